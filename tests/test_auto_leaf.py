"""The table's auto_leaf line: the leaf kind of LEAF_AUTO where no entry names one (host
logic only)."""
import pytest


@pytest.fixture
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


@pytest.fixture
def table(bmm, tmp_path):
    p = tmp_path / "t.txt"
    p.write_text("auto_leaf 3\nleaf 0 512 640 768 1 1 1 0 0\n")
    bmm.bmm_finalize()
    bmm.bmm_autotune_load(str(p))
    yield p
    bmm.bmm_finalize()


def test_auto_leaf_names_the_kind_without_an_entry(bmm, table, tmp_path):
    assert bmm.bmm_leaf_choice(bmm.GF2, 4096, 4096, 4096)[0] == bmm.LEAF_MFMA_F4
    assert bmm.bmm_leaf_choice(bmm.BOOLEAN, 1, 1, 1)[0] == bmm.LEAF_MFMA_F4
    # an entry, an explicit leaf, and products past the fp4 counts keep theirs
    assert bmm.bmm_leaf_choice(bmm.GF2, 512, 640, 768) == (bmm.LEAF_VALU, 1)
    for leaf in (bmm.LEAF_VALU, bmm.LEAF_MFMA_I8):
        o = bmm.Options(leaf=leaf)
        assert bmm.bmm_leaf_choice(bmm.GF2, 4096, 4096, 4096, options=o)[0] == leaf
    assert bmm.bmm_leaf_choice(bmm.GF2, 64, (1 << 24) - 1, 64)[0] == bmm.LEAF_MFMA_F4
    assert bmm.bmm_leaf_choice(bmm.GF2, 64, 1 << 24, 64)[0] == bmm.LEAF_MFMA_I8
    saved = tmp_path / "s.txt"
    bmm.bmm_autotune_save(str(saved))
    assert "auto_leaf 3" in saved.read_text().splitlines()
    bmm.bmm_finalize()
    assert bmm.bmm_leaf_choice(bmm.GF2, 4096, 4096, 4096)[0] == bmm.LEAF_MFMA_I8
    bmm.bmm_autotune_load(str(saved))
    assert bmm.bmm_leaf_choice(bmm.GF2, 4096, 4096, 4096)[0] == bmm.LEAF_MFMA_F4


@pytest.mark.parametrize("line", ["auto_leaf 0", "auto_leaf 4", "auto_leaf x"])
def test_bad_auto_leaf_lines_are_refused(bmm, tmp_path, line):
    p = tmp_path / "t.txt"
    p.write_text(line + "\n")
    with pytest.raises(bmm.BmmError):
        bmm.bmm_autotune_load(str(p))


def test_default_depth_follows_the_leaf(bmm, table):
    """Without a depth entry: leaves of 2048 bits and more with the int8 leaf, of a harmonic
    size of 1250 and more with the fp4 leaf, of which at most two levels breadth first."""
    n = 1 << 16
    _, ds, dp = bmm.bmm_gf2_strassen_workspace(n, n, n, -1)
    assert (ds, dp) == (2, 2)
    _, ds, dp = bmm.bmm_gf2_strassen_workspace(n, n, n, -1, bmm.Options(leaf=bmm.LEAF_MFMA_I8))
    assert (ds, dp) == (1, 4)
    _, ds, dp = bmm.bmm_gf2_strassen_workspace(2048, 2048, 2048, -1)
    assert (ds, dp) == (0, 0)
