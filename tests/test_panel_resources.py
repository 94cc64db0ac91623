"""Register and scratch budgets of the kernels that carry the products: the panel leaf in all
its shapes, the forms for small products and few rows, the VALU leaf's tables, and the
recursion's expansions and compressions.  Two waves per SIMD (at most 256 registers) and no
per-lane scratch, read from their gfx950 descriptors."""
import pytest

from test_kernel_resources import _descriptors, _pick


@pytest.fixture(scope="module")
def panel():
    return _descriptors("leaf_panel.hip")


# shapes of a panel workgroup (RA, RB, far pitches); two formats and semirings each
@pytest.mark.slow
@pytest.mark.parametrize("shape", ["Li2ELi4ELb0E", "Li4ELi2ELb0E", "Li4ELi2ELb1E", "Li2ELi2ELb0E"])
def test_panel_leaf(panel, shape):
    hits = _pick(panel, "leaf_panel_kernel", shape)
    assert len(hits) == 4
    for name, (vgpr, priv) in hits.items():
        # the 128 x 128 form: three workgroups per CU
        assert vgpr <= (168 if shape.startswith("Li2ELi2E") else 256) and priv == 0, (name, vgpr,
                                                                                      priv)


@pytest.mark.slow
@pytest.mark.parametrize("kernel,count", [("leaf_split_kernel", 8), ("leaf_turn_kernel", 6)])
def test_small_and_few_rows(panel, kernel, count):
    hits = _pick(panel, kernel)
    assert len(hits) == count
    for name, (vgpr, priv) in hits.items():
        assert vgpr <= 256 and priv == 0, (name, vgpr, priv)


@pytest.mark.slow
@pytest.mark.parametrize("source,kernel", [("leaf_valu_table.hip", "leaf_valu_table_kernel"),
                                           ("combine.hip", "expand_kernel"),
                                           ("combine.hip", "compress_kernel"),
                                           ("combine.hip", "compress2_kernel"),
                                           ("transpose.hip", "transpose_kernel")])
def test_no_scratch(source, kernel):
    for name, (vgpr, priv) in _pick(_descriptors(source), kernel).items():
        assert vgpr <= 256 and priv == 0, (name, vgpr, priv)


# 64 x 64 wave tiles by 8- and 16-byte loads, two semirings
@pytest.mark.slow
@pytest.mark.parametrize("format", ["Li0ELi2ELi0ELb1E", "Li1ELi2ELi0ELb0E"])
def test_short_k(format):
    hits = _pick(_descriptors("leaf_mfma.hip"), "leaf_mfma_kernel", format, "ELi2ELi2E")
    assert len(hits) == 4
    for name, (vgpr, priv) in hits.items():
        assert vgpr <= 168 and priv == 0, (name, vgpr, priv)
