// Persistent batched leaf: many independent products of uneven sizes in one
// launch.  A work item is a 2 x 2 group of wave tiles of one problem (128 x 64,
// 64 x 64 or 64 x 128 per wave; int8 or E2M1 operands, as the plan chose), so
// the four waves of a workgroup read shared operand rows together.  Items sit
// in kXcds queues, one per XCD: every problem's items, in banded order, are
// split into contiguous ranges over the queues, so the workgroups of one XCD
// walk neighbouring items and share that XCD's L2.  A workgroup takes items
// from the queue of its own XCD (the hardware hands workgroup g to XCD g % 8)
// and, once that queue is empty, from the next that is not; it exits when all
// are empty.  Which XCD runs an item never affects the result.
//
// Wave 0 of a workgroup takes items: lane 0 takes a queue position with one atomic add,
// issued a whole item ahead, and the item's record and problem are read from tables while
// the item before is computed.  The last workgroup to leave sets the queue counters
// back, so a launch is one kernel and can be captured into a HIP graph and replayed.
// Together these took 256 problems of 256 to 1024 from 58 to 50 us, 300 of 256 to 2048 from
// 136 to 122 us, and one of 256 from 18.6 to 12.8 us.  With k in the thousands the matrix
// cores bound an item.
#include <stddef.h>

#include "panel_tile.h"

namespace bmm {
namespace {

// Index of the last segment of a queue whose first position is <= t (every
// queue's first segment starts at 0 and t is below the queue's item count).
__device__ __forceinline__ uint32_t find_segment(const BatchedSeg* __restrict__ segs,
                                                 uint32_t count, uint32_t t) {
  uint32_t lo = 0, hi = count;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (segs[mid].begin <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

constexpr uint32_t kNoItem = ~0u;

// Wave 0's place in the queues: the queue it takes from, and those it knows to be empty.
struct Place {
  int q;
  uint32_t empty;
};

// Lane 0 takes a position of the place's queue; the answer may be on its way (an address
// that is known to be the same in all lanes would have the compiler broadcast it at once).
__device__ __forceinline__ unsigned take(unsigned int* __restrict__ counters, const Place& at,
                                         int lane) {
  int zero = lane;
  asm volatile("" : "+v"(zero));
  unsigned v = 0;
  if (lane == 0) v = atomicAdd(&counters[at.q * kBatchedCounterStride + zero], 1u);
  return v;
}

// The list index of the position t taken at `at`; where the queue was empty, of one of the
// next that is not.  False once every queue is empty (and from then on).  All counters
// are looked at together: trying one queue after the other took a workgroup 5 us at the end.
__device__ __forceinline__ bool settle(const uint32_t* items, const uint64_t* first,
                                       unsigned int* __restrict__ counters, unsigned t, Place& at,
                                       int lane, uint64_t& index) {
  constexpr uint32_t kAll = (1u << kXcds) - 1;
  if (at.empty == kAll) return false;
  while (t >= (unsigned)__builtin_amdgcn_readfirstlane(items[at.q])) {
    at.empty |= 1u << at.q;  // (no counter goes back while a workgroup takes: at most kXcds turns)
    bool none = true;
    if (lane < kXcds)
      none = __hip_atomic_load(&counters[lane * kBatchedCounterStride], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT) >= items[lane];
    at.empty |= (uint32_t)__ballot(none) & kAll;
    if (at.empty == kAll) return false;
    const uint32_t open = ~at.empty & kAll;
    const int from = at.q + 1;  // 1 .. kXcds
    at.q = (from + __builtin_ctz((open | open << kXcds) >> from)) % kXcds;
    t = __builtin_amdgcn_readfirstlane(take(counters, at, lane));
  }
  index = first[at.q] + t;
  return true;
}

// Wave 0 of a workgroup that found every queue empty (its takes have all been answered): the
// last one of the grid sets the counters back for the next launch, as the plan set them up.
__device__ __forceinline__ void leave(unsigned int* __restrict__ counters, int lane) {
  unsigned left = 0;
  if (lane == 0) left = atomicAdd(&counters[kXcds * kBatchedCounterStride], 1u);
  if ((unsigned)__builtin_amdgcn_readfirstlane(left) != gridDim.x - 1) return;
  if (lane <= kXcds)
    __hip_atomic_store(&counters[lane * kBatchedCounterStride],
                       lane < kXcds ? batched_first_take(gridDim.x, lane) : 0u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// Row and column of a problem's item (32-bit divisions where the band fits).
__device__ __forceinline__ void item_coord(const BatchedDesc& d, uint32_t item, int64_t& im,
                                           int64_t& in) {
  if ((uint32_t)d.items_n < (1u << 28))
    band_coord<uint32_t>(item, (uint32_t)d.items_m, (uint32_t)d.items_n, im, in);
  else
    band_coord<int64_t>((int64_t)item, d.items_m, d.items_n, im, in);
}

// The register-fed items keep the 32-bit operand expansion: the persistent loop's own
// state leaves no room for the wide form's registers.
constexpr bool kWide = false;

template <int RA, int RB, int FMT>
__device__ __forceinline__ void run_item(const BatchedDesc& d, int64_t im, int64_t in, int w) {
  const int64_t tm = 2 * im + (w >> 1), tn = 2 * in + (w & 1);
  if (tm >= d.tiles_m || tn >= d.tiles_n) return;  // uniform per wave
  // (the tile reads and writes through global-memory pointers: the table's
  // pointers are device memory)
  const uint64_t* A = d.A;
  const uint64_t* BT = d.BT;
  uint64_t* C = d.C;
  // (the chunked long-k loop of the one-shot leaf measured no faster here: most
  // items are short, and its code doubles the kernel)
  if (d.aligned) {
    mfma::tile<mfma::SEMI_ANY, RA, RB, 2, FMT, 2, 0, kWide>(A, d.lda, BT, d.ldbt, C, d.ldc, d.m,
                                                          d.k, d.n, tm, tn, 0, d.semiring);
  } else {
    mfma::tile<mfma::SEMI_ANY, RA, RB, 1, FMT, 2, 0, kWide>(A, d.lda, BT, d.ldbt, C, d.ldc, d.m,
                                                          d.k, d.n, tm, tn, 0, d.semiring);
  }
}

// One thread per item of a queue.
__global__ void list_kernel(const BatchedDesc* __restrict__ descs,
                            const BatchedSeg* __restrict__ segs, BatchedQueues qs,
                            BatchedItem* __restrict__ list) {
  const int q = blockIdx.y;
  const BatchedSeg* qsegs = segs + qs.seg_off[q];
  for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < qs.items[q];
       t += gridDim.x * blockDim.x) {
    const uint32_t s = find_segment(qsegs, qs.seg_count[q], t);
    const uint32_t p = qsegs[s].problem;
    int64_t im, in;
    item_coord(descs[p], qsegs[s].item_lo + (t - qsegs[s].begin), im, in);
    list[qs.first[q] + t] = BatchedItem{p, (uint32_t)im, (uint32_t)in, 0u};
  }
}

// LDS-staged items (tile 4): the workgroup tile of panel_tile.h, 2 x 2 waves of 128 x 64 (the
// wide shape would spill in the persistent loop).  Everything an item needs is known
// before it starts: while item i is computed, wave 0 has on their way the descriptor of
// item i + 1's problem, the record of item i + 2 and the position of item i + 3, each asked
// for when what it depends on has come with the operands of some first stage, so
// nothing waits for them.  The first stage of the next item is loaded while the results of this one are
// packed and stored (256 problems of 256 to 8192: 963 us, without it 1019; 256 of 256 to 1024:
// 46.6 and 50.0 us).
// All of it goes to LDS directly.
struct alignas(16) Ahead {
  uint32_t desc[2][32];    // of the items at hand and next (0..23: a BatchedDesc)
  uint32_t record[4][4];   // of the items at hand, next and after that
  uint64_t first[kXcds];   // of the queues
  uint32_t items[kXcds];
};
static_assert(sizeof(BatchedDesc) == 96 && sizeof(BatchedItem) == 16, "moved 16 bytes a lane");

struct LookAhead {
  const BatchedDesc* __restrict__ descs;
  const BatchedItem* __restrict__ list;
  unsigned int* __restrict__ counters;
  Ahead* lds;
  int w, lane, it;  // it: the item at hand
  Place at;
  unsigned v;       // the position taken last

  static __device__ __forceinline__ uint32_t address(const void* p) {
    typedef __attribute__((address_space(3))) const unsigned char* lds_ptr;
    return (uint32_t)(uintptr_t)(lds_ptr)p;
  }
  // Ask for the record of item i, and the position after it.
  __device__ __forceinline__ void record(int i) {
    uint64_t index;
    const unsigned t = __builtin_amdgcn_readfirstlane(v);
    v = 0;
    if (settle(lds->items, lds->first, counters, t, at, lane, index)) {
      if (lane == 0) load_lds16(list + index, address(lds->record[i & 3]));
      v = take(counters, at, lane);
    } else if (lane == 0) {
      lds->record[i & 3][0] = kNoItem;
    }
  }
  // Ask for the descriptor of item i's problem.
  __device__ __forceinline__ void descriptor(int i) {
    const uint32_t p = __builtin_amdgcn_readfirstlane(lds->record[i & 3][0]);
    if (p != kNoItem && lane < 6)
      load_lds16(reinterpret_cast<const char*>(descs + p) + 16 * lane, address(lds->desc[i & 1]));
  }
  static __device__ __forceinline__ void arrive() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  }
  __device__ __forceinline__ void operator()() {
    if (w != 0) return;
    record(it + 2);
    descriptor(it + 1);
  }
};

// What of an item is needed after its sums.
struct Result {
  uint64_t* C;
  int64_t ldc, m, n, row0, col0;
  int semiring;
};

template <int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void batched_lds_kernel(
    const BatchedDesc* __restrict__ descs, const BatchedItem* __restrict__ list,
    BatchedQueues qs, unsigned int* __restrict__ counters) {
  __shared__ Ahead lds;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[panel::lds_bytes(4, 2)];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  LookAhead ahead{descs, list, counters, &lds, w, lane, 0, Place{(int)(blockIdx.x % kXcds), 0u},
                  blockIdx.x / kXcds};
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < kXcds; ++q) {
      lds.first[q] = qs.first[q];
      lds.items[q] = qs.items[q];
    }
    ahead.record(0);
    LookAhead::arrive();
    ahead.descriptor(0);
    ahead.record(1);
    LookAhead::arrive();
  }
  __syncthreads();
  using Op = panel::Operands<4, 2, false>;
  // the operands of the item at hand, their first stage on its way
  auto begin = [&](Result& r) {
    const uint32_t* rec = lds.record[ahead.it & 3];
    const uint32_t mine = lds.desc[ahead.it & 1][lane & 31];
    auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)mine, i); };
    auto quad = [&](int i) { return (uint64_t)word(i) | ((uint64_t)word(i + 1) << 32); };
    constexpr int M = offsetof(BatchedDesc, m) / 4, LD = offsetof(BatchedDesc, lda) / 4;
    const uint32_t im = __builtin_amdgcn_readfirstlane(rec[1]);
    const uint32_t in = __builtin_amdgcn_readfirstlane(rec[2]);
    r = Result{(uint64_t*)quad(4), (int64_t)quad(LD + 4), (int64_t)quad(M), (int64_t)quad(M + 4),
               (int64_t)im * Op::TM + (w >> 1) * 128, (int64_t)in * (Op::TN / 64) + (w & 1),
               (int)word(offsetof(BatchedDesc, semiring) / 4)};
    Op op((const uint64_t*)quad(0), (int64_t)quad(LD), (const uint64_t*)quad(2),
          (int64_t)quad(LD + 2), r.m, (int64_t)quad(M + 2), r.n, im, in, w, smem);
    op.load(0, 0);
    return op;
  };
  auto none = [&]() {  // the same for every wave
    return __builtin_amdgcn_readfirstlane(lds.record[ahead.it & 3][0]) == kNoItem;
  };
  if (!none()) {
    Result now, next;
    Op op = begin(next);
    bool more = true;
    while (more) {
      now = next;
      panel::AccV<FMT> acc[4][2];
      panel::sums<mfma::SEMI_ANY, FMT, 4, 2, false>(op, 0, acc, ahead);
      // all waves are done with the operands, and the next item is in LDS
      if (w == 0) LookAhead::arrive();
      __syncthreads();
      ++ahead.it;
      more = !none();
      if (more) op = begin(next);
      panel::store_tile<mfma::SEMI_ANY, FMT, 4, 2>(acc, now.C, now.ldc, now.m, now.n, now.row0,
                                                   now.col0, 0, now.semiring);
    }
  }
  if (w == 0) leave(counters, lane);
}

template <int RA, int RB, int FMT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void batched_kernel(
    const BatchedDesc* __restrict__ descs, const BatchedItem* __restrict__ list,
    BatchedQueues qs, unsigned int* __restrict__ counters) {
  // two (problem, im, in) slots: wave 0 fills one while the others read the other
  __shared__ uint32_t slots[2][3];
  __shared__ uint64_t first[kXcds];
  __shared__ uint32_t items[kXcds];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  Place at{(int)(blockIdx.x % kXcds), 0u};
  auto hand = [&](unsigned v, int slot) {
    uint64_t index;
    const bool more =
        settle(items, first, counters, __builtin_amdgcn_readfirstlane(v), at, lane, index);
    if (lane != 0) return;
    slots[slot][0] = kNoItem;
    if (more) {
      const BatchedItem rec = list[index];
      slots[slot][0] = rec.problem;
      slots[slot][1] = rec.im;
      slots[slot][2] = rec.in;
    }
  };
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < kXcds; ++q) {
      first[q] = qs.first[q];
      items[q] = qs.items[q];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  if (w == 0) hand(blockIdx.x / kXcds, 0);  // (the counters start behind the grid's first items)
  __syncthreads();
  for (int it = 0;; ++it) {
    const uint32_t* cur = slots[it & 1];
    const uint32_t p = __builtin_amdgcn_readfirstlane(cur[0]);
    if (p == kNoItem) break;  // the same for every wave of the workgroup
    const uint32_t im = __builtin_amdgcn_readfirstlane(cur[1]);
    const uint32_t in = __builtin_amdgcn_readfirstlane(cur[2]);
    unsigned v = 0;
    if (w == 0) v = take(counters, at, lane);
    run_item<RA, RB, FMT>(descs[p], im, in, w);
    if (w == 0) hand(v, (it + 1) & 1);
    __syncthreads();
  }
  if (w == 0) leave(counters, lane);
}

template <int RA, int RB, int FMT>
void launch_k(const BatchedDesc* descs, const BatchedItem* list, const BatchedQueues& qs,
              unsigned int* counters, int grid, hipStream_t s) {
  hipLaunchKernelGGL((batched_kernel<RA, RB, FMT>), dim3((unsigned)grid), dim3(256), 0, s, descs,
                     list, qs, counters);
}

template <int FMT>
void launch_fmt(const BatchedDesc* descs, const BatchedItem* list, const BatchedQueues& qs,
                unsigned int* counters, int grid, int tile, hipStream_t s) {
  if (tile == 4)
    hipLaunchKernelGGL((batched_lds_kernel<FMT>), dim3((unsigned)grid), dim3(256), 0, s, descs,
                       list, qs, counters);
  else if (tile == 1) launch_k<4, 2, FMT>(descs, list, qs, counters, grid, s);
  else if (tile == 3) launch_k<2, 4, FMT>(descs, list, qs, counters, grid, s);
  else launch_k<2, 2, FMT>(descs, list, qs, counters, grid, s);
}

}  // namespace

int batched_tile_rows(int tile) { return tile == 1 || tile == 4 ? 128 : 64; }
int batched_tile_cols(int tile) { return tile == 3 ? 128 : 64; }

hipError_t launch_batched_persistent(const BatchedDesc* descs, const BatchedItem* list,
                                     const BatchedQueues& queues, unsigned int* counters,
                                     int grid, int tile, int fmt, hipStream_t s) {
  uint64_t items = 0;
  for (int x = 0; x < kXcds; ++x) items += queues.items[x];
  if (items == 0 || grid <= 0) return hipSuccess;
  if (fmt == mfma::FMT_F4)
    launch_fmt<mfma::FMT_F4>(descs, list, queues, counters, grid, tile, s);
  else
    launch_fmt<mfma::FMT_I8>(descs, list, queues, counters, grid, tile, s);
  return hipGetLastError();
}

hipError_t launch_batched_list(const BatchedDesc* descs, const BatchedSeg* segs,
                               const BatchedQueues& queues, BatchedItem* list, hipStream_t s) {
  uint32_t most = 0;
  for (int q = 0; q < kXcds; ++q) most = most < queues.items[q] ? queues.items[q] : most;
  if (most == 0) return hipSuccess;
  const uint32_t blocks = most / 256 < 1024 ? most / 256 + 1 : 1024;
  hipLaunchKernelGGL(list_kernel, dim3(blocks, kXcds), dim3(256), 0, s, descs, segs, queues, list);
  return hipGetLastError();
}

}  // namespace bmm
