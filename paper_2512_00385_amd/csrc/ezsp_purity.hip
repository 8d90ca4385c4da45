// ezsp_purity.hip -- partition purity and oracle mIoU (Sec. 4.2 "Metrics":
// every superpoint takes the majority ground-truth class of its points; the
// mIoU of that labelling bounds what a classifier on the superpoints can
// reach).
//
// Two ways to the count of every (component, class) pair:
//   - a table of component x class counters while it has at most eight
//     entries a point: blocks count their points in an LDS hash and add each
//     distinct pair once, so that a giant superpoint's pair takes one atomic
//     a block.  A wave per component, or a few lanes where there are at most
//     64 classes, then reads its row for the majority, and the per-class
//     counts come from the rows too.  3M points of a driving tile, 8,500
//     superpoints x 541 classes: 219 us sorted, 109 us counted.
//     Atomics on one 128-byte line take about 10 ns each, however many blocks
//     send them: a small table and a short class list are kept in copies.
//   - else a radix sort of the keys component * n_cls + class; each run of
//     equal keys is one pair, found by a binary search from the run head,
//     and a 64-bit atomicMax of (count, ~class) per component picks the
//     majority.
// Ties go to the smallest class.  Per-class TP, ground-truth and predicted
// counts are exact integers, and one thread forms the mean of
// IoU_c = TP / (gt + pred - TP) in class order, so the result is independent
// of scheduling.
#include <algorithm>

#include "ezsp_internal.h"

namespace ezsp {

namespace {

constexpr int kPuNT = 256;
constexpr int kPuLdsCls = 2048;  // class histograms held in LDS up to here
constexpr int kPuHash = 4096;    // LDS hash slots of a counting block
constexpr int kPuShare = 2816;   // points a counting block takes (load 0.69)
constexpr int kPuNarrow = 64;    // classes up to which a lane keeps one class
constexpr int kPuCntCopies = 16;   // of their per-class counts
constexpr int64_t kPuSpread = 1 << 16;  // entries a table's copies fill

// Entries the counter table may have (32-bit keys); eight a point cost as
// much to clear and read as one pass of the sort.
int64_t table_most(int64_t n) {
  const int64_t most = 8 * n > (1 << 20) ? 8 * n : (1 << 20);
  return most < INT32_MAX ? most : INT32_MAX;
}
// Its entries, 0 when the pairs are sorted instead.
int64_t table_entries(int64_t n, int64_t nc, int64_t n_cls) {
  return nc <= table_most(n) / n_cls ? nc * n_cls : 0;
}

// Copies of a small table, so that 1,000 blocks do not add to the same few
// lines (3M points, ten superpoints x 8 classes in random order: 371 us with
// one table, 130 sorted, 68 with copies).  None while there are few
// blocks: folding them is one more launch.
int32_t table_copies(int64_t n, int64_t entries) {
  const int64_t blocks = (n + kPuShare - 1) / kPuShare;
  const int64_t c = std::min(kPuSpread / entries, blocks / 32);
  return (int32_t)std::max<int64_t>(1, std::min<int64_t>(c, 64));
}

__global__ __launch_bounds__(kPuNT) void k_pu_zero(uint4 *__restrict__ table,
                                                   int64_t vecs,
                                                   unsigned long long *cnt,
                                                   int64_t ncnt) {
  const int64_t t = blockIdx.x * (int64_t)kPuNT + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kPuNT;
  for (int64_t i = t; i < vecs; i += step) table[i] = make_uint4(0, 0, 0, 0);
  for (int64_t i = t; i < ncnt; i += step) cnt[i] = 0;
}

__device__ __forceinline__ uint32_t pair_slot(uint32_t x) {
  return (x * 2654435761u) >> 20;  // Knuth's multiplicative hash, 12 bits
}

// Adds c to a pair's count in the block's hash, or in the table when its
// slots are taken.
__device__ __forceinline__ void pair_add(uint32_t key, uint32_t c,
                                         uint32_t *hkey, uint32_t *hcnt,
                                         uint32_t *table) {
  uint32_t e = pair_slot(key);
  for (int probe = 0; probe < 16; ++probe) {
    const uint32_t prev = atomicCAS(&hkey[e], 0xffffffffu, key);
    if (prev == 0xffffffffu || prev == key) {
      atomicAdd(&hcnt[e], c);
      return;
    }
    e = (e + 1) & (kPuHash - 1);
  }
  atomicAdd(&table[key], c);
}

// Counts the pairs of kPuShare points in this block's copy of the table.
__global__ __launch_bounds__(kPuNT) void k_pu_tally(
    const int32_t *__restrict__ label, const int32_t *__restrict__ cls,
    int32_t n, int32_t nc, int32_t n_cls, uint32_t *__restrict__ tables,
    int64_t entries, int32_t copies, Ctl *ctl) {
  uint32_t *table = tables + (int64_t)(blockIdx.x % copies) * entries;
  static_assert(kPuHash == 4096, "pair_slot gives 12 bits");
  __shared__ uint32_t hkey[kPuHash], hcnt[kPuHash];
  for (int i = threadIdx.x; i < kPuHash; i += kPuNT) {
    hkey[i] = 0xffffffffu;
    hcnt[i] = 0;
  }
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kPuShare;
  constexpr int kPer = kPuShare / kPuNT;
  static_assert(kPer * kPuNT == kPuShare, "whole steps");
  uint32_t key[kPer];
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int64_t p = base + j * kPuNT + threadIdx.x;
    key[j] = 0xffffffffu;
    if (p < n) {
      const uint32_t c = (uint32_t)label[p], y = (uint32_t)cls[p];
      if (c < (uint32_t)nc && y < (uint32_t)n_cls)
        key[j] = c * (uint32_t)n_cls + y;
      else
        bad = true;
    }
  }
  if (bad) raise_err(ctl, kErrBadIndex);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    // the pair of the first lane left, twice, in one addition each: a giant
    // superpoint's pair fills much of a wave
    uint64_t left = __ballot(key[j] != 0xffffffffu);
    bool mine = key[j] != 0xffffffffu;
#pragma unroll
    for (int round = 0; round < 2; ++round) {
      if (!left) break;
      const int first = __ffsll((unsigned long long)left) - 1;
      const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key[j], first);
      const uint64_t same = __ballot(mine && key[j] == k);
      if ((int)(threadIdx.x & (kWave - 1)) == first)
        pair_add(k, (uint32_t)__popcll(same), hkey, hcnt, table);
      mine = mine && key[j] != k;
      left &= ~same;
    }
    if (mine) pair_add(key[j], 1u, hkey, hcnt, table);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kPuHash; i += kPuNT)
    if (hcnt[i]) atomicAdd(&table[hkey[i]], hcnt[i]);
}

// The table's copies added into the first.
__global__ __launch_bounds__(kPuNT) void k_pu_fold(
    uint32_t *__restrict__ table, int64_t entries, int32_t copies) {
  const int64_t i = blockIdx.x * (int64_t)kPuNT + threadIdx.x;
  if (i >= entries) return;
  uint32_t s = 0;
#pragma unroll 8
  for (int32_t q = 0; q < copies; ++q) s += table[q * entries + i];
  table[i] = s;
}

// At most kPuNarrow classes: G lanes per component, lane y of them with class
// y of every component they come to, so that the per-class counts are sums in
// registers; two components in flight.  (With a wave per component 3M
// components of 8 classes took 718 us in all, sorted 307, so 190.)
template <int G>
__global__ __launch_bounds__(kPuNT) void k_pu_rows_narrow(
    const uint32_t *__restrict__ table, int32_t nc, int32_t n_cls,
    int32_t *__restrict__ maj, unsigned long long *cnt) {
  static_assert(G <= kPuNarrow && kPuNarrow == kWave, "a class a lane");
  constexpr int U = 2;
  __shared__ uint32_t h[3 * kPuNarrow];
  if (threadIdx.x < 3 * kPuNarrow) h[threadIdx.x] = 0;
  __syncthreads();
  const int32_t y = threadIdx.x & (G - 1);
  uint32_t tp = 0, gt = 0, pr = 0;
  const int64_t step = (int64_t)gridDim.x * (kPuNT / G);
  for (int64_t c0 = (int64_t)blockIdx.x * (kPuNT / G) + threadIdx.x / G;
       c0 < nc; c0 += U * step) {
    uint32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * step;
      x[u] = c < nc && y < n_cls ? table[c * n_cls + y] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t c = c0 + u * step;
      uint64_t best =
          x[u] ? ((uint64_t)x[u] << 32) | (0xffffffffu - (uint32_t)y) : 0u;
      uint32_t size = x[u];
#pragma unroll
      for (int off = G / 2; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor((unsigned long long)best, off, G);
        best = o > best ? o : best;
        size += __shfl_xor(size, off, G);
      }
      const int32_t by = best ? (int32_t)(0xffffffffu - (uint32_t)best) : -1;
      gt += x[u];
      if (y == by) {
        tp += x[u];
        pr += size;
      }
      if (y == 0 && c < nc) maj[c] = by;
    }
  }
  if (y < n_cls) {
    if (tp) atomicAdd(&h[y], tp);
    if (gt) atomicAdd(&h[kPuNarrow + y], gt);
    if (pr) atomicAdd(&h[2 * kPuNarrow + y], pr);
  }
  __syncthreads();
  cnt += (size_t)(blockIdx.x % kPuCntCopies) * 3 * n_cls;
  if (threadIdx.x < 3 * kPuNarrow) {
    const int32_t q = threadIdx.x / kPuNarrow, i = threadIdx.x % kPuNarrow;
    if (h[threadIdx.x])
      atomicAdd(&cnt[q * n_cls + i], (unsigned long long)h[threadIdx.x]);
  }
}

// A wave per component: its row's majority (-1 when empty), and the row's
// share of the per-class counts.
template <bool LDS>
__global__ __launch_bounds__(kPuNT) void k_pu_rows(
    const uint32_t *__restrict__ table, int32_t nc, int32_t n_cls,
    int32_t *__restrict__ maj, unsigned long long *cnt) {
  __shared__ uint32_t h[LDS ? 3 * kPuLdsCls : 1];
  if (LDS) {
    for (int32_t i = threadIdx.x; i < 3 * n_cls; i += kPuNT) h[i] = 0;
    __syncthreads();
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t wave = (int32_t)(blockIdx.x * (kPuNT / kWave) +
                                 threadIdx.x / kWave);
  const int32_t waves = (int32_t)(gridDim.x * (kPuNT / kWave));
  for (int64_t c = wave; c < nc; c += waves) {
    const uint32_t *row = table + c * n_cls;
    uint64_t best = 0;
    uint32_t size = 0;
#pragma unroll 4
    for (int32_t y = lane; y < n_cls; y += kWave) {
      const uint32_t x = row[y];
      if (x) {
        const uint64_t v = ((uint64_t)x << 32) | (0xffffffffu - (uint32_t)y);
        best = v > best ? v : best;
        size += x;
        if (LDS) atomicAdd(&h[n_cls + y], x);
        else atomicAdd(&cnt[n_cls + y], (unsigned long long)x);
      }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      const uint64_t o = __shfl_xor((unsigned long long)best, off, kWave);
      best = o > best ? o : best;
    }
    size = wave_sum(size);
    if (lane != 0) continue;
    const uint32_t y = 0xffffffffu - (uint32_t)best;
    maj[c] = best ? (int32_t)y : -1;
    if (!best) continue;
    if (LDS) {
      atomicAdd(&h[y], (uint32_t)(best >> 32));
      atomicAdd(&h[2 * n_cls + y], size);
    } else {
      atomicAdd(&cnt[y], (unsigned long long)(best >> 32));
      atomicAdd(&cnt[2 * n_cls + y], (unsigned long long)size);
    }
  }
  if (LDS) {
    __syncthreads();
    for (int32_t i = threadIdx.x; i < 3 * n_cls; i += kPuNT)
      if (h[i]) atomicAdd(&cnt[i], (unsigned long long)h[i]);
  }
}

__global__ __launch_bounds__(kPuNT) void k_pu_keys(
    const int32_t *__restrict__ label, const int32_t *__restrict__ cls,
    int32_t n, int32_t nc, int32_t n_cls, uint64_t *keys, Ctl *ctl) {
  const int32_t p = xcd_tid();
  if (p >= n) return;
  const int32_t c = label[p], y = cls[p];
  if ((uint32_t)c >= (uint32_t)nc || (uint32_t)y >= (uint32_t)n_cls) {
    raise_err(ctl, kErrBadIndex);
    keys[p] = 0;
  } else {
    keys[p] = (uint64_t)c * (uint64_t)n_cls + (uint64_t)y;
  }
}

__global__ __launch_bounds__(kPuNT) void k_pu_clear(unsigned long long *best,
                                                    int32_t nc,
                                                    unsigned long long *cnt,
                                                    int64_t ncnt) {
  const int64_t i = blockIdx.x * (int64_t)kPuNT + threadIdx.x;
  if (i < nc) best[i] = 0;
  if (i < ncnt) cnt[i] = 0;
}

// One thread per run head: the run's length by binary search, then the
// component's (count, ~class) maximum.
__global__ __launch_bounds__(kPuNT) void k_pu_runs(const uint64_t *__restrict__ key,
                                                   int32_t n, int32_t n_cls,
                                                   unsigned long long *best) {
  const int32_t i = xcd_tid();
  if (i >= n) return;
  const uint64_t x = key[i];
  if (i > 0 && key[i - 1] == x) return;
  int32_t lo = i + 1, hi = n;  // first index past the run
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo) / 2;
    if (key[mid] == x) lo = mid + 1;
    else hi = mid;
  }
  const uint64_t count = (uint64_t)(lo - i);
  const uint32_t comp = (uint32_t)(x / (uint64_t)n_cls);
  const uint32_t c = (uint32_t)(x % (uint64_t)n_cls);
  atomicMax(&best[comp], (unsigned long long)((count << 32) | (0xffffffffu - c)));
}

__global__ __launch_bounds__(kPuNT) void k_pu_major(
    const unsigned long long *best, int32_t nc, int32_t *maj) {
  const int32_t c = xcd_tid();
  if (c >= nc) return;
  const unsigned long long b = best[c];
  maj[c] = b ? (int32_t)(0xffffffffu - (uint32_t)(b & 0xffffffffu)) : -1;
}

// Per-class counts: cnt[0..n_cls) TP, [n_cls..2n_cls) ground truth,
// [2n_cls..3n_cls) predicted.
template <bool LDS>
__global__ __launch_bounds__(kPuNT) void k_pu_count(
    const int32_t *__restrict__ label, const int32_t *__restrict__ cls,
    int32_t n, int32_t nc, const int32_t *__restrict__ maj, int32_t n_cls,
    unsigned long long *cnt) {
  __shared__ uint32_t h[LDS ? 3 * kPuLdsCls : 1];
  if (LDS) {
    for (int32_t i = threadIdx.x; i < 3 * n_cls; i += kPuNT) h[i] = 0;
    __syncthreads();
  }
  for (int64_t p = blockIdx.x * (int64_t)kPuNT + threadIdx.x; p < n;
       p += (int64_t)gridDim.x * kPuNT) {
    const int32_t c = label[p], g = cls[p];
    // out-of-range ids were reported by k_pu_keys; skip them here
    if ((uint32_t)c >= (uint32_t)nc || (uint32_t)g >= (uint32_t)n_cls) continue;
    const int32_t y = maj[c];
    if (y < 0) continue;
    if (LDS) {
      atomicAdd(&h[n_cls + g], 1u);
      atomicAdd(&h[2 * n_cls + y], 1u);
      if (g == y) atomicAdd(&h[g], 1u);
    } else {
      atomicAdd(&cnt[n_cls + g], 1ull);
      atomicAdd(&cnt[2 * n_cls + y], 1ull);
      if (g == y) atomicAdd(&cnt[g], 1ull);
    }
  }
  if (LDS) {
    __syncthreads();
    for (int32_t i = threadIdx.x; i < 3 * n_cls; i += kPuNT)
      if (h[i]) atomicAdd(&cnt[i], (unsigned long long)h[i]);
  }
}

// IoU per class in parallel, staged in LDS a chunk of classes at a time,
// then the mean in class order by one thread.  Absent classes are staged as
// 0, which leaves the sum as it is, so that its loop is additions alone: the
// loads of eight classes run ahead of their chain (15 -> 6 us at 541 classes).
constexpr int kPuChunk = 4096;

__global__ __launch_bounds__(kPuNT) void k_pu_final(
    const unsigned long long *cnt, int32_t copies, int32_t n_cls, int32_t n,
    double *iou, Ctl *ctl) {
  __shared__ double v[kPuChunk];
  __shared__ unsigned long long tps[kPuNT / kWave];
  __shared__ int32_t prs[kPuNT / kWave];
  double sum = 0.0;
  int32_t present = 0;
  unsigned long long tp_mine = 0;
  for (int32_t base = 0; base < n_cls; base += kPuChunk) {
    const int32_t len = min(kPuChunk, n_cls - base);
    const int32_t padded = (len + 7) & ~7;
    for (int32_t i = threadIdx.x; i < padded; i += kPuNT) {
      double x = 0.0;
      if (i < len) {
        const int32_t c = base + i;
        unsigned long long tp = 0, gt = 0, pr = 0;
#pragma unroll 4
        for (int32_t q = 0; q < copies; ++q) {
          const unsigned long long *part = cnt + (int64_t)q * 3 * n_cls;
          tp += part[c];
          gt += part[n_cls + c];
          pr += part[2 * n_cls + c];
        }
        tp_mine += tp;
        present += gt ? 1 : 0;
        if (gt) x = __ddiv_rn((double)tp, (double)(gt + pr - tp));
        iou[c] = gt ? x : __builtin_nan("");
      }
      v[i] = x;
    }
    __syncthreads();
    if (threadIdx.x == 0)
      for (int32_t i = 0; i < padded; i += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = v[i + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum = __dadd_rn(sum, x[u]);
      }
    __syncthreads();
  }
  tp_mine = wave_sum(tp_mine);
  present = wave_sum(present);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    tps[threadIdx.x / kWave] = tp_mine;
    prs[threadIdx.x / kWave] = present;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long tp_all = 0;
  int64_t present_all = 0;
  for (int w = 0; w < kPuNT / kWave; ++w) {
    tp_all += tps[w];
    present_all += prs[w];
  }
  ctl->pu_miou = __ddiv_rn(sum, (double)present_all);
  ctl->pu_purity = __ddiv_rn((double)tp_all, (double)n);
  ctl->pu_present = present_all;
}

int key_bits(int64_t nkeys) {  // bits of nkeys - 1, at least 1
  int b = 1;
  while (b < 64 && ((uint64_t)1 << b) < (uint64_t)nkeys) ++b;
  return b;
}

}  // namespace

namespace {

// Workspace of one call: the counter table, or the sort's buffers in its
// place.  Room for both, so that the size grows with each argument and a
// workspace for the largest of them serves all smaller ones, whichever way
// those are counted.
struct PurityWork {
  int64_t entries;  // of the table; 0: sorted
  int32_t copies;   // of the table
  int32_t cnt_copies;
  uint32_t *table;
  uint64_t *keys, *keys2;
  int32_t *hist, *bsum, *total;
  unsigned long long *best;
  int32_t *maj;
  unsigned long long *cnt;
  double *iou;
};

PurityWork take_work(Arena &a, int32_t n, int32_t nc, int32_t n_cls) {
  PurityWork w = {};
  w.entries = table_entries(n, nc, n_cls);
  w.copies = w.entries ? table_copies(n, w.entries) : 1;
  w.cnt_copies = w.entries && n_cls <= kPuNarrow ? kPuCntCopies : 1;
  w.table = a.take<uint32_t>(0);
  const size_t start = a.off;
  w.keys = a.take<uint64_t>(n);
  w.keys2 = a.take<uint64_t>(n);
  w.hist = a.take<int32_t>(radix_hist_ints(n));
  w.bsum = a.take<int32_t>(scan_blocks(radix_hist_ints(n)) + 1);
  w.total = a.take<int32_t>(4);
  w.best = a.take<unsigned long long>(nc);
  const int64_t pairs =
      nc <= INT64_MAX / n_cls ? (int64_t)nc * n_cls : INT64_MAX;
  const size_t table =
      4 * (size_t)std::max(std::min(pairs, table_most(n)), kPuSpread) + 16;
  a.off = std::max(a.off, start + table);
  w.maj = a.take<int32_t>(nc);
  w.cnt = a.take<unsigned long long>(
      3 * (size_t)std::max(n_cls, kPuCntCopies * kPuNarrow));
  w.iou = a.take<double>(n_cls);
  return w;
}

}  // namespace

void purity_reserve(Arena &a, int32_t n, int32_t n_comp, int32_t n_cls) {
  take_work(a, n, n_comp, n_cls);
}

int purity_run(const int32_t *labels, int32_t n, int32_t nc,
               const int32_t *cls, int32_t n_cls, int32_t *majority,
               double *iou, PurityResult *res, Ctl *ctl, Arena &a,
               hipStream_t st) {
  const PurityWork w = take_work(a, n, nc, n_cls);
  int32_t *maj = majority ? majority : w.maj;
  double *iou_out = iou ? iou : w.iou;
  Ctl *hc = pinned_ctl();
  if (!hc) {
    set_error("hipHostMalloc of the control block failed");
    return -5;
  }
  const int nt = kPuNT;
  const int64_t gb = ((int64_t)n + nt - 1) / nt;
  const int64_t ncnt = 3 * (int64_t)n_cls * w.cnt_copies;
  prof_begin("purity", st);
  if (w.entries) {
    const int64_t vecs = (w.entries * w.copies + 3) / 4;
    const int64_t zb = ((vecs > ncnt ? vecs : ncnt) + nt - 1) / nt;
    hipLaunchKernelGGL(k_pu_zero, dim3((unsigned)(zb < 2048 ? zb : 2048)),
                       dim3(nt), 0, st, reinterpret_cast<uint4 *>(w.table),
                       vecs, w.cnt, ncnt);
    hipLaunchKernelGGL(k_pu_tally,
                       dim3((unsigned)(((int64_t)n + kPuShare - 1) / kPuShare)),
                       dim3(nt), 0, st, labels, cls, n, nc, n_cls, w.table,
                       w.entries, w.copies, ctl);
    if (w.copies > 1)
      hipLaunchKernelGGL(k_pu_fold,
                         dim3((unsigned)((w.entries + nt - 1) / nt)), dim3(nt),
                         0, st, w.table, w.entries, w.copies);
    if (n_cls <= kPuNarrow) {
      const auto narrow = [&](auto kernel, int g) {
        const int64_t rb = ((int64_t)nc * g + 2 * nt - 1) / (2 * nt);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(rb < 1024 ? rb : 1024)),
                           dim3(nt), 0, st, w.table, nc, n_cls, maj, w.cnt);
      };
      if (n_cls <= 4) narrow(k_pu_rows_narrow<4>, 4);
      else if (n_cls <= 8) narrow(k_pu_rows_narrow<8>, 8);
      else if (n_cls <= 16) narrow(k_pu_rows_narrow<16>, 16);
      else if (n_cls <= 32) narrow(k_pu_rows_narrow<32>, 32);
      else narrow(k_pu_rows_narrow<64>, 64);
    } else {
      const int64_t rb = ((int64_t)nc + nt / kWave - 1) / (nt / kWave);
      const dim3 rg((unsigned)(rb < 1024 ? rb : 1024));
      if (n_cls <= kPuLdsCls)
        hipLaunchKernelGGL(k_pu_rows<true>, rg, dim3(nt), 0, st, w.table, nc,
                           n_cls, maj, w.cnt);
      else
        hipLaunchKernelGGL(k_pu_rows<false>, rg, dim3(nt), 0, st, w.table, nc,
                           n_cls, maj, w.cnt);
    }
  } else {
    hipLaunchKernelGGL(k_pu_keys, dim3(xcd_grid(gb)), dim3(nt), 0, st, labels,
                       cls, n, nc, n_cls, w.keys, ctl);
    const bool alt = radix_sort_keys(w.keys, w.keys2, n, 0,
                                     key_bits((int64_t)nc * n_cls), w.hist,
                                     w.bsum, w.total, ctl, st);
    const uint64_t *sorted = alt ? w.keys2 : w.keys;
    const int64_t cl = (nc > ncnt ? nc : ncnt);
    hipLaunchKernelGGL(k_pu_clear, dim3((unsigned)((cl + nt - 1) / nt)),
                       dim3(nt), 0, st, w.best, nc, w.cnt, ncnt);
    hipLaunchKernelGGL(k_pu_runs, dim3(xcd_grid(gb)), dim3(nt), 0, st, sorted,
                       n, n_cls, w.best);
    hipLaunchKernelGGL(k_pu_major, dim3(xcd_grid(((int64_t)nc + nt - 1) / nt)),
                       dim3(nt), 0, st, w.best, nc, maj);
    const unsigned cg = (unsigned)(gb < 1024 ? gb : 1024);
    if (n_cls <= kPuLdsCls)
      hipLaunchKernelGGL(k_pu_count<true>, dim3(cg), dim3(nt), 0, st, labels,
                         cls, n, nc, maj, n_cls, w.cnt);
    else
      hipLaunchKernelGGL(k_pu_count<false>, dim3(cg), dim3(nt), 0, st, labels,
                         cls, n, nc, maj, n_cls, w.cnt);
  }
  hipLaunchKernelGGL(k_pu_final, dim3(1), dim3(nt), 0, st, w.cnt,
                     w.cnt_copies, n_cls, n, iou_out, ctl);
  prof_end(st);
  prof_bytes("purity", 8.0 * n + 4.0 * nc + 8.0 * n_cls);
  int rc = read_ctl(ctl, hc, st);
  if (rc) return rc;
  if (hc->err & kErrBadIndex) {
    set_error("label outside [0, n_comp) or class outside [0, n_cls)");
    return -1;
  }
  if (hc->err) {
    set_error("internal check failed in the purity (0x%x)", hc->err);
    return -5;
  }
  res->miou = hc->pu_miou;
  res->purity = hc->pu_purity;
  res->n_present = hc->pu_present;
  return 0;
}

}  // namespace ezsp
