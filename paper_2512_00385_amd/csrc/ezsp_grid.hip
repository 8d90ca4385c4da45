// ezsp_grid.hip -- regular-grid subsampling of a point cloud (Sec. 4.1: every
// cloud is subsampled on a regular grid before it is partitioned).
//
// A point's cell is floor((x_i - o_i) / h) per axis in IEEE fp32 (one
// subtraction, one correctly rounded division, floor), o the coordinate-wise
// minimum of the cloud; the cell keeps its smallest point index, and the kept
// indices come out in increasing order.
//
// Cells go into an open-addressing hash table at load <= 1/2.  An entry is one
// 64-bit word, the cell above the point index, whenever the cloud's cells and
// indices fit 63 bits (3M points: 41 bits of cells): a cell is claimed by a
// 64-bit CAS and lowered to its first index by a 64-bit atomicMin.  Larger
// grids take 16-byte entries (key, first index).  A point loads its entry
// before it tries an atomic and needs none when the cell already holds a
// smaller index: a stale value only costs an atomic that changes nothing,
// since an entry's cell never changes and its index only falls.  One pass
// over the table then flags the kept points, and a scan over the flags writes
// them in point order.  The result does not depend on the order of the
// atomics.  3M points of a driving tile at 10 cm: 0.45 ms with an
// unconditional CAS and atomicMin a point and two random passes over the
// table, 0.16 ms so.
#include "ezsp_internal.h"

namespace ezsp {

namespace {

constexpr uint64_t kCellEmpty = ~0ull;
constexpr float kCellLimit = 2097152.0f;  // 2^21 cells per axis

struct alignas(16) CellEntry {
  unsigned long long key;
  uint32_t first;
  uint32_t pad;
};

// splitmix64 finaliser (Steele, Lea and Flood, 2014)
__device__ __forceinline__ uint64_t cell_hash(uint64_t x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

// Cell of offset v - o; above kCellLimit (or NaN) is out of range.
__device__ __forceinline__ float cell_of(float v, float o, float h) {
  return floorf(__fdiv_rn(__fsub_rn(v, o), h));
}

// Bits of the cell index on each axis, from the bounding box (the largest
// coordinate has the largest cell: each step is monotone), and whether a cell
// and a point index fit one word beside the empty mark.
struct CellBits {
  int b[3];
  bool packed;
};

__device__ __forceinline__ CellBits cell_bits(const int32_t *box, float h,
                                              int index_bits) {
  CellBits c;
  int sum = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float f =
        cell_of(ord2f(box[3 + a]), ord2f(box[a]), h);
    c.b[a] = f >= 0.0f && f < kCellLimit ? 32 - __clz((int)f) : 21;
    sum += c.b[a];
  }
  c.packed = sum + index_bits <= 63;
  return c;
}

// Folds the bounding box, empties the table (8 or 16 bytes an entry) and
// clears the flags.
__global__ __launch_bounds__(256) void k_grid_clear(
    Ctl *ctl, float h, int index_bits, CellEntry *t, int64_t cap,
    uint32_t *__restrict__ flag, int64_t flag_words) {
  __shared__ int32_t box[6];
  fold_box(ctl, box);
  if (blockIdx.x == 0 && threadIdx.x < 6)
    ctl->bbox_enc[threadIdx.x] = box[threadIdx.x];
  const bool packed = cell_bits(box, h, index_bits).packed;
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  uint4 *t4 = reinterpret_cast<uint4 *>(t);
  const int64_t vecs = packed ? cap / 2 : cap;
  const uint32_t last = packed ? 0xffffffffu : 0u;
  for (int64_t i = i0; i < vecs; i += step)
    t4[i] = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, last);
  for (int64_t i = i0; i < flag_words; i += step) flag[i] = 0;
}

template <class T>
__device__ __forceinline__ T peek(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A thread a point, in index order, so that most cells are claimed by their
// first index.  Bound by the table's random lines (3M points 292 -> 80 us).
// look: load the entry before trying the atomics.  It pays where several
// points share a cell; below 2^16 points a load ahead of a CAS that mostly
// follows is one more latency on the path (20,000 points: 10 against 8 us).
__global__ __launch_bounds__(256) void k_grid_insert(
    const float *__restrict__ xyz, int32_t n, float h, bool look,
    int index_bits, CellEntry *t, uint64_t mask, Ctl *ctl) {
  const int32_t p = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (p >= n) return;
  const CellBits bits = cell_bits(ctl->bbox_enc, h, index_bits);
  uint64_t key = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float f =
        cell_of(xyz[3 * (int64_t)p + a], ord2f(ctl->bbox_enc[a]), h);
    if (!(f >= 0.0f && f < kCellLimit)) {  // also NaN from a bad coordinate
      raise_err(ctl, kErrRange);
      return;
    }
    key = (key << bits.b[a]) | (uint64_t)f;
  }
  uint64_t e = cell_hash(key) & mask;
  if (bits.packed) {
    unsigned long long *w = reinterpret_cast<unsigned long long *>(t);
    const unsigned long long v =
        (unsigned long long)((key << index_bits) | (uint64_t)p);
    for (uint64_t probe = 0; probe <= mask; ++probe) {
      unsigned long long cur = look ? peek(&w[e]) : kCellEmpty;
      if (cur == kCellEmpty) {
        cur = atomicCAS(&w[e], (unsigned long long)kCellEmpty, v);
        if (cur == kCellEmpty) return;
      }
      if ((cur >> index_bits) == key) {
        if (v < cur) atomicMin(&w[e], v);
        return;
      }
      e = (e + 1) & mask;
    }
  } else {
    for (uint64_t probe = 0; probe <= mask; ++probe) {
      unsigned long long cur = look ? peek(&t[e].key) : kCellEmpty;
      if (cur == kCellEmpty)
        cur = atomicCAS(&t[e].key, (unsigned long long)kCellEmpty,
                        (unsigned long long)key);
      if (cur == kCellEmpty || cur == key) {
        if ((uint32_t)p < peek(&t[e].first))
          atomicMin(&t[e].first, (uint32_t)p);
        return;
      }
      e = (e + 1) & mask;
    }
  }
  raise_err(ctl, kErrInternal);  // unreachable at load <= 1/2
}

// Flags every entry's point.
__global__ __launch_bounds__(256) void k_grid_mark(
    const Ctl *ctl, float h, int index_bits, const CellEntry *__restrict__ t,
    int64_t cap, uint8_t *__restrict__ flag, int32_t n) {
  const bool packed = cell_bits(ctl->bbox_enc, h, index_bits).packed;
  const ulonglong2 *t2 = reinterpret_cast<const ulonglong2 *>(t);
  const int64_t vecs = packed ? cap / 2 : cap;
  const uint64_t low = ((uint64_t)1 << index_bits) - 1;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < vecs;
       i += (int64_t)gridDim.x * blockDim.x) {
    const ulonglong2 x = t2[i];
    if (x.x != kCellEmpty) {
      const uint64_t p = packed ? x.x & low : x.y & 0xffffffffu;
      if (p < (uint64_t)n) flag[p] = 1;
    }
    if (packed && x.y != kCellEmpty && (x.y & low) < (uint64_t)n)
      flag[x.y & low] = 1;
  }
}

// Scan functor: the flagged points, in order.
struct ScanKeep {
  const uint8_t *flag;
  int32_t *keep;
  __device__ int32_t value(int32_t i) const { return flag[i]; }
  __device__ void emit(int32_t i, int32_t excl, int32_t v) const {
    if (v) keep[excl] = i;
  }
};

int bits_of(int64_t n) {  // bits of n - 1, at least 1
  int b = 1;
  while (b < 31 && ((int64_t)1 << b) < n) ++b;
  return b;
}

uint64_t table_cap(int64_t n) {
  uint64_t cap = 64;
  while (cap < 2 * (uint64_t)n) cap <<= 1;
  return cap;
}

}  // namespace

void grid_reserve(Arena &a, int32_t n) {
  a.take<CellEntry>(table_cap(n));
  a.take<uint32_t>(((size_t)n + 3) / 4);
  a.take<int32_t>(scan_blocks(n) + 1);
}

int grid_run(const float *xyz, int32_t n, float h, int32_t *keep,
             int64_t *n_keep, Ctl *ctl, Arena &a, hipStream_t st) {
  const uint64_t cap = table_cap(n);
  CellEntry *t = a.take<CellEntry>(cap);
  const size_t words = ((size_t)n + 3) / 4;
  uint32_t *flag = a.take<uint32_t>(words);
  const int ib = bits_of(n);
  int32_t *bsum = a.take<int32_t>(scan_blocks(n) + 1);
  Ctl *hc = pinned_ctl();
  if (!hc) {
    set_error("hipHostMalloc of the control block failed");
    return -5;
  }
  const int nt = 256;
  const int64_t gb = (n + nt - 1) / nt;
  prof_begin("grid_subsample", st);
  hipLaunchKernelGGL(k_bbox, dim3((unsigned)(gb < 256 ? gb : 256)), dim3(nt),
                     0, st, xyz, n, ctl);
  const int64_t cb = (int64_t)((cap + nt - 1) / nt);
  const dim3 tg((unsigned)(cb < 4096 ? cb : 4096));
  uint8_t *flag8 = reinterpret_cast<uint8_t *>(flag);
  hipLaunchKernelGGL(k_grid_clear, tg, dim3(nt), 0, st, ctl, h, ib, t,
                     (int64_t)cap, flag, (int64_t)words);
  hipLaunchKernelGGL(k_grid_insert, dim3((unsigned)gb), dim3(nt), 0, st, xyz,
                     n, h, n >= (1 << 16), ib, t, cap - 1, ctl);
  hipLaunchKernelGGL(k_grid_mark, tg, dim3(nt), 0, st, ctl, h, ib, t,
                     (int64_t)cap, flag8, n);
  device_scan(ScanKeep{flag8, keep}, n, bsum, &ctl->n_out, st);
  prof_end(st);
  int rc = read_ctl(ctl, hc, st);
  if (rc) return rc;
  // algorithmic bytes: read xyz, write the kept indices
  prof_bytes("grid_subsample", 12.0 * n + 4.0 * hc->n_out);
  if (hc->err & kErrNonFinite) {
    set_error("non-finite coordinate in xyz");
    return -2;
  }
  if (hc->err & kErrRange) {
    set_error("the cloud spans 2^21 or more cells of size h on some axis");
    return -3;
  }
  if (hc->err) {
    set_error("internal check failed in the grid subsampling (0x%x)",
              hc->err);
    return -5;
  }
  *n_keep = hc->n_out;
  return 0;
}

}  // namespace ezsp
