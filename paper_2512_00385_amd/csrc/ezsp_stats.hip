// ezsp_stats.hip -- per-superpoint size, mean embedding and centroid of a
// labelling (Sec. 3.2: the mean embedding Y_P of a superpoint; App. Alg. A-2,
// component_attributes).  Sums are exact int64 fixed point, so the result
// does not depend on the order in which points are added.
//
// Points are sorted by label (radix sort of packed (label, index) keys) and
// the sorted rows summed in segments.  An atomic per point and dimension
// instead serialises at the memory side on the largest superpoint: 3M points
// of a driving tile, D = 32 with positions, took 242 ms that way (half of
// the points are one ground superpoint) and take 0.43 ms in segments.
#include "ezsp_internal.h"

namespace ezsp {

namespace {

constexpr int kCsNT = 256;
constexpr int kCsU = 4;  // rows in flight per group of lanes

// Raises *dst to the block's maximum; after the first few blocks the value
// is mostly there and a load takes the place of the atomic.
__device__ __forceinline__ void block_max_to(uint32_t m, uint32_t *sm,
                                             uint32_t *dst) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1)
    m = max(m, (uint32_t)__shfl_xor((int)m, off, kWave));
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) sm[threadIdx.x / kWave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kCsNT / kWave; ++w) m = max(m, sm[w]);
    if (m > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(dst, m);
  }
}

// Largest |v| bit pattern this thread sees of v[0, count); patterns from
// 0x7f800000 up are infinities and NaNs.
__device__ __forceinline__ uint32_t max_bits(const float *__restrict__ v,
                                             int64_t count, int64_t t,
                                             int64_t step) {
  uint32_t m = 0;
  int64_t head = 0;
  if ((reinterpret_cast<uintptr_t>(v) & 15) == 0) {
    const uint4 *v4 = reinterpret_cast<const uint4 *>(v);
    const int64_t c4 = count / 4;
    for (int64_t i = t; i < c4; i += 4 * step) {
      uint4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t j = i + u * step;
        x[u] = j < c4 ? v4[j] : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        m = max(max(max(m, x[u].x & 0x7fffffffu), x[u].y & 0x7fffffffu),
                max(x[u].z & 0x7fffffffu, x[u].w & 0x7fffffffu));
    }
    head = 4 * c4;
  }
  for (int64_t i = head + t; i < count; i += step)
    m = max(m, __float_as_uint(v[i]) & 0x7fffffffu);
  return m;
}

// One pass over the inputs: largest |emb| and |xyz|, the sort keys (label in
// the high half, point in the low half), and the sums cleared.
__global__ __launch_bounds__(kCsNT) void k_cs_prep(
    const int32_t *__restrict__ labels, int32_t n, int32_t nc,
    const float *__restrict__ emb, int32_t d, const float *__restrict__ xyz,
    uint64_t *__restrict__ keys, int64_t *size, int64_t *Se, int64_t *Sx,
    Ctl *ctl) {
  __shared__ uint32_t sm[kCsNT / kWave];
  const int64_t t = blockIdx.x * (int64_t)kCsNT + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kCsNT;
  bool bad = false;
  for (int64_t p = t; p < n; p += step) {
    uint32_t c = (uint32_t)labels[p];
    if (c >= (uint32_t)nc) {
      bad = true;
      c = 0;
    }
    keys[p] = ((uint64_t)c << 32) | (uint64_t)p;
  }
  for (int64_t i = t; i < nc; i += step) size[i] = 0;
  for (int64_t i = t; i < (int64_t)nc * d; i += step) Se[i] = 0;
  if (xyz)
    for (int64_t i = t; i < (int64_t)nc * 3; i += step) Sx[i] = 0;
  const uint32_t me = max_bits(emb, (int64_t)n * d, t, step);
  const uint32_t mx = xyz ? max_bits(xyz, (int64_t)n * 3, t, step) : 0u;
  if (max(me, mx) >= 0x7f800000u) raise_err(ctl, kErrNonFinite);
  if (bad) raise_err(ctl, kErrBadIndex);
  block_max_to(me, sm, &ctl->maxabs_bits);
  if (xyz) block_max_to(mx, sm, &ctl->maxabs_x_bits);
}

// Adding 1.5 * 2^52 leaves rint(x) in the low bits of the sum for
// |x| <= 2^51, so the bit patterns add up to the integer sum plus a known
// multiple of the constant: two operations an element instead of the dozen
// of an fp64 to int64 conversion.  |e| * 2^F <= 2^(61 - ceil(log2 n)) by
// the shift rule, so this holds for n > 512; smaller inputs convert.
constexpr double kMagic = 6755399441055744.0;

template <bool MAGIC>
__device__ __forceinline__ uint64_t fixed_bits(float e, double s) {
  if (MAGIC)
    return (uint64_t)__double_as_longlong(__fma_rn((double)e, s, kMagic));
  return (uint64_t)(int64_t)rint((double)e * s);
}

// Segmented sums over the label-sorted points.  A group of G lanes takes E
// consecutive entries, lane i holding dimensions V i .. V i + V - 1 (and
// lanes 0-2 a coordinate each).  A run of equal labels that begins and ends
// inside the group is a whole superpoint and is stored; the group's first
// and last runs go through LDS, where the block joins those of neighbouring
// groups before it adds them with one atomic per value.  The rows of a
// random-order cloud are fetched one by one, which bounds it: at 3M points,
// D = 32 with positions 225 us for 0.45 GB (eight rows in flight a group
// instead of four: 227 us).
template <int G, int V, bool MAGIC>
__global__ __launch_bounds__(kCsNT) void k_cs_segments(
    const uint64_t *__restrict__ keys, int32_t n, int32_t E,
    const float *__restrict__ emb, int32_t d, const float *__restrict__ xyz,
    const Ctl *ctl, int64_t *__restrict__ size, int64_t *__restrict__ Se,
    int64_t *__restrict__ Sx) {
  constexpr int R = kCsNT / G;      // groups a block
  constexpr int W = G * V + 4;      // sums of a run: dims, xyz, count
  __shared__ int32_t run_lab[2 * R];
  __shared__ int64_t run_sum[2 * R][W];
  const int lane = threadIdx.x & (G - 1);
  const int g = threadIdx.x / G;
  const double sF =
      ldexp(1.0, fixshift_rule(__uint_as_float(ctl->maxabs_bits), n));
  const double sX =
      xyz ? ldexp(1.0, fixshift_rule(__uint_as_float(ctl->maxabs_x_bits), n))
          : 0.0;
  if (lane == 0) run_lab[2 * g] = run_lab[2 * g + 1] = -1;

  const int64_t first = ((int64_t)blockIdx.x * R + g) * E;
  const int64_t last = first + E < n ? first + E : n;
  int32_t cur = -1, cnt = 0;
  bool head = true;
  uint64_t acc[V], accx = 0;  // two's complement, wrapping
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0;

  // the current run's sums to LDS slot `slot`, or stored when slot < 0
  auto close = [&](int slot) {
    const uint64_t off =
        MAGIC ? (uint64_t)cnt * (uint64_t)__double_as_longlong(kMagic) : 0u;
    if (slot >= 0) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        run_sum[slot][lane * V + v] = (int64_t)(acc[v] - off);
      if (lane < 3) run_sum[slot][G * V + lane] = (int64_t)(accx - off);
      if (lane == 0) {
        run_sum[slot][G * V + 3] = cnt;
        run_lab[slot] = cur;
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (lane * V + v < d)
          Se[(int64_t)cur * d + lane * V + v] = (int64_t)(acc[v] - off);
      if (xyz && lane < 3)
        Sx[(int64_t)cur * 3 + lane] = (int64_t)(accx - off);
      if (lane == 0) size[cur] = cnt;
    }
    cnt = 0;
    accx = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0;
  };

  for (int64_t i = first; i < last; i += kCsU) {
    int32_t lab[kCsU];
    float e[kCsU][V], x[kCsU];
#pragma unroll
    for (int u = 0; u < kCsU; ++u) {
      const uint64_t key = keys[i + u < last ? i + u : last - 1];
      const int64_t p = (int64_t)(uint32_t)key;
      lab[u] = (int32_t)(key >> 32);
      if (V == 4) {
        const float4 r = lane * 4 < d
                             ? *reinterpret_cast<const float4 *>(
                                   emb + p * d + lane * 4)
                             : make_float4(0.f, 0.f, 0.f, 0.f);
        e[u][0] = r.x;
        e[u][1 % V] = r.y;
        e[u][2 % V] = r.z;
        e[u][3 % V] = r.w;
      } else {
        e[u][0] = lane < d ? emb[p * d + lane] : 0.0f;
      }
      x[u] = (xyz && lane < 3) ? xyz[p * 3 + lane] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kCsU; ++u) {
      if (i + u >= last) break;
      if (lab[u] != cur) {
        if (cur >= 0) {
          close(head ? 2 * g : -1);
          head = false;
        }
        cur = lab[u];
      }
      ++cnt;
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += fixed_bits<MAGIC>(e[u][v], sF);
      accx += fixed_bits<MAGIC>(x[u], sX);
    }
  }
  if (cur >= 0) close(head ? 2 * g : 2 * g + 1);
  __syncthreads();
  // joins equal labels of consecutive runs: thread t takes value t
  const int t = threadIdx.x;
  if (t >= W) return;
  unsigned long long *dst = nullptr;
  int64_t stride = 0;
  if (t < G * V) {
    if (t < d) dst = reinterpret_cast<unsigned long long *>(Se) + t, stride = d;
  } else if (t < G * V + 3) {
    if (xyz)
      dst = reinterpret_cast<unsigned long long *>(Sx) + (t - G * V), stride = 3;
  } else {
    dst = reinterpret_cast<unsigned long long *>(size), stride = 1;
  }
  if (!dst) return;
  int32_t at = -1;
  int64_t sum = 0;
  for (int s = 0; s < 2 * R; ++s) {
    const int32_t l = run_lab[s];
    if (l < 0) continue;
    if (l != at) {
      if (at >= 0) atomicAdd(dst + at * stride, (unsigned long long)sum);
      at = l;
      sum = 0;
    }
    sum += run_sum[s][t];
  }
  if (at >= 0) atomicAdd(dst + at * stride, (unsigned long long)sum);
}

// out = (float)(((double)S / size) * 2^-F), 0 for an empty superpoint.
__global__ __launch_bounds__(kCsNT) void k_cs_mean(
    int32_t nc, int32_t d, int32_t n, const int64_t *__restrict__ size,
    const int64_t *__restrict__ Se, const int64_t *__restrict__ Sx,
    float *__restrict__ mean, float *__restrict__ centroid, Ctl *ctl) {
  const int64_t ne = (int64_t)nc * d;
  const int64_t nx = centroid ? (int64_t)nc * 3 : 0;
  const int64_t t = blockIdx.x * (int64_t)kCsNT + threadIdx.x;
  if (t >= ne + nx) return;
  const bool e = t < ne;
  const int F = fixshift_rule(
      __uint_as_float(e ? ctl->maxabs_bits : ctl->maxabs_x_bits), n);
  if ((t == 0 || t == ne) && F < 16) raise_err(ctl, kErrRange);
  const int64_t i = e ? t : t - ne;
  const int64_t c = e ? i / d : i / 3;
  const int64_t S = e ? Se[i] : Sx[i];
  const double q = size[c] > 0 ? (double)S / (double)size[c] : 0.0;
  (e ? mean : centroid)[i] = (float)(q * ldexp(1.0, -F));
}

int label_bits(int32_t nc) {  // bits of nc - 1
  int b = 0;
  while (b < 31 && ((int64_t)1 << b) < (int64_t)nc) ++b;
  return b;
}

template <int G, int V>
void launch_segments(const uint64_t *keys, int32_t n, const float *emb,
                     int32_t d, const float *xyz, const Ctl *ctl,
                     int64_t *size, int64_t *Se, int64_t *Sx,
                     hipStream_t st) {
  constexpr int R = kCsNT / G;
  // entries a group: up to 64 (fewer atomics a point), fewer while that
  // leaves less than four blocks a CU
  int64_t E = n / (1024 * (int64_t)R) / kCsU * kCsU;
  E = E < kCsU ? kCsU : (E > 64 ? 64 : E);
  const unsigned blocks = (unsigned)((n + R * E - 1) / (R * E));
  if (n > 512)
    hipLaunchKernelGGL((k_cs_segments<G, V, true>), dim3(blocks), dim3(kCsNT),
                       0, st, keys, n, (int32_t)E, emb, d, xyz, ctl, size, Se,
                       Sx);
  else
    hipLaunchKernelGGL((k_cs_segments<G, V, false>), dim3(blocks),
                       dim3(kCsNT), 0, st, keys, n, (int32_t)E, emb, d, xyz,
                       ctl, size, Se, Sx);
}

}  // namespace

void stats_reserve(Arena &a, int32_t n, int64_t n_comp, int32_t d) {
  a.take<int64_t>((size_t)n_comp * d);
  a.take<int64_t>((size_t)n_comp * 3);
  a.take<uint64_t>(n);
  a.take<uint64_t>(n);
  a.take<int32_t>(radix_hist_ints(n));
  a.take<int32_t>(scan_blocks(radix_hist_ints(n)) + 1);
  a.take<int32_t>(4);
}

int stats_run(const int32_t *labels, int32_t n, int32_t nc, const float *emb,
              int32_t d, const float *xyz, int64_t *size, float *emb_mean,
              float *centroid, Ctl *ctl, Arena &a, hipStream_t st) {
  int64_t *Se = a.take<int64_t>((size_t)nc * d);
  int64_t *Sx = a.take<int64_t>((size_t)nc * 3);
  uint64_t *keys = a.take<uint64_t>(n);
  uint64_t *keys2 = a.take<uint64_t>(n);
  int32_t *hist = a.take<int32_t>(radix_hist_ints(n));
  int32_t *bsum = a.take<int32_t>(scan_blocks(radix_hist_ints(n)) + 1);
  int32_t *total = a.take<int32_t>(4);
  // two float4 a thread of the largest array, at most eight blocks a CU
  const int64_t most = (int64_t)(n > nc ? n : nc) * d / 8 / kCsNT + 1;
  hipLaunchKernelGGL(k_cs_prep, dim3((unsigned)(most < 2048 ? most : 2048)),
                     dim3(kCsNT), 0, st, labels, n, nc, emb, d, xyz, keys,
                     size, Se, Sx, ctl);
  const bool alt =
      radix_sort_keys(keys, keys2, n, 32, label_bits(nc), hist, bsum, total,
                      ctl, st);
  const uint64_t *sorted = alt ? keys2 : keys;
  // rows of whole 16-byte vectors are read as such; else a lane a dimension
  const bool vec =
      d % 4 == 0 && (reinterpret_cast<uintptr_t>(emb) & 15) == 0;
  const int32_t lanes = vec ? d / 4 : d;
#define EZSP_CS(G, V)                                                        \
  launch_segments<G, V>(sorted, n, emb, d, xyz, ctl, size, Se, Sx, st)
  if (vec) {
    if (lanes <= 4) EZSP_CS(4, 4);
    else if (lanes <= 8) EZSP_CS(8, 4);
    else EZSP_CS(16, 4);
  } else {
    if (lanes <= 4) EZSP_CS(4, 1);
    else if (lanes <= 8) EZSP_CS(8, 1);
    else if (lanes <= 16) EZSP_CS(16, 1);
    else if (lanes <= 32) EZSP_CS(32, 1);
    else EZSP_CS(64, 1);
  }
#undef EZSP_CS
  const int64_t out = (int64_t)nc * (d + (xyz ? 3 : 0));
  hipLaunchKernelGGL(k_cs_mean, dim3((unsigned)((out + kCsNT - 1) / kCsNT)),
                     dim3(kCsNT), 0, st, nc, d, n, size, Se, Sx, emb_mean,
                     xyz ? centroid : nullptr, ctl);
  // stream-asynchronous: device-detected errors stay in ctl for
  // ezsp_sync_status
  return check_hip(hipGetLastError(), "component statistics launch");
}

}  // namespace ezsp
