// ezsp_loss.hip -- pairwise affinity and the contrastive edge loss over the
// k-nearest-neighbour graph (Sec. 3.1: Eq. softmax, a = exp(-|e_p - e_q| /
// tau); Eq. loss, -log a over intra-class edges and -log(1 - a) over
// inter-class edges, with intra edges dropped at random until they are at
// most a fraction rho of the sample).
//
// Edges are the unordered pairs of the kNN relation.  The slot p*k + j that
// owns a pair is the smallest slot listing it: slot (p, j) owns its pair
// when q = nbr[p*k+j] does not appear earlier in row p and either p < q or
// row q does not list p.  That slot's caller-supplied random word draws the
// pair.  With rho < 1 the sample keeps m = min(n_intra,
// floor(rho * n_inter / (1 - rho))) intra pairs: those whose 64-bit key
// (word, slot) is among the m smallest (keys are distinct, so the m-th
// smallest is a sharp threshold).  Every inter pair is kept.
//
// Distances, affinities, loss terms and gradient contributions are fp32; the
// loss is summed in fp64.  -log a is d / tau and -log(1 - a) is
// -log(-expm1(-d / tau)); the gradient of |e_p - e_q| at e_p = e_q is 0.
//
// Layout: a group of G lanes owns one row p of the table, lane i holding
// V consecutive dimensions (a 16-byte vector where rows allow it) of every
// chunk of G * V.  Lane t also classifies slot t of the row and, once the
// group has its distance, evaluates its affinity and loss term; so the
// transcendental functions run once a slot and not once a lane.
//
// Passes (driving tile of 3M points, k = 8, D = 32, rho = 0.3):
//   k_le_prep    the table packed with the classes, the gradient zeroed, and
//                the share of inter pairs guessed from 16384 slots
//   k_le_pairs   classification, distances, affinities, the inter pairs'
//                loss and gradient, and a histogram of the intra pairs' words
//   k_le_pick    the sample's size, and the histogram bin its threshold is in
//   k_le_sample  the intra pairs below that bin: loss and gradient; those in
//                it are listed
//   k_le_select  the threshold among the listed keys
//   k_le_pairs   (DRAWN) the listed pairs up to the threshold
//   k_le_total   the partial losses added up
// The embedding rows and the neighbours' table rows are gathered once; a
// small sample's rows are gathered again.  Where the guess says that the
// sample is a large part of the pairs, k_le_pairs only classifies, k_le_sample
// only lists, and a second k_le_pairs gathers every row once the threshold is
// known.  When the threshold's bin overflows the list (equal words), the host
// runs the radix select over all slots and that second pass instead
// (k_le_hist, k_le_digit).
//
// The row accumulates the gradient on its own side of every sampled pair it
// lists in registers; the other end q gets its side from its own row when q
// lists p too (a mutual pair), and by atomics from the owner slot otherwise.
// A slot's 16-bit status carries the pair type, whether it owns the pair,
// whether the pair is mutual, and where row q lists p, so a mirror slot can
// read the owner's random word.
#include <algorithm>

#include "ezsp_internal.h"

namespace ezsp {

namespace {

// Slot status: bits 0-1 pair type, bit 2 owner, bit 3 mutual, bits 8-15
// the position of p in row q (mutual pairs).
enum : uint16_t {
  kSlotNone = 0,
  kSlotInter = 1,
  kSlotIntra = 2,
  kSlotOwner = 4,
  kSlotMutual = 8
};

constexpr int kLeNT = 256;
constexpr int kLeGrid = 2048;     // grid-stride kernels: blocks at most
constexpr int kLeBitsMin = 8;     // word bits of the first histogram
constexpr int kLeBitsMax = 12;
constexpr int kLeCopies = 4;      // copies of it (atomics on one address)
constexpr int kLeList = 16384;    // listed keys the threshold is found among
constexpr int kLeTile = 2048;     // slots per step of k_le_sample
constexpr int kLeStage = 1024 + kLeTile;  // keys a block stages for the list
constexpr int kLeGuess = 64;      // blocks that guess, a slot a thread
constexpr unsigned kLeListed = 64;  // blocks that take the listed pairs
// The share of the pairs that makes a guessed sample a large one, with a
// gradient and without (a sampled pair is two gathers and no atomics then).
// 1M points, k = 8, D = 32, whole call in us, pair by pair / through the rows:
// a share of 0.055 760/763, 0.077 871/853, 0.5 1670/785; without a gradient
// 0.21 497/504, 0.5 521/431.
constexpr float kLeLarge = 0.06f, kLeLargePlain = 0.25f;

// Word bits of the first histogram: about half the list's capacity of intra
// pairs a bin, if every other slot owned one.
int hist_bits(int64_t ns) {
  int b = kLeBitsMin;
  while (b < kLeBitsMax && (ns >> (b + 1)) > kLeList / 2) ++b;
  return b;
}

template <class T>
__device__ __forceinline__ T block_sum(T v, T *sh) {
  v = wave_sum(v);
  const int wid = threadIdx.x / kWave;
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) sh[wid] = v;
  __syncthreads();
  T s = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)blockDim.x / kWave; ++w) s += sh[w];
  return s;  // valid in thread 0
}

// Packed table row: the point's class, then its k neighbour ids, padded with
// -1 to a power of two of ints (a multiple of 32 beyond that), so that a row
// of up to 31 ids lies in one 128-byte line.  A slot then fetches its
// neighbour's class and ids in one line instead of two.  At 3M points, k = 8
// (24M slots) the pass went from 1.49 to 1.19 ms for a packing of 0.08.
__host__ __device__ __forceinline__ int32_t packed_ints(int32_t k) {
  return k < 8 ? 8 : (k < 16 ? 16 : (k + 1 + 31) / 32 * 32);
}

// First position of p among the ids of a packed row, or -1.
__device__ __forceinline__ int32_t find_in_row(const int4 *__restrict__ r,
                                               int4 first, int32_t k,
                                               int32_t p) {
  int32_t at = -1;
#pragma unroll 4
  for (int32_t t = k / 4; t > 0; --t) {
    const int4 x = r[t];
    at = x.w == p ? 4 * t + 2 : at;
    at = x.z == p ? 4 * t + 1 : at;
    at = x.y == p ? 4 * t : at;
    at = x.x == p ? 4 * t - 1 : at;
  }
  at = first.w == p ? 2 : at;
  at = first.z == p ? 1 : at;
  return first.y == p ? 0 : at;
}

// A lane's part of an embedding row.
template <int G, int V, int NV>
struct RowPart {
  float v[NV][V];
  __device__ __forceinline__ void load(const float *__restrict__ emb,
                                       int64_t p, int32_t d, int lane,
                                       bool live) {
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const int i = (c * G + lane) * V;
      if (V == 4) {
        const float4 x =
            live && i < d ? *reinterpret_cast<const float4 *>(emb + p * d + i)
                          : make_float4(0.f, 0.f, 0.f, 0.f);
        v[c][0] = x.x;
        v[c][1 % V] = x.y;
        v[c][2 % V] = x.z;
        v[c][3 % V] = x.w;
      } else {
        v[c][0] = live && i < d ? emb[p * d + i] : 0.0f;
      }
    }
  }
};

// Sum over the G lanes of a group, the same in every lane: DPP within 16
// lanes (quad permutes, half-row and row mirrors), shuffles beyond.
template <int G>
__device__ __forceinline__ float group_sum(float x) {
#define EZSP_DPP(ctrl)                                                      \
  x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xf, \
                                               0xf, true))
  if (G >= 2) EZSP_DPP(0xb1);   // quad_perm(1, 0, 3, 2)
  if (G >= 4) EZSP_DPP(0x4e);   // quad_perm(2, 3, 0, 1)
  if (G >= 8) EZSP_DPP(0x141);  // row_half_mirror
  if (G >= 16) EZSP_DPP(0x140);  // row_mirror
#undef EZSP_DPP
  if (G >= 32) x += __shfl_xor(x, 16, kWave);
  if (G >= 64) x += __shfl_xor(x, 32, kWave);
  return x;
}

template <int G, int V, int NV>
__device__ __forceinline__ float squared(const RowPart<G, V, NV> &a,
                                         const RowPart<G, V, NV> &b) {
  float part = 0.0f;
#pragma unroll
  for (int c = 0; c < NV; ++c)
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const float df = a.v[c][v] - b.v[c][v];
      part += df * df;
    }
  return group_sum<G>(part);
}

// grad row p += x.  A lane holds V consecutive dimensions; its atomics would
// leave V - 1 floats between neighbouring lanes', so a row of vectors goes
// through LDS and consecutive lanes add consecutive floats (1M points, k = 8,
// D = 64, rho = 1: 2.18 -> 0.87 ms).  stage: the block's kLeNT * V floats (V > 1).
template <int G, int V, int NV>
__device__ __forceinline__ void add_row(float *grad, int64_t p, int32_t d,
                                        int lane, const RowPart<G, V, NV> &x,
                                        float *stage) {
  if constexpr (V == 1) {
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const int i = c * G + lane;
      if (i < d) unsafeAtomicAdd(grad + p * d + i, x.v[c][0]);
    }
  } else {
    static_assert(V == 4, "16-byte vectors");
    float *mine = stage + ((int)threadIdx.x - lane) * V;  // the group's
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      *reinterpret_cast<float4 *>(mine + lane * V) =
          make_float4(x.v[c][0], x.v[c][1 % V], x.v[c][2 % V], x.v[c][3 % V]);
      // the group is part of one wave, whose LDS accesses stay in order
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int i = c * G * V + v * G + lane;
        if (i < d) unsafeAtomicAdd(grad + p * d + i, mine[v * G + lane]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}
template <int V>
constexpr int stage_floats() { return V == 1 ? 1 : kLeNT * V; }

// d loss / d dist / dist of a pair at distance dist, x = dist / tau
__device__ __forceinline__ float pair_coef(bool intra, float dist, float x,
                                           float inv_tau) {
  if (!(dist > 0.0f)) return 0.0f;
  return intra ? inv_tau / dist : -inv_tau / (expm1f(x) * dist);
}

__device__ __forceinline__ float pair_term(bool intra, float x) {
  return intra ? x : -logf(-expm1f(-x));
}

// Zeroes the gradient and the histogram.
__device__ __forceinline__ void clear_arrays(float *grad, int64_t count,
                                             uint32_t *hist, int32_t nh) {
  const int64_t t = blockIdx.x * (int64_t)kLeNT + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kLeNT;
  for (int64_t i = t; i < nh; i += step) hist[i] = 0;
  if (!grad) return;
  int64_t done = 0;
  if ((reinterpret_cast<uintptr_t>(grad) & 15) == 0) {
    float4 *g4 = reinterpret_cast<float4 *>(grad);
    for (int64_t i = t; i < count / 4; i += step)
      g4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    done = count / 4 * 4;
  }
  for (int64_t i = done + t; i < count; i += step) grad[i] = 0.0f;
}

// Whether the intra sample is guessed to be a large part of the pairs, from
// the guess's counts of inter pairs and of all pairs per block.  The same in
// every lane; whole waves only.
__device__ __forceinline__ bool guessed_large(
    const uint32_t *__restrict__ guess, double rho, bool grad) {
  static_assert(kLeGuess == kWave, "a count a lane");
  const int lane = threadIdx.x & (kWave - 1);
  const float inter = (float)wave_sum(guess[lane]);
  const float all = (float)wave_sum(guess[kLeGuess + lane]);
  const float cap = (float)(rho / (1.0 - rho)) * inter;  // of the sample
  return fminf(all - inter, cap) > (grad ? kLeLarge : kLeLargePlain) * all;
}

// guess: null, or counts of the first kLeGuess blocks' slots (guessed_large;
// the grid has as many blocks then).
__global__ __launch_bounds__(kLeNT) void k_le_prep(
    const int32_t *__restrict__ nbr, int32_t n, int32_t k,
    const int32_t *__restrict__ cls, int4 *__restrict__ table, float *grad,
    int64_t count, uint32_t *hist, int32_t nh, uint32_t *__restrict__ guess) {
  __shared__ uint32_t shu[kLeNT / kWave];
  const bool guesses = guess && blockIdx.x < kLeGuess;  // block-uniform
  int32_t gp = 0, gq = -1, gcp = 0, gcq = 0;
  if (guesses) {
    // a slot of each of as many equal ranges, not at a fixed place in it
    const uint32_t i = blockIdx.x * kLeNT + threadIdx.x;
    const uint32_t ns = (uint32_t)((int64_t)n * k);
    const uint32_t range = max(ns / (kLeGuess * kLeNT), 1u);
    const uint32_t s = i * range + ((i * 2654435761u) >> 8) % range;
    gp = (int32_t)(s / (uint32_t)k);
    gq = s < ns ? nbr[s] : -1;
  }
  clear_arrays(grad, count, hist, nh);
  const bool pair = gq >= 0 && gq < n && gq != gp;
  if (pair) {
    gcp = cls[gp];
    gcq = cls[gq];
  }
  // a thread four ints of a packed row
  const int32_t quads = packed_ints(k) / 4;
  const int64_t step = (int64_t)gridDim.x * kLeNT;
  for (int64_t i = blockIdx.x * (int64_t)kLeNT + threadIdx.x;
       i < (int64_t)n * quads; i += step) {
    const int32_t p = (int32_t)(i / quads);
    const int32_t j = (int32_t)(i - (int64_t)p * quads) * 4 - 1;
    const int32_t *row = nbr + (int64_t)p * k;
    table[i] = make_int4(j < 0 ? cls[p] : (j < k ? row[j] : -1),
                         j + 1 < k ? row[j + 1] : -1,
                         j + 2 < k ? row[j + 2] : -1,
                         j + 3 < k ? row[j + 3] : -1);
  }
  if (!guesses) return;
  const uint32_t inter = block_sum((uint32_t)(pair && gcp != gcq), shu);
  const uint32_t all = block_sum((uint32_t)pair, shu);
  if (threadIdx.x == 0) {
    guess[blockIdx.x] = inter;
    guess[kLeGuess + blockIdx.x] = all;
  }
}

__global__ __launch_bounds__(kLeNT) void k_le_clear(uint32_t *hist,
                                                    int32_t nh) {
  clear_arrays(nullptr, 0, hist, nh);
}

__device__ __forceinline__ uint64_t draw_key(const uint32_t *word, int64_t s) {
  return ((uint64_t)word[s] << 32) | (uint64_t)s;
}

// Loss and gradient of one sampled intra pair by its owner slot, both sides
// by atomics; the term is returned in lane 0 of the group.
template <int G, int V, int NV>
__device__ __forceinline__ double take_pair(
    const float *__restrict__ emb, int32_t d, const int32_t *__restrict__ nbr,
    int32_t k, uint32_t s, float inv_tau, float *grad, uint8_t *sampled,
    int lane, float *stage) {
  const int64_t p = (int64_t)(s / (uint32_t)k);
  const int64_t q = nbr[s];
  RowPart<G, V, NV> a, b;
  a.load(emb, p, d, lane, true);
  b.load(emb, q, d, lane, true);
  const float dist = sqrtf(squared(a, b));
  const float x = dist * inv_tau;
  const float coef = pair_coef(true, dist, x, inv_tau);
  if (grad && coef != 0.0f) {
#pragma unroll
    for (int c = 0; c < NV; ++c)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float g = coef * (a.v[c][v] - b.v[c][v]);
        a.v[c][v] = g;
        b.v[c][v] = -g;
      }
    add_row(grad, p, d, lane, a, stage);
    add_row(grad, q, d, lane, b, stage);
  }
  if (lane != 0) return 0.0;
  if (sampled) sampled[s] = 1;
  return (double)pair_term(true, x);
}

// The listed pairs up to the threshold, by the first kLeListed blocks; a
// thread's terms are returned.
template <int G, int V, int NV>
__device__ __forceinline__ double take_listed(
    const float *__restrict__ emb, int32_t d, const int32_t *__restrict__ nbr,
    int32_t k, float tau, float *__restrict__ grad,
    uint8_t *__restrict__ sampled, const uint64_t *__restrict__ list,
    float *stage, const Ctl *ctl) {
  double lsum = 0.0;
  if (ctl->sel_mode == 2) {
    const uint32_t nc = min(ctl->sel_cand, (uint32_t)kLeList);
    const uint64_t thr = ctl->sel_prefix;
    const float inv_tau = 1.0f / tau;
    const int lane = threadIdx.x & (G - 1);
    const uint32_t blocks = min(gridDim.x, kLeListed);
    for (uint32_t i = (blockIdx.x * kLeNT + threadIdx.x) / G; i < nc;
         i += blocks * (kLeNT / G))
      if (list[i] <= thr)
        lsum += take_pair<G, V, NV>(emb, d, nbr, k, (uint32_t)list[i], inv_tau,
                                    grad, sampled, lane, stage);
  }
  return lsum;
}

// Status of slot (p, j) that lists q != p, 0 <= q < n.
__device__ __forceinline__ uint32_t slot_status(const int4 *__restrict__ prow,
                                                int4 pfirst,
                                                const int4 *__restrict__ qrow,
                                                int32_t k, int32_t p,
                                                int32_t j, int32_t q) {
  const int4 qfirst = qrow[0];
  const int32_t jq = find_in_row(qrow, qfirst, k, p);
  const int32_t jp = find_in_row(prow, pfirst, k, q);
  if (jp != j) return kSlotNone;  // an earlier slot of row p lists q
  uint32_t st = qfirst.x == pfirst.x ? kSlotIntra : kSlotInter;
  if (p < q || jq < 0) st |= kSlotOwner;
  if (jq >= 0) st |= kSlotMutual | (uint32_t)(jq << 8);
  return st;
}

// The classification alone, a slot a thread: statuses, pair counts and the
// block's histogram of the intra pairs' words.  False for an id out of range.
__device__ __forceinline__ bool classify_slots(
    int32_t n, const int32_t *__restrict__ nbr, int32_t k,
    const int4 *__restrict__ table, const uint32_t *__restrict__ word,
    int bits, uint16_t *__restrict__ status, uint32_t *h,
    unsigned long long &edges, unsigned long long &intra) {
  bool inside = true;
  const int64_t ns = (int64_t)n * k, quads = packed_ints(k) / 4;
  for (int64_t s = blockIdx.x * (int64_t)kLeNT + threadIdx.x; s < ns;
       s += (int64_t)gridDim.x * kLeNT) {
    const int32_t p = (int32_t)((uint32_t)s / (uint32_t)k);
    const int32_t j = (int32_t)(s - (int64_t)p * k), q = nbr[s];
    uint32_t st = kSlotNone;
    if (q < -1 || q >= n) {
      inside = false;
    } else if (q >= 0 && q != p) {
      const int4 *prow = table + p * quads;
      st = slot_status(prow, prow[0], table + q * quads, k, p, j, q);
    }
    status[s] = (uint16_t)st;
    if (st & kSlotOwner) {
      ++edges;
      if ((st & 3) == kSlotIntra) {
        ++intra;
        atomicAdd(&h[word[s] >> (32 - bits)], 1u);
      }
    }
  }
  return inside;
}

// Everything that needs every slot: see the head of the file.  Bound by its
// gathers: a random-order cloud fetches an embedding row and a packed table
// row per slot.  Where the sample is guessed to be large it only classifies.
// DRAWN: statuses and the sample's threshold are known.  Where the sample is
// guessed to be large this does the rest, a mirror slot reading its owner's
// word, so that only one-sided pairs need atomics on the far row; else the
// first blocks take the listed pairs up to the threshold.  When the list
// overflowed it waits for another launch (rest), which in the second case
// adds the whole intra sample.
template <int G, int V, int NV, bool DRAWN>
__global__ __launch_bounds__(kLeNT) void k_le_pairs(
    bool rest, const uint32_t *__restrict__ guess, double rho,
    const float *__restrict__ emb, int32_t n, int32_t d,
    const int32_t *__restrict__ nbr, int32_t k,
    const int4 *__restrict__ table, const uint32_t *__restrict__ word,
    float tau, int bits, uint16_t *__restrict__ status,
    float *__restrict__ affinity, float *__restrict__ grad,
    uint8_t *__restrict__ sampled, uint32_t *__restrict__ hist,
    unsigned long long *__restrict__ part_edges,
    unsigned long long *__restrict__ part_intra,
    const uint64_t *__restrict__ list, double *__restrict__ part_loss,
    Ctl *ctl) {
  constexpr int kRows = kLeNT / G;  // rows per block and step
  constexpr int U = NV == 1 ? 4 : (NV == 2 ? 2 : 1);  // gathers in flight
  __shared__ uint32_t h[DRAWN ? 1 : 1 << kLeBitsMax];
  __shared__ double shd[kLeNT / kWave];
  __shared__ unsigned long long shu[kLeNT / kWave];
  __shared__ alignas(16) float stage[stage_floats<V>()];
  const bool large = DRAWN ? ctl->sel_large != 0
                           : guess && guessed_large(guess, rho, grad != nullptr);
  if (DRAWN) {
    const bool wait = !rest && ctl->sel_dense;
    if (wait || (!rest && !large)) {
      const double t = wait || blockIdx.x >= kLeListed
                           ? 0.0
                           : take_listed<G, V, NV>(emb, d, nbr, k, tau, grad,
                                                   sampled, list, stage, ctl);
      const double tl = block_sum(t, shd);
      if (threadIdx.x == 0) part_loss[blockIdx.x] = tl;
      return;
    }
  }
  const bool take_all = !DRAWN && rho >= 1.0;
  const int mode = DRAWN ? ctl->sel_mode : 0;
  const uint64_t thr = DRAWN ? ctl->sel_prefix : 0;
  const int lane = threadIdx.x & (G - 1);
  const int shift0 = (int)(threadIdx.x & (kWave - 1) & ~(G - 1));
  const uint64_t gmask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1);
  const float inv_tau = 1.0f / tau;
  if (!DRAWN)
    for (int i = threadIdx.x; i < (1 << bits); i += kLeNT) h[i] = 0;
  __syncthreads();
  unsigned long long edges = 0, intra = 0;
  double lsum = 0.0;
  bool finite = true, inside = true;
  const int64_t quads = packed_ints(k) / 4;
  const auto finish = [&]() {
    if (!finite) raise_err(ctl, kErrNonFinite);
    if (!inside) raise_err(ctl, kErrBadIndex);
    const double tl = block_sum(lsum, shd);
    if (threadIdx.x == 0) part_loss[blockIdx.x] = tl;
    if (DRAWN) return;
    const unsigned long long te = block_sum(edges, shu);
    const unsigned long long ti = block_sum(intra, shu);
    if (threadIdx.x == 0) {
      part_edges[blockIdx.x] = te;
      part_intra[blockIdx.x] = ti;
    }
    if (take_all) return;
    uint32_t *to = hist + ((size_t)(blockIdx.x % kLeCopies) << bits);
    for (int i = threadIdx.x; i < (1 << bits); i += kLeNT)
      if (h[i]) atomicAdd(&to[i], h[i]);
  };
  if (!DRAWN && large) {
    inside = classify_slots(n, nbr, k, table, word, bits, status, h, edges,
                            intra);
    finish();
    return;
  }
  for (int64_t p = (int64_t)blockIdx.x * kRows + threadIdx.x / G; p < n;
       p += (int64_t)gridDim.x * kRows) {
    const int32_t *row = nbr + p * k;
    RowPart<G, V, NV> ep, acc;
    ep.load(emb, p, d, lane, true);
#pragma unroll
    for (int c = 0; c < NV; ++c)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        finite = finite && isfinite(ep.v[c][v]);
        acc.v[c][v] = 0.0f;
      }
    const int4 *prow = table + p * quads;
    const int4 pfirst = DRAWN ? make_int4(0, 0, 0, 0) : prow[0];
    bool any = false;
    for (int32_t r0 = 0; r0 < k; r0 += G) {
      // lane t classifies slot r0 + t
      const int32_t j = r0 + lane;
      const bool slot = j < k;
      int32_t q = slot ? row[j] : -1;
      if (q < -1 || q >= n) {
        inside = false;
        q = -1;
      }
      uint32_t st = kSlotNone;
      if (DRAWN) {
        st = slot ? status[p * k + j] : kSlotNone;
      } else if (q >= 0 && q != p) {
        st = slot_status(prow, pfirst, table + q * quads, k, (int32_t)p, j, q);
      }
      const bool owner = (st & kSlotOwner) != 0;
      const bool same = (st & 3) == kSlotIntra;
      bool take = (st & 3) == kSlotInter || (take_all && same);
      if (DRAWN) {
        take = take && large;
        if (same)
          take = mode == 1 ||
                 (mode == 2 &&
                  draw_key(word, owner ? p * k + j
                                       : (int64_t)q * k + (st >> 8)) <= thr);
      } else {
        edges += owner;
        intra += owner && same;
        if (!take_all && owner && same)
          atomicAdd(&h[word[p * k + j] >> (32 - bits)], 1u);
      }
      const uint64_t takes = (__ballot(take) >> shift0) & gmask;
      const uint64_t ones = (__ballot(!(st & kSlotMutual)) >> shift0) & gmask;
      const uint64_t sames = (__ballot(same) >> shift0) & gmask;
      if (DRAWN && !large && !takes) continue;
      // the distances of the G slots, U gathers in flight
      float mine = 0.0f;
      const int32_t jn = min(G, k - r0);
      for (int32_t j0 = 0; j0 < jn; j0 += U) {
        RowPart<G, V, NV> eq[U];
        int32_t qs[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          qs[u] = __shfl(q, (j0 + u) & (G - 1), G);
          eq[u].load(emb, qs[u], d, lane, j0 + u < jn && qs[u] >= 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float part = squared(ep, eq[u]);
          mine = lane == j0 + u ? part : mine;
          if (grad && j0 + u < jn && ((takes >> (j0 + u)) & 1)) {
            const float dist = sqrtf(part);
            const float coef = pair_coef((sames >> (j0 + u)) & 1, dist,
                                         dist * inv_tau, inv_tau);
            const bool far = (ones >> (j0 + u)) & 1;
            any = true;
#pragma unroll
            for (int c = 0; c < NV; ++c)
#pragma unroll
              for (int v = 0; v < V; ++v) {
                const float g = coef * (ep.v[c][v] - eq[u].v[c][v]);
                acc.v[c][v] += g;
                eq[u].v[c][v] = -g;
              }
            // q does not list p: the owner slot gives q its side
            if (far && coef != 0.0f)
              add_row(grad, qs[u], d, lane, eq[u], stage);
          }
        }
      }
      if (slot) {
        const float x = sqrtf(mine) * inv_tau;
        if (take && owner) lsum += (double)pair_term(same, x);
        const int64_t s = p * k + j;
        if (!DRAWN) status[s] = (uint16_t)st;
        if (affinity) affinity[s] = q >= 0 ? expf(-x) : 0.0f;
        if (sampled && (!DRAWN || large || take))
          sampled[s] = (take && owner) ? 1 : 0;
      }
    }
    if (any) add_row(grad, p, d, lane, acc, stage);
  }
  finish();
}

// The pair counts, the size of the intra sample, the histogram bin of its
// largest kept key (sel_prefix) and that key's rank in the bin (sel_rank).
// sel_mode: 0 no intra pair is kept, 1 all, 2 those up to a threshold.
// sel_dense: the bin holds more keys than the list.  sel_large: the guess.
constexpr int kLePickNT = 1024;

__global__ __launch_bounds__(kLePickNT) void k_le_pick(
    Ctl *ctl, const uint32_t *__restrict__ guess, bool grad,
    const uint32_t *__restrict__ hist, int bits, double rho,
    const unsigned long long *__restrict__ part_edges,
    const unsigned long long *__restrict__ part_intra, int32_t nparts) {
  __shared__ unsigned long long sh[kLePickNT / kWave];
  __shared__ int64_t wsum[kLePickNT / kWave];
  __shared__ int64_t keep;
  __shared__ bool search;
  unsigned long long e = 0, a = 0;
  for (int32_t i = threadIdx.x; i < nparts; i += kLePickNT) {
    e += part_edges[i];
    a += part_intra[i];
  }
  const unsigned long long edges = block_sum(e, sh);
  const unsigned long long intra = block_sum(a, sh);
  const bool large = guess && guessed_large(guess, rho, grad);
  if (threadIdx.x == 0) {
    const int64_t n_intra = (int64_t)intra;
    const int64_t n_inter = (int64_t)edges - n_intra;
    int64_t m = n_intra;
    if (rho < 1.0) {
      const double cap = floor(
          __ddiv_rn(__dmul_rn(rho, (double)n_inter), __dsub_rn(1.0, rho)));
      if (cap < (double)m) m = (int64_t)cap;
    }
    keep = m;
    ctl->le_edges = edges;
    ctl->le_intra = intra;
    ctl->le_keep = (unsigned long long)m;
    const int mode = m == 0 ? 0 : (m == n_intra ? 1 : 2);
    search = mode == 2;
    ctl->sel_mode = mode;
    ctl->sel_dense = 0;
    ctl->sel_large = large;
    ctl->sel_prefix = mode == 1 ? ~0ull : 0ull;
    ctl->sel_rank = 0;
    ctl->sel_cand = 0;
  }
  __syncthreads();
  const int64_t m = keep;
  if (!search) return;
  // bins in order, each thread a contiguous share
  const int per = ((1 << bits) + kLePickNT - 1) / kLePickNT;
  int64_t c[(1 << kLeBitsMax) / kLePickNT], s = 0, tot;
  for (int i = 0; i < (1 << kLeBitsMax) / kLePickNT; ++i) {
    c[i] = 0;
    const int b = (int)threadIdx.x * per + i;
    if (i < per && b < (1 << bits))
      for (int q = 0; q < kLeCopies; ++q) c[i] += hist[(q << bits) + b];
    s += c[i];
  }
  int64_t before = block_excl_scan<kLePickNT>(s, wsum, &tot);
  for (int i = 0; i < per; ++i) {
    if (before <= m - 1 && m - 1 < before + c[i]) {
      ctl->sel_prefix = (uint64_t)((int)threadIdx.x * per + i);
      ctl->sel_rank = m - 1 - before;
      if (c[i] > kLeList) ctl->sel_dense = 1;
    }
    before += c[i];
  }
}

// The sampled intra pairs below the threshold's bin (all of them in mode 1),
// found by streaming statuses and words; a block lists a tile's pairs in LDS
// and its groups of lanes then share them out.  Keys in the bin are listed;
// no more than that where the sample is guessed to be large.
template <int G, int V, int NV>
__global__ __launch_bounds__(kLeNT) void k_le_sample(
    const float *__restrict__ emb, int32_t d, const int32_t *__restrict__ nbr,
    int32_t k, const uint16_t *__restrict__ status,
    const uint32_t *__restrict__ word, int64_t ns, float tau, int bits,
    float *__restrict__ grad, uint8_t *__restrict__ sampled,
    uint64_t *__restrict__ list, double *__restrict__ part_loss, Ctl *ctl) {
  __shared__ uint32_t sure[kLeTile];
  __shared__ uint64_t stage[kLeStage];
  __shared__ uint32_t n_sure, n_stage, at;
  __shared__ double shd[kLeNT / kWave];
  __shared__ alignas(16) float astage[stage_floats<V>()];
  const bool large = ctl->sel_large != 0;
  const bool idle = ctl->sel_dense != 0 || ctl->sel_mode == 0 ||
                    (large && ctl->sel_mode != 2);
  if (idle) {
    if (threadIdx.x == 0) part_loss[blockIdx.x] = 0.0;
    return;
  }
  const uint64_t bin = ctl->sel_prefix;  // past every bin in mode 1
  const float inv_tau = 1.0f / tau;
  const int lane = threadIdx.x & (G - 1);
  double lsum = 0.0;
  if (threadIdx.x == 0) n_sure = n_stage = 0;
  __syncthreads();
  for (int64_t t0 = (int64_t)blockIdx.x * kLeTile; t0 < ns;
       t0 += (int64_t)gridDim.x * kLeTile) {
#pragma unroll
    for (int j = 0; j < kLeTile / kLeNT; ++j) {
      const int64_t s = t0 + j * kLeNT + threadIdx.x;
      if (s < ns && (status[s] & (3 | kSlotOwner)) == (kSlotIntra | kSlotOwner)) {
        const uint32_t w = word[s];
        const uint64_t b = w >> (32 - bits);
        if (b == bin)
          stage[atomicAdd(&n_stage, 1u)] = ((uint64_t)w << 32) | (uint64_t)s;
        else if (b < bin && !large)
          sure[atomicAdd(&n_sure, 1u)] = (uint32_t)s;
      }
    }
    __syncthreads();
    const uint32_t ne = n_sure, nst = n_stage;
    for (uint32_t i = threadIdx.x / G; i < ne; i += kLeNT / G)
      lsum += take_pair<G, V, NV>(emb, d, nbr, k, sure[i], inv_tau, grad,
                                  sampled, lane, astage);
    const bool flush = nst > 0 && (nst >= kLeStage - kLeTile ||
                                   t0 + (int64_t)gridDim.x * kLeTile >= ns);
    if (flush && threadIdx.x == 0) at = atomicAdd(&ctl->sel_cand, nst);
    __syncthreads();
    if (flush)  // the bin holds at most kLeList keys
      for (uint32_t i = threadIdx.x; i < nst; i += kLeNT)
        if (at + i < (uint32_t)kLeList) list[at + i] = stage[i];
    __syncthreads();
    if (threadIdx.x == 0) {
      n_sure = 0;
      if (flush) n_stage = 0;
    }
    __syncthreads();
  }
  const double t = block_sum(lsum, shd);
  if (threadIdx.x == 0) part_loss[blockIdx.x] = t;
}

// The sel_rank-th smallest of the listed keys, to sel_prefix: a radix select
// in LDS, 8 bits a pass, ending once a digit's bin holds one key.
__global__ __launch_bounds__(kLePickNT) void k_le_select(
    Ctl *ctl, const uint64_t *__restrict__ list, int bits) {
  __shared__ uint64_t key[kLeList];
  __shared__ uint32_t h[256];
  __shared__ uint32_t wsum[kLePickNT / kWave];
  __shared__ uint64_t s_prefix, s_mask;
  __shared__ int64_t s_rank;
  __shared__ uint32_t s_count;
  if (ctl->sel_dense != 0 || ctl->sel_mode != 2) return;
  const uint32_t nc = min(ctl->sel_cand, (uint32_t)kLeList);
  for (uint32_t i = threadIdx.x; i < nc; i += kLePickNT) key[i] = list[i];
  if (threadIdx.x == 0) {
    s_prefix = ctl->sel_prefix << (64 - bits);
    s_mask = ~0ull << (64 - bits);
    s_rank = ctl->sel_rank;
    s_count = nc;
  }
  __syncthreads();
  for (int top = 64 - bits; top > 0 && s_count > 1; top -= 8) {
    const int shift = top > 8 ? top - 8 : 0;
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t prefix = s_prefix, mask = s_mask;
    const int64_t rank = s_rank;
    const uint32_t low = (1u << (top - shift)) - 1;
    for (uint32_t i = threadIdx.x; i < nc; i += kLePickNT)
      if ((key[i] & mask) == prefix)
        atomicAdd(&h[(uint32_t)(key[i] >> shift) & low], 1u);
    __syncthreads();
    const uint32_t c = threadIdx.x < 256 ? h[threadIdx.x] : 0u;
    uint32_t tot;
    const uint32_t before = block_excl_scan<kLePickNT>(c, wsum, &tot);
    if (c > 0 && before <= rank && rank < (int64_t)before + c) {
      s_prefix = prefix | ((uint64_t)threadIdx.x << shift);
      s_mask = mask | ((uint64_t)low << shift);
      s_rank = rank - before;
      s_count = c;
    }
    __syncthreads();
  }
  // the one key left
  for (uint32_t i = threadIdx.x; i < nc; i += kLePickNT)
    if ((key[i] & s_mask) == s_prefix) ctl->sel_prefix = key[i];
}

__global__ __launch_bounds__(kLePickNT) void k_le_total(
    const double *__restrict__ part, int32_t nparts, Ctl *ctl) {
  __shared__ double sh[kLePickNT / kWave];
  double s = 0.0;
  for (int32_t i = threadIdx.x; i < nparts; i += kLePickNT) s += part[i];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) ctl->le_loss = s;
}

// --- the general selection: radix passes over every slot ------------------

__global__ void k_le_dense_start(Ctl *ctl) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  ctl->sel_prefix = 0;
  ctl->sel_mask = 0;
  ctl->sel_rank = (int64_t)ctl->le_keep - 1;
}

// One radix-select pass: histogram of the 8-bit digit at `shift` over the
// intra keys that match the prefix fixed so far.
__global__ __launch_bounds__(kLeNT) void k_le_hist(
    const uint16_t *__restrict__ status, const uint32_t *__restrict__ word,
    int64_t ns, int shift, const Ctl *ctl, uint32_t *hist) {
  if (ctl->sel_mode != 2) return;
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t prefix = ctl->sel_prefix, mask = ctl->sel_mask;
  for (int64_t s = blockIdx.x * (int64_t)kLeNT + threadIdx.x; s < ns;
       s += (int64_t)gridDim.x * kLeNT) {
    if ((status[s] & (3 | kSlotOwner)) != (kSlotIntra | kSlotOwner)) continue;
    const uint64_t key = draw_key(word, s);
    if ((key & mask) == prefix) atomicAdd(&h[(key >> shift) & 255], 1u);
  }
  __syncthreads();
  const uint32_t c = h[threadIdx.x];
  if (c) atomicAdd(&hist[threadIdx.x], c);
}

// Fixes the digit at `shift` (256 threads, one per digit) and clears the
// histogram for the next pass.
__global__ __launch_bounds__(256) void k_le_digit(Ctl *ctl, uint32_t *hist,
                                                  int shift) {
  __shared__ int64_t wsum[256 / kWave];
  __shared__ int64_t tot;
  const bool live = ctl->sel_mode == 2;
  const int64_t c = live ? (int64_t)hist[threadIdx.x] : 0;
  hist[threadIdx.x] = 0;
  const int64_t excl = block_excl_scan<256>(c, wsum, &tot);
  if (!live) return;
  const int64_t r = ctl->sel_rank;
  __syncthreads();
  if (c > 0 && excl <= r && r < excl + c) {
    ctl->sel_rank = r - excl;
    ctl->sel_prefix |= (uint64_t)threadIdx.x << shift;
    ctl->sel_mask |= (uint64_t)0xff << shift;
  }
}

unsigned grid_for(int64_t items) {
  const int64_t b = (items + kLeNT - 1) / kLeNT;
  return (unsigned)(b < kLeGrid ? (b < 1 ? 1 : b) : kLeGrid);
}

// Workspace of one call.
struct LossWork {
  int4 *table;
  uint16_t *status;
  uint32_t *hist;
  uint64_t *list;
  unsigned long long *part_edges, *part_intra;
  double *part_loss;  // of the first k_le_pairs, the second, and k_le_sample:
                      // kLeGrid each
  uint32_t *guess;
};

LossWork take_work(Arena &a, int32_t n, int32_t k) {
  const int64_t ns = (int64_t)n * k;
  LossWork w;
  w.table = a.take<int4>((size_t)n * (packed_ints(k) / 4));
  w.status = a.take<uint16_t>((size_t)ns);
  w.hist = a.take<uint32_t>((size_t)kLeCopies << kLeBitsMax);
  w.list = a.take<uint64_t>(kLeList);
  w.part_edges = a.take<unsigned long long>(kLeGrid);
  w.part_intra = a.take<unsigned long long>(kLeGrid);
  w.part_loss = a.take<double>(3 * kLeGrid);
  w.guess = a.take<uint32_t>(2 * kLeGuess);
  return w;
}

// The kernels of one row layout.
template <int G, int V, int NV>
struct Rows {
  static unsigned blocks(int64_t n) { return grid_for(n * G); }

  template <bool DRAWN>
  static void pairs(const LossArgs &g, const LossWork &w,
                    const uint32_t *guess, int bits, bool rest, Ctl *ctl,
                    hipStream_t st) {
    const unsigned pb = blocks(g.n);
    hipLaunchKernelGGL((k_le_pairs<G, V, NV, DRAWN>), dim3(pb), dim3(kLeNT), 0,
                       st, rest, guess, g.rho, g.emb, g.n, g.d, g.nbr, g.k,
                       w.table, g.word, (float)g.tau, bits, w.status,
                       g.affinity, g.grad, g.sampled, w.hist, w.part_edges,
                       w.part_intra, w.list, w.part_loss + (DRAWN ? pb : 0),
                       ctl);
  }

  // finding the sample's threshold, and with it its sure pairs
  static void sample(const LossArgs &g, const LossWork &w, int bits, Ctl *ctl,
                     unsigned sb, hipStream_t st) {
    const int64_t ns = (int64_t)g.n * g.k;
    hipLaunchKernelGGL((k_le_sample<G, V, NV>), dim3(sb), dim3(kLeNT), 0, st,
                       g.emb, g.d, g.nbr, g.k, w.status, g.word,
                       ns, (float)g.tau, bits, g.grad, g.sampled, w.list,
                       w.part_loss + 2 * blocks(g.n), ctl);
    hipLaunchKernelGGL(k_le_select, dim3(1), dim3(kLePickNT), 0, st, ctl,
                       w.list, bits);
  }
};

template <class R>
int run_rows(const LossArgs &g, const LossWork &w, Ctl *ctl, Ctl *hc,
             hipStream_t st) {
  const int64_t ns = (int64_t)g.n * g.k;
  const int bits = hist_bits(ns);
  const unsigned pb = R::blocks(g.n);
  const int64_t tiles = (ns + kLeTile - 1) / kLeTile;
  const unsigned sb = (unsigned)(tiles < kLeGrid ? tiles : kLeGrid);
  const bool draws = g.rho < 1.0;
  uint32_t *guess = draws ? w.guess : nullptr;
  prof_begin("edge_loss", st);
  const unsigned quads = grid_for((int64_t)g.n * (packed_ints(g.k) / 4));
  hipLaunchKernelGGL(k_le_prep, dim3(std::max(quads, (unsigned)kLeGuess)),
                     dim3(kLeNT), 0, st, g.nbr, g.n, g.k, g.cls, w.table,
                     g.grad, (int64_t)g.n * g.d, w.hist, kLeCopies << bits,
                     guess);
  R::template pairs<false>(g, w, guess, bits, false, ctl, st);
  hipLaunchKernelGGL(k_le_pick, dim3(1), dim3(kLePickNT), 0, st, ctl, guess,
                     g.grad != nullptr, w.hist, bits, g.rho, w.part_edges, w.part_intra, (int32_t)pb);
  if (draws) {
    R::sample(g, w, bits, ctl, sb, st);
    R::template pairs<true>(g, w, guess, bits, false, ctl, st);
  }
  const int32_t parts = (int32_t)(draws ? 2 * pb + sb : pb);
  hipLaunchKernelGGL(k_le_total, dim3(1), dim3(kLePickNT), 0, st, w.part_loss,
                     parts, ctl);
  prof_end(st);
  int rc = read_ctl(ctl, hc, st);
  if (rc || hc->err || !hc->sel_dense) return rc;
  prof_begin("edge_loss", st);
  hipLaunchKernelGGL(k_le_dense_start, dim3(1), dim3(64), 0, st, ctl);
  hipLaunchKernelGGL(k_le_clear, dim3(1), dim3(kLeNT), 0, st, w.hist, 256);
  for (int shift = 56; shift >= 0; shift -= 8) {
    hipLaunchKernelGGL(k_le_hist, dim3(grid_for(ns)), dim3(kLeNT), 0, st,
                       w.status, g.word, ns, shift, ctl, w.hist);
    hipLaunchKernelGGL(k_le_digit, dim3(1), dim3(256), 0, st, ctl, w.hist,
                       shift);
  }
  R::template pairs<true>(g, w, guess, bits, true, ctl, st);
  hipLaunchKernelGGL(k_le_total, dim3(1), dim3(kLePickNT), 0, st, w.part_loss,
                     parts, ctl);
  prof_end(st);
  return read_ctl(ctl, hc, st);
}

}  // namespace

void loss_reserve(Arena &a, int32_t n, int32_t k) {
  take_work(a, n, k);
}

int loss_run(const LossArgs &g, LossResult *res, Ctl *ctl, Arena &a,
             hipStream_t st) {
  const int64_t ns = (int64_t)g.n * g.k;
  const LossWork w = take_work(a, g.n, g.k);
  Ctl *hc = pinned_ctl();
  if (!hc) {
    set_error("hipHostMalloc of the control block failed");
    return -5;
  }
  // 16-byte vectors where every row starts at one; lanes a row: the power
  // of two that covers D, from 4 to 64
  const bool vec = g.d % 4 == 0 &&
                   (reinterpret_cast<uintptr_t>(g.emb) & 15) == 0;
  const int32_t lanes = vec ? g.d / 4 : g.d;
  int rc;
#define EZSP_LE(G, V, NV) rc = run_rows<Rows<G, V, NV>>(g, w, ctl, hc, st)
  if (vec) {
    if (lanes <= 4) EZSP_LE(4, 4, 1);
    else if (lanes <= 8) EZSP_LE(8, 4, 1);
    else if (lanes <= 16) EZSP_LE(16, 4, 1);
    else if (lanes <= 32) EZSP_LE(32, 4, 1);
    else if (lanes <= 64) EZSP_LE(64, 4, 1);
    else if (lanes <= 128) EZSP_LE(64, 4, 2);
    else EZSP_LE(64, 4, 4);
  } else {
    if (lanes <= 4) EZSP_LE(4, 1, 1);
    else if (lanes <= 8) EZSP_LE(8, 1, 1);
    else if (lanes <= 16) EZSP_LE(16, 1, 1);
    else if (lanes <= 32) EZSP_LE(32, 1, 1);
    else if (lanes <= 64) EZSP_LE(64, 1, 1);
    else if (lanes <= 128) EZSP_LE(64, 1, 2);
    else if (lanes <= 256) EZSP_LE(64, 1, 4);
    else if (lanes <= 512) EZSP_LE(64, 1, 8);
    else EZSP_LE(64, 1, 16);
  }
#undef EZSP_LE
  if (rc) return rc;
  // algorithmic bytes: every input read once (embeddings, table, words,
  // classes) and every output written once
  prof_bytes("edge_loss",
             4.0 * g.n * g.d + 8.0 * ns + 4.0 * g.n +
                 (g.affinity ? 4.0 * ns : 0.0) + (g.sampled ? 1.0 * ns : 0.0) +
                 (g.grad ? 4.0 * g.n * g.d : 0.0));
  if (hc->err & kErrNonFinite) {
    set_error("non-finite value in emb");
    return -2;
  }
  if (hc->err & kErrBadIndex) {
    set_error("neighbour id outside [-1, n)");
    return -1;
  }
  if (hc->err) {
    set_error("internal check failed in the edge loss (0x%x)", hc->err);
    return -5;
  }
  res->loss = hc->le_loss;
  res->n_edges = (int64_t)hc->le_edges;
  res->n_intra = (int64_t)hc->le_intra;
  res->n_inter = res->n_edges - res->n_intra;
  res->n_intra_kept = (int64_t)hc->le_keep;
  return 0;
}

}  // namespace ezsp
