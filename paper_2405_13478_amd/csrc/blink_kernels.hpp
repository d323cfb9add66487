// HIP kernels of the dirty-imaging path for gfx950.
//
// Per timestep t (shared by all channels):
//   k_sort_one (lists above SORT_ONE: k_sort_run / k_merge / k_sort_finish) -
//       order the usable baselines by u in metres (exact double comparison, ties
//       by baseline index). Because
//       rint(u * s_c) is non-decreasing in u for every s_c > 0, the baselines of
//       one u cell form a contiguous run of this order at EVERY channel, so one
//       sort serves all channels of the timestep.
// Per chunk of images (t, c):
//   k_bounds  - for every signed u cell, the first sorted position at or beyond
//               it (a scan of the sorted u list at this channel's scale).
//   k_grid_cols / k_grid_cols_half - one wavefront per u cell column: gathers the
//               column's baselines (directly and as conjugates of the mirror
//               column), accumulates sums (and counts) in LDS, applies the
//               weighting, then runs the inverse transform along v and writes
//               the rows of the cutout - the grid never reaches HBM on the image
//               path. k_grid_write (and MODE_GRID of k_grid_cols, with a gridding
//               kernel) write the grid itself.
//   k_rows<N> - two image rows per wavefront: Hermitian extension of the half
//               spectrum (u cells 0..N/2-1), inverse transform along u, real
//               part, FFT shift, 1/W and cutout fused into the store.
// The adjoint (differentiation form) runs the same two passes transposed.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "blink_fft.hpp"
#include "twiddles.inc"

namespace blink {

constexpr double C_LIGHT = 299792458.0;   // m/s
constexpr unsigned long long KEY_MAX = ~0ull;

enum { MODE_IMAGE = 0, MODE_GRID = 1 };
enum { VT_C64 = 0, VT_F16 = 1, VT_BF16 = 2 };

// Cells per metre at frequency f: (f * (N dx)) / c, IEEE double, this order.
__device__ __forceinline__ double cells_per_metre(double f, double ndx) {
  const double p = f * ndx;
  return p / C_LIGHT;
}

// Order-preserving map of a double to an unsigned 64-bit key.
__device__ __forceinline__ unsigned long long order_key(double u) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(u);
  return (b >> 63) ? ~b : (b | (1ull << 63));
}

// The double that order_key maps to a key.
__device__ __forceinline__ double key_value(unsigned long long k) {
  return __longlong_as_double((long long)((k >> 63) ? k & ~(1ull << 63) : ~k));
}

// ============================================================== sort by u
struct SortArgs {
  int T, B;
  int t0;                        // first timestep of this launch (grid.y covers t0 + blockIdx.y)
  const double* uvw;             // [T][B][3]
  const uint8_t* flags;          // [T][B] or null
  unsigned long long* key[2];    // [T][B] ping-pong
  int* idx[2];                   // [T][B]
  int* n_unflagged;              // [T]
  int* n_valid;                  // [T]
  double* su;                    // [T][B] sorted u
  double* sv;                    // [T][B] v in the same order
  int* perm;                     // [T][B] baseline index in the same order
  double* sd;                    // [T][B] delay in the same order, or null (no rotation)
  double pl, pm, pn1;            // phase centre l0, m0 and n0 - 1
  int proj;                      // 1: grid the baselines re-projected onto the new centre's plane
  double eu[3], ev[3];           // with proj: u' = eu . (u, v, w), v' = ev . (u, v, w)
  const double* cable;           // [A] electrical cable lengths (m) or null
  const int* ant1;               // [B] (with cable lengths)
  const int* ant2;               // [B]
  int n_ant;                     // cable length entries; an antenna index outside [0, n_ant) adds 0
  double* vmax;                  // [T] largest |v| of the usable baselines, or null
  // single-image bounds (one channel per timestep): the cell bounds of image t
  // are formed by the sort kernel itself (see k_sort_one)
  int N, kw;                     // grid size, gridding kernel support (0: nearest cell)
  double ndx;                    // fl(N * dx)
  const double* freq;            // [1]
  int* bnd;                      // [T][N + 2]
  int* ncz;                      // [T]
};

// The (u, v) in metres that the imager grids for baseline o of the flat
// [T][B] layout: the baseline's own, or its components along the new
// centre's tangent-plane axes when re-projecting.
__device__ __forceinline__ void plane_uv(const SortArgs& a, size_t o, double& u, double& v) {
  const double* b = a.uvw + o * 3;
  if (a.proj) {
    // written out, so that every caller has the same bits (the sort forms u again)
    u = fma(a.eu[2], b[2], fma(a.eu[0], b[0], a.eu[1] * b[1]));
    v = fma(a.ev[2], b[2], fma(a.ev[0], b[0], a.ev[1] * b[1]));
  } else {
    u = b[0];
    v = b[1];
  }
}

// u l0 + v m0 + w (n0 - 1): the path difference (metres) between the new
// phase centre and zenith for baseline uvw.
__device__ __forceinline__ double geo_delay(const double* uvw, double l0, double m0, double n1) {
  return uvw[0] * l0 + uvw[1] * m0 + uvw[2] * n1;
}

// The delay of baseline b (metres): the geometric term plus, with cable
// lengths, l_ant1 - l_ant2 (a longer path delays that antenna's voltage).
// An antenna index outside [0, n_ant) contributes no cable term, as it
// contributes a zero gain on the gains path.
__device__ __forceinline__ double cable_len(const SortArgs& a, int i) {
  return (unsigned)i < (unsigned)a.n_ant ? a.cable[i] : 0.0;
}
__device__ __forceinline__ double baseline_delay(const SortArgs& a, size_t tb, int b) {
  double d = geo_delay(a.uvw + (tb + b) * 3, a.pl, a.pm, a.pn1);
  if (a.cable != nullptr) d += cable_len(a, a.ant1[b]) - cable_len(a, a.ant2[b]);
  return d;
}

__global__ void k_sort_init(int* a, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

// Bitonic sort of one run of RUN (key, index) pairs in LDS; the pair order is
// total because indices are distinct, so the result equals a stable sort.
template <int RUN>
__global__ void __launch_bounds__(1024) k_sort_run(SortArgs a) {
  __shared__ unsigned long long sk[RUN];
  __shared__ int si[RUN];
  __shared__ int s_unf;
  const int t = a.t0 + blockIdx.y;
  const int base = blockIdx.x * RUN;
  const int len = min(RUN, a.B - base);
  if (threadIdx.x == 0) s_unf = 0;
  __syncthreads();
  int unf = 0;
  for (int i = threadIdx.x; i < RUN; i += blockDim.x) {
    unsigned long long k = KEY_MAX;
    int id = 0x7fffffff;
    if (i < len) {
      const int b = base + i;
      const size_t o = (size_t)t * a.B + b;
      double u, v;
      plane_uv(a, o, u, v);
      const bool flagged = a.flags != nullptr && a.flags[o] != 0;
      unf += flagged ? 0 : 1;
      if (!flagged && isfinite(u) && isfinite(v)) k = order_key(u);
      id = b;
    }
    sk[i] = k;
    si[i] = id;
  }
  if (unf) atomicAdd(&s_unf, unf);
  __syncthreads();
  for (int k = 2; k <= RUN; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < RUN / 2; i += blockDim.x) {
        const int lo = 2 * i - (i & (j - 1));
        const int hi = lo + j;
        const bool up = (lo & k) == 0;
        const unsigned long long ka = sk[lo], kb = sk[hi];
        const int ia = si[lo], ib = si[hi];
        const bool gt = ka > kb || (ka == kb && ia > ib);
        if (gt == up) {
          sk[lo] = kb; sk[hi] = ka;
          si[lo] = ib; si[hi] = ia;
        }
      }
      __syncthreads();
    }
  }
  for (int i = threadIdx.x; i < len; i += blockDim.x) {
    const size_t o = (size_t)t * a.B + base + i;
    a.key[0][o] = sk[i];
    a.idx[0][o] = si[i];
  }
  if (threadIdx.x == 0 && s_unf) atomicAdd(&a.n_unflagged[t], s_unf);
}

// Half-spectrum columns that may hold data, given the clamped u cells of the
// first and the last of nv sorted entries: every entry lies in a column
// |c| <= max(|first|, |last|), and a gridding kernel reaches columns c with
// |c - x_u| <= W/2, i.e. at most floor(W/2 + 1/2) columns beyond the entry's
// nearest one.
__device__ __forceinline__ int nonempty_columns(int cfirst, int clast, int nv, int N, int kw) {
  const int reach = kw > 0 ? (kw + 1) / 2 : 0;
  return nv == 0 ? 0 : min(N / 2, max(clast, -cfirst) + 1 + reach);
}

// ------------------------------------------------ order of one timestep in one launch
// The order of up to SORT_ONE baselines of a timestep, (key, index) ascending
// with the key order_key(u), by one bucket pass instead of a comparison network
// (91 passes with a barrier each for 8,192 keys):
//   1. every thread loads its PER baselines (u, v, flag); a block reduction
//      finds the range of the usable u, their number and the largest |v|;
//   2. u is mapped linearly onto nb buckets. Subtraction, product and
//      truncation never decrease with u, so the buckets are in order of u.
//      Their counts are LDS integer atomics (two 16-bit counts a word), and up to
//      8 baselines a thread keep the count returned as their slot in the bucket;
//   3. a scan turns the counts into each bucket's first sorted position (with 32
//      baselines a thread, its end). Where a bucket has more than SORT_UNEVEN
//      entries (a long baseline beside a dense core, a regular array whose
//      baselines share a few u), 2 and 3 are done again with buckets between
//      THREADS samples of the list, sorted as (key, index) pairs, so that they
//      divide equal u too;
//   4. the keys and indices go to their buckets in LDS, with 32 baselines a
//      thread each bucket from its end down, which leaves its start in the table;
//   5. an entry's position is its bucket's start plus the number of smaller
//      (key, index) pairs in the bucket (about one entry a bucket when u is
//      spread evenly; a centrally condensed array fills some with ten). Buckets
//      above SORT_LIGHT entries are sorted in place by a wavefront each, or by
//      the whole workgroup;
//   6. u, v, index and delay are written in order (index_only: the index
//      alone, see k_sort_gather).
// Where all usable u are equal (a linear array), the order is that of the indices.
// The positions are taken in `shares` parts, whole buckets each: as many as
// fit in LDS, walked by one workgroup per timestep, or by gridDim.x of them
// that each repeat 1-3.
// A share that does not fit in LDS even so (the samples missed where most of a
// long list lies) is ordered by a stable radix sort of the keys instead, four
// bits a pass, skipping digits that all keys share.
// What bounds it: the latency of one workgroup (loads, barriers, LDS atomics),
// not bandwidth; with many long lists the reads of uvw. With 32 baselines a
// thread only their buckets are kept between the steps, two a register (those
// between samples wait in idx[0], which every workgroup of a timestep fills alike):
// with the slots, 45 registers spilled to memory.
// Measured against the networks and merges before it (order, largest |v|, bounds),
// us for one timestep and for 200: 1,000 baselines 30 -> 14 and 32 -> 15; 8,128
// baselines 131 -> 20 and 152 -> 46; 32,640 baselines 188 -> 50 and 877 -> 207. With
// one far baseline, where linear buckets alone took 144 and 169 for 8,128 baselines
// and 481 and 1,718 for 32,640: 51, 92, 162 and 501. At 51 different u: 52, 105, 183
// and 667 (linear buckets alone 52, 140, 191 and 1,584).
constexpr int SORT_ONE = 32768;          // largest list of this kernel (16-bit positions)
constexpr int SORT_LIGHT = 128;          // larger buckets are sorted, not ranked by counting
constexpr int SORT_UNEVEN = 256;         // a larger bucket asks for sampled ones
constexpr int SORT_WAVE_MAX = 2048;      // larger ones are sorted by the whole workgroup
constexpr int SORT_SHARE = 10752;        // entries of a share that fit in LDS beside the bucket ends
constexpr int SORT_SHARES = 8;           // parts of a list
constexpr int SORT_RADIX = 16;           // digits of the radix passes

// Workgroup shapes: lists of up to 1,024 baselines take 256 threads (eight such
// workgroups share a CU), longer ones 1,024.
template <int THREADS>
struct SortWg {
  // buckets for a list of n baselines: about one a baseline, from two a thread on
  __host__ __device__ static constexpr int buckets(int n) {
    int nb = 2 * THREADS;
    while (nb < n && nb < 16384) nb *= 2;
    return nb;
  }
  __host__ __device__ static constexpr int share(int n) { return n < SORT_SHARE ? n : SORT_SHARE; }
  // keys, indices and order of a share; or permutation and digit counts of the radix passes
  __host__ __device__ static constexpr size_t list_bytes(int n) {
    const size_t list = (size_t)((share(n) + 7) & ~7) * 12;
    const size_t radix = (size_t)((n + 7) & ~7) * 2 + (size_t)SORT_RADIX * THREADS * 2;
    return n > SORT_SHARE && radix > list ? radix : list;
  }
  // starts or ends of the buckets (one more than buckets), and beside those of 2 THREADS buckets the samples
  static constexpr int SAMPLES_AT = THREADS + 4;                     // in words
  __host__ __device__ static constexpr size_t table_bytes(int n) {
    const size_t linear = (size_t)(buckets(n) / 2 + 1) * 4, sampled = (size_t)SAMPLES_AT * 4 + (size_t)THREADS * 10;
    return linear > sampled ? linear : sampled;
  }
  __host__ __device__ static constexpr size_t lds_bytes(int n) { return list_bytes(n) + table_bytes(n); }
};

// Exclusive scan of one value per thread over the workgroup; `tot` is one word
// a wavefront that nothing else uses between the barriers.
template <int THREADS>
__device__ __forceinline__ unsigned block_exclusive(unsigned v, unsigned* tot) {
  const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
  unsigned s = v;
  for (int o = 1; o < WAVE; o <<= 1) {
    const unsigned x = __shfl_up(s, o);
    if (lane >= o) s += x;
  }
  if (lane == WAVE - 1) tot[wave] = s;
  __syncthreads();
  unsigned base = 0;
#pragma unroll
  for (int w = 0; w < THREADS / WAVE; ++w) base += w < wave ? tot[w] : 0u;
  return base + s - v;
}

// The key of baseline i: usable ones by u, flagged and non-finite ones last.
__device__ __forceinline__ unsigned long long baseline_key(const SortArgs& a, size_t tb, int i) {
  double u, v;
  plane_uv(a, tb + i, u, v);
  const bool flagged = a.flags != nullptr && a.flags[tb + i] != 0;
  return !flagged && isfinite(u) && isfinite(v) ? order_key(u) : KEY_MAX;
}

// In-place sort of n (key, index) pairs in LDS by `width` threads (rank r of
// them): a bitonic network whose comparators all point the same way (each
// merge starts by comparing mirrored positions), so that it ends at any n.
template <class Sync>
__device__ __forceinline__ void sort_pairs(unsigned long long* key, unsigned short* id, int n, int r, int width,
                                           Sync&& sync) {
  auto exchange = [&](int x, int y) {
    if (y >= n) return;
    const unsigned long long kx = key[x], ky = key[y];
    const unsigned short ix = id[x], iy = id[y];
    if (kx > ky || (kx == ky && ix > iy)) {
      key[x] = ky; key[y] = kx;
      id[x] = iy; id[y] = ix;
    }
  };
  for (int k = 2; k / 2 < n; k <<= 1) {
    for (int p = r; p < (n + k - 1) / k * (k / 2); p += width) {
      const int base = p / (k / 2) * k, q = p % (k / 2);
      exchange(base + q, base + k - 1 - q);
    }
    sync();
    for (int j = k >> 2; j > 0; j >>= 1) {
      for (int p = r; p < (n + 2 * j - 1) / (2 * j) * j; p += width) {
        const int x = 2 * p - (p & (j - 1));
        exchange(x, x + j);
      }
      sync();
    }
  }
}

// Stable radix order of all B keys of the timestep into perm (16-bit indices,
// LDS); cnt: SORT_RADIX x THREADS 16-bit counts (LDS). Thread t owns the
// positions [t per, (t + 1) per), so counts in thread order keep it stable.
template <int THREADS, int PER>
__device__ __forceinline__ void radix_order(const SortArgs& a, size_t tb, unsigned short* perm, unsigned short* cnt,
                                            unsigned* tot, unsigned long long* s_diff) {
  const int tid = threadIdx.x, B = a.B;
  const int per = (B + THREADS - 1) / THREADS;                       // <= PER
  __syncthreads();
  if (tid == 0) *s_diff = 0ull;
  __syncthreads();
  const unsigned long long k0 = baseline_key(a, tb, 0);
  unsigned long long diff = 0ull;
  for (int i = tid; i < B; i += THREADS) {
    diff |= baseline_key(a, tb, i) ^ k0;
    perm[i] = (unsigned short)i;
  }
  for (int o = WAVE / 2; o > 0; o >>= 1) diff |= __shfl_xor(diff, o);
  if (tid % WAVE == 0 && diff != 0ull) atomicOr(s_diff, diff);
  __syncthreads();
  diff = *s_diff;
  for (int sh = 0; sh < 64; sh += 4) {
    if (((diff >> sh) & (SORT_RADIX - 1)) == 0ull) continue;         // one digit for all: no change
    for (int d = 0; d < SORT_RADIX; ++d) cnt[d * THREADS + tid] = 0;
    unsigned id[PER / 2];                                            // two indices a word
    auto digit_of = [&](int i) { return (int)((baseline_key(a, tb, i) >> sh) & (SORT_RADIX - 1)); };
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = tid * per + k;
      int i = 0;
      if (k < per && j < B) {
        i = perm[j];
        ++cnt[digit_of(i) * THREADS + tid];
      }
      if (k % 2 == 0) id[k / 2] = (unsigned)i;
      else id[k / 2] |= (unsigned)i << 16;
      __builtin_amdgcn_sched_barrier(0);                             // bounds the loads in flight
    }
    __syncthreads();
    // exclusive scan in (digit, thread) order: SORT_RADIX consecutive counts a thread
    unsigned sum = 0;
    for (int e = 0; e < SORT_RADIX; ++e) sum += cnt[tid * SORT_RADIX + e];
    unsigned at = block_exclusive<THREADS>(sum, tot);
    for (int e = 0; e < SORT_RADIX; ++e) {
      const unsigned c = cnt[tid * SORT_RADIX + e];
      cnt[tid * SORT_RADIX + e] = (unsigned short)at;
      at += c;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int j = tid * per + k;
      const int i = (int)((id[k / 2] >> (k % 2 * 16)) & 0xffffu);
      if (k < per && j < B) perm[cnt[digit_of(i) * THREADS + tid]++] = (unsigned short)i;
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  }
}

// THREADS (key, index) pairs, one a thread, in ascending order into key, id (LDS):
// a bitonic network, by shuffles where the partner is in the wavefront.
template <int THREADS>
__device__ __forceinline__ void sort_samples(unsigned long long k, int i, unsigned long long* key, unsigned short* id) {
  const int tid = threadIdx.x;
#pragma unroll 1
  for (int run = 2; run <= THREADS; run *= 2) {
#pragma unroll 1
    for (int d = run / 2; d > 0; d /= 2) {
      unsigned long long ko;
      int io;
      if (d < WAVE) {
        ko = __shfl_xor(k, d);
        io = __shfl_xor(i, d);
      } else {
        key[tid] = k;
        id[tid] = (unsigned short)i;
        __syncthreads();
        ko = key[tid ^ d];
        io = id[tid ^ d];
        __syncthreads();
      }
      const bool less = ko < k || (ko == k && io < i);
      const bool low = ((tid & run) == 0) == ((tid & d) == 0);        // keeps the smaller of the two
      if (less == low) { k = ko; i = io; }
    }
  }
  key[tid] = k;
  id[tid] = (unsigned short)i;
  __syncthreads();
}

template <int THREADS, int PER, bool BOUNDS>
__global__ void __launch_bounds__(THREADS) k_sort_one(SortArgs a, int shares, int index_only) {
  static_assert(PER <= 32, "one bit a baseline in okm");
  using W_ = SortWg<THREADS>;
  constexpr int WAVES = THREADS / WAVE;
  constexpr int MAX_HEAVY = SORT_SHARE / SORT_LIGHT + 1;
  extern __shared__ float4 lds_raw[];
  __shared__ unsigned long long s_key[2][WAVES];
  __shared__ double s_vm[WAVES];
  __shared__ int s_cnt[2][WAVES];
  __shared__ unsigned s_tot[WAVES];
  // per share: the positions [p0, p1) it writes, the start ps of the bucket before
  // p0, that bucket b0 and the last one b1
  __shared__ int s_p0[SORT_SHARES], s_p1[SORT_SHARES], s_ps[SORT_SHARES], s_b0[SORT_SHARES], s_b1[SORT_SHARES];
  __shared__ int s_heavy;
  __shared__ unsigned s_big;
  __shared__ unsigned s_list[MAX_HEAVY];             // heavy buckets: start << 16 | size
  __shared__ unsigned long long s_diff;
  const int t = a.t0 + blockIdx.y, g = blockIdx.x, G = gridDim.x;
  const int tid = threadIdx.x, lane = tid % WAVE, wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int B = a.B;
  const size_t tb = (size_t)t * B;
  const int cap = (W_::share(B) + 7) & ~7;
  unsigned long long* keys = reinterpret_cast<unsigned long long*>(lds_raw);
  unsigned short* ids = reinterpret_cast<unsigned short*>(keys + cap);
  unsigned short* ord = ids + cap;
  unsigned* table = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(lds_raw) + W_::list_bytes(B));
  unsigned long long* skey = reinterpret_cast<unsigned long long*>(table + W_::SAMPLES_AT);
  unsigned short* sid = reinterpret_cast<unsigned short*>(skey + THREADS);
  int nb = W_::buckets(B);

  // 1. load and reduce. Up to 8 baselines a thread keep their u in registers; of
  // 32, u is read again: from uvw, or (index_only, where su is not yet written)
  // from a packed copy in su.
  constexpr bool KEEP = PER <= 8;
  constexpr int BATCH = PER < 8 ? PER : 8;                            // baselines at once
  // the thread's number, opaque: what follows from it is formed where it is used
  // (kept across the steps, baseline numbers and addresses spill)
  auto thread = [&]() -> int {
    int i = tid;
    asm volatile("" : "+v"(i));
    return i;
  };
  double u[KEEP ? PER : 1];
  unsigned bs[KEEP ? PER : PER / 2];                                 // bucket and slot << 16, or two buckets
  unsigned okm = 0;
  unsigned long long kmin = KEY_MAX, kmax = 0ull;                    // keys, which tell 0 from -0
  double vm = 0.0;
  int unf = 0;
#pragma unroll 1
  for (int k0 = 0; k0 < PER; k0 += BATCH) {
#pragma unroll
    for (int e = 0; e < BATCH; ++e) {
      const int i = (k0 + e) * THREADS + thread();
      double uk = 0.0;
      if (i < B) {
        double v;
        plane_uv(a, tb + i, uk, v);
        const bool flagged = a.flags != nullptr && a.flags[tb + i] != 0;
        unf += flagged ? 0 : 1;
        if (!flagged && isfinite(uk) && isfinite(v)) {
          okm |= 1u << (k0 + e);
          const unsigned long long k = order_key(uk);
          kmin = min(kmin, k);
          kmax = max(kmax, k);
          vm = fmax(vm, fabs(v));
        }
        if (!KEEP && index_only) a.su[tb + i] = uk;
      }
      if constexpr (KEEP) u[e] = uk;
    }
  }
  auto u_of = [&](int k0, int e) -> double {                         // u of the thread's baseline k0 + e
    if constexpr (KEEP) return u[e];
    const int i = (k0 + e) * THREADS + thread();
    double uk = 0.0, vk;
    if (i < B) {
      if (index_only) uk = a.su[tb + i];
      else plane_uv(a, tb + i, uk, vk);
    }
    return uk;
  };
  for (int w = tid; w <= nb / 2; w += THREADS) table[w] = 0u;
  int val = __popc(okm);
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    kmin = min(kmin, __shfl_xor(kmin, o));
    kmax = max(kmax, __shfl_xor(kmax, o));
    vm = fmax(vm, __shfl_xor(vm, o));
    unf += __shfl_xor(unf, o);
    val += __shfl_xor(val, o);
  }
  if (lane == 0) {
    s_key[0][wave] = kmin; s_key[1][wave] = kmax; s_vm[wave] = vm;
    s_cnt[0][wave] = unf; s_cnt[1][wave] = val;
  }
  if (tid == 0) s_big = 0u;
  __syncthreads();
  {
    const int w = lane % WAVES;
    kmin = s_key[0][w]; kmax = s_key[1][w]; vm = s_vm[w];
    unf = s_cnt[0][w]; val = s_cnt[1][w];
    for (int o = WAVES / 2; o > 0; o >>= 1) {
      kmin = min(kmin, __shfl_xor(kmin, o));
      kmax = max(kmax, __shfl_xor(kmax, o));
      vm = fmax(vm, __shfl_xor(vm, o));
      unf += __shfl_xor(unf, o);
      val += __shfl_xor(val, o);
    }
  }
  // (the same in every lane: scalar registers)
  auto scalar = [](unsigned long long v) {
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return ((unsigned long long)hi << 32) | (unsigned)__builtin_amdgcn_readfirstlane((unsigned)v);
  };
  kmin = scalar(kmin);
  kmax = scalar(kmax);
  const double umin = key_value(kmin), umax = key_value(kmax);       // (of no use when nothing is usable)
  const int nv = __builtin_amdgcn_readfirstlane(val);
  if (g == 0 && tid == 0) {
    a.n_unflagged[t] = unf;
    a.n_valid[t] = nv;
    if (a.vmax != nullptr) a.vmax[t] = vm;
  }

  // 2. buckets (a degenerate range puts all into one)
  double scale = (double)nb / (umax - umin);
  if (!(umax > umin) || !isfinite(scale)) scale = 0.0;
  scale = __longlong_as_double((long long)scalar((unsigned long long)__double_as_longlong(scale)));
  auto linear = [&](double x) -> unsigned {                          // (unusable ones: any bucket)
    return (unsigned)fmin(fmax((x - umin) * scale, 0.0), (double)(nb - 1));
  };
  // with samples: how many of samples 1 .. THREADS - 1 are not above (u, index), of
  // the thread's baselines i0, i0 + THREADS, ..
  auto between = [&](const double (&x)[BATCH], int i0, unsigned (&b)[BATCH]) {
    constexpr int U = BATCH < 4 ? BATCH : 4;                         // searches at once
#pragma unroll
    for (int q = 0; q < BATCH; q += U) {
      unsigned long long k[U];
      unsigned bq[U];
#pragma unroll
      for (int e = 0; e < U; ++e) { k[e] = order_key(x[q + e]); bq[e] = 0u; }
#pragma unroll 1
      for (int h = THREADS / 2; h > 0; h /= 2) {
        unsigned long long ks[U];
#pragma unroll
        for (int e = 0; e < U; ++e) ks[e] = skey[bq[e] + h];
#pragma unroll
        for (int e = 0; e < U; ++e) {
          int up = ks[e] < k[e] ? h : 0;
          if (ks[e] == k[e]) up = (int)sid[bq[e] + h] <= i0 + (q + e) * THREADS ? h : 0;
          bq[e] += up;
        }
      }
#pragma unroll
      for (int e = 0; e < U; ++e) b[q + e] = bq[e];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto entry_of = [&](unsigned b) -> int { return (int)((table[b >> 1] >> ((b & 1u) * 16u)) & 0xffffu); };
  auto count = [&](auto sampled_c) {
    constexpr bool SAMPLED = decltype(sampled_c)::value != 0;
    auto batch = [&](int k0, auto&& put) {
      const int i0 = k0 * THREADS + thread();
      double uk[BATCH];
      unsigned b[BATCH], old[BATCH];
#pragma unroll
      for (int e = 0; e < BATCH; ++e) uk[e] = u_of(k0, e);
      if constexpr (SAMPLED) {
        between(uk, i0, b);
      } else {
#pragma unroll
        for (int e = 0; e < BATCH; ++e) b[e] = linear(uk[e]);
      }
#pragma unroll
      for (int e = 0; e < BATCH; ++e) {
        old[e] = 0u;
        if ((okm >> (k0 + e)) & 1u) {
          if constexpr (KEEP) old[e] = atomicAdd(&table[b[e] >> 1], 1u << ((b[e] & 1u) * 16u));
          else atomicAdd(&table[b[e] >> 1], 1u << ((b[e] & 1u) * 16u));
        }
      }
      put(i0, b, old);
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (KEEP) {
      batch(0, [&](int, const unsigned (&b)[BATCH], const unsigned (&old)[BATCH]) {
#pragma unroll
        for (int e = 0; e < BATCH; ++e) bs[e] = b[e] | (((old[e] >> ((b[e] & 1u) * 16u)) & 0xffffu) << 16);
      });
    } else if constexpr (SAMPLED) {
#pragma unroll 1
      for (int k0 = 0; k0 < PER; k0 += BATCH)
        batch(k0, [&](int i0, const unsigned (&b)[BATCH], const unsigned (&)[BATCH]) {
#pragma unroll
          for (int e = 0; e < BATCH; ++e)
            if ((okm >> (k0 + e)) & 1u) a.idx[0][tb + i0 + e * THREADS] = (int)b[e];
        });
    } else {
#pragma unroll
      for (int k0 = 0; k0 < PER; k0 += BATCH)
        batch(k0, [&](int, const unsigned (&b)[BATCH], const unsigned (&)[BATCH]) {
#pragma unroll
          for (int e = 0; e < BATCH; e += 2) bs[(k0 + e) / 2] = b[e] | (b[e + 1] << 16);
        });
    }
    __syncthreads();
  };
  // 3. starts or ends, in place, and the largest bucket
  auto scan = [&]() {
    const int wpt = nb / 2 / THREADS;                                // words of two counts a thread
    unsigned c[8], sum = 0, big = 0;                                 // counts of up to 16 buckets
    static_assert(W_::buckets(SORT_ONE) / 2 / THREADS <= 8 || THREADS < 1024, "words of counts a thread");
    if (wpt % 4 == 0) {                                              // 16 bytes a lane: few bank conflicts
#pragma unroll
      for (int w = 0; w < 8; w += 4)
        if (w < wpt) *reinterpret_cast<uint4*>(c + w) = *reinterpret_cast<const uint4*>(table + tid * wpt + w);
    } else {
      c[0] = table[tid * wpt];
      c[1] = wpt > 1 ? table[tid * wpt + 1] : 0u;
    }
#pragma unroll
    for (int w = 0; w < 8; ++w)
      if (w < wpt) {
        sum += (c[w] & 0xffffu) + (c[w] >> 16);
        big = max(big, max(c[w] & 0xffffu, c[w] >> 16));
      }
    for (int o = WAVE / 2; o > 0; o >>= 1) big = max(big, __shfl_xor(big, o));
    if (lane == 0) atomicMax(&s_big, big);
    unsigned at = block_exclusive<THREADS>(sum, s_tot);
#pragma unroll
    for (int w = 0; w < 8; ++w)
      if (w < wpt) {
        const unsigned e0 = at + (c[w] & 0xffffu), e1 = e0 + (c[w] >> 16);
        c[w] = KEEP ? at | (e0 << 16) : e0 | (e1 << 16);
        at = e1;
      }
    if (wpt % 4 == 0) {
#pragma unroll
      for (int w = 0; w < 8; w += 4)
        if (w < wpt) *reinterpret_cast<uint4*>(table + tid * wpt + w) = *reinterpret_cast<const uint4*>(c + w);
    } else {
      table[tid * wpt] = c[0];
      if (wpt > 1) table[tid * wpt + 1] = c[1];
    }
    if (tid == THREADS - 1) table[nb / 2] = at;                      // (after the last bucket: nv)
    __syncthreads();
  };
  const bool equal = kmin == kmax;                                   // all usable u: the order is that of the indices
  bool sampled = false;
  if (__builtin_expect(!equal, 1)) {
    count(ic<0>{});
    scan();
    if (__builtin_expect(s_big > (unsigned)SORT_UNEVEN, 0)) {
      const int i = (int)((unsigned)(tid * B) / (unsigned)THREADS);
      __syncthreads();                                               // (s_big is read)
      sort_samples<THREADS>(baseline_key(a, tb, i), i, skey, sid);
      nb = 2 * THREADS;
      sampled = true;
      if (tid == 0) s_big = 0u;
      for (int w = tid; w <= nb / 2; w += THREADS) table[w] = 0u;
      __syncthreads();
      count(ic<1>{});
      scan();
    }
  }

  // 6. the entries at sorted positions [p0, p1), index_at(j) the baseline at
  // position j (p0 - 1 too, for the bounds)
  const double s = BOUNDS ? cells_per_metre(a.freq[0], a.ndx) : 0.0;
  const int H = a.N / 2;
  auto cell = [&](double x) -> int { return (int)fmin(fmax(rint(x * s), (double)-H), (double)H); };
  int* bnd = BOUNDS ? a.bnd + (size_t)t * (a.N + 2) : nullptr;
  auto write = [&](int p0, int p1, auto&& index_at) {
    constexpr int U = 4;                                             // gathers in flight
    for (int j0 = p0; j0 < p1; j0 += U * THREADS) {
      int bi[U];
      double uj[U], vj[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int j = j0 + k * THREADS + tid;
        bi[k] = j < p1 ? index_at(j) : 0;
        uj[k] = vj[k] = 0.0;
        if (j < p1 && !index_only) plane_uv(a, tb + bi[k], uj[k], vj[k]);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int j = j0 + k * THREADS + tid;
        if (j < p1) {
          a.perm[tb + j] = bi[k];
          if (!index_only) {
            a.su[tb + j] = uj[k];
            a.sv[tb + j] = vj[k];
            if (a.sd != nullptr) a.sd[tb + j] = baseline_delay(a, tb, bi[k]);
          }
        }
        if constexpr (BOUNDS) {
          // first sorted position of the cells between the entry before and this one
          const int cj = cell(uj[k]);
          int cp = __shfl_up(cj, 1);
          if (j < p1 && j > 0) {
            if (lane == 0) {
              double ul, vl;
              plane_uv(a, tb + index_at(j - 1), ul, vl);
              cp = cell(ul);
            }
            for (int c = cp + 1; c <= cj; ++c) bnd[c + H] = j;
          }
        }
      }
    }
    if constexpr (BOUNDS) {
      // cells up to the first entry's, and beyond the last one's
      if (p0 == 0 && p1 > 0)
        for (int c = tid - H; c <= cell(umin); c += THREADS) bnd[c + H] = 0;
      if (p1 == nv && p1 > p0)
        for (int c = cell(umax) + 1 + tid; c <= H + 1; c += THREADS) bnd[c + H] = nv;
    }
  };
  if constexpr (BOUNDS) {
    if (g == 0) {
      if (tid == 0) a.ncz[t] = nonempty_columns(nv == 0 ? 0 : cell(umin), nv == 0 ? 0 : cell(umax), nv, a.N, a.kw);
      if (nv == 0)
        for (int c = tid - H; c <= H + 1; c += THREADS) bnd[c + H] = 0;
    }
  }

  if (__builtin_expect(equal, 0)) {
    unsigned short* perm = reinterpret_cast<unsigned short*>(lds_raw);
    int* base = reinterpret_cast<int*>(table);                       // usable ones before each 64 baselines
    static_assert(PER * WAVES <= THREADS, "one count a thread");
    auto ballot_of = [&](int k) { return __ballot((okm >> k) & 1u); };
    for (int k = 0; k < PER; ++k) {
      const unsigned long long usable = ballot_of(k);
      if (lane == 0) base[k * WAVES + wave] = __popcll(usable);
    }
    __syncthreads();
    const unsigned n = tid < PER * WAVES ? (unsigned)base[tid] : 0u;
    const unsigned before = block_exclusive<THREADS>(n, s_tot);
    if (tid < PER * WAVES) base[tid] = (int)before;
    __syncthreads();
    for (int k = 0; k < PER; ++k) {
      const unsigned long long usable = ballot_of(k);
      const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(usable >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)usable, 0u));
      if ((okm >> k) & 1u) perm[base[k * WAVES + wave] + below] = (unsigned short)(k * THREADS + tid);
    }
    __syncthreads();
    write((int)((unsigned)(nv * g) / (unsigned)G), (int)((unsigned)(nv * (g + 1)) / (unsigned)G), [&](int j) { return (int)perm[j]; });
    return;
  }
  if constexpr (!KEEP) {
    if (B > SORT_SHARE && (nv + shares - 1) / shares + 2 * (int)s_big > cap) {
      unsigned short* perm = reinterpret_cast<unsigned short*>(lds_raw);
      radix_order<THREADS, PER>(a, tb, perm, perm + ((B + 7) & ~7), s_tot, &s_diff);
      write((int)((unsigned)(nv * g) / (unsigned)G), (int)((unsigned)(nv * (g + 1)) / (unsigned)G), [&](int j) { return (int)perm[j]; });
      return;
    }
  }
  static_assert(!KEEP || PER * THREADS <= SORT_SHARE, "a short list is one share's worth of LDS");
  // the shares: the buckets after the one that holds position lo - 1, up to the
  // one that holds hi - 1. The bucket before it (from ps) is kept too, as the
  // bounds look at the entry before p0: at most a share and two buckets.
  auto lo_of = [&](int sh) { return (int)((unsigned)(nv * sh) / (unsigned)shares); };   // (below 2^19)
  if (tid < shares) {                                // (what no bucket below writes)
    if (lo_of(tid) == 0) s_p0[tid] = s_ps[tid] = s_b0[tid] = 0;
    if (lo_of(tid + 1) == 0) s_p1[tid] = s_b1[tid] = 0;
  }
  if (tid == 0) s_heavy = 0;
  for (int sh = g; sh < shares; sh += G) {
    const int lo = lo_of(sh), hi = lo_of(sh + 1);
    for (int w = tid; w < nb / 2; w += THREADS) {
      const unsigned h = table[w];
      const int lo16 = (int)(h & 0xffffu), hi16 = (int)(h >> 16);
      const int other = KEEP ? (int)(table[w + 1] & 0xffffu) : w > 0 ? (int)(table[w - 1] >> 16) : 0;
      const int at[3] = {KEEP ? lo16 : other, KEEP ? hi16 : lo16, KEEP ? other : hi16};
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (at[e] < lo && lo <= at[e + 1]) { s_ps[sh] = at[e]; s_p0[sh] = at[e + 1]; s_b0[sh] = 2 * w + e; }
        if (at[e] < hi && hi <= at[e + 1]) { s_p1[sh] = at[e + 1]; s_b1[sh] = 2 * w + e; }
      }
    }
  }
  __syncthreads();
  for (int sh = g; sh < shares; sh += G) {
    const int p0 = s_p0[sh], p1 = s_p1[sh], ps = s_ps[sh];
    const unsigned b0 = s_b0[sh], b1 = s_b1[sh];
    if (p1 <= p0) continue;
    if (sh != g) {
      __syncthreads();                               // the last share is written
      if (tid == 0) s_heavy = 0;
      if (!KEEP && tid == 0 && p0 > 0) {             // the bucket before p0 may have been in it
        const unsigned h = (b0 & 1u) * 16u;
        table[b0 >> 1] = (table[b0 >> 1] & ~(0xffffu << h)) | ((unsigned)p0 << h);
      }
      __syncthreads();
    }
    // 4. keys and indices to their buckets
    if constexpr (!KEEP) {
      if (__builtin_expect(sampled, 0)) {                            // (a thread's own stores)
#pragma unroll
        for (int k = 0; k < PER; k += 2) {
          const int i0 = k * THREADS + thread();
          const unsigned b0k = (okm >> k) & 1u ? (unsigned)a.idx[0][tb + i0] : 0u;
          const unsigned b1k = (okm >> (k + 1)) & 1u ? (unsigned)a.idx[0][tb + i0 + THREADS] : 0u;
          bs[k / 2] = b0k | (b1k << 16);
        }
      }
    }
#pragma unroll
    for (int k0 = 0; k0 < PER; k0 += BATCH) {
      const int i0 = k0 * THREADS + thread();
      double uk[BATCH];
      unsigned b[BATCH];
      int at[BATCH];
#pragma unroll
      for (int e = 0; e < BATCH; ++e) {
        if constexpr (KEEP) b[e] = bs[e] & 0xffffu;
        else b[e] = (bs[(k0 + e) / 2] >> (e % 2 * 16)) & 0xffffu;
      }
#pragma unroll
      for (int e = 0; e < BATCH; ++e) {
        const bool in = ((okm >> (k0 + e)) & 1u) && b[e] >= b0 && b[e] <= b1;
        at[e] = -1;
        if constexpr (KEEP) {
          if (in) at[e] = entry_of(b[e]) - ps + (int)(bs[e] >> 16);
        } else if (in) {
          const unsigned h = (b[e] & 1u) * 16u;
          at[e] = (int)((atomicSub(&table[b[e] >> 1], 1u << h) >> h) & 0xffffu) - 1 - ps;
        }
        uk[e] = at[e] >= 0 ? u_of(k0, e) : 0.0;
      }
#pragma unroll
      for (int e = 0; e < BATCH; ++e)
        if (at[e] >= 0) {
          keys[at[e]] = order_key(uk[e]);
          ids[at[e]] = (unsigned short)(i0 + e * THREADS);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // (of the share's buckets the table now holds the starts)
    auto span_of = [&](unsigned b, int& st, int& en) {
      st = entry_of(b) - ps;
      en = min(entry_of(b + 1u), p1) - ps;
    };
    if (__builtin_expect(s_big > (unsigned)SORT_LIGHT, 0)) {         // heavy buckets of the share
      for (unsigned b = b0 + tid; b <= b1; b += THREADS) {
        int st, en;
        span_of(b, st, en);
        if (en - st > SORT_LIGHT) s_list[atomicAdd(&s_heavy, 1)] = ((unsigned)st << 16) | (unsigned)(en - st);
      }
      __syncthreads();
      const int heavy = s_heavy;
      for (int h = wave; h < heavy; h += WAVES) {
        const int st = (int)(s_list[h] >> 16), n = (int)(s_list[h] & 0xffffu);
        if (n <= SORT_WAVE_MAX) sort_pairs(keys + st, ids + st, n, lane, WAVE, [] { wave_sync(); });
      }
      __syncthreads();
      for (int h = 0; h < heavy; ++h) {
        const int st = (int)(s_list[h] >> 16), n = (int)(s_list[h] & 0xffffu);
        if (n > SORT_WAVE_MAX) sort_pairs(keys + st, ids + st, n, tid, THREADS, [] { __syncthreads(); });
      }
    }
    // 5. rank within the bucket
    for (int p = tid; p < p1 - ps; p += THREADS) {
      const unsigned long long key = keys[p];
      unsigned b;
      if (__builtin_expect(!sampled, 1)) {
        b = linear(key_value(key));
      } else {                                                       // the last bucket that starts at or before p
        b = b0;
#pragma unroll 1
        for (unsigned h = THREADS; h > 0; h /= 2)
          if (b + h <= b1 && entry_of(b + h) - ps <= p) b += h;
      }
      int st, en;
      span_of(b, st, en);
      int at = p;                                                    // heavy buckets are in order already
      if (en - st <= SORT_LIGHT) {
        int same = 0;
        at = st;
#pragma unroll 4
        for (int e = st; e < en; ++e) {
          const unsigned long long ke = keys[e];
          at += ke < key ? 1 : 0;
          same += ke == key ? 1 : 0;
        }
        if (same > 1) {                                              // equal u: by index
          const unsigned short id = ids[p];
#pragma unroll 4
          for (int e = st; e < en; ++e) at += (int)(keys[e] == key) & (int)(ids[e] < id);
        }
      }
      ord[at] = (unsigned short)p;
    }
    __syncthreads();
    write(p0, p1, [&](int j) { return (int)ids[ord[j - ps]]; });
  }
}

// The sorted u, v and delay of the index lists that k_sort_one left, where many
// long lists are ordered at once: 200 workgroups that gather from lists of 783
// KB miss their L2s (4 MiB an XCD) on nearly every line, so the gathers go to
// a launch of their own whose workgroups take the lists of an XCD one after
// the other (workgroup L runs on XCD L mod 8).
__global__ void __launch_bounds__(256) k_sort_gather(SortArgs a, int nt, int blocks) {
  const int L = blockIdx.x, r8 = L >> 3;
  const int tl = (r8 / blocks) * 8 + (L & 7);
  if (tl >= nt) return;
  const int t = a.t0 + tl, j = (r8 % blocks) * 256 + (int)threadIdx.x;
  if (j >= a.n_valid[t]) return;
  const size_t tb = (size_t)t * a.B;
  const int b = a.perm[tb + j];
  double u, v;
  plane_uv(a, tb + b, u, v);
  a.su[tb + j] = u;
  a.sv[tb + j] = v;
  if (a.sd != nullptr) a.sd[tb + j] = baseline_delay(a, tb, b);
}

// Merge neighbouring sorted runs of width w: each element's output position
// is its rank in its own run plus the number of smaller elements in the other
// run (binary search). All (key, index) pairs are distinct.
__global__ void __launch_bounds__(256) k_merge(SortArgs a, int w, int src) {
  const int t = a.t0 + blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.B) return;
  const size_t tb = (size_t)t * a.B;
  const unsigned long long* K = a.key[src] + tb;
  const int* I = a.idx[src] + tb;
  const int pb = (e / (2 * w)) * (2 * w);
  const int lend = min(pb + w, a.B);
  const int rend = min(pb + 2 * w, a.B);
  const unsigned long long mk = K[e];
  const int mi = I[e];
  const bool left = e < lend;
  int lo = left ? lend : pb, hi = left ? rend : lend;
  const int own = left ? e - pb : e - lend;
  while (lo < hi) {  // count of elements of the other run that are smaller
    const int mid = (lo + hi) >> 1;
    const unsigned long long km = K[mid];
    const bool less = km < mk || (km == mk && I[mid] < mi);
    if (less) lo = mid + 1; else hi = mid;
  }
  const int other = left ? lo - lend : lo - pb;
  const int out = pb + own + other;
  a.key[src ^ 1][tb + out] = mk;
  a.idx[src ^ 1][tb + out] = mi;
}

__global__ void __launch_bounds__(256) k_sort_finish(SortArgs a, int src) {
  const int t = a.t0 + blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.B) return;
  const size_t tb = (size_t)t * a.B;
  const unsigned long long k = a.key[src][tb + j];
  const int b = a.idx[src][tb + j];
  double u, v;
  plane_uv(a, tb + b, u, v);
  a.su[tb + j] = u;
  a.sv[tb + j] = v;
  if (a.sd != nullptr) a.sd[tb + j] = baseline_delay(a, tb, b);
  a.perm[tb + j] = b;
  const bool valid = k != KEY_MAX;
  const bool next_invalid = (j + 1 == a.B) || a.key[src][tb + j + 1] == KEY_MAX;
  if (valid && next_invalid) a.n_valid[t] = j + 1;
}

// ============================================================== cell bounds
// largest number of coefficients of the Kaiser-Bessel weight's polynomial (see kb_weight)
constexpr int KB_POLY_TERMS = 25;

struct ImgArgs {
  int T, C, B, N, M, weighting, norm, vis_type;
  double ndx;                   // fl(N * dx)
  const void* vis;              // [T][C][B] c64 or [T][C][B][2] f16/bf16
  const float* vis_scale;       // [C]
  const double* freq;           // [C]
  const int* ant1;              // [B]
  const int* ant2;              // [B]
  const float2* gains;          // [A] or null
  const double* su;             // [T][B]
  const double* sv;             // [T][B]
  const int* perm;              // [T][B]
  const double* sd;             // [T][B] sorted geometric delays (metres) or null: no rotation
  const int* n_valid;           // [T]
  const int* n_unflagged;       // [T]
  const double* vmax;           // [T] largest |v| (metres) of the usable baselines, or null
  int* bnd;                     // [T*C][N + 2]
  int* ncz;                     // [T*C] u-cell columns 0..ncz-1 may be non-empty; the rest are zero
  int ntiles;                   // column tiles per image of the current column kernel
  int* wpart;                   // [T*C][wstride] weight-sum partials, one per column tile
  int* kpart;                   // [T*C][wstride] kept-baseline partials, one per column tile
  int wstride;                  // partial slots per image (>= tiles of any producer kernel)
  int wtiles;                   // partial slots per image written by the current producer kernel
  int img0, nimg;               // this chunk: images [img0, img0 + nimg)
  float2* half;                 // [chunk][N/2][M] column-transformed half spectrum
  float2* grid;                 // MODE_GRID: [T*C][N][N]
  int* counts;                  // MODE_GRID: [T*C][N][N] or null
  float* images;                // [T*C][M][M]
  float* weight_sum;            // [T*C] or null
  int* n_dropped;               // [T*C] or null
  // adjoint
  const float* image_grad;      // [T*C][M][M]
  const float* wsum_in;         // [T*C] weight sums of the forward call, or null (count them)
  float2* gamma;                // [chunk][B] gradient w.r.t. V' per image
  float2* vis_grad;             // [T][C][B]
  float2* pacc;                 // [B] sum over images of gamma conj(V)
  float2* gain_grad;            // [A]
  float2* gfull;                // adjoint with a gridding kernel: [chunk][N/2][N] transformed columns
  int n_ant;
  // Kaiser-Bessel gridding kernel (kw = support in cells, 0 = nearest cell)
  int kw;
  float kbeta;                  // shape
  float kinv;                   // 1 / I0(kbeta)
  double kbeta_d;               // the shape in double (the correction is formed in double)
  double ktaper0_d;             // sinh(beta) / beta: the correction's value at 0 before normalising
  float k2w;                    // 2 / W
  int kpoly_on;                 // 1: weights from kpoly, 0: from cyl_bessel_i0f
  int kpoly_deg;                // degree D of that polynomial (<= KB_POLY_TERMS - 1)
  float kpoly[KB_POLY_TERMS];   // its coefficients in s = 1 - 2 (2d/W)^2, kpoly[k] of s^k, 0 above D
  // kernel gridding with uniform weighting: [chunk][B] per sorted entry, the
  // kept entries (direct and mirrored) at its nearest cell; null otherwise
  int* kdens;
};

// bnd[c + N/2] = first sorted position j with clamp(rint(u_j s)) >= c for
// c in [-N/2, N/2 + 1]; entry N + 1 is always n_valid. The clamped cell is
// non-decreasing along the sorted order (s > 0), so each bound is found either
// by one pass over the list, marking where the cell steps up, or - when the
// list is much longer than the N + 2 bounds - by a binary search per bound.
// Both give that first position. For s <= 0 or a non-finite s every bound
// still lies in [0, n_valid].
// One workgroup per image and segment of the sorted list (`segs` segments an
// image): a call of few images with long lists is bound by the
// latency of its longest workgroup, and the segments of a list are independent.
constexpr int BND_THREADS = 256;

__global__ void __launch_bounds__(BND_THREADS) k_bounds(ImgArgs a, int segs) {
  const int img = blockIdx.x / segs, seg = blockIdx.x - img * segs;
  const int t = img / a.C, ch = img - t * a.C;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const int N = a.N, H = N / 2;
  const double* su = a.su + (size_t)t * a.B;
  const int nv = a.n_valid[t];
  int* bnd = a.bnd + (size_t)img * (N + 2);
  auto ucol = [&](int j) -> int { return (int)fmin(fmax(rint(su[j] * s), (double)-H), (double)H); };
  const int cfirst = nv == 0 ? -H - 1 : ucol(0), clast = nv == 0 ? -H - 1 : ucol(nv - 1);
  if (seg == 0 && threadIdx.x == 0) a.ncz[img] = nonempty_columns(cfirst, clast, nv, N, a.kw);
  if (nv > 16 * (N + 2)) {
    for (int c = (int)threadIdx.x + seg * BND_THREADS - H; c <= H + 1; c += segs * BND_THREADS) {
      int lo = 0, hi = nv;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ucol(mid) >= c) hi = mid; else lo = mid + 1;
      }
      bnd[c + H] = lo;
    }
    return;
  }
  const int lane = threadIdx.x % WAVE;
  const int len = ((a.B + segs - 1) / segs + BND_THREADS - 1) / BND_THREADS * BND_THREADS;
  const int e = (int)min((long long)nv, (long long)(seg + 1) * len);
  constexpr int U = 4;                                       // cells in flight per thread
  for (long long j0 = (long long)seg * len; j0 < e; j0 += U * BND_THREADS) {
    int cj[U], cp[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const long long j = j0 + k * BND_THREADS + (int)threadIdx.x;
      cj[k] = j < e ? ucol((int)j) : 0;
      cp[k] = lane == 0 && j > 0 && j < e ? ucol((int)j - 1) : -H - 1;
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const long long j = j0 + k * BND_THREADS + (int)threadIdx.x;
      const int up = __shfl_up(cj[k], 1);
      if (j < e && j > 0)
        for (int c = (lane == 0 ? cp[k] : up) + 1; c <= cj[k]; ++c) bnd[c + H] = (int)j;
    }
  }
  // the cells up to the first entry's and those beyond the last one's
  if (seg == 0 && nv > 0)
    for (int c = (int)threadIdx.x - H; c <= cfirst; c += BND_THREADS) bnd[c + H] = 0;
  if (seg == segs - 1)
    for (int c = clast + 1 + (int)threadIdx.x; c <= H + 1; c += BND_THREADS) bnd[c + H] = nv;
}

// Largest |v| in metres over the usable baselines of each timestep (one
// workgroup per timestep). Since x -> rint(x |s|) is non-decreasing, every
// gridded row of an image at scale s satisfies |i_v| <= rint(vmax |s|), so the
// rows beyond that bound are known to be empty before the column is gridded.
__global__ void __launch_bounds__(256) k_vmax(const double* __restrict__ sv, const int* __restrict__ n_valid,
                                              int B, double* __restrict__ vmax) {
  __shared__ double red[256];
  const int t = blockIdx.x;
  const double* v = sv + (size_t)t * B;
  const int nv = n_valid[t];
  double m = 0.0;
  for (int j = threadIdx.x; j < nv; j += 256) m = fmax(m, fabs(v[j]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) vmax[t] = red[0];
}

// Zero band of an image's column transforms (see zero_band): the rows beyond
// rint(vmax |s|) are empty. Non-finite or out-of-range bounds give 0.
// reach: rows that an entry touches beyond its nearest one.
template <int N>
__device__ __forceinline__ int column_zero_band(const ImgArgs& a, int t, double s, int reach = 0) {
  if (a.vmax == nullptr) return 0;
  const double vc = rint(a.vmax[t] * fabs(s));
  return (vc >= 0.0 && vc < (double)(N / 2)) ? zero_band(N, (int)vc + 1 + reach) : 0;
}

// Sum of the per-tile partials of one image (read by one wavefront; every
// slot below wtiles was written by exactly one workgroup of the producer).
__device__ __forceinline__ int sum_partials(const int* part, int img, int wstride, int wtiles, int lane) {
  int v = 0;
  for (int i = lane; i < wtiles; i += WAVE) v += part[(size_t)img * wstride + i];
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// The same for partials holding FP32 weight sums (kernel gridding).
__device__ __forceinline__ float sum_partials_f(const int* part, int img, int wstride, int wtiles, int lane) {
  float v = 0.f;
  for (int i = lane; i < wtiles; i += WAVE) v += __int_as_float(part[(size_t)img * wstride + i]);
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ============================================================== visibility load
// g[a1] conj(g[a2]); an antenna index outside [0, n_ant) gives a zero gain.
__device__ __forceinline__ float2 antenna_gain(const float2* g, int i, int n) {
  return (unsigned)i < (unsigned)n ? g[i] : make_float2(0.f, 0.f);
}
template <class A>
__device__ __forceinline__ float2 baseline_gain(const A& a, int b) {
  const float2 g1 = antenna_gain(a.gains, a.ant1[b], a.n_ant);
  const float2 g2 = antenna_gain(a.gains, a.ant2[b], a.n_ant);
  return cmul(g1, cconj(g2));
}
__device__ __forceinline__ float2 load_vis_raw(const ImgArgs& a, size_t off, int ch) {
  float2 v;
  if (a.vis_type == VT_C64) {
    v = static_cast<const float2*>(a.vis)[off];
  } else if (a.vis_type == VT_F16) {
    const __half2 h = static_cast<const __half2*>(a.vis)[off];
    v = __half22float2(h);
    const float sc = a.vis_scale[ch];
    v.x *= sc; v.y *= sc;
  } else {
    const unsigned int w = static_cast<const unsigned int*>(a.vis)[off];
    v.x = __uint_as_float(w << 16);
    v.y = __uint_as_float(w & 0xffff0000u);
    const float sc = a.vis_scale[ch];
    v.x *= sc; v.y *= sc;
  }
  return v;
}
__device__ __forceinline__ float2 load_vis(const ImgArgs& a, size_t off, int b, int ch) {
  float2 v;
  if (a.vis_type == VT_C64) {
    v = static_cast<const float2*>(a.vis)[off];
  } else if (a.vis_type == VT_F16) {
    const __half2 h = static_cast<const __half2*>(a.vis)[off];
    v = __half22float2(h);
    const float sc = a.vis_scale[ch];
    v.x *= sc; v.y *= sc;
  } else {
    const unsigned int w = static_cast<const unsigned int*>(a.vis)[off];
    v.x = __uint_as_float(w << 16);
    v.y = __uint_as_float(w & 0xffff0000u);
    const float sc = a.vis_scale[ch];
    v.x *= sc; v.y *= sc;
  }
  if (a.gains != nullptr) v = cmul(baseline_gain(a, b), v);
  return v;
}

// Geometric phase rotation of a visibility: V exp(+2 pi i d nu / c) for the
// delay d (metres) of its baseline. The phase in cycles is formed in double
// and reduced to [-1/2, 1/2] before the single-precision sine and cosine.
__device__ __forceinline__ float2 rotate_phase(float2 v, double d, double f) {
  const double cyc = d * (f / C_LIGHT);
  const float fr = (float)(cyc - rint(cyc));
  float sn, cs;
  sincospif(2.0f * fr, &sn, &cs);
  return make_float2(v.x * cs - v.y * sn, v.x * sn + v.y * cs);
}

// Grid the column's entries: sorted positions [dlo, dhi) add V' at row i_v,
// positions [clo, chi) (the mirror column) add conj(V') at row -i_v. Both
// ranges are walked as one list, GU x 64 entries per step: every step first
// issues the sorted-list loads of all its entries, then their visibility
// gathers, then the LDS adds, so a wavefront keeps GU times more loads in
// flight. Only this wavefront touches the column, so the LDS adds happen in a
// fixed order (steps in sequence; within a step, sub-steps in sequence and
// lanes in LDS order).
constexpr int GU = 2;

struct ColSpan {                 // the sorted entries of one u-cell column
  int dlo, dhi, clo, chi;        // direct range and mirror (conjugate) range
  __device__ int nd() const { return dhi - dlo; }
  __device__ int total() const { return (dhi - dlo) + (chi - clo); }
};

struct EntryStep {               // GU x 64 entries in registers
  double sv[GU];
  double dl[GU];                 // geometric delay (phase rotation only)
  int bl[GU];
  int row[GU];
  float2 val[GU];
  bool ok[GU], cj[GU];
};

// phase 1: sorted-list loads (v in metres and baseline index) of the step at i0
// (ROT: and the geometric delays for the phase rotation)
template <bool ROT>
__device__ __forceinline__ void step_keys(const ImgArgs& a, const ColSpan& c, int i0, int t, int lane,
                                          EntryStep& e) {
  const size_t tb = (size_t)t * a.B;
  const int nd = c.nd(), total = c.total();
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int i = i0 + u * WAVE + lane;
    e.ok[u] = i < total;
    e.cj[u] = i >= nd;
    const int j = e.cj[u] ? c.clo + (i - nd) : c.dlo + i;
    e.sv[u] = e.ok[u] ? a.sv[tb + j] : 0.0;
    e.bl[u] = e.ok[u] ? a.perm[tb + j] : 0;
    if (ROT) e.dl[u] = e.ok[u] ? a.sd[tb + j] : 0.0;
  }
}

// phase 2: cell rows (FP64) and the visibility gathers of the kept entries
template <int N, bool ROT>
__device__ __forceinline__ void step_gather(const ImgArgs& a, int t, int ch, double s, EntryStep& e) {
  const size_t vb = ((size_t)t * a.C + ch) * a.B;
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const double iv = rint(e.sv[u] * s);
    e.ok[u] = e.ok[u] && fabs(iv) < (double)(N / 2);
    int r = (int)iv;
    if (e.cj[u]) r = -r;
    e.row[u] = r < 0 ? r + N : r;
    e.val[u] = e.ok[u] ? load_vis(a, vb + e.bl[u], e.bl[u], ch) : make_float2(0.f, 0.f);
    if (ROT) e.val[u] = rotate_phase(e.val[u], e.dl[u], a.freq[ch]);
  }
}

// ------------------------------------------------------ LDS accumulation
// LDS floating-point atomic adds are slow on gfx950: measured at about 190
// CU cycles per wave64 ds_add_f32, against about 5 for an integer atomic or a
// plain read-modify-write. The column being gridded is LDS that only its own
// wavefront writes, so the adds are done as plain read-modify-writes, and
// lanes that would touch the same element take turns: each turn, every
// pending lane posts a tag (turn * 64 + 64 - lane) to its key's claim slot
// with an integer atomic max, and the lane whose tag survives adds its value.
// Lanes whose elements coincide share a slot, so no two lanes of one turn touch
// one element; of the lanes sharing a slot the lowest goes first, so each
// element receives its adds in lane order, step after step: the order of the sorted list, whatever the
// grouping into steps. Tags grow with the wavefront's turn counter, so the
// claim slots never need clearing after their initial zeroing. Turns from ballots
// (rank_among_equal, as the signed kernel rows take them) are no faster here, where
// a turn is one add: all-sky columns 1,484 against 1,483 us, widefield 1,511
// against 1,496.
// Slots: a column buffer of up to 256 rows has one per row, so that only lanes
// that really meet on a row wait for each other (2.7 instead of 4 turns a step
// of the all-sky columns); for longer buffers the words would cost a workgroup
// per CU, and key mod 64 stays.
constexpr int CLAIM_TAG = 64;    // tags per turn
__host__ __device__ constexpr int claim_slots(int rows) {
  int n = 64;
  while (n < rows) n *= 2;
  return n <= 256 ? n : 64;
}

template <int SLOTS>
struct Claim {
  unsigned* slot;                // SLOTS words of this wavefront's LDS
  unsigned turn;                 // wave-uniform
};

// Zeroes this wavefront's claim slots (the caller's next wave_sync publishes them).
template <int SLOTS>
__device__ __forceinline__ Claim<SLOTS> claim_init(unsigned* slots, int lane) {
  for (int i = lane; i < SLOTS; i += WAVE) slots[i] = 0u;
  return Claim<SLOTS>{slots, 0u};
}

// dst[idx] += v (and cnt[cidx] += 1 with COUNT) for every active lane; lanes
// with equal idx must pass equal key. Counts are integers, so they take one
// atomic a step outside the turns.
template <bool COUNT, int SLOTS>
__device__ __forceinline__ void wave_add(float2* dst, int idx, int* cnt, int cidx, int key, float2 v, bool active,
                                         Claim<SLOTS>& cl, int lane) {
  if (COUNT && active) __hip_atomic_fetch_add(cnt + cidx, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  bool pending = active;
  while (__ballot(pending) != 0) {
    const unsigned tag = cl.turn * CLAIM_TAG + (unsigned)(CLAIM_TAG - lane);
    unsigned* slot = cl.slot + (key & (SLOTS - 1));
    if (pending) __hip_atomic_fetch_max(slot, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    wave_sync();
    if (pending && *slot == tag) {
      const float2 d = dst[idx];
      dst[idx] = make_float2(d.x + v.x, d.y + v.y);
      pending = false;
    }
    wave_sync();
    ++cl.turn;
  }
}

// phase 3: the LDS adds; kd / kc count the kept direct / conjugate entries
template <bool COUNT, int SLOTS>
__device__ __forceinline__ void step_add(const EntryStep& e, float2* buf, int* cnt, int& kd, int& kc, Claim<SLOTS>& cl,
                                         int lane) {
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    float2 v = e.val[u];
    if (e.cj[u]) v.y = -v.y;
    wave_add<COUNT>(buf, pad(e.row[u]), cnt, e.row[u], e.row[u], v, e.ok[u], cl, lane);
    kd += __popcll(__ballot(e.ok[u] && !e.cj[u]));
    kc += __popcll(__ballot(e.ok[u] && e.cj[u]));
  }
}

// All steps of a column from step i0 on; returns the kept direct and
// conjugate entries (added to kd / kc). The phase-rotated form is a separate
// copy of the loop, so the plain one carries none of its work.
template <int N, bool COUNT, bool ROT, int SLOTS>
__device__ __forceinline__ void grid_steps_t(const ImgArgs& a, const ColSpan& c, int i0, float2* buf, int* cnt,
                                             int t, int ch, double s, int lane, int& kd, int& kc, Claim<SLOTS>& cl) {
  const int total = c.total();
  EntryStep e;
  if (i0 < total) step_keys<ROT>(a, c, i0, t, lane, e);
  for (; i0 < total; i0 += GU * WAVE) {
    step_gather<N, ROT>(a, t, ch, s, e);
    // the next step's lists are in flight during this one's gathers and adds
    EntryStep nx;
    if (i0 + GU * WAVE < total) step_keys<ROT>(a, c, i0 + GU * WAVE, t, lane, nx);
    step_add<COUNT>(e, buf, cnt, kd, kc, cl, lane);
    e = nx;
  }
}
template <int N, bool COUNT, int SLOTS>
__device__ __forceinline__ void grid_steps(const ImgArgs& a, const ColSpan& c, int i0, float2* buf, int* cnt,
                                           int t, int ch, double s, int lane, int& kd, int& kc, Claim<SLOTS>& cl) {
  if (a.sd != nullptr) grid_steps_t<N, COUNT, true>(a, c, i0, buf, cnt, t, ch, s, lane, kd, kc, cl);
  else grid_steps_t<N, COUNT, false>(a, c, i0, buf, cnt, t, ch, s, lane, kd, kc, cl);
}

// ------------------------------------------------------------- kernel gridding
// Kaiser-Bessel weight C(d) = I0(beta sqrt(1 - (2d/W)^2)) / I0(beta), |d| <= W/2.
// I0(beta sqrt(w)) is an entire function of w = 1 - (2d/W)^2 in [0, 1], so a
// polynomial of low degree in s = 2w - 1 in [-1, 1] matches it closely: the
// host interpolates C at Chebyshev points of s and keeps the shortest
// truncation whose dropped Chebyshev terms sum below 2e-8 (degree 11 at
// W = 6 with the default shape). Its coefficients in powers of s are the
// function's expansion around w = 1/2, all positive and summing to about 1,
// so Horner's rule in FP32 loses no accuracy to cancellation. The degree
// picks one of three fixed-length forms (12, 16 or 25 coefficients, zeros
// above the degree), so that the coefficients stay in scalar registers and
// the loops unroll. Beyond 25 coefficients (beta above about 70) the weights
// come from cyl_bessel_i0f.
template <int TERMS>
__device__ __forceinline__ float kb_horner(float s, const float* c) {
  float p = c[TERMS - 1];
#pragma unroll
  for (int k = TERMS - 2; k >= 0; --k) p = fmaf(p, s, c[k]);
  return p;
}

__device__ __forceinline__ float kb_weight(float d, const ImgArgs& a) {
  const float t = d * a.k2w;
  if (a.kpoly_on) {
    const float s = fmaxf(-1.0f, fmaf(-2.0f * t, t, 1.0f));
    if (a.kpoly_deg < 12) return kb_horner<12>(s, a.kpoly);
    if (a.kpoly_deg < 16) return kb_horner<16>(s, a.kpoly);
    return kb_horner<KB_POLY_TERMS>(s, a.kpoly);
  }
  return cyl_bessel_i0f(a.kbeta * sqrtf(fmaxf(0.0f, fmaf(-t, t, 1.0f)))) * a.kinv;
}

// Reciprocal of the correction at xi cycles per cell, 1 / c(xi) with
// c(xi) = [sinh(z)/z] / [sinh(beta)/beta], z = sqrt(beta^2 - (pi W xi)^2)
// (sin(|z|)/|z| beyond pi W |xi| = beta). Formed in double: near a zero of
// c (small beta, pixels near the edge of a full-field image) FP32 would lose
// most of its digits in z.
__device__ __forceinline__ float kb_inv_taper(double xi, const ImgArgs& a) {
  const double b = a.kbeta_d;
  const double x = 3.141592653589793 * (double)a.kw * xi;
  const double z2 = b * b - x * x;
  double f = 1.0;
  if (z2 > 0.0) { const double z = sqrt(z2); f = sinh(z) / z; }
  else if (z2 < 0.0) { const double z = sqrt(-z2); f = sin(z) / z; }
  return (float)(a.ktaper0_d / f);
}

// Rows of a column under kernel gridding. Sizes whose transform starts from
// registers (plan_even up to 2048) keep row j, -N/2 <= j < N/2, at j + N/2
// without padding, so that a footprint is one run of addresses: one base per
// entry and constant offsets, instead of a wrap and a padded index per row. The
// others keep the transform's padded layout.
template <int N>
constexpr bool kb_signed() { return plan_even(N) && N <= 2048; }
template <int N>
__device__ __forceinline__ int kb_row(int r) {        // place of row r, 0 <= r < N
  return kb_signed<N>() ? (r < N / 2 ? r + N / 2 : r - N / 2) : pad(r);
}

// Whether the footprint of a baseline at cell position (xu, xv), each a product
// rounded to double, lies inside |i| < N/2 (H = N/2) on both axes, that is
// ceil(x - W/2) > -N/2 and floor(x + W/2) < N/2. The gridding, the occupancy pass
// and the adjoint ask here: where one of them formed x +- W/2 in one rounding
// (W >= N/2), the adjoint kept a baseline that the others had dropped, and divided
// by an occupancy that nothing had written.
template <int H>
__device__ __forceinline__ bool kb_kept(double xu, double xv, double hw) {
#pragma clang fp contract(off)
  return fabs(xu) + hw < (double)H && fabs(xv) + hw < (double)H;
}

// Number of active lanes below this one with the same BITS-bit key: the lanes
// that agree with it in every bit, from one ballot a bit.
template <int BITS>
__device__ __forceinline__ int rank_among_equal(int key, bool active) {
  unsigned long long same = __ballot(active);
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const unsigned long long ones = __ballot((key >> b) & 1);
    same &= ((key >> b) & 1) ? ones : ~ones;
  }
  return __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
}

// Adds w[k] v to rows j0 + k, k < nrow, of this column for every active lane:
// lanes with the same first row j0 take turns, lowest lane first, and lanes with
// different j0 never reach the same row at the same k, so a turn adds all of its
// lanes' rows in sequence over k. Each element receives its adds in a fixed
// order: step, turn, k. In the signed layout a lane's turn is the number of lanes
// below it with the same j0 (at N = 2048 the same j0 mod 1024, so that rows 1024
// apart take turns too), from ballots (no LDS round trips before a turn, and no
// waiting for lanes whose j0 only shares a claim slot); the other sizes claim
// turns as wave_add does, keyed on j0. nrow is W or W + 1; in the signed layout the
// few lanes with W + 1 add the last one apart (added to all with weight 0, it would
// spread an infinite or NaN visibility to the row after the footprint). Its adds are
// written as fmaf: left to the compiler, the products move out of the turns and
// round by themselves (384 images of 1024^2, W = 6: 1.717e-7 instead of 1.713e-7
// from 64 bits).
// What bounds it: the chain of W + 1 dependent read-modify-writes per turn at 16
// wavefronts per CU (the buffers' LDS), and the weights. 384 images of 1024^2,
// W = 6: the column launch 840 -> 679 us (736 with the layout alone, 697 with the
// ballots, then the row offsets and the keep rule in fewer double operations).
template <int N, bool COUNT, int KMAX, int SLOTS>
__device__ __forceinline__ void kb_add_rows(float2* buf, int* cnt, int j0, int nrow, const float (&w)[KMAX + 1],
                                            float2 v, bool active, int kw, Claim<SLOTS>& cl, int lane) {
  if constexpr (kb_signed<N>()) {
    float2* row = buf + (j0 + N / 2);
    constexpr int BITS = N >= 1024 ? 10 : N >= 512 ? 9 : N >= 256 ? 8 : 7;
    const int below = rank_among_equal<BITS>(j0, active);
    const int rank = active ? below : -1;
    float wl = 0.f;                                    // w[kw]
#pragma unroll
    for (int k = 0; k <= KMAX; ++k) {
      if (k > kw) break;
      wl = w[k];
    }
    for (int t = 0; __ballot(rank >= t) != 0; ++t) {
      if (rank == t) {
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
          if (k >= kw) break;
          const float2 d = row[k];
          row[k] = make_float2(fmaf(w[k], v.x, d.x), fmaf(w[k], v.y, d.y));
          if (COUNT) cnt[j0 + N / 2 + k] += 1;
          wave_sync();
        }
        if (nrow > kw) {                               // the few footprints of W + 1 rows
          const float2 d = row[kw];
          row[kw] = make_float2(fmaf(wl, v.x, d.x), fmaf(wl, v.y, d.y));
          if (COUNT) cnt[j0 + N / 2 + kw] += 1;
        }
        wave_sync();
      }
    }
    return;
  }
  bool pending = active;
  while (__ballot(pending) != 0) {
    const unsigned tag = cl.turn * CLAIM_TAG + (unsigned)(CLAIM_TAG - lane);
    unsigned* slot = cl.slot + (j0 & (SLOTS - 1));
    if (pending) __hip_atomic_fetch_max(slot, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    wave_sync();
    const bool go = pending && *slot == tag;
#pragma unroll
    for (int k = 0; k <= KMAX; ++k) {
      if (k > kw) break;
      if (go && k < nrow) {
        const int r = j0 + k < 0 ? j0 + k + N : j0 + k;
        const float2 d = buf[pad(r)];
        buf[pad(r)] = make_float2(d.x + w[k] * v.x, d.y + w[k] * v.y);
        if (COUNT) cnt[r] += 1;
      }
      wave_sync();
    }
    pending = pending && !go;
    ++cl.turn;
  }
}

// Kernel gridding of u-cell column c: the span holds the sorted entries whose
// nearest column c' lies within floor(W/2 + 1/2) of c (direct) and of -c
// (mirror): |c - x_u| <= W/2 and |x_u - c'| <= 1/2 bound |c - c'|. Each
// direct entry at exact position x adds C(c - x_u) C(j - x_v) V' to the rows j
// of its footprint, each mirror entry (its conjugate, at -x) adds
// C(c + x_u) C(j + x_v) conj(V'). One entry per lane per step; its W + 1
// row weights are formed first (KMAX >= W bounds them at compile time), then
// kb_add_rows adds them. kd / kc count kept entries whose nearest column is
// c (each baseline once); wsum collects this lane's weights.
template <int N, bool COUNT, int KMAX, int SLOTS>
__device__ __forceinline__ void grid_steps_kb(const ImgArgs& a, const ColSpan& sp, int c, float2* buf,
                                              int* cnt, int t, int ch, double s, int lane, int& kd,
                                              int& kc, float& wsum, Claim<SLOTS>& cl, const int* dens) {
  constexpr int H = N / 2;
  const size_t tb = (size_t)t * a.B;
  const size_t vb = ((size_t)t * a.C + ch) * a.B;
  const double hw = 0.5 * a.kw;
  const int kw = a.kw;
  const int nd = sp.nd(), total = sp.total();
  for (int i0 = 0; i0 < total; i0 += WAVE) {
    const int i = i0 + lane;
    bool ok = i < total;
    const bool cj = i >= nd;
    const int j = cj ? sp.clo + (i - nd) : sp.dlo + i;
    double xu = 0.0, xv = 0.0;
    int b = 0;
    if (ok) {
      xu = a.su[tb + j] * s;
      xv = a.sv[tb + j] * s;
      b = a.perm[tb + j];
    }
    ok = ok && kb_kept<H>(xu, xv, hw);
    if (cj) { xu = -xu; xv = -xv; }
    const bool home = ok && rint(xu) == (double)c;
    kd += __popcll(__ballot(home && !cj));
    kc += __popcll(__ballot(home && cj));
    const double du = (double)c - xu;
    const bool in = ok && fabs(du) <= hw;
    float2 v = make_float2(0.f, 0.f);
    float wu = 0.f;
    int j0 = 0, nrow = 0;
    float dhi = 0.f, dlo = 0.f;
    if (in) {
      v = load_vis(a, vb + b, b, ch);
      if (a.sd != nullptr) v = rotate_phase(v, a.sd[tb + j], a.freq[ch]);
      if (cj) v.y = -v.y;
      wu = kb_weight((float)du, a);
      // uniform weighting: the baseline's share of its nearest cell
      if (dens != nullptr) wu = wu / (float)dens[j];
      j0 = (int)ceil(xv - hw);
      nrow = (int)floor(xv + hw) - j0 + 1;       // W or W + 1 rows
      // j0 - x_v in two floats, the first a multiple of 2^-18, so that k + dhi
      // is exact and (k + dhi) + dlo is the double j0 + k - x_v rounded once
      const double d0 = (double)j0 - xv;
      dhi = (float)(rint(d0 * 0x1p18) * 0x1p-18);
      dlo = (float)(d0 - (double)dhi);
    }
    float w[KMAX + 1];
#pragma unroll
    for (int k = 0; k <= KMAX; ++k) {
      w[k] = 0.f;
      if (k > kw) break;
      if (k < nrow) {
        w[k] = wu * kb_weight(((float)k + dhi) + dlo, a);
        wsum += w[k];
      }
    }
    kb_add_rows<N, COUNT, KMAX>(buf, cnt, j0, nrow, w, v, in, kw, cl, lane);
  }
}

// u-cell columns (one wavefront each) per workgroup of the column kernels
__host__ __device__ constexpr int cols_per_wg(int n) { return n <= 1024 ? 8 : (n <= 2048 ? 4 : 2); }

// Uniform weighting with kernel gridding: the weight of a kept baseline is
// 1 / n, n the number of kept entries - direct and mirrored - whose nearest
// cell is the baseline's own. This pass writes n for every kept entry of each
// image of the chunk into a.kdens[li][j] (j its sorted position). One wavefront
// per signed u-cell column c: it counts the kept direct entries of column c and
// the mirrored entries of column -c per row in an LDS row array with integer
// atomics, and reads the counts back for the direct entries. Kept entries have
// |nearest cell| <= N/2 - 1 on both axes, so the columns -N/2+1 .. N/2-1 hold all
// of them. Bound by the latency of a column's loads: a workgroup per image that
// walked its columns took 214 us for 8 images of 1024^2 and 740 for 20 with
// 32,640 baselines; a wavefront per column 12 and 60.
constexpr int DENS_WAVES = 4;
template <int N>
constexpr int dens_tiles() { return (N - 1 + DENS_WAVES - 1) / DENS_WAVES; }

template <int N>
__global__ void __launch_bounds__(DENS_WAVES * WAVE) k_kb_density(ImgArgs a) {
  extern __shared__ int dens_lds[];
  constexpr int H = N / 2;
  const int r8 = (int)(blockIdx.x >> 3);             // (all columns of an image on one XCD, as the column kernel)
  const int li = (r8 / dens_tiles<N>()) * 8 + (int)(blockIdx.x & 7);
  if (li >= a.nimg) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int c = -H + 1 + (r8 % dens_tiles<N>()) * DENS_WAVES + wave;
  if (c >= H) return;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int* bnd = a.bnd + (size_t)img * (N + 2);
  const ColSpan sp{bnd[c + H], bnd[c + 1 + H], bnd[-c + H], bnd[-c + 1 + H]};
  const int nd = sp.nd(), total = sp.total();
  if (nd == 0) return;
  int* rc = dens_lds + wave * N;                     // rc[iv + H]: entries in row iv of the column
  for (int r = lane; r < N; r += WAVE) rc[r] = 0;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const double hw = 0.5 * a.kw;
  const double* su = a.su + (size_t)t * a.B;
  const double* sv = a.sv + (size_t)t * a.B;
  int* out = a.kdens + (size_t)li * a.B;
  // nearest row of entry j (mirrored with mj), or N when it is not kept
  auto row_of = [&](int j, bool mj) -> int {
    const double xu = su[j] * s, xv = sv[j] * s;
    if (!kb_kept<H>(xu, xv, hw)) return N;
    const int r = (int)rint(xv);
    return mj ? -r : r;
  };
  wave_sync();
  for (int i = lane; i < total; i += WAVE) {
    const bool mj = i >= nd;
    const int r = row_of(mj ? sp.clo + (i - nd) : sp.dlo + i, mj);
    if (r != N) atomicAdd(&rc[r + H], 1);
  }
  wave_sync();
  for (int i = lane; i < nd; i += WAVE) {
    const int r = row_of(sp.dlo + i, false);
    if (r != N) out[sp.dlo + i] = rc[r + H];
  }
}

// Twiddle table staged in LDS (one copy per workgroup) where it fits beside
// the transform buffers without lowering occupancy.
template <int N>
struct TwLds { static constexpr bool ON = N <= 1024; };

// CL: copy only the compact table (tw_entries_compact), for transforms that
// form the last stage's higher twiddle powers in registers.
template <int N, bool CL = false>
__device__ __forceinline__ const float2* stage_twiddles(float2* lds_tw) {
  if constexpr (TwLds<N>::ON) {
    const float2* g = TwTable<N>::stages();
    constexpr int NTW = CL ? tw_entries_compact(N) : tw_entries(N);
    for (int i = threadIdx.x; i < NTW; i += blockDim.x) lds_tw[i] = g[i];
    return lds_tw;      // visible after the caller's next __syncthreads
  } else {
    return TwTable<N>::stages();
  }
}

template <int N, int CPW_ = cols_per_wg(N)>
struct Cols {
  static constexpr int STRIDE = padded_len(N);                // complex per column buffer
  static constexpr int CPW = CPW_;
  static constexpr int THREADS = CPW * WAVE;
  static constexpr int TW = TwLds<N>::ON ? tw_entries(N) : 0; // complex twiddles in LDS
  static size_t lds_bytes(bool counts) {
    return (size_t)(CPW * STRIDE + TW) * sizeof(float2) + (counts ? (size_t)CPW * N * sizeof(int) : 0);
  }
  // the gridding kernel adds every wavefront's claim slots after that
  static constexpr int SLOTS = claim_slots(N);
  static size_t grid_lds_bytes(bool counts) { return lds_bytes(counts) + (size_t)CPW * SLOTS * sizeof(unsigned); }
};

// One workgroup = CPW consecutive u-cell columns of one image; one wavefront
// per column. MODE_IMAGE: columns 0..N/2-1 (the half spectrum), transform
// along v, rows of the cutout written to `half`. MODE_GRID (kernel gridding): all
// N columns, weighted grid and counts written out.
// The 1D grid is laid out so that all column tiles of an image share one XCD
// (workgroup L runs on XCD L mod 8): the image's visibility row and the
// timestep's sorted lists are then fetched into a single L2.
// KB: Kaiser-Bessel kernel gridding instead of nearest cell; uniform weighting
// then comes from the per-entry cell occupancy of k_kb_density (a.kdens), so
// UNI (the nearest-cell division by counts) stays off.
// KMAX: largest support W the kernel gridding form handles (rows k = 0 .. W).
// HMC > 0 (KB): the cutout half-width fixed at compile time, so that the last stage
// computes only the rows it stores: columns of 384 images 1024^2 -> 512^2, W = 6,
// 678 -> 653 us.
template <int N, int MODE, bool UNI, int CPW = cols_per_wg(N), bool KB = false, int KMAX = 16, int HMC = 0>
__global__ void __launch_bounds__((Cols<N, CPW>::THREADS)) k_grid_cols(ImgArgs a) {
  static_assert(!(KB && UNI), "kernel gridding weights uniformly through a.kdens");
  static_assert(KB || MODE == MODE_IMAGE, "k_grid_write writes the nearest-cell grids");
  extern __shared__ float4 lds_raw[];
  __shared__ int red[2 * CPW];
  using C_ = Cols<N, CPW>;
  constexpr int H = N / 2;
  constexpr bool CNT = UNI || MODE == MODE_GRID;
  const int L = blockIdx.x;
  const int r8 = L >> 3;
  const int li = (r8 / a.ntiles) * 8 + (L & 7);
  const int tile = r8 % a.ntiles;
  if (li >= a.nimg) return;                          // padding of the last group of 8 images
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  float2* ltw = lds + CPW * C_::STRIDE;
  int* lcnt = reinterpret_cast<int*>(ltw + C_::TW);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int c0 = tile * CPW;
  const int ncols = MODE == MODE_IMAGE ? min(H, a.ncz[img]) : N;
  if (c0 >= ncols) {                                 // the whole tile is empty
    if (threadIdx.x == 0) {
      a.wpart[(size_t)img * a.wstride + tile] = 0;
      a.kpart[(size_t)img * a.wstride + tile] = 0;
    }
    return;
  }
  const int col = c0 + wave;                        // MODE_IMAGE: 0..H-1, MODE_GRID: 0..N-1
  const bool active = col < ncols;
  const int cs = MODE == MODE_IMAGE ? col : (col < H ? col : col - N);  // signed u cell
  float2* buf = lds + wave * C_::STRIDE;
  int* cnt = CNT ? lcnt + wave * N : nullptr;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const float2* tw = MODE == MODE_IMAGE ? stage_twiddles<N>(ltw) : nullptr;

  for (int r = lane; r < C_::STRIDE; r += WAVE) buf[r] = make_float2(0.f, 0.f);
  if (CNT)
    for (int r = lane; r < N; r += WAVE) cnt[r] = 0;
  unsigned* lclaim = reinterpret_cast<unsigned*>(lcnt + (CNT ? CPW * N : 0));
  // (the signed rows of kernel gridding take their turns from ballots; leaving out their
  // slots was slower: 24 images of 512^2, 6-cell kernel, half of 4,950 baselines in 2% of
  // the u range 630 -> 655 us, none faster)
  Claim<C_::SLOTS> cl = claim_init<C_::SLOTS>(lclaim + wave * C_::SLOTS, lane);
  wave_sync();

  int kept_b = 0, wcontrib = 0;
  if (KB && active && cs != H && cs != -H) {
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    const int hk = (a.kw + 1) / 2;                  // see grid_steps_kb
    auto at = [&](int c) { return bnd[min(max(c, -H), H + 1) + H]; };
    const ColSpan span{at(cs - hk), at(cs + hk + 1), at(-cs - hk), at(-cs + hk + 1)};
    int kd = 0, kc = 0;
    float ws = 0.f;
    const int* dens = a.kdens != nullptr ? a.kdens + (size_t)li * a.B : nullptr;
    grid_steps_kb<N, CNT, KMAX>(a, span, cs, buf, cnt, t, ch, s, lane, kd, kc, ws, cl, dens);
    wave_sync();
    kept_b = kd + ((MODE == MODE_IMAGE && cs > 0) ? kc : 0);
    for (int o = WAVE / 2; o > 0; o >>= 1) ws += __shfl_xor(ws, o);
    wcontrib = __float_as_int(((MODE == MODE_IMAGE && cs > 0) ? 2.0f : 1.0f) * ws);
  } else if (!KB && active && cs != H && cs != -H) {
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    const ColSpan span{bnd[cs + H], bnd[cs + 1 + H], bnd[-cs + H], bnd[-cs + 1 + H]};
    int kd = 0, kc = 0;
    grid_steps<N, CNT>(a, span, 0, buf, cnt, t, ch, s, lane, kd, kc, cl);
    wave_sync();
    // baselines counted once: the direct entry of every cell column, plus the
    // conjugate entries of columns whose mirror the image path never visits
    kept_b = kd + (cs > 0 ? kc : 0);
    const int mult = cs > 0 ? 2 : 1;
    if (UNI) {
      int occ = 0;
      for (int r = lane; r < N; r += WAVE) {
        const int n = cnt[r];
        if (n > 0) {
          float2 v = buf[pad(r)];
          v.x = v.x / (float)n;
          v.y = v.y / (float)n;
          buf[pad(r)] = v;
          ++occ;
        }
      }
      for (int o = WAVE / 2; o > 0; o >>= 1) occ += __shfl_xor(occ, o);
      wcontrib = mult * occ;
      wave_sync();
    } else {
      wcontrib = mult * (kd + kc);
    }
  }
  if (lane == 0) { red[wave] = wcontrib; red[CPW + wave] = kept_b; }
  __syncthreads();                                   // also publishes the LDS twiddles
  if (threadIdx.x == 0) {
    int ws = 0, ks = 0;
    float wf = 0.f;                                  // kernel gridding: FP32 weight sums
    for (int i = 0; i < CPW; ++i) {
      ws += red[i];
      wf += __int_as_float(red[i]);
      ks += red[CPW + i];
    }
    a.wpart[(size_t)img * a.wstride + tile] = KB ? __float_as_int(wf) : ws;
    a.kpart[(size_t)img * a.wstride + tile] = ks;
  }

  if constexpr (MODE == MODE_IMAGE && plan_even(N) && N <= 256) {
    // a column takes N / 16 lanes (one first-stage butterfly each), so the first
    // wavefronts transform the tile's columns and the others are done; the
    // exchanges use half of each column's buffer (2,000 images of 128^2 191 -> 161
    // us, 800 of 256^2 166 -> 141; at 512^2, two columns a wavefront, 300 -> 328)
    constexpr int L = N / 16, R = HalfIn<N, L>::R, PER = HalfIn<N, L>::PER;
    const int vec = threadIdx.x / L, ln = threadIdx.x % L;
    if (vec < CPW && c0 + vec < ncols) {
      float2* b = lds + vec * C_::STRIDE;
      HalfIn<N, L> x;
#pragma unroll
      for (int p = 0; p < PER; ++p)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int q = ln + p * L + r * (N / R);
          x.v[p][r] = b[KB ? kb_row<N>(q) : pad(q)];
        }
      wave_sync();
      float2* dst = a.half + ((size_t)li * H + c0 + vec) * a.M;
      const int hm = a.M / 2;
      wave_fft_half_emit<N, +1, 0, false, L>(b, ln, tw, x, [&](auto qb, float2 v) {
        cutout_lane<N, decltype(qb)::value>(ln, hm, [&](unsigned m) { store_at(dst, m, v); });
      });
    }
  } else if constexpr (MODE == MODE_IMAGE && KB && kb_signed<N>()) {
    if (active) {
      float2* dst = a.half + ((size_t)li * H + col) * a.M;
      const int hm = HMC > 0 ? HMC : a.M / 2;
      auto body = [&](auto zbc) {
        constexpr int ZB = decltype(zbc)::value, R = HalfIn<N>::R, zlo = R / 2 - ZB / 2, zhi = R / 2 + ZB / 2;
        HalfIn<N> x;
#pragma unroll
        for (int p = 0; p < HalfIn<N>::PER; ++p)
#pragma unroll
          for (int r = 0; r < R; ++r)
            if ((r < zlo || r >= zhi) && (N / R % WAVE == 0 || lane + p * WAVE < N / R))
              x.v[p][r] = buf[kb_row<N>(lane + p * WAVE + r * (N / R))];
        wave_sync();
        wave_fft_half_emit<N, +1, ZB>(buf, lane, tw, x, [&](auto qb, float2 v) {
          cutout_block<N, decltype(qb)::value>(lane, hm, [&](unsigned m) { store_at(dst, m, v); });
        });
      };
      // a footprint reaches (W + 1) / 2 rows beyond the nearest one
      if (HalfIn<N>::R == 16 && column_zero_band<N>(a, t, s, (a.kw + 1) / 2) >= 4) body(ic<HalfIn<N>::R == 16 ? 4 : 0>{});
      else body(ic<0>{});
    }
  } else if (MODE == MODE_IMAGE) {
    if (active) {
      // rows of the cutout straight from the last stage: output row m holds
      // v-frequency q = (m - M/2) mod N
      float2* dst = a.half + ((size_t)li * H + col) * a.M;
      const int hm = a.M / 2;
      wave_fft_emit<N, +1>(buf, lane, tw, [&](auto qb, float2 v) {
        cutout_block<N, decltype(qb)::value>(lane, hm, [&](unsigned m) { store_at(dst, m, v); });
      });
    }
  } else {
    // write the CPW-column tile row by row (CPW consecutive cells per row)
    float2* g = a.grid + (size_t)img * N * N;
    int* gc = a.counts ? a.counts + (size_t)img * N * N : nullptr;
    for (int e = threadIdx.x; e < N * CPW; e += blockDim.x) {
      const int r = e / CPW, w = e % CPW;
      if (c0 + w < N) {
        g[(size_t)r * N + c0 + w] = lds[w * C_::STRIDE + kb_row<N>(r)];
        if (gc) gc[(size_t)r * N + c0 + w] = lcnt[w * N + (kb_signed<N>() ? kb_row<N>(r) : r)];
      }
    }
  }
}

// ------------------------------------------- column pass, half-length LDS
// The image-mode column kernel (nearest cell) with every LDS exchange of the
// column through N/2 points: the rows below N/2 are gridded (and, with
// uniform weighting, divided by their counts) and handed to the first
// stage's registers, then the rows above, and the stages exchange in two
// rounds (wave_fft_half_emit). Each row receives the same adds in the same
// order as in the full-buffer kernel.
template <int N, int CPW, bool UNI>
struct ColsHalf {
  static constexpr int STRIDE = padded_len(N / 2);
  static constexpr int THREADS = CPW * WAVE;
  // compact twiddle table in LDS: at N = 1024 and 4 columns per workgroup
  // 22.5 KB instead of 26.6 KB, so seven workgroups share a CU instead of six
  static constexpr bool CL = TwLds<N>::ON && compact_last(N);
  static constexpr int TW = TwLds<N>::ON ? tw_entries_compact(N) : 0;
  static constexpr int SLOTS = claim_slots(N / 2);
  static constexpr size_t LDS = (size_t)(CPW * STRIDE + TW) * sizeof(float2) +
                                (UNI ? (size_t)CPW * (N / 2) * sizeof(int) : 0) +
                                (size_t)CPW * SLOTS * sizeof(unsigned);
};

// LDS adds (and counts) of the kept entries of a step whose row lies in half HF
template <int N, int HF, bool COUNT, int SLOTS>
__device__ __forceinline__ void step_add_half(const EntryStep& e, float2* hbuf, int* hcnt, Claim<SLOTS>& cl, int lane) {
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const bool act = e.ok[u] && (e.row[u] >= N / 2) == (HF == 1);
    float2 v = e.val[u];
    if (e.cj[u]) v.y = -v.y;
    const int r = e.row[u] - HF * (N / 2);
    wave_add<COUNT>(hbuf, pad(r), hcnt, r, r, v, act, cl, lane);
  }
}

__device__ __forceinline__ void step_count(const EntryStep& e, int& kd, int& kc) {
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    kd += __popcll(__ballot(e.ok[u] && !e.cj[u]));
    kc += __popcll(__ballot(e.ok[u] && e.cj[u]));
  }
}

template <int N, bool UNI>
__device__ __forceinline__ void zero_half(float2* hbuf, int* hcnt, int lane) {
  for (int r = lane; r < padded_len(N / 2); r += WAVE) hbuf[r] = make_float2(0.f, 0.f);
  if (UNI)
    for (int r = lane; r < N / 2; r += WAVE) hcnt[r] = 0;
}

// Uniform weighting of one half: every occupied cell divided by its count;
// returns this lane's number of occupied cells.
template <int N>
__device__ __forceinline__ int uniform_half(float2* hbuf, const int* hcnt, int lane) {
  int occ = 0;
  for (int r = lane; r < N / 2; r += WAVE) {
    const int n = hcnt[r];
    if (n > 0) {
      float2 v = hbuf[pad(r)];
      v.x = v.x / (float)n;
      v.y = v.y / (float)n;
      hbuf[pad(r)] = v;
      ++occ;
    }
  }
  return occ;
}

// Grids one column in two halves of N/2 rows through hbuf: done(ic<HF>) takes
// half HF before the other half overwrites it. A column of at most GU x 64
// entries (the usual case) keeps its one step of entries in registers for both
// halves; longer columns load them again. COUNT: hcnt counts the entries of
// every cell; UNI: cells are divided by their counts. occ: this lane's occupied
// cells (UNI).
template <int N, bool ROT, bool UNI, bool COUNT, int SLOTS, class Done>
__device__ __forceinline__ void grid_halves(const ImgArgs& a, const ColSpan& c, float2* hbuf, int* hcnt, int t, int ch,
                                            double s, int lane, int& kd, int& kc, int& occ, Claim<SLOTS>& cl,
                                            Done&& done) {
  static_assert(COUNT || !UNI, "uniform weighting needs the counts");
  const int total = c.total();
  const bool one = total <= GU * WAVE;
  EntryStep e;
  static_for<0, 2>([&](auto hf) {
    constexpr int HF = decltype(hf)::value;
    zero_half<N, COUNT>(hbuf, hcnt, lane);
    wave_sync();
    if (one) {
      if (total > 0) {
        if constexpr (HF == 0) {
          step_keys<ROT>(a, c, 0, t, lane, e);
          step_gather<N, ROT>(a, t, ch, s, e);
          step_count(e, kd, kc);
        }
        step_add_half<N, HF, COUNT>(e, hbuf, hcnt, cl, lane);
      }
    } else {
      for (int i0 = 0; i0 < total; i0 += GU * WAVE) {
        EntryStep f;
        step_keys<ROT>(a, c, i0, t, lane, f);
        step_gather<N, ROT>(a, t, ch, s, f);
        step_add_half<N, HF, COUNT>(f, hbuf, hcnt, cl, lane);
        if constexpr (HF == 0) step_count(f, kd, kc);
      }
    }
    wave_sync();
    if (UNI) {
      occ += uniform_half<N>(hbuf, hcnt, lane);
      wave_sync();
    }
    done(hf);
  });
}

// The same with each half handed to the first stage's registers.
template <int N, bool ROT, bool UNI, int ZB, int SLOTS>
__device__ __forceinline__ void grid_col_half(const ImgArgs& a, const ColSpan& c, float2* hbuf, int* hcnt,
                                              HalfIn<N>& in, int t, int ch, double s, int lane, int& kd,
                                              int& kc, int& occ, Claim<SLOTS>& cl) {
  grid_halves<N, ROT, UNI, UNI>(a, c, hbuf, hcnt, t, ch, s, lane, kd, kc, occ, cl, [&](auto hf) {
    half_read<N, HalfIn<N>::R, decltype(hf)::value, ZB>(hbuf, lane, in.v);
    wave_sync();
  });
}

// Same tiling, XCD mapping and outputs as k_grid_cols<N, MODE_IMAGE, UNI, CPW>.
// HMC > 0: the cutout half-width M/2 fixed at compile time (M = N/2 takes
// HMC = N/4), so that the last stage computes only the outputs it stores and
// the cutout tests vanish; 0: read from the arguments.
template <int N, int CPW, bool UNI, int HMC = 0>
__global__ void __launch_bounds__((ColsHalf<N, CPW, UNI>::THREADS)) k_grid_cols_half(ImgArgs a) {
  extern __shared__ float4 lds_raw[];
  using C_ = ColsHalf<N, CPW, UNI>;
  constexpr int H = N / 2;
  const int L = blockIdx.x;
  const int r8 = L >> 3;
  const int li = (r8 / a.ntiles) * 8 + (L & 7);
  const int tile = r8 % a.ntiles;
  if (li >= a.nimg) return;                          // padding of the last group of 8 images
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  float2* ltw = lds + CPW * C_::STRIDE;
  int* lcnt = reinterpret_cast<int*>(ltw + C_::TW);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int c0 = tile * CPW;
  const int ncols = min(H, a.ncz[img]);
  const int col = c0 + wave;                         // u cell 0..H-1
  // one weight / kept-baseline partial per column, written by its wavefront
  int* wslot = a.wpart + (size_t)img * a.wstride + col;
  int* kslot = a.kpart + (size_t)img * a.wstride + col;
  if (c0 >= ncols) {                                 // the whole tile is empty
    if (lane == 0 && col < H) { *wslot = 0; *kslot = 0; }
    return;
  }
  const bool active = col < ncols;
  float2* hbuf = lds + wave * C_::STRIDE;
  int* hcnt = UNI ? lcnt + wave * H : nullptr;
  unsigned* lclaim = reinterpret_cast<unsigned*>(lcnt + (UNI ? CPW * H : 0));
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const float2* tw = stage_twiddles<N, C_::CL>(ltw);
  // the only workgroup barrier: it publishes the LDS twiddles; after it every
  // wavefront grids and transforms its column without waiting for the others
  if (TwLds<N>::ON) __syncthreads();

  ColSpan span{0, 0, 0, 0};
  if (active) {
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    span = ColSpan{bnd[col + H], bnd[col + 1 + H], bnd[-col + H], bnd[-col + 1 + H]};
  }
  // the rest is compiled once per zero band of the first stage and chosen per
  // workgroup (all of its columns belong to one image)
  auto body = [&](auto zbc) {
    constexpr int ZB = decltype(zbc)::value;
    HalfIn<N> in;
    int kd = 0, kc = 0, occ = 0;
    Claim<C_::SLOTS> cl = claim_init<C_::SLOTS>(lclaim + wave * C_::SLOTS, lane);
    if (a.sd != nullptr) grid_col_half<N, true, UNI, ZB>(a, span, hbuf, hcnt, in, t, ch, s, lane, kd, kc, occ, cl);
    else grid_col_half<N, false, UNI, ZB>(a, span, hbuf, hcnt, in, t, ch, s, lane, kd, kc, occ, cl);
    // baselines counted once: the direct entry of every cell column, plus the
    // conjugate entries of columns whose mirror the image path never visits
    const int kept_b = kd + (col > 0 ? kc : 0);
    const int mult = col > 0 ? 2 : 1;
    int wcontrib;
    if (UNI) {
      for (int o = WAVE / 2; o > 0; o >>= 1) occ += __shfl_xor(occ, o);
      wcontrib = mult * occ;
    } else {
      wcontrib = mult * (kd + kc);
    }
    if (lane == 0 && col < H) { *wslot = wcontrib; *kslot = kept_b; }
    if (active) {
      // rows of the cutout straight from the last stage: output row m holds
      // v-frequency q = (m - M/2) mod N
      float2* dst = a.half + ((size_t)li * H + col) * a.M;
      const int hm = HMC > 0 ? HMC : a.M / 2;
      wave_fft_half_emit<N, +1, ZB, C_::CL>(hbuf, lane, tw, in, [&](auto qb, float2 v) {
        cutout_block<N, decltype(qb)::value>(lane, hm, [&](unsigned m) { store_at(dst, m, v); });
      });
    }
  };
  if (HalfIn<N>::R == 16 && column_zero_band<N>(a, t, s) >= 4) body(ic<HalfIn<N>::R == 16 ? 4 : 0>{});
  else body(ic<0>{});
}

// The gridding call's column kernel (nearest cell, all N columns): a wavefront a
// column, 16 columns a workgroup (N <= 1024), so that a row of the tile is a whole
// 128-byte line of the grid; tiles beyond the outermost baseline write zeros
// without passing through LDS. Up to N = 512 the columns lie whole in LDS (32
// images of 512^2 with 8,128 baselines 62 -> 60 us against two halves in turn, 4
// with 32,640 at 51 different u 346 -> 251). Beyond, a wavefront grids one half of
// the rows at a time and the workgroup writes each half. Columns of more than GU x
// 64 entries are walked once a half; tiles with one of more than LONG take half of
// their columns at a time instead, whole ones in two buffers each (in half lines:
// with a few hundred entries a column the halves are faster, 184 against 195 us
// for 32 images of 1024^2 with 32,640 baselines).
// Bound by the 12 bytes a cell that it writes: 32 images of 1024^2 126 -> 97 us,
// 4.2 TB/s (146 us with 8 columns).
template <int N>
struct GridWr {
  static constexpr bool WHOLE = N <= 512;
  static constexpr int LONG = 8 * GU * WAVE;
  static constexpr int CPW = N <= 8 ? 8 : N <= 1024 ? 16 : N <= 2048 ? 8 : 4, THREADS = CPW * WAVE;
  static constexpr int ROWS = WHOLE ? N : N / 2;             // of a column's buffer
  static constexpr int STRIDE = padded_len(ROWS);
  static constexpr int SLOTS = claim_slots(ROWS);
  static constexpr size_t LDS = (size_t)CPW * (STRIDE * sizeof(float2) + ROWS * sizeof(int) + SLOTS * sizeof(unsigned));
  static_assert(WHOLE || padded_len(N) <= 2 * STRIDE, "two buffers hold a whole column");
};

template <int N, bool UNI>
__global__ void __launch_bounds__(GridWr<N>::THREADS) k_grid_write(ImgArgs a) {
  using G_ = GridWr<N>;
  constexpr int H = N / 2, CPW = G_::CPW, ROWS = G_::ROWS;
  extern __shared__ float4 lds_raw[];
  __shared__ int red[2 * CPW];
  const int L = blockIdx.x;
  const int r8 = L >> 3;
  const int li = (r8 / a.ntiles) * 8 + (L & 7);
  const int tile = r8 % a.ntiles;
  if (li >= a.nimg) return;                          // padding of the last group of 8 images
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  int* lcnt = reinterpret_cast<int*>(lds + CPW * G_::STRIDE);
  unsigned* lclaim = reinterpret_cast<unsigned*>(lcnt + CPW * ROWS);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int c0 = tile * CPW, ncol = min(CPW, N - c0);
  const int nz = min(H, a.ncz[img]);
  float2* g = a.grid + (size_t)img * N * N + c0;
  int* gc = a.counts ? a.counts + (size_t)img * N * N + c0 : nullptr;
  if (c0 >= nz && c0 + ncol - 1 <= N - nz) {         // every column |c| >= nz: empty
    for (int e = threadIdx.x; e < N * CPW; e += G_::THREADS) {
      const int r = e / CPW, w = e % CPW;
      if (w < ncol) {
        g[(size_t)r * N + w] = make_float2(0.f, 0.f);
        if (gc) gc[(size_t)r * N + w] = 0;
      }
    }
    if (threadIdx.x == 0) {
      a.wpart[(size_t)img * a.wstride + tile] = 0;
      a.kpart[(size_t)img * a.wstride + tile] = 0;
    }
    return;
  }
  const int col = c0 + wave, cs = col < H ? col : col - N;   // signed u cell
  ColSpan span{0, 0, 0, 0};
  if (col < N && cs != -H) {
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    span = ColSpan{bnd[cs + H], bnd[cs + 1 + H], bnd[-cs + H], bnd[-cs + 1 + H]};
  }
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  int kd = 0, kc = 0, occ = 0;
  Claim<G_::SLOTS> cl = claim_init<G_::SLOTS>(lclaim + wave * G_::SLOTS, lane);
  // rows [r0, r0 + rows) of columns [w0, w0 + cols) of the tile, column w0 + w from buffer w of `stride`
  auto write = [&](int r0, auto rows, int w0, auto cols, int stride) {
    constexpr int RW = decltype(rows)::value, CW = decltype(cols)::value;
    __syncthreads();
    for (int e = threadIdx.x; e < RW * CW; e += G_::THREADS) {
      const int r = e / CW, w = e % CW;
      if (w0 + w < ncol) {
        g[(size_t)(r0 + r) * N + w0 + w] = lds[w * stride + pad(r)];
        if (gc) gc[(size_t)(r0 + r) * N + w0 + w] = lcnt[w * RW + r];
      }
    }
    __syncthreads();
  };
  auto whole = [&](float2* buf, int* cnt) {                  // the wavefront's column, all rows
    for (int r = lane; r < padded_len(N); r += WAVE) buf[r] = make_float2(0.f, 0.f);
    for (int r = lane; r < N; r += WAVE) cnt[r] = 0;
    wave_sync();
    grid_steps<N, true>(a, span, 0, buf, cnt, t, ch, s, lane, kd, kc, cl);
    wave_sync();
    if (UNI) occ += uniform_half<2 * N>(buf, cnt, lane);     // (all N rows)
  };
  if constexpr (G_::WHOLE) {
    whole(lds + wave * G_::STRIDE, lcnt + wave * N);
    write(0, ic<N>{}, 0, ic<CPW>{}, G_::STRIDE);
  } else {
    // every wavefront asks for the tile's entries and, where they are many, for those
    // of all its columns, so that they agree without a barrier
    static_assert(H % CPW == 0, "a tile lies on one side of column N / 2");
    float2* hbuf = lds + wave * G_::STRIDE;
    int* hcnt = lcnt + wave * H;
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    const int u0 = c0 < H ? c0 : c0 - N;
    const int inside = bnd[u0 + CPW + H] - bnd[u0 + H] + bnd[-u0 + 1 + H] - bnd[-u0 - CPW + 1 + H];
    bool few = inside <= G_::LONG;
    if (!few) {
      const int c = u0 + lane;
      few = __ballot(lane < CPW && c != -H &&
                     bnd[c + 1 + H] - bnd[c + H] + bnd[-c + 1 + H] - bnd[-c + H] > G_::LONG) == 0ull;
    }
    if (!few) {
      constexpr int HC = CPW / 2;
      for (int part = 0; part < 2; ++part) {
        if (wave / HC == part) whole(lds + wave % HC * 2 * G_::STRIDE, lcnt + wave % HC * N);
        write(0, ic<N>{}, part * HC, ic<HC>{}, 2 * G_::STRIDE);
      }
    } else {
      auto half = [&](auto hf) { write(decltype(hf)::value * H, ic<H>{}, 0, ic<CPW>{}, G_::STRIDE); };
      if (a.sd != nullptr) grid_halves<N, true, UNI, true>(a, span, hbuf, hcnt, t, ch, s, lane, kd, kc, occ, cl, half);
      else grid_halves<N, false, UNI, true>(a, span, hbuf, hcnt, t, ch, s, lane, kd, kc, occ, cl, half);
    }
  }
  for (int o = WAVE / 2; o > 0; o >>= 1) occ += __shfl_xor(occ, o);
  // baselines are counted once: the direct entry of every column
  if (lane == 0) { red[wave] = UNI ? occ : kd + kc; red[CPW + wave] = kd; }
  __syncthreads();
  if (threadIdx.x == 0) {
    int ws = 0, ks = 0;
    for (int i = 0; i < CPW; ++i) { ws += red[i]; ks += red[CPW + i]; }
    a.wpart[(size_t)img * a.wstride + tile] = ws;
    a.kpart[(size_t)img * a.wstride + tile] = ks;
  }
}

// Weight sums and dropped baselines of the gridding call, a wavefront an image.
__global__ void __launch_bounds__(256) k_grid_finish(ImgArgs a, int n_img) {
  const int img = blockIdx.x * (256 / WAVE) + (int)(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  if (img >= n_img) return;
  const int k = sum_partials(a.kpart, img, a.wstride, a.wtiles, lane);
  const float w = a.kw > 0 ? sum_partials_f(a.wpart, img, a.wstride, a.wtiles, lane)   // kernel gridding: FP32 sums
                           : (float)sum_partials(a.wpart, img, a.wstride, a.wtiles, lane);
  if (lane == 0) {
    if (a.weight_sum) a.weight_sum[img] = w;
    if (a.n_dropped) a.n_dropped[img] = a.n_unflagged[img / a.C] - k;
  }
}

// ============================================================== row pass
template <int N>
struct Rows {
  // buffer stride of 4 mod 32 complex: the workgroup's PPW buffers start on
  // different bank groups, so filling them side by side is conflict-free
  static constexpr int STRIDE = padded_len(N) + ((4 - padded_len(N) % 32) + 32) % 32;
  static constexpr int PPW = N <= 1024 ? 8 : (N <= 2048 ? 4 : 2);  // row pairs (waves) per WG
  static constexpr int THREADS = PPW * WAVE;
  static constexpr int TW = TwLds<N>::ON ? tw_entries(N) : 0;
  static constexpr size_t LDS = (size_t)(PPW * STRIDE + TW) * sizeof(float2);
};

// Inverse transform along u of two cutout rows per wavefront. The half
// spectrum A[k] (k < N/2) of row m and B[k] of row m+1 are packed as
// Z = A_full + i B_full with the Hermitian extensions A_full[N-k] = conj A[k]
// (A_full[N/2] = 0: the Nyquist column is never gridded), so one complex
// transform yields row m as Re z and row m+1 as Im z. The shift, 1/W and the
// cutout are applied as the rows are stored.
// Persistent form: a fixed grid of workgroups walks the (image, row tile)
// list. For N <= 1024, while the transforms of one tile run, the
// half-spectrum slice of the next tile is already in flight into registers,
// so the HBM latency of the loads hides behind the arithmetic of the previous
// tile (larger N would need too many registers and loads per tile instead).
// AL: the cutout half-width M/2 is a multiple of the wavefront width and the
// plan's last-stage blocks are aligned (blocks_aligned), so each block of 64
// output columns is stored or skipped whole.
// KB: the image was gridded with the Kaiser-Bessel kernel; the stores apply
// its correction.
template <int N, bool AL, bool KB>
__global__ void __launch_bounds__(Rows<N>::THREADS) k_rows(ImgArgs a) {
  static_assert(!AL || blocks_aligned(N), "aligned cutout needs aligned blocks");
  extern __shared__ float4 lds_raw[];
  constexpr int H = N / 2;
  constexpr int PPW = Rows<N>::PPW;
  constexpr int ST = Rows<N>::STRIDE;
  constexpr int THR = Rows<N>::THREADS;
  constexpr int EPT = (H * PPW + THR - 1) / THR;     // half-spectrum float4 loads per thread
  constexpr bool PREF = EPT <= 8;
  constexpr int NPRE = PREF ? EPT : 1;
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int M = a.M;
  const int npair = M / 2;
  const int ntr = (npair + PPW - 1) / PPW;           // row tiles per image
  const int total = a.nimg * ntr;
  const float2* tw = stage_twiddles<N>(lds + PPW * ST);
  // kernel gridding: 1 / c((l - M/2) / N) per image column l (the same table
  // serves the rows: the correction is separable), published by the first
  // barrier of the loop
  float* lcorr = reinterpret_cast<float*>(lds + PPW * ST + Rows<N>::TW);
  constexpr bool kbon = KB;
  if (kbon)
    for (int l = threadIdx.x; l < a.M; l += THR) lcorr[l] = kb_inv_taper((double)(l - a.M / 2) / N, a);

  // thread t always serves pair slot t % PPW and columns t / PPW + i * (THR / PPW)
  const int kt = threadIdx.x / PPW, pt = threadIdx.x % PPW;
  auto load = [&](int tile, int i) -> float4 {
    const int li = tile / ntr, p0 = (tile % ntr) * PPW;
    const int nz = min(H, a.ncz[a.img0 + li]);
    const int k = kt + i * (THR / PPW);
    const float4* src = reinterpret_cast<const float4*>(a.half + (size_t)li * H * M) + (p0 + pt);
    return (k < nz && p0 + pt < npair) ? src[(size_t)k * (M / 2)] : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  float4 pre[NPRE];
  int tile = blockIdx.x;
  if (PREF && tile < total) {
#pragma unroll
    for (int i = 0; i < NPRE; ++i) pre[i] = load(tile, i);
  }
#pragma nounroll
  for (; tile < total; tile += gridDim.x) {
    // lane-dependent addresses are recomputed inside the loop: hoisted out of
    // it they would stay live across the transforms and cost occupancy
    int lane_i = lane, ln = threadIdx.x;
    asm volatile("" : "+v"(lane_i), "+v"(ln));
    const int li = tile / ntr, p0 = (tile % ntr) * PPW;
    const int img = a.img0 + li;
    const float W = kbon ? sum_partials_f(a.wpart, img, a.wstride, a.wtiles, lane_i)
                         : (float)sum_partials(a.wpart, img, a.wstride, a.wtiles, lane_i);
    const float scale = a.norm ? (W > 0 ? 1.0f / W : 0.0f) : 1.0f;
    if (p0 == 0 && ln == 0 && a.weight_sum) a.weight_sum[img] = W;
    const int kti = ln / PPW, pti = ln % PPW;
    __syncthreads();                                  // previous tile's rows have left LDS
    auto put = [&](int i, float4 ab) {
      const int k = kti + i * (THR / PPW);
      float2* z = lds + pti * ST;
      if (k == 0) {
        z[pad(0)] = make_float2(ab.x, ab.z);
        z[pad(H)] = make_float2(0.f, 0.f);
      } else {
        z[pad(k)] = make_float2(ab.x - ab.w, ab.y + ab.z);
        z[pad(N - k)] = make_float2(ab.x + ab.w, ab.z - ab.y);
      }
    };
    if constexpr (PREF) {
#pragma unroll
      for (int i = 0; i < NPRE; ++i)
        if (kti + i * (THR / PPW) < H) put(i, pre[i]);
    } else {
      for (int i = 0; kti + i * (THR / PPW) < H; ++i) put(i, load(tile, i));
    }
    __syncthreads();
    if (PREF && tile + (int)gridDim.x < total) {
#pragma unroll
      for (int i = 0; i < NPRE; ++i) pre[i] = load(tile + gridDim.x, i);
    }
    const int pair = p0 + wave;
    if (pair < npair) {
      float2* z = lds + wave * ST;
      float* r0 = a.images + ((size_t)img * M + 2 * pair) * M;
      float* r1 = r0 + M;
      float s0 = scale, s1 = scale;
      if (kbon) {
        s0 *= lcorr[2 * pair];
        s1 *= lcorr[2 * pair + 1];
      }
      int hm = M / 2;
      asm volatile("" : "+s"(hm));   // block tests stay inside the loop (hoisted they spill)
      // image columns of the cutout straight from the last stage: column l
      // holds u-frequency q = (l - M/2) mod N; row 2p is Re z, row 2p+1 is Im z
      wave_fft_emit<N, +1>(z, lane_i, tw, [&](auto qb, float2 v) {
        auto st = [&](unsigned l) {
          const float cl = kbon ? lcorr[l] : 1.0f;
          store_at(r0, l, v.x * s0 * cl);
          store_at(r1, l, v.y * s1 * cl);
        };
        if constexpr (AL) cutout_block_aligned<N, decltype(qb)::value>(lane_i, hm, st);
        else cutout_lane<N, decltype(qb)::value>(lane_i, hm, st);
      });
    }
  }
}

// Row pass with the transforms' exchanges through half-length LDS buffers
// (see wave_fft_half_emit): the same packing, shift, 1/W, cutout and stores
// as k_rows, and the same tiling (one workgroup per row tile, or a
// persistent grid walking the tiles). The workgroup fills the lower halves
// of its PPW packed rows (z[k], k < N/2) from one load of the half-spectrum
// slice, each wavefront takes its first stage's lower inputs, then the upper
// halves (z[N - k]) follow from the same registers. With no prefetch across
// tiles and half the LDS, three workgroups share a CU instead of two.
// Below N = 1024 a row pair takes N / 16 lanes (one first-stage butterfly each)
// instead of a wavefront of which the others would idle, and a workgroup of 128
// or 256 threads as many pairs: 2,000 images of 128^2 110 -> 40 us, 1,000 of
// 512^2 -> 256^2 197 -> 136 us.
template <int N>
struct RowsHalf {
  static constexpr int STRIDE = padded_len(N / 2) + ((4 - padded_len(N / 2) % 32) + 32) % 32;
  static constexpr int L = N / 16 < WAVE ? N / 16 : WAVE;      // lanes per row pair
  // at N = 2048 16 pairs, so that a column's slice is 256 contiguous bytes (128
  // images of 2048^2 960 -> 930 us; at N = 1024 8 are better, 397 against 517)
  static constexpr int THREADS = N == 2048 ? 1024 : N == 1024 ? 512 : N <= 256 ? 128 : 256;
  static constexpr int PPW = THREADS / L;                      // row pairs per workgroup
  static constexpr int TW = TwLds<N>::ON ? tw_entries(N) : 0;
  static constexpr size_t LDS = (size_t)(PPW * STRIDE + TW) * sizeof(float2);
};

// threadIdx.x of a workgroup of whole wavefronts, formed anew from the wavefront's
// number (in a scalar register) where it is asked for, so that no vector register
// keeps it.
__device__ __forceinline__ int thread_number(int wave) {
  int seed = 0;
  asm volatile("" : "+s"(seed));
  return wave * WAVE + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (unsigned)seed));
}

// HMC > 0: the cutout half-width fixed at compile time (see k_grid_cols_half).
template <int N, bool AL, bool KB, int HMC = 0>
__global__ void __launch_bounds__(RowsHalf<N>::THREADS) k_rows_half(ImgArgs a) {
  static_assert(!AL || blocks_aligned(N), "aligned cutout needs aligned blocks");
  extern __shared__ float4 lds_raw[];
  constexpr int H = N / 2;
  constexpr int PPW = RowsHalf<N>::PPW, L = RowsHalf<N>::L;
  constexpr int WAVES = RowsHalf<N>::THREADS / WAVE;
  __shared__ int wred[WAVES];                        // per-wavefront sums of the weight partials
  constexpr int ST = RowsHalf<N>::STRIDE;
  constexpr int THR = RowsHalf<N>::THREADS;
  constexpr int EPT = H / L;                         // half-spectrum float4 loads per thread
  static_assert(H % L == 0 && THR == PPW * L, "a tile's slice is whole columns");
  // At 2048 the 128 registers of 1,024 threads are few: the thread's number and the
  // scales stay out of vector registers. At 1024 there is nothing to save, and it
  // costs 1.3% (7,680 images: 3.72 ms against 3.77).
  constexpr bool FEW = N > 1024;
  static_assert(!FEW || L == WAVE, "a wavefront a row pair");
  constexpr int R0 = HalfIn<N, L>::R;
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int M = HMC > 0 ? 2 * HMC : a.M;
  const int npair = M / 2;
  const int ntr = (npair + PPW - 1) / PPW;           // row tiles per image
  const int total = a.nimg * ntr;
  const float2* tw = stage_twiddles<N>(lds + PPW * ST);
  float* lcorr = reinterpret_cast<float*>(lds + PPW * ST + RowsHalf<N>::TW);
  if (KB)
    for (int l = threadIdx.x; l < a.M; l += THR) lcorr[l] = kb_inv_taper((double)(l - a.M / 2) / N, a);

#pragma nounroll
  for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
    // lane-dependent addresses are formed inside the loop: hoisted out of it
    // they would stay live across the transforms and cost occupancy
    int ln, lane_i;
    if constexpr (FEW) {
      ln = thread_number(wave);
      lane_i = ln % L;
    } else {
      ln = threadIdx.x;
      lane_i = ln % L;
      asm volatile("" : "+v"(lane_i), "+v"(ln));
    }
    auto thread = [&]() { return FEW ? thread_number(wave) : ln; };
    const int vec = L == WAVE ? wave : ln / L;       // this lane's row pair of the tile
    // thread t serves pair slot t % PPW and columns t / PPW + i L; the masks tell
    // the compiler the ranges, so that only i = 0 is ever column 0, and the slots
    // step by constants (pad is linear in steps of 16): 17% fewer vector and half the
    // scalar instructions of a kernel that they bound. Rows of 3,072 images 1024^2 ->
    // 512^2 1,497 -> 1,423 us, 128 of 2048^2 930 -> 893, 384 kernel-gridded 216 -> 200
    const int kt = (ln & (THR - 1)) / PPW, pt = ln & (PPW - 1);
    constexpr bool LIN = L % 16 == 0;
    constexpr int PS = L + L / 16;
    auto lower = [&](int i) { return LIN ? pad(kt) + i * PS : pad(kt + i * L); };
    auto upper = [&](int i) { return LIN ? pad(H - kt) - i * PS : pad(H - kt - i * L); };
    const int li = tile / ntr, p0 = (tile % ntr) * PPW;
    const int img = a.img0 + li;
    const int nz = min(H, a.ncz[img]);               // u cells >= nz are empty
    // the rest of the tile is compiled once per zero band of the first stage
    // and chosen per tile (all of its rows belong to one image)
    auto body = [&](auto zbc) {
      constexpr int ZB = decltype(zbc)::value;
      float4 ab[EPT];
      {
        const float4* src = reinterpret_cast<const float4*>(a.half + (size_t)li * H * M) + p0;
        const unsigned at = (unsigned)(kt * (M / 2) + pt);
        const int nzp = p0 + pt < npair ? nz : 0;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          const unsigned step = (unsigned)(i * L * (M / 2));
          const bool on = kt + i * L < nzp;
          if (HMC > 0) ab[i] = on ? load_at(src + step, at) : make_float4(0.f, 0.f, 0.f, 0.f);
          else ab[i] = on ? load_at(src, at + step) : make_float4(0.f, 0.f, 0.f, 0.f);   // (16 bases would spill)
        }
      }
      // the image's weight sum W from its partials (integers, or FP32 sums with
      // a gridding kernel), split over the workgroup and combined in LDS
      int wli = 0;
      float wlf = 0.f;
      for (int i = thread(); i < a.wtiles; i += THR) {
        const int pv = a.wpart[(size_t)img * a.wstride + i];
        wli += pv;
        wlf += __int_as_float(pv);
      }
      for (int o = WAVE / 2; o > 0; o >>= 1) {
        if (KB) wlf += __shfl_xor(wlf, o);
        else wli += __shfl_xor(wli, o);
      }
      float2* zs = lds + pt * ST;                       // the packed row this thread fills
      float2* z = lds + vec * ST;                       // the packed row its lanes transform
      HalfIn<N, L> in;
      __syncthreads();                                  // previous tile's rows have left LDS
      if (thread() % WAVE == 0) wred[wave] = KB ? __float_as_int(wlf) : wli;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {                   // lower half: z[k] = A[k] + i B[k]
        const float4 v = ab[i];
        zs[lower(i)] = i == 0 && kt == 0 ? make_float2(v.x, v.z) : make_float2(v.x - v.w, v.y + v.z);
      }
      __syncthreads();
      float W;
      if (KB) {
        float f = 0.f;
        for (int w = 0; w < WAVES; ++w) f += __int_as_float(wred[w]);
        W = f;
      } else {
        int n = 0;
        for (int w = 0; w < WAVES; ++w) n += wred[w];
        W = (float)n;
      }
      const float scale = a.norm ? (W > 0 ? 1.0f / W : 0.0f) : 1.0f;
      if (p0 == 0 && thread() == 0 && a.weight_sum) a.weight_sum[img] = W;
      half_read<N, R0, 0, ZB, L>(z, lane_i, in.v);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < EPT; ++i) {                   // upper half: z[N - k] = conj A[k] + i conj B[k]
        const float4 v = ab[i];
        const bool nyq = i == 0 && kt == 0;             // (never gridded)
        zs[nyq ? 0 : upper(i)] = nyq ? make_float2(0.f, 0.f) : make_float2(v.x + v.w, v.z - v.y);
      }
      __syncthreads();
      half_read<N, R0, 1, ZB, L>(z, lane_i, in.v);
      const int pair = p0 + vec;
      if (pair < npair) {
        float* r0 = a.images + ((size_t)img * M + 2 * pair) * M;
        float* r1 = r0 + M;
        float s0 = scale, s1 = scale;
        if (KB) {
          s0 *= lcorr[2 * pair];
          s1 *= lcorr[2 * pair + 1];
        }
        if constexpr (FEW) {                            // (one pair a wavefront: scalars)
          s0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s0)));
          s1 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s1)));
        }
        int hm = HMC > 0 ? HMC : M / 2;
        // block tests stay inside the loop (hoisted they spill)
        if constexpr (HMC == 0) asm volatile("" : "+s"(hm));
        // image columns of the cutout straight from the last stage: column l
        // holds u-frequency q = (l - M/2) mod N; row 2p is Re z, row 2p+1 is Im z
        wave_fft_half_emit<N, +1, ZB, false, L, FEW>(z, lane_i, tw, in, [&](auto qb, float2 v) {
          auto st = [&](unsigned l) {
            const float cl = KB ? lcorr[l] : 1.0f;
            store_at(r0, l, v.x * s0 * cl);
            store_at(r1, l, v.y * s1 * cl);
          };
          if constexpr (AL) cutout_block_aligned<N, decltype(qb)::value>(lane_i, hm, st);
          else cutout_lane<N, decltype(qb)::value>(lane_i, hm, st);
        });
      }
    };
    if (R0 == 16 && zero_band(N, nz) >= 4) body(ic<R0 == 16 ? 4 : 0>{});
    else body(ic<0>{});
  }
}

// ============================================================== dynamic spectra
// Transpose of the image cube [T][C][P] to per-pixel time series [P][C][T]
// with the reference image subtracted on the way. One workgroup per tile of
// DS_TT timesteps x DS_PP pixels of one channel: the rows of the tile (and,
// for a mean over K preceding images, the K rows before it) are read with
// consecutive pixels on consecutive lanes, all loads of a thread issued
// before the first is used; the differences are formed per pixel and staged
// in LDS as [pixel][time]; each pixel's series is then written with
// consecutive timesteps on consecutive lanes. VEC moves 16 bytes per lane
// (P and T multiples of 4, 16-byte aligned arrays).
// Grid: one dimension, workgroup L on XCD L mod 8. The channel varies fastest
// among the workgroups of an XCD, and all time tiles of a pixel tile share
// its XCD, so the series of (p, c) and (p, c + 1), adjacent in the output,
// are written close together into the same L2 and leave it as whole lines.
constexpr int DS_TT = 128, DS_PP = 64, DS_THREADS = 256, DS_KMAX = 128;
constexpr int DS_ST = DS_PP + 1;                              // LDS row stride (floats)

// One LDS buffer of min(DS_TT, T) + K rows (a series shorter than a tile
// needs fewer rows, so more workgroups share a CU): the differences overwrite
// the tile's own rows once every thread has read its window, and the stores
// read them back column-wise (the odd stride keeps both directions off a
// single bank). Rows at or beyond T are never read or written.
__host__ __device__ constexpr int dynspec_rows(int t) { return t < DS_TT ? t : DS_TT; }
__host__ __device__ constexpr size_t dynspec_lds(int k, int t) {
  return (size_t)(dynspec_rows(t) + k) * DS_ST * sizeof(float);
}

template <bool VEC>
__global__ void __launch_bounds__(DS_THREADS) k_dynspec(const float* __restrict__ img, int T, int C, long long P,
                                                        int mode, int K, const float* __restrict__ ref,
                                                        float* __restrict__ out, int npt8) {
  extern __shared__ float4 lds_raw[];
  float* rows = reinterpret_cast<float*>(lds_raw);            // [DS_TT + K][DS_ST]
  const long long L = blockIdx.x;
  const long long r8 = L >> 3;
  const int c = (int)(r8 % C);
  const long long u = (r8 / C) * 8 + (L & 7);                // tile: u = time tile * npt8 + pixel tile
  const long long pt = u % npt8;
  const int tt = (int)(u / npt8);
  const long long p0 = pt * DS_PP;
  const int t0 = tt * DS_TT;
  if (p0 >= P || t0 >= T) return;                             // padding of the pixel tiles to 8
  const int r0 = t0 - K;                                      // first row held (may be < 0)
  const int nrows = dynspec_rows(T) + K;
  if constexpr (VEC) {
    constexpr int Q = DS_PP / 4;                              // float4 per row
    constexpr int MAXI = (DS_TT + DS_KMAX) * Q / DS_THREADS;
    float4 v[MAXI];
#pragma unroll
    for (int i = 0; i < MAXI; ++i) {
      const int e = threadIdx.x + i * DS_THREADS;
      const int r = e / Q, q = e % Q;
      const int t = r0 + r;
      const long long p = p0 + 4 * q;
      v[i] = (r < nrows && t >= 0 && t < T && p < P)
                 ? *reinterpret_cast<const float4*>(img + ((long long)t * C + c) * P + p)
                 : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < MAXI; ++i) {
      const int e = threadIdx.x + i * DS_THREADS;
      const int r = e / Q, q = e % Q;
      if (r < nrows) {
        float* d = rows + r * DS_ST + 4 * q;
        d[0] = v[i].x; d[1] = v[i].y; d[2] = v[i].z; d[3] = v[i].w;
      }
    }
  } else {
    for (int e = threadIdx.x; e < nrows * DS_PP; e += DS_THREADS) {
      const int r = e / DS_PP, jj = e % DS_PP;
      const int t = r0 + r;
      const long long p = p0 + jj;
      rows[r * DS_ST + jj] = (t >= 0 && t < T && p < P) ? img[((long long)t * C + c) * P + p] : 0.0f;
    }
  }
  __syncthreads();
  // thread = (pixel j, segment g of the tile's timesteps)
  const int j = threadIdx.x % DS_PP, g = threadIdx.x / DS_PP;
  constexpr int SEG = DS_TT / (DS_THREADS / DS_PP);
  const float rv = (mode == 2 && p0 + j < P) ? ref[(long long)c * P + p0 + j] : 0.0f;
  double win = 0.0;                                           // sum of the k preceding images
  const int ta = t0 + g * SEG;
  if (mode == 1 && ta < T) {
    const int k = min(K, ta);
    for (int s = ta - k; s < ta; ++s) win += (double)rows[(s - r0) * DS_ST + j];
  }
  float dv[SEG];
#pragma unroll
  for (int i = 0; i < SEG; ++i) {
    const int t = ta + i;
    float d = 0.0f;
    if (t < T) {                                              // rows from T on are not held
      const float x = rows[(t - r0) * DS_ST + j];
      if (mode == 0) {
        d = x;
      } else if (mode == 2) {
        d = x - rv;
      } else {
        // mean of the window: 1/k is exact for k a power of two and within an
        // ulp of double otherwise, far below the final rounding to float
        const int k = min(K, t);
        d = t == 0 ? 0.0f : (float)((double)x - win * (1.0 / (double)k));
        // slide the window to end at t: add x, drop the image K behind
        win += (double)x;
        if (t - K >= 0) win -= (double)rows[(t - K - r0) * DS_ST + j];
      }
    }
    dv[i] = d;
  }
  __syncthreads();                                            // every window has been read
#pragma unroll
  for (int i = 0; i < SEG; ++i)
    if (ta + i < T) rows[(ta + i - r0) * DS_ST + j] = dv[i];
  __syncthreads();
  if constexpr (VEC) {
    constexpr int Q = DS_TT / 4;                              // float4 per pixel series
#pragma unroll
    for (int i = 0; i < DS_PP * Q / DS_THREADS; ++i) {
      const int e = threadIdx.x + i * DS_THREADS;
      const int pj = e / Q, q = e % Q;
      const long long p = p0 + pj;
      const int t = t0 + 4 * q;
      if (p < P && t < T) {
        const float* src = rows + (t - r0) * DS_ST + pj;
        *reinterpret_cast<float4*>(out + (p * C + c) * T + t) =
            make_float4(src[0], src[DS_ST], src[2 * DS_ST], src[3 * DS_ST]);
      }
    }
  } else {
    for (int e = threadIdx.x; e < DS_PP * DS_TT; e += DS_THREADS) {
      const int pj = e / DS_TT, tq = e % DS_TT;
      const long long p = p0 + pj;
      const int t = t0 + tq;
      if (p < P && t < T) out[(p * C + c) * T + t] = rows[(t - r0) * DS_ST + pj];
    }
  }
}

// ============================================================== correlator X-engine
// V_ij = sum_s x_i(s) conj(x_j(s)) for 8-bit complex voltages x[t][c][a][s]
// (real r, imaginary q interleaved), on the matrix cores. Along the bytes of an
// antenna's row the two parts are plain integer dot products:
//   Re V_ij = sum r_i r_j + q_i q_j            = X_i . X_j,
//   Im V_ij = sum q_i r_j - r_i q_j            = X_i . Y_j + sum r_i,
// with X = (r, q, r, q, ...) as stored and Y = (~q, r, ~q, r, ...): the byte
// complement ~q = -q - 1 stands in for -q, which a byte cannot hold at
// q = -128, and costs sum r_i, formed beside the products. So the rows need no
// splitting, and a pair takes two accumulators instead of three (RR + QQ, QR
// and RQ of separate real and imaginary matrices); the operations are as many.
// One workgroup of four wavefronts (2 x 2) computes a tile of 2 WT x 2 WT
// antenna pairs (tile row <= tile column) with v_mfma_i32_32x32x32_i8: lane
// (h, m) holds bytes 16 h .. 16 h + 15 of antenna m's 32-byte step, as A and B
// alike, so the products do not depend on how the matrix cores order them.
// Each byte that enters LDS feeds 2 WT pairs. The rows go through LDS in a ring
// of RING stages of CH bytes a row (twice as many for tiles on the diagonal,
// whose A and B rows are one), loaded straight into LDS, all stages but one
// ahead of the products. LDS 16-byte units are permuted within a row so that
// the 16 rows a read touches at once lie on all banks.
// Sums are exact in int32 for up to 65520 samples. The workgroups of one
// (t, c) run on one XCD, so its voltages are read from HBM once.
// WT = 64 feeds the matrix cores from fewer bytes; WT = 32 has four times the
// workgroups, for calls whose large tiles would leave CUs idle.
typedef int xe_v4i __attribute__((ext_vector_type(4)));
typedef int xe_v16i __attribute__((ext_vector_type(16)));
constexpr int XE_THREADS = 256;
// RR + QQ of S samples reaches 2 S 128^2 in magnitude: below 2^31 up to this S
constexpr int XE_MAX_SAMPLES = 65520;

struct XeArgs {
  const int8_t* volt;           // [T][C][A][S][2]
  float2* vis;                  // [T][C][A(A-1)/2]
  float* autos;                 // [T][C][A] or null
  int T, C, A, S;
  int nt;                       // antenna tiles: ceil(A / (2 WT))
  int npairs;                   // nt (nt + 1) / 2 tile pairs per (t, c)
  long long nimg;               // T * C
};

template <int WT>
struct Xe {
  static constexpr int NB = WT / 32;                   // MFMA blocks per wavefront edge
  static constexpr int TILE = 2 * WT;                  // antennas per workgroup edge
  static constexpr int CH = 128;                       // bytes of a row per stage
  static constexpr int UNITS = CH / 16;                // 16-byte units of a row
  static constexpr int ROWS = 2 * TILE;                // A rows, then B rows
  static constexpr int VPT = ROWS * UNITS / XE_THREADS;// units a thread moves per stage
  static constexpr int BUF = ROWS * UNITS;             // units per stage
  static constexpr int RING = WT == 64 ? 2 : 4;        // stages (twice as many on the diagonal)
  static constexpr size_t LDS = RING * (size_t)BUF * 16;      // 64 KiB: the reach of a load's LDS offset
  static_assert(VPT * RING <= 16 && LDS <= 65536, "xe_wait counts up to 12 loads");
  // place of unit c of row r, and the unit at place c (the same permutation):
  // a row covers half of the banks
  __device__ static int unit(int r, int c) { return r * UNITS + (c ^ ((r >> 1) & 7)); }
};

// 16 bytes a lane from memory to LDS at byte `at` + 16 lane (wave-uniform
// `at`). No register receives the data; xe_wait counts these loads.
__device__ __forceinline__ void xe_load_lds(const int8_t* p, unsigned at) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(at), "v"(p) : "memory", "m0");
}
// Waits until at most `left` of this wavefront's loads are in flight, and for its LDS operations.
__device__ __forceinline__ void xe_wait(int left) {
  switch (left) {
    case 12: asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" : : : "memory"); break;
    case 10: asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)" : : : "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" : : : "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)" : : : "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" : : : "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)" : : : "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory"); break;
  }
}

template <int WT>
__global__ void __launch_bounds__(XE_THREADS, 2) k_xengine(XeArgs a) {
  using X_ = Xe<WT>;
  constexpr int NB = X_::NB, TILE = X_::TILE, CH = X_::CH, UNITS = X_::UNITS, VPT = X_::VPT, BUF = X_::BUF;
  extern __shared__ float4 lds_raw[];                         // alone: 64 KiB from LDS offset 0
  const long long L = blockIdx.x;
  const long long r8 = L >> 3;
  const long long img = (r8 / a.npairs) * 8 + (L & 7);
  if (img >= a.nimg) return;                                  // padding of the last group of 8
  int pr = (int)(r8 % a.npairs);
  int ti = 0;                                                 // tile pair -> (ti <= tj)
  while (pr >= a.nt - ti) { pr -= a.nt - ti; ++ti; }
  const int tj = ti + pr;
  const bool diag = ti == tj;                                 // A and B are the same rows
  const int tid = threadIdx.x, lane = tid % WAVE, wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int wi = wave >> 1, wj = wave & 1;
  const int i0 = ti * TILE + wi * WT, j0 = tj * TILE + wj * WT;   // first antennas of the wavefront's tile
  const bool active = i0 < a.A && j0 < a.A && i0 < j0 + WT;  // else nothing above the diagonal
  const int bytes = a.S * 2;                                  // per antenna row
  const int8_t* base = a.volt + (size_t)img * a.A * bytes;
  uint4* lds = reinterpret_cast<uint4*>(lds_raw);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)lds_raw;

  // this thread's units of a stage: places tid + 256 v, i.e. rows tid / UNITS +
  // v 256 / UNITS. Rows beyond the array read antenna A - 1: their products are
  // not stored.
  const int nv = diag ? VPT / 2 : VPT;
  const int ring = diag ? 2 * X_::RING : X_::RING, buf = diag ? BUF / 2 : BUF;   // stages, units per stage
  const int8_t* src[VPT];
  int col[VPT];                                               // first byte of the unit in its row
#pragma unroll
  for (int v = 0; v < VPT; ++v) {
    const int r = (tid + v * XE_THREADS) / UNITS;
    const int ant = r < TILE ? ti * TILE + r : tj * TILE + (r - TILE);
    col[v] = (X_::unit(r, tid % UNITS) - r * UNITS) * 16;
    src[v] = base + (size_t)min(ant, a.A - 1) * bytes + col[v];
  }
  const int nch = (bytes + CH - 1) / CH;
  auto issue = [&](int ch) {                                  // stage ch mod ring is free
    const int k0 = ch * CH;
    const unsigned st = (unsigned)((ch & (ring - 1)) * buf);
#pragma unroll
    for (int v = 0; v < VPT; ++v)
      if (v < nv) {
        const unsigned at = lds0 + (st + (unsigned)(v * XE_THREADS + wave * WAVE)) * 16u;
        if (k0 + CH <= bytes) {
          xe_load_lds(src[v] + k0, at);
        } else {                                              // the row ends in this stage: zeros beyond
          if (k0 + col[v] < bytes) xe_load_lds(src[v] + k0, at);
          else lds[st + v * XE_THREADS + tid] = make_uint4(0u, 0u, 0u, 0u);
        }
      }
  };

  xe_v16i re[NB][NB], im[NB][NB];
  int rsum[NB];
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    rsum[x] = 0;
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) re[x][y][e] = im[x][y][e] = 0;
  }
  const int h = lane >> 5, m = lane & 31;
  const int arow = wi * WT + m, brow = (diag ? 0 : TILE) + wj * WT + m;
  for (int ch = 0; ch < ring - 1 && ch < nch; ++ch) issue(ch);
  for (int ch = 0; ch < nch; ++ch) {
    // this stage has arrived (at most the ring - 2 after it are in flight), and all
    // wavefronts are done with the stage before it, which the next loads fill
    xe_wait(min(ring - 2, nch - 1 - ch) * nv);
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    if (ch + ring - 1 < nch) issue(ch + ring - 1);
    if (active) {
      const uint4* b = lds + (ch & (ring - 1)) * buf;
#pragma unroll
      for (int st = 0; st < CH / 32; ++st) {
        xe_v4i xa[NB], xb[NB], yb[NB];
#pragma unroll
        for (int x = 0; x < NB; ++x) {
          const uint4 u = b[X_::unit(arow + 32 * x, 2 * st + h)];
          xa[x] = xe_v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) rsum[x] = __builtin_amdgcn_sdot4(xa[x][e], 0x00010001, rsum[x], false);
        }
#pragma unroll
        for (int y = 0; y < NB; ++y) {
          const uint4 u = b[X_::unit(brow + 32 * y, 2 * st + h)];
          xb[y] = xe_v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
#pragma unroll
          for (int e = 0; e < 4; ++e)                         // (r, q) -> (~q, r)
            yb[y][e] = (int)(__builtin_amdgcn_perm(0u, (unsigned)xb[y][e], 0x02030001u) ^ 0x00ff00ffu);
        }
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int y = 0; y < NB; ++y) {
            if (x > y && i0 == j0) continue;                  // wholly below the diagonal
            re[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa[x], xb[y], re[x][y], 0, 0, 0);
            im[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa[x], yb[y], im[x][y], 0, 0, 0);
          }
      }
    }
  }
  // sum r_i of the wavefront's rows: both lane halves of a row (the ring is free)
  __syncthreads();
  int* s_rsum = reinterpret_cast<int*>(lds_raw);
#pragma unroll
  for (int x = 0; x < NB; ++x) {
    const int v = rsum[x] + __shfl_xor(rsum[x], 32);
    if (active && h == 0) s_rsum[wi * WT + 32 * x + m] = v;  // (both wj write the same values)
  }
  __syncthreads();
  if (!active) return;
  // accumulator element e of lane (h, m) in block (x, y) holds row
  // i = i0 + 32 x + 8 (e / 4) + 4 h + e % 4 and column j = j0 + 32 y + m
  const size_t nbl = (size_t)a.A * (a.A - 1) / 2;
  float2* v = a.vis + (size_t)img * nbl;
#pragma unroll
  for (int x = 0; x < NB; ++x)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int ri = 32 * x + 8 * (e / 4) + 4 * h + e % 4;
      const int i = i0 + ri;
      const int rs = s_rsum[wi * WT + ri];
#pragma unroll
      for (int y = 0; y < NB; ++y) {
        const int j = j0 + 32 * y + m;
        if (j < a.A && i < j) {
          const size_t b = (size_t)i * a.A - (size_t)i * (i + 1) / 2 + (j - i - 1);
          v[b] = make_float2((float)re[x][y][e], (float)(im[x][y][e] + rs));
        } else if (a.autos != nullptr && i == j && j < a.A) {
          a.autos[(size_t)img * a.A + i] = (float)re[x][y][e];
        }
      }
    }
}

// The same products with one workgroup of eight wavefronts per spectrum, for
// arrays of up to 256 antennas (NBR blocks of 32 rows): every byte is fetched
// from L2 once instead of twice, 256 contiguous bytes of a row at a time (with
// 64 bytes of each row at a time HBM gave two thirds of that rate), and only
// the blocks on and above the diagonal are computed. The NBR (NBR + 1) / 2
// blocks are dealt to the wavefronts in row order, each wavefront's list known
// at compile time, so that a wavefront reads its row operand once for several
// blocks. Double-buffered: the next 256 bytes of every row are in flight in
// registers during the products of these.
// 512 spectra of 256 antennas x 4096 samples: 617 -> 375 us (0.55 TOP of the
// definition's 8 operations a pair and sample: 1.5 POP/s; 2.9 TB/s of input),
// against 617 with one wavefront per 64 x 64 tile on split real and imaginary
// bytes. With the matrix cores and the loads both busy the clock falls from 2.2
// to 1.8 GHz; products alone took 366 us of the tile form's 535, loads alone 346.
template <int NBR>
struct XeAll {
  static constexpr int THREADS = 512, WAVES = THREADS / WAVE;
  static constexpr int ROWS = 32 * NBR, CH = 256, UNITS = CH / 16;
  static constexpr int VPT = ROWS * UNITS / THREADS;   // units a thread moves per chunk
  static constexpr int BUF = ROWS * UNITS;             // units per buffer
  static constexpr size_t LDS = 2 * (size_t)BUF * 16;
  static constexpr int TOT = NBR * (NBR + 1) / 2;      // blocks on and above the diagonal
  __host__ __device__ static constexpr int first(int w) { return w * TOT / WAVES; }
  __host__ __device__ static constexpr int row(int b) {
    int r = 0;
    while (b >= NBR - r) { b -= NBR - r; ++r; }
    return r;
  }
  __host__ __device__ static constexpr int col(int b) {
    int r = 0;
    while (b >= NBR - r) { b -= NBR - r; ++r; }
    return r + b;
  }
  __device__ static int unit(int r, int c) { return r * UNITS + (c ^ (r & 15)); }
};

template <int NBR, int W>
__device__ __forceinline__ void xe_all_wave(const XeArgs& a, long long img, uint4* lds) {
  using X_ = XeAll<NBR>;
  constexpr int B0 = X_::first(W), NB = X_::first(W + 1) - B0, VPT = X_::VPT;
  const int tid = threadIdx.x, lane = tid % WAVE;
  const int h = lane >> 5, m = lane & 31;
  const int bytes = a.S * 2;
  const int8_t* base = a.volt + (size_t)img * a.A * bytes;
  // unit tid % UNITS of every 32nd row; rows beyond the array read antenna A - 1
  const int uc = tid % X_::UNITS, ur = tid / X_::UNITS;
  unsigned off[VPT];                                          // A * 2 S < 2^25 bytes
#pragma unroll
  for (int v = 0; v < VPT; ++v) off[v] = (unsigned)min(ur + 32 * v, a.A - 1) * (unsigned)bytes + uc * 16;
  uint4 f[VPT];
  auto fetch = [&](int k0) {
    const bool in = k0 + uc * 16 < bytes;                     // (rows are whole units: 2 S is a multiple of 32)
#pragma unroll
    for (int v = 0; v < VPT; ++v)
      f[v] = in ? *reinterpret_cast<const uint4*>(base + k0 + off[v]) : make_uint4(0u, 0u, 0u, 0u);
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int v = 0; v < VPT; ++v) lds[buf * X_::BUF + X_::unit(ur + 32 * v, uc)] = f[v];
  };
  xe_v16i re[NB > 0 ? NB : 1], im[NB > 0 ? NB : 1];
  int rsum[NB > 0 ? NB : 1];                                  // of the blocks on the diagonal
  static_for<0, NB>([&](auto bc) {
    constexpr int b = decltype(bc)::value;
    rsum[b] = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) re[b][e] = im[b][e] = 0;
  });
  if (bytes > 0) {
    fetch(0);
    stage(0);
  }
  __syncthreads();
  int cur = 0;
  for (int k0 = 0; k0 < bytes; k0 += X_::CH) {
    const bool more = k0 + X_::CH < bytes;
    if (more) fetch(k0 + X_::CH);
    const uint4* buf = lds + cur * X_::BUF;
    auto operand = [&](int blk, int st) {
      const uint4 u = buf[X_::unit(32 * blk + m, 2 * st + h)];
      return xe_v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
    };
#pragma unroll 2
    for (int st = 0; st < X_::CH / 32; ++st) {
      xe_v4i xa;
      static_for<0, NB>([&](auto bc) {
        constexpr int b = decltype(bc)::value, x = X_::row(B0 + b), y = X_::col(B0 + b);
        if constexpr (b == 0 || X_::row(B0 + (b > 0 ? b - 1 : 0)) != x) xa = operand(x, st);
        xe_v4i xb = xa, yb;
        if constexpr (x != y) xb = operand(y, st);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) rsum[b] = __builtin_amdgcn_sdot4(xa[e], 0x00010001, rsum[b], false);
#pragma unroll
        for (int e = 0; e < 4; ++e)                           // (r, q) -> (~q, r)
          yb[e] = (int)(__builtin_amdgcn_perm(0u, (unsigned)xb[e], 0x02030001u) ^ 0x00ff00ffu);
        re[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa, xb, re[b], 0, 0, 0);
        im[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xa, yb, im[b], 0, 0, 0);
      });
    }
    if (more) stage(cur ^ 1);
    __syncthreads();
    cur ^= 1;
  }
  // sum r_i of every row, from the wavefronts that hold the diagonal blocks
  int* s_rsum = reinterpret_cast<int*>(lds);
  static_for<0, NB>([&](auto bc) {
    constexpr int b = decltype(bc)::value, x = X_::row(B0 + b);
    if constexpr (x == X_::col(B0 + b)) {
      const int v = rsum[b] + __shfl_xor(rsum[b], 32);
      if (h == 0) s_rsum[32 * x + m] = v;
    }
  });
  __syncthreads();
  const size_t nbl = (size_t)a.A * (a.A - 1) / 2;
  float2* vis = a.vis + (size_t)img * nbl;
  static_for<0, NB>([&](auto bc) {
    constexpr int b = decltype(bc)::value, x = X_::row(B0 + b), y = X_::col(B0 + b);
    const int j = 32 * y + m;
#pragma unroll
    for (int e = 0; e < 16; ++e) {                            // (accumulator layout as in k_xengine)
      const int i = 32 * x + 8 * (e / 4) + 4 * h + e % 4;
      if (j < a.A && i < j) {
        const unsigned p = (unsigned)i * (unsigned)a.A - (unsigned)i * (i + 1) / 2 + (unsigned)(j - i - 1);
        vis[p] = make_float2((float)re[b][e], (float)(im[b][e] + s_rsum[i]));
      } else if (a.autos != nullptr && i == j && j < a.A) {
        a.autos[(size_t)img * a.A + i] = (float)re[b][e];
      }
    }
  });
}

template <int NBR>
__global__ void __launch_bounds__(XeAll<NBR>::THREADS, NBR <= 4 ? 4 : 2) k_xengine_all(XeArgs a) {
  extern __shared__ float4 lds_raw[];
  uint4* lds = reinterpret_cast<uint4*>(lds_raw);
  const long long img = blockIdx.x;
  switch (__builtin_amdgcn_readfirstlane(threadIdx.x / WAVE)) {   // barriers match across the cases
    case 0: xe_all_wave<NBR, 0>(a, img, lds); break;
    case 1: xe_all_wave<NBR, 1>(a, img, lds); break;
    case 2: xe_all_wave<NBR, 2>(a, img, lds); break;
    case 3: xe_all_wave<NBR, 3>(a, img, lds); break;
    case 4: xe_all_wave<NBR, 4>(a, img, lds); break;
    case 5: xe_all_wave<NBR, 5>(a, img, lds); break;
    case 6: xe_all_wave<NBR, 6>(a, img, lds); break;
    default: xe_all_wave<NBR, 7>(a, img, lds); break;
  }
}

// ============================================================== plain 2D FFT
template <int N>
struct Fft2 {
  static constexpr int STRIDE = padded_len(N) + 4;
  static constexpr int VPW = N <= 1024 ? 8 : (N <= 2048 ? 4 : 2);   // vectors per workgroup
  static constexpr int THREADS = VPW * WAVE;
  static constexpr size_t LDS = (size_t)VPW * STRIDE * sizeof(float2);
};

template <int N, int SIGN>
__global__ void __launch_bounds__(Fft2<N>::THREADS) k_fft_rows(const float2* in, float2* out, int nrows) {
  extern __shared__ float4 lds_raw[];
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const long row = (long)blockIdx.x * Fft2<N>::VPW + wave;
  if (row >= nrows) return;
  float2* z = lds + wave * Fft2<N>::STRIDE;
  const float2* s = in + row * N;
  for (int i = lane; i < N; i += WAVE) z[pad(i)] = s[i];
  wave_sync();
  wave_fft<N, SIGN>(z, lane, TwTable<N>::stages());
  float2* d = out + row * N;
  for (int i = lane; i < N; i += WAVE) d[i] = z[pad(i)];
}

template <int N, int SIGN>
__global__ void __launch_bounds__(Fft2<N>::THREADS) k_fft_cols(float2* data) {
  extern __shared__ float4 lds_raw[];
  constexpr int VPW = Fft2<N>::VPW;
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int c0 = blockIdx.x * VPW;
  float2* img = data + (size_t)blockIdx.y * N * N;
  for (int e = threadIdx.x; e < N * VPW; e += blockDim.x) {
    const int r = e / VPW, w = e % VPW;
    if (c0 + w < N) lds[w * Fft2<N>::STRIDE + pad(r)] = img[(size_t)r * N + c0 + w];
  }
  __syncthreads();
  if (c0 + wave < N) wave_fft<N, SIGN>(lds + wave * Fft2<N>::STRIDE, lane, TwTable<N>::stages());
  __syncthreads();
  for (int e = threadIdx.x; e < N * VPW; e += blockDim.x) {
    const int r = e / VPW, w = e % VPW;
    if (c0 + w < N) img[(size_t)r * N + c0 + w] = lds[w * Fft2<N>::STRIDE + pad(r)];
  }
}

// Power-of-two sizes from 128 to 2048: the same two passes with the exchanges
// through half-length LDS buffers (see wave_fft_half_emit), so that twice the
// wavefronts share a CU, and N / 16 lanes per vector (one first-stage butterfly
// each) instead of 64, several vectors a wavefront where N < 1024. Rows go from
// memory to the first stage's registers and from the last stage's to memory.
// Columns are taken CPW at a time, so that a row of the tile is at least one
// whole 128-byte line (8 columns a workgroup moved half lines); their lower and
// upper halves pass through the same buffers, on the way in and out.
// Bound by memory: two passes over 64 images of 1024^2 (2.1 GB) 685 -> 480 us,
// 4.5 of the 5.1 TB/s that a copy reaches; 256^2 704 -> 400 us and 2048^2 1082 ->
// 497 us for as many bytes.
template <int N>
struct FftHalf {
  static constexpr int L = N / 16 < WAVE ? N / 16 : WAVE;   // lanes per vector
  static constexpr int VPV = WAVE / L;                      // vectors per wavefront
  // columns start on different bank groups (4 mod 32 complex, as the row pass)
  static constexpr int STRIDE = padded_len(N / 2) + ((4 - padded_len(N / 2) % 32) + 32) % 32;
  static constexpr int TW = TwLds<N>::ON ? tw_entries(N) : 0;
  static constexpr int RWAVES = 8, RPW = RWAVES * VPV;      // rows per workgroup
  static constexpr int CPW = 4 * VPV > 16 ? 4 * VPV : 16;   // columns per workgroup
  static constexpr int CWAVES = CPW / VPV;
  static constexpr size_t row_lds() { return (size_t)(RPW * STRIDE + TW) * sizeof(float2); }
  static constexpr size_t col_lds() { return (size_t)(CPW * STRIDE + TW) * sizeof(float2); }
};
template <int N>
constexpr bool fft_half() { return plan_even(N) && N >= 128 && N <= 2048; }

template <int N, int SIGN>
__global__ void __launch_bounds__(FftHalf<N>::RWAVES * WAVE) k_fft_rows_half(const float2* in, float2* out, int nrows) {
  using F_ = FftHalf<N>;
  constexpr int L = F_::L, R = HalfIn<N, L>::R, PER = HalfIn<N, L>::PER;
  extern __shared__ float4 lds_raw[];
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int vec = threadIdx.x / L, lane = threadIdx.x % L;  // vector of the workgroup, lane within it
  const long row = (long)blockIdx.x * F_::RPW + vec;
  const float2* s = in + min(row, (long)nrows - 1) * N;     // (spare vectors repeat the last row)
  HalfIn<N, L> x;
#pragma unroll
  for (int p = 0; p < PER; ++p)
#pragma unroll
    for (int r = 0; r < R; ++r) x.v[p][r] = s[lane + L * p + r * (N / R)];
  const float2* tw = stage_twiddles<N>(lds + F_::RPW * F_::STRIDE);
  if (TwLds<N>::ON) __syncthreads();
  float2* d = out + row * N;
  wave_fft_half_emit<N, SIGN, 0, false, L>(lds + vec * F_::STRIDE, lane, tw, x, [&](auto qb, float2 v) {
    if (row < nrows) d[decltype(qb)::value + lane] = v;
  });
}

template <int N, int SIGN>
__global__ void __launch_bounds__(FftHalf<N>::CWAVES * WAVE) k_fft_cols_half(float2* data) {
  using F_ = FftHalf<N>;
  constexpr int L = F_::L, CPW = F_::CPW, ST = F_::STRIDE, H = N / 2, THR = F_::CWAVES * WAVE;
  constexpr int R = HalfIn<N, L>::R, PER = HalfIn<N, L>::PER;
  constexpr int Q = CPW / 2, ROWS = THR / Q, EPT = H / ROWS;   // float4 of a tile row; rows at once; per thread and half
  static_assert(H % ROWS == 0 && N % CPW == 0, "whole tiles");
  constexpr int RL = pick_radix(N / last_stage_ns(N)), PL = N / RL / L;   // last stage: radix, butterflies per lane
  extern __shared__ float4 lds_raw[];
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int vec = threadIdx.x / L, lane = threadIdx.x % L;
  float4* img = reinterpret_cast<float4*>(data + (size_t)blockIdx.y * N * N + blockIdx.x * CPW);
  const int q = threadIdx.x % Q, r0 = threadIdx.x / Q;
  float4 t[EPT];
  auto load = [&](int half) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) t[e] = img[(size_t)(half * H + r0 + e * ROWS) * (N / 2) + q];
  };
  auto put = [&]() {
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      float2* d = lds + 2 * q * ST + pad(r0 + e * ROWS);
      d[0] = make_float2(t[e].x, t[e].y);
      d[ST] = make_float2(t[e].z, t[e].w);
    }
  };
  auto store = [&](int half) {
    int at = r0 * (N / 2) + q;
    asm volatile("" : "+v"(at));                             // (formed again: kept from the loads, addresses spill at 2048)
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const float2* s = lds + 2 * q * ST + pad(r0 + e * ROWS);
      const float2 a = s[0], b = s[ST];
      store_at(img + (size_t)(half * H + e * ROWS) * (N / 2), (unsigned)at, make_float4(a.x, a.y, b.x, b.y));
    }
  };
  const float2* tw = stage_twiddles<N>(lds + CPW * ST);
  float2* buf = lds + vec * ST;                              // this vector's column
  HalfIn<N, L> x;
  load(0);
  put();
  load(1);
  __syncthreads();
  half_read<N, R, 0, 0, L>(buf, lane, x.v);
  __syncthreads();
  put();
  __syncthreads();
  half_read<N, R, 1, 0, L>(buf, lane, x.v);
  wave_sync();
  float2 up[PL][RL / 2];                                     // the outputs from N / 2 on
  wave_fft_half_emit<N, SIGN, 0, false, L>(buf, lane, tw, x, [&](auto qb, float2 v) {
    constexpr int QB = decltype(qb)::value, r = QB / (N / RL), p = QB % (N / RL) / L;
    if constexpr (QB < H) buf[pad(QB + lane)] = v;
    else up[p][r - RL / 2] = v;
  });
  __syncthreads();
  store(0);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PL; ++p)
#pragma unroll
    for (int r = 0; r < RL / 2; ++r) buf[pad(p * L + r * (N / RL) + lane)] = up[p][r];
  __syncthreads();
  store(1);
}

// ============================================================== adjoint
// Weight sums alone (the adjoint needs 1/W before anything else): counts of
// kept entries (natural) or occupied cells (uniform) per half-spectrum column.
template <int N, bool UNI>
__global__ void __launch_bounds__(Cols<N>::THREADS) k_weights(ImgArgs a) {
  extern __shared__ int lw_raw[];
  __shared__ int red[Cols<N>::CPW];
  constexpr int H = N / 2;
  constexpr int CPW = Cols<N>::CPW;
  const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int li = blockIdx.y;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int cs = blockIdx.x * CPW + wave;
  int w = 0;
  if (cs < min(H, a.ncz[img])) {
    int* cnt = lw_raw + wave * N;
    const double s = cells_per_metre(a.freq[ch], a.ndx);
    if (UNI) {
      for (int r = lane; r < N; r += WAVE) cnt[r] = 0;
      wave_sync();
    }
    const int* bnd = a.bnd + (size_t)img * (N + 2);
    const size_t tb = (size_t)t * a.B;
    int kept = 0;
    for (int pass = 0; pass < 2; ++pass) {
      const int c = pass == 0 ? cs : -cs;
      const int lo = bnd[c + H], hi = bnd[c + 1 + H];
      for (int j = lo + lane; j < hi; j += WAVE) {
        const double iv = rint(a.sv[tb + j] * s);
        if (fabs(iv) < (double)H) {
          ++kept;
          if (UNI) {
            int r = (int)iv;
            if (pass) r = -r;
            atomicAdd(&cnt[r < 0 ? r + N : r], 1);
          }
        }
      }
    }
    w = kept;
    if (UNI) {
      wave_sync();
      int occ = 0;
      for (int r = lane; r < N; r += WAVE) occ += cnt[r] > 0;
      w = occ;
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) w += __shfl_xor(w, o);
    w *= (cs > 0 ? 2 : 1);
  }
  if (lane == 0) red[wave] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    int ws = 0;
    for (int i = 0; i < CPW; ++i) ws += red[i];
    a.wpart[(size_t)img * a.wstride + blockIdx.x] = ws;
  }
}

// Adjoint of k_rows: image-gradient rows m, m+1 (zero outside the cutout,
// times 1/W, shift undone) packed as z = a + i b, forward transform, then the
// half-spectrum gradients c_k A[k], c_k B[k] (c_0 = 1, c_k = 2) with
// A[k] = (Z[k] + conj Z[N-k]) / 2 and B[k] = (Z[k] - conj Z[N-k]) / (2i).
// Only the columns that can hold baselines (k < ncz) are stored.
template <int N>
__global__ void __launch_bounds__(Rows<N>::THREADS) k_rows_adj(ImgArgs a) {
  extern __shared__ float4 lds_raw[];
  constexpr int H = N / 2;
  constexpr int PPW = Rows<N>::PPW;
  constexpr int ST = Rows<N>::STRIDE;
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int li = blockIdx.y;
  const int img = a.img0 + li;
  const int M = a.M;
  const int npair = M / 2;
  const int p0 = blockIdx.x * PPW;
  const int nz = min(H, a.ncz[img]);
  const float W = a.wsum_in ? a.wsum_in[img]
                  : a.kw > 0 ? sum_partials_f(a.wpart, img, a.wstride, a.wtiles, lane)
                             : (float)sum_partials(a.wpart, img, a.wstride, a.wtiles, lane);
  const float scale = a.norm ? (W > 0 ? 1.0f / W : 0.0f) : 1.0f;
  const float2* tw = stage_twiddles<N>(lds + PPW * ST);
  __syncthreads();
  const int pair = p0 + wave;
  if (pair < npair) {
    float2* z = lds + wave * ST;
    for (int r = lane; r < ST; r += WAVE) z[r] = make_float2(0.f, 0.f);
    wave_sync();
    const float* g0 = a.image_grad + ((size_t)img * M + 2 * pair) * M;
    const float* g1 = g0 + M;
    // with a gridding kernel the forward pass divided pixel (m, l) by
    // c(q_m / N) c(q_l / N); that diagonal scaling is its own adjoint
    float s0 = scale, s1 = scale;
    if (a.kw > 0) {
      s0 *= kb_inv_taper((double)(2 * pair - M / 2) / N, a);
      s1 *= kb_inv_taper((double)(2 * pair + 1 - M / 2) / N, a);
    }
    for (int l = lane; l < M; l += WAVE) {
      int q = l - M / 2;
      q = q < 0 ? q + N : q;
      const float cl = a.kw > 0 ? kb_inv_taper((double)(l - M / 2) / N, a) : 1.0f;
      z[pad(q)] = make_float2(g0[l] * s0 * cl, g1[l] * s1 * cl);
    }
    wave_sync();
    wave_fft<N, -1>(z, lane, tw);
  }
  __syncthreads();
  float4* dst = reinterpret_cast<float4*>(a.half + (size_t)li * H * M);
  for (int e = threadIdx.x; e < nz * PPW; e += blockDim.x) {
    const int k = e / PPW, p = e % PPW;
    if (p0 + p < npair) {
      const float2* z = lds + p * ST;
      const float2 zk = z[pad(k)];
      const float2 zm = z[pad(k == 0 ? 0 : N - k)];
      float4 o;
      if (k == 0) {
        o = make_float4(zk.x, 0.f, zk.y, 0.f);
      } else {  // 2 A[k] = Z[k] + conj Z[N-k]; 2 B[k] = -i (Z[k] - conj Z[N-k])
        o = make_float4(zk.x + zm.x, zk.y - zm.y, zk.y + zm.y, -(zk.x - zm.x));
      }
      dst[((size_t)k * M + 2 * (p0 + p)) / 2] = o;
    }
  }
}

// Adjoint of k_grid_cols (MODE_IMAGE): column gradient at the cutout rows,
// forward transform along v, cell weight, then gather (degrid) at every
// entry of the column: gamma'_b = w G[i_v] (direct) or conj(w G[-i_v])
// (mirror column), both for i_u = 0. Writes vis_grad = conj(g1 conj g2) gamma'
// and, with gains, gq = gamma' conj(V) for the gain gradient. Same XCD-grouped
// 1D layout and empty-column skip as the forward kernel.
// KBW (adjoint with a gridding kernel): the transformed column is written
// to a.gfull instead, for k_degrid_kb.
template <int N, bool UNI, bool KBW = false>
__global__ void __launch_bounds__(Cols<N>::THREADS) k_cols_adj(ImgArgs a) {
  extern __shared__ float4 lds_raw[];
  constexpr int H = N / 2;
  constexpr int CPW = Cols<N>::CPW;
  const int L = blockIdx.x;
  const int r8 = L >> 3;
  const int li = (r8 / a.ntiles) * 8 + (L & 7);
  const int tile = r8 % a.ntiles;
  if (li >= a.nimg) return;
  const int img = a.img0 + li;
  const int nz = min(H, a.ncz[img]);
  const int c0 = tile * CPW;
  if (c0 >= nz) return;                               // no baseline lives in this tile
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  float2* ltw = lds + CPW * Cols<N>::STRIDE;
  int* lcnt = reinterpret_cast<int*>(ltw + Cols<N>::TW);
  const int wave = threadIdx.x / WAVE, lane = threadIdx.x % WAVE;
  const int t = img / a.C, ch = img - t * a.C;
  const int cs = c0 + wave;
  const bool active = cs < nz;
  float2* buf = lds + wave * Cols<N>::STRIDE;
  int* cnt = UNI ? lcnt + wave * N : nullptr;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const int M = a.M;
  const float2* tw = stage_twiddles<N>(ltw);
  __syncthreads();
  if (!active) return;
  for (int r = lane; r < Cols<N>::STRIDE; r += WAVE) buf[r] = make_float2(0.f, 0.f);
  if (UNI)
    for (int r = lane; r < N; r += WAVE) cnt[r] = 0;
  wave_sync();
  const float2* srcc = a.half + ((size_t)li * H + cs) * M;
  for (int m = lane; m < M; m += WAVE) {
    int q = m - M / 2;
    q = q < 0 ? q + N : q;
    buf[pad(q)] = srcc[m];
  }
  const int* bnd = a.bnd + (size_t)img * (N + 2);
  const int dlo = bnd[cs + H], dhi = bnd[cs + 1 + H];
  const int clo = bnd[-cs + H], chi = bnd[-cs + 1 + H];
  const size_t tb = (size_t)t * a.B;
  if (UNI) {
    for (int pass = 0; pass < 2; ++pass) {
      const int lo = pass ? clo : dlo, hi = pass ? chi : dhi;
      for (int j = lo + lane; j < hi; j += WAVE) {
        const double iv = rint(a.sv[tb + j] * s);
        if (fabs(iv) < (double)H) {
          int r = (int)iv;
          if (pass) r = -r;
          atomicAdd(&cnt[r < 0 ? r + N : r], 1);
        }
      }
    }
  }
  wave_sync();
  wave_fft<N, -1>(buf, lane, tw);
  if constexpr (KBW) {
    float2* g = a.gfull + ((size_t)li * H + cs) * N;
    for (int r = lane; r < N; r += WAVE) g[r] = buf[pad(r)];
    return;
  }
  const size_t vb = (size_t)img * a.B;
  // direct entries (and, for column 0, the conjugate entry of the same baseline)
  for (int pass = 0; pass < (cs == 0 ? 1 : 2); ++pass) {
    const int lo = pass ? clo : dlo, hi = pass ? chi : dhi;
    for (int j = lo + lane; j < hi; j += WAVE) {
      const double iv = rint(a.sv[tb + j] * s);
      if (fabs(iv) < (double)H) {
        const int r = (int)iv;
        const int rp = r < 0 ? r + N : r;
        const int rm = -r < 0 ? -r + N : -r;
        float2 g;
        if (pass == 0) {
          float2 v = buf[pad(rp)];
          if (UNI) v = cscale(v, 1.0f / (float)cnt[rp]);
          g = v;
          if (cs == 0) {
            float2 w = buf[pad(rm)];
            if (UNI) w = cscale(w, 1.0f / (float)cnt[rm]);
            g = cadd(g, cconj(w));
          }
        } else {
          float2 w = buf[pad(rm)];
          if (UNI) w = cscale(w, 1.0f / (float)cnt[rm]);
          g = cconj(w);
        }
        const int b = a.perm[tb + j];
        // gradient with respect to V' = g1 conj(g2) V: the load multiplied V' by
        // exp(+2 pi i d nu / c) (rotation, cables), so its gradient carries the conjugate
        if (a.sd != nullptr) g = rotate_phase(g, -a.sd[tb + j], a.freq[ch]);
        if (a.gains) {
          a.vis_grad[vb + b] = cmul(cconj(baseline_gain(a, b)), g);
          const float2 v = load_vis_raw(a, vb + b, ch);
          a.gamma[(size_t)li * a.B + b] = cmul(g, cconj(v));
        } else {
          a.vis_grad[vb + b] = g;
        }
      }
    }
  }
}

// The gradient of one gridded baseline from the column gradient g at its cell:
// the conjugate of the rotation / cable factor, then vis_grad = conj(g1 conj g2)
// gamma' and, with gains, gq = gamma' conj(V).
__device__ __forceinline__ void put_vis_grad(const ImgArgs& a, int li, int img, int ch, size_t tb, int j, int b, float2 g) {
  const size_t vb = (size_t)img * a.B;
  if (a.sd != nullptr) g = rotate_phase(g, -a.sd[tb + j], a.freq[ch]);
  if (a.gains) {
    a.vis_grad[vb + b] = cmul(cconj(baseline_gain(a, b)), g);
    const float2 v = load_vis_raw(a, vb + b, ch);
    a.gamma[(size_t)li * a.B + b] = cmul(g, cconj(v));
  } else {
    a.vis_grad[vb + b] = g;
  }
}

// First-stage inputs of the adjoint's forward transforms straight from memory:
// x[q] = value(q') for the M cutout positions (q' = q + M/2 mod N < M), zero
// elsewhere. ZB: the zero band of a cutout of at most N - ZB N/16 points, whose
// inputs are not formed.
template <int N, int ZB, int L, class Value>
__device__ __forceinline__ void cutout_inputs(HalfIn<N, L>& in, int lane, int M, Value&& value) {
  constexpr int R = HalfIn<N, L>::R, PER = HalfIn<N, L>::PER;
  constexpr int zlo = R / 2 - ZB / 2, zhi = R / 2 + ZB / 2;
#pragma unroll
  for (int p = 0; p < PER; ++p)
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < zlo || r >= zhi) {
        const int q = lane + p * L + r * (N / R);
        const int m = r < R / 2 ? q + M / 2 : q + M / 2 - N;        // position in the cutout
        const bool in_cut = (N / R % L == 0 || lane + p * L < N / R) && m >= 0 && m < M;
        in.v[p][r] = in_cut ? value(m) : make_float2(0.f, 0.f);
      }
}
// Cutouts of up to half of the grid leave the middle half of every
// transform's inputs zero.
template <int N>
constexpr bool adj_band() { return HalfIn<N>::R == 16; }

// k_rows_adj for power-of-two sizes up to 2048: the rows go from memory to the
// first stage's registers (the empty middle half of a cutout M <= N/2 is neither
// read nor added), the exchanges pass through half-length buffers, and the
// Hermitian split reads Z[k] from the lower half of the outputs and Z[N - k] from
// the upper one through the same buffers.
template <int N>
__global__ void __launch_bounds__(RowsHalf<N>::THREADS) k_rows_adj_half(ImgArgs a) {
  using R_ = RowsHalf<N>;
  constexpr int H = N / 2, PPW = R_::PPW, ST = R_::STRIDE, THR = R_::THREADS, L = R_::L;
  constexpr int EPT = H / L;
  static_assert(H % L == 0 && THR == PPW * L, "a tile's slice is whole columns");
  constexpr int RL = pick_radix(N / last_stage_ns(N)), PL = (N / RL + L - 1) / L;
  extern __shared__ float4 lds_raw[];
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  const int lane = threadIdx.x % L;
  // this lane's row pair of the tile
  const int vec = L == WAVE ? __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE) : (int)(threadIdx.x / L);
  const int li = blockIdx.y;
  const int img = a.img0 + li;
  const int M = a.M;
  const int npair = M / 2;
  const int p0 = blockIdx.x * PPW;
  const int nz = min(H, a.ncz[img]);
  const float W = a.wsum_in ? a.wsum_in[img]
                  : a.kw > 0 ? sum_partials_f(a.wpart, img, a.wstride, a.wtiles, threadIdx.x % WAVE)
                             : (float)sum_partials(a.wpart, img, a.wstride, a.wtiles, threadIdx.x % WAVE);
  const float scale = a.norm ? (W > 0 ? 1.0f / W : 0.0f) : 1.0f;
  const float2* tw = stage_twiddles<N>(lds + PPW * ST);
  const int pair = min(p0 + vec, npair - 1);                   // (spare lanes repeat the last pair)
  const float* g0 = a.image_grad + ((size_t)img * M + 2 * pair) * M;
  const float* g1 = g0 + M;
  // with a gridding kernel the forward pass divided pixel (m, l) by
  // c(q_m / N) c(q_l / N); that diagonal scaling is its own adjoint
  float s0 = scale, s1 = scale;
  if (a.kw > 0) {
    s0 *= kb_inv_taper((double)(2 * pair - M / 2) / N, a);
    s1 *= kb_inv_taper((double)(2 * pair + 1 - M / 2) / N, a);
  }
  if (TwLds<N>::ON) __syncthreads();                           // the twiddles
  float2* z = lds + vec * ST;
  float2 up[PL][RL / 2];                                       // the outputs from N / 2 on
  auto body = [&](auto zbc) {
    constexpr int ZB = decltype(zbc)::value;
    HalfIn<N, L> in;
    cutout_inputs<N, ZB, L>(in, lane, M, [&](int l) {
      const float cl = a.kw > 0 ? kb_inv_taper((double)(l - M / 2) / N, a) : 1.0f;
      return make_float2(g0[l] * s0 * cl, g1[l] * s1 * cl);
    });
    wave_fft_half_emit<N, -1, ZB, false, L>(z, lane, tw, in, [&](auto qb, float2 v) {
      constexpr int QB = decltype(qb)::value, r = QB / (N / RL), p = QB % (N / RL) / L;
      if constexpr (QB < H) z[pad(QB + lane)] = v;
      else up[p][r - RL / 2] = v;
    });
  };
  if (adj_band<N>() && 2 * M <= N) body(ic<adj_band<N>() ? 8 : 0>{});
  else body(ic<0>{});
  __syncthreads();
  // thread t takes pair slot t % PPW and columns t / PPW + i L (slots as in k_rows_half)
  const int kt = threadIdx.x / PPW, pt = threadIdx.x % PPW;
  constexpr bool LIN = L % 16 == 0;
  constexpr int PS = L + L / 16;
  const float2* zs = lds + pt * ST;
  float2 zk[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int k = kt + i * L;
    zk[i] = k < nz ? zs[LIN ? pad(kt) + i * PS : pad(k)] : make_float2(0.f, 0.f);
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PL; ++p)
    if ((N / RL) % L == 0 || lane + p * L < N / RL)
#pragma unroll
      for (int r = 0; r < RL / 2; ++r) z[pad(p * L + r * (N / RL) + lane)] = up[p][r];
  __syncthreads();
  float4* dst = reinterpret_cast<float4*>(a.half + (size_t)li * H * M) + p0;
  const int nzp = p0 + pt < npair ? nz : 0;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int k = kt + i * L;
    if (k < nzp) {
      float4 o;
      if (i == 0 && k == 0) {
        o = make_float4(zk[i].x, 0.f, zk[i].y, 0.f);
      } else {  // 2 A[k] = Z[k] + conj Z[N-k]; 2 B[k] = -i (Z[k] - conj Z[N-k])
        const float2 zm = zs[LIN ? pad(H - kt) - i * PS : pad(H - k)];
        o = make_float4(zk[i].x + zm.x, zk[i].y - zm.y, zk[i].y + zm.y, -(zk[i].x - zm.x));
      }
      store_at(dst, (unsigned)(k * (M / 2) + pt), o);
    }
  }
}

// k_cols_adj for power-of-two sizes up to 2048 (nearest cell): the column goes
// from memory to the first stage's registers, the exchanges pass through a
// half-length buffer, and the entries are gathered from the lower half of the
// transformed column, then from the upper one. Columns of at most GADJ x 64
// entries (the usual case) keep their rows in registers for both. The u = 0
// column adds each entry's two rows, which lie in different halves: its lower
// half waits in registers (`low`, one value per kept entry) or, for longer
// columns, in the entry's vis_grad slot. What binds a long column is one wavefront's
// chain of loads, so those of the next ADJ_AHEAD x 64 entries stay in flight: 2,016
// baselines in the u = 0 column of 16 images of 512^2 take 82 us with loads as they
// are needed, 73 two steps ahead and 70 four ahead; 8,128 baselines with half of them
// in 2% of the u range 90, 82 and 79. (Loaded four at a time and then stored, 92: the
// next loads wait for the stores.) At N = 1024 four ahead would take more than the
// 80 registers that let three workgroups share a CU.
constexpr int GADJ = 4;
template <int N> constexpr int ADJ_AHEAD = N == 1024 ? 3 : 4;

// The twiddle table is the full one, every power rounded once from 64 bits. Formed
// from the compact one, w^2k and w^3k carry the rounding of one and two FP32
// products more: the gradients of 320 images of 1024^2 are then 1.39e-7 from 64
// bits instead of 1.34e-7. Three workgroups of 8 columns share a CU either way.
template <int N, int CPW, bool UNI>
struct ColsAdj {
  static constexpr int STRIDE = padded_len(N / 2);
  static constexpr int THREADS = CPW * WAVE;
  static constexpr int TW = TwLds<N>::ON ? tw_entries(N) : 0;
  static constexpr size_t LDS = (size_t)(CPW * STRIDE + TW) * sizeof(float2) + (UNI ? (size_t)CPW * (N / 2) * sizeof(int) : 0);
};

template <int N, int CPW, bool UNI>
__global__ void __launch_bounds__((ColsAdj<N, CPW, UNI>::THREADS)) k_cols_adj_half(ImgArgs a) {
  using C_ = ColsAdj<N, CPW, UNI>;
  constexpr int H = N / 2;
  constexpr int RL = pick_radix(N / last_stage_ns(N)), PL = (N / RL + WAVE - 1) / WAVE;
  extern __shared__ float4 lds_raw[];
  const int L = blockIdx.x;
  const int r8 = L >> 3;
  const int li = (r8 / a.ntiles) * 8 + (L & 7);
  const int tile = r8 % a.ntiles;
  if (li >= a.nimg) return;
  const int img = a.img0 + li;
  const int nz = min(H, a.ncz[img]);
  const int c0 = tile * CPW;
  if (c0 >= nz) return;                               // no baseline lives in this tile
  float2* lds = reinterpret_cast<float2*>(lds_raw);
  float2* ltw = lds + CPW * C_::STRIDE;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x % WAVE;
  const int t = img / a.C, ch = img - t * a.C;
  const int cs = c0 + wave;
  float2* buf = lds + wave * C_::STRIDE;
  int* cnt = UNI ? reinterpret_cast<int*>(ltw + C_::TW) + wave * H : nullptr;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const int M = a.M;
  const float2* tw = stage_twiddles<N>(ltw);
  if (TwLds<N>::ON) __syncthreads();
  if (cs >= nz) return;
  const float2* srcc = a.half + ((size_t)li * H + cs) * M;
  float2 up[PL][RL / 2];                              // the outputs from N / 2 on
  auto body = [&](auto zbc) {
    constexpr int ZB = decltype(zbc)::value;
    HalfIn<N> in;
    cutout_inputs<N, ZB, WAVE>(in, lane, M, [&](int m) { return srcc[m]; });
    wave_fft_half_emit<N, -1, ZB>(buf, lane, tw, in, [&](auto qb, float2 v) {
      constexpr int QB = decltype(qb)::value, r = QB / (N / RL), p = QB % (N / RL) / WAVE;
      if constexpr (QB < H) buf[pad(QB + lane)] = v;
      else up[p][r - RL / 2] = v;
    });
  };
  if (adj_band<N>() && 2 * M <= N) body(ic<adj_band<N>() ? 8 : 0>{});
  else body(ic<0>{});
  const int* bnd = a.bnd + (size_t)img * (N + 2);
  const ColSpan c{bnd[cs + H], bnd[cs + 1 + H], bnd[-cs + H], bnd[-cs + 1 + H]};
  const size_t tb = (size_t)t * a.B;
  const int nd = c.nd(), total = cs == 0 ? nd : c.total();   // u = 0: its mirror column is itself
  // entry i of the column: its sorted position and its row (N when not kept);
  // mirrored entries take their own row's mirror
  auto place = [&](int i) { return i >= nd ? c.clo + (i - nd) : c.dlo + i; };
  auto row_at = [&](int i, double sv) {
    const double iv = rint(sv * s);
    if (!(fabs(iv) < (double)H)) return N;
    int r = (int)iv;
    if (i >= nd) r = -r;
    return r < 0 ? r + N : r;
  };
  auto entry = [&](int i, int& j, int& row) {
    j = place(i);
    row = i < total ? row_at(i, a.sv[tb + j]) : N;
  };
  int rows[GADJ], js[GADJ];
#pragma unroll
  for (int u = 0; u < GADJ; ++u) entry(u * WAVE + lane, js[u], rows[u]);
  float2 low[GADJ];
#pragma unroll
  for (int u = 0; u < GADJ; ++u) low[u] = make_float2(0.f, 0.f);
  auto half = [&](auto hfc) {
    constexpr int HF = decltype(hfc)::value;
    if (UNI) {                                        // cell counts of this half
      for (int r = lane; r < H; r += WAVE) cnt[r] = 0;
      wave_sync();
      for (int i0 = 0; i0 < c.total(); i0 += GADJ * WAVE) {   // (loads of GADJ x 64 entries in flight)
        double sv[GADJ];
#pragma unroll
        for (int u = 0; u < GADJ; ++u) sv[u] = a.sv[tb + place(min(i0 + u * WAVE + lane, c.total() - 1))];
#pragma unroll
        for (int u = 0; u < GADJ; ++u) {
          const int i = i0 + u * WAVE + lane;
          if (i < c.total()) {
            const int r = row_at(i, sv[u]);
            if (r != N && (r >= H) == (HF == 1)) atomicAdd(&cnt[r - HF * H], 1);
          }
        }
      }
    }
    wave_sync();
    auto at = [&](int row) {                          // the column gradient at a row of this half
      float2 v = buf[pad(row - HF * H)];
      if (UNI) v = cscale(v, 1.0f / (float)cnt[row - HF * H]);
      return v;
    };
    // what this half adds to an entry: direct G[row] if the row lies here,
    // conjugated for mirrored entries; at u = 0 also conj G[mirror row]
    auto part = [&](int i, int row, float2& g) -> bool {
      bool any = false;
      if (row != N && (row >= H) == (HF == 1)) {
        const float2 v = at(row);
        g = cadd(g, i >= nd ? cconj(v) : v);
        any = true;
      }
      if (cs == 0 && row != N) {
        const int rm = row == 0 ? 0 : N - row;
        if ((rm >= H) == (HF == 1)) {
          g = cadd(g, cconj(at(rm)));
          any = true;
        }
      }
      return any;
    };
#pragma unroll
    for (int u = 0; u < GADJ; ++u) {
      const int i = u * WAVE + lane;
      if (cs == 0) {                                  // both halves contribute: written after the second
        part(i, rows[u], low[u]);
        if (HF == 1 && rows[u] != N) put_vis_grad(a, li, img, ch, tb, js[u], a.perm[tb + js[u]], low[u]);
      } else {
        float2 g = make_float2(0.f, 0.f);
        if (part(i, rows[u], g)) put_vis_grad(a, li, img, ch, tb, js[u], a.perm[tb + js[u]], g);
      }
    }
    // longer columns: the loads of the next ADJ_AHEAD x 64 entries are in flight, so that a
    // step waits neither for its own loads nor for the stores just before it
    if (total > GADJ * WAVE) {
      double sv[ADJ_AHEAD<N>];
      int b[ADJ_AHEAD<N>];
      auto fetch = [&](int i, int u) {
        const size_t q = tb + place(min(i, total - 1));
        sv[u] = a.sv[q];
        b[u] = a.perm[q];
      };
#pragma unroll
      for (int u = 0; u < ADJ_AHEAD<N>; ++u) fetch((GADJ + u) * WAVE + lane, u);
#pragma unroll 1
      for (int i0 = GADJ * WAVE; i0 < total; i0 += ADJ_AHEAD<N> * WAVE) {
#pragma unroll
        for (int u = 0; u < ADJ_AHEAD<N>; ++u) {
          if (i0 + u * WAVE >= total) break;
          const int i = i0 + u * WAVE + lane, bu = b[u];
          const int row = i < total ? row_at(i, sv[u]) : N;
          fetch(i + ADJ_AHEAD<N> * WAVE, u);
          if (row == N) continue;
          float2 g = make_float2(0.f, 0.f);
          if (cs == 0) {
            float2* keep = a.vis_grad + (size_t)img * a.B + bu;
            if (HF == 1) g = *keep;
            part(i, row, g);
            if (HF == 0) *keep = g;
            else put_vis_grad(a, li, img, ch, tb, place(i), bu, g);
          } else if (part(i, row, g)) {
            put_vis_grad(a, li, img, ch, tb, place(i), bu, g);
          }
        }
      }
    }
  };
  half(ic<0>{});
  wave_sync();
#pragma unroll
  for (int p = 0; p < PL; ++p)
    if ((N / RL) % WAVE == 0 || lane + p * WAVE < N / RL)
#pragma unroll
      for (int r = 0; r < RL / 2; ++r) buf[pad(p * WAVE + r * (N / RL) + lane)] = up[p][r];
  wave_sync();
  half(ic<1>{});
}

// Adjoint of kernel gridding: gamma'_b = sum over b's footprint cells (j, i)
// of C(i - x_u) C(j - x_v) G2[j][i], G2 = 2 Gh over the whole plane, taken
// from the transformed half-spectrum columns B in a.gfull: G2[j][i] = B[j][i]
// for i > 0 (the row pass packed both Hermitian halves there), B[j][0] +
// conj(B[-j][0]) for i = 0, conj(G2[-j][-i]) for i < 0. This is the
// direct-cell sum plus the conjugate of the mirror-cell sum (the gradient
// image is real, so its transform is Hermitian). One thread per sorted entry
// of each image of the chunk, summing in a fixed order; then the rotation and
// gain factors as in k_cols_adj. Uniform weighting divides by the entry's
// cell occupancy (a.kdens).
template <int N, int KMAX>
__global__ void __launch_bounds__(256) k_degrid_kb(ImgArgs a) {
  constexpr int H = N / 2;
  const int li = blockIdx.y;
  const int img = a.img0 + li;
  const int t = img / a.C, ch = img - t * a.C;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n_valid[t]) return;
  const size_t tb = (size_t)t * a.B;
  const double s = cells_per_metre(a.freq[ch], a.ndx);
  const double hw = 0.5 * a.kw;
  const double xu = a.su[tb + j] * s, xv = a.sv[tb + j] * s;
  if (!kb_kept<H>(xu, xv, hw)) return;               // its gradient stays zero
  const int i0 = (int)ceil(xu - hw), ni = (int)floor(xu + hw) - i0 + 1;
  const int j0 = (int)ceil(xv - hw), nj = (int)floor(xv + hw) - j0 + 1;
  float wv[KMAX + 1];
#pragma unroll
  for (int k = 0; k <= KMAX; ++k) {
    wv[k] = 0.f;
    if (k > a.kw) break;
    if (k < nj) wv[k] = kb_weight((float)((double)(j0 + k) - xv), a);
  }
  const float2* G = a.gfull + (size_t)li * H * N;
  auto at = [&](int r, int c) -> float2 {          // B[r][c], c >= 0
    return G[(size_t)c * N + (r < 0 ? r + N : r)];
  };
  float2 sum = make_float2(0.f, 0.f);
  for (int ii = 0; ii < ni; ++ii) {
    const int c = i0 + ii;
    const float wu = kb_weight((float)((double)c - xu), a);
    float2 col = make_float2(0.f, 0.f);
#pragma unroll
    for (int k = 0; k <= KMAX; ++k) {
      if (k >= nj) break;
      const int r = j0 + k;
      float2 g;
      if (c > 0) g = at(r, c);
      else if (c < 0) g = cconj(at(-r, -c));
      else g = cadd(at(r, 0), cconj(at(-r, 0)));
      col = make_float2(col.x + wv[k] * g.x, col.y + wv[k] * g.y);
    }
    sum = make_float2(sum.x + wu * col.x, sum.y + wu * col.y);
  }
  if (a.kdens != nullptr) sum = cscale(sum, 1.0f / (float)a.kdens[(size_t)li * a.B + j]);
  float2 g = sum;
  const int b = a.perm[tb + j];
  if (a.sd != nullptr) g = rotate_phase(g, -a.sd[tb + j], a.freq[ch]);
  const size_t vb = (size_t)img * a.B;
  if (a.gains) {
    a.vis_grad[vb + b] = cmul(cconj(baseline_gain(a, b)), g);
    const float2 v = load_vis_raw(a, vb + b, ch);
    a.gamma[(size_t)li * a.B + b] = cmul(g, cconj(v));
  } else {
    a.vis_grad[vb + b] = g;
  }
}

__global__ void k_fill2(float2* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = make_float2(0.f, 0.f);
}

// pacc[b] += sum over this chunk's images of gq[li][b]: 64 baselines per
// workgroup, GQ_SLICES image slices per baseline (a wavefront each), slices
// combined in a fixed order. The slices hide the latency of the loads: of 320
// images 4 slices read 80 in sequence (26 us), 16 slices 20.
constexpr int GQ_SLICES = 16;
__global__ void __launch_bounds__(64 * GQ_SLICES) k_gq_reduce(ImgArgs a) {
  __shared__ float2 part[GQ_SLICES][64];
  const int bl = threadIdx.x & 63, sl = threadIdx.x >> 6;
  const int b = blockIdx.x * 64 + bl;
  float2 acc = make_float2(0.f, 0.f);
  if (b < a.B)
#pragma unroll 4
    for (int li = sl; li < a.nimg; li += GQ_SLICES) acc = cadd(acc, a.gamma[(size_t)li * a.B + b]);
  part[sl][bl] = acc;
  __syncthreads();
  if (sl == 0 && b < a.B) {
    float2 sum = a.pacc[b];
    for (int i = 0; i < GQ_SLICES; ++i) sum = cadd(sum, part[i][bl]);
    a.pacc[b] = sum;
  }
}

// gain_grad[a] = sum_{b: a1 = a} g2 p_b + sum_{b: a2 = a} g1 conj(p_b)
__global__ void __launch_bounds__(256) k_gain_grad(ImgArgs a) {
  __shared__ float2 part[256];
  const int ant = blockIdx.x;
  float2 acc = make_float2(0.f, 0.f);
  constexpr int U = 4;                                 // baselines in flight per thread
  for (int b0 = threadIdx.x; b0 < a.B; b0 += U * 256) {
    int a1[U], a2[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * 256;
      a1[u] = b < a.B ? a.ant1[b] : -1;
      a2[u] = b < a.B ? a.ant2[b] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * 256;
      if (b >= a.B || (a1[u] != ant && a2[u] != ant)) continue;
      const float2 p = a.pacc[b];
      if (a1[u] == ant) acc = cadd(acc, cmul(antenna_gain(a.gains, a2[u], a.n_ant), p));
      if (a2[u] == ant) acc = cadd(acc, cmul(antenna_gain(a.gains, a1[u], a.n_ant), cconj(p)));
    }
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) part[threadIdx.x] = cadd(part[threadIdx.x], part[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) a.gain_grad[ant] = part[0];
}

}  // namespace blink
