// Simulated ptychographic measurements on the GPU (Sec. II eq. (1) and
// Sec. IV eq. (16)):
//     I_j = |F D P_j x|^2                       (noise-free intensities)
//     z_j = Pois(I_j * r_p / max_{j,k} I_j[k])  (peak photon rate r_p)
// The maximum is taken over every position and pixel (one scale for the
// whole experiment).  Random numbers come from a counter-based generator,
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, "Parallel random numbers: as
// easy as 1, 2, 3", SC 2011), keyed by the seed and counted by element index,
// so every sample is reproducible and independent of the launch shape.
// Poisson variates: the product-of-uniforms method below mean 10, and
// Hormann's transformed rejection with squeeze (PTRS; W. Hormann, "The
// transformed rejection method for generating Poisson random variables",
// Insurance: Mathematics and Economics 12, 1993) from mean 10 up.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "pmace.h"
#include "pmace_dft.hpp"
#include "pmace_internal.hpp"

namespace pmace {

// ---------------------------------------------------------------------------
// Philox4x32-10: ten rounds of two 32x32->64 multiplies, a xor with the key,
// and a Weyl increment of the key between rounds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint2 k) {
  const uint32_t m0 = 0xD2511F53u, m1 = 0xCD9E8D57u;
  const uint32_t w0 = 0x9E3779B9u, w1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)m0 * c.x, p1 = (uint64_t)m1 * c.z;  // one v_mad_u64_u32 each
    c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k.x, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k.y,
                   (uint32_t)p0);
    k.x += w0;
    k.y += w1;
  }
  return c;
}

// Block n of element `idx`'s stream of uniforms: Philox(counter = (idx lo,
// idx hi, n, 0x50495853), key = seed).
__device__ __forceinline__ uint4 uniform_block(uint32_t i0, uint32_t i1, uint32_t n, uint2 key) {
  return philox4x32_10(make_uint4(i0, i1, n, 0x50495853u), key);
}
// 53 random bits, centred in their interval: never 0
__device__ __forceinline__ double unit_double(uint32_t a, uint32_t b) {
  return ((double)(a >> 5) * 67108864.0 + (double)(b >> 6) + 0.5) * (1.0 / 9007199254740992.0);
}

// Uniform doubles in (0, 1) for element `idx`, two from each block.
struct Uniforms {
  uint2 key;
  uint32_t i0, i1, n;
  uint4 buf;
  int have;
  __device__ Uniforms(uint64_t seed, uint64_t idx)
      : key(make_uint2((uint32_t)seed, (uint32_t)(seed >> 32))),
        i0((uint32_t)idx), i1((uint32_t)(idx >> 32)), n(0), have(0) {}
  __device__ double next() {
    if (have == 0) {
      buf = uniform_block(i0, i1, n++, key);
      have = 2;
    }
    const uint32_t a = have == 2 ? buf.x : buf.z, b = have == 2 ? buf.y : buf.w;
    --have;
    return unit_double(a, b);
  }
};

// Transformed rejection (mean >= 10): one try from two uniforms.  `fast`: the
// squeeze accepted k; else the try has still to pass the exact test.
struct Ptrs {
  double slam, a, b, vr;
  __device__ __forceinline__ explicit Ptrs(double lam)
      : slam(sqrt(lam)), a(-0.059 + 0.02483 * (0.931 + 2.53 * slam)), b(0.931 + 2.53 * slam),
        vr(0.9277 - 3.6224 / (b - 2.0)) {}
  __device__ __forceinline__ bool fast(double lam, double U, double V, double& us, double& k) const {
    us = 0.5 - fabs(U);
    k = floor((2.0 * a / us + b) * U + lam + 0.43);
    return us >= 0.07 && V <= vr;
  }
};

// The exact acceptance test of a try that the squeeze left open.
__device__ __forceinline__ bool ptrs_exact(const Ptrs& t, double lam, double loglam, double invalpha,
                                           double V, double us, double k) {
  return log(V) + log(invalpha) - log(t.a / (us * us) + t.b) <= -lam + k * loglam - lgamma(k + 1.0);
}

// The same decision for less: one logarithm for the left side's three, and
// Stirling's series to 1/n^5 for lgamma(n), n = k + 1 >= 8 (its error is under
// 1/(1680 n^7) < 3e-10).  Where the two sides are nearer than that and than
// 45 roundings of the largest term, the exact test decides.
__device__ __forceinline__ bool ptrs_accept(const Ptrs& t, double lam, double loglam, double invalpha,
                                            double V, double us, double k) {
  const double n = k + 1.0, r = 1.0 / n, r2 = r * r, m = k * loglam;
  const double lg = (n - 0.5) * log(n) - n + 0.91893853320467274 +
                    r * (1.0 / 12.0 - r2 * (1.0 / 360.0 - r2 * (1.0 / 1260.0)));
  const double d = log(V * invalpha / (t.a / (us * us) + t.b)) - ((m - lam) - lg);
  if (n >= 8.0 && fabs(d) > 1e-9 + 1e-14 * (fabs(m) + lam)) return d < 0.0;
  return ptrs_exact(t, lam, loglam, invalpha, V, us, k);
}

__device__ double poisson_draw(double lam, Uniforms& u) {
  if (!(lam > 0.0)) return 0.0;
  if (lam < 10.0) {
    const double L = exp(-lam);
    double p = 1.0;
    int k = 0;
    do {
      ++k;
      p *= u.next();
    } while (p > L && k < 1000);
    return (double)(k - 1);
  }
  const Ptrs t(lam);
  const double loglam = log(lam);
  const double invalpha = 1.1239 + 1.1328 / (t.b - 3.4);
  for (int it = 0; it < 1000; ++it) {  // each try accepts with probability > 0.8
    const double U = u.next() - 0.5;
    const double V = u.next();
    double us, k;
    if (t.fast(lam, U, V, us, k)) return k;
    if (k < 0.0 || (us < 0.013 && V > us)) continue;
    if (ptrs_exact(t, lam, loglam, invalpha, V, us, k)) return k;
  }
  return floor(lam + 0.5);
}

// ---------------------------------------------------------------------------
// Noise-free intensities I_j = |F D P_j x|^2 (F orthonormal) and their
// maximum, with the frames d P_j x formed as the transform loads them and the
// intensities as it stores them.  The maximum is folded per workgroup into
// one atomic (non-negative floats order as their bit patterns, so an
// unsigned max is a float max).
// ---------------------------------------------------------------------------
constexpr int kSimRB = 16;         // rows per workgroup of the row pass (Np > 128)
constexpr int kSimCB = PMACE_CB;   // columns per workgroup of the column pass
static_assert(160 % kSimRB == 0 && 192 % kSimRB == 0 && 256 % kSimRB == 0, "row block");
static_assert(160 % kSimCB == 0 && 192 % kSimCB == 0 && 256 % kSimCB == 0, "column block");

template <int NT>
__device__ __forceinline__ void block_max_to(float v, unsigned* maxbits) {
  static_assert(NT % 64 == 0 && NT <= 1024, "whole wavefronts");
  __shared__ float wmax[NT / 64];
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NT / 64; ++w) v = fmaxf(v, wmax[w]);
    atomicMax(maxbits, __float_as_uint(v));
  }
}

// ctl[0]: the bits of the maximum, ctl[1]: whether a position's patch leaves
// the object.  One workgroup checks every position before anything else is
// launched, and the kernels behind it end at once where one is bad, so nothing
// is read out of range and the output stays as it was, without a wait on the
// host in between.  (Four loads a thread go out together; simulate calls of
// 257 positions of 192^2 without noise take 78 us with it, 76 with the check
// inside the frame kernels, which had then written already.)
constexpr int kCheckT = 1024;
__global__ void __launch_bounds__(kCheckT) sim_check_k(const int2* __restrict__ pos, int J, int n1, int n2, int np,
                                                       unsigned* __restrict__ ctl) {
  bool bad = false;
  for (int j0 = threadIdx.x; j0 < J; j0 += 4 * kCheckT) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + q * kCheckT;
      const int2 p = pos[j < J ? j : j0];
      bad |= p.x < 0 || p.y < 0 || p.x > n1 - np || p.y > n2 - np;
    }
  }
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) {
    ctl[0] = 0u;
    ctl[1] = any ? 1u : 0u;
  }
}

// Np <= 128: one position per workgroup, the whole frame in LDS.
template <int NP>
__global__ void __launch_bounds__(NP * Geo<NP>::A)
sim_small_k(const float2* __restrict__ d, const int2* __restrict__ pos, const float2* __restrict__ x,
            int n2, float* __restrict__ z, unsigned* __restrict__ ctl) {
  if (ctl[1]) return;
  constexpr int A = Geo<NP>::A, B = Geo<NP>::B, S = NP + A, NT = NP * A, M = B / A;
  static_assert(exch_phases<NP>() == 1, "the whole-frame tile exchanges in one round");
  __shared__ float2 tile[NP * S];
  __shared__ float2 tw[NP];
  const int tid = threadIdx.x;
  fill_twiddles<NP>(tw, tid, NT);
  const int j = blockIdx.x;
  const int2 pj = pos[j];
  const int r = tid / A, p = tid % A, c = tid % NP, q = tid / NP;
  const float2* xrow = x + (size_t)(pj.x + r) * n2 + pj.y;
  float2* row = tile + r * S;
  float2 v[B];
#pragma unroll
  for (int nb = 0; nb < B; ++nb) {
    const int cc = p + A * nb;
    v[nb] = cmul(d[r * NP + cc], xrow[cc]);
  }
  __syncthreads();
  row_fwd<NP>(v, row, p, tw);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int ka = 0; ka < A; ++ka) row[p + A * m + B * ka] = v[m * A + ka];
  __syncthreads();
#pragma unroll
  for (int nb = 0; nb < B; ++nb) v[nb] = tile[(q + A * nb) * S + c];
  col_fwd<NP>(v, tile, S, c, q, tw);
  const float scale = 1.f / NP;
  float* zj = z + (size_t)j * NP * NP;
  float mx = 0.f;
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int ka = 0; ka < A; ++ka) {
      const float2 s = cscale(v[m * A + ka], scale);
      const float e = fmaf(s.x, s.x, s.y * s.y);
      zj[(size_t)(q + A * m + B * ka) * NP + c] = e;
      mx = fmaxf(mx, e);
    }
  block_max_to<NT>(mx, ctl);
}

// Np > 128, row pass: frames and forward row DFTs (scaled 1/sqrt(Np)) to fr.
// A workgroup takes one row block of several positions (j, j + groups, ...), so
// the block's probe rows stay in registers, the twiddles are made once, and,
// with no barrier in the loop (a row is transformed within a wave), some waves
// load while others transform.  Simulate call, 900 positions of 256^2: 615 us
// with one position and 32 rows per workgroup, 574 with 16 rows of 3 or 4.
template <int NP>
__global__ void __launch_bounds__(kSimRB * Geo<NP>::A)
sim_rows_k(const float2* __restrict__ d, const int2* __restrict__ pos, const float2* __restrict__ x, int J,
           int groups, int n2, float2* __restrict__ fr, const unsigned* __restrict__ ctl, float sc) {
  if (ctl[1]) return;
  constexpr int A = Geo<NP>::A, B = Geo<NP>::B, M = B / A, S = row_cap<NP>();
  __shared__ float2 tile[kSimRB * S];
  __shared__ float2 tw[NP];
  const int tid = threadIdx.x;
  const int first = blockIdx.x / (NP / kSimRB), rb = blockIdx.x % (NP / kSimRB);
  const int rl = tid / A, p = tid % A, r = rb * kSimRB + rl;
  float2 dv[B], v[B];
#pragma unroll
  for (int nb = 0; nb < B; ++nb) dv[nb] = d[r * NP + p + A * nb];
  fill_twiddles<NP>(tw, tid, kSimRB * A);
  __syncthreads();
#pragma unroll 1
  for (int j = first; j < J; j += groups) {
    const int2 pj = pos[j];
    const float2* xrow = x + (size_t)(pj.x + r) * n2 + pj.y;
#pragma unroll
    for (int nb = 0; nb < B; ++nb) v[nb] = xrow[p + A * nb];
#pragma unroll
    for (int nb = 0; nb < B; ++nb) v[nb] = cmul(dv[nb], v[nb]);
    row_fwd<NP>(v, tile + rl * S, p, tw);
    float2* out = fr + ((size_t)j * NP + r) * NP;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int ka = 0; ka < A; ++ka) out[p + A * m + B * ka] = cscale(v[m * A + ka], sc);
  }
}

// Np > 128, column pass: forward column DFTs (scaled 1/sqrt(Np)) and the
// intensities.
template <int NP>
__global__ void __launch_bounds__(kSimCB * Geo<NP>::A)
sim_cols_k(const float2* __restrict__ fr, float* __restrict__ z, unsigned* __restrict__ ctl, float sc) {
  if (ctl[1]) return;
  constexpr int A = Geo<NP>::A, B = Geo<NP>::B, M = B / A, NT = kSimCB * A;
  __shared__ float2 tile[col_rows<NP>() * kSimCB];
  __shared__ float2 tw[NP];
  const int tid = threadIdx.x;
  fill_twiddles<NP>(tw, tid, NT);
  const int j = blockIdx.x / (NP / kSimCB), cb = blockIdx.x % (NP / kSimCB);
  const int c = tid % kSimCB, q = tid / kSimCB, col = cb * kSimCB + c;
  const size_t base = (size_t)j * NP * NP + col;
  float2 v[B];
#pragma unroll
  for (int nb = 0; nb < B; ++nb) v[nb] = fr[base + (size_t)(q + A * nb) * NP];
  __syncthreads();
  col_fwd<NP>(v, tile, kSimCB, c, q, tw);
  float mx = 0.f;
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int ka = 0; ka < A; ++ka) {
      const float2 s = cscale(v[m * A + ka], sc);
      const float e = fmaf(s.x, s.x, s.y * s.y);
      z[base + (size_t)(q + A * m + B * ka) * NP] = e;
      mx = fmaxf(mx, e);
    }
  block_max_to<NT>(mx, ctl);
}

template <int NP>
hipError_t launch_sim_intensities(int J, const float2* d, const int2* pos, const float2* x, int n2,
                                  float2* fr, float* z, unsigned* ctl, hipStream_t st) {
  if constexpr (NP <= 128) {
    hipLaunchKernelGGL(sim_small_k<NP>, dim3(J), dim3(NP * Geo<NP>::A), 0, st, d, pos, x, n2, z, ctl);
  } else {
    const float sc = 1.f / sqrtf((float)NP);  // 1/sqrt(Np) per pass
    const int groups = J < 256 ? J : 256;  // (each CU holds 4 of the 16 x 256 workgroups at a time)
    hipLaunchKernelGGL(sim_rows_k<NP>, dim3(groups * (NP / kSimRB)), dim3(kSimRB * Geo<NP>::A), 0, st, d, pos,
                       x, J, groups, n2, fr, ctl, sc);
    hipLaunchKernelGGL(sim_cols_k<NP>, dim3(J * (NP / kSimCB)), dim3(kSimCB * Geo<NP>::A), 0, st, fr, z,
                       ctl, sc);
  }
  return hipGetLastError();
}

// Poisson counts in place, PER elements per thread of a workgroup.
//
// A diffraction pattern is dark nearly everywhere: at a peak of 1e6 photons
// 94% of a 256^2 pattern's pixels have a mean under 0.1, 2% one of 1..10 and
// 2.5% one of 10 and more, in clusters.  One element per thread has every wave
// run the FP64 exponential, and the waves of a bright region run the product
// loop, the squeeze and the exact rejection test (logarithms and a lgamma) one
// after the other, each for a few of its lanes.  Here most elements end on
// one integer word: the first uniform lies below (a + 1)/2^32, a its top
// word, and the count is 0 when it is <= exp(-lam), so surely when
// (a + 1)/2^32 <= 1 - lam (tested with slack for the float rounding of both
// sides).  The others are listed in LDS by what they need and drawn by full
// waves: the squeeze of the means of 10 and more, the tries that it leaves
// open, and the product-of-uniforms draws, each lane taking the next element
// as it finishes one.  Every element keeps its own stream and decisions, so
// the counts are poisson_draw's, bit for bit.  Bound by the generator's
// integer multiplies (about 17 64-bit products per element: 200 us for 900
// patterns of 256^2) and the latency of the bright workgroups' draws.  The
// simulate call on those: 1189 us with one element per thread, 645 with this.
constexpr int kPoisT = 256;
// 8 waves per SIMD (64 VGPRs): the rare draws spill, the common path does not.
// Measured, simulate call of 900 patterns of 256^2 at peak 1e6: 1122 us without
// the bound (193 VGPRs, 2 waves), 918 at 6 waves, 934 at 8; with the rotation
// of the groups of workgroups below 672 and 655.
constexpr int kPoisWaves = 8;

// Appends this lane's element to an LDS list (one LDS atomic per wave).
__device__ __forceinline__ void wave_push(bool want, uint16_t v, uint16_t* list, int* count, int step) {
  const unsigned long long m = __ballot(want);
  if (m == 0) return;
  const int lane = threadIdx.x & 63;
  int at = 0;
  if (lane == __ffsll((long long)m) - 1) at = atomicAdd(count, __popcll(m));
  at = __builtin_amdgcn_readlane(at, __ffsll((long long)m) - 1);
  if (want) list[step * (at + __popcll(m & ((1ull << lane) - 1)))] = v;
}

template <int PER>
__global__ void __launch_bounds__(kPoisT, kPoisWaves) poisson_k(float* __restrict__ z,
                                                                const unsigned* __restrict__ ctl,
                                                                double peak, uint64_t seed,
                                                                long long total) {
  constexpr int kPoisN = kPoisT * PER, kPoisIn = PER < 4 ? PER : 4;
  static_assert((1ll << 32) % kPoisN == 0, "a workgroup's elements share the high index word");
  if (ctl[1]) return;
  // lists of elements (offsets in the block): small means from the front of
  // `list`, larger ones from its end; `open` the larger ones the squeeze left
  __shared__ uint16_t list[kPoisN], open[kPoisN];
  __shared__ int n_small, n_large, n_open, next;
  const int tid = threadIdx.x;
  // Bright rows come at the same places of every pattern, and the dispatcher
  // sends workgroup b to XCD b mod 8: each group of 8 is rotated by a hash of
  // its number, or two XCDs would get most of the bright ones.
  unsigned blk8 = blockIdx.x;
  if ((blk8 | 7u) < gridDim.x) blk8 = (blk8 & ~7u) | ((blk8 + (((blk8 >> 3) * 0x9E3779B1u) >> 29)) & 7u);
  const long long base = (long long)blk8 * kPoisN;
  const int n = total - base < kPoisN ? (int)(total - base) : kPoisN;
  const double mx = (double)__uint_as_float(ctl[0]);
  const double scale = mx > 0.0 ? peak / mx : 0.0;
  const uint2 key = make_uint2((uint32_t)seed, (uint32_t)(seed >> 32));
  const uint32_t b0 = (uint32_t)base, b1 = (uint32_t)((unsigned long long)base >> 32);
  float* zb = z + base;
  if (tid == 0) n_small = n_large = n_open = next = 0;
  __syncthreads();
  // kPoisIn elements of a thread in flight at a time
#pragma unroll 1
  for (int k0 = 0; k0 < PER; k0 += kPoisIn) {
    float zv[kPoisIn];
#pragma unroll
    for (int k = 0; k < kPoisIn; ++k) {
      const int i = tid + (k0 + k) * kPoisT;
      zv[k] = i < n ? zb[i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kPoisIn; ++k) {
      const int i = tid + (k0 + k) * kPoisT;
      const double lam = (double)zv[k] * scale;
      const bool pos = lam > 0.0;            // false for NaN: those draw 0, as do the zeros
      const uint32_t a = uniform_block(b0 + (uint32_t)i, b1, 0u, key).x;
      const bool zero =
          !pos || (float)(~a) * 0.999999f >= fmaf((float)lam, 4294967296.f * 1.000001f, 1.f);
      if (zero && i < n) zb[i] = 0.f;
      wave_push(!zero && lam < 10.0, (uint16_t)i, list, &n_small, 1);
      wave_push(!zero && !(lam < 10.0), (uint16_t)i, list + kPoisN - 1, &n_large, -1);
    }
  }
  __syncthreads();
  // means of 10 and more: the first try's squeeze
  const int nl = n_large, ns = n_small;
  for (int e = tid; e < ((nl + 63) & ~63); e += kPoisT) {
    int i = 0;
    bool left = false;
    if (e < nl) {
      i = list[kPoisN - 1 - e];
      const double lam = (double)zb[i] * scale;
      const uint4 w = uniform_block(b0 + (uint32_t)i, b1, 0u, key);
      const Ptrs t(lam);
      double us, k;
      left = !t.fast(lam, unit_double(w.x, w.y) - 0.5, unit_double(w.z, w.w), us, k);
      if (!left) zb[i] = (float)k;
    }
    wave_push(left, (uint16_t)i, open, &n_open, 1);
  }
  __syncthreads();
  // ... and what it left open: from the same try on
  for (int e = tid; e < n_open; e += kPoisT) {
    const int i = open[e];
    const double lam = (double)zb[i] * scale;
    const Ptrs t(lam);
    const double loglam = log(lam);
    const double invalpha = 1.1239 + 1.1328 / (t.b - 3.4);
    double k = 0.0;
    int it = 0;
    for (; it < 1000; ++it) {
      const uint4 w = uniform_block(b0 + (uint32_t)i, b1, (uint32_t)it, key);
      const double V = unit_double(w.z, w.w);
      double us;
      if (t.fast(lam, unit_double(w.x, w.y) - 0.5, V, us, k)) break;
      if (k < 0.0 || (us < 0.013 && V > us)) continue;
      if (ptrs_accept(t, lam, loglam, invalpha, V, us, k)) break;
    }
    zb[i] = (float)(it < 1000 ? k : floor(lam + 0.5));
  }
  // means below 10: the product of uniforms passes exp(-lam), two factors per
  // block of the stream
  int i = -1, k = 0;
  uint32_t blk = 0;
  double p = 1.0, L = 0.0;
  for (;;) {
    if (i < 0) {
      const int e = atomicAdd(&next, 1);
      if (e >= ns) break;
      i = list[e];
      L = exp(-((double)zb[i] * scale));
      p = 1.0;
      k = 0;
      blk = 0;
    }
    const uint4 w = uniform_block(b0 + (uint32_t)i, b1, blk++, key);
    p *= unit_double(w.x, w.y);
    bool done = !(p > L) || ++k >= 1000;
    if (!done) {
      p *= unit_double(w.z, w.w);
      done = !(p > L) || ++k >= 1000;
    }
    if (done) {
      zb[i] = (float)(k < 1000 ? k : 999);
      i = -1;
    }
  }
}

// Elements per thread: with 16, lists are long enough for full waves, once
// there are 8 such workgroups per CU; smaller totals are spread over more
// workgroups, as their time is one workgroup's latency.  Measured, simulate
// calls with 1 / 4 / 16 elements per thread: 36 patterns of 32^2 68 / 70 / 80
// us, 200 of 48^2 76.6 / 76.3 / 82, 300 of 160^2 181 / 156 / 158, 300 of
// 256^2 328 / 268 / 245.
void launch_poisson(float* z, const unsigned* ctl, double peak, uint64_t seed, long long total,
                    hipStream_t st) {
  const auto go = [&](auto per) {
    constexpr int PER = decltype(per)::value, N = kPoisT * PER;
    hipLaunchKernelGGL(poisson_k<PER>, dim3((unsigned)((total + N - 1) / N)), dim3(kPoisT), 0, st, z, ctl,
                       peak, seed, total);
  };
  if (total >= 2048ll * 4096) go(std::integral_constant<int, 16>());
  else if (total >= 128ll * 1024) go(std::integral_constant<int, 4>());
  else go(std::integral_constant<int, 1>());
}

__global__ void philox_k(uint32_t* io, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t* r = io + 6 * (size_t)i;
  const uint4 o = philox4x32_10(make_uint4(r[0], r[1], r[2], r[3]), make_uint2(r[4], r[5]));
  r[0] = o.x;
  r[1] = o.y;
  r[2] = o.z;
  r[3] = o.w;
}

__global__ void poisson_test_k(const double* __restrict__ lam, float* __restrict__ out, uint64_t seed,
                               int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Uniforms u(seed, (uint64_t)i);
  out[i] = (float)poisson_draw(lam[i], u);
}

// Scratch of the allocation-free entry point: the maximum and the position
// flag in the first 256 bytes, then (Np > 128) the frames' row transforms.
// One copy per device, held until the process ends.
constexpr size_t kSimScratchBytes = (size_t)64 << 20;
__device__ __align__(256) unsigned char scratch[kSimScratchBytes];

}  // namespace pmace

namespace {
inline unsigned nblocks(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }
inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Intensities, optional Poisson draws and the scale, into z_d; `fr` holds the
// row transforms (Np > 128), `ctl` the maximum and the position flag, read back
// through the slot, if it is one.  Waits for all of it where the scale is asked
// for, else for the position check only.
pmace_status run_simulation(int32_t n1, int32_t n2, int32_t np, int32_t num_pos, const void* probe_d,
                            const int32_t* pos_d, const void* x_d, double peak_photons, uint64_t seed,
                            float* z_d, float2* fr, unsigned* ctl, pmace::HostSlot& slot, double* scale_out,
                            hipStream_t st) {
  const long long total = (long long)num_pos * np * np;
  const float2* dd = reinterpret_cast<const float2*>(probe_d);
  const int2* pp = reinterpret_cast<const int2*>(pos_d);
  const float2* xx = reinterpret_cast<const float2*>(x_d);
  unsigned words[2];
  const unsigned* host = slot.p ? static_cast<unsigned*>(slot.p) : words;
  const auto read_ctl = [&] {
    if (hipMemcpyAsync(slot.p ? slot.use<void>() : words, ctl, 8, hipMemcpyDeviceToHost, st) != hipSuccess ||
        !slot.wait(st))
      return PMACE_EDEVICE;
    return host[1] ? PMACE_EINVAL : PMACE_OK;
  };
  hipLaunchKernelGGL(pmace::sim_check_k, dim3(1), dim3(pmace::kCheckT), 0, st, pp, num_pos, n1, n2, np, ctl);
  if (!scale_out) {
    const pmace_status s = read_ctl();
    if (s != PMACE_OK) return s;
  }
  hipError_t e = hipErrorInvalidValue;
  switch (np) {
#define PMACE_SIM(N) \
  case N: e = pmace::launch_sim_intensities<N>(num_pos, dd, pp, xx, n2, fr, z_d, ctl, st); break;
    PMACE_SIM(32)
    PMACE_SIM(48)
    PMACE_SIM(64)
    PMACE_SIM(96)
    PMACE_SIM(128)
    PMACE_SIM(160)
    PMACE_SIM(192)
    PMACE_SIM(256)
#undef PMACE_SIM
    default: break;
  }
  if (e != hipSuccess) return PMACE_EDEVICE;
  if (peak_photons > 0.0)
    pmace::launch_poisson(z_d, ctl, peak_photons, seed, total, st);
  if (hipGetLastError() != hipSuccess) return PMACE_EDEVICE;
  if (scale_out) {
    const pmace_status s = read_ctl();
    if (s != PMACE_OK) return s;
    float mx;
    std::memcpy(&mx, &host[0], 4);
    *scale_out = (peak_photons > 0.0 && mx > 0.f) ? peak_photons / (double)mx : 1.0;
  }
  return PMACE_OK;
}


// Device address of `scratch` on each device, looked up once per device.
std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};

unsigned char* scratch_of_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(pmace::scratch)) != hipSuccess || !p) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return static_cast<unsigned char*>(g_scratch_ptr[dev]);
}
}  // namespace

extern "C" {

size_t pmace_simulate_footprint(int32_t np, int32_t num_pos) {
  if (np < 1 || num_pos < 1) return 0;
  return up256((size_t)num_pos * np * np * 8) + 256 + 256;
}

pmace_status pmace_simulate(int32_t n1, int32_t n2, int32_t np, int32_t num_pos, const void* probe_d,
                            const int32_t* pos_d, const void* x_d, double peak_photons,
                            uint64_t seed, float* z_d, void* workspace_d, size_t ws_bytes,
                            double* scale_out, void* hip_stream) {
  if (np < 1 || num_pos < 1 || n1 < np || n2 < np || !probe_d || !pos_d || !x_d || !z_d ||
      !workspace_d || !std::isfinite(peak_photons))
    return PMACE_EINVAL;
  if (np != 32 && np != 48 && np != 64 && np != 96 && np != 128 && np != 160 && np != 192 && np != 256)
    return PMACE_EUNSUPPORTED;
  if (ws_bytes < pmace_simulate_footprint(np, num_pos)) return PMACE_ENOMEM;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  char* base = reinterpret_cast<char*>(up256(reinterpret_cast<size_t>(workspace_d)));
  float2* fr = reinterpret_cast<float2*>(base);
  unsigned* ctl = reinterpret_cast<unsigned*>(base + up256((size_t)num_pos * np * np * 8));
  pmace::HostSlot slot;
  return run_simulation(n1, n2, np, num_pos, probe_d, pos_d, x_d, peak_photons, seed, z_d, fr, ctl, slot, scale_out,
                        st);
}

size_t pmace_simulate_static_max_bytes(void) { return pmace::kSimScratchBytes - 256; }

pmace_status pmace_simulate_static(int32_t n1, int32_t n2, int32_t np, int32_t num_pos,
                                   const void* probe_d, const int32_t* pos_d, const void* x_d,
                                   double peak_photons, uint64_t seed, float* z_d, double* scale_out,
                                   void* hip_stream) {
  if (np < 1 || num_pos < 1 || n1 < np || n2 < np || !probe_d || !pos_d || !x_d || !z_d ||
      !std::isfinite(peak_photons))
    return PMACE_EINVAL;
  if (np != 32 && np != 48 && np != 64 && np != 96 && np != 128 && np != 160 && np != 192 && np != 256)
    return PMACE_EUNSUPPORTED;
  // Np > 128 keeps every frame's row transform in the scratch array
  const size_t frames = np > 128 ? (size_t)num_pos * np * np * 8 : 0;
  if (frames > pmace_simulate_static_max_bytes()) return PMACE_ENOMEM;
  unsigned char* sp = scratch_of_current_device();
  if (!sp) return PMACE_EDEVICE;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  unsigned* ctl = reinterpret_cast<unsigned*>(sp);  // [0] maximum bits, [1] position flag
  float2* fr = reinterpret_cast<float2*>(sp + 256);
  pmace::HostSlot none(pmace::kHostSlot + 1);   // (this entry point allocates nothing at all)
  return run_simulation(n1, n2, np, num_pos, probe_d, pos_d, x_d, peak_photons, seed, z_d, fr, ctl, none,
                        scale_out, st);
}

pmace_status pmace_philox4x32_10(uint32_t* io_d, int32_t n, void* hip_stream) {
  if (!io_d || n < 0) return PMACE_EINVAL;
  if (n == 0) return PMACE_OK;
  hipLaunchKernelGGL(pmace::philox_k, dim3(nblocks(n, 256)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), io_d, n);
  return hipGetLastError() == hipSuccess ? PMACE_OK : PMACE_EDEVICE;
}

pmace_status pmace_poisson(const double* lam_d, float* out_d, int32_t n, uint64_t seed,
                           void* hip_stream) {
  if (!lam_d || !out_d || n < 0) return PMACE_EINVAL;
  if (n == 0) return PMACE_OK;
  hipLaunchKernelGGL(pmace::poisson_test_k, dim3(nblocks(n, 256)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), lam_d, out_d, seed, n);
  return hipGetLastError() == hipSuccess ? PMACE_OK : PMACE_EDEVICE;
}

}  // extern "C"
