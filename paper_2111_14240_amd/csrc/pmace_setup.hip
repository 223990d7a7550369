// Set-up of one reconstruction on the device (gfx950): the probe tables, the
// amplitudes, the starting states and images, and the lists that the
// consensus walks.
//
// Two groups of launches.  The first reads the caller's arrays (probe,
// positions, intensities, starting object) and leaves in the status word
// what the host has to know: a bad value, or a probe with exact zeros.  A
// position outside the object is flagged and kept as (0, 0), so no kernel
// reads out of range whatever the caller passed.  The host then reads the
// status word and the positions in one copy, and launches the second group
// (lists, normaliser, images) from the rows that each chunk covers.
//
// These lists were built on the host, in a vector per tile and per object
// row, sorted and copied: 4.7 ms of a 6.5 ms solve of 400 positions of 256^2
// (five iterations), 0.5 of 0.8 ms for 144 of 64^2.
#include "pmace_dft.hpp"
#include "pmace_internal.hpp"

namespace pmace {

namespace {
constexpr int kPMACE = 0, kSharpPlus = 1;
inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// Whether the states are kept as row spectra, before the host knows of the
// probe's zeros: allowed, and (PMACE) no exact zero seen.
__device__ __forceinline__ bool rows_wanted(const Recon& g, int rowspec_allowed) {
  return rowspec_allowed && (g.method == kSharpPlus || !(*g.status & kStatusProbeZero));
}

// ORs a wave's flags into the status word (one atomic at most).
__device__ __forceinline__ void raise(unsigned* status, unsigned flag) {
  unsigned all = 0;
#pragma unroll
  for (unsigned b = 1; b <= kStatusBadPosition; b <<= 1)
    if (__ballot((flag & b) != 0)) all |= b;
  if (all && (threadIdx.x & 63) == (unsigned)(__ffsll((long long)__ballot(1)) - 1)) atomicOr(status, all);
}
}  // namespace

// Status word, stop flag, counters and history; the twiddle table W_np^m
// (FP64, rounded once; exact zeros at quarter turns).
__global__ void __launch_bounds__(256) setup_clear_k(const Recon g, int* fitem) {
  const int t = threadIdx.x;
  if (t == 0) {
    *g.status = 0u;
    *g.done = 0;
    *fitem = 0;
    g.cursor[0] = g.cursor[1] = 0;
    g.track[0] = 0.0;
    g.track[3] = 0.0;
  }
  if (t == 1 || t == 2 || (t >= 4 && t < 7)) g.track[t] = __builtin_inf();
  if (t < g.np) {
    double s, c;
    sincospi(-2.0 * (double)t / (double)g.np, &s, &c);
    g.twn[t] = make_float2((float)c, (float)s);
  }
}

// Positions (checked) and the per-pixel probe tables, FP64 rounded once:
//   PMACE : d^{-1}/Np^2 (the unnormalised transform pair folded in), |d|^kappa,
//           the d == 0 mark, and the weights on the stored states |d|^kappa / d
//           (|d|^kappa where d == 0: the state is t itself there)
//   SHARP+: conj(d)/Np^2 and conj(d); weights |d|^2
__global__ void __launch_bounds__(256) setup_tables_k(const Recon g, const float2* __restrict__ probe,
                                                      const int2* __restrict__ pos, double kappa,
                                                      double rho, int with_dr) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int np2 = g.np * g.np;
  unsigned flag = 0;
  if (i < g.J) {
    const int2 p = pos[i];
    const bool ok = p.x >= 0 && p.y >= 0 && p.x <= g.n1 - g.np && p.y <= g.n2 - g.np;
    g.pos[i] = ok ? p : make_int2(0, 0);
    if (!ok) flag |= kStatusBadPosition;
  }
  if (i < np2) {
    const float2 d = probe[i];
    if (!(isfinite(d.x) && isfinite(d.y))) flag |= kStatusBadProbe;
    g.d[i] = d;
    const double re = d.x, im = d.y, inv = 1.0 / (double)np2;
    const double mag = hypot(re, im), m2 = re * re + im * im;
    if (g.method == kSharpPlus) {
      g.omega64[i] = mag * mag;
      g.pc[i] = make_float4((float)(re * inv), (float)(-im * inv), d.x, -d.y);
      g.gw[i] = make_float2(0.f, 0.f);
      g.dinv[i] = make_float2(0.f, 0.f);
    } else {
      const double om = pow(mag, kappa);
      float2 di = make_float2(0.f, 0.f), w = make_float2((float)om, 0.f);
      const bool nz = mag != 0.0;
      if (nz) {
        di = make_float2((float)(inv * re / m2), (float)(-inv * im / m2));
        w = make_float2((float)(om * re / m2), (float)(-om * im / m2));
      } else {
        flag |= kStatusProbeZero;
      }
      g.omega64[i] = om;
      g.gw[i] = w;
      g.pc[i] = make_float4(di.x, di.y, (float)om, nz ? 0.f : 1.f);
      // d != 0 must not round to the d == 0 mark: keep the smallest subnormal
      if (nz && di.x == 0.f && di.y == 0.f) di.x = __uint_as_float(1u);
      g.dinv[i] = di;
    }
    if (with_dr) g.dr[i] = make_float2((float)(2.0 * rho * re), (float)(2.0 * rho * im));
  }
  raise(g.status, flag);
}

// The exact zeros of the probe by the threads of the row transforms (A to a
// row), see Recon::zmask.
__global__ void __launch_bounds__(256) setup_zeros_k(const Recon g, int A) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= g.np * A) return;
  const float2* row = g.d + (size_t)(i / A) * g.np + i % A;
  unsigned long long m = 0;
  for (int nb = 0; nb < g.np / A; ++nb) {
    const float2 d = row[A * nb];
    if (d.x == 0.f && d.y == 0.f) m |= 1ull << nb;
  }
  g.zmask[i] = m;
}

int line_threads(int np) {
  switch (np) {
    case 32: return Geo<32>::A;
    case 48: return Geo<48>::A;
    case 64: return Geo<64>::A;
    case 96: return Geo<96>::A;
    case 128: return Geo<128>::A;
    case 160: return Geo<160>::A;
    case 192: return Geo<192>::A;
    default: return Geo<256>::A;
  }
}

// ys = scale sqrt(z), four to a thread.  Bound by memory (8 B per patch pixel).
__global__ void __launch_bounds__(256) setup_amplitudes4_k(const Recon g, const float4* __restrict__ z,
                                                           float scale, long long total4) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total4) return;
  const float4 v = z[i];
  const auto bad = [](float a) { return !(a >= 0.f) || isinf(a); };
  raise(g.status, bad(v.x) || bad(v.y) || bad(v.z) || bad(v.w) ? kStatusBadIntensity : 0u);
  reinterpret_cast<float4*>(g.ys)[i] =
      make_float4(scale * sqrtf(fmaxf(v.x, 0.f)), scale * sqrtf(fmaxf(v.y, 0.f)),
                  scale * sqrtf(fmaxf(v.z, 0.f)), scale * sqrtf(fmaxf(v.w, 0.f)));
}

// The same in any order: z with its zero frequency at the centre, an
// unaligned z, ys in the split agent's coset order (element m of block ab
// holds the frequency (2 m1 + a, 2 m2 + b)).
__global__ void __launch_bounds__(256) setup_amplitudes_k(const Recon g, const float* __restrict__ z,
                                                          float scale, int centered) {
  const int np2 = g.np * g.np, per = (np2 + 255) / 256;
  const int j = blockIdx.x / per, rem = (int)(blockIdx.x % per) * 256 + threadIdx.x;
  if (rem >= np2) return;
  int k = rem / g.np, l = rem - k * g.np;
  if (g.split) {
    const int M = g.np / 2, ab = rem / (M * M), m = rem - ab * M * M;
    k = 2 * (m / M) + (ab >> 1);
    l = 2 * (m % M) + (ab & 1);
  }
  const int h = centered ? g.np / 2 : 0;
  const float zz = z[(size_t)j * np2 + ((k + h) % g.np) * g.np + (l + h) % g.np];
  raise(g.status, !(zz >= 0.f) || isinf(zz) ? kStatusBadIntensity : 0u);
  g.ys[(size_t)j * np2 + rem] = scale * sqrtf(fmaxf(zz, 0.f));
}

// The starting state of one pixel.  Alg. 1: v_j = P_j x0 (= t, xbar = 0),
// stored as d t (t where d == 0).  Alg. 2: s_j = D P_j x0, held as
// t = s - 2 beta d P_j xbar with xbar = x0 (the overlap image of consistent
// frames), i.e. (1 - 2 beta) d x0.
__device__ __forceinline__ float2 start_state(const Recon& g, float2 d, float2 x) {
  const float2 dx = cmul(d, x);
  const float f = g.method == kSharpPlus ? 1.f - g.two_rho : 1.f;
  const bool raw = g.method != kSharpPlus && d.x == 0.f && d.y == 0.f;
  return make_float2(raw ? x.x : dx.x * f, raw ? x.y : dx.y * f);
}

// (The starting object is read from xhat, where setup_object_k has put it.)
__global__ void __launch_bounds__(256) setup_states_k(const Recon g) {
  const int np2 = g.np * g.np, per = (np2 + 255) / 256;
  const int j = blockIdx.x / per, rem = (int)(blockIdx.x % per) * 256 + threadIdx.x;
  if (rem >= np2) return;
  const int r = rem / g.np, c = rem - r * g.np;
  const int2 pj = g.pos[j];
  const float2 x = g.xhat[(size_t)(pj.x + r) * g.n2 + pj.y + c];
  g.t[(size_t)j * np2 + rem] = start_state(g, g.d[rem], x);
}

// Np > 128: the same, each row transformed before it is stored where the
// states are kept as row spectra, F_r(s)/Np (writing the states and
// transforming them in place cost 16 B per patch pixel more).  kRB rows of a
// patch per workgroup.
constexpr int kRB = 16;
static_assert(160 % kRB == 0 && 192 % kRB == 0 && 256 % kRB == 0, "row block");
template <int NP>
__global__ void __launch_bounds__(kRB * Geo<NP>::A) setup_rows_k(const Recon g, int rowspec_allowed) {
  constexpr int A = Geo<NP>::A, B = Geo<NP>::B, M = B / A, S = row_cap<NP>();
  __shared__ float2 tile[kRB * S];
  __shared__ float2 tw[NP];
  const int tid = threadIdx.x;
  const bool rows = rows_wanted(g, rowspec_allowed);
  const int j = blockIdx.x / (NP / kRB), rl = tid / A, p = tid % A;
  const int r = (int)(blockIdx.x % (NP / kRB)) * kRB + rl;
  const int2 pj = g.pos[j];
  const float2* xrow = g.xhat + (size_t)(pj.x + r) * g.n2 + pj.y;
  // all loads ahead of the products (tested and loaded pixel by pixel, this
  // took 98 us for 400 patches of 256^2)
  float2 x[B], d[B];
#pragma unroll
  for (int nb = 0; nb < B; ++nb) {
    const int c = p + A * nb;
    d[nb] = g.d[r * NP + c];
    x[nb] = xrow[c];
  }
#pragma unroll
  for (int nb = 0; nb < B; ++nb) x[nb] = start_state(g, d[nb], x[nb]);
  float2* out = g.t + (size_t)j * NP * NP + (size_t)r * NP;
  load_twiddles<NP>(tw, g.twn, tid, kRB * A);
  if (!rows) {
#pragma unroll
    for (int nb = 0; nb < B; ++nb) out[p + A * nb] = x[nb];
    return;
  }
  __syncthreads();
  row_fwd<NP>(x, tile + rl * S, p, tw);
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int ka = 0; ka < A; ++ka) out[p + A * m + B * ka] = cscale(x[m * A + ka], 1.f / (float)NP);
}

// Split layout: the starting states in their coset blocks (see Recon).
__global__ void __launch_bounds__(256) setup_split_k(const Recon g) {
  const int np2 = g.np * g.np, M = g.np / 2, MM = M * M, per = (np2 + 255) / 256;
  const int j = blockIdx.x / per, rem = (int)(blockIdx.x % per) * 256 + threadIdx.x;
  if (rem >= np2) return;
  const int2 pj = g.pos[j];
  const int ab = rem / MM, m = rem - ab * MM, m1 = m / M, m2 = m % M, a = ab >> 1, b = ab & 1;
  float2 h = make_float2(0.f, 0.f);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int q1 = q >> 1, q2 = q & 1, r = m1 + M * q1, c = m2 + M * q2;
    const float2 f = cmul(g.d[r * g.np + c], g.xhat[(size_t)(pj.x + r) * g.n2 + pj.y + c]);
    h = ((a * q1 + b * q2) & 1) ? csub(h, f) : cadd(h, f);
  }
  g.t[(size_t)j * np2 + rem] = cmul(h, g.twn[a * m1 + b * m2]);
}

// xhat = the starting object, x0 == nullptr standing for 1 + 0i (restricted to the covered pixels later); the
// FP64 normaliser image (the accumulator, not used yet) and S cleared.
__global__ void __launch_bounds__(256) setup_object_k(const Recon g, const float2* __restrict__ x0) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= g.n1 * g.n2) return;
  g.xhat[i] = x0 ? x0[i] : make_float2(1.f, 0.f);
  reinterpret_cast<double*>(g.num)[i] = 0.0;
  g.sold[i] = make_float2(0.f, 0.f);
}

// ---------------------------------------------------------------------------
// Lists
// ---------------------------------------------------------------------------

// Inclusive range test of [p, p + np) against [a, a + w).
__device__ __forceinline__ bool meets(int p, int np, int a, int w) { return p < a + w && p + np > a; }

// Gather tiles of positions [ja, jb): workgroup (tr, panel) writes the tiles
// of tile row tr and up to kPanel tile columns, each with the positions that
// overlap it in ascending order.  The workgroup keeps the positions that meet
// its rows, 256 at a time in order, in LDS; its waves then run over their tile
// columns, 64 positions to a ballot, first to count and then to write.  Where
// a list starts in tile_list is taken from a counter, so it depends on the
// order the workgroups run in; what a tile lists does not.
// `xcd`: tiles of a row ordered so that each XCD runs side-by-side ones.  The
// dispatcher sends workgroup b to XCD b mod 8, and each XCD has its own L2:
// slot b gets tile (b mod 8) q + b / 8 of the row (q = n / 8; the last n mod 8
// stay in place), and the second read of an edge line shared by two tiles
// hits its L2.  Without it (one launch, Np <= 128), rows of a multiple of 8
// tiles are rotated by their number, or the short lists of the object's edge
// columns would all be two XCDs' share.  `slots`: these places from the host,
// without the tiles that list nothing (see SetupChunk).
constexpr int kPanel = 1024;
__global__ void __launch_bounds__(256) setup_tiles_k(const Recon g, int ja, int jb, int lo, int tiles_c,
                                                     int tile0, int xcd, const int* __restrict__ slots) {
  __shared__ int lj[256], lr[256], lc[256], wsum[4];
  __shared__ int count[kPanel], at[kPanel];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lo + (int)blockIdx.x * GT_R, tc0 = (int)blockIdx.y * kPanel;
  const int nt = tiles_c - tc0 < kPanel ? tiles_c - tc0 : kPanel;
  for (int t = tid; t < nt; t += 256) count[t] = 0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int j0 = ja; j0 < jb; j0 += 256) {
      const int j = j0 + tid;
      const int2 p = j < jb ? g.pos[j] : make_int2(0, 0);
      const bool in = j < jb && meets(p.x, g.np, row, GT_R);
      const unsigned long long m = __ballot(in);
      __syncthreads();  // the last batch's lists are done with
      if (lane == 0) wsum[wave] = __popcll(m);
      __syncthreads();
      int base = 0, n = 0;
      for (int w = 0; w < 4; ++w) {
        if (w < wave) base += wsum[w];
        n += wsum[w];
      }
      if (in) {
        const int k = base + __popcll(m & ((1ull << lane) - 1));
        lj[k] = j;
        lr[k] = (p.x - row) * 65536;
        lc[k] = p.y;
      }
      __syncthreads();
      for (int t = wave; t < nt; t += 4) {
        const int c0 = (tc0 + t) * GT_C;
        int cur = pass ? at[t] : 0;
        for (int k0 = 0; k0 < n; k0 += 64) {
          const int k = k0 + lane;
          const bool hit = k < n && meets(lc[k], g.np, c0, GT_C);
          const unsigned long long h = __ballot(hit);
          if (pass && hit)
            g.tile_list[cur + __popcll(h & ((1ull << lane) - 1))] =
                make_int2(lj[k], lr[k] | ((lc[k] - c0) & 0xffff));
          cur += __popcll(h);
        }
        // each tile column belongs to one wave
        if (lane == 0) {
          if (pass) at[t] = cur;
          else count[t] += cur;
        }
      }
    }
    __syncthreads();
    if (pass == 0) {
      const int q = tiles_c / 8;
      for (int t = tid; t < nt; t += 256) {
        const int n = count[t], start = n ? atomicAdd(g.cursor, n) : 0, tc = tc0 + t;
        at[t] = start;
        int slot = xcd && tc < 8 * q ? (tc % q) * 8 + tc / q : tc;
        if (!xcd && tiles_c % 8 == 0) slot = (tc + (int)blockIdx.x) % tiles_c;
        slot += (int)blockIdx.x * tiles_c;
        if (slots) slot = slots[(size_t)blockIdx.x * tiles_c + tc];
        if (slot >= 0) g.tiles[(size_t)tile0 + slot] = make_int4(start, n, row, tc * GT_C);
      }
      __syncthreads();
    }
  }
}

// Row-spectrum states: positions [ja, jb) by descending patch row (so that
// the patch row they have on a given object row ascends), ties in ascending
// order, as (j, row, column).
__global__ void __launch_bounds__(256) setup_order_k(const Recon g, int ja, int jb) {
  __shared__ int4 rows[64];
  const int tid = threadIdx.x, j = ja + (int)blockIdx.x * 256 + tid;
  const int2 p = j < jb ? g.pos[j] : make_int2(0, 0);
  int rank = 0;
  for (int k0 = ja; k0 < jb; k0 += 256) {
    __syncthreads();
    // (rows past the end rank below every row)
    reinterpret_cast<int*>(rows)[tid] = k0 + tid < jb ? g.pos[k0 + tid].x : -1;
    __syncthreads();
#pragma unroll 8
    for (int k = 0; k < 64; ++k) {
      const int4 r = rows[k];
      const int b = j - (k0 + 4 * k);   // positions before j win ties
      rank += (r.x > p.x) | ((r.x == p.x) & (b > 0));
      rank += (r.y > p.x) | ((r.y == p.x) & (b > 1));
      rank += (r.z > p.x) | ((r.z == p.x) & (b > 2));
      rank += (r.w > p.x) | ((r.w == p.x) & (b > 3));
    }
  }
  if (j < jb) g.order[ja + rank] = make_int4(j, p.x, p.y, 0);
}

// Row items of positions [ja, jb): a wave per (object row, CR_W-pixel
// segment), listing the positions whose patch covers the row and meets the
// segment, by patch row (so that a round of the row consensus shares few
// weight rows), then each round of rn entries by patch column (so that the
// entries covering a run of pixels are consecutive in it); ties in ascending
// order.  The consensus sums each pixel in this order.  `rows`: the rows and
// segments from the host, without those that list nothing (see SetupChunk).
__global__ void __launch_bounds__(256) setup_row_items_k(const Recon g, int ja, int jb, int lo, int nitems,
                                                         int nseg, int item0, int rn,
                                                         const int2* __restrict__ rows) {
  const int lane = threadIdx.x & 63;
  const int item = (int)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= nitems) return;
  // segment by segment: row by row, the two segments of a 1280-wide object
  // alternated, and as workgroup b runs on XCD b mod 8 the long first ones all
  // fell to the even XCDs (960 positions of 192^2: consensus 162 -> 101 us)
  const int nrows = nitems / nseg;
  int row, col;
  if (rows) {
    const int2 rc = rows[item];
    row = rc.x;
    col = rc.y;
  } else {
    row = lo + item % nrows;
    col = (item / nrows) * CR_W;
  }
  __shared__ int4 pend[4][128];  // per wave: entries not yet written, in order
  int4* pw = pend[threadIdx.x >> 6];
  const auto covers = [&](const int4& e, int k) {
    return k < jb && (unsigned)(row - e.y) < (unsigned)g.np && meets(e.z, g.np, col, CR_W);
  };
  int n = 0;
  for (int k0 = ja; k0 < jb; k0 += 256) {  // four independent loads a step
    int4 e[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + 64 * q + lane;
      e[q] = g.order[k < jb ? k : ja];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) n += __popcll(__ballot(covers(e[q], k0 + 64 * q + lane)));
  }
  int start = 0;
  if (lane == 0) {
    start = n ? atomicAdd(g.cursor + 1, n) : 0;
    g.citems[item0 + item] = make_int4(start, n, row, col);
  }
  start = __builtin_amdgcn_readfirstlane(start);
  // writes the first m <= 64 pending entries as one round, by column
  int out = start, held = 0;
  const auto round = [&](int m) {
    const int4 e = lane < m ? pw[lane] : make_int4(0, 0, 0x7fffffff, 0);
    int rank = 0;
    for (int k = 0; k < m; ++k) {
      const int c = __builtin_amdgcn_readlane(e.z, k);
      rank += (c < e.z) | ((c == e.z) & (k < lane));
    }
    if (lane < m) g.clist[out + rank] = e;
    out += m;
  };
  for (int k0 = ja; k0 < jb && out + held < start + n; k0 += 64) {
    const int k = k0 + lane;
    const int4 e = g.order[k < jb ? k : ja];
    const bool hit = covers(e, k);
    const unsigned long long h = __ballot(hit);
    if (h == 0) continue;
    if (hit) pw[held + __popcll(h & ((1ull << lane) - 1))] = make_int4(e.x, row - e.y, e.z, 0);
    held += __popcll(h);
    wave_sync();
    while (held >= rn) {
      round(rn);
      held -= rn;
      const int4 a = lane < held ? pw[rn + lane] : make_int4(0, 0, 0, 0);
      const int4 b = 64 + lane < held ? pw[rn + 64 + lane] : make_int4(0, 0, 0, 0);
      wave_sync();
      pw[lane] = a;
      if (64 + lane < 128 - rn) pw[64 + lane] = b;
      wave_sync();
    }
  }
  if (held > 0) round(held);
}

// Lambda = sum_j P_j^t omega (eq. (11)) in FP64 over one chunk's tiles, into
// the accumulator image viewed as FP64, and (PMACE) the consensus sum S of the
// starting states.  These are patches of one object (xhat holds it), so S
// needs the probe tables only; its terms and their order are those of the
// gather over the stored states.  An entry that does not cover the pixel adds
// exactly zero: the object there may be anything (a pixel that no patch covers
// may hold NaN, and 0 NaN is not 0).  GT_K threads share a pixel, thread k adding
// the entries k, k + GT_K, ...; their sums are added in order.  Bound by the
// L2 reads of the tables (24 B per patch pixel).
__global__ void __launch_bounds__(GT_THREADS) setup_sums_k(const Recon g, int first_tile) {
  constexpr int NPX = GT_R * GT_C, U = 8;
  __shared__ double ps[GT_K > 1 ? (GT_K - 1) * NPX : 1];
  __shared__ float2 pt[GT_K > 1 ? (GT_K - 1) * NPX : 1];
  const int tid = threadIdx.x, pxl = tid % NPX, np = g.np;
  const int part = __builtin_amdgcn_readfirstlane(tid / NPX);
  const int4 ti = g.tiles[first_tile + blockIdx.x];
  if (ti.y == 0) return;
  const int lr = pxl / GT_C, lc = pxl % GT_C, R = ti.z + lr, C = ti.w + lc;
  const bool inside = R < g.n1 && C < g.n2;
  const size_t px = inside ? (size_t)R * g.n2 + C : 0;
  const float2 x = g.xhat[px];
  const int2* list = g.tile_list + ti.x;
  double acc = 0.0;
  float ax = 0.f, ay = 0.f;
  for (int i0 = part; i0 < ti.y; i0 += U * GT_K) {
    double om[U];
    float2 d[U], w[U];
    bool in[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int i = i0 + k * GT_K;
      const int2 e = list[i < ti.y ? i : ti.y - 1];
      const unsigned rr = (unsigned)(lr - (e.y >> 16)), cc = (unsigned)(lc - (int)(short)e.y);
      in[k] = rr < (unsigned)np && cc < (unsigned)np && i < ti.y;
      const unsigned o = in[k] ? rr * np + cc : 0u;
      om[k] = in[k] ? g.omega64[o] : 0.0;
      d[k] = g.d[o];
      w[k] = in[k] ? g.gw[o] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      float2 u = start_state(g, d[k], x);
      if (!in[k]) u = make_float2(0.f, 0.f);
      acc += om[k];
      ax = fmaf(w[k].x, u.x, fmaf(-w[k].y, u.y, ax));
      ay = fmaf(w[k].x, u.y, fmaf(w[k].y, u.x, ay));
    }
  }
  if constexpr (GT_K > 1) {
    if (part > 0) {
      ps[(part - 1) * NPX + pxl] = acc;
      pt[(part - 1) * NPX + pxl] = make_float2(ax, ay);
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int k = 0; k < GT_K - 1; ++k) {
      acc += ps[k * NPX + pxl];
      ax += pt[k * NPX + pxl].x;
      ay += pt[k * NPX + pxl].y;
    }
  }
  if (!inside) return;
  reinterpret_cast<double*>(g.num)[px] += acc;
  if (g.method == kPMACE) g.sold[px] = cadd(g.sold[px], make_float2(ax, ay));
}

// Lambda^{-1} (0 where Lambda = 0: no patch, or only zero weights, covers the
// pixel), the starting images, the work items of the NRMSE, the descriptor.
__global__ void __launch_bounds__(256) setup_images_k(const Recon g, Recon* rec, int2* ritems) {
  if (blockIdx.x == 0) {
    const unsigned* src = reinterpret_cast<const unsigned*>(&g);
    for (int w = threadIdx.x; w < (int)(sizeof(Recon) / 4); w += 256)
      reinterpret_cast<unsigned*>(rec)[w] = src[w];
  }
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < g.n_red) ritems[i] = make_int2(0, i);
  if (i >= g.n1 * g.n2) return;
  const double lam = reinterpret_cast<const double*>(g.num)[i];
  const float li = lam != 0.0 ? (float)(1.0 / lam) : 0.f;
  const float2 x = g.xhat[i], zero = make_float2(0.f, 0.f);
  const float2 xh = li > 0.f ? x : zero;
  g.laminv[i] = li;
  g.xhat[i] = xh;
  g.xbar[i] = g.method == kSharpPlus ? xh : zero;
  g.num[i] = zero;
}

hipError_t launch_setup_inputs(const Recon& h, const SetupInputs& in, int* fitem, hipStream_t st) {
  const int np2 = h.np * h.np;
  hipLaunchKernelGGL(setup_clear_k, dim3(1), dim3(256), 0, st, h, fitem);
  hipLaunchKernelGGL(setup_tables_k, dim3(blocks_for(np2 > h.J ? np2 : h.J, 256)), dim3(256), 0, st, h, in.probe,
                     in.pos, in.kappa, in.rho, in.split_allowed);
  hipLaunchKernelGGL(setup_object_k, dim3(blocks_for((long long)h.n1 * h.n2, 256)), dim3(256), 0, st, h, in.x0);
  if (in.split_allowed) return hipGetLastError();  // the rest waits for the layout (launch_setup_states)
  return launch_setup_states(h, in, st);
}

hipError_t launch_setup_states(const Recon& h, const SetupInputs& in, hipStream_t st) {
  const int np2 = h.np * h.np, per = (np2 + 255) / 256;
  const long long total = (long long)h.J * np2;
  // np is a multiple of 16, so whole patches are float4s where z is aligned
  if (!in.centered && !h.split && (reinterpret_cast<size_t>(in.z) & 15) == 0)
    hipLaunchKernelGGL(setup_amplitudes4_k, dim3(blocks_for(total / 4, 256)), dim3(256), 0, st, h,
                       reinterpret_cast<const float4*>(in.z), in.yscale, total / 4);
  else
    hipLaunchKernelGGL(setup_amplitudes_k, dim3((unsigned)h.J * per), dim3(256), 0, st, h, in.z, in.yscale,
                       in.centered);
  if (h.split) {
    hipLaunchKernelGGL(setup_split_k, dim3((unsigned)h.J * per), dim3(256), 0, st, h);
    return hipGetLastError();
  }
  switch (h.np) {
#define PMACE_ROWS(N)                                                                                  \
  case N:                                                                                              \
    hipLaunchKernelGGL(setup_rows_k<N>, dim3((unsigned)h.J * (N / kRB)), dim3(kRB * Geo<N>::A), 0, st, \
                       h, in.rowspec_allowed);                                                         \
    break;
    PMACE_ROWS(160)
    PMACE_ROWS(192)
    PMACE_ROWS(256)
#undef PMACE_ROWS
    default: hipLaunchKernelGGL(setup_states_k, dim3((unsigned)h.J * per), dim3(256), 0, st, h);
  }
  return hipGetLastError();
}

hipError_t launch_setup_lists(const Recon& h, const SetupChunk& k, int tiles_c, int nseg, int rn, hipStream_t st) {
  // the host's lists go where the consensus image will be (4 B a tile and 8 B
  // an item in 8 B a pixel)
  const size_t all = (size_t)k.tiles_r * tiles_c;
  int* slots = k.slots ? reinterpret_cast<int*>(h.xbar) : nullptr;
  int2* rows = k.rows ? reinterpret_cast<int2*>(h.xbar) + (all + 1) / 2 : nullptr;
  if (slots) {
    const hipError_t e = hipMemcpyAsync(slots, k.slots, all * 4, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
  }
  if (rows) {
    const hipError_t e = hipMemcpyAsync(rows, k.rows, (size_t)k.nitems * 8, hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(setup_tiles_k, dim3(k.tiles_r, (tiles_c + kPanel - 1) / kPanel), dim3(256), 0, st, h, k.ja,
                     k.jb, k.lo, tiles_c, k.tile0, h.np > 128 ? 1 : 0, slots);
  if (h.rowspec) {
    hipLaunchKernelGGL(setup_order_k, dim3(blocks_for(k.jb - k.ja, 256)), dim3(256), 0, st, h, k.ja, k.jb);
    hipLaunchKernelGGL(setup_row_items_k, dim3(blocks_for(k.nitems, 4)), dim3(256), 0, st, h, k.ja, k.jb, k.lo,
                       k.nitems, nseg, k.item0, rn, rows);
  }
  hipLaunchKernelGGL(setup_sums_k, dim3(k.ntiles), dim3(GT_THREADS), 0, st, h, k.tile0);
  return hipGetLastError();
}

hipError_t launch_setup_images(const Recon& h, Recon* rec, int2* ritems, hipStream_t st) {
  if (h.has_zero) {
    const int A = line_threads(h.np);
    hipLaunchKernelGGL(setup_zeros_k, dim3(blocks_for(h.np * A, 256)), dim3(256), 0, st, h, A);
  }
  const long long n = (long long)h.n1 * h.n2;
  hipLaunchKernelGGL(setup_images_k, dim3(blocks_for(n, 256)), dim3(256), 0, st, h, rec, ritems);
  return hipGetLastError();
}

}  // namespace pmace
