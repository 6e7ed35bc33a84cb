// Binned matter power spectrum (Koda et al. 2015, Sec. 3.3): P = |delta_k|^2 / V
// over the half space {kz > 0} U {kz = 0, ky > 0} U {kz = 0, ky = 0, kx > 0},
// delta_k = (V / Ng^3) DFT[delta] / W_CIC(k), W_CIC = prod sinc^2(pi n_e / Ng),
// averaged per |k| bin with the mean |k|.  Only |k| <= pi Ng / L is used.
//
// Up to 512 bins (density / momentum spectra: what 64 KB of LDS hold, 441 at
// side 32 and 387 at 2048): k_pk_rows below.  More bins: workgroup (bin b, chunk
// c) visits the (kx, ky) rows of chunk c; a thread walks one row's kz range that
// can fall in bin b (found analytically, each mode then tested exactly), accumulating in FP64
// in a fixed order; the workgroup sums its threads by a fixed tree, and a
// second kernel sums the chunks in order.
#include "cola_device.h"
#include "cola_internal.h"

namespace cola {

constexpr int kPT = 256;

__device__ __forceinline__ double sinc_pi(double x) {  // sin(pi x) / (pi x)
  if (x == 0.0) return 1.0;
  const double a = 3.14159265358979323846 * x;
  return sin(a) / a;
}

__global__ __launch_bounds__(kPT) void k_pk_bin(const float2* __restrict__ spec, int ng, long cols,
                                                double kf, double kmax, double vol_fac,
                                                const double* __restrict__ edges,
                                                int nbins, double* __restrict__ partial, int nchunk,
                                                int deconvolve) {
  __shared__ double sk[kPT], sp[kPT], sn[kPT];
  const int b = blockIdx.y;
  const int c = blockIdx.x;
  const double e0 = edges[b], e1 = edges[b + 1];
  const double lo2 = (e0 / kf) * (e0 / kf), hi2 = (e1 / kf) * (e1 / kf);
  const long nrows = (long)ng * ng;
  const long per = (nrows + nchunk - 1) / nchunk;
  const long r0 = (long)c * per, r1 = r0 + per < nrows ? r0 + per : nrows;
  double ak = 0.0, ap = 0.0, an = 0.0;
  const int h = ng / 2;
  for (long r = r0 + threadIdx.x; r < r1; r += kPT) {
    const int ix = (int)(r / ng), iy = (int)(r - (long)ix * ng);
    const int nx = ix < h ? ix : ix - ng, ny = iy < h ? iy : iy - ng;  // DFT signed indices
    const double p2 = (double)nx * nx + (double)ny * ny;
    if (p2 >= hi2) continue;
    int zlo = 0;
    if (lo2 > p2) zlo = (int)floor(sqrt(lo2 - p2)) - 1;
    if (zlo < 0) zlo = 0;
    int zhi = (int)ceil(sqrt(hi2 - p2)) + 1;
    if (zhi > h) zhi = h;
    const double wxy = sinc_pi((double)nx / ng) * sinc_pi((double)ny / ng);
    for (int nz = zlo; nz <= zhi; ++nz) {
      if (nz == 0 && !(ny > 0 || (ny == 0 && nx > 0))) continue;
      const double n2 = p2 + (double)nz * nz;
      const double kk = kf * sqrt(n2);
      if (kk > kmax) continue;
      if (!(kk >= e0 && kk < e1)) continue;
      const float2 v = spec[r * cols + nz];
      double w = deconvolve ? wxy * sinc_pi((double)nz / ng) : 1.0;
      w = w * w;
      const double re = (double)v.x, im = (double)v.y;
      ap += (re * re + im * im) * vol_fac / (w * w);
      ak += kk;
      an += 1.0;
    }
  }
  sk[threadIdx.x] = ak;
  sp[threadIdx.x] = ap;
  sn[threadIdx.x] = an;
  __syncthreads();
  for (int o = kPT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sk[threadIdx.x] += sk[threadIdx.x + o];
      sp[threadIdx.x] += sp[threadIdx.x + o];
      sn[threadIdx.x] += sn[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* o = partial + ((long)b * nchunk + c) * 3;
    o[0] = sk[0];
    o[1] = sp[0];
    o[2] = sn[0];
  }
}

__global__ void k_pk_reduce(const double* __restrict__ partial, int nbins, int nchunk,
                            double* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  double s0 = 0, s1 = 0, s2 = 0;
  for (int c = 0; c < nchunk; ++c) {
    const double* p = partial + ((long)b * nchunk + c) * 3;
    s0 += p[0];
    s1 += p[1];
    s2 += p[2];
  }
  out[3 * b + 0] = s0;
  out[3 * b + 1] = s1;
  out[3 * b + 2] = s2;
}

// Density / line-of-sight momentum spectra over the same modes and bins:
// per bin, sums of |k|, |d|^2, sign(n_axis) Im(d p*), |p|^2 (each scaled and
// deconvolved like P(k)) and the count; the same fixed-order reduction.
__global__ __launch_bounds__(kPT) void k_pk_cross(const float2* __restrict__ sd, const float2* __restrict__ sp,
                                                  int ng, long cols, double kf, double kmax, double vol_fac,
                                                  const double* __restrict__ edges, int nbins, int axis,
                                                  double* __restrict__ partial, int nchunk) {
  __shared__ double acc[5][kPT];
  const int b = blockIdx.y;
  const int c = blockIdx.x;
  const double e0 = edges[b], e1 = edges[b + 1];
  const double lo2 = (e0 / kf) * (e0 / kf), hi2 = (e1 / kf) * (e1 / kf);
  const long nrows = (long)ng * ng;
  const long per = (nrows + nchunk - 1) / nchunk;
  const long r0 = (long)c * per, r1 = r0 + per < nrows ? r0 + per : nrows;
  double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const int h = ng / 2;
  for (long r = r0 + threadIdx.x; r < r1; r += kPT) {
    const int ix = (int)(r / ng), iy = (int)(r - (long)ix * ng);
    const int nx = ix < h ? ix : ix - ng, ny = iy < h ? iy : iy - ng;
    const double p2 = (double)nx * nx + (double)ny * ny;
    if (p2 >= hi2) continue;
    int zlo = 0;
    if (lo2 > p2) zlo = (int)floor(sqrt(lo2 - p2)) - 1;
    if (zlo < 0) zlo = 0;
    int zhi = (int)ceil(sqrt(hi2 - p2)) + 1;
    if (zhi > h) zhi = h;
    const double wxy = sinc_pi((double)nx / ng) * sinc_pi((double)ny / ng);
    for (int nz = zlo; nz <= zhi; ++nz) {
      if (nz == 0 && !(ny > 0 || (ny == 0 && nx > 0))) continue;
      const double n2 = p2 + (double)nz * nz;
      const double kk = kf * sqrt(n2);
      if (kk > kmax) continue;
      if (!(kk >= e0 && kk < e1)) continue;
      const int na = axis == 0 ? nx : axis == 1 ? ny : nz;
      const double sg = na > 0 ? 1.0 : na < 0 ? -1.0 : 0.0;
      const float2 d = sd[r * cols + nz], p = sp[r * cols + nz];
      double w = wxy * sinc_pi((double)nz / ng);
      w = w * w;
      const double f = vol_fac / (w * w);
      const double dr = d.x, di = d.y, pr = p.x, pi = p.y;
      a[0] += kk;
      a[1] += (dr * dr + di * di) * f;
      a[2] += sg * (di * pr - dr * pi) * f;
      a[3] += (pr * pr + pi * pi) * f;
      a[4] += 1.0;
    }
  }
  for (int q = 0; q < 5; ++q) acc[q][threadIdx.x] = a[q];
  __syncthreads();
  for (int o = kPT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int q = 0; q < 5; ++q) acc[q][threadIdx.x] += acc[q][threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* o = partial + ((long)b * nchunk + c) * 5;
    for (int q = 0; q < 5; ++q) o[q] = acc[q][0];
  }
}

__global__ void k_pk_cross_reduce(const double* __restrict__ partial, int nbins, int nchunk,
                                  double* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int c = 0; c < nchunk; ++c)
    for (int q = 0; q < 5; ++q) s[q] += partial[((long)b * nchunk + c) * 5 + q];
  for (int q = 0; q < 5; ++q) out[5 * b + q] = s[q];
}

// ---------------------------------------------------------------------------
// Spectra of few bins (pk_rows_plan), one pass over the modes.  The sums
// by (bin, chunk) above visit every (kx, ky) row once per bin and take two
// sines per visited mode; here a wave visits each mode of its rows once, and
// the windows come from a table in LDS.  What bounds it is the FP64 arithmetic
// of a mode (a square root and the window) and, with many bins, the runs handed
// over.  768 mesh: 0.9 ms at 1 and 8 bins, 1.1 at 40, 2.1 at 512 (0.9, 1.0, 1.7
// with the lanes' additions left in the order in which the LDS takes them),
// against 5.4, 5.8, 3.4 and 2.9 ms with the sums by (bin, chunk), which remain
// for more bins (their LDS sums no longer fit).
//
// Bins by integers: n2 = nx^2 + ny^2 + nz^2 decides |k| = kf sqrt(n2), so bin b
// is thr[b] <= n2 < thr[b + 1] with thr[b] the smallest n2 whose |k| reaches
// edge b (same expression, same rounding), and |k| <= kmax is n2 < top.
// A lane keeps one nz and goes through the rows, along which n2 changes
// little, so it adds into registers and passes its sums on only when its bin
// changes or its mode is not counted, to LDS sums that belong to its wave alone.
// The sums do not vary from run to run: every run handed over ended in the same
// row (the last one that the wave visited), where the bin does not fall from one
// lane to the next, so the lanes of one bin are found by a look at the lane before
// and add in lane order, one instruction each; a wave's LDS instructions complete
// in their order, and the waves and chunks are added in order.
constexpr int kRowBins = 512;        // largest bin count: LDS of a workgroup, chunks that the partials hold
constexpr int kRowWaves = 4;
constexpr int kRowMaxChunks = 1024;  // workgroups

__device__ __forceinline__ uint32_t first_n2(double e, double kf, bool strict) {
  // smallest integer n2 >= 0 with kf sqrt(n2) >= e (strict: > e); 2^24 where there is none below
  const double q = e / kf;
  if (!(q > 0.0)) return strict && q == 0.0 ? 1u : 0u;
  const double q2 = q * q;
  if (!(q2 < 16777216.0)) return 16777216u;
  uint32_t n = (uint32_t)q2;
  n = n > 2u ? n - 2u : 0u;
  for (;; ++n) {
    const double k = kf * sqrt((double)n);
    if (strict ? k > e : k >= e) return n;
  }
}

// NS sums per bin and the mode count.  CROSS: |k|, |d|^2, sign(n_axis) Im(d p*),
// |p|^2; otherwise |k|, |d|^2.
template <bool CROSS>
__global__ __launch_bounds__(64 * kRowWaves) void k_pk_rows(
    const float2* __restrict__ sd, const float2* __restrict__ sp, int ng, long cols, double kf, double kmax,
    double vol_fac, const double* __restrict__ edges, int nbins, int axis, double* __restrict__ partial,
    int nchunk, int deconvolve) {
  constexpr int NS = CROSS ? 4 : 2, T = 64 * kRowWaves, kU = 4;
  extern __shared__ double smem[];
  double* acc = smem;                                        // [wave][bin][NS]
  double* win = acc + (size_t)kRowWaves * nbins * NS;        // 1 / sinc^4 per axis index
  uint32_t* thr = reinterpret_cast<uint32_t*>(win + ng / 2 + 1);  // nbins + 1
  uint32_t* cnt = thr + nbins + 1;                           // [wave][bin]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = ng / 2;
  for (int i = tid; i < kRowWaves * nbins * NS; i += T) acc[i] = 0.0;
  for (int i = tid; i < kRowWaves * nbins; i += T) cnt[i] = 0u;
  for (int i = tid; i <= h; i += T) {
    const double s = deconvolve ? sinc_pi((double)i / ng) : 1.0;
    win[i] = 1.0 / ((s * s) * (s * s));
  }
  for (int i = tid; i <= nbins; i += T) thr[i] = first_n2(edges[i], kf, false);
  const uint32_t top = first_n2(kmax, kf, true);
  __syncthreads();
  const uint32_t lo = thr[0], hi = min(thr[nbins], top);
  double* wacc = acc + (size_t)wave * nbins * NS;
  uint32_t* wcnt = cnt + wave * nbins;

  double run[NS];                                            // the lane's sums of bin cur
#pragma unroll
  for (int q = 0; q < NS; ++q) run[q] = 0.0;
  uint32_t nrun = 0, tlo, thi;                               // bin cur: tlo <= n2 < thi
  int cur;
  // Hands over the runs of the lanes with out set (every lane of the wave takes
  // part): the lanes of one bin one after the other, no two in one instruction.
  auto flush = [&](bool out) {
    const uint64_t f = __ballot(out);
    if (f == 0) return;
    const uint64_t below = f & ((1ull << lane) - 1);
    const int pb = __shfl(cur, below ? 63 - __builtin_clzll(below) : lane, 64);
    const uint64_t heads = __ballot(out && (below == 0 || pb != cur));
    int rank = -1;                                           // place among the lanes of its bin
    if (out) {
      const uint64_t h = heads & (~0ull >> (63 - lane));
      rank = __popcll(below >> (63 - __builtin_clzll(h)));
      atomicAdd(&wcnt[cur], nrun);
    }
    for (int r = 0; __any(rank >= r); ++r)
      if (rank == r)
#pragma unroll
        for (int q = 0; q < NS; ++q)
          __hip_atomic_fetch_add(&wacc[cur * NS + q], run[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (out) {
#pragma unroll
      for (int q = 0; q < NS; ++q) run[q] = 0.0;
      nrun = 0;
    }
  };

  const int nrows = ng * ng, nw = nchunk * kRowWaves;
  const int gw = (int)blockIdx.x * kRowWaves + wave;
  const int per = (nrows + nw - 1) / nw;
  const int r0 = min(gw * per, nrows), r1 = min(r0 + per, nrows);
  for (int z0 = 0; z0 <= h; z0 += 64) {
    const int nz = z0 + lane;
    const bool zin = nz <= h;
    const double wz = win[zin ? nz : h];
    cur = -1;
    tlo = 1u;
    thi = 0u;
    for (int rb = r0; rb < r1; rb += kU) {
      float2 d[kU], p[kU];
      uint32_t p2[kU];
      int sx[kU], sy[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int r = min(rb + u, nrows - 1);
        const int ix = r / ng, iy = r - ix * ng;
        sx[u] = ix < h ? ix : ix - ng;
        sy[u] = iy < h ? iy : iy - ng;
        p2[u] = rb + u < r1 ? (uint32_t)(sx[u] * sx[u] + sy[u] * sy[u]) : 16777216u;
        const bool in = zin && p2[u] + (uint32_t)(z0 * z0) < hi;
        d[u] = in ? sd[(long)r * cols + nz] : make_float2(0.f, 0.f);
        if constexpr (CROSS) p[u] = in ? sp[(long)r * cols + nz] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        if (p2[u] + (uint32_t)(z0 * z0) >= hi) continue;     // wave-uniform: nothing of the row is left
        const uint32_t n2 = p2[u] + (uint32_t)(nz * nz);
        const bool in = zin && n2 >= lo && n2 < hi && (nz > 0 || sy[u] > 0 || (sy[u] == 0 && sx[u] > 0));
        const bool same = in && n2 >= tlo && n2 < thi;
        flush(nrun > 0 && !same);
        if (!in) continue;
        if (!same) {
          if (cur < 0) {                                     // the last edge not above n2
            int a = 0, e = nbins;
            while (e - a > 1) {
              const int m = (a + e) >> 1;
              if (thr[m] <= n2) a = m; else e = m;
            }
            cur = a;
          } else {                                           // mostly the next bin or the one before
            while (thr[cur + 1] <= n2) ++cur;
            while (thr[cur] > n2) --cur;
          }
          tlo = thr[cur];
          thi = thr[cur + 1];
        }
        const double f = vol_fac * (win[abs(sx[u])] * win[abs(sy[u])] * wz);
        const double dr = d[u].x, di = d[u].y;
        run[0] += kf * sqrt((double)n2);
        run[1] += (dr * dr + di * di) * f;
        if constexpr (CROSS) {
          const double pr = p[u].x, pi = p[u].y;
          const int na = axis == 0 ? sx[u] : axis == 1 ? sy[u] : nz;
          run[2] += (na > 0 ? 1.0 : na < 0 ? -1.0 : 0.0) * (di * pr - dr * pi) * f;
          run[3] += (pr * pr + pi * pi) * f;
        }
        ++nrun;
      }
    }
    flush(nrun > 0);
  }
  __syncthreads();
  for (int b = tid; b < nbins; b += T) {
    double s[NS + 1];
    for (int q = 0; q <= NS; ++q) s[q] = 0.0;
    for (int w = 0; w < kRowWaves; ++w) {
      for (int q = 0; q < NS; ++q) s[q] += acc[((size_t)w * nbins + b) * NS + q];
      s[NS] += (double)cnt[w * nbins + b];
    }
    double* o = partial + ((long)b * nchunk + blockIdx.x) * (NS + 1);
    for (int q = 0; q <= NS; ++q) o[q] = s[q];
  }
}

// Sums the chunks of a bin: one workgroup per bin, strided partial sums and a
// fixed tree.
template <int NV>
__global__ __launch_bounds__(256) void k_pk_rows_reduce(const double* __restrict__ partial, int nchunk,
                                                        double* __restrict__ out) {
  __shared__ double s[NV][256];
  const int b = blockIdx.x, t = threadIdx.x;
  double a[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) a[q] = 0.0;
  for (int c = t; c < nchunk; c += 256)
#pragma unroll
    for (int q = 0; q < NV; ++q) a[q] += partial[((long)b * nchunk + c) * NV + q];
#pragma unroll
  for (int q = 0; q < NV; ++q) s[q][t] = a[q];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o)
#pragma unroll
      for (int q = 0; q < NV; ++q) s[q][t] += s[q][t + o];
    __syncthreads();
  }
  if (t < NV) out[(long)b * NV + t] = s[t][0];
}

namespace {
size_t pk_rows_lds(int ng, int nbins, int ns) {
  return sizeof(double) * ((size_t)kRowWaves * nbins * ns + ng / 2 + 1) +
         sizeof(uint32_t) * (nbins + 1 + (size_t)kRowWaves * nbins);
}
// Whether the row kernel serves nbins bins of nv sums (64 KB of LDS at most),
// and its chunks: at least 16 rows per wave, at most what the partials (cap
// doubles) hold.
bool pk_rows_plan(int ng, int nbins, int nv, long cap, int* nchunk) {
  if (nbins > kRowBins || pk_rows_lds(ng, nbins, nv - 1) > 65536) return false;
  long n = (long)ng * ng / (16 * kRowWaves);
  n = n < kRowMaxChunks ? n : kRowMaxChunks;
  const long fit = cap / ((long)nbins * nv);
  *nchunk = (int)(n < fit ? (n > 0 ? n : 1) : fit);
  return true;
}
}  // namespace

// P(k) adjoint: for half-space modes with |k| <= k_Nyq in bin b,
//   u_k = cbar_b / N_b (V/Ng^3)^2 / V / W_CIC(k)^2,
// and the real field  deltabar(x) = sum_modes 2 u_k Re(X_k e^{ikx})  is written
// as a half spectrum Z for the unnormalised complex-to-real inverse:
//   0 < nz < Ng/2: Z_k = u X_k (the inverse doubles it);  nz = 0: Z_k = u X_k and
//   Z_{-k} = conj(u X_k) (Hermitian plane);  nz = Ng/2: Z_k = 2 u X_k.
// A wave takes whole rows, lanes along nz, and writes every value of Z (zero
// where no bin counts the mode, and in the row padding); bins and windows as
// in k_pk_rows.  An element of the nz = 0 plane outside the half space takes
// its value from its conjugate partner.
__global__ __launch_bounds__(64 * kRowWaves) void k_pk_adj_rows(
    const float2* __restrict__ X, float2* __restrict__ Z, int ng, int cols, double kf, double kmax, double vol_fac,
    const double* __restrict__ edges, int nbins, const double* __restrict__ cbar, const double* __restrict__ sums) {
  extern __shared__ double smem[];
  double* win = smem;
  double* cb = win + ng / 2 + 1;
  uint32_t* thr = reinterpret_cast<uint32_t*>(cb + nbins);
  const int tid = threadIdx.x, lane = tid & 63, h = ng / 2;
  for (int i = tid; i <= h; i += 64 * kRowWaves) {
    const double s = sinc_pi((double)i / ng);
    win[i] = 1.0 / ((s * s) * (s * s));
  }
  for (int i = tid; i < nbins; i += 64 * kRowWaves) {
    const double n = sums[3 * i + 2];
    cb[i] = n > 0 ? cbar[i] / n * vol_fac : 0.0;
  }
  for (int i = tid; i <= nbins; i += 64 * kRowWaves) thr[i] = first_n2(edges[i], kf, false);
  const uint32_t top = first_n2(kmax, kf, true);
  __syncthreads();
  const uint32_t lo = thr[0], hi = min(thr[nbins], top);
  const int nrows = ng * ng, nw = (int)gridDim.x * kRowWaves;
  for (int r = (int)blockIdx.x * kRowWaves + (tid >> 6); r < nrows; r += nw) {
    const int ix = r / ng, iy = r - ix * ng;
    const int nx = ix < h ? ix : ix - ng, ny = iy < h ? iy : iy - ng;
    const uint32_t p2 = (uint32_t)(nx * nx + ny * ny);
    const double wxy = win[abs(nx)] * win[abs(ny)];
    for (int nz = lane; nz < cols; nz += 64) {
      float2 z = make_float2(0.f, 0.f);
      const uint32_t n2 = p2 + (uint32_t)(nz * nz);
      if (nz <= h && n2 >= lo && n2 < hi && n2 > 0) {
        // outside the half space: the partner (-nx, -ny), unless that is outside too
        const bool in = nz > 0 || ny > 0 || (ny == 0 && nx > 0);
        const int jx = (ng - ix) % ng, jy = (ng - iy) % ng;
        const int mx = jx < h ? jx : jx - ng, my = jy < h ? jy : jy - ng;
        if (in || my > 0 || (my == 0 && mx > 0)) {
          int a = 0, e = nbins;
          while (e - a > 1) {
            const int m = (a + e) >> 1;
            if (thr[m] <= n2) a = m; else e = m;
          }
          const double u = cb[a] * (wxy * win[nz]) * (nz == h ? 2.0 : 1.0);
          const float2 x = in ? X[(long)r * cols + nz] : X[((long)jx * ng + jy) * cols];
          z = make_float2((float)(u * x.x), (float)((in ? u : -u) * x.y));
        }
      }
      Z[(long)r * cols + nz] = z;
    }
  }
}

void launch_pk_adj_modes(const float2* X, float2* Z, int ng, double box, const double* edges,
                         int nbins, const double* cbar, const double* sums, hipStream_t s) {
  const double pi = 3.14159265358979323846;
  const double kf = 2.0 * pi / box, kmax = pi * ng / box;
  const double v = box * box * box, n3 = (double)ng * ng * ng;
  const double vol_fac = (v / n3) * (v / n3) / v;
  const int rows = ng * ng;
  const unsigned blocks = (unsigned)(rows / (8 * kRowWaves) < 4096 ? rows / (8 * kRowWaves) : 4096);
  const size_t lds = sizeof(double) * (ng / 2 + 1 + nbins) + sizeof(uint32_t) * (nbins + 1);
  hipLaunchKernelGGL(k_pk_adj_rows, dim3(blocks), dim3(64 * kRowWaves), lds, s, X, Z, ng, (int)padded_cols(ng), kf,
                     kmax, vol_fac, edges, nbins, cbar, sums);
}

void launch_pk_cross(const float2* sd, const float2* sp, int ng, double box, const double* edges, int nbins,
                     int axis, double* partial, int nchunk, double* out, hipStream_t s) {
  const double pi = 3.14159265358979323846;
  const double kf = 2.0 * pi / box;
  const double kmax = pi * ng / box;
  const double v = box * box * box;
  const double n3 = (double)ng * ng * ng;
  const double vol_fac = (v / n3) * (v / n3) / v;
  int nc = 0;
  if (pk_rows_plan(ng, nbins, 5, kPkPartialDoubles, &nc)) {
    hipLaunchKernelGGL(k_pk_rows<true>, dim3((unsigned)nc), dim3(64 * kRowWaves), pk_rows_lds(ng, nbins, 4), s, sd, sp,
                       ng, padded_cols(ng), kf, kmax, vol_fac, edges, nbins, axis, partial, nc, 1);
    hipLaunchKernelGGL(k_pk_rows_reduce<5>, dim3((unsigned)nbins), dim3(256), 0, s, partial, nc, out);
    return;
  }
  hipLaunchKernelGGL(k_pk_cross, dim3((unsigned)nchunk, (unsigned)nbins), dim3(kPT), 0, s, sd, sp, ng,
                     padded_cols(ng), kf, kmax, vol_fac, edges, nbins, axis, partial, nchunk);
  hipLaunchKernelGGL(k_pk_cross_reduce, dim3((unsigned)((nbins + 63) / 64)), dim3(64), 0, s, partial, nbins,
                     nchunk, out);
}

// Sums of |k|, P and the mode count per bin (out: 3 per bin).
void launch_pk_bin(const float2* spec, int ng, double box, const double* edges, int nbins,
                   double* partial, int nchunk, double* out, hipStream_t s, int deconvolve) {
  const double pi = 3.14159265358979323846;
  const double kf = 2.0 * pi / box;
  const double kmax = pi * ng / box;
  const double v = box * box * box;
  const double n3 = (double)ng * ng * ng;
  const double vol_fac = (v / n3) * (v / n3) / v;  // |(V/Ng^3) X|^2 / V
  int nc = 0;
  if (pk_rows_plan(ng, nbins, 3, kPkPartialDoubles, &nc)) {
    hipLaunchKernelGGL(k_pk_rows<false>, dim3((unsigned)nc), dim3(64 * kRowWaves), pk_rows_lds(ng, nbins, 2), s, spec,
                       nullptr, ng, padded_cols(ng), kf, kmax, vol_fac, edges, nbins, 0, partial, nc, deconvolve);
    hipLaunchKernelGGL(k_pk_rows_reduce<3>, dim3((unsigned)nbins), dim3(256), 0, s, partial, nc, out);
    return;
  }
  hipLaunchKernelGGL(k_pk_bin, dim3((unsigned)nchunk, (unsigned)nbins), dim3(kPT), 0, s, spec, ng,
                     padded_cols(ng), kf, kmax, vol_fac, edges, nbins, partial, nchunk, deconvolve);
  hipLaunchKernelGGL(k_pk_reduce, dim3((unsigned)((nbins + 63) / 64)), dim3(64), 0, s, partial, nbins,
                     nchunk, out);
}

// Smoothing + aliasing correction of Jing (2005) (Sec. 3.3): per bin b, the
// sum over its modes of the CIC window's image sum
//   C(k; s_b) = sum_{|m_e| <= kAliasImages} W^2(k + 2 k_N m) (|k + 2 k_N m| / |k|)^s_b,
// W the CIC window sinc^2 per axis continued to the images, s_b = slope[b].
// Per axis the image windows are sinc^4(x + pi m) = sin^4(x) / (x + pi m)^4
// with x = pi n / Ng (1 for m = 0 and 0 otherwise when n = 0).  The terms of
// a mode are summed in FP32 in a fixed order, the modes of a thread and the
// threads of a workgroup in FP64 as in k_pk_bin; partial holds one value per
// (bin, chunk).
constexpr int kAliasImages = 2;

__device__ __forceinline__ void image_windows(int n, int ng, float w[2 * kAliasImages + 1]) {
  if (n == 0) {
#pragma unroll
    for (int m = -kAliasImages; m <= kAliasImages; ++m) w[m + kAliasImages] = m == 0 ? 1.0f : 0.0f;
    return;
  }
  const double x = 3.14159265358979323846 * (double)n / (double)ng;
  const double s = sin(x);
  const double s4 = s * s * s * s;
#pragma unroll
  for (int m = -kAliasImages; m <= kAliasImages; ++m) {
    const double y = x + 3.14159265358979323846 * m;
    const double y2 = y * y;
    w[m + kAliasImages] = (float)(s4 / (y2 * y2));
  }
}

__global__ __launch_bounds__(kPT) void k_pk_alias(int ng, double kf, double kmax,
                                                  const double* __restrict__ edges, int nbins,
                                                  const double* __restrict__ slope,
                                                  double* __restrict__ partial, int nchunk) {
  __shared__ double sc[kPT];
  constexpr int kM = 2 * kAliasImages + 1;
  const int b = blockIdx.y;
  const int c = blockIdx.x;
  const double e0 = edges[b], e1 = edges[b + 1];
  const double lo2 = (e0 / kf) * (e0 / kf), hi2 = (e1 / kf) * (e1 / kf);
  const float hs = (float)(0.5 * slope[b]);
  const long nrows = (long)ng * ng;
  const long per = (nrows + nchunk - 1) / nchunk;
  const long r0 = (long)c * per, r1 = r0 + per < nrows ? r0 + per : nrows;
  double acc = 0.0;
  const int h = ng / 2;
  const float fng = (float)ng;
  for (long r = r0 + threadIdx.x; r < r1; r += kPT) {
    const int ix = (int)(r / ng), iy = (int)(r - (long)ix * ng);
    const int nx = ix < h ? ix : ix - ng, ny = iy < h ? iy : iy - ng;
    const double p2 = (double)nx * nx + (double)ny * ny;
    if (p2 >= hi2) continue;
    int zlo = 0;
    if (lo2 > p2) zlo = (int)floor(sqrt(lo2 - p2)) - 1;
    if (zlo < 0) zlo = 0;
    int zhi = (int)ceil(sqrt(hi2 - p2)) + 1;
    if (zhi > h) zhi = h;
    float wx[kM], wy[kM];
    image_windows(nx, ng, wx);
    image_windows(ny, ng, wy);
    for (int nz = zlo; nz <= zhi; ++nz) {
      if (nz == 0 && !(ny > 0 || (ny == 0 && nx > 0))) continue;
      const double n2 = p2 + (double)nz * nz;
      const double kk = kf * sqrt(n2);
      if (kk > kmax) continue;
      if (!(kk >= e0 && kk < e1)) continue;
      float wz[kM];
      image_windows(nz, ng, wz);
      const float l0 = log2f((float)n2);
      float sum = 0.0f;
#pragma unroll
      for (int mx = 0; mx < kM; ++mx) {
        if (wx[mx] == 0.0f) continue;
        const float kx = (float)nx + fng * (float)(mx - kAliasImages);
#pragma unroll
        for (int my = 0; my < kM; ++my) {
          if (wy[my] == 0.0f) continue;
          const float ky = (float)ny + fng * (float)(my - kAliasImages);
          const float wxy = wx[mx] * wy[my];
#pragma unroll
          for (int mz = 0; mz < kM; ++mz) {
            if (wz[mz] == 0.0f) continue;
            const float kz = (float)nz + fng * (float)(mz - kAliasImages);
            const float k2 = kx * kx + ky * ky + kz * kz;
            sum += wxy * wz[mz] * exp2f(hs * (log2f(k2) - l0));
          }
        }
      }
      acc += (double)sum;
    }
  }
  sc[threadIdx.x] = acc;
  __syncthreads();
  for (int o = kPT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) sc[threadIdx.x] += sc[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(long)b * nchunk + c] = sc[0];
}

__global__ void k_pk_alias_reduce(const double* __restrict__ partial, int nbins, int nchunk,
                                  double* __restrict__ out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  double s = 0.0;
  for (int c = 0; c < nchunk; ++c) s += partial[(long)b * nchunk + c];
  out[b] = s;
}

void launch_pk_alias(int ng, double box, const double* edges, int nbins, const double* slope, double* partial,
                     int nchunk, double* out, hipStream_t s) {
  const double pi = 3.14159265358979323846;
  const double kf = 2.0 * pi / box;
  const double kmax = pi * ng / box;
  hipLaunchKernelGGL(k_pk_alias, dim3((unsigned)nchunk, (unsigned)nbins), dim3(kPT), 0, s, ng, kf, kmax, edges,
                     nbins, slope, partial, nchunk);
  hipLaunchKernelGGL(k_pk_alias_reduce, dim3((unsigned)((nbins + 63) / 64)), dim3(64), 0, s, partial, nbins,
                     nchunk, out);
}

}  // namespace cola
