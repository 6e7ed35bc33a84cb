// Friends-of-friends groups (Koda et al. 2015: Sec. 2.3 runs a FoF halo finder
// on the fly; Sec. 3.1 links at 0.2 times the mean particle separation, 0.37
// for 2LPT).
//
// Two particles are friends when their nearest-image separation is at most b;
// the groups are the connected components, each labelled by its smallest
// particle id (unique, so the output is deterministic).  The link decision is
// made in float32 from the displacement in mesh units, one correctly rounded
// operation per step:
//   q = float(i nm) / float(np),  x = q + d,  dx = x_a - x_b,
//   dx -= nm rint(dx / nm),       r2 = (dx0^2 + dx1^2) + dx2^2 <= b^2.
//
// Search: particles are counted into cells of the mean separation s = nm/np
// (np^3 cells); b < s/2, so friends sit in the same or adjacent cells even
// where rounding moves a particle across a cell face.  A counting sort (count,
// exclusive scan, scatter) lays the positions out by cell, 16 bytes each
// (x, id), so a particle's candidates are a few contiguous ranges: the rest of
// its own cell and the next cell along z, and the 3 cells along z of the four
// other rows of the half shell.  Lanes of a wave mostly share them.
//
// Union-find over the cell order (parent[t] for the t-th particle by cell,
// next to the positions): parent[x] <= x always (a root is only ever
// hooked under a smaller root, by compare-and-swap), so every parent chain
// strictly decreases and each find ends.  Finds halve paths with plain
// coherent stores of a grandparent (a valid ancestor; a non-root never
// becomes a root again, and only roots are hooked, so no hook is undone).
// A failed compare-and-swap means another thread hooked that root first;
// the retry count is bounded and an exceeded bound raises a flag.  A friend
// whose parent is a node that the particle was joined with before is skipped:
// even a stale parent is an ancestor, so the two are connected already.  The last
// passes take every particle's root without halving (see fof_root) and the
// smallest id of each root's group.
//
// What bounds it: the pair tests of crowded cells (a particle's own cell holds
// 19 on average at a = 1), then the root chases of the joins.  256^3 particles
// at a = 1 (600 Mpc/h, 768 mesh): groups and catalogue 18.1 -> 5.4 ms; the link
// pass 15.3 ms when each candidate's id, position (three scattered loads and
// divisions) and root were looked up on their own, 4.3 in cell order, 3.8 with
// the face test, 2.9 + 0.5 with the first parents found beforehand.
#include "cola_device.h"
#include "cola_internal.h"

namespace cola {

namespace {

constexpr int kFofMaxRetry = 1 << 20;

__device__ __forceinline__ uint32_t ld_rel(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void fof_pos(const float* __restrict__ disp, long np3, uint32_t id, int np, int nm,
                                        float x[3]) {
#pragma clang fp contract(off)
  const LatGeom g = lat_geom(np, nm);
  const uint32_t q1 = lat_div(id, g);
  const uint32_t q0 = lat_div(q1, g);
  const uint32_t li[3] = {q0, q1 - q0 * g.np, id - q1 * g.np};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    // i nm / np rounded to float once: the double product is within 2^-52 of a
    // quotient that is a float or 2^-35 from every rounding boundary (LatDivTable)
    const float q = (float)((double)(2u * li[e] * g.nm) * g.inv2);
    x[e] = __fadd_rn(q, disp[e * np3 + id]);
  }
}

__device__ __forceinline__ int fof_cell1(float x, float s_inv, int np) {
  int c = (int)floorf(x * s_inv);
  if ((uint32_t)c >= (uint32_t)np) {
    c %= np;
    if (c < 0) c += np;
  }
  return c;
}

// Cell coordinates up to this keep their rounding below kFofMargin cells.
constexpr float kFofFar = 4096.0f, kFofMargin = 1e-3f;

// Root without writes: the final pass must not halve paths, or a thread that
// read par[x] before another wrote x's root there could overwrite that root
// with an intermediate ancestor.
__device__ __forceinline__ uint32_t fof_root(const uint32_t* par, uint32_t x) {
  for (;;) {
    const uint32_t p = ld_rel(par + x);
    if (p == x) return x;
    x = p;
  }
}

__device__ __forceinline__ uint32_t fof_find(uint32_t* par, uint32_t x) {
  for (;;) {
    const uint32_t p = ld_rel(par + x);
    if (p == x) return x;
    const uint32_t gp = ld_rel(par + p);
    if (gp != p) st_rel(par + x, gp);
    x = gp;
  }
}

}  // namespace

__global__ __launch_bounds__(256) void k_fof_cell(const float* __restrict__ disp, int np, int nm, long np3,
                                                  float s_inv, uint32_t* __restrict__ count,
                                                  uint32_t* __restrict__ key, uint32_t* __restrict__ rank,
                                                  uint32_t* __restrict__ far) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i >= np3) return;
  float x[3];
  fof_pos(disp, np3, (uint32_t)i, np, nm, x);
  const uint32_t c = ((uint32_t)fof_cell1(x[0], s_inv, np) * (uint32_t)np + (uint32_t)fof_cell1(x[1], s_inv, np)) *
                         (uint32_t)np +
                     (uint32_t)fof_cell1(x[2], s_inv, np);
  if (fmaxf(fabsf(x[0]), fmaxf(fabsf(x[1]), fabsf(x[2]))) * s_inv > kFofFar) *far = 1u;
  key[i] = c;
  rank[i] = atomicAdd(&count[c], 1u);
}

// Cell order: (x, id) of the t-th particle.
__global__ __launch_bounds__(256) void k_fof_scatter(const float* __restrict__ disp, int np, int nm, long np3,
                                                     const uint32_t* __restrict__ key,
                                                     const uint32_t* __restrict__ rank,
                                                     const uint32_t* __restrict__ start,
                                                     float4* __restrict__ pos) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i >= np3) return;
  float x[3];
  fof_pos(disp, np3, (uint32_t)i, np, nm, x);
  const uint32_t t = start[key[i]] + rank[i];
  pos[t] = make_float4(x[0], x[1], x[2], __uint_as_float((uint32_t)i));
}

// Squared nearest-image separation in the written order.  Below 0.49 nm the
// quotient rounds to 0 and the image term is exactly 0: no division.
__device__ __forceinline__ float fof_sep2(const float xi[3], const float4& p, float nmf) {
#pragma clang fp contract(off)
  float d[3] = {__fsub_rn(xi[0], p.x), __fsub_rn(xi[1], p.y), __fsub_rn(xi[2], p.z)};
  const float m = fmaxf(fabsf(d[0]), fmaxf(fabsf(d[1]), fabsf(d[2])));
  if (m >= 0.49f * nmf) {
#pragma unroll
    for (int e = 0; e < 3; ++e) d[e] = __fsub_rn(d[e], __fmul_rn(nmf, rintf(__fdiv_rn(d[e], nmf))));
  }
  return __fadd_rn(__fadd_rn(__fmul_rn(d[0], d[0]), __fmul_rn(d[1], d[1])), __fmul_rn(d[2], d[2]));
}

// Joins t and s; returns the root of both (the smaller of the two roots).
__device__ uint32_t fof_union(uint32_t* par, uint32_t t, uint32_t s, uint32_t* flag) {
  int tries = 0;
  for (;;) {
    const uint32_t ri = fof_find(par, t), rj = fof_find(par, s);
    if (ri == rj) return ri;
    const uint32_t hi = ri > rj ? ri : rj, lo = ri > rj ? rj : ri;
    if (atomicCAS(par + hi, hi, lo) == hi) return lo;
    if (++tries >= kFofMaxRetry) {
      atomicOr(flag, 1u);
      return lo;
    }
  }
}

// First parents without any atomics: the earliest friend before t among the
// particles of its own cell and of the cell before it along z.  The trees are
// then flattened, so that the link pass finds most friends under one root.
__global__ __launch_bounds__(256) void k_fof_hook(const float4* __restrict__ pos, int np, int nm, long np3, float s_inv,
                                                  float b2, float reach, const uint32_t* __restrict__ start,
                                                  uint32_t* __restrict__ par) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= np3) return;
  const float4 pi = pos[t];
  const float xi[3] = {pi.x, pi.y, pi.z};
  const int c0 = fof_cell1(xi[0], s_inv, np), c1 = fof_cell1(xi[1], s_inv, np), c2 = fof_cell1(xi[2], s_inv, np);
  const float nmf = (float)nm, uz = xi[2] * s_inv;
  const uint32_t own = ((uint32_t)c0 * np + c1) * (uint32_t)np + c2;
  uint32_t p = (uint32_t)t;
  constexpr int kU = 4;
  for (uint32_t s = start[own - (c2 > 0 && uz - floorf(uz) < reach ? 1 : 0)]; s < (uint32_t)t && p == (uint32_t)t; s += kU) {
    float4 pj[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) pj[u] = pos[min(s + u, (uint32_t)t)];
#pragma unroll
    for (int u = kU - 1; u >= 0; --u)
      if (s + u < (uint32_t)t && fof_sep2(xi, pj[u], nmf) <= b2) p = s + u;
  }
  par[t] = p;
}

__global__ __launch_bounds__(256) void k_fof_flatten(uint32_t* par, long np3) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= np3) return;
  const uint32_t p = ld_rel(par + t);
  if (p != (uint32_t)t) st_rel(par + t, fof_root(par, p));
}

__global__ __launch_bounds__(256) void k_fof_link(const float4* __restrict__ pos, int np, int nm, long np3, float s_inv,
                                                  float b2, float reach, const uint32_t* __restrict__ start,
                                                  uint32_t* par, uint32_t* __restrict__ minid, uint32_t* flag,
                                                  const uint32_t* __restrict__ far) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= np3) return;
  minid[t] = 0xffffffffu;
  const float4 pi = pos[t];
  const float xi[3] = {pi.x, pi.y, pi.z};
  const int c0 = fof_cell1(xi[0], s_inv, np), c1 = fof_cell1(xi[1], s_inv, np), c2 = fof_cell1(xi[2], s_inv, np);
  const float nmf = (float)nm;
  // nodes known to be in t's group, the latest root first
  uint32_t k0 = ld_rel(par + t), k1 = k0, k2 = k0, k3 = k0;
  constexpr int kU = 4;                       // candidates in flight
  auto range = [&](uint32_t s0, uint32_t s1) {
    for (uint32_t s = s0; s < s1; s += kU) {
      float4 pj[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) pj[u] = pos[min(s + u, s1 - 1)];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        if (s + u < s1 && fof_sep2(xi, pj[u], nmf) <= b2) {
          const uint32_t p = __hip_atomic_load(par + s + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (p != k0 && p != k1 && p != k2 && p != k3) {
            const uint32_t r = fof_union(par, (uint32_t)t, s + u, flag);
            k3 = k2;
            k2 = k1;
            k1 = r == k0 ? k1 : k0;
            k0 = r;
            if (p != r) {
              k3 = k2;
              k2 = p;
            }
          }
        }
      }
    }
  };
  // the faces within reach (b in cells, widened by the rounding of the cell
  // coordinates; every face where a coordinate is too large for that bound)
  bool lo[3], hi[3];
  const bool all = *far != 0u;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const float u = xi[e] * s_inv, f = u - floorf(u);
    lo[e] = all || f < reach + kFofMargin;
    hi[e] = all || f > 1.0f - reach - kFofMargin;
  }
  // half shell: the particles after t in the own cell, and the 13 cells that
  // follow (0, 0, 0) in lexicographic order; every unordered pair of adjacent
  // cells is then visited from exactly one side (np >= 3)
  const uint32_t own = ((uint32_t)c0 * np + c1) * (uint32_t)np;
  const bool wrap = hi[2] && c2 + 1 == np;
  range((uint32_t)t + 1, start[own + (hi[2] && !wrap ? c2 + 2 : c2 + 1)]);
  if (wrap) range(start[own], start[own + 1]);
  for (int r = 0; r < 4; ++r) {               // rows (0, 1), (1, -1), (1, 0), (1, 1)
    if (!(r == 0 ? hi[1] : hi[0] && (r == 2 || (r == 1 ? lo[1] : hi[1])))) continue;
    const int a0 = r == 0 ? c0 : (c0 + 1 == np ? 0 : c0 + 1);
    int a1 = c1 + (r == 0 ? 1 : r - 2);
    a1 = a1 < 0 ? np - 1 : a1 == np ? 0 : a1;
    const uint32_t row = ((uint32_t)a0 * np + a1) * (uint32_t)np;
    const int zl = lo[2] && c2 > 0 ? c2 - 1 : c2, zh = hi[2] && !wrap ? c2 + 1 : c2;
    range(start[row + zl], start[row + zh + 1]);
    if (lo[2] && c2 == 0) range(start[row + np - 1], start[row + np]);
    if (wrap) range(start[row], start[row + 1]);
  }
}

// Root of every particle, and the smallest id below each root.
__global__ __launch_bounds__(256) void k_fof_compress(const float4* __restrict__ pos, uint32_t* par, uint32_t* minid,
                                                      long np3) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t >= np3) return;
  const uint32_t r = fof_root(par, (uint32_t)t);   // each thread writes only its own entry
  st_rel(par + t, r);
  const uint32_t id = __float_as_uint(pos[t].w);
  // most members of a large group find a smaller id there already
  if (id < ld_rel(minid + r)) atomicMin(minid + r, id);
}

__global__ __launch_bounds__(256) void k_fof_labels(const float4* __restrict__ pos, const uint32_t* __restrict__ par,
                                                    const uint32_t* __restrict__ minid, long np3,
                                                    uint32_t* __restrict__ labels) {
  const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (t < np3) labels[__float_as_uint(pos[t].w)] = minid[par[t]];
}

void launch_fof(const float* disp, int np, int nm, double b_frac, uint32_t* labels, uint32_t* count,
                uint32_t* start, uint32_t* scan_scratch, uint32_t* key, uint32_t* rank, uint32_t* par, void* pos,
                uint32_t* flag, hipStream_t s) {
  const long np3 = (long)np * np * np;
  const unsigned blocks = (unsigned)((np3 + 255) / 256);
  const double b = b_frac * nm / np;
  const float b2 = (float)(b * b);
  const float s_inv = (float)((double)np / (double)nm);
  float4* p4 = static_cast<float4*>(pos);
  uint32_t* far = flag + 1;
  launch_fill_u32(flag, 2, 0u, s);
  launch_fill_u32(count, np3 + 1, 0u, s);
  hipLaunchKernelGGL(k_fof_cell, dim3(blocks), dim3(256), 0, s, disp, np, nm, np3, s_inv, count, key, rank, far);
  launch_exclusive_scan(count, start, np3, scan_scratch, 0, s);
  hipLaunchKernelGGL(k_fof_scatter, dim3(blocks), dim3(256), 0, s, disp, np, nm, np3, key, rank, start, p4);
  hipLaunchKernelGGL(k_fof_hook, dim3(blocks), dim3(256), 0, s, p4, np, nm, np3, s_inv, b2, (float)b_frac, start, par);
  hipLaunchKernelGGL(k_fof_flatten, dim3(blocks), dim3(256), 0, s, par, np3);
  // the ranks' array then holds the smallest ids
  hipLaunchKernelGGL(k_fof_link, dim3(blocks), dim3(256), 0, s, p4, np, nm, np3, s_inv, b2,
                     (float)b_frac, start, par, rank, flag, far);
  hipLaunchKernelGGL(k_fof_compress, dim3(blocks), dim3(256), 0, s, p4, par, rank, np3);
  hipLaunchKernelGGL(k_fof_labels, dim3(blocks), dim3(256), 0, s, p4, par, rank, np3, labels);
}

// ---------------------------------------------------------------------------
// Halo catalogue of the groups with at least min_members particles, in
// increasing root id: member count, centre of mass (the root's position plus
// the mean nearest-image offset of the members from it, wrapped into
// [0, nm)) and mean velocity.  Offsets and velocities are summed as 64-bit
// fixed point (2^-20 cells, 2^-16 velocity units): integer sums do not
// depend on the order of the atomics, so the catalogue is reproducible.

constexpr double kPosFix = 1048576.0, kVelFix = 65536.0;

// Particle of thread t of a workgroup: 4 x 4 x 16 lattice blocks, a wave on
// 4 x 4 x 4 ids (every supported np is a multiple of 16).  A halo's members are
// compact on the lattice, so a wave meets few halos and adds once for each.
__device__ __forceinline__ long halo_particle(uint32_t b, int t, int np) {
  const uint32_t nbk = (uint32_t)np >> 4, nbj = (uint32_t)np >> 2;
  const uint32_t bk = b % nbk, bj = (b / nbk) % nbj, bi = b / (nbk * nbj);
  const int k = (int)bk * 16 + (t >> 6) * 4 + (t & 3), j = (int)bj * 4 + ((t >> 2) & 3), i = (int)bi * 4 + ((t >> 4) & 3);
  return ((long)i * np + j) * np + k;
}

__global__ __launch_bounds__(256) void k_halo_count(const int32_t* __restrict__ lab, int np, long np3,
                                                    uint32_t* __restrict__ count, uint32_t* bad) {
  const long i = halo_particle(blockIdx.x, threadIdx.x, np);
  const int32_t l = lab[i];
  const bool in = l >= 0 && (long)l < np3;
  if (!in) atomicOr(bad, 1u);   // not a label of this particle set
  // a root (label = id) counts itself alone, the other lanes of one label together
  if (in && (long)l == i) atomicAdd(&count[l], 1u);
  const bool more = in && (long)l != i;
  uint64_t left = __ballot(more);
  while (left) {
    const int32_t l0 = __shfl(l, (int)__builtin_ctzll(left), 64);
    const uint64_t same = __ballot(more && l == l0);
    if ((int)(threadIdx.x & 63) == (int)__builtin_ctzll(same)) atomicAdd(&count[l0], (uint32_t)__popcll(same));
    left &= ~same;
  }
}

__global__ __launch_bounds__(256) void k_halo_flag(const uint32_t* __restrict__ count, long np3, uint32_t minm,
                                                   uint32_t* __restrict__ flg) {
  const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (i < np3) flg[i] = count[i] >= minm ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_halo_roots(const uint32_t* __restrict__ count,
                                                    const uint32_t* __restrict__ flg,
                                                    const uint32_t* __restrict__ hidx, long np3,
                                                    int32_t* __restrict__ root, int32_t* __restrict__ cnt) {
  const long r = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (r < np3 && flg[r]) {
    root[hidx[r]] = (int32_t)r;
    cnt[hidx[r]] = (int32_t)count[r];
  }
}

__global__ __launch_bounds__(256) void k_halo_accum(const float* __restrict__ disp, const float* __restrict__ vel,
                                                    const int32_t* __restrict__ lab,
                                                    const uint32_t* __restrict__ flg,
                                                    const uint32_t* __restrict__ hidx, int np, int nm, long np3,
                                                    unsigned long long* __restrict__ acc) {
#pragma clang fp contract(off)
  const long i = halo_particle(blockIdx.x, threadIdx.x, np);
  const int32_t l = lab[i];
  const bool in = l >= 0 && (long)l < np3 && flg[l];
  uint64_t left = __ballot(in);
  if (!left) return;
  const int h = in ? (int)hidx[l] : -1;
  long long q[6] = {0, 0, 0, 0, 0, 0};
  if (in) {
    float xi[3], xr[3];
    fof_pos(disp, np3, (uint32_t)i, np, nm, xi);
    fof_pos(disp, np3, (uint32_t)l, np, nm, xr);
    const float nmf = (float)nm;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      float dx = __fsub_rn(xi[e], xr[e]);
      dx = __fsub_rn(dx, __fmul_rn(nmf, rintf(__fdiv_rn(dx, nmf))));
      q[e] = llrint((double)dx * kPosFix);
      if (vel) q[3 + e] = llrint((double)vel[e * np3 + i] * kVelFix);
    }
  }
  // one addition per halo, wave and sum (integers: any order gives the same)
  const int lane = threadIdx.x & 63;
  const int nq = vel ? 6 : 3;
  while (left) {
    const int h0 = __shfl(h, (int)__builtin_ctzll(left), 64);
    const bool mine = h == h0;
    long long s[6];
#pragma unroll
    for (int e = 0; e < 6; ++e) s[e] = mine ? q[e] : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int e = 0; e < 6; ++e) s[e] += __shfl_xor(s[e], o, 64);
    long long v = s[0];
#pragma unroll
    for (int e = 1; e < 6; ++e) v = lane == e ? s[e] : v;
    if (lane < nq) atomicAdd(acc + (long)h0 * 6 + lane, (unsigned long long)v);
    left &= ~__ballot(mine);
  }
}

__global__ __launch_bounds__(256) void k_halo_final(const float* __restrict__ disp,
                                                    const int32_t* __restrict__ root,
                                                    const int32_t* __restrict__ cnt,
                                                    const unsigned long long* __restrict__ acc, int np, int nm,
                                                    long np3, int nh, int stride, float* __restrict__ pos,
                                                    float* __restrict__ vout) {
  const int h = blockIdx.x * blockDim.x + threadIdx.x;
  if (h >= nh) return;
  float xr[3];
  fof_pos(disp, np3, (uint32_t)root[h], np, nm, xr);
  const double n = (double)cnt[h];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    double c = (double)xr[e] + (double)(long long)acc[(long)h * 6 + e] / kPosFix / n;
    c -= nm * floor(c / nm);
    float fc = (float)c;                 // rounding can reach nm itself
    if (fc >= (float)nm) fc -= (float)nm;
    pos[(long)e * stride + h] = fc;
    if (vout) vout[(long)e * stride + h] = (float)((double)(long long)acc[(long)h * 6 + 3 + e] / kVelFix / n);
  }
}

void launch_halo_count(const int32_t* lab, int np, int32_t minm, uint32_t* count, uint32_t* flg, uint32_t* hidx,
                       uint32_t* scan_scratch, uint32_t* bad, hipStream_t s) {
  const long np3 = (long)np * np * np;
  const unsigned blocks = (unsigned)((np3 + 255) / 256);
  launch_fill_u32(count, np3, 0u, s);
  hipLaunchKernelGGL(k_halo_count, dim3(blocks), dim3(256), 0, s, lab, np, np3, count, bad);
  hipLaunchKernelGGL(k_halo_flag, dim3(blocks), dim3(256), 0, s, count, np3, (uint32_t)minm, flg);
  launch_exclusive_scan(flg, hidx, np3, scan_scratch, 0, s);
}

void launch_halo_fill(const float* disp, const float* vel, const int32_t* lab, const uint32_t* count,
                      const uint32_t* flg, const uint32_t* hidx, int np, int nm, int nh, int stride,
                      unsigned long long* acc, int32_t* root, int32_t* cnt, float* pos, float* vout,
                      hipStream_t s) {
  const long np3 = (long)np * np * np;
  const unsigned blocks = (unsigned)((np3 + 255) / 256);
  if (nh > 0) launch_fill_u32(reinterpret_cast<uint32_t*>(acc), 12L * nh, 0u, s);
  hipLaunchKernelGGL(k_halo_roots, dim3(blocks), dim3(256), 0, s, count, flg, hidx, np3, root, cnt);
  hipLaunchKernelGGL(k_halo_accum, dim3(blocks), dim3(256), 0, s, disp, vel, lab, flg, hidx, np, nm, np3, acc);
  if (nh > 0)
    hipLaunchKernelGGL(k_halo_final, dim3((unsigned)((nh + 255) / 256)), dim3(256), 0, s, disp, root, cnt, acc,
                       np, nm, np3, nh, stride, pos, vout);
}

}  // namespace cola
