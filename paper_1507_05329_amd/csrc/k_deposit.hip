// Deterministic CIC mass assignment as a gather (no float atomics).
//
// CIC (Koda et al. 2015, Sec. 3.3; Hockney & Eastwood): a particle with home
// cell c and fraction f gives weight prod_e w_{s_e}(f_e) to node c + s.
// One workgroup owns a 16^3 tile of nodes.  The cells that feed those nodes
// are the tile's 16^3 cells plus the one-cell layer below it on each axis
// (a 17^3 region); their particles come from the tile's buckets and from the
// face/edge/corner buckets of the 7 lower neighbour tiles.
//
// Mass (k_deposit_mass): every weight is taken to 64-bit fixed point,
// q = rint(w 2^32), and the tile's nodes add them with integer LDS atomics;
// the integer sum is exact, so the node mass float32(sum) 2^-32 does not
// depend on the order of the particles, the buckets or the workgroups.  The
// particles are streamed, never held, so a region of any size takes one pass.
// What is read are the tile sort's records (fractions and cell in the tile, 16
// bytes in bucket order), not ids and through them displacements.
//
// Weighted deposits (k_deposit_weighted: the transpose of the force readout;
// weights of either sign and any size): the same in 64-bit signed fixed point,
// whose unit follows from the largest weight of the component (k_weight_max)
// and the number of particles in the region, so a node's sum is exact but for
// the rounding of each product to at least 2^-50 of that weight (2^-43 where a
// region holds 2^19 particles), and again does not depend on any order.  A node
// that only weights 2^-27 of the largest or less reach holds fewer bits than a
// float; every user transforms the mesh in float32 next, whose rounding, some
// 2^-24 of a mode that holds the largest weight, lies above what is left out
// there.
#include "cola_device.h"
#include "cola_internal.h"

// Every float operation in this file is a single IEEE rounding (the order is
// part of the result): no fused multiply-add but the one that is written, which
// rounds an exact product to a whole number of units.
#pragma clang fp contract(off)

namespace cola {

constexpr int kTile = 16;                 // nodes per tile side

// Mass deposit.  Node masses in units of 2^-32 particle masses, on 17^3 nodes:
// the layer past each upper face takes what belongs to the next tile (that
// tile adds the same particles itself), so the tile's own particles need no
// test.  39.5 KB: four workgroups per compute unit.
constexpr int kAcc = kTile + 1;
struct NodeSums {
  unsigned long long acc[kAcc * kAcc * kAcc + 1];   // whole 16 bytes
  __device__ __forceinline__ void clear(int threads) {
    for (int i = threadIdx.x; i < kAcc * kAcc * kAcc / 2 + 1; i += threads)
      reinterpret_cast<ulonglong2*>(acc)[i] = make_ulonglong2(0ull, 0ull);
  }
};

// The region's boundary: bucket ranges [c0, c1) of lower neighbour (tx, ty, tz)
// - (dx, dy, dz), nb = 4 dx + 2 dy + dz: the face classes that contain nb.
// One hexadecimal digit per segment, the first one lowest.
constexpr int kBnd = 13;
constexpr uint64_t kBndNb = 0x7655433221111ull, kBndC0 = 0x7675473627531ull, kBndC1 = 0x8886884848642ull;
__device__ __forceinline__ int bnd(uint64_t table, int q) { return (int)(table >> (4 * q)) & 15; }

// The segments in lanes 0 .. kBnd - 1 of every wave, so that a thread's first
// boundary particle can be requested before any barrier.
struct Boundary {
  uint32_t first, pre, total;   // first entry minus the entries before it; entries before it; all of them
  __device__ __forceinline__ Boundary(const uint32_t* __restrict__ off, int tx, int ty, int tz, int nt) {
    const int lane = threadIdx.x & 63;
    uint32_t st = 0, len = 0;
    if (lane < kBnd) {
      const int nb = bnd(kBndNb, lane);
      int ux = tx - (nb >> 2), uy = ty - ((nb >> 1) & 1), uz = tz - (nb & 1);
      if (ux < 0) ux += nt;
      if (uy < 0) uy += nt;
      if (uz < 0) uz += nt;
      const uint32_t* o = off + (((uint32_t)ux * nt + uy) * nt + uz) * 8u;
      st = o[bnd(kBndC0, lane)];
      len = o[bnd(kBndC1, lane)] - st;
    }
    pre = len;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const uint32_t v = __shfl_up(pre, o, 64);
      if (lane >= o) pre += v;
    }
    pre -= len;
    first = st - pre;
    total = __shfl(pre, kBnd, 64);
  }
  // Place of boundary entry x < total in the sorted order, and its neighbour.
  // Every lane of the wave takes part.
  __device__ __forceinline__ uint32_t place(uint32_t x, int& nb) const {
    int q = 0;                                     // last segment with pre <= x
#pragma unroll
    for (int step = 8; step > 0; step >>= 1) {
      const uint32_t p = __shfl(pre, (q + step) & 15, 64);
      if (q + step < kBnd && p <= x) q += step;
    }
    nb = bnd(kBndNb, q);
    return __shfl(first, q, 64) + x;
  }
};

// rint(w 2^32), ties to even, for a weight w in [0, 1] (0 for NaN): below 1 it
// fits 32 bits.
__device__ __forceinline__ unsigned long long fix32(float w) {
  const bool one = w >= 1.0f;
  const uint32_t q = (uint32_t)__builtin_rintf(__fmul_rn(w, 4294967296.0f));   // saturates, 0 for NaN
  return one ? 1ull << 32 : (unsigned long long)q;
}

// Adds a particle's weights to the nodes of offsets k with (k & nb) == nb
// (nb = 0: all 8) of the cell whose offset-0 node is base.
__device__ __forceinline__ void add_mass(NodeSums& sh, const float f[3], int base, int nb) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if ((k & nb) == nb)
      atomicAdd(&sh.acc[base + ((k >> 2) & 1) * kAcc * kAcc + ((k >> 1) & 1) * kAcc + (k & 1)],
                fix32(cic_weight(f, k)));
}

constexpr float kFixInv = 2.3283064365386963e-10f;   // 2^-32
template <int T, int G>
__global__ __launch_bounds__(T) void k_deposit_mass(const float2* __restrict__ fxy, const float2* __restrict__ fzc,
                                                    const uint32_t* __restrict__ off, int nm,
                                                    float* __restrict__ out, long row_stride, int contrast,
                                                    float cinv, long mstride) {
  __shared__ __align__(16) NodeSums sh;
  fxy = mock_ptr(fxy, mstride);
  fzc = mock_ptr(fzc, mstride);
  off = mock_ptr(off, mstride);
  out = mock_ptr(out, mstride);
  const int nt = nm / kTile;
  const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
  const int tx = t / (nt * nt), ty = (t / nt) % nt, tz = t % nt;
  // the tile's own particles: one contiguous range, its first records requested at once
  const uint32_t s0 = off[t * 8u], s1 = off[t * 8u + 8u];
  float2 a[G], b[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint32_t x = s0 + g * T + threadIdx.x;
    if (x < s1) {
      a[g] = fxy[x];
      b[g] = fzc[x];
    }
  }
  const Boundary bd(off, tx, ty, tz, nt);
  const uint32_t total = bd.total;
  int nb = 0;
  float2 ba = make_float2(0.f, 0.f), bb = ba;
  if (total > 0) {
    const uint32_t p = bd.place(min(threadIdx.x, total - 1), nb);
    if (threadIdx.x < total) {
      ba = fxy[p];
      bb = fzc[p];
    }
  }
  sh.clear(T);
  __syncthreads();

  for (uint32_t x0 = s0; x0 < s1; x0 += G * T) {
    if (x0 > s0) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint32_t x = x0 + g * T + threadIdx.x;
        if (x < s1) {
          a[g] = fxy[x];
          b[g] = fzc[x];
        }
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (x0 + g * T + threadIdx.x < s1) {
        const float f[3] = {a[g].x, a[g].y, b[g].x};
        const uint32_t c = __float_as_uint(b[g].y);
        add_mass(sh, f, (int)((((c >> 8) & 15) * kAcc + ((c >> 4) & 15)) * kAcc + (c & 15)), 0);
      }
    }
  }
  for (uint32_t x0 = 0; x0 < total; x0 += T) {     // every lane of a wave takes part in the search
    const uint32_t x = x0 + threadIdx.x;
    if (x0 > 0) {
      const uint32_t p = bd.place(min(x, total - 1), nb);
      if (x < total) {
        ba = fxy[p];
        bb = fzc[p];
      }
    }
    if (x < total) {
      const float f[3] = {ba.x, ba.y, bb.x};
      const uint32_t c = __float_as_uint(bb.y);
      const int lx = nb & 4 ? -1 : (int)((c >> 8) & 15), ly = nb & 2 ? -1 : (int)((c >> 4) & 15),
                lz = nb & 1 ? -1 : (int)(c & 15);
      add_mass(sh, f, (lx * kAcc + ly) * kAcc + lz, nb);
    }
  }
  __syncthreads();

  // four consecutive z nodes per thread and store (rows of the padded
  // layout and tile origins are 16-byte aligned)
  for (int qd = threadIdx.x; qd < kTile * kTile * kTile / 4; qd += T) {
    const int nx = qd >> 6, ny = (qd >> 2) & 15, nz = (qd & 3) * 4;
    const long o = ((long)(tx * kTile + nx) * nm + (ty * kTile + ny)) * row_stride + (tz * kTile + nz);
    unsigned long long q[4];
    float r[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = sh.acc[(nx * kAcc + ny) * kAcc + nz + j];
    // float32(sum): sums below one particle mass (most nodes of a sparse mesh) by one conversion
    if (__any((uint32_t)((q[0] | q[1] | q[2] | q[3]) >> 32))) {
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = __ull2float_rn(q[j]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = __uint2float_rn((uint32_t)q[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      r[j] = __fmul_rn(r[j], kFixInv);
      if (contrast) r[j] = __fsub_rn(__fmul_rn(r[j], cinv), 1.0f);
    }
    *reinterpret_cast<float4*>(out + o) = make_float4(r[0], r[1], r[2], r[3]);
  }
}

// One workgroup per tile; the result does not depend on the shape.  What
// bounds it is a workgroup's chain of requests (bucket starts, records, the
// density's store) with four workgroups per compute unit; sort and deposit
// together, before (ids, then displacements through them) and now: 256^3 / 768^3
// 1.32 -> 0.97 ms, 512^3 / 1024^3 5.25 -> 3.76 ms, 128^3 / 256^3 0.110 -> 0.081 ms.
// Two tiles along z per workgroup, for stores of whole 128-byte lines, took
// 0.74 against 0.76 ms and 2.17 against 2.17 ms (35 against 32 us at 256): not kept;
// nor were conflict-free reads of the sums (0.78 ms) and nontemporal stores (0.89 ms).
// Without its store the kernel takes 0.45 ms (768), without the additions 0.72.
// 1024 threads where a tile holds more than 1024 particles on average: with 256
// threads its records come in many rounds (64^3 / 64^3: 44 us with the ids).
void launch_deposit(const float2* fxy, const float2* fzc, const uint32_t* off, int np, int nm, float* out,
                    long row_stride, int contrast, hipStream_t s, int nmock, long mstride) {
  const long np3 = (long)np * np * np;
  const int nt = nm / kTile;
  const long ntiles = (long)nt * nt * nt;
  const float cinv = (float)((double)nm * nm * nm / (double)np3);
  const dim3 grid((unsigned)ntiles, 1, (unsigned)nmock);
  if (np3 > 1024 * ntiles)
    hipLaunchKernelGGL((k_deposit_mass<1024, 2>), grid, dim3(1024), 0, s, fxy, fzc, off, nm, out, row_stride, contrast,
                       cinv, mstride);
  else
    hipLaunchKernelGGL((k_deposit_mass<256, 2>), grid, dim3(256), 0, s, fxy, fzc, off, nm, out, row_stride, contrast,
                       cinv, mstride);
}

// Weighted deposit of NC components, one after the other in the same node
// sums: particles by id, their cells found again from the displacements; the
// first G particles of a thread and its first boundary particle are fetched
// once, before any barrier, and kept for all components.  What bounds it is the
// clearing and writing of the node sums (three times the mass deposit's); three
// components on 256^3 / 768^3: 2.8 ms, 128^3 / 256^3 0.12 ms, where an ordered float
// sum over particles sorted in LDS took 4.2 and 0.25 ms, and one component per
// workgroup 3.1 ms.  maxw: the bits of the
// largest |weight| per component; where that is not finite the sums are plain
// doubles, so that the nodes out of its reach still get their values.
template <int NC, int T, int G>
__global__ __launch_bounds__(T) void k_deposit_weighted(const float* __restrict__ disp,
                                                        const uint32_t* __restrict__ perm,
                                                        const uint32_t* __restrict__ off, int np, int nm, long np3,
                                                        const float* __restrict__ wt,
                                                        const uint32_t* __restrict__ maxw, float* __restrict__ out,
                                                        long row_stride, long mesh_stride) {
  __shared__ __align__(16) NodeSums sh;
  __shared__ uint32_t bad;                // a position that is not a number
  struct Part {
    float f[3], w[NC];
    int base, nb;
  };
  const int nt = nm / kTile;
  const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
  const int tx = t / (nt * nt), ty = (t / nt) % nt, tz = t % nt;
  const uint32_t s0 = off[t * 8u], s1 = off[t * 8u + 8u];
  const Boundary bd(off, tx, ty, tz, nt);
  const uint32_t total = bd.total;
  auto fetch = [&](Part& p, uint32_t place, int nb, int c0, int c1) {
    const uint32_t id = min(perm[place], (uint32_t)np3 - 1u);
    const float dv[3] = {disp[id], disp[np3 + id], disp[2 * np3 + id]};
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (q >= c0 && q < c1) p.w[q] = wt[q * np3 + id];
    int c[3];
    home_cell_of(dv, id, np, nm, 1.0f, c, p.f);
    const int lx = nb & 4 ? -1 : c[0] & 15, ly = nb & 2 ? -1 : c[1] & 15, lz = nb & 1 ? -1 : c[2] & 15;
    p.base = (lx * kAcc + ly) * kAcc + lz;
    p.nb = nb;
  };
  Part own[G], edge;
  int nb = 0;
#pragma unroll
  for (int g = 0; g < G; ++g)
    if (s0 + g * T + threadIdx.x < s1) fetch(own[g], s0 + g * T + threadIdx.x, 0, 0, NC);
  if (total > 0) {
    const uint32_t p = bd.place(min(threadIdx.x, total - 1), nb);
    if (threadIdx.x < total) fetch(edge, p, nb, 0, NC);
  }
  // n < 2^l particles: products of at most 2^b units, b + l <= 62
  const int l = 32 - __clz((int)(s1 - s0 + total)), b = l < 12 ? 50 : 62 - l;

#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const uint32_t mx = maxw[q];
    const bool fixed = mx < 0x7f800000u;
    const int e = (int)(mx >> 23) - 126;                            // |weight| < 2^e
    const double unit = ldexp(1.0, b - e), inv = ldexp(1.0, e - b);
    auto add = [&](const Part& p) {
      if (!(p.f[0] + p.f[1] + p.f[2] < 4.0f)) bad = 1u;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if ((k & p.nb) == p.nb) {
          unsigned long long* node = &sh.acc[p.base + ((k >> 2) & 1) * kAcc * kAcc + ((k >> 1) & 1) * kAcc + (k & 1)];
          const double v = (double)p.w[q] * (double)cic_weight(p.f, k);   // exact
          if (fixed) {
            const double m = 6755399441055744.0;                    // 1.5 x 2^52: the integer in the low bits
            atomicAdd(node, (unsigned long long)(__double_as_longlong(__fma_rn(v, unit, m)) - __double_as_longlong(m)));
          } else {
            __hip_atomic_fetch_add(reinterpret_cast<double*>(node), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
    };
    if (q > 0) __syncthreads();                                     // the sums before have been read
    sh.clear(T);
    if (q == 0 && threadIdx.x == 0) bad = 0u;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (s0 + g * T + threadIdx.x < s1) add(own[g]);
    if (threadIdx.x < total) add(edge);
    for (uint32_t x = s0 + G * T + threadIdx.x; x < s1; x += T) {
      Part p;
      fetch(p, x, 0, q, q + 1);
      add(p);
    }
    for (uint32_t x0 = T; x0 < total; x0 += T) {                    // every lane of a wave takes part in the search
      const uint32_t x = x0 + threadIdx.x, pl = bd.place(min(x, total - 1), nb);
      if (x < total) {
        Part p;
        fetch(p, pl, nb, q, q + 1);
        add(p);
      }
    }
    __syncthreads();

    float* o = out + q * mesh_stride + ((long)(tx * kTile) * nm + ty * kTile) * row_stride + tz * kTile;
    for (int qd = threadIdx.x; qd < kTile * kTile * kTile / 4; qd += T) {
      const int nx = qd >> 6, ny = (qd >> 2) & 15, nz = (qd & 3) * 4;
      float r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned long long a = sh.acc[(nx * kAcc + ny) * kAcc + nz + j];
        r[j] = fixed ? (float)(((double)(int32_t)(a >> 32) * 4294967296.0 + (double)(uint32_t)a) * inv)
                     : (float)__longlong_as_double((long long)a);
        if (bad) r[j] = __builtin_nanf("");   // the transforms that follow spread it over the mesh
      }
      *reinterpret_cast<float4*>(o + ((long)nx * nm + ny) * row_stride + nz) = make_float4(r[0], r[1], r[2], r[3]);
    }
  }
}

// Largest |w| of each component as float bits (NaN above infinity), into maxw
// (cleared by the caller).
__global__ __launch_bounds__(256) void k_weight_max(const float* __restrict__ wt, long np3, uint32_t* __restrict__ maxw) {
  wt += blockIdx.y * np3;
  uint32_t m = 0;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < np3 / 4; i += gridDim.x * 256L) {   // np3 is a multiple of 4096
    const uint4 v = reinterpret_cast<const uint4*>(wt)[i];
    m = max(max(max(v.x & 0x7fffffffu, v.y & 0x7fffffffu), max(v.z & 0x7fffffffu, v.w & 0x7fffffffu)), m);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  // one atomic per workgroup: those on one address take some 10 ns each
  __shared__ uint32_t wave[4];
  if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(maxw + blockIdx.y, max(max(wave[0], wave[1]), max(wave[2], wave[3])));
}

void launch_deposit_weighted(const float* disp, const uint32_t* perm, const uint32_t* off, int np,
                             int nm, const float* wt, int ncomp, uint32_t* maxw, float* out, long row_stride,
                             long mesh_stride_floats, hipStream_t s) {
  const long np3 = (long)np * np * np;
  const int nt = nm / kTile;
  const long ntiles = (long)nt * nt * nt;
  launch_fill_u32(maxw, ncomp, 0u, s);
  const long blocks = np3 / 4096;
  hipLaunchKernelGGL(k_weight_max, dim3((unsigned)(blocks < 256 ? blocks : 256), (unsigned)ncomp), dim3(256), 0, s, wt,
                     np3, maxw);
  const bool many = np3 > 1024 * ntiles;
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)ntiles), dim3(threads), 0, s, disp, perm, off, np, nm, np3, wt, maxw, out,
                       row_stride, mesh_stride_floats);
  };
  if (ncomp == 3) many ? go(k_deposit_weighted<3, 1024, 1>, 1024) : go(k_deposit_weighted<3, 256, 2>, 256);
  else many ? go(k_deposit_weighted<2, 1024, 1>, 1024) : go(k_deposit_weighted<2, 256, 2>, 256);
}

}  // namespace cola
