// Tile sort for the deterministic CIC deposit: bucket = (16^3 tile of the home
// cell, face class).  Integer atomics only; the order inside a bucket is
// arbitrary (both deposits add integers and do not depend on it).
//
// Two passes over the displacements: the first counts, the second (after the
// scan) finds each particle's place again and writes what the deposit reads
// there, so nothing per particle is kept between them.  Displacements that
// another stream changes between the two get a wrong place, but none outside the
// arrays (the deposits take whatever lies at a place as a valid cell and id).  A
// workgroup of either
// pass takes 1024 particles, four per thread with all loads issued first, and
// counts them by bucket in an LDS table, so that its chain of dependent
// requests (positions, table, one global atomic per bucket) is paid once per
// 1024 particles.
#include "cola_device.h"
#include "cola_internal.h"

namespace cola {

__global__ void k_fill_u32(uint32_t* __restrict__ p, long n, uint32_t v, long mstride) {
  p = mock_ptr(p, mstride);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_u32(uint32_t* p, long n, uint32_t v, hipStream_t s, int nmock, long mstride) {
  if (n <= 0) return;
  long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks, 1, (unsigned)nmock), dim3(256), 0, s, p, n, v,
                     mstride);
}

// LDS table of a workgroup's buckets: open addressing, at most 1024 keys.
constexpr uint32_t kSlots = 2048, kEmpty = 0xffffffffu;
constexpr int kPer = 4;                // particles per thread

struct BinTable {
  uint32_t key[kSlots], cnt[kSlots];
};

__device__ __forceinline__ void table_clear(BinTable& h) {
  for (uint32_t j = threadIdx.x; j < kSlots / 4; j += 256) {
    reinterpret_cast<uint4*>(h.key)[j] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
    reinterpret_cast<uint4*>(h.cnt)[j] = make_uint4(0u, 0u, 0u, 0u);
  }
}

__device__ __forceinline__ uint32_t table_slot(BinTable& h, uint32_t b) {
  uint32_t s = (b * 2654435761u) >> 21;
  for (;;) {
    const uint32_t prev = atomicCAS(&h.key[s], kEmpty, b);
    if (prev == kEmpty || prev == b) return s;
    s = (s + 1) & (kSlots - 1);
  }
}

// Particle u (0 .. 3) of thread t in block b of np^3 / 1024: four sub-cubes of
// subcube_particle stacked along i (8 x 4 x 32 ids, 16 x 4 x 16 when np is not
// a multiple of 32): few buckets per workgroup.
__device__ __forceinline__ long sort_particle(uint32_t b, int t, int u, int np) {
  const int lk = (np & 31) == 0 ? 5 : 4;
  const uint32_t layer = ((uint32_t)np >> lk) * ((uint32_t)np >> 2);   // sub-cubes per layer along i
  const uint32_t bi = b / layer;
  return subcube_particle((bi * kPer + u) * layer + (b - bi * layer), t, np);
}

__global__ __launch_bounds__(256) void k_tile_count(const float* __restrict__ disp, int np, int nm, float dscale,
                                                    long np3, uint32_t* __restrict__ counts, long mstride) {
  __shared__ __align__(16) BinTable h;
  disp = mock_ptr(disp, mstride);
  counts = mock_ptr(counts, mstride);
  const uint32_t blk = xcd_remap(blockIdx.x, gridDim.x);
  long id[kPer];
  float d[kPer][3];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    id[u] = sort_particle(blk, threadIdx.x, u, np);
#pragma unroll
    for (int e = 0; e < 3; ++e) d[u][e] = disp[e * np3 + id[u]];
  }
  table_clear(h);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    int c[3];
    float f[3];
    home_cell_of(d[u], (uint32_t)id[u], np, nm, dscale, c, f);
    atomicAdd(&h.cnt[table_slot(h, bucket_of(c, nm >> 4))], 1u);
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < kSlots; j += 256)
    if (h.key[j] != kEmpty) atomicAdd(&counts[h.key[j]], h.cnt[j]);
}

// cursor: the buckets' starts, advanced to their ends.  REC: fractions and
// cell-in-tile of each particle (fxy, fzc) at its place; PERM: its id.
template <bool REC, bool PERM>
__global__ __launch_bounds__(256) void k_tile_fill(const float* __restrict__ disp, int np, int nm, float dscale,
                                                   long np3, uint32_t* __restrict__ cursor, float2* __restrict__ fxy,
                                                   float2* __restrict__ fzc, uint32_t* __restrict__ perm,
                                                   long mstride) {
  __shared__ __align__(16) BinTable h;
  disp = mock_ptr(disp, mstride);
  cursor = mock_ptr(cursor, mstride);
  const uint32_t blk = xcd_remap(blockIdx.x, gridDim.x);
  long id[kPer];
  float d[kPer][3];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    id[u] = sort_particle(blk, threadIdx.x, u, np);
#pragma unroll
    for (int e = 0; e < 3; ++e) d[u][e] = disp[e * np3 + id[u]];
  }
  table_clear(h);
  __syncthreads();
  uint32_t slot[kPer], rank[kPer], cell[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    int c[3];
    float f[3];
    home_cell_of(d[u], (uint32_t)id[u], np, nm, dscale, c, f);
    slot[u] = table_slot(h, bucket_of(c, nm >> 4));
    rank[u] = atomicAdd(&h.cnt[slot[u]], 1u);
    cell[u] = (uint32_t)(((c[0] & 15) << 8) | ((c[1] & 15) << 4) | (c[2] & 15));
#pragma unroll
    for (int e = 0; e < 3; ++e) d[u][e] = f[e];
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < kSlots; j += 256)
    if (h.key[j] != kEmpty) h.cnt[j] = atomicAdd(&cursor[h.key[j]], h.cnt[j]);
  __syncthreads();
  if constexpr (REC) {
    fxy = mock_ptr(fxy, mstride);
    fzc = mock_ptr(fzc, mstride);
  }
  if constexpr (PERM) perm = mock_ptr(perm, mstride);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const uint32_t p = min(h.cnt[slot[u]] + rank[u], (uint32_t)np3 - 1u);   // past it if the displacements changed
    if constexpr (REC) {
      fxy[p] = make_float2(d[u][0], d[u][1]);
      fzc[p] = make_float2(d[u][2], __uint_as_float(cell[u]));
    }
    if constexpr (PERM) perm[p] = (uint32_t)id[u];
  }
}

// ---------------------------------------------------------------------------
// Exclusive scan.  Up to kScanOne entries: one workgroup.  More: block sums,
// scan of block sums, block scan.  in receives the scan as well (the fill's
// cursor) where both is set.
constexpr int kScanT = 256;
constexpr int kScanPer = 16;
constexpr long kScanChunk = (long)kScanT * kScanPer;
constexpr int kScanOneT = 1024;
constexpr long kScanOne = 65536;

// Exclusive prefix of v over the workgroup (T threads) and the total.
template <int T>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t a = __shfl_up(incl, off, 64);
    if (lane >= off) incl += a;
  }
  __syncthreads();                     // sh may still be read from an earlier call
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const uint32_t s = sh[w];
    before += w < wave ? s : 0u;
    all += s;
  }
  *total = all;
  return before + incl - v;
}

// kV vectors of 4 entries per thread and round, vector j of thread t at 4 (j T + t):
// one round trip to memory bounds it, so a wave's access is 1 KB in a row (32
// entries in a row per thread, 16-byte accesses 128 bytes apart, took 14.8 us
// for the 32768 buckets of a 256 mesh; this order takes 7.2 us).
template <int kV>
__global__ __launch_bounds__(kScanOneT) void k_scan_one(uint32_t* __restrict__ in, uint32_t* __restrict__ out, long n,
                                                        int both, long mstride) {
  constexpr int W = kScanOneT / 64, NS = kV * W;   // wave sums of a round, in the order of the entries
  __shared__ uint32_t sh[NS + 1];
  in = mock_ptr(in, mstride);
  out = mock_ptr(out, mstride);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (long base = 0; base < n; base += 4L * kScanOneT * kV) {
    uint4 v[kV];
    uint32_t loc[kV], incl[kV];
#pragma unroll
    for (int j = 0; j < kV; ++j) {
      const long p = base + 4L * (j * kScanOneT + threadIdx.x);
      if (p + 4 <= n) {
        v[j] = *reinterpret_cast<const uint4*>(in + p);
      } else {
        v[j] = make_uint4(p < n ? in[p] : 0u, p + 1 < n ? in[p + 1] : 0u, p + 2 < n ? in[p + 2] : 0u, 0u);
      }
    }
#pragma unroll
    for (int j = 0; j < kV; ++j) incl[j] = loc[j] = (v[j].x + v[j].y) + (v[j].z + v[j].w);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
      for (int j = 0; j < kV; ++j) {
        const uint32_t a = __shfl_up(incl[j], off, 64);
        if (lane >= off) incl[j] += a;
      }
    }
    if (lane == 63) {
#pragma unroll
      for (int j = 0; j < kV; ++j) sh[j * W + wave] = incl[j];
    }
    __syncthreads();
    if (wave == 0) {
      // exclusive scan of the wave sums, 64 at a time
      uint32_t run = 0;
#pragma unroll
      for (int k = 0; k < NS; k += 64) {
        const uint32_t s = k + lane < NS ? sh[k + lane] : 0u;
        uint32_t a = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t b = __shfl_up(a, off, 64);
          if (lane >= off) a += b;
        }
        if (k + lane < NS) sh[k + lane] = run + a - s;
        run += __shfl(a, 63, 64);
      }
      if (lane == 0) sh[NS] = run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kV; ++j) {
      const long p = base + 4L * (j * kScanOneT + threadIdx.x);
      const uint32_t ex = carry + sh[j * W + wave] + incl[j] - loc[j];
      const uint32_t s1 = ex + v[j].x, s2 = s1 + v[j].y, s3 = s2 + v[j].z;
      const uint4 o = make_uint4(ex, s1, s2, s3);
      if (p + 4 <= n) {
        *reinterpret_cast<uint4*>(out + p) = o;
        if (both) *reinterpret_cast<uint4*>(in + p) = o;
      } else {
        const uint32_t q[3] = {o.x, o.y, o.z};
        for (int u = 0; u < 3; ++u)
          if (p + u < n) {
            out[p + u] = q[u];
            if (both) in[p + u] = q[u];
          }
      }
    }
    carry += sh[NS];
    __syncthreads();                   // sh is written again in the next round
  }
  if (threadIdx.x == 0) out[n] = carry;
}

__global__ __launch_bounds__(kScanT) void k_scan_reduce(const uint32_t* __restrict__ in, long n,
                                                        uint32_t* __restrict__ bsum, long mstride) {
  __shared__ uint32_t sh[kScanT / 64];
  in = mock_ptr(in, mstride);
  bsum = mock_ptr(bsum, mstride);
  const long base = blockIdx.x * kScanChunk;
  uint32_t acc = 0;
  for (int j = 0; j < kScanPer; ++j) {
    const long i = base + (long)j * kScanT + threadIdx.x;
    if (i < n) acc += in[i];
  }
  uint32_t tot;
  block_exclusive_scan<kScanT>(acc, sh, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Scans the block sums in place with one workgroup.
__global__ __launch_bounds__(kScanT) void k_scan_blocksums(uint32_t* __restrict__ bsum, long nb,
                                                           long mstride) {
  __shared__ uint32_t sh[kScanT / 64];
  bsum = mock_ptr(bsum, mstride);
  uint32_t carry = 0;
  for (long base = 0; base < nb; base += kScanT * (long)kScanPer) {
    uint32_t v[kScanPer];
    uint32_t loc = 0;
    for (int j = 0; j < kScanPer; ++j) {
      const long i = base + (long)threadIdx.x * kScanPer + j;
      v[j] = i < nb ? bsum[i] : 0u;
      loc += v[j];
    }
    uint32_t tot;
    uint32_t ex = block_exclusive_scan<kScanT>(loc, sh, &tot) + carry;
    for (int j = 0; j < kScanPer; ++j) {
      const long i = base + (long)threadIdx.x * kScanPer + j;
      if (i < nb) bsum[i] = ex;
      ex += v[j];
    }
    carry += tot;
  }
}

// Four rounds of 1024 entries, four consecutive ones per thread (16-byte
// accesses; the arrays are 16-byte aligned).
__global__ __launch_bounds__(kScanT) void k_scan_apply(uint32_t* __restrict__ in, long n,
                                                       const uint32_t* __restrict__ bsum,
                                                       uint32_t* __restrict__ out, int both, long mstride) {
  __shared__ uint32_t sh[kScanT / 64];
  in = mock_ptr(in, mstride);
  bsum = mock_ptr(bsum, mstride);
  out = mock_ptr(out, mstride);
  constexpr int kR = kScanPer / 4;
  const long base = blockIdx.x * kScanChunk + (long)threadIdx.x * 4;
  uint4 v[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    const long i = base + r * 4L * kScanT;
    if (i + 4 <= n) {
      v[r] = *reinterpret_cast<const uint4*>(in + i);
    } else {
      v[r].x = i < n ? in[i] : 0u;
      v[r].y = i + 1 < n ? in[i + 1] : 0u;
      v[r].z = i + 2 < n ? in[i + 2] : 0u;
      v[r].w = 0u;
    }
  }
  uint32_t carry = bsum[blockIdx.x];
#pragma unroll
  for (int r = 0; r < kR; ++r) {
    const long i = base + r * 4L * kScanT;
    uint32_t tot;
    const uint32_t s1 = v[r].x, s2 = s1 + v[r].y, s3 = s2 + v[r].z;
    const uint32_t ex = block_exclusive_scan<kScanT>(s3 + v[r].w, sh, &tot) + carry;
    const uint4 o = make_uint4(ex, ex + s1, ex + s2, ex + s3);
    carry += tot;
    if (i + 4 <= n) {
      *reinterpret_cast<uint4*>(out + i) = o;
      if (both) *reinterpret_cast<uint4*>(in + i) = o;
    } else {
      const uint32_t q[3] = {o.x, o.y, o.z};
      for (int j = 0; j < 3; ++j)
        if (i + j < n) {
          out[i + j] = q[j];
          if (both) in[i + j] = q[j];
        }
    }
    // out[n] = total, written by the thread that holds element n-1
    if (i < n && n <= i + 4) out[n] = ex + s3 + v[r].w;
  }
}

void launch_exclusive_scan(uint32_t* in, uint32_t* out, long n, uint32_t* scratch, int both,
                           hipStream_t s, int nmock, long mstride) {
  const unsigned z = (unsigned)nmock;
  if (n <= kScanOne) {
    if (n <= 4L * kScanOneT)
      hipLaunchKernelGGL(k_scan_one<1>, dim3(1, 1, z), dim3(kScanOneT), 0, s, in, out, n, both, mstride);
    else
      hipLaunchKernelGGL(k_scan_one<8>, dim3(1, 1, z), dim3(kScanOneT), 0, s, in, out, n, both, mstride);
    return;
  }
  const long nb = (n + kScanChunk - 1) / kScanChunk;
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb, 1, z), dim3(kScanT), 0, s, in, n, scratch, mstride);
  hipLaunchKernelGGL(k_scan_blocksums, dim3(1, 1, z), dim3(kScanT), 0, s, scratch, nb, mstride);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb, 1, z), dim3(kScanT), 0, s, in, n, scratch, out, both,
                     mstride);
}

void launch_tile_sort(const float* disp, int np, int nm, float dscale, const TileSort& ts, hipStream_t s, int nmock,
                      long mstride) {
  const long np3 = (long)np * np * np;   // np is a multiple of 16: whole workgroups
  const long nt = nm / 16, nb = 8 * nt * nt * nt;
  const dim3 grid((unsigned)(np3 / (256 * kPer)), 1, (unsigned)nmock);
  launch_fill_u32(ts.cursor, nb + 1, 0u, s, nmock, mstride);
  hipLaunchKernelGGL(k_tile_count, grid, dim3(256), 0, s, disp, np, nm, dscale, np3, ts.cursor, mstride);
  launch_exclusive_scan(ts.cursor, ts.offsets, nb, ts.scan, 1, s, nmock, mstride);
  if (ts.fxy && ts.perm)
    hipLaunchKernelGGL((k_tile_fill<true, true>), grid, dim3(256), 0, s, disp, np, nm, dscale, np3, ts.cursor, ts.fxy,
                       ts.fzc, ts.perm, mstride);
  else if (ts.fxy)
    hipLaunchKernelGGL((k_tile_fill<true, false>), grid, dim3(256), 0, s, disp, np, nm, dscale, np3, ts.cursor, ts.fxy,
                       ts.fzc, nullptr, mstride);
  else
    hipLaunchKernelGGL((k_tile_fill<false, true>), grid, dim3(256), 0, s, disp, np, nm, dscale, np3, ts.cursor, nullptr,
                       nullptr, ts.perm, mstride);
}

}  // namespace cola
