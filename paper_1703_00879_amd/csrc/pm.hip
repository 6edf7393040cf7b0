// Particle-mesh kernels: CIC deposit, real-space screening, CIC gather fused with the
// COLA kick and drift, stand-alone k-space operators, layout copies and P(k) binning.
//
// Particle p sits in row-major Lagrangian order, p = (ix*np + iy)*np + iz, at
// q = (ix*ratio + 1/2) cells per axis (ratio = nmesh/np, an integer), so its position in
// cells is s = ix*ratio + f with f = 1/2 + u/cell.  The integer and fractional parts are
// kept apart: the CIC offset d = f - floor(f) is exact in single precision, whatever the
// box size, and only u/cell carries rounding.

#include <algorithm>

#include "internal.h"
#include "kspace.h"

namespace cola {

// ------------------------------------------------------------------ helpers
struct CicCell {
  int64_t i0[3], i1[3];   // wrapped mesh coordinates of the two nodes per axis
  float w0[3], w1[3];     // their weights (1 - d, d)
};

__device__ __forceinline__ void cic_axis(int ixq, float u, int nm, int ratio, float inv_cell,
                                         int64_t& i0, int64_t& i1, float& w0, float& w1) {
  const float f = fmaf(u, inv_cell, 0.5f);
  const float fl = floorf(f);
  const float d = f - fl;
  int i = ixq * ratio + (int)fl;
  i %= nm;
  if (i < 0) i += nm;
  i0 = i;
  i1 = (i + 1 == nm) ? 0 : i + 1;
  w0 = 1.f - d;
  w1 = d;
}

static bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
static int ilog2(int v) {
  int l = 0;
  while ((1 << (l + 1)) <= v) ++l;
  return l;
}

static unsigned grid_for(int64_t n, int block, int64_t cap = 1 << 20) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + block - 1) / block, cap));
}

// ------------------------------------------------------------------ fill
__global__ void k_fill(float* __restrict__ p, int64_t n, float v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill(float* p, size_t n, float v, hipStream_t s) {
  ProfScope ps("fill", s);
  hipLaunchKernelGGL(k_fill, dim3(grid_for(n, 256)), dim3(256), 0, s, p, (int64_t)n, v);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ CIC deposit
// rho_j = sum_p m W(x_p - x_j), m = (nmesh/np)^3 so that rho averages to 1.
//
// Device-wide float atomics on a multi-GB mesh resolve beyond the per-XCD L2 caches and
// run far below HBM bandwidth, so the deposit is a counting sort instead:
//  1. count: every particle finds its home tile (the T^3-cell tile holding its lower CIC
//     corner i0) and its class c = bitmask of the axes on which i0 sits on the tile's
//     last layer (c != 0: some corners spill into the next tile), and its rank among the
//     particles of the same (tile, class).  Work-groups take Lagrangian bricks of 4x8x8
//     particles, which land in few tiles, and count in LDS before they add to the
//     global counters;
//  2. scan: exclusive prefix over tiles, then the first place of each class in its tile;
//  3. scatter: every particle writes its CIC record to its class's first place plus its rank
//     (4 bytes a particle written by the count and read here, instead of a second round of
//     returning atomics);
//  4. deposit: one work-group per tile accumulates in LDS the corners that fall inside it
//     -- from every particle of its own tile and from the class-c particles of the seven
//     lower neighbour tiles T - delta with (c & delta) == delta -- and writes the tile
//     once with plain stores, so the mesh needs no zeroing pass.
constexpr int kBrickX = 4, kBrickY = 8, kBrickZ = 8;   // 256 particles per brick
constexpr int kBinBricks = 2;                           // bricks a counting work-group takes at a time
constexpr int kScatterBricks = 2;                       // bricks per scatter work-group
constexpr int kScanBlock = 1024;                        // tiles per scan block
constexpr float kFix = 16777216.f;                      // 2^24: deposit fixed-point unit
// Threads per tile work-group: the LDS accumulator (32 KB for 16^3 cells) allows four
// work-groups per CU, and eight waves each keep more entry loads and LDS atomics in
// flight than four (sixteen measured slower).
constexpr int kDepositThreads = 512;

size_t bins_bytes(int64_t ntiles) {
  const int64_t nblk = (ntiles + kScanBlock - 1) / kScanBlock;
  return align_up((size_t)(17 * ntiles + 2 * nblk + 64) * sizeof(uint32_t));
}

struct BinGeo {
  int np, nm, ratio, nt1, tile;
  int lt;         // log2(tile); the tile side is always a power of two
  int lnp, lnm;   // log2(np), log2(nm) when both are powers of two (the P2 kernels)
  float inv_cell;
  int64_t N;
};

// Lower CIC corner (cell) and offset in [0, 1) of one axis; the same arithmetic as cic_axis().
// For f in (-2^-25, 0) f - floor(f) rounds to 1: such a particle sits on the next cell, which
// cic_axis gives all of its weight.
// P2: nm is a power of two, and the wrap is a mask (exact for negative cells too).
template <bool P2>
__device__ __forceinline__ int axis_cell(int ixq, float u, const BinGeo& g, float& d) {
  const float f = fmaf(u, g.inv_cell, 0.5f);
  float fl = floorf(f);
  d = f - fl;
  if (d >= 1.f) {
    fl += 1.f;
    d = 0.f;
  }
  if (P2) return (ixq * g.ratio + (int)fl) & (g.nm - 1);
  int i = (ixq * g.ratio + (int)fl) % g.nm;
  return i < 0 ? i + g.nm : i;
}

template <bool P2>
__device__ __forceinline__ bool brick_particle(const BinGeo& g, int b, int& ix, int& iy, int& iz,
                                               int64_t& p) {
  const int nbz = (g.np + kBrickZ - 1) / kBrickZ, nby = (g.np + kBrickY - 1) / kBrickY;
  const int nbx = (g.np + kBrickX - 1) / kBrickX;
  if (b >= nbx * nby * nbz) return false;
  int bz, by, bx;
  if (P2 && g.np >= kBrickY) {   // np / 8 bricks per axis, a power of two
    const int l = g.lnp - 3;
    bz = b & ((1 << l) - 1);
    by = (b >> l) & ((1 << l) - 1);
    bx = b >> (2 * l);
  } else {
    bz = b % nbz;
    by = (b / nbz) % nby;
    bx = b / (nbz * nby);
  }
  const int t = threadIdx.x;
  ix = bx * kBrickX + (t >> 6);
  iy = by * kBrickY + ((t >> 3) & 7);
  iz = bz * kBrickZ + (t & 7);
  if (ix >= g.np || iy >= g.np || iz >= g.np) return false;
  p = ((int64_t)ix * g.np + iy) * g.np + iz;
  return true;
}

// CIC record of a particle (12 bytes): per axis, the lower corner's cell inside its home
// tile (bits 28-31) and the offset d in [0, 1) as a 28-bit fraction (bits 0-27), whose
// conversion back to FP32 is exact.  From 2^-5 on, d is a multiple of 2^-28 and the record
// lossless; a smaller d, which f = 1/2 + u/cell may leave with more bits where the two
// nearly cancel, loses less than 2^-28, a sixteenth of the deposit's unit of weight.  Four
// bytes less per particle than a float4 record, written by the scatter and read by the deposit.
struct CicRec {
  uint32_t x, y, z;
};
__device__ __forceinline__ uint32_t rec_axis(int local, float d) {
  return ((uint32_t)local << 28) | (uint32_t)(d * 268435456.f);
}
__device__ __forceinline__ float rec_d(uint32_t v) {
  return (float)(v & 0x0FFFFFFFu) * (1.f / 268435456.f);
}

// A particle's sort key, tile * 8 + class, and its CIC record.
template <bool P2>
__device__ __forceinline__ unsigned bin_key(const BinGeo& g, int ix, int iy, int iz, float ux, float uy,
                                            float uz, CicRec& rec) {
  float dx, dy, dz;
  const int cx = axis_cell<P2>(ix, ux, g, dx);
  const int cy = axis_cell<P2>(iy, uy, g, dy);
  const int cz = axis_cell<P2>(iz, uz, g, dz);
  const int lt = g.lt, m = g.tile - 1;
  const int tile = ((cx >> lt) * g.nt1 + (cy >> lt)) * g.nt1 + (cz >> lt);
  const int cls = ((cx & m) == m ? 1 : 0) | ((cy & m) == m ? 2 : 0) | ((cz & m) == m ? 4 : 0);
  rec = CicRec{rec_axis(cx & m, dx), rec_axis(cy & m, dy), rec_axis(cz & m, dz)};
  return (unsigned)tile * 8u + (unsigned)cls;
}

// Count: cnt[key] += the particles of each key, and rank[] gets every particle's place among
// its key's (in brick order: rank[brick * 256 + thread]).
//
// A work-group takes `iters` pairs of consecutive bricks, each thread one particle of each
// brick, and counts in an LDS hash table first: the lanes of a wave that share a key are
// grouped by ballots (a wave holds an 8 x 8 patch of one lattice plane, so it meets few
// keys), each group makes one LDS add, and each key of the table makes one global add at
// the end.  What bounds the pass otherwise, once many particles from all over the box sit in
// few cells, is the rate of global adds to one cache line of counters, one in 11 ns: 512^3
// particles, a quarter of them in 64 clumps, were counted in 6.3 ms with one global add a
// group and scattered in another 6.3; now 2.0 and 1.55 (unclustered 0.52 + 0.96, now 0.67 +
// 1.0: the rank costs 8 bytes a particle).  A key that finds no slot within kBinProbe goes to
// the global counter directly.
constexpr int kBinIters = 8;        // at most; large runs take all, small ones fill the chip
constexpr int kBinHash = 1024;      // slots: 16 bricks late in a run meet a few hundred keys
constexpr int kBinProbe = 16;
constexpr int kBinGroups = 12;
constexpr uint32_t kBinEmpty = 0xffffffffu, kBinDirect = 0x80000000u;

template <bool P2>
__global__ void __launch_bounds__(256)
k_bin_count(const float* __restrict__ disp, BinGeo g, int iters, uint32_t* __restrict__ cnt,
            uint32_t* __restrict__ rank, int nbricks) {
  constexpr int S = kBinBricks;
  __shared__ uint32_t hkey[kBinHash], hcnt[kBinHash];
  // a particle's (slot << 16 | rank within the work-group), or kBinDirect | its final rank
  __shared__ uint32_t code[kBinIters * S * 256];
  for (int i = threadIdx.x; i < kBinHash; i += 256) {
    hkey[i] = kBinEmpty;
    hcnt[i] = 0u;
  }
  __syncthreads();
  const int first = (int)xcd_block(blockIdx.x, gridDim.x) * S * iters;
  const int lane = (int)__lane_id();
  struct Next {   // the particles of the coming pair of bricks, loaded ahead
    bool valid;
    int ix, iy, iz;
    float ux, uy, uz;
  } nx[S];
  auto issue = [&](int it) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      int64_t p = 0;
      nx[s] = Next{false, 0, 0, 0, 0.f, 0.f, 0.f};
      if (it < iters) nx[s].valid = brick_particle<P2>(g, first + it * S + s, nx[s].ix, nx[s].iy, nx[s].iz, p);
      if (nx[s].valid) {
        nx[s].ux = disp[p];
        nx[s].uy = disp[g.N + p];
        nx[s].uz = disp[2 * g.N + p];
      }
    }
  };
  issue(0);
  for (int it = 0; it < iters; ++it) {
    unsigned kk[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      CicRec rec;
      kk[s] = nx[s].valid ? bin_key<P2>(g, nx[s].ix, nx[s].iy, nx[s].iz, nx[s].ux, nx[s].uy, nx[s].uz, rec)
                          : kBinEmpty;
    }
    issue(it + 1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const unsigned key = kk[s];
      // Group the wave's lanes by key; group i's key and size go to lane i, which makes the
      // group's one add -- all groups' adds go out as a single wave instruction.  The loop is
      // wave-uniform (scalar mask, leader and key: a dozen instructions a group).  After
      // kBinGroups groups the lanes left, whose keys are then nearly all different, add
      // for themselves.
      unsigned long long todo = __ballot(key != kBinEmpty);
      int ng = 0, mygroup = 0;
      uint32_t gcnt = 0, myrank = 0;
      unsigned gkey = 0;
      while (todo != 0ull && ng < kBinGroups) {
        const unsigned lkey = (unsigned)__builtin_amdgcn_readlane((int)key, __builtin_ctzll(todo));
        const bool mine = key == lkey;
        const unsigned long long m = __ballot(mine);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        mygroup = mine ? ng : mygroup;
        myrank = mine ? below : myrank;
        gkey = lane == ng ? lkey : gkey;
        gcnt = lane == ng ? (uint32_t)__popcll(m) : gcnt;
        todo &= ~m;
        ++ng;
      }
      auto add = [&](unsigned k, uint32_t n) -> uint32_t {
        unsigned slot = (k * 2654435761u) >> 22;   // top 10 bits
        for (int probe = 0; probe < kBinProbe; ++probe) {
          const uint32_t was = atomicCAS(&hkey[slot], kBinEmpty, k);
          if (was == kBinEmpty || was == k) return slot << 16 | atomicAdd(&hcnt[slot], n);
          slot = (slot + 1) & (kBinHash - 1);
        }
        return kBinDirect | atomicAdd(&cnt[k], n);
      };
      uint32_t base = 0;
      if (lane < ng) base = add(gkey, gcnt);
      uint32_t c = __shfl(base, mygroup) + myrank;
      if ((todo >> lane) & 1ull) c = add(key, 1u);
      code[(it * S + s) * 256 + threadIdx.x] = c;
    }
  }
  __syncthreads();
  {
    constexpr int V = kBinHash / 256;
    uint32_t k[V], n[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      k[i] = hkey[threadIdx.x + i * 256];
      n[i] = hcnt[threadIdx.x + i * 256];
    }
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (k[i] != kBinEmpty) n[i] = atomicAdd(&cnt[k[i]], n[i]);
#pragma unroll
    for (int i = 0; i < V; ++i) hcnt[threadIdx.x + i * 256] = n[i];
  }
  __syncthreads();
  const int nq = min(iters * S, nbricks - first);
  uint32_t* out = rank + (int64_t)first * 256 + threadIdx.x;
#pragma unroll 4
  for (int q = 0; q < nq; ++q) {
    const uint32_t c = code[q * 256 + threadIdx.x];
    out[q * 256] = (c & kBinDirect) ? c & ~kBinDirect : hcnt[c >> 16] + (c & 0xffffu);
  }
}

// Scatter: the same bricks write their particles' CIC records to entries[cur[key] + rank],
// cur[key] being the key's first place.
template <bool P2>
__global__ void __launch_bounds__(256)
k_bin_scatter(const float* __restrict__ disp, BinGeo g, const uint32_t* __restrict__ cur,
              const uint32_t* __restrict__ rank, CicRec* __restrict__ entries) {
  constexpr int S = kScatterBricks;
  const int b0 = (int)xcd_block(blockIdx.x, gridDim.x) * S;
  bool valid[S];
  int ix[S], iy[S], iz[S];
  float ux[S], uy[S], uz[S];
  uint32_t rk[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    int64_t p = 0;
    ix[s] = iy[s] = iz[s] = 0;
    valid[s] = brick_particle<P2>(g, b0 + s, ix[s], iy[s], iz[s], p);
    ux[s] = uy[s] = uz[s] = 0.f;
    rk[s] = 0;
    if (valid[s]) {
      ux[s] = disp[p];
      uy[s] = disp[g.N + p];
      uz[s] = disp[2 * g.N + p];
      rk[s] = rank[(int64_t)(b0 + s) * 256 + threadIdx.x];
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if (!valid[s]) continue;
    CicRec rec;
    const unsigned key = bin_key<P2>(g, ix[s], iy[s], iz[s], ux[s], uy[s], uz[s], rec);
    entries[cur[key] + rk[s]] = rec;
  }
}

// Particles of a tile, all classes.
__device__ __forceinline__ uint32_t tile_total(const uint32_t* __restrict__ cnt, int64_t tile, uint32_t* c) {
  const uint4* c4 = reinterpret_cast<const uint4*>(cnt + tile * 8);
  const uint4 a = c4[0], b = c4[1];
  c[0] = a.x; c[1] = a.y; c[2] = a.z; c[3] = a.w; c[4] = b.x; c[5] = b.y; c[6] = b.z; c[7] = b.w;
  return c[0] + c[1] + c[2] + c[3] + c[4] + c[5] + c[6] + c[7];
}

// Sum of v over the threads before this one (exclusive scan) of a work-group of 1024 at most;
// total: over all of them.  part: one word a wave.
__device__ __forceinline__ uint32_t group_scan(uint32_t v, uint32_t* part, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  __syncthreads();   // the words of an earlier scan have been read
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
  for (int w = 0; w < waves; ++w) {
    if (w < wave) before += part[w];
    total += part[w];
  }
  return before + inc - v;
}

// Tile totals -> per-block sums (block of kScanBlock tiles).
__global__ void __launch_bounds__(256)
k_scan_reduce(const uint32_t* __restrict__ cnt, uint32_t* __restrict__ bsum, int64_t ntiles) {
  __shared__ uint32_t part[16];
  const int64_t t0 = (int64_t)blockIdx.x * kScanBlock;
  uint32_t s = 0, c[8];
  for (int i = threadIdx.x; i < kScanBlock; i += 256) {
    const int64_t t = t0 + i;
    if (t < ntiles) s += tile_total(cnt, t, c);
  }
  uint32_t total;
  group_scan(s, part, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// Exclusive scan of the block sums (one work-group; nblk <= 4096 for nmesh <= 2048).
__global__ void __launch_bounds__(1024) k_scan_top(uint32_t* __restrict__ bsum, int nblk) {
  __shared__ uint32_t part[16];
  const int t = threadIdx.x;
  const int per = (nblk + 1023) / 1024;
  uint32_t s = 0;
  for (int i = 0; i < per; ++i) {
    const int j = t * per + i;
    if (j < nblk) s += bsum[j];
  }
  uint32_t total, run = group_scan(s, part, total);
  for (int i = 0; i < per; ++i) {
    const int j = t * per + i;
    if (j < nblk) {
      const uint32_t v = bsum[j];
      bsum[j] = run;
      run += v;
    }
  }
}

// Per block: scan of tile totals + block offset -> start[tile]; per-class cursors.  Up to
// kScanAlone blocks (boff null) a block adds up the tiles before its own itself, 32 KB a block
// from the L2 and up to 15 of them, and the two launches before this one are saved (192^3
// cells 14.1 -> 4.6 us, 384^3 13.8 -> 8.2).
constexpr int kScanAlone = 16;
__global__ void __launch_bounds__(kScanBlock)
k_scan_apply(const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ boff,
             uint32_t* __restrict__ start, uint32_t* __restrict__ cur, int64_t ntiles) {
  __shared__ uint32_t part[16];
  const int t = threadIdx.x;
  const int64_t tile = (int64_t)blockIdx.x * kScanBlock + t;
  uint32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  uint32_t offset = 0, total;
  if (boff) {
    offset = boff[blockIdx.x];
  } else if (blockIdx.x > 0) {
    uint32_t s = 0;
    for (unsigned b = 0; b < blockIdx.x; ++b) s += tile_total(cnt, (int64_t)b * kScanBlock + t, c);
    group_scan(s, part, offset);
  }
  const uint32_t tot = tile < ntiles ? tile_total(cnt, tile, c) : 0;
  const uint32_t before = group_scan(tot, part, total);
  if (tile < ntiles) {
    uint32_t run = offset + before;
    start[tile] = run;
    uint32_t cc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      cc[k] = run;
      run += c[k];
    }
    uint4* o4 = reinterpret_cast<uint4*>(cur + tile * 8);
    o4[0] = make_uint4(cc[0], cc[1], cc[2], cc[3]);
    o4[1] = make_uint4(cc[4], cc[5], cc[6], cc[7]);
  }
}

// Fixed-point sum -> density: the two 32-bit halves combine exactly in double (sums stay
// below 2^53), so the one rounding to float gives the correctly rounded v * 2^-24, as a
// direct 64-bit integer conversion would, in a handful of instructions.
__device__ __forceinline__ float fix_to_float(unsigned long long v) {
  const double d = (double)(uint32_t)(v >> 32) * 4294967296.0 + (double)(uint32_t)v;
  return (float)(d * (1.0 / kFix));
}

// One tile.  Its particles come as a list: first its own class-0 particles, whose eight
// corners all lie inside (most of them, contiguous in the sorted records), then the
// segments whose corners need a test: its other classes and, from each lower neighbour
// T - d, every class c with (c & d) == d.  A wave that holds class-0 particles only adds its
// corners at constant offsets from one LDS address without tests, and the first of them are
// loaded while the accumulator is cleared and the segment list built: 1.96 ms for 512^3
// particles on 1024^3 cells, with every corner tested and every record looked up in the
// list 2.02.  What is left is the latency of a tile (counts, records, stores: 7.6 us with
// four tiles a CU; the LDS adds take 0.3 ms of the pass).
template <int T>
__global__ void __launch_bounds__(kDepositThreads)
k_deposit_tiles(const CicRec* __restrict__ entries, const uint32_t* __restrict__ start,
                const uint32_t* __restrict__ cnt, BinGeo g, float* __restrict__ rho, int rpitch,
                int64_t rplane, float mass) {
  // 64-bit fixed-point accumulation in units of 2^-24: integer LDS atomics run several
  // times faster than float ones here, and integer sums do not depend on the order of
  // the particles, so the density mesh is bitwise reproducible.  A contribution is at
  // most the particle mass (nmesh/np)^3 <= 64 (< 2^32 units), and a cell overflows only
  // beyond ~10^12 in mean-density units.
  __shared__ unsigned long long acc[T * T * T];
  const int nt1 = g.nt1;
  const int tile = (int)xcd_block(blockIdx.x, gridDim.x);
  const int tx = tile / (nt1 * nt1), ty = (tile / nt1) % nt1, tz = tile % nt1;
  const uint32_t n0 = cnt[(int64_t)tile * 8], st0 = start[tile];
  const CicRec* own = entries + st0;
  CicRec r0{0u, 0u, 0u};
  if (threadIdx.x < n0) r0 = own[threadIdx.x];
  for (int i = threadIdx.x; i < T * T * T; i += blockDim.x) acc[i] = 0ull;
  // Flatten the segments after the own class-0 particles into one list (at most 1 + 19).
  // Wave 0 builds it with one lane per (d, c): class offsets inside the source tile by an
  // 8-lane scan, list positions by ballot, list offsets by a wave scan.
  __shared__ uint32_t sb[20], so[21];
  __shared__ int sdd[20], nseg;
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x, d = lane >> 3, c = lane & 7;
    const int sx = (tx - (d & 1) + nt1) % nt1, sy = (ty - ((d >> 1) & 1) + nt1) % nt1,
              sz = (tz - ((d >> 2) & 1) + nt1) % nt1;
    const int64_t src = ((int64_t)sx * nt1 + sy) * nt1 + sz;
    const uint32_t nc = cnt[src * 8 + c], st = start[src];
    uint32_t incl = nc;   // inclusive scan over the 8 classes of the source tile
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      const uint32_t t = __shfl_up(incl, o, 8);
      if (c >= o) incl += t;
    }
    const uint32_t rest = __shfl(incl, 7, 8) - n0;   // of the own tile: classes 1 .. 7
    const bool valid = d == 0 ? (c == 1 && rest > 0) : ((c & d) == d && nc > 0);
    const uint32_t n = d == 0 ? rest : nc;
    const unsigned long long vm = __ballot(valid);
    const int pos = __popcll(vm & ((1ull << lane) - 1ull));
    uint32_t x = valid ? n : 0u;   // inclusive scan of the segment lengths over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(x, o, 64);
      if (lane >= o) x += t;
    }
    if (valid) {
      sb[pos] = d == 0 ? st0 + n0 : st + incl - nc;
      so[pos] = n0 + x - n;
      sdd[pos] = d;
    }
    if (lane == 63) {
      nseg = __popcll(vm);
      so[__popcll(vm)] = n0 + x;
    }
  }
  __syncthreads();
  const uint32_t total = so[nseg];
  const float unit = mass * kFix;   // scaling by the power of two commutes with the roundings
  // adds record r of source tile T - d (d < 0: none); the whole wave calls it
  auto add = [&](const CicRec& r, int d) {
    const int cx = (int)(r.x >> 28), cy = (int)(r.y >> 28), cz = (int)(r.z >> 28);
    const float dx = rec_d(r.x), dy = rec_d(r.y), dz = rec_d(r.z);
    const float wx[2] = {unit * (1.f - dx), unit * dx}, wy[2] = {1.f - dy, dy}, wz[2] = {1.f - dz, dz};
    auto val = [&](int o) {
      return (unsigned long long)__float2uint_rn(wx[o & 1] * wy[(o >> 1) & 1] * wz[(o >> 2) & 1]);
    };
    if (__all(d < 0 || (d == 0 && cx < T - 1 && cy < T - 1 && cz < T - 1))) {
      if (d == 0) {
        unsigned long long* at = acc + (cx * T + cy) * T + cz;
#pragma unroll
        for (int o = 0; o < 8; ++o) atomicAdd(at + (o & 1) * T * T + ((o >> 1) & 1) * T + ((o >> 2) & 1), val(o));
      }
    } else if (d >= 0) {
      // the lower corner of a particle of tile T - d lies at (home-tile coordinate - T)
      // on every axis where d is set
      const int lx0 = cx - ((d & 1) ? T : 0), ly0 = cy - (((d >> 1) & 1) ? T : 0),
                lz0 = cz - (((d >> 2) & 1) ? T : 0);
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        const int lx = lx0 + (o & 1), ly = ly0 + ((o >> 1) & 1), lz = lz0 + ((o >> 2) & 1);
        if (lx >= 0 && lx < T && ly >= 0 && ly < T && lz >= 0 && lz < T)
          atomicAdd(&acc[(lx * T + ly) * T + lz], val(o));
      }
    }
  };
  // the list's element e and its source
  int sg = 0;
  auto fetch = [&](uint32_t e, CicRec& r) -> int {
    r = CicRec{0u, 0u, 0u};
    if (e >= total) return -1;
    if (e < n0) {
      r = own[e];
      return 0;
    }
    while (so[sg + 1] <= e) ++sg;
    r = entries[sb[sg] + (e - so[sg])];
    return sdd[sg];
  };
  // batches of KB records per thread: all loads are issued before the LDS accumulation
  constexpr int KB = 4;
  for (uint32_t e0 = 0; e0 < total; e0 += KB * kDepositThreads) {
    CicRec r[KB];
    int dd[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const uint32_t e = e0 + k * kDepositThreads + threadIdx.x;
      if (k == 0 && e0 == 0 && e < n0) {
        r[0] = r0;
        dd[0] = 0;
      } else {
        dd[k] = fetch(e, r[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < KB; ++k)
      if (e0 + k * kDepositThreads < total) add(r[k], dd[k]);   // uniform over the work-group
  }
  __syncthreads();
  // 16-byte stores: T, the row pitch and the plane stride are multiples of 4 floats
  const int ox = tx * T, oy = ty * T, oz = tz * T;
  for (int i4 = threadIdx.x; i4 < T * T * T / 4; i4 += blockDim.x) {
    const int i = 4 * i4;
    const int lx = i / (T * T), ly = (i / T) % T, lz = i % T;
    *reinterpret_cast<float4*>(rho + (int64_t)(ox + lx) * rplane + (int64_t)(oy + ly) * rpitch + oz + lz) =
        make_float4(fix_to_float(acc[i]), fix_to_float(acc[i + 1]), fix_to_float(acc[i + 2]),
                    fix_to_float(acc[i + 3]));
  }
}

static BinGeo bin_geo(const Layout& L) {
  BinGeo g;
  g.np = L.np;
  g.nm = L.nm;
  g.ratio = L.nm / L.np;
  g.nt1 = L.nt1;
  g.tile = L.tile;
  g.inv_cell = L.inv_cell;
  g.N = L.N;
  g.lt = ilog2(L.tile);
  const bool p2 = is_pow2(L.np) && is_pow2(L.nm);
  g.lnp = p2 ? ilog2(L.np) : -1;
  g.lnm = p2 ? ilog2(L.nm) : -1;
  return g;
}

// The density of the particles whose sorted records and segment tables are in `entries`
// and `bins`.
void launch_deposit_tiles(const Layout& L, float* rho, const void* bins, const void* entries_raw,
                          hipStream_t s) {
  const CicRec* entries = static_cast<const CicRec*>(entries_raw);
  const BinGeo g = bin_geo(L);
  const uint32_t* cnt = static_cast<const uint32_t*>(bins);
  const uint32_t* start = cnt + 16 * L.ntiles;
  ProfScope ps("deposit", s);
  const float mass = (float)g.ratio * g.ratio * g.ratio;
  const dim3 grid((unsigned)L.ntiles), block(kDepositThreads);
  switch (L.tile) {
    case 16: hipLaunchKernelGGL(k_deposit_tiles<16>, grid, block, 0, s, entries, start, cnt, g, rho, 2 * L.pitch_m, 2 * L.plane_m, mass); break;
    case 8: hipLaunchKernelGGL(k_deposit_tiles<8>, grid, block, 0, s, entries, start, cnt, g, rho, 2 * L.pitch_m, 2 * L.plane_m, mass); break;
    default: hipLaunchKernelGGL(k_deposit_tiles<4>, grid, block, 0, s, entries, start, cnt, g, rho, 2 * L.pitch_m, 2 * L.plane_m, mass); break;
  }
  COLA_LAUNCH_CHECK();
}

void launch_deposit(const Layout& L, const float* disp, float* rho, void* bins, void* entries_raw,
                    void* ranks, hipStream_t s) {
  CicRec* entries = static_cast<CicRec*>(entries_raw);
  uint32_t* rank = static_cast<uint32_t*>(ranks);
  const BinGeo g = bin_geo(L);
  const bool p2 = g.lnm >= 0;
  const int64_t nblk = (L.ntiles + kScanBlock - 1) / kScanBlock;
  uint32_t* cnt = static_cast<uint32_t*>(bins);
  uint32_t* cur = cnt + 8 * L.ntiles;
  uint32_t* start = cur + 8 * L.ntiles;
  uint32_t* bsum = start + L.ntiles;
  const int64_t nbricks = (int64_t)((L.np + kBrickX - 1) / kBrickX) *
                          ((L.np + kBrickY - 1) / kBrickY) * ((L.np + kBrickZ - 1) / kBrickZ);
  const unsigned bricks = (unsigned)((nbricks + kBinBricks - 1) / kBinBricks);
  {
    ProfScope ps("bin_count", s);
    hipLaunchKernelGGL(k_fill, dim3(grid_for(8 * L.ntiles, 256)), dim3(256), 0, s,
                       reinterpret_cast<float*>(cnt), 8 * L.ntiles, 0.f);
    // more bricks a work-group means fewer global adds; 2048 work-groups still fill the chip
    const int iters = (int)std::max<int64_t>(1, std::min<int64_t>(kBinIters, bricks / 2048));
    const unsigned grid = (bricks + iters - 1) / iters;
    if (p2)
      hipLaunchKernelGGL(k_bin_count<true>, dim3(grid), dim3(256), 0, s, disp, g, iters, cnt, rank, (int)nbricks);
    else
      hipLaunchKernelGGL(k_bin_count<false>, dim3(grid), dim3(256), 0, s, disp, g, iters, cnt, rank, (int)nbricks);
    COLA_LAUNCH_CHECK();
  }
  {
    ProfScope ps("bin_scan", s);
    const bool alone = nblk <= kScanAlone;
    if (!alone) {
      hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nblk), dim3(256), 0, s, cnt, bsum, L.ntiles);
      hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, bsum, (int)nblk);
    }
    hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nblk), dim3(kScanBlock), 0, s, cnt,
                       alone ? nullptr : bsum, start, cur, L.ntiles);
    COLA_LAUNCH_CHECK();
  }
  {
    ProfScope ps("bin_scatter", s);
    const unsigned sgrid = (unsigned)((nbricks + kScatterBricks - 1) / kScatterBricks);
    if (p2)
      hipLaunchKernelGGL(k_bin_scatter<true>, dim3(sgrid), dim3(256), 0, s, disp, g, cur, rank, entries);
    else
      hipLaunchKernelGGL(k_bin_scatter<false>, dim3(sgrid), dim3(256), 0, s, disp, g, cur, rank, entries);
    COLA_LAUNCH_CHECK();
  }
  launch_deposit_tiles(L, rho, bins, entries, s);
}

// ------------------------------------------------------------------ gather + kick + drift
struct GatherDev {
  const float* F3;   // interleaved force mesh, 3 floats per cell, unpadded rows
  float* disp; float* vel;
  const float* psi1; const float* psi2;
  const float* l3; const float* d3;   // interleaved L'' and Delta (MODE 1)
  const double* table; int64_t slice0, slice1;
  float dtk, dtd;
  float* force_out;
  const StepDev* steps; const int* step_ctr;
};

// F_p = sum_corners W F_j (same CIC weights as the deposit); then
// v += dtk (F_p - L''(q_p)), u += dtd v + Delta(q_p)   (kick-drift about the LPT path).
// MODE 0: scale-independent LPT (Psi1, Psi2 per particle, growth scalars from the table);
// MODE 1: scale-dependent LPT (L'' and Delta fields on the particle grid);
// MODE 2: force only (write F_p).
//
// Work order.  Each wave takes 64 consecutive particles of one Lagrangian z-line, so its
// particle loads and (early on) its mesh rows are contiguous.  When the lattice allows
// (np a multiple of 64 and of kGatherBrick), the waves of one XCD are further grouped into
// bricks of kGatherBrick x kGatherBrick z-lines of 64 particles, taken brick after brick:
// the particles an XCD has in flight then form a compact Lagrangian region rather than a
// sheet of one lattice plane, and late in the run, when the particles of a halo come from
// many lattice planes, their force cells are fetched once into that XCD's L2 and reused.
// Otherwise blocks take consecutive particles.
constexpr int kGatherBrick = 16;

template <int MODE>
__global__ void __launch_bounds__(256)
k_gather(GatherDev g, int64_t N, int np, int nm, int ratio, float inv_cell, int bricks) {
  if (MODE != 2 && g.steps) {
    const StepDev& sd = step_entry(g.steps, g.step_ctr);
    g.dtk = sd.dtk;
    g.dtd = sd.dtd;
    g.slice0 = sd.slice0;
    g.slice1 = sd.slice1;
  }
  const unsigned blk = xcd_block(blockIdx.x, gridDim.x);
  int64_t p;
  if (bricks) {
    constexpr int kBlocksPerBrick = kGatherBrick * kGatherBrick / 4;
    const int nbz = np / 64, nby = np / kGatherBrick;
    const int brick = (int)(blk / kBlocksPerBrick);
    const int line = (int)(blk % kBlocksPerBrick) * 4 + (int)(threadIdx.x >> 6);
    const int bz = brick % nbz, by = (brick / nbz) % nby, bx = brick / (nbz * nby);
    const int ix = bx * kGatherBrick + line / kGatherBrick, iy = by * kGatherBrick + line % kGatherBrick;
    p = ((int64_t)ix * np + iy) * np + bz * 64 + (threadIdx.x & 63);
  } else {
    p = blk * (int64_t)blockDim.x + threadIdx.x;
  }
  if (p >= N) return;
  // the particle's own values (velocity, LPT terms) do not depend on its cell: their
  // loads go out first, so that they are in flight while the force corners are fetched
  float uu[3], vv[3], l[3], d[3], s1[3], s2[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) uu[a] = g.disp[a * N + p];
  if (MODE != 2) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      vv[a] = g.vel[a * N + p];
      if (MODE == 0) {
        s1[a] = g.psi1[a * N + p];
        s2[a] = g.psi2[a * N + p];
      } else {
        l[a] = g.l3[3 * p + a];
        d[a] = g.d3[3 * p + a];
      }
    }
  }
  CicCell c;
  {
    const int ip = (int)p;
    const int ix = ip / (np * np), iy = (ip / np) % np, iz = ip % np;
    cic_axis(ix, uu[0], nm, ratio, inv_cell, c.i0[0], c.i1[0], c.w0[0], c.w1[0]);
    cic_axis(iy, uu[1], nm, ratio, inv_cell, c.i0[1], c.i1[1], c.w0[1], c.w1[1]);
    cic_axis(iz, uu[2], nm, ratio, inv_cell, c.i0[2], c.i1[2], c.w0[2], c.w1[2]);
  }
  float f0 = 0.f, f1 = 0.f, f2 = 0.f;
#pragma unroll
  for (int ox = 0; ox < 2; ++ox) {
    const int64_t x = ox ? c.i1[0] : c.i0[0];
    const float wx = ox ? c.w1[0] : c.w0[0];
#pragma unroll
    for (int oy = 0; oy < 2; ++oy) {
      const int64_t y = oy ? c.i1[1] : c.i0[1];
      const float wxy = wx * (oy ? c.w1[1] : c.w0[1]);
      const int64_t row = (x * nm + y) * nm;
      const float* a = g.F3 + 3 * (row + c.i0[2]);
      const float* b = g.F3 + 3 * (row + c.i1[2]);
      const float wa = wxy * c.w0[2], wb = wxy * c.w1[2];
      f0 += wa * a[0] + wb * b[0];
      f1 += wa * a[1] + wb * b[1];
      f2 += wa * a[2] + wb * b[2];
    }
  }
  if (MODE == 2) {
    g.force_out[p] = f0;
    g.force_out[N + p] = f1;
    g.force_out[2 * N + p] = f2;
    return;
  }
  if (MODE == 0) {
    const double* t0 = g.table + g.slice0;
    const double* t1 = g.table + g.slice1;
    const float c1 = (float)t0[2], c2 = (float)t0[5];
    const float e1 = (float)(t1[0] - t0[0]), e2 = (float)(t1[3] - t0[3]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      l[a] = c1 * s1[a] + c2 * s2[a];
      d[a] = e1 * s1[a] + e2 * s2[a];
    }
  }
  const float fv[3] = {f0, f1, f2};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float v = vv[a] + g.dtk * (fv[a] - l[a]);
    g.vel[a * N + p] = v;
    g.disp[a * N + p] = uu[a] + (g.dtd * v + d[a]);
  }
}

void launch_gather(const Layout& L, const GatherArgs& a, hipStream_t s) {
  GatherDev g;
  g.F3 = a.F3;
  g.disp = a.disp; g.vel = a.vel;
  g.psi1 = a.psi1; g.psi2 = a.psi2;
  g.l3 = a.lpp3; g.d3 = a.dlt3;
  g.table = a.table; g.slice0 = a.slice0; g.slice1 = a.slice1;
  g.dtk = (float)a.dtk; g.dtd = (float)a.dtd;
  g.force_out = a.force_out;
  g.steps = a.steps;
  g.step_ctr = a.step_ctr;
  const int ratio = L.nm / L.np;
  const dim3 grid((unsigned)((L.N + 255) / 256)), block(256);
  const int bricks = (L.np % 64 == 0 && L.np % kGatherBrick == 0) ? 1 : 0;
  if (a.force_out) {
    ProfScope ps("gather_force", s);
    hipLaunchKernelGGL(k_gather<2>, grid, block, 0, s, g, L.N, L.np, L.nm, ratio, L.inv_cell,
                       bricks);
  } else if (a.psi1) {
    ProfScope ps("gather_kick_drift", s);
    hipLaunchKernelGGL(k_gather<0>, grid, block, 0, s, g, L.N, L.np, L.nm, ratio, L.inv_cell,
                       bricks);
  } else {
    ProfScope ps("gather_kick_drift", s);
    hipLaunchKernelGGL(k_gather<1>, grid, block, 0, s, g, L.N, L.np, L.nm, ratio, L.inv_cell,
                       bricks);
  }
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ k-Mouflage source
// X* >= 0 with P_X(X*)^2 X* = R, P_X = 1 + m K0 X^(m-1): Newton on y = ln X of
// f(y) = y + 2 ln P_X(e^y) - ln R, which rises with slope between 1 and 2m - 1, from the
// smaller of the two asymptotic roots; returns P_X(X*).  A step of size d leaves an error
// of at most |f''| d^2 / 2 f' <= ((m-1) d / 2)^2, so a wave stops when every lane's last step was
// below 1e-4 / (m-1), where the next is lost in rounding; 24 steps at most.  Most cells take
// three to five.
__device__ __forceinline__ float km_px_at_root(float R, float k0, int m) {
  const bool some = R > 0.f;
  const float mk = (float)m * k0, m1 = (float)(m - 1), lr = __logf(some ? R : 1.f);
  float y = fminf(lr, (lr - 2.f * __logf(mk)) / (float)(2 * m - 1));
  const float tol = 1e-4f / fmaxf(m1, 1.f);
  for (int it = 0; it < 24; ++it) {
    const float t = mk * __expf(m1 * y);   // m K0 X^(m-1)
    const float px = 1.f + t;
    const float f = y + 2.f * __logf(px) - lr;
    const float fp = 1.f + 2.f * m1 * t / px;
    const float d = f / fp;
    y -= d;
    if (__all(!(fabsf(d) > tol) || !some)) break;
  }
  return some ? 1.f + mk * __expf(m1 * y) : 1.f;
}

// A quarter above the bytes at the copy rate (384^3 cells: 1.36 GB, 0.31 ms): 0.39 ms, with 24 steps
// for every cell and 64-bit divisions 1.54.
__global__ void __launch_bounds__(256)
k_kmouflage_source(const float* __restrict__ rho, const float* __restrict__ f3,
                   float* __restrict__ out, float* __restrict__ s_out, int n,
                   int rpitch, int64_t rplane, KmArgs k) {
  if (k.steps) {
    const StepDev& sd = step_entry(k.steps, k.step_ctr);
    k.km_r = sd.km_r;
    k.cn = sd.cn;
    k.c5 = sd.c5;
  }
  CellQuad c;
  if (!cell_quad(n, rpitch, rplane, c)) return;
  float f[12];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const quad_t v = reinterpret_cast<const quad_t*>(f3 + 3 * c.e)[i];
    f[4 * i] = v.x; f[4 * i + 1] = v.y; f[4 * i + 2] = v.z; f[4 * i + 3] = v.w;
  }
  const quad_t d = *reinterpret_cast<const quad_t*>(rho + c.pe);
  quad_t o, so;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float fx = f[3 * i], fy = f[3 * i + 1], fz = f[3 * i + 2];
    const float px = km_px_at_root(k.km_r * (fx * fx + fy * fy + fz * fz), k.k0, k.m);
    const float eps = fminf(1.f, 1.f / px);
    const float dl = d[i] - 1.f;
    o[i] = dl * (k.cn + k.c5 * eps);
    so[i] = dl * eps;
  }
  *reinterpret_cast<quad_t*>(out + c.pe) = o;
  if (s_out) *reinterpret_cast<quad_t*>(s_out + c.pe) = so;
}

void launch_kmouflage_source(const Layout& L, const float* rho, const float* f3, float* out,
                             float* s_out, const KmArgs& k, hipStream_t s) {
  ProfScope ps("kmouflage_source", s);
  hipLaunchKernelGGL(k_kmouflage_source, quad_grid(L.nm), dim3(256), 0, s, rho, f3, out,
                     s_out, L.nm, 2 * L.pitch_m, 2 * L.plane_m, k);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ step table and counter
// Entries of the step table, kStepsPerLaunch at a time by value (2.3 KB of kernel arguments):
// one launch for a run of up to 32 steps where one launch an entry took 4.5 us each.
constexpr int kStepsPerLaunch = 32;
struct StepBatch {
  StepDev v[kStepsPerLaunch];
};
__global__ void k_write_steps(StepDev* steps, int n, StepBatch b) {
  if ((int)threadIdx.x < n) steps[threadIdx.x] = b.v[threadIdx.x];
}
__global__ void k_set_counter(int* ctr, int v) { *ctr = v; }
__global__ void k_step_advance(int* ctr) { *ctr += 1; }

void launch_write_steps(const cola_params& p, const Layout& L, StepDev* steps, hipStream_t s) {
  for (int i0 = 0; i0 < p.n_steps; i0 += kStepsPerLaunch) {
    const int n = std::min(kStepsPerLaunch, p.n_steps - i0);
    StepBatch b;
    for (int i = 0; i < n; ++i) b.v[i] = step_dev(p, L, i0 + i);
    hipLaunchKernelGGL(k_write_steps, dim3(1), dim3(kStepsPerLaunch), 0, s, steps + i0, n, b);
    COLA_LAUNCH_CHECK();
  }
}
void launch_set_counter(int* ctr, int v, hipStream_t s) {
  hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(1), 0, s, ctr, v);
  COLA_LAUNCH_CHECK();
}
void launch_step_advance(int* ctr, hipStream_t s) {
  hipLaunchKernelGGL(k_step_advance, dim3(1), dim3(1), 0, s, ctr);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ force mesh read-out
__global__ void k_split3(const float* __restrict__ f3, float* __restrict__ flat, int64_t M) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < M;
       i += (int64_t)gridDim.x * blockDim.x) {
    flat[i] = f3[3 * i];
    flat[M + i] = f3[3 * i + 1];
    flat[2 * M + i] = f3[3 * i + 2];
  }
}

void launch_split3(const Layout& L, const float* f3, float* flat, hipStream_t s) {
  ProfScope ps("split3", s);
  hipLaunchKernelGGL(k_split3, dim3(grid_for(L.M, 256)), dim3(256), 0, s, f3, flat, L.M);
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ 2LPT source pieces
// d0 <- d0 d1 + d0 d2 + d1 d2 ;  acc <- acc - x^2 - y^2 - z^2, in that order
// (S = sum_{i<j} phi_ii phi_jj - phi_ij^2).  Bound by memory; the three squares in one pass
// instead of one each (384^3: 3 x 151 -> 232 us, 1.13 GB), four values a thread.
__global__ void __launch_bounds__(256)
k_2lpt_diag(quad_t* __restrict__ d0, const quad_t* __restrict__ d1, const quad_t* __restrict__ d2,
            int64_t n4) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x) {
    const quad_t a = d0[i], b = d1[i], c = d2[i];
    quad_t o;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = a[k] * b[k] + a[k] * c[k] + b[k] * c[k];
    d0[i] = o;
  }
}
__global__ void __launch_bounds__(256)
k_2lpt_sub(quad_t* __restrict__ acc, const quad_t* __restrict__ x, const quad_t* __restrict__ y,
           const quad_t* __restrict__ z, int64_t n4) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x) {
    const quad_t a = x[i], b = y[i], c = z[i];
    quad_t o = acc[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      o[k] -= a[k] * a[k];
      o[k] -= b[k] * b[k];
      o[k] -= c[k] * c[k];
    }
    acc[i] = o;
  }
}
// n: a whole padded field, rows of a multiple of four values
void launch_2lpt_diag(float* d0, const float* d1, const float* d2, size_t n, hipStream_t s) {
  ProfScope ps("2lpt_source", s);
  hipLaunchKernelGGL(k_2lpt_diag, dim3(grid_for(n / 4, 256)), dim3(256), 0, s, (quad_t*)d0,
                     (const quad_t*)d1, (const quad_t*)d2, (int64_t)(n / 4));
  COLA_LAUNCH_CHECK();
}
void launch_2lpt_sub(float* acc, const float* x, const float* y, const float* z, size_t n, hipStream_t s) {
  ProfScope ps("2lpt_source", s);
  hipLaunchKernelGGL(k_2lpt_sub, dim3(grid_for(n / 4, 256)), dim3(256), 0, s, (quad_t*)acc,
                     (const quad_t*)x, (const quad_t*)y, (const quad_t*)z, (int64_t)(n / 4));
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ layout copies
__global__ void k_unpad3(const float* __restrict__ a0, const float* __restrict__ a1,
                         const float* __restrict__ a2, const float* __restrict__ b0,
                         const float* __restrict__ b1, const float* __restrict__ b2, float alpha,
                         float beta, float* __restrict__ out, int64_t N, int np, int ppitch,
                         int64_t pplane) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < N;
       p += (int64_t)gridDim.x * blockDim.x) {
    const int ip = (int)p;
    const int64_t q = (int64_t)(ip / (np * np)) * pplane + (int64_t)((ip / np) % np) * ppitch + ip % np;
    float x = alpha * a0[q], y = alpha * a1[q], z = alpha * a2[q];
    if (b0) {
      x += beta * b0[q];
      y += beta * b1[q];
      z += beta * b2[q];
    }
    out[p] = x;
    out[N + p] = y;
    out[2 * N + p] = z;
  }
}

void launch_unpad3(const Layout& L, const float* const f0[3], const float* const f1[3], float alpha,
                   float beta, float* out, hipStream_t s) {
  ProfScope ps("unpad", s);
  hipLaunchKernelGGL(k_unpad3, dim3(grid_for(L.N, 256)), dim3(256), 0, s, f0[0], f0[1], f0[2],
                     f1 ? f1[0] : nullptr, f1 ? f1[1] : nullptr, f1 ? f1[2] : nullptr, alpha, beta,
                     out, L.N, L.np, 2 * L.pitch_p, 2 * L.plane_p);
  COLA_LAUNCH_CHECK();
}

// u = D1(a_0) Psi1 + D2(a_0) Psi2 with the growth factors read from table slice 0
__global__ void k_combine_u0(const float* __restrict__ psi1, const float* __restrict__ psi2,
                             const double* __restrict__ t0, float* __restrict__ disp, int64_t n3) {
  const float c1 = (float)t0[0], c2 = (float)t0[3];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n3;
       i += (int64_t)gridDim.x * blockDim.x)
    disp[i] = c1 * psi1[i] + c2 * psi2[i];
}

void launch_combine_u0(const Layout& L, const float* psi1, const float* psi2, const double* table,
                       float* disp, hipStream_t s) {
  ProfScope ps("combine_u0", s);
  hipLaunchKernelGGL(k_combine_u0, dim3(grid_for(3 * L.N, 256)), dim3(256), 0, s, psi1, psi2, table,
                     disp, 3 * L.N);
  COLA_LAUNCH_CHECK();
}

// Bound by memory: 384^3 cells 69 us (454 MB, partly from the last-level cache), with two
// 64-bit divisions a cell 166.
__global__ void __launch_bounds__(256)
k_unpad_mesh(const float* __restrict__ in, float* __restrict__ out, int n, int rpitch,
             int64_t rplane, float sub) {
  CellQuad c;
  if (!cell_quad(n, rpitch, rplane, c)) return;
  const quad_t v = *reinterpret_cast<const quad_t*>(in + c.pe);
  *reinterpret_cast<quad_t*>(out + c.e) = v - sub;
}

void launch_unpad_mesh(const Layout& L, const float* padded, float* flat, hipStream_t s, float sub) {
  ProfScope ps("unpad_mesh", s);
  hipLaunchKernelGGL(k_unpad_mesh, quad_grid(L.nm), dim3(256), 0, s, padded, flat, L.nm,
                     2 * L.pitch_m, 2 * L.plane_m, sub);
  COLA_LAUNCH_CHECK();
}

// x = (q + u) mod L
__global__ void k_positions(const float* __restrict__ disp, float* __restrict__ xyz, int64_t N,
                            int np, int nm, int ratio, float inv_cell, float cell) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < N;
       p += (int64_t)gridDim.x * blockDim.x) {
    const int ip = (int)p;
    const int ix[3] = {ip / (np * np), (ip / np) % np, ip % np};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float f = 0.5f + disp[a * N + p] * inv_cell;
      const float fl = floorf(f);
      int i = (ix[a] * ratio + (int)fl) % nm;
      if (i < 0) i += nm;
      xyz[a * N + p] = ((float)i + (f - fl)) * cell;
    }
  }
}

void launch_positions(const cola_params& p, const Layout& L, const float* disp, float* xyz,
                      hipStream_t s) {
  ProfScope ps("positions", s);
  hipLaunchKernelGGL(k_positions, dim3(grid_for(L.N, 256)), dim3(256), 0, s, disp, xyz, L.N, L.np,
                     L.nm, L.nm / L.np, L.inv_cell, (float)(p.box / p.nmesh1d));
  COLA_LAUNCH_CHECK();
}

// ------------------------------------------------------------------ power spectrum
__device__ __forceinline__ float sincf_pi(float x) {   // sin(pi x)/(pi x)
  return x == 0.f ? 1.f : sinpif(x) / (3.14159265358979323846f * x);
}

constexpr int kPkMaxBins = 2048;
constexpr int kPkModeBlocks = 512;

// What the shells hold apart from the field: the mode counts and the sums of |k|, and the
// CIC window per axis, wtab[|nu|] = sinc(nu / n).  Both sums depend on |nu_x|, |nu_y| and
// nu_z alone, so one wave takes a row of nu_z for each unordered pair (|nu_x|, |nu_y|) with its
// multiplicity, an eighth of the modes, instead of two LDS atomics for every mode of the
// field (a mode's |k| term is formed in FP32 and summed in FP64, exactly as if each mode
// added its own).  Bound by its LDS atomics: 146 us at n = 1024.
__global__ void __launch_bounds__(256)
k_pk_modes(int n, int nbins, float kf, float* __restrict__ wtab, double* __restrict__ part_k,
           unsigned* __restrict__ part_w) {
  __shared__ double sk[kPkMaxBins];
  __shared__ unsigned sw[kPkMaxBins];
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
    sk[b] = 0.0;
    sw[b] = 0u;
  }
  __syncthreads();
  const int h = n / 2;
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= h; i += blockDim.x) wtab[i] = sincf_pi((float)i / n);
  const int rows = (h + 1) * (h + 2) / 2, waves = gridDim.x * (blockDim.x >> 6);
  for (int r = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); r < rows; r += waves) {
    int a = (int)((sqrtf(8.f * (float)r + 1.f) - 1.f) * 0.5f);   // row r = a (a + 1)/2 + b, b <= a
    while (a * (a + 1) / 2 > r) --a;
    while ((a + 1) * (a + 2) / 2 <= r) ++a;
    const int b = r - a * (a + 1) / 2;
    const unsigned mult = (a == 0 || a == h ? 1u : 2u) * (b == 0 || b == h ? 1u : 2u) * (a != b ? 2u : 1u);
    for (int iz = threadIdx.x & 63; iz <= h; iz += 64) {
      const int n2 = a * a + b * b + iz * iz;
      const int bin = shell_of(n2);
      if (n2 == 0 || bin >= nbins) continue;
      const unsigned w = (iz > 0 && iz < h) ? 2u : 1u;
      atomicAdd(&sk[bin], (double)mult * (double)((float)w * kf * sqrtf((float)n2)));
      atomicAdd(&sw[bin], mult * w);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
    part_k[(int64_t)blockIdx.x * nbins + b] = sk[b];
    part_w[(int64_t)blockIdx.x * nbins + b] = sw[b];
  }
}

// Cross-block reduction per bin in FP64: kPkSeg threads share a bin, each adding every
// kPkSeg-th block with Neumaier compensation, and the first adds their sums in order (a
// fixed order for a given grid); each sum leaves as an FP32 pair hi + lo.  One thread a bin
// walking all blocks took 316 us (512 bins, 1024 blocks: 425 us), this takes 12.
constexpr int kPkSeg = 32;
__global__ void __launch_bounds__(8 * kPkSeg)
k_pk_final(const double* __restrict__ part_p, int nblk_p, const double* __restrict__ part_k,
           const unsigned* __restrict__ part_w, int nblk_k, int nbins, float4* __restrict__ out,
           unsigned long long* __restrict__ counts) {
  __shared__ double rs[2][kPkSeg][8], rc[2][kPkSeg][8];
  __shared__ unsigned long long rw[kPkSeg][8];
  const int lb = threadIdx.x & 7, seg = threadIdx.x >> 3, b = blockIdx.x * 8 + lb;
  auto add = [](double& s, double& c, double x) {
    const double t = s + x;
    c += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
    s = t;
  };
  auto sum = [&](const double* part, int nblk, int which) {
    double s = 0.0, c = 0.0;
    if (b < nbins)
#pragma unroll 8
      for (int i = seg; i < nblk; i += kPkSeg) add(s, c, part[(int64_t)i * nbins + b]);
    rs[which][seg][lb] = s;
    rc[which][seg][lb] = c;
  };
  sum(part_p, nblk_p, 0);
  sum(part_k, nblk_k, 1);
  unsigned long long w = 0;
  if (b < nbins)
#pragma unroll 8
    for (int i = seg; i < nblk_k; i += kPkSeg) w += part_w[(int64_t)i * nbins + b];
  rw[seg][lb] = w;
  __syncthreads();
  if (seg != 0 || b >= nbins) return;
  double v[2];
  for (int q = 0; q < 2; ++q) {
    double s = 0.0, c = 0.0;
    for (int i = 0; i < kPkSeg; ++i) {
      add(s, c, rs[q][i][lb]);
      c += rc[q][i][lb];
    }
    v[q] = s + c;
  }
  for (int i = 1; i < kPkSeg; ++i) w += rw[i][lb];
  const float ph = (float)v[0], kh = (float)v[1];
  out[b] = make_float4(ph, (float)(v[0] - (double)ph), kh, (float)(v[1] - (double)kh));
  counts[b] = w;
}

// scratch: the field's partial sums (at most kPkBlocks rows of nbins), then the modes' (|k|,
// then counts) and the window table
size_t pk_scratch_bytes(const Layout& L, int nbins) {
  return align_up((size_t)nbins * (kPkBlocks * sizeof(double) + kPkModeBlocks * (sizeof(double) + sizeof(unsigned))) +
                  (size_t)(L.nm / 2 + 1) * sizeof(float));
}

void launch_pk(const Layout& L, const FFTPlan& pl, const float2* dk, int nbins, void* scratch, float4* out,
               unsigned long long* counts, hipStream_t s) {
  if (nbins > kPkMaxBins) throw Error{COLA_E_ARG, "nbins exceeds 2048"};
  double* part_p = static_cast<double*>(scratch);
  double* part_k = part_p + (size_t)kPkBlocks * nbins;
  unsigned* part_w = reinterpret_cast<unsigned*>(part_k + (size_t)kPkModeBlocks * nbins);
  float* wtab = reinterpret_cast<float*>(part_w + (size_t)kPkModeBlocks * nbins);
  const float kf = (float)(2.0 * M_PI / L.box);
  const int h = L.nm / 2, rows = (h + 1) * (h + 2) / 2;
  const int mode_blocks = std::min(kPkModeBlocks, (rows + 7) / 8);   // two rows a wave or more
  {
    ProfScope ps("pk_modes", s);
    hipLaunchKernelGGL(k_pk_modes, dim3(mode_blocks), dim3(256), 0, s, L.nm, nbins, kf, wtab, part_k,
                       part_w);
    COLA_LAUNCH_CHECK();
  }
  PkBin a;
  a.pitch = L.pitch_m;
  a.nbins = nbins;
  a.vol = (float)(L.box * L.box * L.box);
  a.wtab = wtab;
  a.part = part_p;
  const int nblk = fft_x_pk(pl, dk, a, s);
  ProfScope ps("pk_final", s);
  hipLaunchKernelGGL(k_pk_final, dim3((nbins + 7) / 8), dim3(8 * kPkSeg), 0, s, part_p, nblk, part_k, part_w,
                     mode_blocks, nbins, out, counts);
  COLA_LAUNCH_CHECK();
}

}  // namespace cola
