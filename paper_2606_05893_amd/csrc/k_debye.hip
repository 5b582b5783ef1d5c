// Resolution check of the grid against the Debye length of the electrons and
// ions (the mesh criterion of the paper's appendix: d_max = 3.4 lambda_D
// alpha_D), per block of b^3 cells.
//
// A workgroup takes a tile of 8^3 cells at a time, which holds whole blocks
// (block divides 8): it streams the tile's binned electrons and ions once, sums
// the moments (count, sum of v, sum of |v|^2) per cell in LDS, joins the cells
// of a block, and forms lambda_D and the criterion there; with one block a tile
// a wave sums it in registers.  Nothing but lambda_D is written.  The
// workgroups' runs of tiles hold as many particles each.
//
// Two kinds of particles go to a global record per block first, cleared where
// there are any and added in by the workgroup of the tile: the ions outside their
// tile (the unbinned tail, and ions that crossed a tile face since the last
// binning), and those of crowded tiles, which many workgroups share, a chunk of
// the push at a time.
//
// Bound: the LDS adds (four FP64 and a count per particle) beside the 48 bytes
// (28 mixed) read per particle.  A check of 10 M electrons and 10 M ions on
// 128x128x512 cells, just binned: 231 us for blocks of 1, 114 for blocks of 8
// (24 bytes read per particle); after steps, which leave some thousand ions
// outside their tiles, 60 more.  All of them in the lowest eighth of the box 235
// and 160, in a 64x64x16 corner 830 and 252; 4 M in one tile of 64^3 cells 505 and
// 129.  (Summing each 2048 particles in a hash table and adding every entry to
// its block's record: 3230 and 630, 1600 and 630, 1510 and 630, 900 and 205.  Equal
// runs of tiles and no crowded ones: 232 and 270, 890 and 930, 5180 and 5200,
// 10300.)
#include <algorithm>
#include <cmath>

#include "pic_ctx.h"

namespace pic {
namespace {

constexpr int kT = 256;
constexpr int kMom = 5;                 // count, sum vx, vy, vz, sum |v|^2
constexpr int kFinBlocks = kRuns;
constexpr int kCells = kTile * kTile * kTile;
// A tile's clearing and finishing in particles' time.
constexpr unsigned kTileCost = 256;

struct BlockGeo {
  int b, bx, by;                        // block edge (cells), blocks per axis
};

__device__ __forceinline__ unsigned block_of(int i, int j, int k,
                                             const BlockGeo& q) {
  return ((unsigned)(k / q.b) * (unsigned)q.by + (unsigned)(j / q.b)) *
             (unsigned)q.bx + (unsigned)(i / q.b);
}

__device__ __forceinline__ void cell_ijk(const Parts& p, long long n,
                                         const GridC& g, int& i, int& j,
                                         int& k) {
  i = (int)floor(p.x[n] * g.inv_dx);
  j = (int)floor(p.y[n] * g.inv_dx);
  k = (int)floor(p.z[n] * g.inv_dx);
  if (i >= g.nx) i -= g.nx;
  if (j >= g.ny) j -= g.ny;
}

__device__ __forceinline__ void cell_ijk(const PartsM& p, long long n,
                                         const GridC& g, int& i, int& j,
                                         int& k) {
  Acc<PartsM>::decode(p.cell[n], g, i, j, k);
}

struct DebyeC {
  double mass[2];        // electron, Cu+ ion
  double w, vol;         // superparticle weight, block volume (b dx)^3
  double e2, eps0, dx, dmax_per_lambda;
};

// lambda_D of a block from its moments (count, sums of v, sum of |v|^2 of
// electrons and ions), tallied.
struct DebyeTally {
  long long checked = 0, unres = 0;
  double lmin = INFINITY, rmax = 0.0;
};

__device__ __forceinline__ double block_lambda(const double (&mom)[2][kMom], const DebyeC& d,
                                               DebyeTally& y) {
  double inv_l2 = 0.0;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const double* r = mom[s];
    const double N = r[0];
    if (!(N >= 2.0)) continue;
    const double sx = r[1], sy = r[2], sz = r[3];
    const double ss = r[4] - ((sx * sx + sy * sy) + sz * sz) / N;
    const double kT_s = (d.mass[s] * ss) / (3.0 * (N - 1.0));
    if (!(kT_s > 0.0)) continue;
    const double n = (N * d.w) / d.vol;
    inv_l2 = inv_l2 + (n * d.e2) / (d.eps0 * kT_s);
  }
  if (!(inv_l2 > 0.0)) return INFINITY;
  const double lam = 1.0 / sqrt(inv_l2);
  const double ratio = d.dx / (d.dmax_per_lambda * lam);
  y.checked += 1;
  if (ratio > 1.0) y.unres += 1;
  y.lmin = fmin(y.lmin, lam);
  y.rmax = fmax(y.rmax, ratio);
  return lam;
}

// The workgroup's tally into its partials, through 4 kT words of LDS.
__device__ __forceinline__ void tally_out(double* lds, const DebyeTally& y,
                                          long long* __restrict__ qpart,
                                          double* __restrict__ part) {
  long long* sc = reinterpret_cast<long long*>(lds);
  long long* su = sc + kT;
  double* smin = lds + 2 * kT;
  double* smax = lds + 3 * kT;
  sc[threadIdx.x] = y.checked;
  su[threadIdx.x] = y.unres;
  smin[threadIdx.x] = y.lmin;
  smax[threadIdx.x] = y.rmax;
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sc[threadIdx.x] += sc[threadIdx.x + o];
      su[threadIdx.x] += su[threadIdx.x + o];
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + o]);
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    qpart[2 * blockIdx.x] = sc[0];
    qpart[2 * blockIdx.x + 1] = su[0];
    part[2 * blockIdx.x] = smin[0];
    part[2 * blockIdx.x + 1] = smax[0];
  }
}

__device__ __forceinline__ unsigned tile_of(int i, int j, int k, const GridC& g) {
  return ((unsigned)(k / kTile) * g.tny + j / kTile) * g.tnx + i / kTile;
}

// The tiles' particles in the chunks of the push: (tile, piece k) covers up to
// kPushChunk of its electrons and of its ions.
struct Chunks {
  const uint32_t* ts[2];                // tile starts: electrons, ions
  const uint2* chunks;
  const unsigned* cstart;               // a tile's first chunk
  unsigned nt;
  unsigned most;                        // chunks of a tile that is not crowded
  bool uneven;                          // equal runs of tiles are not equal work
  __device__ unsigned total() const { return cstart[nt]; }
  __device__ void range(int s, unsigned t, unsigned k, long long& a, long long& b) const {
    a = ts[s][t] + (long long)k * kPushChunk;
    b = ts[s][t + 1];
    if (a > b) a = b;
    if (b - a > kPushChunk) b = a + kPushChunk;
  }
  __device__ bool crowded(unsigned t) const { return cstart[t + 1] - cstart[t] > most; }
};

// The ions outside their tile, found in one pass over the positions: their blocks
// get a bit, their blocks' ion records are cleared and they go to a list, whose
// moments k_debye_add puts in the records.  Workgroup c < nchb scans the binned
// ions of chunk c (if there is one), the others the tail.
struct Strays {
  uint32_t* bits;                       // a bit per block (null: no ion is outside)
  Rec* list;                            // block, ion
  unsigned long long* n;
  unsigned long long cap;               // (never reached: stray_cap)
  __device__ bool has(long long r) const { return bits && (bits[r >> 5] >> (r & 31) & 1u); }
};

__global__ void k_debye_none(Strays S, long long blocks) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *S.n = 0;
  const long long words = (blocks + 31) / 32;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < words;
       i += (long long)gridDim.x * blockDim.x)
    S.bits[i] = 0u;
}

template <class PT>
__global__ void __launch_bounds__(kT) k_debye_find(PT p, long long n, long long n_binned, Chunks C,
                                                   unsigned nchb, GridC g, BlockGeo q, Strays S,
                                                   double* __restrict__ mom) {
  long long a, b, step = kT;
  unsigned own = 0xFFFFFFFFu;
  if (blockIdx.x < nchb) {
    if (blockIdx.x >= C.total()) return;
    own = C.chunks[blockIdx.x].x;
    C.range(1, own, C.chunks[blockIdx.x].y, a, b);
  } else {
    a = n_binned + (long long)(blockIdx.x - nchb) * kT;
    b = n;
    step = (long long)(gridDim.x - nchb) * kT;
  }
  for (long long idx = a + threadIdx.x; idx < b; idx += step) {
    int i, j, k;
    cell_ijk(p, idx, g, i, j, k);
    if (tile_of(i, j, k, g) == own) continue;
    const unsigned r = block_of(i, j, k, q);
    atomicOr(&S.bits[r >> 5], 1u << (r & 31));
    for (int m = kMom; m < 2 * kMom; ++m) mom[(size_t)r * (2 * kMom) + m] = 0.0;
    Rec x;
    x.lo = r;
    x.hi = 0u;
    x.val = (unsigned)idx;
    const unsigned long long slot = atomicAdd(S.n, 1ull);
    if (slot < S.cap) S.list[slot] = x;
  }
}

template <class PT>
__global__ void __launch_bounds__(kT) k_debye_add(PT p, Strays S, double* __restrict__ mom) {
  const long long n = (long long)min(*S.n, S.cap);
  for (long long x = blockIdx.x * (long long)kT + threadIdx.x; x < n;
       x += (long long)gridDim.x * kT) {
    const Rec y = S.list[x];
    double vx, vy, vz;
    Acc<PT>::vel(p, y.val, vx, vy, vz);
    double* rec = mom + (size_t)y.lo * (2 * kMom) + kMom;
    atomicAdd(rec + 0, 1.0);
    atomicAdd(rec + 1, vx);
    atomicAdd(rec + 2, vy);
    atomicAdd(rec + 3, vz);
    atomicAdd(rec + 4, (vx * vx + vy * vy) + vz * vz);
  }
}

// A tile: its first cell, and its blocks (edge 1 << LGB): block(bl) is block bl
// of it, or -1 where the grid ends inside the tile.
template <int LGB>
struct TileGeo {
  int x, y, z;
  __device__ TileGeo(unsigned t, const GridC& g) {
    const unsigned r = t / (unsigned)g.tnx;
    x = (int)(t % (unsigned)g.tnx) * kTile;
    y = (int)(r % (unsigned)g.tny) * kTile;
    z = (int)(r / (unsigned)g.tny) * kTile;
  }
  __device__ __forceinline__ long long block(int bl, const GridC& g, const BlockGeo& q) const {
    constexpr int le = 3 - LGB, m = (1 << le) - 1;   // (kTile = 8)
    const int bx = (x >> LGB) + (bl & m), by = (y >> LGB) + ((bl >> le) & m),
              bz = (z >> LGB) + (bl >> (2 * le));
    if (bx << LGB >= g.nx || by << LGB >= g.ny || bz << LGB >= g.nz) return -1;
    return ((long long)bz * q.by + by) * q.bx + bx;
  }
};
static_assert(kTile == 8, "TileGeo::block");

// Clear the records of crowded tiles.
template <int LGB>
__global__ void __launch_bounds__(kT) k_debye_clear(Chunks C, GridC g, BlockGeo q,
                                                    double* __restrict__ mom) {
  for (unsigned t = blockIdx.x; t < C.nt; t += gridDim.x) {
    if (!C.crowded(t)) continue;
    const TileGeo<LGB> o(t, g);
    for (int bl = threadIdx.x; bl < kCells >> (3 * LGB); bl += kT) {
      const long long r = o.block(bl, g, q);
      if (r < 0) continue;
      for (int m = 0; m < 2 * kMom; ++m) mom[r * (2 * kMom) + m] = 0.0;
    }
  }
}

// A block's record, of its ions alone where no electron is in it, and its sums.
__device__ __forceinline__ void record_read(const double* __restrict__ mom, long long r, bool ions,
                                            double (&mo)[2][kMom]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (s || !ions)
#pragma unroll
    for (int m = 0; m < kMom; ++m) mo[s][m] += mom[r * (2 * kMom) + s * kMom + m];
}
__device__ __forceinline__ void record_add(double* __restrict__ mom, long long r,
                                           const double (&mo)[2][kMom]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
    if (mo[s][0] > 0.0)
#pragma unroll
      for (int m = 0; m < kMom; ++m) atomicAdd(&mom[r * (2 * kMom) + s * kMom + m], mo[s][m]);
}

// ---- blocks of 1, 2 and 4 cells ----------------------------------------------
// A tile's moments in LDS, per cell with those of a block side by side, or where
// a tile has few particles (kFew) per block.
struct TileMom {
  double v[2][4][kCells];
  unsigned n[2][kCells];
};
constexpr unsigned kFew = 1024;

__device__ __forceinline__ void tile_clear(TileMom& L, int places) {
  for (int c = threadIdx.x; c < places; c += kT)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      L.n[s][c] = 0u;
#pragma unroll
      for (int m = 0; m < 4; ++m) L.v[s][m][c] = 0.0;
    }
}

// Particles [a, b) of species s, those inside the tile.
template <int LGB, class PT>
__device__ __forceinline__ void tile_add(TileMom& L, const PT& p, int s, long long a, long long b,
                                         bool few, const TileGeo<LGB>& o, const GridC& g) {
  constexpr int e = kTile >> LGB, w = (1 << LGB) - 1;
  for (long long idx = a + threadIdx.x; idx < b; idx += kT) {
    int i, j, k;
    cell_ijk(p, idx, g, i, j, k);
    double vx, vy, vz;
    Acc<PT>::vel(p, idx, vx, vy, vz);
    i -= o.x;
    j -= o.y;
    k -= o.z;
    // An ion that left its tile is in its block's record.
    if ((unsigned)i >= kTile || (unsigned)j >= kTile || (unsigned)k >= kTile) continue;
    int c = ((k >> LGB) * e + (j >> LGB)) * e + (i >> LGB);
    if (LGB > 0 && !few) c = (((c << LGB | (k & w)) << LGB | (j & w)) << LGB) | (i & w);
    atomicAdd(&L.n[s][c], 1u);
    atomicAdd(&L.v[s][0][c], vx);
    atomicAdd(&L.v[s][1][c], vy);
    atomicAdd(&L.v[s][2][c], vz);
    atomicAdd(&L.v[s][3][c], (vx * vx + vy * vy) + vz * vz);
  }
}

// The tile's sums, each block's passed once to f(block of the tile, moments); all
// threads call it, the sums are consumed.
template <int LGB, class F>
__device__ __forceinline__ void tile_join(TileMom& L, bool few, F f) {
  constexpr int kLgc = 3 * LGB, kNb = kCells >> kLgc;
  if (LGB == 0 || few) {
    for (int c = threadIdx.x; c < kNb; c += kT) {
      double mo[2][kMom];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        mo[s][0] = (double)L.n[s][c];
#pragma unroll
        for (int m = 0; m < 4; ++m) mo[s][m + 1] = L.v[s][m][c];
      }
      f(c, mo);
    }
    __syncthreads();
    return;
  }
  // 2 kMom sums a block over its cells, by one thread each (two for blocks of 4;
  // the cells' order turned by the block, so that the threads of a wave meet
  // other banks), left in LDS for one thread a block.  (Every thread with all the
  // sums of two cells, and then rounds of shuffles: 256 us at 128x128x512 for
  // blocks of 4.)
  constexpr int kLgp = LGB == 2 ? 1 : 0, kSums = 2 * kMom * kNb;
  constexpr int kRounds = ((kSums << kLgp) + kT - 1) / kT;
  double r[kRounds];
#pragma unroll
  for (int z = 0; z < kRounds; ++z) {
    const int x = (z * kT + (int)threadIdx.x) >> kLgp;
    r[z] = 0.0;
    if (x < kSums) {
      const int bl = x & (kNb - 1), m = x / kNb, sp = m >= kMom ? 1 : 0, q = m - sp * kMom;
      constexpr int per = 1 << (kLgc - kLgp);
      const int at = (bl << kLgc) + (threadIdx.x & ((1 << kLgp) - 1));
#pragma unroll 4
      for (int k = 0; k < per; ++k) {
        const int c = at + (((k + bl) & (per - 1)) << kLgp);
        r[z] += q == 0 ? (double)L.n[sp][c] : L.v[sp][q - 1][c];
      }
    }
    if (kLgp) r[z] += __shfl_down(r[z], 1);
  }
  __syncthreads();
  double* w = &L.v[0][0][0];
#pragma unroll
  for (int z = 0; z < kRounds; ++z) {
    const int x = (z * kT + (int)threadIdx.x) >> kLgp;
    if (x < kSums && (threadIdx.x & ((1 << kLgp) - 1)) == 0) w[x] = r[z];
  }
  __syncthreads();
  if (threadIdx.x < kNb) {
    double mo[2][kMom];
#pragma unroll
    for (int m = 0; m < 2 * kMom; ++m) mo[m / kMom][m % kMom] = w[m * kNb + threadIdx.x];
    f(threadIdx.x, mo);
  }
  __syncthreads();
}

// Crowded tiles: two chunks of one per workgroup at a time (one for blocks of
// more than a cell, whose records are few), their sums added to the records.
template <class PT, int LGB>
__global__ void __launch_bounds__(kT) k_debye_pieces(PT pe, PT pi, Chunks C, GridC g, BlockGeo q,
                                                     double* __restrict__ mom) {
  __shared__ TileMom L;
  constexpr unsigned kRun = LGB == 0 ? 2 : 1;
  const unsigned nch = C.total();
  for (unsigned c0 = blockIdx.x; c0 < nch; c0 += gridDim.x) {
    const unsigned t = C.chunks[c0].x;
    if (C.chunks[c0].y % kRun || !C.crowded(t)) continue;
    const unsigned end = min(c0 + kRun, C.cstart[t + 1]);
    const TileGeo<LGB> o(t, g);
    __syncthreads();
    tile_clear(L, kCells);
    __syncthreads();
    for (unsigned c = c0; c < end; ++c)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        long long a, b;
        C.range(s, t, C.chunks[c].y, a, b);
        tile_add(L, s ? pi : pe, s, a, b, false, o, g);
      }
    __syncthreads();
    tile_join<LGB>(L, false, [&](int bl, double (&mo)[2][kMom]) {
      const long long r = o.block(bl, g, q);
      if (r >= 0) record_add(mom, r, mo);
    });
  }
}

// The first tile whose particles, with those of the tiles before it and
// kTileCost a tile, reach target (nt: none); by the workgroup, 256 probes a
// round.
__device__ __forceinline__ unsigned long long tile_weight(const Chunks& C, unsigned t) {
  return (unsigned long long)C.ts[0][t] + C.ts[1][t] + (unsigned long long)kTileCost * t;
}
__device__ unsigned first_tile(const Chunks& C, unsigned long long target) {
  unsigned lo = 0, len = C.nt + 1;      // candidates; the last one holds
  while (len > 1) {
    const unsigned step = (len + kT - 1) / kT;
    const unsigned at = min((threadIdx.x + 1) * step, len) - 1;
    const unsigned c = (unsigned)__syncthreads_count(tile_weight(C, lo + at) < target);
    lo += c * step;
    len = min(step, len - c * step);
  }
  return lo;
}

// The workgroup's tiles, contiguous, one XCD's workgroups side by side: equal runs
// where these hold about as many particles, else runs of equal weight (one tile
// more than the mean is 6 % of 128x128x512 evenly filled cells).
__device__ __forceinline__ void tile_run(const Chunks& C, unsigned& t0, unsigned& t1) {
  const unsigned wg = xcd_block(blockIdx.x, gridDim.x);
  t0 = (unsigned)((unsigned long long)C.nt * wg / gridDim.x);
  t1 = (unsigned)((unsigned long long)C.nt * (wg + 1) / gridDim.x);
  if (C.uneven) {
    const unsigned long long all = tile_weight(C, C.nt);
    t0 = first_tile(C, all * wg / gridDim.x);
    t1 = first_tile(C, all * (wg + 1) / gridDim.x);
  }
}

// Tiles: their moments, and the records of crowded ones and of stray ions, to
// lambda_D.
template <class PT, int LGB>
__global__ void __launch_bounds__(kT) k_debye_tiles(
    PT pe, PT pi, Chunks C, GridC g, BlockGeo q, DebyeC d, Strays S,
    const double* __restrict__ mom, double* __restrict__ lam_out, long long* __restrict__ qpart,
    double* __restrict__ part) {
  __shared__ TileMom L;
  constexpr int kNb = kCells >> (3 * LGB);
  DebyeTally y;
  unsigned t0, t1;
  tile_run(C, t0, t1);
  // Starts of the tile's electrons, ions and chunks, the next tile's loaded a
  // tile ahead: whether and how to clear the sums depends on them.
  struct Starts {
    unsigned e, i, c;
  };
  auto starts = [&](unsigned t) {
    t = min(t, C.nt);
    return Starts{C.ts[0][t], C.ts[1][t], C.cstart[t]};
  };
  Starts a, b = starts(t0), next = starts(t0 + 1);
  for (unsigned t = t0; t < t1; ++t) {
    a = b;
    b = next;
    next = starts(t + 2);
    const bool pieces = b.c - a.c > C.most;
    const TileGeo<LGB> o(t, g);
    const unsigned n = pieces ? 0u : (b.e - a.e) + (b.i - a.i);
    auto finish = [&](int bl, double (&mo)[2][kMom]) {
      const long long r = o.block(bl, g, q);
      if (r < 0) return;
      if (pieces || S.has(r)) record_read(mom, r, !pieces, mo);
      const double lam = block_lambda(mo, d, y);
      if (lam_out) lam_out[r] = lam;
    };
    if (n == 0u) {
      for (int bl = threadIdx.x; (lam_out || S.bits || pieces) && bl < kNb; bl += kT) {
        double mo[2][kMom] = {};
        finish(bl, mo);
      }
      continue;
    }
    const bool few = LGB > 0 && n < kFew;
    tile_clear(L, few ? kNb : kCells);
    __syncthreads();
    tile_add(L, pe, 0, a.e, b.e, few, o, g);
    tile_add(L, pi, 1, a.i, b.i, few, o, g);
    __syncthreads();
    tile_join<LGB>(L, few, finish);
  }
  __syncthreads();
  tally_out(&L.v[0][0][0], y, qpart, part);
}

// ---- blocks of a whole tile ------------------------------------------------------
// No cells, so a wave sums a tile in registers and reads the velocities alone (the
// electrons lie in their tiles, the ions too unless some are strays): 114
// us at 128x128x512 against 268 through LDS.

// Sums of particles [a, b) (IN: those inside the tile) by a wave, a part per lane.
template <class PT, bool IN>
__device__ __forceinline__ void wave_add(double (&mo)[kMom], const PT& p, long long a, long long b,
                                         const TileGeo<3>& o, const GridC& g) {
  // Four at a time, all loads in flight before the first sum.
  constexpr int kN = 4;
  for (long long idx = a + (threadIdx.x & 63); idx < b; idx += 64 * kN) {
    double v[kN][3];
    bool in[kN];
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      const long long x = idx + 64 * u, at = x < b ? x : b - 1;
      Acc<PT>::vel(p, at, v[u][0], v[u][1], v[u][2]);
      in[u] = x < b;
      if (IN) {
        int i, j, k;
        cell_ijk(p, at, g, i, j, k);
        in[u] = in[u] && (unsigned)(i - o.x) < kTile && (unsigned)(j - o.y) < kTile &&
                (unsigned)(k - o.z) < kTile;
      }
    }
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      const double x = in[u] ? v[u][0] : 0.0, y = in[u] ? v[u][1] : 0.0, z = in[u] ? v[u][2] : 0.0;
      mo[0] += in[u] ? 1.0 : 0.0;
      mo[1] += x;
      mo[2] += y;
      mo[3] += z;
      mo[4] += (x * x + y * y) + z * z;
    }
  }
}

template <class PT>
__device__ __forceinline__ void wave_sums(double (&mo)[2][kMom], const PT& pe, const PT& pi,
                                          long long ae, long long be, long long ai, long long bi,
                                          bool strays, const TileGeo<3>& o, const GridC& g) {
  wave_add<PT, false>(mo[0], pe, ae, be, o, g);
  if (strays)
    wave_add<PT, true>(mo[1], pi, ai, bi, o, g);
  else
    wave_add<PT, false>(mo[1], pi, ai, bi, o, g);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int m = 0; m < kMom; ++m)
      for (int x = 32; x > 0; x >>= 1) mo[s][m] += __shfl_down(mo[s][m], x);
}

// Crowded tiles, a chunk per wave.
template <class PT>
__global__ void __launch_bounds__(kT) k_debye_whole_pieces(PT pe, PT pi, Chunks C, GridC g,
                                                           BlockGeo q, bool strays,
                                                           double* __restrict__ mom) {
  const unsigned nch = C.total(), nw = gridDim.x * (kT / 64);
  for (unsigned c = blockIdx.x * (kT / 64) + threadIdx.x / 64; c < nch; c += nw) {
    const unsigned t = C.chunks[c].x;
    if (!C.crowded(t)) continue;
    const TileGeo<3> o(t, g);
    long long ae, be, ai, bi;
    C.range(0, t, C.chunks[c].y, ae, be);
    C.range(1, t, C.chunks[c].y, ai, bi);
    double mo[2][kMom] = {};
    wave_sums(mo, pe, pi, ae, be, ai, bi, strays, o, g);
    if ((threadIdx.x & 63) == 0) record_add(mom, o.block(0, g, q), mo);
  }
}

template <class PT>
__global__ void __launch_bounds__(kT) k_debye_whole(
    PT pe, PT pi, Chunks C, GridC g, BlockGeo q, DebyeC d, Strays S,
    const double* __restrict__ mom, double* __restrict__ lam_out, long long* __restrict__ qpart,
    double* __restrict__ part) {
  __shared__ double lds[4 * kT];
  DebyeTally y;
  unsigned t0, t1;
  tile_run(C, t0, t1);
  for (unsigned t = t0 + threadIdx.x / 64; t < t1; t += kT / 64) {
    const TileGeo<3> o(t, g);
    const bool pieces = C.crowded(t);
    double mo[2][kMom] = {};
    if (!pieces)
      wave_sums(mo, pe, pi, C.ts[0][t], C.ts[0][t + 1], C.ts[1][t], C.ts[1][t + 1],
                S.bits != nullptr, o, g);
    if (threadIdx.x & 63) continue;
    const long long r = o.block(0, g, q);
    if (pieces || S.has(r)) record_read(mom, r, !pieces, mo);
    const double lam = block_lambda(mo, d, y);
    if (lam_out) lam_out[r] = lam;
  }
  tally_out(lds, y, qpart, part);
}

// Fixed-order sum / min / max of the block partials into out[0..3]:
// checked, unresolved (as doubles, exact below 2^53), lambda_min, ratio_max.
__global__ void __launch_bounds__(1024) k_debye_reduce(
    const long long* __restrict__ qpart, const double* __restrict__ part,
    int nblk, double* __restrict__ out) {
  __shared__ long long sc[1024], su[1024];
  __shared__ double smin[1024], smax[1024];
  long long c = 0, u = 0;
  double lmin = INFINITY, rmax = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
    c += qpart[2 * i];
    u += qpart[2 * i + 1];
    lmin = fmin(lmin, part[2 * i]);
    rmax = fmax(rmax, part[2 * i + 1]);
  }
  sc[threadIdx.x] = c;
  su[threadIdx.x] = u;
  smin[threadIdx.x] = lmin;
  smax[threadIdx.x] = rmax;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sc[threadIdx.x] += sc[threadIdx.x + o];
      su[threadIdx.x] += su[threadIdx.x + o];
      smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + o]);
      smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = (double)sc[0];
    out[1] = (double)su[0];
    out[2] = smin[0];
    out[3] = smax[0];
  }
}

template <class PT>
PT species_arrays(pic_ctx* c, int s);
template <>
Parts species_arrays<Parts>(pic_ctx* c, int s) { return c->P[s][c->cur[s]]; }
template <>
PartsM species_arrays<PartsM>(pic_ctx* c, int s) { return c->PM[s][c->cur[s]]; }

template <class PT, int LGB>
void tiles(pic_ctx* c, const BlockGeo& q, const DebyeC& d, double* lam_out) {
  const unsigned nt = (unsigned)c->ntiles;
  const ChunkSpread& sp = parts_spread(c);
  // A tile is crowded when one workgroup (a wave, for whole tiles) to itself
  // would be the last to end: a workgroup reads 400 particles a microsecond and a
  // chunk has up to 4096.  Records of single cells are many, so there more are
  // left to a tile's workgroup.
  const long long fair = LGB == 3 ? std::min(4ll, std::max(1ll, sp.chunks / 2048))
                                  : std::min(8ll, std::max(LGB ? 2ll : 4ll, sp.chunks / 512));
  const Chunks C{{c->tsb[0][c->tcur[0]], c->tsb[2][c->tcur[2]]}, c->chunks, c->cstart, nt,
                 (unsigned)fair, sp.uneven};
  const PT pe = species_arrays<PT>(c, 0), pi = species_arrays<PT>(c, 2);
  const bool crowd = sp.most > fair;
  // The electrons are binned every step.
  const long long tail = c->n[2] - c->n_binned[2];
  const bool strays = tail > 0 || c->ion_moved_accum > 0;
  hipStream_t st = c->stream;
  Strays S{nullptr, c->dbg_list, &c->dc->n_stray,
           (unsigned long long)stray_cap(c->cfg.capacity[2])};
  if (crowd) k_debye_clear<LGB><<<std::min(nt, 1024u), kT, 0, st>>>(C, c->g, q, c->dbg_mom);
  if (strays) {
    S.bits = c->dbg_bits;
    const unsigned nchb = (unsigned)c->nch_bound;
    const unsigned grid = nchb + (tail > 0 ? (unsigned)std::min(256ll, (tail + kT - 1) / kT) : 0u);
    k_debye_none<<<256, kT, 0, st>>>(S, c->ncells >> (3 * LGB));
    k_debye_find<PT><<<grid, kT, 0, st>>>(pi, c->n[2], c->n_binned[2], C, nchb, c->g, q, S,
                                          c->dbg_mom);
    k_debye_add<PT><<<256, kT, 0, st>>>(pi, S, c->dbg_mom);
  }
  if constexpr (LGB == 3) {
    if (crowd)
      k_debye_whole_pieces<PT><<<1024, kT, 0, st>>>(pe, pi, C, c->g, q, strays, c->dbg_mom);
    k_debye_whole<PT><<<kFinBlocks, kT, 0, st>>>(pe, pi, C, c->g, q, d, S, c->dbg_mom, lam_out,
                                                 c->dbg_qpart, c->dbg_part);
  } else {
    if (crowd) k_debye_pieces<PT, LGB><<<1024, kT, 0, st>>>(pe, pi, C, c->g, q, c->dbg_mom);
    k_debye_tiles<PT, LGB><<<kFinBlocks, kT, 0, st>>>(pe, pi, C, c->g, q, d, S, c->dbg_mom,
                                                      lam_out, c->dbg_qpart, c->dbg_part);
  }
}

template <int LGB>
void tiles_any(pic_ctx* c, const BlockGeo& q, const DebyeC& d, double* lam_out) {
  if (c->mixed)
    tiles<PartsM, LGB>(c, q, d, lam_out);
  else
    tiles<Parts, LGB>(c, q, d, lam_out);
}

}  // namespace

long long debye_moment_doubles(long long ncells) { return 2 * kMom * ncells; }

// Moments, lambda_D and the criterion; out[0..3] (device) receives checked,
// unresolved, lambda_min, ratio_max.
void parts_debye(pic_ctx* c, int block, double alpha_D, double* lam_out,
                 double* out) {
  BlockGeo q;
  q.b = block;
  q.bx = c->cfg.nx / block;
  q.by = c->cfg.ny / block;
  DebyeC d;
  d.mass[0] = kMe;
  d.mass[1] = kMcu;
  const double side = (double)block * c->g.dx;
  d.w = (double)c->cfg.w_sp;
  d.vol = (side * side) * side;
  d.e2 = kE * kE;
  d.eps0 = kEps0;
  d.dx = c->g.dx;
  d.dmax_per_lambda = 3.4 * alpha_D;
  if (block == 1)
    tiles_any<0>(c, q, d, lam_out);
  else if (block == 2)
    tiles_any<1>(c, q, d, lam_out);
  else if (block == 4)
    tiles_any<2>(c, q, d, lam_out);
  else
    tiles_any<3>(c, q, d, lam_out);
  k_debye_reduce<<<1, 1024, 0, c->stream>>>(c->dbg_qpart, c->dbg_part,
                                            kFinBlocks, out);
}

}  // namespace pic
