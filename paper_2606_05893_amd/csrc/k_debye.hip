// Resolution check of the grid against the Debye length of the electrons and
// ions (the mesh criterion of the paper's appendix: d_max = 3.4 lambda_D
// alpha_D), per block of b^3 cells.
//
// A workgroup takes a tile of 8^3 cells at a time, which holds whole blocks
// (block divides 8): it streams the tile's binned electrons and ions once, sums
// the moments (count, sum of v, sum of |v|^2) per cell in LDS, joins the cells
// of a block, and forms lambda_D and the criterion there.  Nothing but lambda_D
// is written.  Ions outside their tile (the unbinned tail, and ions that
// crossed a tile face since the last binning) are few: their moments go to a
// global record per block first, in the tiles they flag.
//
// Bound: the LDS adds (four FP64 and a count per particle) beside the 48 bytes
// (28 mixed) read per particle.  On 128x128x512 cells with 10 M electrons and 10
// M ions 246 us for blocks of 1 and of 8 (the read alone 190).  Summing each 2048 particles in a
// hash table and adding every entry to its block's 80-byte record took 3390 and
// 630 us: with blocks of one cell nearly every particle was its own global
// atomic, and the records were cleared, added to and read back.
//
// That form stays where tiles are crowded (more than kCrowded particles on
// average): there a tile per workgroup would leave the chip idle, and a
// workgroup's particles fall into few blocks.
#include <algorithm>
#include <cmath>

#include "pic_ctx.h"

namespace pic {
namespace {

constexpr int kT = 256;
constexpr int kPer = 8;                 // particles per thread
constexpr int kDChunk = kT * kPer;      // particles per workgroup
constexpr int kHash = 1024;             // LDS table entries
constexpr int kMom = 5;                 // count, sum vx, vy, vz, sum |v|^2
constexpr unsigned kEmpty = 0xFFFFFFFFu;
constexpr int kFinBlocks = 1024;
constexpr int kCells = kTile * kTile * kTile;
constexpr long long kCrowded = 8192;

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

// The ions outside their tile.  ADD = false: flag the tiles they are in; true:
// add their moments to their blocks' records.  Workgroup t < ntiles scans tile
// t's binned ions, the others the tail.
template <class PT, bool ADD>
__global__ void __launch_bounds__(kT) k_debye_strays(PT p, long long n, long long n_binned,
                                                     const uint32_t* __restrict__ ts, unsigned nt,
                                                     GridC g, BlockGeo q,
                                                     uint32_t* __restrict__ flag,
                                                     double* __restrict__ mom) {
  long long a, b, step = kT;
  unsigned own = 0xFFFFFFFFu;
  if (blockIdx.x < nt) {
    own = blockIdx.x;
    a = ts[own];
    b = ts[own + 1];
  } else {
    a = n_binned + (long long)(blockIdx.x - nt) * kT;
    b = n;
    step = (long long)(gridDim.x - nt) * kT;
  }
  for (long long idx = a + threadIdx.x; idx < b; idx += step) {
    int i, j, k;
    cell_ijk(p, idx, g, i, j, k);
    const unsigned t = tile_of(i, j, k, g);
    if (t == own) continue;
    if (!ADD) {
      flag[t] = 1u;
      continue;
    }
    double vx, vy, vz;
    Acc<PT>::vel(p, idx, vx, vy, vz);
    double* rec = mom + (size_t)block_of(i, j, k, q) * (2 * kMom) + kMom;
    atomicAdd(rec + 0, 1.0);
    atomicAdd(rec + 1, vx);
    atomicAdd(rec + 2, vy);
    atomicAdd(rec + 3, vz);
    atomicAdd(rec + 4, (vx * vx + vy * vy) + vz * vz);
  }
}

// The blocks of a tile in LDS order (cells of a block are consecutive): block
// bl of the tile, or -1 where the grid ends inside it.
__device__ __forceinline__ long long tile_block(unsigned t, int bl, const GridC& g,
                                                const BlockGeo& q) {
  const int e = kTile / q.b;
  const int tx = (int)(t % g.tnx), ty = (int)(t / g.tnx % g.tny), tz = (int)(t / (g.tnx * g.tny));
  const int bx = tx * e + bl % e, by = ty * e + bl / e % e, bz = tz * e + bl / (e * e);
  if (bx * q.b >= g.nx || by * q.b >= g.ny || bz * q.b >= g.nz) return -1;
  return ((long long)bz * q.by + by) * q.bx + bx;
}

// Clear the stray records of flagged tiles.
__global__ void __launch_bounds__(kT) k_debye_clear(const uint32_t* __restrict__ flag, unsigned nt,
                                                    GridC g, BlockGeo q, double* __restrict__ mom) {
  const int e = kTile / q.b, nb = e * e * e;
  for (unsigned t = blockIdx.x; t < nt; t += gridDim.x) {
    if (!flag[t]) continue;
    for (int bl = threadIdx.x; bl < nb; bl += kT) {
      const long long r = tile_block(t, bl, g, q);
      if (r < 0) continue;
      for (int m = 0; m < 2 * kMom; ++m) mom[r * (2 * kMom) + m] = 0.0;
    }
  }
}

// Tiles: moments per cell in LDS, joined per block, lambda_D.  flag: null when
// no ion is outside its tile.
template <class PT>
__global__ void __launch_bounds__(kT) k_debye_tiles(
    PT pe, PT pi, const uint32_t* __restrict__ tse, const uint32_t* __restrict__ tsi, unsigned nt,
    GridC g, BlockGeo q, DebyeC d, const uint32_t* __restrict__ flag,
    const double* __restrict__ mom, double* __restrict__ lam_out, long long* __restrict__ qpart,
    double* __restrict__ part) {
  __shared__ double hv[2][4][kCells];
  __shared__ unsigned hn[2][kCells];
  const int lgb = 31 - __clz(q.b), e = kTile >> lgb;
  DebyeTally y;
  // Contiguous tiles per workgroup, one XCD's workgroups side by side.
  const unsigned wg = xcd_block(blockIdx.x, gridDim.x);
  const unsigned t0 = (unsigned)((unsigned long long)nt * wg / gridDim.x);
  const unsigned t1 = (unsigned)((unsigned long long)nt * (wg + 1) / gridDim.x);
  for (unsigned t = t0; t < t1; ++t) {
    for (int c = threadIdx.x; c < kCells; c += kT)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        hn[s][c] = 0u;
#pragma unroll
        for (int m = 0; m < 4; ++m) hv[s][m][c] = 0.0;
      }
    __syncthreads();
    const int tx = (int)(t % g.tnx), ty = (int)(t / g.tnx % g.tny), tz = (int)(t / (g.tnx * g.tny));
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const PT p = s ? pi : pe;
      const long long a = (s ? tsi : tse)[t], b = (s ? tsi : tse)[t + 1];
      for (long long idx = a + threadIdx.x; idx < b; idx += kT) {
        int i, j, k;
        cell_ijk(p, idx, g, i, j, k);
        double vx, vy, vz;
        Acc<PT>::vel(p, idx, vx, vy, vz);
        i -= tx * kTile;
        j -= ty * kTile;
        k -= tz * kTile;
        // An ion that left its tile is in its block's stray record.
        if ((unsigned)i >= kTile || (unsigned)j >= kTile || (unsigned)k >= kTile) continue;
        const int bl = ((k >> lgb) * e + (j >> lgb)) * e + (i >> lgb);
        const int w = q.b - 1;
        const int c = (((bl << lgb | (k & w)) << lgb | (j & w)) << lgb) | (i & w);
        atomicAdd(&hn[s][c], 1u);
        atomicAdd(&hv[s][0][c], vx);
        atomicAdd(&hv[s][1][c], vy);
        atomicAdd(&hv[s][2][c], vz);
        atomicAdd(&hv[s][3][c], (vx * vx + vy * vy) + vz * vz);
      }
    }
    __syncthreads();
    const bool strays = flag && flag[t];
    auto finish = [&](int bl, double (&mo)[2][kMom]) {
      const long long r = tile_block(t, bl, g, q);
      if (r < 0) return;
      if (strays)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int m = 0; m < kMom; ++m) mo[s][m] += mom[r * (2 * kMom) + s * kMom + m];
      const double lam = block_lambda(mo, d, y);
      if (lam_out) lam_out[r] = lam;
    };
    if (q.b == 1) {
      for (int c = threadIdx.x; c < kCells; c += kT) {
        double mo[2][kMom];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          mo[s][0] = (double)hn[s][c];
#pragma unroll
          for (int m = 0; m < 4; ++m) mo[s][m + 1] = hv[s][m][c];
        }
        finish(c, mo);
      }
      __syncthreads();
    } else {
      // Two neighbouring cells per thread, then b^3 / 2 lanes of a block.
      double mo[2][kMom];
      const int c = 2 * threadIdx.x;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        mo[s][0] = (double)(hn[s][c] + hn[s][c + 1]);
#pragma unroll
        for (int m = 0; m < 4; ++m) mo[s][m + 1] = hv[s][m][c] + hv[s][m][c + 1];
      }
      const int lanes = (q.b * q.b * q.b) / 2;
      for (int o = (lanes < 64 ? lanes : 64) / 2; o > 0; o >>= 1)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int m = 0; m < kMom; ++m) mo[s][m] += __shfl_down(mo[s][m], o);
      __syncthreads();
      if (lanes > 64) {  // one block: the four waves' sums through LDS
        double* w = &hv[0][0][0];
        if ((threadIdx.x & 63) == 0)
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int m = 0; m < kMom; ++m) w[(threadIdx.x >> 6) * 2 * kMom + s * kMom + m] = mo[s][m];
        __syncthreads();
        if (threadIdx.x == 0)
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int m = 0; m < kMom; ++m) {
              const int o = s * kMom + m;
              mo[s][m] = (w[o] + w[2 * kMom + o]) + (w[4 * kMom + o] + w[6 * kMom + o]);
            }
        __syncthreads();
      }
      if ((threadIdx.x & (lanes - 1)) == 0) finish(threadIdx.x / lanes, mo);
    }
  }
  tally_out(&hv[0][0][0], y, qpart, part);
}

// Moments of one species (slot sidx of the block record) summed per block.
template <class PT>
__global__ void __launch_bounds__(kT) k_debye_acc(PT p, long long n, int sidx,
                                                  GridC g, BlockGeo q,
                                                  double* __restrict__ mom) {
  __shared__ unsigned hk[kHash];
  __shared__ double hv[kMom][kHash];
  const long long base = (long long)blockIdx.x * kDChunk;
  if (base >= n) return;
  for (int t = threadIdx.x; t < kHash; t += kT) {
    hk[t] = kEmpty;
#pragma unroll
    for (int m = 0; m < kMom; ++m) hv[m][t] = 0.0;
  }
  __syncthreads();
  for (int r = 0; r < kPer; ++r) {
    const long long idx = base + (long long)r * kT + threadIdx.x;
    if (idx >= n) break;
    int i, j, k;
    cell_ijk(p, idx, g, i, j, k);
    double vx, vy, vz;
    Acc<PT>::vel(p, idx, vx, vy, vz);
    const unsigned key = block_of(i, j, k, q);
    const double v2 = (vx * vx + vy * vy) + vz * vz;
    unsigned h = (key * 2654435761u) & (kHash - 1);
    int slot = -1;
    for (int probe = 0; probe < 32; ++probe) {
      const unsigned old = atomicCAS(&hk[h], kEmpty, key);
      if (old == kEmpty || old == key) {
        slot = (int)h;
        break;
      }
      h = (h + 1) & (kHash - 1);
    }
    if (slot >= 0) {
      atomicAdd(&hv[0][slot], 1.0);
      atomicAdd(&hv[1][slot], vx);
      atomicAdd(&hv[2][slot], vy);
      atomicAdd(&hv[3][slot], vz);
      atomicAdd(&hv[4][slot], v2);
    } else {
      // Table crowded: straight to the global record.
      double* rec = mom + (size_t)key * (2 * kMom) + sidx * kMom;
      atomicAdd(rec + 0, 1.0);
      atomicAdd(rec + 1, vx);
      atomicAdd(rec + 2, vy);
      atomicAdd(rec + 3, vz);
      atomicAdd(rec + 4, v2);
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kHash; t += kT) {
    const unsigned key = hk[t];
    if (key == kEmpty) continue;
    double* rec = mom + (size_t)key * (2 * kMom) + sidx * kMom;
#pragma unroll
    for (int m = 0; m < kMom; ++m) atomicAdd(rec + m, hv[m][t]);
  }
}

__global__ void k_debye_zero_u32(uint32_t* __restrict__ p, unsigned n) {
  for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    p[i] = 0u;
}

__global__ void k_debye_zero(double* __restrict__ mom, long long n) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
       i += stride)
    mom[i] = 0.0;
}

// lambda_D per block from the global records; block partials of (checked,
// unresolved) counts, the smallest lambda_D and the largest dx / d_max.
__global__ void __launch_bounds__(kT) k_debye_final(
    const double* __restrict__ mom, long long nb, DebyeC d,
    double* __restrict__ lam_out, long long* __restrict__ qpart,
    double* __restrict__ part) {
  DebyeTally y;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long b = blockIdx.x * (long long)blockDim.x + threadIdx.x; b < nb;
       b += stride) {
    double mo[2][kMom];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int m = 0; m < kMom; ++m) mo[s][m] = mom[(size_t)b * (2 * kMom) + s * kMom + m];
    const double lam = block_lambda(mo, d, y);
    if (lam_out) lam_out[b] = lam;
  }
  __shared__ double lds[4 * kT];
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

template <class PT>
void accumulate(pic_ctx* c, const BlockGeo& q) {
  const int sp[2] = {0, 2};
  for (int k = 0; k < 2; ++k) {
    const int s = sp[k];
    const long long n = c->n[s];
    if (n <= 0) continue;
    const unsigned nblk = (unsigned)((n + kDChunk - 1) / kDChunk);
    k_debye_acc<PT><<<nblk, kT, 0, c->stream>>>(species_arrays<PT>(c, s), n,
                                                 k, c->g, q, c->dbg_mom);
  }
}

template <class PT>
void tiles(pic_ctx* c, const BlockGeo& q, const DebyeC& d, double* lam_out) {
  const unsigned nt = (unsigned)c->ntiles;
  const uint32_t* tse = c->tsb[0][c->tcur[0]];
  const uint32_t* tsi = c->tsb[2][c->tcur[2]];
  // The electrons are binned every step.
  const long long tail = c->n[2] - c->n_binned[2];
  uint32_t* flag = nullptr;
  if (tail > 0 || c->ion_moved_accum > 0) {
    flag = c->tile_cursor;  // scratch of the binning passes
    k_debye_zero_u32<<<64, kT, 0, c->stream>>>(flag, nt);
    const unsigned grid = nt + (tail > 0 ? (unsigned)std::min(256ll, (tail + kT - 1) / kT) : 0u);
    k_debye_strays<PT, false><<<grid, kT, 0, c->stream>>>(species_arrays<PT>(c, 2), c->n[2],
                                                          c->n_binned[2], tsi, nt, c->g, q, flag,
                                                          c->dbg_mom);
    k_debye_clear<<<std::min(nt, 1024u), kT, 0, c->stream>>>(flag, nt, c->g, q, c->dbg_mom);
    k_debye_strays<PT, true><<<grid, kT, 0, c->stream>>>(species_arrays<PT>(c, 2), c->n[2],
                                                         c->n_binned[2], tsi, nt, c->g, q, flag,
                                                         c->dbg_mom);
  }
  k_debye_tiles<PT><<<kFinBlocks, kT, 0, c->stream>>>(
      species_arrays<PT>(c, 0), species_arrays<PT>(c, 2), tse, tsi, nt, c->g, q, d, flag,
      c->dbg_mom, lam_out, c->dbg_qpart, c->dbg_part);
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
  const long long nb = (long long)q.bx * q.by * (c->cfg.nz / block);
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
  if (c->n[0] + c->n[2] > kCrowded * c->ntiles) {
    k_debye_zero<<<1024, kT, 0, c->stream>>>(c->dbg_mom, 2 * kMom * nb);
    if (c->mixed)
      accumulate<PartsM>(c, q);
    else
      accumulate<Parts>(c, q);
    k_debye_final<<<kFinBlocks, kT, 0, c->stream>>>(
        c->dbg_mom, nb, d, lam_out, c->dbg_qpart, c->dbg_part);
  } else if (c->mixed) {
    tiles<PartsM>(c, q, d, lam_out);
  } else {
    tiles<Parts>(c, q, d, lam_out);
  }
  k_debye_reduce<<<1, 1024, 0, c->stream>>>(c->dbg_qpart, c->dbg_part,
                                            kFinBlocks, out);
}

}  // namespace pic
