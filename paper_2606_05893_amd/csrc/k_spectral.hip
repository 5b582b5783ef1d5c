// Direct solution of the 7-point Poisson system on the finest level.
//
// With x and y periodic, a plane's 2-D Fourier modes do not couple: mode
// (kx, ky) turns the operator into one tridiagonal system over z with
// d = 2 + 4 sin^2(pi kx/nx) + 4 sin^2(pi ky/ny) on the diagonal and -1 beside
// it.  A solve is therefore real DFTs over x, complex DFTs over y, one
// tridiagonal solve per mode, and the way back: five passes that each read
// and write the field once, in FP64 in both precisions of the library.  It
// works on the residual of the start, r = b - A phi_0, and adds the
// correction to phi_0, so a pass repeated on its own result refines it.
//
// Spectrum layout: the plane's nx * ny reals, in place of the field.  A row
// holds nx/2 complex slots kx; slot 0 packs the two real lines kx = 0 and
// kx = nx/2 as (X_0, X_{nx/2}).  After the y transform, slot 0 of row ky holds
// line 0's mode ky for 0 < ky < ny/2, line nx/2's mode ny - ky for ky > ny/2,
// and both lines' (real) modes for ky = 0 and ny/2.  Every real number of the
// plane is then its own tridiagonal system in z.
//
// Bound: the passes move 12 doubles a node (start and right-hand side or
// density read, spectrum written; four times read and written between the
// transforms; start read, phi written; the check's two reads).  128x128x512
// nodes in FP64, one solve with its residual check: 910 us as four V-cycles,
// 260 us here (x 52 and 42, y 35 each way, z 38, check 32); poisson_solve
// 1269 -> 286 us, on 256x256x1024 in the mixed form 8.8 -> 2.3 ms, on the
// ragged 40x20x36 382 -> 93 us.  The potential is 1e-14 from the exact one
// where the V-cycles stop at 1e-12.
#include <algorithm>

#include "pic_ctx.h"

namespace pic {
namespace {

constexpr int kSpThreads = 256;
constexpr int kSpElems = 8;  // complex values a thread holds in a stage
// Real numbers in LDS lines: one value of padding after every eight, so the
// strided stores of a radix-8 stage fall on different banks.
__host__ __device__ __forceinline__ int pad8(int i) { return i + (i >> 3); }

// Radices of a length-n transform in the order of their stages: powers of
// two as 8s and 4s (registers), odd primes by a direct sum over LDS.
struct FftPlan {
  int n, nst;
  int rad[12];
};

struct SpGrid {
  int nx, ny, nz, k0, np, bc_lo, bc_hi;
  long long nxy;
};

// Start of the solve at a node of plane k: the face value of a Dirichlet
// plane, else the caller's potential or zero.
__device__ __forceinline__ double sp_start(const SpGrid& G, const SpRhs& R,
                                           const double* __restrict__ u0, int k,
                                           long long idx) {
  if (k == 0 && G.bc_lo == PIC_BC_DIRICHLET) return R.v_lo;
  if (k == G.nz && G.bc_hi == PIC_BC_DIRICHLET) return R.v_hi;
  return u0 ? u0[idx] : 0.0;
}

FftPlan make_plan(int n) {
  FftPlan p;
  p.n = n;
  p.nst = 0;
  int a = 0, m = n;
  while (!(m & 1)) {
    m >>= 1;
    ++a;
  }
  while (a > 0) {
    // 16 as 4 x 4 and 4 as one stage: never a radix-2 stage after an 8.
    const int b = a == 4 || a == 2 ? 2 : (a >= 3 ? 3 : a);
    p.rad[p.nst++] = 1 << b;
    a -= b;
  }
  for (int f = 3; m > 1; f += 2)
    while (m % f == 0) {
      p.rad[p.nst++] = f;
      m /= f;
    }
  return p;
}

// v <- its length-R transform with e^{sg 2 pi i / R}.
template <int R>
__device__ __forceinline__ void dft_r(double2* v, double sg) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = make_double2(a.x + b.x, a.y + b.y);
    v[1] = make_double2(a.x - b.x, a.y - b.y);
  } else if constexpr (R == 4) {
    const double2 a = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
    const double2 b = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
    const double2 c = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
    // (v1 - v3) times sg i
    const double2 d = make_double2(-sg * (v[1].y - v[3].y), sg * (v[1].x - v[3].x));
    v[0] = make_double2(a.x + c.x, a.y + c.y);
    v[1] = make_double2(b.x + d.x, b.y + d.y);
    v[2] = make_double2(a.x - c.x, a.y - c.y);
    v[3] = make_double2(b.x - d.x, b.y - d.y);
  } else {
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft_r<4>(e, sg);
    dft_r<4>(o, sg);
    constexpr double h = 0.70710678118654752440;
    const double2 w1 = make_double2(h * (o[1].x - sg * o[1].y), h * (o[1].y + sg * o[1].x));
    const double2 w2 = make_double2(-sg * o[2].y, sg * o[2].x);
    const double2 w3 = make_double2(-h * (o[3].x + sg * o[3].y), h * (sg * o[3].x - o[3].y));
    const double2 w[4] = {o[0], w1, w2, w3};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = make_double2(e[q].x + w[q].x, e[q].y + w[q].y);
      v[q + 4] = make_double2(e[q].x - w[q].x, e[q].y - w[q].y);
    }
  }
}

__device__ __forceinline__ double2 cmul(double2 a, double2 w, double sg) {
  const double wi = sg * w.y;
  return make_double2(fma(a.x, w.x, -(a.y * wi)), fma(a.x, wi, a.y * w.x));
}

// Quotient of small non-negative integers (a < 2^20, n < 2^11) by a float
// reciprocal: the half-step offset keeps the truncation exact.
__device__ __forceinline__ int fdiv(int a, float rn) { return (int)(((float)a + 0.5f) * rn); }

// One self-sorting stage of radix R over all lines of the workgroup: inputs
// j + q N/R, twiddled by e^{sg 2 pi i k q / (Ns R)} with k = j mod Ns (Ns: the
// product of the radices before), outputs (j / Ns) Ns R + k + q Ns.  Every
// thread holds its butterflies in registers between the two barriers, so one
// buffer serves.
template <int R>
__device__ __forceinline__ void stage(double2* buf, const double2* tw, int n, int lines, int stride,
                                      int ns, double sg) {
  constexpr int NB = kSpElems / R;
  const int m = n / R, total = lines * m, tstep = n / (ns * R);
  const float rm = 1.0f / (float)m, rns = 1.0f / (float)ns;
  double2 v[NB][R];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < total) {
      const int line = fdiv(e, rm), j = e - line * m;
      const int k = j - fdiv(j, rns) * ns;
      const double2* src = buf + line * stride;
#pragma unroll
      for (int q = 0; q < R; ++q) v[b][q] = src[pad8(j + q * m)];
#pragma unroll
      for (int q = 1; q < R; ++q)
        if (ns > 1) v[b][q] = cmul(v[b][q], tw[k * q * tstep], sg);
      dft_r<R>(v[b], sg);
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < total) {
      const int line = fdiv(e, rm), j = e - line * m;
      const int jd = fdiv(j, rns), k = j - jd * ns;
      double2* dst = buf + line * stride;
      const int o = jd * ns * R + k;
#pragma unroll
      for (int q = 0; q < R; ++q) dst[pad8(o + q * ns)] = v[b][q];
    }
  }
  __syncthreads();
}

// The same stage for an odd prime radix r, each thread summing its outputs
// from LDS: the input twiddle and the transform's own combine into one power
// of the length-n root per term.
__device__ __forceinline__ void stage_odd(double2* buf, const double2* tw, int n, int lines,
                                          int stride, int ns, int r, double sg) {
  const int m = n / r, total = lines * n, tstep = n / (ns * r);
  const float rn = 1.0f / (float)n, rns = 1.0f / (float)ns, rr = 1.0f / (float)r;
  double2 acc[kSpElems];
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < total) {
      const int line = fdiv(e, rn), pos = e - line * n;
      const int pd = fdiv(pos, rns), k = pos - pd * ns;
      const int jd = fdiv(pd, rr), q = pd - jd * r;
      const double2* src = buf + line * stride;
      const int j = jd * ns + k, step = k * tstep + q * m;
      double2 s = make_double2(0.0, 0.0);
      int w = 0;
      for (int i = 0; i < r; ++i) {
        const double2 t = cmul(src[pad8(j + i * m)], tw[w], sg);
        s.x += t.x;
        s.y += t.y;
        w += step;
        w = w >= n ? w - n : w;
      }
      acc[b] = s;
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < total) {
      const int line = fdiv(e, rn);
      buf[line * stride + pad8(e - line * n)] = acc[b];
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void fft_lines(double2* buf, const double2* tw, const FftPlan& P,
                                          int lines, int stride, double sg) {
  int ns = 1;
  for (int s = 0; s < P.nst; ++s) {
    const int r = P.rad[s];
    if (r == 8)
      stage<8>(buf, tw, P.n, lines, stride, ns, sg);
    else if (r == 4)
      stage<4>(buf, tw, P.n, lines, stride, ns, sg);
    else if (r == 2)
      stage<2>(buf, tw, P.n, lines, stride, ns, sg);
    else
      stage_odd(buf, tw, P.n, lines, stride, ns, r, sg);
    ns *= r;
  }
}

__device__ __forceinline__ void fill_tw(double2* tw, int n) {
  for (int q = threadIdx.x; q < n; q += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * q / n, &sn, &cs);
    tw[q] = make_double2(cs, sn);
  }
}

// x forward: the residual of two neighbouring rows as one complex line.
// Contiguous ranges of lines go to one XCD, so the three planes a residual
// reads stay in its L2.  RHO: f is the caller's density and u its start (null:
// zero), see field_solve_rho; part then also takes the partials of ||b||^2,
// after those of the residual.
template <bool RHO>
__global__ void __launch_bounds__(kSpThreads) k_sp_xfwd(
    SpGrid G, const double* __restrict__ u, const double* __restrict__ f, double* __restrict__ s,
    FftPlan P, int nlines, int lpw, int stride, double* __restrict__ part, SpRhs R) {
  extern __shared__ double2 sm[];
  double2* tw = sm;
  double2* buf = sm + P.n;
  const int nx = G.nx, nyp = G.ny / 2;
  const int wg = xcd_block(blockIdx.x, gridDim.x);
  const int line0 = wg * lpw;
  const int lines = nlines - line0 < lpw ? nlines - line0 : lpw;
  const float rnx = 1.0f / (float)nx;
  double s2 = 0.0, sb = 0.0;
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < lines * nx) {
      const int l = fdiv(e, rnx), i = e - l * nx;
      const int gl = line0 + l;
      const int p = gl / nyp, j = 2 * (gl - p * nyp), k = G.k0 + p;
      const int im = i ? i - 1 : nx - 1, ip = i + 1 < nx ? i + 1 : 0;
      const int jm = j ? j - 1 : G.ny - 1, jp = j + 2 < G.ny ? j + 2 : 0;
      const long long za = (long long)j * nx + i;
      const long long at = (long long)k * G.nxy + za;
      const int kd = k > 0 ? k - 1 : 1, ku = k < G.nz ? k + 1 : G.nz - 1;
      const long long ad = (long long)kd * G.nxy + za, au = (long long)ku * G.nxy + za;
      double fa = f[at], fb = f[at + nx];
      // The nodes (a: row j, b: row j + 1), their x and outer y neighbours,
      // and the planes below and above.
      double ca = 0.0, cb = 0.0, xa = 0.0, xb = 0.0, ym = 0.0, yp = 0.0;
      double da, db, ua, ub;
      if (!RHO || u) {
        const double* pl = u + (long long)k * G.nxy;
        const double* ra = pl + j * nx;
        const double* rb = ra + nx;
        ca = ra[i]; cb = rb[i];
        xa = ra[im] + ra[ip]; xb = rb[im] + rb[ip];
        ym = pl[jm * nx + i]; yp = pl[jp * nx + i];
      }
      if (RHO) {
        fa = sp_rhs(R, k, G.nz, fa);
        fb = sp_rhs(R, k, G.nz, fb);
        // ||b|| of the system with the Dirichlet data on its right.
        const double lo = k == 1 && G.bc_lo == PIC_BC_DIRICHLET ? R.v_lo : 0.0;
        const double hi = k == G.nz - 1 && G.bc_hi == PIC_BC_DIRICHLET ? R.v_hi : 0.0;
        const double ba = (fa + lo) + hi, bb = (fb + lo) + hi;
        sb += ba * ba + bb * bb;
        da = sp_start(G, R, u, kd, ad); db = sp_start(G, R, u, kd, ad + nx);
        ua = sp_start(G, R, u, ku, au); ub = sp_start(G, R, u, ku, au + nx);
      } else {
        da = u[ad]; db = u[ad + nx];
        ua = u[au]; ub = u[au + nx];
      }
      // The stencil sum of one node: x pair, then y pair, then z pair (a
      // Neumann face's mirrored neighbour taken twice).
      const double na = (xa + (ym + cb)) + (da + ua);
      const double nb = (xb + (ca + yp)) + (db + ub);
      const double va = fa - (6.0 * ca - na), vb = fb - (6.0 * cb - nb);
      s2 += va * va + vb * vb;
      buf[l * stride + pad8(i)] = make_double2(va, vb);
    }
  }
  fill_tw(tw, P.n);
  __syncthreads();
  fft_lines(buf, tw, P, lines, stride, -1.0);
  const int nh = nx / 2;
  const float rnh = 1.0f / (float)nh;
#pragma unroll
  for (int b = 0; b < kSpElems / 2; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < lines * nh) {
      const int l = fdiv(e, rnh), kx = e - l * nh;
      const double2 z = buf[l * stride + pad8(kx)];
      const double2 c = buf[l * stride + pad8(kx ? nx - kx : nh)];
      double2 xa, xb;
      if (kx == 0) {
        xa = make_double2(z.x, c.x);
        xb = make_double2(z.y, c.y);
      } else {
        xa = make_double2(0.5 * (z.x + c.x), 0.5 * (z.y - c.y));
        xb = make_double2(0.5 * (z.y + c.y), 0.5 * (c.x - z.x));
      }
      const int gl = line0 + l;
      double* o = s + (long long)gl * 2 * nx + 2 * kx;
      *reinterpret_cast<double2*>(o) = xa;
      *reinterpret_cast<double2*>(o + nx) = xb;
    }
  }
  // Sums of squares of the residual (and of b): one partial per workgroup.
  __syncthreads();
  double* red = reinterpret_cast<double*>(buf);
  const unsigned nw = (blockDim.x + 63) / 64;
  for (int o = 32; o > 0; o >>= 1) {
    s2 += __shfl_down(s2, o);
    if (RHO) sb += __shfl_down(sb, o);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s2;
    if (RHO) red[nw + (threadIdx.x >> 6)] = sb;
  }
  __syncthreads();
  if (threadIdx.x < (RHO ? 2u : 1u)) {
    double a = 0.0;
    for (unsigned w = 0; w < nw; ++w) a += red[threadIdx.x * nw + w];
    part[threadIdx.x * gridDim.x + wg] = a;
  }
}

// Start of a solve from the two sums: ||b||, the counters at zero, and the
// initial check.
__global__ void __launch_bounds__(1024) k_sp_begin(const double* __restrict__ part, int n,
                                                   Counters* dc, double tol) {
  __shared__ double s[2][16];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) {
    a += part[i];
    b += part[n + i];
  }
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_down(a, o);
    b += __shfl_down(b, o);
  }
  if ((threadIdx.x & 63) == 0) {
    s[0][threadIdx.x >> 6] = a;
    s[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int w = 1; w < 16; ++w) {
    a += s[0][w];
    b += s[1][w];
  }
  const double bn = sqrt(b), rr = bn > 0.0 ? sqrt(a) / bn : 0.0;
  dc->b_norm = bn;
  dc->total_charge = 0;
  dc->vcycles = 0;
  dc->refinements = 0;
  dc->rel_res = rr;
  dc->rel_res0 = rr;
  dc->done = 0;
  if (!(rr == rr)) {
    dc->err |= kErrNonFinite;
    dc->done = 1;
  } else if (rr <= tol) {
    dc->done = 1;
  }
}

// y transforms of the columns, lpw neighbouring slots of the flattened
// (plane, slot) list per workgroup, in place.
template <bool INV>
__global__ void __launch_bounds__(kSpThreads) k_sp_y(SpGrid G, double* __restrict__ s, FftPlan P,
                                                     int nlines, int lpw, int stride,
                                                     const Counters* dc) {
  extern __shared__ double2 sm[];
  if (dc->done) return;
  double2* tw = sm;
  double2* buf = sm + P.n;
  const int nh = G.nx / 2, ny = G.ny;
  const int line0 = xcd_block(blockIdx.x, gridDim.x) * lpw;
  const int lines = nlines - line0 < lpw ? nlines - line0 : lpw;
  const float rl = 1.0f / (float)lines;
  double2* sp = reinterpret_cast<double2*>(s);
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < lines * ny) {
      const int j = fdiv(e, rl), l = e - j * lines;
      const int gl = line0 + l, p = gl / nh, kx = gl - p * nh;
      double2* pl = sp + (long long)p * ny * nh;
      double2 v = pl[j * nh + kx];
      if (INV && kx == 0 && j != 0 && 2 * j != ny) {
        // C(ky) = F_0(ky) + i F_N(ky); F(-ky) = conj F(ky).
        const double2 w = pl[(ny - j) * nh];
        v = 2 * j < ny ? make_double2(v.x - w.y, v.y + w.x) : make_double2(w.x + v.y, v.x - w.y);
      }
      buf[l * stride + pad8(j)] = v;
    }
  }
  fill_tw(tw, P.n);
  __syncthreads();
  fft_lines(buf, tw, P, lines, stride, INV ? 1.0 : -1.0);
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < lines * ny) {
      const int j = fdiv(e, rl), l = e - j * lines;
      const int gl = line0 + l, p = gl / nh, kx = gl - p * nh;
      double2 v = buf[l * stride + pad8(j)];
      if (!INV && kx == 0 && j != 0 && 2 * j != ny) {
        // F_0 = (C(ky) + conj C(-ky)) / 2, F_N = (C(ky) - conj C(-ky)) / 2i,
        // F_N stored at the mirrored row.
        const double2 c = buf[l * stride + pad8(ny - j)];
        v = 2 * j < ny ? make_double2(0.5 * (v.x + c.x), 0.5 * (v.y - c.y))
                       : make_double2(0.5 * (c.y + v.y), 0.5 * (v.x - c.x));
      }
      sp[((long long)p * ny + j) * nh + kx] = v;
    }
  }
}

// x inverse and correction: phi = phi_0 + the transform of two rows' slots.
// RHO: phi_0 is u0 (null: zero); u and (unless null) out take phi, with the
// Dirichlet planes' values beside the planes next to them, also where the
// start needs no correction.
template <bool RHO>
__global__ void __launch_bounds__(kSpThreads) k_sp_xinv(SpGrid G, const double* __restrict__ s,
                                                        const double* u0, double* u, double* out,
                                                        FftPlan P, int nlines, int lpw, int stride,
                                                        const Counters* dc, SpRhs R) {
  extern __shared__ double2 sm[];
  const bool done = dc->done;
  if (!RHO && done) return;
  double2* tw = sm;
  double2* buf = sm + P.n;
  const int nx = G.nx, nh = nx / 2;
  const int line0 = xcd_block(blockIdx.x, gridDim.x) * lpw;
  const int lines = nlines - line0 < lpw ? nlines - line0 : lpw;
  if (!done) {
    const float rnh = 1.0f / (float)nh;
#pragma unroll
    for (int b = 0; b < kSpElems / 2; ++b) {
      const int e = threadIdx.x + b * blockDim.x;
      if (e < lines * nh) {
        const int l = fdiv(e, rnh), kx = e - l * nh;
        const double* o = s + (long long)(line0 + l) * 2 * nx + 2 * kx;
        const double2 ga = *reinterpret_cast<const double2*>(o);
        const double2 gb = *reinterpret_cast<const double2*>(o + nx);
        double2* dst = buf + l * stride;
        if (kx == 0) {
          dst[0] = make_double2(ga.x, gb.x);
          dst[pad8(nh)] = make_double2(ga.y, gb.y);
        } else {
          dst[pad8(kx)] = make_double2(ga.x - gb.y, ga.y + gb.x);
          dst[pad8(nx - kx)] = make_double2(ga.x + gb.y, gb.x - ga.y);
        }
      }
    }
    fill_tw(tw, P.n);
    __syncthreads();
    fft_lines(buf, tw, P, lines, stride, 1.0);
  }
  const double sc = 1.0 / ((double)nx * (double)G.ny);
  const float rnx = 1.0f / (float)nx;
  const long long base = (long long)G.k0 * G.nxy;
#pragma unroll
  for (int b = 0; b < kSpElems; ++b) {
    const int e = threadIdx.x + b * blockDim.x;
    if (e < lines * nx) {
      const int l = fdiv(e, rnx), i = e - l * nx;
      const long long at = base + (long long)(line0 + l) * 2 * nx + i;
      double va = !RHO || u0 ? u0[at] : 0.0, vb = !RHO || u0 ? u0[at + nx] : 0.0;
      if (!done) {
        const double2 v = buf[l * stride + pad8(i)];
        va = va + sc * v.x;
        vb = vb + sc * v.y;
      }
      auto put = [&](long long q, double x) {
        u[q] = x;
        if (RHO && out) out[q] = x;
      };
      put(at, va);
      put(at + nx, vb);
      if (RHO) {
        const int k = G.k0 + (int)((line0 + l) / (G.ny / 2));
        if (k == 1 && G.bc_lo == PIC_BC_DIRICHLET) {
          put(at - G.nxy, R.v_lo);
          put(at - G.nxy + nx, R.v_lo);
        }
        if (k == G.nz - 1 && G.bc_hi == PIC_BC_DIRICHLET) {
          put(at + G.nxy, R.v_hi);
          put(at + G.nxy + nx, R.v_hi);
        }
      }
    }
  }
}

__device__ __forceinline__ double ipow(double b, int e) {
  double r = 1.0;
  for (; e; e >>= 1, b *= b)
    if (e & 1) r *= b;
  return r;
}

// The tridiagonal systems -x_{p-1} + d x_p - x_{p+1} = b_p, one per real
// number of the plane, in place.  With d = l + 1/l (0 < l <= 1) the operator
// factors into (1/l)(1 - l S)(1 - l S^-1): two first-order recurrences with
// the one coefficient l give a solution x' with x'_np = 0, and c h_p, h_p =
// sinh((np - p) t) / sinh((np + 1) t) with l = e^-t, sets the lower face.
// Dirichlet: x_{-1} = 0.  Neumann: x_{-1} = x_1 (the row takes its inner
// neighbour twice).  With the Neumann face on top the planes run downwards.
// A thread runs SEG planes of one system in registers; the segments' ends are
// joined through LDS.  No pivots are stored or divided: the pass reads and
// writes the spectrum once.  At 512 planes of 128 x 128: 84 us with the rows'
// addresses kept from the loads to the stores and each join a pass over the
// registers (102 of them spilled), 38 us now; 1024 of 256 x 256 565 -> 254.
template <int SEG>
__global__ void __launch_bounds__(SEG > 32 ? 512 : 1024) k_sp_tri(SpGrid G, double* __restrict__ s,
                                                                  int lgc, const Counters* dc) {
  extern __shared__ double2 sm[];
  if (dc->done) return;
  const int cols = 1 << lgc;
  const int c = threadIdx.x & (cols - 1), sg = threadIdx.x >> lgc;
  const int nsg = blockDim.x >> lgc;
  double* jz = reinterpret_cast<double*>(sm);
  const int col = blockIdx.x * cols + c;
  const bool ok = col < G.nxy;
  const int cc = ok ? col : 0;
  int ky = cc / G.nx;
  const int xr = cc - ky * G.nx;
  int kx = xr >> 1;
  if (kx == 0) {
    const int hy = G.ny / 2;
    if (ky == 0 || ky == hy) {
      kx = (xr & 1) ? G.nx / 2 : 0;
    } else if (ky > hy) {
      kx = G.nx / 2;
      ky = G.ny - ky;
    }
  }
  const bool rev = G.bc_hi == PIC_BC_NEUMANN;
  const bool neu = rev || G.bc_lo == PIC_BC_NEUMANN;
  const int np = G.np, p0 = sg * SEG;
  const int nv = np - p0;                      // planes of this and later segments
  const long long step = rev ? -G.nxy : G.nxy;
  double* base = s + cc + (rev ? (long long)(np - 1) * G.nxy : 0) + p0 * step;
  double b[SEG];
  {
    const double* r = base;
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      b[q] = *r;                               // (past the end: the last plane)
      r += q + 1 < nv ? step : 0;
      // (Eight addresses at a time: all of them beside the loads spill.)
      if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  }
  const double sx = sinpi((double)kx / G.nx), sy = sinpi((double)ky / G.ny);
  const double qq = sx * sx + sy * sy;  // (d - 2) / 4
  const double rt = sqrt(1.0 + qq) + sqrt(qq);
  const double l = 1.0 / (rt * rt);
  const double lseg = ipow(l, SEG);
  // y_p = l (b_p + y_{p-1}), segment-local, then joined.
  double y = 0.0;
#pragma unroll
  for (int q = 0; q < SEG; ++q) {
    y = q < nv ? l * (b[q] + y) : 0.0;
    b[q] = y;
  }
  jz[threadIdx.x] = y;
  __syncthreads();
  y = 0.0;
  for (int q = 0; q < sg; ++q) y = fma(lseg, y, jz[(q << lgc) + c]);
  __syncthreads();
  // x'_p = y_p + l x'_{p+1} from x'_np = 0.
  double w = l * y;
#pragma unroll
  for (int q = 0; q < SEG; ++q) {
    if (q < nv) b[q] += w;
    w *= l;
  }
  double x = 0.0;
#pragma unroll
  for (int q = SEG - 1; q >= 0; --q) {
    x = fma(l, x, b[q]);
    b[q] = x;
  }
  jz[threadIdx.x] = x;
  __syncthreads();
  x = 0.0;
  for (int q = nsg - 1; q > sg; --q) x = fma(lseg, x, jz[(q << lgc) + c]);
  // The join adds w l^(SEG-1-q) to this segment's x'; for the face's
  // coefficient the first two planes take it now, the others with the
  // second exponential, whose powers are the same.
  w = l * x;
  __syncthreads();
  if (sg == 0) {
    const double w1 = w * ipow(l, SEG - 2);
    jz[c] = fma(w1, l, b[0]);
    jz[cols + c] = b[1] + w1;
  }
  __syncthreads();
  const double x0 = jz[c], x1 = jz[cols + c];
  // h_p from its two exponentials, e^{-(p+1)t} and e^{-(2np+1-p)t}.
  const bool flat = qq == 0.0;
  const double l2n = ipow(l, 2 * np + 2);
  const double den = flat ? 1.0 / (double)(np + 1) : 1.0 / (1.0 - l2n);
  double cf = l * x0;
  if (neu) {
    // h_{-1} - h_1
    const double dh = flat ? 2.0 * den : (1.0 - l * l) * (1.0 + ipow(l, 2 * np)) * den;
    cf = (l * x0 - (np > 1 ? x1 : 0.0)) / dh;
  }
  cf *= den;
  if (flat) {
    // (l = 1: the join is w everywhere, the h_p are linear.)
    double h = cf * (double)(np - p0);
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      b[q] += w - h;
      h -= cf;
    }
  } else {
    double ea = -cf * ipow(l, p0 + 1);
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      b[q] += ea;
      ea *= l;
    }
    // Down from the segment's last plane (the last segment's w is zero).
    const int pe = nv < SEG ? np : p0 + SEG;  // one past it
    w = fma(cf, ipow(l, 2 * np + 2 - pe), w);
#pragma unroll
    for (int q = SEG - 1; q >= 0; --q) {
      if (q < nv) {
        b[q] += w;
        w *= l;
      }
    }
  }
  if (ok) {
    // The rows' addresses anew: kept from the loads they spill.
    int z = 0;
    asm volatile("" : "+v"(z));
    double* o = base + z;
#pragma unroll
    for (int q = 0; q < SEG; ++q) {
      if (q < nv) *o = b[q];
      o += step;
      if (q % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Lines per workgroup: what the threads hold, fewer where that would leave
// the chip idle, so at least 512 workgroups (two a CU) as long as each has
// four lines.  poisson_solve with at least 256 / 512 / 1024 / 2048: 118 / 106 /
// 104 / 104 us on 48x48x96, 168 / 152 / 147 / 160 on 120x90x100, 113 / 113 /
// 105 / 106 on 64x64x128; from 128x128x128 on the threads' limit decides.  With
// at least 1 / 2 / 4 / 8 lines: 98 / 98 / 98 / 106 on 64x64x64, 106 / 106 / 106
// / 115 on 48x48x96.
int lines_per_wg(int n, long long nlines) {
  const int most = kSpThreads * kSpElems / n;
  const long long spread = std::max(4LL, (nlines + 511) / 512);
  return (int)std::max(1LL, std::min<long long>(most, spread));
}

struct LineLaunch {
  FftPlan plan;
  int nlines, lpw, stride, threads;
  unsigned grid;
  size_t lds;
};

LineLaunch line_launch(int n, long long nlines) {
  LineLaunch a;
  a.plan = make_plan(n);
  a.nlines = (int)nlines;
  a.lpw = lines_per_wg(n, nlines);
  a.stride = pad8(n) + 1;
  // Enough threads for kSpElems values each.
  a.threads = ((a.lpw * n + kSpElems - 1) / kSpElems + 63) / 64 * 64;
  a.grid = (unsigned)((nlines + a.lpw - 1) / a.lpw);
  a.lds = (size_t)(n + a.lpw * a.stride) * sizeof(double2);
  return a;
}

SpGrid sp_grid(const pic_ctx* c) {
  SpGrid g;
  const pic_config& f = c->cfg;
  g.nx = f.nx; g.ny = f.ny; g.nz = f.nz;
  g.bc_lo = f.bc_lo; g.bc_hi = f.bc_hi;
  g.k0 = f.bc_lo == PIC_BC_DIRICHLET ? 1 : 0;
  g.np = (f.bc_hi == PIC_BC_DIRICHLET ? f.nz - 1 : f.nz) - g.k0 + 1;
  g.nxy = (long long)f.nx * f.ny;
  return g;
}

}  // namespace

bool spectral_direct(const pic_config* f) {
  if (f->mg_levels != 0 || (f->flags & PIC_FLAG_MG_ALL_LEVELS)) return false;
  return f->nx <= kDirectMaxXY && f->ny <= kDirectMaxXY && f->nz < kDirectMaxPlanes;
}

int spectral_partials(const pic_ctx* c) {
  const SpGrid G = sp_grid(c);
  return (int)line_launch(G.nx, (long long)G.np * (G.ny / 2)).grid;
}

void spectral_forward(pic_ctx* c) {
  const SpGrid G = sp_grid(c);
  const LineLaunch a = line_launch(G.nx, (long long)G.np * (G.ny / 2));
  k_sp_xfwd<false><<<a.grid, a.threads, a.lds, c->stream>>>(
      G, c->lev[0].u, c->lev[0].f, c->spec_d, a.plan, a.nlines, a.lpw, a.stride, c->partials,
      SpRhs{});
}

// The passes between the two x transforms.
static void spectral_modes(pic_ctx* c) {
  const SpGrid G = sp_grid(c);
  double* s = c->spec_d;
  const LineLaunch y = line_launch(G.ny, (long long)G.np * (G.nx / 2));
  k_sp_y<false><<<y.grid, y.threads, y.lds, c->stream>>>(G, s, y.plan, y.nlines, y.lpw, y.stride,
                                                         c->dc);
  // Planes a thread holds: a workgroup takes 32 columns (whole 256-byte rows)
  // and as many segments as cover the planes, at most 512 threads' worth with 8
  // and 16 planes and 1024 with 32; past 1024 planes 64, whose registers allow
  // 512 threads, so 16 columns.  The limits of 1024 and 2048 planes are the
  // workgroup's; those of 128 and 256 (256 and 512 would fit) cost nothing:
  // poisson_solve with 8 / 16 / 32 / 64 takes 149 / 147 / 150 / 153 us on
  // 128x128x128, 175 / 172 / 175 / 177 on 128x128x256, with 16 / 32 / 64 275 /
  // 276 / 279 on 128x128x512, with 32 / 64 1931 / 1950 on 256x256x1024.
  const int seg = G.np <= 128 ? 8 : G.np <= 256 ? 16 : G.np <= 1024 ? 32 : 64;
  const int nsg = std::max(1, (G.np + seg - 1) / seg);
  const int lgc = seg == 64 ? 4 : 5;
  const unsigned grid = (unsigned)((G.nxy + (1 << lgc) - 1) >> lgc);
  const int nt = nsg << lgc;
  // The join slots, and the two planes next to the face.
  const size_t lds = (size_t)std::max(nt, 2 << lgc) * sizeof(double);
  if (seg == 8)
    k_sp_tri<8><<<grid, nt, lds, c->stream>>>(G, s, lgc, c->dc);
  else if (seg == 16)
    k_sp_tri<16><<<grid, nt, lds, c->stream>>>(G, s, lgc, c->dc);
  else if (seg == 32)
    k_sp_tri<32><<<grid, nt, lds, c->stream>>>(G, s, lgc, c->dc);
  else
    k_sp_tri<64><<<grid, nt, lds, c->stream>>>(G, s, lgc, c->dc);
  k_sp_y<true><<<y.grid, y.threads, y.lds, c->stream>>>(G, s, y.plan, y.nlines, y.lpw, y.stride,
                                                        c->dc);
}

void spectral_correct(pic_ctx* c) {
  const SpGrid G = sp_grid(c);
  spectral_modes(c);
  const LineLaunch x = line_launch(G.nx, (long long)G.np * (G.ny / 2));
  double* u = c->lev[0].u;
  k_sp_xinv<false><<<x.grid, x.threads, x.lds, c->stream>>>(
      G, c->spec_d, u, u, nullptr, x.plan, x.nlines, x.lpw, x.stride, c->dc, SpRhs{});
}

SpRhs sp_rhs_of(const pic_ctx* c) {
  const double dx = c->g.dx;
  return SpRhs{(dx * dx) / kEps0, 2.0 * dx, c->cfg.v_lo, c->cfg.v_hi, c->cfg.bc_lo,
               c->cfg.bc_hi};
}

void spectral_solve_rho(pic_ctx* c, const SpRhs& R, const double* rho, const double* u0,
                        double* u, double* out, bool first) {
  const SpGrid G = sp_grid(c);
  const LineLaunch x = line_launch(G.nx, (long long)G.np * (G.ny / 2));
  k_sp_xfwd<true><<<x.grid, x.threads, x.lds, c->stream>>>(
      G, u0, rho, c->spec_d, x.plan, x.nlines, x.lpw, x.stride, c->partials, R);
  if (first)
    k_sp_begin<<<1, 1024, 0, c->stream>>>(c->partials, (int)x.grid, c->dc, c->cfg.rel_tol);
  spectral_modes(c);
  k_sp_xinv<true><<<x.grid, x.threads, x.lds, c->stream>>>(
      G, c->spec_d, u0, u, out, x.plan, x.nlines, x.lpw, x.stride, c->dc, R);
}

}  // namespace pic
