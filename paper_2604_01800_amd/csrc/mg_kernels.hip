// Multigrid V-cycle kernels (HIP, gfx950): the preconditioner of the MGPCG
// CG-type (Sec. 2.5, four levels by default).
//
// Level l+1 merges 2 x 2 cells of level l; prolongation is piecewise
// constant and restriction its transpose (sum over the four children), and
// the coarse operators are the Galerkin products P^T A P, which on a tensor
// grid are again five-point operators of 1D arrays (merged widths, the fine
// face factors at surviving faces), so every level runs the same matrix-free
// stencil. Smoothing is the degree-2 Chebyshev semi-iteration on D^-1 A over
// [0.2, 2] (Saad, Sec. 12.3), before the coarse correction from a zero guess
// and after it:
//   pre:   x1 = D^-1 b / theta;  r1 = b - A x1;
//          x2 = x1 + c1 x1 + c2 D^-1 r1
//   post:  x3 = x2 + P e;  r3 = b - A x3;  d = D^-1 r3 / theta;  x4 = x3 + d;
//          r4 = b - A x4;  x5 = x4 + c1 d + c2 D^-1 r4
// with theta, delta the interval's centre and half-width, c1 = rho1 rho0,
// c2 = 2 rho1 / delta (rho0 = delta / theta, rho1 = 1 / (2 theta/delta - rho0)).
// A level costs two launches: down (pre-smoothing, residual, restriction) and
// up (prolongation, both post steps). Each takes two stencil applications on a
// tile with a two-cell halo, recomputed instead of exchanged: the cycle is bound by the
// latency of its dependent launches (3.2 to 6.3 us each at 256^2 to 1024^2, for
// at most 4 MB a vector), not by the bytes or the arithmetic that the wider halo adds. A
// kernel that reads a vector on a halo never writes that vector (other
// workgroups may still be reading it): x2 lives in x, x5 in y. The coarsest
// level is solved exactly by the separable direct method (transforms to the
// eigenbases of both axes, a diagonal scaling, and back) in FP64, with the
// right-hand side's mean removed before and the solution's mean after, i.e. the
// minimum-norm solution.
//
// Vectors are FP32; every kernel returns at once for a solve whose done flag
// is set. The last kernel of the fine level leaves its workgroups' shares of
// r.z, which phase A of the PCG adds up.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "kernels.hpp"
#include "launch_plan.hpp"
#include "mg_internal.hpp"
#include "stencil.hpp"

namespace ppe {

namespace {

struct Cheb {
  float inv_theta, c1, c2;
};

Cheb cheb_consts() {
  const double theta = 0.5 * (kChebHi + kChebLo), delta = 0.5 * (kChebHi - kChebLo);
  const double sigma = theta / delta;
  const double rho0 = 1.0 / sigma, rho1 = 1.0 / (2.0 * sigma - rho0);
  return Cheb{(float)(1.0 / theta), (float)(rho1 * rho0), (float)(2.0 * rho1 / delta)};
}

// Arguments of one level's kernels (passed by value).
struct LevelArgs {
  Coef c;
  int64_t N;               // cells per solve on this level
  const float* b;          // [nb][N]
  float* x;                // [nb][N] x2
  float* y;                // [nb][N] x5
  const int32_t* flags;    // [nb] done codes of the solves
  Cheb k;
  // restriction target / coarse correction source (level l+1)
  float* bc;               // [nb][Nc] coarse right-hand side
  const float* ec;         // [nb][Nc] coarse solution
  int nxc;
  int64_t Nc;
  int bc_t;                // bc is stored transposed ([nxc][nyc])
  int coarsest;            // level l+1 is the coarsest: means are taken there
  double* bpart;           // [nb][P] partial sums of the coarse right-hand side (coarsest only)
  const double* xpart;     // [nb][nyc] row sums of the coarsest solution (coarsest only)
  int nyc;
  double* rzpart;          // fine level: [nb][P] shares of r.z, else NULL
  int P;                   // workgroups per solve of this level
};

}  // namespace

__device__ __forceinline__ float dinv_at(float hyj, float gs, float gn, float hx, float gw, float ge) {
  return 1.0f / fmaxf(diag_of(hyj, gs, gn, hx, gw, ge), 1e-30f);
}

// Tiles of the level kernels: a wavefront's 64 lanes hold 60 owned columns and
// two halo columns on either side (east and west neighbours are DPP wave
// shifts; a stencil application loses one lane at each end), and R owned rows
// between two halo rows above and below. Tiles start on even columns and
// rows, so a 2 x 2 block of children never crosses a tile. XCD banded as the
// 64-column tiles are.
constexpr int kMgH = 2;
constexpr int kMgOwn = kWave - 2 * kMgH;

__device__ __forceinline__ TileXY mg_tile_xy(int nx, int ny, int R) {
  const int gxt = (nx + kMgOwn - 1) / kMgOwn;
  const int gyt = (ny + kWaves * R - 1) / (kWaves * R);
  const int T = gxt * gyt;
  const int per = (T + 7) / 8;
  int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  TileXY o;
  o.valid = t < T;
  if (!o.valid) t = 0;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  o.i0 = (t % gxt) * kMgOwn - kMgH;
  o.j0 = ((t / gxt) * kWaves + w) * R;
  return o;
}

// Rows per wavefront of a level: enough workgroups to cover the chip.
static int mg_rows(int64_t cells) {
  if (cells >= ((int64_t)1 << 20)) return 8;
  if (cells >= ((int64_t)1 << 17)) return 4;
  return 2;
}

static int mg_tiles(int nx, int ny, int R) {
  const int T = ((nx + kMgOwn - 1) / kMgOwn) * ((ny + kWaves * R - 1) / (kWaves * R));
  return 8 * ((T + 7) / 8);
}

// This lane's column of a level tile and the row coefficients of its R + 4
// rows (row q is j0 - 2 + q; the padded arrays read 0 off the grid).
template <int R>
struct MgTile {
  int i, j0;
  bool inx, own;
  float hx, gw, ge;
  float hy[R + 2 * kMgH], gy[R + 2 * kMgH + 1];

  __device__ __forceinline__ MgTile(const Coef& c) {
    const TileXY tl = mg_tile_xy(c.nx, c.ny, R);
    const int lane = threadIdx.x & (kWave - 1);
    i = tl.i0 + lane;
    j0 = tl.j0;
    inx = tl.valid && i >= 0 && i < c.nx;
    own = inx && lane >= kMgH && lane < kWave - kMgH;
#pragma unroll
    for (int q = 0; q < R + 2 * kMgH; ++q) hy[q] = c.hy[j0 - kMgH + q];
#pragma unroll
    for (int q = 0; q < R + 2 * kMgH + 1; ++q) gy[q] = c.gy[j0 - kMgH + q];
    hx = c.hx[i];
    gw = c.gx[i];
    ge = c.gx[i + 1];
  }
  __device__ __forceinline__ float dinv(int q) const { return dinv_at(hy[q], gy[q], gy[q + 1], hx, gw, ge); }
  // (A v) on row q of a column of R + 4 values; lanes 0 and 63 lack a neighbour
  __device__ __forceinline__ float apply(const float (&v)[R + 2 * kMgH], int q) const {
    const float ve = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v[q]), 0x130, 0xf, 0xf, true));
    const float vw = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v[q]), 0x138, 0xf, 0xf, true));
    return stencil5(v[q], ve, vw, v[q + 1], v[q - 1], hy[q], gy[q], gy[q + 1], hx, gw, ge);
  }
};

// Down: pre-smoothing from a zero guess (x2, stored), its residual and the
// restriction of that (sum over 2 x 2 children) to the coarse right-hand side;
// on the way to the coarsest level also the partial sums of the coarse
// right-hand side (its mean is removed there). Bytes per cell: b read, x2
// written, a quarter of a coarse value written (9 B). At 1024^2 one launch of
// 5.2 us replaces two of 4.7 and 3.3 us.
template <int R>
__global__ __launch_bounds__(kBlock) void k_mg_down(LevelArgs a) {
  constexpr int Q = R + 2 * kMgH;
  __shared__ double lds[kWaves];
  const int s = blockIdx.z, nx = a.c.nx, ny = a.c.ny;
  if (a.flags[s] != DONE_NO) return;
  const size_t off = (size_t)s * a.N;
  const uint64_t vbytes = (uint64_t)a.N * 4;
  const MgTile<R> t(a.c);
  const auto bs = make_rsrc(a.b + off, vbytes);
  float b[Q], x1[Q], x2[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) b[q] = bload(bs, cell_off(t.inx, t.j0 - kMgH + q, ny, nx, t.i));
#pragma unroll
  for (int q = 0; q < Q; ++q) x1[q] = b[q] * t.dinv(q) * a.k.inv_theta;
  x2[0] = x2[Q - 1] = 0.f;
  const auto xs = make_rsrc(a.x + off, vbytes);
#pragma unroll
  for (int q = 1; q < Q - 1; ++q) {
    const float r1 = b[q] - t.apply(x1, q);
    x2[q] = x1[q] + a.k.c1 * x1[q] + a.k.c2 * t.dinv(q) * r1;
    if (q >= kMgH && q < kMgH + R) bstore(xs, cell_off(t.own, t.j0 - kMgH + q, ny, nx, t.i), x2[q]);
  }
  const int lane = threadIdx.x & (kWave - 1);
  const auto cs = make_rsrc(a.bc + (size_t)s * a.Nc, (uint64_t)a.Nc * 4);
  double acc = 0.0;
#pragma unroll
  for (int q = kMgH; q < kMgH + R; q += 2) {
    // rows j and j + 1 form one coarse row (j0 and R are even); off the grid
    // both the residual's inputs and its coefficients are 0
    const float v = (b[q] - t.apply(x2, q)) + (b[q + 1] - t.apply(x2, q + 1));
    const float sum = v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
    const int j = t.j0 - kMgH + q;
    const bool w = t.own && (lane & 1) == 0 && j < ny;
    const int jc = j >> 1, ic = t.i >> 1;
    bstore(cs, w ? (uint32_t)(a.bc_t ? ic * (ny >> 1) + jc : jc * a.nxc + ic) * 4u : kOOB, sum);
    if (w) acc += (double)sum;
  }
  if (a.coarsest) {
    acc = block_sum(acc, lds);
    if (threadIdx.x == 0) a.bpart[(size_t)s * a.P + block_linear()] = acc;
  }
}

// Up: coarse correction x3 = x2 + P e and both post-smoothing steps,
//   d = D^-1 (b - A x3) / theta, x4 = x3 + d, x5 = x4 + c1 d + c2 D^-1 (b - A x4);
// reads x2 from x, writes x5 to y. On the fine level b is the PCG residual r
// and x5 is z; the workgroup's share of r.z goes to rzpart. Bytes per cell:
// x2 and b read, a quarter of a coarse value read, x5 written (13 B). At
// 1024^2 one launch of 6.2 us replaces two of 5.2 and 4.8 us.
template <int R>
__global__ __launch_bounds__(kBlock) void k_mg_up(LevelArgs a) {
  constexpr int Q = R + 2 * kMgH;
  __shared__ double lds[kWaves];
  const int s = blockIdx.z, nx = a.c.nx, ny = a.c.ny;
  if (a.flags[s] != DONE_NO) return;
  const size_t off = (size_t)s * a.N;
  const uint64_t vbytes = (uint64_t)a.N * 4;
  const MgTile<R> t(a.c);
  const auto xs = make_rsrc(a.x + off, vbytes), bs = make_rsrc(a.b + off, vbytes);
  const auto es = make_rsrc(a.ec + (size_t)s * a.Nc, (uint64_t)a.Nc * 4);
  float x3[Q], x4[Q], b[Q], d[R], e[Q / 2];
#pragma unroll
  for (int q = 0; q < Q; ++q) x3[q] = bload(xs, cell_off(t.inx, t.j0 - kMgH + q, ny, nx, t.i));
#pragma unroll
  for (int h = 0; h < Q / 2; ++h) {  // the parents of rows 2h and 2h + 1 (0 off the grid)
    const int j = t.j0 - kMgH + 2 * h;
    e[h] = bload(es, (t.inx && j >= 0 && j < ny) ? (uint32_t)((j >> 1) * a.nxc + (t.i >> 1)) * 4u : kOOB);
  }
#pragma unroll
  for (int q = 1; q < Q - 1; ++q) b[q] = bload(bs, cell_off(t.inx, t.j0 - kMgH + q, ny, nx, t.i));
  float emean = 0.f;
  if (a.coarsest) {
    // minimum-norm coarsest solution: subtract its plain mean (fixed-order sum)
    double sum = 0.0;
    for (int u = threadIdx.x; u < a.nyc; u += kBlock) sum += a.xpart[(size_t)s * a.nyc + u];
    emean = (float)(block_sum(sum, lds) / (double)a.Nc);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = t.j0 - kMgH + q;
    x3[q] += (t.inx && j >= 0 && j < ny) ? e[q / 2] - emean : 0.f;
  }
  x4[0] = x4[Q - 1] = 0.f;
#pragma unroll
  for (int q = 1; q < Q - 1; ++q) {
    const float dd = (b[q] - t.apply(x3, q)) * t.dinv(q) * a.k.inv_theta;
    x4[q] = x3[q] + dd;
    if (q >= kMgH && q < kMgH + R) d[q - kMgH] = dd;
  }
  const auto ys = make_rsrc(a.y + off, vbytes);
  double rz = 0.0;
#pragma unroll
  for (int q = kMgH; q < kMgH + R; ++q) {
    const float x5 = x4[q] + a.k.c1 * d[q - kMgH] + a.k.c2 * t.dinv(q) * (b[q] - t.apply(x4, q));
    const uint32_t o = cell_off(t.own, t.j0 - kMgH + q, ny, nx, t.i);
    bstore(ys, o, x5);
    if (o != kOOB) rz += (double)b[q] * (double)x5;
  }
  if (a.rzpart) {
    rz = block_sum(rz, lds);
    if (threadIdx.x == 0) a.rzpart[(size_t)s * a.P + block_linear()] = rz;
  }
}

// r.z partial sums when the fine level is itself the coarsest (one level).
template <int R>
__global__ __launch_bounds__(kBlock) void k_mg_rz(LevelArgs a) {
  __shared__ double lds[kWaves];
  const int s = blockIdx.z, nx = a.c.nx, ny = a.c.ny;
  if (a.flags[s] != DONE_NO) return;
  const size_t off = (size_t)s * a.N;
  const uint64_t vbytes = (uint64_t)a.N * 4;
  const TileXY tl = tile_xy(nx, ny, R);
  const ColIdx ci = col_idx(nx, tl);
  const int j0 = tl.j0;
  float bv[R], xv[R];
  load_rows_own<R>(make_rsrc(a.b + off, vbytes), nx, ny, j0, ci, bv);
  load_rows_own<R>(make_rsrc(a.x + off, vbytes), nx, ny, j0, ci, xv);
  double rz = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) rz += (double)bv[q] * (double)xv[q];
  rz = block_sum(rz, lds);
  if (threadIdx.x == 0) a.rzpart[(size_t)s * a.P + block_linear()] = rz;
}

namespace {
struct CoarseArgs {
  int nxc, nyc;
  int64_t Nc;
  const float* b;        // [nb][Nc]
  float* x;              // [nb][Nc]
  const double* phi;     // [nxc][nxc]
  const double* phiT;    // [nxc][nxc]
  const double* psi;     // [nyc][nyc]
  const double* psiT;    // [nyc][nyc]
  const double* dinv;    // [nyc][nxc]
  double* bh;            // [nb][nyc][nxc]
  const double* bpart;   // [nb][bP] or NULL
  int bP;
  double* xpart;         // [nb][nyc]
  const int32_t* flags;
};
}  // namespace

// sum_q M[q * ld + j] v[q] for q < n (v in LDS), accumulated in q order.
// The matrix loads of 32 terms are issued together before their products, so
// the sum waits for the L2 once per 32 terms instead of once per few.
__device__ __forceinline__ double dot_strided(const double* __restrict__ M, int ld, int j, const double* v, int n) {
  constexpr int B = 32;
  double acc = 0.0;
  int q0 = 0;
  for (; q0 + B <= n; q0 += B) {
    double m[B];
#pragma unroll
    for (int u = 0; u < B; ++u) m[u] = M[(size_t)(q0 + u) * ld + j];
#pragma unroll
    for (int u = 0; u < B; ++u) acc += m[u] * v[q0 + u];
  }
  for (; q0 < n; ++q0) acc += M[(size_t)q0 * ld + j] * v[q0];
  return acc;
}

// Row transform of the coarsest right-hand side (its mean removed):
// bh[j][k] = sum_i phi[i][k] b[j][i]; one workgroup per row.
__global__ __launch_bounds__(kBlock) void k_mg_cfwd(CoarseArgs a) {
  extern __shared__ double row[];
  __shared__ double lds[kWaves];
  const int s = blockIdx.z, j = blockIdx.x;
  if (a.flags[s] != DONE_NO) return;
  double mean = 0.0;
  if (a.bpart) mean = reduce_partials(a.bpart + (size_t)s * a.bP, a.bP, lds) / (double)a.Nc;
  const float* b = a.b + (size_t)s * a.Nc + (size_t)j * a.nxc;
  for (int i = threadIdx.x; i < a.nxc; i += kBlock) row[i] = (double)b[i] - mean;
  __syncthreads();
  double* out = a.bh + (size_t)s * a.Nc + (size_t)j * a.nxc;
  for (int k = threadIdx.x; k < a.nxc; k += kBlock) out[k] = dot_strided(a.phi, a.nxc, k, row, a.nxc);
}

// Column k of the transformed right-hand side: forward transform along y
// (bh[j][k] <- sum_j' psi[j'][j] bh[j'][k]), division by lam_k + mu_j, and the
// inverse transform along y (bh[j][k] <- sum_j' psi[j][j'] c[j'][k]); one
// workgroup per column, in place (no other workgroup touches the column).
__global__ __launch_bounds__(kBlock) void k_mg_ccol(CoarseArgs a) {
  extern __shared__ double col[];  // [2][nyc]
  const int s = blockIdx.z, k = blockIdx.x;
  if (a.flags[s] != DONE_NO) return;
  const int n = a.nyc, m = a.nxc;
  double* c = a.bh + (size_t)s * a.Nc + k;
  double* t = col;
  double* u = col + n;
  for (int j = threadIdx.x; j < n; j += kBlock) t[j] = c[(size_t)j * m];
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += kBlock) u[j] = dot_strided(a.psi, n, j, t, n) * a.dinv[(size_t)j * m + k];
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += kBlock) c[(size_t)j * m] = dot_strided(a.psiT, n, j, u, n);
}

// Back-transform x[j][i] = sum_k phi[i][k] c[j][k] and the row sums of x (the
// fine level's prolongation removes the mean); one workgroup per row.
__global__ __launch_bounds__(kBlock) void k_mg_cbwd(CoarseArgs a) {
  extern __shared__ double row[];
  __shared__ double lds[kWaves];
  const int s = blockIdx.z, j = blockIdx.x;
  if (a.flags[s] != DONE_NO) return;
  const double* c = a.bh + (size_t)s * a.Nc + (size_t)j * a.nxc;
  for (int k = threadIdx.x; k < a.nxc; k += kBlock) row[k] = c[k];
  __syncthreads();
  float* x = a.x + (size_t)s * a.Nc + (size_t)j * a.nxc;
  double sum = 0.0;
  for (int i = threadIdx.x; i < a.nxc; i += kBlock) {
    const double acc = dot_strided(a.phiT, a.nxc, i, row, a.nxc);
    x[i] = (float)acc;
    sum += (double)(float)acc;
  }
  sum = block_sum(sum, lds);
  if (threadIdx.x == 0) a.xpart[(size_t)s * a.nyc + j] = sum;
}

// The coarsest solve for axes of at most kMgSmall cells (a 1024 x 1024 grid at
// four levels has 128 x 128) and few right-hand sides (mg_two_launches): two launches in
// place of the three above. What
// bounds it is the latency of its chain of dense transforms, so every matrix
// value is loaded before the first product needs one: thread (j, part) keeps the
// rows [32 part, 32 part + 32) of each transform's column j in registers, the
// four parts of a sum meet in LDS, and only LDS traffic is left between the
// transforms. The three launches waited on the L2 four times per transform
// with half of their threads idle: 19.1 us at 128 x 128, against 7.7 + 6.0 us here.
// (On FP64 matrix cores, 16 modes per workgroup, the same work took 39 us: eight
// compute units then load all of the matrices.)
//
// The line at 128 cells is this layout's: four parts of 32 rows of two FP64 matrices are 128
// registers of each of 512 threads. An axis of 129 to 256 cells would take twice the rows (more
// registers than a thread of such a workgroup has) or twice the threads (the most a workgroup has, at half
// the registers each), so it keeps the three launches.
constexpr int kMgSmall = 128;
constexpr int kMgParts = 4;
constexpr int kMgPer = kMgSmall / kMgParts;  // matrix rows per thread
constexpr int kMgCB = kMgSmall * kMgParts;   // threads of a workgroup

// Rows q0 .. q0 + 31 of column j of the n x n matrix M (0 outside).
__device__ __forceinline__ void mg_load_col(const double* __restrict__ M, int n, int j, int q0, double (&v)[kMgPer]) {
  const auto rs = make_rsrc(M, (uint64_t)n * n * 8);
#pragma unroll
  for (int u = 0; u < kMgPer; ++u)
    v[u] = bload64(rs, (j < n && q0 + u < n) ? (uint32_t)((q0 + u) * n + j) * 8u : kOOB);
}

// sum over the parts of sum_u m[u] x[q0 + u] (x in LDS, zero past n), for the
// column of this thread; every thread of the column gets the same bits.
__device__ __forceinline__ double mg_dot_parts(const double (&m)[kMgPer], const double* x, int q0, double* red) {
  double acc = 0.0;
#pragma unroll
  for (int u = 0; u < kMgPer; ++u) acc += m[u] * x[q0 + u];
  __syncthreads();  // the reads of red before this sum are done
  red[threadIdx.x] = acc;
  __syncthreads();
  const int j = threadIdx.x & (kMgSmall - 1);
  return ((red[j] + red[kMgSmall + j]) + red[2 * kMgSmall + j]) + red[3 * kMgSmall + j];
}

// Mode k of all rows (one workgroup per mode): bh[j][k] = the solution's
// coefficients in the eigenbasis of x, psi diag(1 / (lam_k + mu_j)) psi^T
// (b - mean) phi, with b transposed ([nxc][nyc], as k_mg_down leaves it).
__global__ __launch_bounds__(kMgCB) void k_mg_modes(CoarseArgs a) {
  __shared__ double red[kMgCB], x[kMgSmall], lds[kMgCB / kWave];
  const int s = blockIdx.z, k = blockIdx.x, n = a.nyc, m = a.nxc;
  if (a.flags[s] != DONE_NO) return;
  const int t = threadIdx.x, j = t & (kMgSmall - 1), q0 = (t / kMgSmall) * kMgPer;
  const auto bs = make_rsrc(a.b + (size_t)s * a.Nc, (uint64_t)a.Nc * 4);
  float bv[kMgPer];
  double psi[kMgPer], psiT[kMgPer];
#pragma unroll
  for (int u = 0; u < kMgPer; ++u)
    bv[u] = bload(bs, (j < n && q0 + u < m) ? (uint32_t)((q0 + u) * n + j) * 4u : kOOB);
  const double ph = t < m ? a.phiT[(size_t)k * m + t] : 0.0;
  double mean = 0.0;
  for (int u = t; u < a.bP; u += kMgCB) mean += a.bpart[(size_t)s * a.bP + u];
  const double dinv = j < n ? a.dinv[(size_t)j * m + k] : 0.0;
  mg_load_col(a.psi, n, j, q0, psi);
  mg_load_col(a.psiT, n, j, q0, psiT);
  __builtin_amdgcn_sched_barrier(0);  // all loads in flight before the first sum
  mean = wave_sum_dpp(mean);
  if ((t & (kWave - 1)) == 0) lds[t / kWave] = mean;
  if (t < kMgSmall) x[t] = ph;
  __syncthreads();
  mean = 0.0;
#pragma unroll
  for (int w = 0; w < kMgCB / kWave; ++w) mean += lds[w];
  mean /= (double)a.Nc;
  double bd[kMgPer];
#pragma unroll
  for (int u = 0; u < kMgPer; ++u) bd[u] = (double)bv[u] - mean;  // phi is 0 past m
  const double T = mg_dot_parts(bd, x, q0, red);
  if (t < kMgSmall) x[t] = t < n ? T : 0.0;
  __syncthreads();
  const double U = mg_dot_parts(psi, x, q0, red) * dinv;
  if (t < kMgSmall) x[t] = U;  // dinv is 0 past n
  __syncthreads();
  const double V = mg_dot_parts(psiT, x, q0, red);
  if (t < n) a.bh[(size_t)s * a.Nc + (size_t)t * m + k] = V;
}

// Row j of the solution, x[j][i] = sum_k phi[i][k] bh[j][k], and its sum (the
// fine level's prolongation removes the mean); one workgroup per row.
__global__ __launch_bounds__(kMgCB) void k_mg_back(CoarseArgs a) {
  __shared__ double red[kMgCB], c[kMgSmall], lds[kWaves];
  const int s = blockIdx.z, j = blockIdx.x, m = a.nxc;
  if (a.flags[s] != DONE_NO) return;
  const int t = threadIdx.x, i = t & (kMgSmall - 1), q0 = (t / kMgSmall) * kMgPer;
  const double cv = t < m ? a.bh[(size_t)s * a.Nc + (size_t)j * m + t] : 0.0;
  double phiT[kMgPer];
  mg_load_col(a.phiT, m, i, q0, phiT);
  __builtin_amdgcn_sched_barrier(0);
  if (t < kMgSmall) c[t] = cv;
  __syncthreads();
  const float x = (float)mg_dot_parts(phiT, c, q0, red);
  if (t < m) a.x[(size_t)s * a.Nc + (size_t)j * m + t] = x;
  const double sum = wave_sum_dpp(t < m ? (double)x : 0.0);
  if ((t & (kWave - 1)) == 0 && t < kMgSmall) lds[t / kWave] = sum;
  __syncthreads();
  if (t == 0) a.xpart[(size_t)s * a.nyc + j] = lds[0] + lds[1];
}

// ---------------------------------------------------------------------------
#define PPE_MG_DISPATCH(R, ...)                                  \
  switch (R) {                                                   \
    case 2: { constexpr int RR = 2; __VA_ARGS__; } break;        \
    case 4: { constexpr int RR = 4; __VA_ARGS__; } break;        \
    default: { constexpr int RR = 8; __VA_ARGS__; } break;       \
  }

void launch_vcycle(const PcgArgs& pa, int nb, hipStream_t s) {
  const MgData& m = *pa.mg;
  const int L = m.L;
  const Cheb k = cheb_consts();
  // the two-launch coarsest solve reads a transposed right-hand side
  const bool small =
      L > 1 && m.nxc <= kMgSmall && m.nyc <= kMgSmall && mg_two_launches(m.nxc, m.nyc, nb, device_cus());
  auto rows = [&](int l) { return mg_rows((int64_t)m.lv[l].nx * m.lv[l].ny * nb); };
  // level l's arguments; the fine level reads the PCG residual and writes z
  auto level = [&](int l) {
    const MgLevel& v = m.lv[l];
    LevelArgs a{};
    a.c = v.c;
    a.N = (int64_t)v.nx * v.ny;
    a.b = l == 0 ? pa.r : v.b;
    a.x = l == 0 ? m.x0 : v.x;
    a.y = l == 0 ? m.z : v.y;
    a.flags = pa.flags;
    a.k = k;
    if (l + 1 < L) {
      const MgLevel& c = m.lv[l + 1];
      a.bc = c.b;
      a.ec = l + 1 == L - 1 ? c.x : c.y;
      a.nxc = c.nx;
      a.Nc = (int64_t)c.nx * c.ny;
      a.coarsest = l + 1 == L - 1;
      a.bc_t = a.coarsest && small;
      a.bpart = m.bpart;
      a.xpart = m.xpart;
      a.nyc = c.ny;
    }
    a.P = mg_tiles(v.nx, v.ny, rows(l));
    a.rzpart = l == 0 ? m.rzpart : nullptr;
    return a;
  };
  for (int l = 0; l + 1 < L; ++l) {
    const LevelArgs a = level(l);
    PPE_MG_DISPATCH(rows(l), k_mg_down<RR><<<dim3(a.P, 1, nb), kBlock, 0, s>>>(a));
  }
  {
    const MgLevel& c = m.lv[L - 1];
    CoarseArgs ca{};
    ca.nxc = m.nxc;
    ca.nyc = m.nyc;
    ca.Nc = (int64_t)m.nxc * m.nyc;
    ca.b = L == 1 ? pa.r : c.b;
    ca.x = L == 1 ? m.z : c.x;
    ca.phi = m.phi;
    ca.phiT = m.phiT;
    ca.psi = m.psi;
    ca.psiT = m.psiT;
    ca.dinv = m.dinv;
    ca.bh = m.bh;
    ca.bpart = L == 1 ? nullptr : m.bpart;
    ca.bP = L == 1 ? 1 : mg_tiles(m.lv[L - 2].nx, m.lv[L - 2].ny, rows(L - 2));
    ca.xpart = m.xpart;
    ca.flags = pa.flags;
    if (small) {
      k_mg_modes<<<dim3(m.nxc, 1, nb), kMgCB, 0, s>>>(ca);
      k_mg_back<<<dim3(m.nyc, 1, nb), kMgCB, 0, s>>>(ca);
    } else {
      const size_t shm = sizeof(double) * m.nxc;
      k_mg_cfwd<<<dim3(m.nyc, 1, nb), kBlock, shm, s>>>(ca);
      k_mg_ccol<<<dim3(m.nxc, 1, nb), kBlock, sizeof(double) * 2 * m.nyc, s>>>(ca);
      k_mg_cbwd<<<dim3(m.nyc, 1, nb), kBlock, shm, s>>>(ca);
    }
  }
  if (L == 1) {
    LevelArgs a = level(0);
    a.x = m.z;
    const dim3 g = stencil_grid(a.c, rows(0), nb);
    a.P = (int)g.x;
    PPE_MG_DISPATCH(rows(0), k_mg_rz<RR><<<g, kBlock, 0, s>>>(a));
    return;
  }
  for (int l = L - 2; l >= 0; --l) {
    const LevelArgs a = level(l);
    PPE_MG_DISPATCH(rows(l), k_mg_up<RR><<<dim3(a.P, 1, nb), kBlock, 0, s>>>(a));
  }
}

int mg_rz_parts(const MgData& m, int nb) {
  const MgLevel& v = m.lv[0];
  const int R = mg_rows((int64_t)v.nx * v.ny * nb);
  return m.L == 1 ? (int)stencil_grid(v.c, R, 1).x : mg_tiles(v.nx, v.ny, R);
}

int mg_max_parts(const MgLevel& v) { return mg_tiles(v.nx, v.ny, 2); }

}  // namespace ppe
