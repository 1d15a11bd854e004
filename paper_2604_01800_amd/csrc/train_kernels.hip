// Training kernels of the DeepONet: weight gradients on BF16 MFMA (split-K
// over pixels, fixed-order reduction), activation-gradient masks, the
// Mesh-Conv local-weight backward, pooling / upsampling / concatenation
// backward, the DeepONet contraction, the residual loss of Eq. 19, and Adam.
#include <algorithm>

#include "common.hpp"
#include "net_common.hpp"
#include "net_kernels.hpp"
#include "train_kernels.hpp"

namespace ppe {

// ---------------------------------------------------------------------------
// Matrix operands whose K dimension runs over pixels, read from an LDS tile
// that keeps each pixel's channels together: ds_read_b64_tr_b16 gives lane i
// of a 16-lane group the four values that column i of a 4 x 16 block holds,
// where lane j points at the block's row j / 4, columns 4 (j % 4) .. + 3. Two of
// them make the eight consecutive pixels of one MFMA 16x16x32 operand; p0 and
// p1 point at the rows of pixels 0..3 and 4..7 of the lane's group.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

__device__ __forceinline__ bf16x8_t tr_frag(const bf16_t* p0, const bf16_t* p1) {
  const s16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p0);
  const s16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p1);
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Weight gradient of a 3x3 layer:
//   dW[co][ci][tap] = sum over pixels p of dPre[p][co] * Xbar[p + off(tap)][ci]
// with Xbar = eta * X (the layer's weighted input), on MFMA 16x16x32 BF16 with
// A = dPre^T (M = 16 MT output channels, K = pixels) and B = shifted Xbar (N = 16
// input channels). A workgroup of CT wavefronts owns 16 MT output and 16 CT
// input channels, wave w the input channels 16 w .. + 15; one set of B operands
// (nine shifted reads of the staged 8 x 16 pixel tile, halo included) feeds MT
// MFMAs per tap. Split z takes the pixel tiles z, z + nsplit, ... of all
// samples, the next tile's loads in flight during the current one's MFMA loop,
// and leaves a partial row in the parameters' layout [co][ci < cin][tap];
// k_reduce_rows sums the rows in a fixed order. The workgroups of one split run
// on one XCD (they read the same pixels). The order of every sum depends on
// nsplit alone, not on the channel tiles.
//
// Bound by the matrix cores and LDS reads about equally (26 8-byte reads for 36
// MFMAs per K-step with MT = 4). An earlier form kept transposed copies of
// dPre and of three column shifts of Xbar in LDS for a 32 x 32 channel tile:
// ten 16-byte reads for nine MFMAs, and transposes through registers. The 14
// layers of 64 samples of 256 x 256: 7.9 -> 1.8 ms.
template <int MT, int CT, int ETA>
__global__ __launch_bounds__(64 * CT) __attribute__((amdgpu_waves_per_eu(2))) void k_wgrad9(
    WgradGeo g, const bf16_t* __restrict__ dp, const bf16_t* __restrict__ x, const bf16_t* __restrict__ eta,
    float* __restrict__ part, int nbx, int nblk, int nsplit) {
  constexpr int TH = 8, TW = 16, LW = TW + 2, NPX = (TH + 2) * LW;
  constexpr int CO = 16 * MT, CI = 16 * CT, NT = 64 * CT;
  // LDS pitches (bf16): four consecutive pixels' 32-byte pieces in distinct banks
  constexpr int XP = CI == 16 ? 16 : CI + 16, DP = CO + 16;
  constexpr int GX = CI / 8, GD = CO / 8;  // 8-channel groups of a staged pixel
  constexpr int NX = (NPX * GX + NT - 1) / NT, ND = (TH * TW * GD + NT - 1) / NT;
  __shared__ __attribute__((aligned(16))) bf16_t s_x[NPX * XP];
  __shared__ __attribute__((aligned(16))) bf16_t s_d[TH * TW * DP];
  // workgroup -> (split, channel block): workgroup b runs on XCD b % 8, so
  // within groups of eight splits the blocks of a split are eight apart
  const int b = blockIdx.x, full = nsplit / 8 * 8 * nblk;
  int split, blk;
  if (b < full) {
    split = (b & 7) + 8 * ((b >> 3) / nblk);
    blk = (b >> 3) % nblk;
  } else {
    split = nsplit / 8 * 8 + (b - full) / nblk;
    blk = (b - full) % nblk;
  }
  const int co0 = (blk % nbx) * CO, ci0 = (blk / nbx) * CI;
  const int tiles_x = (g.W + TW - 1) / TW, tiles_y = (g.H + TH - 1) / TH;
  const int per = tiles_x * tiles_y, tiles = per * g.nb;
  const int lane = threadIdx.x & 63, ct = threadIdx.x >> 6;

  f32x4_t acc[9][MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  uint4 vx[NX], vd[ND], ve[ETA == kEtaChannel ? NX : 1];
  uint32_t ve1[ETA == kEtaNode ? NX : 1];
  auto issue = [&](int t) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // the lane's offsets are recomputed per tile rather than kept in registers
    const int smp = t / per, rem = t - smp * per;
    const int py0 = (rem / tiles_x) * TH, px0 = (rem % tiles_x) * TW;
    // resources based at the tile's first (halo) pixel: lanes outside the
    // image or the channels get an offset past the end and read 0
    const int64_t hp = (int64_t)(py0 - 1) * g.W + px0 - 1, pp = (int64_t)py0 * g.W + px0;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(x + smp * g.x_bstride + hp * g.cin8), (short)0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(dp + smp * g.dp_bstride + pp * g.dp_pitch), (short)0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t er = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(ETA != kEtaNone ? eta + smp * g.e_bstride + hp * (ETA == kEtaChannel ? g.cin8 : 1) : x),
        (short)0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int u = tid + NT * i, px = u / GX, c = ci0 + (u - px * GX) * 8;
      const int ly = px / LW, lx = px - ly * LW, gy = py0 + ly - 1, gx = px0 + lx - 1;
      const bool ok = px < NPX && gy >= 0 && gy < g.H && gx >= 0 && gx < g.W && c < g.cin8;
      const uint32_t rel = (uint32_t)(ly * g.W + lx);
      const uint32_t o = ok ? (rel * (uint32_t)g.cin8 + (uint32_t)c) * 2u : 0x80000000u;
      vx[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)o, 0, 0));
      if constexpr (ETA == kEtaChannel)
        ve[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(er, (int)o, 0, 0));
      if constexpr (ETA == kEtaNode)
        ve1[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(er, (int)(ok ? rel * 2u : 0x80000000u), 0, 0);
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int u = tid + NT * i, px = u / GD, c = co0 + (u - px * GD) * 8;
      const int ly = px / TW, lx = px - ly * TW;
      const bool ok = px < TH * TW && py0 + ly < g.H && px0 + lx < g.W && c < g.cout;
      const uint32_t o = ok ? ((uint32_t)(ly * g.W + lx) * (uint32_t)g.dp_pitch + (uint32_t)c) * 2u : 0x80000000u;
      vd[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(dr, (int)o, 0, 0));
    }
  };
  auto commit = [&]() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int u = tid + NT * i, px = u / GX, c8 = u - px * GX;
      uint4 v = vx[i];
      if constexpr (ETA == kEtaChannel) v = mul_bf16x8(v, ve[i]);
      if constexpr (ETA == kEtaNode) v = mul_bf16x8_s(v, ve1[i]);
      if (px < NPX) *(uint4*)(s_x + px * XP + c8 * 8) = v;
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      const int u = tid + NT * i, px = u / GD, c8 = u - px * GD;
      if (px < TH * TW) *(uint4*)(s_d + px * DP + c8 * 8) = vd[i];
    }
  };
  // this lane's rows of the transposed reads: group q = lane / 16 holds the
  // K-step's pixels 8 q .. 8 q + 7 (tile row q / 2, columns 8 (q % 2) ..)
  const int q = lane >> 4, jr = (lane & 15) >> 2, jc = 4 * (lane & 3);
  const bf16_t* ad = s_d + ((q >> 1) * TW + 8 * (q & 1) + jr) * DP + jc;
  const bf16_t* ax = s_x + ((q >> 1) * LW + 8 * (q & 1) + jr) * XP + ct * 16 + jc;

  if (split < tiles) issue(split);
  for (int t = split; t < tiles; t += nsplit) {
    __syncthreads();  // the previous tile's MFMA loop is done with LDS
    commit();
    __syncthreads();
    if (t + nsplit < tiles) issue(t + nsplit);
#pragma unroll
    for (int st = 0; st < 4; ++st) {  // tile rows 2 st, 2 st + 1
      const bf16_t* pd = ad + st * 2 * TW * DP;
      const bf16_t* px = ax + st * 2 * LW * XP;
      bf16x8_t af[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m) af[m] = tr_frag(pd + m * 16, pd + 4 * DP + m * 16);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const int o = (tap / 3 * LW + tap % 3) * XP;
        const bf16x8_t bf = tr_frag(px + o, px + o + 4 * XP);
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[tap][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[m], bf, acc[tap][m], 0, 0, 0);
      }
    }
  }
  // lane holds dW[co0 + 16 m + 4 (lane >> 4) + j][ci0 + 16 ct + (lane & 15)] per tap
  const int ci = ci0 + ct * 16 + (lane & 15);
  if (ci >= g.cin) return;
  float* ps = part + (int64_t)split * g.cout * g.cin * 9;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int co = co0 + m * 16 + 4 * (lane >> 4) + j;
      if (co >= g.cout) continue;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) ps[((int64_t)co * g.cin + ci) * 9 + tap] = acc[tap][m][j];
    }
}

__device__ __forceinline__ void transpose8x8_bf16(const uint4 (&v)[8], uint4 (&w)[8]) {
  // v[r] holds channels 0..7 of pixel r; w[e] receives pixels 0..7 of channel e
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 a4 = v[2 * j], b4 = v[2 * j + 1];
      const uint32_t a = (e / 2 == 0) ? a4.x : (e / 2 == 1) ? a4.y : (e / 2 == 2) ? a4.z : a4.w;
      const uint32_t b = (e / 2 == 0) ? b4.x : (e / 2 == 1) ? b4.y : (e / 2 == 2) ? b4.z : b4.w;
      o[j] = (e & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
    }
    w[e] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// Weight gradient of a 1x1 layer, dW[co][ci] = sum over pixels p of
// dPre[p][co] * X[p][ci], on MFMA 16x16x32 BF16 with A = dPre^T (M = output
// channels, K = pixels) and B = X (N = input channels). A workgroup owns a
// 128 x 128 (co, ci) tile, so every pixel's data is read once per tile; wave
// w computes the 64 x 64 quarter (w / 2, w % 2) as 4 x 4 MFMA tiles. The
// pixels are taken in stages of 64 (within one sample), stages z, z + nsplit,
// ... for split z. Per stage, thread t < 128 loads an 8-pixel x 8-channel
// block of dPre and thread t >= 128 one of X (coalesced 16-byte loads along
// the channels), transposes it in registers and writes it to LDS as 16-byte
// rows [channel][8 pixels]; the next stage's loads are issued before the
// current stage's MFMA loop. The partial sums are written in the layout
// [co][ci < cin] of the split's row; k_reduce_rows sums the splits in a
// fixed order.
constexpr int kW1T = 128;          // output and input channels per workgroup
constexpr int kW1P = 64;           // pixels per stage
constexpr int kW1PP = kW1P + 8;    // LDS pitch (bf16) of a channel row

__global__ __launch_bounds__(256) void k_wgrad1(WgradGeo g, const bf16_t* __restrict__ dp,
                                                const bf16_t* __restrict__ x, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) bf16_t s_dp[kW1T * kW1PP];
  __shared__ __attribute__((aligned(16))) bf16_t s_x[kW1T * kW1PP];
  const int co0 = blockIdx.x * kW1T, ci0 = blockIdx.y * kW1T;
  const int split = blockIdx.z, nsplit = gridDim.z;
  const int npix = g.H * g.W;
  const int sps = (npix + kW1P - 1) / kW1P;  // stages per sample
  const int stages = sps * g.nb;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  // staging role: operand (0 = dPre, 1 = X), channel group and pixel octet
  const int which = t >> 7, oct = t & 7, cg = (t >> 3) & 15;
  const int ch = (which ? ci0 : co0) + cg * 8;
  const bool ch_ok = which ? ch < g.cin8 : ch < g.cout;
  const int pitch = which ? g.cin8 : g.dp_pitch;
  const bf16_t* src = which ? x : dp;
  const int64_t bstride = which ? g.x_bstride : g.dp_bstride;
  bf16_t* dst = (which ? s_x : s_dp) + (cg * 8) * kW1PP + oct * 8;

  f32x4_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  uint4 v[8];
  auto issue = [&](int st) {
    const int smp = st / sps, p0 = (st - smp * sps) * kW1P + oct * 8;
    const bf16_t* b = src + smp * bstride + ch;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      v[r] = make_uint4(0, 0, 0, 0);
      if (ch_ok && p0 + r < npix) v[r] = *(const uint4*)(b + (int64_t)(p0 + r) * pitch);
    }
  };
  if (split < stages) issue(split);
  for (int st = split; st < stages; st += nsplit) {
    __syncthreads();  // the previous stage's MFMA loop is done with LDS
    {
      uint4 w[8];
      transpose8x8_bf16(v, w);
#pragma unroll
      for (int e = 0; e < 8; ++e) *(uint4*)(dst + e * kW1PP) = w[e];
    }
    __syncthreads();
    if (st + nsplit < stages) issue(st + nsplit);
#pragma unroll
    for (int ks = 0; ks < kW1P / 32; ++ks) {
      const int k = ks * 32 + (lane >> 4) * 8;
      bf16x8_t af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) af[i] = *(const bf16x8_t*)(s_dp + (wm * 64 + i * 16 + (lane & 15)) * kW1PP + k);
#pragma unroll
      for (int j = 0; j < 4; ++j) bf[j] = *(const bf16x8_t*)(s_x + (wn * 64 + j * 16 + (lane & 15)) * kW1PP + k);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
    }
  }
  // lane holds dW[co0 + 64 wm + 16 i + 4 (lane >> 4) + q][ci0 + 64 wn + 16 j + (lane & 15)]
  float* ps = part + (int64_t)split * g.cout * g.cin;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ci = ci0 + wn * 64 + j * 16 + (lane & 15);
    if (ci >= g.cin) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int co = co0 + wm * 64 + i * 16 + 4 * (lane >> 4) + q;
        if (co < g.cout) ps[(int64_t)co * g.cin + ci] = acc[i][j][q];
      }
  }
}

// Whole backward of a 1x1 layer of at most 128 output and input channels (the
// trunk, the head, the narrow up-convolutions) in one pass over its pixels:
//   dW[co][ci] = sum_p d[p][co] x[p][ci],
//   dx[p][ci]  = act'(x[p][ci]) * bf16(sum_co W[co][ci] d[p][co]),
// where x is the layer's input and act' the derivative of the activation that
// made it (1 for ReLU where x > 0, 1 - x^2 for tanh). d is read, or formed
// from the DeepONet contraction y = gamma sum_k B_k T_k: d = bf16(gamma dy S)
// with S the other factor (T for the head, B for the trunk output).
// Stages of 64 pixels: d and x go to LDS as they lie in memory (channels of a
// pixel together). dW takes both operands by transposed reads (K = pixels;
// wave w the quarter (w / 2, w % 2) of the channel square), dx takes d's rows
// as they are and the weights from LDS (wave w the pixels 16 w ..); its result
// replaces d in LDS and leaves as whole 16-byte pieces. The next stage's loads are in flight
// meanwhile.
// 768 B per pixel at 128 channels (d and x read, dx written) where separate launches for
// dW, dx and act' moved 1.8 KB. At 4.2 M pixels a 128 x 128 layer takes 766 us
// (4.3 TB/s; a large copy reaches 5.1) against 286 + 385 + 420. Bound by the barriers of
// a stage (four, 64 pixels apart) and its loads: the wavefronts wait about half of their
// cycles, MFMA busy is 15 %. The bias gradient is a launch of its own (k_bias_grad).
constexpr int kB1P = 64;     // pixels per stage
constexpr int kB1C = 128;    // channels at most
constexpr int kB1DP = kB1C + 16;  // LDS pitch (bf16) of a pixel: see k_wgrad9
constexpr int kB1WP = kB1C + 8;   // LDS pitch of a weight row
enum { kActNone = 0, kActRelu = 1, kActTanh = 2 };

__device__ __forceinline__ uint4 scale8(uint4 a, float c) {
  const uint32_t x[4] = {a.x, a.y, a.z, a.w};
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    o[e] = (uint32_t)f2bf(c * bf2f((bf16_t)(x[e] & 0xffff))) | ((uint32_t)f2bf(c * bf2f((bf16_t)(x[e] >> 16))) << 16);
  return make_uint4(o[0], o[1], o[2], o[3]);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_bwd1x1(Bwd1x1 g,
                                                                                        float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) bf16_t s_d[kB1P * kB1DP];
  __shared__ __attribute__((aligned(16))) bf16_t s_x[kB1P * kB1DP];
  __shared__ __attribute__((aligned(16))) bf16_t s_w[kB1C * kB1WP];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = wv >> 1, wn = wv & 1;
  const int cout = g.cout, cin8 = g.cin8;
  const int nks = (cout + 31) / 32;
  const int sps = (g.hw + kB1P - 1) / kB1P;  // stages per sample
  const int stages = sps * g.nb;
  // channels past cout or cin8 that the products read are zero for the whole launch
  for (int u = tid; u < kB1P * kB1DP / 8; u += 256) {
    *(uint4*)(s_d + u * 8) = make_uint4(0, 0, 0, 0);
    *(uint4*)(s_x + u * 8) = make_uint4(0, 0, 0, 0);
  }
  if (g.dx) {
    const int kq = g.Kp / 8;
    for (int u = tid; u < kB1C * kq; u += 256) {
      const int r = u / kq, q = u - r * kq;
      *(uint4*)(s_w + r * kB1WP + q * 8) =
          r < cin8 ? *(const uint4*)(g.wT + (int64_t)r * g.Kp + q * 8) : make_uint4(0, 0, 0, 0);
    }
  }
  f32x4_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // staging: thread t holds the 8-channel group t % 16 of pixels t / 16 + 16 i
  const int c8 = (tid & 15) * 8, pl = tid >> 4;
  const bool dch = c8 < cout, xch = c8 < cin8;
  const float gam = g.gamma ? g.gamma[0] : 0.f;
  uint4 vd[4], vx[4];
  float vg[4];
  int left = 0;  // pixels of the stage in flight
  int64_t pst = 0;  // its first pixel
  auto issue = [&](int st) {
    const int smp = st / sps, k0 = (st - smp * sps) * kB1P;
    const int64_t p0 = (int64_t)smp * g.hw + k0;
    pst = p0;
    left = min(kB1P, g.hw - k0);
    const bf16_t* db = g.d + p0 * cout + c8;
    const bf16_t* xb = g.x + p0 * cin8 + c8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = pl + 16 * i;
      const bool ok = q < left;
      vd[i] = make_uint4(0, 0, 0, 0);
      vx[i] = make_uint4(0, 0, 0, 0);
      vg[i] = 0.f;
      if (ok && dch) vd[i] = *(const uint4*)(db + q * cout);
      if (ok && xch) vx[i] = *(const uint4*)(xb + q * cin8);
      if (ok && g.gamma) vg[i] = g.dy[p0 + q];
    }
  };
  // transposed reads of a K-step of 32 pixels: group lane / 16 holds pixels
  // 8 (lane / 16) .. + 7
  const int jr = (lane & 15) >> 2, jc = 4 * (lane & 3);
  const bf16_t* td = s_d + (8 * (lane >> 4) + jr) * kB1DP + jc + wm * 64;
  const bf16_t* tx = s_x + (8 * (lane >> 4) + jr) * kB1DP + jc + wn * 64;
  const bf16_t* wrow = s_w + (lane & 15) * kB1WP + (lane >> 4) * 8;
  bf16_t* drow = s_d + (16 * wv + (lane & 15)) * kB1DP;
  const bf16_t* xrow = s_x + (16 * wv + (lane & 15)) * kB1DP;

  if ((int)blockIdx.x < stages) issue(blockIdx.x);
  for (int st = blockIdx.x; st < stages; st += gridDim.x) {
    const int np = left;
    const int64_t p0 = pst;
    __syncthreads();  // the stage before has left LDS
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = pl + 16 * i;
      if (dch) *(uint4*)(s_d + q * kB1DP + c8) = g.gamma ? scale8(vd[i], gam * (g.scale * vg[i])) : vd[i];
      if (xch) *(uint4*)(s_x + q * kB1DP + c8) = vx[i];
    }
    __syncthreads();
    if (st + (int)gridDim.x < stages) issue(st + gridDim.x);
#pragma unroll
    for (int ks = 0; ks < kB1P / 32; ++ks) {
      bf16x8_t af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bf16_t* a = td + ks * 32 * kB1DP + i * 16;
        const bf16_t* b = tx + ks * 32 * kB1DP + i * 16;
        af[i] = tr_frag(a, a + 4 * kB1DP);
        bf[i] = tr_frag(b, b + 4 * kB1DP);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (wm * 64 + i * 16 >= cout) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (wn * 64 + j * 16 < cin8)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
    }
    if (!g.dx) continue;
    uint2 res[8];
    {
      f32x4_t ad[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) ad[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < kB1C / 32; ++ks) {
        if (ks >= nks) break;
        const bf16x8_t bf = *(const bf16x8_t*)(drow + ks * 32 + (lane >> 4) * 8);
#pragma unroll
        for (int m = 0; m < 8; ++m)
          if (m * 16 < cin8)
            ad[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const bf16x8_t*)(wrow + m * 16 * kB1WP + ks * 32), bf,
                                                            ad[m], 0, 0, 0);
      }
      // lane holds dx[pixel 16 wv + (lane & 15)][ci = 16 m + 4 (lane >> 4) + j]
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const uint2 xv = *(const uint2*)(xrow + m * 16 + 4 * (lane >> 4));
        const float o[4] = {bf2f((bf16_t)(xv.x & 0xffff)), bf2f((bf16_t)(xv.x >> 16)), bf2f((bf16_t)(xv.y & 0xffff)),
                            bf2f((bf16_t)(xv.y >> 16))};
        bf16_t r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          r[j] = f2bf(ad[m][j]);
          if (g.act == kActRelu) r[j] = o[j] > 0.f ? r[j] : (bf16_t)0;
          else if (g.act == kActTanh) r[j] = f2bf(bf2f(r[j]) * (1.f - o[j] * o[j]));
        }
        res[m] = make_uint2((uint32_t)r[0] | ((uint32_t)r[1] << 16), (uint32_t)r[2] | ((uint32_t)r[3] << 16));
      }
    }
    __syncthreads();  // every wave is done with d
#pragma unroll
    for (int m = 0; m < 8; ++m)
      if (m * 16 < cin8) *(uint2*)(drow + m * 16 + 4 * (lane >> 4)) = res[m];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = pl + 16 * i;
      if (xch && q < np) *(uint4*)(g.dx + (p0 + q) * cin8 + c8) = *(const uint4*)(s_d + q * kB1DP + c8);
    }
    if (cin8 > cout) {
      // d's columns past cout are zero again before the next stage's products
      __syncthreads();
      for (int u = tid; u < kB1P * ((cin8 - cout) / 8); u += 256) {
        const int w = (cin8 - cout) / 8, r = u / w;
        *(uint4*)(s_d + r * kB1DP + cout + (u - r * w) * 8) = make_uint4(0, 0, 0, 0);
      }
    }
  }
  // lane holds dW[co = 64 wm + 16 i + 4 (lane >> 4) + q][ci = 64 wn + 16 j + (lane & 15)]
  float* ps = part + (int64_t)blockIdx.x * cout * g.cin;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int co = wm * 64 + i * 16 + 4 * (lane >> 4) + q;
      if (co >= cout) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int ci = wn * 64 + j * 16 + (lane & 15);
        if (ci < g.cin) ps[(int64_t)co * g.cin + ci] = acc[i][j][q];
      }
    }
}

// out[k] = scale * sum_b part[b][k] (fixed order, FP64 accumulation). A
// workgroup handles 32 consecutive k; its 8 thread groups sum the rows
// g, g + 8, ... and the 8 group sums are added in order.
__global__ __launch_bounds__(256) void k_reduce_rows(const float* __restrict__ part, int nparts, int64_t len,
                                                     float scale, float* __restrict__ out) {
  __shared__ double red[8][32];
  const int kk = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int64_t k = (int64_t)blockIdx.x * 32 + kk;
  // rows g, g + 8, ... in four interleaved partial sums (their loads in
  // flight together), added in a fixed order
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  if (k < len) {
    int b = g;
    for (; b + 24 < nparts; b += 32) {
      s0 += part[(int64_t)b * len + k];
      s1 += part[(int64_t)(b + 8) * len + k];
      s2 += part[(int64_t)(b + 16) * len + k];
      s3 += part[(int64_t)(b + 24) * len + k];
    }
    for (; b < nparts; b += 8) s0 += part[(int64_t)b * len + k];
  }
  const double s = (s0 + s1) + (s2 + s3);
  red[g][kk] = s;
  __syncthreads();
  if (g == 0 && k < len) {
    double tot = 0.0;
    for (int q = 0; q < 8; ++q) tot += red[q][kk];
    out[k] = (float)(scale * tot);
  }
}

// The same sums for several arrays in one launch: blockIdx.y the table's entry.
__global__ __launch_bounds__(256) void k_reduce_table(RowTable t) {
  __shared__ double red[8][32];
  const RowSum& r = t.row[blockIdx.y];
  if ((int)blockIdx.x * 32 >= r.len) return;
  const int kk = threadIdx.x & 31, g = threadIdx.x >> 5, k = blockIdx.x * 32 + kk;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  if (k < r.len) {
    int b = g;
    for (; b + 24 < r.nparts; b += 32) {
      s0 += r.part[(int64_t)b * r.len + k];
      s1 += r.part[(int64_t)(b + 8) * r.len + k];
      s2 += r.part[(int64_t)(b + 16) * r.len + k];
      s3 += r.part[(int64_t)(b + 24) * r.len + k];
    }
    for (; b < r.nparts; b += 8) s0 += r.part[(int64_t)b * r.len + k];
  }
  red[g][kk] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (g == 0 && k < r.len) {
    double tot = 0.0;
    for (int q = 0; q < 8; ++q) tot += red[q][kk];
    r.out[k] = (float)tot;
  }
}

void launch_reduce_table(const RowTable& t, hipStream_t s) {
  int len = 1;
  for (int k = 0; k < t.n; ++k) len = std::max(len, t.row[k].len);
  k_reduce_table<<<dim3((len + 31) / 32, t.n), 256, 0, s>>>(t);
}

// Bias gradient partials: part[b][c] = sum over workgroup b's pixels of d[p][c].
// Thread t reads 8 channels (c8 = t % (C/8)) of the pixels of phase t / (C/8);
// the phases are summed in LDS in a fixed order. Requires C % 8 == 0, C <= 2048.
// With gamma, d holds a factor S of the DeepONet contraction and the summed
// gradient is bf16(gamma (scale dy) S).
__global__ __launch_bounds__(256) void k_bias_grad(const bf16_t* __restrict__ d, int64_t npix, int pitch, int off,
                                                   int C, const float* __restrict__ gamma,
                                                   const float* __restrict__ dy, float scale,
                                                   float* __restrict__ part) {
  __shared__ float red[256 * 8];
  const int c8n = C / 8;
  const int G = 256 / c8n;  // pixel phases per workgroup
  const int t = threadIdx.x;
  const int c8 = t % c8n, g = t / c8n;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (g < G) {
    // four pixels' loads in flight per thread
    const int64_t step = (int64_t)gridDim.x * G;
    for (int64_t p = (int64_t)blockIdx.x * G + g; p < npix; p += 4 * step) {
      uint4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t pu = p + u * step;
        v[u] = pu < npix ? *(const uint4*)(d + pu * pitch + off + c8 * 8) : make_uint4(0, 0, 0, 0);
        if (gamma && pu < npix) v[u] = scale8(v[u], gamma[0] * (scale * dy[pu]));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t w4[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[2 * e] += bf2f((bf16_t)(w4[e] & 0xffff));
          acc[2 * e + 1] += bf2f((bf16_t)(w4[e] >> 16));
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[t * 8 + e] = acc[e];
  __syncthreads();
  for (int c = t; c < C; c += 256) {
    float sacc = 0.f;
    for (int gg = 0; gg < G; ++gg) sacc += red[(gg * c8n + c / 8) * 8 + (c % 8)];
    part[(int64_t)blockIdx.x * C + c] = sacc;
  }
}

// In-place activation backward: d *= relu'(out) (mode 1) or tanh'(out) (mode 2).
// Eight channels per thread (C, pitches and offsets are multiples of 8).
__global__ void k_act_bwd(bf16_t* __restrict__ d, int dpitch, const bf16_t* __restrict__ out, int opitch, int ooff,
                          int C, int64_t npix, int mode) {
  const int c8n = C / 8;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= npix * c8n) return;
  const int64_t p = idx / c8n;
  const int c = (int)(idx - p * c8n) * 8;
  uint4* dp = (uint4*)(d + p * dpitch + c);
  const uint4 dv = *dp, ov = *(const uint4*)(out + p * opitch + ooff + c);
  const uint32_t a[4] = {dv.x, dv.y, dv.z, dv.w}, b[4] = {ov.x, ov.y, ov.z, ov.w};
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo = bf2f((bf16_t)(a[e] & 0xffff)), hi = bf2f((bf16_t)(a[e] >> 16));
    const float olo = bf2f((bf16_t)(b[e] & 0xffff)), ohi = bf2f((bf16_t)(b[e] >> 16));
    if (mode == 1) {
      lo = olo > 0.f ? lo : 0.f;
      hi = ohi > 0.f ? hi : 0.f;
    } else {
      lo *= 1.f - olo * olo;
      hi *= 1.f - ohi * ohi;
    }
    o[e] = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
  }
  *dp = make_uint4(o[0], o[1], o[2], o[3]);
}

// dst[p][c] = src[p][soff + c], c < C; eight channels per thread.
__global__ void k_copy_ch(const bf16_t* __restrict__ src, int spitch, int soff, bf16_t* __restrict__ dst, int dpitch,
                          int C, int64_t npix) {
  const int c8n = C / 8;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= npix * c8n) return;
  const int64_t p = idx / c8n;
  const int c = (int)(idx - p * c8n) * 8;
  *(uint4*)(dst + p * dpitch + c) = *(const uint4*)(src + p * spitch + soff + c);
}

// Backward of nearest 2x upsampling: coarse[p][c] = sum of the 4 fine pixels,
// eight channels per thread (C a multiple of 8).
__global__ void k_up_bwd(int Hc, int Wc, int C, const bf16_t* __restrict__ fine, int fpitch, int64_t f_bs,
                         bf16_t* __restrict__ coarse, int64_t c_bs) {
  const int c8n = C / 8;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)Hc * Wc * c8n) return;
  const int64_t p = idx / c8n;
  const int c = (int)(idx - p * c8n) * 8;
  const int y = (int)(p / Wc), xx = (int)(p - (int64_t)y * Wc);
  const bf16_t* f = fine + blockIdx.y * f_bs + c;
  uint4 v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    v[q] = *(const uint4*)(f + ((int64_t)(2 * y + (q >> 1)) * 2 * Wc + 2 * xx + (q & 1)) * fpitch);
  uint32_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float lo = 0.f, hi = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t w4[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
      lo += bf2f((bf16_t)(w4[e] & 0xffff));
      hi += bf2f((bf16_t)(w4[e] >> 16));
    }
    o[e] = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
  }
  *(uint4*)(coarse + blockIdx.y * c_bs + p * C + c) = make_uint4(o[0], o[1], o[2], o[3]);
}

// Backward of 2x2 average pooling into the features' gradient, and through
// the features' ReLU: dE = relu'(E) bf16(dE + 0.25 dpool), E the stored
// features (pitch epitch, channel offset eoff); eight channels per thread.
__global__ void k_pool_bwd(int Hc, int Wc, int C, const bf16_t* __restrict__ dpool, int ppitch, int64_t p_bs,
                           const bf16_t* __restrict__ E, int epitch, int eoff, bf16_t* __restrict__ dE, int64_t e_bs) {
  const int c8n = C / 8;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)Hc * Wc * c8n) return;
  const int64_t p = idx / c8n;
  const int c = (int)(idx - p * c8n) * 8;
  const int y = (int)(p / Wc), xx = (int)(p - (int64_t)y * Wc);
  const uint4 gv = *(const uint4*)(dpool + blockIdx.y * p_bs + p * ppitch + c);
  const uint32_t g4[4] = {gv.x, gv.y, gv.z, gv.w};
  const int64_t base = (int64_t)blockIdx.y * 4 * Hc * Wc;  // this sample's first fine pixel
  bf16_t* e = dE + blockIdx.y * e_bs + c;
  uint4 dv[4], ev[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t f = (int64_t)(2 * y + (q >> 1)) * 2 * Wc + 2 * xx + (q & 1);
    dv[q] = *(const uint4*)(e + f * C);
    ev[q] = *(const uint4*)(E + (base + f) * epitch + eoff + c);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t f = (int64_t)(2 * y + (q >> 1)) * 2 * Wc + 2 * xx + (q & 1);
    const uint32_t d4[4] = {dv[q].x, dv[q].y, dv[q].z, dv[q].w}, e4[4] = {ev[q].x, ev[q].y, ev[q].z, ev[q].w};
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float glo = 0.25f * bf2f((bf16_t)(g4[k] & 0xffff)), ghi = 0.25f * bf2f((bf16_t)(g4[k] >> 16));
      float lo = bf2f((bf16_t)(d4[k] & 0xffff)) + glo, hi = bf2f((bf16_t)(d4[k] >> 16)) + ghi;
      lo = bf2f((bf16_t)(e4[k] & 0xffff)) > 0.f ? lo : 0.f;
      hi = bf2f((bf16_t)(e4[k] >> 16)) > 0.f ? hi : 0.f;
      o[k] = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
    }
    *(uint4*)(e + f * C) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// ---------------------------------------------------------------------------
// Per-sample Mesh-Conv local weights (each sample has its own grid): the
// level arrays of sample s start at lv + s * lv_stride. A workgroup computes
// the hidden layer of Phi for 32 pixels, then writes eta[p][c] with the
// channel index fastest across threads.
constexpr int kEtaMPix = 128;  // pixels per workgroup of k_eta_multi
__global__ __launch_bounds__(256) void k_eta_multi(int H, int W, int cin, int cin8, int hid,
                                                   const float* __restrict__ lv, int64_t lv_stride,
                                                   const float* __restrict__ W1, const float* __restrict__ b1,
                                                   const float* __restrict__ W2, const float* __restrict__ b2,
                                                   bf16_t* __restrict__ eta, int64_t e_bs) {
  // Phi's output layer in LDS, transposed ([hid][cin] then b2) so that lanes
  // of consecutive channels read consecutive words; kEtaMPix pixels per
  // workgroup in batches of 32
  extern __shared__ float s_w2[];
  __shared__ float s_h[32][33];
  float* s_b2 = s_w2 + hid * cin;
  for (int u = threadIdx.x; u < cin * hid; u += 256) s_w2[(u % hid) * cin + u / hid] = W2[u];
  for (int u = threadIdx.x; u < cin; u += 256) s_b2[u] = b2[u];
  const int64_t npix = (int64_t)H * W;
  const float* L = lv + blockIdx.y * lv_stride;
  bf16_t* out = eta + blockIdx.y * e_bs;
  for (int64_t p0 = (int64_t)blockIdx.x * kEtaMPix; p0 < min(npix, (int64_t)(blockIdx.x + 1) * kEtaMPix); p0 += 32) {
    __syncthreads();
    for (int u = threadIdx.x; u < 32 * hid; u += 256) {
      const int q = u / hid, a = u - q * hid;
      const int64_t p = min(p0 + q, npix - 1);
      const int j = (int)(p / W), i = (int)(p - (int64_t)j * W);
      const float d0 = L[i], d1 = L[W + i], d2 = L[3 * W + j], d3 = L[3 * W + H + j];
      s_h[q][a] = tanh_nn(b1[a] + W1[a * 4] * d0 + W1[a * 4 + 1] * d1 + W1[a * 4 + 2] * d2 + W1[a * 4 + 3] * d3);
    }
    __syncthreads();
    for (int u = threadIdx.x; u < 32 * cin8; u += 256) {
      const int q = u / cin8, c = u - q * cin8;
      const int64_t p = p0 + q;
      if (p >= npix) continue;
      float e = 0.f;
      if (c < cin) {
        float phi = s_b2[c];
        for (int a = 0; a < hid; ++a) phi += s_w2[a * cin + c] * s_h[q][a];
        e = exp_nn(-phi * phi);
      }
      out[p * cin8 + c] = f2bf(e);
    }
  }
}

// Mesh-Conv local-weight backward. Given dXbar (gradient of the weighted
// input) and the layer input X: dX = eta * dXbar (written in place of dXbar)
// and, through dEta = dXbar * X and eta = exp(-Phi^2), the gradients of Phi's
// parameters. A workgroup handles 32-pixel batches of a contiguous pixel
// range (npb <= 32 pixels per batch, as many as the LDS holds for this
// layer's width). In the channel phase thread t owns the channel slots t % ns + k ns
// (ns = min(cin8, 256), k < KS) and pixel phase t / ns, and issues the loads
// of 8 pixels before using them. In the hidden phase thread t < S (S = the largest
// multiple of hid up to 256) owns hidden unit t % hid and the pixels t / hid,
// t / hid + S / hid, ..., so it accumulates its unit's W1 and b1 gradients
// itself. At the end the per-thread sums are reduced in a fixed order and one
// partial row [W1 (hid*4) | b1 (hid) | W2 (cin*hid) | b2 (cin)] (the layout
// of these parameters in the flat vector) is written. HC = hid rounded up to
// a power of two; KS >= cin8 / 256 channel slots per thread.
constexpr int kEtaPix = 32;
constexpr int kEtaGrp = 8;  // pixels whose loads are in flight together
template <int HC, int KS>
__global__ __launch_bounds__(256) void k_eta_bwd(int H, int W, int cin, int cin8, int hid, int nb,
                                                 const float* __restrict__ lv, int64_t lv_stride,
                                                 const float* __restrict__ W1, const float* __restrict__ b1,
                                                 const float* __restrict__ W2, const float* __restrict__ b2,
                                                 const bf16_t* __restrict__ x, const bf16_t* __restrict__ eta,
                                                 int64_t e_bs, bf16_t* __restrict__ dxb, float* __restrict__ part,
                                                 int npb) {
  extern __shared__ float sm[];
  const int cinp = cin + 1;                 // odd row pitch: rows start in different banks
  float* s_h = sm;                          // [kEtaPix][HC] hidden activations
  float* s_d = s_h + kEtaPix * HC;          // [kEtaPix][4] distances
  float* s_w2 = s_d + kEtaPix * 4;          // [hid][cinp] (transposed)
  float* s_dphi = s_w2 + cinp * hid;        // [npb][cinp]; reused for the final reductions
  __shared__ int s_smp[kEtaPix], s_pix[kEtaPix];  // sample and pixel of each batch pixel
  const int64_t npix = (int64_t)H * W, ntot = npix * nb;
  const int npix32 = H * W;
  const int64_t per = (ntot + gridDim.x - 1) / gridDim.x;
  const int64_t pbeg = blockIdx.x * per, pend = min(ntot, pbeg + per);
  const int t = threadIdx.x;
  const int ns = cin8 < 256 ? cin8 : 256;
  const int phases = 256 / ns;
  const int slot = t % ns, ph = t / ns;
  const bool active = ph < phases;
  const int qstep = 256 / hid, S = qstep * hid;
  const int my_a = t % hid, my_q = t / hid;  // hidden phase (t < S)
  for (int u = t; u < cin * hid; u += 256) s_w2[(u % hid) * cinp + u / hid] = W2[u];
  // the thread's own channels' row of Phi's output layer in registers when it
  // is small enough (else read from LDS)
  constexpr bool W2REG = KS * HC <= 32;
  float aw2[KS][HC], ab2[KS], b2r[KS], w2r[W2REG ? KS : 1][W2REG ? HC : 1];
  float aw1[5] = {0.f, 0.f, 0.f, 0.f, 0.f};  // W1 row and b1 of unit my_a
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const int c = slot + ns * k;
    ab2[k] = 0.f;
    b2r[k] = c < cin ? b2[c] : 0.f;
#pragma unroll
    for (int q = 0; q < HC; ++q) {
      aw2[k][q] = 0.f;
      if (W2REG) w2r[W2REG ? k : 0][W2REG ? q : 0] = (c < cin && q < hid) ? W2[c * hid + q] : 0.f;
    }
  }
  for (int64_t p0 = pbeg; p0 < pend; p0 += npb) {
    const int np = (int)min((int64_t)npb, pend - p0);
    __syncthreads();
    for (int u = t; u < np * hid; u += 256) {
      const int q = u / hid, a = u - q * hid;
      const int gp = (int)(p0 + q);  // the host keeps npix * nb below 2^31
      const int smp = gp / npix32;
      const int p = gp - smp * npix32;
      const int j = p / W, i = p - j * W;
      const float* L = lv + smp * lv_stride;
      const float d0 = L[i], d1 = L[W + i], d2 = L[3 * W + j], d3 = L[3 * W + H + j];
      s_h[q * HC + a] = tanh_nn(b1[a] + W1[a * 4] * d0 + W1[a * 4 + 1] * d1 + W1[a * 4 + 2] * d2 + W1[a * 4 + 3] * d3);
      if (a == 0) {
        s_d[q * 4] = d0;
        s_d[q * 4 + 1] = d1;
        s_d[q * 4 + 2] = d2;
        s_d[q * 4 + 3] = d3;
        s_smp[q] = smp;
        s_pix[q] = p;
      }
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const int c = slot + ns * k;
        if (c >= cin8) continue;
        for (int qb = ph; qb < np; qb += phases * kEtaGrp) {
          float gv[kEtaGrp], xv[kEtaGrp], ev[kEtaGrp];
          int64_t ov[kEtaGrp];
#pragma unroll
          for (int e = 0; e < kEtaGrp; ++e) {
            const int q = qb + phases * e;
            gv[e] = xv[e] = ev[e] = 0.f;
            ov[e] = -1;
            if (q < np) {
              ov[e] = (p0 + q) * cin8 + c;
              gv[e] = bf2f(dxb[ov[e]]);
              xv[e] = bf2f(x[ov[e]]);
              ev[e] = bf2f(eta[s_smp[q] * e_bs + (int64_t)s_pix[q] * cin8 + c]);
            }
          }
#pragma unroll
          for (int e = 0; e < kEtaGrp; ++e) {
            const int q = qb + phases * e;
            if (ov[e] < 0) continue;
            dxb[ov[e]] = f2bf(ev[e] * gv[e]);
            if (c >= cin) continue;
            float phi = b2r[k];
#pragma unroll
            for (int a = 0; a < HC; ++a)
              if (a < hid)
                phi += (W2REG ? w2r[W2REG ? k : 0][W2REG ? a : 0] : s_w2[a * cinp + c]) * s_h[q * HC + a];
            const float ef = exp_nn(-phi * phi);
            const float dphi = gv[e] * xv[e] * (-2.f * phi * ef);
            s_dphi[q * cinp + c] = dphi;
            ab2[k] += dphi;
#pragma unroll
            for (int a = 0; a < HC; ++a)
              if (a < hid) aw2[k][a] += dphi * s_h[q * HC + a];
          }
        }
      }
    }
    __syncthreads();
    // dz[q][a] = (sum_c W2[c][a] dphi[q][c]) (1 - h^2); the unit's W1 / b1 sums
    if (t < S) {
      const float* w = s_w2 + my_a * cinp;
      for (int q = my_q; q < np; q += qstep) {
        const float* f = s_dphi + q * cinp;
        float e0 = 0.f, e1 = 0.f, e2 = 0.f, e3 = 0.f;
        int c = 0;
        for (; c + 4 <= cin; c += 4) {
          e0 += w[c] * f[c];
          e1 += w[c + 1] * f[c + 1];
          e2 += w[c + 2] * f[c + 2];
          e3 += w[c + 3] * f[c + 3];
        }
        for (; c < cin; ++c) e0 += w[c] * f[c];
        const float h = s_h[q * HC + my_a];
        const float dz = ((e0 + e1) + (e2 + e3)) * (1.f - h * h);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) aw1[kk] += dz * s_d[q * 4 + kk];
        aw1[4] += dz;
      }
    }
  }
  const int len = hid * 5 + cin * hid + cin;
  float* row = part + (int64_t)blockIdx.x * len;
  float* red = s_dphi;  // >= 256 * (HC + 1) floats
  // W1 / b1: the threads of one unit, in order of their pixel offset
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < 5; ++kk) red[t * 5 + kk] = t < S ? aw1[kk] : 0.f;
  __syncthreads();
  if (t < hid * 5) {
    const int a = t / 5, kk = t - a * 5;
    float acc = 0.f;
    for (int q = 0; q < qstep; ++q) acc += red[(q * hid + a) * 5 + kk];
    if (kk < 4) row[a * 4 + kk] = acc;
    else row[hid * 4 + a] = acc;
  }
  // W2 / b2: the per-phase sums of each channel
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    __syncthreads();
#pragma unroll
    for (int a = 0; a <= HC; ++a)
      if (a <= hid) red[t * (HC + 1) + a] = a < hid ? aw2[k][a < HC ? a : 0] : ab2[k];
    __syncthreads();
    for (int u = t; u < ns * (hid + 1); u += 256) {
      const int sl = u / (hid + 1), a = u - sl * (hid + 1);
      const int c = sl + ns * k;
      if (c >= cin) continue;
      float acc = 0.f;
      for (int q = 0; q < phases; ++q) acc += red[(q * ns + sl) * (HC + 1) + a];
      if (a < hid) row[hid * 5 + c * hid + a] = acc;
      else row[hid * 5 + cin * hid + c] = acc;
    }
  }
}

// Static channels of the activation buffers of nb samples on their own grids.
__global__ void k_fill_static_multi(int H, int W, int pitch, int coff, const float* __restrict__ lv, int64_t lv_stride,
                                    const uint8_t* const* __restrict__ masks, int moff, bf16_t* __restrict__ buf,
                                    int64_t bstride) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (int64_t)H * W) return;
  const int j = (int)(p / W), i = (int)(p - (int64_t)j * W);
  const float* L = lv + blockIdx.y * lv_stride;
  bf16_t* b = buf + blockIdx.y * bstride + p * pitch;
  if (coff >= 0) {
    b[coff] = f2bf(L[2 * W + i]);
    b[coff + 1] = f2bf(L[3 * W + 2 * H + j]);
  }
  if (moff >= 0) {
    const uint8_t* m = masks ? masks[blockIdx.y] : nullptr;
    b[moff] = f2bf(m ? (float)m[p] : 0.f);
  }
}

// Trunk input channels (normalised centre coordinates, padded to 8).
__global__ void k_trunk_input(int H, int W, const float* __restrict__ tin, int64_t t_stride, bf16_t* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (int64_t)H * W) return;
  const int j = (int)(p / W), i = (int)(p - (int64_t)j * W);
  const float* tt = tin + blockIdx.y * t_stride;
  bf16_t* o = out + ((int64_t)blockIdx.y * H * W + p) * 8;
  o[0] = f2bf(tt[i]);
  o[1] = f2bf(tt[W + j]);
  for (int c = 2; c < 8; ++c) o[c] = 0;
}

// DeepONet contraction s = sum_k B_k T_k (FP32 sum of BF16 operands) and
// y = gamma s; s is kept for gamma's gradient.
// 16 lanes per pixel, 8 basis terms per lane per pass (P % 8 == 0).
__device__ __forceinline__ float dot8(uint4 a, uint4 b) {
  const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    s += bf2f((bf16_t)(x[e] & 0xffff)) * bf2f((bf16_t)(y[e] & 0xffff)) +
         bf2f((bf16_t)(x[e] >> 16)) * bf2f((bf16_t)(y[e] >> 16));
  return s;
}

__device__ __forceinline__ float sum16(float v) {
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 16);
  return v;
}

__global__ __launch_bounds__(256) void k_don_fwd(int64_t n, int P, const bf16_t* __restrict__ B,
                                                 const bf16_t* __restrict__ T, const float* __restrict__ gamma,
                                                 float* __restrict__ y, float* __restrict__ sum) {
  const int64_t p = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int l = threadIdx.x & 15;
  float s = 0.f;
  if (p < n)
    for (int k = l * 8; k < P; k += 128) s += dot8(*(const uint4*)(B + p * P + k), *(const uint4*)(T + p * P + k));
  s = sum16(s);
  if (p < n && l == 0) {
    sum[p] = s;
    y[p] = gamma[0] * s;
  }
}

// The head's output gradient dB = bf16(gamma (scale g) T) as an array, for
// heads too wide for k_bwd1x1.
__global__ __launch_bounds__(256) void k_don_grad(int64_t n, int P, const bf16_t* __restrict__ T,
                                                  const float* __restrict__ gamma, const float* __restrict__ g,
                                                  float scale, bf16_t* __restrict__ dB) {
  const int P8 = P / 8;
  const float gam = gamma[0];
  for (int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x; u < n * P8; u += (int64_t)gridDim.x * 256)
    *(uint4*)(dB + u * 8) = scale8(*(const uint4*)(T + u * 8), gam * (scale * g[u / P8]));
}

// Per-workgroup shares of gamma's gradient, sum of (scale g) s over pixels.
__global__ __launch_bounds__(256) void k_gamma_grad(int64_t n, const float* __restrict__ g, float scale,
                                                    const float* __restrict__ sum, float* __restrict__ part) {
  __shared__ double lds[kWaves];
  double acc = 0.0;
  if ((threadIdx.x & 15) == 0)
    for (int64_t p = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); p < n; p += (int64_t)gridDim.x * 16)
      acc += (double)(scale * g[p]) * (double)sum[p];
  acc = block_sum(acc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = (float)acc;
}

// Residual loss pieces: res = R - Ay (stored), per-workgroup partials of res^2.
__global__ __launch_bounds__(256) void k_loss(int64_t n, const float* __restrict__ R, const float* __restrict__ Ay,
                                              float* __restrict__ res, double* __restrict__ part) {
  __shared__ double lds[kWaves];
  double acc = 0.0;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
    const float v = R[p] - Ay[p];
    res[p] = v;
    acc += (double)v * v;
  }
  acc = block_sum(acc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// Supervised loss pieces, per sample s (blockIdx.y): partial sums of y, e,
// y^2, y e and e^2 ([nb][5][gridDim.x]).
__global__ __launch_bounds__(256) void k_sup_sums(int64_t N, const float* __restrict__ y,
                                                  const double* __restrict__ e, double* __restrict__ part) {
  __shared__ double lds[kWaves];
  const int s = blockIdx.y;
  const float* ys = y + (size_t)s * N;
  const double* es = e + (size_t)s * N;
  double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < N; p += (int64_t)gridDim.x * 256) {
    const double yv = ys[p], ev = es[p];
    a[0] += yv;
    a[1] += ev;
    a[2] += yv * yv;
    a[3] += yv * ev;
    a[4] += ev * ev;
  }
  for (int m = 0; m < 5; ++m) {
    const double v = block_sum(a[m], lds);
    if (threadIdx.x == 0) part[((size_t)s * 5 + m) * gridDim.x + blockIdx.x] = v;
  }
}

// Supervised loss L_s = 1 - a^2 / (b c) with a = y0.e0, b = |y0|^2, c = |e0|^2
// (centred fields) and its gradient, averaged over the nb samples:
// dL/dy = 2 a / (b c nb) (a/b y0 - e0) (zero mean, so the centring needs no
// further projection). A constant y (b = 0) or target (c = 0) gives L = 1
// and no gradient. Every workgroup reduces the partials in the same order.
__global__ __launch_bounds__(256) void k_sup_grad(int64_t N, int nb, const float* __restrict__ y,
                                                  const double* __restrict__ e, const double* __restrict__ part,
                                                  int nparts, float* __restrict__ dy, double* __restrict__ lsamp) {
  __shared__ double lds[kWaves];
  const int s = blockIdx.y;
  double S[5];
  for (int m = 0; m < 5; ++m) S[m] = reduce_partials(part + ((size_t)s * 5 + m) * nparts, nparts, lds);
  const double n = (double)N;
  const double my = S[0] / n, me = S[1] / n;
  const double a = S[3] - n * my * me;
  const double b = S[2] - n * my * my;
  const double c = S[4] - n * me * me;
  const bool ok = b > 0.0 && c > 0.0 && isfinite(a);
  const double L = ok ? 1.0 - a * a / (b * c) : 1.0;
  const double g = ok ? 2.0 * a / (b * c * (double)nb) : 0.0;
  const double ab = ok ? a / b : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) lsamp[s] = L;
  const float* ys = y + (size_t)s * N;
  const double* es = e + (size_t)s * N;
  float* ds = dy + (size_t)s * N;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < N; p += (int64_t)gridDim.x * 256)
    ds[p] = (float)(g * (ab * ((double)ys[p] - my) - (es[p] - me)));
}

// Per-sample partial sums of the A-norm loss: R.y, y.Ay, R.e (FP64).
__global__ __launch_bounds__(256) void k_anorm_sums(int64_t N, const float* __restrict__ y,
                                                    const float* __restrict__ Ay, const float* __restrict__ R,
                                                    const double* __restrict__ e, double* __restrict__ part) {
  __shared__ double lds[kWaves];
  const int s = blockIdx.y;
  const size_t o = (size_t)s * N;
  double a[3] = {0.0, 0.0, 0.0};
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < N; p += (int64_t)gridDim.x * 256) {
    const double yv = y[o + p], rv = R[o + p];
    a[0] += rv * yv;
    a[1] += yv * (double)Ay[o + p];
    a[2] += rv * e[o + p];
  }
  for (int m = 0; m < 3; ++m) {
    const double v = block_sum(a[m], lds);
    if (threadIdx.x == 0) part[((size_t)s * 3 + m) * gridDim.x + blockIdx.x] = v;
  }
}

// A-norm loss L_s = 1 - a^2 / (b c) with a = R.y, b = y.Ay, c = R.e, and its
// gradient averaged over the nb samples (A symmetric):
// dL/dy = (2 a / (b c nb)) (a/b A y - R). b <= 0 or c <= 0 gives L = 1 and no
// gradient. Every workgroup reduces the partials in the same order.
__global__ __launch_bounds__(256) void k_anorm_grad(int64_t N, int nb, const float* __restrict__ Ay,
                                                    const float* __restrict__ R, const double* __restrict__ part,
                                                    int nparts, float* __restrict__ dy, double* __restrict__ lsamp) {
  __shared__ double lds[kWaves];
  const int s = blockIdx.y;
  double S[3];
  for (int m = 0; m < 3; ++m) S[m] = reduce_partials(part + ((size_t)s * 3 + m) * nparts, nparts, lds);
  const double a = S[0], b = S[1], c = S[2];
  const bool ok = b > 0.0 && c > 0.0 && isfinite(a);
  const double L = ok ? 1.0 - a * a / (b * c) : 1.0;
  const double g = ok ? 2.0 * a / (b * c * (double)nb) : 0.0;
  const double ab = ok ? a / b : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) lsamp[s] = L;
  const size_t o = (size_t)s * N;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < N; p += (int64_t)gridDim.x * 256)
    dy[o + p] = (float)(g * (ab * (double)Ay[o + p] - (double)R[o + p]));
}

__global__ void k_sum_parts(const double* __restrict__ part, int n, double scale, double* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  for (int k = 0; k < n; ++k) s += part[k];
  out[0] = scale * s;
}

// Adam (Kingma & Ba 2015, Alg. 1) on the FP32 master parameters. With
// clip > 0 the gradient is first scaled by min(1, clip / ||g||), ||g||^2 being
// the fixed-order sum of the kRedBlocks partial sums in gpart (the same bits
// in every workgroup).
__global__ __launch_bounds__(256) void k_adam(int64_t n, float* __restrict__ w, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                              float b2, float eps, float c1, float c2, const double* __restrict__ gpart,
                                              float clip) {
  __shared__ double lds[kWaves];
  float scale = 1.f;
  if (clip > 0.f) {
    const double gn = sqrt(reduce_partials(gpart, kRedBlocks, lds));
    if (gn > (double)clip) scale = (float)((double)clip / gn);
  }
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const float gk = g[k] * scale;
  const float mk = b1 * m[k] + (1.f - b1) * gk;
  const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  w[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// Sharpness-aware perturbation (Foret et al., 2021): w += rho g / |g|, with
// |g|^2 from the kRedBlocks partials of k_sumsq reduced in the same order by
// every workgroup; no change when g = 0.
__global__ __launch_bounds__(256) void k_sam_perturb(int64_t n, float* w, const float* g, const double* gpart,
                                                     float rho) {
  __shared__ double lds[kWaves];
  const double gn = sqrt(reduce_partials(gpart, kRedBlocks, lds));
  const float scale = gn > 0.0 ? (float)((double)rho / gn) : 0.f;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) w[k] += scale * g[k];
}

// ---------------------------------------------------------------------------
static unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

void launch_wgrad1(const WgradGeo& g, const bf16_t* dp, const bf16_t* x, float* part, int nsplit, hipStream_t s) {
  const dim3 grid1((g.cout + kW1T - 1) / kW1T, (g.cin8 + kW1T - 1) / kW1T, nsplit);
  k_wgrad1<<<grid1, 256, 0, s>>>(g, dp, x, part);
}

bool bwd1x1_fits(int cout, int cin8) { return cout <= kB1C && cin8 <= kB1C; }

// One split per workgroup: 1024 at most (two rounds of the resident
// workgroups), one per 128-pixel tile where there are fewer.
int launch_bwd1x1(const Bwd1x1& g, int64_t tiles, float* part, int64_t cap, hipStream_t s) {
  const int64_t n = std::max<int64_t>(1, std::min<int64_t>({1024, tiles, cap / ((int64_t)g.cout * g.cin8)}));
  k_bwd1x1<<<(unsigned)n, 256, 0, s>>>(g, part);
  return (int)n;
}

// Splits and channel tiles of k_wgrad9. Splits: 1024 / (32 x 32 channel tiles of
// the layer), at most one per pixel tile, and as many rows as the partials
// buffer holds. Per workgroup 64, 32 or 16 input channels, the widest that pads
// the input least; 64 output channels where that leaves two
// workgroups per compute unit, else 32 (64 samples of 256 x 256: 25.1 ms a step, 25.4 with 64 from one per unit).
int launch_wgrad9(const WgradGeo& g, const bf16_t* dp, const bf16_t* x, const bf16_t* eta, float* part, int64_t cap,
                  hipStream_t s) {
  const int64_t tiles = (int64_t)((g.W + 15) / 16) * ((g.H + 7) / 8) * g.nb;
  const int64_t len = (int64_t)g.cout * g.cin8 * 9;
  const int64_t blocks32 = (int64_t)((g.cout + 31) / 32) * ((g.cin8 + 31) / 32);
  const int64_t ns =
      std::max<int64_t>(1, std::min<int64_t>({std::max<int64_t>(1, 1024 / blocks32), tiles, cap / len}));
  const int ct = g.cin8 <= 16 ? 1 : (g.cin8 + 63) / 64 * 64 > (g.cin8 + 31) / 32 * 32 ? 2 : 4;
  const int nby = (g.cin8 + 16 * ct - 1) / (16 * ct);
  const int mt = g.cout > 32 && ns * ((g.cout + 63) / 64) * nby >= 512 ? 4 : 2;
  const int nbx = (g.cout + 16 * mt - 1) / (16 * mt), nblk = nbx * nby;
  const unsigned grid = (unsigned)(ns * nblk);
#define PPE_WG9(MT, CT, ETA) k_wgrad9<MT, CT, ETA><<<grid, 64 * CT, 0, s>>>(g, dp, x, eta, part, nbx, nblk, (int)ns)
#define PPE_WG9_ETA(MT, CT)                            \
  if (!eta) PPE_WG9(MT, CT, kEtaNone);                 \
  else if (g.eta_node) PPE_WG9(MT, CT, kEtaNode);      \
  else PPE_WG9(MT, CT, kEtaChannel)
  if (mt == 4) {
    if (ct == 4) { PPE_WG9_ETA(4, 4); }
    else if (ct == 2) { PPE_WG9_ETA(4, 2); }
    else { PPE_WG9_ETA(4, 1); }
  } else {
    if (ct == 4) { PPE_WG9_ETA(2, 4); }
    else if (ct == 2) { PPE_WG9_ETA(2, 2); }
    else { PPE_WG9_ETA(2, 1); }
  }
#undef PPE_WG9_ETA
#undef PPE_WG9
  return (int)ns;
}

void launch_reduce_rows(const float* part, int nparts, int64_t len, float scale, float* out, hipStream_t s) {
  k_reduce_rows<<<(unsigned)((len + 31) / 32), 256, 0, s>>>(part, nparts, len, scale, out);
}

void launch_bias_grad(const bf16_t* d, int64_t npix, int pitch, int off, int C, const float* gamma, const float* dy,
                      float scale, float* part, int nparts, hipStream_t s) {
  k_bias_grad<<<nparts, 256, 0, s>>>(d, npix, pitch, off, C, gamma, dy, scale, part);
}

void launch_act_bwd(bf16_t* d, int dpitch, const bf16_t* out, int opitch, int ooff, int C, int64_t npix, int mode,
                    hipStream_t s) {
  k_act_bwd<<<nblk(npix * (C / 8)), 256, 0, s>>>(d, dpitch, out, opitch, ooff, C, npix, mode);
}

void launch_copy_ch(const bf16_t* src, int spitch, int soff, bf16_t* dst, int dpitch, int C, int64_t npix,
                    hipStream_t s) {
  k_copy_ch<<<nblk(npix * (C / 8)), 256, 0, s>>>(src, spitch, soff, dst, dpitch, C, npix);
}

void launch_up_bwd(int Hc, int Wc, int C, const bf16_t* fine, int fpitch, int64_t f_bs, bf16_t* coarse, int64_t c_bs,
                   int nb, hipStream_t s) {
  k_up_bwd<<<dim3(nblk((int64_t)Hc * Wc * (C / 8)), nb), 256, 0, s>>>(Hc, Wc, C, fine, fpitch, f_bs, coarse, c_bs);
}

void launch_pool_bwd(int Hc, int Wc, int C, const bf16_t* dpool, int ppitch, int64_t p_bs, const bf16_t* E, int epitch,
                     int eoff, bf16_t* dE, int64_t e_bs, int nb, hipStream_t s) {
  k_pool_bwd<<<dim3(nblk((int64_t)Hc * Wc * (C / 8)), nb), 256, 0, s>>>(Hc, Wc, C, dpool, ppitch, p_bs, E, epitch, eoff,
                                                                        dE, e_bs);
}

void launch_eta_multi(int H, int W, int cin, int cin8, int hid, const float* lv, int64_t lv_stride, const float* W1,
                      const float* b1, const float* W2, const float* b2, bf16_t* eta, int64_t e_bs, int nb,
                      hipStream_t s) {
  const size_t shm = sizeof(float) * ((size_t)hid * cin + cin);
  k_eta_multi<<<dim3((unsigned)(((int64_t)H * W + kEtaMPix - 1) / kEtaMPix), nb), 256, shm, s>>>(
      H, W, cin, cin8, hid, lv, lv_stride, W1, b1, W2, b2, eta, e_bs);
}

int eta_bwd_len(int cin, int hid) { return hid * 5 + cin * hid + cin; }

// LDS of one workgroup of k_eta_bwd, in floats, apart from the dphi rows.
static int64_t eta_bwd_fixed(int cin, int hid, int hc) { return (int64_t)kEtaPix * hc + kEtaPix * 4 + (int64_t)(cin + 1) * hid; }

// LDS available to one workgroup's dynamic allocation: the default 64 KiB
// limit less 1 KiB for the kernel's static arrays.
static int64_t lds_per_block() { return 63 * 1024; }

static int eta_bwd_hc(int hid) { return hid <= 4 ? 4 : hid <= 8 ? 8 : hid <= 16 ? 16 : 32; }

// Pixels per batch that fit the LDS (0: the layer is too wide).
static int eta_bwd_npb(int cin, int hid) {
  const int hc = eta_bwd_hc(hid);
  const int64_t room = lds_per_block() / (int64_t)sizeof(float) - eta_bwd_fixed(cin, hid, hc);
  if (room < 256 * (int64_t)(hc + 1)) return 0;  // the final reductions need this much
  return (int)std::min<int64_t>(kEtaPix, room / (cin + 1));
}

bool eta_bwd_fits(int cin, int cin8, int hid) { return cin8 <= 1024 && eta_bwd_npb(cin, hid) >= 1; }

void launch_eta_bwd(int H, int W, int cin, int cin8, int hid, int nb, const float* lv, int64_t lv_stride,
                    const float* W1, const float* b1, const float* W2, const float* b2, const bf16_t* x,
                    const bf16_t* eta, int64_t e_bs, bf16_t* dxb, float* part, int nparts, hipStream_t s) {
  const int hc = eta_bwd_hc(hid);
  const int npb = eta_bwd_npb(cin, hid);  // >= 1: the caller checked eta_bwd_fits
  const size_t shm = sizeof(float) * (eta_bwd_fixed(cin, hid, hc) +
                                      std::max<int64_t>((int64_t)npb * (cin + 1), 256 * (int64_t)(hc + 1)));
#define PPE_ETA_BWD(HC, KS)                                                                                    \
  k_eta_bwd<HC, KS><<<nparts, 256, shm, s>>>(H, W, cin, cin8, hid, nb, lv, lv_stride, W1, b1, W2, b2, x, eta, \
                                             e_bs, dxb, part, npb)
#define PPE_ETA_BWD_HC(KS)                  \
  if (hc == 4) PPE_ETA_BWD(4, KS);          \
  else if (hc == 8) PPE_ETA_BWD(8, KS);     \
  else if (hc == 16) PPE_ETA_BWD(16, KS);   \
  else PPE_ETA_BWD(32, KS)
  // channel slots per thread: cin8 <= 256 needs one, <= 512 two, <= 1024 four
  if (cin8 <= 256) { PPE_ETA_BWD_HC(1); }
  else if (cin8 <= 512) { PPE_ETA_BWD_HC(2); }
  else { PPE_ETA_BWD_HC(4); }
#undef PPE_ETA_BWD_HC
#undef PPE_ETA_BWD
}

void launch_fill_static_multi(int H, int W, int pitch, int coff, const float* lv, int64_t lv_stride,
                              const uint8_t* const* masks, int moff, bf16_t* buf, int64_t bstride, int nb,
                              hipStream_t s) {
  k_fill_static_multi<<<dim3(nblk((int64_t)H * W), nb), 256, 0, s>>>(H, W, pitch, coff, lv, lv_stride, masks, moff,
                                                                      buf, bstride);
}

void launch_trunk_input(int H, int W, const float* tin, int64_t t_stride, bf16_t* out, int nb, hipStream_t s) {
  k_trunk_input<<<dim3(nblk((int64_t)H * W), nb), 256, 0, s>>>(H, W, tin, t_stride, out);
}

void launch_don_fwd(int64_t n, int P, const bf16_t* B, const bf16_t* T, const float* gamma, float* y, float* sum,
                    hipStream_t s) {
  k_don_fwd<<<(unsigned)((n + 15) / 16), 256, 0, s>>>(n, P, B, T, gamma, y, sum);
}

void launch_don_grad(int64_t n, int P, const bf16_t* T, const float* gamma, const float* g, float scale, bf16_t* dB,
                     hipStream_t s) {
  k_don_grad<<<2048, 256, 0, s>>>(n, P, T, gamma, g, scale, dB);
}

void launch_gamma_grad(int64_t n, const float* g, float scale, const float* sum, float* part, hipStream_t s) {
  k_gamma_grad<<<kGammaParts, 256, 0, s>>>(n, g, scale, sum, part);
}

void launch_loss(int64_t n, const float* R, const float* Ay, float* res, double* part, int nparts, hipStream_t s) {
  k_loss<<<nparts, 256, 0, s>>>(n, R, Ay, res, part);
}

void launch_sup_loss(int64_t N, int nb, const float* y, const double* e, double* part, int nparts, float* dy,
                     double* lsamp, hipStream_t s) {
  k_sup_sums<<<dim3(nparts, nb), 256, 0, s>>>(N, y, e, part);
  k_sup_grad<<<dim3(nparts, nb), 256, 0, s>>>(N, nb, y, e, part, nparts, dy, lsamp);
}

void launch_anorm_loss(int64_t N, int nb, const float* y, const float* Ay, const float* R, const double* e,
                       double* part, int nparts, float* dy, double* lsamp, hipStream_t s) {
  k_anorm_sums<<<dim3(nparts, nb), 256, 0, s>>>(N, y, Ay, R, e, part);
  k_anorm_grad<<<dim3(nparts, nb), 256, 0, s>>>(N, nb, Ay, R, part, nparts, dy, lsamp);
}

// Input gradient of a layer with one local weight per node (or none), given
// g = dXbar, the gradient of the weighted input, and the layer input X:
//   dX = bf16(eta g), where masked also zero where X <= 0 (X a ReLU output),
//   se[p] = dEta[p] = sum_c g[p][c] X[p][c].
// dX replaces g, except that channels [skip_lo, skip_hi) go to the rows of
// `skip` (the encoder's feature gradient) and later ones nowhere (the static
// channels of a decoder concatenation). With `bias`, dX is the gradient of the
// pre-activations of the layer before, and bias[b][c] receives workgroup b's sum
// over its pixels: that layer's bias gradient, in k_bias_grad's order (the same
// pixels per thread and workgroup).
// LP lanes (a power of two, at most 16) share a pixel, lane l taking its
// 8-channel groups l, l + LP, ...; four pixels per thread in flight. se is one
// chain over the channels in order: it passes from lane to lane (DPP row
// shifts), each lane adding its group when its turn comes.
// Bound by HBM: 6 B per channel and pixel. One thread per pixel, with the
// parameter gradients in the same kernel, took 4.5 ms for the 14 layers of 64
// samples of 256 x 256, and separate passes for the mask and the skip channels
// 3.0 ms more; this and k_phi_grad take 2.1 ms.
template <int LP>
__global__ __launch_bounds__(256) void k_eta_dx(EtaDx a) {
  constexpr int PX = 4;
  __shared__ float red[256 * 8];
  const int l = threadIdx.x & (LP - 1);
  const int G = a.cin8 / 8;
  const int64_t step = (int64_t)gridDim.x * (256 / LP);
  float bs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int64_t p0 = (int64_t)blockIdx.x * (256 / LP) + threadIdx.x / LP; p0 < a.npix; p0 += PX * step) {
    float e[PX], se[PX];
#pragma unroll
    for (int u = 0; u < PX; ++u) {
      const int64_t p = p0 + u * step;
      e[u] = a.eta && p < a.npix ? bf2f(a.eta[p]) : 1.f;
      se[u] = 0.f;
    }
    for (int c0 = 0; c0 < G; c0 += LP) {  // all lanes of a pixel together
      const int c8 = c0 + l;
      uint4 gv[PX], xv[PX];
#pragma unroll
      for (int u = 0; u < PX; ++u) {
        const int64_t p = p0 + u * step;
        gv[u] = xv[u] = make_uint4(0, 0, 0, 0);
        if (p < a.npix && c8 < G) {
          gv[u] = *(const uint4*)(a.dxb + p * a.cin8 + c8 * 8);
          xv[u] = *(const uint4*)(a.x + p * a.cin8 + c8 * 8);
        }
      }
#pragma unroll
      for (int u = 0; u < PX; ++u) {
        const int64_t p = p0 + u * step;
        const uint32_t ga[4] = {gv[u].x, gv[u].y, gv[u].z, gv[u].w}, xa[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
        float g[8], x[8];
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          g[2 * k] = bf2f((bf16_t)(ga[k] & 0xffff));
          g[2 * k + 1] = bf2f((bf16_t)(ga[k] >> 16));
          x[2 * k] = bf2f((bf16_t)(xa[k] & 0xffff));
          x[2 * k + 1] = bf2f((bf16_t)(xa[k] >> 16));
        }
        if (a.se) {
          // the chain's value enters at lane 0 and leaves at lane LP - 1
          float v = se[u];
#pragma unroll
          for (int r = 0; r < LP; ++r) {
            float w = v;
#pragma unroll
            for (int k = 0; k < 4; ++k) w += g[2 * k] * x[2 * k] + g[2 * k + 1] * x[2 * k + 1];
            if (LP == 1) {
              v = w;
            } else {
              v = l == r ? w : v;  // lane r's turn
              if (r + 1 < LP) {
                const float from = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x111, 0xf, 0xf, true));
                v = l == r + 1 ? from : v;
              }
            }
          }
          se[u] = LP == 1 ? v : __shfl(v, LP - 1, LP);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float d0 = e[u] * g[2 * k], d1 = e[u] * g[2 * k + 1];
          if (a.mask) {
            d0 = x[2 * k] > 0.f ? d0 : 0.f;
            d1 = x[2 * k + 1] > 0.f ? d1 : 0.f;
          }
          o[k] = (uint32_t)f2bf(d0) | ((uint32_t)f2bf(d1) << 16);
        }
        if (p >= a.npix || c8 >= G) continue;
        const uint4 d = make_uint4(o[0], o[1], o[2], o[3]);
        const int c = c8 * 8;
        if (!a.skip || c < a.skip_lo) *(uint4*)(a.dxb + p * a.cin8 + c) = d;
        else if (c < a.skip_hi) *(uint4*)(a.skip + p * (a.skip_hi - a.skip_lo) + c - a.skip_lo) = d;
        if (a.bias) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            bs[2 * k] += bf2f((bf16_t)(o[k] & 0xffff));
            bs[2 * k + 1] += bf2f((bf16_t)(o[k] >> 16));
          }
        }
      }
    }
    if (a.se) {
#pragma unroll
      for (int u = 0; u < PX; ++u)
        if (l == 0 && p0 + u * step < a.npix) a.se[p0 + u * step] = se[u];
    }
  }
  if (!a.bias) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = bs[e];
  __syncthreads();
  for (int c = threadIdx.x; c < a.cin8; c += 256) {
    float sum = 0.f;
    for (int q = 0; q < 256 / LP; ++q) sum += red[(q * LP + c / 8) * 8 + (c % 8)];
    a.bias[(int64_t)blockIdx.x * a.cin8 + c] = sum;
  }
}

// Lanes per pixel: the widest power of two that the 8-channel groups fill once.
static int eta_dx_lanes(int cin8) {
  const int G = cin8 / 8;
  return G >= 16 ? 16 : G >= 8 ? 8 : G >= 4 ? 4 : G >= 2 ? 2 : 1;
}

bool eta_dx_can_bias(int cin8) { return eta_dx_lanes(cin8) * 8 == cin8; }

void launch_eta_dx(const EtaDx& a, hipStream_t s) {
  const int lp = eta_dx_lanes(a.cin8);
  const unsigned n =
      a.bias ? kBiasParts : (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, (a.npix * lp + 1023) / 1024));
  if (lp == 16) k_eta_dx<16><<<n, 256, 0, s>>>(a);
  else if (lp == 8) k_eta_dx<8><<<n, 256, 0, s>>>(a);
  else if (lp == 4) k_eta_dx<4><<<n, 256, 0, s>>>(a);
  else if (lp == 2) k_eta_dx<2><<<n, 256, 0, s>>>(a);
  else k_eta_dx<1><<<n, 256, 0, s>>>(a);
}

// The layer of workgroup b of a launch over several layers, and b's number
// within the layer's workgroups.
__device__ __forceinline__ const PhiLayer& phi_layer(const PhiArgs& a, int b, int& w) {
  int k = 0;
  while (k + 1 < a.n && a.layer[k + 1].wg0 <= b) ++k;
  w = b - a.layer[k].wg0;
  return a.layer[k];
}

// Local weights (Eq. 17) of all layers with one weight per node, one thread per
// node: eta = exp(-Phi^2), Phi = W2 . tanh(W1 d + b1) + b2 with d the node's four
// distances. Bound by the 2 x 16 transcendentals a node. HC = hidden units
// rounded up to a power of two.
template <int HC>
__global__ __launch_bounds__(256) void k_eta_nodes(PhiArgs a) {
  int w;
  const PhiLayer& y = phi_layer(a, blockIdx.x, w);
  const float *W1 = a.params + y.oW1, *b1 = W1 + a.hid * 4, *W2 = b1 + a.hid, *b2 = W2 + a.hid;
  const int64_t npix = (int64_t)y.H * y.W;
  const int64_t gp = (int64_t)w * 256 + threadIdx.x;
  if (gp >= npix * a.nb) return;
  const int smp = (int)(gp / npix), p = (int)(gp - smp * npix);
  const int j = p / y.W, i = p - j * y.W;
  const float* L = a.lv + smp * a.lv_stride + y.lv_off;
  const float d0 = L[i], d1 = L[y.W + i], d2 = L[3 * y.W + j], d3 = L[3 * y.W + y.H + j];
  float phi = b2[0];
#pragma unroll
  for (int k = 0; k < HC; ++k)
    if (k < a.hid)
      phi += W2[k] * tanh_nn(b1[k] + W1[k * 4] * d0 + W1[k * 4 + 1] * d1 + W1[k * 4 + 2] * d2 + W1[k * 4 + 3] * d3);
  a.eta[y.eta_off + gp] = f2bf(exp_nn(-phi * phi));
}

// Gradients of Phi's parameters of all layers with one weight per node, from
// dEta (se) of every node: through eta = exp(-Phi^2),
//   dPhi = -2 Phi eta dEta,  dz_a = dPhi W2_a (1 - h_a^2),
//   dW1[a][k] += dz_a d_k, db1[a] += dz_a, dW2[a] += dPhi h_a, db2 += dPhi.
// Each thread sums its nodes (grid stride within the layer); the lanes of a wave
// add up by a butterfly of register moves, the waves in order, into one partial
// row per workgroup, [W1 (hid*4) | b1 (hid) | W2 (hid) | b2].
//
// Sum over a wavefront, lanes paired at distance 32, 16, 8, 4, 2, 1 (the row
// rotations by 8 and 4 meet equal values there, so they pair as xor does).
__device__ __forceinline__ float wave_sum_f32(float v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r.x) + __uint_as_float(r.y);
  r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r.x) + __uint_as_float(r.y);
#define PPE_DPP_ADD(C) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C, 0xf, 0xf, true))
  PPE_DPP_ADD(0x128);  // row_ror:8
  PPE_DPP_ADD(0x124);  // row_ror:4
  PPE_DPP_ADD(0x4E);   // quad_perm [2,3,0,1]
  PPE_DPP_ADD(0xB1);   // quad_perm [1,0,3,2]
#undef PPE_DPP_ADD
  return v;
}

template <int HC>
__global__ __launch_bounds__(256) void k_phi_grad(PhiArgs a) {
  constexpr int NV = HC * 6 + 1;  // accumulated values: W1 (4 HC), b1, W2, b2
  __shared__ float s_w[kWaves][NV];
  int w;
  const PhiLayer& y = phi_layer(a, blockIdx.x, w);
  const float *W1 = a.params + y.oW1, *b1 = W1 + a.hid * 4, *W2 = b1 + a.hid, *b2 = W2 + a.hid;
  const int64_t npix = (int64_t)y.H * y.W, ntot = npix * a.nb;
  float acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.f;
  for (int64_t gp = (int64_t)w * 256 + threadIdx.x; gp < ntot; gp += (int64_t)y.nwg * 256) {
    const int smp = (int)(gp / npix), p = (int)(gp - smp * npix);
    const int j = p / y.W, i = p - j * y.W;
    const float* L = a.lv + smp * a.lv_stride + y.lv_off;
    const float d[4] = {L[i], L[y.W + i], L[3 * y.W + j], L[3 * y.W + y.H + j]};
    const float se = a.se[y.eta_off + gp];
    float h[HC];
    float phi = b2[0];
#pragma unroll
    for (int q = 0; q < HC; ++q) {
      h[q] = 0.f;
      if (q < a.hid) {
        h[q] = tanh_nn(b1[q] + W1[q * 4] * d[0] + W1[q * 4 + 1] * d[1] + W1[q * 4 + 2] * d[2] + W1[q * 4 + 3] * d[3]);
        phi += W2[q] * h[q];
      }
    }
    const float dphi = se * (-2.f * phi * exp_nn(-phi * phi));
#pragma unroll
    for (int q = 0; q < HC; ++q) {
      if (q >= a.hid) continue;
      const float dz = dphi * W2[q] * (1.f - h[q] * h[q]);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[q * 4 + k] += dz * d[k];
      acc[HC * 4 + q] += dz;
      acc[HC * 5 + q] += dphi * h[q];
    }
    acc[HC * 6] += dphi;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const float v = wave_sum_f32(acc[k]);
    if (lane == 0) s_w[wv][k] = v;
  }
  __syncthreads();
  const int len = a.hid * 6 + 1;
  float* row = a.part + (int64_t)blockIdx.x * len;
  for (int u = threadIdx.x; u < len; u += 256) {
    // u: W1 (q * 4 + k) | b1 (q) | W2 (q) | b2
    const int k = u < a.hid * 4   ? u
                  : u < a.hid * 5 ? HC * 4 + (u - a.hid * 4)
                  : u < a.hid * 6 ? HC * 5 + (u - a.hid * 5)
                                  : HC * 6;
    float t = 0.f;
    for (int v = 0; v < kWaves; ++v) t += s_w[v][k];
    row[u] = t;
  }
}

#define PPE_PHI_HC(K)                                  \
  if (a.hid <= 8) K<8><<<wg, 256, 0, s>>>(a);          \
  else if (a.hid <= 16) K<16><<<wg, 256, 0, s>>>(a);   \
  else K<32><<<wg, 256, 0, s>>>(a)

void launch_eta_nodes(PhiArgs a, hipStream_t s) {
  int wg = 0;
  for (int k = 0; k < a.n; ++k) {
    a.layer[k].wg0 = wg;
    wg += (int)(((int64_t)a.layer[k].H * a.layer[k].W * a.nb + 255) / 256);
  }
  PPE_PHI_HC(k_eta_nodes);
}

// Workgroups per layer: one node per thread at least, kPhiParts at most.
// Adds the layers' partial rows to the table of sums.
void launch_phi_grad(PhiArgs a, float* grad, RowTable& t, hipStream_t s) {
  const int len = a.hid * 6 + 1;
  int wg = 0;
  for (int k = 0; k < a.n; ++k) {
    const int64_t n = (int64_t)a.layer[k].H * a.layer[k].W * a.nb;
    a.layer[k].wg0 = wg;
    a.layer[k].nwg = (int)std::min<int64_t>(kPhiParts, (n + 255) / 256);
    t.row[t.n++] = RowSum{a.part + (int64_t)wg * len, a.layer[k].nwg, len, grad + a.layer[k].oW1};
    wg += a.layer[k].nwg;
  }
  PPE_PHI_HC(k_phi_grad);
}
#undef PPE_PHI_HC

void launch_sum_parts(const double* part, int n, double scale, double* out, hipStream_t s) {
  k_sum_parts<<<1, 64, 0, s>>>(part, n, scale, out);
}

void launch_adam(int64_t n, float* w, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                 float c1, float c2, const double* gpart, float clip, hipStream_t s) {
  k_adam<<<nblk(n), 256, 0, s>>>(n, w, g, m, v, lr, b1, b2, eps, c1, c2, gpart, clip);
}

void launch_sam_perturb(int64_t n, float* w, const float* g, const double* gpart, float rho, hipStream_t s) {
  k_sam_perturb<<<nblk(n), 256, 0, s>>>(n, w, g, gpart, rho);
}

}  // namespace ppe
