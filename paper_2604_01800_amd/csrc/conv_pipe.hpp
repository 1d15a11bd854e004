// The pipelined 3x3 convolution kernel and its launch, instantiated in a source file each
// for 32 and 64 output channels per workgroup on tiles of 32 rows, and for 32 on tiles of 16.
#pragma once
#include <type_traits>

#include "conv_device.hpp"

namespace ppe {

// Pipelined form of the 3x3 convolution for launches that fill the chip (TH = 32): the
// same implicit GEMM with the same K order (so the same bits), in workgroups of
// eight wavefronts over 32 x 16 pixel tiles, one workgroup per compute unit; and for
// those with at most one 16 x 16 tile per compute unit (TH = 16, four wavefronts, also
// with a split K), which only ever wait for their own loads. What
// bounded k_conv was the wait for an item's loads between two barriers, the vector
// work beside the MFMAs (MFMA busy 6-25 %) and its stores of 8 bytes a lane. Here the
// staged input is double buffered and one barrier separates items: a wavefront in turn
// runs the MFMAs of an item, writes the next one to LDS, issues the loads of a later
// one (two items in flight with 32 output channels and one chunk, layers that are bound
// by memory, and with 16-row tiles) and stores its results; the second half of the
// wavefronts (the other one on each SIMD) does this half a turn later, so that one's vector
// work runs beside the other's MFMAs. Weights stay in LDS for the launch where all chunks fit (WRES), else
// their slices are double buffered too.
// LDS layouts: input pixels of 64 bytes, their 16-byte groups permuted by the
// pixel number (eight consecutive pixels of one group lie in distinct banks);
// weights as MFMA fragments, [step][16-channel tile][lane], read and written
// without conflicts. In a full chunk a K-step is one tap, and the input rows
// that two vertical taps share stay in registers: 18 input and 9 MT weight reads
// for 36 MT MFMAs. The 3x3 layers of a 1024^2 forward took 657 us with k_conv and take
// 514 us; the largest (66 channels, 72 with padding, to 32 at 1024^2) 129 -> 84 us, 0.47
// PFLOP/s and 3.2 TB/s. MFMA busy is 7-34 %; the wavefronts wait 30-61 % of their cycles at
// barriers and for loads, mostly in the start of a launch.

template <int TN, int TH>
struct ConvP {
  using S = ConvShape<TN, 9, TH, TH * 16>;
  static constexpr int MT = TN / 16;
  static constexpr int XB = S::NPIX * 32;        // bf16 of one input buffer
  static constexpr int WB = S::SMAX * MT * 512;  // bf16 of one weight slice
};

// Element offset of 8-channel group c8 of halo pixel p in the input buffer.
__device__ __forceinline__ int convp_slot(int p, int c8) { return p * 32 + ((c8 ^ ((p >> 1) & 3)) * 8); }

// This thread's staged pixels, fixed for the launch: rows and columns of the
// halo tile (ly | lx << 16), and the byte offset of its first weight fragment group
// from the chunk's first column (the others follow at fixed distances).
template <class S>
struct ConvpLane {
  uint32_t yx[S::NU];
  uint32_t wo;
};

template <int TN, int TH>
__device__ __forceinline__ void convp_issue_w(uint4* w, uint32_t wo, __amdgpu_buffer_rsrc_t wr, int ck8,
                                              int kbase) {
  using S = typename ConvP<TN, TH>::S;
  const int n = conv_chunk_steps(9, ck8 * 8) * ConvP<TN, TH>::MT * 64;
#pragma unroll
  for (int i = 0; i < S::NW; ++i) {
    // threads per fragment column: S::NTHR / 64 fragments further on in the list of (step, tile)
    const uint32_t off =
        (int)threadIdx.x + S::NTHR * i < n ? wo + i * (S::NTHR / 64 / ConvP<TN, TH>::MT) * 64 : 0x80000000u;
    w[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wr, (int)off, kbase * 2, 0));
  }
}

template <int TN, int TH>
__device__ __forceinline__ void convp_commit_w(const uint4* w, int ck8, bf16_t* s_w) {
  using S = typename ConvP<TN, TH>::S;
  const int n = conv_chunk_steps(9, ck8 * 8) * ConvP<TN, TH>::MT * 64;
#pragma unroll
  for (int i = 0; i < S::NW; ++i) {
    const int u = threadIdx.x + S::NTHR * i;
    if (u < n) *(uint4*)(s_w + u * 8) = w[i];
  }
}

// Loads of one input chunk (channels c0 .. c0 + 8 ck8 of the tile's halo) that one
// buffer holds: src = that buffer at channel c0 of its sample, pitch its channels
// per pixel, half = it is the coarse source. The resource starts at the halo
// tile's first pixel (which may lie before the image) and every lane outside the
// image or the chunk is out of its range.
template <class S, int ETA>
__device__ __forceinline__ void convp_issue_x(ConvStage<S, ETA>& st, const ConvpLane<S>& ln, const ConvGeo& g,
                                              const bf16_t* src, int pitch, bool half, const bf16_t* eta, int c0,
                                              int py0, int px0, int ck8) {
  int tid = threadIdx.x;
  uint32_t yx[S::NU];
#pragma unroll
  for (int i = 0; i < S::NU; ++i) yx[i] = ln.yx[i];
  if constexpr (S::TN > 32) {
    // recomputed per item (about eight VALU operations a pixel): hoisted out of the item
    // loop, the offsets for every source would not leave registers for 64 channels
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int i = 0; i < S::NU; ++i) asm volatile("" : "+v"(yx[i]));
  }
  const int c8 = tid & 3;
  const int Wc = g.W >> 1;
  const int64_t pb = (int64_t)(py0 - 1) * g.W + px0 - 1;
  const int64_t ub = (int64_t)((py0 >> 1) - 1) * Wc + (px0 >> 1) - 1;
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(src + (half ? ub : pb) * pitch), (short)0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t er = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(eta + (ETA == kEtaNode ? pb : pb * g.cin8 + c0)), (short)0, 0x7fffffff, 0x00020000);
  const bool whole = ck8 == 4 && py0 >= 1 && px0 >= 1 && py0 + S::TH + 1 <= g.H && px0 + kCTW + 1 <= g.W;
  const uint32_t pitch2 = pitch * 2, cb = c8 * 16;
  uint32_t bad[S::NU];
#pragma unroll
  for (int i = 0; i < S::NU; ++i)
    bad[i] = (i + 1) * S::PPR <= S::NPIX || (tid >> 2) + i * S::PPR < S::NPIX ? 0u : 0x80000000u;
  if (!whole) {
    const int ylo = 1 - py0, yn = g.H, xlo = 1 - px0, xn = g.W;  // rows and columns of the image
#pragma unroll
    for (int i = 0; i < S::NU; ++i) {
      const int ly = (int)(yx[i] & 0xffffu), lx = (int)(yx[i] >> 16);
      const bool in = c8 < ck8 && (uint32_t)(ly - ylo) < (uint32_t)yn && (uint32_t)(lx - xlo) < (uint32_t)xn;
      bad[i] = in ? bad[i] : 0x80000000u;
    }
  }
#pragma unroll
  for (int i = 0; i < S::NU; ++i) {
    const uint32_t rel = __umul24(yx[i] & 0xffffu, g.W) + (yx[i] >> 16);
    uint32_t off;
    if (half) {
      const uint32_t t = yx[i] + 0x00010001u;
      off = __umul24(__umul24((t >> 1) & 0x7fffu, Wc) + (t >> 17), pitch2) + cb;
    } else {
      off = __umul24(rel, pitch2) + cb;
    }
    st.x[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off | bad[i]), 0, 0));
    if constexpr (ETA == kEtaNode)
      st.e1[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(er, (int)(rel * 2u | bad[i]), 0, 0);
    if constexpr (ETA == kEtaChannel) {
      const uint32_t eo = __umul24(rel, g.cin8 * 2) + cb;
      st.e[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(er, (int)(eo | bad[i]), 0, 0));
    }
  }
}

template <class S, int ETA>
__device__ __forceinline__ void convp_commit_x(const ConvStage<S, ETA>& st, int ck8, bf16_t* s_x) {
  const int c8 = threadIdx.x & 3, p0 = threadIdx.x >> 2;
  static_assert(S::PPR % 8 == 0 && S::G8 == 4, "a thread's pixels share one permutation");
  if (c8 < ck8) {
    bf16_t* sp = s_x + convp_slot(p0, c8);
#pragma unroll
    for (int i = 0; i < S::NU; ++i) {
      if ((i + 1) * S::PPR <= S::NPIX || p0 + i * S::PPR < S::NPIX) {
        uint4 v = st.x[i];
        if constexpr (ETA == kEtaChannel) v = mul_bf16x8(v, st.e[i]);
        if constexpr (ETA == kEtaNode) v = mul_bf16x8_s(v, st.e1[i]);
        *(uint4*)(sp + i * S::PPR * 32) = v;
      }
    }
  }
}

// A full chunk: K-step = tap. swz[m]: this lane's element offset for a pixel
// congruent to m (mod 8) past the lane's first halo pixel, less that pixel's
// distance.
template <int TN, int TH, bool AHEAD>
__device__ __forceinline__ void convp_mfma_full(f32x4_t (&acc)[TN / 16][4], const bf16_t* s_x, const bf16_t* s_w,
                                                const int (&swz)[8], int lane) {
  constexpr int MT = TN / 16, LW = ConvP<TN, TH>::S::LW;
  bf16x8_t b[6][3];
  auto load_row = [&](int r) {
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int o = r * LW + dx;
      b[r][dx] = *(const bf16x8_t*)(s_x + swz[o & 7] + o * 32);
    }
  };
#pragma unroll
  for (int r = 0; r < 4; ++r) load_row(r);
  const bf16_t* wl = s_w + lane * 8;
  bf16x8_t a[1 + AHEAD][MT];  // this tap's weight fragments and (AHEAD) the next one's
  auto load_a = [&](int tap) {
#pragma unroll
    for (int m = 0; m < MT; ++m) a[AHEAD ? tap & 1 : 0][m] = *(const bf16x8_t*)(wl + (tap * MT + m) * 512);
  };
  if (AHEAD) load_a(0);
#pragma unroll
  for (int dy = 0; dy < 3; ++dy) {
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      const int tap = dy * 3 + dx;
      __builtin_amdgcn_sched_barrier(0);  // no more fragments than these in registers
      if (!AHEAD) load_a(tap);
      else if (tap < 8) load_a(tap + 1);
      if (dx == 2 && dy < 2) load_row(4 + dy);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
          acc[m][nt] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[AHEAD ? tap & 1 : 0][m], b[nt + dy][dx], acc[m][nt], 0, 0, 0);
    }
  }
}

// A chunk of ck8 < 4 channel groups: (tap, group) pairs in the packed order.
template <int TN, int TH>
__device__ __forceinline__ void convp_mfma_part(f32x4_t (&acc)[TN / 16][4], const bf16_t* s_x, const bf16_t* s_w,
                                                int ck8, int lane, int wv) {
  constexpr int MT = TN / 16, LW = ConvP<TN, TH>::S::LW;
  const int steps = conv_chunk_steps(9, ck8 * 8);
  const int p0 = 4 * wv * LW + (lane & 15);
  const int inv = ck8 == 3 ? 22 : 64 / ck8;  // G / ck8 = G * inv >> 6 for G < 28
#pragma unroll 1
  for (int st = 0; st < steps; ++st) {
    const int G = st * 4 + (lane >> 4);
    int tap = (G * inv) >> 6;
    const int c8 = G - tap * ck8;
    if (tap > 8) tap = 8;  // zero-weight padding group: any in-bounds input
    const int dy = (tap * 11) >> 5, p = p0 + dy * (LW - 3) + tap;
    bf16x8_t a[MT], b[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) b[nt] = *(const bf16x8_t*)(s_x + convp_slot(p + nt * LW, c8));
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = *(const bf16x8_t*)(s_w + (st * MT + m) * 512 + lane * 8);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) acc[m][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b[nt], acc[m][nt], 0, 0, 0);
  }
}

// Place of an item in a workgroup's list: chunk (from the launch's first) and tile.
template <int TH>
struct ConvpPos {
  int k, py0, px0;
  __device__ __forceinline__ void next(int nch, int W) {
    if (++k < nch) return;
    k = 0;
    px0 += kCTW;
    if (px0 >= W) px0 = 0, py0 += TH;
  }
};

// ONE: one chunk; PART: the last chunk holds fewer than four channel groups.
template <int TN, int TH, int ETA, bool WRES, bool GRP, bool XU, bool OUTF, bool ONE, bool PART>
__global__ __launch_bounds__(TH * 16) __attribute__((amdgpu_waves_per_eu(TH == 16 && !ONE ? 1 : 2))) void k_convp(
    ConvGeo g, const bf16_t* __restrict__ x, const bf16_t* __restrict__ eta, const bf16_t* __restrict__ wp, int Kp,
    const float* __restrict__ bias, bf16_t* __restrict__ y, int tiles_per_wg, float* __restrict__ kpart_l, int ksplit_l,
    const ConvMember* __restrict__ mem, int nmem, OutFold of) {
  using S = typename ConvP<TN, TH>::S;
  constexpr int MT = ConvP<TN, TH>::MT, XB = ConvP<TN, TH>::XB, WB = ConvP<TN, TH>::WB;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];  // two input buffers, the stores' line buffers, the weight slices
  __shared__ __attribute__((aligned(16))) float s_b[TN];
  bf16_t* s_w = smem + 2 * XB + S::NTHR / 64 * 512;

  // K shares: a member's own, or the launch's (only the 16-row tiles are launched with a split)
  float* kpart = TH == 16 ? kpart_l : nullptr;
  int t0, smp, ksp, nbs, ksplit = TH == 16 ? ksplit_l : 1;
  if constexpr (GRP) {
    int lo = 0, hi = nmem - 1;  // the last member whose first workgroup is <= blockIdx.x
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (mem[mid].wg0 <= (int)blockIdx.x) lo = mid;
      else hi = mid - 1;
    }
    const ConvMember& M = mem[lo];
    if (M.skip && __builtin_amdgcn_readfirstlane(*M.skip) != 0) return;
    g = M.g;
    x = M.x;
    eta = M.eta;
    y = M.y;
    kpart = M.kpart;
    ksplit = M.ks;
    const int local = (int)blockIdx.x - M.wg0;
    ksp = local / M.nwt;
    t0 = (local - ksp * M.nwt) * tiles_per_wg;
    smp = 0;
    nbs = 1;
  } else {
    // workgroup b runs on XCD b % 8: each XCD takes a contiguous band of tiles
    const int G = gridDim.x, per = (G + 7) / 8, b = blockIdx.x;
    const int xcd = b & 7, big = G - 8 * (per - 1);  // the first `big` XCDs hold per workgroups
    t0 = (xcd * per - max(0, xcd - big) + (b >> 3)) * tiles_per_wg;
    smp = blockIdx.z / ksplit;
    ksp = blockIdx.z - smp * ksplit;
    nbs = gridDim.z / ksplit;
  }
  const int tiles_x = (g.W + kCTW - 1) / kCTW;
  const int tiles = tiles_x * ((g.H + TH - 1) / TH);
  const int nt_wg = min(tiles_per_wg, tiles - t0);
  const int co0 = blockIdx.y * TN;
  x += smp * g.x_bstride;
  y += smp * g.y_bstride;
  const bf16_t* x1 = g.x1 ? g.x1 + smp * g.x1_bstride : x;
  const bf16_t* xu = XU ? g.xu + smp * g.xu_bstride : x;
  if (ETA != kEtaNone) eta += smp * g.e_bstride;
  else eta = x;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* s_t = smem + 2 * XB + wv * 512;
  if (threadIdx.x < TN) s_b[threadIdx.x] = (bias && co0 + (int)threadIdx.x < g.cout) ? bias[co0 + threadIdx.x] : 0.f;
  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(wp), (short)0, (int)((int64_t)g.cout * Kp * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t yr =
      __builtin_amdgcn_make_buffer_rsrc(y, (short)0, (int)((int64_t)g.H * g.W * g.y_pitch * 2), 0x00020000);
  const bool pool = g.pool_y != nullptr;
  const __amdgpu_buffer_rsrc_t pr = __builtin_amdgcn_make_buffer_rsrc(
      pool ? g.pool_y + smp * g.pool_bstride : y, (short)0,
      pool ? (int)((int64_t)(g.H / 2) * (g.W / 2) * g.pool_pitch * 2) : 0, 0x00020000);
  const int nch_all = (g.cin8 + S::CK - 1) / S::CK;
  const int cps = (nch_all + ksplit - 1) / ksplit;
  const int c_lo = ksp * cps;
  const int nch = min(cps, nch_all - c_lo);
  const int items = nt_wg * nch;
  if (items <= 0) return;
  auto ck8_of = [&](int k) { return PART ? min(S::CK, g.cin8 - (c_lo + k) * S::CK) / 8 : 4; };
  // chunks of four groups (a share of a split K may end before the partial one)
  const int nfull = PART && c_lo + nch == nch_all ? nch - 1 : nch;

  ConvpLane<S> ln;
#pragma unroll
  for (int i = 0; i < S::NU; ++i) {
    const int p = (threadIdx.x >> 2) + S::PPR * i, ly = p / S::LW, lx = p - ly * S::LW;
    ln.yx[i] = (uint32_t)(ly | lx << 16);
  }
  {
    const int f = threadIdx.x >> 6;
    const int r = (f % MT) * 16 + (lane & 15), q = (f / MT) * 4 + (lane >> 4);
    ln.wo = (uint32_t)(((co0 + r) * Kp + q * 8) * 2);
  }
  int swz[8];  // see convp_mfma_full
  {
    const int p0 = 4 * wv * S::LW + (lane & 15);
#pragma unroll
    for (int m = 0; m < 8; ++m) swz[m] = p0 * 32 + (((lane >> 4) ^ (((p0 + m) >> 1) & 3)) * 8);
  }
  f32x4_t acc[MT][4];
  constexpr int DEPTH = TN == 32 && (ONE || TH == 16) ? 2 : 1;  // items in flight to registers
  ConvStage<S, ETA> stg[DEPTH];
  float4 fpre[OUTF ? MT : 1][4];  // fold weights of the tile in acc

  ConvpPos<TH> pc;  // the item computed
  pc.k = 0;
  pc.py0 = t0 / tiles_x;
  pc.px0 = (t0 - pc.py0 * tiles_x) * kCTW;
  pc.py0 *= TH;
  ConvpPos<TH> pl = pc;              // the next item to load
  int ni = 0, nc = 0, kc = 0;    // items loaded, items written to LDS, chunk of the next one to write
  auto issue = [&](ConvStage<S, ETA>& st) __attribute__((always_inline)) {
    if (ni >= items) return;
    const int c0 = (c_lo + pl.k) * S::CK, ck8 = ck8_of(pl.k), ce = c0 + ck8 * 8;
    if (XU && ce <= g.cu) convp_issue_x<S, ETA>(st, ln, g, xu + c0, g.xu_pitch, true, eta, c0, pl.py0, pl.px0, ck8);
    else if (c0 >= g.c1)
      convp_issue_x<S, ETA>(st, ln, g, x1 + c0 - g.c1, g.x1_pitch, false, eta, c0, pl.py0, pl.px0, ck8);
    else
      convp_issue_x<S, ETA>(st, ln, g, x + c0, g.x_pitch, false, eta, c0, pl.py0, pl.px0, ck8);
    if constexpr (!WRES) convp_issue_w<TN, TH>(st.w, ln.wo, wr, ck8, (c_lo + pl.k) * S::SMAX * 32);
    ++ni;
    pl.next(nch, g.W);
  };
  auto commit = [&](const ConvStage<S, ETA>& st) __attribute__((always_inline)) {
    if (nc >= items) return;
    convp_commit_x<S, ETA>(st, ck8_of(kc), smem + (nc & 1) * XB);
    if constexpr (!WRES) convp_commit_w<TN, TH>(st.w, ck8_of(kc), s_w + (nc & 1) * WB);
    ++nc;
    kc = kc + 1 == nch ? 0 : kc + 1;
  };
  auto mfma = [&](auto part, int it, const ConvpPos<TH>& p) __attribute__((always_inline)) {
    const bf16_t* sx = smem + (it & 1) * XB;
    const bf16_t* sw = s_w + (WRES ? p.k : it & 1) * WB;
    if (p.py0 + 4 * wv >= g.H) return;  // this wavefront's rows lie past the image
    if constexpr (OUTF) {
      if (p.k + 1 == nch) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
          const int py = min(p.py0 + 4 * wv + nt, g.H - 1), px = min(p.px0 + (lane & 15), g.W - 1);
          const float* f = of.fold + ((int64_t)py * g.W + px) * of.pitch;
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const int col = m * 16 + 4 * (lane >> 4);
            fpre[m][nt] = *(const float4*)(f + (col < of.c0 ? col : 0));
          }
        }
      }
    }
    if (p.k == 0) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[m][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    if (PART && (decltype(part)::value || (TH == 16 && !ONE && p.k == nfull)))
      convp_mfma_part<TN, TH>(acc, sx, sw, ck8_of(p.k), lane, wv);
    else if constexpr (!decltype(part)::value) convp_mfma_full<TN, TH, WRES || TN == 32>(acc, sx, sw, swz, lane);
  };
  auto store = [&](const ConvpPos<TH>& p) __attribute__((always_inline)) {
    const int pyr = p.py0 + 4 * wv;
    if (p.k + 1 < nch || pyr >= g.H) return;
    if constexpr (OUTF)
      conv_out_epilogue<MT, 4>(acc, g, s_b, pyr, p.px0 + (lane & 15), of, smp,
                               [&](int m, int nt, int64_t) { return fpre[m][nt]; });
    else
      conv_epilogue<TN, 4, false, false, false>(acc, g, s_b, co0, pyr, p.px0 + (lane & 15), s_t, yr, pr, of, smp, nbs, ksp,
                                                ksplit, kpart);
  };
  // The second half of the wavefronts stages one item further ahead, its barrier
  // between the MFMAs and the writes to LDS: item i + 2's buffer is item i's. (A 1024^2
  // forward takes 568 us without this, 16 mixed grids 3.50 instead of 3.40 ms.) Not with
  // 16-row tiles, whose four wavefronts have a SIMD each, nor with up to four items: there
  // the wait for the second item before the first barrier costs more (a 64^2 forward
  // takes 154.5 us with it and 145.4 without; 1024^2 555.3 and 552.9 with the line at
  // four, 559 at eight).
  const bool late = TH == 32 && (GRP || items > 4) && wv >= S::NTHR / 128;
  // Loads of the first two items and of the resident weights are in flight together.
  {
    ConvStage<S, ETA> s1;
    issue(stg[0]);
    if constexpr (WRES) {
      uint4 w[2][S::NW];
      convp_issue_w<TN, TH>(w[0], ln.wo, wr, ck8_of(0), c_lo * S::SMAX * 32);
      if (nch > 1) convp_issue_w<TN, TH>(w[1], ln.wo, wr, ck8_of(1), (c_lo + 1) * S::SMAX * 32);
      issue(s1);
      convp_commit_w<TN, TH>(w[0], ck8_of(0), s_w);
      if (nch > 1) convp_commit_w<TN, TH>(w[1], ck8_of(1), s_w + WB);
      for (int k = 2; k < nch; k += 2) {
        convp_issue_w<TN, TH>(w[0], ln.wo, wr, ck8_of(k), (c_lo + k) * S::SMAX * 32);
        if (k + 1 < nch) convp_issue_w<TN, TH>(w[1], ln.wo, wr, ck8_of(k + 1), (c_lo + k + 1) * S::SMAX * 32);
        convp_commit_w<TN, TH>(w[0], ck8_of(k), s_w + k * WB);
        if (k + 1 < nch) convp_commit_w<TN, TH>(w[1], ck8_of(k + 1), s_w + (k + 1) * WB);
      }
    } else {
      issue(s1);
    }
    commit(stg[0]);
    if (late) commit(s1);
    else stg[0] = s1;
  }
  if (late) issue(stg[0]);
  if constexpr (DEPTH == 2) issue(stg[1]);
  __syncthreads();
  int it = 0;
  auto step = [&](auto part, ConvStage<S, ETA>& st) __attribute__((always_inline)) {
    mfma(part, it, pc);
    if (late) __syncthreads();
    commit(st);
    issue(st);
    store(pc);
    pc.next(nch, g.W);
    ++it;
    if (!late) __syncthreads();
  };
  const std::bool_constant<PART> last;
  if constexpr (ONE) {
    while (it < items) {
      step(last, stg[0]);
      if constexpr (DEPTH == 2) {
        if (it < items) step(last, stg[1]);
      }
    }
  } else if constexpr (DEPTH == 2) {
    while (it < items) {
      step(std::false_type{}, stg[0]);
      if (it < items) step(std::false_type{}, stg[1]);
    }
  } else {
    for (int t = 0; t < nt_wg; ++t) {
      for (int k = 0; k < nfull; ++k) step(std::false_type{}, stg[0]);
      if (PART && nfull < nch) step(last, stg[0]);
    }
  }
}

// LDS of the pipelined kernel: two input buffers, the line buffers and nw weight slices.
template <int TN, int TH>
static size_t convp_lds(int nw) {
  return (2 * (size_t)ConvP<TN, TH>::XB + TH * 16 / 64 * 512 + (size_t)nw * ConvP<TN, TH>::WB) * sizeof(bf16_t);
}

// Weight slices kept for the launch: all chunks where they fit beside the
// input buffers (160 KB of LDS), else none (two slices in turn).
template <int TN, int TH>
static bool convp_wres(int nch) { return convp_lds<TN, TH>(nch) <= 158 * 1024; }

// The pipelined kernel of a launch: chunks resident or not, one chunk, a partial one.
template <int TN, int TH, int ETA, bool GRP, bool XU, bool OUTF>
static void convp_launch_t(const ConvpLaunch& L, hipStream_t s) {
  auto go = [&](auto wres, auto one, auto pt) {
    k_convp<TN, TH, ETA, decltype(wres)::value, GRP, XU, OUTF, decltype(one)::value, decltype(pt)::value>
        <<<L.grid, TH * 16, convp_lds<TN, TH>(wres ? L.nch : 2), s>>>(L.g, L.x, L.eta, L.wp, L.Kp, L.bias, L.y, L.run,
                                                                      L.kpart, L.ks, L.mem, L.nmem, L.of);
  };
  const std::true_type yes;
  const std::false_type no;
  const bool part = L.part;
  if constexpr (OUTF) {  // (one chunk: the caller's rule)
    part ? go(yes, yes, yes) : go(yes, yes, no);
  } else {
    if constexpr (TN == 32 && !XU) {
      if (L.nch == 1) {
        part ? go(yes, yes, yes) : go(yes, yes, no);
        return;
      }
    }
    // resident slices serve runs of tiles: not the 16-row tiles, of which a workgroup
    // has one or two, nor 64 channels with a coarse source (at least 128 input channels)
    if constexpr (TH == 32 && !(XU && TN == 64)) {
      if (convp_wres<TN, TH>(L.nch)) {
        part ? go(yes, no, yes) : go(yes, no, no);
        return;
      }
    }
    part ? go(no, no, yes) : go(no, no, no);
  }
}

template <int TN, int TH, int ETA>
static void convp_launch_eta(const ConvpLaunch& L, hipStream_t s) {
  if constexpr (TN == 32) {
    if (L.outf) return convp_launch_t<TN, TH, ETA, false, false, true>(L, s);
  }
  if constexpr (TH == 32) {
    if (L.mem) {
      L.xu ? convp_launch_t<TN, TH, ETA, true, true, false>(L, s)
           : convp_launch_t<TN, TH, ETA, true, false, false>(L, s);
      return;
    }
  }
  L.xu ? convp_launch_t<TN, TH, ETA, false, true, false>(L, s)
       : convp_launch_t<TN, TH, ETA, false, false, false>(L, s);
}

template <int TN, int TH>
static void convp_launch(const ConvpLaunch& L, hipStream_t s) {
  if (L.eta_mode == kEtaNone) convp_launch_eta<TN, TH, kEtaNone>(L, s);
  else if (L.eta_mode == kEtaNode) convp_launch_eta<TN, TH, kEtaNode>(L, s);
  else convp_launch_eta<TN, TH, kEtaChannel>(L, s);
}

}  // namespace ppe
