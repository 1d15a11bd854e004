// Device code that both 3x3 convolution kernels share: the tile's shape, staging
// registers, bias and activation, and the stores of a tile's results.
#pragma once
#include "common.hpp"
#include "net_common.hpp"
#include "net_kernels.hpp"

namespace ppe {

constexpr int kCTH = 16, kCTW = 16;  // pixel tile of the convolution kernel

template <int TN_, int TAPS_, int TH_ = kCTH, int NTHR_ = 256>
struct ConvShape {
  static constexpr int TN = TN_, TAPS = TAPS_, TH = TH_, NTHR = NTHR_;
  static constexpr int HALO = TAPS == 9 ? 1 : 0;
  static constexpr int LW = kCTW + 2 * HALO, LH = TH + 2 * HALO;
  static constexpr int NPIX = LW * LH;
  // input channels staged per item: 32 for 3x3 layers, 64 for 1x1 layers (the
  // packed weight layout is the same: a full 64-channel chunk of a 1x1 layer
  // is two full 32-channel chunks)
  static constexpr int CK = TAPS == 9 ? kConvCK : 2 * kConvCK;
  static constexpr int G8 = CK / 8;                             // 8-channel groups of a staged pixel
  static constexpr int PPR = NTHR / G8;                         // pixels staged per round of the workgroup
  static constexpr int CKP = CK + 8;                            // LDS pitch of a staged pixel (bf16)
  static constexpr int SMAX = (TAPS * G8 + 3) / 4;              // K-steps of a full chunk
  static constexpr int WQ = SMAX * 4;                           // 8-value groups of a full weight row
  static constexpr int WKP = SMAX * 32 + 8;                     // LDS pitch of a staged weight row
  static constexpr int NU = (NPIX + PPR - 1) / PPR;             // staged pixels per thread
  static constexpr int NW = (TN * WQ + NTHR - 1) / NTHR;        // weight groups per thread
  // this thread's pixel offsets kept in registers for the launch where they fit
  // (32 output channels per workgroup, 16-row tiles); recomputed per item
  // (about six VALU operations a pixel) elsewhere
  static constexpr bool KEEP = TN == 32 && TH == kCTH;
};

// Registers of one item's loads, between issue and the write to LDS.
template <class S, int ETA>
struct ConvStage {
  static constexpr int NU = S::NU;
  uint4 x[NU], w[S::NW];
  uint4 e[ETA == kEtaChannel ? NU : 1];
  uint32_t e1[ETA == kEtaNode ? NU : 1];
};

// One 4-channel group of the DeepONet output contraction: BF16 activations
// d (two packed pairs) times fold weights w, a product and three FMAs in
// channel order. Both output paths (the separate kernel and the fused
// convolution epilogue) use it, so they round alike.
__device__ __forceinline__ float out_group4(uint2 d, float4 w) {
  float e = __fmul_rn(bf2f((bf16_t)(d.x & 0xffff)), w.x);
  e = __fmaf_rn(bf2f((bf16_t)(d.x >> 16)), w.y, e);
  e = __fmaf_rn(bf2f((bf16_t)(d.y & 0xffff)), w.z, e);
  return __fmaf_rn(bf2f((bf16_t)(d.y >> 16)), w.w, e);
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Orders a wavefront's LDS accesses across its lanes (the hardware keeps their
// order; this keeps the compiler's).
__device__ __forceinline__ void wave_lds_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// A 16-byte buffer store, its whole offset in the vector register: with a scalar
// offset beside it, the store read its data registers after the instructions that
// followed had written them anew (wrong values now and then, on this chip); without
// one the compiler keeps the distance that the store needs.
__device__ __forceinline__ void store_b128(u32x4 v, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, 0);
}

// 2 x 2 average of two rows' four channels (a: upper row, b: lower) with the next
// column's lane: the even lane forms channels 0 and 1 of the group, the odd lane 2 and
// 3 (the neighbour's word by a lane swap within pairs), summed in the order and
// rounding of the pooling kernel from the stored BF16 values.
__device__ __forceinline__ uint32_t conv_pool_word(u32x2 a, u32x2 b, int lane) {
  const bool odd = lane & 1;
  const u32x2 r[2] = {a, b};
  float s0 = 0.f, s1 = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? r[i].x : r[i].y), 0xb1, 0xf, 0xf, true);
    const uint32_t w[2] = {odd ? o : r[i].x, odd ? r[i].y : o};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      s0 += bf2f((bf16_t)(w[k] & 0xffff));
      s1 += bf2f((bf16_t)(w[k] >> 16));
    }
  }
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){0.25f * s0, 0.25f * s1}, bf16x2_t));
}

// Bias and activation of a tile's sums. ReLU and no activation share one maximum
// per value (with 0, or with NaN, which leaves every value as it is): the branch
// costs more than the operation.
template <int MT, int NT>
__device__ __forceinline__ void conv_act(f32x4_t (&acc)[MT][NT], const float* s_b, int act) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const f32x4_t b = *(const f32x4_t*)(s_b + mt * 16 + 4 * (lane >> 4));
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[mt][nt][j] += b[j];
  }
  const float lo = act == 1 ? 0.f : __builtin_nanf("");
  if (act != 2) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < 4; ++j)  // (the builtin maximum canonicalises both operands first)
          asm("v_max_f32 %0, %1, %2" : "=v"(acc[mt][nt][j]) : "v"(acc[mt][nt][j]), "s"(lo));
  } else {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[mt][nt][j] = tanh_nn(acc[mt][nt][j]);
  }
}

// DeepONet output instead of the stored activations (TN = 32 and c0 <= 32: the
// workgroup holds every channel of its pixels). The lane's channel group
// q = 4 mt + (lane >> 4) takes the place of lane q of k_deeponet_out: the same
// BF16-rounded values, the same group sum, and the same pairwise order across
// groups (q ^ 4 within the lane, then lanes ^ 32 and ^ 16), so the result is that
// kernel's bit for bit. fw(mt, nt, pixel): the lane's four fold weights.
template <int MT, int NT, class F>
__device__ __forceinline__ void conv_out_epilogue(f32x4_t (&acc)[MT][NT], const ConvGeo& g, const float* s_b,
                                                  int pyr, int px, const OutFold& of, int smp, F&& fw) {
  const int lane = threadIdx.x & 63;
  conv_act<MT, NT>(acc, s_b, g.act);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int py = pyr + nt;
    const bool pok = py < g.H && px < g.W;
    const int64_t pix = (int64_t)py * g.W + px;
    float sq[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int col = mt * 16 + 4 * (lane >> 4);
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = acc[mt][nt][j];
      const uint2 pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[0], v[1]}, bf16x2_t)),
                        __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[2], v[3]}, bf16x2_t))};
      sq[mt] = 0.f;
      if (pok && col < of.c0) sq[mt] += out_group4(pk, fw(mt, nt, pix));
    }
    float sv = MT == 2 ? sq[0] + sq[1] : sq[0];
    sv += __shfl_xor(sv, 32);
    sv += __shfl_xor(sv, 16);
    if (pok && lane < 16)
      of.y[(int64_t)smp * g.H * g.W + pix] = of.gamma[0] * (sv + of.fold[pix * of.pitch + of.c0]);
  }
}

// Epilogue of one tile: lane holds out[co0 + mt*16 + 4*(lane>>4) + j][pixel (row
// pyr + nt, column px)]; bias, activation and the store (or the K share's
// partial sums, or the DeepONet output); acc is zero again afterwards (ZERO).
template <int TN, int NT, bool UP, bool OUTF, bool ZERO = true>
__device__ __forceinline__ void conv_epilogue(f32x4_t (&acc)[TN / 16][NT], const ConvGeo& g, const float* s_b, int co0,
                                              int pyr, int px, bf16_t* s_t, __amdgpu_buffer_rsrc_t yr,
                                              __amdgpu_buffer_rsrc_t pr, const OutFold& of, int smp, int nbs, int ksp, int ksplit,
                                              float* __restrict__ kpart) {
  constexpr int MT = TN / 16;
  const int lane = threadIdx.x & 63;
  const int WO = UP ? 2 * g.W : g.W;
  const bool pool = g.pool_y != nullptr;
  if (ksplit > 1) {
    // partial sums of this share of K, [ksplit][sample][pixel][gridDim.y * TN] FP32
    const int cp = gridDim.y * TN;
    float* pp = kpart + ((int64_t)ksp * nbs + smp) * g.H * g.W * cp;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int co = co0 + mt * 16 + 4 * (lane >> 4);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int py = pyr + nt;
        if (co < g.cout && py < g.H && px < g.W)
          *(f32x4_t*)(pp + ((int64_t)py * g.W + px) * cp + co) = acc[mt][nt];
        acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
    }
    return;
  }
  if constexpr (OUTF) {
    static_assert(TN == 32 && !UP, "fused output: 32 output channels per workgroup");
    conv_out_epilogue<MT, NT>(acc, g, s_b, pyr, px, of, smp, [&](int mt, int, int64_t pix) {
      return *(const float4*)(of.fold + pix * of.pitch + mt * 16 + 4 * (lane >> 4));
    });
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    return;
  }
  conv_act<MT, NT>(acc, s_b, g.act);
  // store offset: this lane's pixel column and channel, then a scalar per row
  // (lanes past the row or the last channel out of range)
  const int py0 = __builtin_amdgcn_readfirstlane(pyr);
  const int rstep = WO * g.y_pitch * 2, prstep = (g.W >> 1) * g.pool_pitch * 2;
  if constexpr (!UP) {
    // Stores of whole 64-byte lines: the lanes that hold a pixel's channels lie 16
    // apart, and eight bytes a lane at a pixel's stride were one request each (3-6 k
    // cycles a tile at 1024^2, 32 channels, more than its MFMAs). 32 channels of a
    // pixel row go through 1 KB of the wavefront's own LDS, 16-byte groups permuted by
    // the pixel, and out with four consecutive lanes a pixel. LDS takes a wavefront's
    // instructions in order, so the rows follow one another without a wait.
    if ((g.cout | g.y_pitch | g.y_off | (pool ? g.pool_pitch : 0)) % 8 == 0) {
      static_assert(MT % 2 == 0, "pairs of 16 channels");
      const int pl = lane & 15, q = lane >> 4, pt = lane >> 2, ct = lane & 3;
      bf16_t* sw = s_t + pl * 32 + (q & 1) * 4;
      const int wsw = (pl >> 1) & 3;
      bf16_t* w0 = sw + (((q >> 1) ^ wsw) * 8);
      bf16_t* w1 = sw + (((2 + (q >> 1)) ^ wsw) * 8);
      const uint4* rd = (const uint4*)(s_t + pt * 32 + ((ct ^ ((pt >> 1) & 3)) * 8));
      const int pxt = px - pl + pt;  // the pixel and channels this lane stores
      const uint32_t tb = (uint32_t)((pxt * g.y_pitch + g.y_off + co0 + ct * 8) * 2);
      const uint32_t tp = (uint32_t)(((((px - pl) >> 1) + pt) * g.pool_pitch + co0 + ct * 8) * 2);
#pragma unroll
      for (int mp = 0; mp < MT / 2; ++mp) {
        const bool okt = co0 + mp * 32 + ct * 8 < g.cout && pxt < g.W;
        const uint32_t o = okt ? tb + mp * 64u : 0x80000000u;
        u32x2 pk[2][NT];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const f32x4_t v = acc[2 * mp + h][nt];
            pk[h][nt] = u32x2{__builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[0], v[1]}, bf16x2_t)),
                              __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[2], v[3]}, bf16x2_t))};
          }
        u32x4 t[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          *(u32x2*)w0 = pk[0][nt];
          *(u32x2*)w1 = pk[1][nt];
          wave_lds_order();
          t[nt] = *(const u32x4*)rd;
          wave_lds_order();
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (py0 + nt < g.H) store_b128(t[nt], yr, o + (uint32_t)((py0 + nt) * rstep));
        if (pool) {
#pragma unroll
          for (int nt = 0; nt < NT; nt += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
              *(uint32_t*)(s_t + (pl >> 1) * 32 + h * 16 + q * 4 + (pl & 1) * 2) =
                  conv_pool_word(pk[h][nt], pk[h][nt + 1], lane);
            wave_lds_order();
            const u32x4 w = *(const u32x4*)(s_t + (lane & 31) * 8);
            wave_lds_order();
            const bool okp = lane < 32 && co0 + mp * 32 + ct * 8 < g.cout && (px - pl) + 2 * pt < g.W;
            if (py0 + nt < g.H)
              store_b128(w, pr, (okp ? tp + mp * 64u : 0x80000000u) + (uint32_t)(((py0 + nt) >> 1) * prstep));
          }
        }
      }
      if constexpr (ZERO) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
      return;
    }
  }
  const uint32_t obase = (uint32_t)(((UP ? 2 * px : px) * g.y_pitch + g.y_off + co0 + 4 * (lane >> 4)) * 2);
  const uint32_t pbase = (uint32_t)(((px >> 1) * g.pool_pitch + co0 + 4 * (lane >> 4)) * 2);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int col = mt * 16 + 4 * (lane >> 4);  // first of this lane's 4 channels within the workgroup's TN
    const bool ok = co0 + col < g.cout && px < g.W;
    const uint32_t ob = ok ? obase + mt * 32u : 0x80000000u;
    u32x2 pk[NT];  // the stored BF16 values (pooling reads them back)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const f32x4_t v = acc[mt][nt];
      pk[nt] = u32x2{__builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[0], v[1]}, bf16x2_t)),
                     __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){v[2], v[3]}, bf16x2_t))};
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int py = py0 + nt;
      if (py >= g.H) continue;
      if (!UP) {
        __builtin_amdgcn_raw_buffer_store_b64(pk[nt], yr, (int)ob, py * rstep, 0);
      } else {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int bb = 0; bb < 2; ++bb)
            __builtin_amdgcn_raw_buffer_store_b64(pk[nt], yr, (int)ob, (2 * py + a) * rstep + bb * g.y_pitch * 2, 0);
      }
    }
    if (!UP && pool) {
#pragma unroll
      for (int nt = 0; nt < NT; nt += 2) {
        const int py = py0 + nt;
        const uint32_t w = conv_pool_word(pk[nt], pk[nt + 1], lane);
        if (py < g.H)
          __builtin_amdgcn_raw_buffer_store_b32(w, pr, (int)(ok ? pbase + mt * 32u + (lane & 1) * 4u : 0x80000000u),
                                                (py >> 1) * prstep, 0);
      }
    }
    if constexpr (ZERO) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
  }
}

}  // namespace ppe
