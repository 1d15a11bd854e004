// Host-side declarations of the training kernel launchers.
#pragma once
#include "net_common.hpp"

namespace ppe {

struct WgradGeo {
  int H, W, nb;
  int cin8;           // input pitch (channels per pixel of X and eta)
  int cin;            // real input channels (gradient rows written)
  int cout;           // output channels
  int dp_pitch;       // pitch of the output gradient
  int64_t x_bstride, dp_bstride, e_bstride;  // per-sample strides (e_bstride unused without eta)
  int eta_node;       // 1: eta holds one weight per pixel ([H][W] per sample), else one per input channel
};

// Partial rows of a 1x1 layer's weight gradient ([cout][cin] each).
void launch_wgrad1(const WgradGeo& g, const bf16_t* dp, const bf16_t* x, float* part, int nsplit, hipStream_t s);
// Partial rows of a 3x3 layer's weight gradient ([cout][cin][9] each, at most
// cap floats in all); returns their number.
int launch_wgrad9(const WgradGeo& g, const bf16_t* dp, const bf16_t* x, const bf16_t* eta, float* part, int64_t cap,
                  hipStream_t s);
// Backward of a 1x1 layer over nb samples of hw pixels: d [nb][hw][cout], x
// [nb][hw][cin8] its input, wT the packed transposed weights (Kp values per input
// channel), dx [nb][hw][cin8] the gradient of the input before its activation act
// (1 ReLU, 2 tanh, 0 none), or NULL. With gamma: d holds the other factor S of
// the DeepONet contraction and the gradient is bf16(gamma (scale dy) S).
struct Bwd1x1 {
  int hw, nb;
  int cout, cin, cin8;
  const bf16_t* d;
  const bf16_t* x;
  const bf16_t* wT;
  int Kp, act;
  bf16_t* dx;
  const float *gamma, *dy;
  float scale;
};
bool bwd1x1_fits(int cout, int cin8);
// Partial rows [cout][cin] of the weight gradient (at most cap floats, 1024 rows and `tiles` rows); returns their number.
int launch_bwd1x1(const Bwd1x1& g, int64_t tiles, float* part, int64_t cap, hipStream_t s);
// Sums of partial rows, out[k] = sum_b part[b][k] (nparts rows of len), as
// launch_reduce_rows does them, all of a table in one launch.
constexpr int kMaxRows = 72;
struct RowSum {
  const float* part;
  int nparts, len;
  float* out;
};
struct RowTable {
  int n;
  RowSum row[kMaxRows];
};
void launch_reduce_table(const RowTable& t, hipStream_t s);
// Partial rows of a bias gradient, of gamma's, and of a local-weight network's.
constexpr int kBiasParts = 1024, kGammaParts = 2048, kPhiParts = 2048;
void launch_reduce_rows(const float* part, int nparts, int64_t len, float scale, float* out, hipStream_t s);
void launch_bias_grad(const bf16_t* d, int64_t npix, int pitch, int off, int C, const float* gamma, const float* dy,
                      float scale, float* part, int nparts, hipStream_t s);
void launch_act_bwd(bf16_t* d, int dpitch, const bf16_t* out, int opitch, int ooff, int C, int64_t npix, int mode,
                    hipStream_t s);
void launch_copy_ch(const bf16_t* src, int spitch, int soff, bf16_t* dst, int dpitch, int C, int64_t npix,
                    hipStream_t s);
void launch_up_bwd(int Hc, int Wc, int C, const bf16_t* fine, int fpitch, int64_t f_bs, bf16_t* coarse, int64_t c_bs,
                   int nb, hipStream_t s);
// dE = relu'(E) (dE + 0.25 dpool) over the fine pixels (E: pitch epitch,
// channels from eoff, samples contiguous).
void launch_pool_bwd(int Hc, int Wc, int C, const bf16_t* dpool, int ppitch, int64_t p_bs, const bf16_t* E, int epitch,
                     int eoff, bf16_t* dE, int64_t e_bs, int nb, hipStream_t s);
// dX of a layer with one local weight per node (eta, or none when NULL), in
// place of g = dXbar in dxb; mask: through the ReLU that made x; skip: channels
// [skip_lo, skip_hi) go there (pitch skip_hi - skip_lo), later ones nowhere;
// se (or NULL): dEta per pixel; bias (or NULL): kBiasParts partial rows of the sums of
// dX over pixels, where eta_dx_can_bias. All samples contiguous, cin8 channels a pixel.
struct EtaDx {
  int64_t npix;
  int cin8;
  const bf16_t* x;
  const bf16_t* eta;
  bf16_t* dxb;
  int mask;
  bf16_t* skip;
  int skip_lo, skip_hi;
  float* se;
  float* bias;
};
bool eta_dx_can_bias(int cin8);
void launch_eta_dx(const EtaDx& a, hipStream_t s);
// The layers with one local weight per node of a network (four per level at
// most), for one launch over all of them: eta maps forward, and the gradients
// of their parameters from dEta. eta_off: the layer's first element in eta and
// in se; oW1: its parameters W1 | b1 | W2 | b2 in params and grad. part:
// partial rows (at most kPhiParts x (6 hid + 1) floats per layer).
constexpr int kMaxPhi = 24;
struct PhiLayer {
  int H, W;
  int64_t lv_off, oW1, eta_off;
  int wg0, nwg;  // set by the launchers
};
struct PhiArgs {
  int n, nb, hid;
  const float* lv;
  int64_t lv_stride;
  const float* params;
  bf16_t* eta;
  const float* se;
  float* part;
  PhiLayer layer[kMaxPhi];
};
void launch_eta_nodes(PhiArgs a, hipStream_t s);
void launch_phi_grad(PhiArgs a, float* grad, RowTable& t, hipStream_t s);
void launch_eta_multi(int H, int W, int cin, int cin8, int hid, const float* lv, int64_t lv_stride, const float* W1,
                      const float* b1, const float* W2, const float* b2, bf16_t* eta, int64_t e_bs, int nb,
                      hipStream_t s);
int eta_bwd_len(int cin, int hid);
// Whether the local-weight backward handles a layer of cin inputs (pitch cin8)
// and hid hidden units: cin8 <= 1024 and its LDS rows fit the device.
bool eta_bwd_fits(int cin, int cin8, int hid);
void launch_eta_bwd(int H, int W, int cin, int cin8, int hid, int nb, const float* lv, int64_t lv_stride,
                    const float* W1, const float* b1, const float* W2, const float* b2, const bf16_t* x,
                    const bf16_t* eta, int64_t e_bs, bf16_t* dxb, float* part, int nparts, hipStream_t s);
void launch_fill_static_multi(int H, int W, int pitch, int coff, const float* lv, int64_t lv_stride,
                              const uint8_t* const* masks, int moff, bf16_t* buf, int64_t bstride, int nb,
                              hipStream_t s);
void launch_trunk_input(int H, int W, const float* tin, int64_t t_stride, bf16_t* out, int nb, hipStream_t s);
// y = gamma s and s = sum_k B_k T_k per pixel.
void launch_don_fwd(int64_t n, int P, const bf16_t* B, const bf16_t* T, const float* gamma, float* y, float* sum,
                    hipStream_t s);
// dB = bf16(gamma (scale g) T).
void launch_don_grad(int64_t n, int P, const bf16_t* T, const float* gamma, const float* g, float scale, bf16_t* dB,
                     hipStream_t s);
// kGammaParts shares of gamma's gradient, sum of (scale g) sum over n pixels.
void launch_gamma_grad(int64_t n, const float* g, float scale, const float* sum, float* part, hipStream_t s);
void launch_loss(int64_t n, const float* R, const float* Ay, float* res, double* part, int nparts, hipStream_t s);
void launch_sum_parts(const double* part, int n, double scale, double* out, hipStream_t s);
// Supervised loss (scale- and shift-invariant misfit of y against the FP64
// targets e): per-sample losses into lsamp [nb] and dL/dy (batch mean) into
// dy; part holds [nb][5][nparts] partial sums.
void launch_anorm_loss(int64_t N, int nb, const float* y, const float* Ay, const float* R, const double* e,
                       double* part, int nparts, float* dy, double* lsamp, hipStream_t s);
void launch_sup_loss(int64_t N, int nb, const float* y, const double* e, double* part, int nparts, float* dy,
                     double* lsamp, hipStream_t s);
// Adam step; clip > 0 scales the gradient to norm <= clip first, with ||g||^2
// from the kRedBlocks partials in gpart (launch_sumsq on g).
void launch_sam_perturb(int64_t n, float* w, const float* g, const double* gpart, float rho, hipStream_t s);
void launch_adam(int64_t n, float* w, const float* g, float* m, float* v, float lr, float b1, float b2, float eps,
                 float c1, float c2, const double* gpart, float clip, hipStream_t s);

}  // namespace ppe
