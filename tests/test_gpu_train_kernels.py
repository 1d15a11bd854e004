"""The backward kernels of the training step one by one, through the library's
launchers, on ragged sizes: against FP64 sums in plain torch, and bit for bit against
the separate kernels whose place the one-pass ones take.

Tolerances. Operands are BF16, so every product is exact in FP32; a sum of n of them
in FP32 errs by at most n 2^-23 of the sum of their magnitudes (2^-24 a step, twice that
for the rounding inside an MFMA). A result stored in BF16 (eight significant bits) adds 2^-8 of itself.
What follows a stored sum (the activations' derivatives) is compared bit for bit.
Phi's tanh and exponential are good to about 1e-6, which its gradient's terms see
amplified by at most the sum of |W2| and |Phi| (below 10 here): 1e-5 of the terms' magnitudes, a
tenth of the 1e-4 allowed."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

P, I, L, F = C.c_void_p, C.c_int, C.c_int64, C.c_float
BIAS_PARTS, MAX_ROWS, MAX_PHI, PHI_PARTS = 1024, 72, 24, 2048


class WgradGeo(C.Structure):
    _fields_ = [(n, I) for n in "H W nb cin8 cin cout dp_pitch".split()] + \
               [(n, L) for n in "x_bstride dp_bstride e_bstride".split()] + [("eta_node", I)]


class Bwd1x1(C.Structure):
    _fields_ = [(n, I) for n in "hw nb cout cin cin8".split()] + [("d", P), ("x", P), ("wT", P), ("Kp", I), ("act", I),
                                                                 ("dx", P), ("gamma", P), ("dy", P), ("scale", F)]


class ConvGeo(C.Structure):
    _fields_ = [(n, I) for n in "H W cin8 x_pitch c1 x1_pitch".split()] + \
               [("x1", P), ("x1_bstride", L), ("xu", P), ("cu", I), ("xu_pitch", I), ("xu_bstride", L), ("cout", I),
                ("y_pitch", I), ("y_off", I), ("x_bstride", L), ("y_bstride", L), ("e_bstride", L), ("act", I),
                ("eta_node", I), ("pool_y", P), ("pool_pitch", I), ("pool_bstride", L)]


class EtaDx(C.Structure):
    _fields_ = [("npix", L), ("cin8", I), ("x", P), ("eta", P), ("dxb", P), ("mask", I), ("skip", P), ("skip_lo", I),
                ("skip_hi", I), ("se", P), ("bias", P)]


class PhiLayer(C.Structure):
    _fields_ = [("H", I), ("W", I), ("lv_off", L), ("oW1", L), ("eta_off", L), ("wg0", I), ("nwg", I)]


class PhiArgs(C.Structure):
    _fields_ = [("n", I), ("nb", I), ("hid", I), ("lv", P), ("lv_stride", L), ("params", P), ("eta", P), ("se", P),
                ("part", P), ("layer", PhiLayer * MAX_PHI)]


class RowSum(C.Structure):
    _fields_ = [("part", P), ("nparts", I), ("len", I), ("out", P)]


class RowTable(C.Structure):
    _fields_ = [("n", I), ("row", RowSum * MAX_ROWS)]


NAMES = {
    "wgrad1": ("_ZN3ppe13launch_wgrad1ERKNS_8WgradGeoEPKtS4_PfiP12ihipStream_t", None, [P, P, P, P, I, P]),
    "wgrad9": ("_ZN3ppe13launch_wgrad9ERKNS_8WgradGeoEPKtS4_S4_PflP12ihipStream_t", I, [P, P, P, P, P, L, P]),
    "bwd1x1": ("_ZN3ppe13launch_bwd1x1ERKNS_6Bwd1x1ElPflP12ihipStream_t", I, [P, L, P, L, P]),
    "conv": ("_ZN3ppe11launch_convEibRKNS_7ConvGeoEiPKtS4_S4_iPKfPtP12ihipStream_tPfli", None,
             [I, C.c_bool, P, I, P, P, P, I, P, P, P, P, L, I]),
    "pack_t": ("_ZN3ppe21launch_pack_weights_tEPKfiiiiiPtP12ihipStream_t", None, [P, I, I, I, I, I, P, P]),
    "act_bwd": ("_ZN3ppe14launch_act_bwdEPtiPKtiiiliP12ihipStream_t", None, [P, I, P, I, I, I, L, I, P]),
    "don_grad": ("_ZN3ppe15launch_don_gradEliPKtPKfS3_fPtP12ihipStream_t", None, [L, I, P, P, P, F, P, P]),
    "eta_dx": ("_ZN3ppe13launch_eta_dxERKNS_5EtaDxEP12ihipStream_t", None, [P, P]),
    "can_bias": ("_ZN3ppe15eta_dx_can_biasEi", C.c_bool, [I]),
    "phi_grad": ("_ZN3ppe15launch_phi_gradENS_7PhiArgsEPfRNS_8RowTableEP12ihipStream_t", None, [PhiArgs, P, P, P]),
    "eta_nodes": ("_ZN3ppe16launch_eta_nodesENS_7PhiArgsEP12ihipStream_t", None, [PhiArgs, P]),
    "rows": ("_ZN3ppe19launch_reduce_tableERKNS_8RowTableEP12ihipStream_t", None, [P, P]),
}


@pytest.fixture(scope="module")
def K():
    from paper_2604_01800_amd import ppe
    so = ppe.lib()
    out = {}
    for k, (sym, res, args) in NAMES.items():
        f = getattr(so, sym)
        f.restype, f.argtypes = res, args
        out[k] = f
    return out


def rand(shape, seed, relu=False, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=torch.Generator().manual_seed(seed))
    return (t.relu() if relu else t).to(dtype).cuda()


def ptr(t):
    return None if t is None else t.data_ptr()


def close(got, want, mag, terms, rounded=False):
    """|got - want| <= terms 2^-23 mag (+ 2^-8 |want|), elementwise."""
    err = (got.double() - want).abs()
    bar = terms * 2.0 ** -23 * mag + rounded * 2.0 ** -8 * want.abs() + 1e-30
    assert bool((err <= bar).all()), float((err / bar).max())


@pytest.mark.parametrize("H,W,nb,cout,cin", [
    (7, 5, 1, 8, 8), (29, 37, 3, 24, 10), (29, 37, 3, 40, 18), (16, 48, 2, 32, 64), (21, 50, 2, 72, 34),
    (24, 33, 2, 136, 130), (64, 64, 16, 64, 64), (128, 96, 8, 64, 32), (96, 96, 12, 96, 16),
])
@pytest.mark.parametrize("eta_kind", ["none", "node", "channel"])
def test_weight_gradient_3x3(K, H, W, nb, cout, cin, eta_kind):
    cin8 = (cin + 7) // 8 * 8
    x, d = rand((nb, H, W, cin8), 1, relu=True), rand((nb, H, W, cout), 2)
    x[..., cin:] = 0
    node = eta_kind == "node"
    eta = None if eta_kind == "none" else rand((nb, H, W, 1 if node else cin8), 3, dtype=torch.float32).sigmoid().bfloat16()
    g = WgradGeo(H, W, nb, cin8, cin, cout, cout, H * W * cin8, H * W * cout, H * W * (1 if node else cin8), node)
    cap = 4 << 20
    part = torch.zeros(cap, device="cuda")
    n = K["wgrad9"](C.byref(g), ptr(d), ptr(x), ptr(eta), ptr(part), cap, None)
    got = part[:n * cout * cin * 9].view(n, cout, cin, 3, 3).double().sum(0)
    xb = x if eta is None else (eta.float() * x.float()).bfloat16()
    xp = torch.nn.functional.pad(xb[..., :cin].double(), (0, 0, 1, 1, 1, 1))
    D = d.double().reshape(-1, cout)
    for ty in range(3):
        for tx in range(3):
            X = xp[:, ty:ty + H, tx:tx + W].reshape(-1, cin)
            close(got[:, :, ty, tx], D.T @ X, D.abs().T @ X.abs(), H * W * nb)


@pytest.mark.parametrize("H,W,nb,cout,cin,act,tiles", [
    (7, 5, 1, 8, 8, 1, 1), (29, 37, 3, 24, 40, 1, 40), (29, 37, 3, 40, 24, 2, 5), (16, 8, 2, 128, 128, 2, 1000),
    (21, 50, 2, 72, 128, 1, 9), (33, 31, 2, 128, 72, 0, 1000), (64, 48, 4, 128, 128, 2, 11), (13, 11, 2, 8, 128, 1, 2),
    (13, 11, 2, 128, 8, 1, 2), (29, 37, 1, 128, 2, 2, 17),
])
def test_backward_1x1(K, H, W, nb, cout, cin, act, tiles):
    """One pass against FP64 and, bit for bit, against the weight-gradient, input-gradient
    and activation kernels it stands in for."""
    cin8, hw = (cin + 7) // 8 * 8, H * W
    npix = hw * nb
    x = rand((npix, cin8), 1, relu=act == 1)
    if act == 2:
        x = x.float().tanh().bfloat16()
    x[:, cin:] = 0
    d, w = rand((npix, cout), 2), rand((cout, cin), 3, dtype=torch.float32)
    Kp = (cout + 31) // 32 * 32
    wT = torch.zeros((cin8, Kp), dtype=torch.bfloat16, device="cuda")
    K["pack_t"](ptr(w), cout, cin, cin8, 1, Kp, ptr(wT), None)
    assert torch.equal(wT[:cin, :cout], w.bfloat16().T)
    cap = 4 << 20
    part, ref = torch.zeros(cap, device="cuda"), torch.zeros(cap, device="cuda")
    dx, sep = torch.zeros_like(x), torch.zeros_like(x)
    b = Bwd1x1(hw, nb, cout, cin, cin8, ptr(d), ptr(x), ptr(wT), Kp, act, ptr(dx), None, None, 0.0)
    n = K["bwd1x1"](C.byref(b), tiles, ptr(part), cap, None)
    g = WgradGeo(H, W, nb, cin8, cin, cout, cout, hw * cin8, hw * cout, 0, 0)
    K["wgrad1"](C.byref(g), ptr(d), ptr(x), ptr(ref), n, None)
    assert torch.equal(part[:n * cout * cin], ref[:n * cout * cin])
    cg = ConvGeo(H=H, W=W, cin8=cout, x_pitch=cout, c1=cout, cout=cin8, y_pitch=cin8, x_bstride=hw * cout,
                 y_bstride=hw * cin8)
    K["conv"](1, False, C.byref(cg), nb, ptr(d), None, ptr(wT), Kp, None, ptr(sep), None, None, 0, 0)
    if act:
        K["act_bwd"](ptr(sep), cin8, ptr(x), cin8, 0, cin8, npix, act, None)
    assert torch.equal(dx, sep)
    raw = torch.zeros_like(x)  # dx before the activation's derivative
    b.act, b.dx = 0, ptr(raw)
    K["bwd1x1"](C.byref(b), tiles, ptr(ref), cap, None)
    assert torch.equal(part[:n * cout * cin], ref[:n * cout * cin])
    xf = x.float()
    want = torch.where(x > 0, raw, torch.zeros_like(raw)) if act == 1 else \
        (raw.float() * (1 - xf * xf)).bfloat16() if act == 2 else raw
    assert torch.equal(dx, want)
    D, X, Wb = d.double(), x[:, :cin].double(), w.bfloat16().double()
    close(part[:n * cout * cin].view(n, cout, cin).double().sum(0), D.T @ X, D.abs().T @ X.abs(), npix)
    close(raw[:, :cin], D @ Wb, D.abs() @ Wb.abs(), cout, rounded=True)


@pytest.mark.parametrize("npix,hw,P,C0", [(1073 * 2, 1073, 24, 136), (35, 35, 128, 8), (640, 320, 128, 128)])
def test_contraction_gradient(K, npix, hw, P, C0):
    """dB = bf16(gamma (scale dy) T) as an array, and formed where the one-pass kernel reads it."""
    T, dy = rand((npix, P), 1), rand((npix,), 2, dtype=torch.float32)
    gamma, scale = torch.tensor([0.37], device="cuda"), 0.013
    dB = torch.zeros_like(T)
    K["don_grad"](npix, P, ptr(T), ptr(gamma), ptr(dy), scale, ptr(dB), None)
    c = gamma * (torch.tensor(scale, dtype=torch.float32, device="cuda") * dy)
    assert torch.equal(dB, (c[:, None] * T.float()).bfloat16())
    if C0 > 128:
        return
    x, w = rand((npix, C0), 3, relu=True), rand((P, C0), 4, dtype=torch.float32)
    Kp = (P + 31) // 32 * 32
    wT = torch.zeros((C0, Kp), dtype=torch.bfloat16, device="cuda")
    K["pack_t"](ptr(w), P, C0, C0, 1, Kp, ptr(wT), None)
    out = []
    for d, gm, y in ((T, gamma, dy), (dB, None, None)):
        cap = 1 << 20
        part, dx = torch.zeros(cap, device="cuda"), torch.zeros_like(x)
        b = Bwd1x1(hw, npix // hw, P, C0, C0, ptr(d), ptr(x), ptr(wT), Kp, 1, ptr(dx), ptr(gm), ptr(y), scale)
        K["bwd1x1"](C.byref(b), 7, ptr(part), cap, None)
        out.append((part, dx))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("cin8", [8, 16, 24, 32, 40, 64, 72, 128, 144, 264])
@pytest.mark.parametrize("npix", [1, 37, 3219, 70001])
@pytest.mark.parametrize("form", ["plain", "mask", "skip", "noeta"])
def test_input_gradient_and_local_weight_sums(K, cin8, npix, form):
    x, gr = rand((npix, cin8), 1, relu=True), rand((npix, cin8), 2)
    eta = None if form == "noeta" else rand((npix,), 3, dtype=torch.float32).sigmoid().bfloat16()
    dxb, se = gr.clone(), torch.zeros(npix, device="cuda")
    mask = form in ("mask", "noeta")
    bias = torch.zeros((BIAS_PARTS, cin8), device="cuda") if mask and K["can_bias"](cin8) else None
    lo, hi = (8, cin8 - 8) if form == "skip" and cin8 > 16 else (0, 0)
    skip = torch.zeros((npix, hi - lo), dtype=torch.bfloat16, device="cuda") if hi else None
    a = EtaDx(npix, cin8, ptr(x), ptr(eta), ptr(dxb), mask, ptr(skip), lo, hi, None if eta is None else ptr(se),
              ptr(bias))
    K["eta_dx"](C.byref(a), None)
    want = gr.float() * (1.0 if eta is None else eta.float()[:, None])
    if mask:
        want = torch.where(x > 0, want, torch.zeros_like(want))
    want = want.bfloat16()
    if skip is None:
        assert torch.equal(dxb, want)
    else:
        assert torch.equal(dxb[:, :lo], want[:, :lo]) and torch.equal(skip, want[:, lo:hi])
        assert torch.equal(dxb[:, lo:], gr[:, lo:])  # not written
    if eta is not None:
        prod = gr.double() * x.double()
        close(se, prod.sum(1), prod.abs().sum(1), cin8)
    if bias is not None:
        close(bias.double().sum(0), want.double().sum(0), want.double().abs().sum(0), npix // BIAS_PARTS + 257)


@pytest.mark.parametrize("hid,nb,sizes", [(6, 2, [(29, 37), (13, 11), (1, 2)]), (16, 3, [(64, 48)]), (20, 1, [(5, 7)] * 22),
                                          (8, 4, [(300, 500)])])
def test_local_weight_maps_and_parameter_gradients(K, hid, nb, sizes):
    n1 = 6 * hid + 1
    a = PhiArgs(n=len(sizes), nb=nb, hid=hid)
    lv_off, off = 0, 0
    for k, (H, W) in enumerate(sizes):
        a.layer[k] = PhiLayer(H, W, lv_off, k * n1, off, 0, 0)
        lv_off += 3 * (H + W)
        off += H * W * nb
    lv = rand((nb, lv_off), 1, dtype=torch.float32).abs() + 0.5
    params = 0.5 * rand((len(sizes), n1), 2, dtype=torch.float32)
    eta = torch.zeros(off, dtype=torch.bfloat16, device="cuda")
    se = 0.5 + rand((off,), 3, dtype=torch.float32).sigmoid()
    parts = sum(min(PHI_PARTS, (H * W * nb + 255) // 256) for H, W in sizes)
    part, grad = torch.zeros((parts, n1), device="cuda"), torch.zeros((len(sizes), n1), device="cuda")
    a.lv, a.lv_stride, a.params, a.eta, a.se, a.part = ptr(lv), lv_off, ptr(params), ptr(eta), ptr(se), ptr(part)
    K["eta_nodes"](a, None)
    t = RowTable()
    K["phi_grad"](a, ptr(grad), C.byref(t), None)
    assert t.n == len(sizes)
    K["rows"](C.byref(t), None)
    for k, (H, W) in enumerate(sizes):
        y = a.layer[k]
        v = lv[:, y.lv_off:y.lv_off + 3 * (H + W)].double()
        xs = [v[:, q * W:(q + 1) * W][:, None, :].expand(nb, H, W) for q in (0, 1)]
        ys = [v[:, 3 * W + q * H:3 * W + (q + 1) * H][:, :, None].expand(nb, H, W) for q in (0, 1)]
        d = torch.stack(xs + ys, -1).reshape(-1, 4)
        W1, b1, W2, b2 = torch.split(params[k].double(), [4 * hid, hid, hid, 1])
        h = torch.tanh(d @ W1.view(hid, 4).T + b1)
        phi = h @ W2 + b2
        e = torch.exp(-phi * phi)
        s = slice(y.eta_off, y.eta_off + H * W * nb)
        assert float((eta[s].double() - e).abs().max()) <= 2.0 ** -9 + 1e-4
        dphi = se[s].double() * (-2 * phi * e)
        dz = dphi[:, None] * W2 * (1 - h * h)
        got = torch.split(grad[k].double(), [4 * hid, hid, hid, 1])
        for u, terms in ((got[0], (dz[:, :, None] * d[:, None, :]).reshape(-1, 4 * hid)), (got[1], dz),
                         (got[2], dphi[:, None] * h), (got[3], dphi[:, None])):
            assert bool(((u - terms.sum(0)).abs() <= 1e-4 * terms.abs().sum(0)).all())
