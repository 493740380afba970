"""Parity of the HIP path (through the C ABI) with the fp64 CPU oracle, on a real MI355X.

Tolerances (stated target of the build):
  bf16 O : max |err| <= 2e-2 and mean |err| <= 2e-3 for unit-variance inputs.  The gate-extreme
           workload draws Q, K, V with standard deviation 3 (|V| up to ~15, |O| up to ~12), where the
           spacing of bf16 alone exceeds 2e-2; there the bars follow from the arithmetic of a
           bf16 pipeline: probabilities enter the PV product rounded to bf16 (unit roundoff 2^-8)
           and O is stored in bf16, so |err| <= 2^-8 (sum_i P_ti |V_ix| + |O_tx|) elementwise (plus
           5% and 1e-3 for the fp32 steps), and the mean bar scales with the value scale, 3 * 2e-3.
  bf16 L : the row sum is taken in fp32 over the unrounded probabilities, so L is an fp32
           quantity: |err| <= 1e-4 + 1e-5 |L| + 2^-21 * span, where span is the largest gate
           difference that enters any logit, max_t (c_t - c_{max(0, t-w+1)}): c is an fp32 input,
           and any fp32 evaluation of c_i - c_t plus the score rounds a few times at relative
           2^-24 of a number that large (2^-21 = eight such roundings).
  fp32   : ||err||_inf / ||ref||_inf <= 1e-5.
  grads  : relative L2 error <= 1e-2 per tensor (bf16), <= 1e-5 (fp32), against the gradient (the
           oracle on its own fp64 output), and the same bar against Alg. 3 evaluated by the oracle
           on the very O the kernels were given.  The two references differ by the effect of the
           storage rounding of O on D = rowsum(dO * O): -P_ti dD_t in every dS_ti with
           |dD_t| <= 2^-9 sum_x |dO_tx O_tx|.  Over many rows that averages out (it is a few 1e-3
           of the tensor norm at the workload sizes); when a tensor rests on one or two dS entries
           (N of a few tokens) it does not, so for the listed tiny sequences the bar against the
           gradient is 1e-2 plus the CPU-computed relative distance between the two references.
           Beside the tensor norm every row is checked: ||err_t|| <= 3e-2 (||ref_t|| + rms_t ||ref_t||),
           which a single wrong row cannot pass.  A gradient that is identically zero (one key per
           row) is bounded by the fp32 rounding of the two dot products whose difference it is.
The forward entry point is compared with the oracle on the same fp32 prefix c (the oracle's
prefix rounded to fp32); the prefix entry point is compared separately; one chained test runs
alpha -> c -> O entirely on the GPU against the oracle's definition from alpha.
"""
import re

import numpy as np
import pytest
import torch

import gfwa_inputs as gi

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def g():
    import paper_2512_07782_amd as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.load_library()
    return mod


def dev(x: np.ndarray, dtype: str) -> torch.Tensor:
    t = torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def host(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def rel_inf(a, ref):
    return np.abs(a - ref).max() / max(np.abs(ref).max(), 1e-30)


def rel_l2(a, ref):
    return np.linalg.norm((a - ref).ravel()) / max(np.linalg.norm(ref.ravel()), 1e-30)


def note(*a):
    print(*a, flush=True)


def window_span(c, w):
    """Largest gate difference that enters any logit: max_t c_t - c_{max(0, t-w+1)} (c non-decreasing)."""
    c = np.asarray(c, dtype=np.float64)
    N = c.shape[-1]
    r = min(N - 1, int(w) - 1)
    return float((c[..., r:] - c[..., :N - r]).max()) if r > 0 else 0.0


# which workspace the backward calls of run_backward / run_gqa get: the minimum, or the size that selects
# the library's faster variant (dS blocks kept for the dQ pass; bf16, d = 128)
VARIANT = {"fast": False}


@pytest.fixture(params=["min_ws", "fast_ws"])
def ws_variant(request):
    VARIANT["fast"] = request.param == "fast_ws"
    yield request.param
    VARIANT["fast"] = False


def bwd_workspace(g, Q, w):
    B, H, N, d = Q.shape
    size = g.gfwa_backward_fast_workspace_bytes if VARIANT["fast"] else g.gfwa_backward_workspace_bytes
    return torch.empty(size(Q.dtype, B, H, N, d, w), dtype=torch.uint8, device=Q.device)


# ------------------------------------------------------------------------------------------
# gate prefix
# ------------------------------------------------------------------------------------------
@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (2, 3, 37), (1, 2, 4096), (2, 2, 4099), (1, 3, 16384),
                                   (1, 1, 70001)])
def test_gate_prefix(g, oracle, B, H, N):
    note("gate_prefix", B, H, N)
    wl = gi.custom("scan", B, H, N, 64, 8, alpha_mu=0.0, index=7)
    alpha = gi.make_tensor(wl, "alpha")
    c = host(g.gfwa_gate_prefix(dev(alpha, "f32")))
    ref = oracle.gate_prefix(alpha)
    # fp32 result of an fp64-carried scan: a few ulp of the running magnitude
    assert np.abs(c - ref).max() <= 4 * np.finfo(np.float32).eps * ref.max()
    ones = host(g.gfwa_gate_prefix(torch.ones(1, 2, N, device=DEV)))
    np.testing.assert_array_equal(ones[0, 1], np.arange(1, N + 1, dtype=np.float64))


GATE_EPS = 1e-6


@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (2, 3, 37), (1, 2, 4096), (2, 2, 4099), (1, 3, 16384),
                                   (1, 1, 70001)])
def test_gate_activation_prefix(g, oracle, B, H, N):
    note("gate_activation_prefix", B, H, N)
    wl = gi.custom("gact", B, H, N, 64, 8, alpha_mu=-1.0, index=8)
    h, beta = gi.make_gate_inputs(wl)
    c = host(g.gfwa_gate_activation_prefix(dev(h, "f32"), dev(beta, "f32"), GATE_EPS))
    alpha = oracle.gate_activation(h, beta, GATE_EPS)
    ref = oracle.gate_prefix(alpha)
    # each alpha within a few fp32 ulp of itself (exp, log1p, add, divide), summed, plus the scan's own rounding
    assert np.abs(c - ref).max() <= 8 * np.finfo(np.float32).eps * ref.max()
    # the fused call and activation-free scan of the oracle's alpha agree to the same bar
    c2 = host(g.gfwa_gate_prefix(dev(alpha.astype(np.float32), "f32")))
    assert np.abs(c - c2).max() <= 8 * np.finfo(np.float32).eps * ref.max()


@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (2, 3, 37), (1, 2, 4096), (2, 2, 4099), (1, 1, 20487), (1, 2, 1000003),
                                   (4, 16, 16384), (1, 8, 262144)])
@pytest.mark.parametrize("act", [False, True])
def test_gate_prefix_scan_then_propagate(g, oracle, B, H, N, act):
    # the two-launch variant that cuts rows into segments: same definition, same bar as the one-pass scan
    note("gate_prefix_stp", B, H, N, "activation" if act else "plain")
    wl = gi.custom("stp", B, H, N, 64, 8, alpha_mu=-1.0, index=6)
    if act:
        h, beta = gi.make_gate_inputs(wl)
        c = host(g.gfwa_gate_prefix_stp(dev(h, "f32"), dev(beta, "f32"), GATE_EPS))
        ref = oracle.gate_prefix(oracle.gate_activation(h, beta, GATE_EPS))
        one_pass = host(g.gfwa_gate_activation_prefix(dev(h, "f32"), dev(beta, "f32"), GATE_EPS))
    else:
        alpha = gi.make_tensor(wl, "alpha")
        c = host(g.gfwa_gate_prefix_stp(dev(alpha, "f32")))
        ref = oracle.gate_prefix(alpha)
        one_pass = host(g.gfwa_gate_prefix(dev(alpha, "f32")))
    tol = 8 * np.finfo(np.float32).eps * ref.max()
    assert np.abs(c - ref).max() <= tol
    assert np.abs(c - one_pass).max() <= tol


@pytest.mark.parametrize("B,H,N", [
    # two chunks of 4096 of a row take four waves (sixteen with the activation and few rows), longer rows sixteen: both
    # sides, with and without a remainder
    (3, 1, 8191), (1, 2, 8192), (2, 1, 8193), (1, 2, 12288), (1, 1, 12290),
    # rows of one chunk: sixteen waves up to one row per CU, four beyond
    (2, 128, 515), (1, 257, 515), (8, 64, 4096),
    # scan-then-propagate: segments of two and of three chunks
    (2, 150, 49157), (4, 128, 32772)])
@pytest.mark.parametrize("act", [False, True])
def test_gate_scan_wave_counts(g, oracle, B, H, N, act):
    note("gate scan", B, H, N, "activation" if act else "plain")
    wl = gi.custom("gscan", B, H, N, 64, 8, alpha_mu=-1.0, index=17)
    if act:
        h, beta = gi.make_gate_inputs(wl)
        args = (dev(h, "f32"), dev(beta, "f32"), GATE_EPS)
        ref = oracle.gate_prefix(oracle.gate_activation(h, beta, GATE_EPS))
        one_pass = g.gfwa_gate_activation_prefix(*args)
    else:
        alpha = gi.make_tensor(wl, "alpha")
        args = (dev(alpha, "f32"),)
        ref = oracle.gate_prefix(alpha)
        one_pass = g.gfwa_gate_prefix(*args)
    tol = 8 * np.finfo(np.float32).eps * ref.max()  # as above
    for c in (one_pass, g.gfwa_gate_prefix_stp(*args)):
        assert np.abs(host(c) - ref).max() <= tol


def test_gate_activation_elementwise(g, oracle):
    # rows of length 1: c is alpha itself, so the activation is checked element by element, over
    # pre-activations from deeply negative (alpha ~ e^z, where the rounding of 1 + e^z would show) to large
    n = 1 << 16
    z = np.linspace(-80.0, 40.0, n)
    beta = np.exp(0.5 * gi.normal(4242, (n,))).astype(np.float32)
    h = (z / beta).astype(np.float32)
    shape = (256, n // 256, 1)
    a = host(g.gfwa_gate_activation_prefix(dev(h.reshape(shape), "f32"), dev(beta.reshape(shape), "f32"), GATE_EPS))
    ref = oracle.gate_activation(h.reshape(shape), beta.reshape(shape), GATE_EPS)
    # the oracle takes the logarithm of 1 + e^z as Alg. 1 writes it, in fp64: that sum is rounded to
    # 2^-53, so below z ~ -30 the oracle's own value is the less accurate one (it is exactly 0 from -37 on)
    floor = 2.0 ** -52 / (beta.reshape(shape).astype(np.float64) + GATE_EPS)
    far = z.reshape(shape) > -20
    rel = np.abs(a - ref)[far] / ref[far]
    note(f"  alpha worst relative error for z > -20: {rel.max():.3e} ({rel.max() / np.finfo(np.float32).eps:.1f} ulp)")
    # z = beta h is rounded to fp32 on the GPU (relative 2^-24) and d(log alpha)/dz <= 1 for z < 0,
    # so a small alpha ~ e^z inherits |z| half-ulps from its argument on top of the arithmetic's few ulp
    zz = z.reshape(shape)
    assert (np.abs(a - ref) <= np.finfo(np.float32).eps * ref * (8 + np.maximum(-zz, 0)) + floor).all()


def test_gate_activation_extremes(g, oracle):
    # saturated, dead and zero pre-activations, tiny and large amplitudes: no overflow, alpha >= 0
    h = np.array([[[-200.0, -30.0, -1e-3, 0.0, 1e-3, 30.0, 200.0, 3e4] * 5]], dtype=np.float32)
    beta = np.repeat(np.array([1e-3, 0.5, 1.0, 8.0, 100.0], dtype=np.float32), 8).reshape(1, 1, -1)
    c = host(g.gfwa_gate_activation_prefix(dev(h, "f32"), dev(beta, "f32"), GATE_EPS))
    ref = oracle.gate_prefix(oracle.gate_activation(h, beta, GATE_EPS))
    assert np.isfinite(c).all() and (c >= 0).all()
    assert np.abs(c - ref).max() <= 8 * np.finfo(np.float32).eps * ref.max()
    dal = np.ones_like(h)
    dh, dbeta = (host(x) for x in g.gfwa_gate_activation_backward(dev(h, "f32"), dev(beta, "f32"), GATE_EPS,
                                                                  dev(dal, "f32")))
    rh, rb = oracle.gate_activation_backward(h, beta, GATE_EPS, dal)
    assert np.isfinite(dh).all() and np.isfinite(dbeta).all()
    np.testing.assert_allclose(dh, rh, rtol=1e-5, atol=1e-30)
    be = beta.astype(np.float64) + GATE_EPS
    terms = np.abs(h) / be + (np.maximum(beta.astype(np.float64) * h, 0) + 0.7) / be ** 2
    assert (np.abs(dbeta - rb) <= 16 * np.finfo(np.float32).eps * terms + 1e-30).all()


@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (2, 3, 37), (1, 2, 4099), (4, 8, 16384), (1, 1, 4194309)])
def test_gate_activation_backward(g, oracle, B, H, N):
    note("gate_activation_backward", B, H, N)
    wl = gi.custom("gactb", B, H, N, 64, 8, alpha_mu=-1.0, index=9)
    h, beta = gi.make_gate_inputs(wl)
    dal = gi.normal(wl.seed("dO"), h.shape).astype(np.float32)
    dh, dbeta = (host(x) for x in g.gfwa_gate_activation_backward(dev(h, "f32"), dev(beta, "f32"), GATE_EPS,
                                                                  dev(dal, "f32")))
    rh, rb = oracle.gate_activation_backward(h, beta, GATE_EPS, dal)
    np.testing.assert_allclose(dh, rh, rtol=1e-5, atol=1e-30)
    # dbeta is a difference of two terms: a few fp32 ulp of an upper bound of their magnitudes
    be = beta.astype(np.float64) + GATE_EPS
    terms = np.abs(dal) * (np.abs(h) / be + (np.maximum(beta.astype(np.float64) * h, 0) + 0.7) / be ** 2)
    assert (np.abs(dbeta - rb) <= 16 * np.finfo(np.float32).eps * terms + 1e-30).all()
    assert rel_l2(dbeta, rb) <= 1e-6 and rel_l2(dh, rh) <= 1e-6


@pytest.mark.parametrize("B,H,N,d,w", [(1, 2, 300, 128, 64), (2, 2, 1030, 64, 256)])
def test_chain_from_gate_preactivation_bf16(g, oracle, B, H, N, d, w):
    # h, beta -> c (fused) -> forward -> backward -> dalpha -> dh, dbeta, all on the GPU, against the
    # oracle's chain from the same inputs
    note("chain from h, beta", B, H, N, d, w)
    wl = gi.custom("gchain", B, H, N, d, w, "bf16", alpha_mu=-1.0, index=10, backward=True)
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "dO")}
    h, beta = gi.make_gate_inputs(wl)
    alpha = oracle.gate_activation(h, beta, GATE_EPS)
    c_ref = oracle.gate_prefix(alpha)
    O_ref, L_ref = oracle.forward_from_c(ins["Q"], ins["K"], ins["V"], c_ref, wl.w, wl.scale)
    ref = oracle.backward_from_c(ins["Q"], ins["K"], ins["V"], c_ref, ins["dO"], wl.w, wl.scale)
    ref_dh, ref_dbeta = oracle.gate_activation_backward(h, beta, GATE_EPS, ref["dalpha"].reshape(h.shape))
    Qd, Kd, Vd, dOd = (dev(ins[t], "bf16") for t in ("Q", "K", "V", "dO"))
    hd, bd = dev(h, "f32"), dev(beta, "f32")
    cd = g.gfwa_gate_activation_prefix(hd, bd, GATE_EPS)
    Od, Ld = g.gfwa_forward(Qd, Kd, Vd, cd, wl.w, wl.scale)
    dQ, dK, dV, dalpha = g.gfwa_backward(Qd, Kd, Vd, Od, dOd, cd, Ld, wl.w, wl.scale)
    dh, dbeta = g.gfwa_gate_activation_backward(hd, bd, GATE_EPS, dalpha)
    torch.cuda.synchronize()
    LAST["c_span"] = window_span(c_ref, wl.w)
    check_bf16_forward(host(Od), host(Ld), O_ref, L_ref, tag="chain")
    for name, got, want in (("dh", dh, ref_dh), ("dbeta", dbeta, ref_dbeta)):
        r = rel_l2(host(got), want)
        note(f"  chain {name} rel-L2 {r:.3e}")
        assert r <= 1e-2, (name, r)


# ------------------------------------------------------------------------------------------
# forward
# ------------------------------------------------------------------------------------------
LAST = {"c_span": 0.0}  # window_span of the last run


def run_forward(g, oracle, wl, heads=None, want_bound=False):
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha")}
    c64 = oracle.gate_prefix(ins["alpha"])
    c32 = c64.astype(np.float32)
    LAST["c_span"] = window_span(c64, wl.w)
    O, L = g.gfwa_forward(dev(ins["Q"], wl.dtype), dev(ins["K"], wl.dtype), dev(ins["V"], wl.dtype),
                          dev(c32, "f32"), wl.w, wl.scale)
    torch.cuda.synchronize()
    O, L = host(O), host(L)
    if heads is None:
        heads = list(range(wl.B * wl.H))
    sel = lambda x, tr: oracle.select_heads(x, heads, tr)
    if want_bound:
        Vs = sel(ins["V"], 2).astype(np.float64)
        O_ref, L_ref, P = oracle.forward_from_c(sel(ins["Q"], 2), sel(ins["K"], 2), Vs, sel(c32, 1),
                                                wl.w, wl.scale, return_P=True)
        pv = np.stack([band_matmul(P[i], np.abs(Vs[i]), wl.w) for i in range(len(heads))])
        bound = 1.05 * 2.0 ** -8 * (pv + np.abs(O_ref)) + 1e-3
        return sel(O, 2), sel(L, 1), O_ref, L_ref, bound
    O_ref, L_ref = oracle.forward_from_c(sel(ins["Q"], 2), sel(ins["K"], 2), sel(ins["V"], 2),
                                         sel(c32, 1), wl.w, wl.scale)
    return sel(O, 2), sel(L, 1), O_ref, L_ref


def band_matmul(P_band, M, w, block=512):
    """(P @ M) for P given as its band [N, min(w,N)] (row t holds keys max(0,t-w+1)..t)."""
    N = P_band.shape[0]
    out = np.zeros((N, M.shape[1]))
    for a in range(0, N, block):
        b = min(N, a + block)
        k0 = max(0, a - w + 1)
        blk = np.zeros((b - a, b - k0))
        for t in range(a, b):
            lo = max(0, t - w + 1)
            blk[t - a, lo - k0:t + 1 - k0] = P_band[t, :t - lo + 1]
        out[a:b] = blk @ M[k0:b]
    return out


def check_bf16_forward(O, L, O_ref, L_ref, bound=None, value_scale=1.0, tag=""):
    assert np.isfinite(O).all() and np.isfinite(L).all()
    err = np.abs(O - O_ref)
    lerr = np.abs(L - L_ref)
    note(f"  {tag} O max {err.max():.3e} mean {err.mean():.3e}  L max {lerr.max():.3e}")
    if bound is not None:
        note(f"  {tag} worst err/bound {np.max(err / bound):.3f}")
        assert (err <= bound).all()
    else:
        assert err.max() <= 2e-2
    assert err.mean() <= 2e-3 * value_scale
    # L comes from an fp32 row sum of unrounded probabilities; its error is that of the fp32
    # exponent arithmetic on gate differences as large as the span of c over a window
    assert (lerr <= 1e-4 + 1e-5 * np.abs(L_ref) + 2.0 ** -21 * LAST["c_span"]).all()


SMALL_BF16 = [
    # B, H, N, d, w
    (1, 1, 1, 64, 1), (1, 2, 37, 64, 5), (2, 1, 129, 128, 1), (1, 2, 300, 128, 64),
    (1, 1, 257, 64, 100), (1, 2, 1000, 128, 333), (1, 1, 640, 128, 4000), (2, 2, 515, 64, 512),
    (1, 1, 1536, 128, 1024), (1, 1, 700, 128, 32), (1, 1, 450, 64, 33),
]


@pytest.mark.parametrize("B,H,N,d,w", SMALL_BF16)
def test_forward_bf16_small(g, oracle, B, H, N, d, w):
    note("forward bf16 small", B, H, N, d, w)
    wl = gi.custom("small", B, H, N, d, w, "bf16", alpha_mu=-1.0, index=8)
    check_bf16_forward(*run_forward(g, oracle, wl), tag="small")


def test_forward_tiny_f32(g, oracle):
    wl = gi.WORKLOADS["tiny_fwd_f32"]
    note("forward f32", wl)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl)
    note(f"  rel_inf O {rel_inf(O, O_ref):.3e} L {rel_inf(L, L_ref):.3e}")
    assert rel_inf(O, O_ref) <= 1e-5
    assert rel_inf(L, L_ref) <= 1e-5


# (the first three are served by the one-wave-per-row kernels, the next three by the fp32 matrix-core kernels; of windows of one
# key and just over a block many rows, and long ones, go to the matrix cores too)
@pytest.mark.parametrize("B,H,N,d,w", [(1, 2, 77, 64, 9), (2, 1, 130, 128, 500), (1, 1, 65, 128, 1),
                                       (2, 3, 1500, 128, 700), (1, 4, 2100, 64, 300), (1, 4, 1237, 128, 5000),
                                       (4, 16, 5001, 64, 1), (1, 8, 2049, 128, 33)])
def test_forward_f32_ragged(g, oracle, B, H, N, d, w):
    note("forward f32 ragged", B, H, N, d, w)
    wl = gi.custom("f32r", B, H, N, d, w, "f32", alpha_mu=0.0, index=9)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl)
    assert rel_inf(O, O_ref) <= 1e-5 and rel_inf(L, L_ref) <= 1e-5


def test_tiny_f32_chained_from_alpha(g, oracle):
    """alpha -> c -> O all on the GPU against the definition from alpha (fp64 prefix)."""
    wl = gi.WORKLOADS["tiny_fwd_f32"]
    ins = gi.make_inputs(wl)
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    O, L = g.gfwa_forward(dev(ins["Q"], "f32"), dev(ins["K"], "f32"), dev(ins["V"], "f32"), c, wl.w, wl.scale)
    O_ref, L_ref, _ = oracle.forward(ins["Q"], ins["K"], ins["V"], ins["alpha"], wl.w, wl.scale)
    r = rel_inf(host(O), O_ref)
    note(f"  chained tiny f32 rel_inf O {r:.3e}")
    # the fp32 prefix itself carries up to one ulp(c) ~ 1.5e-5 of absolute logit error at c ~ 200
    assert r <= 3e-5


FULL = [("lm_fwd", [0, 21, 42, 63], False), ("long_fwd", [0, 13, 31], False),
        ("gate_extreme_fwd", [0, 3, 5, 12, 15], True)]


@pytest.mark.parametrize("name,heads,mag", FULL)
def test_forward_bf16_full_size(g, oracle, name, heads, mag):
    """BASELINE-size workloads in the launch configuration the benchmark times; the oracle
    checks every row of a sample of (b,h) heads."""
    wl = gi.WORKLOADS[name]
    note("forward full size", wl)
    if mag:
        O, L, O_ref, L_ref, bound = run_forward(g, oracle, wl, heads=heads, want_bound=True)
        check_bf16_forward(O, L, O_ref, L_ref, bound=bound, value_scale=wl.qkv_std, tag=name)
    else:
        O, L, O_ref, L_ref = run_forward(g, oracle, wl, heads=heads)
        check_bf16_forward(O, L, O_ref, L_ref, tag=name)


def test_zero_gate_heads_match_plain_swa(g, oracle):
    """alpha = 0 heads of the gate-extreme workload: the prefix is constant and the bias vanishes."""
    wl = gi.custom("swa", 1, 2, 600, 128, 128, "bf16", alpha_mu=1.0, zero_gate_heads=(0,), index=10)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl)
    check_bf16_forward(O, L, O_ref, L_ref, tag="swa")
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V")}
    O0, _ = oracle.forward_from_c(ins["Q"][0, 0], ins["K"][0, 0], ins["V"][0, 0], np.zeros(wl.N), wl.w, wl.scale)
    assert np.abs(O[0] - O0).max() <= 2e-2


# ------------------------------------------------------------------------------------------
# backward
# ------------------------------------------------------------------------------------------
def run_backward(g, oracle, wl, heads=None, chained=False):
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha", "dO")}
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    if heads is None:
        heads = list(range(wl.B * wl.H))
    sel = lambda x, tr: oracle.select_heads(x, heads, tr)
    ref = oracle.backward_from_c(sel(ins["Q"], 2), sel(ins["K"], 2), sel(ins["V"], 2), sel(c32, 1),
                                 sel(ins["dO"], 2), wl.w, wl.scale)
    Qd, Kd, Vd, dOd = (dev(ins[t], wl.dtype) for t in ("Q", "K", "V", "dO"))
    cd = dev(c32, "f32")
    if chained or len(heads) < wl.B * wl.H:
        Od, Ld = g.gfwa_forward(Qd, Kd, Vd, cd, wl.w, wl.scale)
    else:
        O_ref, L_ref = oracle.forward_from_c(ins["Q"], ins["K"], ins["V"], c32, wl.w, wl.scale)
        Od = dev(O_ref.astype(np.float32), "f32")
        Od = Od.to(torch.bfloat16) if wl.dtype == "bf16" else Od     # torch rounds to nearest even
        Ld = dev(L_ref.astype(np.float32), "f32")
    dQ, dK, dV, dalpha = g.gfwa_backward(Qd, Kd, Vd, Od, dOd, cd, Ld, wl.w, wl.scale,
                                         workspace=bwd_workspace(g, Qd, wl.w))
    torch.cuda.synchronize()
    got = {"dQ": sel(host(dQ), 2), "dK": sel(host(dK), 2), "dV": sel(host(dV), 2), "dalpha": sel(host(dalpha), 1)}
    # Alg. 3 on the stored output the kernels were given (with its dS band when the telescoped form of
    # d(alpha), O(N w^2) on the CPU, is affordable), and the bound of an identically-zero gradient
    direct = wl.N * min(wl.w, wl.N) ** 2 * len(heads) <= 3e8
    ref["saved"] = oracle.backward_from_c(sel(ins["Q"], 2), sel(ins["K"], 2), sel(ins["V"], 2), sel(c32, 1),
                                          sel(ins["dO"], 2), wl.w, wl.scale, O_saved=sel(host(Od), 2),
                                          return_dS=direct)
    if direct:
        ref["saved"]["dalpha_direct"] = oracle.dalpha_direct(ref["saved"]["dS"], wl.w)
    ref["zero"] = zero_gradient_bounds(sel(ins["dO"], 2), sel(ins["V"], 2), sel(ins["Q"], 2), sel(ins["K"], 2),
                                       wl.scale, 1)
    return got, ref


def zero_gradient_bounds(dO, V, Q, K, scale, G):
    """Bounds for gradients that are identically zero, which happens exactly when every row has one key
    (w = 1 or N = 1): P_tt = 1, O_t = v_t, and dS_tt = <dO_t, v_t> - D_t is the difference of two fp32
    dot products of the same d terms added in different orders.  Each is within d/2 roundings of 2^-24
    relative to sum_x |dO_tx v_tx| in the worst case and about sqrt(d) of them typically; the bar takes
    4 * 2^-24 * max_t sum_x |dO_tx v_tx| for |dS_tt| (16 roundings of the full absolute sum).  Then
    |dQ_t| <= scale |dS| max|k|, |dK_i| <= G scale |dS| max|q| (G query heads add up), and every
    d(alpha)_q is a sum of at most 2 N such values."""
    dO, V = np.asarray(dO, dtype=np.float64), np.asarray(V, dtype=np.float64)
    e_dS = 4 * 2.0 ** -24 * np.abs(dO * V).sum(axis=-1).max()
    N = dO.shape[-2]
    return {"dQ": scale * e_dS * np.abs(K).max(), "dK": G * scale * e_dS * np.abs(Q).max(), "dV": 0.0,
            "dalpha": 2 * N * e_dS}


def row_check(got, ref, k, tag):
    """Every row (last axis; 32-element blocks of d(alpha)): ||err_t|| <= 3e-2 (||ref_t|| + rms_t ||ref_t||)."""
    a, b = np.asarray(got), np.asarray(ref)
    if k == "dalpha":
        n = a.shape[-1] // 32 * 32
        if n == 0:
            return
        a, b = a[..., :n].reshape(a.shape[:-1] + (n // 32, 32)), b[..., :n].reshape(b.shape[:-1] + (n // 32, 32))
    err = np.linalg.norm(a - b, axis=-1)
    nr = np.linalg.norm(b, axis=-1)
    rms = np.sqrt((nr ** 2).mean())
    worst = (err / (nr + rms + 1e-300)).max()
    note(f"  {tag} {k} worst row err/(|ref_t| + rms) {worst:.3e}")
    assert worst <= 3e-2, (k, worst)


def check_grads(got, ref, tol, tag="", tiny=False):
    saved = ref.get("saved")
    for k in ("dQ", "dK", "dV", "dalpha"):
        assert np.isfinite(got[k]).all(), k
        nr = np.linalg.norm(ref[k].ravel())
        if nr < 1e-12:                      # one key per row: the gradient is identically zero
            bound = ref["zero"][k]
            note(f"  {tag} {k} zero gradient: max |g| {np.abs(got[k]).max():.3e}, bound {bound:.3e}")
            assert np.abs(got[k]).max() <= bound, k
            continue
        r = rel_l2(got[k], ref[k])
        if saved is None:
            note(f"  {tag} {k} rel-L2 {r:.3e}")
            assert r <= tol, (k, r)
            continue
        rs = rel_l2(got[k], saved[k])
        storage = rel_l2(saved[k], ref[k])   # effect of the storage rounding of O alone, computed on the CPU
        note(f"  {tag} {k} rel-L2 {r:.3e}; against Alg. 3 on the stored O {rs:.3e} (the two references differ by {storage:.3e})")
        assert rs <= tol, (k, rs)
        assert r <= tol + (storage if tiny else 0.0), (k, r)
        if tol >= 1e-3:   # bf16 storage: no single row may be off
            row_check(got[k], saved[k], k, tag)
    # properties the design rests on, on the GPU's own output
    da, ref_da = got["dalpha"], (saved or ref)["dalpha"]
    scale_da = np.abs(ref_da).max()
    if scale_da > 0:
        # alpha_0 shifts every c equally and so changes nothing: d(alpha)[..., 0] = sum_p dc_p = 0 exactly, since
        # every dS_ti enters once as a column and once as a row term.  On the GPU the two terms come from two
        # kernels that each form exp(S_ti - L_t) in fp32 from summands of the size of |L_t| plus the gate span
        # (tens to hundreds), so their values of one dS_ti differ by about 1e-5 relative, with random sign; over
        # the N w' in-window pairs that is a random walk of about 1e-5 sqrt(N w') rms|dS|, a few 1e-4 absolute at
        # every size here (largest seen: 8.6e-5 of max |dalpha| at N = 65536; 2e-7 with fp32 storage, where the
        # kernels share one formula).  Bar: 5e-4 of max |dalpha|, a twentieth of what the other entries may err.
        first = np.abs(da[..., 0]).max()
        note(f"  {tag} |dalpha[..., 0]| {first:.3e} of max |dalpha| {scale_da:.3e}")
        assert first <= (5e-4 if tol >= 1e-3 else 1e-5) * scale_da
    if saved is not None and "dalpha_direct" in saved and np.linalg.norm(saved["dalpha_direct"]) > 1e-12:
        # d(alpha)_q = - sum of dS_ti over in-window pairs with i < q <= t (Sec. 3.3: the gate gradient is the
        # reverse scan of column minus row sums), from the oracle's dS without going through dc
        rd = rel_l2(da, saved["dalpha_direct"])
        note(f"  {tag} dalpha against the telescoped form {rd:.3e}")
        assert rd <= tol


@pytest.mark.parametrize("B,H,N,d,w", [(1, 2, 77, 64, 9), (2, 1, 130, 128, 500), (1, 1, 65, 128, 1),
                                       (1, 1, 256, 64, 64),
                                       # large enough for the fp32 matrix-core kernels
                                       (1, 4, 1100, 128, 400), (2, 2, 1000, 64, 300), (1, 3, 1237, 128, 3000),
                                       (1, 8, 2049, 64, 33), (4, 16, 5001, 128, 1)])
def test_backward_f32(g, oracle, B, H, N, d, w):
    note("backward f32", B, H, N, d, w)
    wl = gi.custom("bf32", B, H, N, d, w, "f32", alpha_mu=-1.0, index=11, backward=True)
    got, ref = run_backward(g, oracle, wl)
    check_grads(got, ref, 1e-5, "f32")


SMALL_BWD = [(1, 1, 1, 64, 1), (1, 2, 37, 64, 5), (2, 1, 129, 128, 1), (1, 2, 300, 128, 64),
             (1, 1, 257, 64, 100), (1, 2, 1000, 128, 333), (1, 1, 640, 128, 4000), (2, 2, 515, 64, 512),
             (1, 1, 1536, 128, 1024), (1, 1, 450, 64, 33)]
# sequences of a few tokens: a gradient tensor rests on a handful of dS entries (N = 2: on one), so the
# storage rounding of O shows undamped in the distance to the gradient (see the module docstring); the three
# leading shapes are the ones a wider seeded sweep found above 1e-2 against the gradient
TINY_BWD = [(1, 1, 2, 128, 34, 0.5, 29), (1, 1, 2, 64, 2, 0.5, 31), (1, 2, 2, 128, 2, -1.0, 12), (1, 1, 3, 64, 3, -1.0, 12),
            (2, 1, 4, 128, 2, -1.0, 12), (1, 1, 5, 64, 100, -1.0, 12), (1, 2, 8, 128, 3, -1.0, 12),
            (1, 1, 16, 64, 16, -1.0, 12), (1, 1, 31, 128, 7, -1.0, 12), (1, 2, 33, 128, 32, -1.0, 12),
            (1, 1, 33, 64, 33, 0.5, 30),
            (1, 1, 6, 64, 322, 0.5, 28)]   # a later sweep's only case above 1e-2 against the exact gradient (dalpha 1.06e-2, 1.2e-6 against Alg. 3 on the stored O)


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("B,H,N,d,w", SMALL_BWD)
def test_backward_bf16_small(g, oracle, ws_variant, B, H, N, d, w, chained):
    note("backward bf16 small", ws_variant, B, H, N, d, w, "chained", chained)
    wl = gi.custom("bsmall", B, H, N, d, w, "bf16", alpha_mu=-1.0, index=12, backward=True)
    got, ref = run_backward(g, oracle, wl, chained=chained)
    check_grads(got, ref, 1e-2, "bf16")


@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("B,H,N,d,w,mu,index", TINY_BWD)
def test_backward_bf16_tiny_sequences(g, oracle, ws_variant, B, H, N, d, w, mu, index, chained):
    note("backward bf16 tiny", ws_variant, B, H, N, d, w, mu, index, "chained", chained)
    wl = gi.custom("fz", B, H, N, d, w, "bf16", alpha_mu=mu, index=index, backward=True)
    got, ref = run_backward(g, oracle, wl, chained=chained)
    check_grads(got, ref, 1e-2, "tiny", tiny=True)


def test_backward_bf16_tiny_grouped(g, oracle, ws_variant):
    # the grouped-query shape of the same sweep: two tokens, three query heads on one key/value head
    wl = gi.custom("fz", 2, 3, 2, 128, 9, "bf16", alpha_mu=-1.0, index=30, backward=True, kv_heads=1)
    note("backward bf16 tiny grouped", ws_variant, wl)
    got, ref = run_gqa(g, oracle, wl)
    check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag="tiny gqa")
    check_grads(got, ref, 1e-2, "tiny gqa", tiny=True)


@pytest.mark.parametrize("name,heads", [("train_bwd", [0, 37, 63]), ("long_bwd", [5, 31])])
def test_backward_bf16_full_size(g, oracle, ws_variant, name, heads):
    wl = gi.WORKLOADS[name]
    note("backward full size", ws_variant, wl)
    got, ref = run_backward(g, oracle, wl, heads=heads)
    check_grads(got, ref, 1e-2, name)


MID = [  # several 256-query workgroups, many key tiles, ragged ends; sampled heads
    # B, H, N, d, w, heads
    (1, 4, 4099, 64, 512, [0, 3]), (1, 2, 5003, 128, 3000, [1]), (2, 2, 2050, 128, 2050, [0, 3]),
    (1, 2, 3001, 64, 7000, [1]),
]


@pytest.mark.parametrize("B,H,N,d,w,heads", MID)
def test_forward_backward_bf16_mid_size(g, oracle, ws_variant, B, H, N, d, w, heads):
    """Sizes between the small exhaustive cases and the benchmark workloads: multi-tile both ways,
    N not a multiple of any tile, windows below, at and above N."""
    note("mid size", ws_variant, B, H, N, d, w)
    wl = gi.custom("mid", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=14, backward=True)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl, heads=heads)
    check_bf16_forward(O, L, O_ref, L_ref, tag="mid")
    got, ref = run_backward(g, oracle, wl, heads=heads)
    check_grads(got, ref, 1e-2, "mid")


@pytest.mark.parametrize("B,H,N,d,w,heads", [
    # more query tiles than resident workgroups (2 per CU at d = 128, 3 at d = 64, 256 CUs), not a multiple of them: the
    # forward deals the tiles of its last round out per XCD; heads from the full first round and from that last one
    (1, 20, 4099, 128, 300, [0, 15, 16, 19]), (1, 25, 4099, 64, 300, [0, 22, 23, 24]), (3, 11, 2100, 128, 77, [0, 30, 31, 32]),
])
def test_forward_bf16_partial_last_round(g, oracle, B, H, N, d, w, heads):
    note("partial last round", B, H, N, d, w)
    wl = gi.custom("plr", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=15)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl, heads=heads)
    check_bf16_forward(O, L, O_ref, L_ref, tag="partial last round")


@pytest.mark.parametrize("H,N,d,w", [(40, 2049, 128, 16), (60, 2049, 64, 16), (36, 2070, 128, 1)])
def test_forward_bf16_after_rows_past_the_end(g, oracle, H, N, d, w):
    # the last query tile of a head has waves without a query, whose made-up rows see no key at all (N + 32 .. with short
    # windows): what they leave in LDS must not reach the tile of another head that the same workgroup takes next
    note("after rows past the end", H, N, d, w)
    wl = gi.custom("past", 1, H, N, d, w, "bf16", alpha_mu=-1.5, index=27)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl)
    check_bf16_forward(O, L, O_ref, L_ref, tag="past the end")


@pytest.mark.parametrize("B,H,N,d,w,heads", [
    # few query tiles: 32 queries per workgroup (last block of one row, window inside a block, window past the sequence)
    (1, 3, 97, 128, 40, [0, 2]), (2, 2, 65, 64, 5000, [0, 3]), (1, 1, 1000, 128, 999, [0]),
    # 64 queries per workgroup
    (1, 32, 701, 128, 1024, [0, 31]), (3, 16, 450, 64, 200, [0, 47]),
    # 128 queries per workgroup: long bands
    (1, 2, 1801, 128, 1600, [0, 1]), (1, 12, 1930, 64, 1901, [0, 11]),
])
def test_forward_bf16_split_band(g, oracle, B, H, N, d, w, heads):
    note("split band", B, H, N, d, w)
    wl = gi.custom("split", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=15)
    O, L, O_ref, L_ref = run_forward(g, oracle, wl, heads=heads)
    check_bf16_forward(O, L, O_ref, L_ref, tag="split band")


def kernels(call):
    """Names (with template arguments) of the library's kernels that `call` runs, as the profiler sees them."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    found = (re.search(r"gfwa::(\w+(<[^>]*>)?)", e.key) for e in prof.key_averages())
    return {m.group(1) for m in found if m}


MANY64, MANY128, TWO_BLOCKS, SPLIT = "fwd_bf16_kernel<64>", "fwd_bf16_kernel<128>", "fwd_two_blocks_bf16_kernel", "fwd_split_bf16_kernel"


@pytest.mark.parametrize("B,H,N,d,w,heads,kernel", [
    # enough work per CU for the kernel of many workgroups on a CU: sequences of one key tile (64 keys at d = 64, 32 at
    # d = 128), one row on either side of a key and of a query tile, windows of one key, inside a tile, at its edge and past the
    # sequence; head counts that divide by the XCDs and that do not; shorter than a key tile, which the split kernel takes;
    # last: a launch that puts two workgroups on a CU instead of three
    (66, 8, 64, 64, 64, [0, 527], MANY64), (5, 81, 65, 64, 9, [0, 404], MANY64), (66, 8, 127, 64, 1, [0, 200], MANY64),
    (5, 81, 128, 64, 5000, [0, 404], MANY64), (24, 16, 129, 64, 64, [0, 383], MANY64), (7, 31, 193, 64, 65, [0, 216], MANY64),
    (10, 20, 321, 64, 128, [0, 199], MANY64), (128, 4, 63, 64, 64, [0, 511], SPLIT),
    # (the two sides of the order of tiles for heads that do not divide by the XCDs, windows of 0.4 N)
    (5, 43, 321, 64, 129, [0, 1, 43, 214], MANY64), (5, 43, 321, 64, 128, [0, 1, 43, 214], MANY64),
    (48, 8, 32, 128, 32, [0, 383], MANY128), (5, 71, 33, 128, 9, [0, 354], MANY128), (48, 8, 127, 128, 1, [0, 200], MANY128),
    (5, 71, 128, 128, 5000, [0, 354], MANY128), (24, 16, 161, 128, 32, [0, 383], MANY128), (7, 31, 193, 128, 65, [0, 216], MANY128),
    (128, 4, 31, 128, 64, [0, 511], SPLIT), (8, 31, 450, 128, 128, [0, 247], MANY128),
    # few workgroups on a CU, d = 128 in steps of 64 keys: sequences of two key tiles, the last tile of one row, of all but one
    # and of three, windows at a tile's edge, one past it and past the sequence; one, two and four workgroups on a CU
    (30, 8, 128, 128, 128, [0, 239], TWO_BLOCKS), (32, 8, 128, 128, 5000, [0, 255], TWO_BLOCKS), (1, 14, 2049, 128, 129, [0, 13], TWO_BLOCKS),
    (1, 15, 2047, 128, 192, [0, 14], TWO_BLOCKS), (2, 58, 450, 128, 300, [0, 115], TWO_BLOCKS), (7, 16, 449, 128, 257, [0, 111], TWO_BLOCKS),
    (1, 14, 7817, 128, 300, [0, 13], TWO_BLOCKS),
    # the lines between the kernels.  d = 64: up to two tiles a CU for heads that divide by the XCDs, one and a half for others; wide
    # split tiles.  d = 128: a tile a CU of short bands, long sequences only; two a CU by length, N > 192; heads in ranges, bands of more
    # than 1024; nearly causal bands; few tiles of another round, in ranges and by length
    (1, 16, 1667, 64, 1048, [0, 15], SPLIT), (4, 13, 939, 64, 311, [0, 51], MANY64), (3, 9, 1855, 64, 1855, [26], SPLIT),
    (1, 7, 4097, 128, 65, [0, 6], TWO_BLOCKS), (1, 7, 4095, 128, 65, [0, 6], SPLIT), (19, 8, 226, 128, 226, [0, 151], TWO_BLOCKS),
    (19, 8, 192, 128, 192, [0, 151], SPLIT), (5, 4, 1921, 128, 1282, [0, 19], SPLIT),
    (7, 9, 1100, 128, 825, [0, 62], TWO_BLOCKS), (7, 9, 1100, 128, 824, [0, 62], MANY128),
    (1, 11, 3193, 128, 492, [0, 10], TWO_BLOCKS), (1, 11, 3193, 128, 191, [0, 10], MANY128),
])
def test_forward_bf16_many_workgroups(g, oracle, B, H, N, d, w, heads, kernel):
    note("many workgroups", B, H, N, d, w)
    wl = gi.custom("many", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=15)
    got = []
    names = kernels(lambda: got.extend(run_forward(g, oracle, wl, heads=heads)))
    assert any(n.startswith(kernel) for n in names), names
    O, L, O_ref, L_ref = got
    check_bf16_forward(O, L, O_ref, L_ref, tag="many workgroups")


@pytest.mark.parametrize("B,H,N,d,w,heads", [
    # the orders of the tiles: heads that do not divide by the XCDs and are one tile each, two tiles, bands just shorter than a tenth of
    # the sequence and a tenth, d = 64 and 128; heads that divide, with a short band; the last tile of one row
    (5, 60, 97, 128, 40, [0, 299]), (3, 100, 65, 64, 50, [0, 299]), (1, 9, 2049, 64, 204, [0, 8]), (1, 9, 2049, 64, 205, [0, 8]),
    (1, 25, 1537, 128, 153, [0, 1, 24]), (1, 25, 1537, 128, 154, [0, 24]), (2, 32, 1025, 128, 70, [0, 1, 63]), (3, 7, 1025, 64, 600, [0, 20]),
])
def test_forward_f32_order_of_tiles(g, oracle, B, H, N, d, w, heads):
    note("f32 order of tiles", B, H, N, d, w)
    wl = gi.custom("order", B, H, N, d, w, "f32", alpha_mu=-1.5, index=29)
    got = []
    names = kernels(lambda: got.extend(run_forward(g, oracle, wl, heads=heads)))
    assert any(n.startswith("fwd_f32_mfma_kernel") for n in names), names
    O, L, O_ref, L_ref = got
    assert rel_inf(O, O_ref) <= 1e-5
    assert (np.abs(L - L_ref) <= 1e-5 * np.abs(L_ref).max() + 1e-5).all()


# ------------------------------------------------------------------------------------------
# grouped-query layout
# ------------------------------------------------------------------------------------------
def run_gqa(g, oracle, wl, groups=None):
    """Forward + backward of a grouped-query workload on the GPU and in the oracle.  `groups`: flat
    key/value head indices (b * Hkv + kv) whose results are compared (all when None)."""
    G = wl.H // wl.Hkv
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha", "dO")}
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    Qd, Kd, Vd, dOd = (dev(ins[t], wl.dtype) for t in ("Q", "K", "V", "dO"))
    cd = dev(c32, "f32")
    Od, Ld = g.gfwa_forward_gqa(Qd, Kd, Vd, cd, wl.w, wl.scale)
    dQ, dK, dV, dalpha = g.gfwa_backward_gqa(Qd, Kd, Vd, Od, dOd, cd, Ld, wl.w, wl.scale,
                                             workspace=bwd_workspace(g, Qd, wl.w))
    torch.cuda.synchronize()
    assert dK.shape == Kd.shape and dV.shape == Vd.shape
    if groups is None:
        groups = list(range(wl.B * wl.Hkv))
    qheads = [(kv // wl.Hkv) * wl.H + (kv % wl.Hkv) * G + j for kv in groups for j in range(G)]
    # the selected groups as a batch of their own: [len(groups), G, N, d] queries on [len(groups), 1, N, d] keys
    shp_q = (len(groups), G, wl.N, wl.d)
    shp_k = (len(groups), 1, wl.N, wl.d)
    sq = lambda x: oracle.select_heads(x, qheads, 2).reshape(shp_q)
    sk = lambda x: oracle.select_heads(x, groups, 2).reshape(shp_k)
    sv = lambda x: oracle.select_heads(x, qheads, 1).reshape(shp_q[:3])
    O_ref, L_ref = oracle.forward_gqa_from_c(sq(ins["Q"]), sk(ins["K"]), sk(ins["V"]), sv(c32), wl.w, wl.scale)
    ref = oracle.backward_gqa_from_c(sq(ins["Q"]), sk(ins["K"]), sk(ins["V"]), sv(c32), sq(ins["dO"]), wl.w, wl.scale)
    got = {"O": sq(host(Od)), "L": sv(host(Ld)), "dQ": sq(host(dQ)), "dK": sk(host(dK)), "dV": sk(host(dV)),
           "dalpha": sv(host(dalpha))}
    ref.update({"O": O_ref, "L": L_ref})
    LAST["c_span"] = window_span(c32, wl.w)
    # Alg. 3 on the stored output the kernels were given, and the bound of an identically-zero gradient
    ref["saved"] = oracle.backward_gqa_from_c(sq(ins["Q"]), sk(ins["K"]), sk(ins["V"]), sv(c32), sq(ins["dO"]), wl.w,
                                              wl.scale, O_saved=sq(host(Od)))
    ref["zero"] = zero_gradient_bounds(sq(ins["dO"]), np.repeat(sk(ins["V"]), G, axis=1), sq(ins["Q"]),
                                       np.repeat(sk(ins["K"]), G, axis=1), wl.scale, G)
    return got, ref


@pytest.mark.parametrize("B,H,Hkv,N,d,w", [(1, 4, 2, 77, 64, 9), (2, 6, 2, 130, 128, 500), (1, 4, 1, 65, 64, 1),
                                           # large enough for the fp32 matrix-core kernels
                                           (1, 8, 2, 1100, 128, 400), (1, 4, 1, 1300, 64, 200)])
def test_gqa_f32(g, oracle, B, H, Hkv, N, d, w):
    note("gqa f32", B, H, Hkv, N, d, w)
    wl = gi.custom("gqa32", B, H, N, d, w, "f32", alpha_mu=-1.0, index=13, backward=True, kv_heads=Hkv)
    got, ref = run_gqa(g, oracle, wl)
    assert rel_inf(got["O"], ref["O"]) <= 1e-5
    assert (np.abs(got["L"] - ref["L"]) <= 1e-5 * np.abs(ref["L"]).max() + 1e-5).all()
    check_grads(got, ref, 1e-5, "gqa f32")


# the one-wave-per-row kernels at the edges of their steps: one full step, one key more, several.  A forward of up to 1024 rows takes
# 64 (d = 64) or 32 keys a step, of more rows 16 or 8, as every backward does
@pytest.mark.parametrize("B,H,Hkv,N,d,w", [(1, 8, 1, 66, 64, 64), (1, 4, 1, 97, 64, 65), (1, 2, 2, 131, 64, 129),
                                           (2, 2, 2, 33, 128, 32), (1, 2, 1, 70, 128, 33),
                                           (2, 8, 8, 130, 64, 16), (1, 12, 4, 97, 64, 17), (1, 9, 3, 131, 128, 8), (2, 5, 5, 129, 128, 9)])
def test_f32_row_steps(g, oracle, B, H, Hkv, N, d, w):
    note("f32 row steps", B, H, Hkv, N, d, w)
    wl = gi.custom("f32s", B, H, N, d, w, "f32", alpha_mu=-1.0, index=18, backward=True, kv_heads=Hkv)
    got, ref = run_gqa(g, oracle, wl)
    assert rel_inf(got["O"], ref["O"]) <= 1e-5
    assert (np.abs(got["L"] - ref["L"]) <= 1e-5 * np.abs(ref["L"]).max() + 1e-5).all()
    check_grads(got, ref, 1e-5, "f32 row steps")


@pytest.mark.parametrize("B,H,Hkv,N,d,w,two", [
    # rows of one step, 8 keys at d = 128, and more of them than 32768: a launch for each pass, the first forms D; just not
    (12, 12, 4, 229, 128, 8, True), (8, 9, 9, 517, 128, 1, True), (9, 61, 61, 61, 128, 8, True),
    (12, 12, 4, 227, 128, 8, False), (12, 12, 4, 229, 128, 9, False), (3, 12, 4, 229, 64, 8, False),
])
def test_backward_f32_rows_in_two_launches(g, oracle, B, H, Hkv, N, d, w, two):
    note("f32 rows, two launches", B, H, Hkv, N, d, w)
    wl = gi.custom("f32two", B, H, N, d, w, "f32", alpha_mu=-1.0, index=30, backward=True, kv_heads=Hkv)
    results = []
    names = launched(g, lambda: results.extend(run_gqa(g, oracle, wl)))
    assert ("bwd_dq" in names) == two and "bwd_rowdot" not in names
    got, ref = results
    check_grads(got, ref, 1e-5, "f32 rows, two launches", tiny=N == 1)


@pytest.mark.parametrize("B,H,Hkv,N,d,w", [(2, 6, 6, 300, 128, 77), (2, 8, 2, 130, 64, 100), (4, 1, 1, 700, 64, 700), (1, 1, 1, 256, 64, 64)])
def test_f32_rows_gate_gradient_cancels(g, oracle, B, H, Hkv, N, d, w):
    # d(alpha)[..., 0] is the sum of every dS as a column minus the sum of every dS as a row: zero.  The two kernels form the same
    # dS bit by bit and add it up in fp64, so what is left is the rounding of the 2 N stored sums, at most 2^-24 of each and
    # independent (four deviations of 2^-24 / sqrt(3) each), and that of the scan, some additions of 2^-24 of a suffix sum
    note("f32 rows, gate gradient", B, H, Hkv, N, d, w)
    wl = gi.custom("f32g", B, H, N, d, w, "f32", alpha_mu=-1.0, index=24, backward=True, kv_heads=Hkv)
    got, ref = run_gqa(g, oracle, wl)
    dc = ref["dalpha"] - np.concatenate([ref["dalpha"][..., 1:], np.zeros_like(ref["dalpha"][..., :1])], axis=-1)
    bound = 2.0 ** -24 * (4 / np.sqrt(3) * np.sqrt((dc ** 2).sum(axis=-1)) + np.abs(ref["dalpha"]).max(axis=-1))
    ratio = (np.abs(got["dalpha"][..., 0]) / bound).max()
    note("  |d(alpha)[..., 0]| over its bound", ratio)
    assert ratio <= 1


# (the one-wave-per-row kernels, the last steps of a row partly filled; the last two: more than 1024 rows, the forward's short steps)
@pytest.mark.parametrize("B,H,Hkv,N,d,w", [(1, 2, 1, 77, 64, 30), (1, 2, 2, 50, 128, 33), (1, 16, 8, 77, 64, 30), (1, 24, 24, 50, 128, 11)])
def test_f32_rows_with_infinities(g, oracle, B, H, Hkv, N, d, w):
    note("f32 rows with infinities", B, H, Hkv, N, d, w)
    wl = gi.custom("f32i", B, H, N, d, w, "f32", alpha_mu=-1.0, index=19, backward=True, kv_heads=Hkv)
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha", "dO")}
    c = dev(oracle.gate_prefix(ins["alpha"]).astype(np.float32), "f32")
    Q, K, V, dO = (dev(ins[t], "f32") for t in ("Q", "K", "V", "dO"))
    O, L = g.gfwa_forward_gqa(Q, K, V, c, w, wl.scale)
    want = [O, *g.gfwa_backward_gqa(Q, K, V, O, dO, c, L, w, wl.scale)]
    # one value column of one key: plus infinity in that column of the rows that see the key, all else as without it
    key, col = N // 2, 5
    Vi = V.clone()
    Vi[:, :, key, col] = float("inf")
    Oi, _ = g.gfwa_forward_gqa(Q, K, Vi, c, w, wl.scale)
    hit = torch.zeros_like(O, dtype=torch.bool)
    hit[:, :, key:key + w, col] = True
    assert (Oi[hit] == float("inf")).all() and torch.equal(Oi[~hit], O[~hit])
    # one gradient entry of one row: what does not depend on the row is as without it
    row = N // 3
    dOi = dO.clone()
    dOi[:, :, row, col] = float("inf")
    dQ, dK, dV, _ = g.gfwa_backward_gqa(Q, K, V, O, dOi, c, L, w, wl.scale)
    keys = torch.arange(N, device=DEV)
    free = (keys < row - w + 1) | (keys > row)
    assert torch.equal(dQ[:, :, keys != row], want[1][:, :, keys != row])
    assert torch.equal(dK[:, :, free], want[2][:, :, free]) and torch.equal(dV[:, :, free], want[3][:, :, free])
    others = torch.arange(d, device=DEV) != col
    assert torch.equal(dV[..., others], want[3][..., others])
    assert (dV[:, :, ~free, col] == float("inf")).all()


# (128 queries per workgroup; 64; 128 with one tile buffer.  One query head per key/value head where the largest value of one
# query would else add up to infinity)
F32_MATRIX_CORE = [(4, 2, 1100, 128, 400), (4, 4, 1300, 64, 300), (64, 64, 193, 64, 65), (300, 300, 97, 128, 40)]


# fp32 storage takes every finite value, and infinities where plain fp32 arithmetic gives a meaning to them, at any size
@pytest.mark.parametrize("H,Hkv,N,d,w", F32_MATRIX_CORE)
def test_f32_matrix_core_range(g, oracle, H, Hkv, N, d, w):
    note("f32 range", H, Hkv, N, d, w)
    wl = gi.custom("f32x", 1, H, N, d, w, "f32", alpha_mu=-2.0, index=20, backward=True, kv_heads=Hkv)
    ins = {t: gi.make_tensor(wl, t).astype(np.float32) for t in ("Q", "K", "V", "alpha", "dO")}
    ins["Q"][..., 0] = 1.0 + np.abs(ins["Q"][..., 0])
    c_host = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    c = dev(c_host, "f32")
    big, key, col = np.finfo(np.float32).max, N // 2, 5
    forward = lambda Q, K, V: g.gfwa_forward_gqa(dev(Q, "f32"), dev(K, "f32"), dev(V, "f32"), c, w, wl.scale)
    clean = [host(x) for x in forward(ins["Q"], ins["K"], ins["V"])]
    hit = np.zeros(clean[0].shape, dtype=bool)
    hit[:, :, key:key + w, col] = True

    def near(got, want, tag):
        note("  ", tag, rel_inf(got, want))
        assert np.isfinite(got).all() and rel_inf(got, want) <= 1e-5, tag

    # an infinite and the largest finite value in one column of V
    for x in (np.inf, big):
        V = ins["V"].copy()
        V[:, :, key, col] = x
        O, L = (host(y) for y in forward(ins["Q"], ins["K"], V))
        near(O[~hit], clean[0][~hit], f"V {x}: other elements")
        near(L, clean[1], "L")
        if np.isinf(x):
            assert (O[hit] == np.inf).all()
        else:
            O_ref, _ = oracle.forward_gqa_from_c(ins["Q"], ins["K"], V, c_host, w, wl.scale)
            near(O[hit], O_ref[hit], "V max")
    # a key nobody may see: the scores are minus infinity, the type's lowest value, or overflow
    K = ins["K"].copy()
    K[:, :, key, 0] = -1e5
    want = [host(x) for x in forward(ins["Q"], K, ins["V"])]
    for x in (-np.inf, -big):
        K[:, :, key, 0] = x
        for got, ref in zip(forward(ins["Q"], K, ins["V"]), want):
            near(host(got), ref, f"K {x}")
    Q, K = ins["Q"].copy(), ins["K"].copy()
    K[..., 0] = 0.0
    want = [host(x) for x in forward(Q, np.where(np.arange(N)[:, None] == key, np.eye(1, d) * -1e5, K).astype(np.float32), ins["V"])]
    Q[..., 0] *= 1e25
    K[:, :, key, 0] = -1.2345678e20
    for got, ref in zip(forward(Q, K, ins["V"]), want):
        near(host(got), ref, "overflowing product")
    # backward: the type's lowest value in K, its largest in V, in dO (scaled so that the results are finite)
    for name, x, shrink in (("K", -big, ()), ("V", big, ("dO",)), ("dO", big, ("V", "dO"))):
        t = {k: ins[k].copy() for k in ("Q", "K", "V", "dO")}
        for k in shrink:
            t[k] = (t[k] * np.float32(2.0 ** -30)).astype(np.float32)
        t[name][:, :, key, 0 if name == "K" else col] = x
        O_ref, L_ref = oracle.forward_gqa_from_c(t["Q"], t["K"], t["V"], c_host, w, wl.scale)
        ref = oracle.backward_gqa_from_c(t["Q"], t["K"], t["V"], c_host, t["dO"], w, wl.scale)
        got = g.gfwa_backward_gqa(*(dev(t[k], "f32") for k in ("Q", "K", "V")), dev(O_ref.astype(np.float32), "f32"), dev(t["dO"], "f32"),
                                  c, dev(L_ref.astype(np.float32), "f32"), w, wl.scale)
        for k, y in zip(("dQ", "dK", "dV", "dalpha"), got):
            r = rel_l2(host(y), ref[k].reshape(y.shape))
            note("  backward", name, x, k, r)
            assert r <= 1e-5, (name, k)


@pytest.mark.parametrize("H,Hkv,N,d,w", F32_MATRIX_CORE)
def test_f32_matrix_core_small_values(g, oracle, H, Hkv, N, d, w):
    # matrices of values of 2^-118, exactly the scaled ones: every result that is linear in the matrix is the scaled one too,
    # to the fp32 bar (2^-149, the spacing of the smallest fp32 values, is 2^-31 of 2^-118)
    note("f32 small values", H, Hkv, N, d, w)
    wl = gi.custom("f32z", 1, H, N, d, w, "f32", alpha_mu=-2.0, index=21, backward=True, kv_heads=Hkv)
    Q, K, V, dO = (dev(gi.make_tensor(wl, t), "f32") for t in ("Q", "K", "V", "dO"))
    c = dev(oracle.gate_prefix(gi.make_tensor(wl, "alpha")).astype(np.float32), "f32")
    tiny = 2.0 ** -118

    def step(Q, K, V, dO, scale=wl.scale):
        O, L = g.gfwa_forward_gqa(Q, K, V, c, w, scale)
        return dict(zip(("O", "dQ", "dK", "dV", "dalpha"), (O, *g.gfwa_backward_gqa(Q, K, V, O, dO, c, L, w, scale))))

    clean = step(Q, K, V, dO)
    ref = {k: host(v) for k, v in clean.items()}
    for name, got, scaled in (("dO", step(Q, K, V, dO * tiny), ("dQ", "dK", "dV", "dalpha")),
                              ("V", step(Q, K, V * tiny, dO), ("O", "dQ", "dK", "dalpha"))):
        for k in ref:
            r = rel_l2(host(got[k]) / (tiny if k in scaled else 1.0), ref[k])
            note("  small", name, k, r)
            assert r <= 1e-5, (name, k)
    # a key (query) matrix that small leaves the gate alone to decide; it is the same matrix in dQ (dK)
    zero = step(Q, torch.zeros_like(K), V, dO)
    assert float(zero["dQ"].abs().max()) == 0.0
    like = step(Q, K, V, dO, scale=2.0 ** -60)  # scores of 2^-60: nothing beside the gate
    for name, got, k in (("K", step(Q, K * tiny, V, dO), "dQ"), ("Q", step(Q * tiny, K, V, dO), "dK")):
        r = rel_l2(host(got[k]) / (tiny * wl.scale), host(like[k]) / 2.0 ** -60)
        note("  small", name, k, r)
        assert r <= 1e-5, (name, k)


@pytest.mark.parametrize("B,H,Hkv,N,d,w,groups", [
    # the matrix-core kernels at the edges of their tiles: 64-, 128- and 256-query tiles with a last row, a last block and a
    # full one, windows of one key, inside one block, across one, past the sequence; sampled heads
    (2, 4, 4, 1025, 64, 97, [0, 7]), (1, 6, 2, 1153, 128, 165, [0, 1]), (2, 32, 32, 1057, 128, 31, [0, 63]),
    (4, 16, 16, 1281, 64, 33, [0, 63]), (8, 32, 32, 256, 128, 500, [0, 255]), (2, 32, 16, 1120, 64, 129, [0, 31]),
    # d = 64, short bands: 64 queries and keys per workgroup
    (6, 64, 64, 129, 64, 1, [0, 383]), (3, 100, 25, 65, 64, 50, [0, 74]), (4, 80, 80, 33, 64, 31, [0, 319]),
    (2, 150, 150, 100, 64, 90, [0, 299]),  # (the forward with 128)
    # d = 128, more sequences that end within 128 than CUs: one tile buffer
    (5, 60, 60, 97, 128, 33, [0, 299]), (1, 260, 130, 128, 128, 128, [0, 129]),
])
def test_f32_matrix_core_tiles(g, oracle, B, H, Hkv, N, d, w, groups):
    note("f32 tiles", B, H, Hkv, N, d, w)
    wl = gi.custom("f32t", B, H, N, d, w, "f32", alpha_mu=-1.0, index=16, backward=True, kv_heads=Hkv)
    results = []
    assert "bwd_rowdot" in launched(g, lambda: results.extend(run_gqa(g, oracle, wl, groups=groups)))  # (not the one-wave-per-row kernels)
    got, ref = results
    assert rel_inf(got["O"], ref["O"]) <= 1e-5
    assert (np.abs(got["L"] - ref["L"]) <= 1e-5 * np.abs(ref["L"]).max() + 1e-5).all()
    check_grads(got, ref, 1e-5, "f32 tiles")


GQA_BF16 = [(1, 4, 1, 300, 128, 64), (2, 8, 2, 515, 64, 512), (1, 4, 2, 1536, 128, 1024), (1, 8, 2, 2050, 64, 700),
            (1, 2, 1, 37, 64, 5), (1, 3, 1, 4099, 128, 300)]


@pytest.mark.parametrize("B,H,Hkv,N,d,w", GQA_BF16)
def test_gqa_bf16(g, oracle, ws_variant, B, H, Hkv, N, d, w):
    note("gqa bf16", ws_variant, B, H, Hkv, N, d, w)
    wl = gi.custom("gqa16", B, H, N, d, w, "bf16", alpha_mu=-1.0, index=14, backward=True, kv_heads=Hkv)
    got, ref = run_gqa(g, oracle, wl)
    check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag="gqa")
    check_grads(got, ref, 1e-2, "gqa bf16")


@pytest.mark.parametrize("name,groups", [("lm_gqa_bwd", [0, 7, 15]), ("long_gqa_bwd", [3])])
def test_gqa_bf16_full_size(g, oracle, ws_variant, name, groups):
    note("gqa full size", ws_variant, name, groups)
    got, ref = run_gqa(g, oracle, gi.WORKLOADS[name], groups=groups)
    check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag=name)
    check_grads(got, ref, 1e-2, name)


@pytest.mark.parametrize("B,H,Hkv,N,d,w,groups", [
    # query tiles and key tiles shared out over groups of waves: 32 and 64 queries per workgroup, 32 keys per workgroup
    (1, 8, 8, 1101, 128, 700, [0, 7]), (3, 16, 16, 450, 64, 200, [0, 47]), (1, 4, 4, 1000, 128, 333, [0, 3]),
    # groups of 8 query heads (the most the split dK/dV pass has room for) and of 9; a last key block of one key
    (1, 8, 1, 769, 64, 300, [0]), (1, 9, 1, 257, 64, 100, [0]), (1, 8, 1, 417, 128, 5000, [0]),
])
def test_backward_bf16_split(g, oracle, ws_variant, B, H, Hkv, N, d, w, groups):
    note("backward split", ws_variant, B, H, Hkv, N, d, w)
    wl = gi.custom("bsplit", B, H, N, d, w, "bf16", alpha_mu=-1.0, index=14, backward=True, kv_heads=Hkv)
    got, ref = run_gqa(g, oracle, wl, groups=groups)
    check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag="split")
    check_grads(got, ref, 1e-2, "split")


def launched(g, call):
    """Names of the kernels that `call` launches."""
    g.gfwa_profile_enable(True)
    call()
    torch.cuda.synchronize()
    g.gfwa_profile_enable(False)
    return {name for name, (_, count) in g.gfwa_profile_read().items() if count}


@pytest.mark.parametrize("B,H,Hkv,N,d,w,one", [
    # both passes in one launch: a workgroup each of a single row, either side of a 32-key and a 64-query block, eight query
    # heads on a key/value head, exactly a workgroup for every CU, more than that with bands of half the sequence
    (1, 1, 1, 1, 64, 4, True), (1, 2, 1, 33, 128, 7, True), (2, 3, 3, 65, 64, 64, True), (1, 8, 1, 97, 64, 1000, True),
    (1, 8, 1, 161, 128, 33, True), (4, 16, 16, 70, 64, 35, True), (2, 6, 2, 449, 128, 225, True),
    # and just not: one head more with a shorter band; a chain of more than 96 blocks at d = 128
    (1, 65, 65, 70, 64, 34, False), (1, 8, 1, 417, 128, 500, False),
    # two rounds: short sequences whose keys fill just the first, less of it and more; longer ones up to 2.1; at d = 128 a long chain of
    # one head and of two
    (5, 15, 15, 91, 64, 91, False), (5, 13, 13, 91, 64, 91, True), (6, 15, 15, 91, 64, 91, True), (1, 32, 8, 673, 64, 673, True),
    (1, 7, 7, 1400, 128, 1400, False), (1, 10, 5, 1441, 128, 1441, True),
])
def test_backward_bf16_one_launch(g, oracle, ws_variant, B, H, Hkv, N, d, w, one):
    note("one launch", ws_variant, B, H, Hkv, N, d, w)
    wl = gi.custom("one", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=23, backward=True, kv_heads=Hkv)
    results = []
    names = launched(g, lambda: results.extend(run_gqa(g, oracle, wl)))
    assert ("bwd_dq" not in names) == one
    got, ref = results
    check_grads(got, ref, 1e-2, "one launch", tiny=N <= 33)


@pytest.mark.parametrize("B,H,Hkv,N,w", [(1, 32, 8, 700, 1024), (1, 16, 8, 1577, 1416)])
def test_large_workspace_does_not_change_the_route_where_dkv_is_split(g, B, H, Hkv, N, w):
    # the split dK/dV pass stores no dS blocks, so the dQ pass is the one that serves the minimum workspace (which
    # forms D itself, without the row-dot launch), not the one that would have read them
    note("large workspace", B, H, Hkv, N, w)
    wl = gi.custom("lws", B, H, N, 128, w, "bf16", alpha_mu=-1.0, index=22, backward=True, kv_heads=Hkv)
    ins = gi.make_inputs(wl)
    Q, K, V, dO = (dev(ins[t], "bf16") for t in ("Q", "K", "V", "dO"))
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    O, L = g.gfwa_forward_gqa(Q, K, V, c, w, wl.scale)
    sizes = [f(torch.bfloat16, B, H, N, 128, w) for f in (g.gfwa_backward_workspace_bytes, g.gfwa_backward_fast_workspace_bytes)]
    assert sizes[1] > sizes[0]  # (with one query head per key/value head the blocks are used)
    results = []
    for n in sizes:
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
        assert launched(g, lambda: results.append(g.gfwa_backward_gqa(Q, K, V, O, dO, c, L, w, wl.scale, workspace=ws))) == {
            "bwd_dq", "bwd_dkv", "gate_grad_scan"}
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,H,Hkv,N,d,w,groups", [
    # the forward and the backward kernels of whole 128-row tiles, where they have a ragged end: last tiles of 3 rows
    # to one row, odd windows, windows past the sequence, grouped heads; sampled heads
    (1, 20, 20, 4099, 128, 301, [0, 19]), (1, 48, 12, 2049, 128, 333, [0, 11]), (2, 100, 100, 513, 128, 1000, [0, 199]),
    (1, 25, 25, 4099, 64, 301, [0, 24]), (1, 40, 10, 3001, 64, 333, [0, 9]), (1, 250, 250, 641, 64, 5000, [0, 249]),
    (1, 8, 8, 5003, 128, 2999, [3]),  # (these, the dQ pass from dS blocks, with the large workspace only)
])
def test_bf16_whole_tiles_ragged(g, oracle, ws_variant, B, H, Hkv, N, d, w, groups):
    note("whole tiles", ws_variant, B, H, Hkv, N, d, w)
    wl = gi.custom("whole", B, H, N, d, w, "bf16", alpha_mu=-1.5, index=23, backward=True, kv_heads=Hkv)
    results = []
    names = launched(g, lambda: results.extend(run_gqa(g, oracle, wl, groups=groups)))
    assert ("bwd_rowdot" in names) == (H > 8 or VARIANT["fast"])  # the launch in front of the whole-tile dQ kernel
    got, ref = results
    check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag="whole tiles")
    check_grads(got, ref, 1e-2, "whole tiles")


def test_backward_d64_two_workgroups_per_cu_repeats_bit_exactly(g):
    # rows leave through inline-assembly stores; with two workgroups of the dK/dV pass on a CU a missing wait state
    # between a store and the next write of its data registers showed as a few wrong elements of dV
    B, H, N, d, w = 4, 8, 2050, 64, 700
    wl = gi.custom("repeat", B, H, N, d, w, "bf16", alpha_mu=-2.0, index=13, backward=True)
    ins = gi.make_inputs(wl)
    Q, K, V, dO = (dev(ins[t], "bf16") for t in ("Q", "K", "V", "dO"))
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    O, L = g.gfwa_forward(Q, K, V, c, w, wl.scale)
    first = g.gfwa_backward(Q, K, V, O, dO, c, L, w, wl.scale)
    for _ in range(4):
        for a, b in zip(g.gfwa_backward(Q, K, V, O, dO, c, L, w, wl.scale), first):
            assert torch.equal(a, b)


def test_gqa_with_one_head_per_group_is_the_plain_call(g, oracle):
    wl = gi.custom("gqa1", 2, 3, 700, 128, 200, "bf16", alpha_mu=-1.0, index=14, backward=True)
    ins = {t: dev(gi.make_tensor(wl, t), "bf16") for t in ("Q", "K", "V", "dO")}
    cd = g.gfwa_gate_prefix(dev(gi.make_tensor(wl, "alpha"), "f32"))
    O1, L1 = g.gfwa_forward(ins["Q"], ins["K"], ins["V"], cd, wl.w, wl.scale)
    O2, L2 = g.gfwa_forward_gqa(ins["Q"], ins["K"], ins["V"], cd, wl.w, wl.scale)
    assert torch.equal(O1, O2) and torch.equal(L1, L2)
    r1 = g.gfwa_backward(ins["Q"], ins["K"], ins["V"], O1, ins["dO"], cd, L1, wl.w, wl.scale)
    r2 = g.gfwa_backward_gqa(ins["Q"], ins["K"], ins["V"], O1, ins["dO"], cd, L1, wl.w, wl.scale)
    for a, b in zip(r1, r2):
        assert torch.equal(a, b)


def test_forward_is_deterministic(g, oracle):
    wl = gi.custom("detf", 1, 2, 1500, 128, 700, "bf16", alpha_mu=-1.0, index=15)
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha")}
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    args = [dev(ins[t], "bf16") for t in ("Q", "K", "V")]
    O1, L1 = g.gfwa_forward(*args, c, wl.w, wl.scale)
    O2, L2 = g.gfwa_forward(*args, c, wl.w, wl.scale)
    torch.cuda.synchronize()
    assert torch.equal(O1, O2) and torch.equal(L1, L2)


def test_backward_is_deterministic(g, oracle, ws_variant):
    wl = gi.custom("det", 1, 2, 700, 128, 200, "bf16", alpha_mu=-1.0, index=13, backward=True)
    a, _ = run_backward(g, oracle, wl, chained=True)
    b, _ = run_backward(g, oracle, wl, chained=True)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k])


def test_outputs_do_not_spill_past_their_buffers(g):
    """Guard bands around O and L stay untouched for a ragged N."""
    wl = gi.custom("guard", 1, 1, 333, 128, 50, "bf16", index=14)
    ins = gi.make_inputs(wl)
    Q, K, V = (dev(ins[t], "bf16") for t in ("Q", "K", "V"))
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    pad = 4096
    Obuf = torch.full((pad + 333 * 128 + pad,), 7.0, dtype=torch.bfloat16, device=DEV)
    Lbuf = torch.full((pad + 333 + pad,), 7.0, dtype=torch.float32, device=DEV)
    O = Obuf[pad:pad + 333 * 128].view(1, 1, 333, 128)
    L = Lbuf[pad:pad + 333].view(1, 1, 333)
    g.gfwa_forward(Q, K, V, c, wl.w, wl.scale, O=O, L=L)
    torch.cuda.synchronize()
    for buf, n in ((Obuf, 333 * 128), (Lbuf, 333)):
        assert (buf[:pad] == 7.0).all() and (buf[pad + n:] == 7.0).all()
    assert not (O == 7.0).all()


def test_step_under_graph_capture_replays_bit_exactly(g, oracle, ws_variant):
    # the whole step (prefix, forward, backward) allocates nothing and clears nothing with memsets, so it
    # can be captured in a HIP graph; every replay must give the eager run's bits, also with other work
    # and synchronizations between the replays
    wl = gi.custom("graph", 1, 4, 3000, 128, 700, "bf16", alpha_mu=-1.0, index=26, backward=True, kv_heads=2)
    ins = {t: dev(gi.make_tensor(wl, t), "bf16") for t in ("Q", "K", "V", "dO")}
    alpha = dev(gi.make_tensor(wl, "alpha"), "f32")
    B, H, N, d = ins["Q"].shape
    c = torch.empty_like(alpha)
    O, L = torch.empty_like(ins["Q"]), torch.empty_like(alpha)
    dQ, dK, dV, dal = torch.empty_like(ins["Q"]), torch.empty_like(ins["K"]), torch.empty_like(ins["V"]), torch.empty_like(alpha)
    ws = bwd_workspace(g, ins["Q"], wl.w)

    def step():
        g.gfwa_gate_prefix(alpha, c)
        g.gfwa_forward_gqa(ins["Q"], ins["K"], ins["V"], c, wl.w, wl.scale, O=O, L=L)
        g.gfwa_backward_gqa(ins["Q"], ins["K"], ins["V"], O, ins["dO"], c, L, wl.w, wl.scale, workspace=ws,
                            dQ=dQ, dK=dK, dV=dV, dalpha=dal)

    outs = (c, O, L, dQ, dK, dV, dal)
    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in outs]
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()                                   # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    for rep in range(3):
        for t in outs:
            t.fill_(float("nan")) if t.is_floating_point() else t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, w_ in zip(outs, want):
            assert torch.equal(t, w_), f"replay {rep}"
        step()                                   # eager work between the replays
        torch.cuda.synchronize()


def test_offsets_beyond_32_bits(g, oracle, ws_variant):
    # 2^31 elements per [B,H,N,d] tensor: element offsets of the last heads do not fit 32 bits.  Inputs
    # are drawn on the GPU (seeded); the oracle gets the first and the last head.
    B, H, N, d, w = 8, 32, 65536, 128, 64
    assert B * H * N * d == 1 << 31
    gen = torch.Generator(device=DEV).manual_seed(31)
    mk = lambda: torch.randn(B, H, N, d, device=DEV, generator=gen, dtype=torch.bfloat16)
    Q, K, V, dO = mk(), mk(), mk(), mk()
    alpha = torch.nn.functional.softplus(torch.randn(B, H, N, device=DEV, generator=gen) - 1.0)
    scale = 1.0 / d ** 0.5
    c = g.gfwa_gate_prefix(alpha)
    O, L = g.gfwa_forward(Q, K, V, c, w, scale)
    ws = bwd_workspace(g, Q, w)   # with the dS blocks: 3.2 GB, block offsets of the last heads beyond 32 bits too
    note("  workspace", ws_variant, ws.numel())
    dQ, dK, dV, dalpha = g.gfwa_backward(Q, K, V, O, dO, c, L, w, scale, workspace=ws)
    torch.cuda.synchronize()
    for b, h in ((0, 0), (B - 1, H - 1)):
        note("  head", b, h)
        pick = lambda t: host(t[b, h])[None, None]
        c_ref = oracle.gate_prefix(pick(alpha))
        assert np.abs(pick(c) - c_ref).max() <= 4 * np.finfo(np.float32).eps * c_ref.max()
        c32 = pick(c)
        O_ref, L_ref = oracle.forward_from_c(pick(Q), pick(K), pick(V), c32, w, scale)
        LAST["c_span"] = window_span(c32, w)
        check_bf16_forward(pick(O), pick(L), O_ref, L_ref, tag="big")
        ref = oracle.backward_from_c(pick(Q), pick(K), pick(V), c32, pick(dO), w, scale)
        ref["saved"] = oracle.backward_from_c(pick(Q), pick(K), pick(V), c32, pick(dO), w, scale, O_saved=pick(O))
        got = {"dQ": pick(dQ), "dK": pick(dK), "dV": pick(dV), "dalpha": pick(dalpha)}
        check_grads(got, ref, 1e-2, "big")


def _random_shapes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        d = int(rng.choice([64, 128]))
        G = int(rng.choice([1, 1, 2, 3, 4]))
        Hkv = int(rng.integers(1, 3))
        N = int(rng.choice([rng.integers(1, 40), rng.integers(40, 300), rng.integers(300, 1400)]))
        w = int(rng.choice([1, rng.integers(2, 70), rng.integers(70, 600), N, N + 17, 4 * N + 1]))
        out.append((int(rng.integers(1, 3)), Hkv * G, Hkv, N, d, max(1, w)))
    return out


# more workgroups than one launch takes (2^32 work items): the forward goes in several, by key/value heads or by the query
# heads of the only one, and the fp32 backward in one launch for each pass
@pytest.mark.parametrize("B,H,Hkv", [(3, (1 << 24) // 3, (1 << 24) // 3), (4, 1 << 22, 1 << 22), (2, 1 << 23, 1 << 21), (1, 1 << 24, 1)])
def test_forward_bf16_at_the_most_heads(g, B, H, Hkv):
    note("most heads", B, H, Hkv)
    gen = torch.Generator(device="cuda").manual_seed(5)
    normal = lambda *shape, dtype=torch.bfloat16: torch.randn(shape, generator=gen, device="cuda", dtype=dtype)
    Q, K, V = normal(B, H, 1, 64), normal(B, Hkv, 1, 64), normal(B, Hkv, 1, 64)
    c = normal(B, H, 1, dtype=torch.float32)
    O, L = (g.gfwa_forward if H == Hkv else g.gfwa_forward_gqa)(Q, K, V, c, 4, 0.125)
    G = H // Hkv
    for lo in range(0, H, 1 << 20):
        part = torch.arange(lo, min(H, lo + (1 << 20)), device="cuda")
        assert (O[:, part] == V[:, part // G]).all()  # one key: its value, and its score
        # 64 additions of 2^-24 of sums that stay below 64, times 0.125
        score = 0.125 * (Q[:, part].double() * K[:, part // G].double()).sum(-1)
        assert (L[:, part].double() - score).abs().max() <= 3e-5


def test_backward_f32_with_more_blocks_than_one_launch_takes(g, oracle):
    B, H, N, d, scale = 2, 1 << 22, 2, 64, 0.125
    note("most blocks", B, H, N, d)
    gen = torch.Generator(device="cuda").manual_seed(6)
    normal = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    Q, K, V, dO = (normal(B, H, N, d) for _ in range(4))
    alpha = normal(B, H, N).exp_()
    c = g.gfwa_gate_prefix(alpha)
    O, L = g.gfwa_forward(Q, K, V, c, N, scale)
    dQ, dK, dV, dalpha = g.gfwa_backward(Q, K, V, O, dO, c, L, N, scale)
    torch.cuda.synchronize()
    for bh in [(0, 0), (0, H // 2), (0, H - 1), (1, 0), (1, 1), (1, H - 1)]:
        one = lambda x: host(x[bh]).astype(np.float32)[None, None]
        ref = oracle.backward(one(Q), one(K), one(V), one(alpha), one(dO), N, scale)
        for name, got in (("dQ", dQ), ("dK", dK), ("dV", dV), ("dalpha", dalpha)):
            assert np.abs(host(got[bh]) - ref[name][0, 0]).max() <= 1e-5 * max(1.0, np.abs(ref[name]).max()), (bh, name)
    for got in (dQ, dK, dV, dalpha):
        assert torch.isfinite(got).all()



@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_random_shapes_forward_backward(g, oracle, ws_variant, dtype):
    if dtype == "f32" and ws_variant == "fast_ws":
        pytest.skip("fp32 storage has one variant")
    # seeded random shapes: ragged N, windows shorter and longer than the sequence, grouped heads
    for case, (B, H, Hkv, N, d, w) in enumerate(_random_shapes(28, 2512)):
        note("random shape", ws_variant, case, (B, H, Hkv, N, d, w), dtype)
        wl = gi.custom("rnd", B, H, N, d, w, dtype, alpha_mu=-1.0, index=28 + case % 4, backward=True, kv_heads=Hkv)
        got, ref = run_gqa(g, oracle, wl)
        if dtype == "bf16":
            check_bf16_forward(got["O"], got["L"], ref["O"], ref["L"], tag=f"rnd{case}")
            check_grads(got, ref, 1e-2, f"rnd{case}")
        else:
            assert rel_inf(got["O"], ref["O"]) <= 1e-5
            assert (np.abs(got["L"] - ref["L"]) <= 1e-5 * np.abs(ref["L"]).max() + 1e-5).all()
            check_grads(got, ref, 1e-5, f"rnd{case}")


def test_gate_kernels_with_pointers_off_the_16_byte_grid(g, oracle):
    # buffers that are 4-byte but not 16-byte aligned: the scan kernels' accesses of four elements at any address, one by one at a row's end
    B, H, N = 2, 3, 1000
    wl = gi.custom("unal", B, H, N, 64, 8, alpha_mu=-1.0, index=5)
    h, beta = gi.make_gate_inputs(wl)
    dal = gi.normal(wl.seed("dO"), h.shape).astype(np.float32)
    n = B * H * N

    def shifted(x):  # same values, storage starting 4 bytes into an allocation
        buf = torch.empty(n + 1, dtype=torch.float32, device=DEV)
        view = buf[1:].view(B, H, N)
        view.copy_(torch.from_numpy(x).to(DEV))
        assert view.data_ptr() % 16 == 4
        return view

    hs, bs, ds = shifted(h), shifted(beta), shifted(dal)
    out = shifted(np.zeros_like(h))
    c = host(g.gfwa_gate_activation_prefix(hs, bs, GATE_EPS, c=out))
    ref = oracle.gate_prefix(oracle.gate_activation(h, beta, GATE_EPS))
    assert np.abs(c - ref).max() <= 8 * np.finfo(np.float32).eps * ref.max()
    c2 = host(g.gfwa_gate_prefix(hs, c=out))
    ref2 = oracle.gate_prefix(h)
    assert np.abs(c2 - ref2).max() <= 4 * np.finfo(np.float32).eps * np.abs(ref2).max() + 1e-6
    dh_o, db_o = shifted(np.zeros_like(h)), shifted(np.zeros_like(h))
    dh, dbeta = g.gfwa_gate_activation_backward(hs, bs, GATE_EPS, ds, dh=dh_o, dbeta=db_o)
    rh, rb = oracle.gate_activation_backward(h, beta, GATE_EPS, dal)
    assert rel_l2(host(dh), rh) <= 1e-6 and rel_l2(host(dbeta), rb) <= 1e-6
