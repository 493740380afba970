"""Bands that the gate has erased before their window ends: the kernels leave those blocks out (csrc/band_reach.h), and nothing shows.

Checked against the oracle, which sums every window to its end, with the bars of test_gpu_parity, and by properties: a far key that outweighs
its decay counts, a far row that is not finite shows in every row that sees it.
"""
import numpy as np
import pytest
import torch

import gfwa_inputs as gi
import test_gpu_parity as par
from test_gpu_parity import DEV, check_bf16_forward, check_grads, dev, host, note, rel_inf

pytestmark = pytest.mark.gpu
g = par.g

# B, H, Hkv, N, d, w, dtype, alpha_mu, the forward kernel (None: this forward is too small to look at norms, the backward does).  Kernels and looks are
# those of 256 CUs.
SPLIT, WHOLE64, F32 = "fwd_split_bf16_kernel", "fwd_bf16_kernel<64>", "fwd_f32_mfma_kernel"
SHAPES = [
    (1, 32, 8, 3073, 128, 3000, "bf16", -1.0, SPLIT + "<128, 8, 4"),   # a last query tile of one row; grouped heads
    (4, 8, 8, 4097, 64, 3000, "bf16", -1.0, WHOLE64),                  # d = 64, whole tiles, the last of one row
    (1, 4, 4, 6146, 128, 4001, "bf16", -2.0, SPLIT + "<128, 8, 4"),    # a last tile of two rows
    (1, 6, 3, 5251, 64, 5251, "bf16", 0.5, SPLIT + "<64, 8, 4"),       # causal, the gate fast: most of every band is erased
    (1, 2, 2, 20000, 128, 14000, "bf16", -5.0, SPLIT + "<128, 8, 4"),  # blocks of 256 keys; more than 64 key tiles of 128 are left of a window
    (3, 6, 6, 6001, 128, 3500, "bf16", -1.5, "bf16_kernel"),           # d = 128, whole tiles
    (1, 12, 2, 6001, 64, 4000, "bf16", -1.0, WHOLE64),                 # six query heads to a key/value head: more than the norms' launch takes at once
    (1, 1, 1, 12801, 128, 8000, "bf16", -2.0, SPLIT + "<128, 4, 1"),   # 32 and 64 queries to a split workgroup
    (1, 2, 2, 9001, 128, 4500, "bf16", -2.0, SPLIT + "<128, 4, 2"),
    (1, 2, 2, 12000, 64, 12000, "bf16", -2.0, SPLIT + "<64, 4, 1"),
    (1, 1, 1, 10990, 64, 10990, "bf16", -2.0, None),                   # both passes of the backward in one launch
    (2, 24, 24, 2048, 128, 1024, "bf16", -1.0, None),
    (1, 8, 4, 2177, 128, 1600, "f32", -1.0, F32 + "<128, 4"),          # fp32: a last tile of one row
    (1, 8, 8, 4100, 64, 3000, "f32", -0.5, F32 + "<64, 4"),
    (2, 16, 8, 2305, 128, 1500, "f32", -1.0, F32 + "<128, 8"),         # 256 queries to a workgroup
]


def inputs(B, H, Hkv, N, d, w, dtype, mu, kind=None):
    wl = gi.custom("reach", B, H, N, d, w, dtype, alpha_mu=mu, index=17, backward=True)
    ins = {t: gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha", "dO")}
    for t in ("K", "V"):
        ins[t] = np.ascontiguousarray(ins[t][:, ::H // Hkv])
    if kind == "rising":  # the gate's prefix falls over a stretch: keys in front of it come back
        ins["alpha"][..., N // 3:N // 3 + 200] *= -1
    if kind == "heavy":   # a key early in the sequence that outweighs the decay over any window here
        # every score with it is about 2 * 64 * d / sqrt(d) and more
        ins["Q"] = gi.round_to_bf16(ins["Q"] + 2.0) if dtype == "bf16" else ins["Q"] + np.float32(2.0)
        ins["K"][:, :, N // 8] = 400.0
    return wl, ins


def step(g, wl, ins, c, keep):
    t = {k: dev(ins[k], wl.dtype) for k in ("Q", "K", "V", "dO")}
    O, L = g.gfwa_forward_gqa(t["Q"], t["K"], t["V"], c, wl.w, wl.scale)
    B, H, N, d = t["Q"].shape
    size = g.gfwa_backward_fast_workspace_bytes if keep else g.gfwa_backward_workspace_bytes
    ws = torch.empty(size(t["Q"].dtype, B, H, N, d, wl.w), dtype=torch.uint8, device=DEV)
    grads = g.gfwa_backward_gqa(t["Q"], t["K"], t["V"], O, t["dO"], c, L, wl.w, wl.scale, workspace=ws)
    torch.cuda.synchronize()
    return dict(zip(("O", "L", "dQ", "dK", "dV", "dalpha"), (O, L) + tuple(grads)))


def check_rows(got, ref, tol, skip=None):
    """Every row against its own size, down to rows of 2^-110 of the largest (weights below 2^-126 are zero)."""
    err, size = np.linalg.norm(got - ref, axis=-1), np.linalg.norm(ref, axis=-1)
    rows = size > 2.0 ** -110 * size.max()
    if skip is not None:
        rows[..., skip] = False
    worst = np.argmax(np.where(rows, err / np.where(size > 0, size, 1), 0))
    note(f"  worst row {worst}: {err.ravel()[worst] / size.ravel()[worst]:.2e}")
    assert (err[rows] <= tol * size[rows]).all(), (worst, err.ravel()[worst], size.ravel()[worst])


def kernels(call):
    """What the profiler calls the kernels that `call` runs (some names it leaves mangled)."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return {e.key for e in prof.key_averages()}


@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu,kernel", SHAPES)
def test_norms_are_looked_at(g, B, H, Hkv, N, d, w, dtype, mu, kernel):
    # the shapes here stand for kernels that shorten their bands: each of them runs, and the norms with it
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, mu)
    t = {k: dev(x, dtype if k != "alpha" else "f32") for k, x in ins.items()}
    c = g.gfwa_gate_prefix(t["alpha"])
    O, L = g.gfwa_forward_gqa(t["Q"], t["K"], t["V"], c, w, wl.scale)
    fwd = kernels(lambda: g.gfwa_forward_gqa(t["Q"], t["K"], t["V"], c, w, wl.scale))
    bwd = kernels(lambda: g.gfwa_backward_gqa(t["Q"], t["K"], t["V"], O, t["dO"], c, L, w, wl.scale))
    assert any("rowdot_reach" in k for k in bwd), bwd
    assert any("key_reach_kernel" in k for k in fwd) == (kernel is not None), fwd
    assert kernel is None or any(kernel in k for k in fwd), fwd


@pytest.mark.parametrize("kind", ["plain", "rising", "heavy"])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu", [s[:8] for s in SHAPES])
def test_erased_bands(g, oracle, B, H, Hkv, N, d, w, dtype, mu, kind):
    note("erased bands", B, H, Hkv, N, d, w, dtype, mu, kind)
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, mu, kind)
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    b, kv = B - 1, Hkv - 1   # the last group of query heads
    hs = slice(kv * (H // Hkv), H)
    pick = lambda x, s: x[b:b + 1, s]
    Q, dO, c = pick(ins["Q"], hs), pick(ins["dO"], hs), pick(c32, hs)
    K, V = pick(ins["K"], slice(kv, kv + 1)), pick(ins["V"], slice(kv, kv + 1))
    O_ref, L_ref = oracle.forward_gqa_from_c(Q, K, V, c, w, wl.scale)
    # (of a "rising" prefix the span is the largest difference of either sign)
    par.LAST["c_span"] = max(par.window_span(c, w), float(np.abs(c).max() - np.abs(c).min()) if kind == "rising" else 0.0)
    ref = None
    for keep in (False, True):
        if keep and (dtype == "f32" or d == 64):
            continue  # no larger workspace here
        out = step(g, wl, ins, dev(c32, "f32"), keep)
        got = {k: pick(host(x), slice(kv, kv + 1) if k in ("dK", "dV") else hs) for k, x in out.items()}
        if dtype == "bf16":
            check_bf16_forward(got["O"].reshape(O_ref.shape), got["L"].reshape(L_ref.shape), O_ref, L_ref, tag=kind)
        else:
            assert rel_inf(got["O"].reshape(O_ref.shape), O_ref) <= 1e-5
        if ref is None:
            ref = oracle.backward_gqa_from_c(Q, K, V, c, dO, w, wl.scale, O_saved=got["O"])
        # bf16 probabilities; the fp32 difference of gates and scores of up to 2^8 in an exponent, a few roundings of it
        heavy = N // 8 if kind == "heavy" else None
        check_rows(got["dV"].reshape(ref["dV"].shape), ref["dV"], 2e-2 if dtype == "bf16" else 1e-4, heavy)
        if kind == "heavy":
            # rows that see the key have all their weight there: its value comes out, and dV of the key is the sum of their dO
            seen = slice(N // 8 + 1, min(N, N // 8 + w))
            np.testing.assert_allclose(got["O"][0, 0, seen], np.broadcast_to(V[0, 0, N // 8], (seen.stop - seen.start, d)), atol=1e-6, rtol=0)
            want = dO[0, :, N // 8:seen.stop].astype(np.float64).sum(axis=(0, 1))
            err = np.linalg.norm(got["dV"][0, 0, N // 8] - want) / np.linalg.norm(want)
            assert err <= (1e-2 if dtype == "bf16" else 1e-5), err
            continue
        # A prefix that falls takes L and the gate up with it, by `fall`, and their difference in an exponent is rounded to 2^-24 of that
        # (2 16 8 2305: fall 80, L up to 90, dalpha at 1.17e-5 with whole bands, too)
        fall = float((np.maximum.accumulate(c, axis=-1) - c).max())
        check_grads({k: got[k].reshape(ref[k].shape) for k in ("dQ", "dK", "dV", "dalpha")}, ref,
                    1e-2 if dtype == "bf16" else 1e-5 + 2.0 ** -24 * 1.4427 * fall, kind)


# slow gates, so that weights lie densely: whole tiles and split kernels of both widths, grouped heads, fp32
FAR = [(1, 8, 8, 5003, 128, 3000, "bf16"), (3, 6, 6, 6001, 128, 3500, "bf16"), (1, 12, 2, 6001, 64, 4000, "bf16"), (4, 8, 8, 4500, 64, 3000, "bf16"),
       (1, 4, 4, 6146, 128, 4001, "bf16"), (1, 8, 4, 4500, 128, 3000, "f32"), (1, 8, 8, 4100, 64, 3000, "f32")]


@pytest.mark.parametrize("decay", [38, 70])   # weights of 2^-55 to 2^-64 and 2^-101 to 2^-110
@pytest.mark.parametrize("which", ["V", "V both", "V masked", "dO", "dO both", "dO masked"])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype", FAR)
def test_weights_that_are_all_a_row_has(g, oracle, B, H, Hkv, N, d, w, dtype, which, decay):
    # A weight that is nothing beside others is all of a row where what the others multiply is small or zero: a far value row that outweighs
    # its decay, alone or with one near the tile that is as heavy and that no query likes, or beside which all others are zero; a far row of dO
    # that does, likewise, or a loss that is masked but for two rows.  Every row of O, dV and dK against its own size.
    note("all a row has", which, decay, B, H, Hkv, N, d, w, dtype)
    if "masked" not in which and decay == 70:
        pytest.skip("rows heavy enough to show have squares beyond fp32")
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, -3.0)
    round_to = gi.round_to_bf16 if dtype == "bf16" else (lambda x: x)
    ins["K"] = round_to(ins["K"] * np.float32(0.25))
    ins["Q"] = round_to(ins["Q"] * np.float32(0.25) + np.float32(0.5))
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    c0 = c32[0, 0].astype(np.float64)
    if which[0] == "V":
        q0 = (N - 300) // 256 * 256   # first row of a query tile of any size
        far = np.nonzero((c0[:q0] <= c0[q0] - decay) & (np.arange(q0) % 64 == 63))[0][-1]   # the block's last row: of its largest weight
        assert far > q0 - w + 300
        near = q0 - 10
        if which != "V":  # (all other scores with it are about -280)
            ins["Q"][:, :, near] *= -1
            ins["K"][:, :, near] = -50.0
        heavy = [far] if which == "V" else [near, far]
        tensor = "V"
    else:
        near = N // 4 // 128 * 128    # first row of a key tile, whose other keys do not see this query
        far = np.nonzero((c0 >= c0[near + 127] + decay) & (np.arange(N) % 64 == 0))[0][0]   # the block's first row
        assert far < near + w
        heavy = [far] if which == "dO" else [near, far]
        tensor = "dO"
    if "masked" in which:
        rest = np.ones(N, bool)
        rest[heavy] = False
        ins[tensor][:, :, rest] = 0.0
    else:
        ins[tensor][:, :, heavy] *= np.float32(2.0 ** 58)
    out = step(g, wl, ins, dev(c32, "f32"), True)
    hs = slice(0, H // Hkv)
    Q, dO, c = (x[:1, hs] for x in (ins["Q"], ins["dO"], c32))
    K, V = ins["K"][:1, :1], ins["V"][:1, :1]
    # bf16 probabilities, dS and outputs; the fp32 difference of gates up to 2^8 in an exponent (2^-24 2^8 1.44), twice
    tol = 1e-2 if dtype == "bf16" else 5e-5
    if which[0] == "V":
        O_ref, _ = oracle.forward_gqa_from_c(Q, K, V, c, w, wl.scale)
        check_rows(host(out["O"])[:1, hs].reshape(O_ref.shape), O_ref, tol)
    else:
        ref = oracle.backward_gqa_from_c(Q, K, V, c, dO, w, wl.scale, O_saved=host(out["O"])[:1, hs])
        check_rows(host(out["dV"])[:1, :1].reshape(ref["dV"].shape), ref["dV"], tol)
        if which == "dO masked":
            check_rows(host(out["dK"])[:1, :1].reshape(ref["dK"].shape), ref["dK"], 2 * tol)


@pytest.mark.parametrize("which,value", [("V", np.inf), ("K", np.nan), ("dO", np.nan), ("Q", np.inf)])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu", [s[:8] for s in (SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[6], SHAPES[12])])
def test_far_rows_that_are_not_finite(g, oracle, B, H, Hkv, N, d, w, dtype, mu, which, value):
    # zero times infinity is NaN: a row that is not finite reaches every row that has it in its window, erased or not
    note("not finite", which, B, H, Hkv, N, d, w, dtype)
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, mu)
    at = N // 5
    ins[which][:, :, at] = value
    out = step(g, wl, ins, g.gfwa_gate_prefix(dev(ins["alpha"], "f32")), True)
    bad = lambda k, s: bool((~torch.isfinite(out[k][:, :, s])).any(dim=-1).all())
    later, earlier = slice(at, min(N, at + w)), slice(max(0, at - w + 1), at + 1)
    if which in ("K", "V"):
        assert bad("O", later) and bad("dQ", later)
    else:
        assert bad("dK", earlier) and (which == "Q" or bad("dV", earlier))


@pytest.mark.parametrize("B,H,N,d,w,dtype", [(3, 6, 6001, 128, 3500, "bf16"), (1, 4, 6146, 128, 4001, "bf16"), (4, 8, 4097, 64, 3000, "bf16"), (1, 1, 12801, 128, 8000, "bf16"),
                                             (1, 2, 12000, 64, 12000, "bf16"), (1, 1, 10990, 64, 10990, "bf16"), (1, 8, 2177, 128, 1600, "f32"),
                                             (1, 8, 4100, 64, 3000, "f32"), (2, 16, 2305, 128, 1500, "f32")])
def test_outputs_over_inputs(g, oracle, B, H, N, d, w, dtype):
    # outputs serve as scratch in front of the kernels, unless they lie over an input that is still read: then the bands stay whole, and the
    # results are the same bit for bit
    note("outputs over inputs", B, H, N, d, w, dtype)
    wl, ins = inputs(B, H, H, N, d, w, dtype, -1.0)
    c = g.gfwa_gate_prefix(dev(ins["alpha"], "f32"))
    want = step(g, wl, ins, c, False)
    t = {k: dev(ins[k], dtype) for k in ("Q", "K", "V", "dO")}
    over = t["Q"].clone()
    O, L = g.gfwa_forward(over, t["K"], t["V"], c, w, wl.scale, O=over)
    assert torch.equal(O, want["O"]) and torch.equal(L, want["L"])
    for name in ("c", "L"):
        x = {"c": c.clone(), "L": L.clone()}
        grads = g.gfwa_backward(t["Q"], t["K"], t["V"], O, t["dO"], x["c"], x["L"], w, wl.scale, dalpha=x[name])
        for k, got in zip(("dQ", "dK", "dV", "dalpha"), grads):
            # What is left out is exactly zero in the backward.  (The split dK/dV kernels, here those with d = 64 and one or two heads, round the
            # products of a band's last block before they add them to the column sums, the other blocks' together with the sum: half an ulp
            # each, 2^-24 of 16 here, of which dalpha adds up thousands: a random walk of 1e-4 at most, of values up to 15.)
            if k == "dalpha" and d == 64 and H < 4:
                assert rel_inf(host(got), host(want[k])) <= 2e-5, (name, k)
            else:
                assert torch.equal(got, want[k]), (name, k, rel_inf(host(got), host(want[k])))
