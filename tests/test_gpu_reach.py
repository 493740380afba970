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

# B, H, Hkv, N, d, w, dtype, alpha_mu: forwards large enough that the norms are asked for
SHAPES = [
    (1, 32, 8, 3073, 128, 3000, "bf16", -1.0),   # a last query tile of one row; whole tiles, grouped heads
    (2, 16, 16, 2311, 64, 1700, "bf16", -1.0),   # d = 64, the last tile has seven rows
    (1, 4, 4, 6146, 128, 4001, "bf16", -2.0),    # split forward, few tiles; a last tile of two rows
    (1, 6, 3, 5251, 64, 5251, "bf16", 0.5),      # causal, split, the gate fast: most of every band is erased
    (1, 2, 2, 20000, 128, 12000, "bf16", -2.0),  # blocks of 256 keys, more than 64 key tiles of 128 in a window
    (2, 24, 24, 2048, 128, 1024, "bf16", -1.5),
    (1, 12, 2, 2500, 64, 1500, "bf16", -1.0),    # six query heads to a key/value head: more than the norms' launch takes at once
    (1, 8, 4, 2177, 128, 1600, "f32", -1.0),     # fp32: a last tile of one row
    (1, 8, 8, 4100, 64, 3000, "f32", -0.5),
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


@pytest.mark.parametrize("keep", [False, True])
@pytest.mark.parametrize("kind", ["plain", "rising", "heavy"])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu", SHAPES)
def test_erased_bands(g, oracle, B, H, Hkv, N, d, w, dtype, mu, kind, keep):
    if keep and (dtype == "f32" or d == 64):
        pytest.skip("no larger workspace here")
    note("erased bands", B, H, Hkv, N, d, w, dtype, mu, kind, keep)
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, mu, kind)
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    out = step(g, wl, ins, dev(c32, "f32"), keep)
    b, kv = B - 1, Hkv - 1   # the last group of query heads
    hs = slice(kv * (H // Hkv), H)
    pick = lambda x, s: x[b:b + 1, s]
    Q, dO, c = pick(ins["Q"], hs), pick(ins["dO"], hs), pick(c32, hs)
    K, V = pick(ins["K"], slice(kv, kv + 1)), pick(ins["V"], slice(kv, kv + 1))
    got = {k: pick(host(x), slice(kv, kv + 1) if k in ("dK", "dV") else hs) for k, x in out.items()}
    O_ref, L_ref = oracle.forward_gqa_from_c(Q, K, V, c, w, wl.scale)
    # (of a "rising" prefix the span is the largest difference of either sign)
    par.LAST["c_span"] = max(par.window_span(c, w), float(np.abs(c).max() - np.abs(c).min()) if kind == "rising" else 0.0)
    if dtype == "bf16":
        check_bf16_forward(got["O"].reshape(O_ref.shape), got["L"].reshape(L_ref.shape), O_ref, L_ref, tag=kind)
    else:
        assert rel_inf(got["O"].reshape(O_ref.shape), O_ref) <= 1e-5
    if kind == "heavy":
        # rows that see the key have all their weight there: its value comes out, and dV of the key is the sum of their dO
        seen = slice(N // 8 + 1, min(N, N // 8 + w))
        np.testing.assert_allclose(got["O"][0, 0, seen], np.broadcast_to(V[0, 0, N // 8], (seen.stop - seen.start, d)), atol=1e-6, rtol=0)
        want = dO[0, :, N // 8:seen.stop].astype(np.float64).sum(axis=(0, 1))
        err = np.linalg.norm(got["dV"][0, 0, N // 8] - want) / np.linalg.norm(want)
        assert err <= (1e-2 if dtype == "bf16" else 1e-5), err
        return
    ref = oracle.backward_gqa_from_c(Q, K, V, c, dO, w, wl.scale, O_saved=got["O"])
    check_grads({k: got[k].reshape(ref[k].shape) for k in ("dQ", "dK", "dV", "dalpha")}, ref, 1e-2 if dtype == "bf16" else 1e-5, kind)


@pytest.mark.parametrize("which", ["V", "dO"])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu", [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[7], SHAPES[8]])
def test_far_rows_that_outweigh_their_decay(g, oracle, B, H, Hkv, N, d, w, dtype, mu, which):
    # one row of 2^58 with small scores: a weight of 2^-58 and less still makes half of an output, so its block must not be left out where
    # blocks of ordinary rows are (from 2^-48 on)
    note("outweigh", which, B, H, Hkv, N, d, w, dtype, mu)
    wl, ins = inputs(B, H, Hkv, N, d, w, dtype, mu)
    for t in ("Q", "K"):
        ins[t] = gi.round_to_bf16(ins[t] * np.float32(0.25)) if dtype == "bf16" else ins[t] * np.float32(0.25)
    at = N // 8 if which == "V" else N - N // 8
    ins[which][:, :, at] *= np.float32(2.0 ** 58)
    c32 = oracle.gate_prefix(ins["alpha"]).astype(np.float32)
    out = step(g, wl, ins, dev(c32, "f32"), True)
    hs = slice(0, H // Hkv)
    Q, dO, c = (x[:1, hs] for x in (ins["Q"], ins["dO"], c32))
    K, V = ins["K"][:1, :1], ins["V"][:1, :1]
    O_ref, _ = oracle.forward_gqa_from_c(Q, K, V, c, w, wl.scale)
    if which == "V":
        got, want = host(out["O"])[:1, hs].reshape(O_ref.shape), O_ref
    else:
        got = host(out["dV"])[:1, :1]
        want = oracle.backward_gqa_from_c(Q, K, V, c, dO, w, wl.scale, O_saved=host(out["O"])[:1, hs])["dV"].reshape(got.shape)
    # every row against its own size: bf16 probabilities and outputs; the fp32 difference of gates up to 2^7 in an exponent (2^-24 2^7 1.44)
    err = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= (1e-2 if dtype == "bf16" else 5e-5), err.max()


@pytest.mark.parametrize("which,value", [("V", np.inf), ("K", np.nan), ("dO", np.nan), ("Q", np.inf)])
@pytest.mark.parametrize("B,H,Hkv,N,d,w,dtype,mu", [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[7]])
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


@pytest.mark.parametrize("B,H,N,d,w,dtype", [(2, 24, 2048, 128, 1400, "bf16"), (1, 4, 6146, 64, 4001, "bf16"), (1, 8, 2177, 128, 1600, "f32")])
def test_outputs_over_inputs(g, oracle, B, H, N, d, w, dtype):
    # outputs serve as scratch in front of the kernels, unless they lie over an input that is still read
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
            # the column sums of the last block of a band may be contracted differently, half an ulp each (2^-24 of 16 here), and
            # dalpha adds up thousands of them: a random walk of 1e-4 at most, of values up to 15
            assert rel_inf(host(got), host(want[k])) <= (2e-5 if k == "dalpha" else 1e-6), (name, k)
