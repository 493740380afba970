"""Gate scans of rows of a few chunks of 4096: segments that add up the row before them by themselves, at the edges of their range."""
import numpy as np
import pytest
import torch

import gfwa_inputs as gi
import test_gpu_parity as par
from test_gpu_parity import GATE_EPS, check_grads, dev, host, note

pytestmark = pytest.mark.gpu
g = par.g


# rows, N: three chunks, the last of one element; as many segments as there are; a workgroup on every CU, and one more row (no segments
# there); with the activation three quarters of that
@pytest.mark.parametrize("rows,N", [(1, 8193), (2, 12288), (3, 65536), (3, 65537), (85, 12285), (86, 12285), (48, 16383), (49, 16383)])
@pytest.mark.parametrize("act", [False, True])
def test_prefix_of_rows_in_segments(g, oracle, rows, N, act):
    note("rows in segments", rows, N, act)
    wl = gi.custom("seg", 1, rows, N, 64, 8, alpha_mu=-1.0, index=21)
    if act:
        h, beta = gi.make_gate_inputs(wl)
        alpha = oracle.gate_activation(h, beta, GATE_EPS)
        x, b = dev(h, "f32"), dev(beta, "f32")
        calls = [lambda: g.gfwa_gate_activation_prefix(x, b, GATE_EPS), lambda: g.gfwa_gate_prefix_stp(x, b, GATE_EPS)]
    else:
        alpha = gi.make_tensor(wl, "alpha")
        x = dev(alpha, "f32")
        calls = [lambda: g.gfwa_gate_prefix(x), lambda: g.gfwa_gate_prefix_stp(x)]
    ref = oracle.gate_prefix(alpha)
    for call in calls:  # the bars of the one-pass scans
        assert np.abs(host(call()) - ref).max() <= (8 if act else 4) * np.finfo(np.float32).eps * ref.max()


@pytest.mark.parametrize("B,H,N,d,w,dtype", [(1, 2, 8193, 64, 24, "bf16"), (1, 3, 12291, 64, 8, "f32"), (1, 1, 32768, 128, 5, "bf16"),
                                             (1, 1, 32769, 64, 5, "bf16")])
def test_gate_gradient_of_rows_in_segments(g, oracle, B, H, N, d, w, dtype):
    note("gate gradient in segments", B, H, N, d, w, dtype)
    wl = gi.custom("seg", B, H, N, d, w, dtype, alpha_mu=-1.0, index=22, backward=True)
    got, ref = par.run_backward(g, oracle, wl)
    check_grads(got, ref, 1e-2 if dtype == "bf16" else 1e-5, "segments")


@pytest.mark.parametrize("act", [False, True])
def test_prefix_over_its_input(g, act):
    x = torch.rand(1, 7, 13000, device=par.DEV)
    b = torch.rand_like(x) + 0.5
    call = (lambda x, c=None: g.gfwa_gate_activation_prefix(x, b, GATE_EPS, c)) if act else (lambda x, c=None: g.gfwa_gate_prefix(x, c))
    want = call(x)
    over = x.clone()
    got = call(over, over)
    assert (got - want).abs().max() <= 4e-7 * want.max()


@pytest.mark.parametrize("rows,N", [(64, 8192), (100, 20000), (32, 16384), (300, 12288)])
def test_chunks_in_front_are_summed_up_by_fours(g, rows, N):
    # scan-then-propagate starts a chunk of 4096 from the sum of those in front, fp32 over four elements and fp64 across, however many launches it
    # takes: its first element is that sum plus one, rounded once (1000 rows of which a workgroup takes two chunks may do otherwise)
    note("sums by fours", rows, N)
    alpha = torch.nn.functional.softplus(torch.randn((1, rows, N), generator=torch.Generator(device=par.DEV).manual_seed(5), device=par.DEV) - 1)
    c = g.gfwa_gate_prefix_stp(alpha)
    a = alpha[0].cpu()
    fours = a[:, :4096].reshape(rows, -1, 4)
    front = ((fours[..., 0] + fours[..., 1]) + (fours[..., 2] + fours[..., 3])).double().sum(-1)
    assert torch.equal(c[0, :, 4096].cpu(), (front + a[:, 4096].double()).float())
