"""bf16 forward with few query tiles and long bands: the shapes of the split kernel on both sides of the lines between them."""
import numpy as np
import pytest

import gfwa_inputs as gi
import test_gpu_parity as par
from test_gpu_parity import check_bf16_forward, dev, host, note

pytestmark = pytest.mark.gpu
g = par.g


# 32, 64, 128 queries to a workgroup at d = 128 (32-query blocks: one and a half and two and a quarter to a CU of 256, odd heads), then d = 64
@pytest.mark.parametrize("B,H,N,d,w", [(1, 1, 2101, 128, 1801), (1, 3, 4065, 128, 1025), (1, 2, 6550, 128, 1700), (1, 2, 8000, 128, 1600),
                                       (1, 3, 6001, 128, 1501), (1, 6, 5990, 128, 1300), (1, 12, 2099, 128, 1800),
                                       (1, 12, 2900, 128, 2900), (1, 12, 3010, 128, 3010), (1, 12, 3010, 64, 3010),
                                       (1, 8, 3000, 64, 2400), (1, 8, 3001, 64, 2200)])
def test_forward_of_long_bands(g, oracle, B, H, N, d, w):
    note("long bands", B, H, N, d, w)
    wl = gi.custom("long", B, H, N, d, w, alpha_mu=-6.0, index=23)
    Q, K, V, alpha = (gi.make_tensor(wl, t) for t in ("Q", "K", "V", "alpha"))
    c32 = oracle.gate_prefix(alpha).astype(np.float32)
    O, L = g.gfwa_forward(dev(Q, "bf16"), dev(K, "bf16"), dev(V, "bf16"), dev(c32, "f32"), w, wl.scale)
    last = lambda x: np.ascontiguousarray(x[-1:, -1:])
    O_ref, L_ref = oracle.forward_gqa_from_c(last(Q), last(K), last(V), last(c32), w, wl.scale)
    par.LAST["c_span"] = par.window_span(c32, w)
    check_bf16_forward(last(host(O)).reshape(O_ref.shape), last(host(L)).reshape(L_ref.shape), O_ref, L_ref, tag="long")
