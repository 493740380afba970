"""The work a user of this library has it do, as cases that a timing program can run.

Four kinds of work, all through the public functions of `paper_2512_07782_amd`:
  prefill  gate preprocessing and the forward of a whole sequence (scoring, prompt processing)
  train    the same, then the backward down to the gate's inputs (one attention layer of a training step)
  decode   one generated token for every sequence of a batch, against the key/value cache
  gates    the gate preprocessing and its derivative alone, on few very long rows

Keys of a case, beside its name:
  kind; B, H, Hkv (query heads, key/value heads), N (sequence length; cache length in `decode`), d, w (window)
  dtype    storage type of the matrices, "bf16" or "f32"
  mu       the gate is softplus(N(mu, 1)); -3 forgets slowly, -1 fast
  act      the gate comes as pre-activation h and amplitude beta (the model's own projection), not as alpha
  stp      scan-then-propagate preprocessing with a workspace that the program keeps
  keep     train: the program keeps the large backward workspace; otherwise the binding allocates the minimum
  static   decode: outputs and scratch are there before the call (gfwa_decode_static)
"""
import math

import torch

import paper_2512_07782_amd as g

DEV = "cuda"
GATE_EPS = 1e-6
TORCH_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}

# What a drawn case may cost at most: the largest listed one of its kind.
MAX_ELEMENTS = 32 * 16384 * 128          # one matrix [B,H,N,d]
MAX_PRODUCTS = {"bf16": 32 * 16384 * 1024 * 128, "f32": 2 * 16 * 4096 * 1024 * 128}  # B H N min(w, N) d
MAX_CACHE = 64 * 8 * 16384 * 128         # one cache [B,Hkv,T,d]
MAX_WINDOWS = 64 * 32 * 1024 * 128       # B H min(w, T) d of a decoding step
MAX_GATES = 16 * 64 * 65536              # one gate tensor [B,H,N]


def _case(kind, B, H, Hkv, N, d, w, dtype="bf16", mu=-2.0, act=False, stp=False, keep=False, static=False, **name):
    return dict(kind=kind, B=B, H=H, Hkv=Hkv, N=N, d=d, w=w, dtype=dtype, mu=mu, act=act, stp=stp, keep=keep, static=static, **name)


def listed():
    return [
        # the smallest call there is: one head, one launch's worth of work, fp32 as a numerics check would run it
        _case("prefill", 1, 1, 1, 256, 64, 64, "f32", mu=0.0, name="tiny_fwd_f32"),
        # a prompt shorter than its window, batch one, grouped heads, gate from the model's projection: serving latency
        _case("prefill", 1, 32, 8, 700, 128, 1024, mu=-2.0, act=True, name="short_prompt"),
        # a fine-tuning step on short ragged sequences
        _case("train", 2, 8, 2, 515, 64, 512, mu=-2.0, act=True, keep=True, name="short_train"),
        # scoring with the language-model shape (64-wide heads, window 512)
        _case("prefill", 4, 16, 16, 4096, 64, 512, mu=-2.0, name="lm_fwd"),
        # a training step of that shape with 4 query heads per key/value head, from the pre-activation
        _case("train", 4, 16, 4, 4096, 64, 512, mu=-2.0, act=True, name="lm_gqa_train"),
        # a sequence that is no multiple of any tile with a window longer than half of it, few heads
        _case("train", 1, 8, 8, 5003, 128, 3000, mu=-1.5, keep=True, name="ragged_train"),
        # the training shape with the workspace the binding allocates by itself
        _case("train", 4, 16, 16, 8192, 128, 1024, mu=-2.0, name="train_bwd"),
        # the benchmark's shape: long sequence, 128-wide heads, the large workspace kept from step to step
        _case("train", 1, 32, 32, 16384, 128, 1024, mu=-3.0, stp=True, keep=True, name="long_train"),
        # fp32 storage at a size that fills the chip
        _case("train", 2, 16, 16, 4096, 128, 1024, "f32", mu=-2.0, name="mid_train_f32"),
        # one conversation: a token's latency, everything allocated beforehand
        _case("decode", 1, 32, 8, 16384, 128, 1024, mu=-2.0, static=True, name="decode_one"),
        # a serving batch of sequences of different lengths
        _case("decode", 64, 32, 8, 16384, 128, 1024, mu=-2.0, name="decode_batch"),
        # gate preprocessing and its derivative on few very long rows
        _case("gates", 1, 8, 8, 262144, 64, 1024, mu=-1.0, act=True, stp=True, name="gates_long"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the range the listed ones span, evenly in their logarithm."""
    kind = rng.choice(["prefill", "prefill", "train", "train", "train", "decode", "decode", "gates"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    group = rng.choice([1, 1, 2, 4])
    Hkv = _log_int(rng, 1, 16)
    H = group * Hkv
    d = rng.choice([64, 128])
    mu = rng.choice([-3.0, -2.0, -1.0])
    act = rng.random() < 0.5
    if kind == "gates":
        while True:
            B, H, N = _log_int(rng, 1, 16), _log_int(rng, 1, 64), _log_int(rng, 64, 262144)
            if B * H * N <= MAX_GATES:
                return _case(kind, B, H, H, N, 64, 1024, mu=mu, act=act, stp=_few_long_rows(B * H, N))
    if kind == "decode":
        while True:
            B, T, w = _log_int(rng, 1, 256), _log_int(rng, 64, 16384), _log_int(rng, 32, 4096)
            if B * Hkv * T * d <= MAX_CACHE and B * H * min(w, T) * d <= MAX_WINDOWS:
                # (the library's own scratch holds 32 MiB: a program with more uses the call with a workspace)
                small = B * H * math.ceil(min(w, T) / 256) * (d + 2) * 4 <= 32 << 20
                return _case(kind, B, H, Hkv, T, d, w, dtype, mu=mu, static=small and rng.random() < 0.3)
    while True:
        B, N, w = _log_int(rng, 1, 8), _log_int(rng, 64, 16384), _log_int(rng, 32, 4096)
        if B * H * N * d <= MAX_ELEMENTS and B * H * N * min(w, N) * d <= MAX_PRODUCTS[dtype]:
            return _case(kind, B, H, Hkv, N, d, w, dtype, mu=mu, act=act, stp=_few_long_rows(B * H, N),
                         keep=kind == "train" and rng.random() < 0.5)


def _few_long_rows(rows, N):
    """When a program takes the segmented preprocessing (as bench.py does)."""
    return rows < 256 and N >= 8192


def prepare(case, seed):
    B, H, Hkv, N, d, w = (case[k] for k in ("B", "H", "Hkv", "N", "d", "w"))
    dt = TORCH_DTYPE[case["dtype"]]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*shape, dtype=dt):
        return torch.randn(shape, generator=gen, device=DEV, dtype=dtype)

    s = dict(case)
    s["scale"] = 1.0 / math.sqrt(d)
    if case["kind"] != "decode":
        if case["act"]:
            s["h"] = normal(B, H, N, dtype=torch.float32) + case["mu"]
            s["beta"] = torch.exp(0.5 * normal(B, H, N, dtype=torch.float32))
        else:
            s["alpha"] = torch.nn.functional.softplus(normal(B, H, N, dtype=torch.float32) + case["mu"])
        s["scan_ws"] = None
        if case["stp"]:
            s["scan_ws"] = torch.empty(g.gfwa_gate_scan_workspace_bytes(B, H, N), dtype=torch.uint8, device=DEV)
    if case["kind"] == "gates":
        s["dalpha"] = normal(B, H, N, dtype=torch.float32)
        return s
    if case["kind"] == "decode":
        s["q"] = normal(B, H, d)
        s["Kc"], s["Vc"] = normal(B, Hkv, N, d), normal(B, Hkv, N, d)
        alpha = torch.nn.functional.softplus(normal(B, H, N, dtype=torch.float32) + case["mu"])
        s["c"] = g.gfwa_gate_prefix(alpha)
        s["alpha_t"] = alpha[:, :, 0].contiguous()
        s["pos"] = torch.randint(N // 4, N, (B,), generator=gen, device=DEV, dtype=torch.int32)
        if case["static"]:
            s["o"] = torch.empty_like(s["q"])
            s["L"] = torch.empty((B, H), dtype=torch.float32, device=DEV)
        else:
            s["workspace"] = torch.empty(g.gfwa_decode_workspace_bytes(B, H, N, d, w), dtype=torch.uint8, device=DEV)
        return s
    s["Q"], s["K"], s["V"] = normal(B, H, N, d), normal(B, Hkv, N, d), normal(B, Hkv, N, d)
    if case["kind"] == "train":
        s["dO"] = normal(B, H, N, d)
        s["workspace"] = None
        if case["keep"]:
            s["workspace"] = torch.empty(g.gfwa_backward_fast_workspace_bytes(dt, B, H, N, d, w), dtype=torch.uint8,
                                         device=DEV)
    return s


def _gate_prefix(s):
    if s["stp"]:
        if s["act"]:
            return g.gfwa_gate_prefix_stp(s["h"], s["beta"], GATE_EPS, workspace=s["scan_ws"])
        return g.gfwa_gate_prefix_stp(s["alpha"], workspace=s["scan_ws"])
    if s["act"]:
        return g.gfwa_gate_activation_prefix(s["h"], s["beta"], GATE_EPS)
    return g.gfwa_gate_prefix(s["alpha"])


def run(s):
    if s["kind"] == "decode":
        if s["static"]:
            o, L = g.gfwa_decode_static(s["q"], s["Kc"], s["Vc"], s["c"], s["pos"], s["w"], s["scale"], s["o"], s["L"],
                                        alpha_t=s["alpha_t"])
        else:
            o, L = g.gfwa_decode(s["q"], s["Kc"], s["Vc"], s["c"], s["pos"], s["w"], s["scale"], alpha_t=s["alpha_t"],
                                 workspace=s["workspace"])
        return {"o": o, "L": L, "c": s["c"]}
    c = _gate_prefix(s)
    if s["kind"] == "gates":
        if not s["act"]:
            return {"c": c}
        dh, dbeta = g.gfwa_gate_activation_backward(s["h"], s["beta"], GATE_EPS, s["dalpha"])
        return {"c": c, "dh": dh, "dbeta": dbeta}
    grouped = s["Hkv"] != s["H"]
    forward = g.gfwa_forward_gqa if grouped else g.gfwa_forward
    O, L = forward(s["Q"], s["K"], s["V"], c, s["w"], s["scale"])
    out = {"c": c, "O": O, "L": L}
    if s["kind"] == "train":
        backward = g.gfwa_backward_gqa if grouped else g.gfwa_backward
        dQ, dK, dV, dalpha = backward(s["Q"], s["K"], s["V"], O, s["dO"], c, L, s["w"], s["scale"],
                                      workspace=s["workspace"])
        out.update(dQ=dQ, dK=dK, dV=dV, dalpha=dalpha)
        if s["act"]:
            out["dh"], out["dbeta"] = g.gfwa_gate_activation_backward(s["h"], s["beta"], GATE_EPS, dalpha)
    return out


def work(case):
    """Every input read once, every output written once; products counted inside the window only."""
    B, H, Hkv, N, d, w = (case[k] for k in ("B", "H", "Hkv", "N", "d", "w"))
    size = 2 if case["dtype"] == "bf16" else 4
    gate = 4 * B * H * N
    inputs = 2 if case["act"] else 1
    if case["kind"] == "gates":
        return {"bytes": gate * (inputs + 1 + (3 if case["act"] else 0)), "flops": 0}
    if case["kind"] == "decode":
        lo = N // 4  # positions are drawn from lo .. N - 1
        keys = sum(min(w, p + 1) for p in range(lo, N)) / (N - lo)
        return {"bytes": B * keys * (2 * Hkv * d * size + 4 * H) + 2 * B * H * d * size + 8 * B * H,
                "flops": 4 * B * H * keys * d}
    wn = min(w, N)
    pairs = B * H * (N * wn - wn * (wn - 1) // 2)
    q_matrix, kv_matrix = B * H * N * d * size, B * Hkv * N * d * size
    if case["kind"] == "prefill":  # Q, K, V, gate in; c, O, L out
        return {"bytes": 2 * q_matrix + 2 * kv_matrix + gate * (inputs + 2), "flops": 4 * pairs * d}
    # Q, K, V, dO, gate in; c, O, L, dQ, dK, dV, dalpha (dh, dbeta) out
    return {"bytes": 4 * q_matrix + 4 * kv_matrix + gate * (inputs + 3 + (2 if case["act"] else 0)),
            "flops": 14 * pairs * d}


def tolerance(case):
    # probabilities and dS are rounded to bf16 between the two products, as are the outputs; fp32 sums otherwise
    if case["dtype"] == "bf16" and case["kind"] != "gates":
        return {"rel": 1e-2}
    return {"rel": 1e-5}
