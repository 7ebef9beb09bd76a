"""Timed cases of the library's hot path, through the Python binding's public calls.

A case is a dict of plain values; ``kind`` says which calls one pass makes:

prefill   ``prefill``: Taylor linear attention over whole sequences, output and final state
swa       ``swa_prefill``: sliding-window attention over whole sequences, output and decode ring
decode    ``decode_fused``: one token of both mixers on their state and ring (device positions: plus
          ``positions_advance``, as a serving loop issues it)
project   ``project_qkv`` and ``project_out``: the projections around a linear-attention layer
gate      ``short_conv_gate``: the gate of a convolution layer, with the state rows for the next call

Values are the ones the repository's workloads draw: N(0, 1) * 0.5 for attention inputs, unit-variance
activations and N(0, 1) / sqrt(K) weights for the projections.
"""
import math

import torch

from paper_2402_18668_amd import based

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
_SIZE = {"bf16": 2, "f32": 4}
_CODE = {"bf16": based.BF16, "f32": based.F32}

# ceilings of a drawn case, each the figure of a listed one
_PREFILL_MFMA = {16: 16 * 16 * 2048 * 128, 32: 2 * 16 * 16384 * 64}   # token-heads x d_v (bf16)
_PREFILL_ROWS = 8 * 16 * 2048 * 273 * 64                              # token-heads x D x d_v (the others)
_SWA = 16 * 16 * 2048 * 128                                           # token-heads x d_h
_DECODE_BYTES = 128 * 16 * (273 * 128 + 273) * 4
_GATE = 16 * 2048 * 7168


def _prefill(name, B, N, d_feat, d_v, dtype="bf16", init=False, packed=False, H=16):
    return {"name": name, "kind": "prefill", "B": B, "H": H, "N": N, "d_feat": d_feat, "d_v": d_v,
            "dtype": dtype, "init": init, "packed": packed}


def _swa(name, B, N, d_h, w, dtype="bf16", rotary=False, H=16):
    return {"name": name, "kind": "swa", "B": B, "H": H, "N": N, "d_h": d_h, "w": w, "dtype": dtype,
            "rotary": rotary}


def _decode(name, B, d_feat, d_v, d_h, w, dtype="bf16", packed=False, rotary=False, device_pos=False, H=16):
    return {"name": name, "kind": "decode", "B": B, "H": H, "d_feat": d_feat, "d_v": d_v, "d_h": d_h, "w": w,
            "dtype": dtype, "packed": packed, "rotary": rotary, "device_pos": device_pos}


def _project(name, B, N, d_model, d_feat, d_v, H=16):
    return {"name": name, "kind": "project", "B": B, "N": N, "d_model": d_model, "H": H, "d_feat": d_feat,
            "d_v": d_v, "dtype": "bf16"}


def _gate(name, B, N, Dc, dtype="bf16"):
    return {"name": name, "kind": "gate", "B": B, "N": N, "Dc": Dc, "dtype": dtype}


def listed():
    return [
        # prompt processing of the 1.3B-shaped layer, a full batch: the benchmark's headline shape
        _prefill("prefill_1p3b", 16, 2048, 16, 128),
        # the same of the 360M-shaped layer: fewer, narrower heads than the chip has room for
        _prefill("prefill_360m", 8, 2048, 16, 64),
        # few long sequences with the larger feature dimension
        _prefill("prefill_long", 2, 16384, 32, 64),
        # one user's prompt of an odd length, continuing a conversation's state: latency
        _prefill("prefill_prompt", 1, 777, 16, 64, init=True),
        # the 360M-shaped layer in fp32: evaluation at full precision
        _prefill("prefill_f32", 8, 2048, 16, 64, dtype="f32"),
        # window layer of the 1.3B-shaped model, a full batch
        _swa("swa_1p3b", 16, 2048, 128, 64),
        # window layer over long sequences, with the positional encoding these layers are trained with
        _swa("swa_long_rotary", 2, 16384, 64, 128, rotary=True),
        # one token for one user of the 360M-shaped model, as a serving loop does it: latency
        _decode("decode_one", 1, 16, 64, 64, 64, packed=True, rotary=True, device_pos=True),
        # one token for a large batch of the 1.3B-shaped model (a model has many layers: state out of cache)
        _decode("decode_1p3b", 128, 16, 128, 128, 64),
        # projections of the 1.3B-shaped layer, a full batch of prompts
        _project("project_1p3b", 16, 2048, 1792, 16, 128),
        # the same for one decoded token of a few sequences: an odd handful of rows against all the weights
        _project("project_decode", 9, 1, 1792, 16, 128),
        # convolution layer of the 1.3B-shaped model
        _gate("gate_1p3b", 16, 2048, 7168),
    ]


def _pairs(d_feat):
    """Distinct features of the map: one row per unordered pair."""
    return 1 + d_feat + d_feat * (d_feat + 1) // 2


def _log_int(rng, lo, hi):
    """An integer of lo .. hi, even over the logarithm."""
    hi = max(lo, hi)
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["prefill"] * 6 + ["swa"] * 4 + ["decode"] * 5 + ["project"] * 3 + ["gate"] * 2)
    H = rng.choice([8, 12, 16, 16, 16, 20, 32])
    if kind == "prefill":
        d_v = rng.choice([64, 128])
        d_feat = rng.choice([16] * 5 + [32] * 3 + [8, 24])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        matrix = dtype == "bf16" and d_feat in (16, 32)
        if matrix:
            most = _PREFILL_MFMA[d_feat] // d_v
        else:
            most = _PREFILL_ROWS // (based.feature_dim(d_feat) * d_v)
        B = _log_int(rng, 1, 32)
        N = _log_int(rng, 16, min(16384, most // (B * H)))
        c = _prefill("", B, N, d_feat, d_v, dtype, init=rng.random() < 0.3, packed=matrix and rng.random() < 0.3, H=H)
    elif kind == "swa":
        d_h, w = rng.choice([64, 128]), rng.choice([16, 32, 64, 64, 128])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        B = _log_int(rng, 1, 32)
        N = _log_int(rng, 16, min(16384, _SWA // (d_h * B * H * (8 if dtype == "f32" else 1))))
        c = _swa("", B, N, d_h, w, dtype, rotary=rng.random() < 0.5, H=H)
    elif kind == "decode":
        d = rng.choice([64, 128])
        d_feat = rng.choice([16, 16, 16, 32])
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        per = H * based.state_stride_floats(d_feat, d) * 4
        device_pos = rng.random() < 0.5
        c = _decode("", _log_int(rng, 1, min(128, _DECODE_BYTES // per)), d_feat, d, d, rng.choice([16, 64, 64, 128]),
                    dtype, packed=rng.random() < 0.5, rotary=device_pos and rng.random() < 0.7, device_pos=device_pos,
                    H=H)
    elif kind == "project":
        d_feat, d_v = rng.choice([(16, 64), (16, 128), (32, 64), (32, 128)])
        if rng.random() < 0.4:
            B, N = _log_int(rng, 1, 128), 1
        else:
            B = _log_int(rng, 1, 16)
            N = _log_int(rng, 16, 2048)
        c = _project("", B, N, 128 * rng.randint(4, 14), d_feat, d_v, H=rng.choice([8, 12, 16, 16]))
    else:
        Dc = 8 * rng.randint(64, 896)
        B = _log_int(rng, 1, 32)
        N = 1 if rng.random() < 0.25 else _log_int(rng, 16, min(16384, _GATE // (B * Dc)))
        c = _gate("", B, N, Dc, "f32" if N * B * Dc < _GATE // 2 and rng.random() < 0.15 else "bf16")
    del c["name"]
    return c


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = _TORCH[case["dtype"]]
    kind, B = case["kind"], case["B"]

    def normal(*shape, scale=0.5, dtype=dt):
        return torch.randn(shape, generator=g, device="cuda").mul_(scale).to(dtype)

    s = {"case": dict(case)}
    if kind == "prefill":
        H, N, dp, dv = case["H"], case["N"], case["d_feat"], case["d_v"]
        s["q"], s["k"], s["v"] = normal(B, H, N, dp), normal(B, H, N, dp), normal(B, H, N, dv)
        s["state"] = based.alloc_packed_state(B, H, dp, dv) if case["packed"] else based.alloc_state(B, H, dp, dv)
        if case["init"]:   # the state of the 64 tokens before
            based.prefill(normal(B, H, 64, dp), normal(B, H, 64, dp), normal(B, H, 64, dv), state=s["state"],
                          packed=case["packed"])
        s["workspace"] = based.alloc_prefill_workspace(B, H, N, dp, dv, _CODE[case["dtype"]])
    elif kind == "swa":
        H, N, dh, w = case["H"], case["N"], case["d_h"], case["w"]
        s["q"], s["k"], s["v"] = normal(B, H, N, dh), normal(B, H, N, dh), normal(B, H, N, dh)
        s["ring"] = based.alloc_swa_ring(B, H, w, dh, dt)
        s["table"] = based.rotary_table(N, dh) if case["rotary"] else None
    elif kind == "decode":
        H, dp, dv, dh, w = case["H"], case["d_feat"], case["d_v"], case["d_h"], case["w"]
        state = based.alloc_state(B, H, dp, dv)
        based.prefill(normal(B, H, 64, dp), normal(B, H, 64, dp), normal(B, H, 64, dv), state=state)
        if case["packed"]:
            state = based.state_pack(state, based.alloc_packed_state(B, H, dp, dv), B, H, dp, dv)
        s["state"] = state
        s["ring"] = normal(B, H, 2, w, dh)
        s["token"] = [normal(B, H, dp), normal(B, H, dp), normal(B, H, dv)]
        s["window"] = [normal(B, H, dh), normal(B, H, dh), normal(B, H, dh)]
        s["table"] = based.rotary_table(32768, dh) if case["rotary"] else None
        if case["device_pos"]:   # sequences of different lengths
            s["pos"] = torch.randint(w, 1024, (B,), generator=g, device="cuda", dtype=torch.int32)
        else:
            s["pos"] = 512
    elif kind == "project":
        H, N, dm, dp, dv = case["H"], case["N"], case["d_model"], case["d_feat"], case["d_v"]
        s["x"] = normal(B, N, dm, scale=1.0)
        s["W"] = normal(H * (2 * dp + dv), dm, scale=dm ** -0.5)
        s["y"] = normal(B, H, N, dv)
        s["Wo"] = normal(dm, H * dv, scale=(H * dv) ** -0.5)
    else:
        N, Dc = case["N"], case["Dc"]
        s["a"], s["c"] = normal(B, N, Dc, scale=1.0), normal(B, N, Dc, scale=1.0)
        s["h"] = normal(3, Dc, scale=3 ** -0.5, dtype=torch.float32)
        s["b1"], s["b2"] = (normal(Dc, scale=0.1, dtype=torch.float32) for _ in range(2))
        s["prev"] = normal(B, 2, Dc, scale=1.0)
        s["last"] = torch.empty_like(s["prev"])
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "prefill":
        y = based.prefill(s["q"], s["k"], s["v"], state=s["state"], has_init=c["init"], workspace=s["workspace"],
                          packed=c["packed"])
        return y, s["state"]
    if kind == "swa":
        y = based.swa_prefill(s["q"], s["k"], s["v"], c["w"], c["d_h"] ** -0.5, ring=s["ring"], rotary=s["table"])
        return y, s["ring"]
    if kind == "decode":
        if not c["device_pos"]:
            s["pos"] += 1
        (q, k, v), (wq, wk, wv) = s["token"], s["window"]
        y_lin, y_swa = based.decode_fused(q, k, v, s["state"], wq, wk, wv, s["ring"], s["pos"], c["w"],
                                          c["d_h"] ** -0.5, packed=c["packed"], rotary=s["table"])
        if c["device_pos"]:
            based.positions_advance(s["pos"])
        return y_lin, y_swa, s["state"], s["ring"]
    if kind == "project":
        q, k, v = based.project_qkv(s["x"], s["W"], c["H"], c["d_feat"], c["d_v"])
        return q, k, v, based.project_out(s["y"], s["Wo"])
    out = based.short_conv_gate(s["a"], s["c"], s["h"], s["b1"], s["b2"], c_prev=s["prev"], c_last=s["last"])
    return out, s["last"]


def work(case):
    kind, B, e = case["kind"], case["B"], _SIZE[case["dtype"]]
    if kind == "prefill":
        U, N, dp, dv = B * case["H"], case["N"], case["d_feat"], case["d_v"]
        rows = _pairs(dp) if case["packed"] else based.feature_dim(dp)
        sym = _pairs(dp)                    # what readout and update cannot do without
        C = min(64, N)                      # tokens of a chunk's masked quadratic block
        return {"bytes": U * N * (2 * dp + 2 * dv) * e + U * rows * (dv + 1) * 4 * (2 if case["init"] else 1),
                "flops": U * N * (4 * sym * (dv + 1) + (C + 1) * (dp + dv + 1))}
    if kind == "swa":
        U, N, dh, w = B * case["H"], case["N"], case["d_h"], case["w"]
        pairs = N * w - w * (w - 1) // 2 if N >= w else N * (N + 1) // 2
        return {"bytes": U * (4 * N + 2 * min(N, w)) * dh * e + (N * dh * 4 if case["rotary"] else 0),
                "flops": U * pairs * 4 * dh}
    if kind == "decode":
        U, dp, dv, dh, w = B * case["H"], case["d_feat"], case["d_v"], case["d_h"], case["w"]
        rows = _pairs(dp) if case["packed"] else based.feature_dim(dp)
        return {"bytes": U * (rows * (dv + 1) * 8 + (2 * dp + 2 * dv + 4 * dh + 2 * (w + 1) * dh) * e),
                "flops": U * (4 * rows * (dv + 1) + 4 * w * dh)}
    if kind == "project":
        M, dm, H, dp, dv = B * case["N"], case["d_model"], case["H"], case["d_feat"], case["d_v"]
        n = H * (2 * dp + dv)
        return {"bytes": (M * (2 * dm + n + H * dv) + dm * (n + H * dv)) * e, "flops": 2 * M * dm * (n + H * dv)}
    n = B * case["N"] * case["Dc"]
    return {"bytes": 3 * n * e + 5 * case["Dc"] * 4 + 4 * B * case["Dc"] * e, "flops": 12 * n}


def tolerance(case):
    # fp32 throughout: sums of a few thousand terms that partly cancel
    return {"rel": 2e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
