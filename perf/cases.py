"""The workloads by which this library's speed is judged, through its public entry points.

A case is one call (or the few calls that belong together) as a training or evaluation program
makes them: attention forward, backward or both on contiguous [B, H, S, D] tensors or on views
of a fused, sequence-major QKV buffer; the QKV linear layer, forward, backward or both; and the
whole attention stage (linear layer, attention, and back).  Sizes are those of the workload table
in ``paper_2507_00394_amd.inputs``, of ``bench.py`` and of the tests, or lie between them.
"""
import math

import torch

from paper_2507_00394_amd import binding as hx

MAX_WORK = 14 * 128 * 32 * 131072 * 131073 // 2   # FLOPs of the largest listed case (fwd + bwd)
MAX_ELEMENTS = 32 * 131072 * 128                  # elements of one of its tensors


def listed():
    attn = dict(path="attn", passes="step", layout="contiguous", B=1, D=128, causal=True, k_mult=1.0)
    return [
        # smallest workload of the table: launches and latency count
        dict(attn, name="tiny_d64", H=2, S=512, D=64),
        # evaluation of a short prompt of no particular length, forward only
        dict(attn, name="short_ragged_fwd", passes="fwd", H=12, S=1500),
        # full (unmasked) attention at an odd length, small head dimension, several samples
        dict(attn, name="full_ragged_d64", B=3, H=9, S=777, D=64, causal=False),
        # backward alone (the forward ran earlier on the stage), short sequences in a micro batch of four
        dict(attn, name="micro_batches_bwd", passes="bwd", B=4, H=16, S=2048),
        # small head dimension at a long sequence
        dict(attn, name="long_d64", H=16, S=16384, D=64),
        # 1.3B layer at 16k tokens
        dict(attn, name="layer_1b_16k", H=16, S=16384),
        # 7B layer at 128k tokens: the headline workload
        dict(attn, name="layer_7b_128k", H=32, S=131072),
        # 13B-like layer shape with two micro batches and a sharpened softmax, at a ragged shorter length
        dict(attn, name="layer_13b_two_mb", B=2, H=40, S=8000, k_mult=2.0),
        # one GPU's share of the heads under 8-way sequence parallelism, views of the fused QKV buffer
        dict(attn, name="share_5_heads_32k", layout="fused", H=5, S=32768),
        # the whole attention stage of one GPU's share of a 1.3B layer: linear layer, attention, and back
        dict(name="stage_2_heads_32k", path="stage", B=1, H=2, S=32768, D=128, K=2048),
        # QKV linear layer, one GPU's share of a 7B layer at 128k tokens
        dict(name="linear_7b_128k", path="linear", passes="step", M=131072, K=4096, N=1536),
        # the same layer in a 1.3B model at few tokens
        dict(name="linear_1b_short", path="linear", passes="step", M=2080, K=2048, N=768),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any length from a few dozen tokens to 128k, 1 to 40 heads, both head
    dimensions, every layout and direction; a linear layer of 32 to 128k tokens."""
    while True:
        kind = rng.choice(["attn", "attn", "attn", "attn", "linear", "linear", "stage"])
        if kind == "attn":
            c = dict(path="attn", passes=rng.choice(["fwd", "bwd", "step", "step"]), layout=rng.choice(["contiguous", "contiguous", "fused"]),
                     B=rng.choice([1, 1, 2, 3, 4]), H=rng.randint(1, 40), S=_log_uniform(rng, 48, 131072), D=rng.choice([64, 128, 128]),
                     causal=rng.random() < 0.8, k_mult=rng.choice([1.0, 1.0, 2.0]))
            if rng.random() < 0.4:
                c["S"] = max(64, c["S"] // 64 * 64)
        elif kind == "linear":
            passes = rng.choice(["fwd", "bwd", "step"])
            M = _log_uniform(rng, 32, 131072)
            if passes != "fwd":
                M = max(32, M // 32 * 32)
            c = dict(path="linear", passes=passes, M=M, K=128 * _log_uniform(rng, 1, 40), N=128 * _log_uniform(rng, 1, 24))
        else:
            H = rng.choice([1, 2, 4, 5])
            c = dict(path="stage", B=1, H=H, S=32 * _log_uniform(rng, 4, 2048), D=128, K=rng.choice([1024, 2048, 4096, 5120]))
        biggest = c["M"] * max(c["K"], c["N"]) if kind == "linear" else c["B"] * c["H"] * c["S"] * c["D"]
        if work(c)["flops"] <= MAX_WORK and biggest <= MAX_ELEMENTS:
            return c


def _normal(gen, *shape, std=1.0):
    x = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    rows = x.view(-1)
    step = 1 << 28   # in pieces: the fp32 draw of a whole tensor would need twice its memory
    for i in range(0, rows.numel(), step):
        part = rows[i:i + step]
        part.copy_(torch.randn(part.numel(), generator=gen, device="cuda") * std)
    return x


def prepare(case, seed):
    """Inputs (iid normal, as in training at initialisation, rounded to bf16), output buffers and the workspace."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = {"case": case}
    bf16 = dict(dtype=torch.bfloat16, device="cuda")
    if case["path"] == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        st.update(a=_normal(gen, M, K), w=_normal(gen, K, N, std=0.02))
        if case["passes"] != "bwd":
            st.update(qkv=torch.empty(M, N, **bf16))
        if case["passes"] != "fwd":
            st.update(g=_normal(gen, M, N), da=torch.empty(M, K, **bf16), dw=torch.empty(K, N, dtype=torch.float32, device="cuda"),
                      ws=torch.empty(hx.helix_qkv_linear_bwd_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda"))
        return st
    B, H, S, D = (case[k] for k in "BHSD")
    st["scale"] = D ** -0.5
    st["lse"] = torch.empty(B, H, S, dtype=torch.float32, device="cuda")
    st["ws"] = torch.empty(hx.helix_attn_bwd_workspace_bytes(B, H, S, D), dtype=torch.uint8, device="cuda")
    if case["path"] == "stage" or case["layout"] == "fused":
        st["dqkv"] = torch.empty(S, B, 3, H, D, **bf16)
        st["o"] = torch.empty(S, B, H, D, **bf16)
        st["dO"] = _normal(gen, S, B, H, D)
        st["qkv"] = torch.empty(S, B, 3, H, D, **bf16)
        if case["path"] == "stage":
            M, K, N = S * B, case["K"], 3 * H * D
            st.update(a=_normal(gen, M, K), w=_normal(gen, K, N, std=0.02), da=torch.empty(M, K, **bf16),
                      dw=torch.empty(K, N, dtype=torch.float32, device="cuda"),
                      lws=torch.empty(hx.helix_qkv_linear_bwd_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda"))
        else:
            st["qkv"].copy_(_normal(gen, S, B, 3, H, D))
            st["qkv"][:, :, 1] *= case["k_mult"]
    else:
        for t in ("q", "k", "v", "dO"):
            st[t] = _normal(gen, B, H, S, D)
        st["k"] *= case["k_mult"]
        st["o"] = torch.empty(B, H, S, D, **bf16)
        for t in ("dq", "dk", "dv"):
            st[t] = torch.empty(B, H, S, D, **bf16)
    if case["path"] == "attn" and case["passes"] == "bwd":
        _attn_fwd(st)
    return st


def _head_major(t):
    return t.permute(1, 2, 0, 3)   # [S, B, H, D] -> logical [B, H, S, D]


def _attn_fwd(st):
    c = st["case"]
    if "qkv" in st:
        q, k, v = (_head_major(st["qkv"][:, :, i]) for i in range(3))
        hx.helix_attn_fwd_strided(q, k, v, _head_major(st["o"]), st["lse"], st["scale"], c.get("causal", True))
    else:
        hx.helix_attn_fwd(st["q"], st["k"], st["v"], st["o"], st["lse"], st["scale"], c["causal"])


def _attn_bwd(st):
    c = st["case"]
    if "qkv" in st:
        q, k, v = (_head_major(st["qkv"][:, :, i]) for i in range(3))
        dq, dk, dv = (_head_major(st["dqkv"][:, :, i]) for i in range(3))
        hx.helix_attn_bwd_strided(q, k, v, _head_major(st["o"]), st["lse"], _head_major(st["dO"]), dq, dk, dv, st["ws"], st["scale"],
                                  c.get("causal", True))
    else:
        hx.helix_attn_bwd(st["q"], st["k"], st["v"], st["o"], st["lse"], st["dO"], st["dq"], st["dk"], st["dv"], st["ws"], st["scale"],
                          c["causal"])


def run(st):
    """One pass; returns every output it writes."""
    c = st["case"]
    if c["path"] == "linear":
        out = []
        if c["passes"] != "bwd":
            hx.helix_qkv_linear_fwd(st["a"], st["w"], st["qkv"])
            out += [st["qkv"]]
        if c["passes"] != "fwd":
            hx.helix_qkv_linear_bwd(st["a"], st["w"], st["g"], st["da"], st["dw"], st["ws"])
            out += [st["da"], st["dw"]]
        return out
    if c["path"] == "stage":
        M, N = c["S"] * c["B"], 3 * c["H"] * c["D"]
        hx.helix_qkv_linear_fwd(st["a"], st["w"], st["qkv"].view(M, N))
        _attn_fwd(st)
        _attn_bwd(st)
        hx.helix_qkv_linear_bwd(st["a"], st["w"], st["dqkv"].view(M, N), st["da"], st["dw"], st["lws"])
        return [st[t] for t in ("qkv", "o", "lse", "dqkv", "da", "dw")]
    out = []
    if c["passes"] != "bwd":
        _attn_fwd(st)
        out += [st["o"], st["lse"]]
    if c["passes"] != "fwd":
        _attn_bwd(st)
        out += [st["dqkv"]] if "qkv" in st else [st["dq"], st["dk"], st["dv"]]
    return out


def work(case):
    """Attention: 4*D FLOPs per unmasked pair forward, 10*D backward (with the score recomputation), bf16 tensors read and
    written once.  Linear layer: 2*M*K*N per product."""
    flops = nbytes = 0
    if case["path"] in ("linear", "stage"):
        M, K, N = (case["M"], case["K"], case["N"]) if case["path"] == "linear" else (case["S"] * case["B"], case["K"], 3 * case["H"] * case["D"])
        passes = case.get("passes", "step")
        if passes != "bwd":
            flops += 2 * M * K * N
            nbytes += 2 * (M * K + K * N + M * N)
        if passes != "fwd":
            flops += 4 * M * K * N
            nbytes += 2 * (M * K + K * N + M * N) + 2 * M * K + 4 * K * N
    if case["path"] in ("attn", "stage"):
        B, H, S, D = (case[k] for k in "BHSD")
        pairs = B * H * (S * (S + 1) // 2 if case.get("causal", True) else S * S)
        tensor, row = 2 * B * H * S * D, 4 * B * H * S
        passes = case.get("passes", "step")
        if passes != "bwd":
            flops += 4 * D * pairs
            nbytes += 4 * tensor + row
        if passes != "fwd":
            flops += 10 * D * pairs
            nbytes += 8 * tensor + row
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the outputs differ by from the same path in 64 bits.  Attention: P and dS are rounded to bf16 before
    the second product and the results once more, 2.4e-3 (2-norm); single values 0.08 of the root mean square, on causal rows and
    columns that few pairs contribute to.  The stage adds the rounding of qkv in front: 3.9e-3 and 0.12.  Linear layer: one
    rounding to bf16, 1.7e-3 and 2^-8 (dw is fp32 and far closer)."""
    if case["path"] == "linear":
        return {"rel": 6e-3, "max": 1.6e-2}
    if case["path"] == "stage":
        return {"rel": 1.5e-2, "max": 0.45}
    return {"rel": 1e-2, "max": 0.33}
