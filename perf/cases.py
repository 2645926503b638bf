"""The decode-time work of one transformer layer on a hybrid cache, as cases that can be timed and compared.

A case is one call (or the two calls of a paged decode step) through ``paper_2501_01792_amd.binding``, on inputs with the
scales of the repository's recipe (``synth.py``), drawn on the GPU.  The layers are those of ``synth.CONFIGS``.  What a
serving loop keeps between steps (weights, the prepared layer, workspaces, block tables, output buffers) is kept in the
state; everything else happens in ``run``.

Paths
  step     hybrid_decode_attn: K/V of the checkpointed tokens regenerated, attention over cached ++ regenerated tokens
  absorbed hybrid_decode_attn_absorbed: the same step without regenerating K/V
  regen    regen_kv: regeneration alone, written behind the cached rows of a K/V cache
  qkv      qkv_current: Q, K, V of the current tokens, K/V written to the cache
  paged    paged_decode_attn on a block table: ragged requests, 16-token blocks, KV and checkpoint blocks mixed
  serve    qkv_current_paged, then paged_decode_attn without regeneration on the query it returned: a serving loop's step
"""
import ctypes
import math

import numpy as np
import torch

from paper_2501_01792_amd import binding as hk, synth

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest call: the contract's tiny layer, bound by launches and latency.
        _case("step_tiny", "step", "tiny", B=4, L_kv=128, L_act=128),
        # An ordinary batch of the 6.7B-shaped layer, half of the context cached.
        _case("step_6.7b", "step", "opt6.7b", B=32, L_kv=512, L_act=512),
        # bf16, a few requests of an odd length: tiles and ranges do not come out even.
        _case("step_13b_bf16_odd", "step", "opt13b", dtype="bf16", B=7, L_kv=383, L_act=1148),
        # The largest: the benchmark's own workload, every context token regenerated.
        _case("step_66b", "step", "opt66b", B=64, L_kv=0, L_act=4096),
        # One request, everything cached: the latency of plain decode attention.
        _case("cached_6.7b_one", "step", "opt6.7b", B=1, L_kv=1999, L_act=0),
        # The step without regeneration, ordinary and large.
        _case("absorbed_6.7b", "absorbed", "opt6.7b", B=32, L_kv=512, L_act=512),
        _case("absorbed_66b", "absorbed", "opt66b", B=64, L_kv=2048, L_act=2048),
        # Three requests that come back to a GPU: their checkpoints become K/V rows of a cache.
        _case("regen_6.7b_bf16_few", "regen", "opt6.7b", dtype="bf16", B=3, L_kv=16, L_act=517),
        # Q, K, V of the current tokens: a batch of 32, and the largest batch of the configurations.
        _case("qkv_6.7b", "qkv", "opt6.7b", B=32),
        _case("qkv_30b", "qkv", "opt30b", B=128),
        # Ragged requests on block tables, half of the blocks checkpoints, regenerated.
        _case("paged_6.7b", "paged", "opt6.7b", B=32, L_min=512, L_max=1024, act_share=0.5),
        # A serving loop's step of a layer: write-back of the current tokens, then attention without regeneration.
        _case("serve_66b", "serve", "opt66b", B=64, L_min=2048, L_max=4096, act_share=0.5),
    ]


def _case(name, path, layer, dtype="f16", **sizes):
    cfg = synth.CONFIGS[layer]
    return {"name": name, "path": path, "d": cfg.d, "heads": cfg.n_heads, "dtype": dtype, **sizes}


def draw(rng):
    layer = rng.choice(sorted(synth.CONFIGS))
    path = rng.choice(["step", "step", "absorbed", "absorbed", "regen", "qkv", "paged", "serve"])
    cfg = synth.CONFIGS[layer]
    case = {"path": path, "d": cfg.d, "heads": cfg.n_heads, "dtype": rng.choice(["f16", "f16", "bf16"])}
    case["B"] = _log_uniform(rng, 1, 128)
    if path == "qkv":
        return case
    # at most 131072 tokens (half of the benchmark's workload) and a context of at most 4096
    L = _log_uniform(rng, 16, min(4096, 131072 // case["B"]))
    if path in ("step", "absorbed"):
        case["L_kv"] = round(rng.choice([0.0, 1.0, rng.random(), rng.random(), rng.random()]) * L)
        case["L_act"] = L - case["L_kv"]
    elif path == "regen":
        case["L_kv"], case["L_act"] = rng.randrange(0, 64), L
    else:
        case["L_min"], case["L_max"] = max(1, L // 2), L
        case["act_share"] = rng.choice([0.0, 0.5, round(rng.random(), 2)])
    return case


def _log_uniform(rng, low, high):
    return max(low, min(high, round(math.exp(rng.uniform(math.log(low), math.log(high))))))


# ----------------------------------------------------------------------------------------------------------- inputs
class _Draw:
    """Normal tensors on the GPU from one seed, at the recipe's scales."""

    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = dtype

    def __call__(self, *shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=self.dtype, device="cuda").normal_(mean, std, generator=self.gen)


def prepare(case, seed):
    el = DTYPES[case["dtype"]]
    draw_n = _Draw(seed, el)
    d, H, B = case["d"], case["heads"], case["B"]
    dh = d // H
    kv_std = 0.02 * d ** 0.5
    shape = hk.make_shape(d, H, dtype=hk.HK_DTYPE_BF16 if el == torch.bfloat16 else hk.HK_DTYPE_F16)
    s = {"path": case["path"], "H": H, "out": torch.empty(B, H, dh, dtype=el, device="cuda")}
    layer = (draw_n(d, std=0.02, mean=1.0), draw_n(d, std=0.02), draw_n(2 * d, d, std=0.02), draw_n(2 * d, std=0.01))
    s["layer"] = layer
    if case["path"] in ("qkv", "serve"):
        s["x"], s["Wq"], s["bq"] = draw_n(B, d), draw_n(d, d, std=0.02), draw_n(d, std=0.01)
        s["qkv_ws"] = hk.new_workspace(hk.hk_qkv_workspace_bytes(shape, B))
    if case["path"] == "qkv":
        s["K"], s["V"] = (torch.zeros(B, H, 4, dh, dtype=el, device="cuda") for _ in range(2))
        return s
    s["layer"] = layer + (hk.prepare_layer(*layer, H),)
    if case["path"] in ("paged", "serve"):
        _prepare_paged(s, case, seed, draw_n, shape, kv_std)
        return s
    L_kv, L_act = case["L_kv"], case["L_act"]
    s["act"] = draw_n(B, L_act, d) if L_act else None
    if case["path"] == "regen":
        s["K"], s["V"] = (torch.zeros(B, H, L_kv + L_act, dh, dtype=el, device="cuda") for _ in range(2))
        s["tok_off"] = L_kv
        s["ws"] = hk.new_workspace(hk.hk_regen_workspace_bytes(shape, B, L_act))
        return s
    s["q"] = draw_n(B, H, dh, std=kv_std)
    s["K"], s["V"] = (draw_n(B, H, L_kv, dh, std=kv_std) if L_kv else None for _ in range(2))
    s["ratio"] = L_kv / (L_kv + L_act)
    size = hk.hk_absorbed_workspace_bytes if case["path"] == "absorbed" else hk.hk_workspace_bytes
    s["ws"] = hk.new_workspace(size(shape, B, L_kv, L_act))
    return s


BLOCK = 16                                             # tokens of a block, as in the repository's measurements


def _lengths(case):
    """Request lengths: part of the case (not of the seed), so that the work is the same for every seed."""
    return np.random.default_rng(case["L_max"] * 1009 + case["B"]).integers(case["L_min"], case["L_max"] + 1, case["B"])


def _block_counts(case):
    blocks = int(sum((int(n) + BLOCK - 1) // BLOCK for n in _lengths(case)))
    act = round(case["act_share"] * blocks)
    return blocks - act, act


def _prepare_paged(s, case, seed, draw_n, shape, kv_std):
    d, H, B = case["d"], case["heads"], case["B"]
    lens = _lengths(case)
    n_kv, n_act = _block_counts(case)
    rng = np.random.default_rng(seed)
    kinds = np.concatenate([rng.permutation(n_kv), ~rng.permutation(n_act)])   # physical blocks in random order
    entries = rng.permutation(kinds).astype(np.int32)
    counts = (lens + BLOCK - 1) // BLOCK
    table = np.zeros((B, int(counts.max())), np.int32)
    at = 0
    for b, n in enumerate(counts):
        table[b, :n] = entries[at:at + n]
        at += n
    s["K"], s["V"] = (draw_n(n_kv, H, BLOCK, d // H, std=kv_std) if n_kv else None for _ in range(2))
    s["act"] = draw_n(n_act, BLOCK, d) if n_act else None
    s["q"] = draw_n(B, H, d // H, std=kv_std)
    s["table"], s["lens"] = torch.from_numpy(table).cuda(), torch.from_numpy(lens.astype(np.int32)).cuda()
    s["cu"] = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)).cuda()
    s["total"], s["n_act"] = int(lens.sum()), n_act
    cache = hk.make_paged_cache(s["K"], s["V"], s["act"], s["table"], s["lens"], s["cu"], s["total"], BLOCK, n_act,
                                el=draw_n.dtype)
    size = hk.lib().hk_paged_absorbed_workspace_bytes if s["path"] == "serve" else hk.lib().hk_paged_workspace_bytes
    s["ws"] = hk.new_workspace(int(size(ctypes.byref(shape), B, ctypes.byref(cache))))


# -------------------------------------------------------------------------------------------------------- one pass
def run(s):
    path = s["path"]
    if path == "step":
        # the step leaves the regenerated rows in its workspace: they are part of what it computes
        if s["act"] is None:
            return hk.hybrid_decode_attn(s["q"], s["K"], s["V"], None, s["layer"], s["ratio"], out=s["out"], workspace=s["ws"])
        return hk.hybrid_decode_attn(s["q"], s["K"], s["V"], s["act"], s["layer"], s["ratio"], out=s["out"], workspace=s["ws"],
                                     return_regen=True)
    if path == "absorbed":
        return hk.hybrid_decode_attn_absorbed(s["q"], s["K"], s["V"], s["act"], s["layer"], s["ratio"], out=s["out"],
                                              workspace=s["ws"])
    if path == "regen":
        return hk.regen_kv(s["act"], *s["layer"][:4], s["H"], K_out=s["K"], V_out=s["V"], tok_off=s["tok_off"],
                           workspace=s["ws"], prepared=s["layer"][4])
    if path == "qkv":
        q = hk.qkv_current(s["x"], *s["layer"], s["Wq"], s["bq"], s["H"], q_out=s["out"], K_dst=s["K"], V_dst=s["V"],
                           tok_pos=1, workspace=s["qkv_ws"])
        return q, s["K"], s["V"]
    q = s["q"]
    if path == "serve":
        q = hk.qkv_current_paged(s["x"], *s["layer"][:4], s["Wq"], s["bq"], s["H"], s["K"], s["V"], s["act"], s["table"],
                                 s["lens"], BLOCK, q_out=q, workspace=s["qkv_ws"])
    out = hk.paged_decode_attn(q, s["K"], s["V"], s["act"], s["table"], s["lens"], BLOCK, s["layer"], n_act_used=s["n_act"],
                               out=s["out"], workspace=s["ws"], absorbed=path == "serve", cu_tokens=s["cu"],
                               total_tokens=s["total"])
    return (q, out, s["K"], s["V"], s["act"]) if path == "serve" else out


# ------------------------------------------------------------------------------------------------- work, tolerance
def work(case):
    """Bytes: every input once and every output once.  Flops: the products of the path's own formulation."""
    d, H, B, path = case["d"], case["heads"], case["B"], case["path"]
    if path == "qkv":
        return {"bytes": 6 * d * d + 10 * B * d, "flops": 6 * B * d * d}
    if path in ("paged", "serve"):
        tokens = int(_lengths(case).sum())
        n_kv, n_act = _block_counts(case)
        M = min(tokens, n_act * BLOCK)
        cached = tokens - M
    else:
        M, cached = B * case["L_act"], B * case["L_kv"]
    if path == "regen":
        return {"bytes": 6 * M * d + 4 * d * d, "flops": 4 * M * d * d}
    weights = 4 * d * d if M else 0
    nbytes = 2 * M * d + 4 * cached * d + weights + 4 * B * d
    if path in ("absorbed", "serve"):
        flops = 4 * cached * d + ((4 * B * d * d + 4 * M * H * d) if M else 0)
        if path == "serve":
            nbytes, flops = nbytes + (6 * d * d - weights) + 8 * B * d, flops + 6 * B * d * d
        return {"bytes": nbytes, "flops": flops}
    return {"bytes": nbytes + (4 * M * d if path == "step" else 0), "flops": 4 * M * d * d + 4 * (M + cached) * d}


# Relative errors, about four times what each path shows against its own definition in 64 bits at the five layers' sizes
# (fp16, bf16): projected rows 3.9e-4, 2.7e-3; attention over regenerated rows 8.2e-4, 6.4e-3 (a 4096-token context at
# d = 9216, where a few tokens carry the softmax); without regenerating 1.3e-3, 4.6e-3.
_REL = {"qkv": (1.6e-3, 1.1e-2), "regen": (1.6e-3, 1.1e-2), "step": (3.2e-3, 2.4e-2), "paged": (3.2e-3, 2.4e-2),
        "absorbed": (5e-3, 1.8e-2), "serve": (5e-3, 1.8e-2)}


def tolerance(case):
    return {"rel": _REL[case["path"]][case["dtype"] == "bf16"]}
