"""The attention kernels at the edges of their 64-token steps, of their ranges and of the merge: lengths around
multiples of 64, fewer pairs than a merge workgroup holds, one to many partials per pair; contiguous and through block
tables, fp16 and bf16, against the CPU oracles.

Tolerances are those of the step's parity tests: fp16 max abs 2e-2 and relative L2 5e-3; bf16 (8 significant bits)
2^-7 of the largest reference value and 5e-3."""
import numpy as np
import pytest
import torch

from oracle import paged_oracle as pgo
from paper_2501_01792_amd import synth
from test_gpu_bf16 import _bf16, _check as _check_bf16
from test_gpu_parity import _check as _check_f16, _gpu, hk  # noqa: F401

pytestmark = pytest.mark.gpu


def _to_gpu(x, dtype):
    """(GPU tensor, the values it holds)"""
    return _bf16(x) if dtype == "bf16" else (_gpu(x.astype(np.float16)), x.astype(np.float16))


def _check(name, got, ref, dtype):
    if dtype == "bf16":
        _check_bf16(name, got, ref)
    else:
        _check_f16(name, got.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("dh,H,B", [(128, 2, 1), (64, 5, 1), (128, 3, 2)])
@pytest.mark.parametrize("L", [1, 63, 64, 65, 128, 193, 700])
def test_cached_attention_at_step_edges(hk, oracle, L, dh, H, B, dtype):
    d = H * dh
    rng = np.random.default_rng(1000 * L + d)
    q, qh = _to_gpu(rng.standard_normal((B, H, dh)), dtype)
    K, Kh = _to_gpu(rng.standard_normal((B, H, L, dh)), dtype)
    V, Vh = _to_gpu(rng.standard_normal((B, H, L, dh)), dtype)
    z = np.zeros(d, np.float16)
    out = hk.hybrid_decode_attn(q, K, V, None, tuple(t.to(q.dtype) for t in (_gpu(z), _gpu(z), torch.zeros(2 * d, d, device="cuda"),
                                                                             torch.zeros(2 * d, device="cuda"))), 1.0)
    torch.cuda.synchronize()
    ref, _, _ = oracle.hybrid_decode_attn(qh, Kh, Vh, None, z, z, np.zeros((2 * d, d), np.float16), np.zeros(2 * d, np.float16), H)
    _check("out", out, ref, dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lens", [[1], [64, 1, 63, 0, 65], [640, 127, 129, 2], [64] * 6, [1000, 3, 500]], ids=str)
@pytest.mark.parametrize("bt", [16, 64])
def test_paged_attention_at_step_edges(hk, lens, bt, dtype):
    """Ranges end inside a step of a pair and are moved to its start: every token is taken once, ranges left empty
    are neutral."""
    cfg = synth.LayerConfig("edges", 384, 3, len(lens), max(lens), 0.5, 71)
    rng = np.random.default_rng(sum(lens))
    B, H, dh, L = cfg.B, cfg.n_heads, cfg.head_dim, cfg.L
    batch = {"act_full": np.zeros((B, L, cfg.d), np.float16), "q": rng.standard_normal((B, H, dh)),
             "K_full": rng.standard_normal((B, H, L, dh)).astype(np.float16),
             "V_full": rng.standard_normal((B, H, L, dh)).astype(np.float16)}
    paged = synth.scatter_into_blocks(cfg, batch, lens, bt, 0.0, seed=5)
    q, qh = _to_gpu(batch["q"], dtype)
    Kp, Kh = _to_gpu(paged["K_pool"].astype(np.float32), dtype)
    Vp, Vh = _to_gpu(paged["V_pool"].astype(np.float32), dtype)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    out = hk.paged_decode_attn(q, Kp, Vp, None, _gpu(paged["block_table"]), _gpu(paged["seq_len"]), bt, None, n_act_used=0,
                               cu_tokens=_gpu(cu), total_tokens=int(cu[-1]))
    torch.cuda.synchronize()
    z = np.zeros(cfg.d, np.float16)
    ref = pgo.paged_decode_attn(qh, Kh, Vh, paged["act_pool"], paged["block_table"], paged["seq_len"], bt, z, z,
                                np.zeros((2 * cfg.d, cfg.d), np.float16), np.zeros(2 * cfg.d, np.float16), H)
    _check("out", out, ref, dtype)


def _with_and_without_an_infinity(call, V, at):
    """call() with V as it is and with V[at] = inf (one element of one token of every pair)."""
    out = call().clone()
    V[at] = float("inf")
    return out, call()


def _only_infinite_at(out, ref, e):
    """The weight of every token is positive here, so the element is infinite; the others do not know of it."""
    assert bool((out[..., e] == float("inf")).all()), "%d NaN" % int(out[..., e].isnan().sum())
    keep = [i for i in range(out.shape[-1]) if i != e]
    assert torch.equal(out[..., keep], ref[..., keep])


# one partial per pair (which no batch of the merge is), several, many; whole steps of 64 tokens
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("dh,H,L,t", [(128, 3, 64, 0), (64, 2, 64, 63), (128, 2, 128, 100), (128, 4, 640, 600), (128, 1, 1280, 1279)])
def test_an_infinite_value_stays_infinite_in_the_merge(hk, dh, H, L, t, dtype):
    rng = np.random.default_rng(L + t)
    q, K, V = (_to_gpu(rng.standard_normal(s), dtype)[0] for s in ((2, H, dh), (2, H, L, dh), (2, H, L, dh)))
    z = torch.zeros(16, dtype=q.dtype, device="cuda")                   # layer parameters: nothing is regenerated
    ref, out = _with_and_without_an_infinity(lambda: hk.hybrid_decode_attn(q, K, V, None, (z, z, z, z), 1.0), V, (..., t, 5))
    _only_infinite_at(out, ref, 5)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lens,block,row", [([64, 128], 3, 15), ([640, 64], 5, 0), ([64], 0, 7)], ids=str)
def test_an_infinite_value_stays_infinite_in_the_paged_merge(hk, lens, block, row, dtype):
    _paged_infinity(hk, lens, block, row, dtype)


def _paged_infinity(hk, lens, block, row, dtype, H=3, dh=128, bt=16):
    """V infinite in one row of one block of request 0; blocks lie in the pool in reverse order."""
    rng = np.random.default_rng(sum(lens))
    counts = [(n + bt - 1) // bt for n in lens]
    pool, table, at = sum(counts), np.zeros((len(lens), max(counts)), np.int32), 0
    for r, c in enumerate(counts):
        table[r, :c] = pool - 1 - np.arange(at, at + c)
        at += c
    q, K, V = (_to_gpu(rng.standard_normal(s), dtype)[0] for s in ((len(lens), H, dh), (pool, H, bt, dh), (pool, H, bt, dh)))
    tab, sl = _gpu(table), _gpu(np.asarray(lens, np.int32))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    cud = _gpu(cu)
    ref, out = _with_and_without_an_infinity(
        lambda: hk.paged_decode_attn(q, K, V, None, tab, sl, bt, None, n_act_used=0, cu_tokens=cud, total_tokens=int(cu[-1])),
        V, (int(table[0, block]), slice(None), row, 5))
    _only_infinite_at(out[:1], ref[:1], 5)
    assert torch.equal(out[1:], ref[1:])


# steps of fewer than 64 tokens, whose missing rows are read from the last one of the range
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("dh,H,L,t", [(128, 3, 1, 0), (64, 2, 65, 64), (128, 32, 1999, 1998), (128, 32, 1999, 61), (64, 5, 700, 63),
                                      (128, 3, 127, 63)])
def test_an_infinite_value_stays_infinite_beside_masked_rows(hk, dh, H, L, t, dtype):
    rng = np.random.default_rng(L + t)
    q, K, V = (_to_gpu(rng.standard_normal(s), dtype)[0] for s in ((1, H, dh), (1, H, L, dh), (1, H, L, dh)))
    z = torch.zeros(16, dtype=q.dtype, device="cuda")
    ref, out = _with_and_without_an_infinity(lambda: hk.hybrid_decode_attn(q, K, V, None, (z, z, z, z), 1.0), V, (..., t, 5))
    _only_infinite_at(out, ref, 5)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lens,block,row", [([65, 64], 4, 0), ([1], 0, 0), ([700, 3], 43, 11)], ids=str)
def test_an_infinite_value_stays_infinite_beside_masked_rows_paged(hk, lens, block, row, dtype):
    _paged_infinity(hk, lens, block, row, dtype)
