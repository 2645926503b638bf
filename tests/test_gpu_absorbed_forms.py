"""The step without regeneration on every form of its two passes over the checkpoint rows (blocks of 32, 64 and 256 rows in the
score pass, one to eight blocks of 16 heads), against the definition in 64 bits (LayerNorm, K/V projection, softmax) for
sampled sequences and heads: at the edges of blocks, tiles and steps, with more blocks than factors fit in LDS at a time,
contiguous and through a block table whose requests have lengths of their own (none at all among them).

Rows differ in spread and mean, and some heads' scores are peaked, so that the blocks of a sequence have references far
apart.  Tolerance: that of the step (relative L2 5e-3); u, w and y are rounded once each to 11 bits (2^-12 / sqrt(3) each of
a row's sum, amplified through the softmax by the spread of the scores, here up to about 8)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import hk  # noqa: F401

pytestmark = pytest.mark.gpu

# (heads, head_dim, sequences, checkpoint rows of each): rows_log2 as absorbed_rows_log2 chooses
SIZES = [
    (1, 64, 1, 1), (3, 64, 2, 63), (5, 128, 3, 65), (17, 64, 2, 257),           # 64-row blocks, narrow layers
    (12, 64, 2, 4500),                                                          # 71 blocks: factors in three stretches
    (33, 64, 2, 1), (36, 64, 3, 31), (40, 64, 2, 97), (72, 64, 1, 33), (100, 64, 2, 64),   # 32-row blocks
    (33, 64, 2, 1100),                                                          # 35 of them: two stretches
    (40, 64, 8, 1025), (33, 64, 100, 83), (50, 64, 5, 1700), (72, 64, 9, 1000), (128, 64, 2, 4099),   # 64-row blocks, wide
    (40, 64, 64, 1025), (33, 64, 2, 33000), (50, 64, 40, 1700), (72, 64, 33, 1990), (100, 64, 11, 6000),   # 256-row blocks
    (81, 64, 2, 70), (96, 64, 9, 1000), (88, 64, 33, 1990),                     # six and seven blocks of heads, each form
    (97, 64, 2, 70), (112, 64, 9, 1000), (104, 64, 11, 6000),
]
ids = ["%dx%d-%dx%d" % s for s in SIZES]


def _layer_and_rows(hk, H, dh, B, L, dtype):
    d = H * dh
    gen = torch.Generator(device="cuda").manual_seed(L * 131 + d)

    def draw(*shape, std, mean=0.0):
        return torch.empty(shape, device="cuda").normal_(mean, std, generator=gen)

    layer = tuple(t.to(dtype) for t in (draw(d, std=0.02, mean=1.0), draw(d, std=0.02), draw(2 * d, d, std=0.02), draw(2 * d, std=0.01)))
    act = torch.empty(B, L, d, dtype=dtype, device="cuda")
    for b in range(B):                                         # rows of spread 0.3 to 3, means up to 2 spreads
        spread = torch.exp2(draw(L, 1, std=1.0).clamp_(-1.7, 1.6))
        act[b] = (spread * (draw(L, d, std=1.0) + draw(L, 1, std=1.0).clamp_(-2, 2))).to(dtype)
    q = draw(B, H, dh, std=1.0) * (0.02 * d ** 0.5)
    q[:, ::3] *= 2.0                                           # every third head peaked
    return layer, act, q.to(dtype)


def _reference(layer, rows, q, H, h):
    """Head h over `rows` [L, d] in float64."""
    ln_w, ln_b, W, b = (t.double() for t in layer)
    d, dh = rows.shape[1], q.shape[0]
    x = rows.double()
    xhat = (x - x.mean(1, keepdim=True)) / torch.sqrt(x.var(1, unbiased=False, keepdim=True) + 1e-5) * ln_w + ln_b
    k, v = (xhat @ W[o + h * dh:o + (h + 1) * dh].T + b[o + h * dh:o + (h + 1) * dh] for o in (0, d))
    return torch.softmax(k @ q.double() * dh ** -0.5, 0) @ v


def _check(out, ref, dtype):
    err = float((out - ref).norm() / ref.norm())
    tol = 5e-3 if dtype == torch.float16 else 1.2e-2           # bf16: the output's own rounding is 2^-9 and the weights' 2^-9
    print("rel_l2 %.2e" % err, flush=True)
    assert err <= tol


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B,L", SIZES, ids=ids)
def test_contiguous(hk, H, dh, B, L, dtype):
    layer, act, q = _layer_and_rows(hk, H, dh, B, L, dtype)
    out = hk.hybrid_decode_attn_absorbed(q, None, None, act, layer + (hk.prepare_layer(*layer, H),), 0.0)
    pairs = [(b, h) for b in sorted({0, B // 2, B - 1}) for h in sorted({0, H // 2, H - 1})]
    _check(torch.stack([out[b, h].double() for b, h in pairs]),
           torch.stack([_reference(layer, act[b], q[b, h], H, h) for b, h in pairs]), dtype)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("block", [16, 64])
@pytest.mark.parametrize("H,dh,B,L", [s for s in SIZES if s[3] > 1 and s[2] > 1], ids=[i for i, s in zip(ids, SIZES) if s[3] > 1 and s[2] > 1])
def test_paged(hk, H, dh, B, L, block, dtype):
    layer, act, q = _layer_and_rows(hk, H, dh, B, L, dtype)
    rng = np.random.default_rng(L)
    lens = rng.integers(max(1, L // 2), L + 1, B)
    lens[0], lens[-1] = L, 0 if B > 2 else max(1, L - 17)
    counts = -(-lens // block)
    total = int(counts.sum())
    perm = rng.permutation(total)
    pool = torch.zeros(total, block, H * dh, dtype=dtype, device="cuda")
    table = np.zeros((B, int(counts.max())), np.int32)
    at = 0
    for b in range(B):
        for i in range(int(counts[b])):
            n = min(block, int(lens[b]) - i * block)
            pool[perm[at], :n] = act[b, i * block:i * block + n]
            table[b, i] = ~perm[at]
            at += 1
    lens_dev = torch.from_numpy(lens.astype(np.int32)).cuda()
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)).cuda()
    out = hk.paged_decode_attn(q, None, None, pool, torch.from_numpy(table).cuda(), lens_dev, block, layer + (hk.prepare_layer(*layer, H),),
                               n_act_used=total, absorbed=True, cu_tokens=cu, total_tokens=int(lens.sum()))
    pairs = [(b, h) for b in sorted({0, B // 2}) for h in sorted({0, H // 2, H - 1})]
    _check(torch.stack([out[b, h].double() for b, h in pairs]),
           torch.stack([_reference(layer, act[b, :int(lens[b])], q[b, h], H, h) for b, h in pairs]), dtype)
    if lens[-1] == 0:
        assert not out[-1].any()
