"""The projection on a prepared layer takes a tile from 32 x 32 to 256 x 256 by the size of the problem; every tile adds
the same products in the same order as the 256 x 256 kernel (which the parity tests compare with the oracle), so the
regenerated rows must be the same bits, at tile edges, with rows left over, with one and several output tiles per compute
unit, with as many k blocks as the load ring has stages and fewer, and every other byte of the caches stays as it was."""
import pytest
import torch

from test_gpu_parity import hk  # noqa: F401

pytestmark = pytest.mark.gpu

# (heads, head_dim, sequences, checkpoint rows of each): comments name the tile that a 256-unit device takes
SIZES = [
    (1, 128, 1, 1), (1, 128, 3, 11), (2, 64, 1, 512),             # 32 x 32; 2 k blocks: fewer than the ring's stages
    (3, 64, 2, 351), (5, 64, 1, 512),                             # 64 x 32
    (1, 128, 1, 2100), (12, 64, 1, 449), (12, 64, 2, 256),        # 64 x 64
    (5, 64, 3, 697), (12, 64, 1, 1023),                           # 128 x 64
    (3, 64, 1, 6001), (12, 128, 1, 701),                          # 128 x 128
    (12, 128, 1, 1537), (5, 64, 1, 8000), (12, 64, 4, 3001),      # 192 x 128
    (12, 64, 1, 4100), (32, 128, 5, 193),                         # 256 x 128
    (72, 128, 1, 5),                                              # 32 x 32, several tiles per compute unit
    (17, 64, 1, 195), (51, 128, 2, 15),                           # 32 x 64
    (72, 128, 3, 17),                                             # 64 x 128
    (56, 128, 1, 500),                                            # 256 x 128
    (72, 128, 1, 300), (12, 128, 1, 2563),                        # 128 x 256
    (12, 64, 1, 6000),                                            # 256 x 256
]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("ln_scale", [1.0, 1e-2, 1e-3, 1e-4])
@pytest.mark.parametrize("H,dh,B,L", [(6, 128, 4, 17), (6, 128, 4, 6000)])        # a small tile; 256 x 256
def test_small_layernorm_weights_keep_the_precision_of_a_prepared_layer(hk, H, dh, B, L, ln_scale, dtype):
    """A small ln_w must not push the prepared weights out of the normal range of their type.  Rows: one rounding of the
    weights and one of the result, each u / sqrt(3) at most in the 2-norm (u = 2^-11; 2^-8, bf16).  Attention without
    regenerated rows: the tolerance of the step, 5e-3."""
    d = H * dh
    gen = torch.Generator(device="cuda").manual_seed(L)

    def draw(*shape, std, mean=0.0):
        return torch.empty(shape, device="cuda").normal_(mean, std, generator=gen)

    layer = tuple(t.to(dtype) for t in (draw(d, std=0.02, mean=1.0) * ln_scale, draw(d, std=0.02) * ln_scale,
                                        draw(2 * d, d, std=0.2), draw(2 * d, std=0.1) * ln_scale))
    prepared = hk.prepare_layer(*layer, H)
    # scores of spread 1.6 whatever ln_w is; weights of 0.2 keep the results themselves in the normal range
    act, q = draw(B, L, d, std=1.0, mean=0.25).to(dtype), draw(B, H, dh, std=0.3 / ln_scale).to(dtype)
    K, V = hk.regen_kv(act, *layer, H, prepared=prepared)
    out = hk.hybrid_decode_attn_absorbed(q, None, None, act, layer + (prepared,), 0.0)

    ln_w, ln_b, W, b = (t.double() for t in layer)
    x = act.double().view(B * L, d)
    xhat = (x - x.mean(1, keepdim=True)) / torch.sqrt(x.var(1, unbiased=False, keepdim=True) + 1e-5) * ln_w + ln_b
    rk, rv = ((xhat @ W.T + b).view(B, L, 2, H, dh).permute(2, 0, 3, 1, 4))
    u = {torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[dtype]
    for name, got, ref, tol in (("K", K, rk, 2 * u / 3 ** 0.5), ("V", V, rv, 2 * u / 3 ** 0.5),
                                ("out", out, (torch.softmax((q.double()[:, :, None] * rk).sum(-1) * dh ** -0.5, 2)[..., None] * rv).sum(2), 5e-3)):
        err = float((got.double() - ref).norm() / ref.norm())
        print("%s: rel_l2 = %.3e" % (name, err), flush=True)
        assert err <= tol, name


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B,L", SIZES)
def test_every_tile_gives_the_same_rows(hk, H, dh, B, L, dtype):
    d = H * dh
    gen = torch.Generator(device="cuda").manual_seed(L * 131 + d)

    def draw(*shape, std, mean=0.0):
        return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=gen)

    layer = (draw(d, std=0.02, mean=1.0), draw(d, std=0.02), draw(2 * d, d, std=0.02), draw(2 * d, std=0.01))
    prepared = hk.prepare_layer(*layer, H)
    act = draw(B, L, d, std=1.0, mean=0.25)
    got = {}
    for tile in (0, 256):
        K, V = (torch.full((B, H, L + 5, dh), -7.0, dtype=dtype, device="cuda") for _ in range(2))
        hk.regen_kv(act, *layer, H, K_out=K, V_out=V, tok_off=3, prepared=prepared, gemm_tile=tile)
        got[tile] = (K, V)
    for a, ref in zip(got[0], got[256]):
        assert torch.equal(a, ref)
        assert bool((a[:, :, :3] == -7.0).all()) and bool((a[:, :, L + 3:] == -7.0).all())
        assert bool((a[:, :, 3:L + 3] != -7.0).any())
