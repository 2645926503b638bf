"""QKV generation in three launches (many rows, wide layers; chosen by rows, width and the size of the workspace) against
the definition in 64 bits: heights of the row tile and their edges, widths that 128 does and does not divide, fewer units
of work than workgroups, q alone, a cache of which only one row may change, and a workspace too small for it.

Tolerances: one rounding of the normalised row and one of the result, each at most u relative per element (u = 2^-11, fp16;
2^-8, bf16) in root mean square below u / sqrt(3), so 2 u / sqrt(3) at most for the two together in the 2-norm."""
import pytest
import torch

from test_gpu_parity import hk  # noqa: F401

pytestmark = pytest.mark.gpu

SIZES = [(12, 64, 65), (12, 64, 96), (6, 128, 97), (13, 64, 128), (13, 64, 70),      # more than 64 rows; d = 832
         (16, 128, 33), (33, 64, 64), (16, 128, 64),                                 # 33 to 64 rows; d = 2112
         (44, 128, 1), (87, 64, 32), (44, 128, 31)]                                  # few rows, wide; d = 5568
UNIT = {torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B", SIZES)
def test_three_launches_match_the_definition(hk, H, dh, B, dtype):
    d = H * dh
    shape = hk.make_shape(d, H, dtype=hk.HK_DTYPE_BF16 if dtype == torch.bfloat16 else hk.HK_DTYPE_F16)
    need = hk.hk_qkv_workspace_bytes(shape, B)
    assert need > 256
    gen = torch.Generator(device="cuda").manual_seed(d * 131 + B)

    def draw(*size, std, mean=0.0):
        return torch.empty(size, dtype=dtype, device="cuda").normal_(mean, std, generator=gen)

    ln_w, ln_b = draw(d, std=0.02, mean=1.0), draw(d, std=0.02)
    Wkv, bkv, Wq, bq = draw(2 * d, d, std=0.02), draw(2 * d, std=0.01), draw(d, d, std=0.02), draw(d, std=0.01)
    x = draw(B, d, std=1.0, mean=0.25)
    x64 = x.double()
    xhat = (x64 - x64.mean(1, keepdim=True)) / torch.sqrt(x64.var(1, unbiased=False, keepdim=True) + shape.ln_eps)
    xhat = xhat * ln_w.double() + ln_b.double()
    ref = (xhat @ Wq.double().T + bq.double(), *(xhat @ Wkv.double().T + bkv.double()).split(d, dim=1))

    def call(nbytes, kv=True):
        K, V = (torch.full((B, H, 3, dh), -7.0, dtype=dtype, device="cuda") for _ in range(2)) if kv else (None, None)
        A = torch.full((B, 3, d), 5.0, dtype=dtype, device="cuda")
        q = hk.qkv_current(x, ln_w, ln_b, Wkv, bkv, Wq, bq, H, K_dst=K, V_dst=V, tok_pos=1, act_dst=A, act_pos=2,
                           workspace=hk.new_workspace(nbytes))
        assert torch.equal(A[:, 2], x) and bool((A[:, :2] == 5.0).all())
        return q, K, V

    got = {n: call(n) for n in (need, 256)}
    for n, (q, K, V) in got.items():
        for name, o, r in (("q", q, ref[0]), ("k", K[:, :, 1], ref[1]), ("v", V[:, :, 1], ref[2])):
            err = float((o.reshape(B, d).double() - r).norm() / r.norm())
            print("workspace %d %s: rel_l2 = %.3e" % (n, name, err), flush=True)
            # the single kernel rounds once more on the way into the product
            assert err <= (2 if n == need else 3) * UNIT[dtype] / 3 ** 0.5
        for c in (K, V):
            assert bool((c[:, :, ::2] == -7.0).all())
    assert torch.equal(call(need, kv=False)[0], got[need][0])           # q does not depend on whether K / V are produced
    assert torch.equal(call(need)[1], got[need][1])                     # the order of the partial sums is fixed
