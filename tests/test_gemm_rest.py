"""The projection on a prepared layer in two launches: full rounds of 256 x 256 tiles, then a smaller tile for the rows that
are left.  The cut is a row of the problem, not of a sequence, so it falls inside sequences here; the rows must be the same
bits as those of the 256 x 256 kernel alone, and every other byte of the caches stays as it was."""
import os
import subprocess

import pytest
import torch

from test_gpu_parity import hk  # noqa: F401

HERE = os.path.dirname(os.path.abspath(__file__))
# (heads, head_dim, sequences, checkpoint rows of each), the second launch's tile on a 256-unit device
SIZES = [
    ((12, 128, 1, 5377), (32, 32)),                             # one row left
    ((12, 128, 4, 1363), (64, 32)),
    ((12, 128, 3, 1839), (32, 64)),
    ((12, 128, 5, 1109), (64, 64)),
    ((12, 128, 1, 11081), (128, 64)),                           # several rounds before it
    ((17, 128, 2, 2117), (64, 128)),
    ((6, 128, 100, 123), (128, 128)),                           # short sequences
    ((6, 128, 1, 13447), (192, 128)),
    ((12, 128, 2, 3653), (256, 128)),
    ((12, 128, 2, 3974), (128, 256)),
]


def test_the_compared_sizes_take_two_launches(tmp_path):
    exe = str(tmp_path / "gemm_plan_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", os.path.join(HERE, "host", "gemm_plan_check.cpp"), "-o", exe])
    args = [str(v) for (H, dh, B, L), _ in SIZES for v in (B * L, H * dh)]
    lines = subprocess.check_output([exe, "256"] + args, text=True).split("\n")
    for ((H, dh, B, L), tile), line in zip(SIZES, lines):
        rows, bm, bn = (int(v) for v in line.split())
        assert 0 < rows < B * L and (bm, bn) == tile, (H, dh, B, L, line)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B,L", [size for size, _ in SIZES])
def test_two_launches_give_the_same_rows(hk, H, dh, B, L, dtype):
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
