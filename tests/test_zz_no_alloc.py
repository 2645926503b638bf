"""hk_hybrid_decode_attn_static (the step on the library's static scratch array, for callers that cannot
allocate) against hk_hybrid_decode_attn, through the C ABI: the same kernels on a different scratch address, so the
results must be bit-identical; and both within the step's tolerance of the oracle.  Two calls in a row, the second
on a smaller input (the array keeps the first call's contents)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import hybridkv_oracle as ho
from paper_2501_01792_amd import binding as hk
from paper_2501_01792_amd import synth

MAX_ABS, REL_L2 = 2e-2, 5e-3


def _run_both(cfg, prepared, gemm_tile=0):
    b = synth.make_batch(cfg)
    g = {k: torch.from_numpy(v).cuda() for k, v in b.items()}
    lp = (g["ln_w"], g["ln_b"], g["Wkv"], g["bkv"])
    if prepared:
        lp = lp + (hk.prepare_layer(*lp, cfg.n_heads),)
    Kc, Vc = (g["K_cache"], g["V_cache"]) if cfg.L_kv else (None, None)
    act = g["act"] if cfg.L_act else None
    ref_gpu = hk.hybrid_decode_attn(g["q"], Kc, Vc, act, lp, cfg.ratio, gemm_tile=gemm_tile)
    out = torch.full_like(ref_gpu, 7.0)
    hk.hybrid_decode_attn_static(g["q"], Kc, Vc, act, lp, cfg.ratio, out, gemm_tile=gemm_tile)
    torch.cuda.synchronize()
    assert torch.equal(out, ref_gpu), "static-scratch call differs from the workspace call on %s" % cfg.name
    ref, _, _ = ho.hybrid_decode_attn(b["q"], b["K_cache"] if cfg.L_kv else None, b["V_cache"] if cfg.L_kv else None,
                                      b["act"] if cfg.L_act else None, b["ln_w"], b["ln_b"], b["Wkv"], b["bkv"], cfg.n_heads)
    got = out.float().cpu().numpy().astype(np.float64)
    err, rel = np.abs(got - ref).max(), np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("%s: max_abs=%.3e rel_l2=%.3e" % (cfg.name, err, rel), flush=True)
    assert err <= MAX_ABS and rel <= REL_L2


@pytest.mark.gpu
def test_static_scratch_call_matches_the_workspace_call_twice_in_a_row():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU path")
    # first a problem that fills most of the array and runs the large-problem projection kernel on a prepared
    # layer brought by the caller (d = 1024, 6 x 1024 checkpoint rows, 256-tiles asked for); then smaller ones that
    # reuse the dirty array: the tiny benchmark layer (small-problem kernel, layer not prepared), then one with no
    # checkpoints at all
    big = synth.LayerConfig("static_big", 1024, 8, 6, 2048, 0.5, 71)
    shape = hk.make_shape(big.d, big.n_heads, gemm_tile=256)
    need = hk.hk_workspace_bytes(shape, big.B, big.L_kv, big.L_act) - hk.hk_prepared_bytes(shape)
    assert hk.HK_STATIC_SCRATCH_BYTES // 2 < need <= hk.HK_STATIC_SCRATCH_BYTES
    _run_both(big, prepared=True, gemm_tile=256)
    _run_both(synth.CONFIGS["tiny"], prepared=False)
    _run_both(synth.LayerConfig("static_all_kv", 768, 12, 3, 200, 1.0, 72), prepared=False)


def _largest_L_act(d, dh, bf16, prepared, B, L_kv):
    """Largest L_act for which the array holds the regenerated rows, their statistics, the room for a prepared layer where
    the call makes one and one partial per 128 positions (at most 4096) and pair."""
    H = d // dh
    up = lambda n: (n + 255) // 256 * 256

    def need(L_act):
        M, positions = B * L_act, B * H * (L_kv + L_act)
        room = up(4 * d * d) + 2 * up(8 * d) if bf16 and not prepared else 0
        return 2 * up(2 * M * d) + up(8 * M) + room + up((min(4096, -(-positions // 128)) + B * H) * (dh + 2) * 4)

    lo, hi = 0, 1 << 20
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if need(mid) <= hk.HK_STATIC_SCRATCH_BYTES else (lo, mid)
    return lo


LIMITS = [(4096, 128, False, True, 1, 0), (4096, 128, False, True, 1, 6000), (4096, 128, False, True, 1, 30000),
          (64, 64, True, False, 1, 0), (768, 64, False, True, 3, 1000), (1024, 128, True, False, 2, 100)]


@pytest.mark.parametrize("d,dh,bf16,prepared,B,L_kv", LIMITS)
def test_static_scratch_call_takes_what_128_positions_a_range_leave_room_for(d, dh, bf16, prepared, B, L_kv):
    """Host check (no GPU) of the limit: a finer cut of the positions must not refuse a step."""
    L_act = _largest_L_act(d, dh, bf16, prepared, B, L_kv)
    FAKE = 0x7F0000001000
    lp = hk.hk_layer_params(FAKE, FAKE, FAKE, FAKE, FAKE if prepared else None)
    shape = hk.make_shape(d, d // dh, dtype=hk.HK_DTYPE_BF16 if bf16 else hk.HK_DTYPE_F16)
    # all checks of sizes passed: the missing query is what is left to complain about
    assert hk.lib().hk_hybrid_decode_attn_static(ctypes.byref(shape), None, FAKE, FAKE, L_kv, FAKE, L_act, B, ctypes.byref(lp),
                                                 L_kv / (L_kv + L_act), FAKE, None) == hk.HK_ERR_NULL
    in_call = hk.hk_prepared_bytes(shape) if bf16 and prepared else 0        # room that a caller with a prepared layer saves
    assert hk.hk_workspace_bytes(shape, B, L_kv, L_act) - in_call <= hk.HK_STATIC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("d,dh,bf16,prepared,B,L_kv", [LIMITS[1], LIMITS[4], LIMITS[5]])
def test_static_scratch_call_at_its_limit_gives_the_bits_of_the_workspace_call(d, dh, bf16, prepared, B, L_kv):
    """The cut that the array's size asks for is that of the workspace call too."""
    H, L_act = d // dh, _largest_L_act(d, dh, bf16, prepared, B, L_kv)
    gen = torch.Generator(device="cuda").manual_seed(d)
    draw = lambda *s, std=1.0, mean=0.0: torch.empty(s, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float16).normal_(mean, std, generator=gen)
    lp = (draw(d, std=0.02, mean=1.0), draw(d, std=0.02), draw(2 * d, d, std=0.02), draw(2 * d, std=0.01))
    if prepared:
        lp = lp + (hk.prepare_layer(*lp, H),)
    q, act, K, V = draw(B, H, dh), draw(B, L_act, d), draw(B, H, L_kv, dh), draw(B, H, L_kv, dh)
    ref = hk.hybrid_decode_attn(q, K, V, act, lp, L_kv / (L_kv + L_act))
    out = torch.full_like(ref, 7.0)
    hk.hybrid_decode_attn_static(q, K, V, act, lp, L_kv / (L_kv + L_act), out)
    assert torch.equal(out, ref)


def test_static_scratch_call_rejects_what_does_not_fit():
    """Host checks (no GPU): a problem beyond the array is refused with its own status before anything else
    happens; the other checks are those of the workspace call."""
    FAKE = 0x7F0000001000
    lp = hk.hk_layer_params(FAKE, FAKE, FAKE, FAKE, None)
    lp_prep = hk.hk_layer_params(FAKE, FAKE, FAKE, FAKE, FAKE)

    def call(shape, L_kv, L_act, B, lp=lp, ratio=0.5, q=FAKE):
        return hk.lib().hk_hybrid_decode_attn_static(ctypes.byref(shape), q, FAKE, FAKE, L_kv, FAKE, L_act, B,
                                                     ctypes.byref(lp), ratio, FAKE, None)

    s67 = hk.make_shape(4096, 32)
    assert call(s67, 512, 512, 32) == hk.HK_ERR_STATIC_LIMIT             # 268 MB of regenerated K/V
    assert call(s67, 512, 512, 32, lp=lp_prep) == hk.HK_ERR_STATIC_LIMIT
    assert "HK_STATIC_SCRATCH_BYTES" in hk.status_string(hk.HK_ERR_STATIC_LIMIT)
    small = hk.make_shape(768, 12)
    assert call(small, 128, 128, 4, ratio=0.25) == hk.HK_ERR_RATIO
    assert call(small, 128, 128, 4, q=None) == hk.HK_ERR_NULL
    assert call(hk.make_shape(768, 11), 128, 128, 4) == hk.HK_ERR_SHAPE
    assert call(small, 0, 0, 4) == hk.HK_ERR_SHAPE
    assert call(small, 128, 128, 0) == hk.HK_OK                          # an empty batch: nothing to do
