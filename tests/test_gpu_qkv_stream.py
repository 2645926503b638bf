"""QKV generation in three launches (many rows, wide layers; chosen by rows, width and the size of the workspace) against
the definition in 64 bits: heights of the row tile and their edges, widths that 128 does and does not divide, fewer units
of work than workgroups, q alone, a cache of which only one row may change, and a workspace too small for it.

Tolerances: one rounding of the normalised row and one of the result, each at most u relative per element (u = 2^-11, fp16;
2^-8, bf16) in root mean square below u / sqrt(3), so 2 u / sqrt(3) at most for the two together in the 2-norm."""
import numpy as np
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


def _paged_inputs(H, dh, B, bt, with_kv, dtype, seed):
    """Inputs and a cache in which the token of a request goes to a KV block, to a checkpoint block, or nowhere: no token,
    masked, an entry outside its pool, a token past the table's last block."""
    d, max_blocks = H * dh, 5
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def draw(*size, std, mean=0.0):
        return torch.empty(size, dtype=dtype, device="cuda").normal_(mean, std, generator=gen)

    p = {"layer": (draw(d, std=0.02, mean=1.0), draw(d, std=0.02), draw(2 * d, d, std=0.02), draw(2 * d, std=0.01)),
         "Wq": draw(d, d, std=0.02), "bq": draw(d, std=0.01), "x": draw(B, d, std=1.0, mean=0.25)}
    rng = np.random.default_rng(seed)
    P_kv, P_act = (B + 2 if with_kv else 0), B + 1
    seq_len = rng.integers(1, max_blocks * bt + 1, B).astype(np.int32)
    seq_len[0], seq_len[1], seq_len[2] = max_blocks * bt, bt + 1, bt                 # last row of all, first row, last row of a block
    seq_len[3] = 0
    seq_len[4] = max_blocks * bt + 1
    mask = np.ones(B, np.int32)
    mask[5::7] = 0
    kv_ids, act_ids = rng.permutation(max(P_kv, 1)), rng.permutation(P_act)
    table = np.full((B, max_blocks), 0x7fffffff, np.int32)
    dst = {}                                                                        # request -> (is checkpoint, block, row)
    for b in range(B):
        t = int(seq_len[b]) - 1
        if t < 0 or t // bt >= max_blocks:
            continue
        act = not with_kv or rng.random() < 0.5
        block = int(act_ids[b]) if act else int(kv_ids[b])
        if b in (6, 8):                                                             # outside its pool
            act, block = not with_kv or b == 6, (P_act if not with_kv or b == 6 else P_kv) + b
        elif mask[b]:
            dst[b] = (act, block, t % bt)
        table[b, t // bt] = ~block if act else block
    p.update(table=torch.from_numpy(table).cuda(), seq_len=torch.from_numpy(seq_len).cuda(), mask=torch.from_numpy(mask).cuda(),
             dst=dst, P_kv=P_kv, P_act=P_act, bt=bt, H=H, dh=dh)
    return p


def _pools(p, dtype):
    K, V = (torch.full((max(p["P_kv"], 1), p["H"], p["bt"], p["dh"]), v, dtype=dtype, device="cuda") for v in (7.0, -7.0))
    return K, V, torch.full((p["P_act"], p["bt"], p["H"] * p["dh"]), 3.0, dtype=dtype, device="cuda")


def _paged_call(hk, p, pools, q, ws):
    K, V, A = pools
    return hk.qkv_current_paged(p["x"], *p["layer"], p["Wq"], p["bq"], p["H"], K if p["P_kv"] else None, V if p["P_kv"] else None, A,
                                p["table"], p["seq_len"], p["bt"], q_out=q, workspace=ws, store_mask=p["mask"])


def _expected(hk, p, ws, dtype):
    """(q, pools): the rows of the contiguous call, which is compared with the definition above, put where they belong."""
    B, H, dh = p["x"].shape[0], p["H"], p["dh"]
    K, V = (torch.zeros(B, H, 1, dh, dtype=dtype, device="cuda") for _ in range(2)) if p["P_kv"] else (None, None)
    q = hk.qkv_current(p["x"], *p["layer"], p["Wq"], p["bq"], H, K_dst=K, V_dst=V, workspace=ws)
    pools = _pools(p, dtype)
    for b, (act, block, row) in p["dst"].items():
        if act:
            pools[2][block, row] = p["x"][b]
        else:
            pools[0][block, :, row], pools[1][block, :, row] = K[b, :, 0], V[b, :, 0]
    return q, pools


PAGED = [(12, 64, 70, 16, True), (12, 64, 130, 32, True), (33, 64, 40, 64, True), (44, 128, 9, 16, True),
         (33, 64, 40, 16, False), (44, 128, 20, 32, False)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B,bt,with_kv", PAGED)
def test_three_launches_write_the_rows_that_the_table_names(hk, H, dh, B, bt, with_kv, dtype):
    """K / V rows and checkpoints land in the blocks of the table, with the bits of the contiguous call; every other byte
    of the pools stays."""
    p = _paged_inputs(H, dh, B, bt, with_kv, dtype, seed=H * dh + B)
    need = hk.hk_qkv_workspace_bytes(hk.make_shape(H * dh, H, dtype=hk.HK_DTYPE_BF16 if dtype == torch.bfloat16 else hk.HK_DTYPE_F16), B)
    assert need > 256
    ws, pools = hk.new_workspace(need), _pools(p, dtype)
    q = _paged_call(hk, p, pools, None, ws)
    ref_q, ref = _expected(hk, p, ws, dtype)
    assert torch.equal(q, ref_q)
    for name, got, want in zip("KVA", pools, ref):
        assert torch.equal(got, want), name
    kinds = [act for act, _, _ in p["dst"].values()]
    assert any(kinds) and (not with_kv or not all(kinds)) and len(p["dst"]) < B


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("H,dh,B,bt,with_kv", [PAGED[0], PAGED[5]])
def test_three_launches_replayed_from_a_graph(hk, H, dh, B, bt, with_kv, dtype):
    """Captured once; every replay works on what the buffers hold then (new rows, new destinations, dirty scratch)."""
    p = _paged_inputs(H, dh, B, bt, with_kv, dtype, seed=1)
    need = hk.hk_qkv_workspace_bytes(hk.make_shape(H * dh, H, dtype=hk.HK_DTYPE_BF16 if dtype == torch.bfloat16 else hk.HK_DTYPE_F16), B)
    assert need > 256
    ws, other, pools = hk.new_workspace(need), hk.new_workspace(need), _pools(p, dtype)
    q = torch.empty(B, H, dh, dtype=dtype, device="cuda")
    _paged_call(hk, p, pools, q, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _paged_call(hk, p, pools, q, ws)
    for replay in range(4):
        new = _paged_inputs(H, dh, B, bt, with_kv, dtype, seed=2 + replay)
        for name in ("x", "table", "seq_len", "mask"):
            p[name].copy_(new[name])
        p["dst"] = new["dst"]
        for t, v in zip(pools, (7.0, -7.0, 3.0)):
            t.fill_(v)
        q.fill_(9.0)
        ws.fill_(255)                                                               # NaN in the rows and parts of the last replay
        graph.replay()
        ref_q, ref = _expected(hk, p, other, dtype)
        torch.cuda.synchronize()
        assert torch.equal(q, ref_q), replay
        for name, got, want in zip("KVA", pools, ref):
            assert torch.equal(got, want), (replay, name)
