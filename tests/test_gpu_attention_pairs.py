"""The attention with a workgroup per (sequence, head) and the attention cut into ranges, on either side of the rule that
chooses between them: one, two and more steps of 64 tokens in one or two segments, workgroups that hold several pairs and are
partly filled, the lengths and numbers of pairs next to the rule's lines (test_attn_pairs_host.py says which form each of these
sizes takes).  Against softmax attention in 64 bits; the same inputs cut into ranges have to agree: by a number of ranges of the
caller's own, or, on a block table, by columns behind the requests' blocks that give the table room for longer rows.

Tolerance: the scores and sums are fp32 (errors of order 1e-6 here), so what is left is the output's one rounding, at most
2^-11 (fp16) or 2^-8 (bf16) of each element, and with it of the norm."""
import numpy as np
import pytest
import torch

from test_gpu_parity import hk  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = {torch.float16: 2.0 ** -11 + 1e-5, torch.bfloat16: 2.0 ** -8 + 1e-5}

# (sequences, heads, head_dim, cached tokens, tokens of the second segment)
SIZES = [(b, h, dh, n, 0) for b, h, dh in [(1, 1, 128), (1, 5, 64), (3, 3, 128)] for n in (1, 63, 64, 65, 127, 128, 129, 256, 257, 513)]
SIZES += [(1, 6, 64, 1024, 0), (1, 6, 64, 1025, 0), (1, 6, 128, 512, 0), (1, 127, 128, 1000, 0), (1, 128, 128, 1024, 0),
          (1, 128, 128, 1025, 0), (4, 45, 128, 1100, 0), (8, 32, 128, 1500, 0), (1, 257, 64, 1536, 0), (1, 257, 64, 1537, 0),
          (7, 64, 128, 2048, 0), (7, 64, 64, 4097, 0)]
SIZES += [(2, 3, 64, n0, n1) for n0, n1 in [(1, 1), (64, 64), (63, 65), (1, 129), (200, 57), (0, 70), (0, 300), (500, 1), (700, 330)]]


def _reference(q, K, V):
    q, K, V = q.double(), K.double(), V.double()
    p = torch.softmax((K * q[:, :, None]).sum(-1) * q.shape[-1] ** -0.5, -1)
    return (p[..., None] * V).sum(2)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("B,H,dh,L_kv,L_act", SIZES, ids=["%dx%dx%d-%d+%d" % s for s in SIZES])
def test_pairs_against_ranges(hk, B, H, dh, L_kv, L_act, dtype):
    d = H * dh
    gen = torch.Generator(device="cuda").manual_seed(17 * L_kv + L_act + d)

    def draw(*shape, std=1.0, mean=0.0):
        return torch.empty(shape, device="cuda").normal_(mean, std, generator=gen).to(dtype)

    q, K, V = draw(B, H, dh), draw(B, H, L_kv, dh, std=1.5), draw(B, H, L_kv, dh)
    act = draw(B, L_act, d) if L_act else None
    layer = ((draw(d, std=0.02, mean=1.0), draw(d, std=0.02), draw(2 * d, d, std=d ** -0.5), draw(2 * d, std=0.1)) if L_act else
             tuple(torch.zeros(8, device="cuda", dtype=dtype) for _ in range(4)))
    ratio = L_kv / (L_kv + L_act)
    cached = (K, V) if L_kv else (None, None)
    got = hk.hybrid_decode_attn(q, *cached, act, layer, ratio, return_regen=bool(L_act))
    if L_act:
        got, K1, V1 = got
        K, V = torch.cat([K, K1], 2), torch.cat([V, V1], 2)
    ref = _reference(q, K, V)
    cut = hk.hybrid_decode_attn(q, *cached, act, layer, ratio, attn_splits=3)
    for name, out in (("chosen", got), ("ranges", cut)):
        err = float((out.double() - ref).norm() / ref.norm())
        print("%s rel_l2 %.2e" % (name, err), flush=True)
        assert err <= TOL[dtype], name


# (heads, head_dim, request lengths, table columns beyond the longest request's)
PAGED = [(3, 128, [513, 0, 1, 512], 0), (3, 128, [512, 64, 65], 0), (40, 128, [1024, 1000, 513], 0), (43, 128, [1024, 1000, 513], 0),
         (43, 128, [1025, 1000, 513], 0), (64, 128, [2100, 1100, 2000, 700], 0), (86, 64, [1500, 1536, 800], 0),
         (86, 64, [1600, 1536, 800], 0), (64, 64, [4096] * 4 + [17, 0, 2000], 0), (64, 64, [4096] * 3 + [17, 0, 300, 2000], 0),
         (64, 128, [100] * 8, 40), (64, 128, [1000] * 8, 1), (64, 128, [1000] * 8, 200),
         (39, 128, [1100 - 7 * i for i in range(65)], 0), (40, 128, [1100 - 7 * i for i in range(64)], 0), (40, 128, [1100] * 64, 0)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
@pytest.mark.parametrize("bt", [16, 128])
@pytest.mark.parametrize("H,dh,lens,spare", PAGED, ids=["%dx%d-%s-%d" % (h, dh, "_".join(map(str, n)) if len(n) < 9 else "%dx%d_to_%d" % (len(n), n[-1], n[0]), s)
                                               for h, dh, n, s in PAGED])
def test_paged_pairs_against_ranges(hk, H, dh, lens, spare, bt, dtype):
    B = len(lens)
    gen = torch.Generator(device="cuda").manual_seed(sum(lens) + H)

    def draw(*shape, std=1.0):
        return torch.empty(shape, device="cuda").normal_(0, std, generator=gen).to(dtype)

    counts = [(n + bt - 1) // bt for n in lens]
    rng = np.random.default_rng(sum(lens))
    order = rng.permutation(sum(counts))
    room_for_ranges = 4097 * 128 // dh                                   # tokens; what lies behind a request's blocks is never used
    table = np.full((B, max(counts) + spare + room_for_ranges // bt), -12345, np.int32)
    for b, at in enumerate(np.cumsum([0] + counts[:-1])):
        table[b, :counts[b]] = order[at:at + counts[b]]
    K, V = draw(len(order), H, bt, dh, std=1.5), draw(len(order), H, bt, dh)
    q = draw(B, H, dh)
    layer = tuple(torch.zeros(8, device="cuda", dtype=dtype) for _ in range(4))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64, device="cuda")
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    chosen, cut = (hk.paged_decode_attn(q, K, V, None, torch.from_numpy(np.ascontiguousarray(t)).cuda(), lens_dev, bt, layer,
                                        cu_tokens=cu, total_tokens=sum(lens)) for t in (table[:, :max(counts) + spare], table))
    for b, n in enumerate(lens):
        if n == 0:
            assert not chosen[b].any() and not cut[b].any()
            continue
        rows = [t[torch.from_numpy(table[b, :counts[b]]).long().cuda()].transpose(0, 1).reshape(1, H, -1, dh)[:, :, :n] for t in (K, V)]
        ref = _reference(q[b:b + 1], *rows)
        for name, out in (("chosen", chosen), ("ranges", cut)):
            err = float((out[b:b + 1].double() - ref).norm() / ref.norm())
            print("request %d %s rel_l2 %.2e" % (b, name, err), flush=True)
            assert err <= TOL[dtype], name


@pytest.mark.parametrize("H,room", [(64, 1008), (64, 2064)], ids=["pairs", "ranges"])
def test_tokens_known_as_a_bound(hk, H, room):
    """One long request among short ones, and the whole room of the table in the place of the tokens' number."""
    B, dh, bt = 8, 128, 16
    lens = [room - 3] + [5, 16, 0, 17, 1, 64, 33]
    gen = torch.Generator(device="cuda").manual_seed(room)
    K, V = (torch.empty(B * room // bt, H, bt, dh, dtype=torch.float16, device="cuda").normal_(generator=gen) for _ in range(2))
    q = torch.empty(B, H, dh, dtype=torch.float16, device="cuda").normal_(generator=gen)
    table = torch.randperm(len(K), generator=gen, device="cuda", dtype=torch.int64).to(torch.int32).view(B, -1)
    layer = tuple(torch.zeros(8, device="cuda", dtype=torch.float16) for _ in range(4))
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int64, device="cuda")
    out = hk.paged_decode_attn(q, K, V, None, table, torch.tensor(lens, dtype=torch.int32, device="cuda"), bt, layer, cu_tokens=cu,
                               total_tokens=B * room)
    for b, n in enumerate(lens):
        rows = [t[table[b].long()].transpose(0, 1).reshape(1, H, -1, dh)[:, :, :n] for t in (K, V)]
        if n == 0:
            assert not out[b].any()
        else:
            ref = _reference(q[b:b + 1], *rows)
            assert float((out[b:b + 1].double() - ref).norm() / ref.norm()) <= TOL[torch.float16], b


@pytest.mark.parametrize("H,room", [(40, 512), (40, 2048)], ids=["pairs", "ranges"])
def test_a_length_beyond_the_table(hk, H, room):
    """A request whose length is more than its row of the table holds reads no entry of another row: with a workgroup per pair its
    context ends with the row; in ranges the tokens beyond are the last block's, again.  (The row that follows it here is one of
    the same tensor that the call is not given.)"""
    B, dh, bt = 3, 128, 16
    gen = torch.Generator(device="cuda").manual_seed(room)
    cols, over = room // bt, 5 * bt
    K, V = (torch.empty(4 * cols, H, bt, dh, dtype=torch.float16, device="cuda").normal_(generator=gen) for _ in range(2))
    q = torch.empty(B, H, dh, dtype=torch.float16, device="cuda").normal_(generator=gen)
    rows = torch.randperm(4 * cols, generator=gen, device="cuda", dtype=torch.int64).to(torch.int32).view(4, cols)
    layer = tuple(torch.zeros(8, device="cuda", dtype=torch.float16) for _ in range(4))

    def step(table, lens):
        cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int64, device="cuda")
        return hk.paged_decode_attn(q, K, V, None, table, torch.tensor(lens, dtype=torch.int32, device="cuda"), bt, layer,
                                    cu_tokens=cu, total_tokens=sum(lens))

    lens = [room - over - 7, 33, room + over]
    got = step(rows[:B], lens)
    if room == 512:
        want = step(rows[:B], lens[:2] + [room])
        assert torch.equal(got, want)
    else:
        longer = torch.cat([rows[:B], rows[:B, -1:].expand(B, over // bt)], 1).contiguous()
        want = step(longer, lens)
        assert float((got.double() - want.double()).norm() / want.double().norm()) <= TOL[torch.float16]
