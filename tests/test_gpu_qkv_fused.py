"""QKV generation on either side of the line from which the last wavefront of a tile finishes it in the streaming kernel: both
heights of the row tile that come there, against the definition in 64 bits with the bounds of the form with a finishing
kernel, Q alone (never on that side) with the same bits, and the same bits on every replay of a graph."""
import pytest
import torch

from test_gpu_parity import hk  # noqa: F401
from test_gpu_qkv_stream import test_three_launches_match_the_definition as _match

pytestmark = pytest.mark.gpu
BOTH = [torch.float16, torch.bfloat16]
SIZES = [(48, 128, 128, t) for t in BOTH] + [(49, 128, 97, t) for t in BOTH] + [(50, 128, 97, t) for t in BOTH] + [(51, 128, 128, t) for t in BOTH] \
    + [(56, 128, 113, torch.float16)] + [(65, 128, 96, t) for t in BOTH] + [(66, 128, 65, torch.bfloat16), (67, 128, 96, torch.bfloat16)]


@pytest.mark.parametrize("H,dh,B,dtype", SIZES, ids=["%dx%d-%d-%s" % (h, e, b, str(t)[6:]) for h, e, b, t in SIZES])
def test_wide_parts_match_the_definition(hk, H, dh, B, dtype):
    _match(hk, H, dh, B, dtype)


def test_replays_have_the_bits_of_the_eager_call(hk):
    H, dh, B = 50, 128, 128
    d = H * dh
    gen = torch.Generator(device="cuda").manual_seed(3)
    ln_w, ln_b, bkv, bq, x, Wkv, Wq = (torch.randn(s, generator=gen, device="cuda").mul_(0.1).half()
                                       for s in ((d,), (d,), (2 * d,), (d,), (B, d), (2 * d, d), (d, d)))
    ws = hk.new_workspace(hk.hk_qkv_workspace_bytes(hk.make_shape(d, H), B))
    q = torch.empty(B, H, dh, dtype=torch.float16, device="cuda")
    K, V = (torch.zeros(B, H, 2, dh, dtype=torch.float16, device="cuda") for _ in range(2))

    def call():
        hk.qkv_current(x, ln_w, ln_b, Wkv, bkv, Wq, bq, H, q_out=q, K_dst=K, V_dst=V, tok_pos=1, workspace=ws)

    call()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (q, K, V)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(8):
        q.zero_(), K.zero_(), V.zero_(), ws.fill_(255)          # nothing is left over in the workspace that a call relies on
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((q, K, V), ref))
