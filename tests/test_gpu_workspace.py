"""The transform blind rotation takes no workspace: a large batch leaves the
context's workspace, and the graphs kept on it, alone; and calls on different
streams still run in the order they were made."""
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, empty  # noqa: E402

W = 2
RINGS = [(32, 1024, 7, 3), (32, 2048, 8, 3), (64, 1024, 6, 4), (64, 2048, 6, 4)]


def make(q, N, bg, l, n=7, seed=95):
    p = si.Params("ws", q, n, 1, N, bg, l, 2, 3, 20, 25)
    return p, fs.Context(p, si.torus(3, seed, p.bsk_words(), q), si.torus(4, seed, p.ksk_words(), q))


@pytest.mark.parametrize("q,N,bg,l", RINGS)
def test_a_large_batch_leaves_the_kept_graph(q, N, bg, l):
    p, ctx = make(q, N, bg, l)
    rows = 6
    col = to_dev(p, si.torus(5, 96, rows * W * (p.n + 1), q).reshape(rows, W, p.n + 1))
    lit = to_dev(p, si.torus(6, 96, W * (p.n + 1), q).reshape(W, p.n + 1))
    mask = empty(p, rows, p.n + 1)
    queries = [dict(col=col, rows=rows, w=W, op="eq", lit_a=lit, mask=mask)]
    ctx.sql_scan_batch(queries, use_graph=True)
    torch.cuda.synchronize()
    ref = mask.clone()
    # (B int8 accumulators would be 8 to 32 KB each)
    B = 3000
    ctx.tfhe_bootstrap_batch(to_dev(p, si.torus(7, 96, B * (p.n + 1), q).reshape(B, p.n + 1)), empty(p, B, N + 1))
    mask.fill_(0)
    ctx.sql_scan_batch(queries, use_graph=True)
    torch.cuda.synchronize()
    assert ctx.graph_stats() == (1, 2, 1)
    assert torch.equal(mask, ref)
    ctx.close()


@pytest.mark.parametrize("q,N,bg,l", RINGS)
def test_calls_on_two_streams_stay_in_order(q, N, bg, l):
    """A key switch on one stream reads what the bootstrap before it on another
    one wrote (the calls of a context are serialized on the device)."""
    p, ctx = make(q, N, bg, l, n=200)
    B = 1024
    d = to_dev(p, si.torus(8, 96, B * (p.n + 1), q).reshape(B, p.n + 1))
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    big, ref, got = empty(p, B, N + 1), empty(p, B, p.n + 1), empty(p, B, p.n + 1)
    ctx.tfhe_bootstrap_batch(d, big)
    ctx.tfhe_keyswitch_batch(big, ref)
    torch.cuda.synchronize()
    for _ in range(3):
        big.fill_(0)
        got.fill_(0)
        torch.cuda.synchronize()
        ctx.tfhe_bootstrap_batch(d, big, stream=s1)
        ctx.tfhe_keyswitch_batch(big, got, stream=s2)
        torch.cuda.synchronize()
        assert torch.equal(got, ref)
    ctx.close()
