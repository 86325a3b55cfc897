"""Gates of one launch that write the same output row: batches that hold the
same query twice, or two queries whose row ranges overlap, into one buffer, and
a server query submitted twice with one result buffer.  All of them compute the
same words for that row, so it holds the words it holds when one of them runs
alone, whichever form of the key switch runs (small launches cut its sums into
slices that are added up)."""
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, empty  # noqa: E402

W = 3
# (key-switch form) int8 products, int8 products at b = 2 and t = 8, gathered rows
SETS = [(32, 64, 256, 8, 2, 2, 5), (32, 33, 1024, 7, 3, 2, 8), (64, 17, 64, 6, 3, 3, 6)]


def make(q, n, N, bg, l, ks_bits, ks_t):
    p = si.Params("shared", q, n, 1, N, bg, l, ks_bits, ks_t, 20, 25)
    ctx = fs.Context(p, si.torus(3, 91, p.bsk_words(), q), si.torus(4, 91, p.ksk_words(), q))
    rows = 60
    col, sel = (to_dev(p, si.torus(s, 92, rows * W * (n + 1), q).reshape(rows, W, n + 1)) for s in (5, 6))
    lit = to_dev(p, si.torus(7, 92, W * (n + 1), q).reshape(W, n + 1))
    return p, ctx, col, sel, lit


@pytest.mark.parametrize("pset", SETS)
@pytest.mark.parametrize("use_graph", [False, True])
def test_queries_of_a_batch_share_their_outputs(pset, use_graph):
    p, ctx, col, sel, lit = make(*pset)

    def query(mask, out, r0, r1):
        return dict(col=col[r0:r1], sel_col=sel[r0:r1], rows=r1 - r0, w=W, op="lt", lit_a=lit, mask=mask[r0:r1],
                    sel_out=out[r0:r1])
    ref = empty(p, 60, p.n + 1), empty(p, 60, W, p.n + 1)
    ctx.sql_scan_batch([query(*ref, 0, 60)], use_graph=False)
    for ranges in (((0, 60), (0, 60)), ((0, 40), (20, 60)), ((0, 1), (0, 60), (0, 60))):
        got = torch.full_like(ref[0], 3), torch.full_like(ref[1], 3)
        ctx.sql_scan_batch([query(*got, r0, r1) for r0, r1 in ranges], use_graph=use_graph)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), ranges
    ctx.close()


@pytest.mark.parametrize("pset", SETS)
def test_a_server_query_submitted_twice(pset):
    p, ctx, col, sel, lit = make(*pset)
    rows = 5
    sums = []
    for times in (1, 2):
        srv = fs.Server(ctx, 1 << 34, max_batch=512)
        out = torch.full_like(empty(p, fs.sum_width(W, rows), p.n + 1), 3)
        ids = [srv.submit(col[:rows], sel[:rows], rows, W, "eq", lit, out) for _ in range(times)]
        for _ in range(1000):
            if all([srv.done(i) for i in ids]):
                break
            srv.step()
        torch.cuda.synchronize()
        srv.close()
        sums.append(out)
    assert torch.equal(sums[0], sums[1])
    ctx.close()
