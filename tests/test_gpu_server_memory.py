"""Memory accounting of the query server: its budget covers all that the server
and its context hold on the device, and the int8 kernels' workspace is held only
once a tuning sends the ticks there."""
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


@pytest.mark.parametrize("q,N,bg,l,n", [(32, 256, 8, 2, 2047), (32, 1024, 7, 3, 255), (32, 2048, 8, 3, 127),
                                        (64, 1024, 6, 4, 127), (64, 2048, 6, 4, 63)])
def test_the_budget_counts_what_is_held(q, N, bg, l, n):
    """(n + 1 words are whole 128-byte lines, so that the rows of the
    key-switching table are as long on the device as they are counted.)"""
    p, ctx = make(q, N, bg, l, n=n)
    fs.Server(ctx, 1 << 36, max_batch=64).close()  # (loads what is loaded once)
    ctx.close()
    torch.cuda.synchronize()
    bsk, ksk = si.torus(3, 95, p.bsk_words(), q), si.torus(4, 95, p.ksk_words(), q)
    before = torch.cuda.mem_get_info()[0]
    ctx = fs.Context(p, bsk, ksk)
    srv = fs.Server(ctx, 1 << 36, max_batch=64)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    counted = srv.bytes_in_use()
    srv.close()
    # held: allocations are rounded up to at most 2 MiB each, about ten of them
    assert abs(held - counted) <= 20 << 20, (held, counted)
    assert p.n * 2 * l * 2 * (N // 2) * 16 * (2 if q == 32 else 3) > 2 * (20 << 20)  # the spectra alone
    with pytest.raises(fs.FheError, match="budget"):
        fs.Server(ctx, counted - 1, max_batch=64)
    fs.Server(ctx, counted, max_batch=64).close()
    ctx.close()


@pytest.mark.parametrize("q,N,bg,l", RINGS)
def test_a_server_retuned_to_the_int8_kernels(q, N, bg, l):
    """The sums of a query served by transforms, of one whose tuning changes to
    int8 products half way, and of one whose budget has no room for their
    workspace (the step fails and changes nothing until the tuning is restored)
    have the same bits."""
    p, ctx = make(q, N, bg, l)
    rows = 5
    col, val = (to_dev(p, si.torus(s, 97, rows * W * (p.n + 1), q).reshape(rows, W, p.n + 1)) for s in (5, 6))
    lit = to_dev(p, si.torus(7, 97, W * (p.n + 1), q).reshape(W, p.n + 1))

    def serve(room, retune_at, restore):
        probe = fs.Server(ctx, 1 << 36, max_batch=64)
        budget = probe.bytes_in_use() + room
        probe.close()
        srv = fs.Server(ctx, budget, max_batch=64)
        out = empty(p, fs.sum_width(W, rows), p.n + 1)
        qid = srv.submit(col, val, rows, W, "lt", lit, out)
        failed, grown = 0, srv.bytes_in_use()
        for tick in range(1000):
            if srv.done(qid):
                break
            if tick == retune_at:
                ctx.set_tuning(split_groups=1 << 20)
            try:
                srv.step()
            except fs.FheError:
                assert restore
                failed += 1
                ctx.set_tuning(split_groups=-1)
        grown = srv.bytes_in_use() - grown
        ctx.set_tuning(split_groups=-1)
        torch.cuda.synchronize()
        assert srv.done(qid)
        srv.close()
        return out, failed, grown
    ref, failed, grown = serve(1 << 30, -1, False)
    assert failed == 0 and grown <= 0
    out, failed, grown = serve(1 << 30, 2, False)
    assert torch.equal(out, ref) and failed == 0 and grown > 0
    out, failed, grown = serve(64 << 10, 2, True)
    assert torch.equal(out, ref) and failed == 1 and grown <= 0
    ctx.close()


def test_the_int8_workspace_gives_way():
    """A server that took the int8 kernels' workspace gives it back when nothing
    runs and a queued query needs the room."""
    p, ctx = make(*RINGS[0])
    rows = 600
    col, val = (to_dev(p, si.torus(s, 97, rows * W * (p.n + 1), p.q).reshape(rows, W, p.n + 1)) for s in (5, 6))
    lit = to_dev(p, si.torus(7, 97, W * (p.n + 1), p.q).reshape(W, p.n + 1))

    def run(srv, count):
        out = empty(p, fs.sum_width(W, count), p.n + 1)
        qid = srv.submit(col[:count], val[:count], count, W, "lt", lit, out)
        for _ in range(20000):
            if srv.done(qid):
                break
            srv.step()
        torch.cuda.synchronize()
        assert srv.done(qid)
        return out
    srv = fs.Server(ctx, 1 << 36, max_batch=64)
    base = srv.bytes_in_use()
    few, many = run(srv, 5), run(srv, rows)
    ctx.set_tuning(split_groups=1 << 20)
    assert torch.equal(run(srv, 5), few)
    srv.step()
    late = srv.bytes_in_use() - base
    srv.close()
    ctx.set_tuning(split_groups=-1)
    srv = fs.Server(ctx, base + late + (64 << 10), max_batch=64)
    ctx.set_tuning(split_groups=1 << 20)
    assert torch.equal(run(srv, 5), few)
    srv.step()
    assert srv.bytes_in_use() == base + late
    ctx.set_tuning(split_groups=-1)
    assert torch.equal(run(srv, rows), many)
    srv.step()
    assert srv.bytes_in_use() == base
    srv.close()
    ctx.close()
