"""One call whose grid would have 2^32 work-items in a single launch: 2^23 and a
few ciphertexts at the rings where a workgroup of 512 threads takes one.  The
inputs repeat every 1009 rows, and every output row holds the words of its input
alone."""
import sys

import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, empty  # noqa: E402


@pytest.mark.parametrize("q,N,bg,l", [(64, 1024, 6, 2), (32, 2048, 8, 1)])
def test_a_call_of_more_than_one_grid(q, N, bg, l):
    p = si.Params("huge", q, 1, 1, N, bg, l, 2, 8, 20, 25)
    B, period = (1 << 23) + 5, 1009
    if torch.cuda.mem_get_info()[0] < int(1.2 * B * (N + 1) * (q // 8)):
        pytest.skip("the outputs (69 GB) do not fit")
    ctx = fs.Context(p, si.torus(3, 98, p.bsk_words(), q), si.torus(4, 98, p.ksk_words(), q))
    few = to_dev(p, si.torus(5, 98, period * (p.n + 1), q).reshape(period, p.n + 1))
    ref = empty(p, period, N + 1)
    ctx.tfhe_bootstrap_batch(few, ref)
    many = few.repeat(B // period + 1, 1)[:B].contiguous()
    out = empty(p, B, N + 1)
    print("huge batch", q, N, "B =", B, flush=True)
    sys.stdout.flush()
    ctx.tfhe_bootstrap_batch(many, out)
    torch.cuda.synchronize()
    for r0 in range(0, B, 512 * period):  # (compared in place, 2 GB at a time)
        rows = out[r0:r0 + 512 * period]
        whole = rows.shape[0] // period
        assert bool((rows[:whole * period].view(whole, period, N + 1) == ref).all()), r0
        tail = rows.shape[0] - whole * period
        assert torch.equal(rows[whole * period:], ref[:tail]), r0
    del out, many, rows
    torch.cuda.empty_cache()
    ctx.close()
