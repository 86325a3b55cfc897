"""A kept graph of sql_scan_batch belongs to the tuning it was captured under:
changing any knob that can change a launch captures anew (also a split threshold
that covers the narrow levels only and leaves the workspace's size as it is),
going back relaunches the earlier graph, and every run gives the same bits."""
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, empty  # noqa: E402


@pytest.mark.parametrize("knob", [{"split_groups": 4}, {"digit_blocks": 4}, {"row_pass": 2}, {"max_batch": 50}])
def test_a_changed_knob_captures_anew(knob):
    p = si.Params("graph", 32, 20, 1, 256, 8, 2, 2, 5, 20, 25)
    ctx = fs.Context(p, si.torus(3, 93, p.bsk_words(), 32), si.torus(4, 93, p.ksk_words(), 32))
    rows, w = 40, 20
    col = to_dev(p, si.torus(5, 94, rows * w * (p.n + 1), 32).reshape(rows, w, p.n + 1))
    lit = to_dev(p, si.torus(6, 94, w * (p.n + 1), 32).reshape(w, p.n + 1))
    mask = empty(p, rows, p.n + 1)
    q = [dict(col=col, rows=rows, w=w, op="eq", lit_a=lit, mask=mask)]
    # a batch that needs the largest workspace first, so that no later one grows it
    ctx.set_tuning(row_pass=2, split_groups=4)
    ctx.sql_mask_scan(col, rows, w, "eq", lit, mask)
    ctx.set_tuning(row_pass=0, split_groups=-1)
    defaults = {"split_groups": -1, "digit_blocks": 0, "row_pass": 0, "max_batch": 65536}
    captures, bits = [], []
    for setting in ({}, knob, {}, knob):
        ctx.set_tuning(**{**defaults, **setting})
        mask.fill_(7)
        ctx.sql_scan_batch(q, use_graph=True)
        torch.cuda.synchronize()
        captures.append(ctx.graph_stats()[0])
        bits.append(mask.clone())
    assert captures == [1, 2, 2, 2]
    assert all(torch.equal(b, bits[0]) for b in bits)
    ctx.close()
