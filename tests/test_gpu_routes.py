"""Which kernels a blind rotation runs on: every knob that chooses between the
transforms and the int8 kernels, the batch sizes where the choice changes, the
rings that have no transforms, and the pair of settings by which the parity
tests compare the two; each with the bits of the plain kernel."""
import numpy as np
import pytest

import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, empty  # noqa: E402

DEFAULTS = {"row_pass": 0, "digit_blocks": 0, "split_groups": -1}
RINGS = [(32, 1024, 7, 3), (32, 2048, 8, 3), (64, 1024, 6, 4), (64, 2048, 6, 4)]
DEFAULT_ROW_PASS = {(32, 1024): 16, (32, 2048): 8, (64, 1024): 4, (64, 2048): 8}
OTHER_ROW_PASS = {(32, 1024): 8, (64, 2048): 4}


def make(q, N, bg, l):
    p = si.Params("route", q, 3, 1, N, bg, l, 2, 8, 20, 25)
    ctx = fs.Context(p, si.torus(3, 99, p.bsk_words(), q), np.zeros(p.ksk_words(), dtype=np.uint64))
    d = to_dev(p, si.torus(4, 99, 40 * (p.n + 1), q).reshape(40, p.n + 1))
    ctx.set_kernel("plain")
    assert ctx.blind_rotation_route(1) == "plain"
    ref = empty(p, 40, N + 1)
    ctx.tfhe_bootstrap_batch(d, ref)
    ctx.set_kernel("mfma")

    def routes(batches=(1, 16, 17, 40), **knobs):
        ctx.set_tuning(**{**DEFAULTS, **knobs})
        for B in batches:
            if B <= 40:
                got = empty(p, B, N + 1)
                ctx.tfhe_bootstrap_batch(d[:B], got)
                torch.cuda.synchronize()
                assert torch.equal(got, ref[:B]), (knobs, B)
        found = [ctx.blind_rotation_route(B) for B in batches]
        ctx.set_tuning(**DEFAULTS)
        return found
    return ctx, routes


@pytest.mark.parametrize("q,N,bg,l", RINGS)
def test_knobs_of_the_transform_rings(q, N, bg, l):
    ctx, routes = make(q, N, bg, l)
    T, I = ["transform"] * 4, ["int8"] * 4
    assert routes() == T
    assert routes(split_groups=0) == T
    assert routes(row_pass=DEFAULT_ROW_PASS[q, N]) == T
    assert routes(row_pass=DEFAULT_ROW_PASS[q, N], split_groups=0) == T
    assert routes(digit_blocks=1) == I
    assert routes(digit_blocks=4, split_groups=0) == I
    if (q, N) in OTHER_ROW_PASS:
        assert routes(row_pass=OTHER_ROW_PASS[q, N]) == I
    assert routes(split_groups=1) == ["int8", "int8", "transform", "transform"]
    assert routes(split_groups=2) == ["int8", "int8", "int8", "transform"]
    assert routes(split_groups=1 << 20) == I  # (the other side of the parity tests)
    ctx.close()


@pytest.mark.parametrize("l,bg", [(2, 8), (1, 8), (3, 7)])
def test_batches_of_the_small_ring(l, bg):
    ctx, routes = make(32, 256, bg, l)
    step = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    if l == 2:
        want = {1: 1, step * 3 // 4: 1, step * 3 // 4 + 1: 0, step: 0, step + 1: 1, step * 3 // 2: 1,
                step * 3 // 2 + 1: 0, 2 * step: 0, 2 * step + 1: 1, 4 * step + step // 2: 1, 4 * step + step // 2 + 1: 0,
                5 * step + 1: 0, 16 * step: 0}
    else:
        want = {1: 1, step // 2: 1, step // 2 + 1: 0, step: 0, step + 1: 0, 16 * step: 0}
    assert routes(tuple(want)) == ["transform" if t else "int8" for t in want.values()]
    assert routes(row_pass=4) == ["transform"] * 4 and routes(row_pass=2) == ["int8"] * 4
    assert routes(split_groups=1) == ["int8", "int8", "transform", "transform"]
    ctx.close()


@pytest.mark.parametrize("q,N,bg,l", [(32, 64, 8, 2), (32, 512, 7, 3), (64, 64, 6, 4), (64, 256, 6, 4),
                                      (64, 512, 6, 4)])
def test_rings_without_transforms(q, N, bg, l):
    ctx, routes = make(q, N, bg, l)
    assert routes() == ["int8"] * 4
    ctx.close()
