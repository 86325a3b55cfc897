"""The transform blind rotation (rings of 1024 and 2048 coefficients, and of 256
at 32-bit words): bit for
bit the int8 path on every ciphertext and the oracle on a few, at the edges of
its launch shapes (one, two or four ciphertexts per workgroup, ragged last
workgroup) and of the gadget (one level, an odd count, more polynomials than
waves, one-bit and eight-bit digits), on inputs at the rounding boundaries,
and with keys and digits of the largest magnitude (the transforms' rounding
error bound is closest there)."""
import sys

import numpy as np
import pytest

import oracle
import seeded_inputs as si
from helpers import edge_lwe

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, from_dev, empty  # noqa: E402


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def both_paths(p, ctx, d, tv=None):
    """Outputs of the default (transform) path and of the int8 path."""
    got, ref = empty(p, d.shape[0], p.N + 1), empty(p, d.shape[0], p.N + 1)
    ctx.tfhe_bootstrap_batch(d, got, testv=tv)
    ctx.set_tuning(split_groups=1 << 20)
    ctx.tfhe_bootstrap_batch(d, ref, testv=tv)
    ctx.set_tuning(split_groups=-1)
    torch.cuda.synchronize()
    return got, ref


@pytest.mark.parametrize("q,N,l,bg", [(32, 1024, 3, 7), (32, 1024, 1, 8), (32, 1024, 5, 6), (32, 1024, 31, 1),
                                      (32, 2048, 3, 8), (32, 2048, 5, 6), (64, 1024, 4, 6), (64, 1024, 1, 8),
                                      (64, 2048, 4, 6), (64, 2048, 3, 8), (64, 2048, 5, 6), (64, 2048, 1, 1),
                                      (32, 256, 2, 8), (32, 256, 1, 8), (32, 256, 3, 7), (32, 256, 31, 1)])
def test_transform_path_parity(q, N, l, bg):
    p = si.Params(f"t{q}_{N}", q, 5, 1, N, bg, l, 2, 8, 20, 25)
    bsk = si.torus(7, 71 + l, p.bsk_words(), q)
    ksk = np.zeros(p.ksk_words(), dtype=np.uint64)
    ctx = fs.Context(p, bsk, ksk)
    tv = oracle.gate_testv(p)
    edge = edge_lwe(p, 72)
    for B in (1, 2, 3, 257, 515, 1539):
        lwe = si.torus(B, 73, B * (p.n + 1), q).reshape(B, p.n + 1)
        if B > len(edge):
            lwe[1:1 + len(edge)] = edge
        say("transform", q, N, l, bg, "B =", B)
        got, ref = both_paths(p, ctx, to_dev(p, lwe))
        assert torch.equal(got, ref), (q, N, l, bg, B)
        if B <= 3:
            g = from_dev(p, got)
            assert np.array_equal(g[B - 1], oracle.bootstrap(p, bsk, lwe[B - 1], tv)), (q, N, l, bg, B)
    ctx.close()


@pytest.mark.parametrize("q,N,l,bg", [(32, 1024, 3, 7), (32, 2048, 3, 8), (64, 1024, 3, 8), (64, 2048, 4, 6),
                                      (64, 2048, 3, 8), (32, 256, 2, 8), (32, 256, 3, 8)])
@pytest.mark.parametrize("sign", [1, -1])
def test_transform_path_largest_sums(q, N, l, bg, sign):
    """Every key limb at the end of its range and, in the first step, every
    digit of the body component at -Bg/2 (the accumulator is half the largest
    negative decomposition and the rotation X^N = -1 doubles it)."""
    M = (1 << q) - 1
    p = si.Params(f"x{q}_{N}", q, 3, 1, N, bg, l, 2, 8, 20, 25)
    widths = (16, 16) if q == 32 else (22, 22, 20)
    word, sh = 0, 0
    for w in widths:
        word += (-(1 << (w - 1)) if sign < 0 else (1 << (w - 1)) - 1) << sh
        sh += w
    bsk = np.full(p.bsk_words(), word & M, dtype=np.uint64)
    ctx = fs.Context(p, bsk, np.zeros(p.ksk_words(), dtype=np.uint64))
    off = sum((1 << (bg - 1)) << (i * bg) for i in range(l)) << (q - l * bg)
    tv = np.full(N, off >> 1, dtype=np.uint64)
    for B in (1, 300, 600):
        lwe = si.torus(B, 74, B * (p.n + 1), q).reshape(B, p.n + 1)
        lwe[:, 0] = 1 << (q - 1)  # abar = N
        lwe[:, p.n] = 0
        say("largest sums", q, N, l, bg, sign, "B =", B)
        got, ref = both_paths(p, ctx, to_dev(p, lwe), tv=to_dev(p, tv))
        assert torch.equal(got, ref), (q, N, l, bg, B)
        assert np.array_equal(from_dev(p, got)[0], oracle.bootstrap(p, bsk, lwe[0], tv))
    ctx.close()


def test_transform_path_look_ups_per_ciphertext():
    """Per-ciphertext test polynomials (radix look-ups) at the 2048-coefficient
    64-bit ring: compare and select of a few rows equal the int8 path's."""
    p = si.Params("tlut", 64, 9, 1, 2048, 6, 4, 3, 6, 20, 51)
    _, _, bsk, ksk = fs.tfhe_keygen(p, si.KEY_SEED_BASE + 75)
    ctx = fs.Context(p, bsk, ksk)
    rows, nb = 5, 3
    col = to_dev(p, si.torus(1, 76, rows * nb * (p.n + 1), 64).reshape(rows, nb, p.n + 1))
    lit = to_dev(p, si.torus(2, 76, nb * (p.n + 1), 64).reshape(nb, p.n + 1))
    outs = []
    for split in (-1, 1 << 20):
        ctx.set_tuning(split_groups=split)
        m, o = empty(p, rows, p.n + 1), empty(p, rows, nb, p.n + 1)
        ctx.sql_radix_mask_scan(col, rows, nb, "lt", lit, m)
        ctx.sql_radix_masked_select(m, col, rows, nb, o)
        torch.cuda.synchronize()
        outs.append((m, o))
    ctx.set_tuning(split_groups=-1)
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    ctx.close()


@pytest.mark.parametrize("knobs,path", [({}, "transform"), ({"row_pass": 16}, "transform"),
                                        ({"split_groups": 0}, "transform"),
                                        ({"row_pass": 16, "split_groups": 0}, "transform"),
                                        ({"row_pass": 8}, "int8"), ({"digit_blocks": 4}, "int8"),
                                        ({"split_groups": 1}, "mixed")])
def test_knobs_and_batch_sizes_keep_the_bits(knobs, path):
    """Every route a knob selects at the 1024-coefficient ring (the transform
    path also for the settings that stood for the old default) gives the same
    bits at batches on both sides of the split threshold."""
    p = si.Params("knobs", 32, 6, 1, 1024, 7, 3, 2, 8, 20, 25)
    ctx = fs.Context(p, si.torus(5, 77, p.bsk_words(), 32), np.zeros(p.ksk_words(), dtype=np.uint64))
    for B in (16, 17, 40):
        d = to_dev(p, si.torus(B, 78, B * (p.n + 1), 32).reshape(B, p.n + 1))
        ref, got = empty(p, B, p.N + 1), empty(p, B, p.N + 1)
        ctx.tfhe_bootstrap_batch(d, ref)
        ctx.set_tuning(**knobs)
        ctx.tfhe_bootstrap_batch(d, got)
        ctx.set_tuning(row_pass=0, digit_blocks=0, split_groups=-1)
        torch.cuda.synchronize()
        assert torch.equal(got, ref), (knobs, path, B)
    ctx.close()


@pytest.mark.parametrize("l,bg", [(2, 8), (3, 7)])
def test_small_ring_batches_on_both_sides_of_the_rule(l, bg):
    """At the 256-coefficient ring the batch decides between the transform and
    the int8 kernel: around the sizes where it changes (and the step sizes of
    the int8 kernel) every ciphertext has the bits it has in a small batch."""
    p = si.Params("small", 32, 9, 1, 256, bg, l, 2, 5, 20, 25)
    bsk = si.torus(11, 79, p.bsk_words(), 32)
    ctx = fs.Context(p, bsk, np.zeros(p.ksk_words(), dtype=np.uint64))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    step = 16 * cus
    top = step + step // 2 + 1
    lwe = si.torus(12, 80, 777 * (p.n + 1), 32).reshape(777, p.n + 1)
    d = to_dev(p, np.tile(lwe, (top // 777 + 1, 1))[:top])
    ref = torch.cat([both_paths(p, ctx, d[:777])[0]] * (top // 777 + 1))[:top]
    tv = oracle.gate_testv(p)
    for i in (0, 776):
        assert np.array_equal(from_dev(p, ref)[i], oracle.bootstrap(p, bsk, lwe[i], tv))
    for B in (step // 2, step // 2 + 1, 12 * cus, 12 * cus + 1, step, step + 1, top - 1, top):
        got = empty(p, B, p.N + 1)
        ctx.tfhe_bootstrap_batch(d[:B].contiguous(), got)
        torch.cuda.synchronize()
        assert torch.equal(got, ref[:B]), B
    ctx.close()


@pytest.mark.parametrize("q,N,l,bg", [(32, 1024, 3, 7), (32, 1024, 5, 6), (32, 2048, 3, 8), (64, 1024, 4, 6),
                                      (64, 2048, 4, 6), (64, 2048, 2, 8)])
def test_batches_that_are_topped_up_with_copies(q, N, l, bg):
    """Batches below the smallest launch are topped up with workgroups that work
    on a ciphertext again and store nothing: around that size every row has the
    int8 path's bits and the memory behind the outputs keeps its own."""
    p = si.Params(f"c{q}_{N}", q, 7, 1, N, bg, l, 2, 8, 20, 25)
    ctx = fs.Context(p, si.torus(13, 81, p.bsk_words(), q), np.zeros(p.ksk_words(), dtype=np.uint64))
    d = to_dev(p, si.torus(14, 82, 70 * (p.n + 1), q).reshape(70, p.n + 1))
    _, ref = both_paths(p, ctx, d)
    for B in (1, 7, 15, 16, 17, 31, 63, 64, 65):
        say("copies", q, N, l, bg, "B =", B)
        buf = torch.full((70, p.N + 1), -7, dtype=d.dtype, device=d.device)
        ctx.tfhe_bootstrap_batch(d[:B].contiguous(), buf[:B])
        torch.cuda.synchronize()
        assert torch.equal(buf[:B], ref[:B]) and bool((buf[B:] == -7).all()), B
    ctx.close()


@pytest.mark.parametrize("l,bg", [(3, 7), (4, 6)])
def test_batches_launched_in_parts(l, bg):
    """Batches of the 1024-coefficient ring whose last round goes out as a
    launch of its own, on both sides of each size where the parts change: every
    row is the int8 path's."""
    p = si.Params("parts", 32, 5, 1, 1024, bg, l, 2, 8, 20, 25)
    ctx = fs.Context(p, si.torus(15, 83, p.bsk_words(), 32), np.zeros(p.ksk_words(), dtype=np.uint64))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    top = 11 * cus + 3
    d = to_dev(p, si.torus(16, 84, 200 * (p.n + 1), 32).reshape(200, p.n + 1)).repeat(top // 200 + 1, 1)[:top].contiguous()
    ref = both_paths(p, ctx, d[:200])[1].repeat(top // 200 + 1, 1)[:top]
    for B in (2 * cus, 2 * cus + 1, 3 * cus, 3 * cus + 1, 4 * cus + 1, 6 * cus, 6 * cus + 1, 7 * cus, 7 * cus + 1,
              8 * cus, 8 * cus + 1, 9 * cus + 1, 10 * cus, 10 * cus + 3, 11 * cus, top):
        say("parts", l, "B =", B)
        buf = torch.full((top, p.N + 1), -7, dtype=d.dtype, device=d.device)
        ctx.tfhe_bootstrap_batch(d[:B], buf[:B])
        torch.cuda.synchronize()
        assert torch.equal(buf[:B], ref[:B]) and bool((buf[B:] == -7).all()), B
    ctx.close()
