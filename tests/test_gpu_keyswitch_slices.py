"""Key switching of small batches, whose sums are cut into slices added
atomically: the bits of every ciphertext equal those of the same ciphertext in
a batch large enough to run unsliced, and the oracle's, at the edges of the
ciphertext groups and where the slices do not divide the sum."""
import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, from_dev, empty  # noqa: E402


@pytest.mark.parametrize("q,n,N,ks_bits,ks_t", [(32, 70, 1024, 2, 8), (32, 15, 64, 2, 5), (32, 130, 256, 4, 7),
                                                (32, 20, 512, 1, 4), (64, 40, 1024, 3, 6), (64, 17, 64, 4, 2)])
def test_sliced_sums(q, n, N, ks_bits, ks_t):
    p = si.Params("slices", q, n, 1, N, 6, 3, ks_bits, ks_t, 20, 25)
    ksk = si.torus(3, 81, p.ksk_words(), q)
    ctx = fs.Context(p, np.zeros(p.bsk_words(), dtype=np.uint64), ksk)
    big = si.torus(4, 82, 300 * (N + 1), q).reshape(300, N + 1)
    d = to_dev(p, big)
    many = d.repeat(256, 1)  # 76,800 ciphertexts: more than one workgroup per CU
    ref = empty(p, many.shape[0], n + 1)
    ctx.tfhe_keyswitch_batch(many, ref)
    for B in (1, 63, 64, 65, 128, 129, 300):
        out = torch.full_like(empty(p, B, n + 1), 5)
        ctx.tfhe_keyswitch_batch(d[:B].contiguous(), out)
        torch.cuda.synchronize()
        assert torch.equal(out, ref[:B]), B
        g = from_dev(p, out)
        assert np.array_equal(g[B - 1], oracle.keyswitch(p, ksk, big[B - 1])), B
    ctx.close()
