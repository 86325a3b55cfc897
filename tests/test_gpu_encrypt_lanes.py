"""Device encryption by 1, 4, 16 or 64 lanes per ciphertext: word for word the
oracle's at the dimensions where the number of lanes changes and at counts around
a workgroup's ciphertexts; and the time follows the words (short ciphertexts do
not pay for a whole wave each)."""
import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from gpu_util import to_dev, from_dev  # noqa: E402


@pytest.mark.parametrize("q", [32, 64])
@pytest.mark.parametrize("n", [1, 3, 8, 9, 31, 32, 33, 64, 65])
def test_words_at_every_number_of_lanes(q, n):
    p = si.Params("enc", q, n, 1, 64, 8, 2, 2, 5, 20, 25)
    s = si.bits(9, si.TAG_LWE_KEY, n)
    for count, start in ((1, 0), (15, 2), (16, 0), (17, 5), (63, 1), (64, 0), (65, 9), (255, 0), (257, 3)):
        masks, errs = si.lwe_randomness(p, 93, count, tag_hi=2, start=start)
        mus = si.torus(94, 95, count, q)
        got = fs.tfhe_lwe_encrypt(p, 93, to_dev(p, s), to_dev(p, mus), start=start, tag_hi=2)
        assert np.array_equal(from_dev(p, got), oracle.lwe_encrypt(p, s, masks, errs, mus)), (q, n, count, start)


def test_time_follows_the_words():
    """10^6 ciphertexts of 8 words write a seventh of what those of 64 write."""
    best = {}
    for n in (8, 64):
        p = si.Params("enc", 32, n, 1, 64, 8, 2, 2, 5, 20, 25)
        key = torch.ones(n, dtype=torch.int32, device="cuda")
        mu = torch.zeros(1000000, dtype=torch.int32, device="cuda")
        times = []
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fs.tfhe_lwe_encrypt(p, 1, key, mu)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        best[n] = min(times)
    assert best[8] < 0.6 * best[64], best
