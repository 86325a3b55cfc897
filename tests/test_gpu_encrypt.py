"""Device encryption, one wave per ciphertext: word for word the oracle's at
dimensions around the 64 lanes of a wave and at counts around the four
ciphertexts of a workgroup, from any start of the stream."""
import numpy as np
import pytest

import oracle
import seeded_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_15413_amd as fs  # noqa: E402
from paper_2510_15413_amd import client  # noqa: E402
from gpu_util import to_dev, from_dev  # noqa: E402


@pytest.mark.parametrize("q", [32, 64])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 630])
def test_encrypt_matches_oracle(q, n):
    p = si.Params("enc", q, n, 1, 64, 8, 2, 2, 5, 20, 25)
    s = si.bits(9, si.TAG_LWE_KEY, n)
    for count, start in ((1, 0), (4, 3), (5, 7), (130, 1)):
        bits = si.bits(count, 91, count)
        masks, errs = si.lwe_randomness(p, 92, count, tag_hi=2, start=start)
        eighth = 1 << (q - 3)
        mus = np.where(bits == 1, eighth, (-eighth) & ((1 << q) - 1)).astype(np.uint64)
        got = client.encrypt_bits(p, 92, to_dev(p, s), torch.from_numpy(bits.astype(np.int64)), tag_hi=2, start=start)
        assert np.array_equal(from_dev(p, got), oracle.lwe_encrypt(p, s, masks, errs, mus)), (q, n, count, start)
        assert torch.equal(client.decrypt_bits(p, to_dev(p, s), got).cpu(), torch.from_numpy(bits.astype(np.int64)))
