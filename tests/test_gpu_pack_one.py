"""Packing one ciphertext to one: c (1 + 2^63 n) mod n^2 for ciphertexts at the
ends of the range and multiples of n, into another buffer and in place."""
import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,seed", [(1024, 1), (2048, 2)])
@pytest.mark.parametrize("count", [1, 16, 37])
def test_one_slot(bits, seed, count):
    import torch
    from paper_2504_03909_amd import he
    p, q = P.keygen(bits, seed)
    n = p * q
    n2 = n * n
    print(f"[gpu-case] pack one slot {bits} {count}", flush=True)
    k = he.Key.from_primes(bits, p, q)
    rng = np.random.default_rng(count)
    vals = ([n2 - 1, 0, 1, n, n2 - n, n + 1] + [int.from_bytes(rng.bytes(bits // 4), "little") % n2 for _ in range(count)])[:count]
    ct = torch.from_numpy(he.ints_to_limbs(vals, 2 * k.limbs)).cuda()
    want = [c * (1 + (1 << 63) * n) % n2 for c in vals]
    packed, _ = he.pack(k, ct, 1)
    assert he.limbs_to_ints(packed.cpu().numpy()) == want
    he._check(he._pack(k.handle, he._ptr(ct), count, 1, he._ptr(ct), he._stream(None)))
    assert he.limbs_to_ints(ct.cpu().numpy()) == want
    k.close()
