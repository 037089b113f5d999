"""Ciphertext division by an inverse taken mod n and lifted to mod n^2: units
next to 0 and n^2, and divisors that are 0 mod n, mod p or mod q only."""
import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 5])
@pytest.mark.parametrize("bits,seed", [(1024, 1), (2048, 2)])
def test_units_and_multiples_of_the_primes(bits, seed, batch):
    import torch
    from paper_2504_03909_amd import he
    print(f"[gpu-case] inverse {bits} batch={batch}", flush=True)
    p, q = P.keygen(bits, seed)
    n = p * q
    n2 = n * n
    k = he.Key.from_primes(bits, p, q)
    units = [1, 2, n2 - 1, n2 - 2, n - 1, n + 1, 5 * n + 1, n2 - n + 1, (1 << 37) + n, n2 >> 1 | 1]
    bad = [0, n, n2 - n, 7 * n, p, q, p * p, q * q, p * q * 3 % n2, 5 * p]
    den = units + bad + units[::-1]
    num = [(3 * i + 7) ** 40 % n2 for i in range(len(den))]

    def dev(v):
        return torch.from_numpy(he.ints_to_limbs(v, 2 * k.limbs)).cuda()
    nb = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = he.hist_subtract(k, dev(num), dev(den), batch=batch, n_bad=nb)
    want = [a * pow(d, -1, n2) % n2 if d % p and d % q else 0 for a, d in zip(num, den)]
    torch.cuda.synchronize()
    assert he.limbs_to_ints(out.cpu().numpy()) == want
    assert int(nb[0]) == len(bad)
