"""The two-digit exponentiations (one, two or 2 G lanes per integer) against
Python integers, at counts whose default plans use every width and a second
launch for the rest, with r at the edges of its range and not a unit mod p or
q (results 0 or a multiple of the prime, where a digit is 0 or the base)."""
import sys

import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def he():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2504_03909_amd import he as H
    return H


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


# The default plans put a wave on every SIMD first (65,536 lanes), so with two
# primes 32,768 ciphertexts fill one lane each, 16,384 two, ..., and the
# remainders go to a wider launch.
COUNTS = [1, 7, 2048 + 3, 4096 + 9, 16384 + 5, 32768 + 3]


@pytest.mark.parametrize("public", [False, True])
@pytest.mark.parametrize("bits,seed", [(1024, 1), (2048, 2)])
def test_widths_and_edge_r(he, bits, seed, public):
    import torch
    p, q = P.keygen(bits, seed)
    n = p * q
    n2 = n * n
    k = he.Key.from_primes(bits, p, q)
    L = k.limbs
    rng = np.random.default_rng(bits + public)
    edge_r = [1, n - 1, p, q, n - p, 3 * q, (1 << (bits - 1)) % n]
    for count in COUNTS if not (public and bits == 2048) else COUNTS[:4]:
        say(f"two-digit exponentiations: {bits} bits, public={public}, {count}")
        m = rng.integers(-(1 << 62), 1 << 62, size=count, dtype=np.int64)
        r = rng.integers(0, 1 << 32, size=(count, L), dtype=np.uint64).astype(np.uint32).view(np.int32)
        r[:, -1] = 0  # below n
        where = sorted(set(list(range(min(count, len(edge_r)))) + list(range(max(0, count - len(edge_r)), count))))
        for j, i in enumerate(where):
            r[i] = he.ints_to_limbs([edge_r[j % len(edge_r)]], L)[0]
        ct = he.encrypt(k, dev(m), r=dev(r), public=public)
        pick = sorted(set(where) | set(rng.choice(count, size=min(count, 4), replace=False).tolist()))
        rows = host(ct)[pick]
        want = [(1 + int(m[i]) * n) * pow(he.limbs_to_ints(r[i][None])[0], n, n2) % n2 for i in pick]
        assert he.limbs_to_ints(rows) == want
        if not public:
            if count < 5000:
                assert torch.equal(ct, he.encrypt(k, dev(m), r=dev(r), public=True))
            unit = np.ones(count, dtype=bool)
            for j, i in enumerate(where):
                unit[i] = edge_r[j % len(edge_r)] % p != 0 and edge_r[j % len(edge_r)] % q != 0
            dm = host(he.decrypt(k, ct)[0])
            assert (dm[unit] == m[unit]).all()
    k.close()


def test_constant_time_at_every_width(he):
    """Masked table reads (fixed windows) give the default path's results
    with one and two lanes per integer as well."""
    import torch
    bits = 1024
    p, q = P.keygen(bits, 1)
    ref, k = he.Key.from_primes(bits, p, q), he.Key.from_primes(bits, p, q)
    k.set_constant_time(True)
    rng = np.random.default_rng(3)
    for count in COUNTS[2:]:
        say(f"constant time, {count}")
        m = dev(rng.integers(-(1 << 62), 1 << 62, size=count, dtype=np.int64))
        ct = he.encrypt(ref, m, seed=4)
        assert torch.equal(ct, he.encrypt(k, m, seed=4))
        assert torch.equal(he.decrypt(k, ct)[0], m)
