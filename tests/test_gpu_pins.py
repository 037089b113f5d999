"""The private-key exponentiations at pinned widths, the pins taken back around
every case, so that the width a case names is the width it runs: r at the edges
of its range and not a unit mod p or q, with plain and with masked tables, and
the shapes the autotuner returns for the benchmark's counts."""
import sys

import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu

KINDS = ("mod_p", "lift", "decrypt")


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def he():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2504_03909_amd import he as H
    return H


@pytest.fixture
def pins(he):
    """pin(key, kind, count, lanes, waves, tail); every pin is taken back."""
    made = []

    def pin(key, kind, count, *shape):
        he.crt_set_shape(key, kind, count, *shape)
        made.append((key, kind, count))
    yield pin
    for key, kind, count in made:
        he.crt_set_shape(key, kind, count, 0)


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


# one unit of 64 integers and a short one, then less than a unit
@pytest.mark.parametrize("count", [67, 5])
@pytest.mark.parametrize("secret", [False, True])
@pytest.mark.parametrize("bits,lanes", [(1024, 1), (1024, 2), (2048, 1), (2048, 4), (2048, 16)])
def test_edge_r_at_a_pinned_width(he, pins, bits, lanes, secret, count):
    p, q = P.keygen(bits, 1 if bits == 1024 else 2)
    n = p * q
    n2 = n * n
    k = he.Key.from_primes(bits, p, q)
    k.set_constant_time(secret)
    say(f"pinned width: {bits} bits, {lanes} lanes, secret={secret}, {count}")
    for kind in KINDS:
        pins(k, kind, count, lanes, 0, 0)
    rng = np.random.default_rng(bits + lanes)
    m = rng.integers(-(1 << 62), 1 << 62, size=count, dtype=np.int64)
    r = rng.integers(0, 1 << 32, size=(count, k.limbs), dtype=np.uint64).astype(np.uint32).view(np.int32)
    edge = [1, n - 1, p, n - q, 0][:count]
    r[:len(edge)] = he.ints_to_limbs(edge, k.limbs)
    ct = he.encrypt(k, dev(m), r=dev(r))
    ri = he.limbs_to_ints(r)
    assert he.limbs_to_ints(host(ct)) == [(1 + int(a) * n) * pow(b, n, n2) % n2 for a, b in zip(m, ri)]
    unit = np.array([b % p != 0 and b % q != 0 for b in ri])
    dm = host(he.decrypt(k, ct)[0])
    assert (dm[unit] == m[unit]).all()
    m2 = dev(np.zeros(count, dtype=np.int64))
    he.decrypt_noalloc(k, ct, m2)
    assert (host(m2)[unit] == m[unit]).all()


@pytest.mark.parametrize("secret", [False, True])
def test_default_plans_of_two_launches(he, pins, secret):
    """A round of waves at two lanes (masked tables too), and counts just above one
    at two lanes and at one (2048 bits), with no pin in their class: whole waves at a
    narrow width, the rest at a wide one."""
    import torch
    bits = 2048
    p, q = P.keygen(bits, 2)
    n = p * q
    n2 = n * n
    k = he.Key.from_primes(bits, p, q)
    k.set_constant_time(secret)
    rng = np.random.default_rng(7)
    for count in (16384, 16384 + 5, 32768 + 3):
        say(f"default plan, {count}, secret={secret}")
        for kind in KINDS:
            pins(k, kind, count, 0)
        m = dev(rng.integers(-(1 << 62), 1 << 62, size=count, dtype=np.int64))
        ct = he.encrypt(k, m, seed=21)
        pick = [0, 1, count // 2, count - 6, count - 1]
        mh = host(m)
        want = [(1 + int(mh[i]) * n) * pow(P.seeded_r(n, bits, 21, i), n, n2) % n2 for i in pick]
        assert he.limbs_to_ints(host(ct)[pick]) == want
        assert torch.equal(he.decrypt(k, ct)[0], m)


def test_tuned_shapes_of_the_benchmark_counts_can_be_pinned(he, pins):
    """he_crt_autotune at 200,000 encryptions and 16,384 decryptions returns shapes
    that he_crt_set_shape takes, with the same ciphertexts and plaintexts."""
    import torch
    bits, enc, dec = 2048, 200_000, 16_384
    p, q = P.keygen(bits, 2)
    k = he.Key.from_primes(bits, p, q)
    say("pinning what the autotuner returned")
    for kind, count in zip(KINDS, (enc, enc, dec)):
        pins(k, kind, count, 0)
    m = dev(np.random.default_rng(8).integers(-(1 << 62), 1 << 62, size=enc, dtype=np.int64))
    ct = he.encrypt(k, m, seed=3)
    tuned = he.crt_autotune(k, enc, dec)
    say(f"tuned: {tuned}")
    assert torch.equal(he.encrypt(k, m, seed=3), ct)
    for kind, count in zip(KINDS, (enc, enc, dec)):
        pins(k, kind, count, 0)
        pins(k, kind, count, *tuned[kind][:3])
    assert torch.equal(he.encrypt(k, m, seed=3), ct)
    assert torch.equal(he.decrypt(k, ct[:dec])[0], m[:dec])
