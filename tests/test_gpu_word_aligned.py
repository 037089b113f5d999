"""Ciphertext buffers aligned to a 32-bit word only (a view into a larger array):
every path gives what it gives on aligned buffers."""
import sys

import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("bits,seed", [(1024, 1), (2048, 2)])
@pytest.mark.parametrize("count", [6, 20_000])   # groups of lanes per integer; one or two lanes
def test_views_at_odd_words(bits, seed, count):
    import torch
    from paper_2504_03909_amd import he
    p, q = P.keygen(bits, seed)
    k = he.Key.from_primes(bits, p, q)
    L = k.limbs

    def odd(t):
        buf = torch.empty(t.numel() + 1, dtype=torch.int32, device="cuda")
        v = buf[1:].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 8 == 4
        return v

    rng = np.random.default_rng(count)
    m = torch.from_numpy(rng.integers(-(1 << 62), 1 << 62, size=count, dtype=np.int64)).cuda()
    say(f"{bits} bits, {count}: encryption")
    ct = he.encrypt(k, m, seed=5)
    out = odd(torch.zeros_like(ct))
    he.encrypt(k, m, seed=5, out=out)
    assert torch.equal(out, ct)
    r = torch.from_numpy(he.ints_to_limbs([3 + i for i in range(count)], L)).cuda()
    assert torch.equal(he.encrypt(k, m, r=odd(r)), he.encrypt(k, m, r=r))
    few = min(count, 600)
    he.encrypt(k, m[:few], seed=5, public=True, out=out[:few])
    assert torch.equal(out[:few], ct[:few])
    say("decryption, packing, products")
    v = odd(ct)
    assert torch.equal(he.decrypt(k, v)[0], m)
    back = torch.empty_like(m)
    he.decrypt_noalloc(k, v, back)
    assert torch.equal(back, m)
    for slots in (1, 3):
        packed, _ = he.pack(k, v, slots)
        assert torch.equal(packed, he.pack(k, ct, slots)[0])
        assert torch.equal(he.decrypt_packed(k, odd(packed), count, slots)[0], m)
    assert torch.equal(he.ct_mul(k, v, v), he.ct_mul(k, ct, ct))
    assert torch.equal(he.hist_subtract(k, v, v.flip(0)), he.hist_subtract(k, ct, ct.flip(0)))
    assert torch.equal(he.to_mont(k, v), he.to_mont(k, ct))
    say("histograms")
    rows = count // 2
    bins = torch.from_numpy(rng.integers(0, 7, size=(2, rows)).astype(np.uint8)).cuda()
    for n in (rows, rows // 2 + 1):
        idx = torch.arange(n, dtype=torch.int32, device="cuda")
        for form, x in ((0, ct), (1, he.to_mont(k, ct))):
            want = he.hist_aggregate(k, x.view(rows, 2, -1), [he.Job(idx, bins, 7)], form=form)[0]
            j = he.Job(idx, bins, 7, odd(torch.zeros_like(want)))
            assert torch.equal(he.hist_aggregate(k, odd(x).view(rows, 2, -1), [j], form=form)[0], want)
    k.close()
