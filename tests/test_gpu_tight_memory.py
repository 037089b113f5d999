"""Histograms on a device whose memory holds the ciphertexts but no second copy of
them in the kernels' form: the same results as with it."""
import sys

import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu

LEFT = 700 << 20   # device memory left free


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("bits,seed,rows", [(1024, 1, 1_600_003), (2048, 2, 900_001)])
def test_without_a_second_copy(bits, seed, rows):
    import torch
    from paper_2504_03909_amd import he
    p, q = P.keygen(bits, seed)
    n2 = (p * q) ** 2
    k = he.Key.from_primes(bits, p, q)
    copy = rows * (640 if bits == 1024 else 1152)
    assert copy > LEFT * 5 // 4
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    ct = torch.empty((rows, 2, 2 * k.limbs), dtype=torch.int32, device="cuda").random_(-(1 << 31), (1 << 31) - 1, generator=g)
    ct[..., -1] = 0  # below n^2
    B = 5
    bins = torch.randint(0, B, (1, rows), device="cuda", generator=g).to(torch.uint8)
    bins[0, :40] = 7                       # out of range
    idx = torch.randperm(rows, device="cuda", generator=g).to(torch.int32)
    small = torch.arange(30, 130, dtype=torch.int32, device="cuda")
    want = {}
    for form in (0, 1):
        say(f"{bits} bits, {rows} rows, form {form}, with room")
        want[form] = he.hist_aggregate(k, ct, [he.Job(idx, bins, B), he.Job(small, bins, B)], form=form)
    torch.cuda.synchronize()
    # the two small nodes against Python integers (form 1: the values are x R)
    vals = he.limbs_to_ints(ct[30:130].cpu().numpy())
    t = bins[0, 30:130].cpu().tolist()
    prod = [1] * (2 * B)
    for i, b in enumerate(t):
        if b < B:
            for s in range(2):
                prod[2 * b + s] = prod[2 * b + s] * vals[2 * i + s] % n2
    assert he.limbs_to_ints(want[0][1].cpu().numpy()) == prod
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(free - LEFT, dtype=torch.uint8, device="cuda")
    try:
        side = torch.cuda.Stream()   # a stream whose workspace holds nothing yet
        side.wait_stream(torch.cuda.current_stream())
        for form in (0, 1):
            say(f"{bits} bits, {rows} rows, form {form}, without room")
            jobs = [he.Job(idx, bins, B, torch.empty_like(want[form][0])), he.Job(small, bins, B, torch.empty_like(want[form][1]))]
            with torch.cuda.stream(side):
                got = he.hist_aggregate(k, ct, jobs, form=form)
            side.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, want[form]))
            for j in jobs:
                j.hist.zero_()
            before = torch.cuda.mem_get_info()[0]
            plan = he.HistPlan(k, ct, jobs, form=form)
            assert before - torch.cuda.mem_get_info()[0] < copy // 2   # the plan made do without the copy
            for _ in range(2):
                plan.launch()
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(plan.hists, want[form]))
                for j in jobs:
                    j.hist.zero_()
            plan.close()
    finally:
        del hold
        torch.cuda.empty_cache()
    k.close()


@pytest.mark.parametrize("secret", [False, True])
def test_exponentiations_on_fewer_blocks(secret):
    """200,000 encryptions and their decryption with 320 MB free, a quarter of the
    window tables that fill the device: the ciphertexts and plaintexts of the full
    launches."""
    import torch
    from paper_2504_03909_amd import he
    bits, n = 2048, 200_000
    p, q = P.keygen(bits, 2)
    k = he.Key.from_primes(bits, p, q)
    k.set_constant_time(secret)
    for kind in ("mod_p", "lift", "decrypt"):
        he.crt_set_shape(k, kind, n, 0)
    say(f"{n} encryptions with room, secret={secret}")
    m = torch.from_numpy(np.random.default_rng(4).integers(-(1 << 62), 1 << 62, size=n, dtype=np.int64)).cuda()
    ct = he.encrypt(k, m, seed=17)
    out, back = torch.empty_like(ct), torch.empty_like(m)
    overflow = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(free - (320 << 20), dtype=torch.uint8, device="cuda")
    try:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        say("without room")
        he.encrypt(k, m, seed=17, out=out, stream=side)
        he._check(he._decrypt(k.handle, he._ptr(out), n, he._ptr(back), None, he._ptr(overflow), side.cuda_stream))
        side.synchronize()
    finally:
        del hold
        torch.cuda.empty_cache()
    assert torch.equal(out, ct) and torch.equal(back, m) and int(overflow.item()) == 0
    k.close()
