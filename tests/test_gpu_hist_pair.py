"""Histogram products in two digits base n against products of Python
integers: every resident row converted or only the jobs' samples (gathered),
from canonical and from Montgomery form, with an empty job between others,
repeated rows, rows and bins out of range, and every number of runs per item
around the item length."""
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


@pytest.mark.parametrize("rows", [40, 90])   # 60 samples: all rows, or the samples gathered
@pytest.mark.parametrize("bits,seed", [(1024, 1), (2048, 2)])
def test_jobs_against_integer_products(he, bits, seed, rows):
    import torch
    say(f"two-digit histograms, {bits} bits, {rows} rows")
    p, q = P.keygen(bits, seed)
    n = p * q
    n2 = n * n
    k = he.Key.from_primes(bits, p, q)
    rng = np.random.default_rng(bits + rows)
    # any residues mod n^2, the ends of the range and multiples of n among them
    vals = [int.from_bytes(rng.bytes(bits // 4), "little") % n2 for _ in range(2 * rows)]
    for j, v in enumerate([0, 1, n2 - 1, n, n2 - n, n - 1, n + 1]):
        vals[3 * j] = v
    ct = dev(he.ints_to_limbs(vals, 2 * k.limbs)).view(rows, 2, -1)
    shapes = [(35, 3, 7), (0, 2, 5), (1, 1, 1), (24, 2, 256)]   # samples, features, bins
    idx, tabs = [], []
    for m, F, B in shapes:
        ix = rng.integers(0, rows, size=m)
        if m > 20:
            ix[:7] = ix[7]                # repeated
            ix[10], ix[15] = rows, 2 ** 31  # not resident
        idx.append(ix.astype(np.uint32).view(np.int32))
        t = rng.integers(0, min(B, 4), size=(F, rows)).astype(np.uint8)
        if B < 256:
            t[:, rng.integers(0, rows, size=3)] = 255  # out of range
        tabs.append(t)
    want = []
    for (m, F, B), ix, t in zip(shapes, idx, tabs):
        h = [[[1, 1] for _ in range(B)] for _ in range(F)]
        for r in ix.view(np.uint32).tolist():
            for f in range(F):
                if r < rows and t[f][r] < B:
                    for s in range(2):
                        h[f][t[f][r]][s] = h[f][t[f][r]][s] * vals[2 * r + s] % n2
        want.append([x for f in h for b in f for x in b])
    for form, x in ((0, ct), (1, he.to_mont(k, ct))):
        for chunk, split, lanes in ((0, 2, 16), (1, 1, 16), (2, 2, 16), (3, 1, 16), (64, 2, 16)) + (
                ((5, 1, 8), (4, 2, 8)) if bits == 2048 else ()):
            jobs = [he.Job(dev(ix) if ix.size else torch.empty(0, dtype=torch.int32, device="cuda"), dev(t), B)
                    for (m, F, B), ix, t in zip(shapes, idx, tabs)]
            hs, _ = he.hist_aggregate_counted(k, x, jobs, form=form, chunk=chunk, split=split, lanes=lanes)
            for h, w in zip(hs, want):
                assert he.limbs_to_ints(host(h)) == w, (form, chunk, split, lanes)
        jobs = [he.Job(dev(ix) if ix.size else torch.empty(0, dtype=torch.int32, device="cuda"), dev(t), B)
                for (m, F, B), ix, t in zip(shapes, idx, tabs)]
        for h, w in zip(he.hist_aggregate(k, x, jobs, form=form), want):
            assert he.limbs_to_ints(host(h)) == w, form
