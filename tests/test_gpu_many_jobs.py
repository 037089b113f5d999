"""Batches of thousands of small jobs: results against products of Python
integers, and the time in proportion to the number of jobs."""
import sys

import numpy as np
import pytest

import oracle.paillier as P

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


def test_thousands_of_jobs():
    import torch
    from paper_2504_03909_amd import he
    bits, rows, n, F, B = 1024, 50_000, 10, 2, 16
    p, q = P.keygen(bits, 1)
    n2 = (p * q) ** 2
    k = he.Key.from_primes(bits, p, q)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    ct = torch.randint(-(1 << 31), 1 << 31, (rows, 2, 2 * k.limbs), device="cuda", generator=g).to(torch.int32)
    ct[..., -1] = 0  # below n^2
    bins = torch.randint(0, B, (F, rows), device="cuda", generator=g).to(torch.uint8)
    perm = torch.randperm(rows, device="cuda", generator=g).to(torch.int32)
    best = {}
    for count in (250, 4000):
        say(f"{count} jobs of {n} samples")
        # every 50th job is empty
        jobs = [he.Job(perm[i * n:i * n + (n if i % 50 else 0)].contiguous(), bins, B) for i in range(count)]
        ms = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            hists = he.hist_aggregate(k, ct, jobs)
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        best[count] = min(ms)
        for i in (0, 1, count // 2 + 1, count - 1):
            rid = jobs[i].sample_idx.cpu().tolist()
            vals = he.limbs_to_ints(ct[rid].cpu().numpy()) if rid else []
            t = bins[:, rid].cpu().numpy() if rid else np.zeros((F, 0), dtype=np.uint8)
            want = [1] * (F * B * 2)
            for f in range(F):
                for j in range(len(rid)):
                    for s in range(2):
                        e = (f * B + int(t[f, j])) * 2 + s
                        want[e] = want[e] * vals[2 * j + s] % n2
            assert he.limbs_to_ints(hists[i].cpu().numpy()) == want, (count, i)
    say(f"ms: {best}")
    # sixteen times the jobs; searched one by one they took some 200 times as long
    assert best[4000] < 32 * best[250], best
    k.close()
