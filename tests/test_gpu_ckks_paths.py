"""CKKS kernels at every ring size: a ciphertext alone and in a batch and over a
used buffer, its noise (below 21 (2 N + 1) by the samples' ranges) the same
integer in every residue, and sums of buffers at any 4-byte alignment."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_n", [12, 13, 14])
def test_ring_sizes_and_alignment(log_n):
    import torch
    from paper_2504_03909_amd import ckks
    print(f"[gpu-case] ckks log_n={log_n}", flush=True)
    ctx = ckks.Context(log_n, 40, 5)
    N = ctx.n
    g = torch.Generator(device="cuda")
    g.manual_seed(log_n)
    pt = torch.stack([torch.randint(0, q, (3, N), dtype=torch.int32, device="cuda", generator=g)
                      for q in ctx.primes], 1)   # [3 vectors, 3 primes, N]
    ct = ctx.encrypt(pt, seed=9, offset=2)
    again = torch.full_like(ct, -1)
    assert torch.equal(ctx.encrypt(pt, seed=9, offset=2, out=again), ct)
    assert torch.equal(ctx.encrypt(pt[1:2], seed=9, offset=3), ct[1:2])   # alone and in a batch
    # noise of each ciphertext: small, centred, the same in every residue
    q = torch.tensor(ctx.primes, device="cuda").view(1, 3, 1)
    diff = (ctx.decrypt(ct).long() - pt.long()) % q
    noise = torch.where(diff > q // 2, diff - q, diff)
    assert torch.equal(noise[:, 0], noise[:, 1]) and torch.equal(noise[:, 0], noise[:, 2])
    assert int(noise.abs().max()) < 21 * (2 * N + 1)
    for off in (0, 1, 2, 3, 4):
        buf = torch.zeros(ct.numel() + 8, dtype=torch.int32, device="cuda")
        x = buf[off:off + ct.numel()].view(ct.shape)
        x.copy_(ct)
        want = (ct.long() + again.long()) % q.view(1, 1, 3, 1)
        assert torch.equal(ctx.add(x, again, out=torch.empty_like(ct)).long(), want), off
        ctx.add(x, again, out=x)
        assert torch.equal(x.long(), want), off
    torch.cuda.synchronize()
