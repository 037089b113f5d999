"""Encryption, decryption and addition of one CKKS context on two streams at once:
the context is only read, so the results are those of one call after the other."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_n", [12, 14])
def test_one_context_on_two_streams(log_n):
    import torch
    from paper_2504_03909_amd import ckks
    print(f"[gpu-case] CKKS on two streams, N = 2^{log_n}", flush=True)
    c = ckks.Context(log_n, 40, 9)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    z = [torch.randn(60, c.slots, dtype=torch.float64, device="cuda", generator=g) for _ in range(2)]
    pt = [c.encode(x) for x in z]
    want = [c.encrypt(p, seed=3, offset=100 * i) for i, p in enumerate(pt)]
    dec = [c.decrypt(w) for w in want]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got, back = [[], []], [[], []]
    out = [[torch.empty_like(w) for _ in range(8)] for w in want]
    torch.cuda.synchronize()
    for k in range(8):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got[i].append(c.encrypt(pt[i], seed=3, offset=100 * i, out=out[i][k]))
                back[i].append(c.decrypt(got[i][k]))
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(x, want[i]) for x in got[i]) and all(torch.equal(x, dec[i]) for x in back[i])
    c.close()
