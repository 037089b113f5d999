"""What the library's host code launches, on a stand-in for the HIP runtime."""
import pytest

from launch_record import record


# ---------------------------------------------------------------- CKKS
CKKS = r"""
h = vp()
assert lib.he_ckks_create(u32(12), u32(40), u64(1), ctypes.byref(h)) == 0
n, count = 1 << 12, 5
pt, ct = vp(0x1000), vp(0x100000)  # never read on the host
for what in ("none", "k_encrypt", "k_sample_enc"):
    rec.rec_fail(what.encode())
    rec.rec_reset()
    rc = lib.he_ckks_encrypt(h, pt, u64(count), u64(1), u64(0), ct, None)
    names = [l[0] for l in launches()]
    i = [k for k, s in enumerate(names) if "k_fill" in s]
    out[what] = [rc, names, [rec.rec_arg0(k) for k in i], [rec.rec_arg1(k) for k in i]]
out["ct"], out["words"] = ct.value, count * 2 * 3 * n
"""


def test_ckks_encrypt_leaves_no_samples_behind_a_failed_launch(tmp_path):
    """The ciphertext buffer holds u, e0 and e1 in clear between the two launches
    of an encryption: if the second is refused they are cleared, and if the first
    is, the second does not run on whatever the buffer held."""
    got = record(tmp_path, CKKS)
    rc, names, _, _ = got["none"]
    assert rc == 0 and len(names) == 2 and "k_sample_enc" in names[0] and "k_encrypt" in names[1]
    rc, names, at, words = got["k_encrypt"]
    assert rc == -6 and [("k_sample_enc" in names[0]), ("k_encrypt" in names[1])] == [True, True]
    assert at == [got["ct"]] and words == [got["words"]], names
    rc, names, _, _ = got["k_sample_enc"]
    assert rc == -6 and len(names) == 1, names
