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


# ---------------------------------------------------- exponentiation shapes
KEYS = r"""
bits, p, q = env["bits"], int(env["p"]), int(env["q"])
plain, secret = key(bits, p, q), key(bits, p, q)
assert lib.he_key_set_constant_time(secret, 1) == 0
A, B = vp(0x100000), vp(0x900000)  # device addresses, never read on the host

def encrypt(k, count):
    rec.rec_reset()
    assert lib.he_encrypt(k, A, u64(count), None, u64(1), u64(0), B, None) == 0
    return launches()

def decrypt(k, count):
    rec.rec_reset()
    assert lib.he_decrypt(k, A, u64(count), B, None, None, None) == 0
    return launches()

def tune(k, enc, dec):
    choice, ms = (u32 * 9)(), (ctypes.c_float * 3)()
    assert lib.he_crt_autotune(k, u64(enc), u64(dec), choice, ms, None) == 0, lib.he_last_error()
    return list(choice), list(ms)
"""


@pytest.fixture(scope="module")
def primes():
    import oracle.paillier as P
    return {bits: [str(x) for x in P.keygen(bits, seed)] for bits, seed in ((1024, 1), (2048, 2))}


@pytest.mark.parametrize("bits", [1024, 2048])
def test_tuning_one_kind_of_key_leaves_the_other_alone(tmp_path, primes, bits):
    """Constant-time keys run other kernels: what was timed for an ordinary key's
    is not used for theirs, and the reverse."""
    got = record(tmp_path, KEYS + r"""
n = 5000
def squared(k):  # the launches of the exponentiations mod p^2 (those mod p are constant-time keys' alone)
    return [l for l in encrypt(k, n) + decrypt(k, n) if "k_pow" in l[0] and "k_powI" not in l[0] and "ELi0E" not in l[0]]

for name, tuned, other in (("plain", plain, secret), ("secret", secret, plain)):
    before, own = squared(other), squared(tuned)
    tune(tuned, n, n)  # every trial takes as long: the first, one lane per integer, stays
    out[name] = [before, squared(other), own, squared(tuned)]
    n *= 4  # another class
""", bits=bits, p=primes[bits][0], q=primes[bits][1])
    for before, after, own, own_after in got.values():
        assert before == after
        assert own != own_after  # the tuner's choice did take effect


def test_masked_decryption_is_planned_on_its_own_kernel(tmp_path, primes):
    """The resident blocks of a constant-time key's decryption are the masked
    kernel's, not those of the kernel with sliding windows."""
    got = record(tmp_path, KEYS + r"""
rec.rec_single(b"Lb1E")  # k_pow_pair<.., .., true>
out["secret"], out["plain"] = decrypt(secret, 60000), decrypt(plain, 60000)
""", bits=2048, p=primes[2048][0], q=primes[2048][1])
    grids = {k: [g for name, g, _ in v if "k_pow" in name] for k, v in got.items()}
    assert max(grids["secret"]) <= 256 and max(grids["plain"]) <= 512, grids


def test_ordinary_keys_do_not_sweep_a_step_they_do_not_have(tmp_path, primes):
    """The exponentiation mod p is constant-time keys' alone: tuning an ordinary key
    launches it for one timing only and changes nothing for those keys."""
    got = record(tmp_path, KEYS + r"""
before = encrypt(secret, 5000)
rec.rec_reset()
choice, ms = tune(plain, 5000, 3000)
out["launches"] = [l[0] for l in launches() if "k_powI" in l[0] or "ELi0E" in l[0]]
out["choice"], out["ms"] = choice, ms
out["same"] = encrypt(secret, 5000) == before
""", bits=2048, p=primes[2048][0], q=primes[2048][1])
    assert 1 <= len(got["launches"]) <= 3, got["launches"]  # a warm-up and two timed runs
    assert got["same"] and got["choice"][0] > 0 and min(got["ms"]) > 0


PINS = KEYS + r"""
def pin(k, kind, count, lanes, waves, tail):
    return lib.he_crt_set_shape(k, u32(kind), u64(count), u32(lanes), u32(waves), u32(tail))

def clear(k, enc, dec):
    for kind, count in ((0, enc), (1, enc), (2, dec)):
        assert pin(k, kind, count, 0, 0, 0) == 0
"""


@pytest.mark.parametrize("bits", [1024, 2048])
@pytest.mark.parametrize("enc,dec", [(5003, 3001), (200000, 16384), (33, 16390)])
def test_what_the_tuner_returns_can_be_pinned(tmp_path, primes, bits, enc, dec):
    """Whichever trial is the fastest: he_crt_set_shape takes what he_crt_autotune
    returned, and the launches are then those the tuner remembered.  lanes 0 takes
    both back."""
    got = record(tmp_path, PINS + r"""
enc, dec = env["enc"], env["dec"]
out["bad"] = []
for name, k in (("plain", plain), ("secret", secret)):
    clear(k, enc, dec)
    default = [encrypt(k, enc), decrypt(k, dec)]
    rec.rec_fastest(-1)
    tune(k, enc, dec)
    trials = rec.rec_timed()
    for fastest in range(trials):
        rec.rec_fastest(fastest)
        choice, _ = tune(k, enc, dec)
        tuned = [encrypt(k, enc), decrypt(k, dec)]
        clear(k, enc, dec)
        if [encrypt(k, enc), decrypt(k, dec)] != default:
            out["bad"].append([name, fastest, "lanes 0 is not the default plan"])
        for i, count in enumerate((enc, enc, dec)):
            if pin(k, i, count, *choice[3 * i:3 * i + 3]) != 0:
                out["bad"].append([name, fastest, choice, lib.he_last_error().decode()])
        if [encrypt(k, enc), decrypt(k, dec)] != tuned:
            out["bad"].append([name, fastest, choice, "other launches"])
    clear(k, enc, dec)
    out[name] = trials
""", bits=bits, p=primes[bits][0], q=primes[bits][1], enc=enc, dec=dec)
    assert got["plain"] >= 9 and got["secret"] >= 13
    assert not got["bad"], got["bad"][:5]


@pytest.mark.parametrize("bits", [1024, 2048])
def test_pins_taken_and_refused(tmp_path, primes, bits):
    """One lane is a pin of every private-key kind; two lanes are none where the
    modulus has 64 limbs; unbuilt widths, waves and tails are refused as ever."""
    got = record(tmp_path, PINS + r"""
out["ok"] = [[kind, lanes, tail] for kind in range(4) for lanes in range(0, 33) for tail in range(0, 33)
             if pin(plain, kind, 777, lanes, 0, tail) == 0]
out["waves"] = [w for w in range(9) if pin(plain, 0, 777, 4, w, 0) == 0]
out["zero"] = [w for w in range(9) if pin(plain, 0, 777, 0, w, 0) == 0]
out["count"] = pin(plain, 0, 0, 4, 0, 0)
for kind in range(4):
    assert pin(plain, kind, 777, 0, 0, 0) == 0
""", bits=bits, p=primes[bits][0], q=primes[bits][1])
    two = bits == 1024
    widths = {0: [1, 2, 4, 8, 16], 1: [1, 2, 4, 8, 16] if two else [1, 4, 8, 16],
              2: [1, 2, 4, 8, 16] if two else [1, 4, 8, 16], 3: [1, 4, 8, 16] if two else [8, 16]}
    want = [[k, 0, 0] for k in widths] + [[k, g, t] for k, ws in widths.items() for g in ws for t in [0] + [x for x in ws if x > g]]
    assert sorted(got["ok"]) == sorted(want)
    assert got["waves"] == [0, 2, 3] and got["zero"] == [0] and got["count"] == -1


@pytest.mark.parametrize("bits", [1024, 2048])
def test_masked_plans_follow_the_masked_kernels_times(tmp_path, primes, bits):
    """At 40,000 values the masked lift and decryption take four lanes or more per
    integer, where the sliding ones take one or two: at 1024 bits a decryption is
    6.3 ms so and was 8.0 planned with the sliding kernels' times."""
    got = record(tmp_path, KEYS + """
out["secret"], out["plain"] = encrypt(secret, 40000) + decrypt(secret, 40000), decrypt(plain, 40000)
""", bits=bits, p=primes[bits][0], q=primes[bits][1])
    width = {k: [int(name.split("ELi")[1].split("E")[0]) for name, _, _ in v if "k_pow_pairI" in name and "ELi0E" not in name]
             for k, v in got.items()}
    assert len(width["secret"]) >= 2 and min(width["secret"]) >= 4, width
    assert width["plain"][0] <= 2, width


def test_packing_one_slot_does_not_enter_the_squarings(tmp_path, primes):
    """One slot is one product by a constant: the kernel built for 64 squarings a
    slot took 1.7 times the former's time at it."""
    got = record(tmp_path, KEYS + r"""
for slots in (1, 2, 31):
    rec.rec_reset()
    assert lib.he_pack(plain, A, u64(1000), u32(slots), B, None) == 0
    out[slots] = [l[0] for l in launches()]
""", bits=2048, p=primes[2048][0], q=primes[2048][1])
    assert len(got["1"]) == 1 and "k_enc_obf" in got["1"][0]
    assert all(len(got[s]) == 1 and "k_pack" in got[s][0] for s in ("2", "31"))


# ---------------------------------------------------------------- histograms
JOBS = KEYS + r"""
class Job(ctypes.Structure):
    _fields_ = [("idx", vp), ("n", u64), ("bins", vp), ("ld", u64), ("F", u32), ("B", u32), ("hist", vp), ("bad", vp)]

rows = env["rows"]
def aggregate(n):
    rec.rec_reset()
    j = Job(A, n, A, rows, 2, 16, B, None)
    rc = lib.he_hist_aggregate(plain, A, u64(rows), env["form"], ctypes.byref(j), u32(1), None)
    return rc, [l[0] for l in launches()]

def plan(n):
    rec.rec_reset()
    j, h = Job(A, n, A, rows, 2, 16, B, None), vp()
    rc = lib.he_hist_plan_create(plain, A, u64(rows), env["form"], ctypes.byref(j), u32(1), u32(0), u32(0), ctypes.byref(h))
    names = [l[0] for l in launches()]
    if rc == 0:
        lib.he_hist_plan_free(h)
    return rc, names
"""


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("n", [200_000, 150_000])  # every row converted, or the samples gathered
def test_histograms_without_memory_for_a_second_copy(tmp_path, primes, form, n):
    """Where the ciphertexts in the kernels' form cannot be allocated (230 MB here),
    a plan and a call run without them, as they did before there was such a copy;
    where not even the partial products can, they are refused."""
    got = record(tmp_path, JOBS + r"""
out["roomy"] = [plan(env["n"]), aggregate(0)]
base = rec.rec_total()
rec.rec_limit(base + (64 << 20))
out["tight"] = [plan(env["n"]), aggregate(env["n"])]
rec.rec_limit(base + (1 << 20))
out["none"] = [plan(env["n"])]
""", bits=2048, p=primes[2048][0], q=primes[2048][1], rows=200_000, n=n, form=form)
    rc, names = got["roomy"][0]
    assert rc == 0 and any("k_hist_pairs" in x for x in names) and any("k_hist_chunkILi2ELi4ELb0E" in x for x in names)
    for rc, names in got["tight"]:
        assert rc == 0 and not any("k_hist_pairs" in x for x in names)
        assert any("k_hist_chunkILi2ELi4ELb1E" in x for x in names)
    assert got["none"][0][0] == -5


@pytest.mark.parametrize("bits", [1024, 2048])
def test_exponentiations_with_little_room_for_tables(tmp_path, primes, bits):
    """One lane per integer on every SIMD takes 0.6 to 1.25 GB of window tables. With
    less memory (as much as the former kernels needed at 2048 bits, then hardly
    more than the operands) encryption and decryption run on fewer blocks, the
    tuner (with the 830 MB it needed then) tries what fits, and only calls without room for their operands fail."""
    got = record(tmp_path, PINS + r"""
n = 200000
def call(name, stream):
    rec.rec_reset()
    if name == "encrypt":
        return lib.he_encrypt(plain, A, u64(n), None, u64(1), u64(0), B, stream)
    if name == "secret":
        return lib.he_encrypt(secret, A, u64(n), None, u64(1), u64(0), B, stream)
    if name == "public":
        return lib.he_encrypt_public(plain, A, u64(n), None, u64(1), u64(0), B, stream)
    return lib.he_decrypt(plain if name == "decrypt" else secret, A, u64(n), B, None, None, stream)

stream = 1
for room in (0, 443, 160, 20):
    for name in ("encrypt", "secret", "public", "decrypt", "secret decrypt"):
        stream += 1  # a stream has its own workspace
        base = rec.rec_total()
        rec.rec_limit(base + (room << 20) if room else (1 << 63))
        rc = call(name, vp(stream))
        out[f"{room} {name}"] = [rc, max([g for s, g, _ in launches() if "k_pow" in s] or [0]), rec.rec_total() - base]
rec.rec_limit(rec.rec_total() + (env["tune"] << 20))
out["tune"] = tune(plain, 20000, 20000)
rec.rec_limit(1 << 63)
""", bits=bits, p=primes[bits][0], q=primes[bits][1], tune=830)
    for name in ("encrypt", "secret", "public", "decrypt", "secret decrypt"):
        full = got[f"0 {name}"]
        assert full[0] == 0 and full[1] >= 256
        for room in (443, 160):
            rc, grid, used = got[f"{room} {name}"]
            assert rc == 0 and 1 <= grid <= full[1] and used <= room << 20, (room, name)
        assert got[f"20 {name}"][0] == -5
    assert got["160 encrypt"][1] < got["0 encrypt"][1] or got["0 encrypt"][2] <= 160 << 20
    choice, ms = got["tune"]
    assert ms[1] > 0 and ms[2] > 0
