"""The library's host-only code (index-file reader, array validation, fixed traversal-order tables) built
for the CPU with the address and undefined-behaviour sanitizers, and run on valid, truncated and corrupted
index files, on out-of-range sizes, and against the oracle's tables.  No GPU."""
import os
import struct
import subprocess

import numpy as np
import pytest

from oracle import pqt_index_io as IO
from oracle import pqt_query as Q

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, EINVAL, EIO, EFORMAT, ENOMEM, EHIP, EUNSUPPORTED = 0, -1, -2, -3, -4, -5, -6


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "sanitizer_driver")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-static-libasan", "-static-libubsan", "-ffp-contract=off",
           os.path.join(ROOT, "tests", "host", "sanitizer_driver.cpp"),
           os.path.join(ROOT, "paper_1702_05911_amd", "csrc", "pqt_host.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def run(*args):
        env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0:detect_leaks=1:abort_on_error=0",
                   UBSAN_OPTIONS="print_stacktrace=1")
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, env=env, timeout=120)
        assert r.returncode == 0 and "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, \
            f"{args}: exit {r.returncode}\n{r.stderr[-2000:]}"
        return r.stdout
    return run


def _rc(out):
    return int(out.split()[1])


def test_valid_files_load(driver, tiny, tiny_pair, tmp_path):
    for name, ix in (("tiny", tiny[3]), ("pair", tiny_pair[3])):
        path = str(tmp_path / f"{name}.pqt")
        IO.write_index(path, ix)
        out = driver("load", path)
        assert _rc(out) == OK
        assert int(out.split()[2]) == int(np.count_nonzero(np.diff(ix.offsets.astype(np.int64))))     # slots that hold a vector


def test_truncated_files_are_format_errors(driver, tiny, tmp_path):
    ix = tiny[3]
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    blob = open(path, "rb").read()
    cut = str(tmp_path / "cut.pqt")
    # every section boundary (multiples of 256 around the section starts), one byte either side, and a few odd places
    places = {0, 1, 8, 63, 64, 255, 256, 257, len(blob) - 1, len(blob) - 100, len(blob) // 2}
    pos = 256
    dp = ix.D // ix.P
    for nbytes in (ix.P * ix.k1 * dp * 4, ix.P * ix.k1 * ix.k2 * dp * 4, ix.M * 256, ix.M * 256, ix.M * 1024,
                   ix.M * ix.k1 * ix.k1 * 4, (ix.H + 1) * 4, ix.N * 4):
        pos = (pos + 255) // 256 * 256 + nbytes
        places |= {pos - 1, pos, pos + 1, (pos + 255) // 256 * 256}
    for n in sorted(p for p in places if 0 <= p < len(blob)):
        with open(cut, "wb") as f:
            f.write(blob[:n])
        assert _rc(driver("load", cut)) == EFORMAT, n
    assert _rc(driver("load", str(tmp_path / "missing.pqt"))) == EIO


def _patched(blob, offset, fmt, value):
    b = bytearray(blob)
    struct.pack_into(fmt, b, offset, value)
    return bytes(b)


def test_corrupted_headers_and_arrays(driver, tiny, tmp_path):
    ix = tiny[3]
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    blob = open(path, "rb").read()
    bad = str(tmp_path / "bad.pqt")
    cases = [
        (b"NOTANIDX" + blob[8:], EFORMAT),
        (_patched(blob, 8, "<I", 2), EFORMAT),                       # version
        (_patched(blob, 12, "<I", 0), EFORMAT),                      # D = 0
        (_patched(blob, 12, "<I", ix.D + 1), EFORMAT),               # D not a multiple of P and M
        (_patched(blob, 16, "<I", 3), EFORMAT),                      # P = 3 does not divide D = 32
        (_patched(blob, 20, "<I", 0xFFFFFFFF), EUNSUPPORTED),        # k1 beyond the limit
        (_patched(blob, 24, "<I", 5000), EUNSUPPORTED),              # k2 beyond the limit
        (_patched(blob, 28, "<I", 0), EFORMAT),                      # M = 0
        (_patched(blob, 32, "<Q", 2 ** 40), EUNSUPPORTED),           # N beyond 32 bits: nothing is allocated
        (_patched(blob, 32, "<Q", ix.N + 1), EFORMAT),               # N larger than the file holds
        (_patched(blob, 40, "<Q", ix.H + 1), EFORMAT),               # H above the number of bins
        (_patched(blob, 40, "<Q", 0), EFORMAT),
        (_patched(blob, 48, "<I", 0), EFORMAT),                      # T = 0
        (_patched(blob, 52, "<I", 1 << 20), EFORMAT),                # C beyond the limit
        (_patched(blob, 56, "<I", 64), EFORMAT),                     # offset_bits
        (_patched(blob, 60, "<I", 7), EFORMAT),                      # code_format
    ]
    for n, (data, want) in enumerate(cases):
        with open(bad, "wb") as f:
            f.write(data)
        out = driver("load", bad)
        assert _rc(out) == want, (n, out)
    # arrays: pointer array not monotone / not spanning the ids, table entry naming a centroid >= k1
    for mutate, want in ((lambda b: b.offsets.__setitem__(5, b.offsets[-1] + 7), EFORMAT),
                         (lambda b: b.offsets.__setitem__(-1, b.offsets[-1] - 1), EFORMAT),
                         (lambda b: b.offsets.__setitem__(0, 1), EFORMAT),
                         (lambda b: b.tbl_j.__setitem__((1, 17), ix.k1), EFORMAT)):
        broken = IO.read_index(path)
        broken.offsets, broken.tbl_j = broken.offsets.copy(), broken.tbl_j.copy()
        mutate(broken)
        IO.write_index(bad, broken)
        assert _rc(driver("load", bad)) == want


def test_pair_code_bytes_are_checked(driver, tiny_pair, tmp_path):
    ix = tiny_pair[3]
    path = str(tmp_path / "pair.pqt")
    IO.write_index(path, ix)
    broken = IO.read_index(path)
    broken.codes = broken.codes.copy()
    broken.codes[17, 2] = ix.k1 * (ix.k1 - 1) // 2                 # one past the last pair
    IO.write_index(path, broken)
    assert _rc(driver("load", path)) == EFORMAT


def test_size_limits(driver):
    ok = dict(D=128, P=2, k1=16, k2=8, M=8, N=1000, H=16384, T=1024, C=4096, fmt=0)

    def rc(**kw):
        v = dict(ok, **kw)
        return driver("sizes", *[v[n] for n in ("D", "P", "k1", "k2", "M", "N", "H", "T", "C", "fmt")]).split()[1:3]
    assert rc() == ["0", "plain"]
    assert rc(H=9973) == ["0", "hashed"]
    assert rc(P=4, H=10_000_019) == ["0", "hashed"]
    assert rc(P=4, k1=256, k2=1024, M=4)[0] == str(EUNSUPPORTED)    # (k1 k2)^4 = 2^72 bins
    assert rc(P=4, k1=256, k2=256, M=4, H=10 ** 9)[0] == str(EUNSUPPORTED)   # (2^16)^4 = 2^64: one too many for 64-bit bin numbers
    assert rc(P=4, k1=256, k2=128, M=4, H=10 ** 9) == ["0", "hashed"]       # 2^60 bins, hashed to 10^9 slots
    assert rc(k1=257)[0] == str(EUNSUPPORTED)
    assert rc(D=8200, M=8, P=2)[0] == str(EUNSUPPORTED)
    assert rc(M=3)[0] == str(EFORMAT)                              # M not a multiple of P
    assert rc(T=8193)[0] == str(EFORMAT)
    assert rc(fmt=1, k1=24)[0] == str(EUNSUPPORTED)                # 276 centroid pairs do not fit a byte
    assert rc(fmt=1, k1=23)[0] == "0"
    assert rc(fmt=1, k1=1, H=64)[0] == str(EUNSUPPORTED)            # no pair of centroids at all


def test_static_order_tables_equal_the_oracles(driver):
    """The ten fixed orders and the nine slope thresholds the library uploads are bit-identical to the oracle's."""
    for R, T in ((1, 1), (4, 16), (7, 30), (16, 100), (32, 1024), (64, 700), (128, 1024), (1024, 8192)):
        lines = driver("static", R, T).strip().split("\n")
        Tn = int(lines[0].split()[1])
        assert Tn == min(T, R * R)
        thr = np.array([float.fromhex(v) for v in lines[1].split()], dtype=np.float32)
        assert np.array_equal(thr, Q.slope_thresholds(np.float32))
        for i, s in enumerate(Q.slopes()):
            got = [tuple(int(v) for v in pair.split(",")) for pair in lines[2 + i].split()]
            if R <= 128:
                assert got == [tuple(t) for t in Q.static_order(R, T, s).tolist()], (R, T, i)
            assert len(got) == Tn and len(set(got)) == Tn


def test_region_size_counts_the_hyperbolic_region(driver):
    for nA, nB, Tn in ((8, 8, 64), (64, 64, 1024), (128, 16, 300), (5, 1000, 37), (1024, 1024, 8192)):
        want = sum(1 for a in range(min(nA, Tn)) for b in range(min(nB, Tn // (a + 1))))
        assert int(driver("region", nA, nB, Tn).split()[1]) == want


@pytest.mark.parametrize("shape, nq, want", [
    # (D, P, k1, list length, C): measured both ways
    ((128, 2, 16, 64, 4096), (1, 67, 300, 1024), 1),
    ((128, 2, 64, 128, 8192), (1, 256, 512, 1024), 1),
    ((960, 2, 64, 64, 2000), (67, 256), 1),
    ((960, 2, 64, 64, 2000), (1, 12, 300, 512, 700, 1024), 0),
    ((960, 4, 64, 64, 1000), (16, 256, 300), 0),
    ((960, 2, 16, 64, 1000), (4, 16, 512), 1),
    ((960, 2, 16, 64, 1000), (1, 700, 1024), 0),
    ((960, 4, 16, 64, 1000), (1, 256, 300), 1),
    ((1024, 2, 16, 64, 2000), (1024,), 0),
    ((512, 2, 64, 64, 1000), (700, 1024), 0),
    ((1536, 2, 16, 64, 1000), (1, 1024), 0),
    ((960, 1, 16, 64, 1000), (1, 1024), 1),
    ((960, 2, 16, 128, 1000), (1, 1024), 1),
])
def test_one_launch_where_it_pays(driver, shape, nq, want):
    """Small batches take one launch where that measured faster than three, and three launches where not."""
    for n in nq:
        assert int(driver("small", *shape, n)) == want, n


def _bf16(x):
    """float32 -> nearest bf16 (ties to even), as float32."""
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _truncate(x):
    """float64 -> float32 towards zero."""
    r = np.asarray(x, np.float64).astype(np.float32)
    over = np.abs(r.astype(np.float64)) > np.abs(x)
    return np.where(over, np.nextafter(r, np.float32(0)), r)


@pytest.mark.parametrize("elem_bytes, D", [(4, 4), (4, 16), (4, 128), (4, 192), (4, 320), (4, 960), (1, 16), (1, 96), (1, 128), (1, 160)])
def test_brute_force_error_bound(driver, elem_bytes, D):
    """The bound that lets the brute-force filter drop a vector, against the filter's arithmetic written out: numbers cut
    into bf16 pieces, piece products added in fp32 with every addition truncated, against float64.  All coordinates of a
    vector are equal (the Cauchy-Schwarz bound is then reached) and their significands the worst of 60,000 for the cut,
    together with the ends of the range."""
    dot, norm = (float.fromhex(v) for v in driver("bound", elem_bytes, D).split())
    grid = (1.0 + np.arange(60_000) / 60_000).astype(np.float32)
    first = _bf16(grid)
    second = _bf16(grid - first)
    left = (grid - first).astype(np.float64) / grid, (grid.astype(np.float64) - first - second) / grid
    worst = np.concatenate([[i for v in left for i in (np.argmax(v), np.argmin(v))], np.argsort(-np.abs(left[0]))[:40],
                            np.argsort(-np.abs(left[1]))[:40], [0, len(grid) - 1]])
    q = grid[worst.astype(int)]
    x = np.array([1, 3, 127, 129, 253, 255], np.float32) if elem_bytes == 1 else q
    q, x = (v.ravel() for v in np.meshgrid(q, x))
    half = _truncate(0.5 * D * x.astype(np.float64) ** 2)             # (its own sum is not what is tested here)
    for order in (1, -1):                                            # products first added to the norm, or last
        hq, hx = _bf16(q), _bf16(x)
        mq, mx = _bf16(q - hq), _bf16(x - hx)
        products = [hx * hq, hx * mq] + ([mx * hq] if elem_bytes == 4 else [])
        s = -half if order == 1 else np.zeros_like(q)
        for p in products:
            p = p.astype(np.float64)
            for _ in range(D):
                s = _truncate(s.astype(np.float64) + p)
        if order == -1:
            s = _truncate(s.astype(np.float64) - half)
        true = D * q.astype(np.float64) * x - 0.5 * D * x.astype(np.float64) ** 2
        bound = dot * D * np.abs(q.astype(np.float64) * x) + norm * D * x.astype(np.float64) ** 2
        assert (np.abs(s - true) <= bound).all(), (np.abs(s - true) / bound).max()


@pytest.mark.parametrize("D", [4, 96, 200, 960])
@pytest.mark.parametrize("small", [1.0, 2.0 ** -12, 2.0 ** -30])
def test_brute_force_halves_error_bound(driver, D, small):
    """The same for products of halves: the query and the longest vector (norm X) scaled to norms of 2^14 .. 2^15, numbers rounded
    to half precision, those below 2^-14 taken for zero, the products added with every addition truncated.  `small`: the other
    vectors' size against the longest's, down to where all of their numbers are taken for zero."""
    dot, norm, flush = (float.fromhex(v) for v in driver("halves", D).split())
    grid = (1.0 + np.arange(40_000) / 40_000).astype(np.float32)
    left = np.abs(grid - grid.astype(np.float16).astype(np.float32)) / grid
    worst = grid[np.concatenate([np.argsort(-left)[:40], [0, len(grid) - 1]])]
    q, x = (v.ravel() for v in np.meshgrid(worst, worst * np.float32(small)))
    X = np.sqrt(D) * 2.0                                            # longest norm: coordinates of two
    to = lambda v: 2.0 ** (14 - np.floor(np.log2(v)))
    sq, sx = to(np.sqrt(D) * q.astype(np.float64)), to(X)
    hq, hx = (np.where(np.abs(v) < 2.0 ** -14, 0.0, v.astype(np.float16).astype(np.float64)) for v in (q * sq, x * sx))
    half = 0.5 * D * x.astype(np.float64) ** 2
    for order in (1, -1):                                            # products first added to the norm, or last
        start = _truncate(-half * sq * sx)
        s = start if order == 1 else np.zeros_like(start)
        for _ in range(D):
            s = _truncate(s.astype(np.float64) + hq * hx)
        if order == -1:
            s = _truncate(s.astype(np.float64) + start)
        true = D * q.astype(np.float64) * x - half
        qn, xn = np.sqrt(D) * q.astype(np.float64), np.sqrt(D) * np.abs(x.astype(np.float64))
        bound = dot * qn * xn + norm * xn ** 2 + flush * qn * X
        assert (np.abs(s / (sq * sx) - true) <= bound).all(), (np.abs(s / (sq * sx) - true) / bound).max()


@pytest.mark.parametrize("D", [4, 128, 960, 1980, 2048, 3072, 4096, 8192])
def test_brute_force_halves_bound_covers_the_pieces(driver, D):
    """The first chunk's values come from bf16 pieces and stay in the list with those of halves, under one window: that of the halves
    (for a vector of norm r, vectors' offset mu and a query of norm q: dot (r + mu)^2 + 2 norm r^2 and dot q (r + mu)) must be
    no narrower than that of the pieces, whatever r and mu."""
    dot, norm, flush = (float.fromhex(v) for v in driver("halves", D).split())
    piece_dot, piece_norm = (float.fromhex(v) for v in driver("bound", 4, D).split())
    assert dot >= piece_dot and flush >= 0
    for mu in (0.0, 0.1, 1.0, 10.0):
        assert dot * (1 + mu) ** 2 + 2 * norm >= piece_dot * (1 + mu) ** 2 + 2 * piece_norm, mu
