"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same
seeded inputs.  Bit-exact on selected clusters, bin order, proposed slots, candidate lists and
top-k ids (by replaying the oracle's discrete logic on the GPU's fp32 values); fp32 distances
within 1e-4 relative (plus the cancellation floor stated in parity_util)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(__file__))
import parity_util as PU  # noqa: E402
from oracle import pqt_build as B  # noqa: E402
from oracle import pqt_index_io as IO  # noqa: E402
from oracle import pqt_query as Q  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pqt():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: no silent fallback")
    import paper_1702_05911_amd.binding as binding
    return binding


def _run_debug(pqt, gix, Y, k, w):
    import torch
    yq = torch.from_numpy(np.ascontiguousarray(Y)).cuda()
    names = tuple(n for n in pqt._TAP_FIELDS if n != "lut" or pqt.pqt_index_info(gix)["code_format"] == 0)
    ids, dists, taps = pqt.pqt_query_batch_debug(gix, yq, k, w, taps=names)
    torch.cuda.synchronize()
    ids2, dists2 = pqt.pqt_query_batch(gix, yq, k, w)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids2) and torch.equal(dists.view(torch.int32), dists2.view(torch.int32)), \
        "debug and plain entry points disagree"
    return PU.to_np(ids), PU.to_np(dists), {n: PU.to_np(t) for n, t in taps.items()}


def _stagewise(pqt, ix, path, Y, k, w, T, C, exact=False, must_match_all=False, order="fullsort", truncate_pairs=False):
    gix = pqt.pqt_index_load(path, 0)
    try:
        pqt.pqt_set_budget(gix, T, C)
        if order == "static":
            pqt.pqt_set_bin_order(gix, pqt.PQT_ORDER_STATIC_SLOPES)
        ids, dists, taps = _run_debug(pqt, gix, Y, k, w)
    finally:
        pqt.pqt_index_free(gix)
    same = decided = 0
    for q in range(Y.shape[0]):
        print(f"query {q}", flush=True)
        tr = PU.check_query_stages(ix, Y[q], taps, q, k, w, T, C, ids, dists, exact=exact, order=order,
                                   truncate_pairs=truncate_pairs)
        s, d = PU.end_to_end_agreement(tr, ids[q], dists[q])
        if exact or must_match_all:
            assert s, f"query {q}: ids differ from the float64 oracle"
        if exact:
            assert np.array_equal(dists[q].astype(np.float64), tr.out_dists), f"query {q}: distances not bit-exact"
        if d:
            assert s, f"query {q}: all decision margins > 1e-5 but ids differ from the oracle"
        same += s
        decided += d
    print("tolerance so far: " + PU.STATS.summary(), flush=True)
    return same, decided


def test_tiny_stagewise(pqt, tiny, tmp_path):
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    same, decided = _stagewise(pqt, ix, path, Y, cfg.k, cfg.w, cfg.T, cfg.C)
    print(f"tiny: {same}/{cfg.nq} queries identical to the float64 oracle end to end, {decided} decided by margin")
    assert same >= 0.9 * cfg.nq


def test_tiny_ragged_batches_and_determinism(pqt, tiny, tmp_path):
    import torch
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    gix = pqt.pqt_index_load(path, 0)
    try:
        yq = torch.from_numpy(Y).cuda()
        full_ids, full_d = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)
        torch.cuda.synchronize()
        for n in (1, 15, 16, 17, 33):
            ids, d = pqt.pqt_query_batch(gix, yq[:n].contiguous(), cfg.k, cfg.w)
            torch.cuda.synchronize()
            assert torch.equal(ids, full_ids[:n]) and torch.equal(d.view(torch.int32), full_d[:n].view(torch.int32))
        ids0, d0 = pqt.pqt_query_batch(gix, yq[:0].contiguous(), cfg.k, cfg.w)
        assert ids0.shape == (0, cfg.k)
        info = pqt.pqt_index_info(gix)
        assert (info["N"], info["D"], info["P"], info["k1"], info["k2"], info["M"], info["H"]) == \
            (cfg.N, cfg.D, cfg.P, cfg.k1, cfg.k2, cfg.M, cfg.H)
    finally:
        pqt.pqt_index_free(gix)


def test_tiny_exhaustive_visits_everything(pqt, tiny, tmp_path):
    """w = k1, T = K, C >= N: every bin is visited, the candidate list is the whole database."""
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    Ys = Y[:6]
    gix = pqt.pqt_index_load(path, 0)
    try:
        pqt.pqt_set_budget(gix, ix.K, cfg.N)
        ids, dists, taps = _run_debug(pqt, gix, Ys, 10, cfg.k1)
    finally:
        pqt.pqt_index_free(gix)
    for q in range(Ys.shape[0]):
        assert int(taps["n_cand"][q]) == cfg.N
        assert np.array_equal(np.sort(taps["cand_ids"][q]), np.arange(cfg.N))
        PU.check_query_stages(ix, Ys[q], taps, q, 10, cfg.k1, ix.K, cfg.N, ids, dists)


def _exact_arithmetic_index(N=3000, seed=5, k1=4, k2=2, P=2):
    """Integer codebooks, integer data and dyadic lambdas: every fp32 operation of the path is
    exact, so the GPU must equal the float64 oracle bit for bit, distances included."""
    from workloads import small_integer_vectors
    rng = np.random.default_rng(seed)
    D, M = 16, 4
    dp = D // P
    C1 = rng.integers(0, 8, size=(P, k1, dp)).astype(np.float32)
    C2 = np.clip(C1[:, :, None, :] + rng.integers(-1, 2, size=(P, k1, k2, dp)), 0, 7).astype(np.float32)
    lams = [0.0, 0.25, 0.5, 0.75, 1.0, -0.25, 1.25, 0.125]
    ent = [(i, j, lam) for i in range(k1) for j in range(i + 1, k1) for lam in lams]
    ti = np.array([[ent[c % len(ent)][0] for c in range(256)]] * M, np.uint8)
    tj = np.array([[ent[c % len(ent)][1] for c in range(256)]] * M, np.uint8)
    tl = np.array([[ent[c % len(ent)][2] for c in range(256)]] * M, np.float32)
    X = small_integer_vectors(N, D, 0, 8, seed=seed, clusters=40)
    Y = small_integer_vectors(64, D, 0, 8, seed=seed + 1, clusters=40)
    ix = B.build_index(X, P, k1, k2, M, T=64, C=512, codebooks=(C1, C2), line_table=(ti, tj, tl))
    return ix, X, Y


def test_exact_arithmetic_index_is_bit_exact(pqt, tmp_path):
    ix, X, Y = _exact_arithmetic_index()
    path = str(tmp_path / "exact.pqt")
    IO.write_index(path, ix)
    for (k, w, T, C) in ((10, 2, 16, 200), (50, 4, 64, 512), (7, 1, 4, 64)):
        same, _ = _stagewise(pqt, ix, path, Y, k, w, T, C, exact=True)
        assert same == Y.shape[0]


def test_exact_arithmetic_wide_lists_heavily_tied_bin_keys(pqt, tmp_path):
    """Integer level-2 distances over wide lists: thousands of bin keys tie, so the ranking pass must cut
    the ties at the T-th tuple by (r1, r2) exactly (region larger than the sort buffer)."""
    ix, X, Y = _exact_arithmetic_index(N=20000, seed=11, k1=16, k2=8)
    path = str(tmp_path / "exact_wide.pqt")
    IO.write_index(path, ix)
    for (k, w, T, C) in ((20, 8, 1020, 4096), (20, 16, 2040, 2000), (10, 8, 510, 512), (10, 4, 300, 512)):
        same, _ = _stagewise(pqt, ix, path, Y[:24], k, w, T, C, exact=True)
        assert same == 24


def test_duplicate_database_ties_broken_by_id(pqt, tmp_path):
    """All vectors identical: one bin, every score tied -> the k smallest ids."""
    ix, X, Y = _exact_arithmetic_index(N=64)
    Xd = np.repeat(X[:1], 1500, axis=0)
    ixd = B.build_index(Xd, ix.P, ix.k1, ix.k2, ix.M, T=16, C=1000, codebooks=(ix.C1, ix.C2),
                        line_table=(ix.tbl_i, ix.tbl_j, ix.tbl_lam))
    path = str(tmp_path / "dup.pqt")
    IO.write_index(path, ixd)
    same, _ = _stagewise(pqt, ixd, path, np.ascontiguousarray(Xd[:3] + 0), 100, ix.k1, 16, 1000, exact=True)
    assert same == 3
    gix = pqt.pqt_index_load(path, 0)
    try:
        import torch
        ids, d = pqt.pqt_query_batch(gix, torch.from_numpy(Xd[:1].copy()).cuda(), 100, ix.k1)
        assert ids[0].tolist() == list(range(100))
    finally:
        pqt.pqt_index_free(gix)


def test_fewer_candidates_than_k_pads(pqt, tiny, tmp_path):
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    Xs = X[:40]
    ixs = B.build_index(Xs, cfg.P, cfg.k1, cfg.k2, cfg.M, T=4, C=64, codebooks=(ix.C1, ix.C2),
                        line_table=(ix.tbl_i, ix.tbl_j, ix.tbl_lam))
    p2 = str(tmp_path / "small.pqt")
    IO.write_index(p2, ixs)
    gix = pqt.pqt_index_load(p2, 0)
    try:
        ids, dists, taps = _run_debug(pqt, gix, Y[:20], 50, 1)
    finally:
        pqt.pqt_index_free(gix)
    for q in range(20):
        PU.check_query_stages(ixs, Y[q], taps, q, 50, 1, 4, 64, ids, dists)
        nc = int(taps["n_cand"][q])
        assert nc < 50 and np.all(ids[q][nc:] == -1) and np.all(np.isinf(dists[q][nc:]))


def test_large_candidate_budgets_change_the_workgroup_shape(pqt, tiny, tmp_path):
    """The re-rank workgroup grows with the candidate budget (a thread holds at most twenty keys):
    budgets on either side of 5120 and 10240, the largest one reaching every vector of the database."""
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    T = (cfg.k1 * cfg.k2) ** 2                                     # every bin of the tiny tree
    for C in (5120, 5121, 10240, 10241, 16384):
        same, _ = _stagewise(pqt, ix, path, Y[:5], cfg.k, cfg.k1, T, C)
        assert same >= 4
    _stagewise(pqt, ix, path, Y[:3], 1000, cfg.k1, T, 16384)        # k large: the short list holds 2048 keys


def test_more_runs_than_the_workgroup_keeps_in_lds(pqt, tmp_path):
    """Two huge clusters and scattered single vectors: the mean run is long, so the workgroup keeps only
    a short run list in LDS (twice what the budget needs at the mean run length), but a query among the
    scattered vectors gathers from more runs than that and reads the rest of its list from memory."""
    rng = np.random.default_rng(12345)
    P, k1, k2, M, D, T, C = 2, 8, 4, 4, 16, 1024, 3000
    centers = rng.normal(size=(2, D)) * 0.01 + np.array([[4.0] * D, [-4.0] * D])
    big = np.repeat(centers, 4940, axis=0) + rng.normal(size=(9880, D)) * 1e-3
    lone = rng.uniform(-1.5, 1.5, size=(120, D))
    X = np.concatenate([big, lone]).astype(np.float32)
    X = X[rng.permutation(X.shape[0])]
    ix = B.build_index(X, P, k1, k2, M, T=T, C=C, train_n=None, iters=8)
    mean_run = X.shape[0] / np.count_nonzero(np.diff(ix.offsets.astype(np.int64)))
    kept = 64
    while kept < T and kept < 2 * C / mean_run:
        kept *= 2
    Y = (lone[:12] + rng.normal(size=(12, D)) * 0.05).astype(np.float32)
    path = str(tmp_path / "skew.pqt")
    IO.write_index(path, ix)
    gix = pqt.pqt_index_load(path, 0)
    try:
        ids, dists, taps = _run_debug(pqt, gix, Y, 20, k1)
    finally:
        pqt.pqt_index_free(gix)
    assert kept < T and int(taps["n_slots"].max()) > kept, "the case does not reach past the LDS run list"
    for q in range(Y.shape[0]):
        PU.check_query_stages(ix, Y[q], taps, q, 20, k1, T, C, ids, dists)


def test_many_medium_runs_are_walked_by_the_wavefront(pqt, tmp_path):
    """Two huge clusters (so the workgroup keeps only 64 runs in LDS) and a few hundred small groups of
    about twenty near-identical vectors: a query among the groups gathers from well over 64 runs whose
    mean length is above sixteen, so a wavefront walks the run list as one, through several blocks of
    64 runs, the later ones read from memory."""
    rng = np.random.default_rng(4242)
    P, k1, k2, M, D, T, C = 2, 8, 4, 4, 16, 1024, 3000
    centers = rng.normal(size=(2, D)) * 0.01 + np.array([[4.0] * D, [-4.0] * D])
    big = np.repeat(centers, 20000, axis=0) + rng.normal(size=(40000, D)) * 1e-3
    spots = rng.uniform(-1.5, 1.5, size=(300, D))
    groups = np.repeat(spots, 20, axis=0) + rng.normal(size=(6000, D)) * 1e-4
    X = np.concatenate([big, groups]).astype(np.float32)
    X = X[rng.permutation(X.shape[0])]
    # the tree is trained on the groups and a few vectors of the big clusters, so that the groups spread over many bins
    C1, C2 = B.train_tree(np.concatenate([groups, big[::2000]]).astype(np.float32), P, k1, k2, iters=8)
    ix = B.build_index(X, P, k1, k2, M, T=T, C=C, codebooks=(C1, C2))
    mean_run = X.shape[0] / np.count_nonzero(np.diff(ix.offsets.astype(np.int64)))
    kept = 64
    while kept < T and kept < 2 * C / mean_run:
        kept *= 2
    Y = (spots[:12] + rng.normal(size=(12, D)) * 0.05).astype(np.float32)
    path = str(tmp_path / "groups.pqt")
    IO.write_index(path, ix)
    gix = pqt.pqt_index_load(path, 0)
    try:
        ids, dists, taps = _run_debug(pqt, gix, Y, 20, k1)
    finally:
        pqt.pqt_index_free(gix)
    nr, nc = taps["n_slots"].astype(np.int64), taps["n_cand"].astype(np.int64)
    print("runs per query", nr.tolist(), "candidates", nc.tolist(), "runs kept in LDS", kept, flush=True)
    walked = (nr > 2 * 64) & (nc >= 16 * nr)
    assert kept == 64 and walked.any(), "no query with more than two blocks of runs of mean length >= 16"
    for q in range(Y.shape[0]):
        PU.check_query_stages(ix, Y[q], taps, q, 20, k1, T, C, ids, dists)


@pytest.mark.parametrize("seed", range(12))
def test_random_shapes(pqt, tmp_path, seed):
    """Seeded random index shapes and budgets inside the documented limits (tree parts, codebook sizes,
    code bytes and format, hashing, bin order, w, T, C, k): every stage against the oracle."""
    from workloads import tiny_mixture
    rng = np.random.default_rng(1000 + seed)
    P = int(rng.choice([1, 2, 2, 4]))
    dp = int(rng.choice([4, 6, 8, 12]))                        # 6: not a multiple of four -> general level-2 path
    D = P * dp
    k1 = int(rng.choice([2, 3, 5, 8, 12]))
    k2 = int(rng.choice([1, 2, 4, 7]))
    per = [m for m in (1, 2, 4) if dp % m == 0]
    M = P * int(rng.choice(per))
    K = (k1 * k2) ** P
    hashed = bool(rng.integers(0, 2)) and K > 64
    H = int(rng.integers(17, min(K, 4096))) if hashed else K
    if H > (1 << 22):                                          # keep the oracle's pointer array small
        H = 4093
    code_format = int(rng.integers(0, 2)) if k1 >= 2 else 0
    N = int(rng.integers(500, 4000))
    X = tiny_mixture(N, d=D, seed=50 + seed)
    Y = tiny_mixture(10, d=D, seed=90 + seed)
    w = int(rng.integers(1, k1 + 1))
    R = w * k2
    T = int(rng.integers(1, min(R ** P, 3000) + 1))
    C = int(rng.integers(1, 2 * N))
    C = min(C, 16384)
    k = int(rng.integers(1, min(C, 300) + 1))
    ix = B.build_index(X, P, k1, k2, M, H=H, T=T, C=C, iters=3, code_format=code_format)
    path = str(tmp_path / f"rand{seed}.pqt")
    IO.write_index(path, ix)
    order = "static" if (P == 2 and H == K and rng.integers(0, 2)) else "fullsort"
    print(f"seed {seed}: P={P} D={D} k1={k1} k2={k2} M={M} H={H} K={K} N={N} w={w} T={T} C={C} k={k} "
          f"codes={code_format} order={order}", flush=True)
    _stagewise(pqt, ix, path, Y, k, w, T, C, order=order)


def test_hashed_index_dedupes_slots(pqt, tiny, tmp_path):
    cfg, X, Y, ix = tiny
    ixh = B.build_index(X[:3000], cfg.P, cfg.k1, cfg.k2, cfg.M, H=97, T=256, C=1024, codebooks=(ix.C1, ix.C2),
                        line_table=(ix.tbl_i, ix.tbl_j, ix.tbl_lam))
    path = str(tmp_path / "hashed.pqt")
    IO.write_index(path, ixh)
    _stagewise(pqt, ixh, path, Y[:24], 10, 4, 256, 1024)
    _stagewise(pqt, ixh, path, Y[:8], 10, cfg.k1, 1024, 3000)


def test_single_part_index(pqt, tmp_path, rng):
    X = rng.normal(size=(2000, 8)).astype(np.float32)
    Y = rng.normal(size=(20, 8)).astype(np.float32)
    ix1 = B.build_index(X, P=1, k1=8, k2=2, M=2, T=16, C=512, iters=5)
    path = str(tmp_path / "p1.pqt")
    IO.write_index(path, ix1)
    _stagewise(pqt, ix1, path, Y, 10, 3, 16, 512)
    _stagewise(pqt, ix1, path, Y, 10, 8, 3, 100)


def test_wide_selection_two_elements_per_lane(pqt, tmp_path, rng):
    """R = w*k2 = 128 > 64 lanes, k1 = 32 (two MFMA column tiles), ragged last tile."""
    X = rng.random(size=(6000, 24)).astype(np.float32)
    Y = rng.random(size=(19, 24)).astype(np.float32)
    ixw = B.build_index(X, P=2, k1=32, k2=16, M=6, T=300, C=700, iters=4)
    path = str(tmp_path / "wide.pqt")
    IO.write_index(path, ixw)
    _stagewise(pqt, ixw, path, Y, 20, 8, 300, 700)
    # R = 256: four list entries per lane; R = 512: lists sorted in LDS
    _stagewise(pqt, ixw, path, Y[:8], 20, 16, 300, 700)
    _stagewise(pqt, ixw, path, Y[:4], 20, 32, 300, 700)


def test_part_dimension_not_a_multiple_of_four(pqt, tmp_path, rng):
    """D/P = 6: the level-2 codebook keeps its plain layout (no 16-byte pieces)."""
    X = rng.random(size=(3000, 12)).astype(np.float32)
    Y = rng.random(size=(21, 12)).astype(np.float32)
    ix6 = B.build_index(X, P=2, k1=8, k2=4, M=4, T=200, C=500, iters=4)
    path = str(tmp_path / "dp6.pqt")
    IO.write_index(path, ix6)
    _stagewise(pqt, ix6, path, Y, 10, 3, 200, 500)


def test_index_from_arrays_matches_index_from_file(pqt, tiny, tmp_path):
    """pqt_index_from_arrays with host arrays and with device arrays answers exactly like the index
    loaded from the file that holds the same arrays."""
    import torch
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    arrays = dict(N=ix.N, H=ix.H, D=ix.D, P=ix.P, k1=ix.k1, k2=ix.k2, M=ix.M, T=ix.T, C=ix.C,
                  C1=ix.C1, C2=ix.C2, tbl_i=ix.tbl_i, tbl_j=ix.tbl_j, tbl_lam=ix.tbl_lam, cc=ix.cc,
                  offsets=ix.offsets, ids=ix.ids, codes=ix.codes)
    on_dev = dict(arrays)
    on_dev["offsets"] = torch.from_numpy(ix.offsets.astype(np.int64)).cuda()
    on_dev["ids"] = torch.from_numpy(ix.ids.astype(np.int32)).cuda()
    on_dev["codes"] = torch.from_numpy(ix.codes).cuda()
    yq = torch.from_numpy(Y).cuda()
    results = []
    for make in (lambda: pqt.pqt_index_load(path, 0), lambda: pqt.pqt_index_from_arrays(arrays, 0),
                 lambda: pqt.pqt_index_from_arrays(on_dev, 0)):
        gix = make()
        try:
            ids, d = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)
            torch.cuda.synchronize()
            results.append((ids.cpu(), d.cpu()))
            info = pqt.pqt_index_info(gix)
            assert (info["N"], info["H"], info["T"], info["C"]) == (ix.N, ix.H, ix.T, ix.C)
        finally:
            pqt.pqt_index_free(gix)
    for ids, d in results[1:]:
        assert torch.equal(ids, results[0][0]) and torch.equal(d.view(torch.int32), results[0][1].view(torch.int32))
    bad = dict(arrays)
    bad["offsets"] = ix.offsets.copy()
    bad["offsets"][3] = bad["offsets"][-1] + 1
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_index_from_arrays(bad, 0)
    assert e.value.code == pqt.PQT_EFORMAT


def _check_exact(pqt, gix, ix, X, Y, k_short, k, w, bit_exact):
    """pqt_query_batch_exact against the oracle: the short list is the line-quantisation top-k_short
    (already checked stage by stage elsewhere; taken from the GPU here), its exact re-ranking must be
    the oracle's on the same list."""
    import torch
    yq = torch.from_numpy(np.ascontiguousarray(Y)).cuda()
    short, _ = pqt.pqt_query_batch(gix, yq, k_short, w)
    ids, d = pqt.pqt_query_batch_exact(gix, yq, k_short, k, w)
    ids_all, d_all = pqt.pqt_query_batch_exact(gix, yq, k_short, k_short, w)
    torch.cuda.synchronize()
    short, ids, d, ids_all, d_all = (PU.to_np(t) for t in (short, ids, d, ids_all, d_all))
    for q in range(Y.shape[0]):
        o_ids, o_d = Q.exact_rerank_short_list(Y[q], X, short[q], k_short)
        have = o_ids >= 0
        # every exact distance within tolerance (compare through the id)
        lookup = dict(zip(o_ids[have].tolist(), o_d[have].tolist()))
        assert sorted(ids_all[q][ids_all[q] >= 0].tolist()) == sorted(o_ids[have].tolist()), "id set of the short list"
        got = np.array([lookup[i] for i in ids_all[q][ids_all[q] >= 0].tolist()])
        gd = d_all[q][ids_all[q] >= 0]
        assert PU.close(gd, got), f"query {q}: exact distances"     # sums of squared differences: relative error only
        # the order is the order of the GPU's own distances, ties by id; the first k are the k-result call
        o = np.lexsort((ids_all[q][ids_all[q] >= 0], gd))
        assert np.array_equal(o, np.arange(o.shape[0])), f"query {q}: not sorted by (distance, id)"
        assert np.array_equal(ids[q], ids_all[q][:k]) and np.array_equal(d[q], d_all[q][:k])
        assert np.all(ids_all[q][have.sum():] == -1) and np.all(np.isinf(d_all[q][have.sum():]))
        if bit_exact:
            assert np.array_equal(ids_all[q], o_ids) and np.array_equal(d_all[q].astype(np.float64)[have], o_d[have])


def test_exact_rerank_of_short_list(pqt, tiny, tmp_path):
    import torch
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    gix = pqt.pqt_index_load(path, 0)
    try:
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_query_batch_exact(gix, torch.from_numpy(Y).cuda(), 50, 10, cfg.w)
        assert e.value.code == pqt.PQT_EINVAL                      # no vectors attached yet
        pqt.pqt_index_set_vectors(gix, X)                          # host array: copied
        _check_exact(pqt, gix, ix, X, Y[:40], 50, 10, cfg.w, bit_exact=False)
        _check_exact(pqt, gix, ix, X, Y[:10], 256, 100, cfg.k1, bit_exact=False)     # more than the candidates of some queries
        Xd = torch.from_numpy(X).cuda()
        pqt.pqt_index_set_vectors(gix, Xd)                         # device tensor: used in place
        _check_exact(pqt, gix, ix, X, Y[:10], 64, 64, cfg.w, bit_exact=False)
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_query_batch_exact(gix, torch.from_numpy(Y).cuda(), 10, 20, cfg.w)   # k > k_short
        assert e.value.code == pqt.PQT_EINVAL
    finally:
        pqt.pqt_index_free(gix)
    # integer data: fp32 and uint8 storage, every operation exact -> equal to the float64 oracle bit for bit
    ixe, Xe, Ye = _exact_arithmetic_index()
    path = str(tmp_path / "exact.pqt")
    IO.write_index(path, ixe)
    gix = pqt.pqt_index_load(path, 0)
    try:
        for stored in (Xe, Xe.astype(np.uint8)):
            pqt.pqt_index_set_vectors(gix, stored)
            _check_exact(pqt, gix, ixe, Xe, Ye[:32], 100, 20, 2, bit_exact=True)
    finally:
        pqt.pqt_index_free(gix)


def _whole_number_index(pqt, N, D, P, k1, k2, M, H=None, T=64, C=1024, fmt=0, distinct=None, seed=3):
    """An index over whole-number vectors built by the library, and its vectors: (index, X on the GPU)."""
    import torch
    from paper_1702_05911_amd import builder
    gen = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randint(0, 32, (N, D), generator=gen, device="cuda").float()
    if distinct:
        X = X[torch.randint(0, distinct, (N,), generator=gen, device="cuda")].contiguous()
    return builder.build_index_native(X, P=P, k1=k1, k2=k2, M=M, H=H, T=T, C=C, iters=4, code_format=fmt), X


@pytest.mark.parametrize("distinct, k, C, nq", [
    (0, 257, 1500, 1100),                  # one result more than threads
    (0, 1000, 4096, 1100),
    (0, 1024, 4096, 1030),                 # the longest list
    (40, 600, 2000, 1100),                 # forty different vectors: crowded bins, the survivors are sorted
    (40, 100, 2000, 1100),                 # fewer results than threads, more survivors: sorted or selected exactly
])
def test_long_result_lists(pqt, distinct, k, C, nq):
    """Result lists longer than the workgroup (256 threads for these batches) against a sort of the tapped scores by
    (score, id): equal, ids and distance bits."""
    import torch
    ix, X = _whole_number_index(pqt, 6000, 16, 2, 4, 4, 4, T=256, C=C, distinct=distinct)
    try:
        Y = X[:nq] + 0.25
        ids, d, taps = pqt.pqt_query_batch_debug(ix, Y, k, 4, taps=("scores", "cand_ids", "n_cand"))
        pid, pd = pqt.pqt_query_batch(ix, Y, k, 4)
        torch.cuda.synchronize()
        col = torch.arange(C, device="cuda")
        free = col[None] >= taps["n_cand"][:, None]
        by_id = torch.argsort(torch.where(free, 1 << 40, taps["cand_ids"]), dim=1, stable=True)
        score = torch.where(free, float("inf"), taps["scores"]).gather(1, by_id)
        order = by_id.gather(1, torch.argsort(score, dim=1, stable=True))[:, :k]
        want = torch.where(free, -1, taps["cand_ids"]).gather(1, order)
        want_d = torch.where(free, float("inf"), taps["scores"]).gather(1, order)
        for got, gd in ((ids, d), (pid, pd)):
            assert torch.equal(got, want) and torch.equal(gd, want_d)
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("M, fmt", [(12, 0), (12, 1), (32, 1), (16, 1), (6, 1)])
def test_code_widths(pqt, tmp_path, M, fmt):
    """Codes read as three, six and sixteen words (M = 16: eight, M = 6 pairs: three, byte by byte): every stage and the
    plain entry point against the oracle."""
    from workloads import tiny_mixture
    X, Y = tiny_mixture(2500, d=2 * M, seed=8), tiny_mixture(12, d=2 * M, seed=9)
    ix = B.build_index(X, 2, 6, 3, M, T=60, C=900, iters=3, code_format=fmt)
    path = str(tmp_path / "width.pqt")
    IO.write_index(path, ix)
    _stagewise(pqt, ix, path, Y, 40, 4, 60, 900)


@pytest.mark.parametrize("M, C", [(12, 400), (12, 3000), (32, 300), (32, 4096)])
def test_wide_pair_codes_by_words_and_bytes(pqt, M, C):
    """(pair, lambda) codes of six and sixteen words are read byte by byte where workgroups of 1,024 threads would not all run at
    once: the same results from calls of 100 queries (words), 300 and 1,024 (bytes) and 1,025 (words, smaller workgroups), and
    from the debug entry point."""
    import torch
    ix, X = _whole_number_index(pqt, 6000, 2 * M, 2, 8, 4, M, T=256, C=C, fmt=1)
    try:
        Y = X[:1025] + 0.25
        ids, d, _ = pqt.pqt_query_batch_debug(ix, Y, 50, 4, taps=("n_tuples",))
        for nq in (100, 300, 1024, 1025):
            got, gd = pqt.pqt_query_batch(ix, Y[:nq].contiguous(), 50, 4)
            assert torch.equal(got, ids[:nq]) and torch.equal(gd, d[:nq]), nq
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("H", [None, 4099])
@pytest.mark.parametrize("C", [30, 60, 120, 400, 3000])
def test_ranking_routes_agree(pqt, C, H):
    """Sparse to full two-part indexes and batches on both sides of every line of the choice between head pass and
    headless ranking: the plain entry point returns what the debug one does, which always ranks all T tuples."""
    import torch
    ix, X = _whole_number_index(pqt, 12_000, 16, 2, 16, 8, 4, H=H, T=700, C=C)
    try:
        for nq in (1, 3, 4, 15, 16, 95, 96, 513, 2048, 2049):
            Y = X[:nq] + 0.25
            ids, d, _ = pqt.pqt_query_batch_debug(ix, Y, min(C, 20), 5, taps=("n_tuples",))
            pid, pd = pqt.pqt_query_batch(ix, Y, min(C, 20), 5)
            assert torch.equal(ids, pid) and torch.equal(d, pd), nq
            if nq <= 513:
                nid, nd = torch.empty_like(ids), torch.empty_like(d)
                pqt.pqt_query_batch_noalloc(ix, Y, min(C, 20), 5, nid, nd)
                assert torch.equal(ids, nid) and torch.equal(d, nd), nq
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("M", [8, 12])
@pytest.mark.parametrize("C", [205, 217, 252, 264])
def test_ranking_routes_agree_for_pair_codes(pqt, M, C):
    """The head pass of large batches of (pair, lambda) codes is left out from a mean need of 88 tuples on (up to eight sub-parts) or 72: on both
    sides of both lines a batch gets what its queries get by themselves."""
    import torch
    rng = np.random.default_rng(29)
    X = rng.integers(0, 64, (3000, 24)).astype(np.float32)
    Y = torch.from_numpy(rng.integers(0, 64, (2100, 24)).astype(np.float32)).cuda()
    from paper_1702_05911_amd import builder
    gix = builder.build_index_native(X, P=2, k1=8, k2=4, M=M, T=500, C=C, train_n=3000, code_format=1)
    try:
        ids, dists = pqt.pqt_query_batch(gix, Y, 20, 6)
        for s in range(0, 2100, 700):
            few = pqt.pqt_query_batch(gix, Y[s:s + 70].contiguous(), 20, 6)
            assert torch.equal(few[0], ids[s:s + 70]) and torch.equal(few[1], dists[s:s + 70])
    finally:
        pqt.pqt_index_free(gix)


@pytest.mark.parametrize("T", [1500, 2500, 6000])
@pytest.mark.parametrize("H, budgets", [(None, (20, 26, 40, 100)), (4099, (150, 240, 400, 900))])
def test_ranking_routes_agree_for_long_lists(pqt, H, budgets, T):
    """As above with more than 1,024 tuples, which no re-rank workgroup ranks: every workgroup size of the full pass, with and
    without a head pass of two and of three levels (the budgets stand for mean numbers of needed tuples on both sides of
    each line)."""
    import torch
    ix, X = _whole_number_index(pqt, 12_000, 16, 2, 16, 12, 4, H=H, T=T, C=1000)
    try:
        for C in budgets:
            pqt.pqt_set_budget(ix, T, C)
            for nq in (1, 256, 257, 512, 513, 1025, 2049):
                Y = X[:nq] + 0.25
                ids, d, _ = pqt.pqt_query_batch_debug(ix, Y, min(C, 20), 8, taps=("n_tuples",))
                pid, pd = pqt.pqt_query_batch(ix, Y, min(C, 20), 8)
                assert torch.equal(ids, pid) and torch.equal(d, pd), (C, nq)
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("D, stored, k_short, k, distinct", [
    (16, "u8", 1, 1, 0),                   # a row is one piece: 64 rows per wavefront
    (48, "u8", 1000, 100, 0),              # three pieces: one lane of four idle
    (128, "u8", 1024, 1024, 0),            # the longest list, all of it returned
    (20, "f32", 257, 63, 0),               # five pieces
    (260, "f32", 65, 64, 0),               # more pieces than lanes
    (32, "u8", 900, 50, 3),                # three different vectors: a bin holds hundreds, all are sorted
    (32, "f32", 700, 699, 0),              # more results asked for than some queries have
])
def test_exact_rerank_edges(pqt, D, stored, k_short, k, distinct):
    """Row widths, list lengths and ties of the exact re-ranking: whole numbers, so the distances are exact and the result
    is a sort of the short list by (distance, id)."""
    import torch
    ix, X = _whole_number_index(pqt, 5000, D, 2, 4, 2, 2, T=64, C=1024 if k_short != 700 else 700, distinct=distinct)
    try:
        if k_short == 700:
            pqt.pqt_set_budget(ix, 3, 700)                           # three tuples: fewer candidates than results
        pqt.pqt_index_set_vectors(ix, X.to(torch.uint8) if stored == "u8" else X)
        Y = X[:9] + 1.0
        short, _ = pqt.pqt_query_batch(ix, Y, k_short, 3)
        ids, d = pqt.pqt_query_batch_exact(ix, Y, k_short, k, 3)
        short = torch.sort(torch.where(short < 0, 1 << 40, short), dim=1).values
        have = short < (1 << 40)
        true = ((X.double()[torch.where(have, short, 0)] - Y.double()[:, None]) ** 2).sum(2)
        true = torch.where(have, true, float("inf"))
        order = torch.argsort(true, dim=1, stable=True)[:, :k]
        assert torch.equal(torch.where(have, short, -1).gather(1, order), ids)
        assert torch.equal(true.gather(1, order).float(), d)
    finally:
        pqt.pqt_index_free(ix)


def test_native_builder(pqt, tiny, tmp_path):
    """pqt_builder_*: vectors streamed in ragged chunks; the saved index satisfies the oracle's
    definitions (bin of every vector, nearest code point, sorted lists) and answers queries exactly as
    the oracle does on that index."""
    import torch
    cfg, X, Y, ix = tiny
    params = dict(N=cfg.N, H=ix.H, D=ix.D, P=ix.P, k1=ix.k1, k2=ix.k2, M=ix.M, T=ix.T, C=ix.C,
                  C1=ix.C1, C2=ix.C2, tbl_i=ix.tbl_i, tbl_j=ix.tbl_j, tbl_lam=ix.tbl_lam, cc=ix.cc)
    Xd = torch.from_numpy(X).cuda()
    b = pqt.pqt_builder_create(params, 0)
    try:
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_builder_finish(b)                              # nothing added yet
        assert e.value.code == pqt.PQT_EINVAL
        for lo, hi in ((0, 1), (1, 4097), (4097, 4097), (4097, cfg.N)):
            pqt.pqt_builder_add(b, Xd[lo:hi].contiguous())
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_builder_add(b, Xd[:1].contiguous())            # more than N
        assert e.value.code == pqt.PQT_EINVAL
        gix = pqt.pqt_builder_finish(b)
    finally:
        pqt.pqt_builder_free(b)
    path = str(tmp_path / "native.pqt")
    try:
        pqt.pqt_index_save(gix, path)
    finally:
        pqt.pqt_index_free(gix)
    nix = IO.read_index(path)
    off = nix.offsets.astype(np.int64)
    assert off[0] == 0 and off[-1] == cfg.N and np.all(np.diff(off) >= 0)
    assert np.array_equal(np.sort(nix.ids), np.arange(cfg.N, dtype=np.uint32))
    for name in ("C1", "C2", "tbl_i", "tbl_j", "tbl_lam", "cc"):
        assert np.array_equal(getattr(nix, name), getattr(ix, name)), name
    slot_of = np.repeat(np.arange(nix.H), np.diff(off))
    want_slots = B.bin_slots_batch(X, nix.C1, nix.C2, nix.H)
    assert np.mean(slot_of != want_slots[nix.ids]) <= 2e-3       # fp32 vs float64 near-ties only
    for s in np.nonzero(np.diff(off) > 1)[0][:200]:
        assert np.all(np.diff(nix.ids[off[s]:off[s + 1]].astype(np.int64)) > 0)   # ids ascend inside a slot
    # codes: the chosen code point is (within fp32 rounding) as near as the nearest one
    # (the encoder takes the smallest of 256 fp32 values of Eq. 9 on the vector's own level-1 distances:
    # the chosen point may lose to the best one by the rounding of both values)
    ds = nix.D // nix.M
    kenc = (PU.kappa(ds) + 8.0) * PU.U32
    for t in np.random.default_rng(3).integers(0, cfg.N, size=300):
        x = X[nix.ids[t]].astype(np.float64)
        Sl = PU.lut_magnitudes(nix, PU.subpart_magnitudes(nix, x))
        for m in range(nix.M):
            pts = B.code_points(B.subpart_centroids(nix.C1, nix.M, m), nix.tbl_i[m], nix.tbl_j[m], nix.tbl_lam[m])
            d = np.sum((pts - x[m * ds:(m + 1) * ds][None]) ** 2, axis=1)
            got, best = int(nix.codes[t, m]), int(np.argmin(d))
            assert d[got] - d[best] <= kenc * (Sl[m, got] + Sl[m, best]), (t, m, got, best)
    # the index is input data: full stage-wise parity on it
    same, _ = _stagewise(pqt, nix, path, Y[:30], cfg.k, cfg.w, cfg.T, cfg.C)
    assert same >= 27


def _distortion(Xp, cen):
    return float(np.mean(np.min(B.sqdist_matrix(Xp, cen), axis=1)))


def test_training_on_the_gpu(pqt, tiny):
    """pqt_train: after one Lloyd iteration every centroid is the mean of the vectors nearest to the start
    centroids (vectors at evenly spaced places of the sample, of the cell for level 2), checked with the
    oracle's distance routine; after twenty the distortion matches the oracle's own Lloyd training; the
    line table is ordered by (i, j, lambda), shares the 256 code points out in proportion to the votes
    the oracle counts, and places them inside the range of the lambdas voted on each line."""
    import torch
    cfg, X, Y, _ = tiny
    P, k1, k2, M, D = cfg.P, cfg.k1, cfg.k2, cfg.M, cfg.D
    dp, ds, n = D // P, D // M, 6000
    Xd = torch.from_numpy(X[:n]).cuda()
    one = pqt.pqt_train(Xd, P=P, k1=k1, k2=k2, M=M, iters=1, n_table=0)
    again = pqt.pqt_train(Xd, P=P, k1=k1, k2=k2, M=M, iters=1, n_table=0)
    for name in one:
        assert np.array_equal(one[name], again[name]), f"{name}: training is not deterministic"
    for p in range(P):
        Xp = X[:n, p * dp:(p + 1) * dp].astype(np.float64)
        start = Xp[(np.arange(k1) * n) // k1]
        lab = np.argmin(B.sqdist_matrix(Xp, start), axis=1)
        for i in range(k1):
            np.testing.assert_allclose(one["C1"][p, i], Xp[lab == i].mean(axis=0), rtol=1e-5, atol=1e-6)
        # level 2: cells of the finished level-1 quantiser, each trained on its own members
        lab1 = np.argmin(B.sqdist_matrix(Xp, one["C1"][p].astype(np.float64)), axis=1)
        for i in range(k1):
            sub = Xp[lab1 == i]
            if sub.shape[0] <= k2:
                continue
            start2 = sub[(np.arange(k2) * sub.shape[0]) // k2]
            lab2 = np.argmin(B.sqdist_matrix(sub, start2), axis=1)
            for j in range(k2):
                if np.any(lab2 == j):
                    np.testing.assert_allclose(one["C2"][p, i, j], sub[lab2 == j].mean(axis=0), rtol=1e-5, atol=1e-6)
    full = pqt.pqt_train(Xd, P=P, k1=k1, k2=k2, M=M, iters=20, n_table=n)
    oC1, oC2 = B.train_tree(X[:n], P, k1, k2, iters=20)
    for p in range(P):
        Xp = X[:n, p * dp:(p + 1) * dp].astype(np.float64)
        g, o = _distortion(Xp, full["C1"][p].astype(np.float64)), _distortion(Xp, oC1[p].astype(np.float64))
        print(f"part {p}: level-1 distortion GPU {g:.6f} oracle {o:.6f}", flush=True)
        assert abs(g - o) <= 0.01 * o
        g2 = _distortion(Xp, full["C2"][p].reshape(k1 * k2, dp).astype(np.float64))
        o2 = _distortion(Xp, oC2[p].reshape(k1 * k2, dp).astype(np.float64))
        assert g2 <= 1.03 * o2 and g2 < g
    np.testing.assert_allclose(full["cc"], B.pair_table(full["C1"], M), rtol=1e-6, atol=1e-9)
    pairs = Q.centroid_pairs(k1)
    for m in range(M):
        ti, tj, tl = full["tbl_i"][m], full["tbl_j"][m], full["tbl_lam"][m]
        ent = list(zip(ti.tolist(), tj.tolist(), tl.tolist()))
        assert ent == sorted(ent) and all(i < j < k1 for i, j, _ in ent)
        bp, bl, _ = B.best_lines(X[:n, m * ds:(m + 1) * ds].astype(np.float64), B.subpart_centroids(full["C1"], M, m))
        use = np.bincount(bp, minlength=len(pairs))
        got = np.zeros(len(pairs), np.int64)
        for i, j, _ in ent:
            got[pairs.index((i, j))] += 1
        quota = use * 256.0 / use.sum()
        # largest-remainder shares lie within one of the exact quota; an fp32 near-tie may move a vote or two
        assert got.sum() == 256 and np.all(np.abs(got - quota) <= 1.0 + 256.0 * 3 / n), (m, np.max(np.abs(got - quota)))
        for q in np.nonzero(got)[0]:
            lams = bl[bp == q]
            mine = tl[(ti == pairs[q][0]) & (tj == pairs[q][1])]
            assert lams.size and mine.min() >= lams.min() - 1e-3 and mine.max() <= lams.max() + 1e-3
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_train(Xd, P=3, k1=k1, k2=k2, M=M)
    assert e.value.code in (pqt.PQT_EINVAL, pqt.PQT_EUNSUPPORTED)


@pytest.mark.parametrize("n,D,P,k1,k2", [
    (63, 8, 1, 4, 2), (65, 2, 2, 3, 5), (1000, 64, 1, 16, 8), (257, 66, 1, 5, 3), (4133, 128, 1, 48, 7), (700, 129, 1, 49, 2),
    (3001, 132, 2, 33, 12), (150_001, 24, 2, 12, 13), (2500, 256, 4, 31, 1),
    (66_001, 16, 1, 13, 12),               # short rows of a large sample: level 1 by whole tiles, level 2 (with fewer centroids) by the step kernel
    (45_001, 64, 2, 8, 9),                 # the other way round
    (45_000, 512, 4, 40, 36),              # 128 dimensions: level 1 by tiles, its 160 groups of level 2 by the step kernel
    (700, 264, 2, 20, 3),                  # rows beyond the tiles': 24 centroids at a time
    (900, 262, 2, 20, 3),                  # the same where they are not read in 16-byte pieces
    (36_000, 520, 1, 120, 2),              # chunks of two of the step kernel's tiles, sums of the second added to the first's
    (36_000, 521, 1, 120, 2),              # the same value by value
    (20_000, 132, 1, 256, 2),              # the same where wavefronts share a tile
])
def test_training_tile_edges(pqt, n, D, P, k1, k2):
    """One Lloyd iteration on small whole numbers, where sums and distances are exact: every centroid is the mean of the vectors
    nearest to the start centroids, rounded once; rows of 1 to 521 values, up to 64 and 128 of them with whole rows on the chip, cells
    on both sides of what a wavefront owns, samples around a tile and beyond one chunk per compute unit.  Level 2 starts from
    centroids that are not whole: a distance of dp squares is off by (dp + 2) 2^-24 of itself at most, and cells near to a vector that lies
    halfway between them to twice that are left out."""
    import torch
    dp = D // P

    def sqdist(x, c):                       # exact for whole numbers
        return (x * x).sum(axis=1)[:, None] + (c * c).sum(axis=1)[None, :] - 2.0 * (x @ c.T)
    X = np.random.default_rng(n).integers(0, 16, (n, D)).astype(np.float32)
    got = pqt.pqt_train(torch.from_numpy(X).cuda(), P=P, k1=k1, k2=k2, M=P, iters=1, n_table=0)
    again = pqt.pqt_train(torch.from_numpy(X).cuda(), P=P, k1=k1, k2=k2, M=P, iters=1, n_table=0)
    seen = 0
    for p in range(P):
        Xp = X[:, p * dp:(p + 1) * dp].astype(np.float64)
        lab = np.argmin(sqdist(Xp, Xp[(np.arange(k1) * n) // k1]), axis=1)
        for i in range(k1):
            if np.any(lab == i):
                np.testing.assert_array_equal(got["C1"][p, i], Xp[lab == i].mean(axis=0).astype(np.float32))
        # the cells of the finished quantiser
        d1 = sqdist(Xp, got["C1"][p].astype(np.float64))
        lab = np.argmin(d1, axis=1)
        close = d1 <= d1.min(axis=1, keepdims=True) * (1.0 + (dp + 2) * 2.0 ** -23)
        open_cells = np.any(close[close.sum(axis=1) > 1], axis=0)
        for i in np.nonzero(~open_cells)[0]:
            sub = Xp[lab == i]
            if sub.shape[0] <= k2:
                continue
            lab2 = np.argmin(sqdist(sub, sub[(np.arange(k2) * sub.shape[0]) // k2]), axis=1)
            for j in range(k2):
                if np.any(lab2 == j):
                    np.testing.assert_array_equal(got["C2"][p, i, j], sub[lab2 == j].mean(axis=0).astype(np.float32))
            seen += 1
    assert seen > 0, "no cell of level 2 was looked at"
    for name in got:
        assert np.array_equal(got[name], again[name]), f"{name}: training is not deterministic"


@pytest.mark.parametrize("k1", [2, 5])           # by the step kernel, and by whole tiles, the last of which ends past 2^32
def test_training_most_vectors(pqt, k1):
    """The most training vectors (2^32 - 2).  Values 0 .. 15 but for the start centroids from the second on, far from these and each other,
    and the last vector, which shares a cell with the last of them; sums are whole numbers below 2^53, so every mean is rounded once."""
    import torch
    n = (1 << 32) - 2
    free, _ = torch.cuda.mem_get_info()
    if free < 80 << 30:
        pytest.skip("needs 80 GB of GPU memory")
    X = torch.empty((n, 1), dtype=torch.float32, device="cuda")
    pattern = (torch.arange(1 << 26, device="cuda") % 16).to(torch.float32).view(-1, 1)
    for s in range(0, n, 1 << 26):
        X[s:s + (1 << 26)] = pattern[:n - s]
    far = {n * j // k1: 4096.0 * j for j in range(1, k1)}
    far[n - 1] = 4096.0 * (k1 - 1) + 1000.0
    for at, value in far.items():
        X[at] = value
    # 2^28 of every value, but one 14 and one 15 less (i mod 16 ends with 13)
    total = (1 << 28) * 120 - 14 - 15 - sum(at % 16 for at in far)
    want = np.array([[total / (n - len(far))]] + [[4096.0 * j] for j in range(1, k1 - 1)] + [[4096.0 * (k1 - 1) + 500.0]]).astype(np.float32)
    try:
        got = pqt.pqt_train(X, P=1, k1=k1, k2=1, M=1, iters=1, n_table=0)
    finally:
        del X, pattern
        torch.cuda.empty_cache()
    np.testing.assert_array_equal(got["C1"][0], want)
    np.testing.assert_array_equal(got["C2"][0, :, 0], want)


def test_pair_lambda_codes(pqt, tiny_pair, tmp_path):
    """Codes stored as (centroid pair, lambda level): stage-wise parity of the query path on an
    oracle-built index; the lut tap is refused; a pair byte beyond the last pair is a format error."""
    import torch
    cfg, X, Y, ix = tiny_pair
    path = str(tmp_path / "pair.pqt")
    IO.write_index(path, ix)
    same, decided = _stagewise(pqt, ix, path, Y[:40], cfg.k, cfg.w, cfg.T, cfg.C)
    assert same >= 36
    # ragged budgets: few candidates, one tuple
    _stagewise(pqt, ix, path, Y[:8], 5, 1, 1, 7)
    gix = pqt.pqt_index_load(path, 0)
    try:
        inf = pqt.pqt_index_info(gix)
        assert inf["code_format"] == pqt.PQT_CODES_PAIR_LAMBDA and inf["code_bytes"] == 2 * cfg.M
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_query_batch_debug(gix, torch.from_numpy(Y[:2]).cuda(), cfg.k, cfg.w, taps=("lut",))
        assert e.value.code == pqt.PQT_EINVAL
        back = pqt.pqt_index_export(gix, ("codes",))["codes"]
        assert np.array_equal(PU.to_np(back), ix.codes)
    finally:
        pqt.pqt_index_free(gix)
    arrays = dict(N=ix.N, H=ix.H, D=ix.D, P=ix.P, k1=ix.k1, k2=ix.k2, M=ix.M, T=ix.T, C=ix.C, C1=ix.C1, C2=ix.C2,
                  cc=ix.cc, offsets=ix.offsets, ids=ix.ids, codes=ix.codes.copy(), code_format=1)
    arrays["codes"][17, 2] = ix.k1 * (ix.k1 - 1) // 2          # one past the last pair
    for on_device in (False, True):
        a = dict(arrays)
        if on_device:
            for n in ("offsets", "ids"):
                a[n] = torch.from_numpy(arrays[n].astype(np.int64)).cuda()
            a["codes"] = torch.from_numpy(arrays["codes"]).cuda()
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_index_from_arrays(a, 0)
        assert e.value.code == pqt.PQT_EFORMAT


@pytest.mark.parametrize("k1, M", [(2, 3), (3, 12), (4, 1), (12, 24), (16, 8), (17, 4), (20, 12), (23, 2), (23, 6)])
def test_pair_table_edges(pqt, tmp_path, k1, M):
    """The table of centroid pairs on the chip: one pair to the most of a byte, odd and even numbers of them (an odd one is
    padded), codes read by words and by bytes, by the small batches' kernel and the others."""
    rng = np.random.default_rng(k1)
    X = rng.integers(0, 32, (900, 24)).astype(np.float32)
    Y = rng.integers(0, 32, (300, 24)).astype(np.float32)
    ix = B.build_index(X, 1, k1, 4, M, T=3 * k1, C=500, iters=3, code_format=1)
    path = str(tmp_path / "pairs.pqt")
    IO.write_index(path, ix)
    _stagewise(pqt, ix, path, Y[:6], 10, 2, 3 * k1, 500)
    import torch
    gix = pqt.pqt_index_load(path, 0)
    try:
        few, _ = pqt.pqt_query_batch(gix, torch.from_numpy(Y[:6]).cuda(), 10, 2)
        many, _ = pqt.pqt_query_batch(gix, torch.from_numpy(np.tile(Y, (8, 1))).cuda(), 10, 2)
        assert torch.equal(many[:6], few) and torch.equal(many[:300], many[2100:])
    finally:
        pqt.pqt_index_free(gix)


def test_pair_code_limits(pqt, tmp_path):
    """The most sub-parts of (pair, lambda) codes with the longest result list and few centroids, where the survivors of the selection
    take more room than the table of pairs, are answered; with the most centroids they are refused (the limit is 16 bytes for each of 256 pairs)."""
    import torch
    rng = np.random.default_rng(5)
    X = rng.integers(0, 32, (3000, 64)).astype(np.float32)
    Y = rng.integers(0, 32, (3, 64)).astype(np.float32)
    ix = B.build_index(X, 2, 5, 16, 64, T=2048, C=2000, iters=2, code_format=1)
    path = str(tmp_path / "few.pqt")
    IO.write_index(path, ix)
    _stagewise(pqt, ix, path, Y, 1024, 5, 2048, 2000)
    path = str(tmp_path / "many.pqt")
    IO.write_index(path, B.build_index(X, 2, 23, 2, 64, T=64, C=100, iters=1, code_format=1))
    gix = pqt.pqt_index_load(path, 0)
    try:
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_query_batch(gix, torch.from_numpy(Y).cuda(), 10, 2)
        assert e.value.code == pqt.PQT_EUNSUPPORTED
    finally:
        pqt.pqt_index_free(gix)


@pytest.mark.parametrize("M", [7, 8, 9, 15, 31, 33, 39, 40, 47, 48, 57, 63, 64])
def test_pair_codes_in_pieces(pqt, tmp_path, M):
    """(pair, lambda) codes that are read in pieces of eight sub-parts: lengths around a piece, and around the two and four that
    long codes are read in.  Whole numbers: a code's score is the same sum in every kernel."""
    import torch
    rng = np.random.default_rng(M)
    X = rng.integers(0, 32, (700, M)).astype(np.float32)
    Y = torch.from_numpy(np.tile(rng.integers(0, 32, (300, M)).astype(np.float32), (8, 1))).cuda()
    ix = B.build_index(X, 1, 5, 4, M, T=20, C=400, iters=3, code_format=1)
    path = str(tmp_path / "pieces.pqt")
    IO.write_index(path, ix)
    _stagewise(pqt, ix, path, Y[:4].cpu().numpy(), 10, 3, 20, 400)
    gix = pqt.pqt_index_load(path, 0)
    try:
        want = pqt.pqt_query_batch_debug(gix, Y[:300].contiguous(), 10, 3, taps=("scores",))[:2]
        for nq in (3, 300, 2400):           # one launch, and three with the largest and the smallest workgroups
            ids, dists = pqt.pqt_query_batch(gix, Y[:nq].contiguous(), 10, 3)
            for first in range(0, nq, 300):
                n = min(300, nq - first)
                assert torch.equal(ids[first:first + n], want[0][:n]) and torch.equal(dists[first:first + n], want[1][:n])
    finally:
        pqt.pqt_index_free(gix)


@pytest.mark.parametrize("many", [0, 12_300])     # more than 8,192 vectors in the second call: 64 per workgroup instead of 16
@pytest.mark.parametrize("N, D, P, k1, k2, M, fmt, offset", [
    (63, 16, 2, 16, 8, 4, 0, 0),           # one vector short of a workgroup; one tile of centroids
    (65, 24, 2, 17, 3, 4, 0, 0),           # one vector in the second workgroup; a second, nearly empty tile of centroids
    (66, 24, 2, 32, 3, 6, 0, 0),           # as many centroids as a lane keeps distances of in registers (33: not)
    (200, 48, 1, 33, 2, 1, 0, 0),          # one sub-part of two slabs, centroids in two passes over them
    (130, 40, 4, 5, 7, 8, 0, 0),           # four tree parts, pieces of one sub-part each
    (129, 30, 2, 6, 4, 6, 0, 0),           # sub-parts of five dimensions: no 16-byte rows
    (100, 16, 2, 8, 1, 4, 0, 1),           # vectors that do not start at a multiple of 16 bytes
    (70, 16, 1, 256, 2, 2, 0, 0),          # the most centroids
    (131, 12, 1, 4, 300, 3, 0, 0),         # more children than threads
    (66, 40, 2, 3, 5, 5 * 2, 0, 0),        # children of four lanes and one more; a part's five 16-byte pieces, one after four
    (130, 32, 1, 4, 9, 4, 0, 0),           # eight children and one more; eight pieces
    (67, 16, 2, 20, 7, 4, 1, 0),           # (pair, lambda) codes
    (130, 16, 2, 7, 3, 4, 0, 0),           # 16-byte rows and numbers of centroids that are no multiple of four, so that a
    (77, 64, 2, 21, 2, 4, 0, 0),           # wavefront's distances outgrow its staged values by an odd number of words
    (70, 32, 4, 15, 4, 4, 1, 0),
    (50, 256, 1, 240, 2, 8, 0, 0),         # distances that do not fit the LDS of the kernel for few vectors
    (17, 64, 2, 16, 4, 64, 0, 0),          # the most sub-parts; one vector in the second workgroup of 16
    (15, 48, 4, 12, 3, 12, 1, 0),          # one vector short of such a workgroup
    (90, 6, 2, 3, 2, 6, 1, 1),             # sub-parts of one dimension
])
def test_builder_edges(pqt, N, D, P, k1, k2, M, fmt, offset, many):
    """Bins, codes and lists at the edges of the placing kernel's tiles, slabs and passes, against the oracle.  Codebooks,
    vectors and lambdas are small whole numbers and multiples of 1/16, so that every distance is exact in fp32 and float64
    and the results are equal, ties included; slots are hashed for the odd H."""
    import torch
    rng = np.random.default_rng(5)
    N += many
    top = 8 if fmt else 16
    dp = D // P
    X = rng.integers(0, top, (N, D)).astype(np.float32)
    C1 = rng.integers(0, top, (P, k1, dp)).astype(np.float32)
    C2 = rng.integers(0, top, (P, k1, k2, dp)).astype(np.float32)
    ti, tj = (rng.integers(0, k1, (M, 256)).astype(np.uint8) for _ in range(2))
    tl = (rng.integers(-8, 25, (M, 256)) / 16.0).astype(np.float32)
    H = max(1, min((k1 * k2) ** P, 1001))
    params = dict(N=N, H=H, D=D, P=P, k1=k1, k2=k2, M=M, T=16, C=16, C1=C1, C2=C2, tbl_i=ti, tbl_j=tj, tbl_lam=tl,
                  cc=B.pair_table(C1, M), code_format=fmt)
    buf = torch.empty((N * D + offset,), dtype=torch.float32, device="cuda")
    Xd = buf[offset:].view(N, D)
    Xd.copy_(torch.from_numpy(X))
    b = pqt.pqt_builder_create(params, 0)
    cut = N // 3
    pqt.pqt_builder_add(b, Xd[:cut])                                 # the second piece starts at an odd row
    pqt.pqt_builder_add(b, Xd[cut:])
    ix = pqt.pqt_builder_finish(b)
    pqt.pqt_builder_free(b)
    try:
        got = {n: t.cpu().numpy() for n, t in pqt.pqt_index_export(ix, ("offsets", "ids", "codes")).items()}
        offsets, ids = B.inverted_lists(B.bin_slots_batch(X, C1, C2, H), H)
        np.testing.assert_array_equal(got["offsets"], offsets)
        np.testing.assert_array_equal(got["ids"], ids)
        codes = B.encode_pair_lambda(X, C1, M) if fmt else B.encode_batch(X, C1, M, ti, tj, tl)
        np.testing.assert_array_equal(got["codes"], codes[ids])
        assert pqt.pqt_index_info(ix)["bytes_index"] >= 4 * (H + 1) + N * (4 + codes.shape[1])
    finally:
        pqt.pqt_index_free(ix)


def test_pair_lambda_native_builder(pqt, tiny_pair, tmp_path):
    """pqt_builder_* with (pair, lambda) codes: every code names a point that is (within fp32 rounding of
    the level-1 distances it is computed from) as near as the nearest code point, with the level nearest
    to the projection on its line; the index answers queries as the oracle does on it."""
    import torch
    cfg, X, Y, ix = tiny_pair
    params = dict(N=cfg.N, H=ix.H, D=ix.D, P=ix.P, k1=ix.k1, k2=ix.k2, M=ix.M, T=ix.T, C=ix.C,
                  C1=ix.C1, C2=ix.C2, cc=ix.cc, code_format=1)
    b = pqt.pqt_builder_create(params, 0)
    try:
        Xd = torch.from_numpy(X).cuda()
        for lo, hi in ((0, 4097), (4097, cfg.N)):
            pqt.pqt_builder_add(b, Xd[lo:hi].contiguous())
        gix = pqt.pqt_builder_finish(b)
    finally:
        pqt.pqt_builder_free(b)
    path = str(tmp_path / "native_pair.pqt")
    try:
        pqt.pqt_index_save(gix, path)
    finally:
        pqt.pqt_index_free(gix)
    nix = IO.read_index(path)
    assert nix.code_format == 1 and nix.codes.shape == (cfg.N, 2 * cfg.M)
    assert np.array_equal(np.sort(nix.ids), np.arange(cfg.N, dtype=np.uint32))
    ds = nix.D // nix.M
    pairs = Q.centroid_pairs(nix.k1)
    same_pair = total = 0
    kenc = (PU.kappa(ds) + 8.0) * PU.U32
    for t in np.random.default_rng(5).integers(0, cfg.N, size=300):
        x = X[nix.ids[t]].astype(np.float64)
        want = B.encode_pair_lambda(X[nix.ids[t]][None], nix.C1, nix.M)[0]
        xr_got, xr_want = Q.reconstruct(nix, nix.codes[t]), Q.reconstruct(nix, want)
        S = PU.subpart_magnitudes(nix, x)
        for m in range(nix.M):
            cen = B.subpart_centroids(nix.C1, nix.M, m)
            xs = x[m * ds:(m + 1) * ds]
            e_got = float(np.sum((xr_got[m * ds:(m + 1) * ds] - xs) ** 2))
            e_want = float(np.sum((xr_want[m * ds:(m + 1) * ds] - xs) ** 2))
            # as near as the nearest code point, up to the rounding of the two fp32 values of Eq. 9 compared
            mags = []
            for code in (nix.codes[t], want):
                ci, cj = pairs[int(code[2 * m])]
                lm = float(Q.lambda_of_level(code[2 * m + 1]))
                mags.append(abs(1 - lm) * S[m, ci] + abs(lm) * S[m, cj] + abs(lm * lm - lm) * float(nix.cc[m, ci, cj]))
            assert e_got - e_want <= kenc * (mags[0] + mags[1]), (t, m, e_got, e_want)
            i, j = pairs[nix.codes[t, 2 * m]]
            lam, _ = B.line_projection(xs, cen[i], cen[j])
            level = int(nix.codes[t, 2 * m + 1])
            if 0 < level < 255:                                               # the level nearest to the projection
                assert abs(float(Q.lambda_of_level(level)) - lam) <= 0.5 / 16 + 1e-4
            else:
                assert lam < -5.96 or lam > 9.9
            same_pair += int(nix.codes[t, 2 * m] == want[2 * m] and level == want[2 * m + 1])
            total += 1
    assert same_pair >= 0.99 * total
    same, _ = _stagewise(pqt, nix, path, Y[:30], cfg.k, cfg.w, cfg.T, cfg.C)
    assert same >= 27


def test_static_slope_order(pqt, tiny, tmp_path, rng):
    """pqt_set_bin_order(PQT_ORDER_STATIC_SLOPES): the tuples are the pre-computed order of the slope the
    oracle picks from the GPU's own lists (bit for bit), everything downstream as usual; switching back
    restores the default answers; unsupported for hashed or four-part indexes."""
    import torch
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    same, _ = _stagewise(pqt, ix, path, Y[:40], cfg.k, cfg.w, cfg.T, cfg.C, order="static")
    assert same >= 36
    for k, w, T, C in ((5, 1, 1, 7), (10, 2, 37, 50), (cfg.k, cfg.k1, cfg.T, cfg.C)):      # ragged tails, R = all leaves
        _stagewise(pqt, ix, path, Y[:6], k, w, T, C, order="static")
    # every slope occurs: scale the second half of the query so that one list rises faster or slower
    slopes = set()
    for f in (0.05, 0.3, 0.6, 0.8, 0.9, 1.0, 1.1, 1.3, 1.7, 3.0, 20.0):
        y = Y[:4].copy()
        y[:, cfg.D // 2:] *= f
        tr = Q.query(ix, y[0], cfg.k, cfg.w, order_method="static")
        slopes.add(Q.choose_slope(tr.Ld[0].astype(np.float32), tr.Ld[1].astype(np.float32)))
        _stagewise(pqt, ix, path, y, cfg.k, cfg.w, cfg.T, cfg.C, order="static")
    assert len(slopes) >= 6, slopes
    gix = pqt.pqt_index_load(path, 0)
    try:
        yq = torch.from_numpy(Y[:50]).cuda()
        ids0, d0 = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)
        pqt.pqt_set_bin_order(gix, pqt.PQT_ORDER_STATIC_SLOPES)
        ids1, _ = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)
        pqt.pqt_set_bin_order(gix, pqt.PQT_ORDER_SUMMED_DISTANCE)
        ids2, d2 = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)
        torch.cuda.synchronize()
        assert torch.equal(ids0, ids2) and torch.equal(d0, d2)
        assert not torch.equal(ids0, ids1)                        # the two orders visit different bins
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_set_bin_order(gix, 7)
        assert e.value.code == pqt.PQT_EINVAL
    finally:
        pqt.pqt_index_free(gix)
    hashed = B.build_index(X[:3000], cfg.P, cfg.k1, cfg.k2, cfg.M, H=1009, T=cfg.T, C=cfg.C, iters=3)
    hpath = str(tmp_path / "hashed.pqt")
    IO.write_index(hpath, hashed)
    gix = pqt.pqt_index_load(hpath, 0)
    try:
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_set_bin_order(gix, pqt.PQT_ORDER_STATIC_SLOPES)
        assert e.value.code == pqt.PQT_EUNSUPPORTED
    finally:
        pqt.pqt_index_free(gix)


def test_brute_force(pqt, tiny, tmp_path):
    """pqt_brute_force against Eq. 1 written out (the oracle's brute_force): integer data bit for bit
    (fp32 and byte storage, several passes over the database, ragged last pass and tile), real-valued
    data within tolerance with the order replayed on the GPU's own distances."""
    import torch
    ixe, Xe, Ye = _exact_arithmetic_index(N=20000, seed=31)
    path = str(tmp_path / "exact.pqt")
    IO.write_index(path, ixe)
    gix = pqt.pqt_index_load(path, 0)
    try:
        yq = torch.from_numpy(Ye).cuda()
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_brute_force(gix, yq, 10)
        assert e.value.code == pqt.PQT_EINVAL                      # no vectors attached
        for stored in (Xe, Xe.astype(np.uint8)):
            pqt.pqt_index_set_vectors(gix, stored)
            for k in (1, 10, 100):
                ids, d = pqt.pqt_brute_force(gix, yq, k)
                torch.cuda.synchronize()
                ids, d = PU.to_np(ids), PU.to_np(d)
                for q in range(0, Ye.shape[0], 7):
                    o_ids, o_d = Q.brute_force(Ye[q], Xe, k)
                    assert np.array_equal(ids[q], o_ids), f"k={k} query {q}"
                    assert np.array_equal(d[q].astype(np.float64), o_d)
    finally:
        pqt.pqt_index_free(gix)
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    gix = pqt.pqt_index_load(path, 0)
    try:
        pqt.pqt_index_set_vectors(gix, X)
        yq = torch.from_numpy(Y).cuda()
        ids, d = pqt.pqt_brute_force(gix, yq, 20)
        ids1, d1 = pqt.pqt_brute_force(gix, yq[:3].contiguous(), 1)
        torch.cuda.synchronize()
        ids, d = PU.to_np(ids), PU.to_np(d)
        assert np.array_equal(PU.to_np(ids1)[:, 0], ids[:3, 0])
        same = 0
        for q in range(cfg.nq):
            o_ids, o_d = Q.brute_force(Y[q], X, 21)
            y64 = Y[q].astype(np.float64)
            xx = np.sum(X[ids[q]].astype(np.float64) ** 2, axis=1)
            exact = np.sum((X[ids[q]].astype(np.float64) - y64[None]) ** 2, axis=1)
            # ||q||^2 + ||x||^2 - 2 q.x accumulated over all D dimensions
            assert PU.close(d[q], exact, np.dot(y64, y64) + xx, PU.kappa(cfg.D)), f"query {q}"
            assert np.array_equal(np.lexsort((ids[q], d[q])), np.arange(20)), "not sorted by (distance, id)"
            gaps = np.diff(o_d) / np.maximum(o_d[1:], 1e-30)
            if np.all(gaps > 1e-4):                                 # no near-ties among the first 21: ids must agree
                assert np.array_equal(ids[q], o_ids[:20]), f"query {q}"
                same += 1
        assert same >= 0.5 * cfg.nq
    finally:
        pqt.pqt_index_free(gix)


@pytest.mark.parametrize("n, D, P, k1, k2, distinct, offset, iters", [
    (255, 6, 2, 3, 2, 0, 0, 1),            # odd slices (no 16-byte rows), one vector short of a tile
    (257, 8, 1, 33, 5, 0, 0, 1),           # one vector in the last tile; twelve centroids a lane, the last of them padding
    (1000, 72, 2, 8, 40, 0, 0, 1),         # slices of nine 16-byte pieces; cells with fewer than k2 members
    (5000, 64, 2, 16, 8, 0, 1, 1),         # vectors that do not start at a multiple of 16 bytes
    (700, 520, 2, 2, 9, 0, 0, 1),          # a wavefront sums a cell in two pieces
    (300, 8, 2, 20, 4, 6, 0, 3),           # fewer distinct vectors than centroids: cells run empty and are re-seeded
    (300, 200, 1, 20, 4, 6, 0, 3),         # the same with more dimensions than a workgroup re-seeds, a last piece of eight
    (2000, 200, 2, 140, 3, 0, 0, 1),       # more cells than compute units: sums are added up 64 dimensions at a time, a last piece of 36
    (900, 132, 2, 140, 2, 6, 0, 2),        # re-seeded there
    (5, 8, 2, 7, 3, 0, 0, 2),              # fewer vectors than centroids
    (600_001, 8, 2, 2, 2, 0, 0, 1),        # more of the step kernel's tiles than workgroups: a workgroup adds up several
    (1000, 40, 1, 130, 2, 0, 0, 1),        # many centroids, few vectors: wavefronts share a tile; a last round of two centroids
    (777, 6, 2, 256, 3, 0, 0, 1),          # the same with odd slices
    (30_001, 16, 2, 2, 200, 0, 0, 1),      # the same at level 2
])
def test_training_edges(pqt, n, D, P, k1, k2, distinct, offset, iters):
    """Tile, slab and piece edges of the training kernels against the oracle's Lloyd iterations.  Whole numbers up to 255:
    level-1 distances of the first iteration are exact; a centroid is a double-precision mean rounded to fp32 (relative
    2^-24, so 1e-6).  The members of the level-2 runs are those of the GPU's own level-1 centroids; a vector whose two
    nearest are closer than fp32 resolves would be a failure of the draw (none with this seed)."""
    import torch
    rng = np.random.default_rng(11)
    X = rng.integers(0, 256, (n, D)).astype(np.float32)
    if distinct:
        X = X[:distinct][rng.integers(0, distinct, n)]
    buf = torch.empty((n * D + offset,), dtype=torch.float32, device="cuda")
    Xd = buf[offset:].view(n, D)
    Xd.copy_(torch.from_numpy(X))
    got = pqt.pqt_train(Xd, P=P, k1=k1, k2=k2, M=P, iters=iters, n_table=0)
    dp = D // P
    for p in range(P):
        Xp = X[:, p * dp:(p + 1) * dp].astype(np.float64)
        np.testing.assert_allclose(got["C1"][p], B.lloyd(Xp, k1, iters), rtol=1e-6, atol=0)
        lab = np.argmin(B.sqdist_matrix(Xp, got["C1"][p].astype(np.float64)), axis=1)
        for i in range(k1):
            sub = Xp[lab == i]
            want = B.lloyd(sub, k2, iters) if len(sub) else np.repeat(got["C1"][p, i][None], k2, axis=0)
            np.testing.assert_allclose(got["C2"][p, i], want, rtol=1e-6, atol=0)


@pytest.mark.parametrize("n, D, k1, M", [(1, 8, 3, 2), (4097, 8, 5, 2), (1024, 48, 24, 8), (3000, 36, 140, 3),
                                         (16_384, 2, 2, 2), (16_385, 6, 2, 1), (50_001, 4, 3, 2)])
def test_line_table_lambdas(pqt, n, D, k1, M):
    """The lambdas of the line table are those at the (t + 1/2) / alloc quantiles of what was voted on the line, which is not
    sorted for them: one vote, a vote more than whole workgroups, (140 centroids) more lines than are counted on the
    chip, and one line or three that have all votes and code points, as many votes as one workgroup reads and more.  Distances of whole numbers are exact, a lambda is their quotient rounded (2^-23 at most); an error of a line rounds by
    2^-22 of b^2 + lambda^2 c^2.  Vectors nearer to a tie than that (the centroids are vectors themselves, and lie on many lines) may
    or may not have voted on a line: its value of some rank is at least that of all who may and at most that of those who must."""
    import torch
    rng = np.random.default_rng(23)
    X = rng.integers(0, 64, (n, D)).astype(np.float32)
    got = pqt.pqt_train(torch.from_numpy(X).cuda(), P=1, k1=k1, k2=1, M=M, iters=0, n_table=n)
    pairs, ds = np.array(Q.centroid_pairs(k1)), D // M
    for m in range(M):
        cen = B.subpart_centroids(got["C1"], M, m).astype(np.float64)
        d = B.sqdist_matrix(X[:, m * ds:(m + 1) * ds].astype(np.float64), cen)
        b2, a2 = d[:, pairs[:, 0]], d[:, pairs[:, 1]]
        c2 = B.sqdist_matrix(cen, cen)[pairs[:, 0], pairs[:, 1]]
        with np.errstate(divide="ignore", invalid="ignore"):
            lam = (b2 - a2 + c2) / (2.0 * c2)
        usable = c2 > 0
        err = np.where(usable, b2 - lam * lam * c2, np.inf)
        near = err <= err.min(axis=1, keepdims=True) + 2.0 ** -21 * np.where(usable, b2 + lam * lam * c2, 0.0).max(axis=1, keepdims=True)
        near &= usable
        ti, tj, tl = (got[a][m] for a in ("tbl_i", "tbl_j", "tbl_lam"))
        for q, (i, j) in enumerate(pairs):
            mine = tl[(ti == i) & (tj == j)]
            if mine.size == 0:
                continue
            may, must = np.sort(lam[near[:, q], q]), np.sort(lam[near[:, q] & (near.sum(axis=1) == 1), q])
            rank = [np.minimum((2 * np.arange(mine.size) + 1) * v.size // (2 * mine.size), v.size - 1) for v in (must, may)]
            low = may[np.maximum(rank[0], 0)]
            high = np.where(rank[1] < must.size, np.append(must, np.inf)[np.minimum(rank[1], must.size)], may[-1])
            slack = 2.0 ** -22 * (1.0 + np.abs(mine))
            assert np.all(mine >= low - slack) and np.all(mine <= high + slack), (m, i, j)


def test_line_table_in_batches(pqt):
    """More votes than are brought together at a time (2^27), in batches of 13 of 64 sub-parts: the values are exact (one line through 0
    and 8, lambda of x = x / 8), and beside the votes' 8 bytes each the call holds little more than one batch's lambdas."""
    import threading
    import torch
    n, M = 10_000_000, 64
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.empty((n, M), dtype=torch.float32, device="cuda")
    for s in range(0, n, 1 << 21):
        X[s:s + (1 << 21)].random_(0, 64, generator=g)
    X[0], X[n // 2] = 0.0, 8.0
    torch.cuda.synchronize()
    free = [torch.cuda.mem_get_info()[0]] * 2                # before, least
    stop = threading.Event()

    def watch():
        while not stop.wait(0.002):
            free[1] = min(free[1], torch.cuda.mem_get_info(0)[0])
    t = threading.Thread(target=watch)
    t.start()
    try:
        got = pqt.pqt_train(X, P=1, k1=2, k2=1, M=M, iters=0, n_table=n)
    finally:
        stop.set()
        t.join()
    assert 8 * M * n <= free[0] - free[1] <= 8 * M * n + (1 << 30)
    rank = torch.from_numpy((2 * np.arange(256) + 1) * n // 512).cuda()
    for m in (0, 12, 13, 25, 26, 63):
        values = torch.bincount(X[:, m].to(torch.int64), minlength=64).cumsum(0)
        want = torch.searchsorted(values, rank, right=True).to(torch.float32).cpu().numpy() / 8.0
        np.testing.assert_array_equal(got["tbl_lam"][m], want)
        assert np.all(got["tbl_i"][m] == 0) and np.all(got["tbl_j"][m] == 1)


@pytest.mark.parametrize("n, D, P, k1, M, zeros", [(700, 16, 2, 7, 4, 0), (333, 64, 2, 21, 4, 0), (500, 32, 4, 15, 8, 0), (900, 40, 2, 16, 8, 0),
                                                   (300, 32, 2, 33, 4, 0), (130, 80, 2, 70, 2, 0), (700, 24, 1, 130, 8, 0), (600, 16, 2, 256, 4, 0),
                                                   (2500, 24, 1, 140, 2, 0.8), (2500, 24, 1, 9, 2, 0.8)])
def test_line_table_edges(pqt, n, D, P, k1, M, zeros):
    """Line votes where 16-byte rows meet numbers of centroids that are no multiple of four (and at sub-parts of five
    dimensions), and of more than 32 centroids, where wavefronts share a sub-part (sub-parts of 40 and of three dimensions, the
    most centroids), and where most vote for one of few lines and of many.  Without iterations the centroids are training
    vectors, whole numbers, so that all distances are exact.
    Shares as in test_training_on_the_gpu: within one of the quota, and a near tie of two lines may move a vote or two."""
    import torch
    rng = np.random.default_rng(17)
    X = rng.integers(0, 64, (n, D)).astype(np.float32)
    # Most vectors zero, but only the first of the centroids: they lie on its lines, with an error of exactly zero, and vote for the first of
    # them.  (Two zero centroids would make every line through them two lines, of the same error but for rounding.)
    centroids = (np.arange(k1) * n) // k1
    none = rng.random(n) < zeros
    none[centroids] = False
    X[none] = 0.0
    if zeros:
        X[0] = 0.0
    got = pqt.pqt_train(torch.from_numpy(X).cuda(), P=P, k1=k1, k2=2, M=M, iters=0, n_table=n)
    pairs, ds = Q.centroid_pairs(k1), D // M
    for m in range(M):
        line, _, _ = B.best_lines(X[:, m * ds:(m + 1) * ds].astype(np.float64), B.subpart_centroids(got["C1"], M, m))
        quota = np.bincount(line, minlength=len(pairs)) * 256.0 / n
        have = np.zeros(len(pairs))
        for i, j in zip(got["tbl_i"][m].tolist(), got["tbl_j"][m].tolist()):
            have[pairs.index((i, j))] += 1
        assert have.sum() == 256 and np.abs(have - quota).max() <= 1.0 + 256.0 * 3 / n, m


@pytest.mark.parametrize("kind, N, D, nq, k", [
    ("bytes", 255, 16, 1, 255),            # one partial chunk, k close to N
    ("bytes", 4096, 96, 257, 100),         # exactly the first chunk; one query past a workgroup's 256
    ("bytes", 4097, 128, 64, 256),         # one vector in the second chunk, largest k
    ("bytes", 70_001, 160, 129, 33),       # more dimensions than the stationary kernel takes
    ("bytes, real queries", 30_000, 128, 65, 50),     # queries with a second bf16 piece
    ("floats", 4100, 4, 3, 7),             # one step of sixteen dimensions, three quarters padding
    ("floats", 20_011, 20, 128, 128),      # an odd number of steps, the last one partial
    ("floats", 9_000, 200, 130, 10),
    ("ties", 30_000, 128, 9, 50),          # all vectors equal: the lists overflow, the exact scan answers
    ("ties, floats", 5_000, 36, 5, 3),
    ("sorted", 40_000, 128, 40, 100),      # vectors stored in order of their first dimension
    ("huge", 5_000, 32, 4, 5),             # squares overflow: the exact scan answers
])
def test_brute_force_edges(pqt, kind, N, D, nq, k):
    """The filter's tile and chunk edges against distances in float64 (on the GPU by torch).  A distance is a sum
    of D squares in fp32: relative error below (D + 2) 2^-24, no floor; ids are those of an ascending sort of the
    call's own distances, and the k-th distance is the true one to that bound."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(7)
    dev = torch.device("cuda")
    if "floats" in kind or kind == "huge":
        X = torch.rand((N, D), generator=gen, device=dev) * (1e25 if kind == "huge" else 1.0)
        Y = torch.rand((nq, D), generator=gen, device=dev) * (1e25 if kind == "huge" else 1.0)
    else:
        X = torch.randint(0, 256, (N, D), generator=gen, device=dev, dtype=torch.int64).to(torch.uint8)
        Y = torch.randint(0, 256, (nq, D), generator=gen, device=dev, dtype=torch.int64).float()
        if "real" in kind:
            Y = Y + torch.rand((nq, D), generator=gen, device=dev)
    if "ties" in kind:
        X[:] = X[0]
    if kind == "sorted":
        X = X[torch.argsort(X[:, 0].to(torch.int32), stable=True)].contiguous()
    ix = pqt.pqt_index_from_arrays(dict(
        N=N, H=1, D=D, P=1, k1=1, k2=1, M=1, T=1, C=256, C1=np.zeros((1, 1, D)), C2=np.zeros((1, 1, 1, D)),
        tbl_i=np.zeros((1, 256)), tbl_j=np.zeros((1, 256)), tbl_lam=np.zeros((1, 256)), cc=np.zeros((1, 1, 1)),
        offsets=np.array([0, N]), ids=np.arange(N), codes=np.zeros((N, 1))))
    try:
        pqt.pqt_index_set_vectors(ix, X)
        for rep in range(2):                                 # the second call works in the first one's memory
            ids, d = pqt.pqt_brute_force(ix, Y, k)
            torch.cuda.synchronize()
            if kind == "huge":
                assert torch.isinf(d).all() and torch.equal(ids, torch.arange(k, device=dev).expand(nq, k))
                continue
            true = torch.stack([((X.double() - y) ** 2).sum(1) for y in Y.double()])
            bound = (D + 2) * 2.0 ** -24
            own = true.gather(1, ids)
            assert (d.double() - own).abs().le(bound * own).all()
            assert (d.double() - true.sort(1).values[:, :k]).abs().le(2 * bound * own).all()
            order = torch.argsort(ids, dim=1, stable=True)
            order = order.gather(1, torch.argsort(d.gather(1, order), dim=1, stable=True))
            assert torch.equal(order, torch.arange(k, device=dev).expand(nq, k)), "not sorted by (distance, id)"
            assert all(len(set(r)) == k for r in ids.cpu().tolist())
            if "bytes" == kind or "ties" == kind or "sorted" == kind:      # whole numbers: exact
                key = true * N + torch.arange(N, device=dev)               # (distance, id), exact in float64
                assert torch.equal(ids, key.sort(1).indices[:, :k])
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("N, D, nq, k, other", [
    (127, 128, 512, 20, ()),                         # less than a tile of 128 vectors, exactly one group of 512 queries
    (4096 + 129, 96, 513, 100, ()),                  # one vector past a tile of the second chunk; one query past a group
    (9001, 112, 640, 10, (600,)),                    # padded dimensions; the first group of bytes, the second not
    (9001, 48, 1024, 10, (255, 1023)),               # the first half of either group, the second half
    (30_000, 128, 130, 250, (3,)),                   # one wavefront's 128 queries and two more, not of bytes
])
@pytest.mark.parametrize("value", [-1.0, 256.0, 127.5, 1e-3])
def test_brute_force_bytes_and_others(pqt, N, D, nq, k, other, value):
    """Byte vectors searched by groups of 512 queries of bytes, and by groups in which one value is not a byte (negative, too
    large, halves with one bf16 piece, with two).  Extreme bytes too: 0 and 255 less 128 are both ends of a signed byte.
    Whole numbers and halves are exact in fp32: ids and distances are those of float64; 1e-3 leaves (D + 2) 2^-24."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(11)
    X = torch.randint(0, 256, (N, D), generator=gen, device="cuda")
    X[::7] = torch.where(X[::7] < 128, 0, 255)
    Y = torch.randint(0, 256, (nq, D), generator=gen, device="cuda").float()
    Y[::3] = torch.where(Y[::3] < 128, 0.0, 255.0)
    for q in other:
        Y[q, q % D] = value
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X.to(torch.uint8))
        ids, d = pqt.pqt_brute_force(ix, Y, k)
        x, y = X.double(), Y.double()
        true = (x * x).sum(1)[None] - 2 * (y @ x.T) + (y * y).sum(1)[:, None]      # below 2^53 / 4: exact but for 1e-3
        exact = torch.ones(nq, dtype=torch.bool, device="cuda")
        exact[list(other)] = value != 1e-3
        want = (true * N + torch.arange(N, device="cuda")).sort(1).indices[:, :k]
        assert torch.equal(ids[exact], want[exact]) and torch.equal(d[exact].double(), true.gather(1, want)[exact])
        rest = true[~exact].gather(1, ids[~exact])
        bound = (D + 2) * 2.0 ** -24
        assert (d[~exact].double() - rest).abs().le(bound * rest).all()
        assert (rest - true[~exact].sort(1).values[:, :k]).abs().le(2 * bound * rest).all()
    finally:
        pqt.pqt_index_free(ix)


def _vectors_only_index(pqt, N, D):
    """An index that holds no more than a collection to search exactly: one bin."""
    return pqt.pqt_index_from_arrays(dict(
        N=N, H=1, D=D, P=1, k1=1, k2=1, M=1, T=1, C=256, C1=np.zeros((1, 1, D)), C2=np.zeros((1, 1, 1, D)),
        tbl_i=np.zeros((1, 256)), tbl_j=np.zeros((1, 256)), tbl_lam=np.zeros((1, 256)), cc=np.zeros((1, 1, 1)),
        offsets=np.array([0, N]), ids=np.arange(N), codes=np.zeros((N, 1))))


@pytest.mark.parametrize("D", [16, 128, 192])
def test_brute_force_keeps_what_the_cut_moves_most(pqt, D):
    """The filter's values of two vectors may be off in opposite directions by all that cutting numbers into pieces can
    cost.  The nearest vector's value is too large, the second nearest's too small, and the nearest comes last in the
    database order (place i is vector i * step mod N), when the list of the best holds the other one only."""
    import math
    import torch
    N = 300_001                                                      # three chunks with one query and one result
    near, second, q = np.float32(1.00388336), np.float32(1.00392914), np.float32(1.00389862)
    assert abs(near - q) < abs(second - q)
    step = int(N * 0.6180339887498949) | 1
    while math.gcd(step, N) != 1:
        step += 2
    last = (N - 1) * step % N
    X = torch.full((N, D), 0.5, device="cuda")                       # (short: the bound grows with the norms)
    X[::2] = -0.5                                                    # (no common centre)
    X[0] = float(second)
    X[last] = float(near)
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X)
        ids, _ = pqt.pqt_brute_force(ix, torch.full((1, D), float(q), device="cuda"), 1)
        assert ids.item() == last
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -66, 2.0 ** -70])
@pytest.mark.parametrize("D", [32, 128])
def test_brute_force_tiny_values(pqt, D, scale):
    """Squares and products near and below the smallest normal fp32 number (2^-126), where the matrix cores need not keep
    what fp32 does: whole numbers times a power of two, so that every exact distance is a multiple of the smallest fp32
    number and results are those of the whole numbers."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(9)
    N, nq, k = 9000, 5, 20
    X = torch.randint(0, 256, (N, D), generator=gen, device="cuda").float()
    Y = torch.randint(0, 256, (nq, D), generator=gen, device="cuda").float()
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X * scale)
        ids, d = pqt.pqt_brute_force(ix, Y * scale, k)
        true = torch.stack([((X.double() - y) ** 2).sum(1) for y in Y.double()])
        assert torch.equal(ids, (true * N + torch.arange(N, device="cuda")).sort(1).indices[:, :k])
        assert torch.equal(d.double(), true.gather(1, ids) * scale ** 2)
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("kind", ["one long vector", "long vectors", "an offset", "a long query", "norms of all sizes"])
def test_brute_force_whatever_the_norms(pqt, kind):
    """Norms that differ and coordinates far from zero: the results are right, and they take about as long as on even data
    (left to the exact scan, which would be right as well, they take more than ten times as long; a factor of four leaves
    room for a busy machine)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(21)
    N, D, nq, k = 60_000, 256, 512, 10
    X = torch.rand((N, D), generator=gen, device="cuda") - 0.5
    Y = torch.rand((nq, D), generator=gen, device="cuda") - 0.5

    def timed(X, Y):
        ix = _vectors_only_index(pqt, N, D)
        try:
            pqt.pqt_index_set_vectors(ix, X)
            times = []
            for _ in range(4):
                begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                begin.record()
                ids, d = pqt.pqt_brute_force(ix, Y, k)
                end.record()
                end.synchronize()
                times.append(begin.elapsed_time(end))
            return min(times[1:]), ids, d
        finally:
            pqt.pqt_index_free(ix)
    even = timed(X, Y)[0]
    if kind == "one long vector":
        X[777] *= 300
    elif kind == "long vectors":
        X[::500] *= 50
    elif kind == "an offset":
        X, Y = X + 15, Y + 15
    elif kind == "a long query":
        Y = Y * 100
    else:
        X = X * torch.exp(torch.randn((N, 1), generator=gen, device="cuda"))
    t, ids, d = timed(X, Y)
    true = torch.cat([((X.double()[None] - y[:, None]) ** 2).sum(2) for y in Y[:40].double().split(4)])
    bound = (D + 2) * 2.0 ** -24
    own = true.gather(1, ids[:40])
    assert (d[:40].double() - own).abs().le(bound * own).all()
    assert (own - true.sort(1).values[:, :k]).abs().le(2 * bound * own).all()
    assert t < 4 * even, (t, even)


@pytest.mark.parametrize("stored, N, D, nq, k, same", [
    ("f32", 60_000, 64, 300, 10, 1000),    # more ties than results, kept to the end
    ("u8", 60_000, 128, 300, 100, 2000),
    ("u8", 60_000, 96, 300, 256, 20_000),  # more than are kept: the exact scan, a part of the database a workgroup
    ("f32", 60_000, 20, 1, 7, 60_000),     # one query, all tied
    ("f32", 700, 2048, 3, 200, 700),       # rows of which the scan holds one query at a time
    ("f32", 700, 2044, 3, 200, 700),       # four such rows and their entries would fill 64 KB of LDS to the byte
    ("f32", 700, 1980, 3, 200, 700),       # the longest of which it holds four
    ("u8", 4500, 16, 5000, 3, 4500),       # more queries than the scan has workgroups
])
def test_brute_force_ties(pqt, stored, N, D, nq, k, same):
    """Groups of equal vectors spread over the database: the smallest ids win, and queries near such a group take at most ten
    times as long as others (measured: 1.5 to 3.6 times; scanned by one workgroup per query 12 to 30 times)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(31)
    # distances are whole numbers in fp32 below 2^24 = 16.8e6: numbers below t lie (t^2 - 1) / 6 apart in the mean square,
    # 1.4e6 for t = 256 and D = 128, 22e6 for D = 2,044, where t = 128 gives 5.6e6
    top = 256 if D <= 128 else 128
    X = torch.randint(0, top, (N, D), generator=gen, device="cuda").float()
    Y = torch.randint(0, top, (nq, D), generator=gen, device="cuda").float()

    def timed(X, Y):
        ix = _vectors_only_index(pqt, N, D)
        try:
            pqt.pqt_index_set_vectors(ix, X.to(torch.uint8) if stored == "u8" else X)
            times = []
            for _ in range(4):
                begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                begin.record()
                ids, d = pqt.pqt_brute_force(ix, Y, k)
                end.record()
                end.synchronize()
                times.append(begin.elapsed_time(end))
            return min(times[1:]), ids, d
        finally:
            pqt.pqt_index_free(ix)
    even = timed(X, Y)[0]
    group = torch.randperm(N, generator=gen, device="cuda")[:same]
    X[group] = X[group[0]].clone()
    Y[::2] = X[group[0]] + (torch.rand((len(Y[::2]), D), generator=gen, device="cuda") < 0.1).float()
    t, ids, d = timed(X, Y)
    for q in range(0, nq, max(1, nq // 50)):
        true = ((X.double() - Y[q].double()) ** 2).sum(1)             # whole numbers: exact in any order
        want = (true * N + torch.arange(N, device="cuda")).sort().indices[:k]
        assert torch.equal(ids[q], want) and torch.equal(d[q].double(), true[want]), q
    print(f"{t:.3f} ms, without ties {even:.3f} ms", flush=True)
    if nq < 1000:
        assert t < 10 * even, (t, even)


@pytest.mark.parametrize("stored, N, D, early, k", [
    ("u8", 60_000, 128, 60, 100),          # too many of the k nearest come first, the others are not kept: scanned
    ("u8", 60_000, 128, 100, 100),         # all of them come first
    ("f32", 60_000, 20, 60, 100),
    ("f32", 300_000, 16, 0, 256),          # none comes before the last chunk
])
def test_brute_force_misleading_order(pqt, stored, N, D, early, k):
    """Neighbours that are not spread over the database order (place i is vector i * step mod N), so that what the first
    vectors let expect of the rest is wrong; other queries of the same call are not affected.  Whole numbers: exact."""
    import math
    import torch
    gen = torch.Generator(device="cuda").manual_seed(51)
    step = int(N * 0.6180339887498949) | 1
    while math.gcd(step, N) != 1:
        step += 2
    X = torch.randint(0, 256, (N, D), generator=gen, device="cuda").float()
    Y = torch.randint(0, 256, (40, D), generator=gen, device="cuda").float()
    places = torch.cat([torch.arange(early), torch.arange(N - (k - early), N)])
    near = Y[7].expand(k, D).clone()
    near[torch.arange(k), torch.arange(k) % D] = (near[torch.arange(k), torch.arange(k) % D] + 1 + torch.arange(k, device="cuda") // D) % 256
    X[(places * step % N).cuda()] = near
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X.to(torch.uint8) if stored == "u8" else X)
        ids, d = pqt.pqt_brute_force(ix, Y, k)
        for q in range(len(Y)):
            true = ((X.double() - Y[q].double()) ** 2).sum(1)
            want = (true * N + torch.arange(N, device="cuda")).sort().indices[:k]
            assert torch.equal(ids[q], want) and torch.equal(d[q].double(), true[want]), q
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("N, D, nq, kind", [
    (70_001, 336, 300, "even"),              # products of halves: an odd number of steps of sixteen dimensions, 256 queries and some
    (40_000, 500, 513, "even"),              # a partial last step; one query past two groups
    (70_001, 336, 300, "a crowd"),           # one query with thousands of vectors in the halves' window: its group keeps to bf16
    (70_001, 336, 300, "an offset"),         # vectors relative to their centre
    (70_001, 336, 300, "small and large"),   # numbers that are zero as scaled halves; a query and vectors far longer than others
    (70_001, 336, 300, "out of range"),      # norms that are not scaled to halves
    (70_001, 336, 300, "half an offset"),    # norms and queries relative to the centre, vectors as they are
    (40_000, 3072, 140, "even"),             # so long that three products of pieces may be off by more than one of halves
    (33_000, 8192, 140, "half an offset"),   # the longest
])
def test_brute_force_halves(pqt, N, D, nq, kind):
    """Float collections large enough to be filtered by products of halves, against distances in float64: a distance is a sum of D
    squares in fp32, relative error below (D + 2) 2^-24, and the k-th distance is the true one to that bound."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(61)
    k = 20
    X = torch.rand((N, D), generator=gen, device="cuda") - 0.5
    Y = torch.rand((nq, D), generator=gen, device="cuda") - 0.5
    if kind == "a crowd":
        X[::7] = Y[5] * (1 + 1e-4 * torch.rand((len(X[::7]), 1), generator=gen, device="cuda")) + 1e-4 * X[::7]
    elif kind == "an offset":
        X, Y = X + 20, Y + 20
    elif kind == "half an offset":
        X, Y = X + 0.5, Y + 0.5
    elif kind == "small and large":
        X[::3] *= 1e-7
        X[::1000] *= 1e4
        Y[7] *= 1e5
        Y[11] *= 1e-6
    elif kind == "out of range":
        X, Y = X * 1e-14, Y * 1e-14
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X)
        for _ in range(2):
            ids, d = pqt.pqt_brute_force(ix, Y, k)
        x = X.double()
        bound = (D + 2) * 2.0 ** -24
        for q in list(range(0, nq, 9)) + [5, 7, 11, nq - 1]:
            true = ((x - Y[q].double()) ** 2).sum(1)
            own = true[ids[q]]
            assert len(set(ids[q].tolist())) == k
            assert (d[q].double() - own).abs().le(bound * own).all(), q
            assert (d[q].double() - true.sort().values[:k]).abs().le(2 * bound * own).all(), q
    finally:
        pqt.pqt_index_free(ix)


def test_brute_force_halves_with_a_crowded_query(pqt):
    """One query of many with thousands of vectors in the halves' window costs little more than its own exact scan: 1.4 times the
    call without it (2.2 with its group kept to bf16 pieces and the others to halves).  Results are right for it and the others."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(62)
    N, D, nq, k = 100_000, 128, 3000, 20
    X = torch.rand((N, D), generator=gen, device="cuda") - 0.5
    Y = torch.rand((nq, D), generator=gen, device="cuda") - 0.5

    def timed(X, Y):
        ix = _vectors_only_index(pqt, N, D)
        try:
            pqt.pqt_index_set_vectors(ix, X)
            times = []
            for _ in range(6):
                begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                begin.record()
                ids, d = pqt.pqt_brute_force(ix, Y, k)
                end.record()
                end.synchronize()
                times.append(begin.elapsed_time(end))
            return min(times[1:]), ids, d
        finally:
            pqt.pqt_index_free(ix)
    even = timed(X, Y)[0]
    X[::7] = Y[5] * (1 + 1e-4 * torch.rand((len(X[::7]), 1), generator=gen, device="cuda")) + 1e-4 * X[::7]
    t, ids, d = timed(X, Y)
    print(f"{t:.3f} ms, without {even:.3f} ms", flush=True)
    bound = (D + 2) * 2.0 ** -24
    for q in (0, 4, 5, 6, 255, 256, nq - 1):
        true = ((X.double() - Y[q].double()) ** 2).sum(1)
        own = true[ids[q]]
        assert len(set(ids[q].tolist())) == k
        assert (d[q].double() - own).abs().le(bound * own).all(), q
        assert (d[q].double() - true.sort().values[:k]).abs().le(2 * bound * own).all(), q
    assert t < 1.8 * even, (t, even)


@pytest.mark.parametrize("stored, D", [("u8", 32), ("f32", 20)])
def test_brute_force_in_rounds(pqt, stored, D):
    """More queries than one round of the workspace holds (16,384): the queries on both sides of the border and the last ones
    get what they get by themselves, and what float64 says; a query of the second round that all vectors tie for is scanned."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(41)
    N, nq, k = 6000, 16_384 + 37, 5
    X = torch.randint(0, 256, (N, D), generator=gen, device="cuda").float()
    X[1000:] = torch.where(torch.rand((N - 1000, 1), generator=gen, device="cuda") < 0.7, X[7], X[1000:])
    Y = torch.randint(0, 256, (nq, D), generator=gen, device="cuda").float()
    Y[-3] = X[7]
    ix = _vectors_only_index(pqt, N, D)
    try:
        pqt.pqt_index_set_vectors(ix, X.to(torch.uint8) if stored == "u8" else X)
        ids, d = pqt.pqt_brute_force(ix, Y, k)
        for part in (slice(0, 9), slice(16_380, 16_390), slice(nq - 9, nq)):
            few, fd = pqt.pqt_brute_force(ix, Y[part].contiguous(), k)
            true = ((X.double()[None] - Y[part].double()[:, None]) ** 2).sum(2)
            want = (true * N + torch.arange(N, device="cuda")).sort(1).indices[:, :k]
            assert torch.equal(few, want) and torch.equal(ids[part], want)
            assert torch.equal(fd, d[part]) and torch.equal(fd.double(), true.gather(1, want))
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("D, P, k1, k2, M, w, H, T, C, k, codes", [
    (32, 2, 16, 8, 8, 8, 0, 1024, 4096, 100, "table"),       # lists of 64, M = 8
    (64, 2, 17, 13, 4, 5, 0, 300, 700, 10, "table"),         # a second tile of one centroid; lists of 65
    (64, 1, 48, 8, 32, 32, 0, 256, 3000, 50, "table"),       # one part, lists of 256 (four a lane), more jobs than wavefronts
    (96, 1, 16, 7, 12, 5, 0, 35, 3000, 50, "table"),         # one part, a list of odd length
    (96, 4, 16, 7, 12, 4, 5003, 1024, 2000, 37, "table"),    # four parts, hashed
    (64, 4, 8, 8, 16, 8, 0, 4096, 16384, 1024, "table"),     # most tuples a workgroup holds, the largest budget and list
    (48, 2, 20, 7, 12, 5, 999, 500, 3001, 37, "pair"),       # pair codes of six words, hashed
    (40, 2, 5, 3, 10, 2, 0, 36, 100, 100, "pair"),           # read byte by byte; fewer tuples than 64; fewer candidates than results
    (96, 2, 16, 16, 6, 16, 0, 128, 5000, 9, "table"),        # read byte by byte
    (512, 2, 64, 4, 8, 4, 0, 256, 1000, 20, "table"),        # large codebooks: one launch up to 256 queries
    (64, 2, 16, 17, 4, 16, 0, 200, 900, 9, "table"),         # lists of 272: three launches
    (36, 2, 9, 4, 2, 4, 0, 64, 500, 9, "table"),             # part dimensions of 18: three launches
])
def test_small_batches(pqt, D, P, k1, k2, M, w, H, T, C, k, codes):
    """Batches of up to 1,024 queries (answered in one launch by workgroups of three sizes, unless said otherwise) against the launches with
    intermediate results and a larger batch: the same ids and distance bits, with budgets that 32 tuples fill, that 64 do, and that
    take the full ranking."""
    import torch
    rng = np.random.default_rng(23)
    N, bins = 20_000, (k1 * k2) ** P
    H = H or min(bins, 1 << 24)
    X = rng.integers(0, 64, (N, D)).astype(np.float32)
    dp, pairs = D // P, k1 * (k1 - 1) // 2
    counts = rng.multinomial(N, rng.dirichlet(np.full(H, 0.3))) if H <= 70_000 else np.bincount(rng.integers(0, H, N), minlength=H)
    offsets = np.concatenate([[0], np.cumsum(counts)])
    C1 = X[rng.permutation(N)[:P * k1]].reshape(P, k1, D)[:, :, :dp]
    C2 = C1[:, :, None] + rng.integers(-8, 9, (P, k1, k2, dp))
    cc = rng.integers(1, 500, (M, k1, k1)).astype(np.float32)
    cc = np.triu(cc, 1) + np.triu(cc, 1).transpose(0, 2, 1)
    code = rng.integers(0, 256, (N, M, 2))
    code[:, :, 0] %= pairs
    ix = pqt.pqt_index_from_arrays(dict(
        N=N, H=H, D=D, P=P, k1=k1, k2=k2, M=M, T=T, C=C, C1=C1, C2=C2, tbl_i=rng.integers(0, k1, (M, 256)),
        tbl_j=rng.integers(0, k1, (M, 256)), tbl_lam=rng.normal(0.5, 0.5, (M, 256)), cc=cc, offsets=offsets, ids=rng.permutation(N),
        codes=code if codes == "pair" else code[:, :, 1], code_format=int(codes == "pair")))
    try:
        Y = torch.from_numpy(X[:1100] + rng.normal(0, 2, (1100, D)).astype(np.float32)).cuda()
        for c in sorted({k, C, max(k, C // 20)}):
            pqt.pqt_set_budget(ix, T, c)
            ids, d = pqt.pqt_query_batch(ix, Y, k, w)                        # three launches
            for nq in (1, 3, 40, 256, 257, 512, 513, 1024):
                few, fd = pqt.pqt_query_batch(ix, Y[:nq].contiguous(), k, w)
                assert torch.equal(few, ids[:nq]) and torch.equal(fd, d[:nq]), (c, nq)
            staged, sd, _ = pqt.pqt_query_batch_debug(ix, Y[:40].contiguous(), k, w, taps=("n_cand",))
            assert torch.equal(staged, ids[:40]) and torch.equal(sd, d[:40])
            if P == 2 and H == bins:                                         # the fixed order
                pqt.pqt_set_bin_order(ix, pqt.PQT_ORDER_STATIC_SLOPES)
                ids, d = pqt.pqt_query_batch(ix, Y, k, w)
                for nq in (1, 256, 257, 513):
                    few, fd = pqt.pqt_query_batch(ix, Y[:nq].contiguous(), k, w)
                    assert torch.equal(few, ids[:nq]) and torch.equal(fd, d[:nq]), (c, nq)
                pqt.pqt_set_bin_order(ix, pqt.PQT_ORDER_SUMMED_DISTANCE)
    finally:
        pqt.pqt_index_free(ix)


@pytest.mark.parametrize("k_short, k, C, same", [
    (257, 10, 2000, 0),                    # one more than the workgroup's threads
    (1000, 1000, 4096, 0),                 # all of the short list is wanted
    (1000, 100, 1100, 0),                  # queries with fewer candidates than that
    (600, 50, 4096, 3000),                 # equal codes: bins too full to place by
])
def test_exact_rerank_of_long_lists(pqt, k_short, k, C, same):
    """Short lists longer than the workgroup come without order: exact re-ranking gets the same vectors as from the ordered list
    of pqt_query_batch, whose exact distances (whole numbers) are taken here."""
    import torch
    rng = np.random.default_rng(29)
    N, D, P, k1, k2, M, H, T, w, nq = 30_000, 32, 2, 16, 8, 8, 2048, 512, 4, 1100
    X = rng.integers(0, 64, (N, D))
    offsets = np.concatenate([[0], np.cumsum(rng.multinomial(N, rng.dirichlet(np.full(H, 0.3))))])
    C1 = X[rng.permutation(N)[:P * k1]].reshape(P, k1, D)[:, :, :D // P]
    code = rng.integers(0, 256, (N, M))
    code[rng.permutation(N)[:same * 9]] = code[0]
    ix = pqt.pqt_index_from_arrays(dict(
        N=N, H=H, D=D, P=P, k1=k1, k2=k2, M=M, T=T, C=C, C1=C1, C2=C1[:, :, None] + rng.integers(-8, 9, (P, k1, k2, D // P)),
        tbl_i=rng.integers(0, k1, (M, 256)), tbl_j=rng.integers(0, k1, (M, 256)), tbl_lam=rng.normal(0.5, 0.5, (M, 256)),
        cc=rng.integers(1, 500, (M, k1, k1)), offsets=offsets, ids=rng.permutation(N), codes=code))
    try:
        x = torch.from_numpy(X.astype(np.uint8)).cuda()
        pqt.pqt_index_set_vectors(ix, x)
        Y = torch.from_numpy(rng.integers(0, 64, (nq, D)).astype(np.float32)).cuda()
        short, _ = pqt.pqt_query_batch(ix, Y, k_short, w)
        true = ((x[short.clamp(min=0)].double() - Y.double()[:, None]) ** 2).sum(2)
        key = torch.where(short >= 0, true * N + short, torch.inf).sort(1).values[:, :k]
        want = torch.where(key.isinf(), -1.0, torch.remainder(key, N)).long()
        for n in (nq, 600, 300, 7):                                  # three launches; one, in workgroups of 256, 512 and 1,024 threads
            ids, d = pqt.pqt_query_batch_exact(ix, Y[:n].contiguous(), k_short, k, w)
            assert torch.equal(ids, want[:n]), n
            assert torch.equal(d.double(), torch.where(key.isinf(), torch.inf, torch.div(key, N, rounding_mode="floor"))[:n]), n
    finally:
        pqt.pqt_index_free(ix)


def test_four_part_index(pqt, tmp_path):
    """P = 4: parts (1,2) and (3,4) are ranked first, then pairs of positions in those two lists."""
    from workloads import tiny_mixture
    X = tiny_mixture(4000, d=32, seed=3)
    Y = tiny_mixture(24, d=32, seed=4)
    ix4 = B.build_index(X, P=4, k1=4, k2=4, M=8, T=512, C=1024, iters=5)
    path = str(tmp_path / "p4.pqt")
    IO.write_index(path, ix4)
    # (k, w, T, C): R = 8 -> pair lists of 64, final region larger than the sort buffer;
    # R = 16 -> pair lists cut at T; R = 4 -> every combination, T not a power of two; a long T
    for (k, w, T, C) in ((10, 2, 256, 1024), (10, 4, 512, 600), (5, 1, 100, 200), (10, 3, 4096, 4000)):
        _stagewise(pqt, ix4, path, Y, k, w, T, C)
    # hashed slots: bins collide, a slot is proposed once
    ixh = B.build_index(X, P=4, k1=4, k2=4, M=8, H=997, T=512, C=1024, codebooks=(ix4.C1, ix4.C2),
                        line_table=(ix4.tbl_i, ix4.tbl_j, ix4.tbl_lam))
    path = str(tmp_path / "p4h.pqt")
    IO.write_index(path, ixh)
    _stagewise(pqt, ixh, path, Y[:12], 10, 2, 300, 1024)
    # more tuples than the table for repeated slots holds: they are found by sorting (slot, tuple) keys
    _stagewise(pqt, ixh, path, Y[:6], 10, 3, 2500, 4000)


def test_four_part_long_lists(pqt, tmp_path):
    """P = 4 with lists of 128 and 64 children and T = 1024: the pair lists are cut at T, the last ranking's
    region has rows of 1024 entries beside rows of 16, so the kernel that deals out units of a row (not rows)
    to its wavefronts runs, and the keys are placed by histogram bin; hashed and unhashed bins."""
    from workloads import tiny_mixture
    X = tiny_mixture(20000, d=32, seed=5)
    Y = tiny_mixture(12, d=32, seed=6)
    ixh = B.build_index(X, P=4, k1=16, k2=16, M=8, H=65537, T=1024, C=3000, iters=4)
    path = str(tmp_path / "p4_long_hashed.pqt")
    IO.write_index(path, ixh)
    # (the oracle with its pair lists cut at T, which its pin test shows to be the same order: the uncut
    # form sorts R^4 tuples)
    _stagewise(pqt, ixh, path, Y, 10, 8, 1024, 3000, truncate_pairs=True)         # R = 128
    _stagewise(pqt, ixh, path, Y[:6], 10, 4, 700, 1500, truncate_pairs=True)      # R = 64, T not a power of two
    ix = B.build_index(X, P=4, k1=8, k2=8, M=8, T=1024, C=3000, iters=4)
    path = str(tmp_path / "p4_long.pqt")
    IO.write_index(path, ix)
    _stagewise(pqt, ix, path, Y, 10, 8, 1024, 3000, truncate_pairs=True)          # R = 64, 2^24 bins, unhashed


def test_four_part_exact_arithmetic_heavily_tied(pqt, tmp_path):
    """P = 4 on the exact-arithmetic index: integer sums tie by the hundreds in the pair lists and in the
    final ranking, so every tie cut by (position, position) is exercised; results must be bit-exact."""
    ix, X, Y = _exact_arithmetic_index(N=6000, seed=21, k1=8, k2=2, P=4)
    path = str(tmp_path / "exact_p4.pqt")
    IO.write_index(path, ix)
    for (k, w, T, C) in ((10, 8, 600, 2000), (10, 4, 256, 512), (20, 8, 2048, 4096), (10, 2, 30, 300)):
        same, _ = _stagewise(pqt, ix, path, Y[:16], k, w, T, C, exact=True)
        assert same == 16


def test_error_codes(pqt, tiny, tmp_path):
    import torch
    cfg, X, Y, ix = tiny
    path = str(tmp_path / "tiny.pqt")
    IO.write_index(path, ix)
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_index_load(str(tmp_path / "missing.pqt"), 0)
    assert e.value.code == pqt.PQT_EIO
    bad = str(tmp_path / "bad.pqt")
    with open(path, "rb") as f:
        blob = f.read()
    with open(bad, "wb") as f:
        f.write(b"NOTANIDX" + blob[8:])
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_index_load(bad, 0)
    assert e.value.code == pqt.PQT_EFORMAT
    with open(bad, "wb") as f:
        f.write(blob[:-100])
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_index_load(bad, 0)
    assert e.value.code == pqt.PQT_EFORMAT
    broken = IO.read_index(path)
    broken.offsets = broken.offsets.copy()
    broken.offsets[5] = broken.offsets[-1] + 7          # not monotone
    IO.write_index(bad, broken)
    with pytest.raises(pqt.PqtError) as e:
        pqt.pqt_index_load(bad, 0)
    assert e.value.code == pqt.PQT_EFORMAT

    gix = pqt.pqt_index_load(path, 0)
    try:
        yq = torch.from_numpy(Y).cuda()
        for k, w in ((0, 2), (cfg.C + 1, 2), (10, 0), (10, cfg.k1 + 1)):
            with pytest.raises(pqt.PqtError) as e:
                pqt.pqt_query_batch(gix, yq, k, w)
            assert e.value.code == pqt.PQT_EINVAL
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_set_budget(gix, 0, 10)
        assert e.value.code == pqt.PQT_EINVAL
        with pytest.raises(pqt.PqtError) as e:
            pqt.pqt_set_budget(gix, 10, 1 << 20)
        assert e.value.code == pqt.PQT_EINVAL
        ids, d = pqt.pqt_query_batch(gix, yq, cfg.k, cfg.w)     # still usable after errors
        torch.cuda.synchronize()
        assert ids.shape == (cfg.nq, cfg.k)
    finally:
        pqt.pqt_index_free(gix)


# ---- full size, in the launch configuration bench.py times -------------------------------------------
@pytest.fixture(scope="module")
def sift_full(pqt, tmp_path_factory):
    """SIFT-shaped 1M x 128 database, 10,000 queries, index trained and built by the library
    (pqt_train, pqt_builder_*; the index is input data for both sides; its validity is checked below)."""
    import torch
    from workloads import CONFIGS, sift_like_tables, sift_like_torch
    from paper_1702_05911_amd import builder
    cfg = CONFIGS["sift"]
    tables = sift_like_tables(cfg.D)
    dev = torch.device("cuda", 0)
    X = sift_like_torch(0, cfg.N, d=cfg.D, seed=cfg.data_seed, tables=tables, device=dev)
    Y = sift_like_torch(0, cfg.nq, d=cfg.D, seed=cfg.query_seed, tables=tables, device=dev)
    path = str(tmp_path_factory.mktemp("sift") / "sift.pqt")
    builder.build_index(path, X, P=cfg.P, k1=cfg.k1, k2=cfg.k2, M=cfg.M, H=cfg.H, T=cfg.T, C=cfg.C,
                        train_n=cfg.train_n, device=0, chunk_rows=1 << 18).close()
    return cfg, X.cpu().numpy(), Y.cpu().numpy(), path, IO.read_index(path)


def test_sift_full_size_index_is_valid(sift_full):
    cfg, X, Y, path, ix = sift_full
    off = ix.offsets.astype(np.int64)
    assert off[0] == 0 and off[-1] == cfg.N and np.all(np.diff(off) >= 0)
    assert np.array_equal(np.sort(ix.ids), np.arange(cfg.N, dtype=np.uint32))
    rng = np.random.default_rng(0)
    mism = 0
    for t in rng.integers(0, cfg.N, size=200):
        slot = int(np.searchsorted(off, t, side="right")) - 1
        x = X[ix.ids[t]]
        mism += slot != B.bin_slot(x, ix.C1, ix.C2, ix.H)
        mism += not np.array_equal(ix.codes[t], B.encode_vector(x, ix.C1, ix.M, ix.tbl_i, ix.tbl_j, ix.tbl_lam))
        if t > 0 and np.searchsorted(off, t - 1, side="right") - 1 == slot:
            assert ix.ids[t - 1] < ix.ids[t]
    assert mism <= 4          # the fp32 builder may settle a near-tie differently from float64


def _full_size_check(pqt, gix, ix, cfg, Y, w, order="fullsort", label="sift"):
    """Properties on every query of the batch bench.py times, and the oracle stage by stage on a sample."""
    ids, dists, taps = _run_debug(pqt, gix, Y, cfg.k, w)
    nc = taps["n_cand"].astype(np.int64)
    assert np.all(nc <= cfg.C) and np.all(nc > 0)
    for q in range(cfg.nq):
        n = int(nc[q])
        sc, cid = taps["scores"][q][:n], taps["cand_ids"][q][:n]
        o = np.lexsort((cid, sc))[:cfg.k]
        assert np.array_equal(ids[q][:len(o)], cid[o]), f"query {q}: top-k is not the k smallest (score, id)"
        assert np.array_equal(dists[q][:len(o)], sc[o])
        assert len(set(cid.tolist())) == n
    same = decided = 0
    sample = list(range(0, cfg.nq, 417))
    for q in sample:
        print(f"{label} w={w} query {q}", flush=True)
        tr = PU.check_query_stages(ix, Y[q], taps, q, cfg.k, w, cfg.T, cfg.C, ids, dists, order=order)
        s, d = PU.end_to_end_agreement(tr, ids[q], dists[q])
        assert s or not d, f"query {q}: margins above threshold but ids differ"
        same += s
        decided += d
    print(f"{label} w={w}: {same}/{len(sample)} sampled queries identical to the float64 oracle, {decided} decided")
    assert same >= 0.8 * len(sample)


@pytest.mark.parametrize("w", [8, 1])
def test_sift_full_size_parity(pqt, sift_full, w):
    cfg, X, Y, path, ix = sift_full
    gix = pqt.pqt_index_load(path, 0)
    try:
        _full_size_check(pqt, gix, ix, cfg, Y, w)
    finally:
        pqt.pqt_index_free(gix)


def test_sift_full_size_static_order(pqt, sift_full):
    cfg, X, Y, path, ix = sift_full
    gix = pqt.pqt_index_load(path, 0)
    try:
        pqt.pqt_set_bin_order(gix, pqt.PQT_ORDER_STATIC_SLOPES)
        _full_size_check(pqt, gix, ix, cfg, Y, cfg.w, order="static", label="sift static order")
    finally:
        pqt.pqt_index_free(gix)


def test_sift_full_size_pair_lambda_codes(pqt, sift_full, tmp_path):
    """The same codebooks and database with (pair, lambda) codes from the library's streaming builder."""
    import torch
    cfg, X, Y, path, ix = sift_full
    params = dict(N=cfg.N, H=ix.H, D=ix.D, P=ix.P, k1=ix.k1, k2=ix.k2, M=ix.M, T=ix.T, C=ix.C,
                  C1=ix.C1, C2=ix.C2, cc=ix.cc, code_format=1)
    b = pqt.pqt_builder_create(params, 0)
    try:
        for lo in range(0, cfg.N, 1 << 18):
            pqt.pqt_builder_add(b, torch.from_numpy(X[lo:lo + (1 << 18)]).cuda())
            torch.cuda.synchronize()
        gix = pqt.pqt_builder_finish(b)
    finally:
        pqt.pqt_builder_free(b)
    ppath = str(tmp_path / "sift_pair.pqt")
    try:
        pqt.pqt_index_save(gix, ppath)
        pix = IO.read_index(ppath)
        off = pix.offsets.astype(np.int64)
        assert pix.code_format == 1 and off[0] == 0 and off[-1] == cfg.N and np.all(np.diff(off) >= 0)
        assert np.array_equal(np.sort(pix.ids), np.arange(cfg.N, dtype=np.uint32))
        # the same bins as the index of the other builder, up to fp32 near-ties
        slot_a = np.empty(cfg.N, np.int64)
        slot_a[pix.ids] = np.repeat(np.arange(pix.H), np.diff(off))
        slot_b = np.empty(cfg.N, np.int64)
        slot_b[ix.ids] = np.repeat(np.arange(ix.H), np.diff(ix.offsets.astype(np.int64)))
        assert np.mean(slot_a != slot_b) <= 2e-3
        _full_size_check(pqt, gix, pix, cfg, Y, cfg.w, label="sift pair codes")
    finally:
        pqt.pqt_index_free(gix)


# ---- the parameter shape of the 100M- and 1B-vector workloads -----------------------------------------
@pytest.mark.parametrize("k1", [32, 64])
def test_large_and_billion_parameter_shape(pqt, tmp_path, k1):
    """D = 128, P = 2, k2 = 16, w = 8 (lists of 128 entries), M = 8, T = 1024, C = 10,000, k = 100, with
    k1 = 32 (the 100M workload) and k1 = 64 (the 1B workload: four MFMA column tiles at level 1), on
    16M SIFT-shaped vectors -- enough for the mean run of a bin to be long, so that the re-rank
    wavefronts walk the run lists as they do at full scale.  Index by the library's streaming builder,
    exported to the oracle through the index file.  4,352 queries in one call (more than a tile per compute
    unit: the launch shapes the benchmark times -- traversal of whole tiles, 512-thread re-rank, head pass +
    in-kernel full ranking) checked stage by stage on a sample; the same queries 64 and 1 per call (the
    small-batch launches: traversal split by tree part, 1024 threads) must return the same bits."""
    import torch
    from workloads import sift_like_tables, sift_like_torch
    from paper_1702_05911_amd import builder
    dev = torch.device("cuda", 0)
    N, D, P, k2, M, w, T, C, k, nq = 1 << 24, 128, 2, 16, 8, 8, 1024, 10_000, 100, 4352
    tables = sift_like_tables(D)

    def chunks(s, n):
        return sift_like_torch(s, n, d=D, seed=0, tables=tables, device=dev, chunk=1 << 19)

    print(f"k1={k1}: building {N:,} vectors", flush=True)
    gix = builder.build_index_native(chunks=chunks, N=N, D=D, P=P, k1=k1, k2=k2, M=M, T=T, C=C,
                                     train_n=200_000, iters=8, device=0, chunk_rows=1 << 20, table_train_n=50_000)
    path = str(tmp_path / f"shape_k1_{k1}.pqt")
    try:
        pqt.pqt_index_save(gix, path)
        ix = IO.read_index(path)
        Yd = sift_like_torch(0, nq, d=D, seed=1, tables=tables, device=dev)
        Y = Yd.cpu().numpy()
        print(f"k1={k1}: one call of {nq} queries, debug and plain entry points", flush=True)
        ids, dists, taps = _run_debug(pqt, gix, Y, k, w)
        nr, nc = taps["n_slots"].astype(np.int64), taps["n_cand"].astype(np.int64)
        print(f"k1={k1}: candidates mean {nc.mean():.0f}, runs mean {nr.mean():.1f}, "
              f"queries whose runs average 8 or more: {np.mean(nr * 8 <= nc):.3f}", flush=True)
        assert np.mean(nc == C) > 0.9 and np.mean(nr * 8 <= nc) > 0.5      # the budget is met, long runs are the rule
        same = decided = 0
        sample = list(range(0, nq, 87))                                      # 51 queries
        for q in sample:
            print(f"k1={k1} query {q}", flush=True)
            tr = PU.check_query_stages(ix, Y[q], taps, q, k, w, T, C, ids, dists)
            s_, d_ = PU.end_to_end_agreement(tr, ids[q], dists[q])
            assert s_ or not d_, f"query {q}: margins above threshold but ids differ"
            same += s_
            decided += d_
        print(f"k1={k1}: {same}/{len(sample)} sampled queries identical to the float64 oracle, {decided} decided; "
              + PU.STATS.summary(), flush=True)
        assert same >= 0.8 * len(sample)
        del taps
        # every query of the batch: the top-k is the k smallest (score, id) of its own candidates is covered by
        # the stage-wise sample; here the small-batch launches against the big one, bit for bit
        ids_t, d_t = torch.from_numpy(ids).cuda(), torch.from_numpy(dists).cuda()
        for B, upto in ((64, 512), (1, 48)):
            print(f"k1={k1}: {B} queries per call", flush=True)
            for o in range(0, upto, B):
                bi, bd = pqt.pqt_query_batch(gix, Yd[o:o + B].contiguous(), k, w)
                assert torch.equal(bi, ids_t[o:o + B]) and torch.equal(bd.view(torch.int32), d_t[o:o + B].view(torch.int32)), \
                    f"batch of {B} at {o}"
        # the small-batch launch stage by stage as well
        ids64, d64, taps64 = _run_debug(pqt, gix, Y[100:164], k, w)
        for q in (0, 31, 63):
            PU.check_query_stages(ix, Y[100 + q], taps64, q, k, w, T, C, ids64, d64)
    finally:
        pqt.pqt_index_free(gix)


@pytest.fixture(scope="module")
def gist_full(pqt, tmp_path_factory):
    """GIST-shaped 1M x 960 database, 1,000 queries, P = 4 with H = K = 2^28 bin slots (the pointer
    array alone is 1 GiB, so its probes are real HBM accesses); index trained and built by the library."""
    import torch
    from workloads import CONFIGS, gist_like_torch
    from paper_1702_05911_amd import builder
    cfg = CONFIGS["gist"]
    dev = torch.device("cuda", 0)
    X = gist_like_torch(0, cfg.N, d=cfg.D, seed=cfg.data_seed, device=dev)
    Y = gist_like_torch(0, cfg.nq, d=cfg.D, seed=cfg.query_seed + 100, device=dev)
    path = str(tmp_path_factory.mktemp("gist") / "gist.pqt")
    builder.build_index(path, X, P=cfg.P, k1=cfg.k1, k2=cfg.k2, M=cfg.M, H=cfg.H, T=cfg.T, C=cfg.C,
                        train_n=cfg.train_n, device=0, chunk_rows=1 << 18).close()
    Xh, Yh = X.cpu().numpy(), Y.cpu().numpy()
    del X, Y
    torch.cuda.empty_cache()
    return cfg, Xh, Yh, path, IO.read_index(path)


def test_gist_full_size_parity(pqt, gist_full):
    cfg, X, Y, path, ix = gist_full
    off = ix.offsets.astype(np.int64)
    assert off[0] == 0 and off[-1] == cfg.N and ix.H == cfg.K
    rng = np.random.default_rng(0)
    mism = 0
    for t in rng.integers(0, cfg.N, size=40):
        slot = int(np.searchsorted(off, t, side="right")) - 1
        mism += slot != B.bin_slot(X[ix.ids[t]], ix.C1, ix.C2, ix.H)
    assert mism <= 2          # the fp32 builder may settle a near-tie differently from float64
    gix = pqt.pqt_index_load(path, 0)
    try:
        ids, dists, taps = _run_debug(pqt, gix, Y, cfg.k, cfg.w)
    finally:
        pqt.pqt_index_free(gix)
    nc = taps["n_cand"].astype(np.int64)
    assert np.all(nc <= cfg.C)
    print(f"gist: candidates per query mean {nc.mean():.1f} min {nc.min()} max {nc.max()}", flush=True)
    for q in range(cfg.nq):
        n = int(nc[q])
        sc, cid = taps["scores"][q][:n], taps["cand_ids"][q][:n]
        o = np.lexsort((cid, sc))[:cfg.k]
        assert np.array_equal(ids[q][:len(o)], cid[o]), f"query {q}: top-k is not the k smallest (score, id)"
        assert np.all(ids[q][len(o):] == -1)
    same = decided = 0
    sample = list(range(0, cfg.nq, 97))
    for q in sample:
        print(f"gist query {q}", flush=True)
        tr = PU.check_query_stages(ix, Y[q], taps, q, cfg.k, cfg.w, cfg.T, cfg.C, ids, dists)
        s, d = PU.end_to_end_agreement(tr, ids[q], dists[q])
        assert s or not d, f"query {q}: margins above threshold but ids differ"
        same += s
        decided += d
    print(f"gist: {same}/{len(sample)} sampled queries identical to the float64 oracle, {decided} decided")
    assert same >= 0.7 * len(sample)
