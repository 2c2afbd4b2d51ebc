"""GPU parity of whole epochs: Alg. 1 and Alg. 2/3 against the oracle, objective within 1e-4."""
import numpy as np
import pytest

import lpc_synth
from oracle import lpco
from _common import gpu_context, oracle_config, oracle_problem, to_dev

pytestmark = pytest.mark.gpu


def _run_both(sp, epochs, **over):
    ctx = gpu_context(sp, **over)
    p, _k = oracle_problem(sp)
    cfg = oracle_config(sp, **over)
    alpc = cfg.algo != lpco.ALGO_LPC
    w_o = sp.w0.copy()
    y_o, z_o = (sp.w0.copy(), sp.w0.copy()) if alpc else (None, None)
    w_g = to_dev(sp.w0)
    y_g, z_g = (to_dev(sp.w0), to_dev(sp.w0)) if alpc else (None, None)
    hist = []
    for s in range(epochs):
        lpco.epoch(p, cfg, w_o, s, y_o, z_o)
        ctx.epoch(w_g, s, y_g, z_g)
        hist.append((lpco.objective(p, w_o), ctx.objective(w_g), lpco.objective(p, w_g.cpu().numpy())))
    assert ctx.take_device_flags() == 0
    ctx.close()
    return hist, w_o, w_g.cpu().numpy()


def test_c1_ten_epochs_objective_parity():
    sp = lpc_synth.make("c1")      # the full tiny config: n=1024, d=64, N=4, B=16, b=2, c*sigma clip, 10 epochs
    hist, w_o, w_g = _run_both(sp, sp.epochs)
    for P_o, P_g, P_og in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)       # spec tolerance
        assert abs(P_g - P_og) <= 1e-5 * abs(P_og)     # the GPU objective of its own iterate
    assert hist[-1][0] < hist[0][0]
    assert np.abs(w_g - w_o).max() <= 1e-3 * max(1.0, np.abs(w_o).max())


@pytest.mark.parametrize("bits,clip_mode,clip", [(32, 0, 1.0), (4, 0, 0.9), (3, 1, 2.0)])
def test_lpc_epochs_small_dense(bits, clip_mode, clip):
    sp = lpc_synth.make("c2", n=2048, d=512, N=4, B=16)
    hist, w_o, w_g = _run_both(sp, 4, bits=bits, clip_mode=clip_mode, clip=clip)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    assert hist[-1][0] < hist[0][0]


def test_quantization_off_tracks_the_oracle_closely():
    # without stochastic rounding the two trajectories differ by float rounding only
    sp = lpc_synth.make("c1", n=512, d=40, N=4, B=8)
    hist, w_o, w_g = _run_both(sp, 5, bits=32)
    assert np.abs(w_g - w_o).max() <= 2e-5 * max(1.0, np.abs(w_o).max())


@pytest.mark.parametrize("algo", [lpco.ALGO_ALPC_SC, lpco.ALGO_ALPC_GC])
@pytest.mark.parametrize("bits", [32, 3])
def test_alpc_epochs_ridge(algo, bits):
    sp = lpc_synth.make("c4", n=2048, d=256, N=4, B=16)
    hist, w_o, w_g = _run_both(sp, 4, algo=algo, bits=bits, tau2=0.5)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    assert hist[-1][0] < hist[0][0]
    if bits == 32:
        assert np.abs(w_g - w_o).max() <= 5e-5 * max(1.0, np.abs(w_o).max())


def test_epoch_is_reproducible():
    import torch
    sp = lpc_synth.make("c2", n=1024, d=256, N=4, B=16)
    ctx = gpu_context(sp)
    a, b = to_dev(sp.w0), to_dev(sp.w0)
    ctx.epoch(a, 0); ctx.epoch(a, 1)
    ctx.epoch(b, 0); ctx.epoch(b, 1)
    assert torch.equal(a, b)
    ctx.close()


@pytest.mark.parametrize("d,B,over", [
    (50_000, 100, {}),                                  # sparse inner iteration, two rounds of rows per worker
    (50_000, 16, dict(scheme=lpco.SCHEME_B)),           # dense-U worker pass (shared scale), large d
    (2048, 70, {}),                                     # small d: many rows of a batch share columns
    (3000, 32, dict(algo=lpco.ALGO_ALPC_GC, L=0.25, tau2=0.5)),
])
def test_csr_epoch_is_reproducible(d, B, over):
    """CSR data: the snapshot gradient and the workers' differences are summed in a fixed order (no float atomics
    whose arrival order could matter), so two runs give the same bits -- and with them the same stochastic
    rounding decisions and the same iterates."""
    import torch
    sp = lpc_synth.make("c3", n=4096, d=d, nnz_mean=30, N=4, B=B)
    runs = []
    for _ in range(3):
        ctx = gpu_context(sp, m=5, **over)
        alpc = ctx.config.algo != 0
        w = to_dev(sp.w0)
        y, z = (to_dev(sp.w0), to_dev(sp.w0)) if alpc else (None, None)
        for s in range(3):
            ctx.epoch(w, s, y, z)
        mu = torch.zeros(sp.d, device="cuda")
        ctx.full_grad(w, mu, None, None)
        U = torch.zeros(sp.N, lpco.d_pad(sp.d), device="cuda")
        ctx.worker_vr_grad(w, to_dev(sp.w0), None, 7, 3, U, None)
        runs.append((w.clone(), mu, U))
        ctx.close()
    assert runs[0][0].abs().max().item() > 0
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("d,bits", [(2048, 2), (40_000, 2), (40_000, 32)])
def test_lpc_epochs_csr(d, bits):
    # sparse rows: small-d single-launch exchange and the large-d path
    sp = lpc_synth.make("c3", n=4096, d=d, nnz_mean=20, N=4, B=16)
    hist, w_o, w_g = _run_both(sp, 3, bits=bits)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    assert hist[-1][0] < hist[0][0]


@pytest.mark.parametrize("scheme", [lpco.SCHEME_B, lpco.SCHEME_C])
@pytest.mark.parametrize("algo", [lpco.ALGO_LPC, lpco.ALGO_ALPC_GC])
def test_shared_scale_schemes_epochs(scheme, algo):
    # Sec. 4.2 (b), (c): parameter-server style exchange with one scale factor for all workers
    name = "c2" if algo == lpco.ALGO_LPC else "c4"
    sp = lpc_synth.make(name, n=2048, d=512, N=4, B=16)
    hist, w_o, w_g = _run_both(sp, 3, algo=algo, scheme=scheme, bits=4, clip_mode=0, clip=1.0, tau2=0.5)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    assert hist[-1][0] < hist[0][0]


@pytest.mark.parametrize("bits,clip_mode,clip,n_full", [(2, 0, 1.0, 0), (5, 0, 0.8, 0), (4, 1, 2.0, 0), (3, 0, 1.0, 2048)])
def test_sparse_inner_iteration_matches_the_oracle_coordinate_by_coordinate(bits, clip_mode, clip, n_full):
    """CSR rows that touch few columns take the sparse passes (head partials + marked tail segments).  The
    oracle works on dense vectors; the iterates must agree coordinate by coordinate except where a float
    rounding difference in u (scatter order) flips a stochastic rounding decision: such a flip moves one
    coordinate of w by eta*delta/N, so only a handful of coordinates may differ, and by little."""
    sp = lpc_synth.make("c3", n=4096, d=50_000, nnz_mean=20, N=4, B=16)
    over = dict(bits=bits, clip_mode=clip_mode, clip=clip, m=6, n_full=n_full)
    hist, w_o, w_g = _run_both(sp, 2, **over)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    scale = max(np.abs(w_o).max(), 1e-12)
    diff = np.abs(w_g - w_o)
    assert np.count_nonzero(w_o) > 1000                      # the iterate has moved on head and tail columns
    assert np.count_nonzero(w_o[8192:]) > 100
    assert (diff > 1e-5 * scale).mean() <= 2e-3              # a few flipped decisions at most
    assert diff.max() <= 0.05 * scale
    # the same support (the L1 prox zeroes exactly the same coordinates, up to those few)
    assert np.count_nonzero((w_o == 0) != (w_g == 0)) <= 2e-3 * sp.d


@pytest.mark.parametrize("nnz_mean,B", [(80, 16), (160, 70)])
def test_sparse_inner_iteration_with_long_rows_and_the_wide_head(nnz_mean, B):
    """d >= 2^17: the sparse passes treat 16384 leading columns densely.  Rows longer than 64 entries: the worker
    pass stages a row's first 64 pairs and takes the rest from memory (head and tail wavefronts both), B = 70 adds
    a second workgroup per worker, hence a second tail plane.  Same agreement with the dense oracle as above."""
    sp = lpc_synth.make("c3", n=2048, d=140_000, nnz_mean=nnz_mean, N=4, B=B)
    rp = sp.csr[0]
    assert (np.diff(rp) > 64).mean() > 0.1
    hist, w_o, w_g = _run_both(sp, 2, bits=3, m=5)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    scale = max(np.abs(w_o).max(), 1e-12)
    diff = np.abs(w_g - w_o)
    assert np.count_nonzero(w_o[:64]) > 32 and np.count_nonzero(w_o[64:16384]) > 1000
    assert np.count_nonzero(w_o[16384:]) > 100
    assert (diff > 1e-5 * scale).mean() <= 2e-3
    assert diff.max() <= 0.05 * scale
    assert np.count_nonzero((w_o == 0) != (w_g == 0)) <= 2e-3 * sp.d


@pytest.mark.parametrize("scheme,bits,clip_mode,clip,d", [
    (lpco.SCHEME_B, 3, 0, 1.0, 50_000), (lpco.SCHEME_C, 4, 0, 0.9, 50_000), (lpco.SCHEME_B, 2, 1, 2.0, 50_000),
    (lpco.SCHEME_C, 3, 0, 1.0, 140_000)])                      # d >= 2^17: 16384 dense head columns
def test_sparse_inner_iteration_with_a_shared_scale_factor(scheme, bits, clip_mode, clip, d):
    """Sec. 4.2 (b), (c) on CSR rows that touch few columns: the sparse worker, statistics and quantizer passes with
    delta = max_i delta_i, then the integer-sum receiver (eq. (5) for scheme (c)).  Coordinate-level agreement
    with the oracle as for scheme (a); the same bits run to run."""
    import torch
    sp = lpc_synth.make("c3", n=4096, d=d, nnz_mean=20, N=4, B=16)
    over = dict(bits=bits, clip_mode=clip_mode, clip=clip, m=6, scheme=scheme)
    hist, w_o, w_g = _run_both(sp, 2, **over)
    for P_o, P_g, _ in hist:
        assert abs(P_g - P_o) <= 1e-4 * abs(P_o)
    scale = max(np.abs(w_o).max(), 1e-12)
    diff = np.abs(w_g - w_o)
    assert np.count_nonzero(w_o) > 1000 and np.count_nonzero(w_o[8192:]) > 100
    assert (diff > 1e-5 * scale).mean() <= 2e-3
    assert diff.max() <= 0.05 * scale
    _h, _w, w_again = _run_both(sp, 2, **over)
    assert np.array_equal(w_g, w_again)


@pytest.mark.parametrize("algo,scheme,bits,clip_mode,clip,B", [
    (lpco.ALGO_ALPC_GC, lpco.SCHEME_A, 3, 0, 1.0, 16), (lpco.ALGO_ALPC_SC, lpco.SCHEME_A, 4, 1, 2.0, 16),
    (lpco.ALGO_ALPC_GC, lpco.SCHEME_B, 4, 0, 0.9, 16), (lpco.ALGO_ALPC_GC, lpco.SCHEME_C, 2, 0, 1.0, 16),
    (lpco.ALGO_ALPC_GC, lpco.SCHEME_A, 3, 0, 1.0, 70),         # B = 70: two workgroups (planes) per vector
    (lpco.ALGO_ALPC_GC, lpco.SCHEME_A, 3, 0, 1.0, -70)])       # ... and d >= 2^17: 16384 dense head columns
def test_sparse_inner_iteration_of_alpc_svrg(algo, scheme, bits, clip_mode, clip, B):
    """Alg. 2 / Alg. 3 on CSR rows that touch few columns: the workers' vectors AND the shared batch's
    full-precision difference take the sparse worker and statistics passes; coordinate-level agreement of x~, y and z
    with the oracle (up to a few flipped rounding decisions) and the same bits run to run."""
    d, B = (140_000, -B) if B < 0 else (50_000, B)
    sp = lpc_synth.make("c3", n=4096, d=d, nnz_mean=20, N=4, B=B)
    over = dict(algo=algo, scheme=scheme, bits=bits, clip_mode=clip_mode, clip=clip, m=6, tau2=0.5, L=0.25,
                sigma=1e-3 if algo == lpco.ALGO_ALPC_SC else 0.0)
    runs = []
    for _ in range(2):
        ctx = gpu_context(sp, **over)
        w_g, y_g, z_g = to_dev(sp.w0), to_dev(sp.w0), to_dev(sp.w0)
        for s in range(2):
            ctx.epoch(w_g, s, y_g, z_g)
        assert ctx.take_device_flags() == 0
        P_g = ctx.objective(w_g)
        ctx.close()
        runs.append((w_g.cpu().numpy(), y_g.cpu().numpy(), z_g.cpu().numpy(), P_g))
    p, _k = oracle_problem(sp)
    cfg = oracle_config(sp, **over)
    w_o, y_o, z_o = sp.w0.copy(), sp.w0.copy(), sp.w0.copy()
    for s in range(2):
        lpco.epoch(p, cfg, w_o, s, y_o, z_o)
    P_o = lpco.objective(p, w_o)
    assert abs(runs[0][3] - P_o) <= 1e-4 * abs(P_o)
    for got, want in zip(runs[0][:3], (w_o, y_o, z_o)):
        scale = max(np.abs(want).max(), 1e-12)
        diff = np.abs(got - want)
        assert np.count_nonzero(want) > 1000
        assert (diff > 1e-5 * scale).mean() <= 2e-3
        assert diff.max() <= 0.05 * scale
    for a, b in zip(runs[0][:3], runs[1][:3]):
        assert np.array_equal(a, b)


def _csr_problem(d, N, B, rows, seed=3):
    """Logistic regression on 2000 unit rows; rows(rng, r) gives row r's columns."""
    sp = lpc_synth.make("c3", n=2000, d=d, nnz_mean=4, N=N, B=B)
    rng = np.random.default_rng(seed)
    cols = [np.sort(np.asarray(rows(rng, r), dtype=np.int32)) for r in range(sp.n)]
    rp = np.zeros(sp.n + 1, dtype=np.int32)
    np.cumsum([c.size for c in cols], out=rp[1:])
    vals = [rng.standard_normal(c.size) / max(1.0, np.sqrt(c.size)) for c in cols]
    sp.csr = (rp, np.concatenate(cols).astype(np.int32), np.concatenate(vals).astype(np.float32))
    sp.w0 = (0.1 * rng.standard_normal(d)).astype(np.float32)
    return sp


def _zipf(d, mean):
    return lambda rng, r: np.unique(np.minimum(d - 1, (rng.pareto(0.7, 1 + r % (2 * mean)) * 2).astype(np.int64)))


def _one_bin(rng, r):  # columns of one owner, a quarter of its own
    return 5 + 256 * (4 + 4 * rng.choice(200, 16, replace=False))


@pytest.mark.parametrize("d,N,B,rows,over", [
    (1, 2, 3, lambda rng, r: [0], {}),                                             # one column, 255 owners without any
    (200, 1, 1, _zipf(200, 4), dict(bits=5)),
    (257, 16, 33, _zipf(257, 10), dict(bits=16, scheme=lpco.SCHEME_C)),
    (1000, 16, 40, _zipf(1000, 8), dict(algo=lpco.ALGO_ALPC_GC, bits=3)),          # seventeen lists, sixteen wavefronts
    (4096, 5, 20, _zipf(4096, 300), {}),                                           # rows past 64 entries
    (5000, 4, 50, lambda rng, r: [] if r % 3 else _zipf(5000, 9)(rng, r), dict(bits=4, clip_mode=1, clip=2.0)),  # empty rows
    (5001, 3, 512, lambda rng, r: list(range(10)) + [10 + r], dict(bits=4)),       # lists past five chunks
    (5003, 3, 200, lambda rng, r: rng.integers(0, 40, 30), dict(bits=6)),          # a row holds a column several times
    (60000, 2, 512, lambda rng, r: rng.choice(60000, 60, replace=False), {}),      # more keys than the builder holds at once
    (262144, 2, 400, _one_bin, {}),                                                # ... all in one bin; lists past 128 columns
    (262144, 2, 512, _one_bin, dict(m=2)),                                         # more than it sorts: the separate launches
    (3000, 2, 4, _zipf(3000, 20), dict(m=131, n_full=700)),                        # a second launch; margins taken by the plan
    (3000, 15, 64, _zipf(3000, 20), dict(algo=lpco.ALGO_ALPC_SC, scheme=lpco.SCHEME_B, bits=4)),
    (2999, 7, 9, _zipf(2999, 6), dict(algo=lpco.ALGO_ALPC_GC, scheme=lpco.SCHEME_C, bits=7, n_full=900, clip_mode=1, clip=1.0))])
def test_csr_epochs_in_one_launch(d, N, B, rows, over):
    """Workgroups by columns, lists of the sampled entries: agreement with the oracle's dense arithmetic up to a few flipped
    rounding decisions (a flip moves a coordinate by eta*delta/N), and the bits of the separate launches (with clipping by c*sigma
    the sums over the coordinates have another order: their last bits reach no scale factor here)."""
    from paper_1901_08924_amd import lpc
    sp = _csr_problem(d, N, B, rows)
    over = dict(dict(m=6, L=0.5, eta=0.4, bits=2, sigma=1e-3, tau2=0.5), **over)
    runs = []
    for form in (-1, 0):
        ctx = gpu_context(sp, **over)
        if form == 0:
            ctx.tune(lpc.TUNE_ITER_FORM, form)
        vec = [to_dev(sp.w0) for _ in range(3)]
        for s in range(2):
            ctx.epoch(vec[0], s, vec[1], vec[2])
        assert ctx.take_device_flags() == 0
        runs.append([v.cpu().numpy() for v in vec])
        ctx.close()
    p, _k = oracle_problem(sp)
    cfg = oracle_config(sp, **over)
    want = [sp.w0.copy() for _ in range(3)]
    for s in range(2):
        lpco.epoch(p, cfg, want[0], s, want[1], want[2])
    P = lpco.objective(p, want[0])
    assert abs(lpco.objective(p, runs[0][0]) - P) <= 1e-4 * abs(P)
    for got, separate, w in zip(*runs, want):
        assert np.array_equal(got, separate)
        diff, scale = np.abs(got - w), np.abs(w).max()
        assert (diff > 1e-5 * scale).mean() <= max(2e-3, 2.0 / d) and diff.max() <= 0.05 * scale


@pytest.mark.parametrize("form", [-1, 0])
@pytest.mark.parametrize("B", [20, 70])
def test_sparse_epochs_of_rows_that_hold_a_column_several_times(B, form):
    """Among the frequent columns that the sparse worker pass keeps a value per row of, up to a row's 64th entry, and among the
    others."""
    from paper_1901_08924_amd import lpc
    sp = _csr_problem(70000, 4, B, lambda rng, r: np.concatenate([rng.integers(0, 70, 20 + r % 50), rng.integers(69990, 70000, 5)]))
    over = dict(m=40, L=0.5, eta=0.4, bits=8)
    ctx = gpu_context(sp, **over)
    ctx.tune(lpc.TUNE_ITER_FORM, form)
    vec, one_launch = _epoch_and_route(ctx, sp)
    assert one_launch == (form == -1) and ctx.take_device_flags() == 0
    ctx.close()
    p, _k = oracle_problem(sp)
    want = sp.w0.copy()
    lpco.epoch(p, oracle_config(sp, **over), want, 0)
    # a flipped rounding decision moves a coordinate by eta * delta / N, 2e-6 of the largest here; entries left out, by 5e-4
    assert np.abs(vec[0] - want).max() <= 1e-5 * np.abs(want).max() and np.abs(want - sp.w0).max() >= 0.05 * np.abs(want).max()


def _epoch_and_route(ctx, sp, epochs=1):
    """x~, y and z after the epochs, and whether the inner loop was one launch."""
    vec = [to_dev(sp.w0) for _ in range(3)]
    ctx.profile_enable(True)
    for s in range(epochs):
        ctx.epoch(vec[0], s, vec[1], vec[2])
    ctx.profile_enable(False)
    counts = ctx.profile_read()
    return np.stack([v.cpu().numpy() for v in vec]), counts["resident"][1] > 0 and counts["vr_rows"][1] == 0


def _spread(d, count):  # one column of each of `count` ranges
    return lambda rng, r: np.arange(count) * (d // count) + rng.integers(0, d // count, count)


@pytest.mark.parametrize("d,B,rows,m,one_launch", [
    (262144, 400, _one_bin, 6, True), (262144, 401, _one_bin, 6, False),  # 6400 entries of one owner, and 6416: what the builder sorts
    (3000, 50, _spread(3000, 20), 4, False), (3000, 50, _spread(3000, 20), 5, True),  # few iterations of few entries
    (3000, 313, _spread(3000, 20), 4, True), (3000, 312, _spread(3000, 20), 4, False),  # ... of 12520 and 12480
    (3000, 512, _spread(3000, 400), 5, False), (3000, 512, _spread(3000, 400), 6, True),  # 204800 in a batch: 40960 and 34133 each
    (524288, 256, _spread(524288, 240), 5, False), (524288, 256, _spread(524288, 240), 6, True),  # u^i sparse: 12288, 10240
    (4000, 512, _spread(4000, 588), 9, False)])                            # 301056 in a batch
def test_csr_epochs_take_one_launch_where_it_pays(d, B, rows, m, one_launch):
    from paper_1901_08924_amd import lpc
    sp = _csr_problem(d, 2, B, rows)
    got = []
    for form in (-1, 0):
        ctx = gpu_context(sp, m=m, L=0.5, eta=0.4, bits=4)
        if form == 0:
            ctx.tune(lpc.TUNE_ITER_FORM, form)
        vec, route = _epoch_and_route(ctx, sp)
        assert route == (one_launch and form == -1) and ctx.take_device_flags() == 0
        got.append(vec)
        ctx.close()
    assert np.array_equal(*got) and not np.array_equal(got[0][0], sp.w0)


@pytest.mark.parametrize("where", ["w", "value", "label", "largest"])
@pytest.mark.parametrize("d,over", [(3000, {}), (50000, {}), (3000, dict(m=1, B=400)), (50000, dict(clip_mode=1, clip=2.0)),
                                    (3000, dict(algo=lpco.ALGO_ALPC_GC)), (50000, dict(algo=lpco.ALGO_ALPC_GC, scheme=lpco.SCHEME_B)),
                                    (3000, dict(scheme=lpco.SCHEME_C))])
def test_csr_epochs_of_numbers_that_are_not_finite(d, over, where):
    """Infinities and NaN in the iterate, in entries and labels, and entries whose margins and sums overflow: the numbers and the
    flag of the separate launches."""
    from paper_1901_08924_amd import lpc
    over = dict(dict(m=6, N=5, B=64, L=0.5, eta=0.4, bits=4, tau2=0.5), **over)
    sp = _csr_problem(d, over["N"], over["B"], _zipf(d, 20) if over["m"] > 1 else _spread(d, 40))
    rng = np.random.default_rng(1)
    some = rng.permutation(sp.n)[:12]
    if where == "w":
        sp.w0[[3, 700, 2900]] = np.inf, np.nan, -np.inf
    elif where == "value":
        sp.csr[2][sp.csr[0][some]] = np.resize([np.inf, np.nan, -np.inf], 12)
    elif where == "label":
        sp.y = sp.y.copy()
        sp.y[some] = np.nan
    else:
        sp.csr[2][:] *= np.float32(2e38) / np.abs(sp.csr[2]).max()
    got = []
    for form in (-1, 0):
        ctx = gpu_context(sp, **over)
        if form == 0:
            ctx.tune(lpc.TUNE_ITER_FORM, form)
        vec, route = _epoch_and_route(ctx, sp, epochs=2 if over["m"] > 1 else 1)
        assert route == (form == -1)
        got.append((vec, ctx.take_device_flags()))
        ctx.close()
    # (one iteration of differences at x~: zeros while the margins are finite)
    assert got[0][1] == got[1][1] == (0 if where == "largest" and over["m"] == 1 else lpc.ENONFINITE)
    assert np.array_equal(got[0][0], got[1][0], equal_nan=True)


@pytest.mark.parametrize("over", [{}, dict(algo=lpco.ALGO_ALPC_GC, scheme=lpco.SCHEME_B)])
def test_csr_epoch_that_gives_up_or_is_refused(over):
    """The caller's vectors are the epoch's or what they were, whatever the waits are given; a launch that does not fit
    takes the separate ones."""
    from paper_1901_08924_amd import lpc
    sp = _csr_problem(3000, 5, 64, _zipf(3000, 20))
    ctx, form0 = (gpu_context(sp, **dict(dict(m=6, bits=4, L=0.5, eta=0.4, tau2=0.5), **over)) for _ in range(2))
    form0.tune(lpc.TUNE_ITER_FORM, 0)

    def epoch(c, spin=1 << 15):
        c.tune(lpc.TUNE_SPIN_LIMIT, spin)
        vec = [to_dev(sp.w0) for _ in range(3)]
        c.profile_enable(True)
        c.epoch(vec[0], 1, vec[1], vec[2])
        c.profile_enable(False)
        one_launch = c.profile_read()["vr_rows"][1] == 0
        return np.stack([v.cpu().numpy() for v in vec]), c.take_device_flags(), one_launch

    want, flags, one_launch = epoch(ctx)
    separate, flags_s, one_launch_s = epoch(form0)
    assert flags == flags_s == 0 and one_launch and not one_launch_s
    assert np.array_equal(want, separate)
    for spin in (0, 1, 2, 4):
        got, flags, _ = epoch(ctx, spin)
        assert np.array_equal(got, want if flags == 0 else np.stack([sp.w0] * 3))
        assert flags == lpc.EDEVICE or (flags == 0 and spin > 0)
    ctx.tune(lpc.TUNE_COMPUTE_UNITS, 255)
    got, flags, one_launch = epoch(ctx)
    assert flags == 0 and not one_launch and np.array_equal(got, separate)
    ctx.tune(lpc.TUNE_COMPUTE_UNITS, 256)
    got, flags, one_launch = epoch(ctx)
    assert flags == 0 and one_launch and np.array_equal(got, want)
    ctx.close()
    form0.close()
