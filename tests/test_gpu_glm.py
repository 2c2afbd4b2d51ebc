"""GPU parity of the gradient passes against the oracle (dense linear models)."""
import numpy as np
import pytest

import lpc_synth
from oracle import lpco
from _common import assert_vectors_do_not_depend_on_the_range, batch_grad_inf, gpu_context, oracle_config, oracle_problem, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [  # name, n, d   (several column tilings, ragged rows, unaligned d)
    ("c1", 1024, 64), ("c1", 517, 100), ("c1", 333, 1000), ("c2", 3000, 4096), ("c2", 1111, 2048),
    ("c4", 700, 8192), ("c4", 256, 777), ("c4", 300, 16384),
]


@pytest.mark.parametrize("name,n,d", SHAPES)
def test_full_gradient(name, n, d):
    import torch
    sp = lpc_synth.make(name, n=n, d=d, N=2, B=8)
    ctx = gpu_context(sp)
    p, _k = oracle_problem(sp)
    rng = np.random.default_rng(1)
    w = (rng.standard_normal(d) * (0.5 / np.sqrt(d) if name != "c2" else 2.0)).astype(np.float32)
    mu = torch.zeros(d, device="cuda")
    z = torch.zeros(n, device="cuda")
    f = torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.full_grad(to_dev(w), mu, z, f)
    mu_o, z_o, f_o = lpco.full_grad(p, w)
    # spec tolerance: max error relative to |mu|_inf at most 1e-5
    assert np.abs(mu.cpu().numpy() - mu_o).max() <= 1e-5 * np.abs(mu_o).max()
    assert np.abs(z.cpu().numpy() - z_o).max() <= 1e-5 * max(1.0, np.abs(z_o).max())
    assert abs(f.item() - f_o) <= 1e-5 * abs(f_o)
    assert abs(ctx.objective(to_dev(w)) - lpco.objective(p, w)) <= 1e-5 * abs(lpco.objective(p, w))
    # reproducible bit for bit (fixed-order reductions, no float atomics)
    mu2 = torch.zeros(d, device="cuda")
    ctx.full_grad(to_dev(w), mu2, None, None)
    assert torch.equal(mu, mu2)
    ctx.close()


def test_full_gradient_partial_snapshot_and_strided_rows():
    import torch
    sp = lpc_synth.make("c2", n=900, d=512, N=2, B=8)
    Xwide = np.zeros((900, 640), dtype=np.float32)
    Xwide[:, :512] = sp.X
    Xwide[:, 512:] = 7.0                       # never read: ldx > d
    from paper_1901_08924_amd import lpc
    cfg = lpc.make_config(N=2, B=8, m=1, bits=4, eta=0.1, n_full=400)
    Xd = to_dev(Xwide)[:, :512]
    ctx = lpc.Context(sp.loss, to_dev(sp.y), cfg, X=Xd, lambda1=sp.lambda1, lambda2=sp.lambda2)
    w = (np.random.default_rng(2).standard_normal(512)).astype(np.float32)
    mu = torch.zeros(512, device="cuda")
    ctx.full_grad(to_dev(w), mu, None, None)
    p, _k = oracle_problem(sp)
    mu_o, _, _ = lpco.full_grad(p, w, n_rows=400)
    assert np.abs(mu.cpu().numpy() - mu_o).max() <= 1e-5 * np.abs(mu_o).max()
    ctx.close()


@pytest.mark.parametrize("name,n,d,N,B", [("c1", 1024, 64, 4, 16), ("c2", 4096, 4096, 8, 64), ("c4", 2048, 8192, 3, 10),
                                           ("c1", 500, 100, 2, 7), ("c4", 512, 777, 5, 1),
                                           # launch shapes of the worker pass with 3, 5, 6 and 8 rows per workgroup
                                           # (chosen so that no CU holds more rows than it must on 256 CUs)
                                           ("c4", 4096, 2048, 8, 64), ("c4", 4096, 2048, 16, 64),
                                           ("c2", 4096, 2048, 16, 96), ("c2", 4096, 2048, 16, 128)])
@pytest.mark.parametrize("cached", [True, False])
def test_worker_vr_gradient(name, n, d, N, B, cached):
    import torch
    sp = lpc_synth.make(name, n=n, d=d, N=N, B=B)
    ctx = gpu_context(sp)
    p, _k = oracle_problem(sp)
    cfg = oracle_config(sp)
    rng = np.random.default_rng(3)
    scale = 2.0 if name == "c2" else 0.5 / np.sqrt(d)
    ws = (rng.standard_normal(d) * scale).astype(np.float32)
    w = (ws + 0.1 * scale * rng.standard_normal(d)).astype(np.float32)
    dw, dws = to_dev(w), to_dev(ws)
    zs = None
    if cached:
        zs = torch.zeros(n, device="cuda")
        ctx.full_grad(dws, torch.zeros(d, device="cuda"), zs, None)
    dp = lpco.d_pad(d)
    for kind, tag, rows in [(1, lpco.TAG_BATCH, N), (2, lpco.TAG_SHARED, 1)]:
        U = torch.full((N, dp), 9.0, device="cuda")
        stats = torch.zeros(N, 4, dtype=torch.float64, device="cuda")
        ctx.worker_vr_grad(dw, dws, zs, 2, 5, U, stats, kind=kind)
        U_o, st_o = lpco.worker_vr_grad(p, cfg, w, ws, 2, 5, tag=tag)
        got = U.cpu().numpy()[:rows]
        # u is a difference of nearly equal per-sample gradients: compare relative to the larger of
        # |grad f_B(w)|_inf and |u|_inf
        for i in range(rows):
            ref_scale = max(batch_grad_inf(sp, w, 2, 5, tag, i), np.abs(U_o[i]).max())
            assert np.abs(got[i] - U_o[i]).max() <= 2e-5 * ref_scale
            assert not got[i, d:].any()
        sg = stats.cpu().numpy()[:rows]
        assert np.array_equal(sg[:, 0], np.abs(got[:, :d]).max(axis=1).astype(np.float64))
        assert np.allclose(sg[:, 1], got[:, :d].astype(np.float64).sum(axis=1), rtol=1e-9, atol=1e-12)
        assert np.allclose(sg[:, 2], (got[:, :d].astype(np.float64) ** 2).sum(axis=1), rtol=1e-9)
    # at the snapshot the difference is exactly zero when the margins are recomputed with the same kernel
    if not cached:
        U = torch.full((N, dp), 9.0, device="cuda")
        ctx.worker_vr_grad(dws, dws, None, 0, 0, U, None)
        assert not U.any().item()
    ctx.close()


@pytest.mark.parametrize("name,d,N,B", [("c1", 90, 8, 64), ("c2", 2048, 16, 16), ("c2", 4096, 8, 64), ("c4", 8192, 16, 8),
                                         ("c2", 20000, 8, 4), ("c3", 50_000, 8, 64)])
def test_worker_vectors_do_not_depend_on_the_range(name, d, N, B):
    sp = lpc_synth.make(name, n=2048, d=d, N=N, B=B, seed=d)
    ctx = gpu_context(sp, clip_mode=lpco.CLIP_CSIGMA, clip=1.0)
    assert_vectors_do_not_depend_on_the_range(ctx, sp)
    ctx.close()


# ---------------------------------------------------------------- CSR rows (sparse text-like design)

CSR_SHAPES = [(2000, 512, 12), (5000, 20_000, 30), (3000, 100_000, 50), (700, 33, 5)]


@pytest.mark.parametrize("n,d,nnz", CSR_SHAPES)
def test_csr_full_gradient(n, d, nnz):
    import torch
    sp = lpc_synth.make("c3", n=n, d=d, nnz_mean=nnz, N=2, B=8)
    ctx = gpu_context(sp)
    p, _k = oracle_problem(sp)
    w = (np.random.default_rng(1).standard_normal(d) * 2.0).astype(np.float32)
    mu = torch.full((d,), 7.0, device="cuda")
    z = torch.zeros(n, device="cuda")
    f = torch.zeros(1, dtype=torch.float64, device="cuda")
    ctx.full_grad(to_dev(w), mu, z, f)
    mu_o, z_o, f_o = lpco.full_grad(p, w)
    assert np.abs(mu.cpu().numpy() - mu_o).max() <= 1e-5 * np.abs(mu_o).max()
    assert np.abs(z.cpu().numpy() - z_o).max() <= 1e-5 * max(1.0, np.abs(z_o).max())
    assert abs(f.item() - f_o) <= 1e-5 * abs(f_o)
    assert abs(ctx.objective(to_dev(w)) - lpco.objective(p, w)) <= 1e-5 * abs(lpco.objective(p, w))
    ctx.close()


@pytest.mark.parametrize("n,d,nnz", CSR_SHAPES)
@pytest.mark.parametrize("cached", [True, False])
def test_csr_worker_vr_gradient(n, d, nnz, cached):
    import torch
    N, B = 4, 16
    sp = lpc_synth.make("c3", n=n, d=d, nnz_mean=nnz, N=N, B=B)
    ctx = gpu_context(sp)
    p, _k = oracle_problem(sp)
    cfg = oracle_config(sp)
    rng = np.random.default_rng(3)
    ws = (rng.standard_normal(d) * 2.0).astype(np.float32)
    w = (ws + 0.2 * rng.standard_normal(d)).astype(np.float32)
    dw, dws = to_dev(w), to_dev(ws)
    zs = None
    if cached:
        zs = torch.zeros(n, device="cuda")
        ctx.full_grad(dws, torch.zeros(d, device="cuda"), zs, None)
    dp = lpco.d_pad(d)
    for kind, tag, rows in [(1, lpco.TAG_BATCH, N), (2, lpco.TAG_SHARED, 1)]:
        U = torch.full((N, dp), 9.0, device="cuda")
        stats = torch.zeros(N, 4, dtype=torch.float64, device="cuda")
        ctx.worker_vr_grad(dw, dws, zs, 1, 3, U, stats, kind=kind)
        U_o, st_o = lpco.worker_vr_grad(p, cfg, w, ws, 1, 3, tag=tag)
        got = U.cpu().numpy()[:rows]
        for i in range(rows):
            ref_scale = max(batch_grad_inf(sp, w, 1, 3, tag, i), np.abs(U_o[i]).max())
            assert np.abs(got[i] - U_o[i]).max() <= 2e-5 * ref_scale
            assert np.array_equal(got[i] != 0, U_o[i] != 0) or np.abs(got[i][(got[i] != 0) != (U_o[i] != 0)]).max() < 1e-6 * ref_scale
        sg = stats.cpu().numpy()[:rows]
        assert np.array_equal(sg[:, 0], np.abs(got[:, :d]).max(axis=1).astype(np.float64))
    ctx.close()
