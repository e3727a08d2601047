"""GPU parity of the on-device calibration (table step 1) against the oracle's fp64 calibration.

* kvc_eigh (fp32 Jacobi) on the 256 key and value covariances of the 8B-shaped workload: eigenvalues
  within 1e-5 of the largest (about 128 fp32 roundings), U diag(lambda) U^T reproducing the
  covariance to the same level, orthonormal columns,
  and each eigenvector whose eigenvalue is separated from the others within the angle that a backward
  error of 1e-5 of the norm allows (a Davis-Kahan bound); every matrix converges.
* kvc_query_variance on the same U (the oracle's, rounded to fp32) within 1e-5 relative.
* kvc_covariance of fp16 activations (ragged and tile-multiple token counts, centred and not, with
  a mean offset) within 1e-4 normwise of the oracle's fp64 sample covariance of the same values.
* The whole chain as the pipeline runs it (exact covariances -> kvc_eigh -> kvc_query_variance ->
  kvc_allocate): tables equal the oracle-calibrated ones on nearly every head, and the total
  modelled distortion agrees to 1e-3.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import alloc as oa
from oracle import calib
from oracle.native import jacobi_eigh
from paper_2609_24298_amd import kvc, pipeline, synth

from oracle_stats import stats_from_covs

pytestmark = pytest.mark.gpu


def log(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def covs8b():
    w = synth.WORKLOADS["llama8b_b8_t32k_2bpd"]
    return w, synth.workload_covs(w, 0)


def _gpu_eigh(S):
    St = torch.as_tensor(S.astype(np.float32), device="cuda")
    n = S.shape[0]
    lam = torch.empty((n, 128), dtype=torch.float32, device="cuda")
    U = torch.empty((n, 128, 128), dtype=torch.float32, device="cuda")
    sw = torch.empty(n, dtype=torch.int32, device="cuda")
    kvc.kvc_eigh(St, lam, U, sw)
    torch.cuda.synchronize()
    return lam.cpu().numpy().astype(np.float64), U.cpu().numpy().astype(np.float64), sw.cpu().numpy()


@pytest.mark.parametrize("side", ["k", "v"])
def test_eigh_matches_oracle(covs8b, side):
    w, covs = covs8b
    S = np.stack([getattr(c, "S_" + side) for c in covs])
    lam, U, sw = _gpu_eigh(S)
    lo, Uo, _ = jacobi_eigh(S)
    assert np.all(sw > 0) and sw.max() <= 20, sw.max()
    worst_l = worst_r = worst_a = 0.0
    for h in range(S.shape[0]):
        lmax = lo[h, 0]
        worst_l = max(worst_l, np.max(np.abs(lam[h] - lo[h])) / lmax)
        worst_r = max(worst_r, np.max(np.abs(U[h] @ np.diag(lam[h]) @ U[h].T - S[h])) / lmax)
        assert np.max(np.abs(U[h].T @ U[h] - np.eye(128))) <= 1e-5, h
        gap = np.abs(lo[h][:, None] - lo[h][None, :]) + np.diag(np.full(128, np.inf))
        gap = gap.min(axis=1)
        # angle between each pair of unit vectors, 2 asin(|u - sign v| / 2) (accurate near zero, where
        # arccos of the dot product is not)
        un = U[h] / np.linalg.norm(U[h], axis=0)
        sg = np.sign(np.sum(un * Uo[h], axis=0))
        ang = 2.0 * np.arcsin(np.minimum(np.linalg.norm(un - sg * Uo[h], axis=0) / 2.0, 1.0))
        bound = 1e-5 * lmax / gap
        ok = gap > 1e-3 * lmax
        assert np.all(ang[ok] <= bound[ok]), (h, np.max(ang[ok] / bound[ok]))
        worst_a = max(worst_a, float(np.max(ang[ok] / bound[ok])) if ok.any() else 0.0)
    assert worst_l <= 1e-5 and worst_r <= 1e-5, (worst_l, worst_r)
    log(f"[eigh {side}] {S.shape[0]} heads: eigenvalue error {worst_l:.1e} of the largest, reconstruction "
        f"{worst_r:.1e}, eigenvector angle at most {worst_a:.2f} of its bound; sweeps {sw.min()}..{sw.max()}")


def test_query_variance_matches_oracle(covs8b):
    w, covs = covs8b
    covs = covs[:64]
    _, Uo, _ = jacobi_eigh(np.stack([c.S_k for c in covs]))
    U32 = Uo.astype(np.float32)
    Sq32 = np.stack([np.stack(c.S_q) for c in covs]).astype(np.float32)
    sig = torch.empty((len(covs), 128), dtype=torch.float32, device="cuda")
    kvc.kvc_query_variance(torch.as_tensor(U32, device="cuda"), torch.as_tensor(Sq32, device="cuda"), sig)
    torch.cuda.synchronize()
    got = sig.cpu().numpy()
    for h in range(len(covs)):
        ref = calib.query_variance(U32[h].astype(np.float64), list(Sq32[h].astype(np.float64)))
        assert np.allclose(got[h], ref, rtol=1e-5, atol=1e-6 * ref.max()), h


@pytest.mark.parametrize("n_tok,centered", [(32768, True), (1000, True), (4096, False)])
def test_covariance_matches_oracle(n_tok, centered):
    rng = np.random.default_rng(n_tok)
    H = 12
    covs = [synth.head_cov(1, 0, h, 1) for h in range(H)]
    x = np.zeros((H, n_tok, 128), dtype=np.float16)
    for h, c in enumerate(covs):
        off = 0.5 * rng.standard_normal(128) * np.sqrt(np.diag(c.S_k)) if h % 2 else 0.0
        x[h] = (synth.draw_tokens_np(c.F_k, n_tok, rng).astype(np.float64) + off).astype(np.float16)
    xt = torch.as_tensor(x.view(np.int16), device="cuda").view(torch.float16)
    cov = torch.empty((H, 128, 128), dtype=torch.float32, device="cuda")
    kvc.kvc_covariance(xt, n_tok, cov, centered)
    torch.cuda.synchronize()
    got = cov.cpu().numpy()
    worst = 0.0
    for h in range(H):
        xf = x[h].astype(np.float64)
        ref = calib.sample_covariance(xf) if centered else (xf.T @ xf) / n_tok
        e = np.max(np.abs(got[h] - ref)) / np.max(np.abs(ref))
        worst = max(worst, e)
        assert e <= 1e-4, (h, e)
    log(f"[covariance n={n_tok} centred={centered}] max normwise error {worst:.1e}")


def test_device_calibration_tables_match_oracle(covs8b):
    w, covs = covs8b
    gst = pipeline.calibrate(covs, "cuda")
    ost = stats_from_covs(covs)
    res = {}
    for name, st in (("gpu", gst), ("oracle", ost)):
        lam = np.stack([s.lam_k for s in st])
        sq = np.stack([s.sigma2_q for s in st])
        res[name] = oa.allocate(lam, sq, oa.AllocOpts(bpd=w.bpd))
    a, b = res["gpu"], res["oracle"]
    same = np.mean((a["r"] == b["r"]) & (a["b"] == b["b"]))
    # both allocations scored with the oracle's weights
    def total(al):
        t = 0.0
        for h, s in enumerate(ost):
            wv = oa.kl_weights(s.lam_k, s.sigma2_q)
            ws = [wv[i] for i in oa.importance_order(wv)]
            t += oa.distortion(ws, int(al["r"][h]), int(al["b"][h]))
        return t
    ta, tb = total(a), total(b)
    log(f"[calibration chain] identical (r, b) on {same:.1%} of {len(covs)} heads; total D {ta:.6e} vs {tb:.6e}")
    assert same >= 0.9
    assert abs(ta - tb) <= 1e-3 * tb


@pytest.mark.parametrize("H,n_tok,centered", [(1, 1, True), (9, 63, True), (17, 64, False), (3, 513, True), (8, 1100, False)])
def test_covariance_chunk_edges(H, n_tok, centered):
    # heads not a multiple of eight, tokens around the 64-token chunks and the 512 of one turn of the wavefronts;
    # fp32 sums of n_tok exact products (n_tok 2^-24 of the sum of magnitudes) and the mean's rounding
    rng = np.random.default_rng(H * 1000 + n_tok)
    x = (rng.standard_normal((H, n_tok + 2, 128)) + 0.25 * rng.standard_normal((H, 1, 128))).astype(np.float16)
    cov = torch.full((H, 128, 128), np.nan, dtype=torch.float32, device="cuda")
    kvc.kvc_covariance(torch.as_tensor(x.view(np.int16), device="cuda").view(torch.float16), n_tok, cov, centered)
    torch.cuda.synchronize()
    got = cov.cpu().numpy().astype(np.float64)
    for h in range(H):
        X = x[h, :n_tok].astype(np.float64)
        ref, mag = X.T @ X / n_tok, np.abs(X).T @ np.abs(X) / n_tok
        if centered:
            ref, mag = ref - np.outer(X.mean(0), X.mean(0)), mag + np.outer(np.abs(X).mean(0), np.abs(X).mean(0))
        assert np.all(np.abs(got[h] - ref) <= (n_tok + 8) * 2.0 ** -24 * mag), h
        assert np.array_equal(got[h], got[h].T), h


@pytest.mark.parametrize("H,n_tok,centered", [(88, 1, False), (81, 256, True), (88, 257, True), (128, 127, True), (200, 384, False),
                                              (256, 129, True), (256, 512, True), (256, 513, True), (600, 800, True), (600, 801, False)])
def test_covariance_short_runs_of_many_heads(H, n_tok, centered):
    # both sides of the lines between a block per head and three; every sixteenth head is checked, the bound as above
    rng = np.random.default_rng(H * 1000 + n_tok)
    x = (rng.standard_normal((H, n_tok, 128), dtype=np.float32) + 0.25 * rng.standard_normal((H, 1, 128), dtype=np.float32)).astype(np.float16)
    cov = torch.full((H, 128, 128), np.nan, dtype=torch.float32, device="cuda")
    kvc.kvc_covariance(torch.as_tensor(x.view(np.int16), device="cuda").view(torch.float16), n_tok, cov, centered)
    torch.cuda.synchronize()
    got = cov.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    for h in sorted(set(range(0, H, 16)) | {H - 1}):
        X = x[h].astype(np.float64)
        ref, mag = X.T @ X / n_tok, np.abs(X).T @ np.abs(X) / n_tok
        if centered:
            ref, mag = ref - np.outer(X.mean(0), X.mean(0)), mag + np.outer(np.abs(X).mean(0), np.abs(X).mean(0))
        assert np.all(np.abs(got[h] - ref) <= (n_tok + 8) * 2.0 ** -24 * mag), h
