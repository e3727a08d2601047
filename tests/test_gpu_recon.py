"""kvc_reconstruct where its tiling can go wrong: ranks around the matrix steps (one or two K-steps of 64
coordinates, with and without a tail group, whole and partial value N-tiles), token ranges that start and
end inside tiles or span many runs of tiles, and an output that is not 16-byte aligned. The reference
dequantizes the oracle's own codes in fp64; 128 exact products summed in fp32 and one rounding by the step
stay within 2^-16 of the largest entry."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oatt
from oracle import native as onat
from paper_2609_24298_amd import kvc

pytestmark = pytest.mark.gpu

CASES = [(r, b) for r in (2, 16, 30, 62, 64, 66, 80, 112, 126, 128) for b in (1, 2, 3, 4, 7, 8)]


@pytest.mark.parametrize("side", [kvc.SIDE_K, kvc.SIDE_V])
@pytest.mark.parametrize("t0,n,shift", [(0, 1, 0), (63, 2, 0), (37, 171, 1), (0, 320, 0)])
def test_reconstruct_ranges(side, t0, n, shift):
    rng = np.random.default_rng(3)
    Ps, ds = [], []
    for r, b in CASES:
        Q, _ = np.linalg.qr(rng.standard_normal((128, 128)))
        Ps.append(Q[:r].astype(np.float16).view(np.uint16))
        ds.append(np.float32(1.9 / 2 ** b))
    offs = np.concatenate([[0], np.cumsum([p.size for p in Ps])[:-1]]).astype(np.int64)
    S = kvc.Side(side, [c[0] for c in CASES], [c[1] for c in CASES], np.array(ds, np.float32),
                 np.concatenate([p.reshape(-1) for p in Ps]), offs, 320)
    x = rng.standard_normal((len(CASES), 320, 128)).astype(np.float16)
    kvc.kvc_encode(S, torch.as_tensor(x.view(np.int16), device="cuda").view(torch.float16), 0, 320)
    buf = torch.full((len(CASES) * n * 128 + 8,), np.nan, dtype=torch.float32, device="cuda")
    out = buf[shift:shift + len(CASES) * n * 128]
    kvc.kvc_reconstruct(S, t0, n, out)
    torch.cuda.synchronize()
    assert torch.isnan(buf[:shift]).all() and torch.isnan(buf[shift + out.numel():]).all()
    got = out.cpu().numpy().reshape(len(CASES), n, 128)
    for u, (r, b) in enumerate(CASES):
        codes = onat.encode_codes(Ps[u], float(ds[u]), b, x[u, t0:t0 + n].view(np.uint16))
        ref = oatt.reconstruct(codes, Ps[u], float(ds[u]), b)
        assert np.max(np.abs(got[u] - ref)) <= 2.0 ** -16 * np.max(np.abs(ref)), (r, b)


@pytest.mark.parametrize("side", [kvc.SIDE_K, kvc.SIDE_V])
def test_reconstruct_basis_at_any_element(side):
    # bases that start at odd elements of the arena reconstruct what aligned ones do, bit for bit
    rng = np.random.default_rng(5)
    ranks, b, n = (2, 30, 64, 66, 128), 3, 70
    Ps = [np.linalg.qr(rng.standard_normal((128, 128)))[0][:r].astype(np.float16).view(np.uint16).reshape(-1) for r in ranks]
    x = torch.as_tensor(rng.standard_normal((len(ranks), n, 128)).astype(np.float16).view(np.int16), device="cuda").view(torch.float16)
    got, codes = [], None
    for gap in (0, 1, 3):
        offs = np.array([gap * (u + 1) + sum(p.size for p in Ps[:u]) for u in range(len(ranks))], dtype=np.int64)
        flat = np.full(int(offs[-1]) + Ps[-1].size, 0x7e00, dtype=np.uint16)
        for o, p in zip(offs, Ps):
            flat[o:o + p.size] = p
        S = kvc.Side(side, ranks, [b] * len(ranks), np.full(len(ranks), 0.4, np.float32), flat, offs, n, codes=codes)
        if codes is None:
            kvc.kvc_encode(S, x, 0, n)
            codes = S.codes
        out = torch.full((len(ranks), n, 128), np.nan, dtype=torch.float32, device="cuda")
        kvc.kvc_reconstruct(S, 0, n, out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
