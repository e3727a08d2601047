"""Bulk encode in pieces that start and end inside tiles: every piece goes through the bulk encoder (more
than four tokens), shares tiles with its neighbours and leaves their codes alone. Ranks with and without a
K tail group, with whole and short value groups, at every code width, as two kvc_encode_kv sides of one
launch; the streams equal the oracle's packing bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import native as onat
from paper_2609_24298_amd import kvc

pytestmark = pytest.mark.gpu

RANKS = (2, 14, 16, 34, 48, 64, 66, 84, 112, 126, 128)
T = 390
PIECES = [(0, 5), (5, 70), (75, 52), (127, 6), (133, 251), (384, 6)]  # inside a tile, across tiles, whole tiles


@pytest.mark.parametrize("b", range(1, 9))
def test_bulk_pieces_bit_exact(b):
    rng = np.random.default_rng(40 + b)
    sides, x, recs = [], [], []
    for side in (kvc.SIDE_K, kvc.SIDE_V):
        Ps = []
        for r in RANKS:
            Q, _ = np.linalg.qr(rng.standard_normal((128, 128)))
            Ps.append(Q[:r].astype(np.float16).view(np.uint16))
        ds = np.full(len(RANKS), 3.0 / 2 ** b, np.float32)
        offs = np.concatenate([[0], np.cumsum([p.size for p in Ps])[:-1]]).astype(np.int64)
        sides.append(kvc.Side(side, RANKS, [b] * len(RANKS), ds, np.concatenate([p.reshape(-1) for p in Ps]), offs, T))
        x.append(rng.standard_normal((len(RANKS), T, 128)).astype(np.float16))
        recs.append((Ps, ds))
    for t0, n in PIECES:
        xk, xv = (torch.as_tensor(np.ascontiguousarray(a[:, t0:t0 + n]).view(np.int16), device="cuda").view(torch.float16) for a in x)
        kvc.kvc_encode_kv(sides[0], sides[1], xk, xv, t0, n)
    torch.cuda.synchronize()
    for S, a, (Ps, ds), side in zip(sides, x, recs, (kvc.SIDE_K, kvc.SIDE_V)):
        for u, r in enumerate(RANKS):
            codes = onat.encode_codes(Ps[u], float(ds[u]), b, a[u].view(np.uint16))
            assert np.array_equal(S.unit_codes(u, T).cpu().numpy(), onat.pack(codes, r, b, side)), (side, r)


@pytest.mark.parametrize("b", [1, 3, 8])
def test_bulk_long_tokens_bit_exact(b):
    # Tokens beyond 126 000 steps have an error bound above half a step, so that every element is settled; the
    # rows after each basis are NaN bits, inside the arena.
    rng = np.random.default_rng(90 + b)
    ranks = (2, 14, 34, 66, 112, 126, 128)
    n, step = 150, np.float32(0.004)
    x = rng.standard_normal((2, len(ranks), n, 128))
    x[:, :, ::3] *= 3000.0
    x[:, :, 1::7] = np.sign(x[:, :, 1::7]) * 65504.0
    x = x.astype(np.float16)
    assert np.linalg.norm(x[:, :, ::3].astype(np.float64), axis=-1).min() > 126000 * float(step)
    for side in (kvc.SIDE_K, kvc.SIDE_V):
        Ps = [np.linalg.qr(rng.standard_normal((128, 128)))[0][:r].astype(np.float16).view(np.uint16) for r in ranks]
        flat = np.full((len(ranks), 128 + 16, 128), 0x7e00, dtype=np.uint16)
        for u, P in enumerate(Ps):
            flat[u, :P.shape[0]] = P
        S = kvc.Side(side, ranks, [b] * len(ranks), np.full(len(ranks), step, np.float32), flat.reshape(-1),
                     np.arange(len(ranks), dtype=np.int64) * 144 * 128, n)
        kvc.kvc_encode(S, torch.as_tensor(x[side].view(np.int16), device="cuda").view(torch.float16), 0, n)
        torch.cuda.synchronize()
        for u, r in enumerate(ranks):
            codes = onat.encode_codes(Ps[u], float(step), b, x[side, u].view(np.uint16))
            assert np.array_equal(S.unit_codes(u, n).cpu().numpy(), onat.pack(codes, r, b, side)), (side, r)
