"""The combine of decode attention where its split can go wrong: one chunk, fewer and more chunks than a
wavefront's lanes, more chunks than one batch of weights holds (512), ragged and empty units, every group size
(one to eight heads share a block; sixteen heads are two partials items of eight) and value ranks around the
four-column reads. The workspace starts as NaN, so an accumulator that the partials did not write shows.

Bound: chunks here are one tile, so the fixed-point weights lose at most 64 x 2^-26 of a chunk's mass; the limbs
of the query are good to 2^-24 of its largest entry, which over 128 coordinates of these codes moves a logit by
at most about 2e-5, a weight by the same share and the output by twice that: 1e-4 of the largest entry."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oatt
from oracle import native as onat
from paper_2609_24298_amd import kvc

from test_gpu_parity import normwise

pytestmark = pytest.mark.gpu

ROWS = [(64, 3, 128, 2), (34, 2, 70, 3), (128, 2, 2, 8)]  # (r_K, b_K, r_V, b_V)
CAP = 33100  # 518 tiles


def _side(side, x, rng, copies):
    Ps, ds, rs, bs = [], [], [], []
    for row in ROWS:
        r, b = row[:2] if side == kvc.SIDE_K else row[2:]
        Q, _ = np.linalg.qr(rng.standard_normal((128, 128)))
        Ps.append(Q[:r].astype(np.float16).view(np.uint16))
        ds.append(np.float32(1.9 / 2 ** b))
        rs.append(r)
        bs.append(b)
    offs = np.concatenate([[0], np.cumsum([p.size for p in Ps])[:-1]]).astype(np.int64)
    S = kvc.Side(side, rs * copies, bs * copies, np.array(ds * copies, np.float32), np.concatenate([p.reshape(-1) for p in Ps]),
                 np.tile(offs, copies), x.shape[1])
    kvc.kvc_encode(S, torch.as_tensor(x.view(np.int16), device="cuda").view(torch.float16).repeat(copies, 1, 1), 0, x.shape[1])
    codes = [onat.encode_codes(Ps[u], ds[u], bs[u], x[u].view(np.uint16)) for u in range(len(ROWS))]
    return S, Ps, ds, bs, codes


def _check(T, copies, groups):
    rng = np.random.default_rng(17)
    xs = [(rng.standard_normal((len(ROWS), T, 128)) * 0.6).astype(np.float16) for _ in range(2)]
    K, Pk, dk, bk, ck = _side(kvc.SIDE_K, xs[0], rng, copies)
    V, Pv, dv, bv, cv = _side(kvc.SIDE_V, xs[1], rng, copies)
    U = K.n_units
    for G in groups:
        q = (rng.standard_normal((U, G, 128)) * 3.0).astype(np.float16)
        q[len(ROWS):] = q[np.arange(len(ROWS), U) % len(ROWS)]
        for lens in ([T, T, T], [T // 3 + 1, 0, T]):
            seq = torch.as_tensor(np.tile(np.array(lens, np.int32), copies), device="cuda")
            ws = torch.full((kvc.kvc_decode_attn_workspace(K, V, G, T),), 255, dtype=torch.uint8, device="cuda")
            out = torch.full((U, G, 128), np.nan, dtype=torch.float32, device="cuda")
            kvc.kvc_decode_attn(K, V, torch.as_tensor(q.view(np.int16), device="cuda").view(torch.float16), G, seq, T, out, ws)
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            for u in range(len(ROWS)):
                if lens[u] == 0:
                    assert not got[u].any(), (G, u)
                    continue
                ref = oatt.decode_attention(ck[u], cv[u], Pk[u], Pv[u], dk[u], dv[u], bk[u], bv[u], q[u].view(np.uint16), lens[u])
                for g in range(G):
                    e = normwise(got[u, g], ref[g])
                    assert e <= 1e-4, (G, u, g, lens[u], e)
            for u in range(len(ROWS), U):
                assert np.array_equal(got[u], got[u % len(ROWS)]), (G, u)


@pytest.mark.parametrize("T", [33, 1100, 4133, CAP])
def test_combine_chunk_counts(T):
    _check(T, 1, (1, 4, 16) if T == CAP else (1, 2, 4, 8, 16))


def test_combine_shared_blocks():
    # 1536 units: blocks of two, four and eight heads
    _check(200, 512, (2, 4, 8, 16))
