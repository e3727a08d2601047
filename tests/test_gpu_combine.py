"""The combine of decode attention where its split can go wrong: one chunk, fewer and more chunks than a
wavefront's lanes, more chunks than one batch of weights holds (512), ragged and empty units, every group size
(one to eight heads share a block; sixteen heads are two partials items of eight) and value ranks around the
four-column reads. The workspace starts as NaN, so an accumulator that the partials did not write shows.

A block merges its chunks in passes: 64 / GB chunks for GB = 1, 2 heads and 32 / GB for 4, 8 where a call's blocks
are all resident, a quarter and half of that where they are not, and every pass but the first is covered for each
but the block of two resident heads, whose second pass starts at 33 chunks: the planner gives units that many
only from about half a million tokens on. So is a second batch of weights for one head (512 chunks); for more
heads, and where blocks are not all resident, a second batch would take millions of tokens.

Bound: the fixed-point weights of a chunk of c tiles lose at most 64 c 2^-26 of its mass, which moves the output by
at most twice that share; the limbs of the query are good to 2^-24 of its largest entry, which over 128
coordinates of these codes moves a logit by at most about 2e-5, a weight by the same share and the output by
twice that. Together 1e-4 + 2^-19 c of the largest entry."""
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


def _chunks(ws_bytes, U, G):
    """Chunks per unit that a workspace of this size was laid out for."""
    def up(n):
        return (n + 255) // 256 * 256
    return (ws_bytes - up(U * 2 * ((G + 3) // 4) * 64 * 16) - up(U * G * 16)) // (U * G * 132 * 4)


def _check(T, copies, groups, min_chunks=None):
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
            n_chunks = _chunks(ws.numel(), U, G)
            tol = 1e-4 + -(-T // (64 * n_chunks)) * 2.0 ** -19
            if min_chunks is not None:
                assert n_chunks >= min_chunks[G], (G, n_chunks)
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
                    assert e <= tol, (G, u, g, lens[u], e)
            for u in range(len(ROWS), U):
                assert np.array_equal(got[u], got[u % len(ROWS)]), (G, u)


@pytest.mark.parametrize("T", [33, 1100, 4133, CAP])
def test_combine_chunk_counts(T):
    _check(T, 1, (1, 4, 16) if T == CAP else (1, 2, 4, 8, 16))


def test_combine_shared_blocks():
    # 1536 units: blocks of two, four and eight heads, not all resident; one or two chunks
    _check(200, 512, (2, 4, 8, 16))


def test_combine_shared_blocks_resident():
    # 300 units: blocks of two, four and eight heads, a second pass for the latter two
    _check(4133, 100, (2, 4, 8), {2: 10, 4: 9, 8: 5})


def test_combine_many_blocks():
    # 1029 units: more blocks than are resident; a second pass for four heads, a third for eight
    _check(4133, 343, (1, 2, 4, 8, 16), {1: 5, 2: 5, 4: 5, 8: 5, 16: 5})


def test_combine_many_blocks_long():
    # 513 units of 33100 tokens: a second pass for one head, a third for two
    _check(CAP, 171, (1, 2), {1: 17, 2: 17})


def test_combine_basis_at_any_element():
    # the value bases start at odd elements of the arena
    rng = np.random.default_rng(23)
    T = 300
    xs = [(rng.standard_normal((len(ROWS), T, 128)) * 0.6).astype(np.float16) for _ in range(2)]
    K = _side(kvc.SIDE_K, xs[0], rng, 1)[0]
    V, Pv, dv, bv, _ = _side(kvc.SIDE_V, xs[1], rng, 1)
    offs = np.array([1, 3, 5], dtype=np.int64) + np.concatenate([[0], np.cumsum([p.size for p in Pv])[:-1]])
    flat = np.full(int(offs[-1]) + Pv[-1].size, 0x7e00, dtype=np.uint16)
    for o, p in zip(offs, Pv):
        flat[o:o + p.size] = p.reshape(-1)
    W = kvc.Side(kvc.SIDE_V, V.r_h, V.b_h, np.array(dv, np.float32), flat, offs, T, codes=V.codes)
    q = torch.as_tensor((rng.standard_normal((3, 4, 128)) * 3.0).astype(np.float16).view(np.int16), device="cuda").view(torch.float16)
    seq = torch.full((3,), T, dtype=torch.int32, device="cuda")
    ws = torch.empty(kvc.kvc_decode_attn_workspace(K, V, 4, T), dtype=torch.uint8, device="cuda")
    outs = [torch.full((3, 4, 128), np.nan, dtype=torch.float32, device="cuda") for _ in range(2)]
    for side, out in zip((V, W), outs):
        kvc.kvc_decode_attn(K, side, q, 4, seq, T, out, ws)
    torch.cuda.synchronize()
    a, b = (o.cpu().numpy() for o in outs)
    assert np.isfinite(a).all() and np.array_equal(a, b)
