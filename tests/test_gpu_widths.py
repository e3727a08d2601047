"""GPU parity of decode attention and reconstruction over every pair of code widths.

The allocator's tables at the measured budgets reach only part of the (b_K, b_V) plane, so this test
builds its own tables: 64 width pairs (b_K, b_V) in {1..8}^2, each on 8 units whose ranks cycle
through {2, 6, 14, 18, 64, 66, 84, 96, 126, 128} (ranks with and without a tail group of r mod 16
coordinates, one and two 64-coordinate K-steps, value N-tiles from 1 to 8). Bases are random
orthonormal rows rounded to fp16, steps scaled to each width. 512 units of 4133 tokens split into
multi-tile context chunks with a ragged last tile. One cache is decoded with every query-group size
G in {1, 2, 4, 8, 16} (the streams do not depend on G) and checked unit by unit against the oracle's
fp64 decode from its own codes; reconstruction of a token range is checked for every unit.

Queries of scale 1.5 against these keys give logits of about 1 nat standard deviation (at full key
rank): nearly flat attention, whose output (about the mean value) hardly moves when some value
fields are read from the wrong place. Every other unit therefore gets queries of scale 6 (about 4
nats): a few tokens then take most of the attention and their value fields show in the output.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oatt
from oracle import native as onat
from paper_2609_24298_amd import kvc

from test_gpu_parity import TOL, normwise
from test_gpu_rope import rope_sigma

pytestmark = pytest.mark.gpu

RANKS = (2, 6, 14, 18, 64, 66, 84, 96, 126, 128)
REPS = 8
T = 4133


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def _table():
    rows = []
    for i, (bk, bv) in enumerate((bk, bv) for bk in range(1, 9) for bv in range(1, 9)):
        for j in range(REPS):
            rows.append((RANKS[(i + j) % 10], bk, RANKS[(i + 3 * j + 5) % 10], bv))
    return rows


def _side(side, rows, rng):
    Ps, ds = [], []
    for rk, bk, rv, bv in rows:
        r, b = (rk, bk) if side == kvc.SIDE_K else (rv, bv)
        Q, _ = np.linalg.qr(rng.standard_normal((128, 128)))
        Ps.append(Q[:r].astype(np.float16).view(np.uint16))
        ds.append(np.float32(rng.uniform(0.6, 1.2) * 1.596 / 2 ** (b - 1) * 0.6))
    rs = [row[0] if side == kvc.SIDE_K else row[2] for row in rows]
    bs = [row[1] if side == kvc.SIDE_K else row[3] for row in rows]
    flat = np.concatenate([p.reshape(-1) for p in Ps])
    offs = np.concatenate([[0], np.cumsum([p.size for p in Ps])[:-1]]).astype(np.int64)
    return kvc.Side(side, rs, bs, np.array(ds, np.float32), flat, offs, T), Ps, ds


@pytest.fixture(scope="module")
def width_cache():
    rows = _table()
    rng = np.random.default_rng(31)
    K, Pk, dk = _side(kvc.SIDE_K, rows, rng)
    V, Pv, dv = _side(kvc.SIDE_V, rows, rng)
    U = len(rows)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4133)
    xk = (torch.randn((U, T, 128), generator=gen, device="cuda") * 0.6).to(torch.float16)
    xv = (torch.randn((U, T, 128), generator=gen, device="cuda") * 0.6).to(torch.float16)
    log(f"[widths] encode {U} units x {T} tokens")
    kvc.kvc_encode_kv(K, V, xk, xv, 0, T)
    torch.cuda.synchronize()
    xkb = xk.view(torch.int16).cpu().numpy().view(np.uint16)
    xvb = xv.view(torch.int16).cpu().numpy().view(np.uint16)
    codes = []
    for u, (rk, bk, rv, bv) in enumerate(rows):
        ck = onat.encode_codes(Pk[u], dk[u], bk, xkb[u])
        cv = onat.encode_codes(Pv[u], dv[u], bv, xvb[u])
        assert np.array_equal(K.unit_codes(u, T).cpu().numpy(), onat.pack(ck, rk, bk, kvc.SIDE_K)), (u, rk, bk)
        assert np.array_equal(V.unit_codes(u, T).cpu().numpy(), onat.pack(cv, rv, bv, kvc.SIDE_V)), (u, rv, bv)
        codes.append((ck, cv))
    log("[widths] streams bit-exact for every unit")
    return rows, K, V, Pk, dk, Pv, dv, codes


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
def test_decode_every_width_pair(width_cache, G):
    rows, K, V, Pk, dk, Pv, dv, codes = width_cache
    U = len(rows)
    rng = np.random.default_rng(100 + G)
    scale = np.where(np.arange(U) % 2 == 0, 1.5, 6.0)[:, None, None]
    q = (rng.standard_normal((U, G, 128)) * scale).astype(np.float16)
    qt = torch.as_tensor(q.view(np.int16), device="cuda").view(torch.float16)
    # lengths: most units attend over everything, some over ragged prefixes
    seq = np.full(U, T, dtype=np.int32)
    seq[::7] = rng.integers(1, T, size=len(seq[::7]))
    nbytes = kvc.kvc_decode_attn_workspace(K, V, G, T)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    out = torch.empty((U, G, 128), dtype=torch.float32, device="cuda")
    log(f"[widths G={G}] decode")
    kvc.kvc_decode_attn(K, V, qt, G, torch.as_tensor(seq, device="cuda"), T, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    worst = {}
    for u, (rk, bk, rv, bv) in enumerate(rows):
        ck, cv = codes[u]
        ref = oatt.decode_attention(ck, cv, Pk[u], Pv[u], dk[u], dv[u], bk, bv, q[u].view(np.uint16), int(seq[u]))
        for g in range(G):
            e = normwise(got[u, g], ref[g])
            worst[(bk, bv)] = max(worst.get((bk, bv), 0.0), e)
            assert e <= TOL, (G, u, (rk, bk, rv, bv), g, e)
    log(f"[widths G={G}] 64 width pairs, max normwise error {max(worst.values()):.2e}")


def test_reconstruct_every_width(width_cache):
    rows, K, V, Pk, dk, Pv, dv, codes = width_cache
    U = len(rows)
    t0, n = 1000, 1100
    for side, S, P, dl in ((kvc.SIDE_K, K, Pk, dk), (kvc.SIDE_V, V, Pv, dv)):
        out = torch.empty((U, n, 128), dtype=torch.float32, device="cuda")
        kvc.kvc_reconstruct(S, t0, n, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        for u, row in enumerate(rows):
            b = row[1] if side == kvc.SIDE_K else row[3]
            c = codes[u][side][t0:t0 + n]
            ref = oatt.reconstruct(c, P[u], dl[u], b)
            assert normwise(got[u], ref) <= 1e-5, (side, u, row)
        log(f"[widths] reconstruct side {'KV'[side]}: every unit within 1e-5")


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("first,units", [(0, 512), (0, 256), (256, 256)])
def test_rope_decode_every_width_pair(width_cache, G, first, units):
    # The RoPE-aware path unpacks K codes itself (whole 16-coordinate groups and the tail group). 512 units split
    # into up to four chunks (blocks of four wavefronts at eight heads), 256 units into eight (blocks of eight),
    # where two units of every width pair are checked. Bound: test_gpu_rope.
    rows, K, V, Pk, dk, Pv, dv, codes = width_cache
    base = 10000.0
    if units < len(rows):
        K, V = kvc.SideRange(K, first, units), kvc.SideRange(V, first, units)
    rng = np.random.default_rng(77)
    scale = np.where(np.arange(units) % 2 == 0, 1.5, 6.0)[:, None, None]
    q = (rng.standard_normal((units, G, 128)) * scale).astype(np.float16)
    qt = torch.as_tensor(q.view(np.int16), device="cuda").view(torch.float16)
    seq = np.full(units, T, dtype=np.int32)
    seq[::5] = rng.integers(1, T, size=len(seq[::5]))
    ws = torch.empty(kvc.kvc_decode_attn_workspace(K, V, G, T), dtype=torch.uint8, device="cuda")
    out = torch.empty((units, G, 128), dtype=torch.float32, device="cuda")
    kvc.kvc_decode_attn_rope(K, V, qt, G, torch.as_tensor(seq, device="cuda"), T, base, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    worst = 0.0
    for i in range(units):
        if units < len(rows) and i % 4 != G.bit_length() % 4:
            continue
        u, n = first + i, int(seq[i])
        rk, bk, rv, bv = rows[u]
        ck, cv = codes[u]
        args = (Pk[u], Pv[u], dk[u], dv[u], bk, bv)
        ref = oatt.decode_attention_rope(ck, cv, *args, q[i].view(np.uint16), n, base)
        lim = 8 * rope_sigma(q[i].view(np.uint16), ck[:n], cv[:n], *args, base)
        for g in range(G):
            e = np.max(np.abs(got[i, g] - ref[g])) / lim[g]
            worst = max(worst, e)
            assert e <= 1.0, (u, (rk, bk, rv, bv), g, e)
    log(f"[widths rope G={G}, units {first} to {first + units}] at most {worst:.2f} of the bound")
