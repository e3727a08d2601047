"""GPU parity of RoPE-aware decode attention (kvc_decode_attn_rope) against the oracle's fp64
decode_attention_rope: the keys' codes hold pre-RoPE keys, the kernel reconstructs them, rotates each at
its stream index and scores the rotated query. Every query-group size, ragged lengths, both common
rotary bases, one layer of the 8B-shaped 32k workload, and every pair of code widths (the 512-unit
table of test_gpu_widths).

Bound (rope_sigma): roundings of the components of query and key, carried to the output to first order. Each
component passes two splits into fp16 halves (2^-24 of it each, and the dropped product of the low halves),
three rotations (the tile's, the query's inside its block, the key's) by an angle of fp32 turns (pi / 2 2^-24, and
2^-24 each of the sine, the cosine and the two products) and the sums of the key's reconstruction
(sqrt(128) 2^-24 / 2): 3 + 3 (pi / 2 + 4) + 6 = 26 roundings of 2^-24 at most, with signs that do not line up, so
that eps = 2^-20 is beyond their standard deviation. A logit then errs by eps |q * k_t| / sqrt(d) (2-norm of the
elementwise product; the logit's own sum is shorter than that of the components' errors), a weight of the
fixed-point softmax by 2^-26 of the largest, and the output by the root of the sum of squares of what these
move. The rank-space average of the codes, whose zero lies at -1/2, is four fp32 roundings of itself (the chunks'
sums, the quotient and the half added at the end). Eight of these standard deviations are allowed. Angles of
frequencies rounded to fp32 err by up to 1e-3 at 32k, one dropped product of the split by 2^-12."""
import math
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import attention as oatt
from oracle import native as onat
from paper_2609_24298_amd import kvc, pipeline, synth

from oracle_stats import oracle_stats
from test_gpu_parity import OracleTables, normwise, x_bits

pytestmark = pytest.mark.gpu


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def rope_sigma(q_bits, ck, cv, Pk, Pv, dk, dv, bk, bv, base):
    """Standard deviation of the largest output entry of one unit's heads (per head)."""
    q = oatt.fp16_to_f64(q_bits)
    k = oatt.rope_rotate(oatt.reconstruct(ck, Pk, dk, bk), np.arange(len(ck)), base)
    z, P = oatt.dequantize(cv, float(dv), bv), oatt.fp16_to_f64(Pv)
    p = oatt.softmax(q @ k.T / math.sqrt(128))
    ds = 2.0 ** -20 * np.sqrt((q * q) @ (k * k).T) / math.sqrt(128)
    w2 = (p * ds) ** 2 + (2.0 ** -26 * p.max(axis=1, keepdims=True)) ** 2
    zbar, v = p @ z, z @ P
    o = zbar @ P
    var = w2 @ (v * v) - 2 * o * (w2 @ v) + o * o * w2.sum(axis=1, keepdims=True)  # sum_t w2 (v - o)^2
    avg = 2.0 ** -22 * (np.abs(zbar) + 0.5 * float(dv))
    return np.sqrt(np.maximum(var, 0.0) + (avg * avg) @ (P * P)).max(axis=1)


def _run(w, T, seq, base, q_scale=1.0, units=None, seed=5):
    st = oracle_stats(w, seed)
    cache = pipeline.Cache(w, seed=seed, stats=st, capacity=T)
    xk = pipeline.draw_unit_tokens(w, st, kvc.SIDE_K, T, seed, "cuda")
    xv = pipeline.draw_unit_tokens(w, st, kvc.SIDE_V, T, seed, "cuda")
    cache.encode(xk, xv, 0, T)
    rng = np.random.default_rng(seed)
    q = (rng.standard_normal((w.n_units, w.group, 128)) * q_scale).astype(np.float16)
    qt = torch.as_tensor(q.view(np.int16), device="cuda").view(torch.float16)
    ws, out = cache.decode_buffers(T)
    kvc.kvc_decode_attn_rope(cache.K, cache.V, qt, w.group, torch.as_tensor(seq, device="cuda"), T, base, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    ot = OracleTables(w, st)
    worst = share = 0.0
    for u in (range(w.n_units) if units is None else units):
        h = w.head_of_unit(u)
        n = int(seq[u])
        res = {}
        for side, x in ((kvc.SIDE_K, xk), (kvc.SIDE_V, xv)):
            r, b = ot.rb(side, h)
            P, dl = ot.basis(side, h)
            res[side] = (onat.encode_codes(P, dl, b, x_bits(x[u][:n])), P, dl, b)
        (ck, Pk, dk, bk), (cv, Pv, dv, bv) = res[kvc.SIDE_K], res[kvc.SIDE_V]
        ref = oatt.decode_attention_rope(ck, cv, Pk, Pv, dk, dv, bk, bv, q[u].view(np.uint16), n, base)
        lim = 8 * rope_sigma(q[u].view(np.uint16), ck[:n], cv[:n], Pk, Pv, dk, dv, bk, bv, base)
        for g in range(w.group):
            worst = max(worst, normwise(got[u, g], ref[g]))
            e = np.max(np.abs(got[u, g] - ref[g]))
            share = max(share, e / lim[g])
            assert e <= lim[g], (u, g, n, e, lim[g])
    return f"max normwise error {worst:.1e}, at most {share:.2f} of its bound"


@pytest.mark.parametrize("G", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("base", [10000.0, 500000.0])
def test_rope_decode_every_group_size(G, base):
    w = synth.Workload(f"rope_g{G}", 1, 4, G, 1, 2000, 2.0)
    seq = np.array([2000, 1999, 65, 1][: w.n_units], dtype=np.int32)
    worst = _run(w, w.tokens, seq, base, q_scale=3.0)
    log(f"[rope G={G} base={base:g}] {worst}")


@pytest.mark.parametrize("q_scale", [2.0, 12.0])
def test_rope_decode_one_layer_of_the_8b_workload(q_scale):
    w0 = synth.WORKLOADS["llama8b_b8_t32k_2bpd"]
    w = synth.Workload("rope_8b_l1", 1, w0.kv_heads, w0.group, w0.batch, w0.tokens, w0.bpd)
    seq = np.full(w.n_units, w.tokens, dtype=np.int32)
    worst = _run(w, w.tokens, seq, 500000.0, q_scale=q_scale, units=[0, 33, w.n_units - 1])
    log(f"[rope 8B layer, 32k, queries of scale {q_scale:g}] {worst}")
