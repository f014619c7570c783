"""GPU parity of the bodies for heads of any row-width mix (rows held in pairs
of row slots), against the fp64 oracle through the C ABI: at each compiled
pair count the splits that fill it, single rows, class boundaries inside a
round of slices, empty 4- and 2-bit slots and many FP16 pivot rows, in the two
scale modes that run these bodies and on both level normalisations.  The frozen
mode checks the generic body on the same shapes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_38169_amd import stepq
import _parity as PT

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)

# (d_k, d_v): heads as (8-bit, 4-bit, 2-bit, FP16 rows)
SHAPES = {
    "dv64-4pairs": (32, 64, [(17, 13, 2, 0), (1, 30, 1, 0), (0, 0, 32, 0), (32, 0, 0, 0), (5, 3, 20, 4)]),
    "dv64-6pairs": (96, 64, [(33, 33, 30, 0), (17, 31, 48, 0), (96, 0, 0, 0), (0, 96, 0, 0), (31, 16, 17, 32)]),
    "dv64-8pairs": (128, 64, [(33, 1, 94, 0), (17, 33, 78, 0), (65, 63, 0, 0), (1, 1, 126, 0), (50, 30, 20, 28)]),
    "dv64-1row": (1, 64, [(1, 0, 0, 0), (0, 1, 0, 0), (0, 0, 1, 0), (0, 0, 0, 1)]),
    "dv128-6pairs": (37, 128, [(9, 17, 11, 0), (1, 1, 35, 0), (37, 0, 0, 0), (0, 33, 4, 0), (7, 5, 1, 24)]),
    "dv128-8pairs": (77, 128, [(25, 31, 21, 0), (9, 17, 51, 0), (0, 77, 0, 0), (45, 0, 0, 32)]),
    "dv128-10pairs": (120, 128, [(41, 33, 46, 0), (25, 17, 78, 0), (119, 1, 0, 0), (30, 44, 26, 20)]),
    "dv128-12pairs": (128, 128, [(33, 17, 78, 0), (17, 33, 78, 0), (49, 18, 61, 0), (64, 48, 0, 16), (30, 20, 46, 32)]),
}


def _bits(rng, dk, heads):
    return np.stack([rng.permutation(np.repeat(np.array([8, 4, 2, 16], np.uint8), h)) for h in heads])


def lv_step(bits, levels):
    """The level step nu of each row: a code q stands for r c nu q."""
    b = bits.astype(np.float64)
    return 2.0 ** (8 - b) if levels == stepq.STEPQ_LEVELS_POW2 else 1.0 / (2.0 ** (b - 1) - 1)


@pytest.mark.parametrize("levels", [stepq.STEPQ_LEVELS_ABSMAX, stepq.STEPQ_LEVELS_POW2])
@pytest.mark.parametrize("mode", [False, True, "row_absmax"])
@pytest.mark.parametrize("act,kda", [("f32", False), ("bf16", True)])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_slot_bodies_one_step(shape, act, kda, mode, levels):
    dk, dv, heads = SHAPES[shape]
    lv = dict(levels=levels)
    print(f"slot bodies {shape} act={act} kda={kda} mode={mode} levels={levels}", flush=True)
    rng = np.random.default_rng(len(shape) * 1000 + dk + 7 * levels)
    bits = _bits(rng, dk, heads)
    Hv, n_slots, B = len(heads), 3, 2
    S = (rng.standard_normal((n_slots, Hv, dk, dv)) * 0.05).astype(np.float32)
    tb = np.broadcast_to(bits[None], (n_slots,) + bits.shape).reshape(-1, dk)
    r, c = oracle.fit_absmax(S.reshape(-1, dk, dv), bits=tb, **lv)
    c = np.where(c > 0, c, 1.0)
    codes, pv = oracle.quantize(S.reshape(-1, dk, dv).astype(np.float64), r, c, tb, **lv)
    pool = stepq.Pool(n_slots, Hv, Hv, dk, dv, bits, device=DEV, levels=levels)
    all_ids = torch.arange(n_slots, dtype=torch.int32, device=DEV)
    up = lambda a, *s: torch.from_numpy(np.ascontiguousarray(a.reshape(*s))).to(DEV)
    pool.import_(all_ids, up(codes, n_slots, Hv, dk, dv), up(r.astype(np.float32), n_slots, Hv, dk),
                 up(c.astype(np.float32), n_slots, Hv, dv))
    pool.import_pivots(all_ids, up(pv.view(np.int16), n_slots, Hv, dk, dv))
    wrow = np.exp(0.3 * rng.standard_normal((Hv, dk))).astype(np.float32)
    pool.set_row_weight(wrow)
    sel = rng.permutation(n_slots)[:B].astype(np.int32)
    q = rng.standard_normal((B, Hv, dk)); q /= np.linalg.norm(q, axis=-1, keepdims=True)
    k = rng.standard_normal((B, Hv, dk)); k /= np.linalg.norm(k, axis=-1, keepdims=True)
    v = rng.standard_normal((B, Hv, dv))
    gate = rng.uniform(0.5, 1.0, (B, Hv, dk)) if kda else rng.uniform(0.9, 1.0, (B, Hv))
    be = rng.uniform(0, 1, (B, Hv))
    dt = torch.bfloat16 if act == "bf16" else torch.float32
    dev_in = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dt) for a in (q, k, v, gate, be)]
    q, k, v, gate, be = (t.float().numpy().astype(np.float64) for t in dev_in)
    o = torch.empty((B, Hv, dv), dtype=torch.float32, device=DEV)
    step = pool.step_kda if kda else pool.step
    step(torch.from_numpy(sel).to(DEV), *(t.to(DEV) for t in dev_in), o, refit=mode)
    g_codes = torch.empty((n_slots, Hv, dk, dv), dtype=torch.int8, device=DEV)
    g_pv = torch.empty((n_slots, Hv, dk, dv), dtype=torch.int16, device=DEV)
    g_r, g_c = torch.empty((n_slots, Hv, dk), device=DEV), torch.empty((n_slots, Hv, dv), device=DEV)
    pool.export(all_ids, g_codes, g_r, g_c)
    pool.export_pivots(all_ids, g_pv)
    torch.cuda.synchronize()
    got = g_codes.cpu().numpy().reshape(-1, dk, dv)
    gpv = g_pv.cpu().numpy().view(np.uint16).reshape(-1, dk, dv)
    gr, gc = g_r.cpu().numpy().reshape(-1, dk), g_c.cpu().numpy().reshape(-1, dv)
    tiles = (sel[:, None] * Hv + np.arange(Hv)[None]).reshape(-1)
    args = (codes[tiles], r[tiles], c[tiles], tb[tiles], q.reshape(-1, dk), k.reshape(-1, dk), v.reshape(-1, dv),
            gate.reshape((-1, dk) if kda else (-1,)), be.reshape(-1))
    if mode is True:
        wt = np.broadcast_to(wrow[None].astype(np.float64), (B, Hv, dk)).reshape(-1, dk)
        new, rn, cn, o_ref, ex, npv = oracle.decode_step_refit(*args, w=wt, want=("y", "c_range"),
                                                               tie_window=PT.TIE_WINDOW, pv=pv[tiles], **lv)
        lo, hi = ex["c_range"]
        if dk == 1:
            # one row: c' = |X| / (r' q_b), and X = d S + beta k (v - d S k) may cancel.  Its fp32 error is at most
            # 4 roundings of the summed magnitudes, so c' may lie that far from the range, relative to |X|
            S0 = codes[tiles][:, 0] * (r[tiles] * c[tiles]) * lv_step(tb[tiles], levels)
            kk, vv, d, b = args[5], args[6], args[7].reshape(-1, 1), args[8][:, None]
            X = d * S0 + b * kk * (vv - d * S0 * kk)
            size = np.abs(d * S0) + np.abs(b * kk) * (np.abs(vv) + np.abs(d * S0 * kk))
            e = 4 * 2.0 ** -24 * size / np.maximum(np.abs(X), 1e-300)
            lo, hi = lo * np.maximum(1 - e, 0.0), hi * (1 + e)
        PT.compare_refit(got[tiles], gr[tiles], gc[tiles], new, rn, cn, ex["y"], (lo, hi), tb[tiles], shape)
        y = ex["y"]
    elif mode == "row_absmax":
        new, rn, cn, o_ref, y, npv = oracle.decode_step_rowmax(*args, want_y=True, pv=pv[tiles], **lv)
        ones = np.ones(cn.shape)
        PT.compare_refit(got[tiles], gr[tiles], gc[tiles], new, rn, cn, y, (ones, ones), tb[tiles], shape)
    else:
        new, o_ref, y, npv = oracle.decode_step(*args, want_y=True, pv=pv[tiles], **lv)
        PT.compare_codes(got[tiles], new, y, shape)
        assert np.array_equal(gr[tiles], r[tiles]) and np.array_equal(gc[tiles], c[tiles])
    PT.compare_pivots(gpv[tiles], npv, y, tb[tiles] == 16, shape)
    PT.compare_out(o.cpu().numpy().reshape(-1, dv), o_ref)
    rest = np.setdiff1d(np.arange(n_slots), sel)
    rt = (rest[:, None] * Hv + np.arange(Hv)[None]).reshape(-1)
    assert np.array_equal(got[rt], codes[rt]) and np.array_equal(gpv[rt], pv[rt])
    assert np.array_equal(gr[rt], r[rt]) and np.array_equal(gc[rt], c[rt])


@pytest.mark.parametrize("kda", [False, True])
@pytest.mark.parametrize("mixed", [False, True])
def test_row_absmax_of_rowmix_heads_in_fp32(mixed, kda):
    """The row-absmax step of heads of 8- and 4-bit rows forms its sums over
    rows in fp32, as that of any other mix does (mixed: a head with a 2-bit row
    puts all in the launch for any mix).  One row of each head has a weight 2^30
    times the others' and codes of 0, so a format scaled to the largest weight
    would leave the others few bits or none.  beta = 0: o is gate (S^T q), held
    to fp32's error bound of that sum."""
    dk = dv = 128
    heads = [(64, 60, 0, 4), (33, 95, 0, 0), (1, 127, 0, 0), (119, 1, 0, 8)]
    rng = np.random.default_rng(11)
    bits = _bits(rng, dk, heads)
    if mixed:
        bits = np.concatenate([bits, _bits(rng, dk, [(60, 67, 1, 0)])])
    B, H = 3, len(bits)
    S = rng.standard_normal((B, H, dk, dv)).astype(np.float32)
    big = np.stack([np.argmax(b != 16) for b in bits])                 # an integer row of each head
    S[:, np.arange(H), big] = 0.0
    r = np.full((B, H, dk), 0.5, np.float32)
    c = np.full((B, H, dv), 8.0, np.float32)
    q, k = (rng.uniform(0.5, 1.0, (B, H, dk)).astype(np.float32) * 2.0 ** -30 for _ in range(2))
    q[:, np.arange(H), big] = 1.0
    v = rng.standard_normal((B, H, dv)).astype(np.float32)
    gate = rng.uniform(0.5, 1.0, (B, H, dk) if kda else (B, H)).astype(np.float32)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    pool = stepq.Pool(B, H, H, dk, dv, bits, device=DEV)
    ids = torch.arange(B, dtype=torch.int32, device=DEV)
    pool.load(ids, up(S), up(r), up(c))
    old = torch.empty((B, H, dk, dv), device=DEV)
    pool.dequant(ids, old)
    o = torch.empty((B, H, dv), device=DEV)
    (pool.step_kda if kda else pool.step)(ids, *(up(a) for a in (q, k, v, gate, np.zeros((B, H), np.float32))), o,
                                          refit="row_absmax")
    torch.cuda.synchronize()
    d = gate.astype(np.float64) if kda else np.broadcast_to(gate.astype(np.float64)[..., None], (B, H, dk))
    terms = (d * q)[..., None] * old.cpu().numpy().astype(np.float64)
    off = np.abs(o.cpu().numpy() - terms.sum(2))
    # per term: 4 roundings of the weight and 2 of its scales; at most 16 + 8 + 4 additions follow
    bound = 34 * 2.0 ** -24 * np.abs(terms).sum(2)
    assert (off <= bound).all(), float((off / bound).max())


@pytest.mark.parametrize("mode", [True, "row_absmax"])
@pytest.mark.parametrize("shape", ["dv64-6pairs", "dv128-6pairs", "dv128-12pairs", "rowmix"])
def test_infinite_and_nan_values_stay_in_their_tile(shape, mode):
    """Infinite and NaN values of v, k, q or a gate make their own tile's o
    non-finite where they enter it, and change no bit of any other tile, in the
    bodies that give slots without a row zero constants."""
    dk, dv, heads = SHAPES.get(shape, (128, 128, [(64, 60, 0, 4), (33, 95, 0, 0), (1, 127, 0, 0), (119, 1, 0, 8)]))
    rng = np.random.default_rng(31)
    bits = _bits(rng, dk, heads)
    Hv, B = len(heads), 6
    S = (rng.standard_normal((B, Hv, dk, dv)) * 0.05).astype(np.float32)
    r = np.sqrt(np.abs(S).mean(-1)).astype(np.float32)
    c = np.full((B, Hv, dv), 0.3, np.float32)
    q, k = (rng.standard_normal((B, Hv, dk)).astype(np.float32) * dk ** -0.5 for _ in range(2))
    v = rng.standard_normal((B, Hv, dv)).astype(np.float32)
    gate, be = rng.uniform(0.5, 1, (B, Hv)).astype(np.float32), rng.uniform(0.2, 1, (B, Hv)).astype(np.float32)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    ids = torch.arange(B, dtype=torch.int32, device=DEV)

    def run(x):
        pool = stepq.Pool(B, Hv, Hv, dk, dv, bits, device=DEV)
        pool.memory.zero_()
        pool.load(ids, up(S), up(r), up(c))
        o = torch.empty((B, Hv, dv), device=DEV)
        pool.step(ids, *(up(t) for t in x), o, refit=mode)
        g = (torch.empty((B, Hv, dk, dv), dtype=torch.int8, device=DEV), torch.empty((B, Hv, dk), device=DEV),
             torch.empty((B, Hv, dv), device=DEV))
        piv = torch.empty((B, Hv, dk, dv), dtype=torch.int16, device=DEV)
        pool.export(ids, *g)
        pool.export_pivots(ids, piv)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (o, *g, piv)]

    clean = run((q, k, v, gate, be))
    assert np.isfinite(clean[0]).all()
    v2, k2, q2, gate2 = v.copy(), k.copy(), q.copy(), gate.copy()
    v2[1, 0, 3], v2[1, 1, 5], k2[2, 0, 0], q2[3, 1, dk - 1], gate2[4, 0] = np.inf, np.nan, np.inf, np.nan, np.nan
    hit = {(1, 0), (1, 1), (2, 0), (3, 1), (4, 0)}
    got = run((q2, k2, v2, gate2, be))
    for b in range(B):
        for h in range(Hv):
            if (b, h) in hit:
                assert not np.isfinite(got[0][b, h]).all(), (b, h)
            else:
                for x, y in zip(clean, got):
                    assert np.array_equal(x[b, h], y[b, h]), (b, h)
    # v enters column by column: o of the others is untouched
    assert np.array_equal(np.isfinite(got[0][1, 0]), np.arange(dv) != 3)
    assert np.array_equal(got[0][1, 0][np.arange(dv) != 3], clean[0][1, 0][np.arange(dv) != 3])
    # q reaches o only: the new state is that of the clean step
    for x, y in zip(clean[1:], got[1:]):
        assert np.array_equal(x[3, 1], y[3, 1])
