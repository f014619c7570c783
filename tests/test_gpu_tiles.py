"""GPU whole-tile operations at their edges: buffers aligned to one element
only, every width with empty slots and FP16 rows, scales whose products leave
the normal range, and infinite and NaN states.  Expected bytes are the plain
fp32 formulas of the boundary pack (IEEE division, rounding to even) and its
inverse in numpy."""
import numpy as np
import pytest
import torch

from paper_2609_38169_amd import stepq

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _odd(shape, dtype):
    """A contiguous tensor whose storage starts one element past an aligned address."""
    n = int(np.prod(shape))
    return torch.zeros(n + 1, dtype=dtype, device=DEV)[1:].view(shape)


def _put(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    out = _odd(a.shape, t.dtype)
    out.copy_(t)
    return out


@pytest.mark.parametrize("levels", [0, 1])
@pytest.mark.parametrize("dk,dv", [(128, 128), (77, 128), (37, 64), (1, 64)])
def test_tile_ops_plain_formulas(dk, dv, levels):
    print(f"tile ops dk={dk} dv={dv} levels={levels}", flush=True)
    rng = np.random.default_rng(dk + dv + levels)
    Hv, n = 4, 3
    bits = np.stack([rng.choice([2, 4, 8], dk), np.full(dk, 8), rng.choice([4, 16], dk, p=[.8, .2]),
                     rng.choice([2, 16], dk, p=[.9, .1])]).astype(np.uint8)
    S = (rng.standard_normal((n, Hv, dk, dv)) * 0.05).astype(np.float32)
    S[0, 0, 0, :4] = [np.inf, -np.inf, np.nan, 0.0]
    S[1, 1, 0, :4] = [3e38, -3e38, 1e-40, -0.0]
    r = np.exp(0.3 * rng.standard_normal((n, Hv, dk))).astype(np.float32) * 0.2
    c = np.exp(0.3 * rng.standard_normal((n, Hv, dv))).astype(np.float32)
    r[2, :, 0], c[2, :, 1] = 1e-25, 1e25          # far from each other: products in and out of range
    r[2, :, -1], c[2, :, 2] = 1e25, 1e-30
    qb = np.float32(2) ** (bits.astype(np.float32) - 1) - 1
    iq = (np.float32(2) ** (bits.astype(np.float32) - 8) if levels else qb).astype(np.float32)
    with np.errstate(all="ignore"):
        y = np.rint((S * iq[None, :, :, None]) / (r[..., None] * c[:, :, None, :])).astype(np.float32)
    q = qb[None, :, :, None]
    y = np.where(np.isnan(y), -q, np.clip(y, -q, q))
    integer = (bits != 16)[None, :, :, None]
    codes = np.where(integer, y, 0).astype(np.int8)
    with np.errstate(all="ignore"):
        half = S.astype(np.float16)

    pool = stepq.Pool(n, Hv, Hv, dk, dv, bits, device=DEV, levels=levels)
    pool.memory.fill_(0x5A)
    ids = torch.tensor([2, 0, 1], dtype=torch.int32, device=DEV)
    pool.load(ids, _put(S), _put(r), _put(c))
    gc, gr, gcol, gp = (_odd((n, Hv, dk, dv), torch.int8), _odd((n, Hv, dk), torch.float32),
                        _odd((n, Hv, dv), torch.float32), _odd((n, Hv, dk, dv), torch.int16))
    pool.export(ids, gc, gr, gcol)
    pool.export_pivots(ids, gp)
    deq = _odd((n, Hv, dk, dv), torch.float32)
    pool.dequant(ids, deq)
    image = pool.memory.clone()
    # the saved form packs to the same image, padding included
    pool.memory.fill_(0xA5)
    pool.import_(ids, gc, gr, gcol)
    pool.import_pivots(ids, gp)
    torch.cuda.synchronize()
    assert torch.equal(image, pool.memory)
    got = gc.cpu().numpy()
    assert np.array_equal(got, codes), np.argwhere(got != codes)[:5]
    assert np.array_equal(gr.cpu().numpy(), r) and np.array_equal(gcol.cpu().numpy(), c)
    want_p = np.where(integer, np.float16(0), half).view(np.int16)
    nan = np.isnan(np.where(integer, np.float16(0), half))
    assert np.array_equal(gp.cpu().numpy()[~nan], want_p[~nan])
    with np.errstate(all="ignore"):
        want = np.where(integer, (r[..., None] * c[:, :, None, :]) * (got.astype(np.float32) / iq[None, :, :, None]),
                        half.astype(np.float32))
    assert np.array_equal(deq.cpu().numpy(), want, equal_nan=True)


def _hard_quotients():
    """(num, r, c), r c = den exactly, of 24 significant bits, whose quotient num / den lies within 2^-42 of the
    midpoint of a half code and the fp32 value beside it, so that a quotient with
    one wrong last bit gives another code.  With the midpoint M / 2^s, M odd of 25
    bits, den = d / M mod 2^t makes den M = num 2^t + d."""
    out = []
    for m in range(127):
        for side in (-1, 1):
            h = np.float32(m + 0.5)
            beside = np.nextafter(h, np.float32(side * 1000))
            M, s = (float(h) + float(beside)) / 2, 0
            while M < 2 ** 24 or M != int(M):
                M, s = M * 2, s + 1
            M = int(M)
            for t in (24, 25, 26):
                inv = pow(M, -1, 2 ** t)
                for d in [x for a in range(1, 33) for x in (-a, a)]:
                    den = d * inv % 2 ** t
                    num = (den * M - d) >> t
                    f = [f for f in (3, 5, 7, 11, 13, 17, 19) if den % f == 0]
                    if 2 ** 23 <= den < 2 ** 24 and 0 < num < 2 ** 24 and f:
                        out.append((num * 2.0 ** (t - s), float(den // f[-1]), float(f[-1])))
    return np.array(out)


def test_pack_rounds_the_divisions_quotient():
    """The codes are those of the correctly rounded quotient, also where the
    exact one is as close to the rounding boundary as 24-bit operands allow."""
    hard = _hard_quotients()
    dk = dv = 128
    rows = []
    for f in np.unique(hard[:, 2]):
        x = hard[hard[:, 2] == f]
        rows += [x[i:i + dk] for i in range(0, len(x) - dk + 1, dk)]
    hard = np.stack(rows)[:, None]                                 # [n][1][dk][3], one c factor per tile
    n = len(hard)
    e = np.exp2(np.arange(dv) // 2 % 16 - 8.0) * np.where(np.arange(dv) % 2, -1.0, 1.0)
    r = (hard[..., 1] * 2.0 ** -24).astype(np.float32)
    c = (hard[:, :, :1, 2] * np.abs(e)).astype(np.float32)
    S = ((hard[..., 0] * 2.0 ** -24)[..., None] * e).astype(np.float32)
    assert np.array_equal(S.astype(np.float64), (hard[..., 0] * 2.0 ** -24)[..., None] * e)
    y = S / (r[..., None] * c[:, :, None, :])
    want = np.clip(np.rint(y), -127, 127).astype(np.int8)
    print(f"hard quotients: {n * dk} rows", flush=True)
    pool = stepq.Pool(n, 1, 1, dk, dv, np.full((1, dk), 8, np.uint8), device=DEV, levels=1)
    ids = torch.arange(n, dtype=torch.int32, device=DEV)
    pool.load(ids, *(torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (S, r, c)))
    got = torch.empty((n, 1, dk, dv), dtype=torch.int8, device=DEV)
    pool.export(ids, got, torch.empty((n, 1, dk), device=DEV), torch.empty((n, 1, dv), device=DEV))
    off = got.cpu().numpy() != want
    assert not off.any(), (int(off.sum()), np.argwhere(off)[:5])
