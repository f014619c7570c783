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
    off = got != codes
    if off.any():
        # another last bit of the quotient than the division's may only show where the value is a half
        with np.errstate(all="ignore"):
            yd = (S.astype(np.float64) * iq[None, :, :, None]) / (r[..., None].astype(np.float64) * c[:, :, None, :])
        assert np.abs(np.abs(yd[off] - np.floor(yd[off])) - 0.5).max() < 1e-5, np.argwhere(off)[:5]
    assert np.array_equal(gr.cpu().numpy(), r) and np.array_equal(gcol.cpu().numpy(), c)
    want_p = np.where(integer, np.float16(0), half).view(np.int16)
    nan = np.isnan(np.where(integer, np.float16(0), half))
    assert np.array_equal(gp.cpu().numpy()[~nan], want_p[~nan])
    with np.errstate(all="ignore"):
        want = np.where(integer, (r[..., None] * c[:, :, None, :]) * (got.astype(np.float32) / iq[None, :, :, None]),
                        half.astype(np.float32))
    assert np.array_equal(deq.cpu().numpy(), want, equal_nan=True)
