"""GPU: rules that choose a form of a launch by its number of tiles change no
bit.  One decode step over a batch is compared with the same step taken in
parts (launches of other lengths), on the two sides of each line."""
import numpy as np
import pytest
import torch

from paper_2609_38169_amd import stepq

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
MAPS = {"layout1": {8: 64, 4: 64}, "layout5": {2: 128}}


def _pool(bits, n_slots, Hqk, seed):
    Hv, dk = bits.shape
    pool = stepq.Pool(n_slots, Hv, Hqk, dk, 128, bits, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(seed)
    S = 0.05 * torch.randn((n_slots, Hv, dk, 128), generator=g, device=DEV)
    r = S.abs().mean(-1).sqrt_()
    top = torch.from_numpy(2.0 ** (bits.astype(np.float32) - 1) - 1).to(DEV)
    c = (S.abs() / (r * top)[..., None]).amax(2) * 1.001
    pool.memory.zero_()
    pool.load(torch.arange(n_slots, dtype=torch.int32, device=DEV), S, r.contiguous(), c.contiguous())
    return pool


def _inputs(B, Hv, Hqk, kda, bf16, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    dt = torch.bfloat16 if bf16 else torch.float32
    unit = lambda x: x / x.norm(dim=-1, keepdim=True)
    q, k = (unit(torch.randn((B, Hqk, 128), generator=g, device=DEV)).to(dt) for _ in range(2))
    v = torch.randn((B, Hv, 128), generator=g, device=DEV).to(dt)
    gate = (1 - 0.1 * torch.rand((B, Hv, 128) if kda else (B, Hv), generator=g, device=DEV)).to(dt)
    return q, k, v, gate, torch.rand((B, Hv), generator=g, device=DEV).to(dt)


def _run(pool, ids, x, kda, parts, adjacent=False, refit=False):
    step = pool.step_kda if kda else pool.step
    o = torch.empty((len(ids), pool.Hv, 128), device=DEV)
    for lo, hi in parts:
        step(ids[lo:hi], *(t[lo:hi] for t in x), o[lo:hi], adjacent=adjacent, refit=refit)
    torch.cuda.synchronize()
    return pool.memory.clone(), o


@pytest.mark.parametrize("kda,bf16", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("layout", list(MAPS))
def test_waves_of_the_columns(layout, kda, bf16):
    """Columns beside the rows (1,537 to 3,072 tiles, more than 8,192 of
    drawn slots) or on waves of their own: 48 | 49, 96 | 97 and 256 | 257
    requests x 32 heads, each also in parts of at most 48."""
    Hv = 32
    rng = np.random.default_rng(7)
    row = np.concatenate([np.full(n, b, np.uint8) for b, n in MAPS[layout].items()])
    bits = np.stack([rng.permutation(row) for _ in range(Hv)])
    for B in (48, 49, 96, 97, 256, 257):
        print(f"waves of the columns {layout} kda={kda} bf16={bf16} B={B}", flush=True)
        x = _inputs(B, Hv, 16, kda, bf16, B)
        ids = torch.arange(B, dtype=torch.int32, device=DEV)
        parts = [(lo, min(B, lo + 48)) for lo in range(0, B, 48)]
        pool = _pool(bits, B, 16, B)
        start = pool.memory.clone()
        want = _run(pool, ids, x, kda, parts)
        for adjacent in (False, True):
            pool.memory.copy_(start)
            got = _run(pool, ids, x, kda, [(0, B)], adjacent)
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (B, adjacent)


@pytest.mark.parametrize("adjacent", [False, True])
@pytest.mark.parametrize("Hv", [6, 20, 32])
def test_rotation_of_combined_launches(Hv, adjacent):
    """Heads @8 and @4 in one combined launch: 4, 5 and 8 tiles a CU, and one
    request more than a residency round, each also in parts."""
    bits = np.stack([np.full(128, 8 if h % 2 else 4, np.uint8) for h in range(Hv)])
    top = 2048 // Hv
    for B in (1024 // Hv, 1024 // Hv + 1, top, top + 1):
        print(f"rotation Hv={Hv} B={B} adjacent={adjacent}", flush=True)
        x = _inputs(B, Hv, Hv // 2, False, False, B)
        ids = torch.arange(B, dtype=torch.int32, device=DEV)
        pool = _pool(bits, B, Hv // 2, B)
        start = pool.memory.clone()
        want = _run(pool, ids, x, False, [(lo, min(B, lo + 16)) for lo in range(0, B, 16)])
        pool.memory.copy_(start)
        got = _run(pool, ids, x, False, [(0, B)], adjacent)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), B
