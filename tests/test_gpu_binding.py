"""The binding's native argument checks: they make every call of plain
arguments; arguments that are not plainly what a call takes reach the Python
checks (which raise, or take them), streams are honoured in every form, and a
closed pool is refused."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2609_38169_amd import stepq

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
B, H, DK, DV = 2, 2, 16, 64


def _pool():
    pool = stepq.Pool(3, H, H, DK, DV, np.full((H, DK), 8, np.uint8), device=DEV)
    ids = torch.arange(3, dtype=torch.int32, device=DEV)
    g = torch.Generator(device=DEV).manual_seed(1)
    S = torch.randn((3, H, DK, DV), generator=g, device=DEV)
    r, c = stepq.stepq_setup_fit(S.cpu())
    pool.load(ids, S, torch.from_numpy(r).to(DEV), torch.from_numpy(c).to(DEV))
    return pool


def _args():
    g = torch.Generator(device=DEV).manual_seed(2)
    rnd = lambda *s: torch.rand(s, generator=g, device=DEV)
    return dict(slot_ids=torch.tensor([2, 0], dtype=torch.int32, device=DEV), q=rnd(B, H, DK), k=rnd(B, H, DK),
                v=rnd(B, H, DV), alpha=rnd(B, H), beta=rnd(B, H), o=torch.zeros((B, H, DV), device=DEV))


BAD = {
    "cpu q": (ValueError, lambda a: a.update(q=a["q"].cpu())),
    "half q": (TypeError, lambda a: a.update(q=a["q"].half())),
    "bf16 k": (TypeError, lambda a: a.update(k=a["k"].bfloat16())),
    "short v": (ValueError, lambda a: a.update(v=a["v"][..., :32].contiguous())),
    "strided k": (ValueError, lambda a: a.update(k=a["k"].repeat(1, 1, 2)[..., ::2])),
    "kda gate": (ValueError, lambda a: a.update(alpha=a["alpha"][..., None].expand(B, H, DK).contiguous())),
    "int64 ids": (TypeError, lambda a: a.update(slot_ids=a["slot_ids"].long())),
    "2-d ids": (ValueError, lambda a: a.update(slot_ids=a["slot_ids"][None])),
    "numpy beta": (TypeError, lambda a: a.update(beta=a["beta"].cpu().numpy())),
    "too many slots": (stepq.StepqError, lambda a: a.update({k: torch.cat([v, v]) for k, v in a.items()})),
}


@pytest.mark.parametrize("what", list(BAD))
def test_bad_arguments_raise(what):
    pool, a = _pool(), _args()
    before = pool.memory.clone()
    err, spoil = BAD[what]
    spoil(a)
    with pytest.raises(err):
        pool.step(**a)
    assert torch.equal(before, pool.memory)


class Subclass(torch.Tensor):
    """A tensor subclass: the native checks leave it to the Python ones."""


def _calls(pool, a, wrap):
    """(name, what the native module is called with, the public call) of every
    device call on copies of the same inputs; wrap changes one tensor each."""
    g = torch.Generator(device=DEV).manual_seed(3)
    rnd = lambda *s: torch.rand(s, generator=g, device=DEV)
    gate, o = rnd(B, H, DK), a["o"]
    ids = a["slot_ids"]
    act = [a["q"], a["k"], a["v"]]
    S, r, c = rnd(B, H, DK, DV), rnd(B, H, DK) + 0.5, rnd(B, H, DV) + 0.5
    codes = torch.zeros((B, H, DK, DV), dtype=torch.int8, device=DEV)
    piv = torch.zeros((B, H, DK, DV), dtype=torch.int16, device=DEV)
    out = torch.zeros((B, H, DK, DV), device=DEV)
    n, P = stepq._native, pool._plain
    step = lambda flags, gt: (P, wrap(ids), *act, gt, a["beta"], o, None, flags)
    KDA, REFIT, ABSMAX = stepq.STEPQ_STEP_KDA_GATE, stepq.STEPQ_STEP_REFIT, stepq.STEPQ_STEP_ROW_ABSMAX
    return [
        ("load", n.scaled, (0, P, wrap(ids), S, r, c, None), lambda: pool.load(wrap(ids), S, r, c)),
        ("step", n.decode, step(0, a["alpha"]), lambda: pool.step(wrap(ids), *act, a["alpha"], a["beta"], o)),
        ("step_kda", n.decode, step(KDA, gate), lambda: pool.step_kda(wrap(ids), *act, gate, a["beta"], o)),
        ("refit", n.decode, step(REFIT, a["alpha"]),
         lambda: pool.step(wrap(ids), *act, a["alpha"], a["beta"], o, refit=True)),
        ("row absmax", n.decode, step(KDA | ABSMAX, gate),
         lambda: pool.step_kda(wrap(ids), *act, gate, a["beta"], o, refit="row_absmax")),
        ("export", n.scaled, (2, P, wrap(ids), codes, r, c, None), lambda: pool.export(wrap(ids), codes, r, c)),
        ("export_pivots", n.tiles, (1, P, wrap(ids), piv, None), lambda: pool.export_pivots(wrap(ids), piv)),
        ("dequant", n.tiles, (0, P, wrap(ids), out, None), lambda: pool.dequant(wrap(ids), out)),
        ("import", n.scaled, (1, P, wrap(ids), codes, r, c, None), lambda: pool.import_(wrap(ids), codes, r, c)),
        ("import_pivots", n.tiles, (2, P, wrap(ids), piv, None), lambda: pool.import_pivots(wrap(ids), piv)),
    ], (o, codes, r, c, piv, out)


def test_native_checks_take_plain_calls_and_leave_the_rest():
    """Every device call of plain tensors is made by the native module (status
    0); with a tensor subclass the module makes none (-1), and the Python
    checks give the same bytes."""
    results = []
    for wrap, status in ((lambda t: t, 0), (lambda t: t.as_subclass(Subclass), -1)):
        pool, a = _pool(), _args()
        calls, outs = _calls(pool, a, wrap)
        assert type(wrap(a["slot_ids"])) is (torch.Tensor if status == 0 else Subclass)
        image = pool.memory.clone()
        for name, fn, args, public in calls:
            assert fn(*args) == status, name
            pool.memory.copy_(image)
            public()
            image = pool.memory.clone()
        torch.cuda.synchronize()
        results.append([image] + [t.clone() for t in outs])
    for x, y in zip(*results):
        assert torch.equal(x, y)


def test_checks_in_python_where_the_module_is_not_built(monkeypatch):
    """A pool of a package built without the module says so once and gives the
    same bytes through the Python checks."""
    results = []
    for built in (True, False):
        if not built:
            monkeypatch.setattr(stepq, "_native", None)
            exists = stepq.os.path.exists
            monkeypatch.setattr(stepq.os.path, "exists", lambda p: not str(p).endswith("_stepq_args.so") and exists(p))
            with pytest.warns(UserWarning, match="_stepq_args"):
                pool = _pool()
        else:
            pool = _pool()
        a = _args()
        calls, outs = _calls(pool, a, lambda t: t)
        for name, fn, args, public in calls:
            assert built or fn(*args) == -1, name
            public()
        torch.cuda.synchronize()
        results.append([pool.memory.clone()] + [t.clone() for t in outs])
    for x, y in zip(*results):
        assert torch.equal(x, y)


def test_stream_forms_agree():
    """The default, object and integer streams, and a Parameter (a plain tensor
    to the native checks), give one result."""
    side = torch.cuda.Stream()
    forms = [None, side, side.cuda_stream, "parameter", "with"]
    images = []
    for f in forms:
        pool, a = _pool(), _args()
        torch.cuda.synchronize()
        if f == "parameter":
            a["q"] = torch.nn.Parameter(a["q"])
            pool.step(**a)
        elif f == "with":
            with torch.cuda.stream(side):
                pool.step(**a)
        else:
            pool.step(**a, stream=f)
        torch.cuda.synchronize()
        images.append((pool.memory.clone(), a["o"].clone()))
    for m, o in images[1:]:
        assert torch.equal(m, images[0][0]) and torch.equal(o, images[0][1])


def test_closed_pool_is_refused():
    pool, a = _pool(), _args()
    pool.close()
    with pytest.raises(stepq.StepqError):
        pool.step(**a)
    with pytest.raises(stepq.StepqError):
        pool.dequant(a["slot_ids"], torch.empty((B, H, DK, DV), device=DEV))


def test_foreign_stream_objects_are_refused():
    """Only torch's streams and integers name a stream: an object that merely
    has an attribute cuda_stream goes through int(), which raises."""
    class Foreign:
        cuda_stream = 0

    pool, a = _pool(), _args()
    before = pool.memory.clone()
    with pytest.raises(TypeError):
        pool.step(**a, stream=Foreign())
    with pytest.raises(TypeError):
        pool.dequant(a["slot_ids"], torch.empty((B, H, DK, DV), device=DEV), stream=Foreign())
    assert torch.equal(before, pool.memory)


def test_default_stream_is_the_current_devices(monkeypatch):
    """Without a stream the calls go to torch's current stream, that of the
    current device, whichever device the pool is on."""
    pool, a = _pool(), _args()
    asked = []
    raw = torch._C._cuda_getCurrentRawStream

    def query(device):
        asked.append(device)
        return raw(0)

    @ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(ctypes.c_int))
    def other_device(out):
        out[0] = 5
        return 0

    class Library:
        hipGetDevice = other_device
        __getattr__ = lambda self, name: getattr(real, name)

    real = stepq.lib()
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", query)
    monkeypatch.setattr(stepq, "_lib", Library())
    monkeypatch.setattr(stepq, "_native", None)
    stepq.native()
    try:
        args = [a[k] for k in ("slot_ids", "q", "k", "v", "alpha", "beta", "o")]
        assert stepq._native.decode(pool._plain, *args, None, 0) == 0
        assert asked == [5]
    finally:
        monkeypatch.undo()
        stepq._native = None
        stepq.native()
