"""The binding's native call path against its general one: the same results for
everything either accepts, and what the native path declines (another container,
number or index type, another dtype, a strided tensor, a CPU tensor) is accepted
or refused by the general path as before."""
import numpy as np
import pytest
import torch

import test_parity_gpu as parity

pytestmark = pytest.mark.gpu

if torch.cuda.device_count() > 0:
    import paper_1906_05936_amd as lsgd
    from paper_1906_05936_amd import _lib
else:
    lsgd = _lib = None

DEV = parity.DEV
GOW = [0, 0, 1, 1]


def state(n=1003):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    new = lambda: torch.randn(n, device=DEV, generator=gen)
    return new(), new(), [new() for _ in range(4)], [torch.zeros(n, device=DEV) for _ in range(2)]


class Declined:
    """_marshal with every call declined."""

    def __getattr__(self, name):
        return lambda *a: None


def test_extension_is_loaded():
    """The native path is there where the library was built."""
    assert _lib._marshal is not None


def test_without_the_extension(monkeypatch):
    p, m, g, r = state()
    lsgd.step(p, m, g, GOW, 2, 0.1, 0.9, 1e-4, r)
    want = [p, m] + r
    monkeypatch.setattr(_lib, "_marshal", None)
    p, m, g, r = state()
    lsgd.step(p, m, g, GOW, 2, 0.1, 0.9, 1e-4, r)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip([p, m] + r, want))


FORMS = {
    "lists": lambda p, m, g, r: dict(),
    "tuples": lambda p, m, g, r: dict(grads=tuple(g), gow=tuple(GOW), replicas=tuple(r)),
    "parameter": lambda p, m, g, r: dict(p=torch.nn.Parameter(p)),
    "two-dimensional": lambda p, m, g, r: dict(p=p[:1000].view(10, 100), m=m[:1000].view(10, 100), grads=[x[:1000] for x in g],
                                               replicas=[x[:1000] for x in r]),
    "numpy indices": lambda p, m, g, r: dict(gow=np.array(GOW)),
    "integer rate": lambda p, m, g, r: dict(lr=1),
    "numpy rate": lambda p, m, g, r: dict(lr=np.float64(0.25)),
    "device rate": lambda p, m, g, r: dict(lr_device=torch.full((1,), 0.5, device=DEV)),
    "stream": lambda p, m, g, r: dict(stream=torch.cuda.Stream()),
}


class Elsewhere(torch.Tensor):
    """A tensor subclass whose elements are those of another tensor."""

    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        if func is torch.Tensor.data_ptr:
            return args[0].real_one.data_ptr()
        return super().__torch_function__(func, types, args, kwargs or {})


def test_subclass_answers_for_its_address():
    """A tensor subclass with __torch_function__ is read through it, whichever
    argument it is."""
    for name in ("p", "m", "g", "r"):
        p, m, g, r = state()
        want = [x.clone() for x in [p, m] + r]
        lsgd.step(want[0], want[1], g, GOW, 2, 0.1, 0.9, 1e-4, want[2:])
        a = dict(p=p, m=m, g=list(g), r=list(r))
        real = a[name] if name in "pm" else a[name][0]
        outer = torch.zeros_like(real).as_subclass(Elsewhere)
        outer.real_one = real
        if name in "pm":
            a[name] = outer
        else:
            a[name][0] = outer
        lsgd.step(a["p"], a["m"], a["g"], GOW, 2, 0.1, 0.9, 1e-4, a["r"])
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip([p, m] + r, want)), name
        assert not outer.as_subclass(torch.Tensor).any()


@pytest.mark.parametrize("form", FORMS)
def test_step_forms_agree(form, monkeypatch):
    got = []
    for native in (True, False):
        if not native:
            monkeypatch.setattr(_lib, "_marshal", Declined())
        p, m, g, r = state()
        a = dict(p=p, m=m, grads=g, gow=GOW, lr=0.1, replicas=r)
        with torch.no_grad():
            a.update(FORMS[form](p, m, g, r))
            torch.cuda.synchronize()
            lsgd.step(a["p"], a["m"], a["grads"], a["gow"], 2, a["lr"], 0.9, 1e-4, a["replicas"],
                      stream=a.get("stream"), lr_device=a.get("lr_device"))
            torch.cuda.synchronize()
        got.append([x.clone() for x in [p, m] + r])
    assert all(torch.equal(x, y) for x, y in zip(*got))
    assert not torch.equal(got[0][0], state()[0])


def bad_calls():
    p, m, g, r = state()
    wide = torch.zeros(2006, device=DEV)[::2]
    return [
        (TypeError, lambda: lsgd.step(p.double(), m, g, GOW, 2, 0.1, 0.9, 0.0)),
        (TypeError, lambda: lsgd.step(p, m, g[:3] + [g[3].bfloat16()], GOW, 2, 0.1, 0.9, 0.0)),
        (ValueError, lambda: lsgd.step(p, wide, g, GOW, 2, 0.1, 0.9, 0.0)),
        (ValueError, lambda: lsgd.step(p, m, g, GOW, 2, 0.1, 0.9, 0.0, [r[0][:-1]])),
        (ValueError, lambda: lsgd.step(p, m, g[:3] + [g[3].cpu()], GOW, 2, 0.1, 0.9, 0.0)),
        (ValueError, lambda: lsgd.step(p.cpu(), m, g, GOW, 2, 0.1, 0.9, 0.0)),
        (ValueError, lambda: lsgd.step(p, m, g, GOW, 2, 0.1, 0.9, 0.0, reduction="sum")),
        (_lib.LsgdError, lambda: lsgd.step(p, m, g, [0, 0, 0, 1], 2, 0.1, 0.9, 0.0)),
        (_lib.LsgdError, lambda: lsgd.step(p, p, g, GOW, 2, 0.1, 0.9, 0.0)),
        (_lib.LsgdError, lambda: lsgd.step(p[1:1001], m[:1000], [x[:1000] for x in g], GOW, 2, 0.1, 0.9, 0.0)),
        (ValueError, lambda: lsgd.group_mean(g, GOW, 2, r[:1])),
        (TypeError, lambda: lsgd.group_mean(g, GOW, 2, [x.bfloat16() for x in r])),
        (TypeError, lambda: lsgd.global_mean(r, m.bfloat16())),
        (ValueError, lambda: lsgd.sgd_step(p, m, g[0][:-1], 0.1, 0.9, 0.0)),
        (TypeError, lambda: lsgd.copy_out(p, [r[0].half()])),
    ]


@pytest.mark.parametrize("k", range(15))
def test_refusals_agree(k, monkeypatch):
    kind, call = bad_calls()[k]
    texts = []
    for native in (True, False):
        if not native:
            monkeypatch.setattr(_lib, "_marshal", Declined())
        with pytest.raises(kind) as e:
            call()
        texts.append(str(e.value))
    assert texts[0] == texts[1]
