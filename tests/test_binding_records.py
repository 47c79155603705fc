"""The step descriptors the binding packs hold, byte for byte, what ctypes gives the same fields, for
every kind of number the fields take (Python and numpy integers of any sign, 0-d tensors, numbers
beyond a field's width, any iterable of three), and refuse what ctypes refuses (no GPU needed)."""
import ctypes as C
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2301_07684_amd import sfq


PX = torch.zeros(5)


def tile(**kw):
    """A tile of no arrays (TileArrays itself takes device tensors only)."""
    t = object.__new__(sfq.TileArrays)
    for f in sfq.TileArrays.__dataclass_fields__.values():
        setattr(t, f.name, None if f.name in ("species", "px", "py", "pz") else f.default)
    t.species, t.px = 0, PX
    for k, v in kw.items():
        setattr(t, k, v)
    return t


def three(v):
    return (C.c_double * 3)(*v)


def by_fields(t):
    return sfq.Tile(species=t.species, product_set=t.product_set, n=t.n, px=t.px.data_ptr(),
                    step_offset=t.step_offset, field_mode=int(t.field_mode),
                    wave_k=three(t.wave_k), wave_pol=three(t.wave_pol),
                    wave_phase0=float(t.wave_phase0))


PRODUCTS = SimpleNamespace(counts=None, **{s: SimpleNamespace(_record=lambda: (0,) * 7)
                                           for s in ("photons", "electrons", "positrons")})


def desc(t, seed=1, step=1):
    return sfq.Handle._desc([t], seed, step, PRODUCTS, SimpleNamespace(t=None))


WHOLE = [0, 7, -1, 2 ** 63, 2 ** 64 + 5, True, np.int64(7), np.int64(-7), np.int32(-7),
         np.uint64(2 ** 63), np.uint8(255), torch.tensor(5), torch.tensor(-5)]


@pytest.mark.parametrize("value", WHOLE, ids=repr)
def test_whole_numbers(value):
    d, _keep = desc(tile(step_offset=value), seed=value, step=value)
    ref = sfq.StepDesc(seed=value, step=value)
    assert (d.seed, d.step) == (ref.seed, ref.step)
    assert bytes(d.tiles[0]) == bytes(by_fields(tile(step_offset=value)))


@pytest.mark.parametrize("field", ["species", "field_mode"])
@pytest.mark.parametrize("value", WHOLE + [2 ** 31, -2 ** 31 - 1, 2 ** 32 + 1], ids=repr)
def test_narrow_whole_numbers(field, value):
    if not isinstance(value, (int, np.integer)):
        value = int(value)
    t = tile(**{field: value})
    d, _keep = desc(t)
    assert bytes(t.to_c()) == bytes(by_fields(t)) == bytes(d.tiles[0])


@pytest.mark.parametrize("make", [lambda: (1, 2), lambda: [0.5, np.float32(2), np.int64(3)],
                                  lambda: iter((1.0, 0.0, 0.0)), lambda: np.arange(3.0),
                                  lambda: torch.tensor([0.0, 1.0, 0.0]), lambda: ()])
def test_vectors(make):
    a, b = tile(wave_k=make(), wave_pol=make()), tile(wave_k=make(), wave_pol=make())
    assert bytes(a.to_c()) == bytes(by_fields(b))


@pytest.mark.parametrize("kw", [dict(species=1.0), dict(species=None), dict(step_offset=1.5),
                                dict(wave_k=(1.0, 0.0, 0.0, 0.0)), dict(wave_k=("1", 0.0, 0.0)),
                                dict(wave_k=None)])
def test_refused_as_by_ctypes(kw):
    with pytest.raises(Exception) as by_ctypes:
        by_fields(tile(**kw))
    with pytest.raises(by_ctypes.type):
        tile(**kw).to_c()


@pytest.mark.parametrize("kw", [dict(seed=1.0), dict(step=None)])
def test_refused_seeds_and_steps(kw):
    with pytest.raises(TypeError):
        desc(tile(), **kw)
