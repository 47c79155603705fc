"""A handle whose launch shape is not set picks one by the step's size and form: the same results,
bit for bit, as the shape 8 x 2048, at the sizes where the rule changes (256 compute units: a
chunk of 256 up to 131,072 particles, one chunk per block up to 8,388,608) and in every form the
rule tells apart, through sfq_step, sfq_step_noalloc and a plan.
"""
import pytest
import torch

from paper_2301_07684_amd import inputs, sfq

pytestmark = pytest.mark.gpu


def tiles(dev, h, n, form, local):
    out = []
    for species, m in ((sfq.ELECTRON, n - n // 3), (sfq.PHOTON, n // 3)):
        if m == 0:
            continue
        w = inputs.plane_wave_t(m, dev, species=species)
        p = w["p"].contiguous()
        kw, fields = {}, [f.clone() for f in (*w["E"], *w["B"])]
        if form == "wave":
            kw = dict(field_mode=sfq.FIELDS_PLANE_WAVE, wave_amp=w["a"], wave_phase=w["phi"])
            fields = [None] * 6
        elif form == "uniform":
            kw = dict(field_mode=sfq.FIELDS_UNIFORM)
            fields = [torch.full((1,), v, dtype=torch.float64, device=dev)
                      for v in (0.0, 200.0, 0.0, 0.0, 0.0, 200.0)]
        tau = None if local else h.init_optical_depth(w["uid"], seed=3) * 0.3
        out.append(sfq.TileArrays(species, *p, *fields, tau=tau, uid=w["uid"],
                                  alive=torch.ones(m, dtype=torch.uint8, device=dev), **kw))
    return out


def result(ts, pb):
    torch.cuda.synchronize()
    out = [getattr(t, f) for t in ts for f in ("px", "py", "pz", "tau", "alive")
           if getattr(t, f) is not None]
    for k, name in enumerate(("photons", "electrons", "positrons")):
        ps, m = getattr(pb, name), pb.host_counts()[k]
        order = torch.argsort(ps.parent[:m])
        out += [getattr(ps, f)[:m][order] for f in ("px", "py", "pz", "tau", "uid", "parent")]
    return out


@pytest.mark.parametrize("form, local", [("arrays", False), ("arrays", True), ("wave", False),
                                         ("uniform", False)])
@pytest.mark.parametrize("n", [1, 257, 131072, 131073, 8388608, 8388609])
@pytest.mark.parametrize("entry", ["step", "noalloc", "plan"])
def test_shape_by_size_gives_the_same_step(form, local, n, entry):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    got = []
    for shape in ((8, 2048), None):
        h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT,
                       decision=sfq.LOCAL if local else sfq.OPTICAL_DEPTH)
        if shape:
            h.set_launch(*shape)
        assert h.get_launch() == (8, 2048)
        ts = tiles(dev, h, n, form, local)
        pb = sfq.ProductBuffers.empty(n // 2 + 64, n // 4 + 64, dev)
        cnt = sfq.Counters(dev)
        kw = dict(seed=3, step=7, products=pb, counters=cnt, push=True)
        if entry == "plan" and not shape:
            plan = h.plan(ts, **kw)
            plan.launch()
            got.append((result(ts, pb), cnt.results()))
            plan.close()
        else:
            call = h.step_noalloc if entry == "noalloc" and not shape else h.step
            call(ts, zero_product_counts=True, **kw)
            got.append((result(ts, pb), cnt.results()))
        h.close()
    (a, ca), (b, cb) = got
    assert ca == cb and ca["processed"] == n and ca["overflow"] == 0
    assert len(a) == len(b) and all(torch.equal(x, y) for x, y in zip(a, b))


def test_reserved_steps_allocate_nothing():
    """sfq_reserve with no shape set holds the queue of every size up to the reserved one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
    h.set_queue(0.1, adaptive=False)
    h.reserve(1200000, 2)
    held = h.queue_bytes()
    for n in (3, 65536, 262145, 524289, 1048577, 1200000):
        for form in ("arrays", "wave", "uniform"):
            ts = tiles(dev, h, n, form, False)
            h.step(ts, seed=1, step=1, products=sfq.ProductBuffers.empty(n, n, dev),
                   counters=sfq.Counters(dev), push=True)
            assert h.queue_bytes() == held, (n, form)
    torch.cuda.synchronize()


@pytest.mark.parametrize("offset", [0, 1, 2, 7, 8, 15, 16, 17])
@pytest.mark.parametrize("n", [1, 15, 256, 257, 12293, 65521])
@pytest.mark.parametrize("shape", [(1, 256), (8, 1024), None])
def test_slices_step_as_their_copies(offset, n, shape):
    """Tiles that start anywhere in larger arrays (their chunks are cut at 128-byte lines) give the
    bits their aligned copies give, and touch nothing beside the slice."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
    if shape:
        h.set_launch(*shape)
    whole = tiles(dev, h, n + 40, "arrays", False)
    got = []
    for copy in (False, True):
        pb, cnt, ts, kept = sfq.ProductBuffers.empty(n + 40, n + 40, dev), sfq.Counters(dev), [], []
        for t in whole:
            if t.n <= offset:
                continue
            m = min(n, t.n - offset)
            full = {f: getattr(t, f).clone() for f in (
                "px", "py", "pz", "ex", "ey", "ez", "bx", "by", "bz", "tau", "uid", "alive")}
            kept.append((full, {f: v.clone() for f, v in full.items()}, m))
            part = {f: v[offset:offset + m].clone() if copy else v[offset:offset + m]
                    for f, v in full.items()}
            ts.append(sfq.TileArrays(t.species, **part))
        if not ts:
            return
        h.step(ts, seed=5, step=2, products=pb, counters=cnt, push=True, zero_product_counts=True)
        got.append((result(ts, pb), cnt.results()))
        for full, before, m in kept:
            for f in full:
                assert torch.equal(full[f][:offset], before[f][:offset])
                assert torch.equal(full[f][offset + m:], before[f][offset + m:])
    (a, ca), (b, cb) = got
    assert ca == cb and all(torch.equal(x, y) for x, y in zip(a, b))
