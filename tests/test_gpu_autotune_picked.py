"""The autotuner's result is never slower than not tuning: the shape the library picks when none is set
is among what it times, and where that is fastest the handle picks again (from the cache too)."""
import json

import pytest
import torch

from paper_2301_07684_amd import autotune, inputs, sfq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 65536, 500000])
def test_picked_shape_is_a_candidate(n, tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
    w = inputs.plane_wave_t(n, dev, species=sfq.ELECTRON)
    p, E, B = (w[k].contiguous() for k in ("p", "E", "B"))
    tiles = [sfq.TileArrays(sfq.ELECTRON, *p, *E, *B, uid=w["uid"],
                            tau=h.init_optical_depth(w["uid"], seed=3))]
    pb, cnt = sfq.ProductBuffers.empty(n, 8, dev), sfq.Counters(dev)
    h.set_launch(1, 4096)                 # a shape set before does not stay
    cache = str(tmp_path / "tune.json")
    res = autotune.tune(h, tiles, pb, cnt, cache_path=cache)
    assert res["ms"] == min(res["timings"].values()) <= res["timings"]["picked"]
    assert res["picked"] == (res["ms"] == res["timings"]["picked"])
    assert h.get_launch() == tuple(res["shape"])

    def queue(prepare):
        """The queue that one step leaves tells which shape it had."""
        k = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
        prepare(k)
        part = [sfq.TileArrays(sfq.ELECTRON, **{
            f: getattr(tiles[0], f)[:n].clone() for f in (
                "px", "py", "pz", "ex", "ey", "ez", "bx", "by", "bz", "uid", "tau")})]
        k.step(part, seed=1, step=1, products=pb, counters=cnt)
        torch.cuda.synchronize()
        return k.queue_bytes()

    # what the cache holds is applied again: a picked entry unsets the shape
    saved = json.load(open(cache))
    (key, entry), = saved.items()
    for picked in (True, False):
        autotune.save_cache({key: dict(entry, shape=[8, 2048], picked=picked)}, cache)

        def from_cache(k):
            k.set_launch(1, 4096)
            r = autotune.tune(k, tiles, pb, cnt, cache_path=cache)
            assert r["cached"] and r["picked"] == picked and k.get_launch() == (8, 2048)

        want = queue(lambda k: None if picked else k.set_launch(8, 2048))
        assert queue(from_cache) == want
    # entries written without the word hold a set shape
    autotune.save_cache({key: {f: v for f, v in dict(entry, shape=[2, 1024]).items()
                               if f != "picked"}}, cache)
    r = autotune.tune(h, tiles, pb, cnt, cache_path=cache)
    assert r["cached"] and h.get_launch() == (2, 1024)


def test_given_candidates_only(tmp_path):
    """Callers that name the candidates get one of them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev, n = torch.device("cuda", 0), 8192
    h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
    w = inputs.plane_wave_t(n, dev, species=sfq.ELECTRON)
    p, E, B = (w[k].contiguous() for k in ("p", "E", "B"))
    tiles = [sfq.TileArrays(sfq.ELECTRON, *p, *E, *B, uid=w["uid"],
                            tau=h.init_optical_depth(w["uid"], seed=3))]
    res = autotune.tune(h, tiles, sfq.ProductBuffers.empty(n, 8, dev), sfq.Counters(dev),
                        cache_path=None, repeats=1, candidates=[(1, 4096), (2, 4096)])
    assert set(res["timings"]) == {"1x4096", "2x4096"} and not res["picked"]
    assert h.get_launch() == tuple(res["shape"])
