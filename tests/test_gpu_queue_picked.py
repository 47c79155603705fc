"""Steps of more emitters than a new handle's queue expects: with no launch shape set they defer no more
particles than at the shape 8 x 2048, whose blocks are more and smaller, and give the same results."""
import pytest
import torch

from paper_2301_07684_amd import inputs, sfq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, fraction", [(9000000, 0.25), (16777216, 0.2)])
def test_dense_first_steps(n, fraction):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    w = inputs.plane_wave_t(n, dev, species=sfq.ELECTRON)
    E, B = w["E"].contiguous(), w["B"].contiguous()
    u = inputs.uniforms_t(5, 0, torch.arange(n, dtype=torch.int64, device=dev))
    made, deferred = [], []
    for shape in ((8, 2048), None):
        h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT)
        if shape:
            h.set_launch(*shape)
        p = w["p"].clone()
        tau = torch.where(u < fraction, 1e-300, 1e9).to(torch.float64)
        tile = sfq.TileArrays(sfq.ELECTRON, *p, *E, *B, uid=w["uid"], tau=tau)
        pb, cnt = sfq.ProductBuffers.empty(n // 3, 8, dev), sfq.Counters(dev)
        h.step([tile], seed=3, step=7, products=pb, counters=cnt)
        torch.cuda.synchronize()
        c = cnt.as_dict()
        deferred.append(c["deferred"])
        assert c["processed"] == n and c["overflow"] == 0 and c["emitted"] > 0.9 * fraction * n
        order = torch.argsort(pb.photons.parent[:c["emitted"]])
        made.append([p, tau, *(getattr(pb.photons, f)[:c["emitted"]][order]
                               for f in ("px", "py", "pz", "tau", "uid", "parent"))])
        h.close()
    assert deferred[1] <= deferred[0] and deferred[0] > 0
    assert all(torch.equal(a, b) for a, b in zip(*made))
