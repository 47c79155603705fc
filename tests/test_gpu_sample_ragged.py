"""The batched samples do not depend on which lanes of a wave are in use: the first n results of a
long call and a call of n give the same bits, for n around the groups of lanes that evaluate one
table patch (16 requests a round, 64 lanes), in every form (MIXED re-evaluates in FP64 only the
lanes whose energy fraction is above 0.999: scattered lanes of a wave)."""
import pytest
import torch

from paper_2301_07684_amd import inputs, sfq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [sfq.FP64, sfq.MIXED])
@pytest.mark.parametrize("approx", [sfq.APPROX_FULL, sfq.APPROX_TRUNCATED])
@pytest.mark.parametrize("pair", [False, True])
def test_prefixes_of_a_call(precision, approx, pair):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev, n = torch.device("cuda", 0), 4099
    h = sfq.Handle(ref_length=inputs.LAMBDA_R, dt=inputs.DT, precision=precision, approx=approx)
    idx = torch.arange(n, dtype=torch.int64, device=dev)
    u = [inputs.uniforms_t(77, k, idx) for k in range(3)]
    gamma, chi, r = 10.0 ** (2 + 3 * u[0]), 10.0 ** (-1 + 4 * u[1]), u[2]
    call = h.sample_pair if pair else h.sample_photon
    whole = call(gamma, chi, r)
    assert all(bool(torch.isfinite(x).all()) and bool((x >= 0).all()) for x in whole)
    for m in (1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 255, 256, 257, 4095):
        part = call(gamma[:m], chi[:m], r[:m])
        assert all(torch.equal(a, b[:m]) for a, b in zip(part, whole)), m
