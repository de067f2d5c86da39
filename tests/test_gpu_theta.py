"""mcg_theta (the stationarity residual of a field as given) on the GPU against the oracle."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 4, 4, 8), (10, 6, 8, 14)])
def test_theta_vs_oracle(S, O, L, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as g
    from paper_0807_0264_amd import api
    U = g.rounded(S.heatbath_field(L, S.sub_seed(7200), 5.7, 3), prec)
    want = O.theta(U)
    assert abs(api.theta(g.links(U, prec)) - want) <= (1e-12 if prec == 0 else 1e-5) * want
