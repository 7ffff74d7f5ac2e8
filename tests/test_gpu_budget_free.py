"""A budget that never binds changes nothing: the budgeted form gives Algorithm 3's
bits, at every kernel of the two (U, padded S) and in both layouts of H."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1702_04458_amd import api, inputs


@pytest.mark.parametrize("U,C,S", [(8, 4, 5), (16, 4, 8), (16, 3, 16), (32, 4, 8), (32, 16, 16), (32, 3, 13), (32, 4, 29),
                                   (64, 8, 8), (64, 4, 16), (64, 4, 24), (64, 2, 33), (64, 3, 47), (64, 8, 64)])
@pytest.mark.parametrize("layout", ["uplink", "downlink"])
@pytest.mark.parametrize("n_sym,eps", [(1, 0.0), (3, 0.3)])
def test_budget_that_never_binds(U, C, S, layout, n_sym, eps):
    print(f"[gpu] free budget U={U} C={C} S={S} {layout} n_sym={n_sym}", file=sys.stderr, flush=True)
    fr = inputs.downlink_frame(inputs.frame_seed(79, S * C + U, n_sym), 9, S * C, U, 64, n_sym=n_sym)
    H, s = torch.from_numpy(fr.H).cuda(), torch.from_numpy(fr.s).cuda()
    if layout == "downlink":
        H = H.transpose(1, 2).contiguous()
    P = torch.full((C,), 1e6, dtype=torch.float32, device="cuda")
    x, beta = api.precode(H, s, C, 1.0, 5, P_cluster=P, power="per_cluster", eps=eps, layout=layout)
    free, _ = api.precode(H, s, C, 1.0, 5, eps=eps, layout=layout)
    torch.cuda.synchronize()
    assert torch.equal(x, free) and bool((beta == 1.0).all())
