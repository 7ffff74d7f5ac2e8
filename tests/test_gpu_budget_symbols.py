"""Budgeted precoding of several symbols: a symbol's bits depend neither on the
symbols before it nor on its place, however strong those are."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import dbp_oracle as O  # noqa: E402
from paper_1702_04458_amd import inputs  # noqa: E402

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1702_04458_amd import api  # noqa: E402


@pytest.mark.parametrize("U,C,S", [(8, 4, 5), (16, 4, 8), (16, 3, 16), (32, 4, 8), (32, 3, 13), (32, 16, 16),
                                   (32, 4, 29), (64, 8, 8), (64, 4, 16), (64, 4, 24), (64, 2, 40), (64, 2, 64)])
@pytest.mark.parametrize("ratio", [1.0, 1e5])
def test_budget_symbols_are_independent(U, C, S, ratio):
    print(f"[gpu] budget symbols U={U} C={C} S={S} ratio={ratio:g}", file=sys.stderr, flush=True)
    n_sc, n_sym = 7, 4
    fr = inputs.downlink_frame(inputs.frame_seed(73, S * C + U, n_sym), n_sc, S * C, U, 64, n_sym=n_sym)
    fr.s[:, 1] *= np.float32(ratio)
    P = torch.tensor([0.02 * (1 + 0.1 * c) for c in range(C)], dtype=torch.float32, device="cuda")
    H, s = torch.from_numpy(fr.H).cuda(), torch.from_numpy(fr.s).cuda()

    def run(v):
        return api.precode(H, v.contiguous(), C, 1.0, 4, P_cluster=P, power="per_cluster")[0]

    x, rev = run(s), run(s.flip(1))
    alone = torch.cat([run(s[:, n:n + 1]) for n in range(n_sym)], 1)
    torch.cuda.synchronize()
    assert torch.equal(x, alone) and torch.equal(x, rev.flip(1))
    ref = O.admm_dl_frame(fr.H, fr.s, C, 1.0, 4, P=P.cpu().numpy().astype(np.float64))
    for n in range(n_sym):
        assert np.linalg.norm(x[:, n].cpu().numpy() - ref[:, n]) <= 1e-5 * np.linalg.norm(ref[:, n])
