"""Precoding with 33 to 64 antennas per cluster for 64 users, where H is read again
for every product and A_c comes from the matrix cores: the edges of the range, both
layouts of H, padding clusters, several symbols, a ball constraint.

Tolerance: 1e-5 relative against the FP64 oracle, the FP32 kernels' bound."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from oracle import dbp_oracle as O
    from paper_1702_04458_amd import api, inputs


@pytest.mark.parametrize("C,S", [(2, 33), (3, 47), (4, 63), (8, 64), (1, 64)])
@pytest.mark.parametrize("layout", ["uplink", "downlink"])
@pytest.mark.parametrize("n_sym,T,eps", [(1, 5, 0.0), (3, 2, 0.3)])
def test_precode_wide_clusters(C, S, layout, n_sym, T, eps):
    print(f"[gpu] precode U=64 C={C} S={S} {layout} n_sym={n_sym} T={T} eps={eps}", file=sys.stderr, flush=True)
    B, U = S * C, 64
    fr = inputs.downlink_frame(inputs.frame_seed(91, B, n_sym), 5, B, U, 16, n_sym=n_sym)
    H = torch.from_numpy(fr.H).cuda()
    if layout == "downlink":
        H = H.transpose(1, 2).contiguous()
    x, _ = api.precode(H, torch.from_numpy(fr.s).cuda(), C, 1.0, T, eps=eps, layout=layout)
    torch.cuda.synchronize()
    ref = O.admm_dl_frame(fr.H, fr.s, C, 1.0, T, eps=eps)
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)


def test_precode_wide_clusters_isolated():
    """A non-finite entry of one cluster's channel or of one subcarrier stays there:
    reads past a cluster's antennas must not bring in its neighbour."""
    print("[gpu] precode U=64 isolation", file=sys.stderr, flush=True)
    C, S, U = 2, 40, 64
    fr = inputs.downlink_frame(inputs.frame_seed(92, 0, 1), 6, S * C, U, 16)
    H = torch.from_numpy(fr.H).cuda()
    s = torch.from_numpy(fr.s).cuda()
    for layout in ("uplink", "downlink"):
        Hl = H if layout == "uplink" else H.transpose(1, 2).contiguous()
        good, _ = api.precode(Hl, s, C, 1.0, 1, layout=layout)
        bad = Hl.clone()
        if layout == "uplink":
            bad[2, S, 5] = float("nan")      # the second cluster's first antenna
        else:
            bad[2, 5, S] = float("nan")
        x, _ = api.precode(bad, s, C, 1.0, 1, layout=layout)
        torch.cuda.synchronize()
        keep = torch.ones_like(good, dtype=torch.bool)
        keep[2, :, S:] = False               # T = 1: no consensus, the first cluster is untouched
        assert torch.equal(x[keep], good[keep])
        assert not torch.isfinite(torch.view_as_real(x[2, 0, S:])).all()
