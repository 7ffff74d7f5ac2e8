"""Detection and precoding away from unit scale: the channel, the receive vectors,
N0 and the penalty scaled along leave the estimates unchanged, so the relative
error must not know the scale as long as the Gram stays in FP32 (amplitudes of
1e-15 to 1e15 here; the forms that keep the whole inverse are left out, they hold
the product of two reciprocals by design).

Tolerance: 1e-5 relative against the FP64 oracle, the FP32 kernels' bound."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from oracle import dbp_oracle as O
    from paper_1702_04458_amd import api, inputs


@pytest.mark.parametrize("U,C,n_sym", [(16, 4, 1), (16, 4, 9), (32, 2, 1), (32, 2, 9)])
@pytest.mark.parametrize("scale", [1e-15, 1e-12, 1e-9, 1e9, 1e12, 1e15])
def test_detect_scales(U, C, n_sym, scale):
    print(f"[gpu] detect scale U={U} n_sym={n_sym} {scale:g}", file=sys.stderr, flush=True)
    fr = inputs.uplink_frame(inputs.frame_seed(75, U, n_sym), 6, 2 * U * C, U, 16, 15.0, n_sym=n_sym)
    H, y = (fr.H * np.float32(scale)).astype(np.complex64), (fr.y * np.float32(scale)).astype(np.complex64)
    rho, N0 = float(np.float32(scale * scale)), float(np.float32(fr.N0 * scale * scale))
    s, _ = api.detect(torch.from_numpy(H).cuda(), torch.from_numpy(y).cuda(), N0, C, rho, 5, hard=False)
    torch.cuda.synchronize()
    ref = O.admm_ul_frame(H, y, C, rho, 5, N0)
    assert np.linalg.norm(s.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("C,S", [(2, 40), (2, 64)])
@pytest.mark.parametrize("scale", [1e-15, 1e-12, 1e-9, 1e9, 1e12, 1e15])
def test_precode_scales(C, S, scale):
    print(f"[gpu] precode scale U=64 S={S} {scale:g}", file=sys.stderr, flush=True)
    fr = inputs.downlink_frame(inputs.frame_seed(76, S, 1), 6, S * C, 64, 64)
    H, rho = (fr.H * np.float32(scale)).astype(np.complex64), float(np.float32(1.0 / scale ** 2))
    x, _ = api.precode(torch.from_numpy(H).cuda(), torch.from_numpy(fr.s).cuda(), C, rho, 5)
    torch.cuda.synchronize()
    ref = O.admm_dl_frame(H, fr.s, C, rho, 5)
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
