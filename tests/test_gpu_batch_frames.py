"""Batches of unlike frames: what one frame of a batch asks for must not change what
another one gets."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1702_04458_amd import api, inputs


def frame(n_sc, U, C, seed, n_sym=1, tiny=False, **kw):
    fr = inputs.uplink_frame(inputs.frame_seed(82, seed, U), max(n_sc, 1), U * C, U, 4, 10.0, n_sym=n_sym)
    y = fr.y * np.float32(1e-6) if tiny else fr.y   # (tiny: every soft value near the threshold at zero)
    return dict(H=torch.from_numpy(fr.H).cuda()[:n_sc], y=torch.from_numpy(y).cuda()[:n_sc], N0=fr.N0, C=C, qam=4, **kw)


def check(frames):
    out = api.detect_batch(frames)
    for f, got in zip(frames, out):
        kw = {k: f[k] for k in ("hard", "status") if k in f}
        want = api.detect(f["H"], f["y"], f["N0"], f["C"], qam=4, **kw)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert (a is None and b is None) or torch.equal(a, b)


@pytest.mark.parametrize("U,C_soft", [(64, 8), (32, 16), (16, 16)])
@pytest.mark.parametrize("n_soft", [0, 5])
def test_batch_soft_frame_of_more_clusters(U, C_soft, n_soft):
    """One subcarrier of one cluster with hard decisions beside a frame of many
    clusters that has none (or is empty): the FP64 pass needs slots of the first
    frame's size only, and its workspace holds one."""
    print(f"[gpu] batch slots U={U} C={C_soft} n_soft={n_soft}", file=sys.stderr, flush=True)
    check([frame(1, U, 1, 1, tiny=True, status=True), frame(n_soft, U, C_soft, 2, hard=False)])


def test_batch_of_many_work_items():
    """24 frames over one channel of 1.4 million subcarriers: more than 2^32 work
    items, with the boundary between two launches inside a frame.  Every frame is
    the single call's result."""
    n_sc, U, C, period = 1_400_000, 8, 9, 1000
    print(f"[gpu] batch 24 x {n_sc} U={U} C={C}", file=sys.stderr, flush=True)
    fr = inputs.uplink_frame(inputs.frame_seed(83, U, C), period, U * C, U, 16, 15.0)
    H = torch.from_numpy(fr.H).cuda().repeat(n_sc // period, 1, 1)
    y = torch.from_numpy(fr.y).cuda().repeat(n_sc // period, 1, 1)
    f = dict(H=H, y=y, N0=fr.N0, C=C, T=1, qam=16, hard=False)
    out = api.detect_batch([f] * 24)
    want, _ = api.detect(H[:period], y[:period], fr.N0, C, 1.0, 1, qam=16, hard=False)
    torch.cuda.synchronize()
    for s, _ in out:
        assert torch.equal(s.view(-1, period, 1, U), want.expand(n_sc // period, period, 1, U))
