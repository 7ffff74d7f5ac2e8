"""The FP64 pass of the exact hard decisions when every subcarrier of a call is
flagged: QPSK with receive vectors of 1e-6, so that every soft value lies within
the guard of the threshold at zero.  The soft outputs must be the FP64 oracle's
rounded to FP32 (one unit in the last place of the subcarrier's largest value)
and the hard decisions the oracle's.  Shapes sit at the edges of the pass: the
chunk (2,048 flags) and slot (256 subcarriers) counts, S not a multiple of the
Gram's row steps, cluster counts below and at the waves of a workgroup, several
symbols."""
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

from test_gpu_parity import STATUS_RESLICED, n0_f32, to_dev  # noqa: E402


def say(msg):
    print(msg, file=sys.stderr, flush=True)


def frame(n_sc, n_sym, B, U, seed):
    fr = inputs.uplink_frame(inputs.frame_seed(61, seed, 10), n_sc, B, U, 4, 10.0, n_sym=n_sym)
    fr.y = (fr.y * np.float32(1e-6)).astype(np.complex64)
    return fr


def check(s, h, fr, C, T, algo, sel):
    if algo == "admm":
        ref = O.admm_ul_frame(fr.H[sel], fr.y[sel], C, 1.0, T, n0_f32(fr.N0))
    else:
        ref = O.dcg_ul_frame(fr.H[sel], fr.y[sel], C, T, n0_f32(fr.N0))
    for i, k in enumerate(sel):
        assert np.abs(s[k] - ref[i]).max() <= 2.0 ** -23 * np.abs(ref[i]).max(), k
    assert np.array_equal(h[sel], O.slice_qam(ref, 4))


@pytest.mark.parametrize("algo,B,U,C,n_sc,n_sym", [
    ("admm", 27, 8, 3, 2049, 1),       # a second chunk of one flag, S = 9
    ("admm", 128, 8, 16, 257, 2),      # 16 waves
    ("admm", 136, 16, 8, 300, 1),      # eight waves, S = 17
    ("admm", 16, 16, 1, 5, 3),         # one cluster, S = U
    ("admm", 198, 32, 6, 259, 1),      # S = 33
    ("admm", 512, 32, 16, 20, 2),      # 16 waves of 32 x 32
    ("admm", 195, 64, 3, 259, 1),      # more subcarriers than slots, S = 65
    ("admm", 512, 64, 8, 12, 2),
    ("cg", 128, 16, 8, 300, 1),
    ("cg", 96, 8, 3, 40, 3),           # symbols of a subcarrier over several workgroups
    ("cg", 512, 64, 8, 9, 17),
])
def test_every_subcarrier_flagged(algo, B, U, C, n_sc, n_sym):
    say(f"[gpu] fix64 {algo} B={B} U={U} C={C} n_sc={n_sc} n_sym={n_sym}")
    T = 4
    fr = frame(n_sc, n_sym, B, U, B + U + C)
    s, h, st = api.detect(to_dev(fr.H), to_dev(fr.y), fr.N0, C, 1.0, T, algo=algo, qam=4, status=True)
    torch.cuda.synchronize()
    assert np.all(st.cpu().numpy() & STATUS_RESLICED)
    sel = np.unique(np.concatenate([np.arange(min(n_sc, 6)), np.arange(max(0, n_sc - 6), n_sc),
                                    np.arange(0, n_sc, max(1, n_sc // 12))]))
    check(s.cpu().numpy(), h.cpu().numpy(), fr, C, T, algo, sel)


@pytest.mark.parametrize("U,shapes", [
    (16, [(128, 8, 70, 1), (64, 4, 1, 2), (256, 16, 33, 1), (51, 3, 300, 1)]),
    (64, [(512, 8, 9, 1), (195, 3, 20, 2), (64, 1, 7, 1)]),
])
def test_every_subcarrier_flagged_batch(U, shapes):
    say(f"[gpu] fix64 batch U={U}")
    T = 4
    frs = [frame(n_sc, n_sym, B, U, 7 * i + U) for i, (B, C, n_sc, n_sym) in enumerate(shapes)]
    outs = api.detect_batch([dict(H=to_dev(f.H), y=to_dev(f.y), N0=f.N0, C=sh[1], T=T, qam=4, status=True)
                             for f, sh in zip(frs, shapes)])
    torch.cuda.synchronize()
    for f, sh, (s, h, st) in zip(frs, shapes, outs):
        assert np.all(st.cpu().numpy() & STATUS_RESLICED)
        sel = np.unique(np.concatenate([np.arange(min(sh[2], 5)), [sh[2] - 1]]))
        check(s.cpu().numpy(), h.cpu().numpy(), f, sh[1], T, "admm", sel)
