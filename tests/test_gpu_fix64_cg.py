"""The FP64 pass of conjugate-gradient detection with every subcarrier flagged, at the
edges of its split of a subcarrier's symbols over workgroups: one subcarrier, as many
workgroups as symbols or fewer, more flagged subcarriers than workgroups, a window of
2,048 flags and one more.  The outputs are the FP64 oracle's rounded to FP32 (one
unit in the last place of the subcarrier's largest value), the decisions its own."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1702_04458_amd import api  # noqa: E402

from test_gpu_fix64 import check, frame  # noqa: E402
from test_gpu_parity import STATUS_RESLICED, to_dev  # noqa: E402


@pytest.mark.parametrize("B,U,C,n_sc,n_sym", [(64, 8, 8, 1, 5), (128, 16, 8, 1, 40), (64, 8, 4, 3, 300), (48, 16, 3, 300, 3),
                                              (32, 8, 4, 129, 2), (24, 8, 3, 2050, 2), (192, 64, 3, 2, 17)])
def test_cg_symbol_split(B, U, C, n_sc, n_sym):
    print(f"[gpu] fix64 cg B={B} U={U} C={C} n_sc={n_sc} n_sym={n_sym}", file=sys.stderr, flush=True)
    T = 3
    fr = frame(n_sc, n_sym, B, U, B + U + n_sym)
    s, h, st = api.detect(to_dev(fr.H), to_dev(fr.y), fr.N0, C, 1.0, T, algo="cg", qam=4, status=True)
    torch.cuda.synchronize()
    assert np.all(st.cpu().numpy() & STATUS_RESLICED)
    sel = np.unique(np.concatenate([np.arange(min(n_sc, 4)), np.arange(max(0, n_sc - 4), n_sc),
                                    np.arange(0, n_sc, max(1, n_sc // 8))]))
    check(s.cpu().numpy(), h.cpu().numpy(), fr, C, T, "cg", sel)
