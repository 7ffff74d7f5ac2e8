"""Calls of more than 2^32 work items, which take several launches (the runtime cuts a
larger launch off without an error): every subcarrier of a repeated frame gets the
result of the short frame, across the boundary between the launches too."""
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1702_04458_amd import _native, api, inputs

PERIOD = 1000


def repeated(t, n):
    return t.repeat(n // PERIOD, *[1] * (t.dim() - 1))


def same(got, want, n):
    return torch.equal(got.view(n // PERIOD, *want.shape), want.expand(n // PERIOD, *want.shape))


def test_cg_of_34_million_subcarriers():
    """U = 8, nine clusters of one antenna: 128 work items per subcarrier."""
    n, U, C = 34_000_000, 8, 9
    print(f"[gpu] CG over {n} subcarriers", file=sys.stderr, flush=True)
    fr = inputs.uplink_frame(inputs.frame_seed(85, U, C), PERIOD, C, U, 16, 20.0)
    H, y = torch.from_numpy(fr.H).cuda(), torch.from_numpy(fr.y).cuda()
    want, _, st = api.detect(H, y, fr.N0, C, T=2, algo="cg", hard=False, status=True)
    got, _, sl = api.detect(repeated(H, n), repeated(y, n), fr.N0, C, T=2, algo="cg", hard=False, status=True)
    torch.cuda.synchronize()
    assert same(got, want, n) and same(sl, st, n)


def test_precode_of_34_million_subcarriers():
    n, U, C = 34_000_000, 8, 9
    print(f"[gpu] precoding over {n} subcarriers", file=sys.stderr, flush=True)
    fr = inputs.downlink_frame(inputs.frame_seed(86, U, C), PERIOD, C, U, 16)
    H, s = torch.from_numpy(fr.H).cuda(), torch.from_numpy(fr.s).cuda()
    P = torch.full((C,), 0.02, dtype=torch.float32, device="cuda")
    want, wb = api.precode(H, s, C, 1.0, 2, P_cluster=P)
    got, gb = api.precode(repeated(H, n), repeated(s, n), C, 1.0, 2, P_cluster=P)
    torch.cuda.synchronize()
    assert same(got, want, n) and same(gb, wb, n)


def test_pack_and_flags_of_17_million_tiles():
    n, B, U, C = 2_120_000, 64, 8, 8
    print(f"[gpu] packed channel of {n * C} tiles", file=sys.stderr, flush=True)
    fr = inputs.uplink_frame(inputs.frame_seed(87, U, C), PERIOD, B, U, 16, 20.0)
    H = torch.from_numpy(fr.H).cuda()
    want = api.pack_channel_h16(H, C)
    got = api.pack_channel_h16(repeated(H, n), C)
    torch.cuda.synchronize()
    body, tail = PERIOD * B * U * 4, PERIOD * C * 4
    big = n // PERIOD
    assert torch.equal(got[:big * body].view(big, body), want[:body].expand(big, body))
    assert torch.equal(got[big * body:].view(big, tail), want[body:].expand(big, tail))

    n = 17_000_000
    x = torch.ones(n, 4, dtype=torch.complex64, device="cuda")
    bad = torch.arange(0, n, 999_983, device="cuda")
    x[bad, 3] = float("nan")
    status = torch.empty(n, dtype=torch.int32, device="cuda")
    _native.check(_native.lib().dbp_flag_nonfinite(x.data_ptr(), n, 4, status.data_ptr(), None))
    torch.cuda.synchronize()
    assert torch.equal(torch.nonzero(status)[:, 0], bad)
