"""Detection of several received vectors per subcarrier as matrix columns, at the
edges of its rule and tiles: the first symbol count that takes it, one, exactly
one and more than one block of eight symbols, padding clusters, ragged rows, a
ragged last workgroup, T = 1.

Tolerance: 1e-5 relative against the FP64 oracle, the FP32 kernels' bound, which
the form does not change (the same products in another order)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from oracle import dbp_oracle as O
    from paper_1702_04458_amd import api, inputs


def say(msg):
    print(msg, file=sys.stderr, flush=True)


def frame(n_sc, n_sym, B, U, seed, qam=16, snr=15.0, corr=0.0):
    fr = inputs.uplink_frame(inputs.frame_seed(81, seed, n_sym), n_sc, B, U, qam, snr, n_sym=n_sym, corr=corr)
    return fr, torch.from_numpy(fr.H).cuda(), torch.from_numpy(fr.y).cuda()


def oracle(fr, C, T, reg="mmse", rho=1.0):
    return O.admm_ul_frame(fr.H, fr.y, C, rho, T, float(np.float32(fr.N0)), reg=reg, box_r=O.box_radius(fr.qam))


CASES = [(16, 3, 19, 4, 5, "mmse"), (16, 8, 16, 8, 5, "box"), (16, 16, 17, 9, 3, "zf"), (16, 4, 33, 14, 1, "mmse"),
         (32, 2, 33, 5, 5, "mmse"), (32, 3, 32, 8, 4, "box"), (32, 8, 37, 9, 5, "mmse"), (32, 16, 32, 17, 2, "zf"),
         (64, 1, 64, 3, 5, "mmse"), (64, 3, 67, 7, 5, "box"), (64, 8, 64, 9, 3, "mmse")]


@pytest.mark.parametrize("U,C,S,n_sym,T,reg", CASES)
def test_symbols_as_columns(U, C, S, n_sym, T, reg):
    say(f"[gpu] symbols U={U} C={C} S={S} n_sym={n_sym} T={T} {reg}")
    n_sc = 21
    fr, H, y = frame(n_sc, n_sym, S * C, U, U + C + S)
    s, h, st = api.detect(H, y, fr.N0, C, 1.0, T, qam=16, reg=reg, status=True)
    soft, _ = api.detect(H, y, fr.N0, C, 1.0, T, qam=16, reg=reg, hard=False)
    torch.cuda.synchronize()
    ref = oracle(fr, C, T, reg)
    for v in (s, soft):
        assert np.linalg.norm(v.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.array_equal(h.cpu().numpy(), O.slice_qam(ref, 16))
    assert not (st.cpu().numpy() & 1).any()


@pytest.mark.parametrize("U,C,S,n_sym,T,reg", [c for c in CASES if c[5] != "box"])
def test_symbols_as_columns_cg(U, C, S, n_sym, T, reg):
    say(f"[gpu] symbols by CG U={U} C={C} S={S} n_sym={n_sym} T={T} {reg}")
    fr, H, y = frame(21, n_sym, S * C, U, U + C + S)
    s, h, st = api.detect(H, y, fr.N0, C, T=T, algo="cg", qam=16, reg=reg, status=True)
    torch.cuda.synchronize()
    ref = O.dcg_ul_frame(fr.H, fr.y, C, T, float(np.float32(fr.N0)), reg=reg)
    assert np.linalg.norm(s.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.array_equal(h.cpu().numpy(), O.slice_qam(ref, 16))
    assert not (st.cpu().numpy() & 1).any()


@pytest.mark.parametrize("U,C", [(16, 4), (32, 4), (64, 2)])
def test_symbols_are_independent(U, C):
    """A symbol with infinities and NaN leaves the others' bits alone, and a
    symbol's bits depend neither on its place nor on the symbols beside it."""
    say(f"[gpu] symbols independent U={U} C={C}")
    n_sc, n_sym = 9, 11
    fr, H, y = frame(n_sc, n_sym, U * C, U, U)
    s, _ = api.detect(H, y, fr.N0, C, qam=16, hard=False)
    y2 = y.clone()
    y2[2, 4, 5] = complex(float("nan"), 0.0)
    y2[3, 10, 0] = complex(float("inf"), 1.0)
    s2, _, st = api.detect(H, y2, fr.N0, C, qam=16, hard=False, status=True)
    rev, _ = api.detect(H, y.flip(1).contiguous(), fr.N0, C, qam=16, hard=False)
    part, _ = api.detect(H, y[:, 3:10].contiguous(), fr.N0, C, qam=16, hard=False)
    torch.cuda.synchronize()
    keep = torch.ones(n_sc, n_sym, dtype=torch.bool, device=s.device)
    keep[2, 4] = keep[3, 10] = False
    assert torch.equal(s2[keep], s[keep])
    assert not torch.isfinite(torch.view_as_real(s2[2, 4])).all() and not torch.isfinite(torch.view_as_real(s2[3, 10])).all()
    assert (st.cpu().numpy() & 1).tolist() == [0, 0, 1, 1, 0, 0, 0, 0, 0]
    assert torch.equal(rev.flip(1), s) and torch.equal(part, s[:, 3:10])


@pytest.mark.parametrize("U", [16, 32, 64])
def test_symbols_in_a_batch(U):
    """Frames on both sides of the rule in one batch: the bits of the single calls."""
    say(f"[gpu] symbols in a batch U={U}")
    frames = []
    for i, (C, n_sc, n_sym) in enumerate([(8, 5, 7), (4, 13, 1), (1, 6, 9), (8, 0, 9), (3, 33, 14), (2, 7, 2)]):
        fr, H, y = frame(max(n_sc, 1), n_sym, U * C, U, i)
        frames.append(dict(H=H[:n_sc], y=y[:n_sc], N0=fr.N0, C=C, qam=16, status=True))
    out = api.detect_batch(frames)
    for f, got in zip(frames, out):
        want = api.detect(f["H"], f["y"], f["N0"], f["C"], qam=16, status=True)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("U,C,n_sym", [(32, 2, 1), (32, 4, 7), (64, 2, 1), (64, 2, 7)])
@pytest.mark.parametrize("corr,rho", [(0.7, 1.0), (0.9, 1.0), (0.9, 0.1)])
def test_block_factors_of_correlated_channels(U, C, n_sym, corr, rho):
    """The block factors at S = U on antenna-correlated channels: an error of the
    order of the conditioning, kappa_2(B_c) u with u = 2^-24 (a Schur complement
    from the explicit inverse of the leading block would lose up to kappa^2 u)."""
    say(f"[gpu] block factors U={U} n_sym={n_sym} corr={corr} rho={rho}")
    fr, H, y = frame(12, n_sym, U * C, U, U + C, corr=corr)
    s, _ = api.detect(H, y, fr.N0, C, rho, 5, qam=16, hard=False)
    torch.cuda.synchronize()
    ref = oracle(fr, C, 5, rho=rho)
    Hc = fr.H.astype(np.complex128).reshape(12, C, U, U)
    ev = np.linalg.eigvalsh(np.swapaxes(Hc.conj(), -1, -2) @ Hc + rho * np.eye(U))
    kappa = (ev[..., -1] / ev[..., 0]).max()
    assert np.linalg.norm(s.cpu().numpy() - ref) <= max(1e-5, kappa * 2.0 ** -24) * np.linalg.norm(ref)


@pytest.mark.parametrize("U,C,S,n_sym", [(16, 3, 19, 4), (16, 8, 16, 9), (32, 3, 33, 5), (32, 8, 32, 9), (64, 1, 67, 3),
                                         (64, 8, 64, 9)])
@pytest.mark.parametrize("h16", [False, True])
def test_symbols_of_a_static_channel(U, C, S, n_sym, h16):
    """Against stored factors: the oracle's result, and for the packed channel, whose
    rounding of H the oracle does not have, the results of one symbol at a time
    (both within 1e-5 of the exact ones of the rounded channel, so 2e-5 apart)."""
    say(f"[gpu] symbols against factors U={U} C={C} S={S} n_sym={n_sym} h16={h16}")
    fr, H, y = frame(19, n_sym, S * C, U, U + S)
    F = api.factor(H, C, 1.0)
    if not h16:
        s, h = api.detect_factored(H, F, y, fr.N0, C, qam=16)
        ref = oracle(fr, C, 5)
        assert np.linalg.norm(s.cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
        assert np.array_equal(h.cpu().numpy(), O.slice_qam(ref, 16))
        return
    packed = api.pack_channel_h16(H, C)

    def run(v):
        return api.detect_factored_h16(packed, F, v, fr.N0, S * C, U, C, qam=16, hard=False)[0]

    want = torch.cat([run(y[:, n:n + 1].contiguous()) for n in range(n_sym)], 1).cpu().numpy()
    assert np.linalg.norm(run(y).cpu().numpy() - want) <= 2e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("U,C,S", [(32, 3, 33), (64, 2, 64)])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("rho", [1.0, 0.01])
def test_symbols_in_mixed_precision(U, C, S, prec, rho):
    """Mixed modes with the FP64 factor rule (S = U or close: on): the oracle's
    decisions, the conditioning flags of a single symbol, and soft values within
    the modes' 1e-3."""
    say(f"[gpu] symbols mixed U={U} C={C} S={S} {prec} rho={rho}")
    n_sym = 9
    fr, H, y = frame(11, n_sym, S * C, U, U + S, snr=20.0)
    s, h, st = api.detect(H, y, fr.N0, C, rho, qam=16, prec=prec, status=True)
    _, _, st1 = api.detect(H, y[:, :1].contiguous(), fr.N0, C, rho, qam=16, prec=prec, status=True)
    torch.cuda.synchronize()
    ref = oracle(fr, C, 5, rho=rho)
    assert np.linalg.norm(s.cpu().numpy() - ref) <= 1e-3 * np.linalg.norm(ref)
    assert np.array_equal(h.cpu().numpy(), O.slice_qam(ref, 16))
    assert torch.equal(st & 4, st1 & 4)
