"""The fp32 r = 128 kernel in the split arithmetic (scan_wide_kernel) against
the oracle, through the C-ABI (needs a GPU): chains of one to a few slots
(prologue, both parities of its slot loop, the last slot), hinted slots of one
to four panels and one to eight row blocks in every order, compact storage,
segments (two-level) and streaming; values that the split cannot hold.

Tolerance: relative Frobenius 1e-5, the fp32 bar; a lost partial product of
the split shows at 2^-16 = 1.5e-5 per slot and above.  Hinted, compact and
streamed results equal the unhinted ones bit for bit (what a hint leaves out
adds exact zeros).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_09204_amd import binding, synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = 1e-5
CYCLES = [(128,), (128, 16), (16, 128), (32, 64, 128), (112, 48, 16, 80), (96, 128, 64), (64,),
          (80, 64)]


def _err(lam, x):
    return oracle.rel_frobenius(lam.cpu().numpy().astype(np.float64),
                                oracle.recurrence(x.A, x.b, x.lamK))


@pytest.mark.parametrize("affine", [True, False])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 9])
@pytest.mark.parametrize("cycle", CYCLES, ids=["-".join(map(str, c)) for c in CYCLES])
def test_wide_hinted_compact_streamed(cycle, K, affine):
    widths = synth.cyclic_widths(K, cycle)
    x = synth.random_chain(5, K, 128, seed=70 + K, widths=widths, affine=affine)
    g = x.to(DEV)
    lam = binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=binding.LBI_ALGO_CHAIN)
    assert _err(lam, x) <= TOL
    hinted = binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, list(widths),
                                          algo=binding.LBI_ALGO_CHAIN)
    assert torch.equal(lam, hinted)
    progress = torch.zeros(5, dtype=torch.int32, device=DEV)
    clock = torch.zeros((5, -(-K // 2)), dtype=torch.int64, device=DEV)
    streamed = binding.lbi_scan_backward_streaming(g.A, g.b, g.lamK, progress, 2, list(widths),
                                                   publish_clock=clock)
    assert torch.equal(lam, streamed)
    assert progress.tolist() == [K] * 5 and bool((clock > 0).all())
    if max(widths) > 64:  # compact storage takes the smallest tile that holds every width
        p = synth.pack_ragged(x)
        c = binding.lbi_scan_backward_ragged(p.A.to(DEV), None if p.b is None else p.b.to(DEV),
                                             p.lamK.to(DEV), list(widths))
        assert torch.equal(synth.unpack_ragged(c.cpu(), widths, 128), lam.cpu())


@pytest.mark.parametrize("B,K", [(3, 37), (70, 128)])
def test_wide_segments_and_products(B, K):
    """Segments in both two-level forms (composites kept; past 256 MiB, scanned
    again), and the exported composites with and without a hint."""
    x = synth.random_chain(B, K, 128, seed=81)
    g = x.to(DEV)
    lam = binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=binding.LBI_ALGO_TWO_LEVEL)
    assert _err(lam, x) <= TOL
    P, c = binding.lbi_scan_suffix_products(g.A[:3], g.b[:3])
    Ph, ch = binding.lbi_scan_suffix_products(g.A[:3], g.b[:3], widths=[128] * (K + 1))
    assert torch.equal(P, Ph) and torch.equal(c, ch)
    Pr, cr = oracle.suffix_composites(x.A[:3], x.b[:3])
    assert oracle.rel_frobenius(P.cpu().numpy().astype(np.float64), Pr) <= TOL
    assert oracle.rel_frobenius(c.cpu().numpy().astype(np.float64), cr) <= TOL


@pytest.mark.parametrize("affine", [True, False])
@pytest.mark.parametrize("cycle", CYCLES, ids=["-".join(map(str, c)) for c in CYCLES])
def test_wide_hinted_products(cycle, affine):
    """The exported composites with narrow widths: slots of one to four panels and row
    blocks of every number, bit for bit the unhinted ones."""
    K = 14
    widths = synth.cyclic_widths(K, cycle)
    x = synth.random_chain(3, K, 128, seed=83, widths=widths, affine=affine)
    g = x.to(DEV)
    P, c = binding.lbi_scan_suffix_products(g.A, g.b)
    Ph, ch = binding.lbi_scan_suffix_products(g.A, g.b, widths=list(widths))
    assert torch.equal(P, Ph) and torch.equal(c, ch)
    Pr, cr = oracle.suffix_composites(x.A, x.b)
    assert oracle.rel_frobenius(Ph.cpu().numpy().astype(np.float64), Pr) <= TOL
    if affine:
        assert oracle.rel_frobenius(ch.cpu().numpy().astype(np.float64), cr) <= TOL


@pytest.mark.parametrize("cycle", [(32, 64, 128), (112, 48, 16, 80)])
def test_wide_hinted_segments(cycle):
    """Segments that are scanned again from their carries (70 x 128: past 256 MiB of
    composites), with segment ends of every width of the cycle."""
    B, K = 70, 128
    widths = synth.cyclic_widths(K, cycle)
    x = synth.random_chain(B, K, 128, seed=84, widths=widths)
    g = x.to(DEV)
    two = binding.LBI_ALGO_TWO_LEVEL
    lam = binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, list(widths), algo=two)
    assert _err(lam, x) <= TOL
    assert torch.equal(lam, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=two))


# A chain's tiles times 2^-e (per slot), and a value planted at row 5, column 7 of a
# tile: what the three-part split cannot hold (infinities, NaN, magnitudes that round
# to an infinity in bf16, values that keep bits below 2^-133).  The finite results
# stay above 2^-116, so that float32 itself keeps all its bits.
RANGE = {"inf": (0, {3: float("inf")}), "inf at the end": (0, {10: float("inf")}),
         "both infinities": (0, {2: float("-inf"), 4: float("inf")}), "nan": (0, {3: float("nan")}),
         "huge": (5, {3: 3.4e38}), "huge at the end": (5, {10: -3.4e38}), "decaying": (10, {}),
         "small at the start": ([112] + [0] * 10, {}), "small at the end": ([0] * 10 + [112], {}),
         "grown, then small": ([112] + [-10] * 10, {}), "fading": ([2] * 38, {}),
         "fading, then grown": ([-4] * 20 + [3] * 28, {}),
         "fading, then grown past the scale": ([-8] * 20 + [3] * 28, {}),
         "vanishing beside a small lambda_K": ([0] * 4 + [-100, 60, 60] + [0] * 4, {})}


@pytest.mark.parametrize("cycle", [None, (32, 64, 128), (128, 16)], ids=["full", "mixed", "thin"])
@pytest.mark.parametrize("affine", [True, False])
@pytest.mark.parametrize("what", list(RANGE))
def test_wide_whole_float32_range(what, affine, cycle):
    """Over the whole range of float32 the default arithmetic gives what the fp32
    matrix cores give: infinities and NaN in the same places (the affine terms are
    finite and change neither; the padding of a hinted call is left out), and the
    finite entries at the parity bar, slot by slot (a slot's norm may be 1e-30 of
    another's), in every form of the launch.  A second, ordinary chain beside the
    planted one keeps its results.

    Entries below float32's normal range are held to its spacing there, 2^-149.

    A finite planted value makes a row of its slot out of one entry of the adjoint
    after it, so that row's relative error is that entry's: the bar times the norm of
    the slot after it over that entry."""
    shift, planted = RANGE[what]
    shift = torch.tensor([shift] * 11 if isinstance(shift, int) else shift)
    K = len(shift)
    widths = synth.cyclic_widths(K, cycle or (128,))
    x = synth.random_chain(2, K, 128, seed=97, widths=widths, affine=affine)
    x.A[0] = torch.ldexp(x.A[0], -shift[:, None, None])
    end = -60 if "small lambda_K" in what else 0
    x.lamK[0] = torch.ldexp(x.lamK[0], torch.tensor(end))
    if affine:  # as large as the adjoint beside it (that float32 holds)
        scale = (end - shift.flip(0).cumsum(0).flip(0)).clamp(min=-120)
        x.b[0] = torch.ldexp(x.b[0], scale[:, None])
    tol = TOL
    finite = [j for j, v in planted.items() if np.isfinite(v)]
    if finite:
        want = oracle.recurrence(x.A, x.b, x.lamK)
        after = np.concatenate([want, x.lamK.double().numpy()[:, None]], axis=1)[0, finite[0] + 1]
        tol = TOL * float(np.linalg.norm(after) / abs(after[7]))
    for j, value in planted.items():
        x.A[0, j, 5, 7] = value
    g = x.to(DEV)
    hint = None if cycle is None else list(widths)
    live = torch.arange(128) < torch.tensor(widths[:K])[:, None]

    def run(algo, math=binding.LBI_MATH_DEFAULT, b=g.b):
        return binding.lbi_scan_backward_ex(g.A, b, g.lamK, hint, math, algo)

    def check(got, exact, pattern, what):
        got, exact, pattern = (t.cpu()[:, live] for t in (got, exact, pattern))
        assert torch.equal(got.isnan(), pattern.isnan()), what
        assert torch.equal(got.isinf(), pattern.isinf()), what
        ok = got.isfinite() & exact.isfinite()
        slot = torch.arange(K).repeat_interleave(torch.tensor(widths[:K]))
        for j in range(K):
            a, e = ((t * ok)[:, slot == j].nan_to_num(0, 0, 0).double() for t in (got, exact))
            err = ((a - e).flatten(1).norm(dim=1) - a[0].numel() ** 0.5 * 2.0 ** -149).clamp(min=0)
            err /= e.flatten(1).norm(dim=1).clamp(min=1e-45)
            assert float(err[0]) <= tol and float(err[1]) <= TOL, (what, j, err)

    fp32 = binding.LBI_MATH_F32_MFMA
    lam = run(binding.LBI_ALGO_CHAIN)
    check(lam, run(binding.LBI_ALGO_CHAIN, fp32), run(binding.LBI_ALGO_CHAIN, fp32, None), "chain")
    two = binding.LBI_ALGO_TWO_LEVEL
    check(run(two), run(two, fp32), run(two, fp32, None), "two-level")
    P, c = binding.lbi_scan_suffix_products(g.A, g.b, hint)
    Pm, _ = binding.lbi_scan_suffix_products(g.A, None, hint, fp32)
    check(P[..., :widths[K]], Pm[..., :widths[K]], Pm[..., :widths[K]], "products")
    if not planted:
        want = oracle.recurrence(x.A, x.b, x.lamK)
        check(lam, torch.from_numpy(want), torch.from_numpy(want), "oracle")
        Pr, cr = oracle.suffix_composites(x.A, x.b)
        check(P, torch.from_numpy(Pr), torch.from_numpy(Pr), "oracle's products")
        if affine:
            check(c, torch.from_numpy(cr), torch.from_numpy(cr), "oracle's affine parts")
    for chunk in (1, 3):
        progress = torch.zeros(2, dtype=torch.int32, device=DEV)
        clock = torch.zeros((2, -(-K // chunk)), dtype=torch.int64, device=DEV)
        streamed = binding.lbi_scan_backward_streaming(g.A, g.b, g.lamK, progress, chunk, hint,
                                                       publish_clock=clock)
        assert torch.equal(streamed.view(torch.int32), lam.view(torch.int32))
        assert progress.tolist() == [K] * 2
        assert bool((clock > 0).all()) and bool((clock.diff(dim=1) >= 0).all())
    if cycle is not None:
        p = synth.pack_ragged(x)
        r = binding.lbi_scan_backward_ragged(p.A.to(DEV), None if p.b is None else p.b.to(DEV),
                                             p.lamK.to(DEV), list(widths)).cpu()
        r = synth.unpack_ragged(r, widths, 128)
        assert torch.equal(r[:, live].view(torch.int32), lam.cpu()[:, live].view(torch.int32))


@pytest.mark.parametrize("cycle", [None, (32, 64, 128)], ids=["full", "mixed"])
def test_wide_range_in_rescanned_segments(cycle):
    """What the split cannot hold, in chains whose segments are folded to their
    aggregates only and scanned again from their carries (past 256 MiB of composites):
    as the fp32 matrix cores give it, the other chains at the parity bar."""
    B, K = 70, 128
    widths = synth.cyclic_widths(K, cycle or (128,))
    x = synth.random_chain(B, K, 128, seed=85, widths=widths, affine=False)
    x.A[0, 40, 5, 7] = float("inf")
    x.A[1, 107, 5, 7] = 3.4e38
    x.A[1, 108:] *= 2.0 ** -3
    x.A[2, 120] = torch.ldexp(x.A[2, 120], torch.tensor(-112))
    x.A[2, :120] = torch.ldexp(x.A[2, :120], torch.tensor(1))
    x.A[3, 16:27] = torch.ldexp(x.A[3, 16:27], torch.tensor(-10))  # within a segment or two
    x.A[3, 27:] = torch.ldexp(x.A[3, 27:], torch.tensor(1))
    g = x.to(DEV)
    hint = None if cycle is None else list(widths)
    lam, want = (binding.lbi_scan_backward_ex(g.A, None, g.lamK, hint, math,
                                              binding.LBI_ALGO_TWO_LEVEL).cpu()
                 for math in (binding.LBI_MATH_DEFAULT, binding.LBI_MATH_F32_MFMA))
    live = torch.arange(128) < torch.tensor(widths[:K])[:, None]
    assert torch.equal(lam[:, live].isnan(), want[:, live].isnan())
    assert torch.equal(lam[:, live].isinf(), want[:, live].isinf())
    ref = oracle.recurrence(x.A[2:], None, x.lamK[2:])
    got = lam[2:].numpy().astype(np.float64)
    for j in range(K):  # slot by slot: a slot's norm may be 1e-30 of another's
        err = np.linalg.norm(got[:, j] - ref[:, j], axis=1) / np.linalg.norm(ref[:, j], axis=1)
        assert err.max() <= 4 * TOL, (j, err.argmax(), err.max())
    ok = want[1][live].isfinite()
    assert bool(ok.all())
    a, b = lam[1][live].double(), want[1][live].double()
    after = want[1, 108]
    factor = float(after.double().norm() / after[7].abs())
    assert float((a - b).norm() / b.norm()) <= factor * TOL
