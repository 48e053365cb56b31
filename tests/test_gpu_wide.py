"""The fp32 r = 128 kernel in the split arithmetic (scan_wide_kernel) against
the oracle, through the C-ABI (needs a GPU): chains of one to a few slots
(prologue, both parities of its slot loop, the last slot), hinted slots of one
to four panels and one to eight row blocks in every order, compact storage,
segments (two-level) and streaming.

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
CYCLES = [(128,), (128, 16), (16, 128), (32, 64, 128), (112, 48, 16, 80), (96, 128, 64)]


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
