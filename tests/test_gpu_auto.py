"""What LBI_ALGO_AUTO runs where its choice depends on the number of chains
(needs a GPU): the two-level scan with the workspace that the query asks for,
and, where that workspace is an offer (the cost model of the other arithmetics
would take the chain scan), the chain scan without it; each bit for bit as the
algorithm named by itself, and all of them against the oracle.

Tolerance: the parity bars, 1e-5 (fp32) and 1e-3 (bf16 with the hi + lo
feedback, which leaves about 1e-5).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_09204_amd import binding, synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = {"f32": 1e-5, "bf16": 1e-3}


def _err(lam, x):
    return oracle.rel_frobenius(lam.cpu().numpy().astype(np.float64),
                                oracle.recurrence(x.A, x.b, x.lamK))


CHAIN, WAVE, TWO = (binding.LBI_ALGO_CHAIN, binding.LBI_ALGO_CHAIN_WAVE,
                    binding.LBI_ALGO_TWO_LEVEL)
# (B, K, r, dtype, affine, AUTO's algorithm, the chain scan without workspace or
# None where the workspace is required)
SHAPES = [(150, 100, 64, "bf16", True, TWO, CHAIN), (150, 70, 64, "bf16", False, CHAIN, CHAIN),
          (256, 130, 32, "bf16", True, TWO, WAVE), (400, 100, 32, "bf16", False, WAVE, WAVE),
          (260, 70, 32, "f32", True, TWO, CHAIN), (90, 33, 16, "bf16", True, WAVE, WAVE),
          (90, 100, 64, "f32", False, TWO, None), (3, 200, 64, "f32", True, TWO, None),
          (20, 37, 128, "f32", True, TWO, None)]


@pytest.mark.parametrize("B,K,r,dtype,affine,algo,less", SHAPES)
def test_auto_with_and_without_workspace(B, K, r, dtype, affine, algo, less):
    x = synth.random_chain(B, K, r, dtype=dtype, seed=91)
    if not affine:
        x.b = None
    g = x.to(DEV)
    lam = binding.lbi_scan_backward(g.A, g.b, g.lamK)
    assert _err(lam, x) <= TOL[dtype]
    assert torch.equal(lam, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=algo))
    assert _err(binding.lbi_scan_backward_noalloc(g.A, g.b, g.lamK), x) <= TOL[dtype]
    little = torch.empty((16,), dtype=torch.uint8, device=DEV)
    if less is not None:
        lam = binding.lbi_scan_backward(g.A, g.b, g.lamK, workspace=little)
        assert torch.equal(lam, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=less))
    else:
        with pytest.raises(binding.LbiError) as e:
            binding.lbi_scan_backward(g.A, g.b, g.lamK, workspace=little)
        assert e.value.status == 5  # LBI_ERR_WORKSPACE


def test_auto_takes_no_workspace_that_overlaps():
    """A workspace that overlaps an argument was never looked at where AUTO ran the
    chain scan; where it now takes the two-level scan if it can, it still does not
    refuse or use such a workspace."""
    x = synth.random_chain(150, 100, 64, dtype="bf16", seed=96)
    g = x.to(DEV)
    want = binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=CHAIN)
    got = binding.lbi_scan_backward(g.A, g.b, g.lamK, workspace=g.A.view(torch.uint8).flatten())
    assert torch.equal(got, want)
    need = binding.lbi_scan_backward_workspace_bytes(150, 100, 64, 1)
    ws = torch.empty((need,), dtype=torch.uint8, device=DEV)
    lam = ws[:4 * want.numel()].view(torch.float32).view_as(want)
    assert torch.equal(binding.lbi_scan_backward(g.A, g.b, g.lamK, lam=lam, workspace=ws), want)


def test_auto_hint_keeps_the_chain_scan():
    """bf16 chains at r = 128, as many as the cost model leaves to the chain scan: they
    run it with and without a widths hint, on the LDS-ring kernel for widths that it
    takes and bit for bit as the unhinted call for others."""
    B, K = 86, 64
    for cycle, algo in (((32, 64, 128), binding.LBI_ALGO_CHAIN_RING), ((16, 128), CHAIN)):
        widths = list(synth.cyclic_widths(K, cycle))
        x = synth.random_chain(B, K, 128, dtype="bf16", seed=94, widths=tuple(widths))
        g = x.to(DEV)
        lam = binding.lbi_scan_backward(g.A, g.b, g.lamK)
        assert torch.equal(lam, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=CHAIN))
        hinted = binding.lbi_scan_backward_widths(g.A, g.b, g.lamK, widths)
        assert torch.equal(hinted, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, widths,
                                                                algo=algo))
        assert _err(hinted, x) <= TOL["bf16"]
        if algo == CHAIN:
            assert torch.equal(hinted, lam)


@pytest.mark.parametrize("K,r,most", [(13, 16, 512), (12, 32, 512), (11, 32, 256)])
def test_auto_tree_batch_limit(K, r, most):
    """fp32 chains within a tree chunk: one tree launch up to a number of them."""
    for B in (most, most + 1):
        x = synth.random_chain(B, K, r, seed=93)
        g = x.to(DEV)
        lam = binding.lbi_scan_backward(g.A, g.b, g.lamK)
        assert _err(lam, x) <= TOL["f32"]
        algo = binding.LBI_ALGO_TREE if B == most else binding.LBI_ALGO_CHAIN
        assert torch.equal(lam, binding.lbi_scan_backward_ex(g.A, g.b, g.lamK, algo=algo))


@pytest.mark.parametrize("algo", ["CHAIN_WAVE", "CHAIN"])
@pytest.mark.parametrize("r", [16, 32, 64])
def test_bf16_affine_exact(algo, r):
    """Signed permutation matrices and small integers: every value that the scan
    forms is an integer below 2^8, so the affine term's sums over lanes have to
    give the oracle's adjoints exactly, from the shortest chains on."""
    gen = torch.Generator().manual_seed(95)
    for B, K in ((3, 1), (3, 2), (5, 3), (2, 4), (7, 40)):
        A = torch.zeros((B, K, r, r))
        for i in range(B):
            for j in range(K):
                sign = 1 - 2 * torch.randint(0, 2, (r,), generator=gen)
                A[i, j, torch.arange(r), torch.randperm(r, generator=gen)] = sign.float()
        b = torch.randint(-3, 4, (B, K, r), generator=gen).float()
        lk = torch.randint(-3, 4, (B, r), generator=gen).float()
        A, b, lk = (t.bfloat16() for t in (A, b, lk))
        lam = binding.lbi_scan_backward_ex(A.to(DEV), b.to(DEV), lk.to(DEV),
                                           algo=getattr(binding, "LBI_ALGO_" + algo))
        assert np.array_equal(lam.cpu().numpy(), oracle.recurrence(A, b, lk)), (B, K)
