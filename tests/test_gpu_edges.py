"""Kernel branches at the sizes where they can go wrong (edges of tiles, remainders, smallest and largest of a range),
against the CPU oracle's primitives in float64."""
import dataclasses

import numpy as np
import pytest

import lp_inputs as LI
from oracle import ops

from gpu_util import compare_step, data_for, generic_params
from test_gpu_kernels import K, dev, host, relerr, rnd, zeros  # noqa: F401  (K is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a_kc,b_kc", [(1, 1), (1, 0), (0, 1), (0, 0)])
@pytest.mark.parametrize("Kd", [65, 72, 127, 136, 200, 1000, 2555])
def test_gemm_reduction_of_any_length(K, Kd, a_kc, b_kc):
    """The 64-deep direct-to-LDS kernel with a partial last k-tile (whole tiles, cut tiles, panels) and the automatic
    choice, twice.  Sums of at most 2555 products in fp32: 1e-6 relative."""
    import torch
    if Kd % 8 and (a_kc or b_kc):
        pytest.skip("a k-contiguous operand has rows of whole 16-byte chunks")
    rng = np.random.default_rng(Kd)
    for (M, N) in ((256, 256), (520, 264), (264, 1032)):
        A, B = rnd(rng, (M, Kd), 1), rnd(rng, (N, Kd), 1)
        Am = A if a_kc else np.ascontiguousarray(A.T)
        Bm = B if b_kc else np.ascontiguousarray(B.T)
        dA, dB = dev(Am, 1), dev(Bm, 1)
        ref = A.astype(np.float64) @ B.astype(np.float64).T
        ws = zeros(2 * 512 * 256 * 256)
        for variant in (0, 20, 21, 22):
            # panel mode needs a few tile columns and ranges shorter than a panel
            if variant == 22 and (N <= 256 or Kd < 1000):
                continue
            outs = []
            for _ in range(2):
                out = zeros(M, N)
                K.lpk_gemm(1, dA, Am.shape[1], a_kc, dB, Bm.shape[1], b_kc, out, N, 1, M, N, Kd, variant=variant, splitk_ws=ws)
                outs.append(out)
            assert relerr(host(outs[0]), ref) <= 2e-6, (M, N, Kd, variant)
            assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("T", [129, 600, 2555])
def test_grouped_weight_gradients_any_rows(K, T):
    """One grouped launch over a row count that is no multiple of a k-tile."""
    import torch
    rng = np.random.default_rng(T)
    shapes = [(64, 192), (192, 64), (64, 64), (320, 128)]
    As = [rnd(rng, (T, m), 1) for m, _ in shapes]
    Bs = [rnd(rng, (T, n), 1) for _, n in shapes]
    ws = zeros(2 * 256 * 256 * 256)
    Cs = [zeros(m, n) for m, n in shapes]
    K.lpk_gemm_grouped([dev(a, 1) for a in As], [dev(b, 1) for b in Bs], Cs, [m for m, _ in shapes], [n for _, n in shapes],
                       T, 0, 0, 0, ws)
    for a, b, c in zip(As, Bs, Cs):
        assert relerr(host(c), a.astype(np.float64).T @ b.astype(np.float64)) <= 2e-6


@pytest.mark.parametrize("vocab", [1001, 1024, 1087, 515])
def test_vocabulary_of_any_size(K, vocab):
    """A step of a decoder whose vocabulary and token count are no multiple of any tile (padded logits)."""
    import paper_2012_03837_amd as lp
    cfg = LI.make_config("cfg3_small", vocab=vocab, seq_len=67, batch=5)
    tr = lp.LocalTrainer(cfg)
    x, y = data_for(cfg)
    compare_step(tr, cfg, generic_params(cfg), x, y, label=f"vocab {vocab}")
    tr.close()
