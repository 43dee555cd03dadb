"""The selection's float64 statistics over the whole range of its exponentials: logits from
nothing to far beyond the exponent range below the maximum, against numpy's float64 (whose exp
differs from the kernels' by about one unit in the last place), and exact zeros where every other
probability vanishes."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

V = 9001  # two full chunks of 4096 and a ragged one


def entropies(z):
    t = z.astype(np.float64) - z.max(-1, keepdims=True).astype(np.float64)
    with np.errstate(under="ignore"):
        e = np.exp(t)
    Z = e.sum(-1)
    return np.log(Z) - (e * t).sum(-1) / Z, 1.0 / Z


@pytest.fixture(scope="module")
def lib():
    import dataclasses
    from paper_2509_04185_amd import Sbd
    shape = dataclasses.replace(synth.TINY, name="exp", vocab=9088, mask_id=9087, n_layers=1)
    lib = Sbd(shape, synth.make_weights(shape, 9900, device="cuda"), max_batch=1, max_seq_len=64, max_block=16)
    yield lib
    lib.close()


def run(lib, z, gamma):
    k = z.shape[0]
    n, pos, tok, H, C = lib.select(torch.from_numpy(z[None]).cuda(), [[1] * k], "eb_entropy", gamma, -1)
    return int(n[0]), H[0].cpu().numpy(), C[0].cpu().numpy()


@pytest.mark.parametrize("lo,hi", [(1e-6, 1e-3), (0.1, 2.0), (2.0, 40.0), (100.0, 700.0), (700.0, 760.0), (760.0, 1e4)])
def test_spreads(lib, lo, hi):
    print(f"[gpu] selection on logits {lo} to {hi} below the maximum", flush=True)
    rng = np.random.default_rng(int(hi * 10) + 1)
    z = (5.0 - rng.uniform(lo, hi, (16, V))).astype(np.float32)
    z[:, ::97] = z.max(-1, keepdims=True) + np.float32(0.25) * np.arange(16, dtype=np.float32)[:, None] % 3
    _, H, C = run(lib, z, 1.0)
    Hr, Cr = entropies(z)
    # sums of 9001 float64 terms in another order, |H| <= 9.2: below 1e-13
    assert np.abs(H - Hr).max() < 1e-13 and np.abs(C - Cr).max() < 1e-13


def test_vanishing_rows(lib):
    """One logit far above the rest: the entropy is exactly zero once no other term is left, and
    such rows are all accepted at threshold 0."""
    print("[gpu] selection on rows with one probability left", flush=True)
    gaps = np.array([700.0, 707.0, 709.0, 720.0, 744.0, 747.0, 799.0, 801.0, 2e3, 1e5, 1e20, 3e38], np.float32)
    z = np.zeros((gaps.size, V), np.float32) - gaps[:, None]
    z[np.arange(gaps.size), 17 + 700 * np.arange(gaps.size)] = 0.0
    n, H, C = run(lib, z, 0.0)
    Hr, _ = entropies(z)
    assert (C == 1.0).all()
    assert ((H == 0.0) == (Hr == 0.0)).all(), (H, Hr)
    assert np.abs(H - Hr).max() <= 1e-13 * np.abs(Hr).max()
    assert n == int((Hr == 0.0).sum()) + int((Hr != 0.0).any())
