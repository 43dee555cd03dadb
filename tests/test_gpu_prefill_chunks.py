"""Prefills on both sides of the sizes at which a chunk changes its kernels, against the oracle:
the 256 rows past which the QKV projection adds every K step in fp32, whole and ragged row
blocks of 128, and the 1024 rows past which a prompt takes several forwards.  The logits of the
last row, and keys and values at every position of both layers.  The projections of this narrow
decoder mostly run as 8-tile column blocks; wider ones are in test_gpu_gemm_plans.py."""
import dataclasses

import numpy as np
import pytest
import torch

import parity
import synth
from oracle import sbd_oracle as O

pytestmark = pytest.mark.gpu

SHAPE = dataclasses.replace(synth.TINY_QK, name="chunks", d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64,
                            ffn_dim=2816, vocab=2176, mask_id=2175)
N_MAX = 2100


@pytest.fixture(scope="module", params=["bf16", "fp8"])
def model(request):
    from paper_2509_04185_amd import Sbd
    make = synth.make_weights_fp8 if request.param == "fp8" else synth.make_weights
    w = make(SHAPE, 9800, device="cuda")
    lib = Sbd(SHAPE, w, max_batch=1, max_seq_len=N_MAX, max_block=16)
    host = O.Model(SHAPE, synth.weights_to_host(w), dtype=np.float64, kv_bf16=True)
    prompt = synth.make_tokens(9800, N_MAX, SHAPE, stream=3)
    cache, _ = host.prefill(prompt)  # causal: every shorter prompt's cache is its beginning
    yield lib, host, prompt, cache
    lib.close()


@pytest.mark.parametrize("n", [1, 33, 256, 257, 300, 385, 511, 1024, 1025, 2065])
def test_prefill_sizes(model, n):
    lib, host, prompt, cache = model
    print(f"[gpu] prefill of {n} tokens, {lib.weight_format} weights", flush=True)
    lib.reset(0)
    logits = lib.prefill(0, prompt[:n])
    k, v = lib.kv_export(0, 0, n)
    torch.cuda.synchronize()
    # one bf16 unit (2^-5 at magnitudes up to 8) where the two sides round differently
    for got, ref, name in ((k, cache.K, "K"), (v, cache.V, "V")):
        for l in range(SHAPE.n_layers):
            parity.close(got[l].float().cpu().numpy(), ref[l][:n], max_abs=0.07, regress=(0.07, 4e-3),
                         label=f"{name} layer {l}: ")
    part = O.SeqCache.from_arrays(np.stack([cache.K[l][:n - 1] for l in range(SHAPE.n_layers)]),
                                  np.stack([cache.V[l][:n - 1] for l in range(SHAPE.n_layers)]), np.float64) \
        if n > 1 else None
    if part is not None:
        ref = host.block_forward([part], prompt[None, n - 1:n], [1]).logits
        parity.close(logits.cpu().numpy(), ref.reshape(-1), label="logits: ")


# 8 KV heads: from 497 rows the attention's workgroups take the whole key range, with one or (past
# 768 rows) two row tiles a wave; with small chunks it takes key splits of one tile a wave.
@pytest.mark.parametrize("head_dim,kv", [(64, "bf16"), (64, "fp8_e4m3"), (128, "bf16"), (128, "fp8_e4m3")])
def test_attention_forms_agree(head_dim, kv):
    from paper_2509_04185_amd import Sbd
    shape = dataclasses.replace(SHAPE, name="forms", n_q_heads=32, n_kv_heads=8, head_dim=head_dim, n_layers=2)
    w = synth.make_weights(shape, 9810, device="cuda")
    one = Sbd(shape, w, max_batch=1, max_seq_len=N_MAX, max_block=16, kv_format=kv)
    many = Sbd(shape, w, max_batch=1, max_seq_len=N_MAX, max_block=16, prefill_chunk=48, kv_format=kv)
    prompt = synth.make_tokens(9810, N_MAX, shape, stream=4)
    for n in (513, 640, 769, 833, 1024, 2000):
        print(f"[gpu] attention of a prefill of {n}, head dim {head_dim}, cache {kv}", flush=True)
        out = []
        for lib in (one, many):
            lib.reset(0)
            out.append((lib.prefill(0, prompt[:n]), *lib.kv_export(0, 0, n)))
        torch.cuda.synchronize()
        (la, ka, va), (lb, kb, vb) = out
        # the same sums in another order: cached values differ where a rounding moves (float
        # errors of 5e-5 against rounding steps of 2^-3 relative, e4m3, or 2^-8, bf16: below 1e-3
        # and 3e-2 of them), and the logits by what those do to the second layer
        frac = 3e-3 if kv != "bf16" else 3e-2
        for x, y in ((ka, kb), (va, vb)):
            assert (x != y).float().mean() < frac
            assert ((x - y).float().norm() / y.float().norm()) < 1e-2
        rel = float((la - lb).norm() / lb.norm())
        print(f"    logits rel-L2 {rel:.2e}", flush=True)
        assert rel < (2e-2 if kv != "bf16" else 4e-3)
    one.close()
    many.close()
