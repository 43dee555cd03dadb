"""The per-row and per-sequence parameters of a forward on both sides of what the embedding
kernel's arguments hold (256 rows, 64 sequences), against the oracle: beyond either limit
they are uploaded."""
import numpy as np
import pytest

import parity
import synth
from oracle import sbd_oracle as O

pytestmark = pytest.mark.gpu

SHAPE = synth.TINY
REGRESS = (5e-3, 6e-4)  # the bound of the synthetic-cache cases
MAX_BATCH, MAX_BLOCK = 66, 6


@pytest.fixture(scope="module")
def model():
    from paper_2509_04185_amd import Sbd
    w = synth.make_weights(SHAPE, 9700, device="cuda")
    lib = Sbd(SHAPE, w, max_batch=MAX_BATCH, max_seq_len=128, max_block=MAX_BLOCK)
    host = O.Model(SHAPE, synth.weights_to_host(w), dtype=np.float64, kv_bf16=True)
    caches = []
    for b in range(MAX_BATCH):
        kk, vv = synth.make_kv(SHAPE, 9700, b, 3 + (29 * b) % 71, device="cuda")
        lib.kv_import(b, 0, kk, vv)
        caches.append(O.SeqCache.from_arrays(synth.to_host_bits(kk), synth.to_host_bits(vv), np.float64))
    yield lib, host, caches
    lib.close()


@pytest.mark.parametrize("B,k", [(1, 1), (64, 4), (65, 3), (43, 6), (66, 6)])
def test_parameter_limits(model, B, k):
    lib, host, caches = model
    print(f"[gpu] forward parameters: {B} x {k}", flush=True)
    toks, is_mask = synth.block_rows(9710 + B, SHAPE, B, k, n_causal=1)
    ids = [(7 * b + 3) % MAX_BATCH for b in range(B)]  # 7 and 66 share no factor: distinct slots
    nc = [1] * B
    got = lib.block_forward(ids, toks, is_mask=is_mask, n_causal=nc)
    ref = host.block_forward([caches[i] for i in ids], toks, nc).logits
    parity.close(got.cpu().numpy(), ref, regress=REGRESS, label=f"{B}x{k}: ")
