"""Launch shapes of the split attention (the per-kernel path and forwards of more than 16
rows) against the oracle, on the tiny decoder.

* A batch whose (sequence, KV head) units alone fill the 256 CUs runs with a single key
  split: the split kernel normalises and stores the attention output itself and no merge is
  launched.  128 sequences of ragged lengths (17 to 136 cached positions), k = 2.
* Query rows of a KV head that fit in 32 (G k <= 32) run as 2 row sets x 4 key parts; more
  rows as 4 x 2.  Both, with several key splits, at k = 8 and k = 20 over 16 sequences.
* Four and more row blocks per KV head with one key split share their keys: one row tile a
  wave up to 1.5 workgroups per CU, two above.  Blocks of 64 rows and of 49 (a ragged last row
  block) at batch 8 and 16, sequences of different lengths, causal and prediction rows mixed.
Each with a bf16 and an e4m3 cache; every sequence is compared with the oracle.
"""
import dataclasses

import numpy as np
import pytest
import torch

import parity
import synth
from oracle import sbd_oracle as O

pytestmark = pytest.mark.gpu

REGRESS = (5e-3, 6e-4)


def build(kv, B, max_seq, max_block, seed, shape=synth.TINY):
    from paper_2509_04185_amd import Sbd
    w = synth.make_weights(shape, seed, device="cuda")
    lib = Sbd(shape, w, max_batch=B, max_seq_len=max_seq, max_block=max_block, kv_format=kv)
    fp8 = kv != "bf16"
    model = O.Model(shape, synth.weights_to_host(w), dtype=np.float64, kv_bf16=not fp8,
                    kv_fp8_exp=0 if fp8 else None)
    return shape, lib, model, fp8


def install(shape, lib, seed, lens, fp8):
    caches = []
    for b, L in enumerate(lens):
        kk, vv = synth.make_kv(shape, seed, b, L, device="cuda")
        lib.kv_import(b, 0, kk, vv)
        c = O.SeqCache.from_arrays(synth.to_host_bits(kk), synth.to_host_bits(vv), np.float64)
        caches.append(c.to_e4m3(0) if fp8 else c)
    return caches


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
def test_single_split_many_sequences(kv):
    B, k = 128, 2
    print(f"[gpu] split attention: {B} sequences, k {k}, {kv} cache (one key split)", flush=True)
    shape, lib, model, fp8 = build(kv, B, 160, 8, 9500)
    lens = [17 + (37 * b) % 120 for b in range(B)]
    caches = install(shape, lib, 9500, lens, fp8)
    toks, is_mask = synth.block_rows(9501, shape, B, k, n_causal=1)
    lib.profile(True)
    lib.profile_read()
    got = lib.block_forward(list(range(B)), toks, is_mask=is_mask, n_causal=[1] * B).cpu().numpy()
    prof = lib.profile_read()
    lib.profile(False)
    # one attention launch per layer and no merge: the single-split path ran
    assert prof["attention"][0] == shape.n_layers and prof.get("attn_merge", (0, 0.0))[0] == 0, prof
    ref = model.block_forward(caches, toks, [1] * B).logits
    parity.close(got, ref, regress=REGRESS, label=f"{B}x{k} {kv}: ")
    lib.close()


@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("k", [8, 20])
def test_row_sets_and_splits(kv, k):
    B = 16
    print(f"[gpu] split attention: {B} sequences, k {k}, {kv} cache", flush=True)
    shape, lib, model, fp8 = build(kv, B, 600, 32, 9510 + k)
    lens = [40 + 31 * b for b in range(B)]       # 40 .. 505 positions
    caches = install(shape, lib, 9510 + k, lens, fp8)
    toks, is_mask = synth.block_rows(9520 + k, shape, B, k, n_causal=3)
    nc = [3] * B
    nc[1] = 0
    got = lib.block_forward(list(range(B)), toks, is_mask=is_mask, n_causal=nc).cpu().numpy()
    ref = model.block_forward(caches, toks, nc).logits
    parity.close(got, ref, regress=REGRESS, label=f"{B}x{k} {kv}: ")
    lib.close()


# 8 KV heads of 4 query heads each: 4 row blocks of 64 rows (49 rows: the last one has 4), so
# 32 B workgroups: 256 and 512 on 256 CUs
@pytest.mark.parametrize("kv", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("B,k", [(8, 64), (16, 64), (8, 49), (16, 49)])
def test_shared_keys_in_blocks(B, k, head_dim, kv):
    print(f"[gpu] shared-key attention: {B} x {k} rows, head dim {head_dim}, {kv} cache", flush=True)
    wide = dataclasses.replace(synth.TINY, name="shared", n_q_heads=32, n_kv_heads=8, head_dim=head_dim)
    shape, lib, model, fp8 = build(kv, B, 400, 64, 9540 + k, wide)
    lens = [1 + (97 * b) % 331 for b in range(B)]       # 1 .. 331 positions
    caches = install(shape, lib, 9540 + k, lens, fp8)
    nc = [(0, 1, k, k // 2, 33)[b % 5] for b in range(B)]
    toks = np.full((B, k), shape.mask_id, dtype=np.int32)
    for b in range(B):
        toks[b, :nc[b]] = synth.make_tokens(9550 + k, max(nc), shape, stream=b)[:nc[b]]
    is_mask = (toks == shape.mask_id).astype(np.uint8)
    lib.profile(True)
    lib.profile_read()
    got = lib.block_forward(list(range(B)), toks, is_mask=is_mask, n_causal=nc)
    prof = lib.profile_read()
    lib.profile(False)
    assert prof["attention"][0] == shape.n_layers and prof.get("attn_merge", (0, 0.0))[0] == 0, prof  # one key split
    again = lib.block_forward(list(range(B)), toks, is_mask=is_mask, n_causal=nc)
    assert torch.equal(got, again)
    ref = model.block_forward(caches, toks, nc).logits
    # e4m3: of the 2^19 values and more that a layer stages a few round to the other code, 1/16 of
    # the value, which the rows of that sequence see with the weight of one key in 65 and more
    parity.close(got.cpu().numpy(), ref, regress=(2e-2, 2e-3) if fp8 else REGRESS, label=f"{B}x{k} d_h {head_dim} {kv}: ")
    lib.close()
