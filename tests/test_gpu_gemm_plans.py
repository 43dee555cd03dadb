"""The kernels that gemm_plan picks for the wide projections of more than 16 rows, against the oracle.

A narrow decoder's projections all run as 8-tile column blocks (test_gpu_gemm_edges.py); blocks
of 12, 14 and 16 tiles, and the QKV projection of prefill chunks in them, take widths of the 8B
decoders.  Each case names the plans (tiles of a column block, K slices) it is there for, and a
CPU test holds gemm_plan to them, so that a planner change cannot leave a kernel without its
test.  bf16 and e4m3 weights."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import parity
import synth
from oracle import sbd_oracle as O

# 1792 gate/up tiles: 128 blocks of 14.  384 QKV tiles.  2312 vocabulary tiles: 144 blocks of 16
# and a half-full one.
LLAMA = dataclasses.replace(synth.LLAMA8B, name="llama_wide", n_layers=2, vocab=36992, mask_id=36991)
QWEN = dataclasses.replace(synth.QWEN8B, name="qwen_wide", n_layers=2, vocab=36992, mask_id=36991)
MAX_ROWS = 1100

# rows, shape, weights: plans (tiles, K slices) of the QKV, O, gate/up and down projections and
# of the LM head; blocks of B x k rows, or a prefill
BLOCKS = [
    # 65 to 128 rows: gate/up in two slices, of 16 tiles and with e4m3 weights of 14
    (LLAMA, "bf16", 5, 13, {"qkv": (8, 5), "o": (8, 8), "gate_up": (16, 2), "down": (8, 8), "lm_head": (16, 1)}),
    (LLAMA, "fp8", 5, 13, {"qkv": (8, 5), "o": (8, 8), "gate_up": (14, 2), "down": (8, 8)}),
    (LLAMA, "bf16", 8, 16, {"gate_up": (16, 2), "lm_head": (16, 1)}),
    (LLAMA, "fp8", 8, 16, {"gate_up": (14, 2)}),
    (LLAMA, "fp8", 6, 16, {"gate_up": (14, 2)}),
    # more: 14 tiles unsplit, 16 tiles in slices
    (LLAMA, "bf16", 10, 16, {"qkv": (16, 5), "o": (8, 4), "gate_up": (14, 1), "down": (16, 8)}),
    (LLAMA, "fp8", 10, 16, {"qkv": (16, 5), "o": (8, 4), "gate_up": (14, 1), "down": (16, 8)}),
    (LLAMA, "fp8", 16, 16, {"qkv": (16, 5), "gate_up": (14, 1), "down": (16, 8)}),
    # 12 tiles: three row tile counts, in slices and not
    (QWEN, "bf16", 2, 13, {"gate_up": (12, 2)}),
    (QWEN, "bf16", 3, 13, {"gate_up": (12, 2)}),
    (QWEN, "bf16", 9, 13, {"gate_up": (12, 2)}),
    (QWEN, "bf16", 13, 13, {"gate_up": (12, 1)}),
]
PREFILLS = [
    # QKV's K steps added in fp32, in 16 tiles with slices, in 12 with and without
    (LLAMA, "bf16", 300, {"qkv": (16, 3), "o": (16, 5), "gate_up": (14, 1), "down": (16, 5)}),
    (LLAMA, "bf16", 512, {"qkv": (12, 2), "o": (16, 4), "gate_up": (14, 1), "down": (16, 4)}),
    (LLAMA, "bf16", 1024, {"qkv": (12, 1), "o": (16, 2), "gate_up": (14, 1), "down": (16, 2)}),
    # e4m3: 16 tiles, with slices and without
    (LLAMA, "fp8", 300, {"qkv": (16, 3), "o": (16, 5), "gate_up": (14, 1), "down": (16, 5)}),
    (LLAMA, "fp8", 640, {"qkv": (16, 2), "o": (16, 3), "gate_up": (14, 1), "down": (16, 3)}),
    (LLAMA, "fp8", 1024, {"qkv": (16, 1), "o": (16, 2), "gate_up": (14, 1), "down": (16, 2)}),
]


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("mt", "nt", "splits", "m_blocks", "n_cb")]


def plans(s, weights, M, fold):
    """gemm_plan's (tiles, K slices) of every projection, with the options launch_gemm passes."""
    from paper_2509_04185_amd import load_library
    f = load_library()._ZN3sbd9gemm_planEiiilbbi
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 3 + [ctypes.c_int64] + [ctypes.c_bool] * 2 + [ctypes.c_int]
    bf16 = weights == "bf16"
    d, qd, n_qkv = s.d_model, s.n_q_heads * s.head_dim, (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim
    cap = 8 * 256 * max(n_qkv, d)  # floats of split-K partials with 256 rows and more (compute_layout)
    out = {}
    for name, tiles, K, nt12, half, nt14 in (("qkv", n_qkv // 16, d, fold and bf16, bf16, 0),
                                             ("o", d // 16, qd, False, False, 0),
                                             ("gate_up", s.ffn_dim // 8, d, bf16, False, 1 if bf16 else 8),
                                             ("down", d // 16, s.ffn_dim, False, False, 0),
                                             ("lm_head", s.vocab // 16, d, False, bf16, 0)):
        p = f(M, tiles, K, cap, nt12, half, nt14)
        out[name] = (p.nt, p.splits)
    return out


@pytest.mark.parametrize("shape,weights,B,k,want", BLOCKS)
def test_plans_of_blocks(shape, weights, B, k, want):
    got = plans(shape, weights, B * k, False)
    assert {n: got[n] for n in want} == want


@pytest.mark.parametrize("shape,weights,n,want", PREFILLS)
def test_plans_of_prefills(shape, weights, n, want):
    got = plans(shape, weights, n, n > 256)
    assert {p: got[p] for p in want} == want


@pytest.fixture(scope="module")
def models():
    made = {}

    def get(shape, weights):
        from paper_2509_04185_amd import Sbd
        key = (shape.name, weights)
        if key not in made:
            for lib, _, _ in made.values():
                lib.close()
            made.clear()  # one at a time: the cases are grouped
            w = (synth.make_weights_fp8 if weights == "fp8" else synth.make_weights)(shape, 9700, device="cuda")
            lib = Sbd(shape, w, max_batch=16, max_seq_len=MAX_ROWS, max_block=16)
            host = O.Model(shape, synth.weights_to_host(w), dtype=np.float32, kv_bf16=True)
            made[key] = (lib, host, w)
        return made[key]

    yield get
    for lib, _, _ in made.values():
        lib.close()


ORDER = sorted(range(len(BLOCKS)), key=lambda i: (BLOCKS[i][0].name, BLOCKS[i][1]))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,weights,B,k,want", [BLOCKS[i] for i in ORDER])
def test_blocks(models, shape, weights, B, k, want):
    lib, host, _ = models(shape, weights)
    print(f"[gpu] {shape.name} {weights}: {B} x {k} rows", flush=True)
    caches = []
    for b in range(B):
        lib.reset(b)
        kk, vv = synth.make_kv(shape, 9700, b, 3 + (29 * b) % 71, device="cuda")
        lib.kv_import(b, 0, kk, vv)
        caches.append(O.SeqCache.from_arrays(synth.to_host_bits(kk), synth.to_host_bits(vv), np.float32))
    toks, is_mask = synth.block_rows(9710 + B, shape, B, k, n_causal=1)
    got = lib.block_forward(list(range(B)), toks, is_mask=is_mask)
    ref = host.block_forward(caches, toks, [1] * B).logits
    # about ten times the error of two layers of the 8B shape (test_gpu_fullsize.py)
    parity.close(got.cpu().numpy(), ref, regress=(5e-3, 6e-4), label=f"{B}x{k}: ")


@pytest.mark.gpu
@pytest.mark.parametrize("shape,weights,n,want", PREFILLS)
def test_prefills(models, shape, weights, n, want):
    lib, host, _ = models(shape, weights)
    print(f"[gpu] {shape.name} {weights}: prefill of {n}", flush=True)
    prompt = synth.make_tokens(9720, n, shape, stream=5)
    lib.reset(0)
    logits = lib.prefill(0, prompt)
    k, v = lib.kv_export(0, 0, n)
    torch.cuda.synchronize()
    cache, ref = host.prefill(prompt)
    # layer 0 is the QKV projection alone: one bf16 unit where the two sides round differently
    # (2^-5 at magnitudes up to 8), at few positions; layer 1 sees what those and every other
    # projection do (test_gpu_prefill.py)
    for got, want_, name in ((k, cache.K, "K"), (v, cache.V, "V")):
        parity.close(got[0].float().cpu().numpy(), want_[0], max_abs=0.07, regress=(0.07, 5e-4), label=f"{name} layer 0: ")
        parity.close(got[1].float().cpu().numpy(), want_[1], max_abs=0.07, regress=(0.07, 4e-3), label=f"{name} layer 1: ")
    parity.close(logits.cpu().numpy(), np.asarray(ref).reshape(-1), regress=(5e-2, 7e-3), label="logits: ")
