"""The benchmark's algorithmic bytes count a weight's own size."""
import bench
import synth


def test_weight_bytes_of_the_dominant_kernels():
    s, M = synth.LLAMA8B, 64
    n_gate_up, n_mlp = 2 * s.ffn_dim * s.d_model, 3 * s.ffn_dim * s.d_model
    assert bench.gate_up_bytes(s, M) - bench.gate_up_bytes(s, M, 1) == n_gate_up
    assert bench.layer_mlp_bytes(s, M) - bench.layer_mlp_bytes(s, M, 1) == n_mlp
    fwd2, _ = bench.step_bytes(s, [100], 16)
    fwd1, _ = bench.step_bytes(s, [100], 16, wbytes=1)
    qd, kvd = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    attn = (qd + 2 * kvd) * s.d_model + s.d_model * qd
    assert fwd2 - fwd1 == s.n_layers * (attn + n_mlp) + s.vocab * s.d_model
