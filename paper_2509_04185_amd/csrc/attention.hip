// Block-hybrid grouped-query attention of the SBD block forward.
//
// For sequence b with cache length L and block rows j = 0..k-1 (stored at positions
// L + j), row j attends to key position kv iff kv < L + j + 1 when j is a causal row
// (j < n_causal) and to every key kv < L + k when j is in the prediction block: the
// inference mask of the paper (App. A, Fig. 3) restricted to the rows of the block.
//
// Work split: one workgroup per (split, KV head x row block, sequence).  The rows of a
// KV head are the group*k (query head, block row) pairs that read it; each wave takes 16
// of them (one MFMA tile) and walks the keys of its split in 32-key steps:
//   S^T = K Q^T   (v_mfma_f32_16x16x32_bf16: keys on M, query rows on N, d_h in 4 steps;
//                  Q as hi + lo bf16, two MFMAs per step)
//   online softmax per query row in base 2 (queries carry log2(e)/sqrt(d_h))
//   O^T += V^T P^T (P as hi + lo bf16 in the B-operand layout straight from the score
//                   tile; V^T comes from the transposed, permuted cache blocks)
// Each split leaves unnormalised (max, sum, O) per row; a merge kernel combines the
// splits with log-sum-exp weights in split order.  K and V blocks are staged in LDS by the
// whole workgroup (see the kernels: attention_body.h for the launches that share a
// workgroup with other phases, attn_split_kernel below for the standalone split kernel).

#include <type_traits>

#include "attention_body.h"

namespace sbd {

// Maximum and sum over the four lanes r, r + 16, r + 32, r + 48 of a row: the lane swaps of
// gfx950 work in the vector unit, where a shuffle is a round trip through LDS in the middle of
// a stage's dependency chain.
__device__ __forceinline__ float row_max4(float v) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
  s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float row_sum4(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// The split kernel of the per-kernel path streams long key ranges, so it is shaped for
// bytes in flight: 8 waves, NRS row sets of 16 query rows times KP = 8 / NRS key parts (4 x 2,
// or 2 x 4 when a row block has at most 32 rows, so that no wave idles); the key positions
// of a ring stage (KP blocks of 32 keys of K and V from a bf16 cache, 2 KP from an fp8 cache;
// copied straight into LDS) are split between the KP waves holding the same 16 query rows,
// so each SIMD has two waves to overlap MFMA, softmax and LDS reads with the stream (an fp8
// wave takes two blocks per stage under one softmax update: the chain of a stage, not its
// bytes, sets its time); a ring of NBUF stages (128 KB) keeps NBUF - 1 stages in flight.  At
// the end the KP key parts of each row set are combined through LDS (log-sum-exp weights,
// in part order) into the split's partial.  LDS reads are ds_read16 (ds_read8 of an fp8
// cache), ordered by hand (see sbd_device.h).
// What a stage costs is its serial chain (LDS reads, scores, softmax, P V), so the chain is
// short: keys are hidden only in blocks that hold some (wave-uniform), a row's maximum crosses
// lanes in the vector unit, sums stay per lane until the end, and the state is rescaled only by
// a block that brings some row a new maximum.  Per layer, before, with that, and with addresses
// formed once: Llama 4 x 32768 116, 108, 98 us (5.5 TB/s), Qwen 8 x 8192 71.6, 58.5, 55.9, e4m3
// cache 8 x 2048 24.0, 22.2, 22.3.
//
// SRT > 0 (many row blocks read the same keys, whole key range per workgroup: prefill): workgroup
// i takes KV head i % n_kv, so that with eight KV heads an XCD reads one head's keys and values
// and they stay in its L2 (cached loads), and the row blocks go from the last to the first.  Rows
// are numbered query head first, so that within each head the blocks that see the most keys start
// before those that see fewer (not over all heads): prompts of 576 tokens 22.8 -> 18.0 us, 768
// 33.2 -> 29.3, the same where the rounds are full.  A wave takes SRT row tiles; with two, every fragment it reads feeds twice the products
// and two chains overlap (a prompt of 4096 in chunks of 1024, per layer: one 377 us, two 342 us;
// e4m3 cache 405 and 345).  The two waves of a SIMD go in step: one of them a phase behind the
// other, softmax beside scores, took a ring stage and was slower (e4m3 cache 360 us against 340 us,
// bf16 340 against 332).
template <int DH, bool KV8, int NRS, int SRT>
__global__ __launch_bounds__(512) void attn_split_kernel(AttnArgs a) {
  constexpr bool SHARED = SRT > 0;
  using KB = KvBlk<DH, KV8>;    // a staged block's layout in LDS
  constexpr int NDT = DH / 16;  // 16-wide dimension tiles
  constexpr int NKS = DH / 32;  // 32-wide reduction steps for the scores
  constexpr int KP = 8 / NRS;                 // key parts
  constexpr int BLK = KB::BYTES;              // bytes of K (or of V) per 32-key block
  constexpr int BPW = KV8 && !SHARED ? 2 : 1;  // blocks per wave and stage
  constexpr int RT = SHARED ? SRT : 1;        // row tiles (16 query rows) per wave
  constexpr int BPS = KP * BPW;               // blocks per stage
  constexpr int STAGE = BPS * 2 * BLK;        // K and V of the stage's blocks
  constexpr int NBUF = (128 * 1024) / STAGE > 8 ? 8 : (128 * 1024) / STAGE;
  constexpr int LPB = BLK / 1024;             // 1 KB wave-loads per part per block
  constexpr int PER_WAVE = STAGE / 1024 / 8;  // wave-loads of one wave per stage
  static_assert(NBUF >= 2 && (NBUF - 2) * PER_WAVE <= 63, "ring shape");
  static_assert(NRS * KP == 8 && (KP - 1) * NRS * 64 * RT * (NDT * 16 + 16) <= NBUF * STAGE, "wave shape");
  __shared__ __attribute__((aligned(16))) char smem[NBUF * STAGE];
  __shared__ int s_kend[8];

  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rs = w % NRS, kh = w / NRS;  // row set (16 rows), key part of each stage
  const int r = lane & 15, grp = lane >> 4;
  const int split = SHARED ? 0 : blockIdx.x, b = blockIdx.z;
  const int g = SHARED ? (int)blockIdx.x % a.n_kv : (int)blockIdx.y / a.n_rowblocks;
  const int rb = SHARED ? (int)gridDim.x / a.n_kv - 1 - (int)blockIdx.x / a.n_kv : (int)blockIdx.y % a.n_rowblocks;
  const SeqParam sp = a.seqs[b];
  const int L = sp.cache_len, nc = sp.n_causal, k = a.k;
  const int G = a.n_q / a.n_kv;
  const int R = G * k;
  // row tile t of this wave: lane's row, its query head and block row, and its last key
  bool row_ok[RT];
  int hq[RT], jr[RT], kend[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int rho = (rb * NRS + rs) * 16 * RT + t * 16 + r;
    row_ok[t] = rho < R;
    hq[t] = g * G + (row_ok[t] ? rho / k : 0);
    jr[t] = row_ok[t] ? rho % k : 0;
    kend[t] = row_ok[t] ? ((jr[t] >= nc) ? L + k : L + jr[t] + 1) : 0;
  }
  const int blk0 = split * a.blocks_per_split, blk_lim = blk0 + a.blocks_per_split;
  int kend_w = 0, kmin_w = INT32_MAX;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    kend_w = max(kend_w, kend[t]);
    kmin_w = min(kmin_w, row_ok[t] ? kend[t] : INT32_MAX);
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    kend_w = max(kend_w, __shfl_xor(kend_w, o));
    kmin_w = min(kmin_w, __shfl_xor(kmin_w, o));
  }
  kmin_w = __builtin_amdgcn_readfirstlane(kmin_w);  // keys every row of this wave sees
  const int blk1 = min(blk_lim, (kend_w + 31) / 32);  // this wave's blocks end here
  int kend_wg = kend_w;
  kend_wg = max(kend_wg, __shfl_xor(kend_wg, 16));
  kend_wg = max(kend_wg, __shfl_xor(kend_wg, 32));
  if (lane == 0) s_kend[w] = kend_wg;

  // queries (B operand, hi and lo): row r, dims 32 s + 8 grp .. + 8; complete before the ring
  i32x4 qf[RT][NKS], ql[RT][NKS];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int64_t qoff = ((int64_t)(b * k + jr[t]) * a.n_q + hq[t]) * DH;
#pragma unroll
    for (int s2 = 0; s2 < NKS; ++s2) {
      qf[t][s2] = row_ok[t] ? *(const i32x4*)(a.q + qoff + 32 * s2 + 8 * grp) : i32x4{0, 0, 0, 0};
      ql[t][s2] = row_ok[t] ? *(const i32x4*)(a.q_lo + qoff + 32 * s2 + 8 * grp) : i32x4{0, 0, 0, 0};
    }
  }
  vm_wait<0>();
  __syncthreads();
  for (int i = 0; i < 8; ++i) kend_wg = max(kend_wg, s_kend[i]);
  const int blk1_wg = min(blk_lim, (kend_wg + 31) / 32);
  const int n_st = blk1_wg > blk0 ? (blk1_wg - blk0 + BPS - 1) / BPS : 0;

  const int64_t hb = attn_head_base(a.layer, sp.slot, g, a.n_slots, a.n_kv, a.cap, DH);
  const char* kbase = static_cast<const char*>(a.kcache) + hb * KB::ES;
  const char* vbase = static_cast<const char*>(a.vcache) + hb * KB::ES;
  const float kv_sc = a.kv_scale;
  // Wave-load u of wave w in stage st: i = w + 8u -> block i / (2 LPB) of the stage, part
  // (i / LPB) % 2 (K, V), 1 KB slice i % LPB; pieces XOR-swizzled (KvBlk).
  const char* src[PER_WAVE];  // of block 0: a block of K, and one of V, is BLK bytes further
#pragma unroll
  for (int u = 0; u < PER_WAVE; ++u) {
    const int idx = w + 8 * u;
    src[u] = KB::src(kbase, vbase, 0, (idx / LPB) % 2, (idx % LPB) * 64 + lane);
  }
  auto issue = [&](int st) {
    char* buf = smem + (st % NBUF) * STAGE;
#pragma unroll
    for (int u = 0; u < PER_WAVE; ++u) {
      const int idx = w + 8 * u;
      const int bi = idx / (2 * LPB), part = (idx / LPB) % 2, sub = idx % LPB;
      const int kb = min(blk0 + BPS * st + bi, blk1_wg - 1);  // past the end: a valid block, never used
      __builtin_amdgcn_global_load_lds((const void*)(src[u] + (int64_t)kb * BLK),
                                       (__attribute__((address_space(3))) void*)(buf + (bi * 2 + part) * BLK + sub * 1024),
                                       16, 0, SHARED ? 0 : 2);  // nt: each cache byte is read once
    }
  };

  f32x4 o[RT][NDT];
  float m_run[RT], l_run[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
  }

  // This wave's blocks of stage st, in two halves: scores, then online softmax and
  // O^T += V^T P^T.  Fragments: KV8 reads 8 bytes and widens them once the reads are complete.
  typedef typename std::conditional<KV8, i32x2, i32x4>::type Frag;
  auto widen = [&](Frag v) -> i32x4 {
    if constexpr (KV8) return e4m3x8_to_bf16(v, kv_sc);
    else return v;
  };
  // LDS byte offsets of the lane's fragments in a stage: key 16 t + r, step s2 and dimension
  // 16 dt + r differ from these by constants (the swizzles depend on r alone)
  uint32_t koff[NKS];
#pragma unroll
  for (int s2 = 0; s2 < NKS; ++s2) koff[s2] = lds_addr(smem) + (uint32_t)(kh * BPW * 2 * BLK + KB::koff(r, s2, grp));
  const uint32_t voff = lds_addr(smem) + (uint32_t)((kh * BPW * 2 + 1) * BLK + KB::voff(r, grp));
  f32x4 sc[RT][BPW][2];
  auto scores = [&](int st) {
    const int kb0 = blk0 + BPS * st + kh * BPW;  // this wave's first block
    if (kb0 >= blk1) return;  // wave-uniform: nothing of its blocks is visible to its rows
    const uint32_t slot = (uint32_t)((st % NBUF) * STAGE);
    Frag kr[BPW][2][NKS];
    static_for<BPW * 2 * NKS>([&](auto I) {
      constexpr int jb = decltype(I)::value / (2 * NKS), t = decltype(I)::value / NKS % 2, s2 = decltype(I)::value % NKS;
      constexpr int off = jb * 2 * BLK + t * 16 * DH * KB::ES;
      if constexpr (KV8) kr[jb][t][s2] = ds_read8<off>(koff[s2] + slot);
      else kr[jb][t][s2] = ds_read16<off>(koff[s2] + slot);
    });
    lds_wait();
#pragma unroll
    for (int jb = 0; jb < BPW; ++jb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s2 = 0; s2 < NKS; ++s2) lds_pin(kr[jb][t][s2]);
    // products of one accumulator stand 2 RT (P V: 4 RT) apart, so that none waits for the last
#pragma unroll
    for (int jb = 0; jb < BPW; ++jb) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) sc[rt][jb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s2 = 0; s2 < NKS; ++s2) {
        i32x4 kf[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          kf[t] = widen(kr[jb][t][s2]);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) sc[rt][jb][t] = mfma16x16x32(kf[t], qf[rt][s2], sc[rt][jb][t]);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) sc[rt][jb][t] = mfma16x16x32(kf[t], ql[rt][s2], sc[rt][jb][t]);
      }
    }
  };
  auto softmax_pv = [&](int st) {
    const int kb0 = blk0 + BPS * st + kh * BPW;
    if (kb0 >= blk1) return;
    const uint32_t slot = (uint32_t)((st % NBUF) * STAGE);
    Frag vr[BPW][NDT];  // requested now: the softmax below hides their latency
    static_for<BPW * NDT>([&](auto I) {
      constexpr int jb = decltype(I)::value / NDT, dt = decltype(I)::value % NDT;
      constexpr int off = jb * 2 * BLK + dt * 16 * 32 * KB::ES;
      if constexpr (KV8) vr[jb][dt] = ds_read8<off>(voff + slot);
      else vr[jb][dt] = ds_read16<off>(voff + slot);
    });
    // sc[rt][jb][t][i]: score of key 32 (kb0 + jb) + 16 t + 4 grp + i for query row r of tile rt;
    // a block at or past blk1 (beyond this wave's last key, or in the next split) counts for nothing
    if (kb0 + BPW > blk1 || 32 * (kb0 + BPW) > kmin_w) {  // wave-uniform: some key is hidden from some row
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int jb = 0; jb < BPW; ++jb)
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (kb0 + jb >= blk1 || 32 * (kb0 + jb) + 16 * t + 4 * grp + i >= kend[rt]) sc[rt][jb][t][i] = -INFINITY;
    }
    i32x4 pf[RT][BPW], pl[RT][BPW];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float mloc = -INFINITY;
#pragma unroll
      for (int jb = 0; jb < BPW; ++jb)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) mloc = fmaxf(mloc, sc[rt][jb][t][i]);
      mloc = row_max4(mloc);
      // a new maximum rescales what the rows hold; most blocks bring none (then the factor is 1)
      if (__any(mloc > m_run[rt])) {
        const float m_new = fmaxf(m_run[rt], mloc);
        // exponents are <= 0 here: the hardware exp2 suffices (results below 2^-126 flush to 0)
        const float scale = (m_run[rt] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run[rt] - m_new);
        l_run[rt] *= scale;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[rt][dt] *= scale;
        m_run[rt] = m_new;
      }
      const float m_use = m_run[rt] == -INFINITY ? 0.f : m_run[rt];  // no key so far: every score is -inf
#pragma unroll
      for (int jb = 0; jb < BPW; ++jb) {
        float p[8];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = __builtin_amdgcn_exp2f(sc[rt][jb][t][i] - m_use);
            p[4 * t + i] = v;
            l_run[rt] += v;  // this lane's keys; the row's four lanes are added at the end
          }
        // P as hi/lo bf16 (B operand): element e holds key 16*(e/4) + 4*grp + e%4.
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p0 = p[2 * e], p1 = p[2 * e + 1];
          const uint32_t hw = pack_bf2(p0, p1);
          pf[rt][jb][e] = (int)hw;
          pl[rt][jb][e] = (int)pack_bf2(p0 - __uint_as_float(hw << 16), p1 - __uint_as_float(hw & 0xffff0000u));
        }
      }
    }
    lds_wait();
#pragma unroll
    for (int jb = 0; jb < BPW; ++jb)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) lds_pin(vr[jb][dt]);
#pragma unroll
    for (int jb = 0; jb < BPW; ++jb) {
      if (kb0 + jb >= blk1) continue;  // wave-uniform
#pragma unroll
      for (int d0 = 0; d0 < NDT; d0 += 4) {
        i32x4 vf[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          vf[u] = widen(vr[jb][d0 + u]);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) o[rt][d0 + u] = mfma16x16x32(vf[u], pf[rt][jb], o[rt][d0 + u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) o[rt][d0 + u] = mfma16x16x32(vf[u], pl[rt][jb], o[rt][d0 + u]);
      }
    }
  };

  // bare s_barrier between stages: the copies are complete once this wave's vmcnt dropped
  auto bar = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  constexpr int D = NBUF - 1;  // stages ahead
  static_assert(D >= 1 && D <= 7, "ring depth");
  for (int st = 0; st < D && st < n_st; ++st) issue(st);
#pragma unroll 1
  for (int c = 0; c < n_st; ++c) {
    const int ahead = min(D - 1, n_st - 1 - c);  // later stages still in flight
    if (ahead >= 6) vm_wait<6 * PER_WAVE>();
    else if (ahead == 5) vm_wait<5 * PER_WAVE>();
    else if (ahead == 4) vm_wait<4 * PER_WAVE>();
    else if (ahead == 3) vm_wait<3 * PER_WAVE>();
    else if (ahead == 2) vm_wait<2 * PER_WAVE>();
    else if (ahead == 1) vm_wait<PER_WAVE>();
    else vm_wait<0>();
    bar();  // every wave's part of stage c is in; every wave is done with stage c - 1
    if (c + D < n_st) issue(c + D);
    scores(c);
    softmax_pv(c);
  }
  __syncthreads();  // the ring is free: it holds the other key parts' states next

#pragma unroll
  for (int t = 0; t < RT; ++t) l_run[t] = row_sum4(l_run[t]);

  // combine the key parts of each row set: parts 1 .. KP - 1 park (m, l, O), part 0 adds
  constexpr int SLOT = NDT * 16 + 16;  // bytes per lane and row tile (16-byte aligned pieces)
  auto park_of = [&](int part, int t) { return smem + ((((part - 1) * NRS + rs) * RT + t) * 64 + lane) * SLOT; };
  if (kh > 0) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      char* park = park_of(kh, t);
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) *(f32x4*)(park + dt * 16) = o[t][dt];
      *(float*)(park + NDT * 16) = m_run[t];
      *(float*)(park + NDT * 16 + 4) = l_run[t];
    }
  }
  __syncthreads();
  if (kh > 0) return;
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (!row_ok[t]) continue;
    float mm = m_run[t];
#pragma unroll
    for (int part = 1; part < KP; ++part) mm = fmaxf(mm, *(const float*)(park_of(part, t) + NDT * 16));
    const float s0 = (m_run[t] == -INFINITY) ? 0.f : exp2f(m_run[t] - mm);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[t][dt] *= s0;
    float ll = l_run[t] * s0;
#pragma unroll
    for (int part = 1; part < KP; ++part) {
      const char* park = park_of(part, t);
      const float mp = *(const float*)(park + NDT * 16), lp = *(const float*)(park + NDT * 16 + 4);
      const float sp_ = (mp == -INFINITY) ? 0.f : exp2f(mp - mm);
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) o[t][dt] += *(const f32x4*)(park + dt * 16) * sp_;
      ll += lp * sp_;
    }
    if (a.n_splits == 1) {  // the whole key range: normalise and store the output (no merge launch)
      const float inv = 1.0f / ll;
      const int64_t orow = (int64_t)b * k + jr[t];
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        i32x2 hi, lo;
        split_bf16x4(o[t][dt] * inv, hi, lo);
        const int64_t dst = aoff(orow, (int64_t)hq[t] * DH + 16 * dt + 4 * grp, (int64_t)a.n_q * DH, a.out_mtiles);
        *(i32x2*)(a.out + dst) = hi;
        *(i32x2*)(a.out_lo + dst) = lo;
      }
      continue;
    }

    // the split's unnormalised (max, sum, O) per row, as attn_split_body leaves them
    const int64_t item = (int64_t)(b * k + jr[t]) * a.n_q + hq[t];
    const int64_t n_items = (int64_t)a.B * k * a.n_q;
    if (grp == 0) {
      float* ml = a.part_ml + ((int64_t)split * n_items + item) * 2;
      ml[0] = mm;
      ml[1] = ll;
    }
    const int64_t po = ((int64_t)split * n_items + item) * DH;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) *(f32x4*)(a.part_o + po + 16 * dt + 4 * grp) = o[t][dt];
  }
}

template <int DH>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
  const int64_t n_items = (int64_t)a.B * a.k * a.n_q;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= n_items) return;
  attn_merge_body<DH, false>(a, item);
}

// Shared keys (SRT) from four row blocks that take the whole key range each: with fewer, most
// keys come from HBM once all the same.  Two row tiles per wave halve the workgroups and make each
// about 1.75 times as long, so one tile is better while half the workgroups leave CUs idle.  Where
// the two meet depends on how unequal the workgroups' ranges are, and the line at 1.5 rounds of
// one-tile workgroups lies between what is best for each (one tile, two, us; W workgroups of one
// tile).  Prompts from their start: 768 rows (W 384) 29.5, 32.6, 960 36.7, 39.5, 1024 42.8, 41.6;
// 1024 rows behind 1024 78, 71.  Blocks of 64 rows, sequences of 250 to 2000 keys: 9 of them (W 288)
// 41, 65, 14 76, 71, 20 75, 75; of 2000 keys each: 8 28, 43, 9 82, 69, 16 90, 78, 20 129, 145.  Equal
// ranges from 1 to 1.5 rounds and from 2 to 3 would be 12 to 17 % better the other way.
template <int DH, bool KV8>
static void launch_split_rs(const AttnArgs& a, dim3 grid, const Exec& ex) {
  const int64_t wgs = (int64_t)a.n_kv * a.n_rowblocks * a.B;
  // a row block of at most 32 rows (one block: n_rowblocks == 1) takes two row sets
  if ((a.n_q / a.n_kv) * a.k <= 32 && a.n_rowblocks == 1)
    SBD_KLAUNCH((attn_split_kernel<DH, KV8, 2, 0>), grid, dim3(512), ex, a);
  else if (a.n_splits > 1 || a.n_rowblocks < 4)
    SBD_KLAUNCH((attn_split_kernel<DH, KV8, 4, 0>), grid, dim3(512), ex, a);
  else if (wgs <= kAttnCus * 3 / 2)
    SBD_KLAUNCH((attn_split_kernel<DH, KV8, 4, 1>), dim3(a.n_kv * a.n_rowblocks, 1, a.B), dim3(512), ex, a);
  else
    SBD_KLAUNCH((attn_split_kernel<DH, KV8, 4, 2>), dim3(a.n_kv * ((a.n_rowblocks + 1) / 2), 1, a.B), dim3(512), ex, a);
}

hipError_t launch_attention_split(const AttnArgs& a, const Exec& ex) {
  dim3 grid(a.n_splits, a.n_kv * a.n_rowblocks, a.B);
  if (a.d_h == 128 && a.kv_fp8)
    launch_split_rs<128, true>(a, grid, ex);
  else if (a.d_h == 128)
    launch_split_rs<128, false>(a, grid, ex);
  else if (a.d_h == 64 && a.kv_fp8)
    launch_split_rs<64, true>(a, grid, ex);
  else if (a.d_h == 64)
    launch_split_rs<64, false>(a, grid, ex);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_attention_merge(const AttnArgs& a, const Exec& ex) {
  const int64_t n_items = (int64_t)a.B * a.k * a.n_q;
  dim3 grid((unsigned)((n_items + 3) / 4));
  if (a.d_h == 128)
    SBD_KLAUNCH(attn_merge_kernel<128>, grid, dim3(256), ex, a);
  else if (a.d_h == 64)
    SBD_KLAUNCH(attn_merge_kernel<64>, grid, dim3(256), ex, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace sbd
