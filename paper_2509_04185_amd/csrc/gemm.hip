// Weight-streaming GEMM for M > 16 rows: y[m][n] = sum_k A[m][k] W[n][k].
//
// Weights are repacked once (pack_kernel) into MFMA fragment order.  A matrix with N rows
// and K columns is cut into 16-row tiles; the 16-byte piece of lane l in step s of tile t
// holds W[16t + l%16][32s + 8(l/16) .. +8], so one 16-byte load per lane reads a 1 KB
// fragment in the B-operand order of v_mfma_f32_16x16x32_bf16.  Tiles are grouped by 8
// (128 rows) and a group's 8 fragments of one step are stored together:
// [N/128 groups][K/32 steps][8 tiles][64 lanes][8] (packed_frag() in sbd_device.h).  The
// gate and up projections share one packed matrix whose tile t holds gate rows 8t..8t+7
// followed by up rows 8t..8t+7, so SwiGLU pairs stay inside one tile.
//
// This kernel serves the block forwards of several sequences (M = batch * k up to a few
// hundred rows) and the prefill chunks; decode-sized products (M <= 16) go through
// gemv.hip.  At these M every projection still reads far more weight bytes than it does
// MFMA work per byte (M flop per weight byte, against a ridge of ~300), so the design
// streams every weight byte from HBM once:
//   - A workgroup owns a column block of NT tiles (8, 12, 14 or 16: gemm_plan) and a row block of
//     MT tiles (up to 128 rows; larger M is cut into row blocks that run on the same XCD
//     and meet the same weights in its L2), and a range of K steps.
//   - Eight waves: four load, four multiply, one of each on a SIMD.  The loading waves bring
//     weights and activations straight into LDS (global_load_lds, no registers) in stages of
//     one K step, a ring of NS stages; the multiplying waves split the block into column
//     halves x row halves, read their weight fragments and the A fragments (hi and lo) of
//     their rows from LDS and run two MFMAs per pair.  A wave issues in order and a load waits
//     for room in the memory pipeline at its issue, so a wave that also loads leaves its
//     matrix core idle for as long; with four waves doing both, gate/up at M = 256 took
//     117 us (Llama 8B, 28672 x 4096; 72 us of it MFMAs), M = 128 (Qwen 8B, 24576 x 4096)
//     67 us, and with the loads on waves of their own 98 and 56 us; chained launches over
//     rotating weights.  Spreading the same loads and reads between the MFMAs of one wave
//     gave 111 and 74 us; separate rings for weights and activations with up to 14 stages of
//     weights in flight gained nothing more (94 and 57 us; slower at M <= 64).
//   - The LDS reads of a row tile's activations are issued one row tile ahead, and a quarter
//     of the next stage's weight fragments with each, between the MFMAs, so the matrix cores
//     wait for nothing but the stage barrier.
//   - When there are too few column blocks to fill the chip, K is split over workgroups
//     of one XCD, all resident at once (plans of one round): each parks its partial tiles
//     in that XCD's L2 and waits for the others, then adds the slices of a share of the row
//     tiles in slice order (deterministic) and runs their epilogue, so the finishing work
//     of a unit is spread over its slices, and in a slice over its four multiplying waves
//     (each a quarter of a row tile's columns, all slices' pieces in flight at once: O
//     projection at M = 32 13.4 -> 11.5 us with the loading waves, 12.4 without this).
// Epilogues (acc in the MFMA D layout: lane l holds column l % 16 of a tile, rows
// 4*(l/16) + i):
//   EPI_SCALED_STORE  out = rinv[m] * y           (QKV projection, LM head)
//   EPI_LOGITS_EB     the same (stores optional) plus the EB softmax statistics of every
//                     row's 64-column chunks (LM head; eb_stats.h)
//   EPI_RESID         x += y; xn = x * g_next as hi/lo; the sum of x^2 over the block's
//                     columns per row (O and down projections: residual add, the next
//                     RMSNorm's inputs)
//   EPI_SWIGLU        act = silu(rinv*gate) * rinv*up as hi/lo (gate/up projection)
// RMSNorm is split across two kernels: the producer writes x * g (gain applied) plus
// partial sums of squares; the consumer adds the partials of a row and scales its fp32
// result by 1/sqrt(mean(x^2) + eps), which equals normalising the input first because the
// scale is constant along a row.

#include <algorithm>
#include <type_traits>

#include "eb_stats.h"

namespace sbd {

template <int MT, int NT, bool W8>
struct MidCfg {
  // multiplying waves across the column block: 2 x 2 waves (each reads half the activation and half
  // the weight fragments of a stage from LDS: 16 KB per 16-tile stage, against 20 KB in a 4 x 1 split)
  static constexpr int WC = 2;
  static constexpr int WM = 4 / WC;            // waves across the row block
  static constexpr int CW = NT / WC;           // tiles per wave
  static constexpr int MTW = MT / WM;          // row tiles per wave
  // weight bytes of a K step: 1 KB per tile in bf16, 512 B in e4m3 (one 1 KB wave-load then
  // carries two tiles' fragments)
  static constexpr int WB = NT * (W8 ? 512 : 1024);
  static constexpr int NWL = WB / 1024;               // weight wave-loads per stage
  static constexpr int NWU = (NWL + 3) / 4;           // of each loading wave (past the last: read again)
  static constexpr int STAGE = NWU * 4096 + 2 * MT * 1024;  // one K step: weights + 2 MT A fragments
  static constexpr int NS = (144 * 1024) / STAGE > 8 ? 8 : (144 * 1024) / STAGE;  // ring stages
  static constexpr int FPW = NWU + MT / 2;            // wave-loads of each loading wave per stage, weights first
  static_assert(MTW >= 1 && MT % 2 == 0 && CW * WC == NT, "unsupported tile shape");
  static_assert(NS >= 3 && (NS - 1) * FPW <= 63, "vmcnt range");
};

// Wait until at most n stages of FPW loads each are still in flight (n in [0, NMAX]).
template <int FPW, int NMAX>
__device__ __forceinline__ void vm_wait_stages(int n) {
  if constexpr (NMAX > 0) {
    if (n >= NMAX) {
      vm_wait<NMAX * FPW>();
      return;
    }
    vm_wait_stages<FPW, NMAX - 1>(n);
  } else {
    vm_wait<0>();
  }
}

// Value of an XCD-local counter, read with an atomic (a load could be served by the CU's own
// L1); the zero comes from an instruction the compiler cannot see through, so the atomic
// stays one.
__device__ __forceinline__ int ctr_peek(int* ctr) {
  int zero;
  asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
  return __hip_atomic_fetch_add(ctr, zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The K slices of a unit (all on one XCD, all resident) wait until every one has parked its
// partials: word 0 of the unit's counter line counts arrivals, word 1 departures, and the
// last to depart resets both for the next launch.  The wait is bounded: one that gives up
// raises the sticky error and the workgroup goes on (its results are then wrong, and the
// next API call reports it).
__device__ __forceinline__ void slices_arrived(const GemmArgs& a, int* ctr, int ks, int what) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores have reached the L2
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    int it = 0;
    while (ctr_peek(ctr) < ks) {
      __builtin_amdgcn_s_sleep(1);
      if (++it > a.spin_limit) {
        atomicOr(a.err, 1);
        atomicExch(a.err + 1, what);
        if (a.err_host != nullptr) {
          __hip_atomic_store(a.err_host + 1, what, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          __hip_atomic_store(a.err_host, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        break;
      }
    }
    if (__hip_atomic_fetch_add(ctr + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == ks - 1) {
      __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_store(ctr + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  __syncthreads();
}

// FOLD: every K step's products of a tile (hi and lo, two MFMAs from zero) are added to its sum
// with ordinary fp32 additions, instead of 2 K / 32 MFMAs accumulating in a row.  The MFMA does
// not round its sum to nearest, and the error of such a chain grows with its length: the keys
// and values of an unsplit QKV projection (K = 4096, 256 MFMAs in a row) round to another bf16
// than the exact ones 1.6 times as often as with five K slices (Qwen 8B prefill of 2048, four
// layers, against float64: keys 5.8e-4 unsplit, 4.6e-4 in slices, 4.4e-4 with FOLD; logits
// 1.5e-4, 0.91e-4, 0.91e-4), while the other projections' chains make no difference (logits
// 0.91e-4 with or without).  It costs two additions per MFMA, 17 % of the kernel at 1024 rows
// (QKV of Llama 8B 91 -> 107 us in 16-tile blocks), so only the QKV projection of prefill
// chunks of more than 256 rows, which need no K slices to fill the chip, takes it.
// SPLIT: K is split over a.splits workgroups (kernels of their own: without the other case's
// epilogue the accumulators are dead once parked, and the slices' sums get their registers).
// W8: the weights are e4m3 bytes (a.Wp8, per-row scales a.wscale) in the same packing, one
// byte per element; a fragment is widened to the bf16 MFMA operand (times its row's scale,
// exact) after its LDS read, so the products are those of the widened bf16 matrix.
template <int MT, int NT, int EPI, bool W8, bool SPLIT, bool FOLD>
__global__ __launch_bounds__(512) void gemm_kernel(GemmArgs a) {
  using Cfg = MidCfg<MT, NT, W8>;
  constexpr int WC = Cfg::WC, CW = Cfg::CW, MTW = Cfg::MTW, NS = Cfg::NS, FPW = Cfg::FPW;
  constexpr int STAGE = Cfg::STAGE;
  constexpr int WB = Cfg::NWU * 4096;  // weight bytes of a stage; A fragments follow
  constexpr int NWU = Cfg::NWU;
  typedef typename std::conditional<W8, i32x2, i32x4>::type WFr;  // a weight fragment in registers
  __shared__ __attribute__((aligned(16))) char smem[NS * STAGE];
  __shared__ float rinv_s[MT * 16];
  __shared__ float ssq_s[4][MT * 16];
  __shared__ double exp_tab[EPI == EPI_LOGITS_EB ? 32 : 1];

  const int lane = threadIdx.x & 63, w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w = w8 & 3;
  const int r = lane & 15, g = lane >> 4;
  const int wc = w % WC, wm = w / WC;

  // Workgroup i runs on XCD i % 8; the m_blocks x splits units of column block cb all sit
  // on XCD cb % 8.  The count is padded to a multiple of 8; padding workgroups leave.
  const int KS = a.splits, MB = a.m_blocks, P = KS * MB;
  const int jx = (int)(blockIdx.x >> 3);
  const int cb = (jx / P) * 8 + (int)(blockIdx.x & 7);
  // a last column block may be half full (n_tiles % NT == 8, LM head with bf16 weights and
  // two waves across the block: the second wave's tiles are past the end)
  const int n_cb = (a.n_tiles + NT - 1) / NT;
  if (cb >= n_cb) return;
  const int mb = (jx % P) / KS, kc = (jx % P) % KS;
  const int uid = cb * MB + mb;
  const int row0 = mb * MT * 16;
  const int S_all = a.K / 32;
  const int s_b = (int)((int64_t)S_all * kc / KS), s_e = (int)((int64_t)S_all * (kc + 1) / KS);
  const int nst = s_e - s_b;
  const int t0 = cb * NT;

  // Barrier between stages.  It waits for nothing of the wave's own: a loading wave has waited for
  // the stage that its barrier hands over, and a multiplying wave's LDS reads of a stage are
  // complete at the lds_wait of its last row tile, before it comes to the next barrier.  The empty
  // asm statements keep the compiler from moving LDS accesses across it.
  auto bar = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (w8 >= 4) {
    // ---- loading wave: load u of a stage fills 1 KB f = w + 4u of it; for u < NWU weight tile
    // t0 + f (bf16) or the tiles t0 + 2f, t0 + 2f + 1 (e4m3: their fragments are adjacent in
    // the packing; f past the last re-reads it), else A fragment f - 4 NWU = 2 * (row tile) +
    // (0: hi, 1: lo).
    constexpr int64_t kWStep = W8 ? kPackStep : kPackStep * 2;
    const char* src[FPW];
    const int64_t a_step = (int64_t)a.a_mtiles * 1024;
#pragma unroll
    for (int u = 0; u < FPW; ++u) {
      const int f = w + 4 * u;
      if (u < NWU) {
        if constexpr (W8) {
          src[u] = (const char*)(a.Wp8 + packed_frag(t0 + 2 * min(f, Cfg::NWL - 1), s_b, S_all)) + lane * 16;
        } else {
          // a half-full block's tiles past the end read the last tile (results discarded)
          constexpr bool kHalf = EPI == EPI_SCALED_STORE || EPI == EPI_LOGITS_EB;
          const int t = t0 + min(f, Cfg::NWL - 1);
          src[u] = (const char*)(a.Wp + packed_frag(kHalf ? min(t, a.n_tiles - 1) : t, s_b, S_all)) + lane * 16;
        }
      } else {
        const int ai = f - 4 * NWU;
        const int row = min(row0 + (ai >> 1) * 16 + r, a.M - 1);  // rows past the end: valid data, results discarded
        src[u] = (const char*)(((ai & 1) ? a.A_lo : a.A) + apack(a.a_row0 + row, (int64_t)s_b * 32 + g * 8, a.a_mtiles));
      }
    }
    int slot = w * 1024;
    auto issue = [&](auto NT_) {
      constexpr int kPolW = decltype(NT_)::value ? 2 : 0;  // nt: read once
#pragma unroll
      for (int u = 0; u < FPW; ++u) {
        if (u < NWU)
          __builtin_amdgcn_global_load_lds((const void*)src[u], (__attribute__((address_space(3))) void*)(smem + slot + u * 4096), 16, 0, kPolW);
        else
          __builtin_amdgcn_global_load_lds((const void*)src[u], (__attribute__((address_space(3))) void*)(smem + slot + u * 4096), 16, 0, 0);
        src[u] += u < NWU ? kWStep : a_step;
      }
      slot = slot + STAGE >= NS * STAGE ? slot + STAGE - NS * STAGE : slot + STAGE;
    };
    auto load = [&](auto NT_) {
#pragma unroll 1
      for (int st = 0; st < NS && st < nst; ++st) issue(NT_);
      vm_wait_stages<FPW, NS - 1>(min(NS - 1, nst - 1));  // stage 0 has landed
      bar();
      // barrier c: stage c + 1 has landed; every wave is done with stage c - 1, whose slot
      // takes stage c - 1 + NS
#pragma unroll 1
      for (int c = 0; c + 1 < nst; ++c) {
        vm_wait_stages<FPW, NS - 2>(min(nst, max(NS, c - 1 + NS)) - 2 - c);
        bar();
        if (c >= 1 && c - 1 + NS < nst) issue(NT_);
      }
    };
    // one row block: every weight byte is read by one workgroup, non-temporal
    if (MB == 1) load(std::true_type{});
    else load(std::false_type{});
    return;  // a wave that has ended no longer counts at the workgroup's barriers
  }

  f32x4 acc[MTW][CW];
#pragma unroll
  for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
    for (int cw = 0; cw < CW; ++cw) acc[mw][cw] = f32x4{0.f, 0.f, 0.f, 0.f};

  // LDS reads of a stage with ds_read16 (sbd_device.h): the compiler would otherwise guard
  // every read of LDS with a wait for all direct loads in flight (it cannot tell the ring
  // slots apart), draining the ring at each step.  Ordering is explicit instead: the barrier
  // before the reads, a wait after them, and the results pinned behind it.  The
  // weights of a stage are read during the stage before (two register sets), its activations
  // one row tile ahead, so LDS reads overlap the matrix work.
  constexpr int WFB = W8 ? 512 : 1024;  // bytes of one weight fragment in LDS
  const uint32_t lds_w = (uint32_t)(uintptr_t)smem + (uint32_t)(wc * CW * WFB + lane * (WFB / 64));
  const uint32_t lds_a = (uint32_t)(uintptr_t)smem + (uint32_t)(WB + wm * MTW * 2048 + lane * 16);
  // the lane's weight scales (row r of each of its tiles); 1 for bf16
  float wsc[CW];
#pragma unroll
  for (int cw = 0; cw < CW; ++cw) wsc[cw] = W8 ? a.wscale[(int64_t)(t0 + wc * CW + cw) * 16 + r] : 1.0f;
  int rslot = 0;  // ring slot (bytes) of the current stage
  // Consumers of a norm: the producer's partial sums of squares of this block's rows,
  // requested before the stream (thread t adds partials of row t / TPR, float4 at a time).
  constexpr int TPR = 256 / (MT * 16);
  constexpr int NPRE = 4;
  const int rr_t = threadIdx.x / TPR, q_t = threadIdx.x % TPR;
  const int m_t = row0 + rr_t;
  const bool norm_in = EPI != EPI_RESID && a.sumsq_in != nullptr;
  const bool vec4 = (a.n_part & 3) == 0;
  const int n4 = a.n_part >> 2;
  const f32x4* prow = reinterpret_cast<const f32x4*>(a.sumsq_in + (int64_t)min(m_t, a.M - 1) * a.n_part);
  f32x4 pre[NPRE];
#pragma unroll
  for (int j = 0; j < NPRE; ++j) {
    const int p4 = q_t + j * TPR;
    pre[j] = (norm_in && vec4 && m_t < a.M && p4 < n4) ? prow[p4] : f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // The epilogue's share of a wave.  One slice: the wave's own accumulators, CW tiles of MTW
  // row tiles.  Split: a quarter of the columns of each of the slice's row tiles (a half of
  // every second one for EB statistics, whose 64-column chunks stay inside one wave, and for
  // blocks of 14 tiles).
  constexpr bool kQuarter = SPLIT && EPI != EPI_LOGITS_EB && NT % 4 == 0;
  constexpr int CWE = kQuarter ? NT / 4 : CW;   // tiles of a row tile
  constexpr int CPR = CWE * 4;                  // float4 pieces of a row
  constexpr int NPASS = 16 * CPR / 64;          // read-back passes per row tile
  const int ct0 = kQuarter ? w * CWE : wc * CW;  // first tile in the block
  const int n_w0 = (t0 + ct0) * 16;              // first output column
  const int n_l = n_w0 + (lane % CPR) * 4;
  f32x4 xcur[NPASS], xnxt[NPASS];
  i32x2 gw{0, 0};
  // EPI_RESID: a lane's residual pieces of the next row tile are requested before the stores
  // of the current one; the gain is the same for every row of the lane
  auto load_x = [&](int rt, f32x4(&xv)[NPASS]) {
#pragma unroll
    for (int j = 0; j < NPASS; ++j) {
      const int m = row0 + rt * 16 + (j * 64 + lane) / CPR;
      xv[j] = *(const f32x4*)(a.x + (int64_t)min(m, a.M - 1) * a.ldx + n_l);  // rows past the end: never stored
    }
  };
  if constexpr (SPLIT && EPI == EPI_RESID) {  // the first row tile's, ahead of the stream: nothing of these depends on it
    gw = *(const i32x2*)(a.g_next + n_l);
    load_x(min(kc, MT - 1), xcur);
  }

  WFr wv0[CW], wv1[CW];
  i32x4 av[2][2];  // [row tile parity][hi, lo]
  bar();  // stage 0 is in
  static_for<CW>([&](auto I) {
    constexpr int i = decltype(I)::value;
    if constexpr (W8) wv0[i] = ds_read8<i * 512>(lds_w);
    else wv0[i] = ds_read16<i * 1024>(lds_w);
  });
  av[0][0] = ds_read16<0>(lds_a);
  av[0][1] = ds_read16<1024>(lds_a);
  lds_wait();
#pragma unroll
  for (int i = 0; i < CW; ++i) lds_pin(wv0[i]);
  lds_pin(av[0][0]);
  lds_pin(av[0][1]);
  constexpr int WPM = (CW + MTW - 1) / MTW;  // weight reads per row tile
  // step cc: MFMAs of stage cc; every accumulator takes hi, then lo (e4m3 fragments are
  // widened once per row tile).  P0: parity of the register pair holding row tile 0.
  f32x4 fold[2][2];                  // FOLD: a step's products of two pairs of tiles
  float facc[FOLD ? MTW : 1][CW][4];  // and the sums (single floats: as vectors they spill)
#pragma unroll
  for (int mw = 0; mw < (FOLD ? MTW : 1); ++mw)
#pragma unroll
    for (int cw = 0; cw < CW; ++cw)
#pragma unroll
      for (int e = 0; e < 4; ++e) facc[mw][cw][e] = 0.f;
  i32x4 wide[W8 ? CW : 1];           // e4m3: the step's widened fragments (FOLD), or one
  if constexpr (FOLD) fold[1][0] = fold[1][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](auto P0, int cc, WFr (&wc_)[CW], WFr (&wn)[CW]) {
    if (cc + 1 < nst) bar();
    const int nslot = rslot + STAGE == NS * STAGE ? 0 : rslot + STAGE;
    __builtin_amdgcn_sched_barrier(0);
    static_for<MTW>([&](auto MW) {
      constexpr int mw = decltype(MW)::value, p = (mw + decltype(P0)::value) & 1, q = p ^ 1;
      constexpr int wleft = CW - mw * WPM, nw = wleft < 0 ? 0 : (wleft < WPM ? wleft : WPM);  // weight reads here
      constexpr bool kNext = mw + 1 == MTW;
      constexpr int NM = 2 * CW;
      static_for<NM>([&](auto I) {
        constexpr int i = decltype(I)::value;
        // reads: the next row tile's hi and lo, then this row tile's share of the next stage's weights
        if constexpr (i == 0) av[q][0] = kNext ? ds_read16<0>(lds_a + nslot) : ds_read16<(mw + 1) * 2048>(lds_a + rslot);
        if constexpr (i == 1) av[q][1] = kNext ? ds_read16<1024>(lds_a + nslot) : ds_read16<(mw + 1) * 2048 + 1024>(lds_a + rslot);
        if constexpr (i >= 2 && i < 2 + WPM && mw * WPM + i - 2 < CW) {
          constexpr int x = mw * WPM + i - 2;
          if constexpr (W8) wn[x] = ds_read8<x * 512>(lds_w + nslot);
          else wn[x] = ds_read16<x * 1024>(lds_w + nslot);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FOLD) {
          // tiles in pairs: lo, lo, hi, hi into fresh registers; meanwhile the pair before is
          // added (the pairs of a step alternate between two register sets: pn is even)
          constexpr int pn = mw * (CW / 2) + i / 4, cw = (i / 4) * 2 + i % 2, h = 1 - (i % 4) / 2, par = pn & 1;
          constexpr int pv = (pn + MTW * CW / 2 - 1) % (MTW * CW / 2), pmw = pv / (CW / 2), pcw = (pv % (CW / 2)) * 2;
          if constexpr (W8) {
            if constexpr (mw == 0 && h == 1) wide[cw] = e4m3x8_to_bf16(wc_[cw], wsc[cw]);
            fold[par][i % 2] = mfma16x16x32(av[p][h], wide[cw], h ? f32x4{0.f, 0.f, 0.f, 0.f} : fold[par][i % 2]);
          } else {
            fold[par][i % 2] = mfma16x16x32(av[p][h], wc_[cw], h ? f32x4{0.f, 0.f, 0.f, 0.f} : fold[par][i % 2]);
          }
          constexpr int e0 = (i % 2) * 2, ft = (i % 4) / 2;  // two of the eight additions
          facc[pmw][pcw + ft][e0] += fold[par ^ 1][ft][e0];
          facc[pmw][pcw + ft][e0 + 1] += fold[par ^ 1][ft][e0 + 1];
        } else if constexpr (W8) {
          constexpr int cw = i / 2, h = i % 2;
          if constexpr (h == 0) wide[0] = e4m3x8_to_bf16(wc_[cw], wsc[cw]);
          acc[mw][cw] = mfma16x16x32(av[p][h], wide[0], acc[mw][cw]);
        } else {
          constexpr int h = i / CW, cw = i % CW;
          acc[mw][cw] = mfma16x16x32(av[p][h], wc_[cw], acc[mw][cw]);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (kNext) {
        lds_wait();
#pragma unroll
        for (int i = 0; i < CW; ++i) lds_pin(wn[i]);
      } else {
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"i"(nw) : "memory");
      }
      lds_pin(av[q][0]);
      lds_pin(av[q][1]);
    });
    rslot = nslot;
  };
#pragma unroll 1
  for (int c = 0; c < nst; c += 2) {
    step(std::integral_constant<int, 0>{}, c, wv0, wv1);
    if (c + 1 < nst) step(std::integral_constant<int, MTW & 1>{}, c + 1, wv1, wv0);
  }

  if constexpr (FOLD) {  // the last step's last pair
    static_assert(MTW * CW % 4 == 0, "an even number of pairs per step");
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
      for (int cw = 0; cw < CW; ++cw)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[mw][cw][e] = facc[mw][cw][e];
    acc[MTW - 1][CW - 2] += fold[1][0];
    acc[MTW - 1][CW - 1] += fold[1][1];
  }

  // ---- K split over workgroups (a plan of one round: every slice of a unit is resident):
  // each slice parks its partial tiles and waits for the others; the epilogue then adds the
  // slices of the row tiles kc, kc + KS, ... of the block in slice order and finishes them
  // (every output is the same sum of the same slices, whichever slice finishes it).
  auto own = [&](int rt) { return !SPLIT || rt % KS == kc; };
  const int64_t zstride = (int64_t)n_cb * MB * 4 * MTW * CW;       // 1 KB (64 x f32x4) pieces per slice
  const int64_t uslot = (int64_t)uid * 4 * (MTW * CW);
  if constexpr (SPLIT) {
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw)
#pragma unroll
      for (int cw = 0; cw < CW; ++cw)
        *(f32x4*)(a.part + ((kc * zstride + uslot + (w * MTW + mw) * CW + cw) * 64 + lane) * 4) = acc[mw][cw];
    slices_arrived(a, a.counters + (int64_t)uid * kCtrStride, KS, 65536 + EPI);
  } else if constexpr (EPI == EPI_RESID) {
    gw = *(const i32x2*)(a.g_next + n_l);
    load_x(wm * MTW, xcur);
  }

  if constexpr (EPI == EPI_LOGITS_EB) exp_table_stage(exp_tab, threadIdx.x);  // read past the barrier below

  // ---- 1/rms of the block's rows (partials beyond the prefetched ones read here)
  if constexpr (EPI != EPI_RESID) {
    float sq = 0.f;
    if (norm_in && m_t < a.M) {
      if (vec4) {
#pragma unroll
        for (int j = 0; j < NPRE; ++j) sq += (pre[j][0] + pre[j][1]) + (pre[j][2] + pre[j][3]);
        for (int p4 = q_t + NPRE * TPR; p4 < n4; p4 += TPR) {
          const f32x4 v = prow[p4];
          sq += (v[0] + v[1]) + (v[2] + v[3]);
        }
      } else {
        for (int p = q_t; p < a.n_part; p += TPR) sq += a.sumsq_in[(int64_t)m_t * a.n_part + p];
      }
    }
#pragma unroll
    for (int o = TPR / 2; o >= 1; o /= 2) sq += __shfl_xor(sq, o);
    if (q_t == 0) rinv_s[rr_t] = norm_in ? 1.0f / sqrtf(sq * a.inv_d + a.eps) : 1.0f;
  }
  __syncthreads();  // rinv_s written; every wave is past the ring, which now stages results

  // ---- epilogue.  Each wave passes its tiles through LDS one row tile at a time (16 rows x
  // 16 CWE columns, rows padded by 4 floats), then lanes own 4 consecutive columns of a row:
  // a row's 16 CWE columns are written by consecutive lanes as whole 16-byte pieces.
  constexpr int LDR = CWE * 16 + 4;  // staged row length (floats)
  float* stg = reinterpret_cast<float*>(smem) + w * 16 * LDR;
  // false only for the empty half of a half-full block (an LM head's last block)
  const bool cols_in = (EPI != EPI_SCALED_STORE && EPI != EPI_LOGITS_EB) || n_w0 < a.n_tiles * 16;
  auto finish = [&](int rt, const f32x4 (&y_)[CWE], const f32x4 (&xv_)[NPASS]) {
    const int rl0 = rt * 16;  // first local row of the row tile
#pragma unroll
    for (int cw = 0; cw < CWE; ++cw)
#pragma unroll
      for (int i = 0; i < 4; ++i) stg[(4 * g + i) * LDR + cw * 16 + r] = y_[cw][i];
    if constexpr (EPI == EPI_SWIGLU) {
      // task: (row, tile tt, half h) -> act columns 8 (tile) + 4 h .. + 3
      constexpr int NT2 = 16 * CWE * 2;
#pragma unroll
      for (int j = 0; j < (NT2 + 63) / 64; ++j) {
        const int idx = j * 64 + lane;
        const int row = idx / (CWE * 2), tt = (idx % (CWE * 2)) >> 1, h = idx & 1;
        const int m = row0 + rl0 + row;
        if (idx < NT2 && m < a.M) {
          const f32x4 gt = *(const f32x4*)(stg + row * LDR + tt * 16 + h * 4);
          const f32x4 up = *(const f32x4*)(stg + row * LDR + tt * 16 + 8 + h * 4);
          const float rv = rinv_s[rl0 + row];
          f32x4 y;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float gv = gt[e] * rv;
            y[e] = gv / (1.0f + expf(-gv)) * (up[e] * rv);
          }
          i32x2 hi, lo;
          split_bf16x4(y, hi, lo);
          const int64_t o = aoff(m, (int64_t)(t0 + ct0 + tt) * 8 + h * 4, a.ld_act, a.o_mtiles);
          *(i32x2*)(a.act + o) = hi;
          *(i32x2*)(a.act_lo + o) = lo;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < NPASS; ++j) {
        const int idx = j * 64 + lane;
        const int row = idx / CPR, pc = idx % CPR;
        const int m = row0 + rl0 + row;
        const int n = n_w0 + pc * 4;
        const f32x4 y = *(const f32x4*)(stg + row * LDR + pc * 4);
        if constexpr (EPI == EPI_SCALED_STORE) {
          if (m < a.M) *(f32x4*)(a.out_f32 + (int64_t)m * a.ldo + n) = y * rinv_s[rl0 + row];
        } else if constexpr (EPI == EPI_LOGITS_EB) {
          if (m < a.M && a.out_f32 != nullptr) *(f32x4*)(a.out_f32 + (int64_t)m * a.ldo + n) = y * rinv_s[rl0 + row];
        } else {  // EPI_RESID
          float s2 = 0.f;
          if (m < a.M) {
            const f32x4 xv = xv_[j] + y;
            *(f32x4*)(a.x + (int64_t)m * a.ldx + n) = xv;
            f32x4 xg;
            xg[0] = xv[0] * __uint_as_float((uint32_t)gw[0] << 16);
            xg[1] = xv[1] * __uint_as_float((uint32_t)gw[0] & 0xffff0000u);
            xg[2] = xv[2] * __uint_as_float((uint32_t)gw[1] << 16);
            xg[3] = xv[3] * __uint_as_float((uint32_t)gw[1] & 0xffff0000u);
            i32x2 hi, lo;
            split_bf16x4(xg, hi, lo);
            const int64_t on = aoff(m, n, a.ldx, a.o_mtiles);
            *(i32x2*)(a.xn + on) = hi;
            *(i32x2*)(a.xn_lo + on) = lo;
            s2 = (xv[0] * xv[0] + xv[1] * xv[1]) + (xv[2] * xv[2] + xv[3] * xv[3]);
          }
#pragma unroll
          for (int o = 1; o < CPR; o <<= 1) s2 += __shfl_xor(s2, o);  // the row's CPR lanes
          if (pc == 0) ssq_s[kQuarter ? w : wc][rl0 + row] = s2;
        }
      }
    }
    if constexpr (EPI == EPI_LOGITS_EB) {
      // the staged row tile again: lane L reduces VPL = 4 CW consecutive columns of row L / 4,
      // 16 / CW lanes per 64-column chunk
      constexpr int VPL = 4 * CW, LPC = 16 / CW;
      static_assert(VPL * LPC == kEbFChunk, "a chunk is 64 columns");
      const int row = lane >> 2, seg = lane & 3;
      const int m = row0 + rl0 + row;
      const int col0 = n_w0 + seg * VPL;
      float mx;
      int arg;
      double z, sz;
      eb_seg_stats<VPL, LPC>(stg + row * LDR + seg * VPL, rinv_s[rl0 + row], col0, a.eb_mask_id, exp_tab, mx,
                             arg, z, sz);
      if (seg % LPC == 0 && m < a.M) eb_chunk_store(a.eb_part, a.eb_arg, a.eb_chunks, m, col0 / kEbFChunk, mx, arg, z, sz);
    }
  };
  if constexpr (SPLIT) {
    const __amdgpu_buffer_rsrc_t rp = buf_rsrc(a.part);
    // the slices' sum of this wave's tiles of row tile rt: NZ slices' pieces in flight at once
    // (indices past the last slice re-read it), added in slice order
    auto add_slices = [&](auto NZ_, int rt, int z0, f32x4 (&sum)[CWE]) {
      constexpr int NZ = decltype(NZ_)::value;
      i32x4 v[NZ][CWE];
#pragma unroll
      for (int zz = 0; zz < NZ; ++zz)
#pragma unroll
        for (int i = 0; i < CWE; ++i) {
          const int ct = ct0 + i;  // tile of the block -> the wave that parked it
          const int pw = (rt / MTW) * WC + ct / CW;
          const int64_t piece = (int64_t)min(z0 + zz, KS - 1) * zstride + uslot + (pw * MTW + rt % MTW) * CW + ct % CW;
          v[zz][i] = ld16_l2(rp, (uint32_t)((piece * 64 + lane) * 16));
        }
#pragma unroll
      for (int zz = 0; zz < NZ; ++zz)
        if (z0 + zz < KS) {
#pragma unroll
          for (int i = 0; i < CWE; ++i) sum[i] += __builtin_bit_cast(f32x4, v[zz][i]);
        }
    };
    constexpr int NZ = CWE >= 7 ? 4 : 8;
#pragma unroll 1
    for (int rt = kc; rt < MT; rt += KS) {
      if constexpr (EPI == EPI_RESID) {
        if (rt + KS < MT) load_x(rt + KS, xnxt);
      }
      if (cols_in && (kQuarter || ((rt - kc) / KS) % Cfg::WM == wm)) {
        f32x4 sum[CWE];
#pragma unroll
        for (int i = 0; i < CWE; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (KS <= 4) {
          add_slices(std::integral_constant<int, 4>{}, rt, 0, sum);
        } else {
          for (int z0 = 0; z0 < KS; z0 += NZ) add_slices(std::integral_constant<int, NZ>{}, rt, z0, sum);
        }
        finish(rt, sum, xcur);
      }
      if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int j = 0; j < NPASS; ++j) xcur[j] = xnxt[j];
      }
    }
  } else {
#pragma unroll
    for (int mw = 0; mw < MTW; ++mw) {
      if constexpr (EPI == EPI_RESID) {
        if (mw + 1 < MTW) load_x(wm * MTW + mw + 1, xnxt);
      }
      if (cols_in) finish(wm * MTW + mw, acc[mw], xcur);
      if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int j = 0; j < NPASS; ++j) xcur[j] = xnxt[j];
      }
    }
  }
  if constexpr (EPI == EPI_RESID) {
    __syncthreads();
    if (threadIdx.x < MT * 16) {
      const int m = row0 + threadIdx.x;
      float s = ssq_s[0][threadIdx.x];
#pragma unroll
      for (int q = 1; q < (kQuarter ? 4 : WC); ++q) s += ssq_s[q][threadIdx.x];
      if (m < a.M && own((int)threadIdx.x / 16)) a.sumsq_out[(int64_t)m * a.n_part_out + cb] = s;
    }
  }
}

// ---- host side: plan and launch

GemmPlan gemm_plan(int M, int n_tiles, int K, int64_t part_cap, bool nt12, bool half_block, int nt14) {
  GemmPlan best{};
  const int mt = M <= 32 ? 2 : (M <= 64 ? 4 : 8);
  const int mb = (M + mt * 16 - 1) / (mt * 16);
  const int S_all = K / 32;
  double best_cost = 1e300;
  // 12-tile blocks (gate/up, and the QKV projection of prefill chunks): Qwen 8B's 1536 gate/up tiles then fill all 32 CUs of an
  // XCD in one round (16 blocks x 2 K slices) where 16-tile blocks leave 8 idle, and so do the
  // 384 tiles of QKV at 1024 rows (32 blocks x 8 row blocks against 24 x 8).  14-tile blocks
  // (gate/up of more than 64 rows): Llama 8B's 1792 tiles are 128 of them, 256 workgroups at
  // 256 rows where 16-tile blocks leave 32 CUs idle; gate/up at 1024 rows 367 -> 353 us, at 256
  // rows 99.9 -> 97.0.  In two K slices (65 to 128 rows) they pay with e4m3 weights (128 rows
  // 57.8 -> 55.7 us, 78 rows 54.1 -> 52.4) and not with bf16 (71.8 us against 66.7 in 16-tile
  // blocks, 78 rows 63.1 against 59.4): the stream of the weights sets the time there, and so it
  // does with fewer rows (64 rows 48.8 -> 53.0 us, 32 rows 39.9 -> 43.7).
  for (int nt : {16, 14, 12, 8}) {
    // half_block: 16-tile blocks also when n_tiles % 16 == 8, the last one half full (one K
    // slice: its empty half would otherwise park and sum nothing)
    const bool half = half_block && nt == 16 && n_tiles % 16 == 8;
    if ((n_tiles % nt && !half) || (nt == 12 && !nt12) || (nt == 14 && (!nt14 || mt < 8))) continue;
    const int n_cb = (n_tiles + nt - 1) / nt;
    for (int ks = 1; ks <= 8; ++ks) {
      if (ks > 1 && (S_all / ks < 4 || half || (nt == 14 && ks > nt14))) break;
      if (ks > 1 && (int64_t)ks * n_cb * nt * 16 * mb * mt * 16 > part_cap) break;
      if (ks > 1 && (int64_t)n_cb * mb * kCtrStride > kLayerCtr0) break;  // one counter line per unit
      // one workgroup per CU, 32 CUs per XCD; units of a column block share its XCD.  The
      // slices of a unit wait for each other, so a split plan runs in one round.
      const int per_xcd = ((n_cb + 7) / 8) * mb * ks;
      if (ks > 1 && per_xcd > kXcdWgs) break;
      const int rounds = (per_xcd + 31) / 32;
      const double steps = (double)S_all / ks;
      const double w_time = steps * nt * 1024.0 / (8e12 / 256);                   // weights at a CU's share of HBM
      const double m_time = steps * nt * mt * 2.0 * 16.0 / 4.0 / 2.4e9;           // MFMA issue, 4 SIMDs
      const double part_bytes = ks > 1 ? 2.0 * ks * n_tiles * 16.0 * mb * mt * 16 * 4 : 0.0;
      const double a_bytes = (double)n_cb * mb * mt * 16 * K * 4;
      // The split's own cost (parked partials, the slices' wait, their sums): a price per batch of
      // slices, fitted to an earlier kernel in which one workgroup added them all, and kept.  Every
      // plan of every projection of both 8B shapes on this kernel, 32 to 1024 rows, both weight
      // formats: the pick is within 3 % of the fastest but for (us, the pick and the fastest) e4m3
      // gate/up at 32 rows, whose weights the model prices at two bytes (8 tiles 31.0, 16 in two
      // slices 26.4; Qwen 29.5, 25.7), Qwen's down projection in 8 slices instead of 7 (32 rows
      // 25.0, 23.4, 64 rows 30.2, 28.1), O at 512 and 1024 rows (16 tiles in 4 slices 41.4, 8 in two
      // 40.4, e4m3 40.2, 37.6; 16 in two 65.4, 8 in one 62.3, e4m3 64.6, 60.0) and e4m3 QKV at 512
      // (16 in two 64.9, 8 in one 62.9).
      const int nacc = (mt / 2) * (nt / 2);  // accumulator tiles per wave (2 x 2 waves)
      const int zb = nacc >= 32 ? 1 : (nacc >= 16 ? 2 : 4);
      const double reduce = ks > 1 ? 1e-6 + 0.6e-6 * ((ks + zb - 1) / zb) : 0.0;
      const double cost = rounds * std::max(w_time, m_time) + 0.5 * part_bytes / 8e12 + a_bytes / 32e12 + reduce;
      if (cost < best_cost) {
        best_cost = cost;
        best = GemmPlan{mt, nt, ks, mb, n_cb};
      }
    }
  }
  return best;
}

template <int MT, int NT, int EPI, bool W8>
static void launch_cfg(const GemmArgs& a, const Exec& ex) {
  const int n_cb = (a.n_tiles + NT - 1) / NT;
  const unsigned grid = (unsigned)(((n_cb + 7) / 8) * 8 * a.splits * a.m_blocks);
  if constexpr (MT == 8 && EPI == EPI_SCALED_STORE) {
    if (a.fold) {
      if (a.splits > 1)
        SBD_KLAUNCH((gemm_kernel<MT, NT, EPI, W8, true, true>), dim3(grid), dim3(512), ex, a);
      else
        SBD_KLAUNCH((gemm_kernel<MT, NT, EPI, W8, false, true>), dim3(grid), dim3(512), ex, a);
      return;
    }
  }
  if constexpr (NT != 14 || W8) {  // 14-tile blocks of bf16 weights: one K slice (gemm_plan)
    if (a.splits > 1) {
      SBD_KLAUNCH((gemm_kernel<MT, NT, EPI, W8, true, false>), dim3(grid), dim3(512), ex, a);
      return;
    }
  }
  SBD_KLAUNCH((gemm_kernel<MT, NT, EPI, W8, false, false>), dim3(grid), dim3(512), ex, a);
}
template <int MT, int NT, int EPI>
static void launch_fmt(const GemmArgs& a, const Exec& ex) {
  if constexpr (NT != 12) {  // 12-tile blocks: bf16 weights only (gemm_plan)
    if (a.Wp8 != nullptr) return launch_cfg<MT, NT, EPI, true>(a, ex);
  }
  launch_cfg<MT, NT, EPI, false>(a, ex);
}

static void launch_fold12(const GemmArgs& a, const Exec& ex) {
  const unsigned grid = (unsigned)(((a.n_tiles / 12 + 7) / 8) * 8 * a.splits * a.m_blocks);
  if (a.splits > 1)
    SBD_KLAUNCH((gemm_kernel<8, 12, EPI_SCALED_STORE, false, true, true>), dim3(grid), dim3(512), ex, a);
  else
    SBD_KLAUNCH((gemm_kernel<8, 12, EPI_SCALED_STORE, false, false, true>), dim3(grid), dim3(512), ex, a);
}

template <int EPI>
static void launch_epi(const GemmArgs& a, int mt, int nt, const Exec& ex) {
  if constexpr (EPI == EPI_SWIGLU) {
    if (nt == 14) return launch_fmt<8, 14, EPI>(a, ex);  // eight row tiles only (gemm_plan)
    if (nt == 12) {
      if (mt == 2) launch_fmt<2, 12, EPI>(a, ex);
      else if (mt == 4) launch_fmt<4, 12, EPI>(a, ex);
      else launch_fmt<8, 12, EPI>(a, ex);
      return;
    }
  }
  if constexpr (EPI == EPI_SCALED_STORE) {
    if (nt == 12) return launch_fold12(a, ex);  // with FOLD only: eight row tiles (launch_gemm)
  }
  if (nt == 16) {
    if (mt == 2) launch_fmt<2, 16, EPI>(a, ex);
    else if (mt == 4) launch_fmt<4, 16, EPI>(a, ex);
    else launch_fmt<8, 16, EPI>(a, ex);
  } else {
    if (mt == 2) launch_fmt<2, 8, EPI>(a, ex);
    else if (mt == 4) launch_fmt<4, 8, EPI>(a, ex);
    else launch_fmt<8, 8, EPI>(a, ex);
  }
}

hipError_t launch_gemm(GemmEpi epi, const GemmArgs& a0, const Exec& ex) {
  if (a0.M < 1 || a0.K < 32 || a0.K % 32 || a0.n_tiles < 8 || a0.n_tiles % 8 || a0.a_mtiles < 1) return hipErrorInvalidValue;
  if (a0.Wp8 != nullptr && a0.wscale == nullptr) return hipErrorInvalidValue;
  if (a0.fold && (epi != EPI_SCALED_STORE || a0.M <= 64)) return hipErrorInvalidValue;  // row blocks of eight tiles
  const bool nt12 = (epi == EPI_SWIGLU || (epi == EPI_SCALED_STORE && a0.fold)) && a0.Wp8 == nullptr;
  const bool half_block = (epi == EPI_SCALED_STORE || epi == EPI_LOGITS_EB) && a0.Wp8 == nullptr;
  const GemmPlan p = gemm_plan(a0.M, a0.n_tiles, a0.K, (a0.part && !a0.no_split) ? a0.part_cap : 0, nt12, half_block,
                               epi != EPI_SWIGLU ? 0 : (a0.Wp8 != nullptr ? 8 : 1));
  if (p.nt == 0) return hipErrorInvalidValue;
  if (p.splits > 1 && (a0.counters == nullptr || (int64_t)p.n_cb * p.m_blocks * kCtrStride > kLayerCtr0))
    return hipErrorInvalidValue;
  if (epi == EPI_RESID && a0.n_part_out != p.n_cb) return hipErrorInvalidValue;
  // the epilogue writes 16-byte (fp32) and 8-byte (bf16) pieces of 4 columns
  if ((epi == EPI_SCALED_STORE && a0.ldo % 4) || (epi == EPI_RESID && a0.ldx % 4) ||
      (epi == EPI_SWIGLU && a0.ld_act % 4) || (epi == EPI_LOGITS_EB && a0.out_f32 && a0.ldo % 4))
    return hipErrorInvalidValue;
  if (epi == EPI_LOGITS_EB && (a0.eb_part == nullptr || a0.eb_arg == nullptr || a0.eb_chunks * kEbFChunk != a0.n_tiles * 16))
    return hipErrorInvalidValue;
  GemmArgs a = a0;
  a.splits = p.splits;
  a.m_blocks = p.m_blocks;
  // the slices of a unit wait for each other: only in a plan of one round (gemm_plan), on a
  // device that keeps every workgroup of an XCD resident at once
  if (p.splits > 1 && (!a0.wait_ok || a0.err == nullptr || ((p.n_cb + 7) / 8) * p.m_blocks * p.splits > kXcdWgs))
    return hipErrorInvalidValue;
  switch (epi) {
    case EPI_SCALED_STORE: launch_epi<EPI_SCALED_STORE>(a, p.mt, p.nt, ex); break;
    case EPI_RESID: launch_epi<EPI_RESID>(a, p.mt, p.nt, ex); break;
    case EPI_SWIGLU: launch_epi<EPI_SWIGLU>(a, p.mt, p.nt, ex); break;
    case EPI_LOGITS_EB: launch_epi<EPI_LOGITS_EB>(a, p.mt, p.nt, ex); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One thread per 16-byte piece of the packed matrix (layout at the top of this file).
// Mode 0: packed row n is src0 row n.  Mode 1 (gate/up): packed tile t holds src0 rows
// 8t..8t+7 then src1 rows 8t..8t+7.
__global__ __launch_bounds__(256) void pack_kernel(const bf16_t* src0, const bf16_t* src1,
                                                   bf16_t* dst, int64_t n_pieces, int K, int mode) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_pieces) return;
  const int S = K / 32;
  const int lane = (int)(i % 64);
  const int64_t tt = (i / 64) % 8;            // tile inside the group
  const int64_t s = (i / 512) % S;            // K step
  const int64_t t = (i / (512 * (int64_t)S)) * 8 + tt;
  const int rr = lane & 15;
  const int64_t k0 = 32 * s + 8 * (lane >> 4);
  const bf16_t* row;
  if (mode == 0)
    row = src0 + (t * 16 + rr) * (int64_t)K;
  else
    row = (rr < 8) ? src0 + (t * 8 + rr) * (int64_t)K : src1 + (t * 8 + rr - 8) * (int64_t)K;
  *(i32x4*)(dst + i * 8) = *(const i32x4*)(row + k0);
}

hipError_t launch_pack(const bf16_t* src0, const bf16_t* src1, bf16_t* dst, int64_t rows, int K,
                       int mode, hipStream_t s) {
  if (rows % 128 || K % 32) return hipErrorInvalidValue;
  const int64_t n_pieces = rows * K / 8;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((n_pieces + 255) / 256)), dim3(256), 0, s, src0,
                     src1, dst, n_pieces, K, mode);
  return hipGetLastError();
}

}  // namespace sbd
