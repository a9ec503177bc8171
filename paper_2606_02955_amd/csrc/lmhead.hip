// lmhead.hip -- the LM head fused with the vocabulary pass on gfx950.
//
// Alg. 1's model call ends in the output projection: a candidate position's
// logits are l_v = sum_k h_k W_vk.  Here they are formed tile by tile on the
// matrix cores (v_mfma_f32_16x16x32_bf16, bf16 operands, float32
// accumulation) and folded straight into the vocabulary pass's online
// (maximum, exponent reference, sum, argmax) state, so no logit reaches HBM;
// the per-position outputs and the selection are then those of
// fdllm_confidence / fdllm_decode_step (Sec. 3 "Notation"; Alg. 1).
//
// Two plans, by the number of positions N = B L:
//   N <= 32     k_lm_stream (d a multiple of 512 up to 4096): W streamed once,
//               hidden operands in registers, logits folded in the kernel;
//   otherwise   MFMA tiles of 256 vocabulary rows x 32 to 256 positions, the
//               width chosen on the device by the number of candidates:
//               k_lm_narrow (at most 128, HBM-bound), k_lm_wide (HBM-bound
//               up to about 200, then bound by the matrix cores);
// each followed by k_lm_finish, which combines the per-workgroup states.
//
// Main loop of the tiles: a workgroup of 8 waves; the hidden dimension streams
// in stages of 64 elements (128 bytes of every weight and hidden row, so each
// load uses whole cache lines) that buffer_load ... lds writes straight into
// LDS, two to four stages resident (up to 160 KiB), one barrier per stage.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <atomic>

#include "fdllm.h"
#include "lm_work.h"
#include "pass_common.h"

namespace fdllm {

// ---------------------------------------------------------------------------
// LM head fused with the vocabulary pass: logits = hidden . W^T are formed
// tile by tile in MFMA accumulators and folded into the per-row online
// (max, exponent reference, sum, argmax) state; no logit is written to HBM.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kLmWaves = 8;                    // waves per workgroup
constexpr int kLmThreads = kLmWaves * kWave;

// Candidate rows of every sequence, compacted (in any order, from run to run
// too: a row's result depends neither on its place in a tile nor on the tile,
// all tiles meet the same vocabulary ranges); default outputs for every other
// position.  One wavefront per sequence.
__global__ void __launch_bounds__(256)
k_lm_compact(const uint8_t* __restrict__ mask, const int32_t* __restrict__ bstart,
             const int32_t* __restrict__ bend, int B, int L, int32_t* __restrict__ rows,
             int32_t* __restrict__ count, RowOut out) {
  const int lane = threadIdx.x % kWave;
  const int b = blockIdx.x * 4 + threadIdx.x / kWave;
  if (b >= B) return;
  const int s = bstart[b], e = bend[b];
  const bool ok = window_ok(s, e, L);
  const size_t row0 = (size_t)b * L;
  for (int q0 = 0; q0 < L; q0 += kWave) {
    const int q = q0 + lane;
    const bool cand = q < L && ok && q >= s && q < e && mask[row0 + q] != 0;
    if (q < L && !cand) store_default(out, row0 + q);
    const unsigned long long bal = __ballot(cand);
    if (bal == 0ull) continue;
    int base = 0;
    if (lane == 0) base = atomicAdd(count, __popcll(bal));
    base = __shfl(base, 0);
    if (cand) rows[base + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)(row0 + q);
  }
}

// The same for at most kLmOneWg positions, in position order, by one
// workgroup: a launch less (no counter to clear first) and one round trip to
// memory, every load issued at once.
constexpr int kLmOneThreads = 1024;
constexpr int kLmOneChunks = 8;
constexpr int kLmOneWg = kLmOneThreads * kLmOneChunks;

__global__ void __launch_bounds__(kLmOneThreads)
k_lm_compact_one(const uint8_t* __restrict__ mask, const int32_t* __restrict__ bstart,
                 const int32_t* __restrict__ bend, int B, int L, int32_t* __restrict__ rows,
                 int32_t* __restrict__ count, RowOut out) {
  constexpr int kWaves = kLmOneThreads / kWave;
  __shared__ int s_n[kLmOneChunks * kWaves];      // candidates of chunk c, wave w
  const int n = B * L;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int s[kLmOneChunks], e[kLmOneChunks], q[kLmOneChunks];
  bool m[kLmOneChunks];
#pragma unroll
  for (int c = 0; c < kLmOneChunks; ++c) {
    const int i = c * kLmOneThreads + (int)threadIdx.x;
    const int ic = i < n ? i : 0;                 // past the end: position 0, not used
    const int b = ic / L;
    q[c] = ic - b * L;
    s[c] = bstart[b];
    e[c] = bend[b];
    m[c] = mask[ic] != 0;
  }
  unsigned long long bal[kLmOneChunks];
#pragma unroll
  for (int c = 0; c < kLmOneChunks; ++c) {
    const int i = c * kLmOneThreads + (int)threadIdx.x;
    const bool cand = i < n && m[c] && window_ok(s[c], e[c], L) && q[c] >= s[c] && q[c] < e[c];
    if (i < n && !cand) store_default(out, (size_t)i);
    bal[c] = __ballot(cand);
    if (lane == 0) s_n[c * kWaves + wave] = __popcll(bal[c]);
  }
  __syncthreads();
  // lane l of every wave: the entries 2 l and 2 l + 1 and an inclusive scan
  static_assert(kLmOneChunks * kWaves == 2 * kWave, "two entries a lane");
  const int n0 = s_n[2 * lane], n1 = s_n[2 * lane + 1];
  int incl = n0 + n1;
#pragma unroll
  for (int x = 1; x < kWave; x <<= 1) {
    const int o = __shfl_up(incl, x);
    if (lane >= x) incl += o;
  }
  const int excl = incl - n0 - n1;
#pragma unroll
  for (int c = 0; c < kLmOneChunks; ++c) {
    const int k = c * kWaves + wave;              // wave-uniform
    const int base = __shfl(excl, k / 2) + (k % 2 ? __shfl(n0, k / 2) : 0);
    if ((bal[c] >> lane) & 1ull)
      rows[base + __popcll(bal[c] & ((1ull << lane) - 1ull))] = c * kLmOneThreads + (int)threadIdx.x;
  }
  if (threadIdx.x == kWave - 1) *count = incl;
}

__global__ void k_lm_zero(int32_t* __restrict__ p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0;
}

// Per-lane online state of one position over the vocabulary entries this
// lane sees.
struct LmState {
  float M, K;
  double S;
  int first;
};

// the exponent reference of a running maximum (kRefFloor before any element)
__device__ __forceinline__ float lm_ref(float M) { return fmaxf(exp_ref(M), kRefFloor); }

// Folds the lane's accumulators of one position, acc[.][0] (vocabulary
// entries base + 16 mi + i, increasing in (mi, i)), into its state.
template <int MI, int NI>
__device__ __forceinline__ void lm_fold_first(LmState& st, f32x4 (&acc)[MI][NI], int base, int v_end,
                                              bool partial) {
  if (partial) {
    // entries past the end take part in nothing: their terms are 0
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[mi][0][i] = 16 * mi + i < v_end - base ? acc[mi][0][i] : kNegInf;
  }
  float tm = kNegInf;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int i = 0; i < 4; ++i) tm = fmaxf(tm, acc[mi][0][i]);
  float K = lm_ref(st.M);      // not kept in a register over the matrix loop
  if (tm > st.M) {
    const float Kn = exp_ref(tm);
    st.S = rescale(st.S, K, Kn);
    K = Kn;
    st.M = tm;
    int f = 0;
#pragma unroll
    for (int mi = MI - 1; mi >= 0; --mi)
#pragma unroll
      for (int i = 3; i >= 0; --i)
        if (acc[mi][0][i] == tm) f = 16 * mi + i;
    st.first = base + f;
  }
  // every term enters a double sum on its own, so the greedy element's term
  // stays exact and s' = (S - e_M) / e_M keeps its relative accuracy
  double sum[2] = {0.0, 0.0};
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[i & 1] += (double)term(acc[mi][0][i], K);
  st.S += sum[0] + sum[1];
}

// Folds all NI positions of a lane.  One body, run NI times with the
// accumulators and states turned by one position each time: a tile's fold is
// run once or twice in a launch, so its instructions come from memory, and
// the time they take to arrive, not the arithmetic, is what it costs
// (unrolled over the positions it added 12 us to a launch of 155 us that
// reads 1 GB of weights for 32 positions).
template <int MI, int NI>
__device__ __forceinline__ void lm_fold(LmState (&st)[NI], f32x4 (&acc)[MI][NI], int base, int v_end,
                                        bool partial) {
#pragma unroll 1
  for (int k = 0; k < NI; ++k) {
    lm_fold_first<MI, NI>(st[0], acc, base, v_end, partial);
    const LmState s0 = st[0];
#pragma unroll
    for (int ni = 0; ni + 1 < NI; ++ni) st[ni] = st[ni + 1];
    st[NI - 1] = s0;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni + 1 < NI; ++ni) acc[mi][ni] = acc[mi][ni + 1];
  }
}

__device__ __forceinline__ void lm_combine(LmState& st, float M2, float K2, double S2, int f2) {
  const float Mn = fmaxf(st.M, M2);
  const int fa = st.M == Mn ? st.first : 0x7fffffff;
  const int fb = M2 == Mn ? f2 : 0x7fffffff;
  ks_combine(st.K, st.S, K2, S2);
  st.M = Mn;
  st.first = min(fa, fb);
}

// ---- work division ----------------------------------------------------------
// lm_work (lm_work.h) on the device, the candidates' number of rounds a lane
// each; every kernel of a call forms the same division for itself.
__device__ __forceinline__ LmWork lm_work_device(int n, int V, int d) {
  LmWork w = lm_work_tiles(n, V);
  if (w.mt > 1) {
    const int lane = lane_id();
    int k = lm_round_ranges(w, lane % kLmRounds);
    unsigned long long t = lm_round_time(w, k, d);
    int at = lane % kLmRounds;                  // the first of the shortest, as lm_work
#pragma unroll
    for (int x = 1; x < kLmRounds; x <<= 1) {
      const unsigned long long t2 = __shfl_xor(t, x);
      const int k2 = __shfl_xor(k, x), at2 = __shfl_xor(at, x);
      if (t2 < t || (t2 == t && at2 < at)) {
        t = t2;
        k = k2;
        at = at2;
      }
    }
    w.k = __builtin_amdgcn_readfirstlane(k);
  }
  return w;
}

// ---- LDS-DMA main loop -----------------------------------------------------
// Stages of kLmBK hidden elements: VT weight rows and PT hidden rows of
// kLmBK * 2 bytes each, written by buffer_load ... lds (each lane of a wave
// instruction fills the next 16 bytes of LDS), WB weight and HB hidden stages
// resident.  Rows are stored unpadded; the 16-byte vector s of row r
// sits in slot s ^ lm_swz(r).  lm_swz was chosen from LDS bank-conflict
// counter measurements of ds_read_b128 patterns on gfx950: with it the
// operand reads (lane l: row l % 16, vector 4 h + l / 16) are conflict-free.
constexpr int kLmBK = 64;                                 // hidden elements per stage
constexpr int kLmSlots = kLmBK / 8;                       // 16-byte vectors per row and stage
constexpr int kLmRowBytes = kLmBK * 2;
constexpr int kLmDmaRows = kWave / kLmSlots;              // rows per wave-wide load
constexpr int kLmWBytes = kLmVt * kLmRowBytes;            // weight part of a stage
constexpr int kLmWDma = kLmVt / kLmDmaRows / kLmWaves;    // weight loads per wave and stage

__device__ __forceinline__ int lm_swz(int r) { return (r & 1) | ((r >> 1) & 2) | ((r << 1) & 4); }

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef int i32x4 __attribute__((ext_vector_type(4)));

// buffer resource of a raw byte range (stride 0, bounds check on the byte
// offset), all four words wave-uniform
__device__ __forceinline__ i32x4 lm_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)base;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}

// one wave-wide 16-byte-per-lane load into LDS: lane i's vector lands at
// byte lds + 16 i.  Issued as inline assembly: the compiler cannot tell which
// buffer such a load writes and would drain every load in flight before the
// next LDS read; the explicit vmcnt waits of lm_sync are the ones needed.
// NT: data that no other workgroup reads (nontemporal).
template <bool NT>
__device__ __forceinline__ void lm_dma(i32x4 rsrc, uint32_t lds, uint32_t voff, int soff) {
  int keep;   // m0 is the compiler's register: saved and restored around the load
  if constexpr (NT)
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\tbuffer_load_dwordx4 %2, %3, %4 offen nt lds\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(keep) : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
  else
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds\n\t"
                 "s_mov_b32 m0, %0"
                 : "=&s"(keep) : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// waits until at most N of this wave's loads are outstanding and its LDS
// reads are done, then meets the other waves; the memory clobber keeps LDS
// accesses on their side
template <int N>
__device__ __forceinline__ void lm_sync() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

#define LM_FENCE() __builtin_amdgcn_sched_barrier(0)

// Shape of a tile's main loop: WV x WP waves over VT x PT, each MI x NI MFMA
// blocks of 16 x 16; WB weight and HB hidden stages resident.
template <int PT_, int WV_, int WB_, int HB_>
struct LmShape {
  static constexpr int PT = PT_, WV = WV_, WP = kLmWaves / WV_, WB = WB_, HB = HB_;
  static constexpr int MI = kLmVt / WV / 16, NI = PT / WP / 16;
  static constexpr int HDma = PT >= 64 ? PT / kLmDmaRows / kLmWaves : 1;   // hidden loads per wave and stage
  static constexpr int HBytes = PT * kLmRowBytes;
  static constexpr int HOff = WB * kLmWBytes;               // hidden buffers after the weight ones
  static constexpr int Bytes = WB * kLmWBytes + HB * HBytes;
};
constexpr size_t kLmLdsBytes = 160 * 1024;
constexpr int kLmStageBytes = 144 * 1024;                   // the narrow tiles' stages

// Rows a multiple of 4 KiB apart have their elements k in the same few memory
// channels, and all workgroups read the same k at the same time.  So half of
// them go through the hidden dimension with each two neighbouring blocks of
// 16 stages (2 KiB of a row) exchanged: 64 positions at d = 4096,
// V = 126464 190 -> 162 us.  The even and the odd blocks are summed apart and
// added at the end, so a logit's bits do not depend on which workgroup formed
// it (equal weight rows tie, whatever their places).
constexpr int kLmFlip = 16;
__device__ __forceinline__ int lm_flip(int g, int nks) {
  return nks % (2 * kLmFlip) == 0 && (g / 8) % 2 ? kLmFlip : 0;
}

// the producer: the next stage this wave loads (tile relative to the
// segment's first, stage within the tile), the buffer it goes to, and the
// lane's load offsets.  Stage i of a tile holds the hidden elements
// [64 k, 64 k + 64) with k = i ^ flip (lm_flip).  Past the last stage the last one is
// loaded again (into a buffer nobody reads any more), so every stage issues
// the same number of loads.
template <class Sh>
struct LmProducer {
  int tile, ks, left, buf;        // weight stages
  int hks, hleft, hbuf;           // hidden stages
  i32x4 wr, hr;
  uint32_t w_voff[kLmWDma], h_voff[Sh::HDma];
  uint32_t lds_w, lds_h;          // the wave's LDS offsets within a stage
};

// weight rows [n0, min(n0 + 256, v_end)); the rows past v_end are out of the
// resource's range: no memory is read for them (they are masked in the fold)
template <class Sh>
__device__ __forceinline__ void lm_tile_setup(LmProducer<Sh>& p, const uint16_t* weight, int n0,
                                              int v_end, int d) {
  p.wr = lm_rsrc(weight + (size_t)n0 * d, (uint32_t)min(kLmVt, v_end - n0) * (uint32_t)d * 2u);
}

struct LmArgs {
  const uint16_t* hidden;
  const uint16_t* weight;
  int32_t* rows;           // candidates, in any order, and their number (workspace)
  int32_t* count;
  WavePartial* partials;
  int d, V;
  uint32_t hid_bytes;
};

// One segment: `cnt` candidates from rank p0 (at most PT) against the
// vocabulary rows [v_beg, v_end); partials at [p0 + i] * stride + split.
// Wave w computes vocabulary rows 16 MI (w % WV) .. of a tile against
// positions 16 NI (w / WV) .. as MI x NI MFMA 16x16x32 blocks, vocabulary
// along the MFMA rows: lane l holds positions 16 ni + l % 16 and, for each,
// vocabulary rows 16 mi + 4 (l / 16) + i of the wave's.
template <class Sh, bool NT>
__device__ __forceinline__ void lm_segment(const LmArgs& a, const int32_t* rows, int p0, int cnt, int v_beg,
                                           int v_end, int flip, int stride, int split) {
  constexpr int MI = Sh::MI, NI = Sh::NI, WV = Sh::WV;
  constexpr int NL = kLmWDma + Sh::HDma;
  // the interleaved schedule: one wave tile of 128 x (48 or 64)
  constexpr bool kInterleaved = MI == 8;
  static_assert(Sh::Bytes <= (int)(Sh::PT <= 128 ? kLmStageBytes : kLmLdsBytes), "stages fit the LDS");
  extern __shared__ __attribute__((aligned(1024))) char lm_lds[];
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int vw = wave % WV, pw = wave / WV;
  const int d = a.d, nks = d / kLmBK;
  const int n_tiles = (v_end - v_beg + kLmVt - 1) / kLmVt;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lm_lds;

  LmProducer<Sh> pr;
  pr.tile = 0;
  pr.ks = 0;
  pr.left = n_tiles * nks;
  pr.buf = 0;
  pr.hks = 0;
  pr.hleft = pr.left;
  pr.hbuf = 0;
  pr.hr = lm_rsrc(a.hidden, a.hid_bytes);
  auto hidden_rows = [&]() {
    const int lr = lane / kLmSlots, ls = lane % kLmSlots;
#pragma unroll
    for (int j = 0; j < Sh::HDma; ++j) {
      const int first = ((wave * Sh::HDma + j) * kLmDmaRows) % Sh::PT;
      const int r = first + lr;
      // positions past the end repeat the others, spread over them
      const int q = p0 + (r < cnt ? r : r % cnt);
      pr.h_voff[j] = (uint32_t)rows[q] * (uint32_t)d * 2u + (uint32_t)((ls ^ lm_swz(r)) * 16);
      if (j == 0) pr.lds_h = lds0 + (uint32_t)(Sh::HOff + first * kLmRowBytes);
    }
  };
  {
    const int lr = lane / kLmSlots, ls = lane % kLmSlots;
#pragma unroll
    for (int j = 0; j < kLmWDma; ++j) {
      const int r = (wave * kLmWDma + j) * kLmDmaRows + lr;
      pr.w_voff[j] = (uint32_t)r * (uint32_t)d * 2u + (uint32_t)((ls ^ lm_swz(r)) * 16);
    }
    pr.lds_w = lds0 + (uint32_t)(wave * kLmWDma * kLmDmaRows * kLmRowBytes);
  }
  lm_tile_setup(pr, a.weight, v_beg, v_end, d);

  // the loads of the producers' stages: H j (j < HDma) of the hidden
  // producer, then W j - HDma of the weight producer
  auto dma = [&](int j) {
    if (j < Sh::HDma)
      lm_dma<false>(pr.hr, pr.lds_h + (uint32_t)(pr.hbuf * Sh::HBytes + j * kWave * 16), pr.h_voff[j],
                    __builtin_amdgcn_readfirstlane((pr.hks ^ flip) * kLmRowBytes));
    else
      lm_dma<NT>(pr.wr, pr.lds_w + (uint32_t)(pr.buf * kLmWBytes + (j - Sh::HDma) * kWave * 16),
                 pr.w_voff[j - Sh::HDma],
                 __builtin_amdgcn_readfirstlane((pr.ks ^ flip) * kLmRowBytes));
  };
  auto advance_w = [&]() {
    if (pr.left > 1) {
      --pr.left;
      if (++pr.ks == nks) {
        pr.ks = 0;
        ++pr.tile;
        lm_tile_setup(pr, a.weight, v_beg + pr.tile * kLmVt, v_end, d);
      }
    }
    pr.buf = pr.buf + 1 == Sh::WB ? 0 : pr.buf + 1;
  };
  auto advance_h = [&]() {
    if (pr.hleft > 1) {
      --pr.hleft;
      if (++pr.hks == nks) pr.hks = 0;
    }
    pr.hbuf = pr.hbuf + 1 == Sh::HB ? 0 : pr.hbuf + 1;
  };

  // operand addresses of this lane: row l % 16 of a 16-row block, 16-byte
  // vector 4 h + l / 16 of the stage's 64 hidden elements in half h
  const uint32_t slot0 = (uint32_t)((lane / 16 ^ lm_swz(lane % 16)) * 16);
  const uint32_t a_addr0 = (uint32_t)((16 * MI * vw + lane % 16) * kLmRowBytes) + slot0;
  const uint32_t b_addr0 = (uint32_t)(Sh::HOff + (16 * NI * pw + lane % 16) * kLmRowBytes) + slot0;
  constexpr uint32_t kHalf = 64;    // half 1: vector 4 + ..., bit 6 of the address (rows are 128 bytes)
  auto lds_at = [&](uint32_t at) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(lm_lds + (at - lds0));
  };

  LmState st[NI];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) st[ni] = LmState{kNegInf, kRefFloor, 0.0, 0x7fffffff};   // K unused here

  auto zero = [&](f32x4 (&acc)[MI][NI]) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[mi][ni][i] = 0.0f;
  };
  auto fold = [&](int t, f32x4 (&acc)[MI][NI]) {
    const int n0 = v_beg + t * kLmVt;
    lm_fold<MI, NI>(st, acc, n0 + 16 * MI * vw + 4 * (lane / 16), v_end, n0 + kLmVt > v_end);
  };

  if constexpr (kInterleaved) {
    // three weight stages and two hidden ones: the weight part, from HBM or
    // the Infinity Cache, runs one stage further ahead than the hidden part,
    // mostly L2 hits.  Both are loaded into the buffers of the stage just
    // read, in the second half of the current stage.
    static_assert(Sh::WB == 3 && Sh::HB == 2 && kLmWDma == 4, "the schedule's waits");
    f32x4 acc[MI][NI];
    bf16x8 fa[8], fb[NI], nfb[NI], na7;
#define LM_M(mi, ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mi], fb[ni], acc[mi][ni], 0, 0, 0)
    // the MFMAs of one half stage on (fa, fb); the operands of the next half
    // stage (weight operands at sa, hidden operands at sb) are read as the
    // registers they replace fall dead; with_loads also issues the stage loads
    auto half = [&](uint32_t sa, uint32_t sb, bool with_loads) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        LM_M(0, ni); LM_FENCE();
        nfb[ni] = lds_at(sb + (uint32_t)(16 * ni * kLmRowBytes)); LM_FENCE();
      }
#pragma unroll
      for (int mi = 1; mi < 8; ++mi) {
        LM_M(mi, 0); LM_FENCE();
        fa[mi - 1] = lds_at(sa + (uint32_t)((mi - 1) * 16 * kLmRowBytes)); LM_FENCE();
        LM_M(mi, 1); LM_FENCE();
        if (with_loads && mi - 1 < NL) { dma(mi - 1); LM_FENCE(); }
        if (mi == 7) { na7 = lds_at(sa + (uint32_t)(7 * 16 * kLmRowBytes)); LM_FENCE(); }
#pragma unroll
        for (int ni = 2; ni < NI; ++ni) {
          LM_M(mi, ni); LM_FENCE();
          if (ni == 2 && with_loads && mi == 7 && NL > 7) { dma(7); LM_FENCE(); }
        }
      }
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[ni] = nfb[ni];
      fa[7] = na7;
    };

    hidden_rows();
    // prologue: stages 0 and 1 of both, and the weight part of stage 2, in
    // flight (in this order), then wait for stage 0
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int j = 0; j < NL; ++j) dma(j);
      advance_h();
      advance_w();
    }
#pragma unroll
    for (int j = Sh::HDma; j < NL; ++j) dma(j);
    advance_w();
    lm_sync<NL + kLmWDma>();
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) fb[ni] = lds_at(lds0 + b_addr0 + ni * 16 * kLmRowBytes);
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) fa[mi] = lds_at(lds0 + a_addr0 + mi * 16 * kLmRowBytes);

    int wbuf = 0, hbuf = 0;     // buffers of the stage being consumed
    for (int t = 0; t < n_tiles; ++t) {
      zero(acc);
      for (int ks = 0; ks < nks; ++ks) {
        const uint32_t cw = lds0 + (uint32_t)wbuf * kLmWBytes, ch = lds0 + (uint32_t)hbuf * Sh::HBytes;
        const int nwbuf = wbuf + 1 == Sh::WB ? 0 : wbuf + 1, nhbuf = hbuf ^ 1;
        const uint32_t nw = lds0 + (uint32_t)nwbuf * kLmWBytes, nh = lds0 + (uint32_t)nhbuf * Sh::HBytes;
        // first half: MFMAs on the stage's half 0, its half 1 read in between
        LM_FENCE();
        half((cw + a_addr0) ^ kHalf, (ch + b_addr0) ^ kHalf, false);
        // every wave has read all of this stage's buffers, and the next stage
        // has landed (only the weight part of the one after is outstanding)
        LM_FENCE();
        lm_sync<kLmWDma>();
        // second half: MFMAs on half 1; the next stage's half 0 read, and the
        // hidden part of the stage after next and the weight part of the one
        // after that loaded into this stage's buffers, in between
        half(nw + a_addr0, nh + b_addr0, true);
        LM_FENCE();
        advance_h();
        advance_w();
        wbuf = nwbuf;
        hbuf = nhbuf;
      }
      fold(t, acc);
    }
#undef LM_M
  } else {
    // narrow tiles, bound by the read of the weights: D stages resident, one
    // barrier a stage; the loads of the stage D - 1 ahead go out first, into
    // the buffers that every wave finished reading before the barrier.  The
    // sums of the even and of the odd 16-stage blocks are kept apart (lm_flip)
    // and, where the registers allow it, formed in chains of 8 stages: the
    // error of a chain of float32 sums grows with its length.
    constexpr int D = Sh::WB, NH = Sh::HDma, kChain = 8;
    static_assert(Sh::HB == D && (D == 3 || D == 4), "equal stages");
    // the weights of the first stages, before the positions are looked up
#pragma unroll
    for (int s = 0; s < D - 1; ++s) {
#pragma unroll
      for (int j = NH; j < NL; ++j) dma(j);
      advance_w();
    }
    hidden_rows();
#pragma unroll
    for (int s = 0; s < D - 1; ++s) {
#pragma unroll
      for (int j = 0; j < NH; ++j) dma(j);
      advance_h();
    }
    int buf = 0, done = 0;
    for (int t = 0; t < n_tiles; ++t) {
      f32x4 cur[MI][NI], other[MI][NI];     // even and odd blocks, in turn
      zero(cur);
      zero(other);
      auto add = [&](f32x4 (&to)[MI][NI], const f32x4 (&x)[MI][NI]) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) to[mi][ni] += x[mi][ni];
      };
      auto stages = [&](f32x4 (&acc)[MI][NI], int count) {
        for (int k = 0; k < count; ++k) {
          // stage `done` has landed: outstanding may be the hidden parts of
          // the prologue's later stages and whole stages issued since
          if (done == 0) lm_sync<(D - 2) * NH>();
          else if (D == 4 && done == 1) lm_sync<NH + NL>();
          else lm_sync<(D - 2) * NL>();
          ++done;
#pragma unroll
          for (int j = 0; j < NL; ++j) dma(j);
          advance_h();
          advance_w();
          const uint32_t cw = lds0 + (uint32_t)buf * kLmWBytes, ch = lds0 + (uint32_t)buf * Sh::HBytes;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            bf16x8 fa[MI], fb[NI];
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) fb[ni] = lds_at(((ch + b_addr0) ^ (h * kHalf)) + ni * 16 * kLmRowBytes);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) fa[mi] = lds_at(((cw + a_addr0) ^ (h * kHalf)) + mi * 16 * kLmRowBytes);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
              for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[mi], fb[ni], acc[mi][ni], 0, 0, 0);
          }
          buf = buf + 1 == D ? 0 : buf + 1;
        }
      };
      for (int k0 = 0; k0 < nks; k0 += kLmFlip) {
        if constexpr (Sh::PT <= 64) {
          for (int k1 = k0; k1 < min(nks, k0 + kLmFlip); k1 += kChain) {
            f32x4 acc[MI][NI];
            zero(acc);
            stages(acc, min(kChain, nks - k1));
            add(cur, acc);
          }
        } else {
          stages(cur, min(kLmFlip, nks - k0));
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) {
            const f32x4 x = cur[mi][ni];
            cur[mi][ni] = other[mi][ni];
            other[mi][ni] = x;
          }
      }
      add(cur, other);
      fold(t, cur);
    }
  }
  // the 4 WV states of a position (lanes l, l + 16, l + 32, l + 48 of the WV
  // waves on its vocabulary rows) meet in LDS, once no load is still writing
  // into it; small loops for the same reason as in lm_fold
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  constexpr int NS = 4 * WV, PP = kLmThreads / Sh::PT < NS ? kLmThreads / Sh::PT : NS;
  constexpr int kPer = NS / PP;                 // states per thread in the first round
  constexpr bool kAll = Sh::PT <= kLmThreads;
  static_assert(kAll && NS % PP == 0 && NS * Sh::PT * 16 <= (int)kLmLdsBytes, "the exchange");
  float* xm = reinterpret_cast<float*>(lm_lds);                       // [NS][PT] maxima
  int* xf = reinterpret_cast<int*>(xm + NS * Sh::PT);                 // their indices
  double* xs = reinterpret_cast<double*>(xf + NS * Sh::PT);           // sums
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const int at = (4 * vw + lane / 16) * Sh::PT + 16 * (NI * pw + ni) + lane % 16;
    xm[at] = st[ni].M;
    xf[at] = st[ni].first;
    xs[at] = st[ni].S;
  }
  __syncthreads();
  const int r = tid % Sh::PT, part = tid / Sh::PT;
  // adds `n` states of position r, from entry s0 on, `step` apart
  auto meet = [&](int s0, int n, int step) {
    LmState c{kNegInf, kRefFloor, 0.0, 0x7fffffff};
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
      const int at = (s0 + k * step) * Sh::PT + r;
      const float m = xm[at];
      lm_combine(c, m, lm_ref(m), xs[at], xf[at]);
    }
    return c;
  };
  if (part < PP) {
    const LmState c = meet(part * kPer, kPer, 1);
    const int at = part * kPer * Sh::PT + r;    // this thread's first entry
    xm[at] = c.M;
    xf[at] = c.first;
    xs[at] = c.S;
  }
  __syncthreads();
  if (part == 0 && r < cnt) {
    const LmState c = meet(0, PP, kPer);
    a.partials[(size_t)(p0 + r) * stride + split] = WavePartial{c.M, c.K, c.S, c.first};
  }
  __syncthreads();   // the next segment loads into the buffers
}

// Workgroup g's segments.  Two kernels, each for its tile widths, both
// launched where the candidates may be either (the other one's workgroups
// leave at once): in one kernel the wide tiles' registers made the narrow
// ones reload spilled values in the fold, and such a reload waits for every
// weight load in flight.
// One: a single position tile, so one segment at most (a loop here made
// k_lm_wide<true> spill registers).
template <bool One, class F>
__device__ __forceinline__ void lm_segments(const LmArgs& a, const LmWork& w, int n, F&& segment) {
  const int g = blockIdx.x;
  const int end = lm_seg_end(w, g);
  int u = lm_seg_first(w, g);
  if (u >= end) return;
  do {
    // uniform values out of divisions: scalar registers
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int s = One ? u : uni(u / w.mt);
    const int p0 = One ? 0 : uni((u - s * w.mt) * w.pt), cnt = One ? n : uni(min(w.pt, n - p0));
    const int v_beg = uni(lm_first(w, s) * w.unit);
    const int v_end = uni((int)min((long long)a.V, (long long)lm_first(w, s + 1) * w.unit));
    segment(p0, cnt, v_beg, v_end, w.k, s);
    u += kLmGroups / kLmXcds;
  } while (!One && u < end);
}

// The candidate positions, in position order, found by every workgroup for
// itself from at most kLmSelf positions (one round trip to memory instead of
// a launch): the first kLmNarrow of them go to `list` (LDS), the number is
// returned.  Workgroup 0 also writes them all out with their number, for the
// kernels that follow, and the default outputs of the other positions.
struct LmCand {
  const uint8_t* mask;
  const int32_t* bstart;
  const int32_t* bend;
  int B, L;
  RowOut out;
};
constexpr int kLmNarrow = 128;                             // most candidates of the narrow kernel
constexpr int kLmSelfChunks = 4;
constexpr int kLmSelf = kLmSelfChunks * kLmThreads;        // 2048

__device__ __forceinline__ int lm_find(const LmCand& c, int32_t* list, int* waves_n, int32_t* rows,
                                       int32_t* count) {
  const int n = c.B * c.L;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int s[kLmSelfChunks], e[kLmSelfChunks], q[kLmSelfChunks];
  bool m[kLmSelfChunks];
#pragma unroll
  for (int k = 0; k < kLmSelfChunks; ++k) {
    const int i = k * kLmThreads + (int)threadIdx.x;
    const int ic = i < n ? i : 0;                          // past the end: position 0, not used
    const int b = (int)((unsigned)ic / (unsigned)c.L);
    q[k] = ic - b * c.L;
    s[k] = c.bstart[b];
    e[k] = c.bend[b];
    m[k] = c.mask[ic] != 0;
  }
  unsigned long long bal[kLmSelfChunks];
#pragma unroll
  for (int k = 0; k < kLmSelfChunks; ++k) {
    const int i = k * kLmThreads + (int)threadIdx.x;
    const bool cand = i < n && m[k] && window_ok(s[k], e[k], c.L) && q[k] >= s[k] && q[k] < e[k];
    if (blockIdx.x == 0 && i < n && !cand) store_default(c.out, (size_t)i);
    bal[k] = __ballot(cand);
    if (lane == 0) waves_n[k * kLmWaves + wave] = __popcll(bal[k]);
  }
  __syncthreads();
  static_assert(kLmSelfChunks * kLmWaves <= kWave, "one lane per (chunk, wave)");
  const int own = lane < kLmSelfChunks * kLmWaves ? waves_n[lane] : 0;
  int incl = own;
#pragma unroll
  for (int x = 1; x < kLmSelfChunks * kLmWaves; x <<= 1) {
    const int o = __shfl_up(incl, x);
    if (lane >= x) incl += o;
  }
  const int total = __builtin_amdgcn_readlane(incl, kLmSelfChunks * kLmWaves - 1);
#pragma unroll
  for (int k = 0; k < kLmSelfChunks; ++k) {
    const int base = __shfl(incl - own, k * kLmWaves + wave);
    if ((bal[k] >> lane) & 1ull) {
      const int at = base + __popcll(bal[k] & ((1ull << lane) - 1ull));
      const int i = k * kLmThreads + (int)threadIdx.x;
      if (at < kLmNarrow) list[at] = i;
      if (blockIdx.x == 0) rows[at] = i;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = total;
  __syncthreads();
  return total;
}

// at most kLmNarrow candidates.  Self: at most kLmSelf positions, compacted
// here; otherwise the candidates were listed before.
template <bool Self>
__global__ void __launch_bounds__(kLmThreads) k_lm_narrow(LmArgs a, LmCand c) {
  // the list sits behind the stages
  extern __shared__ __attribute__((aligned(1024))) char lm_lds[];
  int32_t* list = reinterpret_cast<int32_t*>(lm_lds + kLmStageBytes);
  int n;
  if constexpr (Self) n = lm_find(c, list, list + kLmNarrow, a.rows, a.count);
  else n = *a.count;
  n = __builtin_amdgcn_readfirstlane(n);
  if (n == 0 || n > kLmNarrow) return;
  const LmWork w = lm_work_tiles(n, a.V);
  const int32_t* rows = Self ? list : a.rows;
  const int flip = lm_flip((int)blockIdx.x, a.d / kLmBK);
  lm_segments<true>(a, w, n, [&](int p0, int cnt, int v_beg, int v_end, int stride, int split) {
    if (w.pt == 32) lm_segment<LmShape<32, 8, 4, 4>, true>(a, rows, p0, cnt, v_beg, v_end, flip, stride, split);
    else if (w.pt == 64) lm_segment<LmShape<64, 8, 3, 3>, true>(a, rows, p0, cnt, v_beg, v_end, flip, stride, split);
    else lm_segment<LmShape<128, 4, 3, 3>, true>(a, rows, p0, cnt, v_beg, v_end, flip, stride, split);
  });
}

// One: a single position tile (129..256 candidates), the weights read once;
// otherwise more than 256 candidates.
template <bool One>
__global__ void __launch_bounds__(kLmThreads)
k_lm_wide(LmArgs a) {
  const int n = __builtin_amdgcn_readfirstlane(*a.count);
  if (One ? (n <= 128 || n > kLmMaxPt) : n <= kLmMaxPt) return;
  const LmWork w = One ? lm_work_tiles(n, a.V) : lm_work_device(n, a.V, a.d);
  lm_segments<One>(a, w, n, [&](int p0, int cnt, int v_beg, int v_end, int stride, int split) {
    if (w.pt == 192) lm_segment<LmShape<192, 2, 3, 2>, One>(a, a.rows, p0, cnt, v_beg, v_end, 0, stride, split);
    else lm_segment<LmShape<256, 2, 3, 2>, One>(a, a.rows, p0, cnt, v_beg, v_end, 0, stride, split);
  });
}

// ---------------------------------------------------------------------------
// at most kLsRows positions in all (one sequence's block)
// ---------------------------------------------------------------------------
// With few positions the LM head is bound by reading W once (2 V d bytes;
// the 2 N V d flop are a few percent of the matrix cores' time), and the rate
// of that read depends on how it is issued: streams that each read a few rows
// 8 KiB apart reach ~5 TB/s, a contiguous range per workgroup read by global
// loads ~7 TB/s, the same range by buffer_load ... lds ~6.2 TB/s.  Here every
// workgroup streams a contiguous range of W, kLsBlk whole rows (16 d bytes)
// per block: each wave load instruction reads 1 KiB in address order into
// registers, which are stored to LDS while the next block's loads are in
// flight.
// The 8 waves split the hidden dimension and keep their share of the
// positions' hidden operands in registers for the whole kernel; per block each
// wave runs its MFMAs over its share (A = the block's rows from LDS, B = the
// hidden operands), and 256 threads each sum one (row, position) logit over
// the 8 partial products and fold it into their own running state; the 8 row
// states of a position are combined at the end.  Every workgroup finds the
// candidate positions itself (there are at most 32); workgroup 0 also writes
// them out, with their count, for the finish, and the default outputs of the
// other positions.
constexpr int kLsRows = 32;        // positions served (two 16-column MFMA blocks)
constexpr int kLsWaves = 8;
constexpr int kLsBlk = 8;          // vocabulary rows per block
constexpr int kLsMaxD = 4096;      // hidden operands held in registers: d / 8 per wave
constexpr size_t kLsRedBytes = (size_t)kLsWaves * 2 * kWave * sizeof(f32x4);  // 16 KiB
// two row blocks and two sets of the waves' partial products (160 KiB at
// d = 4096, all of a CU's LDS)
constexpr size_t kLsLdsBytes(int d) { return 2 * (size_t)kLsBlk * d * 2 + 2 * kLsRedBytes; }

__device__ __forceinline__ int ls_swz(int r) { return r & 7; }

// DM = d / 512: 16-byte loads per thread and block; 2 DM 32-element chunks
// of the hidden dimension per wave
template <int DM>
__global__ void __launch_bounds__(kLsWaves * kWave)
k_lm_stream(const uint16_t* __restrict__ hidden, const uint16_t* __restrict__ weight,
            const uint8_t* __restrict__ mask, const int32_t* __restrict__ bstart,
            const int32_t* __restrict__ bend, int B, int L, int V, int32_t* __restrict__ rows,
            int32_t* __restrict__ count, RowOut out, WavePartial* __restrict__ partials,
            int n_split) {
  constexpr int d = DM * 512;
  constexpr int NC = 2 * DM;                                 // 32-element chunks per wave
  constexpr int vec_row = d / 8;                             // 16-byte vectors per row
  constexpr uint32_t blk_bytes = (uint32_t)kLsBlk * d * 2;
  extern __shared__ __attribute__((aligned(1024))) char ls_lds[];
  // the candidate list sits in the second set of partial products, first
  // written after the loop's second barrier
  int32_t* cand_rows = reinterpret_cast<int32_t*>(ls_lds + 2 * blk_bytes + kLsRedBytes);
  int* cand_n = reinterpret_cast<int*>(cand_rows + kLsRows);
  const int t = threadIdx.x;
  const int lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int g = blockIdx.x;
  const int G = gridDim.x;

  // the candidate positions, in position order (B L <= kLsRows)
  if (wave == 0) {
    const int n = B * L;
    bool cand = false;
    if (lane < n) {
      const int b = lane / L, q = lane % L;
      const int s = bstart[b], e = bend[b];
      cand = window_ok(s, e, L) && q >= s && q < e && mask[lane] != 0;
    }
    const unsigned long long bal = __ballot(cand);
    const int idx = __popcll(bal & ((1ull << lane) - 1ull));
    if (cand) cand_rows[idx] = lane;
    if (lane == 0) *cand_n = __popcll(bal);
    if (g == 0) {
      if (cand) rows[idx] = lane;
      else if (lane < n) store_default(out, lane);
      if (lane == 0) *count = __popcll(bal);
    }
  }
  __syncthreads();
  const int nrows = *cand_n;
  if (nrows == 0) return;

  const int nblk = (V + kLsBlk - 1) / kLsBlk;
  const int b_beg = (int)((long long)g * nblk / G), b_end = (int)((long long)(g + 1) * nblk / G);
  const int cnt = b_end - b_beg;
  // partial products of block i in set i % 2: f32x4 [wave][ni][lane]
  float* red = reinterpret_cast<float*>(ls_lds + 2 * blk_bytes);
  const int k0 = wave * (d / kLsWaves);

  // the hidden operands of this wave's share, for positions 16 ni + l % 16
  // (past the count: the first row; their results are not stored)
  u32x4 hb[NC][2];
  {
    const int q0 = lane % 16, q1 = 16 + lane % 16;
    const uint16_t* h0 = hidden + (size_t)cand_rows[q0 < nrows ? q0 : 0] * d + k0 + 8 * (lane / 16);
    const uint16_t* h1 = hidden + (size_t)cand_rows[q1 < nrows ? q1 : 0] * d + k0 + 8 * (lane / 16);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      hb[c][0] = *reinterpret_cast<const u32x4*>(h0 + 32 * c);
      hb[c][1] = *reinterpret_cast<const u32x4*>(h1 + 32 * c);
    }
  }
  // block loads: thread t loads the block's 16-byte vectors j * 512 + t into
  // registers (each wave instruction reads 1 KiB of W in address order) and
  // stores them to LDS slot (row r, vector s ^ ls_swz(r)): the rows are 2 d
  // bytes apart, a multiple of the bank period, and the swizzle puts the
  // operand reads of the 8 rows in distinct banks.
  const u32x4* wv = reinterpret_cast<const u32x4*>(weight);
  u32x4 stg[DM];
  auto load_regs = [&](int i) {
    const int vb = (b_beg + i) * kLsBlk;
#pragma unroll
    for (int j = 0; j < DM; ++j) {
      const int slot = j * kLsWaves * kWave + t;
      const int v = min(vb + slot / vec_row, V - 1);         // rows past V repeat the last
      stg[j] = __builtin_nontemporal_load(wv + (size_t)v * vec_row + slot % vec_row);
    }
  };
  auto store_lds = [&](int buf) {
    u32x4* bl = reinterpret_cast<u32x4*>(ls_lds + buf * blk_bytes);
#pragma unroll
    for (int j = 0; j < DM; ++j) {
      const int slot = j * kLsWaves * kWave + t;
      const int r = slot / vec_row, sv = slot % vec_row;
      bl[r * vec_row + (sv ^ ls_swz(r))] = stg[j];
    }
  };
  // the (row, position) of this thread's running state: threads 0..255 take
  // row fr = t / 32 of every block and position fp = t % 32
  const int fr = t / kLsRows, fp = t % kLsRows;
  const bool folds = t < kLsBlk * kLsRows;
  // where the logit of (fr, fp) sits among the waves' accumulators:
  // ni = fp / 16, lane 16 (fr / 4) + fp % 16, element fr % 4
  const int red_idx = ((fp / 16) * kWave + 16 * (fr / 4) + fp % 16) * 4 + fr % 4;
  LmState st{kNegInf, kRefFloor, 0.0, 0x7fffffff};
  // sums block i's 8 partial products of (fr, fp) and folds the logit
  auto fold = [&](int i) {
    const float* rs = red + (i & 1) * (kLsRedBytes / sizeof(float));
    const int v = (b_beg + i) * kLsBlk + fr;
    if (folds && v < V) {
      float x = rs[red_idx];
#pragma unroll
      for (int w = 1; w < kLsWaves; ++w) x += rs[w * 2 * kWave * 4 + red_idx];
      if (x > st.M) {
        const float Kn = exp_ref(x);
        st.S = rescale(st.S, st.K, Kn);
        st.K = Kn;
        st.M = x;
        st.first = v;
      }
      st.S += (double)term(x, st.K);
    }
  };
  // operand address of this lane in a buffer: row l % 8 (rows 8..15 of the
  // MFMA block repeat rows 0..7), vector k0 / 8 + 4 c + l / 16
  const int ar = lane % kLsBlk;
  const int a_row = ar * vec_row;

  load_regs(0);
  store_lds(0);
  // vmcnt(0): the hidden operands have arrived before the loop, so inside it
  // the only loads in flight are the next block's, waited for at its store
  // (without this the loop would wait for every load at its first MFMAs)
  __builtin_amdgcn_s_waitcnt(0x0f70);
  if (cnt > 1) load_regs(1);
  for (int it = 0; it < cnt; ++it) {
    const int buf = it & 1;
    // one barrier per block: block it is in LDS (stored during the previous
    // iteration), the previous block's partial products are complete, and
    // the fold that read this iteration's set (two blocks back) is done
    __syncthreads();
    const u32x4* bl = reinterpret_cast<const u32x4*>(ls_lds + buf * blk_bytes);
    // two accumulators per column block halve the dependent MFMA chain
    f32x4 acc[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[h][ni][i] = 0.0f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int sv = k0 / 8 + 4 * c + lane / 16;
      const bf16x8 a = __builtin_bit_cast(bf16x8, bl[a_row + (sv ^ ls_swz(ar))]);
#pragma unroll
      for (int ni = 0; ni < 2; ++ni)
        acc[c & 1][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            a, __builtin_bit_cast(bf16x8, hb[c][ni]), acc[c & 1][ni], 0, 0, 0);
    }
    f32x4* redv = reinterpret_cast<f32x4*>(red + buf * (kLsRedBytes / sizeof(float)));
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) redv[(wave * 2 + ni) * kWave + lane] = acc[0][ni] + acc[1][ni];
    // the previous block's logits, while other waves still multiply
    if (it > 0) fold(it - 1);
    // the next block into the buffer every wave finished reading before the
    // barrier above, then the block after it into the registers
    if (it + 1 < cnt) store_lds(buf ^ 1);
    if (it + 2 < cnt) load_regs(it + 2);
  }
  __syncthreads();
  fold(cnt - 1);
  // the row states of a position meet in LDS (the row buffers are free)
  __syncthreads();
  WavePartial* xs = reinterpret_cast<WavePartial*>(ls_lds);
  if (folds) xs[fr * kLsRows + fp] = WavePartial{st.M, st.K, st.S, st.first};
  __syncthreads();
  if (t < kLsRows && t < nrows) {
    LmState c = {xs[t].m, xs[t].K, xs[t].S, xs[t].first};
#pragma unroll
    for (int r = 1; r < kLsBlk; ++r) {
      const WavePartial o = xs[r * kLsRows + t];
      lm_combine(c, o.m, o.K, o.S, o.first);
    }
    partials[(size_t)t * n_split + g] = WavePartial{c.M, c.K, c.S, c.first};
  }
}

// Per candidate row, one wavefront: lane l combines the splits l, l+64, ...
// of the row's contiguous partials, all loaded at once, then a fixed
// butterfly over the lanes (both partners of every step form the same sum)
// and the finish.
constexpr int kLmFinishPer = kLmGroups / kWave;   // partials per lane at most
__device__ __forceinline__ void lm_finish_row(const WavePartial* p, int n_split, int row, RowOut out) {
  const int lane = threadIdx.x % kWave;
  WavePartial q[kLmFinishPer];
#pragma unroll
  for (int i = 0; i < kLmFinishPer; ++i) {
    const int j = lane + i * kWave;
    q[i] = p[j < n_split ? j : 0];
  }
  float M = kNegInf;
#pragma unroll
  for (int i = 0; i < kLmFinishPer; ++i) M = fmaxf(M, q[i].m);
  M = wave_max(M);
  const float K = exp_ref(M);
  double S = 0.0;
  int first = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < kLmFinishPer; ++i) {
    if (lane + i * kWave < n_split) S += rescale(q[i].S, q[i].K, K);
    if (q[i].m == M) first = min(first, q[i].first);
  }
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) S += __shfl_xor(S, d);
  first = wave_min(first);
  if (lane == 0) store_row(out, (size_t)row, finish_row(M, K, S, first));
}

__global__ void __launch_bounds__(256)
k_lm_finish(const int32_t* __restrict__ rows, const int32_t* __restrict__ count,
            const WavePartial* __restrict__ partials, int d, int V, RowOut out) {
  const int r = blockIdx.x * 4 + threadIdx.x / kWave;
  const int n = *count;
  if (r >= n) return;
  const int k = lm_work_device(n, V, d).k;
  lm_finish_row(partials + (size_t)r * k, k, rows[r], out);
}

// the same for the streaming kernel's partials, n_split of every row
__global__ void __launch_bounds__(256)
k_lm_finish_n(const int32_t* __restrict__ rows, const int32_t* __restrict__ count,
              const WavePartial* __restrict__ partials, int n_split, RowOut out) {
  const int k = blockIdx.x * 4 + threadIdx.x / kWave;
  if (k < *count) lm_finish_row(partials + (size_t)k * n_split, n_split, rows[k], out);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// The streaming kernel serves at most kLsRows positions when a block is a
// whole number of 16-byte loads per thread and each wave's share of the hidden
// operands fits its registers; everything else the tiles.  At 32 positions of
// d = 4096, V = 126464 the two take the same 163 us, at 8 positions of
// d = 1024, V = 16000 15.5 us against 20.3 (a tile is 256 rows high, and a
// workgroup's share of a small vocabulary is not); at 64 positions the tiles
// take the 163 us of 32.
static bool lm_streams(long long n, int d) { return n <= kLsRows && d % 512 == 0 && d <= kLsMaxD; }

// the streaming kernel for d = 512 DM
typedef void (*LmStreamFn)(const uint16_t*, const uint16_t*, const uint8_t*, const int32_t*,
                           const int32_t*, int, int, int, int32_t*, int32_t*, RowOut, WavePartial*,
                           int);
static const LmStreamFn kLmStream[kLsMaxD / 512] = {
    k_lm_stream<1>, k_lm_stream<2>, k_lm_stream<3>, k_lm_stream<4>,
    k_lm_stream<5>, k_lm_stream<6>, k_lm_stream<7>, k_lm_stream<8>};

struct LmPlan {
  bool stream;   // k_lm_stream, not the tiles
  int n_split;   // its workgroups
  size_t off_rows, off_partials, off_out, bytes;
};

// One workgroup per compute unit.  k_lm_stream: each a contiguous range of
// row blocks; the tiles: as the number of candidates says, on the device
// (lm_work).
static LmPlan lm_plan(int B, int L, int d, int V, bool need_out) {
  LmPlan p{};
  const long long n = (long long)B * L;
  p.stream = lm_streams(n, d);
  const int nblk = (V + kLsBlk - 1) / kLsBlk;
  p.n_split = nblk < kLmGroups ? nblk : kLmGroups;
  const size_t partials = p.stream ? (size_t)n * p.n_split : lm_max_partials(n, V);
  p.off_rows = 256;
  p.off_partials = p.off_rows + align256((size_t)n * 4);
  p.off_out = p.off_partials + align256(partials * sizeof(WavePartial));
  p.bytes = p.off_out + (need_out ? 3 * align256((size_t)n * 4) : 0);
  return p;
}

static bool lm_sizes_ok(int B, int L, int d, int V) {
  if (B < 0 || L < 1 || V < 1 || d < 64 || d % 64 != 0) return false;
  // hidden is addressed by 32-bit byte offsets (buffer loads)
  return (long long)B * L * d * 2 <= 0xffffffffLL && (long long)V * (d / 8) < 0x7fffffffLL;
}

// The streaming and tiled kernels' dynamic LDS (up to 160 KiB) is above the
// default limit; the limit is raised once per device, before the first launch
// there.
constexpr int kLmMaxDevices = 64;
static std::atomic<bool> lm_lds_allowed[kLmMaxDevices];

static hipError_t lm_allow_lds() {
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev >= 0 && dev < kLmMaxDevices && lm_lds_allowed[dev].load(std::memory_order_acquire))
    return hipSuccess;
  hipError_t a = hipFuncSetAttribute((const void*)k_lm_narrow<true>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLmLdsBytes);
  if (a == hipSuccess)
    a = hipFuncSetAttribute((const void*)k_lm_narrow<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kLmLdsBytes);
  if (a == hipSuccess)
    a = hipFuncSetAttribute((const void*)k_lm_wide<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kLmLdsBytes);
  if (a == hipSuccess)
    a = hipFuncSetAttribute((const void*)k_lm_wide<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kLmLdsBytes);
  for (int i = 0; i < kLsMaxD / 512 && a == hipSuccess; ++i)
    a = hipFuncSetAttribute((const void*)kLmStream[i], hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kLsLdsBytes(512 * (i + 1)));
  if (a == hipSuccess && dev >= 0 && dev < kLmMaxDevices)
    lm_lds_allowed[dev].store(true, std::memory_order_release);
  return a;
}

static hipError_t lm_launch(const void* hidden, const void* weight, int B, int L, int d, int V,
                            const uint8_t* mask, const int32_t* bs, const int32_t* be, RowOut out,
                            char* ws, const LmPlan& p, hipStream_t st) {
  int32_t* count = (int32_t*)ws;
  int32_t* rows = (int32_t*)(ws + p.off_rows);
  WavePartial* part = (WavePartial*)(ws + p.off_partials);
  const hipError_t attr = lm_allow_lds();
  if (attr != hipSuccess) return attr;
  const long long n = (long long)B * L;
  if (p.stream) {
    // the streaming kernel compacts the candidates itself
    hipLaunchKernelGGL(kLmStream[d / 512 - 1], dim3((unsigned)p.n_split), dim3(kLsWaves * kWave),
                       kLsLdsBytes(d), st, (const uint16_t*)hidden, (const uint16_t*)weight, mask,
                       bs, be, B, L, V, rows, count, out, part, p.n_split);
    hipLaunchKernelGGL(k_lm_finish_n, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, rows, count,
                       part, p.n_split, out);
  } else {
    const LmArgs a{(const uint16_t*)hidden, (const uint16_t*)weight, rows, count, part, d, V,
                   (uint32_t)((size_t)B * L * d * 2)};
    const LmCand c{mask, bs, be, B, L, out};
    const dim3 grid(kLmGroups), block(kLmThreads);
    if (n <= kLmSelf) {
      hipLaunchKernelGGL(k_lm_narrow<true>, grid, block, kLmLdsBytes, st, a, c);
    } else {
      if (n <= kLmOneWg) {
        hipLaunchKernelGGL(k_lm_compact_one, dim3(1), dim3(kLmOneThreads), 0, st, mask, bs, be, B, L,
                           rows, count, out);
      } else {
        hipLaunchKernelGGL(k_lm_zero, dim3(1), dim3(64), 0, st, count);
        hipLaunchKernelGGL(k_lm_compact, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, st, mask, bs, be,
                           B, L, rows, count, out);
      }
      hipLaunchKernelGGL(k_lm_narrow<false>, grid, block, kLmLdsBytes, st, a, c);
    }
    // the host knows the span, the device the candidates: the kernels whose
    // range the number is not in return at once
    if (n > kLmNarrow) hipLaunchKernelGGL(k_lm_wide<true>, grid, block, kLmLdsBytes, st, a);
    if (n > kLmMaxPt) hipLaunchKernelGGL(k_lm_wide<false>, grid, block, kLmLdsBytes, st, a);
    hipLaunchKernelGGL(k_lm_finish, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, rows, count, part,
                       d, V, out);
  }
  return hipGetLastError();
}

}  // namespace fdllm

using namespace fdllm;

extern "C" {

fdllm_status fdllm_lmhead_workspace_size(int B, int L, int d, int V, size_t* bytes) {
  if (!bytes) return FDLLM_ERR_INVALID_ARG;
  if (B < 0 || L < 1) return FDLLM_ERR_INVALID_ARG;
  if (!lm_sizes_ok(B, L, d, V)) return FDLLM_ERR_SIZE;
  *bytes = lm_plan(B, L, d, V, true).bytes;
  return FDLLM_OK;
}

static fdllm_status lm_common(const void* hidden, const void* weight, int B, int L, int d, int V,
                              const uint8_t* mask, const int32_t* bs, const int32_t* be,
                              RowOut& out, void* workspace, size_t workspace_bytes, hipStream_t st) {
  if (B < 0 || L < 1) return FDLLM_ERR_INVALID_ARG;
  if (!lm_sizes_ok(B, L, d, V)) return FDLLM_ERR_SIZE;
  if (!hidden || !weight || !mask || !bs || !be) return FDLLM_ERR_INVALID_ARG;
  if (((uintptr_t)hidden % 16) != 0 || ((uintptr_t)weight % 16) != 0) return FDLLM_ERR_INVALID_ARG;
  const bool need_out = !out.tokens || !out.conf || !out.eps;
  const LmPlan p = lm_plan(B, L, d, V, need_out);
  if (!workspace || workspace_bytes < p.bytes) return FDLLM_ERR_WORKSPACE;
  char* ws = (char*)workspace;
  const size_t n = (size_t)B * L;
  if (!out.tokens) out.tokens = (int32_t*)(ws + p.off_out);
  if (!out.conf) out.conf = (float*)(ws + p.off_out + align256(n * 4));
  if (!out.eps) out.eps = (float*)(ws + p.off_out + 2 * align256(n * 4));
  return lm_launch(hidden, weight, B, L, d, V, mask, bs, be, out, ws, p, st) == hipSuccess
             ? FDLLM_OK
             : FDLLM_ERR_HIP;
}

fdllm_status fdllm_lmhead_confidence(const void* hidden, const void* weight, int B, int L, int d,
                                     int V, const uint8_t* mask, const int32_t* block_start,
                                     const int32_t* block_end, int32_t* tokens, float* conf,
                                     float* eps, float* lse, void* workspace,
                                     size_t workspace_bytes, fdllm_stream stream) {
  if (B == 0 && L >= 1) return FDLLM_OK;
  if (!tokens || !conf) return FDLLM_ERR_INVALID_ARG;
  RowOut out{tokens, conf, eps, lse};
  return lm_common(hidden, weight, B, L, d, V, mask, block_start, block_end, out, workspace,
                   workspace_bytes, (hipStream_t)stream);
}

fdllm_status fdllm_lmhead_decode_step(const void* hidden, const void* weight, int B, int L, int d,
                                      int V, uint8_t* mask, const int32_t* block_start,
                                      const int32_t* block_end, int32_t* x, fdllm_selector sel,
                                      float param, const float* eta, float eta_uniform,
                                      int32_t* tokens, float* conf, float* eps, float* lse,
                                      uint8_t* commit, int32_t* n_commit, void* workspace,
                                      size_t workspace_bytes, fdllm_stream stream) {
  if (sel != FDLLM_SEL_THRESHOLD && sel != FDLLM_SEL_FACTOR && sel != FDLLM_SEL_PROFILE &&
      sel != FDLLM_SEL_ROBUST)
    return FDLLM_ERR_INVALID_ARG;
  if (!(eta_uniform == eta_uniform)) return FDLLM_ERR_INVALID_ARG;
  if (B == 0 && L >= 1) return FDLLM_OK;
  if (!x) return FDLLM_ERR_INVALID_ARG;
  RowOut out{tokens, conf, eps, lse};
  hipStream_t st = (hipStream_t)stream;
  const fdllm_status s1 = lm_common(hidden, weight, B, L, d, V, mask, block_start, block_end, out,
                                    workspace, workspace_bytes, st);
  if (s1 != FDLLM_OK) return s1;
  SelectIO io{out.conf, out.eps, mask, block_start, block_end, commit, n_commit, out.tokens, x,
              EtaIn{eta, eta_uniform}};
  return launch_select(sel, io, B, L, param, st) == hipSuccess ? FDLLM_OK : FDLLM_ERR_HIP;
}

}  // extern "C"
