// ART decode attention kernels for gfx950 (MI355X).
//
// One launch computes, for every (sequence b, KV head kvh) group, the
// block-streaming softmax attention of Sec. 3.1 over the group's traversal
// (recency-first, forward, or a supplied block list, Sec. 3.4), the
// magnitude/direction stability test of Sec. 3.2 (Eq. 2) after every block,
// the patience counter of Eq. (3) and the early break of Algorithm 1.
//
// Work decomposition
//   A group's traversal of T blocks is cut into chunks of consecutive
//   blocks (with the default plan, leading chunks of 3 blocks, then chunks
//   of C).  The chunks of all groups form eight chunk-major work lists
//   (list x holds the groups 8r + (x + r) mod 8 of every full run r of eight
//   groups, and the leftover groups g with g mod 8 = x: chunk 0 of each, then
//   chunk 1, ...).  The grid is persistent (as many workgroups as the chip holds);
//   workgroups take list indices from epoch-tagged queue words, so
//   workgroups freed by groups that stopped early move on to the groups that
//   stop late.  Each list is handed out in order and a chunk only waits on
//   earlier chunks of its own group, so every wait targets a chunk that some
//   workgroup already holds: no deadlock whatever the dispatch order.
//
//   Loaders (wavefronts 1..3): the leader claims a chunk when one of the two
//   LDS chunk buffers is free; the loaders stream its 64-token tiles from HBM
//   (16-byte loads, four 64-byte row segments per K load instruction, four
//   256-byte rows per V load instruction), compute the scores of all g query
//   heads with v_mfma_f32_16x16x32_bf16 (tokens are the M rows, query heads
//   the N columns, head dims the reduction), the tile softmax in base 2, and
//   P.V on the same MFMA with P split into three bf16 parts (fp32 accuracy),
//   and leave (m, l, sum p v) for each block in LDS.  Chunks after an
//   announced stop are not loaded, and a loader gives up a chunk mid-way
//   once a stop before it is announced.
//
//   Resolver (wavefront 0), per ready chunk:
//     - folds the blocks' records into the chunk aggregate;
//     - obtains the softmax state after the previous chunk (that chunk's
//       inclusive state, or the nearest inclusive state found by looking
//       back with the aggregates after it folded forward: always the same
//       left fold, so results never depend on timing) and publishes its own
//       inclusive state at once;
//     - replays its blocks from that prefix (normalised running output o(t),
//       increment d = o(t) - o(t-1)) and then runs the stability test on all
//       of them at once (d_scale = |d|, d_direction = 1 - cos from |o|^2,
//       |d|^2 and o.d without cancellation);
//     - publishes a stability summary, and announces "stop at or before this
//       chunk" at once when the chunk's own blocks hold a run of p stable
//       steps; if the chunk can hold the stop (or is the group's last chunk)
//       it looks back the same way over the stability states (entering
//       patience run, stop already found) and either stops inside the chunk
//       (announces the stop, then writes out/lse/stop_block) or, as the last
//       chunk, writes the untruncated result.
//   Cross-workgroup data goes through the workspace with device-coherent
//   accesses only, as the XCDs of MI355X have separate L2 caches (see the
//   workspace helpers below).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "art_internal.h"

namespace art {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kNegInf = -__builtin_inff();

// The kernel's parameters, read where they are used from the kernel argument
// segment through the scalar cache.  fresh() hides the pointer's origin from
// the compiler: it then loads a phase's fields in that phase, instead of
// holding all of them (about 60 registers' worth, with what it derives from
// them) in scalar registers across the whole kernel.  Held so, 140 of them
// were spilled to lanes of vector registers, and 1170 of the kernel's 3600
// instructions (g = 4) were v_readlane to fetch them back.
typedef const __attribute__((address_space(4))) KernelParams Params;
__device__ __forceinline__ Params* fresh(Params* p) {
  __asm__ __volatile__("" : "+s"(p));
  return p;
}
constexpr int kD = kHeadDim;

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// two floats to two bf16 (round to nearest even), one v_cvt_pk_bf16_f32
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);                       // round to nearest even
  return u >> 16;
}

// ---- wavefront reductions over the 16 lanes of a DPP row -------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
constexpr int kQuadXor1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kRowHalfMirror = 0x141; // lane i <- lane 7-i within each 8
constexpr int kRowMirror = 0x140;     // lane i <- lane 15-i within each 16
constexpr int kRowRor4 = 0x124;       // lane i <- lane i-4 of its row of 16 (= i+12)
constexpr int kRowRor8 = 0x128;       // lane i <- lane i-8 (= i+8)

// Every lane of the row ends with the same bits (each step adds the same two
// partial sums, only in swapped operand order).
__device__ __forceinline__ float row_sum(float x) {
  x = x + dpp_f<kQuadXor1>(x);
  x = x + dpp_f<kQuadXor2>(x);
  x = x + dpp_f<kRowHalfMirror>(x);
  x = x + dpp_f<kRowMirror>(x);
  return x;
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, dpp_f<kQuadXor1>(x));
  x = fmaxf(x, dpp_f<kQuadXor2>(x));
  x = fmaxf(x, dpp_f<kRowHalfMirror>(x));
  x = fmaxf(x, dpp_f<kRowMirror>(x));
  return x;
}

__device__ __forceinline__ float read_lane(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
// Maximum and sum over the four rows of 16 lanes (lanes l, l ^ 16, l ^ 32,
// l ^ 48), by gfx950's half swaps: each swap hands every lane both operands
// in the same order, so all four lanes end with the same bits.
__device__ __forceinline__ void swap_rows16(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  a = __int_as_float(r[0]);
  b = __int_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows32(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  a = __int_as_float(r[0]);
  b = __int_as_float(r[1]);
}
__device__ __forceinline__ float rows_max(float x) {
  float a, b;
  swap_rows16(x, a, b);
  swap_rows32(fmaxf(a, b), a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float rows_sum(float x) {
  float a, b;
  swap_rows16(x, a, b);
  swap_rows32(a + b, a, b);
  return a + b;
}

// LDS written by some lanes of this wave, read by others.  LDS operations of
// one wavefront complete in order; this waits for them and keeps the
// compiler from moving memory operations across.
__device__ __forceinline__ void wave_lds_sync() {
  __asm__ __volatile__("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  __asm__ __volatile__("" ::: "memory");
}

// The same ordering without the wait, where only this wave touches the
// memory: the LDS unit executes one wavefront's operations in the order they
// were issued, so a read issued after a write of any lane of the wave sees
// it, and a write issued after a read cannot overtake it.  Only the compiler
// has to be kept from reordering them.
__device__ __forceinline__ void wave_lds_order() {
  __asm__ __volatile__("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  __asm__ __volatile__("" ::: "memory");
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// single hardware instructions (about 1 ulp): the same bits wherever used
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// ---- workspace: cross-workgroup data ---------------------------------------
// Everything one workgroup hands to another (flags, softmax records,
// stability records, the stop announcement) is written and read only with
// agent-scope atomic accesses, which gfx950 performs coherently across the
// XCDs' L2 caches (sc1).  A writer waits for its data stores to complete
// (s_waitcnt vmcnt(0)) before it stores the flag; a reader issues its data
// loads only after the flag load has returned the expected value.  No L2
// write-back or invalidate is needed, so publishing costs a few stores.
__device__ __forceinline__ uint64_t ld_relaxed(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_coh_i32(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_coh_i32(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// wait until this wave's global stores have completed; also a compiler
// barrier for memory operations
__device__ __forceinline__ void stores_complete() {
  __asm__ __volatile__("s_waitcnt vmcnt(0)" ::: "memory");
}
__device__ __forceinline__ void compiler_fence() { __asm__ __volatile__("" ::: "memory"); }

// Flag words: epoch << 24 | state << 20 | payload (20 bits).  The stability
// states carry their data in the payload, so that they are published with a
// single store and read with the flag itself.
__device__ __forceinline__ uint64_t make_flag(uint64_t epoch, uint32_t state, uint32_t payload) {
  return (epoch << 24) | ((uint64_t)state << 20) | (uint64_t)payload;
}
__device__ __forceinline__ uint32_t flag_state(uint64_t v, uint64_t epoch) {
  return (v >> 24) == epoch ? (uint32_t)((v >> 20) & 7u) : 0u;
}
__device__ __forceinline__ uint32_t flag_payload(uint64_t v) { return (uint32_t)(v & 0xfffffu); }

// Bounded waits.  A wave that polls spin_limit times without seeing what it
// waits for gives up: it stores this call's epoch and the timeout status in
// the error word and ends.  Every other wait of the launch reads the error
// word every kErrPollEvery polls and ends as soon as it carries this call's
// epoch, so one give-up drains the whole grid within a few polls per wave
// instead of each dependent wait spinning out its own limit.  (A word left
// by an earlier call carries another epoch: it is reported by the status
// call but does not end this one.)
constexpr uint32_t kTimeoutStatus = 6u;   // ART_ERR_DEVICE_TIMEOUT
constexpr uint32_t kErrPollEvery = 16u;
__device__ __forceinline__ void raise_timeout(Params& P) {
  __hip_atomic_store(P.error_word, (P.epoch << 8) | kTimeoutStatus, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool launch_failed(Params& P) {
  return (ld_relaxed(P.error_word) >> 8) == P.epoch;
}
// Race stress (the build with ART_RACE_STRESS defined, a test build only):
// a pseudo-random delay of up to 7 sleeps of 8128 cycles at every point
// where one workgroup hands data to another or acts on what another handed
// over, keyed by the call, the group, the chunk and the site, so that the
// look-back's producers and consumers meet in orders a plain run rarely
// shows.  Delays only stretch time: every wait stays bounded.
__device__ __forceinline__ void stress_delay(Params& P, int gidx, int k, int site) {
#ifdef ART_RACE_STRESS
  uint32_t h = (uint32_t)P.epoch * 0x9E3779B1u ^ (uint32_t)gidx * 0x85EBCA77u ^
               (uint32_t)k * 0xC2B2AE3Du ^ (uint32_t)site * 0x27D4EB2Fu;
  h ^= h >> 15;
  h *= 0x2C1B3C6Du;
  h ^= h >> 12;
  const uint32_t n = __builtin_amdgcn_readfirstlane((h >> 8) & 7u);
  for (uint32_t i = 0; i < n; ++i) __builtin_amdgcn_s_sleep(127);
#else
  (void)P; (void)gidx; (void)k; (void)site;
#endif
}

// The give-up test of one poll of a wait loop (spin counts the polls made).
__device__ __forceinline__ bool wait_expired(Params& P, uint32_t spin) {
  if (spin >= P.spin_limit) {
    raise_timeout(P);
    return true;
  }
  return (spin % kErrPollEvery) == kErrPollEvery - 1 && launch_failed(P);
}

template <int G>
struct Cfg {
  static constexpr int HPL = G >= 4 ? G / 4 : 1;   // head slots per lane (state layout)
  static constexpr int HC = G > 8 ? 8 : G;          // heads per P.V pass
  static constexpr int REC = G * kD + 2 * G;        // floats per LDS tile record
  static constexpr int REP = G > 8 ? 1 : G > 4 ? 2 : 4;  // copies of the heads over the 16 score columns
  static constexpr int COLS = 16 / REP;             // columns of one copy
  static constexpr int GANG = G > 8 ? 1 : 3;        // blocks the resolver takes at a time (the loads of all in flight)
};

// Per-head softmax state in the "state layout": lane l covers dims
// 8*(l&15) .. +7 of heads (l>>4) + 4*k, k < HPL.  m is in base 2
// (scores * scale * log2 e), L is the mass sum 2^(s - m), o the normalised
// output.  L == 0 is the empty state.
template <int G>
struct State {
  float m[Cfg<G>::HPL];
  float L[Cfg<G>::HPL];
  float o[Cfg<G>::HPL][8];
};

template <int G>
__device__ __forceinline__ void state_clear(State<G>& s) {
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    s.m[k] = kNegInf;
    s.L[k] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s.o[k][e] = 0.f;
  }
}

// s <- s (+) p_0 (+) p_1 ... : softmax-weighted merges of disjoint token
// sets, left to right (the increment form of Appendix A, per head)
//   m' = max(m, m_i), L' = L 2^(m - m') + L_i 2^(m_i - m'),
//   o' = o + w (o_i - o), w = L_i 2^(m_i - m') / L'.
// A run of up to 16 records is merged in two parts.  First, once, lane
// (r, c) takes record c of head r + 4k: the running maxima come from a
// prefix maximum over the 16 lanes of a row (exact), and with them every
// record's factors old = 2^(m - m') and add = L_i 2^(m_i - m'), all records
// at once.  Then step by step: two operations for L', one reciprocal, three
// operations per output.  The results are those of merging one record after
// the other, bit for bit, wherever a run is cut.  (Each record's exponentials
// and their latency inside the step took the resolver 0.55 us a block.)
static_assert(kMaxChunkBlocks <= 16, "a chunk's blocks fit the 16 lanes of a row");
template <int G>
struct Run {
  float m[Cfg<G>::HPL];    // lane (r, c): maximum after record c
  float old[Cfg<G>::HPL];  // factor of the mass before record c
  float add[Cfg<G>::HPL];  // mass that record c adds
};

template <int CTRL>
__device__ __forceinline__ float dpp_old(float old, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, 0xf, 0xf, false));
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;

// m0: the state's maximum (-inf when it is empty), m, L: this lane's record
// (L = 0 past the run's end)
template <int G>
__device__ __forceinline__ void run_factors(Run<G>& f, int k, float m0, float m, float L) {
  const bool v = L > 0.f;
  float x = v ? m : kNegInf;
  x = fmaxf(x, dpp_old<kRowShr1>(kNegInf, x));
  x = fmaxf(x, dpp_old<kRowShr2>(kNegInf, x));
  x = fmaxf(x, dpp_old<kRowShr4>(kNegInf, x));
  x = fmaxf(x, dpp_old<kRowShr8>(kNegInf, x));
  x = fmaxf(x, m0);
  const float before = dpp_old<kRowShr1>(m0, x);
  f.m[k] = x;
  f.old[k] = before == kNegInf ? 0.f : fast_exp2(__fsub_rn(before, x));
  f.add[k] = v ? __fmul_rn(L, fast_exp2(__fsub_rn(m, x))) : 0.f;
}

// the value of lane i < 16 of this lane's row
__device__ __forceinline__ float row_lane(float x, int i, int lane) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * ((lane & 48) | i), __float_as_int(x)));
}

// One step: record i of the run into slot k of the state; `p` is the
// record's output.  d receives the increment.
template <int G>
__device__ __forceinline__ void run_step(State<G>& s, const Run<G>& f, int k, int i, int lane, const float (&p)[8],
                                         float (&d)[8]) {
  const float old = row_lane(f.old[k], i, lane), add = row_lane(f.add[k], i, lane);
  const float Ln = __fadd_rn(__fmul_rn(s.L[k], old), add);
  const float w = add > 0.f ? (s.L[k] > 0.f ? __fmul_rn(add, fast_rcp(Ln)) : 1.f) : 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    d[e] = __fmul_rn(w, __fsub_rn(p[e], s.o[k][e]));
    s.o[k][e] = __fadd_rn(s.o[k][e], d[e]);
  }
  s.L[k] = Ln;
}

// One whole record (in state layout) into the state.
template <int G>
__device__ __forceinline__ void merge(State<G>& s, const State<G>& p) {
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    const bool v1 = s.L[k] > 0.f;
    const bool v2 = p.L[k] > 0.f;
    const float mn = v1 ? (v2 ? fmaxf(s.m[k], p.m[k]) : s.m[k]) : p.m[k];
    const float a = v1 ? __fmul_rn(s.L[k], fast_exp2(__fsub_rn(s.m[k], mn))) : 0.f;
    const float bb = v2 ? __fmul_rn(p.L[k], fast_exp2(__fsub_rn(p.m[k], mn))) : 0.f;
    const float Ln = __fadd_rn(a, bb);
    const float w = v2 ? (v1 ? __fmul_rn(bb, fast_rcp(Ln)) : 1.f) : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      s.o[k][e] = __fadd_rn(s.o[k][e], __fmul_rn(w, __fsub_rn(p.o[k][e], s.o[k][e])));
    s.m[k] = (v1 || v2) ? mn : kNegInf;
    s.L[k] = Ln;
  }
}

// ---- records: workspace (coherent, normalised) and LDS tiles --------------
// LDS block record: o[G][128] | m[G] | L[G], the block's normalised output
// (the loaders normalise it when they write it), its maximum and its mass.
template <int G>
__device__ __forceinline__ void read_output(const float* rec, int k, int lane, float (&o)[8]) {
  const int c = lane & 15;
  int h = (lane >> 4) + 4 * k;
  if (h >= G) h = 0;  // idle slot: read something valid, never used
  const f32x4* src = reinterpret_cast<const f32x4*>(rec + h * kD + c * 8);
  const f32x4 x0 = src[0], x1 = src[1];
  o[0] = x0[0]; o[1] = x0[1]; o[2] = x0[2]; o[3] = x0[3];
  o[4] = x1[0]; o[5] = x1[1]; o[6] = x1[2]; o[7] = x1[3];
}
// Lane (r, c): maximum and mass of block c for head r + 4k (an empty record
// from block nb on).
template <int G>
__device__ __forceinline__ void read_masses(const float* blocks, int nb, int k, int lane, float& m, float& L) {
  const int c = lane & 15;
  int h = (lane >> 4) + 4 * k;
  if (h >= G) h = 0;
  const float* rec = blocks + min(c, nb - 1) * Cfg<G>::REC + G * kD + h;
  m = rec[0];
  L = c < nb ? rec[G] : 0.f;
}

// fn(i) for the blocks 0 .. nb - 1 in order, GANG of them at a time with no
// branch between, so that their loads, weights and row sums overlap; the one
// or two that are left one by one.  (Never a block past nb: its lane
// may lie in another row, and a weight of zero times an infinite output is
// no zero.)
template <int G, class Fn>
__device__ __forceinline__ void gangs_of_blocks(int nb, Fn fn) {
  constexpr int GANG = Cfg<G>::GANG;
  int i = 0;
  for (; i + GANG <= nb; i += GANG)
#pragma unroll
    for (int u = 0; u < GANG; ++u) fn(i + u);
#pragma unroll 1
  for (; i < nb; ++i) fn(i);
}

// The chunk's aggregate: the state of its blocks alone.  The weights of all
// blocks come at once (lane (r, c): block c), then one fused multiply-add
// per block and output.
template <int G>
__device__ __forceinline__ void aggregate(State<G>& s, const float* blocks, int nb, int lane) {
  constexpr int HPL = Cfg<G>::HPL;
  float w[HPL];
#pragma unroll
  for (int k = 0; k < HPL; ++k) {
    float m, L;
    read_masses<G>(blocks, nb, k, lane, m, L);
    const bool v = L > 0.f;
    const float top = row_max(v ? m : kNegInf);
    const float x = v ? __fmul_rn(L, fast_exp2(__fsub_rn(m, top))) : 0.f;
    s.m[k] = top;
    s.L[k] = row_sum(x);
    w[k] = s.L[k] > 0.f ? __fmul_rn(x, fast_rcp(s.L[k])) : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s.o[k][e] = 0.f;
  }
  gangs_of_blocks<G>(nb, [&](int i) {
#pragma unroll
    for (int k = 0; k < HPL; ++k) {
      float p[8];
      read_output<G>(blocks + i * Cfg<G>::REC, k, lane, p);
      const float wi = row_lane(w[k], i, lane);
#pragma unroll
      for (int e = 0; e < 8; ++e) s.o[k][e] = __builtin_fmaf(wi, p[e], s.o[k][e]);
    }
  });
}

// Workspace records go through a buffer resource over the group's record
// area with the sc1 cache policy: agent-coherent 16-byte accesses whose
// completion the compiler tracks like any other load or store.
constexpr int kCoherent = 16;  // buffer cache policy: sc1
constexpr int kLookFirstPasses = 5;  // look-back passes before a chunk publishes its aggregate

__device__ __forceinline__ __amdgpu_buffer_rsrc_t record_rsrc(Params& P, int gidx) {
  const float* base = P.records + (int64_t)gidx * P.max_chunks * 2 * P.record_floats;
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0,
                                           P.max_chunks * 2 * P.record_floats * 4, 0x00020000);
}

// Layout of a workspace record (G*kD + 2G floats).  Head h's outputs fill
// floats h*kD .. h*kD + 127, first the first halves of the sixteen lanes'
// eight coordinates (lane c: dims 8c .. 8c+3 at 4c), then the second halves
// (dims 8c+4 .. 8c+7 at 64 + 4c), so that each store instruction covers
// whole 64-byte segments (256 contiguous bytes per head) and each segment
// leaves the L2 once, not once per half; m and L of head h follow at G*kD + h
// and G*kD + G + h.
template <int G>
__device__ __forceinline__ void publish_state(__amdgpu_buffer_rsrc_t rs, int rec_off, const State<G>& s,
                                              int lane) {
  const int c = lane & 15, r = lane >> 4;
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    const int h = r + 4 * k;
    if (h < G) {
      const int off = (rec_off + h * kD + c * 4) * 4;
      __builtin_amdgcn_raw_buffer_store_b128(f32x4{s.o[k][0], s.o[k][1], s.o[k][2], s.o[k][3]}, rs, off, 0, kCoherent);
      __builtin_amdgcn_raw_buffer_store_b128(f32x4{s.o[k][4], s.o[k][5], s.o[k][6], s.o[k][7]}, rs, off + 256, 0, kCoherent);
      if (c == 0) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s.m[k]), rs, (rec_off + G * kD + h) * 4, 0, kCoherent);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s.L[k]), rs, (rec_off + G * kD + G + h) * 4, 0, kCoherent);
      }
    }
  }
}

__device__ __forceinline__ float ld_record(__amdgpu_buffer_rsrc_t rs, int off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off * 4, 0, kCoherent));
}
template <int G>
__device__ __forceinline__ void fetch_output(__amdgpu_buffer_rsrc_t rs, int rec_off, int k, int lane, float (&o)[8]) {
  const int c = lane & 15;
  int h = (lane >> 4) + 4 * k;
  if (h >= G) h = 0;
  const int off = (rec_off + h * kD + c * 4) * 4;
  const f32x4 x0 = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, kCoherent);
  const f32x4 x1 = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 256, 0, kCoherent);
  o[0] = x0[0]; o[1] = x0[1]; o[2] = x0[2]; o[3] = x0[3];
  o[4] = x1[0]; o[5] = x1[1]; o[6] = x1[2]; o[7] = x1[3];
}
template <int G>
__device__ __forceinline__ void fetch_state(__amdgpu_buffer_rsrc_t rs, int rec_off, State<G>& s, int lane) {
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    int h = (lane >> 4) + 4 * k;
    if (h >= G) h = 0;
    s.m[k] = ld_record(rs, rec_off + G * kD + h);
    s.L[k] = ld_record(rs, rec_off + G * kD + G + h);
    fetch_output<G>(rs, rec_off, k, lane, s.o[k]);
  }
}

// ---- phase 1: one 64-token tile on one wavefront ---------------------------
template <int G>
__device__ __forceinline__ void load_q(Params& P, int b, int kvh, int lane, bf16x8 (&qa)[4]) {
  const int h = lane & (Cfg<G>::COLS - 1);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (h < G) {
      const uint16_t* src = P.q + ((int64_t)b * P.num_q_heads + kvh * G + h) * kD + (4 * s + (lane >> 4)) * 8;
      const u32x4 w = *reinterpret_cast<const u32x4*>(src);
      qa[s] = __builtin_bit_cast(bf16x8, w);
    } else {
      qa[s] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
    }
  }
}

__device__ __forceinline__ int clamp_page(Params& P, int b, int tok) {
  int pg = P.page_table[(int64_t)b * P.max_pages + (tok >> P.page_shift)];
  pg = pg < 0 ? 0 : pg;
  return pg >= P.num_pages ? P.num_pages - 1 : pg;
}

// A 64-token tile on one wavefront.  Both contractions run on
// v_mfma_f32_16x16x32_bf16:
//   - scores transposed, S^T = K Q^T (tokens are the M rows, the query
//     heads of the group the N columns, head dims the reduction), so that
//     each lane ends up holding the probabilities of one head for exactly
//     the eight tokens that the P.V A-operand needs from it;
//   - P.V with P as A (heads x 32 tokens) and V as B (32 tokens x 16 dims).
//     V reaches the B layout (eight tokens of one dim per lane) through LDS,
//     written row-major and read back with ds_read_b64_tr_b16: for groups
//     of up to 4 heads, half tiles through the loader's own staging buffer;
//     for 8 or more, quarter tiles (16 tokens, 4 KiB), through the output
//     part of the very record the tile is about to write when every block
//     is one tile (nothing reads it before the record is written, and the
//     LDS so saved holds longer chunks), else through a 4 KiB staging
//     buffer.  P is split into three bf16 parts (hi + mid + lo carries 24
//     significant bits), so P.V keeps fp32 precision.
// The record written to LDS holds the normalised block output
// sum_j p_hj v_j / l_h [G][128], m_h [G] (base 2) and l_h [G].  pg[n] is the
// (uniform) physical page of 16-token group n.
typedef short v4i16 __attribute__((ext_vector_type(4)));
constexpr int kVPitch = 144;                  // u16 per row of a staging buffer (288 B)
constexpr int kVBufU16 = 32 * kVPitch;        // one half tile: 32 rows
constexpr int kVRow = 128;                    // u16 per row of a quarter-tile stage (256 B)
// Quarter-tile stage: row r's 16-byte piece j sits at piece j ^ 2(r & 3),
// so that the four rows one transposing read touches fall on distinct banks
// (a half-tile buffer pads its rows to 288 bytes for the same end).
__device__ __forceinline__ int vstage_off(int row, int piece) {
  return row * kVRow + ((piece ^ (2 * (row & 3))) << 3);
}

// The first tile of a block writes the block record; each later tile of
// the block (accumulate) is folded into it: both parts rescaled to the
// larger running max and the combined mass, in tile order.
template <int G, bool WIDE>
__device__ void compute_tile(Params& P, int kvh, int L, int tok0, const int (&pg)[4],
                             const bf16x8 (&qa)[4], uint16_t* __restrict__ vbuf,
                             float* __restrict__ rec, bool accumulate) {
  const int lane = threadIdx.x & 63;
  const int lo = lane & 15, g = lane >> 4;
  const int psz_mask = (1 << P.page_shift) - 1;

  if (tok0 >= L) {  // tile past the sequence end: empty partial
    if (accumulate) return;
    for (int i = lane; i < G * kD; i += 64) rec[i] = 0.f;
    if (lane < G) {
      rec[G * kD + lane] = kNegInf;
      rec[G * kD + G + lane] = 0.f;
    }
    return;
  }

  // K: for 16-token group n, lane holds token 16n + lo, dims 32s + 8g .. +7.
  // A 16-aligned group never straddles a page (page_size >= 16, power of
  // two); tokens past L are redirected to token L-1, which lies in the same
  // group or in the last group before it, the group whose page pg[n] then
  // names.  V: lane (lo, g) holds token 4i + g, dims 8lo .. +7; the four
  // tokens of one load instruction are consecutive and lie in group i / 4.
  // All are issued together so that one memory latency covers the tile.
  // Rows less than 16 MiB apart (WIDE false, every usual layout) are addressed
  // from scalar group bases with 24-bit lane products: the general form's
  // 64-bit multiplies per lane (36 of them) kept a tile's first loads waiting.
  u32x4 kr[4][4];
  u32x4 vr[16];
  if constexpr (!WIDE) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int t = min(tok0 + 16 * n, L - 1);
      const char* kb = reinterpret_cast<const char*>(P.k + (int64_t)pg[n] * P.ks_page + (int64_t)kvh * P.ks_head +
                                                     (int64_t)(t & psz_mask) * P.ks_tok);
      const uint32_t ko = __umul24(min(lo, L - 1 - t), (uint32_t)(2 * P.ks_tok)) + 16u * g;
#pragma unroll
      for (int s = 0; s < 4; ++s) kr[n][s] = *reinterpret_cast<const u32x4*>(kb + (ko + 64u * s));
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int t = min(tok0 + 16 * n, L - 1);
      const char* vb = reinterpret_cast<const char*>(P.v + (int64_t)pg[n] * P.vs_page + (int64_t)kvh * P.vs_head +
                                                     (int64_t)(t & psz_mask) * P.vs_tok);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t vo = __umul24(min(4 * j + g, L - 1 - t), (uint32_t)(2 * P.vs_tok)) + 16u * lo;
        vr[4 * n + j] = *reinterpret_cast<const u32x4*>(vb + vo);
      }
    }
  } else {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int tok = min(tok0 + 16 * n + lo, L - 1);
      const uint16_t* kp = P.k + (int64_t)pg[n] * P.ks_page + (int64_t)kvh * P.ks_head +
                           (int64_t)(tok & psz_mask) * P.ks_tok;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        kr[n][s] = *reinterpret_cast<const u32x4*>(kp + (4 * s + g) * 8);
    }
    const uint16_t* vp = P.v + (int64_t)kvh * P.vs_head + lo * 8;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int tok = min(tok0 + 4 * i + g, L - 1);
      vr[i] = *reinterpret_cast<const u32x4*>(vp + (int64_t)pg[i >> 2] * P.vs_page +
                                              (int64_t)(tok & psz_mask) * P.vs_tok);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // S^T[n][r]: token 16n + 4g + r, head lo mod COLS: the 16 columns hold REP
  // copies of the heads, and copy u = lo / COLS keeps the scores of the
  // groups n = REP i + u.  Each lane's softmax work is then NS x 4 tokens in
  // place of 16 with most lanes idle (at g = 4: 4), which with the packed
  // conversions below took a tile's vector ALU instructions from about 650
  // to 200.
  constexpr int REP = Cfg<G>::REP, COLS = Cfg<G>::COLS, NS = 4 / REP;
  const int u = lo / COLS;
  f32x4 St[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    St[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      St[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[n][s]), qa[s], St[n], 0, 0, 0);
  }
  // softmax of the lane's head over the tile: the lane's own tokens, the
  // other copies (lanes lo ^ 8, then lo +- 4 of the row), then the four rows
  // (every lane of a head ends with the same bits: max is exact and each
  // step adds the same two values)
  float sc[NS][4];
  float mx = kNegInf;
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x = St[REP * i][r];
      if constexpr (REP == 2) {
        x = u ? St[2 * i + 1][r] : x;
      } else if constexpr (REP == 4) {
        const float y = (u & 1) ? St[1][r] : x, z = (u & 1) ? St[3][r] : St[2][r];
        x = (u & 2) ? z : y;
      }
      sc[i][r] = x * P.scale_log2;
    }
  if (tok0 + kTile > L) {
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (tok0 + 16 * (REP * i + u) + 4 * g + r >= L) sc[i][r] = kNegInf;
  }
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[i][r]);
  if constexpr (REP >= 2) mx = fmaxf(mx, dpp_f<kRowRor8>(mx));
  if constexpr (REP == 4) mx = fmaxf(mx, dpp_f<kRowRor4>(mx));
  mx = rows_max(mx);
  float ls = 0.f;
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float p = mx == kNegInf ? 0.f : fast_exp2(sc[i][r] - mx);
      sc[i][r] = p;
      ls += p;
    }
  if constexpr (REP >= 2) ls = ls + dpp_f<kRowRor8>(ls);
  if constexpr (REP == 4) ls = ls + dpp_f<kRowRor4>(ls);
  ls = rows_sum(ls);
  if (g == 0 && lo < G && !accumulate) {
    rec[G * kD + lo] = mx;
    rec[G * kD + G + lo] = ls;
  }

  // A operands of the two 32-token K-steps c: element e of lane (lo, g) is
  // p of head lo at token 16(2c + e/4) + 4g + e%4, in three bf16 parts (hi +
  // mid + lo carries 24 significant bits).  Fewer than 16 heads leave rows of
  // A free: up to four heads put the parts in rows h, 4 + h, 8 + h, 12 + h of
  // one operand (the last two hold half of lo each, exactly, so that no row
  // multiplies V by zeros), eight put hi and mid in rows h and 8 + h of one
  // and the halves of lo in those of another.  One product (two) then does
  // the work of three, and the parts' sums are added across the accumulator
  // rows at the end.  The parts reach their rows through the wave's staging
  // memory: row m holds its tokens as [g][n][4], 128 bytes.
  constexpr int NP = G > 8 ? 3 : G > 4 ? 2 : 1;
  uint32_t own[NS][3][2];
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float a0 = sc[i][2 * e], a1 = sc[i][2 * e + 1];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const uint32_t w = pack_bf16(a0, a1);
        own[i][j][e] = w;
        a0 = a0 - bf_lo(w);
        a1 = a1 - bf_hi(w);
        if (G <= 8 && j == 1) {
          a0 = 0.5f * a0;
          a1 = 0.5f * a1;
        }
      }
    }
  bf16x8 a[2][NP];
  if constexpr (G > 8) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        a[c][j] = __builtin_bit_cast(
            bf16x8, u32x4{own[2 * c][j][0], own[2 * c][j][1], own[2 * c + 1][j][0], own[2 * c + 1][j][1]});
  } else {
    const int h = lo & (COLS - 1);
#pragma unroll
    for (int j = 0; j < (G > 4 ? 3 : 4); ++j)
#pragma unroll
      for (int i = 0; i < NS; ++i)
        *reinterpret_cast<u32x2*>(vbuf + (COLS * j + h) * 64 + g * 16 + 4 * (REP * i + u)) =
            u32x2{own[i][j < 3 ? j : 2][0], own[i][j < 3 ? j : 2][1]};
    wave_lds_order();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      a[c][0] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(vbuf + lo * 64 + g * 16 + 8 * c));
      if constexpr (NP == 2)
        a[c][NP - 1] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(vbuf + (16 + h) * 64 + g * 16 + 8 * c));
    }
    wave_lds_order();  // the parts are read before V takes the memory
  }

  // P.V over the two halves of the tile.  B for K-step c and dims
  // 16d .. 16d+15: lane (lo, g) needs V[token of element e][16d + lo]; in
  // each 16-lane group, source lane 4k + q of a transposing read points at
  // row 4g + k of a 16-row quarter (then of the next one), columns
  // 16d + 4q .. +3.
  f32x4 acc[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int rk = lo >> 2, cq = lo & 3;
  if constexpr (G >= 8) {
    // a quarter at a time, the first quarter's B parts (elements 0..3) kept
    // in registers until the second's are read
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      v4i16 r0[8];
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<u32x4*>(vbuf + vstage_off(4 * i + g, lo)) = vr[8 * c + 4 * qh + i];
        wave_lds_order();
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          const v4i16 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) v4i16*)(vbuf + vstage_off(4 * g + rk, 2 * d + (cq >> 1)) +
                                                         4 * (cq & 1)));
          if (qh == 0) {
            r0[d] = r;
          } else {
            const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(r0[d], r, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int j = 0; j < NP; ++j) acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c][j], b, acc[d], 0, 0, 0);
          }
        }
        wave_lds_order();  // the reads of this quarter come before the next one's writes
      }
    }
  } else {
    // a whole half at a time; the row pitch of 288 bytes puts the 16 lanes
    // of a group on 32 distinct banks
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        *reinterpret_cast<u32x4*>(vbuf + (4 * i + g) * kVPitch + 8 * lo) = vr[8 * c + i];
      wave_lds_order();
#pragma unroll
      for (int d = 0; d < 8; ++d) {
        const v4i16 r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) v4i16*)(vbuf + (4 * g + rk) * kVPitch + 16 * d + 4 * cq));
        const v4i16 r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) v4i16*)(vbuf + (16 + 4 * g + rk) * kVPitch + 16 * d + 4 * cq));
        const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
        for (int j = 0; j < NP; ++j) acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c][j], b, acc[d], 0, 0, 0);
      }
      wave_lds_order();  // the reads of this half come before the next half's writes
    }
  }
  // acc[d][r]: row 4g + r of A, dim 16d + lo.  The parts' rows are added by
  // swapping halves (then rows) of two accumulators and adding the pair,
  // which leaves each lane the sums of fewer dims, all lanes at work: ND
  // dims 16 (d + DG dg) + lo of heads HG hg + r.
  constexpr int ND = G > 8 ? 8 : G > 4 ? 4 : 2;
  f32x4 sum[ND];
  if constexpr (G > 8) {
#pragma unroll
    for (int d = 0; d < ND; ++d) sum[d] = acc[d];
  } else {
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_int(acc[d][r]), __float_as_int(acc[d + 4][r]), false, false);
        acc[d][r] = __int_as_float(x[0]) + __int_as_float(x[1]);
      }
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (G > 4) {
          sum[d][r] = acc[d][r];
        } else {
          const auto x = __builtin_amdgcn_permlane16_swap(__float_as_int(acc[d][r]), __float_as_int(acc[d + 2][r]), false, false);
          sum[d][r] = __int_as_float(x[0]) + __int_as_float(x[1]);
        }
      }
  }
  const int h0 = G > 8 ? 4 * g : G > 4 ? 4 * (g & 1) : 0;                      // head of r = 0
  float* const to = rec + h0 * kD + 16 * (G > 8 ? 0 : G > 4 ? 4 * (g >> 1) : 2 * g) + lo;  // its dim of d = 0
  // A block's first tile divides its sums by the mass l_h; a later tile's
  // fold factors come from row 0 of the lanes (g = 0, head lo) through the
  // staging buffer, which the P.V loop no longer reads (a record never
  // stages its own later tiles: records stage only blocks of one tile).
  if (!accumulate) {
    // 1 / l_h of lane h, handed to the lanes that hold head h's sums
    const float inv_l = ls > 0.f ? fast_rcp(ls) : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r < G) {
        float inv = read_lane(inv_l, r);
        if constexpr (G > 4) inv = h0 == 4 ? read_lane(inv_l, 4 + r) : inv;
        if constexpr (G > 8) inv = h0 == 8 ? read_lane(inv_l, 8 + r) : h0 == 12 ? read_lane(inv_l, 12 + r) : inv;
#pragma unroll
        for (int d = 0; d < ND; ++d) to[r * kD + 16 * d] = __fmul_rn(sum[d][r], inv);
      }
    }
    return;
  }
  // fold into the block record: o = (o_rec L_rec so + sum_tile sn) / L_new
  float* scale = reinterpret_cast<float*>(vbuf);
  if (g == 0 && lo < G) {
    const float mo = rec[G * kD + lo], lo_sum = rec[G * kD + G + lo];
    const float mn = fmaxf(mo, mx);
    const float so = mo == kNegInf ? 0.f : fast_exp2(mo - mn);
    const float sn = mx == kNegInf ? 0.f : fast_exp2(mx - mn);
    const float a = __fmul_rn(lo_sum, so);
    const float Ln = __fadd_rn(a, __fmul_rn(ls, sn));
    const float inv = Ln > 0.f ? fast_rcp(Ln) : 0.f;
    rec[G * kD + lo] = mn;
    rec[G * kD + G + lo] = Ln;
    scale[lo] = __fmul_rn(a, inv);
    scale[G + lo] = __fmul_rn(sn, inv);
  }
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r < G) {
      const float so = scale[h0 + r], sn = scale[G + h0 + r];
#pragma unroll
      for (int d = 0; d < ND; ++d) {
        float* x = to + r * kD + 16 * d;
        *x = __fadd_rn(__fmul_rn(*x, so), __fmul_rn(sum[d][r], sn));
      }
    }
  }
  wave_lds_sync();  // the scale factors are read before the buffer is reused
}

// One block of the chunk into the state (the replay's step).
template <int G>
__device__ __forceinline__ void step_block(State<G>& s, const Run<G>& run, const float* blocks, int i, int lane) {
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    float p[8], d[8];
    read_output<G>(blocks + i * Cfg<G>::REC, k, lane, p);
    run_step<G>(s, run, k, i, lane, p, d);
    s.m[k] = row_lane(run.m[k], i, lane);
  }
}

// ---- phase 2 helpers ----------------------------------------------------------
// Chunk geometry: the first lead_chunks chunks of a traversal hold
// lead_blocks blocks each, every later one chunk_blocks.
__device__ __forceinline__ int chunk_start(Params& P, int k) {
  return k < P.lead_chunks ? k * P.lead_blocks
                           : P.lead_chunks * P.lead_blocks + (k - P.lead_chunks) * P.chunk_blocks;
}
__device__ __forceinline__ int chunks_for(Params& P, int T) {
  const int lead_T = P.lead_chunks * P.lead_blocks;
  return T <= lead_T ? (T + P.lead_blocks - 1) / P.lead_blocks
                     : P.lead_chunks + (T - lead_T + P.chunk_blocks - 1) / P.chunk_blocks;
}

struct StabSummary {   // one chunk's own blocks (entering run taken as 0)
  int32_t lead;        // leading stable blocks
  int32_t trail;       // trailing stable blocks
  int32_t len;         // blocks in the chunk
  int32_t fis;         // first block (0-based) where the chunk's own run reaches p, or -1
};
struct StabState {     // after a prefix of chunks
  int32_t stopped;     // 1 if the stop lies in the prefix
  int32_t stop_t;      // 1-based traversal step of the stop
  int32_t run;         // consecutive stable steps ending the prefix (if not stopped)
  int32_t pad;
};

// Payloads: a summary packs lead, trail, len (each <= 16) and fis + 1 in
// five bits each; a stability state packs `stopped` (bit 19) and the run
// (19 bits; traversals are shorter than 2^19 blocks, so it is exact).
__device__ __forceinline__ uint32_t pack_summary(const StabSummary& y) {
  return (uint32_t)y.lead | ((uint32_t)y.trail << 5) | ((uint32_t)y.len << 10) | ((uint32_t)(y.fis + 1) << 15);
}
__device__ __forceinline__ StabSummary unpack_summary(uint32_t p) {
  return StabSummary{(int32_t)(p & 31u), (int32_t)((p >> 5) & 31u), (int32_t)((p >> 10) & 31u),
                     (int32_t)((p >> 15) & 31u) - 1};
}
__device__ __forceinline__ uint32_t pack_stab(const StabState& x) {
  return ((uint32_t)(x.stopped != 0) << 19) | ((uint32_t)x.run & 0x7ffffu);
}
__device__ __forceinline__ StabState unpack_stab(uint32_t p) {
  return StabState{(int32_t)((p >> 19) & 1u), 0, (int32_t)(p & 0x7ffffu), 0};
}

__device__ __forceinline__ StabState stab_fold(StabState x, StabSummary y, int t0, int patience) {
  if (x.stopped) return x;
  StabState r = x;
  if (y.lead > 0 && (int64_t)x.run + y.lead >= patience) {
    r.stopped = 1;
    r.stop_t = t0 + (patience - x.run - 1) + 1;
  } else if (y.fis >= 0) {
    r.stopped = 1;
    r.stop_t = t0 + y.fis + 1;
  } else {
    r.run = (y.lead == y.len) ? x.run + y.len : y.trail;
  }
  return r;
}

// The stop announcement of a group is one word: epoch << 24 | chunk, where
// the chunk holds the stop or lies after it.  Chunks after the announced one
// are moot: loaders skip them and their resolvers give up.
__device__ __forceinline__ bool stop_word_before(uint64_t v, uint64_t epoch, int me) {
  return (v >> kQueueBits) == epoch && (int)(v & ((1ull << kQueueBits) - 1ull)) < me;
}
__device__ __forceinline__ bool stop_announced_before(Params& P, int gidx, int me) {
  return stop_word_before(ld_relaxed(P.stop_word + gidx), P.epoch, me);
}
// Lowers the announcement to chunk k unless this call already announced a
// chunk <= k (a word of an earlier call, whatever its bits, is replaced).
// Several chunks of a group may announce; each compare-and-swap that fails
// saw another announcement land, so the loop ends.  Lane 0 only.
__device__ void announce_stop(Params& P, int gidx, int k) {
  stress_delay(P, gidx, k, 8);
  uint64_t* w = P.stop_word + gidx;
  const uint64_t mine = (P.epoch << kQueueBits) | (uint64_t)k;
  uint64_t cur = ld_relaxed(w);
  for (uint32_t spin = 0; !stop_word_before(cur, P.epoch, k + 1) && spin < P.spin_limit; ++spin)
    if (__hip_atomic_compare_exchange_strong(w, &cur, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT))
      break;
}

// Look-back over the flags of chunks me-1, me-2, ... of group gidx, 64 per
// poll (one per lane): returns the nearest chunk j whose state is >= need_hi
// such that every chunk strictly between j and `me` has state >= need_lo,
// -1 if all chunks 0..me-1 have state >= need_lo and none >= need_hi, or -2
// when a stop in a chunk before `me` has been announced or the spin limit is
// reached (the error word is set then).  Wave-uniform.
__device__ int lookback_scan(Params& P, int gidx, int me, uint32_t need_lo,
                             uint32_t need_hi, int lane) {
  const uint64_t* flags = P.flags + (int64_t)gidx * P.max_chunks;
  int hi = me - 1;
  uint32_t it = 0;
  while (hi >= 0) {
    const int idx = hi - lane;
    const uint32_t st = idx >= 0 ? flag_state(ld_relaxed(flags + idx), P.epoch) : 0u;
    const uint64_t have_hi = __ballot(idx >= 0 && st >= need_hi);
    const uint64_t have_lo = __ballot(idx < 0 || st >= need_lo);
    const int first = have_hi ? __ffsll((unsigned long long)have_hi) - 1 : 64;
    const uint64_t need = first >= 64 ? ~0ull : ((1ull << first) - 1ull);
    if ((have_lo & need) == need) {
      if (first < 64) return hi - first;
      hi -= 64;  // 64 chunks with aggregates but no inclusive state: look further back
      continue;
    }
    if (stop_announced_before(P, gidx, me)) return -2;
    if (wait_expired(P, ++it)) return -2;
    __builtin_amdgcn_s_sleep(2);
  }
  return -1;
}

// One pass of lookback_scan with no wait: the index found, -1 for an empty
// prefix, or -3 when a chunk in the way has not published yet.
__device__ int lookback_once(Params& P, int gidx, int me, uint32_t need_lo,
                             uint32_t need_hi, int lane) {
  const uint64_t* flags = P.flags + (int64_t)gidx * P.max_chunks;
  for (int hi = me - 1; hi >= 0; hi -= 64) {
    const int idx = hi - lane;
    const uint32_t st = idx >= 0 ? flag_state(ld_relaxed(flags + idx), P.epoch) : 0u;
    const uint64_t have_hi = __ballot(idx >= 0 && st >= need_hi);
    const uint64_t have_lo = __ballot(idx < 0 || st >= need_lo);
    const int first = have_hi ? __ffsll((unsigned long long)have_hi) - 1 : 64;
    const uint64_t need = first >= 64 ? ~0ull : ((1ull << first) - 1ull);
    if ((have_lo & need) != need) return -3;
    if (first < 64) return hi - first;
  }
  return -1;
}

// Summaries of consecutive chunks compose (entering run 0 throughout):
// A then B has the blocks of both, leads with A's lead (extended by B's if A
// is stable throughout), trails with B's trail (extended by A's if B is),
// and reaches the patience first inside A, else where A's trailing run and
// B's leading run together reach it, else inside B.  Folding a state with
// A then B equals folding it with the composition (the same integers).
__device__ __forceinline__ StabSummary seg_combine(StabSummary a, StabSummary b, int patience) {
  StabSummary r;
  r.len = a.len + b.len;
  r.lead = a.lead == a.len ? a.len + b.lead : a.lead;
  r.trail = b.trail == b.len ? b.len + a.trail : b.trail;
  if (a.fis >= 0) r.fis = a.fis;
  else if (b.lead > 0 && (int64_t)a.trail + b.lead >= patience) r.fis = a.len + (patience - a.trail) - 1;
  else if (b.fis >= 0) r.fis = a.len + b.fis;
  else r.fis = -1;
  return r;
}

// Stability state on entering chunk `me` of group gidx: the nearest chunk j
// before it that published its stability state, folded with the summaries
// of the chunks between (every chunk between must have published its
// summary).  One backward pass, 64 flags per read (lane u holds chunk
// hi - u): each complete window's summaries are composed across the lanes
// in six shuffle steps and put in front of the composition of the later
// windows.  A flag read once at its summary may later show the chunk's own
// state, which is the fold of every chunk up to it, so the summary already
// used gives the same integers.  Returns false when a stop before `me` has
// been announced or the spin limit is reached.
__device__ bool stab_entering(Params& P, int gidx, int me, StabState& x, int lane) {
  const uint64_t* flags = P.flags + (int64_t)gidx * P.max_chunks;
  StabSummary acc{0, 0, 0, -1};  // composition of the chunks after the window
  int hi = me - 1, j = -1;       // j: the chunk that holds the state, if any
  uint32_t it = 0;
  x = StabState{0, 0, 0, 0};
  while (hi >= 0) {
    const int idx = hi - lane;
    const uint64_t v = idx >= 0 ? ld_relaxed(flags + idx) : 0ull;
    const uint32_t st = idx >= 0 ? flag_state(v, P.epoch) : 0u;
    const uint64_t have_st = __ballot(idx >= 0 && st >= kStabInclusive);
    const uint64_t have_sum = __ballot(idx < 0 || st >= kStabSummary);
    const int first = have_st ? __ffsll((unsigned long long)have_st) - 1 : 64;
    const uint64_t need = first >= 64 ? ~0ull : ((1ull << first) - 1ull);
    if ((have_sum & need) != need) {
      if (stop_announced_before(P, gidx, me)) return false;
      if (wait_expired(P, ++it)) return false;
      __builtin_amdgcn_s_sleep(2);
      continue;
    }
    stress_delay(P, gidx, me, 16);
    // the window's summaries (lanes below `first` that hold a chunk), in
    // chunk order: lane u + d holds the earlier chunk.  Within a window every
    // count is below 2^11, so a summary travels as two words: lead | trail
    // << 16 and len | (fis + 1) << 16.
    const uint32_t pl = flag_payload(v);
    uint32_t w0 = 0u, w1 = 0u;
    if (lane < first && idx >= 0) {
      const StabSummary y = unpack_summary(pl);
      w0 = (uint32_t)y.lead | ((uint32_t)y.trail << 16);
      w1 = (uint32_t)y.len | ((uint32_t)(y.fis + 1) << 16);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t e0 = __shfl_down(w0, d), e1 = __shfl_down(w1, d);
      if ((lane & (2 * d - 1)) == 0 && lane + d < 64) {
        const StabSummary c = seg_combine(
            StabSummary{(int32_t)(e0 & 0xffffu), (int32_t)(e0 >> 16), (int32_t)(e1 & 0xffffu), (int32_t)(e1 >> 16) - 1},
            StabSummary{(int32_t)(w0 & 0xffffu), (int32_t)(w0 >> 16), (int32_t)(w1 & 0xffffu), (int32_t)(w1 >> 16) - 1},
            P.patience);
        w0 = (uint32_t)c.lead | ((uint32_t)c.trail << 16);
        w1 = (uint32_t)c.len | ((uint32_t)(c.fis + 1) << 16);
      }
    }
    w0 = __builtin_amdgcn_readfirstlane(w0);
    w1 = __builtin_amdgcn_readfirstlane(w1);
    const StabSummary wsum{(int32_t)(w0 & 0xffffu), (int32_t)(w0 >> 16), (int32_t)(w1 & 0xffffu),
                           (int32_t)(w1 >> 16) - 1};
    acc = seg_combine(wsum, acc, P.patience);
    if (first < 64) {
      x = unpack_stab(__builtin_amdgcn_readlane(pl, first));
      j = hi - first;
      break;
    }
    hi -= 64;
  }
  // the summaries after chunk j (after none: from chunk 0 on)
  x = stab_fold(x, acc, chunk_start(P, j + 1), P.patience);
  return true;
}

// States whose data sits in the workspace records: the flag goes out once
// the record stores have completed.
__device__ __forceinline__ void publish(Params& P, int gidx, int k, uint32_t state, int lane) {
  stress_delay(P, gidx, k, 1);
  stores_complete();
  if (lane == 0)
    __hip_atomic_store(P.flags + (int64_t)gidx * P.max_chunks + k, make_flag(P.epoch, state, 0),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// States carried in the flag word itself: one store, no wait.
__device__ __forceinline__ void publish_word(Params& P, int gidx, int k, uint32_t state,
                                             uint32_t payload, int lane) {
  stress_delay(P, gidx, k, 2 + (int)state);
  if (lane == 0)
    __hip_atomic_store(P.flags + (int64_t)gidx * P.max_chunks + k, make_flag(P.epoch, state, payload),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int G>
__device__ void write_outputs(Params& P, int b, int kvh, const State<G>& s,
                              int stop, int lane, uint32_t heads = 0xffffffffu,
                              bool write_stop = true) {
  const int c = lane & 15, r = lane >> 4;
#pragma unroll
  for (int k = 0; k < Cfg<G>::HPL; ++k) {
    const int h = r + 4 * k;
    if (h >= G || !((heads >> h) & 1u)) continue;
    const int64_t row = (int64_t)b * P.num_q_heads + kvh * G + h;
    if (P.out_bf16) {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = f32_to_bf16_bits(s.o[k][2 * e]) | (f32_to_bf16_bits(s.o[k][2 * e + 1]) << 16);
      *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(P.out) + row * kD + c * 8) = u32x4{w[0], w[1], w[2], w[3]};
    } else {
      f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(P.out) + row * kD + c * 8);
      dst[0] = f32x4{s.o[k][0], s.o[k][1], s.o[k][2], s.o[k][3]};
      dst[1] = f32x4{s.o[k][4], s.o[k][5], s.o[k][6], s.o[k][7]};
    }
    if (c == 0) {
      // natural log of sum exp(scale q.k): (m + log2 L) * ln 2
      P.lse[row] = (s.m[k] + __log2f(s.L[k])) * 0.69314718055994531f;
    }
  }
  if (write_stop && lane == 0) P.stop_block[(int64_t)b * P.num_kv_heads + kvh] = stop;
}

struct GroupInfo {
  int b, kvh, L, nblk, T, n_chunks;
  const int32_t* list;
};

// Traversal of group gidx (indices are clamped: malformed input never makes
// a kernel read outside the arrays the shape describes).
// From the raw sequence length and list length of the group (the list
// length is ignored for dense traversals).
__device__ __forceinline__ GroupInfo group_info_raw(Params& P, int gidx, int L_raw, int T_raw) {
  GroupInfo g;
  g.b = gidx / P.num_kv_heads;
  g.kvh = gidx - g.b * P.num_kv_heads;
  const int64_t cap = (int64_t)P.max_pages << P.page_shift;
  const int L = L_raw < 0 ? 0 : (int)min((int64_t)L_raw, cap);
  g.L = L;
  g.nblk = (L + P.block_size - 1) / P.block_size;
  g.list = nullptr;
  int T = g.nblk;
  if (P.block_list) {
    const int row = P.list_per_head ? gidx : g.b;
    T = T_raw < 0 ? 0 : min(T_raw, P.max_list);
    g.list = P.block_list + (int64_t)row * P.max_list;
  }
  if (g.nblk == 0) T = 0;
  g.T = min(T, P.t_cap);
  g.n_chunks = chunks_for(P, g.T);
  return g;
}

__device__ __forceinline__ int raw_list_len(Params& P, int gidx) {
  if (!P.block_list) return 0;
  const int b = gidx / P.num_kv_heads;
  return P.block_list_len[P.list_per_head ? gidx : b];
}

template <int G>
__device__ void write_empty_wave(Params& P, int b, int kvh, int lane) {
  for (int i = lane; i < G * kD; i += 64) {
    const int64_t idx = ((int64_t)b * P.num_q_heads + kvh * G) * kD + i;
    if (P.out_bf16) static_cast<uint16_t*>(P.out)[idx] = 0;
    else static_cast<float*>(P.out)[idx] = 0.f;
  }
  if (lane < G) P.lse[(int64_t)b * P.num_q_heads + kvh * G + lane] = kNegInf;
  if (P.per_head) {
    if (lane < G) P.stop_block[(int64_t)b * P.num_q_heads + kvh * G + lane] = 0;
  } else if (lane == 0) {
    P.stop_block[(int64_t)b * P.num_kv_heads + kvh] = 0;
  }
}

constexpr int kLoaders = kWaves - 1;   // wavefronts 1..3 stream tiles
constexpr int kSlots = kChunkSlots;    // chunk buffers in LDS
constexpr int kLenCache = 256;         // sequence lengths kept in LDS
enum SlotState : int { kSlotFree = 0, kSlotLoading = 1, kSlotReady = 2, kSlotEnd = 3 };
// slot metadata words
constexpr int kMetaSeq = 0, kMetaState = 1, kMetaGroup = 2, kMetaChunk = 3, kMetaDone = 4, kMetaAbort = 5;
constexpr int kMetaLen = 6, kMetaListLen = 7;  // raw seq_len and list length of the group

__device__ __forceinline__ int lds_ld(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// the same word for every lane of the wave, in a scalar register
__device__ __forceinline__ int lds_uniform(const int* p) { return __builtin_amdgcn_readfirstlane(lds_ld(p)); }
__device__ __forceinline__ void lds_st(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Work queues.  The chunks of the launch form kQueues chunk-major lists:
// queue x holds n_x groups, and its index i stands for chunk i / n_x of
// group x + kQueues * (i % n_x), rotated within its run of kQueues groups
// (see the claim).  Each
// list is handed out from its own workspace word (call epoch << 24 | next
// index) by one fetch-and-add (claim_issue; claim_finish decodes it), so
// that claims spread over kQueues atomic units.  A workgroup's first claim
// from a queue sends an atomic maximum with this call's epoch and index 0
// ahead of its fetch-and-add (the two reach the word in order), so that a
// word left by an earlier call starts over with no round trip of its own:
// replacing it by compare-and-swap took three dependent round trips with
// every workgroup of the queue on one word (2.5 to 4.4 us of each launch's
// start).  Only a word whose epoch is higher (the workspace last served
// another copy of the library, whose call counter is its own) is replaced
// that way; claims that raced with the replacement retry.
// Every chunk a chunk can wait on belongs to the same group, hence to the
// same list, and each list is handed out in increasing order: a chunk only
// ever waits on chunks that some workgroup already holds.  Lane 0 only /
// wave-uniform result.
__device__ __forceinline__ uint64_t* queue_word(Params& P, int x) {
  return P.queue + (int64_t)x * kQueueStride;
}

__device__ __forceinline__ uint64_t claim_issue(Params& P, int x, bool first, int lane) {
  if (first && lane == 0)
    __hip_atomic_fetch_max(queue_word(P, x), P.epoch << kQueueBits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return lane == 0 ? __hip_atomic_fetch_add(queue_word(P, x), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : 0ull;
}

__device__ int claim_finish(Params& P, int x, uint64_t v, int lane) {
  int q = 0;
  if (lane == 0) {
    uint64_t* w = queue_word(P, x);
    const uint64_t mask = (1ull << kQueueBits) - 1ull;
    if ((v >> kQueueBits) == P.epoch) {
      q = (int)(v & mask);
    } else {
      uint64_t cur = v + 1ull;
      for (uint32_t spin = 0;; ++spin) {
        if ((cur >> kQueueBits) == P.epoch) {
          v = __hip_atomic_fetch_add(w, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((v >> kQueueBits) == P.epoch) {
            q = (int)(v & mask);
            break;
          }
          cur = v + 1ull;
        } else if (__hip_atomic_compare_exchange_strong(w, &cur, (P.epoch << kQueueBits) | 1ull,
                                                        __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT)) {
          q = 0;
          break;
        }
        if (wait_expired(P, spin)) {
          q = 0x7fffffff;
          break;
        }
      }
    }
  }
  return __builtin_amdgcn_readfirstlane(q);
}

// The queues used up so far: epoch << 24 | a bit per queue, in one word that
// no claim touches.  The first claim past a queue's end sets its bit (one
// writer per queue: with every such claim setting it, the word's atomics
// alone took 20 us of a launch), and every claim reads the word along with
// its own atomic, so that a workgroup whose queue is used up passes over the
// others that are, instead of asking each in turn, an atomic and a round
// trip each (the last 5 to 8 us of small launches).  A word of a higher epoch
// (another copy of the library) is never taken for this call's.
__device__ __forceinline__ uint64_t* used_up_word(Params& P) { return P.error_word + kUsedUpWord; }
__device__ __forceinline__ void mark_used_up(Params& P, int x, int lane) {
  if (lane == 0) {
    __hip_atomic_fetch_max(used_up_word(P), P.epoch << kQueueBits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_or(used_up_word(P), 1ull << x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
__device__ __forceinline__ uint32_t used_up_queues(Params& P, uint64_t word) {
  return (word >> kQueueBits) == P.epoch ? __builtin_amdgcn_readfirstlane((uint32_t)word & ((1u << kQueues) - 1u)) : 0u;
}

// Group u of queue x: x + kQueues u, where within every full run of kQueues
// groups the queues rotate by the run's index, so that each list mixes KV
// heads instead of holding one head's groups of every sequence (whose stops
// can fall close together and leave one list's workgroups with the late
// work).  A bijection: every group belongs to one list.
__device__ __forceinline__ int queue_group(int x, int u, int n_groups) {
  const int g = x + kQueues * u;
  return u < n_groups / kQueues ? kQueues * u + (x + u) % kQueues : g;
}

// How many chunks of group u of queue x (lane u, the first 64 groups) are
// still of use: up to the announced stop, or all of its own (at least the
// one that writes an empty traversal's outputs).  Later reads only lower it.
__device__ __forceinline__ int live_chunks(Params& P, const int* s_len, int x, int nx, int n_groups, int lane) {
  int live = 0;
  if (lane < nx) {
    const int g = queue_group(x, lane, n_groups), b = g / P.num_kv_heads;
    const uint64_t sw = P.no_detector ? 0ull : ld_relaxed(P.stop_word + g);
    live = max(group_info_raw(P, g, b < kLenCache ? s_len[b] : P.seq_lens[b], raw_list_len(P, g)).n_chunks, 1);
    if ((sw >> kQueueBits) == P.epoch) live = min(live, (int)(sw & ((1ull << kQueueBits) - 1ull)) + 1);
  }
  return live;
}

// ---- per-query-head termination ---------------------------------------------
// The per-head reading of the test: every query head of a group keeps its
// own patience counter (Eq. 3) and stops on its own; its out and lse are
// those at its own stop (stop_block [batch][num_q_heads] holds each head's
// stop, T for a head that never stops), and the group stops reading blocks
// once its last head has stopped.  The chunk's summaries
// and states of the stability monoid are kept per head in the workspace's
// head area, [chunk][head][8] int32 (lead, trail, len, fis | stopped, run),
// written by lane h for head h and published by the chunk's flag as in the
// group reading.  A summary stays valid after the chunk's state is
// published, so the fold below never meets a changed word.
__device__ __forceinline__ int32_t* head_area(Params& P, int gidx, int k, int G) {
  return P.head_area + ((int64_t)gidx * P.max_chunks + k) * (int64_t)(G * 8);
}

// The nearest chunk before `me` that published its stability state, such
// that every chunk between published its summary: j >= -1, or -2 when a
// stop before `me` has been announced or a wait gave up.
__device__ int stab_scan(Params& P, int gidx, int me, int lane) {
  const uint64_t* flags = P.flags + (int64_t)gidx * P.max_chunks;
  int hi = me - 1;
  uint32_t it = 0;
  while (hi >= 0) {
    const int idx = hi - lane;
    const uint32_t st = idx >= 0 ? flag_state(ld_relaxed(flags + idx), P.epoch) : 0u;
    const uint64_t have_st = __ballot(idx >= 0 && st >= kStabInclusive);
    const uint64_t have_sum = __ballot(idx < 0 || st >= kStabSummary);
    const int first = have_st ? __ffsll((unsigned long long)have_st) - 1 : 64;
    const uint64_t need = first >= 64 ? ~0ull : ((1ull << first) - 1ull);
    if ((have_sum & need) == need) {
      if (first < 64) return hi - first;
      hi -= 64;
      continue;
    }
    if (stop_announced_before(P, gidx, me)) return -2;
    if (wait_expired(P, ++it)) return -2;
    __builtin_amdgcn_s_sleep(2);
  }
  return -1;
}

template <int G>
__device__ void resolve_heads(Params& P, int gidx, int k, const GroupInfo& gi,
                              const float* blocks, const State<G>& pre, const Run<G>& run,
                              uint32_t head_bits, int t0, int nb, int lane) {
  const int n_chunks = gi.n_chunks, T = gi.T;
  const bool mine = lane < G;   // lane h holds head h
  int32_t* my = head_area(P, gidx, k, G) + lane * 8;
  StabSummary sm{0, 0, 0, -1};
  if (mine) {
    int run = 0, lead = 0, fis = -1;
    bool leading = true;
    for (int i = 0; i < nb; ++i) {
      const bool st = (head_bits >> i) & 1u;
      run = st ? run + 1 : 0;
      if (leading) {
        if (st) ++lead;
        else leading = false;
      }
      if (fis < 0 && run >= P.patience) fis = i;
    }
    sm = StabSummary{lead, run, nb, fis};
    st_coh_i32(my + 0, lead);
    st_coh_i32(my + 1, run);
    st_coh_i32(my + 2, nb);
    st_coh_i32(my + 3, fis);
  }
  stores_complete();
  publish_word(P, gidx, k, kStabSummary, 0u, lane);
  // every head reaches its patience inside this chunk: the group's stop lies
  // here or before, whatever the chunks before hold
  const bool all_fis = __all(!mine || sm.fis >= 0);
  if (all_fis && lane == 0) announce_stop(P, gidx, k);
  // no head can stop in a chunk whose first block is unstable for it and
  // whose own runs stay short (the last chunk still writes what is left)
  if (__all(!mine || (sm.lead == 0 && sm.fis < 0)) && k != n_chunks - 1) return;

  // entering state per head: the nearest published state, then the
  // summaries after it
  stress_delay(P, gidx, k, 11);
  const int j = stab_scan(P, gidx, k, lane);
  if (j == -2) return;
  stress_delay(P, gidx, k, 12);
  StabState x{0, 0, 0, 0};
  if (mine && j >= 0) {
    const int32_t* w = head_area(P, gidx, j, G) + lane * 8;
    x.stopped = ld_coh_i32(w + 4);
    x.run = ld_coh_i32(w + 5);
  }
  if (k - (j + 1) <= 4 * G) {
    // a short way back (up to one round trip per head either way): every
    // head folds its own summaries, lane h head h, four chunks' words in
    // flight
    for (int i0 = j + 1; i0 < k; i0 += 4) {
      const int n = min(4, k - i0);
      int32_t v[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (mine && u < n) {
          const int32_t* w = head_area(P, gidx, i0 + u, G) + lane * 8;
#pragma unroll
          for (int f = 0; f < 4; ++f) v[u][f] = ld_coh_i32(w + f);
        }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (mine && u < n)
          x = stab_fold(x, StabSummary{v[u][0], v[u][1], v[u][2], v[u][3]}, chunk_start(P, i0 + u), P.patience);
    }
  } else {
    // a long way back (the last chunk of a traversal with no stop before):
    // 64 chunks per read (lane u: chunk i0 + u), composed across the lanes
    // for each head in turn
    for (int i0 = j + 1; i0 < k; i0 += 64) {
      const bool in = lane < k - i0;
      const int32_t* wc = head_area(P, gidx, in ? i0 + lane : i0, G);
      const int t_win = chunk_start(P, i0);
      for (int h = 0; h < G; ++h) {
        StabSummary c{0, 0, 0, -1};
        if (in) c = StabSummary{ld_coh_i32(wc + h * 8), ld_coh_i32(wc + h * 8 + 1), ld_coh_i32(wc + h * 8 + 2),
                                ld_coh_i32(wc + h * 8 + 3)};
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const StabSummary e{__shfl_down(c.lead, d), __shfl_down(c.trail, d), __shfl_down(c.len, d),
                              __shfl_down(c.fis, d)};
          if ((lane & (2 * d - 1)) == 0 && lane + d < 64) c = seg_combine(c, e, P.patience);
        }
        const StabSummary comp{__builtin_amdgcn_readfirstlane(c.lead), __builtin_amdgcn_readfirstlane(c.trail),
                               __builtin_amdgcn_readfirstlane(c.len), __builtin_amdgcn_readfirstlane(c.fis)};
        if (lane == h) x = stab_fold(x, comp, t_win, P.patience);
      }
    }
  }
  const StabState y = mine ? stab_fold(x, sm, t0, P.patience) : x;
  if (mine) {
    st_coh_i32(my + 4, y.stopped);
    st_coh_i32(my + 5, y.run);
  }
  stores_complete();
  const bool all_before = __all(!mine || x.stopped);
  const bool all_after = __all(!mine || y.stopped);
  if (!all_before && all_after && !all_fis && lane == 0) announce_stop(P, gidx, k);
  publish_word(P, gidx, k, kStabInclusive, 0u, lane);
  if (all_before) return;   // every head stopped before this chunk

  // heads whose stop lies in this chunk: o(t_h) again from the prefix, by
  // the same merges as the replay
  const int rel = (mine && !x.stopped && y.stopped) ? y.stop_t - t0 - 1 : -1;
  int rel_h[G];
  int last_rel = -1;
  uint32_t never = 0;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    rel_h[h] = __builtin_amdgcn_readlane(rel, h);
    last_rel = max(last_rel, rel_h[h]);
    if (!__builtin_amdgcn_readlane((int)y.stopped, h)) never |= 1u << h;
  }
  int32_t* head_stop = P.stop_block + (int64_t)gi.b * P.num_q_heads + gi.kvh * G;
  if (rel >= 0) head_stop[lane] = y.stop_t;
  // one pass of the replay's merges from the prefix: each head stopping
  // here is written at its block; in the group's last chunk, heads that
  // never stopped get the state after the last block (the whole traversal)
  const bool finish = !all_after && k == n_chunks - 1;
  const int upto = finish ? nb - 1 : last_rel;
  if (upto >= 0) {
    State<G> o = pre;
    for (int i = 0; i <= upto; ++i) {
      step_block<G>(o, run, blocks, i, lane);
      uint32_t here = 0;
#pragma unroll
      for (int h = 0; h < G; ++h)
        if (rel_h[h] == i) here |= 1u << h;
      if (here) write_outputs<G>(P, gi.b, gi.kvh, o, 0, lane, here, false);
    }
    if (finish) {
      write_outputs<G>(P, gi.b, gi.kvh, o, T, lane, never, false);
      if (mine && ((never >> lane) & 1u)) head_stop[lane] = T;
    }
  }
}

// Phase 2 for one chunk (resolver wavefront).  `blocks` holds the chunk's
// block records.
template <int G, bool PH>
__device__ void resolve_chunk(Params& P, int gidx, int k, const GroupInfo& gi,
                              const float* blocks, int lane) {
  constexpr int REC = Cfg<G>::REC;
  const int b = gi.b, kvh = gi.kvh, T = gi.T, n_chunks = gi.n_chunks;
  const int t0 = chunk_start(P, k);
  const int nb = min(chunk_start(P, k + 1), T) - t0;
  const bool last = k == n_chunks - 1;
  const __amdgpu_buffer_rsrc_t rs = record_rsrc(P, gidx);
  const int rec_agg = k * 2 * P.record_floats;          // float offsets in the group's area
  const int rec_inc = rec_agg + P.record_floats;

  // the predecessor's flag, read now so that the round trip overlaps the
  // aggregate
  const uint64_t prev_flag = k > 0 ? ld_relaxed(P.flags + (int64_t)gidx * P.max_chunks + (k - 1)) : 0ull;
  State<G> agg;
  aggregate<G>(agg, blocks, nb, lane);

  // Softmax prefix.  Chunk 0 has an empty prefix; when chunk k-1 already
  // holds its inclusive state the prefix is that record; otherwise publish
  // the aggregate first (so that later chunks can fold past this one), look
  // back to the nearest inclusive state and fold the aggregates after it
  // forward, FW records in flight at a time.  Every path computes the same
  // left fold Agg(0) (+) ... (+) Agg(k-1), so the bits never depend on
  // timing.  No chunk follows the last one, so it publishes neither its
  // aggregate nor its inclusive state.
  constexpr int HPL = Cfg<G>::HPL;
  constexpr int FW = 12 / HPL;   // (12 in place of 8: one sequence of 32K tokens 50.4 -> 48.5 us; 16 no better)
  int j;
  if (k == 0) {
    j = -1;
  } else if (flag_state(prev_flag, P.epoch) >= kInclusive) {
    j = k - 1;
  } else {
    // With few chunks of a group in flight (look_first), one pass over the
    // flags often finds the prefix complete, and the aggregate record, one
    // of the two written per chunk, is not needed by anyone; with many, the
    // later chunks need it at once to fold past this one.
    // (compiled for 8 or more heads only: the launches that pass the gate
    // are those of many groups of 8, and the extra code alone measurably
    // slowed the instances for smaller groups)
    j = -3;
    if (G >= 8 && P.look_first) {
      // a few passes, a short sleep apart: a prefix that completes within
      // them spares this chunk its aggregate record (measured: one pass and
      // four more 0.3-0.6 % faster than one, sixteen no better, 32 slower)
      j = lookback_once(P, gidx, k, kAggregate, kInclusive, lane);
      for (int pass = 1; j == -3 && pass < kLookFirstPasses; ++pass) {
        __builtin_amdgcn_s_sleep(8);
        j = lookback_once(P, gidx, k, kAggregate, kInclusive, lane);
      }
    }
    if (j == -3) {
      if (!last) {
        publish_state<G>(rs, rec_agg, agg, lane);
        publish(P, gidx, k, kAggregate, lane);
      }
      j = lookback_scan(P, gidx, k, kAggregate, kInclusive, lane);
    }
    if (j == -2) return;
  }
  stress_delay(P, gidx, k, 9);
  compiler_fence();
  State<G> pre;
  if (j >= 0) {
    fetch_state<G>(rs, j * 2 * P.record_floats + P.record_floats, pre, lane);
  } else {
    state_clear<G>(pre);
  }
  for (int i0 = j + 1; i0 < k; i0 += FW) {
    const int n = min(FW, k - i0);
    float p[FW][HPL][8];
    float m[HPL], L[HPL];
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) {
      int h = (lane >> 4) + 4 * kk;
      if (h >= G) h = 0;
      const int c = lane & 15, at = (i0 + min(c, n - 1)) * 2 * P.record_floats + G * kD + h;
      m[kk] = ld_record(rs, at);
      L[kk] = ld_record(rs, at + G);
      if (c >= n) L[kk] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < FW; ++u)
#pragma unroll
      for (int kk = 0; kk < HPL; ++kk)
        if (u < n) fetch_output<G>(rs, (i0 + u) * 2 * P.record_floats, kk, lane, p[u][kk]);
    Run<G> run;
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) run_factors<G>(run, kk, pre.L[kk] > 0.f ? pre.m[kk] : kNegInf, m[kk], L[kk]);
#pragma unroll
    for (int u = 0; u < FW; ++u)
      if (u < n) {
        float d[8];
#pragma unroll
        for (int kk = 0; kk < HPL; ++kk) run_step<G>(pre, run, kk, u, lane, p[u][kk], d);
      }
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) pre.m[kk] = row_lane(run.m[kk], 15, lane);
  }
  // this chunk's inclusive state, published before the replay: the next
  // chunks wait for it (measured: raising its flag only after the replay's
  // first blocks, to overlap the stores' completion, was 0.5 % slower)
  if (!last || P.no_detector) {
    State<G> inc = pre;
    merge<G>(inc, agg);
    if (!last) {
      publish_state<G>(rs, rec_inc, inc, lane);
      publish(P, gidx, k, kInclusive, lane);
    } else {
      // no stability test (the detector-free baseline): the last chunk
      // holds the output
      write_outputs<G>(P, b, kvh, inc, T, lane);
    }
    if (P.no_detector) return;
  }

  // Replay the chunk's blocks from the prefix with the stability test.  The
  // steps run in order (each needs the state after the previous block); the
  // row sums of |d|^2 and o(t-1).d of block i stay in lane c = i of the
  // head's row with |o(t-1)|^2 (lanes past the chunk's last block are
  // masked out below), and |o(t)|^2 follows as
  // |o(t-1)|^2 + 2 o(t-1).d + |d|^2.  The verdicts of all blocks and heads
  // are then taken at once, lane (r, c) for block c of head r + 4k.  (One
  // verdict after the other and merges with their exponentials inside took
  // 2.0 us for 3 blocks and 5.0 for 9 at g = 4, 7.7 for 9 at g = 8.)
  // The probe weights (Sec. 3.2, x = P o: 1 on the coordinates the test
  // looks at, every probe_stride-th of the head dimension, 0 elsewhere)
  // multiply the partial sums only when the probe is a subsample; this lane
  // holds coordinates 8*(lane&15) .. +7.
  uint32_t stable_bits = 0;
  uint32_t head_bits = 0;   // per-head mode: lane h < G, head h's stable blocks
  State<G> s = pre;   // after the replay: the state after the chunk's last block
  Run<G> run;
  {
    const int c = lane & 15;
    const bool full_probe = P.probe_stride == 1;
    const bool on_acc = P.scale_of_accumulator != 0;
    float pw[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pw[e] = ((8 * c + e) & (P.probe_stride - 1)) == 0 ? 1.f : 0.f;
    float n_prev[HPL];                              // |x|^2 of the state before the next block
    float acc_dx[HPL];
    float q0[HPL], q1[HPL], qdd[HPL], qod[HPL];     // lane (r, c): block c's |x(t-1)|^2, |x(t)|^2, |d|^2, x.d
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) {
      float m, L;
      read_masses<G>(blocks, nb, kk, lane, m, L);
      run_factors<G>(run, kk, pre.L[kk] > 0.f ? pre.m[kk] : kNegInf, m, L);
      float n0 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) n0 = __builtin_fmaf(full_probe ? s.o[kk][e] : s.o[kk][e] * pw[e], s.o[kk][e], n0);
      n_prev[kk] = row_sum(n0);
      q0[kk] = q1[kk] = qdd[kk] = qod[kk] = acc_dx[kk] = 0.f;
    }
    // step i of slot kk; the sums it leaves in lane c = i
    auto step = [&](int i, int kk, bool plain) {
      float p[8], d[8], o0[8];
      read_output<G>(blocks + i * REC, kk, lane, p);
      const float L0 = s.L[kk];
#pragma unroll
      for (int e = 0; e < 8; ++e) o0[e] = s.o[kk][e];
      run_step<G>(s, run, kk, i, lane, p, d);
      float dd = 0.f, od = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        dd = __builtin_fmaf(plain ? d[e] : d[e] * pw[e], d[e], dd);
        od = __builtin_fmaf(plain ? o0[e] : o0[e] * pw[e], d[e], od);
      }
      dd = row_sum(dd);
      od = row_sum(od);
      const float n0 = n_prev[kk], n1 = __fadd_rn(__fadd_rn(n0, __fmul_rn(2.f, od)), dd);   // |x(t)|^2
      n_prev[kk] = n1;
      if (c == i) {
        q0[kk] = n0;
        q1[kk] = n1;
        qdd[kk] = dd;
        qod[kk] = od;
      }
      if (plain) return;
      // change of the unnormalised accumulator L o, each side in its own max
      // reference (L is the mass relative to the running max): on request it
      // takes the place of |d|^2 in the magnitude test below
      float dx2 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dx = __fsub_rn(__fmul_rn(s.L[kk], s.o[kk][e]), __fmul_rn(L0, o0[e]));
        dx2 = __builtin_fmaf(dx * pw[e], dx, dx2);
      }
      dx2 = row_sum(dx2);
      if (c == i) acc_dx[kk] = dx2;
    };
    if (full_probe && !on_acc) {
      gangs_of_blocks<G>(nb, [&](int i) {
#pragma unroll
        for (int kk = 0; kk < HPL; ++kk) step(i, kk, true);
      });
    } else {
#pragma unroll 1
      for (int i = 0; i < nb; ++i)
#pragma unroll
        for (int kk = 0; kk < HPL; ++kk) step(i, kk, false);
    }
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) s.m[kk] = row_lane(run.m[kk], 15, lane);
    uint32_t all = 0xffffu;
#pragma unroll
    for (int kk = 0; kk < HPL; ++kk) {
      const float n0 = q0[kk], n1 = q1[kk], dd = qdd[kk], od = qod[kk];
      // Eq. (2) on the probe: d_scale = |P d| (or the change of P L o);
      // d_direction = 1 - cos(P o_new, P o_old)
      const float d_scale = fast_sqrt(on_acc ? acc_dx[kk] : dd);
      const float nn = __fmul_rn(fast_sqrt(n1), fast_sqrt(n0));
      const float dot = __fadd_rn(n0, od);
      float d_dir;
      if (dot > 0.f) {
        const float num = fmaxf(__fsub_rn(__fmul_rn(n0, dd), __fmul_rn(od, od)), 0.f);
        d_dir = __fmul_rn(num, fast_rcp(__fmul_rn(nn, __fadd_rn(nn, dot))));
      } else {
        d_dir = __fsub_rn(1.f, __fmul_rn(dot, fast_rcp(nn)));
      }
      const bool st = (n0 > 0.f) && (n1 > 0.f) && (d_scale < P.tau) && (d_dir < P.phi);
      // bits 16 r + c: block c of head r + 4k
      const uint64_t bal = __ballot(st);
      if (PH && lane < G && (lane >> 2) == kk) head_bits = (uint32_t)(bal >> (16 * (lane & 3))) & 0xffffu;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r + 4 * kk < G) all &= (uint32_t)(bal >> (16 * r));
    }
    stable_bits = all & ((1u << nb) - 1u);
    head_bits &= (1u << nb) - 1u;
  }

  if constexpr (PH) {
    resolve_heads<G>(P, gidx, k, gi, blocks, pre, run, head_bits, t0, nb, lane);
    return;
  }
  // stability summary of this chunk (entering run 0)
  StabSummary sm;
  {
    int run = 0, lead = 0, fis = -1;
    bool leading = true;
    for (int i = 0; i < nb; ++i) {
      const bool st = (stable_bits >> i) & 1u;
      run = st ? run + 1 : 0;
      if (leading) {
        if (st) ++lead;
        else leading = false;
      }
      if (fis < 0 && run >= P.patience) fis = i;
    }
    sm.lead = lead;
    sm.trail = run;
    sm.len = nb;
    sm.fis = fis;
  }
  publish_word(P, gidx, k, kStabSummary, pack_summary(sm), lane);
  // A run of p stable blocks inside this chunk puts the stop here or earlier,
  // whatever the chunks before hold: the later chunks are moot from now on.
  if (sm.fis >= 0 && lane == 0) announce_stop(P, gidx, k);
  // A chunk whose first block is unstable and whose own run never reaches
  // the patience cannot hold the stop, whatever run it enters with: unless
  // it is the last chunk (which writes the untruncated result) it is done.
  if (sm.lead == 0 && sm.fis < 0 && !last) return;

  // entering stability state, then this chunk's own
  StabState x;
  stress_delay(P, gidx, k, 10);
  if (!stab_entering(P, gidx, k, x, lane)) return;
  const bool stopped_before = x.stopped != 0;
  const StabState y = stab_fold(x, sm, t0, P.patience);
  if (!stopped_before && y.stopped && sm.fis < 0 && lane == 0)  // the stop lies in this chunk
    announce_stop(P, gidx, k);
  publish_word(P, gidx, k, kStabInclusive, pack_stab(y), lane);
  if (!stopped_before && y.stopped) {
    // the stop lies in this chunk: o(t*) again from the prefix, by the same
    // merges as the replay (the same bits)
    State<G> o = pre;
    for (int i = 0; i < y.stop_t - t0; ++i) step_block<G>(o, run, blocks, i, lane);
    write_outputs<G>(P, b, kvh, o, y.stop_t, lane);
  } else if (!y.stopped && last) {
    write_outputs<G>(P, b, kvh, s, T, lane);
  }
}

// ---- the kernel -----------------------------------------------------------------
// Persistent workgroups of four wavefronts.  Wavefronts 1..3 claim chunks
// from the work list and stream their tiles into the LDS chunk buffers in
// turn; wavefront 0 resolves earlier chunks meanwhile.  A chunk is claimed
// only once a buffer is free, and every wait targets a chunk claimed
// earlier, so the launch always makes progress.
template <int G, bool PH, bool WIDE>
__global__ void __launch_bounds__(kThreads, 2) art_decode_kernel(const KernelParams) {
  Params* const args = (Params*)__builtin_amdgcn_kernarg_segment_ptr();
  // the dynamic buffers must start 16-byte aligned (128-bit LDS accesses):
  // the static block below is a multiple of 16 bytes
  extern __shared__ __align__(16) float smem[];
  __shared__ __align__(16) int s_meta[kSlots][8];
  // lengths of the first kLenCache sequences: a dense traversal's claims
  // need no round trip
  __shared__ __align__(16) int s_len[kLenCache];
  static_assert(sizeof(int) * (kSlots * 8 + kLenCache) % 16 == 0,
                "static LDS must keep the dynamic part aligned");
  constexpr int REC = Cfg<G>::REC;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int slot_floats = args->chunk_blocks * REC;

  if (tid < kSlots * 8) (&s_meta[0][0])[tid] = (tid % 8 == kMetaSeq) ? -1 : 0;
  for (int i = tid; i < min(args->batch, kLenCache); i += kThreads) s_len[i] = args->seq_lens[i];
  __syncthreads();

  if (wave == 0) {
    // ---------------- resolver ----------------
    __builtin_amdgcn_s_setprio(3);
    for (int it = 0;; ++it) {
      Params& P = *fresh(args);
      const int slot = it % kSlots;
      int st = kSlotFree;
      for (uint32_t spin = 0;; ++spin) {
        st = lds_ld(&s_meta[slot][kMetaState]);
        if (lds_ld(&s_meta[slot][kMetaSeq]) == it && (st == kSlotReady || st == kSlotEnd)) break;
        if (wait_expired(P, spin)) return;
        __builtin_amdgcn_s_sleep(1);
      }
      if (st == kSlotEnd) return;
      const int gidx = lds_uniform(&s_meta[slot][kMetaGroup]);
      const int k = lds_uniform(&s_meta[slot][kMetaChunk]);
      if (!lds_ld(&s_meta[slot][kMetaAbort])) {
        float* base = smem + slot * slot_floats;
        const GroupInfo gi = group_info_raw(P, gidx, lds_uniform(&s_meta[slot][kMetaLen]),
                                            lds_uniform(&s_meta[slot][kMetaListLen]));
        resolve_chunk<G, PH>(*fresh(args), gidx, k, gi, base, lane);
      }
      wave_lds_sync();
      if (lane == 0) lds_st(&s_meta[slot][kMetaState], kSlotFree);
    }
  }

  // ---------------- loaders ----------------
  const int lw = wave - 1;
  // (a loader's own staging buffer after the chunk buffers, 16-byte aligned:
  // a half tile, or a quarter tile for 8 or more heads; unused when V is
  // staged in the records)
  uint16_t* vbuf = reinterpret_cast<uint16_t*>(smem + ((kSlots * slot_floats + 3) & ~3)) +
                   lw * (G >= 8 ? 16 * kVRow : kVBufU16);
  // leader: the queue it claims from (its own first, as many workgroups to
  // each as it has groups, then the others in turn once its own is used up),
  // the queues that may still hold work (those past
  // the number of groups never do: with two groups, six of eight workgroups
  // spent their first claims on them) and those it has claimed from.  (The
  // first claim issued before the lengths are read, to overlap the two round
  // trips, was no faster on the listed shapes and 2 % slower on others.)
  const int n_queues = min(kQueues, args->batch * args->num_kv_heads);
  int qx = (int)(blockIdx.x % (unsigned)(args->batch * args->num_kv_heads)) % kQueues;
  uint32_t open = (1u << n_queues) - 1u, entered = 0;
  // What is known of the queue's groups (live_chunks; lane u: group u), read
  // by the claim after one that turned out to be of no use.  With it, claims of
  // further such chunks cost one atomic and no read, and the rest of a queue
  // of stopped groups is dropped at once: walking through it, an atomic and
  // two dependent reads per chunk, took the last 10 to 15 us of a launch
  // over lists.
  int live = 0x7fffffff, moot = 0;
  bool stale = false;

  for (int it = 0;; ++it) {
    Params& P = *fresh(args);
    const int n_groups = P.batch * P.num_kv_heads;
    const int slot = it % kSlots;
    if (lw == 0) {
      // leader: wait for the buffer, then claim the next chunk of the list
      bool gave_up = false;
      for (uint32_t spin = 0; lds_ld(&s_meta[slot][kMetaState]) != kSlotFree; ++spin) {
        if (wait_expired(P, spin)) {
          gave_up = true;  // hand out the end marker below
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      int gsel = -1, ksel = -1, len_sel = 0, list_sel = 0;
      while (!gave_up && open) {
        const int nx = (n_groups - qx + kQueues - 1) / kQueues;  // groups in queue qx
        const uint64_t claim = claim_issue(P, qx, !((entered >> qx) & 1u), lane);
        entered |= 1u << qx;
        const uint64_t done = ld_relaxed(used_up_word(P));
        const int i = claim_finish(P, qx, claim, lane);
        const int kh = i / nx, u = i - kh * nx;
        bool used_up = i >= nx * P.work_chunks;
        if (!used_up && stale) {
          live = live_chunks(P, s_len, qx, nx, n_groups, lane);
          stale = false;
        }
        if (!used_up && u < 64 && kh >= __builtin_amdgcn_readlane(live, u)) {
          // a chunk known to be of no use: no read for it.  Now and then the
          // stops are read again; once no group of the queue has a chunk of
          // use in this row, the queue's word is moved to its end.
          used_up = nx > 1 && nx <= 64 && !__any(kh < live);
          if (!used_up) {
            if (++moot % 8 == 0) stale = true;
            continue;
          }
          if (lane == 0)
            __hip_atomic_fetch_max(queue_word(P, qx), (P.epoch << kQueueBits) | (uint64_t)(nx * P.work_chunks),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (used_up) {
          if (i == nx * P.work_chunks) mark_used_up(P, qx, lane);
          // this queue is used up: go on with the next one that is not.
          // (Looking at all the queues' own words for that cost 7-9 % on
          // launches of many groups: the reads meet the other workgroups'
          // claims on the same lines.)
          open &= ~(1u << qx);
          open &= ~used_up_queues(P, done);
          live = 0x7fffffff;
          if (open) {
            const uint32_t after = open & ~((2u << qx) - 1u);
            qx = __builtin_ctz(after ? after : open);
          }
          continue;
        }
        const int g = queue_group(qx, u, n_groups);
        // the group's lengths (for a dense traversal of one of the first
        // kLenCache sequences from LDS, with no round trip); the loaders
        // check for a stop announced before the chunk with their page reads
        const int bq = g / P.num_kv_heads;
        const int L_raw = (bq < kLenCache && !P.block_list) ? lds_ld(&s_len[bq]) : P.seq_lens[bq];
        const int T_raw = raw_list_len(P, g);
        const GroupInfo gi = group_info_raw(P, g, L_raw, T_raw);
        if (gi.n_chunks == 0 && kh == 0) write_empty_wave<G>(P, gi.b, gi.kvh, lane);
        if (kh >= gi.n_chunks || (P.block_list && stop_word_before(ld_relaxed(P.stop_word + g), P.epoch, kh))) {
          stale = P.block_list || P.no_detector;  // (elsewhere the lengths, in LDS, tell it as fast)
          continue;
        }
        gsel = g;
        ksel = kh;
        len_sel = L_raw;
        list_sel = T_raw;
        break;
      }
      // (after a give-up the buffer may still be in the resolver's hands:
      // only the end marker is handed out, its other words stay untouched)
      if (lane == 0 && !gave_up) {
        lds_st(&s_meta[slot][kMetaGroup], gsel);
        lds_st(&s_meta[slot][kMetaChunk], ksel);
        lds_st(&s_meta[slot][kMetaLen], len_sel);
        lds_st(&s_meta[slot][kMetaListLen], list_sel);
        lds_st(&s_meta[slot][kMetaDone], 0);
        lds_st(&s_meta[slot][kMetaAbort], 0);
      }
      wave_lds_sync();
      if (lane == 0) {
        lds_st(&s_meta[slot][kMetaState], gsel >= 0 ? kSlotLoading : kSlotEnd);
        lds_st(&s_meta[slot][kMetaSeq], it);
      }
    }
    // every loader: wait for this iteration's assignment
    int st = kSlotFree;
    for (uint32_t spin = 0;; ++spin) {
      st = lds_ld(&s_meta[slot][kMetaState]);
      if (lds_ld(&s_meta[slot][kMetaSeq]) == it && (st == kSlotLoading || st == kSlotEnd)) break;
      if (wait_expired(P, spin)) return;
      __builtin_amdgcn_s_sleep(1);
    }
    if (st == kSlotEnd) return;
    const int gidx = lds_uniform(&s_meta[slot][kMetaGroup]);
    const int k = lds_uniform(&s_meta[slot][kMetaChunk]);
    const GroupInfo gi = group_info_raw(P, gidx, lds_uniform(&s_meta[slot][kMetaLen]),
                                        lds_uniform(&s_meta[slot][kMetaListLen]));
    const int t0 = chunk_start(P, k);
    const int nb = min(chunk_start(P, k + 1), gi.T) - t0;
    const int tpb = P.tiles_per_block;
    float* blocks = smem + slot * slot_floats;
    bool aborted = false;
    {
      bf16x8 qa[4];
      load_q<G>(P, gi.b, gi.kvh, lane, qa);
      // This wave streams blocks lw, lw + 3, ... of the chunk, each as its
      // tpb tiles in order.  The block list entry and the pages of all its
      // tiles are fetched together once per chunk: lane 4m + n covers
      // 16-token group n of the wave's m-th tile (at most 16 tiles per wave).
      const int n_my = lw < nb ? (nb - lw + kLoaders - 1) / kLoaders * tpb : 0;
      // Bounded speculation: chunk k waits until chunk k - max_ahead of the
      // group has been through the stability test (its summary, or its
      // inclusive state without the test), unless a stop before chunk k is
      // announced meanwhile.  The waited-on chunk was claimed earlier, so
      // it makes progress without this one.
      if (P.max_ahead > 0 && k >= P.max_ahead) {
        const uint64_t* fw = P.flags + (int64_t)gidx * P.max_chunks + (k - P.max_ahead);
        const uint32_t need = P.no_detector ? kInclusive : kStabSummary;
        for (uint32_t spin = 0;; ++spin) {
          if (flag_state(ld_relaxed(fw), P.epoch) >= need) break;
          if (stop_announced_before(P, gidx, k) || wait_expired(P, spin)) {
            aborted = true;
            break;
          }
          __builtin_amdgcn_s_sleep(2);
        }
      }
      // the stop word travels with the page reads: a chunk that lies after
      // an announced stop is given up before any tile is loaded
      const uint64_t sw0 = ld_relaxed(P.stop_word + gidx);
      int my_tok0 = 0x7fffffff, my_page = 0;
      {
        const int m = lane >> 2, n = lane & 3;
        if (m < n_my) {
          const int i = lw + kLoaders * (m / tpb), j = m % tpb;
          const int step = t0 + i;
          int blk;
          if (gi.list) {
            blk = gi.list[step];
            blk = blk < 0 ? 0 : (blk >= gi.nblk ? gi.nblk - 1 : blk);
          } else {
            blk = P.dense_order == 1 ? step : gi.nblk - 1 - step;
          }
          my_tok0 = blk * P.block_size + j * kTile;
          if (my_tok0 < gi.L) my_page = clamp_page(P, gi.b, min(my_tok0 + 16 * n, gi.L - 1));
        }
      }
      if (stop_word_before(sw0, P.epoch, k)) {
        aborted = true;
        // (with one group per queue the claims of its last chunks keep its
        // workgroups from crowding the others: long_512k 208 us, 214 with)
        stale = n_groups > kQueues;
      }
      for (int m = 0; m < n_my && !aborted; ++m) {
        const int i = lw + kLoaders * (m / tpb), j = m % tpb;
        // a stop announced by an earlier chunk makes this chunk's work moot;
        // the flag read here completes while the tile's loads are in flight
        const uint64_t sw = ld_relaxed(P.stop_word + gidx);
        const int tok0 = __builtin_amdgcn_readlane(my_tok0, 4 * m);
        const int pg[4] = {__builtin_amdgcn_readlane(my_page, 4 * m), __builtin_amdgcn_readlane(my_page, 4 * m + 1),
                           __builtin_amdgcn_readlane(my_page, 4 * m + 2), __builtin_amdgcn_readlane(my_page, 4 * m + 3)};
        compute_tile<G, WIDE>(*fresh(args), gi.kvh, gi.L, tok0, pg, qa,
                        P.v_in_record ? reinterpret_cast<uint16_t*>(blocks + i * REC) : vbuf,
                        blocks + i * REC, j > 0);
        if (stop_word_before(sw, P.epoch, k)) {
          aborted = true;
          break;
        }
      }
    }
    wave_lds_sync();
    if (aborted) {
      if (lane == 0) lds_st(&s_meta[slot][kMetaAbort], 1);
    }
    wave_lds_sync();
    stress_delay(P, gidx, k, 13 + lw);
    if (lane == 0) {
      const int done = __hip_atomic_fetch_add(&s_meta[slot][kMetaDone], 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
      if (done == kLoaders - 1) lds_st(&s_meta[slot][kMetaState], kSlotReady);
    }
  }
}

__global__ void fill_zero_kernel(uint32_t* p, size_t n_words) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += stride) p[i] = 0u;
}

template <int G, bool PH, bool WIDE>
int launch_w(const Plan& plan, const KernelParams& params, hipStream_t stream) {
  const int64_t work = (int64_t)plan.n_groups * plan.max_chunks;
  if (work <= 0) return (int)hipSuccess;
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, art_decode_kernel<G, PH, WIDE>, kThreads, plan.lds_bytes);
  if (e != hipSuccess) return (int)e;
  if (per_cu < 1) per_cu = 1;
  // As many workgroups as the chip holds, but no more than the plan allows
  // per group (and never fewer than one per CU).
  const int64_t per_groups = max((int64_t)cus, (int64_t)plan.group_workgroups * plan.n_groups);
  const int64_t grid = min(work, min((int64_t)cus * per_cu, per_groups));
  // Chunks of one group in flight at once: about the launch's chunk buffers
  // over the groups.  Up to 8 (many groups), a chunk of a group of 8 or
  // more heads looks back before it publishes its aggregate (measured: -2 %
  // on 256 groups of g = 8, +5 to +13 % with 32 or more buffers per group).
  // A function of the shape and the device only; the results are the same
  // bits either way.
  KernelParams p = params;
  p.look_first = grid * kChunkSlots <= (int64_t)8 * plan.n_groups ? 1 : 0;
  auto kernel = art_decode_kernel<G, PH, WIDE>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kThreads),
                     plan.lds_bytes, stream, p);
  return (int)hipGetLastError();
}

template <int G, bool PH>
int launch_g(const Plan& plan, const KernelParams& params, hipStream_t stream) {
  return params.wide ? launch_w<G, PH, true>(plan, params, stream) : launch_w<G, PH, false>(plan, params, stream);
}

}  // namespace

int launch_decode(const Plan& plan, const KernelParams& params, hipStream_t stream) {
  switch (plan.group) {
    case 1: return params.per_head ? launch_g<1, true>(plan, params, stream) : launch_g<1, false>(plan, params, stream);
    case 2: return params.per_head ? launch_g<2, true>(plan, params, stream) : launch_g<2, false>(plan, params, stream);
    case 4: return params.per_head ? launch_g<4, true>(plan, params, stream) : launch_g<4, false>(plan, params, stream);
    case 8: return params.per_head ? launch_g<8, true>(plan, params, stream) : launch_g<8, false>(plan, params, stream);
    case 16: return params.per_head ? launch_g<16, true>(plan, params, stream) : launch_g<16, false>(plan, params, stream);
    default: return (int)hipErrorInvalidValue;
  }
}

int launch_fill_zero(void* ptr, size_t bytes, hipStream_t stream) {
  const size_t words = bytes / 4;
  if (words == 0) return (int)hipSuccess;
  size_t blocks = (words + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                     static_cast<uint32_t*>(ptr), words);
  return (int)hipGetLastError();
}

}  // namespace art
