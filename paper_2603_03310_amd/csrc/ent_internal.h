// Internal declarations shared by the HIP translation units of libent.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "ent.h"

namespace ent {

constexpr int kBlock = ENT_BLOCK_SIZE;      // tokens per KV block
constexpr int kRowChunk = ENT_ROW_CHUNK;    // logits per entropy chunk
constexpr int kMinScoreChunk = 16;          // smallest scoring chunk (blocks)
constexpr int kMaxGroup = 16;               // query heads per KV head
constexpr int kMaxBlocksPerSeq = 16384;     // selection keeps all scores in LDS
constexpr int kEstChunkThreads = 256;       // threads of an entropy chunk job (maxima per chunk)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Parameters of the controller (Section 3.3 and Section 5): the signed gain,
// the target entropy, the temperature bounds, the bound on the temperature's
// log step per update, and the entropy offset of the stress tests.
struct Control {
  float eta, h_target, t_min, t_max, rho_t, h_bias;
};
Control make_control(const ent_config& cf);

// Parameters of the block budget and the kept-fraction state (Sections
// 3.2, 3.3, 5): the guarded entropy, the floor, the smallest fraction and
// count, and the bound on how fast the kept fraction may fall.
struct Budget {
  float eps_h, h_min, log_v, kappa_min, dkappa;
  int b_min;
  int keep_first, keep_last;   // blocks always kept at each end of a sequence
  float* kappa;   // nullable [B]: previous kept fraction (NaN = none), updated in place
};

// Arguments of the append body (ent_kv_append), which also runs inside the
// last launch of ent_decode_step_append.
struct AppendArgs {
  const void* k_new;
  const void* v_new;
  const int* tables;
  int* ctx_lens;
  void* kc;
  void* vc;
  float* ksum;
  int Hkv, D, MAXB, P;
  unsigned* flags;
  bool bf16;
};

}  // namespace ent

struct ent_ctx {
  ent_config cfg;
  int device = 0;
  int num_cu = 0;
  int group = 1;            // G = H_q / H_kv
  int chunks = 0;           // entropy chunks per logit row
  int lse_chunks = 0;       // log-sum-exp partials per sequence (finest chunking)
  int decode_grid = 0;      // persistent decode workgroups
  int prologue_grid = 0;    // resident entropy / scoring workgroups
  int b1_occ_plain = 0;     // resident tile-launch workgroups per CU, without the selection inside
  int b1_occ_ticket = 0;    // ... and with it

  void* ws = nullptr;       // one workspace allocation
  size_t ws_bytes = 0;
  float* ent_part = nullptr;      // [max_batch, chunks, 3]  (max, sum, weighted sum)
  float* stats_tmp = nullptr;     // [max_batch, chunks, 2]  row statistics scratch
  float* zbuf = nullptr;          // [max_batch, MAXB, H_q]  block logits
  float* lse_part = nullptr;      // [max_batch, lse_chunks, H_q, 2]
  float* lrow = nullptr;          // [max_batch, H_q]  L_h per sequence
  float* iscores = nullptr;       // [max_batch, MAXB]  block scores when the caller keeps none
  int* kept_phys = nullptr;       // [max_batch, MAXB]  physical blocks of the kept lists
  float* dec_acc = nullptr;       // [decode partial slots, G, d]
  float* dec_ml = nullptr;        // [decode partial slots, G, 2]
  int2* dec_rec = nullptr;        // [decode waves]  cut-segment records of the decode ranges
  float* tmax = nullptr;          // [max_batch, chunks, 256]  per-thread logit maxima (estimators)
  float2* exbuf = nullptr;        // [max_batch, MAXB, H_q]  exact mode: (log mass, mean logit) per block
  unsigned* tickets = nullptr;    // [max_batch]  per-sequence counters of the fused step (zero between launches)
  unsigned* dev_flags = nullptr;  // [1]

  std::string err;
};

namespace ent {

// Whether the controller acts on an estimate (top-k or tail-corrected) of
// the entropy: with k >= |V| both estimates are the exact entropy.
inline bool uses_estimate(const ent_config& cf) {
  return cf.estimator != ENT_EST_EXACT && cf.est_k < cf.vocab;
}

// Launchers (one per kernel family); each returns the launch status.
hipError_t launch_entropy(const ent_ctx* c, int B, const float* logits, long long ld,
                          ent_state st, float* h_out, float* temp_used, float* row_stats,
                          bool controller, hipStream_t s);
hipError_t launch_sample(const ent_ctx* c, int B, const float* logits, long long ld,
                         const float* row_stats, const float* temp_used, const float* uniforms,
                         int* tokens, hipStream_t s);
hipError_t launch_block_summary(const ent_ctx* c, int B, const void* k_cache,
                                const int* tables, const int* ctx_lens, float* ksum,
                                hipStream_t s);
hipError_t launch_block_select(const ent_ctx* c, int B, const void* q, const float* ksum,
                               const void* k_cache, const int* tables, const int* ctx_lens,
                               const float* h, int* kept, int* n_kept, float* scores,
                               float* theta, float* kappa, hipStream_t s);
// Exact token-level scoring: per block and query head (log mass, mean logit)
// into c->exbuf and the per-tile log-sum-exp partials into c->lse_part.
hipError_t launch_exact_scores(const ent_ctx* c, int B, const void* q, const void* k_cache,
                               const int* tables, const int* ctx_lens, hipStream_t s);
// Block scores of the exact mode from c->exbuf and c->lrow.
hipError_t launch_exact_block_scores(const ent_ctx* c, int B, const int* ctx_lens, float* scores,
                                     hipStream_t s);
// Selection phase A: L_h of every sequence into c->lrow from c->lse_part.
hipError_t launch_lse_merge(const ent_ctx* c, int B, const int* ctx_lens, hipStream_t s);
Budget make_budget(const ent_config& cf, float* kappa);
// The pass over logits and block summaries that opens a step:
// entropy chunk triples / row statistics (do_entropy) and block scoring of
// bf16 queries (do_score), in one grid.
struct PrologueArgs {
  int B;
  int do_entropy;
  const float* logits;
  long long ld;
  int V, C;
  const float* temp;
  float* part;          // chunk triples (nullable)
  float* row_stats;     // chunk (max, sum) (nullable)
  float* temp_used;     // nullable: receives temp[b] (written by chunk 0's job)
  float* tmax;          // nullable: per-thread maxima of the chunk, [B, C, 256] (estimators)
  float t_cal;          // calibration temperature: the chunk pass uses temp[b] * t_cal
  int do_score;
  const uint16_t* q;
  const float* ksum;
  const int* tables;
  const int* ctx_lens;
  float* zbuf;
  float* lse_part;
  int Hkv, G, MAXB, P, nch_max;
  float scale;
  unsigned* flags;
};
hipError_t launch_prologue(const ent_ctx* c, const PrologueArgs& a, hipStream_t s);
// fp32 queries: the entropy pass and the block scoring in one launch.  False
// (nothing launched) where the scoring's LDS would cost the entropy workgroups
// residency: launch_prologue and launch_score_valu then.
bool launch_prologue_f32(const ent_ctx* c, const PrologueArgs& a, const float* q, hipStream_t s,
                         hipError_t* e);
int prologue_grid_size(const ent_ctx* c);
// Residency of the fused step's tile launch with and without the selection
// inside (ent_ctx::b1_occ_*).
void step_occupancy(ent_ctx* c);
// The kept-block selection after scoring (L merge, block scores, radix
// select), given each sequence's entropy h.
hipError_t launch_selection(const ent_ctx* c, int B, const int* tables, const int* ctx_lens,
                            const float* h, float* scores, float* theta, int* kept, int* n_kept,
                            float* kappa, hipStream_t s);
// Selection phases B (block scores from c->lrow) and C (radix select).
hipError_t launch_block_scores(const ent_ctx* c, int B, const int* ctx_lens, float* scores,
                               hipStream_t s);
hipError_t launch_select_rows(const ent_ctx* c, int B, const int* tables, const int* ctx_lens,
                              const float* h, const float* scores, float* theta, int* kept,
                              int* n_kept, float* kappa, hipStream_t s);
hipError_t launch_score_valu(const ent_ctx* c, int B, const void* q, const float* ksum,
                             const int* tables, const int* ctx_lens, hipStream_t s);

// Sampling issued in the launch that runs the kept-block selection (the
// fused step), on workgroups of its own; the arguments of ent_sample.
struct SampleArgs {
  const float* logits;
  long long ld;
  int V, C;
  const float* stats;
  const float* temp_used;
  const float* uniforms;
  int* tokens;
  float t_cal;          // calibration temperature: sampling at temp_used[b] * t_cal
};

// kept_phys (nullable): the selection's encoded physical blocks of the same
// kept lists, read instead of kept + tables.
// ap (nullable): an append of one token per sequence, and sp (nullable) the
// sampling of every row, that share the launch merging the split attention
// segments (none of the three reads what another writes).
hipError_t launch_decode(const ent_ctx* c, int B, const void* q, const void* k_cache,
                         const void* v_cache, const int* tables, const int* ctx_lens,
                         const int* kept, const int* n_kept, float* out, float* lse,
                         hipStream_t s, const int* kept_phys = nullptr,
                         const AppendArgs* ap = nullptr, const SampleArgs* sp = nullptr);
hipError_t launch_decode_step(const ent_ctx* c, int B, const float* logits, long long ld,
                              ent_state st, const void* q, const void* k_cache,
                              const void* v_cache, const float* ksum, const int* tables,
                              const int* ctx_lens, const float* uniforms, float* h_out,
                              float* temp_used, float* row_stats, int* kept, int* n_kept,
                              float* out, float* lse, int* tokens, float* scores, float* theta,
                              hipStream_t s, const AppendArgs* ap = nullptr);
AppendArgs make_append_args(const ent_ctx* c, const void* k_new, const void* v_new,
                            const int* tables, int* ctx_lens, void* k_cache, void* v_cache,
                            float* ksum);
hipError_t launch_kv_append(const ent_ctx* c, int B, const void* k_new, const void* v_new,
                            const int* tables, int* ctx_lens, void* k_cache, void* v_cache,
                            float* ksum, hipStream_t s);
hipError_t launch_schedule(int N, const ent_sched_params& p, const float* tau, const int* n_kept,
                           const int* ctx_lens, float* tau_last, float* gain, int* age, int b_sel,
                           int* selected, int* n_selected, float* priority, hipStream_t s);

// Configuration check of ent_init (message, ENT_OK / ENT_E_INVAL /
// ENT_E_UNSUPPORTED in *code), and the message ent_last_error(NULL) returns
// (calls without a context: ent_init, ent_entropy_temperature_noalloc).
std::string config_error(const ent_config* cfg, int* code);
void set_free_error(const std::string& msg);

// Occupancy-derived persistent grid of the decode kernel, and the number of
// partial slots its split segments may use (waves + segments).
int decode_grid_size(const ent_ctx* c);
long long decode_partial_slots(int decode_grid, int max_batch, int num_kv_heads);

}  // namespace ent

// ---------------------------------------------------------------------------
// Device helpers
// ---------------------------------------------------------------------------
#if defined(__HIPCC__)
namespace ent {

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round-to-nearest-even float -> bf16 bits (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// Cross-lane moves on the vector ALU (DPP within rows of 16 lanes, lane swaps
// across them), without LDS latency at every step.  The butterflies below add
// in the order of shuffles and give their bits; the scans add whole rows of 16
// lanes, where a scan by shuffles adds windows that cross them: the same for
// integers, while the float64 sums of wave_scan_d (the sampler's) can differ
// from such a scan's in their last bits.  (A shuffle's result comes
// back after the LDS queue; six of them make one wave reduction, and the
// selection, estimator and sampling bodies chain dozens.)  Against the shuffles:
// sampling alone 17.6 -> 16.1 us, the fp32 tiny step 32.8 -> 31.1, one request
// 27.7 -> 26.2, the 8B step 193.0 -> 190.8, with the tail estimate 259.3 -> 255.1.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ unsigned dpp_u(unsigned old, unsigned v) {
  return static_cast<unsigned>(__builtin_amdgcn_update_dpp(static_cast<int>(old), static_cast<int>(v),
                                                           CTRL, ROWS, 0xf, false));
}
// v of lane (lane ^ M), M = 1, 2, 4, 8 or 16.
template <int M>
__device__ __forceinline__ unsigned xor_lane(unsigned v) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16, "within half a wave");
  if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const unsigned even = r[0], odd = r[1];                // the pair of rows' values
    return (threadIdx.x & 16) ? even : odd;
  } else if constexpr (M == 1) return dpp_u<0xB1>(v, v);          // quad_perm 1, 0, 3, 2
  else if constexpr (M == 2) return dpp_u<0x4E>(v, v);     // quad_perm 2, 3, 0, 1
  else if constexpr (M == 8) return dpp_u<0x128>(v, v);    // row_ror 8
  else {
    const unsigned m = dpp_u<0x141>(v, v);                 // row_half_mirror: lane ^ 7
    return dpp_u<0x1B>(m, m);                              // quad_perm 3, 2, 1, 0: lane ^ 3
  }
}
// op(v, v of lane ^ M) for a commutative op on a 32-bit type, M a power of two.
template <int M, typename T, typename Op>
__device__ __forceinline__ T xor_op(T v, Op op) {
  static_assert(sizeof(T) == 4, "32-bit values");
  const unsigned u = __builtin_bit_cast(unsigned, v);
  if constexpr (M >= 16) {
    // Both halves (or rows) of each pair, in every lane: the lower lanes' in
    // the first, the upper lanes' in the second.
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false)
                           : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned lo = r[0], hi = r[1];
    return op(__builtin_bit_cast(T, lo), __builtin_bit_cast(T, hi));
  } else {
    const unsigned o = xor_lane<M>(u);
    return op(v, __builtin_bit_cast(T, o));
  }
}
struct OpMaxF { __device__ __forceinline__ float operator()(float x, float y) const { return fmaxf(x, y); } };
struct OpAddF { __device__ __forceinline__ float operator()(float x, float y) const { return x + y; } };
struct OpMinU { __device__ __forceinline__ unsigned operator()(unsigned x, unsigned y) const { return min(x, y); } };
struct OpMaxU { __device__ __forceinline__ unsigned operator()(unsigned x, unsigned y) const { return max(x, y); } };
struct OpAddU { __device__ __forceinline__ unsigned operator()(unsigned x, unsigned y) const { return x + y; } };
template <int M>
__device__ __forceinline__ float xor_max(float v) { return xor_op<M>(v, OpMaxF()); }
template <int M>
__device__ __forceinline__ float xor_add(float v) { return xor_op<M>(v, OpAddF()); }

// Butterfly over the wave (result in every lane).
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
  v = xor_op<32>(v, op);
  v = xor_op<16>(v, op);
  v = xor_op<8>(v, op);
  v = xor_op<4>(v, op);
  v = xor_op<2>(v, op);
  return xor_op<1>(v, op);
}
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, OpMaxF()); }
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, OpAddF()); }
__device__ __forceinline__ unsigned wave_min_u(unsigned v) { return wave_reduce(v, OpMinU()); }
__device__ __forceinline__ unsigned wave_max_u(unsigned v) { return wave_reduce(v, OpMaxU()); }
__device__ __forceinline__ unsigned wave_sum_u(unsigned v) { return wave_reduce(v, OpAddU()); }

// Inclusive prefix sums over the wave: within rows of 16 lanes by row shifts,
// then the last lane of row 0 (of 2) to row 1 (3), and lane 31 to rows 2 and 3.
__device__ __forceinline__ unsigned wave_scan_u(unsigned v) {
  v += dpp_u<0x111>(0u, v);
  v += dpp_u<0x112>(0u, v);
  v += dpp_u<0x114>(0u, v);
  v += dpp_u<0x118>(0u, v);
  v += dpp_u<0x142, 0xa>(0u, v);
  v += dpp_u<0x143, 0xc>(0u, v);
  return v;
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_or_zero_d(double v) {
  const uint2 u = __builtin_bit_cast(uint2, v);
  return __builtin_bit_cast(double, make_uint2(dpp_u<CTRL, ROWS>(0u, u.x), dpp_u<CTRL, ROWS>(0u, u.y)));
}
__device__ __forceinline__ double wave_scan_d(double v) {
  v += dpp_or_zero_d<0x111>(v);
  v += dpp_or_zero_d<0x112>(v);
  v += dpp_or_zero_d<0x114>(v);
  v += dpp_or_zero_d<0x118>(v);
  v += dpp_or_zero_d<0x142, 0xa>(v);
  v += dpp_or_zero_d<0x143, 0xc>(v);
  return v;
}
// v of lane i, the same i in every lane of the wave.
__device__ __forceinline__ int lane_at(int v, int i) {
  return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(i));
}
__device__ __forceinline__ float lane_at(float v, int i) {
  return __builtin_bit_cast(float, lane_at(__builtin_bit_cast(int, v), i));
}
__device__ __forceinline__ double lane_at(double v, int i) {
  const int2 u = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(lane_at(u.x, i), lane_at(u.y, i)));
}

__device__ __forceinline__ void raise_flag(unsigned* flags, unsigned f) {
  atomicOr(flags, f);
}

}  // namespace ent
#endif
