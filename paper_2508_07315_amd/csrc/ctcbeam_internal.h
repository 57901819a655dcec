// Internal layouts shared by the host builders and the gfx950 kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

struct ctcbeam_lm;
struct ctcbeam_boost;
struct ctcbeam_opts;

namespace ctcbeam {

constexpr int kThreads = 512;         // threads per workgroup (8 wave64)
constexpr int kWaves = kThreads / 64;
constexpr int kClassThreads = 512;    // threads per workgroup of the class decoder
constexpr int kMaxK = 128;            // beam size limit
constexpr int kMaxKWideV = 64;        // beam size limit above 1024 tokens
constexpr int kLmStage = 4096;        // staged LM arcs per chunk (12-bit slot)
constexpr int kCap = 512;             // survivor pool entries
constexpr uint32_t kExists = 0x80000000u;
constexpr int kFlagLogSumExp = 1;      // recombination by log-sum-exp
constexpr int kFlagBoostRollback = 2;  // pending boosting taken back at the end
constexpr int kFlagNoRowCache = 4;     // LM key rows refilled for every beam every frame
constexpr int kFlagRepeatScore = 8;    // repeated tokens get their LM / boosting terms again
// Workspace: [header, kWsHeaderBytes][status word per utterance, padded to
// 256 B][back-pointers [B, T, K] int32].  The header records the batch size
// of the last decode that used the workspace, so that its status can be read
// back from the workspace alone: {kWsMagic, B, ~B}.
constexpr size_t kWsHeaderBytes = 256;
constexpr uint32_t kWsMagic = 0x42435443u;  // "CTCB"

// LM state record, one per chain level l (context of length l+1):
//   {arc_begin, arc_count | kExists, backoff bits}
// Per-phase clocks of the kernels in profiling builds (-DCTCBEAM_PHASE_CLOCKS):
// a kernel declares uint64_t ph_acc (lane k of each wave holds word k) and
// ph_t0; each CTCBEAM_PHASE_MARK(k) adds the s_memtime cycles since the
// previous mark to word k, CTCBEAM_PHASE_COUNT(k) adds one and
// CTCBEAM_PHASE_ADD(k, n) adds n.  One register
// pair per wave keeps the profiling build's register use close to the
// product's.  Product builds compile none of it.
constexpr int kPhaseWords = 20;
#ifdef CTCBEAM_PHASE_CLOCKS
#define CTCBEAM_PHASE_MARK(k)                                          \
  do {                                                                 \
    const uint64_t now_ = __builtin_amdgcn_s_memtime();                \
    ph_acc += ((threadIdx.x & 63u) == (k)) ? now_ - ph_t0 : 0ull;      \
    ph_t0 = now_;                                                      \
  } while (0)
#define CTCBEAM_PHASE_ADD(k, n)                                                      \
  do {                                                                               \
    ph_acc += ((threadIdx.x & 63u) == (k)) ? static_cast<uint64_t>(n) : 0ull;        \
  } while (0)
#else
#define CTCBEAM_PHASE_ADD(k, n) \
  do {                          \
  } while (0)
#define CTCBEAM_PHASE_MARK(k) \
  do {                        \
  } while (0)
#endif
#define CTCBEAM_PHASE_COUNT(k) CTCBEAM_PHASE_ADD(k, 1)

struct LmLevel {
  uint32_t begin;
  uint32_t count;   // low 31 bits: arcs; bit 31: the context is an entry
  float bo;
};
// LM arc: ln probability of (context, token), next state after emitting token
struct LmArc {
  float logp;
  uint32_t target;
  uint32_t token;
};
// Boosting tree state record.
struct BtNode {
  uint32_t list_begin;
  uint32_t list_count;
  uint32_t pot;        // low 8 bits: pot; bits 8..31: chain nodes (statistics)
  uint32_t chain_arcs; // statistics only
};
struct BtEntry {
  uint32_t token;
  uint32_t key;        // (prio << 26) | (pre << 20) | child
};
constexpr uint32_t kBtChildMask = (1u << 20) - 1;

struct KernelParams {
  const float* logprobs;
  const int32_t* lengths;
  int B, T, V, K;
  float alpha, beta, boost_w, theta;
  int flags;                 // kFlag* bits
  // LM (null when disabled)
  const LmLevel* lm_states;
  const LmArc* lm_arcs;
  const float* lm_unigram;   // [V+1], index V = </s>
  int lm_nlev;
  uint32_t lm_bos_state;
  int lm_states_below_2p23;  // every LM state id fits 23 bits
  int64_t lm_n_states;       // number of LM states
  float lm_absmax;           // bound of |ln P| of a finite LM query
  float lm_max, lm_min;      // upper and lower bound of an LM query (entries of -inf count)
  // boosting (null when disabled)
  const BtNode* bt_nodes;
  const BtEntry* bt_list;
  const uint32_t* bt_root_key;  // [V]
  // workspace / outputs
  uint32_t* ws_header;       // workspace header (written by workgroup 0)
  uint32_t* status;          // [B]
  int32_t* bp;               // [B, T, K]
  int32_t* out_tokens;       // [B, T] or null (then no 1-best output)
  int32_t* out_lengths;      // [B] or null
  float* out_scores;         // [B] or null
  int64_t* stats;            // [B, 8] or null
  // N-best output (nbest_scores null: none; nbest_tokens may be null when
  // T = 0): every slot's final hypothesis ordered by
  // final score, lowest slot on ties; dead slots last, empty, -inf
  int32_t* nbest_tokens;     // [B, K, T]
  int32_t* nbest_lengths;    // [B, K]
  float* nbest_scores;       // [B, K]
};

// Record the batch size in the workspace header (one thread of one workgroup).
__device__ __forceinline__ void write_ws_header(uint32_t* hdr, int B) {
  hdr[0] = kWsMagic;
  hdr[1] = static_cast<uint32_t>(B);
  hdr[2] = ~static_cast<uint32_t>(B);
}

// Kernel variants by labels per lane (V <= 512 * LPT); each dispatches on the
// LM order and on boosting.  Return the launch's hipError_t.
hipError_t launch_lpt1(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt2(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt4(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt8(const KernelParams& p, hipStream_t stream);
// the same for the repeat-scoring variant (CTCBEAM_FLAG_REPEAT_SCORE with an
// LM or boosting)
hipError_t launch_lpt1_rep(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt2_rep(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt4_rep(const KernelParams& p, hipStream_t stream);
hipError_t launch_lpt8_rep(const KernelParams& p, hipStream_t stream);

// Greedy (one hypothesis) kernels by vocabulary: up to 256 tokens (one wave
// per utterance), 1024 and 4096 tokens (four waves).
hipError_t launch_greedy_v256(const KernelParams& p, hipStream_t stream);
hipError_t launch_greedy_v1024(const KernelParams& p, hipStream_t stream);
hipError_t launch_greedy_v4096(const KernelParams& p, hipStream_t stream);

// Writes the header of an empty batch (B = 0: no decode kernel runs).
hipError_t launch_ws_header(uint32_t* hdr, int B, hipStream_t stream);

inline hipError_t launch_greedy(const KernelParams& p, hipStream_t stream) {
  if (p.B == 0) return hipSuccess;
  if (p.V <= 256) return launch_greedy_v256(p, stream);
  if (p.V <= 1024) return launch_greedy_v1024(p, stream);
  return launch_greedy_v4096(p, stream);
}

// The 1-best decode of ctcbeam_decode_ex into a given workspace (host side,
// ctcbeam_host.cpp): validation, parameter block, launch; the C entry
// points' return codes.  set_last_error records the message that
// ctcbeam_last_error returns and passes the code through.
int decode_with_workspace(const float* logprobs, const int32_t* lengths, int B, int T, int V, int K,
                          float alpha, float beta, float boost_w, const ctcbeam_lm* lm,
                          const ctcbeam_boost* boost, void* workspace, size_t workspace_bytes,
                          int32_t* out_tokens, int32_t* out_lengths, float* out_scores,
                          hipStream_t stream, const ctcbeam_opts* opts);
int set_last_error(int code, const char* msg);

// Small-beam decoder (ctcbeam_small.inl): beams of at most 8, at most 1024
// tokens, no LM and no boosting, max recombination.
bool small_beam_eligible(const KernelParams& p);
hipError_t launch_small(const KernelParams& p, hipStream_t stream);

// Class decoder (ctcbeam_class.inl) by vocabulary: up to 512, 1024, 2048 and
// 4096 tokens.
hipError_t launch_class_lpt1(const KernelParams& p, hipStream_t stream);
hipError_t launch_class_lpt2(const KernelParams& p, hipStream_t stream);
hipError_t launch_class_lpt4(const KernelParams& p, hipStream_t stream);
hipError_t launch_class_lpt8(const KernelParams& p, hipStream_t stream);

// Whether the class decoder serves a beam search.  It scores V labels once per
// class of beams instead of once per beam, but spends more dependent steps a
// frame and keeps fewer LM rows in LDS the more tokens there are.  Figures:
// general / class decoder time, 32 utterances of 250 frames, models counted in
// synthetic text (shorter utterances favour the general decoder: 0.85 for 1.00
// at 60 frames, 3000 tokens, 3-gram, K = 12).
// - Beams of one chunk of the general decoder stay there (K = 8, 1024 tokens,
//   3-gram: 0.67), except over character sets, whose few labels leave the
//   general decoder's bound too loose (64 tokens, K = 9..16: 1.3..3.0; 10
//   tokens 1.03..1.3; with phrases from about 144 candidates a frame: 8 tokens,
//   K = 16 0.95..1.10, 16 tokens, K = 9 0.97..1.05).
// - Above 16 beams it is faster throughout (17 beams 0.93..2.1, 24 beams
//   0.98..1.9 with a 2-gram or higher and phrases at 1600 to 4096 tokens).
// - Phrases alone: 1.1 and above, but for K = 3 and 4 over wide vocabularies
//   (2560 tokens 0.97..1.03, 4096 tokens 0.87..0.92).
// - LM and phrases: 1.08 and above from 2049 to 2560 tokens; at 4096 tokens
//   0.75..0.95.  Just below 2048 tokens, where an LDS holds five LM rows and as
//   many boosting rows, it loses for 3- and 4-grams at K = 7..16 (1900 to 2048
//   tokens 0.90..1.04; 1800 tokens 1.03..1.16; other orders 0.96..1.3).
// - LM alone: up to 3072 tokens 0.98..1.11, below 2-grams more, above 4-grams
//   1.3; K = 3 0.96..1.00 for 2- to 4-grams; at 4096 tokens 0.72..0.95.
inline bool class_eligible(const KernelParams& p) {
  const bool lm = p.lm_states != nullptr || p.lm_arcs != nullptr, bt = p.bt_nodes != nullptr;
  const int chunk = p.V <= 512 ? 16 : p.V <= 1024 ? 8 : p.V <= 2048 ? 4 : 2;
  if (p.K <= chunk) return p.V <= 64 && p.K > 8 && (!bt || p.V * p.K >= 144);
  if (p.K > 16) return true;
  if (!lm) return !bt || p.K > 4 || p.V <= 2560;
  if (!bt) return p.V <= 3072 && !(p.V > 2048 && p.K == 3 && p.lm_nlev >= 1 && p.lm_nlev <= 3);
  if (p.V > 1800 && p.V <= 2048 && p.K > 6) return p.lm_nlev != 2 && p.lm_nlev != 3;
  return p.V <= 2560;
}

// The general decoder's forms for beams of several chunks, of which a chunk
// takes 16 / lpt: whether class_eligible leaves it some at lpt labels per lane,
// for an LM of nlev levels (-1: none).
constexpr bool multi_chunk(int lpt, int nlev, bool boosting) {
  if (lpt == 8) return nlev >= 0 || boosting;
  return lpt == 4 && boosting && (nlev == 2 || nlev == 3);
}

inline hipError_t launch_decode(const KernelParams& p, hipStream_t stream) {
  if (p.B == 0) return hipSuccess;
  if (small_beam_eligible(p)) return launch_small(p, stream);
  if (class_eligible(p)) {
    if (p.V <= kClassThreads) return launch_class_lpt1(p, stream);
    if (p.V <= 2 * kClassThreads) return launch_class_lpt2(p, stream);
    if (p.V <= 4 * kClassThreads) return launch_class_lpt4(p, stream);
    return launch_class_lpt8(p, stream);
  }
  // repeat scoring changes nothing without an LM or boosting
  if ((p.flags & kFlagRepeatScore) && (p.lm_states != nullptr || p.lm_arcs != nullptr || p.bt_nodes != nullptr)) {
    if (p.V <= 512) return launch_lpt1_rep(p, stream);
    if (p.V <= 1024) return launch_lpt2_rep(p, stream);
    if (p.V <= 2048) return launch_lpt4_rep(p, stream);
    return launch_lpt8_rep(p, stream);
  }
  if (p.V <= 512) return launch_lpt1(p, stream);
  if (p.V <= 1024) return launch_lpt2(p, stream);
  if (p.V <= 2048) return launch_lpt4(p, stream);
  return launch_lpt8(p, stream);
}

}  // namespace ctcbeam
