// Batched CTC beam search, all frames of one utterance per workgroup (gfx950).
// Included by the per-vocabulary instantiation units (ctcbeam_class_lpt*.hip).
//
// Implements the per-frame step of FlexCTC Algorithm 1 (score update with the
// blank/repeat masks, flat TopK over K*(V+1) candidates, threshold pruning,
// LM/boosting state update for emitting labels, beam update, recombination)
// followed by LM.Final and the transcript read-out of the hypothesis trie
// (Sec. III-A).  Scores follow Eq. 1 with the fp32 fold
//   x = s_k + D[c]; x += beta; x += fl(alpha*LM); x += fl(w*BT)
// for emitting labels (neither blank nor a repeat of the beam's last frame
// label).
//
// The search is a serial chain over frames: each utterance is one persistent
// workgroup of 8 wave64 that loops over its own frames, and the B utterances
// are independent workgroups.  There is no dense contraction, so no MFMA.
// What bounds a frame is the VALU rate of one CU (64 fp32 lanes a cycle) and
// the latency of the dependent phases (LDS round trips, barriers, the loads
// of new LM states).
//
// Classes.  The beams of an utterance sit in few LM and boosting states (64
// beams in about a dozen), and every term of Eq. 1 but s_k depends on the
// state and the label only.  fp32 addition is monotone, so within a class of
// beams with equal states the beam with the highest score bounds every other
// beam's score of each label.  A frame therefore scores V labels once per
// class instead of once per beam, and expands to the class's beams only the
// (class, label) pairs that reach a lower bound of the K-th best candidate.
//
// Per frame:
//   P. classes: every wave names the distinct (LM state, boosting node) pairs
//      of the live beams and finds their rows in LDS, both through small hash
//      tables in LDS.  Rows are kept across frames per LM state (64-bit
//      entries: order, successor state, fl(alpha*LM)) and per boosting node
//      (keys); a state without a row takes one that no class of this frame
//      uses.  A pass takes up to 16 classes, as many as rows are to be had;
//      beams with more take several passes.
//   F. fill of new rows, one wave a row: the unigram + backoff fold of every
//      label (a boosting row: the root keys); then, after a barrier, the
//      explicit arcs of the states' backoff chains over it, in tiles of 64
//      dealt to the waves (64-bit maximum, the longest context wins).
//   C. scoring: V labels of every class with the class's highest score, and
//      the maxima of 8 label groups per class.
//   T. bound: the maxima shifted by each beam's distance from its class's
//      best (less a bound of the rounding) are K * 8 distinct candidates;
//      with the blank and repeat candidates their K-th largest, found through
//      a histogram, bounds the K-th best candidate from below.
//   E. expansion: each wave takes its (class, label) pairs at or above the
//      bound and scores them exactly for the class's beams, lane = beam; the
//      candidates at or above the bound go to a pool in LDS.
//   R. rank: the pool is ranked exactly by (score desc, flat index asc) by
//      counting; the owner of each winner builds its successor record.
//   U. update (every wave, lane j = slot j): prune, recombine.
// A pool overflow (mass ties, or a beam with few live slots) raises the bound
// to the K-th best of the entries that fit and expands again.
//
// Measured against the general decoder, which scored V labels per beam (400
// frames, 1024 tokens; ms a launch): 32 utterances with a 6-gram and 1000
// phrases, 11.3 -> 8.5 at K = 16 and 98 -> 38.6 at K = 128; 64 with a 3-gram
// and 5000 phrases at K = 64, 25.5 -> 13.0.  With 45 tokens, a 3-gram and 50
// phrases (24 utterances of 600 frames, K = 32) 16.8 -> 6.1.  On those inputs a
// frame takes 46 k cycles at K = 16, 74 k at K = 64, 200 k at K = 128 and 25 k
// over 45 tokens (profiling build); at K = 64 the fills take 21 k of it, naming
// classes and rows 15 k, the expansion with its barrier 16 k, the scoring 9 k:
// dependent LDS and memory round trips, not bandwidth.
// Eight waves, two a SIMD, hide those better than four (K = 64: 15.3 against
// 18.4 ms); passes of 16 classes cost fewer phases than passes of 8 (K = 16:
// 9.5 -> 8.9 ms with the arcs dealt out); bounding a class by its best beam
// before a later pass, to skip it, closed too few classes (K = 64: 17.2
// against 13.9 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ctcbeam_internal.h"
#include "ctcbeam_lane.h"

namespace ctcbeam {
namespace classes {

using detail::kNegInf;
using detail::lane_in;
using detail::lse32;
using detail::mix_token;
using detail::no_nan;
using detail::order_key;
using detail::rdlane;
using detail::recomb_shifts;
using detail::wave_incl_scan;
using detail::xor_lane;

// lanes below this one in a wave mask
__device__ __forceinline__ int below(uint64_t m) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                    __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
}
__device__ __forceinline__ int first_of(uint64_t m) { return static_cast<int>(__builtin_ctzll(m)); }
__device__ __forceinline__ uint32_t lane_get(uint32_t v, int l) {
  return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(l << 2, static_cast<int>(v)));
}
__device__ __forceinline__ float lane_get(float v, int l) { return __uint_as_float(lane_get(__float_as_uint(v), l)); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}
// order of LDS accesses between lanes of one wave (LDS operations of a wave
// complete in issue order, so the compiler has to keep it)
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
__device__ __forceinline__ uint32_t row_hash(uint32_t key) { return (key * 0x9E3779B1u) >> 24; }
// wave maximum / minimum (uniform)
__device__ __forceinline__ float wave_max(float v, int lane) {
  v = fmaxf(v, xor_lane(v, 1, lane));
  v = fmaxf(v, xor_lane(v, 2, lane));
  v = fmaxf(v, xor_lane(v, 4, lane));
  v = fmaxf(v, xor_lane(v, 8, lane));
  v = fmaxf(v, xor_lane(v, 16, lane));
  v = fmaxf(v, xor_lane(v, 32, lane));
  return rdlane(v, 0);
}
__device__ __forceinline__ float wave_min(float v, int lane) { return -wave_max(-v, lane); }

// Low word of the order key of a pool entry: the complement of
// slot << 25 | label << 12 | pair id (the slot and the label order ties; the
// pair id, below them, names the entry of the pair table).
constexpr int kSlotShift = 25, kLabelShift = 12;
constexpr uint32_t kLabelMask = 0x1FFFu, kPairMask = 0xFFFu;
constexpr int kOrderShift = 29;  // row entry: context length << 29 | successor state
constexpr uint32_t kStateMask = (1u << kOrderShift) - 1u;
constexpr int kLdsBytes = 160 * 1024;
constexpr int kCT = kClassThreads;
constexpr int kCW = kCT / 64;  // waves of a workgroup
static_assert(kCW == 8, "8 label groups a class, one a wave");

// LPT = labels per lane.  NLEV = levels of the LM's backoff chain above the
// unigrams (-1: no LM).  SPL = beam slots per lane: slot j lives in lane
// j % 64, register set j / 64.
template <int LPT, int NLEV, bool HAS_BT, int SPL>
__global__ void __launch_bounds__(kCT) class_kernel(KernelParams p) {
  constexpr bool HAS_LM = NLEV >= 0;
  constexpr int NL = NLEV > 0 ? NLEV : 0;
  constexpr int NLA = NL > 0 ? NL : 1;
  constexpr bool kRows = HAS_LM || HAS_BT;
  constexpr int KMX = 64 * SPL;
  constexpr int kPool = 256 * SPL;   // pool entries
  constexpr int kHot = 128 * SPL;    // (class, label) pairs a wave collects
  constexpr int kPairs = 16;         // pair table entries of a wave
  // classes a wave scores at once, CG of them with their row loads in flight
  constexpr int NCC = LPT <= 2 ? 16 : 32 / LPT;
  constexpr int kPass = 16;          // classes a pass takes
  static_assert(kHot - kPass > KMX && kPool > KMX, "an overflow leaves more than K candidates");
  constexpr int kFG = NL <= 4 ? 16 : 8;  // new LM rows in the fill's segment table, 64 / kFG lanes each
  constexpr int CG = LPT <= 4 ? 8 / LPT : 1;
  constexpr int RW = 8;
  // beam record of a slot (double-buffered by frame)
  constexpr int kRX = 0, kRHlo = 1, kRHhi = 2, kRLen = 3, kRLast = 4, kRLms = 5, kRBts = 6, kREmit = 7;
  // pair table entry: chain headers of the pair's LM successor, the boosting
  // node's list and pot
  constexpr int PW = 3 * NL + (HAS_BT ? 3 : 0);
  constexpr int kLabels = LPT * kCT;
  constexpr int TU = 6;              // arc tiles of 64 in flight per wave
  constexpr int kBpFrames = SPL == 1 ? 8 : 4;  // frames of back-pointers kept in LDS
  constexpr int kFixed = 1024 + KMX * 10 + kCW * 512 + 128 * 4 + kPool * 16 + kCW * kHot * 4 + 2 * KMX * RW * 4 + kCW * kPairs * (PW > 0 ? PW : 1) * 4 +
                         (kLabels + 64) * 4 + KMX * 8 * 4 + 2 * 64 * 4 + kBpFrames * KMX * 4 + 2048 - KMX * 4;
  // rows of the LM states and boosting nodes; the traceback's tiles after the
  // last frame
  constexpr int kArea = kRows ? ((kLdsBytes - kFixed) & ~255) : 32 * 1024;
  // repeat scoring: the terms of the pool entries and of the slots
  constexpr int kRepBytes = (kPool + 2 * KMX) * 8;

  __shared__ __align__(16) unsigned char s_area[kArea];
  __shared__ uint4 s_pool[kPool];                // order key, LM successor, boosting key
  __shared__ uint32_t s_hot[kCW][kHot];          // a wave's pairs: class | label << 8
  __shared__ __align__(16) uint32_t s_rec[2][KMX * RW];
  __shared__ uint32_t s_pair[kCW * kPairs * (PW > 0 ? PW : 1)];
  __shared__ float s_D[kLabels + 64];            // the frame's row
  __shared__ __align__(16) float s_top[KMX * 8]; // group maxima by class
  __shared__ float s_dm[kCW];                    // the row's maxima by wave
  __shared__ __align__(16) uint32_t s_cht[256];  // lowest slot by hash of its states
  // rows of LM states [0] and boosting nodes [1]: each wave's row by hash of
  // the state; the rows, states and pair ids of a pass's new rows; pots
  __shared__ uint8_t s_rowh[2][kCW][256];
  __shared__ uint32_t s_xrow[2][16], s_xkey[2][16], s_xpid[2][16];
  __shared__ uint32_t s_potB[32];
  // log-sum-exp: order key (score, slot) of a class's best slot where that is
  // not its lowest one, else 0; the lengths and ranks of the final hypotheses after the last frame
  __shared__ unsigned long long s_ctop[KMX];
  __shared__ uint8_t s_cid[KMX], s_cj[KMX];      // class of a leading slot, best slot of a class
  __shared__ uint32_t s_hist[2][64];
  __shared__ int32_t s_bpf[kBpFrames * KMX];
  __shared__ uint64_t s_dup[8][SPL];
  __shared__ uint64_t s_key;
  __shared__ int32_t s_n, s_over, s_best, s_bestlen;
  __shared__ float s_bestscore;
  __shared__ unsigned long long s_st[6];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x;
  const int V = p.V, W = V + 1, K = p.K, T = p.T;
  const float alpha = p.alpha, beta = p.beta, boost_w = p.boost_w;
  const bool rep = kRows && (p.flags & kFlagRepeatScore) != 0;
  const bool lse = (p.flags & kFlagLogSumExp) != 0;
  const bool norows = (p.flags & kFlagNoRowCache) != 0;
  // explicit arcs level by level instead of by the entry's order (state ids
  // that leave no room for it)
  const bool seq = HAS_LM && (norows || p.lm_n_states > static_cast<int64_t>(kStateMask));
  const uint32_t state_mask = seq ? 0xFFFFFFFFu : kStateMask;

  int L = p.lengths[b];
  uint32_t status = 0;
  if (L < 0) { L = 0; status |= 1u; }
  if (L > T) { L = T; status |= 1u; }
  const float* Db = p.logprobs + static_cast<size_t>(b) * T * W;
  int32_t* bpb = p.bp + static_cast<size_t>(b) * T * K;

  // ---- labels of this lane ----
  // Labels run over the workgroup; vocabularies of at most half of it are
  // held by nb waves, and the kCW / nb sets of waves share the classes, so
  // that a character vocabulary does not leave waves idle.
  const int lgnb = LPT > 1 ? 3 : V <= 64 ? 0 : V <= 128 ? 1 : V <= 256 ? 2 : 3;
  const int nb = 1 << lgnb, nsub = kCW >> lgnb;
  const int sub = LPT > 1 ? 0 : wave >> lgnb;
  const int wblk = wave & (nb - 1);
  const int label0 = wblk * 64 + lane;
  // 8 label groups a class, of 8 nb lanes each; the bound uses their maxima
  const auto group_of = [&](int c) __attribute__((always_inline)) {
    const int blk = (c & (kCT - 1)) >> 6;
    return (blk << (3 - lgnb)) + ((c & 63) >> (3 + lgnb));
  };

  // ---- rows ----
  float2* const s_pterm = reinterpret_cast<float2*>(s_area + kArea - kRepBytes);  // rep: terms of the pool entries
  float2* const s_rterm = s_pterm + kPool;                                        // rep: terms of the slots, by frame parity
  const int area = kArea - (rep ? kRepBytes : 0);
  const int VS = (V + 3) & ~3;  // row stride
  int RL = 0, RB = 0;
  {
    if (HAS_LM && HAS_BT) {
      // Boosting rows cost half an LM row, and fewer nodes than states are
      // live: a quarter of the area, three tenths where rows are scarce (2048
      // tokens, 3-gram and 1000 phrases, five rows of each instead of six and
      // three: 1.07x at K = 16, 1.12x at K = 64; but 1024 tokens, K = 16:
      // 0.993x, 930 tokens, 34 phrases, K = 70: 0.98x), and what is left over
      // after the LM rows.
      const int q = area / (4 * VS);     // rows of 4 bytes a label
      RB = max(q >= 4 ? 2 : 1, q >= 24 ? q / 4 : 3 * q / 10);
      RL = min(32, (q - RB) / 2);
      RB = min(32, q - 2 * RL);
    } else if (HAS_LM) {
      RL = min(32, area / (8 * VS));
    } else if (HAS_BT) {
      RB = min(32, area / (4 * VS));
    }
  }
  uint64_t* const lmrow = reinterpret_cast<uint64_t*>(s_area);
  uint32_t* const btrow = reinterpret_cast<uint32_t*>(s_area + (HAS_LM ? 8 * VS * RL : 0));
  const uint32_t rowsL = RL >= 32 ? ~0u : (1u << RL) - 1u;
  const uint32_t rowsB = RB >= 32 ? ~0u : (1u << RB) - 1u;
  uint32_t tagL = 0xFFFFFFFFu, tagB = 0xFFFFFFFFu;  // lane r: the state of row r
  int handL = 0, handB = 0;                         // rows are taken in turn

  float rD[LPT], rDn[LPT];
  uint32_t rcc[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) {
    const int c = label0 + j * kCT;
    const bool ok = c < V;
    rcc[j] = ok ? static_cast<uint32_t>(c) : 0u;
    rDn[j] = ok ? (L > 0 ? Db[c] : 0.0f) : kNegInf;
    rD[j] = kNegInf;
  }
  float rBlankN = L > 0 ? Db[V] : 0.0f;
  float rBlank = 0.0f;

  // ---- beam state: slot lane + 64 h in register set h, in every wave ----
  float sc[SPL], smx[SPL], ral[SPL], rwb[SPL];
  int32_t last[SPL], len[SPL], cls[SPL];
  uint32_t lms[SPL], bts[SPL];
  bool alive[SPL];
#pragma unroll
  for (int h = 0; h < SPL; ++h) {
    alive[h] = h == 0 && lane == 0;
    sc[h] = alive[h] ? 0.0f : kNegInf;
    smx[h] = sc[h];
    ral[h] = rwb[h] = 0.0f;
    last[h] = V;
    len[h] = 0;
    cls[h] = -1;
    // (a unigram LM has one row)
    lms[h] = NL > 0 ? p.lm_bos_state : 0u;
    bts[h] = 0u;
  }
#ifdef CTCBEAM_PHASE_CLOCKS
  const bool want_stats = false;
#else
  const bool want_stats = p.stats != nullptr;
#endif
  // bound of the magnitude of a candidate's added terms (the rounding of two
  // folds of one label differs by at most a few ulps of the partial sums)
  const float term_max = fabsf(beta) + (HAS_LM ? fabsf(alpha) * p.lm_absmax : 0.0f) + (HAS_BT ? 64.0f * fabsf(boost_w) : 0.0f);

  // upper bound of those terms (a boosted token gains at most one unit)
  const float term_most = beta + (HAS_LM ? (alpha >= 0.0f ? alpha * p.lm_max : alpha * p.lm_min) : 0.0f) +
                          (HAS_BT ? (boost_w >= 0.0f ? boost_w : -64.0f * boost_w) : 0.0f);

  int rcur = 0;
  for (int i = tid; i < 2 * kCW * 256; i += kCT) (&s_rowh[0][0][0])[i] = 0;
  if (tid < 64) {
    s_hist[0][lane] = 0u;
    s_hist[1][lane] = 0u;
    *reinterpret_cast<uint4*>(&s_cht[4 * lane]) = make_uint4(~0u, ~0u, ~0u, ~0u);
#pragma unroll
    for (int h = 0; h < SPL; ++h) s_ctop[lane + 64 * h] = 0ull;
  }
  if (tid == 0) {
    uint32_t* r = s_rec[0];
    for (int w = 0; w < RW; ++w) r[w] = 0u;
    r[kRLast] = static_cast<uint32_t>(V) | (kPairMask << 16);  // no pair
    r[kRLms] = lms[0];
    if (rep) s_rterm[0] = make_float2(0.0f, 0.0f);
    s_n = 0;
    s_over = 0;
    if (want_stats) {
      // the initial beam's chain is scanned in frame 0
      unsigned long long ns = 0, na = 0;
      for (int l = 0; l < NL; ++l) {
        const LmLevel hd = p.lm_states[static_cast<size_t>(p.lm_bos_state) * NL + l];
        if (L > 0 && (hd.count & kExists)) {
          ns += 1;
          na += hd.count & ~kExists;
        }
      }
      s_st[0] = L > 0 ? 1 : 0;
      s_st[1] = ns;
      s_st[2] = na;
      s_st[3] = s_st[4] = s_st[5] = 0;
    }
  }
  int hpar = 0;
  __syncthreads();
#ifdef CTCBEAM_PHASE_CLOCKS
  uint64_t ph_acc = 0ull;
  uint64_t ph_t0 = __builtin_amdgcn_s_memtime();
#endif

  for (int t = 0; t < L; ++t) {
    // ---- the frame's row ----
#pragma unroll
    for (int jj = 0; jj < LPT; ++jj) {
      rD[jj] = rDn[jj];
      if (label0 + jj * kCT < V) s_D[label0 + jj * kCT] = rD[jj];
    }
    rBlank = rBlankN;
    if (K > kPass) {
      float m = rD[0];
#pragma unroll
      for (int jj = 1; jj < LPT; ++jj) m = fmaxf(m, rD[jj]);
      m = wave_max(m, lane);
      if (lane == 0) s_dm[wave] = m;
    }
    // The next row is loaded behind the first fill: loads return in order,
    // and the fill waits for its arcs.
    bool ahead = t + 1 < L;
    const auto load_ahead = [&]() __attribute__((always_inline)) {
      const float* rowp = Db + static_cast<size_t>(t + 1) * W;
#pragma unroll
      for (int jj = 0; jj < LPT; ++jj) {
        const int c = label0 + jj * kCT;
        if (c < V) rDn[jj] = __builtin_nontemporal_load(rowp + c);
      }
      rBlankN = __builtin_nontemporal_load(rowp + V);
      ahead = false;
    };
    if (norows) tagL = tagB = 0xFFFFFFFFu;

    // ---- blank candidates and their bound ----
    float xblank[SPL];
    float tb = __builtin_huge_valf();
    int na = 0;
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      na += __popcll(__ballot(alive[h]));
      xblank[h] = no_nan(sc[h] + rBlank);
      if (lane + 64 * h < K) tb = fminf(tb, xblank[h]);
    }
    const bool full = na == K;  // uniform
    tb = full ? wave_min(tb, lane) : kNegInf;
    float tau = -__FLT_MAX__;
    // an overflow's bound: candidates must reach this order key too
    bool kmode = false;
    uint64_t kmin = 0ull;
    int poff = 0;      // pool entries placed without the counter (blanks and repeats)
    int carry = 0;     // pool entries of earlier chunks
    bool first = true; // the frame's first chunk (it adds the blanks and repeats)
    int gbase = 0;     // classes of earlier passes
    int npair = 0;     // pair table entries this wave used
    // The pairs a chunk expanded last (lane i: entry npair + i): the chain
    // headers and the boosting node of the successor, loaded with the
    // expansion and stored when the loads had time to return.
    LmLevel ph[NLA];
    BtNode pn{0u, 0u, 0u, 0u};
    int pend = 0;
    const auto store_pairs = [&]() __attribute__((always_inline)) {
      if (PW > 0 && pend > 0) {  // uniform
        if (lane < pend) {
          uint32_t* h = s_pair + (wave * kPairs + npair + lane) * PW;
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            h[3 * l] = ph[l].begin;
            h[3 * l + 1] = ph[l].count;
            h[3 * l + 2] = __float_as_uint(ph[l].bo);
          }
          if (HAS_BT) {
            h[3 * NL] = pn.list_begin;
            h[3 * NL + 1] = pn.list_count;
            h[3 * NL + 2] = pn.pot & 0xFFu;
          }
        }
        npair += pend;
        pend = 0;
      }
    };
    // ---- P. classes: the live slots by (LM state, boosting node), numbered by
    // their lowest slot.  Every wave enters all slots in the shared table (the
    // entries only fall, so its own operations suffice for its reads); slots
    // whose hash meets another state stand alone. ----
    int CT = 0;
    bool lead[SPL];
    {
      uint32_t hs[SPL];
      int ld[SPL];
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        hs[h] = kRows ? ((lms[h] * 0x9E3779B1u) ^ (bts[h] * 0x85EBCA6Bu)) >> 24 : 0u;
        if (alive[h]) atomicMin(&s_cht[hs[h]], static_cast<uint32_t>(lane + 64 * h));
      }
      wave_lds_fence();
#pragma unroll
      for (int h = 0; h < SPL; ++h) ld[h] = alive[h] ? static_cast<int>(s_cht[hs[h]]) : lane + 64 * h;
      float lx[SPL];
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        const uint32_t* r = s_rec[rcur] + ld[h] * RW;
        lx[h] = __uint_as_float(r[kRX]);
        const bool same = (!HAS_LM || r[kRLms] == lms[h]) && (!HAS_BT || r[kRBts] == bts[h]);
        ld[h] = same ? ld[h] : lane + 64 * h;
        lx[h] = same ? lx[h] : sc[h];
      }
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        lead[h] = alive[h] && ld[h] == lane + 64 * h;
        const uint64_t m = __ballot(lead[h]);
        if (lead[h]) {
          const int id = CT + below(m);
          s_cid[lane + 64 * h] = static_cast<uint8_t>(id);
          if (!lse) s_cj[id] = static_cast<uint8_t>(lane + 64 * h);
        }
        CT += __popcll(m);
      }
      wave_lds_fence();
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        cls[h] = alive[h] ? static_cast<int>(s_cid[ld[h]]) : -1;
        smx[h] = lx[h];
      }
      if (lse) {
        // slots are in score order, unless log-sum-exp merges raised some: a
        // class's best slot is its highest score's lowest slot.  Only slots
        // above their leading slot's score compete (few; one address takes
        // its atomics one after the other)
#pragma unroll
        for (int h = 0; h < SPL; ++h)
          if (alive[h] && sc[h] > lx[h])
            atomicMax(&s_ctop[cls[h]], static_cast<unsigned long long>(order_key(sc[h], static_cast<uint32_t>(lane + 64 * h))));
        wave_lds_fence();
#pragma unroll
        for (int h = 0; h < SPL; ++h) {
          const uint64_t top = alive[h] ? s_ctop[cls[h]] : 0ull;  // 0: the leading slot
          const uint32_t u = static_cast<uint32_t>(top >> 32);
          smx[h] = top != 0ull ? __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u) : lx[h];
          if (top != 0ull ? ~static_cast<uint32_t>(top) == static_cast<uint32_t>(lane + 64 * h) : lead[h])
            s_cj[cls[h]] = static_cast<uint8_t>(lane + 64 * h);
        }
        wave_lds_fence();
      }
    }
    // the rows of live states
    const auto live_rows = [&](int kind, const uint32_t (&key)[SPL], uint32_t tag) __attribute__((always_inline)) {
      uint32_t m = 0u;
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        const int q = s_rowh[kind][wave][row_hash(key[h])];
        const uint32_t tq = lane_get(tag, q);
        m |= (alive[h] && tq == key[h]) ? 1u << q : 0u;
      }
      m |= xor_lane(m, 1, lane);
      m |= xor_lane(m, 2, lane);
      m |= xor_lane(m, 4, lane);
      if (K > 8) m |= xor_lane(m, 8, lane);
      if (K > 16) m |= xor_lane(m, 16, lane);
      if (K > 32) m |= xor_lane(m, 32, lane);
      return rdlane(m, 0);
    };
    uint32_t liveL = 0u, liveB = 0u;
    if (HAS_LM) liveL = live_rows(0, lms, tagL);
    if (HAS_BT) liveB = live_rows(1, bts, tagB);

    // Passes of up to kPass classes, as far as their rows fit.  After the
    // first pass the classes that cannot reach the bound any more are left
    // out: they are the last ones.
    for (;;) {
      if (!first && !lse && K > kPass && gbase < CT) {
        // no emission of a slot exceeds its score + the row's maximum + beta
        // + the largest LM term + one boosted token
        float dm = s_dm[lane & (kCW - 1)];
        dm = fmaxf(dm, xor_lane(dm, 1, lane));
        dm = fmaxf(dm, xor_lane(dm, 2, lane));
        dm = fmaxf(dm, xor_lane(dm, 4, lane));
        int keep = 0;
#pragma unroll
        for (int h = 0; h < SPL; ++h) {
          const float most = (sc[h] + (dm + term_most)) + 2e-6f * (fabsf(sc[h]) + fabsf(dm) + term_max);
          // (a class's lowest slot is its best, and the slots are in order)
          keep += __popcll(__ballot(lead[h] && !(most < tau)));
        }
        CT = min(CT, max(keep, gbase));
      }
      if (gbase >= CT) break;  // uniform
      int nfl = 0, nfb = 0;         // rows to fill
      uint32_t fl = 0u, fb = 0u;    // lane f: pair id | row << 16
      uint32_t flk = 0u, fbk = 0u;  // lane f: LM state / boosting node
      int C = min(CT - gbase, kPass);
      // lane i < C: class gbase + i; its best slot, rows and highest score
      const int cJ = s_cj[gbase + min(lane, C - 1)];
      uint32_t cP = 0u;   // LM row | boosting row << 8
      float cS;
      {
        const uint32_t* r = s_rec[rcur] + cJ * RW;
        const uint32_t k1 = r[kRLms], k2 = r[kRBts], pd = r[kRLast] >> 16;
        if (SPL == 1 || CT <= 64) {
          cS = lane_get(smx[0], cJ & 63);
          if (SPL > 1) {
            const float up = lane_get(smx[SPL - 1], cJ & 63);
            cS = cJ >= 64 ? up : cS;
          }
        } else {
          const float lo = lane_get(smx[0], cJ & 63), up = lane_get(smx[SPL - 1], cJ & 63);
          cS = cJ >= 64 ? up : lo;
        }
        // Rows of the pass's classes (kind 0: LM states, 1: boosting nodes):
        // the row in place, or for each other state, in class order, a row
        // that no class of the pass uses, rather one of no live state, in
        // turn.  Straight-line code over the lanes: class lanes, row lanes and
        // filler lanes exchange through LDS (a loop over the new states took
        // 500 cycles a state).  Every wave computes the same.
        const auto place = [&](int kind, uint32_t key, uint32_t& tag, uint32_t rows, uint32_t& live, int& hand, int& nf,
                               uint32_t& f, uint32_t& fk) __attribute__((always_inline)) {
          uint8_t* const tbl = s_rowh[kind][wave];
          int q = tbl[row_hash(key)];
          const uint32_t tq = lane_get(tag, q);
          const bool hit = lane < C && tq == key;
          uint32_t used = hit ? 1u << q : 0u;
          used |= xor_lane(used, 1, lane);
          used |= xor_lane(used, 2, lane);
          used |= xor_lane(used, 4, lane);
          used |= xor_lane(used, 8, lane);
          used = rdlane(used, 0);
          bool miss = lane < C && !hit;
          const uint64_t mm = __ballot(miss);
          if (mm != 0ull) {  // uniform
            uint32_t fr = rows & ~used;
            if (fr == 0u && (mm & 1ull) != 0ull) {
              // the first class of a pass takes a row in any case
              C = 1;
              fr = rows;
              miss = lane == 0;
            }
            // the first class of each new state, and its number
            int fi = lane;
            const uint32_t kk = miss ? key : 0xFFFFFFFFu;
            const auto probe = [&](uint32_t o, int d) __attribute__((always_inline)) { fi = o == kk ? lane - d : fi; };
            probe(detail::dpp_shr_ones<1>(kk), 1);
            probe(detail::dpp_shr_ones<2>(kk), 2);
            probe(detail::dpp_shr_ones<3>(kk), 3);
            probe(detail::dpp_shr_ones<4>(kk), 4);
            probe(detail::dpp_shr_ones<5>(kk), 5);
            probe(detail::dpp_shr_ones<6>(kk), 6);
            probe(detail::dpp_shr_ones<7>(kk), 7);
            probe(detail::dpp_shr_ones<8>(kk), 8);
            probe(detail::dpp_shr_ones<9>(kk), 9);
            probe(detail::dpp_shr_ones<10>(kk), 10);
            probe(detail::dpp_shr_ones<11>(kk), 11);
            probe(detail::dpp_shr_ones<12>(kk), 12);
            probe(detail::dpp_shr_ones<13>(kk), 13);
            probe(detail::dpp_shr_ones<14>(kk), 14);
            probe(detail::dpp_shr_ones<15>(kk), 15);
            const bool firstof = miss && fi == lane;
            const uint64_t fm = __ballot(firstof);
            const int n = below(fm);
            const int F = __popc(fr);
            const uint64_t over = __ballot(firstof && n >= F);
            if (over != 0ull) C = first_of(over);  // the pass ends before this class
            const int M = min(__popcll(fm), F);
            // the free rows in order
            const uint32_t p0 = fr & ~live, p1 = fr & live, hi = ~0u << hand;
            const int r0 = lane >= hand ? __builtin_amdgcn_mbcnt_lo(p0 & hi, 0u)
                                        : __popc(p0 & hi) + __builtin_amdgcn_mbcnt_lo(p0 & ~hi, 0u);
            const int at = ((p0 >> (lane & 31)) & 1u) ? r0 : __popc(p0) + static_cast<int>(__builtin_amdgcn_mbcnt_lo(p1, 0u));
            const bool taken = lane < 32 && ((fr >> (lane & 31)) & 1u) != 0u && at < M;
            if (taken) s_xrow[kind][at & 15] = static_cast<uint32_t>(lane);
            if (firstof && n < M) {
              s_xkey[kind][n & 15] = key;
              s_xpid[kind][n & 15] = pd;
            }
            live |= static_cast<uint32_t>(__ballot(taken));
            wave_lds_fence();
            const uint32_t nk = s_xkey[kind][at & 15];
            tag = taken ? nk : tag;
            const uint32_t nfi = lane_get(static_cast<uint32_t>(n), fi);
            const uint32_t rq = s_xrow[kind][nfi & 15u];
            q = miss ? static_cast<int>(rq) : q;
            const uint32_t fr_row = s_xrow[kind][lane & 15], fr_key = s_xkey[kind][lane & 15], fr_pid = s_xpid[kind][lane & 15];
            f = fr_pid | (fr_row << 16);
            fk = fr_key;
            // one at a time: two states of one hash must leave the same row in
            // every wave's table
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              if (i >= M) break;  // uniform
              if (lane == i) tbl[row_hash(fr_key)] = static_cast<uint8_t>(fr_row);
              wave_lds_fence();
            }
            // (no row is free where the first class has one and fills the area)
            if (M > 0) hand = static_cast<int>(rdlane(fr_row, M - 1) + 1u) & 31;
            nf = M;
          }
          return static_cast<uint32_t>(q);
        };
        if constexpr (HAS_LM) cP = place(0, k1, tagL, rowsL, liveL, handL, nfl, fl, flk);
        if constexpr (HAS_BT) cP |= place(1, k2, tagB, rowsB, liveB, handB, nfb, fb, fbk) << 8;
      }
      CTCBEAM_PHASE_ADD(16, nfl);  // rows filled
      CTCBEAM_PHASE_ADD(18, nfb);
      CTCBEAM_PHASE_ADD(12, C);  // classes
      CTCBEAM_PHASE_MARK(13);

      // ---- F. fill the new rows ----
      if (kRows && nfl + nfb > 0) {  // uniform
        // Segment table of kFG LM rows, lane f * (64 / kFG) + l: the explicit
        // arcs of level l of new row f's chain, and the backoff weights of the
        // longer contexts (zeros past the last level).
        constexpr int kSL = 64 / kFG;  // lanes a row
        uint32_t sg_begin = 0u, sg_cnt = 0u, sg_row = 0u;
        float sg_bo = 0.0f, sg_f[NLA];
        int tincl = 0, texcl = 0, ntile = 0;
        const auto segments = [&](int g) __attribute__((always_inline)) {
          const int f = g * kFG + lane / kSL, l = lane % kSL;
          const uint32_t info = lane_get(fl, f & 63);
          const uint32_t sk = lane_get(flk, f & 63);
          const bool ok = f < nfl && l < NL;
          const uint32_t pd = info & 0xFFFFu;
          sg_row = info >> 16;
          sg_begin = sg_cnt = 0u;
          sg_bo = 0.0f;
          if (ok && first && pd != kPairMask) {  // (later passes may overwrite the pair table)
            const uint32_t* h = s_pair + pd * PW + 3 * l;
            sg_begin = h[0];
            sg_cnt = h[1] & ~kExists;
            sg_bo = __uint_as_float(h[2]);
          } else if (ok) {
            const LmLevel hd = p.lm_states[static_cast<size_t>(sk) * NL + l];
            sg_begin = hd.begin;
            sg_cnt = hd.count & ~kExists;
            sg_bo = hd.bo;
          }
          const int nt = static_cast<int>((sg_cnt + 63u) >> 6);
          tincl = wave_incl_scan(nt, lane);
          texcl = tincl - nt;
          ntile = rdlane(tincl, 63);
#pragma unroll
          for (int k = 0; k + 1 < NL; ++k) {
            const float o = lane_get(sg_bo, (lane + k + 1) & 63);
            sg_f[k] = l + k + 1 < NL ? o : 0.0f;
          }
        };
        LmArc a[TU];
        int asg[TU];
        const auto load_tiles = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
          for (int u = 0; u < TU; ++u) {
            const int tt = t0 + u * kCW;
            a[u].token = 0xFFFFFFFFu;
            asg[u] = 0;
            if (tt < ntile) {  // uniform
              const int sg = __popcll(__ballot(tincl <= tt));
              const uint32_t qs = (static_cast<uint32_t>(tt - rdlane(texcl, sg)) << 6) + static_cast<uint32_t>(lane);
              const bool ok = qs < rdlane(sg_cnt, sg);
              const LmArc x = p.lm_arcs[rdlane(sg_begin, sg) + (ok ? qs : 0u)];
              a[u].logp = x.logp;
              a[u].target = x.target;
              a[u].token = ok ? x.token : 0xFFFFFFFFu;
              asg[u] = sg;
            }
          }
        };
        const auto store_tiles = [&](int t0, int level) __attribute__((always_inline)) {
#pragma unroll
          for (int u = 0; u < TU; ++u) {
            const int l = asg[u] % kSL;
            if (t0 + u * kCW < ntile && (level < 0 || l == level)) {  // uniform
              // the backoff weights of the longer contexts, which lack this
              // token, in ascending order
              float v = a[u].logp;
#pragma unroll
              for (int k = 0; k + 1 < NL; ++k) v = v + rdlane(sg_f[k], asg[u]);
              const float av = alpha * v;
              uint64_t* const row = lmrow + rdlane(sg_row, asg[u]) * static_cast<uint32_t>(VS);
              if (a[u].token < static_cast<uint32_t>(V)) {
                uint64_t* e = row + a[u].token;
                if (seq) {
                  *e = (static_cast<uint64_t>(a[u].target) << 32) | __float_as_uint(av);
                } else {
                  const uint32_t hi = (static_cast<uint32_t>(l + 1) << kOrderShift) | a[u].target;
                  atomicMax(reinterpret_cast<unsigned long long*>(e),
                            (static_cast<unsigned long long>(hi) << 32) | __float_as_uint(av));
                }
              }
            }
          }
        };
        const int ngrp = (nfl + kFG - 1) / kFG;
        if (NL > 0 && nfl > 0) {
          segments(0);
          load_tiles(wave);
        }
        // one wave a row: the unigram + backoff fold of every label, or the
        // root keys of a boosting row and its node's list over them
        for (int jb = wave; jb < nfl + nfb; jb += kCW) {  // uniform per wave
          if (HAS_LM && jb < nfl) {
            const uint32_t info = rdlane(fl, jb);
            uint64_t* const row = lmrow + (info >> 16) * static_cast<uint32_t>(VS);
            float bo[NLA];
            if (jb < kFG) {
#pragma unroll
              for (int l = 0; l < NL; ++l) bo[l] = rdlane(sg_bo, jb * kSL + l);
            } else {
              // (past the first group of the segment table)
              const uint32_t pd = info & 0xFFFFu, sk = rdlane(flk, jb);
#pragma unroll
              for (int l = 0; l < NL; ++l)
                bo[l] = (first && pd != kPairMask) ? __uint_as_float(uniform(s_pair[pd * PW + 3 * l + 2]))
                                                   : __uint_as_float(uniform(__float_as_uint(p.lm_states[static_cast<size_t>(sk) * NL + l].bo)));
            }
            for (int c0 = 0; c0 < V; c0 += 1024) {
              float4 u4[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int c = c0 + 256 * i + 4 * lane;
                u4[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                // (the array holds V + 1 values)
                if (c + 3 <= V) u4[i] = *reinterpret_cast<const float4*>(p.lm_unigram + c);
                else if (c < V) u4[i] = make_float4(p.lm_unigram[c], c + 1 < V ? p.lm_unigram[c + 1] : 0.0f, c + 2 < V ? p.lm_unigram[c + 2] : 0.0f, 0.0f);
              }
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int c = c0 + 256 * i + 4 * lane;
                const auto fold = [&](float v) __attribute__((always_inline)) {
#pragma unroll
                  for (int l = 0; l < NL; ++l) v = v + bo[l];
                  const float av = alpha * v;
                  return __float_as_uint(av);
                };
                if (c < V) {  // (the row's stride is padded to 4)
                  uint4* e = reinterpret_cast<uint4*>(row + c);
                  const uint32_t uc = static_cast<uint32_t>(c);
                  e[0] = make_uint4(fold(u4[i].x), uc, fold(u4[i].y), uc + 1u);
                  e[1] = make_uint4(fold(u4[i].z), uc + 2u, fold(u4[i].w), uc + 3u);
                }
              }
            }
          }
          if (HAS_BT && jb >= nfl) {
            const int j = jb - nfl;
            const uint32_t info = rdlane(fb, j), nk = rdlane(fbk, j);
            const uint32_t r = info >> 16;
            uint32_t* const row = btrow + r * static_cast<uint32_t>(VS);
            const uint32_t pd = info & 0xFFFFu;
            uint32_t base, cnt, pot;
            if (first && pd != kPairMask) {
              const uint32_t hv = s_pair[pd * PW + (lane < PW ? lane : 0)];
              base = rdlane(hv, 3 * NL);
              cnt = rdlane(hv, 3 * NL + 1);
              pot = rdlane(hv, 3 * NL + 2);
            } else {
              const BtNode nd = p.bt_nodes[nk];
              base = uniform(nd.list_begin);
              cnt = uniform(nd.list_count);
              pot = uniform(nd.pot) & 0xFFu;
            }
            if (lane == 0) s_potB[r] = pot;
            BtEntry be{0xFFFFFFFFu, 0u};
            if (static_cast<uint32_t>(lane) < cnt) be = p.bt_list[base + static_cast<uint32_t>(lane)];
            for (int c = 4 * lane; c < V; c += 256) {
              uint4 k4 = make_uint4(0u, 0u, 0u, 0u);
              if (c + 3 < V) k4 = *reinterpret_cast<const uint4*>(p.bt_root_key + c);
              else k4 = make_uint4(p.bt_root_key[c], c + 1 < V ? p.bt_root_key[c + 1] : 0u, c + 2 < V ? p.bt_root_key[c + 2] : 0u, 0u);
              *reinterpret_cast<uint4*>(row + c) = k4;
            }
            // (the stores of one wave keep their order)
            wave_lds_fence();
            for (uint32_t q0 = 0u; q0 < cnt; q0 += 64u) {
              const uint32_t q = q0 + static_cast<uint32_t>(lane);
              if (q0 > 0u && q < cnt) be = p.bt_list[base + q];
              if (q < cnt && be.token < static_cast<uint32_t>(V)) row[be.token] = be.key;
            }
          }
        }
        if constexpr (NL > 0) {
          if (nfl > 0) {  // uniform
            __syncthreads();  // folds in place
            for (int g = 0; g < ngrp; ++g) {
              const bool kept = ngrp == 1;  // the table and first tiles are in registers
              if (!kept) segments(g);
              if (!seq) {
                for (int t0 = wave; t0 < ntile; t0 += kCW * TU) {
                  if (!kept || t0 != wave) load_tiles(t0);
                  store_tiles(t0, -1);
                }
              } else {
                for (int l = 0; l < NL; ++l) {
                  for (int t0 = wave; t0 < ntile; t0 += kCW * TU) {
                    load_tiles(t0);
                    store_tiles(t0, l);
                  }
                  __syncthreads();
                }
              }
            }
          }
        }
        CTCBEAM_PHASE_MARK(0);
        __syncthreads();  // rows complete
        CTCBEAM_PHASE_MARK(1);
      }
      if (ahead) load_ahead();
      // lane i: LM row | boosting row << 8 | pot << 16
      uint32_t cR = cP;
      if (HAS_BT) cR = (cP & 0xFFFFu) | (s_potB[(cP >> 8) & 31u] << 16);

      for (int c0 = 0; c0 < C; c0 += NCC * nsub) {
        const int nq = min(C - c0, NCC * nsub);
        // ---- C. scoring: class c0 + sub + r * nsub in registers r ----
        float rm[NCC];  // the class's maximum over this lane's labels
        float lmax = kNegInf;
#pragma unroll
        for (int r0 = 0; r0 < NCC; r0 += CG) {
          if (sub + r0 * nsub < nq) {  // uniform
            uint64_t ent[CG][LPT];
            uint32_t key[CG][LPT];
            float sm[CG];
            int po[CG];
#pragma unroll
            for (int i = 0; i < CG; ++i) {
              const int ci = c0 + min(sub + (r0 + i) * nsub, nq - 1);
              sm[i] = rdlane(cS, ci);
              const uint32_t cr = rdlane(cR, ci);
              po[i] = static_cast<int>(cr >> 16);
#pragma unroll
              for (int jj = 0; jj < LPT; ++jj) {
                if (HAS_LM) ent[i][jj] = lmrow[(cr & 0xFFu) * static_cast<uint32_t>(VS) + rcc[jj]];
                if (HAS_BT) key[i][jj] = btrow[((cr >> 8) & 0xFFu) * static_cast<uint32_t>(VS) + rcc[jj]];
              }
            }
#pragma unroll
            for (int i = 0; i < CG; ++i) {
              const bool have = sub + (r0 + i) * nsub < nq;  // uniform
#pragma unroll
              for (int jj = 0; jj < LPT; ++jj) {
                float x = sm[i] + rD[jj];
                x = x + beta;
                if (HAS_LM) x = x + __uint_as_float(static_cast<uint32_t>(ent[i][jj]));
                if (HAS_BT) x = x + boost_w * static_cast<float>(static_cast<int>((key[i][jj] >> 20) & 63u) - po[i]);
                if (i > 0) x = have ? x : kNegInf;
                rm[r0 + i] = jj == 0 ? x : fmaxf(rm[r0 + i], x);
              }
              lmax = fmaxf(lmax, rm[r0 + i]);
            }
          } else {
#pragma unroll
            for (int i = 0; i < CG; ++i) rm[r0 + i] = kNegInf;
          }
        }
        // Maxima of the label groups, 8 classes at a time: a transposed
        // reduction halves the classes a lane carries at each of the lane-bit
        // steps 1, 2, 4, leaving lane l with class 4(l&1) + 2(l>>1&1) +
        // (l>>2&1), then reduces over the group's other lane bits.
#pragma unroll
        for (int s8 = 0; s8 < NCC; s8 += 8) {
          if (sub + s8 * nsub < nq) {  // uniform
            float m8[8], m4[4], m2[2];
#pragma unroll
            for (int i = 0; i < 8; ++i) m8[i] = s8 + i < NCC ? rm[s8 + i < NCC ? s8 + i : 0] : kNegInf;
            const bool b0 = lane_in(0xAAAAAAAAAAAAAAAAull), b1 = lane_in(0xCCCCCCCCCCCCCCCCull),
                       b2 = lane_in(detail::kLanesBit2);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              m4[q] = fmaxf(b0 ? m8[q + 4] : m8[q], xor_lane(b0 ? m8[q] : m8[q + 4], 1, lane));
#pragma unroll
            for (int q = 0; q < 2; ++q)
              m2[q] = fmaxf(b1 ? m4[q + 2] : m4[q], xor_lane(b1 ? m4[q] : m4[q + 2], 2, lane));
            float m1 = fmaxf(b2 ? m2[1] : m2[0], xor_lane(b2 ? m2[0] : m2[1], 4, lane));
            if (lgnb >= 1) m1 = fmaxf(m1, xor_lane(m1, 8, lane));
            if (lgnb >= 2) m1 = fmaxf(m1, xor_lane(m1, 16, lane));
            if (lgnb >= 3) m1 = fmaxf(m1, xor_lane(m1, 32, lane));
            const int r = s8 + ((lane & 1) << 2) + (lane & 2) + ((lane >> 2) & 1);
            const int q = sub + r * nsub;
            if ((lane & ((8 << lgnb) - 1)) < 8 && q < nq)
              s_top[(gbase + c0 + q) * 8 + (wblk << (3 - lgnb)) + (lane >> (3 + lgnb))] = m1;
          }
        }
        CTCBEAM_PHASE_MARK(2);
        __syncthreads();  // B: group maxima, the row in s_D
        CTCBEAM_PHASE_MARK(3);

        // ---- T. bound ----
        const int gdone = gbase + c0 + nq;  // classes scored so far
        float xrep[SPL];                    // repeat candidates
#pragma unroll
        for (int h = 0; h < SPL; ++h) {
          xrep[h] = kNegInf;
          if (alive[h] && last[h] != V) {
            float x = sc[h] + s_D[last[h]];
            if (rep) {
              if (HAS_LM) x = x + ral[h];
              if (HAS_BT) x = x + rwb[h];
            }
            xrep[h] = x;
          }
        }
        // a beam's candidate at its class's maximum m of a group, bounded
        // from below (d: distance of the beam's score from its class's best)
        const auto lower = [&](float m, float d) __attribute__((always_inline)) {
          return (m - d) - 2e-6f * (fabsf(m) + d + term_max);
        };
        if (K <= 8) {
          // lane 8 g + k: slot k, group g.  Two sets of distinct candidates,
          // one in each row of 16 lanes: the (slot, half of the groups)
          // maxima; the 8 group maxima and the repeat candidates.
          const int k = lane & 7, g = lane >> 3;
          const int lg0 = last[0] == V ? 15 : group_of(last[0]);
          const uint32_t pk = lane_get((cls[0] >= 0 && cls[0] < gdone ? static_cast<uint32_t>(cls[0]) : 0xFFu) |
                                           (static_cast<uint32_t>(lg0) << 8), k);
          const float dk = lane_get(smx[0] - sc[0], k);
          const float rpv = lane_get(xrep[0], k);
          const bool ok = (pk & 0xFFu) != 0xFFu && static_cast<int>(pk >> 8) != g;
          const float mk = s_top[(ok ? (pk & 0xFFu) : 0u) * 8 + g];
          const float v = ok ? lower(mk, dk) : kNegInf;
          float hm = fmaxf(v, xor_lane(v, 8, lane));
          hm = fmaxf(hm, xor_lane(hm, 16, lane));  // lanes 0..31: groups 0..3, lanes 32..63: 4..7
          const float oh = xor_lane(hm, 32, lane);
          float gm = fmaxf(v, xor_lane(v, 1, lane));
          gm = fmaxf(gm, xor_lane(gm, 2, lane));
          gm = fmaxf(gm, xor_lane(gm, 4, lane));
          const float gmv = lane_get(gm, (lane & 7) * 8);
          float u = kNegInf;
          u = lane_in(0xFFull) ? hm : u;
          u = lane_in(0xFF00ull) ? oh : u;
          u = lane_in(0xFF0000ull) ? gmv : u;
          u = lane_in(0xFF000000ull) ? rpv : u;
          const float kv = detail::row_max_last(detail::row_ge_count(u) >= static_cast<uint32_t>(K) ? u : kNegInf);
          tau = fmaxf(tau, fmaxf(fmaxf(rdlane(kv, 15), rdlane(kv, 31)), tb));
        } else {
          // histogram of the candidates' distances from the best, 64 bins
          // down to the bound of the blanks (at most 32; 24 with dead slots)
          float best = kNegInf;
          for (int i = lane; i < gdone * 8; i += 64) best = fmaxf(best, s_top[i]);
          best = wave_max(best, lane);
          // (a best of +inf gives no range)
          const float R = !(best < __builtin_huge_valf()) ? 0.0f : full ? fminf(best - tb, 32.0f) : 24.0f;
          const float lo = best - R;
          const float scale = 64.0f / R;
          const auto add = [&](float v) __attribute__((always_inline)) {
            // (a NaN or an empty range adds nothing)
            if (v >= lo && R > 0.0f) atomicAdd(&s_hist[hpar][min(63, max(0, static_cast<int>((best - v) * scale)))], 1u);
          };
          if (wave == kCW - 1) s_hist[hpar ^ 1][lane] = 0u;
#pragma unroll
          for (int h = 0; h < SPL; ++h) {
            const bool in = cls[h] >= 0 && cls[h] < gdone;
            const int lg0 = last[h] == V ? -1 : group_of(last[h]);
            const float d = smx[h] - sc[h];
            const float m = s_top[(in ? cls[h] : 0) * 8 + wave];
            if (in && wave != lg0) add(lower(m, d));
            if (wave == 0 && alive[h]) add(xblank[h]);
            if (wave == 1) add(xrep[h]);
          }
          __syncthreads();  // H: histogram complete
          const int incl = wave_incl_scan(static_cast<int>(s_hist[hpar][lane]), lane);
          hpar ^= 1;
          const uint64_t m = __ballot(incl >= K);
          if (m != 0ull) {
            const float t1 = best - static_cast<float>(first_of(m) + 1) * (R * (1.0f / 64.0f));
            tau = fmaxf(tau, t1 - 4e-6f * (fabsf(best) + R));
          }
          tau = fmaxf(tau, tb);
        }
        // an infinite bound admits every finite candidate and no -inf one
        tau = fmaxf(tau, -__FLT_MAX__);
        CTCBEAM_PHASE_MARK(14);

        // ---- E. expansion into the pool ----
        store_pairs();  // the chunk's before
        for (;;) {
          if (first) {
            // blanks and repeats: every wave knows their places
            int at[2][SPL];
            bool in[2][SPL];
            int n = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
              for (int h = 0; h < SPL; ++h) {
                const float x = q == 0 ? xblank[h] : xrep[h];
                in[q][h] = alive[h] && x >= tau;
                if (kmode) {
                  const uint32_t c = static_cast<uint32_t>(q == 0 ? V : last[h]);
                  in[q][h] = in[q][h] && order_key(x, (static_cast<uint32_t>(lane + 64 * h) << kSlotShift) | (c << kLabelShift) | kPairMask) >= kmin;
                }
                const uint64_t m = __ballot(in[q][h]);
                at[q][h] = n + below(m);
                n += __popcll(m);
              }
            }
            poff = n;  // at most 2 K <= kPool
            if (wave < 2) {
#pragma unroll
              for (int h = 0; h < SPL; ++h) {
                const float x = wave == 0 ? xblank[h] : xrep[h];
                const uint32_t c = static_cast<uint32_t>(wave == 0 ? V : last[h]);
                if (wave == 0 ? in[0][h] : in[1][h]) {
                  const uint64_t key = order_key(x, (static_cast<uint32_t>(lane + 64 * h) << kSlotShift) | (c << kLabelShift) | kPairMask);
                  s_pool[wave == 0 ? at[0][h] : at[1][h]] = make_uint4(static_cast<uint32_t>(key), static_cast<uint32_t>(key >> 32), 0u, 0u);
                }
              }
            }
          }
          if (__ballot(lmax >= tau) != 0ull) {  // uniform: many waves hold no pair
            int nh = 0;
#pragma unroll
            for (int r = 0; r < NCC; ++r) {
              const int q = sub + r * nsub;
              if (__ballot(rm[r] >= tau) != 0ull) {  // uniform; few classes: their labels are scored again
                const float sm = rdlane(cS, c0 + q);
                const uint32_t cr = rdlane(cR, c0 + q);
#pragma unroll
                for (int jj = 0; jj < LPT; ++jj) {
                  float x = sm + rD[jj];
                  x = x + beta;
                  if (HAS_LM) x = x + __uint_as_float(static_cast<uint32_t>(lmrow[(cr & 0xFFu) * static_cast<uint32_t>(VS) + rcc[jj]]));
                  if (HAS_BT) {
                    const uint32_t key = btrow[((cr >> 8) & 0xFFu) * static_cast<uint32_t>(VS) + rcc[jj]];
                    x = x + boost_w * static_cast<float>(static_cast<int>((key >> 20) & 63u) - static_cast<int>(cr >> 16));
                  }
                  bool hot = x >= tau;
                  if (kmode) {
                    // the key of the best slot's candidate: every pair that
                    // passes has one, but for that slot's repeat
                    const uint32_t bs = static_cast<uint32_t>(rdlane(cJ, c0 + q));
                    hot = hot && order_key(x, (bs << kSlotShift) | (rcc[jj] << kLabelShift)) >= kmin;
                  }
                  const uint64_t m = __ballot(hot);
                  const int at = nh + below(m);
                  if (hot && at < kHot) s_hot[wave][at] = static_cast<uint32_t>(c0 + q) | (rcc[jj] << 8);
                  nh += __popcll(m);
                }
              }
            }
            if (nh > kHot) {
              if (lane == 0) s_over = 1;
              nh = kHot;
            }
            wave_lds_fence();
            CTCBEAM_PHASE_ADD(19, nh);  // pairs expanded
            for (int h0 = 0; h0 < nh; h0 += 64) {
              // lane i: pair h0 + i
              const int n = min(64, nh - h0);
              const uint32_t e = s_hot[wave][lane < n ? h0 + lane : h0];
              const uint32_t ci = e & 0xFFu, c = e >> 8;
              const uint32_t cr = lane_get(cR, static_cast<int>(ci));
              const float d = s_D[c];
              float av = 0.0f, bv = 0.0f;
              uint32_t tg = 0u, bk = 0u;
              if (HAS_LM) {
                const uint64_t en = lmrow[(cr & 0xFFu) * static_cast<uint32_t>(VS) + c];
                av = __uint_as_float(static_cast<uint32_t>(en));
                tg = static_cast<uint32_t>(en >> 32) & state_mask;
              }
              if (HAS_BT) {
                bk = btrow[((cr >> 8) & 0xFFu) * static_cast<uint32_t>(VS) + c];
                bv = boost_w * static_cast<float>(static_cast<int>((bk >> 20) & 63u) - static_cast<int>(cr >> 16));
              }
              const int np = (PW > 0 && h0 == 0) ? min(n, kPairs - npair) : 0;  // uniform
              if (np > 0 && lane < np) {
#pragma unroll
                for (int l = 0; l < NL; ++l) ph[l] = p.lm_states[static_cast<size_t>(tg) * NL + l];
                if (HAS_BT) pn = p.bt_nodes[bk & kBtChildMask];
              }
              if (h0 == 0) pend = np;  // (the chunk's first 64 pairs)
              const uint32_t pidv = lane < np ? static_cast<uint32_t>(wave * kPairs + npair + lane) : kPairMask;
              for (int u0 = 0; u0 < n; u0 += 4) {
                // four pairs at a time, one counter round trip
                float x[4][SPL];
                uint64_t m[4][SPL];
                int total = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const int u = u0 + i;
#pragma unroll
                  for (int h = 0; h < SPL; ++h) {
                    m[i][h] = 0ull;
                    x[i][h] = 0.0f;
                  }
                  if (u < n) {  // uniform
                    const int gc = gbase + static_cast<int>(rdlane(ci, u));
                    const uint32_t cu = rdlane(c, u);
                    const float du = rdlane(d, u), au = rdlane(av, u), bu = rdlane(bv, u);
#pragma unroll
                    for (int h = 0; h < SPL; ++h) {
                      float y = sc[h] + du;
                      y = y + beta;
                      if (HAS_LM) y = y + au;
                      if (HAS_BT) y = y + bu;
                      x[i][h] = y;
                      bool keep = cls[h] == gc && static_cast<uint32_t>(last[h]) != cu && y >= tau;
                      if (kmode)
                        keep = keep && order_key(y, (static_cast<uint32_t>(lane + 64 * h) << kSlotShift) | (cu << kLabelShift)) >= kmin;
                      m[i][h] = __ballot(keep);
                      total += __popcll(m[i][h]);
                    }
                  }
                }
                if (total > 0) {  // uniform
                  int base = 0;
                  if (lane == 0) base = atomicAdd(&s_n, total);
                  base = __builtin_amdgcn_readfirstlane(base) + poff;
                  if (base + total > kPool && lane == 0) s_over = 1;
#pragma unroll
                  for (int i = 0; i < 4; ++i) {
                    const int u = u0 + i;
                    if (u < n) {  // uniform
                      const uint32_t cu = rdlane(c, u), tu = rdlane(tg, u), ku = rdlane(bk, u), pu = rdlane(pidv, u);
                      const float au = rdlane(av, u), bu = rdlane(bv, u);
#pragma unroll
                      for (int h = 0; h < SPL; ++h) {
                        const int at = base + below(m[i][h]);
                        if (((m[i][h] >> lane) & 1ull) != 0ull && at < kPool) {
                          const uint64_t key = order_key(x[i][h], (static_cast<uint32_t>(lane + 64 * h) << kSlotShift) | (cu << kLabelShift) | pu);
                          s_pool[at] = make_uint4(static_cast<uint32_t>(key), static_cast<uint32_t>(key >> 32), tu, ku);
                          if (rep) s_pterm[at] = make_float2(au, bu);
                        }
                        base += __popcll(m[i][h]);
                      }
                    }
                  }
                }
              }
            }
          }
          CTCBEAM_PHASE_MARK(4);
          __syncthreads();  // C: pool complete
          CTCBEAM_PHASE_MARK(5);
          if (s_over == 0) break;  // uniform
          // Overflow: the K-th best of the entries that fit bounds the K-th
          // best candidate; keep what reaches it and expand this chunk
          // again.  More than K entries fit (a full pool, or a wave's full
          // list, of whose pairs at most kPass have no candidate), all of them
          // at or above the last bound, so it rises each time and this ends.
          CTCBEAM_PHASE_COUNT(17);
          constexpr int EPT = kPool / kCT > 0 ? kPool / kCT : 1;  // entries a thread
          const int n = min(poff + s_n, kPool);
          uint64_t key[EPT];
          uint4 ent[EPT];
          float2 term[EPT];
#pragma unroll
          for (int h = 0; h < EPT; ++h) {
            const int e = tid + h * kCT;
            ent[h] = s_pool[e < n ? e : 0];
            term[h] = make_float2(0.0f, 0.0f);
            if (rep) term[h] = s_pterm[e < n ? e : 0];
            key[h] = e < n ? (static_cast<uint64_t>(ent[h].y) << 32) | ent[h].x : 0ull;
            int rk = 0;
            for (int f = 0; f < n; ++f) {
              const uint64_t o = *reinterpret_cast<const uint64_t*>(&s_pool[f]);
              rk += o > key[h] ? 1 : 0;
            }
            // (without the pair id, which may change)
            if (e < n && rk == K - 1) s_key = key[h] & ~static_cast<uint64_t>(kPairMask);
          }
          __syncthreads();
          const uint64_t nk = n >= K ? s_key : kmin;
          const bool stuck = n < K || (kmode && nk <= kmin);  // uniform; not reached: the bound rises
          kmin = nk;
          kmode = true;
          {
            const uint32_t u = static_cast<uint32_t>(kmin >> 32);
            if (n >= K) tau = fmaxf(tau, __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u));
          }
          __syncthreads();
          if (tid == 0) {
            s_over = 0;
            if (!stuck) s_n = 0;
          }
          __syncthreads();
          if (stuck) {
            status |= 4u;
            break;
          }
          if (!first) {
            // keep the earlier chunks' entries that reach the bound
#pragma unroll
            for (int h = 0; h < EPT; ++h) {
              if (tid + h * kCT < carry && key[h] >= kmin) {
                const int at = atomicAdd(&s_n, 1);
                s_pool[at] = ent[h];
                if (rep) s_pterm[at] = term[h];
              }
            }
            poff = 0;
          }
          pend = 0;
          __syncthreads();
          carry = s_n;  // (0 in the first chunk)
          __syncthreads();
        }
        first = false;
        carry = min(poff + s_n, kPool);  // (the next chunk adds after barrier B)
        CTCBEAM_PHASE_COUNT(10);  // chunks
      }
      gbase += C;
    }
    if (ahead) load_ahead();
    if (first) __syncthreads();  // no live slot: the pool is empty

    // ---- R. rank; successors ----
    if (wave == kCW - 1) {
      *reinterpret_cast<uint4*>(&s_cht[4 * lane]) = make_uint4(~0u, ~0u, ~0u, ~0u);
      if (lse) {
#pragma unroll
        for (int h = 0; h < SPL; ++h) s_ctop[lane + 64 * h] = 0ull;
      }
    }
    const int N = min(poff + s_n, kPool);
    {
      // 1 << lg neighbouring lanes count for one entry
      const int lg = N <= kCT / 8 ? 3 : N <= kCT / 4 ? 2 : N <= kCT / 2 ? 1 : 0;  // uniform
      const int G = 1 << lg;
      const uint32_t* prec = s_rec[rcur];
      uint32_t* nrec = s_rec[rcur ^ 1];
      int32_t* bpf = s_bpf + (t & (kBpFrames - 1)) * K;
      for (int eb = 0; eb < N; eb += kCT) {  // uniform
        const int e = eb + (tid >> lg), g = tid & (G - 1);
        const bool act = e < N;
        const uint4 me = s_pool[act ? e : 0];
        const uint64_t key = (static_cast<uint64_t>(me.y) << 32) | me.x;
        const uint32_t flat = ~me.x;
        const uint32_t par = flat >> kSlotShift;
        const uint32_t c = (flat >> kLabelShift) & kLabelMask;
        // the parent's record (inactive lanes name a valid entry's)
        const uint32_t* src = static_cast<const uint32_t*>(__builtin_assume_aligned(prec + par * RW, 16));
        const uint4 r0 = *reinterpret_cast<const uint4*>(src), r1 = *reinterpret_cast<const uint4*>(src + 4);
        int rk = 0;
#pragma unroll 4
        for (int i = g; i < N; i += G) {
          const uint64_t o = *reinterpret_cast<const uint64_t*>(&s_pool[i]);
          rk += o > key ? 1 : 0;
        }
        if (lg >= 1) rk += static_cast<int>(xor_lane(static_cast<uint32_t>(rk), 1, lane));
        if (lg >= 2) rk += static_cast<int>(xor_lane(static_cast<uint32_t>(rk), 2, lane));
        if (lg >= 3) rk += static_cast<int>(xor_lane(static_cast<uint32_t>(rk), 4, lane));
        if (act && g == 0 && rk < K) {
          const bool emit = c != static_cast<uint32_t>(V) && c != (r1.x & 0xFFFFu);
          uint64_t h = (static_cast<uint64_t>(r0.z) << 32) | r0.y;
          const uint64_t hm = mix_token(h, c);
          h = emit ? hm : h;
          const uint32_t u = me.y;
          uint32_t* dst = static_cast<uint32_t*>(__builtin_assume_aligned(nrec + rk * RW, 16));
          *reinterpret_cast<uint4*>(dst) =
              make_uint4((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u, static_cast<uint32_t>(h),
                         static_cast<uint32_t>(h >> 32), r0.w + (emit ? 1u : 0u));
          *reinterpret_cast<uint4*>(dst + 4) =
              make_uint4(c | ((emit ? (flat & kPairMask) : kPairMask) << 16), (NL > 0 && emit) ? me.z : r1.y,
                         (HAS_BT && emit) ? (me.w & kBtChildMask) : r1.z, emit ? 1u : 0u);
          if (rep) s_rterm[(rcur ^ 1) * KMX + rk] = emit ? s_pterm[e] : s_rterm[rcur * KMX + par];
          bpf[rk] = static_cast<int32_t>((par << 16) | c);
        }
      }
      if (tid >= N && tid < K) bpf[tid] = -1;
    }
    store_pairs();
    CTCBEAM_PHASE_ADD(15, N);  // pool entries
    CTCBEAM_PHASE_MARK(6);
    __syncthreads();  // D: successor records complete
    CTCBEAM_PHASE_MARK(7);
    if (tid == 0) s_n = 0;
    if (((t + 1) & (kBpFrames - 1)) == 0 || t + 1 == L) {  // uniform
      // the back-pointers of the last frames go out together: a store holds
      // the wave's next load wait
      const int f0 = t & ~(kBpFrames - 1);
      const int n = (t + 1 - f0) * K;
      for (int q = tid; q < n; q += kCT) bpb[static_cast<size_t>(f0) * K + q] = s_bpf[q];
    }

    // ---- U. prune, recombine, take the new beam (lane = slot) ----
    rcur ^= 1;
    const int nsel = min(K, N);
    float x[SPL];
    bool alive0[SPL], dup[SPL];
    uint32_t klo[SPL], khi[SPL];
    {
      float best = kNegInf;
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        const int js = lane + 64 * h;
        const bool valid = js < nsel;
        const uint32_t* src = static_cast<const uint32_t*>(__builtin_assume_aligned(s_rec[rcur] + (valid ? js : 0) * RW, 16));
        const uint4 r0 = *reinterpret_cast<const uint4*>(src);
        const uint4 r1 = *reinterpret_cast<const uint4*>(src + 4);
        x[h] = valid ? __uint_as_float(r0.x) : kNegInf;
        // prune (Algorithm 1: below best - theta -> -inf)
        if (h == 0) best = rdlane(x[0], 0);
        if (valid && x[h] < best - p.theta) x[h] = kNegInf;
        last[h] = valid ? static_cast<int32_t>(r1.x & 0xFFFFu) : V;
        len[h] = valid ? static_cast<int32_t>(r0.w) : 0;
        lms[h] = r1.y;
        bts[h] = r1.z;
        if (rep) {
          const float2 tm = s_rterm[rcur * KMX + (valid ? js : 0)];
          ral[h] = tm.x;
          rwb[h] = tm.y;
        }
        alive0[h] = valid && x[h] != kNegInf;
        // recombination key: the 64-bit transcript hash with the length and
        // the ends-in-blank flag folded in; dead slots use all ones
        const uint32_t meta = (static_cast<uint32_t>(len[h]) & 0x3FFFFFFFu) | ((last[h] == V ? 1u : 0u) << 30);
        uint64_t key = ((static_cast<uint64_t>(r0.z) << 32) | r0.y) ^ (static_cast<uint64_t>(meta + 1u) * 0xD6E8FEB86659FD93ull);
        if (!alive0[h]) key = ~0ull;
        klo[h] = static_cast<uint32_t>(key);
        khi[h] = static_cast<uint32_t>(key >> 32);
        dup[h] = false;
        if (want_stats && wave == 0 && alive0[h] && r1.w != 0u) atomicAdd(&s_st[5], 1ull);
      }
    }
    if (K <= 16) {
      // the slots sit in one 16-lane row: compare with the lower ones
      dup[0] = (K <= 8 ? recomb_shifts<1, 7>(klo[0], khi[0]) : recomb_shifts<1, 15>(klo[0], khi[0])) && alive0[0];
    } else {
      // each wave finds the duplicates among its share of the slots
      uint64_t mine[SPL];
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        mine[h] = 0ull;
        const uint64_t live = __ballot(alive0[h]);
        for (int i = wave; i < 64 && i + 64 * h < nsel; i += kCW) {  // uniform
          const uint32_t l0 = rdlane(klo[h], i), h0 = rdlane(khi[h], i);
          uint64_t low = __ballot(klo[h] == l0 && khi[h] == h0) & ((1ull << i) - 1ull);
          if (SPL > 1 && h > 0) low |= __ballot(klo[0] == l0 && khi[0] == h0);
          if (low != 0ull) mine[h] |= (1ull << i) & live;
        }
        // (per-lane address: a uniform one, s_dup[wave] in lane 0, lengthens
        // other live ranges and costs 3 % at K = 94 without models)
        if (lane < 1) s_dup[wave + lane][h] = mine[h];
      }
      __syncthreads();
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        const uint64_t m = s_dup[lane & 7][h];
        uint32_t ml = static_cast<uint32_t>(m), mh = static_cast<uint32_t>(m >> 32);
        ml |= xor_lane(ml, 1, lane);
        mh |= xor_lane(mh, 1, lane);
        ml |= xor_lane(ml, 2, lane);
        mh |= xor_lane(mh, 2, lane);
        ml |= xor_lane(ml, 4, lane);
        mh |= xor_lane(mh, 4, lane);
        dup[h] = (((lane < 32 ? ml : mh) >> (lane & 31)) & 1u) != 0u;
      }
    }
    if (lse) {  // uniform
      // Each duplicate, in slot order, is merged into the first live slot of
      // its transcript (a lower slot, which is not a duplicate itself).
      float xs[SPL];
#pragma unroll
      for (int h = 0; h < SPL; ++h) xs[h] = x[h];
#pragma unroll
      for (int hj = 0; hj < SPL; ++hj) {
        uint64_t dm = __ballot(dup[hj]);
        while (dm) {
          const int jj = first_of(dm);
          dm &= dm - 1ull;
          const uint32_t l0 = rdlane(klo[hj], jj), h0 = rdlane(khi[hj], jj);
          int to = -1;  // the duplicate itself matches, so some slot does
#pragma unroll
          for (int h = SPL - 1; h >= 0; --h) {
            const uint64_t same = __ballot(alive0[h] && klo[h] == l0 && khi[h] == h0);
            if (same) to = first_of(same) + 64 * h;
          }
          const float xj = rdlane(xs[hj], jj);
#pragma unroll
          for (int h = 0; h < SPL; ++h)
            if (lane + 64 * h == to && to != jj + 64 * hj) x[h] = lse32(x[h], xj);
        }
      }
    }
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      alive[h] = alive0[h] && !dup[h];
      sc[h] = alive[h] ? x[h] : kNegInf;
      if (want_stats && wave == 0 && alive[h] && t + 1 < L) {
        // chain work of the next frame
        unsigned long long ns = 0, nar = 0;
        for (int l = 0; l < NL; ++l) {
          const LmLevel hd = p.lm_states[static_cast<size_t>(lms[h]) * NL + l];
          if (hd.count & kExists) {
            ns += 1;
            nar += hd.count & ~kExists;
          }
        }
        atomicAdd(&s_st[0], 1ull);
        if (ns) atomicAdd(&s_st[1], ns);
        if (nar) atomicAdd(&s_st[2], nar);
        if (HAS_BT) {
          const BtNode nd = p.bt_nodes[bts[h]];
          if (nd.pot >> 8) atomicAdd(&s_st[3], static_cast<unsigned long long>(nd.pot >> 8));
          if (nd.chain_arcs) atomicAdd(&s_st[4], static_cast<unsigned long long>(nd.chain_arcs));
        }
      }
    }
    CTCBEAM_PHASE_MARK(8);
    CTCBEAM_PHASE_COUNT(9);  // frames
  }
#ifdef CTCBEAM_PHASE_CLOCKS
  if (p.stats && lane < kPhaseWords) {
    int64_t* pw = p.stats + static_cast<size_t>(p.B) * 8 + (static_cast<size_t>(b) * 8 + wave) * kPhaseWords;
    pw[lane] = static_cast<int64_t>(ph_acc);
  }
#endif

  // ---- LM.Final, order of the final hypotheses ----
  const bool nbest = p.nbest_scores != nullptr;
  uint32_t* const s_len = reinterpret_cast<uint32_t*>(s_ctop);  // by rank
  uint32_t* const s_rank = s_len + KMX;                         // by slot
  float sj[SPL];  // wave 0: final score of the slot, -inf for a dead one
#pragma unroll
  for (int h = 0; h < SPL; ++h) sj[h] = kNegInf;
  if (wave == 0) {
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      const int js = lane + 64 * h;
      float s = sc[h];
      if (HAS_LM && js < K && s != kNegInf) {
        // ln P(</s> | state) through the backoff chain; </s> is the last arc
        // of a state's sorted arcs when present
        float v = p.lm_unigram[V];
        for (int l = 0; l < NL; ++l) {
          const LmLevel hd = p.lm_states[static_cast<size_t>(lms[h]) * NL + l];
          v = v + hd.bo;
          const uint32_t n = hd.count & ~kExists;
          if (n > 0u) {
            const LmArc a = p.lm_arcs[hd.begin + n - 1u];
            if (a.token == static_cast<uint32_t>(V)) v = a.logp;
          }
        }
        const float av = alpha * v;
        s = s + av;
      }
      if (HAS_BT && (p.flags & kFlagBoostRollback) && js < K && s != kNegInf) {
        // the pending boosting of an unfinished phrase is taken back
        const float wb = boost_w * static_cast<float>(-static_cast<int>(p.bt_nodes[bts[h]].pot & 0xFFu));
        s = s + wb;
      }
      sj[h] = (js < K && s > kNegInf) ? s : kNegInf;
    }
    // rank of each slot: final score descending, lowest slot on ties (a NaN
    // would leave ranks without a slot)
    int rank[SPL];
#pragma unroll
    for (int h = 0; h < SPL; ++h) rank[h] = 0;
    for (int i = 0; i < K; ++i) {
      const float si = (i < 64) ? rdlane(sj[0], i) : rdlane(sj[SPL - 1], i & 63);
#pragma unroll
      for (int h = 0; h < SPL; ++h) rank[h] += (si > sj[h] || (si == sj[h] && i < lane + 64 * h)) ? 1 : 0;
    }
    int bj = 0;  // K >= 1: some slot has rank 0
#pragma unroll
    for (int h = SPL - 1; h >= 0; --h) {
      const uint64_t top = __ballot(lane + 64 * h < K && rank[h] == 0);
      if (top) bj = first_of(top) + 64 * h;
    }
    const float bs = (bj < 64) ? rdlane(sj[0], bj) : rdlane(sj[SPL - 1], bj & 63);
    const int blen = (bj < 64) ? rdlane(len[0], bj) : rdlane(len[SPL - 1], bj & 63);
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      const int js = lane + 64 * h;
      const int nlen = (js < K && sj[h] != kNegInf) ? len[h] : 0;
      if (nbest && js < K) {
        p.nbest_scores[static_cast<size_t>(b) * K + rank[h]] = sj[h];
        p.nbest_lengths[static_cast<size_t>(b) * K + rank[h]] = nlen;
        s_len[rank[h]] = static_cast<uint32_t>(nlen);
        s_rank[js] = static_cast<uint32_t>(rank[h]);
      }
    }
    if (lane == 0) {
      s_best = bj;
      s_bestscore = bs;
      s_bestlen = blen;
    }
    if (want_stats && lane == 0) {
      // wave 0 made every update of s_st (LDS operations of one wave complete
      // in order)
      int64_t* so = p.stats + static_cast<size_t>(b) * 8;
      so[0] = L;
#pragma unroll
      for (int q = 0; q < 6; ++q) so[1 + q] = static_cast<int64_t>(s_st[q]);
      so[7] = 0;
    }
  }
  __syncthreads();
  const int best = s_best;
  const float bscore = s_bestscore;
  const bool have = bscore != kNegInf;
  const int nout = have ? s_bestlen : 0;
  int32_t* ot = p.out_tokens ? p.out_tokens + static_cast<size_t>(b) * T : nullptr;
  if (ot)
    for (int tt = nout + tid; tt < T; tt += kCT) ot[tt] = -1;
  if (tid == 0 && p.out_scores) {
    p.out_scores[b] = bscore;
    if (p.out_lengths) p.out_lengths[b] = nout;
  }
  int32_t* nbt = nbest ? p.nbest_tokens + static_cast<size_t>(b) * K * T : nullptr;
  if (nbest) {
    // padding of every row past its transcript
    for (int r = 0; r < K; ++r) {
      const int n = static_cast<int>(s_len[r]);
      for (int tt = n + tid; tt < T; tt += kCT) nbt[static_cast<size_t>(r) * T + tt] = -1;
    }
  }

  // ---- traceback through the back-pointers, staged in LDS tiles ----
  // 1-best: lane 0 of wave 0 walks the best slot.  N-best: lane j of wave 0
  // walks slots j + 64 h (every slot with a final score) and writes the rows of
  // their ranks.
  if (have && L > 0) {
    int32_t* const s_bp = reinterpret_cast<int32_t*>(s_area);
    const int tile_frames = kArea / 4 / K;
    bool walker[SPL];
    int jb[SPL], cnext[SPL], pos[SPL];
    int32_t* orow[SPL];
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      const int js = lane + 64 * h;
      walker[h] = (wave == 0) && (nbest ? sj[h] != kNegInf : (h == 0 && lane == 0));
      jb[h] = nbest ? js : best;
      cnext[h] = -1;
      orow[h] = nullptr;
      pos[h] = 0;
      if (walker[h]) {
        orow[h] = nbest ? nbt + static_cast<size_t>(s_rank[js]) * T : ot;
        pos[h] = nbest ? len[h] : nout;
      }
    }
    for (int hi = L; hi > 0;) {
      const int lo = hi > tile_frames ? hi - tile_frames : 0;
      __syncthreads();
      const int n = (hi - lo) * K;
      const int32_t* src = bpb + static_cast<size_t>(lo) * K;
      for (int q = tid; q < n; q += kCT) s_bp[q] = src[q];
      __syncthreads();
#pragma unroll
      for (int h = 0; h < SPL; ++h) {
        if (walker[h]) {
          for (int tt = hi - 1; tt >= lo; --tt) {
            const uint32_t e = static_cast<uint32_t>(s_bp[(tt - lo) * K + jb[h]]);
            const int cl = static_cast<int>(e & 0xFFFFu);
            const int par = static_cast<int>(e >> 16);
            if (tt < L - 1 && cnext[h] != V && cnext[h] != cl) {
              if (pos[h] > 0) {
                --pos[h];
                if (orow[h]) orow[h][pos[h]] = cnext[h];
              }
            }
            cnext[h] = cl;
            jb[h] = par;
          }
        }
      }
      hi = lo;
    }
    bool bad = false;
#pragma unroll
    for (int h = 0; h < SPL; ++h) {
      if (walker[h]) {
        if (cnext[h] != V && cnext[h] >= 0 && pos[h] > 0) {
          --pos[h];
          if (orow[h]) orow[h][pos[h]] = cnext[h];
        }
        bad = bad || pos[h] != 0;
      }
    }
    if (wave == 0 && __ballot(bad) != 0ull) status |= 2u;
  }
  if (tid == 0) {
    p.status[b] = status;
    if (b == 0) write_ws_header(p.ws_header, p.B);
  }
}

template <int LPT, int NLEV, int SPL>
hipError_t launch_class_nlev(const KernelParams& p, hipStream_t s) {
  dim3 grid(p.B), block(kCT);
  if (p.bt_nodes != nullptr)
    hipLaunchKernelGGL((class_kernel<LPT, NLEV, true, SPL>), grid, block, 0, s, p);
  else
    hipLaunchKernelGGL((class_kernel<LPT, NLEV, false, SPL>), grid, block, 0, s, p);
  return hipGetLastError();
}

template <int LPT, int SPL>
hipError_t launch_class_spl(const KernelParams& p, hipStream_t s) {
  if (p.lm_states == nullptr && p.lm_arcs == nullptr) return launch_class_nlev<LPT, -1, SPL>(p, s);
  switch (p.lm_nlev) {
    case 0: return launch_class_nlev<LPT, 0, SPL>(p, s);
    case 1: return launch_class_nlev<LPT, 1, SPL>(p, s);
    case 2: return launch_class_nlev<LPT, 2, SPL>(p, s);
    case 3: return launch_class_nlev<LPT, 3, SPL>(p, s);
    case 4: return launch_class_nlev<LPT, 4, SPL>(p, s);
    case 5: return launch_class_nlev<LPT, 5, SPL>(p, s);
    case 6: return launch_class_nlev<LPT, 6, SPL>(p, s);
    case 7: return launch_class_nlev<LPT, 7, SPL>(p, s);
    default: return hipErrorInvalidValue;
  }
}

// beams above 64 take two slots per lane (vocabularies of at most 1024
// tokens; the host rejects the rest)
template <int LPT>
hipError_t launch_class_lpt(const KernelParams& p, hipStream_t s) {
  if constexpr (LPT * kCT <= 1024) {
    if (p.K > 64) return launch_class_spl<LPT, 2>(p, s);
  } else {
    if (p.K > 64) return hipErrorInvalidValue;
  }
  return launch_class_spl<LPT, 1>(p, s);
}

}  // namespace classes
}  // namespace ctcbeam
