// Small-beam decoder: K <= 8 hypotheses, V <= 1024 tokens, no LM and no
// phrase boosting (gfx950).  Included by ctcbeam_small.hip.
//
// Same search as the general decoder (FlexCTC Algorithm 1 with the Eq. 1
// fold x = s_k + D[c], x += beta for emitting labels; TopK by (score desc,
// flat index asc); pruning; recombination; read-out of the hypothesis trie,
// Sec. III-A), laid out for the beam sizes of the paper's main tables
// (K = 4..8) without a language model.
//
// What bounds it is the serial chain of the frames: the beam of frame t is
// known only when frame t - 1 is done.  The work that does not depend on the
// beam is therefore taken out of that chain.  Without models a label's score
// depends on the beam only through s_k, and fp32 addition is monotone, so the
// candidates of every beam are ordered as D is, and the K best of a frame lie
// among few (beam, label rank) positions: with the live beams in descending
// order of score, a candidate of beam i with the label of rank r (rank by D
// descending, label ascending) has at least (i + 1) r - 1 emitting candidates
// of no lower score before it (each beam's repeat label, which emits nothing,
// is taken off), so those with (i + 1) r > K are not needed.  That leaves
// sum_i (K / (i + 1) + 1) = 28 candidates at K = 8; with 8 blanks and 8
// repeats a frame's selection is 44 entries: one per lane of one wave.
//
// One workgroup of 4 wave64 per utterance, one wave per SIMD:
// * waves 1..3 make, a batch of frames ahead, each frame's list of its K + 2
//   best labels (a bound from the lane maxima, the values that reach it
//   gathered, ranked by counting) and leave the row in LDS for the repeats;
// * wave 0 runs the chain alone, without a barrier inside a batch: read the
//   beam, one candidate per lane, rank by counting, successors, prune,
//   recombine.
//
// A candidate left out ties the K-th best at most.  K further lanes carry the
// best score left out of each beam; when one of them reaches the K-th best, or
// two entries have equal scores, the frame is settled by the exact keys
// (score, flat index), and the places at the K-th best score go to the lowest
// flat indices of all candidates with that score.
//
// The chain of wave 0 bounds it, about 2.5 k cycles a frame (423 us for 400
// frames): a wave alone on its SIMD issues a dependent instruction every 7 to 8
// cycles and waits about 130 for LDS.  So the rank takes the signs of
// differences instead of compares and carries, a winner brings its new
// transcript hash with it (formed in every entry's lane while the scores settle
// in LDS) instead of reading its parent's afterwards, and the next frame's list
// entry is read a frame ahead (32 utterances of 400 frames, V = 1024, K = 8:
// 0.68 -> 0.43 ms; the form before the lists, with every label scored for every
// beam behind three barriers a frame, took 1.48).  The lists themselves cost
// nothing that shows.  One utterance of 50 frames, V = 32, K = 4: 0.114 ->
// 0.038 ms with the code warm, 0.170 -> 0.089 ms for a first call on new inputs,
// which is mostly the launch and cold code.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ctcbeam_internal.h"
#include "ctcbeam_lane.h"

namespace ctcbeam {
namespace small {

using detail::kNegInf;
using detail::lanemask_lt;
using detail::mix_token;
using detail::order_key;
using detail::rdlane;

constexpr int kST = 256;             // threads: 4 wave64
constexpr int kSW = kST / 64;        // waves
constexpr int kVmax = 1024;          // labels (blank handled apart)
constexpr int kKmax = 8;             // beam slots
constexpr int kFP = 2;               // frames a list wave makes per batch
constexpr int kF = kFP * (kSW - 1);  // frames of a batch
constexpr int kList = kKmax + 2;     // list entries of a frame
constexpr int kGather = 64;          // values gathered for a list

// order of LDS accesses between lanes of one wave (LDS operations of a wave
// complete in issue order, so the compiler has to keep it)
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
// One frame's M best labels by value descending and label ascending, where the
// gather does not hold all values that reach the bound tau (ties, or many
// labels of few lanes): M rounds of "best key below the previous one".
template <int NJ>
__device__ __forceinline__ void extract_list(const float (&v)[NJ], int M, int lane, uint2* list) {
  uint64_t prev = ~0ull;
#pragma unroll 1
  for (int r = 0; r < M; ++r) {
    uint64_t best = 0ull;
    float bv = kNegInf;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const uint64_t key = v[j] != kNegInf ? order_key(v[j], static_cast<uint32_t>(lane + 64 * j)) : 0ull;
      if (key < prev && key > best) {
        best = key;
        bv = v[j];
      }
    }
    uint64_t wb = best;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t o = __shfl_xor(wb, off);
      wb = o > wb ? o : wb;
    }
    if (wb == 0ull) break;  // uniform: nothing finite left
    if (best == wb) list[r] = make_uint2(__float_as_uint(bv), 0xFFFFFFFFu - static_cast<uint32_t>(wb));
    prev = wb;
  }
}

// The M best labels of each of NQ frames, by value descending and label
// ascending; lane l holds labels l + 64 j (-inf past V and for NaN) and the
// frames' rows are in LDS.  list[q] gets (value, label) pairs, entries past the
// finite values (-inf, V).  The frames go through each step together: a step
// is a chain of dependent instructions.
template <int NJ, int NQ, int GS, int LS, int RS>
__device__ __forceinline__ void make_lists(const float (&v)[NQ][NJ], int M, int V, int lane, const float* row,
                                           uint64_t* gather, uint2* list) {
  float tau[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    float top = v[q][0];
#pragma unroll
    for (int j = 1; j < NJ; ++j) top = fmaxf(top, v[q][j]);
    tau[q] = detail::wave_sort_desc<64>(top, lane);
  }
  uint32_t bits[NQ];
  int n[NQ], at[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    // M lanes reach the M-th largest lane maximum, so the M best values do
    const float t = rdlane(tau[q], M - 1);
    bits[q] = 0u;
#pragma unroll
    for (int j = 0; j < NJ; ++j) bits[q] |= (v[q][j] >= t && v[q][j] != kNegInf) ? (1u << j) : 0u;
    const int cnt = __popc(bits[q]);
    const int incl = detail::wave_incl_scan(cnt, lane);
    n[q] = rdlane(incl, 63);
    at[q] = incl - cnt;
    if (lane < M) list[q * LS + lane] = make_uint2(__float_as_uint(kNegInf), static_cast<uint32_t>(V));
    gather[q * GS + lane] = 0ull;
  }
  wave_lds_fence();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (n[q] <= kGather) {  // uniform
      for (uint32_t m = bits[q]; m != 0u; m &= m - 1u) {  // usually none or one
        const uint32_t c = static_cast<uint32_t>(lane + 64 * __builtin_ctz(m));
        gather[q * GS + at[q]++] = order_key(row[q * RS + c], c);
      }
    }
  }
  wave_lds_fence();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    if (n[q] <= kGather) {  // uniform
      const uint64_t key = gather[q * GS + lane];  // 0: none
      int rank = 0;
#pragma unroll
      for (int i = 0; i < 10; ++i) {
        const ulonglong2 o = reinterpret_cast<const ulonglong2*>(gather + q * GS)[i];
        rank += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0);
      }
      for (int i = 10; 2 * i < n[q]; ++i) {  // uniform trip count
        const ulonglong2 o = reinterpret_cast<const ulonglong2*>(gather + q * GS)[i];
        rank += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0);
      }
      if (key != 0ull && rank < M) {
        const uint32_t c = 0xFFFFFFFFu - static_cast<uint32_t>(key);
        list[q * LS + rank] = make_uint2(__float_as_uint(row[q * RS + c]), c);
      }
    } else {
      extract_list<NJ>(v[q], M, lane, list + q * LS);
    }
  }
}

// NJ = labels per lane of a list wave (V <= 64 NJ)
template <int NJ>
__global__ void __launch_bounds__(kST) small_kernel(KernelParams p) {
  constexpr int kRow = NJ * 64 + 4;  // labels and the blank of a frame
  constexpr int kRowWords = 2 * kF * kRow;
  constexpr int kStageWords = kRowWords > 4096 ? kRowWords : 4096;
  // rows of two batches of frames; the traceback's tiles after the last frame
  __shared__ __align__(16) uint32_t s_big[kStageWords];
  __shared__ uint2 s_list[2][kF][kList];  // (value, label)
  __shared__ __align__(16) uint64_t s_gather[kSW - 1][kFP][kGather];
  __shared__ int s_bp[2][kF * kKmax];     // back-pointers of a batch
  // the beam as the scoring sees it, by live position (slot order; dead
  // positions score -inf): score bits, last label, slot, the last label's
  // value in the frame
  __shared__ uint4 s_beam[kKmax];
  __shared__ uint4 s_hash[kKmax];  // transcript hash lo, hi, length, 0
  __shared__ __align__(16) float s_x[64];       // scores ranked
  __shared__ __align__(16) uint64_t s_key[64];  // keys ranked (equal scores)
  __shared__ uint32_t s_tie[kKmax];             // winners at the K-th best score
  __shared__ int s_best, s_bestlen;
  __shared__ float s_bestscore;
  __shared__ int s_nblen[kKmax], s_nbrank[kKmax];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x;
  const int V = p.V, W = V + 1, K = p.K, T = p.T;
  const float beta = p.beta;
  const bool want_stats = p.stats != nullptr;

  int L = p.lengths[b];
  uint32_t status = 0;
  if (L < 0) { L = 0; status |= 1u; }
  if (L > T) { L = T; status |= 1u; }
  const float* Db = p.logprobs + static_cast<size_t>(b) * T * W;
  int32_t* bpb = p.bp + static_cast<size_t>(b) * T * K;
  float* const s_row = reinterpret_cast<float*>(s_big);
  const int nbatch = (L + kF - 1) / kF;

  // ---- the beam (wave 0, slot k in lane k) ----
  float sc = (lane == 0) ? 0.0f : kNegInf;
  int last = V, len = 0;
  uint32_t hlo = 0u, hhi = 0u;
  // counters (wave 0 lanes, summed at the end)
  uint32_t st_alive = 0u, st_emit = 0u;

  // ---- wave 0: the entry of this lane ----
  // emitting candidates (position ei, label rank er), then the blanks, the
  // repeats and the best candidates left out (er = K / (ei + 1) + 1)
  int ei = 0, er = 0, nent = 0;
  bool k_emit = false, k_blank = false, k_rep = false, k_out = false;
  {
    int at = 0;
    for (int i = 0; i < K; ++i) {
      const int n = K / (i + 1) + 1;
      if (lane >= at && lane < at + n) {
        k_emit = true;
        ei = i;
        er = lane - at;
      }
      at += n;
    }
    nent = at + 2 * K;
    const int q = lane - at;
    if (q >= 0 && q < 3 * K) {
      const int g = q / K;
      ei = q - g * K;
      k_blank = g == 0;
      k_rep = g == 1;
      k_out = g == 2;
      if (k_out) er = K / (ei + 1) + 1;
    }
  }
  const bool k_any = k_emit || k_blank || k_rep || k_out;
  const bool k_label = k_emit || k_out;  // lanes that read the list

  // ---- waves 1..3: frames ahead ----
  // (frames past the end repeat the last one; nothing reads them)
  float rn[kFP][NJ], rb[kFP];
  const auto load_rows = [&](int n) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < kFP; ++q) {
      const int t = min(n * kF + (wave - 1) * kFP + q, L - 1);
      const float* rowp = Db + static_cast<size_t>(t) * W;
#pragma unroll
      for (int j = 0; j < NJ; ++j) rn[q][j] = __builtin_nontemporal_load(rowp + min(lane + 64 * j, V));
      rb[q] = rowp[V];
    }
  };
  const auto make_frames = [&](int n) __attribute__((always_inline)) {
    const int f0 = (n & 1) * kF + (wave - 1) * kFP;
    float* row = s_row + f0 * kRow;
    float v[kFP][NJ];
#pragma unroll
    for (int q = 0; q < kFP; ++q) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int c = lane + 64 * j;
        const float d = rn[q][j];
        v[q][j] = (c < V && d == d) ? d : kNegInf;
        if (c < V) row[q * kRow + c] = v[q][j];
      }
      if (lane == 0) row[q * kRow + V] = rb[q];
    }
    make_lists<NJ, kFP, kGather, kList, kRow>(v, K + 2, V, lane, row, s_gather[wave - 1][0],
                                              &s_list[0][0][0] + f0 * kList);
  };
  // back-pointers of batch n to global memory
  const auto store_bp = [&](int n) __attribute__((always_inline)) {
    const int cnt = min(kF, L - n * kF) * K;
    if (wave == 1 && lane < cnt) bpb[static_cast<size_t>(n) * kF * K + lane] = s_bp[n & 1][lane];
  };
  static_assert(kF * kKmax <= 64, "a batch's back-pointers are stored by one wave");

  // profiling builds: wave 0's cycles of the entries, the rank, the winners, the
  // equal scores, the successors, the recombination, the new beam, the batch's
  // barrier; then frames, frames with equal scores, searches over all labels
#ifdef CTCBEAM_PHASE_CLOCKS
  uint64_t ph_acc = 0ull;
  uint64_t ph_t0 = __builtin_amdgcn_s_memtime();
#endif

  // round n: wave 0 decodes batch n, waves 1..3 make batch n + 1.  Two loops with
  // the same barriers: in one, each side's lane masks would stay live through
  // the other's
  if (wave != 0) {
    if (nbatch > 0) load_rows(0);
    for (int n = -1; n < nbatch; ++n) {
      if (n + 1 < nbatch) {
        make_frames(n + 1);
        if (n + 2 < nbatch) load_rows(n + 2);
      }
      if (n > 0) store_bp(n - 1);
      detail::lds_barrier();
    }
    if (nbatch > 0) store_bp(nbatch - 1);
  } else {
    if (lane < kKmax) {
      s_beam[lane] = make_uint4(__float_as_uint(lane == 0 ? 0.0f : kNegInf), static_cast<uint32_t>(V), 0u, 0u);
      s_hash[lane] = make_uint4(0u, 0u, 0u, 0u);
    }
    detail::lds_barrier();
    for (int n = 0; n < nbatch; ++n) {
      const int nf = min(kF, L - n * kF);
      const float* row0 = s_row + ((n & 1) * kF) * kRow;
      // the last labels' values in the batch's first row, which was not there
      // before
      wave_lds_fence();
      if (lane < kKmax) s_beam[lane].w = __float_as_uint(row0[s_beam[lane].y]);
      wave_lds_fence();
      uint2 le = s_list[n & 1][0][er];
      float dblank = row0[V];
      for (int f = 0; f < nf; ++f) {
        const float* row = row0 + f * kRow;
        wave_lds_fence();
        const uint4 br = s_beam[ei];
        const uint4 hr = s_hash[ei];
        const float si = __uint_as_float(br.x);
        const int li = static_cast<int>(br.y);
        const float drep = __uint_as_float(br.w);
        // the candidate of this lane
        const int c = k_label ? static_cast<int>(le.y) : k_rep ? li : V;
        const float d = k_label ? __uint_as_float(le.x) : k_rep ? drep : dblank;
        float x = si + d;
        const float xe = x + beta;
        x = k_label ? xe : x;
        // the repeat of the beam's last frame label emits nothing; no repeat
        // after a blank; NaN candidates are none (selects, not branches)
        const int off = k_rep ? V : k_emit ? li : -1;
        const int me = k_rep ? li : c;
        x = (me == off) ? kNegInf : x;
        const float xn = (x == x) ? x : kNegInf;
        x = k_any ? xn : kNegInf;
        const float xo = k_out ? x : kNegInf;  // the best candidate left out of position ei
        if (k_out) x = kNegInf;
        const bool evalid = x != kNegInf;
        CTCBEAM_PHASE_MARK(0);
        s_x[lane] = x;
        wave_lds_fence();
        // while the scores settle: the transcript this candidate would have
        const uint64_t ph = (static_cast<uint64_t>(hr.y) << 32) | hr.x;
        const uint64_t eh = k_emit ? mix_token(ph, static_cast<uint32_t>(c)) : ph;
        const int el = static_cast<int>(hr.z) + (k_emit ? 1 : 0);
        // and the next frame's list entry and blank
        const int fn = min(f + 1, nf - 1);
        const uint2 le_next = s_list[n & 1][fn][er];
        const float db_next = row0[fn * kRow + V];
        // rank: the scores above this one, as the signs of the differences
        // gathered in four words (a compare and its carry need wait states
        // between them; a difference that rounds to zero reads as equal)
        uint32_t w0 = 0u, w1 = 0u, w2 = 0u, w3 = 0u;
        const auto above = [&](int q) __attribute__((always_inline)) {
          const float4 o = reinterpret_cast<const float4*>(s_x)[q];
          w0 = __builtin_amdgcn_alignbit(w0, __float_as_uint(x - o.x), 31u);
          w1 = __builtin_amdgcn_alignbit(w1, __float_as_uint(x - o.y), 31u);
          w2 = __builtin_amdgcn_alignbit(w2, __float_as_uint(x - o.z), 31u);
          w3 = __builtin_amdgcn_alignbit(w3, __float_as_uint(x - o.w), 31u);
        };
#pragma unroll
        for (int q = 0; q < 5; ++q) above(q);
        if (nent > 20) {  // uniform
#pragma unroll
          for (int q = 5; q < 11; ++q) above(q);
        }
        int rank = (__popc(w0) + __popc(w1)) + (__popc(w2) + __popc(w3));
        CTCBEAM_PHASE_MARK(1);
        int nfin = min(K, static_cast<int>(__popcll(__ballot(evalid))));
        // the winner of rank r goes to lane r, marked in bit 20 (others write to
        // lane 63, which no winner reads: K <= 8)
        bool top = evalid && rank < K;
        const int epk = (1 << 20) | (c << 3) | ((k_emit ? 1 : 0) << 14) | (static_cast<int>(br.z) << 15);
        const int dst = (top ? rank : 63) << 2;
        int pk = __builtin_amdgcn_ds_permute(dst, epk);
        float wx = __int_as_float(__builtin_amdgcn_ds_permute(dst, __float_as_int(x)));
        uint32_t whlo = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(dst, static_cast<int>(eh)));
        uint32_t whhi = static_cast<uint32_t>(__builtin_amdgcn_ds_permute(dst, static_cast<int>(eh >> 32)));
        int wlen = __builtin_amdgcn_ds_permute(dst, el);
        // equal scores leave a rank without an entry or put more than K there,
        // or a score left out reaches the K-th best (with K of them)
        const float xk = rdlane(wx, K - 1);
        const uint64_t odd = __ballot(lane < nfin && pk == 0) | (nfin == K ? __ballot(xo != kNegInf && xo >= xk) : 0ull);
        const bool slow = odd != 0ull || static_cast<int>(__popcll(__ballot(top))) != nfin;
        CTCBEAM_PHASE_MARK(2);
        if (slow) {  // uniform, rare
          CTCBEAM_PHASE_COUNT(10);
          const uint64_t key = evalid ? order_key(x, static_cast<uint32_t>(ei * W + c)) : 0ull;
          s_key[lane] = key;
          wave_lds_fence();
          rank = 0;
#pragma unroll
          for (int m = 0; m < 22; ++m) {  // 44 entries; keys past them are 0
            const ulonglong2 o = reinterpret_cast<const ulonglong2*>(s_key)[m];
            rank += (o.x > key ? 1 : 0) + (o.y > key ? 1 : 0);
          }
          top = evalid && rank < K;
          const int to = (top ? rank : 63) << 2;
          pk = __builtin_amdgcn_ds_permute(to, epk);
          wx = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(x)));
          const float xt = rdlane(wx, K - 1);
          if (nfin == K && __ballot(xo != kNegInf && xo >= xt) != 0ull) {  // uniform
            // candidates left out may equal the K-th best score: its places go
            // to the lowest flat indices of all candidates with that score
            CTCBEAM_PHASE_COUNT(11);
            const int ngt = static_cast<int>(__popcll(__ballot(evalid && x > xt)));
            const int need = K - ngt;
            int have = 0;
            if (lane < kKmax) s_tie[lane] = static_cast<uint32_t>(V << 3);
            wave_lds_fence();
            for (int i = 0; i < K && have < need; ++i) {  // uniform
              const uint4 bi = s_beam[i];
              const float s = __uint_as_float(bi.x);
              const int l0 = static_cast<int>(bi.y);
              if (s == kNegInf) continue;  // dead position (uniform)
              for (int c0 = 0; c0 <= V && have < need; c0 += 64) {
                const int cc = c0 + lane;
                float y = kNegInf;
                if (cc <= V) {
                  y = s + row[cc];
                  if (cc < V && cc != l0) y = y + beta;
                }
                const uint64_t m = __ballot(y == xt);
                const int at = have + static_cast<int>(__popcll(m & lanemask_lt()));
                if (y == xt && at < need)
                  s_tie[at] = static_cast<uint32_t>(i | (cc << 3) | ((cc < V && cc != l0 ? 1 : 0) << 14) |
                                                    (static_cast<int>(bi.z) << 15));
                have += static_cast<int>(__popcll(m));
              }
            }
            wave_lds_fence();
            if (lane >= ngt && lane < K) {
              wx = xt;
              pk = static_cast<int>(s_tie[lane - ngt]);
            }
          }
          // the winners' transcripts, from their parents (slot k in lane k)
          const int from = ((pk >> 15) & 7) << 2;
          const uint32_t plo = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(hlo)));
          const uint32_t phi = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(from, static_cast<int>(hhi)));
          const int plen = __builtin_amdgcn_ds_bpermute(from, len);
          const bool em = ((pk >> 14) & 1) != 0;
          const uint64_t h0 = (static_cast<uint64_t>(phi) << 32) | plo;
          const uint64_t h1 = mix_token(h0, static_cast<uint32_t>((pk >> 3) & 2047));
          whlo = static_cast<uint32_t>(em ? h1 : h0);
          whhi = static_cast<uint32_t>((em ? h1 : h0) >> 32);
          wlen = plen + (em ? 1 : 0);
        }
        CTCBEAM_PHASE_MARK(3);
        CTCBEAM_PHASE_COUNT(9);
        const bool valid = lane < nfin;
        float xw = valid ? wx : kNegInf;
        const int wc = (pk >> 3) & 2047;
        const int par = (pk >> 15) & 7;
        const bool emit = valid && ((pk >> 14) & 1);
        // the label's value in the next frame of the batch
        const float dn = (f + 1 < nf) ? row[kRow + min(wc, V)] : 0.0f;

        // counters: the beams entering this frame
        if (want_stats && lane < K && sc != kNegInf) st_alive += 1u;

        // prune (Algorithm 1: below best - theta -> -inf)
        const float lim = rdlane(xw, 0) - p.theta;
        const uint64_t h = (static_cast<uint64_t>(whhi) << 32) | whlo;
        const int nlen = wlen;
        const int nlast = valid ? wc : V;
        if (valid && xw < lim) xw = kNegInf;
        if (want_stats && xw != kNegInf && emit) st_emit += 1u;
        CTCBEAM_PHASE_MARK(4);
        // recombination: same transcript hash, length and ends-in-blank flag as
        // a live lower slot (slots in lanes 0..7 of one 16-lane row)
        const bool alive0 = valid && xw != kNegInf;
        const uint32_t meta = (static_cast<uint32_t>(nlen) & 0x3FFFFFFFu) | ((nlast == V ? 1u : 0u) << 30);
        uint64_t rkey = h ^ (static_cast<uint64_t>(meta + 1u) * 0xD6E8FEB86659FD93ull);
        if (!alive0) rkey = ~0ull;
        const bool dup = detail::recomb_shifts<1, 7>(static_cast<uint32_t>(rkey), static_cast<uint32_t>(rkey >> 32)) && alive0;
        const bool alive = alive0 && !dup;
        CTCBEAM_PHASE_MARK(5);
        if (lane < K) s_bp[n & 1][f * K + lane] = valid ? ((par << 16) | wc) : -1;

        // the beam after this frame
        sc = alive ? xw : kNegInf;
        last = nlast;
        len = nlen;
        hlo = whlo;
        hhi = whhi;
        le = le_next;
        dblank = db_next;
        // as the next frame's scoring sees it: the live slots first, the
        // other positions score -inf
        const uint64_t am = __ballot(alive && lane < K);
        const int na = static_cast<int>(__popcll(am));
        const int below = static_cast<int>(__popcll(am & lanemask_lt()));
        const bool liv = alive && lane < K;
        if (lane < kKmax) {
          const int pos = liv ? below : na + lane - below;
          s_beam[pos] = make_uint4(__float_as_uint(liv ? sc : kNegInf), static_cast<uint32_t>(liv ? last : V),
                                   static_cast<uint32_t>(lane), __float_as_uint(dn));
          s_hash[pos] = make_uint4(hlo, hhi, static_cast<uint32_t>(len), 0u);
        }
        CTCBEAM_PHASE_MARK(6);
      }
      detail::lds_barrier();
      CTCBEAM_PHASE_MARK(7);
    }
  }
  __syncthreads();

  // ---- the order of the final hypotheses (wave 0) ----
  const bool nbest = p.nbest_scores != nullptr;
  // (without models the final score is the beam's; -inf for a dead slot)
  const float sj = (lane < K && sc > kNegInf) ? sc : kNegInf;
  if (wave == 0) {
    // rank: final score descending, lowest slot on ties (a NaN would leave
    // ranks without a slot)
    int rank = 0;
    for (int i = 0; i < K; ++i) {
      const float si = rdlane(sj, i);
      rank += (si > sj || (si == sj && i < lane)) ? 1 : 0;
    }
    const int bj = static_cast<int>(__builtin_ctzll(__ballot(lane < K && rank == 0)));
    const int nlen = (lane < K && sj != kNegInf) ? len : 0;
    if (nbest && lane < K) {
      p.nbest_scores[static_cast<size_t>(b) * K + rank] = sj;
      p.nbest_lengths[static_cast<size_t>(b) * K + rank] = nlen;
      s_nblen[rank] = nlen;
      s_nbrank[lane] = rank;
    }
    const float bsc = rdlane(sj, bj);
    const int blen = rdlane(len, bj);
    if (lane == 0) {
      s_best = bj;
      s_bestscore = bsc;
      s_bestlen = blen;
    }
    if (want_stats) {
      uint32_t a0 = st_alive, a3 = st_emit;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        a0 += __shfl_xor(a0, off);
        a3 += __shfl_xor(a3, off);
      }
      if (lane == 0) {
        int64_t* so = p.stats + static_cast<size_t>(b) * 8;
        so[0] = L;
        so[1] = a0;
        so[2] = 0;
        so[3] = 0;
        so[4] = 0;
        so[5] = 0;
        so[6] = a3;
        so[7] = 0;
      }
    }
  }
  __syncthreads();
  const int best = s_best;
  const float bscore = s_bestscore;
  const bool have = bscore != kNegInf;
  const int nout = have ? s_bestlen : 0;
  int32_t* ot = p.out_tokens ? p.out_tokens + static_cast<size_t>(b) * T : nullptr;
  if (ot)
    for (int tt = nout + tid; tt < T; tt += kST) ot[tt] = -1;
  if (tid == 0 && p.out_scores) {
    p.out_scores[b] = bscore;
    if (p.out_lengths) p.out_lengths[b] = nout;
  }
  int32_t* nbt = nbest ? p.nbest_tokens + static_cast<size_t>(b) * K * T : nullptr;
  if (nbest) {
    for (int r = 0; r < K; ++r) {
      const int n = s_nblen[r];
      for (int tt = n + tid; tt < T; tt += kST) nbt[static_cast<size_t>(r) * T + tt] = -1;
    }
  }

  // ---- traceback through the back-pointers, staged in LDS tiles ----
  // 1-best: lane 0 of wave 0 walks the best slot; N-best: lane k of wave 0
  // walks live slot k into the row of its rank
  const bool walker = wave == 0 && (nbest ? sj != kNegInf : (lane == 0 && have));
  if (have && L > 0) {
    uint32_t* stg = s_big;
    const int tile_frames = kStageWords / K;
    int jb = nbest ? lane : best, cnext = -1, pos = 0;
    int32_t* orow = nullptr;
    if (walker) {
      orow = nbest ? nbt + static_cast<size_t>(s_nbrank[lane]) * T : ot;
      pos = nbest ? len : nout;
    }
    for (int hi = L; hi > 0;) {
      const int lo = hi > tile_frames ? hi - tile_frames : 0;
      __syncthreads();
      const int n = (hi - lo) * K;
      const int32_t* src = bpb + static_cast<size_t>(lo) * K;
      for (int q = tid; q < n; q += kST) stg[q] = static_cast<uint32_t>(src[q]);
      __syncthreads();
      if (walker) {
        for (int tt = hi - 1; tt >= lo; --tt) {
          const uint32_t e = stg[(tt - lo) * K + jb];
          const int cl = static_cast<int>(e & 0xFFFFu);
          const int pr = static_cast<int>(e >> 16);
          if (tt < L - 1 && cnext != V && cnext != cl && pos > 0) {
            --pos;
            if (orow) orow[pos] = cnext;
          }
          cnext = cl;
          jb = pr < K ? pr : 0;  // a live slot's ancestors are live: pr < K (else the walk ends unbalanced)
        }
      }
      hi = lo;
    }
    if (walker && cnext != V && cnext >= 0 && pos > 0) {
      --pos;
      if (orow) orow[pos] = cnext;
    }
    if (wave == 0 && __ballot(walker && pos != 0) != 0ull) status |= 2u;
  }
#ifdef CTCBEAM_PHASE_CLOCKS
  CTCBEAM_PHASE_MARK(8);
  if (p.stats && lane < kPhaseWords) {
    int64_t* pw = p.stats + static_cast<size_t>(p.B) * 8 + (static_cast<size_t>(b) * 8 + wave) * kPhaseWords;
    pw[lane] = static_cast<int64_t>(ph_acc);
  }
#endif
  if (tid == 0) {
    p.status[b] = status;
    if (b == 0) write_ws_header(p.ws_header, p.B);
  }
}

template <int NJ>
hipError_t launch(const KernelParams& p, hipStream_t s) {
  hipLaunchKernelGGL(small_kernel<NJ>, dim3(p.B), dim3(kST), 0, s, p);
  return hipGetLastError();
}

}  // namespace small

// The small-beam decoder serves beams of at most 8 without an LM or boosting:
// the entries of K = 8 fill one wave's lanes, and a label's order in every beam
// is its order in D only where no model adds to it (0.43 against 1.72 ms in
// the general decoder at K = 8 on 32 utterances of 400 frames, V = 1024).
bool small_beam_eligible(const KernelParams& p) {
  if (p.bt_nodes != nullptr || p.lm_states != nullptr || p.lm_arcs != nullptr) return false;
  if (p.K > small::kKmax || p.V > small::kVmax) return false;
  return (p.flags & (kFlagNoRowCache | kFlagLogSumExp | kFlagRepeatScore)) == 0;
}

hipError_t launch_small(const KernelParams& p, hipStream_t s) {
  if (p.V <= 64) return small::launch<1>(p, s);
  if (p.V <= 256) return small::launch<4>(p, s);
  return small::launch<16>(p, s);
}

}  // namespace ctcbeam
