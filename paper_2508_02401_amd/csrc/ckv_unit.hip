// gfx950 (MI355X) top-N selection and retain/evict of CompressKV's
// prefill-end token selection (arXiv 2508.02401, Sec. 3.3: the tokens with the
// N highest averaged scores keep their KV pairs, the others are evicted), for
// a batch of layers in one launch or for one layer.
//
// After the pooling kernel has written the scores and first-level histograms,
// one workgroup of 512 threads takes a selection unit (layer, prompt,
// selection group) from the threshold to the compact cache, with no further
// kernel boundary or device-wide atomic:
//   1. the bin of the 4096-bin histogram (key bits 30..19) holding the N-th
//      largest key;
//   2. the exact threshold: the keys of that bin listed in LDS (when at most
//      kCandCap) and ranked there, or ranked by further histogram passes over
//      the scores, 12 bits at a time, until the threshold key is exact or
//      every key of the bin is kept;
//   3. two LDS bitmaps per segment of 131072 tokens, one of the kept keys
//      (above the threshold) and one of the keys equal to it; walking them in
//      token order keeps the lowest-index equal keys, writes the indices in
//      ascending order and copies their K/V rows (or leaves the copies to a
//      gather launch when the batch keeps many rows per unit).
// For a prompt of at most 131072 tokens whose threshold bin fits in LDS,
// steps 2 and 3 read the scores once: the same pass marks the keys above the
// bin and the bin's keys.
// One layer has few units (8 for 8 KV heads), so a unit is split into parts:
// each part's workgroup repeats steps 1 and 2, whose reads are a few hundred
// KB from L2, and writes and copies only its share of the kept rows.
// Keys are the fp32 bit patterns of the scores (scores >= 0, so integer
// order is score order); ties go to the lower token index.
#include "ckv_device.h"

namespace ckv {
namespace {

using namespace dev;

constexpr int kUT = 512;                   // threads per unit workgroup
constexpr int kUW = kUT / 64;              // its waves
constexpr int kCandCap = 8192;             // threshold-bin keys ranked in LDS
constexpr int kSegWords = 4096;            // bitmap words of one output segment
constexpr int kSegTokens = kSegWords * 32; // tokens of one output segment
constexpr int kUnitList = 1024;            // kept rows listed per copy round
constexpr int kScanLoads = 8;               // 16-byte score loads in flight per thread
constexpr int kScanBatch = 4 * kScanLoads;  // scores per thread of a scan batch
constexpr int kBatchTokens = kUT * kScanBatch;  // tokens of one scan batch
constexpr int kWaveTokens = 64 * kScanBatch;    // consecutive tokens of a wave in a batch
static_assert(kSegWords % kUT == 0 && kSegTokens == kUnitTokens, "bitmap words per thread");
static_assert(kHistBins % kUT == 0 && kSegTokens % kBatchTokens == 0, "whole batches");

struct UnitLds {
  uint32_t hist[kHistBins];
  uint2 cand[kCandCap];      // (key, token) of the threshold bin's keys
  alignas(16) uint32_t kmap[kSegWords];  // keys above the threshold
  alignas(16) uint32_t emap[kSegWords];  // keys equal to it
  int32_t ltok[kUnitList];
  uint32_t wsum[kUW];
  uint32_t res[3];
  uint32_t n_cand;
};

// Bin of an LDS histogram of nbins (<= kHistBins) bins holding the need-th
// largest key (1 <= need <= total count): res = (bin, keys in higher bins,
// keys in the bin), for every thread.
constexpr int kBinsPer = kHistBins / kUT;
__device__ void find_bin_unit(UnitLds& sm, int nbins, uint32_t need) {
  const int per = (nbins + kUT - 1) / kUT;
  const int top = nbins - 1 - per * (int)threadIdx.x;
  uint32_t c[kBinsPer];
  uint32_t local = 0;
#pragma unroll
  for (int i = 0; i < kBinsPer; ++i) {
    c[i] = i < per && top - i >= 0 ? sm.hist[top - i] : 0u;
    local += c[i];
  }
  uint32_t tot;
  const uint32_t above = block_excl_scan<kUT>(local, sm.wsum, tot);
  if (above < need && need <= above + local) {
    uint32_t run = above;
    bool found = false;
#pragma unroll
    for (int i = 0; i < kBinsPer; ++i) {
      if (!found && need <= run + c[i]) {
        sm.res[0] = (uint32_t)(top - i);
        sm.res[1] = run;
        sm.res[2] = c[i];
        found = true;
      }
      run += c[i];
    }
  }
  __syncthreads();
}

// The kernel runs each step once or twice, so a launch pays for the bytes of
// code it passes through (every 64 of them come from L2 first): one copy of
// each step, loops over inlined variants.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// A wave's 2048 consecutive scores of the batch at base: load k takes tokens
// 256 k + 4 lane .. + 3 of them (score rows are 4-byte aligned). Tokens at or
// past Ls get any score.
__device__ __forceinline__ void load_batch(const CKV_GLOBAL float* sc, int64_t base, int64_t Ls,
                                           f32x4* v) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const CKV_GLOBAL float* p = sc + base + wave * kWaveTokens;
  const int64_t left64 = Ls - base - wave * kWaveTokens;
  const int left = left64 > kWaveTokens ? kWaveTokens : (int)left64;  // scores of this wave
  if (left <= 0) return;
  if (left == kWaveTokens) {
#pragma unroll
    for (int k = 0; k < kScanLoads; ++k) v[k] = *(const CKV_GLOBAL f32x4u*)(p + k * 256 + 4 * lane);
    return;
  }
  // the row ends here: whole vectors inside it, then the one that straddles
  // the end (if any) score by score
  const int whole = left & ~3, rest = left & 3;
  if (whole > 0) {
#pragma unroll
    for (int k = 0; k < kScanLoads; ++k) {
      const int at = k * 256 + 4 * lane;
      v[k] = *(const CKV_GLOBAL f32x4u*)(p + (at < whole ? at : 0));
    }
  }
  if (rest > 0) {
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
    r.x = p[whole];
    if (rest > 1) r.y = p[whole + 1];
    if (rest > 2) r.z = p[whole + 2];
#pragma unroll
    for (int k = 0; k < kScanLoads; ++k)
      if (k * 256 + 4 * lane == whole) v[k] = r;
  }
}

// Adds the keys of [0, Ls) whose bits above `shift` equal prefix to an LDS
// histogram of their next bits, kHistLoads 16-byte loads in flight per thread.
constexpr int kHistLoads = 4;
__device__ __forceinline__ void hist_scores(UnitLds& sm, const CKV_GLOBAL float* sc, int64_t Ls,
                                            uint32_t prefix, int shift, int nshift, uint32_t nmask) {
  auto add = [&](float x) {
    const uint32_t key = score_key(x);
    if ((key >> shift) == prefix) atomicAdd(&sm.hist[(key >> nshift) & nmask], 1u);
  };
  const int64_t whole = Ls & ~(int64_t)3;
  if ((int64_t)threadIdx.x < Ls - whole) add(sc[whole + threadIdx.x]);
  for (int64_t j0 = 4 * (int64_t)threadIdx.x; j0 < whole; j0 += 4 * kUT * kHistLoads) {
    f32x4 v[kHistLoads];
#pragma unroll
    for (int k = 0; k < kHistLoads; ++k) {
      const int64_t j = j0 + k * 4 * kUT;
      v[k] = *(const CKV_GLOBAL f32x4u*)(sc + (j < whole ? j : j0));
    }
#pragma unroll
    for (int k = 0; k < kHistLoads; ++k)
      if (j0 + k * 4 * kUT < whole) {
        add(v[k].x);
        add(v[k].y);
        add(v[k].z);
        add(v[k].w);
      }
  }
}

// 8 x 8 transpose of the 4-bit pieces of m over each group of 8 lanes: lane s of
// the group gets piece s of lane 0 in bits 0..3, of lane 1 in bits 4..7, ...
__device__ __forceinline__ uint32_t transpose_nibbles(uint32_t m) {
  const int lane = threadIdx.x & 63;
  auto step = [&](int d, uint32_t low) {  // swap with the lane d away: `low` marks the kept low pieces
    const uint32_t o = __shfl_xor(m, d);
    const int sh = 4 * d;
    m = lane & d ? (m & ~low) | ((o & ~low) >> sh) : (m & low) | ((o & low) << sh);
  };
  step(1, 0x0F0F0F0Fu);
  step(2, 0x00FF00FFu);
  step(4, 0x0000FFFFu);
  return m;
}

// Marks a batch's scores: the bitmap words (from token seg0, below lim) of the
// tokens with bits(score) > hi go to kmap, of those from lo to hi to emap. A
// lane collects a bit per score and mask in registers, 4 per load, and eight
// lanes exchange their pieces into words of 32 consecutive tokens. Balloting
// per 64 keys and storing each row from one lane made 131072 scores take 33
// us.
__device__ __forceinline__ void mark_batch(UnitLds& sm, const f32x4* v, int64_t base, int64_t seg0,
                                           int64_t lim, int lo, int hi) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t above = 0, from = 0;
#pragma unroll
  for (int k = 0; k < kScanLoads; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int x = __float_as_int(v[k][i]);
      above |= x > hi ? 1u << (4 * k + i) : 0u;
      from |= x >= lo ? 1u << (4 * k + i) : 0u;
    }
  above = transpose_nibbles(above);
  from = transpose_nibbles(from);
  // this lane's word: tokens 256 (lane % 8) + 32 (lane / 8) .. + 31 of the wave's
  const int64_t t = base + wave * kWaveTokens + 256 * (lane & 7) + 32 * (lane >> 3);
  const int64_t left = lim - t;
  const uint32_t valid = left >= 32 ? ~0u : (left <= 0 ? 0u : (1u << left) - 1u);
  const int w = (int)((t - seg0) >> 5);
  sm.kmap[w] = above & valid;
  sm.emap[w] = from & ~above & valid;
}

// K and V rows tok[0 .. n) (tokens of the prompt) of KV head g to output rows
// row0 .. row0 + n - 1, kListCopies 16-byte pieces of each in flight per thread.
constexpr int kListCopies = 4;
__device__ __forceinline__ void copy_list(const LayerArgs& a, const SeqArgs& sq, int g, int row0,
                                          int n, const int32_t* tok) {
  const int nv = a.d * a.elt / 16;  // 8, 16 or 32 pieces per row
  const int nv_log2 = nv == 8 ? 3 : (nv == 16 ? 4 : 5);
  const int c = threadIdx.x & (nv - 1), rpt = kUT >> nv_log2;
  const int64_t rs = sq.kv_st * a.elt, head = (int64_t)g * sq.kv_sh * a.elt + c * 16;
  const CKV_GLOBAL char* kb = to_global(static_cast<const char*>(sq.k)) + head;
  const CKV_GLOBAL char* vb = to_global(static_cast<const char*>(sq.v)) + head;
  const int64_t o0 = (((int64_t)g * sq.n_ret + row0) << nv_log2) + c;
  CKV_GLOBAL u32x4* ko = to_global(static_cast<u32x4*>(sq.k_out)) + o0;
  CKV_GLOBAL u32x4* vo = to_global(static_cast<u32x4*>(sq.v_out)) + o0;
#pragma unroll 1
  for (int i0 = threadIdx.x >> nv_log2; i0 < n; i0 += rpt * kListCopies) {
    u32x4 kr[kListCopies], vr[kListCopies];
#pragma unroll
    for (int q = 0; q < kListCopies; ++q) {
      const int i = i0 + q * rpt;
      const int64_t off = tok[i < n ? i : i0] * rs;
      kr[q] = *(const CKV_GLOBAL u32x4*)(kb + off);
      vr[q] = *(const CKV_GLOBAL u32x4*)(vb + off);
    }
#pragma unroll
    for (int q = 0; q < kListCopies; ++q) {
      const int i = i0 + q * rpt;
      if (i < n) {
        ko[(int64_t)i << nv_log2] = kr[q];
        vo[(int64_t)i << nv_log2] = vr[q];
      }
    }
  }
}

// Marks every score of [seg0, lim) (at most kSegTokens) into the bitmaps of the
// segment, the words past it cleared. v holds the first batch; two batches are
// on the way while one is marked.
__device__ __forceinline__ void mark_segment(UnitLds& sm, const CKV_GLOBAL float* sc, f32x4* v,
                                             int64_t seg0, int64_t lim, uint32_t prefix, int shift) {
  const int scanned = (int)((lim - seg0 + kBatchTokens - 1) / kBatchTokens) * (kBatchTokens / 32);
  for (int i = scanned + threadIdx.x; i < kSegWords; i += kUT) sm.emap[i] = sm.kmap[i] = 0u;
  // bits of the scores whose key equals prefix above shift: lo .. hi. Negative
  // scores rank as 0, so prefix 0 takes them too.
  const int lo = prefix == 0 ? INT32_MIN : (int)(prefix << shift);
  const int hi = (int)(((prefix + 1) << shift) - 1u);
  f32x4 v1[kScanLoads] = {};
  if (seg0 + kBatchTokens < lim) load_batch(sc, seg0 + kBatchTokens, lim, v1);
#pragma unroll 1
  for (int64_t base = seg0; base < lim; base += kBatchTokens) {
    f32x4 v2[kScanLoads] = {};
    if (base + 2 * kBatchTokens < lim) load_batch(sc, base + 2 * kBatchTokens, lim, v2);
    mark_batch(sm, v, base, seg0, lim, lo, hi);
#pragma unroll
    for (int k = 0; k < kScanLoads; ++k) {
      v[k] = v1[k];
      v1[k] = v2[k];
    }
  }
  __syncthreads();
}

// Ranks the set bits of a bitmap: sm.hist[w] = bits below word w. Returns how
// many there are.
static_assert(kSegWords <= kHistBins, "word ranks fit in the histogram");
__device__ __forceinline__ uint32_t rank_words(UnitLds& sm, const uint32_t* map) {
  constexpr int kPer = kSegWords / kUT;
  uint32_t n[kPer], sum = 0, tot;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    n[i] = __popc(map[threadIdx.x * kPer + i]);
    sum += n[i];
  }
  uint32_t at = block_excl_scan<kUT>(sum, sm.wsum, tot);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    sm.hist[threadIdx.x * kPer + i] = at;
    at += n[i];
  }
  __syncthreads();
  return tot;
}

// Token of the segment whose bit is the r-th set one (r below the total): a
// search over the word ranks, then over the word. Every row finds its own
// token; walking a thread's 256 tokens bit by bit left most lanes idle, as
// kept tokens cluster.
__device__ __forceinline__ uint32_t token_of_rank(const UnitLds& sm, const uint32_t* map, uint32_t r) {
  uint32_t w = 0;  // last word with rank <= r
#pragma unroll 1
  for (uint32_t d = kSegWords / 2; d > 0; d >>= 1) w += sm.hist[w + d] <= r ? d : 0u;
  uint32_t m = map[w], n = r - sm.hist[w], t = w * 32;
#pragma unroll
  for (uint32_t d = 16; d > 0; d >>= 1) {
    const uint32_t c = __popc(m & ((1u << d) - 1u));
    if (n >= c) {
      n -= c;
      m >>= d;
      t += d;
    }
  }
  return t;
}

// Part `part` of n_parts of prompt s's selection unit g: the unit's output rows, KV
// head by KV head when the selection is shared, are dealt out in consecutive shares.
__device__ __forceinline__ void unit_body(const LayerArgs& a, int s, int g, int part, int n_parts,
                                          bool copy, UnitLds& sm) {
  const int tid = threadIdx.x;
  const SeqArgs& sq = a.seq[s];
  const int64_t Ls = sq.L - a.tail;
  const int n_ret = sq.n_ret;
  // ranked rows: 0 .. n_keep - 1; the rows after them are the tokens from
  // tail0 on (the window, kept by rule, or every token when the budget is L)
  const int n_keep = sq.n_keep < 0 ? 0 : sq.n_keep;
  const int tail0 = sq.n_keep < 0 ? 0 : (int)Ls;
  // the KV heads whose rows this selection keeps: its own, or all of them;
  // this part's heads gk0 .. gk1 and, on head gk, its rows row_a(gk) .. row_b(gk)
  const int h0 = a.shared ? 0 : g;
  const int64_t rows_all = (int64_t)(a.shared ? a.n_kv : 1) * n_ret;
  const int64_t m0 = rows_all * part / n_parts, m1 = rows_all * (part + 1) / n_parts;
  if (m0 >= m1) return;
  const int gk0 = h0 + (int)(m0 / n_ret), gk1 = h0 + (int)((m1 - 1) / n_ret) + 1;
  const int first_a = (int)(m0 - (int64_t)(gk0 - h0) * n_ret);
  const int last_b = (int)(m1 - (int64_t)(gk1 - 1 - h0) * n_ret);
  auto row_a = [&](int gk) { return gk == gk0 ? first_a : 0; };
  auto row_b = [&](int gk) { return gk == gk1 - 1 ? last_b : n_ret; };
  // the index row is written with the first head's rows
  const int ia = gk0 == h0 ? first_a : n_ret, ib = gk0 == h0 ? row_b(gk0) : n_ret;
  if (!copy && ia >= ib) return;
  const CKV_GLOBAL float* sc = to_global(sq.scores) + (int64_t)g * Ls;
  CKV_GLOBAL int32_t* out = to_global(sq.idx) + (int64_t)g * n_ret;
  // whether any of this part's rows is ranked (rows start below n_keep)
  const bool ranked = n_keep > 0 && (gk1 > gk0 + 1 || first_a < n_keep);

  // keys compare on (key >> shift) against prefix: those above are kept, and
  // of the cnt equal to it the `need` lowest-index ones
  uint32_t prefix = 0, need = 0, cnt = 0;
  int shift = kHistShift;
  constexpr int kPer = kSegWords / kUT;  // bitmap words per thread
  f32x4 v[kScanLoads];
  bool marked = false;
  if (ranked) {
    // 1. the first-level bin from the pooling kernel's histogram; the first
    // batch of scores is in flight meanwhile
    const CKV_GLOBAL uint32_t* ghist = to_global(sq.hist) + (int64_t)g * kHistBins;
    uint32_t hv[kHistBins / kUT];
#pragma unroll
    for (int k = 0; k < kHistBins / kUT; ++k) hv[k] = ghist[tid + k * kUT];
    load_batch(sc, 0, Ls, v);
#pragma unroll
    for (int k = 0; k < kHistBins / kUT; ++k) sm.hist[tid + k * kUT] = hv[k];
    __syncthreads();
    need = (uint32_t)n_keep;
    // 2. the exact threshold, level by level
    bool in_lds = false;
    int nb = kHistBits;
#pragma unroll 1
    for (;;) {
      find_bin_unit(sm, 1 << nb, need);
      prefix = (prefix << nb) | sm.res[0];
      need -= sm.res[1];
      cnt = sm.res[2];
      __syncthreads();
      if (!marked && Ls <= kSegTokens && (need == cnt || cnt <= (uint32_t)kCandCap)) {
        // the keys above the bin and the keys in it into the bitmaps, in one
        // pass; unless the whole bin is kept, the bin's tokens are listed in
        // token order and their keys read back
        mark_segment(sm, sc, v, 0, Ls, prefix, shift);
        marked = true;
        if (need < cnt && shift > 0) {
          rank_words(sm, sm.emap);
          for (uint32_t c = tid; c < cnt; c += kUT) {
            const uint32_t t = token_of_rank(sm, sm.emap, c);
            sm.cand[c] = make_uint2(score_key(sc[t]), t);
          }
          __syncthreads();
          for (int i = tid; i < kSegWords; i += kUT) sm.emap[i] = 0u;  // for the threshold's equals
          if (tid == 0) sm.n_cand = cnt;
          in_lds = true;
        }
      }
      if (shift == 0 || need >= cnt) break;
      nb = shift < 12 ? shift : 12;
      const int nshift = shift - nb;
      const uint32_t nmask = (1u << nb) - 1u;
      for (int i = tid; i <= (int)nmask; i += kUT) sm.hist[i] = 0u;
      __syncthreads();
      if (in_lds) {
        const uint32_t n = sm.n_cand;
        for (uint32_t c = tid; c < n; c += kUT) {
          const uint32_t key = sm.cand[c].x;
          if ((key >> shift) == prefix) atomicAdd(&sm.hist[(key >> nshift) & nmask], 1u);
        }
      } else {
        hist_scores(sm, sc, Ls, prefix, shift, nshift, nmask);
        load_batch(sc, 0, Ls, v);
      }
      __syncthreads();
      shift = nshift;
    }
    if (in_lds) {
      // the listed keys settle against the exact threshold: above it kept,
      // equal to it ranked by token
      const uint32_t n = sm.n_cand;
      for (uint32_t c = tid; c < n; c += kUT) {
        const uint2 e = sm.cand[c];
        const uint32_t p = e.x >> shift, bit = 1u << (e.y & 31u);
        if (p > prefix) atomicOr(&sm.kmap[e.y >> 5], bit);
        else if (p == prefix) atomicOr(&sm.emap[e.y >> 5], bit);
      }
      __syncthreads();
    }
  }

  // 3. ascending output, one segment of tokens at a time, then the rows after
  // the ranked ones
  uint32_t eq_carry = 0;
  int pos_carry = 0;
#pragma unroll 1
  for (int64_t seg0 = 0;; seg0 += kSegTokens) {
    const bool tail = !ranked || seg0 >= Ls || pos_carry >= n_keep;
    int lo = n_keep, hi = n_ret;  // rows of this step
    if (!tail) {
      if (!marked) {
        const int64_t seg1 = Ls - seg0 < kSegTokens ? Ls : seg0 + kSegTokens;
        if (seg0 > 0) load_batch(sc, seg0, seg1, v);
        mark_segment(sm, sc, v, seg0, seg1, prefix, shift);
      }
      // equal keys in token order: the first `need` are kept
      uint32_t em[kPer], ne = 0, tot_eq;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        em[i] = sm.emap[tid * kPer + i];
        ne += __popc(em[i]);
      }
      const uint32_t eq_rank = eq_carry + block_excl_scan<kUT>(ne, sm.wsum, tot_eq);
      uint32_t left = eq_rank < need ? need - eq_rank : 0u;
      if (ne > 0 && left > 0) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          uint32_t e = em[i], n = __popc(e);
          if (n > left) {  // drop the highest tokens past `left`
            uint32_t k = 0;
            for (; left > 0; --left, e &= e - 1u) k |= e & (0u - e);
            e = k;
            n = 0;
          }
          left -= n;
          sm.kmap[tid * kPer + i] |= e;
        }
      }
      eq_carry += tot_eq;
      const int kept = (int)rank_words(sm, sm.kmap);  // a thread reads the words that it wrote
      lo = pos_carry;
      hi = pos_carry + kept < n_keep ? pos_carry + kept : n_keep;
      pos_carry += kept;
    }
    // kUnitList rows of a head at a time: their tokens into LDS and the index
    // row (with the first head), then the copies
#pragma unroll 1
    for (int gk = gk0; gk < gk1; ++gk) {
      const int ra = row_a(gk) < lo ? lo : row_a(gk), rb = row_b(gk) < hi ? row_b(gk) : hi;
      if (!copy && gk != h0) break;
#pragma unroll 1
      for (int r0 = ra; r0 < rb; r0 += kUnitList) {
        const int r1 = rb - r0 < kUnitList ? rb : r0 + kUnitList;
        for (int r = r0 + tid; r < r1; r += kUT) {
          const int t = tail ? tail0 + r - n_keep
                             : (int)(seg0 + token_of_rank(sm, sm.kmap, (uint32_t)(r - lo)));
          sm.ltok[r - r0] = t;
          if (gk == h0) out[r] = t;
        }
        __syncthreads();
        if (copy) copy_list(a, sq, gk, r0, r1 - r0, sm.ltok);
        __syncthreads();
      }
    }
    if (tail) break;
  }
}

__global__ __launch_bounds__(kUT) void select_unit_kernel(const MultiArgs m) {
  __shared__ UnitLds sm;
  const int l = blockIdx.x / m.per_layer;
  const LayerArgs& a = layer_args(m, l);
  const int u = blockIdx.x - l * m.per_layer, s = u / a.n_sg;
  unit_body(a, s, u - s * a.n_sg, 0, 1, m.unit_copy != 0, sm);
}

// One layer, the parts of every unit as dealt out. Bound by its chain of dependent
// steps (a dozen barriers, three trips to memory): 13 us at 1024 tokens, 21 us at
// 32768 with 2048 rows of 8 heads kept, where filter, resolve and compact took
// 20 and 32 us. Two prompts of 24571 and 9001 tokens that share one selection
// for 8 heads had all copies made by the few ranges holding kept tokens: 58
// us, now 17 us.
__global__ __launch_bounds__(kUT) void select_parts_kernel(const LayerArgs a, const UnitParts p) {
  __shared__ UnitLds sm;
  args_ready(args_touch<sizeof(LayerArgs) + sizeof(UnitParts)>());
  const int b = blockIdx.x;
  int s = 0, u, part, parts = p.same;  // part of unit u of prompt s
  if (parts > 0) {
    u = b / parts;
    part = b - u * parts;
    s = u / a.n_sg;
    u -= s * a.n_sg;
  } else {
    while (s + 1 < a.num_seqs && b >= p.first[s + 1]) ++s;
    parts = p.parts[s];
    u = (b - p.first[s]) / parts;
    part = b - p.first[s] - u * parts;
  }
  unit_body(a, s, u, part, parts, a.do_gather != 0, sm);
}

}  // namespace

hipError_t launch_select_units(const MultiArgs& m, hipStream_t st, const Timing& tm) {
  return launch(select_unit_kernel, m.n_layers * m.per_layer, kUT, st, tm, m);
}

hipError_t launch_select_parts(const LayerArgs& a, const UnitParts& p, hipStream_t st, const Timing& tm) {
  void* args[] = {const_cast<LayerArgs*>(&a), const_cast<UnitParts*>(&p)};
  return hipExtLaunchKernel(reinterpret_cast<const void*>(select_parts_kernel),
                            dim3(p.first[a.num_seqs]), dim3(kUT), args, 0, st, tm.start, tm.stop, 0);
}

}  // namespace ckv
