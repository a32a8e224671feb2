// gfx950 (MI355X) kernels of CompressKV's layer-error profile (arXiv
// 2508.02401, Sec. 3.4, Eq. 6-8): decode attention of T query tokens over a
// full or a compressed KV cache, and the W_O-projected error ratio of every
// decoding step.
//
// decode_kernel: one workgroup per (KV head g, chunk of the cache), for up to
//   64 query rows (a group's G heads x T tokens, head-major) in 32-row blocks.
//   Each wave walks 32-key tiles of its own, staged in LDS that no other wave
//   touches, so the loop has no barrier. Per tile: S^T = K Q^T (keys x rows)
//   with MFMA, an online max and sum per row, P = exp2(S - m), O += P V with
//   MFMA. The waves' (max, sum, O) meet in LDS and leave as one partial.
// decode_rows_kernel_16 / _f32: the same for 65 to 128 query rows, a 32-row
//   block per wave and the key tiles shared by the workgroup.
// decode_merge_kernel: per (KV head, row): the chunks' partials rescaled to
//   the common max and summed, divided by the sum: out[t][h][:].
// project_kernel: Y = W_O X for the 2T columns X = [A_full | A_comp - A_full]
//   with fp32 MFMA, one workgroup per 32 rows of W_O and 32 columns, then the
//   column sums of Y^2 over its rows as one partial.
// error_kernel: the partials summed per column; ratio_t = sqrt(num_t) /
//   (sqrt(den_t) + eps) and e = sum_t ratio_t.
// Everything accumulates in fp32: the ratios compare two attention outputs
// that may differ in their third digit, which plain bf16 products would
// blur. fp32 inputs use fp32 MFMA (32x32x2); 16-bit inputs use 16-bit MFMA
// with the probabilities split into high and low parts.
#include <math.h>

#include "ckv_device.h"

namespace ckv {
namespace {

using namespace dev;

constexpr int kDecThreads = kDecodeThreads;
constexpr int kDecWaves = kDecThreads / 64;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <int DT>
__device__ __forceinline__ float elt_load(const void* base, int64_t i) {
  if constexpr (DT == 0) {
    const uint16_t u = static_cast<const CKV_GLOBAL uint16_t*>(to_global(static_cast<const uint16_t*>(base)))[i];
    return __uint_as_float((uint32_t)u << 16);
  } else if constexpr (DT == 1) {
    return (float)static_cast<const CKV_GLOBAL _Float16*>(to_global(static_cast<const _Float16*>(base)))[i];
  } else {
    return to_global(static_cast<const float*>(base))[i];
  }
}

// The 16 / element-bytes elements of a 16-byte piece, in fp32.
template <int DT>
__device__ __forceinline__ void unpack16(const u32x4 u, float* f) {
  if constexpr (DT == 2) {
    f[0] = __uint_as_float(u.x);
    f[1] = __uint_as_float(u.y);
    f[2] = __uint_as_float(u.z);
    f[3] = __uint_as_float(u.w);
  } else {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (DT == 0) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
      } else {
        f[2 * i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] & 0xFFFFu));
        f[2 * i + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] >> 16));
      }
    }
  }
}

// EPV = 16 / element-bytes consecutive elements at element offset off, in fp32.
template <int DT>
__device__ __forceinline__ void load_row16(const void* base, int64_t off, float* f) {
  unpack16<DT>(*reinterpret_cast<const CKV_GLOBAL u32x4*>(to_global(static_cast<const char*>(base)) +
                                                          off * Elt<DT>::bytes),
               f);
}

// ---------------------------------------------------------------------------
// Decode attention, one partial per (KV head, chunk).
// ---------------------------------------------------------------------------
// The (max in exp2 units, sum) pairs [n_kv][n_chunks][R] that follow a
// prompt's O partials [n_kv][n_chunks][R][d].
__device__ __forceinline__ float2* partial_ml(const DecodeArgs& a, int n_kv, int R, int D) {
  return reinterpret_cast<float2*>(a.part + (int64_t)n_kv * a.n_chunks * R * D);
}

template <int DT, int D>
__global__ __launch_bounds__(kDecThreads) void decode_rows_kernel_f32(const DecodeBatch B) {
  args_ready(args_touch<sizeof(DecodeBatch)>());
  constexpr int KB = 32;      // keys per block
  constexpr int KS = D + 1;   // LDS row stride: lanes reading one column of 32 rows hit 32 banks
  __shared__ float kl[KB * KS];  // K block [key][d], fp32
  __shared__ float vl[KB * KS];  // V block [key][d], fp32
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this workgroup's prompt (a uniform scan over at most kMaxDecodeSeqs)
  int si = 0;
  while (si + 1 < B.n && (int)blockIdx.x >= B.blk_off[si + 1]) ++si;
  const DecodeArgs& a = B.s[si];
  const int lb = (int)blockIdx.x - B.blk_off[si];
  const int g = lb / a.n_chunks, chunk = lb - g * a.n_chunks;
  const int G = B.H / B.n_kv;
  const int R = G * a.T;                    // query rows of the group
  const int qb = wave;                      // this wave's 32-row block of them
  const bool active = qb * 32 < R;
  const int64_t j0 = (int64_t)chunk * a.chunk;
  const int64_t j1 = j0 + a.chunk < a.n ? j0 + a.chunk : a.n;
  const int nkb = (int)((j1 - j0 + KB - 1) / KB);

  // this lane's query row (column of S^T and row of O): r = head-in-group * T + t
  const int r = qb * 32 + l32;
  const bool row_ok = active && r < R;
  float q[D / 2];  // lane half h holds elements 2i + h
  {
    const int hl = row_ok ? r / a.T : 0, t = row_ok ? r - (r / a.T) * a.T : 0;
    const int64_t qoff = (int64_t)t * a.q_st + (int64_t)(g * G + hl) * a.q_sh;
#pragma unroll
    for (int i = 0; i < D / 2; ++i) q[i] = row_ok ? elt_load<DT>(a.q, qoff + 2 * i + h) : 0.f;
  }
  f32x16 o[D / 32];
#pragma unroll
  for (int nb = 0; nb < D / 32; ++nb) o[nb] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  const float alpha = B.alpha;
  const int64_t kv_base = (int64_t)g * a.kv_sh;

  // K and V blocks of 32 keys go through LDS in fp32; each thread loads NLD
  // 16-byte pieces of both per block, and the next block's loads are issued
  // before the current block is reduced, so they overlap its MFMA work
  constexpr int EPV = 16 / Elt<DT>::bytes;              // elements per 16-byte load
  constexpr int NLD = KB * D / EPV / kDecThreads;       // loads per thread per block
  static_assert(NLD >= 1 && KB * D / EPV % kDecThreads == 0, "block loads");
  u32x4 kr[NLD], vr[NLD];
  auto issue = [&](int kb) {
    const int64_t t0 = j0 + (int64_t)kb * KB;
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e = tid + u * kDecThreads;
      const int key = e / (D / EPV), c = (e - key * (D / EPV)) * EPV;
      const int64_t tok = t0 + key < j1 ? t0 + key : j1 - 1;  // past the chunk: a valid row
      const int64_t off = (kv_base + tok * a.kv_st + c) * Elt<DT>::bytes;
      // each cache row is read once: non-temporal loads
      kr[u] = __builtin_nontemporal_load(reinterpret_cast<const CKV_GLOBAL u32x4*>(to_global(static_cast<const char*>(a.k)) + off));
      vr[u] = __builtin_nontemporal_load(reinterpret_cast<const CKV_GLOBAL u32x4*>(to_global(static_cast<const char*>(a.v)) + off));
    }
  };
  issue(0);
  for (int kb = 0; kb < nkb; ++kb) {
    const int64_t t0 = j0 + (int64_t)kb * KB;
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e = tid + u * kDecThreads;
      const int key = e / (D / EPV), c = (e - key * (D / EPV)) * EPV;
      const bool in = t0 + key < j1;  // keys past the chunk hold 0
      float kf[EPV], vf[EPV];
      unpack16<DT>(kr[u], kf);
      unpack16<DT>(vr[u], vf);
#pragma unroll
      for (int i = 0; i < EPV; ++i) {
        kl[key * KS + c + i] = in ? kf[i] : 0.f;
        vl[key * KS + c + i] = in ? vf[i] : 0.f;
      }
    }
    __syncthreads();
    if (kb + 1 < nkb) issue(kb + 1);
    if (active) {
      // S^T[key][row]: lane (row l32, half h) receives keys acc_row(v, h)
      f32x16 s = f32x16{};
#pragma unroll
      for (int i = 0; i < D / 2; ++i) s = mfma_f32(kl[l32 * KS + 2 * i + h], q[i], s);
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = acc_row(v, h);
        s[v] = t0 + key < j1 ? s[v] * alpha : -INFINITY;  // exp2 units
        mx = fmaxf(mx, s[v]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32));  // the row's max over both lane halves
      const float m_new = fmaxf(m_run, mx);
      const float resc = m_run == -INFINITY ? 0.f : exp2f(m_run - m_new);
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = m_new == -INFINITY ? 0.f : exp2f(s[v] - m_new);
        psum += s[v];
      }
      l_run = l_run * resc + psum;
      m_run = m_new;
#pragma unroll
      for (int nb = 0; nb < D / 32; ++nb) {
        // O^T[n][row] += V^T P^T: lane half h supplies key acc_row(v, h), the
        // key of its P value s[v]; the result's column is the lane's own row,
        // so the rescale is the lane's own
        f32x16 acc = o[nb] * resc;
#pragma unroll
        for (int v = 0; v < 16; ++v)
          acc = mfma_f32(vl[acc_row(v, h) * KS + nb * 32 + l32], s[v], acc);
        o[nb] = acc;
      }
    }
    __syncthreads();
  }
  if (!active) return;
  // the partial of this wave: (max, sum) per row, and O rows
  l_run += __shfl_xor(l_run, 32);
  if (!row_ok) return;
  const int64_t slot = (int64_t)g * a.n_chunks + chunk;
  if (h == 0) partial_ml(a, B.n_kv, R, D)[slot * R + r] = make_float2(m_run, l_run);
  float* part = a.part + (slot * R + r) * D;
  // o[nb][v]: O^T[nb*32 + acc_row(v, h)][row l32]
#pragma unroll
  for (int nb = 0; nb < D / 32; ++nb)
#pragma unroll
    for (int v = 0; v < 16; ++v) part[nb * 32 + acc_row(v, h)] = o[nb][v];
}

// 8 (16-bit) or 4 (fp32) fp32 values -> one operand chunk, and for 16-bit types
// the chunk of the rounded remainders.
template <int DT>
__device__ __forceinline__ void split_chunk(const float* x, uint4& hi, uint4& lo) {
  if constexpr (DT == 2) {
    hi = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]),
                    __float_as_uint(x[3]));
  } else if constexpr (DT == 0) {
    bf16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h[i] = (__bf16)x[i];
      l[i] = (__bf16)(x[i] - (float)h[i]);
    }
    hi = __builtin_bit_cast(uint4, h);
    lo = __builtin_bit_cast(uint4, l);
  } else {
    f16x8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      h[i] = (_Float16)x[i];
      l[i] = (_Float16)(x[i] - (float)h[i]);
    }
    hi = __builtin_bit_cast(uint4, h);
    lo = __builtin_bit_cast(uint4, l);
  }
}

// 16-bit inputs (bf16, f16): the same decode with 16-bit MFMA (32x32x16) at
// fp32-level accuracy. Q, K and V are exact in the MFMA type; the
// probabilities are split into a high part (rounded to the type) and a low
// part (the rounded remainder), and O += P V is the sum of two MFMAs, which
// leaves a relative error near 2^-16 (bf16) or 2^-22 (f16) instead of
// 2^-8 or 2^-11.
// Blocks of 64 keys keep the staging registers small enough for two
// workgroups per CU (two waves per SIMD): one workgroup reduces a block while
// the other's loads are in flight.
template <int DT, int D>
__global__ __launch_bounds__(kDecThreads) __attribute__((amdgpu_waves_per_eu(2)))
void decode_rows_kernel_16(const DecodeBatch B) {
  args_ready(args_touch<sizeof(DecodeBatch)>());
  constexpr int SB = 32;              // keys per MFMA tile (a sub-block)
  constexpr int NSB = 2;              // sub-blocks staged per block
  constexpr int KB = SB * NSB;        // keys per block
  constexpr int NC = D / 16;          // 16-element contraction chunks of a row
  constexpr int KROW = D * 2 + 16;    // K and V row bytes in LDS, padded by one 16-byte chunk
  __shared__ __align__(16) unsigned char kl[KB * KROW];  // K block [key][d], raw 16-bit
  __shared__ __align__(16) unsigned char vl[KB * KROW];  // V block [key][d], raw 16-bit
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this workgroup's prompt (a uniform scan over at most kMaxDecodeSeqs)
  int si = 0;
  while (si + 1 < B.n && (int)blockIdx.x >= B.blk_off[si + 1]) ++si;
  const DecodeArgs& a = B.s[si];
  const int lb = (int)blockIdx.x - B.blk_off[si];
  const int g = lb / a.n_chunks, chunk = lb - g * a.n_chunks;
  const int G = B.H / B.n_kv;
  const int R = G * a.T;
  const int qb = wave;  // this wave's 32-row block of the query rows
  const bool active = qb * 32 < R;
  const int64_t j0 = (int64_t)chunk * a.chunk;
  const int64_t j1 = j0 + a.chunk < a.n ? j0 + a.chunk : a.n;
  const int nkb = (int)((j1 - j0 + KB - 1) / KB);

  // query row r = head-in-group * T + t; lane half h holds elements
  // 16c + 8h .. 16c + 8h + 7 of it (exact: queries have the MFMA's type)
  const int r = qb * 32 + l32;
  const bool row_ok = active && r < R;
  uint4 qh[NC];
  {
    const int hl = row_ok ? r / a.T : 0, t = row_ok ? r - (r / a.T) * a.T : 0;
    const int64_t qoff = (int64_t)t * a.q_st + (int64_t)(g * G + hl) * a.q_sh;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const u32x4 x = *reinterpret_cast<const CKV_GLOBAL u32x4*>(
          to_global(static_cast<const char*>(a.q)) + (qoff + 16 * c + 8 * h) * 2);
      qh[c] = row_ok ? make_uint4(x.x, x.y, x.z, x.w) : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  f32x16 o[D / 32];
#pragma unroll
  for (int nb = 0; nb < D / 32; ++nb) o[nb] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  const float alpha = B.alpha;
  const int64_t kv_base = (int64_t)g * a.kv_sh;

  // every block of KB keys is staged by all threads (16-byte loads, the next
  // block's issued before the current one is reduced)
  constexpr int NLD = KB * D / 8 / kDecThreads;  // 16-byte loads per thread per block
  static_assert(NLD >= 1 && KB * D / 8 % kDecThreads == 0, "block loads");
  u32x4 kr[NLD], vr[NLD];
  auto issue = [&](int kb) {
    const int64_t t0 = j0 + (int64_t)kb * KB;
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e = tid + u * kDecThreads;
      const int key = e / (D / 8), c = (e - key * (D / 8)) * 8;
      const int64_t tok = t0 + key < j1 ? t0 + key : j1 - 1;  // past the chunk: a valid row
      const int64_t off = (kv_base + tok * a.kv_st + c) * 2;
      // each cache row is read once: non-temporal loads
      kr[u] = __builtin_nontemporal_load(reinterpret_cast<const CKV_GLOBAL u32x4*>(to_global(static_cast<const char*>(a.k)) + off));
      vr[u] = __builtin_nontemporal_load(reinterpret_cast<const CKV_GLOBAL u32x4*>(to_global(static_cast<const char*>(a.v)) + off));
    }
  };
  issue(0);
  for (int kb = 0; kb < nkb; ++kb) {
    const int64_t t0 = j0 + (int64_t)kb * KB;
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
      const int e = tid + u * kDecThreads;
      const int key = e / (D / 8), c = (e - key * (D / 8)) * 8;
      const bool in = t0 + key < j1;  // keys past the chunk hold 0
      const u32x4 kz = in ? kr[u] : u32x4{0u, 0u, 0u, 0u};
      const u32x4 vz = in ? vr[u] : u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(kl + key * KROW + c * 2) = kz;
      *reinterpret_cast<u32x4*>(vl + key * KROW + c * 2) = vz;
    }
    __syncthreads();
    if (kb + 1 < nkb) issue(kb + 1);
    for (int sb = 0; active && sb < NSB; ++sb) {
      const int64_t ts = t0 + sb * SB;  // first key of the sub-block
      if (ts >= j1) break;
      // S^T[key][row] = K Q^T; lane (row l32, half h) receives keys
      // acc_row(v, h) of the sub-block
      f32x16 s = f32x16{};
      const unsigned char* krow = kl + (sb * SB + l32) * KROW;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const uint4 kc = *reinterpret_cast<const uint4*>(krow + (16 * c + 8 * h) * 2);
        s = mfma_chunk<DT>(kc, qh[c], s);
      }
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = ts + acc_row(v, h) < j1 ? s[v] * alpha : -INFINITY;  // exp2 units
        mx = fmaxf(mx, s[v]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float resc = m_run == -INFINITY ? 0.f : fast_exp2(m_run - m_new);
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = fast_exp2(s[v] - m_new);
        psum += s[v];
      }
      l_run = l_run * resc + psum;
      m_run = m_new;
      // P^T operands: MFMA step m takes this lane's keys acc_row(8m .. 8m+7, h)
      // = 16m + 4h + (0..3) and 16m + 8 + 4h + (0..3), in that order
      uint4 ph[2], pl[2];
      {
        float p0[8], p1[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          p0[i] = s[i];
          p1[i] = s[8 + i];
        }
        split_chunk<DT>(p0, ph[0], pl[0]);
        split_chunk<DT>(p1, ph[1], pl[1]);
      }
#pragma unroll
      for (int nb = 0; nb < D / 32; ++nb) {
        // O^T[n][row] += V^T P^T: lane (n = nb*32 + l32, half h) supplies V of
        // the same 8 keys, gathered from the row-major tile (the lanes of a
        // half read 32 consecutive elements of one key row)
        f32x16 acc = o[nb] * resc;
        const unsigned char* vcol = vl + (sb * SB) * KROW + (nb * 32 + l32) * 2;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          uint32_t e[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int key = 16 * m + 8 * (j >> 2) + 4 * h + (j & 3);
            e[j] = *reinterpret_cast<const uint16_t*>(vcol + key * KROW);
          }
          const uint4 va = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16,
                                      e[6] | e[7] << 16);
          acc = mfma_chunk<DT>(va, ph[m], acc);
          acc = mfma_chunk<DT>(va, pl[m], acc);
        }
        o[nb] = acc;
      }
    }
    __syncthreads();
  }
  if (!active) return;
  l_run += __shfl_xor(l_run, 32);
  if (!row_ok) return;
  const int64_t slot = (int64_t)g * a.n_chunks + chunk;
  if (h == 0) partial_ml(a, B.n_kv, R, D)[slot * R + r] = make_float2(m_run, l_run);
  float* part = a.part + (slot * R + r) * D;
#pragma unroll
  for (int nb = 0; nb < D / 32; ++nb)
#pragma unroll
    for (int v = 0; v < 16; ++v) part[nb * 32 + acc_row(v, h)] = o[nb][v];
}

// Wait until at most n vector-memory operations of this wave are outstanding
// and its LDS operations are done; nothing is moved across.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x070 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

// exp2 of a logit's distance to the maximum. fp32 caches keep weights below
// 2^-126, which the bare instruction flushes to zero; V may be that large. The
// 16-bit types' weights are rounded to high and low parts that end sooner.
template <int DT>
__device__ __forceinline__ float weight_exp2(float x) {
  return DT == 2 ? exp2f(x) : fast_exp2(x);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));

// Up to 32 * NQ query rows. A cache row is read once, so the bound is the
// stream: what counts is how much of it is in flight and that no wave waits
// for another. Every wave therefore owns its tiles: 32 keys of K and of V go
// straight from memory into the wave's part of LDS, and the next tile's K is
// requested as soon as this tile's K is in registers, before its contraction
// (the same for V), so a CU has 64 to 128 KB requested nearly all the time. V
// is transposed for the second contraction by ds_read_b64_tr_b16 (16 reads a
// tile; gathering it with 2-byte reads took 64 and as many packs). The waves'
// results are added in LDS, and only rows that exist are written out.
// Shared 64-key blocks behind two barriers, with half the waves idle at up to
// 32 rows and a 32-row partial per wave, took 122 us + 27 us for the merge on
// four caches of 8192 to 98304 tokens (403 MB of K and V); this takes 64 + 5 us,
// 6.3 TB/s.
template <int DT, int D, int NQ>
__global__ __launch_bounds__(kDecThreads) __attribute__((amdgpu_waves_per_eu(DT != 2 && NQ == 1 ? 2 : 1)))
void decode_kernel(const DecodeBatch B) {
  constexpr int EB = Elt<DT>::bytes;
  constexpr int ROWB = D * EB;       // bytes per cache row
  constexpr int NV = ROWB / 16;      // 16-byte chunks per row: 8, 16 or 32
  constexpr int NC = NV / 2;         // operand chunks per lane
  constexpr int KT = 32;             // keys per tile
  constexpr int VEC = KT * NV;       // 16-byte chunks per tile
  constexpr int PT = VEC / 64;       // load instructions per tile
  constexpr int RPL = 64 / NV;       // tile rows per load instruction
  constexpr int NB = D / 32;
  __shared__ uint4 kl[kDecWaves][VEC];  // chunk c of row t at position c ^ swz(t)
  __shared__ uint4 vl[kDecWaves][VEC];
  __shared__ float2 ml[kDecWaves][32];
  const uint32_t touched = args_touch<sizeof(DecodeBatch)>();
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int si = 0;
  while (si + 1 < B.n && (int)blockIdx.x >= B.blk_off[si + 1]) ++si;
  const DecodeArgs& a = B.s[si];
  const int lb = (int)blockIdx.x - B.blk_off[si];
  const int g = lb / a.n_chunks, chunk = lb - g * a.n_chunks;
  const int G = B.H / B.n_kv;
  const int R = G * a.T;
  const int64_t j0 = (int64_t)chunk * a.chunk;
  const int64_t j1 = j0 + a.chunk < a.n ? j0 + a.chunk : a.n;
  const int nt = (int)((j1 - j0 + KT - 1) / KT);
  const int64_t rs = a.kv_st * EB;
  const char* kbase = static_cast<const char*>(a.k) + ((int64_t)g * a.kv_sh + j0 * a.kv_st) * EB;
  const char* vbase = static_cast<const char*>(a.v) + ((int64_t)g * a.kv_sh + j0 * a.kv_st) * EB;
  const int rows = (int)(j1 - j0);
  const float alpha = B.alpha;
  args_ready(touched);

  auto swz = [](int t) { return ROWB >= 256 ? (t & 15) : ((t >> 1) & 7); };
  // load i of a tile brings rows i * RPL .. + RPL - 1; this lane's chunk of row
  // t goes to position lane % NV, so it is chunk (lane % NV) ^ swz(t)
  const int lrow = lane / NV, lpos = lane % NV;
  const int64_t lane_off = lrow * rs;
  // tile tl of base: non-temporal, each cache row is read once. Rows past the
  // chunk read its last row instead.
  auto fetch = [&](const char* base, int tl, uint4* slot) {
    const char* tb = base + (int64_t)tl * KT * rs;
    if (tl * KT + KT <= rows) {
#pragma unroll
      for (int i = 0; i < PT; ++i)
        __builtin_amdgcn_global_load_lds(
            reinterpret_cast<const uint4*>(tb + (int64_t)i * RPL * rs + lane_off +
                                           (lpos ^ swz(i * RPL + lrow)) * 16),
            slot + i * 64, 16, 0, 2);
    } else {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int t = i * RPL + lrow;
        const int tc = tl * KT + t < rows ? t : rows - 1 - tl * KT;
        __builtin_amdgcn_global_load_lds(
            reinterpret_cast<const uint4*>(tb + tc * rs + (lpos ^ swz(t)) * 16), slot + i * 64, 16,
            0, 2);
      }
    }
  };
  int tile = wave;
  if (tile < nt) {
    fetch(kbase, tile, kl[wave]);
    fetch(vbase, tile, vl[wave]);
  }

  // query row r = head-in-group * T + t; lane half h holds chunks 2c + h of it,
  // 16-bit queries exactly (alpha is applied to the logits)
  uint4 q[NQ][NC];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int r = j * 32 + l32;
    const bool row_ok = r < R;
    const int hl = row_ok ? r / a.T : 0, t = row_ok ? r - hl * a.T : 0;
    const int64_t qoff = ((int64_t)t * a.q_st + (int64_t)(g * G + hl) * a.q_sh) * EB;
    const CKV_GLOBAL u32x4* src =
        (const CKV_GLOBAL u32x4*)(to_global(static_cast<const char*>(a.q)) + qoff) + h;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const u32x4 x = src[2 * c];
      q[j][c] = row_ok ? make_uint4(x.x, x.y, x.z, x.w) : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  f32x16 o[NQ][NB];
  float m_run[NQ], l_run[NQ];  // the maximum in exp2 units
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) o[j][nb] = f32x16{};
    m_run[j] = -INFINITY;
    l_run[j] = 0.f;
  }
  // byte offset of V chunk column group (nb, jj) in a 16-key half of the tile:
  // lane i of a 16-lane group reads columns 4 * (i % 4) .. + 3 of key
  // 8 * jj + 4 * h + i / 4, and receives column i of the 4 keys
  const int i16 = lane & 15;
  auto v_off = [&](int nb, int jj) {
    const int key = 8 * jj + 4 * h + (i16 >> 2);
    const int col = nb * 32 + (lane & 16) + 4 * (i16 & 3);
    return key * ROWB + ((col >> 3) ^ swz(key)) * 16 + (col & 7) * 2;
  };

  for (; tile < nt; tile += kDecWaves) {
    const bool more = tile + kDecWaves < nt;
    wait_vm<PT>();  // this tile's K; its V may still be on the way
    uint4 kr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) kr[c] = kl[wave][l32 * NV + ((2 * c + h) ^ swz(l32))];
    wait_vm<63>();  // K is in registers: its part of LDS is free
    if (more) fetch(kbase, tile + kDecWaves, kl[wave]);
    const int left = rows - tile * KT;  // keys of this tile that exist, if below KT
    f32x16 s[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) s[j] = f32x16{};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int j = 0; j < NQ; ++j) s[j] = mfma_chunk<DT>(kr[c], q[j][c], s[j]);
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      if (left < KT) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (acc_row(v, h) >= left) s[j][v] = -INFINITY;
      }
      float mx = s[j][0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[j][v]);
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      // the scaled maximum is kept as rounded: it must be the very number that
      // the weights below were and will be taken against, so that a row whose
      // maximum stays is rescaled by exactly 1 when another row's moves. A
      // product rounded anew, m * alpha inside a fused multiply-add, is off by
      // its rounding error, the same way at every rescale: 3e-4 of the result
      // after 256 tiles at logits up to 255
      const float m_new = fmaxf(m_run[j], mx * alpha);
      const float ms = m_new == -INFINITY ? 0.f : m_new;
      if (__any(m_new > m_run[j])) {  // some row's maximum moved: rescale
        const float resc = m_run[j] == -INFINITY ? 0.f : weight_exp2<DT>(m_run[j] - m_new);
        l_run[j] *= resc;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) o[j][nb] *= resc;
        m_run[j] = m_new;
      }
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[j][v] = weight_exp2<DT>(fmaf(s[j][v], alpha, -ms));
        psum += s[j][v];
      }
      l_run[j] += psum;
    }
    if (more) wait_vm<PT>();  // this tile's V; the next K may still be on the way
    else wait_vm<0>();
    if (left < KT) {  // rows past the chunk count as zeros
#pragma unroll
      for (int i = 0; i < PT; ++i)
        if (i * RPL + lrow >= left) vl[wave][i * 64 + lane] = make_uint4(0u, 0u, 0u, 0u);
      wait_vm<63>();
    }
    const char* vt = reinterpret_cast<const char*>(vl[wave]);
    if constexpr (DT != 2) {
      // P^T operands: MFMA step m takes this lane's keys acc_row(8m .. 8m+7, h)
      // = 16m + 4h + (0..3) and 16m + 8 + 4h + (0..3), in that order
      uint4 vr[2][NB];
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          typedef __attribute__((address_space(3))) s16x4* LdsPtr;
          const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (LdsPtr)(vt + v_off(nb, 0) + m * 16 * ROWB));
          const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (LdsPtr)(vt + v_off(nb, 1) + m * 16 * ROWB));
          const uint2 a2 = __builtin_bit_cast(uint2, lo4), b2 = __builtin_bit_cast(uint2, hi4);
          vr[m][nb] = make_uint4(a2.x, a2.y, b2.x, b2.y);
        }
      wait_vm<63>();  // V is in registers
      if (more) fetch(vbase, tile + kDecWaves, vl[wave]);
#pragma unroll
      for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          float p[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) p[i] = s[j][8 * m + i];
          uint4 ph, pl;
          split_chunk<DT>(p, ph, pl);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) o[j][nb] = mfma_chunk<DT>(vr[m][nb], ph, o[j][nb]);
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) o[j][nb] = mfma_chunk<DT>(vr[m][nb], pl, o[j][nb]);
        }
    } else {
      auto v_elem = [&](int v, int nb) {
        const int key = acc_row(v, h), col = nb * 32 + l32;
        return *reinterpret_cast<const float*>(vt + key * ROWB + ((col >> 2) ^ swz(key)) * 16 +
                                               (col & 3) * 4);
      };
      if constexpr (NQ == 1) {
        float vr[16][NB];
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) vr[v][nb] = v_elem(v, nb);
        wait_vm<63>();
        if (more) fetch(vbase, tile + kDecWaves, vl[wave]);
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) o[0][nb] = mfma_f32(vr[v][nb], s[0][v], o[0][nb]);
      } else {
        // the fp32 queries and outputs of two query blocks leave no registers
        // for a whole tile of V: it is read along, and requested after
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const float x = v_elem(v, nb);
#pragma unroll
            for (int j = 0; j < NQ; ++j) o[j][nb] = mfma_f32(x, s[j][v], o[j][nb]);
          }
        wait_vm<63>();
        if (more) fetch(vbase, tile + kDecWaves, vl[wave]);
      }
    }
  }

  // the waves' results, rescaled to the common maximum and added in wave order,
  // one query block at a time through the tiles' LDS. A wave's O^T (32 rows of
  // D floats) fills its K and V parts when elements are 2 bytes (columns below
  // and from D / 2), its K part when they are 4. 16-byte chunks of row r are
  // XOR-ed with r % 8.
  constexpr int OC = EB == 2 ? D / 8 : D / 4;  // 16-byte chunks of a row in one part
  float2* pml = partial_ml(a, B.n_kv, R, D);
  const int64_t slot = (int64_t)g * a.n_chunks + chunk;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    if (j * 32 >= R) break;
    __syncthreads();
    const float l = l_run[j] + __shfl_xor(l_run[j], 32);
    if (h == 0)
      ml[wave][l32] = make_float2(m_run[j], l);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int c = nb * 8 + v4 * 2 + h;  // chunk of the row: columns 4c .. 4c + 3
        float4* part = reinterpret_cast<float4*>(c < OC ? kl[wave] : vl[wave]);
        part[l32 * OC + ((c % OC) ^ (l32 & 7))] =
            make_float4(o[j][nb][4 * v4], o[j][nb][4 * v4 + 1], o[j][nb][4 * v4 + 2],
                        o[j][nb][4 * v4 + 3]);
      }
    __syncthreads();
    const int n_rows = R - j * 32 < 32 ? R - j * 32 : 32;
    for (int e = tid; e < n_rows * (D / 4); e += kDecThreads) {
      const int rr = e / (D / 4), c = e - rr * (D / 4), r = j * 32 + rr;
      float m = ml[0][rr].x;
#pragma unroll
      for (int w = 1; w < kDecWaves; ++w) m = fmaxf(m, ml[w][rr].x);
      float ls = 0.f;
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < kDecWaves; ++w) {
        const float2 x = ml[w][rr];
        if (x.x == -INFINITY) continue;  // a wave without keys
        const float f = exp2f(x.x - m);
        const float4* part = reinterpret_cast<const float4*>(c < OC ? kl[w] : vl[w]);
        const float4 y = part[rr * OC + ((c % OC) ^ (rr & 7))];
        ls += x.y * f;
        acc.x += y.x * f;
        acc.y += y.y * f;
        acc.z += y.z * f;
        acc.w += y.w * f;
      }
      if (a.direct) {  // the only chunk: the result itself (4-byte aligned)
        const int hl = r / a.T, t = r - hl * a.T;
        float* out = a.out + ((int64_t)t * B.H + g * G + hl) * D + 4 * c;
        out[0] = acc.x / ls;
        out[1] = acc.y / ls;
        out[2] = acc.z / ls;
        out[3] = acc.w / ls;
      } else {
        *reinterpret_cast<float4*>(a.part + (slot * R + r) * D + 4 * c) = acc;
        if (c == 0) pml[slot * R + r] = make_float2(m, ls);
      }
    }
  }
}

// out[t][h][:] from the chunks' partials, one workgroup per (prompt, query
// row): D / 4 lanes take four columns each, and the 256 / (D / 4) thread groups
// take every such chunk in turn with U of them in flight, then meet in LDS in a
// fixed order. One thread per output walking all slots 16 at a time was a
// chain of up to 16 trips to memory (27 us for four caches of 8192 to 98304
// tokens, now 4.6 us).
template <int D>
__global__ __launch_bounds__(kDecThreads) void decode_merge_kernel(const DecodeBatch B) {
  constexpr int C4 = D / 4, NG = kDecThreads / C4, U = 8;
  __shared__ float4 acc_l[NG][C4];
  __shared__ float2 ml_l[NG];
  args_ready(args_touch<sizeof(DecodeBatch)>());
  int si = 0;
  while (si + 1 < B.n && (int)blockIdx.x >= B.mrg_off[si + 1]) ++si;
  const DecodeArgs& a = B.s[si];
  const int G = B.H / B.n_kv;
  const int R = G * a.T;
  const int lr = (int)blockIdx.x - B.mrg_off[si];
  const int g = lr / R, r = lr - g * R;
  const int c = threadIdx.x % C4, ng = threadIdx.x / C4;
  const int n = a.n_chunks;
  const CKV_GLOBAL f32x4* po =
      (const CKV_GLOBAL f32x4*)to_global(a.part) + ((int64_t)g * n * R + r) * C4 + c;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const CKV_GLOBAL f32x2* pm =
      (const CKV_GLOBAL f32x2*)to_global(partial_ml(a, B.n_kv, R, D)) + (int64_t)g * n * R + r;
  // running maximum: the sums are rescaled whenever a chunk's exceeds it
  float m = -INFINITY, l = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = ng; s0 < n; s0 += NG * U) {
    f32x2 x[U];
    f32x4 y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s0 + u * NG < n ? s0 + u * NG : s0;
      x[u] = pm[(int64_t)s * R];
      y[u] = po[(int64_t)s * R * C4];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u * NG >= n || x[u].x == -INFINITY) continue;
      if (x[u].x > m) {
        const float f = exp2f(m - x[u].x);  // 0 while nothing has been added
        l *= f;
        acc *= f;
        m = x[u].x;
      }
      const float f = exp2f(x[u].x - m);
      l += x[u].y * f;
      acc += y[u] * f;
    }
  }
  acc_l[ng][c] = make_float4(acc.x, acc.y, acc.z, acc.w);
  if (c == 0) ml_l[ng] = make_float2(m, l);
  __syncthreads();
  if (threadIdx.x >= D) return;
  // thread d adds column d of every group
  const int d = threadIdx.x;
  float mm = ml_l[0].x;
#pragma unroll
  for (int i = 1; i < NG; ++i) mm = fmaxf(mm, ml_l[i].x);
  float ls = 0.f, s = 0.f;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    if (ml_l[i].x == -INFINITY) continue;
    const float f = exp2f(ml_l[i].x - mm);
    ls += ml_l[i].y * f;
    s += reinterpret_cast<const float*>(&acc_l[i][d / 4])[d & 3] * f;
  }
  const int hl = r / a.T, t = r - hl * a.T;
  a.out[((int64_t)t * B.H + g * G + hl) * D + d] = s / ls;
}

// ---------------------------------------------------------------------------
// Projection and error ratios.
// ---------------------------------------------------------------------------
// Workgroup (row block rb, column block cb, K range ks): the 32 x 32 tile of
// Y = W X over the ks-th of n_split K ranges, that range split over the
// workgroup's waves, the waves' sums added in LDS in a fixed order and the
// tile written to part_y. K is taken 16 at a time: lane half h holds
// k0 + 8h .. k0 + 8h + 7 of its W row (one 16-byte load for 2-byte weights)
// and of its X column, and MFMA m pairs k0 + m with k0 + 8 + m. K is a
// multiple of 16 (H * d with d in {64, 128}).
constexpr int kProjThreads = 256;
constexpr int kProjWaves = kProjThreads / 64;

template <int DT>
__global__ __launch_bounds__(kProjThreads) void project_kernel(const ErrorArgs a) {
  __shared__ float red[kProjWaves][32][33];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = tid >> 6;
  const int rb = blockIdx.x, cb = blockIdx.y, ks = blockIdx.z;
  const int row = rb * 32 + l32, col = cb * 32 + l32;
  const int rrow = row < a.D ? row : a.D - 1;  // rows past D compute a copy, not used
  const int T = a.T;
  const bool full_col = col < T, diff_col = col >= T && col < 2 * T;
  const int tcol = full_col ? col : (diff_col ? col - T : 0);
  const int64_t n16 = a.K / 16;
  const int64_t per_ks = (n16 + a.n_split - 1) / a.n_split;
  const int64_t k0 = ks * per_ks, k1 = k0 + per_ks < n16 ? k0 + per_ks : n16;
  const int64_t per = (k1 - k0 + kProjWaves - 1) / kProjWaves;
  const int64_t b0 = k0 + wave * per, b1 = b0 + per < k1 ? b0 + per : k1;
  const CKV_GLOBAL float* af = to_global(a.a_full) + (int64_t)tcol * a.K;
  const CKV_GLOBAL float* ac = to_global(a.a_comp) + (int64_t)tcol * a.K;
  f32x16 acc = f32x16{};
  // U batches of 16 k per step, all their loads issued before their MFMAs
  constexpr int U = 4;
  for (int64_t b = b0; b < b1; b += U) {
    float w[U][8], x[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = b + u < b1;
      const int64_t k = (in ? b + u : b0) * 16 + 8 * h;
      if constexpr (DT == 2) {
        load_row16<2>(a.w, (int64_t)rrow * a.w_stride + k, w[u]);
        load_row16<2>(a.w, (int64_t)rrow * a.w_stride + k + 4, w[u] + 4);
      } else {
        load_row16<DT>(a.w, (int64_t)rrow * a.w_stride + k, w[u]);
      }
      const f32x4 f0 = *reinterpret_cast<const CKV_GLOBAL f32x4*>(af + k);
      const f32x4 f1 = *reinterpret_cast<const CKV_GLOBAL f32x4*>(af + k + 4);
      const f32x4 c0 = *reinterpret_cast<const CKV_GLOBAL f32x4*>(ac + k);
      const f32x4 c1 = *reinterpret_cast<const CKV_GLOBAL f32x4*>(ac + k + 4);
      const float fv[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
      const float cv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
      for (int m = 0; m < 8; ++m)
        x[u][m] = !in ? 0.f : (full_col ? fv[m] : (diff_col ? cv[m] - fv[m] : 0.f));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int m = 0; m < 8; ++m) acc = mfma_f32(w[u][m], x[u][m], acc);
  }
  // acc[v]: row rb*32 + acc_row(v, h), column cb*32 + l32
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][acc_row(v, h)][l32] = acc[v];
  __syncthreads();
  float* tile = a.part_y + (((int64_t)ks * gridDim.x + rb) * gridDim.y + cb) * 1024;
  for (int e = tid; e < 1024; e += kProjThreads) {
    const int r = e >> 5, c = e & 31;
    float y = 0.f;
#pragma unroll
    for (int wv = 0; wv < kProjWaves; ++wv) y += red[wv][r][c];
    tile[e] = y;
  }
}

// 16-bit W_O: the columns of X = [A_full | A_comp - A_full] (fp32) split into
// two 16-bit parts in W_O's type, high = X rounded, low = X - high rounded,
// so that the 16-bit MFMA of W_O with high and then low gives W_O X to about
// 16 significant bits (W_O itself is exact in its type). x_hl is
// [2][n_cols][K]; columns from 2T on are zero.
template <int DT>
__global__ __launch_bounds__(kProjThreads) void xsplit_kernel(const ErrorArgs a) {
  const int64_t n = (int64_t)a.n_cols * a.K;
  for (int64_t e = (int64_t)blockIdx.x * kProjThreads + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * kProjThreads) {
    const int col = (int)(e / a.K);
    const int64_t k = e - (int64_t)col * a.K;
    float x = 0.f;
    if (col < a.T) x = a.a_full[(int64_t)col * a.K + k];
    else if (col < 2 * a.T)
      x = a.a_comp[(int64_t)(col - a.T) * a.K + k] - a.a_full[(int64_t)(col - a.T) * a.K + k];
    uint16_t hi, lo;
    if constexpr (DT == 0) {  // bf16, round to nearest even (X is finite)
      auto rne = [](float v) {
        const uint32_t u = __float_as_uint(v);
        return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
      };
      hi = rne(x);
      lo = rne(x - __uint_as_float((uint32_t)hi << 16));
    } else {
      const _Float16 h = (_Float16)x;
      const _Float16 l = (_Float16)(x - (float)h);
      hi = __builtin_bit_cast(uint16_t, h);
      lo = __builtin_bit_cast(uint16_t, l);
    }
    a.x_hl[e] = hi;
    a.x_hl[n + e] = lo;
  }
}

// 16-bit W_O: workgroup (row blocks 4*bx .. 4*bx+3, column block cb, K range
// ks); wave w computes the 32 x 32 tile of row block 4*bx + w over the K
// range with the 32x32x16 MFMA (W_O rows against the high and then the low
// part of X, one accumulator) and writes it to part_y.
//
// Every load of the workgroup is issued at the start, so that the whole
// range is in flight at once: W_O in tiles of 32 rows x 128 k (8 KB, at most
// kProjTiles per wave) into registers with contiguous loads (lane l of load i
// takes 16-byte chunk l % 16 of tile row 4i + l / 16), and the X tiles the
// four waves share (both parts, 32 columns) into LDS by all threads. A tile
// of W_O then goes through the wave's LDS region. In LDS, chunk c of row (or
// column) r sits at position c ^ (r % 16); lane half h of lane l32 reads
// chunk 2j + h of row l32 for the j-th 16-k step of the tile, as its X column
// does.
constexpr int kProjTileK = 128;                                // k per tile
constexpr int kProjTileLoads = 32 * kProjTileK * 2 / 16 / 64;  // 16-byte W_O loads per lane: 8
constexpr int kProjTiles = kProjRangeK / kProjTileK;           // tiles per K range: 2
constexpr int kProjXChunks = kProjTiles * 2 * 32 * (kProjTileK / 8);  // 16-byte X chunks: 2048
constexpr int kProjXLoads = kProjXChunks / kProjThreads;              // per thread: 8

template <int DT>
__global__ __launch_bounds__(kProjThreads) void project16_kernel(const ErrorArgs a) {
  __shared__ uint4 wl[kProjWaves][32 * (kProjTileK / 8)];  // a W_O tile per wave, 8 KB
  __shared__ uint4 xl[kProjXChunks];                        // [tile][part][col][chunk], 32 KB
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wave = tid >> 6;
  const int n_rb = (a.D + 31) / 32;
  const int rb = blockIdx.x * kProjWaves + wave, cb = blockIdx.y, ks = blockIdx.z;
  const int64_t n16 = a.K / 16;
  const int64_t per_ks = (n16 + a.n_split - 1) / a.n_split;
  const int64_t k0 = ks * per_ks, k1 = k0 + per_ks < n16 ? k0 + per_ks : n16;  // in 16-k steps
  const int n_steps = k1 > k0 ? (int)(k1 - k0) : 0;  // <= kProjTiles * 8 (checked on the host)
  const CKV_GLOBAL uint16_t* w0 = to_global(static_cast<const uint16_t*>(a.w));
  const CKV_GLOBAL uint16_t* x0 = to_global(a.x_hl);
  // this wave's W_O tiles (rows past D or k past the range: zeros)
  u32x4 t[kProjTiles][kProjTileLoads];
#pragma unroll
  for (int tl = 0; tl < kProjTiles; ++tl)
#pragma unroll
    for (int i = 0; i < kProjTileLoads; ++i) {
      const int r = 4 * i + lane / 16, c = lane % 16;
      const int row = rb * 32 + r;
      const bool ok = rb < n_rb && row < a.D && tl * 8 + c / 2 < n_steps;
      const int64_t off =
          ok ? (int64_t)row * a.w_stride + (k0 + tl * 8) * 16 + 8 * c : 0;
      t[tl][i] = ok ? *reinterpret_cast<const CKV_GLOBAL u32x4*>(w0 + off) : u32x4{0u, 0u, 0u, 0u};
    }
  // the shared X tiles: chunk e = ((tile * 2 + part) * 32 + col) * 16 + c
  u32x4 xv[kProjXLoads];
#pragma unroll
  for (int i = 0; i < kProjXLoads; ++i) {
    const int e = i * kProjThreads + tid;
    const int c = e % 16, col = (e / 16) % 32, part = (e / 512) % 2, tl = e / 1024;
    const bool ok = tl * 8 + c / 2 < n_steps;
    const int64_t off = ok ? ((int64_t)part * a.n_cols + cb * 32 + col) * a.K +
                                 (k0 + tl * 8) * 16 + 8 * c
                           : 0;
    xv[i] = ok ? *reinterpret_cast<const CKV_GLOBAL u32x4*>(x0 + off) : u32x4{0u, 0u, 0u, 0u};
  }
#pragma unroll
  for (int i = 0; i < kProjXLoads; ++i) {
    const int e = i * kProjThreads + tid;
    const int c = e % 16, rc = e / 16;  // rc = (tile * 2 + part) * 32 + col
    xl[rc * 16 + (c ^ (rc & 15))] = make_uint4(xv[i].x, xv[i].y, xv[i].z, xv[i].w);
  }
  __syncthreads();
  if (rb >= n_rb) return;  // after the barrier: these waves only helped load X
  uint4* tile = wl[wave];
  f32x16 acc = f32x16{};
#pragma unroll
  for (int tl = 0; tl < kProjTiles; ++tl) {
    if (tl * 8 >= n_steps) break;
#pragma unroll
    for (int i = 0; i < kProjTileLoads; ++i) {
      const int r = 4 * i + lane / 16, c = lane % 16;
      tile[r * 16 + (c ^ (r & 15))] = make_uint4(t[tl][i].x, t[tl][i].y, t[tl][i].z, t[tl][i].w);
    }
    __builtin_amdgcn_wave_barrier();
    const uint4* xh = xl + (tl * 2 + 0) * 32 * 16;
    const uint4* xlo = xl + (tl * 2 + 1) * 32 * 16;
#pragma unroll
    for (int j = 0; j < kProjTileK / 16; ++j) {
      const int pos = (2 * j + h) ^ (l32 & 15);
      const uint4 wv = tile[l32 * 16 + pos];
      acc = mfma_chunk<DT>(wv, xh[l32 * 16 + pos], acc);
      acc = mfma_chunk<DT>(wv, xlo[l32 * 16 + pos], acc);
    }
    __builtin_amdgcn_wave_barrier();  // the next tile's stores come after these reads
  }
  // acc[v]: row rb*32 + acc_row(v, h), column cb*32 + l32
  float* out = a.part_y + (((int64_t)ks * n_rb + rb) * gridDim.y + cb) * 1024;
#pragma unroll
  for (int v = 0; v < 16; ++v) out[acc_row(v, h) * 32 + l32] = acc[v];
}

// Workgroup (rb, cb): Y = the n_split partial tiles added in order, then
// per column the sum of Y^2 over the tile's rows (rows past D excluded) into
// part[rb][col].
__global__ __launch_bounds__(kProjThreads) void square_kernel(const ErrorArgs a) {
  constexpr int RG = kProjThreads / 32;  // row groups: thread t sums rows t/32, t/32 + RG, ...
  __shared__ float colsum[RG][32];
  const int rb = blockIdx.x, cb = blockIdx.y, nrb = gridDim.x, ncb = gridDim.y;
  const int c = threadIdx.x & 31, rg = threadIdx.x >> 5;
  float sq = 0.f;
  for (int r = rg; r < 32; r += RG) {
    if (rb * 32 + r >= a.D) break;
    // the n_split partials in order, loaded 16 at a time
    float y = 0.f;
    for (int ks0 = 0; ks0 < a.n_split; ks0 += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        v[u] = ks0 + u < a.n_split ? a.part_y[(((int64_t)(ks0 + u) * nrb + rb) * ncb + cb) * 1024 + r * 32 + c]
                                   : 0.f;
#pragma unroll
      for (int u = 0; u < 16; ++u) y += v[u];
    }
    sq += y * y;
  }
  colsum[rg][c] = sq;
  __syncthreads();
  if (threadIdx.x < 32) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < RG; ++i) t += colsum[i][c];
    const int col = cb * 32 + c;
    if (col < 2 * a.T) a.part[(int64_t)rb * 2 * a.T + col] = t;
  }
}

// One workgroup: num_t and den_t summed over the row blocks (kDecWaves
// threads per step and column kind, each over every kDecWaves-th block, then
// combined in a fixed order), the ratios and their sum in step order.
__global__ __launch_bounds__(kDecThreads) void error_kernel(const ErrorArgs a) {
  constexpr int kSplit = 8;                         // threads per column
  constexpr int kCols = kDecThreads / kSplit;       // columns per round
  __shared__ float part_l[kSplit][kCols];
  __shared__ float col_l[kCols];
  const int n_rb = (a.D + 31) / 32;
  const int j = threadIdx.x % kSplit, cl = threadIdx.x / kSplit;
  float total = 0.f;
  for (int c0 = 0; c0 < 2 * a.T; c0 += kCols) {
    const int col = c0 + cl;
    float acc = 0.f;
    if (col < 2 * a.T) {
      // row blocks j, j + kSplit, ... in that order, kBatch loads in flight
      constexpr int kBatch = 8;
      for (int rb0 = j; rb0 < n_rb; rb0 += kSplit * kBatch) {
        float v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const int rb = rb0 + u * kSplit;
          v[u] = rb < n_rb ? a.part[(int64_t)rb * 2 * a.T + col] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) acc += v[u];
      }
    }
    part_l[j][cl] = acc;
    __syncthreads();
    if (threadIdx.x < kCols) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < kSplit; ++i) v += part_l[i][threadIdx.x];
      col_l[threadIdx.x] = v;
    }
    __syncthreads();
    // columns c0 .. c0 + kCols - 1 hold den (col < T) or num (col >= T) of
    // their steps; a step's pair lands in the same round when T <= kCols / 2
    if (threadIdx.x == 0) {
      for (int i = 0; i < kCols && c0 + i < 2 * a.T; ++i) part_l[0][i] = col_l[i];
    }
    __syncthreads();
    if (threadIdx.x < kCols && c0 + threadIdx.x < 2 * a.T)
      a.part[(int64_t)n_rb * 2 * a.T + c0 + threadIdx.x] = part_l[0][threadIdx.x];
    __syncthreads();
  }
  // the column sums sit after the row-block partials; ratios in step order
  const float* sums = a.part + (int64_t)n_rb * 2 * a.T;
  if (threadIdx.x == 0) {
    for (int t = 0; t < a.T; ++t) {
      const float r = sqrtf(sums[a.T + t]) / (sqrtf(sums[t]) + a.eps);
      a.ratio[t] = r;
      total += r;
    }
    *a.e = total;
  }
}

// The decode kernel of a batch whose largest prompt has `rows` query rows per
// KV head.
template <int DT, int D>
hipError_t launch_dec(const DecodeBatch& b, int rows, hipStream_t st) {
  const Timing tm;
  const int grid = b.blk_off[b.n];
  if (rows <= 32) return launch(decode_kernel<DT, D, 1>, grid, kDecThreads, st, tm, b);
  if (rows <= 64) return launch(decode_kernel<DT, D, 2>, grid, kDecThreads, st, tm, b);
  if constexpr (DT == 2) return launch(decode_rows_kernel_f32<2, D>, grid, kDecThreads, st, tm, b);
  else return launch(decode_rows_kernel_16<DT, D>, grid, kDecThreads, st, tm, b);
}

}  // namespace

hipError_t launch_decode(int dtype, const DecodeBatch& b, hipStream_t st) {
  int rows = 0;
  for (int i = 0; i < b.n; ++i) {
    const int r = b.H / b.n_kv * b.s[i].T;
    rows = r > rows ? r : rows;
  }
  hipError_t e;
  if (dtype == 0) e = b.d == 64 ? launch_dec<0, 64>(b, rows, st) : launch_dec<0, 128>(b, rows, st);
  else if (dtype == 1) e = b.d == 64 ? launch_dec<1, 64>(b, rows, st) : launch_dec<1, 128>(b, rows, st);
  else e = b.d == 64 ? launch_dec<2, 64>(b, rows, st) : launch_dec<2, 128>(b, rows, st);
  if (e != hipSuccess || b.mrg_off[b.n] == 0) return e;
  const Timing tm;
  return b.d == 64 ? launch(decode_merge_kernel<64>, b.mrg_off[b.n], kDecThreads, st, tm, b)
                   : launch(decode_merge_kernel<128>, b.mrg_off[b.n], kDecThreads, st, tm, b);
}

hipError_t launch_error(int w_dtype, const ErrorArgs& a, hipStream_t st) {
  const Timing tm;
  const int n_rb = (a.D + 31) / 32;
  const dim3 grid(n_rb, (2 * a.T + 31) / 32, a.n_split);
  const dim3 tiles(grid.x, grid.y);
  hipError_t e;
  if (w_dtype == 2) {
    e = launch(project_kernel<2>, grid, kProjThreads, st, tm, a);
  } else {
    // 16-bit W_O: split X once, then one wave per 32 x 32 tile and K range
    const int64_t n = (int64_t)a.n_cols * a.K;
    const int xg = (int)((n + kProjThreads - 1) / kProjThreads);  // one element per thread
    e = w_dtype == 0 ? launch(xsplit_kernel<0>, xg, kProjThreads, st, tm, a)
                     : launch(xsplit_kernel<1>, xg, kProjThreads, st, tm, a);
    if (e != hipSuccess) return e;
    const dim3 g16((n_rb + kProjWaves - 1) / kProjWaves, grid.y, a.n_split);
    e = w_dtype == 0 ? launch(project16_kernel<0>, g16, kProjThreads, st, tm, a)
                     : launch(project16_kernel<1>, g16, kProjThreads, st, tm, a);
  }
  if (e != hipSuccess) return e;
  if ((e = launch(square_kernel, tiles, kProjThreads, st, tm, a)) != hipSuccess) return e;
  return launch(error_kernel, 1, kDecThreads, st, tm, a);
}

}  // namespace ckv
