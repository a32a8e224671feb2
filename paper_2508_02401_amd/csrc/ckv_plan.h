// Launch plans that are plain arithmetic on sizes: how decode attention and one
// layer's selection are cut into workgroups. No HIP in here, so that the rules can be tested on the host.
#pragma once

#include <stdint.h>

namespace ckv {

// Decode workgroups per CU that a launch is cut for, by the kernel that takes
// `rows` query rows per KV head: two, but one where the kernel's registers
// (over 256 of a SIMD's 512) or its LDS (over 80 of 160 KB) admit no second:
// fp32 at d = 128, 16-bit at d = 128 and fp32 with 33 to 64 rows. With 33 to 64
// rows at d = 64 in 16 bits, and up to 32 rows at d = 64 in fp32, two would fit,
// but one with twice the keys is as fast or faster: 2 KV heads, one cache of
// 131072 tokens, 64 rows, 25.4 us against 28.0 (four of 65536: 38.0 against
// 36.9); fp32, 8 rows, four of 65536: 54.9 us against 62.2.
inline int decode_wgs_per_cu(bool f32, int head_dim, int rows) {
  if (rows <= 32) return f32 ? 1 : 2;
  if (rows <= 64) return 1;
  return f32 && head_dim == 128 ? 1 : 2;
}

// Tokens per decode workgroup for one launch over cnt caches of n[i] tokens, the
// same for every prompt: a multiple of one 32-key tile, at least a tile per
// wave (128), for about `target` workgroups over all caches and KV heads, as
// many as are resident at once. A few workgroups more would run after the
// others: 516 of them took 122 us on four caches of 196608 tokens in all,
// where 512 are resident; so the chunk grows until they are one round, but at
// most to twice the even share. Where that is not enough (caches x KV heads
// near or past `target`, which no chunk length can bring down) the even share
// stays: workgroups of any number then share the work, and the longest is no
// longer than two even rounds. Growing on made it one workgroup per cache and
// head: 32 KV heads, one cache of 131072 tokens and sixteen of 1024 took 1580
// us, 32 of 544 workgroups with 89% of the bytes.
inline int64_t decode_chunk_len(int64_t target, int64_t n_kv, int32_t cnt, const int64_t* n) {
  int64_t sum_n = 0, max_n = 0;
  for (int32_t i = 0; i < cnt; ++i) {
    sum_n += n[i];
    max_n = n[i] > max_n ? n[i] : max_n;
  }
  int64_t even = (sum_n * n_kv + target - 1) / target;
  even = (even + 31) / 32 * 32;
  if (even < 128) even = 128;
  if (even >= max_n) return max_n < 128 ? 128 : (max_n + 31) / 32 * 32;  // one chunk each
  for (int64_t c = even; c <= 2 * even; c += (c + 32 * 32 - 1) / (32 * 32) * 32) {
    int64_t wgs = 0;
    for (int32_t i = 0; i < cnt; ++i) wgs += (n[i] + c - 1) / c * n_kv;
    if (wgs <= target) return c;
  }
  return even;
}

// Most partial rows (chunks of a KV head times its query rows) that the launches
// over cnt caches can need, for these row counts and cache lengths or smaller
// ones: rows is the largest prompt's, tiles the sum over the caches of
// ceil(n / 128). A launch has at most one chunk per 128 keys, and at most its even
// share's count plus one per cache and head. Fewer rows may mean more chunks (the
// 32-row kernel is cut for twice the workgroups of the 64-row one) and, in a mixed
// batch, two launches; a size that grew with neither would refuse a program
// that sizes its buffer once, for its longest caches and most tokens.
inline int64_t decode_partial_rows(bool f32, int head_dim, int64_t cus, int64_t n_kv, int32_t cnt,
                                   int64_t tiles, int64_t rows, bool mixed) {
  auto most = [&](int64_t r) {  // of one launch whose largest prompt has r rows
    const int64_t by_share = cus * decode_wgs_per_cu(f32, head_dim, (int)r) + cnt * n_kv;
    return (tiles * n_kv < by_share ? tiles * n_kv : by_share) * r;
  };
  int64_t few = most(rows < 32 ? rows : 32);
  if (rows > 32) {
    const int64_t f = most(rows < 64 ? rows : 64);
    few = f > few ? f : few;
  }
  if (rows <= 64) return few;
  const int64_t many = most(rows);
  return mixed ? few + many : (few > many ? few : many);
}

// Whether the prompts with at most 64 query rows of a batch that also has prompts
// with more are launched apart, given their cached tokens times KV heads. The
// kernel for more rows gives a prompt one wave per 32 rows, so a one-token
// prompt there leaves three of four waves idle, but a launch pair of its own
// costs about 9 us. 16 bits, 15 one-token caches beside one of 300 tokens with
// 112 rows, 4 KV heads: 246000 keys 39.7 us together and 41.5 apart, 492000 keys
// 64.9 and 60.6; the fp32 kernel's waves are slower: 31000 keys 36 and 51, 61000
// keys 61 and 58, 123000 keys 99 and 69.
inline bool decode_split_pays(bool f32, int64_t few_keys) {
  return few_keys >= (f32 ? 1 << 16 : 1 << 18);
}

// Workgroups of one layer's selection units when each unit is split into parts
// that copy a share of its kept rows: prompt s's units have parts[s] workgroups
// each, unit after unit from first[s] on. Where all units have as many (one prompt
// above all), `same` says so: a division finds the prompt without the reads of
// first[] and parts[], which cost the start of the launch 0.3 us.
constexpr int kPlanSeqs = 16;  // most prompts of a layer call
constexpr int kPartRows = 16;  // kept rows per part (at least, where a unit has so many)
struct UnitParts {
  int32_t same;  // parts of every unit, or 0 where they differ
  int32_t first[kPlanSeqs + 1];
  int32_t parts[kPlanSeqs];
};

// Workgroups that the parts of a layer call may be, for its kept rows in all and
// its longest prompt's scored tokens: one round (a unit workgroup's LDS fills a
// CU) when the prompts are short or a part of half a round would copy more than
// 256 rows, else half a round. The other half is what a caller's other streams
// run on meanwhile: layers of 32768 tokens, 2048 kept by each of 8 heads, over
// four streams took 49.6 us each with a whole round, 43.4 with half, over two
// 50.7 and 47.6; on one stream 61.0 and 60.6. Short prompts' K passes leave CUs
// free by themselves: 4013 tokens on one stream took 42.0 us with a round, 42.7
// with half. With 32768 of 65000 tokens kept the copies count: 128 and 145 us.
constexpr int64_t kPartShort = 8192;
inline int64_t part_round(int64_t cus, int64_t total_rows, int64_t scored) {
  return scored < kPartShort || total_rows > cus / 2 * 256 ? cus : cus / 2;
}

// Deals a round of `cus` workgroups out over the units, one to each and the others
// by the rows that a unit keeps, rows[s] of each head and unit of prompt s; units
// past cus run in further rounds, unsplit. A unit that copies for several heads
// (a shared selection) gets a multiple of them where it gets as many, so that no
// part ends one head's rows and starts another's, two turns in a row (two prompts
// of 24571 and 9001 tokens, 8 heads: 52.1 us with parts over head ends, 50.5
// without). Returns the most rows of a part. The same count for every unit made a
// long prompt's parts the last to end: 16 prompts of 8 KV heads, one keeping 8192
// rows a head and the others 128, took 187 us, now 130.
inline int64_t deal_unit_parts(int64_t cus, int32_t num_seqs, int32_t n_sg, int32_t heads,
                               const int64_t* rows, UnitParts& p) {
  const int64_t units = (int64_t)num_seqs * n_sg, more = cus > units ? cus - units : 0;
  int64_t total = 0, most = 0;
  for (int32_t s = 0; s < num_seqs; ++s) total += rows[s] * n_sg;
  p.first[0] = p.same = 0;
  for (int32_t s = 0; s < num_seqs; ++s) {
    const int64_t unit_rows = rows[s] * heads;
    const int64_t share = 1 + more * rows[s] / total, useful = unit_rows / kPartRows;
    int64_t n = share < useful ? share : (useful > 1 ? useful : 1);
    if (n > heads) n -= n % heads;
    p.parts[s] = (int32_t)n;
    p.same = s == 0 || p.same == n ? p.parts[s] : 0;
    p.first[s + 1] = p.first[s] + p.parts[s] * n_sg;
    const int64_t r = (unit_rows + n - 1) / n;
    most = r > most ? r : most;
  }
  return most;
}

}  // namespace ckv
