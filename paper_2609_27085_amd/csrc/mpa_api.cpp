// C ABI of the mixed paged-attention library: host-side validation, the
// varlen planner (decode rows -> split-K work items, prefill chunks -> query
// tiles) and the launch sequence.  Every check runs before the first launch.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <functional>
#include <mutex>
#include <queue>
#include <unordered_set>
#include <vector>

#include "mpa.h"
#include "mpa_internal.h"

namespace {

using mpa::kBlock;
constexpr int kMaskWords = 8;  // CU-mask words: devices of up to 256 CUs

struct Batch {
  std::vector<int> decode;   // sequence ids with q_len == 1
  std::vector<int> prefill;  // sequence ids with q_len > 1
};

int check_shape(const mpa_shape* sh) {
  if (!sh) return MPA_ERR_INVALID;
  if (sh->num_seqs < 0 || sh->num_q_heads <= 0 || sh->num_kv_heads <= 0 || sh->num_blocks < 0 ||
      sh->max_blocks_per_seq < 0 || sh->total_q_tokens < 0 || !isfinite(sh->scale) || !(sh->scale > 0.f))
    return MPA_ERR_INVALID;
  if (sh->dtype != MPA_BF16 && sh->dtype != MPA_F32 && sh->dtype != MPA_FP8) return MPA_ERR_UNSUPPORTED;
  if (sh->dtype == MPA_FP8 && !(isfinite(sh->k_scale) && sh->k_scale > 0.f && isfinite(sh->v_scale) &&
                                sh->v_scale > 0.f))
    return MPA_ERR_INVALID;
  if (sh->head_dim != 64 && sh->head_dim != 128) return MPA_ERR_UNSUPPORTED;
  if (sh->block_size != kBlock) return MPA_ERR_UNSUPPORTED;
  if (sh->num_q_heads % sh->num_kv_heads != 0) return MPA_ERR_UNSUPPORTED;
  if (sh->num_q_heads / sh->num_kv_heads > 16) return MPA_ERR_UNSUPPORTED;
  return MPA_OK;
}

// The MFMA prefill launch's work units (query tiles x KV heads) over the
// chunks, and the most KV splits any chunk's prefix allows.
void prefill_units(const mpa_shape* sh, const std::vector<int>& prefill, const int32_t* seq_lens,
                   const int32_t* qsl, long* units, int* most) {
  const int qt = mpa::kPrefillRowsMfma / (sh->num_q_heads / sh->num_kv_heads);
  *units = 0;
  *most = 1;
  for (int s : prefill) {
    const int C = qsl[s + 1] - qsl[s];
    *units += (long)(C + qt - 1) / qt * sh->num_kv_heads;
    *most = std::max(*most, std::min(1 + (seq_lens[s] - C) / 64 / mpa::kPrefillMinSplitTiles, 64));
  }
}

// Whether the planner starts from whole chunks (one KV split each): MFMA
// batches with at least two workgroups per CU or no prefix long enough to
// split.
bool prefill_whole(const mpa_shape* sh, const std::vector<int>& prefill, const int32_t* seq_lens,
                   const int32_t* qsl) {
  long units;
  int most;
  prefill_units(sh, prefill, seq_lens, qsl, &units, &most);
  return units >= 2L * mpa::kPrefillSplitTarget || most == 1;
}

// Validates the host metadata.
int check_batch(const mpa_shape* sh, const int32_t* seq_lens, const int32_t* qsl, const int32_t* bt_host,
                bool append_only) {
  int rc = check_shape(sh);
  if (rc != MPA_OK) return rc;
  const int S = sh->num_seqs;
  if (S > 0 && (!seq_lens || !qsl)) return MPA_ERR_INVALID;
  if (S == 0) return sh->total_q_tokens == 0 ? MPA_OK : MPA_ERR_INVALID;
  if (qsl[0] != 0 || qsl[S] != sh->total_q_tokens) return MPA_ERR_INVALID;
  for (int s = 0; s < S; ++s) {
    const int ql = qsl[s + 1] - qsl[s];
    const int L = seq_lens[s];
    if (ql < 0 || L < 0 || ql > L) return MPA_ERR_INVALID;
    if (ql == 0) continue;
    if (sh->num_blocks == 0) return MPA_ERR_INVALID;  // nothing could hold its KV
    const long nblk = ((long)L + kBlock - 1) / kBlock;
    if (nblk > sh->max_blocks_per_seq) return MPA_ERR_INVALID;
    if (bt_host) {
      const long first = append_only ? (long)(L - ql) / kBlock : 0;
      for (long j = first; j < nblk; ++j) {
        const int32_t id = bt_host[(size_t)s * sh->max_blocks_per_seq + j];
        if (id < 0 || id >= sh->num_blocks) return MPA_ERR_INVALID;
      }
    }
  }
  return MPA_OK;
}

// The sequences of a valid batch by kind.
Batch classify(const mpa_shape* sh, const int32_t* qsl) {
  Batch b;
  for (int s = 0; s < sh->num_seqs; ++s) {
    const int ql = qsl[s + 1] - qsl[s];
    if (ql == 1) b.decode.push_back(s);
    if (ql > 1) b.prefill.push_back(s);
  }
  return b;
}

// The tuning overrides in the environment, read at each call: the value when
// it is a whole number in [lo, hi] and a multiple of `step`, else -1 (not set).
// The planner and the memo's key both go through these, so that an override
// that is not taken plans (and is remembered) as none at all.
int env_override(const char* name, long lo, long hi, long step) {
  const char* e = getenv(name);
  if (!e) return -1;
  char* end = nullptr;
  const long v = strtol(e, &end, 10);
  return end != e && v >= lo && v <= hi && v % step == 0 ? (int)v : -1;
}
int env_split_tokens() { return env_override("MPA_SPLIT_TOKENS", kBlock, 1024, kBlock); }
int env_prefill_splits() { return env_override("MPA_PREFILL_SPLITS", 1, 64, 1); }
int env_decode_range() { return env_override("MPA_DECODE_RANGE", 0, 1 << 26, 1); }  // in tokens below 2^31

// How a decode row of L keys is split at nominal split size S: into
// n = ceil(L / S) parts of equal size, rounded up to whole cache blocks, so
// that the waves of a launch stream about the same number of bytes (a fixed
// size S with a short remainder would leave the short waves idle while the
// full ones finish).  The last part ends at L; `parts` can be below n when
// the rounding makes the earlier parts cover L sooner.
struct RowSplit {
  int parts;
  int tokens;  // keys per part, a multiple of the block size
};

RowSplit row_split(int L, int S) {
  const int n = std::max(1, (L + S - 1) / S);
  const int per = (L + n - 1) / n;
  const int tokens = std::max(kBlock, (per + kBlock - 1) / kBlock * kBlock);
  return {std::max(1, (L + tokens - 1) / tokens), tokens};
}

// KV tokens per decode split.  Every (split, KV head) is one wave, and a
// wave's time is about proportional to its tokens plus a fixed start-up cost,
// so the step takes about ceil(waves / slots) * (split + overhead), where
// slots is the number of waves the device runs at once.  The split is the
// multiple of 16 in [128, 1024] that minimises that estimate (more, smaller
// splits fill the last round of waves; fewer, larger ones cut start-up and
// merge work).  MPA_SPLIT_TOKENS (a multiple of 16, at most 1024) overrides
// it for tuning sweeps.
int choose_split(const mpa_shape* sh, const Batch& b, const int32_t* seq_lens) {
  if (const int v = env_split_tokens(); v > 0) return v;
  if (b.decode.empty()) return 1024;
  const long slots = mpa::decode_wave_slots(sh->dtype, sh->head_dim, false);
  const long overhead = 64;
  long best_cost = -1;
  int best = 1024;
  long tokens = 0;
  for (int s : b.decode) tokens += seq_lens[s];
  for (int split = 128; split <= 1024; split += kBlock) {
    // no split makes fewer parts than this many, so most splits are ruled out
    // without a pass over the rows
    const long fewest = std::max((long)b.decode.size(), (tokens + split - 1) / split) * sh->num_kv_heads;
    if (best_cost >= 0 && (fewest + slots - 1) / slots * (split + overhead) >= best_cost) continue;
    long items = 0;
    for (int s : b.decode) items += row_split(seq_lens[s], split).parts;
    const long waves = items * sh->num_kv_heads;
    const long cost = ((waves + slots - 1) / slots) * (split + overhead);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = split;
    }
  }
  return best;
}

int row_blocks(int L) { return (int)(((long)L + kBlock - 1) / kBlock); }

// The fewest blocks per wave at which a launch's rows are dealt to the waves
// as ranges of equal size (the streaming decode kernel) instead of each row
// being split on its own.  Below it the waves' few blocks do not pay for the
// wider launch and the rows cut at odd places; measured on 8 to 192 rows of
// 512-8,192 and 2,048-16,384 tokens (blocks per wave: time of row splits ->
// of ranges, decode and merge), the two meet at
//   bf16, d 128: 12 blocks 58.6 -> 61.4 us, 24 100.6 -> 99.4, 42 169.7 ->
//                165.8, 102 417 -> 385;
//   bf16, d 64:  6 blocks 28.3 -> 29.1 us, 10 38.8 -> 37.3, 26 82.9 -> 77.7;
//   fp8,  d 128: 51 blocks 113.5 -> 115.3 us (row splits fill one round of
//                waves), 61 152.8 -> 143.7 (two rounds), 139 322 -> 284;
//   fp8,  d 64:  12 blocks 22.6 -> 22.5 us, 22 33.5 -> 30.9, 139 158 -> 140;
//   f32:         21 blocks 121.8 -> 123.3 us, 26 146.6 -> 144.5, 51 376 -> 354.
int range_min_blocks(int dtype, int head_dim) {
  if (dtype == MPA_F32) return 24;
  if (dtype == MPA_FP8) return head_dim == 128 ? 60 : 12;
  return head_dim == 128 ? 24 : 10;
}

// bf16 and f32 launches of ranges hold waves for three quarters of the device's
// slots, whole workgroups of a CU each: 192 of 256 CUs draw all that the memory
// gives, with less contention among them (32 / 8 heads, steps of 6-200 rows,
// all slots -> three quarters: bf16 281 MB 116.0 -> 113.8 us, 3.2 GB 520.6 ->
// 503.9, 6.5 GB 990 -> 966; f32 703 -> 674; 7 / 8 of them between the two, 2 / 3
// slower), and on three quarters of the CUs, where a partitioned step runs its
// decode, they are still one round (256 rows of 4-8K beside 4,096 tokens, decode
// there: 1,264 -> 965 us).  Ranges of fewer blocks than this lose more to
// being longer (64-wide heads, 10 blocks: 37.7 -> 39.3), and so do fp8 launches,
// whose small workgroups leave waves on every CU short (276.6 -> 302.3).
constexpr long kFewerWavesBlocks = 14;

// Whether ranges of `range` blocks pay by the rows they meet.  A wave goes over
// the rows of its range one after another, and each costs it a start (and its
// new token a wait), about a block's time and more at fp8 and in a step that
// appends; the launch takes as long as its most crowded range.  Measured as
// row splits -> ranges (us, 32 / 8 heads, step with its tokens), with the rows
// past the first in the most crowded range over its blocks:
//   bf16, d 128: 0.06 354 -> 314, 0.15 417 -> 399, 0.24 221 -> 244, 0.25 416
//     -> 427 (100 rows of 64 keys behind 4 of 131,072), 0.41 805 -> 994 (248
//     rows of 1-64 behind 8);
//   bf16, d 64: 0.07 174 -> 161, 0.15 83.1 -> 82.8, 0.24 110 -> 125;
//   f32: 0.1 198 -> 194, 0.2 191 -> 189, 0.24 423 -> 459;
//   fp8, d 128: 0.05 197 -> 182, 0.25 236 -> 264, 0.41 448 -> 575;
//   fp8, d 64: 0.08 90.3 -> 90.5 (83.8 -> 81.7 without tokens), 0.24 65 -> 83.
// fp8 rows whose splits fill at most one round of waves are split (d 64: 128
// rows of 1,100 35.1 -> 38.8, 256 of 2,000 98.4 -> 100.4; more rounds, 256 of
// 100-8,000 without tokens 83.8 -> 81.7; d 128: 128 of 3,000 134 -> 141, two
// rounds, 256 of 2,000 203 -> 201), and so are bf16 rows of 64-wide heads whose
// ranges are the shortest and whose splits are few to merge (256 of 400 49.0
// -> 50.4; with 16 parts a row 128 of 3,000 44.5 -> 42.6).
bool ranges_pay(const mpa_shape* sh, const Batch& b, const int32_t* seq_lens, size_t c0, size_t c1, int range,
                int* split) {
  int most = 0, here = 0;
  long at = 0, last = -1;  // the last range met, by `here` rows so far
  for (size_t k = c0; k < c1; ++k) {
    const int nb = row_blocks(seq_lens[b.decode[k]]);
    here = at / range == last ? here + 1 : 1;
    most = std::max(most, here);
    if ((at + nb - 1) / range > at / range) here = 1;
    last = (at + nb - 1) / range;
    at += nb;
  }
  const bool fp8 = sh->dtype == MPA_FP8;
  if ((most - 1) * (fp8 ? 8 : 5) > range) return false;
  const bool shortest = sh->dtype == MPA_BF16 && sh->head_dim == 64 && range < 14;
  if (!fp8 && !shortest) return true;
  if (*split == 0) *split = choose_split(sh, b, seq_lens);
  long items = 0;
  for (size_t k = c0; k < c1; ++k) items += row_split(seq_lens[b.decode[k]], *split).parts;
  if (fp8) return items * sh->num_kv_heads > mpa::decode_wave_slots(sh->dtype, sh->head_dim, false);
  return items >= 4 * (long)(c1 - c0);
}

// The launches that take one workgroup per (row, KV head) (decode_short_kernel)
// with no row split: at most so many pairs, of rows of at most so many keys.
// Measured against row splits and their merge (decode half, us; 12.3 is what
// the host takes to issue a call), splits -> this:
//   bf16, d 128: 8 rows of 8 heads of up to 700 keys 16.6 -> 13.0, 1,024 16.3
//     -> 14.7, 1,500 16.7 -> 19.2; 64 rows of 1,024 40.3 -> 37.5;
//   bf16, d 64: 64 rows of 2 heads, 2,048 keys 16.7 -> 15.6, 3,000 20.2 -> 21.5;
//   fp8, d 128: 32 rows of 8 heads, 1,024 keys 17.2 -> 15.8; 64 rows of 700
//     22.2 -> 23.1 (the split kernel reads the codes by 16 bytes);
//   f32, d 128: 32 rows of 2 heads, 256 keys 19.5 -> 12.7, 700 20.9 -> 23.1.
int short_row(int dtype, int head_dim) { return (dtype == MPA_F32 ? 512 : 1024) * (128 / head_dim); }
long short_pairs(int dtype) { return dtype == MPA_BF16 ? 512 : 256; }

// One decode launch: rows [c0, c1) of Batch::decode.
struct DecodeLaunch {
  size_t c0 = 0, c1 = 0;
  int range_blocks = 0;  // DecodePlan::range_blocks
  long items = 0;        // parts of its rows
  bool split = false;    // some row has several parts
};

// A row's parts when its nb blocks begin at block `at` of the launch's.
long range_parts(long at, long nb, int range) { return (at + nb - 1) / range - at / range + 1; }

// The decode launches, with ranges where they pay (`ranges`) or all rows
// split on their own.  `split` takes the nominal part size when it is needed
// and 0.  MPA_DECODE_RANGE (blocks; 0: none) overrides the choice of ranges
// for tuning sweeps and tests; MPA_SPLIT_TOKENS asks for row splits.
std::vector<DecodeLaunch> decode_layout(const mpa_shape* sh, const Batch& b, const int32_t* seq_lens, int* split,
                                        bool ranges) {
  std::vector<DecodeLaunch> out;
  const int range_env = env_decode_range();
  const int forced = range_env < 0 && env_split_tokens() > 0 ? 0 : range_env;
  const long slots = ranges && forced != 0 ? mpa::decode_wave_slots(sh->dtype, sh->head_dim, true) : 0;
  for (size_t c0 = 0; c0 < b.decode.size(); c0 += mpa::kMaxPlanSeqs) {
    DecodeLaunch d;
    d.c0 = c0;
    d.c1 = std::min(b.decode.size(), c0 + mpa::kMaxPlanSeqs);
    long blocks = 0;
    for (size_t k = d.c0; k < d.c1; ++k) blocks += row_blocks(seq_lens[b.decode[k]]);
    int longest = 0;
    for (size_t k = d.c0; k < d.c1; ++k) longest = std::max(longest, seq_lens[b.decode[k]]);
    if (forced < 0 && longest <= short_row(sh->dtype, sh->head_dim) &&
        (long)(d.c1 - d.c0) * sh->num_kv_heads <= short_pairs(sh->dtype))
      d.range_blocks = -1;
    else if (ranges && blocks < (1L << 30)) {  // block counts are 32 bits in the plan
      auto range_over = [&](long waves) {
        const long per_head = std::max(1L, waves / sh->num_kv_heads);
        return (blocks + per_head - 1) / per_head;
      };
      long range = range_over(slots);
      if (forced > 0) {
        d.range_blocks = forced;
      } else if (slots > 0 && range >= range_min_blocks(sh->dtype, sh->head_dim)) {
        if (sh->dtype != MPA_FP8 && range >= kFewerWavesBlocks) range = range_over(slots * 3 / 4);
        if (ranges_pay(sh, b, seq_lens, d.c0, d.c1, (int)range, split)) d.range_blocks = (int)range;
      }
    }
    if (d.range_blocks == 0 && *split == 0) *split = choose_split(sh, b, seq_lens);
    long at = 0;
    for (size_t k = d.c0; k < d.c1; ++k) {
      const int L = seq_lens[b.decode[k]];
      const long parts = d.range_blocks > 0   ? range_parts(at, row_blocks(L), d.range_blocks)
                         : d.range_blocks < 0 ? 1
                                              : (long)row_split(L, *split).parts;
      at += row_blocks(L);
      d.items += parts;
      d.split |= parts > 1;
    }
    out.push_back(d);
  }
  return out;
}

// Query tokens per prefill tile: 256 (token, head) rows for the MFMA kernel
// (bf16 and fp8 caches), 64 for the generic kernel (f32).
int q_tile(const mpa_shape* sh) {
  const int rows = sh->dtype == MPA_F32 ? mpa::kPrefillRows : mpa::kPrefillRowsMfma;
  return rows / (sh->num_q_heads / sh->num_kv_heads);
}

// Launch errors are read with hipGetLastError() after each launch.  That
// call also returns an error left behind by an earlier runtime call on this
// thread that nobody collected -- e.g. hipErrorNotReady from another
// library's stream or event query -- so it is cleared once, after
// validation, before this call's first launch.
void clear_stale_hip_error() { (void)hipGetLastError(); }

size_t workspace_bytes(const mpa_shape* sh, long items) {
  const size_t per = (size_t)sh->num_q_heads * (sh->head_dim + 2) * sizeof(float);
  return items * per;
}

// The prefill work, in launch order: each segment is tokens [tok0, tok0 +
// ntok) of a chunk (whole query tiles, or the chunk's rest) in nsplit KV
// splits.  A segment's query tiles times its splits and the KV heads are its
// workgroups, and each workgroup holds a whole CU.  With several splits the
// cached prefix is divided into parts of kPrefillMinSplitTiles 64-key tiles
// or more; the last split also takes the chunk's own keys (and the causal
// diagonal), so every split holds keys of every row.  bf16 and fp8 caches (the
// MFMA kernel); f32 chunks are not split.
struct PrefillSegment {
  int seq = 0, tok0 = 0, ntok = 0;
  int nsplit = 1;
  int tiles = 0;        // 64-key tiles of every split but the last
  long item_base = 0;   // first workspace slot of its partials
};

// `want` splits, or as many as the prefix of `prefix` keys allows.
void split_segment(PrefillSegment* g, int prefix, int want) {
  const int np = prefix / 64;  // whole 64-key tiles of the prefix
  const int ct = (g->ntok + 63) / 64;
  const int n = std::min({want, 1 + np / mpa::kPrefillMinSplitTiles, 64});
  g->nsplit = std::max(1, n);
  g->tiles = n < 2 ? 0 : std::min((np + ct + n - 1) / n, np / (n - 1));
}

// Every chunk whole or in up to `want` splits, in batch order.
std::vector<PrefillSegment> split_layout(const Batch& b, const int32_t* seq_lens, const int32_t* qsl, int want) {
  std::vector<PrefillSegment> out(b.prefill.size());
  for (size_t k = 0; k < b.prefill.size(); ++k) {
    const int s = b.prefill[k];
    out[k].seq = s;
    out[k].ntok = qsl[s + 1] - qsl[s];
    split_segment(&out[k], seq_lens[s] - out[k].ntok, want);
  }
  return out;
}

// The makespan of jobs dealt in order, each `copies` times over, to `slots`
// slots that take the next job when free.  When the copies divide the slots
// the schedule is that many times the same one, so one is simulated.
double list_makespan(const std::vector<double>& jobs, int copies, int slots) {
  if (slots % copies == 0) {
    slots /= copies;
    copies = 1;
  }
  if ((long)jobs.size() * copies <= slots) return jobs.empty() ? 0.0 : *std::max_element(jobs.begin(), jobs.end());
  std::vector<double> heap((size_t)slots, 0.0);  // when each slot is free, least first
  double makespan = 0.0;
  for (double job : jobs)
    for (int c = 0; c < copies; ++c) {
      const double end = heap[0] + job;
      makespan = std::max(makespan, end);
      size_t i = 0;
      for (;;) {  // the first slot is free at `end`: sift it down
        size_t k = 2 * i + 1;
        if (k >= heap.size()) break;
        if (k + 1 < heap.size() && heap[k + 1] < heap[k]) ++k;
        if (heap[k] >= end) break;
        heap[i] = heap[k];
        i = k;
      }
      heap[i] = end;
    }
  return makespan;
}

// The work units of segment g in unit order, in query tiles of qt tokens:
// f(64-key tiles of the unit).
template <typename F>
void segment_units(const PrefillSegment& g, const int32_t* seq_lens, const int32_t* qsl, int qt, F f) {
  const int P = seq_lens[g.seq] - (qsl[g.seq + 1] - qsl[g.seq]) + g.tok0;  // keys before the segment
  for (int q = 0; q < (g.ntok + qt - 1) / qt; ++q) {
    const int all = (P + std::min(q * qt + qt, g.ntok) + 63) / 64;
    for (int x = 0; x < g.nsplit; ++x) f(x == g.nsplit - 1 ? all - x * g.tiles : g.tiles);
  }
}

// Predicted device time of the prefill launches for a split layout: per
// launch (kMaxPrefillSeqs chunks), the makespan of its workgroups -- each
// wg_us + tile_us per 64-key tile -- dealt in launch order (the longest
// query tiles first) to `slots` slots that take the next workgroup when
// free; plus, when a chunk of the launch is split, the merge: merge_us +
// merge_row_us per partial (token, q head, split) row.  A launch whose time
// cannot be below `cutoff` may be given its lower bound instead.
// `work_us` (may be null) takes the work of all slots.
double prefill_time(const mpa_shape* sh, const int32_t* seq_lens, const int32_t* qsl,
                    const std::vector<PrefillSegment>& segments, double wg_us, double tile_us, int slots,
                    double merge_us, double merge_row_us, double cutoff = INFINITY, double* work_us = nullptr) {
  const int qt = q_tile(sh);
  double total = 0.0;
  std::vector<double> jobs;
  if (work_us) *work_us = 0.0;
  for (size_t c0 = 0; c0 < segments.size(); c0 += mpa::kMaxPrefillSeqs) {
    const size_t c1 = std::min(segments.size(), c0 + mpa::kMaxPrefillSeqs);
    jobs.clear();  // the work units' times, in unit order
    double partial_rows = 0.0, work = 0.0, shortest = INFINITY;
    for (size_t k = c0; k < c1; ++k) {
      const PrefillSegment& g = segments[k];
      if (g.nsplit > 1) partial_rows += (double)g.ntok * sh->num_q_heads * g.nsplit;
      segment_units(g, seq_lens, qsl, qt, [&](int tiles) {
        jobs.push_back(wg_us + tile_us * tiles);
        work += jobs.back();
        shortest = std::min(shortest, jobs.back());
      });
    }
    if (work_us) *work_us += work * sh->num_kv_heads;
    std::reverse(jobs.begin(), jobs.end());  // blockIdx order: the last unit first, each unit once per KV head
    const double merge = partial_rows > 0 ? merge_us + merge_row_us * partial_rows : 0.0;
    const long units = (long)jobs.size() * sh->num_kv_heads;
    const double bound = std::max(work * sh->num_kv_heads / slots, (units + slots - 1) / slots * shortest);
    total += (units && bound + merge >= cutoff ? bound : list_makespan(jobs, sh->num_kv_heads, slots)) + merge;
  }
  return total;
}

// The planner's own figures for prefill_time (those of mpa_default_rates),
// fixed so that a batch always gets the same plan.
constexpr double kPlanWgUs = 18.0;
constexpr double kPlanTileUs = 1.85;
constexpr double kPlanMergeUs = 3.0;
constexpr double kPlanMergeRowUs = 1.6e-4;
// Balancing a launch that fills the device: what a partial row costs there
// beside the merge (its units store 4 bytes an element, not 2, and run more
// often), fitted to 22 batches of 200-4,000 us; without it the five batches
// whose every chunk was cut in two came out 1-8 % slower than predicted even.
constexpr double kPlanBalanceRowUs = 5e-4;

// The segments (without their workspace slots).
//
// A batch with fewer than two workgroups per CU gets the split count (1, 2,
// ...), for all its chunks, with the shortest predicted prefill time, the
// fewer splits on a tie; counts past the point where every chunk's prefix is
// cut as finely as allowed, or past 8 workgroups per CU, are not tried.
//
// A larger one keeps its chunks whole where their makespan is close to the
// work over the CUs.  The kernel dispatches its units from the last segment
// backwards, each from its longest query tile (the one that sees the most
// keys), so segments are ordered by their longest unit: the longest go first
// and the short ones fill the end of the launch.  Where that leaves more than
// 3 % of the launch idle, chunks whose units are long against a CU's share
// are split (to shares of 1/1.5, 1/2 or 1/3), and then the first query tiles
// of the last segment to run (a quarter of a round of them in 4 splits, or a
// round in 3), whichever is predicted shortest.  Measured on 22 batches of up
// to 4 chunks (us, whole chunks -> this): 3,025 tokens on 613 keys and 439 on
// 35,613 789 -> 659, 6,291 on 15,587 (tail) 3,409 -> 3,166, 2,490 / 1,215 / 423
// on 0 / 1,850 / 36,264 (fp8, d 64) 649 -> 264; none more than 1 % slower.
// With `balance` false only the order is chosen.
// MPA_PREFILL_SPLITS (1..64) overrides the choice for tuning sweeps.
std::vector<PrefillSegment> prefill_segments(const mpa_shape* sh, const Batch& b, const int32_t* seq_lens,
                                             const int32_t* qsl, bool balance) {
  std::vector<PrefillSegment> best = split_layout(b, seq_lens, qsl, 1);
  if (sh->dtype == MPA_F32 || b.prefill.empty()) return best;
  if (const int v = env_prefill_splits(); v > 0) return split_layout(b, seq_lens, qsl, v);
  const int slots = mpa::kPrefillSplitTarget;
  double row_us = kPlanMergeRowUs, margin = 1e-9;
  auto time = [&](const std::vector<PrefillSegment>& v, double cutoff, double* work = nullptr) {
    return prefill_time(sh, seq_lens, qsl, v, kPlanWgUs, kPlanTileUs, slots, kPlanMergeUs, row_us, cutoff, work);
  };
  double best_t = INFINITY;
  auto take_if_shorter = [&](std::vector<PrefillSegment>& v) {
    const double t = time(v, best_t);
    if (t < best_t * (1.0 - margin)) {
      best_t = t;
      best = v;
    }
  };
  long units;
  int most;  // the most splits any chunk can take
  prefill_units(sh, b.prefill, seq_lens, qsl, &units, &most);
  if (!prefill_whole(sh, b.prefill, seq_lens, qsl)) {
    for (int want = 1; want <= most && (want == 1 || units * want <= 8L * slots); ++want) {
      std::vector<PrefillSegment> v = split_layout(b, seq_lens, qsl, want);
      take_if_shorter(v);
    }
    return best;
  }
  auto prefix = [&](const PrefillSegment& g) { return seq_lens[g.seq] - (qsl[g.seq + 1] - qsl[g.seq]) + g.tok0; };
  auto longest = [&](const PrefillSegment& g) {  // tiles of the segment's longest unit
    const int all = (prefix(g) + g.ntok + 63) / 64;
    return std::max(g.tiles, all - (g.nsplit - 1) * g.tiles);
  };
  auto order = [&](std::vector<PrefillSegment>& v) {
    std::stable_sort(v.begin(), v.end(), [&](const PrefillSegment& x, const PrefillSegment& y) {
      return longest(x) != longest(y) ? longest(x) < longest(y) : seq_lens[x.seq] < seq_lens[y.seq];
    });
  };
  order(best);
  if (!balance || most == 1 || units < 2L * slots || best.size() >= (size_t)mpa::kMaxPrefillSeqs) return best;
  double work;
  row_us = kPlanBalanceRowUs;
  margin = 0.04;  // of the prediction, which was up to 9 % low on the batches above
  time(best, 0.0, &work);
  const double share = work / slots;
  // Dealt in any order the units end within the longest one of the share, so
  // most large launches are even without a simulation (60 chunks of 8,192
  // tokens, 10 KV heads: 3.8 ms of host time)
  int unit = 0;
  for (const PrefillSegment& g : best) unit = std::max(unit, longest(g));
  if (kPlanWgUs + kPlanTileUs * unit < 0.03 * share) return best;
  best_t = time(best, INFINITY);
  if (best_t < 1.03 * share) return best;
  const std::vector<PrefillSegment> whole = best;
  for (double parts : {1.5, 2.0, 3.0}) {
    std::vector<PrefillSegment> v = whole;
    bool any = false;
    for (PrefillSegment& g : v) {
      const double unit = kPlanTileUs * ((prefix(g) + g.ntok + 63) / 64);
      const int want = (int)std::min(16.0, ceil(unit * parts / share));
      if (want > 1) split_segment(&g, prefix(g), want);
      any |= g.nsplit > 1;
    }
    if (!any) continue;
    order(v);
    take_if_shorter(v);
  }
  if (best_t < 1.03 * share || best[0].nsplit > 1) return best;
  margin = 0.01;  // few partial rows: within 3 %
  const int qt = q_tile(sh);
  const int round = std::max(1, slots / sh->num_kv_heads);  // query tiles of one round
  const std::vector<PrefillSegment> from = best;
  for (int n : {4, 3}) {
    const int tail = std::max(1, n == 4 ? round / 4 : round);
    PrefillSegment head = from[0];
    PrefillSegment rest = head;
    head.ntok = std::min(head.ntok, tail * qt);
    rest.tok0 += head.ntok;
    rest.ntok -= head.ntok;
    split_segment(&head, prefix(head), n);
    if (head.nsplit < 2) continue;
    std::vector<PrefillSegment> v(1, head);
    if (rest.ntok > 0) v.push_back(rest);
    v.insert(v.end(), from.begin() + 1, from.end());
    take_if_shorter(v);
  }
  return best;
}

// The makespan of jobs dealt in order, each `copies` times over, to CUs that
// hold up to `per` of them at once: first one to every CU, then a second, then
// to whichever has room.  A job on a CU that holds k runs at rate[k - 1].
double shared_makespan(const std::vector<double>& jobs, int copies, int per, std::array<double, 3> rate) {
  size_t cus = mpa::kPrefillSplitTarget;
  if (cus % (size_t)copies == 0) {  // that many times the same schedule
    cus /= copies;
    copies = 1;
  }
  const size_t total = jobs.size() * (size_t)copies;
  if (total <= cus) return jobs.empty() ? 0.0 : *std::max_element(jobs.begin(), jobs.end());
  struct Cu {
    double left[3], at;  // of its jobs, at that time
    int n;
  };
  std::vector<Cu> cu(cus, Cu{{0.0, 0.0, 0.0}, 0.0, 0});
  size_t next = 0;
  for (int r = 0; r < per; ++r)
    for (size_t c = 0; c < cus && next < total; ++c) cu[c].left[cu[c].n++] = jobs[next++ / copies];
  using Event = std::pair<double, int>;  // when a CU's shortest job ends
  std::priority_queue<Event, std::vector<Event>, std::greater<Event>> events;
  auto push = [&](int c) {
    const Cu& u = cu[c];
    if (u.n > 0) events.push({u.at + *std::min_element(u.left, u.left + u.n) / rate[u.n - 1], c});
  };
  for (size_t c = 0; c < cus; ++c) push((int)c);
  double end = 0.0;
  while (!events.empty()) {
    const Event e = events.top();
    events.pop();
    Cu& u = cu[e.second];
    const double done = *std::min_element(u.left, u.left + u.n);
    int n = 0;
    for (int k = 0; k < u.n; ++k)
      if (u.left[k] > done) u.left[n++] = u.left[k] - done;
    u.n = n;
    u.at = end = e.first;
    while (u.n < per && next < total) u.left[u.n++] = jobs[next++ / copies];
    push(e.second);
  }
  return end;
}

// (token, head) rows per workgroup of the bf16 launch of segments [c0, c1).
// The planner counts workgroups of 256 rows (eight waves, one to a CU).
// Launches of few of them may run as workgroups of 128 (four waves, two to a
// CU, or three at head_dim 64): a prompt's tiles grow from one 64-key tile to
// the chunk's length, and half tiles let a long and a short one share a CU and
// fill each other's gaps.  They read K and V twice as often for it, which
// costs up to a tenth where the tiles are alike (a long prefix), so a launch
// takes the form with the shorter predicted time: whole tiles from the makespan
// of the launch order, half tiles from that of CUs which share their rate among
// the workgroups they hold, both with the work per CU (a tile takes longer the
// more CUs are busy).  The figures are fitted to 399 launches, those close to
// the line by what the wrong form costs.  On 230 others of the same ranges the
// form taken is 0.2 % slower than the better one in the mean, and past 13 us
// never slower than whole tiles.  Measured (us, 256 -> 128 rows):
//   d 128: 1,003 tokens of 32 / 8 heads on 500 41.4 -> 33.4, on 2,000 61.0 ->
//     64.2; 2,027 on 0 53.5 -> 49.4, on 8,000 261 -> 272, on 32,000 883 -> 942;
//     3,001 on 0 82.7 -> 79.4, 3,201 87.7 -> 92.2; 2,987 on 2,000 165.9 -> 176.6;
//   d 64: 2,038 of 16 / 2 on 0 38.9 -> 29.5, on 32,000 (KV-split) 301 -> 317;
//     2,539 of 32 / 8 on 2,000 95.8 -> 85.2, on 32,000 755 -> 728.
// The model is not asked where it was not fitted: KV-split launches of
// 128-wide heads stay whole, those of 64-wide heads from 1,024 workgroups on
// are half tiles (0.93-0.97 of the time in 12 launches), and other launches
// past 448, or at 128-wide heads past 128 with several chunks (which meet on a
// CU in no particular order), stay whole.
int prefill_rows_bf16(const mpa_shape* sh, const std::vector<PrefillSegment>& segments, size_t c0, size_t c1,
                      const int32_t* seq_lens, const int32_t* qsl) {
  const int qt = q_tile(sh);
  const bool d64 = sh->head_dim == 64;
  long groups = 0;
  bool split = false;
  for (size_t k = c0; k < c1; ++k) {
    groups += (long)(segments[k].ntok + qt - 1) / qt * segments[k].nsplit * sh->num_kv_heads;
    split |= segments[k].nsplit > 1;
  }
  if (d64 && groups >= 1024) return mpa::kPrefillRowsHalf;
  if (groups >= (d64 || c1 - c0 == 1 ? 448 : 128) || (split && !d64)) return mpa::kPrefillRowsMfma;
  std::vector<double> jobs;  // the workgroups' 64-key tiles and a start, in launch order
  double per_cu = 0.0, longest = 0.0;
  auto make_jobs = [&](int rows, double start) {
    jobs.clear();
    per_cu = longest = 0.0;
    for (size_t k = c0; k < c1; ++k)
      segment_units(segments[k], seq_lens, qsl, rows / (sh->num_q_heads / sh->num_kv_heads), [&](int tiles) {
        jobs.push_back(start + tiles);
        per_cu += tiles;
        longest = std::max(longest, (double)tiles);
      });
    std::reverse(jobs.begin(), jobs.end());
    per_cu *= (double)sh->num_kv_heads / mpa::kPrefillSplitTarget;
  };
  double whole, half;
  make_jobs(mpa::kPrefillRowsMfma, d64 ? 6.0 : 8.0);
  whole = list_makespan(jobs, sh->num_kv_heads, mpa::kPrefillSplitTarget);
  whole = d64 ? 9.46 + 0.66 * whole + 0.327 * per_cu + 0.096 * longest
              : 6.13 + 0.694 * whole + 0.482 * per_cu + 0.444 * longest;
  make_jobs(mpa::kPrefillRowsHalf, d64 ? 2.0 : 8.0);
  if (d64)
    half = 11.43 + 0.408 * per_cu + 0.284 * shared_makespan(jobs, sh->num_kv_heads, 3, {1.0, 0.8, 0.65});
  else
    half = 3.8 + 0.376 * per_cu + 0.744 * shared_makespan(jobs, sh->num_kv_heads, 2, {1.0, 0.75, 0.0});
  return half < whole ? mpa::kPrefillRowsHalf : mpa::kPrefillRowsMfma;
}

// (token, head) rows per workgroup of the f32 launch of segments [c0, c1): 64
// (a tile: four waves of 16 rows, all their keys each) or 16 (eight waves, an
// eighth of the keys each, merged in LDS; four workgroups to a tile).  A wave
// needs 2,048 MFMA cycles per 16 keys and 128 dims in either form.  Up to two
// tiles of a launch run on a CU at once, so one of up to 512 takes as long as
// its longest tile or its longest pair (tile i and i + 256 of the launch);
// 16-row workgroups spread over four times the slots, at the price of reading
// K and V for 16 rows, not 64.  The form with the shorter predicted time is
// taken.  The figures, in 16-key blocks, are fitted to 234 launches of 128-512
// tiles (rms 2-3 %); on those the keys form, where taken, was at most 0.1 %
// slower than tiles, and the better form was missed by 5 % at most.  Measured
// (us, tiles -> keys; tokens on prefix):
//   d 128: 128 tiles (8 / 2 heads, 1,024 on 500) 115.9 -> 56.7, 200 (1,600 on
//     2,000) 262.9 -> 244.2, on 8,000 670 -> 745; 248 (1,984 on 500) 183.5 ->
//     148.9, 256 (32 / 8, 512 on 500) 79.9 -> 88.2, 264 (528 on 500) 137.3 ->
//     103.4, 496 (992 on 500) 215.9 -> 213.3, 504 (8 / 2, 4,032 on 500) 601 -> 470;
//   d 64: 128 (16 / 2, 512 on 500) 43.8 -> 23.9, 200 (64 / 8, 200 on 0) 13.5 ->
//     18.6, 496 (496 on 0) 32.3 -> 47.1, 496 (16 / 2, 1,984 on 0) 111.0 -> 101.3.
// Larger launches keep whole tiles (600 tiles: 0.82-1.42 of their time in the
// keys form, which the model does not tell apart).
int prefill_rows_f32(const mpa_shape* sh, const std::vector<PrefillSegment>& segments, size_t c0, size_t c1,
                     const int32_t* seq_lens, const int32_t* qsl) {
  const int G = sh->num_q_heads / sh->num_kv_heads;
  const int qt = q_tile(sh);
  const int hkv = sh->num_kv_heads;
  const size_t slots = mpa::kPrefillSplitTarget;
  size_t tiles = 0;
  for (size_t k = c0; k < c1; ++k) tiles += (size_t)(segments[k].ntok + qt - 1) / qt * hkv;
  if (tiles > 2 * slots) return mpa::kPrefillRows;
  const bool d64 = sh->head_dim == 64;
  std::vector<int> blocks;   // of the tiles, in launch order, each once per KV head
  std::vector<double> jobs;  // the 16-row workgroups of one KV head, in launch order
  for (size_t k = c1; k-- > c0;) {
    const PrefillSegment& g = segments[k];
    const int P = seq_lens[g.seq] - (qsl[g.seq + 1] - qsl[g.seq]) + g.tok0;
    for (int q = (g.ntok + qt - 1) / qt; q-- > 0;) {
      const int first = q * qt;
      blocks.insert(blocks.end(), hkv, row_blocks(P + std::min(first + qt, g.ntok)));
      for (int sub = 0; sub < 4 && first + sub * 16 / G < g.ntok; ++sub) {
        const int nb = row_blocks(P + std::min(first + std::min((sub * 16 + 15) / G + 1, qt), g.ntok));
        jobs.push_back((d64 ? 2.35 : 3.4) + (d64 ? 1.18 : 2.75) * ((nb + 7) / 8));
      }
    }
  }
  int longest = 0, pair = 0;
  for (size_t i = 0; i < tiles; ++i) {
    longest = std::max(longest, blocks[i]);
    if (i + slots < tiles) pair = std::max(pair, blocks[i] + blocks[i + slots]);
  }
  const double whole = (d64 ? 6.1 : 6.5) + std::max((d64 ? 0.611 : 1.138) * longest, (d64 ? 0.566 : 1.323) * pair);
  const double keys = (d64 ? 4.5 : 3.7) + list_makespan(jobs, hkv, (int)slots);
  return keys < 0.98 * whole ? mpa::kPrefillRowsKeys : mpa::kPrefillRows;
}

// The same for a launch of any cache type.
int prefill_rows(const mpa_shape* sh, const std::vector<PrefillSegment>& segments, size_t c0, size_t c1,
                 const int32_t* seq_lens, const int32_t* qsl) {
  if (sh->dtype == MPA_F32) return prefill_rows_f32(sh, segments, c0, c1, seq_lens, qsl);
  if (sh->dtype == MPA_FP8) return mpa::kPrefillRowsMfma;
  return prefill_rows_bf16(sh, segments, c0, c1, seq_lens, qsl);
}

// Gives split segments their workspace slots, from first_item on; returns the
// number of slots given.
long assign_prefill_items(std::vector<PrefillSegment>* segments, long first_item) {
  long n = 0;
  for (PrefillSegment& g : *segments)
    if (g.nsplit > 1) {
      g.item_base = first_item + n;
      n += (long)g.nsplit * g.ntok;
    }
  return n;
}

// Everything a step's launches follow from.  The partial results of split
// decode rows come first in the workspace, those of split chunks after them.
struct StepPlan {
  Batch batch;
  int split = 0;  // nominal tokens per part of rows split on their own
  std::vector<DecodeLaunch> decode;
  std::vector<PrefillSegment> prefill;
  std::vector<int> prefill_rows;      // (token, head) rows per workgroup of each prefill launch
  long items = 0;                     // workspace slots
  bool decode_split = false, prefill_split = false;  // some row / chunk has several parts
};

StepPlan make_plan(const mpa_shape* sh, const int32_t* seq_lens, const int32_t* qsl) {
  StepPlan p;
  p.batch = classify(sh, qsl);
  auto total = [](const std::vector<DecodeLaunch>& v) {
    long n = 0;
    for (const auto& d : v) n += d.items;
    return n;
  };
  p.decode = decode_layout(sh, p.batch, seq_lens, &p.split, true);
  p.prefill = prefill_segments(sh, p.batch, seq_lens, qsl, true);
  auto place = [&] {
    const long ditems = total(p.decode);
    p.items = ditems + assign_prefill_items(&p.prefill, ditems);
    return workspace_bytes(sh, p.items) <= MPA_SCRATCH_BYTES;
  };
  if (!place() && env_decode_range() < 0) {
    // Ranges cut every row, also short ones, and balancing splits chunks, so
    // their partial results can take more room than those of row splits and
    // whole chunks.  A step past the fixed array of
    // mpa_append_attention_noalloc does without them where that takes less.
    p.prefill = prefill_segments(sh, p.batch, seq_lens, qsl, false);
    if (!place()) {
      const std::vector<DecodeLaunch> rows = decode_layout(sh, p.batch, seq_lens, &p.split, false);
      if (total(rows) < total(p.decode)) {
        p.decode = rows;
        place();
      }
    }
  }
  if (p.split == 0 && !p.decode.empty() && p.decode[0].range_blocks > 0)
    p.split = (int)std::min((long)INT32_MAX, (long)p.decode[0].range_blocks * kBlock);
  if (p.split == 0) p.split = std::max(1024, short_row(sh->dtype, sh->head_dim));  // no row is split
  for (const auto& d : p.decode) p.decode_split |= d.split;
  for (const auto& c : p.prefill) p.prefill_split |= c.nsplit > 1;
  for (size_t c0 = 0; c0 < p.prefill.size(); c0 += mpa::kMaxPrefillSeqs)
    p.prefill_rows.push_back(
        prefill_rows(sh, p.prefill, c0, std::min(p.prefill.size(), c0 + mpa::kMaxPrefillSeqs), seq_lens, qsl));
  return p;
}

// The plan of a valid batch, from a per-thread memo of the last one: one step
// asks for its plan several times (workspace sizing, the append, each
// attention half, the step model).  The key is everything the plan depends
// on: the shape's heads, head_dim and dtype, the exact seq_lens and
// query_start_loc, the device (its wave capacity) and the tuning overrides
// in the environment.  The reference holds until the thread's next call.
const StepPlan& step_plan(const mpa_shape* sh, const int32_t* seq_lens, const int32_t* qsl) {
  struct Memo {
    int32_t key[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
    std::vector<int32_t> seq_lens, qsl;
    StepPlan plan;
  };
  thread_local Memo m;
  // an empty batch may come without metadata (check_batch accepts null
  // arrays when num_seqs is 0): its query_start_loc is {0}
  static const int32_t kEmptyQsl[1] = {0};
  if (sh->num_seqs == 0 && !qsl) qsl = kEmptyQsl;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  const int32_t key[8] = {sh->num_q_heads, sh->num_kv_heads, sh->head_dim, (int32_t)sh->dtype, dev,
                          env_split_tokens(), env_prefill_splits(), env_decode_range()};
  const size_t n = (size_t)sh->num_seqs;
  if (memcmp(key, m.key, sizeof key) != 0 || m.seq_lens.size() != n || m.qsl.size() != n + 1 ||
      (n && memcmp(m.seq_lens.data(), seq_lens, n * sizeof(int32_t)) != 0) ||
      memcmp(m.qsl.data(), qsl, (n + 1) * sizeof(int32_t)) != 0) {
    m.key[0] = -1;  // no plan while it is made
    m.seq_lens.assign(seq_lens, seq_lens + n);
    m.qsl.assign(qsl, qsl + n + 1);
    m.plan = make_plan(sh, seq_lens, qsl);
    memcpy(m.key, key, sizeof key);
  }
  return m.plan;
}

// MPA_DEBUG=1 (read per call): before an append, the cache slots it writes
// must be pairwise distinct, and none may hold a key that a sequence of the
// step reads (prefix blocks shared between sequences are read-only).  Needs
// the host copy of the block tables; without it the check cannot run and
// the call is rejected.  Costs a pass over every key of the step.
bool debug_checks() {
  const char* e = getenv("MPA_DEBUG");
  return e && e[0] == '1' && e[1] == '\0';
}

int check_append_slots(const mpa_shape* sh, const int32_t* seq_lens, const int32_t* qsl, const int32_t* bt) {
  if (!bt) return MPA_ERR_INVALID;
  std::unordered_set<int64_t> written;
  auto slot_of = [&](int s, int p) {
    return (int64_t)bt[(size_t)s * sh->max_blocks_per_seq + p / kBlock] * kBlock + p % kBlock;
  };
  for (int s = 0; s < sh->num_seqs; ++s) {
    const int ql = qsl[s + 1] - qsl[s];
    for (int p = seq_lens[s] - ql; p < seq_lens[s]; ++p)
      if (!written.insert(slot_of(s, p)).second) return MPA_ERR_INVALID;  // two tokens, one slot
  }
  for (int s = 0; s < sh->num_seqs; ++s) {
    const int ql = qsl[s + 1] - qsl[s];
    if (ql == 0) continue;
    for (int p = 0; p < seq_lens[s] - ql; ++p)
      if (written.count(slot_of(s, p))) return MPA_ERR_INVALID;  // overwrites a key that is read
  }
  return MPA_OK;
}

// Whether single tokens are written with non-temporal stores.  What they leave
// in part-written lines slows the decode that follows when it streams more
// than the caches hold; below that a plain store is complete sooner.  Append
// and decode, us, plain -> non-temporal: bf16 none slower (256 rows of 300, 2
// heads of 128, 78 MB 30.5 -> 30.5; 256 of 600, 8 heads 133.7 -> 130.0); f32
// 26 MB 25.1 -> 26.0, 59 MB 27.9 -> 29.6, 134 MB 32.1 -> 32.7, 315 MB 69.8 ->
// 66.7; fp8 26 MB 27.8 -> 29.6, 92 MB 28.0 -> 29.2, 184 MB (100 rows of 900 in
// the mean) 47.9 -> 46.3, 393 MB (128 of 1,500) 79.9 -> 78.3, but 157 and 315
// MB as 256 rows of 300 and 600 38.8 -> 42.3 and 80.4 -> 84.8: a store there
// is a single code, 2,048 of them for a row's token.
bool token_stores_stream(const mpa_shape* sh, const Batch& b, const int32_t* seq_lens) {
  if (sh->dtype == MPA_BF16) return true;
  double keys = 0.0;
  for (int s : b.decode) keys += seq_lens[s];
  if (sh->dtype == MPA_FP8 && keys < 800.0 * b.decode.size()) return false;
  return keys * sh->num_kv_heads * sh->head_dim * 2 * (sh->dtype == MPA_F32 ? 4 : 1) >= 160e6;
}

// The append launches (plain, or with the rotary embedding when rope is
// given).
int run_append(const mpa_shape* shape, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
               const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
               const int32_t* seq_lens_host, const int32_t* query_start_loc_host, const int32_t* block_tables_host,
               const mpa::RopeArgs* rope, void* stream, bool multi_only = false) {
  int rc = check_batch(shape, seq_lens_host, query_start_loc_host, block_tables_host, true);
  if (rc != MPA_OK) return rc;
  if (shape->total_q_tokens == 0) return MPA_OK;
  if (debug_checks()) {
    rc = check_append_slots(shape, seq_lens_host, query_start_loc_host, block_tables_host);
    if (rc != MPA_OK) return rc;
  }
  if (!k_new || !v_new || !k_cache || !v_cache || !block_tables || !seq_lens || !query_start_loc)
    return MPA_ERR_INVALID;
  mpa::AppendArgs a;
  a.k_new = k_new;
  a.v_new = v_new;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.block_tables = block_tables;
  a.hkv = shape->num_kv_heads;
  a.mb = shape->max_blocks_per_seq;
  a.nb = shape->num_blocks;
  a.inv_k_scale = shape->dtype == MPA_FP8 ? 1.f / shape->k_scale : 1.f;
  a.inv_v_scale = shape->dtype == MPA_FP8 ? 1.f / shape->v_scale : 1.f;
  const Batch b = classify(shape, query_start_loc_host);
  a.nt = token_stores_stream(shape, b, seq_lens_host);
  clear_stale_hip_error();
  // multi-token sequences one wave per (cache block, KV head); with the rotary
  // embedding (appended by no attention call) the single tokens beside them
  // too, where one launch holds all
  std::vector<int> blocks(b.prefill);
  bool tokens_left = !multi_only;
  if (rope && !b.prefill.empty() && b.prefill.size() + b.decode.size() <= (size_t)mpa::kMaxPrefillSeqs) {
    blocks.insert(blocks.end(), b.decode.begin(), b.decode.end());
    tokens_left = false;
  }
  for (size_t c0 = 0; c0 < blocks.size(); c0 += mpa::kMaxPrefillSeqs) {
    mpa::AppendBlockPlan p;
    p.n_seqs = (int32_t)(std::min(blocks.size(), c0 + mpa::kMaxPrefillSeqs) - c0);
    int units = 0, tokens = 0;
    for (int k = 0; k < p.n_seqs; ++k) {
      const int s = blocks[c0 + k];
      const int ql = query_start_loc_host[s + 1] - query_start_loc_host[s];
      const int pos0 = seq_lens_host[s] - ql;
      p.seq[k] = s;
      p.row0[k] = query_start_loc_host[s];
      p.pos0[k] = pos0;
      p.ntok[k] = ql;
      p.unit_start[k] = units;
      p.tok_start[k] = tokens;
      units += (pos0 + ql - 1) / kBlock - pos0 / kBlock + 1;
      tokens += ql;
    }
    p.unit_start[p.n_seqs] = units;
    p.tok_start[p.n_seqs] = tokens;
    if (mpa::launch_append_blocks(a, p, rope, shape->dtype, shape->head_dim, (hipStream_t)stream) != hipSuccess)
      return MPA_ERR_HIP;
  }
  // single-token sequences one wave per token, unless the decode kernel
  // appends them
  for (size_t c0 = 0; tokens_left && c0 < b.decode.size(); c0 += mpa::kMaxPlanSeqs) {
    mpa::AppendPlan p;
    p.n_seqs = (int32_t)(std::min(b.decode.size(), c0 + mpa::kMaxPlanSeqs) - c0);
    for (int k = 0; k < p.n_seqs; ++k) {
      const int s = b.decode[c0 + k];
      p.seq[k] = s;
      p.row[k] = query_start_loc_host[s];
      p.pos[k] = seq_lens_host[s] - 1;
    }
    hipError_t e = rope ? mpa::launch_rope_append(a, p, *rope, shape->dtype, shape->head_dim, (hipStream_t)stream)
                        : mpa::launch_append(a, p, shape->dtype, shape->head_dim, (hipStream_t)stream);
    if (e != hipSuccess) return MPA_ERR_HIP;
  }
  return MPA_OK;
}

}  // namespace

namespace {

// The rate of a decode launch whose rows are dealt as ranges, over that of
// row splits (mpa_rates::decode_gbs): 6,550-7,040 GB/s on the agentic, lent,
// budget and longctx steps against the 5,880 fitted to row splits.
constexpr double kRangeSpeed = 1.145;
// The same launch on 1, 2 and 3 quarters of the CUs, over the share of its
// speed that row splits keep there (mpa_rates::coexec_decode_q1..q3): one round
// of workgroups on three quarters, three on one (0.476 of the speed on the
// whole device, 14 steps) and an uneven two on half of them (0.667).
constexpr double kRangeShare[4] = {1.0, 0.9, 0.8, 1.0};
// And what side by side the halves lose then, over coexec_slowdown's excess of
// 1: on 14 steps (agentic, lent, budget and longctx over several seeds, two TP4
// shares) the picks with 1.06 and 130 us are 1.2 % slower than the best mode
// in the mean and none slower than one stream; with 1.15, agentic (seed 0) runs
// on one stream at 3,664 us (3,372 with decode on a quarter) and budget4096 at
// 1,352 (1,240 on three).
constexpr double kRangeOverlap = 0.4;

// The step-time model (mpa_predict_step), shared with the mode planner.
mpa_step_time model_step(const mpa_shape* shape, const StepPlan& plan, const int32_t* seq_lens_host,
                         const int32_t* qsl_host, const mpa_rates& r) {
  const Batch& b = plan.batch;
  const double elem = 2.0;  // bf16
  const double row_bytes = (double)shape->num_kv_heads * shape->head_dim * elem;  // one token's K (or V)
  mpa_step_time t = {0.0, 0.0, 0.0, 0.0};

  // append, launch by launch as run_append issues them: every new token's K
  // and V read once and written once
  for (size_t c0 = 0; c0 < b.decode.size(); c0 += mpa::kMaxPlanSeqs) {
    const double tokens = (double)(std::min(b.decode.size(), c0 + mpa::kMaxPlanSeqs) - c0);
    t.append_us += r.append_fixed_us + 4.0 * row_bytes * tokens / (r.append_gbs * 1e3);
  }
  for (size_t c0 = 0; c0 < b.prefill.size(); c0 += mpa::kMaxPrefillSeqs) {
    double tokens = 0.0;
    for (size_t k = c0; k < std::min(b.prefill.size(), c0 + mpa::kMaxPrefillSeqs); ++k)
      tokens += qsl_host[b.prefill[k] + 1] - qsl_host[b.prefill[k]];
    t.append_us += std::max(r.append_block_us, 4.0 * row_bytes * tokens / (r.append_block_gbs * 1e3));
  }

  // decode, launch by launch as run_attention issues them
  const double head_bytes = 2.0 * shape->head_dim * elem;  // K + V of one token and KV head
  for (const DecodeLaunch& d : plan.decode) {
    double bytes = 0.0, wave = 0.0;
    for (size_t k = d.c0; k < d.c1; ++k) {
      const int L = seq_lens_host[b.decode[k]];
      bytes += (double)L * head_bytes * shape->num_kv_heads;
      // the most keys one wave goes over; a short row's eight waves share it
      const int part = d.range_blocks < 0 ? short_row(shape->dtype, shape->head_dim) / 8 : row_split(L, plan.split).tokens;
      if (d.range_blocks <= 0) wave = std::max(wave, (double)std::min(L, part) * head_bytes);
    }
    if (d.range_blocks > 0) wave = (double)d.range_blocks * kBlock * head_bytes;
    const double gbs = r.decode_gbs * (d.range_blocks > 0 ? kRangeSpeed : 1.0);
    t.decode_us += r.decode_fixed_us + std::max(bytes / (gbs * 1e3), wave / (r.decode_wave_gbs * 1e3));
    if (d.split) t.decode_us += r.merge_us;
  }

  // prefill: each launch's workgroups, in launch order (longest query tiles
  // first), on prefill_slots slots that take the next workgroup when free
  t.prefill_us = prefill_time(shape, seq_lens_host, qsl_host, plan.prefill, r.prefill_wg_us, r.prefill_tile_us,
                              r.prefill_slots, r.prefill_merge_us, r.prefill_merge_row_us);
  bool few = false;
  for (int s : b.prefill) few |= seq_lens_host[s] - (qsl_host[s + 1] - qsl_host[s]) < mpa::kFewKeys;
  if (few) t.prefill_us += r.prefill_fixup_us;
  t.step_us = t.append_us + t.decode_us + t.prefill_us;
  return t;
}

int check_model_inputs(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host,
                       const mpa_rates& r) {
  int rc = check_batch(shape, seq_lens_host, qsl_host, nullptr, false);
  if (rc != MPA_OK) return rc;
  if (shape->dtype != MPA_BF16) return MPA_ERR_UNSUPPORTED;
  if (!(r.append_gbs > 0) || !(r.append_block_gbs > 0) || !(r.decode_gbs > 0) || !(r.decode_wave_gbs > 0) ||
      r.prefill_slots <= 0)
    return MPA_ERR_INVALID;
  return MPA_OK;
}

}  // namespace

extern "C" {

const char* mpa_status_string(int status) {
  switch (status) {
    case MPA_OK: return "ok";
    case MPA_ERR_INVALID: return "invalid argument or batch metadata";
    case MPA_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case MPA_ERR_WORKSPACE: return "workspace missing, too small or not 16-byte aligned";
    case MPA_ERR_HIP: return "HIP launch error";
    case MPA_ERR_SCRATCH: return "batch needs more than the library's fixed scratch array (MPA_SCRATCH_BYTES)";
    default: return "unknown status";
  }
}

int mpa_get_plan_info(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host,
                      mpa_plan_info* info) {
  if (!info) return MPA_ERR_INVALID;
  int rc = check_batch(shape, seq_lens_host, qsl_host, nullptr, false);
  if (rc != MPA_OK) return rc;
  const StepPlan& plan = step_plan(shape, seq_lens_host, qsl_host);
  const Batch& b = plan.batch;
  info->num_decode_seqs = (int32_t)b.decode.size();
  info->num_prefill_seqs = (int32_t)b.prefill.size();
  // the nominal part size: that of the first launch's ranges, if it has them
  const bool ranged = !plan.decode.empty() && plan.decode[0].range_blocks > 0;
  info->split_tokens = ranged ? (int32_t)std::min((long)INT32_MAX, (long)plan.decode[0].range_blocks * kBlock) : plan.split;
  info->num_decode_items = 0;
  for (const auto& d : plan.decode) info->num_decode_items += (int32_t)d.items;
  long tiles = 0;
  const int qt = q_tile(shape);
  int max_split = b.prefill.empty() ? 0 : 1;
  for (const PrefillSegment& g : plan.prefill) {
    tiles += (long)(g.ntok + qt - 1) / qt * g.nsplit;
    max_split = std::max(max_split, g.nsplit);
  }
  info->num_prefill_tiles = (int32_t)(tiles * shape->num_kv_heads);
  info->prefill_max_splits = max_split;
  info->decode_launches = (int32_t)plan.decode.size();
  return MPA_OK;
}

int mpa_get_prefill_rows(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host, int32_t launch,
                         int32_t* rows) {
  if (!rows || launch < 0) return MPA_ERR_INVALID;
  int rc = check_batch(shape, seq_lens_host, qsl_host, nullptr, false);
  if (rc != MPA_OK) return rc;
  const StepPlan& plan = step_plan(shape, seq_lens_host, qsl_host);
  if ((size_t)launch >= plan.prefill_rows.size()) return MPA_ERR_INVALID;
  *rows = plan.prefill_rows[launch];
  return MPA_OK;
}

void mpa_default_rates(mpa_rates* r) {
  if (!r) return;
  // Least-squares fit (log error) to the phase times bench.py measured on
  // one MI355X for decode8b, lent, agentic, budget0/256/1024/4096 and
  // longctx (seed 0, each phase less the ~5 us of its event record); the
  // merge, few-key and wave figures are single kernel times from rocprofv3.
  // The append figures are fitted to the append phases alone: the
  // per-token launch from decode8b and budget0, the per-block launch (a
  // latency floor, then about 3.7 TB/s) from lent, budget4096 and longctx.
  r->append_fixed_us = 3.9;
  r->append_gbs = 545.0;
  r->append_block_us = 17.0;
  r->append_block_gbs = 3700.0;
  // decode: refitted to the decode half alone after its cache reads became
  // non-temporal (the fit puts the launch's fixed cost inside the rate)
  r->decode_fixed_us = 0.0;
  r->decode_gbs = 5880.0;
  r->decode_wave_gbs = 4.8;
  r->merge_us = 5.0;
  // prefill: refitted to the prefill half alone (lent, agentic, the budget
  // chunks, longctx) on two devices whose prefill rates differ by 5-7 %,
  // the mean of the two least-squares fits (12 + 1.80 per tile and 11.9 +
  // 1.76 against 12.1 + 1.85)
  r->prefill_wg_us = 12.0;
  r->prefill_tile_us = 1.80;
  r->prefill_merge_us = 3.0;
  r->prefill_merge_row_us = 1.6e-4;
  // A partitioned step's fixed cost beyond the model (the cross-stream waits,
  // and interference that the slowdown factor underrates on short steps):
  // fitted with coexec_slowdown, on a grid, to the four modes measured on
  // agentic, lent, budget4096, budget1024 and longctx, and on the TP4 shares
  // of agentic, lent and budget4096: the lowest mean regret of the
  // planner's choice with no choice slower than one stream is at slowdown
  // 1.10; the slowdown is one grid step above it (1.15), a margin for the
  // few percent that step times move between devices
  r->coexec_fixed_us = 130.0;
  // the few-key rows' second pass over their first key tile adds less than
  // a tile to one workgroup, which the makespan absorbs
  r->prefill_fixup_us = 0.0;
  r->prefill_slots = 256;
  // CU-partitioned co-execution (mpa_plan_coexec), measured on agentic, lent,
  // budget4096, budget1024 and longctx, each half alone on its CU set: the
  // decode half's speed on 1, 2 and 3 quarters of every XCD's CUs relative
  // to the whole device, the prefill half's likewise (faster than its share
  // of the CUs: fewer CUs contend for the same HBM and L2), medians over the
  // five; and the slowdown of the two halves side by side over the slower of
  // them alone (shared HBM, L2 and MALL)
  r->coexec_decode_q1 = 0.53;
  r->coexec_decode_q2 = 0.83;
  r->coexec_decode_q3 = 1.0;
  r->coexec_prefill_q1 = 0.33;
  r->coexec_prefill_q2 = 0.60;
  r->coexec_prefill_q3 = 0.73;
  r->coexec_slowdown = 1.15;
}

int mpa_predict_step(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host,
                     const mpa_rates* rates, mpa_step_time* out) {
  if (!out) return MPA_ERR_INVALID;
  mpa_rates def;
  mpa_default_rates(&def);
  const mpa_rates& r = rates ? *rates : def;
  int rc = check_model_inputs(shape, seq_lens_host, qsl_host, r);
  if (rc != MPA_OK) return rc;
  *out = model_step(shape, step_plan(shape, seq_lens_host, qsl_host), seq_lens_host, qsl_host, r);
  return MPA_OK;
}

int mpa_plan_coexec(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host,
                    const mpa_rates* rates, int32_t* mode, double* predicted_us) {
  if (!mode) return MPA_ERR_INVALID;
  mpa_rates def;
  mpa_default_rates(&def);
  const mpa_rates& r = rates ? *rates : def;
  int rc = check_model_inputs(shape, seq_lens_host, qsl_host, r);
  if (rc != MPA_OK) return rc;
  double dfrac[4] = {1.0, r.coexec_decode_q1, r.coexec_decode_q2, r.coexec_decode_q3};
  const double pfrac[4] = {1.0, r.coexec_prefill_q3, r.coexec_prefill_q2, r.coexec_prefill_q1};
  if (!(r.coexec_slowdown >= 1.0)) return MPA_ERR_INVALID;
  for (int k = 1; k <= 3; ++k)
    if (!(dfrac[k] > 0) || !(pfrac[k] > 0)) return MPA_ERR_INVALID;
  if (!(r.coexec_fixed_us >= 0.0)) return MPA_ERR_INVALID;
  const StepPlan& plan = step_plan(shape, seq_lens_host, qsl_host);
  const Batch& b = plan.batch;
  bool ranges = false;
  for (const auto& d : plan.decode) ranges |= d.range_blocks > 0;
  for (int k = 1; ranges && k <= 3; ++k) dfrac[k] *= kRangeShare[k];
  const double slowdown = ranges ? 1.0 + (r.coexec_slowdown - 1.0) * kRangeOverlap : r.coexec_slowdown;
  const mpa_step_time serial = model_step(shape, plan, seq_lens_host, qsl_host, r);
  double t[4];
  t[0] = serial.decode_us + serial.prefill_us;
  // The prefill half on the (4 - k) / 4 of the CUs: its workgroups' makespan
  // on that share of the slots relative to all of them (more rounds when the
  // batch has few workgroups), times the per-CU speed measured on that share
  // (pfrac against the share itself), and never faster than alone on the
  // whole device.
  const double all_slots = prefill_time(shape, seq_lens_host, qsl_host, plan.prefill, r.prefill_wg_us, r.prefill_tile_us,
                                        r.prefill_slots, 0.0, 0.0);
  for (int k = 1; k <= 3; ++k) {
    if (b.decode.empty() || b.prefill.empty()) {
      t[k] = INFINITY;  // nothing to overlap
      continue;
    }
    const double share = (4 - k) / 4.0;
    const int slots = std::max(1, (int)lround(r.prefill_slots * share));
    const double rounds = prefill_time(shape, seq_lens_host, qsl_host, plan.prefill, r.prefill_wg_us, r.prefill_tile_us,
                                       slots, 0.0, 0.0) /
                          all_slots;
    const double prefill_k = serial.prefill_us * std::max(1.0, rounds * share / pfrac[k]);
    t[k] = std::max(serial.decode_us / dfrac[k], prefill_k) * slowdown + r.coexec_fixed_us;
  }
  int best = 0;
  for (int k = 1; k <= 3; ++k)
    if (t[k] < t[best]) best = k;
  *mode = best;
  if (predicted_us)
    for (int k = 0; k < 4; ++k) predicted_us[k] = t[k];
  return MPA_OK;
}

int mpa_partition_streams(int32_t mode, void** decode_stream, void** prefill_stream) {
  if (mode < 1 || mode > 3 || !decode_stream || !prefill_stream) return MPA_ERR_INVALID;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MPA_ERR_HIP;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0 ||
      cus > 32 * kMaskWords)
    return MPA_ERR_HIP;
  static std::mutex lock;
  static hipStream_t made[64][3][2];
  std::lock_guard<std::mutex> guard(lock);
  hipStream_t* pair = made[dev][mode - 1];
  if (!pair[0]) {
    // CU i (the mask's numbering) goes to the decode half when (i / 8) % 4 <
    // mode: `mode` quarters of every XCD whether the numbering runs XCD by
    // XCD or interleaves them
    uint32_t dmask[kMaskWords] = {0}, pmask[kMaskWords] = {0};
    for (int i = 0; i < cus; ++i) ((i / 8) % 4 < mode ? dmask : pmask)[i / 32] |= 1u << (i % 32);
    const uint32_t words = (uint32_t)((cus + 31) / 32);
    hipStream_t d = nullptr, p = nullptr;
    if (hipExtStreamCreateWithCUMask(&d, words, dmask) != hipSuccess) return MPA_ERR_HIP;
    if (hipExtStreamCreateWithCUMask(&p, words, pmask) != hipSuccess) {
      (void)hipStreamDestroy(d);
      return MPA_ERR_HIP;
    }
    pair[0] = d;
    pair[1] = p;
  }
  *decode_stream = pair[0];
  *prefill_stream = pair[1];
  return MPA_OK;
}

size_t mpa_workspace_size(const mpa_shape* shape, const int32_t* seq_lens_host, const int32_t* qsl_host) {
  if (check_batch(shape, seq_lens_host, qsl_host, nullptr, false) != MPA_OK) return 0;
  const StepPlan& plan = step_plan(shape, seq_lens_host, qsl_host);
  return plan.decode_split || plan.prefill_split ? workspace_bytes(shape, plan.items) : 0;
}

int mpa_kv_append(const mpa_shape* shape, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                  const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
                  const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
                  const int32_t* block_tables_host, void* stream) {
  return run_append(shape, k_new, v_new, k_cache, v_cache, block_tables, seq_lens, query_start_loc, seq_lens_host,
                    query_start_loc_host, block_tables_host, nullptr, stream);
}

int mpa_kv_append_rope(const mpa_shape* shape, void* q, const void* k_new, const void* v_new, void* k_cache,
                       void* v_cache, const int32_t* block_tables, const int32_t* seq_lens,
                       const int32_t* query_start_loc, const int32_t* seq_lens_host,
                       const int32_t* query_start_loc_host, const int32_t* block_tables_host,
                       const float* rope_cos_sin, int32_t rope_dim, int32_t rope_max_pos, void* stream) {
  if (!shape) return MPA_ERR_INVALID;
  if (rope_dim <= 0 || rope_dim % 16 != 0 || rope_dim > shape->head_dim || rope_max_pos <= 0)
    return MPA_ERR_INVALID;
  if (shape->total_q_tokens > 0 && (!q || !rope_cos_sin)) return MPA_ERR_INVALID;
  if (seq_lens_host && shape->num_seqs > 0)
    for (int s = 0; s < shape->num_seqs; ++s)
      if (seq_lens_host[s] > rope_max_pos) return MPA_ERR_INVALID;  // a position past the table
  mpa::RopeArgs r;
  r.q = q;
  r.cos_sin = rope_cos_sin;
  r.hq = shape->num_q_heads;
  r.half = rope_dim / 2;
  return run_append(shape, k_new, v_new, k_cache, v_cache, block_tables, seq_lens, query_start_loc, seq_lens_host,
                    query_start_loc_host, block_tables_host, &r, stream);
}

}  // extern "C"

namespace {

enum Phase { kDecode = 1, kPrefill = 2 };

int run_attention(int phases, const mpa_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                  const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
                  const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
                  const int32_t* block_tables_host, void* out, float* lse, void* workspace,
                  size_t workspace_bytes_given, void* stream, const void* k_new = nullptr,
                  const void* v_new = nullptr, bool validate_only = false) {
  int rc = check_batch(shape, seq_lens_host, query_start_loc_host, block_tables_host, false);
  if (rc != MPA_OK) return rc;
  // The plan is the whole batch's, whichever phase runs: the two halves
  // together equal the mixed call exactly, and their partial results lie in
  // disjoint parts of the workspace, so they can run concurrently.
  const StepPlan& plan = step_plan(shape, seq_lens_host, query_start_loc_host);
  const bool decode = (phases & kDecode) && !plan.batch.decode.empty();
  const bool prefill = (phases & kPrefill) && !plan.batch.prefill.empty();
  if (!decode && !prefill) return MPA_OK;
  if (!q || !k_cache || !v_cache || !block_tables || !seq_lens || !query_start_loc || !out)
    return MPA_ERR_INVALID;
  const long items = plan.items;
  const bool any_split = (decode && plan.decode_split) || (prefill && plan.prefill_split);
  if (any_split) {
    const size_t need = workspace_bytes(shape, items);
    if (!workspace || workspace_bytes_given < need || ((uintptr_t)workspace & 15) != 0) return MPA_ERR_WORKSPACE;
  }
  mpa::AttnArgs a;
  a.q = q;
  a.k_cache = k_cache;
  a.v_cache = v_cache;
  a.block_tables = block_tables;
  a.seq_lens = seq_lens;
  a.qsl = query_start_loc;
  a.out = out;
  a.lse = lse;
  a.ws_o = any_split ? static_cast<float*>(workspace) : nullptr;
  a.ws_ml = any_split ? a.ws_o + (size_t)items * shape->num_q_heads * shape->head_dim : nullptr;
  a.hq = shape->num_q_heads;
  a.hkv = shape->num_kv_heads;
  a.mb = shape->max_blocks_per_seq;
  a.nb = shape->num_blocks;
  // fp8 caches: the key scale folds into the softmax scale, the value scale
  // into the output (and the split partials)
  const bool fp8 = shape->dtype == MPA_FP8;
  a.scale_log2 = shape->scale * 1.4426950408889634f * (fp8 ? shape->k_scale : 1.f);
  a.v_scale = fp8 ? shape->v_scale : 1.f;
  a.k_new = k_new;
  a.v_new = v_new;
  a.inv_k_scale = fp8 ? 1.f / shape->k_scale : 1.f;
  a.inv_v_scale = fp8 ? 1.f / shape->v_scale : 1.f;
  if (validate_only) return MPA_OK;
  hipStream_t st = (hipStream_t)stream;
  clear_stale_hip_error();

  // Decode rows, in launches of up to kMaxPlanSeqs sequences; split rows are
  // merged after their launch.
  long base = 0;
  for (const DecodeLaunch& d : plan.decode) {
    if (!decode) break;
    mpa::DecodePlan p;
    p.n_seqs = (int32_t)(d.c1 - d.c0);
    p.item_base = (int32_t)base;
    p.range_blocks = d.range_blocks;
    p.n_ranges = 0;
    int acc = 0, at = 0;
    for (int k = 0; k < p.n_seqs; ++k) {
      const int s = plan.batch.decode[d.c0 + k];
      const int L = seq_lens_host[s];
      p.seq[k] = s;
      p.item_start[k] = acc;
      if (d.range_blocks < 0) {
        p.part[k] = 0;
        acc += 1;
      } else if (d.range_blocks > 0) {
        p.part[k] = at;
        acc += (int)range_parts(at, row_blocks(L), d.range_blocks);
        at += row_blocks(L);
      } else {
        const RowSplit rs = row_split(L, plan.split);
        p.part[k] = rs.tokens;
        acc += rs.parts;
      }
    }
    p.part[p.n_seqs] = at;
    if (d.range_blocks > 0) p.n_ranges = (int32_t)(((long)at + d.range_blocks - 1) / d.range_blocks);
    p.item_start[p.n_seqs] = acc;
    base += acc;
    hipError_t e = mpa::launch_decode(a, p, acc, shape->dtype, shape->head_dim, st);
    if (e == hipSuccess && d.split) e = mpa::launch_merge(a, p, shape->dtype, shape->head_dim, st);
    if (e != hipSuccess) return MPA_ERR_HIP;
  }
  // Prefill segments, in launches of up to kMaxPrefillSeqs; KV-split ones are
  // merged after their launch.
  for (size_t c0 = 0; prefill && c0 < plan.prefill.size(); c0 += mpa::kMaxPrefillSeqs) {
    mpa::PrefillPlan p;
    p.n_seqs = (int32_t)(std::min(plan.prefill.size(), c0 + mpa::kMaxPrefillSeqs) - c0);
    p.rows = plan.prefill_rows[c0 / mpa::kMaxPrefillSeqs];
    // 16-row workgroups are quarters of a 64-row tile
    p.q_tile = std::max(p.rows, mpa::kPrefillRows) / (shape->num_q_heads / shape->num_kv_heads);
    const int qt = p.q_tile;
    int acc = 0, rows = 0;
    for (int k = 0; k < p.n_seqs; ++k) {
      const PrefillSegment& g = plan.prefill[c0 + k];
      p.seq[k] = g.seq;
      p.tok0[k] = g.tok0;
      p.ntok[k] = g.ntok;
      p.tile_start[k] = acc;
      p.nsplit[k] = g.nsplit;
      p.split_tiles[k] = g.tiles;
      p.item_base[k] = (int32_t)g.item_base;
      p.row_start[k] = rows;
      acc += (g.ntok + qt - 1) / qt * g.nsplit;
      if (g.nsplit > 1) rows += g.ntok;
    }
    p.tile_start[p.n_seqs] = acc;
    p.row_start[p.n_seqs] = rows;
    hipError_t e = mpa::launch_prefill(a, p, acc, shape->dtype, shape->head_dim, st);
    if (e != hipSuccess) return MPA_ERR_HIP;
    if (rows > 0) {
      e = mpa::launch_prefill_merge(a, p, shape->dtype, shape->head_dim, st);
      if (e != hipSuccess) return MPA_ERR_HIP;
    }
  }
  return MPA_OK;
}

// The append and the attention of the rows in `phases`, in one call: the
// attention's checks (the workspace included) and the append's run first,
// so an error means nothing was launched; then the multi-token rows' block
// append (prefill phase), and the attention, whose decode kernel writes the
// decode rows' new tokens itself.
int run_fused(int phases, const mpa_shape* shape, const void* q, const void* k_new, const void* v_new,
              void* k_cache, void* v_cache, const int32_t* block_tables, const int32_t* seq_lens,
              const int32_t* query_start_loc, const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
              const int32_t* block_tables_host, void* out, float* lse, void* workspace, size_t workspace_bytes_given,
              void* stream) {
  int rc = run_attention(phases, shape, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc, seq_lens_host,
                         query_start_loc_host, block_tables_host, out, lse, workspace, workspace_bytes_given, stream,
                         nullptr, nullptr, true);
  if (rc != MPA_OK) return rc;
  if (shape->total_q_tokens > 0 && (!k_new || !v_new)) return MPA_ERR_INVALID;
  if (phases & kPrefill) {
    rc = run_append(shape, k_new, v_new, k_cache, v_cache, block_tables, seq_lens, query_start_loc, seq_lens_host,
                    query_start_loc_host, block_tables_host, nullptr, stream, true);
    if (rc != MPA_OK) return rc;
  } else if (debug_checks()) {
    rc = check_append_slots(shape, seq_lens_host, query_start_loc_host, block_tables_host);
    if (rc != MPA_OK) return rc;
  }
  return run_attention(phases, shape, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc, seq_lens_host,
                       query_start_loc_host, block_tables_host, out, lse, workspace, workspace_bytes_given, stream,
                       k_new, v_new);
}

}  // namespace

extern "C" {

int mpa_mixed_paged_attention(const mpa_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                              const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
                              const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
                              const int32_t* block_tables_host, void* out, float* lse, void* workspace,
                              size_t workspace_bytes_given, void* stream) {
  return run_attention(kDecode | kPrefill, shape, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc,
                       seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                       workspace_bytes_given, stream);
}

int mpa_append_attention(const mpa_shape* shape, const void* q, const void* k_new, const void* v_new,
                         void* k_cache, void* v_cache, const int32_t* block_tables, const int32_t* seq_lens,
                         const int32_t* query_start_loc, const int32_t* seq_lens_host,
                         const int32_t* query_start_loc_host, const int32_t* block_tables_host, void* out,
                         float* lse, void* workspace, size_t workspace_bytes_given, void* stream) {
  return run_fused(kDecode | kPrefill, shape, q, k_new, v_new, k_cache, v_cache, block_tables, seq_lens,
                   query_start_loc, seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                   workspace_bytes_given, stream);
}

int mpa_append_decode_attention(const mpa_shape* shape, const void* q, const void* k_new, const void* v_new,
                                void* k_cache, void* v_cache, const int32_t* block_tables, const int32_t* seq_lens,
                                const int32_t* query_start_loc, const int32_t* seq_lens_host,
                                const int32_t* query_start_loc_host, const int32_t* block_tables_host, void* out,
                                float* lse, void* workspace, size_t workspace_bytes_given, void* stream) {
  return run_fused(kDecode, shape, q, k_new, v_new, k_cache, v_cache, block_tables, seq_lens, query_start_loc,
                   seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                   workspace_bytes_given, stream);
}

int mpa_append_prefill_attention(const mpa_shape* shape, const void* q, const void* k_new, const void* v_new,
                                 void* k_cache, void* v_cache, const int32_t* block_tables, const int32_t* seq_lens,
                                 const int32_t* query_start_loc, const int32_t* seq_lens_host,
                                 const int32_t* query_start_loc_host, const int32_t* block_tables_host, void* out,
                                 float* lse, void* workspace, size_t workspace_bytes_given, void* stream) {
  return run_fused(kPrefill, shape, q, k_new, v_new, k_cache, v_cache, block_tables, seq_lens, query_start_loc,
                   seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                   workspace_bytes_given, stream);
}

int mpa_decode_attention(const mpa_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
                         const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
                         const int32_t* block_tables_host, void* out, float* lse, void* workspace,
                         size_t workspace_bytes_given, void* stream) {
  return run_attention(kDecode, shape, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc,
                       seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                       workspace_bytes_given, stream);
}

int mpa_prefill_attention(const mpa_shape* shape, const void* q, const void* k_cache, const void* v_cache,
                          const int32_t* block_tables, const int32_t* seq_lens, const int32_t* query_start_loc,
                          const int32_t* seq_lens_host, const int32_t* query_start_loc_host,
                          const int32_t* block_tables_host, void* out, float* lse, void* workspace,
                          size_t workspace_bytes_given, void* stream) {
  return run_attention(kPrefill, shape, q, k_cache, v_cache, block_tables, seq_lens, query_start_loc,
                       seq_lens_host, query_start_loc_host, block_tables_host, out, lse, workspace,
                       workspace_bytes_given, stream);
}

}  // extern "C"
