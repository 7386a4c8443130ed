// Host-side launch interface between the C-ABI dispatcher and the kernel translation units.
#pragma once

#include "tb_common.h"

namespace tb {

// Raises a kernel's dynamic-LDS limit to `bytes` (hipFuncSetAttribute) unless an earlier launch
// on the same device already raised it at least that far: the attribute call costs a few
// microseconds, which matters for calls that take ten.  `kernel` is the host-side kernel symbol.
hipError_t grant_dynamic_lds(const void* kernel, size_t bytes);

// Resolved pointers into the caller's workspace for the GLOBAL path.
struct GlobalWs {
  void* keys[8];      // packed keys per order, B * group_cap entries of 8 or 16 bytes
  uint32_t* inv[8];   // offset dictionary ids per order, B * group_cap entries
  int32_t wide[8];    // 1 when the order uses 16-byte keys
  void* tables;       // hash tables / counters in HBM (groups too large for LDS), or the
                      // per-partition dictionary sizes of the partitioned kernels, else null
  int32_t* overflow;  // [B], partitioned kernels only (else null): non-zero where a partition of
                      // the group received more distinct n-grams than it can number; the score
                      // kernels turn such a group's score into NaN
  int32_t* arrivals;  // [B], hierarchical-key kernels only (else null; the same words as
                      // `overflow`): how many of a group's count workgroups have finished; the
                      // dictionary kernel zeroes it, and in a whole call the last count workgroup
                      // to arrive scores the sentence
};

// Integer statistics (either the caller's arrays or workspace scratch; never null).
struct StatPtrs {
  int32_t* clipped;   // [B, N]
  int32_t* total;     // [B, N]
  int32_t* closest;   // [B]
  int32_t* distinct;  // [B, N]
  int64_t* corpus;    // [2N+2]
};

// Launch shape shared by the dictionary and count/clip kernels: every thread keeps up to
// `items` of its group's n-grams in registers (threads * items >= group_cap).
struct DictPlan {
  int threads;          // workgroup size (256, 512 or 1024)
  int items;            // register-resident n-grams per thread: 2, 4, 6, 8 or 12
  int narrow_orders[8]; // orders with 8-byte keys, and how many
  int n_narrow;
  int slot32_mask;      // bit n: order n's keys fit 32 bits (4-byte table entries, 2x the slots)
  int narrow_slots;     // hash-table slots (power of two, >= 4/3 group_cap), 8-byte entries
  size_t narrow_lds;
  int wide_orders[8];   // orders with 16-byte keys
  int n_wide;
  int wide_slots;       // 4-byte tag:position entries
  int wide_compact;     // 1: keys within 64 + 18 bits, only their low halves are staged in LDS
  size_t wide_lds, wide_table_off;
};
struct CountPlan {
  int threads, items;
  int fields;   // 1: one 16-bit LDS field per sequence (count_fields_kernel); 0: pair phases
  int words;    // 32-bit words per dictionary entry in the fields kernel
  size_t lds_bytes;
};
struct FusedPlan {
  int threads, blocks;     // workgroup size; blocks of 64 positions per wavefront
  int keep;                // 1: a pass starts above order 2
  uint32_t pass_ends;      // see FusedArgs
  int log2_slots, id_bits;
  int first_payload, first_key_bits, later_payload, later_key_bits;
  int array_bytes;
  int table_and_counters;  // 16-byte units
  uint32_t off_sym, off_sums;
  size_t lds_bytes;
};

// Groups within one LDS table whose (prefix id, last token) keys fit 31 bits: one workgroup per
// group builds the dictionaries of all orders on hierarchical 32-bit keys, and one workgroup per
// group (or per share of its orders) counts and clips all of them at once.
struct HierPlan {
  int threads, items;        // workgroup size; token positions / slots per thread
  int table_slots;           // power of two > group_cap, 4-byte entries
  size_t dict_lds;
  int words;                 // count/clip: 32-bit words of 16-bit fields per entry
  int count_threads, count_rows;  // count/clip: workgroup size; 16-byte id requests per thread
  int count_pairs_fit;       // count/clip: the counters of two orders fit one workgroup's LDS
};
bool plan_hier(int64_t group_cap, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits,
               HierPlan* plan);
// cand_distinct [B, N]: written by the dictionary pass, read by the count/clip pass
hipError_t launch_hier_dictionary(const Problem& pb, const GlobalWs& ws, const HierPlan& plan,
                                  const StatPtrs& st, int32_t* cand_distinct, hipStream_t s);
// rouge_overlap != null: ROUGE-N instead -- only order N is counted, and overlap[B, R] receives
// per reference the sum over n-grams of min(candidate count, the reference's count)
// tail != null (BLEU only): the last workgroup of a group to finish also computes what the
// sentence score kernel computes (closest reference length, Section 3.4's score into tail->out),
// which then is not to be launched; needs ws.arrivals zeroed by the dictionary pass
struct ScoreTail {
  ScoreParams sp;
  void* out;  // [B] fp32 or bfloat16 (sp.out_bf16)
};
hipError_t launch_hier_count_clip(const Problem& pb, const GlobalWs& ws, const HierPlan& plan,
                                  const StatPtrs& st, const int32_t* cand_distinct,
                                  hipStream_t s, int32_t* rouge_overlap = nullptr,
                                  const ScoreTail* tail = nullptr);

// Groups beyond the LDS plans: table and counters live in the workspace.
struct BigPlan {
  int64_t slots;          // hash-table slots per (group, order): power of two >= 2 * group_cap
  int64_t table_entries;  // slots + padding, 8 bytes each
};
// Groups of up to 2 097 152 n-gram slots beyond the LDS plans: P workgroups per (group, order),
// each with the dictionary entries / counters of one hash partition in LDS.
struct PartPlan {
  int log2_parts;     // P = 1 << log2_parts workgroups per (group, order), 2 .. 512
  int id_cap;         // ids a partition may hand out
  int words;          // count/clip: 32-bit counter words per id
  int refs_per_pass;  // count/clip: 0 = every sequence has its field; else references per pass
  int fields_per_word;  // 2: 16-bit counters, 1: 32-bit (a stride above 65 535)
  int64_t id_stride;  // id range per group: max(group_cap, P * id_cap)
  size_t dict_lds, count_lds;
  int count_in_dictionary;  // the counter fields of a partition fit the dictionary table's LDS
};
bool plan_part(int64_t group_cap, int64_t cand_stride, int64_t ref_stride, int R, int N,
               const int32_t* key_bytes, PartPlan* plan);
// bytes the partitioned kernels need at GlobalWs::tables
size_t part_workspace_bytes(int64_t B, int N, int64_t group_cap, const PartPlan& plan);
// whole_call: the count/clip pass follows at once and nobody else reads the id array, so ids are
// stored only where a later order's keys are derived from them and, if
// plan.count_in_dictionary, the dictionary kernel also does the count/clip pass's work, which is
// then not to be launched.  from_tokens: pb.cand / pb.refs are set and the keys are built from
// them; otherwise they are read from ws.keys as the pack kernel left them
hipError_t launch_part_dictionary(const Problem& pb, const GlobalWs& ws, const PartPlan& plan,
                                  const StatPtrs& st, bool whole_call, bool from_tokens,
                                  hipStream_t s);
// rouge_overlap != null: ROUGE-N instead, as for launch_hier_count_clip
hipError_t launch_part_count_clip(const Problem& pb, const GlobalWs& ws, const PartPlan& plan,
                                  const StatPtrs& st, hipStream_t s,
                                  int32_t* rouge_overlap = nullptr);

// Whole calls on the same groups: equal n-grams of a chunk merged before they are dealt out to
// partitions, tables with the candidate's n-grams only (tb_runs.hip).  group_distinct: the caller
// wants the dictionary sizes (the references' n-grams are then entered, too).
struct RunsPlan {
  int items;                    // positions per thread of the sorting kernel: 1, 2 or 4
  int num_orders;               // 1..N, or order N alone (ROUGE-N)
  int orders_each;              // orders a sorting workgroup takes one after the other
  int parts, log2_slots;
  int beyond, log2_parts, sub_bits;  // n-grams of more than 64 bits
  int cand_chunks, ref_chunks, chunks;
  int words, wide_fields;
  uint32_t off_counters, off_prefix, off_runs;
  size_t lds_bytes;
};
bool plan_runs(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits,
               bool rouge, bool group_distinct, RunsPlan* plan);
// its share of the partitioned kernels' workspace: N * B * group_cap keys of 8 bytes,
// multiplicities of (at least) 2 and places of 4
struct RunsBuffers {
  uint64_t* keys;
  uint16_t* times;
  uint32_t* places;
  int32_t* overflow;  // [B]
};
RunsBuffers runs_buffers(const Problem& pb, const GlobalWs& ws, const PartPlan& plan);
// rouge_overlap != null: ROUGE-N, as for launch_hier_count_clip
hipError_t launch_runs(const Problem& pb, const RunsPlan& plan, const RunsBuffers& buffers,
                       const StatPtrs& st, bool group_distinct, int32_t* rouge_overlap,
                       hipStream_t s);

// Whole calls on the same groups, BLEU of up to four orders and ROUGE-1 and -2, every position dealt out once
// (tb_deal.hip); in the same share of the workspace.
struct DealPlan {
  int items;                                // positions per thread of the dealing kernel: 1 or 2
  int first_kind, kinds, all_parts, parts[3], parts_before[3];
  int all;                                  // the references' n-grams are entered, too (group_distinct)
  int cand_chunks, ref_chunks, chunks;
  int words, halves, capacity, window[3], id_bits, log2_first, log2_pair, log2_item;
  uint32_t off_tokens, off_lead, off_sums, off_places, off_scratch;
  size_t lds_bytes;
};
bool plan_deal(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int32_t vocab, bool rouge,
               bool group_distinct, DealPlan* plan);
hipError_t launch_deal(const Problem& pb, const DealPlan& plan, const RunsBuffers& buffers,
                       const StatPtrs& st, const ScoreParams& sp, void* out_bleu_or_null,
                       int32_t* rouge_overlap, hipStream_t s);

bool plan_big(int64_t group_cap, int N, BigPlan* plan);
hipError_t launch_big_dictionary(const Problem& pb, const GlobalWs& ws, const BigPlan& plan,
                                 const StatPtrs& st, hipStream_t s);
// rouge_overlap != null: ROUGE-N instead, as for launch_hier_count_clip
hipError_t launch_big_count_clip(const Problem& pb, const GlobalWs& ws, const BigPlan& plan,
                                 const StatPtrs& st, hipStream_t s,
                                 int32_t* rouge_overlap = nullptr);

bool plan_dictionary(int64_t group_cap, const int32_t* key_bytes, int N, int bits,
                     DictPlan* plan);
bool plan_count(int64_t group_cap, int64_t cand_stride, int64_t ref_stride, int R,
                CountPlan* plan);
// Whether TB_PATH_AUTO resolves a shape to the FUSED path.  (The kernel itself takes larger groups:
// plan_fused.  The line stays where callers know it, because what a path reports as group_distinct
// depends on it.)
bool fused_path_takes(int64_t cand_stride, int64_t ref_stride, int R, int bits);
bool plan_fused(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits,
                bool rouge, FusedPlan* plan);
// Whether the plan's workgroups have a compute unit each, and with it the kernel that has more registers.
bool fused_alone(int64_t B, const FusedPlan& plan);

// The kernels that serve a whole call: the fused one, those for dealt positions or for sorted runs, or the GLOBAL path's
// stages.
enum class Route { kFused, kDealt, kRuns, kStaged };
Route route_of_call(int32_t B, int32_t R, int64_t cand_stride, int64_t ref_stride, const tb_config_t* cfg, bool rouge,
                    bool group_distinct);

hipError_t launch_pack(const Problem& pb, const GlobalWs& ws, hipStream_t s);
hipError_t launch_dictionary(const Problem& pb, const GlobalWs& ws, const DictPlan& plan,
                             int32_t* distinct, hipStream_t s);
hipError_t launch_count_clip(const Problem& pb, const GlobalWs& ws, const CountPlan& plan,
                             const StatPtrs& st, hipStream_t s);
// sentence_scores: out_bleu[B] per-sentence scores; corpus_sums: fill st.corpus;
// corpus_score: additionally write the corpus score to out_bleu[0] (not with sentence_scores).
// overflow: GlobalWs::overflow or null.  known_closest: st.closest is filled already and no group
// can have overflowed.  own_counts: this call's kernels have filled st.clipped, so that no count is
// above its candidate's length
hipError_t launch_finalize(const Problem& pb, const StatPtrs& st, const ScoreParams& sp,
                           bool sentence_scores, bool corpus_sums, bool corpus_score,
                           void* out_bleu, hipStream_t s, const int32_t* overflow = nullptr,
                           bool known_closest = false, bool own_counts = true);
// ROUGE-N scores from overlap counts (GLOBAL path): precision, recall, F of the best reference.
struct RougeOut;
hipError_t launch_rouge_finalize(const Problem& pb, const ScoreParams& sp, const int32_t* overlap,
                                 const RougeOut& out, hipStream_t s);
// ROUGE-N outputs of the fused kernel (order n = pb.N): see tensorrouge_n.
struct RougeOut {
  void* prf;         // [B, 3] fp32 or bfloat16 (ScoreParams::out_bf16)
  int32_t* overlap;  // [B, R] or null
  int32_t* best;     // [B] or null
  float beta2;
};
// rouge == null: BLEU (statistics, st.distinct among them if want_distinct, and, if
// out_bleu_or_null, per-sentence scores).
hipError_t launch_fused(const Problem& pb, const FusedPlan& plan, const StatPtrs& st,
                        const ScoreParams& sp, void* out_bleu_or_null, bool want_distinct,
                        hipStream_t s, const RougeOut* rouge = nullptr);

}  // namespace tb
