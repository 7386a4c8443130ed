// The library's plans and what else of it runs on the host, callable from Python (compiled and loaded
// by test_plans.py).
#include "tb_kernels.h"

extern "C" {

// tables an order's n-grams are dealt to, slots of one, partitions; false: no such plan
bool runs_plan(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits, bool rouge,
               bool group_distinct, int64_t* out) {
  tb::RunsPlan p;
  if (!tb::plan_runs(B, cand_stride, ref_stride, R, N, bits, rouge, group_distinct, &p)) return false;
  out[0] = int64_t(p.parts) << p.sub_bits;
  out[1] = int64_t(1) << (p.log2_slots - p.sub_bits);
  out[2] = p.parts;
  out[3] = p.chunks;
  out[4] = int64_t(p.lds_bytes);
  return true;
}

// of the same plan: positions per thread of the sorting kernel, counter words, whether counters have 32 bits, bits of
// an n-gram that choose a part of the table
bool runs_shape(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits, bool group_distinct,
                int32_t* out) {
  tb::RunsPlan p;
  if (!tb::plan_runs(B, cand_stride, ref_stride, R, N, bits, false, group_distinct, &p)) return false;
  out[0] = p.items;
  out[1] = p.words;
  out[2] = p.wide_fields;
  out[3] = p.sub_bits;
  return true;
}

// kinds; partitions, slots and candidate's positions of each; ids; slots of their table; members in a window (of any kind);
// partitions of all kinds; chunks; LDS bytes; first kind; false: no such plan
bool deal_plan(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int32_t vocab, bool rouge,
               bool group_distinct, int64_t* out) {
  tb::DealPlan p;
  if (!tb::plan_deal(B, cand_stride, ref_stride, R, N, vocab, rouge, group_distinct, &p)) return false;
  out[0] = p.kinds;
  out[13] = p.first_kind;
  for (int kind = 0; kind < 3; ++kind) out[1 + kind] = p.parts[kind];
  out[4] = int64_t(1) << p.log2_first;
  out[5] = int64_t(1) << p.log2_pair;
  out[6] = int64_t(1) << p.log2_item;
  out[7] = p.capacity;
  out[8] = int64_t(1) << p.id_bits;
  out[9] = p.window[0] | p.window[1] | p.window[2];
  out[10] = p.all_parts;
  out[11] = p.chunks;
  out[12] = int64_t(p.lds_bytes);
  return true;
}

// log2 of the slots; bits of an id and of the widest key; pass_ends; LDS bytes; wavefronts; blocks of one
// of them; whether ids are kept between passes; whether a workgroup has its unit to itself; false: no such plan
bool fused_plan(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits, bool rouge,
                int64_t* out) {
  tb::FusedPlan p;
  if (!tb::plan_fused(B, cand_stride, ref_stride, R, N, bits, rouge, &p)) return false;
  out[0] = p.log2_slots;
  out[1] = p.id_bits;
  out[2] = p.first_key_bits > p.later_key_bits ? p.first_key_bits : p.later_key_bits;
  out[3] = p.pass_ends;
  out[4] = int64_t(p.lds_bytes);
  out[5] = p.threads / 64;
  out[6] = p.blocks;
  out[7] = p.keep;
  out[8] = tb::fused_alone(B, p);
  return true;
}

// which kernels serve a whole call: 0 the fused one, 1 dealt positions, 2 sorted runs, 3 stages
int route(int32_t B, int32_t R, int64_t cand_stride, int64_t ref_stride, int N, int32_t vocab, bool rouge,
          bool group_distinct) {
  tb_config_t cfg{};
  cfg.max_n = N;
  cfg.vocab_size = vocab;
  return int(tb::route_of_call(B, R, cand_stride, ref_stride, &cfg, rouge, group_distinct));
}

bool fused_path(int64_t cand_stride, int64_t ref_stride, int R, int bits) {
  return tb::fused_path_takes(cand_stride, ref_stride, R, bits);
}

uint32_t first_free_slot(uint32_t x, uint32_t y, uint32_t z) { return tb::first_free_slot(x, y, z); }

}  // extern "C"
