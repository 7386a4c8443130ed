// Whole calls on groups beyond one LDS table (12 289 .. 2 097 152 n-gram slots) that the kernels which deal every
// position out once (tb_deal.hip) do not take or are slower on (more than four orders or 20-bit tokens, few positions,
// many references: takes_deal in tb_api.hip), in two kernels:
//
//   runs_sort_kernel   one workgroup per (group, order, chunk of 1024..4096 positions of one
//                      sequence): builds the chunk's n-grams from the token row (Section 3.1),
//                      merges equal ones, sorts what is left by hash partition and writes it as
//                      one run per partition, with the runs' places
//   runs_count_kernel  one workgroup per (group, order, partition): gathers the partition's runs,
//                      enters the candidate's n-grams into an LDS table, looks the references' up,
//                      adds the multiplicities into one counter per sequence and clips
//                      (Sections 3.2-3.3)
//
// What bounds it, and why this split:
//   * Tokens are Zipf-distributed: one token makes up a tenth of a text, so one partition of order 1
//     received twenty times its share, and its workgroup alone took 70 of 111 us on a text of
//     262 144 tokens.  Merged per chunk, a frequent n-gram arrives once per chunk.  The merging is not
//     exact, and need not be: of the positions whose keys hash to the same word one is kept there, and
//     those equal to it add themselves to its count; any other is passed on as it is.  (One LDS store,
//     two reads and, for duplicates, one addition a position; no probing.)
//   * A chunk writes into the place of its own positions, so no workgroup needs to know how much the
//     others have: no histogram kernel, no cursors.  A chunk lies in one sequence, so no slot numbers
//     are stored.  Per n-gram 8 bytes of key and 2 of multiplicity pass through memory.
//   * Only the candidate's n-grams occupy the table unless the size of the group's dictionary is
//     asked for; 4096 entries with their counters are 48 KB (one or, with 64 KB, up to three
//     references), so two workgroups of 1024 threads share a compute unit.
//   * n-grams of more than 64 bits: the partition number is (hash of the low 64 bits) xor (the bits
//     above them), so partition and low bits identify the n-gram and the key stays 8 bytes.  Where the
//     plan has fewer partitions than that takes, up to four more bits choose a part of the table.  Such a
//     part is a table of its own, of 64 slots at the least: the plan has to leave it room for more than
//     its share (has_room).
//
// Measured (us a call, before on the partitioned kernels -> here, whichever kernel takes them now): one text of 262 144 tokens with its
// reference 110.7 -> 33 (sorting 12.5, counting 17.6, score 3); 16 groups of two times 8192 36 -> 22; 100 of
// two times 20 000 276 -> 137 (sorting 55, counting 80); 300 of nine times 4096 1111 -> 354; 20 of nine
// times 4096 with 18-bit tokens 147 -> 48; ROUGE-2 of one text of 100 000 80 -> 20.  The number of
// partitions is as many as the tables need, filled up to whole rounds of 512 workgroups (a power of two
// only with longer n-grams): counting 110 us before, with 16 tables a third full, for the 100 groups.
//
// Keys are exact.  A table that is full (which takes tokens chosen to collide: see has_room) is reported
// through TB_DEV_TABLE_OVERFLOW and scored NaN.
#include <cmath>

#include "tb_kernels.h"

namespace tb {

namespace {

constexpr int kRunThreads = 1024;
constexpr int kMaxRunParts = 512;
constexpr int kMaxChunks = kRunThreads;  // per group: one thread each reads a run's place
constexpr int kSubBits = 4;              // at most; above the 12 bits of a multiplicity - 1
constexpr int kSubs = 1 << kSubBits;
constexpr unsigned long long kFree = ~0ull;

struct RunsArgs {
  Problem pb;
  StatPtrs st;
  uint64_t* run_key;        // [num_orders][B * group_cap]
  uint16_t* run_times;      // the same: multiplicity - 1 | part of the table << 12
  uint32_t* run_at;         // [num_orders][B][chunks][P]: first of the run within its chunk | size << 16
  int32_t* overflow;        // [B]
  int32_t* rouge_overlap;   // [B, R] or null
  int first_order, num_orders;
  int orders_each;          // orders a sorting workgroup handles one after the other
  int parts, log2_slots;
  int log2_parts, sub_bits; // with n-grams of more than 64 bits, where parts = 1 << log2_parts
  int beyond;               // 1: there are some
  int cand_chunks, ref_chunks, chunks;  // of the candidate, of one reference, of a group
  int words, wide_fields;   // counter words per entry; 1: 32-bit counters, 0: two of 16 bits a word
  int enter_refs;           // 1: the references' n-grams are entered, too, and distinct ones counted
  uint32_t off_counters, off_prefix, off_runs;
};

// (Both halves are multiplied: an exclusive or of shifted halves gives the same hash to all n-grams
// whose frequent tokens, small numbers, cancel; the call on one text of 262 144 tokens then took 52.6 us
// instead of 38.9.)
__device__ __forceinline__ uint32_t run_hash(uint64_t key) {
  const uint32_t h = uint32_t(key) * 0x9E3779B1u + uint32_t(key >> 32) * 0xC2B2AE3Du;
  return h ^ (h >> 15);
}
// (independent of the top bits of h, which pick the table slot, and of the probe step)
__device__ __forceinline__ uint32_t second_hash(uint32_t h) { return h * 0x85EBCA6Bu + 0x27D4EB2Fu; }

// Chunk c of a group: its sequence and first position.
struct Chunk {
  int seq, first;
};
template <int CHUNK>
__device__ __forceinline__ Chunk chunk_of(const RunsArgs& a, int c) {
  Chunk k;
  const int q = max(c - a.cand_chunks, 0);
  const int j = a.pb.R > 1 ? q / a.ref_chunks : 0;
  k.seq = c < a.cand_chunks ? 0 : 1 + j;
  k.first = (c < a.cand_chunks ? c : q - j * a.ref_chunks) * CHUNK;
  return k;
}
// Where a chunk's n-grams lie among the group's slots.
__device__ __forceinline__ int chunk_base(const RunsArgs& a, const Chunk& k) {
  return (k.seq == 0 ? 0 : int(a.pb.cand_stride) + (k.seq - 1) * int(a.pb.ref_stride)) + k.first;
}

// ITEMS: positions per thread.  68 KB of LDS with four: two workgroups on a compute unit.
//
// Bound by latency: 1.4 to 2.6 of a workgroup's 5.7 us pass until the tokens are there, and six barriers
// follow (time stamps of each step, one text of 262 144 tokens).  Where there are more workgroups than
// the chip holds, each therefore takes several orders of its chunk (100 groups of two times 20 000
// tokens: 63 us, then 55).
template <int ITEMS>
__global__ __launch_bounds__(kRunThreads, 8) void runs_sort_kernel(RunsArgs a) {
  constexpr int kChunk = ITEMS * kRunThreads;
  constexpr int kLog2Chunk = ITEMS == 4 ? 12 : ITEMS == 2 ? 11 : 10;
  static_assert((1 << kLog2Chunk) == kChunk, "chunk");
  __shared__ uint64_t key[kChunk];
  __shared__ uint32_t token[kChunk + 8];
  __shared__ uint32_t kept[kChunk];       // by hash: position kept there | its duplicates << 12; in
                                          // the end: what run_times receives
  __shared__ int in_part[kMaxRunParts], first_of[kMaxRunParts];
  __shared__ int scan_scratch[17];
  const Problem& pb = a.pb;
  const int tid = threadIdx.x, parts = a.parts;
  const int c = blockIdx.x, g = blockIdx.z;
  const int idx_begin = int(blockIdx.y) * a.orders_each;
  const int idx_end = min(idx_begin + a.orders_each, a.num_orders);
  const Chunk me = chunk_of<kChunk>(a, c);

  const RefRows rr = ref_rows(pb, g);
  int len = 0;
  int64_t row;
  const void* base;
  if (me.seq == 0) {  // uniform
    len = clamped_len(uniform_load(pb.cand_len, g), pb.cand_stride, nullptr);
    base = pb.cand;
    row = int64_t(g) * pb.cand_stride;
  } else {
    const int64_t r = rr.row0 + me.seq - 1;
    if (me.seq <= rr.used) len = clamped_len(uniform_load(pb.ref_len, r), pb.ref_stride, nullptr);
    base = pb.refs;
    row = r * pb.ref_stride;
  }
  row += me.first;
  // (every token inside the length is looked at, also where no n-gram starts)
  const int staged = min(max(len - me.first, 0), kChunk + a.first_order + idx_end - 2);

  bool bad = false;
  auto put = [&](int i, int32_t t) {
    const bool outside = uint32_t(t) >= uint32_t(pb.vocab);  // reported and taken as 0
    bad |= outside;
    token[i] = outside ? 0u : uint32_t(t);
  };
  if (staged > 0) {  // uniform
    int32_t t[ITEMS];
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
      t[u] = load_token(base, row + min(u * kRunThreads + tid, staged - 1), pb.tok64);
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
      if (u * kRunThreads + tid < staged) put(u * kRunThreads + tid, t[u]);
    if (kChunk + tid < staged) put(kChunk + tid, load_token(base, row + kChunk + tid, pb.tok64));
  }
  if (tid < kMaxRunParts) in_part[tid] = 0;
  if (c == 0) {  // what the partitions' workgroups add to
    if (tid >= idx_begin && tid < idx_end) {
      const int64_t stat = int64_t(g) * pb.N + a.first_order + tid - 1;
      a.st.clipped[stat] = 0;
      a.st.distinct[stat] = 0;
    }
    if (idx_begin == 0 && tid == 0) a.overflow[g] = 0;
    if (a.rouge_overlap && idx_begin == 0 && tid < pb.R)
      a.rouge_overlap[int64_t(g) * pb.R + tid] = 0;
  }
  if (bad && pb.status) atomicOr(pb.status, TB_DEV_TOKEN_RANGE);
  __syncthreads();

  const int bits = pb.bits;
  uint64_t lo[ITEMS];
  uint32_t hi[ITEMS];  // the bits beyond 64
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) lo[u] = 0, hi[u] = 0;
  int built = 0;  // tokens in lo and hi
#pragma unroll 1
  for (int idx = idx_begin; idx < idx_end; ++idx) {
    const int n = a.first_order + idx;
    const int count = min(max(len - n + 1 - me.first, 0), kChunk);
    const bool wide = n * bits > 64;
#pragma unroll 1
    for (; built < n; ++built) {
#pragma unroll
      for (int u = 0; u < ITEMS; ++u) {
        if (wide) hi[u] = (hi[u] << bits) | uint32_t(lo[u] >> (64 - bits));
        lo[u] = (lo[u] << bits) | token[u * kRunThreads + tid + built];  // (beyond `count`: not used)
      }
    }
    uint32_t h[ITEMS], where[ITEMS];  // where: partition (| part of the table << log2_parts)
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int k = u * kRunThreads + tid;
      h[u] = run_hash(lo[u]);
      const uint32_t h2 = second_hash(h[u]);
      where[u] = a.beyond ? (h2 >> (32 - a.log2_parts - a.sub_bits)) ^ hi[u]
                          : __umulhi(h2, uint32_t(parts));
      if (k < count) {
        key[k] = lo[u];
        kept[h[u] >> (32 - kLog2Chunk)] = uint32_t(k);
      }
    }
    auto part_at = [&](int u) { return a.beyond ? where[u] & uint32_t(parts - 1) : where[u]; };
    __syncthreads();
    int rank[ITEMS];  // -1: merged into another position
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int k = u * kRunThreads + tid;
      rank[u] = -1;
      if (k < count) {
        uint32_t* const word = &kept[h[u] >> (32 - kLog2Chunk)];
        const int w = int(*word & 0xFFFu);
        // (the bits beyond 64 belong to the first token)
        if (w != k && key[w] == lo[u] && (!wide || token[w] == token[k]))
          atomicAdd(word, 0x1000u);
        else
          rank[u] = atomicAdd(&in_part[part_at(u)], 1);
      }
    }
    __syncthreads();
    uint32_t times[ITEMS];
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int k = u * kRunThreads + tid;
      times[u] = 0u;
      if (rank[u] >= 0) {
        const uint32_t word = kept[h[u] >> (32 - kLog2Chunk)];
        if (int(word & 0xFFFu) == k) times[u] = word >> 12;
        if (a.beyond) times[u] |= (where[u] >> a.log2_parts) << 12;
      }
    }
    const int mine = tid < parts ? in_part[tid] : 0;
    int total;
    const int first = block_exclusive_scan(mine, scan_scratch, &total);
    if (tid < parts) {
      first_of[tid] = first;
      in_part[tid] = 0;
      a.run_at[((int64_t(idx) * pb.B + g) * a.chunks + c) * parts + tid] =
          uint32_t(first) | (uint32_t(mine) << 16);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      if (rank[u] >= 0) {
        const int at = first_of[part_at(u)] + rank[u];
        key[at] = lo[u];
        kept[at] = times[u];
      }
    }
    __syncthreads();
    const int64_t out = (int64_t(idx) * pb.B + g) * pb.group_cap + chunk_base(a, me);
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int i = u * kRunThreads + tid;
      if (i < total) {
        a.run_key[out + i] = key[i];
        a.run_times[out + i] = uint16_t(kept[i]);
      }
    }
    if (idx + 1 < idx_end) __syncthreads();  // key and kept are written again
  }
}

// Bound by latency, too: 4.3 of a workgroup's 11.7 us until its runs' places and first members are there,
// 3.8 (at most 7.9) for the candidate's entries, 1.4 for the look-ups, 1.5 for the sweep (the same time
// stamps).
template <int CHUNK>
__global__ __launch_bounds__(kRunThreads, 8) void runs_count_kernel(RunsArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int scan_scratch[17];
  __shared__ int s_cand_members;
  __shared__ int s_overlap[kWave];  // ROUGE-N: this partition's overlap with each reference
  const Problem& pb = a.pb;
  const int tid = threadIdx.x, nt = kRunThreads;
  const int parts = a.parts;
  const int p = blockIdx.x, idx = blockIdx.y, g = blockIdx.z;
  const int n = a.first_order + idx;
  const int T = 1 << a.log2_slots, W = a.words;
  unsigned long long* const table = reinterpret_cast<unsigned long long*>(smem);  // T, and for the
  // key that looks like a free slot one entry for each part of the table behind them
  uint32_t* const counters = reinterpret_cast<uint32_t*>(smem + a.off_counters);
  int* const prefix = reinterpret_cast<int*>(smem + a.off_prefix);
  int2* const runs = reinterpret_cast<int2*>(smem + a.off_runs);  // x + i: member i; y: sequence

  const int64_t slots = (int64_t(idx) * pb.B + g) * pb.group_cap;
  uint32_t at = 0;
  if (tid < a.chunks)
    at = a.run_at[((int64_t(idx) * pb.B + g) * a.chunks + tid) * parts + p];
  {
    uint4* const t4 = reinterpret_cast<uint4*>(table);
    for (int q = tid; q < (T + kSubs) / 2; q += nt) t4[q] = make_uint4(~0u, ~0u, ~0u, ~0u);
    uint4* const c4 = reinterpret_cast<uint4*>(counters);
    for (int q = tid; q < (T + kSubs) / 4 * W; q += nt) c4[q] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < kWave) s_overlap[tid] = 0;
  }
  int members;
  {
    const int size = int(at >> 16);
    const int before = block_exclusive_scan(size, scan_scratch, &members);
    if (tid < a.chunks) {
      const Chunk k = chunk_of<CHUNK>(a, tid);
      prefix[tid] = before;
      runs[tid] = make_int2(chunk_base(a, k) + int(at & 0xFFFFu) - before, k.seq);
    }
    if (tid == a.cand_chunks) s_cand_members = before;
  }
  __syncthreads();
  const int cand_members = s_cand_members;

  int half = 1;
  while (2 * half < a.chunks) half *= 2;
  constexpr int kBatch = 2;
  struct Batch {
    uint64_t key[kBatch];
    uint32_t word[kBatch];
    int seq[kBatch];
  };
  // members [base, base + 2 * nt) that lie before `end` > 0
  auto fetch = [&](Batch& b, int base, int end) {
    int i[kBatch], c[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      i[u] = min(base + u * nt + tid, end - 1);
      c[u] = 0;  // becomes the last run that starts at or before member i
    }
    for (int step = half; step; step >>= 1) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int q = c[u] + step;
        if (q < a.chunks && prefix[q] <= i[u]) c[u] = q;
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int2 run = runs[c[u]];
      b.seq[u] = run.y;
      b.key[u] = a.run_key[slots + run.x + i[u]];
      b.word[u] = a.run_times[slots + run.x + i[u]];
    }
  };

  const int log2_part = a.log2_slots - a.sub_bits;
  const uint32_t part_mask = (1u << log2_part) - 1u;
  bool lost = false;
  int created = 0;
  auto count_in = [&](uint32_t s, uint32_t word, int seq) {
    const uint32_t times = (word & 0xFFFu) + 1u;
    if (a.wide_fields)
      atomicAdd(&counters[__umul24(s, uint32_t(W)) + uint32_t(seq)], times);
    else
      atomicAdd(&counters[__umul24(s, uint32_t(W)) + uint32_t(seq >> 1)], times << (16 * (seq & 1)));
  };
  auto enter = [&](uint64_t key, uint32_t word, int seq) {
    const uint32_t sub = word >> 12;
    uint32_t s;
    if (key == kFree) {
      s = uint32_t(T) + sub;
      created += atomicCAS(&table[s], kFree, 0ull) == kFree ? 1 : 0;
    } else {
      const uint32_t h = run_hash(key), step = (h >> 3) | 1u, part = sub << log2_part;
      uint32_t q = (h >> (32 - a.log2_slots)) & part_mask;
      unsigned long long old = atomicCAS(&table[part | q], kFree, key);
      uint32_t rounds = 0;
      while (old != kFree && old != key && rounds < part_mask) {
        q = (q + step) & part_mask;
        old = atomicCAS(&table[part | q], kFree, key);
        ++rounds;
      }
      if (old != kFree && old != key) {
        lost = true;
        return;
      }
      created += old == kFree ? 1 : 0;
      s = part | q;
    }
    count_in(s, word, seq);
  };
  auto look_up = [&](uint64_t key, uint32_t word, int seq) {
    const uint32_t sub = word >> 12;
    uint32_t s;
    if (key == kFree) {
      s = uint32_t(T) + sub;
      if (table[s] == kFree) return;
    } else {
      const uint32_t h = run_hash(key), step = (h >> 3) | 1u, part = sub << log2_part;
      uint32_t q = (h >> (32 - a.log2_slots)) & part_mask;
      unsigned long long old = table[part | q];
      uint32_t rounds = 0;
      while (old != kFree && old != key && rounds < part_mask) {
        q = (q + step) & part_mask;
        old = table[part | q];
        ++rounds;
      }
      if (old != key) return;
      s = part | q;
    }
    count_in(s, word, seq);
  };

  Batch cand, ref;
  if (cand_members > 0) fetch(cand, 0, cand_members);  // uniform
  if (members > cand_members) fetch(ref, cand_members, members);
  for (int base = 0; base < cand_members; base += kBatch * nt) {
    if (base) fetch(cand, base, cand_members);
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (base + u * nt + tid < cand_members) enter(cand.key[u], cand.word[u], 0);
  }
  __syncthreads();
  for (int base = cand_members; base < members; base += kBatch * nt) {
    if (base != cand_members) fetch(ref, base, members);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (base + u * nt + tid < members) {
        if (a.enter_refs)
          enter(ref.key[u], ref.word[u], ref.seq[u]);
        else
          look_up(ref.key[u], ref.word[u], ref.seq[u]);
      }
    }
  }
  if (lost) {
    if (pb.status) atomicOr(pb.status, TB_DEV_TABLE_OVERFLOW);
    a.overflow[g] = 1;
  }
  __syncthreads();

  // maximum over the references, minimum with the candidate, sum
  int part = 0;
  if (W == 1) {  // one reference: four entries a request
    for (int q = tid; q < (T + kSubs) / 4; q += nt) {
      const uint4 e = reinterpret_cast<const uint4*>(counters)[q];
      part += int(min(e.x & 0xFFFFu, e.x >> 16) + min(e.y & 0xFFFFu, e.y >> 16) +
                  min(e.z & 0xFFFFu, e.z >> 16) + min(e.w & 0xFFFFu, e.w >> 16));
    }
  }
  for (int s = tid; W > 1 && s < T + kSubs; s += nt) {
    const uint32_t* const e = counters + __umul24(uint32_t(s), uint32_t(W));
    const uint32_t w0 = e[0];
    const uint32_t cc = a.wide_fields ? w0 : w0 & 0xFFFFu;
    uint32_t most = a.wide_fields ? 0u : w0 >> 16;
    for (int q = 1; q < W; ++q) {
      const uint32_t w = e[q];
      most = max(most, a.wide_fields ? w : max(w & 0xFFFFu, w >> 16));
    }
    part += int(min(cc, most));
    if (a.rouge_overlap && cc) {
      for (int j = 1; j <= pb.R; ++j) {
        const uint32_t w = e[a.wide_fields ? j : j >> 1];
        const uint32_t both = min(cc, a.wide_fields ? w : (j & 1) ? w >> 16 : w & 0xFFFFu);
        if (both) atomicAdd(&s_overlap[j - 1], int(both));
      }
    }
  }
  const int clipped = block_sum(part, scan_scratch);  // (its barriers complete s_overlap)
  if (a.rouge_overlap && tid < pb.R) {
    const int both = W == 1 ? clipped : s_overlap[tid];
    if (both) atomicAdd(&a.rouge_overlap[int64_t(g) * pb.R + tid], both);
  }
  const int64_t stat = int64_t(g) * pb.N + n - 1;
  if (a.enter_refs) {
    __syncthreads();  // (scan_scratch is used again)
    const int distinct = block_sum(created, scan_scratch);
    if (tid == 0 && distinct) atomicAdd(&a.st.distinct[stat], distinct);
  }
  if (tid == 0) {
    if (clipped) atomicAdd(&a.st.clipped[stat], clipped);
    if (p == 0) {
      const int len = clamped_len(uniform_load(pb.cand_len, g), pb.cand_stride, nullptr);
      a.st.total[stat] = max(len - n + 1, 0);
    }
  }
}

template <int ITEMS>
hipError_t launch_items(const RunsArgs& a, const RunsPlan& plan, hipStream_t s) {
  const auto count = runs_count_kernel<ITEMS * kRunThreads>;
  hipError_t e = grant_dynamic_lds(reinterpret_cast<const void*>(count), plan.lds_bytes);
  if (e != hipSuccess) return e;
  const int shares = (a.num_orders + a.orders_each - 1) / a.orders_each;
  hipLaunchKernelGGL(runs_sort_kernel<ITEMS>, dim3(a.chunks, shares, a.pb.B), dim3(kRunThreads), 0,
                     s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(count, dim3(a.parts, a.num_orders, a.pb.B), dim3(kRunThreads),
                     plan.lds_bytes, s, a);
  return hipGetLastError();
}

// Whether a table (or part of one) of `slots` slots holds what a hash sends to it of `entries` distinct
// n-grams dealt to `tables` of them.  The number is binomial; that it reaches k is less likely than
// exp(k - mean - k log(k / mean)) (Chernoff), here exp(-40): with 2^31 tables in a call, 1e-8.  Half full
// on average is room enough from 256 slots on; 128 may expect 51, 64 may expect 16.
bool has_room(int64_t entries, int64_t tables, int64_t slots) {
  const double mean = double(entries) / double(tables), k = double(slots);
  return mean < k && k - mean - k * std::log(k / mean) <= -40.0;
}

}  // namespace

bool plan_runs(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits,
               bool rouge, bool group_distinct, RunsPlan* plan) {
  RunsPlan& p = *plan;
  const int64_t cap = cand_stride + R * ref_stride;
  if (R >= kWave || cap > int64_t(4096) * kMaxRunParts || B > 65535) return false;
  p.wide_fields = cand_stride > 65535 || ref_stride > 65535;
  p.words = p.wide_fields ? R + 1 : (R + 2) / 2;
  p.num_orders = rouge ? 1 : N;
  const int64_t pairs = B * p.num_orders;

  // positions per thread: as many as leave every compute unit a workgroup
  p.items = 4;
  while (p.items > 1 && pairs * cap < int64_t(256) * p.items * kRunThreads) p.items /= 2;
  auto split = [&] {
    const int64_t chunk = p.items * kRunThreads;
    p.cand_chunks = int((cand_stride + chunk - 1) / chunk);
    p.ref_chunks = int((ref_stride + chunk - 1) / chunk);
    return p.cand_chunks + int64_t(R) * p.ref_chunks;
  };
  while (p.items < 4 && split() > kMaxChunks) p.items *= 2;
  const int64_t chunks = split();
  if (chunks > kMaxChunks) return false;
  p.chunks = int(chunks);

  auto lds_for = [&](int log2_slots) {
    const size_t T = size_t(1) << log2_slots;
    p.off_counters = uint32_t((T + kSubs) * 8);
    p.off_runs = p.off_counters + uint32_t((T + kSubs) * 4 * p.words);
    p.off_prefix = p.off_runs + uint32_t(8 * p.chunks);
    p.lds_bytes = (p.off_prefix + 4 * size_t(p.chunks) + 15) & ~size_t(15);
    p.log2_slots = log2_slots;
    return p.lds_bytes + 1024;  // (the kernel's static arrays)
  };
  // entries a table may be expected to hold: half its slots.  The largest table (up to 4096 slots)
  // of which two fit a compute unit; a larger one only where there would be too many partitions.
  const int64_t entries = group_distinct ? cap : cand_stride;
  int log2_slots = 12;
  while (log2_slots > 10 && lds_for(log2_slots) > size_t(kLdsBudget) / 2) --log2_slots;
  while (log2_slots < 13 && (entries >> (log2_slots - 1)) >= kMaxRunParts) ++log2_slots;
  if (lds_for(log2_slots) > size_t(kLdsBudget)) return false;
  const int64_t half_full = int64_t(1) << (log2_slots - 1);
  int64_t parts = (entries + half_full - 1) / half_full;
  // the chip holds 512 workgroups of the counting kernel: more partitions than the tables ask for, until
  // the last round of workgroups is a full one, but none of less than 512 n-grams
  const int64_t rounds = (pairs * parts + 511) / 512;
  const int64_t fill = rounds * 512 / pairs, most = entries / 512;
  const int64_t more = fill < most ? fill : most;
  parts = more > parts ? more : parts;
  if (parts > kMaxRunParts && half_full * kMaxRunParts >= entries) parts = kMaxRunParts;
  if (parts < 2) parts = 2;
  // bits of an n-gram beyond 64 (they have to lie in its first token)
  const int beyond = N * bits - 64;
  p.beyond = beyond > 0;
  p.log2_parts = p.sub_bits = 0;
  if (p.beyond) {
    if (beyond > bits) return false;
    int lg = 1;
    while ((int64_t(1) << lg) < parts) ++lg;
    while (lg + kSubBits < beyond) ++lg;
    // one partition more instead of one part of a table: the parts keep their n-grams and get twice the
    // slots.  (8192 tokens of 18 bits with 16 references: 32 n-grams in 64 slots, now in 128.)  Where
    // partitions would become too many or too small, larger tables.
    auto sub_bits = [&] { return beyond > lg ? beyond - lg : 0; };
    while (!has_room(entries, int64_t(1) << (lg + sub_bits()), int64_t(1) << (log2_slots - sub_bits()))) {
      if ((int64_t(2) << lg) <= kMaxRunParts && entries >> (lg + 1) >= 64)
        ++lg;
      else if (++log2_slots > 13 || lds_for(log2_slots) > size_t(kLdsBudget))
        return false;
    }
    parts = int64_t(1) << lg;
    if (entries / parts < 64) return false;  // partitions of a few n-grams: not worth it
    p.log2_parts = lg;
    p.sub_bits = sub_bits();
  }
  if (parts > kMaxRunParts) return false;
  p.parts = int(parts);
  // orders a sorting workgroup takes: as many as leave the chip two full rounds of workgroups
  p.orders_each = p.num_orders;
  while (p.orders_each > 1 &&
         B * ((p.num_orders + p.orders_each - 1) / p.orders_each) * chunks < 1024)
    p.orders_each = (p.orders_each + 1) / 2;
  // the runs' places lie where the partitioned kernels keep the ids of a group's slots
  return chunks * parts <= cap;
}

hipError_t launch_runs(const Problem& pb, const RunsPlan& plan, const RunsBuffers& buffers,
                       const StatPtrs& st, bool group_distinct, int32_t* rouge_overlap,
                       hipStream_t s) {
  RunsArgs a;
  a.pb = pb;
  a.st = st;
  a.run_key = buffers.keys;
  a.run_times = buffers.times;
  a.run_at = buffers.places;
  a.overflow = buffers.overflow;
  a.rouge_overlap = rouge_overlap;
  a.num_orders = plan.num_orders;
  a.first_order = rouge_overlap ? pb.N : 1;
  a.orders_each = plan.orders_each;
  a.parts = plan.parts;
  a.log2_parts = plan.log2_parts;
  a.sub_bits = plan.sub_bits;
  a.beyond = plan.beyond;
  a.log2_slots = plan.log2_slots;
  a.cand_chunks = plan.cand_chunks;
  a.ref_chunks = plan.ref_chunks;
  a.chunks = plan.chunks;
  a.words = plan.words;
  a.wide_fields = plan.wide_fields;
  a.enter_refs = group_distinct ? 1 : 0;
  a.off_counters = plan.off_counters;
  a.off_prefix = plan.off_prefix;
  a.off_runs = plan.off_runs;
  if (plan.items == 4) return launch_items<4>(a, plan, s);
  if (plan.items == 2) return launch_items<2>(a, plan, s);
  return launch_items<1>(a, plan, s);
}

}  // namespace tb
