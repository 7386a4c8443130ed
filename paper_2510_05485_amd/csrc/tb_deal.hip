// Whole calls on groups beyond one LDS table, BLEU of up to four orders and ROUGE-1 and -2, in two kernels:
//
//   deal_kernel   one workgroup per (group, chunk of 1024 or 2048 positions of one sequence): deals the
//                 chunk's positions out to partitions three times, as three kinds of members: its tokens by a
//                 hash of the token, its pairs by a hash of both, its 4-grams by a hash of the first three
//                 tokens.  Equal ones are merged, what is left is written as one run per partition, with the
//                 runs' places
//   tally_kernel  one workgroup per (group, partition of a kind): gathers the partition's runs, enters the
//                 candidate's members into an LDS table, looks the references' up, counts and clips; orders 3
//                 and 4 in one go
//
// The sorted runs (tb_runs.hip) do the same for one order at a time: every position is dealt out four times
// there, each time with six barriers, and four workgroups count a partition's share, each with its own trips to
// memory.  Here the tokens are read once and the barriers are shared.  Orders 3 and 4 go together because an
// n-gram that is new to the candidate at order 3 is new at order 4, too, and the 4-gram that goes on like the
// first one does needs no entry (as in the fused kernel).  Order 2 stays apart: the most frequent pair of a
// Zipf-distributed text is a fiftieth of it, and the partition that received all 4-grams that start with it took
// five times as long as the others.  One workgroup for all kinds of a partition was tried, too: its tables left
// room for shares of 640 positions only, and what a workgroup costs however little it has (places, clearing,
// sums) ate the gain (50 groups of two times 20 000: 66.6 us a call, 61.5 like this).
//
// Equal ones are merged as in the sorted runs: of the positions whose keys hash to the same word one is kept
// there, and those equal to it add themselves to its count; any other is passed on as it is.
//
// What bounds it.  Dealing: 7.7 us a workgroup, six barriers' worth of LDS and memory latency, two of them on a
// unit, and the 19 bytes a position that it writes.  Tallying: latency, too (one text of 262 144 tokens: 356 vector and
// 347 scalar instructions of a wavefront, which waits 64 % of its cycles; 37 MB fetched for the 11.5 that were
// written: a partition's places lie a row of partitions apart), and the longest workgroups.
//
// Measured (us a call, sorted runs -> this): one text of 262 144 tokens with its reference 32.6 -> 25.8; 11 groups of two
// times 90 000 96.7 -> 59; 50 of two times 20 000 80.4 -> 57; 16 of two times 12 500 32 -> 22.6; two of 174 762
// with two references 65 -> 40.  Of these the scores inside the counting kernel, instead of in one of their own, and
// arguments read where they are used 2 to 4 us each (113 scalar registers were moved to lanes and back, then 33; with the
// code for crowded partitions 84 to 102).
//
// Keys are exact.  What the tables hold is bounded by the hashes whatever the tokens are, except for 4-grams:
// where many different ones start with the same three tokens and ids run out, orders 3 and 4 are counted again, each
// on its own, order 4 in shares that the group's workgroups take in turn (see tally_crowd).  A table that is full
// then (which takes tokens chosen to collide) is reported through TB_DEV_TABLE_OVERFLOW and scored NaN.
#include <cmath>

#include "tb_kernels.h"
#include "tb_score.h"

namespace tb {

namespace {

constexpr int kThreads = 1024;
constexpr int kKinds = 3;
constexpr int kMaxParts = 2 * kThreads;  // of all kinds (a thread of the dealing kernel scans two counts)
constexpr int kTallyThreads = 1024;
constexpr int kMaxDealChunks = kTallyThreads;  // per group: one thread each reads a run's place
constexpr int kTokenBits = 20;
constexpr uint32_t kNoToken = (1u << kTokenBits) - 1u;  // behind the end of a sequence
constexpr uint32_t kGivenBack = ~0u;  // in the place of an id's token
constexpr uint32_t kAlone = 3;  // shares of a crowded partition that its own workgroup takes by itself
constexpr int kCrowds = 64;     // crowded partitions of a group whose shares others are told of

struct DealArgs {
  Problem pb;
  StatPtrs st;
  uint64_t* pair;    // [B * group_cap]: tokens 0 and 1 | multiplicity - 1, from bit 40 on
  uint64_t* rest;    // tokens 1 to 3 of a 4-gram
  uint32_t* lead;    // its token 0 | multiplicity - 1, from bit 20 on
  uint32_t* first;   // token | multiplicity - 1, from bit 20 on
  uint32_t* run_at;  // [B][chunks][parts of all kinds]: first of the run within its chunk | size << 16
  int32_t* overflow; // [B]
  int32_t* rouge_overlap;  // [B, R] or null
  unsigned long long* arrived;  // [B, N]: sum of the partitions' matches | partitions and shares of them << 24 | shares
                                // there are << 40 | spoilt ones << 52
  int32_t* complete;  // [B]: orders all of whose partitions have arrived
  // Crowded partitions (see tally_crowd):
  int32_t* crowds;      // [B]: how many
  int32_t* crowd;       // [B][kCrowds]: partition << 16 | shares, or 0
  int32_t* next_share;  // [B][kCrowds]: shares that have been taken
  ScoreParams sp;
  void* out;          // per-sentence scores, or null
  int first_kind, kinds, all_parts;  // kinds first_kind .. kinds - 1
  int parts[kKinds], parts_before[kKinds];  // of each kind; of the kinds before it
  int log2_chunk;
  int cand_chunks, ref_chunks, chunks;  // of the candidate, of one reference, of a group
  // tally_kernel
  int words;         // per counter
  int capacity;      // ids of order 3 and 4 n-grams
  uint32_t per_member;  // 2^32 / members of a share
  int window[kKinds];  // members of a kind that the marks are for, a multiple of 64
  int id_bits, log2_first, log2_pair, log2_item;
  // LDS: table and counters at 0, (4-grams: tokens under the ids,) marks, and for all kinds
  uint32_t off_tokens, off_lead, off_sums, off_places, off_scratch;
};

struct DealChunk {
  int seq, first;
};
__device__ __forceinline__ DealChunk deal_chunk(const DealArgs& a, int c) {
  DealChunk k;
  const int q = max(c - a.cand_chunks, 0);
  const int j = a.pb.R > 1 ? q / a.ref_chunks : 0;
  k.seq = c < a.cand_chunks ? 0 : 1 + j;
  k.first = (c < a.cand_chunks ? c : q - j * a.ref_chunks) << a.log2_chunk;
  return k;
}
// Where a chunk's n-grams lie among the group's slots.
__device__ __forceinline__ int deal_base(const DealArgs& a, const DealChunk& k, int* seq) {
  *seq = k.seq;
  return (k.seq == 0 ? 0 : int(a.pb.cand_stride) + (k.seq - 1) * int(a.pb.ref_stride)) + k.first;
}

// Hashes of one, two, three and four tokens: top bits choose the partition.
__device__ __forceinline__ uint32_t hash1(uint32_t t0) { return t0 * 0x9E3779B1u + 0x6A09E667u; }
__device__ __forceinline__ uint32_t mix(uint32_t h) { return (h ^ (h >> 15)) * 0xC2B2AE3Du; }
__device__ __forceinline__ uint32_t hash2(uint32_t t0, uint32_t t1) { return mix(t0 * 0x9E3779B1u + t1 * 0x85EBCA6Bu); }
__device__ __forceinline__ uint32_t hash3(uint32_t t0, uint32_t t1, uint32_t t2) {
  return mix(t0 * 0x9E3779B1u + t1 * 0x85EBCA6Bu + t2 * 0x27D4EB2Fu);
}
__device__ __forceinline__ uint32_t hash4(uint32_t h3, uint32_t t3) { return mix(h3 + t3 * 0x165667B1u); }
// (The partition is the high word of hash * parts: the low word's top bits choose the slot.)

// A store that leaves the XCD's L2 at once.  (Ordinary ones wait there for the end of the kernel, which then takes
// as long as it takes to write them all.)
template <typename T>
__device__ __forceinline__ void write_through(T* at, T v) {
  __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int ITEMS>
__global__ __launch_bounds__(kThreads, 8) void deal_kernel(DealArgs a) {
  constexpr int kChunk = ITEMS * kThreads;
  constexpr int kLog2Chunk = ITEMS == 2 ? 11 : 10;
  static_assert((1 << kLog2Chunk) == kChunk, "chunk");
  struct Out {
    uint64_t pair[kChunk], rest[kChunk];
    uint32_t lead[kChunk], first[kChunk];
  };
  union Space {
    uint32_t kept[kKinds][kChunk];  // by hash: position kept there | its duplicates << 12
    Out out;
  };
  __shared__ Space space;
  __shared__ uint32_t token[kChunk + 8];
  __shared__ int in_part[2 * kThreads];
  __shared__ int kind_base[kKinds + 1];
  __shared__ int scan_scratch[17];
  const Problem& pb = a.pb;
  const int tid = threadIdx.x, kinds = a.kinds, first_kind = a.first_kind;
  const int c = blockIdx.x, g = blockIdx.y;
  const DealChunk me = deal_chunk(a, c);
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
  const int left = max(len - me.first, 0);
  const int staged = min(left, kChunk + 3);

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
      t[u] = load_token(base, row + min(u * kThreads + tid, staged - 1), pb.tok64);
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
      if (u * kThreads + tid < staged) put(u * kThreads + tid, t[u]);
    if (kChunk + tid < staged) put(kChunk + tid, load_token(base, row + kChunk + tid, pb.tok64));
  }
  reinterpret_cast<int2*>(in_part)[tid] = make_int2(0, 0);
  if (c == 0) {  // what the partitions' workgroups add to
    if (tid < pb.N) {
      a.st.clipped[int64_t(g) * pb.N + tid] = 0;
      a.st.distinct[int64_t(g) * pb.N + tid] = 0;
    }
    if (tid == 0) a.overflow[g] = a.complete[g] = a.crowds[g] = 0;
    if (tid < kCrowds) a.crowd[g * kCrowds + tid] = a.next_share[g * kCrowds + tid] = 0;
    if (tid < pb.N) a.arrived[int64_t(g) * pb.N + tid] = 0;
    if (a.rouge_overlap && tid < pb.R) a.rouge_overlap[int64_t(g) * pb.R + tid] = 0;
  }
  if (bad && pb.status) atomicOr(pb.status, TB_DEV_TOKEN_RANGE);
  __syncthreads();

  uint32_t t[ITEMS][4], h[ITEMS][kKinds];
  // (4-grams by all of their tokens: by three, as they are dealt, all that go on otherwise than the one kept would be
  // passed on, of two different tokens every second position: one text of 262 144 of them 92.6 us a call, now 19.6)
  auto slot = [&](int u, int kind) {
    return (kind == 2 ? hash4(h[u][2], t[u][3]) : h[u][kind]) >> (32 - kLog2Chunk);
  };
  // tokens from its position on that a member of the kind has, and one that others are merged into
  auto is_member = [&](int u, int kind) { return left - (u * kThreads + tid) > kind; };
  // (of three orders the fourth token is none: two texts of 100 000, a quarter of them behind one beginning, 107 us a
  // call, now 25)
  const uint32_t fourth = pb.N > 3 ? ~0u : 0u;
  const int merge_left = pb.N > 3 ? 3 : 2;
  auto merges = [&](int u, int kind) { return left - (u * kThreads + tid) > (kind == 2 ? merge_left : kind); };
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
    const int k = u * kThreads + tid;
#pragma unroll
    for (int j = 0; j < 4; ++j) t[u][j] = token[k + j];
    if (left - k <= 3 || !fourth) t[u][3] = kNoToken;
    h[u][0] = hash1(t[u][0]);
    h[u][1] = hash2(t[u][0], t[u][1]);
    h[u][2] = hash3(t[u][0], t[u][1], t[u][2]);
#pragma unroll
    for (int kind = 0; kind < kKinds; ++kind)
      if (kind >= first_kind && kind < kinds && merges(u, kind)) space.kept[kind][slot(u, kind)] = uint32_t(k);
  }
  __syncthreads();
  // (Reads of all kinds first, whether they count or not: with a branch around each, a wavefront waited for six
  // chains of three LDS accesses one after the other.)
  bool merged[ITEMS][kKinds];
  int part[ITEMS][kKinds];
  {
    uint32_t w[ITEMS][kKinds];
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
#pragma unroll
      for (int kind = 0; kind < kKinds; ++kind)
        w[u][kind] = space.kept[kind][slot(u, kind)] & uint32_t(kChunk - 1);
    uint32_t differs[ITEMS][kKinds];
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
#pragma unroll
      for (int kind = 0; kind < kKinds; ++kind) {
        differs[u][kind] = 0;
#pragma unroll
        for (int j = 0; j < (kind == 2 ? 4 : kind + 1); ++j)
          differs[u][kind] |= (token[w[u][kind] + j] ^ t[u][j]) & (j == 3 ? fourth : ~0u);
      }
#pragma unroll
    for (int u = 0; u < ITEMS; ++u)
#pragma unroll
      for (int kind = 0; kind < kKinds; ++kind) {
        merged[u][kind] = merges(u, kind) && w[u][kind] != uint32_t(u * kThreads + tid) && differs[u][kind] == 0u;
        part[u][kind] = a.parts_before[kind] + int(__umulhi(h[u][kind], uint32_t(a.parts[kind])));
      }
  }
  int rank[ITEMS][kKinds];
  uint32_t member = 0;  // by bits: what is passed on
#pragma unroll
  for (int u = 0; u < ITEMS; ++u)
#pragma unroll
    for (int kind = 0; kind < kKinds; ++kind) {
      rank[u][kind] = 0;
      if (kind < first_kind || kind >= kinds) continue;  // uniform
      if (merged[u][kind]) {
        atomicAdd(&space.kept[kind][slot(u, kind)], 0x1000u);
      } else if (is_member(u, kind)) {
        rank[u][kind] = atomicAdd(&in_part[part[u][kind]], 1);
        member |= 1u << (u * kKinds + kind);
      }
    }
  __syncthreads();
  uint32_t times[ITEMS][kKinds];
#pragma unroll
  for (int u = 0; u < ITEMS; ++u)
#pragma unroll
    for (int kind = 0; kind < kKinds; ++kind) {
      const uint32_t word = space.kept[kind][slot(u, kind)];
      times[u][kind] = merges(u, kind) && int(word & 0xFFFu) == u * kThreads + tid ? word >> 12 : 0u;
    }
  const int2 mine = reinterpret_cast<const int2*>(in_part)[tid];
  int total;
  const int before = block_exclusive_scan(mine.x + mine.y, scan_scratch, &total);
#pragma unroll
  for (int kind = 0; kind <= kKinds; ++kind) {
    const int q = kind < kinds ? a.parts_before[kind] : a.all_parts;  // (its members begin where all before it end)
    if (tid == q / 2) kind_base[kind] = before + (q & 1 ? mine.x : 0);
    if (q == 2 * kThreads && tid == 0) kind_base[kind] = total;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int q = 2 * tid + j, size = j ? mine.y : mine.x;
    if (q >= a.all_parts) continue;
    const int kind = kinds > 2 && q >= a.parts_before[2] ? 2 : kinds > 1 && q >= a.parts_before[1] ? 1 : 0;
    const int first = before + (j ? mine.x : 0) - kind_base[kind];
    in_part[q] = first;
    write_through(a.run_at + (int64_t(g) * a.chunks + c) * a.all_parts + q, uint32_t(first) | uint32_t(size) << 16);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ITEMS; ++u)
#pragma unroll
    for (int kind = 0; kind < kKinds; ++kind)
      if (kind >= first_kind && kind < kinds) rank[u][kind] += in_part[part[u][kind]];
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
#pragma unroll
    for (int kind = 0; kind < kKinds; ++kind) {
      if (!(member >> (u * kKinds + kind) & 1u)) continue;
      const int at = rank[u][kind];
      if (kind == 0) space.out.first[at] = t[u][0] | times[u][0] << kTokenBits;
      if (kind == 1)
        space.out.pair[at] = uint64_t(t[u][0]) | uint64_t(t[u][1]) << kTokenBits |
                             uint64_t(times[u][1]) << (2 * kTokenBits);
      if (kind == 2) {
        space.out.rest[at] = uint64_t(t[u][1]) | uint64_t(t[u][2]) << kTokenBits |
                             uint64_t(t[u][3]) << (2 * kTokenBits);
        space.out.lead[at] = t[u][0] | times[u][2] << kTokenBits;
      }
    }
  }
  __syncthreads();
  int seq;
  const int64_t out = int64_t(g) * pb.group_cap + deal_base(a, me, &seq);
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
    const int i = u * kThreads + tid;
    if (i < kind_base[1]) write_through(a.first + out + i, space.out.first[i]);
    if (kinds > 1 && i < kind_base[2] - kind_base[1]) write_through(a.pair + out + i, space.out.pair[i]);
    if (kinds > 2 && i < kind_base[3] - kind_base[2]) {
      write_through(a.rest + out + i, space.out.rest[i]);
      write_through(a.lead + out + i, space.out.lead[i]);
    }
  }
}

__device__ __forceinline__ int wave_inclusive_max(int v) {  // of values >= 0
  v = max(v, dpp_or_zero<0x111, 0xf, 0xf>(v));  // row_shr:1
  v = max(v, dpp_or_zero<0x112, 0xf, 0xf>(v));  // row_shr:2
  v = max(v, dpp_or_zero<0x114, 0xf, 0xf>(v));  // row_shr:4
  v = max(v, dpp_or_zero<0x118, 0xf, 0xf>(v));  // row_shr:8
  v = max(v, dpp_or_zero<0x142, 0xa, 0xf>(v));  // row_bcast:15 into rows 1 and 3
  return max(v, dpp_or_zero<0x143, 0xc, 0xf>(v));  // row_bcast:31 into rows 2 and 3
}

template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds(uint32_t offset) {
  typedef __attribute__((address_space(3))) T* Ptr;
  return (Ptr)(uintptr_t)(offset);
}
template <typename T>
__device__ __forceinline__ T lds_cas(uint32_t at, T desired, T expected = 0) {
  __hip_atomic_compare_exchange_strong((T*)lds<T>(at), &expected, desired, __ATOMIC_RELAXED,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return expected;
}
__device__ __forceinline__ uint32_t lds_add(uint32_t at, uint32_t v) {
  return __hip_atomic_fetch_add((uint32_t*)lds<uint32_t>(at), v, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_add_only(uint32_t at, uint32_t v) {
  __hip_atomic_fetch_add((uint32_t*)lds<uint32_t>(at), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t lds_peek(uint32_t at) {  // (as it is now)
  return __hip_atomic_load((uint32_t*)lds<uint32_t>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
typedef uint32_t Quad __attribute__((ext_vector_type(4)));

// One reference: a counter is one less than the candidate's count, less what the reference has had of it; what
// the reference finds is a match.  More: counters of the candidate (one less) and of each reference, two a word
// where no sequence is longer than 65 535, and a pass over them in the end.
// With the sizes of the group's dictionaries (kAll...) the references' n-grams are entered, too, and every
// occurrence is counted.
enum Counters { kOneReference, kHalves, kWords, kAllHalves, kAllWords };

// The kernel's arguments, read through the argument segment where they are used (loads of a by-value parameter all stand
// at the entry and occupy scalar registers throughout); and read once more by who calls this again.
__device__ __forceinline__ const DealArgs& arguments() {
  typedef const char __attribute__((address_space(4)))* Segment;
  Segment at = (Segment)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(at));
  return *(const DealArgs*)at;
}

// What a workgroup of the tallying kernel works with.  (The rare parts below have an object of their own, from
// arguments that are read again: shared with the usual part, their values took its scalar registers, 95 of which
// were moved to lanes and back.)
template <int KIND, Counters COUNTERS>
struct Tally {
  static constexpr bool ONE = COUNTERS == kOneReference, HALVES = COUNTERS == kHalves || COUNTERS == kAllHalves;
  static constexpr bool ALL = COUNTERS == kAllHalves || COUNTERS == kAllWords;
  static constexpr int kWaves = kTallyThreads / kWave;
  struct Member {
    uint64_t key;   // pair, or the rest of a 4-gram
    uint32_t word;  // token, or the first one of a 4-gram
    int f;
  };
  struct Item {
    uint32_t t0;
    uint64_t rest;
  };

  const DealArgs& a;
  const int tid, lane, wave, g, N;
  const uint32_t parts;
  // (LDS: the table at 0, its counters behind it, then what follows here)
  const uint32_t lost_at, ids_at, again_at;
  const uint32_t table_bytes, slots_bytes;
  const uint32_t counters4, used_bytes;  // KIND 2: order 4's
  const int window;
  const uint32_t cand_marks, ref_marks;
  const int64_t slots;
  // 4-grams: ids, and the tokens under them
  const uint32_t id_limit, capacity, bucket_mask;
  int run_size, before, members, cand_members;
  uint32_t matches = 0, matches4 = 0;  // (4-grams)

  __device__ __forceinline__ explicit Tally(const DealArgs& args)
      : a(args), tid(threadIdx.x), lane(tid & (kWave - 1)), wave(__builtin_amdgcn_readfirstlane(tid / kWave)),
        g(blockIdx.y), N(a.pb.N), parts(uint32_t(a.parts[KIND])),
        lost_at(a.off_sums), ids_at(lost_at + 4u), again_at(lost_at + 8u),
        table_bytes(KIND == 0 ? 4u << a.log2_first : KIND == 1 ? 8u << a.log2_pair : 4u << a.log2_item),
        slots_bytes(KIND == 0 ? 4u << a.log2_first : KIND == 1 ? 4u << a.log2_pair : 4u * uint32_t(a.capacity)),
        counters4(table_bytes + slots_bytes * uint32_t(ONE ? 1 : a.words)),
        used_bytes(KIND < 2 ? counters4 : counters4 + slots_bytes * uint32_t(N < 4 ? 0 : ONE ? 1 : a.words)),
        window(a.window[KIND]),
        cand_marks(KIND < 2 ? used_bytes : (a.off_lead + 4u * uint32_t(a.capacity) + 15u) & ~15u),
        ref_marks(cand_marks + 2u * uint32_t(window)), slots(int64_t(g) * a.pb.group_cap),
        id_limit(1u << a.id_bits), capacity(uint32_t(a.capacity)), bucket_mask(((4u << a.log2_item) - 1u) & ~15u) {}

  __device__ __forceinline__ auto scratch(int i) const { return lds<int>(a.off_scratch + 4u * uint32_t(i)); }
  __device__ __forceinline__ auto place_of(int run) const { return lds<int>(a.off_places + 4u * uint32_t(run)); }
  __device__ __forceinline__ auto before_of(int run) const { return place_of(a.chunks + run); }
  __device__ __forceinline__ auto seq_of(int run) const { return place_of(2 * a.chunks + run); }
  __device__ __forceinline__ void clear(uint32_t from, uint32_t to) const {
    for (uint32_t q = from + 16u * uint32_t(tid); q < to; q += 16u * kTallyThreads) *lds<Quad>(q) = Quad(0u);
  }
  __device__ __forceinline__ uint32_t load_place(int partition) const {
    if (tid >= a.chunks) return 0u;
    return a.run_at[(int64_t(g) * a.chunks + tid) * a.all_parts + a.parts_before[KIND] + partition];
  }

  // Members: those of the candidate's chunks, then those of the references'.
  __device__ __forceinline__ void gather(uint32_t place) {
    run_size = int(place >> 16);
    before = wave_inclusive_scan(run_size);
    if (lane == kWave - 1) *scratch(wave) = before;
    __syncthreads();
    const int of_waves = row_inclusive_scan(*scratch(lane & (kWaves - 1)));
    members = lane_value(of_waves, kWaves - 1);
    if (wave > 0) before += __builtin_amdgcn_readlane(of_waves, (wave - 1) & 15);
    before -= run_size;
    if (tid == a.cand_chunks) *scratch(16) = before;
    // where a run's members are: x + member; and whose they are
    if (tid < a.chunks) {
      int seq;
      const int base = deal_base(a, deal_chunk(a, tid), &seq);
      *place_of(tid) = base + int(place & 0xFFFFu) - before;
      if (KIND == 2) *before_of(tid) = before;
      if (!ONE) *seq_of(tid) = seq;
    }
  }
  // Windows of `window` members, in blocks of 64 that the wavefronts take in turn.  A run marks its first member
  // in the window and every member at a multiple of 64: the largest mark up to a lane is its run.
  __device__ __forceinline__ void mark(uint32_t marks, int begin, int size) const {
    const int lo = max(before - begin, 0), hi = min(before + run_size - begin, size);
#pragma unroll 1
    for (int i = lo; i < hi; i = (i | (kWave - 1)) + 1) *lds<uint16_t>(marks + 2u * uint32_t(i)) = uint16_t(tid + 1);
  }
  __device__ __forceinline__ Member load(int i, int run, bool cand) const {
    Member m;
    const int64_t at = slots + i + *place_of(run);
    m.f = cand ? 0 : ONE ? 1 : *seq_of(run);
    m.key = 0;
    m.word = 0;
    if (KIND == 0) m.word = a.first[at];
    if (KIND == 1) m.key = a.pair[at];
    if (KIND == 2) m.key = a.rest[at], m.word = a.lead[at];
    return m;
  }
  // block of a window of `size` > 64 * block members from `begin` on
  __device__ __forceinline__ Member fetch(uint32_t marks, int begin, int size, int block, bool cand) const {
    const uint32_t mark = marks + 2u * uint32_t(block * kWave + lane);
    const int run = wave_inclusive_max(*lds<uint16_t>(mark)) - 1;
    *lds<uint16_t>(mark) = 0;  // (for the next window)
    // (behind the last member: the last one again)
    return load(begin + min(block * kWave + lane, size - 1), run, cand);
  }

  // Adds `times` occurrences in sequence f to the counter; `is_new`: the candidate's first.
  __device__ __forceinline__ void count(uint32_t at, uint32_t times, int f, bool is_new, uint32_t& matched) const {
    if (f == 0) {
      lds_add_only(at, times - (is_new && !ALL ? 1u : 0u));
    } else if (ONE) {
      const int had = int(lds_add(at, 0u - times)) + 1;
      matched += uint32_t(min(max(had, 0), int(times)));
    } else {
      lds_add_only(at + uint32_t(HALVES ? f >> 1 : f) * slots_bytes, HALVES ? times << (16 * (f & 1)) : times);
    }
  }
  // Tables of whole keys, probed slot by slot.
  template <typename Key>
  __device__ __forceinline__ void do_key(Key key, uint32_t s, uint32_t times, int f) {
    constexpr uint32_t kSize = sizeof(Key);
    Key old = *lds<Key>(s);
    if (f > 0 && !ALL) {
      for (uint32_t left = table_bytes; old != key && old != 0 && left; left -= kSize) {
        s = (s + kSize) & (table_bytes - 1u);
        old = *lds<Key>(s);
      }
      if (old != key) return;
    } else {
      uint32_t left = table_bytes;
      while (true) {
        if (old == 0) old = lds_cas<Key>(s, key);
        if (old == 0 || old == key || left == 0) break;
        s = (s + kSize) & (table_bytes - 1u);
        old = *lds<Key>(s);
        left -= kSize;
      }
      if (old != 0 && old != key) {  // (full)
        *lds<uint32_t>(lost_at) = 1u;
        return;
      }
    }
    count(table_bytes + s / (kSize / 4u), times, f, old == 0, matches);
  }
  __device__ __forceinline__ void do_first(uint32_t word, int f) {
    const uint32_t t = word & kNoToken;
    do_key<uint32_t>(t + 1u, (hash1(t) * parts) >> (32 - a.log2_first) << 2, (word >> kTokenBits) + 1u, f);
  }
  __device__ __forceinline__ void do_pair(uint64_t word, int f) {
    const uint32_t h = hash2(uint32_t(word) & kNoToken, uint32_t(word >> kTokenBits) & kNoToken);
    do_key<uint64_t>((word & ((1ull << (2 * kTokenBits)) - 1ull)) | 1ull << 63, (h * parts) >> (32 - a.log2_pair) << 3,
                     uint32_t(word >> (2 * kTokenBits)) + 1u, f);
  }

  __device__ __forceinline__ Item load_item(uint32_t id) const {
    return Item{*lds<uint32_t>(a.off_lead + 4u * id), *lds<uint64_t>(a.off_tokens + 8u * id)};
  }
  static __device__ __forceinline__ bool same(const Item& x, const Item& y, int n) {
    const uint64_t mask = n == 3 ? (1ull << (2 * kTokenBits)) - 1ull : ~0ull;
    return x.t0 == y.t0 && ((x.rest ^ y.rest) & mask) == 0ull;
  }
  static __device__ __forceinline__ uint32_t last_of(const Item& x) { return uint32_t(x.rest >> (2 * kTokenBits)); }
  static __device__ __forceinline__ uint32_t item_hash(const Item& x) {
    return hash3(x.t0, uint32_t(x.rest) & kNoToken, uint32_t(x.rest >> kTokenBits) & kNoToken);
  }
  // An id that a lane took and had no use for, where there are no new ones; `capacity`: none found.  (Each lane looks at
  // places of its own: where lanes lose many ids, the first ones will do, and few lost are no use.)
  __device__ __forceinline__ uint32_t id_given_back() const {
    uint32_t h = uint32_t(tid) * 0x85EBCA6Bu;
#pragma unroll 1
    for (int tries = 0; tries < 24 && !lds_peek(again_at); ++tries) {
      h = h * 0x9E3779B1u + 0x7F4A7C15u;
      const uint32_t id = __umulhi(h, capacity), at = a.off_lead + 4u * id;
      if (lds_peek(at) == kGivenBack && lds_cas<uint32_t>(at, 0u, kGivenBack) == kGivenBack) return id;
    }
    *lds<uint32_t>(again_at) = 1u;
    return capacity;
  }
  // The id of the n-gram of order n (3 or 4) with hash h, and the item under it; it is entered if it is the
  // candidate's and not there.  false: not there, or no id left for it.  Who enters one takes an id, writes the
  // tokens under it and then swaps it in; where another lane was first, the id is given back.  (Ids that were lost
  // there ran out on texts of few different tokens, which all lanes enter at once: two of 100 000, 13 different ones,
  // 122 us a call, now 25.  The lanes with the n-gram of the first one used to wait for its id instead: that took
  // longer than it saved, 50 groups of two times 20 000 61.1 us, now 60.2.)
  __device__ __forceinline__ bool resolve(const Item& x, uint32_t h, int n, int f, uint32_t& id, Item& found,
                                          bool& is_new) const {
    uint32_t s = ((h * parts) >> (30 - a.log2_item)) & bucket_mask;
    const uint32_t mine = h << (a.id_bits + 1) | uint32_t(n - 2) << a.id_bits;
    Quad e;
    is_new = false;
    // (buckets of four, filled front to back: a free slot ends the search)
    while (true) {
      e = *lds<Quad>(s);
      id = min(min(e.x ^ mine, e.y ^ mine), min(e.z ^ mine, e.w ^ mine));
      if (id < id_limit) {
        found = load_item(id);
        if (same(found, x, n)) return true;
#pragma unroll 1
        for (uint32_t k = 0; k < 16u; k += 4u) {  // another one with the same bits: each entry of its own
          id = *lds<uint32_t>(s + k) ^ mine;
          if (id >= id_limit) continue;
          found = load_item(id);
          if (same(found, x, n)) return true;
        }
      }
      if (e.w == 0u) break;
      s = (s + 16u) & bucket_mask;
    }
    if (f > 0 && !ALL) return false;
    const uint64_t entering = __builtin_amdgcn_ballot_w64(true);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(uint32_t(entering >> 32),
                                                    __builtin_amdgcn_mbcnt_lo(uint32_t(entering), 0u));
    uint32_t next = 0;
    if (rank == 0) next = lds_add(ids_at, uint32_t(__popcll(entering)));
    uint32_t own = uint32_t(__builtin_amdgcn_readfirstlane(int(next))) + rank;
    if (__builtin_expect(own >= capacity, 0)) {
      own = id_given_back();
      if (own >= capacity) return false;
    }
    *lds<uint64_t>(a.off_tokens + 8u * own) = x.rest;
    *lds<uint32_t>(a.off_lead + 4u * own) = x.t0;
    asm volatile("" ::: "memory");  // (a wavefront's LDS accesses happen in their order)
    // (the slots from the first one that was free on are looked at one by one, so that what has been entered
    // since is seen)
    s += first_free_slot(e.x, e.y, e.z);
    while (true) {
      const uint32_t old = lds_cas<uint32_t>(s, mine + own);
      if (old == 0u) {
        is_new = true;
        id = own;
        found = x;
        break;
      }
      id = old ^ mine;
      if (id < id_limit) {
        found = load_item(id);
        if (same(found, x, n)) break;
      }
      s = (s + 4u) & (bucket_mask | 12u);
    }
    *lds<uint32_t>(a.off_lead + 4u * own) = is_new ? x.t0 : kGivenBack;  // (a branch: 2 % of the call)
    return true;
  }
  __device__ __forceinline__ void do_item(uint64_t rest, uint32_t lead, int f) {
    const uint32_t times = (lead >> kTokenBits) + 1u;
    const Item x{lead & kNoToken, rest};
    const uint32_t h = item_hash(x);
    Item found;
    uint32_t id;
    bool is_new;
    if (!resolve(x, h, 3, f, id, found, is_new)) return;
    // (one that is new at order 3 is new at order 4, too)
    if (f == 0 && is_new && times == 1u && !ALL) return;
    count(table_bytes + 4u * id, times, f, is_new, matches);
    // (behind the end there is no fourth token)
    if (N < 4 || last_of(x) == kNoToken) return;
    if (last_of(x) != last_of(found) && !resolve(x, hash4(h, last_of(x)), 4, f, id, found, is_new)) return;
    count(counters4 + 4u * id, times, f, is_new, matches4);
  }

  // The candidate's members, or the references'; m: the wavefront's first block.
  __device__ __forceinline__ void side(bool cand, Member m) {
    const uint32_t marks = cand ? cand_marks : ref_marks;
    int begin = cand ? 0 : cand_members;
    const int end = cand ? cand_members : members;
#pragma unroll 1
    while (true) {
      const int size = min(end - begin, window);
#pragma unroll 1
      for (int block = wave; block * kWave < size; block += kWaves) {
        const Member now = m;
        if ((block + kWaves) * kWave < size) m = fetch(marks, begin, size, block + kWaves, cand);
        const int f = cand ? 0 : ONE ? 1 : now.f;
        if (block * kWave + lane < size) {
          if (KIND == 2) do_item(now.key, now.word, f);
          if (KIND == 1) do_pair(now.key, f);
          if (KIND == 0) do_first(now.word, f);
        }
      }
      begin += window;
      if (begin >= end) break;
      const int next = min(end - begin, window);
      __syncthreads();
      if (KIND == 2 && lds_peek(again_at)) break;  // uniform: what is counted is of no use
      mark(marks, begin, next);
      __syncthreads();
      if (wave * kWave < next) m = fetch(marks, begin, next, wave, cand);
    }
  }
  // The candidate's n-grams clipped; `there`: the entries (of which every occurrence is counted).
  __device__ __forceinline__ uint32_t sweep(uint32_t at, uint32_t& there) const {
    uint32_t part = 0;
    for (uint32_t k = at + 4u * uint32_t(tid); k < at + slots_bytes; k += 4u * kTallyThreads) {
      const uint32_t head = *lds<uint32_t>(k);
      const uint32_t of_cand = (HALVES ? head & 0xFFFFu : head) + (ALL ? 0u : 1u);
      uint32_t most = HALVES ? head >> 16 : 0u;
      for (int w = 1; w < a.words; ++w) {
        const uint32_t word = *lds<uint32_t>(k + uint32_t(w) * slots_bytes);
        most = max(most, HALVES ? max(word & 0xFFFFu, word >> 16) : word);
      }
      part += min(of_cand, most);
      if (ALL) there += (of_cand | most) != 0u ? 1u : 0u;
    }
    return part;
  }
  __device__ __forceinline__ void add_to(uint32_t at, uint32_t part) const {
    const int sum = wave_sum(int(part));
    if (lane == 0 && sum) lds_add_only(at, uint32_t(sum));
  }
  // Order n's sums, of the counters at `at` or as matched.
  __device__ __forceinline__ void add_up(int n, uint32_t at, uint32_t matched) const {
    uint32_t there = 0;
    add_to(lost_at + 12u + 4u * uint32_t(n), ONE ? matched : sweep(at, there));
    if (ALL) add_to(lost_at + 28u + 4u * uint32_t(n), there);
  }
  __device__ __forceinline__ uint32_t report_loss() const {
    const uint32_t lost = *lds<uint32_t>(lost_at);  // uniform
    if (tid == 0 && lost) {
      if (a.pb.status) atomicOr(a.pb.status, TB_DEV_TABLE_OVERFLOW);
      a.overflow[g] = 1;
    }
    return lost;
  }
  // (wavefront 0) The partition's sums, from LDS; of a share of order 4 (not `own`): that order's.
  // The last partition (or share of one) of an order to arrive writes the order's statistics, and the last of these
  // scores the sentence: one round trip to memory for a workgroup, three for the last one, where a kernel of its own
  // took 3.5 us.  Everything that passes between workgroups goes through atomics whose answers are awaited.
  __device__ __forceinline__ void arrive(uint32_t lost, bool own) const {
    const Problem& pb = a.pb;
    const int n0 = KIND + lane;  // order n0 + 1
    const int64_t stat = int64_t(g) * N + n0;
    bool last = false;
    if (lane < (KIND == 2 ? 2 : 1) && n0 < N && (own || n0 == 3)) {
      if (ALL) atomicAdd(&a.st.distinct[stat], int(*lds<uint32_t>(lost_at + 32u + 4u * uint32_t(n0))));
      const unsigned long long add = *lds<uint32_t>(lost_at + 16u + 4u * uint32_t(n0)) | 1ull << 24 | (lost ? 1ull << 52 : 0ull);
      const unsigned long long all = add + __hip_atomic_fetch_add(&a.arrived[stat], add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t shares = uint32_t(all >> 40) & 0xFFFu;  // (of order 4)
      if (KIND == 2 && shares) *lds<uint32_t>(called_at()) = 1u;
      if ((uint32_t(all >> 24) & 0xFFFFu) == parts + shares) {
        const int len = clamped_len(uniform_load(pb.cand_len, g), pb.cand_stride, nullptr);
        a.st.clipped[stat] = int32_t(all & 0xFFFFFFull);
        a.st.total[stat] = max(len - n0, 0);
        if (a.out)
          last = __hip_atomic_fetch_add(&a.complete[g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == N - 1;
      }
    }
    if (!__builtin_amdgcn_ballot_w64(last)) return;  // uniform
    unsigned long long all = 0;
    if (lane < N) all = __hip_atomic_load(&a.arrived[int64_t(g) * N + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int c = clamped_len(uniform_load(pb.cand_len, g), pb.cand_stride, pb.status);
    const RefRows rows = ref_rows(pb, g, true);
    const int r = closest_ref_len(c, pb.ref_len + rows.row0, rows.used, pb.ref_stride, pb.status);
    const float brevity = expf(1.0f - float(r) / float(c));
    const float score = bleu_from_stats_wave<int>(int(all & 0xFFFFFFull), max(c - lane, 0), c, r, brevity, lane_weight(a.sp), a.sp);
    const bool spoilt = __builtin_amdgcn_ballot_w64(all >> 52 != 0) != 0;
    if (lane == 0) {
      a.st.closest[g] = r;
      store_score(a.out, g, spoilt ? __int_as_float(0x7FC00000) : score, a.sp.out_bf16);
    }
  }

  // ---- 4-grams where ids run out (see tally_crowd).
  // LDS words: whether there are shares of crowded partitions to be taken; and for what is passed on to all threads.
  __device__ __forceinline__ uint32_t called_at() const { return lost_at + 48u; }
  __device__ __forceinline__ uint32_t told_at() const { return lost_at + 52u; }
  // Members that take up ids.
  __device__ __forceinline__ uint32_t entries() const { return uint32_t(ALL ? members : cand_members); }

  // One order on its own: n-grams whose hash falls into the share, in `pieces` rounds, and in more of them where one
  // has too many all the same.  Each wavefront takes a sixteenth of the members, one behind the other, whose runs then
  // need no search.  It requests several blocks at a time (most of the time is the way from memory) and puts those
  // members that are the share's together to full blocks, which are then entered or looked up.
  __device__ __forceinline__ void count_alone(int n, uint32_t index, uint32_t of, uint32_t pieces) {
    constexpr int kAhead = 4;
    constexpr uint64_t kTokens = (1ull << (3 * kTokenBits)) - 1ull;
    const uint32_t first_pieces = pieces;
    auto hash_of = [&](const Item& x) { return n == 3 ? item_hash(x) : hash4(item_hash(x), last_of(x)); };
    auto move = [&](int place, uint32_t v) { return uint32_t(__builtin_amdgcn_ds_permute(place << 2, int(v))); };
#pragma unroll 1
    for (uint32_t done = 0; done < pieces;) {
      __syncthreads();
      clear(0, counters4);
      clear(a.off_lead, cand_marks);
      if (tid == 0) *lds<uint32_t>(ids_at) = 0u, *lds<uint32_t>(again_at) = 0u;
      matches = 0;
      const uint32_t all = of * pieces, mine = index * pieces + done;
      // (in the end one lane of a wavefront after the other: sixteen ids at most are then taken in vain)
      const int turns = pieces < 16u * first_pieces ? 1 : kWave;
#pragma unroll 1
      for (int refs = 0; refs < 2; ++refs) {
        const int begin = refs ? cand_members : 0, end = refs ? members : cand_members;
        const int blocks = (end - begin + kWave - 1) / kWave;
        int at = begin + wave * blocks / kWaves * kWave;  // (uniform)
        const int stop = min(begin + (wave + 1) * blocks / kWaves * kWave, end);
        int run = 0;
        if (at < stop) {
#pragma unroll 1
          for (int step = kMaxDealChunks / 2; step; step /= 2)
            if (run + step < a.chunks && *before_of(run + step) <= min(at + lane, stop - 1)) run += step;
        }
        // An n-gram that many lanes have met: what a lane sees of it is added up in a register first.
        uint32_t often0 = ~0u, often1 = 0, often2 = 0;  // its tokens
        uint32_t often_at = 0, times_often = 0;
        int f = 0;
        // Lanes 0 .. pending - 1: members to be entered or looked up (the sequence from bit 60 of the key on).
        uint64_t key = 0;
        uint32_t word = 0;
        int pending = 0;
        __syncthreads();
        uint64_t next_key[kAhead];
        uint32_t next_word[kAhead];
        int loaded = 0;
#pragma unroll 1
        while (at < stop || pending > 0) {
          uint64_t more_key = 0;
          uint32_t more_word = 0;
          if (at < stop) {
            if (loaded == 0) {
#pragma unroll
              for (int k = 0; k < kAhead; ++k) {
                const int i = min(at + k * kWave + lane, stop - 1);
#pragma unroll 1
                while (run + 1 < a.chunks && *before_of(run + 1) <= i) ++run;
                const Member m = load(i, run, refs == 0);
                next_key[k] = m.key | uint64_t(m.f) << (3 * kTokenBits);
                next_word[k] = m.word;
              }
              loaded = kAhead;
            }
            bool counts = at + lane < stop;
            const uint64_t own = next_key[0];
            const uint32_t own_word = next_word[0];
            --loaded;
            at += kWave;
#pragma unroll
            for (int k = 0; k + 1 < kAhead; ++k) next_key[k] = next_key[k + 1], next_word[k] = next_word[k + 1];
            const Item x{own_word & kNoToken, own & kTokens};
            const int of_seq = refs ? ONE ? 1 : int(own >> (3 * kTokenBits)) : 0;
            if (times_often && of_seq != f) {
              count(often_at, times_often, f, false, matches);
              times_often = 0;
            }
            f = of_seq;
            if (n == 4) {
              counts &= last_of(x) != kNoToken;
            } else if (counts && same(x, Item{often0, uint64_t(often2) << 32 | often1}, 3)) {
              times_often += (own_word >> kTokenBits) + 1u;
              counts = false;
            }
            if (all > 1u) counts &= __umulhi(hash_of(x) * 0x9E3779B1u, all) == mine;
            const uint64_t going = __builtin_amdgcn_ballot_w64(counts);
            if (going) {
              // Lanes that have one move it behind those waiting, the others theirs behind these (a permutation).
              const int rank = int(__builtin_amdgcn_mbcnt_hi(uint32_t(going >> 32),
                                                             __builtin_amdgcn_mbcnt_lo(uint32_t(going), 0u)));
              const int place = pending + (counts ? rank : __popcll(going) + lane - rank);
              more_key = uint64_t(move(place, uint32_t(own >> 32))) << 32 | move(place, uint32_t(own));
              more_word = move(place, own_word);
              if (lane >= pending) key = more_key, word = more_word;
              pending += __popcll(going);
            }
            if (pending < kWave && at < stop) continue;
          }
          const bool counts = lane < pending;
          const Item x{word & kNoToken, key & kTokens};
          const uint32_t times = (word >> kTokenBits) + 1u;
          const int seq = refs ? ONE ? 1 : int(key >> (3 * kTokenBits)) : 0;
          const uint32_t h = hash_of(x);
          key = more_key, word = more_word;  // (lanes 0 .. pending - 65)
          pending = max(pending - kWave, 0);
#pragma unroll 1
          for (int turn = 0; turn < turns; ++turn) {
            bool there = false, is_new;
            uint32_t id = 0;
            if (counts && (turns == 1 || turn == lane)) {
              Item found;
              there = resolve(x, h, n, seq, id, found, is_new);
              if (there) count(table_bytes + 4u * id, times, seq, is_new, matches);
            }
            if (n == 3) {
              const uint64_t have = __builtin_amdgcn_ballot_w64(there);
              if (!have) continue;
              const int first = __ffsll((unsigned long long)have) - 1;
              const uint32_t first_id = uint32_t(__builtin_amdgcn_readlane(int(id), first));
              if (__popcll(__builtin_amdgcn_ballot_w64(there && id == first_id)) < kWave / 4) continue;
              if (times_often) count(often_at, times_often, f, false, matches);
              times_often = 0;
              often_at = table_bytes + 4u * first_id;
              const Item often = load_item(first_id);
              often0 = uint32_t(__builtin_amdgcn_readfirstlane(int(often.t0)));
              often1 = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(often.rest))));
              often2 = uint32_t(__builtin_amdgcn_readfirstlane(int(often.rest >> 32)));
            }
          }
        }
        if (times_often) count(often_at, times_often, f, false, matches);
      }
      __syncthreads();
      if (!*lds<uint32_t>(again_at)) {  // uniform
        add_up(n, table_bytes, matches);
        ++done;
      } else if (pieces < first_pieces << 8) {
        pieces *= 2;
        done *= 2;
      } else {
        if (tid == 0) *lds<uint32_t>(lost_at) = 1u;
        break;
      }
    }
  }
};

// What is left to do where ids ran out.  Many different 4-grams with the same first three tokens crowd a partition: a
// twentieth of a text of 262 144 tokens behind one beginning are 13 000 ids, where a partition has 1900.  The workgroup
// of such a partition (`own`) counts order 3 on its own, where they are one n-gram, and divides order 4 into shares by
// the hash of all four tokens.  Of more than kAlone it makes them known before it arrives, and every workgroup of the
// group's 4-grams that sees with its own arrival that there are some takes shares until none is left.  Nobody waits for
// another one: who makes shares known takes what is left of them.
//
// Measured (us a call; one text of 262 144 tokens, so much of it behind one beginning with another token behind it each
// time; the partition's workgroup counting in rounds -> this; the sorted runs take 40): 0.5 % 243 -> 79, 1 % 342 -> 96,
// 5 % 1940 -> 69, an eighth 7780 -> 92, a quarter 22 960 -> 123; 50 texts of 20 000, a quarter 740 -> 102 (84).  A pass
// over few members is a chain of latencies, the first one with instructions that no other workgroup has brought along.
// Told of at the start by the dealing kernel, or by the number of members, shares come earlier (0.5 % 49), but either
// took the usual texts 1 to 3 %, or texts of few different tokens with as many members for crowded ones.
template <Counters COUNTERS>
__device__ __forceinline__ void tally_crowd(int p, int members, int cand_members, bool own) {
  typedef Tally<2, COUNTERS> T;
  if (own) {
    uint32_t pieces;
    {
      T t(arguments());
      t.members = members;
      t.cand_members = cand_members;
      pieces = 1u + __umulhi(t.entries(), t.a.per_member);
      if (t.N > 3 && pieces > kAlone) {
        __syncthreads();
        if (t.tid == 0) {
          const int e = __hip_atomic_fetch_add(&t.a.crowds[t.g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (e < kCrowds) {
            // (answers awaited: known before it is counted, counted before the partition arrives)
            const int was = __hip_atomic_exchange(&t.a.crowd[t.g * kCrowds + e], p << 16 | int(pieces), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long add = (unsigned long long)(pieces + uint32_t(was)) << 40;  // (it was 0)
            const unsigned long long before = __hip_atomic_fetch_add(&t.a.arrived[int64_t(t.g) * t.N + 3], add,
                                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lds<uint32_t>(t.called_at()) = uint32_t((before + add) >> 40);
          }
          *lds<int>(t.told_at()) = e;
        }
        __syncthreads();
        if (*lds<int>(t.told_at()) < kCrowds) pieces = 0;  // uniform
      }
      t.count_alone(3, 0u, 1u, 1u);
    }
    if (pieces && arguments().pb.N > 3) {  // (more crowded partitions than can be told of)
      T t(arguments());
      t.members = members;
      t.cand_members = cand_members;
      t.count_alone(4, 0u, 1u, pieces);
    }
    const T t(arguments());
    __syncthreads();
    const uint32_t lost = t.report_loss();
    if (t.wave == 0) t.arrive(lost, true);
    __syncthreads();
    if (!*lds<uint32_t>(t.called_at())) return;  // uniform
  }
#pragma unroll 1
  for (int e = 0; e < kCrowds;) {
    T t(arguments());
    __syncthreads();
    if (t.tid == 0) {  // (one thread looks: another one might see something else already)
      const int crowds = __hip_atomic_load(&t.a.crowds[t.g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int crowd = __hip_atomic_load(&t.a.crowd[t.g * kCrowds + e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int share = e < crowds ? 0xFFFF : -1;  // (not told of yet: its own workgroup comes to it; none)
      if (crowd) share = __hip_atomic_fetch_add(&t.a.next_share[t.g * kCrowds + e], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *lds<int>(t.told_at()) = crowd;
      *lds<int>(t.told_at() + 4u) = share;
      *lds<uint32_t>(t.lost_at) = *lds<uint32_t>(t.lost_at + 28u) = *lds<uint32_t>(t.lost_at + 44u) = 0u;
    }
    __syncthreads();
    const int crowd = __builtin_amdgcn_readfirstlane(*lds<int>(t.told_at()));
    const int share = __builtin_amdgcn_readfirstlane(*lds<int>(t.told_at() + 4u));
    if (share < 0) return;
    if (share >= (crowd & 0xFFFF)) {
      ++e;
      continue;
    }
    t.gather(t.load_place(crowd >> 16));
    __syncthreads();
    t.cand_members = __builtin_amdgcn_readfirstlane(*t.scratch(16));
    t.count_alone(4, uint32_t(share), uint32_t(crowd & 0xFFFF), 1u);
    __syncthreads();
    const uint32_t lost = t.report_loss();
    if (t.wave == 0) t.arrive(lost, false);
  }
}

// One partition's members of one kind.
template <int KIND, Counters COUNTERS>
__device__ __forceinline__ void tally_kind(const DealArgs& a, int p) {
  typedef Tally<KIND, COUNTERS> T;
  typedef typename T::Member Member;
  constexpr bool ONE = T::ONE, HALVES = T::HALVES;
  T t(a);
  const uint32_t place = t.load_place(p);
  t.clear(0, t.used_bytes);
  t.clear(KIND < 2 ? t.cand_marks : a.off_lead, t.cand_marks + 4u * uint32_t(t.window));  // (no id is given back yet)
  t.clear(a.off_sums, a.off_places);
  t.gather(place);
  __syncthreads();
  t.cand_members = __builtin_amdgcn_readfirstlane(*t.scratch(16));
  t.mark(t.cand_marks, 0, min(t.cand_members, t.window));
  t.mark(t.ref_marks, t.cand_members, min(t.members - t.cand_members, t.window));
  __syncthreads();
  // (of so many members ids run out: not tried first)
  bool counted = KIND < 2 || 2u * t.entries() <= 5u * t.capacity;  // uniform
  if (counted) {
    Member m{0, 0, 0}, later{0, 0, 0};
    const int cand_size = min(t.cand_members, t.window), refs_size = min(t.members - t.cand_members, t.window);
    if (t.wave * kWave < cand_size) m = t.fetch(t.cand_marks, 0, cand_size, t.wave, true);
    // (on their way while the candidate's are entered)
    if (t.wave * kWave < refs_size) later = t.fetch(t.ref_marks, t.cand_members, refs_size, t.wave, false);
    t.side(true, m);
    __syncthreads();
    // (uniform: only what is entered can set it; with ALL the references' n-grams are, too)
    if (KIND == 2 && !T::ALL) counted = !lds_peek(t.again_at);
    if (counted) {
      t.side(false, later);
      __syncthreads();
      if (KIND == 2 && T::ALL) counted = !lds_peek(t.again_at);  // uniform
    }
  }
  if (counted) {
    const bool rouge = KIND < 2 && a.rouge_overlap;  // uniform
    const uint32_t overlaps_at = t.lost_at + 64u;
    if (rouge && !ONE) {  // the overlap with each reference
      for (int f = 1; f <= a.pb.R; ++f) {
        uint32_t part = 0;
        for (uint32_t k = t.table_bytes + 4u * uint32_t(t.tid); k < t.table_bytes + t.slots_bytes; k += 4u * kTallyThreads) {
          const uint32_t head = *lds<uint32_t>(k), word = *lds<uint32_t>(k + uint32_t(HALVES ? f >> 1 : f) * t.slots_bytes);
          part += HALVES ? min((head & 0xFFFFu) + 1u, f & 1 ? word >> 16 : word & 0xFFFFu) : min(head + 1u, word);
        }
        t.add_to(overlaps_at + 4u * uint32_t(f), part);
      }
    }
    if (ONE || !rouge) t.add_up(KIND + 1, t.table_bytes, t.matches);
    if (KIND == 2 && t.N > 3) t.add_up(4, t.counters4, t.matches4);
    __syncthreads();
    const uint32_t lost = t.report_loss();
    if (rouge) {
      const uint32_t at = ONE ? t.lost_at + 16u + 4u * uint32_t(KIND) : overlaps_at + 4u * uint32_t(t.tid + 1);
      if (t.tid < a.pb.R && *lds<uint32_t>(at))
        atomicAdd(&a.rouge_overlap[int64_t(t.g) * a.pb.R + t.tid], int(*lds<uint32_t>(at)));
      return;
    }
    if (t.wave == 0) t.arrive(lost, true);
    if (KIND < 2 || t.N < 4) return;
    __syncthreads();
    if (!*lds<uint32_t>(t.called_at())) return;  // uniform
  }
  if constexpr (KIND == 2) tally_crowd<COUNTERS>(p, t.members, t.cand_members, !counted);
}
template <Counters COUNTERS>
__global__ __launch_bounds__(kTallyThreads, 8) void tally_kernel(DealArgs by_value) {
  const DealArgs& a = arguments();
  int p = blockIdx.x;  // (the kind with the most work first)
  if (a.kinds > 2) {
    if (p < a.parts[2]) return tally_kind<2, COUNTERS>(a, p);
    p -= a.parts[2];
  }
  if (a.kinds > 1) {
    if (p < a.parts[1]) return tally_kind<1, COUNTERS>(a, p);
    p -= a.parts[1];
  }
  tally_kind<0, COUNTERS>(a, p);
}

int log2_ceil(int64_t v) {
  int b = 0;
  while ((int64_t(1) << b) < v) ++b;
  return b;
}

// Whether a table of `slots` holds what a hash sends to it of its binomial share (see has_room in tb_runs.hip:
// less likely than exp(-40) not to).
bool deal_has_room(int64_t share, int64_t slots) {
  const double mean = double(share), k = double(slots);
  return mean < k && k - mean - k * std::log(k / mean) <= -40.0;
}

template <int ITEMS>
hipError_t launch_items(const DealArgs& a, const DealPlan& plan, hipStream_t s) {
  hipLaunchKernelGGL(deal_kernel<ITEMS>, dim3(a.chunks, a.pb.B), dim3(kThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto tally = [&](auto kernel) {
    e = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), plan.lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(a.all_parts, a.pb.B), dim3(kTallyThreads), plan.lds_bytes, s, a);
    return hipGetLastError();
  };
  if (plan.all) return plan.halves ? tally(tally_kernel<kAllHalves>) : tally(tally_kernel<kAllWords>);
  return a.pb.R == 1 ? tally(tally_kernel<kOneReference>)
         : plan.halves ? tally(tally_kernel<kHalves>) : tally(tally_kernel<kWords>);
}

}  // namespace

// What the choice of the shares weighs (14 shapes of one to three references, all shares; us a call):
//   * A workgroup's start (its runs' places, clearing, marks) costs as much as some 500 members, so shares are as
//     large as the LDS of two workgroups a unit allows: one reference, 50 groups of two times 20 000, shares of
//     320, 640 and 1280 4-grams 99.9, 71.5 and 61.5; 11 groups of 180 000 120.9, 71.3 and 62.8.
//   * Where the chip is not full, smaller ones down to that: 16 groups of two times 8192 640 4-grams 21.3, 1280
//     22.7; one text of 30 000 480 16.5, 1280 18.8, 160 20.
//   * A share of the candidate brings one of each reference with it.  9 groups of 25 236 with three references of
//     27 025: 480 4-grams 42.8, 1280 49.5, 320 50.0.
//   * A 4-gram costs 1.6 times a pair, and a token, of which most are merged, half as much.  With more references,
//     whose counters need more LDS, the table of tokens is the first that does not fit: smaller shares of them
//     leave the others larger ones (19 groups of 20 809 with two references of 20 000 54.4 -> 51.4, two orders 38.8 ->
//     34.0).
//   * Tables of tokens and pairs at most half full: a wavefront probes as long as its unluckiest lane.  With up to
//     two thirds, 22 groups of two times 17 000, two orders, 28.4 instead of 24.0, 4 of two times 50 000 29.3 instead
//     of 26.9.
//   * Where the partitions do not fit one round of 512 workgroups at that, shares grow as far as the LDS of two of them a
//     unit lets them, up to 48 / (1 + R) steps.  It was 32, which left a third of the LDS unused with three references:
//     of 89 shapes whose shares that changes 0.95 of the time on average (three references 0.93, two 0.99, the worst of
//     all 1.08; 41 groups of 10 622 with three references of 12 054, two orders, 49.6 -> 45.0, 27 of 7687 with three
//     of 8643 46.0 -> 38.5, 33 of 10 083 with one of 9617 35.6 -> 29.8).
bool plan_deal(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int32_t vocab, bool rouge,
               bool group_distinct, DealPlan* plan) {
  DealPlan& p = *plan;
  const int64_t cap = cand_stride + R * ref_stride;
  if (N > (rouge ? 2 : 4) || R >= kWave || B > 65535 || vocab >= int32_t(kNoToken)) return false;
  p.kinds = N < 3 ? N : 3;
  p.first_kind = rouge ? N - 1 : 0;
  p.all = group_distinct;
  p.halves = cand_stride <= 65535 && ref_stride <= 65535;
  p.window[0] = p.window[1] = p.window[2] = kWave;
  p.words = R == 1 && !p.all ? 1 : p.halves ? (R + 2) / 2 : 1 + R;
  p.items = B * cap < 256 * 2 * kThreads ? 1 : 2;  // (one workgroup for every compute unit)
  auto split = [&] {
    const int64_t chunk = p.items * kThreads;
    p.cand_chunks = int((cand_stride + chunk - 1) / chunk);
    p.ref_chunks = int((ref_stride + chunk - 1) / chunk);
    return p.cand_chunks + int64_t(R) * p.ref_chunks;
  };
  if (cap > int64_t(2) * kThreads * kMaxDealChunks) return false;
  if (split() > kMaxDealChunks) p.items = 2;
  const int64_t chunks = split();
  if (chunks > kMaxDealChunks) return false;
  p.chunks = int(chunks);

  // shares: positions whose n-grams are entered, as a partition of each kind may expect them
  const int64_t entries = p.all ? cap : cand_stride;
  auto fits = [&](int scale) {
    int64_t share[kKinds] = {(R == 1 ? 256 : 192) * scale, 128 * scale, 80 * scale};
    int log2_slots[kKinds];
    p.all_parts = 0;
    for (int kind = 0; kind < kKinds; ++kind) {
      int64_t parts = (entries + share[kind] - 1) / share[kind];
      if (parts < 2) parts = 2;
      share[kind] = (entries + parts - 1) / parts;
      const bool used = kind >= p.first_kind && kind < p.kinds;
      p.parts[kind] = int(used ? parts : 1);
      p.parts_before[kind] = used ? p.all_parts : 0;
      if (used) p.all_parts += int(parts);
      log2_slots[kind] = log2_ceil(2 * share[kind]);
      while (!deal_has_room(share[kind], int64_t(1) << log2_slots[kind])) ++log2_slots[kind];
    }
    // ids: the most frequent three tokens of a Zipf-distributed text start one of 370 of its 4-grams
    p.capacity = int((share[2] + share[2] / 4 + entries / 512 + 128 + 7) & ~int64_t(7));
    p.id_bits = log2_ceil(p.capacity);
    p.log2_first = log2_slots[0];
    p.log2_pair = log2_slots[1];
    p.log2_item = log2_ceil(2 * share[2]);
    while ((int64_t(3) << p.log2_item) < 4 * int64_t(p.capacity)) ++p.log2_item;
    const uint32_t ids = uint32_t(p.capacity), counter = 4u * uint32_t(p.words);
    p.off_tokens = ((4u << p.log2_item) + counter * ids * (N > 3 ? 2u : 1u) + 15u) & ~15u;
    p.off_lead = p.off_tokens + 8u * ids;
    const uint32_t tables[kKinds] = {(4u + counter) << p.log2_first, (8u + counter) << p.log2_pair,
                                     (p.off_lead + 4u * ids + 15u) & ~15u};
    // marks: of pairs for a quarter more than the share, of 4-grams for as many (a partition may have a frequent
    // beginning), of tokens, of which most are merged, for three quarters
    p.off_sums = 0;
    for (int kind = p.first_kind; kind < p.kinds; ++kind) {
      p.window[kind] = int((kind ? 5 * share[1] : 3 * share[0]) / 4 + 127) & ~(kWave - 1);
      const uint32_t end = tables[kind] + 4u * uint32_t(p.window[kind]);
      if (p.off_sums < end) p.off_sums = end;
    }
    p.off_places = p.off_sums + 64 + (rouge ? 4 * kWave : 0);
    p.off_scratch = p.off_places + 4u * uint32_t(3 * p.chunks);
    p.lds_bytes = p.off_scratch + 4 * 17;
    return p.all_parts <= kMaxParts && chunks * p.all_parts <= (p.kinds - p.first_kind) * cap;
  };
  const int most = 48 / (1 + R) < 2 ? 2 : 48 / (1 + R), least = (12 + R) / (1 + R) < 2 ? 2 : (12 + R) / (1 + R);
  int scale = 0;
  for (int s = 1; s <= most; ++s) {
    if (!fits(s)) continue;
    if (p.lds_bytes > size_t(kLdsBudget) / 2 / 1280 * 1280) break;
    scale = s;
    if (s >= least && B * p.all_parts <= 512) break;
  }
  return scale > 0 && fits(scale);
}

hipError_t launch_deal(const Problem& pb, const DealPlan& plan, const RunsBuffers& buffers, const StatPtrs& st,
                       const ScoreParams& sp, void* out_bleu_or_null, int32_t* rouge_overlap, hipStream_t s) {
  DealArgs a;
  a.pb = pb;
  a.st = st;
  const size_t n = size_t(pb.B) * size_t(pb.group_cap);
  uint64_t* at = buffers.keys;  // N * n of them
  a.pair = at;
  if (pb.N > 1) at += n;
  a.rest = at;
  if (pb.N > 2) at += n;
  a.first = reinterpret_cast<uint32_t*>(at);
  a.lead = a.first + n;
  a.run_at = buffers.places;
  a.overflow = buffers.overflow;
  a.rouge_overlap = rouge_overlap;
  a.arrived = reinterpret_cast<unsigned long long*>(buffers.times);  // (N * n words there)
  a.complete = reinterpret_cast<int32_t*>(a.arrived + size_t(pb.B) * pb.N);
  a.crowds = a.complete + pb.B;
  a.crowd = a.crowds + pb.B;  // (a group has more than 12 288 slots)
  a.next_share = a.crowd + size_t(pb.B) * kCrowds;
  a.per_member = uint32_t((int64_t(20) << 32) / (17 * int64_t(plan.capacity)));
  a.sp = sp;
  a.out = out_bleu_or_null;
  a.first_kind = plan.first_kind;
  a.kinds = plan.kinds;
  a.all_parts = plan.all_parts;
  for (int kind = 0; kind < kKinds; ++kind) {
    a.window[kind] = plan.window[kind];
    a.parts[kind] = plan.parts[kind];
    a.parts_before[kind] = plan.parts_before[kind];
  }
  a.log2_chunk = plan.items == 2 ? 11 : 10;
  a.cand_chunks = plan.cand_chunks;
  a.ref_chunks = plan.ref_chunks;
  a.chunks = plan.chunks;
  a.words = plan.words;
  a.capacity = plan.capacity;
  a.id_bits = plan.id_bits;
  a.log2_first = plan.log2_first;
  a.log2_pair = plan.log2_pair;
  a.log2_item = plan.log2_item;
  a.off_tokens = plan.off_tokens;
  a.off_lead = plan.off_lead;
  a.off_sums = plan.off_sums;
  a.off_places = plan.off_places;
  a.off_scratch = plan.off_scratch;
  return plan.items == 2 ? launch_items<2>(a, plan, s) : launch_items<1>(a, plan, s);
}

}  // namespace tb
