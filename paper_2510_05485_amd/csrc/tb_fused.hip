// FUSED kernel: the whole per-sentence pipeline for one sentence group in one workgroup.
//
// Tokens are read from HBM once; dictionary and counters never leave LDS; one score (plus optional
// integer statistics) goes out.  What bounds it: instruction issue.  A lone small group pays seven or
// eight cycles per instruction of its longest wavefront.  A full chip issues, per cycle and compute unit,
// 0.73 vector and 0.48 scalar instructions (512 x 1024 with four references), 0.83 and 0.59 (1024 x 2048),
// 0.71 and 0.54 (4096 x 512 with two): 71 to 84 % of the 1.7 that a mix of both kinds reaches at most
// (counters of rocprofv3; 1.5 of vector instructions alone, 1.0 of scalar ones), the scalar ones from
// loops, masks and bookkeeping.  LDS is not the limit (0.07 to 0.09 instructions; a random 16-byte read
// takes 12.5 cycles per wavefront, a 4-byte one 6.5, a compare-and-swap 12).  So:
//   * Symbols.  Order 1 turns every token into the candidate position that holds its first
//     occurrence there (its "symbol"), or into "absent" (-1).  An n-gram of order n >= 2 is then
//     named by (id of the (n-1)-gram that starts at the same position, symbol of its last token):
//     at most 2 * log2(candidate stride) bits whatever n and the vocabulary are.  Once the symbols
//     of all positions are in LDS, a thread walks all orders of its positions on its own: a
//     candidate position enters its n-grams one order after the other (an id is known as soon as
//     the entry is), a reference position looks its n-grams up until one is absent (a candidate
//     n-gram extends only prefixes the candidate contains).  No barrier lies between the orders.
//   * Implied n-grams.  An id is the candidate position of one occurrence.  The n-gram that goes on
//     like the candidate does there (the prefix's id p, then the symbol at p + n - 1) takes the same id
//     without an entry; only other continuations are entered and looked up.  Every (n-1)-gram but the
//     candidate's last has one implied continuation, so the entries of orders lo..hi are at most the
//     distinct n-grams of order hi less those of order lo - 1, plus one an order: never more than
//     candidate positions, where four orders used to enter up to four times as many.  Tables take a
//     quarter of the room or fill a quarter as far, from order 3 on few lanes enter anything at all
//     (1024 x 2048 43.8 -> 35.7 us, 128 x 8192 46.5 -> 37.5, 4096 x 2048 with two references 143 -> 127).
//   * Entries that carry the id.  A table entry is one 32-bit word (remainder | probe count | id).
//     The key is multiplied by an odd constant modulo 2^key_bits (a bijection); the top bits of the
//     product pick the home bucket and the remaining bits are stored.  Bucket and probe count give
//     back the home bucket (the probe step depends on the remainder only), so (bucket, remainder,
//     probe count) identifies the key exactly, and one LDS read answers both "is it this key" and
//     "what is its id": no second array and no second dependent read.
//   * Buckets of four slots, filled front to back.  A look-up reads a bucket with one request and
//     is straight-line code: only a full bucket without the key makes it go on.
//   * A group's positions are dealt to the wavefronts in blocks of 64 that lie in one sequence, so
//     sequence, row, counter word and addend of a block are scalars.
//   * The orders of a pass put their number into the key and share one table, each with counters of
//     its own.  How many orders that are is the plan's choice: all of them (fewest barriers), or
//     fewer where LDS is short (table and counters are then swept and cleared in between).
//
// Counters: 16-bit fields per candidate id and reference (the offset of Section 3.3 step 1 keeps
// sequences apart the same way).  With one reference, and for ROUGE-N, a look-up sees by the counter it
// decreases whether the candidate has the n-gram once more (step 3's minimum); with more, a pass over
// the counters takes the maximum over the references.  Wavefront 0 forms brevity penalty, smoothing and
// geometric mean (Section 3.4), one order per lane.  Mode kRouge scores ROUGE-N for n = N.
//
// Measured on gfx950 (us of GPU time, 4 orders; in brackets the kernel that counted first occurrences and did not
// put together what is left of blocks, the one that entered every n-gram and swept its counters, and the one
// before that, with a barrier per insertion and look-up of each order): 16 x 256 tokens with one reference 5.9
// (6.0, 6.7, 9.5), 256 x 1088 8.0 (8.3, 9.4, 12.8), 512 x 1024 with four references 17.0 (17.5, 19.8, 22.8), 4096 x
// 512 with two and the batch's sums 30.3 (32.0, 47.7, 50.5), 4096 x 2048 with two 95 (102, 145, 171), 1000 x 96 with
// up to eight 10.1 (10.3, 10.5, 13.7), ROUGE-2 of 512 x 512 with three 6.9 (7.1, 9.6, 12.5; 7.2 on
// one kernel with the other orders); 128 x 5000 with one 18.9 (21.7, 28.5; 55 on three staged kernels), 128 x 8192 27.5
// (31.2, 46.6; 98 on the partitioned ones).
#include <type_traits>

#include "tb_kernels.h"
#include "tb_score.h"

// Phase time stamps for tuning builds only (-DTB_STAMPS), as in the hierarchical kernels.
#ifdef TB_STAMPS
__device__ unsigned long long tb_fused_stamps[8192 * 32];
#define TB_FSTAMP(i) \
  do { if (threadIdx.x == 0 && blockIdx.x < 8192) tb_fused_stamps[blockIdx.x * 32 + (i)] = wall_clock64(); } while (0)
extern "C" int tb_debug_stamps_fused(unsigned long long* host, int count) {
  return int(hipMemcpyFromSymbol(host, HIP_SYMBOL(tb_fused_stamps), size_t(count) * 8));
}
#else
#define TB_FSTAMP(i) do {} while (0)
#endif

namespace tb {

namespace {

constexpr int kMaxSeqs = kWave;     // candidate + references, one lane each
constexpr int kPadSymbols = 8;      // absent symbols behind every sequence: orders up to 8
constexpr int kMaxBlocks = 24;      // per wavefront
constexpr int kApartBlocks = 3;     // up to here what is left of a wavefront's blocks is not put together
constexpr size_t sums_bytes(bool rouge) { return 64 + 16 + (rouge ? kMaxSeqs * 4 : 0); }

// A kernel's plain arguments as they lie at the start of its argument segment.
struct PlainArgs {
  const void* cand;
  const int32_t* cand_lens;
  const void* refs;
  const int32_t* ref_lens;
  const int32_t* ref_count;
  const int32_t* ref_offsets;
  uint32_t cand_shape, ref_shape;
};
constexpr int kRegisterArgs = sizeof(PlainArgs);
#ifdef TB_PRELOADED_WORDS
static_assert(4 * TB_PRELOADED_WORDS == kRegisterArgs, "the build asks for other arguments in registers");
#endif

// The eight plain arguments before it come in scalar registers (the build asks for 56 bytes), so that
// the lengths are requested at once; what else is read before the tokens arrive stands first here and
// is read in one request meanwhile.  Before, the prologue waited for the argument segment six times in
// turn: 16 x 256 6.74 -> 6.64 us, 39 x 336 with two references, two orders, 6.31 -> 6.21.
struct FusedArgs {
  int32_t* status;         // may be null
  int vocab;
  int table_and_counters;  // 16-byte units of table and counters together
  uint32_t off_sym, off_sums;
  int progress_priority;   // 1: wavefronts of a workgroup that is behind get the higher priority
  int log2_slots;
  int id_bits;             // ids (candidate positions) are below 2^id_bits
  int64_t ref_rows;        // CSR lists: number of reference rows
  uint32_t pass_ends;      // bits 4(n - 1)..: last order of the stretch that starts with order n >= 2;
                           // bit 0: order 1 is a pass of its own; bit 1: the others are one pass, not one
                           // for each stretch
  int first_payload, first_key_bits;  // payload bits and key bits (order within the pass | payload)
                                      // of the table that order 1 is in
  int later_payload, later_key_bits;  // ... of the passes behind it
  int array_bytes;         // of one array of counter words, a word per id
  int want_distinct;
  float beta2;             // ROUGE-N: beta squared
  StatPtrs st;
  ScoreParams sp;
  void* out;               // per-sentence scores (fp32 or bfloat16: sp.out_bf16), or null
  void* rouge_prf;         // ROUGE-N of order N: [B, 3] (same type)
  int32_t* rouge_overlap;  // [B, R] or null
  int32_t* rouge_best;     // [B] or null
};

// LDS by byte offset.  (The kernel has dynamic LDS only, which starts at offset 0; going through the
// array's name would cost an addition of that 0 per access.)
template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds(uint32_t offset) {
  typedef __attribute__((address_space(3))) T* Ptr;
  return (Ptr)(uintptr_t)(offset);
}
__device__ __forceinline__ uint32_t lds_cas(uint32_t at, uint32_t desired) {  // expects 0
  uint32_t expected = 0u;
  __hip_atomic_compare_exchange_strong((uint32_t*)lds<uint32_t>(at), &expected, desired,
                                       __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
  return expected;
}
__device__ __forceinline__ uint32_t lds_add(uint32_t at, uint32_t v) {  // returns what was there
  return __hip_atomic_fetch_add((uint32_t*)lds<uint32_t>(at), v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The table of one pass, at LDS offset 0: buckets of four slots, filled front to back.  0: free slot;
// probe counts start at 1, so no entry is 0 (nor below id_limit).
struct SymbolTable {
  __device__ __forceinline__ uint32_t home(uint32_t h) const { return (h >> home_shift) & bucket_mask; }
  uint32_t bucket_mask;  // byte offsets of buckets
  int home_shift;        // 30 - log2(slots)
  int log2_buckets;
  uint32_t multiplier;   // odd << (32 - key bits)
  uint32_t id_limit;     // 1 << id_bits
  uint32_t limit;        // the same in a vector register: with the shift count one instruction may not
                         // read two scalar registers
  uint32_t longest;      // largest probe count an entry can hold, << id_bits
  uint32_t lost_at;      // LDS word set to 1 when a probe sequence reaches that count

  // (an odd number of buckets further, from the remainder alone)
  __device__ __forceinline__ uint32_t step(uint32_t remainder) const {
    return ((remainder >> 16) & ~31u) | 16u;
  }
  __device__ __forceinline__ static uint32_t match(const uint4& e, uint32_t mine) {
    return min(min(min(e.x ^ mine, e.y ^ mine), e.z ^ mine), e.w ^ mine);
  }
  __device__ __forceinline__ static uint4 bucket(uint32_t at) {
    typedef uint32_t Quad __attribute__((ext_vector_type(4)));
    const Quad q = *lds<Quad>(at);
    return make_uint4(q.x, q.y, q.z, q.w);
  }
  struct Probe {
    uint32_t x;     // the key's id if it was found, else at least id_limit
    uint32_t s;     // the bucket that was read last, and what it held
    uint4 e;
    uint32_t mine;  // the key's entry there, without an id
  };
  // Reads buckets until one holds the key or is not full; ends, because the odd step visits every
  // bucket and the plan keeps the table at most 3/4 full.  known(): the answer is `id` (the lane asks
  // all the same, which is less than a branch, but not for a second bucket).
  template <typename Known>
  __device__ __forceinline__ Probe probe(uint32_t h, Known known, uint32_t id) const {
    Probe p;
    p.s = home(h);
    p.e = bucket(p.s);
    __builtin_amdgcn_sched_barrier(0);  // (whatever known() waits for is on its way with the bucket)
    p.mine = (h << log2_buckets) + limit;
    p.x = known() ? id : match(p.e, p.mine);
    if (min(p.x, p.e.w) >= id_limit) {
      const uint32_t remainder = h << log2_buckets;
      do {
        p.s = (p.s + step(remainder)) & bucket_mask;
        p.mine = min(p.mine + id_limit, remainder + longest);
        p.e = bucket(p.s);
        p.x = match(p.e, p.mine);
      } while (min(p.x, p.e.w) >= id_limit);
      if (__builtin_expect(p.mine == remainder + longest, 0)) *lds<uint32_t>(lost_at) = 1u;
    }
    return p;
  }
  template <typename Known>
  __device__ __forceinline__ uint32_t find(uint32_t h, Known known, uint32_t id) const {
    return probe(h, known, id).x;
  }
  // Id of the key, entered as `id` where it is not there.  LOOK: buckets are read before anything is
  // swapped.  A wavefront that swaps from slot to slot does so as often as its slowest lane finds one
  // taken, six times in a table that fills up to the half.  A swap that fails (lanes of this or another
  // wavefront entered something there) goes on with the next slot.
  template <bool LOOK>
  __device__ __forceinline__ uint32_t claim(uint32_t h, uint32_t id) const {
    uint32_t s = home(h), mine = (h << log2_buckets) + limit;
    if (LOOK) {
      const Probe p = probe(h, [] { return false; }, 0u);
      if (p.x < id_limit) return p.x;
      s = p.s + first_free_slot(p.e.x, p.e.y, p.e.z);
      mine = p.mine;
    }
    uint32_t old = lds_cas(s, mine + id);
    uint32_t x = old ^ mine;
    if (min(old, x) >= id_limit) {  // neither free nor the key
      const uint32_t remainder = h << log2_buckets;
      do {
        const bool leaves = (s & 12u) == 12u;  // (selects, no branch)
        s = (s + (leaves ? step(remainder) - 12u : 4u)) & (bucket_mask | 12u);
        mine = min(mine + (leaves ? id_limit : 0u), remainder + longest);
        old = lds_cas(s, mine + id);
        x = old ^ mine;
      } while (min(old, x) >= id_limit);
      if (__builtin_expect(mine == remainder + longest, 0)) *lds<uint32_t>(lost_at) = 1u;
    }
    return old == 0u ? id : x;
  }
};

// What a kernel is for.  With one or two references lengths, rows and counters of a block are known
// without a look at other lanes, and no register holds what depends on the number of references.
// kRouge: ROUGE-1 and -2, kRougeLonger the others.  (One kernel for both moved 19 to 24 scalar registers to lanes
// of a vector register and back in ROUGE-1 and -2, too, and took a branch around the orders behind order 2: ROUGE-2
// of 512 x 512 with three references 7.16 -> 6.87 us, of 700 x 512 8.63 -> 8.25, ROUGE-1 of 1435 x 503 with one 7.43 -> 7.23,
// with three 10.44 -> 10.12.)
enum Mode { kOneReference, kTwoReferences, kReferences, kRouge, kRougeLonger };

// The value of sequence f.  (Arguments by value: a choice between variables that closures refer to is
// made between their addresses, which keeps all of them in memory.)
template <bool THREE, typename T>
__device__ __forceinline__ T pick(int f, T cand, T ref, T ref1) {
  T v = cand;
  if (f >= 1) v = ref;
  if (THREE && f >= 2) v = ref1;
  return v;
}

// BLOCKS: blocks of 64 positions per wavefront.  KEEP: a pass starts above order 2, with the ids of
// the order below.  ALONE: the kernel that has more registers.
template <int BLOCKS, bool KEEP, Mode MODE, bool ALONE>
__device__ __forceinline__
void fused_group(const void* cand, const int32_t* cand_lens, const void* refs,
                  const int32_t* ref_lens, const int32_t* ref_count, const int32_t* ref_offsets,
                  uint32_t cand_shape, uint32_t ref_shape) {
  // The struct behind the plain arguments is read through the kernel-argument segment where its fields are used: loads of a
  // by-value parameter all stand at the entry and would occupy scalar registers throughout.
  typedef const char __attribute__((address_space(4)))* Segment;
  const FusedArgs& a =
      *(const FusedArgs*)((Segment)__builtin_amdgcn_kernarg_segment_ptr() + kRegisterArgs);
  constexpr bool ROUGE = MODE == kRouge || MODE == kRougeLonger, SHORT = MODE == kRouge;
  constexpr bool ONE = MODE == kOneReference, TWO = MODE == kTwoReferences;
  constexpr bool FEW = ONE || TWO;
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));
  const int cs = cand_shape & 0xFFFFu, R = ONE ? 1 : TWO ? 2 : (cand_shape >> 16) & 0xFFu;
  const int log2_waves = cand_shape >> 24;
  const int rs = ref_shape & 0xFFFFu, N = (ref_shape >> 16) & 0xFFu;
  const bool wide = ref_shape >> 24;  // int64 token ids
  const int nwaves = 1 << log2_waves, nt = kWave << log2_waves;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int g = blockIdx.x;
  TB_FSTAMP(0);

  // Lengths (0 for a reference not in use) and rows of the sequences; with several references lane j of
  // every wavefront holds those of sequence j, and the prefix of the sequences' block counts
  int raw_cand = uniform_load(cand_lens, g);
  // (no branch: with neither counts nor lists a length is read, and not used)
  const int32_t* const rows = ref_offsets ? ref_offsets : ref_count ? ref_count : cand_lens;
  int rows0 = uniform_load(rows, g), rows1 = uniform_load(rows, g + (ref_offsets ? 1 : 0));
  int64_t row0 = int64_t(g) * R;
  int raw_ref = 0, raw_ref1 = 0;
  if (FEW) {
    if (!ref_offsets) {
      raw_ref = uniform_load(ref_lens, row0);
      if (TWO) raw_ref1 = uniform_load(ref_lens, row0 + 1);
    }
  } else {
    if (!ref_offsets && lane >= 1 && lane <= R) raw_ref = ref_lens[row0 + lane - 1];
  }
  // (in one request while the lengths are on their way)
  int table_and_counters = a.table_and_counters, vocab_size = a.vocab;
  uint32_t sym_at = a.off_sym;
  // per order: sums (8 words), distinct n-grams (8 words)
  uint32_t part_at = a.off_sums;
  int progress = a.progress_priority, lg = a.log2_slots, id_bits = a.id_bits;
  asm volatile("" : "+s"(table_and_counters), "+s"(vocab_size), "+s"(sym_at), "+s"(part_at),
               "+s"(progress), "+s"(lg), "+s"(id_bits), "+s"(raw_cand), "+s"(rows0), "+s"(rows1));
  int used = R;
  bool odd = false;  // counts or lists that had to be clamped
  if (ref_offsets) {  // uniform
    const RefRows rr = listed_rows(rows0, rows1, a.ref_rows, R, &odd);
    row0 = rr.row0;
    used = rr.used;
    if (FEW) {
      if (used > 0) raw_ref = uniform_load(ref_lens, row0);
      if (TWO && used > 1) raw_ref1 = uniform_load(ref_lens, row0 + 1);
    } else if (lane >= 1 && lane <= used) {
      raw_ref = ref_lens[row0 + lane - 1];
    }
  } else if (ref_count) {
    used = min(max(rows0, 1), R);
    odd = rows0 != used;
    if (TWO) raw_ref1 = used > 1 ? raw_ref1 : 0;
    if (!FEW) raw_ref = lane <= used ? raw_ref : 0;
  }
  const bool prio = progress != 0;
  const uint32_t lost_at = part_at + 64;  // non-zero: a probe sequence was too long to be counted
  const uint32_t overlap_at = lost_at + 4;        // ROUGE: overlap with each reference
  const uint32_t closest_at = lost_at + 4;        // BLEU: closest reference length, brevity penalty
  const uint32_t sequence_at = part_at + uint32_t(sums_bytes(ROUGE));  // a byte for each block: its reference (see LISTED)
  if (prio) __builtin_amdgcn_s_setprio(3);

  const uint32_t token_bytes = wide ? 8u : 4u;
  const uint64_t cand_row = reinterpret_cast<uint64_t>(cand) + uint64_t(uint32_t(g)) * (uint32_t(cs) * token_bytes);
  const uint64_t ref_row = reinterpret_cast<uint64_t>(refs) + uint64_t(row0) * (uint32_t(rs) * token_bytes);
  const int cand_len = min(max(raw_cand, 0), cs);
  const int ref_len = min(max(raw_ref, 0), rs), ref_len1 = min(max(raw_ref1, 0), rs);
  const int my_len = pick<false>(FEW || lane > 0 ? 1 : 0, cand_len, ref_len, 0);
  const bool clamped = cand_len != raw_cand || ref_len != raw_ref || ref_len1 != raw_ref1 || odd;
  if (__builtin_amdgcn_ballot_w64(clamped)) {  // uniform
    if (wave == 0 && clamped && a.status) atomicOr(a.status, TB_DEV_LENGTH_RANGE);
  }
  const int cand_blocks = (cand_len + kWave - 1) >> 6;
  int block_ends, block_begins = 0, ends = 0;
  const int begin1 = cand_blocks + ((ref_len + kWave - 1) >> 6);  // (FEW: of the second reference)
  uint64_t row_at = 0;
  if (FEW) {
    block_ends = begin1 + ((ref_len1 + kWave - 1) >> 6);
  } else {
    const int my_seq_blocks = (my_len + kWave - 1) >> 6;
    block_ends = wave_inclusive_scan(my_seq_blocks);
    block_begins = block_ends - my_seq_blocks;
    ends = lane <= R ? block_ends : 0x7FFFFFFF;
    row_at = lane == 0 ? cand_row : ref_row + uint64_t(uint32_t(lane - 1) * uint32_t(rs)) * token_bytes;
  }
  const int blocks =
      min(FEW ? block_ends : lane_value(block_ends, kWave - 1), BLOCKS << log2_waves);
  auto sequence_of = [&](int b) __attribute__((always_inline)) {  // of block b < blocks
    if (FEW) return (b >= cand_blocks ? 1 : 0) + (TWO && b >= begin1 ? 1 : 0);
    return int(__popcll(__builtin_amdgcn_ballot_w64(ends <= b)));
  };
  auto reference_of = [&](int b) __attribute__((always_inline)) {  // the same, of a block behind the candidate's
    if (FEW) {
      int f = 1;
      if (TWO && b >= begin1) f = 2;
      return f;
    }
    return sequence_of(b);
  };
  // position of block b of sequence f in its row
  auto first_of = [&](int b, int f) __attribute__((always_inline)) {
    if (FEW) return (b - pick<TWO>(f, 0, cand_blocks, begin1)) << 6;
    return (b - __builtin_amdgcn_readlane(block_begins, f)) << 6;
  };
  auto length_of = [&](int f) __attribute__((always_inline)) {
    if (FEW) return pick<TWO>(f, cand_len, ref_len, ref_len1);
    return int(__builtin_amdgcn_readlane(my_len, f));
  };
  auto lane_value64 = [](uint64_t v, int from) __attribute__((always_inline)) {
    return uint64_t(uint32_t(__builtin_amdgcn_readlane(int(v >> 32), from))) << 32 |
           uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), from));
  };
  auto row_of = [&](int f) __attribute__((always_inline)) {
    if (FEW) return pick<TWO>(f, cand_row, ref_row, ref_row + uint32_t(rs) * token_bytes);
    return lane_value64(row_at, f);
  };
  // Closest reference length, the shorter one on ties (no reference at all: 0).
  auto closest_length = [&]() __attribute__((always_inline)) {
    if (FEW) {
      const int d0 = abs(ref_len - cand_len), d1 = abs(ref_len1 - cand_len);
      const bool other = TWO && used > 1 && (d1 < d0 || (d1 == d0 && ref_len1 < ref_len));
      return pick<TWO>(other ? 2 : 1, 0, ref_len, ref_len1);
    }
    const bool is_ref = lane >= 1 && lane <= used;
    const int key = is_ref ? abs(my_len - cand_len) << 15 | my_len : 0x7FFFFFFF;
    return used > 0 ? wave_min(key) & 0x7FFF : 0;
  };

  SymbolTable table;
  auto set_key_bits = [&](int key_bits) __attribute__((always_inline)) {
    const int count_bits = min(32 - key_bits + lg - 2 - id_bits, 32 - id_bits);
    table.multiplier = 0x9E3779B1u << (32 - key_bits);
    table.longest = ((1u << count_bits) - 1u) << id_bits;
  };
  const uint32_t cnt_at = 4u << lg;
  uint32_t array_bytes = 0;
  int want = 0;
  // (pinned, so that nothing of this is left for after the barrier)
  auto set_up = [&]() __attribute__((always_inline)) {
    table.bucket_mask = (((1u << lg) - 1u) << 2) & ~15u;
    table.home_shift = 30 - lg;
    table.log2_buckets = lg - 2;
    table.id_limit = 1u << id_bits;
    table.lost_at = lost_at;
    set_key_bits(a.first_key_bits);
    array_bytes = uint32_t(a.array_bytes);
    want = a.want_distinct;
    asm volatile("v_mov_b32 %0, %1" : "=v"(table.limit) : "s"(table.id_limit));
    asm volatile("" : "+s"(table.bucket_mask), "+s"(table.home_shift), "+s"(table.log2_buckets),
                 "+s"(table.id_limit), "+s"(table.multiplier), "+s"(table.longest), "+s"(array_bytes),
                 "+s"(want));
  };

  // This wavefront's blocks are wave, wave + nwaves, ... (the candidate's come first).  val[i]: the
  // token, then the symbol, of the lane's position (KEEP: then the id of the last finished order).
  int32_t val[BLOCKS];
#pragma unroll
  for (int i = 0; i < BLOCKS; ++i)  // (blocks that are not there hold any value: nothing reads it)
    val[i] = __builtin_nondeterministic_value(0);
  // Lane i: positions that the wavefront's block i has, and where its tokens are.  Chosen block by block
  // from two or three sequences these are scalar instructions (33 a block with two references), of which a
  // unit issues one a cycle for all its wavefronts: us of the call with the choice per block and like this,
  // one order with two references 825 x 643 9.5 -> 8.2, 101 x 1194 7.3 -> 6.5, four orders 11.1 -> 10.3;
  // 256 x 1088 with one 8.4 -> 8.1.  One or two blocks have too few.
  constexpr bool ALL_AT_ONCE = FEW && BLOCKS >= 3;
  int block_left = 0;
  uint64_t block_at = 0;
  if (ALL_AT_ONCE) {
    const int b = wave + (lane << log2_waves), f = sequence_of(b), first = first_of(b, f);
    block_left = length_of(f) - first;
    block_at = row_of(f) + uint32_t(first) * token_bytes;
  }
  // Tokens are requested; while they are on their way, table slots become free, counters zero, symbols
  // behind the sequences absent.
  auto stage = [&](auto token_type) __attribute__((always_inline)) {
    typedef decltype(token_type) Token;
    typedef std::make_unsigned_t<Token> UToken;
    Token raw[BLOCKS];
    int left[BLOCKS];  // positions of the block inside the sequence
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) {
      const int b = wave + (i << log2_waves);
      raw[i] = 0;
      left[i] = 0;
      // (uniform; blocks that are not there are not touched any more.  With more references the other
      // form is the better one: the values set above need no registers)
      if (FEW && b >= blocks) break;
      if (b >= blocks) continue;
      uint64_t at;
      if (ALL_AT_ONCE) {
        left[i] = __builtin_amdgcn_readlane(block_left, i);
        at = lane_value64(block_at, i);
      } else {
        const int f = sequence_of(b), first = first_of(b, f);
        left[i] = length_of(f) - first;
        at = row_of(f) + uint32_t(first) * token_bytes;
      }
      typedef const Token __attribute__((address_space(1)))* GlobalToken;
      raw[i] = reinterpret_cast<GlobalToken>(at)[uint32_t(min(lane, left[i] - 1))];
    }
    set_up();
    for (uint32_t q = tid; q < uint32_t(table_and_counters); q += nt)
      *lds<Quad>(16u * q) = Quad(0u);
    if (wave == 0 && lane <= R) {
      const int behind = FEW ? pick<TWO>(lane, cand_blocks, begin1, block_ends) : block_ends;
      *lds<Quad>(sym_at + uint32_t(2 * kWave) * behind + uint32_t(2 * kPadSymbols) * lane) = Quad(~0u);
    }
    if (tid < 17) *lds<uint32_t>(part_at + 4 * tid) = 0u;  // (lost_at, too)
    if (ROUGE && tid < kMaxSeqs) *lds<uint32_t>(overlap_at + 4 * tid) = 0u;
    const UToken vocab = UToken(uint32_t(vocab_size));
    bool bad = false;
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) {
      if (FEW && wave + (i << log2_waves) >= blocks) break;  // uniform
      // a token outside the vocabulary is reported and taken as 0
      const bool outside = UToken(raw[i]) >= vocab;
      const bool here = lane < left[i];
      bad |= outside & here;
      val[i] = here ? (outside ? 0 : int32_t(raw[i])) : -1;
    }
    if (__builtin_amdgcn_ballot_w64(bad)) {  // uniform
      if (bad && a.status) atomicOr(a.status, TB_DEV_TOKEN_RANGE);
    }
  };
  if (wide) {
    stage(int64_t(0));
  } else {
    stage(int32_t(0));
  }
  __syncthreads();
  TB_FSTAMP(1);

  // The blocks at hand are val[0], ..., finished ones rotate to the end (a register array cannot be
  // indexed by a loop counter).  A rotation moves all of them, so they are taken in groups of up to
  // four, as far as full ones go (128 x 8192 48.5 -> 46.7 us, 128 x 5000 29.5 -> 28.7); where only order 1
  // keeps them in registers, in twos (4096 x 2048 with two references 109.0 -> 106.5; four are no better, and
  // with more references, whose kernels are short of registers, twos cost a tenth).
  constexpr bool LOOK = KEEP || BLOCKS > 6;  // (see claim)
  // (Order 1 of a table that is for more orders, or for one order only, enters few of its slots' worth: with
  // three references or more 1 % faster without the look, with fewer 4 % slower where many tokens are the same.)
  constexpr bool LOOK_FIRST = KEEP || (LOOK && MODE != kReferences);
  constexpr int GROUP = !KEEP ? (FEW && BLOCKS >= 8 ? 2 : 1) : BLOCKS >= 8 ? 4 : BLOCKS >= 4 ? 2 : 1;
  auto rotate = [&](auto by) __attribute__((always_inline)) {
    constexpr int n = decltype(by)::value;
    int32_t first[n];
#pragma unroll
    for (int u = 0; u < n; ++u) first[u] = val[u];
#pragma unroll
    for (int i = 0; i + n < BLOCKS; ++i) val[i] = val[i + n];
#pragma unroll
    for (int u = 0; u < n; ++u) val[BLOCKS - n + u] = first[u];
  };
  // f(val[k]) for the blocks from i to `end`; f may change the value
  auto each_block = [&](int& i, int end, auto&& f) __attribute__((always_inline)) {
    if (GROUP > 1) {
#pragma unroll 1
      for (; i + GROUP <= end; i += GROUP) {
#pragma unroll
        for (int u = 0; u < GROUP; ++u) f(val[u]);
        rotate(std::integral_constant<int, GROUP>{});
      }
    }
#pragma unroll 1
    for (; i < end; ++i) {
      f(val[0]);
      rotate(std::integral_constant<int, 1>{});
    }
  };

  // Counters: 16-bit fields, two a word, the words of all ids in one array per pair of fields.  A position
  // whose n-gram has the position's own id (its first occurrence) is not counted: no reference asks for
  // other ids, so a field that nothing was added to stands for one occurrence in the candidate.  (ROUGE-1 and -2
  // count every occurrence: with hardly an n-gram's second one behind it, the branch costs more than it saves.)
  //   * One reference, and ROUGE-N: a field is one less than the n-gram's count in the candidate, less
  //     what the reference has had of it so far (a negative lower half borrows from the upper one).  A
  //     reference's n-gram that does not find it negative is a match, and matches are all that is asked
  //     for: no pass over the counters, which cost a lone workgroup of 16 x 256 tokens 1600 of 15000
  //     cycles, and one with eight references of 464 tokens (ROUGE-1) 7 of 11 us.
  //   * Two references: the same less the reference's count, one field each; the smaller one is (one less
  //     than) what the candidate has beyond both.
  //   * More: one less than the count in the candidate, then the counts in the references.
  constexpr bool EVERY = SHORT;
  constexpr bool matching = ONE || ROUGE;
  constexpr bool differences = MODE != kReferences;
  const int order_fields = differences ? R : R + 1;
  const uint32_t ref_unit = differences ? ~0u : 1u;
  const int first_ref = differences ? -1 : 0;  // field of reference 0, which does not exist
  auto array_of = [&](int field) __attribute__((always_inline)) { return cnt_at + uint32_t(field >> 1) * array_bytes; };
  auto count_candidate = [&](int order, uint32_t id) __attribute__((always_inline)) {
    if (ROUGE) {
      uint32_t at = cnt_at + 4u * id;
#pragma unroll 1
      for (int j = R; j > 0; j -= 2, at += array_bytes) lds_add(at, j > 1 ? 0x10001u : 1u);
    } else {
      const int field = order * order_fields;
      lds_add(array_of(field) + 4u * id, (TWO ? 0x10001u : 1u) << (16 * (field & 1)));
    }
  };
  // the counter's word before reference f's n-gram was counted, if it is wanted
  auto count_reference = [&](int order, int f, uint32_t id) __attribute__((always_inline)) {
    const int field = (ROUGE ? 0 : order * order_fields) + first_ref + f;
    const uint32_t at = array_of(field) + 4u * id, unit = ref_unit << (16 * (field & 1));
    if (matching) return lds_add(at, unit);
    lds_add(at, unit);
    return 0u;
  };
  // whether the field was not negative, with EVERY positive (low + 65536 * high, each within 32767)
  auto is_match = [&](int order, int f, uint32_t word) __attribute__((always_inline)) {
    const int odd = ((ROUGE ? 0 : order * order_fields) + first_ref + f) & 1;
    if (EVERY) return int32_t(word << (odd ? 0 : 16)) > (odd ? 0x7FFF : 0);
    return int32_t(word << (odd ? 0 : 16)) >= (odd ? -0x8000 : 0);
  };
  // Of this lane, orders 1, 2 and the ones behind them that a stretch has: the reference's matches, and
  // the candidate's positions whose n-gram has another position's id.
  // (Two orders in the halves of a word, the second one in the upper half.)
  uint32_t match12 = 0, matches[2] = {0, 0};
  uint32_t repeat12 = 0, repeats[2] = {0, 0};
  int overlap = 0;                           // ROUGE: lane f: matches with reference f
  const int my_cand_blocks = (max(cand_blocks - wave, 0) + nwaves - 1) >> log2_waves;
  const int my_blocks = (max(blocks - wave, 0) + nwaves - 1) >> log2_waves;
  // byte offset of the symbol of this lane's position in the wavefront's first block, and from
  // block to block (behind sequence f lie kPadSymbols * f more)
  const uint32_t first_sym = sym_at + 2u * uint32_t(kWave * wave + lane);
  const uint32_t sym_stride = 2u * uint32_t(nt);

  const uint32_t id_limit = table.id_limit;
  const bool want_distinct = want;

  // What is left of blocks is put together to full ones (COMPACT; not where a wavefront has few).
  constexpr bool COMPACT = BLOCKS > kApartBlocks && !SHORT;
  constexpr bool LISTED = COMPACT && !FEW;  // the references of positions are looked up

  // ---- order 1: tokens become symbols
  {
    int i = 0, b = wave;
    uint32_t id = uint32_t(kWave * wave + lane), s = first_sym;
    each_block(i, my_cand_blocks, [&](int32_t& v) __attribute__((always_inline)) {
      int32_t got = -1;
      if (v >= 0) {
        got = int32_t(table.claim<LOOK_FIRST>(uint32_t(v) * table.multiplier, id));
        if (EVERY || got != int32_t(id)) {
          if (!ROUGE || N == 1) count_candidate(0, uint32_t(got));
          if (!ROUGE) ++repeat12;
        }
      }
      *lds<int16_t>(s) = int16_t(got);
      if (SHORT) v = got;
      id += nt;
      s += sym_stride;
      b += nwaves;
    });
    if (!ROUGE && wave == nwaves - 1) {
      // the lengths' part of the score, for the tail: by the wavefront that has the fewest blocks
      const int best = closest_length();
      *lds<int32_t>(closest_at) = best;
      *lds<float>(closest_at + 4) = expf(1.0f - float(best) / float(cand_len));
    }
    __syncthreads();
    TB_FSTAMP(2);
    each_block(i, my_blocks, [&](int32_t& v) __attribute__((always_inline)) {
      const int f = reference_of(b);
      int32_t got = -1;
      bool match = false;
      if (v >= 0) {
        const uint32_t x = table.find(uint32_t(v) * table.multiplier, [] { return false; }, 0u);
        if (x < id_limit) {
          got = int32_t(x);
          if (!ROUGE || N == 1) {
            const uint32_t word = count_reference(0, f, x);
            if (matching) match = is_match(0, f, word);
          }
        }
      }
      *lds<int16_t>(s + uint32_t(2 * kPadSymbols) * f) = int16_t(got);
      if (LISTED && N > 2) *lds<uint8_t>(sequence_at + uint32_t(b)) = uint8_t(f);
      if (!ROUGE) match12 += match ? 1u : 0u;
      if (ROUGE && N == 1) {
        const int of_block = __popcll(__builtin_amdgcn_ballot_w64(match));
        overlap += lane == f ? of_block : 0;
      }
      if (SHORT) v = got;
      s += sym_stride;
      b += nwaves;
    });
  }
  TB_FSTAMP(3);

  // A stretch is up to three orders that a block takes in one go, a pass one stretch or several with
  // one table (from order 5 on): the next stretch's insertions go beside the look-ups before them as
  // those of order 2 go beside the look-ups of order 1.  (A pass for each stretch, with its sums, its
  // clearing and three barriers more: eight orders of 457 x 10 with three references 10.9 us instead of
  // 9.8, of 3946 x 21 17.0 instead of 15.5; 517 drawn shapes of five to eight orders 1.09 of its speed.)
  constexpr int DEPTH = KEEP ? 3 : 2;  // orders of a stretch behind order 2 (without KEEP there are four at most)
  // KEEP: blocks of val that hold what is left of the candidate's and of the references' positions (from
  // my_cand_blocks on)
  int kept_cand = 0, kept = my_cand_blocks;
  int swept = 0, counted = 0, hi = 1;
  bool pass_ends = a.pass_ends & 1u;
#pragma unroll 1
  while (true) {
    // ---- sums of the orders, two in the halves of a word (neither exceeds the positions), in LDS, where
    // the tail's lanes find theirs: matches of a stretch, or for a whole pass min(count, largest reference
    // count) of the candidate's n-grams; with two references what the candidate has of them beyond both
    // (the rest of them is that minimum)
    auto add_up = [&](uint32_t at, int n, uint32_t part) __attribute__((always_inline)) {
      part = uint32_t(row_inclusive_scan(int(part)));
      if ((lane & 15) == 15) lds_add(at + 4u * uint32_t(n - 1), part);
    };
    auto add_orders = [&](uint32_t at, uint32_t first, const uint32_t (&more)[2]) __attribute__((always_inline)) {
      if (counted < 2) add_up(at, 1, first);
      if (hi > 2) {
        const int n = KEEP ? max(counted, 2) + 1 : 3;
        add_up(at, n, more[0]);
        if (KEEP && hi > n + 1) add_up(at, n + 2, more[1]);
      }
    };
    if (!ROUGE && (pass_ends || (KEEP && hi > 1))) {
      if (matching && my_cand_blocks < my_blocks) {  // (uniform)
        add_orders(part_at, match12, matches);
        match12 = matches[0] = matches[1] = 0;
      }
      if ((TWO || want_distinct) && my_cand_blocks > 0) {
        add_orders(part_at + 32, repeat12, repeats);
        repeat12 = repeats[0] = repeats[1] = 0;
      }
      counted = hi;
    }
    if (pass_ends) {
      if (hi == N && prio) __builtin_amdgcn_s_setprio(0);
      if (ROUGE) {
        if (hi == N && lane >= 1 && lane <= R) lds_add(overlap_at + 4u * uint32_t(lane - 1), uint32_t(overlap));
      } else if (!matching) {
        __syncthreads();
        if (TWO) {
          const uint32_t at = cnt_at + 4u * uint32_t(tid);
#pragma unroll 1
          for (int n = swept + 1; n <= hi; n += 2) {
            uint32_t part = 0;
            uint32_t e = at + uint32_t(n - 1 - swept) * array_bytes;
            const uint32_t second = n < hi ? array_bytes : 0u;
#pragma unroll 1
            for (int k = tid; k < cand_len; k += nt, e += 4u * uint32_t(nt)) {
              const int32_t v0 = *lds<int32_t>(e), v1 = *lds<int32_t>(e + second);
              const int32_t low0 = int16_t(v0), low1 = int16_t(v1);
              part += uint32_t(max(min(low0, (v0 - low0) >> 16) + 1, 0)) |
                      uint32_t(max(min(low1, (v1 - low1) >> 16) + 1, 0)) << 16;
            }
            if (n == hi) part &= 0xFFFFu;
            add_up(part_at, n, part);
          }
        } else {
          typedef uint16_t Halves __attribute__((ext_vector_type(2)));
          auto max_halves = [](uint32_t a, uint32_t b) __attribute__((always_inline)) {
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(
                __builtin_bit_cast(Halves, a), __builtin_bit_cast(Halves, b)));
          };
          // Two orders have order_fields words: the first order's count and first reference in word 0,
          // the second order's count in word `middle`, in the upper half if the last reference of the
          // first order has the lower one.  Words of both are read side by side: one after the other
          // they are two chains of dependent steps, which is better only where registers are so short that
          // what is read side by side goes through scratch (24 blocks, shared units: 860 x 343 with 16 references
          // of 1184, eight orders, 150 -> 115 us; 170 shapes 1.024, the slowest 0.975).
          constexpr bool BOTH = BLOCKS <= 16 || ALONE;
          const int middle = order_fields >> 1;
          const bool shared = order_fields & 1;
          // (where nothing has been added to a position's fields, no reference has)
          auto least = [](uint32_t count, uint32_t most) __attribute__((always_inline)) {
            return min(count + 1u, max(most & 0xFFFFu, most >> 16));
          };
#pragma unroll 1
          for (int n = swept + 1; n <= hi; n += 2) {
            const bool two = n < hi;
            uint32_t part = 0;
            uint32_t e = array_of((n - 1 - swept) * order_fields) + 4u * uint32_t(tid);
            const uint32_t to_middle = two || shared ? uint32_t(middle) * array_bytes : 0u;
            const uint32_t to_other = two ? to_middle : 0u;
#pragma unroll 1
            for (int k = tid; k < cand_len; k += nt, e += 4u * uint32_t(nt)) {
              const uint32_t head = *lds<uint32_t>(e), second = *lds<uint32_t>(e + to_middle);
              uint32_t most0 = head >> 16, most1 = shared ? 0u : second >> 16;
              if (shared) most0 = max_halves(most0, second & 0xFFFFu);
              if (!BOTH) {
                auto most_of = [&](uint32_t& most, int w, int end) __attribute__((always_inline)) {  // words w..end - 1
                  uint32_t at = e + uint32_t(w) * array_bytes;
#pragma unroll 1
                  for (; w < end; ++w, at += array_bytes) most = max_halves(most, *lds<uint32_t>(at));
                };
                most_of(most0, 1, middle);
                part += least(head & 0xFFFFu, most0);
                if (two) {
                  most_of(most1, middle + 1, order_fields);
                  part += least(shared ? second >> 16 : second & 0xFFFFu, most1) << 16;
                }
                continue;
              }
              uint32_t at = e;
              int w = 1;
#pragma unroll 1
              for (; w + 1 < middle; w += 2) {
                at += array_bytes;
                const uint32_t v0 = *lds<uint32_t>(at), v1 = *lds<uint32_t>(at + to_other);
                at += array_bytes;
                const uint32_t u0 = *lds<uint32_t>(at), u1 = *lds<uint32_t>(at + to_other);
                most0 = max_halves(most0, max_halves(v0, u0));
                most1 = max_halves(most1, max_halves(v1, u1));
              }
              if (w < middle) {
                at += array_bytes;
                const uint32_t v0 = *lds<uint32_t>(at), v1 = *lds<uint32_t>(at + to_other);
                most0 = max_halves(most0, v0);
                most1 = max_halves(most1, v1);
              }
              part += least(head & 0xFFFFu, most0);
              if (two) {
                if (shared) most1 = max_halves(most1, *lds<uint32_t>(at + array_bytes + to_middle));
                part += least(shared ? second >> 16 : second & 0xFFFFu, most1) << 16;
              }
            }
            add_up(part_at, n, part);
          }
        }
      }
      __syncthreads();
      if (hi == N) break;
      for (uint32_t q = tid; q < uint32_t(table_and_counters); q += nt)
        *lds<Quad>(16u * q) = Quad(0u);
      __syncthreads();
      swept = hi;
      set_key_bits(a.later_key_bits);
    }
    // ---- orders lo..hi
    const int lo = hi + 1;
    hi = int((a.pass_ends >> (4 * hi)) & 15u);
    pass_ends = hi == N || !(a.pass_ends & 2u);
    // Two workgroups share a compute unit and its arbiter serves the older wavefronts first: left
    // alone, the one dispatched first finishes early and its mate runs alone on a half-empty unit.
    // The workgroup that is behind therefore gets the higher priority.
    if (prio) {
      if (lo == 2)
        __builtin_amdgcn_s_setprio(2);
      else
        __builtin_amdgcn_s_setprio(1);
    }
    // the order within the pass is the key's top bits: a constant added to the product
    const int payload = swept == 0 ? __builtin_amdgcn_readfirstlane(a.first_payload)
                                   : __builtin_amdgcn_readfirstlane(a.later_payload);
    const uint32_t tag_unit = table.multiplier << payload;
    auto hash_of = [&](int n, uint32_t prefix, uint32_t last) __attribute__((always_inline)) {
      return ((prefix << id_bits) | last) * table.multiplier + uint32_t(n - 1 - swept) * tag_unit;
    };
    // Order 2 is for all positions of a block, and what goes on from it is a word: the position as
    // blocks number them (64 * block + lane) and, in the upper half, its id; -1: nothing.  Orders from
    // `next` on take such words.
    const bool dense = !KEEP || lo == 2;
    const int next = dense ? 3 : lo;
    const bool deeper = !SHORT && (KEEP || hi > 2);
    const uint32_t ahead = 2u * uint32_t(next - 1), other = sym_at + ahead;
    auto word_of = [](uint32_t position, uint32_t id) __attribute__((always_inline)) { return int32_t(position | id << 16); };

    // The candidate's n-gram at `position`; repeated(id): its id is that of another position.  (The n-gram
    // that goes on like the candidate does at the prefix's id has that id.)  A position that has its own id
    // is through: all longer n-grams at it have the same, they go on like it does, and none is counted.
    auto enter = [&](int n, uint32_t position, uint32_t prefix, int32_t last, int32_t implied,
                     auto&& repeated) __attribute__((always_inline)) {
      uint32_t id = prefix;
      if (last != implied) id = table.claim<LOOK>(hash_of(n, prefix, uint32_t(last)), position);
      if (!EVERY && id == position) return;
      if (!ROUGE || n == N) count_candidate(n - 1 - swept, id);
      repeated(id);
    };
    // Orders from `next` on, of lanes that have gone on so far; left: the word of those that go on from there.
    auto enter_step = [&](auto depth, uint32_t position, uint32_t prefix, const int32_t (&lasts)[DEPTH],
                          int32_t& left, auto&& again) __attribute__((always_inline)) {
      constexpr int d = decltype(depth)::value;
      if (lasts[d] < 0) return;  // (an absent symbol: no n-gram here)
      const int32_t implied = *lds<int16_t>(other + 2u * prefix + 2u * d);
      enter(next + d, position, prefix, lasts[d], implied, [&](uint32_t id) __attribute__((always_inline)) {
        if (!ROUGE) repeats[d >> 1] += d & 1 ? 0x10000u : 1u;
        if (d == DEPTH - 1 || next + d == hi) {  // (uniform)
          left = word_of(position, id);
        } else {
          if constexpr (d + 1 < DEPTH) again(std::integral_constant<int, d + 1>{}, position, id, lasts, left, again);
        }
      });
    };
    auto enter_more = [&](int32_t word) __attribute__((always_inline)) {
      int32_t left = -1;
      const uint32_t position = uint32_t(word) & 0xFFFFu;
      if (word >= 0) {
        int32_t lasts[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) lasts[d] = *lds<int16_t>(other + 2u * position + 2u * d);
        enter_step(std::integral_constant<int, 0>{}, position, uint32_t(word) >> 16, lasts, left, enter_step);
      }
      return left;
    };
    // The n-gram of reference f; found(id, what count_reference returned).  Lanes drop out where an n-gram is
    // not the candidate's, and stay out for the orders behind it.
    auto look_up = [&](int n, int f, uint32_t prefix, int32_t last, uint32_t implied_at, auto&& found) __attribute__((always_inline)) {
      const int32_t implied = *lds<int16_t>(implied_at);
      const uint32_t id = table.find(hash_of(n, prefix, uint32_t(last)), [&] { return implied == last; }, prefix);
      if (id >= id_limit) return;
      uint32_t word = 0;
      if (!ROUGE || n == N) word = count_reference(n - 1 - swept, f, id);
      found(id, word);
    };
    auto look_up_step = [&](auto depth, int f, uint32_t position, uint32_t prefix, const int32_t (&lasts)[DEPTH],
                            int32_t& left, auto&& again) __attribute__((always_inline)) {
      constexpr int d = decltype(depth)::value;
      if (lasts[d] < 0) return;
      look_up(next + d, f, prefix, lasts[d], other + 2u * prefix + 2u * d, [&](uint32_t id, uint32_t counter) __attribute__((always_inline)) {
        if (d == DEPTH - 1 || next + d == hi) {  // (uniform)
          left = word_of(position, id);
        } else {
          if constexpr (d + 1 < DEPTH) again(std::integral_constant<int, d + 1>{}, f, position, id, lasts, left, again);
        }
        if (ROUGE) {
          if (next + d == N && is_match(0, f, counter)) lds_add(overlap_at + 4u * uint32_t(f - 1), 1u);
        } else if (matching) {
          matches[d >> 1] += is_match(next + d - 1 - swept, f, counter) ? (d & 1 ? 0x10000u : 1u) : 0u;
        }
      });
    };
    // block: of the wavefront's, where words are still in the place of their positions
    auto look_up_more = [&](int32_t word, int block) __attribute__((always_inline)) {
      int32_t left = -1;
      const uint32_t position = uint32_t(word) & 0xFFFFu;
      int f = 1;
      if (!FEW && !LISTED) f = reference_of(wave + (block << log2_waves));  // (all lanes take part)
      if (word >= 0) {
        if (LISTED) f = *lds<uint8_t>(sequence_at + (position >> 6));
        if (TWO) f = position >= uint32_t(begin1) * kWave ? 2 : 1;
        const uint32_t own = other + 2u * position + uint32_t(2 * kPadSymbols) * f;
        int32_t lasts[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) lasts[d] = *lds<int16_t>(own + 2u * d);
        look_up_step(std::integral_constant<int, 0>{}, f, position, uint32_t(word) >> 16, lasts, left, look_up_step);
      }
      return left;
    };
    // A block's order 2, and without COMPACT the orders behind it at once.
    const bool at_once = !COMPACT && !SHORT && hi > 2;
    int i = 0, b = wave;
    uint32_t id = uint32_t(kWave * wave + lane), s = first_sym;
    auto enter_block = [&]() __attribute__((always_inline)) {
      int32_t left = -1;
      const int32_t prefix = *lds<int16_t>(s), last = *lds<int16_t>(s + 2);
      int32_t lasts[DEPTH];
#pragma unroll
      for (int d = 0; !COMPACT && !SHORT && d < DEPTH; ++d) lasts[d] = *lds<int16_t>(s + 4 + 2u * d);
      if (last >= 0 && (EVERY || prefix != int32_t(id))) {
        const int32_t implied = *lds<int16_t>(sym_at + 2u * uint32_t(prefix) + 2u);
        enter(2, id, uint32_t(prefix), last, implied, [&](uint32_t got) __attribute__((always_inline)) {
          if (!ROUGE) repeat12 += 0x10000u;
          if (at_once)
            enter_step(std::integral_constant<int, 0>{}, id, got, lasts, left, enter_step);
          else
            left = word_of(id, got);
        });
      }
      id += nt;
      s += sym_stride;
      b += nwaves;
      return left;
    };
    auto look_up_block = [&]() __attribute__((always_inline)) {
      const int f = reference_of(b);
      const uint32_t own = s + uint32_t(2 * kPadSymbols) * f;
      const int32_t prefix = *lds<int16_t>(own), last = *lds<int16_t>(own + 2);
      int32_t lasts[DEPTH];
#pragma unroll
      for (int d = 0; !COMPACT && !SHORT && d < DEPTH; ++d) lasts[d] = *lds<int16_t>(own + 4 + 2u * d);
      int32_t left = -1;
      bool match = false;
      if ((int32_t(uint32_t(prefix) << id_bits) | last) >= 0) {
        look_up(2, f, uint32_t(prefix), last, sym_at + 2u * uint32_t(prefix) + 2u, [&](uint32_t got, uint32_t counter) __attribute__((always_inline)) {
          if (at_once)
            look_up_step(std::integral_constant<int, 0>{}, f, id, got, lasts, left, look_up_step);
          else
            left = word_of(id, got);
          if (ROUGE) match = is_match(0, f, counter);
          else if (matching) match12 += is_match(1 - swept, f, counter) ? 0x10000u : 0u;
        });
      }
      if (ROUGE && N == 2) {
        const int of_block = __popcll(__builtin_amdgcn_ballot_w64(match));
        overlap += lane == f ? of_block : 0;
      }
      id += nt;
      s += sym_stride;
      b += nwaves;
      return left;
    };
    // Blocks i..end - 1 of the candidate or of the references: order 2 of each (first), and the orders
    // behind it (more) of what is left, where COMPACT puts that together to full blocks: of the candidate's
    // positions a tenth to a quarter go on behind order 2, of the references' a quarter to a half, but hardly
    // a block is without one.  KEEP: the orders behind it follow later.  `kept`: where the next block is kept.
    auto all_blocks = [&](int end, int& kept, auto&& first, auto&& more) __attribute__((always_inline)) {
      int32_t waiting = -1;  // lanes 0 .. pending - 1: words of blocks before
      int pending = 0;
      auto go_on = [&](int32_t word) __attribute__((always_inline)) {
        if (KEEP) {
          // (a branch: chosen without one, every register of val would be)
          asm volatile("" : "+s"(kept));
          val[kept++] = word;
        } else {
          more(word, 0);
        }
      };
#pragma unroll 1
      for (; i < end; ++i) {
        int32_t word = first();
        if (!deeper || (!COMPACT && !KEEP)) continue;
        const uint64_t going = __builtin_amdgcn_ballot_w64(word >= 0);
        if (COMPACT) {
          // Lanes that go on move behind those waiting, the others behind these (a permutation).
          const int n = __popcll(going);
          const int rank = int(__builtin_amdgcn_mbcnt_hi(uint32_t(going >> 32),
                                                         __builtin_amdgcn_mbcnt_lo(uint32_t(going), 0u)));
          const int place = word >= 0 ? rank : n + lane - rank;
          const int32_t moved = __builtin_amdgcn_ds_permute((place + pending) << 2, word);
          const bool behind = lane >= pending;
          word = behind ? moved : waiting;
          waiting = word;
          pending += n;
          if (pending < kWave) continue;
          waiting = behind ? -1 : moved;
          pending -= kWave;
        }
        go_on(word);
      }
      if (COMPACT && pending > 0) go_on(waiting);
    };
    // KEEP: the orders from `next` on of what is left
    auto kept_blocks = [&](int k, int end, auto&& more) __attribute__((always_inline)) {
      if (next > hi || (dense && !COMPACT)) return;
#pragma unroll 1
      for (; k < end; ++k)
        if (__builtin_amdgcn_ballot_w64(val[k] >= 0)) val[k] = more(val[k], k);
    };
    const auto enter_words = [&](int32_t word, int) __attribute__((always_inline)) { return enter_more(word); };
    if (dense) all_blocks(my_cand_blocks, kept_cand, enter_block, enter_words);
    if (KEEP) kept_blocks(0, kept_cand, enter_words);
    __syncthreads();
    TB_FSTAMP(2 * lo);
    if (dense) {
      i = my_cand_blocks;
      all_blocks(my_blocks, kept, look_up_block, look_up_more);
    }
    if (KEEP) kept_blocks(my_cand_blocks, kept, look_up_more);
    TB_FSTAMP(2 * lo + 1);
  }
  TB_FSTAMP(20);
  const bool lost = *lds<uint32_t>(lost_at);
  if (lost) {
    // Token ids chosen to collide: count by comparing n-grams, without a table.
    __syncthreads();
    if (tid < 16) *lds<uint32_t>(part_at + 4 * tid) = 0u;
    if (ROUGE && tid < kMaxSeqs) *lds<uint32_t>(overlap_at + 4 * tid) = 0u;
    __syncthreads();
    // (pointers from the argument segment again: they need no registers until here)
    const Segment args = (Segment)__builtin_amdgcn_kernarg_segment_ptr();
    const PlainArgs& plain = *(const PlainArgs*)args;
    const char* const cand_row = static_cast<const char*>(plain.cand) + uint64_t(uint32_t(g)) * (uint32_t(cs) * token_bytes);
    const char* const ref_row = static_cast<const char*>(plain.refs) + uint64_t(row0) * (uint32_t(rs) * token_bytes);
    const int32_t* const ref_lens = plain.ref_lens;
    auto token = [&](const char* row, int i) __attribute__((always_inline)) {
      const uint64_t t = wide ? *reinterpret_cast<const uint64_t*>(row + 8 * int64_t(i))
                              : *reinterpret_cast<const uint32_t*>(row + 4 * int64_t(i));
      return t >= uint64_t(a.vocab) ? 0 : int32_t(t);
    };
#pragma unroll 1
    for (int n = ROUGE ? N : 1; n <= N; ++n) {
#pragma unroll 1
      for (int k = tid; k + n <= cand_len; k += nt) {
        // occurrences in row[0 .. len - 1] of the n-gram at candidate position k (at most one is
        // wanted with `once`)
        auto occurrences = [&](const char* row, int len, bool once) __attribute__((always_inline)) {
          int found = 0;
#pragma unroll 1
          for (int i = 0; i + n <= len && !(once && found); ++i) {
            int j = 0;
            while (j < n && token(row, i + j) == token(cand_row, k + j)) ++j;
            found += j == n ? 1 : 0;
          }
          return found;
        };
        if (occurrences(cand_row, k + n - 1, true)) continue;  // not its first occurrence
        const int cc = occurrences(cand_row, cand_len, false);
        int mx = 0;
#pragma unroll 1
        for (int j = 0; j < used; ++j) {
          const int len = min(max(ref_lens[row0 + j], 0), rs);
          const int c = occurrences(
              ref_row + int64_t(j) * rs * token_bytes, len, false);
          mx = max(mx, c);
          if (ROUGE) lds_add(overlap_at + 4u * j, uint32_t(min(cc, c)));
        }
        lds_add(part_at + 4u * uint32_t(n - 1), uint32_t(max(cc - mx, 0)));
        lds_add(part_at + 32u + 4u * uint32_t(n - 1), 1u);
      }
    }
    __syncthreads();
  }

  // wavefront 0: lane n < N owns order n + 1 (statistics out, one logarithm each)
  if (wave == 0) {
    const int c = cand_len;
    if (!ROUGE) {
      // (what the tail reads of the arguments: one request, with the sums)
      // (a word holds the sum of the order in the lower half and, in the upper one, of the next order)
      const uint32_t at = part_at + 4u * uint32_t(lane & 7);
      const uint32_t here = *lds<uint32_t>(at), before = *lds<uint32_t>(lane & 7 ? at - 4u : lost_at);
      const int sum = int((here & 0xFFFFu) + (before >> 16));
      int repeated = 0;  // (lost: the distinct n-grams)
      if (TWO || want_distinct) {
        const uint32_t here = *lds<uint32_t>(at + 32u), before = *lds<uint32_t>(lane & 7 ? at + 28u : lost_at);
        repeated = int((here & 0xFFFFu) + (before >> 16));
      }
      const int best = __builtin_amdgcn_readfirstlane(*lds<int32_t>(closest_at));
      const float brevity = *lds<float>(closest_at + 4);
      int32_t *clipped = a.st.clipped, *total = a.st.total, *closest = a.st.closest;
      void* out = a.out;
      ScoreParams sp;
      sp.N = N;
      sp.smoothing = a.sp.smoothing;
      sp.param = a.sp.param;
      sp.out_bf16 = a.sp.out_bf16;
      asm volatile("" : "+s"(clipped), "+s"(total), "+s"(closest), "+s"(out), "+s"(sp.smoothing),
                   "+s"(sp.param), "+s"(sp.out_bf16));
      const float w = lane_weight(a.sp);
      // (two references: among the sum is every position that is no id, for a counter that nothing was added
      // to stands for one occurrence: those that repeat another's n-gram, and those behind the last one)
      const int tn = max(c - lane, 0), cn = lost ? tn - sum : TWO ? c - (sum - repeated) : sum;
      const float score = bleu_from_stats_wave<int>(cn, tn, c, best, brevity, w, sp);
      if (lane == 0) {
        if (out) store_score(out, g, score, sp.out_bf16);
        closest[g] = best;
      }
      if (lane < N) {
        clipped[int64_t(g) * N + lane] = cn;
        total[int64_t(g) * N + lane] = tn;
        if (want_distinct) a.st.distinct[int64_t(g) * N + lane] = lost ? repeated : tn - repeated;
      }
    } else {
      // lane j = 1..used: reference j - 1.  F is proportional to overlap / (cand + beta^2 ref)
      // n-grams; the best reference is the first one with the largest such quotient.
      const bool ref_lane = lane >= 1 && lane <= used;
      const int ov = ref_lane ? int(*lds<uint32_t>(overlap_at + 4 * ((lane - 1) & (kMaxSeqs - 1)))) : 0;
      const float ct = float(max(c - N + 1, 0)), rt = float(max(my_len - N + 1, 0));
      const float key = (ref_lane && ov > 0) ? float(ov) / __fmaf_rn(a.beta2, rt, ct) : 0.0f;
      if (a.rouge_overlap && lane >= 1 && lane <= R)
        a.rouge_overlap[int64_t(g) * R + lane - 1] = ov;
      int best_j = 1;
      float best_key = __int_as_float(lane_value(__float_as_int(key), 1));
      for (int j = 2; j <= used; ++j) {
        const float kj = __int_as_float(lane_value(__float_as_int(key), j));
        if (kj > best_key) {
          best_key = kj;
          best_j = j;
        }
      }
      const float p = ct > 0.0f ? float(ov) / ct : 0.0f;
      const float r = rt > 0.0f ? float(ov) / rt : 0.0f;
      const float f = (p + r > 0.0f) ? (1.0f + a.beta2) * p * r / (r + a.beta2 * p) : 0.0f;
      if (lane == best_j) {
        store_score(a.rouge_prf, int64_t(g) * 3 + 0, p, a.sp.out_bf16);
        store_score(a.rouge_prf, int64_t(g) * 3 + 1, r, a.sp.out_bf16);
        store_score(a.rouge_prf, int64_t(g) * 3 + 2, f, a.sp.out_bf16);
        if (a.rouge_best) a.rouge_best[g] = best_j - 1;
      }
    }
  }
  TB_FSTAMP(21);
}

// (The scalar-register cap keeps two 1024-thread workgroups on a compute unit: eight wavefronts per
// SIMD need at most 80 scalar registers each on this hardware.)
template <int BLOCKS, bool KEEP, Mode MODE>
__global__ __launch_bounds__(1024, 8) __attribute__((amdgpu_num_sgpr(80)))
void fused_kernel(const void* cand, const int32_t* cand_lens, const void* refs,
                  const int32_t* ref_lens, const int32_t* ref_count, const int32_t* ref_offsets,
                  uint32_t cand_shape, uint32_t ref_shape, FusedArgs by_value) {
  fused_group<BLOCKS, KEEP, MODE, false>(cand, cand_lens, refs, ref_lens, ref_count, ref_offsets, cand_shape,
                                  ref_shape);
}
// The same where a compute unit has one workgroup at a time: its wavefronts, four per SIMD, may have all
// scalar registers (25 to 50 of them move to lanes of a vector register and back otherwise) and 128
// vector registers (with 64, the values of 24 blocks and the sweep's do not fit).  us, plans of few
// blocks: 3 x 124 with three references 9.84 -> 9.41, 142 x 93 with eight 10.5 -> 10.3, 16 x 256 6.03 -> 5.98;
// of 8 to 16: 1 to 3 % (128 x 8192 34.2 -> 33.8, 128 x 2500 with four references 24.1 -> 23.4); of 24, with three
// references or more, a fifth (128 x 5000 with three 53.8 -> 45.1, 700 of them 155 -> 128, 800 x 2400 with eight
// 176 -> 149).
template <int BLOCKS, bool KEEP, Mode MODE>
__global__ __launch_bounds__(1024, 4)
void fused_kernel_alone(const void* cand, const int32_t* cand_lens, const void* refs,
                        const int32_t* ref_lens, const int32_t* ref_count, const int32_t* ref_offsets,
                        uint32_t cand_shape, uint32_t ref_shape, FusedArgs by_value) {
  fused_group<BLOCKS, KEEP, MODE, true>(cand, cand_lens, refs, ref_lens, ref_count, ref_offsets, cand_shape,
                                  ref_shape);
}

// The kernels read the struct behind the plain arguments, and some of these again, from the argument
// segment, where arguments lie like the members of a struct.
template <typename... Args>
constexpr size_t last_argument_at(void (*)(Args...)) {
  size_t end = 0, at = 0;
  ((at = (end + alignof(Args) - 1) / alignof(Args) * alignof(Args), end = at + sizeof(Args)), ...);
  return at;
}
static_assert(last_argument_at(decltype(&fused_kernel<2, false, kRouge>){}) == kRegisterArgs);
static_assert(last_argument_at(decltype(&fused_kernel_alone<2, false, kRouge>){}) == kRegisterArgs);

int log2_ceil(int64_t v) {
  int b = 0;
  while ((int64_t(1) << b) < v) ++b;
  return b;
}

template <int BLOCKS, bool KEEP, Mode MODE, bool ALONE>
hipError_t launch_shape(const Problem& pb, const FusedArgs& a, const FusedPlan& plan, hipStream_t s) {
  const auto kernel = [] {  // (the other one is not to be instantiated)
    if constexpr (ALONE)
      return fused_kernel_alone<BLOCKS, KEEP, MODE>;
    else
      return fused_kernel<BLOCKS, KEEP, MODE>;
  }();
  hipError_t e = grant_dynamic_lds(reinterpret_cast<const void*>(kernel), plan.lds_bytes);
  if (e != hipSuccess) return e;
  const uint32_t cand_shape = uint32_t(pb.cand_stride) | uint32_t(pb.R) << 16 |
                              uint32_t(log2_ceil(plan.threads / kWave)) << 24;
  const uint32_t ref_shape = uint32_t(pb.ref_stride) | uint32_t(pb.N) << 16 |
                             uint32_t(pb.tok64 ? 1 : 0) << 24;
  hipLaunchKernelGGL(kernel, dim3(uint32_t(pb.B)), dim3(plan.threads), plan.lds_bytes, s, pb.cand,
                     pb.cand_len, pb.refs, pb.ref_len, pb.ref_count, pb.ref_offsets, cand_shape,
                     ref_shape, a);
  return hipGetLastError();
}
template <int BLOCKS, bool KEEP, bool ALONE>
hipError_t launch_mode(const Problem& pb, const FusedArgs& a, const FusedPlan& plan, hipStream_t s) {
  if (a.rouge_prf) {
    if constexpr (!KEEP) {
      if (pb.N <= 2) return launch_shape<BLOCKS, KEEP, kRouge, ALONE>(pb, a, plan, s);
    }
    return launch_shape<BLOCKS, KEEP, kRougeLonger, ALONE>(pb, a, plan, s);
  }
  return pb.R == 1   ? launch_shape<BLOCKS, KEEP, kOneReference, ALONE>(pb, a, plan, s)
         : pb.R == 2 ? launch_shape<BLOCKS, KEEP, kTwoReferences, ALONE>(pb, a, plan, s)
                     : launch_shape<BLOCKS, KEEP, kReferences, ALONE>(pb, a, plan, s);
}
template <int BLOCKS, bool KEEP>
hipError_t launch_keep(const Problem& pb, const FusedArgs& a, const FusedPlan& plan, hipStream_t s) {
  if (fused_alone(pb.B, plan)) return launch_mode<BLOCKS, KEEP, true>(pb, a, plan, s);
  // (plans for shared units have two blocks or more)
  if constexpr (BLOCKS > 1) return launch_mode<BLOCKS, KEEP, false>(pb, a, plan, s);
  return hipErrorInvalidValue;
}
template <int BLOCKS>
hipError_t launch_blocks(const Problem& pb, const FusedArgs& a, const FusedPlan& plan, hipStream_t s) {
  return plan.keep ? launch_keep<BLOCKS, true>(pb, a, plan, s)
                   : launch_keep<BLOCKS, false>(pb, a, plan, s);
}

constexpr size_t kLdsUnit = 1280;  // LDS is handed out in units of this size

}  // namespace

// One workgroup a unit: no more of them than units, or LDS for one only.
bool fused_alone(int64_t B, const FusedPlan& plan) {
  return B <= 256 || plan.lds_bytes > kLdsBudget / 2;
}

bool fused_path_takes(int64_t cand_stride, int64_t ref_stride, int R, int bits) {
  if (R + 1 > kMaxSeqs) return false;
  const int64_t cap = cand_stride + int64_t(R) * ref_stride;
  if (cap > 12 * 1024 || cand_stride > 4096 || ref_stride > 65535) return false;
  if (bits > 31 || (uint64_t(cand_stride) << bits) > 0xFFFFFFFFull) return false;
  int64_t slots = 256;
  while (slots * 3 < cand_stride * 4) slots *= 2;
  const int64_t nwaves = cap <= 1024 ? 4 : cap <= 2048 ? 8 : 16;
  const int64_t list = ((R * ref_stride + nwaves - 1) / nwaves + kWave - 1) / kWave * kWave * nwaves;
  const int64_t bytes = slots * 6 + ((cand_stride * ((R + 2) / 2) * 4 + 15) & ~int64_t(15)) +
                        cand_stride * 4 + (((cap + 4) * (bits <= 16 ? 2 : 4) + 3) & ~int64_t(3)) +
                        list * 4;
  return bytes + 1024 <= kLdsBudget;
}

namespace {

// Passes of a plan.  Fills in pass_ends and the key widths; false: the key is too wide.
enum Passes {
  kTogether,         // all orders share a table
  kFirstApart,       // order 1 on its own, then all others
  kStretches,        // orders 1 to 4, 5 to 7, 8: a table for each stretch
  kFirstStretches,   // order 1 on its own, then 2 to 4, 5 to 7, 8
  kPairs,
  kSingle,           // every order on its own
};
bool set_passes(int passes, int N, int bits, FusedPlan* plan, int* orders_per_pass) {
  FusedPlan& p = *plan;
  static const uint32_t kEnds[6] = {0x90u, 0x92u, 0x90u, 0x92u, 0x154u, ~0u};  // bit n: a stretch ends with order n
  p.pass_ends = (N == 1 || (kEnds[passes] & 2u)) ? 1u : 0u;
  if (passes <= kFirstApart) p.pass_ends |= 2u;
  for (int n = 2; n <= N; ++n) {
    int end = n;
    while (end < N && !((kEnds[passes] >> end) & 1u)) ++end;
    p.pass_ends |= uint32_t(end) << (4 * (n - 1));
  }
  static const int kOrders[6] = {8, 7, 4, 3, 2, 1};
  const int most = (passes == kFirstApart || passes == kFirstStretches) && N > 1 ? N - 1 : N;
  *orders_per_pass = kOrders[passes] < most ? kOrders[passes] : most;
  const int tag_bits = log2_ceil(*orders_per_pass);
  p.later_payload = 2 * p.id_bits;
  p.later_key_bits = p.later_payload + tag_bits;
  p.first_payload = p.first_key_bits = bits;
  if (!(p.pass_ends & 1u)) {
    p.first_payload = bits > p.later_payload ? bits : p.later_payload;
    p.first_key_bits = p.first_payload + tag_bits;
  }
  p.keep = N > 4 || (passes >= kPairs && N > 2);  // (more than one stretch above order 1)
  return p.first_key_bits <= 32 && p.later_key_bits <= 32;
}

}  // namespace

// What the choice weighs (all plans of 113 shapes timed, 8 to 4096 groups of 24 to 4096 tokens with one
// to eight references, one to four orders; on average the choice is 1.4 % behind the best plan of a
// shape, more than a tenth behind in five of them):
//   * A pass costs its barriers, its sums, clearing the table and the block loop again, but has the
//     counters of its orders only.  Up to four workgroups on a unit, all at once, want their exact share
//     of LDS, whatever passes that takes (1024 x 2048: pairs, four a unit, 25.4 us; orders 1 to 4
//     together, three a unit, 33.3).  Where there are more, fewer passes win with down to half as many of
//     them side by side (4096 x 512 with two references: pairs, sixteen a unit, 32.0; orders 1 to 4 together, eight,
//     28.0; 2493 x 711 with two, ten and seven a unit, 34.3 and 30.4).  Every order on its own only where nothing
//     else fits.
//   * A table that is nearly full costs more than anything else: probe sequences of the wavefront's
//     slowest lane grow from 1 to 4 requests between a quarter and three quarters.  More than twelve
//     slots a position, six for one order, cost more to clear than they save (38 x 1425 with three
//     references, one order: 7.2 -> 6.9 us).
//   * 32 wavefronts a unit hide latency (16 take 512 x 1024 with four references from 17.8 to 19.6 us);
//     a workgroup with fewer blocks than wavefronts idles, and with two blocks or less per wavefront its
//     prologue outweighs them.
//   * More than 12 to 16 blocks a wavefront are short of registers where workgroups share a unit (of 24, 28 to
//     54 vector registers go to scratch): these get more wavefronts, and the LDS of as many workgroups as then
//     fit (5340 x 242 with six references, 17 blocks, 76.8 us; 9 blocks of four wavefronts 51.0; 13 blocks and
//     more in 300 drawn shapes: 1.09 of the speed).  Two wavefronts, and four with more than one order, gain from 13
//     blocks on (1.13 and 1.07); four with one order, one, and eight with more than two orders from 17 on (13 to
//     16: 0.9 to 1.0 with twice the wavefronts); eight with one or two orders never do (0.97).  Two workgroups of
//     16 wavefronts keep up to 24 blocks: they are faster with scratch than one a unit without it (90 shapes: 1.23).
bool plan_fused(int64_t B, int64_t cand_stride, int64_t ref_stride, int R, int N, int bits,
                bool rouge, FusedPlan* plan) {
  if (R + 1 > kMaxSeqs || cand_stride > 12288 || ref_stride > 65535 || bits > 31) return false;
  const int64_t blocks =
      (cand_stride + kWave - 1) / kWave + R * ((ref_stride + kWave - 1) / kWave);
  if (blocks > kMaxBlocks * 16) return false;
  FusedPlan& p = *plan;
  p.id_bits = cand_stride > 1 ? log2_ceil(cand_stride) : 1;
  p.array_bytes = (int(cand_stride) * 4 + 15) & ~15;
  const int order_fields = rouge || R <= 2 ? R : R + 1;
  const size_t sym_bytes = (size_t(blocks * kWave + (R + 1) * kPadSymbols) * 2 + 15) & ~size_t(15);
  const int resident = int(B > 256 * 32 ? 32 : (B + 255) / 256);  // workgroups a unit gets, if they fit

  // r workgroups on a unit; the table may be half full if no n-gram repeats (three quarters: full)
  auto fits = [&](int passes, int r, bool full) {
    int orders;
    if (!set_passes(passes, N, bits, plan, &orders)) return false;
    int waves = 1;
    if (resident <= 1) {  // the chip is not full: a wavefront for (nearly) each block
      while (waves < 16 && 4 * waves < 3 * blocks) waves *= 2;
    } else {
      while (waves < 16 && 2 * waves <= 32 / r && blocks > waves * (waves < 4 ? 2 : waves < 8 ? 3 : 4))
        waves *= 2;
    }
    // blocks a wavefront takes at most (see above), and workgroups that the wavefronts then leave room for
    auto most = [&]() -> int64_t {
      if (r < 2 || (waves == 8 && N <= 2)) return kMaxBlocks;
      return waves == 2 || (waves == 4 && N > 1) ? 12 : 16;
    };
    while (waves < 16 && blocks > most() * waves) waves *= 2;
    if (r > 32 / waves) r = 32 / waves;
    // All orders of a pass together enter at most as many n-grams as the candidate has positions.
    const int64_t entries = cand_stride;
    const int widest = p.first_key_bits > p.later_key_bits ? p.first_key_bits : p.later_key_bits;
    int lg_min = 6;
    while ((int64_t(full ? 3 : 2) << lg_min) < 4 * entries) ++lg_min;
    // bits for the probe count.  A sequence that reaches the largest count sends the whole
    // workgroup to the loop without a table, so ordinary tokens must not get there.  Every bucket
    // further is reached by an eighth of the sequences at half load, by 0.43 of them at three
    // quarters (look-ups and insertions of 128 x 8192 and 64 x 6144 Zipf-distributed tokens counted
    // on the CPU): fifteen buckets were reached by 1e-9 of the groups and by one in twenty, sixty-three
    // would be by 1e-19.
    while (32 - widest + lg_min - 2 - p.id_bits < (full ? 6 : 4)) ++lg_min;
    int lg = lg_min;
    while ((int64_t(1) << lg) < (N == 1 ? 6 : 12) * entries) ++lg;
    const bool listed = N > 2 && blocks > kApartBlocks * waves && (rouge || R > 2);  // (see LISTED)
    const size_t sums = sums_bytes(rouge) + (listed ? size_t(blocks + 15) & ~size_t(15) : 0);
    const size_t share = size_t(kLdsBudget) / r / kLdsUnit * kLdsUnit;
    const size_t counters = size_t(((rouge ? 1 : orders) * order_fields + 1) / 2) * p.array_bytes;
    for (; lg >= lg_min; --lg) {
      const size_t front = (size_t(4) << lg) + counters;
      p.lds_bytes = front + sym_bytes + sums;
      if (p.lds_bytes > share) continue;
      p.threads = waves * kWave;
      p.blocks = int((blocks + waves - 1) / waves);
      p.log2_slots = lg;
      p.table_and_counters = int(front / 16);
      p.off_sym = uint32_t(front);
      p.off_sums = uint32_t(front + sym_bytes);
      return true;
    }
    return false;
  };
  for (int full = 0; full < 2; ++full) {
    auto some_fits = [&](int passes, int r) {  // (up to order 4 there is one stretch)
      return (N > 4 || passes < kStretches || passes > kFirstStretches) && fits(passes, r, full);
    };
    int r = resident < 1 ? 1 : resident;
    if (r > 4) {
      const int shares[3] = {r, r * 7 / 10, r / 2};
      for (int passes = kTogether; passes <= kPairs; ++passes)
        for (int share : shares) {
          // (Counters of five orders and more with three references or more take so much LDS that a table
          // for each stretch is better than fewer workgroups: 3615 x 26 with 16, eight orders, 39.4 -> 30.5 us.)
          if (N > 4 && R > 2 && passes <= kFirstApart && share < r) break;
          if (some_fits(passes, share)) return true;
        }
      r = r / 2 - 1;
    }
    for (; r >= 1; --r)
      for (int passes = kTogether; passes <= (r > 1 ? kPairs : kSingle); ++passes)
        if (some_fits(passes, r)) return true;
  }
  return false;
}

hipError_t launch_fused(const Problem& pb, const FusedPlan& plan, const StatPtrs& st,
                        const ScoreParams& sp, void* out_bleu_or_null, bool want_distinct,
                        hipStream_t s, const RougeOut* rouge) {
  FusedArgs a;
  a.status = pb.status;
  a.vocab = pb.vocab;
  a.ref_rows = pb.ref_rows;
  a.st = st;
  a.sp = sp;
  a.out = out_bleu_or_null;
  a.rouge_prf = rouge ? rouge->prf : nullptr;
  a.rouge_overlap = rouge ? rouge->overlap : nullptr;
  a.rouge_best = rouge ? rouge->best : nullptr;
  a.beta2 = rouge ? rouge->beta2 : 1.0f;
  a.pass_ends = plan.pass_ends;
  a.log2_slots = plan.log2_slots;
  a.id_bits = plan.id_bits;
  a.first_payload = plan.first_payload;
  a.first_key_bits = plan.first_key_bits;
  a.later_payload = plan.later_payload;
  a.later_key_bits = plan.later_key_bits;
  a.array_bytes = plan.array_bytes;
  a.want_distinct = want_distinct ? 1 : 0;
  a.table_and_counters = plan.table_and_counters;
  a.off_sym = plan.off_sym;
  a.off_sums = plan.off_sums;
  const int by_threads = 2048 / plan.threads;
  const int by_lds = int(size_t(kLdsBudget) / plan.lds_bytes);
  const int resident = 256 * (by_threads < by_lds ? by_threads : (by_lds < 1 ? 1 : by_lds));
  a.progress_priority = pb.B <= 2 * resident ? 1 : 0;
  if (plan.blocks <= 1) return launch_blocks<1>(pb, a, plan, s);
  if (plan.blocks <= 2) return launch_blocks<2>(pb, a, plan, s);
  if (plan.blocks <= 3) return launch_blocks<3>(pb, a, plan, s);
  if (plan.blocks <= 4) return launch_blocks<4>(pb, a, plan, s);
  if (plan.blocks <= 5) return launch_blocks<5>(pb, a, plan, s);
  if (plan.blocks <= 6) return launch_blocks<6>(pb, a, plan, s);
  if (plan.blocks <= 8) return launch_blocks<8>(pb, a, plan, s);
  if (plan.blocks <= 12) return launch_blocks<12>(pb, a, plan, s);
  if (plan.blocks <= 16) return launch_blocks<16>(pb, a, plan, s);
  return launch_blocks<kMaxBlocks>(pb, a, plan, s);
}

}  // namespace tb
