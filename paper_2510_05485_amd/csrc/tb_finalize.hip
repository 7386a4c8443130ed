// Score assembly from the integer statistics (paper Section 3.4): per-sentence scores, and the
// corpus variant that sums numerators, denominators and lengths over the batch first.
#include <type_traits>

#include "tb_kernels.h"
#include "tb_score.h"

namespace tb {

struct FinalArgs {
  Problem pb;
  StatPtrs st;
  ScoreParams sp;
  void* out;  // fp32 or bfloat16 scores (sp.out_bf16)
  const int32_t* overflow;  // [B] or null: groups whose dictionary overflowed score NaN
};

// One lane per sentence.
__global__ __launch_bounds__(256) void sentence_score_kernel(FinalArgs a) {
  const Problem& pb = a.pb;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pb.B) return;
  const int c = clamped_len(pb.cand_len[i], pb.cand_stride, pb.status);
  const RefRows rr = ref_rows(pb, i, true);
  const int r = closest_ref_len(c, pb.ref_len + rr.row0, rr.used, pb.ref_stride, pb.status);
  a.st.closest[i] = r;
  int cl[8], to[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    cl[n] = (n < pb.N) ? a.st.clipped[int64_t(i) * pb.N + n] : 0;
    to[n] = (n < pb.N) ? a.st.total[int64_t(i) * pb.N + n] : 0;
  }
  // a group whose statistics are not trustworthy must not pass for a reward
  const bool spoilt = a.overflow && a.overflow[i] != 0;
  store_score(a.out, i, spoilt ? __int_as_float(0x7FC00000) : bleu_from_stats<int>(cl, to, c, r, a.sp),
              a.sp.out_bf16);
}

// A single workgroup strides over the batch and reduces the 2N+2 integer sums; wavefront 0 forms
// the corpus score, one order per lane.
//
// Bound by latency: B * (4N + 8) bytes that other XCDs have just written come back through one
// compute unit.  So the statistics of four sentences per thread are requested together (one memory
// round trip per 4096 sentences), the totals are recomputed from the lengths instead of read, and
// KNOWN_CLOSEST (the per-sentence pass has stored the closest reference lengths, as the fused
// kernel does) reads them instead of walking the references again.  Measured at B = 4096, N = 4,
// R = 2: 25 us with a round trip per field and sentence.
// FOUR_ORDERS: N = 4, one 16-byte request per sentence.  Sum: int32_t where the host knows that no sum
// leaves it (B times the longer stride; not for counts that the caller brings), else int64_t, added up
// across lanes 20 bits at a time.  With sums of 64 bits everywhere and a loop over the wavefronts' parts
// in LDS, which waited for each, the kernel took 5.4 us instead of 3.5 (2000 x 64 corpus BLEU 12.4 ->
// 10.5, 1024 x 2048 35.0 -> 33.0).
template <bool KNOWN_CLOSEST, bool FOUR_ORDERS, typename Sum>
__global__ __launch_bounds__(1024) void corpus_kernel(FinalArgs a, int write_score) {
  constexpr int kUnroll = 4, kOrders = FOUR_ORDERS ? 4 : 8;
  struct __attribute__((packed, aligned(4))) Quad {  // the caller's array may be 4-byte aligned
    int32_t v[4];
  };
  constexpr int kRows = 2 * kOrders + 4;  // sums, four (16 lanes each) to a register of wavefront 0
  __shared__ int32_t part[kRows][16];
  __shared__ int s_spoilt;
  const Problem& pb = a.pb;
  const int tid = threadIdx.x, nt = blockDim.x, N = pb.N;
  if (tid == 0) s_spoilt = 0;
  // clipped, total, candidate lengths, closest reference lengths
  Sum acc[2 * kOrders + 2];
#pragma unroll
  for (int k = 0; k < 2 * kOrders + 2; ++k) acc[k] = 0;
  bool spoilt = false;  // some group's dictionary overflowed
  for (int base = 0; base < pb.B; base += kUnroll * nt) {
    int c[kUnroll], r[kUnroll], cl[kUnroll][kOrders];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {  // (clamped rows: unconditional loads, masked below)
      const int i = min(base + u * nt + tid, pb.B - 1);
      c[u] = pb.cand_len[i];
      if (KNOWN_CLOSEST) r[u] = a.st.closest[i];
      const int32_t* row = a.st.clipped + int64_t(i) * N;
      if (FOUR_ORDERS) {
        const Quad q = *reinterpret_cast<const Quad*>(row);
#pragma unroll
        for (int n = 0; n < 4; ++n) cl[u][n] = q.v[n];
      } else {
#pragma unroll
        for (int n = 0; n < kOrders; ++n) cl[u][n] = row[min(n, N - 1)];
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int i = base + u * nt + tid;
      if (i >= pb.B) continue;
      c[u] = clamped_len(c[u], pb.cand_stride, pb.status);
      if (!KNOWN_CLOSEST) {
        const RefRows rr = ref_rows(pb, i, true);
        r[u] = closest_ref_len(c[u], pb.ref_len + rr.row0, rr.used, pb.ref_stride, pb.status);
        a.st.closest[i] = r[u];
        spoilt |= a.overflow && a.overflow[i] != 0;
      }
#pragma unroll
      for (int n = 0; n < kOrders; ++n) {
        acc[n] += cl[u][n];
        acc[kOrders + n] += max(c[u] - n, 0);
      }
      acc[2 * kOrders] += c[u];
      acc[2 * kOrders + 1] += r[u];
    }
  }
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  if (!KNOWN_CLOSEST) {
    __syncthreads();  // s_spoilt is cleared
    if (spoilt) s_spoilt = 1;
  }
  Sum tot[kRows / 4] = {};  // lane 16 q + 15: sum 4 k + q
  constexpr int kStep = sizeof(Sum) == 4 ? 32 : 20;
#pragma unroll 1
  for (int shift = 0; shift < int(8 * sizeof(Sum)); shift += kStep) {
    if (shift) __syncthreads();  // the parts before have been read
#pragma unroll
    for (int k = 0; k < 2 * kOrders + 2; ++k) {
      const int v = wave_inclusive_scan(
          sizeof(Sum) == 4 ? int(acc[k]) : int((int64_t(acc[k]) >> shift) & 0xFFFFF));
      if (lane == kWave - 1) part[k][wave] = v;
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int k = 0; k < kRows / 4; ++k) {
        const int v = row_inclusive_scan(part[min(4 * k + lane / 16, 2 * kOrders + 1)][lane & 15]);
        tot[k] += Sum(sizeof(Sum) == 4 ? int64_t(v) : int64_t(uint32_t(v)) << shift);
      }
    }
  }
  if (wave == 0) {
    const int row = lane / 16;
    if ((lane & 15) == 15) {
#pragma unroll
      for (int k = 0; k < kOrders / 4; ++k) {
        const int n = 4 * k + row;
        if (n < N) {
          a.st.corpus[n] = tot[k];
          a.st.corpus[N + n] = tot[kOrders / 4 + k];
        }
      }
      if (row < 2) a.st.corpus[2 * N + row] = tot[kRows / 4 - 1];
    }
    if (write_score) {
      // the value that lane `from` holds, in every lane (a lane may ask for another one)
      auto value_of = [&](Sum v, int from) {
        const uint64_t w = uint64_t(int64_t(v));
        const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(4 * from, int(uint32_t(w))));
        if (sizeof(Sum) == 4) return Sum(int32_t(lo));
        const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(4 * from, int(uint32_t(w >> 32))));
        return Sum(uint64_t(hi) << 32 | lo);
      };
      const int from = 16 * (lane & 3) + 15;  // lane n: order n + 1
      Sum cn = value_of(tot[0], from), tn = value_of(tot[kOrders / 4], from);
      if (!FOUR_ORDERS) {
        const Sum cn1 = value_of(tot[1], from), tn1 = value_of(tot[kOrders / 4 + 1], from);
        cn = lane & 4 ? cn1 : cn;
        tn = lane & 4 ? tn1 : tn;
      }
      const Sum c = value_of(tot[kRows / 4 - 1], 15), r = value_of(tot[kRows / 4 - 1], 31);
      const float brevity = expf(1.0f - float(r) / float(c));
      const float score = bleu_from_stats_wave<Sum>(cn, tn, c, r, brevity, lane_weight(a.sp), a.sp);
      if (lane == 0)
        store_score(a.out, 0, s_spoilt ? __int_as_float(0x7FC00000) : score, a.sp.out_bf16);
    }
  }
}

// ROUGE-N from the overlap counts of the GLOBAL path, one lane per candidate: precision, recall
// and F against every reference in use; the best reference is the first one with the largest
// overlap / (candidate n-grams + beta^2 * reference n-grams), to which F is proportional (the
// same single-precision quotient as the fused kernel forms: both paths choose alike).
struct RougeFinalArgs {
  Problem pb;
  ScoreParams sp;
  const int32_t* overlap;   // [B, R] from the count pass
  void* prf;                // [B, 3]
  int32_t* overlap_out;     // [B, R] caller's array, or null (then `overlap` is the caller's)
  int32_t* best;            // [B] or null
  float beta2;
};

__global__ __launch_bounds__(256) void rouge_score_kernel(RougeFinalArgs a) {
  const Problem& pb = a.pb;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pb.B) return;
  const int N = pb.N, R = pb.R;
  const RefRows rr = ref_rows(pb, i, true);
  const int used = rr.used;
  const int c = clamped_len(pb.cand_len[i], pb.cand_stride, pb.status);
  const float ct = float(max(c - N + 1, 0));
  int best_j = 0;
  float best_key = -1.0f, best_rt = 0.0f;
  int best_ov = 0;
  for (int j = 0; j < R; ++j) {
    const int ov = j < used ? a.overlap[int64_t(i) * R + j] : 0;
    if (a.overlap_out) a.overlap_out[int64_t(i) * R + j] = ov;
    if (j >= used) continue;
    const int len = clamped_len(pb.ref_len[rr.row0 + j], pb.ref_stride, pb.status);
    const float rt = float(max(len - N + 1, 0));
    const float key = ov > 0 ? float(ov) / __fmaf_rn(a.beta2, rt, ct) : 0.0f;
    if (key > best_key) {
      best_key = key;
      best_j = j;
      best_rt = rt;
      best_ov = ov;
    }
  }
  const float p = ct > 0.0f ? float(best_ov) / ct : 0.0f;
  const float r = best_rt > 0.0f ? float(best_ov) / best_rt : 0.0f;
  const float f = (p + r > 0.0f) ? (1.0f + a.beta2) * p * r / (r + a.beta2 * p) : 0.0f;
  store_score(a.prf, int64_t(i) * 3 + 0, p, a.sp.out_bf16);
  store_score(a.prf, int64_t(i) * 3 + 1, r, a.sp.out_bf16);
  store_score(a.prf, int64_t(i) * 3 + 2, f, a.sp.out_bf16);
  if (a.best) a.best[i] = best_j;
}

hipError_t launch_rouge_finalize(const Problem& pb, const ScoreParams& sp, const int32_t* overlap,
                                 const RougeOut& out, hipStream_t s) {
  RougeFinalArgs a;
  a.pb = pb;
  a.sp = sp;
  a.overlap = overlap;
  a.prf = out.prf;
  a.overlap_out = (out.overlap && out.overlap != overlap) ? out.overlap : nullptr;
  a.best = out.best;
  a.beta2 = out.beta2;
  hipLaunchKernelGGL(rouge_score_kernel, dim3((pb.B + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize(const Problem& pb, const StatPtrs& st, const ScoreParams& sp,
                           bool sentence_scores, bool corpus_sums, bool corpus_score,
                           void* out_bleu, hipStream_t s, const int32_t* overflow,
                           bool known_closest, bool own_counts) {
  FinalArgs a;
  a.pb = pb;
  a.st = st;
  a.sp = sp;
  a.out = out_bleu;
  a.overflow = overflow;
  if (sentence_scores) {
    const int blocks = (pb.B + 255) / 256;
    hipLaunchKernelGGL(sentence_score_kernel, dim3(blocks), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (corpus_sums || corpus_score) {
    const int score = corpus_score ? 1 : 0;
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, s, a, score);
    };
    const int64_t longer = pb.cand_stride > pb.ref_stride ? pb.cand_stride : pb.ref_stride;
    const bool narrow = own_counts && pb.B * longer < (int64_t(1) << 31);
    auto choose = [&](auto known, auto four) {
      constexpr bool k = decltype(known)::value, f = decltype(four)::value;
      narrow ? launch(corpus_kernel<k, f, int32_t>) : launch(corpus_kernel<k, f, int64_t>);
    };
    auto choose_orders = [&](auto known) {
      pb.N == 4 ? choose(known, std::true_type{}) : choose(known, std::false_type{});
    };
    if (known_closest || sentence_scores)
      choose_orders(std::true_type{});
    else
      choose_orders(std::false_type{});
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace tb
