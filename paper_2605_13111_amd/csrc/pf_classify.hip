// Offline tri-pattern head classification (Sec. 4.1; pre-processing and harmonic folding as in the appendix
// paragraph on the FFT analysis stage), then a vote per head.
// All arithmetic is fp64: the decisions (thresholds, peak bin) are taken in the precision a host implementation
// would use.  Three kernels share the steps:
//   pf_classify_batch_kernel   sequences of 4 to 72 frames (the paper analyses 69): a workgroup's sequences side by side in LDS, the
//                              spectra of 16 at a time as a matrix product on the fp64 matrix cores
//   pf_classify_rounds_kernel  73 to 256 frames, and some shorter ones in launches of medium size: the same products, 16 sequences at a time
//                              through LDS
//   pf_classify_kernel         launches of few sequences, and the longest (their tables do not fit beside 16 sequences in LDS): one workgroup
//                              per sequence, a direct DFT
#include <hip/hip_runtime.h>
#include <math.h>
#include <type_traits>
#include "pf_internal.h"

constexpr int CLS_THREADS = 256;
constexpr int CLS_MAX_HIST = 1024;      // longest historical sequence (frames)
constexpr int CLS_HARMONICS = 4;        // harmonics folded onto a fundamental, weights 1/j
constexpr double CLS_TIE_REL = 1e-9;    // folded scores this close count as equal: the lowest bin wins

struct ClassifyParams {
  const float *logits;                  // [n_prompts][n_heads][n_hist]
  int32_t *prompt_type;                 // [n_prompts][n_heads]
  double *prompt_period;                // [n_prompts][n_heads] or null
  int n_hist;
  double alpha, beta;
};

__device__ __forceinline__ double block_sum(double v, double *s_red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  __syncthreads();
  if (lane == 0) s_red[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < CLS_THREADS / 64; ++w) t += s_red[w];
  return t;
}

__global__ __launch_bounds__(CLS_THREADS) void pf_classify_kernel(ClassifyParams P) {   // one workgroup per (prompt, head) sequence
  __shared__ double s_a[CLS_MAX_HIST];           // the sequence, then the pre-processed difference
  __shared__ double s_cos[CLS_MAX_HIST], s_sin[CLS_MAX_HIST];
  __shared__ double s_amp[CLS_MAX_HIST / 2 + 1];
  __shared__ double s_score[CLS_MAX_HIST / 2 + 1];
  __shared__ double s_red[CLS_THREADS / 64];
  __shared__ int s_k;
  const int tid = threadIdx.x;
  const int n = P.n_hist;
  const float *a = P.logits + (size_t)blockIdx.x * n;

  // ---- sign rates and mean of the raw sequence ----
  double cnt = 0.0, sum = 0.0;
  for (int t = tid; t < n; t += CLS_THREADS) {
    const double v = (double)a[t];
    s_a[t] = v;
    cnt += v > 0.0 ? 1.0 : 0.0;
    sum += v;
  }
  const double n_pos = block_sum(cnt, s_red);
  const double total = block_sum(sum, s_red);
  const double r_pos = n_pos / (double)n, r_neg = 1.0 - r_pos;
  int type = -1;
  double period = INFINITY;
  if (r_pos >= P.alpha) type = PF_ANCHOR;
  else if (r_neg >= P.alpha) type = PF_VEIL;
  if (type < 0) {                                  // uniform over the workgroup
    // ---- dominant period: difference, mean removal, Hann window, spectrum, harmonic folding ----
    const int N = n - 1;
    if (N >= 3) {
      __syncthreads();
      double dsum = 0.0;
      double d_mine[CLS_MAX_HIST / CLS_THREADS];
      for (int m = tid, i = 0; m < N; m += CLS_THREADS, ++i) {
        d_mine[i] = s_a[m + 1] - s_a[m];
        dsum += d_mine[i];
      }
      const double dmean = block_sum(dsum, s_red) / (double)N;   // (the barriers inside also order the reads above)
      for (int m = tid, i = 0; m < N; m += CLS_THREADS, ++i) {
        const double w = 0.5 - 0.5 * cospi(2.0 * (double)m / (double)(N - 1));
        s_a[m] = (d_mine[i] - dmean) * w;
        double sn, cs;
        sincospi(2.0 * (double)m / (double)N, &sn, &cs);
        s_cos[m] = cs;
        s_sin[m] = sn;
      }
      __syncthreads();
      const int nb = N / 2;
      for (int k = tid; k <= nb; k += CLS_THREADS) {
        double re = 0.0, im = 0.0;
        int j = 0;                                 // (k * m) mod N
        for (int m = 0; m < N; ++m) {
          re += s_a[m] * s_cos[j];
          im -= s_a[m] * s_sin[j];
          j += k;
          if (j >= N) j -= N;
        }
        s_amp[k] = sqrt(re * re + im * im);
      }
      __syncthreads();
      double best = 0.0;
      for (int k = 1 + tid; k <= nb; k += CLS_THREADS) {
        double sc = 0.0;
        for (int h = 1; h <= CLS_HARMONICS; ++h)
          if (h * k <= nb) sc += s_amp[h * k] / (double)h;
        s_score[k] = sc;
        best = fmax(best, sc);
      }
      // maximum over the workgroup, then the lowest bin within the tie band
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) best = fmax(best, __shfl_down(best, o, 64));
      __syncthreads();
      if ((tid & 63) == 0) s_red[tid >> 6] = best;
      if (tid == 0) s_k = 0x7fffffff;
      __syncthreads();
      best = fmax(fmax(s_red[0], s_red[1]), fmax(s_red[2], s_red[3]));
      if (best > 0.0 && isfinite(best)) {
        int kmin = 0x7fffffff;
        for (int k = 1 + tid; k <= nb; k += CLS_THREADS)
          if (s_score[k] >= best * (1.0 - CLS_TIE_REL)) { kmin = k; break; }
        if (kmin != 0x7fffffff) atomicMin(&s_k, kmin);
        __syncthreads();
        period = (double)N / (double)s_k;
      }
    }
    if (period < P.beta) type = PF_WAVE;
    else type = (total / (double)n) > 0.0 ? PF_ANCHOR : PF_VEIL;   // mean-score fallback
  }
  if (tid == 0) {
    P.prompt_type[blockIdx.x] = type;
    if (P.prompt_period) P.prompt_period[blockIdx.x] = period;
  }
}

// ---------------------------------------------------------------------------------------------------
// Batched form.  A workgroup takes a contiguous run of sequences, one per compute unit where the launch is large, and keeps them in LDS
// as they lie in memory; a sequence that the sign rates decide is finished there, the others are listed, and every wave then takes 16
// listed sequences at a time from the raw values to the result.  The differences x of length N are folded,
// e[m] = x[m] + x[N-m], o[m] = x[m] - x[N-m], so that re X[k] = sum_m e[m] cos(2 pi k m / N) and
// im X[k] = -sum_m o[m] sin(2 pi k m / N) run over m = 0 .. N/2 only, and both are products of a [16 x N/2] and a
// [N/2 x 16] matrix on v_mfma_f64_16x16x4 (A: lane l holds row l % 16, inner index l / 16; B: column l % 16, inner index
// l / 16; result: register r of lane l is row l / 16 + 4 r, column l % 16).  Every lane folds its A operands (a quarter of the inner
// indices) from the raw values straight into registers; the B operands, the same for all waves, lie in LDS as the lanes read them.
// The amplitudes of a sequence go where its raw values were.
// Bound: the chain of one workgroup, and the fetching of its code, most of which runs once: 92 160 sequences of 69 frames take
// 21 us (with 62 us before: four waves in rounds of 16 sequences between barriers, folded into LDS, twiddles gathered by index), of
// which their 25 MB need 5 and the votes 4.  On the way: raw values through registers into padded rows 25 us, with every loop
// unrolled (3200 instructions instead of 2200) 29.  6400 take 13.0 us against 13.8, 23 040 of 72 frames 14.8 against 23.7, 92 160 of
// 24 frames 16.0 against 36.1; few sequences, and some lengths in launches of medium size, are left to the forms below.
// ---------------------------------------------------------------------------------------------------
constexpr int CLS_BATCH_MIN = 4;        // shortest sequence with a spectrum (three differences)
constexpr int CLS_STEPS = 9;            // matrix steps: sequences of at most 72 frames (with 16, for 128 frames, the folded operands of a
                                        // wave no longer fit its 128 registers: 23 040 of 100 frames took 30 us, in the form below 28)
constexpr int CLS_WAVES = 16;           // of the batched form
constexpr int CLS_BATCH_THREADS = CLS_WAVES * 64;
constexpr int CLS_LDS = 159 * 1024;     // of the 160 KB of a compute unit
constexpr int CLS_WGS = 256;            // workgroups of a large launch, one per compute unit
constexpr int CLS_REST = 4;             // bins beyond a multiple of 16 that are not worth a matrix product of their own
typedef __attribute__((ext_vector_type(4))) double f64x4;
typedef double __attribute__((may_alias)) amp_t;   // an amplitude in the place of raw values: its accesses are ordered with those of the floats

struct ClassifyBatchParams {
  ClassifyParams c;
  int n_seq, per_wg, cap;               // sequences: all, of a workgroup, of one round
};
__host__ __device__ constexpr int cls_inner(int N) { return (N / 2 + 1 + 3) / 4 * 4; }      // inner length, padded to the matrix step
__host__ __device__ constexpr int cls_groups(int N) { return (N / 2 + 15) / 16; }           // bins 1 .. N/2, 16 at a time
static_assert(cls_inner(71) == 4 * CLS_STEPS && cls_inner(72) > 4 * CLS_STEPS, "72 frames are 71 differences");
__host__ __device__ constexpr int cls_table(int n) { return (n + 1) & ~1; }                 // what follows starts on a 16-byte border
// LDS layout in doubles: B operands [groups][CLS_STEPS][cos | sin][64]; tables cos, sin, window [cls_table each]; then floats: raw sequences
// [cap][n] and a copy's overhang; then ints: listed sequences [cap]
constexpr int CLS_COPY = 64 * 4;        // floats of one wave's copy
__host__ __device__ constexpr size_t cls_lds_bytes(int n, int cap) {
  return sizeof(double) * ((size_t)cls_groups(n - 1) * CLS_STEPS * 128 + 3 * (size_t)cls_table(n)) + sizeof(float) * ((size_t)cap * n + CLS_COPY) +
         sizeof(int) * (size_t)cap;
}

// A lane's value of the lane d further on in its group of 16 (d = 8, 4, 2, 1: an exchange of halves for what is summed or compared
// over all 16)
template <int D>
__device__ __forceinline__ int row_turn(int x) { return __builtin_amdgcn_update_dpp(x, x, 0x120 | D, 0xf, 0xf, false); }   // row_ror
template <int D>
__device__ __forceinline__ double row_turn(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)row_turn<D>((int)(unsigned)u), hi = (unsigned)row_turn<D>((int)(unsigned)(u >> 32));
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// Sum over the four lanes 16 apart
__device__ __forceinline__ int quarter_sum(int x) {
  auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = a[0] + a[1];
  auto b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return b[0] + b[1];
}
__device__ __forceinline__ double quarter_sum(double x) {
  auto half = [](double v, auto swap) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    auto lo = swap((unsigned)u), hi = swap((unsigned)(u >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi[0] << 32 | (unsigned)lo[0]) +
           __builtin_bit_cast(double, (unsigned long long)hi[1] << 32 | (unsigned)lo[1]);
  };
  x = half(x, [](unsigned v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
  return half(x, [](unsigned v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
}

__global__ __launch_bounds__(CLS_BATCH_THREADS) void pf_classify_batch_kernel(ClassifyBatchParams B) {
  extern __shared__ __attribute__((aligned(16))) double s_batch_mem[];
  __shared__ int s_count, s_hi, s_lo;
  typedef __attribute__((address_space(3))) void *lptr_t;
  constexpr int S = CLS_STEPS, GROUPS = (4 * S - 1 + 15) / 16;     // bin groups at most (N / 2 <= 4 S - 1)
  const ClassifyParams &P = B.c;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int n = P.n_hist, N = n - 1, nb = N / 2;
  const int groups = cls_groups(N), steps = cls_inner(N) / 4;
  // the last group as a matrix product, unless it has a few bins only
  const int rest = nb - 16 * (groups - 1), full = rest <= CLS_REST ? groups - 1 : groups;
  const int nt = cls_table(n);
  double *s_b = s_batch_mem, *s_cos = s_b + groups * S * 128, *s_sin = s_cos + nt, *s_win = s_sin + nt;
  float *s_raw = (float *)(s_win + nt);
  int *s_list = (int *)(s_raw + B.cap * n + CLS_COPY);
  const int seq0 = blockIdx.x * B.per_wg, seq1 = pf_min(seq0 + B.per_wg, B.n_seq);

  auto finish = [&](int seq, int type, double period) {
    P.prompt_type[seq] = type;
    if (P.prompt_period) P.prompt_period[seq] = period;
  };
  // a round's raw values, as they lie in memory, straight into LDS: 1 KB per copy where they start on a 16-byte border, else 256 bytes;
  // the last copy's overhang reads zeros (beyond the descriptor's end) and lands behind the last sequence
  auto request = [&](int sb, int rows) {
    const float *from = P.logits + (size_t)sb * n;
    const int bytes = rows * n * (int)sizeof(float);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)from, 0, bytes, 0x00020000u);
    if (((uintptr_t)from & 15) == 0) {
      for (int o = wave * 1024; o < bytes; o += CLS_WAVES * 1024)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)((char *)s_raw + o), 16, lane * 16, o, 0, 0);
    } else {
      for (int o = wave * 256; o < bytes; o += CLS_WAVES * 256)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)((char *)s_raw + o), 4, lane * 4, o, 0, 0);
    }
  };
  request(seq0, pf_min(B.cap, seq1 - seq0));                       // travels while the tables are made
  static_assert(8 * CLS_STEPS <= 512, "a table is made by half the threads");
  {
    const int m = tid & 511;
    const bool win = tid >= 512;
    if (m < N) {                                                   // one copy of the sine for both tables: this code runs once and is fetched for it
      double sn, cs;
      sincospi(2.0 * (double)m / (double)(win ? N - 1 : N), &sn, &cs);
      if (win) s_win[m] = 0.5 - 0.5 * cs;
      else s_cos[m] = cs, s_sin[m] = sn;
    }
  }
  // The sign rates decide by whole numbers: at least s_hi positive values is an Anchor sequence, at most s_lo a Veil one
  // (the same quotients and comparisons as for one sequence, made once for every count)
  if (wave == CLS_WAVES - 1) {
    int hi = n + 1, lo = -1;
    for (int c0 = 0; c0 <= n; c0 += 64) {
      const double r_pos = (double)(c0 + lane) / (double)n;
      const bool anchor = c0 + lane <= n && r_pos >= P.alpha, veil = c0 + lane <= n && !anchor && 1.0 - r_pos >= P.alpha;
      const unsigned long long am = __builtin_amdgcn_ballot_w64(anchor), vm = __builtin_amdgcn_ballot_w64(veil);
      if (am) hi = pf_min(hi, c0 + __builtin_ctzll(am));
      if (vm) lo = c0 + 63 - __builtin_clzll(vm);
    }
    if (lane == 0) {
      s_hi = hi;
      s_lo = lo;
      s_count = 0;
    }
  }
  __syncthreads();
  // j = k m mod N by a multiplication: k m < 2^11, and the quotient is exact while k m N < 2^22
  const int inv = (1 << 22) / N + 1;
  for (int e = tid; e < groups * S * 64; e += CLS_BATCH_THREADS) { // bin k (columns beyond the last repeat it), inner index m
    const int l = e & 63, gs = e >> 6, g = gs / S, m = 4 * (gs - g * S) + (l >> 4);
    const int km = m <= nb ? pf_min(1 + g * 16 + (l & 15), nb) * m : 0, j = km - (int)(((long long)km * inv) >> 22) * N;
    s_b[gs * 128 + l] = s_cos[j];
    s_b[gs * 128 + 64 + l] = s_sin[j];
  }

  for (int sb = seq0; sb < seq1; sb += B.cap) {
    const int rows = pf_min(B.cap, seq1 - sb);
    if (sb > seq0) request(sb, rows);
    __builtin_amdgcn_s_waitcnt(0x0F70);                            // this wave's copies have landed
    __syncthreads();

    // ---- sign rates: 16 sequences per wave, four lanes each ----
    const int hi = s_hi, lo = s_lo;
    for (int r0 = wave * 16; r0 < rows; r0 += CLS_WAVES * 16) {
      const int row = r0 + l16;
      const float *a = s_raw + pf_min(row, rows - 1) * n;
      int lq_c = lq;
      asm volatile("" : "+v"(lq_c));               // places and tests are worked out here: held through the kernel they would take its registers
      float v[2 * S];                                              // all reads in flight
#pragma unroll
      for (int i = 0; i < 2 * S; ++i) v[i] = a[pf_min(4 * i + lq_c, N)];
      int pos = 0;
#pragma unroll
      for (int i = 0; i < 2 * S; ++i) pos += v[i] > 0.0f && 4 * i + lq_c < n ? 1 : 0;
      pos = quarter_sum(pos);
      const bool settled = pos >= hi || pos <= lo, mine = lq == 0 && row < rows;
      if (mine && settled) finish(sb + row, pos >= hi ? PF_ANCHOR : PF_VEIL, INFINITY);
      const unsigned long long und = __builtin_amdgcn_ballot_w64(mine && !settled);
      if (und) {
        int next = 0;
        if (lane == 0) next = atomicAdd(&s_count, __builtin_popcountll(und));
        next = __builtin_amdgcn_readfirstlane(next) + __builtin_popcountll(und & ((1ull << lane) - 1ull));
        if (mine && !settled) s_list[next] = row;
      }
    }
    __syncthreads();
    const int listed = s_count;

    // ---- 16 listed sequences per wave and turn: difference, mean removal (the differences sum to last - first), window, folding
    // into the A operands; spectra; folded scores, their maximum, the lowest bin in the tie band ----
    for (int b0 = wave * 16; b0 < listed; b0 += CLS_WAVES * 16) {
      double e[S], o[S], total = 0.0;
      const int first = s_list[pf_min(b0 + l16, listed - 1)] * n;
      {
        const float *a = s_raw + first;
        int lq_b = lq;
        asm volatile("" : "+v"(lq_b));             // as above
        const double dmean = ((double)a[N] - (double)a[0]) / (double)N;
        // the sum of all values comes from the same reads: m = 0 .. nb, N-m+1 for the pairs, and nb + 1 remain
        if (lq == 0) total = (double)a[nb + 1];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const int m = 4 * s + lq_b, q = N - m;                   // m and q coincide at N/2 and have no partner at 0
          const bool in = m <= nb, pair = in && m != 0 && q != m;
          const int mi = in ? m : 0, qi = pair ? q : 0;
          const double am = (double)a[mi], aq = (double)a[qi + 1];
          const double x = in ? ((double)a[mi + 1] - am - dmean) * s_win[mi] : 0.0;
          const double y = (aq - (double)a[qi] - dmean) * s_win[qi];
          e[s] = pair ? x + y : x;
          o[s] = pair ? x - y : 0.0;
          total += (in ? am : 0.0) + (pair ? aq : 0.0);
          if (s % 3 == 2) __builtin_amdgcn_sched_barrier(0);       // three steps' reads in flight
        }
      }
      total = quarter_sum(total);
      // The raw values of these sequences are in registers now (LDS operations of one wave complete in order), and the amplitudes of
      // bins 1 .. nb go where they were: nb doubles from the first 8-byte border on
      amp_t *const s_amp = (amp_t *)s_raw - 1;
      int at[4];                                                   // of this lane's four results
#pragma unroll
      for (int r = 0; r < 4; ++r) at[r] = (s_list[pf_min(b0 + lq + 4 * r, listed - 1)] * n + 1) >> 1;
#pragma unroll 1
      for (int g = 0; g < full; ++g) {
        f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
        const double *pb = s_b + g * S * 128 + lane;
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (s < steps) {                                         // uniform
            re = __builtin_amdgcn_mfma_f64_16x16x4f64(e[s], pb[s * 128], re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f64_16x16x4f64(o[s], pb[s * 128 + 64], im, 0, 0, 0);
          }
        const int k = 1 + g * 16 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k <= nb && b0 + lq + 4 * r < listed) s_amp[at[r] + k] = sqrt(re[r] * re[r] + im[r] * im[r]);
      }
      // a few bins left over, two at a time: a lane adds up its own inner indices of its sequence, the four lanes of a sequence are
      // added, and two of them keep a bin each
#pragma unroll 1
      for (int i = 0; i < rest && full < groups; i += 2) {
        double re[2] = {0.0, 0.0}, im[2] = {0.0, 0.0};
        const double *pb = s_b + full * S * 128 + lq * 16 + i;
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (s < steps) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              re[j] += e[s] * pb[s * 128 + j];
              im[j] += o[s] * pb[s * 128 + 64 + j];
            }
          }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          re[j] = quarter_sum(re[j]);
          im[j] = quarter_sum(im[j]);
        }
        const double x = lq == 0 ? re[0] : re[1], y = lq == 0 ? im[0] : im[1];
        if (lq < 2 && i + lq < rest && b0 + l16 < listed) s_amp[((first + 1) >> 1) + 1 + full * 16 + i + lq] = sqrt(x * x + y * y);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      int k = 0;                                                   // lane 16 lq + r writes the result of sequence lq + 4 r
#pragma unroll 1
      for (int r = 0; r < 4; ++r) {
        const amp_t *amp = s_amp + ((s_list[pf_min(b0 + lq + 4 * r, listed - 1)] * n + 1) >> 1);
        double sc[GROUPS], best = 0.0;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
          const int kg = 1 + g * 16 + l16;
          double v[CLS_HARMONICS];                                 // all in flight
#pragma unroll
          for (int h = 1; h <= CLS_HARMONICS; ++h) v[h - 1] = amp[pf_min(h * kg, nb)];
          constexpr double w[CLS_HARMONICS] = {1.0, 0.5, 1.0 / 3.0, 0.25};
          sc[g] = 0.0;
#pragma unroll
          for (int h = 1; h <= CLS_HARMONICS; ++h) sc[g] = h * kg <= nb ? sc[g] + v[h - 1] * w[h - 1] : sc[g];
          best = fmax(best, sc[g]);
        }
        best = fmax(best, row_turn<8>(best));
        best = fmax(best, row_turn<4>(best));
        best = fmax(best, row_turn<2>(best));
        best = fmax(best, row_turn<1>(best));
        const bool peak = best > 0.0 && isfinite(best);
        int kmin = CLS_MAX_HIST;                                   // the lane's lowest bin, then the sequence's (none: beyond the last)
#pragma unroll
        for (int g = GROUPS - 1; g >= 0; --g)
          if (peak && 1 + g * 16 + l16 <= nb && sc[g] >= best * (1.0 - CLS_TIE_REL)) kmin = 1 + g * 16 + l16;
        kmin = pf_min(kmin, row_turn<8>(kmin));
        kmin = pf_min(kmin, row_turn<4>(kmin));
        kmin = pf_min(kmin, row_turn<2>(kmin));
        kmin = pf_min(kmin, row_turn<1>(kmin));
        if (l16 == r) k = kmin;
      }
      // the sum is with lane l16 = sequence: fetched from there
      const int which = lq + 4 * l16;
      const double sum = __shfl(total, which & 15, 64);
      if (l16 < 4 && b0 + which < listed) {
        const double period = k <= nb ? (double)N / (double)k : (double)INFINITY;
        finish(sb + s_list[b0 + which], period < P.beta ? PF_WAVE : sum / (double)n > 0.0 ? PF_ANCHOR : PF_VEIL, period);
      }
    }
    __syncthreads();                               // the next round's values go into the same places
    if (tid == 0) s_count = 0;
  }
}

// ---------------------------------------------------------------------------------------------------
// Batched form for sequences whose operands do not fit beside each other in LDS or registers (73 to 256 frames), and for those where it
// is the shorter one (see the dispatch).  A workgroup walks
// a contiguous run of sequences, 16 at a time (four per wave): a sequence that the sign
// rates decide is finished there; the others' windowed and folded differences go into an LDS buffer of `cap` rows, and when the
// buffer is full (or the run ends) their spectra are computed together, as above; the twiddles are read from a table of
// N points by the index k m mod N, which every lane carries along by adding 4 k mod N.
// ---------------------------------------------------------------------------------------------------
constexpr int CLS_FEW_SEQ = 768;        // fewer: a workgroup each
// Shorter and longer sequences than these, but fewer, go by rounds though they would fit the batched form
constexpr int CLS_BATCH_FROM = 11, CLS_BATCH_TO = 70, CLS_BATCH_SEQ = 4608;
constexpr int CLS_ROUNDS_HIST = 256;    // its longest sequence (16 rows and the tables: 72 KB of LDS)
constexpr int CLS_ROUNDS_LDS = 53 * 1024;  // three workgroups per compute unit where that leaves at least one round's rows
constexpr int CLS_ROUNDS_WAVES = 4;            // of the batched form
constexpr int CLS_ROUNDS_THREADS = CLS_ROUNDS_WAVES * 64;
constexpr int CLS_ROUNDS_PER_WAVE = 4;
constexpr int CLS_ROUNDS_MAX_CAP = 64;         // rows of the buffer at most
constexpr int CLS_ROUNDS_WGS = 768;      // workgroups of a large launch: three per compute unit, all resident

// LDS layout in doubles: tables cos, sin, window [N each]; e and o rows [cap][ld] each; amplitudes [cap][la]; row sums
// [cap]; then ints: sequence of each row [cap]; then floats: raw sequences [16][n_hist]
__host__ __device__ constexpr int cls_rounds_ld(int N) { return cls_inner(N) | 1; }                // odd: 16 rows start in different banks
__host__ __device__ constexpr int cls_rounds_la(int N) { return (N / 2 + 1) | 1; }
__host__ __device__ constexpr size_t cls_rounds_lds_bytes(int n_hist, int cap) {
  return sizeof(double) * (3 * (size_t)n_hist + (size_t)cap * (2 * cls_rounds_ld(n_hist - 1) + cls_rounds_la(n_hist - 1) + 1)) +
         sizeof(int) * (size_t)cap + sizeof(float) * CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE * (size_t)n_hist;
}

static_assert(cls_rounds_lds_bytes(CLS_ROUNDS_HIST, CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE) <= 160 * 1024 - 256, "one round of the longest sequence fits");

__global__ __launch_bounds__(CLS_ROUNDS_THREADS) void pf_classify_rounds_kernel(ClassifyBatchParams B) {
  extern __shared__ double s_mem[];
  __shared__ int s_count, s_hi, s_lo;
  const ClassifyParams &P = B.c;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
  const int n = P.n_hist, N = n - 1, nb = N / 2;
  const int ld = cls_rounds_ld(N), la = cls_rounds_la(N), inner = cls_inner(N);
  double *s_cos = s_mem, *s_sin = s_cos + n, *s_win = s_sin + n;
  double *s_e = s_win + n, *s_o = s_e + (size_t)B.cap * ld, *s_amp = s_o + (size_t)B.cap * ld;
  double *s_tot = s_amp + (size_t)B.cap * la;
  int *s_seq = (int *)(s_tot + B.cap);
  float *s_raw = (float *)(s_seq + B.cap) + (size_t)wave * CLS_ROUNDS_PER_WAVE * n;
  for (int m = tid; m < N; m += CLS_ROUNDS_THREADS) {
    double sn, cs;
    sincospi(2.0 * (double)m / (double)N, &sn, &cs);
    s_cos[m] = cs;
    s_sin[m] = sn;
    s_win[m] = 0.5 - 0.5 * cospi(2.0 * (double)m / (double)(N - 1));
  }
  // The sign rates decide by whole numbers: at least s_hi positive values is an Anchor sequence, at most s_lo a Veil one
  // (the same quotients and comparisons as for one sequence, made once for every count)
  if (tid == 0) {
    s_count = 0;
    s_hi = n + 1;
    s_lo = -1;
  }
  __syncthreads();
  for (int c = tid; c <= n; c += CLS_ROUNDS_THREADS) {
    const double r_pos = (double)c / (double)n;
    if (r_pos >= P.alpha) atomicMin(&s_hi, c);
    else if (1.0 - r_pos >= P.alpha) atomicMax(&s_lo, c);
  }
  __syncthreads();
  const int hi = s_hi, lo = s_lo;

  auto finish = [&](int seq, int type, double period) {
    P.prompt_type[seq] = type;
    if (P.prompt_period) P.prompt_period[seq] = period;
  };
  const int seq0 = blockIdx.x * B.per_wg, seq1 = pf_min(seq0 + B.per_wg, B.n_seq);
  // a wave's four sequences are consecutive in memory and travel as one flat run
  constexpr int FLAT = (CLS_ROUNDS_PER_WAVE * CLS_ROUNDS_HIST + 63) / 64;
  const int flat = CLS_ROUNDS_PER_WAVE * n;
  float ahead[FLAT];
  auto request = [&](int sb) {
    const int first = pf_min(sb + wave * CLS_ROUNDS_PER_WAVE, B.n_seq - 1);
    const float *from = P.logits + (size_t)first * n;
    const int most = pf_min(B.n_seq - first, CLS_ROUNDS_PER_WAVE) * n - 1;
#pragma unroll
    for (int i = 0; i < FLAT; ++i)
      if (i * 64 < flat) ahead[i] = from[pf_min(i * 64 + lane, most)];
  };
  request(seq0);
  for (int sb = seq0; sb < seq1; sb += CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE) {
    // ---- four sequences per wave: raw values (requested one round ahead), sign rates ----
#pragma unroll
    for (int i = 0; i < FLAT; ++i)
      if (i * 64 < flat) {                         // uniform
        if (i * 64 + lane < flat) s_raw[i * 64 + lane] = ahead[i];
      }
    request(sb + CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE);
    // the wave's own rows of s_raw are read by other lanes below (LDS operations of one wave complete in order)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // 16 lanes per row
    const float *a = s_raw + lq * n;
    int pos = 0;
    double total = 0.0;
    for (int t = l16; t < n; t += 16) {
      const float v = a[t];
      pos += v > 0.0f ? 1 : 0;
      total += (double)v;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      pos += __shfl_xor(pos, o, 16);
      total += __shfl_xor(total, o, 16);
    }
    const int seq = sb + wave * CLS_ROUNDS_PER_WAVE + lq;
    const bool settled = pos >= hi || pos <= lo, und = seq < seq1 && !settled;
    if (l16 == 0 && seq < seq1 && settled) finish(seq, pos >= hi ? PF_ANCHOR : PF_VEIL, INFINITY);
    const unsigned long long und_rows = __builtin_amdgcn_ballot_w64(und && l16 == 0);
    if (und_rows) {
      int next = 0;
      if (lane == 0) next = atomicAdd(&s_count, __builtin_popcountll(und_rows));
      next = __builtin_amdgcn_readfirstlane(next);
      const int row = next + __builtin_popcountll(und_rows & ((1ull << (lane & 48)) - 1ull));
      if (und) {
        if (l16 == 0) {
          s_seq[row] = seq;
          s_tot[row] = total;
        }
        // difference, mean removal (the differences sum to last - first), window, folding
        const double dmean = ((double)a[N] - (double)a[0]) / (double)N;
        double *e = s_e + row * ld, *o = s_o + row * ld;
        for (int m = l16; m < inner; m += 16) {
          const int q = N - m;                     // m and q coincide at N/2 and have no partner at 0
          const bool in = m <= nb, pair = in && m != 0 && q != m;
          const int mi = in ? m : 0, qi = pair ? q : 0;
          const double x = in ? ((double)a[mi + 1] - (double)a[mi] - dmean) * s_win[mi] : 0.0;
          const double y = ((double)a[qi + 1] - (double)a[qi] - dmean) * s_win[qi];
          e[m] = pair ? x + y : x;
          o[m] = pair ? x - y : 0.0;
        }
      }
    }
    __syncthreads();
    const int rows = s_count;
    const bool last = sb + CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE >= seq1;
    if (rows == 0 || (!last && rows + CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE <= B.cap)) {
      __syncthreads();                             // every wave has read the count before a faster one appends again
      continue;
    }

    // ---- spectra: one task = 16 rows x 16 bins (k = 1 ..), both parts.  Rows beyond the last hold old values;
    // their results are not read ----
    const int row_groups = pf_ceil_div(rows, 16), bin_groups = pf_ceil_div(nb, 16);
    for (int task = wave; task < row_groups * bin_groups; task += CLS_ROUNDS_WAVES) {
      const int rg = task / bin_groups, k = 1 + (task - rg * bin_groups) * 16 + l16;
      const double *pe = s_e + (size_t)(rg * 16 + l16) * ld + lq, *po = s_o + (size_t)(rg * 16 + l16) * ld + lq;
      // k m mod N for this lane's m = lq, and its step from one m to the next (columns beyond the last bin repeat it)
      const int kk = pf_min(k, nb);
      int j = kk * lq, step = 4 * kk;              // at most 3 N / 2 and 2 N
      if (j >= N) j -= N;
      if (step >= N) step -= N;
      if (step >= N) step -= N;
      f64x4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
      double ae = pe[0], ao = po[0], bc = s_cos[j], bs = s_sin[j];      // operands one step ahead of their product
      for (int m = 4; m <= inner; m += 4) {
        const double ce = ae, co = ao, cc = bc, cs = bs;
        j += step;
        if (j >= N) j -= N;
        const int mn = pf_min(m, inner - 4);
        ae = pe[mn], ao = po[mn], bc = s_cos[j], bs = s_sin[j];
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(ce, cc, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(co, cs, im, 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (k <= nb) s_amp[(size_t)(rg * 16 + lq + 4 * r) * la + k] = sqrt(re[r] * re[r] + im[r] * im[r]);
    }
    __syncthreads();

    // ---- folded scores, their maximum, the lowest bin in the tie band: 16 lanes per row ----
    for (int row0 = wave * 4; row0 < rows; row0 += CLS_ROUNDS_WAVES * 4) {
      const int row = row0 + lq;
      const double *amp = s_amp + (size_t)pf_min(row, rows - 1) * la;
      double sc[CLS_ROUNDS_HIST / 32], best = 0.0;
#pragma unroll
      for (int i = 0; i < CLS_ROUNDS_HIST / 32; ++i) {
        const int k = 1 + i * 16 + l16;
        sc[i] = 0.0;
        if (i * 16 < nb) {                         // uniform: bins beyond the last are not looked at
          if (k <= nb) sc[i] = amp[k];
          if (2 * k <= nb) sc[i] += amp[2 * k] * 0.5;
          if (3 * k <= nb) sc[i] += amp[3 * k] * (1.0 / 3.0);
          if (4 * k <= nb) sc[i] += amp[4 * k] * 0.25;
          best = fmax(best, sc[i]);
        }
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) best = fmax(best, __shfl_xor(best, o, 16));
      int kmin = 0;
      if (best > 0.0 && isfinite(best)) {
#pragma unroll
        for (int i = CLS_ROUNDS_HIST / 32 - 1; i >= 0; --i)
          if (i * 16 < nb && 1 + i * 16 + l16 <= nb && sc[i] >= best * (1.0 - CLS_TIE_REL)) kmin = 1 + i * 16 + l16;
      }
      // the lane's lowest bin, then the row's (0 = none)
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        const int other = __shfl_xor(kmin, o, 16);
        kmin = kmin == 0 || (other != 0 && other < kmin) ? other : kmin;
      }
      if (l16 == 0 && row < rows) {
        const double period = kmin > 0 ? (double)N / (double)kmin : (double)INFINITY;
        const int type = period < P.beta ? PF_WAVE : s_tot[row] / (double)n > 0.0 ? PF_ANCHOR : PF_VEIL;
        finish(s_seq[row], type, period);
      }
    }
    if (tid == 0) s_count = 0;
    __syncthreads();
  }
}

// Majority vote over the prompts; equal counts go to the smaller type code.  64 heads per workgroup, one per lane, the
// prompts dealt to its 16 waves (one thread per head walking all prompts alone took 71 us for 256 prompts).  Bound: the loads' latency;
// each wave has eight in flight, also where fewer are left (an unrolled loop's remainder goes one by one: 84 prompts x 34 heads of 133
// frames 19.5 us in all, so 18.8; sixteen in flight 19.6, four 19.0), and no more than it has prompts (with eight whatever there is the
// vote of 4 prompts took 1.96 us, now 1.72).  Eight in a row stand by themselves: with a branch in front of each, and three comparisons
// behind each instead of a shift and an add, 92 160 sequences of 69 frames took 22.7 us in all, now 21.9 (22.4 before either).
constexpr int CLS_VOTE_WAVES = 16, CLS_VOTE_AHEAD = 8;
__global__ __launch_bounds__(CLS_VOTE_WAVES * 64) void pf_classify_vote_kernel(const int32_t *prompt_type, int32_t *head_type, int n_prompts, int n_heads) {
  __shared__ int s_votes[CLS_VOTE_WAVES][3][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x * 64 + lane;
  int votes[3] = {0, 0, 0};
  if (h < n_heads) {
    const unsigned step = (unsigned)CLS_VOTE_WAVES * n_heads;
    unsigned at = (unsigned)wave * n_heads + h;                    // below 2^30 wherever there is a prompt (checked on the host)
#pragma unroll 1
    for (int left = n_prompts - wave; left > 0; left -= CLS_VOTE_WAVES * CLS_VOTE_AHEAD) {
      int t[CLS_VOTE_AHEAD];                                       // all in flight, also where fewer are left
      if (left > (CLS_VOTE_AHEAD - 1) * CLS_VOTE_WAVES) {          // (the branches are uniform)
#pragma unroll
        for (int i = 0; i < CLS_VOTE_AHEAD; ++i) t[i] = prompt_type[at + i * step];
        at += CLS_VOTE_AHEAD * step;
      } else {
#pragma unroll
        for (int i = 0; i < CLS_VOTE_AHEAD; ++i) t[i] = 3;
#pragma unroll
        for (int i = 0; i < CLS_VOTE_AHEAD; ++i) {
          if (left <= i * CLS_VOTE_WAVES) break;
          t[i] = prompt_type[at + i * step];
        }
      }
      unsigned counts = 0;                                         // a byte per type, the fourth for what is not there
#pragma unroll
      for (int i = 0; i < CLS_VOTE_AHEAD; ++i) counts += 1u << (8 * t[i]);
#pragma unroll
      for (int c = 0; c < 3; ++c) votes[c] += counts >> (8 * c) & 255;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) s_votes[wave][c][lane] = votes[c];
  __syncthreads();
  if (wave != 0 || h >= n_heads) return;
  for (int w = 1; w < CLS_VOTE_WAVES; ++w)
#pragma unroll
    for (int c = 0; c < 3; ++c) votes[c] += s_votes[w][c][lane];
  int best = 0;
  if (votes[1] > votes[best]) best = 1;
  if (votes[2] > votes[best]) best = 2;
  head_type[h] = best;
}

extern "C" int pf_classify_heads(const float *logits, int n_prompts, int n_heads, int n_hist, double alpha, double beta,
                                 int32_t *head_type, int32_t *prompt_type, double *prompt_period, void *stream) {
  if (!logits || !head_type || !prompt_type) return PF_ERR_INVALID_ARG;
  if (n_prompts < 1 || n_heads < 1 || n_hist < 1) return PF_ERR_INVALID_ARG;
  if ((long long)n_prompts * n_heads > (1ll << 30)) return PF_ERR_INVALID_ARG;
  if (n_hist > CLS_MAX_HIST) return PF_ERR_UNSUPPORTED;
  if (!(alpha > 0.0) || !(alpha <= 1.0) || !(beta > 0.0)) return PF_ERR_INVALID_ARG;
  ClassifyParams P;
  P.logits = logits;
  P.prompt_type = prompt_type;
  P.prompt_period = prompt_period;
  P.n_hist = n_hist;
  P.alpha = alpha;
  P.beta = beta;
  // Few sequences finish earlier in a workgroup each: of 240 frames 48 take 13.8 us against 23.1 us in batches, 400 17.8 against
  // 23.4 (1920 of 200 frames 56.6 against 21.5); of 69 frames 48 take 8.5 (11.4 in batches, 11.5 by rounds; kernels alone), 756 10.1 (11.8, 12.0), 1276
  // 12.3 (12.1, 12.2), 2000 16.8 (12.0, 12.1); of 13 frames 756 8.2 (9.4, 9.5), 1276 10.0 (9.7, 9.7).
  // The batched form's tables and its few left-over bins have to pay: 2000 of 8 frames 9.6 against 9.4 by rounds, 4000 9.9 against 9.6, 6400 10.2
  // against 10.6; of 72 2000 12.7 against 12.3, 4000 13.1 against 12.6, 6400 13.2 against 14.4; between 11 and 70 frames it is
  // the shorter one throughout (1000 of 12 frames 9.5 both, of 69 11.8 against 12.0).
  const int n_seq = n_prompts * n_heads;
  const bool few = n_seq < CLS_FEW_SEQ, batch = n_seq >= CLS_BATCH_SEQ || (n_hist >= CLS_BATCH_FROM && n_hist <= CLS_BATCH_TO);
  if (n_hist < CLS_BATCH_MIN || n_hist > CLS_ROUNDS_HIST || few) {
    hipLaunchKernelGGL(pf_classify_kernel, dim3(n_seq), dim3(CLS_THREADS), 0, (hipStream_t)stream, P);
  } else if (batch && cls_inner(n_hist - 1) <= 4 * CLS_STEPS) {
    // a workgroup per compute unit, as many sequences each, in as few rounds of equal size as LDS allows
    ClassifyBatchParams B;
    B.c = P;
    B.n_seq = n_seq;
    B.per_wg = pf_ceil_div(B.n_seq, CLS_WGS);
    const size_t tables = cls_lds_bytes(n_hist, 0), each = cls_lds_bytes(n_hist, 1) - tables;
    B.cap = pf_ceil_div(B.per_wg, pf_ceil_div(B.per_wg, (int)((CLS_LDS - tables) / each)));
    hipLaunchKernelGGL(pf_classify_batch_kernel, dim3(pf_ceil_div(B.n_seq, B.per_wg)), dim3(CLS_BATCH_THREADS),
                       cls_lds_bytes(n_hist, B.cap), (hipStream_t)stream, B);
  } else {
    // the longer the buffer, the fuller its groups of 16 rows
    ClassifyBatchParams B;
    B.c = P;
    B.n_seq = n_seq;
    B.cap = CLS_ROUNDS_MAX_CAP;
    while (B.cap > CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE && cls_rounds_lds_bytes(n_hist, B.cap) > CLS_ROUNDS_LDS) B.cap -= 16;
    const int batches = pf_ceil_div(B.n_seq, CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE);
    B.per_wg = pf_ceil_div(batches, CLS_ROUNDS_WGS) * CLS_ROUNDS_WAVES * CLS_ROUNDS_PER_WAVE;
    hipLaunchKernelGGL(pf_classify_rounds_kernel, dim3(pf_ceil_div(B.n_seq, B.per_wg)), dim3(CLS_ROUNDS_THREADS),
                       cls_rounds_lds_bytes(n_hist, B.cap), (hipStream_t)stream, B);
  }
  PF_HIP_CHECK(hipGetLastError());
  hipLaunchKernelGGL(pf_classify_vote_kernel, dim3(pf_ceil_div(n_heads, 64)), dim3(CLS_VOTE_WAVES * 64), 0, (hipStream_t)stream,
                     prompt_type, head_type, n_prompts, n_heads);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}
