// Offline tri-pattern head classification (Sec. 4.1; pre-processing and harmonic folding as in the appendix
// paragraph on the FFT analysis stage), then a vote per head.
// All arithmetic is fp64: the decisions (thresholds, peak bin) are taken in the precision a host implementation
// would use.  Two kernels share the steps:
//   pf_classify_batch_kernel   sequences of 4 to CLS_BATCH_HIST frames (the paper analyses 69): the spectra of 16
//                              sequences at a time as a matrix product on the fp64 matrix cores
//   pf_classify_kernel         others, and launches of few long ones: one workgroup per sequence, a direct DFT (their tables do not fit beside
//                              16 sequences in LDS)
#include <hip/hip_runtime.h>
#include <math.h>
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
// Batched form.  A workgroup walks a contiguous run of sequences, 16 at a time (four per wave): a sequence that the sign
// rates decide is finished there; the others' windowed differences go into an LDS buffer of `cap` rows, and when the
// buffer is full (or the run ends) their spectra are computed together.  The differences x of length N are folded,
// e[m] = x[m] + x[N-m], o[m] = x[m] - x[N-m], so that re X[k] = sum_m e[m] cos(2 pi k m / N) and
// im X[k] = -sum_m o[m] sin(2 pi k m / N) run over m = 0 .. N/2 only, and both are products of a [16 x N/2] and a
// [N/2 x 16] matrix on v_mfma_f64_16x16x4 (A: lane l holds row l % 16, inner index l / 16; B: column l % 16, inner index
// l / 16; result: register r of lane l is row l / 16 + 4 r, column l % 16).  The twiddles are read from a table of
// N points by the index k m mod N, which every lane carries along by adding 4 k mod N.
// What it replaces, one workgroup per sequence (the form above), spent its time on barriers, on an fp64 table of N sines
// per sequence and on three integer instructions and two LDS gathers per multiply-add: 410 us for 92 160 sequences of 69
// frames, of which the bytes need 6 us.  This form takes 60 us: reading 14, counting and folding 12, the matrix products
// and amplitudes 23, the scores 10 (each measured by leaving the later ones out); it is bound by the latency of those
// short chains at three waves per SIMD.  More, smaller workgroups (1024 of 32 rows: 79 us), larger ones of eight waves
// (72 us) and fewer (512 of 64 rows: 62 us) lose more to half-full row groups and barriers than they hide.
// ---------------------------------------------------------------------------------------------------
constexpr int CLS_FEW_HIST = 80, CLS_FEW_SEQ = 768;   // longer sequences than this, but fewer: a workgroup each
constexpr int CLS_BATCH_HIST = 256;     // longest sequence of the batched form (16 rows and the tables: 72 KB of LDS)
constexpr int CLS_BATCH_MIN = 4;        // shortest sequence with a spectrum (three differences)
constexpr int CLS_BATCH_LDS = 53 * 1024;  // three workgroups per compute unit where that leaves at least one round's rows
constexpr int CLS_WAVES = 4;            // of the batched form
constexpr int CLS_BATCH_THREADS = CLS_WAVES * 64;
constexpr int CLS_ROWS_PER_WAVE = 4;
constexpr int CLS_MAX_CAP = 64;         // rows of the buffer at most
constexpr int CLS_BATCH_WGS = 768;      // workgroups of a large launch: three per compute unit, all resident
typedef __attribute__((ext_vector_type(4))) double f64x4;

struct ClassifyBatchParams {
  ClassifyParams c;
  int n_seq, per_wg, cap;
};
// LDS layout in doubles: tables cos, sin, window [N each]; e and o rows [cap][ld] each; amplitudes [cap][la]; row sums
// [cap]; then ints: sequence of each row [cap]; then floats: raw sequences [16][n_hist]
__host__ __device__ constexpr int cls_inner(int N) { return (N / 2 + 1 + 3) / 4 * 4; }      // inner length, padded to the matrix step
__host__ __device__ constexpr int cls_ld(int N) { return cls_inner(N) | 1; }                // odd: 16 rows start in different banks
__host__ __device__ constexpr int cls_la(int N) { return (N / 2 + 1) | 1; }
__host__ __device__ constexpr size_t cls_lds_bytes(int n_hist, int cap) {
  return sizeof(double) * (3 * (size_t)n_hist + (size_t)cap * (2 * cls_ld(n_hist - 1) + cls_la(n_hist - 1) + 1)) +
         sizeof(int) * (size_t)cap + sizeof(float) * CLS_WAVES * CLS_ROWS_PER_WAVE * (size_t)n_hist;
}

static_assert(cls_lds_bytes(CLS_BATCH_HIST, CLS_WAVES * CLS_ROWS_PER_WAVE) <= 160 * 1024 - 256, "one round of the longest sequence fits");

__global__ __launch_bounds__(CLS_BATCH_THREADS) void pf_classify_batch_kernel(ClassifyBatchParams B) {
  extern __shared__ double s_mem[];
  __shared__ int s_count, s_hi, s_lo;
  const ClassifyParams &P = B.c;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
  const int n = P.n_hist, N = n - 1, nb = N / 2;
  const int ld = cls_ld(N), la = cls_la(N), inner = cls_inner(N);
  double *s_cos = s_mem, *s_sin = s_cos + n, *s_win = s_sin + n;
  double *s_e = s_win + n, *s_o = s_e + (size_t)B.cap * ld, *s_amp = s_o + (size_t)B.cap * ld;
  double *s_tot = s_amp + (size_t)B.cap * la;
  int *s_seq = (int *)(s_tot + B.cap);
  float *s_raw = (float *)(s_seq + B.cap) + (size_t)wave * CLS_ROWS_PER_WAVE * n;
  for (int m = tid; m < N; m += CLS_BATCH_THREADS) {
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
  for (int c = tid; c <= n; c += CLS_BATCH_THREADS) {
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
  constexpr int FLAT = (CLS_ROWS_PER_WAVE * CLS_BATCH_HIST + 63) / 64;
  const int flat = CLS_ROWS_PER_WAVE * n;
  float ahead[FLAT];
  auto request = [&](int sb) {
    const int first = pf_min(sb + wave * CLS_ROWS_PER_WAVE, B.n_seq - 1);
    const float *from = P.logits + (size_t)first * n;
    const int most = pf_min(B.n_seq - first, CLS_ROWS_PER_WAVE) * n - 1;
#pragma unroll
    for (int i = 0; i < FLAT; ++i)
      if (i * 64 < flat) ahead[i] = from[pf_min(i * 64 + lane, most)];
  };
  request(seq0);
  for (int sb = seq0; sb < seq1; sb += CLS_WAVES * CLS_ROWS_PER_WAVE) {
    // ---- four sequences per wave: raw values (requested one round ahead), sign rates ----
#pragma unroll
    for (int i = 0; i < FLAT; ++i)
      if (i * 64 < flat) {                         // uniform
        if (i * 64 + lane < flat) s_raw[i * 64 + lane] = ahead[i];
      }
    request(sb + CLS_WAVES * CLS_ROWS_PER_WAVE);
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
    const int seq = sb + wave * CLS_ROWS_PER_WAVE + lq;
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
    const bool last = sb + CLS_WAVES * CLS_ROWS_PER_WAVE >= seq1;
    if (rows == 0 || (!last && rows + CLS_WAVES * CLS_ROWS_PER_WAVE <= B.cap)) {
      __syncthreads();                             // every wave has read the count before a faster one appends again
      continue;
    }

    // ---- spectra: one task = 16 rows x 16 bins (k = 1 ..), both parts.  Rows beyond the last hold old values;
    // their results are not read ----
    const int row_groups = pf_ceil_div(rows, 16), bin_groups = pf_ceil_div(nb, 16);
    for (int task = wave; task < row_groups * bin_groups; task += CLS_WAVES) {
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
    for (int row0 = wave * 4; row0 < rows; row0 += CLS_WAVES * 4) {
      const int row = row0 + lq;
      const double *amp = s_amp + (size_t)pf_min(row, rows - 1) * la;
      double sc[CLS_BATCH_HIST / 32], best = 0.0;
#pragma unroll
      for (int i = 0; i < CLS_BATCH_HIST / 32; ++i) {
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
        for (int i = CLS_BATCH_HIST / 32 - 1; i >= 0; --i)
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
// prompts dealt to its 16 waves (one thread per head walking all prompts alone took 71 us for 256 prompts).
constexpr int CLS_VOTE_WAVES = 16;
__global__ __launch_bounds__(CLS_VOTE_WAVES * 64) void pf_classify_vote_kernel(const int32_t *prompt_type, int32_t *head_type, int n_prompts, int n_heads) {
  __shared__ int s_votes[CLS_VOTE_WAVES][3][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = blockIdx.x * 64 + lane;
  int votes[3] = {0, 0, 0};
  if (h < n_heads) {
#pragma unroll 4
    for (int p = wave; p < n_prompts; p += CLS_VOTE_WAVES) {
      const int t = prompt_type[(size_t)p * n_heads + h];
#pragma unroll
      for (int c = 0; c < 3; ++c) votes[c] += t == c ? 1 : 0;
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
  // Few long sequences finish earlier in a workgroup each: of 240 frames 48 take 13.8 us against 23.1 us in batches, 400 17.8 against
  // 23.4 (1920 of 200 frames 56.6 against 21.5); of 100 frames 48 take 12.9 against 13.7, of 69 or fewer as long either way.
  const bool few = n_hist > CLS_FEW_HIST && (long long)n_prompts * n_heads < CLS_FEW_SEQ;
  if (n_hist >= CLS_BATCH_MIN && n_hist <= CLS_BATCH_HIST && !few) {
    // the longer the buffer, the fuller its groups of 16 rows; 48 rows for the paper's 69 frames
    ClassifyBatchParams B;
    B.c = P;
    B.n_seq = n_prompts * n_heads;
    B.cap = CLS_MAX_CAP;
    while (B.cap > CLS_WAVES * CLS_ROWS_PER_WAVE && cls_lds_bytes(n_hist, B.cap) > CLS_BATCH_LDS) B.cap -= 16;
    const int batches = pf_ceil_div(B.n_seq, CLS_WAVES * CLS_ROWS_PER_WAVE);
    B.per_wg = pf_ceil_div(batches, CLS_BATCH_WGS) * CLS_WAVES * CLS_ROWS_PER_WAVE;
    hipLaunchKernelGGL(pf_classify_batch_kernel, dim3(pf_ceil_div(B.n_seq, B.per_wg)), dim3(CLS_BATCH_THREADS),
                       cls_lds_bytes(n_hist, B.cap), (hipStream_t)stream, B);
  } else {
    hipLaunchKernelGGL(pf_classify_kernel, dim3(n_prompts * n_heads), dim3(CLS_THREADS), 0, (hipStream_t)stream, P);
  }
  PF_HIP_CHECK(hipGetLastError());
  hipLaunchKernelGGL(pf_classify_vote_kernel, dim3(pf_ceil_div(n_heads, 64)), dim3(CLS_VOTE_WAVES * 64), 0, (hipStream_t)stream,
                     prompt_type, head_type, n_prompts, n_heads);
  PF_HIP_CHECK(hipGetLastError());
  return PF_OK;
}
