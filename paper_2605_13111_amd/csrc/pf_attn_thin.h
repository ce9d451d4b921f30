// Thin work items of the pipelined attention kernel: 32 query rows against a run of a head's keys, the keys split over
// the eight waves of the workgroup.  Included by pf_attn.hip (uses its operand layouts and helpers).
//
// A full item gives every wave 32 query rows of its own and lets all eight share each K/V tile; where fewer query rows are
// left (the last query tile of a head, small launches), most waves of such an item would have nothing to do and the item
// would still take a full item's time.  Here all eight waves hold the SAME 32 query rows and walk different keys: each
// streams its own 32-key steps of K and V through a private part of LDS (no barriers in the loop), and the eight partial
// results are merged once at the end through LDS.
//
// Per step and wave: 16 copies of 1 KB (head_dim 128), 24 LDS fragment reads, 16 MFMAs, the softmax of 16 scores per lane.
// Bound: the copies, 128 KB per eight steps through the compute unit's 64 B/clk return path.  K of the next step is sent
// as soon as this step's K fragments are in registers (before the softmax), V of the next as soon as this step's V^T
// fragments are, so that on average 12 KB per wave are in flight.
#ifndef PF_ATTN_THIN_H
#define PF_ATTN_THIN_H

constexpr int THIN_WAVES = 8;
constexpr int THIN_KEYS = 32;                                   // keys per step
template <int D>
struct Thin {
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int TENSOR_BYTES = THIN_KEYS * ROW_BYTES;    // one step of one tensor
  static constexpr int WAVE_BYTES = 2 * TENSOR_BYTES;
  static constexpr int COPY_ROWS = 1024 / ROW_BYTES;            // rows per copy instruction (64 lanes x 16 bytes)
  static constexpr int NCOPY = THIN_KEYS / COPY_ROWS;           // copies per step and tensor
  static constexpr int CHUNKS = ROW_BYTES / 16;                 // 16-byte chunks per row
  static constexpr int NKS = D / 16, NDB = D / 32;
  static constexpr int LD = D + 4;                              // row stride of a staged partial result (floats)
  static constexpr int STAGE_FLOATS = THIN_WAVES * THIN_KEYS * LD + 2 * THIN_WAVES * 32;   // O, then m and l, of all waves
  static constexpr int SMEM_BYTES = THIN_WAVES * WAVE_BYTES > STAGE_FLOATS * 4 ? THIN_WAVES * WAVE_BYTES : STAGE_FLOATS * 4;
  // Position of 16-byte chunk c of row r inside the row: c ^ swz(r).  K fragments are read 32 rows x one chunk at a time, V^T
  // fragments as 64 bytes from each of four rows; with these permutations the lanes of a read cover all banks evenly
  // (head_dim 128 as in the full items; head_dim 64: two rows share the 64 banks).
  static __device__ constexpr int swz_k(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
  static __device__ constexpr int swz_v(int r) { return D == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; }
};

// The keys of one wave: where the step's rows sit.  A "run" is a stretch of keys whose rows are a fixed stride apart: a history
// frame, or the chunk.
struct ThinRun {
  const __bf16 *k, *v;        // row of key t0
  int t0, end;                // keys [t0, end) of the head's sequence
  long long stride;           // elements between rows
  int j;                      // which frame; n_sel: the chunk
};
template <int D>
__device__ __forceinline__ ThinRun thin_run(int j, int slot, const HeadKV &H) {   // slot: of frame j
  ThinRun R;
  R.j = j;
  if (j >= H.n_sel) {
    R.t0 = H.hist_tokens;
    R.end = H.lkv;
    R.k = H.k_cur;
    R.v = H.v_cur;
    R.stride = H.cur_stride;
  } else {
    const long long e = (long long)slot * H.tpf * D;
    R.t0 = j * H.tpf;
    R.end = R.t0 + H.tpf;
    R.k = H.k_pool + e;
    R.v = H.v_pool + e;
    R.stride = D;
  }
  return R;
}
// The run that key t lies in, and the slot of the frame after it, which is read a run ahead where frames are long, so that it is there
// when a step crosses the border; shorter ones may be stepped over, and there it is looked up where it is wanted (where they are shorter
// than a step, only for the chunk: their rows are looked up one by one anyway, and with the run of every step looked up before that 12
// heads x 497 queries, 120 frames of 31 tokens took 53.4 us, now 51.9; 24 heads x 28, 97 frames of 9, 14.8, now 14.7).
constexpr int THIN_AHEAD = PF_BK;
struct ThinRuns {
  ThinRun at;
  int next_slot;
};
template <int D>
__device__ __forceinline__ int thin_next_slot(int j, const HeadKV &H) {
  return j + 1 < H.n_sel ? H.slots[j + 1] : 0;
}
template <int D, bool LONG = true>                               // LONG: frames may be long
__device__ __forceinline__ void thin_locate(ThinRuns &R, int t, const HeadKV &H) {
  const int j = t >= H.hist_tokens ? H.n_sel : __builtin_amdgcn_readfirstlane(t / H.tpf);
  const int slot = j < H.n_sel ? H.slots[j] : 0;
  if (LONG && H.tpf >= THIN_AHEAD) R.next_slot = thin_next_slot<D>(j, H);
  R.at = thin_run<D>(j, slot, H);
}
template <int D, int ROWS = THIN_KEYS>                           // ROWS: of a step
__device__ __forceinline__ void thin_follow(ThinRuns &R, int t, const HeadKV &H) {
  if (__builtin_expect(t < R.at.end || R.at.j >= H.n_sel, 1)) return;
  if (H.tpf >= THIN_AHEAD) {                                     // no frame is stepped over
    const int slot = R.next_slot;
    R.next_slot = thin_next_slot<D>(R.at.j + 1, H);
    R.at = thin_run<D>(R.at.j + 1, slot, H);
  } else if (H.tpf >= ROWS || t >= H.hist_tokens) {              // shorter frames' rows are looked up one by one: R.at stays behind
    thin_locate<D>(R, t, H);
  }
}

// Send the copies of one tensor's rows t .. t+ROWS-1, the first of them in R.at (or beyond the sequence), into `dst` (a place whose row
// number in its tile is a multiple of 16, the period of the chunk permutations; ROWS / Thin<D>::COPY_ROWS instructions whichever way).
// thin_copy_border is for rows that do not all lie in R.at: a step that crosses a border takes its rows from R.at and the run after it by a
// select per lane.  Where every lane looked its row up for itself (a division, a slot from memory, the address), the waves with such
// steps held their workgroup up by 5 us: 5 heads x 666 queries at 333 tokens per frame, two layers 40.8 -> 36.6 us, 20 heads x 400
// queries at 200 102 -> 83, 12 heads x 48 at 48 32 -> 23; head_dim 64, 5 heads x 4680 queries without history 84 -> 78.
template <int D, bool IS_V, int ROWS = THIN_KEYS, bool LONG = true>
__device__ __forceinline__ void thin_copy_border(ThinRuns &Rs, int t, const HeadKV &H, char *dst, int lane) {
  typedef Thin<D> C;
  constexpr int NC = ROWS / C::COPY_ROWS;
  typedef const __attribute__((address_space(1))) void *gptr_t;
  typedef __attribute__((address_space(3))) void *lptr_t;
  const ThinRun &R = Rs.at;
  // Rare: per-lane values are worked out here, not held in registers through the loop
  int lane_l = lane;
  asm volatile("" : "+v"(lane_l));
  if (__builtin_expect(H.tpf >= ROWS || R.j >= H.n_sel, 1)) {    // one border at most; rows past the sequence's end repeat the last key
    const ThinRun N = thin_run<D>(R.j + 1, LONG && H.tpf >= THIN_AHEAD ? Rs.next_slot : thin_next_slot<D>(R.j, H), H);
#pragma unroll                                                   // in a loop of turns of two: 9 heads x 1788 queries without history, six layers 284 -> 289 us
    for (int G = 0; G < NC; ++G) {
      const int row = G * C::COPY_ROWS + lane_l / C::CHUNKS;
      const int tt = pf_min(t + row, H.lkv - 1);
      const bool over = tt >= R.end;
      const char *b = (const char *)(over ? (IS_V ? N.v : N.k) : (IS_V ? R.v : R.k));
      const long long off = (long long)(tt - (over ? N.t0 : R.t0)) * (over ? (int)N.stride : (int)R.stride) * 2;
      const int c = (lane_l % C::CHUNKS) ^ (IS_V ? C::swz_v(row) : C::swz_k(row));
      __builtin_amdgcn_global_load_lds((gptr_t)(b + off + c * 16), (lptr_t)(dst + G * 1024), 16, 0, 0);
    }
    return;
  }
  // Frames shorter than a step.  Two copies: every lane finds its row (4 heads x 48 queries, head_dim 64: 6.46 us, 6.53 with the code
  // for more of them)
  if constexpr (NC <= 2) {
    for (int G = 0; G < NC; ++G) {
      const int row = G * C::COPY_ROWS + lane_l / C::CHUNKS;
      const int tt = pf_min(t + row, H.lkv - 1);
      const bool in_chunk = tt >= H.hist_tokens;
      const int th = in_chunk ? 0 : tt;
      const int j = th / H.tpf;
      const long long e_hist = ((long long)pf_max(H.slots[j], 0) * H.tpf + (th - j * H.tpf)) * D;
      const long long e = in_chunk ? (long long)(tt - H.hist_tokens) * H.cur_stride : e_hist;
      const __bf16 *b = (in_chunk ? (IS_V ? H.v_cur : H.k_cur) : (IS_V ? H.v_pool : H.k_pool)) + e;
      const int c = (lane_l % C::CHUNKS) ^ (IS_V ? C::swz_v(row) : C::swz_k(row));
      __builtin_amdgcn_global_load_lds((gptr_t)((const char *)b + c * 16), (lptr_t)(dst + G * 1024), 16, 0, 0);
    }
    return;
  }
  // More: lane i finds row i (a division, a slot from memory), every copy's lanes ask for theirs.  With a look-up in front of every
  // copy each waited for the slot and, as loads return in order, for the copies before it: 24 heads x 56 queries at 28 tokens per
  // frame, three layers 48.3 -> 35.4 us, 12 heads x 62 at 31 59.3 -> 40.3.  (Row numbers fit 32 bits: 2^31 rows are 549 GB.)
  const int tr = pf_min(t + (lane_l & (ROWS - 1)), H.lkv - 1);
  const int th = tr >= H.hist_tokens ? 0 : tr;
  const int j = th / H.tpf;
  const int at_row = pf_max(H.slots[j], 0) * H.tpf + (th - j * H.tpf);
  const int found = tr >= H.hist_tokens ? tr - H.hist_tokens : at_row;
#pragma unroll
  for (int G = 0; G < NC; ++G) {
    const int row = G * C::COPY_ROWS + lane_l / C::CHUNKS;
    const bool in_chunk = pf_min(t + row, H.lkv - 1) >= H.hist_tokens;
    const char *b = (const char *)(in_chunk ? (IS_V ? H.v_cur : H.k_cur) : (IS_V ? H.v_pool : H.k_pool));
    const unsigned row_b = in_chunk ? (unsigned)H.cur_stride * 2 : D * 2;
    const unsigned long long off = (unsigned long long)(unsigned)__builtin_amdgcn_ds_bpermute(row * 4, found) * row_b;
    const int c = (lane_l % C::CHUNKS) ^ (IS_V ? C::swz_v(row) : C::swz_k(row));
    __builtin_amdgcn_global_load_lds((gptr_t)(b + off + c * 16), (lptr_t)(dst + G * 1024), 16, 0, 0);
  }
}

template <int D, bool IS_V, int ROWS = THIN_KEYS, bool LONG = true>
__device__ __forceinline__ void thin_copy(ThinRuns &Rs, int t, const HeadKV &H, char *dst, int lane) {
  typedef Thin<D> C;
  constexpr int NC = ROWS / C::COPY_ROWS;
  typedef __attribute__((address_space(3))) void *lptr_t;
  const ThinRun &R = Rs.at;
  const int rr = lane / C::CHUNKS, p = lane % C::CHUNKS;
  if (__builtin_expect(t + ROWS <= R.end, 1)) {                  // whole step inside the run: scalar base, per-lane offset
    const long long e = (long long)(t - R.t0) * R.stride;
    const unsigned row_b = (unsigned)(R.stride * 2);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)((IS_V ? R.v : R.k) + e), 0, (int)(ROWS * row_b), 0x00020000u);
    const unsigned low = (unsigned)((p ^ (IS_V ? C::swz_v(rr) : C::swz_k(rr))) << 4);
    static_for<0, NC>([&](auto gi) {
      constexpr int G = decltype(gi)::value;
      constexpr unsigned flip = (unsigned)((IS_V ? C::swz_v(G * C::COPY_ROWS) : C::swz_k(G * C::COPY_ROWS)) << 4);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)(dst + G * 1024), 16, (low ^ flip) + (unsigned)rr * row_b, G * C::COPY_ROWS * row_b, 0, 0);
    });
  } else {
    thin_copy_border<D, IS_V, ROWS, LONG>(Rs, t, H, dst, lane);
  }
}

template <int N>
__device__ __forceinline__ void thin_wait_vm() {                 // at most N vector-memory operations outstanding
  static_assert(N < 64, "vmcnt field");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void thin_wait_lds() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
  __builtin_amdgcn_sched_barrier(0);
}

// Fragment reads by hand: the compiler would wait for all outstanding copies before an LDS read it knows about
template <int OFF = 0>
__device__ __forceinline__ void thin_read_k(u32x4 &f, unsigned a) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f) : "v"(a), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void thin_read_vt(u32x2 &f, unsigned a) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f) : "v"(a), "n"(OFF));
}

// Keys [ta, tb) of the item for this wave: O^T, reference maximum and row sum of query rows q0 .. q0+31.
template <int D>
__device__ __forceinline__ void thin_keys(const AttnParams &P, const PfWorkItem &it, const HeadKV &H, int q0, int ta, int tb, char *mem,
                                          int lane, f32x16 (&o)[D / 32], float &m_run, float &l_run) {
  typedef Thin<D> C;
  const int l32 = lane & 31, g = lane >> 5;
  const float c = P.scale_log2;
  char *memK = mem, *memV = mem + C::TENSOR_BYTES;
  ThinRuns R;
  thin_locate<D>(R, ta, H);
  thin_copy<D, false>(R, ta, H, memK, lane);
  thin_copy<D, true>(R, ta, H, memV, lane);
  bf16x8 qf[C::NKS];
  {
    const int row = pf_min(q0 + l32, P.q_tokens - 1);
    const __bf16 *qh = P.q + (size_t)pf_item_head(it) * P.head_stride + (size_t)row * P.tok_stride + 8 * g;
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) qf[ks] = *(const bf16x8 *)(qh + ks * 16);
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) asm volatile("" : "+v"(qf[ks]));   // the compiler waits here, not inside the loop
  }
  const unsigned ldsK = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)memK;
  const unsigned ldsV = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)memV;
  // this lane's fragments: K row l32, chunk 2 ks + g -> ak ^ (ks << 5); V^T rows 4g + (lane & 15) / 4 (+8, +16 ...), channel
  // block db -> av ^ (db << 6)
  const unsigned ak = ldsK + l32 * C::ROW_BYTES + ((g ^ C::swz_k(l32)) << 4);
  unsigned av;
  {
    const int rowv = 4 * g + ((lane & 15) >> 2);
    const int c0 = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    av = ldsV + rowv * C::ROW_BYTES + ((c0 ^ C::swz_v(rowv)) << 4) + 8 * (lane & 1);
  }
  float mc = m_run * c;
  constexpr int NVF = 2 * C::NDB;                                // V^T fragments of a step, two LDS reads each
  constexpr int VRING = NVF < 6 ? NVF : 6;                       // requested ahead (at most 15 LDS reads may be in flight)
  for (int t = ta; t < tb; t += THIN_KEYS) {
    const bool more = t + THIN_KEYS < tb;
    // ---- S^T = K Q^T ----
    thin_wait_vm<C::NCOPY>();                                    // K of this step has landed (its V may still travel)
    u32x4 kf[C::NKS];
    static_for<0, C::NKS>([&](auto i) {
      constexpr int I = decltype(i)::value;
      thin_read_k(kf[I], ak ^ (unsigned)(I << 5));
    });
    f32x16 s;
    static_for<0, C::NKS>([&](auto i) {
      constexpr int I = decltype(i)::value;
      thin_wait_lds<C::NKS - 1 - I>();
      const f32x16 zero = {};
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[I]), qf[I], I == 0 ? zero : s, 0, 0, 0);
    });
    __builtin_amdgcn_sched_barrier(0);
    if (more) {                                                  // K's place is free: its fragments are in registers
      thin_follow<D>(R, t + THIN_KEYS, H);
      thin_copy<D, false>(R, t + THIN_KEYS, H, memK, lane);
    }
    const int valid = H.lkv - t;                                 // ragged end of the head's sequence
    if (__builtin_expect(valid < THIN_KEYS, 0)) {
      int g_l = g;
      asm volatile("" : "+v"(g_l));                              // rare, as above
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + 4 * g_l + (i & 3) >= valid) s[i] = -INFINITY;
    }
    // ---- online softmax, one query column per lane (as in the full items) ----
    bf16x8 pf[2];
    float ts[2];
    auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float e0 = fast_exp2(fmaf(s[i], c, -mc)), e1 = fast_exp2(fmaf(s[i + 1], c, -mc));
        ts[0] = i == 0 ? e0 : ts[0] + e0;
        ts[1] = i == 0 ? e1 : ts[1] + e1;
        pf[i >> 3][i & 7] = (__bf16)e0;
        pf[i >> 3][(i & 7) + 1] = (__bf16)e1;
      }
    };
    weights();
    asm volatile("" : "+v"(pf[0]), "+v"(pf[1]));                 // rounded here: sunk past the branch, all 16 weights would stay in registers
    if (__builtin_expect(tile_sum_too_large(ts[0] + ts[1]), 0)) {
      float mx = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
      const float m_new = fmaxf(m_run, partner_max(mx));
      const float alpha = fast_exp2((m_run - m_new) * c);
      m_run = m_new;
      mc = m_new * c;
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
      weights();
    }
    l_run += ts[0] + ts[1];
    // ---- O^T += V^T P^T ----
    if (more) thin_wait_vm<C::NCOPY>();                          // V of this step has landed (K of the next may still travel)
    else thin_wait_vm<0>();
    u32x2 vl[NVF], vh[NVF];
    auto vread = [&](auto i) {
      constexpr int I = decltype(i)::value, OFF = (I / C::NDB) * 16 * C::ROW_BYTES;
      const unsigned a = av ^ (unsigned)((I % C::NDB) << 6);
      thin_read_vt<OFF>(vl[I], a);
      thin_read_vt<OFF + 8 * C::ROW_BYTES>(vh[I], a);
    };
    static_for<0, VRING>([&](auto i) { vread(i); });
    static_for<0, NVF>([&](auto i) {
      constexpr int I = decltype(i)::value;
      constexpr int NEWEST = I + VRING - 1 < NVF - 1 ? I + VRING - 1 : NVF - 1;
      thin_wait_lds<2 * (NEWEST - I)>();
      const u32x4 a4 = __builtin_shufflevector(vl[I], vh[I], 0, 1, 2, 3);
      o[I % C::NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a4), pf[I / C::NDB], o[I % C::NDB], 0, 0, 0);
      if constexpr (I + VRING < NVF) vread(IntC<I + VRING>());
      __builtin_amdgcn_sched_barrier(0);
    });
    if (more) thin_copy<D, true>(R, t + THIN_KEYS, H, memV, lane);
  }
}

// One thin item.  smem: Thin<D>::SMEM_BYTES; every thread of the workgroup (512) calls this, nothing in smem is in use.
template <int D>
__device__ __forceinline__ void thin_item(const AttnParams &P, const PfWorkItem &it, char *smem, int32_t *sFlagp, int tid) {
  typedef Thin<D> C;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const float c = P.scale_log2;
  HeadKV H;
  attn_setup_head<D>(P, it, H, tid);
  const int key0 = it.kt0 * PF_BK, key1 = pf_min(it.kt1 * PF_BK, H.lkv);
  const int steps = pf_ceil_div(key1 - key0, THIN_KEYS);
  const int ta = key0 + (steps * wave / THIN_WAVES) * THIN_KEYS, tb = pf_min(key0 + (steps * (wave + 1) / THIN_WAVES) * THIN_KEYS, key1);
  float *sO = (float *)smem, *sM = sO + THIN_WAVES * 32 * C::LD, *sL = sM + THIN_WAVES * 32;
  constexpr int VPT = 32 * D / (THIN_WAVES * 64);                // output values per thread
  const int r = tid / (D / VPT), d0 = (tid % (D / VPT)) * VPT;   // ... of query row r of the group, channels d0 ..
  f32x16 o[C::NDB];
#pragma unroll
  for (int db = 0; db < C::NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.0f;
  float m_run = -3.0e38f, l_run = 0.0f;
  if (ta < tb) thin_keys<D>(P, it, H, it.q0, ta, tb, smem + wave * C::WAVE_BYTES, lane, o, m_run, l_run);
  // ---- the waves' results -> LDS (their key buffers are done with), then one thread per VPT output values ----
  __syncthreads();
  {
    const float lsum = partner_sum(l_run);
    float *row = sO + (wave * 32 + l32) * C::LD;
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *(float4 *)(row + db * 32 + 8 * i4 + 4 * g) = make_float4(o[db][i4 * 4], o[db][i4 * 4 + 1], o[db][i4 * 4 + 2], o[db][i4 * 4 + 3]);
    if (g == 0) {
      sM[wave * 32 + l32] = m_run;
      sL[wave * 32 + l32] = lsum;
    }
  }
  __syncthreads();
  float mmax = sM[r], lsum = 0.0f, acc[VPT];
#pragma unroll
  for (int w = 1; w < THIN_WAVES; ++w) mmax = fmaxf(mmax, sM[w * 32 + r]);
#pragma unroll
  for (int i = 0; i < VPT; ++i) acc[i] = 0.0f;
#pragma unroll
  for (int w = 0; w < THIN_WAVES; ++w) {
    const float f = fast_exp2((sM[w * 32 + r] - mmax) * c);
    lsum += f * sL[w * 32 + r];
#pragma unroll
    for (int i = 0; i < VPT; ++i) acc[i] += f * sO[(w * 32 + r) * C::LD + d0 + i];
  }
  if (it.nseg > 1) {
    constexpr int BQ = 32, NT = THIN_WAVES * 64, NV = VPT / 4;
    f32x4 v[NV];
#pragma unroll
    for (int i = 0; i < VPT; ++i) v[i / 4][i % 4] = acc[i];
    attn_park<D, BQ, NT, 0>(P, it, v, tid);
    if (d0 == 0) attn_park_row<D, BQ>(P, it, r, mmax, lsum);
    if (!attn_arrive(P, it, sFlagp, tid)) return;
    attn_merge<D, BQ, NT, 0>(P, it, v, r, lsum, tid);
#pragma unroll
    for (int i = 0; i < VPT; ++i) acc[i] = v[i / 4][i % 4];
  }
  const float inv = 1.0f / lsum;
  typedef __attribute__((ext_vector_type(VPT))) __bf16 out_t;
  out_t w;
#pragma unroll
  for (int i = 0; i < VPT; ++i) w[i] = (__bf16)(acc[i] * inv);
  if (it.q0 + r < P.q_tokens) *(out_t *)(P.out + (size_t)pf_item_head(it) * P.head_stride + (size_t)(it.q0 + r) * P.tok_stride + d0) = w;
}

#endif  // PF_ATTN_THIN_H
