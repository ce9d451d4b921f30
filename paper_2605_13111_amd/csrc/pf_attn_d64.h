// Attention for head_dim 64: 4 waves x 32 query rows per work item, four workgroups per compute unit.  Included by
// pf_attn.hip behind pf_attn_thin.h, whose copies, tile layout and waits it shares.
//
// Bound: the vector ALU.  A 64-key tile costs a wave 16 MFMAs (512 cycles) but the softmax of 32 scores per lane (~700
// cycles of fma, exp2, add and rounding), so what counts is that the four waves of a SIMD keep its vector ALU busy while
// others wait for LDS, copies or their own MFMAs: at most 128 registers per wave, two tile stages (32 KB) per workgroup, tiles
// copied global -> LDS directly (no staging registers), fragments read a few ahead of their MFMA.
// Measured: 16 heads x 4680 queries x up to 512 key tiles 598 -> 465 us (706 -> 908 TFLOP/s; 64 heads: 980) against tiles
// staged through registers at two workgroups per compute unit; since then 457 -> 441 by a cheaper merge and -> 432 by copies that
// follow runs.  Not better: three workgroups (479 us), eight waves per
// workgroup (481), the next tile's scores computed between this tile's weights (523: needs 168 registers).  Without its
// copies the kernel would take 11 % less, without the PV half 25 % less.
#ifndef PF_ATTN_D64_H
#define PF_ATTN_D64_H

constexpr int D64_WAVES = 4;
constexpr int D64_STAGES = 2;
constexpr int D64_TENSOR_BYTES = PF_BK * 128;                    // one tensor's tile
constexpr int D64_STAGE_BYTES = 2 * D64_TENSOR_BYTES;
constexpr int D64_ROWS = PF_BK / D64_WAVES;                      // rows of every tile that one wave copies
constexpr int D64_SMEM = D64_STAGES * D64_STAGE_BYTES > attn_stage_floats(D64_WAVES * 32, 64) * 4 ? D64_STAGES * D64_STAGE_BYTES
                                                                                                  : attn_stage_floats(D64_WAVES * 32, 64) * 4;
static_assert(D64_ROWS % 16 == 0, "a wave's rows start at a multiple of the chunk permutations' period");

// Sixteen rows of K and V, two groups of eight each (see Thin<64>); the second groups' immediate offset moves their LDS destination too.
__device__ __forceinline__ void d64_copy_rows(__amdgpu_buffer_rsrc_t k, __amdgpu_buffer_rsrc_t v, char *to, unsigned k0, unsigned k1, unsigned v0,
                                              unsigned s0, unsigned s1) {
  typedef __attribute__((address_space(3))) void *lptr_t;
  static_assert(D64_ROWS == 2 * Thin<64>::COPY_ROWS && Thin<64>::swz_v(Thin<64>::COPY_ROWS) == 0, "two groups, V chunks permuted alike");
  __builtin_amdgcn_raw_ptr_buffer_load_lds(k, (lptr_t)to, 16, k0, s0, 0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(k, (lptr_t)to, 16, k1, s1, 1024, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(v, (lptr_t)(to + D64_TENSOR_BYTES), 16, v0, s0, 0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(v, (lptr_t)(to + D64_TENSOR_BYTES), 16, v0, s1, 1024, 0);
}

// RUNS: copies follow runs of tiles.  What a run costs to set up has to be spread over some tiles: 22 heads x 80 queries, 19 frames of
// 80 tokens take 24.1 us without and 27.1 with runs, 40 heads x 256, 20 frames of 128, 38.9 and 40.5; at 200 tokens per frame both forms
// take as long (22 x 200 x 19 frames 22.9 and 23.2, 12 x 600 x 40 frames 39.5 and 38.6), and from there on runs gain (12 x 768 x 40 frames of
// 256 47.2 and 46.3; 24 heads x 1200 queries without history 20.7 and 19.8).  A long chunk is a run of its own: from eight tiles
// on, runs gain at frames of two tiles already (24 heads x 600 queries without history 12.7 and 12.3, behind 40 frames of 200 tokens 39.5 and
// 38.6); one of six loses with history in front of it (40 heads x 390, a frame of 195 tokens 13.0 and 13.5).
__device__ __host__ constexpr bool d64_follows_runs(int tpf, int q_tokens) {
  return tpf >= 4 * PF_BK || (tpf >= 2 * PF_BK && q_tokens >= 8 * PF_BK);
}
template <bool RUNS>
__global__ __launch_bounds__(D64_WAVES * 64, 4) void pf_attn_d64_kernel(AttnParams P) {
  typedef Thin<64> C;
  __shared__ __attribute__((aligned(1024))) char smem[D64_SMEM];
  __shared__ int32_t sFlag;
  const PfWorkItem it = P.items[blockIdx.x];
  if (it.head_sel < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  HeadKV H;
  attn_setup_head<64>(P, it, H, tid);
  const float c = P.scale_log2;
  const int key0 = it.kt0 * PF_BK, n_tiles = it.kt1 - it.kt0;
  // a wave whose query rows all lie beyond the chunk's end only sends its share of the copies and meets the barriers
  const bool has_rows = it.q0 + wave * 32 < P.q_tokens;

  // This wave's rows of tile u are keys tw + 64 u .. + D64_ROWS - 1.  As long as they stay in one run, only a scalar offset moves on
  // from tile to tile (32 heads x 4096 queries x 36864 keys 981 -> 997 TFLOP/s).
  const int tw = key0 + wave * D64_ROWS;
  ThinRuns R;
  if constexpr (RUNS) thin_locate<64>(R, pf_min(tw, H.lkv - 1), H);
  else R.at.end = 0, R.at.j = -1;
  __amdgpu_buffer_rsrc_t run_k = __builtin_amdgcn_make_buffer_rsrc((void *)H.k_pool, 0, 0, 0x00020000u), run_v = run_k;
  unsigned run_soff = 0, run_tile = 0, run_second = 0, run_k0 = 0, run_k1 = 0, run_v0 = 0;
  int run_n = 0;                                                 // tiles left that continue the run
  char *const mine = smem + wave * (D64_ROWS * C::ROW_BYTES);
  auto copy_tile = [&](int u, unsigned stage) __attribute__((always_inline)) {
    if constexpr (!RUNS) {
      if (u >= n_tiles) return;
      const int t = tw + u * PF_BK;
      if (t >= R.at.end) thin_locate<64, false>(R, pf_min(t, H.lkv - 1), H);
      thin_copy<64, false, D64_ROWS, false>(R, t, H, mine + stage, lane);
      thin_copy<64, true, D64_ROWS, false>(R, t, H, mine + stage + D64_TENSOR_BYTES, lane);
      return;
    }
    if (__builtin_expect(run_n <= 0, 0)) {
      if (u < n_tiles) {
        const int t = tw + u * PF_BK;
        thin_follow<64, D64_ROWS>(R, t, H);
        const int room = R.at.end - t - D64_ROWS;
        const unsigned rb = (unsigned)(R.at.stride * 2);
        run_tile = PF_BK * rb;
        if (room < 0) {
          thin_copy_border<64, false, D64_ROWS>(R, t, H, mine + stage, lane);
          thin_copy_border<64, true, D64_ROWS>(R, t, H, mine + stage + D64_TENSOR_BYTES, lane);
        } else {
          run_n = __builtin_amdgcn_readfirstlane(pf_min(pf_min(room / PF_BK + 1, n_tiles - u), 1 << (__builtin_clz(run_tile) - 1)));   // offsets stay below 2^31
          int lane_l = lane;
          asm volatile("" : "+v"(lane_l));                       // worked out here, not held in registers through the loop
          const int rr = lane_l / C::CHUNKS, p = lane_l % C::CHUNKS;
          const unsigned low = (unsigned)((p ^ C::swz_k(rr)) << 4), lrow = (unsigned)rr * rb;
          run_k0 = low + lrow;
          run_k1 = (low ^ (unsigned)(C::swz_k(C::COPY_ROWS) << 4)) + lrow;
          run_v0 = (unsigned)((p ^ C::swz_v(rr)) << 4) + lrow;
          run_soff = 0;
          run_second = C::COPY_ROWS * rb - 1024;                 // the second group's immediate offset moves its source by 1024 already
          const long long e = (long long)(t - R.at.t0) * R.at.stride;
          run_k = __builtin_amdgcn_make_buffer_rsrc((void *)(R.at.k + e), 0, (int)(run_tile * (unsigned)run_n), 0x00020000u);
          run_v = __builtin_amdgcn_make_buffer_rsrc((void *)(R.at.v + e), 0, (int)(run_tile * (unsigned)run_n), 0x00020000u);
        }
      }
    }
    if (__builtin_expect(run_n > 0, 1)) {
      --run_n;
      d64_copy_rows(run_k, run_v, mine + stage, run_k0, run_k1, run_v0, run_soff, run_soff + run_second);
      run_soff += run_tile;
    }
  };
  copy_tile(0, 0);
  f32x16 o[1][2];
  float m_run[1], l_run[1];
  attn_zero<64, 1>(o, m_run, l_run);
  bf16x8 qf[1][4];
  attn_load_q<64, 1>(P, it, qf, tid);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(qf[0][ks]));   // the compiler waits here, not inside the loop
  float mc = m_run[0] * c;
  const unsigned lds0 = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) char *)smem;
  const unsigned ak = lds0 + l32 * C::ROW_BYTES + ((g ^ C::swz_k(l32)) << 4);
  unsigned av;
  {
    const int rowv = 4 * g + ((lane & 15) >> 2);
    const int c0 = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    av = lds0 + D64_TENSOR_BYTES + rowv * C::ROW_BYTES + ((c0 ^ C::swz_v(rowv)) << 4) + 8 * (lane & 1);
  }

  for (int u = 0; u < n_tiles; ++u) {
    const unsigned stage = (u & 1) * D64_STAGE_BYTES;
    thin_wait_vm<0>();                                           // this wave's share of tile u has landed
    __builtin_amdgcn_s_barrier();                                // ... everyone's has, and everyone is done with tile u-1
    copy_tile(u + 1, stage ^ D64_STAGE_BYTES);
    if (!has_rows) continue;
    // ---- S^T = K Q^T: fragment 2 ks + kb = key block kb, k-step ks, four ahead ----
    f32x16 s[2];
    {
      u32x4 kf[8];
      auto kread = [&](auto i) {
        constexpr int I = decltype(i)::value, KB = I & 1, KSTEP = I >> 1;
        thin_read_k<KB * 32 * C::ROW_BYTES>(kf[I], (ak + stage) ^ (unsigned)(KSTEP << 5));
      };
      static_for<0, 4>([&](auto i) { kread(i); });
      static_for<0, 8>([&](auto i) {
        constexpr int I = decltype(i)::value, KB = I & 1, KSTEP = I >> 1;
        thin_wait_lds<(I + 3 < 7 ? 3 : 7 - I)>();
        const f32x16 zero = {};
        s[KB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[I]), qf[0][KSTEP], KSTEP == 0 ? zero : s[KB], 0, 0, 0);
        if constexpr (I + 4 < 8) kread(IntC<I + 4>());
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    const int valid = H.lkv - (key0 + u * PF_BK);                // ragged end of the head's sequence
    if (__builtin_expect(valid < PF_BK, 0)) {
      int g_l = g;
      asm volatile("" : "+v"(g_l));
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kb * 32 + 8 * (i >> 2) + 4 * g_l + (i & 3) >= valid) s[kb][i] = -INFINITY;
    }
    // ---- online softmax, one query column per lane ----
    bf16x8 pf[4];
    float ts[2];
    auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float e0 = fast_exp2(fmaf(s[kb][i], c, -mc)), e1 = fast_exp2(fmaf(s[kb][i + 1], c, -mc));
          ts[0] = kb + i == 0 ? e0 : ts[0] + e0;
          ts[1] = kb + i == 0 ? e1 : ts[1] + e1;
          pf[kb * 2 + (i >> 3)][i & 7] = (__bf16)e0;
          pf[kb * 2 + (i >> 3)][(i & 7) + 1] = (__bf16)e1;
        }
    };
    weights();
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(pf[i]));   // rounded here: sunk past the branch, all 32 weights would stay in registers
    if (__builtin_expect(tile_sum_too_large(ts[0] + ts[1]), 0)) {
      float mx = s[0][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kb][i]);
      const float m_new = fmaxf(m_run[0], partner_max(mx));
      const float alpha = fast_exp2((m_run[0] - m_new) * c);
      m_run[0] = m_new;
      mc = m_new * c;
      l_run[0] *= alpha;
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[0][db][i] *= alpha;
      weights();
    }
    l_run[0] += ts[0] + ts[1];
    // ---- O^T += V^T P^T: fragment 2 s16 + db = 16 keys, channel block db (two transpose reads each), four ahead ----
    {
      u32x2 vl[8], vh[8];
      auto vread = [&](auto i) {
        constexpr int I = decltype(i)::value, OFF = (I >> 1) * 16 * C::ROW_BYTES;
        const unsigned a = (av + stage) ^ (unsigned)((I & 1) << 6);
        thin_read_vt<OFF>(vl[I], a);
        thin_read_vt<OFF + 8 * C::ROW_BYTES>(vh[I], a);
      };
      static_for<0, 4>([&](auto i) { vread(i); });
      static_for<0, 8>([&](auto i) {
        constexpr int I = decltype(i)::value;
        thin_wait_lds<2 * (I + 3 < 7 ? 3 : 7 - I)>();
        const u32x4 a4 = __builtin_shufflevector(vl[I], vh[I], 0, 1, 2, 3);
        o[0][I & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a4), pf[I >> 1], o[0][I & 1], 0, 0, 0);
        if constexpr (I + 4 < 8) vread(IntC<I + 4>());
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  __syncthreads();
  attn_epilogue<64, 1, D64_WAVES>(P, it, o, m_run, l_run, (float *)smem, &sFlag, tid);
}

#endif  // PF_ATTN_D64_H
