// gemm_tile_kernel: the decoder's bf16 GEMM for calls of many rows (prefill,
// large batches, wide multi-draft windows) and for any call whose K has one
// logical split.  Included by model.hip after GemmArgs and the epilogue modes.
//
// C[m, n] = sum_k A[m, k] W[n, k].  A workgroup of WM x WN waves computes a
// tile of MT rows x CT columns over all of K; each wave holds RG x CG blocks
// of 32 x 32.  Every element is ((0 + p_0) + p_1) + ... over the logical K
// splits (g.ksplit), p_s the in-order MFMA accumulation of split s: the
// weight-streaming kernels' bits.
//
// Bound by feeding the matrix cores.  Per 64-k chunk a CU of the 128 x 256
// tile has 1,024 cycles of products, about 1,000 of direct global -> LDS
// copies (the copies alone, measured) and 900 of LDS traffic, so all three
// must run at once:
//   * whole-line 64-k chunks (128 bytes of a row) in a ring of NS stages,
//     copied NS - 1 chunks ahead; a bare barrier per chunk;
//   * a wave's copies are spread between its products -- issued in one go
//     they hold the wave up for 16 cycles each, every wave at once (754 ->
//     700 TFLOP/s without);
//   * the fragments of half a chunk are read under the products of the other
//     half, two reads after each of the first products (802 -> 754 without).
// 8832 x 8192 outputs, K = 1536: 283 us (785 TFLOP/s); the kernel this
// replaces (registers to LDS, double-buffered, 128 x 128 tiles, one barrier
// that drained every load per chunk) took 545 us (408 TFLOP/s).
#pragma once

namespace dvs {

typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

// The bf16 and top-1 epilogues of a tile of MT x CT summed values in LDS (fp32,
// row-major), by NT threads.  Columns past the call's are skipped; a 32-column block lies
// in one segment.
template <int MT, int CT, int NT, int EPI>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& g, const float* __restrict__ s_sum,
                                              int tid, int lane, int m0, int c0) {
  constexpr int CB = CT / 32;
  auto seg_of = [&](int col) {
    int si = 0;
    if (g.nseg > 1 && col >= g.seg[1].n0) si = 1;
    if (g.nseg > 2 && col >= g.seg[2].n0) si = 2;
    return si;
  };
  if constexpr (EPI == EPI_SWIGLU) {
    // a unit: 4 gate columns of a block and the 4 up columns 16 further on
    constexpr int UNITS = MT * CB * 4;
    const GemmSeg sg = g.seg[0];
#pragma unroll 4
    for (int u = tid; u < UNITS; u += NT) {
      const int r = u / (CB * 4), b = (u / 4) % CB, c = (u % 4) * 4;
      const int row = m0 + r, f = (c0 >> 1) + b * 16 + c;
      if (row >= g.M || f >= sg.n) continue;
      const f32x4 gt = *(const f32x4*)(s_sum + r * CT + b * 32 + c);
      const f32x4 up = *(const f32x4*)(s_sum + r * CT + b * 32 + 16 + c);
      __bf16 act[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = (float)(__bf16)gt[i], o = (float)(__bf16)up[i];
        act[i] = (__bf16)(v / (1.0f + expf(-v)) * o);
      }
      __bf16* dst = (__bf16*)sg.C + (size_t)row * sg.n + f;
      if ((sg.n & 3) == 0 && f + 4 <= sg.n) {
        *(u32x2*)dst = __builtin_bit_cast(u32x2, act);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (f + i < sg.n) dst[i] = act[i];
      }
    }
  } else if constexpr (EPI == EPI_ARGMAX) {
    // a unit is 8 columns of a block's row; the 4 units of a block row are
    // adjacent lanes
    constexpr int UNITS = MT * CB * 4;
    const int NB = (g.ncols + 31) / 32;
    bool nonfinite = false;
    static_assert(UNITS % NT == 0, "whole lane quads");
    for (int u = tid; u < UNITS; u += NT) {
      const int r = u / (CB * 4), b = (u / 4) % CB, q = u % 4;
      const int row = m0 + r, cb = c0 / 32 + b;
      const bool live = row < g.M && cb < NB;
      uint64_t kv = 0;
      if (live) {
        const f32x4 t0 = *(const f32x4*)(s_sum + r * CT + b * 32 + q * 8);
        const f32x4 t1 = *(const f32x4*)(s_sum + r * CT + b * 32 + q * 8 + 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int col = cb * 32 + q * 8 + i;
          const uint64_t k = col < g.ncols ? pack_logit(i < 4 ? t0[i] : t1[i - 4], col, nonfinite) : 0;
          kv = k > kv ? k : kv;
        }
      }
#pragma unroll
      for (int off = 1; off < 4; off <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)kv, off);
        const uint32_t hi = __shfl_xor((uint32_t)(kv >> 32), off);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        kv = o > kv ? o : kv;
      }
      if (live && q == 0) g.part[(size_t)row * NB + cb] = kv;
    }
    if (__any(nonfinite) && lane == 0) set_err(g.err, DVS_ERR_NONFINITE);
  } else if (EPI == EPI_BF16 && g.rope_tab != nullptr) {
    // a unit: columns c .. c+3 of a block's first half and their partners 16
    // further on (dims i and i + D/2 of a head, or plain columns for V).
    // Element by element: a vector conversion of the rotated floats rounds
    // double -> float -> bf16 in two steps where the scalar one (and so the
    // other kernels) ends in a single rounding; they differ in 1 of 10^5.
    constexpr int UNITS = MT * CB * 4;
    const int D = g.rope_D, half = D / 2;
#pragma unroll 2
    for (int u = tid; u < UNITS; u += NT) {
      const int r = u / (CB * 4), b = (u / 4) % CB, c = (u % 4) * 4;
      const int row = m0 + r, col = c0 + b * 32;
      if (row >= g.M || col >= g.ncols) continue;
      const int si = seg_of(col);
      const GemmSeg sg = g.seg[si];
      const int cs = col - sg.n0;
      const f32x4 x1 = *(const f32x4*)(s_sum + r * CT + b * 32 + c);
      const f32x4 x2 = *(const f32x4*)(s_sum + r * CT + b * 32 + 16 + c);
      __bf16 y1[4], y2[4];
      int d1 = cs + c, d2 = cs + 16 + c;
      if (si < 2) {
        const int hd = cs / D, i = (cs - hd * D) / 2 + c;
        const double2* tab = g.rope_tab + (size_t)row * half + i;
        d1 = hd * D + i;
        d2 = d1 + half;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double2 t = tab[e];
          float o1, o2;
          rope_rotate((float)(__bf16)x1[e], (float)(__bf16)x2[e], t.x, t.y, o1, o2);
          y1[e] = (__bf16)o1;
          y2[e] = (__bf16)o2;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          y1[e] = (__bf16)x1[e];
          y2[e] = (__bf16)x2[e];
        }
      }
      __bf16* dst = (__bf16*)sg.C + (size_t)row * sg.n;
      *(u32x2*)(dst + d1) = __builtin_bit_cast(u32x2, y1);
      *(u32x2*)(dst + d2) = __builtin_bit_cast(u32x2, y2);
    }
  } else {
    static_assert(EPI == EPI_BF16, "fp32 results are stored by the kernel");
    constexpr int UNITS = MT * CT / 4;
    static_assert(UNITS % NT == 0, "whole rounds");
#pragma unroll 8
    for (int u = tid; u < UNITS; u += NT) {
      const int r = u / (CT / 4), cc = (u % (CT / 4)) * 4;
      const int row = m0 + r, gcol = c0 + cc;
      const GemmSeg sg = g.seg[seg_of(gcol)];
      const int col = gcol - sg.n0;
      if (row >= g.M || col >= sg.n) continue;
      const f32x4 t = *(const f32x4*)(s_sum + r * CT + cc);
      __bf16* dst = (__bf16*)sg.C + (size_t)row * sg.n + col;
      if ((sg.n & 3) == 0 && col + 4 <= sg.n) {
        *(bf16x4*)dst = __builtin_convertvector(t, bf16x4);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (col + i < sg.n) dst[i] = (__bf16)t[i];
      }
    }
  }
}

// ALIGNED = false: operands that do not all start on 16 bytes (a weight that
// begins inside another tensor).  Direct global -> LDS copies are only used on
// 16-byte addresses; these go through registers, by loads of any alignment.
template <int WM, int WN, int RG, int CG, int NS, int EPI, bool ALIGNED = true>
__global__ void __launch_bounds__(WM * WN * 64, (NS * (WM * RG + WN * CG) * 4096 <= 81920 && WM * WN == 4) ? 2 : 1)
gemm_tile_kernel(GEMM_HEAD_PARAMS, GemmArgs g) {
  constexpr int NW = WM * WN, NT = NW * 64;
  constexpr int MT = WM * RG * 32, CT = WN * CG * 32;    // tile rows, columns
  constexpr int KC = 64, RB = KC * 2;
  constexpr int STB = (MT + CT) * RB;                    // bytes of a stage
  constexpr int NCP = (MT + CT) / 8;                     // 1 KB copies per stage
  constexpr int PW = NCP / NW;                           // ... per wave
  static_assert(NCP % NW == 0, "copies per wave");
  static_assert(PW * (NS - 1) < 64, "vmcnt range");
  constexpr int LDS_B = NS * STB > MT * CT * 4 ? NS * STB : MT * CT * 4;
  static_assert(LDS_B <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char s_ring[LDS_B];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int nct = (ncols + CT - 1) / CT, nrt = n_rt;
  // order: strips of GM row tiles, column-major inside; each XCD takes a
  // contiguous run of the sequence
  constexpr int GM = MT >= 256 ? 4 : 8;
  const int total = nct * nrt;
  const int per = (total + 7) / 8;
  const int p = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || p >= total) return;
  const int strip = p / (GM * nct), q = p - strip * (GM * nct);
  const int gm = min(GM, nrt - strip * GM);
  const int ct = q / gm, rt = strip * GM + (q - ct * gm);
  const int m0 = rt * MT, c0 = ct * CT;

  auto sw = [](int row) { return (row >> 1) & 7; };
  const int crow = lane >> 3, cchk = lane & 7;
  const bool rope_call = EPI == EPI_BF16 && rope_D != 0;
  const __bf16* src[PW];
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    const int row = (w * PW + i) * 8 + crow;             // row of the stage: A rows, then W rows
    if (w * PW + i < MT / 8) {
      src[i] = hA + (size_t)min(m0 + row, M - 1) * K;
    } else {
      const int cw = row - MT;                           // column of the tile
      const int col = c0 + cw;
      const __bf16* base;
      int rowi, n;
      if (EPI == EPI_SWIGLU) {
        rowi = (col >> 5) * 16 + (col & 15);
        base = (col & 16) ? hW1 : hW0;
        n = n1;
      } else {
        const ColSeg cs = col_seg(col, hW0, hW1, hW2, ncols, n1, n2);
        rowi = col - cs.n0;
        n = cs.n;
        base = cs.W;
        if (rope_call && cs.si < 2) {
          const int hd = rowi / rope_D, cp = rowi - hd * rope_D;
          const int bh = cp >> 5, c = cp & 31;
          rowi = hd * rope_D + (c < 16 ? bh * 16 + c : rope_D / 2 + bh * 16 + c - 16);
        }
      }
      src[i] = base + (size_t)(rowi < n ? rowi : 0) * K;
    }
    src[i] += (cchk ^ sw(row)) << 3;
  }
  const int nch = K / KC;
  const int cps = nch / g.ksplit;                        // chunks per split
  auto issue_one = [&](int t, int slot, int i) {         // copy i of the wave's PW copies of chunk t
    char* dst = s_ring + slot * STB + (w * PW + i) * 1024;
    if constexpr (ALIGNED)
      __builtin_amdgcn_global_load_lds((const void*)(src[i] + t * KC), (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    else
      *(u32x4*)(dst + lane * 16) = *(const u32x4_a2*)(src[i] + t * KC);
  };
  const int wr = w / WN, wc = w % WN;
  // Fragments are read half a chunk (two 16-k steps) ahead of their products:
  // the second half of chunk t under the products of its first, the first
  // half of chunk t + 1 under the products of the second.
  int off[4];                                            // the lane's bytes of step ks in a 32-row group
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) off[ks] = l32 * RB + (((2 * ks + hh) ^ sw(l32)) << 4);
  bf16x8 fa[2][2][RG], fb[2][2][CG];
  constexpr int NR = 2 * (RG + CG);                      // fragment reads of half a chunk
  auto read_one = [&](int slot, auto hc, auto ic) {
    constexpr int h = decltype(hc)::value, i = decltype(ic)::value;
    constexpr int k2 = i / (RG + CG), j = i % (RG + CG);
    const char* st = s_ring + slot * STB;
    if constexpr (j < RG)
      fa[h][k2][j] = *(const bf16x8*)(st + (wr * RG + j) * 4096 + off[2 * h + k2]);
    else
      fb[h][k2][j - RG] = *(const bf16x8*)(st + MT * RB + (wc * CG + j - RG) * 4096 + off[2 * h + k2]);
  };
  f32x16 acc[RG][CG], sum[RG][CG];
#pragma unroll
  for (int a = 0; a < RG; ++a)
#pragma unroll
    for (int b = 0; b < CG; ++b) sum[a][b] = f32x16{};
  // The products of half a chunk, with copies [lo, hi) of chunk tn (into slot
  // sn) spread between them: issued in one go they would hold the wave up
  // while the load path takes them (16 cycles each, all waves at once).
  auto products = [&](auto hc, auto fresh, auto loc, auto hic, int tn, int sn, int rslot) {
    constexpr int h = decltype(hc)::value, lo = decltype(loc)::value, hi = decltype(hic)::value;
    constexpr int NM = 2 * RG * CG;                      // products
    static_for<0, NM>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr int k2 = j / (RG * CG), a = (j / CG) % RG, b = j % CG;
      acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          fa[h][k2][a], fb[h][k2][b], h == 0 && k2 == 0 && decltype(fresh)::value ? f32x16{} : acc[a][b], 0, 0, 0);
      constexpr int r0 = NR * j / (NM / 2) < NR ? NR * j / (NM / 2) : NR, r1 = NR * (j + 1) / (NM / 2) < NR ? NR * (j + 1) / (NM / 2) : NR;
      constexpr int jl = j - NM / 2;
      constexpr int c0i = jl < 0 ? lo : lo + (hi - lo) * jl / (NM / 2), c1i = jl < 0 ? lo : lo + (hi - lo) * (jl + 1) / (NM / 2);
      __builtin_amdgcn_sched_barrier(0);
      static_for<r0, r1>([&](auto ic) { read_one(rslot, IC<1 - h>{}, ic); });
      if constexpr (c1i > c0i) {
        if (tn < nch) static_for<c0i, c1i>([&](auto ic) { issue_one(tn, sn, decltype(ic)::value); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // fp32 results are stored from the accumulators: 32 lanes write 128 bytes
  // of a row, without the two barriers and the trip through LDS of the bf16
  // epilogues, which regroup columns.  The residual's values come first of
  // all where the registers allow, under the products (rows and columns past
  // the end read the last one's).  Whole calls, through LDS -> from the
  // accumulators: 1024-row step of four layers 1002 -> 987 us, 2176-row step
  // with fp32 logits 1776 -> 1753 us, prefill of 8832 rows 2727 -> 2700 us.
  // One workgroup per CU over several tiles, the next one's copies under the
  // stores of the last, was slower than the dispatcher's rounds (1017, 1789,
  // 2841 us).
  constexpr bool ADD = EPI == EPI_F32_ADD, EARLY = ADD && RG * CG <= 2;
  const int mw = m0 + wr * RG * 32 + 4 * hh, cw = c0 + wc * CG * 32 + l32;
  float* __restrict__ C = ADD ? (float*)hW1 : (float*)g.seg[0].C;
  f32x16 old[ADD ? RG : 1][ADD ? CG : 1];
  auto load_old = [&]() {
#pragma unroll
    for (int a = 0; a < RG; ++a)
#pragma unroll
      for (int b = 0; b < CG; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          old[a][b][i] = C[(size_t)min(mw + a * 32 + 8 * (i >> 2) + (i & 3), M - 1) * ncols + min(cw + b * 32, ncols - 1)];
  };
  if constexpr (EARLY) load_old();
  static_for<0, NS>([&](auto c) {
    if (decltype(c)::value < nch) static_for<0, PW>([&](auto i) { issue_one(decltype(c)::value, decltype(c)::value, decltype(i)::value); });
  });
  if (NS <= nch) ws_wait_vmcnt<(NS - 1) * PW>();
  else ws_wait_vmcnt<0>();
  ring_barrier();
  static_for<0, NR>([&](auto ic) { read_one(0, IC<0>{}, ic); });
  constexpr int PH = PW / 2;                             // copies under the second half's products
  int t = 0, slot = 0, prev = 0;
  int tn = nch;                                          // chunk whose copies PH.. are due (none yet)
  auto chunk = [&](auto fresh) {
    // the first half's fragments have arrived (they were read under the last
    // chunk's products) before the second half's reads go out
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    products(IC<0>{}, fresh, IC<PH>{}, IC<PW>{}, tn, prev, slot);
    __builtin_amdgcn_sched_barrier(0);
    // chunk t + 1 has landed, and every wave holds its fragments of chunk t,
    // whose slot takes chunk t + NS
    if (t + NS - 1 < nch) ws_wait_vmcnt<(NS - 2) * PW>();
    else ws_wait_vmcnt<0>();
    ring_barrier();
    tn = t + NS;
    prev = slot;
    ++t;
    slot = slot + 1 == NS ? 0 : slot + 1;
    // (reads past the last chunk: unused)
    products(IC<1>{}, IC<0>{}, IC<0>{}, IC<PH>{}, tn, prev, slot);
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int s = 0; s < g.ksplit; ++s) {
    chunk(IC<1>{});
    for (int i = 1; i < cps; ++i) chunk(IC<0>{});
#pragma unroll
    for (int a = 0; a < RG; ++a)
#pragma unroll
      for (int b = 0; b < CG; ++b) sum[a][b] += acc[a][b];
  }
  if constexpr (EPI == EPI_F32 || ADD) {
    if constexpr (ADD && !EARLY) load_old();
#pragma unroll
    for (int a = 0; a < RG; ++a)
#pragma unroll
      for (int b = 0; b < CG; ++b) {
        if constexpr (ADD) {
#pragma unroll
          for (int i = 0; i < 16; ++i) sum[a][b][i] = old[a][b][i] + sum[a][b][i];
          asm volatile("" : "+v"(sum[a][b]));   // (not one load at a time under the conditions below)
        }
        if (cw + b * 32 < ncols)
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int row = mw + a * 32 + 8 * (i >> 2) + (i & 3);
            if (row < M) C[(size_t)row * ncols + cw + b * 32] = sum[a][b][i];
          }
      }
  } else {
    __syncthreads();
    float* s_sum = (float*)s_ring;
#pragma unroll
    for (int a = 0; a < RG; ++a)
#pragma unroll
      for (int b = 0; b < CG; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          s_sum[((wr * RG + a) * 32 + 8 * (i >> 2) + 4 * hh + (i & 3)) * CT + (wc * CG + b) * 32 + l32] = sum[a][b][i];
    __syncthreads();
    tile_epilogue<MT, CT, NT, EPI>(g, s_sum, tid, lane, m0, c0);
  }
}

}  // namespace dvs
