// Kernels of the bf16 backward pass whose waves work on keys of their own, without barriers.
// See the head of mrt_bf16.hip for the register layouts.  Their accumulators take more registers than the
// 256 an instruction can name; the file is compiled so that a product's results stay in those unless they
// live from step to step (build.py).
#include "mrt_bwd_tiles.hpp"

namespace mrt {

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// ---------------------------------------------------------------------------------------
// Stage L backward at t = T (nothing in dQ to add to) of streamed key ranges, up to six query tiles, after a forward call that left
// its row statistics: rows and columns in one sweep, one workgroup of four waves per (m, j).
//
// A wave owns 32 key rows at a time and every query row, so L and dZ of those keys never leave it: the
// logits are formed with the queries on the accumulator rows (Q and dO of the column sit in LDS, alpha_L
// and Y rows go from global memory straight into matrix operands), which makes L and dZ the operands of
// dY = L^T dO and d alpha_L = scale dZ^T Q as they are.  Only dQ += scale dZ alpha_L contracts over the
// keys: dZ and alpha_L pass through LDS of the wave's own for that, and every wave keeps a dQ of its own,
// added up at the end.  The sweep has no barrier; the loads of a wave's next 32 keys are in flight while it
// forms the results of these.  A compute unit holds one workgroup (two with up to two query tiles; at 64
// features three, two and one of two, four and six tiles), so what is left over its bytes is the load of Q, dO
// and O ahead of the sweep and the sum of the four dQ behind it, which nothing overlaps.
//
// Against the rows of twelve waves with LDS rings and two barriers every 64 keys (k_bwdm_l_rows_ring, which
// stays for calls without the statistics): 480p clip, 90 rows, 642 -> 535 us (its bytes take 416 at the copy
// rate); 20 rows of 17 columns, 12 tiles, 21 heads 292 -> 151; 64 features, 36 rows, 10 heads 74 -> 46, 16
// rows, 2 heads 34 -> 18.  Longest key ranges first (all heads) cost 2 % of the clip's step, non-temporal
// loads 3 %.
// ---------------------------------------------------------------------------------------
template <int D, int NLT>
__global__ __launch_bounds__(256, NLT == 2 ? 2 : 1) void k_bwdm_l_keys(BwdParams bp) {
  const KParams& p = bp.k;
  constexpr int NW = 4, KEYS = 32, LD = D + 16, KS1 = D / 32, NVT = D / 16, ROWS = 16 * NLT, LZ = ROWS + 8, NS = NLT / 2;
  constexpr int CPR = D / 8;
  // Q | dO | per wave alpha_L rows, dZ [nk][l] | row statistics; afterwards the waves' dQ tiles
  constexpr int kTiles = 2 * ROWS * LD + NW * KEYS * (LD + LZ);
  __shared__ __attribute__((aligned(16))) u16 lds[kTiles];
  __shared__ __attribute__((aligned(16))) float lse_s[ROWS], delta_s[ROWS];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, c = lane & 15;
  u16 *Qs = lds, *dOs = lds + ROWS * LD, *Kt = lds + 2 * ROWS * LD + wave * KEYS * (LD + LZ), *Zt = Kt + KEYS * LD;
  const int b1 = p.b1, b2 = p.b2;
  const int j = blockIdx.x, ml = blockIdx.y, m = p.m0 + ml, bhl = blockIdx.z, bh = p.bh0 + bhl;
  const int a = m / p.c2, bq = m - a * p.c2;
  const int NK = visible_key_tile_rows(a, p.c1k, p.ct, p.qt0) * p.c2 * b1;
  const size_t NKtot = (size_t)p.ntk * b1;
  const int b = bh / p.H, hd = bh - b * p.H;
  const size_t row0 = (((size_t)bhl * p.ntq + ml) * b2 + j) * NKtot, qr0 = (((size_t)bhl * p.ntq + ml) * b2 + j) * b1;
  const u16* aLp = (const u16*)p.aL + row0 * D;
  const u16* Yp = (const u16*)p.Y + row0 * D;
  const float* cLp = p.cL + row0;
  const long long qcol = axis_offset(p.cmap, bq * b2 + j);
  const u16* Qp = (const u16*)p.Q + b * p.qs.batch + hd * p.qs.head + qcol * p.qs.token;
  const u16* dOp = (const u16*)bp.dO + b * p.os.batch + hd * p.os.head + qcol * p.os.token;

  // a wave's 32 keys: operand rows (lane column = key) and c_L.  Lanes beyond the range repeat its last key,
  // results included, which they store once more (a branch around a store would make the next loads' waits
  // include every store); only dQ must not count it again.
  bf16x8 ka[2][KS1], ya[2][KS1];
  float cl[2];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const int nk = k0 + 16 * kt + c, at = nk < NK ? nk : NK - 1;
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        ka[kt][ks] = ld_global_16B(aLp + (size_t)at * D + 32 * ks + 8 * g);
        ya[kt][ks] = ld_global_16B(Yp + (size_t)at * D + 32 * ks + 8 * g);
      }
      cl[kt] = cLp[at];
    }
  };
  // the point where a chunk's loads are waited for: at the end of the loop body, where the count of the stores
  // issued after them is exact (at its head the first pass, which has none, would make it wait for those too)
  auto landed = [&]() {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        u32x4 k4 = __builtin_bit_cast(u32x4, ka[kt][ks]), y4 = __builtin_bit_cast(u32x4, ya[kt][ks]);
        asm volatile("" : "+v"(k4), "+v"(y4));
        ka[kt][ks] = __builtin_bit_cast(bf16x8, k4);
        ya[kt][ks] = __builtin_bit_cast(bf16x8, y4);
      }
      asm volatile("" : "+v"(cl[kt]));
    }
  };
  {
    RowRegs<D, ROWS, 256> rq, ro;
    rq.load(Qp, tile_rows(p, a, p.qs.token), b1, tid);
    ro.load(dOp, tile_rows(p, a, p.os.token), b1, tid);
    f32x4 o32[RowRegs<D, ROWS, 256>::N][2];
#pragma unroll
    for (int i = 0; i < RowRegs<D, ROWS, 256>::N; ++i) {
      const int r = (tid + 256 * i) / CPR, rc = r < b1 ? r : b1 - 1;
      const float* at = bp.o32 + (qr0 + rc) * D + 8 * (tid % CPR);
      o32[i][0] = *(const f32x4*)at;
      o32[i][1] = *(const f32x4*)(at + 4);
    }
    if (tid < ROWS) lse_s[tid] = tid < b1 ? bp.lse[qr0 + tid] : INFINITY;      // (rows beyond b1: weights of zero)
    fetch(KEYS * wave);
    rq.template store<LD>(Qs, tid);
    ro.template store<LD>(dOs, tid);
    // delta[l] = sum_nk L[l, nk] (dO[l] . Y[nk]) = dO[l] . O[l]
#pragma unroll
    for (int i = 0; i < RowRegs<D, ROWS, 256>::N; ++i) {
      const bf16x8 x = as_bf16x8(ro.v[i]);
      float t = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) t = fmaf((float)x[e], o32[i][e / 4][e % 4], t);
      t = CPR == 16 ? row16_sum(t) : row8_sum(t);
      const int r = (tid + 256 * i) / CPR;
      if (tid % CPR == 0) delta_s[r] = r < b1 ? t : 0.f;
    }
  }
  const float scale2 = p.scale * kLog2e;
  f32x4 dq[NLT][NVT];
#pragma unroll
  for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) dq[lt][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  landed();

  for (int k0 = KEYS * wave; k0 < NK; k0 += KEYS * NW) {
    bf16x8 zb[NS][2], lb[NS][2];              // dZ and L as operands: 32 query rows x 16 keys
    float zsum[2] = {0.f, 0.f}, bias[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      bias[kt] = -cl[kt] * kLog2e;
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) *(uint4*)(Kt + (16 * kt + c) * LD + 32 * ks + 8 * g) = __builtin_bit_cast(uint4, ka[kt][ks]);
    }
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      f32x4 s[2][2], dp[2][2];                // [query tile of the pair][key tile]
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u16 *qa = Qs + (32 * st + 16 * h + c) * LD + 8 * g, *oa = dOs + (32 * st + 16 * h + c) * LD + 8 * g;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) s[h][kt] = dp[h][kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) {
          const bf16x8 q = ld_lds_16B(qa + 32 * ks), o = ld_lds_16B(oa + 32 * ks);
#pragma unroll
          for (int kt = 0; kt < 2; ++kt) {
            s[h][kt] = mfma(q, ka[kt][ks], s[h][kt]);
            dp[h][kt] = mfma(o, ya[kt][ks], dp[h][kt]);
          }
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 lse = *(const f32x4*)(lse_s + 32 * st + 16 * h + 4 * g), delta = *(const f32x4*)(delta_s + 32 * st + 16 * h + 4 * g);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float L = exp2_fast(fmaf(s[h][kt][r], scale2, bias[kt]) - lse[r]);
            s[h][kt][r] = L;
            dp[h][kt][r] = L * (dp[h][kt][r] - delta[r]);
            zsum[kt] += dp[h][kt][r];
          }
        }
      }
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        lb[st][kt] = pack8(s[0][kt], s[1][kt]);
        zb[st][kt] = pack8(dp[0][kt], dp[1][kt]);
        const uint4 z = k0 + 16 * kt + c < NK ? __builtin_bit_cast(uint4, zb[st][kt]) : uint4{0u, 0u, 0u, 0u};
        u16* at = Zt + (16 * kt + c) * LZ + 32 * st + 4 * g;
        *(uint2*)at = uint2{z.x, z.y};
        *(uint2*)(at + 16) = uint2{z.z, z.w};
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch(k0 + KEYS * NW);
    __builtin_amdgcn_sched_barrier(0);
    // dQ[l] += dZ[l, nk] alpha_L[nk]
    {
      bf16x8 zq[NLT];
#pragma unroll
      for (int lt = 0; lt < NLT; ++lt) zq[lt] = ld_columns<LZ>(Zt, 16 * lt, lane);
      pv_step_multi<D, NLT, LD>(Kt, zq, NLT, dq, lane);
    }
    // d alpha_L[nk] = scale sum_l dZ[l, nk] Q[l], then dY[nk] = sum_l L[l, nk] dO[l]
#pragma unroll
    for (int out = 0; out < 2; ++out) {
      f32x4 oc[2][NVT];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) oc[kt][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        pv_step_multi<D, 2, LD>((out ? dOs : Qs) + 32 * st * LD, out ? lb[st] : zb[st], 2, oc, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const size_t at = row0 + (k0 + 16 * kt + c < NK ? k0 + 16 * kt + c : NK - 1);
        if (out) {
          store_ws_row<D>((u16*)bp.dY + at * D, oc[kt], 1.0f, g);
        } else {
          store_ws_row<D>((u16*)bp.daL + at * D, oc[kt], p.scale, g);
          bp.dcL[at] = -xsum(zsum[kt]);
        }
      }
    }
    landed();
  }

  // dQ: the waves' tiles through LDS, as many query tiles at a time as fit
  constexpr int kTileBytes = NW * NVT * 64 * 16, kAtOnce = kTiles * 2 / kTileBytes, PAIRS = D / 32;
  static_assert(kAtOnce >= 1, "LDS of a query tile's four parts");
  f32x4* part = (f32x4*)lds;
  const TokRows drow = tile_rows(p, a, D);
  float* dQp = bp.dQ + ((size_t)bh * p.Nq + qcol) * D;
#pragma unroll
  for (int l0 = 0; l0 < NLT; l0 += kAtOnce) {
    __syncthreads();
#pragma unroll
    for (int lt = l0; lt < (l0 + kAtOnce < NLT ? l0 + kAtOnce : NLT); ++lt)
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) part[(((lt - l0) * NW + wave) * NVT + vt) * 64 + lane] = dq[lt][vt];
    __syncthreads();
    const int n = (l0 + kAtOnce < NLT ? kAtOnce : NLT - l0) * PAIRS;
    for (int i = wave; i < n; i += NW) {
      const int lt = i / PAIRS, q = i - lt * PAIRS, l = 16 * (l0 + lt) + c;
      f32x4 x[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4* at = part + (lt * NW * NVT + 2 * q + h) * 64 + lane;
        x[h] = ((at[0] + at[NVT * 64]) + (at[2 * NVT * 64] + at[3 * NVT * 64])) * p.scale;
      }
      if (l < b1) {
        f32x4* to = (f32x4*)(dQp + drow(l) + 32 * q + 8 * g);
        to[0] = x[0];
        to[1] = x[1];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Stage R backward of one key tile (b2 <= 16), bf16 workspace: a workgroup is ONE wave, which owns whole key
// blocks and walks their query tiles.
//
// K of the block sits in LDS, V in registers as matrix operands, dK and dV of its keys in accumulators;
// the 16 rows of abar, d alpha_L and dY of a step go from global memory into operands and from there into
// LDS of the wave's own, where the products over the columns read them transposed.  R and scale dS, formed
// with the columns on the lanes, are transposed through LDS too.  Nothing is shared with another wave, so
// there is no barrier, and the next step's rows are in flight while this one is formed.
//
// What bounds it is how many of these chains run side by side: eight to sixteen a compute unit (registers),
// five before, when tiles padded to 32 rows took 28 KB (64 features) or 48 KB of LDS (36 rows of 8 columns, 12 tiles,
// 10 heads, 64 features 110 -> 46 us).  For two to four key tiles the workgroups of k_bwdm_r stay, whose waves
// share a step: written for several tiles, one wave took 407 us instead of 357 (20 rows of 17 columns, 21
// heads), 43 instead of 41 ((90,37), 18 heads), 640 instead of 597 (480p clip, 52 columns), few blocks most of
// all (43 rows of 20 columns, one head 47 instead of 28).
// ---------------------------------------------------------------------------------------
__device__ inline f32x4 mfma16(s16x4 a, s16x4 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }

template <int D, bool LAST>
__global__ __launch_bounds__(64, 2) void k_bwdm_r_wave(BwdParams bp, int first, int nitems) {
  const KParams& p = bp.k;
  constexpr int LD = D + 16, KS1 = D / 32, NVT = D / 16, LR = 16 + 8;
  __shared__ __attribute__((aligned(16))) u16 Ks[16 * LD];               // K[n, k, i, :]
  __shared__ __attribute__((aligned(16))) u16 As[16 * LD];               // abar[m, n, k, j, :]
  __shared__ __attribute__((aligned(16))) u16 Gs[16 * LD];               // d alpha_L[m, n, j, k, :]
  __shared__ __attribute__((aligned(16))) u16 Ys[LAST ? 16 * LD : 8];    // dY[m, n, j, k, :]
  __shared__ __attribute__((aligned(16))) u16 RT[16 * LR], ST[16 * LR];  // R[j][i], scale dS[j][i]
  const int lane = threadIdx.x, g = lane >> 4, c = lane & 15;
  const int b1 = p.b1, b2 = p.b2;
  const int perrow = p.c2 * b1;                 // key blocks per (batch, head) and key tile row
  const int level = perrow * (nitems / (p.ntk * b1));      // ... and all heads of the pass
  const size_t NKtot = (size_t)p.ntk * b1;
  const float scale2 = p.scale * kLog2e;

  // one work item: a key block.  Key tile rows slowest: under a mask the blocks of the first rows are seen
  // by the most query tiles, and a wave takes one of every row instead of whichever its stride meets.
  struct Item {
    int nk, bhl, bh, k, an, bn, ml0;
    long long krow;
  };
  auto decode = [&](int w) {
    Item it;
    it.an = w / level;
    const int rest = w - it.an * level;
    it.bhl = rest / perrow;
    const int in = rest - it.bhl * perrow;
    it.bn = in / b1;
    it.k = in - it.bn * b1;
    it.nk = it.an * perrow + in;
    it.bh = p.bh0 + it.bhl;
    it.krow = row_offset(p, it.an, it.k);
    it.ml0 = 0;
    while (it.ml0 < p.ntq && it.an >= visible_key_tile_rows((p.m0 + it.ml0) / p.c2, p.c1k, p.ct, p.qt0)) ++it.ml0;
    return it;
  };

  // the columns of a step (lane column = j); lanes beyond b2 repeat the last one
  bf16x8 qv[KS1], gv[KS1], yv[LAST ? KS1 : 1];
  float dcl = 0.f;
  auto fetch = [&](const Item& it, int ml) {
    const int m = p.m0 + ml, a = m / p.c2, bq = m - a * p.c2;
    const int jc = c < b2 ? c : b2 - 1;
    const size_t jr = (((size_t)it.bhl * p.ntq + ml) * b2 + jc) * NKtot + it.nk;
    const u16* ap;
    if (first) {
      const int b = it.bh / p.H, hd = it.bh - b * p.H;
      ap = (const u16*)p.Q + b * p.qs.batch + hd * p.qs.head +
           (row_offset(p, a, it.k) + axis_offset(p.cmap, bq * b2 + jc)) * p.qs.token;
    } else {
      ap = (const u16*)p.aR + ((((size_t)it.bhl * p.ntq + ml) * NKtot + it.nk) * b2 + jc) * D;
    }
    dcl = bp.dcL[jr];
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) {
      qv[ks] = ld_global_16B(ap + 32 * ks + 8 * g);
      gv[ks] = ld_global_16B((const u16*)bp.daL + jr * D + 32 * ks + 8 * g);
      if (LAST) yv[ks] = ld_global_16B((const u16*)bp.dY + jr * D + 32 * ks + 8 * g);
    }
  };
  // waits for a step's rows at the end of the step before it, where the stores issued since are counted
  auto landed = [&]() {
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) {
      u32x4 x = __builtin_bit_cast(u32x4, qv[ks]), y = __builtin_bit_cast(u32x4, gv[ks]);
      asm volatile("" : "+v"(x), "+v"(y));
      qv[ks] = __builtin_bit_cast(bf16x8, x);
      gv[ks] = __builtin_bit_cast(bf16x8, y);
      if (LAST) {
        u32x4 z = __builtin_bit_cast(u32x4, yv[ks]);
        asm volatile("" : "+v"(z));
        yv[ks] = __builtin_bit_cast(bf16x8, z);
      }
    }
    asm volatile("" : "+v"(dcl));
  };

  int w = blockIdx.x;                     // the host launches at most nitems workgroups
  Item cur = decode(w);
  if (cur.ml0 < p.ntq) fetch(cur, cur.ml0);
  const bool live = c < b2;               // this lane's column, and its key
  while (true) {
    // K into LDS, V into operands; rows beyond b2 are zeros
    bf16x8 vv[KS1];
    {
      const int b = cur.bh / p.H, hd = cur.bh - b * p.H;
      const u16* Kp = (const u16*)p.K + b * p.ks.batch + hd * p.ks.head;
      const u16* Vp = (const u16*)p.V + b * p.vs.batch + hd * p.vs.head;
      bf16x8 kk[KS1];
      const long long tok = cur.krow + axis_offset(p.cmap, cur.bn * b2 + (live ? c : b2 - 1));
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        kk[ks] = ld_global_16B(Kp + tok * p.ks.token + 32 * ks + 8 * g);
        if (LAST) vv[ks] = ld_global_16B(Vp + tok * p.vs.token + 32 * ks + 8 * g);
      }
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        const uint4 zero = {0u, 0u, 0u, 0u};
        *(uint4*)(Ks + c * LD + 32 * ks + 8 * g) = live ? __builtin_bit_cast(uint4, kk[ks]) : zero;
        if (LAST) vv[ks] = as_bf16x8(live ? __builtin_bit_cast(uint4, vv[ks]) : zero);
      }
    }
    const int w2 = w + (int)gridDim.x;
    const bool more = w2 < nitems;
    const Item nxt = more ? decode(w2) : cur;
    f32x4 oK[NVT], oV[LAST ? NVT : 1];
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) {
      oK[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (LAST) oV[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    landed();
    for (int ml = cur.ml0; ml < p.ntq; ++ml) {
      // S^T and dR^T: rows i = 4 g + r, lane column j
      f32x4 s = {0.f, 0.f, 0.f, 0.f}, dr = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        const bf16x8 k = ld_lds_16B(Ks + c * LD + 32 * ks + 8 * g);
        s = mfma(k, qv[ks], s);
        dr = mfma(k, gv[ks], dr);
        if (LAST) dr = mfma(vv[ks], yv[ks], dr);
      }
      const float dc = dcl;
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) {
        const uint4 zero = {0u, 0u, 0u, 0u};
        const int at = c * LD + 32 * ks + 8 * g;
        *(uint4*)(As + at) = live ? __builtin_bit_cast(uint4, qv[ks]) : zero;
        *(uint4*)(Gs + at) = live ? __builtin_bit_cast(uint4, gv[ks]) : zero;
        if (LAST) *(uint4*)(Ys + at) = live ? __builtin_bit_cast(uint4, yv[ks]) : zero;
      }
      __builtin_amdgcn_sched_barrier(0);
      // the next step: the next query tile, or the next block's first
      if (ml + 1 < p.ntq) fetch(cur, ml + 1);
      else fetch(nxt, nxt.ml0 < p.ntq ? nxt.ml0 : p.ntq - 1);
      __builtin_amdgcn_sched_barrier(0);

      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] = 4 * g + r < b2 ? s[r] * scale2 : -INFINITY;
        mx = fmaxf(mx, s[r]);
      }
      mx = xmax(mx);
      float sum = 0.f;
      f32x4 ex;                                      // 2^(logit - maximum): R times the sum
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] -= mx;
        ex[r] = exp2_fast(s[r]);
        sum += ex[r];
      }
      sum = xsum(sum);
      const float inv = 1.0f / sum, lsum = log2_fast(sum);
      float dot = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float R = ex[r] * inv;                               // 0 beyond b2
        const float dR = 4 * g + r < b2 ? dr[r] + dc * fmaf(s[r] - lsum, kLn2, 1.0f) : 0.f;
        ex[r] = R;
        dr[r] = dR;
        dot = fmaf(R, dR, dot);
      }
      dot = xsum(dot);
#pragma unroll
      for (int r = 0; r < 4; ++r) dr[r] = p.scale * ex[r] * (dr[r] - dot);   // scale dS
      typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
      const bf16x4 R = {(__bf16)ex[0], (__bf16)ex[1], (__bf16)ex[2], (__bf16)ex[3]};
      const bf16x4 S = {(__bf16)dr[0], (__bf16)dr[1], (__bf16)dr[2], (__bf16)dr[3]};
      {
        const uint2 zero = {0u, 0u};
        *(uint2*)(RT + c * LR + 4 * g) = live ? __builtin_bit_cast(uint2, R) : zero;
        *(uint2*)(ST + c * LR + 4 * g) = live ? __builtin_bit_cast(uint2, S) : zero;
      }
      // d abar[j] = sum_i (scale dS[j, i]) K[i]
      {
        f32x4 o[NVT];
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) o[vt] = f32x4{0.f, 0.f, 0.f, 0.f};
        const u16* at = Ks + (4 * g + (c >> 2)) * LD + 8 * (c & 3);
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt)
          o[vt] = mfma16(ld_lds_tr(at + 32 * (vt >> 1) + 4 * (vt & 1)), __builtin_bit_cast(s16x4, S), o[vt]);
        const int nk = cur.nk;
        if (first && bp.dq_from_r) {
          const int m = p.m0 + ml, a = m / p.c2, bq = m - a * p.c2;
          if (live) {
            const long long tok = row_offset(p, a, cur.k) + axis_offset(p.cmap, bq * b2 + c);
            store_rows_f32<D>(bp.dQ + ((size_t)cur.bh * p.Nq + tok) * D, o, 1.0f, g, true);
          }
        } else {
          const size_t ablk = (((size_t)cur.bhl * p.ntq + ml) * NKtot + nk) * b2;
          store_ws_row<D>((u16*)bp.dA + (ablk + (live ? c : b2 - 1)) * D, o, 1.0f, g);   // (the last column, once more)
        }
      }
      // dK += R^T d alpha_L + scale dS^T abar, dV += R^T dY over the step's columns
      {
        const int rc = (4 * g + (c >> 2)) * LR + 4 * (c & 3), xc = (4 * g + (c >> 2)) * LD + 8 * (c & 3);
        const s16x4 bR = ld_lds_tr(RT + rc), bS = ld_lds_tr(ST + rc);
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) {
          const int at = xc + 32 * (vt >> 1) + 4 * (vt & 1);
          const s16x4 xg = ld_lds_tr(Gs + at), xa = ld_lds_tr(As + at);
          s16x4 xy;
          if (LAST) xy = ld_lds_tr(Ys + at);
          oK[vt] = mfma16(xg, bR, oK[vt]);
          oK[vt] = mfma16(xa, bS, oK[vt]);
          if (LAST) oV[vt] = mfma16(xy, bR, oV[vt]);
        }
      }
      landed();
    }
    if (live) {
      const long long tok = cur.krow + axis_offset(p.cmap, cur.bn * b2 + c);
      float* to = bp.dK + ((size_t)cur.bh * p.Nkv + tok) * D;
      if (first && !bp.accumulate) store_rows_f32_nt<D>(to, oK, 1.0f, g);
      else store_rows_f32<D>(to, oK, 1.0f, g, bp.accumulate != 0);
      if (LAST) store_rows_f32_nt<D>(bp.dV + ((size_t)cur.bh * p.Nkv + tok) * D, oV, 1.0f, g);
    }
    if (!more) break;
    if (cur.ml0 >= p.ntq && nxt.ml0 < p.ntq) fetch(nxt, nxt.ml0);     // (a block that no query tile sees fetched nothing)
    cur = nxt;
    w = w2;
  }
}

template <int D>
hipError_t keys_d(const BwdParams& bp, dim3 grid, int nlt, hipStream_t s) {
  if (nlt <= 2) k_bwdm_l_keys<D, 2><<<grid, 256, 0, s>>>(bp);      // (an operand holds two query tiles)
  else if (nlt <= 4) k_bwdm_l_keys<D, 4><<<grid, 256, 0, s>>>(bp);
  else k_bwdm_l_keys<D, 6><<<grid, 256, 0, s>>>(bp);
  return hipGetLastError();
}

template <int D, bool LAST>
hipError_t r_wave_d(const BwdParams& bp, int nitems, bool first, hipStream_t s) {
  static const int resident = resident_workgroups(k_bwdm_r_wave<D, LAST>, 64);
  k_bwdm_r_wave<D, LAST><<<dim3(nitems < resident ? nitems : resident), 64, 0, s>>>(bp, first ? 1 : 0, nitems);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_bf16_keys(const BwdParams& bp, dim3 grid, int nlt, hipStream_t s) {
  return bp.k.d == 128 ? keys_d<128>(bp, grid, nlt, s) : keys_d<64>(bp, grid, nlt, s);
}

hipError_t launch_bwd_bf16_r_wave(const BwdParams& bp, int nitems, bool first, bool last, hipStream_t s) {
  if (bp.k.d == 128) return last ? r_wave_d<128, true>(bp, nitems, first, s) : r_wave_d<128, false>(bp, nitems, first, s);
  return last ? r_wave_d<64, true>(bp, nitems, first, s) : r_wave_d<64, false>(bp, nitems, first, s);
}

}  // namespace mrt
