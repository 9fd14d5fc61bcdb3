// Dense softmax attention baseline on the bf16 matrix unit (Sec. 2.2), chunk-causal by token.
// See the head of mrt_bf16.hip for the register layouts.
//
// Eight waves, two to a SIMD, each owning QT query tiles of 16.  A step of 64 keys is a vector phase
// (maxima, exponentials, packing, the refill of the LDS ring) and a matrix phase (first product of the
// next step, second product of this one, their LDS reads), and the two halves of the workgroup run one
// phase apart: one wave of a SIMD feeds the matrix unit while the other one has the vector ALU.  The
// barrier that ends every phase keeps them so.  (Without it the waves drift into step and the two
// units take turns: a matrix unit busy 35 % of the time.)  What bounds the kernel then is the vector
// phase (vector instructions issue at half rate under the other wave's products) and about 150 clocks
// of barrier per phase; hence phases of 64 keys (two chunks).  The sums of the probabilities are fp32
// additions of the unrounded values: a product with ones over the rounded ones takes them off the
// vector ALU (3 to 6 % of a call), but shortens the denominator by up to 2^-8 where the roundings agree.
//
// LDS rows are padded to D + 16 elements (288 bytes at D = 128): the 16-byte key reads and the
// transposed value reads of 16 contiguous features then both run free of bank conflicts (4.0 and 2.8
// clocks per wave instruction and CU measured; a 16-byte XOR swizzle 6.0 and 4.0).
//
// WK = 1: every wave sees all keys.  WK = 2: waves w and w + 4 share their queries and take one half of
// every 64 keys (half the queries per workgroup, so twice the workgroups); the halves are merged at the
// end.
//
// PART: a workgroup takes one of `parts` runs of 64-key pairs and leaves its accumulators, references and
// sums in fp32 for k_dense_merge; for calls of few queries (dense_shape).
#include "mrt_internal.hpp"
#include "mrt_bf16_tiles.hpp"

#include <algorithm>

namespace mrt {

namespace {

// A query's softmax reference is raised only when a logit exceeds it by more than this (base 2):
// every probability is then at most 2^kGrow, and the ratio sum(p v) / sum(p) does not depend on it.
constexpr float kGrow = 8.0f;
constexpr float kNoKey = -__FLT_MAX__;   // reference of a query that has seen no key
// Beyond this the rounding of a reference, which its own logit's exponent would contain (one fma), is no
// longer small beside kGrow: every step then counts as one that raises it, and there the exponents are
// formed from logits that are rounded first.  (A choice between the two on the common path costs a
// quarter of the call at 64 features: it parts the exponentials from the rest of the vector phase.)
constexpr float kFarRef = 0x1p20f;
constexpr int kDenseWaves = 8, kDenseThreads = 64 * kDenseWaves;
// LDS ring of 64-key pairs of chunks: while pair i is consumed, pair i + 1 is resident, pair i + 2 is
// being written and pair i + 3 is in flight from global memory.
constexpr int kDenseSlots = 4;
constexpr int kAhead = 5;    // operand reads ahead of their products (3, 5 and 7 measured alike)
template <int D> constexpr int kDenseLd = D + 16;                          // elements per LDS row
template <int D> constexpr int kDenseSlot = 2 * 64 * kDenseLd<D>;          // 64 keys, then 64 values
template <int D> constexpr size_t kDenseLds = (size_t)kDenseSlots * kDenseSlot<D> * 2;

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// 64 rows of D bf16 between global memory and LDS.  Buffer loads return zeros beyond the last row, so
// no load is clamped or conditional.
template <int D>
struct DenseTile {
  static constexpr int CPR = D / 8, N = 64 * CPR / kDenseThreads, RSTEP = kDenseThreads / CPR;
  u32x4 v[N];
  // at: byte offset of the tile's first row
  __device__ inline void load(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned at, unsigned rowbytes) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + (at + (unsigned)(i * RSTEP) * rowbytes), 0, 0);
  }
  __device__ inline void store(u16* dst, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) *(u32x4*)(dst + (tid / CPR + i * RSTEP) * kDenseLd<D> + 8 * (tid % CPR)) = v[i];
  }
};

// Keys query q sees: the frames up to the end of its own chunk, a prefix.
__host__ __device__ inline int dense_visible(const KParams& p, int q) {
  if (p.cc == 0) return p.Nkv;
  const long long lim = (long long)((p.qoff + q / p.hw) / p.cc + 1) * p.cc * p.hw;
  return lim < p.Nkv ? (int)lim : p.Nkv;
}

// Partial results of a call whose keys are split over `n` workgroups per query tile: every part's
// accumulators, softmax reference and sum of a query (row = (part, head, query)).
struct DenseParts {
  float* o;     // [part][bh][q][D]
  float2* ml;   // [part][bh][q]
  int n;
};

// (64 features: two workgroups to a compute unit)
template <int D, int QT, int WK, bool PART>
__global__ __launch_bounds__(kDenseThreads, D == 64 ? 4 : 2) void k_bf16_dense(KParams p, DenseParts parts) {
  using Tile = DenseTile<D>;
  constexpr int KS1 = D / 32, NVT = D / 16, LD = kDenseLd<D>, WQ = kDenseWaves / WK, WGQ = 16 * QT * WQ;
  constexpr int NS = 2 / WK, NT = 2 * NS;                 // 32-key chunks / 16-key tiles of a wave's step
  extern __shared__ __attribute__((aligned(16))) u16 dense_lds[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int wq = wave % WQ, wk = wave / WQ;
  const bool second = wave >= kDenseWaves / 2;           // the half that runs one phase behind
  auto visible = [&](int q) { return dense_visible(p, q); };
  // Workgroups reach the eight XCDs in turn: hand each XCD a contiguous run of (head, query tile)
  // units, so that the units that stream the same keys share its L2.  (Under a mask that gives the
  // query tiles of a head different key counts the natural order spreads the long ones evenly.)
  const int nx = (p.Nq + WGQ - 1) / WGQ, total = gridDim.x, xcd = blockIdx.x & 7;
  int unit = blockIdx.x;
  if (visible(0) == visible(p.Nq - 1)) unit = xcd * (total >> 3) + (xcd < (total & 7) ? xcd : (total & 7)) + (blockIdx.x >> 3);
  const int run = unit / nx, q0 = (unit - run * nx) * WGQ;         // run = (head, part)
  const int bh = PART ? run / parts.n : run, part = PART ? run - bh * parts.n : 0;
  const int b = bh / p.H, hd = bh - b * p.H;
  const int qw0 = q0 + 16 * QT * wq;                      // this wave's first query
  const int nkeys = visible(q0 + WGQ - 1 < p.Nq ? q0 + WGQ - 1 : p.Nq - 1), nfree = visible(q0);

  const u16* Qp = (const u16*)p.Q + b * p.qs.batch + hd * p.qs.head;
  bf16x8 qv[QT][KS1];
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int qi = qw0 + 16 * q + c, qc = qi < p.Nq ? qi : p.Nq - 1;
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) qv[q][ks] = ld_global_16B(Qp + (long long)qc * p.qs.token + 32 * ks + 8 * g);
  }

  const unsigned krow = (unsigned)p.ks.token * 2u, vrow = (unsigned)p.vs.token * 2u;     // bytes per token
  // 256 queries: the first half's 128 stop at key `mid`, and a pair of chunks ends there, so that no value
  // hidden from all of them meets their weights of zero (0 x inf); the rest is the second half's alone
  const int mid = WK == 1 ? visible(q0 + WGQ / 2 - 1 < p.Nq ? q0 + WGQ / 2 - 1 : p.Nq - 1) : nkeys;
  const int nmid = (mid + 63) >> 6, npairs = nmid + ((nkeys - mid + 63) >> 6);
  auto first_key = [&](int pr) { return pr < nmid ? 64 * pr : mid + 64 * (pr - nmid); };
  const int p0 = PART ? part * npairs / parts.n : 0, p1 = PART ? (part + 1) * npairs / parts.n : npairs;   // this part's pairs
  const u16* Kp = (const u16*)p.K + b * p.ks.batch + hd * p.ks.head;
  const u16* Vp = (const u16*)p.V + b * p.vs.batch + hd * p.vs.head;
  const unsigned kvoff = (unsigned)(tid / Tile::CPR) * krow + 16u * (tid % Tile::CPR);
  const unsigned vvoff = (unsigned)(tid / Tile::CPR) * vrow + 16u * (tid % Tile::CPR);
  Tile kt, vt;
  // (pairs past the end re-read the last one; nobody reads their slot, or only as masked keys)
  auto fetch = [&](int pr) {
    const int last = PART && p1 > p0 ? p1 : npairs, at = pr < last ? pr : last - 1, end = at < nmid ? mid : nkeys;
    const unsigned key = (unsigned)first_key(at), rows = (unsigned)(end - 1);
    kt.load(__builtin_amdgcn_make_buffer_rsrc((void*)Kp, 0, rows * krow + 2 * D, 0x00020000), kvoff, key * krow, krow);
    vt.load(__builtin_amdgcn_make_buffer_rsrc((void*)Vp, 0, rows * vrow + 2 * D, 0x00020000), vvoff, key * vrow, vrow);
  };
  auto commit = [&](int slot) {
    u16* at = dense_lds + slot * kDenseSlot<D>;
    kt.store(at, tid);
    vt.store(at + 64 * LD, tid);
  };

  const float scale2 = p.scale * kLog2e;
  bf16x8 pb[QT][NS];
  f32x4 s[QT][NT], o[QT][NVT];
  float mref[QT], thr[QT];                // reference, the raw logit that would raise it (kFarRef: any would)
  float mul[QT], off[QT];                 // a step's exponents are s mul - off: scale and reference, or 1 and 0 (kFarRef)
  float lrun[QT];                         // this lane's sum of the (unrounded) probabilities
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    mref[q] = off[q] = kNoKey; mul[q] = scale2; thr[q] = -INFINITY; lrun[q] = 0.f;
#pragma unroll
    for (int vt = 0; vt < NVT; ++vt) o[q][vt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // A wave's keys of a pair start at row 32 wk (WK = 2) or 0.
  const int koff = (WK == 2 ? 32 * wk * LD : 0) + c * LD + 8 * g;
  const int voff = 64 * LD + (WK == 2 ? 32 * wk * LD : 0) + (4 * g + (c >> 2)) * LD + 4 * (c & 3);
  // The matrix phase: s = logits of the next step's keys (pair in kslot), o += the probabilities'
  // product with this step's values (pair in vslot).  Operands are read from LDS kAhead groups of
  // products ahead of their use, in this fixed order.
  constexpr int NK_OPS = NT * KS1, NV_OPS = NS * NVT, OPS = NK_OPS + NV_OPS;
  bf16x8 op[OPS];
  auto read_op = [&](int i, const u16* ka, const u16* va) {
    if (i < NK_OPS) {
      op[i] = ld_lds_16B(ka + 16 * (i % NT) * LD + 32 * (i / NT));
    } else {
      const u16* at = va + 32 * ((i - NK_OPS) / NVT) * LD + 16 * ((i - NK_OPS) % NVT);
      op[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(ld_lds_tr(at), ld_lds_tr(at + 16 * LD), 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  auto matrix = [&](int kslot, int vslot, bool with_v) {
    const u16* ka = dense_lds + kslot * kDenseSlot<D> + koff;
    const u16* va = dense_lds + vslot * kDenseSlot<D> + voff;
#pragma unroll
    for (int i = 0; i < kAhead; ++i) read_op(i, ka, va);
#pragma unroll
    for (int i = 0; i < OPS; ++i) {
      if (!with_v && i >= NK_OPS) break;
      if (i + kAhead < (with_v ? OPS : NK_OPS)) read_op(i + kAhead, ka, va);
      if (i < NK_OPS) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
          s[q][i % NT] = mfma(op[i], qv[q][i / NT], i < NT ? f32x4{0.f, 0.f, 0.f, 0.f} : s[q][i % NT]);
      } else {
        const int st = (i - NK_OPS) / NVT, vt = (i - NK_OPS) % NVT;
#pragma unroll
        for (int q = 0; q < QT; ++q) o[q][vt] = mfma(op[i], pb[q][st], o[q][vt]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto top = [&](int q) {
    float m = fmaxf(s[q][0][0], s[q][0][1]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t > 0) m = fmaxf(m, fmaxf(s[q][t][0], s[q][t][1]));
      m = fmaxf(m, fmaxf(s[q][t][2], s[q][t][3]));
    }
    return m;
  };
  // the raw logits of the keys from c0 on are complete: mask them where they reach beyond a query's
  // keys or the pair's end, raise the references they exceed, and form the probabilities
  auto soften = [&](int c0, int end) {
    if (c0 + 16 * NT > nfree) {
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        const int qi = qw0 + 16 * q + c, seen = visible(qi < p.Nq ? qi : p.Nq - 1), lim = seen < end ? seen : end;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (c0 + 16 * t + 4 * g + r >= lim) s[q][t][r] = -INFINITY;
      }
    }
    bool above = false;
#pragma unroll
    for (int q = 0; q < QT; ++q) above |= top(q) > thr[q];
    if (__builtin_amdgcn_ballot_w64(above) != 0) {
#pragma unroll
      for (int q = 0; q < QT; ++q) {
        const float mnew = fmaxf(mref[q], mul_rounded(xmax(top(q)), scale2));
        const float f = exp2_fast(mref[q] - mnew);
        const bool far = mnew > kNoKey && fabsf(mnew) > kFarRef;
        mref[q] = mnew;
        mul[q] = far ? 1.0f : scale2;
        off[q] = far ? 0.0f : mnew;
        thr[q] = (mnew + (far ? -INFINITY : kGrow)) / scale2;     // (no branch: it would part the loop)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[q][t][r] = far ? mul_rounded(s[q][t][r], scale2) - mnew : s[q][t][r];
        lrun[q] *= f;
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) o[q][vt] = o[q][vt] * f;
      }
    }
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[q][t][r] = exp2_fast(fmaf(s[q][t][r], mul[q], -off[q]));
          sum += s[q][t][r];
        }
      lrun[q] += sum;
#pragma unroll
      for (int st = 0; st < NS; ++st) pb[q][st] = pack8(s[q][2 * st], s[q][2 * st + 1]);
    }
  };
  auto phase_end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };

  fetch(p0);
  const Tile k0 = kt, v0 = vt;
  fetch(p0 + 1);
  const Tile k1 = kt, v1 = vt;
  fetch(p0 + 2);
  k0.store(dense_lds + (p0 & (kDenseSlots - 1)) * kDenseSlot<D>, tid);
  v0.store(dense_lds + (p0 & (kDenseSlots - 1)) * kDenseSlot<D> + 64 * LD, tid);
  k1.store(dense_lds + ((p0 + 1) & (kDenseSlots - 1)) * kDenseSlot<D>, tid);
  v1.store(dense_lds + ((p0 + 1) & (kDenseSlots - 1)) * kDenseSlot<D> + 64 * LD, tid);
  __syncthreads();
  matrix(p0 & (kDenseSlots - 1), 0, false);
  if (second) __syncthreads();
  auto step = [&](int i, int end, bool mine) {
    if (mine) soften(first_key(i) + (WK == 2 ? 32 * wk : 0), end);
    // pair i + 2 into the slot of pair i - 2, which both halves left at least a phase ago (the other
    // half may still be reading pairs i - 1 and i)
    commit((i + 2) & (kDenseSlots - 1));
    fetch(i + 3);
    phase_end();
    __builtin_amdgcn_s_setprio(1);
    if (mine) matrix((i + 1) & (kDenseSlots - 1), i & (kDenseSlots - 1), true);
    __builtin_amdgcn_s_setprio(0);
    phase_end();
  };
  for (int i = p0; i < (PART && p1 < nmid ? p1 : nmid); ++i) step(i, mid, true);
  if constexpr (WK == 1) {
    for (int i = PART && p0 > nmid ? p0 : nmid; i < p1; ++i) step(i, nkeys, second);
  }
  if (!second) __syncthreads();

  if constexpr (WK == 2) {
    // the second half's reference, sum and accumulators, merged into the first half's
    f32x4* xo = (f32x4*)dense_lds + (size_t)wq * (QT * (NVT + 1)) * 64 + lane;
    __syncthreads();
    if (wk == 1) {
#pragma unroll
      for (int q = 0; q < QT; ++q) {
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) xo[(q * (NVT + 1) + vt) * 64] = o[q][vt];
        xo[(q * (NVT + 1) + NVT) * 64] = f32x4{mref[q], lrun[q], 0.f, 0.f};
      }
    }
    __syncthreads();
    if (wk == 1) return;
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const f32x4 ml = xo[(q * (NVT + 1) + NVT) * 64];
      const float m = fmaxf(mref[q], ml[0]), f0 = exp2_fast(mref[q] - m), f1 = exp2_fast(ml[0] - m);
      lrun[q] = lrun[q] * f0 + ml[1] * f1;
      mref[q] = m;
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) o[q][vt] = o[q][vt] * f0 + xo[(q * (NVT + 1) + vt) * 64] * f1;
    }
  }
  if constexpr (PART) {
    const long long row0 = ((long long)part * (total / (nx * parts.n)) + bh) * p.Nq;
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int qi = qw0 + 16 * q + c;
      const float lsum = xsum(lrun[q]);
      if (qi < p.Nq) {
        float* row = parts.o + (row0 + qi) * D + 4 * g;
#pragma unroll
        for (int vt = 0; vt < NVT; ++vt) *(f32x4*)(row + 16 * vt) = o[q][vt];
        if (g == 0) parts.ml[row0 + qi] = make_float2(mref[q], lsum);
      }
    }
    return;
  }
  u16* Op = (u16*)p.O + b * p.os.batch + hd * p.os.head;
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int qi = qw0 + 16 * q + c;
    const float lsum = xsum(lrun[q]), inv = lsum > 0.f ? 1.0f / lsum : 0.f;
    if (qi < p.Nq) {
      u16* row = Op + (long long)qi * p.os.token + 4 * g;
#pragma unroll
      for (int vt = 0; vt < NVT; ++vt) {
        const f32x4 x = o[q][vt] * inv;
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
        *(bf16x4*)(row + 16 * vt) = bf16x4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
      }
    }
  }
}

// O from the parts: every part's sum and accumulators against the largest reference.  A thread owns
// four features of a query and has eight parts in flight at once: what it waits for is memory.
template <int D>
__global__ __launch_bounds__(256) void k_dense_merge(KParams p, DenseParts parts, int rows) {
  constexpr int TPR = D / 4, AHEAD = 8;
  const int row = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, f = 4 * (threadIdx.x % TPR);
  if (row >= rows) return;
  float m = kNoKey, lsum = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < parts.n; i0 += AHEAD) {
    float2 ml[AHEAD];
    f32x4 po[AHEAD];
#pragma unroll
    for (int e = 0; e < AHEAD; ++e) {
      const size_t at = (size_t)(i0 + e < parts.n ? i0 + e : parts.n - 1) * rows + row;
      ml[e] = parts.ml[at];
      po[e] = *(const f32x4*)(parts.o + at * D + f);
    }
    float top = m;
#pragma unroll
    for (int e = 0; e < AHEAD; ++e) top = fmaxf(top, ml[e].x);
    const float keep = exp2_fast(m - top);
    m = top;
    lsum *= keep;
    o = o * keep;
#pragma unroll
    for (int e = 0; e < AHEAD; ++e)
      if (i0 + e < parts.n) {
        const float w = exp2_fast(ml[e].x - m);
        lsum += ml[e].y * w;
        o = o + po[e] * w;
      }
  }
  const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
  const f32x4 x = o * inv;
  const int bh = row / p.Nq, q = row - bh * p.Nq, b = bh / p.H, hd = bh - b * p.H;
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  *(bf16x4*)((u16*)p.O + b * p.os.batch + hd * p.os.head + (long long)q * p.os.token + f) =
      bf16x4{(__bf16)x[0], (__bf16)x[1], (__bf16)x[2], (__bf16)x[3]};
}

template <int D, int QT, int WK, bool PART>
hipError_t run_dense(const KParams& kp, int nbh, const DenseParts& parts, hipStream_t s) {
  const hipError_t e = hipFuncSetAttribute((const void*)k_bf16_dense<D, QT, WK, PART>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDenseLds<D>);
  if (e != hipSuccess) return e;
  constexpr int wgq = 16 * QT * kDenseWaves / WK;
  k_bf16_dense<D, QT, WK, PART><<<(kp.Nq + wgq - 1) / wgq * nbh * parts.n, kDenseThreads, kDenseLds<D>, s>>>(kp, parts);
  if constexpr (PART) {
    const int rows = nbh * kp.Nq, rpw = 256 / (D / 4);
    k_dense_merge<D><<<(rows + rpw - 1) / rpw, 256, 0, s>>>(kp, parts, rows);
  }
  return hipGetLastError();
}

// A call takes as many rounds as its workgroups fill the chip; the shape with the least rounds x cost.
//
// 128 features: a workgroup occupies a compute unit.  A round of 4680 keys costs 61, 79 and 126 us for
// workgroups of 64 (QT = 1, WK = 2), 128 (QT = 2, WK = 2) and 256 (QT = 2) queries (one head of 4680
// tokens 59 | 78 | 122 us, 5 heads 120 | 80 | 123, 12 heads 233 | 159 | 130, 16 heads 294 | 238 | 256).
// Where a mask gives the query tiles different key counts the short ones fill the last round, and the
// largest shape, which reads the keys least often, is taken at 112 (24 heads of 12 one-frame chunks of
// 320 tokens 203 | 173 | 162, 10 heads of 2 chunks of 4680 tokens 575 | 444 | 399).
//
// 64 features: two workgroups of 64 or 128 queries share a compute unit; a round of up to one per unit
// costs 40 and 57 us, of up to two 54 and 90 (one head of 4680 tokens 38 | 57, 5 heads 53 | 58, 8 heads
// 92 | 87, 16 heads 145 | 134; 40 heads of 1560 tokens 43 | 52).  Workgroups of 256, one per unit, take
// 88 a round: never ahead of 128 by more than 3 %, behind by up to 1.5 x.  Under a mask the workgroups
// count by their share of the longest one's keys (12 heads of 3 chunks of 1040 tokens 50 | 63, 16 heads
// 63 | 64, 32 heads 101 | 98).
//
// Splitting the keys.  Calls of few queries leave most of the chip idle however small their workgroups
// are (one head of 816 queries, 3264 keys: 26 workgroups of 64 queries, 43.6 us), so `parts` workgroups
// share the keys of a query tile and a second launch merges their partial results.  `time` is a model of
// a call fitted to 700 measured shapes of 29 calls (rounds x steps of 64 keys x microseconds a step, the merge
// launch, the partial results' bytes) and, for calls under a mask, to another 1600: there one round lasts as long
// as its longest workgroup, and of several the units that finish early take the next one's workgroups.  A split
// has to promise 6 %: 928 drawn calls that are split so take 0.64 of the unsplit time on average, four of them
// more than that time, up to 1.034.  (Counted as if units could finish early in a single round, 128 features, or as if
// workgroups beyond the last full round cost nothing, 64, calls under a mask took up to 1.43 of the unsplit time.)
// (2 heads of 816 queries of 3264 keys 43.6 -> 19 us, one
// head of 7080 of 21240 244 -> 88, 4 heads of 1989 of 7956 96 -> 49, 6 heads of 7020 of 21060 501 -> 415;
// 64 features: one head of 3240 of 12960 96 -> 30.  No split: 384 keys 10.6 (two parts 12.6), 12 heads of
// 4680 of 4680 132 (155), under a mask 15 heads of 3240 of 6480 172 (201).)
constexpr int kMostParts = 32;
constexpr size_t kMostPartsBytes = (size_t)128 << 20;       // of partial results
constexpr long long kMostSplitRows = 1 << 18;               // 2^18 rows of two parts are more than that

size_t dense_parts_bytes(int rows, int parts, int d) { return (size_t)rows * parts * (d + 2) * sizeof(float); }

struct DenseShape {
  int queries, parts;    // queries per workgroup, workgroups that share the keys of one query tile
};

DenseShape dense_shape(const KParams& kp, int nbh, bool may_split) {
  const long long cus = compute_units(), first = dense_visible(kp, 0), last = dense_visible(kp, kp.Nq - 1);
  auto wgs = [&](int queries) { return (long long)((kp.Nq + queries - 1) / queries) * nbh; };
  DenseShape best;
  if (kp.d == 64) {
    auto cost = [&](int queries, long long one, long long two) {
      const long long n = (wgs(queries) * (first + last) + 2 * last - 1) / (2 * last), rest = n % (2 * cus);
      return n / (2 * cus) * two + (rest > cus ? two : rest > 0 ? one : 0);
    };
    best = {cost(64, 40, 54) < cost(128, 57, 90) ? 64 : 128, 1};
  } else {
    auto cost = [&](int queries, long long unit) { return (wgs(queries) + cus - 1) / cus * unit; };
    const long long c256 = cost(256, first == last ? 126 : 112), c128 = cost(128, 79), c64 = cost(64, 61);
    best = {c64 < c128 && c64 < c256 ? 64 : c128 < c256 ? 128 : 256, 1};
  }
  if (!may_split || (long long)kp.Nq * nbh > kMostSplitRows) return best;
  const long long pairs = (last + 63) / 64;
  auto time = [&](int queries, int parts) {
    const double steps = (double)((pairs + parts - 1) / parts), share = (double)(first + last) / (2 * last);
    const long long n = wgs(queries) * parts;
    double us = 0;
    if (kp.d == 64) {
      const double one = queries == 64 ? 0.45 : 0.72, two = queries == 64 ? 0.67 : 1.12;
      const long long rest = n % (2 * cus);
      double full = n / (2 * cus) * two + (rest > cus ? two : rest > 0 ? one : 0);
      if (first != last)
        full = n > 2 * cus ? std::max(two, n * share / (2 * cus) * two + 0.7 * one)
                           : one + (two - one) * std::min(1.0, std::max(0.0, (n - cus) / 64.0));
      us = 6.0 + full * steps;
      if (parts > 1) us += 4.2;
    } else {
      const long long rounds = (n + cus - 1) / cus;
      const double full = first == last ? (double)rounds : std::min((double)rounds, std::max(1.0, n * share / cus + 0.8));
      us = 3.4 + 4.1 * rounds + full * steps * (queries == 64 ? 0.71 : queries == 128 ? 1.02 : 1.56);
      if (parts > 1) us += 5.5;
    }
    const double mb = 1e-6 * 2 * dense_parts_bytes(kp.Nq * nbh, parts, kp.d);      // written, read
    return parts > 1 ? us + mb / (kp.d == 64 ? 3.0 : 5.7) : us;
  };
  const DenseShape one = best;
  // Queries of one run (a workgroup, or its half if it has 256) meet the values of every key that one of
  // them sees, with weights of zero where they don't: an infinite value hidden from some of them shows in
  // them all.  A split takes no run longer than the unsplit call's that a chunk could end inside.
  auto run_ok = [&](int queries) {
    const long long run = std::min(queries, 128);
    return first == last || run <= one.queries || ((long long)kp.cc * kp.hw % run == 0 && (long long)kp.qoff * kp.hw % run == 0);
  };
  double least = time(one.queries, 1) / 1.06;
  for (int queries = 64; queries <= (kp.d == 64 ? 128 : 256); queries *= 2) {
    if (!run_ok(queries)) continue;
    for (int parts = 2; parts <= kMostParts && parts <= pairs; ++parts) {
      if (dense_parts_bytes(kp.Nq * nbh, parts, kp.d) > kMostPartsBytes || wgs(queries) * parts > 6 * cus) break;
      const double us = time(queries, parts);
      if (us < least) { least = us; best = {queries, parts}; }
    }
  }
  return best;
}

template <int D, bool PART>
hipError_t run_dense_d(const KParams& kp, int nbh, int queries, const DenseParts& parts, hipStream_t s) {
  if (queries == 64) return run_dense<D, 1, 2, PART>(kp, nbh, parts, s);
  if constexpr (D == 128)
    if (queries == 256) return run_dense<D, 2, 1, PART>(kp, nbh, parts, s);
  return run_dense<D, 2, 2, PART>(kp, nbh, parts, s);
}

}  // namespace

size_t bf16_dense_workspace_bytes(const KParams& kp, int nbh) {
  const DenseShape shape = dense_shape(kp, nbh, true);
  return shape.parts > 1 ? dense_parts_bytes(kp.Nq * nbh, shape.parts, kp.d) : 0;
}

hipError_t launch_bf16_dense(const KParams& kp, int nbh, void* workspace, size_t workspace_bytes, hipStream_t s) {
  DenseShape shape = dense_shape(kp, nbh, workspace != nullptr);
  if (shape.parts > 1 && workspace_bytes < dense_parts_bytes(kp.Nq * nbh, shape.parts, kp.d)) shape = dense_shape(kp, nbh, false);
  const size_t rows = (size_t)kp.Nq * nbh * shape.parts;
  const DenseParts parts = {(float*)workspace, (float2*)((float*)workspace + rows * kp.d), shape.parts};
  if (kp.d == 128)
    return shape.parts > 1 ? run_dense_d<128, true>(kp, nbh, shape.queries, parts, s) : run_dense_d<128, false>(kp, nbh, shape.queries, parts, s);
  return shape.parts > 1 ? run_dense_d<64, true>(kp, nbh, shape.queries, parts, s) : run_dense_d<64, false>(kp, nbh, shape.queries, parts, s);
}

}  // namespace mrt
