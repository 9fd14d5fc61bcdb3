// fp32 path: fp32 arithmetic and fp32 intermediates; every contraction runs on the matrix unit in
// fp32 (v_mfma_f32_16x16x4_f32: an fp32 dot product in another summation order).
//
// Used for f32 storage (the 1e-4 parity class) and, on request, as a device-side
// cross-check for bf16 storage.  Same three stages as the bf16 path:
//   stage R      one workgroup per (m, n, k): Z_R, R = softmax_i, c_L, alpha_L, (Y)
//   stage L out  one workgroup per (m, j): online softmax over nk, O = L Y
//   stage L ref  one workgroup per (m, j): alpha_R / c_R of the next iteration
// Equation references: App. A.1 / A.2 update equations.
//
// What bounds these kernels is the fp32 matrix rate (64 flop per clock and SIMD, a sixteenth of the
// bf16 rate), so the layout is chosen to feed it from registers and 16-byte LDS reads with nothing
// in between.  Lane (g = lane / 16, c = lane % 16) supplies A[c][k = g] and B[k = g][c] of a step and
// holds C[4g + r][c] in register r.
//   * First products contract over features, which are contiguous in both operands: with feature
//     16 ks + 4 g + e as slot g of step (ks, e), a lane's operands of four steps are 16 contiguous
//     bytes.
//   * Queries sit on the N side, so a query's logits live in one lane column.  Register r of a logit
//     tile (keys 16 t + 4 g + r) is as it stands the B operand of second-product step (t, r), whose
//     slot g is that key: probabilities never move.
//   * Its A operand is a value row's features: lane c reads the 16 bytes at feature
//     64 blk + 4 perm(c), one read for four output tiles e; with perm(a) = 4 (a % 4) + a / 4 register
//     r of the four tiles is feature 64 blk + 16 r + 4 g + e, i.e. 16-byte stores whose four lane
//     rows are contiguous.
// Feature counts are padded to D = 64 or 128 (zeros); LDS rows are padded by four floats, which
// makes both 16-byte reads conflict-free.  VEC: rows are 16-byte aligned (8 for bf16 storage) and
// their length is a multiple of four; the other variant loads and stores single elements.
//
// Measured against the kernels they replaced (1024 threads, operands element by element from LDS,
// softmax by one thread per row): 4680 tokens, 12 heads of 128, regular (90,52), T = 2: stage R
// 94 -> 35 us and 133 -> 52 us (last), refine 276 -> 59 us, output 258 -> 58 us, the call 772 -> 195 us
// (the fp32 matrix unit alone needs 73 us with the tiles' padding); one head of 576 tokens and 64
// features 28.9 -> 15.3 us.  The error against 64 bits fell from 5.5e-7 to 3.0e-7.
#include "mrt_internal.hpp"
#include "mrt_bf16_tiles.hpp"

namespace mrt {

namespace {

__device__ inline f32x4 mfma4(f32x4 a, f32x4 b, f32x4 acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
  return acc;
}

// ---- rows of four features -------------------------------------------------------------------
template <typename T> struct Quad;
template <> struct Quad<float> {
  typedef f32x4 raw;
  static __device__ inline f32x4 widen(raw x) { return x; }
  static __device__ inline float one(float x) { return x; }
};
template <> struct Quad<u16> {
  typedef __attribute__((ext_vector_type(4))) u16 raw;
  static __device__ inline float one(u16 x) { return __uint_as_float((uint32_t)x << 16); }
  static __device__ inline f32x4 widen(raw x) { return f32x4{one(x[0]), one(x[1]), one(x[2]), one(x[3])}; }
};
// features v .. v + 3 of the row at p, zero from d on (the load itself is unconditional)
template <bool VEC, typename T>
__device__ inline f32x4 ld4(const T* p, int v, int d) {
  f32x4 x;
  if constexpr (VEC) {
    x = Quad<T>::widen(*(const typename Quad<T>::raw*)(p + (v < d ? v : 0)));
    if (v >= d) x = f32x4{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float one = Quad<T>::one(p[v + e < d ? v + e : 0]);
      x[e] = v + e < d ? one : 0.f;
    }
  }
  return x;
}
template <bool VEC>
__device__ inline void st4(float* p, f32x4 x, int v, int d) {
  if constexpr (VEC) {
    if (v < d) *(f32x4*)(p + v) = x;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (v + e < d) p[v + e] = x[e];
  }
}
template <bool VEC>
__device__ inline void st4(u16* p, f32x4 x, int v, int d) {
  if constexpr (VEC) {
    typedef typename Quad<u16>::raw raw;
    if (v < d) *(raw*)(p + v) = raw{f2bf(x[0]), f2bf(x[1]), f2bf(x[2]), f2bf(x[3])};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (v + e < d) p[v + e] = f2bf(x[e]);
  }
}

template <int D> constexpr int kLd = D + 4;   // LDS row stride in floats

// second product, one step group of four keys per lane row: o[blk][e] += Val[row + 4 g + r, :] p[r]
template <int D>
__device__ inline void pv4(const float* row0, f32x4 p, f32x4 (&o)[D / 64][4], int g, int c) {
  const float* at = row0 + (4 * g) * kLd<D> + 4 * (4 * (c & 3) + (c >> 2));
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int blk = 0; blk < D / 64; ++blk) {
      const f32x4 a = *(const f32x4*)(at + r * kLd<D> + 64 * blk);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[blk][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], p[r], o[blk][e], 0, 0, 0);
    }
}
template <int D>
__device__ inline void zero(f32x4 (&o)[D / 64][4]) {
#pragma unroll
  for (int blk = 0; blk < D / 64; ++blk)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[blk][e] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// the lane column's row of the second product, times mul
template <int D, bool VEC, typename T>
__device__ inline void store_out(T* row, const f32x4 (&o)[D / 64][4], float mul, int g, int d) {
#pragma unroll
  for (int blk = 0; blk < D / 64; ++blk)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      st4<VEC>(row, f32x4{o[blk][0][r], o[blk][1][r], o[blk][2][r], o[blk][3][r]} * mul, 64 * blk + 16 * r + 4 * g, d);
}

// ROWS rows of a token-indexed (or workspace) array between their global loads and the LDS tile;
// rows from `valid` on are zeros (their loads re-read the last valid row)
template <int D, int ROWS, int NTHR, bool VEC, typename T>
struct Rows32 {
  static constexpr int CPR = D / 4, TOTAL = ROWS * CPR, N = (TOTAL + NTHR - 1) / NTHR;
  f32x4 v[N];
  template <typename RowFn>
  __device__ inline void load(const T* src, RowFn rowoff, int valid, int d, int tid) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = tid + i * NTHR < TOTAL ? tid + i * NTHR : TOTAL - 1;
      const int r = idx / CPR;
      v[i] = ld4<VEC>(src + rowoff(r < valid ? r : valid - 1), 4 * (idx % CPR), d);
    }
  }
  __device__ inline void store(float* dst, int valid, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = tid + i * NTHR, r = idx / CPR;
      if (idx < TOTAL) *(f32x4*)(dst + r * kLd<D> + 4 * (idx % CPR)) = r < valid ? v[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
};

// ---------------------------------------------------------------------------------------
// stage R:  for one (m, n, k):
//   Z_R[j,i] = scale * sum_v A[j,v] K[n,k,i,v]        A = Q[m,k,j,:] at t=1 (L = identity),
//                                                      A = alpha_R/c_R from the workspace later
//   R = softmax_i Z_R;  c_L[j] = sum_i R log R;  alpha_L[j,:] = sum_i R[j,i] K[i,:];  Y likewise
// NT = ceil(b2 / 16) waves, one query tile each; K in LDS, then V in the same place (its loads are
// in flight from the start), so that a workgroup takes 34 KB at b2 = 52 and four share a CU.
// ---------------------------------------------------------------------------------------
template <int NT, int D, typename TIn, bool LAST, bool VEC>
__global__ __launch_bounds__(64 * NT, 3) void k_f32_stage_r(KParams p, int first) {
  constexpr int KS = D / 16, NTHR = 64 * NT, ROWS = 16 * NT;
  __shared__ __attribute__((aligned(16))) float tile[ROWS * kLd<D>];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int d = p.d, b1 = p.b1, b2 = p.b2;
  const int nk = blockIdx.x, ml = blockIdx.y, m = p.m0 + ml, bhl = blockIdx.z, bh = p.bh0 + bhl;
  const int n = nk / b1, k = nk - n * b1;
  const int a = m / p.c2, bq = m - a * p.c2;
  const int an = n / p.c2, bn = n - an * p.c2;
  if (an >= visible_key_tile_rows(a, p.c1k, p.ct, p.qt0)) return;
  const int b = bh / p.H, hd = bh - b * p.H;

  // block-grid rows a*b1 + k (queries) and an*b1 + k (keys); columns bq*b2 + j and bn*b2 + i
  const long long qrow = row_offset(p, a, k), krow = row_offset(p, an, k);
  const TIn* Qp = (const TIn*)p.Q + b * p.qs.batch + hd * p.qs.head + qrow * p.qs.token;
  const TIn* Kp = (const TIn*)p.K + b * p.ks.batch + hd * p.ks.head + krow * p.ks.token;
  const TIn* Vp = (const TIn*)p.V + b * p.vs.batch + hd * p.vs.head + krow * p.vs.token;
  const size_t NKtot = (size_t)p.ntk * b1;

  const int j = 16 * wave + c, jc = j < b2 ? j : b2 - 1;
  Rows32<D, ROWS, NTHR, VEC, TIn> rk, rv;
  rk.load(Kp, [&](int r) { return axis_offset(p.cmap, bn * b2 + r) * p.ks.token; }, b2, d, tid);
  f32x4 q[KS];
  if (first) {
    const TIn* row = Qp + axis_offset(p.cmap, bq * b2 + jc) * p.qs.token;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = ld4<VEC>(row, 16 * ks + 4 * g, d);
  } else {
    const float* row = (const float*)p.aR + ((((size_t)bhl * p.ntq + ml) * NKtot + nk) * b2 + jc) * d;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = ld4<VEC>(row, 16 * ks + 4 * g, d);
  }
  if (LAST) rv.load(Vp, [&](int r) { return axis_offset(p.cmap, bn * b2 + r) * p.vs.token; }, b2, d, tid);
  rk.store(tile, b2, tid);
  __syncthreads();

  f32x4 s[NT];
#pragma unroll
  for (int it = 0; it < NT; ++it) s[it] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    f32x4 ka[NT];
#pragma unroll
    for (int it = 0; it < NT; ++it) ka[it] = *(const f32x4*)(tile + (16 * it + c) * kLd<D> + 16 * ks + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int it = 0; it < NT; ++it)
        s[it] = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[it][e], q[ks][e], s[it], 0, 0, 0);
  }
  // softmax over i and sum_i R log R = (sum_i e z) / sum - log(sum)
  float mx = -INFINITY;
#pragma unroll
  for (int it = 0; it < NT; ++it)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[it][r] = 16 * it + 4 * g + r < b2 ? mul_rounded(p.scale, s[it][r]) : -INFINITY;
      mx = fmaxf(mx, s[it][r]);
    }
  mx = xmax(mx);
  float sum = 0.f, ent = 0.f;
#pragma unroll
  for (int it = 0; it < NT; ++it)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = 16 * it + 4 * g + r < b2;
      const float z = ok ? s[it][r] - mx : 0.f;
      const float e = ok ? expf(z) : 0.f;
      sum += e;
      ent = fmaf(e, z, ent);
      s[it][r] = e;
    }
  sum = xsum(sum);
  ent = xsum(ent);
  const float inv = 1.0f / sum;
  const size_t row = (((size_t)bhl * p.ntq + ml) * b2 + j) * NKtot + nk;
  if (g == 0 && j < b2) p.cL[row] = ent * inv - logf(sum);
#pragma unroll
  for (int it = 0; it < NT; ++it) s[it] = s[it] * inv;

  f32x4 o[D / 64][4];
  zero<D>(o);
#pragma unroll
  for (int it = 0; it < NT; ++it) pv4<D>(tile + 16 * it * kLd<D>, s[it], o, g, c);
  if (j < b2) store_out<D, VEC>((float*)p.aL + row * d, o, 1.0f, g, d);
  if constexpr (LAST) {
    __syncthreads();                  // every wave is done with K: the tile now holds V
    rv.store(tile, b2, tid);
    __syncthreads();
    zero<D>(o);
#pragma unroll
    for (int it = 0; it < NT; ++it) pv4<D>(tile + 16 * it * kLd<D>, s[it], o, g, c);
    if (j < b2) store_out<D, VEC>((float*)p.Y + row * d, o, 1.0f, g, d);
  }
}

// ---------------------------------------------------------------------------------------
// Online softmax of one query tile (16 rows, the wave's B operand q) over a key array, 16 keys at a
// time through two LDS slots: while the waves work on a chunk the next one's loads are in flight;
// they are committed to the other slot before the chunk's closing barrier.
// ---------------------------------------------------------------------------------------
constexpr int kChunk32 = 16;
template <int D, bool WITH_V> constexpr int kSlot32 = kChunk32 * kLd<D> * (WITH_V ? 2 : 1) + kChunk32;   // floats
constexpr float kGrow32 = 8.0f;   // the reference is raised when a logit exceeds it by more than this

struct Online32 {
  float m = -INFINITY, l = 0.f;   // reference (same in the four lanes of a query), this lane's sum
};

// NW waves; `wkeys`: the keys from here on are hidden from every query of this wave, which leaves out the
// chunks that start there (0: the wave owns no query).  `cut`, then every `step` keys: a chunk ends there
// too (0: nowhere).  bias(key) is subtracted from the scaled logits, hide(key) hides a key from the
// lane's query.
template <int D, int NW, bool WITH_V, bool VEC, typename TK, typename Bias, typename Hide>
__device__ inline void flash32(const TK* kbase, long long kstride, const TK* vbase, long long vstride, int nkeys, int d,
                               float scale, const f32x4 (&q)[D / 16], int wkeys, int cut, int step, float* lds, Bias bias,
                               Hide hide,
                               Online32& st, f32x4 (&o)[D / 64][4], int tid) {
  constexpr int KS = D / 16, NTHR = 64 * NW, LD = kLd<D>, SLOT = kSlot32<D, WITH_V>;
  const int lane = tid & 63, g = lane >> 4, c = lane & 15;
  Rows32<D, kChunk32, NTHR, VEC, TK> rk, rv;
  float rb = 0.f;
  int valid = 0;                  // rows of the fetched chunk
  auto fetch = [&](int c0) {
    if (step > 0 && c0 >= cut) cut += step;
    const int end = step > 0 && cut < nkeys ? cut : nkeys;
    valid = end - c0 < kChunk32 ? end - c0 : kChunk32;
    rk.load(kbase + c0 * kstride, [&](int r) { return r * kstride; }, valid, d, tid);
    if (WITH_V) rv.load(vbase + c0 * vstride, [&](int r) { return r * vstride; }, valid, d, tid);
    const int r = tid & 15;
    const float x = bias(c0 + (r < valid ? r : valid - 1));
    rb = r < valid ? -x : -INFINITY;
  };
  auto commit = [&](float* slot) {
    rk.store(slot, kChunk32, tid);
    // value rows past the end are zeros: a copy of the last one times a weight of zero is NaN where it holds an infinity
    if (WITH_V) rv.store(slot + kChunk32 * LD, valid, tid);
    if (tid < kChunk32) slot[kChunk32 * LD * (WITH_V ? 2 : 1) + tid] = rb;
  };
  fetch(0);
  commit(lds);
  __syncthreads();
  int cur = 0;
  for (int c0 = 0, next; c0 < nkeys; c0 = next, cur ^= 1) {
    const float* slot = lds + cur * SLOT;
    next = c0 + valid;
    fetch(next < nkeys ? next : c0);                               // past the end: the last chunk again
    if (c0 < wkeys) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
      for (int ks = 0; ks < KS; ks += 2) {
        s0 = mfma4(*(const f32x4*)(slot + c * LD + 16 * ks + 4 * g), q[ks], s0);
        s1 = mfma4(*(const f32x4*)(slot + c * LD + 16 * ks + 16 + 4 * g), q[ks + 1], s1);
      }
      const f32x4 bi = *(const f32x4*)(slot + kChunk32 * LD * (WITH_V ? 2 : 1) + 4 * g);
      f32x4 z;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[r] = fmaf(scale, s0[r] + s1[r], bi[r]);
        if (hide(c0 + 4 * g + r)) z[r] = -INFINITY;
      }
      const float zm = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
      if (__builtin_amdgcn_ballot_w64(zm > st.m + kGrow32) != 0) {     // also the first finite logit
        const float mnew = fmaxf(st.m, xmax(zm));
        const float f = mnew == -INFINITY ? 1.0f : expf(st.m - mnew);
        st.m = mnew;
        st.l *= f;
        if (WITH_V) {
#pragma unroll
          for (int blk = 0; blk < D / 64; ++blk)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[blk][e] = o[blk][e] * f;
        }
      }
      const float ref = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[r] = expf(z[r] - ref);
        st.l += z[r];
      }
      if (WITH_V) pv4<D>(slot + kChunk32 * LD, z, o, g, c);
    }
    commit(lds + (cur ^ 1) * SLOT);
    __syncthreads();
  }
}

// Query tile of wave `wave` of column j of query tile row a: row l = 16 wave + c (rows beyond b1
// repeat the last one and are not stored).
template <int D, bool VEC, typename TIn>
__device__ inline void load_q32(const TIn* Qp, const TokRows& qrow, int l, int b1, int d, int g, f32x4 (&q)[D / 16]) {
  const TIn* row = Qp + qrow(l < b1 ? l : b1 - 1);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) q[ks] = ld4<VEC>(row, 16 * ks + 4 * g, d);
}

// Addresses of a stage L workgroup: column j of query tile m of one (batch, head).
template <typename TIn>
struct Column32 {
  int j, ml, m, a, NK, b1, b2;
  size_t NKtot, row0, unit;
  long long qtok0;
  const TIn* Q;
  TIn* O;
  const float *aL, *Y, *cL;
  __device__ inline explicit Column32(const KParams& p) {
    j = blockIdx.x; ml = blockIdx.y; m = p.m0 + ml; b1 = p.b1; b2 = p.b2;
    const int bhl = (int)gridDim.z - 1 - (int)blockIdx.z, bh = p.bh0 + bhl;   // last head first, as the bf16 path
    a = m / p.c2;
    const int bq = m - a * p.c2, b = bh / p.H, hd = bh - b * p.H;
    NK = visible_key_tile_rows(a, p.c1k, p.ct, p.qt0) * p.c2 * b1;
    NKtot = (size_t)p.ntk * b1;
    unit = (size_t)bhl * p.ntq + ml;
    row0 = (unit * b2 + j) * NKtot;
    qtok0 = axis_offset(p.cmap, bq * b2 + j);
    Q = (const TIn*)p.Q + b * p.qs.batch + hd * p.qs.head + qtok0 * p.qs.token;
    O = (TIn*)p.O + b * p.os.batch + hd * p.os.head + qtok0 * p.os.token;
    aL = (const float*)p.aL + row0 * p.d;
    Y = (const float*)p.Y + row0 * p.d;
    cL = p.cL + row0;
  }
};

// ---------------------------------------------------------------------------------------
// stage L, last iteration:  Z_L[l,nk] = scale * sum_v alpha_L[nk,v] Q[m,l,j,v] - c_L[nk];
// L = softmax over visible nk;  O[l,:] = sum_nk L[l,nk] Y[nk,:].  NW >= ceil(b1 / 16) waves.
// ---------------------------------------------------------------------------------------
template <int NW, int D, typename TIn, bool VEC>
__global__ __launch_bounds__(64 * NW, NW > 8 ? 3 : (NW > 2 ? 4 : 2)) void k_f32_stage_l_out(KParams p) {
  __shared__ __attribute__((aligned(16))) float lds[2 * kSlot32<D, true>];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const Column32<TIn> col(p);
  const int l = 16 * wave + c, b1 = col.b1, d = p.d;
  f32x4 q[D / 16], o[D / 64][4];
  load_q32<D, VEC>(col.Q, tile_rows(p, col.a, p.qs.token), l, b1, d, g, q);
  zero<D>(o);
  Online32 st;
  const int lim = p.rl > 0 ? visible_key_rows(p, l < b1 ? l : b1 - 1) : 0x7fffffff;
  flash32<D, NW, true, VEC>(col.aL, d, col.Y, d, col.NK, d, p.scale, q, 16 * wave < b1 ? col.NK : 0, 0, 0, lds,
                            [&](int key) { return col.cL[key]; }, [&](int key) { return key >= lim; }, st, o, tid);
  const float lsum = xsum(st.l);
  const TokRows orow = tile_rows(p, col.a, p.os.token);
  if (l < b1) store_out<D, VEC>(col.O + orow(l), o, 1.0f / lsum, g, d);
}

// The Q tile of a column in LDS: NLT * 16 rows, those beyond b1 zero.
template <int D, bool VEC, typename TIn>
__device__ inline void stage_q32(float* Qs, const TIn* Qp, const TokRows& qrow, int rows, int b1, int d, int tid, int nthr) {
  constexpr int CPR = D / 4, BATCH = 8;
  const int total = rows * CPR;
  for (int i0 = tid; i0 < total; i0 += BATCH * nthr) {
    f32x4 v[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int idx = i0 + i * nthr, r = idx / CPR;
      v[i] = ld4<VEC>(Qp + qrow(r < b1 ? r : b1 - 1), 4 * (idx % CPR), d);
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int idx = i0 + i * nthr, r = idx / CPR;
      if (idx < total) *(f32x4*)(Qs + r * kLd<D> + 4 * (idx % CPR)) = r < b1 ? v[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
}

// A column sum of weights below this may have lost terms to underflow: alpha_R / c_R is then formed
// from the weights relative to the column's maximum (the same ratio).
constexpr float kTinySum = 0x1p-80f;

// alpha_R / c_R of the lane's key column and, for the backward pass, the statistics behind it.
template <int D, bool VEC, typename TIn>
__device__ inline void store_abar(const KParams& p, const Column32<TIn>& col, int nk, const f32x4 (&o)[D / 64][4],
                                  float csum, float shift, int g) {
  if (nk >= col.NK) return;
  const size_t at = (col.unit * col.NKtot + nk) * col.b2 + col.j;
  store_out<D, VEC>((float*)p.aR + at * p.d, o, 1.0f / csum, g, p.d);
  if (p.cmx_out != nullptr && g == 0) {
    p.cmx_out[at] = shift;
    p.cinv_out[at] = 1.0f / csum;
  }
}

// ---------------------------------------------------------------------------------------
// stage L, earlier iterations, at most 192 key rows: one wave per key tile (its rows of alpha_L in
// registers), the logits of every query tile formed once with the queries on the accumulator rows
// and kept; row statistics are exchanged between the waves, then
//   alpha_R[nk,:] / c_R[nk] = sum_l L[l,nk] Q[l,:] / sum_l L[l,nk].
// ---------------------------------------------------------------------------------------
template <int NLT, int D, typename TIn, bool VEC>
__global__ __launch_bounds__(768, 3) void k_f32_stage_l_refine_one(KParams p) {
  constexpr int KS = D / 16, LROWS = 16 * NLT, LD = kLd<D>;
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  const int tid = threadIdx.x, nthr = blockDim.x, nw = nthr >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, c = lane & 15;
  float* Qs = dyn;                       // [LROWS][LD]
  float* lse = Qs + LROWS * LD;          // [LROWS]
  float* red_m = lse + LROWS;            // [nw][LROWS]
  float* red_s = red_m + nw * LROWS;     // [nw][LROWS]
  const Column32<TIn> col(p);
  const int b1 = col.b1, d = p.d, NK = col.NK;
  const int nk = 16 * wave + c, nkc = nk < NK ? nk : NK - 1;
  f32x4 kb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kb[ks] = ld4<VEC>(col.aL + (size_t)nkc * d, 16 * ks + 4 * g, d);
  const float cl = col.cL[nkc];
  stage_q32<D, VEC>(Qs, col.Q, tile_rows(p, col.a, p.qs.token), LROWS, b1, d, tid, nthr);
  __syncthreads();

  f32x4 z[NLT];
  auto logits = [&]() {
#pragma unroll
    for (int lt = 0; lt < NLT; lt += 2) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
      const float* at = Qs + (16 * lt + c) * LD + 4 * g;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s0 = mfma4(*(const f32x4*)(at + 16 * ks), kb[ks], s0);
        s1 = mfma4(*(const f32x4*)(at + 16 * LD + 16 * ks), kb[ks], s1);
      }
      z[lt] = s0;
      z[lt + 1] = s1;
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * lt + 4 * g + r;
        const bool hidden = nk >= NK || (p.rl > 0 && nk >= visible_key_rows(p, l));
        z[lt][r] = hidden ? -INFINITY : fmaf(p.scale, z[lt][r], -cl);
      }
  };
  logits();
  // this wave's share of every row's statistics; the exponentials stay in place of the logits
#pragma unroll
  for (int lt = 0; lt < NLT; ++lt) {
    f32x4 mr, sr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      mr[r] = row16_max(z[lt][r]);
      z[lt][r] = expf(z[lt][r] - (mr[r] == -INFINITY ? 0.f : mr[r]));
      sr[r] = row16_sum(z[lt][r]);
    }
    if (c == 0) {
      *(f32x4*)(red_m + wave * LROWS + 16 * lt + 4 * g) = mr;
      *(f32x4*)(red_s + wave * LROWS + 16 * lt + 4 * g) = sr;
    }
  }
  __syncthreads();
  // per row: log-sum-exp and, in place of every wave's sum, what turns its exponentials into weights
  for (int l = tid; l < LROWS; l += nthr) {
    float M = -INFINITY, S = 0.f;
    for (int w = 0; w < nw; ++w) M = fmaxf(M, red_m[w * LROWS + l]);
    const float Ms = M == -INFINITY ? 0.f : M;
    for (int w = 0; w < nw; ++w) S = fmaf(red_s[w * LROWS + l], expf(red_m[w * LROWS + l] - Ms), S);
    lse[l] = Ms + logf(S);
    const float inv = l < b1 ? 1.0f / S : 0.f;
    for (int w = 0; w < nw; ++w) red_s[w * LROWS + l] = expf(red_m[w * LROWS + l] - Ms) * inv;
  }
  __syncthreads();
  float csum = 0.f, shift = 0.f;
#pragma unroll
  for (int lt = 0; lt < NLT; ++lt) {
    z[lt] = z[lt] * *(const f32x4*)(red_s + wave * LROWS + 16 * lt + 4 * g);
    csum += (z[lt][0] + z[lt][1]) + (z[lt][2] + z[lt][3]);
  }
  csum = xsum(csum);
  if (__builtin_expect(__any(nk < NK && !(csum > kTinySum)), 0)) {
    logits();
    float cm = -INFINITY;
#pragma unroll
    for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int l = 16 * lt + 4 * g + r;
        z[lt][r] = l < b1 ? z[lt][r] - lse[l] : -INFINITY;
        cm = fmaxf(cm, z[lt][r]);
      }
    cm = xmax(cm);
    shift = cm == -INFINITY ? 0.f : cm;
    csum = 0.f;
#pragma unroll
    for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[lt][r] = expf(z[lt][r] - shift);
        csum += z[lt][r];
      }
    csum = xsum(csum);
  }
  f32x4 o[D / 64][4];
  zero<D>(o);
#pragma unroll
  for (int lt = 0; lt < NLT; ++lt) pv4<D>(Qs + 16 * lt * LD, z[lt], o, g, c);
  store_abar<D, VEC>(p, col, nk, o, csum, shift, g);
}

// ---------------------------------------------------------------------------------------
// stage L, earlier iterations, longer key ranges: pass 1 finds the row log-sum-exps (flash32 without
// values), pass 2 deals the key tiles to the waves and forms each tile's logits again, one query
// tile at a time.  NW >= ceil(b1 / 16) waves.
// ---------------------------------------------------------------------------------------
template <int NW, int D, typename TIn, bool VEC>
__global__ __launch_bounds__(64 * NW, NW > 8 ? 3 : 4) void k_f32_stage_l_refine(KParams p) {
  constexpr int KS = D / 16, LD = kLd<D>;
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const Column32<TIn> col(p);
  const int b1 = col.b1, d = p.d, NK = col.NK, nlt = (b1 + 15) >> 4;
  float* ring = dyn;                              // two chunk slots
  float* lse = ring + 2 * kSlot32<D, false>;      // [16 nlt]
  float* Qs = lse + 16 * nlt;                     // [16 nlt][LD]
  const TokRows qrow = tile_rows(p, col.a, p.qs.token);
  const int l = 16 * wave + c;
  {
    f32x4 q[KS], o[D / 64][4];
    load_q32<D, VEC>(col.Q, qrow, l, b1, d, g, q);
    stage_q32<D, VEC>(Qs, col.Q, qrow, 16 * nlt, b1, d, tid, 64 * NW);
    Online32 st;
    const int lim = p.rl > 0 ? visible_key_rows(p, l < b1 ? l : b1 - 1) : 0x7fffffff;
    flash32<D, NW, false, VEC>(col.aL, d, col.aL, d, NK, d, p.scale, q, 16 * wave < b1 ? NK : 0, 0, 0, ring,
                               [&](int key) { return col.cL[key]; }, [&](int key) { return key >= lim; }, st, o, tid);
    const float lsum = xsum(st.l);
    if (wave < nlt && g == 0) lse[l] = st.m + logf(lsum);
  }
  __syncthreads();
  for (int t = wave; 16 * t < NK; t += NW) {
    const int nk = 16 * t + c, nkc = nk < NK ? nk : NK - 1;
    f32x4 kb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kb[ks] = ld4<VEC>(col.aL + (size_t)nkc * d, 16 * ks + 4 * g, d);
    const float cl = col.cL[nkc];
    // log L[l, nk] of query tile lt (rows beyond b1 and hidden keys: -inf)
    auto logits = [&](int lt) {
      const float* at = Qs + (16 * lt + c) * LD + 4 * g;
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
      for (int ks = 0; ks < KS; ks += 2) {
        s0 = mfma4(*(const f32x4*)(at + 16 * ks), kb[ks], s0);
        s1 = mfma4(*(const f32x4*)(at + 16 * ks + 16), kb[ks + 1], s1);
      }
      f32x4 z;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int lr = 16 * lt + 4 * g + r;
        const bool hidden = lr >= b1 || (p.rl > 0 && nk >= visible_key_rows(p, lr));
        z[r] = hidden ? -INFINITY : fmaf(p.scale, s0[r] + s1[r], -cl) - lse[lr];
      }
      return z;
    };
    f32x4 o[D / 64][4];
    float csum, shift = 0.f;
    auto run = [&]() {
      zero<D>(o);
      csum = 0.f;
      for (int lt = 0; lt < nlt; ++lt) {
        f32x4 w = logits(lt);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          w[r] = expf(w[r] - shift);
          csum += w[r];
        }
        pv4<D>(Qs + 16 * lt * LD, w, o, g, c);
      }
      csum = xsum(csum);
    };
    run();
    if (__builtin_expect(__any(nk < NK && !(csum > kTinySum)), 0)) {
      float cm = -INFINITY;
      for (int lt = 0; lt < nlt; ++lt) {
        const f32x4 z = logits(lt);
#pragma unroll
        for (int r = 0; r < 4; ++r) cm = fmaxf(cm, z[r]);
      }
      cm = xmax(cm);
      shift = cm == -INFINITY ? 0.f : cm;
      run();
    }
    store_abar<D, VEC>(p, col, nk, o, csum, shift, g);
  }
}

// ---------------------------------------------------------------------------------------
// dense baseline: softmax(scale Q K^T + mask) V, one query tile per wave
// ---------------------------------------------------------------------------------------
constexpr int kDenseWaves32 = 8, kDenseQ32 = 16 * kDenseWaves32;

// MASKED: chunk-causal (a kernel of its own: the shorter chunks' bookkeeping costs 4 % of a
// call at 64 features)
template <int D, typename TIn, bool VEC, bool MASKED>
__global__ __launch_bounds__(64 * kDenseWaves32, 4) void k_f32_dense(KParams p) {
  __shared__ __attribute__((aligned(16))) float lds[2 * kSlot32<D, true>];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int q0 = blockIdx.x * kDenseQ32, bh = blockIdx.y, d = p.d;
  const int b = bh / p.H, hd = bh - b * p.H;
  const TIn* Qp = (const TIn*)p.Q + b * p.qs.batch + hd * p.qs.head;
  const TIn* Kp = (const TIn*)p.K + b * p.ks.batch + hd * p.ks.head;
  const TIn* Vp = (const TIn*)p.V + b * p.vs.batch + hd * p.vs.head;
  const int qi = q0 + 16 * wave + c, qc = qi < p.Nq ? qi : p.Nq - 1;
  f32x4 q[D / 16], o[D / 64][4];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) q[ks] = ld4<VEC>(Qp + (long long)qc * p.qs.token, 16 * ks + 4 * g, d);
  zero<D>(o);
  // the keys query row r sees: a prefix, up to the end of its own chunk
  auto visible = [&](int r) {
    if (p.cc == 0) return p.Nkv;
    const long long most = (long long)((p.qoff + r / p.hw) / p.cc + 1) * p.cc * p.hw;
    return most < p.Nkv ? (int)most : p.Nkv;
  };
  auto last_of = [&](int r) { return r < p.Nq ? r : p.Nq - 1; };
  const int nkeys = visible(last_of(q0 + kDenseQ32 - 1)), lim = visible(qc);
  int wkeys = q0 + 16 * wave < p.Nq ? nkeys : 0;
  if (MASKED && wkeys > 0) wkeys = __builtin_amdgcn_readfirstlane(visible(last_of(q0 + 16 * wave + 15)));
  Online32 st;
  // chunks end where a query of this workgroup stops seeing keys: a wave whose queries stop there leaves the
  // next chunk out, and no value hidden from all of them gets to meet their weights of zero (0 x inf)
  flash32<D, kDenseWaves32, true, VEC>(Kp, p.ks.token, Vp, p.vs.token, nkeys, d, p.scale, q, wkeys, MASKED ? visible(q0) : 0,
                                       MASKED ? p.cc * p.hw : 0, lds, [](int) { return 0.f; },
                                       [&](int key) { return MASKED && key >= lim; }, st, o, tid);
  const float lsum = xsum(st.l);
  TIn* Op = (TIn*)p.O + b * p.os.batch + hd * p.os.head;
  if (qi < p.Nq) store_out<D, VEC>(Op + (long long)qi * p.os.token, o, lsum > 0.f ? 1.0f / lsum : 0.f, g, d);
}

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Rows of four features can be moved as one access: aligned bases, strides and row length.
template <typename TIn>
bool vec_ok(const KParams& kp) {
  const void* ptrs[4] = {kp.Q, kp.K, kp.V, kp.O};
  const mrt_strides* st[4] = {&kp.qs, &kp.ks, &kp.vs, &kp.os};
  if (kp.d % 4) return false;
  for (int i = 0; i < 4; ++i)
    if ((uintptr_t)ptrs[i] % (4 * sizeof(TIn)) || st[i]->token % 4 || st[i]->head % 4 || st[i]->batch % 4) return false;
  return true;
}

// Rows that cannot be moved so take the element-by-element variants of the same sizes.  (One variant, of the
// largest size, for all of them made small problems pay for it: blocks of 16 x 16 at 6 features 28 -> 91 us,
// 40 heads of them 67 -> 256; unaligned 24 x 24 at 64 features 56 -> 88.)
template <int NT, int D, typename TIn, bool VEC>
hipError_t run_r(const KParams& kp, dim3 grid, bool first, bool last, hipStream_t s) {
  if (last) k_f32_stage_r<NT, D, TIn, true, VEC><<<grid, 64 * NT, 0, s>>>(kp, first);
  else k_f32_stage_r<NT, D, TIn, false, VEC><<<grid, 64 * NT, 0, s>>>(kp, first);
  return hipGetLastError();
}
template <int D, typename TIn, bool VEC>
hipError_t run_r_d(const KParams& kp, dim3 grid, bool first, bool last, hipStream_t s) {
  switch ((kp.b2 + 15) / 16) {
    case 1: return run_r<1, D, TIn, VEC>(kp, grid, first, last, s);
    case 2: return run_r<2, D, TIn, VEC>(kp, grid, first, last, s);
    case 3: return run_r<3, D, TIn, VEC>(kp, grid, first, last, s);
    case 4: return run_r<4, D, TIn, VEC>(kp, grid, first, last, s);
    case 5: return run_r<5, D, TIn, VEC>(kp, grid, first, last, s);
    case 6: return run_r<6, D, TIn, VEC>(kp, grid, first, last, s);
  }
  return hipErrorInvalidValue;
}
template <typename TIn>
hipError_t run_r_t(const KParams& kp, dim3 grid, bool first, bool last, hipStream_t s) {
  if (kp.b2 > 96 || kp.d > 128) return hipErrorInvalidValue;
  if (vec_ok<TIn>(kp))
    return kp.d <= 64 ? run_r_d<64, TIn, true>(kp, grid, first, last, s) : run_r_d<128, TIn, true>(kp, grid, first, last, s);
  return kp.d <= 64 ? run_r_d<64, TIn, false>(kp, grid, first, last, s) : run_r_d<128, TIn, false>(kp, grid, first, last, s);
}

// Key ranges the one-pass refine kernel takes: twelve waves of one key tile each is the largest
// workgroup whose kept logits (48 registers at b1 = 192) leave three waves per SIMD.  It forms the
// logits once, the streamed kernel twice.
constexpr int kOnePassRows = 192;

template <int NW, int D, typename TIn, bool VEC>
hipError_t run_l(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  hipError_t e;
  if (last) {
    k_f32_stage_l_out<NW, D, TIn, VEC><<<grid, 64 * NW, 0, s>>>(kp);
    return hipGetLastError();
  }
  const int nk_max = kp.ntk * kp.b1;
  if (nk_max <= kOnePassRows) {
    // one wave per key tile; NW here is the (even) number of query tiles
    const int nw = (nk_max + 15) / 16;
    const size_t lds = ((size_t)16 * NW * (kLd<D> + 1) + 2 * (size_t)nw * 16 * NW) * 4;
    if ((e = allow_lds(k_f32_stage_l_refine_one<NW, D, TIn, VEC>, lds)) != hipSuccess) return e;
    k_f32_stage_l_refine_one<NW, D, TIn, VEC><<<grid, 64 * nw, lds, s>>>(kp);
    return hipGetLastError();
  }
  const int rows = 16 * ((kp.b1 + 15) / 16);
  const size_t lds = (2 * (size_t)kSlot32<D, false> + (size_t)rows * (kLd<D> + 1)) * 4;
  if ((e = allow_lds(k_f32_stage_l_refine<NW, D, TIn, VEC>, lds)) != hipSuccess) return e;
  k_f32_stage_l_refine<NW, D, TIn, VEC><<<grid, 64 * NW, lds, s>>>(kp);
  return hipGetLastError();
}
template <int D, typename TIn, bool VEC>
hipError_t run_l_d(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  switch ((kp.b1 + 31) / 32) {
    case 1: return run_l<2, D, TIn, VEC>(kp, grid, last, s);
    case 2: return run_l<4, D, TIn, VEC>(kp, grid, last, s);
    case 3: return run_l<6, D, TIn, VEC>(kp, grid, last, s);
    case 4: return run_l<8, D, TIn, VEC>(kp, grid, last, s);
    case 5: return run_l<10, D, TIn, VEC>(kp, grid, last, s);
    case 6: return run_l<12, D, TIn, VEC>(kp, grid, last, s);
  }
  return hipErrorInvalidValue;
}
template <typename TIn>
hipError_t run_l_t(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  if (kp.b1 > 192 || kp.d > 128) return hipErrorInvalidValue;
  if (vec_ok<TIn>(kp)) return kp.d <= 64 ? run_l_d<64, TIn, true>(kp, grid, last, s) : run_l_d<128, TIn, true>(kp, grid, last, s);
  return kp.d <= 64 ? run_l_d<64, TIn, false>(kp, grid, last, s) : run_l_d<128, TIn, false>(kp, grid, last, s);
}

template <int D, typename TIn, bool VEC>
hipError_t run_dense(const KParams& kp, dim3 grid, hipStream_t s) {
  if (kp.cc > 0) k_f32_dense<D, TIn, VEC, true><<<grid, 64 * kDenseWaves32, 0, s>>>(kp);
  else k_f32_dense<D, TIn, VEC, false><<<grid, 64 * kDenseWaves32, 0, s>>>(kp);
  return hipGetLastError();
}
template <typename TIn>
hipError_t run_dense_t(const KParams& kp, dim3 grid, hipStream_t s) {
  if (vec_ok<TIn>(kp)) return kp.d <= 64 ? run_dense<64, TIn, true>(kp, grid, s) : run_dense<128, TIn, true>(kp, grid, s);
  return kp.d <= 64 ? run_dense<64, TIn, false>(kp, grid, s) : run_dense<128, TIn, false>(kp, grid, s);
}

}  // namespace

hipError_t launch_f32_stage_r(const KParams& kp, int dtype, int nbh, bool first, bool last,
                              hipStream_t s) {
  dim3 grid(kp.ntk * kp.b1, kp.ntq, nbh);
  return dtype == MRT_F32 ? run_r_t<float>(kp, grid, first, last, s) : run_r_t<u16>(kp, grid, first, last, s);
}

hipError_t launch_f32_stage_l(const KParams& kp, int dtype, int nbh, bool last, hipStream_t s) {
  dim3 grid(kp.b2, kp.ntq, nbh);
  return dtype == MRT_F32 ? run_l_t<float>(kp, grid, last, s) : run_l_t<u16>(kp, grid, last, s);
}

hipError_t launch_f32_dense(const KParams& kp, int dtype, int nbh, hipStream_t s) {
  dim3 grid((kp.Nq + kDenseQ32 - 1) / kDenseQ32, nbh);
  return dtype == MRT_F32 ? run_dense_t<float>(kp, grid, s) : run_dense_t<u16>(kp, grid, s);
}

}  // namespace mrt
