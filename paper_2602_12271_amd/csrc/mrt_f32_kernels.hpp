// fp32 path: fp32 arithmetic and fp32 intermediates; every contraction runs on the matrix unit, as
// products of operands split into bf16 parts that add up to them or in fp32 (v_mfma_f32_16x16x4_f32).
//
// Used for f32 storage (the 1e-4 parity class) and, on request, as a device-side
// cross-check for bf16 storage.  Same three stages as the bf16 path:
//   stage R      one workgroup per (m, n, k): Z_R, R = softmax_i, c_L, alpha_L, (Y)
//   stage L out  one workgroup per (m, j): online softmax over nk, O = L Y
//   stage L ref  one workgroup per (m, j): alpha_R / c_R of the next iteration
// Equation references: App. A.1 / A.2 update equations.
//
// fp32 products go at 64 flop per clock and SIMD, a sixteenth of the bf16 rate, and block the vector ALU
// of the SIMD's other waves.  So operands are split into three bf16 parts as they reach LDS or registers
// and a product is six bf16 products (mrt_f32_split.hpp; layout as in the bf16 path).  What bounds the
// split kernels is the vector ALU: eleven instructions split two numbers, against which the products
// take a third of the time.  A compute unit must hold two or three workgroups, or their loads and
// barriers show: six waves (2, 2, 1, 1 on the SIMDs, every workgroup's alike) only double up at 128 registers a
// wave (measured with waves that only wait: 128 registers, 512 workgroups in one round, 136 in two).  The bounds cost
// local memory: the refine of six, eight and ten query tiles at 128 features keeps 150 to 290 bytes a lane there, most
// of them for its rare second logits, the output of six and eight tiles with more than 192 keys 260 and 180.
// 4680 tokens, 12 heads of 128, regular (90,52), T = 2: stage R 35 -> 31 us and 52 -> 42 us (last),
// refine 59 -> 42 us, output 58 -> 41 us, the call 195 -> 145 us (in graphs 141); dense baseline 1318 -> 975 us;
// the error against 64 bits 3.0e-7 -> 2.7e-7.
//
// fp32 operands remain where rows are moved element by element, for the smallest blocks (see run_r) and
// where a product was an infinity or a NaN or operands were very small or huge.  The layout feeds the
// matrix unit from registers and 16-byte LDS reads with nothing in between: lane (g = lane / 16,
// c = lane % 16) supplies A[c][k = g] and B[k = g][c] of a step and holds C[4g + r][c] in register r.
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
// d % 4 == 0; the other variant moves single elements.
#pragma once
#include "mrt_internal.hpp"
#include "mrt_f32_split.hpp"

namespace mrt {

namespace {

// A tile of a first product with fp32 operands: four sums side by side, each of every fourth step (one sum of all
// steps rounds as often as there are steps, up to 32: over 36 calls of small blocks, drawn, the error against 64 bits
// is 0.91 of what it was; small calls are 0.5 % longer, others not).
struct Sums4 {
  f32x4 s[4];
  __device__ inline Sums4() {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void add(f32x4 a, f32x4 b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], s[e], 0, 0, 0);
  }
  __device__ inline f32x4 total() const { return (s[0] + s[1]) + (s[2] + s[3]); }
};

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
// features v .. v + 3 of the row at p (the load itself is unconditional); from d on they are zeros, where
// rows are moved by four only once blank4 has seen them
template <bool VEC, typename T>
__device__ inline f32x4 ld4(const T* p, int v, int d) {
  f32x4 x;
  if constexpr (VEC) {
    x = Quad<T>::widen(*(const typename Quad<T>::raw*)(p + (v < d ? v : 0)));
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
__device__ inline f32x4 blank4(f32x4 x, int v, int d) {
  return VEC && v >= d ? f32x4{0.f, 0.f, 0.f, 0.f} : x;
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

// ROWS rows of a token-indexed (or workspace) array between their global loads and the LDS tile (fp32
// rows or split planes); rows from `valid` on are zeros (their loads re-read the last valid row)
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
  // PLANE: rows from one split plane to the next; SEE: what `watch` looks for in the rows split
  template <bool SPLIT, int SEE, int PLANE = ROWS>
  __device__ inline void store(float* dst, int valid, int d, int tid, Watch& watch) {
    const bool blank = valid < ROWS || d < D;        // (as they were loaded: the zeros are not looked at)
    if (blank) {
      if constexpr (SPLIT) watch.see_split<SEE>(v);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int idx = tid + i * NTHR;
        v[i] = blank4<true>(v[i], idx / CPR < valid ? 4 * (idx % CPR) : D, d);
      }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int idx = tid + i * NTHR, r = idx / CPR;
      const f32x4 x = v[i];
      if (idx < TOTAL) {
        if constexpr (SPLIT) store_split<D, PLANE>((u16*)dst, r, idx % CPR, x);
        else *(f32x4*)(dst + r * kLd<D> + 4 * (idx % CPR)) = x;
      }
    }
    if constexpr (SPLIT)
      if (!blank) watch.see_split<SEE>(v);
  }
};

// A wave's operand of the first product: sixteen rows, lane column c's at `row`.  SEE: what `watch` looks for
// in them.
template <int D, bool SPLIT>
struct Query32 {
  f32x4 v[D / 16];
  template <bool VEC, int SEE, typename T>
  __device__ inline void load(const T* row, int d, int g, Watch&) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) v[ks] = ld4<VEC>(row, 16 * ks + 4 * g, d);
    if (d < D) {
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) v[ks] = blank4<VEC>(v[ks], 16 * ks + 4 * g, d);
    }
  }
};
template <int D>
struct Query32<D, true> {
  Split8 v[D / 32];
  template <bool VEC, int SEE, typename T>
  __device__ inline void load(const T* row, int d, int g, Watch& watch) {
    f32x4 x[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) x[ks] = ld4<VEC>(row, 32 * (ks >> 1) + 8 * g + 4 * (ks & 1), d);
    if (d < D) {
      watch.see_split<SEE>(x);
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) x[ks] = blank4<VEC>(x[ks], 32 * (ks >> 1) + 8 * g + 4 * (ks & 1), d);
    }
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) v[ks] = split8(x[2 * ks], x[2 * ks + 1]);
    if (d == D) watch.see_split<SEE>(x);
  }
};

// The lane column's row of a second product.
template <int D, bool SPLIT>
struct Out32 {
  f32x4 v[D / 64][4];
  __device__ inline void clear() { zero<D>(v); }
  __device__ inline void scale(float f) {
#pragma unroll
    for (int blk = 0; blk < D / 64; ++blk)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[blk][e] = v[blk][e] * f;
  }
  __device__ inline void show(Watch&) const {}
  template <bool VEC, typename T>
  __device__ inline void store(T* row, float mul, int g, int d) const { store_out<D, VEC>(row, v, mul, g, d); }
};
template <int D>
struct Out32<D, true> {
  f32x4 v[D / 16];
  __device__ inline void clear() {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) v[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ inline void scale(float f) {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) v[t] = v[t] * f;
  }
  __device__ inline void show(Watch& w) const {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) w.see(v[t]);
  }
  template <bool VEC, typename T>
  __device__ inline void store(T* row, float mul, int g, int d) const {
#pragma unroll
    for (int t = 0; t < D / 16; ++t) st4<VEC>(row, v[t] * mul, 32 * (t >> 1) + 8 * g + 4 * (t & 1), d);
  }
};

// Sixteen weights a lane column and tile, as the operand of the second product with a whole tile of rows.
template <int NT, bool SPLIT>
struct Weights32 {
  f32x4 w[NT];
  __device__ inline explicit Weights32(const f32x4 (&s)[NT]) {
#pragma unroll
    for (int it = 0; it < NT; ++it) w[it] = s[it];
  }
  template <int D, int ROWS>
  __device__ inline void product(const float* tile, Out32<D, false>& o, int g, int c) const {
    o.clear();
#pragma unroll
    for (int it = 0; it < NT; ++it) pv4<D>(tile + 16 * it * kLd<D>, w[it], o.v, g, c);
  }
};
template <int NT>
struct Weights32<NT, true> {
  Split8 w[(NT + 1) / 2];
  __device__ inline explicit Weights32(const f32x4 (&s)[NT]) {
#pragma unroll
    for (int st = 0; st < (NT + 1) / 2; ++st)
      w[st] = split8(s[2 * st], 2 * st + 1 < NT ? s[2 * st + 1 < NT ? 2 * st + 1 : 0] : f32x4{0.f, 0.f, 0.f, 0.f});
  }
  template <int D, int ROWS>
  __device__ inline void product(const float* tile, Out32<D, true>& o, int g, int c) const {
    o.clear();
#pragma unroll
    for (int st = 0; st < (NT + 1) / 2; ++st) pv_split<D, ROWS>((const u16*)tile + 32 * st * kLdS<D>, w[st], o.v, 16 * g + c);
  }
};

// A workgroup's work with split operands and, if `Watch` met something unusual anywhere in it, once more with
// fp32 operands.  work(std::bool_constant, place, again) passes
// what it saw to again(watch) and returns the answer, the same in all threads: whether it will be called once
// more.  Results that may take the place of an input (O that of Q) are stored after the question; others may
// be stored before, as the second run writes them again.  `split` = false: with fp32 operands only.
struct Place {
  int x, y, z, tid;       // block and thread
};
template <bool SPLIT, typename Work>
__device__ inline void run_split(Work work, bool split = true) {
  Place at{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, (int)threadIdx.x};
  if constexpr (SPLIT) {
    __shared__ int found;
    if (threadIdx.x == 0) found = 0;       // seen by all after the first of the work's barriers
    auto again = [&](const Watch& watch) {
      if (__builtin_amdgcn_ballot_w64(watch.unusual()) != 0) found = 1;
      __syncthreads();
      return found != 0;
    };
    if (__builtin_expect(split, 1))
      if (__builtin_expect(!work(std::true_type{}, at, again), 1)) return;
    // an opaque copy: addresses are formed again instead of kept in registers through the first run
    asm("" : "+s"(at.x), "+s"(at.y), "+s"(at.z), "+v"(at.tid));
  }
  work(std::false_type{}, at, [](const Watch&) { return false; });
}

// ---------------------------------------------------------------------------------------
// stage R:  for one (m, n, k):
//   Z_R[j,i] = scale * sum_v A[j,v] K[n,k,i,v]        A = Q[m,k,j,:] at t=1 (L = identity),
//                                                      A = alpha_R/c_R from the workspace later
//   R = softmax_i Z_R;  c_L[j] = sum_i R log R;  alpha_L[j,:] = sum_i R[j,i] K[i,:];  Y likewise
// NT = ceil(b2 / 16) waves, one query tile each; K in LDS, then V in the same place, so that a workgroup
// takes 49 KB at b2 = 52 and three share a CU.  V's loads are in flight from the start or, where the
// registers are short, from the end of the logits.
// ---------------------------------------------------------------------------------------
template <int NT> constexpr int kRowsR = 32 * ((NT + 1) / 2);    // whole 32-row steps of the second product

// SPLIT: products of split operands, the tile as three bf16 planes.
template <int NT, int D, typename TIn, bool LAST, bool VEC, bool SPLIT, typename Again>
__device__ inline bool stage_r_32(const Place& at, const KParams& p, int first, float* tile, Again again) {
  constexpr int NTHR = 64 * NT, ROWS = SPLIT ? kRowsR<NT> : 16 * NT, STAGED = 16 * NT;
  constexpr bool EARLY_V = !SPLIT || NT * D <= 128;      // there are registers for the values beside the operand
  const int tid = at.tid, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int d = p.d, b1 = p.b1, b2 = p.b2;
  const int nk = at.x, ml = at.y, m = p.m0 + ml, bhl = at.z, bh = p.bh0 + bhl;
  const int n = nk / b1, k = nk - n * b1;
  const int a = m / p.c2, bq = m - a * p.c2;
  const int an = n / p.c2, bn = n - an * p.c2;
  const int b = bh / p.H, hd = bh - b * p.H;

  // block-grid rows a*b1 + k (queries) and an*b1 + k (keys); columns bq*b2 + j and bn*b2 + i
  const long long qrow = row_offset(p, a, k), krow = row_offset(p, an, k);
  const TIn* Qp = (const TIn*)p.Q + b * p.qs.batch + hd * p.qs.head + qrow * p.qs.token;
  const TIn* Kp = (const TIn*)p.K + b * p.ks.batch + hd * p.ks.head + krow * p.ks.token;
  const TIn* Vp = (const TIn*)p.V + b * p.vs.batch + hd * p.vs.head + krow * p.vs.token;
  const size_t NKtot = (size_t)p.ntk * b1;

  const int j = 16 * wave + c, jc = j < b2 ? j : b2 - 1;
  Watch watch(p.scale);
  Rows32<D, STAGED, NTHR, VEC, TIn> rk, rv;
  rk.load(Kp, [&](int r) { return axis_offset(p.cmap, bn * b2 + r) * p.ks.token; }, b2, d, tid);
  Query32<D, SPLIT> q;
  if (first) q.template load<VEC, kSeeNone>(Qp + axis_offset(p.cmap, bq * b2 + jc) * p.qs.token, d, g, watch);
  else q.template load<VEC, kSeeNone>((const float*)p.aR + ((((size_t)bhl * p.ntq + ml) * NKtot + nk) * b2 + jc) * d, d, g, watch);
  auto load_v = [&]() {
    if (LAST) rv.load(Vp, [&](int r) { return axis_offset(p.cmap, bn * b2 + r) * p.vs.token; }, b2, d, tid);
  };
  if (EARLY_V) load_v();
  rk.template store<SPLIT, kSeeSmall | kSeeHuge, ROWS>(tile, b2, d, tid, watch);
  if constexpr (ROWS > STAGED) {
    // the second half of the last step of the second products: zeros
    constexpr int PIECES = (ROWS - STAGED) * kLdS<D> / 8;
    for (int i = tid; i < 3 * PIECES; i += NTHR)
      *(uint4*)((u16*)tile + (i / PIECES * ROWS + STAGED) * kLdS<D> + 8 * (i % PIECES)) = uint4{0u, 0u, 0u, 0u};
  }
  __syncthreads();

  f32x4 s[NT];
  if constexpr (SPLIT) {
#pragma unroll
    for (int it = 0; it < NT; it += 2) {
      const u16* rows = (const u16*)tile + 16 * it * kLdS<D>;
      if (it + 1 < NT) logits_split<D, ROWS, 2>(rows, q.v, s + it, g, c);
      else logits_split<D, ROWS, 1>(rows, q.v, s + it, g, c);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int it = 0; it < NT; ++it) watch.see(s[it]);
    if (!EARLY_V) load_v();           // into the registers the operand had
  } else {
#pragma unroll
    for (int it = 0; it < NT; ++it) {
      Sums4 sums;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) sums.add(*(const f32x4*)(tile + (16 * it + c) * kLd<D> + 16 * ks + 4 * g), q.v[ks]);
      s[it] = sums.total();
      if (NT > 3) __builtin_amdgcn_sched_barrier(0);      // (the second run of a split kernel: few registers, not speed)
    }
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
      // weights of e^-200 are 0; a difference of two huge logits may be infinite, and 0 times it is no entropy
      const float z = ok ? fmaxf(s[it][r] - mx, -200.f) : 0.f;
      const float e = ok ? (SPLIT ? exp_near(z) : expf(z)) : 0.f;
      sum += e;
      ent = fmaf(e, z, ent);
      s[it][r] = e;
    }
  sum = xsum(sum);
  ent = xsum(ent);
  constexpr float W = SPLIT ? kWeight : 1.f;
  const float inv = 1.0f / sum;
  const size_t row = (((size_t)bhl * p.ntq + ml) * b2 + j) * NKtot + nk;
  if (g == 0 && j < b2) p.cL[row] = ent * inv - logf(sum * (1.f / W));
#pragma unroll
  for (int it = 0; it < NT; ++it) s[it] = s[it] * (inv * W);

  Weights32<NT, SPLIT> w(s);
  Out32<D, SPLIT> o;
  w.template product<D, ROWS>(tile, o, g, c);
  o.show(watch);
  if (j < b2) o.template store<VEC>((float*)p.aL + row * d, 1.f / W, g, d);
  if constexpr (LAST) {
    __syncthreads();                  // every wave is done with K: the tile now holds V
    rv.template store<SPLIT, kSeeSmall, ROWS>(tile, b2, d, tid, watch);
    __syncthreads();
    w.template product<D, ROWS>(tile, o, g, c);
    o.show(watch);
    if (j < b2) o.template store<VEC>((float*)p.Y + row * d, 1.f / W, g, d);
  }
  return again(watch);
}

template <int NT, int D, typename TIn, bool LAST, bool VEC, bool SPLIT>
__global__ __launch_bounds__(64 * NT, 3) void k_f32_stage_r(KParams p, int first) {
  constexpr int FLOATS = SPLIT ? kRowsR<NT> * kRowFloats<D> : 16 * NT * kLd<D>;
  static_assert(FLOATS >= 16 * NT * kLd<D>, "the tile holds fp32 rows too");
  __shared__ __attribute__((aligned(16))) float tile[FLOATS];
  {
    const int an = (int)blockIdx.x / p.b1 / p.c2, a = (p.m0 + (int)blockIdx.y) / p.c2;
    if (an >= visible_key_tile_rows(a, p.c1k, p.ct, p.qt0)) return;
  }
  run_split<SPLIT>([&](auto split, const Place& at, auto again) {
    return stage_r_32<NT, D, TIn, LAST, VEC, decltype(split)::value>(at, p, first, tile, again);
  });
}

// ---------------------------------------------------------------------------------------
// Online softmax of one query tile (16 rows, the wave's operand q) over a key array.  fp32 operands: 16
// keys at a time through two LDS slots; while the waves work on a chunk the next one's loads are in
// flight, and they are committed to the other slot before the chunk's closing barrier.  Split operands:
// 32 keys at a time (a whole step of the second product) through one slot of 49 KB at 128 features, so
// that two or three workgroups share a compute unit and cover each other's commits and barriers.
// ---------------------------------------------------------------------------------------
template <int D, bool SPLIT> constexpr int kChunk32 = SPLIT ? 32 : 16;
template <int D, bool WITH_V, bool SPLIT>
constexpr int kSlot32 = kChunk32<D, SPLIT> * (SPLIT ? kRowFloats<D> : kLd<D>) * (WITH_V ? 2 : 1) + kChunk32<D, SPLIT>;   // floats
// the loop's LDS: what the run with split operands takes, and the one with fp32 operands after it
constexpr int max_of(int a, int b) { return a > b ? a : b; }
template <int D, bool WITH_V, bool VEC>
constexpr int kRing32 = max_of(VEC ? kSlot32<D, WITH_V, true> : 0, 2 * kSlot32<D, WITH_V, false>);
constexpr float kGrow32 = 8.0f;   // the reference is raised when a logit exceeds it by more than this

struct Online32 {
  float m = -INFINITY, l = 0.f;   // reference (same in the four lanes of a query), this lane's sum (SPLIT: with the weights' factor)
};

// NW waves; `wkeys`: the keys from here on are hidden from every query of this wave, which leaves out the
// chunks that start there (0: the wave owns no query).  `cut`, then every `step` keys: a chunk ends there
// too (0: nowhere).  bias(key) is subtracted from the scaled logits, hide(key) hides a key from the
// lane's query.  `watch` sees the logits and the values that are split (SPLIT only; the caller has it see q).
template <int D, int NW, bool WITH_V, bool VEC, bool SPLIT, typename TK, typename Bias, typename Hide>
__device__ inline void flash32(const TK* kbase, long long kstride, const TK* vbase, long long vstride, int nkeys, int d,
                               float scale, const Query32<D, SPLIT>& q, int wkeys, int cut, int step, float* lds, Bias bias,
                               Hide hide,
                               Online32& st, Out32<D, SPLIT>& o, Watch& watch, int tid) {
  constexpr int CH = kChunk32<D, SPLIT>, NTHR = 64 * NW, NT = CH / 16;
  constexpr int KV = CH * (SPLIT ? kRowFloats<D> : kLd<D>), SLOT = kSlot32<D, WITH_V, SPLIT>, BIAS = KV * (WITH_V ? 2 : 1);
  const int lane = tid & 63, g = lane >> 4, c = lane & 15;
  Rows32<D, CH, NTHR, VEC, TK> rk, rv;
  float rb = 0.f;
  int valid = 0;                  // rows of the fetched chunk
  auto fetch_k = [&](int c0) {
    if (step > 0 && c0 >= cut) cut += step;
    const int end = step > 0 && cut < nkeys ? cut : nkeys;
    valid = end - c0 < CH ? end - c0 : CH;
    rk.load(kbase + c0 * kstride, [&](int r) { return r * kstride; }, valid, d, tid);
    const int r = tid & (CH - 1);
    const float x = bias(c0 + (r < valid ? r : valid - 1));
    rb = r < valid ? -x : -INFINITY;
  };
  auto fetch_v = [&](int c0) {
    if (WITH_V) rv.load(vbase + c0 * vstride, [&](int r) { return r * vstride; }, valid, d, tid);
  };
  auto commit_k = [&](float* slot) {
    rk.template store<SPLIT, kSeeNone>(slot, CH, d, tid, watch);
    if (tid < CH) slot[BIAS + tid] = rb;
  };
  // value rows past the end are zeros: a copy of the last one times a weight of zero is NaN where it holds an infinity
  auto commit_v = [&](float* slot, int rows) {
    if (WITH_V) rv.template store<SPLIT, kSeeSmall>(slot + KV, rows, d, tid, watch);
  };
  fetch_k(0);
  if constexpr (SPLIT) {
    commit_k(lds);
    fetch_v(0);
  } else {
    fetch_v(0);
    commit_k(lds);
    commit_v(lds, valid);
  }
  __syncthreads();
  int cur = 0;
  for (int c0 = 0, next; c0 < nkeys; c0 = next, cur ^= 1) {
    const float* slot = lds + (SPLIT ? 0 : cur * SLOT);
    const int rows = valid;
    next = c0 + rows;
    if constexpr (!SPLIT) {
      fetch_k(next < nkeys ? next : c0);                           // past the end: the last chunk again
      fetch_v(next < nkeys ? next : c0);
    }
    [[maybe_unused]] Split8 w;
    if (c0 < wkeys) {
      f32x4 z[NT];
      if constexpr (SPLIT) {
        logits_split<D, CH, NT>((const u16*)slot, q.v, z, g, c);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t) watch.see(z[t]);
      } else {
        Sums4 sums;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) sums.add(*(const f32x4*)(slot + c * kLd<D> + 16 * ks + 4 * g), q.v[ks]);
        z[0] = sums.total();
      }
      float zm = -INFINITY;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const f32x4 bi = *(const f32x4*)(slot + BIAS + 16 * t + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          z[t][r] = fmaf(scale, z[t][r], bi[r]);
          if (hide(c0 + 16 * t + 4 * g + r)) z[t][r] = -INFINITY;
          zm = fmaxf(zm, z[t][r]);
        }
      }
      if (__builtin_amdgcn_ballot_w64(zm > st.m + kGrow32) != 0) {     // also the first finite logit
        const float mnew = fmaxf(st.m, xmax(zm));
        const float f = mnew == -INFINITY ? 1.0f : expf(st.m - mnew);
        st.m = mnew;
        st.l *= f;
        if (WITH_V) o.scale(f);
      }
      const float ref = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          z[t][r] = SPLIT ? exp_near(z[t][r] - ref) : expf(z[t][r] - ref);
          st.l += z[t][r];
        }
      if constexpr (WITH_V) {
        if constexpr (SPLIT) w = split8(z[0], z[1]);
        else pv4<D>(slot + KV, z[0], o.v, g, c);
      }
    }
    if constexpr (!SPLIT) {
      commit_k(lds + (cur ^ 1) * SLOT);
      commit_v(lds + (cur ^ 1) * SLOT, valid);
      __syncthreads();
    } else {
      // the values are committed and the next keys requested beside the logits, the next keys committed
      // and their values requested beside the second product: one set of rows in registers at a time
      commit_v(lds, rows);
      if (next < nkeys) fetch_k(next);
      __syncthreads();
      if constexpr (WITH_V)
        if (c0 < wkeys) pv_split<D, CH>((const u16*)(slot + KV), w, o.v, lane);
      if (next >= nkeys) break;
      commit_k(lds);
      fetch_v(next);
      __syncthreads();
    }
  }
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
  __device__ inline explicit Column32(const Place& at, const KParams& p) {
    j = at.x; ml = at.y; m = p.m0 + ml; b1 = p.b1; b2 = p.b2;
    const int bhl = (int)gridDim.z - 1 - at.z, bh = p.bh0 + bhl;   // last head first, as the bf16 path
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
template <int NW, int D, typename TIn, bool VEC, bool SPLIT, typename Again>
__device__ inline bool stage_l_out_32(const Place& at, int l0, const KParams& p, float* lds, Again again) {
  const int tid = at.tid, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const Column32<TIn> col(at, p);
  const int l = l0 + 16 * wave + c, b1 = col.b1, d = p.d;
  Query32<D, SPLIT> q;
  Out32<D, SPLIT> o;
  Watch watch(p.scale);
  // rows beyond b1 repeat the last one and are not stored
  q.template load<VEC, kSeeSmall | kSeeHuge>(col.Q + tile_rows(p, col.a, p.qs.token)(l < b1 ? l : b1 - 1), d, g, watch);
  o.clear();
  Online32 st;
  const int lim = p.rl > 0 ? visible_key_rows(p, l < b1 ? l : b1 - 1) : 0x7fffffff;
  flash32<D, NW, true, VEC, SPLIT>(col.aL, d, col.Y, d, col.NK, d, p.scale, q, l0 + 16 * wave < b1 ? col.NK : 0, 0, 0, lds,
                            [&](int key) { return col.cL[key]; }, [&](int key) { return key >= lim; }, st, o, watch, tid);
  o.show(watch);
  const float lsum = xsum(st.l);
  if (again(watch)) return true;
  const TokRows orow = tile_rows(p, col.a, p.os.token);
  if (l < b1) o.template store<VEC>(col.O + orow(l), 1.0f / lsum, g, d);
  return false;
}
// fp32 operands; with split operands: longer key ranges than the kernel below takes
template <int NW, int D, typename TIn, bool VEC, bool SPLIT>
__global__ __launch_bounds__(64 * NW, NW > 8 ? 3 : (NW > 2 ? 4 : 2)) void k_f32_stage_l_out(KParams p) {
  __shared__ __attribute__((aligned(16))) float lds[kRing32<D, true, SPLIT>];
  run_split<SPLIT>([&](auto split, const Place& at, auto again) {
    return stage_l_out_32<NW, D, TIn, VEC, decltype(split)::value>(at, 0, p, lds, again);
  });
}

// ---------------------------------------------------------------------------------------
// The same with split operands and at most 16 NT key rows (one key tile row, or two narrow ones): the
// query operand's registers are free before the outputs' are needed.  The key range passes as chunks of
// 32 rows through two LDS slots, alpha_L first: every logit stays in registers, the softmax is formed
// once, then the rows of Y pass.  One chunk is in registers between global memory and LDS.
// ---------------------------------------------------------------------------------------
template <int NW, int NT, int D, typename TIn, typename Again>
__device__ inline bool stage_l_out_res_32(const Place& at, int l0, const KParams& p, float* lds, Again again) {
  constexpr int NTHR = 64 * NW, SLOT = 32 * kRowFloats<D>;
  const int tid = at.tid, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const Column32<TIn> col(at, p);
  const int l = l0 + 16 * wave + c, b1 = col.b1, d = p.d, NK = col.NK, nch = (NK + 31) >> 5;
  float* bias = lds + 2 * SLOT;          // [16 NT]
  Rows32<D, 32, NTHR, true, float> rows;
  Watch watch(p.scale);
  // chunk i of alpha_L, then of Y (i >= nch)
  auto fetch = [&](int i) {
    const int r0 = 32 * (i < nch ? i : i - nch);
    rows.load((i < nch ? col.aL : col.Y) + (size_t)r0 * d, [&](int r) { return r * d; }, NK - r0 < 32 ? NK - r0 : 32, d, tid);
  };
  auto commit = [&](int i) {
    const int left = NK - 32 * (i < nch ? i : i - nch);
    rows.template store<true, kSeeNone>(lds + (i & 1) * SLOT, left < 32 ? left : 32, d, tid, watch);      // rows past the end: zeros
    if (i >= nch) watch.see_split<kSeeSmall>(rows.v);
  };
  // chunk i is done: i + 1 goes to the other slot, i + 2 is requested
  auto advance = [&](int i) {
    if (i + 1 < 2 * nch) commit(i + 1);
    if (i + 2 < 2 * nch) fetch(i + 2);
    __syncthreads();
  };
  fetch(0);
  for (int i = tid; i < 16 * NT; i += NTHR) bias[i] = i < NK ? -col.cL[i] : -INFINITY;
  f32x4 z[NT];
  {
    Query32<D, true> q;
    q.template load<true, kSeeSmall | kSeeHuge>(col.Q + tile_rows(p, col.a, p.qs.token)(l < b1 ? l : b1 - 1), d, g, watch);
    commit(0);
    fetch(1);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT / 2; ++i) {
      if (i < nch) {
        logits_split<D, 32, 2>((const u16*)(lds + (i & 1) * SLOT), q.v, z + 2 * i, g, c);
        __builtin_amdgcn_sched_barrier(0);
        watch.see(z[2 * i]);
        watch.see(z[2 * i + 1]);
        advance(i);
      } else {
        z[2 * i] = z[2 * i + 1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  const int lim = p.rl > 0 ? visible_key_rows(p, l < b1 ? l : b1 - 1) : 0x7fffffff;
  float mx = -INFINITY, sum = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const f32x4 bi = *(const f32x4*)(bias + 16 * t + 4 * g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[t][r] = fmaf(p.scale, z[t][r], bi[r]);
      if (16 * t + 4 * g + r >= lim) z[t][r] = -INFINITY;
      mx = fmaxf(mx, z[t][r]);
    }
  }
  mx = xmax(mx);
  const float ref = mx == -INFINITY ? 0.f : mx;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      z[t][r] = exp_near(z[t][r] - ref);
      sum += z[t][r];
    }
  Out32<D, true> o;
  o.clear();
#pragma unroll
  for (int i = 0; i < NT / 2; ++i)
    if (i < nch) {
      pv_split<D, 32>((const u16*)(lds + ((nch + i) & 1) * SLOT), split8(z[2 * i], z[2 * i + 1]), o.v, lane);
      if (i + 1 < nch) advance(nch + i);
    }
  o.show(watch);
  const float lsum = xsum(sum);
  if (again(watch)) return true;
  if (l < b1) o.template store<true>(col.O + tile_rows(p, col.a, p.os.token)(l), 1.0f / lsum, g, d);
  return false;
}
// `parts` workgroups share a column's rows, 16 NW each
template <int NW, int NT, int D, typename TIn>
__global__ __launch_bounds__(64 * NW, NW > 4 ? 4 : 3) void k_f32_stage_l_out_res(KParams p, int parts) {
  __shared__ __attribute__((aligned(16))) float lds[max_of(2 * 32 * kRowFloats<D> + 16 * NT, 2 * kSlot32<D, true, false>)];
  run_split<true>([&](auto split, const Place& at, auto again) {
    const int j = at.x / parts, l0 = 16 * NW * (at.x - j * parts);
    const Place of{j, at.y, at.z, at.tid};
    if constexpr (decltype(split)::value) return stage_l_out_res_32<NW, NT, D, TIn>(of, l0, p, lds, again);
    else return stage_l_out_32<NW, D, TIn, true, false>(of, l0, p, lds, again);
  });
}

// The Q tile of a column in LDS: NLT * 16 rows (ROWS: the planes' stride where it is split), those
// beyond b1 zero.
template <int D, int ROWS, bool VEC, bool SPLIT, int SEE, typename TIn>
__device__ inline void stage_q32(float* Qs, const TIn* Qp, const TokRows& qrow, int rows, int b1, int d, int tid, int nthr,
                                 Watch& watch) {
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
      const f32x4 x = blank4<true>(v[i], r < b1 ? 4 * (idx % CPR) : D, d);
      if (idx < total) {
        if constexpr (SPLIT) store_split<D, ROWS>((u16*)Qs, r, idx % CPR, x);
        else *(f32x4*)(Qs + r * kLd<D> + 4 * (idx % CPR)) = x;
      }
    }
    if constexpr (SPLIT) watch.see_split<SEE>(v);
  }
}

// A column sum of weights below this may have lost terms to underflow: alpha_R / c_R is then formed
// from the weights relative to the column's maximum (the same ratio).
template <bool SPLIT> constexpr float kTinySum = 0x1p-80f * (SPLIT ? kWeight : 1.f);

// alpha_R / c_R of the lane's key column and, for the backward pass, the statistics behind it.  `o` and
// `csum` have the weights' factor.
template <int D, bool VEC, bool SPLIT, typename TIn>
__device__ inline void store_abar(const KParams& p, const Column32<TIn>& col, int nk, const Out32<D, SPLIT>& o,
                                  float csum, float shift, Watch& watch, int g) {
  if (nk >= col.NK) return;
  const size_t at = (col.unit * col.NKtot + nk) * col.b2 + col.j;
  o.template store<VEC>((float*)p.aR + at * p.d, 1.0f / csum, g, p.d);
  if (p.cmx_out != nullptr && g == 0) {
    p.cmx_out[at] = shift;
    p.cinv_out[at] = (SPLIT ? kWeight : 1.f) / csum;
  }
  o.show(watch);
}

// ---------------------------------------------------------------------------------------
// stage L, earlier iterations, at most 192 key rows: one wave per key tile (its rows of alpha_L in
// registers), the logits of every query tile formed once with the queries on the accumulator rows
// and kept; row statistics are exchanged between the waves, then
//   alpha_R[nk,:] / c_R[nk] = sum_l L[l,nk] Q[l,:] / sum_l L[l,nk].
// ---------------------------------------------------------------------------------------
template <int NLT, int D, typename TIn, bool VEC, bool SPLIT, typename Again>
__device__ inline bool stage_l_refine_one_32(const Place& at, const KParams& p, float* dyn, Again again) {
  constexpr int LROWS = 16 * NLT, LD = kLd<D>;
  const int tid = at.tid, nthr = blockDim.x, nw = nthr >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, g = lane >> 4, c = lane & 15;
  float* Qs = dyn;                       // [LROWS][LD] or planes
  float* lse = Qs + LROWS * (SPLIT ? kRowFloats<D> : LD);   // [LROWS]
  float* red_m = lse + LROWS;            // [nw][LROWS]
  float* red_s = red_m + nw * LROWS;     // [nw][LROWS]
  const Column32<TIn> col(at, p);
  const int b1 = col.b1, d = p.d, NK = col.NK;
  const int nk = 16 * wave + c, nkc = nk < NK ? nk : NK - 1;
  const float cl = col.cL[nkc];
  f32x4 z[NLT];
  Watch watch(p.scale);
  Query32<D, SPLIT> first;
  first.template load<VEC, kSeeNone>(col.aL + (size_t)nkc * d, d, g, watch);
  stage_q32<D, LROWS, VEC, SPLIT, kSeeSmall | kSeeHuge>(Qs, col.Q, tile_rows(p, col.a, p.qs.token), LROWS, b1, d, tid, nthr, watch);
  __syncthreads();

  auto logits = [&](const Query32<D, SPLIT>& kb) {
#pragma unroll
    for (int lt = 0; lt < NLT; lt += 2) {
      if constexpr (SPLIT) {
        logits_split<D, LROWS, 2>((const u16*)Qs + 16 * lt * kLdS<D>, kb.v, z + lt, g, c);
        watch.see(z[lt]);
        watch.see(z[lt + 1]);
      } else {
        const float* at = Qs + (16 * lt + c) * LD + 4 * g;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          Sums4 sums;
#pragma unroll
          for (int ks = 0; ks < D / 16; ++ks) sums.add(*(const f32x4*)(at + 16 * i * LD + 16 * ks), kb.v[ks]);
          z[lt + i] = sums.total();
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
      for (int r = 0; r < 4; ++r) z[lt][r] = nk < NK ? fmaf(p.scale, z[lt][r], -cl) : -INFINITY;
    if (p.rl > 0) {
#pragma unroll
      for (int lt = 0; lt < NLT; ++lt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (nk >= visible_key_rows(p, 16 * lt + 4 * g + r)) z[lt][r] = -INFINITY;
    }
  };
  logits(first);
  // this wave's share of every row's statistics; the exponentials stay in place of the logits
#pragma unroll
  for (int lt = 0; lt < NLT; ++lt) {
    f32x4 mr, sr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      mr[r] = row16_max(z[lt][r]);
      const float at = z[lt][r] - (mr[r] == -INFINITY ? 0.f : mr[r]);
      z[lt][r] = SPLIT ? exp_near(at) : expf(at);
      sr[r] = row16_sum(z[lt][r]);
    }
    if (c == 0) {
      *(f32x4*)(red_m + wave * LROWS + 16 * lt + 4 * g) = mr;
      *(f32x4*)(red_s + wave * LROWS + 16 * lt + 4 * g) = sr;
    }
  }
  __syncthreads();
  // per row: log-sum-exp and, in place of every wave's sum, what turns its exponentials into weights
  constexpr float W = SPLIT ? kWeight : 1.f;
  for (int l = tid; l < LROWS; l += nthr) {
    float M = -INFINITY, S = 0.f;
    for (int w = 0; w < nw; ++w) M = fmaxf(M, red_m[w * LROWS + l]);
    const float Ms = M == -INFINITY ? 0.f : M;
    for (int w = 0; w < nw; ++w) S = fmaf(red_s[w * LROWS + l], expf(red_m[w * LROWS + l] - Ms), S);
    lse[l] = Ms + logf(S * (1.f / W));
    const float inv = l < b1 ? W / S : 0.f;
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
  if (__builtin_expect(__any(nk < NK && !(csum > kTinySum<SPLIT>)), 0)) {
    Query32<D, SPLIT> kb;               // read again rather than kept (nor its addresses)
    int reread = nkc;
    asm("" : "+v"(reread));
    kb.template load<VEC, kSeeNone>(col.aL + (size_t)reread * d, d, g, watch);
    logits(kb);
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
        z[lt][r] = SPLIT ? exp_near(z[lt][r] - shift) : expf(z[lt][r] - shift);
        csum += z[lt][r];
      }
    csum = xsum(csum);
  }
  Out32<D, SPLIT> o;
  const Weights32<NLT, SPLIT> w(z);
  w.template product<D, LROWS>(Qs, o, g, c);
  store_abar<D, VEC>(p, col, nk, o, csum, shift, watch, g);
  return again(watch);
}
template <int NLT, int D, bool SPLIT>
constexpr size_t refine_one_32_lds(int nw) {
  return ((size_t)16 * NLT * ((SPLIT ? kRowFloats<D> : kLd<D>) + 1) + 2 * (size_t)nw * 16 * NLT) * 4;
}
// (Two query tiles, 64 features, fp32 operands: 82 registers without the bound of six waves a SIMD, and one
// workgroup of six key tiles less a unit: 48 x 48 in tiles of 24 x 24, 8 heads 75 -> 71 us.)
template <int NLT, int D, bool VEC, bool SPLIT>
constexpr int kRefineOneWaves = NLT > 6 ? 3 : (NLT == 2 && D == 64 && VEC && !SPLIT ? 6 : 4);
template <int NLT, int D, typename TIn, bool VEC, bool SPLIT>
__global__ __launch_bounds__(768, (kRefineOneWaves<NLT, D, VEC, SPLIT>)) void k_f32_stage_l_refine_one(KParams p) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  run_split<SPLIT>([&](auto split, const Place& at, auto again) {
    return stage_l_refine_one_32<NLT, D, TIn, VEC, decltype(split)::value>(at, p, dyn, again);
  });
}

// ---------------------------------------------------------------------------------------
// stage L, earlier iterations, longer key ranges: pass 1 finds the row log-sum-exps (flash32 without
// values), pass 2 deals the key tiles to the waves and forms each tile's logits again, one query
// tile at a time.  NW >= ceil(b1 / 16) waves.
// ---------------------------------------------------------------------------------------
template <int NW, int D, typename TIn, bool VEC, bool SPLIT, typename Again>
__device__ inline bool stage_l_refine_32(const Place& at, const KParams& p, float* lse, float* dyn, Again again) {
  constexpr int LD = kLd<D>, MAXROWS = 16 * NW;
  const int tid = at.tid, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const Column32<TIn> col(at, p);
  const int b1 = col.b1, d = p.d, NK = col.NK, nlt = (b1 + 15) >> 4;
  const TokRows qrow = tile_rows(p, col.a, p.qs.token);
  const int l = 16 * wave + c;
  // the chunks of the first pass and the Q tile of the second take the same LDS
  float* Qs = dyn;
  Watch watch(p.scale);
  {
    Query32<D, SPLIT> q;
    Out32<D, SPLIT> o;
    q.template load<VEC, kSeeSmall | kSeeHuge>(col.Q + qrow(l < b1 ? l : b1 - 1), d, g, watch);
    Online32 st;
    const int lim = p.rl > 0 ? visible_key_rows(p, l < b1 ? l : b1 - 1) : 0x7fffffff;
    flash32<D, NW, false, VEC, SPLIT>(col.aL, d, col.aL, d, NK, d, p.scale, q, 16 * wave < b1 ? NK : 0, 0, 0, dyn,
                               [&](int key) { return col.cL[key]; }, [&](int key) { return key >= lim; }, st, o, watch, tid);
    const float lsum = xsum(st.l);
    if (wave < nlt && g == 0) lse[l] = st.m + logf(lsum * (SPLIT ? 1.f / kWeight : 1.f));
  }
  __syncthreads();
  stage_q32<D, MAXROWS, VEC, SPLIT, kSeeNone>(Qs, col.Q, qrow, 32 * ((nlt + 1) / 2), b1, d, tid, 64 * NW, watch);
  __syncthreads();
  for (int t = wave; 16 * t < NK; t += NW) {
    const int nk = 16 * t + c, nkc = nk < NK ? nk : NK - 1;
    Query32<D, SPLIT> kb;
    kb.template load<VEC, kSeeNone>(col.aL + (size_t)nkc * d, d, g, watch);
    const float cl = col.cL[nkc];
    // log L[l, nk] of query tiles lt and lt + 1 (rows beyond b1 and hidden keys: -inf)
    auto logits = [&](int lt, f32x4 (&z)[2]) {
      if constexpr (SPLIT) {
        logits_split<D, MAXROWS, 2>((const u16*)Qs + 16 * lt * kLdS<D>, kb.v, z, g, c);
        watch.see(z[0]);
        watch.see(z[1]);
      } else {
        const float* at = Qs + (16 * lt + c) * LD + 4 * g;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          Sums4 sums;
#pragma unroll
          for (int ks = 0; ks < D / 16; ++ks) sums.add(*(const f32x4*)(at + 16 * i * LD + 16 * ks), kb.v[ks]);
          z[i] = sums.total();
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int lr = 16 * (lt + i) + 4 * g + r;
          const bool hidden = lr >= b1 || (p.rl > 0 && nk >= visible_key_rows(p, lr));
          z[i][r] = hidden ? -INFINITY : fmaf(p.scale, z[i][r], -cl) - lse[lr];
        }
    };
    Out32<D, SPLIT> o;
    float csum, shift = 0.f;
    auto run = [&]() {
      o.clear();
      csum = 0.f;
      for (int lt = 0; lt < nlt; lt += 2) {
        f32x4 w[2];
        logits(lt, w);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            w[i][r] = SPLIT ? exp_near(w[i][r] - shift) : expf(w[i][r] - shift);
            csum += w[i][r];
          }
        if constexpr (SPLIT) {
          pv_split<D, MAXROWS>((const u16*)Qs + 16 * lt * kLdS<D>, split8(w[0], w[1]), o.v, lane);
        } else {
          pv4<D>(Qs + 16 * lt * LD, w[0], o.v, g, c);
          pv4<D>(Qs + 16 * (lt + 1) * LD, w[1], o.v, g, c);
        }
      }
      csum = xsum(csum);
    };
    run();
    if (__builtin_expect(__any(nk < NK && !(csum > kTinySum<SPLIT>)), 0)) {
      float cm = -INFINITY;
      for (int lt = 0; lt < nlt; lt += 2) {
        f32x4 z[2];
        logits(lt, z);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) cm = fmaxf(cm, z[i][r]);
      }
      cm = xmax(cm);
      shift = cm == -INFINITY ? 0.f : cm;
      run();
    }
    store_abar<D, VEC>(p, col, nk, o, csum, shift, watch, g);
  }
  return again(watch);
}
template <int NW, int D, bool SPLIT>
constexpr int kRefineFloats32 = max_of(kRing32<D, false, SPLIT>, 16 * NW * max_of(kLd<D>, SPLIT ? kRowFloats<D> : 0));
template <int NW, int D, typename TIn, bool VEC, bool SPLIT>
__global__ __launch_bounds__(64 * NW, 3) void k_f32_stage_l_refine(KParams p) {
  extern __shared__ __attribute__((aligned(16))) float dyn[];
  run_split<SPLIT>([&](auto split, const Place& at, auto again) {
    return stage_l_refine_32<NW, D, TIn, VEC, decltype(split)::value>(at, p, dyn + kRefineFloats32<NW, D, SPLIT>, dyn, again);
  });
}

// ---------------------------------------------------------------------------------------
// dense baseline: softmax(scale Q K^T + mask) V, one query tile per wave
// ---------------------------------------------------------------------------------------
constexpr int kDenseWaves32 = 8, kDenseQ32 = 16 * kDenseWaves32;

// MASKED: chunk-causal (a kernel of its own: the shorter chunks' bookkeeping costs 4 % of a
// call at 64 features)
template <int D, typename TIn, bool VEC, bool MASKED, bool SPLIT, typename Again>
__device__ inline bool dense_32(const Place& at, const KParams& p, float* lds, Again again) {
  const int tid = at.tid, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int q0 = at.x * kDenseQ32, bh = at.y, d = p.d;
  const int b = bh / p.H, hd = bh - b * p.H;
  const TIn* Qp = (const TIn*)p.Q + b * p.qs.batch + hd * p.qs.head;
  const TIn* Kp = (const TIn*)p.K + b * p.ks.batch + hd * p.ks.head;
  const TIn* Vp = (const TIn*)p.V + b * p.vs.batch + hd * p.vs.head;
  const int qi = q0 + 16 * wave + c, qc = qi < p.Nq ? qi : p.Nq - 1;
  Query32<D, SPLIT> q;
  Out32<D, SPLIT> o;
  Watch watch(p.scale);
  q.template load<VEC, kSeeSmall | kSeeHuge>(Qp + (long long)qc * p.qs.token, d, g, watch);
  o.clear();
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
  flash32<D, kDenseWaves32, true, VEC, SPLIT>(Kp, p.ks.token, Vp, p.vs.token, nkeys, d, p.scale, q, wkeys, MASKED ? visible(q0) : 0,
                                       MASKED ? p.cc * p.hw : 0, lds, [](int) { return 0.f; },
                                       [&](int key) { return MASKED && key >= lim; }, st, o, watch, tid);
  o.show(watch);
  const float lsum = xsum(st.l);
  if (again(watch)) return true;
  TIn* Op = (TIn*)p.O + b * p.os.batch + hd * p.os.head;
  if (qi < p.Nq) o.template store<VEC>(Op + (long long)qi * p.os.token, lsum > 0.f ? 1.0f / lsum : 0.f, g, d);
  return false;
}
// A few keys do not pay for splitting the queries: up to these the operands stay fp32 (us with split and with
// fp32 operands, 12 heads; 64 features: 16 keys 4.4, 3.8, 32 keys 4.4, 4.8; 128 features: 16 keys 7.3, 4.8, 64 keys
// 11.5, 10.4, 80 keys 17.0, 17.3, 96 keys 17.6, 20.2; masked, where chunks of 32 keys are cut short, two chunks
// of 40 keys 21.3, 17.3, of 80 keys 30.7, about 27, of 96 keys 30.0, 30.6).
template <int D, bool MASKED>
constexpr int kFewKeys32 = D == 64 ? 16 : (MASKED ? 160 : 64);
template <int D, typename TIn, bool VEC, bool MASKED>
__global__ __launch_bounds__(64 * kDenseWaves32, 4) void k_f32_dense(KParams p) {
  __shared__ __attribute__((aligned(16))) float lds[kRing32<D, true, VEC>];
  run_split<VEC>([&](auto split, const Place& at, auto again) {
    return dense_32<D, TIn, VEC, MASKED, decltype(split)::value>(at, p, lds, again);
  }, p.Nkv > kFewKeys32<D, MASKED>);
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
//
// Where fp32 operands stay: blocks of one tile, whose second products would fill half a step of split
// operands and whose few products do not pay for the splitting (blocks of 16 x 16 at 64 features, one to
// 32 heads: the call with split operands 13 % longer; at one head the last launch 5.4 against 7.3 us), and
// two tiles, or the last launch of three, where the key side is at most 48 rows: a few heads of them are one
// chain of latencies (24 x 24 at 64 features, calls of 1 to 8 heads: all launches split 1.04 of the time, of
// 12 to 40 heads 0.96 .. 0.98; 40 x 33 at 128 features, last launch split 1.02, 0.98; 90 rows of 26 columns,
// 12 heads 0.98, 64 of 20, 24 heads 0.93).  The choice is the block's and the features', not the heads', the
// sequences' or the passes': a head's bits do not depend on what shares its call.
constexpr int kShortRows = 48;
template <int NT, int D, typename TIn, bool VEC>
hipError_t run_r(const KParams& kp, dim3 grid, bool first, bool last, hipStream_t s) {
  const bool small = kp.ntk * kp.b1 <= kShortRows;
  if (last) {
    constexpr bool ALWAYS = VEC && NT > 3;
    const bool split = VEC && NT > 1 && (ALWAYS || !small);
    if constexpr (VEC && NT > 1)
      if (split) k_f32_stage_r<NT, D, TIn, true, VEC, true><<<grid, 64 * NT, 0, s>>>(kp, first);
    if constexpr (!ALWAYS)
      if (!split) k_f32_stage_r<NT, D, TIn, true, VEC, false><<<grid, 64 * NT, 0, s>>>(kp, first);
  } else {
    constexpr bool ALWAYS = VEC && NT > 2;
    const bool split = VEC && NT > 1 && (ALWAYS || !small);
    if constexpr (VEC && NT > 1)
      if (split) k_f32_stage_r<NT, D, TIn, false, VEC, true><<<grid, 64 * NT, 0, s>>>(kp, first);
    if constexpr (!ALWAYS)
      if (!split) k_f32_stage_r<NT, D, TIn, false, VEC, false><<<grid, 64 * NT, 0, s>>>(kp, first);
  }
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
// logits once, the streamed kernel twice.  Twelve query tiles of split operands at 128 features are
// 144 KB, and with the row statistics of eleven waves more than a compute unit has: those blocks (161 rows and
// more) take the streamed kernel too, and are ahead of the one-pass kernel with fp32 operands by as much as
// others (calls of 176 x 30, 1 to 24 heads 115 .. 432 us -> 87 .. 360).
constexpr int kOnePassRows = 192;
constexpr size_t kMaxLds = 160 * 1024;
template <int NLT, int D, bool SPLIT> constexpr bool kOnePass = !(NLT == 12 && D == 128 && SPLIT);
static_assert(refine_one_32_lds<12, 128, true>(11) > kMaxLds && refine_one_32_lds<10, 128, true>(12) + 16 <= kMaxLds &&
              refine_one_32_lds<12, 128, false>(12) + 16 <= kMaxLds && refine_one_32_lds<12, 64, true>(12) + 16 <= kMaxLds, "");

template <int NW, int NT, int D, typename TIn>
hipError_t run_out_res(const KParams& kp, dim3 grid, int parts, hipStream_t s) {
  k_f32_stage_l_out_res<NW, NT, D, TIn><<<dim3(parts * grid.x, grid.y, grid.z), 64 * NW, 0, s>>>(kp, parts);
  return hipGetLastError();
}
template <int NW, int D, typename TIn, bool VEC, bool SPLIT>
hipError_t run_l_as(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  const int nk_max = kp.ntk * kp.b1;
  if (last) {
    if constexpr (SPLIT) {
      if (nk_max <= 96) {
        if constexpr (NW > 2 && NW <= 6) return run_out_res<NW, 6, D, TIn>(kp, grid, 1, s);      // (run_l: not two)
      } else if (nk_max <= 192) {
        // at most four waves a workgroup: three of them share a compute unit, where one of six to twelve
        // waves would have it alone (the logits of 192 keys leave 168 registers a wave)
        const int tiles = (kp.b1 + 15) / 16, parts = (tiles + 3) / 4;
        switch ((tiles + parts - 1) / parts) {
          case 4: return run_out_res<4, 12, D, TIn>(kp, grid, parts, s);
          case 3: return run_out_res<3, 12, D, TIn>(kp, grid, parts, s);
          default: return run_out_res<2, 12, D, TIn>(kp, grid, parts, s);
        }
      }
    }
    k_f32_stage_l_out<NW, D, TIn, VEC, SPLIT><<<grid, 64 * NW, 0, s>>>(kp);
    return hipGetLastError();
  }
  hipError_t e;
  if constexpr (kOnePass<NW, D, SPLIT>)
    if (nk_max <= kOnePassRows) {
      // one wave per key tile; NW here is the (even) number of query tiles
      const int nw = (nk_max + 15) / 16;
      const size_t lds1 = refine_one_32_lds<NW, D, SPLIT>(nw);
      if ((e = allow_lds(k_f32_stage_l_refine_one<NW, D, TIn, VEC, SPLIT>, lds1)) != hipSuccess) return e;
      k_f32_stage_l_refine_one<NW, D, TIn, VEC, SPLIT><<<grid, 64 * nw, lds1, s>>>(kp);
      return hipGetLastError();
    }
  const size_t lds = ((size_t)kRefineFloats32<NW, D, SPLIT> + 16 * NW) * 4;
  if ((e = allow_lds(k_f32_stage_l_refine<NW, D, TIn, VEC, SPLIT>, lds)) != hipSuccess) return e;
  k_f32_stage_l_refine<NW, D, TIn, VEC, SPLIT><<<grid, 64 * NW, lds, s>>>(kp);
  return hipGetLastError();
}
template <int NW, int D, typename TIn, bool VEC>
hipError_t run_l(const KParams& kp, dim3 grid, bool last, hipStream_t s) {
  if constexpr (VEC && NW == 2) {
    // up to 32 query rows two waves would split what twelve times as many products do not pay for: fp32
    // operands up to the key rows of the one-pass kernels (4 rows, 96 columns, 40 heads: output launch 12 us
    // against 23, refine 14 against 16; calls with fp32 and with split operands here: 30 rows, 52 columns, 128
    // features, one head 0.99 against 1.03 of fp32 operands everywhere, 40 heads 0.87 against 0.94; 144 key rows of
    // 24 x 24 tiles, one head 0.98 against 1.04, 24 heads 0.97 against 0.99; 192 key rows 0.99 .. 1.04 against
    // 0.98 .. 1.00)
    if (kp.ntk * kp.b1 >= kOnePassRows) return run_l_as<NW, D, TIn, true, true>(kp, grid, last, s);
    return run_l_as<NW, D, TIn, true, false>(kp, grid, last, s);
  } else {
    return run_l_as<NW, D, TIn, VEC, VEC>(kp, grid, last, s);
  }
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
}  // namespace mrt
