// The middle of a ring product whose first and last four transform stages run in the lift
// and the reconstruction (lift_cols.hip, crt_cols.hip): the other stages of the forward
// transforms over contiguous rows of N / 16 points, the pointwise products, and the
// matching stages of the inverse transforms, in one pass over the residues.  Rows of up to
// 256 points take rows_fused_kernel (kernels.hip); this file has rows of 512 to 4096.
#include <algorithm>

#include "device_common.h"

namespace fhe {

// A row of n = 2^S points is held by T = n / 16 threads with 16 values each, in three
// register phases of four, four and S - 8 stages: elements {u T + t}, then 16 sub-columns
// per block of T elements, then {16 t + u}.  The exchange between the first two phases
// crosses waves where T > 64; the other one stays inside a wave's 1024 elements.
template <int S>
struct MidRow {
  static constexpr int n = 1 << S, T = n / 16, C = T / 16;
  static constexpr int THREADS = T > 128 ? T : 128, RPW = THREADS / T;  // rows per workgroup
  static constexpr int C2 = 4096 / n;  // phase 2: twiddles per thread of its first stage
  static constexpr int LDS_ROW = n + n / 16;

  static constexpr __device__ __forceinline__ int pad(int e) { return e + (e >> 4); }
  // element of register r of thread t in phase I; positions of the thread's part and the
  // register's part add (their bits are disjoint)
  template <int I>
  static constexpr __device__ __forceinline__ int elem(int r, int t) {
    return I == 0 ? r * T + t : (I == 1 ? (t / C) * T + r * C + t % C : 16 * t + r);
  }
};

// A phase's twiddles of one thread: the stage of c groups per thread has its c entries at
// [c, 2 c).
struct Tw16 {
  uint32_t w[16];
};

// Phase I's twiddles: the stage with c groups per thread starts at table index
// mult c G + (thread's block) c, G the groups of the phase's first stage over the row.
template <int S, int I>
__device__ __forceinline__ void load_phase_tw(Tw16& w, TwTab tw, int mult, int t) {
  typedef MidRow<S> M;
  constexpr int G = I == 0 ? 1 : (I == 1 ? 16 : M::T);
  const int b = mult * G + (I == 0 ? 0 : (I == 1 ? t / M::C : t));
  if (I < 2 || M::C2 <= 1) tw.run<1>(b, w.w + 1);
  if (I < 2 || M::C2 <= 2) tw.run<2>(2 * b, w.w + 2);
  if (I < 2 || M::C2 <= 4) tw.run<4>(4 * b, w.w + 4);
  tw.run<8>(8 * b, w.w + 8);
}

template <int S, int I, int NP>
__device__ __forceinline__ void fwd_phase(uint32_t (&x)[NP][16], const Tw16& w, const Mod& M) {
#pragma unroll
  for (int c = I == 2 ? MidRow<S>::C2 : 1; c <= 8; c *= 2) {
    const int h = 8 / c;
#pragma unroll
    for (int g = 0; g < c; ++g)
#pragma unroll
      for (int r = 0; r < NP; ++r)
#pragma unroll
        for (int u = 2 * h * g; u < 2 * h * g + h; ++u) ct_bfly(x[r][u], x[r][u + h], w.w[c + g], M);
  }
}

template <int S, int I, int NP>
__device__ __forceinline__ void inv_phase(uint32_t (&x)[NP][16], const Tw16& w, const Mod& M) {
#pragma unroll
  for (int c = 8; c >= (I == 2 ? MidRow<S>::C2 : 1); c /= 2) {
    const int h = 8 / c;
#pragma unroll
    for (int g = 0; g < c; ++g)
#pragma unroll
      for (int r = 0; r < NP; ++r)
#pragma unroll
        for (int u = 2 * h * g; u < 2 * h * g + h; ++u) gs_bfly(x[r][u], x[r][u + h], w.w[c + g], M);
  }
}

// Registers of phase I to those of phase J, NB rows at a time through NB buffers.
template <int S, int I, int J, int NP, int NB>
__device__ __forceinline__ void mid_exchange(uint32_t (&x)[NP][16], uint32_t* const (&l)[NB], int t) {
  typedef MidRow<S> M;
  constexpr bool across = (I == 0 || J == 0) && M::T > 64;
#pragma unroll
  for (int r0 = 0; r0 < NP; r0 += NB) {
    // the buffers have been read: by every wave, or (before the first round, whose writes
    // stay in the region that this wave read last) by this one
    if (across && r0 > 0) __syncthreads();
    else slot_sync();
#pragma unroll
    for (int r = r0; r < NP && r < r0 + NB; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        l[r - r0][M::pad(M::template elem<I>(0, t)) + M::pad(M::template elem<I>(u, 0))] = x[r][u];
    if (across) __syncthreads();
    else slot_sync();
#pragma unroll
    for (int r = r0; r < NP && r < r0 + NB; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        x[r][u] = l[r - r0][M::pad(M::template elem<J>(0, t)) + M::pad(M::template elem<J>(u, 0))];
  }
}

// All row stages of NP forward transforms: values in [-2q, 2q) at elements u T + t, left in
// [0, 2q) at 16 t + u.  A phase's twiddles are issued before the exchange that precedes it.
template <int S, int NP, int NB>
__device__ __forceinline__ void mid_forward(uint32_t (&x)[NP][16], uint32_t* const (&l)[NB], int t, TwTab tw, int mult,
                                            const Mod& M) {
  Tw16 w0, w1, w2;
  load_phase_tw<S, 0>(w0, tw, mult, t);
  load_phase_tw<S, 1>(w1, tw, mult, t);
  __builtin_amdgcn_sched_barrier(0);
  fwd_phase<S, 0, NP>(x, w0, M);
  mid_exchange<S, 0, 1, NP, NB>(x, l, t);
  load_phase_tw<S, 2>(w2, tw, mult, t);
  __builtin_amdgcn_sched_barrier(0);
  fwd_phase<S, 1, NP>(x, w1, M);
  mid_exchange<S, 1, 2, NP, NB>(x, l, t);
  fwd_phase<S, 2, NP>(x, w2, M);
#pragma unroll
  for (int r = 0; r < NP; ++r)
#pragma unroll
    for (int u = 0; u < 16; ++u) x[r][u] = fwd_lift(x[r][u], M);
}

// The row stages of NP inverse transforms, values in [0, 2q) from 16 t + u to u T + t; w2
// holds phase 2's twiddles (loaded before the products).
template <int S, int NP, int NB>
__device__ __forceinline__ void mid_inverse(uint32_t (&x)[NP][16], uint32_t* const (&l)[NB], int t, TwTab itw, int mult,
                                            const Mod& M, const Tw16& w2) {
  Tw16 w0, w1;
  inv_phase<S, 2, NP>(x, w2, M);
  __builtin_amdgcn_sched_barrier(0);
  load_phase_tw<S, 1>(w1, itw, mult, t);
  __builtin_amdgcn_sched_barrier(0);
  mid_exchange<S, 2, 1, NP, NB>(x, l, t);
  load_phase_tw<S, 0>(w0, itw, mult, t);
  inv_phase<S, 1, NP>(x, w1, M);
  mid_exchange<S, 1, 0, NP, NB>(x, l, t);
  inv_phase<S, 0, NP>(x, w0, M);
}

template <int S, int MODE>
__device__ __forceinline__ void rows_mid_kernel_body(const RowsArgs& a, const Blk bk) {
  typedef MidRow<S> M;
  constexpr int n = M::n, T = M::T, RPW = M::RPW, NB = MODE == ROWS_RELIN ? 1 : 2;
  __shared__ uint32_t lds[NB][RPW * M::LDS_ROW];
  const int s = threadIdx.x / T, t = threadIdx.x % T;
  const int N = 1 << a.logN;
  constexpr int ROWS = 16;  // rows of a transform
  // Workgroup w runs on XCD w % 8.  The rows, ordered by prime, are cut into eight runs of
  // equal length, one per XCD: a prime's table and key rows are read into one L2, and the
  // XCDs finish together whatever K is.
  const int per_prime = a.cnum * (ROWS / RPW), total = a.K * per_prime, chunk = (total + 7) / 8;
  const int li = bk.x >> 3, item = (bk.x & 7) * chunk + li;
  if (li >= chunk || item >= total) return;  // whole workgroup exits
  const int p = item / per_prime, rem = item % per_prime;
  // consecutive items: the ciphertexts of one row, which share its twiddles
  const int c = rem % a.cnum, row0 = (rem / a.cnum) * RPW;
  const Mod Q(a.pc[p]);
  const uint32_t q = Q.q, two_q = Q.two_q, qneg = Q.qneg;
  const TwTab tw = tw_table(a.tw, p), itw = tw_table(a.itw, p);
  const int sg = T >= 64 ? __builtin_amdgcn_readfirstlane(row0 + s) : row0 + s;
  const int mult = ROWS + sg;
  const long long KN = (long long)a.K * N;
  const long long base = (long long)p * N + (long long)row0 * n;
  const uint32_t lane = 4u * (uint32_t)(s * n + t);
  const uint32_t row_bytes = 4u * RPW * n;
  uint32_t* lb[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) lb[b] = lds[b] + s * M::LDS_ROW;

  if constexpr (MODE == ROWS_TENSOR) {  // in place: slots 0..3 in, 0..2 out
    const __amdgpu_buffer_rsrc_t rs = row_buffer(wave_uniform(a.data + (long long)c * a.group_stride + base),
                                                 (uint32_t)(3 * KN * 4) + row_bytes);
    uint32_t x[4][16];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        x[r][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)lane, (int)(4 * (r * KN + u * T)), 0);
    mid_forward<S, 4, NB>(x, lb, t, tw, mult, Q);
    Tw16 w2;
    load_phase_tw<S, 2>(w2, itw, mult, t);  // in flight during the products
    __builtin_amdgcn_sched_barrier(0);
    // products as in rows_fused_kernel: inputs and outputs in [0, 2q)
    uint32_t d[3][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      d[0][u] = redc_lazy(mad64(x[0][u], x[2][u], 0), q, qneg);
      d[1][u] = csub(redc_lazy(mad64(x[0][u], x[3][u], mad64(x[1][u], x[2][u], 0)), q, qneg), two_q);
      d[2][u] = redc_lazy(mad64(x[1][u], x[3][u], 0), q, qneg);
    }
    mid_inverse<S, 3, NB>(d, lb, t, itw, mult, Q, w2);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        __builtin_amdgcn_raw_buffer_store_b32(d[r][u], rs, (int)lane, (int)(4 * (r * KN + u * T)), 0);
  } else if constexpr (MODE == ROWS_RELIN) {  // d2 rows times the key's two rows, to out
    const uint32_t bytes = (uint32_t)(KN * 4) + row_bytes;
    const __amdgpu_buffer_rsrc_t rk = row_buffer(wave_uniform(a.key + base), bytes);
    const __amdgpu_buffer_rsrc_t ri =
        row_buffer(wave_uniform(a.data + (long long)c * a.group_stride + base), row_bytes);
    uint32_t x[1][16], k[2][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[0][u] = __builtin_amdgcn_raw_buffer_load_b32(ri, (int)lane, 4 * u * T, 0);
    mid_forward<S, 1, NB>(x, lb, t, tw, mult, Q);
    // the key's rows are stored so that thread t's element 16 t + u sits at u T + t; all 32
    // words are issued together
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      k[0][u] = __builtin_amdgcn_raw_buffer_load_b32(rk, (int)lane, 4 * u * T, 0);
      k[1][u] = __builtin_amdgcn_raw_buffer_load_b32(rk, (int)lane, (int)(4 * (KN + u * T)), 0);
    }
    Tw16 w2;
    load_phase_tw<S, 2>(w2, itw, mult, t);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      // x in [0, 2q), key canonical: results in [0, 2q)
      k[0][u] = redc_lazy(mad64(x[0][u], k[0][u], 0), q, qneg);
      k[1][u] = redc_lazy(mad64(x[0][u], k[1][u], 0), q, qneg);
    }
    mid_inverse<S, 2, NB>(k, lb, t, itw, mult, Q, w2);
    const __amdgpu_buffer_rsrc_t ro = row_buffer(wave_uniform(a.out + (long long)c * a.out_stride + base), bytes);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        __builtin_amdgcn_raw_buffer_store_b32(k[r][u], ro, (int)lane, (int)(4 * (r * KN + u * T)), 0);
  } else {  // ring: a times b, in place of a
    const __amdgpu_buffer_rsrc_t ra =
        row_buffer(wave_uniform(a.data + (long long)c * a.group_stride + base), row_bytes);
    const __amdgpu_buffer_rsrc_t rb =
        row_buffer(wave_uniform(a.data2 + (long long)(c % a.data2_groups) * a.data2_stride + base), row_bytes);
    uint32_t x[2][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      x[0][u] = __builtin_amdgcn_raw_buffer_load_b32(ra, (int)lane, 4 * u * T, 0);
      x[1][u] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)lane, 4 * u * T, 0);
    }
    mid_forward<S, 2, NB>(x, lb, t, tw, mult, Q);
    Tw16 w2;
    load_phase_tw<S, 2>(w2, itw, mult, t);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t y[1][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) y[0][u] = redc_lazy(mad64(x[0][u], x[1][u], 0), q, qneg);  // [0, 2q)
    mid_inverse<S, 1, NB>(y, lb, t, itw, mult, Q, w2);
#pragma unroll
    for (int u = 0; u < 16; ++u) __builtin_amdgcn_raw_buffer_store_b32(y[0][u], ra, (int)lane, 4 * u * T, 0);
  }
}

// What bounds it: VALU issue.  2^16 points, 106 primes, 4 ciphertexts (tensor): 5 000 VALU
// instructions per wave, 40% of them 32-bit products at 4 clocks, adds at 2.4: 237 us of
// issue of the 323 us that a launch takes.  The tensor and ring forms are held to 128
// registers (4 waves per SIMD; 3 took 8% longer), the relinearization form to 96 (5).  Two
// ciphertexts per workgroup, sharing the row's key words and twiddles, needed 168 registers
// in that form and took 5% longer.
constexpr int mid_waves(int mode) { return mode == ROWS_RELIN ? 5 : 4; }

template <int S, int MODE>
__global__ __launch_bounds__(MidRow<S>::THREADS) __attribute__((amdgpu_waves_per_eu(mid_waves(MODE)))) void rows_mid_kernel(
    RowsArgs a) {
  rows_mid_kernel_body<S, MODE>(a, own_blk());
}

// The same over the cells of a stage-batched plan: one launch, each workgroup in its
// cell's segment (cell_of) with that cell's arguments.
template <int S, int MODE>
__global__ __launch_bounds__(MidRow<S>::THREADS) __attribute__((amdgpu_waves_per_eu(mid_waves(MODE)))) void rows_mid_kernel_multi(
    const RowsArgs* __restrict__ cells, const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  rows_mid_kernel_body<S, MODE>(cells[c], bk);
}

// The tensor and ring forms for few rows: a wave for each input polynomial, so that a
// product's forward transforms run side by side, and then its inverse ones; the values
// pass through the LDS in between.  Rows of up to 1024 points (N = 2^13 and 2^14), 1024 / n
// of them per workgroup, so that a wave's threads share a polynomial.
//
// What bounds it: at N = 2^14, 438 bits a product has 496 rows for 1024 SIMDs, and a wave's
// own chain (four forward transforms, the products and three inverse ones, 5 000
// instructions) sets the time; here the chain is one of each.  Tensor form, us (rows of
// 2^10): 15.4 -> 10.8 at 496, 24.2 -> 16.0 at 992, 28.7 -> 25.5 at 1984, 46.7 -> 44.8 at
// 3968; an HE-mult at N = 2^14, 438 bits: 66.5 -> 59.7.
template <int S, int MODE>
struct MidSplit {
  static constexpr int WAVES = MODE == ROWS_TENSOR ? 4 : 2, T = MidRow<S>::T, RPW = 64 / T;
};

// Where it is taken: rows in units of 1024 points, per compute unit.  Once every SIMD has
// its four waves of the other form, which loads a row's twiddles once for all polynomials,
// that one is as fast: ring form 8.0 -> 7.7 us at 496 rows, 11.8 -> 9.7 at 992, 20.2 ->
// 17.4 at 2976, 21.3 -> 21.4 at 3968; tensor form (above) up to 4096.  The relinearization
// form, which has one forward transform, gains nothing (11.4 -> 10.9 at 720 rows, 13.1 ->
// 15.8 at 1440).  A stage-batched plan, whose launches hold several cells' rows, keeps the
// other form.
constexpr int mid_split_rows(int mode) { return mode == ROWS_TENSOR ? 16 : (mode == ROWS_RING ? 12 : 0); }

template <int S, int MODE>
__global__ __launch_bounds__((64 * MidSplit<S, MODE>::WAVES)) void rows_mid_split_kernel(RowsArgs a) {
  typedef MidRow<S> M;
  typedef MidSplit<S, MODE> W;
  constexpr int n = M::n, T = M::T, RPW = W::RPW, ROWS = 16;
  __shared__ uint32_t lds[W::WAVES][RPW * M::LDS_ROW];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = (threadIdx.x & 63) / T, t = threadIdx.x % T;
  const int N = 1 << a.logN;
  // the order of the rows over the XCDs as in rows_mid_kernel
  const int per_prime = a.cnum * (ROWS / RPW), total = a.K * per_prime, chunk = (total + 7) / 8;
  const int li = blockIdx.x >> 3, item = (blockIdx.x & 7) * chunk + li;
  if (li >= chunk || item >= total) return;  // whole workgroup exits
  const int p = item / per_prime, rem = item % per_prime;
  const int c = rem % a.cnum, row0 = (rem / a.cnum) * RPW;
  const Mod Q(a.pc[p]);
  const uint32_t q = Q.q, two_q = Q.two_q, qneg = Q.qneg;
  const TwTab tw = tw_table(a.tw, p), itw = tw_table(a.itw, p);
  const int mult = ROWS + row0 + s;
  const long long KN = (long long)a.K * N;
  const long long base = (long long)p * N + (long long)row0 * n;
  const uint32_t lane = 4u * (uint32_t)(s * n + t);
  const uint32_t bytes = 4u * RPW * n;
  uint32_t* const lb[1] = {lds[wave] + s * M::LDS_ROW};
  // this thread's element u of the wave r's polynomial, between the transforms
  auto at = [&](int r, int u) -> uint32_t& { return lds[r][s * M::LDS_ROW + 17 * t + u]; };

  const uint32_t* src = a.data + (long long)c * a.group_stride;
  if (MODE == ROWS_TENSOR) src += wave * KN;
  if (MODE == ROWS_RING && wave == 1) src = a.data2 + (long long)(c % a.data2_groups) * a.data2_stride;
  const __amdgpu_buffer_rsrc_t ri = row_buffer(wave_uniform(src + base), bytes);
  uint32_t x[1][16];
#pragma unroll
  for (int u = 0; u < 16; ++u) x[0][u] = __builtin_amdgcn_raw_buffer_load_b32(ri, (int)lane, 4 * u * T, 0);
  mid_forward<S, 1, 1>(x, lb, t, tw, mult, Q);
#pragma unroll
  for (int u = 0; u < 16; ++u) at(wave, u) = x[0][u];
  Tw16 w2;
  load_phase_tw<S, 2>(w2, itw, mult, t);
  __syncthreads();
  if (MODE == ROWS_TENSOR) {
    if (wave == 1) {
#pragma unroll
      for (int u = 0; u < 16; ++u)
        x[0][u] = csub(redc_lazy(mad64(at(0, u), at(3, u), mad64(x[0][u], at(2, u), 0)), q, qneg), two_q);
    } else if (wave != 3) {
      const int l = wave == 0 ? 0 : 1;  // d0 = x0 x2, d2 = x1 x3
#pragma unroll
      for (int u = 0; u < 16; ++u) x[0][u] = redc_lazy(mad64(at(l, u), at(l + 2, u), 0), q, qneg);
    }
    __syncthreads();  // every wave's values have been read
    if (wave == 3) return;
  } else {
    if (wave == 1) return;
#pragma unroll
    for (int u = 0; u < 16; ++u) x[0][u] = redc_lazy(mad64(x[0][u], at(1, u), 0), q, qneg);
  }
  mid_inverse<S, 1, 1>(x, lb, t, itw, mult, Q, w2);
  uint32_t* const dst = a.data + (long long)c * a.group_stride + (MODE == ROWS_TENSOR ? wave * KN : 0);
  const __amdgpu_buffer_rsrc_t ro = row_buffer(wave_uniform(dst + base), bytes);
#pragma unroll
  for (int u = 0; u < 16; ++u) __builtin_amdgcn_raw_buffer_store_b32(x[0][u], ro, (int)lane, 4 * u * T, 0);
}

template <int S, int MODE>
static hipError_t rows_mid(const RowsArgs& a, hipStream_t st) {
  const int total = a.K * a.cnum * (16 / MidRow<S>::RPW);
  // algorithmic HBM bytes per prime, as in the fused pass of kernels.hip
  const int b_rows = a.data2_stride ? std::min(a.data2_groups, a.cnum) : 1;
  const double rows = MODE == ROWS_TENSOR ? 7.0 * a.cnum
                                          : (MODE == ROWS_RELIN ? 3.0 * a.cnum + 2.0 : 2.0 * a.cnum + b_rows);
  Bracket br(KID_ROWS_FUSED, st, 4.0 * rows * a.K * (double)(1 << a.logN));
  if constexpr (S <= 10 && mid_split_rows(MODE) > 0) {
    typedef MidSplit<S, MODE> W;
    const int items = a.K * a.cnum * (16 / W::RPW);
    if (!launch_sink() && items <= mid_split_rows(MODE) * a.cus) {
      hipLaunchKernelGGL((rows_mid_split_kernel<S, MODE>), dim3(8 * ((items + 7) / 8)), dim3(64 * W::WAVES), 0, st, a);
      return hipGetLastError();
    }
  }
  const hipError_t e = emit((const void*)rows_mid_kernel<S, MODE>, (const void*)rows_mid_kernel_multi<S, MODE>,
                            dim3(8 * ((total + 7) / 8)), dim3(MidRow<S>::THREADS), 0, st, a);
  return e != hipSuccess ? e : hipGetLastError();
}

template <int S>
static hipError_t rows_mid_mode(const RowsArgs& a, int mode, hipStream_t st) {
  switch (mode) {
    case ROWS_TENSOR: return rows_mid<S, ROWS_TENSOR>(a, st);
    case ROWS_RELIN: return rows_mid<S, ROWS_RELIN>(a, st);
    case ROWS_RING: return rows_mid<S, ROWS_RING>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rows_mid(const RowsArgs& a, int mode, hipStream_t st) {
  if (a.cnum <= 0) return hipSuccess;
  // a workgroup's buffers span up to 3 K N words past their base (32-bit byte offsets)
  if (((3LL * a.K << a.logN) + 4096) * 4 >= 0x70000000LL) return hipErrorInvalidValue;
  switch (a.logN - 4) {
    case 9: return rows_mid_mode<9>(a, mode, st);
    case 10: return rows_mid_mode<10>(a, mode, st);
    case 11: return rows_mid_mode<11>(a, mode, st);
    case 12: return rows_mid_mode<12>(a, mode, st);
    default: return hipErrorInvalidValue;
  }
}

// The first four stages on their own, after a lift that cannot take them: a thread holds one
// column {c + (N / 16) u} of a transform; residues in [0, 2q) in, [-2q, 2q) out.
__device__ __forceinline__ void cols16_kernel_body(const NttArgs& a, const Blk bk) {
  const int cols = 1 << (a.logN - 4);  // at least 64: a wave's columns are one transform's
  const long long w = (long long)bk.x * 256 + threadIdx.x;
  const int tr = __builtin_amdgcn_readfirstlane((int)(w >> (a.logN - 4)));
  if (tr >= a.ntr) return;
  const int g = tr / a.per_group, r = tr % a.per_group, p = r % a.K;
  const uint32_t c4 = 4u * (uint32_t)(w & (cols - 1));
  const __amdgpu_buffer_rsrc_t rb = row_buffer(
      wave_uniform(a.data + (long long)g * a.group_stride + ((long long)r << a.logN)), 4u << a.logN);
  uint32_t x[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) x[u] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)c4, 4 * u * cols, 0);
  cols16_forward(x, tw_table(a.tw, p), Mod(a.pc[p]));
#pragma unroll
  for (int u = 0; u < 16; ++u) __builtin_amdgcn_raw_buffer_store_b32(x[u], rb, (int)c4, 4 * u * cols, 0);
}

__global__ __launch_bounds__(256) void cols16_kernel(NttArgs a) { cols16_kernel_body(a, own_blk()); }

__global__ __launch_bounds__(256) void cols16_kernel_multi(const NttArgs* __restrict__ cells,
                                                           const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  cols16_kernel_body(cells[c], bk);
}

hipError_t launch_cols16(const NttArgs& a0, int ntr, hipStream_t st) {
  if (ntr <= 0) return hipSuccess;
  if (ntr % a0.K != 0 || a0.per_group % a0.K != 0 || a0.logN < 10) return hipErrorInvalidValue;
  NttArgs a = a0;
  a.ntr = ntr;
  const long long threads = (long long)ntr << (a.logN - 4);
  // algorithmic HBM bytes: every element of every transform read and written once
  Bracket br(KID_NTT_FWD_COLS, st, 8.0 * ntr * (double)(1 << a.logN));
  const hipError_t e = emit((const void*)cols16_kernel, (const void*)cols16_kernel_multi,
                            dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace fhe
