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

// A phase's twiddles of one thread: the stage of c groups per thread has its c pairs at
// [c - 1, 2 c - 1).
struct Tw15 {
  uint2 w[15];
};

// Phase I's twiddles: the stage with c groups per thread starts at table index
// mult c G + (thread's block) c, G the groups of the phase's first stage over the row.
// MIR: minus the inverse ones, from the forward table read backwards (mirror_tw) at the
// mirrored multiplier.
template <int S, int I, bool MIR>
__device__ __forceinline__ void load_phase_tw(Tw15& w, TwTab tw, int mult, int t) {
  typedef MidRow<S> M;
  constexpr int G = I == 0 ? 1 : (I == 1 ? 16 : M::T);
  const int blk = I == 0 ? 0 : (I == 1 ? t / M::C : t);
#pragma unroll
  for (int c = I == 2 ? M::C2 : 1; c <= 8; c *= 2) {
    const int b = MIR ? mult * c * G - (blk + 1) * c : mult * c * G + blk * c;
    if (I == 0 || c == 1) {  // wave-uniform (scalar loads), or a single entry
#pragma unroll
      for (int g = 0; g < c; ++g) w.w[c - 1 + (MIR ? c - 1 - g : g)] = tw[b + g];
    } else {
#pragma unroll
      for (int g = 0; g < c; g += 2) {
        const v4i_t v = tw.pair(b + g);
        w.w[c - 1 + (MIR ? c - 1 - g : g)] = make_uint2((uint32_t)v[0], (uint32_t)v[1]);
        w.w[c - 1 + (MIR ? c - 2 - g : g + 1)] = make_uint2((uint32_t)v[2], (uint32_t)v[3]);
      }
    }
  }
}

template <int S, int I, int NP>
__device__ __forceinline__ void fwd_phase(uint32_t (&x)[NP][16], const Tw15& w, uint32_t q, uint32_t two_q) {
#pragma unroll
  for (int c = I == 2 ? MidRow<S>::C2 : 1; c <= 8; c *= 2) {
    const int h = 8 / c;
#pragma unroll
    for (int g = 0; g < c; ++g)
#pragma unroll
      for (int r = 0; r < NP; ++r)
#pragma unroll
        for (int u = 2 * h * g; u < 2 * h * g + h; ++u) ct_bfly(x[r][u], x[r][u + h], w.w[c - 1 + g], q, two_q);
  }
}

template <int S, int I, int NP>
__device__ __forceinline__ void inv_phase(uint32_t (&x)[NP][16], const Tw15& w, uint32_t q, uint32_t two_q) {
#pragma unroll
  for (int c = 8; c >= (I == 2 ? MidRow<S>::C2 : 1); c /= 2) {
    const int h = 8 / c;
#pragma unroll
    for (int g = 0; g < c; ++g) {
      const uint2 f = w.w[c - 1 + g];
      const uint2 v = I == 0 && MidRow<S>::T >= 64
                          ? mirror_tw_s(make_uint2(__builtin_amdgcn_readfirstlane(f.x), __builtin_amdgcn_readfirstlane(f.y)))
                          : mirror_tw(f);
#pragma unroll
      for (int r = 0; r < NP; ++r)
#pragma unroll
        for (int u = 2 * h * g; u < 2 * h * g + h; ++u) gs_bfly_neg(x[r][u], x[r][u + h], v, q, two_q);
    }
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

// All row stages of NP forward transforms: values in [0, 4q) at elements u T + t, left in
// [0, 2q) at 16 t + u.  A phase's twiddles are issued before the exchange that precedes it.
template <int S, int NP, int NB>
__device__ __forceinline__ void mid_forward(uint32_t (&x)[NP][16], uint32_t* const (&l)[NB], int t, TwTab tw, int mult,
                                            uint32_t q, uint32_t two_q) {
  Tw15 w0, w1, w2;
  load_phase_tw<S, 0, false>(w0, tw, mult, t);
  load_phase_tw<S, 1, false>(w1, tw, mult, t);
  __builtin_amdgcn_sched_barrier(0);
  fwd_phase<S, 0, NP>(x, w0, q, two_q);
  mid_exchange<S, 0, 1, NP, NB>(x, l, t);
  fwd_phase<S, 1, NP>(x, w1, q, two_q);
  __builtin_amdgcn_sched_barrier(0);  // the registers do not hold two phases' twiddles
  load_phase_tw<S, 2, false>(w2, tw, mult, t);
  __builtin_amdgcn_sched_barrier(0);
  mid_exchange<S, 1, 2, NP, NB>(x, l, t);
  fwd_phase<S, 2, NP>(x, w2, q, two_q);
#pragma unroll
  for (int r = 0; r < NP; ++r)
#pragma unroll
    for (int u = 0; u < 16; ++u) x[r][u] = csub(x[r][u], two_q);
}

// The row stages of NP inverse transforms, values in [0, 2q) from 16 t + u to u T + t; w2
// holds phase 2's twiddles (loaded before the products).
template <int S, int NP, int NB>
__device__ __forceinline__ void mid_inverse(uint32_t (&x)[NP][16], uint32_t* const (&l)[NB], int t, TwTab tw,
                                            int mirror, uint32_t q, uint32_t two_q, const Tw15& w2) {
  Tw15 w0, w1;
  inv_phase<S, 2, NP>(x, w2, q, two_q);
  __builtin_amdgcn_sched_barrier(0);
  load_phase_tw<S, 1, true>(w1, tw, mirror, t);
  __builtin_amdgcn_sched_barrier(0);
  mid_exchange<S, 2, 1, NP, NB>(x, l, t);
  load_phase_tw<S, 0, true>(w0, tw, mirror, t);
  inv_phase<S, 1, NP>(x, w1, q, two_q);
  mid_exchange<S, 1, 0, NP, NB>(x, l, t);
  inv_phase<S, 0, NP>(x, w0, q, two_q);
}

// CG ciphertexts per row of the relinearization form: they share the row's twiddles and
// key words.
template <int S, int MODE, int CG>
__device__ __forceinline__ void rows_mid_kernel_body(const RowsArgs& a, const Blk bk) {
  typedef MidRow<S> M;
  constexpr int n = M::n, T = M::T, RPW = M::RPW, NB = MODE == ROWS_RELIN && CG == 1 ? 1 : 2;
  static_assert(CG == 1 || MODE == ROWS_RELIN, "only the relinearization form groups ciphertexts");
  __shared__ uint32_t lds[NB][RPW * M::LDS_ROW];
  const int s = threadIdx.x / T, t = threadIdx.x % T;
  const int N = 1 << a.logN;
  constexpr int ROWS = 16;  // rows of a transform
  // Workgroup w runs on XCD w % 8.  The rows, ordered by prime, are cut into eight runs of
  // equal length, one per XCD: a prime's table and key rows are read into one L2, and the
  // XCDs finish together whatever K is.
  const int ncg = (a.cnum + CG - 1) / CG;
  const int per_prime = ncg * (ROWS / RPW), total = a.K * per_prime, chunk = (total + 7) / 8;
  const int li = bk.x >> 3, item = (bk.x & 7) * chunk + li;
  if (li >= chunk || item >= total) return;  // whole workgroup exits
  const int p = item / per_prime, rem = item % per_prime;
  // consecutive items: the groups of ciphertexts of one row, which share its twiddles
  const int c = (rem % ncg) * CG, row0 = (rem / ncg) * RPW;
  const PrimeC pc = a.pc[p];
  const uint32_t q = pc.q, two_q = pc.two_q, qneg = pc.qneg;
  const TwTab tw = tw_table(a.tw, p);
  const int sg = T >= 64 ? __builtin_amdgcn_readfirstlane(row0 + s) : row0 + s;
  const int mult = ROWS + sg, mirror = 2 * ROWS - sg;
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
        x[r][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(lane + 4u * u * T), (int)(4 * r * KN), 0);
    mid_forward<S, 4, NB>(x, lb, t, tw, mult, q, two_q);
    Tw15 w2;
    load_phase_tw<S, 2, true>(w2, tw, mirror, t);  // in flight during the products
    __builtin_amdgcn_sched_barrier(0);
    // products as in rows_fused_kernel: inputs and outputs in [0, 2q)
    uint32_t d[3][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      d[0][u] = redc_lazy(mad64(x[0][u], x[2][u], 0), q, qneg);
      d[1][u] = csub(redc_lazy(mad64(x[0][u], x[3][u], mad64(x[1][u], x[2][u], 0)), q, qneg), two_q);
      d[2][u] = redc_lazy(mad64(x[1][u], x[3][u], 0), q, qneg);
    }
    mid_inverse<S, 3, NB>(d, lb, t, tw, mirror, q, two_q, w2);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int u = 0; u < 16; ++u)
        __builtin_amdgcn_raw_buffer_store_b32(d[r][u], rs, (int)(lane + 4u * u * T), (int)(4 * r * KN), 0);
  } else if constexpr (MODE == ROWS_RELIN) {  // d2 rows times the key's two rows, to out
    const uint32_t bytes = (uint32_t)(KN * 4) + row_bytes;
    const __amdgpu_buffer_rsrc_t rk = row_buffer(wave_uniform(a.key + base), bytes);
    uint32_t x[CG][16], k[2 * CG][16];
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      // a ciphertext past the last reads zeros and stores nothing (an empty buffer)
      const bool in = c + g < a.cnum;
      const __amdgpu_buffer_rsrc_t ri = row_buffer(
          wave_uniform(a.data + (in ? (long long)(c + g) * a.group_stride + base : 0)), in ? row_bytes : 0);
#pragma unroll
      for (int u = 0; u < 16; ++u) x[g][u] = __builtin_amdgcn_raw_buffer_load_b32(ri, (int)(lane + 4u * u * T), 0, 0);
    }
    mid_forward<S, CG, NB>(x, lb, t, tw, mult, q, two_q);
    // the key's rows are stored so that thread t's element 16 t + u sits at u T + t; all 32
    // words are issued together
    uint32_t kw[2][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      kw[0][u] = __builtin_amdgcn_raw_buffer_load_b32(rk, (int)(lane + 4u * u * T), 0, 0);
      kw[1][u] = __builtin_amdgcn_raw_buffer_load_b32(rk, (int)(lane + 4u * u * T), (int)(4 * KN), 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 16; ++u)
#pragma unroll
      for (int g = CG - 1; g >= 0; --g) {
        // x in [0, 2q), key canonical: results in [0, 2q)
        k[2 * g][u] = redc_lazy(mad64(x[g][u], kw[0][u], 0), q, qneg);
        k[2 * g + 1][u] = redc_lazy(mad64(x[g][u], kw[1][u], 0), q, qneg);
      }
    Tw15 w2;
    load_phase_tw<S, 2, true>(w2, tw, mirror, t);
    mid_inverse<S, 2 * CG, NB>(k, lb, t, tw, mirror, q, two_q, w2);
#pragma unroll
    for (int g = 0; g < CG; ++g) {
      const bool in = c + g < a.cnum;
      const __amdgpu_buffer_rsrc_t ro =
          row_buffer(wave_uniform(a.out + (in ? (long long)(c + g) * a.out_stride + base : 0)), in ? bytes : 0);
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int u = 0; u < 16; ++u)
          __builtin_amdgcn_raw_buffer_store_b32(k[2 * g + r][u], ro, (int)(lane + 4u * u * T), (int)(4 * r * KN), 0);
    }
  } else {  // ring: a times b, in place of a
    const __amdgpu_buffer_rsrc_t ra =
        row_buffer(wave_uniform(a.data + (long long)c * a.group_stride + base), row_bytes);
    const __amdgpu_buffer_rsrc_t rb =
        row_buffer(wave_uniform(a.data2 + (long long)(c % a.data2_groups) * a.data2_stride + base), row_bytes);
    uint32_t x[2][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      x[0][u] = __builtin_amdgcn_raw_buffer_load_b32(ra, (int)(lane + 4u * u * T), 0, 0);
      x[1][u] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)(lane + 4u * u * T), 0, 0);
    }
    mid_forward<S, 2, NB>(x, lb, t, tw, mult, q, two_q);
    Tw15 w2;
    load_phase_tw<S, 2, true>(w2, tw, mirror, t);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t y[1][16];
#pragma unroll
    for (int u = 0; u < 16; ++u) y[0][u] = redc_lazy(mad64(x[0][u], x[1][u], 0), q, qneg);  // [0, 2q)
    mid_inverse<S, 1, NB>(y, lb, t, tw, mirror, q, two_q, w2);
#pragma unroll
    for (int u = 0; u < 16; ++u) __builtin_amdgcn_raw_buffer_store_b32(y[0][u], ra, (int)(lane + 4u * u * T), 0, 0);
  }
}

template <int S, int MODE, int CG>
__global__ __launch_bounds__(MidRow<S>::THREADS) __attribute__((amdgpu_waves_per_eu(3))) void rows_mid_kernel(
    RowsArgs a) {
  rows_mid_kernel_body<S, MODE, CG>(a, own_blk());
}

// The same over the cells of a stage-batched plan: one launch, each workgroup in its
// cell's segment (cell_of) with that cell's arguments.
template <int S, int MODE, int CG>
__global__ __launch_bounds__(MidRow<S>::THREADS) __attribute__((amdgpu_waves_per_eu(3))) void rows_mid_kernel_multi(
    const RowsArgs* __restrict__ cells, const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  rows_mid_kernel_body<S, MODE, CG>(cells[c], bk);
}

template <int S, int MODE, int CG>
static hipError_t rows_mid(const RowsArgs& a, hipStream_t st) {
  const int total = a.K * ((a.cnum + CG - 1) / CG) * (16 / MidRow<S>::RPW);
  // algorithmic HBM bytes per prime, as in the fused pass of kernels.hip
  const int b_rows = a.data2_stride ? std::min(a.data2_groups, a.cnum) : 1;
  const double rows = MODE == ROWS_TENSOR ? 7.0 * a.cnum
                                          : (MODE == ROWS_RELIN ? 3.0 * a.cnum + 2.0 : 2.0 * a.cnum + b_rows);
  Bracket br(KID_ROWS_FUSED, st, 4.0 * rows * a.K * (double)(1 << a.logN));
  const hipError_t e = emit((const void*)rows_mid_kernel<S, MODE, CG>, (const void*)rows_mid_kernel_multi<S, MODE, CG>,
                            dim3(8 * ((total + 7) / 8)), dim3(MidRow<S>::THREADS), 0, st, a);
  return e != hipSuccess ? e : hipGetLastError();
}

template <int S>
static hipError_t rows_mid_mode(const RowsArgs& a, int mode, hipStream_t st) {
  switch (mode) {
    case ROWS_TENSOR: return rows_mid<S, ROWS_TENSOR, 1>(a, st);
    case ROWS_RELIN: return a.cnum > 1 ? rows_mid<S, ROWS_RELIN, 2>(a, st) : rows_mid<S, ROWS_RELIN, 1>(a, st);
    case ROWS_RING: return rows_mid<S, ROWS_RING, 1>(a, st);
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

// The four outer stages on their own, where the lift or the reconstruction cannot take
// them: a thread holds one column {c + (N / 16) u} of a transform; forward values in
// [0, 4q) out, inverse ones canonical, times the final factor if there is one.
template <bool INV>
__device__ __forceinline__ void cols16_kernel_body(const NttArgs& a, const Blk bk) {
  const int cols = 1 << (a.logN - 4);  // at least 64: a wave's columns are one transform's
  const long long w = (long long)bk.x * 256 + threadIdx.x;
  const int tr = __builtin_amdgcn_readfirstlane((int)(w >> (a.logN - 4)));
  if (tr >= a.ntr) return;
  const int g = tr / a.per_group, r = tr % a.per_group, p = r % a.K;
  const uint32_t c4 = 4u * (uint32_t)(w & (cols - 1));
  const __amdgpu_buffer_rsrc_t rb = row_buffer(
      wave_uniform(a.data + (long long)g * a.group_stride + ((long long)r << a.logN)), 4u << a.logN);
  const PrimeC pc = a.pc[p];
  const uint32_t q = pc.q, two_q = pc.two_q;
  const TwTab tw = tw_table(a.tw, p);
  uint32_t x[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) x[u] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)c4, 4 * u * cols, 0);
  if (!INV) cols16_forward(x, tw, q, two_q);
  else if (a.scale) cols16_inverse<true>(x, tw, a.scale[p], a.scale_w[p], q, two_q);
  else cols16_inverse<false>(x, tw, make_uint2(0, 0), make_uint2(0, 0), q, two_q);
#pragma unroll
  for (int u = 0; u < 16; ++u) __builtin_amdgcn_raw_buffer_store_b32(x[u], rb, (int)c4, 4 * u * cols, 0);
}

template <bool INV>
__global__ __launch_bounds__(256) void cols16_kernel(NttArgs a) {
  cols16_kernel_body<INV>(a, own_blk());
}
template <bool INV>
__global__ __launch_bounds__(256) void cols16_kernel_multi(const NttArgs* __restrict__ cells,
                                                           const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  cols16_kernel_body<INV>(cells[c], bk);
}

hipError_t launch_cols16(const NttArgs& a0, int ntr, bool inverse, hipStream_t st) {
  if (ntr <= 0) return hipSuccess;
  if (ntr % a0.K != 0 || a0.per_group % a0.K != 0 || a0.logN < 10) return hipErrorInvalidValue;
  NttArgs a = a0;
  a.ntr = ntr;
  const long long threads = (long long)ntr << (a.logN - 4);
  // algorithmic HBM bytes: every element of every transform read and written once
  Bracket br(inverse ? KID_NTT_INV_COLS : KID_NTT_FWD_COLS, st, 8.0 * ntr * (double)(1 << a.logN));
  const hipError_t e =
      inverse ? emit((const void*)cols16_kernel<true>, (const void*)cols16_kernel_multi<true>,
                     dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a)
              : emit((const void*)cols16_kernel<false>, (const void*)cols16_kernel_multi<false>,
                     dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace fhe
