// CRT reconstruction (residues -> limbs, on the i8 matrix cores) with the last four inverse
// transform stages.
#include <algorithm>

#include "device_common.h"

namespace fhe {

// Residues -> limbs (the reconstruction step of Section 5.1 / Eq. garner_mrc, here in its
// direct CRT form).  With M = q_0 ... q_(K-1), c_k = [(M/q_k)^-1]_(q_k) and the inverse
// NTT's final factor including c_k, a transform output x_k (any representative) gives
// y_k = x_k + d_k, d_k = [2^e c_k]_(q_k), CRT coordinates of Y = X + 2^e in [0, 2^(e+1))
// (X the signed exact product, |X| < 2^e).  Then
//   Y = sum_k y_k (M/q_k) - alpha M,   alpha = floor(sum_k y_k / q_k),
// and the output is X mod 2^outbits = (Y - 2^e) mod 2^outbits.  No y_k has to be reduced:
// a multiple of q_k more adds the same multiple of M to the sum and to alpha M.  The d_k
// are constants, so sum_k d_k (M/q_k) joins the constant row and sum_k d_k / q_k the
// constant of the quotient; what is left per residue is x_k itself, in [0, 2 q_k).
// The prime count leaves Y / M < 2^-16, so alpha is exact from the sum in fixed point
// sum_k x_k floor(2^54 / q_k): a truncated reciprocal is short by less than 2^-54, so that
// the x_k below 2 q_k and the d_k below q_k lose less than K 3 2^30 2^-54, 2^-14 for the up
// to 256 primes, and an offset of 2^-10 covers it.
//
// The column sums sum_k x_k V_kl, V_kl = limb l of (M/q_k) mod 2^(32 Lout), are a dense
// integer contraction [coefficients x K] x [K x Lout] and run on the i8 matrix cores:
// x_k - 0x80808080 and V_kl are split into 4 balanced base-256 digits each (digits in
// [-128, 127]; the digits of x_k - 0x80808080 are the bytes of x_k ^ 0x80808080, and limbs
// of V are taken in [-0x80808080, 0x7F7F7F7F]), the 16 digit-plane products accumulate
// exactly in int32 (|sum| <= K 2^14), and the VALU recombines sum_(a,b) 2^(8(a+b)) C_ab per
// limb (the 7 diagonal sums in int32, then 64-bit multiply-adds), adds alpha [-M] and the
// constant row (limbs mod 2^(32 Lout)), and propagates the carries.
//
// A workgroup of 8 waves takes 16 columns {c + (N / 16) u} of a polynomial, 256
// coefficients.  Per 32 primes, thread (prime, column) runs the column's 16-point stages
// and leaves the values in LDS; then wave w takes rows 2 w and 2 w + 1, a unit of 32
// coefficients whose digit planes of all primes it collects in registers for the products.
// MFMA v_mfma_i32_32x32x32_i8: lane (c, h) = (lane mod 32, lane / 32) supplies B bytes
// k = 32 kb + 16 h + i (i < 16) of coefficient column c, and A bytes of row c for the same
// k; its accumulator holds rows 8 j + 4 h + i.  Rows of a tile are (digit plane b of V,
// limb 8 t + l'), row = 8 b + l', so lane half h ends with all four planes of limbs
// 8 t + 4 h + i.
//
// What bounds it: instruction issue.  For 158 primes and 98 limbs an item takes 47 000
// clocks: stages and digit planes 24 000 (VALU), products and carries 23 000 (16 600 of them
// matrix instructions).  Neither all of an item's loads ahead, nor the next item's stages
// beside the products, nor workgroups half an item apart changed its time by more than 1%.
// 2^16 coefficients, 8 polynomials: 260 us (12 polynomials, 106 primes, 49 limbs: 225); the
// separate column pass of eight stages and reconstruction took 140 + 175 (140 + 131).

// 4 x 32-bit words -> their byte plane a (a < 4) as 4 packed bytes, for all planes.
__device__ __forceinline__ void byte_planes(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t& p0,
                                            uint32_t& p1, uint32_t& p2, uint32_t& p3) {
  // v_perm_b32: result byte i = byte sel_i of {src0 (bytes 4..7), src1 (bytes 0..3)}
  const uint32_t lo01 = __builtin_amdgcn_perm(w1, w0, 0x05010400u);  // w0.0 w1.0 w0.1 w1.1
  const uint32_t hi01 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);  // w0.2 w1.2 w0.3 w1.3
  const uint32_t lo23 = __builtin_amdgcn_perm(w3, w2, 0x05010400u);
  const uint32_t hi23 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
  p0 = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);  // w0.0 w1.0 w2.0 w3.0
  p1 = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
  p2 = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
  p3 = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

// Exchange buffers: two (one barrier per 32 primes) where the table still fits beside them.
template <int NKB>
constexpr int crt_bufs() { return NKB <= 5 ? 2 : 1; }

constexpr int kCrtRow = 32 * 16 + 48;  // exchange words per row u: rows and prime halves on different banks
constexpr int kCrtTw = 20;             // words of a prime's twiddles (four primes on different banks)

// Dynamic LDS: the digit table (LDSA), the exchange buffers, twiddles and constants.
static size_t crt_lds(int nkb, int bufs, int ntiles, bool table) {
  return ((table ? (size_t)ntiles * nkb * 256 : 0) + (size_t)bufs * 16 * kCrtRow + (size_t)32 * nkb * (kCrtTw + 3) +
          16 * ntiles) * 4;
}

template <int NKB, bool LDSA>
__device__ __forceinline__ void crt_cols_kernel_body(const CrtArgs& a, const Blk bk) {
  constexpr int WAVES = 8, BUFS = crt_bufs<NKB>();
  extern __shared__ v4i sA[];
  uint32_t* const s_x = (uint32_t*)(sA + (LDSA ? a.ntiles * NKB * 64 : 0));
  uint32_t* const s_tw = s_x + BUFS * 16 * kCrtRow;  // [prime]: final factor, its second half or entry 1, entries 2..15
  uint32_t* const s_q = s_tw + 32 * NKB * kCrtTw;
  uint32_t* const s_qn = s_q + 32 * NKB;
  uint32_t* const s_r = s_qn + 32 * NKB;
  uint32_t* const s_mneg = s_r + 32 * NKB;
  uint32_t* const s_eneg = s_mneg + 8 * a.ntiles;
  for (int k = threadIdx.x; k < 32 * NKB; k += 64 * WAVES) {
    const bool in = k < a.K;
    s_q[k] = in ? a.pc[k].q : 1u;
    s_qn[k] = in ? a.pc[k].qneg : 0u;
    s_r[k] = in ? a.rq[k] : 0u;  // rows past K add nothing to the quotient
  }
  for (int i = threadIdx.x; i < 32 * NKB * 16; i += 64 * WAVES) {
    const int k = i >> 4, e = i & 15;
    const uint32_t* src = a.scale && e < 2 ? (e ? a.scale_w : a.scale) + k : a.itw + (long long)k * kNMax + e;
    s_tw[k * kCrtTw + e] = k < a.K ? *src : 0u;
  }
  for (int l = threadIdx.x; l < 8 * a.ntiles; l += 64 * WAVES) {
    s_mneg[l] = a.mneg[l];
    s_eneg[l] = a.eneg[l];
  }
  if (LDSA)
    for (int f = threadIdx.x; f < a.ntiles * NKB * 64; f += 64 * WAVES) sA[f] = a.A[f];
  __syncthreads();
  const v4i* At = LDSA ? sA : a.A;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this thread's lane as (c, h), and its prime and column of a block of 32 primes; made
  // opaque again for each item, or the offsets derived from them would be hoisted out of the
  // item loop, each holding a register
  uint32_t lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5, pr = threadIdx.x >> 4, col = lane & 15;
  const uint32_t row = 4u * (uint32_t)a.N;                       // bytes between residue (or limb) rows
  const uint64_t frac0 = a.frac0;
  const bool scaled = a.scale != nullptr;

  // Workgroup w runs on XCD w % 8; an XCD's workgroups take neighbouring blocks of columns,
  // which share cache lines.
  const int nblk = a.N >> 8, total = a.npoly * nblk, chunk = (total + 7) / 8;
  const int first = (int)(bk.x & 7) * chunk, end = min(first + chunk, total), step = (int)(bk.nx >> 3);
  int item = first + (int)(bk.x >> 3);
  if (item >= end) return;  // whole workgroup exits

  // residues of primes 32 kb + pr, this thread's column; rows at or beyond K read as zero
  auto source = [&](int it, uint32_t& left) {
    const int z = it / nblk;
    const uint32_t j0 = 16u * (uint32_t)(it % nblk);
    left = 4u * ((uint32_t)a.K * (uint32_t)a.N - j0);
    return wave_uniform(a.res + (long long)(z / a.per_group) * a.gstride + (long long)(z % a.per_group) * a.pstride + j0);
  };
  auto fetch = [&](uint32_t (&x)[16], const uint32_t* xb, uint32_t left, int kb) {
    const __amdgpu_buffer_rsrc_t rs = row_buffer(xb, left);
    const uint32_t off = (32u * kb + pr) * row + 4u * col;
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, (int)(u * (row >> 4)), 0);
  };
  // the last four inverse stages of this thread's column of block kb
  auto stages = [&](uint32_t (&x)[16], int kb) {
    const uint32_t k = 32u * kb + pr;
    const Mod M(s_q[k], s_qn[k]);
    const uint32_t* const tp = s_tw + k * kCrtTw;
    uint32_t w[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] = tp[e];
#pragma unroll
    for (int m = 8; m >= 2; m /= 2) {
      const int d = 8 / m;
#pragma unroll
      for (int g = 0; g < m; ++g)
#pragma unroll
        for (int u = 2 * d * g; u < 2 * d * g + d; ++u) gs_bfly(x[u], x[u + d], w[m + g], M);
    }
    if (scaled) {  // the last stage with the final factor folded in
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t xs = x[u], ys = x[u + 8];
        x[u] = mont_s(xs + ys + M.neg2q, w[0], M);
        x[u + 8] = mont_s(xs - ys, w[1], M);
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) gs_bfly(x[u], x[u + 8], w[1], M);
    }
  };
  uint32_t nb = 0;  // blocks of primes done, modulo the buffers
  auto store = [&](const uint32_t (&x)[16]) {
    uint32_t* const xw = s_x + (BUFS == 2 ? (nb & 1) * 16 * kCrtRow : 0) + pr * 16 + (pr >> 4) * 32 + col;
#pragma unroll
    for (int u = 0; u < 16; ++u) xw[u * kCrtRow] = x[u];
  };
  uint32_t left;
  const uint32_t* xb = source(item, left);
  // Residues of every block: as a block's digit planes take their 16 registers, the
  // residues they came from leave 16, so all of an item's loads can be in flight at once.
  uint32_t xv[NKB][16];
  fetch(xv[0], xb, left, 0);

  for (; item < end; item += step) {
    const int z = item / nblk;
    const uint32_t j0 = 16u * (uint32_t)(item % nblk);
    opaque(lane);
    opaque(c);
    opaque(h);
    opaque(pr);
    opaque(col);

    // phase 1: the last transform stages, then x_k's part of the quotient and digit planes.
    // Between two barriers a wave reads its unit of one block and runs the stages of the next
    // while the reads are in flight.
    v4i B[NKB][4];
    uint64_t frac = 0;  // sum_k x_k floor(2^54 / q_k)
#pragma unroll
    for (int kb = 1; kb < NKB; ++kb) fetch(xv[kb], xb, left, kb);
    __builtin_amdgcn_sched_barrier(0);
    stages(xv[0], 0);
    store(xv[0]);
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      __syncthreads();
      uint32_t s[16];
      uint4 rq[4];
      {
        const uint32_t* const xr = s_x + (BUFS == 2 ? (nb & 1) * 16 * kCrtRow : 0) +
                                   (2 * wave + (c >> 4)) * kCrtRow + h * (16 * 16 + 32) + (c & 15);
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = xr[16 * i];
        const uint4* const rp = (const uint4*)(s_r + 32 * kb + 16 * h);
#pragma unroll
        for (int i = 0; i < 4; ++i) rq[i] = rp[i];
      }
      ++nb;
      __builtin_amdgcn_sched_barrier(0);
      if (kb + 1 < NKB) stages(xv[kb + 1], kb + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        frac += (uint64_t)s[4 * r] * rq[r].x;
        frac += (uint64_t)s[4 * r + 1] * rq[r].y;
        frac += (uint64_t)s[4 * r + 2] * rq[r].z;
        frac += (uint64_t)s[4 * r + 3] * rq[r].w;
        asm volatile("" : "+v"(frac));  // here, or all blocks' residues stay live to the end
        uint32_t p0, p1, p2, p3;
        byte_planes(s[4 * r], s[4 * r + 1], s[4 * r + 2], s[4 * r + 3], p0, p1, p2, p3);
        p0 ^= 0x80808080u;
        p1 ^= 0x80808080u;
        p2 ^= 0x80808080u;
        p3 ^= 0x80808080u;
        // materialised here: left to the compiler, the planes may be recomputed later
        opaque(p0);
        opaque(p1);
        opaque(p2);
        opaque(p3);
        B[kb][0][r] = (int)p0;
        B[kb][1][r] = (int)p1;
        B[kb][2][r] = (int)p2;
        B[kb][3][r] = (int)p3;
      }
      if (kb + 1 < NKB) {
        if (BUFS == 1) __syncthreads();  // the one buffer has been read
        store(xv[kb + 1]);
      }
    }
    if (BUFS == 1) __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    frac = sum_lane_halves(frac) + frac0;
    const uint32_t alpha = (uint32_t)(frac >> 54);
    if (item + step < end) {  // the next block's first residues, in flight during the products
      xb = source(item + step, left);
      fetch(xv[0], xb, left, 0);
    }
    // opaque multipliers of mad_i64 (the unit multipliers distinct per term of a sum)
    uint32_t one0 = 1, one1 = 1, one2 = 1, one3 = 1, m8 = 256, m16 = 65536, m24 = 16777216;
    opaque_s(one0);
    opaque_s(one1);
    opaque_s(one2);
    opaque_s(one3);
    opaque_s(m8);
    opaque_s(m16);
    opaque_s(m24);

    // phase 2, per tile of 8 limbs: the digit-plane products, recombination, carries.
    // Lane half h holds limbs l = 8 t + 4 h + i (i < 4) with C_ab = acc_a[4 b + i] (y plane
    // a, V plane b) and diagonal sums S_p = sum_(a+b=p) C_ab.  S_4..S_6 weigh 2^0..2^16 in
    // limb l + 1: inside the lane they join the next limb's sums, from the top limb they
    // leave with the carry.
    uint32_t* o = wave_uniform((z < a.first1 ? a.out + (long long)z * a.ostride
                                             : a.out1 + (long long)(z - a.first1) * a.ostride) + j0);
    uint32_t out_off = 4u * h * row + (2u * wave + (c >> 4)) * (row >> 4) + 4u * (c & 15);
    opaque(out_off);
    const int topbits = a.outbits - 32 * (a.Lout - 1);
    int64_t cin = 0;  // carry into the tile (used in lane half 0)
    v16i acc0, acc1, acc2, acc3;
    v4i Af[NKB];  // the next tile's fragments
    auto fragments = [&](int t) {
      const v4i* Ap = At + ((long long)t * NKB) * 64 + lane;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) Af[kb] = Ap[kb * 64];
    };
    auto products = [&]() {
      acc0 = v16i{};
      acc1 = v16i{};
      acc2 = v16i{};
      acc3 = v16i{};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af[kb], B[kb][0], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af[kb], B[kb][1], acc1, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af[kb], B[kb][2], acc2, 0, 0, 0);
        acc3 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af[kb], B[kb][3], acc3, 0, 0, 0);
      }
    };
    // tile sums: tt[i][p] = T_p of limb i (S_p plus S_(p+4) of limb i - 1), s4..s6 of limb 3
    int32_t tt[4][4], s4, s5, s6;
    auto sums = [&]() {
      s4 = s5 = s6 = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        tt[i][0] = acc0[i] + s4;
        tt[i][1] = acc0[4 + i] + acc1[i] + s5;
        tt[i][2] = acc0[8 + i] + acc1[4 + i] + acc2[i] + s6;
        tt[i][3] = acc0[12 + i] + acc1[8 + i] + acc2[4 + i] + acc3[i];
        s4 = acc1[12 + i] + acc2[8 + i] + acc3[4 + i];
        s5 = acc2[12 + i] + acc3[8 + i];
        s6 = acc3[12 + i];
      }
    };
    auto finish = [&](int t, bool last) {
      uint32_t ol[4];
      int64_t u = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int limb = 8 * t + 4 * h + i;
        // |T_p| <= 4 K 2^14 < 2^25, alpha < 3 K < 2^10: the limb value fits 64 bits with the constant and carry
        int64_t v = (int64_t)((uint64_t)alpha * s_mneg[limb] + s_eneg[limb]);
        v = mad_i64(tt[i][0], one0, v);
        v = mad_i64(tt[i][1], m8, v);
        v = mad_i64(tt[i][2], m16, v);
        v = mad_i64(tt[i][3], m24, v);
        if (i > 0) v = mad_i64((int32_t)(u >> 32), one1, v);
        u = v;
        ol[i] = (uint32_t)v;
      }
      int64_t carry = mad_i64(s4, one0, 0);
      carry = mad_i64(s5, m8, carry);
      carry = mad_i64(s6, m16, carry);
      carry = mad_i64((int32_t)(u >> 32), one1, carry);
      // carry across the lane halves: half 0 takes the carry into the tile, passes its
      // carry out to half 1, whose carry out enters the next tile
      carry = mad_i64(add_carry4(ol, h == 0 ? cin : 0), one2, carry);
      const int64_t mid = from_lane_below(carry);
      carry = mad_i64(add_carry4(ol, h == 1 ? mid : 0), one3, carry);
      cin = from_lane_above(carry);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int limb = 8 * t + 4 * h + i;
        uint32_t w = ol[i];
        if (last) {
          if (limb >= a.Lout) continue;
          if (limb == a.Lout - 1 && topbits < 32) w &= (1u << topbits) - 1u;
        }
        store_at(o, out_off + i * row, w);
      }
    };
    fragments(0);
    for (int t = 0; t < a.ntiles - 1; ++t) {
      products();
      sums();
      fragments(t + 1);  // on their way while this tile is finished
      finish(t, false);
      o += 8 * a.N;
    }
    products();
    sums();
    finish(a.ntiles - 1, true);
  }
}

template <int NKB, bool LDSA>
__global__ __launch_bounds__(512) void crt_cols_kernel(CrtArgs a) {
  crt_cols_kernel_body<NKB, LDSA>(a, own_blk());
}

// The same over the cells of a stage-batched plan: one launch, each workgroup in its
// cell's segment (cell_of) with that cell's arguments.
template <int NKB, bool LDSA>
__global__ __launch_bounds__(512) void crt_cols_kernel_multi(const CrtArgs* __restrict__ cells,
                                                             const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  crt_cols_kernel_body<NKB, LDSA>(cells[c], bk);
}

template <int NKB, bool LDSA>
static void crt_cols(const CrtArgs& a, hipStream_t st) {
  const size_t lds = crt_lds(NKB, crt_bufs<NKB>(), a.ntiles, LDSA);
  static bool attr = false;  // allow the full LDS of the device for this instantiation (once)
  if (!attr)
    attr = hipFuncSetAttribute((const void*)crt_cols_kernel<NKB, LDSA>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               a.lds_max) == hipSuccess;
  // persistent workgroups, a multiple of 8: two per compute unit where the LDS and the
  // registers (up to two k-blocks) hold them
  const int per_cu = NKB <= 2 && 2 * lds <= (size_t)a.lds_max ? 2 : 1;
  const int chunk = (a.npoly * (a.N >> 8) + 7) / 8;
  const unsigned grid = 8u * (unsigned)std::max(1, std::min(chunk, per_cu * a.cus / 8));
  (void)emit((const void*)crt_cols_kernel<NKB, LDSA>, (const void*)crt_cols_kernel_multi<NKB, LDSA>, dim3(grid),
             dim3(512), lds, st, a);
}

template <int NKB>
static hipError_t crt_cols_lds(const CrtArgs& a, hipStream_t st) {
  if (crt_lds(NKB, crt_bufs<NKB>(), a.ntiles, true) <= (size_t)a.lds_max) crt_cols<NKB, true>(a, st);
  else crt_cols<NKB, false>(a, st);
  return hipGetLastError();
}

hipError_t launch_crt_cols(CrtArgs a, int npoly, hipStream_t st) {
  a.npoly = npoly;
  if (npoly == 0) return hipSuccess;
  if (a.N < 1024) return hipErrorInvalidValue;
  // algorithmic HBM bytes: K residues read and Lout limbs written per coefficient
  Bracket br(KID_CRT, st, 4.0 * npoly * a.N * (double)(a.K + a.Lout));
  switch ((a.K + 31) / 32) {
    case 1: return crt_cols_lds<1>(a, st);
    case 2: return crt_cols_lds<2>(a, st);
    case 3: return crt_cols_lds<3>(a, st);
    case 4: return crt_cols_lds<4>(a, st);
    case 5: return crt_cols_lds<5>(a, st);
    case 6: return crt_cols_lds<6>(a, st);
    case 7: return crt_cols_lds<7>(a, st);
    case 8: return crt_cols_lds<8>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fhe
