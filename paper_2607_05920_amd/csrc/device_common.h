// Device helpers shared by the kernel files: opaque registers, buffer resources, lane
// exchanges, workgroup coordinates, twiddle tables and the lazy butterflies; and the
// host's launch helper.
#pragma once
#include <utility>
#include <vector>

#include "fhe_internal.h"

namespace fhe {

typedef v4i_t v4i;
typedef int v16i __attribute__((ext_vector_type(16)));

// Makes a register value opaque to the optimizer.  Uses here: multipliers that must
// stay 64-bit multiply-adds (not shifts and adds), values that must be computed where
// written (not re-derived later), and per-iteration offsets of persistent loops (not
// hoisted out of the loop, where each would hold a register).
__device__ __forceinline__ void opaque(uint32_t& v) { asm volatile("" : "+v"(v)); }

// The same for a value in a scalar register.
__device__ __forceinline__ void opaque_s(uint32_t& v) { asm volatile("" : "+s"(v)); }

// A pointer the caller knows to be equal on every lane of the wave, moved to scalar
// registers: buffer resources need it there, and stores through it take the scalar
// base + 32-bit lane offset form (no 64-bit address arithmetic per lane).
template <typename T>
__device__ __forceinline__ T* wave_uniform(T* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((uint64_t)hi << 32) | lo);
}

// Raw buffer over `bytes` bytes from the wave-uniform `base`.  Loads at lane offsets at
// or beyond `bytes` return zero (the buffer range check), which stands in for clamping
// and masking rows past the end of a polynomial.
// `bytes` is uniform too: it is moved to a scalar register, so that a value the compiler
// happened to compute in vector registers does not make the descriptor divergent (which
// would wrap every access in a loop over lanes).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const uint32_t* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)__builtin_amdgcn_readfirstlane(bytes),
                                           0x00020000);
}

__device__ __forceinline__ uint32_t buffer_word(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, (int)byte_off, 0, 0);
}

// Limb rows of one coefficient per lane.  Rows at or beyond the buffer's end read as zero.
struct LimbRows {
  __amdgpu_buffer_rsrc_t r;
  uint32_t lane, row;  // byte offset of the lane's coefficient, bytes between rows
  // rows l < `rows` of the polynomial at the wave-uniform `base`, N coefficients a row
  __device__ __forceinline__ LimbRows(const uint32_t* base, int rows, int N, uint32_t coeff)
      : r(row_buffer(wave_uniform(base), 4u * (uint32_t)rows * (uint32_t)N)), lane(4u * coeff), row(4u * (uint32_t)N) {}
  __device__ __forceinline__ uint32_t operator[](int l) const { return buffer_word(r, lane + (uint32_t)l * row); }
  template <int B>
  __device__ __forceinline__ void block(uint32_t (&v)[B], int l0) const {
#pragma unroll
    for (int i = 0; i < B; ++i) v[i] = (*this)[l0 + i];
  }
};

// A limb-serial kernel's rows first.. of x (and of y), `n` of them, B at a time: f(block of x,
// block of y, first row's number) in turn, with the next block already in flight.
//
// What bounds these kernels: with few waves the rows' latency, with many the memory's rate,
// which is highest while reads and stores go on side by side.  A load per limb inside the
// carry chain waits for memory limb by limb; large blocks read, then store, the whole chip
// in step; and a load after a block's stores waits for them too, as both are counted in
// order.  Small blocks, the next one asked for before this one is stored, do well at both
// ends.  us with a row at a time, with blocks of 16, with these (N = 2^16): automorphism of
// 49 limbs 14.1, 10.7, 7.4, of 4 x 49 21.7, 25.5, 21.3; rescaling 49 limbs 18.3, 12.2, 9.9,
// 8 x 49 89, 76, 76; BGV rescaling 8 x 14 19.4, 22.3, 18.4; sum of 8 x 14 26.3, 27.5, 25.9;
// composition at 1555 bits 33.0, 19.2, 17.7, of 4 53.7, 48.3, 46.9.
template <int B, typename F>
__device__ __forceinline__ void limb_blocks(const LimbRows& x, int xfirst, const LimbRows& y, int yfirst, int n, F f) {
  uint32_t x0[B], y0[B], x1[B], y1[B];
  x.block(x0, xfirst);
  y.block(y0, yfirst);
  for (int l = 0; l < n; l += 2 * B) {
    x.block(x1, xfirst + l + B);
    y.block(y1, yfirst + l + B);
    __builtin_amdgcn_sched_barrier(0);
    f(x0, y0, l);
    if (l + B >= n) break;
    x.block(x0, xfirst + l + 2 * B);
    y.block(y0, yfirst + l + 2 * B);
    __builtin_amdgcn_sched_barrier(0);
    f(x1, y1, l + B);
  }
}
template <int B, typename F>
__device__ __forceinline__ void limb_blocks(const LimbRows& x, int xfirst, int n, F f) {
  uint32_t x0[B], x1[B];
  x.block(x0, xfirst);
  for (int l = 0; l < n; l += 2 * B) {
    x.block(x1, xfirst + l + B);
    __builtin_amdgcn_sched_barrier(0);
    f(x0, l);
    if (l + B >= n) break;
    x.block(x0, xfirst + l + 2 * B);
    __builtin_amdgcn_sched_barrier(0);
    f(x1, l + B);
  }
}

// Global store at a byte offset from a wave-uniform base (the global address space is
// stated: the pointer's provenance is lost through the scalar move).
__device__ __forceinline__ void store_at(uint32_t* base, uint32_t byte_off, uint32_t v) {
  typedef __attribute__((address_space(1))) char gchar;
  typedef __attribute__((address_space(1))) uint32_t gu32;
  *(gu32*)((gchar*)base + byte_off) = v;
}

// a * b + c as one v_mad_i64_i32.  b must be opaque (a register the compiler cannot
// see the value of), or the product is strength-reduced into shifts and adds; and two
// terms of one sum must not share a multiplier register, or the compiler merges them
// into a 64 x 64-bit product.  (Not inline asm: a compiler-visible instruction gets
// the wait states after the matrix-core op that produced its operand.)
__device__ __forceinline__ int64_t mad_i64(int32_t a, uint32_t b, int64_t c) { return (int64_t)a * (int32_t)b + c; }

// Exchanges between the wave's lane halves with v_permlane32_swap (a vector op, no LDS
// round trip).  swap(x, x) returns {r0, r1}: r0 holds, in lanes 32..63, x of the lane 32
// below (lanes 0..31 keep theirs); r1 holds, in lanes 0..31, x of the lane 32 above.
__device__ __forceinline__ int64_t from_lane_below(int64_t x) {  // valid in lanes 32..63
  const uint32_t lo = (uint32_t)x, hi = (uint32_t)((uint64_t)x >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return (int64_t)(((uint64_t)u[0] << 32) | l[0]);
}
__device__ __forceinline__ int64_t from_lane_above(int64_t x) {  // valid in lanes 0..31
  const uint32_t lo = (uint32_t)x, hi = (uint32_t)((uint64_t)x >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return (int64_t)(((uint64_t)u[1] << 32) | l[1]);
}
// x plus x of the lane 32 apart, in every lane
__device__ __forceinline__ uint64_t sum_lane_halves(uint64_t x) {
  const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto u = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return ((((uint64_t)u[0] << 32) | l[0])) + ((((uint64_t)u[1] << 32) | l[1]));
}

// o += cin over 4 limbs (unsigned words, least significant first), cin signed 64-bit:
// one add-with-carry chain over (cin_lo, cin_hi, ext, ext), ext the sign extension.
// Returns the signed carry out of the top limb, in {-1, 0, 1}.
__device__ __forceinline__ int32_t add_carry4(uint32_t (&o)[4], int64_t cin) {
  const uint32_t lo = (uint32_t)cin, hi = (uint32_t)((uint64_t)cin >> 32);
  const uint32_t ext = (uint32_t)((int32_t)hi >> 31);
  uint32_t co;
  asm("v_add_co_u32 %0, vcc, %0, %5\n\t"
      "v_addc_co_u32 %1, vcc, %1, %6, vcc\n\t"
      "v_addc_co_u32 %2, vcc, %2, %7, vcc\n\t"
      "v_addc_co_u32 %3, vcc, %3, %7, vcc\n\t"
      "v_addc_co_u32 %4, vcc, 0, %7, vcc"
      : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]), "=&v"(co)
      : "v"(lo), "v"(hi), "v"(ext)
      : "vcc");
  return (int32_t)co;
}

// Workgroup coordinates within one launch's grid.  A kernel body takes them as an
// argument, so that it runs either as its own launch (own_blk) or as one cell's
// segment of a stage-batched launch over many cells (cell_of).
struct Blk {
  uint32_t x, y, nx;  // block index (x, y) and the grid's width in x
};

__device__ __forceinline__ Blk own_blk() { return Blk{blockIdx.x, blockIdx.y, gridDim.x}; }

// The cell that workgroup blockIdx.x of a stage-batched launch belongs to: seg[c].off
// (ascending, multiples of 8, so that a workgroup's XCD, blockIdx.x mod 8, is the one
// its own launch would give it) is the first workgroup of cell c, whose own grid is
// gx x gy.  Workgroups past a cell's grid (the rounding to 8) take -1 and exit.
__device__ __forceinline__ int cell_of(const CellSeg* seg, int ncells, Blk& bk) {
  const uint32_t w = blockIdx.x;
  int lo = 0, hi = ncells;  // the last cell with off <= w
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (seg[mid].off <= w) lo = mid;
    else hi = mid;
  }
  const CellSeg sg = seg[lo];
  const uint32_t l = w - sg.off;
  if (l >= sg.gx * sg.gy) return -1;
  bk = Blk{l % sg.gx, l / sg.gx, sg.gx};
  return lo;
}

// A pointer read from memory (a stage-batched launch's table of cell arguments) is
// generic to the compiler, and its loads become flat loads into vector registers even
// where the address is wave-uniform.  Held as a global-memory pointer, its loads are
// global ones, or scalar ones where uniform, as in a single launch.
template <typename T>
using gptr = const __attribute__((address_space(1))) T*;

// One prime's twiddle table (32-bit words, Montgomery form) through such a pointer.
struct TwTab {
  gptr<uint32_t> p;
  __device__ __forceinline__ uint32_t operator[](int i) const { return p[i]; }
  // CNT consecutive entries from i (a multiple of CNT, a power of two) in loads of up to 16
  // bytes
  template <int CNT>
  __device__ __forceinline__ void run(int i, uint32_t* w) const {
    if (CNT == 1) {
      w[0] = p[i];
    } else if (CNT == 2) {
      const uint64_t v = *(gptr<uint64_t>)(p + i);
      w[0] = (uint32_t)v;
      w[1] = (uint32_t)(v >> 32);
    } else {
#pragma unroll
      for (int e = 0; e < CNT; e += 4) {
        const v4i_t v = *(gptr<v4i_t>)(p + i + e);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[e + k] = (uint32_t)v[k];
      }
    }
  }
};
__device__ __forceinline__ TwTab tw_table(const uint32_t* t, int p) {
  return TwTab{(gptr<uint32_t>)t + (long long)p * kNMax};
}

// A prime as the butterflies use it: the same for the whole wave, or (second form) one per
// lane.  neg2q is -2q, opaque, so that adding it stays one operation of a three-input add.
struct Mod {
  uint32_t q, two_q, qneg, neg2q;
  __device__ __forceinline__ explicit Mod(const PrimeC& c)
      : q(__builtin_amdgcn_readfirstlane(c.q)), two_q(2 * q), qneg(__builtin_amdgcn_readfirstlane(c.qneg)),
        neg2q(0u - 2 * q) {
    asm("" : "+s"(neg2q));
  }
  __device__ __forceinline__ Mod(uint32_t q_, uint32_t qneg_) : q(q_), two_q(2 * q_), qneg(qneg_), neg2q(0u - 2 * q_) {
    asm("" : "+v"(neg2q));
  }
};

// Signed Montgomery product: y w 2^-32 mod q in (0, 2q) for |y| < 2q and w in [0, q).
// T = y w + q 2^32 lies within 2 q^2 of q 2^32, and m q, m the signed word that clears T's
// low half, within q 2^31 of 0; with 2 q^2 < q 2^31 (q < 2^30) the high word of T + m q is
// in (0, 2q).  Three operations, a four-byte twiddle, and y may be a plain difference.
__device__ __forceinline__ uint32_t mont_s(uint32_t y, uint32_t w, const Mod& M) {
  int64_t T = (int64_t)(int32_t)y * (int32_t)w + (int64_t)((uint64_t)M.q << 32);
  asm("" : "+v"(T));  // its low half as it is (the compiler would multiply again for it)
  const uint32_t m = (uint32_t)T * M.qneg;
  return (uint32_t)((uint64_t)((int64_t)(int32_t)m * (int32_t)M.q + T) >> 32);
}

// Lazy Cooley-Tukey butterfly.  Forward values are held less 2q: words in [-2q, 2q), two's
// complement, which the product takes as they are; with t = Y w in (0, 2q) and x = X or
// X + 2q in [0, 2q) (an unsigned minimum), X + t - 2q and x - t are in [-2q, 2q) again:
// 7 operations.  FIRST: X is in [0, 2q) already (the transform's first stage).
template <bool FIRST = false>
__device__ __forceinline__ void ct_bfly(uint32_t& X, uint32_t& Y, uint32_t w, const Mod& M) {
  const uint32_t x = FIRST ? X : min(X, X + M.two_q);
  const uint32_t t = mont_s(Y, w, M);
  X = x + t + M.neg2q;
  Y = x - t;
}
// A forward value in [-2q, 2q) to [0, 2q).
__device__ __forceinline__ uint32_t fwd_lift(uint32_t X, const Mod& M) { return min(X, X + M.two_q); }

// Lazy Gentleman-Sande butterfly: X, Y in [0, 2q) -> [0, 2q); 7 operations.
__device__ __forceinline__ void gs_bfly(uint32_t& X, uint32_t& Y, uint32_t w, const Mod& M) {
  const uint32_t x = X, y = Y;
  X = csub(x + y, M.two_q);
  Y = mont_s(x - y, w, M);
}

// The limbs of input polynomial z of a lift.
__device__ __forceinline__ const uint32_t* lift_source(const LiftArgs& a, uint32_t z) {
  if (a.interleave4) {
    const uint32_t i = z & 3u, c = z >> 2;
    return a.in_ptrs ? a.in_ptrs[i * (uint32_t)(a.npoly >> 2) + c] : a.in4[i] + (long long)c * a.in_stride;
  }
  if (a.in_ptrs) return a.in_ptrs[z];
  if ((int)z >= a.first2) return a.limbs2 + (long long)((int)z - a.first2) * a.in_stride;
  if ((int)z >= a.first1) return a.limbs1 + (long long)((int)z - a.first1) * a.in_stride;
  return a.limbs + (long long)z * a.in_stride;
}

// The first four stages of a transform on one column {c + (N / 16) u}, u < 16: forward
// stages of 1, 2, 4 and 8 groups (table entries 1..15), values in [0, 2q) to [-2q, 2q).
__device__ __forceinline__ void cols16_forward(uint32_t (&x)[16], TwTab tw, const Mod& M) {
#pragma unroll
  for (int m = 1; m <= 8; m *= 2) {
    const int h = 8 / m;
#pragma unroll
    for (int g = 0; g < m; ++g) {
      const uint32_t w = tw[m + g];
#pragma unroll
      for (int u = 2 * h * g; u < 2 * h * g + h; ++u) {
        if (m == 1) ct_bfly<true>(x[u], x[u + h], w, M);
        else ct_bfly(x[u], x[u + h], w, M);
      }
    }
  }
}

// Every LDS exchange of the row passes stays inside one T-thread slot, and a slot
// (T <= 16 threads) never straddles two waves: a wave-level ordering point is enough
// between the writes and the reads (a wave's LDS accesses are performed in order), so
// the two waves of a workgroup never wait for each other.
__device__ __forceinline__ void slot_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Issues a launch of `single` (one struct argument), or records it with its
// stage-batched entry point `multi` while a sink is installed.
template <typename A>
inline hipError_t emit(const void* single, const void* multi, dim3 grid, dim3 block, size_t lds, hipStream_t st,
                       const A& a) {
  if (LaunchSink* sink = launch_sink()) {
    LaunchRec r;
    r.multi = multi;
    r.grid = grid;
    r.block = block;
    r.lds = lds;
    r.args.assign((const char*)&a, (const char*)&a + sizeof(A));
    sink->recs.push_back(std::move(r));
    return hipSuccess;
  }
  void* args[] = {(void*)&a};
  return hipLaunchKernel(single, grid, block, args, lds, st);
}

}  // namespace fhe
