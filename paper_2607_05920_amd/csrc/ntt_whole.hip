// Standalone negacyclic transforms in one pass over memory: a workgroup holds a whole
// transform in registers (2^V values per thread) and exchanges through LDS, so each
// residue is read once and written once, and the natural order costs one more LDS
// exchange instead of a permutation pass over memory.  The same butterfly network, tables
// and results as the two-pass transforms of kernels.hip.
#include "device_common.h"

namespace fhe {

// A transform of 2^LG points runs in phases of up to V stages.  Phase I works on blocks of
// B elements (B = 2^LG after the stages before it), each cut into B / G sub-columns of
// G = 2^stages elements a distance B / G apart; a thread holds R / G sub-columns (R = 2^V).
// Sub-column k of thread t is numbered so that after the first exchange every exchange
// stays inside a wave: waves hold contiguous elements (LG < 16), or, for 2^16 points, the
// same 2 x 2048 elements (one run in each half of the transform).
//
// What bounds it: 2^13 and 2^14 points move 2.4-3.7 TB/s (read + write) with two or more
// workgroups per compute unit, VALU issue and the exchanges together.  2^16 points fill one
// compute unit (1024 threads x 64 values; the LDS takes half a transform at a time, so an
// exchange runs in two rounds): about 26 us of VALU issue of 46 a transform, and loads and
// stores that nothing overlaps.
template <int LG, int V>
struct Whole {
  static constexpr int R = 1 << V, T = 1 << (LG - V);
  static constexpr int NPH = V == 6 ? 3 : (LG + V - 1) / V;
  static constexpr int HALVES = V == 6 ? 2 : 1;  // exchange rounds: the LDS holds 2^LG / HALVES values
  static constexpr int RH = R / HALVES;            // registers per round
  static constexpr int LDS_WORDS = ((1 << LG) / HALVES) + ((1 << LG) / HALVES >> V);

  static constexpr int before(int I) { return V == 6 ? (I == 0 ? 0 : 1 + 5 * I) : V * I; }
  static constexpr int stages(int I) { return (I + 1 < NPH ? before(I + 1) : LG) - before(I); }
  static constexpr int B(int I) { return 1 << (LG - before(I)); }
  static constexpr int G(int I) { return 1 << stages(I); }

  // LDS position of element e of a round, free of bank conflicts for runs of lanes and for
  // lanes R elements apart.  Positions (and reversed indices) of values with disjoint bits
  // add, so an element's is the thread's plus a constant of the register.
  static constexpr __device__ __forceinline__ int pad(int e) { return e + (e >> V); }
  static constexpr __device__ __forceinline__ int rev(int e) {
    int r = 0;
    for (int b = 0; b < LG; ++b) r |= ((e >> b) & 1) << (LG - 1 - b);
    return r;
  }

  template <int I>
  static constexpr __device__ __forceinline__ int subcol(int k, int t) {
    constexpr int W = T < 64 ? T : 64, KG = R / G(I);
    if (KG == 1) return t;
    constexpr int KH = KG / HALVES;  // per half
    return (k / KH) * (T * KH) + (t / W) * (W * KH) + (k % KH) * W + t % W;
  }
  template <int I>
  static constexpr __device__ __forceinline__ int elem(int r, int t) {  // register r = k G + u
    constexpr int C = B(I) / G(I);
    const int w = subcol<I>(r / G(I), t);
    return (w / C) * B(I) + (r % G(I)) * C + w % C;
  }
  // LDS position of register r of its round: thread part (base<I>(t)) + constant part
  template <int I>
  static __device__ __forceinline__ int base(int t) { return pad(elem<I>(0, t)); }
  template <int I>
  static constexpr __device__ __forceinline__ int offset(int r) {
    return pad(elem<I>(r, 0) - (r / RH) * ((1 << LG) / HALVES));
  }

  // orders the writes of an exchange between phases I and I + 1 before its reads
  template <int I>
  static __device__ __forceinline__ void sync() {
    if (I == 0 && T > 64) __syncthreads();
    else slot_sync();
  }

  template <int I, int J>
  static __device__ __forceinline__ void exchange(uint32_t (&x)[R], uint32_t* lds, int t) {
    uint32_t* const lw = lds + base<I>(t);
    uint32_t* const lr = lds + base<J>(t);
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
      if (h > 0) sync<(I < J ? I : J)>();  // the previous round has been read
#pragma unroll
      for (int r = h * RH; r < (h + 1) * RH; ++r) lw[offset<I>(r)] = x[r];
      sync<(I < J ? I : J)>();
#pragma unroll
      for (int r = h * RH; r < (h + 1) * RH; ++r) x[r] = lr[offset<J>(r)];
    }
  }

  // Table index of the first group of sub-column k's block: stage j's group g is at
  // (index << j) + g.
  template <int I>
  static __device__ __forceinline__ int tw_base(int k, int t) {
    constexpr int C = B(I) / G(I);
    const int b = (1 << before(I)) + subcol<I>(k, t) / C;
    return C >= 64 ? __builtin_amdgcn_readfirstlane(b) : b;  // one block per wave: scalar loads
  }

  template <int I>
  static __device__ __forceinline__ void forward(uint32_t (&x)[R], TwTab tw, int t, const Mod& M) {
    constexpr int g_ = G(I);
#pragma unroll
    for (int k = 0; k < R / g_; ++k) {
      const int b = tw_base<I>(k, t);
#pragma unroll
      for (int j = 0; j < stages(I); ++j) {
        const int h = g_ >> (j + 1);
        if (V == 6) __builtin_amdgcn_sched_barrier(0);  // later stages' twiddles loaded this early would spill
#pragma unroll
        for (int g = 0; g < (1 << j); ++g) {
          const uint32_t w = tw[(b << j) + g];
#pragma unroll
          for (int u = 2 * h * g; u < 2 * h * g + h; ++u) {
            if (I == 0 && j == 0) ct_bfly<true>(x[k * g_ + u], x[k * g_ + u + h], w, M);
            else ct_bfly(x[k * g_ + u], x[k * g_ + u + h], w, M);
          }
        }
      }
    }
  }

  // FOLD: leave the last stage (one group over the whole transform) to the caller
  template <int I, bool FOLD>
  static __device__ __forceinline__ void inverse(uint32_t (&x)[R], TwTab tw, int t, const Mod& M) {
    constexpr int g_ = G(I);
#pragma unroll
    for (int k = 0; k < R / g_; ++k) {
      const int b = tw_base<I>(k, t);
#pragma unroll
      for (int j = stages(I) - 1; j >= (FOLD ? 1 : 0); --j) {
        const int h = g_ >> (j + 1);
        if (V == 6) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < (1 << j); ++g) {
          const uint32_t w = tw[(b << j) + g];
#pragma unroll
          for (int u = 2 * h * g; u < 2 * h * g + h; ++u) gs_bfly(x[k * g_ + u], x[k * g_ + u + h], w, M);
        }
      }
    }
  }

  // Loads or stores the registers in the transform's own (bit-reversed) order from or to
  // phase NPH - 1: sub-columns are contiguous runs of G elements.
  template <bool STORE>
  static __device__ __forceinline__ void runs(uint32_t (&x)[R], __amdgpu_buffer_rsrc_t rb, int t) {
    constexpr int I = NPH - 1, g_ = G(I);
    static_assert(B(I) == g_, "the last phase's sub-columns are contiguous");
#pragma unroll
    for (int k = 0; k < R / g_; ++k) {
      const int o = 4 * g_ * subcol<I>(k, t);
      if (g_ >= 4) {
#pragma unroll
        for (int v = 0; v < g_ / 4; ++v) {
          uint32_t* y = x + k * g_ + 4 * v;
          if (STORE) {
            __builtin_amdgcn_raw_buffer_store_b128(v4i_t{(int)y[0], (int)y[1], (int)y[2], (int)y[3]}, rb, o, 16 * v, 0);
          } else {
            const v4i_t w = __builtin_amdgcn_raw_buffer_load_b128(rb, o, 16 * v, 0);
            y[0] = (uint32_t)w[0];
            y[1] = (uint32_t)w[1];
            y[2] = (uint32_t)w[2];
            y[3] = (uint32_t)w[3];
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < g_; ++u) {
          if (STORE) __builtin_amdgcn_raw_buffer_store_b32(x[k * g_ + u], rb, o, 4 * u, 0);
          else x[k * g_ + u] = __builtin_amdgcn_raw_buffer_load_b32(rb, o, 4 * u, 0);
        }
      }
    }
  }

  // Through LDS, so that memory sees runs of lanes: natural order (NAT) at the reversed
  // positions, where a round holds one half of the natural order, i.e. the elements of one
  // parity; or the transform's own order, where a round holds the registers of one half.
  // The own order takes it where a thread's runs of 32 elements would go out 16 bytes a lane
  // (2^16, 106 x 64: 1413 -> 1216 us; 2^15 forward, 106 x 16: 151 -> 137; its inverse, which
  // loads whole lines either way, 147 without it).
  template <bool STORE, bool NAT>
  static __device__ __forceinline__ void through(uint32_t (&x)[R], uint32_t* lds, __amdgpu_buffer_rsrc_t rb, int t) {
    constexpr int I = NPH - 1, half = (1 << LG) / HALVES;
    static_assert(HALVES == 1 || G(I) % 2 == 0, "an element's parity is its register's");
    static_assert(NAT || R / G(I) == HALVES, "a thread's runs are one per round");
    uint32_t* const ln = lds + pad(t);
    uint32_t* const lv = lds + pad(NAT ? (int)(__brev((unsigned)elem<I>(0, t)) >> (32 - LG)) : elem<I>(0, t));
    auto in = [](int r, int h) { return HALVES == 1 || (NAT ? r % 2 : r / RH) == h; };
    auto at = [](int r, int h) { return pad((NAT ? rev(elem<I>(r, 0)) : elem<I>(r, 0)) - h * half); };
#pragma unroll
    for (int h = 0; h < HALVES; ++h) {
      if (STORE || h > 0) __syncthreads();  // the LDS's previous contents have been read
      if (STORE) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (in(r, h)) lv[at(r, h)] = x[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RH; ++r)
          __builtin_amdgcn_raw_buffer_store_b32(ln[pad(r * T)], rb, 4 * t, 4 * (h * half + r * T), 0);
      } else {
        uint32_t y[RH];
#pragma unroll
        for (int r = 0; r < RH; ++r) y[r] = __builtin_amdgcn_raw_buffer_load_b32(rb, 4 * t, 4 * (h * half + r * T), 0);
#pragma unroll
        for (int r = 0; r < RH; ++r) ln[pad(r * T)] = y[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (in(r, h)) x[r] = lv[at(r, h)];
      }
    }
    if (!STORE) __syncthreads();
  }

  template <int I>
  static __device__ __forceinline__ void forward_from(uint32_t (&x)[R], uint32_t* lds, TwTab tw, int t, const Mod& M) {
    forward<I>(x, tw, t, M);
    if constexpr (I + 1 < NPH) {
      exchange<I, I + 1>(x, lds, t);
      forward_from<I + 1>(x, lds, tw, t, M);
    }
  }
  template <int I>
  static __device__ __forceinline__ void inverse_from(uint32_t (&x)[R], uint32_t* lds, TwTab tw, int t, const Mod& M) {
    inverse<I, I == 0>(x, tw, t, M);
    if constexpr (I > 0) {
      exchange<I, I - 1>(x, lds, t);
      inverse_from<I - 1>(x, lds, tw, t, M);
    }
  }
};

// Workgroup w runs on XCD w % 8 (round-robin dispatch).  The transforms, ordered by prime,
// are cut into eight runs of equal length, one per XCD: a prime's twiddle table is read
// into one L2 (two at a run's end), and the XCDs finish together whatever K is.
// (Persistent workgroups, whose waves load the next transform as soon as they have stored
// this one, measured 0-20% slower.)
template <int LG, int V, bool INV, bool NAT>
__global__ __launch_bounds__((Whole<LG, V>::T)) void ntt_whole_kernel(NttArgs a) {
  typedef Whole<LG, V> W;
  __shared__ uint32_t lds[W::LDS_WORDS];
  const int t = threadIdx.x;
  const int chunk = (a.ntr + 7) / 8;
  const int l = blockIdx.x >> 3, item = (blockIdx.x & 7) * chunk + l;
  if (l >= chunk || item >= a.ntr) return;  // whole workgroup exits
  const int npp = a.ntr / a.K;              // transforms per prime
  const int p = item / npp, jg = item % npp;
  const int pk = a.per_group / a.K;  // polynomials per group
  const long long row = (long long)(jg / pk) * a.group_stride + ((long long)(jg % pk) * a.K + p) * (1 << LG);
  const __amdgpu_buffer_rsrc_t rb = row_buffer(wave_uniform(a.data + row), 4u << LG);
  const Mod M(a.pc[p]);
  const uint32_t q = M.q;
  const TwTab tw = tw_table(a.tw, p);
  uint32_t x[W::R];
  if (!INV) {
#pragma unroll
    for (int r = 0; r < W::R; ++r) x[r] = __builtin_amdgcn_raw_buffer_load_b32(rb, 4 * t, 4 * r * W::T, 0);
    W::template forward_from<0>(x, lds, tw, t, M);
#pragma unroll
    for (int r = 0; r < W::R; ++r) x[r] = csub(fwd_lift(x[r], M), q);
    if constexpr (NAT || V >= 5) W::template through<true, NAT>(x, lds, rb, t);
    else W::template runs<true>(x, rb, t);
  } else {
    if constexpr (NAT || V == 6) W::template through<false, NAT>(x, lds, rb, t);
    else W::template runs<false>(x, rb, t);
    W::template inverse_from<W::NPH - 1>(x, lds, tw, t, M);
    // the last stage with the final factor folded in, as in the two-pass form
    const uint32_t sc = a.scale[p], sw = a.scale_w[p];
#pragma unroll
    for (int u = 0; u < W::R / 2; ++u) {
      const uint32_t xs = x[u], ys = x[u + W::R / 2];
      x[u] = csub(mont_s(xs + ys + M.neg2q, sc, M), q);
      x[u + W::R / 2] = csub(mont_s(xs - ys, sw, M), q);
    }
#pragma unroll
    for (int r = 0; r < W::R; ++r) __builtin_amdgcn_raw_buffer_store_b32(x[r], rb, 4 * t, 4 * r * W::T, 0);
  }
}

template <int LG, int V, bool INV, bool NAT>
static hipError_t ntt_whole(const NttArgs& a, hipStream_t st) {
  // algorithmic HBM bytes: every element of every transform read and written once
  Bracket br(INV ? KID_NTT_INV_COLS : KID_NTT_FWD_COLS, st, 8.0 * a.ntr * (double)(1 << LG));
  hipLaunchKernelGGL((ntt_whole_kernel<LG, V, INV, NAT>), dim3(8 * ((a.ntr + 7) / 8)), dim3(Whole<LG, V>::T), 0, st, a);
  return hipGetLastError();
}

template <int LG, int V>
static hipError_t ntt_whole_dir(const NttArgs& a, bool inverse, bool natural, hipStream_t st) {
  if (inverse) return natural ? ntt_whole<LG, V, true, true>(a, st) : ntt_whole<LG, V, true, false>(a, st);
  return natural ? ntt_whole<LG, V, false, true>(a, st) : ntt_whole<LG, V, false, false>(a, st);
}

// Where one workgroup per transform is the faster form (us, two passes [and the permutation]
// against one; N, primes x polynomials):
//   up to 2^14 always: 2^10, 106 x 64: 69 -> 16, natural order 108 -> 16; 2^13, 31 x 16:
//   20.7 -> 13.0, natural 77 -> 13; 2^14, 9 x 1: 10.6 -> 9.4, 106 x 64: 452 -> 243.
//   2^15: a transform takes 18 us on its one compute unit, so few of them are faster in two
//   passes over many: 31 x 2: 14.7 against 18.8, 31 x 4: 21.1 against 20.5 (inverse 18.6
//   against 19.8), 31 x 6: 27.9 against 21.0.  So from five transforms per eight compute
//   units on; with the second round's first transforms it gains less, but no more turns it:
//   11 x 24 (1.03 rounds) 42.0 -> 38.4, inverse 41.1 -> 37.0, 13 x 40 (2.03) 65.9 -> 58.9,
//   63.3 -> 58.1, 33 x 32 (4.1) 119 -> 96, 113 -> 99.  Natural order adds a permutation pass
//   to the two: 5 x 1: 14 against 19, 4 x 8: 26.4 -> 18.3, 31 x 4: 52 -> 20; from one per
//   eight units on.
//   2^16: 46 us a round of one transform per compute unit, against 50 of two passes (54
//   beyond the last-level cache): faster where the last round is nearly full or one of
//   many: 31 x 8: 54.1 -> 50.1, 32 x 12 (1.5 rounds): 76.8 against 88.6, 32 x 16: 96.8 ->
//   93.4, 53 x 16 (3.3 rounds): 153 against 172, 106 x 16 (6.6): 350 -> 340, 106 x 64: 1474
//   -> 1216.  Natural order: 31 x 4: 92 -> 41, 106 x 64: 6798 -> 1233; 5 x 1: 17 against 42;
//   4 x 16: 66 -> 39; from one per four units on.
bool ntt_whole_wanted(int logN, bool natural, long long ntransforms, int cus) {
  if (logN <= 14) return true;
  if (logN == 15) return 8 * ntransforms >= (natural ? 1 : 5) * (long long)cus;
  if (natural) return 4 * ntransforms >= cus;
  const long long slots = (ntransforms + cus - 1) / cus * cus;  // at most one in 16 idle, or 8 full rounds
  return ntransforms > 8LL * cus || 15 * slots <= 16 * ntransforms;
}

hipError_t launch_ntt_whole(const NttArgs& a0, int ntr, bool inverse, bool natural, hipStream_t st) {
  if (ntr <= 0) return hipSuccess;
  if (ntr % a0.K != 0 || a0.per_group % a0.K != 0 || (inverse && (!a0.scale || !a0.scale_w)))
    return hipErrorInvalidValue;
  NttArgs a = a0;
  a.ntr = ntr;
  switch (a.logN) {
    case 10: return ntt_whole_dir<10, 4>(a, inverse, natural, st);
    case 11: return ntt_whole_dir<11, 4>(a, inverse, natural, st);
    case 12: return ntt_whole_dir<12, 4>(a, inverse, natural, st);
    case 13: return ntt_whole_dir<13, 4>(a, inverse, natural, st);
    case 14: return ntt_whole_dir<14, 4>(a, inverse, natural, st);
    case 15: return ntt_whole_dir<15, 5>(a, inverse, natural, st);
    case 16:
      return ntt_whole_dir<16, 6>(a, inverse, natural, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fhe
