// The lift (limbs -> residues) with the first four forward transform stages: a workgroup
// takes 64 columns {c + (N / 16) u} of a polynomial, so that the residues it makes on the
// matrix cores go through their 16-point stages before they are stored, and no separate
// pass reads and writes them.
#include <algorithm>

#include "device_common.h"

namespace fhe {

// The digit planes, tables and reduction are those of lift_mfma_kernel (kernels.hip); here
// wave u of 16 holds row u of the block (its 64 columns are two units of 32 coefficients,
// whose limbs stay in registers for every prime), and the workgroup goes through the
// primes 16 at a time:
//   products   each wave: two tiles of 8 primes, both units per table fragment
//   exchange   residues to LDS as [prime][row][column], one barrier
//   stages     wave w: the 64 columns of prime w of the step, one per lane; its twiddles
//              are wave-uniform (scalar loads); 256-byte runs out
// The LDS holds two exchange buffers and two steps' table fragments: one barrier per step,
// the stages a step behind the products.
//
// What bounds it: instruction issue (the VALU about 75% busy between the barriers, the
// matrix instructions beside it) and, in the first quarter of a block, its limbs' loads.  At
// 16 waves of 128 registers the limbs, accumulators and a fragment just fit up to 7 k-blocks
// (56 limbs); larger ones take the separate lift and column pass.  2^16 coefficients, 49
// limbs, 106 primes, 16 polynomials: 221 us; the separate lift and column pass of eight
// stages took 146 and 161 (the other four stages are in the middle pass now, which went from
// 256 to 323).
template <int NKB>
__device__ __forceinline__ void lift_cols_kernel_body(const LiftArgs& a, const Blk bk) {
  constexpr int XS = 16 * 64 + 8;  // words per prime: the lane halves' stores fall on different banks
  __shared__ uint32_t sx[2][16 * XS];
  __shared__ v4i sa[2][2 * NKB * 64];
  __shared__ uint4 sc[2][16];
  const uint32_t tid = threadIdx.x, lane = tid & 63, c = lane & 31, h = lane >> 5;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Workgroup w runs on XCD w % 8: the a.nsplit workgroups that share a block (each takes
  // its own primes) run on one XCD, whose L2 then holds the block's limbs.
  const int nblk = a.N >> 10, units = a.npoly * nblk;
  const int l = bk.x >> 3, unit = (l / a.nsplit) * 8 + (int)(bk.x & 7), split = l % a.nsplit;
  if (unit >= units) return;  // whole workgroup exits
  const int steps = (a.K + 15) / 16, per = (steps + a.nsplit - 1) / a.nsplit;
  const int s0 = split * per, s1 = min(s0 + per, steps);
  if (s0 >= s1) return;
  const uint32_t z = (uint32_t)(unit / nblk);
  const uint32_t j0 = wave * ((uint32_t)a.N >> 4) + 64u * (uint32_t)(unit % nblk);  // this wave's first coefficient
  const uint32_t row = 4u * (uint32_t)a.N;  // bytes between limb (or residue) rows

  auto fetch = [&](int s) {  // this thread's share of a step's fragments
    const uint32_t at = (uint32_t)(2 * s * NKB * 64) + tid;
    return tid < 2 * NKB * 64 && at < (uint32_t)(a.ntiles * NKB * 64) ? a.A[at] : v4i{};
  };
  auto constants = [&](int s) {
    const int p = min(16 * s + (int)(tid & 15), a.K - 1);
    const uint64_t o = a.off[p];
    return make_uint4(a.pc[p].q, a.pc[p].qneg, (uint32_t)o, (uint32_t)(o >> 32));
  };

  // limbs 8 kb + 4 h + r; rows at or beyond L read as zero, where the table is zero too
  const uint32_t* src = wave_uniform(lift_source(a, z) + j0);
  const __amdgpu_buffer_rsrc_t rs = row_buffer(src, 4u * ((uint32_t)a.L * (uint32_t)a.N - j0));
  const uint32_t in_off = 4u * h * row + 4u * c;
  v4i B[2][NKB];
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int v = 0; v < 2; ++v) B[v][kb][r] = (int)buffer_word(rs, in_off + (8 * kb + r) * row + 128u * v);
  {
    const v4i f = fetch(s0);
    if (tid < 2 * NKB * 64) sa[s0 & 1][tid] = f;
    if (tid < 16) sc[s0 & 1][tid] = constants(s0);
  }
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int v = 0; v < 2; ++v) B[v][kb][r] ^= (int)0x80808080u;
  __syncthreads();
  uint32_t one = 1, m8 = 256, m16 = 65536, m24 = 16777216;  // opaque multipliers of mad_i64
  opaque_s(one);
  opaque_s(m8);
  opaque_s(m16);
  opaque_s(m24);
  uint32_t* const out = a.res + (long long)z * a.out_stride + (j0 - wave * ((uint32_t)a.N >> 4));

  // the products of step s: residues of its 16 primes in [0, 2q) to the step's buffer
  auto products = [&](int s) {
    uint32_t* const xw = sx[s & 1] + 4 * h * XS + wave * 64 + c;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (2 * s + g >= a.ntiles) break;
      v16i acc0 = {}, acc1 = {};
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const v4i Af = sa[s & 1][(g * NKB + kb) * 64 + lane];
        acc0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af, B[0][kb], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(Af, B[1][kb], acc1, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint4 k = sc[s & 1][8 * g + 4 * h + i];
        const int64_t o = (int64_t)(((uint64_t)k.w << 32) | k.z);
        int64_t v = mad_i64(acc0[i], one, o);
        v = mad_i64(acc0[4 + i], m8, v);
        v = mad_i64(acc0[8 + i], m16, v);
        v = mad_i64(acc0[12 + i], m24, v);
        xw[(8 * g + i) * XS] = redc_lazy((uint64_t)v, k.x, k.y);
        v = mad_i64(acc1[i], one, o);
        v = mad_i64(acc1[4 + i], m8, v);
        v = mad_i64(acc1[8 + i], m16, v);
        v = mad_i64(acc1[12 + i], m24, v);
        xw[(8 * g + i) * XS + 32] = redc_lazy((uint64_t)v, k.x, k.y);
      }
    }
  };
  // the stages of step s: this wave's prime, one column per lane
  auto stages = [&](int s) {
    const int p = 16 * s + (int)wave;
    if (p >= a.K) return;
    uint32_t x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = sx[s & 1][wave * XS + u * 64 + lane];
    cols16_forward(x, tw_table(a.tw, p), Mod(a.pc[p]));
    const __amdgpu_buffer_rsrc_t ro = row_buffer(wave_uniform(out + (long long)p * a.N), row);
#pragma unroll
    for (int u = 0; u < 16; ++u)
      __builtin_amdgcn_raw_buffer_store_b32(x[u], ro, (int)(4u * lane), (int)(u * (row >> 4)), 0);
  };
  // Between two barriers a wave has the products of step s and the stages of step s - 1 to
  // do, in either order: half the waves of each SIMD take the products first and half the
  // stages, so that the matrix cores and the VALU work side by side.
  const int first = (int)(wave >> 3);
  for (int s = s0; s <= s1; ++s) {
    v4i f = {};
    if (s + 1 < s1) f = fetch(s + 1);
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
      if (k == first) {
        if (s < s1) products(s);
      } else {
        if (s > s0) stages(s - 1);
      }
    }
    if (s + 1 < s1) {
      if (tid < 2 * NKB * 64) sa[(s + 1) & 1][tid] = f;
      if (tid < 16) sc[(s + 1) & 1][tid] = constants(s + 1);
    }
    __syncthreads();
  }
}

template <int NKB>
__global__ __launch_bounds__(1024) void lift_cols_kernel(LiftArgs a) {
  lift_cols_kernel_body<NKB>(a, own_blk());
}

// The same over the cells of a stage-batched plan: one launch, each workgroup in its
// cell's segment (cell_of) with that cell's arguments.
template <int NKB>
__global__ __launch_bounds__(1024) void lift_cols_kernel_multi(const LiftArgs* __restrict__ cells,
                                                               const CellSeg* __restrict__ seg, int ncells) {
  Blk bk;
  const int c = cell_of(seg, ncells, bk);
  if (c < 0) return;
  lift_cols_kernel_body<NKB>(cells[c], bk);
}

template <int NKB>
static hipError_t lift_cols(const LiftArgs& b, hipStream_t st) {
  const int units = b.npoly * (b.N >> 10);
  (void)emit((const void*)lift_cols_kernel<NKB>, (const void*)lift_cols_kernel_multi<NKB>,
             dim3(8 * ((units + 7) / 8) * b.nsplit), dim3(1024), 0, st, b);
  if (LaunchSink* sink = launch_sink()) sink->recs.emplace_back();  // the place of the separate column pass
  return hipGetLastError();
}

hipError_t launch_lift_cols(const LiftArgs& a, int npoly, hipStream_t st, const Tuning& t) {
  if (npoly <= 0) return hipSuccess;
  if (t.lift_primes != 0 || !a.A || a.nkb > 7 || a.N < 1024) {  // the two passes on their own
    hipError_t e = launch_lift(a, npoly, st, t);
    NttArgs n{};
    n.data = a.res;
    n.logN = __builtin_ctz((unsigned)a.N);
    n.K = n.per_group = a.K;
    n.group_stride = a.out_stride;
    n.tw = a.tw;
    n.pc = a.pc;
    return e != hipSuccess ? e : launch_cols16(n, npoly * a.K, st);
  }
  LiftArgs b = a;
  b.npoly = npoly;
  // Few blocks: their primes are shared out over workgroups (each reads the block's limbs)
  // until there is one for each compute unit.
  const int units = npoly * (a.N >> 10), steps = (a.K + 15) / 16;
  b.nsplit = std::max(1, std::min(steps, a.cus / std::max(units, 1)));
  // algorithmic HBM bytes: L limbs read and K residues written per coefficient
  Bracket br(KID_LIFT, st, 4.0 * npoly * a.N * (double)(a.L + a.K));
  switch (b.nkb) {
    case 1: return lift_cols<1>(b, st);
    case 2: return lift_cols<2>(b, st);
    case 3: return lift_cols<3>(b, st);
    case 4: return lift_cols<4>(b, st);
    case 5: return lift_cols<5>(b, st);
    case 6: return lift_cols<6>(b, st);
    case 7: return lift_cols<7>(b, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fhe
