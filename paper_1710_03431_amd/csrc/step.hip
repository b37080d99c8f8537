// Persistent trajectory kernel: batched quantum-jump stepping in the
// instantaneous eigenbasis (Sec. IV waiting-time procedure; App. C validity;
// jump-type law App. B eq. Pi(t); jump update Sec. III eq. jump).
//
// One workgroup (WV = 4 or 8 wavefronts) owns a tile of TT = 8*TQ trajectories for the whole
// anneal; their amplitudes stay in LDS.  Per grid step g (from s_{g-1} to s_g):
//   1. C <- O_g C on MFMA, written as C + Delta_g C (identity split) so the
//      accumulator starts from C.  Real Delta times complex C is one real GEMM
//      on the re and im column tiles.
//   2. C' = d_g o C with d_b = exp(-i e_b dt - Gamma_b dt / 2): the no-jump
//      propagator of the diagonal H_eff (Sec. III eq. Heff), fused into the
//      GEMM epilogue together with the per-trajectory squared norm.
//   3. A trajectory whose squared norm falls to its threshold r crosses: a
//      wavefront takes it, finds the crossing time (Newton on the log of
//      sum_b |c_b|^2 e^{-Gamma_b tau}), draws the source level with weight
//      q_b Gamma_b and the (qubit, target) with weight R[i][b][a], applies the
//      jump, renormalises, records it and draws a new threshold; repeated
//      until the step's time is used up.  FP64 arithmetic in every mode.
//   4. Ground-cluster population per trajectory; per-tile sums go to a
//      [tile][g] buffer reduced afterwards in a fixed order.
// Phases of the whole step are applied in step 2; the jump path only applies
// real factors (decays, omega = 0 elements, normalisation) or collapses to a
// single level whose phase is that of d_a, which equals applying the step's
// phases at its end.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <algorithm>
#include <limits>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "common.hpp"
#include "ctx.hpp"
#include "philox.hpp"

namespace aqt {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Accumulator layouts of the 16x16 MFMAs (lane l, accumulator element i -> row;
// the column is always l % 16): the FP64 16x16x4 interleaves rows by 4, the FP32
// and BF16 variants keep four consecutive rows per lane.
struct ModeF64 {
  using T = double;
  using Acc = d4;
  static constexpr int KC = 4;
  __device__ static constexpr int row(int lane, int i) { return (lane >> 4) + 4 * i; }
};
struct ModeF32 {
  using T = float;
  using Acc = f4;
  static constexpr int KC = 4;
  __device__ static constexpr int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};
struct ModeBF16 {
  using T = float;
  using Acc = f4;
  static constexpr int KC = 32;
  __device__ static constexpr int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};
// 16-level instances: BF16 16x16x16 MFMA (four BF16 per lane and operand).
struct ModeBF16K16 {
  using T = float;
  using Acc = f4;
  static constexpr int KC = 16;
  __device__ static constexpr int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};
typedef short s16x4 __attribute__((ext_vector_type(4)));

struct StepArgs {
  int M, n, nq;
  int M_run;             // grid points processed (M, or fewer when autotuning)
  int width;             // trajectories of a one-wavefront tile if fewer than 8 TQ (else 0)
  int NP, TQ;            // padded levels and column tiles of this instance (batched runs)
  int64_t tiles;         // workgroup tiles of this instance
  int64_t t_base;        // first trajectory of this launch and its first row of `partial`
  int64_t tile0;         // (a run may take several launches of different tile widths)
  double* pgs_sum;       // [M] (batched runs reduce into these)
  double* pgs_sumsq;
  const double* tbeg;    // [M] start time of the step into grid g
  const double* tlen;    // [M] its length
  int64_t K;
  uint64_t seed, iid, traj0;
  int cap;
  const void* dlt_a;     // Delta fragments (hi for BF16)
  const void* dlt_b;     // Delta lo fragments (BF16 only)
  const void* dre;       // [M][NP] state precision
  const void* dim;
  const double* cinit;   // [NP]
  const double* Gamma;   // [M][NP]
  const double* d64re;   // [M][NP]
  const double* d64im;
  const double* R;       // [M][nq][NP][NP]
  const double* Rcol;    // [M][nq][NP][4] row sum, sum below the diagonal, diagonal of R
  const double* ehalf;   // [M][NP] exp(+Gamma dt / 2)
  const double* zdiag;   // [M][nq][NP]
  const float4* chf;     // FP32 runs: [M][nq][NP] (row sum, sum below the diagonal, diagonal, z_bb), else null
  const double* E;       // [M][NP]
  const int* gs;         // [M]
  double* partial;       // [tiles][M][2]
  int64_t* jump_totals;
  int32_t* jump_count;
  aqt_jump* jumps;
  int32_t* net_gs;
  int64_t* net_hist;
  int hist_lo, hist_hi;
  double* final_state;
  int* flags;            // AQT_RUN_* flags of the context (OR-ed)
};

// The kernels read their arguments where the launch left them (kernel-argument segment or
// the batch's argument array), as scalar loads from constant memory.  Held in registers for a
// whole kernel, the forty-odd pointers overflow the scalar registers into vector-register
// lanes (500 lane reads at 32 levels), so code off the step's main path takes them afresh.
using CArgs = const __attribute__((address_space(4))) StepArgs;
__device__ __forceinline__ CArgs& fresh(CArgs& a) {
  CArgs* p = &a;
  asm volatile("" : "+s"(p));
  return *p;
}

__device__ __forceinline__ d4 mfma_k4(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma_k4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Round-to-nearest-even FP32 -> BF16 of two values (inputs are finite), the first in the low half.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{x, y}), bf16x2));
}
__device__ __forceinline__ float bf16_low(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_high(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// hi/lo BF16 split of 4 floats: x ~ hi + lo with |x - hi - lo| <= 2^-17 |x|.  x holds the rest
// x - hi - lo on return; it has at most 8 significant bits, so hi, lo and the rest as three
// BF16 words are x exactly.
__device__ __forceinline__ void split4(float* x, uint2& hi, uint2& lo) {
#pragma clang fp contract(off)
  hi = make_uint2(bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]));
  x[0] -= bf16_low(hi.x);
  x[1] -= bf16_high(hi.x);
  x[2] -= bf16_low(hi.y);
  x[3] -= bf16_high(hi.y);
  lo = make_uint2(bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]));
  x[0] -= bf16_low(lo.x);
  x[1] -= bf16_high(lo.x);
  x[2] -= bf16_low(lo.y);
  x[3] -= bf16_high(lo.y);
}

// A-operand fragments of Delta read by one load per lane: 16 bytes of consecutive k
// chunks for the K = 4 MFMAs (frag_chunks of them), hi/lo BF16 words of one chunk for
// the K = 16 and K = 32 ones.
template <class Mode>
constexpr int frag_chunks() {
  return Mode::KC == 4 ? static_cast<int>(16 / sizeof(typename Mode::T)) : 1;
}
template <class Mode>
struct Frag {
  typename Mode::T v __attribute__((ext_vector_type(frag_chunks<Mode>())));
};
template <>
struct Frag<ModeBF16K16> {
  uint2 h, l;
};
template <>
struct Frag<ModeBF16> {
  uint4 h, l;
};

template <class Mode>
__device__ __forceinline__ Frag<Mode> load_frag(CArgs& a, size_t idx, unsigned lane = 0) {
  Frag<Mode> f;
  if constexpr (Mode::KC == 4) {
    f = (static_cast<const Frag<Mode>*>(a.dlt_a) + idx)[lane];
  } else if constexpr (Mode::KC == 16) {
    f.h = (static_cast<const uint2*>(a.dlt_a) + idx)[lane];
    f.l = (static_cast<const uint2*>(a.dlt_b) + idx)[lane];
  } else {
    f.h = (static_cast<const uint4*>(a.dlt_a) + idx)[lane];
    f.l = (static_cast<const uint4*>(a.dlt_b) + idx)[lane];
  }
  return f;
}

// Loads of A fragments kept in flight: a ring of PF loads per unit, refilled
// PF loads ahead and, at the end of a step, with the first ones of the next
// step, so the loads overlap the epilogue and the jump handler.  A row of Delta is
// latency-bound L2 traffic, so the loads are 16 bytes a lane (4-byte loads of single
// chunks: 256 levels FP32, a step of an 8-trajectory tile 12.0 us against 9.9, of a
// 16-trajectory tile 31.4 us against 14.4); rings of 2, 4 and 8 such loads measured
// 14.4, 14.5 and 14.6 us there and 28.0, 27.5 and 28.7 us with 40 trajectories.
template <class Mode, int NP>
constexpr int prefetch_depth() {
  constexpr int NKG = NP / Mode::KC / frag_chunks<Mode>();
  constexpr int want = (Mode::KC == 4) ? 4 : 2;
  return NKG < want ? NKG : want;
}

// ----------------------------------------------------------- jump handler --
// Tile layout in LDS: S[q] holds column tile q (8 trajectories) column-major; column
// c = (t & 7) + 8 * part carries the real (part 0) or imaginary (part 1) part of local
// trajectory t = 8 q + (c & 7).
// Columns are padded so that an MFMA operand read (row 4 k + lane / 16 of column lane % 16)
// meets distinct banks: 4 floats, and 2 doubles, which are read half a wavefront at a time
// (4 doubles: two-way conflicts).
template <class T>
constexpr int col_pad() {
  return sizeof(T) == 8 ? 2 : 4;
}
// One trajectory's column, by level.
template <class T>
struct PlainCol {
  T* p;
  __device__ __forceinline__ T get(int x) const { return p[x]; }
  __device__ __forceinline__ void set(int x, T v) const { p[x] = v; }
};
template <int NP, class T>
struct PlainTile {
  using Col = PlainCol<T>;
  T c[16][NP + col_pad<T>()];
  __device__ __forceinline__ Col col(int i) { return Col{&c[i][0]}; }
  // four rows of one column per lane: consecutive ones in the FP32 layout, else every fourth
  template <class Acc>
  __device__ __forceinline__ void load4(int lane, int rt, Acc& v) const {
    if constexpr (sizeof(T) == 4) {
      v = *reinterpret_cast<const Acc*>(&c[lane & 15][rt * 16 + 4 * (lane >> 4)]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = c[lane & 15][rt * 16 + (lane >> 4) + 4 * i];
    }
  }
  template <class Acc>
  __device__ __forceinline__ void store4(int lane, int rt, const Acc& v) {
    if constexpr (sizeof(T) == 4) {
      *reinterpret_cast<Acc*>(&c[lane & 15][rt * 16 + 4 * (lane >> 4)]) = v;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) c[lane & 15][rt * 16 + (lane >> 4) + 4 * i] = v[i];
    }
  }
};
// BF16 runs keep every amplitude as the three BF16 words of split4, whose sum it is: the
// products read their B operand as it stands.  (Splitting FP32 amplitudes in the k loop had
// every wavefront split the whole tile every step: 14000 of 40000 cycles at 256 levels with 40
// trajectories, where the epilogue, once per amplitude, takes 1800; FP32 words beside the split
// ones would not fit the LDS.)  8 words of padding spread the 16-byte operand reads.
template <int NP>
struct SplitCol {
  static constexpr int kWord = 16 * (NP + 8);   // distance between the words of an amplitude
  uint16_t* p;
  static __device__ __forceinline__ float up(uint16_t w) { return __uint_as_float(static_cast<uint32_t>(w) << 16); }
  __device__ __forceinline__ float get(int x) const { return (up(p[x]) + up(p[x + kWord])) + up(p[x + 2 * kWord]); }
  __device__ __forceinline__ void set(int x, float v) const {
    // (a product in v must not fuse with the subtraction: the words have to add up to v as rounded)
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint16_t w = static_cast<uint16_t>(bf16_pair(v, 0.f));
      p[x + k * kWord] = w;
      v -= up(w);
    }
  }
};
template <int NP>
struct SplitTile {
  using Col = SplitCol<NP>;
  uint16_t w[3][16][NP + 8];
  __device__ __forceinline__ Col col(int i) { return Col{&w[0][i][0]}; }
  __device__ __forceinline__ void load4(int lane, int rt, f4& v) const {
    const int r = rt * 16 + 4 * (lane >> 4);
    uint2 u[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) u[k] = *reinterpret_cast<const uint2*>(&w[k][lane & 15][r]);
    v[0] = (bf16_low(u[0].x) + bf16_low(u[1].x)) + bf16_low(u[2].x);
    v[1] = (bf16_high(u[0].x) + bf16_high(u[1].x)) + bf16_high(u[2].x);
    v[2] = (bf16_low(u[0].y) + bf16_low(u[1].y)) + bf16_low(u[2].y);
    v[3] = (bf16_high(u[0].y) + bf16_high(u[1].y)) + bf16_high(u[2].y);
  }
  __device__ __forceinline__ void store4(int lane, int rt, const f4& v) {
    const int r = rt * 16 + 4 * (lane >> 4);
    float x[4] = {v[0], v[1], v[2], v[3]};
    uint2 hi, lo;
    split4(x, hi, lo);
    *reinterpret_cast<uint2*>(&w[0][lane & 15][r]) = hi;
    *reinterpret_cast<uint2*>(&w[1][lane & 15][r]) = lo;
    *reinterpret_cast<uint2*>(&w[2][lane & 15][r]) = make_uint2(bf16_pair(x[0], x[1]), bf16_pair(x[2], x[3]));
  }
};
template <int NP, class Mode>
using TileCols = typename std::conditional<Mode::KC == 32, SplitTile<NP>, PlainTile<NP, typename Mode::T>>::type;

constexpr int kStepTables = 5;
// Wavefronts per workgroup.  Eight (two per SIMD) let one wave's LDS and load waits
// hide behind the other's MFMAs where each wave still has a large share of the
// GEMM (BF16, 256 levels, 40 trajectories, before the operand loads were pinned: 12.3 us a step
// against 19.3 with four); 64 levels
// keep four.
template <int NP, class Mode>
constexpr int waves_for() {
  return NP >= 128 ? 8 : 4;
}
// Exchange with lane ^ 8 (the other part of the same amplitude) by DPP row
// rotation: within each row of 16 lanes, rotating by 8 maps lane i to i ^ 8.
__device__ __forceinline__ float xor8(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, false));
}
__device__ __forceinline__ double xor8(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u & 0xffffffffu), 0x128, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), 0x128, 0xf, 0xf, false);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo));
}

// A crossing is handled by a segment of SEG consecutive lanes (seg_width): a
// wavefront serves 64 / SEG crossings at once.  Reductions, scans, ballots and broadcasts stay inside the segment, and
// are built from DPP row operations (rows of 16 lanes) and row-pair swaps rather
// than LDS-routed shuffles; every lane of a segment receives a bit-identical sum.
template <int CTRL, int ROWS = 0xf, bool BOUND = false>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, BOUND));
}
template <int CTRL, int ROWS = 0xf, bool BOUND = false>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u & 0xffffffffu), CTRL, ROWS, 0xf, BOUND);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, ROWS, 0xf, BOUND);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo));
}
// v + (the same register of the partner row): rows 0+1 and 2+3 (W = 16), or the two
// halves of the wavefront (W = 32); both operands of the swap are v, so the two
// results hold the pair's values in every lane and their sum needs no select.
template <int W>
__device__ __forceinline__ float swap_add(float v) {
  const int x = __builtin_bit_cast(int, v);
  const auto s = (W == 16) ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                           : __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return __builtin_bit_cast(float, static_cast<int>(s[0])) + __builtin_bit_cast(float, static_cast<int>(s[1]));
}
template <int W>
__device__ __forceinline__ double swap_add(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const int lo = static_cast<int>(u & 0xffffffffu), hi = static_cast<int>(u >> 32);
  const auto sl = (W == 16) ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                            : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto sh = (W == 16) ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                            : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  const double a = __builtin_bit_cast(double, (static_cast<uint64_t>(static_cast<uint32_t>(sh[0])) << 32) |
                                                  static_cast<uint32_t>(sl[0]));
  const double b = __builtin_bit_cast(double, (static_cast<uint64_t>(static_cast<uint32_t>(sh[1])) << 32) |
                                                  static_cast<uint32_t>(sl[1]));
  return a + b;
}
template <int SEG, class V>
__device__ __forceinline__ V seg_sum(V v) {
  static_assert(SEG == 16 || SEG == 32 || SEG == 64, "segments are whole rows");
  v += dpp<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);   // row_half_mirror
  v += dpp<0x140>(v);   // row_mirror: the row total in every lane of the row
  if constexpr (SEG >= 32) v = swap_add<16>(v);
  if constexpr (SEG == 64) v = swap_add<32>(v);
  return v;
}
// Inclusive scan over the segment's lanes in lane order.
template <int SEG, class V>
__device__ __forceinline__ V seg_scan(V v) {
  static_assert(SEG == 16 || SEG == 32 || SEG == 64, "segments are whole rows");
  v += dpp<0x111, 0xf, true>(v);   // row_shr:1 (zero shifted in)
  v += dpp<0x112, 0xf, true>(v);   // row_shr:2
  v += dpp<0x114, 0xf, true>(v);   // row_shr:4
  v += dpp<0x118, 0xf, true>(v);   // row_shr:8: inclusive scan of each row
  if constexpr (SEG >= 32) v += dpp<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
  if constexpr (SEG == 64) v += dpp<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
  return v;
}
// Lanes per crossing: one 16-lane row for up to 32 levels (four crossings per
// wavefront), half a wavefront for 64 levels, the whole wavefront above.
template <int NP>
__host__ __device__ constexpr int seg_width() {
  return NP <= 32 ? 16 : (NP == 64 ? 32 : kWave);
}
template <int SEG>
__device__ __forceinline__ uint64_t seg_ballot(bool pred, int base) {
  const uint64_t m = __ballot(pred);
  return (SEG == 64) ? m : (m >> base) & ((1ull << (SEG & 63)) - 1ull);
}
// Value of segment lane `idx` (segment-uniform) in every lane of the segment.
template <int SEG>
__device__ __forceinline__ float seg_read(float v, int idx, int base) {
  if constexpr (SEG == 64) return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), idx));
  else return __shfl(v, base + idx, kWave);
}
template <int SEG>
__device__ __forceinline__ double seg_read(double v, int idx, int base) {
  if constexpr (SEG == 64) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), idx));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u >> 32), idx));
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
  } else {
    return __shfl(v, base + idx, kWave);
  }
}
template <int SEG>
__device__ __forceinline__ uint32_t seg_read(uint32_t v, int idx, int base) {
  if constexpr (SEG == 64) return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), idx));
  else return __shfl(v, base + idx, kWave);
}

// First index x = lane + SEG j (chunk-major order) whose running sum of w exceeds thr,
// with `start` added in front; -1 if none.  Chunk totals first (independent sums),
// then one scan of the chunk the threshold falls in (the next chunk if rounding of
// the scan keeps it below).  Also returns the last index with w > 0 in *lastpos.
template <int SEG, int PL, class H>
__device__ __forceinline__ int seg_pick(const H (&w)[PL], H thr, H start, int base, int* lastpos) {
  H tot[PL];
#pragma unroll
  for (int j = 0; j < PL; ++j) tot[j] = seg_sum<SEG>(w[j]);
  H prefix = start;
  int hit = -1, last = -1;
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    if (hit < 0 && prefix + tot[j] > thr) {
      const H cum = seg_scan<SEG>(w[j]) + prefix;
      // cum is non-decreasing, so the first index exceeding thr carries weight; the
      // weight test only keeps a scan rounded below the chunk total from picking the
      // next chunk's (possibly empty) first level
      const uint64_t h = seg_ballot<SEG>(cum > thr && w[j] > H(0), base);
      if (h) hit = first_set_lane(h) + SEG * j;
    }
    prefix += tot[j];
    const uint64_t pz = seg_ballot<SEG>(w[j] > H(0), base);
    if (pz) last = last_set_lane(pz) + SEG * j;
  }
  *lastpos = last;
  return hit;
}

// Uniform draws of one trajectory served from Philox blocks computed in parallel:
// lane l of the segment holds block B0 + l (four words), so one generator
// evaluation covers the next 4 SEG draws; later draws fall back to a direct
// evaluation.
template <int SEG>
struct DrawCache {
  uint64_t B0;
  uint64_t w0, w1, w2, w3;
  uint64_t seed, iid, traj;
  int base;
  __device__ void fill(uint64_t seed_, uint64_t iid_, uint64_t traj_, uint64_t first_draw, int base_, int sl) {
    seed = seed_;
    iid = iid_;
    traj = traj_;
    base = base_;
    B0 = first_draw >> 2;
    const Philox4 r = philox4x64_10(traj, B0 + sl, 0, 0, seed, iid);
    w0 = r.w[0];
    w1 = r.w[1];
    w2 = r.w[2];
    w3 = r.w[3];
  }
  __device__ double operator()(uint64_t d) const {
    const uint64_t rel = (d >> 2) - B0;
    if (rel >= static_cast<uint64_t>(SEG)) return draw_uniform(seed, iid, traj, d);
    const unsigned k = static_cast<unsigned>(d & 3);
    const uint64_t mine = k == 0 ? w0 : (k == 1 ? w1 : (k == 2 ? w2 : w3));
    const uint32_t lo = seg_read<SEG>(static_cast<uint32_t>(mine & 0xffffffffu), static_cast<int>(rel), base);
    const uint32_t hi = seg_read<SEG>(static_cast<uint32_t>(mine >> 32), static_cast<int>(rel), base);
    return uniform_open01((static_cast<uint64_t>(hi) << 32) | lo);
  }
};

// Per-trajectory cache of Philox blocks in LDS: block x of trajectory t's stream sits in
// slot x & 3, and blocks b[t] and b[t] + 1 are there, b[t] = (3 m + 1) / 4 after m jumps, so
// that the draws of the next jump (3m+1, 3m+2 and the threshold 3m+3) are waiting.  One jump
// moves b[t] on by at most one block; a wavefront without a crossing of its own computes that
// block b[t] + 2 while the handlers run (rng_ahead).  A trajectory it could not serve (several
// jumps in one step, or every wavefront handling a crossing) is listed and refilled by
// wavefront 0 at the start of the next step (rng_refill).
struct RngCache {
  uint64_t (*w)[16];
  uint64_t* b;
  int* list;
  int* n;
};

// Block x of trajectory t into its slot.
__device__ __forceinline__ void rng_block(CArgs& a, int64_t tb, int t, uint64_t x, RngCache rc) {
  const Philox4 r = philox4x64_10(a.traj0 + static_cast<uint64_t>(tb + t), x, 0, 0, a.seed, a.iid);
#pragma unroll
  for (int k = 0; k < 4; ++k) rc.w[t][4 * (x & 3) + k] = r.w[k];
}

// Blocks B and B + 1, B = (3 m + 1) / 4, for n trajectories (list, or 0..n-1 when list
// is null; m = 0 when m_of is null): one wavefront, two lanes per trajectory.
__device__ void rng_refill(CArgs& a, int64_t tb, int n, const int* list, const int* m_of, RngCache rc,
                           int lane) {
  for (int i0 = 0; i0 < 2 * n; i0 += kWave) {
    const int i = i0 + lane;
    if (i < 2 * n) {
      const int t = list ? list[i >> 1] : (i >> 1);
      const int half = i & 1;
      const uint64_t mm = m_of ? static_cast<uint64_t>(m_of[t]) : 0ull;
      const uint64_t B = (3ull * mm + 1ull) >> 2;
      rng_block(a, tb, t, B + half, rc);
      if (half == 0) rc.b[t] = B;
    }
  }
}

// One wavefront, lane t of the trajectories in `mask` with m jumps so far: the block that the
// cache lacks after one more jump.  Its slot holds neither of the two blocks in use.
__device__ __forceinline__ void rng_ahead(CArgs& a, int64_t tb, uint64_t mask, int m, RngCache rc, int lane) {
  const uint64_t B = (3ull * static_cast<uint64_t>(m) + 1ull) >> 2, Bn = (3ull * static_cast<uint64_t>(m) + 4ull) >> 2;
  if (((mask >> lane) & 1ull) && Bn != B) rng_block(a, tb, lane, B + 2, rc);
}

// Orders LDS accesses of the lanes of one wavefront (which executes them in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Convergence of the crossing-time iteration: a step below tol * dt ends it.
template <class H>
__device__ constexpr H newton_tol() {
  return sizeof(H) == 8 ? H(1e-15) : H(4.0f * 1.1920929e-7f);
}

// One wavefront finishes step g for local trajectory t whose amplitudes after
// the fused propagator are in S (the threshold pass found the FP64 sum of |S|^2
// at or below r).  The handler computes in the state precision H = T: FP64 runs
// keep every step in FP64 (jump times and channels as the FP64 oracle's), mixed-
// precision runs take the crossing time, the channel scans and the renormalisation
// in FP32 (native exponentials, 32-bit shuffles).  The crossing test itself and
// the observable sums stay in FP64 in every mode.
// cre, cim: the trajectory's columns in LDS (real and imaginary parts by level).  WAVE: the
// one-wavefront kernel, which hands over Gamma and e^{G dt / 2} of this lane's levels in
// registers (tw) and keeps the Philox cache filled itself (rc.b = end of the filled blocks).
template <class T, int PL>
struct LaneTables {
  T G[PL], up[PL];
};
template <int NP, class T, bool STAGED, bool WAVE, class Col>
__device__ void finish_crossing(CArgs& args, int g, int t, int64_t jloc, Col cre, Col cim,
                                const double* s_r, double* s_rn, int* s_m, int* s_cnt, int* s_net, double* s_p,
                                int* s_kind, RngCache rc, bool ahead, int gsz, const double* tg, const float4* chs,
                                const LaneTables<T, NP / seg_width<NP>()>& tw) {
  using H = T;
  constexpr int SEG = seg_width<NP>();
  constexpr int PL = NP / SEG;
  CArgs& a = fresh(args);
  const int lane = threadIdx.x & (SEG - 1);                    // lane within the segment
  const int base = (threadIdx.x & (kWave - 1)) & ~(SEG - 1);   // first lane of the segment
  const double dt = a.tlen[g];
  const uint64_t traj = a.traj0 + static_cast<uint64_t>(jloc);   // Philox counter word 0
  // grid point g's Gamma, e^{G dt/2}, E and phase factors: staged in LDS (kStepTables rows
  // of NP) or read from the tables
  const size_t gofs = static_cast<size_t>(g) * NP;
  const double* Gam = STAGED ? tg : a.Gamma + gofs;
  const double* Eh = STAGED ? tg + NP : a.ehalf + gofs;
  const double* Eg = STAGED ? tg + 2 * NP : a.E + gofs;
  const double* Pre = STAGED ? tg + 3 * NP : a.d64re + gofs;
  const double* Pim = STAGED ? tg + 4 * NP : a.d64im + gofs;
  H sr[PL], si[PL], G[PL], up[PL];
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    const int x = lane + SEG * j;
    if constexpr (WAVE) {
      G[j] = tw.G[j];
      up[j] = tw.up[j];
    } else {
      G[j] = static_cast<H>(Gam[x]);
      up[j] = static_cast<H>(Eh[x]);
    }
    sr[j] = cre.get(x);
    si[j] = cim.get(x);
  }
  double r = s_r[t];
  int m = s_m[t];
  const int m0 = m;
  int cnt = s_cnt[t];
  int net = s_net[t];
  const double tk = a.tbeg[g];
  // the crossing test of the whole step, in FP64 as in the threshold pass:
  // sum_b |c_b|^2 e^{-G_b dt} = sum |S|^2
  double nu0 = 0.0;
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    const double xr = sr[j], xi = si[j];
    nu0 = fma(xr, xr, fma(xi, xi, nu0));
  }
  nu0 = seg_sum<SEG>(nu0);
  if (nu0 > r) {
    // no crossing after all (the threshold pass summed in another order): S stays
    double pg = 0.0;
#pragma unroll
    for (int j = 0; j < PL; ++j)
      if (lane + SEG * j < gsz) pg += static_cast<double>(sr[j]) * sr[j] + static_cast<double>(si[j]) * si[j];
    pg = seg_sum<SEG>(pg);
    if (lane == 0) {
      s_p[t] = pg / nu0;
      s_rn[t] = r;
    }
    return;
  }
  // draws of the next jump: the cached blocks; past them the segment's lanes evaluate blocks in
  // parallel (WAVE: into the cache, which only this wavefront touches)
  uint64_t Bc = rc.b[t];
  DrawCache<SEG> far;
  bool far_ready = false;
  auto fill_cache = [&](int m) {
    const uint64_t B = (3ull * static_cast<uint64_t>(m) + 1ull) >> 2;
    if (((3ull * static_cast<uint64_t>(m) + 3ull) >> 2) < Bc) return;
    // blocks below B are spent: slots of B .. B + 3 are free from Bc on
    const uint64_t x = max(B, Bc) + static_cast<uint64_t>(lane);
    if (x < B + 4) rng_block(a, jloc - t, t, x, rc);
    wave_lds_fence();
    Bc = B + 4;
  };
  auto draw = [&](uint64_t d) -> double {
    if constexpr (WAVE) {
      return uniform_open01(rc.w[t][d & 15]);
    } else {
      if ((d >> 2) - Bc < 2) return uniform_open01(rc.w[t][d & 15]);
      if (!far_ready) {
        far.fill(a.seed, a.iid, traj, d, base, lane);
        far_ready = true;
      }
      return far(d);
    }
  };
  // amplitudes at the start of the step's decay: undo the fused e^{-G dt / 2}
  H cr[PL], ci[PL];
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    cr[j] = sr[j] * up[j];
    ci[j] = si[j] * up[j];
  }
  const double* Rc = a.Rcol + static_cast<size_t>(g) * a.nq * NP * 4;
  double tau_e = 0.0;
  int guard = 0;
  for (; guard < AQT_MAX_JUMPS_PER_STEP; ++guard) {   // jumps within one step
    const H rem = static_cast<H>(dt - tau_e);
    if (guard > 0) {
      // after a jump: does the norm reach the next threshold within the rest of the step?
      H h[PL], part = H(0);
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        h[j] = exp(H(-0.5) * G[j] * rem);
        part += (cr[j] * cr[j] + ci[j] * ci[j]) * (h[j] * h[j]);
      }
      const H nu_end = seg_sum<SEG>(part);
      if (static_cast<double>(nu_end) > r) {
#pragma unroll
        for (int j = 0; j < PL; ++j) {
          cr[j] *= h[j];
          ci[j] *= h[j];
        }
        break;
      }
    }
    // crossing time: Newton on log sum_b w_b e^{-G_b tau} = log r from tau = 0
    H w[PL], hf[PL];
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      w[j] = cr[j] * cr[j] + ci[j] * ci[j];
      hf[j] = H(1);
    }
    H tau = H(0);
    const H logr = static_cast<H>(log(r));
    for (int it = 0; it < 100; ++it) {
      H s0 = H(0), s1 = H(0);
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        const H e = w[j] * (hf[j] * hf[j]);
        s0 += e;
        s1 += G[j] * e;
      }
      s0 = seg_sum<SEG>(s0);
      s1 = seg_sum<SEG>(s1);
      const H f = log(s0) - logr;
      // converged once the log-ratio is at rounding level: further steps only follow
      // the noise of the sums (for a slowly decaying level that noise exceeds tol dt)
      if (fabs(f) <= H(8) * std::numeric_limits<H>::epsilon()) break;
      const H fp = -s1 / s0;
      if (fp == H(0)) {
        tau = rem;
#pragma unroll
        for (int j = 0; j < PL; ++j) hf[j] = exp(H(-0.5) * G[j] * tau);
        break;
      }
      const H stp = -f / fp;
      if (!(stp > H(0))) break;
      const H tn = fmin(tau + stp, rem);
      const bool done = (tn - tau <= newton_tol<H>() * static_cast<H>(dt)) || (tn >= rem);
      tau = tn;
#pragma unroll
      for (int j = 0; j < PL; ++j) hf[j] = exp(H(-0.5) * G[j] * tau);
      if (done) break;
    }
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      cr[j] *= hf[j];
      ci[j] *= hf[j];
    }
    tau_e += static_cast<double>(tau);
    if constexpr (WAVE) fill_cache(m);
    const H u1 = static_cast<H>(draw(3ull * m + 1));
    const H u2 = static_cast<H>(draw(3ull * m + 2));
    // source level b: first index whose running sum of q_b Gamma_b exceeds u1 * total
    int b = -1;
    {
      H wq[PL];
#pragma unroll
      for (int j = 0; j < PL; ++j) wq[j] = (cr[j] * cr[j] + ci[j] * ci[j]) * G[j];
      H tot = H(0);
#pragma unroll
      for (int j = 0; j < PL; ++j) tot += wq[j];
      tot = seg_sum<SEG>(tot);
      int lastpos = -1;
      b = seg_pick<SEG, PL, H>(wq, u1 * tot, H(0), base, &lastpos);
      if (b < 0) b = lastpos;
    }
    if (b < 0) {
      // no populated level decays (a rounding-level crossing): nothing can jump
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        const H f = exp(H(-0.5) * G[j] * static_cast<H>(dt - tau_e));
        cr[j] *= f;
        ci[j] *= f;
      }
      break;
    }
    // qubit i and target a: inverse CDF over R[g][i][b][a] in i-major, a-minor order,
    // taken in stages -- the qubit from the row sums, then the diagonal (omega = 0)
    // element from the sum below it, and only for a != b a scan of the row --
    // which selects the same (i, a) as one pass over the whole list.
    int qi = 0, ta = b;
    {
      H thr, before, lo_q, dg_q;
      if (a.nq <= SEG) {
        // one channel per lane
        H rs = H(0), rlo = H(0), rdg = H(0);
        if (lane < a.nq) {
          if (chs) {   // staged in LDS
            const float4 c4 = chs[lane * NP + b];
            rs = static_cast<H>(c4.x);
            rlo = static_cast<H>(c4.y);
            rdg = static_cast<H>(c4.z);
          } else {
            const double* c4 = Rc + (static_cast<size_t>(lane) * NP + b) * 4;
            rs = static_cast<H>(c4[0]);
            rlo = static_cast<H>(c4[1]);
            rdg = static_cast<H>(c4[2]);
          }
        }
        const H cum_i = seg_scan<SEG>(rs);
        const H tot = seg_read<SEG>(cum_i, SEG - 1, base);
        thr = u2 * tot;
        const uint64_t hit_i = seg_ballot<SEG>(cum_i > thr && lane < a.nq, base);
        const uint64_t pos_i = seg_ballot<SEG>(rs > H(0), base);
        qi = hit_i ? first_set_lane(hit_i) : last_set_lane(pos_i);
        if (qi < 0) qi = 0;
        before = (qi > 0) ? seg_read<SEG>(cum_i, qi - 1, base) : H(0);
        lo_q = seg_read<SEG>(rlo, qi, base);
        dg_q = seg_read<SEG>(rdg, qi, base);
      } else {
        // more channels than lanes: channel lane + SEG j sits in chunk j; the chosen
        // channel's diagonal bounds are read once it is known
        constexpr int CQ = kWave / SEG;
        H rs[CQ];
#pragma unroll
        for (int j = 0; j < CQ; ++j) {
          const int ch = lane + SEG * j;
          rs[j] = (ch < a.nq) ? static_cast<H>(Rc[(static_cast<size_t>(ch) * NP + b) * 4]) : H(0);
        }
        H tot = H(0);
#pragma unroll
        for (int j = 0; j < CQ; ++j) tot += seg_sum<SEG>(rs[j]);
        thr = u2 * tot;
        int lastq = -1;
        qi = seg_pick<SEG, CQ, H>(rs, thr, H(0), base, &lastq);
        if (qi < 0) qi = lastq;
        if (qi < 0) qi = 0;
        const double* c4 = Rc + (static_cast<size_t>(qi) * NP + b) * 4;
        lo_q = static_cast<H>(c4[1]);
        dg_q = static_cast<H>(c4[2]);
        before = H(0);
#pragma unroll
        for (int j = 0; j < CQ; ++j) before += seg_sum<SEG>((lane + SEG * j < qi) ? rs[j] : H(0));
      }
      const H rel = thr - before;
      if (!(rel >= lo_q && rel < lo_q + dg_q)) {
        const double* row = a.R + ((static_cast<size_t>(g) * a.nq + qi) * NP + b) * NP;
        H v[PL];
#pragma unroll
        for (int j = 0; j < PL; ++j) {
          const int x = lane + SEG * j;
          v[j] = (x < NP) ? static_cast<H>(row[x]) : H(0);
        }
        int lastpos = -1;
        const int hit = seg_pick<SEG, PL, H>(v, thr, before, base, &lastpos);
        ta = (hit >= 0) ? hit : (lastpos >= 0 ? lastpos : b);
      }
    }
    int kind;
    if (ta != b) {
      // collapse to level ta, carrying the step phase e^{-i e_a dt}
      const double pr = Pre[ta];
      const double pim = Pim[ta];
      const double inv = 1.0 / sqrt(pr * pr + pim * pim);
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        const int x = lane + SEG * j;
        cr[j] = (x == ta) ? static_cast<H>(pr * inv) : H(0);
        ci[j] = (x == ta) ? static_cast<H>(pim * inv) : H(0);
      }
      kind = (Eg[ta] <= Eg[b]) ? AQT_KIND_RELAX : AQT_KIND_EXCITE;
      if (ta < gsz && b >= gsz) ++net;
      else if (b < gsz && ta >= gsz) --net;
    } else {
      const double* zd = a.zdiag + (static_cast<size_t>(g) * a.nq + qi) * NP;
      H z[PL];
      if (chs) {
#pragma unroll
        for (int j = 0; j < PL; ++j) {
          const int x = lane + SEG * j;
          z[j] = (x < NP) ? static_cast<H>(chs[qi * NP + x].w) : H(0);
        }
      } else {
#pragma unroll
        for (int j = 0; j < PL; ++j) {
          const int x = lane + SEG * j;
          z[j] = (x < NP) ? static_cast<H>(zd[x]) : H(0);
        }
      }
#pragma unroll
      for (int j = 0; j < PL; ++j) {
        cr[j] *= z[j];
        ci[j] *= z[j];
      }
      kind = AQT_KIND_DEPHASE;
    }
    H nrm = H(0);
#pragma unroll
    for (int j = 0; j < PL; ++j) nrm += cr[j] * cr[j] + ci[j] * ci[j];
    nrm = seg_sum<SEG>(nrm);
    const H inv = H(1) / sqrt(nrm);
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      cr[j] *= inv;
      ci[j] *= inv;
    }
    if (lane == 0) {
      if (a.jumps && cnt >= a.cap) atomicOr(a.flags, AQT_RUN_RECORDS_TRUNCATED);
      if (cnt < a.cap && a.jumps) {
        aqt_jump rec;
        rec.t = tk + tau_e;
        rec.step = g - 1;
        rec.qubit = static_cast<int16_t>(qi);
        rec.kind = static_cast<int16_t>(kind);
        rec.from_level = b;
        rec.to_level = ta;
        a.jumps[jloc * a.cap + cnt] = rec;
      }
      atomicAdd(&s_kind[kind], 1);
    }
    ++cnt;
    ++m;
    r = draw(3ull * m);
  }
  if (guard == AQT_MAX_JUMPS_PER_STEP && lane == 0) atomicOr(a.flags, AQT_RUN_JUMP_LIMIT);
  double pg = 0.0, pt = 0.0;
#pragma unroll
  for (int j = 0; j < PL; ++j) {
    const int x = lane + SEG * j;
    const double xr = cr[j], xi = ci[j];
    const double w2 = xr * xr + xi * xi;
    pt += w2;
    if (x < gsz) pg += w2;
    cre.set(x, cr[j]);
    cim.set(x, ci[j]);
  }
  pg = seg_sum<SEG>(pg);
  pt = seg_sum<SEG>(pt);
  if (lane == 0) {
    s_p[t] = pg / pt;
    s_rn[t] = r;
    s_m[t] = m;
    s_cnt[t] = cnt;
    s_net[t] = net;
    if constexpr (WAVE) {
      rc.b[t] = Bc;
    } else {
      const uint64_t B = (3ull * static_cast<uint64_t>(m) + 1ull) >> 2;
      if (ahead && m == m0 + 1) rc.b[t] = B;
      else if (B != Bc) rc.list[atomicAdd(rc.n, 1)] = t;
    }
  }
}

// Per-grid-point tables the jump handler reads, staged in LDS each step in the FP32
// kernels: loaded from HBM/L2 ahead of the GEMM, stored after it, so a crossing finds
// them at LDS latency.  (The BF16 and FP64 kernels run out of registers holding them
// across the GEMM and read them from the tables.)
template <class Mode>
constexpr bool stage_tables() {
  return Mode::KC == 4 && sizeof(typename Mode::T) == 4;
}
// The channel entries of a grid point (per channel and level: R's row sum, its part
// below the diagonal, its diagonal, z_bb) as well, in the FP32 kernels with 128 or
// more levels when they fit kChanStage entries: the channel draw and the dephasing
// factors of a crossing then need no dependent global load.  (The smaller-level
// kernels keep their LDS for more resident workgroups.)
constexpr int kChanStage = 2048;
template <class Mode, int NP>
constexpr bool stage_channels() {
  return stage_tables<Mode>() && NP >= 128;
}

// --------------------------------------------------------------- kernel ----
// Work split of the overlap GEMM over the WV wavefronts: each wave owns the row tiles
// rt = wave (mod WV) for every column tile (one A fragment feeds TQ MFMAs).  The k loop is
// outermost so each wave keeps UPW*TQ independent accumulator chains in flight.
template <int NP, int TQ, class Mode, int WV>
struct TileShared {
  using T = typename Mode::T;
  static constexpr int TT = 8 * TQ;
  TileCols<NP, Mode> S[TQ];
  double nu[WV][TT];   // partial squared norms per wavefront, accumulated in FP64
  double r[2][TT];   // waiting-time thresholds: read from r[g & 1], written to r[(g + 1) & 1]
  double p[TT];
  int m[TT], cnt[TT], net[TT];
  int kind[3];
  uint64_t rng[TT][16];  // Philox blocks of each trajectory's next draws (RngCache)
  uint64_t rngb[TT];
  int rfl[TT];           // trajectories whose blocks are to be refreshed
  int nrfl;
  double tg[kStepTables][NP];   // the step's Gamma, e^{G dt/2}, E, phase re/im (jump handler)
  float4 chs[stage_channels<Mode, NP>() ? kChanStage : 1];   // the step's channel entries (jump handler)
};

__device__ __forceinline__ const double* step_table(CArgs& a, int which) {
  return which == 0 ? a.Gamma : which == 1 ? a.ehalf : which == 2 ? a.E : which == 3 ? a.d64re : a.d64im;
}

template <int NP, int TQ, class Mode, int WV>
__device__ void run_tile(CArgs& a, int64_t tile, TileShared<NP, TQ, Mode, WV>& sh) {
  using T = typename Mode::T;
  using Acc = typename Mode::Acc;
  constexpr int NRT = NP / 16;
  constexpr int TT = 8 * TQ;
  static_assert(NRT % WV == 0, "every wavefront owns the same number of row tiles");
  constexpr int UPW = NRT / WV;             // row tiles per wave
  constexpr int NKC = NP / Mode::KC;
  constexpr int FW = frag_chunks<Mode>();   // k chunks per fragment load
  constexpr int NKG = NKC / FW;
  static_assert(TT <= kWave, "tile must fit one wavefront for the decision pass");

  auto& S = sh.S;
  auto& s_nu = sh.nu;
  double* s_p = sh.p;
  int* s_m = sh.m;
  int* s_cnt = sh.cnt;
  int* s_net = sh.net;
  int* s_kind = sh.kind;

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wave
  const int64_t tb = a.t_base + tile * TT;
  const int lc = lane & 15;          // MFMA output column
  const int part = (lane >> 3) & 1;  // 0: real part, 1: imaginary part

  const RngCache rc{sh.rng, sh.rngb, sh.rfl, &sh.nrfl};
  if (tid < TT) {
    const int64_t j = tb + tid;
    sh.r[1][tid] = (j < a.K) ? draw_uniform(a.seed, a.iid, a.traj0 + j, 0) : 2.0;   // read at g = 1
    s_m[tid] = 0;
    s_cnt[tid] = 0;
    s_net[tid] = 0;
  }
  if (tid < 3) s_kind[tid] = 0;
  if (tid == 0) sh.nrfl = 0;
  if (wave == WV - 1) rng_refill(a, tb, TT, nullptr, nullptr, rc, lane);   // m = 0: blocks 0 and 1

  int rt_u[UPW];
#pragma unroll
  for (int u = 0; u < UPW; ++u) rt_u[u] = (wave + WV * u) % NRT;   // (the modulo shows the range: 32-bit offsets)
  Acc acc[UPW][TQ];
  // fragment load (g, row tile, k group) lives at ((g * NRT + rt) * NKG + k) * 64 + lane
  size_t fbase[UPW];
#pragma unroll
  for (int u = 0; u < UPW; ++u) fbase[u] = static_cast<size_t>(rt_u[u]) * NKG * kWave + lane;
#define frag_index(gg, u, k) \
  (static_cast<size_t>(gg) * (NRT * NKG * kWave) + fbase[u] + static_cast<size_t>(k) * kWave)
  constexpr int PF = prefetch_depth<Mode, NP>();
  static_assert(NKG % PF == 0, "prefetch depth must divide the k groups");
  Frag<Mode> ring[PF][UPW];
  if (a.M_run > 2) {
#pragma unroll
    for (int s2 = 0; s2 < PF; ++s2)
#pragma unroll
      for (int u = 0; u < UPW; ++u)
        ring[s2][u] = load_frag<Mode>(a, frag_index(2, u, s2));
  }

  // The accumulators keep C between steps (the identity split starts from C);
  // only column tiles touched by the jump handler are reloaded from LDS.
  unsigned dirty = 0;
  // channel entries staged per step when the kernel keeps room for them and they fit
  constexpr int CHPT = stage_channels<Mode, NP>() ? (kChanStage + WV * 64 - 1) / (WV * 64) : 1;
  const int nch_e = a.nq * NP;
  const bool ch_on = stage_channels<Mode, NP>() && a.chf != nullptr && nch_e <= kChanStage;

  for (int g = 1; g < a.M_run; ++g) {
    const int gsz = a.gs[g];
    // jumps so far of trajectory `lane`, read where no handler runs (for rng_ahead)
    const int m_lane = (g > 1 && wave == WV - 1 && lane < TT) ? s_m[lane] : 0;
    // Philox blocks for the trajectories that jumped in the previous step (their
    // handlers listed them before the last barrier; this step's handlers read the
    // blocks only after the barrier that follows the GEMM)
    if (g > 1 && wave == 0) {
      const int nr = __builtin_amdgcn_readfirstlane(sh.nrfl);
      if (nr) {
        rng_refill(a, tb, nr, sh.rfl, s_m, rc, lane);
        if (lane == 0) sh.nrfl = 0;
      }
    }
    // ---- 1. C + Delta C (or the initial state at g = 1)
    if (g == 1) {
#pragma unroll
      for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int qq = 0; qq < TQ; ++qq)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = rt_u[u] * 16 + Mode::row(lane, i);
            acc[u][qq][i] = part ? T(0) : static_cast<T>(a.cinit[row]);
          }
    } else if (dirty) {
#pragma unroll
      for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int qq = 0; qq < TQ; ++qq)
          if ((dirty >> qq) & 1u) S[qq].load4(lane, rt_u[u], acc[u][qq]);
    }
    // the step's phase factors, loaded ahead of the GEMM (used by the epilogue)
    T dpre[UPW][4], dpim[UPW][4];
    {
      const T* dr = static_cast<const T*>(a.dre) + static_cast<size_t>(g) * NP;
      const T* di = static_cast<const T*>(a.dim) + static_cast<size_t>(g) * NP;
#pragma unroll
      for (int u = 0; u < UPW; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dpre[u][i] = dr[rt_u[u] * 16 + Mode::row(lane, i)];
          dpim[u][i] = di[rt_u[u] * 16 + Mode::row(lane, i)];
        }
    }
    constexpr bool STAGED = stage_tables<Mode>();
    constexpr int NTG = kStepTables * NP, TGPT = STAGED ? (NTG + WV * 64 - 1) / (WV * 64) : 1;
    double tgv[TGPT];
#pragma unroll
    for (int k = 0; k < TGPT; ++k) {
      const int f = tid + k * WV * 64;
      tgv[k] = (STAGED && f < NTG) ? step_table(a, f / NP)[static_cast<size_t>(g) * NP + f % NP] : 0.0;
    }
    float4 chv[CHPT];
#pragma unroll
    for (int k = 0; k < CHPT; ++k) {
      const int f = tid + k * WV * 64;
      chv[k] = (ch_on && f < nch_e) ? a.chf[static_cast<size_t>(g) * nch_e + f] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (g > 1) {
      T bnx[TQ];
      if constexpr (Mode::KC == 4) {
#pragma unroll
        for (int qq = 0; qq < TQ; ++qq) bnx[qq] = S[qq].c[lc][lane >> 4];
      }
      // two wavefronts share each SIMD, and with equal priorities they issue so that one
      // finishes its share early and leaves the other to run the tail of the GEMM alone
      // (8% slower in FP32); one of each pair at a raised priority keeps both issuing to
      // the end (waves 0-3 measured 0.6% faster than waves 4-7 in FP32, 0.7% in FP64
      // against equal priorities).
      if (WV == 8 && wave < 4) __builtin_amdgcn_s_setprio(1);
      // (unrolled: left to itself the compiler keeps a loop for the widest FP32 tile, whose
      // rotated ring waits on loads just issued; 25.7 us against 24.1)
#pragma unroll
      for (int kg = 0; kg < NKG; kg += PF) {
#pragma unroll
        for (int s2 = 0; s2 < PF; ++s2) {
          Frag<Mode> av[UPW];
#pragma unroll
          for (int u = 0; u < UPW; ++u) av[u] = ring[s2][u];
          // refill this slot PF loads ahead (next step's first ones at the end)
          // (after the last step the slot reloads grid M_run - 1: in bounds, unused)
          const int kn = kg + s2 + PF;
          const int gn = min(kn < NKG ? g : g + 1, a.M_run - 1);
          const int kk = kn < NKG ? kn : kn - NKG;
#pragma unroll
          for (int u = 0; u < UPW; ++u)
            ring[s2][u] = load_frag<Mode>(a, frag_index(gn, u, kk));
          // The unrolled loop is one block, in which the scheduler moves these loads down to the
          // products that use them: pinned, 256 levels take 6.9 us a step against 8.0 with 8
          // FP32 trajectories, 23.3 against 24.2 with 40, and 6.6 against 9.1 with 16 in BF16.
          // FP64 (24 trajectories) already keeps them apart, and only loses freedom (0.7%).
          if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0);
          if constexpr (Mode::KC == 4) {
            // B for this chunk was read one chunk ahead; read the next one now (on
            // the last chunk that is chunk 0 again: unused)
#pragma unroll
            for (int w = 0; w < FW; ++w) {
              const int k = (kg + s2) * FW + w;
              T bcur[TQ];
#pragma unroll
              for (int qq = 0; qq < TQ; ++qq) bcur[qq] = bnx[qq];
              const bool wraps = s2 == PF - 1 && w == FW - 1;   // only here: fixed offsets elsewhere
              const int krn = (wraps ? 4 * (k + 1) & (NP - 1) : 4 * (k + 1)) + (lane >> 4);
#pragma unroll
              for (int qq = 0; qq < TQ; ++qq) bnx[qq] = S[qq].c[lc][krn];
#pragma unroll
              for (int u = 0; u < UPW; ++u)
#pragma unroll
                for (int qq = 0; qq < TQ; ++qq) acc[u][qq] = mfma_k4(av[u].v[w], bcur[qq], acc[u][qq]);
            }
          } else {
            const int k0 = 32 * (kg + s2) + 8 * (lane >> 4);
            bf16x8 bh[TQ], bl[TQ];
#pragma unroll
            for (int qq = 0; qq < TQ; ++qq) {
              bh[qq] = *reinterpret_cast<const bf16x8*>(&S[qq].w[0][lc][k0]);
              bl[qq] = *reinterpret_cast<const bf16x8*>(&S[qq].w[1][lc][k0]);
            }
#pragma unroll
            for (int u = 0; u < UPW; ++u) {
              const bf16x8 ah = __builtin_bit_cast(bf16x8, av[u].h);
              const bf16x8 al = __builtin_bit_cast(bf16x8, av[u].l);
#pragma unroll
              for (int qq = 0; qq < TQ; ++qq) {
                Acc c = acc[u][qq];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[qq], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[qq], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[qq], c, 0, 0, 0);
                acc[u][qq] = c;
              }
            }
          }
        }
      }
    }
    if (WV == 8) __builtin_amdgcn_s_setprio(0);
    // the step tables for this step's handlers (the previous step's handlers are done)
    if constexpr (STAGED) {
#pragma unroll
      for (int k = 0; k < TGPT; ++k) {
        const int f = tid + k * WV * 64;
        if (f < NTG) sh.tg[f / NP][f % NP] = tgv[k];
      }
    }
    if (ch_on) {
#pragma unroll
      for (int k = 0; k < CHPT; ++k) {
        const int f = tid + k * WV * 64;
        if (f < nch_e) sh.chs[f] = chv[k];
      }
    }
    __syncthreads();   // every wave has finished reading S
    // ---- 2. C' = d o C and the squared norms (partial sums per wave).
    // The squares of state-precision amplitudes are exact in FP64 and every sum of
    // them (per lane, across lanes, across slots) is taken in FP64, so the threshold
    // test sees the norm of the stored state to FP64 rounding whatever the state
    // precision: a compensated norm, not a state-precision running sum.
    {
      double nacc[TQ];
#pragma unroll
      for (int qq = 0; qq < TQ; ++qq) nacc[qq] = 0.0;
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        const int rt = rt_u[u];
        T drv[4], div[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          drv[i] = dpre[u][i];
          div[i] = dpim[u][i];
        }
#pragma unroll
        for (int qq = 0; qq < TQ; ++qq) {
          double nrm = 0.0;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const T y = acc[u][qq][i];
            const T yp = xor8(y);       // the other part of the same amplitude
            const T yr = part ? yp : y, yi = part ? y : yp;
            const T c = part ? (drv[i] * yi + div[i] * yr) : (drv[i] * yr - div[i] * yi);
            acc[u][qq][i] = c;
            const double cd = static_cast<double>(c);
            nrm = fma(cd, cd, nrm);
          }
          S[qq].store4(lane, rt, acc[u][qq]);
          nacc[qq] += nrm;
        }
      }
#pragma unroll
      for (int qq = 0; qq < TQ; ++qq) {
        double nrm = nacc[qq];
        nrm += xor8(nrm);
        nrm = swap_add<16>(nrm);
        nrm = swap_add<32>(nrm);
        if (lane < 8) s_nu[wave][qq * 8 + lane] = nrm;
      }
    }
    __syncthreads();
    // ---- 3. threshold test.  Every wavefront takes it for all TT trajectories (lane t,
    // the same FP64 sums in the same order), so each knows the crossing set from a
    // ballot, without a list or another barrier; the thresholds it reads are not
    // written this step (the handlers write the other buffer).  Wavefront 0 records
    // the ground-cluster weight of the trajectories that do not cross and carries
    // their thresholds over.
    const double* s_r = sh.r[g & 1];
    double* s_rn = sh.r[(g + 1) & 1];
    uint64_t cmask;
    {
      bool cross = false;
      double nu = 0.0;
      const bool valid = lane < TT && tb + lane < a.K;
      if (lane < TT) {
#pragma unroll
        for (int sl = 0; sl < WV; ++sl) nu += s_nu[sl][lane];
        cross = valid && nu <= s_r[lane];
      }
      cmask = __ballot(cross);
      if (wave == 0 && lane < TT && !cross) {
        double gw = 0.0;
        if (valid) {
          const auto cre = S[lane >> 3].col(lane & 7), cim = S[lane >> 3].col((lane & 7) + 8);
          for (int row = 0; row < gsz; ++row) {
            const double re = static_cast<double>(cre.get(row));
            const double im = static_cast<double>(cim.get(row));
            gw += re * re + im * im;
          }
        }
        s_p[lane] = valid ? gw / nu : 0.0;
        s_rn[lane] = s_r[lane];
      }
    }
    const int ncross = __popcll(cmask);
    {
      // 64 / SEG crossings per wavefront, one per segment of SEG lanes; crossing e is
      // the trajectory of the e-th set bit of the mask
      constexpr int SEG = seg_width<NP>();
      constexpr int NSEG = kWave / SEG;
      const int seg = (tid & (kWave - 1)) / SEG;
      // the last wavefront, when it has no crossing of its own, computes the Philox blocks
      const bool ahead = ncross <= (WV - 1) * NSEG;
      if (ahead && ncross && wave == WV - 1) rng_ahead(a, tb, cmask, m_lane, rc, lane);
      for (int e0 = wave * NSEG; e0 < ncross; e0 += WV * NSEG) {
        const int e = e0 + seg;
        if (e < ncross) {
          uint64_t mm = cmask;
          for (int k = 0; k < e; ++k) mm &= mm - 1;
          const int t = __builtin_ctzll(mm);
          finish_crossing<NP, T, STAGED, false>(a, g, t, tb + t, S[t >> 3].col(t & 7), S[t >> 3].col((t & 7) + 8),
                                                s_r, s_rn, s_m, s_cnt, s_net, s_p, s_kind, rc, ahead, gsz,
                                                &sh.tg[0][0], ch_on ? sh.chs : nullptr, {});
        }
      }
    }
    __syncthreads();
    // column tiles whose amplitudes the handler rewrote
    dirty = 0;
#pragma unroll
    for (int q = 0; q < TQ; ++q)
      if ((cmask >> (8 * q)) & 0xffull) dirty |= 1u << q;
    // ---- 4. per-tile observable sums (wave 0)
    if (wave == 0) {
      const double p = (lane < TT) ? s_p[lane] : 0.0;
      const double sp = seg_sum<64>(p);
      const double sq = seg_sum<64>(p * p);
      if (lane == 0) {
        double* dst = a.partial + (static_cast<size_t>(a.tile0 + tile) * a.M + g) * 2;
        dst[0] = sp;
        dst[1] = sq;
      }
    }
  }
  // ---- per-trajectory results
  if (tid < TT && tb + tid < a.K) {
    const int64_t j = tb + tid;
    if (a.jump_count) a.jump_count[j] = s_cnt[tid];
    if (a.net_gs) a.net_gs[j] = s_net[tid];
    if (a.net_hist) {
      int v = s_net[tid];
      v = v < a.hist_lo ? a.hist_lo : (v > a.hist_hi ? a.hist_hi : v);
      atomicAdd(reinterpret_cast<unsigned long long*>(&a.net_hist[v - a.hist_lo]), 1ull);
    }
  }
  if (a.final_state) {
    for (int e = tid; e < TT * a.n; e += blockDim.x) {
      const int t = e / a.n, x = e - t * a.n;
      const int64_t j = tb + t;
      if (j < a.K) {
        a.final_state[(j * a.n + x) * 2 + 0] = static_cast<double>(S[t >> 3].col(t & 7).get(x));
        a.final_state[(j * a.n + x) * 2 + 1] = static_cast<double>(S[t >> 3].col((t & 7) + 8).get(x));
      }
    }
  }
  if (a.jump_totals && tid < 3 && s_kind[tid])
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.jump_totals[tid]),
              static_cast<unsigned long long>(s_kind[tid]));
  __syncthreads();   // the shared tile state may be reused by the caller
#undef frag_index
}

// ------------------------------------------------- one wavefront per tile ----
// Up to kWaveLevels levels a tile belongs to one wavefront, which keeps its amplitudes in
// the accumulators for the whole anneal and meets no barrier.  The four-wavefront tile
// above spends its step there on latency that has nothing to hide behind: at 16 levels one
// wavefront multiplies while three wait at three barriers, and each step waits for its own
// table loads (4400 cycles for four MFMAs).  Here
//   * the MFMA B operand is made from the accumulators by lane-row exchanges (none in
//     FP64 and in the K = 16 BF16 form, whose accumulator and operand layouts agree);
//   * Delta, the phase factors and the handler's decay tables are loaded one step ahead;
//   * thresholds and norms sit in lanes: lane t holds trajectory t, a step without a
//     crossing never touches LDS;
//   * a pass over the crossings takes 64 / seg_width of them (one per segment) through a
//     small LDS column buffer;
//   * Philox blocks are computed for all trajectories of the tile at once, up to four
//     blocks ahead, when a crossing finds its cache empty.
// Microseconds a step, four wavefronts -> one: 16 levels, 1000 trajectories FP64 1.77 -> 1.15,
// FP32 2.44 -> 0.99; 32 levels, 10^5 trajectories FP32 27.3 -> 18.5, BF16 26.9 -> 16.4, FP64
// 71.9 -> 32.7.  At 64 levels it spills (FP32, 30000 trajectories 15.6 -> 41), so the
// four-wavefront tile stays there.
constexpr int kWaveLevels = 32;

template <int NP, int TQ, class Mode>
struct WaveShared {
  using T = typename Mode::T;
  static constexpr int TT = 8 * TQ;
  static constexpr int NSEG = kWave / seg_width<NP>();
  T X[NSEG][2][NP + col_pad<T>()];   // columns of the crossings of a pass
  double r[TT], p[TT];
  uint64_t rng[TT][16], rngb[TT];
  int m[TT], cnt[TT], net[TT];
  int kind[3];
};

// Swap the odd 16-lane rows of x with the even rows of y (W = 16), or the upper half of x
// with the lower half of y (W = 32).
template <int W>
__device__ __forceinline__ void row_swap(uint32_t& x, uint32_t& y) {
  const auto s = (W == 16) ? __builtin_amdgcn_permlane16_swap(x, y, false, false)
                           : __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = s[0];
  y = s[1];
}

// B operands of one column tile from its accumulators c[row tile] (rows 4 (lane / 16) + i,
// FP64 lane / 16 + 4 i): B of k chunk k holds row 4 k + lane / 16.
template <int NRT>
__device__ __forceinline__ void wave_operand(const d4 (&c)[NRT], double (&b)[4 * NRT]) {
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
    for (int i = 0; i < 4; ++i) b[4 * rt + i] = c[rt][i];
}
template <int NRT>
__device__ __forceinline__ void wave_operand(const f4 (&c)[NRT], float (&b)[4 * NRT]) {
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(c[rt][i]);
    row_swap<32>(v[0], v[2]);
    row_swap<32>(v[1], v[3]);
    row_swap<16>(v[0], v[1]);
    row_swap<16>(v[2], v[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[4 * rt + i] = __uint_as_float(v[i]);
  }
}

template <int NP, int TQ, class Mode>
__device__ void run_wave(CArgs& a, int64_t tile, WaveShared<NP, TQ, Mode>& sh) {
  using T = typename Mode::T;
  using Acc = typename Mode::Acc;
  constexpr int NRT = NP / 16, TT = 8 * TQ, NKC = NP / Mode::KC;
  constexpr int FW = frag_chunks<Mode>(), NKG = NKC / FW;
  constexpr int SEG = seg_width<NP>(), NSEG = kWave / SEG, PL = NP / SEG;
  static_assert(TT <= kWave, "one lane per trajectory");
  const int lane = threadIdx.x & (kWave - 1);
  const int width = a.width ? a.width : TT;
  const int64_t tb = a.t_base + tile * width;
  const int lc = lane & 15;
  const int part = (lane >> 3) & 1;
  const bool valid = lane < width && tb + lane < a.K;
  const int tl = lane < TT ? lane : 0;   // this lane's trajectory in the LDS arrays
  const RngCache rc{sh.rng, sh.rngb, nullptr, nullptr};

  if (lane < TT) {
    sh.m[lane] = 0;
    sh.cnt[lane] = 0;
    sh.net[lane] = 0;
    sh.rngb[lane] = 0;
  }
  if (lane < 3) sh.kind[lane] = 0;
  wave_lds_fence();
  // Philox blocks up to four from the one of the next jump's first draw, kWave / TT at a time
  constexpr int LPT = kWave / TT;
  auto refill = [&]() {
    const int t = lane / LPT;
    const uint64_t B = (3ull * static_cast<uint64_t>(sh.m[t]) + 1ull) >> 2, end = sh.rngb[t];
    const uint64_t x = end + static_cast<uint64_t>(lane % LPT);
    if (x < B + 4) rng_block(a, tb, t, x, rc);
    wave_lds_fence();
    if (lane % LPT == 0) sh.rngb[t] = min(end + static_cast<uint64_t>(LPT), B + 4);
    wave_lds_fence();
  };
  refill();
  double r = valid ? uniform_open01(sh.rng[tl][0]) : 2.0;   // draw 0
  if (lane < TT) sh.r[lane] = r;

  // Delta fragments and tables of the next step
  Frag<Mode> A[NRT][NKG];
  T npre[NRT][4], npim[NRT][4];
  double nG[PL], nup[PL];
  // (uniform base plus a 32-bit lane offset: one offset register for all of them)
  const unsigned ul = lane, row0 = Mode::row(lane, 0);
  auto load_delta = [&](int g) {
    const size_t g0 = static_cast<size_t>(g) * (NRT * NKG * kWave);
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int k = 0; k < NKG; ++k) A[rt][k] = load_frag<Mode>(a, g0 + (rt * NKG + k) * kWave, ul);
  };
  auto load_tables = [&](int g) {
    const T* dr = static_cast<const T*>(a.dre) + static_cast<size_t>(g) * NP;
    const T* di = static_cast<const T*>(a.dim) + static_cast<size_t>(g) * NP;
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        npre[rt][i] = (dr + (rt * 16 + Mode::row(0, i)))[row0];
        npim[rt][i] = (di + (rt * 16 + Mode::row(0, i)))[row0];
      }
    const double* Gg = a.Gamma + static_cast<size_t>(g) * NP;
    const double* Eg = a.ehalf + static_cast<size_t>(g) * NP;
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      nG[j] = (Gg + SEG * j)[ul & (SEG - 1)];
      nup[j] = (Eg + SEG * j)[ul & (SEG - 1)];
    }
  };
  const int glast = a.M_run - 1;
  load_tables(min(1, glast));
  load_delta(min(2, glast));
  int gs_next = a.gs[min(1, glast)];

  Acc acc[TQ][NRT];
#pragma unroll
  for (int q = 0; q < TQ; ++q)
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc[q][rt][i] = part ? T(0) : static_cast<T>(a.cinit[rt * 16 + Mode::row(lane, i)]);

  for (int g = 1; g <= glast; ++g) {
    const int gsz = gs_next;
    T dre[NRT][4], dim[NRT][4];
    LaneTables<T, PL> tw;
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dre[rt][i] = npre[rt][i];
        dim[rt][i] = npim[rt][i];
      }
#pragma unroll
    for (int j = 0; j < PL; ++j) {
      tw.G[j] = static_cast<T>(nG[j]);
      tw.up[j] = static_cast<T>(nup[j]);
    }
    const int gn = min(g + 1, glast);
    load_tables(gn);
    gs_next = a.gs[gn];
    // ---- 1. C + Delta C, the k chunks of each accumulator in ascending order
    if (g > 1) {
#pragma unroll
      for (int q = 0; q < TQ; ++q) {
        if constexpr (Mode::KC == 4) {
          T b[4 * NRT];
          wave_operand<NRT>(acc[q], b);
#pragma unroll
          for (int k = 0; k < NKC; ++k)
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) acc[q][rt] = mfma_k4(A[rt][k / FW].v[k % FW], b[k], acc[q][rt]);
        } else {
          uint32_t h[NRT][2], l[NRT][2];
#pragma unroll
          for (int rt = 0; rt < NRT; ++rt) {
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = acc[q][rt][i];
            uint2 hh, ll;
            split4(x, hh, ll);
            h[rt][0] = hh.x;
            h[rt][1] = hh.y;
            l[rt][0] = ll.x;
            l[rt][1] = ll.y;
          }
          if constexpr (Mode::KC == 16) {
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) {
              const s16x4 ah = __builtin_bit_cast(s16x4, A[rt][0].h), al = __builtin_bit_cast(s16x4, A[rt][0].l);
              const s16x4 bh = __builtin_bit_cast(s16x4, make_uint2(h[0][0], h[0][1]));
              const s16x4 bl = __builtin_bit_cast(s16x4, make_uint2(l[0][0], l[0][1]));
              Acc c = acc[q][rt];
              c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh, c, 0, 0, 0);
              c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bl, c, 0, 0, 0);
              c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh, c, 0, 0, 0);
              acc[q][rt] = c;
            }
          } else {
            // chunk k: lane row j holds rows 32 k + 8 j .. + 7 (two 4-row words of row tile 2k + j / 2)
#pragma unroll
            for (int k = 0; k < NKC; ++k) {
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                row_swap<32>(h[2 * k][e], h[2 * k + 1][e]);
                row_swap<16>(h[2 * k][e], h[2 * k + 1][e]);
                row_swap<32>(l[2 * k][e], l[2 * k + 1][e]);
                row_swap<16>(l[2 * k][e], l[2 * k + 1][e]);
              }
              const bf16x8 bh = __builtin_bit_cast(bf16x8, make_uint4(h[2 * k][0], h[2 * k][1], h[2 * k + 1][0], h[2 * k + 1][1]));
              const bf16x8 bl = __builtin_bit_cast(bf16x8, make_uint4(l[2 * k][0], l[2 * k][1], l[2 * k + 1][0], l[2 * k + 1][1]));
#pragma unroll
              for (int rt = 0; rt < NRT; ++rt) {
                const bf16x8 ah = __builtin_bit_cast(bf16x8, A[rt][k].h), al = __builtin_bit_cast(bf16x8, A[rt][k].l);
                Acc c = acc[q][rt];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, c, 0, 0, 0);
                acc[q][rt] = c;
              }
            }
          }
        }
      }
      load_delta(gn);
    }
    // ---- 2. C' = d o C; squared norms and ground-cluster weights in FP64, lane t's
    // trajectory t selected from the column sums
    double nu = 0.0, gw = 0.0;
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      double nq = 0.0, gq = 0.0;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        double sq[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const T y = acc[q][rt][i];
          const T yp = xor8(y);       // the other part of the same amplitude
          const T yr = part ? yp : y, yi = part ? y : yp;
          const T drv = dre[rt][i], div = dim[rt][i];
          const T c = part ? (drv * yi + div * yr) : (drv * yr - div * yi);
          acc[q][rt][i] = c;
          const double cd = static_cast<double>(c);
          sq[i] = cd;
          nq = fma(cd, cd, nq);
        }
        if (rt * 16 < gsz) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double v = (rt * 16 + Mode::row(lane, i) < gsz) ? sq[i] : 0.0;
            gq = fma(v, v, gq);
          }
        }
      }
      nq += xor8(nq);
      nq = swap_add<16>(nq);
      nq = swap_add<32>(nq);
      gq += xor8(gq);
      gq = swap_add<16>(gq);
      gq = swap_add<32>(gq);
      if ((lane >> 3) == q) {
        nu = nq;
        gw = gq;
      }
    }
    // ---- 3. threshold test and crossings
    const uint64_t cmask = __ballot(valid && nu <= r);
    double p = valid ? gw / nu : 0.0;
    if (cmask) {
      // two jumps of every crossing need blocks up to (3 m + 6) / 4
      for (;;) {
        const bool lack = ((cmask >> lane) & 1ull) &&
                          ((3ull * static_cast<uint64_t>(sh.m[tl]) + 6ull) >> 2) >= sh.rngb[tl];
        if (!__ballot(lack)) break;
        refill();
      }
      uint64_t left = cmask;
      while (left) {
        // the lowest NSEG crossings; seg's own is the seg-th of them
        uint64_t sel = 0;
        int t = 0;
        const int seg = lane / SEG;
        int n = 0;
#pragma unroll
        for (int e = 0; e < NSEG; ++e)
          if (left) {
            const int te = __builtin_ctzll(left);
            left &= left - 1;
            sel |= 1ull << te;
            if (seg == e) t = te;
            ++n;
          }
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
          if (!((sel >> (8 * q)) & 0xffull)) continue;
          const int tq = 8 * q + (lane & 7);
          if ((sel >> tq) & 1ull) {
            T* x = &sh.X[__popcll(sel & ((1ull << tq) - 1ull))][part][0];
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
              for (int i = 0; i < 4; ++i) x[rt * 16 + Mode::row(lane, i)] = acc[q][rt][i];
          }
        }
        wave_lds_fence();
        if (seg < n)
          finish_crossing<NP, T, false, true>(a, g, t, tb + t, PlainCol<T>{&sh.X[seg][0][0]}, PlainCol<T>{&sh.X[seg][1][0]}, sh.r, sh.r, sh.m,
                                              sh.cnt, sh.net, sh.p, sh.kind, rc, false, gsz, nullptr, nullptr, tw);
        wave_lds_fence();
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
          if (!((sel >> (8 * q)) & 0xffull)) continue;
          const int tq = 8 * q + (lane & 7);
          if ((sel >> tq) & 1ull) {
            const T* x = &sh.X[__popcll(sel & ((1ull << tq) - 1ull))][part][0];
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[q][rt][i] = x[rt * 16 + Mode::row(lane, i)];
          }
        }
        wave_lds_fence();
      }
      if ((cmask >> lane) & 1ull) {
        r = sh.r[lane];
        p = sh.p[lane];
      }
    }
    // ---- 4. per-tile observable sums
    const double sp = seg_sum<64>(p);
    const double sq = seg_sum<64>(p * p);
    if (lane == 0) {
      double* dst = a.partial + (static_cast<size_t>(a.tile0 + tile) * a.M + g) * 2;
      *reinterpret_cast<double2*>(dst) = make_double2(sp, sq);
    }
  }
  // ---- per-trajectory results
  if (valid) {
    const int64_t j = tb + lane;
    if (a.jump_count) a.jump_count[j] = sh.cnt[lane];
    if (a.net_gs) a.net_gs[j] = sh.net[lane];
    if (a.net_hist) {
      int v = sh.net[lane];
      v = v < a.hist_lo ? a.hist_lo : (v > a.hist_hi ? a.hist_hi : v);
      atomicAdd(reinterpret_cast<unsigned long long*>(&a.net_hist[v - a.hist_lo]), 1ull);
    }
  }
  if (a.final_state) {
#pragma unroll
    for (int q = 0; q < TQ; ++q) {
      const int64_t j = tb + 8 * q + (lane & 7);
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int x = rt * 16 + Mode::row(lane, i);
          if (8 * q + (lane & 7) < width && j < a.K && x < a.n) a.final_state[(j * a.n + x) * 2 + part] = static_cast<double>(acc[q][rt][i]);
        }
    }
  }
  if (a.jump_totals && lane < 3 && sh.kind[lane])
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.jump_totals[lane]),
              static_cast<unsigned long long>(sh.kind[lane]));
  wave_lds_fence();   // the shared state may be reused by the caller
}

// Tile body of a level count: one wavefront up to kWaveLevels levels.
template <int NP, int TQ, class Mode, bool WAVE = (NP <= kWaveLevels)>
struct Tile {
  static constexpr int WV = 1;
  using Shared = WaveShared<NP, TQ, Mode>;
  static __device__ __forceinline__ void run(CArgs& a, int64_t tile, Shared& sh) {
    run_wave<NP, TQ, Mode>(a, tile, sh);
  }
};
template <int NP, int TQ, class Mode>
struct Tile<NP, TQ, Mode, false> {
  static constexpr int WV = waves_for<NP, Mode>();
  using Shared = TileShared<NP, TQ, Mode, WV>;
  static __device__ __forceinline__ void run(CArgs& a, int64_t tile, Shared& sh) {
    run_tile<NP, TQ, Mode, WV>(a, tile, sh);
  }
};

// Wavefronts per SIMD the register allocation must leave room for.  The FP32 / BF16
// four-wavefront tile at 64 levels is bound by the latency of jump handling: three.  The
// one-wavefront tiles and FP64 at 64 levels: two (three and four measured equal or slower
// there, up to 31 against 20 us a step at 32 levels, 64-trajectory tiles, from spills).
// Larger levels: the compiler's choice.
template <int NP, class Mode>
constexpr int min_waves_per_simd() {
  return NP > 64 ? 1 : (NP <= kWaveLevels || sizeof(typename Mode::T) == 8) ? 2 : 3;
}

template <int NP, int TQ, class Mode>
__global__ __launch_bounds__((Tile<NP, TQ, Mode>::WV * 64))
__attribute__((amdgpu_waves_per_eu(min_waves_per_simd<NP, Mode>()))) void k_trajectories(StepArgs) {
  using Body = Tile<NP, TQ, Mode>;
  __shared__ typename Body::Shared sh;
  Body::run(*(CArgs*)__builtin_amdgcn_kernarg_segment_ptr(), blockIdx.x, sh);   // its one argument
}

// Compensated (Neumaier) running sum: s + c carries the rounding error of every addition.
struct CompSum {
  double s = 0.0, c = 0.0;
  __device__ void add(double x) {
    const double t = s + x;
    c += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
    s = t;
  }
  __device__ double value() const { return s + c; }
};

// Sums of the per-tile observables of one run over its tiles.  A workgroup takes kRedG
// consecutive grid points (one 256-byte row segment of `partial` per tile) and splits the
// tiles over kRedT threads per grid point, each with its own compensated sums, which are
// then added in thread order: with one thread per grid point a run of 1563 tiles and 500
// points waited 460 us for its loads on two workgroups; this takes 37 us.
constexpr int kRedG = 16, kRedT = 16;
__device__ void reduce_tiles(const double* __restrict__ partial, int64_t tiles, int M, double K,
                             double* __restrict__ sum, double* __restrict__ sumsq) {
  __shared__ double part[kRedT][kRedG][4];
  const int gl = threadIdx.x % kRedG, tl = threadIdx.x / kRedG;
  const int g = blockIdx.x * kRedG + gl;
  CompSum cs, cq;
  if (g > 0 && g < M) {
    for (int64_t t = tl; t < tiles; t += kRedT) {
      const double2 v = *reinterpret_cast<const double2*>(partial + (t * M + g) * 2);
      cs.add(v.x);
      cq.add(v.y);
    }
  }
  part[tl][gl][0] = cs.s;
  part[tl][gl][1] = cs.c;
  part[tl][gl][2] = cq.s;
  part[tl][gl][3] = cq.c;
  __syncthreads();
  if (tl || g >= M) return;
  double s = K, q = K;   // g = 0: every trajectory starts in the ground state of H(0)
  if (g > 0) {
    for (int k = 1; k < kRedT; ++k) {
      cs.add(part[k][gl][0]);
      cs.c += part[k][gl][1];
      cq.add(part[k][gl][2]);
      cq.c += part[k][gl][3];
    }
    s = cs.value();
    q = cq.value();
  }
  if (sum) sum[g] = s;
  if (sumsq) sumsq[g] = q;
}

__global__ __launch_bounds__(kRedG * kRedT) void k_reduce_partials(const double* __restrict__ partial, int64_t tiles,
                                                                   int M, double K, double* __restrict__ sum,
                                                                   double* __restrict__ sumsq) {
  reduce_tiles(partial, tiles, M, K, sum, sumsq);
}

// Column-tile counts instantiated per level count and precision.
constexpr int kTQ[] = {1, 2, 3, 4, 5, 8};

__host__ __device__ constexpr bool tq_allowed(int NP, int TQ, bool f64) {
  return (NP <= 64) ? (TQ != 3 && TQ != 5 && !(f64 && NP == 64 && TQ == 8))
                    : (TQ <= 5 && !(f64 && TQ > 4));
}

// ------------------------------------------------------------- batched ----
// Many instances in few persistent launches.  Items (instance, tile) are grouped by
// padded level count and tile width; one launch per group (largest levels first)
// has its workgroups pull the group's items from an atomic queue (longest first)
// and run each with the trajectory kernel's tile body, wavefront count and
// occupancy floor.
struct BatchItem {
  int inst;
  int tile;
};

constexpr int kLevelClasses[] = {256, 128, 64, 32, 16};   // launch order
constexpr int kTileClasses[] = {1, 2, 4, 8};              // column tiles
constexpr int kNumClasses = 20;                           // (levels, tile) groups

__global__ void k_batch_reset(int* counter, int n) {
  if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < n) counter[threadIdx.x] = 0;
}

// BF16 runs of 16-level instances use the K = 16 MFMA, as in the single-instance launch
template <int NP, class Mode>
using BatchMode = typename std::conditional<NP == 16 && Mode::KC == 32, ModeBF16K16, Mode>::type;

// column tiles a batch may use: 1, 2, 4, 8 up to 64 levels, 1, 2 above
__host__ __device__ constexpr bool batch_tq(int NP, int TQ, bool f64) {
  return tq_allowed(NP, TQ, f64) && ((NP <= 64) ? (TQ == 1 || TQ == 2 || TQ == 4 || TQ == 8) : (TQ == 1 || TQ == 2));
}

template <int NP, int TQ, class Mode>
__global__ __launch_bounds__((Tile<NP, TQ, BatchMode<NP, Mode>>::WV * 64))
__attribute__((amdgpu_waves_per_eu(min_waves_per_simd<NP, BatchMode<NP, Mode>>()))) void k_batch(
    const StepArgs* __restrict__ args, const BatchItem* __restrict__ items, int n_items, int* counter) {
  using Body = Tile<NP, TQ, BatchMode<NP, Mode>>;
  __shared__ typename Body::Shared sh;
  __shared__ int s_item;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(counter, 1);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
    if (it >= n_items) break;
    const int inst = __builtin_amdgcn_readfirstlane(items[it].inst);
    const int tile = __builtin_amdgcn_readfirstlane(items[it].tile);
    Body::run(*reinterpret_cast<CArgs*>(reinterpret_cast<uintptr_t>(args + inst)), tile, sh);
  }
}

__global__ __launch_bounds__(kRedG * kRedT) void k_reduce_batch(const StepArgs* __restrict__ args) {
  const StepArgs& a = args[blockIdx.y];
  reduce_tiles(a.partial, a.tiles, a.M, static_cast<double>(a.K), a.pgs_sum, a.pgs_sumsq);
}

template <class Mode, int NP>
hipError_t launch_tq(int TQ, const StepArgs& a, int64_t blocks, hipStream_t st) {
  constexpr bool f64 = sizeof(typename Mode::T) == 8;
#define AQT_CASE(tq)                                                                          \
  if constexpr (tq_allowed(NP, tq, f64)) {                                                    \
    if (TQ == tq) {                                                                           \
      hipLaunchKernelGGL((k_trajectories<NP, tq, Mode>), dim3(static_cast<unsigned>(blocks)), \
                         dim3(Tile<NP, tq, Mode>::WV * 64), 0, st, a);                         \
      return hipGetLastError();                                                               \
    }                                                                                         \
  }
  AQT_CASE(1) AQT_CASE(2) AQT_CASE(3) AQT_CASE(4) AQT_CASE(5) AQT_CASE(8)
#undef AQT_CASE
  return hipErrorInvalidValue;
}

template <class Mode>
hipError_t launch_mode(int NP, int TQ, const StepArgs& a, int64_t blocks, hipStream_t st) {
  switch (NP) {
    case 16:
      if constexpr (Mode::KC == 4) return launch_tq<Mode, 16>(TQ, a, blocks, st);
      else return launch_tq<ModeBF16K16, 16>(TQ, a, blocks, st);
    case 32: return launch_tq<Mode, 32>(TQ, a, blocks, st);
    case 64: return launch_tq<Mode, 64>(TQ, a, blocks, st);
    case 128: return launch_tq<Mode, 128>(TQ, a, blocks, st);
    case 256: return launch_tq<Mode, 256>(TQ, a, blocks, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

namespace {

// Launches of one run: widths (column tiles of 8 trajectories per workgroup) and
// workgroups, widest first.
struct TilePlan {
  int n = 0;
  int tq[8];
  int64_t wgs[8];
  int width = 0;   // StepArgs::width of its tiles
  int64_t tiles() const {
    int64_t t = 0;
    for (int i = 0; i < n; ++i) t += wgs[i];
    return t;
  }
  void add(int w, int64_t count) {
    tq[n] = w;
    wgs[n++] = count;
  }
};

// Width of the explicit `tile` parameter (trajectories per workgroup); 0 if unsupported.
int explicit_tq(int NP, int precision, int tile) {
  const int tq = tile / 8;
  const bool f64 = precision == AQT_FP64;
  if (tile % 8 || !(tq == 1 || tq == 2 || tq == 4 || tq == 5 || tq == 8)) return 0;
  if (NP > 64 && f64 && tq > 2) return 0;   // 24 and 32 are chosen by plan_tiles only
  return tq_allowed(NP, tq, f64) ? tq : 0;
}

// Explicit tiles of half a column tile, as small launches up to kWaveLevels levels take them.
bool explicit_narrow(int NP, int tile) { return tile == 4 && NP <= kWaveLevels; }

// Split of K trajectories over the chip.  One-wavefront tiles: 8 trajectories while the
// launch fits the chip at once (two wavefronts per SIMD), else 16; 4 of the 8 columns while that
// fits, so that all crossings of a step are handled in one pass of four lane segments (32 levels FP32, us a step:
// 16000 trajectories 4.3 with 8, 5.1 with 16, 8.1 with 32; 10^5: 24.7, 18.5, 19.4 and 19.9
// with 64).  At 64 levels several workgroups share a CU: one launch with the widest tile
// that still gives every CU a workgroup.  Above, a CU holds
// one workgroup, so a launch takes rounds of one tile per CU and a round costs the step
// time of its width whether or not the CUs are full: the run is cut into the cheapest set
// of widths whose sum covers the column tiles that fall to each CU.  Step times in
// 0.1 us, measured at 256 levels on the 2000-point anneal: FP64 rises linearly (the GEMM
// binds), so what counts is not to pay for idle columns: 10^4 trajectories (4.9 columns a
// CU) take 3 + 2 (46.2 us a step) instead of three rounds of 2 (56.8); FP32 and BF16 gain
// from width up to 5 (4096 FP32 trajectories on 256 tiles of 16: 11.1 us instead of 19.1 on 128
// tiles of 32).  At 128 levels a step of 1 to 5 columns takes, in the same unit, FP64 44, 69, 94
// (up to 3), FP32 34, 49, 62, 74, 87 and BF16 26, 35, 41, 47, 55: for up to 8 columns a CU the
// sets chosen here are the best by these in FP32 and BF16 (or within 2%), and in FP64 but for 6 and
// 8 columns (2 + 2 + 2 instead of 3 + 3: 10%, 7%).
TilePlan plan_tiles(int NP, int precision, int64_t K, int cus) {
  const int64_t cols = (K + 7) / 8;
  const bool f64 = precision == AQT_FP64;
  TilePlan plan;
  if (NP <= kWaveLevels) {
    if (cols <= 4 * static_cast<int64_t>(cus)) {
      plan.width = 4;
      plan.add(1, (K + 3) / 4);
      return plan;
    }
    const int w = cols <= 8 * static_cast<int64_t>(cus) ? 1 : 2;
    plan.add(w, (cols + w - 1) / w);
    return plan;
  }
  if (NP <= 64) {
    int best = 1;
    for (int tq : kTQ)
      if (tq_allowed(NP, tq, f64) && (cols + tq - 1) / tq >= cus) best = tq;
    plan.add(best, (cols + best - 1) / best);
    return plan;
  }
  constexpr int kW = 5;
  static constexpr int kCost[3][kW] = {{119, 189, 287, 380, 1 << 20},   // FP64 (1, 2, 3, 4 columns)
                                       {69, 111, 151, 191, 233},        // FP32
                                       {51, 66, 82, 97, 114}};          // BF16
  const int* cost = kCost[f64 ? 0 : (precision == AQT_FP32 ? 1 : 2)];
  int widest = 1;
  for (int w = 1; w <= kW; ++w)
    if (tq_allowed(NP, w, f64)) widest = w;
  int64_t per_cu = (cols + cus - 1) / cus;   // columns each CU takes
  int64_t count[kW + 1] = {};
  constexpr int kExact = 40;                 // beyond this many columns, widest tiles first
  if (per_cu > kExact) {
    count[widest] = (per_cu - kExact + widest - 1) / widest;
    per_cu -= count[widest] * widest;
  }
  int best[kExact + 1] = {0}, with[kExact + 1] = {0};
  for (int c = 1; c <= per_cu; ++c) {
    best[c] = INT32_MAX;
    for (int w = 1; w <= widest; ++w) {
      const int v = best[c > w ? c - w : 0] + cost[w - 1];
      if (v <= best[c]) {
        best[c] = v;
        with[c] = w;
      }
    }
  }
  for (int64_t c = per_cu; c > 0; c -= with[c]) ++count[with[c]];
  int64_t left = cols;
  for (int w = widest; w >= 1 && left > 0; --w) {
    if (!count[w]) continue;
    const int64_t wgs = std::min<int64_t>(count[w] * cus, (left + w - 1) / w);
    plan.add(w, wgs);
    left -= wgs * w;
  }
  return plan;
}

// One launch of w column tiles a workgroup.
TilePlan single_width(const aqt_run_params* p, int w) {
  TilePlan plan;
  plan.add(w, (p->n_traj + 8 * w - 1) / (8 * w));
  return plan;
}

// The widest tile alone: the fewest per-tile sums.
TilePlan widest_plan(const aqt_ctx* ctx, const aqt_run_params* p) {
  int w = 1;
  for (int tq : kTQ)
    if (tq_allowed(ctx->NP, tq, p->precision == AQT_FP64)) w = tq;
  return single_width(p, w);
}

double partial_bytes(const aqt_ctx* ctx, const TilePlan& plan) {
  return static_cast<double>(plan.tiles()) * ctx->M * 2 * sizeof(double);
}

// Up to 32 levels the 16-trajectory tiles keep n_traj n_grid bytes of per-tile sums.  Beyond
// this many, tiles of 32 run instead: half the sums and the same time at such sizes (32 levels,
// 400000 trajectories, us a step with 16, 32 and 64: FP64 141, 143, 189; FP32 74, 69, 88; BF16
// 65, 60, 79).
constexpr double kMaxPartialBytes = 4.0 * (1u << 30);

// Plan of a run (explicit or chosen width); empty for an unsupported explicit tile.
TilePlan run_plan(const aqt_ctx* ctx, const aqt_run_params* p) {
  if (!p->tile) {
    const TilePlan plan = plan_tiles(ctx->NP, p->precision, p->n_traj, ctx->cus > 0 ? ctx->cus : 256);
    return (ctx->NP <= kWaveLevels && partial_bytes(ctx, plan) > kMaxPartialBytes) ? single_width(p, 4) : plan;
  }
  TilePlan plan;
  if (explicit_narrow(ctx->NP, p->tile)) {
    plan.width = p->tile;
    plan.add(1, (p->n_traj + p->tile - 1) / p->tile);
    return plan;
  }
  const int tq = explicit_tq(ctx->NP, p->precision, p->tile);
  if (tq) plan.add(tq, (p->n_traj + 8 * tq - 1) / (8 * tq));
  return plan;
}

// Enqueues the trajectory kernel and the observable reduction with the per-tile sums
// in `partial` ([tiles][M][2] doubles; every entry g >= 1 is written before it is read).
aqt_status enqueue_run(aqt_ctx* ctx, const aqt_run_params* p, const aqt_outputs* o, const TilePlan& plan,
                       double* partial) {
  const int prec = p->precision;
  const int64_t tiles = plan.tiles();
  StepArgs a{};
  a.M = ctx->M;
  a.M_run = ctx->M;
  a.NP = ctx->NP;
  a.tiles = tiles;
  a.pgs_sum = o->pgs_sum;
  a.pgs_sumsq = o->pgs_sumsq;
  a.n = ctx->n;
  a.nq = ctx->tab_nch;   // jump channels
  a.tbeg = ctx->tbeg.as<double>();
  a.tlen = ctx->tlen.as<double>();
  a.K = p->n_traj;
  a.seed = p->seed;
  a.iid = p->instance_id;
  a.traj0 = p->traj_offset;
  a.cap = p->record_capacity;
  a.dlt_a = ctx->pk_a.p;
  a.dlt_b = ctx->pk_b.p;
  a.dre = ctx->pk_dre.p;
  a.dim = ctx->pk_dim.p;
  a.cinit = ctx->cinit.as<double>();
  a.Gamma = ctx->Gamma.as<double>();
  a.d64re = ctx->dre.as<double>();
  a.d64im = ctx->dim.as<double>();
  a.R = ctx->R.as<double>();
  a.Rcol = ctx->Rcol.as<double>();
  a.ehalf = ctx->ehalf.as<double>();
  a.zdiag = ctx->zdiag.as<double>();
  a.chf = (prec == AQT_FP32) ? ctx->pk_ch.as<float4>() : nullptr;
  a.E = ctx->E.as<double>();
  a.gs = ctx->gs.as<int>();
  a.partial = partial;
  a.jump_totals = o->jump_totals;
  a.jump_count = o->jump_count;
  a.jumps = o->jumps;
  a.net_gs = o->net_gs;
  a.net_hist = o->net_hist;
  a.hist_lo = o->hist_lo;
  a.hist_hi = o->hist_hi;
  a.final_state = o->final_state;
  a.flags = ctx->run_flags.as<int>();

  hipError_t e = hipSuccess;
  for (int i = 0; i < plan.n && e == hipSuccess; ++i) {
    a.TQ = plan.tq[i];
    a.width = plan.width;
    if (prec == AQT_FP64) e = launch_mode<ModeF64>(ctx->NP, a.TQ, a, plan.wgs[i], ctx->stream);
    else if (prec == AQT_FP32) e = launch_mode<ModeF32>(ctx->NP, a.TQ, a, plan.wgs[i], ctx->stream);
    else e = launch_mode<ModeBF16>(ctx->NP, a.TQ, a, plan.wgs[i], ctx->stream);
    a.t_base += (plan.width ? plan.width : 8 * a.TQ) * plan.wgs[i];
    a.tile0 += plan.wgs[i];
  }
  if (e != hipSuccess) return ctx->fail(AQT_EHIP, std::string("trajectory kernel launch: ") + hipGetErrorString(e));
  if (o->pgs_sum || o->pgs_sumsq) {
    hipLaunchKernelGGL(k_reduce_partials, dim3((ctx->M + kRedG - 1) / kRedG), dim3(kRedG * kRedT), 0, ctx->stream,
                       partial, tiles, ctx->M, static_cast<double>(p->n_traj), o->pgs_sum, o->pgs_sumsq);
    e = hipGetLastError();
    if (e != hipSuccess) return ctx->fail(AQT_EHIP, std::string("reduction launch: ") + hipGetErrorString(e));
  }
  return AQT_OK;
}

// ---------------------------------------------------------- no allocation ----
// Per-tile observable sums of aqt_run_noalloc: a fixed buffer in device memory, one
// copy per device (held until the process ends).  Host code never passes `scratch`
// itself to a kernel: its device address comes from hipGetSymbolAddress, taken once
// per device with that device current, and only that address is used.
constexpr size_t kScratchBytes = static_cast<size_t>(AQT_NOALLOC_SCRATCH_BYTES);
static __device__ __align__(256) double scratch[kScratchBytes / sizeof(double)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};

}  // namespace

aqt_status launch_run(aqt_ctx* ctx, const aqt_run_params* p, const aqt_outputs* o) {
  const int prec = p->precision;
  aqt_status s = check_step_decay(ctx, prec);
  if (s != AQT_OK) return s;
  s = pack_for_precision(ctx, prec);
  if (s != AQT_OK) return s;
  TilePlan plan = run_plan(ctx, p);
  if (!plan.n) return ctx->fail(AQT_EINVAL, "unsupported tile size for this level count and precision");
  hipError_t e = ctx->partial.reserve(static_cast<size_t>(partial_bytes(ctx, plan)));
  for (int tq : kTQ) {   // a chosen width whose sums do not fit gives way to wider ones
    if (e == hipSuccess || p->tile) break;
    if (!tq_allowed(ctx->NP, tq, prec == AQT_FP64)) continue;
    const TilePlan wider = single_width(p, tq);
    if (wider.tiles() >= plan.tiles()) continue;
    (void)hipGetLastError();
    plan = wider;
    e = ctx->partial.reserve(static_cast<size_t>(partial_bytes(ctx, plan)));
  }
  if (e != hipSuccess) return ctx->fail(AQT_ENOMEM, "workspace allocation failed");
  return enqueue_run(ctx, p, o, plan, ctx->partial.as<double>());
}

aqt_status setup_noalloc_scratch(aqt_ctx* ctx) {
  const int dev = ctx->device;
  if (dev < 0 || dev >= kMaxDevices) return ctx->fail(AQT_EINVAL, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_done[dev]) {
    void* ptr = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));   // the device is current
    g_scratch_ptr[dev] = (g_scratch_err[dev] == hipSuccess) ? ptr : nullptr;
    g_scratch_done[dev] = true;
  }
  if (g_scratch_err[dev] != hipSuccess)
    return ctx->fail(AQT_EHIP, std::string("scratch address: ") + hipGetErrorString(g_scratch_err[dev]));
  return AQT_OK;
}

aqt_status launch_run_noalloc(aqt_ctx* ctx, const aqt_run_params* p, const aqt_outputs* o) {
  const int prec = p->precision;
  aqt_status s = check_step_decay(ctx, prec);
  if (s != AQT_OK) return s;
  if (ctx->packed_for != prec)
    return ctx->fail(AQT_ESTATE, "the step operands of this precision are not resident; one aqt_run in this "
                                 "precision after the tables were loaded packs them");
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (ctx->device >= 0 && ctx->device < kMaxDevices) base = g_scratch_ptr[ctx->device];
  }
  if (!base) return ctx->fail(AQT_ESTATE, "the device scratch buffer has no address (aqt_create did not set it up)");
  TilePlan plan = run_plan(ctx, p);
  if (!plan.n) return ctx->fail(AQT_EINVAL, "unsupported tile size for this level count and precision");
  if (!p->tile && partial_bytes(ctx, plan) > static_cast<double>(kScratchBytes)) plan = widest_plan(ctx, p);
  const double need = partial_bytes(ctx, plan);
  if (need > static_cast<double>(kScratchBytes))
    return ctx->fail(AQT_EINVAL, "the run needs " + std::to_string(static_cast<long long>(need)) +
                                     " bytes of per-tile sums (tiles x n_grid x 16), more than the " +
                                     std::to_string(kScratchBytes) + "-byte no-allocation buffer");
  return enqueue_run(ctx, p, o, plan, static_cast<double*>(base));
}

}  // namespace aqt

// ================================================================ batches ===
struct aqt_batch {
  int device = 0;
  hipStream_t capture_stream = nullptr;   // private stream used only for graph capture
  hipStream_t stream = nullptr;           // launch stream (the first context's)
  std::string err;
  int precision = AQT_FP32;
  int n = 0;
  std::vector<aqt_ctx*> ctxs;
  std::vector<aqt::StepArgs> hargs;
  std::vector<int> tiles_per_inst;        // trajectories per workgroup tile chosen per instance
  aqt::DevBuf dargs, ditems, dcounter;
  aqt::DevBuf sums;                       // per-tile sums of every instance
  int n_items = 0;
  int class_off[20] = {};                 // items of each (levels, tile) group
  int class_cnt[20] = {};
  int class_grid[20] = {};                // persistent workgroups per group launch
  // groups after the first run on side streams forked from and joined back into the
  // launch stream, so that one group's tail overlaps the next group's work
  hipStream_t side[3] = {nullptr, nullptr, nullptr};
  hipEvent_t fork = nullptr;
  hipEvent_t join[3] = {nullptr, nullptr, nullptr};
  bool use_graph = false;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  aqt_status fail(aqt_status s, const std::string& m) {
    err = m;
    return s;
  }
};

namespace aqt {
namespace {

// Items of a launch per (levels, tile) group: [off, off + cnt) of the item array.
struct ClassSpans {
  int off[kNumClasses] = {};
  int cnt[kNumClasses] = {};
};

int batch_class(int NP, int TQ) {
  int l = -1, t = -1;
  for (int c = 0; c < 5; ++c)
    if (kLevelClasses[c] == NP) l = c;
  for (int c = 0; c < 4; ++c)
    if (kTileClasses[c] == TQ) t = c;
  return (l < 0 || t < 0) ? -1 : 4 * l + t;
}

// Calls f.template operator()<NP, TQ>() for the (levels, tile) group c, if the batch allows it.
template <class Mode, class F>
hipError_t with_class(int c, const F& f) {
  constexpr bool f64 = sizeof(typename Mode::T) == 8;
  hipError_t e = hipErrorInvalidValue;
  auto tq = [&](auto np_tag) {
    constexpr int NP = decltype(np_tag)::value;
    switch (kTileClasses[c % 4]) {
      case 1: if constexpr (batch_tq(NP, 1, f64)) e = f.template operator()<NP, 1>(); break;
      case 2: if constexpr (batch_tq(NP, 2, f64)) e = f.template operator()<NP, 2>(); break;
      case 4: if constexpr (batch_tq(NP, 4, f64)) e = f.template operator()<NP, 4>(); break;
      default: if constexpr (batch_tq(NP, 8, f64)) e = f.template operator()<NP, 8>(); break;
    }
  };
  switch (kLevelClasses[c / 4]) {
    case 256: tq(std::integral_constant<int, 256>{}); break;
    case 128: tq(std::integral_constant<int, 128>{}); break;
    case 64: tq(std::integral_constant<int, 64>{}); break;
    case 32: tq(std::integral_constant<int, 32>{}); break;
    default: tq(std::integral_constant<int, 16>{}); break;
  }
  return e;
}

template <class Mode>
struct LaunchGroup {
  const StepArgs* dargs;
  const BatchItem* items;
  int n;
  int* counter;
  int grid;
  hipStream_t st;
  template <int NP, int TQ>
  hipError_t operator()() const {
    hipLaunchKernelGGL((k_batch<NP, TQ, Mode>), dim3(grid), dim3(Tile<NP, TQ, BatchMode<NP, Mode>>::WV * 64), 0, st,
                       dargs, items, n, counter);
    return hipGetLastError();
  }
};

template <class Mode>
struct GroupOccupancy {
  int* blocks;
  template <int NP, int TQ>
  hipError_t operator()() const {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch<NP, TQ, Mode>,
                                                        Tile<NP, TQ, BatchMode<NP, Mode>>::WV * 64, 0);
  }
};

// One reset of the group counters, then one persistent launch per non-empty group:
// the first on st, the others on the side streams (forked after the reset, joined
// back into st), so the groups run concurrently.
template <class Mode>
hipError_t enqueue_mode(const aqt_batch* b, const StepArgs* dargs, const BatchItem* items, const ClassSpans& sp,
                        int* counter, hipStream_t st) {
  hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(64), 0, st, counter, kNumClasses);
  hipError_t e = hipGetLastError();
  bool forked = false, used[3] = {false, false, false};
  int k = 0;   // non-empty groups so far
  for (int c = 0; c < kNumClasses && e == hipSuccess; ++c) {
    if (!sp.cnt[c]) continue;
    hipStream_t s = st;
    if (k > 0 && b->side[0]) {
      if (!forked) {
        e = hipEventRecord(b->fork, st);
        forked = true;
      }
      const int j = (k - 1) % 3;
      if (e == hipSuccess && !used[j]) {
        e = hipStreamWaitEvent(b->side[j], b->fork, 0);
        used[j] = true;
      }
      s = b->side[j];
    }
    ++k;
    if (e != hipSuccess) break;
    e = with_class<Mode>(c, LaunchGroup<Mode>{dargs, items + sp.off[c], sp.cnt[c], counter + c, b->class_grid[c], s});
  }
  for (int j = 0; j < 3 && e == hipSuccess; ++j)
    if (used[j]) {
      e = hipEventRecord(b->join[j], b->side[j]);
      if (e == hipSuccess) e = hipStreamWaitEvent(st, b->join[j], 0);
    }
  return e;
}

hipError_t enqueue_batch(const aqt_batch* b, const StepArgs* dargs, const BatchItem* items, const ClassSpans& sp,
                         int* counter, hipStream_t st) {
  if (b->precision == AQT_FP64) return enqueue_mode<ModeF64>(b, dargs, items, sp, counter, st);
  if (b->precision == AQT_FP32) return enqueue_mode<ModeF32>(b, dargs, items, sp, counter, st);
  return enqueue_mode<ModeBF16>(b, dargs, items, sp, counter, st);
}

// Resident workgroups per CU of group c's kernel (0 if the group is not allowed).
template <class Mode>
int class_occupancy(int c) {
  int blocks = 0;
  const hipError_t e = with_class<Mode>(c, GroupOccupancy<Mode>{&blocks});
  return e == hipSuccess ? (blocks > 0 ? blocks : 1) : 0;
}

int class_occupancy_for(int c, int precision) {
  if (precision == AQT_FP64) return class_occupancy<ModeF64>(c);
  if (precision == AQT_FP32) return class_occupancy<ModeF32>(c);
  return class_occupancy<ModeBF16>(c);
}

bool batch_tq_ok(int NP, int tq, int precision) {
  return batch_class(NP, tq) >= 0 && batch_tq(NP, tq, precision == AQT_FP64);
}

// Items of all instances grouped by (levels, tile), largest levels first, longest first
// within a group (work per item ~ TQ * (M-1) * NP^2).
std::vector<BatchItem> build_items(const std::vector<StepArgs>& args, ClassSpans* sp) {
  std::vector<std::pair<double, BatchItem>> v[kNumClasses];
  for (int i = 0; i < static_cast<int>(args.size()); ++i) {
    const StepArgs& a = args[i];
    const double w = static_cast<double>(a.TQ) * (a.M_run - 1) * (64.0 + static_cast<double>(a.NP) * a.NP);
    const int c = batch_class(a.NP, a.TQ);
    for (int64_t t = 0; t < a.tiles; ++t) v[c].push_back({w, BatchItem{i, static_cast<int>(t)}});
  }
  std::vector<BatchItem> out;
  for (int c = 0; c < kNumClasses; ++c) {
    std::stable_sort(v[c].begin(), v[c].end(), [](const auto& x, const auto& y) { return x.first > y.first; });
    sp->off[c] = static_cast<int>(out.size());
    sp->cnt[c] = static_cast<int>(v[c].size());
    for (auto& p : v[c]) out.push_back(p.second);
  }
  return out;
}

// Trajectories a tile of a batch's instances up to kWaveLevels levels, from the 8-trajectory
// columns of all of them.  A one-wavefront tile handles its crossings one pass after another, so
// what ends a batch is the jumps of its longest anneals, and narrow tiles spread them.  4 (half
// the columns, as in plan_tiles) up to 8 columns a CU: 24 instances, 200 points, with 4 and with 8
// take 5.1 and 9.0 ms in FP64 at one column a CU, 6.1 and 10.1 at 8, FP32 3.7 and 6.3, 4.0 and 6.7
// (at 16 a CU 4 is still ahead, 7.4 to 10.4; the line is as far as small batches were tried when
// it was drawn).  8 up to 256 a CU, 16 beyond (ms with 8, 16
// and 32; 24 instances, 24 a CU: FP64 11.3, 18.6, 32.9, FP32 7.1, 12.4, 22.4; 60 instances, 240 a
// CU, 100 points: 58.9, 62.8, 74.6 and 34.7, 37.5, 43.7; 24 instances, 469 a CU: 74.3, 69.3, 71.6
// and 43.4, 40.7, 44.7).  Timing the first steps, which have few jumps, picks wider tiles than
// that (60 instances of 2048, 200 points, BF16: 27.0 ms against 14.4), so they are not timed.
int wave_batch_tile(int64_t cols, int cus) {
  return cols <= 8 * static_cast<int64_t>(cus) ? 4 : cols <= 256 * static_cast<int64_t>(cus) ? 8 : 16;
}

// Time each allowed tile size per level count above kWaveLevels on a shortened anneal (outputs
// discarded) and keep the fastest per trajectory-step.
aqt_status autotune(aqt_batch* b) {
  const int tune_steps = 24;
  std::vector<int> nps;
  for (auto& a : b->hargs)
    if (a.NP > kWaveLevels && std::find(nps.begin(), nps.end(), a.NP) == nps.end()) nps.push_back(a.NP);
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
    return b->fail(AQT_EHIP, "event creation failed");
  aqt_status st = AQT_OK;
  DevBuf dargs, ditems, dctr, scratch;
  if (dctr.reserve(kNumClasses * sizeof(int)) != hipSuccess) st = b->fail(AQT_ENOMEM, "tuning allocation failed");
  for (int np : nps) {
    if (st != AQT_OK) break;
    double best_t = 1e300;
    int best_tq = 1;
    for (int tq : kTQ) {
      if (!batch_tq_ok(np, tq, b->precision)) continue;
      std::vector<StepArgs> ta;
      size_t scratch_need = 0;
      double traj_steps = 0.0;
      for (size_t i = 0; i < b->hargs.size(); ++i) {
        StepArgs a = b->hargs[i];
        if (a.NP != np) continue;
        a.TQ = tq;
        a.M_run = std::min(a.M, tune_steps + 1);
        a.tiles = (a.K + 8 * tq - 1) / (8 * tq);
        a.jump_totals = nullptr;
        a.jump_count = nullptr;
        a.jumps = nullptr;
        a.cap = 0;
        a.net_gs = nullptr;
        a.net_hist = nullptr;
        a.final_state = nullptr;
        a.pgs_sum = a.pgs_sumsq = nullptr;
        scratch_need = std::max(scratch_need, static_cast<size_t>(a.tiles) * a.M * 2 * sizeof(double));
        traj_steps += static_cast<double>(a.K) * (a.M_run - 1);
        ta.push_back(a);
      }
      if (scratch.reserve(scratch_need) != hipSuccess) {
        st = b->fail(AQT_ENOMEM, "tuning allocation failed");
        break;
      }
      for (auto& a : ta) a.partial = scratch.as<double>();   // shared scratch, contents discarded
      ClassSpans sp;
      std::vector<BatchItem> items = build_items(ta, &sp);
      if (dargs.reserve(ta.size() * sizeof(StepArgs)) != hipSuccess ||
          ditems.reserve(items.size() * sizeof(BatchItem)) != hipSuccess) {
        st = b->fail(AQT_ENOMEM, "tuning allocation failed");
        break;
      }
      (void)hipMemcpyAsync(dargs.p, ta.data(), ta.size() * sizeof(StepArgs), hipMemcpyHostToDevice, b->stream);
      (void)hipMemcpyAsync(ditems.p, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice, b->stream);
      double t_ms = 1e300;
      for (int rep = 0; rep < 2; ++rep) {
        (void)hipEventRecord(e0, b->stream);
        if (enqueue_batch(b, dargs.as<StepArgs>(), ditems.as<BatchItem>(), sp, dctr.as<int>(), b->stream) !=
            hipSuccess) {
          st = b->fail(AQT_EHIP, "tuning launch failed");
          break;
        }
        (void)hipEventRecord(e1, b->stream);
        if (hipEventSynchronize(e1) != hipSuccess) {
          st = b->fail(AQT_EHIP, "tuning run failed");
          break;
        }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        if (rep) t_ms = std::min(t_ms, static_cast<double>(ms));   // first repetition warms up
      }
      if (st != AQT_OK) break;
      const double per = t_ms / traj_steps;
      if (per < best_t) {
        best_t = per;
        best_tq = tq;
      }
    }
    for (size_t i = 0; i < b->hargs.size(); ++i)
      if (b->hargs[i].NP == np && b->tiles_per_inst[i] == 0) b->tiles_per_inst[i] = 8 * best_tq;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return st;
}

}  // namespace
}  // namespace aqt

extern "C" {

aqt_status aqt_batch_create(aqt_batch** out, aqt_ctx* const* ctxs, int n, const aqt_run_params* params,
                            const aqt_outputs* outs, int flags) {
  using namespace aqt;
  if (!out) return AQT_EINVAL;
  *out = nullptr;
  if (!ctxs || !params || !outs || n < 1) return AQT_EINVAL;
  aqt_batch* b = new (std::nothrow) aqt_batch();
  if (!b) return AQT_ENOMEM;
  auto bail = [&](aqt_status s) {
    if (s != AQT_OK) {
      // keep the object so the caller can read the message, then destroy it
      *out = b;
      return s;
    }
    return s;
  };
  b->n = n;
  b->ctxs.assign(ctxs, ctxs + n);
  b->device = ctxs[0] ? ctxs[0]->device : 0;
  b->stream = ctxs[0] ? ctxs[0]->stream : nullptr;
  b->precision = params[0].precision;
  b->use_graph = (flags & 1) != 0;
  const bool tune = (flags & 2) != 0;
  if (hipSetDevice(b->device) != hipSuccess) return bail(b->fail(AQT_EHIP, "hipSetDevice failed"));
  if (hipEventCreateWithFlags(&b->fork, hipEventDisableTiming) != hipSuccess)
    return bail(b->fail(AQT_EHIP, "event creation failed"));
  for (int j = 0; j < 3; ++j)
    if (hipStreamCreateWithFlags(&b->side[j], hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&b->join[j], hipEventDisableTiming) != hipSuccess)
      return bail(b->fail(AQT_EHIP, "stream creation failed"));
  for (int i = 0; i < n; ++i) {
    aqt_ctx* c = ctxs[i];
    if (!c) return bail(b->fail(AQT_EINVAL, "null context in batch"));
    if (!c->have_tables) return bail(b->fail(AQT_ESTATE, "every context needs tables before batching"));
    if (c->device != b->device) return bail(b->fail(AQT_EINVAL, "all contexts must be on one device"));
    if (params[i].precision != b->precision) return bail(b->fail(AQT_EINVAL, "one precision per batch"));
    if (params[i].n_traj < 1) return bail(b->fail(AQT_EINVAL, "n_traj must be >= 1"));
    if (params[i].record_capacity > 0 && !outs[i].jumps)
      return bail(b->fail(AQT_EINVAL, "record_capacity > 0 needs a jumps buffer"));
    if (outs[i].net_hist && outs[i].hist_hi < outs[i].hist_lo) return bail(b->fail(AQT_EINVAL, "hist_hi < hist_lo"));
    if (params[i].tile && !explicit_narrow(c->NP, params[i].tile) && (params[i].tile % 8 || !batch_tq_ok(c->NP, params[i].tile / 8, b->precision)))
      return bail(b->fail(AQT_EINVAL, "unsupported tile size in batch"));
    if (batch_class(c->NP, 1) < 0) return bail(b->fail(AQT_EINVAL, "unsupported level count in batch"));
    aqt_status s = check_step_decay(c, b->precision);
    if (s == AQT_OK) s = pack_for_precision(c, b->precision);
    if (s != AQT_OK) return bail(b->fail(s, c->err));
  }
  for (int i = 0; i < n; ++i)   // packed on the members' streams, read on the first one's
    if (hipStreamSynchronize(ctxs[i]->stream) != hipSuccess) return bail(b->fail(AQT_EHIP, "packing failed"));
  b->tiles_per_inst.assign(n, 0);
  for (int i = 0; i < n; ++i) b->tiles_per_inst[i] = params[i].tile;
  // provisional args (TQ fixed below)
  b->hargs.resize(n);
  for (int i = 0; i < n; ++i) {
    aqt_ctx* c = ctxs[i];
    StepArgs a{};
    a.M = c->M;
    a.M_run = c->M;
    a.n = c->n;
    a.nq = c->tab_nch;   // jump channels
    a.NP = c->NP;
    a.tbeg = c->tbeg.as<double>();
    a.tlen = c->tlen.as<double>();
    a.K = params[i].n_traj;
    a.seed = params[i].seed;
    a.iid = params[i].instance_id;
    a.traj0 = params[i].traj_offset;
    a.cap = params[i].record_capacity;
    a.dlt_a = c->pk_a.p;
    a.dlt_b = c->pk_b.p;
    a.dre = c->pk_dre.p;
    a.dim = c->pk_dim.p;
    a.cinit = c->cinit.as<double>();
    a.Gamma = c->Gamma.as<double>();
    a.d64re = c->dre.as<double>();
    a.d64im = c->dim.as<double>();
    a.R = c->R.as<double>();
    a.Rcol = c->Rcol.as<double>();
    a.ehalf = c->ehalf.as<double>();
    a.zdiag = c->zdiag.as<double>();
    a.E = c->E.as<double>();
    a.gs = c->gs.as<int>();
    a.jump_totals = outs[i].jump_totals;
    a.jump_count = outs[i].jump_count;
    a.jumps = outs[i].jumps;
    a.net_gs = outs[i].net_gs;
    a.net_hist = outs[i].net_hist;
    a.hist_lo = outs[i].hist_lo;
    a.hist_hi = outs[i].hist_hi;
    a.final_state = outs[i].final_state;
    a.pgs_sum = outs[i].pgs_sum;
    a.pgs_sumsq = outs[i].pgs_sumsq;
    a.flags = c->run_flags.as<int>();
    a.TQ = 1;
    a.tiles = (a.K + 7) / 8;
    b->hargs[i] = a;
  }
  const int cus = ctxs[0]->cus > 0 ? ctxs[0]->cus : 256;
  for (int c = 0; c < kNumClasses; ++c) b->class_grid[c] = cus * class_occupancy_for(c, b->precision);
  if (tune) {
    aqt_status s = autotune(b);
    if (s != AQT_OK) return bail(s);
  }
  int64_t wave_cols = 0;   // 8-trajectory columns of the instances that take one-wavefront tiles
  for (int i = 0; i < n; ++i)
    if (b->hargs[i].NP <= kWaveLevels) wave_cols += (b->hargs[i].K + 7) / 8;
  for (int i = 0; i < n; ++i) {
    const StepArgs& a = b->hargs[i];
    int& tile = b->tiles_per_inst[i];
    if (!tile && a.NP <= kWaveLevels) tile = wave_batch_tile(wave_cols, cus);
    if (!tile) {
      // heuristic: the largest allowed tile that still gives every CU several items
      int best = 1;
      for (int tq : kTQ)
        if (batch_tq_ok(a.NP, tq, b->precision)) best = tq;
      tile = 8 * std::min(best, 4);
    }
  }
  // per-tile sums of every instance, in one buffer of the batch: the contexts' own ones move with
  // their runs.  Chosen widths whose sums do not fit give way to wider ones.
  std::vector<size_t> sums(n);
  for (;;) {
    size_t need = 0;
    for (int i = 0; i < n; ++i) {
      StepArgs& a = b->hargs[i];
      const int tile = b->tiles_per_inst[i];
      a.TQ = std::max(1, tile / 8);
      a.width = tile < 8 ? tile : 0;
      a.tiles = (a.K + tile - 1) / tile;
      sums[i] = need;
      need += (static_cast<size_t>(a.tiles) * a.M * 2 * sizeof(double) + 255) & ~size_t(255);
    }
    if (b->sums.reserve(need) == hipSuccess) break;
    (void)hipGetLastError();
    bool wider = false;
    for (int i = 0; i < n; ++i)
      if (!params[i].tile && batch_tq_ok(b->hargs[i].NP, 2 * b->tiles_per_inst[i] / 8, b->precision)) {
        b->tiles_per_inst[i] *= 2;
        wider = true;
      }
    if (!wider) return bail(b->fail(AQT_ENOMEM, "workspace allocation failed"));
  }
  for (int i = 0; i < n; ++i) b->hargs[i].partial = reinterpret_cast<double*>(b->sums.as<char>() + sums[i]);
  ClassSpans sp;
  std::vector<BatchItem> items = build_items(b->hargs, &sp);
  b->n_items = static_cast<int>(items.size());
  for (int c = 0; c < kNumClasses; ++c) {
    b->class_off[c] = sp.off[c];
    b->class_cnt[c] = sp.cnt[c];
  }
  if (b->dargs.reserve(n * sizeof(StepArgs)) != hipSuccess ||
      b->ditems.reserve(items.size() * sizeof(BatchItem)) != hipSuccess ||
      b->dcounter.reserve(kNumClasses * sizeof(int)) != hipSuccess)
    return bail(b->fail(AQT_ENOMEM, "batch allocation failed"));
  if (hipMemcpy(b->dargs.p, b->hargs.data(), n * sizeof(StepArgs), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(b->ditems.p, items.data(), items.size() * sizeof(BatchItem), hipMemcpyHostToDevice) != hipSuccess)
    return bail(b->fail(AQT_EHIP, "batch upload failed"));
  if (b->use_graph) {
    if (hipStreamCreate(&b->capture_stream) != hipSuccess) return bail(b->fail(AQT_EHIP, "stream creation failed"));
    if (hipStreamBeginCapture(b->capture_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
      return bail(b->fail(AQT_EHIP, "graph capture failed to start"));
    hipError_t e = enqueue_batch(b, b->dargs.as<StepArgs>(), b->ditems.as<BatchItem>(), sp, b->dcounter.as<int>(),
                                 b->capture_stream);
    int maxM = 0;
    for (auto& a : b->hargs) maxM = std::max(maxM, a.M);
    hipLaunchKernelGGL(k_reduce_batch, dim3((maxM + kRedG - 1) / kRedG, n), dim3(kRedG * kRedT), 0, b->capture_stream,
                       b->dargs.as<StepArgs>());
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(b->capture_stream, &g);
    if (e != hipSuccess || e2 != hipSuccess || !g) return bail(b->fail(AQT_EHIP, "graph capture failed"));
    b->graph = g;
    if (hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0) != hipSuccess)
      return bail(b->fail(AQT_EHIP, "graph instantiation failed"));
  }
  *out = b;
  return AQT_OK;
}

aqt_status aqt_batch_launch(aqt_batch* b) {
  using namespace aqt;
  if (!b) return AQT_EINVAL;
  if (!b->dargs.p) return b->fail(AQT_ESTATE, "batch was not created successfully");
  if (hipSetDevice(b->device) != hipSuccess) return b->fail(AQT_EHIP, "hipSetDevice failed");
  if (b->use_graph) {
    if (hipGraphLaunch(b->exec, b->stream) != hipSuccess) return b->fail(AQT_EHIP, "graph launch failed");
    return AQT_OK;
  }
  ClassSpans sp;
  for (int c = 0; c < kNumClasses; ++c) {
    sp.off[c] = b->class_off[c];
    sp.cnt[c] = b->class_cnt[c];
  }
  if (enqueue_batch(b, b->dargs.as<StepArgs>(), b->ditems.as<BatchItem>(), sp, b->dcounter.as<int>(), b->stream) !=
      hipSuccess)
    return b->fail(AQT_EHIP, "batch launch failed");
  int maxM = 0;
  for (auto& a : b->hargs) maxM = std::max(maxM, a.M);
  hipLaunchKernelGGL(k_reduce_batch, dim3((maxM + kRedG - 1) / kRedG, b->n), dim3(kRedG * kRedT), 0, b->stream,
                     b->dargs.as<StepArgs>());
  if (hipGetLastError() != hipSuccess) return b->fail(AQT_EHIP, "batch reduction launch failed");
  return AQT_OK;
}

aqt_status aqt_batch_tiles(const aqt_batch* b, int32_t* tile_per_instance) {
  if (!b || !tile_per_instance) return AQT_EINVAL;
  for (int i = 0; i < b->n; ++i) tile_per_instance[i] = b->tiles_per_inst.empty() ? 0 : b->tiles_per_inst[i];
  return AQT_OK;
}

const char* aqt_batch_last_error(const aqt_batch* b) { return b ? b->err.c_str() : "null batch"; }

void aqt_batch_destroy(aqt_batch* b) {
  if (!b) return;
  (void)hipSetDevice(b->device);
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  else (void)hipDeviceSynchronize();
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  if (b->capture_stream) (void)hipStreamDestroy(b->capture_stream);
  for (int j = 0; j < 3; ++j) {
    if (b->side[j]) (void)hipStreamSynchronize(b->side[j]);
    if (b->side[j]) (void)hipStreamDestroy(b->side[j]);
    if (b->join[j]) (void)hipEventDestroy(b->join[j]);
  }
  if (b->fork) (void)hipEventDestroy(b->fork);
  delete b;
}

}  // extern "C"
