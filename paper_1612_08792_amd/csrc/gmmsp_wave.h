// Device helpers shared by the per-cell kernels (gmmsp_kernels.hip,
// gmmsp_cov3.hip, gmmsp_modes.hip): scalar-load pointers, FP64 constants and
// the wave-wide butterfly reduce-scatter.  Not part of the public ABI.
#pragma once

#include "gmmsp_internal.h"

namespace gmmsp {

#define AS4 __attribute__((address_space(4)))

// Uniform reads through the constant address space compile to scalar loads.
template <typename T>
__device__ __forceinline__ const AS4 T* cptr(const T* p) {
  return (const AS4 T*)(p);
}

constexpr double kLog2e = 1.4426950408889634074;
constexpr double kLn2 = 0.69314718055994530942;
constexpr double kLn2Pi = 1.8378770664093454836;

// The number of stopped images to pinned host memory (done_out, nullable), by
// the gather that follows the stop rule: a separate copy of the counter was a
// launch of its own, 3.5 us and a gap per pass of a run to the stop rule.
__device__ __forceinline__ void report_done(const DevPtrs& P, int32_t* done_out) {
  if (done_out && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(done_out, *P.n_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Butterfly reduce-scatter of per-lane sums across a 64-lane wave.  Each step
// halves the number of values: in a pair of partner lanes the one whose keep
// bit is 0 keeps the even entries summed with its partner's, the other the odd
// ones.  Keep bits go 5, 4, 3, 2, 1, 0: each step consumes the lowest bit of an
// entry's index, so after the six steps lane l holds the wave total of entry
// 64 q + bitrev6(l) at position q.

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// keep bit 5 (lanes 0-31 keep even entries): v_permlane32_swap exchanges the
// upper half of the first operand with the lower half of the second.
template <int N, int CAP>
__device__ __forceinline__ void bfly_swap32(float (&v)[CAP]) {
  static_assert(2 * ((N + 1) / 2) <= CAP, "butterfly reads past the array");
  if (N & 1) v[N] = 0.f;
#pragma unroll
  for (int i = 0; i < (N + 1) / 2; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * i]),
                                                    __float_as_uint(v[2 * i + 1]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

// keep bit 4: v_permlane16_swap exchanges odd 16-lane rows of the first operand
// with even rows of the second.
template <int N, int CAP>
__device__ __forceinline__ void bfly_swap16(float (&v)[CAP]) {
  static_assert(2 * ((N + 1) / 2) <= CAP, "butterfly reads past the array");
  if (N & 1) v[N] = 0.f;
#pragma unroll
  for (int i = 0; i < (N + 1) / 2; ++i) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[2 * i]),
                                                    __float_as_uint(v[2 * i + 1]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}

// keep bit BIT, partner given by the DPP control CTRL (an involution inside a
// 16-lane row that flips BIT and keeps the higher bits)
template <int N, int BIT, int CTRL, int CAP>
__device__ __forceinline__ void bfly_dpp(float (&v)[CAP], int lane) {
  static_assert(2 * ((N + 1) / 2) <= CAP, "butterfly reads past the array");
  const bool hi = ((lane >> BIT) & 1) != 0;
  if (N & 1) v[N] = 0.f;
#pragma unroll
  for (int i = 0; i < (N + 1) / 2; ++i) {
    const float a = v[2 * i], b = v[2 * i + 1];
    const float send = hi ? a : b;
    const float keep = hi ? b : a;
    v[i] = keep + dpp<CTRL>(send);
  }
}

// N per-lane values (the array holds at least 2 ceil(N / 2)); afterwards lane
// l holds the wave total of entry 64 q + bitrev6(l) in v[q].
template <int N, int CAP>
__device__ __forceinline__ void wave_reduce_scatter(float (&v)[CAP], int lane) {
  constexpr int N1 = (N + 1) / 2, N2 = (N1 + 1) / 2, N3 = (N2 + 1) / 2, N4 = (N3 + 1) / 2,
                N5 = (N4 + 1) / 2;
  bfly_swap32<N>(v);
  bfly_swap16<N1>(v);
  bfly_dpp<N2, 3, 0x128>(v, lane);  // row_ror:8, partner lane ^ 8
  bfly_dpp<N3, 2, 0x141>(v, lane);  // row_half_mirror, partner lane ^ 7
  bfly_dpp<N4, 1, 0x4E>(v, lane);   // quad_perm [2,3,0,1], partner lane ^ 2
  bfly_dpp<N5, 0, 0xB1>(v, lane);   // quad_perm [1,0,3,2], partner lane ^ 1
}

// ---------------------------------------------------------------------------
// Record offsets through LDS.  A VALU FMA reads at most one scalar register, so
// the offset of a whitening FMA (the addend beside a scalar record factor) has
// to come from a vector register.  The per-cell kernels keep the nine slots'
// offsets (at most 5 per record) in the wave's own block of LDS, kOffStride
// floats per slot, and read them back by broadcast each round: LDS reads issue
// on their own port, so this costs no VALU issue and no scalar registers.
// ---------------------------------------------------------------------------
constexpr int kOffStride = 8;
constexpr int kOffBlock = kSlots * kOffStride;  // floats per wave

// lanes 0..kSlots-1 copy the offsets idx[0..N) of their slot's record (rec_cell:
// the cell's slot-0 record, slot s at s * rec_stride floats); every lane of the wave may read the
// block after the call.  Only the calling wave touches its block, so a wave
// barrier orders the writes before the reads.
template <int N>
__device__ __forceinline__ void stage_offsets(float* woff, const float* rec_cell, size_t rec_stride,
                                              const int (&idx)[N], int lane) {
  static_assert(N <= 5, "at most five offsets per record");
  if (lane < kSlots) {
    const float* g = rec_cell + (size_t)lane * rec_stride;
#pragma unroll
    for (int i = 0; i < N; ++i) woff[lane * kOffStride + i] = g[idx[i]];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// the offsets of slot s: four by one 16-byte read, the fifth by one more
template <int N>
__device__ __forceinline__ void load_offsets(const float* woff, int s, float (&o)[N]) {
  const float4 q = *reinterpret_cast<const float4*>(woff + s * kOffStride);
  const float v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < N && i < 4; ++i) o[i] = v[i];
  if constexpr (N > 4) o[4] = woff[s * kOffStride + 4];
}

// ---------------------------------------------------------------------------
// Posterior export: 64 pixels of a cell, one per lane, nine floats each.  A
// lane storing its own nine floats would touch 64 different cache lines per
// store instruction; instead the wave turns the 64 x 9 values in its LDS and
// writes them in address order, 64 consecutive floats per store within a row
// of the cell (36 w bytes).  Bound by the 36 B written and 12 B read per
// pixel: on 32 x 3840x2160 (12.7 GB) the export takes 2.98 ms, 4.3 TB/s, the
// rate of a large copy; with each lane storing its own floats it took 4.50 ms
// (and the caller cleared the buffer first, 1.40 ms).
// ---------------------------------------------------------------------------
constexpr int kStageR = 64 * kSlots + 64;  // floats per wave: the values, the pixels' offsets

// v: the lane's nine posteriors; ofs: its pixel's offset (pixels) from the
// pixel that `dst` stands for; the first n lanes hold pixels (n may be <= 0:
// nothing is written).  Every lane of the wave calls it; st is the wave's own
// block.  The stride of nine floats per lane is odd, so neither the writes nor
// the reads of LDS conflict.
__device__ __forceinline__ void store_posteriors(float* st, float* dst, uint32_t ofs, int n, int lane,
                                                 const float (&v)[kSlots]) {
  uint32_t* so = reinterpret_cast<uint32_t*>(st + 64 * kSlots);
#pragma unroll
  for (int s = 0; s < kSlots; ++s) st[lane * kSlots + s] = v[s];
  so[lane] = ofs;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int it = 0; it < kSlots; ++it) {
    const int i = 64 * it + lane, k = i / kSlots;
    if (k < n) dst[(size_t)so[k] * kSlots + (i - k * kSlots)] = st[i];
  }
  // the next call's writes stay behind these reads
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Labels and posteriors of few cells: the four waves of a block share a cell, in
// rounds of pixels taken in turn.  A wave per cell leaves SIMDs without a wave
// below 1024 cells and, some way beyond, too few to hide the loads; but a cell of few
// rounds leaves most of four waves idle.  Labels with a wave each / shared, us: one
// 481x321 (442 cells, 3 rounds) 9.4 / 9.3, the split ones' posteriors 9.6 / 8.8;
// 1768 such cells 10.9 / 10.8, 2652 12.7 / 13.4, 3536 14.7 / 15.8; 3234 cells of one
// round 10.0 / 13.2; of four rounds 1980 12.9 / 12.6, 3960 18.1 / 19.4; of seven 3312
// 25.3 / 23.7, 4554 29.2 / 29.2.  The other models' rounds are half as long: 3x3
// block, 3094 cells of six rounds 16.1 / 14.8; 3234 of two 10.5 / 11.7.  Posteriors turn
// at the same places.  Beyond 4096 cells a wave each has the chip full: posteriors
// of 64 uneven images (46 773 cells) 283 / 298, of 32 x 3840x2160 2960 / 3190.
// ---------------------------------------------------------------------------
constexpr int kSplitCells = 4096;
constexpr int kSplitPerRound = 2048 / 3;

// round: pixels that a wave takes in one round
inline int label_waves(const DevPtrs& P, int round) {
  const int rounds = (P.cell_px + round - 1) / round;
  return rounds > 1 && P.n_cell <= kSplitCells && P.n_cell / kSplitPerRound < rounds ? 4 : 1;
}

// A pixel's log-likelihood term (log2 units) on a 2^-22 grid: the integer-valued
// FP64 sums of these are exact, so L does not depend on how the pixels are dealt.
__device__ __forceinline__ double ll_term(float lg) { return (double)rintf(lg * 0x1p22f); }

// L of the cell from the lanes' sums of ll_term, by the WPC waves that share it
// (four: the whole block calls it)
template <int WPC>
__device__ __forceinline__ void store_cell_ll(double* llp, double ll, double cst) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) ll += __shfl_xor(ll, m, 64);
  if constexpr (WPC == 1) {
    if ((threadIdx.x & 63) == 0) *llp = fma(kLn2, ll * 0x1p-22, cst);
  } else {
    static_assert(WPC == kWavesPerBlock, "a block per cell");
    __shared__ double s_ll[kWavesPerBlock];
    if ((threadIdx.x & 63) == 0) s_ll[threadIdx.x >> 6] = ll;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 1; k < WPC; ++k) ll += s_ll[k];
      *llp = fma(kLn2, ll * 0x1p-22, cst);
    }
  }
}

}  // namespace gmmsp
