// Segmentation accuracy measures of Sec. IV on gfx950, per image of a batch:
// boundary recall (BR), under-segmentation error (Eq. ue) and achievable
// segmentation accuracy (Eq. asa) of a superpixel label map against a
// ground-truth region map.
//
//   * a boundary pixel of a map is one whose right or lower neighbour carries
//     another value; a ground-truth boundary pixel is recovered when a
//     superpixel boundary pixel lies in the 5 x 5 square around it;
//   * UE = (1/N) sum_g sum_{k : 20 |s_k n s_g| > |s_k|} |s_k| - 1 (eps = 0.05
//     compared exactly), ASA = (1/N) sum_k max_g |s_k n s_g|.
//
// Superpixel labels lie in [0, S_b) (S_b given per image, by default the
// image's seed-grid size K_b) and region ids in [0, G_b); the overlaps
// |s_k n s_g| are counted per superpixel (S_b G_b < 2^31), see OverlapImg.
// Every result is a ratio of exact integer counts.
#include "gmmsp_internal.h"

#include <algorithm>

namespace gmmsp {

namespace {

constexpr int kT = 256;
constexpr int kR = 2;  // boundary tolerance in pixels (square window)

// The overlaps of an image, OverlapImg, an S x G table:
//   * G <= kDense, or G > kRatio S: the dense counts;
//   * else each superpixel's row holds kSlots16 keys (g + 1, 0 empty) and their
//     counts, 128 bytes, and only those are cleared and read.  A superpixel
//     that meets more regions than that is flagged, and its row cleared whole and
//     counted anew as a dense one by k_m_rescan.
// Up to 128 regions dense rows cost no more than slots (264 us with 16 slots for 84
// regions, 246 dense; 45 regions 255 and 229).  A dense table of
// 8 x 3840x2160 with 10 500 segments and some 2000 regions per image is 680 MB, of
// which almost all is zero: clearing it took 100 us, reading it 119 (261 us a call
// with slots).  With more than 8 S regions a superpixel meets more than 8 on average
// and often more than 16, and dense rows are not dearer before it does: 8.1 and 10.2
// S regions for 510 superpixels 279 and 279 us with slots, 256 and 257 dense (6.6 S:
// 257 with slots); 21 S, where most are flagged, 4250 and 281.
constexpr int kSlots16 = 16;
constexpr int kSlotInts = 2 * kSlots16;
constexpr int kDense = 128;

constexpr int kRatio = 8;

__host__ __device__ inline bool slots_for(int64_t S, int G) { return G > kDense && G <= kRatio * S; }
__device__ __forceinline__ bool has_slots(const OverlapImg& O) { return slots_for(O.K, O.G); }
// the slots of superpixel k, on the first cache line that begins in its row
__device__ __forceinline__ int64_t slots_at(const OverlapImg& O, int64_t k) {
  static_assert(kDense >= 2 * kSlotInts, "a whole line in every row");
  return (O.tab + k * O.G + kSlotInts - 1) & ~(int64_t)(kSlotInts - 1);
}

// n4 16-byte words from T.flag on (flags, sums, error word, dense tables), and the
// slots of image blockIdx.y
__global__ __launch_bounds__(kT) void k_m_clear(const OverlapImg* ov, OverlapPtrs T, int64_t n4) {
  int4* const a = reinterpret_cast<int4*>(T.flag);
  const int64_t blk = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t step = (int64_t)gridDim.x * gridDim.y * kT;
  for (int64_t i = blk * kT + threadIdx.x; i < n4; i += step) a[i] = make_int4(0, 0, 0, 0);
  const OverlapImg O = ov[blockIdx.y];
  if (!has_slots(O)) return;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < (int64_t)O.K * (kSlotInts / 4);
       i += (int64_t)gridDim.x * kT)
    reinterpret_cast<int4*>(T.tab + slots_at(O, i / (kSlotInts / 4)))[i % (kSlotInts / 4)] =
        make_int4(0, 0, 0, 0);
}

__device__ __forceinline__ int ld_dev(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// superpixel k is to be counted anew (image blockIdx.y); a store only where it is
// news, as stores to one line follow one another
__device__ __forceinline__ void flag_label(const OverlapImg& O, const OverlapPtrs& T, int k) {
  if (ld_dev(T.flag + O.row + k)) return;
  __hip_atomic_store(T.flag + O.row + k, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(T.flag + blockIdx.y, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// n pixels more of superpixel k in region g
__device__ __forceinline__ void add_overlap(const OverlapImg& O, const OverlapPtrs& T, int k, int g,
                                            int n) {
  if (!has_slots(O)) {
    atomicAdd(T.tab + O.tab + (int64_t)k * O.G + g, n);
    return;
  }
  int* const row = T.tab + slots_at(O, k);
  const int h = (int)(((unsigned)g * 2654435761u) >> 28);
  static_assert(kSlots16 == 16, "a hash of four bits");
  // (a flagged row is counted anew: its slots need no more)
  const int flagged = ld_dev(T.flag + O.row + k);
  int q = ld_dev(row + h);
  if (flagged) return;
#pragma unroll 1
  for (int p = 0; p < kSlots16; ++p) {
    const int e = (h + p) & (kSlots16 - 1);
    if (p) q = ld_dev(row + e);
    if (q == 0) {
      q = atomicCAS(row + e, 0, g + 1);
      if (q == 0) q = g + 1;
    }
    if (q == g + 1) {
      atomicAdd(row + kSlots16 + e, n);
      return;
    }
  }
  flag_label(O, T, k);
}

// A block's LDS table of pairs (the place k G + g in the image's table; -1: empty)
// and their pixels.  A pair that finds no entry within kProbes is added to a dense
// table in memory by itself, or has its superpixel counted anew where that has
// slots: with as many pairs as pixels (noise) look-ups over all the entries and the
// slots behind them took 36 to 47 ms for 8 x 3840x2160.
constexpr int kProbes = 8;

template <int BITS>
struct PairTable {
  static constexpr int kN = 1 << BITS;
  int key[kN], cnt[kN];
  __device__ __forceinline__ void clear() {
    for (int e = threadIdx.x; e < kN; e += kT) {
      key[e] = -1;
      cnt[e] = 0;
    }
  }
  __device__ __forceinline__ bool add(int k, int n) {
    int q = (int)(((unsigned)k * 2654435761u) >> (32 - BITS));
#pragma unroll 1
    for (int p = 0; p < kProbes; ++p, q = (q + 1) & (kN - 1)) {
      int at = __hip_atomic_load(key + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (at == -1) {
        at = atomicCAS(key + q, -1, k);
        if (at == -1) at = k;
      }
      if (at == k) {
        atomicAdd(cnt + q, n);
        return true;
      }
    }
    return false;
  }
};

// Tiles of the pixel pass: 64 columns, R rows per wave.  16 rows read 1.3 labels
// per pixel; with 4, a batch of up to kSmallTiles tiles has four times the blocks
// and a quarter of the serial work in each.
constexpr int kMW = 64;
constexpr int kSmallTiles = 512;

__host__ __device__ inline int m_tiles(int W, int H, int rows) {
  return ((W + kMW - 1) / kMW) * ((H + 4 * rows - 1) / (4 * rows));
}

__device__ __forceinline__ int clampi(int x, int hi) { return min(max(x, 0), hi); }

// What boundary pixels beside the tile widen to in it, by the two bits of their
// columns from left to right, four bits each: columns x0, x0 + 1 from x0 - 2 (one)
// and x0 - 1 (both); columns x0 + 62, x0 + 63 from x0 + 64 (both) and x0 + 65 (one).
constexpr unsigned kLeft = 0x3310, kRight = 0x3230;

// Overlap counts, and per block the boundary recall counts.  A lane per column of
// the tile: a row's boundary pixels are one ballot and widening them by two columns
// a few operations on the mask, so the 5 x 5 test of a row is five masks.  Each lane
// then counts the runs of equal (k, g) down its column (a few in 16 rows, so they
// are marked first and looked up after) in the block's LDS table, which the block
// adds to the overlaps once.  Bound by the issue of the rows' operations and the 8 B
// per pixel: 8 x 3840x2160 takes 230 us, 269 us with a look-up in each row; 399 us
// with the boundary map of a 64 x 16 tile in LDS and runs along the rows.

template <int R>
__global__ __launch_bounds__(kT) void k_m_pix(const ImgDesc* img, const OverlapImg* ov,
                                              OverlapPtrs T, const int32_t* sp, const int32_t* gt,
                                              int* br_part, int max_blocks) {
  __shared__ PairTable<(R > 4 ? 9 : 8)> tab;
  __shared__ int pair[kT / 64][R][2][64];  // the labels and regions of the waves' rows
  __shared__ int wsum[kT / 64][2];
  const int b = blockIdx.y;
  const ImgDesc& I = img[b];
  const int W = I.W, H = I.H;
  if ((int)blockIdx.x >= m_tiles(W, H, R)) return;  // the whole block
  const int tiles_x = (W + kMW - 1) / kMW;
  const int x0 = (blockIdx.x % tiles_x) * kMW;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int yw = (blockIdx.x / tiles_x) * (4 * R) + wv * R;  // the wave's first row
  const OverlapImg O = ov[b];
  tab.clear();
  __syncthreads();
  int nhit = 0, ngb = 0;
  if (yw < H) {
    const int32_t* S = sp + I.pix_off;
    const int32_t* Gt = gt + I.pix_off;
    const int xc = min(x0 + lane, W - 1);
    // beside the tile: lanes 0 .. 4 the labels of columns x0 - 2, x0 - 1, x0 + 64,
    // x0 + 65, x0 + 66; lane 63 the region of column x0 + 64.  Places outside the
    // image repeat its edge, which makes no boundary there.
    const int xs = lane == 63 ? x0 + 64 : x0 + (lane < 2 ? lane - 2 : 62 + min(lane, 4));
    const unsigned long long in_x = __ballot(x0 + lane < W);
    const unsigned in_side = (unsigned)__ballot(xs >= 0 && xs < W) & 15;
    int h[R + 5], e[R + 5], g[R + 1];  // rows yw - 2 on; of regions, yw on
    {
      const int32_t* ph = S + (int64_t)clampi(yw - kR, H - 1) * W + xc;
      const int32_t* pg = Gt + (int64_t)yw * W + xc;
      const int ys = lane == 63 ? yw : yw - kR;
      const int32_t* pe = (lane == 63 ? Gt : S) + (int64_t)clampi(ys, H - 1) * W + clampi(xs, W - 1);
#pragma unroll
      for (int j = 0; j < R + 5; ++j) {
        h[j] = *ph;
        e[j] = *pe;
        if (j < R + 1) g[j] = *pg;
        ph += (unsigned)(yw - kR + j) < (unsigned)(H - 1) ? W : 0;
        pe += (unsigned)(ys + j) < (unsigned)(H - 1) ? W : 0;
        pg += yw + j < H - 1 ? W : 0;
      }
    }
    // the superpixel boundary pixels of row yw - 2 + j, two columns wider on both sides
    auto wide = [&](int j) {
      int right = __shfl_down(h[j], 1, 64);
      const int beside = __builtin_amdgcn_readlane(e[j], 2);
      right = lane == 63 ? beside : right;
      int eright = __shfl_down(e[j], 1, 64);
      const int first = __builtin_amdgcn_readlane(h[j], 0);
      eright = lane == 1 ? first : eright;
      const int y = yw - kR + j;
      unsigned long long m = __ballot(((right ^ h[j]) | (h[j + 1] ^ h[j])) != 0) & in_x;
      const unsigned s = (unsigned)__ballot(((eright ^ e[j]) | (e[j + 1] ^ e[j])) != 0) & in_side;
      m |= m << 1 | m << 2 | m >> 1 | m >> 2;
      m |= kLeft >> (4 * (s & 3)) & 3;                            // from columns x0 - 2, x0 - 1
      m |= (unsigned long long)(kRight >> (4 * (s >> 2)) & 3) << 62;  // from x0 + 64, x0 + 65
      return y >= 0 && y < H ? m : 0ull;
    };
    const int rows = min(R, H - yw);
    unsigned starts = 1;  // bit u: a run of this lane's column starts in row u
    unsigned long long D[5] = {0, wide(0), wide(1), wide(2), wide(3)};
#pragma unroll
    for (int u = 0; u < R; ++u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) D[j] = D[j + 1];
      D[4] = wide(u + 4);
      int right = __shfl_down(g[u], 1, 64);
      right = lane == 63 ? e[u] : right;
      unsigned long long gb = __ballot(((right ^ g[u]) | (g[u + 1] ^ g[u])) != 0) & in_x;
      gb = u < rows ? gb : 0;
      ngb += __popcll(gb);
      nhit += __popcll(gb & (D[0] | D[1] | D[2] | D[3] | D[4]));
      pair[wv][u][0][lane] = h[u + kR];
      pair[wv][u][1][lane] = g[u];
      if (u > 0) starts |= ((h[u + kR] ^ h[u + kR - 1]) | (g[u] ^ g[u - 1])) != 0 ? 1u << u : 0u;
      __builtin_amdgcn_sched_barrier(0);  // (rows in turn: their masks do not fit the registers)
    }
    bool bad = false;
    starts = x0 + lane < W ? starts & ((1u << rows) - 1) : 0;
#pragma unroll 1
    while (starts) {
      const int u = __builtin_ctz(starts);
      starts &= starts - 1;
      const int n = (starts ? __builtin_ctz(starts) : rows) - u;
      const int k = pair[wv][u][0][lane], g = pair[wv][u][1][lane];
      if ((unsigned)k >= (unsigned)O.K || (unsigned)g >= (unsigned)O.G) {
        bad = true;
        continue;
      }
      if (tab.add(k * O.G + g, n)) continue;
      if (has_slots(O)) flag_label(O, T, k);
      else add_overlap(O, T, k, g, n);
    }
    if (__ballot(bad) && lane == 0) atomicOr(T.err, 1);
  }
  if (lane == 0) {
    wsum[wv][0] = nhit;
    wsum[wv][1] = ngb;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < tab.kN; e += kT) {
    const int key = tab.key[e];
    if (key >= 0) add_overlap(O, T, key / O.G, key % O.G, tab.cnt[e]);
  }
  if (threadIdx.x < 2) {
    int t = 0;
    for (int w = 0; w < kT / 64; ++w) t += wsum[w][threadIdx.x];
    br_part[((int64_t)b * max_blocks + blockIdx.x) * 2 + threadIdx.x] = t;
  }
}

// The rows of flagged superpixels cleared, a wave each.
__global__ __launch_bounds__(kT) void k_m_clear_rows(const OverlapImg* ov, OverlapPtrs T) {
  const OverlapImg O = ov[blockIdx.y];
  if (!T.flag[blockIdx.y]) return;
  const int lane = threadIdx.x & 63;
  for (int64_t k = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6); k < O.K;
       k += (int64_t)gridDim.x * (kT / 64)) {
    if (!T.flag[O.row + k]) continue;
    for (int g = lane; g < O.G; g += 64) T.tab[O.tab + k * O.G + g] = 0;
  }
}

// The pixels of flagged superpixels counted into their rows: a lane per column of 16
// rows, its runs gathered in the block's LDS table as in k_m_pix.  One background
// superpixel over half of 8 x 3840x2160 among 10 764: 400 us a call; 1070 with each
// run added to memory, 735 with dense tables for all.
__global__ __launch_bounds__(kT) void k_m_rescan(const ImgDesc* img, const OverlapImg* ov,
                                                 OverlapPtrs T, const int32_t* sp,
                                                 const int32_t* gt) {
  __shared__ PairTable<9> tab;
  const OverlapImg O = ov[blockIdx.y];
  if (!T.flag[blockIdx.y]) return;
  const ImgDesc& I = img[blockIdx.y];
  const int W = I.W, H = I.H;
  const int tiles_x = (W + kMW - 1) / kMW;
  constexpr int kRows = 16;
  if ((int)blockIdx.x >= m_tiles(W, H, kRows)) return;  // the whole block
  tab.clear();
  __syncthreads();
  const int x = (blockIdx.x % tiles_x) * kMW + (threadIdx.x & 63);
  const int y0 = (blockIdx.x / tiles_x) * (4 * kRows) + (threadIdx.x >> 6) * kRows;
  int* const row0 = T.tab + O.tab;
  int k[kRows], g[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const bool in = x < W && y0 + u < H;
    const int64_t i = I.pix_off + (int64_t)(y0 + u) * W + x;
    k[u] = in ? sp[i] : -1;
    g[u] = in ? gt[i] : -1;
  }
  int cur = -1, cnt = 0;  // the run's pair, its pixels
  bool flagged = false;   // of the label of the row before
  auto put = [&]() {
    if (cur >= 0 && !tab.add(cur, cnt)) atomicAdd(row0 + cur, cnt);
  };
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    if (u == 0 || k[u] != k[u - 1]) flagged = (unsigned)k[u] < (unsigned)O.K && T.flag[O.row + k[u]];
    const int key = flagged && (unsigned)g[u] < (unsigned)O.G ? k[u] * O.G + g[u] : -1;
    if (key != cur) {
      put();
      cur = key;
      cnt = 0;
    }
    ++cnt;
  }
  put();
  __syncthreads();
  for (int e = threadIdx.x; e < tab.kN; e += kT)
    if (tab.key[e] >= 0) atomicAdd(row0 + tab.key[e], tab.cnt[e]);
}

// Sixteen lanes per superpixel, a block where its row is longer than kLong (10 764
// regions, 510 superpixels: 2171 us a call with sixteen lanes, 281 with a block): |s_k|,
// the leaking overlaps, the largest overlap; and the blocks' boundary counts.  A block sums its share of one image and adds the
// four totals to the image's sums (T.sum_stride integers apart: see metrics_sum_stride).
constexpr int kLong = 256;

__global__ __launch_bounds__(kT) void k_m_rows(const ImgDesc* img, const OverlapImg* ov,
                                               OverlapPtrs T, const int* br_part, int max_blocks,
                                               int rows) {
  __shared__ int64_t red[kT / 64][4];
  __shared__ int s_size[kT / 64], s_best[kT / 64];
  const int b = blockIdx.y;
  const OverlapImg O = ov[b];
  const int t = threadIdx.x & 15;
  const bool has = has_slots(O), any = T.flag[b] != 0;
  int64_t a[4] = {0, 0, 0, 0};
  const int nb = m_tiles(img[b].W, img[b].H, rows);
  for (int i = blockIdx.x * kT + threadIdx.x; i < nb; i += gridDim.x * kT) {
    a[0] += br_part[((int64_t)b * max_blocks + i) * 2 + 0];
    a[1] += br_part[((int64_t)b * max_blocks + i) * 2 + 1];
  }
  for (int64_t k = (int64_t)blockIdx.x * (kT / 16) + threadIdx.x / 16; k < O.K;
       k += (int64_t)gridDim.x * (kT / 16)) {
    const bool slots = has && !(any && T.flag[O.row + k]);
    const int n = slots ? kSlots16 : O.G;
    if (n > kLong) continue;
    const int* r = T.tab + (slots ? slots_at(O, k) + kSlots16 : O.tab + k * O.G);
    const int c0 = t < n ? r[t] : 0, c1 = t + 16 < n ? r[t + 16] : 0;
    int size = c0 + c1, best = max(c0, c1);
    for (int g = 32 + t; g < n; g += 16) {
      size += r[g];
      best = max(best, r[g]);
    }
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
      size += __shfl_xor(size, o, 64);
      best = max(best, __shfl_xor(best, o, 64));
    }
    int leak = (20LL * c0 > (int64_t)size) + (20LL * c1 > (int64_t)size);
    for (int g = 32 + t; g < n; g += 16) leak += 20LL * r[g] > (int64_t)size;
    a[2] += (int64_t)size * leak;  // (this lane's share of the leaking overlaps)
    if (t == 0) a[3] += best;
  }
  if (O.G > kLong && (!has || any)) {
    for (int64_t k = blockIdx.x; k < O.K; k += gridDim.x) {  // (the whole block)
      if (has && !T.flag[O.row + k]) continue;
      const int* r = T.tab + O.tab + k * O.G;
      int size = 0, best = 0;
#pragma unroll 4
      for (int g = threadIdx.x; g < O.G; g += kT) {
        size += r[g];
        best = max(best, r[g]);
      }
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        size += __shfl_xor(size, o, 64);
        best = max(best, __shfl_xor(best, o, 64));
      }
      if ((threadIdx.x & 63) == 0) {
        s_size[threadIdx.x >> 6] = size;
        s_best[threadIdx.x >> 6] = best;
      }
      __syncthreads();
      size = best = 0;
#pragma unroll
      for (int w = 0; w < kT / 64; ++w) {
        size += s_size[w];
        best = max(best, s_best[w]);
      }
      int leak = 0;
      // (none leaks if the largest does not)
      if (20LL * best > (int64_t)size) {
#pragma unroll 4
        for (int g = threadIdx.x; g < O.G; g += kT) leak += 20LL * r[g] > (int64_t)size;
      }
      a[2] += (int64_t)size * leak;
      if (threadIdx.x == 0) a[3] += best;
      __syncthreads();  // s_size and s_best are rewritten
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) a[c] += __shfl_xor(a[c], o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][c] = a[c];
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    int64_t v = 0;
    for (int w = 0; w < kT / 64; ++w) v += red[w][threadIdx.x];
    if (v) atomicAdd((unsigned long long*)(T.sums + (int64_t)T.sum_stride * b + threadIdx.x),
                     (unsigned long long)v);
  }
}

}  // namespace

bool overlap_has_slots(int64_t n_lab, int n_gt) { return slots_for(n_lab, n_gt); }

// A cache line per image keeps the images' atomics from waiting for each other (nr
// of k_m_rows each).  The 96 bytes that it adds per image come out of the workspace
// that S labels leave: 16 bytes each are allowed for and the flags take 4.
int metrics_sum_stride(int64_t n_labels, int n_img) { return n_labels >= 16 * (int64_t)n_img + 64 ? 16 : 4; }

int metrics_tile_rows(int max_w, int max_h, int n_img) {
  return (int64_t)m_tiles(max_w, max_h, 16) * n_img <= kSmallTiles ? 4 : 16;
}

int metrics_max_blocks(int max_w, int max_h, int rows) { return m_tiles(max_w, max_h, rows); }

hipError_t metrics_launch(const DevPtrs& P, int rows, int max_blocks, int64_t max_rows, bool slots,
                          const OverlapImg* ov, const OverlapPtrs& T, int64_t clear_bytes,
                          int max_gt, const int32_t* sp, const int32_t* gt, int* br_part,
                          hipStream_t s) {
  const int64_t n4 = clear_bytes / 16;
  // some 8192 blocks; at least one per image
  const int64_t want = std::max((n4 + kT - 1) / kT, slots ? P.n_img * ((max_rows * (kSlotInts / 4) + kT - 1) / kT) : 1);
  const unsigned nc = (unsigned)std::max<int64_t>(std::min<int64_t>(want, 8192) / P.n_img, 1);
  hipLaunchKernelGGL(k_m_clear, dim3(nc, P.n_img), dim3(kT), 0, s, ov, T, n4);
  const dim3 g(max_blocks, P.n_img);
  if (rows == 16)
    hipLaunchKernelGGL(k_m_pix<16>, g, dim3(kT), 0, s, P.img, ov, T, sp, gt, br_part, max_blocks);
  else
    hipLaunchKernelGGL(k_m_pix<4>, g, dim3(kT), 0, s, P.img, ov, T, sp, gt, br_part, max_blocks);
  // up to 128 blocks per image: their atomics on the image's line follow one another
  const int64_t per = max_gt > kLong ? 1 : 64;  // superpixels a block takes before it goes round
  const unsigned nr = (unsigned)std::min<int64_t>((max_rows + per - 1) / per, 128);
  if (slots) {
    hipLaunchKernelGGL(k_m_clear_rows, dim3(nr, P.n_img), dim3(kT), 0, s, ov, T);
    hipLaunchKernelGGL(k_m_rescan, g, dim3(kT), 0, s, P.img, ov, T, sp, gt);
  }
  hipLaunchKernelGGL(k_m_rows, dim3(nr, P.n_img), dim3(kT), 0, s, P.img, ov, T, br_part, max_blocks,
                     rows);
  return hipGetLastError();
}

}  // namespace gmmsp
