// Connectivity post-processing (Algorithm 1, last step; the paragraph on
// enforcing connectivity in Sec. III-C) for a batch of label maps on gfx950.
//
// The paper sorts the isolated pieces of the superpixels by size, ascending,
// and merges each piece smaller than a quarter of the desired superpixel size,
// in that order, into the neighbouring superpixel closest in colour; a merged
// piece's size becomes zero and its destination's size grows by it.
//
// Definitions (pieces are "segments"):
//   * a segment is a 4-connected component of equal label; its id is the
//     raster index of its first pixel; small means 4 size < v_x v_y;
//   * colours are the segments' own mean Lab colours, fixed for the whole
//     procedure, from integer sums of the pixel colours quantised to 2^-20;
//   * the neighbours of a segment are the current segments holding a
//     4-neighbour of any pixel merged into it so far; the destination is the
//     one at the smallest squared colour distance (FP64, no fused
//     multiply-add), ties to the smallest id.
//
// Parallel form of the sequential procedure.  A small segment's decision
// reads only (a) its own size and pixels, which change only when small
// segments adjacent to it are merged into it, and (b) the current owner of
// each neighbouring pixel, which changes only for neighbouring small
// segments.  So the clusters of small segments joined by adjacency never
// influence each other: each cluster runs the procedure in the global order
// restricted to it, and all clusters run in parallel.  Merges into a large
// segment from several clusters only add to its size, which no decision reads
// (a large segment is never merged).
//
// Steps: pixel union-find of equal-label 4-neighbours, in 64 x 64 tiles in
// LDS and then across tile borders (roots are the minimum index, so the
// partition and ids are unique whatever the order of the atomics); ranks of
// the roots in raster order (segment indices, in id order); sizes and integer
// colour sums, gathered per block in LDS and added with integer atomics
// (exact); per-source pixel lists; a pass over the small segments that merges
// those whose neighbours are all large and joins the others into clusters;
// per-cluster lists; the merges of each cluster (8 or 16 lanes, a wave or a block);
// the output ids.  The number of segments stays on the device: kernels over
// segments read it and stride over them, so nothing waits for the host.
#include "gmmsp_internal.h"

#include <math.h>

#include <algorithm>

namespace gmmsp {

namespace {

constexpr int kT = 256;
constexpr int kScanPer = 16;                // elements per thread of the scan
constexpr int kScanBlock = kScanPer * 256;  // elements per block of the scan

// loads and stores of state other threads update (device-coherent: served by
// the L2, never by a possibly stale L1 line)
__device__ __forceinline__ int ld_dev(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// root of x in a forest with parent[x] <= x (every link points to a smaller
// index, so the walk strictly decreases and ends)
__device__ int uf_find(int* par, int x) {
  int y = ld_dev(par + x);
  while (y != x) {
    x = y;
    y = ld_dev(par + x);
  }
  return x;
}

// join the sets of a and b by hanging the larger root under the smaller; a
// failed compare-and-swap returns the newer, strictly smaller parent, so the
// loop ends
__device__ void uf_unite(int* par, int a, int b) {
  a = uf_find(par, a);
  b = uf_find(par, b);
  while (a != b) {
    if (a < b) {
      const int t = a;
      a = b;
      b = t;
    }
    const int old = atomicCAS(par + a, a, b);
    if (old == a) return;
    a = uf_find(par, old);
    b = uf_find(par, b);
  }
}

__device__ double colour_dist2(const double* a, const double* b) {
#pragma clang fp contract(off)
  const double dL = a[0] - b[0];
  const double da = a[1] - b[1];
  const double db = a[2] - b[2];
  return (dL * dL + da * da) + db * db;
}

// merge parent walk: a segment points to the segment it was merged into
__device__ __forceinline__ int m_find(const int* mpar, int t) {
  int u = ld_dev(mpar + t);
  while (u != t) {
    t = u;
    u = ld_dev(mpar + t);
  }
  return t;
}

// ---- pixel components ------------------------------------------------------
// A block labels a 64 x 64 tile, consecutive rows per wave: every pixel first
// points, in LDS, at the head of its horizontal run of equal label (masks from
// ballots), then each overlap of two equal runs on adjacent rows is joined once, by
// its first pixel, from head to head (union-find with LDS atomics, roots the
// smallest tile-local raster index, which is also the smallest global index); the
// run's head then finds the root for its run.  The block writes each pixel's tile
// root as a global index and keeps the labels and roots of the tile's first and
// last columns in a side buffer; the tile borders are then joined in global memory
// from those and from the tiles' first rows.  Roots stay the minimum index of their
// set throughout.  Bound by the latency of the LDS chains and the 8 B per pixel:
// 8 x 3840x2160 takes 210 us; 387 us when the waves took rows in turn, so that the
// links ran from row to row, and every pixel followed them to its root.

constexpr int kTW = 64, kTH = 64;  // tile of the component labelling
constexpr int kSide = 4 * kTH;     // first-column labels, roots; last-column labels, roots
// Waves per block of the tile kernels: four fill the chip on large batches; up to
// kSmallTiles tiles (two blocks per CU) sixteen shorten a block's serial rows.
// Tile labelling and segment pass of one 481x321 image (48 tiles): 24.3 + 18.3 us
// with four, 12.4 + 12.5 us with sixteen (now 9 + 11.7).
constexpr int kSmallTiles = 512;

__device__ int lds_find(int* lp, int x) {
  int y = __hip_atomic_load(lp + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  while (y != x) {
    x = y;
    y = __hip_atomic_load(lp + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  return x;
}

__device__ void lds_unite(int* lp, int a, int b) {
  a = lds_find(lp, a);
  b = lds_find(lp, b);
  while (a != b) {
    if (a < b) {
      const int t = a;
      a = b;
      b = t;
    }
    const int old = atomicCAS(lp + a, a, b);
    if (old == a) return;
    a = lds_find(lp, old);
    b = lds_find(lp, b);
  }
}

template <int WAVES>  // per block
__global__ __launch_bounds__(64 * WAVES) void k_cc_tile(const ImgDesc* img, const int32_t* labels,
                                                        int* par, int* side, int max_tiles) {
  __shared__ int lp[kTW * kTH];
  const int b = blockIdx.y;
  const ImgDesc& I = img[b];
  const int W = I.W, H = I.H;
  const int tiles_x = (W + kTW - 1) / kTW, tiles_y = (H + kTH - 1) / kTH;
  if ((int)blockIdx.x >= tiles_x * tiles_y) return;  // the whole block
  const int x0 = (blockIdx.x % tiles_x) * kTW, y0 = (blockIdx.x / tiles_x) * kTH;
  const int64_t off = I.pix_off;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int x = x0 + lane;
  const unsigned long long in_x = __ballot(x < W), upto = (2ull << lane) - 1ull;  // bits 0..lane
  // the wave's rows and, first, the tile's row above them: labels, and masks of the
  // pixels that start a run (pixels outside the image are runs of their own)
  constexpr int kRows = kTH / WAVES;
  const int ty0 = wv * kRows;
  const int rows = min(kRows, H - y0 - ty0);  // <= 0: none
  int32_t labs[kRows + 1];
#pragma unroll
  for (int q = 0; q <= kRows; ++q) {
    const int y = y0 + ty0 + q - 1;
    labs[q] = x < W && y >= y0 && y < H ? labels[off + (int64_t)y * W + x] : 0;
  }
  unsigned long long heads[kRows + 1];
#pragma unroll
  for (int q = 0; q <= kRows; ++q) {
    const int32_t left = __shfl_up(labs[q], 1, 64);
    heads[q] = __ballot(left != labs[q]) | 1ull | ~in_x;
    if (q == 0) continue;
    const int l = (ty0 + q - 1) * kTW;
    lp[l + lane] = l + 63 - __builtin_clzll(heads[q] & upto);
  }
  __syncthreads();
  // Vertical joins, row after row from above, so that a run's head meets heads that
  // already point near their root: the first pixel of each overlap of equal runs.
#pragma unroll
  for (int q = 1; q <= kRows; ++q) {
    if (q - 1 >= rows || ty0 + q == 1) continue;
    const unsigned long long eq = __ballot(labs[q] == labs[q - 1]) & in_x;
    const int l = (ty0 + q - 1) * kTW;
    if (eq & ~(eq << 1 & ~heads[q] & ~heads[q - 1]) & (1ull << lane))
      lds_unite(lp, l + 63 - __builtin_clzll(heads[q] & upto),
                l - kTW + 63 - __builtin_clzll(heads[q - 1] & upto));
  }
  __syncthreads();
  int* sd = side + ((size_t)b * max_tiles + blockIdx.x) * kSide;
  const int xl = min(kTW, W - x0) - 1;  // the tile's last column
#pragma unroll
  for (int q = 1; q <= kRows; ++q) {
    if (q - 1 >= rows) continue;
    const int ty = ty0 + q - 1;
    // the run's head finds the root for its run
    const int head = 63 - __builtin_clzll(heads[q] & upto);
    int r = head == lane ? lds_find(lp, ty * kTW + lane) : 0;
    r = __shfl(r, head, 64);
    const int g = (int)(off + (int64_t)(y0 + r / kTW) * W + x0 + r % kTW);
    if (x < W) par[off + (int64_t)(y0 + ty) * W + x] = g;
    if (lane == 0) {
      sd[ty] = labs[q];
      sd[kTH + ty] = g;
    }
    if (lane == xl) {
      sd[2 * kTH + ty] = labs[q];
      sd[3 * kTH + ty] = g;
    }
  }
}

// Joins across tile borders, one block per tile: wave 0 joins the tile's first
// row to the row above it, wave 1 its first column to the column on its left
// (from the side buffer).  As inside the tiles, only the first pixel of each
// overlap of equal runs along the border joins.
__global__ __launch_bounds__(128) void k_cc_border(const ImgDesc* img, const int32_t* labels,
                                                   int* par, const int* side, int max_tiles) {
  const int b = blockIdx.y;
  const ImgDesc& I = img[b];
  const int W = I.W, H = I.H;
  const int tiles_x = (W + kTW - 1) / kTW, tiles_y = (H + kTH - 1) / kTH;
  if ((int)blockIdx.x >= tiles_x * tiles_y) return;
  const int x0 = (blockIdx.x % tiles_x) * kTW, y0 = (blockIdx.x / tiles_x) * kTH;
  const int t = threadIdx.x & 63;
  int32_t a = 0, c = 0;
  int ra = 0, rc = 0;
  bool in;
  if (threadIdx.x < 64) {  // first row against the row above
    if (y0 == 0) return;
    in = x0 + t < W;
    const int64_t i = I.pix_off + (int64_t)y0 * W + x0 + t;
    if (in) {
      a = labels[i];
      c = labels[i - W];
      ra = ld_dev(par + i);
      rc = ld_dev(par + i - W);
    }
  } else {  // first column against the last column of the tile on the left
    if (x0 == 0) return;
    in = y0 + t < H;
    const int* me = side + ((size_t)b * max_tiles + blockIdx.x) * kSide;
    const int* lf = me - kSide;
    if (in) {
      a = me[t];
      ra = me[kTH + t];
      c = lf[2 * kTH + t];
      rc = lf[3 * kTH + t];
    }
  }
  const int32_t ap = __shfl_up(a, 1, 64), cp = __shfl_up(c, 1, 64);
  if (!in || a != c) return;
  if (t > 0 && ap == a && cp == a) return;  // joined through the previous pixel
  uf_unite(par, ra, rc);
}

// Segment numbering: the roots of the pixel forest (par[i] == i) in raster
// order.  Each block of kScanBlock pixels counts its roots and writes each
// root's rank within the block (at the root only); a root's segment index is
// that rank plus the exclusive scan of the block counts.
__global__ __launch_bounds__(kT) void k_root_rank(const int* par, int n, int* rank, int* bsum) {
  __shared__ int sh[kT];
  const int base = blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  int v[kScanPer];
  if (base + kScanPer <= n) {  // par is 256-byte aligned: four 16-byte loads
#pragma unroll
    for (int k = 0; k < kScanPer / 4; ++k) {
      const int4 w = reinterpret_cast<const int4*>(par + base)[k];
      v[4 * k] = w.x == base + 4 * k;
      v[4 * k + 1] = w.y == base + 4 * k + 1;
      v[4 * k + 2] = w.z == base + 4 * k + 2;
      v[4 * k + 3] = w.w == base + 4 * k + 3;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) v[k] = base + k < n && par[base + k] == base + k;
  }
  int t = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) t += v[k];
  sh[threadIdx.x] = t;
  __syncthreads();
  for (int o = 1; o < kT; o <<= 1) {
    const int u = (int)threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += u;
    __syncthreads();
  }
  int run = sh[threadIdx.x] - t;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (v[k]) rank[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == kT - 1) bsum[blockIdx.x] = sh[kT - 1];
}

// one block: exclusive scan of the block totals of n (or *n_dev) elements, in
// chunks of kScanBlock; their sum to *total (nullable)
__global__ __launch_bounds__(kT) void k_scan_totals(int* bsum, int n, const int* n_dev, int* total) {
  __shared__ int sh[kT];
  const int nb = ((n_dev ? *n_dev : n) + kScanBlock - 1) / kScanBlock;
  int carry = 0;
  for (int c0 = 0; c0 < nb; c0 += kScanBlock) {
    const int base = c0 + threadIdx.x * kScanPer;
    int v[kScanPer];
    int t = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = base + k < nb ? bsum[base + k] : 0;
      t += v[k];
    }
    sh[threadIdx.x] = t;
    __syncthreads();
    for (int o = 1; o < kT; o <<= 1) {
      const int u = (int)threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += u;
      __syncthreads();
    }
    int run = carry + sh[threadIdx.x] - t;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
      if (base + k < nb) bsum[base + k] = run;
      run += v[k];
    }
    carry += sh[kT - 1];
    __syncthreads();  // sh is rewritten by the next chunk
  }
  if (threadIdx.x == 0 && total) *total = carry;
}

// ---- segments ---------------------------------------------------------------

// counters of a call, at the head of the side buffer once the tile borders are
// joined: pixels listed, clustered sources, listed sources, clusters by class
enum Counter {
  N_PX = 0, N_CLUSTERED = 1, N_LISTED = 2, N_TEAM8 = 3, N_TEAM16 = 4, N_WAVE = 5, N_BLOCK = 6,
  N_COUNTERS = 16
};

__global__ __launch_bounds__(kT) void k_seg_zero(const int* n_seg_dev, int n_img, int* size0,
                                                 unsigned long long* colsum, int* ccnt, int* cursor,
                                                 int* ccur, int* cnt, int* counts) {
  const int n_seg = *n_seg_dev;
  const int i0 = blockIdx.x * kT + threadIdx.x, step = gridDim.x * kT;
  if (i0 < N_COUNTERS) cnt[i0] = 0;
  for (int i = i0; i < 4 * n_img; i += step) counts[i] = 0;
  for (int s = i0; s < n_seg; s += step) {
    size0[s] = 0;
    ccnt[s] = 0;
    cursor[s] = 0;
    ccur[s] = 0;
  }
  for (int64_t s = i0; s < 3 * (int64_t)n_seg; s += step) colsum[s] = 0ull;
}

// Segment of each pixel, segment roots, and the sizes and integer colour sums
// (exact, so the order of the additions does not matter), on the 64 x 64 tiles of
// the component labelling.  A pixel's parent is its tile's root of its component
// unless the pixel is such a root itself, so only the roots walk the forest and
// read their rank; the others find them through LDS.  Each lane then takes a
// column of 16 rows and adds up runs of equal segment in registers; a run's totals
// go to the segment's entry of an LDS table, and the block adds each entry once
// with integer atomics.  Roots beyond the table's kTab entries (a checkerboard
// has 4096) go to memory directly.  Bound by the 20 B per pixel (parents, colours,
// segments); 8 x 3840x2160 took 857 us when every pixel walked the
// forest and every row was summed with six shuffle steps of 64-bit values, 543
// with a table of 512 entries (four blocks per CU) and 64-bit integer sums, and
// takes 453 us.
constexpr int kTab = 384;

__device__ __forceinline__ void add_stats(int s, int cnt, const long long (&q)[3], int* size0,
                                          unsigned long long* colsum) {
  if (cnt) atomicAdd(size0 + s, cnt);
#pragma unroll
  for (int c = 0; c < 3; ++c) atomicAdd(colsum + 3 * (int64_t)s + c, (unsigned long long)q[c]);
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_seg_assign(const ImgDesc* img, const float* lab,
                                                   const int* par, const int* rank,
                                                   const int* boff, int* segid,
                                                   int* seg_root, int* seg_img, int* size0,
                                                   unsigned long long* colsum) {
  // a root: its table entry, or ~ its segment beyond the table; else kTab + the
  // tile-local index of its parent
  __shared__ int ref[kTW * kTH];
  __shared__ int tseg[kTab], tcnt[kTab];
  __shared__ unsigned long long tsum[3][kTab];
  __shared__ int n_tab;
  const int b = blockIdx.y;
  const ImgDesc& I = img[b];
  const int W = I.W, H = I.H;
  const int tiles_x = (W + kTW - 1) / kTW;
  if ((int)blockIdx.x >= tiles_x * ((H + kTH - 1) / kTH)) return;  // the whole block
  const int x0 = (blockIdx.x % tiles_x) * kTW, y0 = (blockIdx.x / tiles_x) * kTH;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int off = (int)I.pix_off;
  const bool xin = x0 + lane < W;
  constexpr int kRows = kTH / WAVES;  // consecutive rows of a wave
  static_assert(kRows % 4 == 0, "rows in fours");
  const int ty0 = wv * kRows;
  for (int e = threadIdx.x; e < kTab; e += 64 * WAVES) {
    tcnt[e] = 0;
    tsum[0][e] = tsum[1][e] = tsum[2][e] = 0ull;
  }
  if (threadIdx.x == 0) n_tab = 0;
  __syncthreads();
  // (fewer than 2^31 pixels in a batch, but a row past the image may lie beyond)
  const unsigned i0 = (unsigned)off + (unsigned)(y0 + ty0) * (unsigned)W + (unsigned)(x0 + lane);
  // the segment of tile root i: its root's rank
  auto resolve = [&](int i) {
    int r = i, y = par[r];
    while (y != r) {
      r = y;
      y = par[y];
    }
    const int s = rank[r] + boff[r / kScanBlock];
    if (r == i) {
      seg_root[s] = i;
      seg_img[s] = b;
    }
    return s;
  };
  const int rows = min(kRows, H - y0 - ty0);  // <= 0: none
  int pr[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) pr[u] = xin && u < rows ? par[i0 + (unsigned)u * W] : -1;
  const int base = off + y0 * W + x0;  // the tile's first pixel
  const float inv_w = 1.0f / (float)W;
  unsigned beyond = 0;  // bit u: the pixel of row u is a root beyond the table
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int i = (int)(i0 + (unsigned)u * W), l = (ty0 + u) * kTW + lane;
    // the parent's place, row d / W and column d % W: inside this tile, and not the
    // pixel itself?  (a parent precedes its pixel, so d < 64 W and the quotient is
    // below 64, at most one off before the correction)
    const int d = pr[u] - base;
    int py = (int)((float)d * inv_w);
    int px = d - py * W;
    if (px < 0) {
      --py;
      px += W;
    } else if (px >= W) {
      ++py;
      px -= W;
    }
    if (pr[u] < 0) continue;
    if (pr[u] != i && d >= 0 && px < min(kTW, W - x0)) {
      ref[l] = kTab + py * kTW + px;
      continue;
    }
    const int e = atomicAdd(&n_tab, 1);
    if (e < kTab) {
      tseg[e] = l;  // its place, until the table's roots are resolved together
      ref[l] = e;
    } else {
      beyond |= 1u << u;
    }
  }
  for (; beyond; beyond &= beyond - 1) {
    const int u = __builtin_ctz(beyond);
    ref[(ty0 + u) * kTW + lane] = ~resolve((int)(i0 + (unsigned)u * W));
  }
  __syncthreads();
  const int n = min(n_tab, kTab);
  for (int e = threadIdx.x; e < n; e += 64 * WAVES) {
    const int l = tseg[e];
    tseg[e] = resolve((int)((unsigned)off + (unsigned)(y0 + l / kTW) * (unsigned)W +
                            (unsigned)(x0 + l % kTW)));
  }
  __syncthreads();
  // the run's reference (as in ref), its pixels, and its colours in units of 2^-20:
  // integers below 2^31 each, so their sums in FP64 are exact
  int run = 0, cnt = 0;
  double q[3] = {0.0, 0.0, 0.0};
  auto add = [&](int n, const long long (&v)[3]) {
    if (run >= 0) {
      if (n) atomicAdd(tcnt + run, n);
#pragma unroll
      for (int c = 0; c < 3; ++c) atomicAdd(&tsum[c][run], (unsigned long long)v[c]);
    } else {
      add_stats(~run, n, v, size0, colsum);
    }
  };
#pragma unroll 1
  for (int u0 = 0; u0 < rows; u0 += 4) {
    // four rows' colours in flight
    float col[4][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = xin && u0 + k < rows;
      const float* z = lab + 3 * (int64_t)(in ? i0 + (unsigned)(u0 + k) * W : 0u);
#pragma unroll
      for (int c = 0; c < 3; ++c) col[k][c] = in ? z[c] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!xin || u0 + k >= rows) continue;
      int v = ref[(ty0 + u0 + k) * kTW + lane];
      while (v >= kTab) v = ref[v - kTab];
      segid[i0 + (unsigned)(u0 + k) * W] = v >= 0 ? tseg[v] : ~v;
      if (v != run) {
        if (cnt) add(cnt, {(long long)q[0], (long long)q[1], (long long)q[2]});
        run = v;
        cnt = 0;
        q[0] = q[1] = q[2] = 0.0;
      }
      ++cnt;
      // (the product is exact in FP32, and below 2^31 so is its rounding there; larger
      // colours and NaN, which compares false, are rounded in FP64 and added by
      // themselves)
      if (fabsf(col[k][0]) < 2047.f && fabsf(col[k][1]) < 2047.f && fabsf(col[k][2]) < 2047.f) {
#pragma unroll
        for (int c = 0; c < 3; ++c) q[c] += (double)rintf(col[k][c] * 0x1p20f);
      } else {
        add(0, {(long long)rint((double)col[k][0] * 1048576.0), (long long)rint((double)col[k][1] * 1048576.0),
                (long long)rint((double)col[k][2] * 1048576.0)});
      }
    }
  }
  if (cnt) add(cnt, {(long long)q[0], (long long)q[1], (long long)q[2]});
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += 64 * WAVES) {
    const long long t[3] = {(long long)tsum[0][e], (long long)tsum[1][e], (long long)tsum[2][e]};
    add_stats(tseg[e], tcnt[e], t, size0, colsum);
  }
}

// Block-wide exclusive prefix of v (kT threads); the total to every thread.
__device__ __forceinline__ int block_prefix(int v, int* sh, int& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) sh[wv] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kT / 64; ++w) {
    if (w < wv) before += sh[w];
    total += sh[w];
  }
  __syncthreads();  // sh may be rewritten
  return before + incl - v;
}

// The block's share of n elements, a contiguous chunk of whole groups of PER
// elements (so that its segments span few images and one atomic serves many):
// [begin, end).
template <int PER>
__device__ __forceinline__ void block_chunk(int n, int& begin, int& end) {
  const int groups = (n + PER - 1) / PER, per = (groups + gridDim.x - 1) / gridDim.x;
  begin = (int)min((int64_t)blockIdx.x * per * PER, (int64_t)n);
  end = (int)min((int64_t)begin + (int64_t)per * PER, (int64_t)n);
}

// A count per image of the segments whose predicate holds.  Each wave keeps it for
// the image it is in and adds it to memory when the image changes; at the end the
// block adds its waves' last counts together.  (Atomics on one cache line take
// about 10 ns each: one per wave and 64 segments took 300 us on 2.67 million.)
struct ImageCount {
  int b = -1, c = 0;  // wave-uniform
  __device__ __forceinline__ void add(int* counts, int column, int img, bool valid, bool pred) {
    unsigned long long v = __ballot(valid);
    while (v) {  // the images of this wave's segments: mostly one
      const int first = __ffsll(v) - 1;
      const int i = __shfl(img, first, 64);
      const unsigned long long mine = __ballot(valid && img == i);
      if (i != b) {
        if (c && (threadIdx.x & 63) == 0) atomicAdd(counts + 4 * b + column, c);
        b = i;
        c = 0;
      }
      c += __popcll(__ballot(valid && img == i && pred));
      v &= ~mine;
    }
  }
  __device__ __forceinline__ void finish(int* counts, int column) {
    __shared__ int sb[kT / 64], sc[kT / 64];
    if ((threadIdx.x & 63) == 0) {
      sb[threadIdx.x >> 6] = b;
      sc[threadIdx.x >> 6] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 0; w < kT / 64; ++w) {
        int t = sc[w];
        if (w + 1 < kT / 64 && sb[w + 1] == sb[w]) sc[w + 1] += t;
        else if (t) atomicAdd(counts + 4 * sb[w] + column, t);
      }
    }
  }
};

constexpr int kPer = 4;  // segments per thread between two block-wide prefixes

// means (in place of the sums), owners, cluster parents (a large segment's is -1,
// which marks it large from here on, a small one's itself), the small segments
// per image, and room in the pixel list for the small segments of two or more
// pixels, in any order (poff -1: no list; a single pixel is the segment's root)
__global__ __launch_bounds__(kT) void k_seg_prep(const ImgDesc* img, const int* n_seg_dev,
                                                 const int* seg_img, const int* size0,
                                                 unsigned long long* colsum, int* mpar, int* cpar,
                                                 int* poff, int* cnt, int* counts) {
  __shared__ int sh[kT / 64];
  __shared__ int base_s;
  const int n_seg = *n_seg_dev;
  int begin, end;
  block_chunk<kT>(n_seg, begin, end);
  ImageCount ic;
  for (int s0 = begin; s0 < end; s0 += kPer * kT) {
    int want[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int s = s0 + k * kT + threadIdx.x;
      const bool in = s < end;
      int n = 0, b = 0;
      bool small = false;
      if (in) {
        n = size0[s];
        b = seg_img[s];
        double* mean = reinterpret_cast<double*>(colsum + 3 * (int64_t)s);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const long long q = (long long)colsum[3 * (int64_t)s + c];
          mean[c] = (double)q / (double)n * 0x1p-20;
        }
        small = 4LL * n < (int64_t)img[b].vx * img[b].vy;
        mpar[s] = s;
        cpar[s] = small ? s : -1;
      }
      ic.add(counts, 1, b, in, small);
      want[k] = small && n > 1 ? n : 0;
      sum += want[k];
    }
    int total;
    int at = block_prefix(sum, sh, total);
    if (threadIdx.x == 0) base_s = total ? atomicAdd(cnt + N_PX, total) : 0;
    __syncthreads();
    at += base_s;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int s = s0 + k * kT + threadIdx.x;
      if (s < end) poff[s] = want[k] ? at : -1;
      at += want[k];
    }
    __syncthreads();  // base_s is rewritten
  }
  ic.finish(counts, 1);
}

// the pixel lists, four consecutive pixels of the batch per thread
__global__ __launch_bounds__(kT) void k_px_fill(int n_pix, const int* segid, const int* poff,
                                                int* cursor, int* plist) {
  const int64_t i0 = 4 * ((int64_t)blockIdx.x * kT + threadIdx.x);
  if (i0 >= n_pix) return;
  int s[4], p[4];
  if (i0 + 4 <= n_pix) {  // segid is 256-byte aligned
    const int4 w = *reinterpret_cast<const int4*>(segid + i0);
    s[0] = w.x; s[1] = w.y; s[2] = w.z; s[3] = w.w;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = i0 + k < n_pix ? segid[i0 + k] : -1;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k] = s[k] >= 0 ? (k > 0 && s[k] == s[k - 1] ? p[k - 1] : poff[s[k]]) : -1;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (p[k] >= 0) plist[p[k] + atomicAdd(cursor + s[k], 1)] = (int)(i0 + k);
}

constexpr int kOwnPixels = 4;  // pixels that a thread visits by itself

// One thread per small segment (a wave for the pixels of a segment of more than
// kOwnPixels).  If its neighbours are all large (they never
// merge, so they own themselves) its visit depends on nothing else and is made
// here; otherwise it joins its small neighbours' cluster.  Bound by the gathers
// of the neighbours' indices and means.  On 8 x 3840x2160 after T = 10 (2.58
// million small segments, 1.61 million of them alone) it takes
// 439 us; a pass over all pixels for the clusters and one thread per cluster, with
// the lone segments taking the general path, took 536 + 1586 us.
__global__ __launch_bounds__(kT) void k_merge_single(const ImgDesc* img, const int* n_seg_dev,
                                                     const int* seg_img, const int* seg_root,
                                                     const int* size0, const int* poff,
                                                     const int* plist, const int* segid,
                                                     const double* mean, int* cpar, int* mpar,
                                                     int* clist, int* cnt) {
  __shared__ int sh[kT / 64];
  __shared__ int base_s;
  const int n_seg = *n_seg_dev;
  int begin, end;
  block_chunk<kT>(n_seg, begin, end);
  for (int s0 = begin; s0 < end; s0 += kPer * kT) {
    unsigned clustered = 0;  // bit k: segment s0 + k kT + threadIdx.x
#pragma unroll 1
    for (int k = 0; k < kPer && s0 + k * kT < end; ++k) {
      const int s = s0 + k * kT + threadIdx.x;
      // (the sign of cpar, unlike its value, does not change here: plain loads)
      const bool mine = s < end && cpar[s] >= 0;
      int np = 0, p0 = 0, root = 0, W = 1, H = 0, off = 0;
      if (mine) {
        const ImgDesc& I = img[seg_img[s]];
        W = I.W;
        H = I.H;
        off = (int)I.pix_off;
        np = size0[s];
        p0 = poff[s];
        root = seg_root[s];
      }
      int best = -1;
      double bd = 0.0;
      bool joined = false;
      // neighbour e of pixel u of segment sg, colour mg
      auto visit = [&](int sg, const double* mg, int j, int e, int w, int h, int of, int& last) {
        const int x = j % w, y = j / w;
        const bool in = e == 0 ? y > 0 : e == 1 ? y + 1 < h : e == 2 ? x > 0 : x + 1 < w;
        if (!in) return;
        const int o = segid[of + j + (e == 0 ? -w : e == 1 ? w : e == 2 ? -1 : 1)];
        if (o == sg || o == last) return;  // itself, or the neighbour just seen
        last = o;
        if (cpar[o] >= 0) {
          joined = true;
          if (o < sg) uf_unite(cpar, sg, o);  // (the other segment joins the rest)
          return;
        }
        const double d = colour_dist2(mg, mean + 3 * (int64_t)o);
        if (best < 0 || d < bd || (d == bd && o < best)) {
          best = o;
          bd = d;
        }
      };
      if (np <= kOwnPixels) {
        const double* m = mean + 3 * (int64_t)s;
        const double ms[3] = {np ? m[0] : 0.0, np ? m[1] : 0.0, np ? m[2] : 0.0};
        int last = s;
        for (int u = 0; u < np; ++u) {
          const int j = (p0 >= 0 ? plist[p0 + u] : root) - off;
#pragma unroll
          for (int e = 0; e < 4; ++e) visit(s, ms, j, e, W, H, off, last);
        }
      }
      // the pixels of a larger segment over the whole wave
      for (unsigned long long big = __ballot(np > kOwnPixels); big; big &= big - 1) {
        const int l = __ffsll(big) - 1;
        const int sg = __shfl(s, l, 64), pp = __shfl(p0, l, 64), n4 = 4 * __shfl(np, l, 64);
        const int w = __shfl(W, l, 64), h = __shfl(H, l, 64), of = __shfl(off, l, 64);
        const int keep_best = best;
        const double keep_bd = bd;
        const bool keep_joined = joined;
        const double* m = mean + 3 * (int64_t)sg;
        const double mg[3] = {m[0], m[1], m[2]};
        best = -1;
        joined = false;
        int last = sg;
        for (int u = (int)(threadIdx.x & 63); u < n4; u += 64)
          visit(sg, mg, plist[pp + (u >> 2)] - of, u & 3, w, h, of, last);
        joined = __ballot(joined) != 0;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
          const double od = __shfl_xor(bd, o, 64);
          const int ob = __shfl_xor(best, o, 64);
          if (ob >= 0 && (best < 0 || od < bd || (od == bd && ob < best))) {
            best = ob;
            bd = od;
          }
        }
        if ((int)(threadIdx.x & 63) != l) {  // lane l keeps the result, the others theirs
          best = keep_best;
          bd = keep_bd;
          joined = keep_joined;
        }
      }
      // (no small neighbour, so cpar[s] = s: nothing else joins this segment)
      if (joined) clustered |= 1u << k;
      else if (mine && best >= 0) mpar[s] = best;
    }
    int total;
    int at = block_prefix(__popc(clustered), sh, total);
    if (threadIdx.x == 0) base_s = total ? atomicAdd(cnt + N_CLUSTERED, total) : 0;
    __syncthreads();
    at += base_s;
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (clustered >> k & 1) clist[at++] = s0 + k * kT + threadIdx.x;
    __syncthreads();  // base_s is rewritten
  }
}

// the clustered sources per cluster root
__global__ __launch_bounds__(kT) void k_cl_count(const int* clist, const int* cnt, int* cpar,
                                                 int* ccnt) {
  const int n = cnt[N_CLUSTERED];
  for (int i = blockIdx.x * kT + threadIdx.x; i < n; i += gridDim.x * kT) {
    const int s = clist[i];
    const int r = uf_find(cpar, s);
    st_dev(cpar + s, r);  // (an ancestor: finds that pass through it stay right)
    atomicAdd(ccnt + r, 1);
  }
}

// clusters of at most kTeam8 sources go to 8 lanes, of at most kTeam16 to 16
// lanes, others to a wave
constexpr int kTeam8 = 4, kTeam16 = 12;

// Room in the cluster lists and the lists of clusters by class, in any order: those
// for 8 lanes from team[0] up, those for 16 lanes from team[half - 1] down.
__global__ __launch_bounds__(kT) void k_cl_alloc(const int* clist, const int* cpar, const int* ccnt,
                                                 int* coff, int* cnt, int* team, int half, int* wave) {
  __shared__ int sh[kT / 64];
  __shared__ int base_s[4];
  const int n = cnt[N_CLUSTERED];
  int begin, end;
  block_chunk<kT>(n, begin, end);
  for (int i0 = begin; i0 < end; i0 += kPer * kT) {
    int root[kPer], c[kPer], n_list = 0, n8 = 0, n16 = 0, nw = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = i0 + k * kT + threadIdx.x;
      const int r = i < end ? clist[i] : -1;
      root[k] = r >= 0 && cpar[r] == r ? r : -1;
      c[k] = root[k] >= 0 ? ccnt[r] : 0;
      n_list += c[k];
      if (root[k] >= 0) (c[k] <= kTeam8 ? n8 : c[k] <= kTeam16 ? n16 : nw) += 1;
    }
    static_assert(kPer * kT < 65536, "two classes share a prefix, 16 bits each");
    int all_list, all_teams, all_waves;
    int at0 = block_prefix(n_list, sh, all_list);
    const int at = block_prefix(n8 | n16 << 16, sh, all_teams);
    int atw = block_prefix(nw, sh, all_waves);
    if (threadIdx.x == 0) base_s[0] = atomicAdd(cnt + N_LISTED, all_list);
    if (threadIdx.x == 64) base_s[1] = atomicAdd(cnt + N_TEAM8, all_teams & 0xFFFF);
    if (threadIdx.x == 128) base_s[2] = atomicAdd(cnt + N_TEAM16, all_teams >> 16);
    if (threadIdx.x == 192) base_s[3] = atomicAdd(cnt + N_WAVE, all_waves);
    __syncthreads();
    at0 += base_s[0];
    int at8 = base_s[1] + (at & 0xFFFF), at16 = base_s[2] + (at >> 16);
    atw += base_s[3];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (root[k] < 0) continue;
      coff[root[k]] = at0;
      at0 += c[k];
      if (c[k] <= kTeam8) team[at8++] = root[k];
      else if (c[k] <= kTeam16) team[half - 1 - at16++] = root[k];
      else wave[atw++] = root[k];
    }
    __syncthreads();  // base_s is rewritten
  }
}

// Cluster lists (any order): the sources, and beside each its size and where its
// pixels are (an offset in the pixel list, or ~ the one pixel), so that a merge
// finds them one load behind the list.
__global__ __launch_bounds__(kT) void k_cl_fill(const int* clist, const int* cnt, const int* cpar,
                                                const int* coff, const int* size0, const int* poff,
                                                const int* seg_root, int* ccur, int* list,
                                                int* lsize, int* lpix) {
  const int n = cnt[N_CLUSTERED];
  for (int i = blockIdx.x * kT + threadIdx.x; i < n; i += gridDim.x * kT) {
    const int s = clist[i], r = cpar[s];
    const int at = coff[r] + atomicAdd(ccur + r, 1);
    const int p = poff[s];
    list[at] = s;
    lsize[at] = size0[s];
    lpix[at] = p >= 0 ? p : ~seg_root[s];
  }
}

// pixel u of a listed source
__device__ __forceinline__ int list_pixel(int where, int u, const int* plist) {
  return where >= 0 ? plist[where + u] : ~where;
}

// Clusters: the procedure in rounds, all of a cluster's sources at once.
//
// A source's visit reads its own pixels and size and the owners of its
// neighbouring pixels.  Of what an undecided source v can still change, a
// source s sees only merges of v itself when v currently owns a neighbour of s
// (a merge into v changes v's pixels and size, which s does not read).  So s
// can be decided as soon as no undecided segment that owns a neighbour of s
// precedes it in (size, id) order, and its decision is then the one of the
// sequential procedure.  Two sources decided in the same round do not own
// neighbours of each other (the later one would have waited), so their merges
// commute.  The first undecided source is always ready: every round decides
// at least one.  The depth is that of a greedy pass over the order (18 rounds
// for 202 825 sources of a noisy 4K image, half of the rest decided in each).
//
// A round drops the entries of decided sources and of pairs that have become one
// segment, then makes two passes over the rest: the first marks the sources that
// must wait and takes each source's smallest colour distance, the second the
// smallest id at that distance; then the ready sources are decided and the owner
// links shortened to the roots.
//
// With the state in LDS the entries are spread over the lanes.  Bound by the
// latency of LDS and of the gathers that set a cluster up.  Four sizes of team:
// 8 or 16 lanes and 1.8 or 3.4 KB of LDS for up to 4 or 12 sources (94 % of the
// clusters have at most 8), a wave and 14 KB for more (11 waves per CU hide each
// other's latency), and a block of 1024 threads for what does not fit those (twice
// as fast as one of 512), in LDS or, for a cluster larger still, with the state in
// memory (a noisy image can be one cluster of a million sources).  On the labels of
// 8 x 3840x2160 after T = 10 (2.67 million segments, 169 000 clusters of 2 to 852
// sources) the teams take 299 us, the waves 167 and the blocks 254; 370, 300 and
// 377 us when every round passed over all entries.  Visiting the sources of a
// cluster one after the other, on one thread up to 16 sources and then a wave, took
// 1586 + 12 470 us.
constexpr unsigned short kNone = 0xFFFF;

template <int CAP, int PX>  // members + external neighbours; pixels of the members
struct ClusterLds {
  static constexpr int kHashBits = CAP == 16 ? 5 : CAP == 32 ? 6 : CAP == 128 ? 8 : 11;  // twice CAP entries
  static constexpr int kHash = 1 << kHashBits;
  static_assert(kHash == 2 * CAP && kHash < kNone, "16-bit indices");
  unsigned long long key[CAP];   // (size, id) of a member; the id of an external neighbour
  unsigned long long bd[CAP];    // smallest distance of the round (bits of a double >= 0)
  unsigned long long bk[CAP];    // 0: must wait; else 1 + (id << 16 | local index) at bd
  double mean[CAP][3];
  int sz[CAP];                   // current size of each member
  int pref[CAP];                 // first pixel of each member
  int pix[CAP];                  // where its pixels are (list_pixel)
  int hkey[kHash];               // segment id -> local index
  unsigned short hval[kHash];
  unsigned short own[CAP];       // owner (local index); itself while it is a segment
  unsigned ent[4 * PX];          // entries: member << 16 | neighbour (local indices)
  unsigned char open[CAP];       // 1: not yet decided
  int wave_n[2][CAP > 128 ? 16 : 1];  // entries kept per wave of a block
  int n_loc, n_pix, overflow;
};

template <int T>
__device__ __forceinline__ void team_sync() {
  if constexpr (T <= 64) {  // lanes of one wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// table slot of segment id; a new id gets the next local index
template <int CAP, int PX>
__device__ int lds_slot(ClusterLds<CAP, PX>& S, int id) {
  constexpr int kHash = ClusterLds<CAP, PX>::kHash;
  int e = (int)(((unsigned)id * 2654435761u) >> (32 - ClusterLds<CAP, PX>::kHashBits));
  for (int probe = 0; probe < kHash; ++probe, e = (e + 1) & (kHash - 1)) {
    // (a plain read first: most neighbours are the same few large segments)
    int k = __hip_atomic_load(&S.hkey[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (k == id) return e;
    if (k == -1) k = atomicCAS(&S.hkey[e], -1, id);
    if (k == -1) {
      const int x = atomicAdd(&S.n_loc, 1);
      S.hval[e] = (unsigned short)(x < CAP ? x : kNone);
      if (x < CAP) {
        S.key[x] = (unsigned)id;
        S.own[x] = (unsigned short)x;
        S.open[x] = 0;
      } else {
        S.overflow = 1;
      }
    }
    if (k == -1 || k == id) return e;
  }
  S.overflow = 1;
  return -1;
}

// what the merges read and write
struct MergePtrs {
  const ImgDesc* img;
  const int *seg_img, *list, *lsize, *lpix, *plist, *segid;
  const double* mean;
  int *ccnt, *coff, *mpar;
  // the block merges with the state in memory
  const int *size0, *poff, *seg_root;
  int *cpar, *link, *tail, *work0, *work1;
};

// One cluster (root r) by the T threads of a team, t = 0 .. T - 1.  False, with
// nothing written to memory, if it does not fit.
template <int T, int CAP, int PX>
__device__ bool merge_rounds(ClusterLds<CAP, PX>& S, int t, int r, const MergePtrs& M) {
  const int n = M.ccnt[r], l0 = M.coff[r];
  const ImgDesc& I = M.img[M.seg_img[r]];
  if (n > CAP) return false;
  const int W = I.W, H = I.H;
  const int off = (int)I.pix_off;
  const int64_t desired = (int64_t)I.vx * I.vy;
  for (int e = t; e < ClusterLds<CAP, PX>::kHash; e += T) S.hkey[e] = -1;
  if (t == 0) {
    S.n_loc = S.n_pix = S.overflow = 0;
  }
  team_sync<T>();
  // the members, in any order: ids, sizes, first pixels
  for (int q = t; q < n; q += T) {
    const int g = M.list[l0 + q], sz = M.lsize[l0 + q];
    S.pix[q] = M.lpix[l0 + q];
    S.pref[q] = atomicAdd(&S.n_pix, sz);
    S.sz[q] = sz;
    S.key[q] = ((unsigned long long)sz << 32) | (unsigned)g;
    S.own[q] = (unsigned short)q;
    S.open[q] = 1;
    int e = (int)(((unsigned)g * 2654435761u) >> (32 - ClusterLds<CAP, PX>::kHashBits));
    while (atomicCAS(&S.hkey[e], -1, g) != -1) e = (e + 1) & (ClusterLds<CAP, PX>::kHash - 1);
    S.hval[e] = (unsigned short)q;
  }
  if (t == 0) S.n_loc = n;
  team_sync<T>();
  const int np = S.n_pix;
  if (np > PX) return false;
  for (int q = t; q < n; q += T) {
    const int p0 = S.pref[q], sz = S.sz[q];
    for (int u = 0; u < sz; ++u) S.ent[4 * (p0 + u)] = (unsigned)q << 16;
  }
  team_sync<T>();
  // the neighbours (up, down, left, right) of every pixel: table slots first
  for (int u = t; u < np; u += T) {
    const int q = (int)(S.ent[4 * u] >> 16);
    const int g = (int)(unsigned)S.key[q];
    const int j = list_pixel(S.pix[q], u - S.pref[q], M.plist) - off;
    const int x = j % W, y = j / W;
    const int* at = M.segid + off + j;
    int nb[4];
    nb[0] = y > 0 ? at[-W] : g;
    nb[1] = y + 1 < H ? at[W] : g;
    nb[2] = x > 0 ? at[-1] : g;
    nb[3] = x + 1 < W ? at[1] : g;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int e = nb[k] != g ? lds_slot(S, nb[k]) : -1;
      S.ent[4 * u + k] = (unsigned)q << 16 | (e >= 0 ? (unsigned)e : (unsigned)kNone);
    }
  }
  team_sync<T>();
  if (S.overflow) return false;
  for (int u = t; u < 4 * np; u += T) {
    const unsigned e = S.ent[u], slot = e & 0xFFFFu;
    if (slot != kNone) S.ent[u] = (e & 0xFFFF0000u) | S.hval[slot];
  }
  const int nl = S.n_loc;
  for (int i = t; i < nl; i += T) {
    const double* m = M.mean + 3 * (int64_t)(unsigned)S.key[i];
    S.mean[i][0] = m[0];
    S.mean[i][1] = m[1];
    S.mean[i][2] = m[2];
  }
  // The entries of undecided sources between different segments, moved to the
  // front in place, as entries of the current owners: what is dropped stays
  // dropped, so a round's work halves with its sources.  (A chunk is read by every
  // thread before any of it is overwritten, and the writes lie behind the reads.)
  auto compact = [&](int live) {
    int out = 0, par = 0;
    for (int base = 0; base < live; base += T) {
      const int u = base + t;
      unsigned v = 0;
      bool keep = false;
      if (u < live) {
        v = S.ent[u];
        if ((v & 0xFFFFu) != kNone) {
          const unsigned s = S.own[v >> 16], o = S.own[v & 0xFFFFu];
          keep = s != o && S.open[s];
          v = s << 16 | o;
        }
      }
      const unsigned long long m = __ballot(keep);
      if constexpr (T <= 64) {  // this team's lanes of the wave's ballot
        const unsigned long long mine = T == 64 ? m : m >> ((threadIdx.x & 63) & ~(T - 1)) & ((1ull << (T & 63)) - 1);
        team_sync<T>();
        if (keep) S.ent[out + __popcll(mine & ((1ull << t) - 1))] = v;
        out += __popcll(mine);
      } else {
        const int lane = t & 63, wv = t >> 6;
        if (lane == 0) S.wave_n[par][wv] = __popcll(m);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < T / 64; ++w) {
          const int c = S.wave_n[par][w];
          if (w < wv) before += c;
          total += c;
        }
        if (keep) S.ent[out + before + __popcll(m & ((1ull << lane) - 1))] = v;
        out += total;
        par ^= 1;
      }
    }
    team_sync<T>();
    return out;
  };
  team_sync<T>();
  int live = 4 * np;
  while (true) {
    // owner links shortened to the roots (an owner read here while it is being
    // shortened is an ancestor), the undecided sources' minima reset
    int any = 0;
    for (int q = t; q < n; q += T) {
      int x = S.own[q];
      while (S.own[x] != x) x = S.own[x];
      S.own[q] = (unsigned short)x;
      if (S.open[q]) {
        S.bd[q] = ~0ull;
        S.bk[q] = ~0ull;
        any = 1;
      }
    }
    if constexpr (T <= 64) {  // this team's lanes of the wave's ballot
      const unsigned long long m = __ballot(any) >> ((threadIdx.x & 63) & ~(T - 1));
      if ((T == 64 ? m : m & ((1ull << (T & 63)) - 1)) == 0) break;
      team_sync<T>();
    } else {
      if (!__syncthreads_or(any)) break;
    }
    live = compact(live);
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
      for (int u = t; u < live; u += T) {
        const unsigned v = S.ent[u];
        const int s = (int)(v >> 16), o = (int)(v & 0xFFFFu);
        if (S.open[o] && S.key[o] < S.key[s]) {
          S.bk[s] = 0;  // (the smallest value: no minimum raises it again)
          continue;
        }
        const unsigned long long d =
            (unsigned long long)__double_as_longlong(colour_dist2(S.mean[s], S.mean[o]));
        // (a value that does not lower the minimum needs no atomic: the lanes of a
        // source mostly meet the same few neighbours, and LDS atomics on one
        // address follow one another)
        if (pass == 0) {
          if (d < S.bd[s]) atomicMin(&S.bd[s], d);
        } else if (d == S.bd[s]) {
          const unsigned long long k = (((S.key[o] & 0xFFFFFFFFull) << 16) | (unsigned)o) + 1;
          if (k < S.bk[s]) atomicMin(&S.bk[s], k);
        }
      }
      team_sync<T>();
    }
    for (int q = t; q < n; q += T) {
      const unsigned long long k = S.bk[q];
      if (!S.open[q] || k == 0) continue;
      S.open[q] = 0;
      if (4LL * S.sz[q] >= desired || k == ~0ull) continue;  // grown, or no neighbour
      const int o = (int)((k - 1) & 0xFFFF);
      S.own[q] = (unsigned short)o;
      if (o < n) atomicAdd(&S.sz[o], S.sz[q]);
    }
    team_sync<T>();
  }
  // the final owners, as segment ids (a large segment's size is read by no
  // decision and no output)
  for (int q = t; q < n; q += T)
    M.mpar[(int)(unsigned)S.key[q]] = (int)(unsigned)S.key[S.own[q]];
  team_sync<T>();  // the state is rewritten by the next cluster
  return true;
}

// Small clusters, 8 lanes (even blocks) or 16 lanes (odd blocks) each; what does
// not fit goes to the waves' list.
template <int T, int CAP, int PX>
__device__ __forceinline__ void merge_teams(ClusterLds<CAP, PX>* S, const MergePtrs& M, int* cnt,
                                            int* wave, const int* team, int step, int n) {
  const int t = threadIdx.x % T, g = threadIdx.x / T;
  constexpr int kG = 64 / T;
  for (int c = (blockIdx.x >> 1) * kG + g; c < n; c += (gridDim.x >> 1) * kG) {
    const int r = team[c * step];
    if (!merge_rounds<T, CAP, PX>(S[g], t, r, M) && t == 0) wave[atomicAdd(cnt + N_WAVE, 1)] = r;
    team_sync<T>();
  }
}

__global__ __launch_bounds__(64) void k_merge_team(MergePtrs M, int* cnt, const int* team, int half,
                                                   int* wave) {
  __shared__ union {
    ClusterLds<16, 32> s8[8];
    ClusterLds<32, 64> s16[4];
  } S;
  if (blockIdx.x & 1)
    merge_teams<16>(S.s16, M, cnt, wave, team + half - 1, -1, cnt[N_TEAM16]);
  else
    merge_teams<8>(S.s8, M, cnt, wave, team, 1, cnt[N_TEAM8]);
}

// Larger clusters, a wave each; what does not fit is listed in rest.
__global__ __launch_bounds__(64) void k_merge_wave(MergePtrs M, int* cnt, const int* wave, int* rest) {
  __shared__ ClusterLds<128, 256> S;
  const int t = threadIdx.x, n = cnt[N_WAVE];
  for (int c = blockIdx.x; c < n; c += gridDim.x) {
    const int r = wave[c];
    if (!merge_rounds<64>(S, t, r, M) && t == 0) rest[atomicAdd(cnt + N_BLOCK, 1)] = r;
    team_sync<64>();
  }
}

// The clusters left over, a block each: in LDS if they fit, else with the state in
// memory and lists of the sources to look at.
//
// A source that some undecided owner of a neighbour precedes waits for that one:
// nothing else can make it ready.  It is entered in that owner's list of waiters and
// looked at again when the owner is decided, so a source is looked at as often as it
// meets another one to wait for (3.4 times in noise), and a round costs what changed in
// it.  (With passes over all entries in every round, noise, of which a round decides
// some ten sources, took 1.7 s for 192 x 192 pixels, 0.46 s one source after the
// other; it takes 46 ms.)  A source that has grown to a quarter of the desired size will
// do nothing at its turn, so it is decided at once.  Every undecided source is in
// the next list or waits for an undecided one that precedes it; the first of all
// waits for none, so every round decides a source.
//
// Per segment: size in ccnt; head, the first waiter (kNoWaiter, or kDecided), in
// coff; the next waiter in cpar (a large segment's is -1); the segments merged into a
// source are linked from it by link, tail the last of them.  A cluster's own ccnt and
// coff are read before its segments' entries of them serve for this.  Owners are
// changed between barriers that no look-up crosses, and two sources decided
// between the same ones do not own neighbours of each other.
constexpr int kHugeT = 1024;
constexpr int kNoWaiter = -1, kDecided = -2, kLastWaiter = INT32_MAX;
constexpr int kWide = 128;      // sources in a list from which on a lane takes one each
constexpr int kLanePixels = 8;  // of up to so many pixels; a wave takes a larger one

// a source's look at its neighbours
struct Look {
  int best = -1, blocker = -1;
  double bd = 0.0;
};

// current owner of segment nb, the walk shortened for the next one (no owner
// changes meanwhile)
__device__ __forceinline__ int owner_of(int* mpar, int nb) {
  const int u = ld_dev(mpar + nb);
  const int t = m_find(mpar, u);
  if (t != u) st_dev(mpar + nb, t);
  return t;
}

// neighbour k of pixel j (of member m) for source s, colour ms
__device__ __forceinline__ void look_at(const MergePtrs& M, const ImgDesc& I, int off, int s, int key,
                                        const double* ms, int m, int j, int k, Look& L) {
  const int W = I.W, H = I.H;
  const int x = j % W, y = j / W;
  const bool in = k == 0 ? y > 0 : k == 1 ? y + 1 < H : k == 2 ? x > 0 : x + 1 < W;
  if (!in) return;
  const int nb = M.segid[off + j + (k == 0 ? -W : k == 1 ? W : k == 2 ? -1 : 1)];
  if (nb == m) return;
  const int o = owner_of(M.mpar, nb);
  if (o == s) return;
  if (ld_dev(M.cpar + o) != -1 && ld_dev(M.coff + o) != kDecided) {
    const int ko = M.size0[o];
    if (ko < key || (ko == key && o < s)) {
      L.blocker = o;
      return;
    }
  }
  const double d = colour_dist2(ms, M.mean + 3 * (int64_t)o);
  if (L.best < 0 || d < L.bd || (d == L.bd && o < L.best)) {
    L.best = o;
    L.bd = d;
  }
}

__device__ __forceinline__ int seg_pixel(const MergePtrs& M, int m, int u) {
  const int p = M.poff[m];
  return p >= 0 ? M.plist[p + u] : M.seg_root[m];
}

// one lane
__device__ Look look_lane(const MergePtrs& M, const ImgDesc& I, int off, int s) {
  Look L;
  const int key = M.size0[s];
  const double* m3 = M.mean + 3 * (int64_t)s;
  const double ms[3] = {m3[0], m3[1], m3[2]};
  for (int m = s; m >= 0 && L.blocker < 0; m = ld_dev(M.link + m)) {
    const int np = M.size0[m];
    for (int u = 0; u < np && L.blocker < 0; ++u) {
      const int j = seg_pixel(M, m, u) - off;
#pragma unroll
      for (int k = 0; k < 4; ++k) look_at(M, I, off, s, key, ms, m, j, k, L);
    }
  }
  return L;
}

// the whole wave; s and the result are the same in every lane
__device__ Look look_wave(const MergePtrs& M, const ImgDesc& I, int off, int s) {
  Look L;
  const int lane = threadIdx.x & 63;
  const int key = M.size0[s];
  const double* m3 = M.mean + 3 * (int64_t)s;
  const double ms[3] = {m3[0], m3[1], m3[2]};
  int m = s;
  while (m >= 0) {
    // up to sixteen members of up to 16 pixels, four lanes each, then a larger one
    int mine = -1, large = -1;
    for (int c = 0; c < 16 && m >= 0 && large < 0; ++c) {
      if (M.size0[m] > 16) large = m;
      else if (c == lane >> 2) mine = m;
      m = ld_dev(M.link + m);
    }
    if (mine >= 0) {
      const int np = M.size0[mine];
      for (int u = 0; u < np; ++u)
        look_at(M, I, off, s, key, ms, mine, seg_pixel(M, mine, u) - off, lane & 3, L);
    }
    if (large >= 0) {
      const int n4 = 4 * M.size0[large];
      for (int u = lane; u < n4; u += 64)
        look_at(M, I, off, s, key, ms, large, seg_pixel(M, large, u >> 2) - off, u & 3, L);
    }
    const unsigned long long blocked = __ballot(L.blocker >= 0);
    if (blocked) {
      L.blocker = __shfl(L.blocker, __ffsll(blocked) - 1, 64);
      return L;
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double od = __shfl_xor(L.bd, o, 64);
    const int ob = __shfl_xor(L.best, o, 64);
    if (ob >= 0 && (L.best < 0 || od < L.bd || (od == L.bd && ob < L.best))) {
      L.best = ob;
      L.bd = od;
    }
  }
  return L;
}

// one cluster (root r, n sources from place l0 of the list on), the whole block
__device__ void merge_lists(const MergePtrs& M, int r, int n, int l0) {
  __shared__ int n_next;
  const int t = threadIdx.x, lane = t & 63;
  const ImgDesc& I = M.img[M.seg_img[r]];
  const int off = (int)I.pix_off;
  const int64_t desired = (int64_t)I.vx * I.vy;
  int* const size = M.ccnt;
  int* const head = M.coff;
  for (int q = t; q < n; q += kHugeT) {
    const int s = M.list[l0 + q];
    st_dev(size + s, M.lsize[l0 + q]);
    st_dev(head + s, kNoWaiter);
    st_dev(M.link + s, -1);
    st_dev(M.tail + s, s);
  }
  if (t == 0) n_next = 0;
  __syncthreads();  // (the places of lpix serve as a list from here on)
  const int* src = M.list + l0;
  int* dst = M.work0 + l0;
  int cnt = n;
  // a decided source's waiters go to the next list
  auto release = [&](int w) {
    while (w >= 0 && w != kLastWaiter) {
      const int nx = ld_dev(M.cpar + w);
      st_dev(dst + atomicAdd(&n_next, 1), w);
      w = nx;
    }
  };
  for (int round = 0; cnt > 0 && round < n; ++round) {
    const bool wide = cnt > kWide;
    const int per = wide ? kHugeT : kHugeT / 64;
    for (int base = 0; base < cnt; base += per) {
      // this lane's source (of a wave's one source: lane 0's)
      const int q = base + (wide ? t : t >> 6);
      int s = q < cnt ? ld_dev(src + q) : -1;
      if (s >= 0 && ld_dev(head + s) == kDecided) s = -1;
      Look L;
      if (wide) {
        const int np = s >= 0 ? ld_dev(size + s) : 0;
        if (s >= 0 && np <= kLanePixels) L = look_lane(M, I, off, s);
        for (unsigned long long big = __ballot(np > kLanePixels); big; big &= big - 1) {
          const int l = __ffsll(big) - 1;
          const Look B = look_wave(M, I, off, __shfl(s, l, 64));
          if (lane == l) L = B;
        }
      } else if (s >= 0) {  // (the same in the whole wave)
        L = look_wave(M, I, off, s);
        if (lane != 0) s = -1;
      }
      if (s >= 0 && L.blocker >= 0) {
        const int w = atomicExch(head + L.blocker, s);
        st_dev(M.cpar + s, w >= 0 ? w : kLastWaiter);
        s = -1;
      }
      __syncthreads();
      if (s >= 0) {
        release(atomicExch(head + s, kDecided));
        const int o = L.best;
        if (o >= 0) {
          st_dev(M.mpar + s, o);
          if (ld_dev(M.cpar + o) != -1) {  // a source, or one that was: not a large segment
            const int sz = ld_dev(size + s);
            const int old = atomicAdd(size + o, sz);
            if (ld_dev(head + o) != kDecided) {
              const int ln = atomicExch(M.link + o, s), tl = ld_dev(M.tail + s);
              st_dev(M.link + tl, ln);
              if (ln < 0) st_dev(M.tail + o, tl);
            }
            if (4LL * old < desired && 4LL * (old + sz) >= desired)
              release(atomicExch(head + o, kDecided));
          }
        }
      }
      __syncthreads();
    }
    cnt = n_next;
    src = dst;
    dst = (dst == M.work0 + l0 ? M.work1 : M.work0) + l0;
    __syncthreads();  // every thread has read n_next
    if (t == 0) n_next = 0;
    __syncthreads();
  }
  // the walks shortened for the output
  for (int q = t; q < n; q += kHugeT) owner_of(M.mpar, M.list[l0 + q]);
}

__global__ __launch_bounds__(kHugeT) void k_merge_block(MergePtrs M, const int* cnt, const int* rest) {
  __shared__ ClusterLds<1024, 4608> S;
  const int nr = cnt[N_BLOCK];
  for (int c = blockIdx.x; c < nr; c += gridDim.x) {
    const int r = rest[c];
    if (merge_rounds<kHugeT>(S, threadIdx.x, r, M)) continue;
    const int n = M.ccnt[r], l0 = M.coff[r];
    __syncthreads();  // every thread has read n and l0
    merge_lists(M, r, n, l0);
    __syncthreads();  // (n_next is used again)
  }
}

// ranks of the final segments: for each segment the number of final segments
// before it in its block of kScanBlock, and the block counts
__global__ __launch_bounds__(kT) void k_final_rank(const int* n_seg_dev, const int* mpar, int* rank,
                                                   int* bsum) {
  __shared__ int sh[kT / 64];
  const int n = *n_seg_dev;
  if ((int64_t)blockIdx.x * kScanBlock >= n) return;  // the whole block
  const int base = blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  int v[kScanPer];
  int t = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = base + k < n && mpar[base + k] == base + k;
    t += v[k];
  }
  int total;
  int run = block_prefix(t, sh, total);
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) rank[base + k] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// output value of each segment: the id of its final segment (compact = 0),
// or the rank of that segment among the image's final segments in id order
// (compact = 1; rank = final segments before it in the batch minus those before
// the image's first segment); the segments and merged segments per image
__global__ __launch_bounds__(kT) void k_seg_out(const ImgDesc* img, int n_img, const int* n_seg_dev,
                                                const int* seg_img, const int* segid,
                                                const int* mpar, const int* seg_root,
                                                const int* rank, const int* boff, int compact,
                                                int* val, int* counts) {
  const int n_seg = *n_seg_dev;
  int begin, end;
  block_chunk<kT>(n_seg, begin, end);
  ImageCount ic;
  for (int s0 = begin; s0 < end; s0 += kT) {
    const int s = s0 + threadIdx.x;
    const bool in = s < end;
    int b = 0;
    bool merged = false;
    if (in) {
      b = seg_img[s];
      int t = s;  // (the owners are final: plain loads)
      for (int u = mpar[t]; u != t; u = mpar[t]) t = u;
      merged = t != s;
      const int64_t off = img[b].pix_off;
      if (compact) {
        const int f = segid[off];
        val[s] = rank[t] + boff[t / kScanBlock] - (rank[f] + boff[f / kScanBlock]);
      } else {
        val[s] = (int)(seg_root[t] - off);
      }
    }
    ic.add(counts, 2, b, in, merged);
  }
  ic.finish(counts, 2);
  if (blockIdx.x == 0) {
    for (int b = threadIdx.x; b < n_img; b += kT)
      counts[4 * b] = (b + 1 < n_img ? segid[img[b + 1].pix_off] : n_seg) - segid[img[b].pix_off];
  }
}

// the output, four consecutive pixels of the batch per thread (VEC: out is
// 16-byte aligned)
template <bool VEC>
__global__ __launch_bounds__(kT) void k_final(int n_pix, const int* segid, const int* val,
                                              int32_t* out) {
  const int64_t i0 = 4 * ((int64_t)blockIdx.x * kT + threadIdx.x);
  if (i0 >= n_pix) return;
  if (VEC && i0 + 4 <= n_pix) {
    const int4 w = *reinterpret_cast<const int4*>(segid + i0);
    const int a = val[w.x];
    const int b = w.y == w.x ? a : val[w.y];
    const int c = w.z == w.y ? b : val[w.z];
    const int d = w.w == w.z ? c : val[w.w];
    *reinterpret_cast<int4*>(out + i0) = make_int4(a, b, c, d);
  } else {
    for (int64_t i = i0; i < i0 + 4 && i < n_pix; ++i) out[i] = val[segid[i]];
  }
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

}  // namespace

size_t conn_scan_blocks(int64_t n) { return (size_t)((n + kScanBlock - 1) / kScanBlock); }

size_t conn_tiles(int W, int H) {
  return (size_t)((W + kTW - 1) / kTW) * (size_t)((H + kTH - 1) / kTH);
}

size_t conn_side_ints(int n_img, int max_tiles) { return (size_t)n_img * max_tiles * kSide; }

hipError_t conn_launch(const ConnPtrs& C, const ImgDesc* img, int n_img, int max_tiles,
                       const float* lab, const int32_t* labels, int compact,
                       int32_t* out, hipStream_t s) {
  const int n = (int)C.n_pix;
  const dim3 gt(max_tiles, n_img);
  const bool few = (int64_t)max_tiles * n_img <= kSmallTiles;
  if (few)
    hipLaunchKernelGGL(k_cc_tile<16>, gt, dim3(1024), 0, s, img, labels, C.par, C.side, max_tiles);
  else
    hipLaunchKernelGGL(k_cc_tile<4>, gt, dim3(256), 0, s, img, labels, C.par, C.side, max_tiles);
  hipLaunchKernelGGL(k_cc_border, dim3(max_tiles, n_img), dim3(128), 0, s, img, labels, C.par,
                     C.side, max_tiles);
  // roots in raster order: ranks within blocks, then the scan of the block counts
  const int nb = (n + kScanBlock - 1) / kScanBlock;
  hipLaunchKernelGGL(k_root_rank, dim3(nb), dim3(kT), 0, s, C.par, n, C.scan, C.bsum);
  hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(kT), 0, s, C.bsum, n, (const int*)nullptr, C.total);
  // Kernels over segments: at most one segment per pixel, strided beyond 4096
  // blocks.  (The tile borders are joined: the side buffer now holds the
  // counters and, behind them, the list of the largest clusters.  A cluster in
  // it has more than 256 pixels, or more than 128 members and neighbours, of
  // which p pixels have at most 5 p: 26 pixels or more.  The buffer has kSide
  // entries per tile of 4096 pixels.)
  static_assert(kSide >= N_COUNTERS + kTW * kTH / 26 + 1, "the largest clusters' list");
  int* const cnt = C.side;
  int* const rest = C.side + N_COUNTERS;
  const dim3 gs(std::min(blocks(n), 4096u));
  // where a block ends in atomics on shared counters, fewer and longer ones
  const dim3 ga(std::min(blocks(n), 1024u));
  const double* mean = reinterpret_cast<const double*>(C.colsum);
  // (tail: list cursors of the clusters until the block merges)
  hipLaunchKernelGGL(k_seg_zero, gs, dim3(kT), 0, s, C.total, n_img, C.size0, C.colsum, C.ccnt,
                     C.cursor, C.tail, cnt, C.counts);
  // (bsum still holds the block offsets of the root ranks here)
  if (few)
    hipLaunchKernelGGL(k_seg_assign<16>, gt, dim3(1024), 0, s, img, lab, C.par, C.scan, C.bsum,
                       C.segid, C.seg_root, C.seg_img, C.size0, C.colsum);
  else
    hipLaunchKernelGGL(k_seg_assign<4>, gt, dim3(256), 0, s, img, lab, C.par, C.scan, C.bsum,
                       C.segid, C.seg_root, C.seg_img, C.size0, C.colsum);
  hipLaunchKernelGGL(k_seg_prep, ga, dim3(kT), 0, s, img, C.total, C.seg_img, C.size0, C.colsum,
                     C.mpar, C.cpar, C.poff, cnt, C.counts);
  // the pixel union-find array is free now: it holds the sources' pixel lists
  const dim3 g4(blocks((C.n_pix + 3) / 4));
  hipLaunchKernelGGL(k_px_fill, g4, dim3(kT), 0, s, n, C.segid, C.poff, C.cursor, C.par);
  // (next: the clustered sources, until the block merges' links)
  hipLaunchKernelGGL(k_merge_single, gs, dim3(kT), 0, s, img, C.total, C.seg_img, C.seg_root, C.size0,
                     C.poff, C.par, C.segid, mean, C.cpar, C.mpar, C.next, cnt);
  hipLaunchKernelGGL(k_cl_count, gs, dim3(kT), 0, s, C.next, cnt, C.cpar, C.ccnt);
  // The root-rank array is free until the final ranks: clusters for 8 and 16 lanes
  // in its first half, for a wave in its second.  Each has two sources or more, so
  // half the segments bound either, also when all of the first move on.
  const int half = n / 2;
  int* const team = C.scan;
  int* const wave = C.scan + half;
  hipLaunchKernelGGL(k_cl_alloc, ga, dim3(kT), 0, s, C.next, C.cpar, C.ccnt, C.coff, cnt, team, half,
                     wave);
  // (beside the list: sizes in the working sizes, pixels in the pixel cursors)
  hipLaunchKernelGGL(k_cl_fill, gs, dim3(kT), 0, s, C.next, cnt, C.cpar, C.coff, C.size0, C.poff,
                     C.seg_root, C.tail, C.list, C.size, C.cursor);
  const MergePtrs M{img, C.seg_img, C.list, C.size, C.cursor, C.par, C.segid, mean,
                    C.ccnt, C.coff, C.mpar, C.size0, C.poff, C.seg_root, C.cpar, C.next, C.tail,
                    C.scan, C.cursor};
  hipLaunchKernelGGL(k_merge_team, dim3(std::min(2 * blocks(n), 8192u)), dim3(64), 0, s, M, cnt, team,
                     half, wave);
  hipLaunchKernelGGL(k_merge_wave, dim3(std::min(blocks(n), 3584u)), dim3(64), 0, s, M, cnt, wave, rest);
  // (next and tail are free now, and so is the root-rank array)
  hipLaunchKernelGGL(k_merge_block, dim3(std::min(blocks(n), 256u)), dim3(kHugeT), 0, s, M, cnt, rest);
  // final segments ranked in id order; each segment's output value (into the
  // working sizes, no longer needed); the output
  if (compact) {
    hipLaunchKernelGGL(k_final_rank, dim3(nb), dim3(kT), 0, s, C.total, C.mpar, C.scan, C.bsum);
    hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(kT), 0, s, C.bsum, 0, C.total, (int*)nullptr);
  }
  hipLaunchKernelGGL(k_seg_out, ga, dim3(kT), 0, s, img, n_img, C.total, C.seg_img, C.segid, C.mpar,
                     C.seg_root, C.scan, C.bsum, compact, C.size, C.counts);
  if (((uintptr_t)out & 15) == 0)
    hipLaunchKernelGGL(k_final<true>, g4, dim3(kT), 0, s, n, C.segid, C.size, out);
  else
    hipLaunchKernelGGL(k_final<false>, g4, dim3(kT), 0, s, n, C.segid, C.size, out);
  return hipGetLastError();
}

}  // namespace gmmsp
