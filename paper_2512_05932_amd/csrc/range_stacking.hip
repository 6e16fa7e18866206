// Range stacking (section II-C, Alg. 2) with a separable kernel
// kappa*eta = H * V: the rendered intensities are split into depth slices
// (time bins); every slice is correlated with the kernel, separably (a pass
// along the rows with H, then along the columns with V); each pixel keeps
// the nearest slice whose correlation reaches rho_min and that value.
//
// A depth slice holds few of the image's pixels, so the correlations are
// evaluated over the pixels that a slice has and not over the image:
//   1. k_rs_rows: the pixel records row by row, and the largest shade of every
//      slice.  A slice whose largest shade times sum H times sum V stays below
//      rho_min reaches it nowhere and is skipped (slice skipping).
//   2. k_rs_present: for every image row and block of kCols output columns, a
//      bitmap of the slices that the row's window (the block and the kernel's
//      half extent on both sides) holds.
//   3. k_range_stacking: a workgroup per tile of kCols x kRows output pixels,
//      every wave with its share of the slices, see there.
// The sums run over the same terms in the same order as a correlation of the
// whole slice (ascending columns, then ascending rows; the terms left out are
// zero).
#include <algorithm>

#include "engine.h"

namespace lidar {

namespace {

constexpr int kCols = 64, kRows = kRangeStackRows;  // output tile: columns (lanes) x rows
constexpr int kThreads = 256;
constexpr int kTileWaves = 8, kTileThreads = 64 * kTileWaves;
constexpr int kDense = 8;                     // window columns correlated together
constexpr int kMaxHalf = kRsMaxHalf;          // M, N <= 127
// 64-row groups of a tile's window rows, 64-column groups of its window columns
constexpr int kRowGroups = (kRows + 2 * kMaxHalf + 63) / 64;
constexpr int kMaxColGroups = (kCols + 2 * kMaxHalf + 63) / 64;
constexpr int kMapRows = 16;                  // image rows of a workgroup of k_rs_present

// Bitwise OR over the 64 lanes (all active), as a uniform value.
template <int CTRL, int ROW_MASK>
__device__ inline unsigned dpp_or(unsigned v)
{
    return v | (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}

__device__ inline unsigned wave_or(unsigned x)
{
    x = dpp_or<0xb1, 0xf>(x);
    x = dpp_or<0x4e, 0xf>(x);
    x = dpp_or<0x141, 0xf>(x);
    x = dpp_or<0x140, 0xf>(x);
    x = dpp_or<0x142, 0xa>(x);
    x = dpp_or<0x143, 0xc>(x);
    return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}

// Row-major copy of the pixel records and the largest shade of every slice
// (time bin) over the image (FP32 bits of non-negative values compare as
// integers).
// The pre-pass's 4-column blocks put a row's records 32 H bytes apart, often a
// power of two; row by row, a wave reads a window row's records in whole lines
// at one scalar base and constant lane offsets.
// Neighbouring pixels share few slices, so global atomics would serialise on
// their addresses (3.1 ms for 4096 x 512 pixels): a workgroup keeps the maxima
// of its share of the tiles in LDS, where a plain read decides whether the
// atomic is needed at all, and adds the slices it saw to the global maxima at
// the end. 12 us in all for that image.
constexpr int kMaxGroups = 512;                // two workgroups per CU
constexpr int kCopyRows = 16;                  // copy tile: kCols columns x kCopyRows rows

__global__ __launch_bounds__(kThreads)
void k_rs_rows(RangeStackArgs a, int* smax)
{
    extern __shared__ int lmax[];               // [R]
    __shared__ int2 t[kCopyRows][kCols + 1];
    const int tid = threadIdx.x;
    for (int i = tid; i < a.R; i += kThreads) lmax[i] = 0;
    const long tr = (a.H + kCopyRows - 1) / kCopyRows, tiles = tr * ((a.W4 + kCols - 1) / kCols);
    for (long tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const long u0 = tile / tr * kCols;
        const int v0 = (int)(tile % tr) * kCopyRows;
        __syncthreads();                         // the maxima are cleared, the last tile is written
#pragma unroll
        for (int p = 0; p < kCols * kCopyRows / kThreads; ++p) {
            const int e = p * kThreads + tid, j = e % 4, r = e / 4 % kCopyRows, b = e / (4 * kCopyRows);
            if (v0 + r >= a.H || u0 + 4 * b >= a.W4) continue;
            const int2 rec = a.pix[(((u0 >> 2) + b) * a.H + v0 + r) * 4 + j];
            t[r][4 * b + j] = rec;
            if (rec.x >= 0 && rec.x < a.R && rec.y > lmax[rec.x]) atomicMax(lmax + rec.x, rec.y);
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < kCols * kCopyRows / kThreads; ++p) {
            const int e = p * kThreads + tid, c = e % kCols, r = e / kCols;
            if (v0 + r < a.H && u0 + c < a.W4) a.rows[(long)(v0 + r) * a.W4 + u0 + c] = t[r][c];
        }
    }
    __syncthreads();
    for (int i = tid; i < a.R; i += kThreads)
        if (lmax[i] > 0) atomicMax(smax + i, lmax[i]);
}

__global__ void k_rs_clear(int* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Slices of the windows of image rows lr0 .. lr1 - 1, one bitmap per row and
// column block: word w of row v at ((block) words + w) (lr1 - lr0) + v - lr0.
// A row holds a slice through a pixel of positive shade; slices that cannot
// reach rho_min are left out.  A workgroup takes kMapRows rows of a block
// through an LDS bitmap.  Bound by the
// reads (every record is read 1 + 2 M / kCols times, from L2): 18 us for 4096 x
// 512 pixels and a kernel 69 columns wide.
__global__ __launch_bounds__(kThreads)
void k_rs_present(RangeStackArgs a, int lr0, int lr1)
{
    extern __shared__ unsigned map[];                  // [words][kMapRows]
    const int rows = lr1 - lr0, words = (a.R + 31) / 32, tid = threadIdx.x;
    const int row_groups = (rows + kMapRows - 1) / kMapRows;
    const int blk = blockIdx.x / row_groups;
    const int r0 = (blockIdx.x - blk * row_groups) * kMapRows;
    for (int i = tid; i < words * kMapRows; i += kThreads) map[i] = 0u;
    __syncthreads();
    const long c0 = std::max<long>((long)blk * kCols - a.M, 0);
    const int cols = (int)(std::min<long>((long)blk * kCols + kCols + a.M, a.W) - c0);
    for (int i = tid; i < cols * kMapRows; i += kThreads) {
        const int r = i / cols, c = i - r * cols;
        if (r0 + r >= rows) break;
        const int2 rec = a.rows[(long)(lr0 + r0 + r) * a.W4 + c0 + c];
        if (rec.x >= 0 && rec.x < a.R && rec.y > 0 && __int_as_float(a.smax[rec.x]) * a.bound >= a.rho_min)
            atomicOr(&map[(rec.x >> 5) * kMapRows + r], 1u << (rec.x & 31));
    }
    __syncthreads();
    unsigned* out = a.present + (long)blk * words * rows;
    for (int i = tid; i < words * kMapRows; i += kThreads) {
        const int w = i / kMapRows, r = i % kMapRows;
        if (r0 + r < rows) out[(long)w * rows + r0 + r] = map[i];
    }
}

// Output rows o0 .. o1 - 1 from the bitmaps of rows lr0 .. lr1 - 1 (the rows and
// their halo of N inside the image).  Every wave walks the slices of the
// tile's window from the nearest on, 32 at a time: lane l holds the words of
// window rows l, l + 64, ..., their union gives the slices and a ballot per
// slice its rows.  Wave w evaluates the slices w, w + kTileWaves, ...: each
// row of the slice is correlated with H (every pixel of the slice is one
// multiply-add over the lanes, H read from LDS shifted by the lane), and the
// row's sums enter the tile's kRows correlations with one scalar of V each.
// A pixel keeps the smallest slice that reaches rho_min (the largest key's
// complement: one 64-bit LDS minimum of slice and value); the workgroup is
// done when every pixel has a slice nearer than those left.
// The work is a multiply-add per (pixel of the window, tile) and kRows per
// (row, slice), with no barrier between slices and no step for an absent
// one.  The slices go round the waves because tiles differ widely (165 to 348
// (row, slice) pairs on average, 6632 at most, where box sides are seen at a
// grazing angle).  A workgroup per 32 x 16 tile that staged each slice's
// rows in LDS took 4209 us for 4096 x 512 pixels (1200 bins, 69 x 83 kernel),
// bound by its barriers; a wave per tile of 8 rows 3452 us, bound by the
// largest tile; this kernel 540 to 750 us over scenes.  It is bound by the
// instructions of the largest tiles: about 160 vector instructions per (row,
// slice), and the CU that has such a tile works on after the others (all
// tiles have begun after 200 us).
template <int CG, int RG>                              // 64-column and 64-row groups of the window
__global__ __launch_bounds__(kTileThreads)
void k_range_stacking(RangeStackArgs a, int o0, int o1, int lr0, int lr1)
{
    // H at window column minus lane, zero outside the kernel
    constexpr int kShift = kCols - 1;
    __shared__ float hs[64 * CG + kShift];
    __shared__ unsigned long long found[kRows][kCols]; // slice, value of the nearest so far
    const int M2 = 2 * a.M, N2 = 2 * a.N, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // tiles column block by column block: neighbours, which cost alike, go to
    // different XCDs
    const int per_block = (o1 - o0 + kRows - 1) / kRows;
    const int tile = blockIdx.x, blk = tile / per_block;
    const int v0 = o0 + (tile - blk * per_block) * kRows;
    const int u0 = blk * kCols;
    for (int i = tid; i < 64 * CG + kShift; i += kTileThreads)
        hs[i] = i >= kShift && i - kShift <= M2 ? a.hk[i - kShift] : 0.0f;
    for (int i = tid; i < kRows * kCols; i += kTileThreads)
        found[i / kCols][i % kCols] =
            u0 + i % kCols < a.W && v0 + i / kCols < o1 ? (unsigned long long)a.R << 32 : 0ull;
    __syncthreads();
    // this lane's window columns 64 k + lane: byte offsets from the window's
    // first one inside the image, and which lanes have one
    const int first = max(u0 - a.M, 0);
    unsigned off[CG];
    bool inside[CG];
#pragma unroll
    for (int k = 0; k < CG; ++k) {
        const long c = (long)u0 - a.M + 64 * k + lane;
        inside[k] = c >= 0 && c < a.W;
        off[k] = (unsigned)((inside[k] ? c : first) - first) * 8u;
    }
    const int words = (a.R + 31) / 32, rows = lr1 - lr0;
    const unsigned* map = a.present + (long)blk * words * rows;
    bool have[RG];
    int rel[RG];
#pragma unroll
    for (int k = 0; k < RG; ++k) {
        const int wr = 64 * k + lane, v = v0 - a.N + wr;
        have[k] = wr < kRows + N2 && v >= lr0 && v < lr1;
        rel[k] = have[k] ? v - lr0 : 0;
    }
    auto load_words = [&](int w, unsigned (&x)[RG]) {
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            x[k] = 0u;
            if (have[k]) x[k] = *gptr(map + (long)w * rows + rel[k]);
        }
    };
    auto fetch = [&](int wr, int2 (&rec)[CG]) {
        const char* base = (const char*)(a.rows + (long)(v0 - a.N + wr) * a.W4 + first);
#pragma unroll
        for (int k = 0; k < CG; ++k) {
            const gint2 t = *gptr((const gint2*)(base + off[k]));
            rec[k] = make_int2(t.x, t.y);
        }
    };
    unsigned bits[RG], bits_next[RG];
    load_words(0, bits_next);
    for (int w = 0; w < words; ++w) {
        unsigned any = 0u;
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            bits[k] = bits_next[k];
            any |= bits[k];
        }
        if (w + 1 < words) load_words(w + 1, bits_next);
        // this wave's slices of the word
        unsigned slices = wave_or(any) & (0x01010101u << wave);
        static_assert(kTileWaves == 8, "every eighth slice of a word");
        if (!slices) continue;
        // done when every pixel has a slice nearer than this word's
        bool open = false;
#pragma unroll
        for (int t = 0; t < kRows; ++t) open |= (int)(found[t][lane] >> 32) >= 32 * w;
        if (__ballot(open) == 0ull) break;
        for (; slices; slices &= slices - 1u) {
            const int bit = __builtin_ctz(slices), s = 32 * w + bit;
            float acc[kRows];
#pragma unroll
            for (int t = 0; t < kRows; ++t) acc[t] = 0.0f;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                // the window rows 64 g .. that hold s
                unsigned long long held = __ballot((bits[g] >> bit) & 1u);
                if (!held) continue;
                int wr = 64 * g + __builtin_ctzll(held);
                int2 cur[CG], ahead[CG];
                fetch(wr, cur);
                for (;;) {
                    held &= held - 1ull;
                    const int nwr = held ? 64 * g + __builtin_ctzll(held) : wr;
                    fetch(nwr, ahead);                 // the next row's records, over this row's work
                    // output row t takes V at the window row minus t (vk is zero
                    // on kRows - 1 entries on both sides)
                    struct Taps { float w[kRows]; };
                    const Taps v = load_uniform((const Taps*)(a.vk + (wr - (kRows - 1))));
                    // the row's correlation with H: its pixels of s in ascending
                    // columns, one multiply-add each over the lanes, in blocks of
                    // kDense columns that hold one; the other slices' pixels are
                    // zeros there (they leave the sum as it is)
                    float row = 0.0f;
                    unsigned long long px[CG];
#pragma unroll
                    for (int k = 0; k < CG; ++k) {
                        const bool mine = inside[k] && cur[k].x == s;
                        px[k] = __ballot(mine);
                        if (!px[k]) continue;
                        const int x = mine ? cur[k].y : 0;
                        const float* h = hs + (64 * k + kShift - lane);
                        const unsigned half[2] = {(unsigned)px[k], (unsigned)(px[k] >> 32)};
#pragma unroll
                        for (int b = 0; b < 64; b += kDense) {
                            if (!(half[b / 32] & (((1u << kDense) - 1u) << (b % 32)))) continue;
                            float hv[kDense];
#pragma unroll
                            for (int j = 0; j < kDense; ++j) hv[j] = h[b + j];
#pragma unroll
                            for (int j = 0; j < kDense; ++j)
                                row = fmaf(hv[j], __int_as_float(__builtin_amdgcn_readlane(x, b + j)), row);
                        }
                    }
                    if (__ballot(!isfinite(row)) == 0ull) {
#pragma unroll
                        for (int t = 0; t < kRows; ++t) acc[t] = fmaf(v.w[kRows - 1 - t], row, acc[t]);
                    } else {
                        // an infinity or NaN: exactly the terms inside the kernel
                        row = 0.0f;
#pragma unroll
                        for (int k = 0; k < CG; ++k)
                            for (; px[k]; px[k] &= px[k] - 1ull) {
                                const int i = __builtin_ctzll(px[k]), m = 64 * k + i - lane;
                                const float x = __int_as_float(__builtin_amdgcn_readlane(cur[k].y, i));
                                if (m >= 0 && m <= M2) row = fmaf(hs[m + kShift], x, row);
                            }
#pragma unroll
                        for (int t = 0; t < kRows; ++t)
                            if (wr - t >= 0 && wr - t <= N2) acc[t] = fmaf(a.vk[wr - t], row, acc[t]);
                    }
                    if (!held) break;
                    wr = nwr;
#pragma unroll
                    for (int k = 0; k < CG; ++k) cur[k] = ahead[k];
                }
            }
#pragma unroll
            for (int t = 0; t < kRows; ++t)
                if (acc[t] >= a.rho_min)
                    atomicMin(&found[t][lane], (unsigned long long)s << 32 | __float_as_uint(acc[t]));
        }
    }
    __syncthreads();
    for (int i = tid; i < kRows * kCols; i += kTileThreads) {
        const int u = u0 + i % kCols, v = v0 + i / kCols;
        if (u >= a.W || v >= o1) continue;
        const unsigned long long f = found[i / kCols][i % kCols];
        a.s_nearest[(long)v * a.W + u] = (int32_t)(f >> 32);
        a.xi_nearest[(long)v * a.W + u] = __uint_as_float((unsigned)f);
    }
}

template <int CG>
static void launch_tiles(hipStream_t s, long tiles, int row_groups, const RangeStackArgs& a, int o0, int o1, int lr0,
                         int lr1)
{
    const dim3 grid((unsigned)tiles), block(kTileThreads);
    switch (row_groups) {
    case 1: hipLaunchKernelGGL((k_range_stacking<CG, 1>), grid, block, 0, s, a, o0, o1, lr0, lr1); break;
    case 2: hipLaunchKernelGGL((k_range_stacking<CG, 2>), grid, block, 0, s, a, o0, o1, lr0, lr1); break;
    default: hipLaunchKernelGGL((k_range_stacking<CG, kRowGroups>), grid, block, 0, s, a, o0, o1, lr0, lr1);
    }
}

}  // namespace

// The bitmaps of as many rows as the workspace holds are built at a time (all
// rows of the usual images; a halo of 2 N rows is built again for every band).
size_t range_stacking_map_words(int W, int H, int N, int R)
{
    constexpr size_t kMost = 16u << 20;                // 64 MB
    const size_t per_row = (size_t)((W + kCols - 1) / kCols) * ((R + 31) / 32);
    const size_t least = per_row * std::min<size_t>(H, 2 * (size_t)N + kRows);
    return std::max(least, std::min(per_row * H, kMost));
}

hipError_t launch_range_stacking(hipStream_t s, const RangeStackArgs& a, int* smax_scratch, unsigned* map,
                                 size_t map_words)
{
    if (a.M > kMaxHalf || a.N > kMaxHalf || a.R > kMaxBins) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rs_clear, dim3((a.R + 255) / 256), dim3(256), 0, s, smax_scratch, a.R);
    const long tiles = (long)((a.W4 + kCols - 1) / kCols) * ((a.H + kCopyRows - 1) / kCopyRows);
    RangeStackArgs b = a;
    b.smax = smax_scratch;
    b.present = map;
    hipLaunchKernelGGL(k_rs_rows, dim3((unsigned)std::min<long>(tiles, kMaxGroups)), dim3(kThreads),
                       sizeof(int) * (size_t)a.R, s, b, smax_scratch);
    const long nblk = (a.W + kCols - 1) / kCols, words = (a.R + 31) / 32;
    const long held = (long)(map_words / (size_t)(nblk * words));
    const long band = held >= a.H ? a.H : (held - 2L * a.N) / kRows * kRows;
    if (band <= 0) return hipErrorInvalidValue;
    for (long o0 = 0; o0 < a.H; o0 += band) {
        const int o1 = (int)std::min<long>(o0 + band, a.H);
        const int lr0 = (int)std::max<long>(o0 - a.N, 0), lr1 = (int)std::min<long>((long)o1 + a.N, a.H);
        const long mg = nblk * ((lr1 - lr0 + kMapRows - 1) / kMapRows);
        hipLaunchKernelGGL(k_rs_present, dim3((unsigned)mg), dim3(kThreads), sizeof(unsigned) * words * kMapRows, s,
                           b, lr0, lr1);
        const long tg = nblk * ((o1 - o0 + kRows - 1) / kRows);
        const int rg = (kRows + 2 * a.N + 63) / 64;
        switch ((kCols + 2 * a.M + 63) / 64) {
        case 1:
        case 2: launch_tiles<2>(s, tg, rg, b, (int)o0, o1, lr0, lr1); break;
        case 3: launch_tiles<3>(s, tg, rg, b, (int)o0, o1, lr0, lr1); break;
        default: launch_tiles<kMaxColGroups>(s, tg, rg, b, (int)o0, o1, lr0, lr1);
        }
    }
    return hipGetLastError();
}

}  // namespace lidar
