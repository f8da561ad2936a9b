// Separable filter for gfx950: two 1-D ranged inner products in a row (dot product, Section
// III-B Eq. 3), the window centred as in the bilateral-filter call of Section VI-A (offset -k/2):
//     t[n,p1,p2] = sum_{a2<k} kx[a2] * x[n, p1, p2 + a2 - k/2]
//     y[n,p1,p2] = sum_{a1<k} ky[a1] * t[n, p1 + a1 - k/2, p2]
// with coordinates clamped to the image.  Both passes run in one launch and the intermediate
// t never leaves LDS (it overwrites the staged input there): 8 algorithmic bytes per pixel (one fp32 read, one fp32 written).
//
// A workgroup owns TH x 64 output pixels of one image.  The covering sub-tensor (Section IV-A,
// Eq. 9: (TH + k - 1) x (64 + k - 1)) is staged in LDS with the clamping resolved there.  A
// row-pass unit keeps RC adjacent outputs of one staged row in registers and reads the
// RC + k - 1 inputs they need as 16-byte runs; a column-pass unit keeps a PR x PC patch and
// reads k + PR - 1 runs of PC columns.  In the row pass neighbouring lanes take neighbouring
// rows; the row pitches are 4 mod 8 floats, which spreads the 16-byte accesses of 16 lanes over
// all banks (the padding layout of Section IV-B).
//
// Three forms (SepForm, merit_internal.h), chosen by the plan from the window and the number of tiles.  What bounds
// them: on large frames the multiply-adds (9.9 us of 24 at k = 30 on 4x1080x1920, at the probe's rate), the LDS reads
// and the memory of a tile one after the other, so they want many workgroups in different phases; on small ones the
// chain of one tile, so they want it cut into many threads.  us a launch (18 in a graph, over three sets of buffers), one
// persistent form of 256 threads that requested its next tile -> these:
//   TILES       one tile a workgroup, no request ahead: six or seven workgroups a compute unit instead of three
//               (4x1080x1920: k = 3 12.7 -> 12.3, 8 14.9 -> 13.7, 12 17.0 -> 15.1, 16 19.4 -> 16.8, 20 21.7 -> 19.2, 24
//               23.7 -> 21.6, 28 25.5 -> 25.3)
//   PERSISTENT  k > 28, where 64 staged rows would be half halo: 96 rows, four workgroups a compute unit that walk the
//               tiles (k = 30 23.7 -> 23.4, 32 24.5 -> 24.3; 64 rows 10 % more); and any window on more tiles than
//               a launch has workgroups, or on request of more than 64 staged rows
//   FEW         up to three tiles a compute unit: 512 threads, 2 x 2 patches (2x600x1280: k = 30 8.6 -> 7.9, 20 8.1 ->
//               7.2; 380x936: 30 6.8 -> 4.4, 8 4.3 -> 3.6), and where the tiles do not fill the chip shorter ones
//               (624x172: k = 20 6.6 -> 3.8, 0.5 more on 44-row tiles)
//
// The staged columns start at x0 - c4, c4 = k/2 rounded up to 4, so that (for W % 4 == 0) every
// group of four staged columns is one aligned 16-byte run of the image, entirely inside it or
// entirely outside (then it is four copies of the edge pixel): the staging is 16-byte loads
// without a branch, and the row pass reads its window c4 - k/2 columns further right.  Any other
// W >= 4 the same: fp32 rows start on 4-byte boundaries, which is all a 16-byte load or store
// needs, and the group that the row's end cuts is loaded so that it ends with the row, its pixels
// picked out of the four.  (Such widths were staged element by element: k = 13 on 2x678x1861
// 23.0 us -> 9.3, k = 6 on 2x806x869 12.0 -> 6.6, k = 17 on 1080x1919 20.3 -> 10.5.)
#include "merit_internal.h"

namespace merit {

typedef float float4v __attribute__((ext_vector_type(4)));

// K = window length (compile time: every tap index is an immediate, the sliding windows live
// in renamed registers and no zero tap is multiplied).  RAGGED = W % 4 != 0 (an instance of its
// own: as a run-time condition it cost the aligned rows 1.5 %)
template <int K, bool RAGGED, int FORM>
__global__ __launch_bounds__((FORM == SEP_FEW ? 512 : 256), 4) void merit_sepfilter_tile(SepParams p, const float *__restrict__ x,
                                                           const float *__restrict__ kx,
                                                           const float *__restrict__ ky, float *__restrict__ y)
{
    constexpr int NT = FORM == SEP_FEW ? 512 : 256, ROWS = sep_rows(FORM), RC = sep_rc(FORM);
    constexpr int PR = FORM == SEP_FEW ? 2 : 4, PC = FORM == SEP_FEW ? 2 : 4;     // rows and columns of a column-pass patch
    constexpr bool LONG = K > 8;                                  // one window, or a few rows of a patch, in registers at a time
    typedef float run __attribute__((ext_vector_type(PC)));
    constexpr int TW = 64;
    constexpr int C = K / 2, C4 = (C + 3) / 4 * 4, D = C4 - C;    // staged column 0 = image column x0 - C4
    constexpr int NWR = (D + RC + K - 1 + 3) / 4;                 // 16-byte groups a row-pass unit reads
    constexpr int K4 = (K + 3) / 4;
    extern __shared__ __align__(16) float smem[];
    const int RH = p.TH + K - 1;                          // staged rows
    float *in = smem;                                     // [RH][PI]; later the row-pass result
    float *wxl = in + RH * p.PI;                          // [4*K4]
    float *wyl = wxl + 4 * K4;                            // [4*K4]

    const int tid = threadIdx.x;
    const int ntiles = p.N * p.tiles_y * p.tiles_x;
    struct Tile {
        int n, x0, y0;
    };
    auto tile_at = [&](int t) {
        const uint32_t q0 = fdiv((uint32_t)t, p.div_tiles_x);
        Tile T;
        T.n = (int)fdiv(q0, p.div_tiles_y);
        T.x0 = (t - (int)q0 * p.tiles_x) * TW;
        T.y0 = ((int)q0 - T.n * p.tiles_y) * p.TH;
        return T;
    };

    // The taps live in LDS and are read into vector registers at the start of each pass:
    // measured on gfx950, a multiply-add stream whose tap sits in a scalar register issues
    // one wavefront instruction per 4.2-4.6 clocks, with all operands in vector registers
    // one per 2.4-3.0 clocks (two or more wavefronts per SIMD).
    if (tid < 4 * K4) {
        wxl[tid] = tid < K ? kx[min(tid, K - 1)] : 0.0f;
        wyl[tid] = tid < K ? ky[min(tid, K - 1)] : 0.0f;
    }
    // Staging: every element is a real (clamped) pixel.  A thread owns one 4-column group of
    // the staged rows r = tid / 32 + (NT / 32) j; every load of a tile is issued before its first
    // LDS write (one memory round trip a tile).
    constexpr int SB = ROWS / (NT / 32);
    const int P4 = p.PI >> 2, W4 = p.W >> 2;              // P4 <= 32 for every K <= 32
    const bool vec = !RAGGED || p.W >= 4;
    constexpr int lg = 5;                                 // lanes per staged row
    const int cg = tid & ((1 << lg) - 1);
    const bool live = cg < P4;
    constexpr int rstep = NT >> lg;
    float4v pre[SB];
    auto issue = [&](const Tile &T, int r0) {
        const int g4 = ((T.x0 - C4) >> 2) + cg;           // image 4-column group (may be outside)
        // uniform image base + 32-bit element offsets (the plan keeps H*W below 2^31)
        const float *img = x + (size_t)T.n * p.H * p.W;
        const uint32_t col = RAGGED ? (uint32_t)min(max(4 * g4, 0), p.W - 4) : 4u * (uint32_t)min(max(g4, 0), W4 - 1);
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int gy = min(max(T.y0 - C + r0 + rstep * b, 0), p.H - 1);
            const float *src = img + (col + (uint32_t)gy * (uint32_t)p.W);
            if (RAGGED) __builtin_memcpy(&pre[b], src, 16);
            else pre[b] = *reinterpret_cast<const float4v *>(src);
        }
    };
    auto commit = [&](const Tile &T, int r0) {
        const int g4 = ((T.x0 - C4) >> 2) + cg;
        const bool inside = g4 >= 0 && g4 < W4;           // else: four copies of the edge pixel
        const bool left = g4 < 0;
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int r = r0 + rstep * b;
            const float edge = left ? pre[b].x : pre[b].w;
            float4v o;
            o.x = inside ? pre[b].x : edge; o.y = inside ? pre[b].y : edge;
            o.z = inside ? pre[b].z : edge; o.w = inside ? pre[b].w : edge;
            if (live && r < RH) reinterpret_cast<float4v *>(in)[r * P4 + cg] = o;
        }
        // the group that the row's end cuts: its first pixels lie behind those it shares with its neighbour (written once
        // more, so that the common form above stays as short as it is)
        if (RAGGED && g4 == W4) {
            const int cut = p.W & 3;                      // pixels of the group that exist
#pragma unroll
            for (int b = 0; b < SB; ++b) {
                const int r = r0 + rstep * b;
                float4v o = pre[b];
                o.x = cut == 1 ? pre[b].w : (cut == 2 ? pre[b].z : pre[b].y);
                o.y = cut == 3 ? pre[b].z : pre[b].w;
                o.z = pre[b].w;
                if (live && r < RH) reinterpret_cast<float4v *>(in)[r * P4 + cg] = o;
            }
        }
    };

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Every XCD sweeps its
    // own contiguous eighth of the raster-ordered tile list (a band of tile rows), its workgroups
    // side by side: horizontally adjacent tiles, which share the cache lines of their halo columns,
    // and vertically adjacent ones, which share k - 1 halo rows, meet in one L2 at about the same
    // time.  (With runs of four tiles per XCD in raster order over the whole chip the vertical
    // neighbours sat on other XCDs: 1.72 times the image was fetched at k = 30.)
    const int nwg = (int)gridDim.x;
    int t = (int)blockIdx.x, tstep = nwg, tend = ntiles;
    if (FORM != SEP_PERSISTENT) {
        t = (int)xcd_band_item(blockIdx.x, nwg >> 3, nwg & 7);
    } else if (nwg % 8 == 0) {
        const int xcd = t & 7, slot = t >> 3;
        t = (int)(((long long)xcd * ntiles) >> 3) + slot;         // slot < nwg / 8 <= the band's length
        tend = (int)(((long long)(xcd + 1) * ntiles) >> 3);
        tstep = nwg >> 3;
    }
    for (; t < tend; t += tstep) {                        // t < tend at first: the grid never exceeds the tile list
        const Tile T = tile_at(t);
        const int x0 = T.x0, y0 = T.y0;
        if (vec) {
            issue(T, tid >> lg);
            commit(T, tid >> lg);
        } else {
            const float *img = x + (size_t)T.n * p.H * p.W;
            const int total = RH * p.PI;
            for (int e = tid; e < total; e += NT) {
                const int r = e / p.PI;
                const int cc = e - r * p.PI;
                const int gy = min(max(y0 - C + r, 0), p.H - 1);
                const int gx = min(max(x0 - C4 + cc, 0), p.W - 1);
                in[e] = img[(size_t)gy * p.W + gx];
            }
        }
        __syncthreads();

        // row pass: unit = (RC-column group, staged row), rows fastest; output column j of the
        // unit = sum_a kx[a] * staged column (RC cg + j + D + a).  The results replace the staged
        // input in place (columns 0..63 of each row): every unit is computed into registers
        // first, and a barrier separates the last read from the first write.
        constexpr int RU = TW / RC * ROWS / NT;           // units per thread
        float acc[RU][RC];
        float wx[4 * K4];
#pragma unroll
        for (int g = 0; g < K4; ++g) {
            const float4v w = *reinterpret_cast<const float4v *>(wxl + 4 * g);
            wx[4 * g] = w.x; wx[4 * g + 1] = w.y; wx[4 * g + 2] = w.z; wx[4 * g + 3] = w.w;
        }
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            const int u = min(tid + NT * k, (TW / RC) * RH - 1);
            const int cgr = (int)fdiv((uint32_t)u, p.div_rh);
            const int r = u - cgr * RH;
            const float *src = in + r * p.PI + RC * cgr;
            float win[4 * NWR];
#pragma unroll
            for (int g = 0; g < NWR; ++g) {
                const float4v h = *reinterpret_cast<const float4v *>(src + 4 * g);
                win[4 * g] = h.x; win[4 * g + 1] = h.y; win[4 * g + 2] = h.z; win[4 * g + 3] = h.w;
            }
#pragma unroll
            for (int j = 0; j < RC; ++j) acc[k][j] = 0.0f;
#pragma unroll
            for (int a = 0; a < K; ++a)
#pragma unroll
                for (int j = 0; j < RC; ++j) acc[k][j] = fmaf(wx[a], win[j + D + a], acc[k][j]);
            // long windows: one unit's window at a time in registers.  The empty statement
            // consumes the sums and clobbers memory, so these multiply-adds stay above it and
            // the next unit's reads below it.
            if constexpr (LONG && RU > 1)
                asm volatile("" : "+v"(acc[k][0]), "+v"(acc[k][1]), "+v"(acc[k][2]), "+v"(acc[k][3]),
                                  "+v"(acc[k][4]), "+v"(acc[k][5]), "+v"(acc[k][6]), "+v"(acc[k][7]) : : "memory");
        }
        __syncthreads();
        float *mid = in;                                  // [RH][PI], columns 0..63
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            const int u = tid + NT * k;
            if (u < (TW / RC) * RH) {
                const int cgr = (int)fdiv((uint32_t)u, p.div_rh);
                const int r = u - cgr * RH;
                float *dst = mid + r * p.PI + RC * cgr;
#pragma unroll
                for (int j = 0; j < RC; j += 4)
                    *reinterpret_cast<float4v *>(dst + j) = (float4v){acc[k][j], acc[k][j + 1], acc[k][j + 2], acc[k][j + 3]};
            }
        }
        __syncthreads();

        // column pass: unit = PR rows x PC columns, column groups fastest: one LDS read or store
        // a row.  Row q of the K + PR - 1 rows a unit reads feeds output row i with tap
        // q - i.
        float *out = y + (size_t)T.n * p.H * p.W;
        float wy[4 * K4];
#pragma unroll
        for (int g = 0; g < K4; ++g) {
            const float4v w = *reinterpret_cast<const float4v *>(wyl + 4 * g);
            wy[4 * g] = w.x; wy[4 * g + 1] = w.y; wy[4 * g + 2] = w.z; wy[4 * g + 3] = w.w;
        }
        constexpr int CG = TW / PC;
        for (int u = tid; u < (p.TH / PR) * CG; u += NT) {
            const int rg = u / CG, cg2 = u % CG;
            const float *src = mid + (PR * rg) * p.PI + PC * cg2;
            run o[PR];
#pragma unroll
            for (int i = 0; i < PR; ++i)
#pragma unroll
                for (int j = 0; j < PC; ++j) o[i][j] = 0.0f;
            // QC rows at a time: their reads, then their multiply-adds (for long windows the
            // scheduler must not pull all K + PR - 1 reads to the front: PC registers each)
            constexpr int QC = LONG ? 16 / PC : 32 / PC;
#pragma unroll
            for (int q0 = 0; q0 < K + PR - 1; q0 += QC) {
                run v[QC];
#pragma unroll
                for (int e = 0; e < QC; ++e)
                    if (q0 + e < K + PR - 1) v[e] = *reinterpret_cast<const run *>(src + (q0 + e) * p.PI);
#pragma unroll
                for (int e = 0; e < QC; ++e) {
                    const int q = q0 + e;
#pragma unroll
                    for (int i = 0; i < PR; ++i)
                        if (q < K + PR - 1 && q - i >= 0 && q - i < K)
#pragma unroll
                            for (int j = 0; j < PC; ++j) o[i][j] = fmaf(wy[q - i], v[e][j], o[i][j]);
                }
                if constexpr (LONG)
#pragma unroll
                    for (int i = 0; i < PR; ++i) asm volatile("" : "+v"(o[i]) : : "memory");
            }
            const int gx = x0 + PC * cg2;
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                const int gy = y0 + PR * rg + i;
                if (gy >= p.H) continue;
                float *dst = out + (size_t)gy * p.W + gx;
                if (!RAGGED) {
                    if (gx < p.W) *reinterpret_cast<run *>(dst) = o[i];
                } else if (gx + PC - 1 < p.W) {
                    __builtin_memcpy(dst, &o[i], 4 * PC);
                } else {
#pragma unroll
                    for (int j = 0; j < PC - 1; ++j)
                        if (gx + j < p.W) dst[j] = o[i][j];
                }
            }
        }
        if (FORM != SEP_PERSISTENT) break;                // one tile a workgroup
        __syncthreads();                                  // the staged tile is free again
    }
}

template <int K, bool RAGGED, int FORM>
static hipError_t launch_sep_form(const SepParams &p, const float *x, const float *kx, const float *ky, float *y,
                                  hipStream_t s, int64_t ntiles)
{
    static std::atomic<int> raised{0};
    if (hipError_t e = raise_lds_limit_once(reinterpret_cast<const void *>(merit_sepfilter_tile<K, RAGGED, FORM>), raised);
        e != hipSuccess)
        return e;
    // persistent workgroups: as many as are resident (the registers allow four a compute unit as well)
    int64_t grid = ntiles;
    if (FORM == SEP_PERSISTENT) {
        const int64_t slots = (int64_t)device_cu_count() * p.wg_per_cu;
        if (grid > slots) grid = slots;
    }
    hipLaunchKernelGGL((merit_sepfilter_tile<K, RAGGED, FORM>), dim3((uint32_t)grid), dim3(FORM == SEP_FEW ? 512 : 256),
                       (size_t)p.lds_bytes, s, p, x, kx, ky, y);
    return hipGetLastError();
}

template <int K>
static hipError_t launch_sep(const SepParams &p, const float *x, const float *kx, const float *ky, float *y,
                             hipStream_t s, int64_t ntiles)
{
    const bool ragged = (p.W & 3) != 0;
    if (p.form == SEP_FEW)
        return ragged ? launch_sep_form<K, true, SEP_FEW>(p, x, kx, ky, y, s, ntiles)
                      : launch_sep_form<K, false, SEP_FEW>(p, x, kx, ky, y, s, ntiles);
    if constexpr (sep_many(K) == SEP_TILES)
        if (p.form == SEP_TILES)
            return ragged ? launch_sep_form<K, true, SEP_TILES>(p, x, kx, ky, y, s, ntiles)
                          : launch_sep_form<K, false, SEP_TILES>(p, x, kx, ky, y, s, ntiles);
    if (p.form != SEP_PERSISTENT) return hipErrorInvalidValue;
    return ragged ? launch_sep_form<K, true, SEP_PERSISTENT>(p, x, kx, ky, y, s, ntiles)
                  : launch_sep_form<K, false, SEP_PERSISTENT>(p, x, kx, ky, y, s, ntiles);
}

hipError_t launch_sepfilter(const SepParams &p, const float *x, const float *kx, const float *ky, float *y,
                            hipStream_t s)
{
    const int64_t ntiles = (int64_t)p.N * p.tiles_y * p.tiles_x;
    if (ntiles == 0) return hipSuccess;
    switch (p.k) {
#define MERIT_SEP_CASE(Kv) case Kv: return launch_sep<Kv>(p, x, kx, ky, y, s, ntiles)
#define MERIT_SEP_CASE8(B)                                                                           \
    MERIT_SEP_CASE(B + 1); MERIT_SEP_CASE(B + 2); MERIT_SEP_CASE(B + 3); MERIT_SEP_CASE(B + 4);      \
    MERIT_SEP_CASE(B + 5); MERIT_SEP_CASE(B + 6); MERIT_SEP_CASE(B + 7); MERIT_SEP_CASE(B + 8)
        MERIT_SEP_CASE8(0); MERIT_SEP_CASE8(8); MERIT_SEP_CASE8(16); MERIT_SEP_CASE8(24);
#undef MERIT_SEP_CASE8
#undef MERIT_SEP_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace merit
