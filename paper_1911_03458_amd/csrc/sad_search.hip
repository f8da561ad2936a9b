// Block-matching motion estimation for gfx950: two-level ranged inner product.
//
// k = (by, bx | dy, dx, i, j).  Inner level: L1 distance (Section III-B, Eq. 4)
// between the current block and the reference block displaced by the search
// indices (index pattern of Section III-C, Eq. 8):
//     M(cur)[p,a] = cur[by*B + i,          bx*B + j         ]
//     M(ref)[p,a] = ref[by*B + i + dy - R, bx*B + j + dx - R]   (clamped to the frame)
// Outer level: min / argmin over (dy,dx), ties to the lowest raster index.
//
// The reference search window (B+2R)^2, i.e. the minimal covering sub-tensor of
// Section IV-A, Eq. 9, is staged once in LDS with the clamping resolved there;
// candidates then read it branch-free.  Four pixels per lane-op with v_sad_u8.
// The (sad, raster index) pair is packed into one u32 key so that integer min
// gives the lexicographic minimum, reduced across the wavefront with DPP.
#include "merit_internal.h"

namespace merit {

constexpr int KEY_SHIFT = 14;                 // raster index < 2^14 (R <= 63)
constexpr uint32_t KEY_MASK = (1u << KEY_SHIFT) - 1u;

// min over the 64 lanes of a wavefront; the result is valid in lane 63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_min_step(uint32_t v)
{
    // lanes whose source is disabled or out of range keep the identity 0xffffffff
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)0xffffffff, (int)v, CTRL, ROW_MASK, 0xf, false);
    return o < v ? o : v;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = dpp_min_step<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
    v = dpp_min_step<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
    v = dpp_min_step<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_min_step<0x140, 0xf>(v);   // row_mirror: every lane holds its row's min
    v = dpp_min_step<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_min_step<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// v + (the lanes below in the same group of G = 8 or 16 lanes): the last lane of every
// group holds the group's sum.  Lanes shifted in from outside a 16-lane row read 0.
template <int G>
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
    if (G == 16) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
    return v;
}

// Stage the clamped search window of block (by,bx) as bytes win[wy*pitch + wx],
// wy,wx in [0, B+2R), four bytes per thread-iteration.
__device__ __forceinline__ void stage_window(const SadParams &p, const uint8_t *__restrict__ ref,
                                             uint32_t *win32, int gy0, int gx0, int rows, int cols4,
                                             FastDiv div_cols4, int pitch4, int tid, int nthreads)
{
    // (four pixels are one load on any byte boundary: frames whose rows are not whole dwords used to be fetched a byte at
    // a time: 326x550, 16x16 blocks, R = 8: 12.8 -> 9.5 us on the kernel for any shape)
    const int n = rows * cols4;
    for (int i = tid; i < n; i += nthreads) {
        const int wy = (int)fdiv((uint32_t)i, div_cols4);
        const int w4 = i - wy * cols4;
        const int gy = min(max(gy0 + wy, 0), p.H - 1);
        const int gx = gx0 + 4 * w4;
        const uint8_t *row = ref + (size_t)gy * p.W;
        uint32_t v;
        if (gx >= 0 && gx + 3 < p.W) {
            __builtin_memcpy(&v, row + gx, 4);
        } else {
            v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int cx = min(max(gx + b, 0), p.W - 1);
                v |= (uint32_t)row[cx] << (8 * b);
            }
        }
        win32[wy * pitch4 + w4] = v;
    }
}

// The same for frames of 16 and more columns, 16 pixels a load and all of a thread's loads in flight before the first is
// written (one by one they were ten trips to memory in a row).  A load that crosses an edge of its row is moved inside it,
// its pixels moved back and the edge's pixel repeated beside them.  PITCH4: dwords of a staged row (a multiple of 4).
template <int ROWS, int COLS16, int PITCH4, int NTHREADS>
__device__ __forceinline__ void stage_window16(const SadParams &p, const uint8_t *__restrict__ ref, uint32_t *win32, int gy0,
                                               int gx0, int tid)
{
    constexpr int U = ROWS * COLS16, NU = (U + NTHREADS - 1) / NTHREADS;
    static_assert(PITCH4 % 4 == 0 && PITCH4 >= 4 * COLS16, "16-byte rows");
    uint4 v[NU];
    int moved[NU];                                                 // pixels by which the load was moved right
    // (wavefronts whose further units are all past the last one: none of those)
    const int first = __builtin_amdgcn_readfirstlane(tid & ~63);
#pragma unroll
    for (int k = 0; k < NU; ++k) {
        if (k > 0 && first + NTHREADS * k >= U) break;
        const int u = min(tid + NTHREADS * k, U - 1);
        const int wy = u / COLS16, gx = gx0 + 16 * (u - wy * COLS16);
        const int at = min(max(gx, 0), p.W - 16);
        moved[k] = at - gx;
        __builtin_memcpy(&v[k], ref + (size_t)min(max(gy0 + wy, 0), p.H - 1) * p.W + at, 16);
    }
#pragma unroll
    for (int k = 0; k < NU; ++k) {
        if (k > 0 && first + NTHREADS * k >= U) break;
        if (moved[k] != 0) {
            const int n = min(abs(moved[k]), 16);
            uint64_t lo = ((uint64_t)v[k].y << 32) | v[k].x, hi = ((uint64_t)v[k].w << 32) | v[k].z;
            if (moved[k] > 0) {                                    // past the left edge: up by n, the first pixel below
                const uint64_t e = (lo & 0xff) * 0x0101010101010101ull;
                const uint64_t l = n >= 8 ? e : (lo << (8 * n)) | (e >> (64 - 8 * n));
                const uint64_t h = n >= 16 ? e : n > 8 ? (lo << (8 * n - 64)) | (e >> (128 - 8 * n)) : n == 8 ? lo : (hi << (8 * n)) | (lo >> (64 - 8 * n));
                lo = l; hi = h;
            } else {                                               // past the right edge: down by n, the last pixel above
                const uint64_t e = (hi >> 56) * 0x0101010101010101ull;
                const uint64_t h = n >= 8 ? e : (hi >> (8 * n)) | (e << (64 - 8 * n));
                const uint64_t l = n >= 16 ? e : n > 8 ? (hi >> (8 * n - 64)) | (e << (128 - 8 * n)) : n == 8 ? hi : (lo >> (8 * n)) | (hi << (64 - 8 * n));
                lo = l; hi = h;
            }
            v[k] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
        }
        const int u = tid + NTHREADS * k;
        if (U % NTHREADS == 0 || u < U) *reinterpret_cast<uint4 *>(win32 + u / COLS16 * PITCH4 + 4 * (u % COLS16)) = v[k];
    }
}

// Pixels x .. x + 3 of a row of W >= 4, those past its end repeating the last one, from one load on any byte boundary.
__device__ __forceinline__ uint32_t row_dword(const uint8_t *__restrict__ row, int x, int W)
{
    const int at = min(x, W - 4);
    uint32_t v;
    __builtin_memcpy(&v, row + at, 4);
    const uint64_t more = ((uint64_t)((v >> 24) * 0x01010101u) << 32) | v;
    return (uint32_t)(more >> (8 * min(x - at, 4)));
}

// ---------------------------------------------------------------------------
// Generic kernel: one workgroup per block, one lane per candidate (strided).
// Any B that is a multiple of 4 (<= 32) and any R <= 63.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void merit_sad_generic(SadParams p, const uint8_t *__restrict__ cur,
                                                        const uint8_t *__restrict__ ref,
                                                        int32_t *__restrict__ sad, int32_t *__restrict__ mv)
{
    extern __shared__ __align__(16) uint32_t lds32[];
    const int tid = threadIdx.x;
    const int pitch4 = p.pitch >> 2;
    const int B4 = p.B >> 2;
    uint32_t *win32 = lds32;                                  // [win][pitch4] (+1 dword slack)
    uint32_t *cur32 = lds32 + p.win * pitch4 + 1;             // [B][B4]
    uint32_t *red = cur32 + p.B * B4;                         // [4]

    const uint32_t blk = xcd_band_item(blockIdx.x, p.xq, p.xr);   // a band of block rows per XCD
    const int by = (int)(blk / (uint32_t)p.nbx);
    const int bx = (int)(blk - (uint32_t)by * p.nbx);

    stage_window(p, ref, win32, by * p.B - p.R, bx * p.B - p.R, p.win, (p.win + 3) >> 2,
                 p.div_win4, pitch4, tid, 256);
    // current block; pixels past the frame edge (frames the block does not divide) repeat the
    // edge pixel, as the reference window does
    for (int i = tid; i < p.B * B4; i += 256) {
        const int r = i / B4, c4 = i - r * B4;
        const uint8_t *row = cur + (size_t)min(by * p.B + r, p.H - 1) * p.W;
        const int gx = bx * p.B + 4 * c4;
        uint32_t v;
        if (gx + 3 < p.W) {
            __builtin_memcpy(&v, row + gx, 4);
        } else {
            v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) v |= (uint32_t)row[min(gx + b, p.W - 1)] << (8 * b);
        }
        cur32[i] = v;
    }
    __syncthreads();

    uint32_t best = 0xffffffffu;
    const int ncand = p.n * p.n;
    for (int c = tid; c < ncand; c += 256) {
        const int dyi = (int)fdiv((uint32_t)c, p.div_n);       // dy + R
        const int dxi = c - dyi * p.n;                         // dx + R
        uint32_t acc = 0;
        for (int i = 0; i < p.B; ++i) {
            const int byte0 = (dyi + i) * p.pitch + dxi;
            const uint32_t sh = (uint32_t)(byte0 & 3);
            const uint32_t *w = win32 + (byte0 >> 2);
            uint32_t lo = w[0];
            for (int j4 = 0; j4 < B4; ++j4) {
                const uint32_t hi = w[j4 + 1];
                const uint32_t r4 = __builtin_amdgcn_alignbyte(hi, lo, sh);
                acc = __builtin_amdgcn_sad_u8(cur32[i * B4 + j4], r4, acc);
                lo = hi;
            }
        }
        const uint32_t key = (acc << KEY_SHIFT) | (uint32_t)c;
        best = key < best ? key : best;
    }
    best = wave_min_u32(best);
    if ((tid & 63) == 0) red[tid >> 6] = best;
    __syncthreads();
    if (tid == 0) {
        uint32_t k = red[0];
        for (int w = 1; w < 4; ++w) k = red[w] < k ? red[w] : k;
        const uint32_t c = k & KEY_MASK;
        const int dyi = (int)(c / (uint32_t)p.n);
        sad[blk] = (int32_t)(k >> KEY_SHIFT);
        mv[2 * blk + 0] = dyi - p.R;
        mv[2 * blk + 1] = (int)c - dyi * p.n - p.R;
    }
}

// ---------------------------------------------------------------------------
// Row-scan kernel for 16x16 blocks, R = 32 or 16: candidates are eliminated by a lower bound first.
//
// Bound by the vector ALU: the full scan is 64 v_sad_u8 a candidate, 56 us of them on a full-HD frame.  Most candidates
// need not be scanned: the sixteen 4x4 sums of a block and of its candidate differ by no more than the pixels do (the
// triangle inequality; multilevel successive elimination, Gao, Duanmu and Zou 2000), and compare in eight v_sad_u16.
//   1. A workgroup (four adjacent blocks, two wavefronts each) stages the joint search window in LDS, and from it the 4x4
//      sums at every position.
//   2. Lane l owns the candidates dx = l - R.  It walks the rows of sums; a row is fetched once for the four candidates
//      whose block rows it holds.  All bounds of the column stay in registers.
//   3. The candidate with the lowest bound is evaluated, a dword per lane; then every candidate whose bound is not above
//      the best sum so far (three of 4225, at the median, on a moving scene with sensor noise).  The key (sum, raster
//      index) decides ties as the full scan does: the result is the same for any input.
//   4. Blocks that this cannot help are scanned in full: those whose pixels differ from their 4x4 means by more than
//      the means do from the block's (flat or noisy ones, recognised before anything is built), and those with more
//      candidates left than a tenth of the scan's time.
// The full scan: the wavefront walks the window rows top to bottom; for window row r a lane byte-aligns its 16 reference
// pixels once (4 x v_alignbyte) and adds them into the partial sums of the (up to) sixteen candidates dy = r - i that
// use this row as block row i (4 x v_sad_u8 each).  Sixteen accumulators rotate: candidate dy completes at row dy + 15
// and its slot restarts for dy + 16.
// Four blocks a workgroup, a block inside a frame of whole dwords: its pixels come from memory once more, as scalar loads
// (64 v_readlane less a wavefront; the loads' latency shows on smaller frames, which have the other form).
// The 65th column at R = 32: its bounds one candidate per lane, its sums too with four blocks a workgroup, else sixteen lanes
// to a candidate.
// BPW: blocks per workgroup: four, the rows of a block's candidates split between two wavefronts, or one, split among four
// (R = 16 as well, on frames of 64 to 1200 blocks: 288x416 11.0 us on the kernel below -> 7.0, 480x640 11.2 -> 9.6).
// Workgroups go round-robin to the XCDs, not in bands of block rows: a band of sky or water would be the whole work of
// one of them (1080x1920: 77 us in bands, 53).
//
// us a launch, R = 32, full scan (one wavefront a block, in a kernel of its own) -> this: moving scenes with sensor noise,
// 1080x1920 75.3 -> 51, 720x1280 40.6 -> 27.7, 480x640 24.0 -> 14.9, 120x160 16.8 -> 8.6; smooth textures that move by
// block, 1088x1920, 75.3 -> 35.7; two unrelated scenes 76.8 -> 68.5; a still picture 76 -> 47.  Where every block is scanned,
// by two or four wavefronts that share its rows, large frames are slower: white noise 1080x1920 75.4 both, 995x1906 76.0 ->
// 78.1, 2160x3840 283 -> 287, 540x960 24.3 -> 24.7, 720x1280 40.7 -> 43.4 (480x640: 24.0 -> 16.9); a random texture that
// moves by block, 1080x1920, 75.5 -> 77.3.  (A single wavefront a block there, the other one idle: 95 at 1080x1920.)  With every block decided by its bounds a full-HD frame takes 27 us; the rest
// is the scans of a sixth of the blocks, which come in clusters and are dealt to the compute units by position.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void load_aligned16(const uint32_t *rowp, uint32_t sh, uint32_t (&r)[4])
{
    const uint32_t d0 = rowp[0], d1 = rowp[1], d2 = rowp[2], d3 = rowp[3], d4 = rowp[4];
    r[0] = __builtin_amdgcn_alignbyte(d1, d0, sh);
    r[1] = __builtin_amdgcn_alignbyte(d2, d1, sh);
    r[2] = __builtin_amdgcn_alignbyte(d3, d2, sh);
    r[3] = __builtin_amdgcn_alignbyte(d4, d3, sh);
}

// the sum over a wavefront's lanes, the same for all
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    v = group_sum_u32<16>(v);                                                                     // lane 15 of every row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);               // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);               // row_bcast:31
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// Row (lane % 16) of the block of which every lane holds a dword (row lane / 4).
__device__ __forceinline__ void rows_of_lanes(uint32_t cl, int lane, uint32_t (&crow)[4])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) crow[j] = (uint32_t)__builtin_amdgcn_ds_bpermute((4 * (lane & 15) + j) * 4, (int)cl);
}

// The full scan of ND candidate rows from d0 on of block wb, whose pixels are `cl` (four per lane) and, unless that is null,
// at `block` in memory, in rows of W4 dwords: the lowest key, the same for all lanes.  The column past the 64th, where there
// is one: of these rows (column = 0), of all rows (1), or not (-1).
template <int R, int ND, int PITCH4>
__device__ __forceinline__ uint32_t scan_rows(const uint32_t *lds32, uint32_t cl, const uint32_t *__restrict__ block, int W4,
                                              int wb, int d0, int lane, int column)
{
    constexpr int N = 2 * R + 1, NCOL = N < 64 ? N : 64, NLEFT = N - NCOL;
    static_assert(ND <= 64, "a candidate row per lane");
    // (a value to the compiler: with offsets that it knows it fetches the rows of all steps first, into registers that are
    // not there)
    int pitch = PITCH4;
    asm("" : "+s"(pitch));
    uint32_t c[16][4];                                             // the current block, wave-uniform
    if (block) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) c[i][j] = block[i * W4 + j];
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) c[i][j] = (uint32_t)__builtin_amdgcn_readlane((int)cl, 4 * i + j);
    }
    const int o = 16 * wb + min(lane, NCOL - 1);                   // idle lanes repeat the last column
    const uint32_t sh = (uint32_t)(o & 3);
    const uint32_t *base = lds32 + d0 * pitch + (o >> 2);
    uint32_t acc[16];
    uint32_t lbest = 0xffffffffu;                                  // (sum << 7) | row

    // one window row: block rows i in [ilo, ihi] accumulate into slot (rot - i) & 15, whose sum starts with row 0;
    // then candidate `fin` (if >= 0), which sits in slot (rot + 1) & 15, is complete
    auto step = [&](const uint32_t *rowp, int ilo, int ihi, int rot, int fin) __attribute__((always_inline)) {
        uint32_t r4[4];
        load_aligned16(rowp, sh, r4);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i < ilo || i > ihi) continue;
            const int slot = (rot - i) & 15;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[slot] = __builtin_amdgcn_sad_u8(c[i][j], r4[j], i + j == 0 ? 0u : acc[slot]);
        }
        if (fin >= 0) {
            const int slot = (rot + 1) & 15;
            const uint32_t key = (acc[slot] << 7) | (uint32_t)fin;
            lbest = key < lbest ? key : lbest;
        }
    };
    if constexpr (ND < 32) {
#pragma unroll
        for (int r = 0; r < ND + 15; ++r) step(base + r * pitch, max(0, r - ND + 1), min(15, r), r & 15, r - 15);
    } else {
        constexpr int NS = ND - 15, NSB = NS / 16, NSR = NS % 16;  // rows 15 .. ND - 1 use all 16 block rows
#pragma unroll
        for (int r = 0; r < 15; ++r) step(base + r * pitch, 0, r, r, -1);
#pragma unroll 1
        for (int k = 0; k < NSB; ++k) {
            const uint32_t *rp = base + (15 + 16 * k) * pitch;
#pragma unroll
            for (int j = 0; j < 16; ++j) step(rp + j * pitch, 0, 15, (15 + j) & 15, 16 * k + j);
        }
#pragma unroll
        for (int j = 0; j < NSR; ++j)
            step(base + (15 + 16 * NSB + j) * pitch, 0, 15, (15 + j) & 15, 16 * NSB + j);
#pragma unroll
        for (int e = 1; e <= 15; ++e)
            step(base + (ND - 1 + e) * pitch, e, 15, (ND - 1 + e) & 15, ND - 1 + e - 15);
    }
    uint32_t key = lane < NCOL ? ((lbest >> 7) << KEY_SHIFT) | ((uint32_t)(d0 + (int)(lbest & 127u)) * N + (uint32_t)lane) : 0xffffffffu;
    // (the condition on the pitch, always true, keeps this apart from the scan: in one block with it the compiler fetches all
    // rows first, into registers that are not there)
    if (NLEFT > 0 && ND > 24 && pitch != 0 && column >= 0) {       // the last column: a candidate row per lane
        const int ol = 16 * wb + NCOL;
        const uint32_t sl = (uint32_t)(ol & 3);
        // (idle lanes repeat the last row; of all rows the 65th is below)
        const int dl = column > 0 ? lane : d0 + min(lane, ND - 1);
        const uint32_t *lp = lds32 + dl * pitch + (ol >> 2);
        uint32_t a = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            uint32_t r4[4];
            load_aligned16(lp + i * pitch, sl, r4);
#pragma unroll
            for (int j = 0; j < 4; ++j) a = __builtin_amdgcn_sad_u8(c[i][j], r4[j], a);
        }
        a = (a << KEY_SHIFT) | (uint32_t)(dl * N + NCOL);
        key = a < key ? a : key;
    }
    if (NLEFT > 0 && pitch != 0 && (ND <= 24 || column > 0)) {     // ... sixteen lanes to a candidate, a row each
        uint32_t crow[4];
        rows_of_lanes(cl, lane, crow);
        const int ol = 16 * wb + NCOL;
        const int end = ND <= 24 ? d0 + ND : N;
#pragma unroll 1
        for (int i = ND <= 24 ? d0 : N - 1; i < end; i += 4) {
            const int dy = min(i + (lane >> 4), end - 1);
            uint32_t r4[4], a = 0;
            load_aligned16(lds32 + (dy + (lane & 15)) * pitch + (ol >> 2), (uint32_t)(ol & 3), r4);
#pragma unroll
            for (int j = 0; j < 4; ++j) a = __builtin_amdgcn_sad_u8(crow[j], r4[j], a);
            a = (group_sum_u32<16>(a) << KEY_SHIFT) | (uint32_t)(dy * N + NCOL);
            if ((lane & 15) == 15) key = a < key ? a : key;        // (whole in the last lane of the sixteen)
        }
    }
    return wave_min_u32(key);
}

template <int R, int BPW>
__global__ __launch_bounds__(BPW == 4 ? 512 : 256, R == 32 ? 8 : 4) void merit_sad_rowscan16(SadParams p, const uint8_t *__restrict__ cur,
                                                                             const uint8_t *__restrict__ ref,
                                                                             int32_t *__restrict__ sad, int32_t *__restrict__ mv)
{
    static_assert(BPW == 1 || BPW == 4, "blocks per workgroup");
    constexpr int N = 2 * R + 1, ROWS = 16 + 2 * R;
    constexpr int WPB = BPW == 1 ? 4 : 2, NW = BPW * WPB, NT = 64 * NW;           // wavefronts per block, per workgroup
    constexpr int ND = (N + WPB - 1) / WPB;                        // candidate rows per wavefront
    constexpr int NCOL = N < 64 ? N : 64, NLEFT = N - NCOL;        // candidate columns that are lanes; the rest
    static_assert(N >= 16 && NLEFT <= 1 && ND <= 64, "R = 8 .. 32");
    constexpr int SROWS = ROWS - 3, SCOLS = sad_rowscan16_cols(R, BPW);            // 4x4 sums: rows, halves of a row
    constexpr int NSEG = NT / SCOLS, SEG = (SROWS + NSEG - 1) / NSEG;             // rows per thread when they are built
    constexpr int MOST = SAD_LIST;                                 // candidates worth evaluating one by one
    constexpr int pitch4 = sad_rowscan16_pitch4(R, BPW);

    extern __shared__ __align__(16) uint32_t lds32[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wb = wv / WPB, part = wv % WPB;                      // block inside the workgroup, share of its candidates
    uint16_t *sums = reinterpret_cast<uint16_t *>(lds32 + ROWS * pitch4);         // [SROWS][SCOLS]
    uint32_t *red = lds32 + ROWS * pitch4 + SROWS * SCOLS / 2;     // [2][NW]
    uint32_t *result = red + 2 * NW;                               // [BPW] keys
    uint16_t *list = reinterpret_cast<uint16_t *>(result + BPW) + wv * MOST;      // this wavefront's [MOST]
    const int by = (int)(blockIdx.x / (uint32_t)p.groups_x);
    const int bx0 = (int)(blockIdx.x - (uint32_t)by * p.groups_x) * BPW;
    const int bx = min(bx0 + wb, p.nbx - 1);                       // (ragged last group: the last block again, not stored)

    // the current block, four pixels per lane: row lane / 4, columns 4 (lane % 4) .. + 3; pixels past the frame's edge
    // repeat the edge
    const uint32_t cl = row_dword(cur + (size_t)min(by * 16 + (lane >> 2), p.H - 1) * p.W, bx * 16 + 4 * (lane & 3), p.W);
    if (p.W >= 16) stage_window16<ROWS, (16 * BPW + 2 * R) / 16, pitch4, NT>(p, ref, lds32, by * 16 - R, bx0 * 16 - R, tid);
    else stage_window(p, ref, lds32, by * 16 - R, bx0 * 16 - R, ROWS, (16 * BPW + 2 * R) / 4, p.div_win4, pitch4, tid, NT);

    // its 4x4 sums: the rows of a 4x4 are lanes 4 apart
    uint32_t s4 = __builtin_amdgcn_sad_u8(cl, 0, 0);
    s4 += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s4, 0x124, 0xf, 0xf, true);          // row_ror:4
    s4 += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s4, 0x128, 0xf, 0xf, true);          // row_ror:8
    // (four blocks a workgroup: by one wavefront of a block, for both; with one block, where the chain of a block is the whole
    // launch, by each: the answer is then there without a trip through LDS, 8.6 against 9.1 us on 120x160)
    bool bounds = false;
    if (BPW == 1 || part == 0) {
        // (means rounded down; four lanes hold each 4x4 sum)
        const uint32_t mean = wave_sum_u32(s4) >> 6;               // of the 4x4 sums
        const uint32_t coarse = wave_sum_u32(s4 > mean ? s4 - mean : mean - s4) >> 2;
        const uint32_t fine = wave_sum_u32(__builtin_amdgcn_sad_u8(cl, (s4 >> 4) * 0x01010101u, 0));
        bounds = coarse >= fine;
        if (lane == 0) red[wv] = bounds ? 1u : 0u;
    }
    if (tid < BPW) result[tid] = 0xffffffffu;
    __syncthreads();
    if (BPW != 1) bounds = __builtin_amdgcn_readfirstlane((int)red[wb * WPB]) != 0;

    const int d0 = min(part * ND, N - ND);                         // first candidate row (the last share overlaps)
    uint32_t best = 0xffffffffu;                                   // wave-uniform (sum << 14) | raster index
    bool scan = !bounds;
    uint32_t any_bounds = 0;
#pragma unroll
    for (int i = 0; i < NW; i += WPB) any_bounds |= red[i];
    if (any_bounds != 0) {
        const int seg = tid / SCOLS, x = tid - seg * SCOLS;
        if (seg < NSEG) {
            const uint32_t sh = (uint32_t)(x & 3);
            const int y0 = min(seg * SEG, SROWS - SEG);            // (the last segment overlaps the one before: the same values)
            const uint32_t *src = lds32 + y0 * pitch4 + (x >> 2);
            uint16_t *dst = sums + y0 * SCOLS + x;
            auto row4 = [&](const uint32_t *r) __attribute__((always_inline)) {
                return __builtin_amdgcn_sad_u8(__builtin_amdgcn_alignbyte(r[1], r[0], sh), 0, 0);
            };
            uint32_t h[4];
#pragma unroll
            for (int i = 0; i < 3; ++i) h[i] = row4(src + i * pitch4);
            uint32_t s = h[0] + h[1] + h[2];
#pragma unroll
            for (int y = 0; y < SEG; ++y) {
                h[3] = row4(src + (y + 3) * pitch4);
                s += h[3];
                dst[y * SCOLS] = (uint16_t)s;
                s -= h[0];
                h[0] = h[1]; h[1] = h[2]; h[2] = h[3];
            }
        }
        __syncthreads();

        uint32_t lb[ND], lb_left = 0xffffffffu, low = 0xffffffffu;
        if (bounds) {
            uint32_t sp[4][2];                                     // the block's sums, in the same pairs, wave-uniform
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    sp[a][j] = (uint32_t)__builtin_amdgcn_readlane((int)s4, 16 * a + 2 * j) |
                               (uint32_t)__builtin_amdgcn_readlane((int)s4, 16 * a + 2 * j + 1) << 16;
            auto pair = [](const uint16_t *at) __attribute__((always_inline)) {       // the sums at x and x + 4
                ushort2v v;
                v.x = at[0]; v.y = at[4];
                return __builtin_bit_cast(uint32_t, v);
            };
            const uint16_t *src = sums + d0 * SCOLS + 16 * wb + min(lane, NCOL - 1);
#pragma unroll
            for (int y = 0; y < ND + 12; ++y) {
                const uint32_t v0 = pair(src + y * SCOLS), v1 = pair(src + y * SCOLS + 8);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const int dy = y - 4 * a;
                    if (dy < 0 || dy >= ND) continue;
                    lb[dy] = __builtin_amdgcn_sad_u16(sp[a][0], v0, a == 0 ? 0u : lb[dy]);
                    lb[dy] = __builtin_amdgcn_sad_u16(sp[a][1], v1, lb[dy]);
                }
            }
#pragma unroll
            for (int dy = 0; dy < ND; ++dy) {
                const uint32_t k = (lb[dy] << 7) | (uint32_t)dy;
                low = k < low ? k : low;
            }
            low = lane < NCOL ? ((low >> 7) << KEY_SHIFT) | ((uint32_t)(d0 + (int)(low & 127u)) * N + (uint32_t)lane) : 0xffffffffu;
            if constexpr (NLEFT > 0) {                             // the last column: candidate row d0 + lane
                uint32_t v = 0;
                const uint16_t *end = sums + (d0 + min(lane, ND - 1)) * SCOLS + 16 * wb + NCOL;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    v = __builtin_amdgcn_sad_u16(sp[a][0], pair(end + 4 * a * SCOLS), v);
                    v = __builtin_amdgcn_sad_u16(sp[a][1], pair(end + 4 * a * SCOLS + 8), v);
                }
                if (lane < ND) {
                    lb_left = v;
                    const uint32_t k = (v << KEY_SHIFT) | ((uint32_t)(d0 + lane) * N + NCOL);
                    low = k < low ? k : low;
                }
            }
            low = wave_min_u32(low);
        }
        if (lane == 0) red[NW + wv] = low;
        __syncthreads();
        if (bounds) {
            // the block's candidate with the lowest bound, a dword per lane
            uint32_t first = red[NW + wb * WPB];
#pragma unroll
            for (int i = 1; i < WPB; ++i) first = min(first, red[NW + wb * WPB + i]);
            first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(first & KEY_MASK));
            {
                const int dy = (int)(first / (uint32_t)N), o = 16 * wb + (int)first - dy * N;
                const uint32_t *r = lds32 + (dy + (lane >> 2)) * pitch4 + (o >> 2) + (lane & 3);
                best = (wave_sum_u32(__builtin_amdgcn_sad_u8(cl, __builtin_amdgcn_alignbyte(r[1], r[0], (uint32_t)(o & 3)), 0)) << KEY_SHIFT) | first;
            }
            const uint32_t most = best >> KEY_SHIFT;
            // the candidates that are left, if any: a bit for each row of a lane's column
            if ((low >> KEY_SHIFT) <= most) {
                constexpr int NM = (ND + 31) / 32;
                uint32_t m[NM], left = 0;
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    m[i] = 0;
#pragma unroll
                    for (int dy = min(32 * i + 31, ND - 1); dy >= 32 * i; --dy) m[i] = m[i] + m[i] + (lb[dy] <= most ? 1u : 0u);
                    if (lane >= NCOL) m[i] = 0;
                    left += (uint32_t)__popc(m[i]);
                }
                const bool last = NLEFT > 0 && lb_left <= most;
                left += last ? 1u : 0u;
                // their places in the list: the sum over the lanes up to this one
                uint32_t upto = group_sum_u32<16>(left);
                upto += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)upto, 0x142, 0xa, 0xf, false);
                upto += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)upto, 0x143, 0xc, 0xf, false);
                const int count = __builtin_amdgcn_readlane((int)upto, 63);
                if (count > MOST) {
                    scan = true;
                } else if (count > 0) {
                    int at = (int)(upto - left);
                    if (last) list[at++] = (uint16_t)(lane << 7 | NCOL);
#pragma unroll
                    for (int i = 0; i < NM; ++i)
                        while (m[i] != 0) {
                            list[at++] = (uint16_t)((32 * i + __builtin_ctz(m[i])) << 7 | lane);
                            m[i] &= m[i] - 1;
                        }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // (this wavefront's own: no barrier)
                    // sixteen lanes to a candidate, a block row each
                    uint32_t crow[4];
                    rows_of_lanes(cl, lane, crow);
                    uint32_t key = 0xffffffffu;
#pragma unroll 1
                    for (int i = 0; i < count; i += 8) {
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            const int e = list[min(i + 4 * k + (lane >> 4), count - 1)];
                            const int dy = d0 + (e >> 7), dx = e & 127, o = 16 * wb + dx;
                            uint32_t r4[4], a = 0;
                            load_aligned16(lds32 + (dy + (lane & 15)) * pitch4 + (o >> 2), (uint32_t)(o & 3), r4);
#pragma unroll
                            for (int j = 0; j < 4; ++j) a = __builtin_amdgcn_sad_u8(crow[j], r4[j], a);
                            a = (group_sum_u32<16>(a) << KEY_SHIFT) | (uint32_t)(dy * N + dx);
                            key = a < key ? a : key;                   // (whole in lane 15 of the sixteen)
                        }
                    }
                    key = wave_min_u32((lane & 15) == 15 ? key : 0xffffffffu);
                    best = key < best ? key : best;
                }
            }
        }
    }
    if (scan) {
        const bool whole = BPW == 4 && (p.W & 3) == 0 && by * 16 + 16 <= p.H && bx * 16 + 16 <= p.W;
        const uint32_t *block = whole ? reinterpret_cast<const uint32_t *>(cur + (size_t)by * 16 * p.W + bx * 16) : nullptr;
        // no block of the workgroup with bounds: both wavefronts of each scan, and one of them takes its last column, four such
        // wavefronts on four SIMDs (one block a workgroup, one of its four wavefronts: 120x160 6.5 -> 7.8 us; not there)
        const int column = WPB == 2 && any_bounds == 0 ? (part == ((wb ^ wb >> 1) & 1) ? 1 : -1) : 0;
        best = min(best, scan_rows<R, ND, pitch4>(lds32, cl, block, p.W >> 2, wb, d0, lane, column));
    }
    if (lane == 0) atomicMin(&result[wb], best);
    __syncthreads();
    if (tid >= BPW || bx0 + tid >= p.nbx) return;
    best = result[tid];
    const uint32_t blk = (uint32_t)by * p.nbx + bx0 + tid;
    const uint32_t cidx = best & KEY_MASK;
    const int dyi = (int)(cidx / (uint32_t)N);
    sad[blk] = (int32_t)(best >> KEY_SHIFT);
    mv[2 * blk + 0] = dyi - R;
    mv[2 * blk + 1] = (int)cidx - dyi * N - R;
}

// ---------------------------------------------------------------------------
// Row-scan kernel, two blocks per wavefront: for search ranges whose 2R+1 candidate columns
// fill only half a wavefront (R <= 19), each 32-lane half owns one block, so a workgroup
// covers eight horizontally adjacent blocks.  The walk over the window rows is the one
// described above with B block rows and B rotating accumulators; the current block lives
// in vector registers (it differs between the halves).  Columns beyond the 32nd are run
// one candidate per lane.  B = 8 or 16.  (16x16 blocks with R = 8: 17 of 32 lanes have a column, and it is still
// 14.7 us against 40.2 of the kernel that takes any shape, on 1080x1920; 7.7 against 13.1 on 326x552.)
// ---------------------------------------------------------------------------
template <int B4>
__device__ __forceinline__ void load_aligned_row(const uint32_t *rowp, uint32_t sh, uint32_t (&r)[B4])
{
    uint32_t d[B4 + 1];
#pragma unroll
    for (int j = 0; j <= B4; ++j) d[j] = rowp[j];
#pragma unroll
    for (int j = 0; j < B4; ++j) r[j] = __builtin_amdgcn_alignbyte(d[j + 1], d[j], sh);
}

// min over each 32-lane half of a wavefront; valid in lanes 31 and 63
__device__ __forceinline__ uint32_t half_wave_min_u32(uint32_t v)
{
    v = dpp_min_step<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
    v = dpp_min_step<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
    v = dpp_min_step<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_min_step<0x140, 0xf>(v);   // row_mirror: every lane holds its row's min
    v = dpp_min_step<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    return v;
}

template <int B, int R, bool ANY>
__global__ __launch_bounds__(256) void merit_sad_rowscan_pair(SadParams p, const uint8_t *__restrict__ cur,
                                                             const uint8_t *__restrict__ ref,
                                                             int32_t *__restrict__ sad, int32_t *__restrict__ mv)
{
    static_assert(B == 8 || B == 16, "accumulator rotation needs a power of two");
    static_assert(2 * R >= B - 1 && 2 * R + 1 <= 40, "steady state needs 2R >= B-1; at most 8 extra columns");
    constexpr int N = 2 * R + 1, ROWS = B + 2 * R, B4 = B / 4;
    constexpr int NMAIN = N < 32 ? N : 32;          // candidate columns that are lane columns
    constexpr int NLEFT = N - NMAIN;                // the rest: one candidate per lane
    constexpr int NS = 2 * R - B + 2, NSB = NS / B, NSR = NS % B;   // rows B-1 .. 2R use all B block rows

    extern __shared__ __align__(16) uint32_t lds32[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pitch4 = p.pitch >> 2;
    const uint32_t g = xcd_band_item(blockIdx.x, p.xq, p.xr);     // a band of block rows per XCD
    const int by = (int)(g / (uint32_t)p.groups_x);
    const int bx0 = (int)(g - (uint32_t)by * p.groups_x) * 8;

    stage_window(p, ref, lds32, by * B - R, bx0 * B - R, ROWS, pitch4 - 1, p.div_win4, pitch4, tid, 256);
    __syncthreads();
    const int bxl = 2 * wv + hb;                    // block inside the workgroup's window
    const int bx = bx0 + bxl;
    const bool live = bx < p.nbx;                   // ragged last group: the half computes, nothing is written

    uint32_t c[B][B4];
    {
        // rows past the last one (H % B != 0) repeat it; dwords past the end of a row
        // (W % B != 0, W % 4 == 0) are four copies of its last pixel
        const uint32_t *cp = reinterpret_cast<const uint32_t *>(cur);
        const int W4 = p.W >> 2;
        const int d0 = min(bx, p.nbx - 1) * B4;
        if ((p.W & (B - 1)) == 0) {                  // whole blocks per row: the plain loads
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int row = min(by * B + i, p.H - 1);
#pragma unroll
                for (int j = 0; j < B4; ++j) c[i][j] = cp[row * W4 + d0 + j];
            }
        } else if (ANY && (p.W & 3) != 0) {          // rows on any byte boundary
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int row = min(by * B + i, p.H - 1);
#pragma unroll
                for (int j = 0; j < B4; ++j) c[i][j] = row_dword(cur + (size_t)row * p.W, 4 * (d0 + j), p.W);
            }
        } else {
#pragma unroll
            for (int i = 0; i < B; ++i) {
                const int row = min(by * B + i, p.H - 1);
#pragma unroll
                for (int j = 0; j < B4; ++j) {
                    const uint32_t v = cp[row * W4 + min(d0 + j, W4 - 1)];
                    c[i][j] = d0 + j < W4 ? v : (v >> 24) * 0x01010101u;
                }
            }
        }
    }

    // row (lane & (B-1)) of this half's current block, for the split tail below
    uint32_t crow[B4];
    {
        const uint32_t *cp = reinterpret_cast<const uint32_t *>(cur);
        const int W4 = p.W >> 2;
        const int row = min(by * B + (l32 & (B - 1)), p.H - 1);
        const int d0 = min(bx, p.nbx - 1) * B4;
        if (ANY && (p.W & 3) != 0) {
#pragma unroll
            for (int j = 0; j < B4; ++j) crow[j] = row_dword(cur + (size_t)row * p.W, 4 * (d0 + j), p.W);
        } else {
#pragma unroll
            for (int j = 0; j < B4; ++j) {
                const uint32_t v = cp[row * W4 + min(d0 + j, W4 - 1)];
                crow[j] = d0 + j < W4 ? v : (v >> 24) * 0x01010101u;
            }
        }
    }

    uint32_t best = 0xffffffffu;                    // (sad << 14) | raster index
    {
        const int dxi = l32;
        const int o = B * bxl + min(dxi, NMAIN - 1);          // idle lanes repeat the last column
        const uint32_t sh = (uint32_t)(o & 3);
        const uint32_t *base = lds32 + (o >> 2);
        uint32_t acc[B];
#pragma unroll
        for (int k = 0; k < B; ++k) acc[k] = 0;
        uint32_t lbest = 0xffffffffu;               // (sad << 7) | (dy + R)

        auto step = [&](const uint32_t *rowp, int ilo, int ihi, int rot, int fin) __attribute__((always_inline)) {
            uint32_t r4[B4];
            load_aligned_row<B4>(rowp, sh, r4);
#pragma unroll
            for (int i = 0; i < B; ++i) {
                if (i < ilo || i > ihi) continue;
                const int slot = (rot - i) & (B - 1);
#pragma unroll
                for (int j = 0; j < B4; ++j) acc[slot] = __builtin_amdgcn_sad_u8(c[i][j], r4[j], acc[slot]);
            }
            if (fin >= 0) {
                const int slot = (rot + 1) & (B - 1);
                const uint32_t key = (acc[slot] << 7) | (uint32_t)fin;
                lbest = key < lbest ? key : lbest;
                acc[slot] = 0;
            }
        };

#pragma unroll
        for (int r = 0; r < B - 1; ++r) step(base + r * pitch4, 0, r, r, -1);
#pragma unroll 1
        for (int k = 0; k < NSB; ++k) {
            const uint32_t *rp = base + (B - 1 + B * k) * pitch4;
#pragma unroll
            for (int j = 0; j < B; ++j) step(rp + j * pitch4, 0, B - 1, (B - 1 + j) & (B - 1), B * k + j);
        }
#pragma unroll
        for (int j = 0; j < NSR; ++j)
            step(base + (B - 1 + B * NSB + j) * pitch4, 0, B - 1, (B - 1 + j) & (B - 1), B * NSB + j);
#pragma unroll
        for (int e = 1; e <= B - 1; ++e)
            step(base + (2 * R + e) * pitch4, e, B - 1, (2 * R + e) & (B - 1), 2 * R + e - (B - 1));

        if (dxi < NMAIN) {
            const uint32_t dyi = lbest & 127u;
            best = ((lbest >> 7) << KEY_SHIFT) | (dyi * (uint32_t)N + (uint32_t)dxi);
        }
    }

    if (NLEFT > 0) {
        // what does not fill a pass of 32 candidates (one candidate at N = 33) is split B
        // lanes per candidate, a block row each
        constexpr int NCAND = NLEFT * N;
        constexpr int REM = NCAND % 32;
        constexpr bool SPLIT = REM > 0 && REM <= 32 / B;
        constexpr int NFULL = SPLIT ? NCAND - REM : NCAND;
#pragma unroll 1
        for (int c0 = 0; c0 < NFULL; c0 += 32) {
            const int cand = min(c0 + l32, NCAND - 1);         // idle lanes recompute the last candidate
            const int dyi = cand / NLEFT;
            const int dxi = NMAIN + (cand - dyi * NLEFT);
            const int o = B * bxl + dxi;
            const uint32_t sh = (uint32_t)(o & 3);
            const uint32_t *base = lds32 + dyi * pitch4 + (o >> 2);
            uint32_t a = 0;
#pragma unroll
            for (int i = 0; i < B; ++i) {
                uint32_t r4[B4];
                load_aligned_row<B4>(base + i * pitch4, sh, r4);
#pragma unroll
                for (int j = 0; j < B4; ++j) a = __builtin_amdgcn_sad_u8(c[i][j], r4[j], a);
            }
            const uint32_t key = (a << KEY_SHIFT) | (uint32_t)(dyi * N + dxi);
            best = key < best ? key : best;
        }
        if (SPLIT) {
            const int i = l32 & (B - 1);
            const int ci = NFULL + l32 / B;
            const int cand = min(ci, NCAND - 1);
            const int dyi = cand / NLEFT;
            const int dxi = NMAIN + (cand - dyi * NLEFT);
            const int o = B * bxl + dxi;
            uint32_t r4[B4];
            load_aligned_row<B4>(lds32 + (dyi + i) * pitch4 + (o >> 2), (uint32_t)(o & 3), r4);
            uint32_t a = 0;
#pragma unroll
            for (int j = 0; j < B4; ++j) a = __builtin_amdgcn_sad_u8(crow[j], r4[j], a);
            a = group_sum_u32<B>(a);
            const uint32_t key = (a << KEY_SHIFT) | (uint32_t)(dyi * N + dxi);
            if (i == B - 1 && ci < NCAND) best = key < best ? key : best;
        }
    }

    best = half_wave_min_u32(best);
    if (l32 == 31 && live) {
        const uint32_t blk = (uint32_t)by * p.nbx + bx;
        const uint32_t cidx = best & KEY_MASK;
        const int dyi = (int)(cidx / (uint32_t)N);
        sad[blk] = (int32_t)(best >> KEY_SHIFT);
        mv[2 * blk + 0] = dyi - R;
        mv[2 * blk + 1] = (int)cidx - dyi * N - R;
    }
}

// ---------------------------------------------------------------------------
// Row-scan kernel, seven blocks per wavefront: 8x8 blocks with R = 4, whose nine candidate columns fill 63 of the 64 lanes.
// The walk over the window rows is the one described above, eight accumulators rotating over the nine rows of candidates:
// 144 v_sad_u8 for nine candidates of seven blocks, where the kernel for any shape spends a workgroup on 81 candidates and
// as much again on its window.  A workgroup is four block rows of seven blocks, so that their windows share a staged area of
// 40 x 64 pixels (1.4 times the blocks' own, 2.1 for a single row of 28 blocks); that and the current blocks are one 16-byte
// load a thread each.  Bound by the launch and this one trip to memory.
// us a launch in a graph, kernel for any shape -> this: 64x64 3.3 -> 2.8, 480x640 8.2 -> 3.0, 822x1002 17.8 -> 3.4, 1080x1920
// 40.0 -> 4.6.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void merit_sad_rowscan_seven(SadParams p, const uint8_t *__restrict__ cur,
                                                              const uint8_t *__restrict__ ref,
                                                              int32_t *__restrict__ sad, int32_t *__restrict__ mv)
{
    constexpr int B = 8, R = 4, N = 2 * R + 1, BW = 7, PITCH4 = SEVEN_PITCH4;
    __shared__ __align__(16) uint32_t win32[SEVEN_ROWS * PITCH4], cur32[4 * B * PITCH4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t g = xcd_band_item(blockIdx.x, p.xq, p.xr);     // a band of block rows per XCD
    const int gy = (int)(g / (uint32_t)p.groups_x);
    const int bx0 = (int)(g - (uint32_t)gy * p.groups_x) * BW, by0 = gy * 4;

    // (64 columns of both; the planner asks for rows of 16 pixels)
    stage_window16<SEVEN_ROWS, 4, PITCH4, 256>(p, ref, win32, by0 * B - R, bx0 * B - R, tid);
    stage_window16<4 * B, 4, PITCH4, 256>(p, cur, cur32, by0 * B, bx0 * B, tid);
    __syncthreads();

    const int bl = min(lane / N, BW - 1), dx = lane < N * BW ? lane - bl * N : 0;         // (the last lane repeats a column)
    uint32_t c[B][2];
#pragma unroll
    for (int i = 0; i < B; ++i) {
        const uint2 v = *reinterpret_cast<const uint2 *>(cur32 + (B * wv + i) * PITCH4 + 2 * bl);
        c[i][0] = v.x; c[i][1] = v.y;
    }
    const int o = B * bl + dx;
    const uint32_t sh = (uint32_t)(o & 3);
    const uint32_t *base = win32 + B * wv * PITCH4 + (o >> 2);
    uint32_t acc[N], best = 0xffffffffu;
#pragma unroll
    for (int r = 0; r < B + 2 * R; ++r) {
        const uint32_t d0 = base[r * PITCH4], d1 = base[r * PITCH4 + 1], d2 = base[r * PITCH4 + 2];
        const uint32_t r0 = __builtin_amdgcn_alignbyte(d1, d0, sh), r1 = __builtin_amdgcn_alignbyte(d2, d1, sh);
#pragma unroll
        for (int dy = 0; dy < N; ++dy) {
            const int i = r - dy;
            if (i < 0 || i >= B) continue;
            acc[dy] = __builtin_amdgcn_sad_u8(c[i][0], r0, i == 0 ? 0u : acc[dy]);
            acc[dy] = __builtin_amdgcn_sad_u8(c[i][1], r1, acc[dy]);
        }
        if (r >= B - 1) best = min(best, (acc[r - B + 1] << KEY_SHIFT) | (uint32_t)((r - B + 1) * N));
    }
    best += (uint32_t)dx;
    // the lowest of a block's nine lanes, in its first one (what the others take from their neighbours is not used)
    auto down = [&](uint32_t v, int by) __attribute__((always_inline)) {
        return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (lane + by), (int)v);
    };
    const uint32_t ninth = down(best, 8);
#pragma unroll
    for (int k = 4; k >= 1; k >>= 1) best = min(best, down(best, k));
    best = min(best, ninth);
    const int by = by0 + wv, bx = bx0 + bl;
    if (dx != 0 || lane >= N * BW || by >= p.nby || bx >= p.nbx) return;
    const uint32_t blk = (uint32_t)by * p.nbx + bx, cidx = best & KEY_MASK;
    const int dyi = (int)(cidx / (uint32_t)N);
    sad[blk] = (int32_t)(best >> KEY_SHIFT);
    mv[2 * blk + 0] = dyi - R;
    mv[2 * blk + 1] = (int)cidx - dyi * N - R;
}

// ---------------------------------------------------------------------------
hipError_t launch_sad(const SadParams &p, const uint8_t *cur, const uint8_t *ref, int32_t *sad,
                      int32_t *mv, hipStream_t s)
{
    const uint32_t nblocks = (uint32_t)(p.nby * p.nbx);
    if (nblocks == 0) return hipSuccess;
    const int pitch4 = p.pitch >> 2;
    if (p.variant == SAD_ROWSCAN_B16) {
        const uint32_t grid = (uint32_t)(p.nby * p.groups_x);
        const auto k = p.R == 32 ? (p.bpw == 1 ? merit_sad_rowscan16<32, 1> : merit_sad_rowscan16<32, 4>)
                                 : (p.bpw == 1 ? merit_sad_rowscan16<16, 1> : merit_sad_rowscan16<16, 4>);
        hipLaunchKernelGGL(k, dim3(grid), dim3(p.bpw == 1 ? 256 : 512), sad_rowscan16_lds(p), s, p, cur, ref, sad, mv);
        return hipGetLastError();
    }
    if (p.variant == SAD_ROWSCAN_PAIR) {
        const uint32_t grid = (uint32_t)(p.nby * p.groups_x);
        const size_t lds_bytes = (size_t)((p.B + 2 * p.R) * pitch4 + 1) * 4;
        // (the instances for whole dwords gain 2 and 0.5 % on these two; on the others they lose 1 %)
        const bool any = (p.W & 3) != 0;
        void (*k)(SadParams, const uint8_t *, const uint8_t *, int32_t *, int32_t *) = nullptr;
        if (p.B == 8 && p.R == 16) k = any ? merit_sad_rowscan_pair<8, 16, true> : merit_sad_rowscan_pair<8, 16, false>;
        else if (p.B == 16 && p.R == 16) k = any ? merit_sad_rowscan_pair<16, 16, true> : merit_sad_rowscan_pair<16, 16, false>;
        else if (p.B == 8 && p.R == 8) k = merit_sad_rowscan_pair<8, 8, true>;
        else if (p.B == 16 && p.R == 8) k = merit_sad_rowscan_pair<16, 8, true>;
        else return hipErrorInvalidValue;
        hipLaunchKernelGGL(k, dim3(grid), dim3(256), lds_bytes, s, p, cur, ref, sad, mv);
        return hipGetLastError();
    }
    if (p.variant == SAD_ROWSCAN_SEVEN) {
        const uint32_t grid = (uint32_t)((p.nby + 3) / 4 * p.groups_x);
        hipLaunchKernelGGL(merit_sad_rowscan_seven, dim3(grid), dim3(256), 0, s, p, cur, ref, sad, mv);
        return hipGetLastError();
    }
    const size_t lds_bytes = (size_t)(p.win * pitch4 + 1 + p.B * (p.B >> 2) + 4) * 4;
    hipLaunchKernelGGL(merit_sad_generic, dim3(nblocks), dim3(256), lds_bytes, s, p, cur, ref, sad, mv);
    return hipGetLastError();
}

const char *sad_kernel_name(const SadParams &p)
{
    if (p.variant == SAD_ROWSCAN_B16) return p.R == 32 ? "merit_sad_rowscan16<32>" : "merit_sad_rowscan16<16>";
    if (p.variant == SAD_ROWSCAN_PAIR)
        return p.B == 16 ? (p.R == 16 ? "merit_sad_rowscan_pair<16,16>" : "merit_sad_rowscan_pair<16,8>") : (p.R == 16 ? "merit_sad_rowscan_pair<8,16>" : "merit_sad_rowscan_pair<8,8>");
    if (p.variant == SAD_ROWSCAN_SEVEN) return "merit_sad_rowscan_seven";
    return "merit_sad_generic";
}

}  // namespace merit
