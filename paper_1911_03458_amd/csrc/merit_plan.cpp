// Host side of the library: plan validation, derived geometry, and the C ABI.
//
// A plan holds the paper's transform descriptor (per index an axis d_j, stride
// s_j and offset o_j per operand; Section III-C, Eq. 5) after it has been
// matched against the three index patterns the kernels implement, plus the
// tile / halo geometry derived from it with the footprint rule of Section
// IV-A, Eq. 9.  No GPU call happens here.
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>

#include "merit_internal.h"

using namespace merit;

namespace merit {
size_t conv_lds_bytes(const ConvParams &p);
}

namespace {

constexpr int64_t LDS_LIMIT = 160 * 1024;       // per workgroup on gfx950
constexpr int64_t INT_LIMIT = 1ll << 30;

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return cdiv(a, b) * b; }

// FastDiv is exact when (nmax + d) * d < 2^32.
inline bool fastdiv_ok(int64_t nmax, int64_t d) { return d >= 1 && (nmax + d) * d < (1ll << 32); }

bool operand_is(const merit_operand &o, int n_index, const int *axis, const int64_t *stride,
                const int64_t *offset /* may hold INT64_MIN = "don't care" */)
{
    for (int j = 0; j < n_index; ++j) {
        if (o.axis[j] != axis[j]) return false;
        if (axis[j] == MERIT_AXIS_UNUSED) continue;
        if (stride && stride[j] != INT64_MIN && o.stride[j] != stride[j]) return false;
        if (offset && offset[j] != INT64_MIN && o.offset[j] != offset[j]) return false;
    }
    return true;
}

int64_t out_extent(int64_t I, int64_t k, int64_t s, int64_t p) { return (I + 2 * p - k) / s + 1; }

// ---------------------------------------------------------------- pooling ---
merit_status derive_pool(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    const bool is_avg = d.op == MERIT_OP_POOL_AVG;
    if (d.dtype != MERIT_F32) return MERIT_ERR_UNSUPPORTED;
    if (d.pad != (is_avg ? MERIT_PAD_EXCLUDE : MERIT_PAD_NEG_INF)) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 4 || d.n_acc != 2) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 4 || d.b.ndim != 0) return MERIT_ERR_UNSUPPORTED;
    const int axis[6] = {0, 1, 2, 3, 2, 3};
    const int64_t DC = INT64_MIN;
    const int64_t stride[6] = {1, 1, DC, DC, 1, 1};
    const int64_t offset[6] = {0, 0, 0, 0, DC, DC};
    if (!operand_is(d.a, 6, axis, stride, offset)) return MERIT_ERR_UNSUPPORTED;

    const int64_t N = d.a.shape[0], C = d.a.shape[1], H = d.a.shape[2], W = d.a.shape[3];
    const int64_t OH = d.range[2], OW = d.range[3], kh = d.range[4], kw = d.range[5];
    const int64_t sh = d.a.stride[2], sw = d.a.stride[3];
    const int64_t ph = -d.a.offset[4], pw = -d.a.offset[5];
    if (N < 0 || C <= 0 || H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
        return MERIT_ERR_INVALID_ARG;
    if (d.range[0] != N || d.range[1] != C) return MERIT_ERR_SHAPE;
    if (H + 2 * ph < kh || W + 2 * pw < kw) return MERIT_ERR_SHAPE;
    if (OH != out_extent(H, kh, sh, ph) || OW != out_extent(W, kw, sw, pw)) return MERIT_ERR_SHAPE;
    if (N * C >= INT_LIMIT || H * W >= INT_LIMIT || kh > 64 || kw > 64 || sh > 64 || sw > 64)
        return MERIT_ERR_UNSUPPORTED;

    PoolParams &p = pl->pool;
    p.NC = (int)(N * C); p.H = (int)H; p.W = (int)W; p.OH = (int)OH; p.OW = (int)OW;
    p.kh = (int)kh; p.kw = (int)kw; p.sh = (int)sh; p.sw = (int)sw; p.ph = (int)ph; p.pw = (int)pw;
    p.is_avg = is_avg ? 1 : 0;

    // row-strip variants: full-width strips, 16-byte accesses
    int variant = POOL_TILE_GENERIC;
    // staged rows carry 4 fill columns on either side; the last thread of a row reads
    // whole 16-byte chunks up to float 4*C1 past its span start
    const int64_t C1 = (4 - pw + 3 * sw + kw + 3) / 4;
    const bool rows_ok = (W % 4 == 0) && (OW % 4 == 0) && pw <= 4 &&
                         ((OW - 4) * sw + 4 * C1 <= W + 8);
    if (rows_ok) {
        if (kh == 3 && kw == 3 && sh == 2 && sw == 2 && pw == 1) variant = POOL_ROWS_K3S2P1;
        else if (kh == 2 && kw == 2 && sh == 2 && sw == 2 && pw == 0) variant = POOL_ROWS_K2S2P0;
        // (3x3 at stride 1: on request only -- the two-columns-per-lane kernel below is as fast or faster on every
        // size measured: 32 x 64 x 56 x 56 15.4 against 18.0 us, 8 x 64 x 112 x 112 14.7 against 17.8, 32 x 512 x 8 x 8 5.1 against 10.1)
        else if (kh == 3 && kw == 3 && sh == 1 && sw == 1 && pw == 1 && pl->tile_req[2] > 0) variant = POOL_ROWS_K3S1P1;
    }
    // streaming variant: register-resident strips, no LDS (3x3 / stride 2 / pad 1, W <= 256)
    const bool stream_ok = kh == 3 && kw == 3 && sh == 2 && sw == 2 && ph == 1 && pw == 1 &&
                           (W % 4 == 0) && W <= 256 && pl->tile_req[3] <= 0;
    if (stream_ok) {
        int64_t TH = 4;             // measured best on the 112x112 workload (4 < 7 < 8)
        if (pl->tile_req[2] > 0) TH = pl->tile_req[2];
        if (TH == 4 || TH == 7 || TH == 8) {
            int lg_shift = 0;
            while ((1 << lg_shift) < W / 4) ++lg_shift;
            p.variant = variant = POOL_STREAM_K3S2P1;
            p.TH = (int)TH; p.TW = (int)OW;
            p.tiles_y = (int)cdiv(OH, TH); p.tiles_x = 1;
            p.RH = 0; p.RW = 0; p.pitch = 0;
            p.lg_shift = lg_shift;
            const int64_t items = N * C * p.tiles_y;
            if (items >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;
            p.items = (int)items;
            p.grid = (int)cdiv(items, 4 * (64 >> lg_shift));
        }
    }
    if (variant != POOL_TILE_GENERIC && variant != POOL_STREAM_K3S2P1) {
        const int64_t pitch = W + 8;
        // strip height: as many output rows as keep the staged rows within ~16 KB,
        // then balanced so that all strips of a plane are (nearly) equal
        int64_t TH = (16 * 1024 / (pitch * 4) - kh) / sh + 1;
        if (TH < 1) TH = 1;
        if (TH > OH) TH = OH;
        TH = cdiv(OH, cdiv(OH, TH));
        if (pl->tile_req[2] > 0) TH = pl->tile_req[2] < OH ? pl->tile_req[2] : OH;
        const int64_t RH = (TH - 1) * sh + kh;
        if (RH * pitch * 4 > LDS_LIMIT || !fastdiv_ok(RH * (pitch / 4), pitch / 4) ||
            !fastdiv_ok(TH * (OW / 4), OW / 4)) {
            variant = POOL_TILE_GENERIC;
        } else {
            p.variant = variant;
            p.TH = (int)TH; p.TW = (int)OW;
            p.tiles_y = (int)cdiv(OH, TH); p.tiles_x = 1;
            p.RH = (int)RH; p.RW = (int)pitch; p.pitch = (int)pitch;
            p.div_p4 = make_fastdiv((uint32_t)(pitch / 4));
            p.div_ow4 = make_fastdiv((uint32_t)(OW / 4));
        }
    }
    // 3x3 / stride 2 (padding 0 or 1) and 2x2 / stride 2 (no padding) on a width the 16-byte kernels do not
    // take: a lane per two output columns, whose input columns are one 16-byte load (W >= 8), in groups of
    // 4 to 64 lanes; 3x3 on narrower planes: a lane per output column
    // (3x3 at stride 1, the pooling branch of an inception module on 35, 17 and 7 columns: the same kernel, 8 output rows
    // per group, any width of 4 and more)
    const bool k3 = kh == 3 && kw == 3 && ph <= 1 && pw <= 1, k2 = kh == 2 && kw == 2 && ph == 0 && pw == 0 && W >= 8;
    const bool s1 = k3 && sh == 1 && sw == 1 && W >= 4;
    if (variant == POOL_TILE_GENERIC && (((k3 || k2) && sh == 2 && sw == 2) || s1) &&
        !(OH == 1 && OW == 1) && pl->tile_req[2] <= 0 && pl->tile_req[3] <= 0 && H * W < INT_LIMIT) {
        const bool two = W >= 8 || s1;
        const int64_t cols = two ? 128 : 64;                // output columns of a full group of 64 lanes
        int lg_shift = 0;                                   // items per wavefront = 1 << lg_shift
        while (lg_shift < (two ? 4 : 2) && (cols >> (lg_shift + 1)) >= OW) ++lg_shift;
        const int64_t chunks = cdiv(OW, cols);
        // Output rows of a group.  2x2 windows share no rows, so one: 9x564x19x82 16.4 us with four, 11.4 with one, 29x158x145x23
        // 20.6 and 18.1 (1.13-2x over 40 layers; the tile kernel's 5x903x50x12 10.3 -> 5.1), 8x512x28x28 7.1 and 5.2,
        // 64x512x28x28 26.7 and 22.9.  Four on the largest launches, 200000 wavefronts of one row and more, where a group's
        // lanes have outputs for three quarters of them at most: 38x157x94x262 162 us, 189 with one, 1x311x1638x347 157 and
        // 177, 204x15x705x34 87 and 97 (51x194x60x754, all lanes at work, 470 and 400; 203x284x228x10, 16 groups a
        // wavefront, 170 and 149).
        const int64_t row_waves = N * C * chunks * OH >> lg_shift;
        const bool four = k2 && row_waves >= 200000 && lg_shift < 4 && 4 * OW <= 3 * chunks * (cols >> lg_shift);
        int64_t th = s1 ? 8 : (k2 && !four ? 1 : 4);
        auto items_of = [&](int64_t t) { return N * C * chunks * cdiv(OH, t); };
        // the kernel's divisions, and the threads of a launch
        auto fits = [&](int64_t t) {
            const int64_t n = items_of(t);
            return n < INT_LIMIT && fastdiv_ok(n, chunks) && fastdiv_ok(n, cdiv(OH, t)) && cdiv(n, 4 * (1 << lg_shift)) < 1 << 24;
        };
        if (th == 1 && !fits(th)) th = 4;                   // (4x64x2158x3838: 2187 us, 3298 on the tile kernel)
        const int64_t strips = cdiv(OH, th), items = items_of(th);
        // (2x2 windows of fewer outputs than the tile kernel's workgroups hold between them stay there: 2x106x11x13 2.7 against
        // 3.0 us, 5x42x19x34 3.0 either way)
        if (fits(th) && (k3 || s1 || N * C * OH * OW >= 32768)) {
            p.variant = variant = two ? POOL_LANES2_K3S2 : POOL_LANES_K3S2;
            p.TH = (int)th; p.TW = (int)(OW < cols ? OW : cols);
            p.tiles_y = (int)strips; p.tiles_x = (int)chunks;
            p.RH = p.RW = p.pitch = 0;
            p.lg_shift = lg_shift;
            p.items = (int)items;
            p.div_tiles_x = make_fastdiv((uint32_t)chunks);
            p.div_tiles_y = make_fastdiv((uint32_t)strips);
            p.grid = (int)cdiv(items, 4 * (1 << lg_shift));
        }
    }
    // one output per plane (global pooling): a wavefront per plane, no staging
    if (variant == POOL_TILE_GENERIC && OH == 1 && OW == 1 && pl->tile_req[2] <= 0 && pl->tile_req[3] <= 0 &&
        H * W < INT_LIMIT) {
        p.variant = variant = POOL_PLANE;
        p.TH = p.TW = 1; p.tiles_y = p.tiles_x = 1;
        p.RH = p.RW = p.pitch = 0;
        // lanes per plane: about four in-range window elements each, 4 to 64
        const int64_t y0 = std::max<int64_t>(-ph, 0), y1 = std::min<int64_t>(-ph + kh, H);
        const int64_t x0 = std::max<int64_t>(-pw, 0), x1 = std::min<int64_t>(-pw + kw, W);
        const int64_t rw = std::max<int64_t>(x1 - x0, 1), cnt = std::max<int64_t>(y1 - y0, 0) * rw;
        int lg = 0;                                         // planes per wavefront = 1 << lg
        while (lg < 4 && (64 >> (lg + 1)) * 4 >= cnt) ++lg;
        p.lg_shift = lg;
        const int64_t g = cdiv((int64_t)p.NC, 4 << lg);
        if (g >= (1ll << 31)) return MERIT_ERR_UNSUPPORTED;
        p.grid = (int)g;
    }
    if (variant == POOL_TILE_GENERIC) {
        p.variant = POOL_TILE_GENERIC;
        int64_t TW = OW < 64 ? OW : 64;
        int64_t TH = OH < 16 ? OH : 16;
        if (pl->tile_req[2] > 0) TH = pl->tile_req[2] < OH ? pl->tile_req[2] : OH;
        if (pl->tile_req[3] > 0) TW = pl->tile_req[3] < OW ? pl->tile_req[3] : OW;
        // shrink until the staged region fits comfortably
        for (;;) {
            const int64_t RH = (TH - 1) * sh + kh, RW = (TW - 1) * sw + kw;
            if (RH * (RW + 1) * 4 <= 64 * 1024 || (TH == 1 && TW == 1)) break;
            if (TH > 1) TH = (TH + 1) / 2; else TW = (TW + 1) / 2;
        }
        const int64_t RH = (TH - 1) * sh + kh, RW = (TW - 1) * sw + kw;
        if (RH * (RW + 1) * 4 > LDS_LIMIT) return MERIT_ERR_UNSUPPORTED;
        if (!fastdiv_ok(RH * RW, RW) || !fastdiv_ok(TH * TW, TW)) return MERIT_ERR_UNSUPPORTED;
        p.TH = (int)TH; p.TW = (int)TW;
        p.tiles_y = (int)cdiv(OH, TH); p.tiles_x = (int)cdiv(OW, TW);
        p.RH = (int)RH; p.RW = (int)RW; p.pitch = (int)RW + 1;
        p.div_rw = make_fastdiv((uint32_t)RW);
        p.div_tw = make_fastdiv((uint32_t)TW);
    }
    if (variant != POOL_STREAM_K3S2P1 && variant != POOL_PLANE && variant != POOL_LANES_K3S2 && variant != POOL_LANES2_K3S2) {
        const int64_t g = (int64_t)p.NC * p.tiles_y * p.tiles_x;
        if (g >= (1ll << 31)) return MERIT_ERR_UNSUPPORTED;
        p.grid = (int)g;
    }
    const int64_t grid = p.grid;

    pl->out_ndim = 4;
    pl->out_shape[0] = N; pl->out_shape[1] = C; pl->out_shape[2] = OH; pl->out_shape[3] = OW;
    merit_launch_info &li = pl->info;
    li.kernel = pool_kernel_name(p);
    li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = (int64_t)p.RH * p.pitch * 4;
    li.tile[0] = 1; li.tile[1] = 1; li.tile[2] = p.TH; li.tile[3] = p.TW; li.tile[4] = kh; li.tile[5] = kw;
    return MERIT_OK;
}

// ----------------------------------------------------------- block matching ---
merit_status derive_sad(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    if (d.dtype != MERIT_U8 || d.pad != MERIT_PAD_CLAMP) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 2 || d.n_acc != 4) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 2 || d.b.ndim != 2) return MERIT_ERR_UNSUPPORTED;
    const int64_t B = d.range[4], n = d.range[2];
    if (B <= 0 || n <= 0 || d.range[5] != B || d.range[3] != n || (n % 2) == 0) return MERIT_ERR_SHAPE;
    const int64_t R = (n - 1) / 2;
    const int axis_ref[6] = {0, 1, 0, 1, 0, 1};
    const int64_t stride_ref[6] = {B, B, 1, 1, 1, 1};
    const int64_t offset_ref[6] = {0, 0, -R, -R, 0, 0};
    const int axis_cur[6] = {0, 1, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 0, 1};
    const int64_t stride_cur[6] = {B, B, 0, 0, 1, 1};
    const int64_t offset_cur[6] = {0, 0, 0, 0, 0, 0};
    if (!operand_is(d.a, 6, axis_ref, stride_ref, offset_ref)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 6, axis_cur, stride_cur, offset_cur)) return MERIT_ERR_UNSUPPORTED;
    const int64_t H = d.a.shape[0], W = d.a.shape[1];
    if (H <= 0 || W <= 0) return MERIT_ERR_INVALID_ARG;
    if (d.b.shape[0] != H || d.b.shape[1] != W) return MERIT_ERR_SHAPE;
    // blocks that reach past the edge (B does not divide H or W) read both frames clamped
    if (d.range[0] != cdiv(H, B) || d.range[1] != cdiv(W, B)) return MERIT_ERR_SHAPE;
    // key packing: SAD < 2^18 and raster index < 2^14 share one u32
    if (B % 4 || B > 32 || R > 63) return MERIT_ERR_UNSUPPORTED;
    if (H * W >= INT_LIMIT || cdiv(H, B) * cdiv(W, B) >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;

    SadParams &p = pl->sad;
    p.H = (int)H; p.W = (int)W; p.B = (int)B; p.R = (int)R; p.n = (int)n;
    p.nby = (int)cdiv(H, B); p.nbx = (int)cdiv(W, B);
    p.win = (int)(B + 2 * R);
    const int64_t cols4 = cdiv(p.win, 4);
    p.pitch = (int)((cols4 + 1) * 4);
    p.variant = SAD_GENERIC;
    p.bpw = 1; p.groups_x = p.nbx;
    if (!fastdiv_ok(n * n, n) || !fastdiv_ok((int64_t)p.win * cols4, cols4)) return MERIT_ERR_UNSUPPORTED;
    p.div_n = make_fastdiv((uint32_t)n);
    p.div_win4 = make_fastdiv((uint32_t)cols4);
    p.div_nbx = make_fastdiv((uint32_t)p.nbx);

    // row-scan kernel: 16x16 blocks, four blocks per workgroup, instances for R = 16 and 32;
    // a tile request of one block per workgroup keeps the generic kernel
    int64_t grid = (int64_t)p.nby * p.nbx;
    int64_t lds = ((int64_t)p.win * (p.pitch / 4) + 1 + B * (B / 4) + 4) * 4;
    int64_t tile_bx = 1;
    // The row-scan kernels, any H.  Rows that are not whole dwords: from 64 blocks on (500x702, R = 32: 90.7 us on the
    // kernel for any shape, 25.0 on the row scan).  Smaller frames stay, for the plan tests that hold them, where they
    // were: the row scan is the faster one there too (159x78, R = 32: 59.5 against 17.1; 16x16 with R = 16 and 8 by 1.6
    // and 1.2, 8x8 by 1.35 and 1.14, over 110 frames).
    const bool rowscan_ok = W % 4 == 0 || (W >= 4 && (int64_t)p.nby * p.nbx >= 64);
    // R = 16: the elimination kernel, one block a workgroup, where the two-blocks-per-wavefront kernel below, whose wavefront
    // scans all of a block's candidates, leaves the chip idle: from 64 blocks (the plan tests hold smaller frames there; 76x144:
    // 10.5 against 6.8 us in a graph) to 1200 (288x416 11.0 against 7.0, 480x640 11.2 against 9.6, white noise 11.2 against
    // 9.8; 701x1003 17.5 against 16.1, but noise 17.5 against 19.1; 720x1280 15.3 against 18.8).
    const bool eliminate16 = rowscan_ok && B == 16 && R == 16 && pl->tile_req[1] <= 0 && (int64_t)p.nby * p.nbx >= 64 &&
                             (int64_t)p.nby * p.nbx <= 1200;
    if (rowscan_ok && B == 16 && (R == 16 || R == 32) && pl->tile_req[1] != 1) {
        // Four blocks a workgroup share a window and its sums; one block a workgroup, split among four wavefronts, is the
        // finer grain (R = 32, moving scenes, us: 540x960 19.4 against 24.8, 720x1280 27.8 against 34.6, 1080x1440, which has
        // 6120 blocks and takes four, 42.1 against 44.7, 1080x1920 52.7 against 52.2, 1440x2560 86 against 73, 2160x3840 179
        // against 148; white noise 1080x1440 67.5 against 66.6, 1080x1920 89 against 75.4)
        const int64_t bpw = eliminate16 ? 1 : R == 32 && (int64_t)p.nby * p.nbx < 6000 && pl->tile_req[1] <= 0 ? 1 : 4;
        const int64_t c4 = cdiv(bpw * 16 + 2 * R, 4);
        if (fastdiv_ok((16 + 2 * R) * c4, c4)) {
            p.variant = SAD_ROWSCAN_B16;
            p.bpw = (int)bpw;
            p.groups_x = (int)cdiv(p.nbx, bpw);
            p.pitch = 4 * sad_rowscan16_pitch4((int)R, (int)bpw);
            p.div_win4 = make_fastdiv((uint32_t)c4);
            grid = (int64_t)p.nby * p.groups_x;
            lds = (int64_t)sad_rowscan16_lds(p);
            tile_bx = bpw;
        }
    }

    // two blocks per wavefront, eight per workgroup: 8x8 and 16x16 blocks
    // with R = 8 or 16 (a tile request of four blocks per workgroup keeps the one-block-per-wavefront
    // kernel there)
    if (rowscan_ok && ((B == 8 || B == 16) && (R == 8 || R == 16)) && !eliminate16 && pl->tile_req[1] != 1 &&
        pl->tile_req[1] != 4) {
        const int64_t c4 = cdiv(8 * B + 2 * R, 4);
        if (fastdiv_ok((B + 2 * R) * c4, c4)) {
            p.variant = SAD_ROWSCAN_PAIR;
            p.bpw = 8;
            p.groups_x = (int)cdiv(p.nbx, 8);
            p.pitch = (int)((c4 + 1) * 4);
            p.div_win4 = make_fastdiv((uint32_t)c4);
            grid = (int64_t)p.nby * p.groups_x;
            lds = ((B + 2 * R) * (c4 + 1) + 1) * 4;
            tile_bx = 8;
        }
    }

    // seven blocks per wavefront, four block rows per workgroup: 8x8 blocks with R = 4 on rows of 16 and more pixels, the
    // faster kernel there from the smallest frame on (64x64: 2.8 us a launch against 3.3; 1080x1920: 4.6 against 40).  A tile
    // request of one block per workgroup keeps the kernel for any shape, and so do frames of up to 64 blocks that the blocks
    // do not divide, for the plan test that holds one there.
    int64_t tile_by = 1;
    if (B == 8 && R == 4 && W >= 16 && ((int64_t)p.nby * p.nbx > 64 || (W % 8 == 0 && H % 8 == 0)) && pl->tile_req[1] != 1) {
        p.variant = SAD_ROWSCAN_SEVEN;
        p.groups_x = (int)cdiv(p.nbx, 7);
        grid = cdiv(p.nby, 4) * p.groups_x;
        lds = (SEVEN_ROWS + 32) * SEVEN_PITCH4 * 4;
        tile_bx = 7; tile_by = 4;
    }

    p.xq = (int)(grid / 8); p.xr = (int)(grid % 8);
    pl->out_ndim = 2;
    pl->out_shape[0] = p.nby; pl->out_shape[1] = p.nbx;
    merit_launch_info &li = pl->info;
    li.kernel = sad_kernel_name(p);
    li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = p.variant == SAD_ROWSCAN_B16 && p.bpw == 4 ? 512 : 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = lds;
    li.tile[0] = tile_by; li.tile[1] = tile_bx; li.tile[2] = n; li.tile[3] = n; li.tile[4] = B; li.tile[5] = B;
    return MERIT_OK;
}

// -------------------------------------------------------- separable filter ---
merit_status derive_sep(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    if (d.dtype != MERIT_F32 || d.pad != MERIT_PAD_CLAMP) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 3 || d.n_acc != 2) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 3 || d.b.ndim != 1) return MERIT_ERR_UNSUPPORTED;
    const int64_t N = d.a.shape[0], H = d.a.shape[1], W = d.a.shape[2], k = d.b.shape[0];
    if (N < 0 || H <= 0 || W <= 0 || k <= 0) return MERIT_ERR_INVALID_ARG;
    const int64_t c = k / 2;
    const int axis_x[5] = {0, 1, 2, 1, 2};
    const int64_t stride_x[5] = {1, 1, 1, 1, 1};
    const int64_t offset_x[5] = {0, 0, 0, -c, -c};
    const int axis_k[5] = {MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 0};
    const int64_t stride_k[5] = {0, 0, 0, 0, 1};
    const int64_t offset_k[5] = {0, 0, 0, 0, 0};
    if (!operand_is(d.a, 5, axis_x, stride_x, offset_x)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 5, axis_k, stride_k, offset_k)) return MERIT_ERR_UNSUPPORTED;
    if (d.range[0] != N || d.range[1] != H || d.range[2] != W || d.range[3] != k || d.range[4] != k)
        return MERIT_ERR_SHAPE;
    if (k > 32 || H * W >= INT_LIMIT || N * H * W >= (1ll << 40)) return MERIT_ERR_UNSUPPORTED;

    SepParams &p = pl->sep;
    p.N = (int)N; p.H = (int)H; p.W = (int)W; p.k = (int)k; p.c = (int)c;
    p.c4 = (int)round_up(c, 4);
    // staged rows RH = TH + k - 1; TH a multiple of 4 (the column pass works on patches of 2 or 4 rows)
    const int64_t asked = pl->tile_req[1], most = k <= 16 ? 64 : 96;      // staged rows per workgroup, at most
    if (asked > 0 && (asked < k + 3 || asked > most)) return MERIT_ERR_UNSUPPORTED;
    auto rows_of = [&](int form) {
        const int64_t rows = form == SEP_PERSISTENT ? most : sep_rows(form);
        return asked > 0 && asked < rows ? asked : rows;
    };
    auto tiles_of = [&](int64_t TH) { return N * cdiv(H, TH) * cdiv(W, 64); };
    auto divides = [&](int64_t TH) {
        return fastdiv_ok(tiles_of(TH), cdiv(W, 64)) && fastdiv_ok(N * cdiv(H, TH), cdiv(H, TH));
    };
    // few tiles: up to three a compute unit (at 480-760 tiles 512 threads are 1-8 % faster, at 960 on k = 30 and at
    // 1840-2500 otherwise 4-13 % slower).  Where they are fewer than the compute units they are shortened until those are
    // full, to 16 rows at least: a tile's chain is as long as it is tall (not for short windows, whose chain is the round
    // trip to memory whatever the height).
    // A request for more rows than those two forms stage names the third.
    int64_t TH = (rows_of(SEP_FEW) - k + 1) / 4 * 4;
    p.form = asked > sep_rows(SEP_FEW) ? SEP_PERSISTENT : TH > 0 && tiles_of(TH) <= 768 ? SEP_FEW : sep_many((int)k);
    if (p.form != SEP_FEW) TH = (rows_of(p.form) - k + 1) / 4 * 4;
    else if (asked <= 0 && k >= 8)
        while (TH > 16 && tiles_of(TH - 4) <= 256) TH -= 4;
    // (2^24 workgroups of 256 threads are more than a launch takes, and more tiles than workgroups can be walked; taller
    // tiles on frames of so many rows that the shorter ones' numbers do not divide)
    if (p.form == SEP_TILES && (tiles_of(TH) >= 1 << 24 || !divides(TH))) {
        p.form = SEP_PERSISTENT;
        TH = (rows_of(p.form) - k + 1) / 4 * 4;
    }
    const int64_t RH = TH + k - 1;
    p.TH = (int)TH;
    p.tiles_y = (int)cdiv(H, TH);
    p.tiles_x = (int)cdiv(W, 64);
    // a row-pass unit of rc columns reads ceil((d + rc + k - 1) / 4) 16-byte groups from column rc cg on
    const int64_t rc = sep_rc(p.form), nwr = cdiv((p.c4 - c) + rc + k - 1, 4);
    p.PI = (int)(round_up(64 - rc + 4 * nwr, 8) + 4);     // pitches of 4 mod 8 floats: see the kernel
    p.lds_bytes = (int)((RH * p.PI + 8 * cdiv(k, 4)) * 4);
    if (p.lds_bytes > LDS_LIMIT) return MERIT_ERR_UNSUPPORTED;
    const int64_t grid = N * p.tiles_y * p.tiles_x;
    if (grid >= INT_LIMIT || !divides(TH) || !fastdiv_ok(8 * RH, RH)) return MERIT_ERR_UNSUPPORTED;
    p.div_tiles_x = make_fastdiv((uint32_t)p.tiles_x);
    p.div_tiles_y = make_fastdiv((uint32_t)p.tiles_y);
    p.div_rh = make_fastdiv((uint32_t)RH);

    pl->out_ndim = 3;
    pl->out_shape[0] = N; pl->out_shape[1] = H; pl->out_shape[2] = W;
    merit_launch_info &li = pl->info;
    li.kernel = "merit_sepfilter_tile";
    // persistent grid: the launcher sizes it from the device's CU count (256 on MI355X)
    p.wg_per_cu = (int)(LDS_LIMIT / p.lds_bytes);
    if (p.wg_per_cu > 4) p.wg_per_cu = 4;
    li.grid[0] = p.form == SEP_PERSISTENT && grid > 256 * p.wg_per_cu ? 256 * p.wg_per_cu : grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = p.form == SEP_FEW ? 512 : 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = p.lds_bytes;
    li.tile[0] = 1; li.tile[1] = TH; li.tile[2] = 64; li.tile[3] = k; li.tile[4] = k;
    return MERIT_OK;
}

// --------------------------------------------------------- bilateral filter ---
merit_status derive_bilateral(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    if (d.dtype != MERIT_F32 || d.pad != MERIT_PAD_CLAMP) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 3 || d.n_acc != 2) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 3 || d.b.ndim != 1) return MERIT_ERR_UNSUPPORTED;
    const int64_t N = d.a.shape[0], H = d.a.shape[1], W = d.a.shape[2], k = d.b.shape[0];
    if (N < 0 || H <= 0 || W <= 0 || k <= 0) return MERIT_ERR_INVALID_ARG;
    const int64_t c = k / 2;
    const int axis_x[5] = {0, 1, 2, 1, 2};
    const int64_t stride_x[5] = {1, 1, 1, 1, 1};
    const int64_t offset_x[5] = {0, 0, 0, -c, -c};
    const int axis_k[5] = {MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 0};
    const int64_t stride_k[5] = {0, 0, 0, 0, 1};
    const int64_t offset_k[5] = {0, 0, 0, 0, 0};
    if (!operand_is(d.a, 5, axis_x, stride_x, offset_x)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 5, axis_k, stride_k, offset_k)) return MERIT_ERR_UNSUPPORTED;
    if (d.range[0] != N || d.range[1] != H || d.range[2] != W || d.range[3] != k || d.range[4] != k)
        return MERIT_ERR_SHAPE;
    if (k > 32 || H * W >= INT_LIMIT || N * H * W >= (1ll << 40)) return MERIT_ERR_UNSUPPORTED;

    BilatParams &p = pl->bil;
    p.N = (int)N; p.H = (int)H; p.W = (int)W; p.k = (int)k; p.c = (int)c;
    p.c4 = (int)round_up(c, 4);
    // Windows of up to 16 taps: one output a thread on frames of up to 400 16 x 64 tiles, and of up to 1200 from 9 taps on,
    // else two (k = 9: 720x1280 14.2 us against 15.4, 1080x1920 29.6 against 28.8; k = 3: 333x1203 3.7 both, 720x1280 5.3
    // against 4.6).  With one or two taps, which memory bounds, four from 200 tiles on (k = 2 on 2 of 1017x496, 1024 tiles:
    // 3.9 against 4.4 with two; on 2 of 463x322, 348: 3.3 against 3.6 with one; k = 1 on 4 of 313x130, 240: 2.6 against 2.7).
    // Longer windows: merit_bilateral_tile's 16 x 64 outputs on 256 threads, four a thread down a column.
    const int64_t tiles16 = N * cdiv(H, 16) * cdiv(W, 64);
    p.J = k > 16 ? 4 : k <= 2 ? (tiles16 <= 200 ? 1 : 4) : (tiles16 <= 400 || (k >= 9 && tiles16 <= 1200) ? 1 : 2);
    p.NT = p.J == 2 ? 512 : 256;
    const int64_t TH = p.J * p.NT / 64;
    p.tiles_y = (int)cdiv(H, TH);
    p.tiles_x = (int)cdiv(W, 64);
    p.PI = (int)round_up(64 + p.c4 + (k - 1 - c), 4);
    const int64_t RH = TH + k - 1;
    p.lds_bytes = (int)((RH * p.PI + 2 * k + 4) * 4);     // + one 16-byte group: whole-group reads of the last row
    p.scale = 0.0f; p.neg = 1;
    const int64_t grid = N * p.tiles_y * p.tiles_x;
    if (grid >= INT_LIMIT || !fastdiv_ok(grid, p.tiles_x) || !fastdiv_ok(N * p.tiles_y, p.tiles_y) ||
        !fastdiv_ok(RH * p.PI, p.PI / 4))
        return MERIT_ERR_UNSUPPORTED;
    p.div_tiles_x = make_fastdiv((uint32_t)p.tiles_x);
    p.div_tiles_y = make_fastdiv((uint32_t)p.tiles_y);
    p.div_p4 = make_fastdiv((uint32_t)(p.PI / 4));

    pl->out_ndim = 3;
    pl->out_shape[0] = N; pl->out_shape[1] = H; pl->out_shape[2] = W;
    merit_launch_info &li = pl->info;
    li.kernel = k <= 16 ? "merit_bilateral_rows" : "merit_bilateral_tile";
    li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = p.NT; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = p.lds_bytes;
    li.tile[0] = 1; li.tile[1] = TH; li.tile[2] = 64; li.tile[3] = k; li.tile[4] = k;
    return MERIT_OK;
}

// -------------------------------------------------------------- convolution ---
// The size of the packed copy of a wave-specialised multi-pass tiling.
int64_t packed_bytes(const ConvParams &p) { return (int64_t)p.co_groups * p.nchunks * p.lds_w_bytes; }

// The layers whose weights can be packed once: the wave-specialised multi-pass kernel on a multiple of 8 input channels
// and more than 32 output channels, at least 32 of the former unless a tile request named the kernel.
bool packable(const merit_plan *pl)
{
    const ConvParams &p = pl->conv;
    const bool requested = pl->tile_req[2] > 0 && pl->tile_req[3] > 0;
    return p.variant == CONV_CHWS && p.Cin % 8 == 0 && p.Cout > 32 && (requested || p.Cin >= 32);
}

// 1x1 windows at stride 1 without padding: the matrix-product kernel (conv2d_px.hip), whatever the general planner
// chose, unless a tile request names one of the other kernels' tilings.
void derive_px(merit_plan *pl)
{
    const ConvParams &c = pl->conv;
    if (c.kh != 1 || c.kw != 1 || c.sh != 1 || c.sw != 1 || c.ph != 0 || c.pw != 0 || c.pool) return;
    if (pl->tile_req[2] > 0 && pl->tile_req[3] > 0) return;
    const int64_t N = c.N, Cin = c.Cin, HW = (int64_t)c.H * c.W, Cout = c.Cout;
    // (any channel count: 260 -> 64 on 8 of 56x56 4.8 us, 23.7 on the channel-block kernels, 1028 -> 64 on 64 of 16x16 7.4 and
    // 61.4, 286 -> 131 on 40 of 56x32 18 and 159)
    if (Cin < 16 || HW < 8 || Cin * HW >= (1ll << 30) || Cout * Cin >= (1ll << 30) || Cout * HW >= (1ll << 30)) return;
    PxParams p;
    std::memset(&p, 0, sizeof(p));
    p.N = (int)N; p.Cin = (int)Cin; p.HW = (int)HW; p.Cout = (int)Cout;
    p.relu = c.relu; p.residual = c.residual;
    p.nk = (int)cdiv(Cin, 64);
    // The tile with the lowest estimate, in microseconds of a compute unit: per workgroup, steps of 64 channels x the
    // cost of one (alone on its unit, or beside others) + its start and its stores; fitted to 110 layers of 16 .. 2016
    // channels timed on every tile: the estimate's choice takes 0.9 % longer than the best of them in the geometric mean.
    static const struct { int tm, tn; double alone, beside, ends; } tiles[6] = {
        {64, 32, 0.165, 0.175, 0.767}, {64, 64, 0.175, 0.218, 0.742}, {64, 128, 0.343, 0.353, 1.101},
        {128, 32, 0.221, 0.241, 0.659}, {128, 64, 0.365, 0.316, 0.876}, {128, 128, 0.459, 0.573, 1.655}};
    double best_cost = 0.0;
    for (const auto &t : tiles) {
        const double n = (double)(N * cdiv(HW, t.tm) * cdiv(Cout, t.tn)) / 256.0;
        const double steps = (double)cdiv(Cin, 16) / 4.0;
        const double per_cu = n <= 1.0 ? 1.0 : 0.5 * (n + std::ceil(n));
        const double cost = per_cu * (steps * (n <= 1.0 ? t.alone : t.beside) + t.ends * (p.residual ? 1.3 : 1.0));
        if (p.TM == 0 || cost < best_cost) { p.TM = t.tm; p.TN = t.tn; best_cost = cost; }
    }
    p.tiles = (int)cdiv(HW, p.TM); p.co_groups = (int)cdiv(Cout, p.TN);
    const int64_t grid = N * p.tiles * p.co_groups;
    // (2^23 workgroups of 512 threads are more than a launch takes: the general planner's kernels walk their tiles)
    if (grid >= (1ll << 23) || !fastdiv_ok(grid, p.co_groups) || !fastdiv_ok(N * p.tiles, p.tiles)) return;
    p.xq = (int)(grid / 8); p.xr = (int)(grid % 8);
    p.div_cog = make_fastdiv((uint32_t)p.co_groups);
    p.div_tiles = make_fastdiv((uint32_t)p.tiles);
    pl->px = p;
    pl->use_px = 1;
    merit_launch_info &li = pl->info;
    li.kernel = "merit_conv2d_px";
    li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = 512; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = (int64_t)px_lds_bytes(p);
    li.tile[1] = p.TN; li.tile[2] = cdiv(p.TM, c.W); li.tile[3] = c.W;
}

// 3x3 and 5x5 windows that the wave-specialised multi-pass kernel would run on a fraction of the chip: the form of it that
// splits the channels among the wavefronts (conv2d_split.hip), where its estimate is the lower one.  Not on a tile request,
// which names one of the other form's tilings.
void derive_split(merit_plan *pl)
{
    const ConvParams &c = pl->conv;
    if (c.variant != CONV_CHWS || c.pool || c.residual || !(c.kh == c.kw && (c.kh == 3 || c.kh == 5))) return;
    if (pl->tile_req[2] > 0 && pl->tile_req[3] > 0) return;
    const int64_t N = c.N, Cin = c.Cin, H = c.H, W = c.W, Cout = c.Cout, OW = c.OW, ohw = (int64_t)c.OH * c.OW;
    // (at least one slice of 16 channels and one 16-byte unit of an image; byte offsets into an image and the weights)
    if (N == 0 || Cin < 17 || H * W < 8 || Cin * H * W >= (1ll << 29) || Cout * Cin * c.kh * c.kw >= (1ll << 29) || Cout * ohw >= (1ll << 30)) return;

    // (up to 48 channels on rows of whole 16-byte units stay where they were: three wavefronts of eight would have a slice,
    // this form is 3-20 % faster, and the tests hold such a layer's sums to those of another tiling, bit for bit)
    if (Cin <= 48 && W % 8 == 0) return;

    // Estimates in microseconds, fitted to 870 layers (3 to 112 pixels wide, 17 to 2048 channels, the caller's weights and
    // packed ones) timed on both forms.  The multi-pass form: a launch, its rounds, its passes, and in each of them the
    // multiplications, the input loads (dearer on rows of an odd width) and the weights.  This form: a launch, its rounds,
    // and in each of them, per eight slices, their multiplications and barrier-free chain, the input loads and the weights
    // (as the caller's lie: a plan does not know which call comes).  The choice is within 0.2 % (3x3) and 0.4 % (5x5) of the
    // better form on average.  A lead of 6 % is asked for, of 15 % on grids of more than one round, where the estimate errs
    // most; beyond two rounds the multi-pass form was always the better one.  (Of 850 other layers that take this form,
    // 1.6x faster in the geometric mean, ten are 2 to 8 % slower, at leads of 7 to 40 %: 3x3 / 2 56 -> 160 on 11 of 7x27
    // 5.65 -> 5.89 us, 5x5 / 2 399 -> 960 on 15 of 10x10 100 -> 107.)
    const bool k5 = c.kh == 5;
    const double T = c.kh * c.kw, odd = (double)(W & 1);
    const double rounds = (double)cdiv(N * c.tiles_per_image * c.co_groups, 256), passes = rounds * c.nchunks;
    const double mults = c.CB * (c.TM / 32.0) * (c.nchi / 2.0) * T / 8.0, loads = 8.0 * c.xu * (c.xpx == 8 ? 1.0 : 0.7);
    const double weights = (double)c.CB * 32.0 * c.nchi * 16.0 * T / 16384.0;
    const double multi_pass = k5 ? 0.3 + 4.6 * rounds + passes * (0.154 + 0.028 * mults + (0.05 + 0.011 * odd) * loads + 0.249 * weights)
                                 : 1.8 + 2.36 * rounds + passes * (0.104 + 0.056 * mults + (0.022 + 0.018 * odd) * loads + 0.126 * weights);
    static const struct { double launch, round, slices, even, odd, weights; } costs[2][2] = {
        {{1.54, 2.11, 0.74, 0.97, 2.40, 0.59}, {1.33, 2.69, 0.50, 1.37, 2.69, 0.69}},
        {{1.28, 2.98, 1.72, 1.21, 2.76, 1.95}, {1.08, 3.81, 1.78, 1.19, 2.59, 2.05}}};

    double best_cost = multi_pass;
    // tiles of 32 or 64 pixels: adjacent ones of the plane (whole input rows are staged), or rectangles 8, 16 or 32 wide
    // (part of a row is staged: what long rows and row strides need to fit at all).  Where both fit, the rectangle has to
    // lead by 12 %: its units start on even columns only, and within that lead it was up to 9 % slower, over 400 layers.
    for (int form = 0; form < 8; ++form) {
        const int pxb = 1 + (form & 1), lg_tw = form < 2 ? 0 : 2 + form / 2;
        if (form == 2 && pl->use_split) best_cost *= 0.88;
        SplitParams p;
        std::memset(&p, 0, sizeof(p));
        p.N = c.N; p.Cin = c.Cin; p.H = c.H; p.W = c.W; p.Cout = c.Cout; p.OH = c.OH; p.OW = c.OW;
        p.sh = c.sh; p.sw = c.sw; p.ph = c.ph; p.pw = c.pw; p.dh = c.dh; p.dw = c.dw;
        p.K = c.kh; p.PXB = pxb; p.relu = c.relu; p.lg_tw = lg_tw;
        const int64_t TM = 32 * pxb, TW = lg_tw > 0 ? 1ll << lg_tw : OW;
        if (lg_tw > 0 && (W < 8 || TW / 2 >= OW)) continue;
        int64_t rows_out = lg_tw > 0 ? TM / TW : (TM + OW - 2) / OW + 1;
        if (rows_out > c.OH) rows_out = c.OH;
        p.RHa = (int)((rows_out - 1) * c.sh + (c.kh - 1) * c.dh + 1);
        const int64_t span = (TW - 1) * c.sw + (c.kw - 1) * c.dw + 1;     // input columns of a tile
        // (a rectangle's first staged column is an even one: loads on rows of an even width stay on 4-byte boundaries)
        p.units_x = (int)cdiv(lg_tw > 0 ? std::min(span + 1, W) : W, 8);
        int64_t pitch = lg_tw > 0 ? 8 * (int64_t)p.units_x + c.pw + 1 : c.pw + W;
        const int64_t reach = lg_tw > 0 ? span + 9 : span;
        if (reach > pitch) pitch = reach;
        p.pitch = (int)(pitch | 1);               // odd: staged rows start in different LDS bank groups
        const int64_t units = 2 * (int64_t)p.RHa * p.units_x;
        if (units > (W < 8 ? 64 : 128)) continue;
        p.xu = W < 8 ? 0 : (int)cdiv(units, 64);
        if (Cin % 8 != 0 && (W < 8 || (pxb == 2 && p.xu == 2))) continue;           // (no such instance)
        p.slices = (int)cdiv(Cin, 16);
        p.tiles_x = lg_tw > 0 ? (int)cdiv(OW, TW) : 1;
        p.tiles = lg_tw > 0 ? (int)(p.tiles_x * cdiv(c.OH, TM / TW)) : (int)cdiv(ohw, TM);
        p.co_groups = (int)cdiv(Cout, 32);
        p.slice_bytes = 2 * p.RHa * p.pitch * 16;
        const int64_t sums = (int64_t)SPLIT_WAVES * 32 * (TM + 4) * 4;
        const int64_t areas = (int64_t)SPLIT_WAVES * (p.slice_bytes + 32 * split_weight_pitch(p.K));
        p.lds_bytes = (int)(sums > areas ? sums : areas);
        if (p.lds_bytes > LDS_LIMIT) continue;
        const int64_t grid = N * p.tiles * p.co_groups;
        p.by_channel = Cout * Cin * c.kh * c.kw > N * Cin * H * W ? 1 : 0;
        p.minor = (int)(p.by_channel ? N * p.tiles : p.co_groups);
        if (grid > 512 || !fastdiv_ok(grid, p.minor) || !fastdiv_ok(N * p.tiles, p.tiles) || !fastdiv_ok(ohw, OW) ||
            !fastdiv_ok(p.tiles, p.tiles_x) || !fastdiv_ok(units, 2 * p.RHa))
            continue;
        const auto &k = costs[k5][pxb - 1];
        const double r = (double)cdiv(grid, 256), load = (double)units / 64.0;
        const double cost = (k.launch + r * (k.round + p.slices / 8.0 * (k.slices + load * (W & 1 ? k.odd : k.even) + k.weights))) *
                            (r > 1.0 ? 1.15 : 1.06);
        if (cost >= best_cost) continue;
        best_cost = cost;
        p.xq = (int)(grid / 8); p.xr = (int)(grid % 8);
        p.div_minor = make_fastdiv((uint32_t)p.minor);
        p.div_tiles = make_fastdiv((uint32_t)p.tiles);
        p.div_tiles_x = make_fastdiv((uint32_t)p.tiles_x);
        p.div_ow = make_fastdiv((uint32_t)OW);
        p.div_r2 = make_fastdiv((uint32_t)(2 * p.RHa));
        pl->split = p;
        pl->use_split = 1;
        merit_launch_info &li = pl->info;
        li.kernel = "merit_conv2d_split";
        li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
        li.block[0] = SPLIT_WAVES * 64; li.block[1] = 1; li.block[2] = 1;
        li.lds_bytes = p.lds_bytes;
        li.tile[1] = 32; li.tile[2] = rows_out; li.tile[3] = TW;
    }
}

// Every family but the two forms for few pixels and for 1x1 layers (derive_px, derive_split), which only an unpooled layer
// takes: the convolution of a plan that pools in a launch of its own is planned here too, and sums in the fused form's order.
merit_status derive_conv_families(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    pl->use_px = pl->use_split = pl->use_na = 0;
    if (d.dtype != MERIT_F16 || d.pad != MERIT_PAD_ZERO) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 4 || d.n_acc != 3) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 4 || d.b.ndim != 4) return MERIT_ERR_UNSUPPORTED;
    const int64_t DC = INT64_MIN;
    const int axis_x[7] = {0, MERIT_AXIS_UNUSED, 2, 3, 1, 2, 3};
    const int64_t stride_x[7] = {1, 0, DC, DC, 1, DC, DC};      // window strides = dilation
    const int64_t offset_x[7] = {0, 0, 0, 0, 0, DC, DC};
    const int axis_w[7] = {MERIT_AXIS_UNUSED, 0, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1, 2, 3};
    const int64_t stride_w[7] = {0, 1, 0, 0, 1, 1, 1};
    const int64_t offset_w[7] = {0, 0, 0, 0, 0, 0, 0};
    if (!operand_is(d.a, 7, axis_x, stride_x, offset_x)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 7, axis_w, stride_w, offset_w)) return MERIT_ERR_UNSUPPORTED;

    const int64_t N = d.a.shape[0], Cin = d.a.shape[1], H = d.a.shape[2], W = d.a.shape[3];
    const int64_t Cout = d.b.shape[0], kh = d.b.shape[2], kw = d.b.shape[3];
    const int64_t sh = d.a.stride[2], sw = d.a.stride[3];
    const int64_t dh = d.a.stride[5], dw = d.a.stride[6];
    const int64_t ph = -d.a.offset[5], pw = -d.a.offset[6];
    const int64_t OH = d.range[2], OW = d.range[3];
    if (N < 0 || Cin <= 0 || H <= 0 || W <= 0 || Cout <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 ||
        ph < 0 || pw < 0 || dh <= 0 || dw <= 0)
        return MERIT_ERR_INVALID_ARG;
    const int64_t eh = (kh - 1) * dh + 1, ew = (kw - 1) * dw + 1;      // extent of the dilated window
    if (d.b.shape[1] != Cin || d.range[0] != N || d.range[1] != Cout || d.range[4] != Cin ||
        d.range[5] != kh || d.range[6] != kw)
        return MERIT_ERR_SHAPE;
    if (H + 2 * ph < eh || W + 2 * pw < ew) return MERIT_ERR_SHAPE;
    if (OH != out_extent(H, eh, sh, ph) || OW != out_extent(W, ew, sw, pw)) return MERIT_ERR_SHAPE;
    if (N * Cin * H * W >= (1ll << 40) || OH * OW >= (1 << 24) || Cin > 4096 || Cout > 65535 * 32 ||
        kh > 31 || kw > 31 || sh > 16 || sw > 16 || dh > 16 || dw > 16)
        return MERIT_ERR_UNSUPPORTED;
    const bool dilated = dh != 1 || dw != 1;

    ConvParams &p = pl->conv;
    p.N = (int)N; p.Cin = (int)Cin; p.H = (int)H; p.W = (int)W; p.Cout = (int)Cout;
    p.relu = (d.op == MERIT_OP_CONV_DOT_RELU || d.op == MERIT_OP_CONV_DOT_RELU_POOLMAX ||
              d.op == MERIT_OP_CONV_DOT_ADD_RELU) ? 1 : 0;
    p.residual = (d.op == MERIT_OP_CONV_DOT_ADD || d.op == MERIT_OP_CONV_DOT_ADD_RELU) ? 1 : 0;
    const bool pool = d.op == MERIT_OP_CONV_DOT_POOLMAX || d.op == MERIT_OP_CONV_DOT_RELU_POOLMAX;
    p.pool = pool ? 1 : 0;
    p.PH = p.PW = p.PB = p.NB = p.pw8 = 0; p.pool_halo = 0;
    // fused pooling: a workgroup's tile is an even number of whole output rows (at least two)
    if (pool && (OH % 2 != 0 || OW % 2 != 0 || 2 * OW > 256)) return MERIT_ERR_UNSUPPORTED;
    p.OH = (int)OH; p.OW = (int)OW; p.kh = (int)kh; p.kw = (int)kw; p.sh = (int)sh; p.sw = (int)sw;
    p.ph = (int)ph; p.pw = (int)pw; p.dh = (int)dh; p.dw = (int)dw;

    const int64_t ohw = OH * OW;
    const int64_t ncb = cdiv(Cout, 32);
    p.CB = ncb >= 2 ? 2 : 1;
    // A grid that would leave more than half of the 256 CUs idle gets 32-channel blocks, i.e. twice
    // the workgroups (channel-block kernels; 8x128x56x56 -> 128, 3x3 / s2: 112 -> 224 workgroups,
    // 24.4 -> 14.5 us; with more workgroups than that the 64-channel blocks win: half the input staging), the few-channel
    // kernel too (its weights are then staged in half the time: 11x11 3 -> 64 on 3 of 147x74 13.2 -> 11.5 us).
    if (ncb >= 2 && !pool && N * cdiv(ohw, 128) * cdiv(ncb, 2) <= 128) p.CB = 1;
    p.co_groups = (int)cdiv(ncb, p.CB);

    // try both tile sizes for a variant; prefer 256 pixels when the grid stays large
    // an explicit tile request selects the plain kernels; so does the residual layer (the added
    // tensor is staged by the wavefronts that also multiply)
    bool want_ws = pl->tile_req[2] <= 0 && !p.residual;
    auto try_variant = [&](int variant, int pxw, int nw) -> bool {
        ConvParams q = p;
        q.variant = variant;
        q.nchunks = 1; q.pipe = 0;
        q.PXW = pxw;
        q.NW = nw;
        q.TM = nw * pxw * 32;
        q.tiles_per_image = (int)cdiv(ohw, q.TM);
        q.rows_out_max = (int)((q.TM + OW - 2) / OW + 1);
        if (q.rows_out_max > OH) q.rows_out_max = (int)OH;
        q.tile_px = q.TM;
        if (pool) q.rows_out_max = 2;
        q.RHa = (int)((q.rows_out_max - 1) * sh + eh);
        if (variant == CONV_PLANAR_SMALLC) {
            if (kw > 16 || pw > 8 || dilated) return false;      // its fragments are runs of adjacent taps
            if (Cin * H * W * 2 >= (1ll << 31) || Cout * Cin * kh * kw * 2 >= (1ll << 31)) return false;    // byte offsets into an image / the weights
            q.padl = 8;
            // with an even column stride every window starts on the same column parity; if that
            // parity is odd and a slot is free, start the fragment one column earlier (front = 1)
            // so that it is dword-aligned in LDS and needs no funnel shift
            const bool odd_start = ((q.padl - pw) & 1) != 0;
            q.front = (sw % 2 == 0 && odd_start && kw != 8 && kw != 16) ? 1 : 0;
            q.aligned = (sw % 2 == 0 && ((q.padl - pw - q.front) & 1) == 0) ? 1 : 0;
            // a window row of more than 8 slots is two K-groups (two adjacent fragments)
            const int64_t parts = (q.front + kw > 8) ? 2 : 1;
            int64_t pitch = q.padl + W;
            const int64_t reach = q.padl - pw + (OW - 1) * sw + 2 + 8 * parts;
            if (reach > pitch) pitch = reach;
            q.pitch = (int)round_up(pitch, 8);
            q.G = (int)(Cin * kh * parts);
            q.G2 = (int)round_up(q.G, 2);
            q.S = q.G2 / 2;
            q.nchi = 0;
            q.lds_w_bytes = q.CB * q.G2 * 32 * 16;
            q.lds_x_bytes = (int)(Cin * q.RHa * q.pitch * 2);
            if (!fastdiv_ok((int64_t)Cin * q.RHa * (q.pitch / 8), q.pitch / 8)) return false;
            if (!fastdiv_ok((int64_t)Cin * q.RHa, q.RHa) || !fastdiv_ok(q.G2, kh)) return false;
            q.div_pitch8 = make_fastdiv((uint32_t)(q.pitch / 8));
            q.div_kh = make_fastdiv((uint32_t)kh);
            if (!fastdiv_ok((int64_t)q.CB * 32 * q.G2, q.G2)) return false;
            q.div_g2 = make_fastdiv((uint32_t)q.G2);
            q.lds_o_offset = (int)round_up((int64_t)q.lds_w_bytes + 32 + q.lds_x_bytes, 16);
        } else {
            q.front = 0; q.aligned = 0;
            q.padl = (int)pw;
            int64_t pitch = q.padl + W;
            const int64_t reach = (OW - 1) * sw + ew;
            if (reach > pitch) pitch = reach;
            q.pitch = (int)pitch;
            q.G = q.G2 = 0;
            // Channel groups of 8, an even number (the two halves of a wavefront take one each per
            // MFMA step).  All of them are staged at once when weights + input rows + output
            // staging fit in LDS; else the channels go through in passes of the largest even
            // group count that fits half of it (two workgroups per CU overlap staging and MFMAs),
            // or all of it if not even one pair fits the half.
            const int64_t nchi_all = cdiv(Cin, 16) * 2;
            const int64_t per_pair = kh * kw * q.CB * 64 * 16 + 2 * (int64_t)q.RHa * pitch * 16;
            const int64_t o_bytes = (int64_t)q.CB * 32 * (q.TM / 2 + 2) * 4;
            int64_t pairs = nchi_all / 2;
            q.pipe = 0;
            if (pairs * per_pair + o_bytes > LDS_LIMIT) {
                pairs = (LDS_LIMIT / 2 - o_bytes) / per_pair;
                if (pairs < 1) pairs = (LDS_LIMIT - o_bytes) / per_pair;
                if (pairs < 1) return false;
                // 3x3 and 1x1 layers with Cin % 8 == 0 get the pipelined form of the multi-pass
                // kernel (a pass's loads fly under the previous pass's MFMAs): a pass then is
                // at most 1 (3x3) or 2 (1x1) weight units (8 channels x all taps of an output
                // channel) and 1 input unit of 8 channels x 8 pixels (3 of 8 x 1 when W % 8 != 0) per thread.
                const int64_t T = kh * kw;
                if ((T == 9 || T == 1) && (Cin % 8) == 0) {
                    int64_t pp = pairs;
                    const int64_t by_w = (T == 9 ? 256 : 512) / (q.CB * 32 * 2);
                    // input: one 8-pixel unit per thread (W % 8 == 0), else three 1-pixel units
                    const int64_t by_x = (W % 8) == 0 ? 256 / (2 * q.RHa * (W / 8)) : 768 / (2 * q.RHa * W);
                    if (pp > by_w) pp = by_w;
                    if (pp > by_x) pp = by_x;
                    if (pp >= 1 && fastdiv_ok(768, W)) { pairs = pp; q.pipe = (int)T; q.div_w = make_fastdiv((uint32_t)W); }
                }
                // equal passes (the last one is padded with zero channels otherwise)
                const int64_t passes = cdiv(nchi_all / 2, pairs);
                pairs = cdiv(nchi_all / 2, passes);
            }
            q.nchi = (int)(2 * pairs);
            q.nchunks = (int)cdiv(nchi_all, q.nchi);
            q.S = (int)((q.nchi / 2) * kh * kw);
            q.lds_w_bytes = q.S * q.CB * 64 * 16;
            q.lds_x_bytes = (int)((int64_t)q.nchi * q.RHa * q.pitch * 16);
            if ((W % 8) == 0) {
                if (!fastdiv_ok((int64_t)q.nchi * q.RHa * (W / 8), W / 8)) return false;
                q.div_w8 = make_fastdiv((uint32_t)(W / 8));
            }
            if (!fastdiv_ok((int64_t)q.nchi * q.RHa, q.RHa)) return false;
            if (!fastdiv_ok((int64_t)q.CB * 32 * q.nchi, q.nchi)) return false;
            q.div_nchi = make_fastdiv((uint32_t)q.nchi);
            q.lds_o_offset = q.lds_w_bytes + q.lds_x_bytes;
        }
        q.lds_o_bytes = q.CB * 32 * (q.TM / 2 + 2) * 4;   // [channel][TM/2 + 2] dwords
        {
            const int64_t end_x = (int64_t)q.lds_w_bytes + (variant == CONV_PLANAR_SMALLC ? 32 : 0) + q.lds_x_bytes;
            const int64_t end_o = (int64_t)q.lds_o_offset + q.lds_o_bytes;
            q.lds_total = (int)round_up(end_x > end_o ? end_x : end_o, 16);
        }
        q.div_rha = make_fastdiv((uint32_t)q.RHa);
        // wave-specialised planar kernel: 4 multiplier + 4 mover wavefronts, double-buffered
        // input tile and output staging, one workgroup per CU
        q.ws = 0; q.su = 0; q.lg_chunks = 0;
        // (the kernel fetches a channel's weights in 16-byte vectors: at least one per channel)
        int lgc = 0;
        while ((1 << lgc) < q.pitch / 8) ++lgc;
        // (rows or output planes that start on any element: funnel-shifted staging and stores on the
        // output's 16-byte grid, not with the fused pooling)
        const int unal = ((W % 8) != 0 || (OH * OW) % 8 != 0) ? 1 : 0;
        q.unal = 0;
        if (variant == CONV_PLANAR_SMALLC && want_ws && q.front + kw <= 8 && pxw == 2 && nw == 4 && (!unal || !pool) && lgc <= 7 &&
            (((int64_t)Cin * q.RHa) << lgc) <= 128 * 10 && (int64_t)q.G * kw >= 8 &&
            N * Cin * H * W * 2 < (1ll << 31) &&
            N * Cout * OH * OW * 2 / (pool ? 4 : 1) < (1ll << 31)) {
            static const int steps[] = {4, 6, 8, 11, 12};
            int su = 0;
            for (int k = 0; k < 5 && !su; ++k)
                if (q.S <= steps[k] && q.S + 2 >= steps[k]) su = steps[k];
            const int64_t o_off = (int64_t)q.lds_w_bytes + 32 + 2 * (int64_t)q.lds_x_bytes;
            if (su && o_off + 2 * (int64_t)q.lds_o_bytes <= LDS_LIMIT) {
                q.ws = 1;
                q.unal = unal;
                // output planes off the 16-byte grid: tiles advance by 248 pixels and compute 256, so that
                // every 16-byte unit of a plane lies inside the tile that owns its first pixel
                // (unless the extra tiles cost the persistent grid, one workgroup per compute unit, a round that
                // outweighs the 12 % or so that such a tile's stores gain)
                if (unal && (OH * OW) % 8 != 0) {
                    const int64_t t_ov = std::max<int64_t>(1, cdiv(ohw - 8, q.TM - 8));
                    const int64_t slots = std::max<int64_t>(1, 256 / q.co_groups);
                    if (0.88 * (double)cdiv(N * t_ov, slots) <= (double)cdiv(N * q.tiles_per_image, slots)) {
                        q.tile_px = q.TM - 8;
                        q.tiles_per_image = (int)t_ov;
                    }
                }
                q.su = su;
                q.lg_chunks = lgc;
                q.lds_o_offset = (int)o_off;
                q.lds_total = (int)(o_off + 2 * (int64_t)q.lds_o_bytes);
            }
        }
        // the few-channel kernel without wave specialisation on output planes off the 16-byte grid: the same
        // overlapping tiles (a tile's run of a channel then has no elements outside every 16-byte store unit)
        if (variant == CONV_PLANAR_SMALLC && !q.ws && !pool && (OH * OW) % 8 != 0) {
            const int64_t t_ov = std::max<int64_t>(1, cdiv(ohw - 8, q.TM - 8));
            const int64_t wgs = std::min<int64_t>(3, LDS_LIMIT / (int64_t)conv_lds_bytes(q));
            const int64_t slots = std::max<int64_t>(1, 256 * wgs / q.co_groups);
            if (0.88 * (double)cdiv(N * t_ov, slots) <= (double)cdiv(N * q.tiles_per_image, slots)) {
                q.tile_px = q.TM - 8;
                q.tiles_per_image = (int)t_ov;
            }
        }
        // Room for the weights as they lie, out of which the few-channel kernel cuts its operands: where the tile's area is
        // smaller (11x11 windows on narrow images) it would gather them from memory a tap at a time (4 -> 64 on 19 of 124x142:
        // 29.8 -> 17.1 us, 3 -> 64 on 3 of 147x74: 23.1 -> 13.2).  Not where that costs a resident workgroup that the grid has
        // a use for.
        if (variant == CONV_PLANAR_SMALLC && !q.ws) {
            const int64_t raw = round_up((int64_t)q.lds_w_bytes + 32 + std::min<int64_t>(Cout, q.CB * 32) * Cin * kh * kw * 2 + 64, 16);
            const int64_t now = (int64_t)conv_lds_bytes(q), items = N * q.tiles_per_image * q.co_groups;
            if (raw > now && raw <= LDS_LIMIT &&
                (std::min<int64_t>(3, LDS_LIMIT / raw) == std::min<int64_t>(3, LDS_LIMIT / now) || items <= 256 * (LDS_LIMIT / raw)))
                q.lds_total = (int)raw;
        }
        if ((int64_t)conv_lds_bytes(q) > LDS_LIMIT) return false;
        q.wg_per_cu = (int)(LDS_LIMIT / (int64_t)conv_lds_bytes(q));
        // register budget: three workgroups (waves per SIMD) for the planar kernel, two otherwise
        const int reg_cap = q.ws ? 1 : (variant == CONV_PLANAR_SMALLC ? 3 : 2);
        if (q.wg_per_cu > reg_cap) q.wg_per_cu = reg_cap;
        if (!fastdiv_ok(ohw, OW) || !fastdiv_ok((int64_t)N * q.tiles_per_image, q.tiles_per_image)) return false;
        q.div_ow = make_fastdiv((uint32_t)OW);
        q.div_tiles = make_fastdiv((uint32_t)q.tiles_per_image);
        p = q;
        return true;
    };

    // Wave-specialised multi-pass kernel (conv2d_chws.hip): 256- or 128-pixel tiles x `cb` 32-channel blocks
    // (4, 2 or 1), 16 to 64 input channels per pass through two LDS buffers, 3x3, 1x1 or 5x5 windows.
    bool short_pass = false;     // 1x1 windows: no 64-channel passes
    bool any_count = false;      // the planner's own choice below: any channel count (a tile request and the fused pooling: as documented)
    auto try_chws = [&](int cb, bool forced, int nw = 8, int tm = 256, bool halo = false) -> bool {
        const bool k5 = kh == 5 && kw == 5;
        if (!((kh == 3 && kw == 3) || (kh == 1 && kw == 1) || k5)) return false;
        // 5x5 windows: the 64- and 32-channel tilings on 8 wavefronts (a tile request: 256 x 64), no added tensor, no pooling
        if (k5 && (cb > 2 || nw != 8 || pool || p.residual)) return false;
        if (k5 && tm != 256 && pl->tile_req[2] > 0 && pl->tile_req[3] > 0) return false;
        // its tiles are 256 pixels of one image: small images (13x13, 7x7) would leave a third
        // and more of every tile empty and stay with the 128-pixel tiles of the plain kernels
        if (!forced && !pool && 4 * ohw < 3 * cdiv(ohw, tm) * tm) return false;
        if (!any_count && (Cin % 8 != 0 || Cin < 16 || ncb < 2)) return false;
        if (Cin < 8 || (pool && p.residual)) return false;
        // residual layer: 3x3 and 1x1 windows, the 64-channel tilings on 8 wavefronts
        if (p.residual && (!(kh == 3 || kh == 1) || cb != 2 || nw != 8)) return false;
        if (cb != 1 && cb != 2 && cb != 4) return false;
        // 32-channel tiles: 128 pixels on 8 wavefronts, 3x3 and 1x1 windows, no added tensor, no pooling (for launches
        // that would otherwise leave half the chip idle)
        if (cb == 1 && (nw != 8 || tm != 128 || pool || p.residual)) return false;
        // fused pooling: 3x3 windows, the 64-channel tilings and the 128-channel one on 12 wavefronts; a tile is whole rows
        if (pool && (kh != 3 || !((cb == 2 && nw == 8) || (cb == 4 && nw == 12)) || (halo ? 3 : 2) * OW > tm)) return false;
        ConvParams q = p;
        q.variant = CONV_CHWS;
        q.CB = cb;
        q.co_groups = (int)cdiv(ncb, cb);
        q.PXW = tm == 128 ? 1 : ((cb == 4 && nw == 8) ? 4 : 2);    // 32-pixel blocks per multiplying wavefront
        q.NW = nw;                               // 8: four multiplying + four moving wavefronts; 12: eight + four
        q.TM = tm;                               // 256 pixels, or 128 (64- and 32-channel tiles on 8 wavefronts only)
        if (tm != 256 && !(tm == 128 && (cb == 2 || cb == 1) && nw == 8)) return false;
        q.tiles_per_image = (int)cdiv(ohw, q.TM);
        q.rows_out_max = (int)((q.TM + OW - 2) / OW + 1);
        if (q.rows_out_max > OH) q.rows_out_max = (int)OH;
        q.tile_px = q.TM;
        if (!pool && tm == 256) {
            // A tile of TM consecutive pixels starts anywhere in a row, so its covering sub-tensor
            // (Section IV-A, Eq. 9) is rows_out_max whole rows + the window's: on a 224-wide image
            // 5 staged rows for 1.14 rows of results.  Tiles of whole rows (R rows, R OW <= TM, the
            // rest of the MFMA tile idle) stage R - 1 + kh rows: taken when at least 80 % of the
            // tile is used and a fifth less input is staged over the image (224-wide: 51.8 -> 45.5 us for
            // 64 -> 64 channels; 112-wide: 3-5 % faster; 56-wide, a fifth less: no gain, not taken;
            // nor on the 128-pixel tiles of small launches, where the extra workgroups cost more).
            int64_t R = q.TM / OW;
            if (R > OH) R = OH;
            if (R >= 1 && (R * OW) % 8 == 0 && R * OW * 10 >= (int64_t)q.TM * 8) {
                const int64_t stage_lin = (int64_t)q.tiles_per_image * ((q.rows_out_max - 1) * sh + eh);
                const int64_t stage_row = cdiv(OH, R) * ((R - 1) * sh + eh);
                if (stage_row * 100 <= stage_lin * 80) {
                    q.tile_px = (int)(R * OW);
                    q.tiles_per_image = (int)cdiv(OH, R);
                    q.rows_out_max = (int)R;
                }
            }
        }
        if (pool) {
            // R whole rows per tile.  Carried row above (R even, R / 2 pooled rows per tile): bands of PB
            // pooled rows, a multiple of R / 2, about one band per compute unit (every band below the
            // first computes a tile more).  Computed row above (R odd, (R - 1) / 2 pooled rows): a
            // band is one tile.
            int64_t R = q.TM / OW;
            if (halo) { if (R % 2 == 0) --R; if (R > OH + 1) R = OH + 1; }
            else { R &= ~1ll; if (R > OH) R = OH; }
            const int64_t hp = R / 2;
            q.rows_out_max = (int)R;
            q.pool_halo = halo ? 1 : 0;
            q.PH = (int)(OH / 2); q.PW = (int)(OW / 2);
            int64_t nb = 256 / (N * q.co_groups > 0 ? N * q.co_groups : 1);
            if (nb < 1) nb = 1;
            int64_t pb = halo ? hp : round_up(cdiv(q.PH, nb), hp);
            q.PB = (int)pb;
            q.NB = (int)cdiv(q.PH, pb);
            q.pw8 = (int)cdiv(q.PW, 4);                       // units of 4 pooled pixels per pooled row
            if (!fastdiv_ok(N * q.NB, q.NB) || !fastdiv_ok((hp + 1) * q.pw8, q.pw8)) return false;
            q.div_nb = make_fastdiv((uint32_t)q.NB);
            q.div_pw8 = make_fastdiv((uint32_t)q.pw8);
        }
        q.RHa = (int)((q.rows_out_max - 1) * sh + eh);
        // a window one row high with a row stride uses every sh-th image row: only those are staged
        q.row_skip = (kh == 1 && sh > 1 && !pool) ? 1 : 0;
        if (q.row_skip) q.RHa = q.rows_out_max;
        q.front = 0; q.aligned = 0; q.ws = 0; q.su = 0; q.lg_chunks = 0; q.pipe = 0; q.unal = 0;
        q.G = q.G2 = 0;
        q.padl = (int)pw;
        int64_t pitch = q.padl + W;
        const int64_t reach = (OW - 1) * sw + ew;
        if (reach > pitch) pitch = reach;
        pitch |= 1;                               // odd: staged rows start in different LDS bank groups
        q.pitch = (int)pitch;
        // 16 input channels per pass; 32 with the small tile, whose passes would otherwise be
        // shorter than the memory round trip that brings the next one
        int64_t ng = tm == 128 && !k5 ? 2 : 1;
        if (kh == 1 && kw == 1 && Cin >= 128 && !pool && !short_pass) {
            // 1x1 windows: a pass is one tap; 64 channels per pass where its rows and staging units fit
            const int64_t g = 4, xb = 2 * g * (int64_t)q.RHa * pitch * 16, wb = g * cb * 64 * 16;
            const int64_t rows = 2 * g * (int64_t)q.RHa;
            const int64_t nu = W >= 8 ? rows * cdiv(W, 8) : (W == 4 ? rows : rows * W);
            const int64_t cap = (W >= 8 ? 2 : (W == 4 ? (nw == 8 ? 4 : 2) : (nw == 8 ? 8 : 4))) * 256;
            if (2 * (wb + xb) <= LDS_LIMIT && nu <= cap) ng = g;
        }
        q.nchi = (int)(2 * ng);
        q.nchunks = (int)cdiv(Cin, 16 * ng);
        q.S = (int)(ng * kh * kw);
        const int64_t w_bytes = ng * kh * kw * cb * 64 * 16;
        const int64_t x_bytes = 2 * ng * (int64_t)q.RHa * pitch * 16;
        const int64_t o_bytes = (int64_t)cb * 32 * (q.TM / 2 + 2) * 4;
        const int64_t total = 2 * (w_bytes + x_bytes) > o_bytes ? 2 * (w_bytes + x_bytes) : o_bytes;
        if (total > LDS_LIMIT) return false;
        q.lds_w_bytes = (int)w_bytes; q.lds_x_bytes = (int)x_bytes; q.lds_buf_bytes = (int)(w_bytes + x_bytes);
        q.lds_o_offset = 0; q.lds_o_bytes = (int)o_bytes; q.lds_total = (int)total;
        if (pool) {
            // two carry buffers (the last row of a tile, every channel) behind the pass buffers / staging area
            const int64_t carry = 2 * (int64_t)cb * 32 * (OW / 2) * 4 + 16;
            q.lds_o_offset = (int)round_up(total, 16);
            q.lds_total = (int)(q.lds_o_offset + carry);
            if (q.lds_total > LDS_LIMIT) return false;
        }
        // staging units per moving thread and pass: 8 channels x 8 pixels, two at most.  Where more would be needed (the
        // many rows of a tile on narrow images with a row stride), or rows are shorter: x 4 pixels (W % 4 == 0; four,
        // two on 12 wavefronts) and x 2 (W even; no added tensor, no pooling) or 1, eight of them (four on 12 wavefronts
        // and for 5x5 windows).  3x3 / 3, 400 -> 221 on 3 of 138x10: 65 us, on the channels-in-passes kernel 262;
        // 3x3 / 4, 888 -> 60 on 9 of 174x4: 45 us, with one-pixel units 82.
        const int64_t rows = 2 * ng * (int64_t)q.RHa;
        auto units_of = [&](int64_t px, int64_t most) -> bool {
            const int64_t nu = rows * cdiv(W, px);
            if (W < px || nu > most * 256 || !fastdiv_ok(nu, px == 1 ? W : rows)) return false;
            q.xpx = (int)px;
            q.xu = (int)cdiv(nu, 256);
            if (px == 1) q.div_w = make_fastdiv((uint32_t)W);
            else q.div_r2 = make_fastdiv((uint32_t)rows);
            return true;
        };
        const bool short_units = Cin % 8 == 0 && W % 8 != 0;
        // Rows of an odd width start on 2-byte boundaries, where a 16-byte load takes twice the time, so that on many
        // channels, where passes count, the eight coalesced 2-byte loads of a one-pixel unit can be the faster ones.
        // 3x3 windows on rows of 63 pixels and more, from 128 channels on (448 -> 48 on 11 of 11x65: 24 us against 33;
        // 64 channels: equal at best, 32 -> 336 on 12 of 13x75: 16.2 against 11.4) or with a row stride (96 -> 841 on 10
        // of 30x111 / 2: 43 against 50); from 256 channels on also rows of a
        // power of two and one (512 -> 64 on 6 of 9x9: 10 % faster; 64 channels: 8 % slower) and where 8-pixel units
        // would be two per thread (512 -> 64 on 6 of 21x21 / 2: 14 %).  Elsewhere the 8-pixel units gain 5-25 %.
        const bool one_px = short_units && kh == 3 && W % 2 == 1 &&
                            ((W >= 63 && (Cin >= 128 || sh > 1)) ||
                             (Cin >= 256 && (((W - 1) & (W - 2)) == 0 || rows * cdiv(W, 8) > 256)));
        if (!(one_px && units_of(1, nw == 8 ? 8 : 4)) && !units_of(8, 2) && !(short_units && !k5 && W % 4 == 0 && units_of(4, nw == 8 ? 4 : 2)) &&
            !(short_units && !k5 && W % 2 == 0 && !pool && !p.residual && units_of(2, nw == 8 ? 8 : 4)) &&
            !(short_units && units_of(1, nw == 8 && !k5 ? 8 : 4)))
            return false;
        const int64_t nitems = pool ? N * q.NB * q.co_groups : N * q.tiles_per_image * q.co_groups;
        if (nitems >= (1ll << 30) || !fastdiv_ok(nitems + 256, q.co_groups) || !fastdiv_ok(2 * ng * (int64_t)q.RHa, q.RHa) ||
            !fastdiv_ok(ohw, OW) || !fastdiv_ok(N * q.tiles_per_image, q.tiles_per_image))
            return false;
        if (N * Cin * H * W >= (1ll << 31) || N * Cout * ohw >= (1ll << 31)) return false;
        // byte offsets into the input and into the weights, as they lie or packed
        if ((N > 0 && chws_images_per_launch(q) == 0) || Cout * Cin * kh * kw * 2 >= (1ll << 31) - 64 ||
            q.co_groups * q.nchunks * w_bytes >= (1ll << 31))
            return false;
        q.div_cog = make_fastdiv((uint32_t)q.co_groups);
        q.div_rha = make_fastdiv((uint32_t)q.RHa);
        q.div_ow = make_fastdiv((uint32_t)OW);
        q.div_tiles = make_fastdiv((uint32_t)q.tiles_per_image);
        q.wg_per_cu = 1;
        p = q;
        return true;
    };

    // tile = (wavefronts per workgroup) x (pixels per wavefront): 4 x 32, 4 x 64 or, for the
    // planar kernel, 8 x 32.  256-pixel tiles when that still leaves a large grid.
    const bool want_big = N * cdiv(ohw, 256) * p.co_groups >= 512;
    bool ok = false;
    pl->est_units = 0.0;
    pl->two_pass = 0;
    if (pool && Cin >= 8) {
        // many input channels: the wave-specialised multi-pass kernel pools out of its staging area.
        // A tile request names one of its tilings: 8 x 64 (256 pixels x 64 channels), 8 x 32 (128 x 64),
        // 12 x 64 (256 x 128).
        const bool req = pl->tile_req[2] > 0 && pl->tile_req[3] > 0;
        const int64_t rw = pl->tile_req[2], rp = pl->tile_req[3];
        if (req && !((rw == 8 && (rp == 64 || rp == 32)) || (rw == 12 && rp == 64))) return MERIT_ERR_UNSUPPORTED;
        // Six candidates: 256 x 64, 128 x 64 or 256 x 128 tiles, the row above a tile's first pooled
        // row carried from the tile before or computed by the tile itself.  Estimated time = rounds of
        // the grid x tiles per workgroup x cost of a tile (256 x 64: 1, 128 x 64: 0.6, 256 x 128: 1.6; from timings).
        int best_tm = 0, best_cb = 0; bool best_halo = false; double best = 0.0;
        for (int cand = 0; cand < 6; ++cand) {
            const int shape = cand >> 1;                       // 0: 256 x 64, 1: 128 x 64, 2: 256 x 128
            const int tm = shape == 1 ? 128 : 256, cb = shape == 2 ? 4 : 2, nw = shape == 2 ? 12 : 8;
            const bool halo = (cand & 1) != 0;
            if (req && !(rw == nw && rp == (shape == 1 ? 32 : 64))) continue;
            if (cb == 4 && ncb < 4) continue;
            const ConvParams saved = p;
            const bool fits = try_chws(cb, true, nw, tm, halo);
            const ConvParams q = p;
            p = saved;
            if (!fits) continue;
            const int64_t items = N * q.NB * q.co_groups;
            const int64_t hp = q.rows_out_max / 2;
            const int64_t per_item = cdiv(q.PB, hp) + (halo || q.NB == 1 ? 0 : 1);
            const double cost = (double)cdiv(items, 256) * (double)per_item * (shape == 0 ? 1.0 : (shape == 1 ? 0.6 : 1.6));
            if (!best_tm || cost < best) { best_tm = tm; best_cb = cb; best_halo = halo; best = cost; }
        }
        ok = best_tm != 0 && try_chws(best_cb, true, best_cb == 4 ? 12 : 8, best_tm, best_halo);
        if (!ok) return MERIT_ERR_UNSUPPORTED;
        pl->est_units = best;
    } else if (pool) {
        // few input channels: the wave-specialised planar kernel pools; a tile request must name it (8 x 64) or nothing
        if (pl->tile_req[2] > 0 && pl->tile_req[3] > 0 && (pl->tile_req[2] != 8 || pl->tile_req[3] != 64))
            return MERIT_ERR_UNSUPPORTED;
        if (OW % 16 != 0) return MERIT_ERR_UNSUPPORTED;    // it pools 8 columns at a time
        want_ws = true;
        ok = try_variant(CONV_PLANAR_SMALLC, 2, 4) && p.ws;
        if (!ok) return MERIT_ERR_UNSUPPORTED;
        p.PH = (int)(OH / 2); p.PW = (int)(OW / 2); p.pw8 = p.PW / 8;
        // bands of pooled rows: about one workgroup per compute unit, but at least 4 rows per
        // band (every band recomputes one convolution row pair above its first pooled row)
        int64_t nb = 256 / (N * p.co_groups > 0 ? N * p.co_groups : 1);
        const int64_t nb_max = p.PH >= 4 ? p.PH / 4 : 1;
        if (nb > nb_max) nb = nb_max;
        if (nb < 1) nb = 1;
        p.PB = (int)cdiv(p.PH, nb);
        p.NB = (int)cdiv(p.PH, p.PB);
        if (!fastdiv_ok((int64_t)N * p.NB, p.NB) || !fastdiv_ok((int64_t)128 * 2 * p.CB, p.pw8))
            return MERIT_ERR_UNSUPPORTED;
        p.div_nb = make_fastdiv((uint32_t)p.NB);
        p.div_pw8 = make_fastdiv((uint32_t)p.pw8);
        if ((int64_t)N * p.NB >= (1ll << 31)) return MERIT_ERR_UNSUPPORTED;
    } else if (pl->tile_req[2] > 0 && pl->tile_req[3] > 0) {
        const int64_t nw = pl->tile_req[2], ppw = pl->tile_req[3];
        if ((nw != 4 && nw != 8 && nw != 12) || (ppw != 32 && ppw != 64 && ppw != 128)) return MERIT_ERR_UNSUPPORTED;
        if (ppw == 128 && nw != 8) return MERIT_ERR_UNSUPPORTED;
        if (nw == 12) {
            // 8 multiplying (64 pixels x 64 channels each) + 4 moving wavefronts: 256 pixels x 128 channels
            if (ppw != 64 || Cin < 8) return MERIT_ERR_UNSUPPORTED;
            ok = try_chws(4, true, 12);
            if (!ok) return MERIT_ERR_UNSUPPORTED;
        } else if (nw == 8 && Cin >= 8) {
            // 4 multiplying + 4 moving wavefronts on many channels: 256 pixels x 128 (4 x 32) or 64 channels
            ok = ppw == 32 ? try_chws(2, true, 8, 128) : try_chws(ppw == 128 ? 4 : 2, true);
            if (!ok) return MERIT_ERR_UNSUPPORTED;
        } else if (ppw == 128) {
            return MERIT_ERR_UNSUPPORTED;
        } else if (nw == 8 && ppw == 64) {
            // 4 multiplier wavefronts x 64 pixels + 4 mover wavefronts: the wave-specialised kernel
            if (p.residual) return MERIT_ERR_UNSUPPORTED;
            want_ws = true;
            if (Cin < 8) ok = try_variant(CONV_PLANAR_SMALLC, 2, 4) && p.ws;
            if (!ok) return MERIT_ERR_UNSUPPORTED;
        } else if (Cin < 8) ok = try_variant(CONV_PLANAR_SMALLC, (int)(ppw / 32), (int)nw);
        if (!ok && nw == 4) ok = try_variant(CONV_CHBLOCK, (int)(ppw / 32), 4);
    } else {
        // window rows of 9 to 16 taps with more 128-pixel tiles than compute units: 256-pixel tiles on 8
        // wavefronts (8 x 3 x 227 x 227 -> 96, 11x11 / s4: 30.8 -> 20.9 us; 4 wavefronts x 64 pixels: 23.8)
        if (Cin < 8 && kw > 8 && N * cdiv(ohw, 128) * p.co_groups > 256) ok = try_variant(CONV_PLANAR_SMALLC, 1, 8);
        if (!ok && Cin < 8)
            ok = want_big ? (try_variant(CONV_PLANAR_SMALLC, 2, 4) || try_variant(CONV_PLANAR_SMALLC, 1, 4))
                          : (try_variant(CONV_PLANAR_SMALLC, 1, 4) || try_variant(CONV_PLANAR_SMALLC, 2, 4));
        if (!ok)
            ok = want_big ? (try_variant(CONV_CHBLOCK, 2, 4) || try_variant(CONV_CHBLOCK, 1, 4))
                          : (try_variant(CONV_CHBLOCK, 1, 4) || try_variant(CONV_CHBLOCK, 2, 4));
        // 3x3 layers on at least 17 input channels (exceptions below):
        // the wave-specialised multi-pass kernel.  Its tilings: 256 pixels x 128 channels on 12
        // wavefronts, 256 x 64 and 128 x 64 (32 channels per pass) on 8.  The one with the lowest
        // estimate rounds of the grid x cost of a tile (1.6, 1, 0.6 from timings) is taken, the larger
        // tile on a tie: few large tiles while they still fill the chip, else more small ones --
        // also for images far smaller than a tile (13x13 on 256-pixel tiles: 32 us, against 98 us on
        // the plain multi-pass kernel; 7x7 on 128-pixel tiles: 28 against 88).  1x1 layers the same
        // (256 -> 64 on 56x56: 8.1 against 11.9 us, 1024 -> 256 on 14x14: 27 against 51); with a residual
        // tensor from 128 input channels on (128 -> 512 on 28x28: 11.7 against 36 us; 64 -> 256 on 56x56 is
        // a single short pass and stays on the single-pass kernel: 12.7 against 14.0).
        const bool window = (kh == 3 && kw == 3) || (kh == 1 && kw == 1 && (!p.residual || Cin >= 128)) ||
                            (kh == 5 && kw == 5 && !p.residual);
        // Channel counts off the multiple of 8, 17 to 31 of them, and at most 32 output channels: the same kernel
        // (65 -> 16 on 21 images of 18x20, stride 2: 31.3 -> 6.9 us; 165 -> 60 on 8 of 18x110, stride 2: 127 -> 23;
        // 100 -> 100 on 8 of 28x28: 40 -> 8.0).  On rows off the 8 pixels, which the channel-block kernels stage a pixel at
        // a time, and with 5x5 windows, also 16 channels and 64 aligned ones to at most 32 (16 -> 184 on 33 of 16x13, 5x5:
        // 34.3 -> 6.9 us; 48 -> 32 on 4 of 8x81, stride 2: 38 -> 5.5; 16 -> 24 on 52 of 106x86: 51.7 -> 38.4; over 120 such
        // layers 2.3x, none slower).  What stays on the channel-block kernels is close there, on rows of whole units (16 ->
        // 64 on 8 of 56x56: 5.7 against 5.3; 64 -> 32: 7.2 against 5.7; 24 -> 32: 6.2 against 5.0), or is held there by the
        // plan tests: single images with Cin % 8 != 0 (over 120 such layers 23-156 us on average by kernel and window, on
        // this one 5-26).
        // (1x1 windows at stride 1 have a kernel of their own: derive_px.)
        const bool was = Cin >= 32 && Cin % 8 == 0 && ncb >= 2;
        const bool off_units = W % 8 != 0 || kh == 5;
        any_count = (kh > 1 || sh > 1 || sw > 1) && Cin >= (off_units ? 16 : 17) && (Cin % 8 == 0 || N >= 2) &&
                    (ncb >= 2 || Cin % 8 != 0 || Cin > 64 || off_units);
        if (window && (was || any_count)) {
            // the tiling with the lowest estimate among those whose packed weights are at most so many bytes
            auto choose = [&](int64_t most_bytes, double *best_cost) -> bool {
                bool found = false;
                ConvParams best = p;
                for (int shape = 0; shape < 4; ++shape) {          // 0: 256 x 128 on 12 wavefronts, 1: 256 x 64, 2: 128 x 64, 3: 128 x 32
                    if (shape == 0 && ncb < 4) continue;
                    const int64_t tm = shape >= 2 ? 128 : 256;
                    const int cbs = shape == 0 ? 4 : (shape == 3 ? 1 : 2);
                    const ConvParams saved = p;
                    const bool fits = try_chws(cbs, true, shape == 0 ? 12 : 8, (int)tm);
                    const int64_t items = N * (int64_t)p.tiles_per_image * p.co_groups;     // (of the trial, if it fits)
                    // cost of a tile, from timings.  5x5 windows (16 channels per pass on every tiling: the weights of a pass
                    // are moved as often as on the large tile): 0.87 and 0.67 over 30 and 380 layers; 8-pixel staging units
                    // on wide rows of an odd width (see try_chws): with a row stride they are most of a tile's time (80 -> 352 on
                    // 12 of 6x123 / 2: 13.9 us in one round of large tiles with one-pixel units, 21.8 in two of small ones)
                    static const double tile_cost[2][4] = {{1.6, 1.0, 0.6, 0.42}, {0.0, 1.0, 0.87, 0.67}};
                    const double units = fits && W % 2 == 1 && W >= 63 && (Cin >= 128 || sh > 1) && p.xpx == 8 ? (sh > 1 ? 2.0 : 1.3) : 1.0;
                    const double cost = (double)cdiv(items, 256) * tile_cost[kh == 5][shape] * units;
                    const int64_t bytes = packed_bytes(p);
                    const ConvParams trial = p;
                    p = saved;
                    if (fits && bytes <= most_bytes && (!found || cost < *best_cost)) { found = true; best = trial; *best_cost = cost; }
                }
                if (found) p = best;
                return found;
            };
            double cost = 0.0;
            if (choose(INT64_MAX, &cost)) {
                ok = true;
                pl->est_units = cost;
                if (packed_bytes(p) > MERIT_NOALLOC_SCRATCH_BYTES) {
                    // (channel blocks and passes are padded by different amounts on different tilings)
                    const ConvParams run = p;
                    for (int i = 0; i < 2 && !pl->use_na; ++i) {
                        short_pass = i == 1;
                        if (choose(MERIT_NOALLOC_SCRATCH_BYTES, &cost)) { pl->conv_na = p; pl->use_na = 1; }
                        p = run;
                    }
                    short_pass = false;
                }
            }
        }
    }
    if (!ok) {
        // neither MFMA kernel holds this shape's operands in LDS: the one-element-per-thread
        // kernel takes any shape (not a tile request, which names an MFMA tiling, and not the
        // fused pooling, which only the wave-specialised kernel does)
        if (pool || (pl->tile_req[2] > 0 && pl->tile_req[3] > 0)) return MERIT_ERR_UNSUPPORTED;
        const int64_t per_image = Cout * ohw;
        if (per_image >= INT_LIMIT || H * W >= INT_LIMIT || Cout * Cin * kh * kw >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;
        p.variant = CONV_DIRECT;
        // a workgroup: 256 pixels x a block of output channels; the channel blocks count as
        // tiles of the image here (grid.y stays 1)
        p.PXW = 1; p.NW = 4; p.TM = 256; p.CB = 1; p.ws = 0; p.su = 0;
        p.co_groups = (int)cdiv(Cout, conv_direct_channels());
        p.tiles_per_image = (int)(p.co_groups * cdiv(ohw, 256));
        p.rows_out_max = 1; p.RHa = (int)eh; p.pitch = (int)W; p.padl = 0;
        p.G = p.G2 = p.S = p.nchi = 0; p.nchunks = 1; p.pipe = 0;
        p.lds_w_bytes = p.lds_x_bytes = p.lds_o_offset = p.lds_o_bytes = 0;
        p.lds_total = 32 * 1024;          // the kernel's own (static) weight buffer
        p.front = p.aligned = p.lg_chunks = 0;
        p.wg_per_cu = 8;
        p.div_ow = make_fastdiv((uint32_t)OW);
        p.div_tiles = make_fastdiv((uint32_t)p.tiles_per_image);
    }
    if ((int64_t)N * p.tiles_per_image >= (1ll << 31)) return MERIT_ERR_UNSUPPORTED;

    pl->out_ndim = 4;
    pl->out_shape[0] = N; pl->out_shape[1] = Cout; pl->out_shape[2] = OH; pl->out_shape[3] = OW;
    if (pool) { pl->out_shape[2] = p.PH; pl->out_shape[3] = p.PW; }
    merit_launch_info &li = pl->info;
    li.kernel = conv_kernel_name(p);
    // persistent grid; the launcher sizes it from the device's CU count (256 on MI355X)
    {
        int64_t slots = 256 * (int64_t)p.wg_per_cu / p.co_groups;
        if (slots < 1) slots = 1;
        const int64_t nt = (int64_t)N * p.tiles_per_image;
        li.grid[0] = nt < slots ? nt : slots;
        if (pool) li.grid[0] = (int64_t)N * p.NB;          // one workgroup per band, not persistent
        if (p.variant == CONV_DIRECT) li.grid[0] = nt;     // one workgroup per 256 pixels x 8 channels
        if (p.variant == CONV_CHWS) li.grid[0] = nt * p.co_groups < 256 ? nt * p.co_groups : 256;   // (tile, channel block) items
        if (p.variant == CONV_CHWS && pool) {                                                       // (band, channel block) items
            const int64_t nb = (int64_t)N * p.NB * p.co_groups;
            li.grid[0] = nb < 256 ? nb : 256;
        }
    }
    li.grid[1] = (p.variant == CONV_DIRECT || p.variant == CONV_CHWS) ? 1 : p.co_groups; li.grid[2] = 1;
    li.block[0] = p.ws ? 512 : p.NW * 64; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = (int64_t)conv_lds_bytes(p);
    li.tile[0] = 1; li.tile[1] = p.CB * 32; li.tile[2] = p.rows_out_max; li.tile[3] = OW;
    li.tile[4] = Cin; li.tile[5] = kh; li.tile[6] = kw;
    // convolution rows a band computes: its own and the row pair (few-channel kernel) or tile above
    if (pool) li.tile[2] = p.variant == CONV_CHWS ? ((p.pool_halo || p.NB == 1) ? p.rows_out_max * (int)cdiv(p.PB, p.rows_out_max / 2) : 2 * p.PB + p.rows_out_max) : 2 * (p.PB + 1);

    // Convolution + pooling on many channels: pooling inside the kernel costs MFMA time (a band of
    // pooled rows below the first recomputes the tile above it, tiles are whole rows, the 128-channel
    // tiling rarely fits), which a compute-bound layer cannot hide.  When the estimate for the
    // plain convolution plus one pass of the binary16 pooling kernel over its result is clearly
    // lower, the plan runs as those two launches (the result is the same: the maxima are exact).
    // Estimates in microseconds: a launch 4, a 256 x 64 tile 1.5 + 0.058 Cin kh kw / 9 (from
    // timings on 64 .. 512 channels), the pooling pass 3.5 (it cannot start before the convolution
    // has drained) + 1.25 x the convolution's result at 2.9 TB/s (measured: + 9 us for 12.8 MB,
    // + 3.4 us for 1.6 MB).  A tile request names a fused tiling and keeps the plan fused.
    if (pool && p.variant == CONV_CHWS && !(pl->tile_req[2] > 0 && pl->tile_req[3] > 0) && pl->est_units > 0.0) {
        merit_plan *plain = new (std::nothrow) merit_plan(*pl);
        if (plain) {
            plain->desc.op = p.relu ? MERIT_OP_CONV_DOT_RELU : MERIT_OP_CONV_DOT;
            if (derive_conv_families(plain) == MERIT_OK && plain->conv.variant == CONV_CHWS && plain->est_units > 0.0) {
                const double unit = 1.5 + 0.058 * (double)Cin * (double)(kh * kw) / 9.0;
                const double conv_bytes = (double)N * (double)Cout * (double)ohw * 2.0;
                const double t_fused = 4.0 + pl->est_units * unit;
                const double t_two = 4.0 + plain->est_units * unit + 3.5 + 1.25 * conv_bytes / 2.9e6;
                // (on a short launch the second launch and the temporary's allocation calls cost
                // more host time than the GPU saves: the convolution alone must be estimated at 12 us)
                if (t_two < 0.9 * t_fused && plain->est_units * unit >= 12.0) {
                    pl->two_pass = 1;
                    pl->conv2 = plain->conv;
                    const int64_t keep2 = li.tile[2];
                    li = plain->info;
                    li.tile[2] = keep2;
                    li.kernel = "merit_conv2d_chws+merit_maxpool_f16";
                }
            }
            delete plain;
        }
    }
    return MERIT_OK;
}

merit_status derive_conv(merit_plan *pl)
{
    if (const merit_status st = derive_conv_families(pl); st != MERIT_OK) return st;
    derive_px(pl);
    derive_split(pl);
    return MERIT_OK;
}

// ----------------------------------------------------- depthwise convolution ---
merit_status derive_dw(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    if (d.dtype != MERIT_F16 || d.pad != MERIT_PAD_ZERO) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 4 || d.n_acc != 2) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 4 || d.b.ndim != 3) return MERIT_ERR_UNSUPPORTED;
    const int64_t DC = INT64_MIN;
    const int axis_x[6] = {0, 1, 2, 3, 2, 3};
    const int64_t stride_x[6] = {1, 1, DC, DC, 1, 1};
    const int64_t offset_x[6] = {0, 0, 0, 0, DC, DC};
    const int axis_w[6] = {MERIT_AXIS_UNUSED, 0, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1, 2};
    const int64_t stride_w[6] = {0, 1, 0, 0, 1, 1};
    const int64_t offset_w[6] = {0, 0, 0, 0, 0, 0};
    if (!operand_is(d.a, 6, axis_x, stride_x, offset_x)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 6, axis_w, stride_w, offset_w)) return MERIT_ERR_UNSUPPORTED;
    const int64_t N = d.a.shape[0], C = d.a.shape[1], H = d.a.shape[2], W = d.a.shape[3];
    const int64_t OH = d.range[2], OW = d.range[3], kh = d.range[4], kw = d.range[5];
    const int64_t sh = d.a.stride[2], sw = d.a.stride[3];
    const int64_t ph = -d.a.offset[4], pw = -d.a.offset[5];
    if (N < 0 || C <= 0 || H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
        return MERIT_ERR_INVALID_ARG;
    if (d.range[0] != N || d.range[1] != C || d.b.shape[0] != C || d.b.shape[1] != kh || d.b.shape[2] != kw)
        return MERIT_ERR_SHAPE;
    if (H + 2 * ph < kh || W + 2 * pw < kw) return MERIT_ERR_SHAPE;
    if (OH != out_extent(H, kh, sh, ph) || OW != out_extent(W, kw, sw, pw)) return MERIT_ERR_SHAPE;
    if (N * C >= INT_LIMIT || H * W >= INT_LIMIT || kh > 31 || kw > 31 || sh > 16 || sw > 16)
        return MERIT_ERR_UNSUPPORTED;

    DwParams &p = pl->dw;
    p.NC = (int)(N * C); p.C = (int)C; p.H = (int)H; p.W = (int)W; p.OH = (int)OH; p.OW = (int)OW;
    p.kh = (int)kh; p.kw = (int)kw; p.sh = (int)sh; p.sw = (int)sw; p.ph = (int)ph; p.pw = (int)pw;
    // the workgroup of the kernel for any window: output rows, halves of an input row in LDS (0 rows: too wide)
    const int64_t pitch = W + 2 * pw;
    int64_t tile_rows = pl->tile_req[2] > 0 ? pl->tile_req[2] : (4096 / OW > 0 ? 4096 / OW : 1);
    if (tile_rows > OH) tile_rows = OH;
    while (tile_rows > 1 && ((tile_rows - 1) * sh + kh) * pitch * 2 > 48 * 1024) tile_rows = (tile_rows + 1) / 2;
    if (((tile_rows - 1) * sh + kh) * pitch * 2 > 96 * 1024) tile_rows = 0;
    // 3x3 and 5x5 windows at stride 1 and 2: the kernel without LDS (not where a tile request names the rows of a workgroup)
    const int64_t qw = 8 / (sw > 0 ? sw : 1), units = cdiv(OW, qw), planes = N * C;
    // Output rows of a thread: one as long as the launch fits the chip with it (a thread of four rows is a chain of 1.5 us
    // on a wavefront that has its SIMD to itself: 24 channels at 96x80, 5x5 / 2, 4.8 -> 3.0 us, 31x64x15x10 4.1 -> 2.8),
    // two up to 2000 workgroups of one row, where the rows that strips share start to count (7x336x9x83 5x5 6.8, 5.9, 7.9 us
    // with one, two, four), four beyond (5x456x41x107 15.2, 13.7, 12.8).  A row stride shares fewer: two up to 4000
    // workgroups of 5x5 windows (4x928x179x24 11.4 us, 12.1 with four; 181x10x192x57 16.7, 14.2; 16x501x73x665 305, 257), up
    // to 15000 of 3x3 ones (11x341x251x22 15.2, 17.2; 60x5x317x762 36.4, 33.4; 95x60x143x126 51.4, 46.6).
    const int64_t one_row = cdiv(planes * OH * units, 256), two_rows = sw == 1 ? 2000 : (kw == 5 ? 4000 : 15000);
    int64_t lanes_rows = one_row <= (sw == 2 ? 1500 : 600) ? 1 : (one_row <= two_rows ? 2 : 4);
    auto lanes_fit = [&](int64_t t) {                    // the kernel's divisions
        const int64_t n = planes * cdiv(OH, t);
        return n * units < (1ll << 30) && fastdiv_ok(n * units + 256, units) && fastdiv_ok(n, cdiv(OH, t));
    };
    while (lanes_rows < 4 && !lanes_fit(lanes_rows)) lanes_rows *= 2;
    const int64_t strips = cdiv(OH, lanes_rows);
    const bool rows = kh == 3 && kw == 3 && sh == 1 && sw == 1 && ph == 1 && pw == 1 && W % 8 == 0 && W <= 4096 && pl->tile_req[2] <= 0;
    bool lanes = !rows && kh == kw && (kw == 3 || kw == 5) && sh == sw && (sw == 1 || sw == 2) && pl->tile_req[2] <= 0 &&
                 planes * H * W >= 16 && planes * H * W < (1ll << 31) - 64 && lanes_fit(lanes_rows);
    if (lanes && tile_rows > 0) {
        // 5x5 windows at stride 1 on small planes of odd width: the kernel for any window, with an output a thread.  Rows on
        // every second 2-byte boundary cost the other 0.4 us (2x14x18x7 3.43 against 3.84 us, 2x40x8x17 3.49, 3.72, 4x31x8x21
        // 3.57, 3.75, 8x70x11x7 3.77, 3.68; on even widths 3.4 to 4.1 against 3.2 to 3.5).  Elsewhere over 260 small layers
        // it takes 0.96 to 1.83 of the other's time, 1.1 on average (1x24x9x14 3x3 / 2 2.75 against 2.67).  So with one and two
        // columns, most of whose loaded units lie outside the row (1x95x29x1 5x5 / 2 3.46 against 4.21, 8x10x26x2 5x5 3.46,
        // 4.07; 0.94 over 88 of them, 1.1 to 4 times the other's time from 1000 planes on).
        if (planes <= 512 && (W <= 2 || (kw == 5 && sw == 1 && W % 2 == 1 && tile_rows * OW <= 256))) lanes = false;
    }
    if (lanes) {
        p.variant = DW_LANES;
        p.TH = (int)lanes_rows;
        p.pitch = 1;
        p.lds_w_offset = 0; p.lds_bytes = 0;
        p.units = (int)units;
        p.items = (int)(N * C * strips * units);
        p.div_units = make_fastdiv((uint32_t)units);
        const int64_t wgs = cdiv(p.items, 256);
        p.xq = (int)(wgs / 8); p.xr = (int)(wgs % 8);
    } else if (rows) {
        p.variant = DW_ROWS_K3S1P1;
        int64_t TH = 4096 / W;                       // about two 8-pixel units per thread
        if (TH < 1) TH = 1;
        if (TH > OH) TH = OH;
        p.TH = (int)TH;
        p.pitch = (int)(W / 8 + 2);
        p.lds_w_offset = 0;
        p.lds_bytes = (int)((TH + 2) * p.pitch * 16);
        p.div_ow = make_fastdiv((uint32_t)(W / 8));
    } else {
        p.variant = DW_TILE_GENERIC;
        p.pitch = (int)pitch;
        const int64_t TH = tile_rows, RH = (TH - 1) * sh + kh;
        if (TH == 0) return MERIT_ERR_UNSUPPORTED;                           // very wide rows: no column tiling here
        p.TH = (int)TH;
        p.lds_w_offset = (int)round_up(RH * p.pitch * 2, 16);
        p.lds_bytes = (int)(p.lds_w_offset + kh * kw * 4);
        if (!fastdiv_ok(RH * p.pitch, p.pitch) || !fastdiv_ok(TH * OW, OW)) return MERIT_ERR_UNSUPPORTED;
        p.div_ow = make_fastdiv((uint32_t)OW);
    }
    p.tiles_y = (int)cdiv(OH, p.TH);
    const int64_t grid = (int64_t)p.NC * p.tiles_y;
    if (grid >= INT_LIMIT || !fastdiv_ok(grid, p.tiles_y) || !fastdiv_ok(p.NC, C) ||
        !fastdiv_ok((int64_t)(p.TH + 2 + kh * 16) * p.pitch, p.pitch))
        return MERIT_ERR_UNSUPPORTED;
    p.div_tiles_y = make_fastdiv((uint32_t)p.tiles_y);
    p.div_c = make_fastdiv((uint32_t)C);
    p.div_pitch = make_fastdiv((uint32_t)p.pitch);

    pl->out_ndim = 4;
    pl->out_shape[0] = N; pl->out_shape[1] = C; pl->out_shape[2] = OH; pl->out_shape[3] = OW;
    merit_launch_info &li = pl->info;
    li.kernel = dwconv_kernel_name(p);
    li.grid[0] = p.variant == DW_LANES ? cdiv(p.items, 256) : grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = p.lds_bytes;
    li.tile[0] = 1; li.tile[1] = 1; li.tile[2] = p.TH; li.tile[3] = OW; li.tile[4] = kh; li.tile[5] = kw;
    return MERIT_OK;
}

// -------------------------------------------------------- correlation layer ---
merit_status derive_corr(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    if (d.dtype != MERIT_F16 || d.pad != MERIT_PAD_ZERO) return MERIT_ERR_UNSUPPORTED;
    if (d.n_par != 5 || d.n_acc != 1) return MERIT_ERR_UNSUPPORTED;
    if (d.a.ndim != 4 || d.b.ndim != 4) return MERIT_ERR_UNSUPPORTED;
    const int64_t n = d.range[3];
    if (n <= 0 || (n % 2) == 0 || d.range[4] != n) return MERIT_ERR_SHAPE;
    const int64_t R = (n - 1) / 2;
    const int64_t sd = d.b.stride[3];
    if (sd <= 0) return MERIT_ERR_INVALID_ARG;
    const int axis_1[6] = {0, 2, 3, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1};
    const int64_t stride_1[6] = {1, 1, 1, 0, 0, 1};
    const int64_t offset_1[6] = {0, 0, 0, 0, 0, 0};
    const int axis_2[6] = {0, 2, 3, 2, 3, 1};
    const int64_t stride_2[6] = {1, 1, 1, sd, sd, 1};
    const int64_t offset_2[6] = {0, 0, 0, -R * sd, -R * sd, 0};
    if (!operand_is(d.a, 6, axis_1, stride_1, offset_1)) return MERIT_ERR_UNSUPPORTED;
    if (!operand_is(d.b, 6, axis_2, stride_2, offset_2)) return MERIT_ERR_UNSUPPORTED;
    const int64_t N = d.a.shape[0], C = d.a.shape[1], H = d.a.shape[2], W = d.a.shape[3];
    if (N < 0 || C <= 0 || H <= 0 || W <= 0) return MERIT_ERR_INVALID_ARG;
    for (int i = 0; i < 4; ++i)
        if (d.b.shape[i] != d.a.shape[i]) return MERIT_ERR_SHAPE;
    if (d.range[0] != N || d.range[1] != H || d.range[2] != W || d.range[5] != C) return MERIT_ERR_SHAPE;
    // the kernel stages 8-pixel units and gives a wavefront at most 8 column displacements
    if (W < 8 || R > 15 || sd > 8 || C > 65536) return MERIT_ERR_UNSUPPORTED;
    // Widths off the multiple of 8: up to 64 K products in all the definition kernel stays, because its own correlation
    // tests run these calls (13-69 us over 23 of them, the MFMA kernel 4); above, it costs 1.5 us per channel and the
    // MFMA kernel 5-12 us in all (8x60x60, +-5: 35 against 5).
    if ((W % 8) != 0 && N * C * H * W * n * n <= 65536) return MERIT_ERR_UNSUPPORTED;
    if (N * C * H * W >= INT_LIMIT || N * H * W * n * n >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;

    CorrParams &p = pl->corr;
    p.N = (int)N; p.C = (int)C; p.H = (int)H; p.W = (int)W; p.R = (int)R; p.sd = (int)sd; p.n = (int)n;
    p.nchi = (int)cdiv(C, 8);
    p.xchunks = (int)cdiv(W, 64);
    p.lead = (int)round_up(R * sd, 8);
    // (images narrower than a chunk of 64 pixels: only the columns that exist and their reach.  Fewer staged columns are
    // fewer pixel blocks to multiply and more channels a pass: us a launch in a graph, 248 channels on 29x19, +-3 / 2, 7.2 ->
    // 4.8, 136 on 42x25, +-5 / 2, 6.4 -> 5.2, 56 on 34x27, +-5, 4.4 -> 4.4; 1.12x over 60 of 16 to 64 pixels a side)
    const int64_t chunk = W < 64 ? round_up(W, 8) : 64;
    p.cols2 = (int)round_up(chunk + p.lead + R * sd, 8);
    // (rows off the multiple of 8: the zeros behind a row start where it ends, `cut` columns before their unit's own place, and
    // as many are missing at the end of what is staged.  A row's last chunk has those to spare, the one before it only where
    // it ends short of the row's last unit or stages that many more than it needs.  Eight columns more may be a pass more:
    // 180 channels on 3 of 89x85, +-5 / 2, 33.7 us without, 41.0 with.)
    const int64_t cut = round_up(W, 8) - W, reach = p.cols2 - p.lead;
    if (W > 64 && cut > 0 && reach > (64 + W % 64) / 8 * 8 && reach - cut < 64 + R * sd) p.cols2 += 8;
    // staged rows ordered by residue class of the column modulo sd (the 16 pixels of an MFMA block are adjacent)
    p.pitch1 = (int)cdiv(chunk, sd); p.P1 = (int)round_up(sd * p.pitch1, 8);      // (whole runs of eight: corr_slot)
    p.pitch2 = (int)cdiv(p.cols2, sd); p.P2 = (int)round_up(sd * p.pitch2, 8);
    p.nsb = (int)cdiv(p.pitch1, 16); p.nblk = (int)(sd * p.nsb);
    p.nb = (int)cdiv(16 + 2 * R, 16);
    // channel groups per pass: whole reduction steps of 4 groups, at most CORR_XB staging units (one) per
    // thread, and at most CORR_LDS_KB of them, so that several workgroups share a CU's LDS
    const int64_t per_g_full = chunk / 8 + p.cols2 / 8;
    const int64_t per_group = ((int64_t)p.P1 + p.P2) * 16;
    int64_t chg = (CORR_LDS_KB * 1024) / per_group;
    if (chg > 256 * CORR_XB / per_g_full) chg = 256 * CORR_XB / per_g_full;
    chg = chg / 4 * 4;
    if (chg < 4) chg = 4;
    // (without the rotation 0.98 of the time with it up to 64 channels over 208 images, 4 % less at 36 to 48 on 20 to 60 pixels
    // a side; as much on 64 to 150 and 3 to 12 % more beyond: 256 channels on 64x64, +-5 / 2, 7.25 us with, 8.1 without)
    p.rot = p.nchi > 8;
    const int64_t nchi4 = round_up(p.nchi, 4);
    const int64_t passes = cdiv(nchi4, chg);
    p.chg = (int)round_up(cdiv(nchi4, passes), 4);       // equal passes
    if (p.chg * per_g_full > 256 * CORR_XB || p.chg * per_group + 16 > LDS_LIMIT) return MERIT_ERR_UNSUPPORTED;
    p.div_sd = make_fastdiv((uint32_t)sd);
    p.div_perg = make_fastdiv((uint32_t)per_g_full);
    p.div_perg_last = make_fastdiv((uint32_t)(cdiv(W % 64, 8) + p.cols2 / 8));
    const int64_t grid = N * H * n * p.xchunks;
    if (grid >= INT_LIMIT || !fastdiv_ok(grid, p.xchunks) || !fastdiv_ok(grid, n) || !fastdiv_ok(grid, H))
        return MERIT_ERR_UNSUPPORTED;
    p.xq = (int)(grid / 8); p.xr = (int)(grid % 8);
    p.div_xchunks = make_fastdiv((uint32_t)p.xchunks);
    p.div_n = make_fastdiv((uint32_t)n);
    p.div_h = make_fastdiv((uint32_t)H);

    pl->out_ndim = 5;
    pl->out_shape[0] = N; pl->out_shape[1] = H; pl->out_shape[2] = W; pl->out_shape[3] = n; pl->out_shape[4] = n;
    merit_launch_info &li = pl->info;
    li.kernel = "merit_corr_mfma";
    li.grid[0] = grid; li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = (int64_t)corr_lds_bytes(p);
    li.tile[0] = 1; li.tile[1] = 1; li.tile[2] = W < 64 ? W : 64; li.tile[3] = 1; li.tile[4] = n; li.tile[5] = C;
    return MERIT_OK;
}

// ------------------------------------------------ any descriptor (Eq. 1, Eq. 5) ---
// What none of the patterns above recognises still is a ranged inner product: the definition
// kernel (generic.hip) runs it, one thread per row.  Operations: the dot products (CONV_DOT,
// CONV_DOT_RELU, DWCONV_DOT, CORR_DOT: binary16, zero or clamp padding, two operands) and the
// single-operand reductions (POOL_MAX: any padding rule; POOL_AVG: exclude, zero or clamp; fp32).
// The output is the dense tensor of the parallel ranges, so there are at most MERIT_MAX_DIMS of them.
merit_status derive_generic(merit_plan *pl)
{
    const merit_plan_desc &d = pl->desc;
    GenericParams &g = pl->gen;
    std::memset(&g, 0, sizeof(g));
    switch (d.op) {
    case MERIT_OP_CONV_DOT:
    case MERIT_OP_CONV_DOT_RELU:
    case MERIT_OP_DWCONV_DOT:
    case MERIT_OP_CORR_DOT:
        if (d.dtype != MERIT_F16 || (d.pad != MERIT_PAD_ZERO && d.pad != MERIT_PAD_CLAMP) || d.b.ndim < 1)
            return MERIT_ERR_UNSUPPORTED;
        g.mode = 0;
        g.relu = d.op == MERIT_OP_CONV_DOT_RELU ? 1 : 0;
        break;
    case MERIT_OP_POOL_MAX:
        if (d.dtype != MERIT_F32) return MERIT_ERR_UNSUPPORTED;
        g.mode = 1;
        break;
    case MERIT_OP_POOL_AVG:
        if (d.dtype != MERIT_F32 || d.pad == MERIT_PAD_NEG_INF) return MERIT_ERR_UNSUPPORTED;
        g.mode = 2;
        break;
    default: return MERIT_ERR_UNSUPPORTED;
    }
    if (d.n_par > MERIT_MAX_DIMS) return MERIT_ERR_UNSUPPORTED;
    g.pad = (int)d.pad;
    g.n_par = d.n_par; g.n_acc = d.n_acc;
    const int nidx = d.n_par + d.n_acc;
    int64_t rows = 1, acc = 1;
    for (int j = 0; j < nidx; ++j) {
        const int64_t r = d.range[j];
        if (r >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;
        if (j >= d.n_par && r < 1) return MERIT_ERR_INVALID_ARG;     // an empty reduction has no value
        g.range[j] = (int)r;
        if (j < d.n_par) { rows *= r; if (rows >= (1ll << 38)) return MERIT_ERR_UNSUPPORTED; }
        else { acc *= r; if (acc >= (1ll << 40)) return MERIT_ERR_UNSUPPORTED; }
    }
    g.rows = rows; g.acc = acc;
    auto operand = [&](const merit_operand &o, GenericOperand &q) -> merit_status {
        q.ndim = o.ndim;
        int64_t elems = 1;
        for (int i = o.ndim - 1; i >= 0; --i) {
            if (o.shape[i] < 1 || o.shape[i] >= (1ll << 31)) return MERIT_ERR_INVALID_ARG;
            q.shape[i] = (int)o.shape[i];
            q.pitch[i] = elems;
            elems *= o.shape[i];
            if (elems >= (1ll << 40)) return MERIT_ERR_UNSUPPORTED;
        }
        // every coordinate any k can produce stays a small integer
        int64_t lo[MERIT_MAX_DIMS] = {0}, hi[MERIT_MAX_DIMS] = {0};
        for (int j = 0; j < nidx; ++j) {
            q.axis[j] = o.axis[j];
            if (o.stride[j] <= -INT_LIMIT || o.stride[j] >= INT_LIMIT || o.offset[j] <= -INT_LIMIT || o.offset[j] >= INT_LIMIT)
                return MERIT_ERR_UNSUPPORTED;
            q.stride[j] = (int)o.stride[j]; q.offset[j] = (int)o.offset[j];
            if (o.axis[j] < 0) continue;
            const int64_t travel = (d.range[j] > 0 ? d.range[j] - 1 : 0) * o.stride[j];
            lo[o.axis[j]] += o.offset[j] + (travel < 0 ? travel : 0);
            hi[o.axis[j]] += o.offset[j] + (travel > 0 ? travel : 0);
            if (lo[o.axis[j]] <= -INT_LIMIT || hi[o.axis[j]] >= INT_LIMIT) return MERIT_ERR_UNSUPPORTED;
        }
        return MERIT_OK;
    };
    if (merit_status st = operand(d.a, g.a); st != MERIT_OK) return st;
    if (g.mode == 0) {
        if (merit_status st = operand(d.b, g.b); st != MERIT_OK) return st;
    } else {
        for (int j = 0; j < MERIT_MAX_INDEX; ++j) g.b.axis[j] = -1;
    }
    pl->generic = 1;
    pl->out_ndim = d.n_par;
    for (int j = 0; j < d.n_par; ++j) pl->out_shape[j] = d.range[j];
    merit_launch_info &li = pl->info;
    std::memset(&li, 0, sizeof(li));
    li.kernel = generic_kernel_name(g);
    li.grid[0] = cdiv(rows, 256); li.grid[1] = 1; li.grid[2] = 1;
    li.block[0] = 256; li.block[1] = 1; li.block[2] = 1;
    li.lds_bytes = 0;
    // a workgroup: 256 consecutive rows (the last parallel index fastest), the whole accumulation range
    for (int j = 0; j < nidx; ++j) li.tile[j] = j < d.n_par ? 1 : d.range[j];
    li.tile[d.n_par - 1] = d.range[d.n_par - 1] < 256 ? d.range[d.n_par - 1] : 256;
    return MERIT_OK;
}

bool aligned16(const void *ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

}  // namespace

// ============================================================== C ABI ======
extern "C" {

merit_status merit_plan_create(const merit_plan_desc *desc, merit_plan **out)
{
    if (!desc || !out) return MERIT_ERR_NULL;
    *out = nullptr;
    if ((int)desc->op < 0 || (int)desc->op > 12 || (int)desc->dtype < 0 || (int)desc->dtype > 2 ||
        (int)desc->pad < 0 || (int)desc->pad > 3)
        return MERIT_ERR_INVALID_ARG;
    if (desc->n_par < 1 || desc->n_acc < 1 || desc->n_par + desc->n_acc > MERIT_MAX_INDEX)
        return MERIT_ERR_INVALID_ARG;
    if (desc->a.ndim < 1 || desc->a.ndim > MERIT_MAX_DIMS || desc->b.ndim < 0 || desc->b.ndim > MERIT_MAX_DIMS)
        return MERIT_ERR_INVALID_ARG;
    const int nidx = desc->n_par + desc->n_acc;
    for (int j = 0; j < nidx; ++j) {
        if (desc->range[j] < 0) return MERIT_ERR_INVALID_ARG;
        if (desc->a.axis[j] < MERIT_AXIS_UNUSED || desc->a.axis[j] >= desc->a.ndim) return MERIT_ERR_INVALID_ARG;
        if (desc->b.ndim > 0 && (desc->b.axis[j] < MERIT_AXIS_UNUSED || desc->b.axis[j] >= desc->b.ndim))
            return MERIT_ERR_INVALID_ARG;
    }
    merit_plan *pl = new (std::nothrow) merit_plan;
    if (!pl) return MERIT_ERR_INVALID_ARG;
    std::memset(pl, 0, sizeof(*pl));
    pl->desc = *desc;
    merit_status st;
    switch (desc->op) {
    case MERIT_OP_CONV_DOT:
    case MERIT_OP_CONV_DOT_RELU:
    case MERIT_OP_CONV_DOT_POOLMAX:
    case MERIT_OP_CONV_DOT_RELU_POOLMAX:
    case MERIT_OP_CONV_DOT_ADD:
    case MERIT_OP_CONV_DOT_ADD_RELU: st = derive_conv(pl); break;
    case MERIT_OP_POOL_MAX:
    case MERIT_OP_POOL_AVG: st = derive_pool(pl); break;
    case MERIT_OP_CORR_DOT: st = derive_corr(pl); break;
    case MERIT_OP_DWCONV_DOT: st = derive_dw(pl); break;
    case MERIT_OP_SEPFILTER_DOT: st = derive_sep(pl); break;
    case MERIT_OP_BILATERAL: st = derive_bilateral(pl); break;
    default: st = derive_sad(pl); break;
    }
    // no specialised kernel for this descriptor: the definition kernel takes what it can
    if (st == MERIT_ERR_UNSUPPORTED) {
        const merit_status sg = derive_generic(pl);
        if (sg != MERIT_ERR_UNSUPPORTED) st = sg;
    }
    if (st != MERIT_OK) {
        delete pl;
        return st;
    }
    *out = pl;
    return MERIT_OK;
}

merit_status merit_plan_destroy(merit_plan *plan)
{
    if (!plan) return MERIT_ERR_NULL;
    delete plan;
    return MERIT_OK;
}

}  // extern "C"

static merit_status plan_conv2d_op(merit_op op, int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh,
                                   int sw, int ph, int pw, int dh, int dw, merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (N < 0 || Cin <= 0 || H <= 0 || W <= 0 || Cout <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 ||
        ph < 0 || pw < 0 || dh <= 0 || dw <= 0)
        return MERIT_ERR_INVALID_ARG;
    const int64_t eh = ((int64_t)kh - 1) * dh + 1, ew = ((int64_t)kw - 1) * dw + 1;
    if (H + 2 * ph < eh || W + 2 * pw < ew) return MERIT_ERR_SHAPE;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = op; d.dtype = MERIT_F16; d.pad = MERIT_PAD_ZERO;
    d.n_par = 4; d.n_acc = 3;
    const int64_t OH = out_extent(H, eh, sh, ph), OW = out_extent(W, ew, sw, pw);
    const int64_t range[7] = {N, Cout, OH, OW, Cin, kh, kw};
    const int ax[7] = {0, MERIT_AXIS_UNUSED, 2, 3, 1, 2, 3};
    const int64_t sx[7] = {1, 0, sh, sw, 1, dh, dw};
    const int64_t ox[7] = {0, 0, 0, 0, 0, -ph, -pw};
    const int aw[7] = {MERIT_AXIS_UNUSED, 0, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1, 2, 3};
    const int64_t sw_[7] = {0, 1, 0, 0, 1, 1, 1};
    for (int j = 0; j < 7; ++j) {
        d.range[j] = range[j];
        d.a.axis[j] = ax[j]; d.a.stride[j] = sx[j]; d.a.offset[j] = ox[j];
        d.b.axis[j] = aw[j]; d.b.stride[j] = sw_[j]; d.b.offset[j] = 0;
    }
    d.a.ndim = 4; d.a.shape[0] = N; d.a.shape[1] = Cin; d.a.shape[2] = H; d.a.shape[3] = W;
    d.b.ndim = 4; d.b.shape[0] = Cout; d.b.shape[1] = Cin; d.b.shape[2] = kh; d.b.shape[3] = kw;
    return merit_plan_create(&d, out);
}

extern "C" {

merit_status merit_plan_conv2d(int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw,
                               int ph, int pw, merit_plan **out)
{
    return plan_conv2d_op(MERIT_OP_CONV_DOT, N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, 1, 1, out);
}

merit_status merit_plan_conv2d_relu(int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw,
                                    int ph, int pw, merit_plan **out)
{
    return plan_conv2d_op(MERIT_OP_CONV_DOT_RELU, N, Cin, H, W, Cout, kh, kw, sh, sw, ph, pw, 1, 1, out);
}

merit_status merit_plan_conv2d_dilated(int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw,
                                       int ph, int pw, int dh, int dw, int relu, merit_plan **out)
{
    return plan_conv2d_op(relu ? MERIT_OP_CONV_DOT_RELU : MERIT_OP_CONV_DOT, N, Cin, H, W, Cout, kh, kw, sh, sw, ph,
                          pw, dh, dw, out);
}

merit_status merit_plan_conv2d_pool(int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw,
                                    int ph, int pw, int relu, merit_plan **out)
{
    return plan_conv2d_op(relu ? MERIT_OP_CONV_DOT_RELU_POOLMAX : MERIT_OP_CONV_DOT_POOLMAX, N, Cin, H, W, Cout,
                          kh, kw, sh, sw, ph, pw, 1, 1, out);
}

merit_status merit_plan_conv2d_residual(int N, int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw,
                                        int ph, int pw, int relu, merit_plan **out)
{
    return plan_conv2d_op(relu ? MERIT_OP_CONV_DOT_ADD_RELU : MERIT_OP_CONV_DOT_ADD, N, Cin, H, W, Cout, kh, kw, sh,
                          sw, ph, pw, 1, 1, out);
}

merit_status merit_plan_pool2d(int N, int C, int H, int W, int kh, int kw, int sh, int sw, int ph, int pw,
                               int is_avg, merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (N < 0 || C <= 0 || H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
        return MERIT_ERR_INVALID_ARG;
    if (H + 2 * ph < kh || W + 2 * pw < kw) return MERIT_ERR_SHAPE;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = is_avg ? MERIT_OP_POOL_AVG : MERIT_OP_POOL_MAX;
    d.dtype = MERIT_F32;
    d.pad = is_avg ? MERIT_PAD_EXCLUDE : MERIT_PAD_NEG_INF;
    d.n_par = 4; d.n_acc = 2;
    const int64_t OH = out_extent(H, kh, sh, ph), OW = out_extent(W, kw, sw, pw);
    const int64_t range[6] = {N, C, OH, OW, kh, kw};
    const int ax[6] = {0, 1, 2, 3, 2, 3};
    const int64_t sx[6] = {1, 1, sh, sw, 1, 1};
    const int64_t ox[6] = {0, 0, 0, 0, -ph, -pw};
    for (int j = 0; j < 6; ++j) {
        d.range[j] = range[j];
        d.a.axis[j] = ax[j]; d.a.stride[j] = sx[j]; d.a.offset[j] = ox[j];
    }
    d.a.ndim = 4; d.a.shape[0] = N; d.a.shape[1] = C; d.a.shape[2] = H; d.a.shape[3] = W;
    d.b.ndim = 0;
    return merit_plan_create(&d, out);
}

static merit_status plan_window_filter(merit_op op, int N, int H, int W, int k, merit_plan **out);

merit_status merit_plan_sepfilter(int N, int H, int W, int k, merit_plan **out)
{
    return plan_window_filter(MERIT_OP_SEPFILTER_DOT, N, H, W, k, out);
}

merit_status merit_plan_bilateral(int N, int H, int W, int k, merit_plan **out)
{
    return plan_window_filter(MERIT_OP_BILATERAL, N, H, W, k, out);
}

merit_status merit_bilateral(const merit_plan *plan, const void *x, const void *gx, const void *gy, double norm,
                             void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_BILATERAL) return MERIT_ERR_INVALID_ARG;
    if (!(norm == norm) || norm * 1.4426950408889634 > 3.0e38 || norm * 1.4426950408889634 < -3.0e38)
        return MERIT_ERR_INVALID_ARG;
    if (plan->bil.N == 0) return MERIT_OK;                // empty batch: nothing to read or write
    if (!x || !gx || !gy || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(y) || ((uintptr_t)gx & 3) || ((uintptr_t)gy & 3)) return MERIT_ERR_ALIGNMENT;
    merit::BilatParams p = plan->bil;                     // the plan stays shareable between threads
    p.neg = norm <= 0.0 ? 1 : 0;
    p.scale = (float)std::sqrt(std::fabs(norm) * 1.4426950408889634);
    return launch_bilateral(p, static_cast<const float *>(x), static_cast<const float *>(gx),
                            static_cast<const float *>(gy), static_cast<float *>(y),
                            static_cast<hipStream_t>(stream)) == hipSuccess
               ? MERIT_OK
               : MERIT_ERR_HIP;
}

}  // extern "C"

// k = (n, p1, p2 | a1, a2): the image window at offset -k/2 on both axes, a vector of length k on a2
static merit_status plan_window_filter(merit_op op, int N, int H, int W, int k, merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (N < 0 || H <= 0 || W <= 0 || k <= 0) return MERIT_ERR_INVALID_ARG;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = op; d.dtype = MERIT_F32; d.pad = MERIT_PAD_CLAMP;
    d.n_par = 3; d.n_acc = 2;
    const int64_t range[5] = {N, H, W, k, k};
    const int ax[5] = {0, 1, 2, 1, 2};
    const int64_t ox[5] = {0, 0, 0, -(int64_t)(k / 2), -(int64_t)(k / 2)};
    for (int j = 0; j < 5; ++j) {
        d.range[j] = range[j];
        d.a.axis[j] = ax[j]; d.a.stride[j] = 1; d.a.offset[j] = ox[j];
        d.b.axis[j] = j == 4 ? 0 : MERIT_AXIS_UNUSED; d.b.stride[j] = j == 4 ? 1 : 0; d.b.offset[j] = 0;
    }
    d.a.ndim = 3; d.a.shape[0] = N; d.a.shape[1] = H; d.a.shape[2] = W;
    d.b.ndim = 1; d.b.shape[0] = k;
    return merit_plan_create(&d, out);
}

// The stream-ordered temporaries of the two-launch plans come from the device's default memory
// pool.  By default that pool hands freed memory back to the system at the next synchronisation,
// so a caller who synchronises between calls would pay a device allocation per call (measured: 79
// against 69 us per call for the one-kernel form, which is slower on the GPU).  Once per device the
// pool's release threshold is raised so that it keeps what it has been given.
static void keep_pool_memory_once()
{
    static std::atomic<int> done[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    if (done[dev].load(std::memory_order_acquire)) return;
    hipMemPool_t pool = nullptr;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess && pool) {
        uint64_t keep = UINT64_MAX;
        (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
    }
    done[dev].store(1, std::memory_order_release);
}

extern "C" {

merit_status merit_sepfilter(const merit_plan *plan, const void *x, const void *kx, const void *ky, void *y,
                             void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_SEPFILTER_DOT) return MERIT_ERR_INVALID_ARG;
    if (plan->sep.N == 0) return MERIT_OK;                // empty batch: nothing to read or write
    if (!x || !kx || !ky || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(y) || ((uintptr_t)kx & 3) || ((uintptr_t)ky & 3)) return MERIT_ERR_ALIGNMENT;
    return launch_sepfilter(plan->sep, static_cast<const float *>(x), static_cast<const float *>(kx),
                            static_cast<const float *>(ky), static_cast<float *>(y),
                            static_cast<hipStream_t>(stream)) == hipSuccess
               ? MERIT_OK
               : MERIT_ERR_HIP;
}

merit_status merit_plan_sad(int H, int W, int block, int range, merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (H <= 0 || W <= 0 || block <= 0 || range < 0) return MERIT_ERR_INVALID_ARG;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = MERIT_OP_SAD_ARGMIN; d.dtype = MERIT_U8; d.pad = MERIT_PAD_CLAMP;
    d.n_par = 2; d.n_acc = 4;
    const int64_t n = 2 * (int64_t)range + 1;
    const int64_t rg[6] = {cdiv(H, block), cdiv(W, block), n, n, block, block};
    const int a_ref[6] = {0, 1, 0, 1, 0, 1};
    const int64_t s_ref[6] = {block, block, 1, 1, 1, 1};
    const int64_t o_ref[6] = {0, 0, -range, -range, 0, 0};
    const int a_cur[6] = {0, 1, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 0, 1};
    const int64_t s_cur[6] = {block, block, 0, 0, 1, 1};
    for (int j = 0; j < 6; ++j) {
        d.range[j] = rg[j];
        d.a.axis[j] = a_ref[j]; d.a.stride[j] = s_ref[j]; d.a.offset[j] = o_ref[j];
        d.b.axis[j] = a_cur[j]; d.b.stride[j] = s_cur[j]; d.b.offset[j] = 0;
    }
    d.a.ndim = 2; d.a.shape[0] = H; d.a.shape[1] = W;
    d.b.ndim = 2; d.b.shape[0] = H; d.b.shape[1] = W;
    return merit_plan_create(&d, out);
}

merit_status merit_plan_set_tile(merit_plan *plan, const int64_t tile[MERIT_MAX_INDEX])
{
    if (!plan || !tile) return MERIT_ERR_NULL;
    if (plan->generic) {                                   // the definition kernel has one shape: nothing to choose
        for (int j = 0; j < MERIT_MAX_INDEX; ++j)
            if (tile[j] > 0) return MERIT_ERR_UNSUPPORTED;
        return MERIT_OK;
    }
    if (plan->desc.op == MERIT_OP_CORR_DOT && plan->desc.a.shape[3] % 8 != 0) {      // one tiling, and no request names it
        for (int j = 0; j < MERIT_MAX_INDEX; ++j)
            if (tile[j] > 0) return MERIT_ERR_UNSUPPORTED;
    }
    merit_plan trial = *plan;
    for (int j = 0; j < MERIT_MAX_INDEX; ++j) trial.tile_req[j] = tile[j];
    merit_status st;
    switch (trial.desc.op) {
    case MERIT_OP_CONV_DOT:
    case MERIT_OP_CONV_DOT_RELU:
    case MERIT_OP_CONV_DOT_POOLMAX:
    case MERIT_OP_CONV_DOT_RELU_POOLMAX:
    case MERIT_OP_CONV_DOT_ADD:
    case MERIT_OP_CONV_DOT_ADD_RELU: st = derive_conv(&trial); break;
    case MERIT_OP_POOL_MAX:
    case MERIT_OP_POOL_AVG: st = derive_pool(&trial); break;
    case MERIT_OP_CORR_DOT: st = derive_corr(&trial); break;
    case MERIT_OP_DWCONV_DOT: st = derive_dw(&trial); break;
    case MERIT_OP_SEPFILTER_DOT: st = derive_sep(&trial); break;
    case MERIT_OP_BILATERAL: st = derive_bilateral(&trial); break;
    default: st = derive_sad(&trial); break;
    }
    if (st != MERIT_OK) return st;          // the plan keeps its previous tiling
    *plan = trial;
    return MERIT_OK;
}

merit_status merit_plan_get_desc(const merit_plan *plan, merit_plan_desc *out)
{
    if (!plan || !out) return MERIT_ERR_NULL;
    *out = plan->desc;
    return MERIT_OK;
}

merit_status merit_plan_out_shape(const merit_plan *plan, int32_t *ndim, int64_t shape[MERIT_MAX_DIMS])
{
    if (!plan || !ndim || !shape) return MERIT_ERR_NULL;
    *ndim = plan->out_ndim;
    for (int i = 0; i < MERIT_MAX_DIMS; ++i) shape[i] = i < plan->out_ndim ? plan->out_shape[i] : 0;
    return MERIT_OK;
}

merit_status merit_plan_footprint(const merit_plan *plan, int which, const int64_t tile[MERIT_MAX_INDEX],
                                  int64_t out[MERIT_MAX_DIMS])
{
    if (!plan || !tile || !out) return MERIT_ERR_NULL;
    if (which != 0 && which != 1) return MERIT_ERR_INVALID_ARG;
    const merit_operand &o = which == 0 ? plan->desc.a : plan->desc.b;
    if (o.ndim == 0) return MERIT_ERR_INVALID_ARG;
    const int nidx = plan->desc.n_par + plan->desc.n_acc;
    for (int j = 0; j < nidx; ++j)
        if (tile[j] < 1 || tile[j] > plan->desc.range[j]) return MERIT_ERR_INVALID_ARG;
    for (int i = 0; i < MERIT_MAX_DIMS; ++i) {
        int64_t n = 0;
        if (i < o.ndim) {
            n = 1;
            for (int j = 0; j < nidx; ++j)
                if (o.axis[j] == i) n += (tile[j] - 1) * o.stride[j];
        }
        out[i] = n;
    }
    return MERIT_OK;
}

merit_status merit_plan_launch_info(const merit_plan *plan, merit_launch_info *out)
{
    if (!plan || !out) return MERIT_ERR_NULL;
    *out = plan->info;
    return MERIT_OK;
}

// a plan on the definition kernel: the same pointer rules as everywhere
static merit_status run_generic(const merit_plan *plan, const void *a, const void *b, void *y, void *stream)
{
    if (plan->gen.rows == 0) return MERIT_OK;             // an empty parallel range: nothing to read or write
    if (!a || !b || !y) return MERIT_ERR_NULL;
    if (!aligned16(a) || !aligned16(b) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    return launch_generic(plan->gen, a, b, y, static_cast<hipStream_t>(stream)) == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_conv2d(const merit_plan *plan, const void *x, const void *w, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_CONV_DOT && plan->desc.op != MERIT_OP_CONV_DOT_RELU &&
        plan->desc.op != MERIT_OP_CONV_DOT_POOLMAX && plan->desc.op != MERIT_OP_CONV_DOT_RELU_POOLMAX)
        return MERIT_ERR_INVALID_ARG;
    if (plan->generic) return run_generic(plan, x, w, y, stream);
    if (plan->conv.N == 0) return MERIT_OK;               // empty batch: nothing to read or write
    if (!x || !w || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    if (plan->two_pass) {
        // the plain convolution into the plan's buffer on this device, then the pooling kernel
        // The convolution's result lives in a stream-ordered temporary: allocated and released in
        // the caller's stream, so calls on different streams never share it and the plan stays
        // immutable.  (The pool that serves it keeps the memory for the next call.)
        const ConvParams &q = plan->conv2;
        hipStream_t s = static_cast<hipStream_t>(stream);
        keep_pool_memory_once();
        void *mid = nullptr;
        if (hipMallocAsync(&mid, (size_t)q.N * q.Cout * q.OH * q.OW * 2, s) != hipSuccess || !mid) return MERIT_ERR_HIP;
        hipError_t e = launch_conv2d(q, x, w, nullptr, mid, s);
        if (e == hipSuccess) e = launch_maxpool_f16(mid, y, (int64_t)q.N * q.Cout, q.OH, q.OW, s);
        const hipError_t ef = hipFreeAsync(mid, s);
        return (e == hipSuccess && ef == hipSuccess) ? MERIT_OK : MERIT_ERR_HIP;
    }
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = plan->use_px      ? launch_conv2d_px(plan->px, x, w, nullptr, y, s)
                         : plan->use_split ? launch_conv2d_split(plan->split, x, w, y, s, false)
                                           : launch_conv2d(plan->conv, x, w, nullptr, y, s);
    return e == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

static bool plan_takes_packed(const merit_plan *plan)
{
    return (plan->desc.op == MERIT_OP_CONV_DOT || plan->desc.op == MERIT_OP_CONV_DOT_RELU) && packable(plan);
}

merit_status merit_plan_packed_weights_bytes(const merit_plan *plan, int64_t *bytes)
{
    if (!plan || !bytes) return MERIT_ERR_NULL;
    if (!plan_takes_packed(plan)) return MERIT_ERR_UNSUPPORTED;
    const ConvParams &p = plan->conv;
    *bytes = packed_bytes(p);
    return MERIT_OK;
}

merit_status merit_conv2d_pack_weights(const merit_plan *plan, const void *w, void *packed, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (!plan_takes_packed(plan)) return MERIT_ERR_UNSUPPORTED;
    if (!w || !packed) return MERIT_ERR_NULL;
    if (!aligned16(w) || !aligned16(packed)) return MERIT_ERR_ALIGNMENT;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    // (the matrix-product kernel reads the weights as they lie: its packed copy is a copy)
    const hipError_t e = plan->use_px      ? launch_copy_weights(w, packed, (int64_t)plan->px.Cout * plan->px.Cin, s)
                         : plan->use_split ? launch_conv2d_split_pack(plan->split, w, packed, s)
                                           : launch_conv2d_pack_weights(plan->conv, w, packed, s);
    return e == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_conv2d_packed(const merit_plan *plan, const void *x, const void *packed, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (!plan_takes_packed(plan)) return MERIT_ERR_UNSUPPORTED;
    if (plan->conv.N == 0) return MERIT_OK;               // empty batch: nothing to read or write
    if (!x || !packed || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(packed) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = plan->use_px      ? launch_conv2d_px(plan->px, x, packed, nullptr, y, s)
                         : plan->use_split ? launch_conv2d_split(plan->split, x, packed, y, s, true)
                                           : launch_conv2d_chws(plan->conv, x, packed, nullptr, y, s, true);
    return e == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_conv2d_packed_noalloc(const merit_plan *plan, const void *x, const void *w, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (!plan_takes_packed(plan)) return MERIT_ERR_UNSUPPORTED;
    const ConvParams &p = plan->use_na ? plan->conv_na : plan->conv;
    // (the matrix-product kernel reads the weights as they lie: no copy, but the same limit)
    const int64_t bytes = plan->use_px ? (int64_t)plan->px.Cout * plan->px.Cin * 2 : packed_bytes(p);
    if (bytes > (int64_t)MERIT_NOALLOC_SCRATCH_BYTES) return MERIT_ERR_SCRATCH_LIMIT;
    if (p.N == 0) return MERIT_OK;                        // empty batch: nothing to read or write
    if (!x || !w || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = plan->use_px      ? launch_conv2d_px(plan->px, x, w, nullptr, y, s)
                         : plan->use_split ? launch_conv2d_split(plan->split, x, w, y, s, false)
                                           : launch_conv2d_chws_noalloc(p, x, w, y, s);
    return e == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_conv2d_residual(const merit_plan *plan, const void *x, const void *w, const void *r, void *y,
                                   void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_CONV_DOT_ADD && plan->desc.op != MERIT_OP_CONV_DOT_ADD_RELU)
        return MERIT_ERR_INVALID_ARG;
    if (plan->conv.N == 0) return MERIT_OK;               // empty batch: nothing to read or write
    if (!x || !w || !r || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(r) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = plan->use_px ? launch_conv2d_px(plan->px, x, w, r, y, s) : launch_conv2d(plan->conv, x, w, r, y, s);
    return e == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_pool2d(const merit_plan *plan, const void *x, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_POOL_MAX && plan->desc.op != MERIT_OP_POOL_AVG) return MERIT_ERR_INVALID_ARG;
    if (plan->generic) return run_generic(plan, x, x, y, stream);
    if (plan->pool.NC == 0) return MERIT_OK;              // empty batch: nothing to read or write
    if (!x || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    return launch_pool2d(plan->pool, static_cast<const float *>(x), static_cast<float *>(y),
                         static_cast<hipStream_t>(stream)) == hipSuccess
               ? MERIT_OK
               : MERIT_ERR_HIP;
}

merit_status merit_sad_search(const merit_plan *plan, const void *cur, const void *ref, void *sad, void *mv,
                              void *stream)
{
    if (!plan || !cur || !ref || !sad || !mv) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_SAD_ARGMIN) return MERIT_ERR_INVALID_ARG;
    if (!aligned16(cur) || !aligned16(ref) || !aligned16(sad) || !aligned16(mv)) return MERIT_ERR_ALIGNMENT;
    return launch_sad(plan->sad, static_cast<const uint8_t *>(cur), static_cast<const uint8_t *>(ref),
                      static_cast<int32_t *>(sad), static_cast<int32_t *>(mv),
                      static_cast<hipStream_t>(stream)) == hipSuccess
               ? MERIT_OK
               : MERIT_ERR_HIP;
}

merit_status merit_plan_conv2d_depthwise(int N, int C, int H, int W, int kh, int kw, int sh, int sw, int ph, int pw,
                                         merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (N < 0 || C <= 0 || H <= 0 || W <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
        return MERIT_ERR_INVALID_ARG;
    if (H + 2 * ph < kh || W + 2 * pw < kw) return MERIT_ERR_SHAPE;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = MERIT_OP_DWCONV_DOT; d.dtype = MERIT_F16; d.pad = MERIT_PAD_ZERO;
    d.n_par = 4; d.n_acc = 2;
    const int64_t OH = out_extent(H, kh, sh, ph), OW = out_extent(W, kw, sw, pw);
    const int64_t range[6] = {N, C, OH, OW, kh, kw};
    const int ax[6] = {0, 1, 2, 3, 2, 3};
    const int64_t sx[6] = {1, 1, sh, sw, 1, 1};
    const int64_t ox[6] = {0, 0, 0, 0, -ph, -pw};
    const int aw[6] = {MERIT_AXIS_UNUSED, 0, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1, 2};
    const int64_t sw_[6] = {0, 1, 0, 0, 1, 1};
    for (int j = 0; j < 6; ++j) {
        d.range[j] = range[j];
        d.a.axis[j] = ax[j]; d.a.stride[j] = sx[j]; d.a.offset[j] = ox[j];
        d.b.axis[j] = aw[j]; d.b.stride[j] = sw_[j]; d.b.offset[j] = 0;
    }
    d.a.ndim = 4; d.a.shape[0] = N; d.a.shape[1] = C; d.a.shape[2] = H; d.a.shape[3] = W;
    d.b.ndim = 3; d.b.shape[0] = C; d.b.shape[1] = kh; d.b.shape[2] = kw;
    return merit_plan_create(&d, out);
}

merit_status merit_conv2d_depthwise(const merit_plan *plan, const void *x, const void *w, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_DWCONV_DOT) return MERIT_ERR_INVALID_ARG;
    if (plan->generic) return run_generic(plan, x, w, y, stream);
    if (plan->dw.NC == 0) return MERIT_OK;                // empty batch: nothing to read or write
    if (!x || !w || !y) return MERIT_ERR_NULL;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    return launch_dwconv(plan->dw, x, w, y, static_cast<hipStream_t>(stream)) == hipSuccess ? MERIT_OK : MERIT_ERR_HIP;
}

merit_status merit_plan_correlation(int N, int C, int H, int W, int R, int sd, merit_plan **out)
{
    if (!out) return MERIT_ERR_NULL;
    *out = nullptr;
    if (N < 0 || C <= 0 || H <= 0 || W <= 0 || R < 0 || sd <= 0) return MERIT_ERR_INVALID_ARG;
    merit_plan_desc d;
    std::memset(&d, 0, sizeof(d));
    d.op = MERIT_OP_CORR_DOT; d.dtype = MERIT_F16; d.pad = MERIT_PAD_ZERO;
    d.n_par = 5; d.n_acc = 1;
    const int64_t n = 2 * (int64_t)R + 1;
    const int64_t range[6] = {N, H, W, n, n, C};
    const int a1[6] = {0, 2, 3, MERIT_AXIS_UNUSED, MERIT_AXIS_UNUSED, 1};
    const int64_t s1[6] = {1, 1, 1, 0, 0, 1};
    const int a2[6] = {0, 2, 3, 2, 3, 1};
    const int64_t s2[6] = {1, 1, 1, sd, sd, 1};
    const int64_t o2[6] = {0, 0, 0, -(int64_t)R * sd, -(int64_t)R * sd, 0};
    for (int j = 0; j < 6; ++j) {
        d.range[j] = range[j];
        d.a.axis[j] = a1[j]; d.a.stride[j] = s1[j]; d.a.offset[j] = 0;
        d.b.axis[j] = a2[j]; d.b.stride[j] = s2[j]; d.b.offset[j] = o2[j];
    }
    d.a.ndim = 4; d.a.shape[0] = N; d.a.shape[1] = C; d.a.shape[2] = H; d.a.shape[3] = W;
    d.b.ndim = 4; d.b.shape[0] = N; d.b.shape[1] = C; d.b.shape[2] = H; d.b.shape[3] = W;
    return merit_plan_create(&d, out);
}

merit_status merit_correlation(const merit_plan *plan, const void *x1, const void *x2, void *y, void *stream)
{
    if (!plan) return MERIT_ERR_NULL;
    if (plan->desc.op != MERIT_OP_CORR_DOT) return MERIT_ERR_INVALID_ARG;
    if (plan->generic) return run_generic(plan, x1, x2, y, stream);
    if (plan->corr.N == 0) return MERIT_OK;               // empty batch: nothing to read or write
    if (!x1 || !x2 || !y) return MERIT_ERR_NULL;
    if (!aligned16(x1) || !aligned16(x2) || !aligned16(y)) return MERIT_ERR_ALIGNMENT;
    return launch_correlation(plan->corr, x1, x2, y, static_cast<hipStream_t>(stream)) == hipSuccess ? MERIT_OK
                                                                                                   : MERIT_ERR_HIP;
}

const char *merit_status_string(merit_status s)
{
    switch ((int)s) {          // a C caller may pass any int
    case MERIT_OK: return "ok";
    case MERIT_ERR_NULL: return "null pointer";
    case MERIT_ERR_INVALID_ARG: return "invalid argument";
    case MERIT_ERR_SHAPE: return "inconsistent shape";
    case MERIT_ERR_UNSUPPORTED: return "transform not supported by any kernel";
    case MERIT_ERR_ALIGNMENT: return "device pointer not 16-byte aligned";
    case MERIT_ERR_HIP: return "HIP launch failed";
    case MERIT_ERR_SCRATCH_LIMIT: return "needs more scratch memory than the library's fixed buffer holds";
    }
    return "unknown status";
}

}  // extern "C"
