// 2-D convolution for gfx950, many input channels on few output pixels: the channels split among the wavefronts.
//
// k = (n, co, oy, ox | ci, ky, kx) (Section III-C, Eq. 6), reduced with the dot product (Section III-B, Eq. 3) on
// v_mfma_f32_32x32x16_f16, as in conv2d_chws.hip.  There a workgroup's channels go through LDS in passes, one barrier
// each, and a launch of a few dozen tiles spends its time in that chain (memory round trip, transposition, barrier, a few
// MFMAs) while the rest of the chip is idle.  Here
//   * tiles are small (32 or 64 pixels x 32 output channels), so that there are more of them;
//   * each of the eight wavefronts owns every eighth slice of 16 input channels for the whole tile, fetches and stages it
//     by itself in an LDS area of its own, and multiplies it: no barrier until the partial sums meet at the end;
//   * the weights as they lie (16 channels x all taps of an output channel are contiguous) are fetched in the order of
//     memory, handed through LDS to the lanes whose output channel they are, and cut into MFMA operands in registers;
//     packed, they are those operands and go straight to registers.
// Bound by the loads of a slice: 16-byte loads of 8 lanes in 8 rows of pixels each (twice the time on rows of an odd
// width), 2-3 us per eight slices on one workgroup per compute unit; a workgroup's start and its sums are 2 us more.
//
// us a launch, multi-pass form -> this one (graph of twenty launches over four input sets):
//   256 -> 256 on 8 images of 14x14         12.3 -> 9.0, packed 10.7 -> 7.2
//   512 -> 512 on 8 of 7x7                  20.6 -> 12.7
//   512 -> 512 on 28x28                     18.6 -> 13.0
//   40 -> 40 on 2 of 31x18                  5.8 -> 4.2
//   432 -> 196 on 23x26, stride 2, packed   24.8 -> 10.5
//   5x5 680 -> 22 on 3 of 47x11, stride 2   83 -> 36
// Tiles are adjacent pixels of the plane, for which whole input rows are staged, or rectangles 8, 16 or 32 pixels wide, for
// which the columns they need are: long rows and row strides did not fit otherwise, and left such layers to a few dozen
// tiles of the other form.  Rectangles, us a launch, before -> with them (41 of 400 layers of 7 to 112 pixels a side take
// them, 1.37x in the geometric mean):
//   536 -> 32 on 14x109                      50.2 -> 14.8
//   414 -> 32 on 3 of 32x92, stride 2        28.0 -> 9.8
//   5x5 72 -> 56 on 6 of 16x105, stride 2    16.1 -> 7.9
//   264 -> 264 on 34x41                      11.9 -> 10.3
// and on larger launches the other form keeps (64 -> 64 on 8 of 56x56 6.8 against 19, 256 -> 256 on 56x56 12.0 against 20):
// its wavefronts share what they stage.
#include "merit_internal.h"

#include <atomic>

namespace merit {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t OOB = 0x80000000u;      // a buffer offset past every tensor: zeros come back
constexpr int WAVES = SPLIT_WAVES, NT = WAVES * 64;

}  // namespace

// K: window edge (3 or 5).  PXB: 32-pixel blocks of the tile.  XU: staging units of 8 channels x 8 pixels per lane and
// slice (0: one, of rows shorter than 8 pixels).  RAGGED: Cin % 8 != 0.
template <int K, int PXB, int XU, bool PACKED, bool RAGGED>
__global__ __launch_bounds__(NT, 2) void merit_conv2d_split(SplitParams p, const uint16_t *__restrict__ x,
                                                           const uint16_t *__restrict__ w, uint16_t *__restrict__ y)
{
    static_assert(!(PACKED && RAGGED), "packed weights: whole groups of 8 channels");
    constexpr int T = K * K, TM = 32 * PXB;
    constexpr int NXU = XU == 0 ? 1 : XU;
    constexpr int OPITCH = TM + 4;                        // staging of the sums: [WAVES][32][OPITCH] floats
    // 3x3 windows: the operands of a slice are cut out of the raw weights at once, and the next slice's are on their way
    // meanwhile; 5x5 windows (100 registers of them) are cut tap by tap and fetched again behind the last tap
    constexpr bool EARLY = !PACKED && K == 3;
    // Raw weights of a slice, 3x3 windows: 18 chunks of 16 bytes for each of the 32 output channels, fetched four lanes to a
    // row (a lane that fetched its own output channel's row would have 64 lanes in 64 places: 64 cycles a load instead of
    // 16) and handed to the lanes that multiply them through LDS, in rows whose pitch puts 16 of them into 16 different
    // bank groups.  5x5 windows, whose 25 chunks a group leave no registers for that: each lane its own row.
    constexpr int WPITCH = split_weight_pitch(K);

    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, c32 = lane & 31;

    // An XCD's share of the list is a contiguous band: of pixel tiles with all their channel blocks, or, where the weights
    // are the larger operand, of channel blocks with all their tiles, so that its L2 fetches its share of that operand only.
    const int item = (int)xcd_band_item(blockIdx.x, p.xq, p.xr);
    const int major = (int)fdiv((uint32_t)item, p.div_minor), minor = item - major * p.minor;
    const int tile = p.by_channel ? minor : major, cg = p.by_channel ? major : minor;
    const int n = (int)fdiv((uint32_t)tile, p.div_tiles);
    const int ohw = p.OH * p.OW;
    // a run of TM adjacent pixels from m0 on, or a rectangle at (oyA, oxA); image column of staged column 0
    const int at = tile - n * p.tiles;
    int m0 = at * TM, oyA, oxA = 0, colA = -p.pw;
    if (p.lg_tw == 0) {
        oyA = (int)fdiv((uint32_t)m0, p.div_ow);
    } else {
        const int ty = (int)fdiv((uint32_t)at, p.div_tiles_x);
        oyA = ty * (TM >> p.lg_tw);
        oxA = (at - ty * p.tiles_x) << p.lg_tw;
        colA = min(oxA * p.sw - p.pw, p.W - 8) & ~1;         // (units are whole: the last one of a row ends with it)
    }
    const int yA = oyA * p.sh - p.ph;
    const int chbytes = p.H * p.W * 2;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x + (size_t)n * p.Cin * p.H * p.W), 0, p.Cin * chbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(w), 0, PACKED ? p.co_groups * p.slices * T * 1024 : p.Cout * p.Cin * T * 2, 0x00020000);

    // ---- what a lane loads of every slice ----
    uint8_t *area = smem + wave * (p.slice_bytes + (PACKED ? 0 : 32 * WPITCH));      // [group][row][pitch][8 channels]
    uint8_t *warea = area + p.slice_bytes;                                         // [32][WPITCH]
    uint32_t x_voff[NXU];
    int x_lds[NXU], x_hh[NXU];
    {
        const int nu = 2 * p.RHa * p.units_x;
#pragma unroll
        for (int k = 0; k < NXU; ++k) {
            // consecutive lanes: consecutive staged rows (the pitch is odd: their LDS writes start in different banks)
            const int u = lane + 64 * k, uc = min(u, nu - 1);
            const int xc = (int)fdiv((uint32_t)uc, p.div_r2);
            const int q = uc - xc * 2 * p.RHa;
            const int hh = q >= p.RHa ? 1 : 0;
            const int gy = yA + q - hh * p.RHa;
            const int col = XU == 0 ? 0 : min(max(colA, 0) + 8 * xc, p.W - 8);       // (a row's last unit ends with the row)
            x_hh[k] = u < nu ? hh : 2;
            x_voff[k] = u < nu && gy >= 0 && gy < p.H ? (uint32_t)(((hh * 8 * p.H + gy) * p.W + col) * 2) : OOB;
            x_lds[k] = (q * p.pitch + col - colA) * 16;
        }
    }

    // The last slice starts earlier where it would not be whole, so that it ends with the last channel (Cin >= 17); the
    // channels that it shares with the slice before it are zeros in both operands.
    auto first_channel = [&](int sl) __attribute__((always_inline)) { return min(sl * 16, p.Cin - 16); };

    uint32x4 xv[NXU][8];
    uint32_t xmoved[XU == 0 ? 8 : 1];                     // bits by which a short row's load was moved to stay inside the image
    uint32x4 wl[PACKED || K == 3 ? T : 1];                // raw 3x3: chunks in the order of memory; packed: the operand of each tap
    uint32_t wr[PACKED ? 1 : 4 * T];                      // raw: this lane's 8 channels x T taps
    auto issue_x = [&](int sl) __attribute__((always_inline)) {
        const int ch0 = first_channel(sl);
        const int early = sl < p.slices ? sl * 16 - ch0 : 16;          // (past the last slice: everything out of range)
        const uint32_t base = (uint32_t)ch0 * (uint32_t)chbytes;
#pragma unroll
        for (int k = 0; k < NXU; ++k) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const bool in = (RAGGED ? c : 0) + 8 * x_hh[k] >= early;
                uint32_t voff = in ? x_voff[k] + (uint32_t)(c * chbytes) : OOB;
                if constexpr (XU == 0) {
                    const uint32_t moved = moved_to_end(base + voff, (uint32_t)(p.Cin * chbytes));
                    xmoved[c] = 8u * moved;
                    voff -= moved;
                }
                xv[k][c] = __builtin_amdgcn_raw_buffer_load_b128(rx, voff, base, 0);
            }
        }
    };
    uint32_t w_voff[3];
    if constexpr (K == 3) {
        const int q = lane >> 2, d = lane >> 1;            // output channels: q, q + 16; d for the last two chunks
        const uint32_t row = (uint32_t)p.Cin * (uint32_t)(2 * T);
        w_voff[0] = cg * 32 + q < p.Cout ? (uint32_t)(cg * 32 + q) * row + (lane & 3) * 16 : OOB;
        w_voff[1] = cg * 32 + 16 + q < p.Cout ? (uint32_t)(cg * 32 + 16 + q) * row + (lane & 3) * 16 : OOB;
        w_voff[2] = cg * 32 + d < p.Cout ? (uint32_t)(cg * 32 + d) * row + 256 + (lane & 1) * 16 : OOB;
    } else {
        w_voff[0] = cg * 32 + c32 < p.Cout ? (uint32_t)((cg * 32 + c32) * p.Cin + 8 * h) * (uint32_t)(2 * T) : OOB;
    }
    auto issue_w = [&](int sl) __attribute__((always_inline)) {
        if constexpr (!PACKED) {
            const int ch0 = first_channel(sl);
            const uint32_t at = (uint32_t)ch0 * (uint32_t)(2 * T);
            const bool past = sl >= p.slices;
            if constexpr (K == 3) {
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const uint32_t voff = i < 8 ? w_voff[i & 1] + 64 * (i >> 1) : w_voff[2];
                    wl[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, past ? OOB : voff, at, 0);
                }
            } else {
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const uint32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, past ? OOB : w_voff[0] + 16 * i, at, 0);
                    wr[4 * i] = v.x; wr[4 * i + 1] = v.y; wr[4 * i + 2] = v.z; wr[4 * i + 3] = v.w;
                }
            }
        }
    };
    auto hand_over = [&](int sl) __attribute__((always_inline)) {
        if constexpr (!PACKED) {
            if constexpr (K == 3) {
                uint8_t *d0 = warea + (lane >> 2) * WPITCH + (lane & 3) * 16, *d2 = warea + (lane >> 1) * WPITCH + 256 + (lane & 1) * 16;
#pragma unroll
                for (int i = 0; i < 9; ++i)
                    *reinterpret_cast<uint32x4 *>(i < 8 ? d0 + (i & 1) * 16 * WPITCH + 64 * (i >> 1) : d2) = wl[i];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const uint8_t *src = warea + c32 * WPITCH + h * T * 16;
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    const uint32x4 v = *reinterpret_cast<const uint32x4 *>(src + 16 * i);
                    wr[4 * i] = v.x; wr[4 * i + 1] = v.y; wr[4 * i + 2] = v.z; wr[4 * i + 3] = v.w;
                }
            }
            if (sl == p.slices - 1) {
                // the slice before's channels: zeros
                const int skip = min(max(sl * 16 - first_channel(sl) - 8 * h, 0), 8) * T;       // halves
#pragma unroll
                for (int i = 0; i < 4 * T; ++i) wr[i] &= 2 * i >= skip ? ~0u : (2 * i + 1 >= skip ? 0xffff0000u : 0u);
            }
        }
    };
    auto issue_wp = [&](int sl, int t) __attribute__((always_inline)) {       // packed: the operand of one tap
        wl[t] = __builtin_amdgcn_raw_buffer_load_b128(rw, sl < p.slices ? (uint32_t)lane * 16u : OOB,
                                                      (uint32_t)((cg * p.slices + min(sl, p.slices - 1)) * T + t) * 1024u, 0);
    };

    int sl = wave;
    const bool any = sl < p.slices;
    if (any) {
        issue_x(sl);
        if constexpr (PACKED) {
#pragma unroll
            for (int t = 0; t < T; ++t) issue_wp(sl, t);
        } else issue_w(sl);
    }
    // the zeros left and right of the image (rows above and below it come as zeros from memory)
    for (int i = lane; i < (p.slice_bytes >> 4); i += 64) reinterpret_cast<uint4 *>(area)[i] = make_uint4(0, 0, 0, 0);

    // ---- what a lane multiplies: a pixel of each block ----
    int xa[PXB];
#pragma unroll
    for (int pb = 0; pb < PXB; ++pb) {
        int oy, ox;
        if (p.lg_tw == 0) {
            const int m = min(m0 + pb * 32 + c32, ohw - 1);
            oy = (int)fdiv((uint32_t)m, p.div_ow);
            ox = m - oy * p.OW;
        } else {
            const int m = pb * 32 + c32;
            oy = min(oyA + (m >> p.lg_tw), p.OH - 1);
            ox = min(oxA + (m & ((1 << p.lg_tw) - 1)), p.OW - 1);
        }
        xa[pb] = ((h * p.RHa + (oy - oyA) * p.sh) * p.pitch + ox * p.sw - p.pw - colA) * 16;
    }
    floatx16 acc[PXB];
#pragma unroll
    for (int pb = 0; pb < PXB; ++pb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[pb][r] = 0.0f;

    // the operand of tap t out of the raw weights: halves c T + t of the channels c of the group
    auto cut = [&](int t) __attribute__((always_inline)) {
        uint32x4 f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e0 = 2 * j * T + t, e1 = (2 * j + 1) * T + t;
            const uint32_t sel = ((e0 & 1) ? 0x0302u : 0x0100u) | ((e1 & 1) ? 0x07060000u : 0x05040000u);
            f[j] = __builtin_amdgcn_perm(wr[e1 >> 1], wr[e0 >> 1], sel);
        }
        return f;
    };
    auto commit_x = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NXU; ++k) {
            if (x_hh[k] > 1) continue;
            if constexpr (XU == 0) {
                // (the last channel's last row: only there can a load have been moved)
                if (s == p.slices - 1) {
#pragma unroll
                    for (int c = 0; c < 8; ++c)
                        if (xmoved[c] != 0) {
                            const uint4 m = shift_down(make_uint4(xv[k][c].x, xv[k][c].y, xv[k][c].z, xv[k][c].w), (int)xmoved[c]);
                            xv[k][c].x = m.x; xv[k][c].y = m.y; xv[k][c].z = m.z; xv[k][c].w = m.w;
                        }
                }
            }
#pragma unroll
            for (int px = 0; px < 8; ++px) {
                if (XU == 0 && px >= p.W) break;
                const uint32_t sel = (px & 1) ? 0x07060302u : 0x05040100u;
                uint4 d;
                d.x = __builtin_amdgcn_perm(xv[k][1][px >> 1], xv[k][0][px >> 1], sel);
                d.y = __builtin_amdgcn_perm(xv[k][3][px >> 1], xv[k][2][px >> 1], sel);
                d.z = __builtin_amdgcn_perm(xv[k][5][px >> 1], xv[k][4][px >> 1], sel);
                d.w = __builtin_amdgcn_perm(xv[k][7][px >> 1], xv[k][6][px >> 1], sel);
                *reinterpret_cast<uint4 *>(area + x_lds[k] + 16 * px) = d;
            }
        }
    };

    for (; sl < p.slices; sl += WAVES) {
        // The area is this wavefront's own, and its LDS accesses take effect in program order: what the fences keep in
        // order is the compiler.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        commit_x(sl);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int next = sl + WAVES;                      // (past the last one: every load out of range)
        hand_over(sl);
        uint32x4 fr[EARLY ? T : 1];
        if constexpr (EARLY) {
#pragma unroll
            for (int t = 0; t < T; ++t) fr[t] = cut(t);
        }
        issue_x(next);
        if constexpr (EARLY) issue_w(next);

        uint32x4 a[2][PXB];
        auto load = [&](int t) __attribute__((always_inline)) {
            const int off = (t / K * p.dh * p.pitch + t % K * p.dw) * 16;
#pragma unroll
            for (int pb = 0; pb < PXB; ++pb) a[t & 1][pb] = *reinterpret_cast<const uint32x4 *>(area + xa[pb] + off);
        };
        load(0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t + 1 < T) load(t + 1);
            uint32x4 b;
            if constexpr (PACKED) b = wl[t];
            else if constexpr (EARLY) b = fr[t];
            else b = cut(t);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pb = 0; pb < PXB; ++pb)
                acc[pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a[t & 1][pb]),
                                                                 __builtin_bit_cast(half8, b), acc[pb], 0, 0, 0);
            if constexpr (PACKED) issue_wp(next, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!PACKED && !EARLY) issue_w(next);
    }

    // ---- partial sums -> LDS (over the areas) -> 16-byte units of the output ----
    __syncthreads();
    float *st = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int pb = 0; pb < PXB; ++pb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // registers 4q .. 4q + 3 of a lane: pixels 8q + 4h .. + 3 of channel lane % 32
            const floatx4 v = {acc[pb][4 * q], acc[pb][4 * q + 1], acc[pb][4 * q + 2], acc[pb][4 * q + 3]};
            *reinterpret_cast<floatx4 *>(st + (wave * 32 + c32) * OPITCH + pb * 32 + 8 * q + 4 * h) = v;
        }
    __syncthreads();
    const half2v z = {(_Float16)0.0f, (_Float16)0.0f};
    const int live = min(WAVES, p.slices);                 // wavefronts that had a slice
    for (int u = tid; u < 32 * (TM / 8); u += NT) {
        const int c = u / (TM / 8), oc = cg * 32 + c;
        int px = m0 + 8 * (u % (TM / 8)), left = ohw - px;          // pixels that there are
        if (p.lg_tw != 0) {
            const int m = 8 * (u % (TM / 8)), oy = oyA + (m >> p.lg_tw), ox = oxA + (m & ((1 << p.lg_tw) - 1));
            px = oy * p.OW + ox;
            left = oy < p.OH ? p.OW - ox : 0;
        }
        if (left <= 0 || oc >= p.Cout) continue;
        float f[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) f[k] = 0.0f;
        for (int s = 0; s < live; ++s) {
            const floatx4 *src = reinterpret_cast<const floatx4 *>(st + (s * 32 + c) * OPITCH + 8 * (u % (TM / 8)));
            const floatx4 lo = src[0], hi = src[1];
#pragma unroll
            for (int k = 0; k < 4; ++k) { f[k] += lo[k]; f[4 + k] += hi[k]; }
        }
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            half2v e;
            e.x = (_Float16)f[2 * k]; e.y = (_Float16)f[2 * k + 1];
            if (p.relu) e = __builtin_elementwise_max(e, z);           // clipping the rounded value = rounding the clipped value
            o[k] = __builtin_bit_cast(uint32_t, e);
        }
        uint16_t *dst = y + ((size_t)n * p.Cout + oc) * ohw + px;
        if (left >= 8) {
            const uint4 v = make_uint4(o[0], o[1], o[2], o[3]);
            __builtin_memcpy(dst, &v, 16);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < left) dst[k] = (uint16_t)(o[k >> 1] >> (16 * (k & 1)));
        }
    }
}

// The operands of the kernel above in the order it takes them: [channel block][slice][tap][lane] of 16 bytes.
__global__ __launch_bounds__(256) void merit_conv2d_split_pack_w(SplitParams p, int T, const uint16_t *__restrict__ w,
                                                                 uint4 *__restrict__ packed, uint32_t units)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= units) return;
    const int lane = (int)(i & 63u);
    const uint32_t q = i >> 6, b = q / (uint32_t)T;
    const int t = (int)(q - b * (uint32_t)T);
    const int cg = (int)(b / (uint32_t)p.slices), sl = (int)(b - (uint32_t)cg * (uint32_t)p.slices);
    const int co = cg * 32 + (lane & 31), ci = min(sl * 16, p.Cin - 16) + (lane >> 5) * 8;
    uint32_t d[4] = {0, 0, 0, 0};
    if (co < p.Cout && ci >= sl * 16)                     // (a group of the slice before: zeros)
        for (int c = 0; c < 8; ++c)
            d[c >> 1] |= (uint32_t)w[((size_t)co * p.Cin + ci + c) * T + t] << (16 * (c & 1));
    packed[i] = make_uint4(d[0], d[1], d[2], d[3]);
}

namespace {

template <int K, int PXB, int XU, bool PACKED, bool RAGGED>
hipError_t launch_one(const SplitParams &p, const void *x, const void *w, void *y, hipStream_t s)
{
    static std::atomic<int> raised{0};
    void (*k)(SplitParams, const uint16_t *, const uint16_t *, uint16_t *) = merit_conv2d_split<K, PXB, XU, PACKED, RAGGED>;
    if (hipError_t e = raise_lds_limit_once(reinterpret_cast<const void *>(k), raised); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((uint32_t)(p.N * p.tiles * p.co_groups)), dim3(NT), (size_t)p.lds_bytes, s, p,
                       reinterpret_cast<const uint16_t *>(x), reinterpret_cast<const uint16_t *>(w),
                       reinterpret_cast<uint16_t *>(y));
    return hipGetLastError();
}

template <int K, int PXB, int XU>
hipError_t launch_form(const SplitParams &p, const void *x, const void *w, void *y, hipStream_t s, bool packed)
{
    if (p.Cin % 8 != 0) {
        if constexpr (XU == 0 || (PXB == 2 && XU == 2)) return hipErrorInvalidValue;       // (the planner makes no such plan)
        else return packed ? hipErrorInvalidValue : launch_one<K, PXB, XU, false, true>(p, x, w, y, s);
    }
    return packed ? launch_one<K, PXB, XU, true, false>(p, x, w, y, s) : launch_one<K, PXB, XU, false, false>(p, x, w, y, s);
}

template <int K, int PXB>
hipError_t launch_units(const SplitParams &p, const void *x, const void *w, void *y, hipStream_t s, bool packed)
{
    switch (p.xu) {
    case 0: return launch_form<K, PXB, 0>(p, x, w, y, s, packed);
    case 1: return launch_form<K, PXB, 1>(p, x, w, y, s, packed);
    case 2: return launch_form<K, PXB, 2>(p, x, w, y, s, packed);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_conv2d_split(const SplitParams &p, const void *x, const void *w, void *y, hipStream_t s, bool packed)
{
    if ((int64_t)p.N * p.tiles * p.co_groups == 0) return hipSuccess;
    switch (p.K * 10 + p.PXB) {
    case 31: return launch_units<3, 1>(p, x, w, y, s, packed);
    case 32: return launch_units<3, 2>(p, x, w, y, s, packed);
    case 51: return launch_units<5, 1>(p, x, w, y, s, packed);
    case 52: return launch_units<5, 2>(p, x, w, y, s, packed);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv2d_split_pack(const SplitParams &p, const void *w, void *packed, hipStream_t s)
{
    const int T = p.K * p.K;
    const uint32_t units = (uint32_t)((int64_t)p.co_groups * p.slices * T * 64);
    hipLaunchKernelGGL(merit_conv2d_split_pack_w, dim3((units + 255) / 256), dim3(256), 0, s, p, T,
                       reinterpret_cast<const uint16_t *>(w), reinterpret_cast<uint4 *>(packed), units);
    return hipGetLastError();
}

}  // namespace merit
