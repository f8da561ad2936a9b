// 2-D convolution for gfx950, windows of one pixel at stride 1: a matrix product per image.
//
// k = (n, co, p | ci) with p the pixel of the plane: y[n] = w . x[n], w [Cout][Cin], x[n] [Cin][H W] (Eq. 6 with a 1x1
// window, reduced with the dot product, Eq. 3, on v_mfma_f32_32x32x16_f16).
//
// A workgroup of eight wavefronts owns TM pixels x TN output channels of one image.  The input channels go through two
// LDS buffers in steps of 64.  What bounds these layers is not the matrix cores but the chain of a step -- memory round
// trip, LDS, barrier -- on launches that have one workgroup per compute unit, so:
//   * D steps are in flight in registers (16-byte loads, one to four per thread and step), issued D steps ahead;
//   * a step that the channels fill has no check, no select and no shift, and no branch lies round a load whose data
//     leaves it: where paths with different loads in flight meet, the compiler waits for all of them (1024 -> 256 on 8 of
//     14x14 8.5 us with such branches, with the loads of cut units shifted and with the last step's checks in every step,
//     5.6 without; the loads alone take 4.0);
//   * nothing is transposed by hand: the pixels of a channel lie in LDS as they lie in memory, and the operand a lane
//     feeds to the MFMA (eight channels of one pixel) comes out of ds_read_b64_tr_b16, which transposes on the way;
//   * all wavefronts load, and all multiply: where TM x TN has fewer than eight 32 x 32 blocks the wavefronts split
//     the 64 channels of each step instead (KS ways) and their partial sums meet in the fp32 staging area;
//   * workgroups are many and small, several to a compute unit, so that one's chain hides the other's.
// LDS rows are swizzled in 64-byte (pixels) and 16-byte (weights) chunks: the four rows of a transposing read and the
// sixteen rows of a weight read fall into different banks without padding.
//
// Planes of any size (H W >= 8): a 16-byte unit of eight pixels lies on any 2-byte boundary, which a global load or
// store takes; the unit that a plane's end would cut ends with the plane and has some pixels of the one before it once
// more.  Channels the same, but there the ones that come twice are zeroed.
//
// us a launch, the branches and shifts of before -> now (inputs from the Infinity Cache):
//   1024 -> 256 on 8 images of 14x14                8.5 -> 5.6      (24.6 on the wave-specialised multi-pass kernel)
//   256 -> 1024 on 8 of 14x14                       5.5 -> 4.2
//   1568 -> 392 on 3 of 25x17                       13.3 -> 9.2
//   392 -> 1568 on 3 of 25x17                       10.0 -> 7.4     (128 x 128 tiles; 8.4 on 128 x 64)
//   512 -> 128 on 25 of 53x19                       11.5 -> 9.7     (5.3 us at the copy rate)
//   576 -> 16 on 36x111                             5.7 -> 4.1
//   32 -> 64 on 32 of 64x64                         7.5 -> 6.7      (2.1 us at the copy rate; 8.2 on the multi-pass kernel)
// Tried: wavefronts that each split the channels and never meet before the sums (5.7 us on the first of these, 1.5-3x
// slower where the tiles fill the chip); six steps in flight, which is slower everywhere.
#include "merit_internal.h"

#include <atomic>

namespace merit {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int KB = 64;                     // input channels per step
constexpr int NT = 512;

// One 16-byte load, off in bytes on any 2-byte boundary.  A vector type throughout: a struct of four dwords the compiler
// splits into two 8-byte loads wherever a later step looks at its halves.
__device__ __forceinline__ u32x4 load16(const uint16_t *base, uint32_t off)
{
    typedef uint32_t u32x4_2 __attribute__((ext_vector_type(4), aligned(2)));
    return *reinterpret_cast<const u32x4_2 *>(reinterpret_cast<const uint8_t *>(base) + off);
}

// Eight pixels of a row to where they lie.  A unit that ends with the plane has some of the one before it: the same
// values once more, but for the added tensor's, which may be the output itself and which that unit's thread has read.
template <bool RES>
__device__ __forceinline__ void store_unit(uint16_t *row, int px, int HW, u32x4 v)
{
    uint16_t *dst = row + min(px, HW - 8);
    if (!RES || px + 8 <= HW) {
        __builtin_memcpy(dst, &v, 16);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (HW - 8 + k >= px) dst[k] = (uint16_t)(v[k >> 1] >> (16 * (k & 1)));
    }
}

// A unit of eight channels without its first `cut` ones, which the unit before it has (8 and more: all of them).
__device__ __forceinline__ u32x4 zero_first(u32x4 v, int cut)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] &= (2 * j >= cut ? 0xffffu : 0u) | (2 * j + 1 >= cut ? 0xffff0000u : 0u);
    return v;
}

// 64-byte chunk of a staged pixel row that row r keeps in place of chunk c
template <int TM>
__device__ __forceinline__ int xchunk(int c, int r)
{
    return TM >= 128 ? c ^ (r & 3) : (TM == 64 ? c ^ ((r >> 1) & 1) : c);
}

}  // namespace

// TM pixels x TN channels on WM x WN x KS = 8 wavefronts; D steps in flight; RES: an added tensor of the output's shape.
template <int TM, int TN, int WM, int WN, int KS, int D, int MINW, bool RES>
__global__ __launch_bounds__(NT, MINW) void merit_conv2d_px(PxParams p, const uint16_t *__restrict__ x,
                                                         const uint16_t *__restrict__ w, const uint16_t *res, uint16_t *y)
{
    static_assert(WM * WN * KS == 8, "eight wavefronts");
    constexpr int PXB = TM / (32 * WM), CHB = TN / (32 * WN);
    constexpr int XPITCH = TM * 2, XBYTES = KB * XPITCH, WBYTES = TN * KB * 2, BUF = XBYTES + WBYTES;
    constexpr int XUNITS = KB * TM / 8, WUNITS = TN * KB / 8;            // 16-byte units of a step
    constexpr int XU = (XUNITS + NT - 1) / NT, WU = (WUNITS + NT - 1) / NT;
    constexpr int U8 = TM / 8;                                          // units per pixel row
    constexpr int OPITCH = TM + 4, HPITCH = TM + 8;                     // staging: [KS][TN][OPITCH] floats, or [TN][HPITCH] halves
    constexpr int OUNITS = TN * U8, OU = (OUNITS + NT - 1) / NT;

    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, c32 = lane & 31;

    // channel blocks of one pixel tile are neighbours on one XCD: its L2 reads the tile once
    const int item = (int)xcd_band_item(blockIdx.x, p.xq, p.xr);
    const int tile = (int)fdiv((uint32_t)item, p.div_cog);
    const int co0 = (item - tile * p.co_groups) * TN;
    const int n = (int)fdiv((uint32_t)tile, p.div_tiles);
    const int px0 = (tile - n * p.tiles) * TM;
    const int HW = p.HW, Cin = p.Cin, nk_full = Cin / KB;
    const uint16_t *xn = x + (size_t)n * Cin * HW;

    // ---- what a thread loads of every step.  A unit of eight pixels that the plane's end would cut ends with the plane:
    // some of its pixels are computed, and stored, twice, the same ----
    int x_row[XU], x_lds[XU], w_k[WU], w_lds[WU];
    uint32_t x_px[XU], x_off[XU], w_off[WU];
#pragma unroll
    for (int i = 0; i < XU; ++i) {
        const int u = min(tid + NT * i, XUNITS - 1);
        const int r = u / U8, c = u % U8;
        x_row[i] = r;
        x_px[i] = 2u * (uint32_t)min(px0 + 8 * c, HW - 8);
        x_off[i] = (uint32_t)r * (2u * (uint32_t)HW) + x_px[i];
        x_lds[i] = r * XPITCH + (xchunk<TM>(c >> 2, r) << 6) + (c & 3) * 16;
    }
#pragma unroll
    for (int i = 0; i < WU; ++i) {
        const int u = min(tid + NT * i, WUNITS - 1);
        const int r = u / (KB / 8), c = u % (KB / 8);
        w_k[i] = 8 * c;
        w_off[i] = 2u * ((uint32_t)min(co0 + r, p.Cout - 1) * (uint32_t)Cin);         // (channels past Cout: never stored)
        w_lds[i] = XBYTES + r * (KB * 2) + ((c ^ ((r >> 1) & 7)) * 16);
    }

    u32x4 xr[D][XU], wr[D][WU];
    auto issue = [&](int s, int slot) __attribute__((always_inline)) {               // a whole step
        const uint16_t *xs = xn + (size_t)(s * KB) * HW, *ws = w + s * KB;
#pragma unroll
        for (int i = 0; i < XU; ++i) xr[slot][i] = load16(xs, x_off[i]);
#pragma unroll
        for (int i = 0; i < WU; ++i) wr[slot][i] = load16(ws, w_off[i] + 2u * w_k[i]);
    };
    auto commit = [&](int slot, int b) __attribute__((always_inline)) {
        uint8_t *buf = smem + b * BUF;
#pragma unroll
        for (int i = 0; i < XU; ++i)
            if (XUNITS % NT == 0 || tid + NT * i < XUNITS) *reinterpret_cast<u32x4 *>(buf + x_lds[i]) = xr[slot][i];
#pragma unroll
        for (int i = 0; i < WU; ++i)
            if (WUNITS % NT == 0 || tid + NT * i < WUNITS) *reinterpret_cast<u32x4 *>(buf + w_lds[i]) = wr[slot][i];
    };
    // the step that the channels do not fill: no loads, no staging and no MFMAs for rows of which none exists (a third
    // of the time of a layer on 32 channels)
    const int k_rest = nk_full * KB;
    auto issue_rest = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < XU; ++i)
            if (k_rest + NT * i / U8 < Cin) {
                const int u8 = k_rest + (x_row[i] & ~7), ch = min(u8, Cin - 8) + (x_row[i] & 7);
                xr[slot][i] = load16(xn, (uint32_t)ch * (2u * (uint32_t)HW) + x_px[i]);
            }
#pragma unroll
        for (int i = 0; i < WU; ++i) wr[slot][i] = load16(w, w_off[i] + 2u * (uint32_t)min(k_rest + w_k[i], Cin - 8));
    };
    auto commit_rest = [&](int slot, int b) __attribute__((always_inline)) {
        uint8_t *buf = smem + b * BUF;
#pragma unroll
        for (int i = 0; i < XU; ++i) {
            if (k_rest + NT * i / U8 >= ((Cin + 15) & ~15)) continue;
            const int u8 = k_rest + (x_row[i] & ~7);
            const bool ok = u8 < Cin && min(u8, Cin - 8) + (x_row[i] & 7) >= u8;
            u32x4 v = xr[slot][i];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = ok ? v[j] : 0u;
            if (XUNITS % NT == 0 || tid + NT * i < XUNITS) *reinterpret_cast<u32x4 *>(buf + x_lds[i]) = v;
        }
#pragma unroll
        for (int i = 0; i < WU; ++i) {
            const u32x4 v = zero_first(wr[slot][i], max(k_rest + w_k[i] + 8 - Cin, 0));
            if (WUNITS % NT == 0 || tid + NT * i < WUNITS) *reinterpret_cast<u32x4 *>(buf + w_lds[i]) = v;
        }
    };

    // ---- what a wavefront multiplies ----
    const int wk = wave % KS, wm = (wave / KS) % WM, wn = wave / (KS * WM);
    int xa[PXB], wa[CHB], wsw[CHB];
#pragma unroll
    for (int pb = 0; pb < PXB; ++pb) {
        // lane address of a transposing read: row (lane & 15) / 4 of the four, 8 bytes of the 32 pixels' 64
        const int r = 8 * h + ((lane & 15) >> 2);
        const int col = (wm * PXB + pb) * 64;                                          // bytes
        xa[pb] = r * XPITCH + (xchunk<TM>(col >> 6, r) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    }
#pragma unroll
    for (int cb = 0; cb < CHB; ++cb) {
        const int r = (wn * CHB + cb) * 32 + c32;
        wa[cb] = XBYTES + r * (KB * 2);
        wsw[cb] = (r >> 1) & 7;
    }
    floatx16 acc[CHB][PXB];
#pragma unroll
    for (int cb = 0; cb < CHB; ++cb)
#pragma unroll
        for (int pb = 0; pb < PXB; ++pb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][pb][r] = 0.0f;

    auto multiply = [&](int s, int b, bool last) __attribute__((always_inline)) {
        uint8_t *buf = smem + b * BUF;
        constexpr int STEPS = KB / 16 / KS;
        half8 a[2][PXB], bw[2][CHB];
        auto load = [&](int t) __attribute__((always_inline)) {
            const int st = wk * STEPS + t;
#pragma unroll
            for (int pb = 0; pb < PXB; ++pb) {
                typedef __attribute__((address_space(3))) short4v *lds4;
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(buf + xa[pb] + (16 * st) * XPITCH));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(buf + xa[pb] + (16 * st + 4) * XPITCH));
                a[t & 1][pb] = __builtin_bit_cast(half8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
            for (int cb = 0; cb < CHB; ++cb)
                bw[t & 1][cb] = *reinterpret_cast<const half8 *>(buf + wa[cb] + (((2 * st + h) ^ wsw[cb]) << 4));
        };
        // the reads of step t + 1 are issued before the MFMAs of step t, and no others (all at once they spill)
        if (last && s * KB + 16 * wk * STEPS >= Cin) return;
        load(0);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (last && s * KB + 16 * (wk * STEPS + t) >= Cin) break;
            if (t + 1 < STEPS) load(t + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int cb = 0; cb < CHB; ++cb)
#pragma unroll
                for (int pb = 0; pb < PXB; ++pb)
                    acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[t & 1][pb], bw[t & 1][cb], acc[cb][pb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- the steps: what the channels leave over first, then the whole ones in groups of D, the next group's loads going
    // out as this one's registers come free.  No branch round a load whose data is not used inside it: where paths with
    // different loads in flight meet, the compiler waits for all of them. ----
    u32x4 rr[RES ? OU : 1];
    auto load_added = [&]() __attribute__((always_inline)) {
        if constexpr (RES) {
#pragma unroll
            for (int i = 0; i < OU; ++i) {
                const int u = min(tid + NT * i, OUNITS - 1);
                const int c = u / U8, px = px0 + 8 * (u % U8);
                rr[i] = load16(res + (size_t)n * p.Cout * HW,
                               2u * ((uint32_t)min(co0 + c, p.Cout - 1) * (uint32_t)HW + (uint32_t)min(px, HW - 8)));
            }
        }
    };
    const bool rest = k_rest < Cin;
    if (nk_full == 0) {
        issue_rest(0);
        load_added();
        commit_rest(0, 0);                                              // (the only step has the only buffer)
        __syncthreads();
        multiply(0, 0, true);
    } else {
        const int last = nk_full - 1;
        if (rest) issue_rest(D - 1);
#pragma unroll
        for (int i = 0; i < D - 1; ++i) issue(min(i, last), i);
        if (rest) commit_rest(D - 1, 1);
        issue(min(D - 1, last), D - 1);
        load_added();
        if (rest) {
            __syncthreads();
            multiply(nk_full, 1, true);
        }
        int s = 0;
        for (; s + D < nk_full; s += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                commit(i, (s + i) & 1);
                issue(min(s + i + D, last), i);
                __syncthreads();
                multiply(s + i, (s + i) & 1, false);
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (s + i < nk_full) {
                commit(i, (s + i) & 1);
                __syncthreads();
                multiply(s + i, (s + i) & 1, false);
            }
        }
    }

    // ---- sums -> staging [channel][pixel] (over the buffers) -> 16-byte units to memory.  Whole sums that nothing is
    // added to are rounded on the way in; partial ones, or an added tensor's, are staged in fp32 ----
    __syncthreads();
    constexpr bool HALF = KS == 1 && !RES;
    float *st = reinterpret_cast<float *>(smem);
    const half2v z = {(_Float16)0.0f, (_Float16)0.0f};
    auto rounded = [&](float a, float b) __attribute__((always_inline)) {
        half2v e;
        e.x = (_Float16)a; e.y = (_Float16)b;
        if (p.relu) e = __builtin_elementwise_max(e, z);             // clipping the rounded value = rounding the clipped value
        return __builtin_bit_cast(uint32_t, e);
    };
#pragma unroll
    for (int cb = 0; cb < CHB; ++cb)
#pragma unroll
        for (int pb = 0; pb < PXB; ++pb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // registers 4q .. 4q + 3 of a lane: pixels 8q + 4h .. + 3 of channel lane % 32
                const int ch = (wn * CHB + cb) * 32 + c32, px = (wm * PXB + pb) * 32 + 8 * q + 4 * h;
                const floatx4 v = {acc[cb][pb][4 * q], acc[cb][pb][4 * q + 1], acc[cb][pb][4 * q + 2], acc[cb][pb][4 * q + 3]};
                if constexpr (HALF)
                    *reinterpret_cast<uint2 *>(smem + (ch * HPITCH + px) * 2) = make_uint2(rounded(v[0], v[1]), rounded(v[2], v[3]));
                else
                    *reinterpret_cast<floatx4 *>(st + (wk * TN + ch) * OPITCH + px) = v;
            }
    __syncthreads();
    uint16_t *yn = y + (size_t)n * p.Cout * HW;
#pragma unroll
    for (int i = 0; i < OU; ++i) {
        const int u = tid + NT * i;
        const int c = u / U8, px = px0 + 8 * (u % U8), co = co0 + c;
        if ((OUNITS % NT != 0 && u >= OUNITS) || px >= HW || co >= p.Cout) continue;
        u32x4 o;
        if constexpr (HALF) {
            o = *reinterpret_cast<const u32x4 *>(smem + (c * HPITCH + 8 * (u % U8)) * 2);
        } else {
            float f[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) f[k] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const floatx4 *src = reinterpret_cast<const floatx4 *>(st + (ks * TN + c) * OPITCH + 8 * (u % U8));
                const floatx4 a = src[0], b = src[1];
#pragma unroll
                for (int k = 0; k < 4; ++k) { f[k] += a[k]; f[4 + k] += b[k]; }
            }
            if constexpr (RES) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t d = rr[i][k];             // (a cast of the vector's element itself takes element 0)
                    const half2v e = __builtin_bit_cast(half2v, d);
                    f[2 * k] += (float)e.x; f[2 * k + 1] += (float)e.y;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = rounded(f[2 * k], f[2 * k + 1]);
        }
        store_unit<RES>(yn + (size_t)co * HW, px, HW, o);
    }
}

namespace {

template <int TM, int TN, int WM, int WN, int KS, int D, int MINW, bool RES>
hipError_t launch_one(const PxParams &p, const void *x, const void *w, const void *res, void *y, hipStream_t s)
{
    static std::atomic<int> raised{0};
    const size_t lds = px_lds_bytes(p);
    const auto k = merit_conv2d_px<TM, TN, WM, WN, KS, D, MINW, RES>;
    if (hipError_t e = raise_lds_limit_once(reinterpret_cast<const void *>(k), raised); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((uint32_t)(p.N * p.tiles * p.co_groups)), dim3(NT), lds, s, p,
                       reinterpret_cast<const uint16_t *>(x), reinterpret_cast<const uint16_t *>(w),
                       reinterpret_cast<const uint16_t *>(res), reinterpret_cast<uint16_t *>(y));
    return hipGetLastError();
}

template <int TM, int TN, int WM, int WN, int KS, int D, int MINW>
hipError_t launch_tile(const PxParams &p, const void *x, const void *w, const void *res, void *y, hipStream_t s)
{
    if (res) return launch_one<TM, TN, WM, WN, KS, D, MINW, true>(p, x, w, res, y, s);
    return launch_one<TM, TN, WM, WN, KS, D, MINW, false>(p, x, w, res, y, s);
}

}  // namespace

size_t px_lds_bytes(const PxParams &p)
{
    const size_t bufs = (p.nk > 1 ? 2 : 1) * (size_t)KB * 2 * (p.TM + p.TN);
    const size_t blocks = (size_t)(p.TM / 32) * (p.TN / 32);
    const size_t ks = blocks >= 8 ? 1 : 8 / blocks;
    const size_t staging = ks == 1 && !p.residual ? (size_t)p.TN * (p.TM + 8) * 2 : ks * p.TN * (p.TM + 4) * 4;
    return bufs > staging ? bufs : staging;
}

__global__ __launch_bounds__(256) void merit_conv2d_copy_w(const uint4 *__restrict__ w, uint4 *__restrict__ packed, uint32_t n)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < n) packed[i] = w[i];
}

hipError_t launch_copy_weights(const void *w, void *packed, int64_t halves, hipStream_t s)
{
    const uint32_t n = (uint32_t)(halves / 8);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(merit_conv2d_copy_w, dim3((n + 255) / 256), dim3(256), 0, s, reinterpret_cast<const uint4 *>(w),
                       reinterpret_cast<uint4 *>(packed), n);
    return hipGetLastError();
}

hipError_t launch_conv2d_px(const PxParams &p, const void *x, const void *w, const void *res, void *y, hipStream_t s)
{
    if ((p.residual != 0) != (res != nullptr)) return hipErrorInvalidValue;
    if ((int64_t)p.N * p.tiles * p.co_groups == 0) return hipSuccess;
    switch (p.TM * 1000 + p.TN) {
    case 64032: return launch_tile<64, 32, 2, 1, 4, 4, 4>(p, x, w, res, y, s);
    case 64064: return launch_tile<64, 64, 2, 2, 2, 3, 4>(p, x, w, res, y, s);
    case 64128: return launch_tile<64, 128, 2, 4, 1, 2, 4>(p, x, w, res, y, s);
    case 128032: return launch_tile<128, 32, 4, 1, 2, 1, 6>(p, x, w, res, y, s);
    case 128064:          // (with the added tensor's 16 registers, two workgroups per compute unit instead of three)
        if (res) return launch_one<128, 64, 4, 2, 1, 2, 4, true>(p, x, w, res, y, s);
        return launch_one<128, 64, 4, 2, 1, 1, 6, false>(p, x, w, res, y, s);
    case 128128: return launch_tile<128, 128, 4, 2, 1, 1, 4>(p, x, w, res, y, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace merit
