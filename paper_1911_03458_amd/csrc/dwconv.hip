// Depthwise convolution for gfx950: k = (n, c, oy, ox | ky, kx),
//     M(x)[p,a] = x[n, c, oy*sh + ky - ph, ox*sw + kx - pw]      (0 outside the image)
//     M(w)[p,a] = w[c, ky, kx]
// reduced with the dot product (Section III-B, Eq. 3).  The channel index is parallel, so
// there is no contraction for the matrix cores: the op moves 4 bytes per output element and
// does kh*kw multiply-adds on them — HBM-bound, plain vector arithmetic in fp32.
//
// A workgroup owns TH output rows of one (n,c) plane.  The input rows they need are one
// contiguous span of the plane (the minimal covering sub-tensor of Section IV-A, Eq. 9),
// staged in LDS with the zero padding resolved there; windows are then read branch-free.
#include "merit_internal.h"

namespace merit {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float h2f(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

__device__ __forceinline__ uint16_t f2h(float f)
{
    const _Float16 h = (_Float16)f;                        // round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}

// ---------------------------------------------------------------------------
// Generic kernel: any window / stride / padding / width; scalar accesses.
// LDS: [RH][pitch] halves, pitch = W + 2*pw, then the kh*kw weights as floats.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void merit_dwconv_tile(DwParams p, const uint16_t *__restrict__ x,
                                                        const uint16_t *__restrict__ w, uint16_t *__restrict__ y)
{
    extern __shared__ __align__(16) uint8_t smem[];
    uint16_t *xl = reinterpret_cast<uint16_t *>(smem);
    float *wf = reinterpret_cast<float *>(smem + p.lds_w_offset);

    const int tid = threadIdx.x;
    const uint32_t nc = fdiv(blockIdx.x, p.div_tiles_y);
    const int strip = (int)(blockIdx.x - nc * (uint32_t)p.tiles_y);
    const int c = (int)(nc - fdiv(nc, p.div_c) * (uint32_t)p.C);
    const int oy0 = strip * p.TH;
    const int y0 = oy0 * p.sh - p.ph;
    const int rows = min(p.TH, p.OH - oy0);
    const int RH = (rows - 1) * p.sh + p.kh;
    const uint16_t *xp = x + (size_t)nc * p.H * p.W;

    for (int i = tid; i < p.kh * p.kw; i += 256) wf[i] = h2f(w[(size_t)c * p.kh * p.kw + i]);
    for (int i = tid; i < RH * p.pitch; i += 256) {
        const int r = (int)fdiv((uint32_t)i, p.div_pitch);
        const int col = i - r * p.pitch;
        const int gy = y0 + r, gx = col - p.pw;
        uint16_t v = 0;
        if (gy >= 0 && gy < p.H && gx >= 0 && gx < p.W) v = xp[(size_t)gy * p.W + gx];
        xl[i] = v;
    }
    __syncthreads();

    uint16_t *yp = y + (size_t)nc * p.OH * p.OW;
    for (int o = tid; o < rows * p.OW; o += 256) {
        const int ty = (int)fdiv((uint32_t)o, p.div_ow);
        const int ox = o - ty * p.OW;
        const uint16_t *win = xl + (ty * p.sh) * p.pitch + ox * p.sw;
        float acc = 0.0f;
        for (int ky = 0; ky < p.kh; ++ky)
            for (int kx = 0; kx < p.kw; ++kx) acc = fmaf(h2f(win[ky * p.pitch + kx]), wf[ky * p.kw + kx], acc);
        yp[(size_t)(oy0 + ty) * p.OW + ox] = f2h(acc);
    }
}

// ---------------------------------------------------------------------------
// 3x3, stride 1, padding 1, W % 8 == 0 (the MobileNet layer).  LDS rows are
// [8 zero halves][W halves][8 zero halves], so every 16-byte chunk is aligned; rows are
// copied with 16-byte loads.  A thread makes 8 adjacent outputs from three aligned 16-byte
// reads per window row (it needs the last half of the chunk on its left, its own chunk and
// the first half of the chunk on its right) and stores them as one 16-byte run.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void merit_dwconv_rows_k3s1p1(DwParams p, const uint16_t *__restrict__ x,
                                                               const uint16_t *__restrict__ w,
                                                               uint16_t *__restrict__ y)
{
    extern __shared__ __align__(16) uint8_t smem[];
    uint4 *xl = reinterpret_cast<uint4 *>(smem);            // [RH][pitch8] chunks of 8 halves
    const int tid = threadIdx.x;
    const uint32_t nc = fdiv(blockIdx.x, p.div_tiles_y);
    const int strip = (int)(blockIdx.x - nc * (uint32_t)p.tiles_y);
    const int c = (int)(nc - fdiv(nc, p.div_c) * (uint32_t)p.C);
    const int oy0 = strip * p.TH;
    const int rows = min(p.TH, p.OH - oy0);
    const int RH = rows + 2;
    const int W8 = p.W >> 3, pitch8 = W8 + 2;
    const uint16_t *xp = x + (size_t)nc * p.H * p.W;

    // weights: nine wave-uniform loads
    float wk[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) wk[i] = h2f(w[(size_t)c * 9 + i]);

    // batches of SB chunks per thread, every load issued before the first LDS write (one memory
    // round trip per batch); a chunk outside the plane re-reads the plane's first bytes and is zeroed
    constexpr int SB = 4;
    const int total = RH * pitch8;
    for (int i0 = tid; i0 < total; i0 += 256 * SB) {
        uint4 v[SB];
        bool in[SB];
#pragma unroll
        for (int b = 0; b < SB; ++b) {
            const int i = min(i0 + 256 * b, total - 1);
            const int r = (int)fdiv((uint32_t)i, p.div_pitch);
            const int c8 = i - r * pitch8;                  // 0 and W8+1 are the zero chunks
            const int gy = oy0 - 1 + r;
            in[b] = gy >= 0 && gy < p.H && c8 >= 1 && c8 <= W8;
            v[b] = *reinterpret_cast<const uint4 *>(in[b] ? xp + (size_t)gy * p.W + 8 * (c8 - 1) : xp);
        }
#pragma unroll
        for (int b = 0; b < SB; ++b)
            if (i0 + 256 * b < total) xl[i0 + 256 * b] = in[b] ? v[b] : make_uint4(0, 0, 0, 0);
    }
    __syncthreads();

    uint16_t *yp = y + (size_t)nc * p.OH * p.OW;
    for (int o = tid; o < rows * W8; o += 256) {
        const int ty = (int)fdiv((uint32_t)o, p.div_ow);     // div_ow holds W8 for this variant
        const int x8 = o - ty * W8;
        float acc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
            const uint4 *row = xl + (ty + ky) * pitch8 + x8;  // chunks x8 (left), x8+1 (own), x8+2 (right)
            const half8 l = __builtin_bit_cast(half8, row[0]);
            const half8 m = __builtin_bit_cast(half8, row[1]);
            const half8 r = __builtin_bit_cast(half8, row[2]);
            float v[10];
            v[0] = (float)l[7];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[1 + k] = (float)m[k];
            v[9] = (float)r[0];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) acc[k] = fmaf(v[k + kx], wk[ky * 3 + kx], acc[k]);
        }
        uint4 out;
        out.x = (uint32_t)f2h(acc[0]) | ((uint32_t)f2h(acc[1]) << 16);
        out.y = (uint32_t)f2h(acc[2]) | ((uint32_t)f2h(acc[3]) << 16);
        out.z = (uint32_t)f2h(acc[4]) | ((uint32_t)f2h(acc[5]) << 16);
        out.w = (uint32_t)f2h(acc[6]) | ((uint32_t)f2h(acc[7]) << 16);
        *reinterpret_cast<uint4 *>(yp + (size_t)(oy0 + ty) * p.OW + 8 * x8) = out;
    }
}

// ---------------------------------------------------------------------------
// K x K windows (3 or 5) at stride S (1 or 2), any padding, any width: no LDS, no barrier.
//
// A thread makes QW = 8 / S adjacent outputs of TR rows.  Bound by memory and by the launch on all but the largest of
// these layers, so what counts is few, wide, early loads: the input columns an output row needs are one 16-byte load
// and one of 4 or 8 bytes per input row, on any 2-byte boundary, all rows requested before the first is used; what lies
// outside the plane is masked to zero.  The last unit of a row starts earlier where it would be cut (the outputs it
// shares with its neighbour are stored twice, with the same values), so every store is whole, but for rows of fewer
// outputs than a unit.
// us a launch, merit_dwconv_tile or TR = 4 throughout -> this: 1x24x96x80 5x5 / 2 4.8 -> 3.0, 4x192x16x28 3x3 4.2 -> 2.9,
// 31x64x15x10 3x3 4.3 -> 2.8, 1x176x90x20 5x5 5.0 -> 3.3, 7x336x9x83 5x5 8.1 -> 5.9, 8x96x112x112 3x3 / 2 8.3 (4.0 at the copy
// rate).  On rows of whole 16-byte chunks merit_dwconv_rows_k3s1p1 keeps the 3x3 layer (32x32x64x64: 5.5 against 6.3).
// TR: 1, 2 or 4, by the launch's size (the plan); the rows that strips share are read by both, from L2.
// ---------------------------------------------------------------------------
template <int K, int S, int TR>
__global__ __launch_bounds__(256) void merit_dwconv_lanes(DwParams p, const uint16_t *__restrict__ x,
                                                         const uint16_t *__restrict__ w, uint16_t *__restrict__ y)
{
    constexpr int QW = 8 / S;                              // outputs of a row
    constexpr int L = (QW - 1) * S + K;                    // input columns they need: 10, 12, 9, 11
    constexpr int D = (L + 1) / 2;                         // dwords loaded per row: 5, 6, 5, 6
    constexpr int RH = (TR - 1) * S + K;                   // input rows

    const uint32_t item = xcd_band_item(blockIdx.x, p.xq, p.xr) * 256u + threadIdx.x;
    if (item >= (uint32_t)p.items) return;
    const uint32_t q = fdiv(item, p.div_units);            // (plane, strip)
    const int u = (int)(item - q * (uint32_t)p.units);
    const uint32_t nc = fdiv(q, p.div_tiles_y);
    const int oy0 = (int)(q - nc * (uint32_t)p.tiles_y) * TR;
    const int ox0 = max(min(u * QW, p.OW - QW), 0);        // (rows of fewer outputs: one unit, stored one by one)
    const int c = (int)(nc - fdiv(nc, p.div_c) * (uint32_t)p.C);
    const int gx0 = ox0 * S - p.pw, gy0 = oy0 * S - p.ph;

    // which of the 2 D halves are inside the row
    uint32_t mask[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int a = gx0 + 2 * d, b = a + 1;
        mask[d] = (a >= 0 && a < p.W ? 0x0000ffffu : 0u) | (b >= 0 && b < p.W ? 0xffff0000u : 0u);
    }
    const int total = p.NC * p.H * p.W;                    // (below 2^31: the planner)
    const int plane = (int)nc * p.H * p.W;
    uint32_t v[RH][D];
    int moved[RH];                                         // halves by which a load was moved to stay inside the tensor
#pragma unroll
    for (int r = 0; r < RH; ++r) {
        const int e = plane + min(max(gy0 + r, 0), p.H - 1) * p.W + gx0;
        const int at = min(max(e, 0), total - 2 * D);
        moved[r] = e - at;
        __builtin_memcpy(v[r], x + at, 4 * D);
    }
    uint16_t wh[K * K];
    __builtin_memcpy(wh, w + c * K * K, 2 * K * K);
    float wk[K * K];
#pragma unroll
    for (int i = 0; i < K * K; ++i) wk[i] = h2f(wh[i]);
    // the tensor's first and last units: back to where they belong, a half at a time (what comes in is masked)
    bool any = false;
#pragma unroll
    for (int r = 0; r < RH; ++r) any |= moved[r] != 0;
    if (any) {
#pragma unroll
        for (int r = 0; r < RH; ++r) {
            for (int m = moved[r]; m > 0; --m) {
#pragma unroll
                for (int d = 0; d < D; ++d) v[r][d] = (v[r][d] >> 16) | (d + 1 < D ? v[r][d + 1] << 16 : 0u);
            }
            for (int m = moved[r]; m < 0; ++m) {
#pragma unroll
                for (int d = D - 1; d >= 0; --d) v[r][d] = (v[r][d] << 16) | (d > 0 ? v[r][d - 1] >> 16 : 0u);
            }
        }
    }

    float acc[TR][QW];
#pragma unroll
    for (int t = 0; t < TR; ++t)
#pragma unroll
        for (int k = 0; k < QW; ++k) acc[t][k] = 0.0f;
#pragma unroll
    for (int r = 0; r < RH; ++r) {
        const bool in = gy0 + r >= 0 && gy0 + r < p.H;
        float f[2 * D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const uint32_t m = in ? v[r][d] & mask[d] : 0u;
            f[2 * d] = h2f((uint16_t)m);
            f[2 * d + 1] = h2f((uint16_t)(m >> 16));
        }
#pragma unroll
        for (int t = 0; t < TR; ++t) {
            const int ky = r - t * S;                      // an output's rows arrive in window scan order
            if (ky < 0 || ky >= K) continue;
#pragma unroll
            for (int k = 0; k < QW; ++k)
#pragma unroll
                for (int kx = 0; kx < K; ++kx) acc[t][k] = fmaf(f[k * S + kx], wk[ky * K + kx], acc[t][k]);
        }
    }
    uint16_t *yp = y + (size_t)nc * p.OH * p.OW + ox0;
#pragma unroll
    for (int t = 0; t < TR; ++t) {
        if (oy0 + t >= p.OH) break;
        uint32_t o[QW / 2];
#pragma unroll
        for (int k = 0; k < QW / 2; ++k) o[k] = (uint32_t)f2h(acc[t][2 * k]) | ((uint32_t)f2h(acc[t][2 * k + 1]) << 16);
        uint16_t *dst = yp + (size_t)(oy0 + t) * p.OW;
        if (p.OW >= QW) {
            __builtin_memcpy(dst, o, 2 * QW);
        } else {
#pragma unroll
            for (int k = 0; k < QW; ++k)
                if (k < p.OW) dst[k] = (uint16_t)(o[k >> 1] >> (16 * (k & 1)));
        }
    }
}

hipError_t launch_dwconv(const DwParams &p, const void *x, const void *w, void *y, hipStream_t s)
{
    const int64_t grid = p.variant == DW_LANES ? ((int64_t)p.items + 255) / 256 : (int64_t)p.NC * p.tiles_y;
    if (grid == 0) return hipSuccess;
    const uint16_t *xs = reinterpret_cast<const uint16_t *>(x);
    const uint16_t *ws = reinterpret_cast<const uint16_t *>(w);
    uint16_t *ys = reinterpret_cast<uint16_t *>(y);
    if (p.lds_bytes > 64 * 1024) {     // wide rows: more dynamic LDS than a kernel gets by default
        static std::atomic<int> raised_rows{0}, raised_tile{0};
        const bool rows = p.variant == DW_ROWS_K3S1P1;
        if (hipError_t e = raise_lds_limit_once(rows ? reinterpret_cast<const void *>(merit_dwconv_rows_k3s1p1)
                                                     : reinterpret_cast<const void *>(merit_dwconv_tile),
                                                rows ? raised_rows : raised_tile);
            e != hipSuccess)
            return e;
    }
    if (p.variant == DW_LANES) {
        const dim3 g((uint32_t)grid), b(256);
#define MERIT_DW_LANES(K, S)                                                                                     \
    case K * 10 + S:                                                                                             \
        if (p.TH == 1) hipLaunchKernelGGL((merit_dwconv_lanes<K, S, 1>), g, b, 0, s, p, xs, ws, ys);             \
        else if (p.TH == 2) hipLaunchKernelGGL((merit_dwconv_lanes<K, S, 2>), g, b, 0, s, p, xs, ws, ys);        \
        else hipLaunchKernelGGL((merit_dwconv_lanes<K, S, 4>), g, b, 0, s, p, xs, ws, ys);                       \
        break
        switch (p.kw * 10 + p.sw) {
        MERIT_DW_LANES(3, 1);
        MERIT_DW_LANES(3, 2);
        MERIT_DW_LANES(5, 1);
        MERIT_DW_LANES(5, 2);
        default: return hipErrorInvalidValue;
        }
#undef MERIT_DW_LANES
        return hipGetLastError();
    }
    if (p.variant == DW_ROWS_K3S1P1)
        hipLaunchKernelGGL(merit_dwconv_rows_k3s1p1, dim3((uint32_t)grid), dim3(256), (size_t)p.lds_bytes, s, p, xs, ws, ys);
    else
        hipLaunchKernelGGL(merit_dwconv_tile, dim3((uint32_t)grid), dim3(256), (size_t)p.lds_bytes, s, p, xs, ws, ys);
    return hipGetLastError();
}

const char *dwconv_kernel_name(const DwParams &p)
{
    if (p.variant == DW_LANES) return "merit_dwconv_lanes";
    return p.variant == DW_ROWS_K3S1P1 ? "merit_dwconv_rows_k3s1p1" : "merit_dwconv_tile";
}

}  // namespace merit
