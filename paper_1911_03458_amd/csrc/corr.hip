// Correlation layer for gfx950 (Section III-C, Eq. 8):
//     M(I1)[p,a] = I1[b, a1, p1, p2]
//     M(I2)[p,a] = I2[b, a1, p1 + (p3-R)*sd, p2 + (p4-R)*sd]      (0 outside the image)
// with k = (b, p1, p2, p3, p4 | a1) and the dot product over the channel index a1
// (Section III-B, Eq. 3).  Output y[b,p1,p2,p3,p4], binary16, fp32 accumulation.
//
// A workgroup owns (b, p1, p3, a run of 64 pixels p2, or what a narrower image has): one row of
// the first tensor and one (displaced) row of the second.  For that pair of rows the layer is a banded matrix product:
// with the pixels p2 as rows, the columns q of the second row as columns and the channels as
// the reduction axis, D = X1^T X2 holds y[.., p2, p3, p4] at q = p2 + (p4-R)*sd.  Only columns
// congruent to p2 modulo sd are ever needed, so a block of 16 pixels of one residue class is
// multiplied with the 16+2R columns of the same class around it, in blocks of 16
// (v_mfma_f32_16x16x32_f16, a third of the products are wanted ones at R = 5); the matrix
// cores do in a few hundred cycles what the vector dot products took most of the kernel for.
// Both rows are staged in LDS with the channel axis innermost, eight channels = 16 bytes per
// pixel, transposed in registers on the way (v_perm_b32): exactly the operand a lane feeds to
// the MFMA.  Positions are ordered by residue class so that the 16 pixels of a block are
// adjacent.  Channels go through LDS in passes of `chg` groups of eight; the loads of the next
// pass are in flight while the current one is multiplied.  Needs W >= 8, R <= 15, sd <= 8.
// Rows of any width: a unit's eight pixels lie on any 2-byte boundary (a 16-byte global load needs no more), and the unit
// that the row's end cuts ends with the row, which keeps every load inside the tensor.
// What bounds it: not the matrix cores but a pass's chain of loads, LDS writes and barriers, and on 256 channels the rows
// themselves, each of which 2R+1 workgroups stage.  So the loads go out together (with the zeroing beside them each waited
// for its own round trip), only by lanes that have something to load, and on many channels the writes fall into all bank
// groups.  us a launch of 20 in a graph, before -> with that: 256 channels at 64x64, +-5 at stride 2: 9.0 -> 7.3; 208 at
// 63x46, +-3: 7.8 -> 5.9; 80 at 64x58, +-4: 6.1 -> 5.0; 48 at 52x40, +-5: 4.6 -> 4.4; 40 at 33x18, +-3: 3.8 -> 3.8; 1.12x
// over 400 images of 8 to 150 pixels a side, of which six (the shortest launches, 3.5 us) lost 4 to 6 %.
#include "merit_internal.h"

namespace merit {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16 bytes on a 16-byte boundary, or on any 2-byte one
template <bool ANY>
__device__ __forceinline__ u32x4 load16(const uint8_t *src)
{
    typedef uint32_t u32x4_2 __attribute__((ext_vector_type(4), aligned(2)));
    if constexpr (ANY) return *reinterpret_cast<const u32x4_2 *>(src);
    else return *reinterpret_cast<const u32x4 *>(src);
}

// Where item `at` (a pixel's eight channels, 16 bytes) of channel group g lies in its staged row.  The lanes of a write are
// eight items apart, two bank groups of the sixteen: with ROT each run of eight is rotated by its place and its group.
template <bool ROT>
__device__ __forceinline__ int corr_slot(int at, int g)
{
    return ROT ? (at & ~7) | ((at + (at >> 3) + g) & 7) : at;
}

static_assert(CORR_XB == 1, "a thread stages one unit a pass");

// NB = 16-column blocks of the second row per pixel block, BPW = pixel blocks per wavefront, RAGGED = W % 8 != 0.  ROT: the
// plan's choice (CorrParams::rot); what it costs where it does not pay are the instructions, so an instance of its own.
template <int NB, int BPW, bool RAGGED, bool ROT>
__global__ __launch_bounds__(256, 4) void merit_corr_mfma(CorrParams p, const uint16_t *__restrict__ x1,
                                                       const uint16_t *__restrict__ x2, uint16_t *__restrict__ y)
{
    extern __shared__ __align__(16) uint8_t smem[];
    uint4 *a1l = reinterpret_cast<uint4 *>(smem);                 // [chg][P1]
    uint4 *a2l = a1l + p.chg * p.P1;                              // [chg][P2]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each XCD takes a band of image rows: its L2 then fetches that band and its halo rows of
    // the second tensor, not both whole tensors
    uint32_t g = xcd_band_item(blockIdx.x, p.xq, p.xr);
    // work item -> (b, p1, p3, pixel chunk), chunk fastest
    const uint32_t q0 = fdiv(g, p.div_xchunks);
    const int xc = (int)(g - q0 * (uint32_t)p.xchunks);
    const uint32_t q1 = fdiv(q0, p.div_n);
    const int p3 = (int)(q0 - q1 * (uint32_t)p.n);
    const int b = (int)fdiv(q1, p.div_h);
    const int p1 = (int)(q1 - (uint32_t)b * (uint32_t)p.H);

    const int px0 = xc * 64, yy = p1 + (p3 - p.R) * p.sd;
    const bool rowok = yy >= 0 && yy < p.H;
    const int wchunk = min(64, p.W - px0);                        // pixels of this chunk

    // The staging unit of this thread, the same in every pass: 8 adjacent pixels x 8 channels of one row, eight 16-byte
    // loads (one per channel), transposed to eight 16-byte LDS items (one per pixel).  The units of a pass form one list:
    // for each channel group the chunk's units of the first tensor, then those of the second.  Units start at multiples of
    // 8; those outside the row are zeros.
    const int npx8 = min(8, (p.W - px0 + 7) >> 3);                // units of the first tensor's chunk
    const uint32_t per_g = (uint32_t)(npx8 + (p.cols2 >> 3));
    const int sg = (int)fdiv((uint32_t)tid, npx8 == 8 ? p.div_perg : p.div_perg_last);       // channel group of the pass
    const int unit = tid - sg * (int)per_g;
    const bool second = unit >= npx8;
    const int run = second ? unit - npx8 : unit;
    const int gx = (second ? px0 - p.lead : px0) + 8 * run;
    const bool colok = gx >= 0 && gx < p.W;
    const bool stages = rowok && sg < p.chg && colok;
    // (RAGGED: the unit that the row's end cuts ends with the row, its shared pixels are written twice, the same; the units
    // of zeros behind it follow where it ends)
    const int shift = RAGGED && gx + 8 > p.W ? -p.W & 7 : 0;
    const uint32_t chbytes = 2u * (uint32_t)p.H * (uint32_t)p.W, last = (uint32_t)(p.C - 1) * chbytes;
    const uint8_t *src = reinterpret_cast<const uint8_t *>((second ? x2 : x1) + (size_t)b * p.C * p.H * p.W) +
                         2u * ((uint32_t)(second ? yy : p1) * (uint32_t)p.W + (uint32_t)(colok ? gx - shift : 0));

    // The loads of a pass, without a select or a branch on their data: whatever uses a value here makes every load wait
    // for its own round trip before the next one goes out.  Channels past the last: the last one's pixels, zeroed when
    // they are written to LDS.
    u32x4 v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = (u32x4){0, 0, 0, 0};         // (units outside the row stay that)
    auto issue = [&](int chi0) __attribute__((always_inline)) {
        if (!stages || (chi0 + sg) * 8 >= p.C) return;            // (a lane that loads costs the address unit its cycles)
        const uint32_t off = (uint32_t)((chi0 + sg) * 8) * chbytes;
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = load16<RAGGED>(src + min(off + c * chbytes, last));
    };
    issue(0);                                                     // before anything that the loads do not need

    const int l16 = lane & 15, kg = lane >> 4;
    floatx4 acc[BPW][NB];
#pragma unroll
    for (int t = 0; t < BPW; ++t)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[t][nb] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    // (uniform: else every product is 0, and the workgroup has only zeros to store.  What the staging needs is computed
    // inside: before the branch it was a cost of every displaced row beside the image as well, 3x16x16x82, +-8 / 3, 7.7 us
    // against 7.3, 4x55x9x93, +-6 / 3, 5.8 against 5.5.  The loads are not: inside they go out later, 4 to 16 % slower.)
    if (rowok) {
        u32x4 *lds0 = reinterpret_cast<u32x4 *>(smem) + (second ? p.chg * p.P1 + sg * p.P2 : sg * p.P1);
        const int pitch = second ? p.pitch2 : p.pitch1;
        // where its pixels go: by residue class of the column; to the spare item behind the rows what lies left of the chunk
        int item[8], col = 8 * run - shift, cls, at;
        {
            const int c0 = RAGGED ? max(col, 0) : col;
            const int idx = (int)fdiv((uint32_t)c0, p.div_sd);
            cls = c0 - idx * p.sd;
            at = cls * pitch + idx;
        }
        auto next_col = [&]() __attribute__((always_inline)) {
            const bool wrap = ++cls == p.sd;
            at += wrap ? 1 - (p.sd - 1) * pitch : pitch;
            cls = wrap ? 0 : cls;
        };
        const int spare = (int)(reinterpret_cast<u32x4 *>(smem) + p.chg * (p.P1 + p.P2) - lds0);
#pragma unroll
        for (int px = 0; px < 8; ++px) {
            const bool there = !RAGGED || col + px >= 0;
            item[px] = there ? corr_slot<ROT>(at, sg) : spare;
            if (there) next_col();
        }

        auto commit = [&](int chi0, int ng) __attribute__((always_inline)) {
            if ((chi0 + ng) * 8 > p.C) {                              // uniform: the last pass, where channels are missing
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const bool ok = (chi0 + sg) * 8 + c < p.C;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[c][j] = ok ? v[c][j] : 0u;
                }
            }
            if (sg >= ng) return;
#pragma unroll
            for (int px = 0; px < 8; ++px) {
                const uint32_t sel = (px & 1) ? 0x07060302u : 0x05040100u;
                u32x4 d;
#pragma unroll
                for (int q = 0; q < 4; ++q) d[q] = __builtin_amdgcn_perm(v[2 * q + 1][px >> 1], v[2 * q][px >> 1], sel);
                lds0[item[px]] = d;
            }
        };

        // this lane's operand positions: pixel (lane & 15) of block (class c, sub-block s) and the
        // columns q = pixel0 - R*sd + sd*j of the same class, j = 16*nb + (lane & 15); positions
        // past the staged ones are clamped (their products are never stored)
        int apos[BPW], bpos[BPW][NB];
#pragma unroll
        for (int t = 0; t < BPW; ++t) {
            const uint32_t bl = (uint32_t)min(wave + 4 * t, p.nblk - 1);
            const uint32_t s = fdiv(bl, p.div_sd);
            const uint32_t c = bl - s * (uint32_t)p.sd;
            apos[t] = corr_slot<ROT>(min((int)c * p.pitch1 + 16 * (int)s + l16, p.P1 - 1), kg);
            const uint32_t ec = (uint32_t)(p.lead - p.R * p.sd) + c;
            const uint32_t ei = fdiv(ec, p.div_sd);
            const uint32_t cls2 = ec - ei * (uint32_t)p.sd;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                bpos[t][nb] = corr_slot<ROT>(min((int)cls2 * p.pitch2 + (int)ei + 16 * (int)s + 16 * nb + l16, p.P2 - 1), kg);
        }

        // groups of the pass that starts at chi0, padded to whole reduction steps (the padding is staged as zeros)
        auto groups_of = [&](int chi0) { return min(p.chg, ((p.nchi - chi0) + 3) & ~3); };
        for (int chi0 = 0; chi0 < p.nchi; chi0 += p.chg) {
            const int ng = groups_of(chi0);
            if (chi0 > 0) __syncthreads();                        // previous pass has been read
            commit(chi0, ng);
            __syncthreads();
            // the next pass's loads are in flight while this one is multiplied
            if (chi0 + p.chg < p.nchi) issue(chi0 + p.chg);
#pragma unroll
            for (int t = 0; t < BPW; ++t) {
                if (wave + 4 * t >= p.nblk) break;                // uniform
                const uint4 *ap = a1l + kg * p.P1;
                const uint4 *bp = a2l + kg * p.P2;
                for (int ks = 0; ks < ng; ks += 4) {              // (four groups on: rotated by four)
                    const half8 a = __builtin_bit_cast(half8, ap[ks * p.P1 + (apos[t] ^ (ROT ? ks & 4 : 0))]);
                    half8 bq[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) bq[nb] = __builtin_bit_cast(half8, bp[ks * p.P2 + (bpos[t][nb] ^ (ROT ? ks & 4 : 0))]);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[t][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, bq[nb], acc[t][nb], 0, 0, 0);
                }
            }
        }
    }

    // D[i][j]: lane holds column j = lane & 15 and rows i = 4*(lane >> 4) + r.  Row i is pixel
    // i of the block, column 16*nb + j is displacement p4 = 16*nb + j - i.
    uint16_t *yrow = y + (((size_t)b * p.H + p1) * p.W + px0) * p.n * p.n + (size_t)p3 * p.n;
#pragma unroll
    for (int t = 0; t < BPW; ++t) {
        const int bl = wave + 4 * t;
        if (bl >= p.nblk) break;                                  // uniform
        const uint32_t s = fdiv((uint32_t)bl, p.div_sd);
        const int c = bl - (int)s * p.sd;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 4 * kg + r;
            const int px = c + p.sd * (16 * (int)s + i);          // pixel inside the chunk
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int p4 = 16 * nb + l16 - i;
                if (px < wchunk && p4 >= 0 && p4 < p.n) {
                    const _Float16 h = (_Float16)acc[t][nb][r];   // round to nearest even
                    yrow[(size_t)px * p.n * p.n + p4] = __builtin_bit_cast(uint16_t, h);
                }
            }
        }
    }
}

size_t corr_lds_bytes(const CorrParams &p)
{
    return ((size_t)p.chg * (p.P1 + p.P2) + 1) * 16;      // and the spare item (see the kernel)
}

template <int NB, int BPW, bool RAGGED, bool ROT>
static hipError_t launch_corr(const CorrParams &p, const void *x1, const void *x2, void *y, hipStream_t s,
                              uint32_t grid)
{
    static std::atomic<int> raised{0};
    if (hipError_t e = raise_lds_limit_once(reinterpret_cast<const void *>(merit_corr_mfma<NB, BPW, RAGGED, ROT>), raised);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL((merit_corr_mfma<NB, BPW, RAGGED, ROT>), dim3(grid), dim3(256), corr_lds_bytes(p), s, p,
                       reinterpret_cast<const uint16_t *>(x1), reinterpret_cast<const uint16_t *>(x2),
                       reinterpret_cast<uint16_t *>(y));
    return hipGetLastError();
}

hipError_t launch_correlation(const CorrParams &p, const void *x1, const void *x2, void *y, hipStream_t s)
{
    const int64_t grid = (int64_t)p.N * p.H * p.n * p.xchunks;
    if (grid == 0) return hipSuccess;
    const uint32_t gx = (uint32_t)grid;
    const int bpw = (p.nblk + 3) / 4;
    if (bpw < 1 || bpw > 2) return hipErrorInvalidValue;
    const int v = p.nb * 2 + (bpw - 1);
#define MERIT_CORR(RAGGED, ROT)                                              \
    switch (v) {                                                             \
    case 2: return launch_corr<1, 1, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    case 3: return launch_corr<1, 2, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    case 4: return launch_corr<2, 1, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    case 5: return launch_corr<2, 2, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    case 6: return launch_corr<3, 1, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    case 7: return launch_corr<3, 2, RAGGED, ROT>(p, x1, x2, y, s, gx);      \
    default: return hipErrorInvalidValue;                                    \
    }
    if (p.W % 8 != 0 && p.rot) MERIT_CORR(true, true)
    if (p.W % 8 != 0) MERIT_CORR(true, false)
    if (p.rot) MERIT_CORR(false, true)
    MERIT_CORR(false, false)
#undef MERIT_CORR
}

}  // namespace merit
