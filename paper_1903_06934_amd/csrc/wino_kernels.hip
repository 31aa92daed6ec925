// HIP kernels for gfx950: stride-1 3x3 layers by fast filtering,
// F(2x2, 3x3) of S. Winograd's minimal filtering algorithms (Winograd, 1980;
// for convolution layers Lavin & Gray, 2015): a 2 x 2 tile of outputs takes
// 16 multiplications a channel instead of 36.
//
//   Y = At [ sum over channels of (G g Gt) o (Bt d B) ] A
//   Bt = | 1  0 -1  0 |   G = |  1    0    0  |   At = | 1  1  1  0 |
//        | 0  1  1  0 |       | 1/2  1/2  1/2 |        | 0  1 -1 -1 |
//        | 0 -1  1  0 |       | 1/2 -1/2  1/2 |
//        | 0  1  0 -1 |       |  0    0    1  |
//
// The sum over channels is 16 matrix products (one per point of the
// transformed tile), run on v_mfma_f32_16x16x4f32 in fp32 throughout.
//
// A 5 x 5 filter is the sum of four 3 x 3 ones (parts (a, b), a, b < 2) at
// offsets (2 a, 2 b): part (a, b) holds the taps (2 a + i, 2 b + j), i, j < 3,
// without those that an earlier part holds (i = 0 where a > 0, j = 0 where
// b > 0).  All four add up in the transformed domain, 64 multiplications
// instead of 100 for 2 x 2 outputs; to the products they are further channels.
// The offsets are even so that the patches keep their alignment.
#include "internal.h"
#include "tile_offsets.h"

#include <algorithm>

namespace miconv {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

namespace {

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
}

// Buffer load of four words a lane straight into LDS (256 consecutive words).
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, float *lds, uint32_t voff,
                                      uint32_t soff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LDS_AS void *)lds, 16, voff, soff, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void fence()
{
    __asm__ volatile("" ::: "memory");
}

// V = Bt d B.
__device__ __forceinline__ void input_transform(const float (&d)[16], float (&v)[16])
{
    float t[16];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        t[j] = d[j] - d[8 + j];
        t[4 + j] = d[4 + j] + d[8 + j];
        t[8 + j] = d[8 + j] - d[4 + j];
        t[12 + j] = d[4 + j] - d[12 + j];
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        v[4 * i] = t[4 * i] - t[4 * i + 2];
        v[4 * i + 1] = t[4 * i + 1] + t[4 * i + 2];
        v[4 * i + 2] = t[4 * i + 2] - t[4 * i + 1];
        v[4 * i + 3] = t[4 * i + 1] - t[4 * i + 3];
    }
}

// Four words of LDS.
__device__ __forceinline__ f32x4 lds_b128(const float *base, int word)
{
    return *(LDS_AS const f32x4 *)(base + word);
}

// A patch row of a tile and channel, by buffer loads: off holds one offset per
// load (out of range: zero), soff the row's and stage's.  MODE 1 (first column
// odd): columns 0, (1, 2), 3; MODE 2 (even): columns (0, 1), (2, 3).  The pairs
// start at even columns, so on even widths a pair lies inside a row or outside;
// on odd ones (ODD) the pair at the last column takes its second word from
// past the row, which `keep` (0 for that lane, else all ones) clears.  MODE 0:
// one word each.
template <int MODE>
struct Patch {
    static constexpr int LOADS = MODE == 0 ? 4 : MODE == 1 ? 3 : 2;  // a row
    // First column of load l, and whether it is a pair.
    static constexpr int col(int l) { return MODE == 0 ? l : MODE == 1 ? l + l / 2 : 2 * l; }
    static constexpr bool pair(int l) { return MODE == 2 || (MODE == 1 && l == 1); }
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int MODE>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, const uint32_t *off,
                                         uint32_t soff, float *d)
{
#pragma unroll
    for (int l = 0; l < Patch<MODE>::LOADS; l++) {
        const int c = Patch<MODE>::col(l);
        if (Patch<MODE>::pair(l)) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off[l], soff, 0);
            const uint32_t hi = v[1];
            d[c] = __uint_as_float(v[0]);
            d[c + 1] = __uint_as_float(hi);
        } else {
            d[c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off[l], soff, 0));
        }
    }
}
// Clears the words past the row (once the loads are due).
template <int MODE>
__device__ __forceinline__ void clear_past(const uint32_t (&keep)[2], float *d)
{
    if (MODE == 1) {
        d[2] = __uint_as_float(__float_as_uint(d[2]) & keep[0]);
    } else {
        d[1] = __uint_as_float(__float_as_uint(d[1]) & keep[0]);
        d[3] = __uint_as_float(__float_as_uint(d[3]) & keep[1]);
    }
}

// Whether a sum is neither an infinity nor a NaN.
__device__ __forceinline__ bool is_finite(float v)
{
    return fabsf(v) < __builtin_inff();
}

// The kernel's arguments, read from the argument segment anew: for code that
// runs once an output tile, so that its arguments do not hold scalar registers
// (and, spilled to vector lanes, cost MFMA time) during the main loop.
template <class Args>
__device__ __forceinline__ const Args &cold_args()
{
    typedef const __attribute__((address_space(4))) Args *Ptr;
    Ptr p = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(p));
    return *(const Args *)p;
}

// Work of one workgroup: the rounds of whole output tiles (tile = round
// nwg + its place), then its share of the stages of the remaining tiles.
struct Unit {
    int tile, s0, s1, slab;  // stages [s0, s1); slab -1: the whole tile
};
// First stage, among those of the remaining tiles, of workgroup w's share.
__device__ __forceinline__ int share(const WinoWork &a, int w)
{
    return w * a.share + min(w, a.share_rem);
}
__device__ __forceinline__ Unit wino_unit(const WinoWork &a, int w, int k)
{
    Unit u;
    if (k < a.rounds) {
        u.tile = k * a.nwg + w;
        u.s0 = 0;
        u.s1 = a.nstage;
        u.slab = -1;
        return u;
    }
    const int lo = share(a, w), hi = share(a, w + 1);
    const int t0 = (int)fast_div((uint32_t)lo, a.d_nstage), cut = min(hi, (t0 + 1) * a.nstage);
    const int i = k - a.rounds;
    u.tile = a.rounds * a.nwg + t0 + i;
    u.s0 = i ? 0 : lo - t0 * a.nstage;
    u.s1 = i ? hi - cut : cut - t0 * a.nstage;
    u.slab = u.s0 == 0 && u.s1 == a.nstage ? -1 : w + t0 + i;
    return u;
}

// Y = At m A of one (row, tile): y = {00, 01, 10, 11}.
__device__ __forceinline__ f32x4 output_transform(const float (&m)[16])
{
    float z[2][4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        z[0][j] = m[j] + m[4 + j] + m[8 + j];
        z[1][j] = m[4 + j] - m[8 + j] - m[12 + j];
    }
    return f32x4{z[0][0] + z[0][1] + z[0][2], z[0][1] - z[0][2] - z[0][3],
                 z[1][0] + z[1][1] + z[1][2], z[1][1] - z[1][2] - z[1][3]};
}

// Place of a tile in the output.
struct TileAt {
    int img, ty, tx;
};
__device__ __forceinline__ TileAt tile_at(const WinoArgs &a, int t)
{
    const int row = (int)fast_div((uint32_t)t, a.d_qt);
    TileAt r;
    r.tx = t - row * a.Qt;
    r.img = (int)fast_div((uint32_t)row, a.d_pt);
    r.ty = row - r.img * a.Pt;
    return r;
}

// The 2 x 2 outputs of output channel oc at a tile (zero where there are none).
__device__ __forceinline__ f32x4 load_tile(const WinoArgs &a, const TileAt &at, int oc)
{
    const int p = 2 * at.ty, q = 2 * at.tx;
    const float *const o = a.out + (long long)at.img * a.out_img_stride + (long long)oc * a.out_hw +
                           (long long)p * a.Q + q;
    const bool two_p = p + 1 < a.P, two_q = q + 1 < a.Q;
    return f32x4{o[0], two_q ? o[1] : 0.f, two_p ? o[a.Q] : 0.f, two_p && two_q ? o[a.Q + 1] : 0.f};
}

// Stores the 2 x 2 outputs (bias added) of output channel oc at a tile.
__device__ __forceinline__ void store_tile(const WinoArgs &a, const TileAt &at, int oc, f32x4 y)
{
    const int p = 2 * at.ty, q = 2 * at.tx;
    float *const o = a.out + (long long)at.img * a.out_img_stride + (long long)oc * a.out_hw +
                     (long long)p * a.Q + q;
    const bool two_p = p + 1 < a.P;
    if ((a.Q & 1) == 0) {
        *(f32x2 *)o = f32x2{y[0], y[1]};
        if (two_p)
            *(f32x2 *)(o + a.Q) = f32x2{y[2], y[3]};
    } else {
        const bool two_q = q + 1 < a.Q;
        o[0] = y[0];
        if (two_q)
            o[1] = y[1];
        if (two_p) {
            o[a.Q] = y[2];
            if (two_q)
                o[a.Q + 1] = y[3];
        }
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward and backward-data (WinoArgs).
//
// A workgroup of eight waves (one a CU, persistent) computes output tiles of
// 64 channels x 64 tiles (256 pixels); a wave takes 32 channels of 16 tiles at
// all 16 points: 32 accumulator blocks, 128 registers, two waves a SIMD.
// A stage is eight source channels.  Per stage a wave loads the 4 x 4 patches
// of 16 tiles and four channels into registers (a lane one patch; padding
// through the buffer's range check, so any map width and padding runs), turns
// them into V with 32 additions and puts V into LDS in the MFMA's lane order,
// where the waves of both channel halves read it; the transformed filters U
// come by direct-to-LDS loads in the same order.  All LDS operands are 16-byte
// reads of consecutive lanes.
//
// What bounds it: on gfx950 a VALU instruction does not run beside an fp32
// MFMA of its SIMD (measured with two waves a SIMD: one v_add after every MFMA
// takes 39 cycles a pair instead of 32, six 51), so the transform's additions cost
// MFMA time (128 channels on 112 x 112: 0.70 MFMA-busy, no LDS conflicts);
// sharing V between the two channel halves halves them (a first version with
// the transform in every wave, two workgroups of four waves a CU, ran its
// steady state at 0.76 of the MFMA rate), and they run in one burst.
//
// The stages of a workgroup's output tiles follow one another without a gap:
// in stage j the patches of stage j + 2 are loaded, V of stage j + 1 written,
// and after the barrier near its end (every read of stage j is in registers
// by then) U of stage j + 2 is requested and the first operands of stage j + 1
// read, so a tile's start costs no latency and its end only the output
// transform.  The tiles left after the whole rounds are cut along the
// channels so that every workgroup gets the same number of stages; their
// partial sums go to slabs that wino_finish_kernel adds in a fixed order.
//
// Measured against the direct plans (forward, batch 32 unless said, ms):
// 64 -> 64 on 224 x 224 maps 0.534 (0.868), 128 on 112 x 112 0.487 (0.835),
// 256 on 56 x 56 0.464 (0.818), 512 on 28 x 28 0.462 (0.819), 512 on 14 x 14
// 0.139 (0.257); batch 128, 384 on 13 x 13 in two groups 0.160 (0.227); batch
// 64, 512 on 7 x 7 0.098 (0.164): 0.60-0.73 of the fp32 MFMA peak in executed
// operations.  Error against 64 bits 3.0e-7 (4.2e-7) of the norm with 128
// channels, 4.6e-7 (5.9e-7) with 512.  Tried: the two waves of a SIMD
// transforming in different groups (15 % slower), the additions spread over
// the MFMAs, a few after each (2 % slower), U requested after group 6's MFMAs
// (2 %), a raised wave priority around the MFMAs (4 %), one wave a SIMD with 64
// channels by 16 tiles and the transform in every wave (25 %).
// ---------------------------------------------------------------------------
template <int MODE, bool ODD>
__global__ __launch_bounds__(512, 2) void wino_gemm_kernel(const WinoArgs a)
{
    constexpr int STG = 2 * 4 * 4 * 256;  // words of U, and of V, per stage
    constexpr int NOFF = 4 * Patch<MODE>::LOADS;
    __shared__ __attribute__((aligned(16))) float U0[STG], U1[STG], V0[STG], V1[STG];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2, tg = wave & 3;  // channel half (of 64, of 8), tile group
    const int kr = lane >> 4, lc = lane & 15;
    // Workgroups of one XCD (hardware ids congruent mod 8) take neighbouring
    // output tiles, which share their filters or their source rows in its L2.
    const int per = a.nwg >> 3, rem = a.nwg & 7, xcd = blockIdx.x & 7;
    const int w = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);

    const __amdgpu_buffer_rsrc_t rX = make_rsrc(a.src, a.src_bytes);
    const __amdgpu_buffer_rsrc_t rU = make_rsrc(a.U, a.u_bytes);
    const uint32_t stage_bytes = 32u * (uint32_t)a.src_hw;
    const int ncb = a.ncb;

    // Cursor of the loads, two stages ahead of the MFMAs.
    Unit pu{};
    int pk = -1, ps = 0;     // unit, stage
    int pc = 0;              // its channel block (of the part)
    uint32_t pu_base = 0;    // its filters
    uint32_t off[NOFF];      // its patches
    uint32_t keep[2] = {~0u, ~0u};
    bool more = true;
    auto advance = [&]() __attribute__((always_inline)) {
        if (pk >= 0) {
            ps++;
            pc++;
            if (ps < pu.s1 && pc < ncb)
                return;
        }
        const WinoArgs &a = cold_args<WinoArgs>();
        if (pk < 0 || ps >= pu.s1) {
            const int nunits = a.rounds + (a.rest ? 2 : 0);
            do {
                if (++pk >= nunits) {
                    more = false;
                    return;
                }
                pu = wino_unit(a, w, pk);
            } while (pu.s0 >= pu.s1);
            ps = pu.s0;
        }
        const int part = (int)fast_div((uint32_t)ps, a.d_ncb);
        pc = ps - part * ncb;
        const int ph = part / a.parts, pw = part - ph * a.parts;
        const int gm = (int)fast_div((uint32_t)pu.tile, a.d_tblocks);  // (group, channel block)
        const int tb = pu.tile - gm * a.tblocks, g = (int)fast_div((uint32_t)gm, a.d_mblocks);
        pu_base = (uint32_t)gm * (uint32_t)a.nstage * (STG * 4u);
        const int t = tb * 64 + tg * 16 + lc;
        const TileAt at = tile_at(a, min(t, a.tiles - 1));
        const int h0 = 2 * (at.ty + ph) + a.off, w0 = 2 * (at.tx + pw) + a.off;
        const uint32_t base = ((uint32_t)at.img * a.src_img_words +
                               (uint32_t)(g * a.cin + 4 * half + kr) * (uint32_t)a.src_hw) * 4u;
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int l = 0; l < Patch<MODE>::LOADS; l++) {
                const int c = Patch<MODE>::col(l);
                const bool ok = (unsigned)(h0 + i) < (unsigned)a.src_h &&
                                (unsigned)(w0 + c) < (unsigned)a.src_w;
                off[i * Patch<MODE>::LOADS + l] =
                    ok ? base + (uint32_t)((h0 + i) * a.src_w + w0 + c) * 4u : kOob;
            }
        if constexpr (ODD) {
            keep[0] = w0 + (MODE == 1 ? 2 : 1) == a.src_w ? 0u : ~0u;
            keep[1] = w0 + 3 == a.src_w ? 0u : ~0u;
        }
    };
    auto load_patch = [&](float (&d)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; i++)
            load_row<MODE>(rX, off + i * Patch<MODE>::LOADS, (uint32_t)pc * stage_bytes, d + 4 * i);
    };
    auto load_u = [&](float *Ud, uint32_t base, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < 4; l++) {
            const int i = wave + 8 * l;
            dma16(rU, Ud + i * 256, (uint32_t)lane * 16u + (uint32_t)i * 1024u,
                  base + (uint32_t)s * (STG * 4u));
        }
    };
    // (Before the cursor moves on: keep is that of the patches in d.)
    auto write_v = [&](float *Vd, float (&d)[16]) __attribute__((always_inline)) {
        float v[16];
        if constexpr (ODD) {
#pragma unroll
            for (int i = 0; i < 4; i++)
                clear_past<MODE>(keep, d + 4 * i);
        }
        input_transform(d, v);
#pragma unroll
        for (int q = 0; q < 4; q++)
            *(LDS_AS f32x4 *)(Vd + ((half * 4 + tg) * 4 + q) * 256 + lane * 4) =
                f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    };

    f32x4 acc[2][16];
    f32x4 u[4][2], v[4];
    float d[16];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int p = 0; p < 16; p++)
                acc[b][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // Operands of group g8 (step g8 / 4, points 4 (g8 % 4) ..) of a stage.
    auto read_ops = [&](const float *Uc, const float *Vc, int g8) __attribute__((always_inline)) {
        const int step = g8 >> 2, q = g8 & 3;
#pragma unroll
        for (int b = 0; b < 2; b++)
            u[q][b] = lds_b128(Uc, ((step * 4 + half * 2 + b) * 4 + q) * 256 + lane * 4);
        v[q] = lds_b128(Vc, ((step * 4 + tg) * 4 + q) * 256 + lane * 4);
    };
    // Outputs of unit un: to its slab, or (whole tiles) with the bias to the
    // output, by buffer stores whose range check drops what lies outside it.
    auto finish = [&](const Unit &un) __attribute__((always_inline)) {
        const WinoArgs &c = cold_args<WinoArgs>();
        const int M = c.M, P = c.P, Q = c.Q, hw = c.out_hw;
        const int gm = (int)fast_div((uint32_t)un.tile, c.d_tblocks), tb = un.tile - gm * c.tblocks;
        const int g = (int)fast_div((uint32_t)gm, c.d_mblocks), mb = gm - g * c.mblocks;
        const int t = tb * 64 + tg * 16 + lc, row0 = half * 32 + 4 * kr, m0 = mb * 64 + row0;
        const TileAt at = tile_at(c, min(t, c.tiles - 1));
        const int p = 2 * at.ty, q = 2 * at.tx;
        const __amdgpu_buffer_rsrc_t rO = make_rsrc(c.out, c.out_bytes);
        const __amdgpu_buffer_rsrc_t rB = make_rsrc(c.bias, c.bias ? (uint32_t)(c.groups * M) * 4u : 0u);
        const uint32_t o0 = ((uint32_t)at.img * (uint32_t)c.out_img_stride +
                             (uint32_t)(g * M + m0) * (uint32_t)hw + (uint32_t)(p * Q + q)) * 4u;
        const bool two_p = p + 1 < P, two_q = q + 1 < Q;
        float bv[2][4];
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                bv[b][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    rB, (g * M + min(m0 + b * 16 + r, M - 1)) * 4, 0, 0));
        float zero = 0.f;  // a NaN once an output is not finite
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                float x[16];
#pragma unroll
                for (int k = 0; k < 16; k++)
                    x[k] = acc[b][k][r];
                f32x4 y = output_transform(x);
                if (un.slab >= 0) {
                    *(f32x4 *)(c.slabs + (size_t)un.slab * 16384 +
                               ((row0 + b * 16 + r) * 64 + tg * 16 + lc) * 4) = y;
                    continue;
                }
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    y[k] += bv[b][r];
                    zero = fmaf(y[k], 0.f, zero);
                }
                const TileOffsets o =
                    tile_offsets(o0 + (uint32_t)((b * 16 + r) * hw) * 4u, (uint32_t)Q * 4u,
                                 t < c.tiles && m0 + b * 16 + r < M, two_p, two_q);
                if ((Q & 1) == 0) {
                    __builtin_amdgcn_raw_buffer_store_b64(
                        u32x2{__float_as_uint(y[0]), __float_as_uint(y[1])}, rO, o.at[0], 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(
                        u32x2{__float_as_uint(y[2]), __float_as_uint(y[3])}, rO, o.at[2], 0, 0);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[k]), rO, o.at[k], 0, 0);
                }
            }
        // (Lanes outside the output hold sums of valid or zero operands.)
        if (un.slab < 0 && !(zero == 0.f))
            *c.flag = 1;  // wino_finish_kernel looks the outputs over
    };

    // The MFMAs' cursor.
    Unit cu{};
    int ck = -1, cs = 0;
    auto step_cursor = [&]() __attribute__((always_inline)) {
        if (ck >= 0 && ++cs < cu.s1)
            return;
        const WinoArgs &a = cold_args<WinoArgs>();
        const int nunits = a.rounds + (a.rest ? 2 : 0);
        do {
            if (++ck >= nunits)
                return;
            cu = wino_unit(a, w, ck);
        } while (cu.s0 >= cu.s1);
        cs = cu.s0;
    };

    // One stage: MFMAs from (Uc, Vc); the next stage is (Un, Vn).  have1, have2:
    // there is a stage one, two further on.
    bool have1, have2;
    auto stage = [&](float *Uc, float *Vc, float *Un, float *Vn) __attribute__((always_inline)) {
#pragma unroll
        for (int g8 = 0; g8 < 8; g8++) {
            const int q = g8 & 3;
            if (g8 == 6) {
                // Every read of this stage is in registers and this wave's
                // part of the next one has landed; after the barrier that
                // holds for all waves.
                __builtin_amdgcn_s_waitcnt(0);
                fence();
                __builtin_amdgcn_s_barrier();
                fence();
                if (have2)
                    load_u(Uc, pu_base, ps);
            }
            read_ops(g8 < 6 ? Uc : Un, g8 < 6 ? Vc : Vn, (g8 + 2) & 7);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int b = 0; b < 2; b++)
                    acc[b][4 * q + j] = mfma16(u[q][b][j], v[q][j], acc[b][4 * q + j]);
            __builtin_amdgcn_sched_barrier(0);
            if (g8 == 0) {
                if (have1)
                    write_v(Vn, d);
                __builtin_amdgcn_sched_barrier(0);
                advance();
                have2 = more;
                if (have2)
                    load_patch(d);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (cs + 1 == cu.s1) {
            finish(cu);
            clear();
        }
        step_cursor();
        const bool on = have1;
        have1 = have2;
        return on;
    };

    advance();
    if (!more)
        return;
    load_u(U0, pu_base, ps);
    load_patch(d);
    write_v(V0, d);
    step_cursor();
    advance();
    have1 = more;
    if (have1) {
        load_u(U1, pu_base, ps);
        load_patch(d);
    }
    clear();
    __builtin_amdgcn_s_waitcnt(0);
    fence();
    __builtin_amdgcn_s_barrier();
    fence();
    read_ops(U0, V0, 0);
    read_ops(U0, V0, 1);
    // The operands read past a workgroup's last stage are not used.
    while (stage(U0, V0, U1, V1) && stage(U1, V1, U0, V0)) {
    }
}

// Direct sums, over channels and taps in order, of the outputs in `bad` (bit k:
// output (k >> 1, k & 1)) of the tile `at` of output channel oc.  All lanes of a
// wave call it, on the same channel: a lane loads its tile's patch once for all
// four outputs, and one word of the channel's filter for the others.  The
// padding's zeros are multiplied too (by an infinite tap, to a NaN), as in the
// direct plans.
//
// Waiting for the loads bounds it: a channel's are all requested together.  With
// every output plus infinity a forward pass takes 3.3 ms on 64 -> 64 channels,
// 112 x 112, batch 32 (one thread an output: 23; the direct plan: 0.25), 3.4 on 512
// -> 512, 14 x 14 (11; 0.27); with NaNs, which end a sum, 0.25 and 0.15; with one
// infinite input 0.21 (0.35) and 0.65 (4.3).
template <int R>
__device__ __forceinline__ void wino_direct(const WinoArgs &a, const TileAt &at, int oc, int bad, f32x4 &y)
{
    constexpr int D = R + 1, T = R * R;
    const int lane = threadIdx.x & 63, g = oc / a.M, m = oc - g * a.M;
    const int h0 = 2 * at.ty + a.off, w0 = 2 * at.tx + a.off;
    const __amdgpu_buffer_rsrc_t rX = make_rsrc(a.src, a.src_bytes);
    const __amdgpu_buffer_rsrc_t rW = make_rsrc(a.w, (uint32_t)(a.groups * a.M * a.cin) * (T * 4u));
    // Backward-data: the filters of one input channel, taps mirrored.
    const uint32_t tap = (uint32_t)(a.flip ? T - 1 - lane : lane) * 4u;
    const uint32_t wbase = (uint32_t)(a.flip ? g * a.cin * a.M + m : oc * a.cin) * (T * 4u);
    const uint32_t wstep = (a.flip ? a.M : 1) * (T * 4u), xstep = (uint32_t)a.src_hw * 4u;
    const uint32_t base = ((uint32_t)at.img * a.src_img_words + (uint32_t)(g * a.cin) * (uint32_t)a.src_hw) * 4u;
    uint32_t off[D * D];
#pragma unroll
    for (int e = 0; e < D * D; e++) {
        const int h = h0 + e / D, q = w0 + e % D;
        off[e] = (unsigned)h < (unsigned)a.src_h && (unsigned)q < (unsigned)a.src_w
                     ? base + (uint32_t)(h * a.src_w + q) * 4u
                     : kOob;
    }
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    int live = bad;  // what is not a NaN yet (a NaN stays one)
    for (int c = 0; c < a.cin && __builtin_amdgcn_ballot_w64(live != 0); c++) {
        float d[D][D], wt[T];
        const int xs = __builtin_amdgcn_readfirstlane((int)((uint32_t)c * xstep));
        const float wl = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
            rW, lane < T ? (int)tap : (int)kOob,
            __builtin_amdgcn_readfirstlane((int)(wbase + (uint32_t)c * wstep)), 0));
#pragma unroll
        for (int e = 0; e < D * D; e++)
            d[e / D][e % D] = __uint_as_float(
                __builtin_amdgcn_raw_buffer_load_b32(rX, (int)off[e], xs, 0));
#pragma unroll
        for (int t = 0; t < T; t++)
            wt[t] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wl), t));
#pragma unroll
        for (int i = 0; i < D; i++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int r = i - (k >> 1);
                if (r < 0 || r >= R)
                    continue;
#pragma unroll
                for (int z = 0; z < R; z++)
                    s[k] = fmaf(d[i][(k & 1) + z], wt[r * R + z], s[k]);
            }
        live = 0;
#pragma unroll
        for (int k = 0; k < 4; k++)
            live |= s[k] == s[k] ? bad & (1 << k) : 0;
    }
    const float bv = a.bias ? a.bias[oc] : 0.f;
#pragma unroll
    for (int k = 0; k < 4; k++)
        y[k] = bad & (1 << k) ? s[k] + bv : y[k];
}

// The workgroup whose share holds the first stage of remaining tile r.
__device__ __forceinline__ int wino_first_share(const WinoWork &a, int r)
{
    const int lo = r * a.nstage, big = a.share_rem * (a.share + 1);
    int w = lo < big || a.share == 0 ? lo / (a.share + 1) : a.share_rem + (lo - big) / a.share;
    while (share(a, w + 1) <= lo)
        w++;
    return w;
}

// Adds the slabs of the tiles that were cut (their parts in the order of their
// channels) and, where an infinity or a NaN came out -- the transforms mix the
// pixels of a tile, so that an infinity in x may become a NaN, or a finite
// result overflow -- recomputes the output directly.  A block is 256 (channel,
// tile) pairs of one cut output tile; then all blocks look through the output
// if the GEMM raised the flag, a wave for 64 tiles of a channel.
template <int R>
__global__ __launch_bounds__(256) void wino_finish_kernel(const WinoArgs a)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int whole = a.rounds * a.nwg;  // output tiles before the remaining ones
    const int rows = (whole + a.rest) * 64, place = (int)blockIdx.x * 4 + wave;
    // First (cut = true) the wave's row of a cut tile, if it has one; then, on
    // the flag, its share of all rows of the others.
    bool cut = true;
    for (int u = whole * 64 + place;; u += (int)gridDim.x * 4) {
        const int tile = u >> 6, r = tile - whole, row = u & 63;
        const int gm = tile / a.tblocks, tb = tile - gm * a.tblocks;
        const int g = gm / a.mblocks, m = (gm - g * a.mblocks) * 64 + row;
        const int t = tb * 64 + lane;
        if (u < rows && m < a.M) {
            const int hi = (r + 1) * a.nstage;
            int w = r >= 0 ? wino_first_share(a, r) : 0;
            if ((r >= 0 && share(a, w + 1) < hi) == cut) {
                const TileAt at = tile_at(a, min(t, a.tiles - 1));
                const int oc = g * a.M + m;
                f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
                if (cut) {
                    for (; w < a.nwg && share(a, w) < hi; w++) {
                        if (share(a, w) == share(a, w + 1))
                            continue;
                        const f32x4 s = *(const f32x4 *)(a.slabs + (size_t)(w + r) * 16384 + (row * 64 + lane) * 4);
                        y = f32x4{y[0] + s[0], y[1] + s[1], y[2] + s[2], y[3] + s[3]};
                    }
                    const float bv = a.bias ? a.bias[oc] : 0.f;
                    y = f32x4{y[0] + bv, y[1] + bv, y[2] + bv, y[3] + bv};
                } else {
                    y = load_tile(a, at, oc);
                }
                int bad = 0;
#pragma unroll
                for (int k = 0; k < 4; k++)
                    bad |= is_finite(y[k]) || t >= a.tiles ? 0 : 1 << k;
                if (__builtin_amdgcn_ballot_w64(bad != 0))
                    wino_direct<R>(cold_args<WinoArgs>(), at, oc, bad, y);
                if (t < a.tiles && (cut || bad))
                    store_tile(cold_args<WinoArgs>(), at, oc, y);
            }
        }
        if (cut) {
            if (!__builtin_amdgcn_readfirstlane(*a.flag))
                return;
            cut = false;
            u = place - (int)gridDim.x * 4;
        } else if (u >= rows) {
            return;
        }
    }
}

// Filter transform U = G g Gt into the order the GEMM reads: word
// ((((gm nstage + s) 2 + step) 4 + b) 4 + q) 256 + lane 4 + j is point 4 q + j
// of row m = 64 mb + 16 b + lane % 16, channel c = 8 (s % ncb) + 4 step + lane / 16
// of group g, gm = g mblocks + mb (zero past M), part s / ncb of the filter.  flip (backward-data): row m is
// input channel m, channel c filter c, the taps mirrored.  Also lowers the flag.
__global__ __launch_bounds__(256) void wino_filter_kernel(const WinoArgs a, float *__restrict__ U)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0)
        *a.flag = 0;
    const int lane = i & 63, b = (i >> 6) & 3, step = (i >> 8) & 1;
    const int r = i >> 9, gm = r / a.nstage, s = r - gm * a.nstage;
    const int g = gm / a.mblocks, mb = gm - g * a.mblocks;
    const int part = s / a.ncb, ph = part / a.parts, pw = part - ph * a.parts;
    const int m = mb * 64 + b * 16 + (lane & 15);
    const int c = (s - part * a.ncb) * 8 + step * 4 + (lane >> 4);
    float k[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (m < a.M) {
        const int taps = a.R * a.R;
        const float *src = a.flip ? a.w + ((size_t)(g * a.cin + c) * a.M + m) * taps
                                  : a.w + ((size_t)(g * a.M + m) * a.cin + c) * taps;
#pragma unroll
        for (int j = 0; j < 9; j++) {
            const int i = j / 3, z = j - 3 * i, t = (2 * ph + i) * a.R + 2 * pw + z;
            if ((ph == 0 || i > 0) && (pw == 0 || z > 0))
                k[j] = src[a.flip ? taps - 1 - t : t];
        }
    }
    float t[12];
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const float e = 0.5f * (k[j] + k[6 + j]), o = 0.5f * k[3 + j];
        t[j] = k[j];
        t[3 + j] = e + o;
        t[6 + j] = e - o;
        t[9 + j] = k[6 + j];
    }
    float *dst = U + (((size_t)r * 2 + step) * 4 + b) * 1024 + lane * 4;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float e = 0.5f * (t[3 * q] + t[3 * q + 2]), o = 0.5f * t[3 * q + 1];
        *(f32x4 *)(dst + q * 256) = f32x4{t[3 * q], e + o, e - o, t[3 * q + 2]};
    }
}

// ---------------------------------------------------------------------------
// Backward-weight (WinoWgArgs): the adjoint in the filters, F(3x3, 2x2) with
// the same points.  Per 2 x 2 tile of dy and the 4 x 4 patch of x under it,
//   dw = Ct [ sum over tiles of (H dy Ht) o (Bt x B) ] C
//   H = | 1  0 |   Ct = | 1 1/2  1/2  0 |
//       | 1  1 |        | 0 1/2 -1/2  0 |
//       | 1 -1 |        | 0 1/2  1/2 -1 |
//       | 0  1 |
// (the halves of the transform of dy stand in Ct).  The sum over tiles is 16
// matrix products of filters by channels whose reduction is the tiles.
//
// As the forward GEMM: eight waves, 64 filters x 64 channels, a wave 32 x 16
// at all 16 points, a stage eight tiles.  Both operands are transformed by
// the waves (12 and 32 additions a stage and lane) and shared through LDS.
// The eight tiles of a stage lie in one tile row, cw columns of 8 / cw images;
// the stages of such a strip run down the tile rows, so that a lane keeps the
// lower two rows of its patch for the next stage, its offsets move by a scalar
// and a row outside the image is the same for all lanes.
//
// Measured against the direct plans (ms; batch 32 unless said): 64 -> 64 on
// 224 x 224 maps 0.537 (0.903), 128 on 112 x 112 0.468 (0.899), 256 on 56 x 56
// 0.486 (0.864), 512 on 28 x 28 0.517 (0.865), 512 on 14 x 14 0.182 (0.275);
// batch 128, 384 on 13 x 13 in two groups 0.196 (0.290): 0.6-0.7 of the fp32
// MFMA peak in executed operations on the even maps, 0.42-0.46 where 7 tile
// columns leave one lane in eight idle.  Error against 64 bits 1.0e-6 (1.4e-6)
// of the norm for 128 channels on 112 x 112, 3.8e-7 (4.8e-7) for 512 on 14 x 14.
// The loads must not stand in a branch: where the branches meet the compiler
// copies their results and so waits for them (0.68 instead of 0.49 ms on
// 56 x 56 maps).
// ---------------------------------------------------------------------------
namespace {

constexpr int WG_Q = 272;               // words of one (step, block, q): 4 rows of 16 lanes, 68 apart,
constexpr int WG_STEP = 16 * WG_Q + 16; // for distinct banks in the eight tiles' writes (the counters
                                        // still show 3 conflict cycles an LDS instruction)
constexpr int WG_STG = 2 * WG_STEP;
constexpr int WG_SLAB = 64 * 64 * 9 + 64;  // words: [k][c][tap], then the bias gradient

__device__ __forceinline__ void dy_transform(const float (&g)[4], float (&v)[16])
{
    const float r[2][4] = {{g[0], g[0] + g[1], g[0] - g[1], g[1]},
                           {g[2], g[2] + g[3], g[2] - g[3], g[3]}};
#pragma unroll
    for (int j = 0; j < 4; j++) {
        v[j] = r[0][j];
        v[4 + j] = r[0][j] + r[1][j];
        v[8 + j] = r[0][j] - r[1][j];
        v[12 + j] = r[1][j];
    }
}

// Ct m C: taps in row-major order.
__device__ __forceinline__ void tap_transform(const float (&m)[16], float (&w)[9])
{
    float z[3][4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const float s = 0.5f * (m[4 + j] + m[8 + j]);
        z[0][j] = m[j] + s;
        z[1][j] = 0.5f * (m[4 + j] - m[8 + j]);
        z[2][j] = s - m[12 + j];
    }
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const float s = 0.5f * (z[i][1] + z[i][2]);
        w[3 * i] = z[i][0] + s;
        w[3 * i + 1] = 0.5f * (z[i][1] - z[i][2]);
        w[3 * i + 2] = s - z[i][3];
    }
}

// Output tile: part of the filter, channel block and (group, filter block).
struct WgTile {
    int gm, cb, part, ph, pw;
};
__device__ __forceinline__ WgTile wg_tile(const WinoWgArgs &a, int tile)
{
    WgTile t;
    const int n = (int)fast_div((uint32_t)tile, a.d_parts);
    t.part = tile - n * a.parts * a.parts;
    t.ph = t.part / a.parts;
    t.pw = t.part - t.ph * a.parts;
    t.gm = (int)fast_div((uint32_t)n, a.d_cblocks);
    t.cb = n - t.gm * a.cblocks;
    return t;
}

}  // namespace

template <int MODE>
__global__ __launch_bounds__(512, 2) void wino_wgrad_kernel(const WinoWgArgs a)
{
    // Loads a row of a patch and of dy.  (Odd widths load single words: pairs
    // cleared as in wino_gemm_kernel take registers that this kernel lacks, 0.274
    // instead of 0.196 ms on 13 x 13 maps.)
    constexpr int XL = Patch<MODE>::LOADS, YL = MODE == 0 ? 2 : 1;
    __shared__ __attribute__((aligned(16))) float Y0[WG_STG], Y1[WG_STG], X0[WG_STG], X1[WG_STG];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fg = wave >> 2, cg = wave & 3;  // filter half, channel block of the MFMAs
    const int kr = lane >> 4, lc = lane & 15;
    const int tl = lane & 7, c8 = lane >> 3;  // tile and channel (filter) of the transforms
    const int per = a.nwg >> 3, rem = a.nwg & 7, xcd = blockIdx.x & 7;
    int w = xcd * per + min(xcd, rem) + (int)(blockIdx.x >> 3);
    if (a.rounds == 0) {
        // Few output tiles, each cut over several workgroups: neighbours take
        // the same part of different tiles, which reads the same pixels.
        const int r = a.nwg / a.rest, e = a.nwg - r * a.rest, q = w / a.rest;
        const int t = q < r ? w - q * a.rest : (w - r * a.rest) * a.rest / e;
        w = t * r + (t * e + a.rest - 1) / a.rest + min(q, r);
    }
    // LDS words of the transforms' writes and the MFMAs' reads.
    const int wr = (tl >> 2) * WG_STEP + (wave >> 1) * 4 * WG_Q + (tl & 3) * 68 +
                   ((wave & 1) * 8 + c8) * 4;
    const int rd = kr * 68 + lc * 4;

    // Cursor of the loads, two stages ahead of the MFMAs.
    Unit pu{};
    int pk = -1, ps = 0, pty = 0, ph0 = 0;  // unit, stage, tile row, first patch row of row 0
    bool more = true, fresh = true;      // fresh: the strip's first stage here
    uint32_t xo[XL], yo[YL];
    auto advance = [&]() __attribute__((always_inline)) {
        if (pk >= 0) {
            ps++;
            pty++;
            fresh = false;
            if (ps < pu.s1 && pty < a.Pt)
                return;
        }
        const WinoWgArgs &c = cold_args<WinoWgArgs>();
        if (pk < 0 || ps >= pu.s1) {
            const int nunits = c.rounds + (c.rest ? 2 : 0);
            do {
                if (++pk >= nunits) {
                    more = false;
                    return;
                }
                pu = wino_unit(c, w, pk);
            } while (pu.s0 >= pu.s1);
            ps = pu.s0;
        }
        fresh = true;
        const int st = (int)fast_div((uint32_t)ps, c.d_pt);  // (image group, strip)
        pty = ps - st * c.Pt;
        const int ig = (int)fast_div((uint32_t)st, c.d_strips), strip = st - ig * c.nstrip;
        const WgTile tile = wg_tile(c, pu.tile);
        const int cb = tile.cb, gm = tile.gm;
        const int g = (int)fast_div((uint32_t)gm, c.d_kblocks), kb = gm - g * c.kblocks;
        const int tx = strip * c.cw + (tl & (c.cw - 1));
        const int img = ig * (8 >> c.cw_log) + (tl >> c.cw_log);
        const int k = kb * 64 + wave * 8 + c8, ch = cb * 64 + wave * 8 + c8;
        const bool in = tx < c.Qt && img < c.nimg;
        const int w0 = 2 * (tx + tile.pw) + c.off;
        ph0 = 2 * tile.ph + c.off;
        const uint32_t xb = ((uint32_t)img * c.x_img_words + (uint32_t)((g * c.Cg + ch) * c.HW)) * 4u;
#pragma unroll
        for (int l = 0; l < XL; l++) {
            const int col = w0 + Patch<MODE>::col(l);
            xo[l] = in && ch < c.Cg && (unsigned)col < (unsigned)c.W ? xb + (uint32_t)col * 4u : kOob;
        }
        const uint32_t yb = ((uint32_t)img * c.dy_img_words + (uint32_t)((g * c.Kg + k) * c.PQ)) * 4u;
#pragma unroll
        for (int l = 0; l < YL; l++)
            yo[l] = in && k < c.Kg && 2 * tx + l < c.Q ? yb + (uint32_t)(2 * tx + l) * 4u : kOob;
    };
    // Rows i, i + 1 of the patches of tile row pty into d.  (A row outside the
    // image reads zero through an empty buffer: a branch around the load would
    // make the compiler wait for it where the branches meet.)
    auto load_x = [&](int i, float (&d)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const int h = 2 * pty + ph0 + i + r;
            const bool ok = more && (unsigned)h < (unsigned)a.H;
            load_row<MODE>(make_rsrc(a.x, ok ? a.x_bytes : 0u), xo,
                           ok ? (uint32_t)(h * a.W) * 4u : 0u, d + 4 * r);
        }
    };
    auto load_y = [&](float (&g)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const bool ok = more && 2 * pty + r < a.P;
            const __amdgpu_buffer_rsrc_t rY = make_rsrc(a.dy, ok ? a.dy_bytes : 0u);
            const uint32_t soff = ok ? (uint32_t)((2 * pty + r) * a.Q) * 4u : 0u;
            if constexpr (YL == 1) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rY, (int)yo[0], soff, 0);
                const uint32_t hi = v[1];
                g[2 * r] = __uint_as_float(v[0]);
                g[2 * r + 1] = __uint_as_float(hi);
            } else {
#pragma unroll
                for (int l = 0; l < YL; l++)
                    g[2 * r + l] =
                        __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rY, (int)yo[l], soff, 0));
            }
        }
    };
    float db = 0.f;  // this lane's filter and tiles, of the stages transformed so far
    auto write = [&](float *Yd, float *Xd, const float (&lo)[8], const float (&hi)[8],
                     const float (&g)[4]) __attribute__((always_inline)) {
        float d[16], v[16];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            d[j] = lo[j];
            d[8 + j] = hi[j];
        }
        input_transform(d, v);
#pragma unroll
        for (int q = 0; q < 4; q++)
            *(LDS_AS f32x4 *)(Xd + wr + q * WG_Q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        dy_transform(g, v);
#pragma unroll
        for (int q = 0; q < 4; q++)
            *(LDS_AS f32x4 *)(Yd + wr + q * WG_Q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        db += v[5];  // the sum of the tile
    };

    f32x4 acc[2][16];
    f32x4 u[2][2], v[2];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int p = 0; p < 16; p++)
                acc[b][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto read_ops = [&](const float *Yc, const float *Xc, int g8) __attribute__((always_inline)) {
        const int step = g8 >> 2, q = g8 & 3;
#pragma unroll
        for (int b = 0; b < 2; b++)
            u[q & 1][b] = lds_b128(Yc, rd + step * WG_STEP + ((fg * 2 + b) * 4 + q) * WG_Q);
        v[q & 1] = lds_b128(Xc, rd + step * WG_STEP + (cg * 4 + q) * WG_Q);
    };
    // Sums of unit un: to its slab, or (whole tiles) to dw and db.
    // add: onto what an earlier part of the unit has stored there.
    auto finish = [&](const Unit &un, bool add, bool end, float bias) __attribute__((always_inline)) {
        const WinoWgArgs &c = cold_args<WinoWgArgs>();
        const WgTile tile = wg_tile(c, un.tile);
        const int cb = tile.cb, gm = tile.gm, part = tile.part;
        const int g = (int)fast_div((uint32_t)gm, c.d_kblocks), kb = gm - g * c.kblocks;
        float *const slab = un.slab >= 0 ? c.slabs + (size_t)un.slab * WG_SLAB : nullptr;
        const int Kg = c.Kg, Cg = c.Cg, ch = cb * 64 + cg * 16 + lc;
        const int R = c.R, i0 = tile.ph > 0, j0 = tile.pw > 0;  // taps that an earlier part holds
        float *const dw = c.dw + (size_t)g * Kg * Cg * R * R + 2 * tile.ph * R + 2 * tile.pw;
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int row = fg * 32 + b * 16 + 4 * kr + r, k = kb * 64 + row;
                float x[16], t[9];
#pragma unroll
                for (int p = 0; p < 16; p++)
                    x[p] = acc[b][p][r];
                tap_transform(x, t);
                // (Loads together, then stores: not each store behind its load.)
                if (slab) {
                    float *const o = slab + (row * 64 + cg * 16 + lc) * 9;
                    if (add) {
#pragma unroll
                        for (int j = 0; j < 9; j++)
                            t[j] += o[j];
                    }
#pragma unroll
                    for (int j = 0; j < 9; j++)
                        o[j] = t[j];
                } else if (k < Kg && ch < Cg) {
                    float *const o = dw + ((size_t)k * Cg + ch) * R * R;
                    if (add) {
#pragma unroll
                        for (int j = 0; j < 9; j++)
                            if (j / 3 >= i0 && j % 3 >= j0)
                                t[j] += o[j / 3 * R + j % 3];
                    }
#pragma unroll
                    for (int j = 0; j < 9; j++)
                        if (j / 3 >= i0 && j % 3 >= j0)
                            o[j / 3 * R + j % 3] = t[j];
                }
            }
        if (!end)
            return;
        // The eight tiles' sums of a filter, in a fixed order.
        bias += __shfl_xor(bias, 1);
        bias += __shfl_xor(bias, 2);
        bias += __shfl_xor(bias, 4);
        if (tl == 0) {
            if (slab)
                slab[64 * 64 * 9 + wave * 8 + c8] = bias;
            else if (c.db && cb == 0 && part == 0 && kb * 64 + wave * 8 + c8 < Kg)
                c.db[g * Kg + kb * 64 + wave * 8 + c8] = bias;
        }
    };

    // The MFMAs' cursor.  A unit's sums are stored every `part` stages, in equal
    // parts of at most c.most, so that no accumulation runs longer than that.
    Unit cu{};
    int ck = -1, cs = 0, part = 0, left = 0;
    auto step_cursor = [&]() __attribute__((always_inline)) {
        if (ck >= 0 && ++cs < cu.s1)
            return;
        const WinoWgArgs &c = cold_args<WinoWgArgs>();
        const int nunits = c.rounds + (c.rest ? 2 : 0);
        do {
            if (++ck >= nunits)
                return;
            cu = wino_unit(c, w, ck);
        } while (cu.s0 >= cu.s1);
        cs = cu.s0;
        const int len = cu.s1 - cu.s0;
        int n = 1;
        while (n * c.most < len)
            n++;
        part = left = (len + n - 1) / n;
    };

    // As in wino_gemm_kernel: MFMAs from (Yc, Xc), transforms of the next stage
    // into (Yn, Xn) from the patch rows lo, hi, loads of the one after it into
    // hi's successor lo (and hi's own rows, where it opens a strip).
    bool have1, have2;
    float g[4];
    auto stage = [&](float *Yc, float *Xc, float *Yn, float *Xn, float (&lo)[8],
                     float (&hi)[8]) __attribute__((always_inline)) {
        const bool last = cs + 1 == cu.s1, store = last || left == 1;
        left--;
        float bias = 0.f;  // of this unit, once its last stage is transformed
#pragma unroll
        for (int g8 = 0; g8 < 8; g8++) {
            const int q = g8 & 3;
            if (g8 == 7) {
                __builtin_amdgcn_s_waitcnt((15 | 3 << 14) | (7 << 4));  // LDS; loads may fly on
                fence();
                __builtin_amdgcn_s_barrier();
                fence();
            }
            read_ops(g8 < 7 ? Yc : Yn, g8 < 7 ? Xc : Xn, (g8 + 1) & 7);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; j++)
#pragma unroll
                for (int b = 0; b < 2; b++)
                    acc[b][4 * q + j] = mfma16(u[q & 1][b][j], v[q & 1][j], acc[b][4 * q + j]);
            __builtin_amdgcn_sched_barrier(0);
            if (g8 == 0) {
                if (last) {  // the unit's stages are all transformed
                    bias = db;
                    db = 0.f;
                }
                if (have1)
                    write(Yn, Xn, lo, hi, g);
                __builtin_amdgcn_sched_barrier(0);
                advance();
                have2 = more;
                if (fresh)
                    load_x(0, hi);
                load_x(2, lo);
                load_y(g);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (store) {
            finish(cu, cs + 1 - cu.s0 > part, last, bias);
            clear();
            left = part;
        }
        step_cursor();
        const bool on = have1;
        have1 = have2;
        return on;
    };

    float ra[8], rb[8];
    advance();
    if (!more)
        return;
    load_x(0, ra);
    load_x(2, rb);
    load_y(g);
    write(Y0, X0, ra, rb, g);
    step_cursor();
    advance();
    have1 = more;
    if (have1) {
        if (fresh)
            load_x(0, rb);
        load_x(2, ra);
        load_y(g);
    }
    clear();
    __builtin_amdgcn_s_waitcnt(0);
    fence();
    __builtin_amdgcn_s_barrier();
    fence();
    read_ops(Y0, X0, 0);
    // The operands read past a workgroup's last stage are not used.
    while (stage(Y0, X0, Y1, X1, rb, ra) && stage(Y1, X1, Y0, X0, ra, rb)) {
    }
}

// Direct sums of the filter gradients `bad` (bit j: tap j of the tile's part) of
// filter row and channel (row, ch) of an output tile.  All lanes of a wave call
// it: a lane sums every 64th 2 x 2 tile of dy, from the 4 x 4 patch of x under
// it, then the lanes' sums are added in a fixed order.  The padding's zeros are
// multiplied too, as in the direct plans.
//
// With every gradient plus infinity the pass takes 8.0 ms on 64 -> 64 channels,
// 112 x 112, batch 32 (a block an element, one after another: 80; the direct plan:
// 0.25), 4.4 on 512 -> 512, 14 x 14 (31; 0.29); with NaNs 0.18 (1.7) and 0.87 (2.1).
__device__ __forceinline__ void wino_wgrad_direct(const WinoWgArgs &a, const WgTile &wt, int row, int ch,
                                                  int bad, float (&t)[9])
{
    const int lane = threadIdx.x & 63;
    const int g = wt.gm / a.kblocks, k = (wt.gm - g * a.kblocks) * 64 + row, c = wt.cb * 64 + ch;
    const __amdgpu_buffer_rsrc_t rX = make_rsrc(a.x, a.x_bytes), rY = make_rsrc(a.dy, a.dy_bytes);
    const int xs = __builtin_amdgcn_readfirstlane((g * a.Cg + c) * a.HW * 4);
    const int ys = __builtin_amdgcn_readfirstlane((g * a.Kg + k) * a.PQ * 4);
    const int tiles = a.nimg * a.Pt * a.Qt;
#pragma unroll
    for (int j = 0; j < 9; j++)
        t[j] = 0.f;
    int live = bad;  // what no lane has as a NaN yet (a NaN stays one)
    for (int i0 = 0, step = 0; i0 < tiles && live; i0 += 64, step++) {
        const int i = i0 + lane, r = (int)fast_div((uint32_t)i, a.d_qt), tx = i - r * a.Qt;
        const int img = (int)fast_div((uint32_t)r, a.d_pt), ty = r - img * a.Pt;
        const int h0 = i < tiles ? 2 * (ty + wt.ph) + a.off : -4, w0 = 2 * (tx + wt.pw) + a.off;
        const uint32_t yo = (uint32_t)img * a.dy_img_words + (uint32_t)(2 * ty * a.Q + 2 * tx);
        const uint32_t xo = (uint32_t)img * a.x_img_words + (uint32_t)(h0 * a.W + w0);
        const bool row2 = 2 * ty + 1 < a.P, col2 = 2 * tx + 1 < a.Q;
        float y[4], x[16];
#pragma unroll
        for (int e = 0; e < 4; e++)
            y[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rY, i < tiles && (e < 2 || row2) && (e % 2 == 0 || col2)
                        ? (int)((yo + (uint32_t)(e / 2 * a.Q + e % 2)) * 4u)
                        : (int)kOob,
                ys, 0));
#pragma unroll
        for (int e = 0; e < 16; e++)
            x[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rX, (unsigned)(h0 + e / 4) < (unsigned)a.H && (unsigned)(w0 + e % 4) < (unsigned)a.W
                        ? (int)((xo + (uint32_t)(e / 4 * a.W + e % 4)) * 4u)
                        : (int)kOob,
                xs, 0));
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const bool ok = i < tiles && (e < 2 || row2) && (e % 2 == 0 || col2);
#pragma unroll
            for (int j = 0; j < 9; j++) {
                const float v = fmaf(y[e], x[4 * (e / 2 + j / 3) + e % 2 + j % 3], t[j]);
                t[j] = ok ? v : t[j];  // no pixel, no product
            }
        }
        if ((step & 3) == 3) {
#pragma unroll
            for (int j = 0; j < 9; j++)
                live &= __builtin_amdgcn_ballot_w64(t[j] != t[j]) ? ~(1 << j) : ~0;
        }
    }
#pragma unroll
    for (int j = 0; j < 9; j++)
#pragma unroll
        for (int d = 1; d < 64; d *= 2)
            t[j] += __shfl_xor(t[j], d);
}

// Ends the pass: adds the slabs of cut output tiles, and recomputes filter
// gradients that are not finite as direct sums (see wino_finish_kernel).  A
// block is 32 quads of one tile's words, eight threads to a quad: each sums
// every eighth slab, then the eight sums are added in order.
constexpr int WG_BLOCKS = WG_SLAB / 128 + 1;
__global__ __launch_bounds__(256) void wino_wgrad_finish_kernel(const WinoWgArgs a)
{
    __shared__ f32x4 part[8][32];
    __shared__ int bad[32];
    const int tile = blockIdx.x / WG_BLOCKS, r = tile - a.rounds * a.nwg;
    const int lane = threadIdx.x & 31, j = threadIdx.x >> 5;
    const int e = ((blockIdx.x - tile * WG_BLOCKS) * 32 + lane) * 4;
    const WgTile wt = wg_tile(a, tile);
    const int gm = wt.gm, cb = wt.cb, g = gm / a.kblocks, kb = gm - g * a.kblocks, taps = a.R * a.R;
    // Word m of filter row `row` of the tile: channel m / 9, tap (m % 9 / 3, m % 3)
    // of the part; -1 for a tap that an earlier part holds.
    float *const dw = a.dw + ((size_t)(g * a.Kg + kb * 64) * a.Cg + cb * 64) * taps;
    auto place = [&](int row, int m) {
        if (a.parts == 1)
            return (long long)row * a.Cg * 9 + m;
        const int c = m / 9, i = (m - c * 9) / 3, z = m - c * 9 - i * 3;
        return (i == 0 && wt.ph > 0) || (z == 0 && wt.pw > 0)
                   ? -1LL
                   : ((long long)row * a.Cg + c) * taps + (2 * wt.ph + i) * a.R + 2 * wt.pw + z;
    };
    const int hi = (r + 1) * a.nstage, w0 = r >= 0 ? wino_first_share(a, r) : 0;
    const bool cut = r >= 0 && share(a, w0 + 1) < hi;  // else its workgroup has written dw
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    if (cut) {
        if (e < WG_SLAB)
            for (int w = w0 + j; w < a.nwg && share(a, w) < hi; w += 8)
                if (share(a, w) < share(a, w + 1)) {
                    const f32x4 y = *(const f32x4 *)(a.slabs + (size_t)(w + r) * WG_SLAB + e);
                    s = f32x4{s[0] + y[0], s[1] + y[1], s[2] + y[2], s[3] + y[3]};
                }
        part[j][lane] = s;
    }
    __syncthreads();
    int mask = 0;
    if (j == 0 && e < WG_SLAB) {
        if (cut)
#pragma unroll
            for (int i = 1; i < 8; i++) {
                const f32x4 y = part[i][lane];
                s = f32x4{s[0] + y[0], s[1] + y[1], s[2] + y[2], s[3] + y[3]};
            }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int n = e + i, row = n / 576, m = n - row * 576;
            if (n >= 64 * 64 * 9) {
                const int k = kb * 64 + n - 64 * 64 * 9;
                if (cut && a.db && cb == 0 && wt.part == 0 && k < a.Kg)
                    a.db[g * a.Kg + k] = s[i];
            } else if (kb * 64 + row < a.Kg && cb * 64 + m / 9 < a.Cg) {
                const long long at = place(row, m);
                if (at < 0)
                    continue;
                if (cut)
                    dw[at] = s[i];
                mask |= is_finite(cut ? s[i] : dw[at]) ? 0 : 1 << i;
            }
        }
    }
    if (j == 0)
        bad[lane] = mask;
    if (!__syncthreads_or(mask))
        return;
    // A wave for each (filter row, channel) among the block's words.
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int n0 = (blockIdx.x - tile * WG_BLOCKS) * 128;
    for (int q = n0 / 9 + wave; q * 9 < min(n0 + 128, 64 * 64 * 9); q += 4) {
        const int n = q * 9 + l - n0;
        const int which = (int)__builtin_amdgcn_ballot_w64(l < 9 && (unsigned)n < 128u &&
                                                           (bad[(n & 127) >> 2] >> (n & 3) & 1));
        if (!which)
            continue;
        float t[9];
        wino_wgrad_direct(cold_args<WinoWgArgs>(), wt, q >> 6, q & 63, which, t);
        if (l == 0)
#pragma unroll
            for (int j = 0; j < 9; j++)
                if (which & (1 << j))
                    dw[place(q >> 6, (q & 63) * 9 + j)] = t[j];
    }
}

// ---------------------------------------------------------------- launches
// Parts of an R x R filter along an axis (R = 3 or 5).
static int wino_parts(int R)
{
    return (R - 1) / 2;
}

// Channel blocks of 64, stages of 8 channels (cin is a multiple of 8) of a part.
size_t wino_filter_words(int M, int cin, int groups, int R)
{
    return (size_t)groups * ((M + 63) / 64) * (cin / 8) * wino_parts(R) * wino_parts(R) * 8192;
}

// Work of n output tiles of nstage stages on cus workgroups, each at least
// `least` stages.
static WinoWork wino_work(long long n, int nstage, int cus, int least)
{
    WinoWork w{};
    const long long most = n * nstage / least;
    w.nwg = (int)(most < 1 ? 1 : most < cus ? most : cus);
    w.nstage = nstage;
    w.rounds = (int)(n / w.nwg);
    w.rest = (int)(n % w.nwg);
    w.share = (int)((long long)w.rest * nstage / w.nwg);
    w.share_rem = (int)((long long)w.rest * nstage % w.nwg);
    w.d_nstage = make_fastdiv(nstage);
    return w;
}

WinoWork wino_plan(int M, int cin, int groups, int R, int nimg, int P, int Q, int cus)
{
    const long long tiles = (long long)nimg * ((P + 1) / 2) * ((Q + 1) / 2);
    return wino_work((long long)groups * ((M + 63) / 64) * ((tiles + 63) / 64),
                     cin / 8 * wino_parts(R) * wino_parts(R), cus, 4);
}

size_t wino_slab_bytes(const WinoWork &w)
{
    return w.rest ? (size_t)(w.nwg + w.rest) * 65536 : 0;
}

hipError_t launch_wino(WinoArgs a, const WinoWork &p, float *U, hipStream_t stream)
{
    static_cast<WinoWork &>(a) = p;
    a.U = U;
    a.Pt = (a.P + 1) / 2;
    a.Qt = (a.Q + 1) / 2;
    a.tiles = a.nimg * a.Pt * a.Qt;
    a.tblocks = (a.tiles + 63) / 64;
    a.mblocks = (a.M + 63) / 64;
    a.parts = wino_parts(a.R);
    a.ncb = a.cin / 8;
    a.d_ncb = make_fastdiv(a.ncb);
    a.d_tblocks = make_fastdiv(a.tblocks);
    a.d_mblocks = make_fastdiv(a.mblocks);
    a.d_qt = make_fastdiv(a.Qt);
    a.d_pt = make_fastdiv(a.Pt);
    const long long fb = (long long)a.groups * a.mblocks * a.nstage * 2;
    wino_filter_kernel<<<dim3((unsigned)fb), 256, 0, stream>>>(a, U);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    if (a.before && (e = hipEventRecord(a.before, stream)) != hipSuccess)
        return e;
    const dim3 grid((unsigned)p.nwg);
    const int mode = (a.off & 1 ? 0 : 2) + (a.src_w & 1);
    if (mode == 0)
        wino_gemm_kernel<1, false><<<grid, 512, 0, stream>>>(a);
    else if (mode == 1)
        wino_gemm_kernel<1, true><<<grid, 512, 0, stream>>>(a);
    else if (mode == 2)
        wino_gemm_kernel<2, false><<<grid, 512, 0, stream>>>(a);
    else
        wino_gemm_kernel<2, true><<<grid, 512, 0, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if (a.after && (e = hipEventRecord(a.after, stream)) != hipSuccess)
        return e;
    const dim3 blocks((unsigned)std::max(p.rest * 16, 8 * p.nwg));
    if (a.R == 3)
        wino_finish_kernel<3><<<blocks, 256, 0, stream>>>(a);
    else
        wino_finish_kernel<5><<<blocks, 256, 0, stream>>>(a);
    return hipGetLastError();
}

// Output tiles of backward-weight, and the threads of its last launch.
static long long wino_wgrad_tiles(int Kg, int Cg, int groups, int R)
{
    return (long long)groups * ((Kg + 63) / 64) * ((Cg + 63) / 64) * wino_parts(R) * wino_parts(R);
}

long long wino_wgrad_finish_threads(int Kg, int Cg, int groups, int R)
{
    return wino_wgrad_tiles(Kg, Cg, groups, R) * WG_BLOCKS * 256;
}

// Columns of a stage's eight tiles: 8, or 4 of two or 2 of four images where
// that leaves fewer lanes idle (28 x 28 maps, 14 tiles wide, 512 channels:
// 0.521 ms with 2 columns, 0.560 with 8; one column of eight images was 17-28 %
// slower than 8 columns with one idle on 14 x 14 maps: its loads touch eight
// times the cache lines).
WinoWork wino_wgrad_plan(int Kg, int Cg, int groups, int R, int nimg, int P, int Q, int cus, int *cw)
{
    const int Pt = (P + 1) / 2, Qt = (Q + 1) / 2;
    auto strips = [&](int c) { return (long long)((Qt + c - 1) / c) * ((nimg + 8 / c - 1) / (8 / c)); };
    *cw = 8;
    for (int c : {4, 2})
        if (strips(c) < strips(*cw))
            *cw = c;
    return wino_work(wino_wgrad_tiles(Kg, Cg, groups, R), (int)(strips(*cw) * Pt), cus, 8);
}

size_t wino_wgrad_slab_bytes(const WinoWork &w)
{
    return w.rest ? (size_t)(w.nwg + w.rest) * WG_SLAB * 4 : 0;
}

hipError_t launch_wino_wgrad(WinoWgArgs a, const WinoWork &p, int cw, hipStream_t stream)
{
    static_cast<WinoWork &>(a) = p;
    a.cw = cw;
    a.cw_log = cw == 8 ? 3 : cw == 4 ? 2 : 1;
    a.Pt = (a.P + 1) / 2;
    a.Qt = (a.Q + 1) / 2;
    a.nstrip = (a.Qt + cw - 1) / cw;
    a.kblocks = (a.Kg + 63) / 64;
    a.cblocks = (a.Cg + 63) / 64;
    a.d_pt = make_fastdiv(a.Pt);
    a.d_qt = make_fastdiv(a.Qt);
    a.d_strips = make_fastdiv(a.nstrip);
    a.parts = wino_parts(a.R);
    a.d_parts = make_fastdiv(a.parts * a.parts);
    a.d_cblocks = make_fastdiv(a.cblocks);
    a.d_kblocks = make_fastdiv(a.kblocks);
    hipError_t e;
    if (a.before && (e = hipEventRecord(a.before, stream)) != hipSuccess)
        return e;
    const dim3 grid((unsigned)p.nwg);
    if (a.W & 1)
        wino_wgrad_kernel<0><<<grid, 512, 0, stream>>>(a);
    else if (a.off & 1)
        wino_wgrad_kernel<1><<<grid, 512, 0, stream>>>(a);
    else
        wino_wgrad_kernel<2><<<grid, 512, 0, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess ||
        (a.after && (e = hipEventRecord(a.after, stream)) != hipSuccess))
        return e;
    const long long blocks = ((long long)p.rounds * p.nwg + p.rest) * WG_BLOCKS;
    wino_wgrad_finish_kernel<<<dim3((unsigned)blocks), 256, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace miconv
