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
#include "internal.h"

namespace miconv {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

namespace {

constexpr uint32_t kOob = 0x80000000u;  // beyond any buffer of < 2^31 bytes

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

// The 4 x 4 patch of a tile and channel, by buffer loads: off holds one offset
// per load (out of range: zero), soff the stage's.  MODE 0: one word each;
// 1: columns 0, (1, 2), 3; 2: columns (0, 1), (2, 3).
template <int MODE>
struct Patch {
    static constexpr int LOADS = MODE == 0 ? 4 : MODE == 1 ? 3 : 2;  // a row
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int MODE>
__device__ __forceinline__ void load_patch(__amdgpu_buffer_rsrc_t r,
                                           const uint32_t (&off)[4 * Patch<MODE>::LOADS],
                                           uint32_t soff, float (&d)[16])
{
    constexpr int L = Patch<MODE>::LOADS;
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int l = 0; l < L; l++) {
            const int c = MODE == 0 ? l : MODE == 1 ? (l ? l + l / 2 : 0) : 2 * l;  // first column
            if (MODE == 2 || (MODE == 1 && l == 1)) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off[i * L + l], soff, 0);
                d[4 * i + c] = __uint_as_float(v[0]);
                d[4 * i + c + 1] = __uint_as_float(v[1]);
            } else {
                d[4 * i + c] =
                    __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off[i * L + l], soff, 0));
            }
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
__device__ __forceinline__ const WinoArgs &cold_args()
{
    typedef const __attribute__((address_space(4))) WinoArgs *Ptr;
    Ptr p = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(p));
    return *(const WinoArgs *)p;
}

// Work of one workgroup: the rounds of whole output tiles (tile = round
// nwg + its place), then its share of the stages of the remaining tiles.
struct Unit {
    int tile, s0, s1, slab;  // stages [s0, s1); slab -1: the whole tile
};
// First stage, among those of the remaining tiles, of workgroup w's share.
__device__ __forceinline__ int share(const WinoArgs &a, int w)
{
    return w * a.share + min(w, a.share_rem);
}
__device__ __forceinline__ Unit wino_unit(const WinoArgs &a, int w, int k)
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
    u.slab = u.s0 == 0 && u.s1 == a.nstage ? -1 : 2 * w + i;
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
// MFMA of its SIMD (measured: one v_add after every MFMA takes 39 cycles a
// pair instead of 32, six 50), so the transform's additions cost MFMA time;
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
template <int MODE>
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

    // Cursor of the loads, two stages ahead of the MFMAs.
    Unit pu{};
    int pk = -1, ps = 0;     // unit, stage
    uint32_t pu_base = 0;    // its filters
    uint32_t off[NOFF];      // its patches
    bool more = true;
    auto advance = [&]() __attribute__((always_inline)) {
        if (pk >= 0 && ++ps < pu.s1)
            return;
        const WinoArgs &a = cold_args();
        const int nunits = a.rounds + (a.rest ? 2 : 0);
        do {
            if (++pk >= nunits) {
                more = false;
                return;
            }
            pu = wino_unit(a, w, pk);
        } while (pu.s0 >= pu.s1);
        ps = pu.s0;
        const int gm = (int)fast_div((uint32_t)pu.tile, a.d_tblocks);  // (group, channel block)
        const int tb = pu.tile - gm * a.tblocks, g = (int)fast_div((uint32_t)gm, a.d_mblocks);
        pu_base = (uint32_t)gm * (uint32_t)a.nstage * (STG * 4u);
        const int t = tb * 64 + tg * 16 + lc;
        const TileAt at = tile_at(a, min(t, a.tiles - 1));
        const int h0 = 2 * at.ty + a.off, w0 = 2 * at.tx + a.off;
        const uint32_t base = ((uint32_t)at.img * a.src_img_words +
                               (uint32_t)(g * a.cin + 4 * half + kr) * (uint32_t)a.src_hw) * 4u;
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int l = 0; l < Patch<MODE>::LOADS; l++) {
                const int c = MODE == 0 ? l : MODE == 1 ? (l ? l + l / 2 : 0) : 2 * l;
                const bool ok = (unsigned)(h0 + i) < (unsigned)a.src_h &&
                                (unsigned)(w0 + c) < (unsigned)a.src_w;
                off[i * Patch<MODE>::LOADS + l] =
                    ok ? base + (uint32_t)((h0 + i) * a.src_w + w0 + c) * 4u : kOob;
            }
    };
    auto load_u = [&](float *Ud, uint32_t base, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < 4; l++) {
            const int i = wave + 8 * l;
            dma16(rU, Ud + i * 256, (uint32_t)lane * 16u + (uint32_t)i * 1024u,
                  base + (uint32_t)s * (STG * 4u));
        }
    };
    auto write_v = [&](float *Vd, const float (&d)[16]) __attribute__((always_inline)) {
        float v[16];
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
        const WinoArgs &c = cold_args();
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
        const uint32_t o1 = p + 1 < P ? 0u : kOob;  // the tile's second row
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
                const uint32_t o = t < c.tiles && m0 + b * 16 + r < M
                                       ? o0 + (uint32_t)((b * 16 + r) * hw) * 4u
                                       : kOob;
                const uint32_t oq = o | o1, Qb = (uint32_t)Q * 4u;
                if ((Q & 1) == 0) {
                    __builtin_amdgcn_raw_buffer_store_b64(
                        u32x2{__float_as_uint(y[0]), __float_as_uint(y[1])}, rO, o, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(
                        u32x2{__float_as_uint(y[2]), __float_as_uint(y[3])}, rO, oq + Qb, 0, 0);
                } else {
                    const uint32_t s = q + 1 < Q ? 0u : kOob;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[0]), rO, o, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[1]), rO, (o | s) + 4, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[2]), rO, oq + Qb, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y[3]), rO, (oq | s) + Qb + 4, 0, 0);
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
        const WinoArgs &a = cold_args();
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
                    load_patch<MODE>(rX, off, (uint32_t)ps * stage_bytes, d);
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
    load_patch<MODE>(rX, off, (uint32_t)ps * stage_bytes, d);
    write_v(V0, d);
    step_cursor();
    advance();
    have1 = more;
    if (have1) {
        load_u(U1, pu_base, ps);
        load_patch<MODE>(rX, off, (uint32_t)ps * stage_bytes, d);
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

// One output pixel directly: the sum over channels and taps in order.
__device__ float wino_direct(const WinoArgs &a, int img, int oc, int p, int q)
{
    const int g = oc / a.M, m = oc - g * a.M;
    float s = 0.f;
    for (int c = 0; c < a.cin; c++) {
        const float *x = a.src + (size_t)img * a.src_img_words + (size_t)(g * a.cin + c) * a.src_hw;
        const float *wt = a.flip ? a.w + ((size_t)(g * a.cin + c) * a.M + m) * 9
                                 : a.w + ((size_t)(g * a.M + m) * a.cin + c) * 9;
        for (int r = 0; r < 3; r++)
            for (int z = 0; z < 3; z++) {
                const int h = p + a.off + r, w = q + a.off + z, k = r * 3 + z;
                if ((unsigned)h < (unsigned)a.src_h && (unsigned)w < (unsigned)a.src_w)
                    s = fmaf(x[h * a.src_w + w], wt[a.flip ? 8 - k : k], s);
            }
    }
    return s + (a.bias ? a.bias[oc] : 0.f);
}

// The workgroup whose share holds the first stage of remaining tile r.
__device__ __forceinline__ int wino_first_share(const WinoArgs &a, int r)
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
// if the GEMM raised the flag.
__global__ __launch_bounds__(256) void wino_finish_kernel(const WinoArgs a)
{
    if (a.rest) {
        const int r = blockIdx.x >> 4, e = (blockIdx.x & 15) * 256 + threadIdx.x;
        const int hi = (r + 1) * a.nstage;
        int w = wino_first_share(a, r);
        if (share(a, w + 1) < hi) {
            f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
            for (; w < a.nwg && share(a, w) < hi; w++) {
                const int lo_w = share(a, w);
                if (lo_w == share(a, w + 1))
                    continue;
                const int slab = 2 * w + (lo_w / a.nstage == r ? 0 : 1);
                const f32x4 s = *(const f32x4 *)(a.slabs + (size_t)slab * 16384 + e * 4);
                y = f32x4{y[0] + s[0], y[1] + s[1], y[2] + s[2], y[3] + s[3]};
            }
            const int tile = a.rounds * a.nwg + r;
            const int gm = tile / a.tblocks, tb = tile - gm * a.tblocks;
            const int g = gm / a.mblocks, m = (gm - g * a.mblocks) * 64 + (e >> 6);
            const int t = tb * 64 + (e & 63);
            if (m < a.M && t < a.tiles) {
                const TileAt at = tile_at(a, t);
                const int oc = g * a.M + m;
                const float bv = a.bias ? a.bias[oc] : 0.f;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    y[k] += bv;
                    if (!is_finite(y[k]))
                        y[k] = wino_direct(a, at.img, oc, 2 * at.ty + (k >> 1), 2 * at.tx + (k & 1));
                }
                store_tile(a, at, oc, y);
            }
        }
    }
    if (*a.flag) {
        const long long total = (long long)a.nimg * a.out_img_stride;
        for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total;
             i += (long long)gridDim.x * 256) {
            if (is_finite(a.out[i]))
                continue;
            const int img = (int)(i / a.out_img_stride);
            const long long r = i - (long long)img * a.out_img_stride;
            const int oc = (int)(r / a.out_hw), pq = (int)(r - (long long)oc * a.out_hw);
            const int p = pq / a.Q, q = pq - p * a.Q;
            // A cut output tile's pixels are another block's (above).
            const int g = oc / a.M, t = (img * a.Pt + p / 2) * a.Qt + q / 2;
            const int rest = (g * a.mblocks + (oc - g * a.M) / 64) * a.tblocks + t / 64 - a.rounds * a.nwg;
            if (rest >= 0) {
                const int w = wino_first_share(a, rest);
                if (share(a, w + 1) < (rest + 1) * a.nstage)
                    continue;
            }
            a.out[i] = wino_direct(a, img, oc, p, q);
        }
    }
}

// Filter transform U = G g Gt into the order the GEMM reads: word
// ((((gm nstage + s) 2 + step) 4 + b) 4 + q) 256 + lane 4 + j is point 4 q + j
// of row m = 64 mb + 16 b + lane % 16, channel c = 8 s + 4 step + lane / 16 of
// group g, gm = g mblocks + mb (zero past M).  flip (backward-data): row m is
// input channel m, channel c filter c, the taps mirrored.  Also lowers the flag.
__global__ __launch_bounds__(256) void wino_filter_kernel(const WinoArgs a, float *__restrict__ U)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0)
        *a.flag = 0;
    const int lane = i & 63, b = (i >> 6) & 3, step = (i >> 8) & 1;
    const int r = i >> 9, gm = r / a.nstage, s = r - gm * a.nstage;
    const int g = gm / a.mblocks, mb = gm - g * a.mblocks;
    const int m = mb * 64 + b * 16 + (lane & 15), c = s * 8 + step * 4 + (lane >> 4);
    float k[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (m < a.M) {
        const float *src = a.flip ? a.w + ((size_t)(g * a.cin + c) * a.M + m) * 9
                                  : a.w + ((size_t)(g * a.M + m) * a.cin + c) * 9;
#pragma unroll
        for (int j = 0; j < 9; j++)
            k[j] = src[a.flip ? 8 - j : j];
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

// ---------------------------------------------------------------- launches
// Channel blocks of 64, stages of 8 channels (cin is a multiple of 8).
size_t wino_filter_words(int M, int cin, int groups)
{
    return (size_t)groups * ((M + 63) / 64) * (cin / 8) * 8192;
}

WinoPlan wino_plan(int M, int cin, int groups, int nimg, int P, int Q, int cus)
{
    WinoPlan p{};
    const long long tiles = (long long)nimg * ((P + 1) / 2) * ((Q + 1) / 2);
    const long long n = (long long)groups * ((M + 63) / 64) * ((tiles + 63) / 64);
    const long long stages = n * (cin / 8);
    // At least four stages a workgroup.
    p.nwg = (int)(stages / 4 < 1 ? 1 : stages / 4 < cus ? stages / 4 : cus);
    p.rounds = (int)(n / p.nwg);
    p.rest = (int)(n % p.nwg);
    p.slab_bytes = p.rest ? (size_t)p.nwg * 2 * 65536 : 0;
    return p;
}

hipError_t launch_wino(WinoArgs a, const WinoPlan &p, float *U, hipStream_t stream)
{
    a.U = U;
    a.Pt = (a.P + 1) / 2;
    a.Qt = (a.Q + 1) / 2;
    a.tiles = a.nimg * a.Pt * a.Qt;
    a.tblocks = (a.tiles + 63) / 64;
    a.mblocks = (a.M + 63) / 64;
    a.nstage = a.cin / 8;
    a.nwg = p.nwg;
    a.rounds = p.rounds;
    a.rest = p.rest;
    a.share = p.rest * a.nstage / p.nwg;
    a.share_rem = p.rest * a.nstage % p.nwg;
    a.d_nstage = make_fastdiv(a.nstage);
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
    // Pairs of columns load together where no pair straddles the map's edge:
    // even widths, from the column whose number is even.
    const dim3 grid((unsigned)p.nwg);
    if (a.src_w & 1)
        wino_gemm_kernel<0><<<grid, 512, 0, stream>>>(a);
    else if (a.off & 1)
        wino_gemm_kernel<1><<<grid, 512, 0, stream>>>(a);
    else
        wino_gemm_kernel<2><<<grid, 512, 0, stream>>>(a);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if (a.after && (e = hipEventRecord(a.after, stream)) != hipSuccess)
        return e;
    wino_finish_kernel<<<dim3(p.rest ? (unsigned)p.rest * 16 : 64), 256, 0, stream>>>(a);
    return hipGetLastError();
}

}  // namespace miconv
