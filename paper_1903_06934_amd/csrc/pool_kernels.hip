// Pooling layer (forward and backward), max with argmax mask or average.
// Memory-bound.  Planes that fit in LDS: one workgroup per (n, c) plane (or
// several small ones), staged once with consecutive loads.  Larger planes: one
// thread per written element, windows read through the caches.  Indices are
// decoded with constant-divisor division.
#include "internal.h"

namespace miconv {

namespace {

// Window of output index p along an axis: inside the image [lo, hi), and
// the extent of the window clipped to the padded image (the average's
// divisor counts padding but not the overhang past it).
struct Win {
    int lo, hi, ext;
};

__device__ __forceinline__ Win window(int p, int stride, int pad, int filt, int in)
{
    const int start = p * stride - pad;
    const int end = min(start + filt, in + pad);
    return Win{max(start, 0), min(end, in), end - start};
}

template <bool MAX>
__global__ __launch_bounds__(256) void pool_fwd_kernel(const float *__restrict__ x,
                                                       float *__restrict__ y,
                                                       int *__restrict__ mask, int H, int W,
                                                       int R, int S, int stride, int pad,
                                                       FastDiv pq, FastDiv q_, uint32_t total)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += gridDim.x * blockDim.x) {
        const uint32_t nc = fast_div(i, pq), pix = i - nc * pq.d;
        const uint32_t p = fast_div(pix, q_), q = pix - p * q_.d;
        const Win wh = window((int)p, stride, pad, R, H), ww = window((int)q, stride, pad, S, W);
        const float *xp = x + (size_t)nc * H * W;
        if constexpr (MAX) {
            // First maximum in row-major order; the window always holds an
            // image element (pad < window, and no window lies past the image),
            // so arg is set.
            float best = -__builtin_inff();
            int arg = -1;
            for (int h = wh.lo; h < wh.hi; h++)
                for (int w = ww.lo; w < ww.hi; w++) {
                    const float v = xp[h * W + w];
                    if (v > best) {
                        best = v;
                        arg = h * W + w;
                    }
                }
            y[i] = best;
            if (mask)
                mask[i] = arg;
        } else {
            float sum = 0.f;
            for (int h = wh.lo; h < wh.hi; h++)
                for (int w = ww.lo; w < ww.hi; w++)
                    sum += xp[h * W + w];
            y[i] = sum / (float)(wh.ext * ww.ext);
        }
    }
}

// dx[h][w] gathers, in the order of the windows (p, then q), the dy of every
// window that covers it: all of it for max when the window's argmax is this
// element, dy / area for the average.  No atomics: each thread writes one dx.
template <bool MAX>
__global__ __launch_bounds__(256) void pool_bwd_kernel(const float *__restrict__ dy,
                                                       const int *__restrict__ mask,
                                                       float *__restrict__ dx, int H, int W,
                                                       int P, int Q, int R, int S, int stride,
                                                       int pad, FastDiv hw, FastDiv w_,
                                                       FastDiv st_, uint32_t total)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += gridDim.x * blockDim.x) {
        const uint32_t nc = fast_div(i, hw), pix = i - nc * hw.d;
        const int h = (int)fast_div(pix, w_), w = (int)(pix - (uint32_t)h * w_.d);
        // windows p with p stride - pad <= h < p stride - pad + R
        const int hp = h + pad, wp = w + pad;  // >= 0
        const int p0 = hp < R ? 0 : (int)fast_div((uint32_t)(hp - R), st_) + 1;
        const int p1 = min((int)fast_div((uint32_t)hp, st_), P - 1);
        const int q0 = wp < S ? 0 : (int)fast_div((uint32_t)(wp - S), st_) + 1;
        const int q1 = min((int)fast_div((uint32_t)wp, st_), Q - 1);
        const size_t base = (size_t)nc * P * Q;
        float acc = 0.f;
        for (int p = p0; p <= p1; p++)
            for (int q = q0; q <= q1; q++) {
                const size_t o = base + (size_t)p * Q + q;
                if constexpr (MAX) {
                    // Both loads issued together; the select keeps the sum's order.
                    const float g = dy[o];
                    acc += mask[o] == (int)pix ? g : 0.f;
                } else {
                    const Win wh = window(p, stride, pad, R, H), ww = window(q, stride, pad, S, W);
                    acc += dy[o] / (float)(wh.ext * ww.ext);
                }
            }
        dx[i] = acc;
    }
}

// Whole-plane variants, for planes that fit in LDS: a workgroup stages one
// (n, c) plane with consecutive (coalesced) loads, then computes that
// plane's outputs from LDS, so every input byte is read from HBM once and in
// order.  Same arithmetic in the same order as the kernels above: the
// results are identical bit for bit.
template <bool MAX>
__global__ __launch_bounds__(256) void pool_fwd_plane_kernel(const float *__restrict__ x,
                                                             float *__restrict__ y,
                                                             int *__restrict__ mask, int H, int W,
                                                             int R, int S, int stride, int pad,
                                                             FastDiv q_, uint32_t P,
                                                             uint32_t planes)
{
    extern __shared__ float xs[];
    const uint32_t hw = (uint32_t)H * (uint32_t)W, pq = P * q_.d;
    for (uint32_t nc = blockIdx.x; nc < planes; nc += gridDim.x) {
        const float *xp = x + (size_t)nc * hw;
        for (uint32_t i = threadIdx.x; i < hw; i += blockDim.x)
            xs[i] = xp[i];
        __syncthreads();
        for (uint32_t o = threadIdx.x; o < pq; o += blockDim.x) {
            const uint32_t p = fast_div(o, q_), q = o - p * q_.d;
            const Win wh = window((int)p, stride, pad, R, H), ww = window((int)q, stride, pad, S, W);
            const size_t out = (size_t)nc * pq + o;
            if constexpr (MAX) {
                float best = -__builtin_inff();
                int arg = -1;
                for (int h = wh.lo; h < wh.hi; h++)
                    for (int w = ww.lo; w < ww.hi; w++) {
                        const float v = xs[h * W + w];
                        if (v > best) {
                            best = v;
                            arg = h * W + w;
                        }
                    }
                y[out] = best;
                if (mask)
                    mask[out] = arg;
            } else {
                float sum = 0.f;
                for (int h = wh.lo; h < wh.hi; h++)
                    for (int w = ww.lo; w < ww.hi; w++)
                        sum += xs[h * W + w];
                y[out] = sum / (float)(wh.ext * ww.ext);
            }
        }
        __syncthreads();  // the plane's reads are done before the next one lands
    }
}

template <bool MAX>
__global__ __launch_bounds__(256) void pool_bwd_plane_kernel(const float *__restrict__ dy,
                                                             const int *__restrict__ mask,
                                                             float *__restrict__ dx, int H, int W,
                                                             int P, int Q, int R, int S,
                                                             int stride, int pad, FastDiv w_,
                                                             FastDiv st_, uint32_t planes)
{
    extern __shared__ float gs[];  // dy plane, then (max) the mask plane
    int *ms = (int *)(gs + P * Q);
    const uint32_t hw = (uint32_t)H * (uint32_t)W, pq = (uint32_t)P * (uint32_t)Q;
    const uint32_t rows = blockDim.x / (uint32_t)W;
    for (uint32_t nc = blockIdx.x; nc < planes; nc += gridDim.x) {
        for (uint32_t i = threadIdx.x; i < pq; i += blockDim.x) {
            gs[i] = dy[(size_t)nc * pq + i];
            if constexpr (MAX)
                ms[i] = mask[(size_t)nc * pq + i];
        }
        __syncthreads();
        // Thread t keeps column w = t % W of rows t / W, t / W + rows, ...
        // (rows = blockDim.x / W rows at a time, W <= blockDim.x), so the
        // column's window range is decoded once and each row's once per row.
        if (threadIdx.x < rows * (uint32_t)W) {
            const int w = (int)(threadIdx.x - fast_div(threadIdx.x, w_) * w_.d);
            const int wp = w + pad;
            const int q0 = wp < S ? 0 : (int)fast_div((uint32_t)(wp - S), st_) + 1;
            const int q1 = min((int)fast_div((uint32_t)wp, st_), Q - 1);
            for (int h = (int)fast_div(threadIdx.x, w_); h < H; h += (int)rows) {
                const int pix = h * W + w;
                const int hp = h + pad;
                const int p0 = hp < R ? 0 : (int)fast_div((uint32_t)(hp - R), st_) + 1;
                const int p1 = min((int)fast_div((uint32_t)hp, st_), P - 1);
                float acc = 0.f;
                for (int p = p0; p <= p1; p++)
                    for (int q = q0; q <= q1; q++) {
                        const int o = p * Q + q;
                        if constexpr (MAX) {
                            acc += ms[o] == pix ? gs[o] : 0.f;
                        } else {
                            const Win wh = window(p, stride, pad, R, H),
                                      ww = window(q, stride, pad, S, W);
                            acc += gs[o] / (float)(wh.ext * ww.ext);
                        }
                    }
                dx[(size_t)nc * hw + pix] = acc;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// 2 x 2 and 3 x 3 windows at stride 2 (F), the windows that networks use, on
// planes that fit in LDS.  A workgroup takes `per` planes, which lie side by
// side in memory.  Same values in the same order as the kernels above.
//
// What bound the general whole-plane kernels: one four-byte load a wave in
// flight at a time, and loops over windows whose LDS reads each waited for the
// one before.  Here the planes arrive in 16-byte loads that are all requested
// before the first is waited for, and a window's reads are unrolled; backward,
// a thread computes a 2 x 2 block of dx from the one (F = 2) or four windows
// over it.  96 planes of 55 x 55 at batch 128, 3 x 3, max: both passes 146.6 ->
// 109.4 us (kernels 44.0 + 62.4), 4.0 TB/s of the 4.6-4.9 that a copy moves.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
}

// n words of a buffer (rounded up to four: the rest reads zero) into LDS; a
// second buffer beside it where there is one.
template <bool TWO>
__device__ __forceinline__ void stage_words(const void *a, uint32_t *la, const void *b,
                                            uint32_t *lb, uint32_t n)
{
    constexpr int U = TWO ? 2 : 4;  // loads of a thread and buffer in flight
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a, n * 4u), rb = make_rsrc(b, n * 4u);
    const uint32_t nv = (n + 3) / 4;
    for (uint32_t v0 = threadIdx.x; v0 < nv; v0 += U * 256) {
        u32x4 va[U], vb[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            va[u] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(v0 + u * 256) * 16, 0, 0);
            if constexpr (TWO)
                vb[u] = __builtin_amdgcn_raw_buffer_load_b128(rb, (int)(v0 + u * 256) * 16, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (v0 + u * 256 < nv) {
                *(u32x4 *)(la + (v0 + u * 256) * 4) = va[u];
                if constexpr (TWO)
                    *(u32x4 *)(lb + (v0 + u * 256) * 4) = vb[u];
            }
    }
}

// FULL: every window lies inside the image.
template <bool MAX, int F, bool FULL>
__global__ __launch_bounds__(256) void pool_fwd_s2_kernel(const float *__restrict__ x,
                                                          float *__restrict__ y,
                                                          int *__restrict__ mask, int H, int W,
                                                          int pad, FastDiv pq_, FastDiv q_,
                                                          uint32_t planes, uint32_t per)
{
    extern __shared__ __attribute__((aligned(16))) float xs[];
    const uint32_t hw = (uint32_t)H * (uint32_t)W;
    const uint32_t n0 = blockIdx.x * per, n = min(per, planes - n0);
    stage_words<false>(x + (size_t)n0 * hw, (uint32_t *)xs, nullptr, nullptr, n * hw);
    __syncthreads();
    for (uint32_t o = threadIdx.x; o < n * pq_.d; o += 256) {
        const uint32_t j = fast_div(o, pq_), pix = o - j * pq_.d;
        const uint32_t p = fast_div(pix, q_), q = pix - p * q_.d;
        const int h0 = 2 * (int)p - pad, w0 = 2 * (int)q - pad;
        const float *xp = xs + j * hw;
        float v[F][F], best = -__builtin_inff(), sum = 0.f;
        bool ok[F][F];
        int arg = -1;
#pragma unroll
        for (int r = 0; r < F; r++)
#pragma unroll
            for (int s = 0; s < F; s++) {
                ok[r][s] = FULL || ((unsigned)(h0 + r) < (unsigned)H && (unsigned)(w0 + s) < (unsigned)W);
                v[r][s] = xp[ok[r][s] ? (h0 + r) * W + w0 + s : 0];
            }
#pragma unroll
        for (int r = 0; r < F; r++)
#pragma unroll
            for (int s = 0; s < F; s++) {
                if constexpr (MAX) {
                    const bool more = ok[r][s] && v[r][s] > best;
                    best = more ? v[r][s] : best;
                    arg = more ? (h0 + r) * W + w0 + s : arg;
                } else {
                    sum = ok[r][s] ? sum + v[r][s] : sum;
                }
            }
        const size_t out = (size_t)n0 * pq_.d + o;
        if constexpr (MAX) {
            y[out] = best;
            if (mask)
                mask[out] = arg;
        } else {
            const int eh = FULL ? F : min(h0 + F, H + pad) - h0;
            const int ew = FULL ? F : min(w0 + F, W + pad) - w0;
            y[out] = sum / (float)(eh * ew);
        }
    }
}

// Block (a, b) of a plane is padded rows 2 a, 2 a + 1 and columns 2 b, 2 b + 1:
// windows a (and, F = 3, a - 1 for the first row) by b (and b - 1).
template <bool MAX, int F>
__global__ __launch_bounds__(256) void pool_bwd_s2_kernel(const float *__restrict__ dy,
                                                          const int *__restrict__ mask,
                                                          float *__restrict__ dx, int H, int W,
                                                          int P, int Q, int pad, FastDiv ab_,
                                                          FastDiv b_, uint32_t planes, uint32_t per)
{
    extern __shared__ __attribute__((aligned(16))) float gs[];  // dy, then (max) the mask
    const uint32_t hw = (uint32_t)H * (uint32_t)W, pq = (uint32_t)P * (uint32_t)Q;
    const uint32_t n0 = blockIdx.x * per, n = min(per, planes - n0);
    int *const ms = (int *)gs + (per * pq + 3) / 4 * 4;
    stage_words<MAX>(dy + (size_t)n0 * pq, (uint32_t *)gs, MAX ? mask + (size_t)n0 * pq : nullptr,
                     (uint32_t *)ms, n * pq);
    __syncthreads();
    constexpr int L = F - 2;  // windows before a and b
    for (uint32_t i = threadIdx.x; i < n * ab_.d; i += 256) {
        const uint32_t j = fast_div(i, ab_), e = i - j * ab_.d;
        const int a = (int)fast_div(e, b_), b = (int)(e - (uint32_t)a * b_.d);
        float g[L + 1][L + 1];
        int m[L + 1][L + 1];
#pragma unroll
        for (int r = 0; r <= L; r++)
#pragma unroll
            for (int s = 0; s <= L; s++) {
                const int p = a - L + r, q = b - L + s;
                const bool ok = (unsigned)p < (unsigned)P && (unsigned)q < (unsigned)Q;
                const uint32_t o = ok ? j * pq + (uint32_t)(p * Q + q) : 0u;
                g[r][s] = ok ? gs[o] : 0.f;
                if constexpr (MAX) {
                    m[r][s] = ms[o];
                } else {
                    const Win wh = window(p, 2, pad, F, H), ww = window(q, 2, pad, F, W);
                    g[r][s] = ok ? g[r][s] / (float)(wh.ext * ww.ext) : 0.f;
                }
            }
        const int h0 = 2 * a - pad, w0 = 2 * b - pad;
        float d[2][2];
#pragma unroll
        for (int y = 0; y < 2; y++)
#pragma unroll
            for (int x = 0; x < 2; x++) {
                const int pix = (h0 + y) * W + w0 + x;
                float acc = 0.f;
#pragma unroll
                for (int r = y ? L : 0; r <= L; r++)
#pragma unroll
                    for (int s = x ? L : 0; s <= L; s++)
                        acc += !MAX || m[r][s] == pix ? g[r][s] : 0.f;
                d[y][x] = acc;
            }
        float *const o = dx + (size_t)(n0 + j) * hw;
#pragma unroll
        for (int y = 0; y < 2; y++) {
            if ((unsigned)(h0 + y) >= (unsigned)H)
                continue;
            float *const row = o + (h0 + y) * W + w0;
            if (w0 >= 0 && w0 + 1 < W) {
                __builtin_memcpy(row, d[y], 8);
            } else {
                if (w0 >= 0 && w0 < W)
                    row[0] = d[y][0];
                if (w0 + 1 >= 0 && w0 + 1 < W)
                    row[1] = d[y][1];
            }
        }
    }
}

// Planes of at least kPlaneMin elements whose staged data fits in kPlaneLds
// bytes take the whole-plane kernels (smaller planes leave most of a
// workgroup idle: AlexNet's 13 x 13 pool5 ran at half the speed that way).
constexpr size_t kPlaneLds = 48 * 1024;
constexpr long long kPlaneMin = 512;

unsigned pool_grid(uint32_t total)
{
    uint32_t b = (total + 255) / 256;
    return b < 65536u ? b : 65536u;
}

// The stride-2 kernels' windows, on planes that fit, and their planes a
// workgroup: enough for about 1024 elements.  Measured (general / these, us,
// forward and backward): 3 x 3 max on 13 x 13 planes, 256 at batch 128, 12.4 /
// 12.4 and 20.2 / 14.1; 27 x 27 38.4 / 24.5 and 50.0 / 33.8; average with
// padding on 56 x 56, 64 at batch 64, 20.0 / 15.6 and 46.4 / 19.7; 2 x 2 on
// 104 x 104, 128 at batch 32, 116.6 / 47.3 and 72.7 / 59.7; 512 planes of 7 x 7
// at batch 64 12.3 / 11.8 and 9.9 / 9.7.  Not on small planes (below kPlaneMin) of
// fewer than kS2Min elements, which are few workgroups and so wait for the staging
// (3-4 us either way): backward 3.0 / 3.6 on 58 planes of 11 x 11, 3.2 / 4.3 on 812
// of 4 x 4, forward 2-8 % more; a tie or better from kS2Min on.  Forward 3 x 3
// windows all inside the image gain there too (5-19 %).
constexpr long long kS2Min = 1 << 19;
bool s2_applies(int R, int S, int stride, int pad, int H, int W, uint32_t planes, bool inside)
{
    return stride == 2 && R == S && (R == 2 || R == 3) && pad < R &&
           ((long long)H * W >= kPlaneMin || (long long)H * W * planes >= kS2Min ||
            (inside && R == 3));
}
uint32_t s2_planes(int H, int W, uint32_t planes)
{
    const uint32_t per = 1024u / ((uint32_t)H * (uint32_t)W);
    return per < 1u ? 1u : per < planes ? per : planes;
}

}  // namespace

hipError_t launch_pool_fwd(bool max_mode, const float *x, float *y, int *mask, int N, int C, int H,
                           int W, int R, int S, int stride, int pad, int P, int Q,
                           hipStream_t stream)
{
    const uint32_t total = (uint32_t)((long long)N * C * P * Q);
    const uint32_t planes = (uint32_t)((long long)N * C);
    const size_t lds = (size_t)H * W * sizeof(float);
    const bool full = pad == 0 && 2 * (P - 1) + R <= H && 2 * (Q - 1) + R <= W;
    if (s2_applies(R, S, stride, pad, H, W, planes, full) && lds <= kPlaneLds) {
        const uint32_t per = s2_planes(H, W, planes);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((planes + per - 1) / per), dim3(256),
                               (per * lds + 15) / 16 * 16, stream, x, y, max_mode ? mask : nullptr,
                               H, W, pad, make_fastdiv(P * Q), make_fastdiv(Q), planes, per);
            return hipGetLastError();
        };
        if (max_mode)
            return R == 2 ? full ? go(pool_fwd_s2_kernel<true, 2, true>)
                                 : go(pool_fwd_s2_kernel<true, 2, false>)
                          : full ? go(pool_fwd_s2_kernel<true, 3, true>)
                                 : go(pool_fwd_s2_kernel<true, 3, false>);
        return R == 2 ? full ? go(pool_fwd_s2_kernel<false, 2, true>)
                             : go(pool_fwd_s2_kernel<false, 2, false>)
                      : full ? go(pool_fwd_s2_kernel<false, 3, true>)
                             : go(pool_fwd_s2_kernel<false, 3, false>);
    }
    if (lds <= kPlaneLds && (long long)H * W >= kPlaneMin) {
        const dim3 grid(planes < 1048576u ? planes : 1048576u);
        if (max_mode)
            hipLaunchKernelGGL(pool_fwd_plane_kernel<true>, grid, dim3(256), lds, stream, x, y,
                               mask, H, W, R, S, stride, pad, make_fastdiv(Q), (uint32_t)P,
                               planes);
        else
            hipLaunchKernelGGL(pool_fwd_plane_kernel<false>, grid, dim3(256), lds, stream, x, y,
                               nullptr, H, W, R, S, stride, pad, make_fastdiv(Q), (uint32_t)P,
                               planes);
        return hipGetLastError();
    }
    if (max_mode)
        hipLaunchKernelGGL(pool_fwd_kernel<true>, dim3(pool_grid(total)), dim3(256), 0, stream, x,
                           y, mask, H, W, R, S, stride, pad, make_fastdiv(P * Q),
                           make_fastdiv(Q), total);
    else
        hipLaunchKernelGGL(pool_fwd_kernel<false>, dim3(pool_grid(total)), dim3(256), 0, stream,
                           x, y, nullptr, H, W, R, S, stride, pad, make_fastdiv(P * Q),
                           make_fastdiv(Q), total);
    return hipGetLastError();
}

hipError_t launch_pool_bwd(bool max_mode, const float *dy, const int *mask, float *dx, int N,
                           int C, int H, int W, int R, int S, int stride, int pad, int P, int Q,
                           hipStream_t stream)
{
    const uint32_t total = (uint32_t)((long long)N * C * H * W);
    const uint32_t planes = (uint32_t)((long long)N * C);
    const size_t lds = (size_t)P * Q * (max_mode ? 2 : 1) * sizeof(float);
    if (s2_applies(R, S, stride, pad, H, W, planes, false) && lds <= kPlaneLds) {
        const uint32_t per = s2_planes(H, W, planes);
        const int A = (H + pad + 1) / 2, B = (W + pad + 1) / 2;
        const size_t bytes = ((size_t)per * P * Q * sizeof(float) + 15) / 16 * 16;
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((planes + per - 1) / per), dim3(256),
                               max_mode ? 2 * bytes : bytes, stream, dy, max_mode ? mask : nullptr,
                               dx, H, W, P, Q, pad, make_fastdiv(A * B), make_fastdiv(B), planes,
                               per);
            return hipGetLastError();
        };
        if (max_mode)
            return R == 2 ? go(pool_bwd_s2_kernel<true, 2>) : go(pool_bwd_s2_kernel<true, 3>);
        return R == 2 ? go(pool_bwd_s2_kernel<false, 2>) : go(pool_bwd_s2_kernel<false, 3>);
    }
    if (lds <= kPlaneLds && (long long)H * W >= kPlaneMin && W <= 256) {
        const dim3 grid(planes < 1048576u ? planes : 1048576u);
        if (max_mode)
            hipLaunchKernelGGL(pool_bwd_plane_kernel<true>, grid, dim3(256), lds, stream, dy, mask,
                               dx, H, W, P, Q, R, S, stride, pad, make_fastdiv(W),
                               make_fastdiv(stride), planes);
        else
            hipLaunchKernelGGL(pool_bwd_plane_kernel<false>, grid, dim3(256), lds, stream, dy,
                               nullptr, dx, H, W, P, Q, R, S, stride, pad, make_fastdiv(W),
                               make_fastdiv(stride), planes);
        return hipGetLastError();
    }
    if (max_mode)
        hipLaunchKernelGGL(pool_bwd_kernel<true>, dim3(pool_grid(total)), dim3(256), 0, stream,
                           dy, mask, dx, H, W, P, Q, R, S, stride, pad, make_fastdiv(H * W),
                           make_fastdiv(W), make_fastdiv(stride), total);
    else
        hipLaunchKernelGGL(pool_bwd_kernel<false>, dim3(pool_grid(total)), dim3(256), 0, stream,
                           dy, nullptr, dx, H, W, P, Q, R, S, stride, pad, make_fastdiv(H * W),
                           make_fastdiv(W), make_fastdiv(stride), total);
    return hipGetLastError();
}

}  // namespace miconv
