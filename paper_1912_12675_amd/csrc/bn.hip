// Batch norm (+ residual, + ReLU) forward and backward whose statistics no
// convolution formed, and per-channel sums (bias gradients), for gfx950.
//
// All of it is bound by memory: the forward reads y twice (statistics, then
// apply) and writes z, the backward reads dz, z and y twice and writes dy.
// Elements move as float4 (V = 4) where a plane's size and the pointers
// allow, else one by one (V = 1); sums are taken in double, each with one
// owner and a fixed order.
//
// Planes of 64 units and more ("wide"): grid (channel, part); a part is a
// range of images, and the apply kernels merge a channel's parts themselves,
// after their own loads are issued.  Smaller planes ("flat"): neighbouring
// channels share cache lines, so a workgroup takes as many whole channels as
// fit 256 units of one image and walks images; a wave per channel then merges
// the parts, and the apply kernels look its coefficients up.
//
// 128 x 64 x 32 x 32 with an identity residual and ReLU (us, before: one
// float at a time, 64-bit index divisions): statistics 30 -> 7, apply 25 -> 14
// (100 MB), backward sums 30 -> 17, apply 29 -> 24 (168 MB), merges 9 -> none.
#include <algorithm>

#include "internal.h"

namespace psw {
namespace {

constexpr int kBlock = 256;

template <int V>
struct Vec {
    float v[V];
};
template <int V>
__device__ __forceinline__ Vec<V> load_v(const float* p)
{
    Vec<V> r;
    if constexpr (V == 4) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        r.v[0] = t.x, r.v[1] = t.y, r.v[2] = t.z, r.v[3] = t.w;
    } else {
        r.v[0] = *p;
    }
    return r;
}
template <int V>
__device__ __forceinline__ void store_v(float* p, const Vec<V>& r)
{
    if constexpr (V == 4)
        store_stream4(p, make_float4(r.v[0], r.v[1], r.v[2], r.v[3]));
    else
        store_stream(p, r.v[0]);
}

// Two sums over the block at once, fixed order; results valid in thread 0.
__device__ __forceinline__ void block_sum2(double& a, double& b, double* sh)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        sh[2 * wave] = a;
        sh[2 * wave + 1] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int i = 1; i < kBlock / 64; ++i) {
            a += sh[2 * i];
            b += sh[2 * i + 1];
        }
    __syncthreads();
}

// What is summed per element: SUM x; STATS y and y^2; GRAD g and g xhat with
// g = dz [z > 0] (relu) or dz.
enum { SUM, STATS, GRAD };
struct SumArgs {
    const float* x;  // x, y or dz
    const float* z;
    const float* y;
    const float* mean;
    const float* invstd;
    double* part;    // [c][parts][2]
    int n, c, hw, parts, relu;
};

template <int MODE, int V>
struct Sums {
    double s1 = 0.0, s2 = 0.0, mu = 0.0, is = 0.0;
    __device__ __forceinline__ void channel(const SumArgs& a, int ch)
    {
        if (MODE == GRAD) {
            mu = (double)a.mean[ch];
            is = (double)a.invstd[ch];
        }
    }
    __device__ __forceinline__ void add(const Vec<V>& x, const Vec<V>& z, const Vec<V>& y, int relu)
    {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const double v = x.v[e];
            if (MODE == SUM) {
                s1 += v;
            } else if (MODE == STATS) {
                s1 += v;
                s2 += v * v;
            } else {
                const double g = (relu && !(z.v[e] > 0.f)) ? 0.0 : v;
                s1 += g;
                s2 += g * ((double)y.v[e] - mu) * is;
            }
        }
    }
};

// wide planes: block (channel, part), each thread every 256th unit
template <int MODE, int V>
__global__ __launch_bounds__(kBlock) void chan_sums_wide(SumArgs a)
{
    __shared__ double sh[2 * kBlock / 64];
    const int ch = blockIdx.x, upc = a.hw / V;
    const int i0 = (int)((int64_t)a.n * blockIdx.y / a.parts), i1 = (int)((int64_t)a.n * (blockIdx.y + 1) / a.parts);
    Sums<MODE, V> s;
    s.channel(a, ch);
    int img = i0, u = threadIdx.x;
    while (u >= upc) {
        u -= upc;
        ++img;
    }
    constexpr int B = MODE == GRAD ? 2 : 4;  // units in flight
    while (img < i1) {
        Vec<V> x[B], z[B], y[B];
        bool ok[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            ok[b] = img < i1;
            const size_t at = ok[b] ? ((size_t)img * a.c + ch) * a.hw + (size_t)u * V : 0;
            x[b] = load_v<V>(a.x + at);
            if (MODE == GRAD) {
                y[b] = load_v<V>(a.y + at);
                if (a.relu) z[b] = load_v<V>(a.z + at);
            }
            u += kBlock;
            while (u >= upc) {
                u -= upc;
                ++img;
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (ok[b]) s.add(x[b], z[b], y[b], a.relu);
    }
    block_sum2(s.s1, s.s2, sh);
    if (threadIdx.x == 0) {
        double* p = a.part + ((size_t)ch * a.parts + blockIdx.y) * 2;
        p[0] = s.s1;
        p[1] = s.s2;
    }
}

// flat planes: block (group of channels, part), a thread one unit of each of
// its images; a channel's threads meet in LDS in order.  Where the channels
// are fewer than a block's threads hold, the threads take `side` images at a
// time (16 channels of 1x1, 400,000 images: 131 us forward without, 53 now).
template <int MODE, int V>
__global__ __launch_bounds__(kBlock) void chan_sums_flat(SumArgs a, int group, int side)
{
    __shared__ double sh[2][kBlock];
    const int upc = a.hw / V, width = group * upc;  // units of one image in this block
    const int sub = (int)threadIdx.x / width, unit = (int)threadIdx.x - sub * width;
    const int lc = unit / upc, ch = blockIdx.x * group + lc;
    const bool live = sub < side && ch < a.c;
    const int i0 = (int)((int64_t)a.n * blockIdx.y / a.parts), i1 = (int)((int64_t)a.n * (blockIdx.y + 1) / a.parts);
    Sums<MODE, V> s;
    if (live) {
        s.channel(a, ch);
        const size_t at = (size_t)ch * a.hw + (unit - lc * upc) * V, step = (size_t)a.c * a.hw;
        constexpr int B = 4;
        for (int img = i0 + sub; img < i1; img += B * side) {
            Vec<V> x[B], z[B], y[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const size_t o = at + (size_t)min(img + b * side, i1 - 1) * step;
                x[b] = load_v<V>(a.x + o);
                if (MODE == GRAD) {
                    y[b] = load_v<V>(a.y + o);
                    if (a.relu) z[b] = load_v<V>(a.z + o);
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (img + b * side < i1) s.add(x[b], z[b], y[b], a.relu);
        }
    }
    sh[0][threadIdx.x] = s.s1;
    sh[1][threadIdx.x] = s.s2;
    __syncthreads();
    const int t = threadIdx.x;
    for (int left = side; left > 1;) {  // the images side by side, halved in order
        const int keep = (left + 1) / 2;
        if (sub < left - keep) {
            sh[0][t] += sh[0][t + keep * width];
            sh[1][t] += sh[1][t + keep * width];
        }
        __syncthreads();
        left = keep;
    }
    const int mine = (int)blockIdx.x * group + t;  // thread t < group: channel t of the block
    if (t < group && mine < a.c) {
        double s1 = 0.0, s2 = 0.0;
        for (int u = t * upc; u < (t + 1) * upc; ++u) {
            s1 += sh[0][u];
            s2 += sh[1][u];
        }
        double* p = a.part + ((size_t)mine * a.parts + blockIdx.y) * 2;
        p[0] = s1;
        p[1] = s2;
    }
}

// a channel's parts summed by one wave, fixed order; the result in every lane
__device__ __forceinline__ void wave_parts(const double* part, int ch, int parts, double& s1, double& s2)
{
    s1 = s2 = 0.0;
    for (int p = threadIdx.x & 63; p < parts; p += 64) {
        s1 += part[((size_t)ch * parts + p) * 2];
        s2 += part[((size_t)ch * parts + p) * 2 + 1];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_xor(s1, off, 64);
        s2 += __shfl_xor(s2, off, 64);
    }
}

__global__ __launch_bounds__(kBlock) void chan_sum_out(int c, int parts, const double* part, float* out)
{
    const int ch = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (ch >= c) return;
    double s1, s2;
    wave_parts(part, ch, parts, s1, s2);
    if ((threadIdx.x & 63) == 0) out[ch] = (float)s1;
}

struct BnFwdArgs {
    const float* y;
    const float* gamma;
    const float* beta;
    const float* res;
    int rc, rh, rw, relu;
    float eps, momentum;
    float* z;
    float* save_mean;
    float* save_invstd;
    float* run_mean;
    float* run_var;
    float* save_scale;
    const double* part;
    int n, c, h, w, parts;
    float* coef;        // flat: [c][2] scale, shift
    int img0, imgs;     // wide: the images of this launch
};

// a channel's coefficients from its sums; store: also the saved and running statistics
__device__ __forceinline__ void bn_fwd_coef(const BnFwdArgs& a, int ch, double s1, double s2, bool store, float& scale,
                                            float& shift)
{
    const double count = (double)a.n * a.h * a.w;
    const double mean = s1 / count;
    double var = s2 / count - mean * mean;
    if (var < 0.0) var = 0.0;
    const double invstd = 1.0 / sqrt(var + (double)a.eps);
    const double sc = (double)a.gamma[ch] * invstd;
    scale = (float)sc;
    shift = (float)((double)a.beta[ch] - mean * sc);
    if (!store) return;
    a.save_mean[ch] = (float)mean;
    a.save_invstd[ch] = (float)invstd;
    if (a.run_mean) a.run_mean[ch] = (float)((1.0 - a.momentum) * a.run_mean[ch] + a.momentum * mean);
    if (a.run_var)
        a.run_var[ch] = (float)((1.0 - a.momentum) * a.run_var[ch] +
                                a.momentum * (count > 1.0 ? var * count / (count - 1.0) : var));
    if (a.save_scale) {
        a.save_scale[ch] = scale;
        a.save_scale[a.c + ch] = shift;
    }
}

__global__ __launch_bounds__(kBlock) void bn_fwd_merge(BnFwdArgs a)
{
    const int ch = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (ch >= a.c) return;
    double s1, s2;
    wave_parts(a.part, ch, a.parts, s1, s2);
    if ((threadIdx.x & 63) == 0) bn_fwd_coef(a, ch, s1, s2, true, a.coef[2 * ch], a.coef[2 * ch + 1]);
}

// the residual of V elements of channel ch from in-plane offset off
template <int V>
__device__ __forceinline__ Vec<V> residual(const BnFwdArgs& a, int img, int ch, int off, bool identity)
{
    Vec<V> r;
    if (identity) return load_v<V>(a.res + ((size_t)img * a.c + ch) * (a.h * a.w) + off);
    // option A: subsampled, zero-padded channels
    const int cc = ch - (a.c - a.rc) / 2, fh = a.rh / a.h, fw = a.rw / a.w;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int hh = (off + e) / a.w, ww = off + e - hh * a.w;
        r.v[e] = cc >= 0 && cc < a.rc ? a.res[(((size_t)img * a.rc + cc) * a.rh + hh * fh) * a.rw + ww * fw] : 0.f;
    }
    return r;
}

template <int V>
__device__ __forceinline__ Vec<V> bn_fwd_one(const BnFwdArgs& a, const Vec<V>& y, const Vec<V>& r, float sc, float sf)
{
    Vec<V> o;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        float v = __fmaf_rn(y.v[e], sc, sf);
        if (a.res) v += r.v[e];
        o.v[e] = a.relu ? fmaxf(v, 0.f) : v;
    }
    return o;
}

// wide: block (channel, U * 256 units of it), channels first; both on the x
// dimension of the grid, since the others end at 65,535
template <int V, int U>
__global__ __launch_bounds__(kBlock) void bn_fwd_apply_wide(BnFwdArgs a)
{
    __shared__ double sh[2 * kBlock / 64];
    __shared__ float coef[2];
    const int ch = blockIdx.x % a.c, blk = blockIdx.x / a.c, hw = a.h * a.w, upc = hw / V, units = a.imgs * upc;
    const bool identity = a.res && a.rc == a.c && a.rh == a.h && a.rw == a.w;
    size_t at[U];
    Vec<V> y[U], r[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int u = min((blk * U + q) * kBlock + (int)threadIdx.x, units - 1);
        const int img = u / upc, off = (u - img * upc) * V;
        at[q] = ((size_t)(a.img0 + img) * a.c + ch) * hw + off;
        y[q] = load_v<V>(a.y + at[q]);
        if (a.res) r[q] = residual<V>(a, a.img0 + img, ch, off, identity);
    }
    double s1 = 0.0, s2 = 0.0;
    for (int p = threadIdx.x; p < a.parts; p += kBlock) {
        s1 += a.part[((size_t)ch * a.parts + p) * 2];
        s2 += a.part[((size_t)ch * a.parts + p) * 2 + 1];
    }
    block_sum2(s1, s2, sh);
    if (threadIdx.x == 0) bn_fwd_coef(a, ch, s1, s2, blk == 0 && a.img0 == 0, coef[0], coef[1]);
    __syncthreads();
    const float sc = coef[0], sf = coef[1];
#pragma unroll
    for (int q = 0; q < U; ++q)
        if ((blk * U + q) * kBlock + (int)threadIdx.x < units)
            store_v<V>(a.z + at[q], bn_fwd_one<V>(a, y[q], r[q], sc, sf));
}

// flat: a thread one unit of an image, for `per` images; `side` images at a
// time where an image has fewer units than a block threads.  Blocks over an
// image first, over images next, on the x dimension of the grid.
struct FlatAt {
    int u, img, end, step;
    __device__ __forceinline__ FlatAt(int ups, int n, int bx, int side, int per)
    {
        const int xb = (int)(blockIdx.x % bx), yb = (int)(blockIdx.x / bx);
        const int sub = side > 1 ? (int)threadIdx.x / ups : 0;
        u = xb * kBlock + (int)threadIdx.x - sub * ups;
        img = yb * per * side + sub;
        end = u < ups && sub < side ? min((yb + 1) * per * side, n) : 0;
        step = side;
    }
};

template <int V>
__global__ __launch_bounds__(kBlock) void bn_fwd_apply_flat(BnFwdArgs a, int bx, int side, int per)
{
    const int hw = a.h * a.w, ups = a.c * (hw / V);
    const FlatAt f(ups, a.n, bx, side, per);
    if (f.img >= f.end) return;
    const int ch = f.u / (hw / V), off = (f.u - ch * (hw / V)) * V;
    const bool identity = a.res && a.rc == a.c && a.rh == a.h && a.rw == a.w;
    const float sc = a.coef[2 * ch], sf = a.coef[2 * ch + 1];
    for (int img = f.img; img < f.end; img += f.step) {
        const size_t at = (size_t)img * ((size_t)a.c * hw) + (size_t)f.u * V;
        const Vec<V> y = load_v<V>(a.y + at);
        Vec<V> r = y;
        if (a.res) r = residual<V>(a, img, ch, off, identity);
        store_v<V>(a.z + at, bn_fwd_one<V>(a, y, r, sc, sf));
    }
}

struct BnBwdArgs {
    const float* dz;
    const float* z;
    const float* y;
    const float* gamma;
    const float* mean;
    const float* invstd;
    int relu;
    float* dy;
    float* dgamma;
    float* dbeta;
    float* dres;  // identity residual only
    int res_accumulate;
    const double* part;
    int n, c, hw, parts;
    float* coef;     // flat: [c][3]
    int img0, imgs;  // wide: the images of this launch
};

__device__ __forceinline__ void bn_bwd_coef(const BnBwdArgs& a, int ch, double s1, double s2, bool store, float* k)
{
    const double count = (double)a.n * a.hw;
    k[0] = (float)((double)a.gamma[ch] * (double)a.invstd[ch]);
    k[1] = (float)(s1 / count);
    k[2] = (float)(s2 / count);
    if (store) {
        a.dbeta[ch] = (float)s1;
        a.dgamma[ch] = (float)s2;
    }
}

__global__ __launch_bounds__(kBlock) void bn_bwd_merge(BnBwdArgs a)
{
    const int ch = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (ch >= a.c) return;
    double s1, s2;
    wave_parts(a.part, ch, a.parts, s1, s2);
    if ((threadIdx.x & 63) == 0) bn_bwd_coef(a, ch, s1, s2, true, a.coef + 3 * ch);
}

template <int V>
struct BwdIn {
    Vec<V> g, z, y, old;
    __device__ __forceinline__ void load(const BnBwdArgs& a, size_t at)
    {
        g = load_v<V>(a.dz + at);
        y = load_v<V>(a.y + at);
        if (a.relu) z = load_v<V>(a.z + at);
        if (a.dres && a.res_accumulate) old = load_v<V>(a.dres + at);
    }
    __device__ __forceinline__ void finish(const BnBwdArgs& a, size_t at, float mu, float is, float k0, float k1, float k2)
    {
        Vec<V> o, d;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float gm = (a.relu && !(z.v[e] > 0.f)) ? 0.f : g.v[e];
            const float xh = (y.v[e] - mu) * is;
            o.v[e] = k0 * (gm - k1 - xh * k2);
            d.v[e] = a.res_accumulate ? old.v[e] + gm : gm;
        }
        store_v<V>(a.dy + at, o);
        if (a.dres) store_v<V>(a.dres + at, d);
    }
};

template <int V, int U>
__global__ __launch_bounds__(kBlock) void bn_bwd_apply_wide(BnBwdArgs a)
{
    __shared__ double sh[2 * kBlock / 64];
    __shared__ float coef[3];
    const int ch = blockIdx.x % a.c, blk = blockIdx.x / a.c, upc = a.hw / V, units = a.imgs * upc;
    size_t at[U];
    BwdIn<V> in[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int u = min((blk * U + q) * kBlock + (int)threadIdx.x, units - 1);
        const int img = u / upc;
        at[q] = ((size_t)(a.img0 + img) * a.c + ch) * a.hw + (size_t)(u - img * upc) * V;
        in[q].load(a, at[q]);
    }
    double s1 = 0.0, s2 = 0.0;
    for (int p = threadIdx.x; p < a.parts; p += kBlock) {
        s1 += a.part[((size_t)ch * a.parts + p) * 2];
        s2 += a.part[((size_t)ch * a.parts + p) * 2 + 1];
    }
    block_sum2(s1, s2, sh);
    const float mu = a.mean[ch], is = a.invstd[ch];
    if (threadIdx.x == 0) bn_bwd_coef(a, ch, s1, s2, blk == 0 && a.img0 == 0, coef);
    __syncthreads();
    const float k0 = coef[0], k1 = coef[1], k2 = coef[2];
#pragma unroll
    for (int q = 0; q < U; ++q)
        if ((blk * U + q) * kBlock + (int)threadIdx.x < units) in[q].finish(a, at[q], mu, is, k0, k1, k2);
}

template <int V>
__global__ __launch_bounds__(kBlock) void bn_bwd_apply_flat(BnBwdArgs a, int bx, int side, int per)
{
    const int ups = a.c * (a.hw / V);
    const FlatAt f(ups, a.n, bx, side, per);
    if (f.img >= f.end) return;
    const int ch = f.u / (a.hw / V);
    const float mu = a.mean[ch], is = a.invstd[ch];
    const float k0 = a.coef[3 * ch], k1 = a.coef[3 * ch + 1], k2 = a.coef[3 * ch + 2];
    for (int img = f.img; img < f.end; img += f.step) {
        const size_t at = (size_t)img * ((size_t)a.c * a.hw) + (size_t)f.u * V;
        BwdIn<V> in;
        in.load(a, at);
        in.finish(a, at, mu, is, k0, k1, k2);
    }
}

// option-A shortcut backward: dres[n][cr][hr][wr] gets g[n][cr+lo][hr/sh][wr/sw]
// at subsampled positions and zero elsewhere; V consecutive columns a thread
template <int V>
__global__ __launch_bounds__(kBlock) void shortcut_a_bwd(int units, int c, int h, int w, int rc, int rh, int rw,
                                                         const float* dz, const float* z, int relu, float* dres,
                                                         int accumulate)
{
    const int i = (int)blockIdx.x * kBlock + (int)threadIdx.x;
    if (i >= units) return;
    const int upr = rw / V;
    const int row = i / upr, w0 = (i - row * upr) * V;  // row of [n][rc][rh]
    const int ncr = row / rh, hr = row - ncr * rh;
    const int img = ncr / rc, cr = ncr - img * rc;
    const int sh = rh / h, sw = rw / w;
    Vec<V> g;
    const bool on = hr % sh == 0;
    const size_t j = (((size_t)img * c + cr + (c - rc) / 2) * h + hr / sh) * w;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int wr = w0 + e;
        float v = 0.f;
        if (on && wr % sw == 0) {
            v = dz[j + wr / sw];
            if (relu && !(z[j + wr / sw] > 0.f)) v = 0.f;
        }
        g.v[e] = v;
    }
    float* o = dres + (size_t)row * rw + w0;
    if (accumulate) {
        const Vec<V> old = load_v<V>(o);
#pragma unroll
        for (int e = 0; e < V; ++e) g.v[e] = old.v[e] + g.v[e];
    }
    store_v<V>(o, g);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// parts per channel of the wide kernels, and of every channel_sum
int channel_splits(int n, int c)
{
    int sp = (1024 + c - 1) / c;
    if (sp > n) sp = n;
    if (sp < 1) sp = 1;
    return sp;
}

bool is_flat(int hw, int v) { return hw / v < 64; }

int flat_group(int c, int upc) { return std::min(kBlock / upc, c); }  // whole channels of a block

// parts of the flat kernels: about 512 workgroups, at least four images each
int flat_parts(int n, int c, int hw, int v)
{
    const int group = flat_group(c, hw / v), blocks = (c + group - 1) / group;
    int p = (512 + blocks - 1) / blocks;
    if (p > (n + 3) / 4) p = (n + 3) / 4;
    if (p < 1) p = 1;
    return p;
}

int bn_parts(int n, int c, int hw, int v) { return is_flat(hw, v) ? flat_parts(n, c, hw, v) : channel_splits(n, c); }

template <int MODE>
void launch_sums(const SumArgs& a, int v, const Work& wk, hipStream_t st)
{
    if (is_flat(a.hw, v)) {
        // Fewer channels a block, and images side by side in their place, while
        // a part's images are more than a thread should take in turn and the
        // workgroups too few (a bias of 512 channels of 2x2 has the workspace for
        // two parts: 14.8 us with 256 channels a block).
        const int upc = a.hw / v, images = (a.n + a.parts - 1) / a.parts;
        int group = flat_group(a.c, upc);
        auto side_of = [&](int g) { return std::min(kBlock / (g * upc), images); };
        while (group * upc > 32 && images > 4 * side_of(group) && (int64_t)(a.c + group - 1) / group * a.parts < 256)
            group = (group + 1) / 2;
        const int side = side_of(group);
        const dim3 grid((unsigned)((a.c + group - 1) / group), (unsigned)a.parts);
        if (v == 4)
            PSW_LAUNCH(kname("chan_sums_flat", MODE, 4), wk, (chan_sums_flat<MODE, 4>), grid, dim3(kBlock), 0, st, a, group,
                       side);
        else
            PSW_LAUNCH(kname("chan_sums_flat", MODE, 1), wk, (chan_sums_flat<MODE, 1>), grid, dim3(kBlock), 0, st, a, group,
                       side);
    } else {
        const dim3 grid((unsigned)a.c, (unsigned)a.parts);
        if (v == 4)
            PSW_LAUNCH(kname("chan_sums_wide", MODE, 4), wk, (chan_sums_wide<MODE, 4>), grid, dim3(kBlock), 0, st, a);
        else
            PSW_LAUNCH(kname("chan_sums_wide", MODE, 1), wk, (chan_sums_wide<MODE, 1>), grid, dim3(kBlock), 0, st, a);
    }
}

// units per thread of the wide apply kernels: the largest of 4, 2, 1 that
// still gives 1024 workgroups (four per CU)
int wide_units(int64_t units_total)
{
    for (int u = 4; u > 1; u /= 2)
        if (units_total / ((int64_t)u * kBlock) >= 1024) return u;
    return 1;
}

// images of one launch: units of an image counted in 32 bits, `threads` in all
// for an image (a grid ends at 2^32)
int slice_images(int n, int64_t units_per_image, int64_t threads)
{
    const int64_t most = std::min((INT32_MAX - 8 * kBlock) / units_per_image, (int64_t)INT32_MAX / threads);
    return (int)std::max<int64_t>(1, std::min<int64_t>(n, most));
}

// the flat apply kernels' launch: blocks over an image, images side by side
// and one after another, and the blocks in all
struct FlatGrid {
    int bx, side, per;
    int64_t blocks;
    FlatGrid(int n, int64_t ups)
    {
        bx = (int)((ups + kBlock - 1) / kBlock);
        side = ups < kBlock ? kBlock / (int)ups : 1;
        const int rows = (n + side - 1) / side;  // groups of images
        per = 1;
        while (per < 8 && per * 2 <= rows && (int64_t)bx * (rows / (per * 2)) >= 1024) per *= 2;
        blocks = (int64_t)bx * ((rows + per - 1) / per);
    }
};

}  // namespace

size_t channel_sum_ws_bytes(int n, int c, int hw)
{
    (void)hw;
    return (size_t)c * channel_splits(n, c) * 2 * sizeof(double);
}

hipError_t channel_sum(int n, int c, int hw, const float* x, float* out, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (ws_bytes < channel_sum_ws_bytes(n, c, hw)) return hipErrorInvalidValue;
    const int v = hw % 4 == 0 && aligned16(x) ? 4 : 1;
    SumArgs a{};
    a.x = x;
    a.part = (double*)ws;
    a.n = n; a.c = c; a.hw = hw;
    a.parts = std::min(bn_parts(n, c, hw, v), channel_splits(n, c));
    const double elems = (double)n * c * hw;
    launch_sums<SUM>(a, v, Work{elems, kF * elems}, st);
    PSW_LAUNCH(kname("chan_sum_out"), (Work{(double)c * a.parts, 16.0 * c * a.parts + kF * c}), chan_sum_out,
               dim3((unsigned)((c + 3) / 4)), dim3(kBlock), 0, st, c, a.parts, (const double*)ws, out);
    return hipGetLastError();
}

size_t bn_ws_bytes(int n, int c, int h, int w)
{
    // the sums' parts for either width of unit, the flat kernels' coefficients
    int p = channel_splits(n, c);
    for (int v : {1, 4})
        if (h * w % v == 0) p = std::max(p, bn_parts(n, c, h * w, v));
    return (size_t)c * p * 2 * sizeof(double) + (size_t)c * 3 * sizeof(float) + 256;
}

hipError_t bn_fwd(int n, int c, int h, int w, const float* y, const float* gamma, const float* beta, const float* res,
                  int rc, int rh, int rw, int relu, float eps, float momentum, float* z, float* save_mean,
                  float* save_invstd, float* run_mean, float* run_var, void* ws, size_t ws_bytes, hipStream_t st,
                  float* save_scale)
{
    if (ws_bytes < bn_ws_bytes(n, c, h, w)) return hipErrorInvalidValue;
    const int hw = h * w;
    const bool identity = res && rc == c && rh == h && rw == w;
    const int v = hw % 4 == 0 && aligned16(y) && aligned16(z) && (!identity || aligned16(res)) ? 4 : 1;
    const double total = (double)n * c * hw;
    SumArgs s{};
    s.x = y;
    s.part = (double*)ws;
    s.n = n; s.c = c; s.hw = hw;
    s.parts = bn_parts(n, c, hw, v);
    launch_sums<STATS>(s, v, Work{3.0 * total, kF * total}, st);
    BnFwdArgs a{y, gamma, beta, res, rc, rh, rw, relu, eps, momentum, z, save_mean, save_invstd, run_mean, run_var,
                save_scale, s.part, n, c, h, w, s.parts, (float*)(s.part + (size_t)c * s.parts * 2), 0, n};
    const double rbytes = res ? kF * (double)n * std::min(c, rc) * hw : 0.0;
    const Work wk{3.0 * total, kF * 2.0 * total + rbytes + 16.0 * c * s.parts};
    if (is_flat(hw, v)) {
        PSW_LAUNCH(kname("bn_fwd_merge"), (Work{2.0 * c * s.parts, 16.0 * c * s.parts + 6 * kF * c}), bn_fwd_merge,
                   dim3((unsigned)((c + 3) / 4)), dim3(kBlock), 0, st, a);
        const FlatGrid f(n, (int64_t)c * (hw / v));
        const dim3 grid((unsigned)f.blocks);
        if (v == 4)
            PSW_LAUNCH(kname("bn_fwd_apply_flat", 4), wk, bn_fwd_apply_flat<4>, grid, dim3(kBlock), 0, st, a, f.bx, f.side,
                       f.per);
        else
            PSW_LAUNCH(kname("bn_fwd_apply_flat", 1), wk, bn_fwd_apply_flat<1>, grid, dim3(kBlock), 0, st, a, f.bx, f.side,
                       f.per);
        return hipGetLastError();
    }
    const int U = wide_units((int64_t)n * (hw / v) * c);
    for (int i0 = 0, step = slice_images(n, hw / v, (int64_t)c * (hw / v)); i0 < n; i0 += step) {
        a.img0 = i0;
        a.imgs = std::min(step, n - i0);
        const dim3 grid((unsigned)(c * (((int64_t)a.imgs * (hw / v) + U * kBlock - 1) / (U * kBlock))));
#define PSW_BN(V_, U_) \
    PSW_LAUNCH(kname("bn_fwd_apply_wide", V_, U_), wk, (bn_fwd_apply_wide<V_, U_>), grid, dim3(kBlock), 0, st, a)
        if (v == 4 && U == 4) PSW_BN(4, 4);
        else if (v == 4 && U == 2) PSW_BN(4, 2);
        else if (v == 4) PSW_BN(4, 1);
        else if (U == 4) PSW_BN(1, 4);
        else if (U == 2) PSW_BN(1, 2);
        else PSW_BN(1, 1);
#undef PSW_BN
    }
    return hipGetLastError();
}

hipError_t bn_bwd(int n, int c, int h, int w, const float* dz, const float* z, const float* y, const float* gamma,
                  const float* save_mean, const float* save_invstd, int relu, float* dy, float* dgamma,
                  float* dbeta, float* dres, int rc, int rh, int rw, int res_accumulate, void* ws, size_t ws_bytes,
                  hipStream_t st)
{
    if (ws_bytes < bn_ws_bytes(n, c, h, w)) return hipErrorInvalidValue;
    const int hw = h * w;
    const bool identity = dres && rc == c && rh == h && rw == w;
    const int v = hw % 4 == 0 && aligned16(dz) && aligned16(z) && aligned16(y) && aligned16(dy) &&
                          (!identity || aligned16(dres)) ? 4 : 1;
    const double total = (double)n * c * hw;
    SumArgs s{dz, z, y, save_mean, save_invstd, (double*)ws, n, c, hw, bn_parts(n, c, hw, v), relu};
    launch_sums<GRAD>(s, v, Work{5.0 * total, (relu ? 3 : 2) * kF * total}, st);
    BnBwdArgs a{dz, z, y, gamma, save_mean, save_invstd, relu, dy, dgamma, dbeta, identity ? dres : nullptr,
                res_accumulate, s.part, n, c, hw, s.parts, (float*)(s.part + (size_t)c * s.parts * 2), 0, n};
    const Work wk{6.0 * total, kF * ((relu ? 4.0 : 3.0) + (identity ? 1.0 + res_accumulate : 0.0)) * total};
    if (is_flat(hw, v)) {
        PSW_LAUNCH(kname("bn_bwd_merge"), (Work{2.0 * c * s.parts, 16.0 * c * s.parts + 7 * kF * c}), bn_bwd_merge,
                   dim3((unsigned)((c + 3) / 4)), dim3(kBlock), 0, st, a);
        const FlatGrid f(n, (int64_t)c * (hw / v));
        const dim3 grid((unsigned)f.blocks);
        if (v == 4)
            PSW_LAUNCH(kname("bn_bwd_apply_flat", 4), wk, bn_bwd_apply_flat<4>, grid, dim3(kBlock), 0, st, a, f.bx, f.side,
                       f.per);
        else
            PSW_LAUNCH(kname("bn_bwd_apply_flat", 1), wk, bn_bwd_apply_flat<1>, grid, dim3(kBlock), 0, st, a, f.bx, f.side,
                       f.per);
    } else {
        const int U = std::min(wide_units((int64_t)n * (hw / v) * c), 2);  // four tensors per unit in registers
        for (int i0 = 0, step = slice_images(n, hw / v, (int64_t)c * (hw / v)); i0 < n; i0 += step) {
            a.img0 = i0;
            a.imgs = std::min(step, n - i0);
            const dim3 grid((unsigned)(c * (((int64_t)a.imgs * (hw / v) + U * kBlock - 1) / (U * kBlock))));
#define PSW_BN(V_, U_) \
    PSW_LAUNCH(kname("bn_bwd_apply_wide", V_, U_), wk, (bn_bwd_apply_wide<V_, U_>), grid, dim3(kBlock), 0, st, a)
            if (v == 4 && U == 2) PSW_BN(4, 2);
            else if (v == 4) PSW_BN(4, 1);
            else if (U == 2) PSW_BN(1, 2);
            else PSW_BN(1, 1);
#undef PSW_BN
        }
    }
    if (dres && !identity) {
        const int vr = rw % 4 == 0 && aligned16(dres) ? 4 : 1;
        const int64_t upi = (int64_t)rc * rh * (rw / vr);  // units of an image
        for (int i0 = 0, step = slice_images(n, upi, upi); i0 < n; i0 += step) {
            const int64_t units = std::min(step, n - i0) * upi;
            const Work ws2{0.0, kF * ((1.0 + res_accumulate) * units * vr + (relu ? 2.0 : 1.0) * n * rc * hw)};
            const dim3 grid((unsigned)((units + kBlock - 1) / kBlock));
            const size_t so = (size_t)i0 * c * hw, ro = (size_t)i0 * upi * vr;
            if (vr == 4)
                PSW_LAUNCH(kname("shortcut_a_bwd", 4), ws2, shortcut_a_bwd<4>, grid, dim3(kBlock), 0, st, (int)units, c, h,
                           w, rc, rh, rw, dz + so, z + so, relu, dres + ro, res_accumulate);
            else
                PSW_LAUNCH(kname("shortcut_a_bwd", 1), ws2, shortcut_a_bwd<1>, grid, dim3(kBlock), 0, st, (int)units, c, h,
                           w, rc, rh, rw, dz + so, z + so, relu, dres + ro, res_accumulate);
        }
    }
    return hipGetLastError();
}

}  // namespace psw
