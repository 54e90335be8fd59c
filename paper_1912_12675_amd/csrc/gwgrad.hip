// Backward-weight of a convolution for the shapes without a kernel of their
// own, on the bf16 matrix cores: fp32 operands as three bfloat16 parts
// (split.h), or rounded once in bf16 mode.  Kernels of 1, 3 or 5 columns; other
// widths stay on the implicit GEMM (conv.hip).
//
//   dW[k][c][r][s] = sum_{img,p,q} dy[img][k][p][q] x[img][c][p st + r - pad][q st + s - pad]
//
// The reduction runs over images and output pixels.  Eight images at one
// pixel are a 16-byte unit of eight bfloat16, so a tap, which moves the pixel
// of x, moves whole units: every operand read is an aligned 16 bytes, and a
// value is loaded and split once for all taps.  (Eight pixels of a row as a
// unit would need a copy of x per column of the kernel.)
//
// A workgroup owns BM output channels and CT blocks of 16 input channels at
// RG rows of S taps, and walks its share of the chunks: a chunk is PX units of
// dy (TO image octets x TH rows x TW columns, powers of two chosen on the
// host) and the pixels of x they meet.  The next chunk is loaded into
// registers while the matrix cores work on this one.  A matrix step takes
// four units (lane group g the g-th); the WK waves that share an output
// block take the steps in turn and meet in LDS in wave order.  Each workgroup
// writes one dW-shaped partial sum (its part); reduce_splits adds the parts
// in a fixed order.
//
// Measured with the reduction, batch 128, against the implicit GEMM (fp32):
// 3x3 64 -> 64 at 32x32 336 -> 77 us, 256 -> 256 at 8x8 299 -> 64 us (151
// TFLOP/s), 512 -> 512 at 4x4 364 -> 62 us, 5x5 64 -> 192 at 16x16 597 -> 138
// us; bf16 mode 464 -> 56, 395 -> 39, 425 -> 37, 767 -> 78 us.
#include "internal.h"
#include "split.h"

namespace psw {
namespace {

struct GwArgs {
    const float* x;   // [n][C][H][W]
    const float* dy;  // [n][K][P][Q]
    float* part;      // [z][K][C][R][S]
    int n, C, H, W, K, P, Q, R, S, st, pad;
    int lw, lh;       // log2 of the chunk's columns and rows
    int tiles_h, tiles_w, chunks;
    int z, per;       // parts, chunks per part
    int kblocks, cblocks, rblocks;
    int by_xcd;       // parts are dealt to the XCDs in turn
};

template <int NS, int BM, int WM, int CT, int RG, int S, int PX>
__global__ __launch_bounds__(256, 2) void conv_split_wgrad(GwArgs a)
{
    constexpr int NT = 256, WK = 4 / WM, MT = BM / WM / 16;
    constexpr int TAPS = CT * RG * S;
    // bf16 rows of five taps: few parts and long sums, so the steps of a chunk
    // take two sums in turn
    constexpr bool TWO = NS == 1 && S == 5 && PX / 4 / WK >= 2;
    constexpr int DI = BM * PX, DV = DI / NT;  // units of dy, per thread
    constexpr int XV = 3;                       // units of x per thread and staging pass
    static_assert(DI % NT == 0, "units");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int combos = a.kblocks * a.cblocks * a.rblocks;
    int zi, combo;
    if (a.by_xcd) {  // the blocks of one part read the same tiles: one XCD, one after another
        const int slot = (int)(blockIdx.x >> 3);
        combo = slot % combos;
        zi = slot / combos * 8 + (int)(blockIdx.x & 7);
    } else {
        combo = (int)blockIdx.x % combos;
        zi = (int)blockIdx.x / combos;
    }
    if (zi >= a.z) return;
    const int k0 = combo % a.kblocks * BM;
    const int c0 = combo / a.kblocks % a.cblocks * (16 * CT);
    const int r0 = combo / (a.kblocks * a.cblocks) * RG;
    const int ch_begin = zi * a.per, ch_end = min(ch_begin + a.per, a.chunks);

    const int TW = 1 << a.lw, TH = 1 << a.lh, TO = PX >> (a.lw + a.lh);
    const int HC = (TW - 1) * a.st + S, HR = (TH - 1) * a.st + RG;
    const int XP = TO * HR * HC, XROW = XP | 1;  // units of one channel of x; odd row
    const int XI = 16 * CT * XP;
    sp_v8b* const Ds = reinterpret_cast<sp_v8b*>(smem);  // [NS][BM][PX], unit u of row m at u ^ (m % PX)
    sp_v8b* const Xs = Ds + NS * DI;                     // [NS][16 CT][XROW]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wk = wave / WM;
    const int g = lane >> 4, j = lane & 15;
    const int PQ = a.P * a.Q, HW = a.H * a.W;

    // chunk -> first octet, first output row and column
    auto chunk_at = [&](int ch, int* oct, int* p0, int* q0) {
        *q0 = ch % a.tiles_w * TW;
        *p0 = ch / a.tiles_w % a.tiles_h * TH;
        *oct = ch / (a.tiles_w * a.tiles_h) * TO;
    };
    const Buffer dyb = make_buffer(a.dy, (int64_t)a.n * a.K * PQ * 4);
    const Buffer xb = make_buffer(a.x, (int64_t)a.n * a.C * HW * 4);

    float dr[DV][8], xr[XV][8];
    // Eight images of one element: `src` its byte offset in the first of them,
    // or kOutside.  Images past the last lie past the buffer's end and read as
    // zero; so that the hardware's check covers them, the whole offset is the
    // lane's then (four to eleven images, a comparison and a choice a load as it
    // was, now: 1x1 4 -> 40 at 20x17 19.8 us, 16.7; 128 -> 64 at 28x28 stride 2 28.1,
    // 23.2; 3x3 16 -> 16 at 14x14 stride 2 13.5, 11.8).
    auto load_unit = [&](const Buffer& b, int src, int stride, bool whole, float(&r)[8]) {
        if (whole) {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = buffer_load(b, src, e * stride);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = buffer_load(b, (int)((unsigned)src + (unsigned)(e * stride)), 0);
        }
    };
    auto load_x = [&](int idx, int oct, int p0, int q0, bool whole, float(&r)[8]) {
        const int c = idx / XP, u = idx - c * XP;
        const int o = u / (HR * HC), rem = u - o * (HR * HC);
        const int hr = rem / HC, hc = rem - hr * HC;
        const int ih = p0 * a.st + r0 - a.pad + hr, iw = q0 * a.st - a.pad + hc, img = (oct + o) * 8;
        const bool in = idx < XI && c0 + c < a.C && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W && img < a.n;
        load_unit(xb, in ? (((img * a.C + c0 + c) * a.H + ih) * a.W + iw) * 4 : kOutside, a.C * HW * 4, whole, r);
    };
    auto load_chunk = [&](int ch) {
        int oct, p0, q0;
        chunk_at(ch, &oct, &p0, &q0);
        const bool whole = (oct + TO) * 8 <= a.n;
#pragma unroll
        for (int v = 0; v < DV; ++v) {
            const int idx = tid + v * NT, m = idx / PX, u = idx % PX;
            const int q = q0 + (u & (TW - 1)), p = p0 + ((u >> a.lw) & (TH - 1)), img = (oct + (u >> (a.lw + a.lh))) * 8;
            const bool in = k0 + m < a.K && p < a.P && q < a.Q && img < a.n;
            load_unit(dyb, in ? ((img * a.K + k0 + m) * PQ + p * a.Q + q) * 4 : kOutside, a.K * PQ * 4, whole, dr[v]);
        }
#pragma unroll
        for (int v = 0; v < XV; ++v)
            if (v * NT < XI) load_x(tid + v * NT, oct, p0, q0, whole, xr[v]);
    };
    auto put = [&](sp_v8b* dst, int stride, const float(&r)[8]) {
        sp_v8b parts[NS];
        split8<NS>(r, parts);
#pragma unroll
        for (int s = 0; s < NS; ++s) dst[s * stride] = parts[s];
    };
    auto store_chunk = [&](int ch) {
#pragma unroll
        for (int v = 0; v < DV; ++v) {
            const int idx = tid + v * NT, m = idx / PX, u = idx % PX;
            put(Ds + m * PX + (u ^ (m & (PX - 1))), DI, dr[v]);
        }
#pragma unroll
        for (int v = 0; v < XV; ++v) {
            const int idx = tid + v * NT, c = idx / XP;
            if (idx < XI) put(Xs + c * XROW + idx - c * XP, 16 * CT * XROW, xr[v]);
        }
        if (XV * NT < XI) {  // more units than the registers hold
            int oct, p0, q0;
            chunk_at(ch, &oct, &p0, &q0);
            for (int idx = tid + XV * NT; idx < XI; idx += NT) {
                const int c = idx / XP;
                float r[8];
                load_x(idx, oct, p0, q0, (oct + TO) * 8 <= a.n, r);
                put(Xs + c * XROW + idx - c * XP, 16 * CT * XROW, r);
            }
        }
    };

    sp_v4f acc[MT][TAPS];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < TAPS; ++t) acc[mt][t] = sp_v4f{0.f, 0.f, 0.f, 0.f};

    sp_v4f odd[TWO ? MT : 1][TWO ? TAPS : 1];
#pragma unroll
    for (int mt = 0; mt < (TWO ? MT : 1); ++mt)
#pragma unroll
        for (int t = 0; t < (TWO ? TAPS : 1); ++t) odd[mt][t] = sp_v4f{0.f, 0.f, 0.f, 0.f};
    if (ch_begin < ch_end) load_chunk(ch_begin);
    for (int ch = ch_begin; ch < ch_end; ++ch) {
        __syncthreads();
        store_chunk(ch);
        __syncthreads();
        if (ch + 1 < ch_end) load_chunk(ch + 1);
#pragma unroll
        for (int q = 0; q < PX / 4 / WK; ++q) {
            const int u = (q * WK + wk) * 4 + g;  // this lane group's unit
            const int tw = u & (TW - 1), th = (u >> a.lw) & (TH - 1), to = u >> (a.lw + a.lh);
            const sp_v8b* xp = Xs + j * XROW + (to * HR + th * a.st) * HC + tw * a.st;
            sp_v8b av[MT][NS];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    av[mt][s] = Ds[s * DI + ((wm * MT + mt) * 16 + j) * PX + (u ^ (j & (PX - 1)))];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int r = 0; r < RG; ++r)
#pragma unroll
                    for (int s = 0; s < S; ++s) {
                        sp_v8b bv[NS];
#pragma unroll
                        for (int k = 0; k < NS; ++k) bv[k] = xp[(k * CT + ct) * 16 * XROW + r * HC + s];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            {
                            const int t = (ct * RG + r) * S + s;
                            sp_v4f& sum = TWO && q % 2 ? odd[TWO ? mt : 0][TWO ? t : 0] : acc[mt][t];
                            mfma_split<NS, false>(av[mt], bv, sum, sum);
                        }
                    }
        }
    }

    if constexpr (TWO)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int t = 0; t < TAPS; ++t) acc[mt][t] += odd[mt][t];
    if constexpr (WK > 1) {  // the waves' sums, in wave order, MT tiles at a time
        float* red = reinterpret_cast<float*>(smem);
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            __syncthreads();
            if (wk > 0)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<sp_v4f*>(red + (((wk - 1) * WM + wm) * MT + mt) * 256 + lane * 4) = acc[mt][t];
            __syncthreads();
            if (wk == 0)
#pragma unroll
                for (int q = 0; q < WK - 1; ++q)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt][t] +=
                            *reinterpret_cast<const sp_v4f*>(red + ((q * WM + wm) * MT + mt) * 256 + lane * 4);
        }
        if (wk > 0) return;
    }

    float* out = a.part + (size_t)zi * a.K * a.C * a.R * a.S;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = k0 + (wm * MT + mt) * 16 + 4 * g + i;
            if (k >= a.K) continue;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int c = c0 + ct * 16 + j;
                if (c >= a.C) continue;
                float* o = out + ((size_t)k * a.C + c) * a.R * S + r0 * S;
#pragma unroll
                for (int r = 0; r < RG; ++r)
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        if (RG == 1 || r0 + r < a.R) o[r * S + s] = acc[mt][(ct * RG + r) * S + s][i];
            }
        }
    // sums to form again (split.h; where a chunk reaches past dy's plane its
    // zeros meet x); one that has become NaN stays so
    Again redo;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int q = 0; q < TAPS; ++q) redo.add<NS>(acc[mt][q]);
    if (redo.any()) {
#pragma unroll 1
        for (int q = 0; q < MT * TAPS * 4; ++q) {
            const int i = q & 3, tt = (q >> 2) % TAPS, mt = (q >> 2) / TAPS;
            const int k = k0 + (wm * MT + mt) * 16 + 4 * g + i, c = c0 + tt / (RG * S) * 16 + j;
            const int r = r0 + tt / S % RG, s = tt % S;
            if (k >= a.K || c >= a.C || r >= a.R) continue;
            float* o = out + (((size_t)k * a.C + c) * a.R + r) * S + s;
            if (!again<NS>(*o)) continue;
            float v = 0.f;
            for (int ch = ch_begin; ch < ch_end && v == v; ++ch) {
                int oct, p0, q0;
                chunk_at(ch, &oct, &p0, &q0);
                for (int u = 0; u < PX; ++u) {
                    const int qq = q0 + (u & (TW - 1)), pp = p0 + ((u >> a.lw) & (TH - 1));
                    const int ih = pp * a.st + r - a.pad, iw = qq * a.st + s - a.pad;
                    const bool in = ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
                    if (pp >= a.P || qq >= a.Q) continue;
                    for (int e = 0; e < 8; ++e) {
                        const int img = (oct + (u >> (a.lw + a.lh))) * 8 + e;
                        if (img >= a.n) break;
                        const float xv = in ? a.x[((img * a.C + c) * a.H + ih) * a.W + iw] : 0.f;
                        v = fmaf(operand<NS>(a.dy[(img * a.K + k) * PQ + pp * a.Q + qq]), operand<NS>(xv), v);
                    }
                }
            }
            *o = v;
        }
    }
}

constexpr size_t kLdsMax = 160 * 1024;

template <int NS, int BM, int WM, int CT, int RG, int S, int PX>
size_t gw_lds(const GwArgs& a)
{
    const int TW = 1 << a.lw, TH = 1 << a.lh, TO = PX >> (a.lw + a.lh);
    const size_t xp = (size_t)TO * ((TH - 1) * a.st + RG) * ((TW - 1) * a.st + S);
    const size_t main = (size_t)NS * 16 * (BM * PX + 16 * CT * (xp | 1));
    const size_t red = (size_t)(4 / WM - 1) * BM * 64;  // (WK-1) waves x MT tiles x 256 floats, per row of waves
    return main > red ? main : red;
}

template <int NS, int BM, int WM, int CT, int RG, int S, int PX>
hipError_t gw_launch(GwArgs a, int max_splits, int* splits, const Work& wk, hipStream_t st)
{
    constexpr int LP = PX == 16 ? 4 : 3;
    // Chunk of PX units: the least of all chunks' staging, in units a thread
    // loads.  Neighbouring lanes load neighbouring columns, so units of rows
    // shorter than 8 count more (32 bytes a row are a sector), units past the
    // registers are waited for, and a chunk's barriers are four units more.  The
    // fewest chunks alone, as it was, took one pixel of 128 images where a plane is
    // no multiple of 8 (us, 128 images, fp32: 1x1 64 -> 256 at 28x28 643, 87; 3x3 192 ->
    // 384 at 13x13 1,238, 320; 5x5 64 -> 96 at 27x27 2,274, 437; 3x3 64 -> 64 at 33x33
    // 586, 105; of 58 measured shapes in both modes within 17% of the best choice).
    int64_t best = 0;
    double best_cost = 0.0;
    for (int lw = 0; lw <= LP; ++lw)
        for (int lh = 0; lw + lh <= LP; ++lh) {
            const int tw = 1 << lw, th = 1 << lh, to = PX >> (lw + lh);
            if (((tw >> 1) >= a.Q && lw) || ((th >> 1) >= a.P && lh)) continue;
            const int64_t ch = (int64_t)((a.Q + tw - 1) / tw) * ((a.P + th - 1) / th) * (((a.n + 7) / 8 + to - 1) / to);
            const int hc = (tw - 1) * a.st + S;
            const double x = 16.0 * CT * to * ((th - 1) * a.st + RG) * hc / 256;
            auto row = [](int columns) { return columns >= 8 ? 1.0 : columns >= 4 ? 1.6 : columns >= 2 ? 3.0 : 8.0; };
            const double cost = ch * (4.0 + BM * PX / 256 * row(tw) + x * row(hc) + (x > 3.0 ? x - 3.0 : 0.0));
            if (!best || cost < best_cost) {
                best = ch;
                best_cost = cost;
                a.lw = lw;
                a.lh = lh;
                a.tiles_w = (a.Q + tw - 1) / tw;
                a.tiles_h = (a.P + th - 1) / th;
            }
        }
    if (best > INT32_MAX) return hipErrorNotSupported;
    const size_t lds = gw_lds<NS, BM, WM, CT, RG, S, PX>(a);
    if (lds > kLdsMax) return hipErrorNotSupported;
    a.chunks = (int)best;
    a.kblocks = (a.K + BM - 1) / BM;
    a.cblocks = (a.C + 16 * CT - 1) / (16 * CT);
    a.rblocks = (a.R + RG - 1) / RG;
    const int64_t combos = (int64_t)a.kblocks * a.cblocks * a.rblocks;
    // two workgroups per CU as far as there are chunks (a chunk is a round
    // trip to memory whatever its size, so small layers spread out fully)
    int64_t z = (512 + combos - 1) / combos;
    if (z > a.chunks) z = a.chunks;
    if (z > max_splits) z = max_splits;
    if (z >= 8) z = z / 8 * 8;
    a.per = (int)((a.chunks + z - 1) / z);
    a.z = (a.chunks + a.per - 1) / a.per;
    a.by_xcd = a.z >= 8;
    // Up to three images a unit's eight are mostly absent, and the workspace
    // bounds the parts: past so many units a thread stages in turn the implicit
    // GEMM's slices of 16 (bf16: 32) pixels take less (fp32, one image, us: 64 -> 64
    // at 28x28 39 against 22, 64 -> 128 at 56x56 stride 2 47 and 24, 512 -> 512 at
    // 4x4 19 and 61; two images of the second 29 and 27, of the first 21 and 24;
    // bf16 one image 24 -> 56 at 29x23 stride 2 31 and 26, of the first 31 and 34).
    const int TW = 1 << a.lw, TH = 1 << a.lh, TO = PX >> (a.lw + a.lh);
    const int64_t units = (16 * CT * TO * ((TH - 1) * a.st + RG) * ((TW - 1) * a.st + S) + 255) / 256 + BM * PX / 256;
    const int bk = NS == 1 ? 32 : 16;
    const int64_t depth = ((int64_t)a.n * a.P * a.Q + max_splits - 1) / max_splits, slices = (depth + bk - 1) / bk;
    if (a.n < 4 && a.per * units > (NS == 1 ? 10 * slices + 10 * a.n : 3 * slices + 2 * a.n)) return hipErrorNotSupported;
    *splits = a.z;
    const int64_t blocks = (a.by_xcd ? (a.z + 7) / 8 * 8 : a.z) * combos;
    if (blocks > INT32_MAX) return hipErrorNotSupported;
    PSW_LAUNCH(kname("conv_split_wgrad", NS, BM, WM, CT, RG, S, PX), wk, (conv_split_wgrad<NS, BM, WM, CT, RG, S, PX>),
               dim3((unsigned)blocks), dim3(256), lds, st, a);
    return hipGetLastError();
}

template <int NS, int BM, int WM, int PX>
hipError_t gw_taps(const GwArgs& a, int ms, int* sp, const Work& wk, hipStream_t st)
{
    if (a.R == 3 && a.S == 3) return gw_launch<NS, BM, WM, 1, 3, 3, PX>(a, ms, sp, wk, st);
    if (a.S == 5) return gw_launch<NS, BM, WM, 1, 1, 5, PX>(a, ms, sp, wk, st);
    if (a.S == 3) return gw_launch<NS, BM, WM, 1, 1, 3, PX>(a, ms, sp, wk, st);
    if (a.S == 1 && a.C <= 16) return gw_launch<NS, BM, WM, 1, 1, 1, PX>(a, ms, sp, wk, st);
    if (a.S == 1) return gw_launch<NS, BM, WM, 4, 1, 1, PX>(a, ms, sp, wk, st);
    return hipErrorNotSupported;
}

template <int NS>
hipError_t gw_rows(const GwArgs& a, int ms, int* sp, const Work& wk, hipStream_t st)
{
    if (a.K <= 16) return gw_taps<NS, 16, 1, 16>(a, ms, sp, wk, st);
    // half-size tiles and chunks where 64 x 16 ones would be fewer than two per
    // CU (37 images, 24 -> 56 at 29x23, stride 2: 26 -> 16 us)
    const int64_t units = (int64_t)((a.n + 7) / 8) * a.P * a.Q / 16 * ((a.K + 63) / 64) * ((a.C + 15) / 16);
    if (units < 512 && a.S > 1) return gw_taps<NS, 32, 2, 8>(a, ms, sp, wk, st);
    if (a.K <= 32) return gw_taps<NS, 32, 1, 16>(a, ms, sp, wk, st);
    // a 1x1 chunk has one tap to multiply per loaded value: smaller chunks, three
    // workgroups a CU (128 -> 192 at 16x16 b128 52 -> 34 us).  Up to 16 channels one
    // block of them (fp32, us, four blocks and one: 16 images 4 -> 6 at 21x11 stride 2
    // 15.0, 8.9; 16 -> 32 at 14x14 15.5, 10.7; 128 images 4 -> 40 at 20x17 18.4, 13.1)
    if (a.S == 1 && a.C > 16) return gw_launch<NS, 64, 2, 4, 1, 1, 8>(a, ms, sp, wk, st);
    return gw_taps<NS, 64, 2, 16>(a, ms, sp, wk, st);
}

}  // namespace

// Partial sums of dW (each K x C x R x S) for `*splits` <= max_splits parts of
// the reduction; hipErrorNotSupported (nothing launched) for kernels without
// a configuration (other than 1, 3 or 5 columns) and where the implicit GEMM is faster.
hipError_t conv_general_wgrad(const ConvShape& cs, const float* x, const float* dy, float* part, int max_splits,
                              int* splits, int bf16, hipStream_t st)
{
    // byte offsets are 31 bits, and with seven images past the last one 32
    if ((int64_t)cs.n * cs.c * cs.h * cs.w * 4 > INT32_MAX || (int64_t)cs.n * cs.k * cs.p * cs.q * 4 > INT32_MAX ||
        (int64_t)cs.c * cs.h * cs.w * 4 > INT32_MAX / 8 || (int64_t)cs.k * cs.p * cs.q * 4 > INT32_MAX / 8)
        return hipErrorNotSupported;
    if (max_splits < 1) return hipErrorNotSupported;
    GwArgs a{};
    a.x = x; a.dy = dy; a.part = part;
    a.n = cs.n; a.C = cs.c; a.H = cs.h; a.W = cs.w;
    a.K = cs.k; a.P = cs.p; a.Q = cs.q; a.R = cs.r; a.S = cs.s;
    a.st = cs.stride; a.pad = cs.pad;
    const Work wk = conv_work(cs);
    return bf16 ? gw_rows<1>(a, max_splits, splits, wk, st) : gw_rows<3>(a, max_splits, splits, wk, st);
}

}  // namespace psw
