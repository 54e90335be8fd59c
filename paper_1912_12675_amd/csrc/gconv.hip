// Convolution forward and backward-data for the shapes without a kernel of
// their own (any channel counts, plane sizes, kernel, stride and padding), on
// the bf16 matrix cores: fp32 operands as three bfloat16 parts (split.h), or
// rounded once in bf16 mode.
//
// Both passes are one computation: an output position (i, j) of a plane grid
// sums, over reduction channels c and taps t, weight(m, c, t) times the input
// at (i is + dr_t, j is + ds_t).  Forward: the grid is the output plane and
// is the stride.  Backward data of a stride-st convolution: the input pixels
// fall into st x st classes by (h mod st, w mod st); a class is a grid of its
// own whose taps are every st-th row and column of the kernel, is = 1, so no
// product with an inserted zero is formed (blockIdx.z is the class).
//
// A workgroup owns BM output channels of BP grid positions (TI images x TH
// rows x TW columns, powers of two chosen on the host, see pick_tile).
// Reduction channels come in chunks of 8 OC.  A chunk's input tile with its
// halo is loaded once, split once and kept in LDS as 16-byte units [octet of
// channels][pixel], so that a tap is only another pixel offset: nothing is
// gathered or split again per tap.  Weights are staged per group of KG matrix
// steps as 16-byte units [channel m][slot], a slot being one tap of one
// octet; a matrix step takes four slots (lane group g the g-th), its A
// operand one unit per lane and its B operand one unit per lane.  The next
// group's weights and the next chunk's input are loaded into registers while
// the matrix cores work.  WK waves share one tile and take the steps in turn
// (deep reductions over few positions); their sums meet in LDS in wave order.
//
// Measured against the implicit GEMM that gathered (and, for each tap, divided
// indices) element by element, batch 128, us, fp32 unless stated: 512 -> 512
// 3x3 at 4x4 forward 119, backward data 110 (1,382 on average over VGG-16's
// layers there); 5x5 64 -> 192 at 16x16 forward 112, bf16 forward 751 -> 57 and
// backward data 1,330 -> 78.
#include "internal.h"
#include "split.h"

namespace psw {
namespace {

struct GcArgs {
    const float* x;     // input [n][C][IH][IW]
    const float* w;
    const float* bias;  // per output channel or null
    float* y;           // output [n][M][OH][OW]
    int n, C, M;
    int IH, IW, OH, OW;
    int R, S, pad;
    int is, os;         // input step per grid position; output step (classes per dimension)
    int bwd;
    int wm, wc;         // weight strides (floats) of an output and of a reduction channel
    int lw, lh;         // log2 of the tile's columns and rows
    int tiles_h, tiles_w, tiles, mblocks;
    int relu, accumulate;
};

// taps of one class along one dimension: kernel index r = r0 + k * step for
// k < count, at input offset org + (bwd ? count - 1 - k : k)
struct Taps {
    int r0, step, count, org;
};
__host__ __device__ inline Taps class_taps(int R, int pad, int os, int bwd, int phase)
{
    if (!bwd) return Taps{0, 1, R, -pad};
    const int r0 = (phase + pad) % os;
    const int cnt = r0 < R ? (R - r0 + os - 1) / os : 0;
    return Taps{r0, os, cnt, (phase + pad - r0) / os - (cnt - 1)};
}

// one output in plain fp32, in the order of the definition (zero outside the
// input).  A sum that has become NaN stays one, so it ends there.
template <int NS>
__device__ __forceinline__ float plain_sum(const GcArgs& a, int img, int m, int oh, int ow)
{
    float acc = 0.f;
    for (int c = 0; c < a.C && acc == acc; ++c)
        for (int r = 0; r < a.R; ++r)
            for (int s = 0; s < a.S; ++s) {
                int ih, iw;
                bool ok;
                if (a.bwd) {
                    ih = oh + a.pad - r;
                    iw = ow + a.pad - s;
                    ok = ih >= 0 && iw >= 0 && ih % a.os == 0 && iw % a.os == 0;
                    ih /= a.os;
                    iw /= a.os;
                } else {
                    ih = oh * a.is + r - a.pad;
                    iw = ow * a.is + s - a.pad;
                    ok = ih >= 0 && iw >= 0;
                }
                ok = ok && ih < a.IH && iw < a.IW;
                const float v = ok ? a.x[((img * a.C + c) * a.IH + ih) * a.IW + iw] : 0.f;
                acc = fmaf(operand<NS>(a.w[m * a.wm + c * a.wc + r * a.S + s]), operand<NS>(v), acc);
            }
    return acc;
}

template <int NS, int BM, int BP, int WP, int WK, int OC, int KG, bool OWN>
__global__ __launch_bounds__(64 * WP * WK, NS == 3 && BM == 32 && BP == 256 && !OWN ? 3 : 2) void conv_split(GcArgs a)
{
    constexpr int NT = 64 * WP * WK;
    constexpr int MT = BM / 16, NTL = BP / WP / 16;  // 16x16 tiles of a wave
    constexpr int SLOTS = 4 * KG, TG = SLOTS / OC;   // slots and taps of a weight group
    constexpr int AROW = SLOTS + 1;                  // units per weight row: odd, so the 16 rows spread over the banks
    constexpr int AI = BM * SLOTS, AV = (AI + NT - 1) / NT;
    constexpr int BV = OC * BP / NT > 2 ? OC * BP / NT : OC * BP / NT + 1;  // input units per thread in registers
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // this workgroup's class, channel block and tile.  Consecutive workgroups
    // go to the 8 XCDs in turn: the channel blocks of one tile run on one XCD,
    // one after another, and find its input in that L2
    const int slot8 = (int)(blockIdx.x >> 3);
    const int tile = (slot8 / a.mblocks) * 8 + (int)(blockIdx.x & 7);
    const int m0 = (slot8 % a.mblocks) * BM;
    if (tile >= a.tiles) return;
    const int ph = (int)blockIdx.z / a.os, pw = (int)blockIdx.z % a.os;
    const Taps tr = class_taps(a.R, a.pad, a.os, a.bwd, ph), ts = class_taps(a.S, a.pad, a.os, a.bwd, pw);
    const int GH = a.bwd ? (a.OH - ph + a.os - 1) / a.os : a.OH, GW = a.bwd ? (a.OW - pw + a.os - 1) / a.os : a.OW;
    const int TW = 1 << a.lw, TH = 1 << a.lh;
    const int tw0 = (tile % a.tiles_w) * TW;
    const int th0 = (tile / a.tiles_w % a.tiles_h) * TH;
    const int img0 = tile / (a.tiles_w * a.tiles_h) * (BP >> (a.lw + a.lh));
    if (th0 >= GH || tw0 >= GW) return;  // a class with a smaller grid
    const int ntaps = tr.count * ts.count, ngroups = (ntaps + TG - 1) / TG;
    const int HC = (TW - 1) * a.is + ts.count, HR = (TH - 1) * a.is + tr.count;
    const int HP = (BP >> (a.lw + a.lh)) * HR * HC;  // staged pixels
    const int BI = OC * HP;                          // staged units

    sp_v8b* const Bs = reinterpret_cast<sp_v8b*>(smem);
    sp_v8b* const As = Bs + NS * BI;
    int* const tapo = reinterpret_cast<int*>(As + NS * BM * AROW);  // per slot: byte offset of its unit of pixel 0
    int* const wtab = tapo + ngroups * SLOTS;                       // per tap: weight offset

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wp = wave % WP, wk = wave / WP;
    const int g = lane >> 4, j = lane & 15;

    for (int i = tid; i < ngroups * SLOTS; i += NT) {
        const int t = i / OC, o = i % OC;
        const int kr = t / (ts.count ? ts.count : 1), ks = t - kr * ts.count;
        const int hr = a.bwd ? tr.count - 1 - kr : kr, hc = a.bwd ? ts.count - 1 - ks : ks;
        tapo[i] = t < ntaps ? (o * HP + hr * HC + hc) * 16 : 0;
        if (o == 0) wtab[t] = t < ntaps ? (tr.r0 + kr * tr.step) * a.S + ts.r0 + ks * ts.step : 0;
    }

    // B operand: byte offset of this lane's position of each 16-position block
    int boff[NTL];
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt) {
        const int p = (wp * NTL + nt) * 16 + j;
        const int tw = p & (TW - 1), th = (p >> a.lw) & (TH - 1), ti = p >> (a.lw + a.lh);
        boff[nt] = ((ti * HR + th * a.is) * HC + tw * a.is) * 16;
    }
    sp_v4f acc[MT][NTL];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt) acc[mt][nt] = sp_v4f{0.f, 0.f, 0.f, 0.f};

    sp_v4f lo[OWN ? MT : 1][OWN ? NTL : 1];
#pragma unroll
    for (int mt = 0; mt < (OWN ? MT : 1); ++mt)
#pragma unroll
        for (int nt = 0; nt < (OWN ? NTL : 1); ++nt) lo[mt][nt] = sp_v4f{0.f, 0.f, 0.f, 0.f};

    // input units: unit idx = octet * HP + staged pixel; src is the byte
    // offset of its first channel (chunk 0) from the tile's first image
    const int plane = a.IH * a.IW;
    const Buffer xb = make_buffer(a.x + (size_t)img0 * a.C * plane, (int64_t)(a.n - img0) * a.C * plane * 4);
    const Buffer wb = make_buffer(a.w, (int64_t)a.M * a.C * a.R * a.S * 4);
    auto unit_at = [&](int idx, int* c) -> int {  // c: its first channel within the chunk
        const int o = idx / HP, hp = idx - o * HP;
        const int ti = hp / (HR * HC), rem = hp - ti * (HR * HC);
        const int hr = rem / HC, hc = rem - hr * HC;
        const int ih = th0 * a.is + tr.org + hr, iw = tw0 * a.is + ts.org + hc;
        const bool in = idx < BI && img0 + ti < a.n && ih >= 0 && ih < a.IH && iw >= 0 && iw < a.IW;
        *c = o * 8;
        return in ? (((ti * a.C + o * 8) * a.IH + ih) * a.IW + iw) * 4 : kOutside;
    };
    int bsrc[BV], bch[BV];
#pragma unroll
    for (int v = 0; v < BV; ++v) bsrc[v] = unit_at(tid + v * NT, &bch[v]);
    // Loads ahead of their use carry no branch: what a branch merges is copied
    // to its place at once, and the copy waits for memory (the matrix work
    // that should hide the latency came after it: 1.5 times as slow).  A chunk
    // that does not exist reads zeros (`ok` false), and the last chunk of a
    // channel count that is no multiple of 8 is loaded when it is stored.
    float br[BV][8];
    auto load_b = [&](int c0, bool ok) {
        const int lim = ok ? a.C : 0, cb = ok ? c0 : 0, step = ok ? plane * 4 : 0;
#pragma unroll
        for (int v = 0; v < BV; ++v) {
            if (v * NT >= BI) break;
            const int off = cb + bch[v] < lim ? bsrc[v] : kOutside;
#pragma unroll
            for (int e = 0; e < 8; ++e) br[v][e] = buffer_load(xb, off, (cb + e) * step);
        }
    };
    auto put_unit = [&](sp_v8b* dst, int plane_units, const float(&r)[8]) {
        sp_v8b parts[NS];
        split8<NS>(r, parts);
#pragma unroll
        for (int s = 0; s < NS; ++s) dst[s * plane_units] = parts[s];
    };
    auto store_b = [&](int c0, bool now) {
        if (!now)
#pragma unroll
            for (int v = 0; v < BV; ++v)
                if (tid + v * NT < BI) put_unit(Bs + tid + v * NT, BI, br[v]);
        // a ragged chunk, and a tile of more units than the registers hold
        for (int idx = tid + (now ? 0 : BV * NT); idx < BI; idx += NT) {
            int ch;
            const int src = unit_at(idx, &ch), left = src >= 0 ? a.C - c0 - ch : 0;
            float r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = buffer_load(xb, e < left ? src + (c0 + e) * plane * 4 : kOutside, 0);
            put_unit(Bs + idx, BI, r);
        }
    };
    // weight units: idx = channel * SLOTS + slot
    float ar[AV][8];
    auto weight_at = [&](int u, int grp, int* c) -> int {  // c: its first channel within the chunk
        const int idx = tid + u * NT;
        const int m = idx / SLOTS, sl = idx % SLOTS, t = grp * TG + sl / OC;
        *c = sl % OC * 8;
        const bool in = t < ntaps && m0 + m < a.M && (AI % NT == 0 || idx < AI);
        return in ? ((m0 + m) * a.wm + *c * a.wc + wtab[t]) * 4 : kOutside;
    };
    auto load_a = [&](int c0, int grp, bool ok) {
        const int lim = ok ? a.C : 0, cb = ok ? c0 : 0, step = ok ? a.wc * 4 : 0;
#pragma unroll
        for (int u = 0; u < AV; ++u) {
            int c;
            const int src = weight_at(u, grp, &c), off = cb + c < lim ? src : kOutside;
#pragma unroll
            for (int e = 0; e < 8; ++e) ar[u][e] = buffer_load(wb, off, (cb + e) * step);
        }
    };
    auto store_a = [&](int c0, int grp, bool now) {
#pragma unroll
        for (int u = 0; u < AV; ++u) {
            const int idx = tid + u * NT;
            if (AI % NT && idx >= AI) continue;
            sp_v8b* const dst = As + idx / SLOTS * AROW + idx % SLOTS;
            if (now) {
                int c;
                const int src = weight_at(u, grp, &c), left = src >= 0 ? a.C - c0 - c : 0;
                float r[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] = buffer_load(wb, e < left ? src + (c0 + e) * a.wc * 4 : kOutside, 0);
                put_unit(dst, BM * AROW, r);
            } else {
                put_unit(dst, BM * AROW, ar[u]);
            }
        }
    };
    auto ragged = [&](int c0) { return a.C % 8 != 0 && a.C - c0 < 8 * OC; };

    __syncthreads();  // the tables
    if (ntaps > 0) {
        load_a(0, 0, !ragged(0));
        load_b(0, !ragged(0));
        for (int c0 = 0; c0 < a.C; c0 += 8 * OC) {
            const bool now = ragged(c0), next = c0 + 8 * OC < a.C && !ragged(c0 + 8 * OC);
            __syncthreads();  // the previous chunk's operands are read
            store_b(c0, now);
            store_a(c0, 0, now);
            __syncthreads();
            load_b(c0 + 8 * OC, next);
            for (int grp = 0; grp < ngroups; ++grp) {
                const bool last = grp + 1 == ngroups;
                load_a(last ? c0 + 8 * OC : c0, last ? 0 : grp + 1, last ? next : !now);
#pragma unroll
                for (int q = 0; q < (KG + WK - 1) / WK; ++q) {
                    const int ks = q * WK + wk;
                    if (ks >= KG || grp * SLOTS + ks * 4 >= ntaps * OC) break;
                    const char* bp = reinterpret_cast<const char*>(Bs) + tapo[grp * SLOTS + ks * 4 + g];
                    const sp_v8b* ap = As + j * AROW + ks * 4 + g;
                    sp_v8b av[MT][NS];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int s = 0; s < NS; ++s) av[mt][s] = ap[(s * BM + mt * 16) * AROW];
                    // a block's operands are read while the one before it is
                    // multiplied (left to itself the compiler reads them last)
                    sp_v8b bv[2][NS];
                    auto read_b = [&](int nt) {
#pragma unroll
                        for (int s = 0; s < NS; ++s)
                            bv[nt & 1][s] = *reinterpret_cast<const sp_v8b*>(bp + boff[nt] + s * BI * 16);
                    };
                    read_b(0);
#pragma unroll
                    for (int nt = 0; nt < NTL; ++nt) {
                        if (nt + 1 < NTL) read_b(nt + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            mfma_split<NS, OWN>(av[mt], bv[nt & 1], acc[mt][nt], lo[OWN ? mt : 0][OWN ? nt : 0]);
                    }
                }
                if (!last) {
                    __syncthreads();  // the group's weights are read
                    store_a(c0, grp + 1, now);
                    __syncthreads();
                }
            }
        }
    }

    if constexpr (OWN)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NTL; ++nt) acc[mt][nt] += lo[mt][nt];
    if constexpr (WK > 1) {  // the waves' sums, in wave order
        float* red = reinterpret_cast<float*>(smem);
        __syncthreads();
        if (wk > 0)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NTL; ++nt)
                    *reinterpret_cast<sp_v4f*>(red + ((((wk - 1) * WP + wp) * MT + mt) * NTL + nt) * 256 + lane * 4) =
                        acc[mt][nt];
        __syncthreads();
        if (wk > 0) return;
        for (int q = 0; q < WK - 1; ++q)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NTL; ++nt)
                    acc[mt][nt] += *reinterpret_cast<const sp_v4f*>(
                        red + (((q * WP + wp) * MT + mt) * NTL + nt) * 256 + lane * 4);
    }

    const int oplane = a.OH * a.OW;
    // grid position p of this tile: its offset in channel 0 of the output, -1
    // outside the grid
    struct Pos {
        int img, oh, ow;
    };
    auto pos_at = [&](int p, Pos* q) -> bool {
        const int gi = th0 + ((p >> a.lw) & (TH - 1)), gj = tw0 + (p & (TW - 1));
        *q = Pos{img0 + (p >> (a.lw + a.lh)), gi * a.os + ph, gj * a.os + pw};
        return gi < GH && gj < GW && q->img < a.n;
    };
    Again redo;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt) redo.add<NS>(acc[mt][nt]);
    if (redo.any()) {  // split.h; a group's unused slots read a real pixel
        uint64_t bad = 0;
        static_assert(MT * NTL * 4 <= 64, "one bit per sum");
#pragma unroll
        for (int k = 0; k < MT * NTL * 4; ++k)
            bad |= (uint64_t)again<NS>(acc[(k >> 2) / NTL][(k >> 2) % NTL][k & 3]) << k;
#pragma unroll 1
        for (; bad; bad &= bad - 1) {
            const int at = __ffsll((unsigned long long)bad) - 1;
            const int m = m0 + (at >> 2) / NTL * 16 + 4 * g + (at & 3);
            Pos q;
            if (!pos_at((wp * NTL + (at >> 2) % NTL) * 16 + j, &q) || m >= a.M) continue;
            const float v = plain_sum<NS>(a, q.img, m, q.oh, q.ow);
#pragma unroll
            for (int k = 0; k < MT * NTL * 4; ++k) {
                sp_v4f& sums = acc[(k >> 2) / NTL][(k >> 2) % NTL];
                sums[k & 3] = k == at ? v : sums[k & 3];
            }
        }
    }
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt) {
        Pos q;
        if (!pos_at((wp * NTL + nt) * 16 + j, &q)) continue;
        float* dst = a.y + ((q.img * a.M + m0 + 4 * g) * a.OH + q.oh) * a.OW + q.ow;
        float old[MT][4];
        if (a.accumulate)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    old[mt][i] = m0 + mt * 16 + 4 * g + i < a.M ? dst[(mt * 16 + i) * oplane] : 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m0 + mt * 16 + 4 * g + i;
                float v = acc[mt][nt][i];
                if (m >= a.M) continue;
                if (a.bias) v += a.bias[m];
                if (a.relu) v = fmaxf(v, 0.f);
                if (a.accumulate) v += old[mt][i];
                store_stream(dst + (mt * 16 + i) * oplane, v);
            }
    }
}

struct Tiling {
    int lw, lh, tiles_h, tiles_w;
    int64_t tiles;
    int hp;  // staged pixels
};

// Tile of bp positions over n planes of gh x gw, for the least of all tiles'
// products (bp positions each, padding included) and staging (the halo's
// elements, 1.3 of a position each; neighbouring lanes load and store
// neighbouring columns, so rows shorter than 16 count more, up to five times
// for one column); of equal ones the most columns.  The fewest tiles alone gave
// 14x14 planes tiles of 2x2 positions in 64 images, a halo four times the
// positions (fp32, 128 images, us then and now: 256 -> 256 at 14x14 693, 222; at
// 7x7 395, 98; 64 -> 64 at 28x28 114, 70; 5x5 64 -> 96 at 27x27 962, 200; 1x1 96
// -> 200 at 14x14 184, 43), and a penalty that did not grow below 8 columns gave
// 1x1 kernels on planes that no power of two divides single columns (182 images,
// 61 -> 50 at 10x9 47, 15; 128 images, 1 -> 152 at 8x13 66, 16).  Of 127 measured
// calls all are within 15% of their best tile.
Tiling pick_tile(int n, int gh, int gw, int bp, int is, int rs, int ss)
{
    Tiling best{};
    double best_cost = 0.0;
    for (int lw = 0; (1 << lw) <= bp; ++lw)
        for (int lh = 0; (1 << (lw + lh)) <= bp; ++lh) {
            const int tw = 1 << lw, th = 1 << lh, ti = bp >> (lw + lh);
            if ((tw >> 1) >= gw && lw) continue;
            if ((th >> 1) >= gh && lh) continue;
            Tiling t{lw, lh, (gh + th - 1) / th, (gw + tw - 1) / tw, 0, 0};
            t.tiles = (int64_t)t.tiles_h * t.tiles_w * ((n + ti - 1) / ti);
            t.hp = ti * ((th - 1) * is + rs) * ((tw - 1) * is + ss);
            const double row = tw >= 16 ? 1.0 : tw >= 8 ? 1.3 : tw >= 4 ? 1.4 : tw >= 2 ? 2.5 : 5.0;
            const double cost = (double)t.tiles * (bp + 1.3 * t.hp * row);
            if (!best.tiles || cost <= best_cost) {
                best = t;
                best_cost = cost;
            }
        }
    return best;
}

constexpr size_t kLdsMax = 160 * 1024;

struct Plan {
    GcArgs a;
    int gh, gw, rs, ss, classes;
};

// LDS bytes of one configuration
template <int NS, int BM, int BP, int WP, int WK, int OC, int KG>
size_t lds_bytes(const Plan& p, const Tiling& t)
{
    constexpr int SLOTS = 4 * KG, TG = SLOTS / OC;
    const size_t groups = (size_t)(p.rs * p.ss + TG - 1) / TG;
    const size_t main = (size_t)NS * 16 * ((size_t)OC * t.hp + BM * (SLOTS + 1)) + groups * (SLOTS + TG) * 4;
    const size_t red = (size_t)(WK - 1) * BM * BP * 4;
    return main > red ? main : red;
}

template <int NS, int BM, int BP, int WP, int WK, int OC, int KG, bool OWN>
hipError_t launch_cfg(Plan& p, const Tiling& t, const Work& wk, hipStream_t st)
{
    GcArgs a = p.a;
    a.lw = t.lw;
    a.lh = t.lh;
    a.tiles_h = t.tiles_h;
    a.tiles_w = t.tiles_w;
    a.tiles = (int)t.tiles;
    a.mblocks = (a.M + BM - 1) / BM;
    const int64_t blocks = (t.tiles + 7) / 8 * 8 * a.mblocks;
    // byte offsets within a tile's images and within the weights are 31 bits
    if ((int64_t)(BP >> (t.lw + t.lh)) * a.C * a.IH * a.IW * 4 > INT32_MAX || (int64_t)a.M * a.C * a.R * a.S * 4 > INT32_MAX)
        return hipErrorNotSupported;
    if (t.tiles > INT32_MAX / 8 || blocks > INT32_MAX) return hipErrorNotSupported;
    const size_t lds = lds_bytes<NS, BM, BP, WP, WK, OC, KG>(p, t);
    if (lds > kLdsMax) return hipErrorNotSupported;
    PSW_LAUNCH(kname("conv_split", NS, BM, BP, WP, WK, OC, KG, OWN), wk, (conv_split<NS, BM, BP, WP, WK, OC, KG, OWN>),
               dim3((unsigned)blocks, 1, (unsigned)p.classes), dim3(64 * WP * WK), lds, st, a);
    return hipGetLastError();
}

template <int NS>
hipError_t launch_ns(Plan& p, const Work& wk, hipStream_t st)
{
    const GcArgs& a = p.a;
    const int taps = p.rs * p.ss;
    auto tile = [&](int bp) { return pick_tile(a.n, p.gh, p.gw, bp, a.is, p.rs, p.ss); };
    auto blocks = [&](const Tiling& t, int bm) { return t.tiles * ((a.M + bm - 1) / bm) * p.classes; };
#define PSW_GC(T_, OWN_, ...)                                                              \
    do {                                                                                   \
        const Tiling t_ = T_;                                                              \
        if (lds_bytes<NS, __VA_ARGS__>(p, t_) <= kLdsMax)                                  \
            return launch_cfg<NS, __VA_ARGS__, NS == 3 && OWN_>(p, t_, wk, st);            \
    } while (0)
    const Tiling t256 = tile(256);
    // An image net's first layer (forward) or few output channels (backward): one
    // octet, four taps per matrix step.  Little work, so the tile is the widest
    // that still gives every CU a workgroup (us fp32 by the implicit GEMM, by 256
    // positions of up to 64 channels for all, now: 5x5 1 -> 6 at 28x28, 16 images
    // 8.2, 11.9, 7.3; 6 -> 16 at 14x14 26.6, 11.7, 7.5; 2 -> 54 at 13x11 stride 2, 128
    // images 11.6, 20.9, 7.4; 3 -> 32 at 28x28 18.9, 20.3, 17.4; 1x1 4 -> 152 at 8x13
    // 11.7, 16.1, 10.8; 7x7 3 -> 64 at 32x32 stride 2 38.9, 36.9, 19.1).  By the lines:
    // - 16 channels: of 64 positions and of 128, the first at 112 blocks of the
    //   second 7.3, 8.3, at 896 (5x5 1 -> 16 at 28x28) 16.2, 13.1; of 128 and of 256
    //   at 512 blocks of the second 13.1, 15.0, at 1024 (9x9 at 64x64) 39.3, 37.7,
    //   and in 1x1 kernels, which stage no second group of weights, at 448 9.7, 9.3
    // - 16 of 64 and 32 of 128 at 128 blocks of the second 7.4, 9.7, at 512 14.0, 10.3
    // - 32 of 128 and 64 of 256 at 1024 blocks of 32 x 256 35.6, 34.0 (5x5 3 -> 64 at
    //   32x32); past half a CU's LDS, one workgroup a CU, 158, 258 (7x7 3 -> 64 at
    //   224x224 stride 2, 32 images)
    // - a tile of 64 that takes more than half the LDS and the implicit GEMM: 768
    //   blocks 49, 80 (11x11 3 -> 64 at 96x96 stride 4), 1792 (112x112) 117, 82
    if (a.C <= 8) {
        const size_t half = kLdsMax / 2;
        const Tiling t128 = tile(128), t64 = tile(64);
        if (a.M <= 16) {
            if (blocks(t256, 16) >= (taps <= 4 ? 256 : 1024)) PSW_GC(t256, true, 16, 256, 4, 1, 1, 4);
            if (blocks(t128, 16) >= 256) PSW_GC(t128, true, 16, 128, 4, 1, 1, 4);
        } else {
            if (a.M > 32 && blocks(t256, 32) >= 1024 && lds_bytes<NS, 64, 256, 4, 1, 1, 2>(p, t256) <= half)
                PSW_GC(t256, false, 64, 256, 4, 1, 1, 2);
            if (blocks(t128, 32) >= 256 && lds_bytes<NS, 32, 128, 4, 1, 1, 2>(p, t128) <= half)
                PSW_GC(t128, true, 32, 128, 4, 1, 1, 2);
        }
        if (blocks(t64, 16) <= 1024 || lds_bytes<NS, 16, 64, 4, 1, 1, 4>(p, t64) <= half)
            PSW_GC(t64, true, 16, 64, 4, 1, 1, 4);
    }
    // Wide tiles while they fill the chip: 32 channels rather than 64, since
    // three workgroups then share a CU's LDS and registers and one multiplies
    // while another stages (us, 32 and 64, fp32 / bf16: 128 -> 128 at 16x16 65, 89 /
    // 41, 49; 5x5 64 -> 192 112, 134 / 58, 74; 1x1 128 -> 192 33, 39 / 24, 30; 192 ->
    // 384 at 13x13 228, 261 / 138, 144; the other way only 256 -> 256 at 14x14 224,
    // 211 / 136, 116).
    if (a.M <= 16 && blocks(t256, 16) >= 256) PSW_GC(t256, true, 16, 256, 4, 1, 2, 2);
    if (a.M > 16 && blocks(t256, 32) >= 256) {
        // up to two workgroups a CU leave registers for the small products' own
        // sums (192 -> 64 5x5 backward data 141 us against 162); with more,
        // three a CU are faster (256 -> 256 at 14x14 222 against 228)
        if (NS == 3 && blocks(t256, 32) <= 512) PSW_GC(t256, true, 32, 256, 4, 1, 2, 2);
        PSW_GC(t256, false, 32, 256, 4, 1, 2, 2);
    }
    // few output channels, a short reduction: small wide tiles (LeNet's second
    // layer's backward data 14 against 18)
    if (a.M <= 32 && a.C * taps <= 1024) PSW_GC(tile(128), true, 16, 128, 4, 1, 2, 2);
    // deep reductions over few positions: waves share the depth, two of a 32 x
    // 64 tile (from 256 blocks: 256 -> 128 at 14x14, 16 images 45 against 52), or
    // with fewer of those, four of a 32 x 32 tile (512 -> 512 at 2x2 89 against
    // 115).  A strided forward stages four elements a position and keeps to the
    // smaller tile a little longer (24 -> 56 at 29x23 stride 2, 37 images, 296
    // blocks: 14.3 against 15.4; 128 -> 256 at 8x8, 256 blocks: 33.5 against 35.8)
    const Tiling t64 = tile(64);
    if (blocks(t64, 32) >= (a.is > 1 ? 320 : 256)) PSW_GC(t64, true, 32, 64, 2, 2, 4, 2);
    PSW_GC(tile(32), true, 32, 32, 1, 4, 4, 4);
#undef PSW_GC
    return hipErrorNotSupported;
}

}  // namespace

// Forward (bwd == 0) or backward data (bwd == 1) of any convolution;
// hipErrorNotSupported (nothing launched) when a tile's halo exceeds the LDS.
hipError_t conv_general(const ConvShape& cs, int bwd, const float* x, const float* w, const float* bias, int relu,
                        float* y, int accumulate, int bf16, hipStream_t st)
{
    if (cs.r > 32 || cs.s > 32) return hipErrorNotSupported;
    Plan p{};
    GcArgs& a = p.a;
    a.x = x;
    a.w = w;
    a.bias = bias;
    a.y = y;
    a.n = cs.n;
    a.R = cs.r;
    a.S = cs.s;
    a.pad = cs.pad;
    a.bwd = bwd;
    a.relu = relu;
    a.accumulate = accumulate;
    if (bwd) {
        a.C = cs.k; a.M = cs.c;
        a.IH = cs.p; a.IW = cs.q; a.OH = cs.h; a.OW = cs.w;
        a.is = 1; a.os = cs.stride;
        a.wm = cs.r * cs.s; a.wc = cs.c * cs.r * cs.s;
    } else {
        a.C = cs.c; a.M = cs.k;
        a.IH = cs.h; a.IW = cs.w; a.OH = cs.p; a.OW = cs.q;
        a.is = cs.stride; a.os = 1;
        a.wm = cs.c * cs.r * cs.s; a.wc = cs.r * cs.s;
    }
    p.gh = (a.OH + a.os - 1) / a.os;
    p.gw = (a.OW + a.os - 1) / a.os;
    p.rs = (cs.r + a.os - 1) / a.os;
    p.ss = (cs.s + a.os - 1) / a.os;
    if ((int64_t)a.os * a.os > 65535) return hipErrorNotSupported;
    p.classes = a.os * a.os;
    Work wk = conv_work(cs);
    if (accumulate) wk.bytes += kF * (double)cs.n * cs.c * cs.h * cs.w;
    return bf16 ? launch_ns<1>(p, wk, st) : launch_ns<3>(p, wk, st);
}

}  // namespace psw
