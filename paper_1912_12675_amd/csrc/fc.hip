// Fully connected products on the bf16 matrix cores: C[m][n] (+)= sum_k
// A(m, k) B(k, n), fp32 operands as three bfloat16 parts (split.h), or rounded
// once in bf16 mode.  Forward y = x w^T, backward dx = dy w and dw = dy^T x
// differ in which index of an operand is contiguous in memory.
//
// A workgroup owns BM x BN of C and walks k in stages of 32 KG: both tiles are
// loaded into registers a stage ahead (16 bytes a lane along k, or lanes along
// the row index), split, and kept in LDS as 16-byte units of eight k.  The
// matrix instruction's rows are C's columns, so that a lane ends with four
// consecutive elements of a row of C.  WK waves share one tile and take the
// matrix steps of a stage in turn: with few outputs and a deep reduction the
// chip is filled and memory kept busy by the stages' depth, not by more
// outputs; their sums meet in LDS in wave order, so results do not depend on
// timing.
//
// Measured at 128 x 16384 x 4096 against the gemm that staged scalars (us,
// fp32 / bf16): forward 2,238 -> 204 / 167, dx 655 -> 163, dw 258 -> 140 (268
// MB of weights read, read and written: 40-50 us each at memory's rate, 110 at
// the fp32 matrix rate; timed over repeated calls, a trace shows 220, 160 and 175).
// Forward is bound by the delivery of x to every block of columns, dx and dw
// by their stages' phases following one another.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "split.h"

namespace psw {
namespace {

struct GsArgs {
    const float* A;     // AK: [m][k], row stride lda; else [k][m]
    const float* B;     // BK: [n][k], row stride ldb; else [k][n]
    float* C;           // [M][N]
    const float* bias;  // per column n, or null
    int M, N, K;
    int lda, ldb;
    int nblocks, mblocks;
    int relu, accumulate;
    int vec;            // C rows are 16-byte aligned
    int kchunk;         // k of one part (blockIdx.y), a multiple of the stage
    int64_t part;       // floats from one part's C to the next
};

template <bool AK, bool BK>
__device__ __forceinline__ float plain_dot(const GsArgs& a, int m, int n, int k0, int k1)
{
    float v = 0.f;
    for (int k = k0; k < k1 && v == v; ++k)
        v = fmaf(AK ? a.A[(int64_t)m * a.lda + k] : a.A[(int64_t)k * a.lda + m],
                 BK ? a.B[(int64_t)n * a.ldb + k] : a.B[(int64_t)k * a.ldb + n], v);
    return v;
}

// eight k of one row: `off` its lane offset (kOutside: none), `left` how many
// of the eight exist (a stage past the end of k)
template <bool KC>
__device__ __forceinline__ void load_k8(Buffer b, int off, int ld, bool whole, int left, float (&r)[8])
{
    if (KC && whole) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 u = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
        const f4 v = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(b, off, 16, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            r[e] = u[e];
            r[4 + e] = v[e];
        }
    } else if (whole) {
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = buffer_load(b, off, e * ld * 4);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            r[e] = buffer_load(b, off >= 0 && e < left ? off + e * (KC ? 4 : ld * 4) : kOutside, 0);
    }
}

template <int NS, int BM, int BN, int WM, int WN, int WK, int KG, bool AK, bool BK, bool FAR>
__global__ __launch_bounds__(64 * WM * WN * WK, WM * WN * WK > 8 ? 4 : 2) void gemm_split(GsArgs a)
{
    constexpr int NT = 64 * WM * WN * WK, KU = 4 * KG, ROW = KU + 1;  // units per row; odd row of units
    constexpr int MT = BM / WM / 16, NTL = BN / WN / 16;
    // registers for a second sum: the small products' or, in bf16, of every other step
    constexpr bool OWN = MT * NTL <= 4 && (NS == 3 || KG / WK % 2 == 0);
    constexpr int AI = BM * KU, BI = BN * KU, AV = (AI + NT - 1) / NT, BV = (BI + NT - 1) / NT;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    sp_v8b* const As = reinterpret_cast<sp_v8b*>(smem);  // [NS][BM][ROW]
    sp_v8b* const Bs = As + NS * BM * ROW;               // [NS][BN][ROW]

    // consecutive workgroups go to the 8 XCDs in turn: the row blocks of one
    // column block run on one XCD, one after another (with fewer than eight
    // column blocks, in plain order over all XCDs)
    const int slot = (int)(blockIdx.x >> 3);
    int nb = slot / a.mblocks * 8 + (int)(blockIdx.x & 7), mb = slot % a.mblocks;
    if (a.nblocks < 8) {
        nb = (int)blockIdx.x % a.nblocks;
        mb = (int)blockIdx.x / a.nblocks;
    }
    if (nb >= a.nblocks) return;
    const int m0 = mb * BM, n0 = nb * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);
    const int g = lane >> 4, j = lane & 15;

    const int kbeg = (int)blockIdx.y * a.kchunk, kend = (int)min((int64_t)a.K, (int64_t)kbeg + a.kchunk);
    float* const C = a.C + blockIdx.y * a.part;

    float ar[AV][8], br[BV][8];
    // eight k of row r0 + row of one operand from stage k0's octet o
    auto load_op = [&](auto kc, const float* p, int ld, int rows, int r0, int row, bool in, int o, int k0, bool whole,
                       float(&r)[8]) {
        constexpr bool KC = decltype(kc)::value;
        if constexpr (FAR) {
            const float* q = KC ? p + (int64_t)(r0 + row) * ld : p + r0 + row;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = k0 + o * 8 + e;
                const bool ok = in && k < kend;
                const float v = *(ok ? q + (KC ? (int64_t)k : (int64_t)k * ld) : p);
                r[e] = ok ? v : 0.f;
            }
        } else {
            const Buffer b = KC ? make_buffer(p + (int64_t)r0 * ld + k0, ((int64_t)(rows - r0) * ld - k0) * 4)
                                : make_buffer(p + (int64_t)k0 * ld + r0, ((int64_t)(a.K - k0) * ld - r0) * 4);
            load_k8<KC>(b, in ? (KC ? row * ld + o * 8 : row + o * 8 * ld) * 4 : kOutside, ld, whole, kend - k0 - o * 8,
                        r);
        }
    };
    auto load = [&](int k0) {
        const bool whole = k0 + 8 * KU <= kend;
#pragma unroll
        for (int v = 0; v < AV; ++v) {
            const int idx = tid + v * NT, row = AK ? idx / KU : idx % BM, o = AK ? idx % KU : idx / BM;
            load_op(std::bool_constant<AK>{}, a.A, a.lda, a.M, m0, row, m0 + row < a.M && (AI % NT == 0 || idx < AI), o, k0,
                    whole, ar[v]);
        }
#pragma unroll
        for (int v = 0; v < BV; ++v) {
            const int idx = tid + v * NT, row = BK ? idx / KU : idx % BN, o = BK ? idx % KU : idx / BN;
            load_op(std::bool_constant<BK>{}, a.B, a.ldb, a.N, n0, row, n0 + row < a.N && (BI % NT == 0 || idx < BI), o, k0,
                    whole, br[v]);
        }
    };
    auto put = [&](sp_v8b* dst, int stride, const float(&r)[8]) {
        sp_v8b parts[NS];
        split8<NS>(r, parts);
#pragma unroll
        for (int s = 0; s < NS; ++s) dst[s * stride] = parts[s];
    };
    auto store = [&]() {
#pragma unroll
        for (int v = 0; v < AV; ++v) {
            const int idx = tid + v * NT, row = AK ? idx / KU : idx % BM, o = AK ? idx % KU : idx / BM;
            if (AI % NT == 0 || idx < AI) put(As + row * ROW + o, BM * ROW, ar[v]);
        }
#pragma unroll
        for (int v = 0; v < BV; ++v) {
            const int idx = tid + v * NT, row = BK ? idx / KU : idx % BN, o = BK ? idx % KU : idx / BN;
            if (BI % NT == 0 || idx < BI) put(Bs + row * ROW + o, BN * ROW, br[v]);
        }
    };

    sp_v4f acc[NTL][MT];
#pragma unroll
    for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = sp_v4f{0.f, 0.f, 0.f, 0.f};

    sp_v4f lo[OWN ? NTL : 1][OWN ? MT : 1];
#pragma unroll
    for (int nt = 0; nt < (OWN ? NTL : 1); ++nt)
#pragma unroll
        for (int mt = 0; mt < (OWN ? MT : 1); ++mt) lo[nt][mt] = sp_v4f{0.f, 0.f, 0.f, 0.f};

    load(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += 8 * KU) {
        __syncthreads();
        store();
        __syncthreads();
        if (k0 + 8 * KU < kend) load(k0 + 8 * KU);
#pragma unroll
        for (int q = 0; q < KG / WK; ++q) {
            const int u = (q * WK + wk) * 4 + g;
            if (k0 + (q * WK + wk) * 32 >= kend) break;
            const sp_v8b* ap = As + (wm * MT * 16 + j) * ROW + u;
            const sp_v8b* bp = Bs + (wn * NTL * 16 + j) * ROW + u;
            sp_v8b bv[NTL][NS];
#pragma unroll
            for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
                for (int s = 0; s < NS; ++s) bv[nt][s] = bp[(s * BN + nt * 16) * ROW];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                sp_v8b av[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s) av[s] = ap[(s * BM + mt * 16) * ROW];
#pragma unroll
                for (int nt = 0; nt < NTL; ++nt) {
                    sp_v4f& second = lo[OWN ? nt : 0][OWN ? mt : 0];
                    mfma_split<NS, OWN>(bv[nt], av, NS == 1 && OWN && q % 2 ? second : acc[nt][mt], second);
                }
            }
        }
    }

    if constexpr (OWN)
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] += lo[nt][mt];
    if constexpr (WK > 1) {  // the waves' sums, in wave order
        float* red = reinterpret_cast<float*>(smem);
        __syncthreads();
        if (wk > 0)
#pragma unroll
            for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    *reinterpret_cast<sp_v4f*>(red + ((((wk - 1) * WN + wn) * WM + wm) * NTL * MT + nt * MT + mt) * 256 +
                                               lane * 4) = acc[nt][mt];
        __syncthreads();
        if (wk > 0) return;
        for (int q = 0; q < WK - 1; ++q)
#pragma unroll
            for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[nt][mt] += *reinterpret_cast<const sp_v4f*>(
                        red + (((q * WN + wn) * WM + wm) * NTL * MT + nt * MT + mt) * 256 + lane * 4);
    }

    const int mrow = m0 + wm * MT * 16 + j, ncol = n0 + wn * NTL * 16 + 4 * g;
    if constexpr (NS == 3) {
        Again redo;
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) redo.add<NS>(acc[nt][mt]);
        if (redo.any()) {
            uint64_t bad = 0;
            static_assert(MT * NTL * 4 <= 64, "one bit per sum");
#pragma unroll
            for (int k = 0; k < MT * NTL * 4; ++k)
                bad |= (uint64_t)again<NS>(acc[(k >> 2) / MT][(k >> 2) % MT][k & 3]) << k;
#pragma unroll 1
            for (; bad; bad &= bad - 1) {
                const int at = __ffsll((unsigned long long)bad) - 1;
                const int m = mrow + (at >> 2) % MT * 16, n = ncol + (at >> 2) / MT * 16 + (at & 3);
                if (m >= a.M || n >= a.N) continue;
                const float v = plain_dot<AK, BK>(a, m, n, kbeg, kend);
#pragma unroll
                for (int k = 0; k < MT * NTL * 4; ++k) {
                    sp_v4f& sums = acc[(k >> 2) / MT][(k >> 2) % MT];
                    sums[k & 3] = k == at ? v : sums[k & 3];
                }
            }
        }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = mrow + mt * 16;
        if (m >= a.M) continue;
#pragma unroll
        for (int nt = 0; nt < NTL; ++nt) {
            const int n = ncol + nt * 16;
            float* dst = C + (int64_t)m * a.N + n;
            sp_v4f v = acc[nt][mt];
            if (a.vec && n + 4 <= a.N) {
                if (a.bias) v += sp_v4f{a.bias[n], a.bias[n + 1], a.bias[n + 2], a.bias[n + 3]};
                if (a.relu)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
                if (a.accumulate) v += *reinterpret_cast<const sp_v4f*>(dst);
                __builtin_nontemporal_store(v, reinterpret_cast<sp_v4f*>(dst));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float s = v[i];
                    if (n + i >= a.N) continue;
                    if (a.bias) s += a.bias[n + i];
                    if (a.relu) s = fmaxf(s, 0.f);
                    dst[i] = a.accumulate ? dst[i] + s : s;
                }
            }
        }
    }
}

// Forward of a batch of few rows (both operands contiguous along k).  A
// workgroup owns 16 MT rows by 16 columns, and its WK waves take the steps of
// 32 k in turn, each for the whole tile: no operand is used by two waves, so
// there are no barriers.  Four neighbouring lanes load 64 bytes of a row, and
// the wave's own LDS turns 16 rows of 4 pieces into the operands' order: loads
// in that order (a row's four pieces 16 lanes apart) took a cycle of address
// processing a lane, and bound the kernel (us before, now: 128 x 16384 x 4096
// 285, 228; 128 x 4096 x 4096 72, 53; 16 x 16384 x 4096 62, 50; 128 x 4096 x
// 10 14.4, 8.6).  The order of k within a step is free as long as A and B
// agree, so two pieces 64 bytes apart are a bf16 operand as they stand, and
// eight operands of the fp32 instruction.  The weights are read once and the
// next step's operands are in flight while the matrix cores work.  fp32 uses
// the fp32 instructions: a split costs the vector units 208 cycles an operand,
// eight of nine operands are the batch's, and each would serve one block of
// columns (the tiled kernel takes 370 us at 128 x 16384 x 4096).
template <bool BF, int MT, int WK>
__global__ __launch_bounds__(64 * WK) void gemm_rows(GsArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wk = tid >> 6;
    const int g = lane >> 4, j = lane & 15;
    const int n0 = (int)blockIdx.x * 16, m0 = (int)blockIdx.y * 16 * MT;
    const Buffer ab = make_buffer(a.A + (int64_t)m0 * a.lda, (int64_t)(a.M - m0) * a.lda * 4);
    const Buffer bb = make_buffer(a.B + (int64_t)n0 * a.ldb, (int64_t)(a.N - n0) * a.ldb * 4);
    // lane l loads piece l % 4 of row l / 4 of a block of 16 rows
    const int lr = lane >> 2, lp = lane & 3;
    int aoff[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
        aoff[mt] = m0 + mt * 16 + lr < a.M ? ((mt * 16 + lr) * a.lda + lp * 4) * 4 : kOutside;
    const int boff = n0 + lr < a.N ? (lr * a.ldb + lp * 4) * 4 : kOutside;
    const int full = a.K / 32;

    sp_v4f acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = sp_v4f{0.f, 0.f, 0.f, 0.f};
    typedef float f4 __attribute__((ext_vector_type(4)));
    f4 ar[MT][2], br[2];
    // Half h (16 k) of whole step ks; past the last step nothing is read.
    auto load_a = [&](int ks, int h) {
        const int none = ks < full ? 0 : kOutside, at = ks < full ? ks * 128 + h * 64 : 0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            ar[mt][h] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(ab, aoff[mt] | none, at, 0));
    };
    auto load_b = [&](int ks) {
        const int none = ks < full ? 0 : kOutside, at = ks < full ? ks * 128 : 0;
        br[0] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(bb, boff | none, at, 0));
        br[1] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(bb, (boff + 64) | none, at, 0));
    };
    // The wave's own LDS, 1 KB a block of rows: piece p of row r at unit
    // 4 r + (p ^ (r >> 2)), so that neither the stores by rows nor the reads
    // by pieces meet in a bank.  A wave's LDS operations are done in order:
    // no barrier, the compiler only keeps to that order.
    f4* const own = reinterpret_cast<f4*>(smem) + wk * MT * 64;
    const int put = lr * 4 + (lp ^ (lr >> 2)), get = j * 4 + (g ^ (j >> 2));
    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    f4 av[MT][2], bv[2];
    auto swap_b = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            own[put] = br[h];
            fence();
            bv[h] = own[get];
            fence();
        }
    };
    auto put_a = [&](int h) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) own[mt * 64 + put] = ar[mt][h];
        fence();
    };
    auto mul = [&](int h) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[mt][h] = own[mt * 64 + get];
        fence();
        if constexpr (BF) {
            if (h == 0) return;
            auto bf8 = [](const f4(&r)[2]) {
                float t[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = r[e / 4][e % 4];
                sp_v8b p[1];
                split8<1>(t, p);
                return p[0];
            };
            const sp_v8b b8 = bf8(bv);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b8, bf8(av[mt]), acc[mt], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[h][e], av[mt][h][e], acc[mt], 0, 0, 0);
        }
    };
    load_b(wk);
    load_a(wk, 0);
    load_a(wk, 1);
    for (int ks = wk; ks < full; ks += WK) {
        swap_b();
        load_b(ks + WK);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            put_a(h);
            load_a(ks + WK, h);
            mul(h);
        }
    }
    if (full * 32 < a.K && full % WK == wk) {  // the last step's missing k are zero
        auto part = [&](Buffer b, int off, f4(&r)[2]) {
            const int left = off >= 0 ? a.K - full * 32 - lp * 4 : 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = e / 4 * 16 + e % 4;
                r[e / 4][e % 4] = buffer_load(b, k < left ? off + full * 128 + k * 4 : kOutside, 0);
            }
        };
        part(bb, boff, br);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) part(ab, aoff[mt], ar[mt]);
        swap_b();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            put_a(h);
            mul(h);
        }
    }

    // the waves' sums, in wave order; wave w finishes row blocks w, w + WK, ...
    float* red = reinterpret_cast<float*>(smem);
    if (WK > 1) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<sp_v4f*>(red + (wk * MT + mt) * 256 + lane * 4) = acc[mt];
        __syncthreads();
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (mt % WK != wk) continue;
        sp_v4f v = *reinterpret_cast<const sp_v4f*>(red + mt * 256 + lane * 4);
        for (int q = 1; q < WK; ++q) v += *reinterpret_cast<const sp_v4f*>(red + (q * MT + mt) * 256 + lane * 4);
        const int m = m0 + mt * 16 + j, n = n0 + 4 * g;
        if (m >= a.M) continue;
        float* dst = a.C + (int64_t)m * a.N + n;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (a.bias && n + i < a.N) v[i] += a.bias[n + i];
            if (a.relu) v[i] = fmaxf(v[i], 0.f);
        }
        if (a.vec && n + 4 <= a.N) {
            *reinterpret_cast<sp_v4f*>(dst) = v;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n + i < a.N) dst[i] = v[i];
        }
    }
}

// column sums out[c] = sum_r x[r][c] in double, rows in order within each of
// four lanes of a column, then the lanes in order
__global__ __launch_bounds__(256) void col_sum_k(int rows, int cols, const float* x, float* out)
{
    __shared__ double sh[4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
    double s = 0.0;
    if (c < cols) {
        int r = q;
        for (; r + 28 < rows; r += 32) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = x[(int64_t)(r + 4 * e) * cols + c];
#pragma unroll
            for (int e = 0; e < 8; ++e) s += (double)v[e];
        }
        for (; r < rows; r += 4) s += (double)x[(int64_t)r * cols + c];
    }
    sh[q][threadIdx.x & 63] = s;
    __syncthreads();
    if (q == 0 && c < cols)
        out[c] = (float)(((sh[0][threadIdx.x] + sh[1][threadIdx.x]) + sh[2][threadIdx.x]) + sh[3][threadIdx.x]);
}

// Backward products of few rows, few k and many columns (classifiers of a
// handful of samples over a wide input): V columns a thread, MR rows in
// registers, A by uniform loads, k in order.  A row of B is read once and
// memory is the bound; the 64 x 64 tile spends its time on padding (fp32, dx and
// dw, us: 4 samples 1,200,000 -> 10 229, 8 samples 60,000 -> 10 17.4).
template <int NS, int MR, int V, bool AK>
__global__ __launch_bounds__(256) void gemm_thin(GsArgs a)
{
    typedef float fv __attribute__((ext_vector_type(V)));
    const int64_t n = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (n >= a.N) return;
    const int m0 = (int)blockIdx.y * MR;
    fv acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m] = 0.f;
    auto step = [&](int k, fv b) {
#pragma unroll
        for (int e = 0; e < V; ++e) b[e] = operand<NS>(b[e]);
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            const int row = min(m0 + m, a.M - 1);
            const float v = operand<NS>(AK ? a.A[(int64_t)row * a.lda + k] : a.A[(int64_t)k * a.lda + row]);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[m][e] = fmaf(v, b[e], acc[m][e]);
        }
    };
    auto row_of_b = [&](int k) { return *reinterpret_cast<const fv*>(a.B + (int64_t)k * a.ldb + n); };
    constexpr int U = 4;  // rows of B in flight
    int k = 0;
    for (; k + U <= a.K; k += U) {
        fv b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = row_of_b(k + u);
#pragma unroll
        for (int u = 0; u < U; ++u) step(k + u, b[u]);
    }
    for (; k < a.K; ++k) step(k, row_of_b(k));
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        if (m0 + m >= a.M) break;
        fv* dst = reinterpret_cast<fv*>(a.C + (int64_t)(m0 + m) * a.N + n);
        if (a.accumulate) acc[m] = *dst + acc[m];
        __builtin_nontemporal_store(acc[m], dst);
    }
}

template <int NS, int BM, int BN, int WM, int WN, int WK, int KG, bool AK, bool BK, bool FAR = false>
hipError_t gs_launch(GsArgs a, const Work& wk, hipStream_t st, int parts = 1)
{
    a.mblocks = (a.M + BM - 1) / BM;
    a.nblocks = (a.N + BN - 1) / BN;
    const int64_t blocks = (int64_t)(a.nblocks < 8 ? a.nblocks : (a.nblocks + 7) / 8 * 8) * a.mblocks;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    if (parts == 1) a.kchunk = INT32_MAX / (32 * KG) * (32 * KG);
    constexpr size_t main = (size_t)NS * 16 * (BM + BN) * (4 * KG + 1), red = (size_t)(WK - 1) * BM * BN * 4;
    PSW_LAUNCH(kname("gemm_split", NS, BM, BN, WM, WN, WK, KG, AK, BK, FAR), wk,
               (gemm_split<NS, BM, BN, WM, WN, WK, KG, AK, BK, FAR>), dim3((unsigned)blocks, (unsigned)parts),
               dim3(64 * WM * WN * WK), main > red ? main : red, st, a);
    return hipGetLastError();
}

constexpr int64_t kRowsL2 = 4 << 20;  // bytes

// The depth in parts of a multiple of 64 k, whose sums meet in the workspace:
// where a wave of the one-launch tile would add up more than 16 steps of 32 k
// and the tiles leave the chip room.
struct Parts {
    int64_t tiles;  // of 64 x 64
    bool deep;      // few outputs over a deep k
    bool near, far; // lane offsets: every tile's in 31 bits, not even the 64 x 64 tile's
    int parts, kchunk;
    Parts(const GsArgs& a, int bf16, size_t ws_bytes)
    {
        const int64_t ld = std::max(a.lda, a.ldb);
        // 512 k of a row-contiguous operand or 128 rows of another are the most
        // of any tile here, 64 of either the most of the 64 x 64 tile; past
        // that, plain loads
        near = ld * 512 * 4 <= INT32_MAX;
        far = ld * 64 * 4 > INT32_MAX;
        tiles = (int64_t)((a.M + 63) / 64) * ((a.N + 63) / 64);
        deep = a.K > 512 && (int64_t)((a.M + 15) / 16) * ((a.N + 15) / 16) <= 256;
        const int waves = !near || tiles >= 128 ? 1 : deep ? 16 : 4;
        parts = 1;
        kchunk = 0;
        if (a.K <= 512 * waves || tiles >= 512) return;
        const int64_t least = bf16 ? 128 : 64;
        int64_t z = std::min((1024 + tiles - 1) / tiles, (a.K + least - 1) / least);
        z = std::min(z, (int64_t)(ws_bytes / ((size_t)a.M * a.N * sizeof(float))));
        if (z <= 1) return;
        kchunk = (int)(((a.K + z - 1) / z + 63) / 64 * 64);
        parts = (a.K + kchunk - 1) / kchunk;
    }
};

// Tiles, each with the reason it is there (fp32, us; 128 rows unless said):
// the largest that leaves work for the whole chip, except that
//  - 128 x 128 pays only over many tiles: dw 4096 x 16384, k 128: 140 (64 x 64
//    179; bf16 104 and 86, but 31 and 39 at 4096 x 4096, k 256); dx 128 x 16384, k
//    4096, is 128 tiles of it: 281 (64 x 64 166);
//  - few outputs over a deep k take 16 waves on k: 16 x 227, k 4096: 20.
template <int NS, bool AK, bool BK>
hipError_t gs_pick(GsArgs a, const Work& wk, float* ws, size_t ws_bytes, hipStream_t st)
{
    auto blocks = [&](int bm, int bn) { return (int64_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    const Parts d(a, NS == 1, ws ? ws_bytes : 0);
    if (d.parts > 1 || !d.near) {
        GsArgs p = a;
        if (d.parts > 1) {
            p.kchunk = d.kchunk;
            p.C = ws;
            p.part = (int64_t)a.M * a.N;
            p.vec = a.N % 4 == 0 && (uintptr_t)ws % 16 == 0;
            p.accumulate = 0;
        }
        const hipError_t e = d.far ? gs_launch<NS, 64, 64, 2, 2, 1, 2, AK, BK, true>(p, wk, st, d.parts)
                                   : gs_launch<NS, 64, 64, 2, 2, 1, 2, AK, BK>(p, wk, st, d.parts);
        if (e != hipSuccess || d.parts == 1) return e;
        return reduce_parts(ws, d.parts, p.part, a.C, a.accumulate, st);
    }
    // bf16 forward of more than 64 rows whose x is larger than the L2 (see gemm())
    if constexpr (NS == 1 && AK && BK)
        if (a.M > 64 && a.M <= 256 && (int64_t)a.M * a.K * 4 > kRowsL2)
            return gs_launch<NS, 128, 16, 1, 1, 4, 4, AK, BK>(a, wk, st);
    if (blocks(128, 128) >= 512) return gs_launch<NS, 128, 128, 2, 2, 1, 1, AK, BK>(a, wk, st);
    if (d.tiles >= 128) return gs_launch<NS, 64, 64, 2, 2, 1, 2, AK, BK>(a, wk, st);
    if (d.deep) return gs_launch<NS, 16, 16, 1, 1, 16, 16, AK, BK>(a, wk, st);
    if (blocks(32, 32) >= 64) return gs_launch<NS, 32, 32, 1, 1, 4, 4, AK, BK>(a, wk, st);
    return gs_launch<NS, 16, 16, 1, 1, 4, 4, AK, BK>(a, wk, st);
}

template <int NS, int MR, bool AK>
hipError_t thin_launch(const GsArgs& a, const Work& wk, hipStream_t st)
{
    const unsigned rows = (unsigned)((a.M + MR - 1) / MR);
    if (a.vec && (uintptr_t)a.B % 16 == 0 && a.N >= 1 << 18)
        PSW_LAUNCH(kname("gemm_thin", NS, MR, 4, AK), wk, (gemm_thin<NS, MR, 4, AK>), dim3((unsigned)((a.N + 1023) / 1024), rows),
                   dim3(256), 0, st, a);
    else
        PSW_LAUNCH(kname("gemm_thin", NS, MR, 1, AK), wk, (gemm_thin<NS, MR, 1, AK>), dim3((unsigned)((a.N + 255) / 256), rows),
                   dim3(256), 0, st, a);
    return hipGetLastError();
}

template <bool BF, int MT, int WK>
hipError_t rows_launch(const GsArgs& a, const Work& wk, hipStream_t st)
{
    PSW_LAUNCH(kname("gemm_rows", BF, MT, WK), wk, (gemm_rows<BF, MT, WK>),
               dim3((unsigned)((a.N + 15) / 16), (unsigned)((a.M + 16 * MT - 1) / (16 * MT))), dim3(64 * WK),
               (size_t)WK * MT * 1024, st, a);
    return hipGetLastError();
}

template <bool BF>
hipError_t rows_pick(const GsArgs& a, int64_t most, const Work& wk, hipStream_t st)
{
    // the most rows per workgroup that still leave a workgroup for every
    // other CU (the columns' operands are then read once or twice); else 16
    // rows and 16 waves on the depth of k
    const int64_t cols = (a.N + 15) / 16;
    if (most >= 8 && a.M > 64 && cols * ((a.M + 127) / 128) >= 128) return rows_launch<BF, 8, 8>(a, wk, st);
    if (most >= 4 && a.M > 32 && cols * ((a.M + 63) / 64) >= 128) return rows_launch<BF, 4, 8>(a, wk, st);
    if (most >= 2 && a.M > 16 && cols * ((a.M + 31) / 32) >= 128) return rows_launch<BF, 2, 8>(a, wk, st);
    return a.K > 512 ? rows_launch<BF, 1, 16>(a, wk, st) : rows_launch<BF, 1, 4>(a, wk, st);
}

template <bool AK, bool BK>
hipError_t gemm(GsArgs a, int bf16, float* ws, size_t ws_bytes, hipStream_t st)
{
    const Work wk{2.0 * a.M * a.N * (double)a.K,
                  kF * ((double)a.M * a.K + (double)a.K * a.N + (1.0 + a.accumulate) * a.M * (double)a.N)};
    a.vec = a.N % 4 == 0 && (uintptr_t)a.C % 16 == 0;
    // Forward of up to 256 rows: the weights' traffic and the depth of k decide,
    // not the matrix rate: gemm_rows.  Not over many columns and few k, where
    // its eight waves a workgroup have a step each or none (us at 128 x 64 ->
    // 30,000: rows 32.8, tiles 9.0; 256 x 300 -> 4096: 17.5, 11.5; 128 x 300 ->
    // 4096, 128 tiles: 9.4, 11.2).  bf16 with an x past an XCD's 4 MB of L2
    // (fp32, re-read by every block of columns) takes the LDS tile of 128 rows
    // where its workgroups of 16 columns fill the chip (tile, rows: 256 x 8192 ->
    // 8192 196, 340; 200 x 6000 -> 3000 79, 98; 128 x 16384 -> 4096 167, 172; 256 x
    // 16384 -> 2048 159, 147; 128 x 8200 -> 1024 84, 43)
    if constexpr (AK && BK) {
        const int64_t most = INT32_MAX / 64 / std::max(a.lda, a.ldb);  // blocks of 16 rows in 31 bits
        const bool tiles = a.M > 32 && a.K <= 1024 && (int64_t)((a.M + 63) / 64) * ((a.N + 63) / 64) >= 256;
        const bool past = bf16 && a.N >= 2560 && a.M > 64 && (int64_t)a.M * a.K * 4 > kRowsL2;
        if (most >= 1 && a.M <= 256 && !tiles && !past)
            return bf16 ? rows_pick<true>(a, most, wk, st) : rows_pick<false>(a, most, wk, st);
    }
    if constexpr (!BK)  // columns enough for a workgroup of one each on half the CUs
        if (a.M <= 32 && a.K <= 128 && a.N >= 1 << 15) {
            if (a.M <= 4) return bf16 ? thin_launch<1, 4, AK>(a, wk, st) : thin_launch<3, 4, AK>(a, wk, st);
            return bf16 ? thin_launch<1, 16, AK>(a, wk, st) : thin_launch<3, 16, AK>(a, wk, st);
        }
    return bf16 ? gs_pick<1, AK, BK>(a, wk, ws, ws_bytes, st) : gs_pick<3, AK, BK>(a, wk, ws, ws_bytes, st);
}

}  // namespace

hipError_t fc_gemm_fwd(int n, int in, int out, const float* x, const float* w, const float* b, int relu, float* y,
                       int bf16, hipStream_t st)
{
    GsArgs a{};
    a.A = x; a.B = w; a.C = y; a.bias = b; a.relu = relu;
    a.M = n; a.N = out; a.K = in;
    a.lda = in;  // x[n][i]
    a.ldb = in;  // w[o][i]
    return gemm<true, true>(a, bf16, nullptr, 0, st);
}

size_t fc_gemm_bwd_ws_bytes(int n, int in, int out)
{
    GsArgs a{};
    a.M = n; a.N = in; a.K = out;
    a.lda = out;
    a.ldb = in;
    const Parts d(a, 0, SIZE_MAX);  // bf16 takes as many or fewer
    return d.parts > 1 ? (size_t)d.parts * n * in * sizeof(float) : 0;
}

hipError_t fc_gemm_bwd(int n, int in, int out, const float* x, const float* w, const float* dy, float* dx,
                       int dx_accumulate, float* dw, float* db, int bf16, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (dx) {
        GsArgs a{};
        a.A = dy; a.B = w; a.C = dx; a.accumulate = dx_accumulate;
        a.M = n; a.N = in; a.K = out;
        a.lda = out;  // dy[n][o]
        a.ldb = in;   // w[o][i], k = o
        const hipError_t e = gemm<true, false>(a, bf16, (float*)ws, ws_bytes, st);
        if (e != hipSuccess) return e;
    }
    GsArgs a{};
    a.A = dy; a.B = x; a.C = dw;
    a.M = out; a.N = in; a.K = n;
    a.lda = out;  // dy[n][o], k = n
    a.ldb = in;   // x[n][i], k = n
    const hipError_t e = gemm<false, false>(a, bf16, nullptr, 0, st);
    if (e != hipSuccess || !db) return e;
    // the column sums of dy (not a product, so never rounded to bf16)
    PSW_LAUNCH(kname("col_sum_k"), (Work{(double)n * out, kF * ((double)n * out + out)}), col_sum_k,
               dim3((unsigned)((out + 63) / 64)), dim3(256), 0, st, n, out, dy, db);
    return hipGetLastError();
}

}  // namespace psw
