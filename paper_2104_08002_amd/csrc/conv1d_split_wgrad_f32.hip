// FP32 backward-weight on the bf16 matrix instructions (each float the sum of three bfloat16 numbers, a product the six
// largest of their nine products; see conv1d_split_f32.hip).
//
// The contraction runs over positions: A = dy (16 filters x 32 positions), B = x shifted by the tap (32 positions x 16
// channels).  x sits in LDS as [part][8 channels][position] and is read with the transposing LDS read, so a tap is a row
// offset whatever the dilation; dy sits in operand order.  A workgroup (one per CU) owns a strip of units of QC positions,
// 16 filters, 16 channels and TW NTW taps.  Eight of its waves multiply: wave v owns NTW of the taps and every WK-th
// k-step of 32 positions (TW WK = 8), and the WK sums of a tap are added in a fixed order.  The other eight load, split and
// write the next unit meanwhile (two units in LDS, the loads of two more in registers).
// Partial tiles and second stage are those of the small-channel kernel, ws[(pair * strips + strip) * S + s][16][16]; a layer
// of one strip (few positions, or 129 block pairs and more) has neither.
//
// With many taps the matrix instructions bound it, at the clock they are granted with values as dense as these (C = K = 64,
// S = 33: 1.2 PFLOP/s in the first stage, a large product of matrices 1.33 on such values); with few the loads and the splitting
// do (S = 5: 62 us, about 55 without the products).  While every wave did both, one filter or two blocks at a time, loads one
// wave's share of a unit ahead and in lanes that fell on 16 rows (64 cache accesses a load instead of 4) it took, in us, then
// and now, both stages (normal values; events around launches back to back, both builds in turn on one card; a trace of four
// launches reads up to 15 % more of either): N = 8, C = K = 64, W = 20000: S = 5, d = 1 96 and 63, S = 33, d = 4 234 and 217,
// S = 51, d = 8 350 and 313; N = 16, C = K = 15, W = 60000, S = 51, d = 8 150 and 125; N = 12, C = 24, K = 40, W = 4999, S = 7, d = 3
// 44 and 21; N = 20, C = K = 48, W = 3001, S = 17, d = 3 64 and 36; N = 8, C = K = 256, W = 2000, S = 3 155 and 86.
#include "conv1d_split_f32.h"

namespace conv1d {
namespace {
using namespace sp;

constexpr int kRole = 512;  // threads that multiply, and as many that stage
constexpr int kMaxUnit = kRole / 2;  // positions: a staging thread has one 16-byte slot of dy
constexpr int kXTasks = 3;           // and at most so many of x
// Two running sums of a tap, one for every other unit, where the registers allow: half as many roundings of each.
constexpr bool two_sums(int ntw) { return ntw <= 7; }
constexpr bool four_steps(int ntw) { return ntw <= 9 && ntw != 7; }  // dy of four k-steps fits beside the sums

struct SwfArgs {
    const float* x;
    const float* dy;
    float* ws;  // nullptr: one strip, straight into dw
    float* dw;
    int C, K, W, Q, S, d, P;
    long x_sn, dy_sn, dw_sk, dw_sc;
    int N, qc, upr, nunits, strips, tw_sh, tgroups, kblocks, cblocks, lx, lxp;
};

typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_at4;  // four floats from any float on

// XT: slots of x of a staging thread
template <int NTW, int XT>
__global__ __launch_bounds__(2 * kRole, 4) void split_wgrad_f32_kernel(SwfArgs a) {
    extern __shared__ u32x4 lds[];
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int block_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tid = threadIdx.x & (kRole - 1), wave = block_wave & 7;
    const int QC = a.qc, TW = 1 << a.tw_sh, WK = 8 >> a.tw_sh;
    const int tw = wave & (TW - 1), wk = wave >> a.tw_sh;
    const int ndy = QC * 2, nx = 2 * a.lxp;   // 16-byte slots per part
    const int stage = 3 * (ndy + nx);

    int id = xcd_logical_id(blockIdx.x, gridDim.x);
    const int cb = id % a.cblocks;
    id /= a.cblocks;
    const int kb = id % a.kblocks;
    id /= a.kblocks;
    const int tg = id % a.tgroups, strip = id / a.tgroups;
    const int k0 = kb * 16, c0 = cb * 16, s0 = tg * (NTW << a.tw_sh);
    const int u_begin = static_cast<int>(static_cast<long>(strip) * a.nunits / a.strips);
    const int u_end = static_cast<int>(static_cast<long>(strip + 1) * a.nunits / a.strips);

    // Loads are issued without a branch, where lanes have nothing to load too: the compiler counts them to wait for the
    // older ones alone, and past a branch it waits for all.  Consecutive lanes load consecutive positions (64 lanes in 16
    // rows take the cache 64 accesses).
    struct Set {
        float dv[8], xv[XT][8];
    };
    Set sets[2];
    // byte offsets in a sample, which the plan keeps below 2^32
    const int half = wave >> 2, xpos = tid & 255;  // this thread's 8 channels and its first position
    unsigned xrow[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) xrow[e] = 4u * static_cast<unsigned>(min(c0 + 8 * half + e, a.C - 1) * a.W);
    const int dyi = min(tid, ndy - 1), dym = dyi / (QC / 8), dyj = dyi - dym * (QC / 8);  // filter, and which 8 of 32 positions
    const unsigned dyrow = 4u * static_cast<unsigned>(min(k0 + dym, a.K - 1) * a.Q);
    const int dyq = 32 * (dyj >> 2) + 4 * (dyj & 3);
    // the filters of a position are turned by it, so that neither the lanes that write (positions) nor those that read
    // (filters) meet in a bank
    const int dyslot = dyj * 16 + ((dym ^ dyj) & 15);
    const bool whole_rows = k0 + 16 <= a.K, whole_channels = c0 + 16 <= a.C;
    // a row's last loads go on into the next row, the tensor's last ones begin up to 3 elements early
    const unsigned dyend = 4u * static_cast<unsigned>(a.K * a.Q - 4);
    auto dy_offset = [&](int q) { return dyrow + 4u * static_cast<unsigned>(min(q, a.Q - 1)); };
    auto request = [&](int u, Set& set) __attribute__((always_inline)) {
        const int n = u / a.upr, q0 = (u - n * a.upr) * QC;
        const char* dyb = reinterpret_cast<const char*>(a.dy + n * a.dy_sn);
        const char* xb = reinterpret_cast<const char*>(a.x + n * a.x_sn);
        const unsigned last = n == a.N - 1 ? dyend : 0xffffffffu;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4_at4 v = *reinterpret_cast<const f32x4_at4*>(dyb + min(dy_offset(q0 + dyq + 16 * h), last));
#pragma unroll
            for (int e = 0; e < 4; ++e) set.dv[4 * h + e] = v[e];
        }
        const int col0 = q0 + s0 * a.d - a.P;
#pragma unroll
        for (int k = 0; k < XT; ++k) {
            const unsigned col = 4u * static_cast<unsigned>(clampi(col0 + min(xpos + 256 * k, a.lx - 1), 0, a.W - 1));
#pragma unroll
            for (int e = 0; e < 8; ++e) set.xv[k][e] = *reinterpret_cast<const float*>(xb + (xrow[e] + col));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto park = [&](int u, u32x4* b, const Set& set) __attribute__((always_inline)) {
        const int n = u / a.upr, q0 = (u - n * a.upr) * QC;
        // The matrix instruction cuts sums off towards minus infinity, which adds up over millions of terms: every other
        // unit of the layer is multiplied with -dy and subtracted, so that the offsets cancel, within a strip or, where
        // strips have a unit or two, between them.  (Counted from the strip's first unit they did not cancel in strips of
        // one: C = K = 15, S = 7, 66000 columns of 80 % zeros 3.6e-7 of the gradient, FP32 instruction 1.8e-7.)
        const unsigned sign = (u & 1) ? 0x80000000u : 0u;
        const bool early = n == a.N - 1 && q0 + QC > a.Q - 4;
        const bool dy_inside = whole_rows && q0 + QC <= a.Q;
        if (64 * wave < ndy) {
            const int q = q0 + dyq;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = set.dv[e];
            if (early) {
#pragma unroll
                for (int h = 0; h < 8; h += 4) {
                    const unsigned off = dy_offset(q + 4 * h);
                    const unsigned sh = off > dyend ? (off - dyend) >> 2 : 0u;
                    v[h] = sh & 1 ? v[h + 1] : v[h];
                    v[h + 1] = sh & 1 ? v[h + 2] : v[h + 1];
                    v[h + 2] = sh & 1 ? v[h + 3] : v[h + 2];
                    v[h] = sh & 2 ? v[h + 2] : v[h];
                    v[h + 1] = sh & 2 ? v[h + 3] : v[h + 1];
                }
            }
            if (!dy_inside) {
                const int left = k0 + dym < a.K ? a.Q - q : 0;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (16 * (e >> 2) + (e & 3) >= left) v[e] = 0.f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(__float_as_uint(v[e]) ^ sign);
            const Split8 s = split8(v);
            u32x4* o = b + dyslot;
            if (tid < ndy) {
                o[0] = s.h;
                o[ndy] = s.m;
                o[2 * ndy] = s.l;
            }
        }
        u32x4* xs = b + 3 * ndy + half * a.lxp;
        const int col0 = q0 + s0 * a.d - a.P;
        const bool x_inside = whole_channels && col0 >= 0 && col0 + a.lx <= a.W;
#pragma unroll
        for (int k = 0; k < XT; ++k) {
            if (64 * (wave & 3) + 256 * k >= a.lx) break;
            const int pos = xpos + 256 * k, col = col0 + pos;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = set.xv[k][e];
            if (!x_inside) {
                const int cleft = (col >= 0 && col < a.W) ? a.C - c0 - 8 * half : 0;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e >= cleft) v[e] = 0.f;
            }
            const Split8 s = split8(v);
            if (pos < a.lx) {
                xs[pos] = s.h;
                xs[nx + pos] = s.m;
                xs[2 * nx + pos] = s.l;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // f(unit, its place in the strip modulo 2) and a barrier, over the strip.  (With a way out in the middle of the loop the
    // compiler could not count the loads either.)
    auto each_unit = [&](auto f) __attribute__((always_inline)) {
        int u = u_begin;
        for (; u + 1 < u_end; u += 2) {
            f(u, std::integral_constant<int, 0>{});
            __syncthreads();
            f(u + 1, std::integral_constant<int, 1>{});
            __syncthreads();
        }
        if (u < u_end) {
            f(u, std::integral_constant<int, 0>{});
            __syncthreads();
        }
    };
    if (block_wave >= 8) {
        request(u_begin, sets[0]);
        if (u_end - u_begin == 1) {
            // no loads of units that are not there (C = K = 4, W = 3992, S = 1 7.3 us with them, now 6.7; N = 21, C = K = 4, W = 584,
            // S = 49, d = 8 11.2 and 10.0)
            park(u_begin, lds, sets[0]);
            __syncthreads();
            __syncthreads();
            return;
        }
        request(min(u_begin + 1, u_end - 1), sets[1]);
        park(u_begin, lds, sets[0]);
        request(min(u_begin + 2, u_end - 1), sets[0]);
        __syncthreads();
        each_unit([&](int u, auto par) __attribute__((always_inline)) {
            constexpr int PAR = decltype(par)::value;
            Set& set = sets[1 - PAR];
            if (u + 1 < u_end) park(u + 1, lds + (1 - PAR) * stage, set);
            request(min(u + 3, u_end - 1), set);
        });
        return;  // (a barrier does not wait for waves that have ended)
    }

    // Running sums of a tap; sums[1] is that of every other unit, whose products have the other sign.  Their roundings are
    // what the error of a gradient is made of, so up to four k-steps are summed by themselves first (C = K = 64, S = 33, d = 4,
    // W = 20000, N = 8: 2.4e-7 with an addition per k-step, now 1.6e-7; as one chain of matrix instructions, which cut off at the
    // size of the sum so far, 2.1e-7).
    constexpr int NS = two_sums(NTW) ? 2 : 1;
    f32x4 sums[NS][NTW];
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int s = 0; s < NS; ++s) sums[s][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // rows of 8 channels, two planes: this lane's piece of rows 4 g .. 4 g + 3
    const int piece = 2 * (((l16 >> 1) & 1) * a.lxp + 4 * g + (l16 >> 2)) + (l16 & 1);
    __syncthreads();
    each_unit([&](int, auto par) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        const u32x4* cur = lds + PAR * stage;
        const int xs0 = 2 * (PAR * stage + 3 * ndy + tw * NTW * a.d);
        // H k-steps, WK apart
        auto steps = [&](int ks, auto count) __attribute__((always_inline)) {
            constexpr int H = decltype(count)::value;
            u32x4 y[H][3];
            int at = piece, mine = g;
            opaque(at);  // or addresses of every copy of this code are kept in registers of their own
            opaque(mine);
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int row = 4 * (ks + h * WK) + mine;
#pragma unroll
                for (int i = 0; i < 3; ++i) y[h][i] = cur[i * ndy + row * 16 + ((l16 ^ row) & 15)];
            }
            // the next reads are issued in front of the products of these, and no earlier (left to itself the compiler reads
            // further ahead and spills)
            u32x4 b[2][3];
            at += xs0 + 64 * ks;
            auto read = [&](int r) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const u32x2* p = reinterpret_cast<const u32x2*>(lds) + at + i * 2 * nx;
                    const u32x2 lo = read_tr(p), hi = read_tr(p + 32);
                    b[r & 1][i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                }
                // one running index, not one register per tap and part
                at += r % H == H - 1 ? 2 * a.d - 64 * WK * (H - 1) : 64 * WK;
                opaque(at);
            };
            read(0);
            f32x4 total;
#pragma unroll
            for (int r = 0; r < H * NTW; ++r) {
                if (r + 1 < H * NTW) read(r + 1);
                __builtin_amdgcn_sched_barrier(0);
                const int t = r / H, h = r % H;
                f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 6; ++k) part = mfma(y[h][kPartB[k]], b[r & 1][kPartA[k]], part);
                total = h == 0 ? part : total + part;
                if (h == H - 1) {
                    f32x4& sum = sums[PAR % NS][t];
                    sum = NS == 1 && PAR ? sum - total : sum + total;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int ks = wk;
        if constexpr (four_steps(NTW))
            for (; ks + 3 * WK < QC / 32; ks += 4 * WK) steps(ks, std::integral_constant<int, 4>{});
        for (; ks + WK < QC / 32; ks += 2 * WK) steps(ks, std::integral_constant<int, 2>{});
        if (ks < QC / 32) steps(ks, std::integral_constant<int, 1>{});
    });
    f32x4 acc[NTW];
#pragma unroll
    for (int i = 0; i < NTW; ++i) acc[i] = NS == 2 ? sums[0][i] - sums[NS - 1][i] : sums[0][i];

    // the k-step shares of a tap, the upper half of them to the lower (one after the other: 0.4 us more for the eight of S = 5)
    f32x4* red = reinterpret_cast<f32x4*>(lds);
    for (int half = WK / 2; half > 0; half /= 2) {
        f32x4* mine = red + ((wk & (half - 1)) * TW + tw) * NTW * 64 + lane;
        if (wk >= half && wk < 2 * half)
#pragma unroll
            for (int i = 0; i < NTW; ++i) mine[i * 64] = acc[i];
        __syncthreads();
        if (wk < half)
#pragma unroll
            for (int i = 0; i < NTW; ++i) acc[i] += mine[i * 64];
        __syncthreads();
    }
    if (wk != 0) return;
    const float turn = (u_begin & 1) ? -1.f : 1.f;  // such a strip added up its units with the opposite sign
    float* ws = a.ws + (static_cast<long>(kb * a.cblocks + cb) * a.strips + strip) * a.S * 256;
    float* dw = a.dw + (k0 + 4 * g) * a.dw_sk + (c0 + l16) * a.dw_sc;
#pragma unroll
    for (int i = 0; i < NTW; ++i) {
        const int s = s0 + tw * NTW + i;
        if (s < a.S)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (a.ws) ws[s * 256 + (4 * g + j) * 16 + l16] = turn * acc[i][j];
                else if (k0 + 4 * g + j < a.K && c0 + l16 < a.C) dw[j * a.dw_sk + s] = turn * acc[i][j];
            }
    }
}

struct Plan {
    bool ok;
    int ntw, grid;
    SwfArgs a;
    size_t lds;
    long most;  // strips that the workspace holds
    double roundings;
};

// positions of a plane of 8 channels, rounded up so that the two planes of a read begin in different halves of the banks
long padded(long lx) { return ((lx + 7) & ~15L) + 8; }

// N = 2, C = K = 4, W = 256, S = 5, d = 2, two units: 9.0 us in two strips, 8.8 in one (C = K = 32, W = 500, S = 17, d = 4 9.4
// and 8.9); three units (N = 3, C = K = 16, W = 256, S = 9, d = 2): 9.3 in three strips, 10.5 in one.
constexpr long kOneStrip = 2;

// taps of a wave, within the 128 registers of 16 waves
constexpr int kTaps[] = {3, 5, 7, 9, 13};

// Roundings of a weight gradient before its second stage: a strip of `longest` units of `steps` k-steps per wave, then the
// WK shares of a tap as a tree and, where every other unit has a sum of its own, the difference of the two.
double roundings(int ntw, int WK, int steps, long longest) {
    const int left = four_steps(ntw) ? steps % 4 : steps, adds = (steps - left) / 4 + left / 2 + left % 2;
    double r = chain_roundings(adds * (two_sums(ntw) ? (longest + 1) / 2 : longest)) + (two_sums(ntw) && longest > 1 ? 1 : 0);
    for (; WK > 1; WK /= 2) r += 1;
    return r;
}

// The least that any tile of either kernel rounds off: one k-step an addition, in the best number of shares.
double least_roundings(const WgradProblem& p, long most) {
    const long steps = static_cast<long>(p.N) * cdiv(p.Q, 32), strips = most < steps ? most : steps, per_strip = (steps + strips - 1) / strips;
    double least = chain_roundings(per_strip);
    for (int WK = 2; WK <= 8; WK *= 2) {
        const double r = chain_roundings((per_strip + WK - 1) / WK) + chain_roundings(WK);
        if (r < least) least = r;
    }
    return least;
}

// the fastest tile, or the fastest of at most so many roundings
Plan search(const WgradProblem& p, const double* most_roundings) {
    Plan best{};
    if (p.bf16 || p.dw_sc != p.S || static_cast<long>(p.N) * p.Q < kMinTerms) return best;
    if (static_cast<long>(p.K) * p.Q < 4) return best;  // dy is loaded by four elements of a sample
    const size_t wsb = smallc_wgrad_f32_blocks_workspace(p);  // the partial tiles take no more than that kernel's
    if (wsb == 0) return best;
    const int cblocks = cdiv(p.C, 16), kblocks = cdiv(p.K, 16);
    const long most = static_cast<long>(wsb / (static_cast<size_t>(cblocks) * kblocks * p.S * 1024));
    double best_cost = 0;
    for (const int ntw : kTaps) {
        for (int tw_sh = 0; tw_sh <= 3; ++tw_sh) {
            const int taps = ntw << tw_sh, tgroups = cdiv(p.S, taps), WK = 8 >> tw_sh;
            if (tw_sh > 0 && tgroups == cdiv(p.S, taps / 2)) continue;  // half the waves would do
            const long per_strip = static_cast<long>(cblocks) * kblocks * tgroups;
            const long halo = static_cast<long>(taps - 1) * p.d;
            const long turns = (most * per_strip + 255) / 256, one = per_strip < 256 ? 256 / per_strip : 1;
            long before = 0;
            // units whose x is one, two or three positions per staging thread, and small ones for short rows
            for (int i = 0; i < 6; ++i) {
                long QC = i < 3 ? ((i + 1) * (kRole / 2) - halo) & ~31L : 32L << (i - 3);
                const long fits = (static_cast<long>(kLdsAll / 96) - 2 * (halo + 23)) / 4;  // 2 stages of 3 parts
                if (QC > fits) QC = fits & ~31L;
                if (QC > kMaxUnit) QC = kMaxUnit;
                if (QC < 32 || QC == before) continue;
                before = QC;
                const long lx = QC + halo, lxp = padded(lx);
                const size_t stage = static_cast<size_t>(3 * (2 * QC + 2 * lxp)) * 16;
                const size_t red = WK > 1 ? static_cast<size_t>(taps) * (WK / 2) * 1024 : 0;
                const size_t lds = red > 2 * stage ? red : 2 * stage;
                if (2 * lx > kXTasks * kRole || lds > kLdsAll) continue;
                const int steps = cdiv(QC / 32, WK);
                // one k-step per addition and one running sum: not over more, shorter units than this
                if (steps == 1 && !two_sums(ntw) && QC < kMaxUnit && QC < p.Q) continue;
                const int upr = static_cast<int>((static_cast<unsigned>(p.Q) + static_cast<unsigned>(QC) - 1) / static_cast<unsigned>(QC));
                const long nunits = static_cast<long>(p.N) * upr;
                if (nunits > 0x3fffffffL) continue;
                // As many strips as the workspace holds, but no few workgroups over a whole number per CU: six pairs of
                // blocks in 43 strips took two turns, 34 us, where 42 strips take 26.  One turn at most where the k-steps
                // that are summed by themselves more than make up for the longer sums of fewer strips (with as many: N = 53,
                // C = 40, K = 7, W = 9177, S = 51, d = 16 1.8e-7 off where 1.6e-7 in all strips).
                const long by_itself = (steps < 2 ? 1 : steps >= 4 && four_steps(ntw) ? 4 : 2) * (two_sums(ntw) ? 2 : 1);
                long strips = most;
                if (turns > 1 && one * by_itself >= 2 * most) strips = one;
                else if (turns > 1 && most * per_strip < turns * 230 && 256 * (turns - 1) >= per_strip) strips = 256 * (turns - 1) / per_strip;
                if (strips > nunits) strips = nunits;
                // one strip while a few units cost less than the second stage, which it does without
                if (nunits <= kOneStrip) strips = 1;
                if (most_roundings && strips > 0 && roundings(ntw, WK, steps, (nunits + strips - 1) / strips) > *most_roundings)
                    strips = most < nunits ? most : nunits;
                if (strips < 1 || strips * per_strip > (1 << 20)) continue;
                const long longest = static_cast<unsigned>(nunits + strips - 1) / static_cast<unsigned>(strips);  // units of the longest strip
                if (most_roundings && roundings(ntw, WK, steps, longest) > *most_roundings) continue;
                // Cycles of a unit on one SIMD, the products of its two multiplying waves beside what its two staging waves
                // do; a fit to all tiles on 17 layers (C, K 4 ... 256, 1 ... 51 taps): what is taken is within 9 % of the
                // fastest, 2 % on average.
                const double mm = steps * (270.0 * ntw + 200.0), staging = 950.0 * (1 + cdiv(2 * lx, kRole));
                const double unit = mm > staging ? mm + 0.26 * staging : staging + 0.26 * mm;
                const double waves = static_cast<double>((strips * per_strip + 255) / 256);
                const double cost = waves * (unit * longest + 11000 + WK * taps * 42.0) + (strips > 1 ? 7000 : 0);
                if (best.ok && cost >= best_cost) continue;
                best_cost = cost;
                best.ok = true;
                best.ntw = ntw;
                best.lds = lds;
                best.grid = static_cast<int>(strips * per_strip);
                SwfArgs& a = best.a;
                a.qc = static_cast<int>(QC); a.upr = upr; a.nunits = static_cast<int>(nunits); a.strips = static_cast<int>(strips);
                a.tw_sh = tw_sh; a.tgroups = tgroups; a.lx = static_cast<int>(lx); a.lxp = static_cast<int>(lxp);
            }
        }
    }
    if (!best.ok) return best;
    SwfArgs& a = best.a;
    best.most = most;
    const int WK = 8 >> a.tw_sh;
    best.roundings = roundings(best.ntw, WK, cdiv(a.qc / 32, WK), cdiv(a.nunits, a.strips));
    a.x = static_cast<const float*>(p.x);
    a.dy = static_cast<const float*>(p.dy);
    a.ws = a.strips > 1 ? static_cast<float*>(p.ws) : nullptr;
    a.dw = p.dw; a.dw_sk = p.dw_sk; a.dw_sc = p.dw_sc;
    a.N = p.N; a.C = p.C; a.K = p.K; a.W = p.W; a.Q = p.Q; a.S = p.S; a.d = p.d; a.P = p.P;
    a.x_sn = p.x_sn; a.dy_sn = p.dy_sn;
    a.cblocks = cblocks; a.kblocks = kblocks;
    return best;
}

// The fastest tile may keep fewer sums than the kernel of several filter blocks, which takes all strips and mostly eight
// shares: no tile rounds more often than that kernel would.  Error against 64 bits in 1e-7, time in us, of the fastest tile,
// of this rule and of that kernel: N = 33, C = K = 160, W = 957, S = 33, d = 12 2.3, 1.4 and 1.4, 326, 388 and 727; N = 8,
// C = 144, K = 160, W = 11290, S = 25, d = 4 2.5, 2.0 and 2.1, 635, 842 and 1319; N = 41, C = 42, K = 40, W = 55280, S = 46,
// d = 16 3.4, 2.6 and 3.4, 3120, 3060 and 4280.  One layer in 25 takes another tile for it.  A few roundings are less than
// those of the steps and of the second stage, and are not compared; nor is what no tile can round less often (another search
// is 1 us of host time, which would show in the short launches that have so few).  Errors of 340 drawn layers of more than 3000
// weights over that kernel's: 0.94 in the median, more than 1.03 in one (1.07); the worst seen is a short sum, whose additions
// within a unit count too: N = 4, C = K = 19, W = 2772, S = 33, d = 4 1.23e-7 for 1.11e-7.
constexpr double kFewRoundings = 8;

Plan make_plan(const WgradProblem& p) {
    const Plan fastest = search(p, nullptr);
    if (!fastest.ok || fastest.roundings <= kFewRoundings || fastest.roundings <= least_roundings(p, fastest.most)) return fastest;
    double most = split_f32_wgrad_pair_roundings(p);
    if (most < kFewRoundings) most = kFewRoundings;
    if (fastest.roundings <= most) return fastest;
    const Plan fewer = search(p, &most);
    return fewer.ok ? fewer : fastest;  // (no layer of 50000 of all kinds was without one)
}

template <int NTW>
hipError_t run(const Plan& pl, hipStream_t st) {
    const int xt = cdiv(pl.a.lx, kRole / 2);
    auto kern = xt == 1 ? split_wgrad_f32_kernel<NTW, 1> : xt == 2 ? split_wgrad_f32_kernel<NTW, 2> : split_wgrad_f32_kernel<NTW, 3>;
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), pl.lds);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3(pl.grid), dim3(2 * kRole), pl.lds, st, pl.a);
}

}  // namespace

bool split_f32_wgrad_tile(const WgradProblem& p, SplitTile* t) {
    if (split_f32_wgrad_pair_tile(p, t)) return true;
    const Plan pl = make_plan(p);
    if (pl.ok) *t = SplitTile{1, pl.ntw, cdiv(pl.a.nunits, pl.a.strips), pl.grid, pl.roundings, cdiv(pl.a.lx, kRole / 2)};
    return pl.ok;
}

bool split_f32_wgrad_supported(const WgradProblem& p) {
    SplitTile t;
    return split_f32_wgrad_tile(p, &t);
}

hipError_t split_f32_wgrad_launch(const WgradProblem& p, hipStream_t st, bool* taken) {
    hipError_t e = split_f32_wgrad_pair_launch(p, st, taken);
    if (*taken) return e;
    const Plan pl = make_plan(p);
    *taken = pl.ok;
    if (!pl.ok) return hipSuccess;
    switch (pl.ntw) {
        case 3: e = run<3>(pl, st); break;
        case 5: e = run<5>(pl, st); break;
        case 7: e = run<7>(pl, st); break;
        case 9: e = run<9>(pl, st); break;
        case 13: e = run<13>(pl, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess || pl.a.strips == 1) return e;
    return smallc_wgrad_reduce_launch(pl.a.ws, p.dw, p.K, p.C, p.S, p.dw_sk, p.dw_sc, pl.a.strips, st);
}

}  // namespace conv1d
