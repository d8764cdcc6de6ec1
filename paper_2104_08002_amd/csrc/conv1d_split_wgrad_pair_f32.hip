// FP32 backward-weight on the bf16 matrix instructions, two or four blocks of 16 filters per workgroup, in waves that
// split as well as multiply (see conv1d_split_wgrad_f32.hip for the kernel that has waves for each, the splitting and the
// partial tiles).
//
// x is split once for all blocks of a workgroup.  That is what counts where workgroups of one pair of blocks leave CUs idle,
// for the workspace has one or two partial tiles per pair then (129 to 255 pairs), and where x is mostly the halo of the taps.
// N = 8, C = K = 192, W = 12616, S = 17, d = 4 1000 us, waves for each 1122; N = 54, C = K = 182, W = 4424, S = 15, d = 2 2390 and
// 2951; N = 30, C = K = 115, W = 2192, S = 49, d = 16 579 and 665.
//
// A = dy (16 filters x 32 positions), B = x shifted by the tap.  x sits in LDS as [part][position] rows of 16 channels and is
// read with the transposing LDS read; dy sits in operand order.  Eight waves: wave v owns NTW of the TW NTW taps and every
// WK-th k-step of 32 positions (TW WK = 8), and the WK sums of a tap are added in a fixed order.  Units are double-buffered
// in LDS with their loads one unit ahead in registers; half of the waves split and write the next unit before they multiply,
// the other half after, so that the matrix units have work meanwhile.
#include "conv1d_split_f32.h"

namespace conv1d {
namespace {
using namespace sp;

constexpr int kThreads = 512;
// 16-byte slots of dy and x a thread stages per unit, and register sets
constexpr int kDyTasks = 2, kXTasks = 3;
constexpr int num_sets(int fbw, int ntw) { return fbw * ntw <= 6 ? 2 : 1; }

struct SwfArgs {
    const float* x;
    const float* dy;
    float* ws;
    int C, K, W, Q, S, d, P;
    long x_sn, dy_sn;
    int qc_sh, upr, nunits, strips, tw_sh, tgroups, kgroups, cblocks, lx, vec;
};

template <int FBW, int NTW>
__global__ __launch_bounds__(kThreads, 2) void split_wgrad_pair_f32_kernel(SwfArgs a) {
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int QC = 1 << a.qc_sh, TW = 1 << a.tw_sh, WK = 8 >> a.tw_sh;
    const int tw = wave & (TW - 1), wk = wave >> a.tw_sh;
    const int ndy = FBW * QC * 2, nx = 2 * a.lx;   // 16-byte slots per part
    const int stage = 3 * (ndy + nx);

    int id = xcd_logical_id(blockIdx.x, gridDim.x);
    const int cb = id % a.cblocks;
    id /= a.cblocks;
    const int kg = id % a.kgroups;
    id /= a.kgroups;
    const int tg = id % a.tgroups, strip = id / a.tgroups;
    const int k0 = kg * 16 * FBW, c0 = cb * 16, s0 = tg * (NTW << a.tw_sh);
    const int u_begin = static_cast<int>(static_cast<long>(strip) * a.nunits / a.strips);
    const int u_end = static_cast<int>(static_cast<long>(strip + 1) * a.nunits / a.strips);

    constexpr int NSET = num_sets(FBW, NTW);
    struct Set {
        float dv[kDyTasks][8], xv[kXTasks][8];
    };
    Set sets[NSET];
    // byte offsets in a sample, which the plan keeps below 2^32: uniform base + 32-bit offset, one register per row
    unsigned xrow[8], dyrow[kDyTasks];
#pragma unroll
    for (int e = 0; e < 8; ++e) xrow[e] = 4u * static_cast<unsigned>(min(c0 + 8 * (tid & 1) + e, a.C - 1) * a.W);
#pragma unroll
    for (int k = 0; k < kDyTasks; ++k) {
        const int f = min(tid + k * kThreads, ndy - 1) >> (a.qc_sh + 1);
        dyrow[k] = 4u * static_cast<unsigned>(min(k0 + 16 * f + (tid & 15), a.K - 1) * a.Q);
    }
    auto request = [&](int u, Set& set) __attribute__((always_inline)) {
        auto& dv = set.dv;
        auto& xv = set.xv;
        const int n = u / a.upr, q0 = (u - n * a.upr) << a.qc_sh;
        const char* dyb = reinterpret_cast<const char*>(a.dy + n * a.dy_sn);
        const char* xb = reinterpret_cast<const char*>(a.x + n * a.x_sn);
#pragma unroll
        for (int k = 0; k < kDyTasks; ++k) {
            if (k * kThreads >= ndy) break;
            const int j = (min(tid + k * kThreads, ndy - 1) >> 4) & (QC / 8 - 1);
            const int q = q0 + 32 * (j >> 2) + 4 * (j & 3);
            if (a.vec) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(dyb + (dyrow[k] + 4u * min(q + 16 * h, a.Q - 4)));
#pragma unroll
                    for (int e = 0; e < 4; ++e) dv[k][4 * h + e] = v[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    dv[k][e] = *reinterpret_cast<const float*>(dyb + (dyrow[k] + 4u * min(q + 16 * (e >> 2) + (e & 3), a.Q - 1)));
            }
        }
        const int col0 = q0 + s0 * a.d - a.P;
#pragma unroll
        for (int k = 0; k < kXTasks; ++k) {
            if (k * kThreads >= nx) break;
            const unsigned col = 4u * clampi(col0 + min((tid + k * kThreads) >> 1, a.lx - 1), 0, a.W - 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) xv[k][e] = *reinterpret_cast<const float*>(xb + (xrow[e] + col));
        }
    };
    auto park = [&](int u, u32x4* b, Set& set) __attribute__((always_inline)) {
        auto& dv = set.dv;
        auto& xv = set.xv;
        const int n = u / a.upr, q0 = (u - n * a.upr) << a.qc_sh;
        // The matrix instruction cuts sums off towards minus infinity, which adds up over millions of terms: every other
        // unit of the layer is multiplied with -dy and subtracted, so that the offsets cancel, within a strip or, where
        // strips have a unit or two, between them.  (Counted from the strip's first unit they did not cancel in strips of
        // one: C = K = 15, S = 7, 66000 columns of 80 % zeros 3.6e-7 of the gradient, FP32 instruction 1.8e-7.)
        const unsigned sign = (u & 1) ? 0x80000000u : 0u;
#pragma unroll
        for (int k = 0; k < kDyTasks; ++k) {
            const int i = tid + k * kThreads;
            if (i < ndy) {
                const int j = (i >> 4) & (QC / 8 - 1), f = i >> (a.qc_sh + 1);
                const int left = k0 + 16 * f + (i & 15) < a.K ? a.Q - (q0 + 32 * (j >> 2) + 4 * (j & 3)) : 0;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    dv[k][e] = 16 * (e >> 2) + (e & 3) >= left ? 0.f : __uint_as_float(__float_as_uint(dv[k][e]) ^ sign);
                const Split8 s = split8(dv[k]);
                b[i] = s.h;
                b[ndy + i] = s.m;
                b[2 * ndy + i] = s.l;
            }
        }
        u32x4* xs = b + 3 * ndy;
        const int col0 = q0 + s0 * a.d - a.P;
#pragma unroll
        for (int k = 0; k < kXTasks; ++k) {
            const int i = tid + k * kThreads;
            if (i < nx) {
                const int col = col0 + (i >> 1);
                const int cleft = (col >= 0 && col < a.W) ? a.C - c0 - 8 * (i & 1) : 0;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e >= cleft) xv[k][e] = 0.f;
                const Split8 s = split8(xv[k]);
                xs[i] = s.h;
                xs[nx + i] = s.m;
                xs[2 * nx + i] = s.l;
            }
        }
    };

    f32x4 acc[NTW][FBW];
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int f = 0; f < FBW; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};

    // unit u, the PAR-th of the strip modulo 2
    auto unit = [&](int u, auto par) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        const u32x4* cur = lds + PAR * stage;
        auto refill = [&] {
            Set& set = sets[(PAR + 1) % NSET];
            if (u + 1 < u_end) park(u + 1, lds + (1 - PAR) * stage, set);
            if (u + 1 + NSET < u_end) request(u + 1 + NSET, set);
        };
        if (wave & 4) refill();
        const u32x4* dys = cur + g * 16 + l16;
        // rows of 16 channels are 4 transposing reads wide: this lane's piece of rows 4 g .. 4 g + 3
        const int xs0 = 2 * (PAR * stage + 3 * ndy) + (4 * g + (l16 >> 2)) * 4 + (l16 & 3) + tw * NTW * a.d * 4;
        for (int ks = wk; ks < QC / 32; ks += WK) {
            u32x4 y[FBW][3];
#pragma unroll
            for (int f = 0; f < FBW; ++f)
#pragma unroll
                for (int i = 0; i < 3; ++i) y[f][i] = dys[i * ndy + f * (QC * 2) + ks * 64];
            // the reads of the next tap are issued in front of the products of this one, and no earlier (left to itself the
            // compiler reads further ahead and spills)
            u32x4 b[2][3];
            int at = xs0 + 128 * ks;
            auto read = [&](int t) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const u32x2* p = reinterpret_cast<const u32x2*>(lds) + at + i * 2 * nx;
                    const u32x2 lo = read_tr(p), hi = read_tr(p + 64);
                    b[t & 1][i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                }
                at += 4 * a.d;
                opaque(at);  // one running index, not one register per tap and part
            };
            read(0);
#pragma unroll
            for (int t = 0; t < NTW; ++t) {
                if (t + 1 < NTW) read(t + 1);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 part[FBW];
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int f = 0; f < FBW; ++f)
                        part[f] = mfma(y[f][kPartB[k]], b[t & 1][kPartA[k]], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : part[f]);
#pragma unroll
                for (int f = 0; f < FBW; ++f) acc[t][f] = PAR ? acc[t][f] - part[f] : acc[t][f] + part[f];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!(wave & 4)) refill();
        __syncthreads();
    };
    if (u_begin < u_end) {
        request(u_begin, sets[0]);
        if (NSET == 2 && u_begin + 1 < u_end) request(u_begin + 1, sets[NSET - 1]);
        park(u_begin, lds, sets[0]);
        if (u_begin + NSET < u_end) request(u_begin + NSET, sets[0]);
    }
    __syncthreads();
    for (int u = u_begin; u < u_end; u += 2) {
        unit(u, std::integral_constant<int, 0>{});
        if (u + 1 < u_end) unit(u + 1, std::integral_constant<int, 1>{});
    }

    // the k-step shares of a tap, left to right
    f32x4* red = reinterpret_cast<f32x4*>(lds);
    for (int r = 1; r < WK; ++r) {
        if (wk == r)
#pragma unroll
            for (int i = 0; i < NTW; ++i)
#pragma unroll
                for (int f = 0; f < FBW; ++f) red[((tw * NTW + i) * FBW + f) * 64 + lane] = acc[i][f];
        __syncthreads();
        if (wk == 0)
#pragma unroll
            for (int i = 0; i < NTW; ++i)
#pragma unroll
                for (int f = 0; f < FBW; ++f) acc[i][f] += red[((tw * NTW + i) * FBW + f) * 64 + lane];
        __syncthreads();
    }
    if (wk != 0) return;
    const float turn = (u_begin & 1) ? -1.f : 1.f;  // such a strip added up its units with the opposite sign
#pragma unroll
    for (int f = 0; f < FBW; ++f) {
        const int kb = kg * FBW + f;
        if (16 * kb >= a.K) continue;
        float* ws = a.ws + (static_cast<long>(kb * a.cblocks + cb) * a.strips + strip) * a.S * 256;
#pragma unroll
        for (int i = 0; i < NTW; ++i) {
            const int s = s0 + tw * NTW + i;
            if (s < a.S)
#pragma unroll
                for (int j = 0; j < 4; ++j) ws[s * 256 + (4 * g + j) * 16 + l16] = turn * acc[i][f][j];
        }
    }
}

struct Plan {
    bool ok;
    int fbw, ntw, grid;
    SwfArgs a;
    size_t lds;
};

// Filter blocks and taps of a wave.  Shapes of one block are priced, not run: where one of them would be the fastest, the
// kernel that has waves for each is faster still (see taken_plan).
constexpr int kShapes[][2] = {{1, 3}, {1, 5}, {1, 7}, {1, 9}, {1, 13}, {2, 2}, {2, 3}, {2, 5}, {2, 7}, {2, 9}, {4, 2}, {4, 3}};

// the other kernel loads dy by four elements of a sample
bool few_outputs(const WgradProblem& p) { return static_cast<long>(p.K) * p.Q < 4; }

Plan make_plan(const WgradProblem& p) {
    Plan best{};
    if (p.bf16 || p.dw_sc != p.S || static_cast<long>(p.N) * p.Q < kMinTerms) return best;
    const size_t wsb = smallc_wgrad_f32_blocks_workspace(p);  // the partial tiles take no more than that kernel's
    if (wsb == 0) return best;
    const int cblocks = cdiv(p.C, 16), kblocks = cdiv(p.K, 16);
    const long most = static_cast<long>(wsb / (static_cast<size_t>(cblocks) * kblocks * p.S * 1024));
    double best_cost = 0;
    constexpr int kUnitSizes = 5;  // units of 32 << i positions
    struct {
        int upr;
        long nunits, strips;
        double longest;  // units of the longest strip
    } cut[kUnitSizes];
    for (int i = 0; i < kUnitSizes; ++i) {
        auto& c = cut[i];
        c.upr = cdiv(p.Q, 32 << i);
        c.nunits = static_cast<long>(p.N) * c.upr;
        c.strips = most < c.nunits ? most : c.nunits;
        c.longest = c.strips < 1 ? 0.0 : static_cast<double>((c.nunits + c.strips - 1) / c.strips);
    }
    for (const auto& sh : kShapes) {
        const int fbw = sh[0], ntw = sh[1];
        if (few_outputs(p) ? fbw != 2 : fbw > 1 && ntw > 2 && fbw / 2 >= kblocks) continue;  // half the filter blocks would do: such a shape loses anyway
        const int kgroups = cdiv(kblocks, fbw);
        for (int tw_sh = 0; tw_sh <= 3; ++tw_sh) {
            const int taps = ntw << tw_sh, tgroups = cdiv(p.S, taps), WK = 8 >> tw_sh;
            const long per_strip = static_cast<long>(cblocks) * kgroups * tgroups;
            for (int i = 3 - tw_sh; i < kUnitSizes; ++i) {  // a k-step at least for every wave of a tap
                const int qc_sh = 5 + i, QC = 1 << qc_sh;
                const auto& c = cut[i];
                const long lx = QC + static_cast<long>(taps - 1) * p.d;
                const long ndy = static_cast<long>(fbw) * QC * 2;
                const size_t stage = static_cast<size_t>(3 * (ndy + 2 * lx)) * 16;
                const size_t red = WK > 1 ? static_cast<size_t>(taps) * fbw * 1024 : 0;
                const size_t lds = red > 2 * stage ? red : 2 * stage;
                if (ndy > kDyTasks * kThreads || 2 * lx > kXTasks * kThreads || lds > kLdsAll) continue;
                if (c.nunits > 0x3fffffffL || c.strips < 1 || c.strips * per_strip > (1 << 20)) continue;
                // cycles of a unit on one SIMD's two waves: matrix instructions, LDS reads of all eight, splitting
                const double steps = QC / 32 >> (3 - tw_sh);
                const double mm = 2 * steps * ntw * fbw * 96;
                const double rd = 8 * steps * (3.0 * fbw + 3.0 * ntw) * 8;
                const double staging = 1500 + (cdiv(ndy, kThreads) + cdiv(2 * lx, kThreads)) * 2 * 300.0;
                const double unit = (mm > rd ? mm : rd) + 0.5 * staging;
                const double waves = static_cast<double>((c.strips * per_strip + 255) / 256);
                const double cost = waves * (unit * c.longest + 10000 + WK * taps * fbw * 16.0);
                if (best.ok && cost >= best_cost) continue;
                best_cost = cost;
                best.ok = true;
                best.fbw = fbw;
                best.ntw = ntw;
                best.lds = lds;
                best.grid = static_cast<int>(c.strips * per_strip);
                SwfArgs& a = best.a;
                a.qc_sh = qc_sh; a.upr = c.upr; a.nunits = static_cast<int>(c.nunits); a.strips = static_cast<int>(c.strips);
                a.tw_sh = tw_sh; a.tgroups = tgroups; a.kgroups = kgroups; a.lx = static_cast<int>(lx);
            }
        }
    }
    if (!best.ok) return best;
    SwfArgs& a = best.a;
    a.x = static_cast<const float*>(p.x);
    a.dy = static_cast<const float*>(p.dy);
    a.ws = static_cast<float*>(p.ws);
    a.C = p.C; a.K = p.K; a.W = p.W; a.Q = p.Q; a.S = p.S; a.d = p.d; a.P = p.P;
    a.x_sn = p.x_sn; a.dy_sn = p.dy_sn;
    a.cblocks = cblocks;
    a.vec = p.Q % 4 == 0 && p.dy_sn % 4 == 0 && (reinterpret_cast<uintptr_t>(p.dy) & 15) == 0;
    return best;
}

template <int FBW, int NTW>
hipError_t run(const Plan& pl, hipStream_t st) {
    auto kern = split_wgrad_pair_f32_kernel<FBW, NTW>;
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), pl.lds);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3(pl.grid), dim3(kThreads), pl.lds, st, pl.a);
}

// Layers of 129 to 255 pairs of blocks, one workgroup of which would leave up to half of the CUs idle, and of many pairs with
// a halo of 600 positions and more, over 60 layers drawn from 4 ... 256 channels and 5 ... 51 taps (fewer taps: N = 1, C = K =
// 200, W = 2000, S = 3 22 us here, 17 in the other kernel).  Not where one block per workgroup is the best that can be done
// here, one in thirty of them: x is split for that block alone then, and over 19 such layers the other kernel takes 0.47 to
// 0.97 of the time (N = 5, C = K = 198, W = 6153, S = 49, d = 3 890 and 741 us; N = 1, C = K = 238, W = 232, S = 17, d = 4 29
// and 14), in one 1.04 (N = 48, C = 210, K = 208, W = 2788, S = 39, d = 16 3170 and 3300), with smaller errors in all.
// And samples of one to three outputs, of whose dy the other kernel cannot load four elements (N = 56, C = 256, K = 1,
// W = 303, S = 51, d = 6 26 us, on FP32 products 93; N = 16, C = 4, K = 1, W = 9, S = 8 9 and 13).
Plan taken_plan(const WgradProblem& p) {
    const long pairs = static_cast<long>(cdiv(p.C, 16)) * cdiv(p.K, 16);
    const bool idle = pairs > 128 && pairs < 256 && p.S >= 5;
    const bool halo = (p.S - 1L) * p.d >= 600 && pairs >= 48;
    if (!idle && !halo && !few_outputs(p)) return Plan{};
    Plan pl = make_plan(p);
    pl.ok = pl.ok && pl.fbw > 1;
    return pl;
}

double plan_roundings(const Plan& pl) {
    if (!pl.ok) return 0.0;
    const int WK = 8 >> pl.a.tw_sh;
    return chain_roundings(static_cast<long>((1 << pl.a.qc_sh) / 32 / WK) * cdiv(pl.a.nunits, pl.a.strips)) + chain_roundings(WK);
}

}  // namespace

double split_f32_wgrad_pair_roundings(const WgradProblem& p) { return plan_roundings(make_plan(p)); }

bool split_f32_wgrad_pair_tile(const WgradProblem& p, SplitTile* t) {
    const Plan pl = taken_plan(p);
    if (pl.ok) *t = SplitTile{pl.fbw, pl.ntw, cdiv(pl.a.nunits, pl.a.strips), pl.grid, plan_roundings(pl), 0};
    return pl.ok;
}

hipError_t split_f32_wgrad_pair_launch(const WgradProblem& p, hipStream_t st, bool* taken) {
    const Plan pl = taken_plan(p);
    *taken = pl.ok;
    if (!pl.ok) return hipSuccess;
    hipError_t e;
    switch (pl.fbw * 16 + pl.ntw) {
        case 32 + 2: e = run<2, 2>(pl, st); break;
        case 32 + 3: e = run<2, 3>(pl, st); break;
        case 32 + 5: e = run<2, 5>(pl, st); break;
        case 32 + 7: e = run<2, 7>(pl, st); break;
        case 32 + 9: e = run<2, 9>(pl, st); break;
        case 64 + 3: e = run<4, 3>(pl, st); break;
        case 64 + 2: e = run<4, 2>(pl, st); break;
        default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    return smallc_wgrad_reduce_launch(pl.a.ws, p.dw, p.K, p.C, p.S, p.dw_sk, p.dw_sc, pl.a.strips, st);
}

}  // namespace conv1d
