// FP32 forward / backward-data on the bf16 matrix instructions.
//
// v_mfma_f32_16x16x4_f32 does 1/16 of the operations per cycle that v_mfma_f32_16x16x32_bf16 does, and the FP32 passes
// were bound by it.  Here each float is the sum of three bfloat16 numbers (conv1d_split_f32.h) and a product is the six
// largest of their nine products, exact in the matrix unit and added in FP32: 6/16 of the FP32 matrix time.  The
// products left out are at most 2^-24 of the whole, half a unit in the last place of an FP32 product.  The sum of the six
// over 32 terms is added to the running sums in FP32, so a sum of n terms is rounded n/32 times at full size where the
// FP32 instruction rounded it n/4 times.
// One pass, N = 8, C = K = 64, W = 20000, FP32 instruction and three parts: S = 5, d = 1 116 and 52 us, S = 33, d = 4 447 and
// 222 us, S = 51, d = 8 658 and 297 us (225 TFLOP/s, 54 % of the rate of six bf16 products).
//
// One workgroup: 16 FBW filters x 64 PB output columns of one sample, wave v the columns 16 PB v ..  A step is one
// matrix instruction deep (32 = 4 lane groups x 8 channels): PL planes of 8 channels times 4/PL taps.  The input
// window of PL planes sits in LDS as [part][plane][position] slots of 8 channels, so any dilation is a slot offset; the
// weights of one step are gathered from (K, C, S), split and written to LDS one step ahead, double-buffered, one
// barrier per step; the waves take turns at that.  Workgroups that share a CU multiply while others stage.
#include "conv1d_split_f32.h"

namespace conv1d {
namespace {
using namespace sp;

constexpr int kThreads = 256;

struct SpArgs {
    const float* in;
    const float* wt;
    float* out;
    Epilogue epi;
    int R, M, Win, Wout, S, d, P;
    long w_sm, w_sr, in_sn, out_sn;
    int w_s0, w_ss;
    int pl_sh, nstages, nsteps, wlen, qtiles, fgroups, vec;
};

template <int FBW, int PB>
__global__ __launch_bounds__(kThreads, 2) void split_corr_f32_kernel(SpArgs a) {
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int PL = 1 << a.pl_sh, TP = 4 >> a.pl_sh;
    const int part = PL * a.wlen;
    u32x4* xs = lds;
    u32x4* ws = lds + 3 * part;  // [2][FBW][3][64]

    int id = xcd_logical_id(blockIdx.x, gridDim.x);
    const int fg = id % a.fgroups;
    id /= a.fgroups;
    const int qt = id % a.qtiles, n = id / a.qtiles;
    const int q0 = qt * (64 * PB), m0 = fg * (16 * FBW);
    const float* inb = a.in + n * a.in_sn;

    // Weight entries: FBW waves hold one step's, the other waves those of the steps after it (NG groups of waves in turn),
    // so that a group's loads have NG steps to arrive.  With all of them one step ahead a step of a workgroup alone on its
    // CU took as long as the loads, about 1 us (C = K = 64, S = 33, d = 4, up to 16000 columns: 68 us a pass).
    constexpr int NG = 4 / FBW;
    const bool has_entry = wave < NG * FBW;
    const int ef = wave % FBW, em = m0 + ef * 16 + l16;  // filter of this thread's entry; lane group g has plane and tap
    // byte offsets in the weights, which the plan keeps below 2^32
    const unsigned wrow = 4u * static_cast<unsigned>(min(em, a.M - 1) * a.w_sm + a.w_s0);
    const unsigned wchan = 4u * static_cast<unsigned>(a.w_sr), wlast = static_cast<unsigned>(a.R - 1) * wchan;
    const int eplane = g & (PL - 1), etap = g >> a.pl_sh;
    const int total = a.nstages * a.nsteps;
    int due = wave / FBW;  // step, counted over all stages, of the entry in wv
    int wstage = 0, wstep = due;
    float wv[8];
    int cleft = 0;
    auto request = [&] {
        if (!has_entry || due >= total) return;
        while (wstep >= a.nsteps) {
            wstep -= a.nsteps;
            ++wstage;
        }
        const int tap = wstep * TP + etap, c = 8 * (wstage * PL + eplane);
        const unsigned row = wrow + 4u * static_cast<unsigned>(min(tap, a.S - 1) * a.w_ss);
        cleft = (em < a.M && tap < a.S) ? a.R - c : 0;
        unsigned at = static_cast<unsigned>(c) * wchan;
#pragma unroll
        for (int j = 0; j < 8; ++j, at += wchan)
            wv[j] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.wt) + (row + min(at, wlast)));
    };
    // entry of the given step, if this wave has it.  Channels, taps and filters the layer does not have count as zero; put
    // right here, so that nothing waits for the loads before the products of a step are done
    auto park = [&](int step, int buf) {
        if (!has_entry || due != step || step >= total) return;
        // The matrix instruction cuts sums off towards minus infinity: every other step is multiplied with -w and
        // subtracted, so that the offsets cancel (C = 24, S = 7, 6 steps: mean error of the outputs over their norm
        // -1.6e-8 without).
        const unsigned sign = (step & 1) ? 0x80000000u : 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) wv[j] = j >= cleft ? 0.f : __uint_as_float(__float_as_uint(wv[j]) ^ sign);
        const Split8 s = split8(wv);
        u32x4* e = ws + (buf * FBW + ef) * 192 + lane;
        e[0] = s.h;
        e[64] = s.m;
        e[128] = s.l;
        due += NG;
        wstep += NG;
        request();
    };

    f32x4 acc[PB][FBW];
#pragma unroll
    for (int t = 0; t < PB; ++t)
#pragma unroll
        for (int f = 0; f < FBW; ++f) acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};

    request();
    int buf = 0, next = 1;  // step after the current one, counted over all stages
    const int rd0 = (g & (PL - 1)) * a.wlen + (g >> a.pl_sh) * a.d + wave * (16 * PB) + l16;
    for (int stage = 0; stage < a.nstages; ++stage) {
        const int col0 = q0 - a.P;
        // four slots per thread in flight
        for (int i0 = tid; i0 < part; i0 += 4 * kThreads) {
            float v[4][8];
            int cl[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + k * kThreads, part - 1);
                const int plane = (i >= a.wlen) + (i >= 2 * a.wlen) + (i >= 3 * a.wlen);
                const int c = 8 * (stage * PL + plane), col = col0 + i - plane * a.wlen;
                const float* p = inb + clampi(col, 0, a.Win - 1);
                cl[k] = (col >= 0 && col < a.Win) ? a.R - c : 0;
#pragma unroll
                for (int j = 0; j < 8; ++j) v[k][j] = p[static_cast<long>(min(c + j, a.R - 1)) * a.Win];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 + k * kThreads;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j >= cl[k]) v[k][j] = 0.f;
                const Split8 s = split8(v[k]);
                if (i < part) {
                    xs[i] = s.h;
                    xs[part + i] = s.m;
                    xs[2 * part + i] = s.l;
                }
            }
        }
        if (stage == 0) park(0, 0);
        __syncthreads();
        int rd = rd0;
        for (int step = 0; step < a.nsteps; ++step, ++next, rd += TP * a.d) {
            const float turn = (next & 1) ? 1.f : -1.f;  // odd steps have -w
            u32x4 w[FBW][3];
#pragma unroll
            for (int f = 0; f < FBW; ++f)
#pragma unroll
                for (int i = 0; i < 3; ++i) w[f][i] = ws[(buf * FBW + f) * 192 + i * 64 + lane];
            constexpr int U = FBW >= 3 ? 1 : 2;  // column blocks in turn: no product waits for the one before
            // the reads of the next blocks in front of the products of these, and no earlier (registers)
            u32x4 xr[2][U][3];
            auto read = [&](int t0) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (t0 + u < PB)
#pragma unroll
                        for (int i = 0; i < 3; ++i) xr[(t0 / U) & 1][u][i] = xs[i * part + rd + 16 * (t0 + u)];
            };
            read(0);
            if constexpr (NG > 1) park(next, buf ^ 1);  // under the latency of the reads; with one group the loads are not here yet
#pragma unroll
            for (int t0 = 0; t0 < PB; t0 += U) {
                if (t0 + U < PB) read(t0 + U);
                __builtin_amdgcn_sched_barrier(0);
                const auto& x = xr[(t0 / U) & 1];
                f32x4 sum[U][FBW];
#pragma unroll
                for (int k = 0; k < 6; ++k)
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (t0 + u < PB)
#pragma unroll
                            for (int f = 0; f < FBW; ++f)
                                sum[u][f] = mfma(x[u][kPartA[k]], w[f][kPartB[k]], k == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[u][f]);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (t0 + u < PB)
#pragma unroll
                        for (int f = 0; f < FBW; ++f)
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[t0 + u][f][i] = __builtin_fmaf(turn, sum[u][f][i], acc[t0 + u][f][i]);
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
            if constexpr (NG == 1) park(next, buf);
            __syncthreads();
        }
    }

    float* out = a.out;
    const long ob = n * a.out_sn;
#pragma unroll
    for (int f = 0; f < FBW; ++f) {
        const int m = m0 + 16 * f + l16;
        if (m >= a.M) continue;
        const float bias = epi_bias(a.epi, m);
        const long row = ob + static_cast<long>(m) * a.Wout;
#pragma unroll
        for (int t = 0; t < PB; ++t) {
            const int q = q0 + (wave * PB + t) * 16 + 4 * g;
            const f32x4 v = epi_apply4(a.epi, acc[t][f], bias);
            if (a.vec) {
                if (q < a.Wout) *reinterpret_cast<f32x4*>(out + row + q) = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (q + i < a.Wout) out[row + q + i] = v[i];
            }
        }
    }
}

struct Tile {
    int fbw, pb;
};
// sums, weights and inputs within 256 registers
constexpr Tile kTiles[] = {{1, 1}, {1, 2}, {1, 4}, {1, 5}, {1, 6}, {1, 8}, {2, 4}, {2, 5}, {2, 6}, {2, 8}, {3, 4}, {3, 5}, {3, 6}, {4, 4}, {4, 5}};

struct Plan {
    bool ok;
    Tile tile;
    SpArgs a;
    size_t lds;
    long grid;
};

// A tile with 1 << sh planes per step on this layer, and its time as a model of cycles: `alone`, a workgroup with its CU
// to itself, which is a chain of reads, products and barriers; `busy`, what it takes of the pipes it shares with others,
// most of it the gather of weights, whose 64 lanes fall on 64 cache lines.  The constants are a fit to the forward times
// of these tiles on 22 layers (C, K 4 ... 256, 1 ... 51 taps) at 500 ... 2.4 million columns; tile and planes picked by it
// are within 21 % of the fastest everywhere, 2 % on average.  Small launches get narrow tiles: 64 columns take 36 us where
// 256 take 49 on 2000 columns of C = K = 64, S = 33, d = 4 (FP32 instruction 61 us).
struct Fit {
    bool ok;
    int nsteps, nstages, planes, by_regs;
    long columns, wlen, most_slots;  // columns of a window, slots of a plane of it, and how many 32-bit columns allow
    long per_sample;                 // workgroups of a sample
    size_t lds;
    double alone, busy;
    int resident(size_t bytes) const {
        const int by_lds = bytes > kLdsAll ? 0 : static_cast<int>(static_cast<unsigned>(kLdsAll) / static_cast<unsigned>(bytes));
        return by_lds < by_regs ? by_lds : by_regs;
    }
    double time(long grid, int resident) const {
        const long slots = 256L * resident, full = (grid - 1) / slots, last = (grid - full * slots + 255) / 256;
        const double whole = alone > resident * busy ? alone : resident * busy;
        return full * whole + (alone > last * busy ? alone : last * busy);
    }
    // The time of a launch, with planes rounded up to begin in the same bank (C = K = 48, S = 17, d = 3: 40.0 -> 38.8 us) where
    // that costs no time: where a CU has room for fewer workgroups so, if these suffice.  N = 43, C = K = 112, W = 600, S = 17,
    // d = 2 (three for four) 91 and 85 us, but C = 15, K = 5, N = 48, W = 24848, S = 5, d = 8 (five turns of three for four of
    // four) 29.5 and 31.9, and N = 19, C = K = 172, W = 1624, S = 5, d = 10 (one for two, or a smaller tile) 88 and 110.
    double settle(long grid) {
        const int bare = resident(lds);
        const double t = time(grid, bare);
        const long rounded = (columns + 15) & ~15L;
        if (planes == 1 || rounded == columns || rounded > most_slots) return t;
        const size_t bytes = lds + static_cast<size_t>(rounded - columns) * 48 * planes;
        const int now = resident(bytes);
        if (now < 1) return t;
        const double r = now < bare ? time(grid, now) : t;
        if (r > t || (r == t && now < bare && grid > 256L * now)) return t;
        wlen = rounded;
        lds = bytes;
        return r;
    }
};
Fit fit(const CorrProblem& p, Tile t, int sh) {
    Fit f{};
    const int tp = 4 >> sh;
    f.nsteps = cdiv(p.S, tp);
    f.nstages = cdiv(p.R, 8 << sh);
    f.columns = f.wlen = 64L * t.pb + (static_cast<long>(f.nsteps) * tp - 1) * p.d;
    f.lds = (static_cast<size_t>(f.wlen) * 3 * (1 << sh) + 2 * t.fbw * 192) * 16;
    if (f.wlen > 16384 || f.lds > kLdsAll) return f;
    const long columns = static_cast<long>(cdiv(p.Wout, 64 * t.pb)) * 64 * t.pb;  // the last tile may end behind the row
    f.most_slots = (1L << 31) - (columns - 64 * t.pb - p.P);
    if (columns > 1L << 31 || f.wlen > f.most_slots) return f;  // 32-bit columns in the kernel
    f.planes = 1 << sh;
    f.by_regs = 512 / (94 + 12 * t.fbw + 4 * t.fbw * t.pb);
    f.per_sample = static_cast<long>(cdiv(p.Wout, 64 * t.pb)) * cdiv(cdiv(p.M, 16), t.fbw);
    const double window = static_cast<double>(f.columns << sh);
    const double mm = 150.0 * t.fbw * t.pb, loads = 610.0 * t.fbw + 31.0 * (t.fbw + t.pb);
    f.alone = f.nstages * (f.nsteps * (240.0 + 350.0 * t.fbw + (22.0 + 100.0 * t.fbw) * t.pb + (t.fbw > 2 ? 1000.0 : 0.0)) + 6 * window);
    f.busy = f.nstages * (f.nsteps * (mm > loads ? mm : loads) + 3.6 * window);
    f.ok = true;
    return f;
}

// Planes per step (1 << result), which decides the order of an output's sum: from what a sample is, not from how many there
// are, so that a sample's result does not depend on its batch.  The least of matrix time plus what steps and windows cost
// beside it over the tiles of 256 columns and more; workgroups that share a CU hide half of the latter.  -1: none fits.
// Long rows of many filters and taps take one plane, four taps a step: the windows are short beside the steps then, and their
// workgroups share CUs three at a time.  W = 60000, one plane and two: C = K = 64, d = 1, S = 40 N = 1 115 and 115 us, N = 4 372
// and 385, S = 47 128 and 130, 424 and 441, S = 51 137 and 139, 456 and 499; C = K = 128, N = 4 S = 43 1520 and 1640, S = 51
// 1770 and 1910; d = 8 and 16 the same tiles either way, within 0.5 %; N = 2, C = K = 45, W = 55001, S = 43, d = 5 128 and 144.
// Shorter rows lose with one where the batch is small (N = 1, W = 20000, C = K = 64, S = 51: 83.7 and 81.5) and gain where it is
// not (N = 4: 172 and 178).  Not where four taps a step pad the taps by more than two do (S = 41, 42, 45, 46, 49, 50): the
// sums are longer by these zeros, 2 % more error (C = K = 64, S = 41 1.77e-7 and 1.73e-7), for between 2 % more and 8 % less
// time.
constexpr int kLongTaps = 40;
constexpr long kLongRows = 2400000;  // filters x columns of a sample

int planes_shift(const CorrProblem& p) {
    if (p.S >= kLongTaps && cdiv(p.S, 4) * 4 <= cdiv(p.S, 2) * 2 && static_cast<long>(p.M) * p.Wout >= kLongRows)
        for (const Tile t : kTiles)
            if (t.pb >= 4 && 16 * (t.fbw - 1) < p.M && fit(p, t, 0).ok) return 0;
    int best = -1;
    double best_cost = 0;
    for (const Tile t : kTiles) {
        if (t.pb < 4 || 16 * (t.fbw - 1) >= p.M) continue;  // (no more filter blocks than there are: those tiles lose anyway)
        for (int sh = 0; sh <= 2; ++sh) {
            const Fit f = fit(p, t, sh);
            if (!f.ok) continue;
            const double beside = f.nsteps * 600.0 + 1000.0 + (f.columns << sh) * 2.0;
            const double cost = f.per_sample * f.nstages * (f.nsteps * 96.0 * t.fbw * t.pb + (2 * f.lds <= kLdsAll ? 0.5 : 1.0) * beside);
            if (best >= 0 && cost >= best_cost) continue;
            best_cost = cost;
            best = sh;
        }
    }
    return best;
}

Plan make_plan(const CorrProblem& p) {
    Plan best{};
    if (p.bf16 || p.accumulate || p.epi.out_bf16 || p.tail.ws || static_cast<long>(p.R) * p.S < kMinTerms) return best;
    if (static_cast<long>(p.M) * p.R * p.S >= 1L << 30) return best;  // 32-bit byte offsets in the weights
    const int sh = planes_shift(p);
    if (sh < 0) return best;
    Fit bf{};
    double best_time = 0;
    for (const Tile t : kTiles) {
        if (16 * (t.fbw - 1) >= p.M) continue;
        Fit f = fit(p, t, sh);
        if (!f.ok) continue;
        const long grid = p.N * f.per_sample;
        if (grid > 0x7fffffffL / kThreads) continue;
        const double time = f.settle(grid);
        if (best.ok && time >= best_time) continue;
        best.ok = true;
        best_time = time;
        best.tile = t;
        best.grid = grid;
        best.a.pl_sh = sh;
        bf = f;
    }
    if (!best.ok) return best;
    best.lds = bf.lds;
    SpArgs& a = best.a;
    a.in = static_cast<const float*>(p.in);
    a.wt = static_cast<const float*>(p.wt);
    a.out = p.out;
    a.epi = p.epi;
    a.R = p.R; a.M = p.M; a.Win = p.Win; a.Wout = p.Wout; a.S = p.S; a.d = p.d; a.P = p.P;
    a.w_sm = p.w_sm; a.w_sr = p.w_sr; a.in_sn = p.in_sn; a.out_sn = p.out_sn;
    a.w_s0 = p.w_s0; a.w_ss = p.w_ss;
    a.nstages = bf.nstages; a.nsteps = bf.nsteps; a.wlen = static_cast<int>(bf.wlen);
    a.qtiles = cdiv(p.Wout, 64 * best.tile.pb);
    a.fgroups = cdiv(cdiv(p.M, 16), best.tile.fbw);
    a.vec = p.Wout % 4 == 0 && p.out_sn % 4 == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15) == 0;
    return best;
}

template <int FBW, int PB>
hipError_t run(const Plan& pl, hipStream_t st) {
    auto kern = split_corr_f32_kernel<FBW, PB>;
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), pl.lds);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3(static_cast<unsigned>(pl.grid)), dim3(kThreads), pl.lds, st, pl.a);
}

template <size_t... I>
hipError_t run_tile(const Plan& pl, hipStream_t st, std::index_sequence<I...>) {
    hipError_t e = hipErrorInvalidValue;
    (void)((pl.tile.fbw == kTiles[I].fbw && pl.tile.pb == kTiles[I].pb && (e = run<kTiles[I].fbw, kTiles[I].pb>(pl, st), true)) || ...);
    return e;
}

}  // namespace

bool split_f32_corr_supported(const CorrProblem& p) { return make_plan(p).ok; }

bool split_f32_corr_tile(const CorrProblem& p, SplitTile* t) {
    const Plan pl = make_plan(p);
    *t = SplitTile{pl.tile.fbw, pl.tile.pb, 1 << pl.a.pl_sh, pl.grid, 0.0, 0};
    return pl.ok;
}

hipError_t split_f32_corr_launch(const CorrProblem& p, hipStream_t st, bool* taken) {
    const Plan pl = make_plan(p);
    *taken = pl.ok;
    if (!pl.ok) return hipSuccess;
    return run_tile(pl, st, std::make_index_sequence<sizeof(kTiles) / sizeof(kTiles[0])>{});
}

}  // namespace conv1d
