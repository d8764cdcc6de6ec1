// FP32 forward / backward-data on the bf16 matrix instructions.
//
// v_mfma_f32_16x16x4_f32 does 1/16 of the operations per cycle that v_mfma_f32_16x16x32_bf16 does, and the FP32 passes
// were bound by it.  Here each float is the sum of three bfloat16 numbers (conv1d_split_f32.h) and a product is the six
// largest of their nine products, exact in the matrix unit and added in FP32: 6/16 of the FP32 matrix time.  The
// products left out are at most 2^-24 of the whole, half a unit in the last place of an FP32 product.  The sum of the six
// over 32 terms is added to the running sums in FP32, so a sum of n terms is rounded n/32 times at full size where the
// FP32 instruction rounded it n/4 times.
//
// One workgroup: 16 FBW filters x 64 PB output columns of one sample, wave v the columns 16 PB v ..  A step is one
// matrix instruction deep (32 = 4 lane groups x 8 channels): PL planes of 8 channels times 4/PL taps.  The input
// window of PL planes sits in LDS as [part][plane][position] slots of 8 channels, so any dilation is a slot offset; the
// weights of one step are gathered from (K, C, S), split and written to LDS one step ahead, double-buffered, one
// barrier per step.  Workgroups are kept to half the LDS and 256 registers: two share a CU, and one multiplies while
// the other stages.
#include "conv1d_split_f32.h"

namespace conv1d {
namespace {
using namespace sp;

constexpr int kThreads = 256;
constexpr size_t kLdsHalf = 80 * 1024, kLdsAll = 160 * 1024;

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
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g = lane >> 4;
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

    // the weight entry of this thread: filter em, lane group g's plane and tap of the step
    const int em = m0 + (tid >> 6) * 16 + l16;
    const bool has_entry = tid < FBW * 64;
    const float* wrow = a.wt + min(em, a.M - 1) * a.w_sm + a.w_s0;
    const int eplane = g & (PL - 1), etap = g >> a.pl_sh;
    float wv[8];
    int cleft = 0;
    auto request = [&](int stage, int step) {
        if (!has_entry) return;
        const int tap = step * TP + etap, c = 8 * (stage * PL + eplane);
        const float* p = wrow + static_cast<long>(min(tap, a.S - 1)) * a.w_ss;
        cleft = (em < a.M && tap < a.S) ? a.R - c : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) wv[j] = p[min(c + j, a.R - 1) * a.w_sr];
    };
    // channels, taps and filters the layer does not have count as zero; put right here, so that nothing waits for the
    // loads before the products of a step are done
    auto park = [&](int buf) {
        if (!has_entry) return;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j >= cleft) wv[j] = 0.f;
        const Split8 s = split8(wv);
        u32x4* e = ws + (buf * FBW + (tid >> 6)) * 192 + lane;
        e[0] = s.h;
        e[64] = s.m;
        e[128] = s.l;
    };

    f32x4 acc[PB][FBW];
#pragma unroll
    for (int t = 0; t < PB; ++t)
#pragma unroll
        for (int f = 0; f < FBW; ++f) acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};

    request(0, 0);
    int buf = 0;
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
        if (stage == 0) park(0);
        __syncthreads();
        int rd = rd0;
        for (int step = 0; step < a.nsteps; ++step, rd += TP * a.d) {
            const bool more = step + 1 < a.nsteps || stage + 1 < a.nstages;
            if (more) request(step + 1 < a.nsteps ? stage : stage + 1, step + 1 < a.nsteps ? step + 1 : 0);
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
                        for (int f = 0; f < FBW; ++f) acc[t0 + u][f] += sum[u][f];
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
            if (more) park(buf);
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

struct Plan {
    bool ok;
    int fbw, pb;
    SpArgs a;
    size_t lds;
    long grid;
};

// Planes per step (1 << result), which decides the order of an output's sum: from what a sample is, not from how many there
// are, so that a sample's result does not depend on its batch.  The least of matrix time plus what steps and windows cost
// beside it over the tiles; workgroups that share a CU hide half of the latter.  -1: no tile fits.
int planes_shift(const CorrProblem& p) {
    int best = -1;
    double best_cost = 0;
    for (int fbw = 1; fbw <= 4; ++fbw) {
        for (int pb = 4; pb <= 8; ++pb) {
            if (pb == 7 || fbw * pb > 20) continue;
            const double tiles = static_cast<double>(cdiv(p.Wout, 64 * pb)) * cdiv(cdiv(p.M, 16), fbw);
            for (int sh = 0; sh <= 2; ++sh) {
                const int tp = 4 >> sh, nsteps = cdiv(p.S, tp), nstages = cdiv(p.R, 8 << sh);
                const long wlen = 64L * pb + (static_cast<long>(nsteps) * tp - 1) * p.d;
                const size_t lds = (static_cast<size_t>(wlen) * 3 * (1 << sh) + 2 * fbw * 192) * 16;
                if (wlen > 16384 || lds > kLdsAll) continue;
                const double beside = nsteps * 600.0 + 1000.0 + (wlen << sh) * 2.0;
                const double cost = tiles * nstages * (nsteps * 96.0 * fbw * pb + (lds <= kLdsHalf ? 0.5 : 1.0) * beside);
                if (best >= 0 && cost >= best_cost) continue;
                best_cost = cost;
                best = sh;
            }
        }
    }
    return best;
}

Plan make_plan(const CorrProblem& p) {
    Plan best{};
    if (p.bf16 || p.accumulate || p.epi.out_bf16 || p.tail.ws || static_cast<long>(p.R) * p.S < kMinTerms) return best;
    const int sh = planes_shift(p);
    if (sh < 0) return best;
    const int mb = cdiv(p.M, 16);
    double best_cost = 0;
    for (int fbw = 1; fbw <= 4; ++fbw) {
        for (int pb = 4; pb <= 8; ++pb) {
            if (pb == 7 || fbw * pb > 20) continue;  // sums, weights and inputs within 256 registers
            const int qtiles = cdiv(p.Wout, 64 * pb), fgroups = cdiv(mb, fbw);
            const long grid = static_cast<long>(p.N) * qtiles * fgroups;
            if (grid > 0x7fffffffL / kThreads) continue;
            const int tp = 4 >> sh, nsteps = cdiv(p.S, tp), nstages = cdiv(p.R, 8 << sh);
            const long wlen = 64L * pb + (static_cast<long>(nsteps) * tp - 1) * p.d;
            const size_t lds = (static_cast<size_t>(wlen) * 3 * (1 << sh) + 2 * fbw * 192) * 16;
            if (wlen > 16384 || lds > kLdsAll) continue;
            // cycles of the busiest CU: matrix time of its workgroups, plus what a step and a window cost beside it;
            // a workgroup alone on its CU hides none of that
            const double staging = nsteps * 400.0 + 3000.0 + (wlen << sh) * 6.0;
            const double mm = static_cast<double>(nsteps) * fbw * pb * 96;
            const long per_cu = (grid + 255) / 256;
            const bool shared = lds <= kLdsHalf && per_cu > 1;
            const double lds_reads = static_cast<double>(nsteps) * (3 * pb + 3 * fbw) * 4 * 8;
            const double busy = mm > lds_reads ? mm : lds_reads;
            const double cost = nstages * per_cu * (busy + (shared ? 0.3 : 1.0) * staging);
            if (best.ok && cost >= best_cost) continue;
            best_cost = cost;
            best.ok = true;
            best.fbw = fbw;
            best.pb = pb;
            best.lds = lds;
            best.grid = grid;
            SpArgs& a = best.a;
            a.in = static_cast<const float*>(p.in);
            a.wt = static_cast<const float*>(p.wt);
            a.out = p.out;
            a.epi = p.epi;
            a.R = p.R; a.M = p.M; a.Win = p.Win; a.Wout = p.Wout; a.S = p.S; a.d = p.d; a.P = p.P;
            a.w_sm = p.w_sm; a.w_sr = p.w_sr; a.in_sn = p.in_sn; a.out_sn = p.out_sn;
            a.w_s0 = p.w_s0; a.w_ss = p.w_ss;
            a.pl_sh = sh; a.nstages = nstages; a.nsteps = nsteps; a.wlen = static_cast<int>(wlen);
            a.qtiles = qtiles; a.fgroups = fgroups;
            a.vec = p.Wout % 4 == 0 && p.out_sn % 4 == 0 && (reinterpret_cast<uintptr_t>(p.out) & 15) == 0;
        }
    }
    return best;
}

template <int FBW, int PB>
hipError_t run(const Plan& pl, hipStream_t st) {
    auto kern = split_corr_f32_kernel<FBW, PB>;
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), pl.lds);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3(static_cast<unsigned>(pl.grid)), dim3(kThreads), pl.lds, st, pl.a);
}

template <int FBW>
hipError_t run_pb(const Plan& pl, hipStream_t st) {
    switch (pl.pb) {
        case 4: return run<FBW, 4>(pl, st);
        case 5: return run<FBW, 5>(pl, st);
        case 6:
            if constexpr (FBW <= 3) return run<FBW, 6>(pl, st);
            break;
        case 8:
            if constexpr (FBW <= 2) return run<FBW, 8>(pl, st);
            break;
        default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool split_f32_corr_supported(const CorrProblem& p) { return make_plan(p).ok; }

hipError_t split_f32_corr_launch(const CorrProblem& p, hipStream_t st) {
    const Plan pl = make_plan(p);
    if (!pl.ok) return hipErrorInvalidValue;
    switch (pl.fbw) {
        case 1: return run_pb<1>(pl, st);
        case 2: return run_pb<2>(pl, st);
        case 3: return run_pb<3>(pl, st);
        default: return run_pb<4>(pl, st);
    }
}

}  // namespace conv1d
