// Backward of the fused epilogue (bias + ReLU) in front of the two backward passes:
//   dy[n][k][q] = gy[n][k][q] where the activation was positive, 0 elsewhere (gy * 0 or 1, so NaN and Inf stay visible)
//   dbias[k]    = sum over n, q of that, before it is rounded to dy's type.
// Bound by memory: gy read once, one bit per element, dy written once.  N = 56, K = 16, Q = 20000 in bfloat16: mask 9.4 us
// (3.9 TB/s), gradient 15.8 us (4.7 TB/s, what a large copy reaches), sum over the waves 2.8 us.  As separate elementwise
// passes and a reduction (compare 12, multiplication by a boolean tensor 51, cast to float 17, sum 29 us) every element
// crossed memory seven times.
#include "conv1d_internal.h"

namespace conv1d {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64, kThreads = 256;
constexpr int kInFlight = 4;         // groups of 8 elements a lane has in flight
constexpr long kChunk = 8 * kWave;   // groups of 8 elements per wave: 8 per lane, so that small batches fill the chip too

template <bool BF16>
__device__ __forceinline__ void load8(const void* p, long i, float (&v)[8]) {
    if constexpr (BF16) {
        const bf16x8 t = *reinterpret_cast<const bf16x8*>(static_cast<const unsigned short*>(p) + i);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = static_cast<float>(t[e]);
    } else {
        const f32x4 a = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p) + i);
        const f32x4 b = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p) + i + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = a[e];
            v[4 + e] = b[e];
        }
    }
}

// bit i & 7 of byte i >> 3: element i of y is positive
template <bool BF16>
__global__ __launch_bounds__(kThreads) void relu_mask_kernel(const void* y, unsigned char* positive, long n, int vec) {
    const long g0 = static_cast<long>(blockIdx.x) * (kThreads * kInFlight) + threadIdx.x;
    float v[kInFlight][8];
#pragma unroll
    for (int k = 0; k < kInFlight; ++k) {
        const long i = 8 * (g0 + k * kThreads);
        if (vec && i + 8 <= n) {
            load8<BF16>(y, i, v[k]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[k][e] = i + e < n ? load_elem<BF16>(y, i + e) : 0.f;
        }
    }
#pragma unroll
    for (int k = 0; k < kInFlight; ++k) {
        const long g = g0 + k * kThreads;
        unsigned bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) bits |= (v[k][e] > 0.f ? 1u : 0u) << e;
        if (8 * g < n) positive[g] = static_cast<unsigned char>(bits);
    }
}

struct GradArgs {
    const void* gy;
    const unsigned char* positive;  // nullptr: no ReLU
    void* dy;                       // nullptr: not wanted (equal to gy)
    float* partial;                 // [K][N][chunks]; nullptr: no bias
    int N, K, Q, chunks, vec_in, vec_out;
    long first, units;              // first of the launch, and all of them: N * K * chunks
};

// A wave has one chunk of one row (n, k).  Groups of 8 elements are counted over the whole tensor, so that they are aligned
// and match the bytes of the mask whatever Q is; the ones at the ends of a row are shared with its neighbours.
template <bool IN16, bool OUT16>
__global__ __launch_bounds__(kThreads) void epilogue_grad_kernel(GradArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const long unit = a.first + static_cast<long>(blockIdx.x) * (kThreads / kWave) + (threadIdx.x >> 6);
    if (unit >= a.units) return;
    const long row = unit / a.chunks, chunk = unit - row * a.chunks;
    const long r0 = row * a.Q, r1 = r0 + a.Q, n_all = static_cast<long>(a.N) * a.K * a.Q;
    const long g0 = (r0 >> 3) + chunk * kChunk, g1 = min(((r1 - 1) >> 3) + 1, g0 + kChunk);
    float sum = 0.f;
    for (long g = g0 + lane; g < g1; g += kInFlight * kWave) {
        float v[kInFlight][8];
        unsigned bits[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const long at = g + k * kWave, i = 8 * at;
            bits[k] = 0;
            if (at >= g1) continue;
            bits[k] = a.positive ? a.positive[at] : 0xffu;
            if (a.vec_in && i + 8 <= n_all) {
                load8<IN16>(a.gy, i, v[k]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[k][e] = i + e < n_all ? load_elem<IN16>(a.gy, i + e) : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const long at = g + k * kWave, i = 8 * at;
            if (at >= g1) continue;
            const bool whole = i >= r0 && i + 8 <= r1;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[k][e] *= (bits[k] >> e) & 1 ? 1.f : 0.f;
            if (a.dy) {
                if (a.vec_out && whole) {
                    if constexpr (OUT16) {
                        bf16x8 t;
#pragma unroll
                        for (int e = 0; e < 8; ++e) t[e] = static_cast<__bf16>(v[k][e]);
                        *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(a.dy) + i) = t;
                    } else {
                        float* o = static_cast<float*>(a.dy) + i;
                        *reinterpret_cast<f32x4*>(o) = f32x4{v[k][0], v[k][1], v[k][2], v[k][3]};
                        *reinterpret_cast<f32x4*>(o + 4) = f32x4{v[k][4], v[k][5], v[k][6], v[k][7]};
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (i + e >= r0 && i + e < r1) {
                            if constexpr (OUT16) static_cast<__bf16*>(a.dy)[i + e] = static_cast<__bf16>(v[k][e]);
                            else static_cast<float*>(a.dy)[i + e] = v[k][e];
                        }
                }
            }
            if (!whole) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (i + e < r0 || i + e >= r1) v[k][e] = 0.f;
            }
            sum += ((v[k][0] + v[k][1]) + (v[k][2] + v[k][3])) + ((v[k][4] + v[k][5]) + (v[k][6] + v[k][7]));
        }
    }
    if (!a.partial) return;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_down(sum, o, kWave);
    if (lane == 0) {
        const long n = row / a.K, k = row - n * a.K;
        a.partial[(k * a.N + n) * a.chunks + chunk] = sum;
    }
}

// one wave per filter, in 64 bits: the error of a gradient is that of its partial sums
__global__ __launch_bounds__(kWave) void bias_grad_kernel(const float* partial, float* dbias, long per) {
    const float* p = partial + blockIdx.x * per;
    double sum = 0.0;
#pragma unroll 4
    for (long i = threadIdx.x; i < per; i += kWave) sum += static_cast<double>(p[i]);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) sum += __shfl_down(sum, o, kWave);
    if (threadIdx.x == 0) dbias[blockIdx.x] = static_cast<float>(sum);
}

// groups of 8 a row of Q elements can touch, in chunks of one wave
long row_chunks(int Q) { return ((static_cast<long>(Q) + 14) / 8 + kChunk - 1) / kChunk; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// workgroups of a launch: what is more is launched in pieces
constexpr long kMostBlocks = 0x7fffffffL / kThreads;

}  // namespace

size_t epilogue_grad_workspace(int N, int K, int Q) { return 4 * static_cast<size_t>(N) * K * row_chunks(Q); }

hipError_t relu_mask_launch(const void* y, int bf16, unsigned char* positive, long n, hipStream_t st) {
    constexpr long per_block = 8L * kThreads * kInFlight;
    const int vec = aligned16(y);
    for (long at = 0; at < n; at += kMostBlocks * per_block) {
        const long left = n - at, blocks = (left + per_block - 1) / per_block;
        const dim3 grid(static_cast<unsigned>(blocks < kMostBlocks ? blocks : kMostBlocks));
        const void* from = static_cast<const char*>(y) + at * (bf16 ? 2 : 4);
        const hipError_t e = launch_kernel(bf16 ? relu_mask_kernel<true> : relu_mask_kernel<false>, grid, dim3(kThreads), 0, st, from,
                                           positive + at / 8, left, vec);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t epilogue_grad_launch(const void* gy, int in16, const unsigned char* positive, void* dy, int out16, float* dbias, float* ws,
                                int N, int K, int Q, hipStream_t st) {
    GradArgs a{};
    a.gy = gy; a.positive = positive; a.dy = dy; a.partial = dbias ? ws : nullptr;
    a.N = N; a.K = K; a.Q = Q;
    const long chunks = row_chunks(Q);
    a.chunks = static_cast<int>(chunks);
    a.vec_in = aligned16(gy);
    a.vec_out = aligned16(dy);
    a.units = static_cast<long>(N) * K * chunks;
    if (in16 && !out16) return hipErrorInvalidValue;
    auto kern = in16 ? epilogue_grad_kernel<true, true> : out16 ? epilogue_grad_kernel<false, true> : epilogue_grad_kernel<false, false>;
    constexpr long per_block = kThreads / kWave;
    for (a.first = 0; a.first < a.units; a.first += kMostBlocks * per_block) {
        const long blocks = (a.units - a.first + per_block - 1) / per_block;
        const dim3 grid(static_cast<unsigned>(blocks < kMostBlocks ? blocks : kMostBlocks));
        const hipError_t e = launch_kernel(kern, grid, dim3(kThreads), 0, st, a);
        if (e != hipSuccess) return e;
    }
    if (!dbias) return hipSuccess;
    return launch_kernel(bias_grad_kernel, dim3(static_cast<unsigned>(K)), dim3(kWave), 0, st, ws, dbias, static_cast<long>(N) * chunks);
}

}  // namespace conv1d
