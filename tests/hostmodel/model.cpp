// Runtime of the host-side bounds model: runs the library's kernels (compiled as CPU code through hip_cpu_shim.h)
// workgroup by workgroup and thread by thread, with every tensor of a call placed against an inaccessible guard
// page, and reports the first access that leaves a tensor.  TEST INFRASTRUCTURE, never part of the product library.
#include "hip_cpu_shim.h"

#include <setjmp.h>
#include <signal.h>
#include <stdio.h>
#include <sys/mman.h>
#include <unistd.h>

#include <vector>

#include "../../include/conv1d.h"
#include "conv1d_internal.h"  // (this file is compiled from a copy that sits beside the kernels' sources)

namespace hostmodel {

thread_local Idx g_thread, g_block, g_grid, g_bdim;

namespace {
const size_t kPage = 4096;
// inaccessible address space on either side of every tensor: a wrong sample or row index lands megabytes away
const size_t kGuard = size_t(1) << 28;
struct Region {
    char* map = nullptr;
    size_t map_bytes = 0;
    char* data = nullptr;
    size_t bytes = 0;
    const char* name = "";
};
std::vector<Region> g_regions;
Region g_lds;
sigjmp_buf g_jump;
volatile sig_atomic_t g_armed = 0;
void* volatile g_fault_addr = nullptr;

// [guard zone][pages for `bytes`][guard zone]; the data ends at the trailing guard (end_aligned: up to 15 bytes of
// slack keep the 16-byte alignment the fast kernels ask for) or starts right behind the leading one
Region make_region(size_t bytes, bool end_aligned, const char* name) {
    Region r;
    r.name = name;
    r.bytes = bytes;
    const size_t body = (bytes + kPage - 1) / kPage * kPage + (bytes == 0 ? kPage : 0);
    r.map_bytes = body + 2 * kGuard;
    r.map = static_cast<char*>(mmap(nullptr, r.map_bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
    if (r.map == MAP_FAILED) {
        r.map = nullptr;
        return r;
    }
    mprotect(r.map + kGuard, body, PROT_READ | PROT_WRITE);
    r.data = end_aligned ? r.map + kGuard + ((body - bytes) & ~static_cast<size_t>(15)) : r.map + kGuard;
    return r;
}
void free_region(Region& r) {
    if (r.map) munmap(r.map, r.map_bytes);
    r = Region{};
}

// the same with the last byte right before the guard, whatever alignment beyond `align` that leaves
Region make_exact(size_t bytes, size_t align, const char* name) {
    Region r = make_region(bytes, true, name);
    if (r.map) r.data = r.map + r.map_bytes - kGuard - (bytes + align - 1) / align * align;
    return r;
}

void on_fault(int, siginfo_t* info, void*) {
    if (!g_armed) _exit(139);
    g_fault_addr = info->si_addr;
    siglongjmp(g_jump, 1);
}
}  // namespace

int g_launches = 0;  // kernel launches of the last hostmodel_run

void* dynamic_lds() { return g_lds.data; }

// Runs a call of the library with faults caught: 0, 100 - its status, or 1 with a message about the access that left its
// tensor.
template <typename Call>
int guarded(int pass, char* msg, int msglen, Call call) {
    struct sigaction sa, old_segv, old_bus;
    memset(&sa, 0, sizeof(sa));
    sa.sa_sigaction = on_fault;
    sa.sa_flags = SA_SIGINFO | SA_NODEFER;
    sigaction(SIGSEGV, &sa, &old_segv);
    sigaction(SIGBUS, &sa, &old_bus);
    g_launches = 0;
    int rc;
    if (sigsetjmp(g_jump, 1) == 0) {
        g_armed = 1;
        const int st = call();
        g_armed = 0;
        rc = st == CONV1D_OK ? 0 : 100 - st;
    } else {
        g_armed = 0;
        const char* fa = static_cast<const char*>(g_fault_addr);
        const char* where = "no tensor of this call";
        long off = 0;
        for (const auto& r : g_regions)
            if (fa >= r.map && fa < r.map + r.map_bytes) {
                where = r.name;
                off = fa - r.data;
            }
        if (g_lds.map && fa >= g_lds.map && fa < g_lds.map + g_lds.map_bytes) {
            where = g_lds.name;
            off = fa - g_lds.data;
        }
        if (msg && msglen > 0)
            snprintf(msg, msglen, "access outside %s (address %p, byte offset %ld from its start) by workgroup (%u,%u) thread %u of a kernel of pass %d",
                     where, static_cast<const void*>(fa), off, g_block.x, g_block.y, g_thread.x, pass);
        rc = 1;
    }
    sigaction(SIGSEGV, &old_segv, nullptr);
    sigaction(SIGBUS, &old_bus, nullptr);
    return rc;
}

void run_grid(dim3 grid, dim3 block, size_t lds_bytes, const std::function<void()>& fn) {
    ++g_launches;
    free_region(g_lds);
    g_lds = make_region(lds_bytes, true, "dynamic LDS");
    g_grid = Idx{grid.x, grid.y, grid.z};
    g_bdim = Idx{block.x, block.y, block.z};
    for (unsigned by = 0; by < grid.y; ++by)
        for (unsigned bx = 0; bx < grid.x; ++bx) {
            g_block = Idx{bx, by, 0};
            for (unsigned t = 0; t < block.x; ++t) {
                g_thread = Idx{t, 0, 0};
                fn();
            }
        }
}

}  // namespace hostmodel

using namespace hostmodel;

// pass: 0 conv1d_fwd, 1 conv1d_bwd_data, 2 conv1d_bwd_weight, 3 conv1d_bwd, 4 conv1d_fwd_ex (bias, ReLU, bfloat16 output
// when dtype is bfloat16), 5 conv1d_bwd_data_ex (bfloat16 output), 6 conv1d_bwd_ex (bfloat16 dx).  placement: 0 tensors end at a guard page, 1 tensors
// start behind one, 2 as 0 with every tensor shifted by one element (the element-aligned paths).
// Returns 0 (every access inside its tensor), 1 (an access left its tensor; msg says where), or 100 - status when the
// library refused the call.
extern "C" int hostmodel_run(int pass, int N, int C, int K, int W, int S, int d, int P, int dtype, int variant, int placement,
                             char* msg, int msglen) {
    const long Q = static_cast<long>(W) + 2L * P - static_cast<long>(S - 1) * d;
    if (Q < 1) return 100 - CONV1D_EINVAL;
    const size_t e = dtype == CONV1D_BF16 ? 2 : 4;
    const bool out16 = dtype == CONV1D_BF16 && pass >= 4;
    const size_t shift = placement == 2 ? 1 : 0;
    const bool end_aligned = placement != 1;
    const size_t nx = static_cast<size_t>(N) * C * W, ny = static_cast<size_t>(N) * K * Q, nw = static_cast<size_t>(K) * C * S;
    for (auto& r : g_regions) free_region(r);
    g_regions.clear();
    auto tensor = [&](size_t elems, size_t esize, const char* name) -> char* {
        // a bfloat16 tensor may be read up to its next 4-byte boundary (include/conv1d.h)
        const size_t bytes = ((elems + shift) * esize + 3) & ~static_cast<size_t>(3);
        g_regions.push_back(make_region(bytes, end_aligned, name));
        return g_regions.back().data;
    };
    char* x = tensor(nx, e, "x");
    char* w = tensor(nw, e, "w");
    char* dy = tensor(ny, e, "dy");
    char* y = tensor(ny, out16 ? 2 : 4, "y");
    char* dx = tensor(nx, out16 ? 2 : 4, "dx");
    char* dw = tensor(nw, 4, "dw");
    char* bias = tensor(K, 4, "bias");
    const size_t wsb = conv1d_bwd_weight_workspace_bytes(N, C, K, W, S, d, P, dtype);
    g_regions.push_back(make_region(wsb + 256, false, "workspace"));
    char* ws = g_regions.back().data;
    if (shift) {  // one element into each allocation: only element alignment is left
        x += e; w += e; dy += e; y += out16 ? 2 : 4; dx += out16 ? 2 : 4; dw += 4;
    }
    conv1d_set_variant(variant);
    const int rc = guarded(pass, msg, msglen, [&] {
        switch (pass) {
            case 0: return conv1d_fwd(x, w, reinterpret_cast<float*>(y), N, C, K, W, S, d, P, dtype, nullptr);
            case 1: return conv1d_bwd_data(dy, w, reinterpret_cast<float*>(dx), N, C, K, W, S, d, P, dtype, nullptr);
            case 2: return conv1d_bwd_weight(x, dy, reinterpret_cast<float*>(dw), ws, wsb, N, C, K, W, S, d, P, dtype, nullptr);
            case 3: return conv1d_bwd(x, dy, w, reinterpret_cast<float*>(dx), reinterpret_cast<float*>(dw), ws, wsb, N, C, K, W, S, d, P, dtype, nullptr);
            case 4: return conv1d_fwd_ex(x, w, reinterpret_cast<float*>(bias), y, N, C, K, W, S, d, P, dtype,
                                         CONV1D_EPI_RELU | (out16 ? CONV1D_EPI_OUT_BF16 : 0), nullptr);
            case 5: return conv1d_bwd_data_ex(dy, w, dx, N, C, K, W, S, d, P, dtype, out16 ? CONV1D_EPI_OUT_BF16 : 0, nullptr);
            case 6: return conv1d_bwd_ex(x, dy, w, dx, reinterpret_cast<float*>(dw), ws, wsb, N, C, K, W, S, d, P, dtype,
                                         out16 ? CONV1D_EPI_OUT_BF16 : 0, nullptr);
            default: return static_cast<int>(CONV1D_EINVAL);
        }
    });
    conv1d_set_variant(0);
    return rc;
}

// The backward of the epilogue on N K Q elements: conv1d_relu_mask of an output and conv1d_epilogue_bwd with that mask (when
// relu), into dy (when want_dy) and dbias (when bias).  placement 0: every
// tensor ends at a guard page exactly, on the alignment of its elements alone; 1: it starts behind one, 16-byte aligned; 2:
// it ends at one, 16-byte aligned, up to 15 bytes before it.
extern "C" int hostmodel_run_epilogue(int N, int K, int Q, int in16, int out16, int relu, int want_dy, int bias, int placement,
                                      char* msg, int msglen) {
    const size_t n = static_cast<size_t>(N) * K * Q;
    for (auto& r : g_regions) free_region(r);
    g_regions.clear();
    auto tensor = [&](size_t bytes, size_t align, const char* name) -> char* {
        g_regions.push_back(placement == 0 ? make_exact(bytes, align, name) : make_region(bytes, placement == 2, name));
        return g_regions.back().data;
    };
    const size_t ei = in16 ? 2 : 4, eo = out16 ? 2 : 4, wsb = conv1d_epilogue_bwd_workspace_bytes(N, K, Q);
    char* y = tensor(n * ei, ei, "y");
    char* gy = tensor(n * ei, ei, "gy");
    char* mask = tensor((n + 7) / 8, 1, "mask");
    char* dy = tensor(n * eo, eo, "dy");
    float* db = reinterpret_cast<float*>(tensor(4 * static_cast<size_t>(K), 4, "dbias"));
    char* ws = tensor(wsb, 4, "workspace");
    return guarded(7, msg, msglen, [&] {
        if (relu) {
            const int st = conv1d_relu_mask(y, mask, n, in16 ? CONV1D_BF16 : CONV1D_FP32, nullptr);
            if (st != CONV1D_OK) return st;
        }
        return conv1d_epilogue_bwd(gy, relu ? mask : nullptr, want_dy ? dy : nullptr, bias ? db : nullptr, bias ? ws : nullptr,
                                   bias ? wsb : 0, N, K, Q, in16 ? CONV1D_BF16 : CONV1D_FP32, out16 ? CONV1D_BF16 : CONV1D_FP32, nullptr);
    });
}

extern "C" const char* hostmodel_kernel_name(int pass, int N, int C, int K, int W, int S, int d, int P, int dtype) {
    return conv1d_kernel_name(pass, N, C, K, W, S, d, P, dtype);
}

extern "C" int hostmodel_launches() { return g_launches; }
extern "C" void hostmodel_reset_launches() { g_launches = 0; }

// Tile of the FP32 kernels in three bfloat16 parts for a pass (0 forward, 1 backward-data, 2 backward-weight): t[0 .. 4] as
// conv1d::SplitTile (without its roundings); returns 0 where the pass cannot run on them.
extern "C" int hostmodel_split_tile(int pass, int N, int C, int K, int W, int S, int d, int P, long* t) {
    const int Q = W + 2 * P - (S - 1) * d;
    conv1d::SplitTile r{};
    bool ok;
    if (pass == 2) {
        conv1d::WgradProblem p{};
        p.N = N; p.C = C; p.K = K; p.W = W; p.Q = Q; p.S = S; p.d = d; p.P = P;
        p.x_sn = static_cast<long>(C) * W; p.dy_sn = static_cast<long>(K) * Q; p.dw_sk = static_cast<long>(C) * S; p.dw_sc = S;
        ok = conv1d::split_f32_wgrad_tile(p, &r);
    } else {
        conv1d::CorrProblem p{};
        p.N = N; p.S = S; p.d = d;
        p.R = pass == 0 ? C : K; p.M = pass == 0 ? K : C; p.Win = pass == 0 ? W : Q; p.Wout = pass == 0 ? Q : W;
        p.P = pass == 0 ? P : (S - 1) * d - P;
        ok = conv1d::split_f32_corr_tile(p, &r);
    }
    t[0] = r.filter_blocks; t[1] = r.columns_or_taps; t[2] = r.planes_or_units; t[3] = r.grid; t[4] = r.x_slots;
    return ok;
}

// Roundings of a weight gradient's sums in the tile taken (0: none is) and in that of the kernel of several filter blocks.
extern "C" void hostmodel_wgrad_roundings(int N, int C, int K, int W, int S, int d, int P, double* r) {
    conv1d::WgradProblem p{};
    p.N = N; p.C = C; p.K = K; p.W = W; p.Q = W + 2 * P - (S - 1) * d; p.S = S; p.d = d; p.P = P;
    p.x_sn = static_cast<long>(C) * W; p.dy_sn = static_cast<long>(K) * p.Q; p.dw_sk = static_cast<long>(C) * S; p.dw_sc = S;
    conv1d::SplitTile t{};
    r[0] = conv1d::split_f32_wgrad_tile(p, &t) ? t.roundings : 0.0;
    r[1] = conv1d::split_f32_wgrad_pair_roundings(p);
}

// The multiply-high division of the kernels against the plain one: the first n <= nmax whose quotient differs, -1 if
// none does, -2 if make_fastdiv refuses the pair (it must refuse every pair for which the quotient could be wrong).
extern "C" long hostmodel_fastdiv_mismatch(long d, long nmax) {
    conv1d::FastDiv f;
    if (!conv1d::make_fastdiv(f, d, nmax)) return -2;
    for (long n = 0; n <= nmax; ++n)
        if (conv1d::fast_div(static_cast<int>(n), f) != static_cast<int>(n / d)) return n;
    return -1;
}
