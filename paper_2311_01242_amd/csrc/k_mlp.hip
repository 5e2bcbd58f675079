// Warm-start MLP on gfx950: bfloat16 GEMM operands on the matrix cores
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation), FP32 bias / GELU / MSE /
// Adam, FP32 master weights with a bfloat16 copy for the products.
//
// A project addition on top of the method: the network maps a bond-stretch
// geometry descriptor to UCCSD amplitudes, trained on the converged
// amplitudes that plain VQE produces along the scan (Sec. 3.1 "Results for
// bond stretching" is the scan this stands in for); VQE started from its
// prediction is compared with VQE from the Hartree-Fock point (Eq. 1).
//
// Layer l: z_l = a_{l-1} W_l^T + b_l; a_l = GELU(z_l) (exact erf form) for
// hidden layers; the last layer is linear.  Loss: mean squared error.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <type_traits>
#include <vector>

#include "internal.h"

typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace vqe {

#define HIPCHK_M(expr)                                                                      \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(VQE_EDEVICE, std::string("HIP error in ") + #expr + ": " +         \
                                         hipGetErrorString(e_));                            \
    } while (0)

// float -> bfloat16, round to nearest even (NaN stays NaN)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

__device__ __forceinline__ float gelu_f(float z) {
    return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
}

__device__ __forceinline__ float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
           z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// A training step is L forward launches, L - 1 for dL/dz and one for every
// gradient with its Adam update (37-256-256-360 on 160 rows: 6 launches, 42 us
// a step; as 16 launches of products from strided 2-byte reads, activation,
// loss, column sums and Adam apart it was 104 us).  Launch latency and one
// round trip to L2 per launch bound it: the products are 157 MFLOP a step.
//
// bf16 operands are kept twice, row-major and transposed, with rows padded to
// multiples of 32 elements (zeros), so that every product reads both operands
// in 16-byte pieces along its inner dimension.
constexpr int kMaxLayers = 8;

struct MlpLayer {
    int fi, fo, fip, fop;     // widths, padded
    int64_t woff, boff;       // parameter offsets of W [fo][fi] and b [fo]
    uint16_t *w, *wt;         // W: [fo][fip]; W^T: [fi][fop]
    uint16_t *a, *at;         // the layer's input: [B][fip]; [fi][bp]
    float* z;                 // its pre-activation [B][fo]
    uint16_t *d, *dt;         // dL/dz: [B][fop]; [fo][bp]
    float* dtf;               // dL/dz in fp32: [fo][bp]
};

struct MlpArgs {
    MlpLayer l[kMaxLayers];
    int L, B, bp;             // layers; rows; row capacity, a multiple of 32
    float *p, *m, *v, *g;     // parameters, Adam moments, gradient
    const float* y;           // targets [B][fo of the last layer]
    float *lpart, *loss, *trace;   // loss partials (one per output tile), loss, its trace
    int *t, *tnext;           // steps taken; the step being taken
    int trace_cap;
    float lr, b1, b2, eps;
};

// One wave's 16 x 16 tile of A B^T, A [M][sa] and B [N][sb] with the inner
// dimension contiguous; rows past the end repeat the last one (their results
// are not stored).  Operand fragments of v_mfma_f32_16x16x32_bf16: lane l
// holds A[l%16][8(l/16)+r] and B[8(l/16)+r][l%16], r = 0..7; the result is
// D[4(l/16)+r][l%16], r = 0..3.  Eight blocks of 32 are in flight at once:
// at these sizes the product is a round trip to L2, not arithmetic.  MASK:
// elements from K on (stale rows of a larger batch) are cleared.
template <bool MASK>
__device__ __forceinline__ f32x4 tile_product(const uint16_t* __restrict__ A, int M, int sa,
                                              const uint16_t* __restrict__ B, int N, int sb, int ti, int tj, int K) {
    const int lane = threadIdx.x & 63, kq = (lane >> 4) * 8;
    const s16x8* pa = reinterpret_cast<const s16x8*>(A + int64_t(min(ti + (lane & 15), M - 1)) * sa + kq);
    const s16x8* pb = reinterpret_cast<const s16x8*>(B + int64_t(min(tj + (lane & 15), N - 1)) * sb + kq);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int nk = (K + 31) / 32;
    for (int k0 = 0; k0 < nk; k0 += 8) {
        s16x8 a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int kb = min(k0 + u, nk - 1);
            a[u] = pa[kb * 4];
            b[u] = pb[kb * 4];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (k0 + u >= nk) break;
            if (MASK && (k0 + u) * 32 + 32 > K) {
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    if ((k0 + u) * 32 + kq + r >= K) a[u][r] = b[u][r] = 0;
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u]),
                                                          __builtin_bit_cast(bf16x8, b[u]), acc, 0, 0, 0);
        }
    }
    return acc;
}

// Rows ii .. ii + 3 (below M) of column jj of a row-major and a transposed
// bf16 array (and an fp32 transposed one, if given).
__device__ __forceinline__ void store4(const float (&v)[4], int ii, int M, int jj, uint16_t* __restrict__ rm, int srm,
                                       uint16_t* __restrict__ tr, float* __restrict__ trf, int str) {
    uint16_t h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        h[r] = f2bf(v[r]);
        if (ii + r < M) rm[int64_t(ii + r) * srm + jj] = h[r];
    }
    uint16_t* q = tr + int64_t(jj) * str + ii;
    float* qf = trf ? trf + int64_t(jj) * str + ii : nullptr;
    if (ii + 3 < M) {   // ii and the stride are multiples of 4: 8- and 16-byte aligned
        *reinterpret_cast<uint2*>(q) = make_uint2(uint32_t(h[0]) | (uint32_t(h[1]) << 16),
                                                  uint32_t(h[2]) | (uint32_t(h[3]) << 16));
        if (qf) *reinterpret_cast<float4*>(qf) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (ii + r < M) {
                q[r] = h[r];
                if (qf) qf[r] = v[r];
            }
    }
}

// src [rows][cols] -> bf16 row-major [rows][srm] and transposed [cols][str].
__global__ void k_pack(const float* __restrict__ src, int64_t n, int cols, uint16_t* __restrict__ rm, int srm,
                       uint16_t* __restrict__ tr, int str) {
    for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n;
         e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t i = e / cols;
        const int j = int(e - i * cols);
        const uint16_t h = f2bf(src[e]);
        rm[i * srm + j] = h;
        tr[int64_t(j) * str + i] = h;
    }
}

// Layer l forward: z = a W^T + b; a hidden layer stores GELU(z) as the next
// layer's input.  The last layer of a training pass (TRAIN) also forms dL/dz =
// 2 (z - y) / (B N) and its tile's part of the loss.
template <bool TRAIN>
__global__ void __launch_bounds__(64) k_mlp_fwd(MlpArgs n, int l) {
    const MlpLayer& q = n.l[l];
    const int ti = blockIdx.y * 16, tj = blockIdx.x * 16, lane = threadIdx.x;
    const int ii = ti + (lane >> 4) * 4, jj = tj + (lane & 15);
    const bool col = jj < q.fo, last = l == n.L - 1;
    const float bias = n.p[q.boff + min(jj, q.fo - 1)];
    float yv[4] = {0.f, 0.f, 0.f, 0.f};
    if (TRAIN && last) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            yv[r] = n.y[int64_t(min(ii + r, n.B - 1)) * q.fo + min(jj, q.fo - 1)];
    }
    const f32x4 acc = tile_product<false>(q.a, n.B, q.fip, q.w, q.fo, q.fip, ti, tj, q.fip);
    float c[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c[r] = acc[r] + bias;
        if (col && ii + r < n.B) q.z[int64_t(ii + r) * q.fo + jj] = c[r];
    }
    if (!last) {
        const MlpLayer& x = n.l[l + 1];
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = gelu_f(c[r]);
        if (col) store4(v, ii, n.B, jj, x.a, x.fip, x.at, nullptr, n.bp);
    } else if (TRAIN) {
        const float sc = 2.0f / float(int64_t(n.B) * q.fo);
        float v[4], s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = c[r] - yv[r];
            if (col && ii + r < n.B) s += d * d;
            v[r] = sc * d;
        }
        if (col) store4(v, ii, n.B, jj, q.d, q.fop, q.dt, q.dtf, n.bp);
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
        if (lane == 0) n.lpart[int64_t(blockIdx.y) * gridDim.x + blockIdx.x] = s;
        if (lane == 0 && blockIdx.x == 0 && blockIdx.y == 0) *n.tnext = *n.t + 1;
    }
}

// dL/dz of layer l - 1: (dL/dz_l W_l) GELU'(z_{l-1}).
__global__ void __launch_bounds__(64) k_mlp_back(MlpArgs n, int l) {
    const MlpLayer& q = n.l[l];
    const MlpLayer& x = n.l[l - 1];
    const int ti = blockIdx.y * 16, tj = blockIdx.x * 16, lane = threadIdx.x;
    const int ii = ti + (lane >> 4) * 4, jj = tj + (lane & 15);
    float zv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) zv[r] = x.z[int64_t(min(ii + r, n.B - 1)) * x.fo + min(jj, x.fo - 1)];
    const f32x4 acc = tile_product<false>(q.d, n.B, q.fop, q.wt, q.fi, q.fop, ti, tj, q.fop);
    float v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = acc[r] * gelu_grad_f(zv[r]);
    if (jj < q.fi) store4(v, ii, n.B, jj, x.d, x.fop, x.dt, x.dtf, n.bp);
}

__device__ __forceinline__ float adam_step(const MlpArgs& n, int64_t k, float gk, float mk, float vk, float pk,
                                           float c1, float c2) {
    // the roundings spelled out: contraction that varies with the surrounding
    // code would change which weights round up in bf16
    mk = __fmaf_rn(1.0f - n.b1, gk, __fmul_rn(n.b1, mk));
    vk = __fmaf_rn(gk, __fmul_rn(1.0f - n.b2, gk), __fmul_rn(n.b2, vk));
    n.m[k] = mk;
    n.v[k] = vk;
    pk = pk - n.lr * (mk / c1) / (sqrtf(vk / c2) + n.eps);
    n.p[k] = pk;
    return pk;
}

// Every layer's weight gradient dW[j][k] = sum_i dz[i][j] a[i][k] (one wave
// per 16 x 16 tile), bias gradient (one wave per output, lane u adding rows u,
// u + 64, ... in order, then a butterfly) and the loss (one wave), then, with
// ADAM, the update of the fp32 parameters and the bf16 copies in place.  Wave
// id: the layers' weight tiles, their biases, the loss.
template <bool ADAM>
__global__ void __launch_bounds__(64) k_mlp_update(MlpArgs n) {
    const int lane = threadIdx.x;
    float c1 = 1.f, c2 = 1.f;
    if (ADAM) {
        const float step = float(*n.tnext);   // the count of this step, from 1
        c1 = 1.0f - powf(n.b1, step);
        c2 = 1.0f - powf(n.b2, step);
    }
    int64_t id = blockIdx.x;
    for (int l = 0; l < n.L; ++l) {
        const MlpLayer& q = n.l[l];
        const int tk = (q.fi + 15) / 16, tiles = ((q.fo + 15) / 16) * tk;
        if (id < tiles) {
            const int ti = int(id / tk) * 16, tj = int(id % tk) * 16;
            const int ii = ti + (lane >> 4) * 4, jj = tj + (lane & 15);
            const bool col = jj < q.fi;
            float mo[4], vo[4], po[4];
            if (ADAM) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t k = q.woff + int64_t(min(ii + r, q.fo - 1)) * q.fi + min(jj, q.fi - 1);
                    mo[r] = n.m[k];
                    vo[r] = n.v[k];
                    po[r] = n.p[k];
                }
            }
            const f32x4 acc = tile_product<true>(q.dt, q.fo, n.bp, q.at, q.fi, n.bp, ti, tj, n.B);
            float w[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                w[r] = 0.f;
                if (!col || ii + r >= q.fo) continue;
                const int64_t k = q.woff + int64_t(ii + r) * q.fi + jj;
                if (ADAM) w[r] = adam_step(n, k, acc[r], mo[r], vo[r], po[r], c1, c2);
                else n.g[k] = acc[r];
            }
            if (ADAM && col) store4(w, ii, q.fo, jj, q.w, q.fip, q.wt, nullptr, q.fop);
            return;
        }
        id -= tiles;
    }
    for (int l = 0; l < n.L; ++l) {
        const MlpLayer& q = n.l[l];
        if (id < q.fo) {
            const float* d = q.dtf + id * n.bp;
            float s = 0.f;
            for (int i = lane; i < n.B; i += 64) s += d[i];
#pragma unroll
            for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
            if (lane == 0) {
                const int64_t k = q.boff + id;
                if (ADAM) (void)adam_step(n, k, s, n.m[k], n.v[k], n.p[k], c1, c2);
                else n.g[k] = s;
            }
            return;
        }
        id -= q.fo;
    }
    // the loss: the tiles' parts, lane u adding parts u, u + 64, ... in order
    const MlpLayer& q = n.l[n.L - 1];
    const int64_t parts = int64_t((q.fo + 15) / 16) * ((n.B + 15) / 16);
    double s = 0.0;
    for (int64_t i = lane; i < parts; i += 64) s += double(n.lpart[i]);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
    if (lane == 0) {
        const float v = float(s / double(int64_t(n.B) * q.fo));
        *n.loss = v;
        if (ADAM) {
            const int step = *n.tnext - 1;
            if (step < n.trace_cap) n.trace[step] = v;
            *n.t = step + 1;
        }
    }
}

}  // namespace vqe

using namespace vqe;

// ============================================================== C ABI (MLP)

struct vqe_mlp {
    int L = 0;
    std::vector<int> w;             // widths, L + 1
    std::vector<int64_t> woff, boff;  // parameter offsets of W_l and b_l
    int64_t P = 0;
    int dev = 0;
    hipStream_t st = nullptr;
    float *p = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
    int* t = nullptr;               // device step counters: steps taken, the step being taken
    float* loss = nullptr;
    MlpLayer layer[kMaxLayers] = {};
    // batch buffers
    int bcap = 0;                   // rows, a multiple of 32
    float *y = nullptr, *x = nullptr, *lpart = nullptr;
    float* trace = nullptr;
    int trace_cap = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int graph_batch = 0;
    float graph_hp[4] = {0, 0, 0, 0};
    std::vector<void*> allocs;
    ~vqe_mlp() {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(dev);
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        for (void* a : allocs) (void)hipFree(a);
        if (st) (void)hipStreamDestroy(st);
        (void)hipSetDevice(cur);
    }
};

namespace {

int mlp_alloc(vqe_mlp* n, void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, std::max<size_t>(bytes, 16));
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? VQE_ENOMEM : VQE_EDEVICE,
                    std::string("MLP allocation: ") + hipGetErrorString(e));
    n->allocs.push_back(*p);
    return VQE_OK;
}

template <class T>
int mlp_alloc_t(vqe_mlp* n, T** p, size_t count) {
    return mlp_alloc(n, reinterpret_cast<void**>(p), count * sizeof(T));
}

int ensure_batch(vqe_mlp* n, int B) {
    if (B <= n->bcap) return VQE_OK;
    HIPCHK_M(hipStreamSynchronize(n->st));
    // buffers for the new capacity (old ones stay allocated until free), their
    // padding cleared once: the kernels write live entries only
    B = (B + 31) & ~31;
    size_t total = 0;
    for (int pass = 0; pass < 2; ++pass) {   // sizes, then one allocation cut up
        char* base = nullptr;
        if (pass == 1) {
            if (int rc = mlp_alloc(n, reinterpret_cast<void**>(&base), total)) return rc;
            HIPCHK_M(hipMemsetAsync(base, 0, total, n->st));
        }
        total = 0;
        auto take = [&](auto** p, size_t count) {
            *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(base + total);
            total += (count * sizeof(**p) + 255) & ~size_t(255);
        };
        MlpLayer scratch[kMaxLayers] = {};
        float *x, *y, *lpart;
        for (int l = 0; l < n->L; ++l) {
            MlpLayer& q = pass == 1 ? n->layer[l] : scratch[l];
            const MlpLayer& d = n->layer[l];
            take(&q.a, size_t(B) * d.fip);
            take(&q.at, size_t(d.fi) * B);
            take(&q.z, size_t(B) * d.fo);
            take(&q.d, size_t(B) * d.fop);
            take(&q.dt, size_t(d.fo) * B);
            take(&q.dtf, size_t(d.fo) * B);
        }
        take(pass == 1 ? &n->x : &x, size_t(B) * n->w[0]);
        take(pass == 1 ? &n->y : &y, size_t(B) * n->w[n->L]);
        take(pass == 1 ? &n->lpart : &lpart, size_t((B + 15) / 16) * ((n->w[n->L] + 15) / 16));
    }
    n->bcap = B;
    if (n->exec) {
        (void)hipGraphExecDestroy(n->exec);
        n->exec = nullptr;
    }
    if (n->graph) {
        (void)hipGraphDestroy(n->graph);
        n->graph = nullptr;
    }
    return VQE_OK;
}

int blocks(int64_t n) { return int(std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 1024))); }

MlpArgs mlp_args(const vqe_mlp* n, int B) {
    MlpArgs a{};
    std::copy(n->layer, n->layer + n->L, a.l);
    a.L = n->L;
    a.B = B;
    a.bp = n->bcap;
    a.p = n->p;
    a.m = n->m;
    a.v = n->v;
    a.g = n->g;
    a.y = n->y;
    a.lpart = n->lpart;
    a.loss = n->loss;
    a.trace = n->trace;
    a.t = n->t;
    a.tnext = n->t + 1;
    a.trace_cap = n->trace ? n->trace_cap : 0;
    return a;
}

// B rows of inputs into the first layer's operands.
void enqueue_input(vqe_mlp* n, int B) {
    const MlpLayer& q = n->layer[0];
    hipLaunchKernelGGL(k_pack, dim3(blocks(int64_t(B) * q.fi)), dim3(256), 0, n->st, n->x, int64_t(B) * q.fi, q.fi,
                       q.a, q.fip, q.at, n->bcap);
}

void enqueue_forward(vqe_mlp* n, const MlpArgs& a, bool train) {
    for (int l = 0; l < n->L; ++l) {
        const dim3 grid((n->w[l + 1] + 15) / 16, (a.B + 15) / 16);
        if (train) hipLaunchKernelGGL(k_mlp_fwd<true>, grid, dim3(64), 0, n->st, a, l);
        else hipLaunchKernelGGL(k_mlp_fwd<false>, grid, dim3(64), 0, n->st, a, l);
    }
}

// After a training forward pass: dL/dz of the hidden layers, then every
// gradient with the loss, applied by Adam or stored (into n->g).
void enqueue_backward(vqe_mlp* n, const MlpArgs& a, bool adam) {
    for (int l = n->L - 1; l > 0; --l)
        hipLaunchKernelGGL(k_mlp_back, dim3((n->w[l] + 15) / 16, (a.B + 15) / 16), dim3(64), 0, n->st, a, l);
    int64_t waves = 1;
    for (int l = 0; l < n->L; ++l)
        waves += int64_t((n->w[l] + 15) / 16) * ((n->w[l + 1] + 15) / 16) + n->w[l + 1];
    if (adam) hipLaunchKernelGGL(k_mlp_update<true>, dim3(unsigned(waves)), dim3(64), 0, n->st, a);
    else hipLaunchKernelGGL(k_mlp_update<false>, dim3(unsigned(waves)), dim3(64), 0, n->st, a);
}

int check_rows(const vqe_mlp* n, int B, const float* x) {
    if (!n || !x) return fail(VQE_EINVAL, "null pointer argument");
    if (B < 1 || B > 65536) return fail(VQE_ERANGE, "batch must be in [1, 65536]");
    if (!std::all_of(x, x + int64_t(B) * n->w[0], [](float v) { return std::isfinite(v); }))
        return fail(VQE_EINVAL, "non-finite input");
    return VQE_OK;
}

}  // namespace

extern "C" int vqe_mlp_create(int n_layers, const int32_t* widths, void* stream, vqe_mlp** out) {
    if (!out || !widths) return fail(VQE_EINVAL, "null pointer argument");
    *out = nullptr;
    if (n_layers < 1 || n_layers > 8) return fail(VQE_ERANGE, "n_layers must be in [1, 8]");
    for (int l = 0; l <= n_layers; ++l)
        if (widths[l] < 1 || widths[l] > 8192) return fail(VQE_ERANGE, "widths must be in [1, 8192]");
    auto* n = new vqe_mlp();
    std::unique_ptr<vqe_mlp> guard(n);
    n->L = n_layers;
    n->w.assign(widths, widths + n_layers + 1);
    for (int l = 0; l < n_layers; ++l) {
        n->woff.push_back(n->P);
        n->P += int64_t(n->w[l]) * n->w[l + 1];
        n->boff.push_back(n->P);
        n->P += n->w[l + 1];
    }
    (void)stream;   // the network orders its work on a stream of its own
    HIPCHK_M(hipGetDevice(&n->dev));
    HIPCHK_M(hipStreamCreateWithFlags(&n->st, hipStreamNonBlocking));
    // the fp32 vectors with the counters, and the bf16 weights, one cleared
    // allocation each
    const size_t pad = size_t(n->P + 63) & ~size_t(63);
    if (int rc = mlp_alloc_t(n, &n->p, 4 * pad + 64)) return rc;
    HIPCHK_M(hipMemsetAsync(n->p, 0, (4 * pad + 64) * sizeof(float), n->st));
    n->m = n->p + pad;
    n->v = n->m + pad;
    n->g = n->v + pad;
    n->loss = n->g + pad;
    n->t = reinterpret_cast<int*>(n->loss + 1);
    size_t words = 0;
    for (int l = 0; l < n_layers; ++l) {
        MlpLayer& q = n->layer[l];
        q.fi = n->w[l];
        q.fo = n->w[l + 1];
        q.fip = (q.fi + 31) & ~31;
        q.fop = (q.fo + 31) & ~31;
        q.woff = n->woff[l];
        q.boff = n->boff[l];
        words += size_t(q.fo) * q.fip + size_t(q.fi) * q.fop;   // multiples of 32 each
    }
    uint16_t* h = nullptr;
    if (int rc = mlp_alloc_t(n, &h, words)) return rc;
    HIPCHK_M(hipMemsetAsync(h, 0, words * sizeof(uint16_t), n->st));
    for (int l = 0; l < n_layers; ++l) {
        MlpLayer& q = n->layer[l];
        q.w = h;
        q.wt = h + size_t(q.fo) * q.fip;
        h = q.wt + size_t(q.fi) * q.fop;
    }
    HIPCHK_M(hipStreamSynchronize(n->st));
    *out = guard.release();
    return VQE_OK;
}

extern "C" int vqe_mlp_n_params(const vqe_mlp* n, int64_t* count) {
    if (!n || !count) return fail(VQE_EINVAL, "null pointer argument");
    *count = n->P;
    return VQE_OK;
}

extern "C" int vqe_mlp_set_params(vqe_mlp* n, const float* params) {
    if (!n || !params) return fail(VQE_EINVAL, "null pointer argument");
    if (!std::all_of(params, params + n->P, [](float v) { return std::isfinite(v); }))
        return fail(VQE_EINVAL, "non-finite parameter");
    HIPCHK_M(hipMemcpyAsync(n->p, params, n->P * sizeof(float), hipMemcpyHostToDevice, n->st));
    for (int l = 0; l < n->L; ++l) {
        const MlpLayer& q = n->layer[l];
        hipLaunchKernelGGL(k_pack, dim3(blocks(int64_t(q.fi) * q.fo)), dim3(256), 0, n->st, n->p + q.woff,
                           int64_t(q.fi) * q.fo, q.fi, q.w, q.fip, q.wt, q.fop);
    }
    HIPCHK_M(hipMemsetAsync(n->m, 0, n->P * sizeof(float), n->st));
    HIPCHK_M(hipMemsetAsync(n->v, 0, n->P * sizeof(float), n->st));
    HIPCHK_M(hipMemsetAsync(n->t, 0, 2 * sizeof(int), n->st));
    HIPCHK_M(hipGetLastError());
    HIPCHK_M(hipStreamSynchronize(n->st));
    return VQE_OK;
}

extern "C" int vqe_mlp_get_params(const vqe_mlp* n, float* params) {
    if (!n || !params) return fail(VQE_EINVAL, "null pointer argument");
    HIPCHK_M(hipMemcpyAsync(params, n->p, n->P * sizeof(float), hipMemcpyDeviceToHost, n->st));
    HIPCHK_M(hipStreamSynchronize(n->st));
    return VQE_OK;
}

extern "C" int vqe_mlp_forward(vqe_mlp* n, int B, const float* x, float* y) {
    if (int rc = check_rows(n, B, x)) return rc;
    if (!y) return fail(VQE_EINVAL, "null output");
    if (int rc = ensure_batch(n, B)) return rc;
    HIPCHK_M(hipMemcpyAsync(n->x, x, size_t(B) * n->w[0] * sizeof(float), hipMemcpyHostToDevice,
                            n->st));
    enqueue_input(n, B);
    enqueue_forward(n, mlp_args(n, B), false);
    HIPCHK_M(hipGetLastError());
    HIPCHK_M(hipMemcpyAsync(y, n->layer[n->L - 1].z, size_t(B) * n->w[n->L] * sizeof(float),
                            hipMemcpyDeviceToHost, n->st));
    HIPCHK_M(hipStreamSynchronize(n->st));
    return VQE_OK;
}

extern "C" int vqe_mlp_loss_grad(vqe_mlp* n, int B, const float* x, const float* y, float* loss,
                                 float* grad) {
    if (int rc = check_rows(n, B, x)) return rc;
    if (!y || !loss) return fail(VQE_EINVAL, "null pointer argument");
    if (int rc = ensure_batch(n, B)) return rc;
    HIPCHK_M(hipMemcpyAsync(n->x, x, size_t(B) * n->w[0] * sizeof(float), hipMemcpyHostToDevice,
                            n->st));
    HIPCHK_M(hipMemcpyAsync(n->y, y, size_t(B) * n->w[n->L] * sizeof(float), hipMemcpyHostToDevice,
                            n->st));
    enqueue_input(n, B);
    const MlpArgs args = mlp_args(n, B);
    enqueue_forward(n, args, true);
    enqueue_backward(n, args, false);
    HIPCHK_M(hipGetLastError());
    HIPCHK_M(hipMemcpyAsync(loss, n->loss, sizeof(float), hipMemcpyDeviceToHost, n->st));
    if (grad)
        HIPCHK_M(hipMemcpyAsync(grad, n->g, n->P * sizeof(float), hipMemcpyDeviceToHost, n->st));
    HIPCHK_M(hipStreamSynchronize(n->st));
    return VQE_OK;
}

extern "C" int vqe_mlp_train(vqe_mlp* n, int B, const float* x, const float* y, int steps, float lr,
                             float beta1, float beta2, float eps, float* loss_trace) {
    if (int rc = check_rows(n, B, x)) return rc;
    if (!y) return fail(VQE_EINVAL, "null targets");
    if (steps < 0) return fail(VQE_ERANGE, "steps < 0");
    if (!(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return fail(VQE_EINVAL, "invalid Adam hyper-parameters");
    if (!std::all_of(y, y + int64_t(B) * n->w[n->L], [](float v) { return std::isfinite(v); }))
        return fail(VQE_EINVAL, "non-finite target");
    if (int rc = ensure_batch(n, B)) return rc;
    // loss trace indexed by the step counter relative to this call
    int t0 = 0;
    HIPCHK_M(hipMemcpyAsync(&t0, n->t, sizeof(int), hipMemcpyDeviceToHost, n->st));
    HIPCHK_M(hipStreamSynchronize(n->st));
    if (n->trace_cap < t0 + steps) {
        void* tr = nullptr;
        if (int rc = mlp_alloc(n, &tr, size_t(t0 + steps + 1024) * sizeof(float))) return rc;
        n->trace = static_cast<float*>(tr);
        n->trace_cap = t0 + steps + 1024;
        if (n->exec) {   // the captured graph refers to the old trace buffer
            (void)hipGraphExecDestroy(n->exec);
            n->exec = nullptr;
            (void)hipGraphDestroy(n->graph);
            n->graph = nullptr;
        }
    }
    HIPCHK_M(hipMemcpyAsync(n->x, x, size_t(B) * n->w[0] * sizeof(float), hipMemcpyHostToDevice,
                            n->st));
    HIPCHK_M(hipMemcpyAsync(n->y, y, size_t(B) * n->w[n->L] * sizeof(float), hipMemcpyHostToDevice,
                            n->st));
    enqueue_input(n, B);
    const float hp[4] = {lr, beta1, beta2, eps};
    if (n->exec && (n->graph_batch != B || std::memcmp(hp, n->graph_hp, sizeof(hp)) != 0)) {
        (void)hipGraphExecDestroy(n->exec);
        n->exec = nullptr;
        (void)hipGraphDestroy(n->graph);
        n->graph = nullptr;
    }
    if (!n->exec) {
        // one training step: forward, dL/dz, gradients with Adam
        MlpArgs args = mlp_args(n, B);
        args.lr = lr;
        args.b1 = beta1;
        args.b2 = beta2;
        args.eps = eps;
        HIPCHK_M(hipStreamBeginCapture(n->st, hipStreamCaptureModeThreadLocal));
        enqueue_forward(n, args, true);
        enqueue_backward(n, args, true);
        hipGraph_t g = nullptr;
        const hipError_t ce = hipStreamEndCapture(n->st, &g);
        n->graph = g;
        HIPCHK_M(ce);
        HIPCHK_M(hipGraphInstantiate(&n->exec, n->graph, nullptr, nullptr, 0));
        n->graph_batch = B;
        std::memcpy(n->graph_hp, hp, sizeof(hp));
    }
    for (int s = 0; s < steps; ++s) HIPCHK_M(hipGraphLaunch(n->exec, n->st));
    if (loss_trace && steps > 0)
        HIPCHK_M(hipMemcpyAsync(loss_trace, n->trace + t0, size_t(steps) * sizeof(float),
                                hipMemcpyDeviceToHost, n->st));
    HIPCHK_M(hipStreamSynchronize(n->st));
    return VQE_OK;
}

extern "C" void vqe_mlp_free(vqe_mlp* n) { delete n; }
