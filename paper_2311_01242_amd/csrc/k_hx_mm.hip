// H-apply of a molecular Hamiltonian as matrix products on the FP64 matrix
// cores (Sec. 2.1.1, Eq. 1): lambda = H phi and Re <phi|lambda> on the
// reference's (N, S_z) sector with real amplitudes, in string-product order.
//
// With the sign (-1)^f(a, b), f the number of (alpha, beta) occupied pairs
// whose alpha orbital comes after the beta one in the register, taken into
// the amplitudes (the order conversions apply it), no Jordan-Wigner chain
// crosses from one spin to the other, and a Hamiltonian of Eq. 2 is
//     H = Ha x 1 + 1 x Hb + sum_{P, R} G[P][R] E_P x E_R
// with Ha, Hb the same-spin parts (dense matrices over the alpha and beta
// strings), P the alpha moves (the orbital pairs p < q with E = a+_p a_q +
// a+_q a_p, then the occupations n_p) and R the beta ones.
//
// * k_hx_same: Ha phi + phi Hb, one product of inner length NA + NB.
// * k_hx_cross: for a row a the alpha moves that a admits pick na (oa - na)
//   partner rows; with the row itself (its occupations summed into one
//   coefficient row) they are the K inputs of T = A B, A[R][k] = +-G[P_k][R],
//   B[k] the partner rows; then lambda(a, b) adds T[R][b ^ x_R] over the beta
//   moves R that b admits, from LDS.  Against walking the (alpha move, beta
//   move) pairs one by one from LDS (two 8-byte gathers per pair) this takes
//   M/(nb (ob - nb) + nb) times the flops (about 2), all of them on the matrix
//   cores, and one 8-byte gather per beta move instead of two per pair.
//
// Measured, H-apply with its order conversions, walking kernel -> here: one
// state of 24 qubits 690 -> 268 us, of 20 qubits 53 -> 28, of 16 qubits 54 (in
// a batch of one) -> 19; 49 states of 20 qubits 970 -> 387 us, 60 of 17 qubits
// 213 -> 82, 20 of 12 qubits 25 -> 18.  k_hx_cross then runs at 43 TFLOP/s on
// 49 states of 20 qubits (265 us; the FP64 matrix peak is 78.6): its products
// take half the time, the rest is the gathers and each row's first loads.
#include <hip/hip_runtime.h>

#include "device_common.h"

namespace vqe {

using d4 = __attribute__((ext_vector_type(4))) double;

// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and
// D[4 v + l / 16][l % 16] for v = 0 .. 3.
__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// State and block of a workgroup.  xs > 0 (a batch of xs states): workgroup
// id i (dispatched to XCD i mod 8) works on state 8 q + (i mod 8), so that all
// of a state's workgroups share one XCD's L2.
__device__ __forceinline__ bool mm_place(int xs, int nblk, int& state, int& blk) {
    state = blockIdx.y;
    blk = blockIdx.x;
    if (xs > 0) {
        const int slot = int(blockIdx.x >> 3), q = slot / nblk;
        blk = slot - q * nblk;
        state = 8 * q + int(blockIdx.x & 7);
    }
    return xs == 0 || state < xs;
}

// aux = Ha phi + phi Hb: 2 x 2 waves of TM x TM tiles of 16 x 16, operands
// from memory to registers (a lane's four A values of a 16-deep block are 32
// contiguous bytes, the block's k taken in the order that makes them so; B
// reads 128-byte row segments), the next block's loads in flight during the
// current one's products.  The matrices' padding (to multiples of 16) is
// zero, so that a clamped operand beside it adds nothing.
template <int TM>
__global__ void __launch_bounds__(256) k_hx_same(const StateDesc* __restrict__ sd, CiMmArgs mm, int xs, int ntn,
                                                 int nblk) {
    int st, blk;
    if (!mm_place(xs, nblk, st, blk)) return;
    const StateDesc& s = sd[st];
    const int NA = mm.na_str, NB = mm.nb_str, NAp = mm.na_pad, NBp = mm.nb_pad;
    const double* __restrict__ phi = reinterpret_cast<const double*>(s.lam);
    const double* __restrict__ ha = s.ci_ha;
    const double* __restrict__ hb = s.ci_hb;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int i = lane & 15, g = lane >> 4;
    const int m0 = ((blk / ntn) * 2 + (w >> 1)) * 16 * TM, n0 = ((blk % ntn) * 2 + (w & 1)) * 16 * TM;
    if (m0 >= NA || n0 >= NB) return;   // no barriers below
    int mr[TM], mh[TM], nc[TM], nh[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        mr[t] = min(m0 + 16 * t + i, NA - 1);    // row of phi
        mh[t] = min(m0 + 16 * t + i, NAp - 1);   // row of Ha
        nc[t] = min(n0 + 16 * t + i, NB - 1);    // column of phi
        nh[t] = min(n0 + 16 * t + i, NBp - 1);   // column of Hb
    }
    d4 acc[TM][TM];
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TM; ++y) acc[x][y] = d4{0.0, 0.0, 0.0, 0.0};
    const int ka = NAp / 16, nk = ka + NBp / 16;
    auto load = [&](int kb, double (&a)[TM][4], double (&b)[TM][4]) {
        if (kb < ka) {
            const int k0 = kb * 16 + 4 * g;
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[t][j] = ldg64(ha + size_t(mh[t]) * NAp + k0 + j);
                    b[t][j] = ldg64(phi + size_t(min(k0 + j, NA - 1)) * NB + nc[t]);
                }
        } else {
            const int k0 = (kb - ka) * 16 + 4 * g;
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[t][j] = ldg64(phi + size_t(mr[t]) * NB + min(k0 + j, NB - 1));
                    b[t][j] = ldg64(hb + size_t(k0 + j) * NBp + nh[t]);
                }
        }
    };
    auto products = [&](const double (&a)[TM][4], const double (&b)[TM][4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int y = 0; y < TM; ++y) acc[x][y] = mfma64(a[x][j], b[y][j], acc[x][y]);
    };
    double a0[TM][4], b0[TM][4], a1[TM][4], b1[TM][4];
    load(0, a0, b0);
    int kb = 0;
    for (; kb + 2 <= nk; kb += 2) {
        load(kb + 1, a1, b1);
        products(a0, b0);
        load(kb + 2 < nk ? kb + 2 : nk - 1, a0, b0);
        products(a1, b1);
    }
    if (kb < nk) products(a0, b0);
    double* out = reinterpret_cast<double*>(s.aux);
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
        for (int y = 0; y < TM; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + 16 * x + 4 * v + g, n = n0 + 16 * y + i;
                if (m < NA && n < NB) stgv(out + size_t(m) * NB + n, acc[x][y][v]);
            }
}

// The same for sizes that leave the chip idle: one 16 x 16 tile per workgroup,
// its W waves take every W-th block of the inner dimension and their parts are
// added through LDS in wave order.
template <int W>
__global__ void __launch_bounds__(64 * W) k_hx_same_split(const StateDesc* __restrict__ sd, CiMmArgs mm, int xs,
                                                          int ntn, int nblk) {
    __shared__ double part[W][256];
    int st, blk;
    if (!mm_place(xs, nblk, st, blk)) return;
    const StateDesc& s = sd[st];
    const int NA = mm.na_str, NB = mm.nb_str, NAp = mm.na_pad, NBp = mm.nb_pad;
    const double* __restrict__ phi = reinterpret_cast<const double*>(s.lam);
    const double* __restrict__ ha = s.ci_ha;
    const double* __restrict__ hb = s.ci_hb;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int m0 = (blk / ntn) * 16, n0 = (blk % ntn) * 16;   // below NA and NB
    const int mr = min(m0 + i, NA - 1), nc = min(n0 + i, NB - 1);
    const int ka = NAp / 16, nk = ka + NBp / 16;
    auto load = [&](int kb, double (&a)[4], double (&b)[4]) {
        if (kb < ka) {
            const int k0 = kb * 16 + 4 * g;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = ldg64(ha + size_t(m0 + i) * NAp + k0 + j);
                b[j] = ldg64(phi + size_t(min(k0 + j, NA - 1)) * NB + nc);
            }
        } else {
            const int k0 = (kb - ka) * 16 + 4 * g;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = ldg64(phi + size_t(mr) * NB + min(k0 + j, NB - 1));
                b[j] = ldg64(hb + size_t(k0 + j) * NBp + n0 + i);
            }
        }
    };
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    constexpr int D = 4;   // blocks in flight
    double a[D][4], b[D][4];
#pragma unroll
    for (int u = 0; u < D; ++u) load(min(w + u * W, nk - 1), a[u], b[u]);
    for (int kb = w; kb < nk; kb += D * W) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (kb + u * W < nk) {
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = mfma64(a[u][j], b[u][j], acc);
            }
            load(min(kb + (u + D) * W, nk - 1), a[u], b[u]);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) part[w][v * 64 + lane] = acc[v];
    __syncthreads();
    double* out = reinterpret_cast<double*>(s.aux);
    for (int e = tid; e < 256; e += 64 * W) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < W; ++u) v += part[u][e];
        const int m = m0 + 4 * (e >> 6) + ((e & 63) >> 4), n = n0 + (e & 15);
        if (m < NA && n < NB) stgv(out + size_t(m) * NB + n, v);
    }
}

// One workgroup per row: W waves, each NT column tiles of 16, KS k-steps of 4
// (B in registers, read once).  The beta moves go in chunks of 16: a chunk's
// T (16 x columns) is formed, stored to LDS, and gathered by every column from
// its list of the chunk's moves.  The next chunk's rows of G (staged in LDS for
// the waves) and the chunk's list entries are read ahead.  One T buffer and at most 128 registers, so
// that up to 256 beta strings four workgroups share a compute unit and fill
// each other's waits.
template <int W, int NT, int KS>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4))) k_hx_cross(const StateDesc* __restrict__ sd, CiMmArgs mm, int xs) {
    constexpr int BS = 64 * W;
    constexpr int kList = W < 16 ? 12 : 4;   // list entries of a chunk held in registers
    constexpr int kStage = (64 * KS + BS - 1) / BS;
    extern __shared__ double sh_mm[];
    int st, ia;
    if (!mm_place(xs, mm.na_str, st, ia)) return;
    const StateDesc& s = sd[st];
    const int NB = mm.nb_str, TS = mm.t_stride, nch = mm.m_pad / 16;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    double* A = sh_mm;                // [2][4 KS][16]: a chunk's rows of G
    double* T = A + 128 * KS;         // [16][TS], then a zero
    double* red = T + 16 * TS + 1;    // [W]
    const double* __restrict__ phi = reinterpret_cast<const double*>(s.lam);
    const double* __restrict__ G = s.ci_g;
    // the row's inputs: partner row, row of G, sign (taken into B)
    const uint32_t* rl = mm.rows + size_t(ia) * mm.kpad;   // kpad = 4 KS
    uint32_t r[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) r[ks] = ldg32(rl + 4 * ks + g);
    // the thread's elements of A: input e / 16, beta move e % 16 of the chunk
    int ga[kStage];
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
        const int e = min(tid + BS * u, 64 * KS - 1);
        ga[u] = int((ldg32(rl + (e >> 4)) >> 16) & 0x3fffu) * mm.m_pad + (e & 15);
    }
    static_assert(NT * 16 * W <= BS, "a column per thread");
    const int cn = min(tid, NB - 1);   // the thread's column
    double* out = reinterpret_cast<double*>(s.aux) + size_t(ia) * NB;
    double sig = ldg64(out + cn);
    double B[NT][KS], av[kStage];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            B[t][ks] = ldg64(phi + size_t(r[ks] & 0xffffu) * NB + min((w * NT + t) * 16 + i, NB - 1));
#pragma unroll
    for (int u = 0; u < kStage; ++u) av[u] = ldg64(G + ga[u]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const double v = __hiloint2double(__double2hiint(B[t][ks]) ^ int(r[ks] & 0x80000000u), __double2loint(B[t][ks]));
            B[t][ks] = (r[ks] & kMmNone) ? 0.0 : v;
        }
    auto stage = [&](int buf) {
#pragma unroll
        for (int u = 0; u < kStage; ++u) A[buf * 64 * KS + min(tid + BS * u, 64 * KS - 1)] = av[u];
    };
    stage(0);
    if (tid == 0) T[16 * TS] = 0.0;
    const uint32_t* lst = mm.cols + cn;
    for (int ch = 0; ch < nch; ++ch) {
        // the chunk's list entries (a multiple of 4) and the next chunk of A, in
        // flight during the products
        const int ne = mm.cnt[ch];
        uint32_t en[kList];
        if constexpr (W < 16) {
#pragma unroll
            for (int q = 0; q < kList; q += 4)
                if (q < ne) {
#pragma unroll
                    for (int e = q; e < q + 4; ++e) en[e] = ldg32(lst + size_t(e) * NB);
                }
        }
        const int nx = (ch + 1 < nch ? ch + 1 : ch) * 16;
#pragma unroll
        for (int u = 0; u < kStage; ++u) av[u] = ldg64(G + ga[u] + nx);
        __syncthreads();   // A is there, the last chunk's T no longer read
        double a[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[ks] = A[(ch & 1) * 64 * KS + (4 * ks + g) * 16 + i];
        // one column tile after the other: the four waves of a SIMD hide each
        // other's dependent products, and one accumulator leaves the registers
        // that four need
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int c0 = (w * NT + t) * 16;
            if (c0 < TS) {
                d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma64(a[ks], B[t][ks], acc);
#pragma unroll
                for (int v = 0; v < 4; ++v) T[(4 * v + g) * TS + c0 + i] = acc[v];
            }
        }
        stage((ch + 1) & 1);
        __syncthreads();
        // list entry: 8 x the LDS element of T (from T's start; the zero past
        // T for padding), bit 0 the sign
        auto element = [&](uint32_t x) {
            const double v = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(T) + (x & ~7u));
            return __hiloint2double(__double2hiint(v) ^ int(x << 31), __double2loint(v));
        };
        if (w * 64 < NB) {
#pragma unroll
            for (int q = 0; q < (W < 16 ? kList : 0); q += 4)
                if (q < ne) {
                    const double v0 = element(en[q]), v1 = element(en[q + 1]), v2 = element(en[q + 2]),
                                 v3 = element(en[q + 3]);
                    sig += (v0 + v1) + (v2 + v3);
                }
            for (int e = W < 16 ? kList : 0; e < ne; e += 4) {
                uint32_t x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = ldg32(lst + size_t(e + u) * NB);
                sig += (element(x[0]) + element(x[1])) + (element(x[2]) + element(x[3]));
            }
        }
        lst += size_t(ne) * NB;
    }
    double acc = 0.0;
    if (tid < NB) {
        stgv(out + tid, sig);
        acc = ldg64(phi + size_t(ia) * NB + tid) * sig;
    }
    acc = wave_total(acc);
    if (lane == 0) red[w] = acc;
    __syncthreads();
    if (tid == 0) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < W; ++u) v += red[u];
        s.part_e[ia] = v;
    }
}

// Shapes: waves and column tiles per wave by the number of beta strings,
// k-steps by the row's moves.
#define VQE_MM_KS(X, W, NT) X(W, NT, 3) X(W, NT, 5) X(W, NT, 6) X(W, NT, 7) X(W, NT, 8) X(W, NT, 10) X(W, NT, 11)
#define VQE_MM_SHAPES(X) \
    VQE_MM_KS(X, 4, 1) VQE_MM_KS(X, 4, 2) VQE_MM_KS(X, 4, 4) VQE_MM_KS(X, 8, 4) VQE_MM_KS(X, 16, 4)

struct MmShape {
    int w, nt, ks;
    const void* fn;
};
#define VQE_MM_ENTRY(W, NT, KS) {W, NT, KS, reinterpret_cast<const void*>(&k_hx_cross<W, NT, KS>)},
static const MmShape kMmShapes[] = {VQE_MM_SHAPES(VQE_MM_ENTRY)};
#undef VQE_MM_ENTRY

static const MmShape* mm_shape(const CiMmArgs& mm) {
    const int ks = (mm.krow + 1 + 3) / 4;
    for (const MmShape& sh : kMmShapes)
        if (sh.w * sh.nt * 16 >= mm.nb_str && sh.ks >= ks) return &sh;   // ascending in both
    return nullptr;
}

static size_t mm_lds(const CiMmArgs& mm, const MmShape& sh) {
    return sizeof(double) * (size_t(128) * sh.ks + size_t(16) * mm.t_stride + 1 + sh.w);
}

int mm_prepare(CiMmArgs* mm) {
    const MmShape* sh = mm_shape(*mm);
    if (!sh) return 1;
    mm->kpad = 4 * sh->ks;
    const size_t lds = mm_lds(*mm, *sh);
    if (lds > size_t(160) << 10) return 1;
    if (lds > size_t(64) << 10 &&
        hipFuncSetAttribute(sh->fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10) != hipSuccess)
        return 1;
    return 0;
}

void launch_hx_mm(const StateDesc* sd, int count, const CiMmArgs& mm, hipStream_t st) {
    const MmShape* sh = mm_shape(mm);
    // (24 qubits: 4,536 states of 924 rows with 1,024 threads each)
    for (const int most = states_per_launch(int64_t(mm.na_str) * 64 * sh->w); count > most; count -= most, sd += most)
        launch_hx_mm(sd, most, mm, st);
    // 64 x 64 tiles when those fill the chip, else 16 x 16 with the inner
    // dimension split over the waves
    const int t64 = ((mm.na_str + 63) / 64) * ((mm.nb_str + 63) / 64);
    const bool big = int64_t(t64) * count >= 192;
    const int edge = big ? 64 : 16;
    const int ntm = (mm.na_str + edge - 1) / edge, ntn = (mm.nb_str + edge - 1) / edge;
    const int xs = count >= 8 ? count : 0;
    auto grid = [&](int nblk) {
        return xs ? dim3(unsigned(8 * ((count + 7) / 8) * nblk), 1, 1) : dim3(unsigned(nblk), unsigned(count), 1);
    };
    if (big)
        hipLaunchKernelGGL(k_hx_same<2>, grid(ntm * ntn), dim3(256), 0, st, sd, mm, xs, ntn, ntm * ntn);
    else
        hipLaunchKernelGGL(k_hx_same_split<4>, grid(ntm * ntn), dim3(256), 0, st, sd, mm, xs, ntn, ntm * ntn);
    const size_t lds = mm_lds(mm, *sh);
#define VQE_MM_LAUNCH(W, NT, KS)                                                                              \
    if (sh->w == W && sh->nt == NT && sh->ks == KS)                                                           \
        hipLaunchKernelGGL((k_hx_cross<W, NT, KS>), grid(mm.na_str), dim3(64 * W), lds, st, sd, mm, xs);
    VQE_MM_SHAPES(VQE_MM_LAUNCH)
#undef VQE_MM_LAUNCH
}

}  // namespace vqe
