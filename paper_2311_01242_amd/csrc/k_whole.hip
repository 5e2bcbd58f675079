// Ansatz passes of a whole state in one workgroup (Sec. 2.1.2; the objective
// of Sec. 2.1.1, Eq. 1, and its gradient by the reverse sweep), for sectors
// whose amplitudes fit one compute unit's LDS: real amplitudes in
// string-product order (alpha string times beta string), phi alone in the
// forward pass, phi and lambda side by side in the reverse sweep.
//
// Against the tiled runs of k_packed.hip this takes one launch per pass
// instead of one per run, no order conversions around the H-apply (it reads
// phi and writes lambda in this order), no staging between runs, and a gate's
// step covers all of its pairs at once: a step costs its chain (LDS read,
// rotation, LDS write, barrier: about 0.2 us forward and 0.35 us back at 16
// qubits) almost whatever the number of pairs, so wide steps are the cheap
// ones.  Measured, forward + reverse, tiled runs -> here: UCCSD 16 qubits, one
// state 170 + 199 -> 73 + 130 us; 17 qubits, 60 states 261 + 354 -> 125 + 224,
// 400 states 525 + 914 -> 216 + 461; k-UpCCGSD (k = 2) 17 qubits, 60 states
// 177 + 248 -> 117 + 244.  No size was found where the tiled runs win.
#include "device_common.h"

namespace vqe {

// LDS of both passes, dynamic and from address 0 on: the amplitudes (8 bytes
// in the forward pass, 16 in the reverse sweep), kWholeIdle dummies, the gates'
// (cos, sin), and in the reverse sweep the waves' totals.
constexpr int kWholeAhead = 4;   // gates a list entry is loaded ahead

using u32x2 = __attribute__((ext_vector_type(2))) uint32_t;
using d2 = __attribute__((ext_vector_type(2))) double;

// LDS accesses by absolute address: the kernels have no static LDS, so their
// dynamic LDS starts at 0 and an entry is an address as it is.
template <typename T>
__device__ __forceinline__ T whole_at(uint32_t off) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T*>(uintptr_t(off));
}
template <typename T>
__device__ __forceinline__ void whole_put(uint32_t off, T v) {
    *reinterpret_cast<__attribute__((address_space(3))) T*>(uintptr_t(off)) = v;
}

// One gate on N pairs of a thread: an entry is two LDS offsets (in units of 8
// bytes; an amplitude's slot), the pair ordered so that its sign is +: a
// rotation by -s of (D, E) is one by s of (E, D).  The pairs of a gate are
// disjoint, so all are read before the first is written.  Lanes without a pair
// rotate a dummy (no mask between the barrier and the reads); the entries
// fill the lanes in order, so a wave whose first lane has a dummy has nothing
// to do (`idle`: the dummies' first offset).
template <bool REVERSE, int N>
__device__ __forceinline__ void whole_pairs(const u32x2* e, double c, double s, uint32_t idle, double& acc) {
    if (uint32_t(__builtin_amdgcn_readfirstlane(int(e[0].x))) >= idle) return;
    if constexpr (!REVERSE) {
        double d[N], f[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            d[u] = whole_at<double>(e[u].x);
            f[u] = whole_at<double>(e[u].y);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            givens(d[u], f[u], c, s);
            whole_put(e[u].x, d[u]);
            whole_put(e[u].y, f[u]);
        }
    } else {
        d2 d[N], f[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            d[u] = whole_at<d2>(e[u].x * 2u);
            f[u] = whole_at<d2>(e[u].y * 2u);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            double fD = d[u].x, lD = d[u].y, fE = f[u].x, lE = f[u].y;
            // Re <lambda|A phi>: A|D> = |E>, A|E> = -|D>
            acc = fma(lE, fD, acc);
            acc = fma(-lD, fE, acc);
            givens(fD, fE, c, -s);   // U^dag
            givens(lD, lE, c, -s);
            whole_put(e[u].x * 2u, d2{fD, lD});
            whole_put(e[u].y * 2u, d2{fE, lE});
        }
    }
}

// Every gate of the program in order (REVERSE: backwards), segment by segment.
// A segment of narrow gates (passes == 0): at most one pair per thread and
// gate, entries ent[row * BS + thread], row the gate's number among its
// segment's, loaded kWholeAhead gates ahead into slot t % kWholeAhead (the
// loop is unrolled and free of other loads, so that a gate waits for its own
// slot only).  A segment of wide gates: `passes` pairs per thread and gate,
// read and rotated kU at once, the next kU entries read meanwhile.
// totals(n, acc, g): the threads' parts of the n gates g, g -+ 1, ... (n <= 8).
template <int BS, bool REVERSE, typename Totals>
__device__ __forceinline__ void whole_gates(const WholeArgs& w, const double2* par, Totals totals) {
    const int tid = threadIdx.x;
    const uint32_t idle = 8u * uint32_t(w.nE);
    // nothing moves across: an address formed gates early waits for its entry
    auto barrier = [] {
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int si = 0; si < w.nseg; ++si) {
        const WholeSeg sg = ldc(w.seg + (REVERSE ? w.nseg - 1 - si : si));
        const int ng = sg.g1 - sg.g0;
        const u32x2* ent = reinterpret_cast<const u32x2*>(w.ent) + sg.ent;
        auto row = [&](int t) { return REVERSE ? ng - 1 - t : t; };
        auto gate = [&](int t) { return sg.g0 + row(t); };
        if (sg.passes == 0) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<u32x2*>(ent), 0, int(uint32_t(ng) * uint32_t(BS * 8)), 0x00020000);
            const uint32_t voff = uint32_t(tid) * 8u;
            u32x2 eq[kWholeAhead];
            auto load = [&](int t, u32x2& e) {   // clamped at the end: reloaded, unused
                e = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, uint32_t(row(min(t, ng - 1))) * uint32_t(BS * 8), 0);
            };
#pragma unroll
            for (int d = 0; d < kWholeAhead; ++d) load(d, eq[d]);
            double2 cs_next = par[gate(0)];
            auto step = [&](int t, auto slot, double& acc) {
                constexpr int q = decltype(slot)::value % kWholeAhead;
                const double2 cs = cs_next;
                cs_next = par[gate(min(t + 1, ng - 1))];
                acc = 0.0;
                whole_pairs<REVERSE, 1>(&eq[q], cs.x, cs.y, idle, acc);
                load(t + kWholeAhead, eq[q]);
                barrier();
            };
            int t0 = 0;
            for (; t0 + 8 <= ng; t0 += 8) {
                double acc[8];
                unroll_n<8>([&](auto slot) { step(t0 + decltype(slot)::value, slot, acc[decltype(slot)::value]); });
                totals(8, acc, gate(t0));
            }
            if (t0 < ng) {
                double acc[8];
                unroll_n<8>([&](auto slot) {
                    constexpr int u = decltype(slot)::value;
                    acc[u] = 0.0;
                    if (t0 + u < ng) step(t0 + u, slot, acc[u]);
                });
                totals(ng - t0, acc, gate(t0));
            }
        } else {
            constexpr int kU = 4;   // pairs in flight per thread
            const int np = sg.passes;
            u32x2 next[kU];
            auto fetch = [&](int t, int u0, u32x2 (&e)[kU]) {
                const u32x2* l = ent + size_t(row(t)) * np * BS + tid;
#pragma unroll
                for (int u = 0; u < kU; ++u) e[u] = l[min(u0 + u, np - 1) * BS];
            };
            fetch(0, 0, next);
            for (int t = 0; t < ng; ++t) {
                const double2 cs = par[gate(t)];
                double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                for (int u0 = 0; u0 < np; u0 += kU) {
                    u32x2 cur[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) cur[u] = next[u];
                    const bool last = u0 + kU >= np;
                    fetch(last ? min(t + 1, ng - 1) : t, last ? 0 : u0 + kU, next);
                    const int n = min(np - u0, kU);
                    if (n == 4) whole_pairs<REVERSE, 4>(cur, cs.x, cs.y, idle, acc[0]);
                    else if (n == 3) whole_pairs<REVERSE, 3>(cur, cs.x, cs.y, idle, acc[0]);
                    else if (n == 2) whole_pairs<REVERSE, 2>(cur, cs.x, cs.y, idle, acc[0]);
                    else whole_pairs<REVERSE, 1>(cur, cs.x, cs.y, idle, acc[0]);
                }
                barrier();
                totals(1, acc, gate(t));
            }
        }
    }
}

template <int BS>
__global__ void __launch_bounds__(BS) k_whole_fwd(const StateDesc* __restrict__ sd, WholeArgs w) {
    extern __shared__ __align__(16) unsigned char lds_whole[];
    const StateDesc& s = sd[blockIdx.x];
    const int tid = threadIdx.x;
    double* psi = reinterpret_cast<double*>(lds_whole);                    // [nE + kWholeIdle]
    double2* par = reinterpret_cast<double2*>(psi + w.nE + kWholeIdle);    // [M] (cos, sin)
    for (int j = tid; j < w.M; j += BS) {
        const GateDesc g = s.gates[j];
        double sn, c;
        sincos(g.scale * s.theta[g.param], &sn, &c);
        par[j] = make_double2(c, sn);
        stg2(s.cs + j, make_double2(c, sn));   // the reverse sweep's
    }
    for (int k = tid; k < w.nE + kWholeIdle; k += BS) psi[k] = k == w.ref ? (w.ref_neg ? -1.0 : 1.0) : 0.0;
    __syncthreads();
    whole_gates<BS, false>(w, par, [](int, const double (&)[8], int) {});
    double* out = reinterpret_cast<double*>(s.lam);   // where the H-apply reads phi
    for (int k = tid; k < w.nE; k += BS) stgv(out + k, psi[k]);
}

// Reverse sweep: per gate Re <lambda|A_j phi>, then U_j^dag on both vectors.
// The wave totals of up to eight gates are taken at once (wave_totals8) and
// summed over the waves at the next call, barriers in between; the energy's
// partials are summed by the first wave.
template <int BS>
__global__ void __launch_bounds__(BS) k_whole_adj(const StateDesc* __restrict__ sd, WholeArgs w, int nplanes,
                                                  int nblk_e) {
    extern __shared__ __align__(16) unsigned char lds_whole[];
    constexpr int kW = BS / 64;
    const StateDesc& s = sd[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    double2* pl = reinterpret_cast<double2*>(lds_whole);                   // [nE + kWholeIdle] (phi, lambda)
    double2* par = pl + w.nE + kWholeIdle;                                 // [M]
    double* red = reinterpret_cast<double*>(par + w.M);                    // [2][8][kW]
    const double* phi = reinterpret_cast<const double*>(s.lam);
    const double* lam = reinterpret_cast<const double*>(s.aux);
    for (int j = tid; j < w.M; j += BS) par[j] = ldg2(s.cs + j);
    for (int k = tid; k < w.nE; k += BS) {
        double l = ldg64(lam + k);
        for (int z = 1; z < nplanes; ++z) l += ldg64(lam + size_t(z) * w.nE + k);
        pl[k] = make_double2(ldg64(phi + k), l);
    }
    for (int k = tid; k < kWholeIdle; k += BS) pl[w.nE + k] = make_double2(0.0, 0.0);
    if (tid < 64) {
        double e = 0.0;
        for (int b = lane; b < nblk_e; b += 64) e += s.part_e[b];
        e = wave_total(e);
        if (lane == 0) s.out_e[0] = e;
    }
    __syncthreads();
    int n_prev = 0, g_prev = 0, buf = 0;
    auto collect = [&]() {   // the gates of the last call; thread u adds gate u's waves
        if (tid < n_prev) {
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < kW; ++u) v += red[((buf ^ 1) * 8 + tid) * kW + u];
            s.out_g[g_prev - tid] = v;
        }
    };
    whole_gates<BS, true>(w, par, [&](int n, const double (&acc)[8], int g) {
        const double tot = wave_totals8(acc, lane);
        if ((tid & 7) == 0) red[(buf * 8 + (lane >> 3)) * kW + (tid >> 6)] = tot;
        collect();   // a barrier has passed since its totals were written
        n_prev = n;
        g_prev = g;
        buf ^= 1;
    });
    __syncthreads();
    collect();
}

static size_t whole_lds(int nE, int M, int threads, bool adj) {
    return size_t(nE + kWholeIdle) * (adj ? 16 : 8) + size_t(M) * sizeof(double2) +
           (adj ? 2 * 8 * size_t(threads / 64) * sizeof(double) : 0);
}

#define VQE_WHOLE_SIZES(X) X(64) X(128) X(256) X(512) X(1024)

// Threads of both passes for gates of cnt[0 .. M) pairs: the fewest clocks of
// the gate steps, a step taken as a chain of 300 for each kU pairs of a thread
// and 25 of the LDS pipe for each wave with a pair, and 10 for each wave at
// the barrier.
int whole_prepare(int nE, int M, const int* cnt, int* threads) {
    struct Shape {
        int bs;
        const void *fwd, *adj;
    };
#define VQE_WHOLE_ENTRY(BS) \
    {BS, reinterpret_cast<const void*>(&k_whole_fwd<BS>), reinterpret_cast<const void*>(&k_whole_adj<BS>)},
    static const Shape shapes[] = {VQE_WHOLE_SIZES(VQE_WHOLE_ENTRY)};
#undef VQE_WHOLE_ENTRY
    const Shape* sh = nullptr;
    double best = 0.0;
    for (const Shape& x : shapes) {
        double t = 0.0;
        for (int j = 0; j < M; ++j) {
            const int per = (cnt[j] + x.bs - 1) / x.bs;
            t += 300.0 * ((per + 3) / 4) + 25.0 * ((cnt[j] + 63) / 64) + 10.0 * (x.bs / 64) + (per > 1 ? 150.0 : 0.0);
        }
        if (sh == nullptr || t < best) {
            best = t;
            sh = &x;
        }
    }
    *threads = sh->bs;
    if (nE > kWholeMax || whole_lds(nE, M, sh->bs, true) > size_t(160) << 10) return 1;
    for (const void* f : {sh->fwd, sh->adj})
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10) != hipSuccess) return 1;
    return 0;
}

void launch_whole(const StateDesc* sd, int count, const WholeArgs& w, bool adj, int nplanes, int nblk_e,
                  hipStream_t st) {
    const size_t lds = whole_lds(w.nE, w.M, w.threads, adj);
#define VQE_WHOLE_LAUNCH(BS)                                                                                \
    if (w.threads == BS) {                                                                                  \
        if (adj)                                                                                            \
            hipLaunchKernelGGL((k_whole_adj<BS>), dim3(count), dim3(BS), lds, st, sd, w, nplanes, nblk_e);  \
        else                                                                                                \
            hipLaunchKernelGGL((k_whole_fwd<BS>), dim3(count), dim3(BS), lds, st, sd, w);                   \
    }
    VQE_WHOLE_SIZES(VQE_WHOLE_LAUNCH)
#undef VQE_WHOLE_LAUNCH
}

}  // namespace vqe
