// Ansatz passes of a whole state in one workgroup (Sec. 2.1.2; the objective
// of Sec. 2.1.1, Eq. 1, and its gradient by the reverse sweep), for sectors
// whose amplitudes fit one compute unit's LDS: real amplitudes in
// string-product order (alpha string times beta string), phi alone in the
// forward pass, phi and lambda side by side in the reverse sweep.
//
// Against the tiled runs of k_packed.hip this takes one launch per pass
// instead of one per run, no order conversions around the H-apply (it reads
// phi and writes lambda in this order), no staging between runs, and a gate's
// step covers all of its pairs at once.  What bounds a step: the wave's serial
// instruction stream (12 qubits, one or two waves: about 0.14 us forward, 0.2
// back), from 300 pairs on the LDS accesses (16 qubits: 0.19 and 0.34 us).
// Measured, forward + reverse, us, tiled runs -> whole states with a barrier
// and 8-byte entries per gate -> here: UCCSD 60 states of 14 qubits 99 -> 65,
// 16 qubits, one state 369 -> 203 -> 192; 17 qubits, 60 states 615 -> 349 -> 357,
// 400 states 1439 -> 677 -> 681; k-UpCCGSD (k = 2), 60 states, 16 qubits 304 ->
// 222 -> 169, 17 qubits 425 -> 361 -> 346.  (14 qubits: the first figure is the
// second form's.)
// Against the tiled runs' present form (its best threads and block bits), whole
// calls with gradient, us, here / tiled, 2 / 60 / 400 states: UCCSD 14 qubits 129 /
// 176, 136 / 193, 187 / 332; 15 qubits 161 / 217, 179 / 260, 315 / 517; 16 qubits
// 255 / 243, 289 / 329, 657 / 860; 17 qubits 418 / 282, 477 / 468, 1127 / 1456;
// k-UpCCGSD 16 qubits 231 / 253, 262 / 297, 596 / 803; 17 qubits 402 / 293, 461 / 436,
// 1104 / 1304; UCCSD on 20 qubits with 4 electrons (2,025 strings) 204 / 356, 216 /
// 390, 307 / 801.  So a state alone on its compute unit is slower here in the
// largest sectors only; lone states take tiles there (whole_as_tiles), batches
// are not told apart by their number of states.
#include "device_common.h"

#include <algorithm>

namespace vqe {

// LDS of both passes, dynamic and from address 0 on: the amplitudes (8 bytes
// in the forward pass, 16 in the reverse sweep), kWholeIdle dummies, the gates'
// (cos, sin) and one more.

using d2 = __attribute__((ext_vector_type(2))) double;

// LDS accesses by absolute address: the kernels have no static LDS, so their
// dynamic LDS starts at 0 and an entry's index times 8 or 16 is an address.
template <typename T>
__device__ __forceinline__ T whole_at(uint32_t off) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T*>(uintptr_t(off));
}
template <typename T>
__device__ __forceinline__ void whole_put(uint32_t off, T v) {
    *reinterpret_cast<__attribute__((address_space(3))) T*>(uintptr_t(off)) = v;
}

// One gate on N pairs of a thread: an entry is the pair's two indices, ordered
// so that its sign is +: a rotation by -s of (D, E) is one by s of (E, D).  The
// pairs of a gate are disjoint, so all are read before the first is written.
// Places without a pair rotate a dummy.
template <bool REVERSE, int N>
__device__ __forceinline__ void whole_pairs(const uint32_t* e, double c, double s, double& acc) {
    uint32_t p[N], q[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        p[u] = (e[u] & 0xffffu) << (REVERSE ? 4 : 3);
        q[u] = (e[u] >> 16) << (REVERSE ? 4 : 3);
    }
    if constexpr (!REVERSE) {
        double d[N], f[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            d[u] = whole_at<double>(p[u]);
            f[u] = whole_at<double>(q[u]);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            givens(d[u], f[u], c, s);
            whole_put(p[u], d[u]);
            whole_put(q[u], f[u]);
        }
    } else {
        d2 d[N], f[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            d[u] = whole_at<d2>(p[u]);
            f[u] = whole_at<d2>(q[u]);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            double fD = d[u].x, lD = d[u].y, fE = f[u].x, lE = f[u].y;
            // Re <lambda|A phi>: A|D> = |E>, A|E> = -|D>
            acc = fma(lE, fD, acc);
            acc = fma(-lD, fE, acc);
            givens(fD, fE, c, -s);   // U^dag
            givens(lD, lE, c, -s);
            whole_put(p[u], d2{fD, lD});
            whole_put(q[u], d2{fE, lE});
        }
    }
}

// Every gate of the program in order (REVERSE: backwards), segment by segment.
// As in the tiled runs, a wave's serial instruction stream is what a step
// costs, so a narrow gate's step (1, 2 or, up to 256 threads, 4 places per
// thread) has no branch but the one around the barrier, which only ends a
// stretch of gates (the waves own whole groups of strings, WaveSplit in
// vqe_device.hip): entries ent[(row * places + place) * BS + thread], row the
// gate's number among its segment's, are loaded kListAhead gates ahead into slot
// t % kListAhead, past the segment's ends too (unused).  A segment of wide gates:
// `passes` places per thread and gate, read and rotated kU at once, the next kU
// entries read meanwhile (each waits for its load: 16 qubits with 256 threads, 2
// places, 221 us forward this way).
// totals(n, acc, g): the threads' parts of the n gates g, g -+ 1, ... (n <= 8).
template <int BS, bool REVERSE, typename Totals>
__device__ __forceinline__ void whole_gates(const WholeArgs& w, const double2* par, Totals totals) {
    const int tid = threadIdx.x;
    auto step_end = [](bool meet) {   // nothing moves across: an address formed early waits for its entry
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_sched_barrier(0);
        if (BS == 1024 || __builtin_expect(meet, 0)) __syncthreads();   // (16 waves: after every gate)
        __builtin_amdgcn_sched_barrier(0);
    };
    // bit u: the waves meet after the u-th gate from g on in the pass
    auto meets = [&](int g) -> uint32_t {
        const int bit = REVERSE ? g : g + 8;   // w.meet's bit j + 8: between gates j and j + 1
        const uint64_t v = uint64_t(ldc(w.meet + (bit >> 5))) | uint64_t(ldc(w.meet + (bit >> 5) + 1)) << 32;
        const uint32_t m = uint32_t(v >> (bit & 31)) & 0xffu;
        return REVERSE ? __builtin_bitreverse32(m) >> 24 : m;   // gate g - u: between g - u - 1 and g - u
    };
    auto narrow = [&](const WholeSeg& sg, auto places) {
        constexpr int NP = decltype(places)::value;
        constexpr uint32_t rowb = NP * BS * 4u;
        const int ng = sg.g1 - sg.g0;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(w.ent + sg.ent - kListAhead * NP * BS), 0,
                                              int(uint32_t(ng + 2 * kListAhead) * rowb), 0x00020000);
        const uint32_t voff = uint32_t(tid) * 4u;
        uint32_t row = uint32_t(kListAhead + (REVERSE ? ng - 1 : 0)) * rowb;   // of the next load
        uint32_t eq[kListAhead][NP];
        auto load = [&](uint32_t (&e)[NP]) {
#pragma unroll
            for (int v = 0; v < NP; ++v)
                e[v] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff + uint32_t(v) * BS * 4u, row, 0);
            row += REVERSE ? 0u - rowb : rowb;
        };
#pragma unroll
        for (int d = 0; d < kListAhead; ++d) load(eq[d]);
        const int first = REVERSE ? sg.g1 - 1 : sg.g0;
        double2 cs_ahead = par[first];
        auto round = [&](int t0, auto full_tag) {
            constexpr bool FULL = decltype(full_tag)::value;
            const int g = REVERSE ? first - t0 : first + t0;
            const uint32_t meet = meets(g);
            double acc[8];
            unroll_n<8>([&](auto uu) {
                constexpr int u = decltype(uu)::value;
                acc[u] = 0.0;
                if (FULL || t0 + u < ng) {
                    const double2 cs = cs_ahead;
                    cs_ahead = par[g + (REVERSE ? -(u + 1) : u + 1)];   // (past the segment: unused)
                    // (16 waves: divided in order, the last ones often without a pair)
                    if (BS < 1024 || (uint32_t(__builtin_amdgcn_readfirstlane(int(eq[u][0]))) & 0xffffu) < uint32_t(w.nE))
                        whole_pairs<REVERSE, NP>(eq[u], cs.x, cs.y, acc[u]);
                    // (formed here, not where it is used)
                    if constexpr (REVERSE) __asm__ volatile("" : "+v"(acc[u]));
                    load(eq[u]);
                    step_end((meet >> u) & 1u);
                }
            });
            totals(FULL ? 8 : ng - t0, acc, g);
        };
        static_assert(kListAhead == 8, "a round of slots is a batch of totals");
        int t0 = 0;
        for (; t0 + 8 <= ng; t0 += 8) round(t0, std::true_type{});
        if (t0 < ng) round(t0, std::false_type{});
    };
    for (int si = 0; si < w.nseg; ++si) {
        const WholeSeg sg = ldc(w.seg + (REVERSE ? w.nseg - 1 - si : si));
        const int ng = sg.g1 - sg.g0;
        const uint32_t* ent = w.ent + sg.ent;
        if (sg.passes == 1) {
            narrow(sg, std::integral_constant<int, 1>{});
        } else if (sg.passes == 2) {
            narrow(sg, std::integral_constant<int, 2>{});
        } else if (BS <= 256 && sg.passes == 4) {
            narrow(sg, std::integral_constant<int, 4>{});
        } else {
            constexpr int kU = 4;   // pairs in flight per thread
            const int np = sg.passes;
            auto row = [&](int t) { return REVERSE ? ng - 1 - t : t; };
            uint32_t next[kU];
            auto fetch = [&](int t, int u0, uint32_t (&e)[kU]) {
                const uint32_t* l = ent + size_t(row(t)) * np * BS + tid;
#pragma unroll
                for (int u = 0; u < kU; ++u) e[u] = l[min(u0 + u, np - 1) * BS];
            };
            fetch(0, 0, next);
            for (int t = 0; t < ng; ++t) {
                const int g = sg.g0 + row(t);
                const double2 cs = par[g];
                double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                for (int u0 = 0; u0 < np; u0 += kU) {
                    uint32_t cur[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) cur[u] = next[u];
                    const bool last = u0 + kU >= np;
                    fetch(last ? min(t + 1, ng - 1) : t, last ? 0 : u0 + kU, next);
                    // (the wave's places are filled in order)
                    if ((uint32_t(__builtin_amdgcn_readfirstlane(int(cur[0]))) & 0xffffu) >= uint32_t(w.nE)) continue;
                    const int n = min(np - u0, kU);
                    if (n == 4) whole_pairs<REVERSE, 4>(cur, cs.x, cs.y, acc[0]);
                    else if (n == 3) whole_pairs<REVERSE, 3>(cur, cs.x, cs.y, acc[0]);
                    else if (n == 2) whole_pairs<REVERSE, 2>(cur, cs.x, cs.y, acc[0]);
                    else whole_pairs<REVERSE, 1>(cur, cs.x, cs.y, acc[0]);
                }
                step_end(meets(g) & 1u);
                totals(1, acc, g);
            }
        }
    }
    __syncthreads();
}

template <int BS>
__global__ void __launch_bounds__(BS) k_whole_fwd(const StateDesc* __restrict__ sd, WholeArgs w) {
    extern __shared__ __align__(16) unsigned char lds_whole[];
    const StateDesc& s = sd[blockIdx.x];
    const int tid = threadIdx.x;
    double* psi = reinterpret_cast<double*>(lds_whole);                    // [nE + kWholeIdle]
    double2* par = reinterpret_cast<double2*>(psi + w.nE + kWholeIdle + (w.nE & 1));   // [M + 1] (cos, sin)
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
// The wave totals of up to eight gates are taken at once (wave_totals8) into
// part_g, the waves summed after the last gate; the energy's partials are
// summed by the first wave.
template <int BS>
__global__ void __launch_bounds__(BS) k_whole_adj(const StateDesc* __restrict__ sd, WholeArgs w, int nplanes,
                                                  int nblk_e) {
    extern __shared__ __align__(16) unsigned char lds_whole[];
    constexpr int kW = BS / 64;
    const StateDesc& s = sd[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    double2* pl = reinterpret_cast<double2*>(lds_whole);                   // [nE + kWholeIdle] (phi, lambda)
    double2* par = pl + w.nE + kWholeIdle;                                 // [M + 1]
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
    whole_gates<BS, true>(w, par, [&](int n, const double (&acc)[8], int g) {
        const double tot = wave_totals8(acc, lane);
        const int u = lane >> 3;
        if ((lane & 7) == 0 && u < n) s.part_g[size_t(g - u) * kWholeWaves + (tid >> 6)] = tot;
    });
    for (int j = tid; j < w.M; j += BS) {
        double v = 0.0;
#pragma unroll
        for (int u = 0; u < kW; ++u) v += s.part_g[size_t(j) * kWholeWaves + u];
        s.out_g[j] = v;
    }
}

static size_t whole_lds(int nE, int M, bool adj) {
    return size_t(nE + kWholeIdle + (nE & 1)) * (adj ? 16 : 8) + size_t(M + 1) * sizeof(double2);
}

#define VQE_WHOLE_SIZES(X) X(64) X(128) X(256) X(512) X(1024)

// Threads of both passes for gates of cnt[0 .. M) pairs, by the clocks of the
// gate steps: 200 for a wave's step of one place, 50 for each further one, 35
// of the LDS pipe for each wave and place, with a wave's places 85% filled; 16
// waves (1,024 threads) divide every gate in order, meet after each (150) and
// skip waves without a pair.  Measured, forward + reverse, us: 60 states of 14
// qubits with 64 / 128 / 256 / 512 threads 112 / 65 / 65 / 76, 15 qubits 212 / 145 / 96
// / 114, 16 qubits with 128 / 256 / 512 279 / 212 / 195; 400 states of 17 qubits 512
// threads 792, 1,024 with owned groups 794, divided in order 677.
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
            const int nw = x.bs / 64, fill = nw == 1 ? 64 : nw == 16 ? 1024 : x.bs * 85 / 100;
            const int per = std::max(1, (cnt[j] + fill - 1) / fill);
            const int places = nw == 16 ? (cnt[j] + 63) / 64 : nw * per;
            t += 150.0 + 50.0 * per + 35.0 * places + (nw == 16 ? 150.0 : 0.0);
        }
        if (sh == nullptr || t < best) {
            best = t;
            sh = &x;
        }
    }
    *threads = sh->bs;
    if (nE > kWholeMax || whole_lds(nE, M, true) > size_t(160) << 10) return 1;
    for (const void* f : {sh->fwd, sh->adj})
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10) != hipSuccess) return 1;
    return 0;
}

void launch_whole(const StateDesc* sd, int count, const WholeArgs& w, bool adj, int nplanes, int nblk_e,
                  hipStream_t st) {
    const size_t lds = whole_lds(w.nE, w.M, adj);
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
