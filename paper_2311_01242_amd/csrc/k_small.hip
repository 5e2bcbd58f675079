// Whole-state evaluation in one workgroup for programs that conserve the
// number of set qubits (Sec. 2.1.1, Eq. 1 and its gradient): the pUCCD
// ansatz in the hard-core-boson form (qubit p = spatial orbital p occupied by
// a pair; its pair moves change the pair count of no state) conserves the
// number of pairs k, so a state prepared from the reference lives on the
// C(n, k) strings of k set qubits.  When that sector is small, a state's
// amplitudes on it (ranked in increasing string order) fit one workgroup's
// LDS, and the forward pass, the H-apply and the reverse sweep each run in
// one workgroup per state.  Everything a phase reads more than once (the
// strings, the rank table, the gates with their angles, the Hamiltonian's
// tables) is staged in LDS first with wide loads, so the per-gate and
// per-term steps touch no memory outside the workgroup.
//
// A gate pairs D (its annihilated qubits set, its created ones clear) with
// E = D ^ x by a Givens rotation whose sign is csign (-1)^{|D & chain|}; the
// thread holding D's rank updates both amplitudes, the pairs of one gate are
// disjoint, and one barrier separates gates.  lambda = H phi is formed on the
// sector only: output string b takes, for every subgroup of every x-group of
// H, the subgroup's term at b times phi at b ^ x when that string is in the
// sector (E and the gradient need lambda on the sector only, as phi and A_j
// phi live there).  The H-apply splits each string's subgroups over several
// threads when the workgroup has more threads than the sector has strings,
// and adds the parts in a fixed order.  The H-apply writes the energy and the
// reverse sweep the per-gate gradient sums directly (no separate reduction
// launches).  Amplitudes are real (double) or complex (double2), as the rest
// of the sector paths: the pair moves are real rotations and H is a real
// matrix.
#include <mutex>

#include "device_common.h"

namespace vqe {

constexpr int kSmallThreads = 256;   // forward pass and reverse sweep
constexpr int kSmallHxThreads = 1024;
constexpr int kSmallMaxSlices = 8;   // threads per string in the H-apply

static_assert(sizeof(GroupDesc) == 16 && sizeof(SubDesc) == 8, "descriptor sizes staged in LDS");

// A gate as the kernels use it: masks, sign, and its (cos, sin).
struct SmallGate {
    uint32_t x, pd, chain;
    float csign;
    double c, s;
};
static_assert(sizeof(SmallGate) == 32, "SmallGate layout");

// A term of the staged Hamiltonian: flip (bit 15: leads out of the sector)
// and sign mask, and its table.
struct SmallTerm {
    uint32_t xw, pos;
    int32_t tab;
};
static_assert(kSmallMaxN <= 15, "a term's masks have 15 bits");

__host__ __device__ inline size_t small_r16(size_t v) { return (v + 15) & ~size_t(15); }

// Threads per string in the H-apply.
__host__ __device__ inline int small_slices(int nsec) {
    const int s = kSmallHxThreads / (nsec > 0 ? nsec : 1);
    return s < 1 ? 1 : (s > kSmallMaxSlices ? kSmallMaxSlices : s);
}

// Copy nbytes (even) from global memory to LDS, both 16-byte aligned: 16-byte
// pieces with four loads per thread issued before their stores, then the
// remainder in 2-byte pieces.
template <int NT>
__device__ __forceinline__ void small_copy(void* dst, const void* src, size_t nbytes) {
    const uint4* s4 = static_cast<const uint4*>(src);
    uint4* d4 = static_cast<uint4*>(dst);
    const int n16 = int(nbytes >> 4);
    int t = threadIdx.x;
    for (; t + 3 * NT < n16; t += 4 * NT) {
        const uint4 a = s4[t], b = s4[t + NT], c = s4[t + 2 * NT], d = s4[t + 3 * NT];
        d4[t] = a;
        d4[t + NT] = b;
        d4[t + 2 * NT] = c;
        d4[t + 3 * NT] = d;
    }
    for (; t < n16; t += NT) d4[t] = s4[t];
    const int rem = int(nbytes & 15) >> 1;
    if (int(threadIdx.x) < rem) {
        const size_t o = (size_t(n16) << 3) + threadIdx.x;   // in 2-byte units
        static_cast<uint16_t*>(dst)[o] = static_cast<const uint16_t*>(src)[o];
    }
}

// Fixed-order workgroup total of NT threads: wave totals, then every thread
// adds them in wave order.  Contains barriers: every thread calls it.
template <int NT>
__device__ __forceinline__ double small_block_total(double v, double* red) {
    v = wave_total(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) r += red[i];
    __syncthreads();
    return r;
}

// LDS layout (byte offsets, every region 16-byte aligned): amplitude
// vectors, H-apply partial sums, gates, Hamiltonian, rank table, strings.
struct SmallLayout {
    size_t vec, part, gates, ham, rank, str, total;
};

enum SmallPhase { kSmallFwd = 0, kSmallHx = 1, kSmallAdj = 2 };

__host__ __device__ inline SmallLayout small_layout(const SmallSpace& sp, int phase) {
    SmallLayout l;
    const size_t vbytes = size_t(sp.vbytes) * size_t(sp.nsec);   // one vector's amplitudes
    l.vec = 0;
    l.part = l.vec + (phase == kSmallAdj ? 2 : 1) * small_r16(vbytes);   // phi [, lambda]
    const int sl = small_slices(sp.nsec);
    l.gates = l.part + (phase == kSmallHx && sl > 1 ? small_r16(size_t(sl) * vbytes) : 0);
    l.ham = l.gates + (phase == kSmallHx ? 0 : sizeof(SmallGate) * size_t(sp.M));
    l.rank = l.ham + (phase == kSmallHx ? small_r16(size_t(sp.ham_lds)) : 0);
    l.str = l.rank + small_r16(2 * (size_t(1) << sp.n));
    l.total = l.str + small_r16(4 * size_t(sp.nsec));
    return l;
}

// Stage the sector's strings and the rank table into LDS.
template <int NT>
__device__ __forceinline__ void small_stage_space(const SmallSpace& sp, uint32_t* str, int16_t* rank) {
    small_copy<NT>(str, sp.str, 4 * size_t(sp.nsec));
    small_copy<NT>(rank, sp.rank, 2 * (size_t(1) << sp.n));
}

// What a thread needs of a gate besides the amplitudes: the partner of each of
// its KT strings (rank, or -1 when the string is no D of the gate) and the
// sign.  It depends on nothing the gates change, so it is looked up one gate
// ahead, beside the current gate's pairs: what bounds a step is its chain of
// LDS reads (string, rank, amplitudes).  512 states of 11 orbitals and 7 pairs
// (330 strings, 28 gates): forward 15.2 -> 13.3 us, reverse 19.3 -> 16.0; most of
// the rest is the staging's loads.
constexpr uint32_t kSmallNone = ~0u;
template <int KT>
struct SmallPairs {
    double c, s;
    int re[KT];
    bool neg[KT];
    __device__ __forceinline__ void find(const SmallGate& g, const uint32_t (&str)[KT], const int16_t* rank) {
        c = g.c;
        s = g.s;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const bool hit = str[k] != kSmallNone && (str[k] & g.x) == g.pd;
            const int r = rank[hit ? str[k] ^ g.x : 0u];
            re[k] = hit ? r : -1;
            neg[k] = (__popc(str[k] & g.chain) & 1) != (g.csign < 0.0f);
        }
    }
};

// The thread's strings t, t + kSmallThreads, ...; kSmallNone past the sector.
template <int KT>
__device__ __forceinline__ void small_strings(const uint32_t* str, int nsec, uint32_t (&mine)[KT]) {
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int t = int(threadIdx.x) + k * kSmallThreads;
        mine[k] = t < nsec ? str[t] : kSmallNone;
    }
}

// Forward pass: |ref> then U_M ... U_1; phi and the gates' (cos, sin) out.
template <typename V, int KT>
__global__ void __launch_bounds__(kSmallThreads) k_small_fwd(const StateDesc* __restrict__ sd, SmallSpace sp) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallLayout L = small_layout(sp, kSmallFwd);
    const StateDesc& s = sd[blockIdx.y];
    V* psi = reinterpret_cast<V*>(smem + L.vec);
    SmallGate* gs = reinterpret_cast<SmallGate*>(smem + L.gates);
    uint32_t* str = reinterpret_cast<uint32_t*>(smem + L.str);
    int16_t* rank = reinterpret_cast<int16_t*>(smem + L.rank);
    small_stage_space<kSmallThreads>(sp, str, rank);
    for (int t = threadIdx.x; t < sp.nsec; t += kSmallThreads)
        psi[t] = t == sp.ref_rank ? vunit(V{}) : vzero<V>();
    for (int j = threadIdx.x; j < s.M; j += kSmallThreads) {
        const GateDesc g = s.gates[j];
        double sn, c;
        sincos(g.scale * s.theta[g.param], &sn, &c);
        s.cs[j] = make_double2(c, sn);
        gs[j] = SmallGate{g.x, g.pd, g.chain, float(g.csign), c, sn};
    }
    __syncthreads();
    uint32_t mine[KT];
    small_strings<KT>(str, sp.nsec, mine);
    SmallPairs<KT> cur, next;
    if (s.M > 0) cur.find(gs[0], mine, rank);
    for (int j = 0; j < s.M; ++j) {
        next.find(gs[min(j + 1, s.M - 1)], mine, rank);
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const int t = int(threadIdx.x) + k * kSmallThreads;
            if (cur.re[k] >= 0) {
                V a = psi[t], b = psi[cur.re[k]];
                givens(a, b, cur.c, cur.neg[k] ? -cur.s : cur.s);
                psi[t] = a;
                psi[cur.re[k]] = b;
            }
        }
        __syncthreads();
        cur = next;
    }
    V* phi = reinterpret_cast<V*>(s.phi);
    for (int t = threadIdx.x; t < sp.nsec; t += kSmallThreads) phi[t] = psi[t];
}

// lambda = H phi on the sector, and E = Re <phi|lambda> into out_e.
template <typename V>
__global__ void __launch_bounds__(kSmallHxThreads) k_small_hx(const StateDesc* __restrict__ sd, SmallSpace sp) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallLayout L = small_layout(sp, kSmallHx);
    double* red = reinterpret_cast<double*>(smem + L.total);   // [waves]
    const StateDesc& s = sd[blockIdx.y];
    const int nsec = sp.nsec;
    V* psi = reinterpret_cast<V*>(smem + L.vec);
    V* part = reinterpret_cast<V*>(smem + L.part);
    V* lam = reinterpret_cast<V*>(s.lam);
    uint32_t* str = reinterpret_cast<uint32_t*>(smem + L.str);
    int16_t* rank = reinterpret_cast<int16_t*>(smem + L.rank);
    small_stage_space<kSmallHxThreads>(sp, str, rank);
    small_copy<kSmallHxThreads>(psi, s.phi, sizeof(V) * size_t(nsec));
    // the state's own Hamiltonian fits the staged region when the launch has one
    const bool hlds = sp.ham_lds > 0 && small_ham_bytes(s.G, s.nsub, s.ntab) <= size_t(sp.ham_lds);
    double e = 0.0;
    if (hlds) {
        // a term is one record, read by all lanes at once; the terms of the
        // group without a flip need only their sign and value, which is what
        // most of a seniority-zero Hamiltonian's are.  Bound by the instructions
        // of its 16 waves after the staging's loads (512 states of 330 strings:
        // 26.8 us with group, subgroup and rank read for every term, 24.5 so)
        double* tabs = reinterpret_cast<double*>(smem + L.ham);
        SmallTerm* terms = reinterpret_cast<SmallTerm*>(smem + L.ham + small_r16(8 * size_t(s.ntab)));
        small_copy<kSmallHxThreads>(tabs, s.tabs, 8 * size_t(s.ntab));
        int* diag = reinterpret_cast<int*>(red);   // free until the energy's sum
        if (threadIdx.x < 2) diag[threadIdx.x] = 0;
        __syncthreads();
        for (int gi = threadIdx.x; gi < s.G; gi += kSmallHxThreads) {
            const GroupDesc gd = s.groups[gi];
            if (gd.x == 0) {   // one group at most
                diag[0] = gd.sub_begin;
                diag[1] = gd.sub_end;
            }
            // (bits beyond n occur in no string; a flip of one leads out of the sector)
            const uint32_t x = gd.x >= (1u << sp.n) ? 0x8000u : gd.x;
            for (int si = gd.sub_begin; si < gd.sub_end; ++si) {
                terms[si].xw = x;
                terms[si].pos = gd.pos;
            }
        }
        __syncthreads();
        for (int si = threadIdx.x; si < s.nsub; si += kSmallHxThreads) {
            const SubDesc sub = s.subs[si];
            terms[si].xw |= (uint32_t(sub.w) & 0x7fffu) << 16;
            terms[si].tab = int32_t(sub.tab);
        }
        const int d0 = diag[0], d1 = diag[1];
        __syncthreads();
        // thread (slice q, string r) takes every sl-th term from the q-th on
        const int sl = small_slices(nsec);
        for (int i = threadIdx.x; i < sl * nsec; i += kSmallHxThreads) {
            const int r = i % nsec, q = i / nsec;
            const uint32_t b = str[r];
            double dd = 0.0;
#pragma unroll 4
            for (int si = d0 + q; si < d1; si += sl) {
                const SmallTerm m = terms[si];
                const double t = tabs[m.tab + ((m.pos & 7u) ? pext_pos(b, m.pos) : 0u)];
                dd += (__popc(b & (m.xw >> 16)) & 1) ? -t : t;
            }
            V acc = vzero<V>();
            axpy(acc, dd, psi[r]);
            const int nt = s.nsub - (d1 - d0);
#pragma unroll 2
            for (int k = q; k < nt; k += sl) {
                const SmallTerm m = terms[k < d0 ? k : k + (d1 - d0)];
                const uint32_t x = m.xw & 0xffffu;
                const int rp = x & 0x8000u ? -1 : int(rank[(b ^ x) & ((1u << sp.n) - 1u)]);
                const uint32_t u = (m.pos & 7u) == 2u
                                       ? ((b >> ((m.pos >> 3) & 31u)) & 1u) | ((b >> ((m.pos >> 8) & 31u)) & 1u) << 1
                                       : pext_pos(b, m.pos);
                const double t = tabs[m.tab + u];
                const double d = rp < 0 ? 0.0 : (__popc(b & (m.xw >> 16)) & 1) ? -t : t;
                axpy(acc, d, psi[max(rp, 0)]);
            }
            if (sl > 1) {
                part[size_t(q) * nsec + r] = acc;
            } else {
                lam[r] = acc;
                e += redot(psi[r], acc);
            }
        }
        if (sl > 1) {
            __syncthreads();
            for (int r = threadIdx.x; r < nsec; r += kSmallHxThreads) {
                V acc = vzero<V>();
                for (int q = 0; q < sl; ++q) vadd(acc, part[size_t(q) * nsec + r]);
                lam[r] = acc;
                e += redot(psi[r], acc);
            }
        }
    } else {
        __syncthreads();
        for (int r = threadIdx.x; r < nsec; r += kSmallHxThreads) {
            const uint32_t b = str[r];
            V acc = vzero<V>();
            for (int gi = 0; gi < s.G; ++gi) {
                const GroupDesc gd = s.groups[gi];
                const uint32_t p = b ^ gd.x;
                if (p >= (1u << sp.n)) continue;
                const int rp = rank[p];
                if (rp < 0) continue;
                axpy(acc, group_coeff(gd, s.subs, s.tabs, b), psi[rp]);
            }
            lam[r] = acc;
            e += redot(psi[r], acc);
        }
    }
    const double tot = small_block_total<kSmallHxThreads>(e, red);
    if (threadIdx.x == 0) s.out_e[0] = tot;
}

// Reverse sweep: per gate (last first) each wave's part of Re <lambda|A_j phi>
// into LDS, then U_j^dag on phi and lambda in the same pass; the per-gate sums
// (waves added in fixed order) into out_g at the end.
template <typename V, int KT>
__global__ void __launch_bounds__(kSmallThreads) k_small_adj(const StateDesc* __restrict__ sd, SmallSpace sp) {
    constexpr int kWaves = kSmallThreads / 64;
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallLayout L = small_layout(sp, kSmallAdj);
    const StateDesc& s = sd[blockIdx.y];
    V* psi = reinterpret_cast<V*>(smem + L.vec);
    V* lam = reinterpret_cast<V*>(smem + L.vec + small_r16(sizeof(V) * size_t(sp.nsec)));
    SmallGate* gs = reinterpret_cast<SmallGate*>(smem + L.gates);
    uint32_t* str = reinterpret_cast<uint32_t*>(smem + L.str);
    int16_t* rank = reinterpret_cast<int16_t*>(smem + L.rank);
    double* part = reinterpret_cast<double*>(smem + L.total);   // [M][waves] gradient partials
    small_stage_space<kSmallThreads>(sp, str, rank);
    small_copy<kSmallThreads>(psi, s.phi, sizeof(V) * size_t(sp.nsec));
    small_copy<kSmallThreads>(lam, s.lam, sizeof(V) * size_t(sp.nsec));
    for (int j = threadIdx.x; j < s.M; j += kSmallThreads) {
        const GateDesc g = s.gates[j];
        const double2 cs = s.cs[j];
        gs[j] = SmallGate{g.x, g.pd, g.chain, float(g.csign), cs.x, cs.y};
    }
    __syncthreads();
    uint32_t mine[KT];
    small_strings<KT>(str, sp.nsec, mine);
    SmallPairs<KT> cur, next;
    if (s.M > 0) cur.find(gs[s.M - 1], mine, rank);
    for (int t0 = 0; t0 < s.M; t0 += 8) {   // the wave totals of eight gates at once
        double acc[8];
        unroll_n<8>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            const int j = s.M - 1 - t0 - u;
            acc[u] = 0.0;
            if (j < 0) return;
            next.find(gs[max(j - 1, 0)], mine, rank);
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                const int t = int(threadIdx.x) + k * kSmallThreads, re = cur.re[k];
                if (re >= 0) {
                    V fD = psi[t], fE = psi[re], lD = lam[t], lE = lam[re];
                    // A|D> = s|E>, A|E> = -s|D>: <lam|A phi> = s (lam_E^* phi_D - lam_D^* phi_E)
                    const double v = redot(lE, fD) - redot(lD, fE);
                    acc[u] += cur.neg[k] ? -v : v;
                    const double ss = cur.neg[k] ? cur.s : -cur.s;   // U^dag: rotation by -theta
                    givens(fD, fE, cur.c, ss);
                    givens(lD, lE, cur.c, ss);
                    psi[t] = fD;
                    psi[re] = fE;
                    lam[t] = lD;
                    lam[re] = lE;
                }
            }
            __syncthreads();
            cur = next;
        });
        const double tot = wave_totals8(acc, threadIdx.x & 63);
        const int j = s.M - 1 - t0 - int((threadIdx.x & 63) >> 3);
        if ((threadIdx.x & 7) == 0 && j >= 0) part[size_t(j) * kWaves + (threadIdx.x >> 6)] = tot;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < s.M; j += kSmallThreads) {
        double r = 0.0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) r += part[size_t(j) * kWaves + i];
        s.out_g[j] = r;
    }
}

size_t small_lds(const SmallSpace& sp, int phase) {
    const size_t base = small_layout(sp, phase).total;
    if (phase == kSmallHx) return base + 8 * size_t(kSmallHxThreads / 64);
    return phase == kSmallAdj ? base + 8 * size_t(kSmallThreads / 64) * size_t(sp.M) : base;
}

// The launches' LDS must fit the CU's 160 KiB; beyond 64 KiB the kernels are
// allowed the whole of it (once).  None has static LDS, which would come on top.
int small_prepare(const SmallSpace& sp) {
    constexpr size_t kMax = size_t(160) << 10;
    size_t lds = 0;
    for (int ph = 0; ph < 3; ++ph) lds = std::max(lds, small_lds(sp, ph));
    if (lds > kMax) return 1;
    if (lds <= (64u << 10)) return 0;
    static std::once_flag once;
    static int rc = 0;
    std::call_once(once, [] {
#define VQE_SMALL_FNS(V)                                                                                             \
    reinterpret_cast<const void*>(&k_small_hx<V>), reinterpret_cast<const void*>(&k_small_fwd<V, 1>),               \
        reinterpret_cast<const void*>(&k_small_fwd<V, 2>), reinterpret_cast<const void*>(&k_small_fwd<V, 4>),       \
        reinterpret_cast<const void*>(&k_small_fwd<V, 8>), reinterpret_cast<const void*>(&k_small_adj<V, 1>),       \
        reinterpret_cast<const void*>(&k_small_adj<V, 2>), reinterpret_cast<const void*>(&k_small_adj<V, 4>),       \
        reinterpret_cast<const void*>(&k_small_adj<V, 8>)
        const void* fs[] = {VQE_SMALL_FNS(double2), VQE_SMALL_FNS(double)};
#undef VQE_SMALL_FNS
        for (const void* f : fs)
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(kMax)) != hipSuccess) rc = 1;
        if (rc) (void)hipGetLastError();   // not the next launch's
    });
    return rc;
}

template <typename V, int KT>
static void launch_small_gates(int phase, const StateDesc* sd, int count, const SmallSpace& sp, hipStream_t st) {
    const size_t lds = small_lds(sp, phase);
    if (phase == kSmallFwd)
        hipLaunchKernelGGL((k_small_fwd<V, KT>), dim3(1, count), dim3(kSmallThreads), lds, st, sd, sp);
    else
        hipLaunchKernelGGL((k_small_adj<V, KT>), dim3(1, count), dim3(kSmallThreads), lds, st, sd, sp);
}

template <typename V>
static void launch_small_t(int phase, const StateDesc* sd, int count, const SmallSpace& sp, hipStream_t st) {
    static_assert(kSmallMaxSector <= 8 * kSmallThreads, "strings per thread");
    if (phase == kSmallHx)
        hipLaunchKernelGGL(k_small_hx<V>, dim3(1, count), dim3(kSmallHxThreads), small_lds(sp, phase), st, sd, sp);
    else if (sp.nsec <= kSmallThreads)
        launch_small_gates<V, 1>(phase, sd, count, sp, st);
    else if (sp.nsec <= 2 * kSmallThreads)
        launch_small_gates<V, 2>(phase, sd, count, sp, st);
    else if (sp.nsec <= 4 * kSmallThreads)
        launch_small_gates<V, 4>(phase, sd, count, sp, st);
    else
        launch_small_gates<V, 8>(phase, sd, count, sp, st);
}

void launch_small(int phase, const StateDesc* sd, int count, const SmallSpace& sp, hipStream_t st) {
    if (sp.vbytes == 8)
        launch_small_t<double>(phase, sd, count, sp, st);
    else
        launch_small_t<double2>(phase, sd, count, sp, st);
}

}  // namespace vqe
