// Ansatz kernels on the packed sector layout (Sec. 2.1.2; the objective of
// Sec. 2.1.1, Eq. 1, and its gradient by the reverse sweep).
//
// Every UCCSD gate conserves the alpha and beta electron counts, so a state
// prepared from the reference |HF> has nonzero amplitudes only in the
// reference's (N, S_z) sector.  The packed layout stores exactly those
// amplitudes: strings b are grouped in blocks by their high bits h = b >> L,
// block h holds the in-sector strings with that high part ordered by
// (rank of the low alpha string, rank of the low beta string) among strings
// of their popcounts, and blocks follow each other in increasing h from
// base[h].  Empty blocks take no space.  The reference is entry 0.
//
// L is at least the number of electrons, so the reference lies in block 0.
// A gate pairs D (annihilated orbitals occupied, created ones empty) with
// E = D ^ x.  Consecutive gates whose high orbitals (the annihilated and
// created ones above the block bits) fit a window of at most 4 high bits form
// a run, applied tile by tile: a tile is the set of blocks whose high parts
// agree outside the window (those the run's gates pair), staged in LDS one
// after the other, all the run's gates applied, written back.  For UCCSD on
// the reference the occupied orbitals are low, so D and E differ in the
// high bits of the created orbitals only; generalised excitations may also
// annihilate high orbitals.
#include <type_traits>

#include "device_common.h"

namespace vqe {

template <typename V>
__global__ void k_packed_hf(const StateDesc* __restrict__ sd, int64_t size) {
    const StateDesc& s = sd[blockIdx.y];
    V* phi = reinterpret_cast<V*>(s.phi);
    for (int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; k < size;
         k += int64_t(gridDim.x) * blockDim.x)
        nt_store(phi + k, k == 0 ? vunit(V{}) : vzero<V>());
}

// VEC = 1: forward pass on phi.  VEC = 2: reverse sweep on phi and lambda
// with per-gate, per-tile partials of Re <lambda|A_j phi> (A_j = T_j - T_j^dag).
// V: amplitude type (double2, or double for real states).
// Tile entry k (blocks one after the other) is staged by thread k % BS
// (2 EPT BS covers the largest tile of the run); a gate's pairs come from the
// run's precomputed list for the tile's class, one pair per thread per pass.
// The tile's geometry is its host-built descriptor (one scalar read), so the
// tile loads, the gate parameters and the first list entries are all in
// flight together before the first wait.
// What bounds it, one state of 20 qubits (a run of 46 gates, forward): 2.5 us of
// loads before the first gate, then each wave's serial instruction stream.  A
// gate took 436 cycles, 328 of them without its pair's work: address and clamp
// arithmetic, two branches, a parity test; barriers and bank conflicts next to
// nothing.  Hence a step of 20 instructions that branches only to a barrier (an
// entry is two LDS offsets, the sign their order, absent pairs a dummy), and, as
// the waits that remain are then the barriers', waves that own whole groups of
// strings (WaveSplit in vqe_device.hip) and meet once per stretch of gates.
// Forward + reverse, us: one state of 18 qubits 281 -> 243, 20 qubits 432 -> 356,
// 22 qubits 690 -> 577, 24 qubits 1363 -> 1277; 49 states of 20 qubits, where LDS is
// busy half of the time, 1507 -> 1481.
template <int VEC, int BS, int EPT, typename V>
__global__ void __launch_bounds__(BS) k_prun(const StateDesc* __restrict__ sd, PackedRun run,
                                             const PackedGate* __restrict__ pg) {
    extern __shared__ double2 sh[];
    const StateDesc& s = sd[blockIdx.y];
    // both passes cover the run's live tiles only (all of them without a list);
    // gradient partials go to the tile's position in the launch
    const TileDesc tb = ldc(run.tdesc + blockIdx.x);
    const int po = int(blockIdx.x);
    const int tid = threadIdx.x;
    if (tb.nE == 0) {   // an empty tile: zero gradient partials
        if (VEC == 2)
            for (int jl = tid; jl < run.g1 - run.g0; jl += BS)
                s.part_g[size_t(run.g0 + jl) * s.gstride + po] = 0.0;
        return;
    }
    const int nE = tb.nE;
    const uint32_t hb0 = tb.hbase << run.L;
    const int nV = run.max_entries + 2;   // a vector: the tile and the lists' idle pair
    V* shp = reinterpret_cast<V*>(sh);
    V* shl = shp + nV;
    // the reverse sweep on real amplitudes keeps (phi, lambda) of an entry
    // side by side, so that a pair's four values take two 16-byte LDS reads
    // and two writes
    constexpr bool kPL = VEC == 2 && std::is_same<V, double>::value;
    double2* shpl = sh;
    constexpr bool fwd = VEC == 1;
    const int ng = run.g1 - run.g0;
    // the tile class's pair lists: gate j's list at lbase + j * stride.  Each
    // thread's first entry of a gate is loaded kListAhead gates ahead (the
    // first kListAhead before the tile loads) into slot t % kListAhead of eq;
    // the gate loops are unrolled so that every slot index is a constant, so a
    // gate waits only for its own entry's load and the list reads' latency
    // overlaps kListAhead gate steps.  The loads run past both ends of the
    // class's lists, unused (the lists' array has room for that): no clamp
    const uint32_t* lbase = run.ent + tb.ent;
    const int stride = tb.stride, span = tb.span;
    const uint32_t rowb = uint32_t(stride) * 4u;
    const __amdgpu_buffer_rsrc_t lrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(lbase - kListAhead * stride), 0, int(uint32_t(ng + 2 * kListAhead) * rowb), 0x00020000);
    const bool has_slot = __builtin_amdgcn_readfirstlane(tid) < span;   // whole waves
    const uint32_t voff = uint32_t(has_slot ? tid : 0) * 4u;
    uint32_t row = uint32_t(kListAhead + (fwd ? 0 : ng - 1)) * rowb;   // of the next load
    uint32_t eq[kListAhead];
#pragma unroll
    for (int d = 0; d < kListAhead; ++d) {
        eq[d] = __builtin_amdgcn_raw_buffer_load_b32(lrs, voff, row, 0);
        row += fwd ? rowb : 0u - rowb;
    }
    // per-gate parameters of this tile after the tile (2 double2 per gate):
    // (cos, sgn sin) and (sgn, 0), sgn the gate's pair sign from the tile's
    // high bits outside the window (the window's part is in each entry);
    // staged once; the first is read by broadcast in the gate loop, the
    // second (reverse sweep) applied to the gate's tile total at the end
    const RunLds lay = tiled_run_lds(VEC, sizeof(V), run.max_entries, ng, BS / 64);
    double2* gpar = sh + lay.par / 16;
    // the state index of each staged entry, kept for the write-back
    int gix[2 * EPT];
    {   // all loads first (clamped into the tile), then the LDS stores
        V vp[2 * EPT], vl[2 * EPT];
#pragma unroll
        for (int u = 0; u < 2 * EPT; ++u) {
            gix[u] = tile_index(tb, run.nblk, min(tid + BS * u, nE - 1));
            vp[u] = ldgv(reinterpret_cast<const V*>(s.phi) + gix[u]);
            if (VEC == 2) vl[u] = ldgv(reinterpret_cast<const V*>(s.lam) + gix[u]);
        }
        for (int j = tid; j < ng; j += BS) {
            const PackedGate g = pg[j];
            const double2 cs = s.cs[run.g0 + j];
            const double sgn = g.csign * parity_sign(hb0 & g.chhi);
            gpar[2 * j] = make_double2(cs.x, sgn * cs.y);
            gpar[2 * j + 1] = make_double2(sgn, 0.0);
        }
        // unconditional stores (a clamped slot rewrites the last entry with its
        // own value), so that every load is waited for on every path
#pragma unroll
        for (int u = 0; u < 2 * EPT; ++u) {
            const int k = min(tid + BS * u, nE - 1);
            if constexpr (kPL) {
                shpl[k] = make_double2(vp[u], vl[u]);
            } else {
                shp[k] = vp[u];
                if (VEC == 2) shl[k] = vl[u];
            }
        }
        if (tid < 2) {   // the idle pair
            shp[(kPL ? 2 : 1) * (run.max_entries + tid)] = V{};
            if (VEC == 2) (kPL ? shp + 1 : shl)[(kPL ? 2 : 1) * (run.max_entries + tid)] = V{};
        }
    }
    __syncthreads();
    // one pair; its part of the reverse sweep's Re <lambda|A_j phi>, A|D> =
    // s|E>, A|E> = -s|D>, with the entry's part of s; the tile's, common to the
    // gate, comes in when its total is stored
    auto at = [&](V* v, uint32_t off) -> V& {
        return *reinterpret_cast<V*>(reinterpret_cast<char*>(v) + off * uint32_t(sizeof(V) / 8));
    };
    auto pair = [&](uint32_t e, const double2& cs, double& acc) {
        if constexpr (kPL) {
            const uint32_t o0 = (e << 1) & 0x1fff0u, o1 = (e >> 15) & 0x1fff0u;
            double2* q0 = reinterpret_cast<double2*>(reinterpret_cast<char*>(shpl) + o0);
            double2* q1 = reinterpret_cast<double2*>(reinterpret_cast<char*>(shpl) + o1);
            double2 d = *q0, f = *q1;
            acc += d.x * f.y - d.y * f.x;
            givens(d.x, f.x, cs.x, -cs.y);   // U^dag: rotation by -theta
            givens(d.y, f.y, cs.x, -cs.y);
            *q0 = d;
            *q1 = f;
        } else {
            const uint32_t o0 = e & 0xffffu, o1 = e >> 16;
            V d = at(shp, o0), f = at(shp, o1);
            if constexpr (fwd) {
                givens(d, f, cs.x, cs.y);
            } else {
                V lD = at(shl, o0), lE = at(shl, o1);
                acc += redot(lE, d) - redot(lD, f);
                givens(d, f, cs.x, -cs.y);
                givens(lD, lE, cs.x, -cs.y);
                at(shl, o0) = lD;
                at(shl, o1) = lE;
            }
            at(shp, o0) = d;
            at(shp, o1) = f;
        }
    };
    // one gate: its pairs (one per thread per pass), returning the thread's
    // part of the gate's total; the slot's entry for gate t + kListAhead is
    // loaded meanwhile, and the next gate's (cos, sgn sin) read.  A place
    // without a pair rotates the idle pair, so the step branches only to a
    // barrier: what bounds it is the wave's serial instruction stream (about 20 per
    // gate forward, 10 to 20 cycles each), not its LDS accesses or arithmetic.  LONG (a list
    // longer than its span): the thread's later entries are read in the gate
    // itself; the gate loops are built separately for the two cases, so that
    // the common one has no other list reads than the slots'.  Between gates
    // whose entries are the same waves' there is no barrier: a wave's LDS
    // accesses are carried out in order, so it does not even wait for its
    // writes.  Nothing moves across a gate's end: an address formed early would
    // wait for its entry's load there
    double2 cs_ahead = gpar[fwd ? 0 : 2 * (ng - 1)];
    auto gate_step = [&](int jl, const double2* next, auto slot, auto long_tag, uint32_t meet) -> double {
        constexpr int q = decltype(slot)::value;
        constexpr bool LONG = decltype(long_tag)::value;
        const double2 cs = cs_ahead;
        cs_ahead = *next;
        double acc = 0.0;
        pair(eq[q], cs, acc);
        if constexpr (LONG) {
            for (int i = tid + span; i < stride; i += span) {
                const uint32_t e = ldg32(lbase + size_t(jl) * stride + i);
                if (uint32_t(__builtin_amdgcn_readfirstlane(int(e))) == run.idle) break;   // the wave's last
                pair(e, cs, acc);
            }
        }
        // (formed here: left to the round's end, where it is used, it would
        // keep the pair's amplitudes in registers)
        if constexpr (!fwd) __asm__ volatile("" : "+v"(acc));
        // the slot's next entry, issued once this gate's entry is dead (so
        // that it can take the same register)
        eq[q] = __builtin_amdgcn_raw_buffer_load_b32(lrs, voff, row, 0);
        row += fwd ? rowb : 0u - rowb;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect((meet >> q) & 1u, 0)) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        return acc;
    };
    // Whole rounds of slots run without per-gate bounds, so every one issues
    // the same loads and a gate waits for its own slot only; the last, partial
    // one checks each gate.  The reverse sweep takes the wave totals of a
    // round's gates together after them (wave_totals8) into wsum; the waves
    // are added after the last gate.
    double* wsum = reinterpret_cast<double*>(sh + lay.wsum / 16);   // [ng][BS / 64], VEC = 2 only
    auto meets = [&](int t0) -> uint32_t {   // of the gates t0 .. t0 + 7, t0 a multiple of 8
        const uint64_t m = fwd ? (t0 < 64 ? run.meet_fwd[0] : run.meet_fwd[1])
                               : (t0 < 64 ? run.meet_adj[0] : run.meet_adj[1]);
        return uint32_t(m >> (t0 & 63)) & 0xffu;
    };
    auto round = [&](int t0, auto long_tag, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        const uint32_t meet = meets(t0);
        const int j0 = fwd ? t0 : ng - 1 - t0;
        double acc[kListAhead];
        unroll_n<kListAhead>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            acc[u] = 0.0;
            if (FULL || t0 + u < ng)   // (past the last gate: unused parameters)
                acc[u] = gate_step(fwd ? j0 + u : j0 - u, gpar + 2 * j0 + (fwd ? 2 * (u + 1) : -2 * (u + 1)), uu,
                                   long_tag, meet);
        });
        if constexpr (!fwd) {
            static_assert(kListAhead == 8, "wave_totals8 takes eight gates");
            const double tot = wave_totals8(acc, tid & 63);
            const int u = (tid & 63) >> 3;
            if ((tid & 7) == 0 && (FULL || t0 + u < ng)) wsum[(j0 - u) * (BS / 64) + (tid >> 6)] = tot;
        }
    };
    auto gates = [&](auto long_tag) {
        int t0 = 0;
        for (; t0 + kListAhead <= ng; t0 += kListAhead) round(t0, long_tag, std::true_type{});
        if (t0 < ng) round(t0, long_tag, std::false_type{});
    };
    if (!has_slot) {   // a wave without pairs only meets the others
        for (int t0 = 0; t0 < ng; t0 += 8)
            for (int k = __builtin_popcount(meets(t0)); k > 0; --k) __syncthreads();
    } else if (stride > span) {
        gates(std::true_type{});
    } else {
        gates(std::false_type{});
    }
    __syncthreads();
    if constexpr (!fwd) {
        for (int jl = tid; jl < ng; jl += BS) {
            double v = 0.0;
            for (int w = 0; w < span / 64; ++w) v += wsum[jl * (BS / 64) + w];
            s.part_g[size_t(run.g0 + jl) * s.gstride + po] = v * gpar[2 * jl + 1].x;
        }
    }
#pragma unroll
    for (int u = 0; u < 2 * EPT; ++u) {
        const int k = tid + BS * u;
        if (k < nE) {
            if constexpr (kPL) {
                const double2 pl = shpl[k];
                stgv(reinterpret_cast<double*>(s.phi) + gix[u], pl.x);
                stgv(reinterpret_cast<double*>(s.lam) + gix[u], pl.y);
            } else {
                stgv(reinterpret_cast<V*>(s.phi) + gix[u], shp[k]);
                if (VEC == 2) stgv(reinterpret_cast<V*>(s.lam) + gix[u], shl[k]);
            }
        }
    }
}

// Zero-angle reverse sweep of a gate pool (ADAPT-VQE pool gradients): every
// gate at angle 0 is the identity, so phi and lambda are only read and the
// gates are independent.  One launch covers every (run, tile): block b works
// on tile b - blk0[r] of run r = blk_run[b]; after staging the tile, each
// wave takes whole gates (w, w + BS/64, ...) and its 64 lanes split the
// gate's pair list, so a gate's tile partial of Re <lambda|A_j phi> is one
// wave total, stored without a block barrier.
template <int BS, int EPT, typename V>
__global__ void __launch_bounds__(BS) k_ppool(const StateDesc* __restrict__ sd,
                                              const PackedRun* __restrict__ runs,
                                              const int32_t* __restrict__ blk_run,
                                              const int32_t* __restrict__ blk0,
                                              const PackedGate* __restrict__ pg_all,
                                              const HxTables* __restrict__ tabsrc,
                                              const int32_t* __restrict__ base) {
    extern __shared__ double2 sh[];
    __shared__ HxTables T;
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(tabsrc);
        uint32_t* dst = reinterpret_cast<uint32_t*>(&T);
        for (int i = threadIdx.x; i < int(sizeof(HxTables) / 4); i += BS) dst[i] = src[i];
    }
    __syncthreads();
    const StateDesc& s = sd[blockIdx.y];
    const int r = ldc(blk_run + blockIdx.x);
    const PackedRun run = ldc(runs + r);
    const int o = int(blockIdx.x) - ldc(blk0 + r);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng = run.g1 - run.g0;
    TileBlocks tb;
    tile_blocks(T, run, o, base, tb);
    if (tb.nE == 0) {
        for (int jl = tid; jl < ng; jl += BS) s.part_g[size_t(run.g0 + jl) * s.gstride + o] = 0.0;
        return;
    }
    const int nE = tb.nE;
    const uint32_t hb0 = tb.hbase << run.L;
    V* shp = reinterpret_cast<V*>(sh);
    V* shl = shp + nE;
    {
        V vp[2 * EPT], vl[2 * EPT];
#pragma unroll
        for (int u = 0; u < 2 * EPT; ++u) {
            const int k = min(tid + BS * u, nE - 1);
            const int64_t gi = tile_global(tb, run.nblk, k);
            vp[u] = ldgv(reinterpret_cast<const V*>(s.phi) + gi);
            vl[u] = ldgv(reinterpret_cast<const V*>(s.lam) + gi);
        }
#pragma unroll
        for (int u = 0; u < 2 * EPT; ++u) {
            const int k = min(tid + BS * u, nE - 1);
            shp[k] = vp[u];
            shl[k] = vl[u];
        }
    }
    __syncthreads();
    const int cls = tb.cls;
    const PackedGate* pg = pg_all + run.g0;
    const int2 lc = ldc(run.info + cls);
    const int stride = lc.y & 0xffff;
    // a gate's parameters and first kPoolAhead x 64 entries are loaded while the
    // wave's gate before it is summed: a round trip for each was what the sweep
    // took (875 operators on 20 qubits 49.8 us, so and with as much LDS as the
    // amplitudes take 34.5; 512 threads 38.1, 1,024 58.3)
    constexpr int kPoolAhead = 4;
    struct Gate {
        double csign;
        uint32_t chhi, e[kPoolAhead];
    };
    auto load = [&](int jl, Gate& g) {
        const int j = min(jl, ng - 1);
        const PackedGate q = ldc(pg + j);
        g.csign = q.csign;
        g.chhi = q.chhi;
        const uint32_t* lst = run.ent + lc.x + size_t(j) * stride;
#pragma unroll
        for (int u = 0; u < kPoolAhead; ++u) g.e[u] = lane + 64 * u < stride ? ldg32(lst + lane + 64 * u) : run.idle;
    };
    Gate cur, next;
    load(w, next);
    for (int jl = w; jl < ng; jl += BS / 64) {
        cur = next;
        load(jl + BS / 64, next);
        const double sgn_hi = cur.csign * parity_sign(hb0 & cur.chhi);
        double acc = 0.0;
        auto pair = [&](uint32_t e) {
            const int k = pair_first(e), ie = pair_second(e);
            const V fD = shp[k], fE = shp[ie], lD = shl[k], lE = shl[ie];
            acc += sgn_hi * (redot(lE, fD) - redot(lD, fE));
        };
#pragma unroll
        for (int u = 0; u < kPoolAhead; ++u)
            if (cur.e[u] != run.idle) pair(cur.e[u]);
        const uint32_t* lst = run.ent + lc.x + size_t(jl) * stride;
        for (int i = lane + 64 * kPoolAhead; i < stride; i += 64) {
            const uint32_t e = ldg32(lst + i);
            if (e == run.idle) break;
            pair(e);
        }
        acc = wave_total(acc);
        if (lane == 0) s.part_g[size_t(run.g0 + jl) * s.gstride + o] = acc;
    }
}

// Launch shapes (threads per tile, entries per thread).
#define VQE_PACKED_SHAPES(X)                                                                  \
    X(64, 1) X(64, 2) X(64, 4) X(64, 8) X(256, 1) X(256, 2) X(256, 3) X(256, 5) X(512, 1)     \
    X(512, 2) X(512, 3) X(1024, 1) X(1024, 2)

struct PShape {
    int bs, ept;
};
#define VQE_SHAPE_ENTRY(B, E) {B, E},
constexpr PShape kPShapes[] = {VQE_PACKED_SHAPES(VQE_SHAPE_ENTRY)};
#undef VQE_SHAPE_ENTRY
constexpr int kNumPShapes = int(sizeof(kPShapes) / sizeof(kPShapes[0]));

int packed_shape(int max_block, int min_threads) {
    int best = -1;
    for (int pass = 0; pass < 2 && best < 0; ++pass)   // second pass: any thread count
        for (int i = 0; i < kNumPShapes; ++i) {
            const PShape& p = kPShapes[i];
            if ((pass == 0 && p.bs < min_threads) || p.bs * p.ept < max_block) continue;
            if (best < 0 || p.bs * p.ept < kPShapes[best].bs * kPShapes[best].ept) best = i;
        }
    return best;
}

int packed_shape_threads(int shape) { return kPShapes[shape].bs; }

using PackedLauncher = void (*)(const StateDesc*, int, const PackedRun&, const PackedGate*, hipStream_t);

template <int VEC, int BS, int EPT, typename V>
static void launch_one(const StateDesc* sd, int count, const PackedRun& run, const PackedGate* pg,
                       hipStream_t st) {
    const size_t lds = tiled_run_lds(VEC, sizeof(V), run.max_entries, run.g1 - run.g0, BS / 64).total;
    const int nx = run.live ? run.nlive : run.ntiles;
    if (nx == 0) return;   // a run with no live tile: nothing to do, no partials
    hipLaunchKernelGGL((k_prun<VEC, BS, EPT, V>), dim3(nx, count), dim3(BS), lds, st, sd, run, pg);
}

#define VQE_FWD_ENTRY(B, E) &launch_one<1, B, E, double2>,
#define VQE_ADJ_ENTRY(B, E) &launch_one<2, B, E, double2>,
#define VQE_FWD_REAL(B, E) &launch_one<1, B, E, double>,
#define VQE_ADJ_REAL(B, E) &launch_one<2, B, E, double>,
static const PackedLauncher kFwdLaunch[] = {VQE_PACKED_SHAPES(VQE_FWD_ENTRY)};
static const PackedLauncher kAdjLaunch[] = {VQE_PACKED_SHAPES(VQE_ADJ_ENTRY)};
static const PackedLauncher kFwdLaunchR[] = {VQE_PACKED_SHAPES(VQE_FWD_REAL)};
static const PackedLauncher kAdjLaunchR[] = {VQE_PACKED_SHAPES(VQE_ADJ_REAL)};
#undef VQE_FWD_ENTRY
#undef VQE_ADJ_ENTRY
#undef VQE_FWD_REAL
#undef VQE_ADJ_REAL

void launch_packed_run(const StateDesc* sd, int count, const PackedRun& run, const PackedGate* pg,
                       bool adjoint, bool real, hipStream_t st) {
    if (adjoint)
        (real ? kAdjLaunchR : kAdjLaunch)[run.shape_adj](sd, count, run, pg, st);
    else
        (real ? kFwdLaunchR : kFwdLaunch)[run.shape](sd, count, run, pg, st);
}

using PoolLauncher = void (*)(const StateDesc*, int, const PoolSweep&, const HxTables*,
                              const int32_t*, hipStream_t);

template <int BS, int EPT, typename V>
static void launch_pool_one(const StateDesc* sd, int count, const PoolSweep& ps,
                            const HxTables* tabs, const int32_t* base, hipStream_t st) {
    hipLaunchKernelGGL((k_ppool<BS, EPT, V>), dim3(ps.nblk, count), dim3(BS), ps.lds / sizeof(double2) * sizeof(V), st, sd, ps.runs,
                       ps.blk_run, ps.blk0, ps.gates, tabs, base);
}

#define VQE_POOL_ENTRY(B, E) &launch_pool_one<B, E, double2>,
#define VQE_POOL_REAL(B, E) &launch_pool_one<B, E, double>,
static const PoolLauncher kPoolLaunch[] = {VQE_PACKED_SHAPES(VQE_POOL_ENTRY)};
static const PoolLauncher kPoolLaunchR[] = {VQE_PACKED_SHAPES(VQE_POOL_REAL)};
#undef VQE_POOL_ENTRY
#undef VQE_POOL_REAL

void launch_pool_sweep(const StateDesc* sd, int count, const PoolSweep& ps, const HxTables* tabs,
                       const int32_t* base, bool real, hipStream_t st) {
    if (ps.nblk > 0) (real ? kPoolLaunchR : kPoolLaunch)[ps.shape](sd, count, ps, tabs, base, st);
}

void launch_packed_hf(const StateDesc* sd, int count, int64_t size, bool real, hipStream_t st) {
    const int nblk = blocks_for(uint64_t(size));
    if (real)
        hipLaunchKernelGGL(k_packed_hf<double>, dim3(nblk, count), dim3(kBlock), 0, st, sd, size);
    else
        hipLaunchKernelGGL(k_packed_hf<double2>, dim3(nblk, count), dim3(kBlock), 0, st, sd, size);
}

int packed_enable_lds(size_t bytes) {
    hipError_t e = hipSuccess;
    auto set = [&](const void* f) {
        hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
        if (r != hipSuccess) e = r;
    };
#define VQE_SET_ENTRY(B, E)                                                 \
    set(reinterpret_cast<const void*>(&k_prun<1, B, E, double2>));          \
    set(reinterpret_cast<const void*>(&k_prun<2, B, E, double2>));          \
    set(reinterpret_cast<const void*>(&k_ppool<B, E, double2>));            \
    set(reinterpret_cast<const void*>(&k_prun<1, B, E, double>));           \
    set(reinterpret_cast<const void*>(&k_prun<2, B, E, double>));           \
    set(reinterpret_cast<const void*>(&k_ppool<B, E, double>));
    VQE_PACKED_SHAPES(VQE_SET_ENTRY)
#undef VQE_SET_ENTRY
    return e == hipSuccess ? 0 : 1;
}

}  // namespace vqe
