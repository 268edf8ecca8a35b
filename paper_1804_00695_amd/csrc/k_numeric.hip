// k_numeric.hip -- numeric phase (Sec. 2.1, Fig. "spgemmexp") as the
// row-range fused multiply-add kernel of the chunking algorithms
// (Secs. 3.2.2 and 3.3.1): C_i += sum over k in row i of A, k in [k_lo, k_hi),
// of a_ik * B_k, optionally starting from the values already in C (the
// partial result of earlier row parts of B).
//
// LDS path: G lanes own a row of C. Its (sorted) columns are loaded once into
// an LDS hash mapping column -> position in the row, next to an LDS array of
// fp64 accumulators in row order. When C has few enough columns, a table slot
// packs column and position into one 32-bit word. The entries of row i of A are
// taken in stored order, G at a time. With 8 lanes or a whole wave per row their
// (entry, position in B_k) pairs are laid end to end, one per lane, and lanes of a
// step that belong to different entries add entry by entry; with 16 or 32 lanes
// a step is one entry, whose lanes hold distinct columns of B_k. Either way every
// c_ij receives its terms in ascending k -- the order of the row-wise
// formulation. Products are rounded before the add (compiled without
// contraction), so the result equals a sequential dense-accumulator evaluation bit
// for bit. The B loads of a batch of steps are all issued, without branches, before
// the first of them is used, to hide HBM/L2 latency.
//
// Spill path (rows with more outputs than the largest LDS class holds): the
// row's outputs are cut into windows of consecutive positions of C, each a
// task of its own with the LDS table and accumulators of one wave. A window
// streams the whole row of A, its rows of B narrowed to the window's column
// range (by binary search in B's sorted columns for long rows, by a range
// test for short ones), 64 (entry, B position) pairs per step; the adds of a
// step go in rounds so that every c_ij still gets its terms in ascending k.
#include <climits>
#include <cstdio>
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "postab.h"
#include "profile.h"

namespace mls {

constexpr int kNumDepth = 4;   // steps whose B loads are issued together (8 where LDS caps occupancy at 4)
constexpr int kNumWinCap = 1024;   // table slots of a spill window (CAP / 2 positions)
constexpr int kWinDepth = 8;       // spill window: steps of 64 pairs whose B loads are issued together
constexpr bool kNumFlat = true;    // flattened pairs for the classes of at most kNumFlatMaxG lanes per row
constexpr int kNumFlatMaxG = 8;

__device__ __forceinline__ void nwave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

constexpr int nw_num(int row_bytes, int rows_per_wave, int lds = 65536)
{
    int per_wave = row_bytes * rows_per_wave;
    int nw = lds / per_wave;
    return nw > 4 ? 4 : (nw < 1 ? 1 : nw);
}

// Hash a row's columns (column -> position) and set its accumulators (0, or
// the values already in C when accumulating). Each lane loads D of its
// columns (then values) before inserting them, so the loads overlap instead
// of each waiting on the previous insert (D = 2 for 32 or more lanes per
// row: few columns per lane, and few registers to spare at 8 waves per SIMD).
template <int G>
constexpr int ins_depth() { return G >= 32 ? 2 : 4; }

template <int G, typename TAB>
__device__ __forceinline__ void insert_row(TAB &tab, double *acc,
                                           const MLS_G int32_t *__restrict__ cols,
                                           const MLS_G double *__restrict__ vals, int off, int n, int lane,
                                           bool accumulate)
{
    constexpr int kInsDepth = ins_depth<G>();
    if constexpr (kInsDepth == 1) {
        for (int e = lane; e < n; e += G) {
            tab.insert(cols[off + e], e);
            acc[e] = accumulate ? vals[off + e] : 0.0;
        }
        return;
    }
    for (int e0 = lane; e0 < n; e0 += G * kInsDepth) {
        int jv[kInsDepth];
#pragma unroll
        for (int u = 0; u < kInsDepth; ++u) {
            const int e = e0 + u * G;
            jv[u] = e < n ? cols[off + e] : -1;
        }
#pragma unroll
        for (int u = 0; u < kInsDepth; ++u)
            if (jv[u] >= 0) tab.insert(jv[u], e0 + u * G);
        if (accumulate) {
            double v[kInsDepth];
#pragma unroll
            for (int u = 0; u < kInsDepth; ++u) {
                const int e = e0 + u * G;
                v[u] = e < n ? vals[off + e] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kInsDepth; ++u) {
                const int e = e0 + u * G;
                if (e < n) acc[e] = v[u];
            }
        } else {
#pragma unroll
            for (int u = 0; u < kInsDepth; ++u) {
                const int e = e0 + u * G;
                if (e < n) acc[e] = 0.0;
            }
        }
    }
}

constexpr int num_row_bytes(int CAP, int G, bool PACK)
{
    return CAP * (PACK ? 4 : 8) + (CAP / 2) * 8 + G * 16;
}

// Where a row of the bin lives: product t, output size nc, the start of its
// C entries (cs) and its A entry range [ps, pe), all local (a slot without a
// row: nc = 0 and an empty range).
struct RowMeta {
    int t, nc, cs, ps, pe;
};

// The descriptor of product t: the kernel argument for a single product (its
// fields then live in scalar registers), else the batch's descriptor array.
template <bool MULTI>
__device__ __forceinline__ Prob prob_of(const Batch &b, int t)
{
    if (!MULTI) return b.p0;
    return get_prob_batch(b, t);
}

// Rows are software-pipelined across loop iterations, and every load of that
// pipeline is issued without a branch around it (a lane with nothing to load
// reads a constant word instead), so its first use can sit a row or more
// behind it: a use inside a branch would make the wave wait at the branch.

// A row's metadata as loaded: output size and row pointers before their
// offsets are subtracted (row_final), product t for a batch. A slot with no
// row reads zeros: no outputs and an empty range of A, so every step of the
// row loop is empty for it.
struct RowRaw {
    int t, nc, c0, a0, a1;
};

template <bool MULTI>
__device__ __forceinline__ RowRaw row_issue(const Batch &b, const Sched &sc, int g, ProbCache &pc)
{
    RowRaw r{0, 0, 0, 0, 0};
    const bool on = g >= 0;
    int i = g;
    if (MULTI && on) {
        r.t = find_prob_cached(b.abase, b.nprob, g, pc);
        i = g - pc.lo;
    }
    const Prob P = prob_of<MULTI>(b, r.t);
    const MLS_G int32_t *zero = (const MLS_G int32_t *)k_zeros4;
    const MLS_G int32_t *pv = on ? gp(sc.val) + g : zero;
    const MLS_G int32_t *pcr = on ? gp(P.crp) + i : zero;
    const MLS_G int32_t *par = on ? gp(P.arp) + i : zero;
    r.nc = *pv;
    r.c0 = *pcr;
    r.a0 = par[0];
    r.a1 = par[1];
    return r;
}

template <bool MULTI>
__device__ __forceinline__ RowMeta row_final(const Batch &b, const RowRaw &r)
{
    const Prob P = prob_of<MULTI>(b, r.t);
    RowMeta m;
    m.t = r.t;
    m.nc = r.nc;
    m.cs = r.c0 - P.c_off;
    m.ps = r.a0 - P.a_off;
    m.pe = r.a1 - P.a_off;
    return m;
}

// The first chunk of a row: entries ps + lane of row i of A (column -1 past
// the row) and the row pointers of B at their columns, as loaded (zeros for
// columns outside [k_lo, k_hi), which then give an empty range).
struct FirstChunk {
    int ka;
    double sa;
    int r0, r1;
};

__device__ __forceinline__ void first_a(const Prob &P, const RowMeta &m, int lane, FirstChunk &f)
{
    const bool on = m.ps + lane < m.pe;
    const MLS_G int32_t *pk = on ? gp(P.aci) + m.ps + lane : (const MLS_G int32_t *)k_ones4;
    const MLS_G double *pa = on ? gp(P.aval) + m.ps + lane : (const MLS_G double *)k_zeros4;
    f.ka = *pk;
    f.sa = *pa;
}

__device__ __forceinline__ void first_b(const Prob &P, FirstChunk &f)
{
    const bool in = f.ka >= P.k_lo && f.ka < P.k_hi;
    const MLS_G int32_t *pb = in ? gp(P.brp) + (f.ka - P.k_lo) : (const MLS_G int32_t *)k_zeros4;
    f.r0 = pb[0];
    f.r1 = pb[1];
}

// Wave-wide flattened steps: the (entry, B position) pairs of a staged chunk,
// entry-major (so in ascending k), 64 per step whatever the rows of B, D steps
// with their loads in flight. The chunk's non-empty entries are compacted in
// par: (first B position - first pair, -, a). A bit per pair tells where an
// entry starts, so a lane's entry is a count of the bits up to it; eb holds
// the entries that started before the tile, less one. Lanes of a step that
// belong to different entries may hit the same output: they add entry by
// entry (one wave's LDS adds take effect in program order), which keeps every
// c_ij's terms in ascending k. Columns outside [jlo, jhi] are another
// window's. Returns whether a column was not found.
// A step's rounds of adds: one per entry that has pairs in it, or (FEW) per entry
// that has an output in the window. Short rows of B make many entries per step,
// and a window takes few of their pairs, as rows of up to 32 are not narrowed:
// chunks of kWinRounds entries per step and more are taken so. Rows of 6000
// outputs, rows of B of 1, 2, 4, 8 and 16 entries: 4139, 2231, 1471, 911 and 691 us
// with a round for each, 2021, 1301, 1079, 844 and 601 us so (one add per
// collision, which needs a word of LDS per output and three passes over it: 1915,
// 1356, 1183, 1126 and 1077). Rows of 1500 outputs in one table, whose pairs all
// hit, lose by it: rows of B of 1 entry 3336, 4626 us (8978 by collisions).
constexpr int kWinRounds = 8;

template <int D, bool FEW, typename TAB>
__device__ __forceinline__ bool flat_tile(const TAB &tab, double *acc, const int4 *par, uint32_t *flags,
                                          int lane, int base, int first, bool nonempty, int total, int &eb,
                                          const MLS_G int32_t *bci, const MLS_G double *bval, int jlo, int jhi)
{
    if (lane < 2 * D) flags[lane] = 0u;
    nwave_sync();
    const int at = first - base;
    if (nonempty && (uint32_t)at < (uint32_t)(kWave * D)) atomicOr(flags + (at >> 5), 1u << (at & 31));
    nwave_sync();
    int jv[D], rel[D], more[D];
    bool ok[D];
    double av[D], bv[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const uint2 m = *(const uint2 *)(flags + 2 * d);
        const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)m.x);
        const uint32_t m1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)m.y);
        const uint64_t starts = ((uint64_t)m1 << 32) | m0, after = starts >> 1;   // after: lanes 1 and up
        rel[d] = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(after >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)after, 0u));
        more[d] = __popcll(after);
        const int e0 = eb + (int)(starts & 1u);
        const int pp = base + d * kWave + lane;
        ok[d] = pp < total;
        const int4 pr = par[e0 + rel[d]];
        const uint32_t q = (uint32_t)(pr.x + or_last(ok[d], pp, total - 1));   // (past the pairs: the last one again)
        jv[d] = bci[q];
        bv[d] = bval[q];
        av[d] = __hiloint2double(pr.w, pr.z);
        eb = e0 + more[d];
    }
    // every load is issued before the first use of a loaded column
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) ok[d] = ok[d] && jv[d] >= jlo && jv[d] <= jhi;
    uint32_t posv[D];
    tab.template lookup_n<D>(jv, ok, posv);
#pragma unroll
    for (int d = 0; d < D; ++d) asm volatile("" ::"v"(bv[d]));
    bool bad = false;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const bool hit = ok[d] && posv[d] <= TAB::kMaxPos;
        bad |= ok[d] && !hit;
        const double t = av[d] * bv[d];
        if constexpr (!FEW) {
            for (int r = 0; r <= more[d]; ++r)
                if (hit && rel[d] == r) atomicAdd(acc + posv[d], t);
        } else {
            for (unsigned long long pend = __ballot(hit); pend;) {
                const bool mine = hit && rel[d] == __builtin_amdgcn_readlane(rel[d], __ffsll((long long)pend) - 1);
                if (mine) atomicAdd(acc + posv[d], t);
                pend &= ~__ballot(mine);
            }
        }
    }
    return bad;
}

constexpr int kFlatWords = 16;   // start bits of a tile of 8 steps

template <int DEPTH, bool WIN, typename TAB>
__device__ __forceinline__ bool flat_chunk(const TAB &tab, double *acc, int4 *par, uint32_t *flags,
                                           int lane, int q0, int q1, double a, const MLS_G int32_t *bci,
                                           const MLS_G double *bval, int jlo, int jhi)
{
    static_assert(2 * DEPTH <= kFlatWords, "start bits");
    const int np = q1 > q0 ? q1 - q0 : 0;
    const int incl = group_scan_incl<kWave>(np, lane);
    const int total = group_total<kWave>(np, incl);
    const int first = incl - np;
    const unsigned long long ne = __ballot(np > 0);
    if (np > 0)
        par[__popcll(ne & ((1ull << lane) - 1ull))] = make_int4(q0 - first, 0, __double2loint(a), __double2hiint(a));
    bool bad = false;
    int eb = -1;
    auto tiles = [&](auto few) {
        constexpr bool FEW = decltype(few)::value;
        for (int base = 0; base < total;) {
            // (the tail in smaller tiles: a step past the pairs costs as much as any)
            const int steps = (total - base + kWave - 1) / kWave;
            if (steps > DEPTH / 2) {
                bad |= flat_tile<DEPTH, FEW>(tab, acc, par, flags, lane, base, first, np > 0, total, eb, bci, bval,
                                             jlo, jhi);
                base += DEPTH * kWave;
            } else {
                bad |= flat_tile<2, FEW>(tab, acc, par, flags, lane, base, first, np > 0, total, eb, bci, bval, jlo,
                                         jhi);
                base += 2 * kWave;
            }
        }
    };
    if (WIN && total <= kWave / kWinRounds * __popcll(ne)) tiles(std::true_type{});
    else tiles(std::false_type{});
    nwave_sync();
    return bad;
}

// FLAT: the (entry, B position) pairs of a staged chunk are flattened, G at a
// time, one per lane (for rows of B shorter than G, which would leave lanes
// idle).

// Waves per SIMD that the LDS of one workgroup (NW waves) leaves resident:
// 160 KB per CU, 4 SIMDs, at most 8 waves each.
constexpr int lds_waves_per_simd(int wg_bytes, int nw)
{
    int wgs = 163840 / wg_bytes;
    int w = wgs * nw / 4;
    return w > 8 ? 8 : (w < 1 ? 1 : w);
}

// MAXLDS: LDS bytes of a workgroup that set how many waves it has (1 to 4)
template <int G, int CAP, bool PACK, bool MULTI, bool FLAT, int MAXLDS = 65536>
struct NumShape {
    static constexpr int W = kWave / G;
    static constexpr int XW = G == kWave && !FLAT ? kFlatWords : 0;   // start bits of a wave's pairs
    static constexpr int NW = nw_num(num_row_bytes(CAP, G, PACK) + 4 * XW, W, MAXLDS);
    static constexpr int OCC = lds_waves_per_simd(NW * W * (num_row_bytes(CAP, G, PACK) + 4 * XW), NW);
    // where LDS already limits a SIMD to 4 waves, registers are free for
    // twice the steps in flight
    static constexpr int DEPTH = OCC <= 4 ? 2 * kNumDepth : kNumDepth;
    // waves per SIMD the kernel is compiled for: the LDS bound, capped so the
    // row pipeline's registers fit without spills (a reload from scratch
    // would wait for every load issued before it): 7 waves (72 VGPRs), 6
    // (80) where a wave owns a row, 5 (96) for the flattened steps or for batches
    static constexpr int OCC_CAP = (FLAT || MULTI) ? 5 : (G == kWave ? 6 : 7);
    static constexpr int OCC_R = OCC < OCC_CAP ? OCC : OCC_CAP;
    // the next row's first chunk is prefetched where registers allow (at
    // most 5 waves per SIMD); otherwise a row loads its first chunk when it
    // starts
    static constexpr bool PF = !MULTI && OCC_R <= 5;
    // LDS of a workgroup: tables (and start bits), staged entries of A
    // (q0, q1, a), accumulators
    static constexpr int TW = PACK ? CAP : 2 * CAP;   // table words per row
    static constexpr int LDS_PAR = (NW * W * (TW + XW) * 4 + 15) / 16 * 16;
    static constexpr int LDS_ACC = LDS_PAR + NW * W * G * 16;
    static constexpr int LDS = LDS_ACC + NW * W * (CAP / 2) * 8;
};

// The rows of one bin on the workgroups vblk of vgrid; lds: NumShape::LDS bytes
// of this workgroup.
template <int G, int CAP, bool PACK, bool MULTI, bool FLAT, int MAXLDS>
__device__ __forceinline__ void num_lds_rows(const Batch &b, const Sched &sc, int bin, char *lds, int vblk, int vgrid)
{
    using Shape = NumShape<G, CAP, PACK, MULTI, FLAT, MAXLDS>;
    constexpr int kNumDepth = Shape::DEPTH;
    constexpr bool PF = Shape::PF;
    // Where a wave owns a row, its pairs are flattened over the 64 lanes
    // (flat_chunk): rows of B are long there (the host picks G from their mean
    // length), and one entry of A per step would leave lanes idle or, past 64
    // entries, chain a load, a lookup and a load per step. Numeric phase of the
    // restriction times the 81-point elasticity operator on 48^3 nodes: 1050 us
    // with one step at a time, 711 us in steps of one entry,
    // 452 us flattened.
    constexpr bool LONG = G == kWave && !FLAT;
    static_assert(FLAT || G % kNumDepth == 0, "the staged entries are read kNumDepth at a time");
    constexpr int W = kWave / G;
    constexpr int XW = Shape::XW;
    constexpr int NW = Shape::NW;
    constexpr int TW = Shape::TW;
    uint32_t *s_tab = (uint32_t *)lds;
    int4 *s_par = (int4 *)(lds + Shape::LDS_PAR);
    double *s_acc = (double *)(lds + Shape::LDS_ACC);

    const int wave = threadIdx.x >> 6;
    if (wave >= NW) return;
    const int lw = threadIdx.x & 63;
    const int slot = lw / G, lane = lw % G;
    const int rs = wave * W + slot;
    // 2-slot buckets where 32 lanes own a row, else 4-slot ones. A 4-slot bucket
    // costs more instructions, a 2-slot one more probes past it, in which one
    // lane holds up the others: restriction times the 81-point elasticity
    // operator, 64 lanes and tables 43 % full, 559 us with 2 and 452 with 4
    // slots; 27-point stencil square on 128^3, 32 lanes, 2377 with 2 and 2632
    // with 4.
    PosTab<CAP, PACK, (G == 32 ? 2 : 4)> tab{s_tab + rs * TW};
    double *acc = s_acc + rs * (CAP / 2);
    int4 *par = s_par + rs * G;
    uint32_t *flags = s_tab + NW * W * TW + rs * XW;   // LONG only

    const int n_bin = gp(sc.bin_count)[bin];
    const int start = bin_start(sc.bin_count, bin);
    const int ntasks = (n_bin + W - 1) / W;
    TaskIter it = task_iter<MAXLDS != 65536>(ntasks, NW, -1, vblk, vgrid);
    // Rows of a slot overlap: with PF three are in flight (the row after next
    // has its perm entry loading; the next row its metadata, then its first
    // chunk: A entries during this row's insert and steps, B row pointers
    // after them), so a row starts with all of its dependent index loads
    // done. Without PF (fewer registers), the next row's perm entry loads
    // from the start of a row and its metadata from the middle.
    int task = next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it);
    const bool h_cur = task >= 0 && task * W + slot < n_bin;
    const int g_raw = bin_row_issue(sc.perm, sc.err, b.na, start + task * W + slot, h_cur);
    int task_n = -1, g_n = -1;
    bool h_n = false;
    if constexpr (PF) {
        task_n = task >= 0 ? next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it) : -1;
        h_n = task_n >= 0 && task_n * W + slot < n_bin;
        g_n = bin_row_issue(sc.perm, sc.err, b.na, start + task_n * W + slot, h_n);
    }
    ProbCache pc;
    RowRaw mr = row_issue<MULTI>(b, sc, bin_row_checked(sc.err, b.na, g_raw, h_cur), pc);
    FirstChunk f;
    if constexpr (PF) {
        const RowMeta m0 = row_final<MULTI>(b, mr);
        const Prob P0 = prob_of<MULTI>(b, m0.t);
        first_a(P0, m0, lane, f);
        first_b(P0, f);
        asm volatile("" ::"v"(f.ka), "v"(f.sa), "v"(f.r0), "v"(f.r1), "v"(g_n));
    }
    // the loop starts with no load of the prologue pending: the wait counts
    // at the top of the loop are computed over both ways into it, and a load
    // pending from the prologue would make the first use there also wait
    // for the loads the previous row issued last
    asm volatile("" ::"v"(mr.nc), "v"(mr.c0), "v"(mr.a0), "v"(mr.a1));
    while (task >= 0) {
        // PF: the row after next; else the next row
        const int task_x = (!PF || task_n >= 0) ? next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it) : -1;
        const bool h_x = task_x >= 0 && task_x * W + slot < n_bin;
        const int g_x = bin_row_issue(sc.perm, sc.err, b.na, start + task_x * W + slot, h_x);
        RowRaw mr_n;
        if constexpr (PF) mr_n = row_issue<MULTI>(b, sc, bin_row_checked(sc.err, b.na, g_n, h_n), pc);

        const RowMeta m = row_final<MULTI>(b, mr);
        const Prob P = prob_of<MULTI>(b, m.t);
        const int nc = m.nc;
        tab.open(nc, lane, G);
        // descriptor fields into registers once per row, as global pointers
        const MLS_G int32_t *__restrict__ aci = gp(P.aci);
        const MLS_G double *__restrict__ aval = gp(P.aval);
        const MLS_G int32_t *__restrict__ brp = gp(P.brp);
        const MLS_G int32_t *__restrict__ bci = gp(P.bci);
        const MLS_G double *__restrict__ bval = gp(P.bval);
        const MLS_G int32_t *__restrict__ cci = gp(P.cci);
        MLS_G double *__restrict__ cval = gpw(P.cval);
        const int b_off = P.b_off, k_lo = P.k_lo, k_hi = P.k_hi;
        const bool accumulate = P.accumulate != 0;
        const int cs = m.cs, ps = m.ps, pe = m.pe;
        // the first chunk of row i of A: loaded during the previous row (PF),
        // else its entries now and its B row pointers after the insert
        if constexpr (!PF) first_a(P, m, lane, f);
        // a step over a part of B's rows skips the rows (of one chunk) with no
        // entry in it: most rows of A reach only a few parts
        bool skip = false;
        if (P.ranged) {
            // (the empty asm keeps the test, and the wait for the entries,
            // inside this branch)
            int kk = f.ka;
            asm volatile("" : "+v"(kk));
            const unsigned long long bal = __ballot(kk >= k_lo && kk < k_hi);
            const unsigned long long gm = (G == 64 ? ~0ull : ((1ull << G) - 1ull)) << (slot * G);
            skip = pe - ps <= G && (bal & gm) == 0ull;
        }
        nwave_sync();
        if (!skip) insert_row<G>(tab, acc, cci, cval, cs, nc, lane, accumulate);
        nwave_sync();
        if constexpr (!PF) {
            mr_n = row_issue<MULTI>(b, sc, bin_row_checked(sc.err, b.na, g_x, h_x), pc);
            first_b(P, f);
        }
        int ka = f.ka;
        double sa = f.sa;
        bool bad = false;
        const int pe_w = skip ? ps : pe;
        // stage a chunk: (q0, q1, a) of its entry pc + lane, from the B row
        // pointers as loaded; FLAT: the group's pair offsets and pair count
        int eq0 = 0, eq1 = 0;   // LONG: this lane's entry of the chunk
        double ea = 0.0;
        int fe_first = 0;       // FLAT: first pair of this lane's entry, if it has any
        bool fe_any = false;
        auto stage = [&](int q0r, int q1r, double a) -> int {
            const int sq0 = q0r - b_off, sq1 = q1r - b_off;
            int tot = 0;
            if constexpr (LONG) {
                eq0 = sq0;
                eq1 = sq1;
                ea = a;
                asm volatile("" : "+v"(ea));   // waited for here, not where the two ways join
                return tot;
            }
            if constexpr (FLAT) {
                // the non-empty entries compacted: (first B position - first pair, -, a)
                const int np = sq1 > sq0 ? sq1 - sq0 : 0;
                const int incl = group_scan_incl<G>(np, lane);
                tot = group_total<G>(np, incl) - 1;
                fe_first = incl - np;
                fe_any = np > 0;
                const uint32_t ne = (uint32_t)(__ballot(fe_any) >> (slot * G)) & 0xffu;
                if (fe_any)
                    par[__popc(ne & ((1u << lane) - 1u))] =
                        make_int4(sq0 - fe_first, 0, __double2loint(a), __double2hiint(a));
            } else {
                // (first, last B position, a); an empty row of B is (1, 0)
                const bool any = sq1 > sq0;
                par[lane] = make_int4(any ? sq0 : 1, any ? sq1 - 1 : 0, __double2loint(a), __double2hiint(a));
            }
            return tot;
        };
        // the first chunk is staged here from what was loaded during the
        // previous row (unused when the row has no chunk), the later ones in
        // the chunk loop: no loaded value reaches a point where the two ways
        // join, where its wait would also cover the loads issued since
        int last = stage(f.r0, f.r1, f.sa);   // FLAT: the chunk's last pair
        // PF: the next row's first A entries load during this row's steps
        RowMeta mn{};
        Prob Pn{};
        if constexpr (PF) {
            mn = row_final<MULTI>(b, mr_n);
            Pn = prob_of<MULTI>(b, mn.t);
            first_a(Pn, mn, lane, f);
        }
        for (int pc = ps; pc < pe_w; pc += G) {
            if (pc != ps) {
                // a later chunk: the B row pointers of the entries of A loaded
                // during the previous chunk
                const bool in = ka >= k_lo && ka < k_hi;
                const MLS_G int32_t *pb = in ? brp + (ka - k_lo) : (const MLS_G int32_t *)k_zeros4;
                last = stage(pb[0], pb[1], sa);
            }
            nwave_sync();
            // the next chunk's entries of A are in flight during this chunk's
            // steps (loaded without a branch: a default written into their
            // registers before a conditional load would wait for the loads of
            // the previous chunk, and with them for everything issued since)
            {
                const bool on = pc + G + lane < pe;
                ka = *(on ? aci + pc + G + lane : (const MLS_G int32_t *)k_ones4);
                sa = *(on ? aval + pc + G + lane : (const MLS_G double *)k_zeros4);
            }
            const int n = FLAT ? 0 : min(G, pe - pc);
            if constexpr (FLAT) {
                // kNumDepth * 8 pairs per tile, one bit per pair where an entry
                // starts (OR-ed over the group by DPP): a pair's entry is the count
                // of the bits up to it. Lanes of a step that belong to different
                // entries may hit the same output: they add entry by entry, so the
                // terms arrive in ascending k (one wave's LDS adds take effect in
                // program order).
                static_assert(G == 8 && (kNumDepth == 4 || kNumDepth == 8), "a tile of 32 or 64 pairs");
                int eb = -1;   // entries started before the tile, less one
                for (int base = 0; base <= last; base += G * kNumDepth) {
                    int jv[kNumDepth], rel[kNumDepth];
                    bool ok[kNumDepth];
                    double av[kNumDepth], bv[kNumDepth];
#pragma unroll
                    for (int h = 0; h < kNumDepth / 4; ++h) {
                        const int at = fe_first - base - 32 * h;
                        uint32_t m = fe_any && (uint32_t)at < 32u ? 1u << at : 0u;
                        m = group_or8(m);
#pragma unroll
                        for (int d4 = 0; d4 < 4; ++d4) {
                            const int d = 4 * h + d4;
                            const int pp = base + d * G + lane;
                            const int e0 = eb + __popc(m & ((2u << (8 * d4)) - 1u));   // the step's first lane's entry
                            const int en = eb + __popc(m & ((2u << (8 * d4 + lane)) - 1u));
                            rel[d] = en - e0;
                            ok[d] = pp <= last;
                            const int4 pr = par[en];   // (past the pairs: the last entry's last pair again)
                            const uint32_t q = (uint32_t)(pr.x + or_last(ok[d], pp, last));
                            jv[d] = bci[q];
                            bv[d] = bval[q];
                            av[d] = __hiloint2double(pr.w, pr.z);
                        }
                        eb += __popc(m);
                    }
                    // (every load before the first use of a loaded column)
                    __builtin_amdgcn_sched_barrier(0);
                    uint32_t posv[kNumDepth];
                    tab.template lookup_n<kNumDepth>(jv, ok, posv);
#pragma unroll
                    for (int d = 0; d < kNumDepth; ++d) asm volatile("" ::"v"(bv[d]));
#pragma unroll
                    for (int d = 0; d < kNumDepth; ++d) {
                        const bool hit = ok[d] && posv[d] <= tab.kMaxPos;
                        bad |= ok[d] && !hit;
                        const double t = av[d] * bv[d];
                        const int rk = hit ? rel[d] : -1;
                        for (int rr = 0;; ++rr) {
                            if (rk == rr) atomicAdd(acc + posv[d], t);
                            if (!__ballot(rk > rr)) break;
                        }
                    }
                }
            }
            // kNumDepth staged steps, no row of B longer than G: their B loads are
            // issued together, then accumulated in step order
            auto batch = [&](int u0, const int2 (&qr)[kNumDepth]) {
                int jv[kNumDepth];
                bool ok[kNumDepth];
                double bv[kNumDepth], av[kNumDepth];
                // lanes past their row of B load its last entry again (B's first for
                // an empty row; neither looked up nor added), so no branch
                // surrounds the loads
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) {
                    const int q = qr[d].x + lane;
                    ok[d] = q <= qr[d].y;
                    const uint32_t qi = (uint32_t)or_last(ok[d], q, qr[d].y);
                    jv[d] = bci[qi];
                    bv[d] = bval[qi];
                }
                // keep the scheduler from hoisting uses of the loaded columns
                // above the later loads (each would wait for a load)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) av[d] = *((const double *)(par + u0 + d) + 1);
                // positions first (independent LDS reads), then the adds in step
                // order; within a step the lanes hold distinct columns of B_k, so
                // no two lanes add to the same slot and every slot gets its terms
                // in ascending k. The LDS fp64 add rounds like a plain add.
                uint32_t posv[kNumDepth];
                tab.template lookup_n<kNumDepth>(jv, ok, posv);
                // every loaded value is consumed on every path (an empty asm
                // use), so no load is left pending into the next batch
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) asm volatile("" ::"v"(bv[d]));
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) {
                    const bool hit = ok[d] && posv[d] <= tab.kMaxPos;
                    bad |= ok[d] && !hit;
                    if (hit) atomicAdd(acc + posv[d], av[d] * bv[d]);
                }
            };
            if constexpr (LONG)
                bad |= flat_chunk<kNumDepth, false>(tab, acc, par, flags, lane, eq0, eq1, ea, bci, bval,
                                             INT_MIN, INT_MAX);
            for (int u0 = 0; !LONG && u0 < n; u0 += kNumDepth) {
                // The staged entries are read together (all G are written every
                // chunk, those past the row as empty ranges, and G is a multiple of
                // kNumDepth).
                int2 qr[kNumDepth];
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) qr[d] = *(const int2 *)(par + u0 + d);
                bool longs = false;   // a step whose row of B is longer than G
#pragma unroll
                for (int d = 0; d < kNumDepth; ++d) longs |= qr[d].y - qr[d].x >= G;
                if (__ballot(longs)) {
                    // one step at a time, each through all of its row of B: its
                    // entries have distinct columns, so the order is kept
#pragma unroll 1
                    for (int d = 0; d < kNumDepth; ++d) {
                        const int4 pr = par[u0 + d];
                        const double a = __hiloint2double(pr.w, pr.z);
                        for (int q = pr.x + lane; q <= pr.y; q += G) {
                            const uint32_t pos = tab.lookup(bci[q]);
                            if (pos <= tab.kMaxPos) atomicAdd(acc + pos, a * bval[q]);
                            else bad = true;
                        }
                    }
                    continue;
                }
                batch(u0, qr);
            }
            nwave_sync();
        }
        // the next row's metadata is taken before this row's stores are
        // issued (a wait for it at the next row's start would also wait for
        // the stores: the counter covers both)
        asm volatile("" ::"v"(mr_n.nc), "v"(mr_n.c0), "v"(mr_n.a0), "v"(mr_n.a1));
        // PF: the next row's B row pointers (its A entries arrived during the steps)
        if constexpr (PF) first_b(Pn, f);
        if (bad) atomicOr(sc.err, kErrStructure);
        if (!skip)
            for (int e = lane; e < nc; e += G) cval[cs + e] = acc[e];
        else if (!accumulate)
            for (int e = lane; e < nc; e += G) cval[cs + e] = 0.0;
        nwave_sync();
        if constexpr (PF) {
            task = task_n;
            task_n = task_x;
            g_n = g_x;
            h_n = h_x;
        } else {
            task = task_x;
        }
        mr = mr_n;
    }
}

template <int G, int CAP, bool PACK, bool MULTI, bool FLAT>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(
    NumShape<G, CAP, PACK, MULTI, FLAT>::OCC_R))) void k_num_lds(Batch b, Sched sc, int bin)
{
    __shared__ __attribute__((aligned(16))) char s_mem[NumShape<G, CAP, PACK, MULTI, FLAT>::LDS];
    num_lds_rows<G, CAP, PACK, MULTI, FLAT, 65536>(b, sc, bin, s_mem, (int)blockIdx.x, (int)gridDim.x);
}

// first position in cols[lo, hi) whose column is >= j
__device__ __forceinline__ int lower_col(const MLS_G int32_t *cols, int lo, int hi, int j)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cols[mid] < j) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// the same, expected near lo: steps that double from lo on, then a search
// between the last two (their reads stay in the lines that the window's pairs
// are read from)
__device__ __forceinline__ int lower_col_near(const MLS_G int32_t *cols, int lo, int hi, int j)
{
    int step = 8;
    while (lo + step < hi && cols[lo + step] < j) {
        lo += step + 1;
        step *= 2;
    }
    return lower_col(cols, lo, min(lo + step, hi), j);
}

// Tasks of the spill rows, one workgroup: wstart[r] = first task of the r-th
// row of the spill bin, wstart[n] = the total. A row has ceil(nc / m) windows,
// one per task or (blocks, and more than kWinSpread windows) win_block of its
// entries. Latency bound (perm, then
// the row's size and entries): four rows per thread in flight. 20400 spill
// rows of the R-MAT 16 square: 87 us with 256 rows per step, 31 us.
__global__ __launch_bounds__(kWinScanWG) void k_win_scan(Batch b, Sched sc, int m, int blocks)
{
    constexpr int NW = kWinScanWG / kWave, R = 4;
    __shared__ int s_red[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = gp(sc.bin_count)[kBinSpill];
    const int start = bin_start(sc.bin_count, kBinSpill);
    MLS_G int32_t *ws = gpw(sc.wstart);
    ProbCache pc;
    int carry = 0;
    // (one step's rows may have few windows; more spill rows have at least 5 each)
    if (blocks && n <= kWinScanWG * R) {
        int w = 0;
        for (int r = (int)threadIdx.x; r < n; r += kWinScanWG) {
            const int g = bin_row(sc.perm, sc.err, b.na, start + r);
            w += g >= 0 ? (gp(sc.val)[g] + m - 1) / m : 0;
        }
        w = group_sum<kWave>(w);
        if (lane == 0) s_red[wave] = w;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int x = 0; x < NW; ++x) all += s_red[x];
        blocks = all > kWinSpread;
        __syncthreads();
    }
    for (int r0 = 0; r0 < n; r0 += kWinScanWG * R) {
        const int r = r0 + (int)threadIdx.x * R;
        int g[R], c[R], sum = 0;
#pragma unroll
        for (int x = 0; x < R; ++x) g[x] = r + x < n ? bin_row(sc.perm, sc.err, b.na, start + r + x) : -1;
#pragma unroll
        for (int x = 0; x < R; ++x) {
            c[x] = g[x] >= 0 ? (gp(sc.val)[g[x]] + m - 1) / m : 0;
            if (blocks && g[x] >= 0) {
                const int t = b.nprob == 1 ? 0 : find_prob_cached(b.abase, b.nprob, g[x], pc);
                const MLS_G int32_t *arp = gp(get_prob(b, t).arp) + (g[x] - (b.nprob == 1 ? 0 : pc.lo));
                const int per = win_block(arp[1] - arp[0]);
                c[x] = (c[x] + per - 1) / per;
            }
        }
#pragma unroll
        for (int x = 0; x < R; ++x) sum += c[x];
        const int incl = group_scan_incl<kWave>(sum, lane);
        if (lane == kWave - 1) s_red[wave] = incl;
        __syncthreads();
        int off = carry + incl - sum;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            off += x < wave ? s_red[x] : 0;
            carry += s_red[x];
        }
#pragma unroll
        for (int x = 0; x < R; ++x) {
            if (r + x < n) ws[r + x] = off;
            off += c[x];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) ws[n] = carry;
}

// LDS of one spill window: table, accumulators, staged entries, the start bits
// of their pairs and where the window ended in the entries' rows of B
constexpr int win_bytes(int CAP, bool PACK)
{
    return CAP * (PACK ? 4 : 8) + (CAP / 2) * 8 + kWave * 16 + kFlatWords * 4 + kWinCarry * 2;
}

// A window streams the whole row of A, its rows of B narrowed to the window's
// columns, as flattened pairs (flat_chunk). What bounds it: the latency of the
// dependent loads per window (a third of the issue slots are used, 4 waves per
// SIMD by LDS): the task's row, the entries of A, their rows of B and the
// searches in them, then the pairs. R-MAT 16 square, 306000 windows: 4.06 ms
// with a window per task, 2.78 ms with win_block windows per task, where the
// first column of a window needs no search and its last is searched from there.
template <int CAP, bool PACK, int MAXLDS = 65536>
struct WinShape {
    static constexpr int M = CAP / 2;   // positions of C per window
    static constexpr int NW = nw_num(win_bytes(CAP, PACK), 1, MAXLDS);
    static constexpr int TW = PACK ? CAP : 2 * CAP;
    static constexpr int LDS_PAR = NW * TW * 4;
    static constexpr int LDS_ACC = LDS_PAR + NW * kWave * 16;
    static constexpr int LDS_FLAGS = LDS_ACC + NW * M * 8;
    static constexpr int LDS_OFF = LDS_FLAGS + NW * kFlatWords * 4;
    static constexpr int LDS = LDS_OFF + NW * kWinCarry * 2;
};

// lds: WinShape::LDS bytes of this workgroup
template <int CAP, bool PACK, bool MULTI, int MAXLDS>
__device__ __forceinline__ void num_win_rows(const Batch &b, const Sched &sc, char *lds)
{
    using Shape = WinShape<CAP, PACK, MAXLDS>;
    constexpr int G = kWave;
    constexpr int M = Shape::M;
    constexpr int NW = Shape::NW;
    constexpr int TW = Shape::TW;
    uint32_t *s_tab = (uint32_t *)lds;
    int4 *s_par = (int4 *)(lds + Shape::LDS_PAR);    // staged entries: (first B position, -, a)
    double *s_acc = (double *)(lds + Shape::LDS_ACC);
    uint32_t *flags = (uint32_t *)(lds + Shape::LDS_FLAGS) + (threadIdx.x >> 6) * kFlatWords;

    const int wave = threadIdx.x >> 6;
    if (wave >= NW) return;
    const int lane = threadIdx.x & 63;
    PosTab<CAP, PACK, 2> tab{s_tab + wave * TW};
    double *acc = s_acc + wave * M;
    int4 *par = s_par + wave * G;

    const int n_bin = gp(sc.bin_count)[kBinSpill];
    const int start = bin_start(sc.bin_count, kBinSpill);
    const MLS_G int32_t *wst = gp(sc.wstart);
    const int ntasks = n_bin > 0 ? wst[n_bin] : 0;
    uint16_t *off = (uint16_t *)(lds + Shape::LDS_OFF) + wave * kWinCarry;
    // one counter over all tasks: their work varies too much (a hub row's
    // windows are consecutive and long) for per-XCD slabs
    if (ntasks == 0) return;
    int32_t *cursor = sc.task_cursor + kBinSpill * kXcd;
    ProbCache pcache;
    for (;;) {
        int u = 0;
        if (lane == 0) u = atomicAdd(cursor, 1);
        u = __builtin_amdgcn_readlane(u, 0);
        if (u >= ntasks) break;
        const int r = find_last_wave(wst, n_bin, u);   // the row of task u
        const int g = bin_row(sc.perm, sc.err, b.na, start + r);
        if (g < 0) continue;
        int t = 0, i = g;
        if (MULTI) {
            t = find_prob_cached(b.abase, b.nprob, g, pcache);
            i = g - pcache.lo;
        }
        const Prob P = prob_of<MULTI>(b, t);
        const MLS_G int32_t *__restrict__ aci = gp(P.aci);
        const MLS_G double *__restrict__ aval = gp(P.aval);
        const MLS_G int32_t *__restrict__ brp = gp(P.brp);
        const MLS_G int32_t *__restrict__ bci = gp(P.bci);
        const MLS_G double *__restrict__ bval = gp(P.bval);
        const MLS_G int32_t *__restrict__ cci = gp(P.cci);
        MLS_G double *__restrict__ cval = gpw(P.cval);
        const int b_off = P.b_off, k_lo = P.k_lo, k_hi = P.k_hi;
        const bool accumulate = P.accumulate != 0;
        const int nc = gp(sc.val)[g];
        const int cr = gp(P.crp)[i] - P.c_off;
        const int ps = gp(P.arp)[i] - P.a_off, pe = gp(P.arp)[i + 1] - P.a_off;
        // (one window per task where k_win_scan gave the row as many tasks)
        const int w0 = wst[r];
        const int per = wst[r + 1] - w0 == (nc + M - 1) / M ? 1 : win_block(pe - ps);
        const bool narrow = nc > M;
        bool bad = false;
        // first positions of the task's windows in the row
        const int cb = (u - w0) * per * M, ce = min(nc, cb + per * M);
        for (int c0 = cb; c0 < ce; c0 += M) {
            const int cs = cr + c0;
            const int n = min(M, nc - c0);
            // columns the window takes: from its first to its last column, open
            // below for the row's first window and above for its last, so that
            // a column outside the whole row still fails the lookup
            const int jlo = c0 == 0 ? INT_MIN : cci[cs];
            const int jhi = c0 + n == nc ? INT_MAX : cci[cs + n - 1];
            tab.open(n, lane, G);
            nwave_sync();
            insert_row<G>(tab, acc, cci, cval, cs, n, lane, accumulate);
            nwave_sync();
            for (int pc = ps; pc < pe; pc += G) {
                // stage the chunk: entry pc + lane's row of B, narrowed to the
                // window's columns when it is long, and its pair count; the
                // task's next window starts where this one ends
                int sq0 = 0, sq1 = 0;
                double sa = 0.0;
                if (pc + lane < pe) {
                    const int ka = aci[pc + lane];
                    sa = aval[pc + lane];
                    if (ka >= k_lo && ka < k_hi) {
                        sq0 = brp[ka - k_lo] - b_off;
                        sq1 = brp[ka - k_lo + 1] - b_off;
                        if (narrow && sq1 - sq0 > 32) {
                            const int q = sq0, e = pc - ps + lane;
                            const int at = c0 > cb ? (int)off[e] : 0xffff;
                            if (at != 0xffff) sq0 += at;
                            else if (jlo != INT_MIN) sq0 = lower_col(bci, sq0, sq1, jlo);
                            if (jhi != INT_MAX) sq1 = lower_col_near(bci, sq0, sq1, jhi + 1);
                            if (c0 + M < ce) off[e] = (uint16_t)min(sq1 - q, 0xffff);
                        }
                    }
                }
                bad |= flat_chunk<kWinDepth, true>(tab, acc, par, flags, lane, sq0, sq1, sa, bci, bval, jlo, jhi);
            }
            for (int e = lane; e < n; e += G) cval[cs + e] = acc[e];
            nwave_sync();
        }
        if (bad) atomicOr(sc.err, kErrStructure);
    }
}

template <int CAP, bool PACK, bool MULTI>
__global__ __launch_bounds__(kWG) void k_num_win(Batch b, Sched sc)
{
    __shared__ __attribute__((aligned(16))) char s_mem[WinShape<CAP, PACK>::LDS];
    num_win_rows<CAP, PACK, MULTI, 65536>(b, sc, s_mem);
}

// Products of few rows: every class and the spill windows in one launch, the
// workgroups divided among the bins by their work (each bin with rows gets at
// least one). The classes' own launches cost at least 4.7 us of stream time
// each, empty or not, and seven of them (with the window scan) are saved. A
// workgroup has as many waves per class as kAllLds holds, and the rows of the
// largest class (33 KB each) run as windows, so that LDS leaves six workgroups
// resident per CU (registers leave four). Numeric phase of 5000 random rows of 36 outputs 46 -> 22 us, of
// the 64x64 Laplacian square 36 -> 15 us.
constexpr int kAllLds = 24576;

using NumAll0 = NumShape<8, kFillCap[0], true, false, true, kAllLds>;
using NumAll1 = NumShape<32, kFillCap[1], true, false, false, kAllLds>;
using NumAll2 = NumShape<64, kFillCap[2], true, false, false, kAllLds>;
using NumAll3 = NumShape<64, kFillCap[3], true, false, false, kAllLds>;
using NumAllW = WinShape<kNumWinCap, true, kAllLds>;
static_assert(NumAll0::LDS <= kAllLds && NumAll1::LDS <= kAllLds && NumAll2::LDS <= kAllLds &&
              NumAll3::LDS <= kAllLds && NumAllW::LDS <= kAllLds, "one LDS buffer for every part");

__global__ __launch_bounds__(kWG) void k_num_all(Batch b, Sched sc)
{
    __shared__ __attribute__((aligned(16))) char s_mem[kAllLds];
    // rows (windows) per workgroup of each part
    const int per[kNumClasses + 1] = {NumAll0::W * NumAll0::NW, NumAll1::W * NumAll1::NW, NumAll2::NW, NumAll3::NW,
                                      1, NumAllW::NW};
    int vblk, vgrid;
    switch (part_of_block(sc, per, vblk, vgrid)) {
    case 0: num_lds_rows<8, kFillCap[0], true, false, true, kAllLds>(b, sc, 0, s_mem, vblk, vgrid); break;
    case 1: num_lds_rows<32, kFillCap[1], true, false, false, kAllLds>(b, sc, 1, s_mem, vblk, vgrid); break;
    case 2: num_lds_rows<64, kFillCap[2], true, false, false, kAllLds>(b, sc, 2, s_mem, vblk, vgrid); break;
    case 3: num_lds_rows<64, kFillCap[3], true, false, false, kAllLds>(b, sc, 3, s_mem, vblk, vgrid); break;
    case kNumClasses: num_win_rows<kNumWinCap, true, false, kAllLds>(b, sc, s_mem); break;
    }
}

// ---------------------------------------------------------------------------

template <typename K>
static int persistent_grid_n(K kernel, int threads)
{
    static int cus = device_cu_count();
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return cus * per_cu;
}

template <int G, int CAP, bool PACK, bool MULTI, bool FLAT>
static void launch_num_variant(const Batch &b, const Sched &sc, int bin, hipStream_t s)
{
    constexpr int NW = NumShape<G, CAP, PACK, MULTI, FLAT>::NW;
    static int grid = persistent_grid_n(k_num_lds<G, CAP, PACK, MULTI, FLAT>, NW * kWave);
    static char name[64];
    if (!name[0])
        snprintf(name, sizeof(name), "num_lds_G%d_C%d%s%s%s", G, CAP, PACK ? "_p" : "", MULTI ? "_b" : "", FLAT ? "_f" : "");
    ProfScope ps(name, s);
    hipLaunchKernelGGL((k_num_lds<G, CAP, PACK, MULTI, FLAT>), dim3(grid), dim3(NW * kWave), 0, s, b, sc, bin);
}

template <int G, int CAP, bool PACK>
static void launch_num_multi(const Batch &b, const Sched &sc, int bin, hipStream_t s)
{
    constexpr bool FLAT = kNumFlat && G <= kNumFlatMaxG;
    if (b.nprob > 1) launch_num_variant<G, CAP, PACK, true, FLAT>(b, sc, bin, s);
    else launch_num_variant<G, CAP, PACK, false, FLAT>(b, sc, bin, s);
}

// The packed table needs every column index below PackBits<CAP>::kMaxCols.
template <int G, int CAP>
static void launch_num_class(const Batch &b, const Sched &sc, int bin, hipStream_t s)
{
    if (b.max_ncols > 0 && (uint32_t)b.max_ncols <= PackBits<CAP>::kMaxCols)
        launch_num_multi<G, CAP, true>(b, sc, bin, s);
    else
        launch_num_multi<G, CAP, false>(b, sc, bin, s);
}

template <int CAP, bool PACK, bool MULTI>
static void launch_num_win(const Batch &b, const Sched &sc, hipStream_t s)
{
    constexpr int NW = WinShape<CAP, PACK>::NW;
    static int grid = persistent_grid_n(k_num_win<CAP, PACK, MULTI>, NW * kWave);
    static char name[64];
    if (!name[0]) snprintf(name, sizeof(name), "num_spill_C%d%s%s", CAP, PACK ? "_p" : "", MULTI ? "_b" : "");
    ProfScope ps(name, s);
    hipLaunchKernelGGL(k_win_scan, dim3(1), dim3(kWinScanWG), 0, s, b, sc, CAP / 2, 1);
    hipLaunchKernelGGL((k_num_win<CAP, PACK, MULTI>), dim3(grid), dim3(NW * kWave), 0, s, b, sc);
}

static void launch_num_spill(const Batch &b, const Sched &sc, hipStream_t s)
{
    constexpr int CAP = kNumWinCap;
    const bool pack = b.max_ncols > 0 && (uint32_t)b.max_ncols <= PackBits<CAP>::kMaxCols;
    if (b.nprob > 1) {
        if (pack) launch_num_win<CAP, true, true>(b, sc, s);
        else launch_num_win<CAP, false, true>(b, sc, s);
    } else {
        if (pack) launch_num_win<CAP, true, false>(b, sc, s);
        else launch_num_win<CAP, false, false>(b, sc, s);
    }
}

void launch_numeric_groups(const Batch &b, const Sched &sc, int G1, int G2, const int32_t *n_bin, hipStream_t s)
{
    if (b.na <= 0) return;
    auto rows = [&](int bin) { return !n_bin || n_bin[bin] > 0; };
    if (rows(0)) launch_num_class<8, kFillCap[0]>(b, sc, 0, s);
    if (rows(1)) {
        switch (G1) {
        case 8: launch_num_class<8, kFillCap[1]>(b, sc, 1, s); break;
        case 16: launch_num_class<16, kFillCap[1]>(b, sc, 1, s); break;
        case 64: launch_num_class<64, kFillCap[1]>(b, sc, 1, s); break;
        default: launch_num_class<32, kFillCap[1]>(b, sc, 1, s); break;
        }
    }
    if (rows(2)) {
        if (G2 >= 64) launch_num_class<64, kFillCap[2]>(b, sc, 2, s);
        else launch_num_class<32, kFillCap[2]>(b, sc, 2, s);
    }
    if (rows(3)) launch_num_class<64, kFillCap[3]>(b, sc, 3, s);
    if (rows(4)) launch_num_class<64, kFillCap[4]>(b, sc, 4, s);
    if (rows(kBinSpill)) launch_num_spill(b, sc, s);
}

bool small_rows_fit(const Batch &b)
{
    return b.nprob == 1 && b.na > 0 && b.na <= kSmallRows && b.max_ncols > 0 &&
           (uint32_t)b.max_ncols <= PackBits<kFillCap[4]>::kMaxCols;
}

// Two launches or one per class, by the outputs and their mean per row. Numeric
// phase in us, by class / two launches (rows x outputs, entries of A times of B):
//   up to 512 outputs, always two: 4 x 450 (22 x 20) 44 / 19, 20000 x 450 139 / 130
//   up to 2048, 2^20 outputs: 1000 x 900 (45 x 20) 54 / 34, 4000 x 900 82 / 96, 4 x
//     1500 (15 x 100) 50 / 26, 1000 x 1500 59 / 98; and, past 1024, from 2^24 on,
//     where their windows overtake the 4096-slot class again: 4000 x 1500 138 / 169,
//     10000 x 1500 287 / 300, 20000 x 1500 573 / 541, 20000 x 1776 (30 x 60) 723 / 632
//   more (windows either way), 2^24: 4 x 2500 (25 x 100) 90 / 26, 4000 x 2500 239 / 218,
//     10000 x 2500 402 / 451, 16 x 20000 (200 x 100) 109 / 51, 250 x 20000 260 / 220,
//     1000 x 20000 590 / 661
bool num_small_fit(const Batch &b, int64_t outputs)
{
    if (!small_rows_fit(b)) return false;
    const int64_t mean = outputs / b.na;
    if (mean <= 512) return true;
    if (mean <= 2048) return outputs <= 1ll << 20 || (mean > 1024 && outputs >= 1ll << 24);
    return outputs <= 1ll << 24;
}

// Two rows per workgroup in the larger classes, and two windows of 512 outputs in
// the spill bin: from the rows alone, a few long ones had too few workgroups (16
// rows of 20000 outputs: 658 us).
int small_rows_grid(int na, int64_t outputs)
{
    const int64_t want = na / 2 + kNumBins + outputs / kNumWinCap;
    return want < kSmallGrid ? (int)want : kSmallGrid;
}

void launch_numeric_small(const Batch &b, const Sched &sc, int64_t outputs, hipStream_t s)
{
    launch_bin_small(b, sc, kNumWinCap / 2, 1, s);
    ProfScope ps("num_all", s);
    hipLaunchKernelGGL(k_num_all, dim3(small_rows_grid(b.na, outputs)), dim3(kWG), 0, s, b, sc);
}

void launch_numeric(const Batch &b, const Sched &sc, int G, hipStream_t s)
{
    launch_numeric_groups(b, sc, G, G >= 64 ? 64 : 32, nullptr, s);
}

}  // namespace mls
