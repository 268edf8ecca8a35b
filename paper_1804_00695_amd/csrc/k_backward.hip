// k_backward.hip -- adjoint of loss(A, B) = sum_ij W_ij (A*B)_ij with W given
// on the pattern of C = A*B (the product's reverse mode; not in the paper):
//   dA_ik = sum_{j in B_k} W_ij b_kj      (only on the pattern of A)
//   dB_kj = sum_{i : k in A_i} a_ik W_ij  (only on the pattern of B)
// Fused, with no dense or product-sized intermediate: G lanes own row i;
// W_i goes into an LDS hash (column -> W value); the pairs (entry (i, k),
// entry of B_k) of a chunk of A_i are flattened, one per lane: each looks up
// W_ij, adds W_ij b_kj to the entry's dA sum in LDS and a_ik W_ij into dB
// with a device fp64 atomic.
// Rows of W too long for LDS are cut into windows of consecutive positions of
// W_i, each a task of one wave with its own LDS hash; a window streams the
// row of A with its rows of B narrowed to the window's column range, and adds
// its part of dA_ik with a device atomic.
//
// Also here: CSR transpose (count, scan, scatter, per-row sort) and a masked
// gather out[e] = X(row(e), col(e)) over a pattern, used by the unfused
// per-call adjoint (W B^T masked to pat(A), A^T W masked to pat(B)).
#include <algorithm>
#include <climits>
#include <cstdio>

#include "common.h"
#include "launch.h"
#include "postab.h"
#include "profile.h"

namespace mls {

constexpr int kBwdUnroll = 4;

__device__ __forceinline__ void bwd_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

constexpr int nw_bwd(int row_bytes, int rows_per_wave, int lds = 65536)
{
    int per_wave = row_bytes * rows_per_wave;
    int nw = lds / per_wave;
    return nw > 4 ? 4 : (nw < 1 ? 1 : nw);
}

// W_i's hash: column keys (-1 empty) in buckets of 4 slots (16 bytes), W
// values beside them. A column takes the first empty slot at or after the
// start of its home bucket, so a bucket's filled slots are a prefix of it and
// a bucket whose last slot is empty ends a search.
__device__ __forceinline__ uint32_t w_home(int logcap, int j) { return hslot32((uint32_t)j, logcap - 2) << 2; }

__device__ __forceinline__ void w_insert(int *key, double *wv, int logcap, int j, double w)
{
    const uint32_t cmask = (1u << logcap) - 1u;
    uint32_t h = w_home(logcap, j);
    for (uint32_t probe = 0; probe <= cmask; probe += 4) {
        const int4 k = *(const int4 *)(key + h);
        int sl = k.x == -1 ? 0 : (k.y == -1 ? 1 : (k.z == -1 ? 2 : (k.w == -1 ? 3 : 4)));
        for (; sl < 4; ++sl)
            if (atomicCAS(key + h + sl, -1, j) == -1) { wv[h + sl] = w; return; }
        h = (h + 4u) & cmask;
    }
}

// slot of column j given the keys k of its home bucket h, or -1 when absent
__device__ __forceinline__ int w_slot(const int *key, int logcap, int j, uint32_t h, int4 k)
{
    const int sl = k.x == j ? 0 : (k.y == j ? 1 : (k.z == j ? 2 : (k.w == j ? 3 : -1)));
    if (sl >= 0) return (int)h + sl;
    if (k.w == -1) return -1;
    const uint32_t cmask = (1u << logcap) - 1u;
    for (uint32_t probe = 4; probe <= cmask; probe += 4) {   // the home bucket is full: rarely
        h = (h + 4u) & cmask;
        const int4 v = *(const int4 *)(key + h);
        const int s2 = v.x == j ? 0 : (v.y == j ? 1 : (v.z == j ? 2 : (v.w == j ? 3 : -1)));
        if (s2 >= 0) return (int)h + s2;
        if (v.w == -1) return -1;
    }
    return -1;
}

// slots of D columns (-2 where jv < 0), the home buckets of a pair read
// before either is searched, then the W values of all D read together
template <int D>
__device__ __forceinline__ void w_lookup_n(const int *key, const double *wv, int logcap, const int (&jv)[D],
                                           int (&sl)[D], double (&w)[D])
{
    static_assert(D % 2 == 0, "looked up in pairs");
#pragma unroll
    for (int d0 = 0; d0 < D; d0 += 2) {
        uint32_t hv[2];
        int4 kv[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) hv[d] = jv[d0 + d] >= 0 ? w_home(logcap, jv[d0 + d]) : 0u;
#pragma unroll
        for (int d = 0; d < 2; ++d) kv[d] = *(const int4 *)(key + hv[d]);
#pragma unroll
        for (int d = 0; d < 2; ++d) sl[d0 + d] = jv[d0 + d] >= 0 ? w_slot(key, logcap, jv[d0 + d], hv[d], kv[d]) : -2;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) w[d] = wv[sl[d] >= 0 ? sl[d] : 0];
}

// LDS of one row: W_i's hash (wide: key and value per slot; packed: a
// column -> position table and the values by position), the staged entries
// of A (B position, a_ik, their dA sums) and, for groups of 32 or 64 lanes, the
// start bits of a tile of pairs
constexpr int bwd_flag_words(int G) { return G >= 32 ? G * kBwdUnroll / 32 : 0; }

constexpr int bwd_row_bytes(int CAP, int G, bool PACK)
{
    return (PACK ? CAP * 4 + (CAP / 2) * 8 : CAP * 12) + G * 20 + bwd_flag_words(G) * 4;
}

// Waves per workgroup that keep the most waves resident on a CU (160 KB of
// LDS, 32 waves), given the LDS of one wave and the most a workgroup may have.
constexpr int nw_bwd_best(int wave_bytes, int lds)
{
    int best = 1, best_w = 0;
    for (int nw = 1; nw <= 4; ++nw) {
        int wgs = 163840 / (nw * wave_bytes);
        int w = wgs * nw;
        if (w > 32) w = 32;
        if (lds < nw * wave_bytes) w = 0;   // a workgroup's LDS stays within lds
        if (w >= best_w) { best = nw; best_w = w; }
    }
    return best;
}

// Rows of W in LDS: G lanes own row i. The pairs (entry of A_i, position in
// B_k) of a staged chunk of A_i are flattened and taken G at a time, one per
// lane: W_ij is looked up, a_ik W_ij goes to dB with a device atomic and
// W_ij b_kj to the entry's dA sum in LDS, written out once per entry.
// Latency: a row's metadata (size, row pointers of W and A) is loaded while
// the previous row runs, the first chunk of A_i while W_i is hashed, each
// lane's columns and values of W_i kInsDepth at a time before they are
// inserted, and the next chunk of A_i while the current one's pairs run.
constexpr int kBwdInsDepth = 4;

struct BwdMeta {
    int nw, ws0, ps, pe;
};

// The loads of a row's metadata (size of W_i, row pointers of W and A),
// issued without a branch around them (a slot without a row reads zeros: no
// entries) so that their first use can sit a row later.
__device__ __forceinline__ BwdMeta bwd_meta_issue(const Prob &P, const Sched &sc, int g)
{
    const bool on = g >= 0;
    const MLS_G int32_t *zero = (const MLS_G int32_t *)k_zeros4;
    const MLS_G int32_t *pv = on ? gp(sc.val) + g : zero;
    const MLS_G int32_t *pc = on ? gp(P.crp) + g : zero;
    const MLS_G int32_t *pa = on ? gp(P.arp) + g : zero;
    BwdMeta m;
    m.nw = *pv;
    m.ws0 = *pc;
    m.ps = pa[0];
    m.pe = pa[1];
    return m;
}

// A row's first chunk, located in advance: entries ps + lane of A_i (column
// -1 and value 0 past the row), then their rows' bounds in B (zeros past the
// row: no pairs).
struct BwdFirst {
    int ka;
    double sa;
    int q0, q1;
};

__device__ __forceinline__ void bwd_first_a(const Prob &P, const BwdMeta &m, int lane, BwdFirst &f)
{
    const bool on = m.ps + lane < m.pe;
    f.ka = *(on ? gp(P.aci) + m.ps + lane : (const MLS_G int32_t *)k_ones4);
    f.sa = *(on ? gp(P.aval) + m.ps + lane : (const MLS_G double *)k_zeros4);
}

__device__ __forceinline__ void bwd_first_b(const Prob &P, BwdFirst &f)
{
    const MLS_G int32_t *pb = f.ka >= 0 ? gp(P.brp) + f.ka : (const MLS_G int32_t *)k_zeros4;
    f.q0 = pb[0];
    f.q1 = pb[1];
}

template <int G, int CAP, bool PACK, int MAXLDS = 65536>
struct BwdShape {
    static constexpr int W = kWave / G;
    static constexpr int NW = nw_bwd_best(bwd_row_bytes(CAP, G, PACK) * W, MAXLDS);
    static constexpr int WV = PACK ? CAP / 2 : CAP;   // W values per row: by position, or by slot
    static constexpr int LDS_WV = NW * W * CAP * 4;
    static constexpr int LDS_PA = LDS_WV + NW * W * WV * 8;
    static constexpr int LDS_DA = LDS_PA + NW * W * G * 8;
    static constexpr int LDS_FLAGS = LDS_DA + NW * W * G * 8;
    static constexpr int LDS_PQ = LDS_FLAGS + NW * W * bwd_flag_words(G) * 4;
    static constexpr int LDS = LDS_PQ + NW * W * G * 4;
};

// The rows of one bin on the workgroups vblk of vgrid; lds: BwdShape::LDS bytes
// of this workgroup.
template <int G, int CAP, bool PACK, int MAXLDS>
__device__ __forceinline__ void bwd_lds_rows(const Batch &b, const Sched &sc, int bin, double *dA, double *dB,
                                             char *lds, int vblk, int vgrid)
{
    using Shape = BwdShape<G, CAP, PACK, MAXLDS>;
    constexpr int W = Shape::W;
    constexpr int NW = Shape::NW;
    constexpr int WV = Shape::WV;
    int *s_key = (int *)lds;
    double *s_wv = (double *)(lds + Shape::LDS_WV);
    double *s_pa = (double *)(lds + Shape::LDS_PA);
    double *s_da = (double *)(lds + Shape::LDS_DA);
    uint32_t *s_flags = (uint32_t *)(lds + Shape::LDS_FLAGS);   // start bits, read four words at a time
    int *s_pq = (int *)(lds + Shape::LDS_PQ);

    const int wave = threadIdx.x >> 6;
    if (wave >= NW) return;
    const int lw = threadIdx.x & 63;
    const int slot = lw / G, lane = lw % G;
    const int rs = wave * W + slot;
    int *key = s_key + rs * CAP;
    double *wv = s_wv + rs * WV;
    PosTab<CAP, true, 4> ptab{(uint32_t *)key};   // PACK: column -> position of W_i
    double *pa = s_pa + rs * G;
    double *da = s_da + rs * G;
    int *pq = s_pq + rs * G;
    uint32_t *flags = s_flags + rs * bwd_flag_words(G);   // groups of 32 or 64 lanes

    const Prob P = b.p0;
    const MLS_G int32_t *__restrict__ aci = gp(P.aci);
    const MLS_G double *__restrict__ aval = gp(P.aval);
    const MLS_G int32_t *__restrict__ brp = gp(P.brp);
    const MLS_G int32_t *__restrict__ bci = gp(P.bci);
    const MLS_G double *__restrict__ bval = gp(P.bval);
    const MLS_G int32_t *__restrict__ wci = gp(P.cci);
    const MLS_G double *__restrict__ wval = gp(P.cval);
    MLS_G double *__restrict__ gdA = gpw(dA);
    const int n_bin = gp(sc.bin_count)[bin];
    const int start = bin_start(sc.bin_count, bin);
    const int ntasks = (n_bin + W - 1) / W;
    TaskIter it = task_iter<MAXLDS != 65536>(ntasks, NW, -1, vblk, vgrid);
    // Three rows of a slot are in flight: the row after next has its perm
    // entry loading, the next row its metadata, then its first chunk (entries
    // of A_i while this row's W_i is hashed, their B row bounds after this
    // row's pairs), so a row starts with its dependent index loads done.
    int task = next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it);
    const bool h_cur = task >= 0 && task * W + slot < n_bin;
    const int g_raw = bin_row_issue(sc.perm, sc.err, b.na, start + task * W + slot, h_cur);
    int task_n = task >= 0 ? next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it) : -1;
    bool h_n = task_n >= 0 && task_n * W + slot < n_bin;
    int g_n = bin_row_issue(sc.perm, sc.err, b.na, start + task_n * W + slot, h_n);
    BwdMeta m = bwd_meta_issue(P, sc, bin_row_checked(sc.err, b.na, g_raw, h_cur));
    BwdFirst f;
    bwd_first_a(P, m, lane, f);
    bwd_first_b(P, f);
    // no prologue load is left pending into the loop (the wait counts at its
    // top are computed over both ways into it)
    asm volatile("" ::"v"(f.q0), "v"(f.q1), "v"(f.sa), "v"(g_n), "v"(m.nw), "v"(m.ws0), "v"(m.ps), "v"(m.pe));
    while (task >= 0) {
        const int task_x = task_n >= 0 ? next_task_wave(sc.task_cursor + bin * kXcd, ntasks, it) : -1;
        const bool h_x = task_x >= 0 && task_x * W + slot < n_bin;
        const int g_x = bin_row_issue(sc.perm, sc.err, b.na, start + task_x * W + slot, h_x);
        const BwdMeta mn = bwd_meta_issue(P, sc, bin_row_checked(sc.err, b.na, g_n, h_n));
        const int nw = m.nw, ws0 = m.ws0, ps = m.ps, pe = m.pe;
        int logcap = ilog2_ceil(2 * nw);
        if (logcap < 5) logcap = 5;
        if constexpr (PACK) {
            ptab.open(nw, lane, G);
        } else {
            for (int h = lane; h < 1 << logcap; h += G) key[h] = -1;
        }
        // this row's first chunk was located during the previous row
        int ka = f.ka;
        double sa = f.sa;
        int fq0 = f.q0, fq1 = f.q1;
        bwd_sync();
        for (int e0 = lane; e0 < nw; e0 += G * kBwdInsDepth) {
            int jv[kBwdInsDepth];
            double wj[kBwdInsDepth];
#pragma unroll
            for (int u = 0; u < kBwdInsDepth; ++u) {
                const int e = e0 + u * G;
                jv[u] = -1;
                wj[u] = 0.0;
                if (e < nw) { jv[u] = wci[ws0 + e]; wj[u] = wval[ws0 + e]; }
            }
#pragma unroll
            for (int u = 0; u < kBwdInsDepth; ++u) {
                if (jv[u] < 0) continue;
                if constexpr (PACK) {
                    ptab.insert(jv[u], e0 + u * G);
                    wv[e0 + u * G] = wj[u];
                } else {
                    w_insert(key, wv, logcap, jv[u], wj[u]);
                }
            }
        }
        bwd_sync();
        bool bad = false;
        // the chunk loop runs to the wave's longest row, so that the group
        // scans (cross-lane shuffles) run with every lane present
        int nch = (pe - ps + G - 1) / G;
        for (int o = 32; o >= 1; o >>= 1) nch = max(nch, __shfl_xor(nch, o, kWave));
        // stage a chunk: its non-empty entries compacted (first B position - first
        // pair, a_ik and zeroed dA sums); returns the chunk's pair count
        int first = 0, rank = 0;   // this lane's entry: its first pair, its place
        bool any = false;
        auto stage = [&](int q0, int q1, double a) -> int {
            const int np = q1 > q0 ? q1 - q0 : 0;
            const int incl = group_scan_incl<G>(np, lane);
            const int tot = group_total<G>(np, incl);
            first = incl - np;
            any = np > 0;
            const unsigned long long ne = __ballot(any) >> (slot * G);
            rank = __popcll(ne & ((1ull << lane) - 1ull));
            if (any) {
                pq[rank] = q0 - first;
                pa[rank] = a;
            }
            da[lane] = 0.0;
            return tot;
        };
        // the first chunk from what was located during the previous row, the
        // later ones in the loop: no loaded value reaches a point where two
        // ways join (its wait there would cover every load issued since)
        int total = stage(fq0, fq1, sa);
        // the next row's first entries of A load during this row's pairs
        bwd_first_a(P, mn, lane, f);
        for (int c = 0; c < nch; ++c) {
            const int pc = ps + c * G;
            if (c > 0) {
                const MLS_G int32_t *pb = pc + lane < pe ? brp + ka : (const MLS_G int32_t *)k_zeros4;
                total = stage(pb[0], pb[1], sa);
            }
            // the next chunk's entries of A are in flight during this chunk's
            // pairs (no branch: see the numeric kernel's chunk loop)
            {
                const bool on = pc + G + lane < pe;
                ka = *(on ? aci + pc + G + lane : (const MLS_G int32_t *)k_ones4);
                sa = *(on ? aval + pc + G + lane : (const MLS_G double *)k_zeros4);
            }
            bwd_sync();
            // the dB adds of a batch are issued after the next batch's loads:
            // the wait for those loads then does not include them (the
            // counter covers loads and atomics in issue order)
            int dq[kBwdUnroll];
            double dv[kBwdUnroll];
#pragma unroll
            for (int d = 0; d < kBwdUnroll; ++d) { dq[d] = -1; dv[d] = 0.0; }
            int eb = -1;   // entries started before the tile, less one
            for (int base = 0; base < total; base += G * kBwdUnroll) {
                // a bit per pair of the tile where an entry starts: a pair's entry is
                // the count of the bits up to it (from DPP ORs for groups of up to 16
                // lanes, through LDS for wider ones)
                constexpr int NB = G * kBwdUnroll / 32;   // words of bits
                uint32_t m[NB];
                const int at0 = first - base;
                if constexpr (G <= 16) {
#pragma unroll
                    for (int x = 0; x < NB; ++x) {
                        const int at = at0 - 32 * x;
                        m[x] = group_or8(any && (uint32_t)at < 32u ? 1u << at : 0u);
                        if constexpr (G == 16) m[x] |= (uint32_t)dpp_move<0x140>((int)m[x]);   // the other half of 16
                    }
                } else {
                    if (lane < NB) flags[lane] = 0u;
                    bwd_sync();
                    if (any && (uint32_t)at0 < 32u * NB) atomicOr(flags + (at0 >> 5), 1u << (at0 & 31));
                    bwd_sync();
#pragma unroll
                    for (int x = 0; x < NB; x += 4) {
                        const uint4 v = *(const uint4 *)(flags + x);
                        m[x] = v.x; m[x + 1] = v.y; m[x + 2] = v.z; m[x + 3] = v.w;
                    }
                    bwd_sync();
                }
                int qv[kBwdUnroll], ev[kBwdUnroll], jv[kBwdUnroll];
                bool ok[kBwdUnroll];
                double bv[kBwdUnroll];
                // loads without branches (past the pairs, the last one again), all
                // issued before any use
#pragma unroll
                for (int d = 0; d < kBwdUnroll; ++d) {
                    const int pp = base + d * G + lane;
                    int en;
                    if constexpr (G == 64) {
                        const uint64_t mm = ((uint64_t)m[2 * d + 1] << 32) | m[2 * d];
                        en = eb + __popcll(mm & (lane == 63 ? ~0ull : (2ull << lane) - 1ull));
                        eb += __popcll(mm);
                    } else {
                        const int sh = d * G % 32;
                        const uint32_t w = m[d * G / 32];
                        en = eb + __popc(w & ((2u << (sh + lane)) - 1u));
                        if (sh + G == 32) eb += __popc(w);
                    }
                    ok[d] = pp < total;
                    ev[d] = en;
                    qv[d] = pq[en] + or_last(ok[d], pp, total - 1);
                    jv[d] = bci[(uint32_t)qv[d]];
                    bv[d] = bval[(uint32_t)qv[d]];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int d = 0; d < kBwdUnroll; ++d)
                    if (dq[d] >= 0) atomicAdd(dB + dq[d], dv[d]);
                bool hit[kBwdUnroll];
                double w[kBwdUnroll];
                if constexpr (PACK) {
                    // positions in W_i's row, then the values by position
                    uint32_t pos[kBwdUnroll];
                    ptab.template lookup_n<kBwdUnroll>(jv, ok, pos);
#pragma unroll
                    for (int d = 0; d < kBwdUnroll; ++d) {
                        hit[d] = ok[d] && pos[d] <= ptab.kMaxPos;
                        w[d] = wv[hit[d] ? pos[d] : 0u];
                    }
                } else {
                    int sl[kBwdUnroll];
#pragma unroll
                    for (int d = 0; d < kBwdUnroll; ++d) jv[d] = ok[d] ? jv[d] : -1;
                    w_lookup_n<kBwdUnroll>(key, wv, logcap, jv, sl, w);
#pragma unroll
                    for (int d = 0; d < kBwdUnroll; ++d) hit[d] = sl[d] >= 0;
                }
#pragma unroll
                for (int d = 0; d < kBwdUnroll; ++d) asm volatile("" ::"v"(bv[d]));
#pragma unroll
                for (int d = 0; d < kBwdUnroll; ++d) {
                    bad |= ok[d] && !hit[d];
                    dq[d] = -1;
                    if (!hit[d]) continue;
                    if (dA) atomicAdd(da + ev[d], w[d] * bv[d]);
                    if (dB) { dq[d] = qv[d]; dv[d] = pa[ev[d]] * w[d]; }
                }
            }
#pragma unroll
            for (int d = 0; d < kBwdUnroll; ++d)
                if (dq[d] >= 0) atomicAdd(dB + dq[d], dv[d]);
            bwd_sync();
            if (dA && pc + lane < pe) gdA[pc + lane] = any ? da[rank] : 0.0;
            bwd_sync();
        }
        // the next row's B row bounds (its entries of A arrived during the pairs)
        bwd_first_b(P, f);
        if (bad) atomicOr(sc.err, kErrStructure);
        bwd_sync();
        task = task_n;
        task_n = task_x;
        g_n = g_x;
        h_n = h_x;
        m = mn;
    }
}

template <int G, int CAP, bool PACK>
__global__ __launch_bounds__(kWG) void k_bwd_lds(Batch b, Sched sc, int bin, double *dA, double *dB)
{
    __shared__ __attribute__((aligned(16))) char s_mem[BwdShape<G, CAP, PACK>::LDS];
    bwd_lds_rows<G, CAP, PACK, 65536>(b, sc, bin, dA, dB, s_mem, (int)blockIdx.x, (int)gridDim.x);
}

__device__ __forceinline__ int bsearch_w(const MLS_G int32_t *cols, int n, int j)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (cols[mid] < j) lo = mid + 1; else hi = mid;
    }
    return (lo < n && cols[lo] == j) ? lo : -1;
}

// first position in cols[lo, hi) whose column is >= j
__device__ __forceinline__ int lower_col_w(const MLS_G int32_t *cols, int lo, int hi, int j)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (cols[mid] < j) lo = mid + 1; else hi = mid;
    }
    return lo;
}

constexpr int kBwdWinCap = 1024;   // table slots of a spill window (CAP / 2 positions of W_i)
constexpr int kBwdWinDepth = 2;    // batches of 64 pairs whose B loads are issued together

// LDS of one spill window: hash keys and W values, staged entries, their
// first pair, and the entries' dA parts
constexpr int bwd_win_bytes(int CAP) { return CAP * 12 + kWave * 16 + (kWave + 1) * 4 + kWave * 8; }

// Tasks of the spill rows come from k_win_scan, one window (of M positions of
// W_i) each.
// A window's (entry, B position) pairs are flattened, 64 per step: each pair
// adds a_ik W_ij into dB with a device atomic and W_ij b_kj into its entry's
// dA part in LDS; the parts go to dA with one device atomic per entry.
template <int CAP, int MAXLDS = 65536>
struct BwdWinShape {
    static constexpr int NW = nw_bwd(bwd_win_bytes(CAP), 1, MAXLDS);
    static constexpr int LDS_WV = NW * CAP * 4;
    static constexpr int LDS_PAR = LDS_WV + NW * CAP * 8;
    static constexpr int LDS_DA = LDS_PAR + NW * kWave * 16;
    static constexpr int LDS_POFF = LDS_DA + NW * kWave * 8;
    static constexpr int LDS = LDS_POFF + NW * (kWave + 1) * 4;
};

// lds: BwdWinShape::LDS bytes of this workgroup
template <int CAP, int MAXLDS>
__device__ __forceinline__ void bwd_win_rows(const Batch &b, const Sched &sc, double *dA, double *dB, char *lds)
{
    using Shape = BwdWinShape<CAP, MAXLDS>;
    constexpr int G = kWave;
    constexpr int M = CAP / 2;
    constexpr int NW = Shape::NW;
    int *s_key = (int *)lds;
    double *s_wv = (double *)(lds + Shape::LDS_WV);
    int4 *s_par = (int4 *)(lds + Shape::LDS_PAR);    // staged entries: (first B position, -, a)
    double *s_da = (double *)(lds + Shape::LDS_DA);
    int *s_poff = (int *)(lds + Shape::LDS_POFF);    // first pair of each staged entry, then the total

    const int wave = threadIdx.x >> 6;
    if (wave >= NW) return;
    const int lane = threadIdx.x & 63;
    int *key = s_key + wave * CAP;
    double *wv = s_wv + wave * CAP;
    int4 *par = s_par + wave * G;
    int *poff = s_poff + wave * (G + 1);
    double *da = s_da + wave * G;

    const Prob P = b.p0;
    const MLS_G int32_t *__restrict__ arp = gp(P.arp);
    const MLS_G int32_t *__restrict__ aci = gp(P.aci);
    const MLS_G double *__restrict__ aval = gp(P.aval);
    const MLS_G int32_t *__restrict__ brp = gp(P.brp);
    const MLS_G int32_t *__restrict__ bci = gp(P.bci);
    const MLS_G double *__restrict__ bval = gp(P.bval);
    const MLS_G int32_t *__restrict__ wrp = gp(P.crp);
    const MLS_G int32_t *__restrict__ wci = gp(P.cci);
    const MLS_G double *__restrict__ wval = gp(P.cval);
    const int n_bin = gp(sc.bin_count)[kBinSpill];
    const int start = bin_start(sc.bin_count, kBinSpill);
    const MLS_G int32_t *wst = gp(sc.wstart);
    const int nwin = n_bin > 0 ? wst[n_bin] : 0;
    // one counter over all windows: their work varies too much (a hub row's
    // windows are consecutive and long) for per-XCD slabs
    if (nwin == 0) return;
    int32_t *cursor = sc.task_cursor + kBinSpill * kXcd;
    for (;;) {
        int u = 0;
        if (lane == 0) u = atomicAdd(cursor, 1);
        u = __builtin_amdgcn_readlane(u, 0);
        if (u >= nwin) break;
        const int r = find_last_wave(wst, n_bin, u);   // the row holding window u
        const int i = bin_row(sc.perm, sc.err, b.na, start + r);
        if (i < 0) continue;
        const int nw = gp(sc.val)[i];
        const int c0 = (u - wst[r]) * M;
        const int ws0 = wrp[i] + c0;
        const int n = min(M, nw - c0);
        const bool narrow = nw > M;
        // open below for the row's first window and above for its last, so
        // that a column outside the whole row still fails the lookup
        const int jlo = c0 == 0 ? INT_MIN : wci[ws0];
        const int jhi = c0 + n == nw ? INT_MAX : wci[ws0 + n - 1];
        int logcap = ilog2_ceil(2 * n);
        if (logcap < 5) logcap = 5;
        const int cap = 1 << logcap;
        for (int h = lane; h < cap; h += G) key[h] = -1;
        bwd_sync();
        for (int e0 = lane; e0 < n; e0 += G * kBwdInsDepth) {
            int jv[kBwdInsDepth];
            double wj[kBwdInsDepth];
#pragma unroll
            for (int u = 0; u < kBwdInsDepth; ++u) {
                const int e = e0 + u * G;
                jv[u] = -1;
                wj[u] = 0.0;
                if (e < n) { jv[u] = wci[ws0 + e]; wj[u] = wval[ws0 + e]; }
            }
#pragma unroll
            for (int u = 0; u < kBwdInsDepth; ++u)
                if (jv[u] >= 0) w_insert(key, wv, logcap, jv[u], wj[u]);
        }
        bwd_sync();
        bool bad = false;
        const int ps = arp[i], pe = arp[i + 1];
        for (int pc = ps; pc < pe; pc += G) {
            int sq0 = 0, sq1 = 0;
            double sa = 0.0;
            if (pc + lane < pe) {
                const int k = aci[pc + lane];
                sa = aval[pc + lane];
                sq0 = brp[k];
                sq1 = brp[k + 1];
                if (narrow && sq1 - sq0 > 32) {
                    if (jlo != INT_MIN) sq0 = lower_col_w(bci, sq0, sq1, jlo);
                    if (jhi != INT_MAX) sq1 = lower_col_w(bci, sq0, sq1, jhi + 1);
                }
            }
            const int np = sq1 > sq0 ? sq1 - sq0 : 0;
            int incl = group_scan_incl<G>(np, lane);
            const int total = group_total<G>(np, incl);
            poff[lane] = incl - np;
            if (lane == 0) poff[G] = total;
            par[lane] = make_int4(sq0, 0, __double2loint(sa), __double2hiint(sa));
            da[lane] = 0.0;
            bwd_sync();
            for (int base = 0; base < total; base += G * kBwdWinDepth) {
                int ev[kBwdWinDepth], qv[kBwdWinDepth], jv[kBwdWinDepth];
                double bv[kBwdWinDepth], av[kBwdWinDepth];
#pragma unroll
                for (int d = 0; d < kBwdWinDepth; ++d) {
                    jv[d] = -1; ev[d] = 0; qv[d] = 0; bv[d] = 0.0; av[d] = 0.0;
                    const int pp = base + d * G + lane;
                    if (pp < total) {
                        int lo = 0, hi = G - 1;   // largest e with poff[e] <= pp
                        while (lo < hi) {
                            const int mid = (lo + hi + 1) >> 1;
                            if (poff[mid] <= pp) lo = mid; else hi = mid - 1;
                        }
                        const int4 pr = par[lo];
                        ev[d] = lo;
                        qv[d] = pr.x + (pp - poff[lo]);
                        av[d] = __hiloint2double(pr.w, pr.z);
                        jv[d] = bci[qv[d]];
                        bv[d] = bval[qv[d]];
                    }
                }
                int jw[kBwdWinDepth], sl[kBwdWinDepth];
                double w[kBwdWinDepth];
#pragma unroll
                for (int d = 0; d < kBwdWinDepth; ++d) jw[d] = (jv[d] >= jlo && jv[d] <= jhi) ? jv[d] : -1;
                w_lookup_n<kBwdWinDepth>(key, wv, logcap, jw, sl, w);
#pragma unroll
                for (int d = 0; d < kBwdWinDepth; ++d) {
                    if (sl[d] == -1) bad = true;
                    if (sl[d] < 0) continue;
                    if (dA) atomicAdd(da + ev[d], w[d] * bv[d]);
                    if (dB) atomicAdd(dB + qv[d], av[d] * w[d]);
                }
            }
            bwd_sync();
            if (dA && pc + lane < pe && da[lane] != 0.0) atomicAdd(dA + pc + lane, da[lane]);
            bwd_sync();
        }
        if (bad) atomicOr(sc.err, kErrStructure);
    }
}

template <int CAP>
__global__ __launch_bounds__(kWG) void k_bwd_win(Batch b, Sched sc, double *dA, double *dB)
{
    __shared__ __attribute__((aligned(16))) char s_mem[BwdWinShape<CAP>::LDS];
    bwd_win_rows<CAP, 65536>(b, sc, dA, dB, s_mem);
}

// Products of few rows: every class and the spill windows in one launch, the
// rows of the largest class as windows (as the numeric phase's k_num_all, with
// the same saving: 5000 random rows of 36 outputs 52 -> 23 us).
constexpr int kBwdAllLds = 24576;

using BwdAll0 = BwdShape<8, kFillCap[0], true, kBwdAllLds>;
using BwdAll1 = BwdShape<32, kFillCap[1], true, kBwdAllLds>;
using BwdAll2 = BwdShape<64, kFillCap[2], true, kBwdAllLds>;
using BwdAll3 = BwdShape<64, kFillCap[3], true, kBwdAllLds>;
using BwdAllW = BwdWinShape<kBwdWinCap, kBwdAllLds>;
static_assert(BwdAll0::LDS <= kBwdAllLds && BwdAll1::LDS <= kBwdAllLds && BwdAll2::LDS <= kBwdAllLds &&
              BwdAll3::LDS <= kBwdAllLds && BwdAllW::LDS <= kBwdAllLds, "one LDS buffer for every part");

__global__ __launch_bounds__(kWG) void k_bwd_all(Batch b, Sched sc, double *dA, double *dB)
{
    __shared__ __attribute__((aligned(16))) char s_mem[kBwdAllLds];
    const int per[kNumClasses + 1] = {BwdAll0::W * BwdAll0::NW, BwdAll1::W * BwdAll1::NW, BwdAll2::NW, BwdAll3::NW,
                                      1, BwdAllW::NW};
    int vblk, vgrid;
    switch (part_of_block(sc, per, vblk, vgrid)) {
    case 0: bwd_lds_rows<8, kFillCap[0], true, kBwdAllLds>(b, sc, 0, dA, dB, s_mem, vblk, vgrid); break;
    case 1: bwd_lds_rows<32, kFillCap[1], true, kBwdAllLds>(b, sc, 1, dA, dB, s_mem, vblk, vgrid); break;
    case 2: bwd_lds_rows<64, kFillCap[2], true, kBwdAllLds>(b, sc, 2, dA, dB, s_mem, vblk, vgrid); break;
    case 3: bwd_lds_rows<64, kFillCap[3], true, kBwdAllLds>(b, sc, 3, dA, dB, s_mem, vblk, vgrid); break;
    case kNumClasses: bwd_win_rows<kBwdWinCap, kBwdAllLds>(b, sc, dA, dB, s_mem); break;
    }
}

// As num_small_fit; the adjoint's windows hold one wave per workgroup there. By
// class / two launches in us: 20000 x 100 (17 x 6) 75 / 66; 4000 x 250 (12 x 20) 50 /
// 46, 10000 x 250 74 / 86, 1000 x 900 (45 x 20) 60 / 38, 4000 x 900 93 / 101, 250 x 1500
// (15 x 100) 61 / 52, 1000 x 1500 70 / 109; 1000 x 2500 (25 x 100) 160 / 137, 4000 x 2500
// 363 / 411, 64 x 20000 (200 x 100) 155 / 114, 250 x 20000 295 / 315.
bool bwd_small_fit(const Batch &b, int64_t outputs)
{
    if (!small_rows_fit(b)) return false;
    const int64_t mean = outputs / b.na;
    return outputs <= (mean <= 128 ? 1ll << 21 : (mean <= 2048 ? 1ll << 20 : 1ll << 22));
}

void launch_backward_small(const Batch &b, const Sched &sc, double *dA, double *dB, int64_t outputs, hipStream_t s)
{
    launch_bin_small(b, sc, kBwdWinCap / 2, 0, s);
    ProfScope ps("bwd_all", s);
    hipLaunchKernelGGL(k_bwd_all, dim3(small_rows_grid(b.na, 2 * outputs)), dim3(kWG), 0, s, b, sc, dA, dB);
}

template <typename K>
static int bwd_grid(K kernel, int threads)
{
    static int cus = device_cu_count();
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return cus * per_cu;
}

template <int G, int CAP, bool PACK>
static void launch_bwd_variant(const Batch &b, const Sched &sc, int bin, double *dA, double *dB, hipStream_t s)
{
    constexpr int NW = BwdShape<G, CAP, PACK>::NW;
    static int grid = bwd_grid(k_bwd_lds<G, CAP, PACK>, NW * kWave);
    static char name[64];
    if (!name[0]) snprintf(name, sizeof(name), "bwd_lds_G%d_C%d%s", G, CAP, PACK ? "_p" : "");
    ProfScope ps(name, s);
    hipLaunchKernelGGL((k_bwd_lds<G, CAP, PACK>), dim3(grid), dim3(NW * kWave), 0, s, b, sc, bin, dA, dB);
}

// The packed table needs every column index of W below PackBits<CAP>::kMaxCols.
template <int G, int CAP>
static void launch_bwd_class(const Batch &b, const Sched &sc, int bin, double *dA, double *dB, hipStream_t s)
{
    if (b.max_ncols > 0 && (uint32_t)b.max_ncols <= PackBits<CAP>::kMaxCols)
        launch_bwd_variant<G, CAP, true>(b, sc, bin, dA, dB, s);
    else
        launch_bwd_variant<G, CAP, false>(b, sc, bin, dA, dB, s);
}

void launch_backward(const Batch &b, const Sched &sc, const double *wval, double *dA, double *dB, int G,
                     hipStream_t s)
{
    (void)wval;
    if (b.na <= 0) return;
    launch_bwd_class<8, kFillCap[0]>(b, sc, 0, dA, dB, s);
    switch (G) {
    case 8: launch_bwd_class<8, kFillCap[1]>(b, sc, 1, dA, dB, s); break;
    case 16: launch_bwd_class<16, kFillCap[1]>(b, sc, 1, dA, dB, s); break;
    case 64: launch_bwd_class<64, kFillCap[1]>(b, sc, 1, dA, dB, s); break;
    default: launch_bwd_class<32, kFillCap[1]>(b, sc, 1, dA, dB, s); break;
    }
    // the pairs are flattened, so lanes are filled whatever the rows of B: from
    // the 1024-slot class on, a whole wave per row (one row's LDS per wave)
    // keeps the most waves resident (300000 rows of about 160 outputs: 32
    // lanes 1250-1365 us, 64 lanes 841-911 us)
    launch_bwd_class<64, kFillCap[2]>(b, sc, 2, dA, dB, s);
    launch_bwd_class<64, kFillCap[3]>(b, sc, 3, dA, dB, s);
    launch_bwd_class<64, kFillCap[4]>(b, sc, 4, dA, dB, s);
    constexpr int NWW = BwdWinShape<kBwdWinCap>::NW;
    static int win_grid = bwd_grid(k_bwd_win<kBwdWinCap>, NWW * kWave);
    ProfScope ps("bwd_spill", s);
    hipLaunchKernelGGL(k_win_scan, dim3(1), dim3(kWinScanWG), 0, s, b, sc, kBwdWinCap / 2, 0);
    hipLaunchKernelGGL(k_bwd_win<kBwdWinCap>, dim3(win_grid), dim3(NWW * kWave), 0, s, b, sc, dA, dB);
}

// ---------------------------------------------------------------------------
// Deterministic adjoint: every entry of dA and of dB is the sequential sum of
// one lane, in the order of the row-wise formulation -- dA_ik over the columns
// j of B_k in ascending order, dB_kj over the rows i of column k of A in
// ascending order (read from the transpose of A) -- with each product rounded
// before it is added. The result does not depend on scheduling, so repeated
// calls agree bit for bit. W_ij is found by binary search in W_i's ascending
// columns (no LDS table, no atomics on the outputs); a triple whose column j
// is missing from W_i sets the structure error.

// G lanes own a row of A (of B): rows of W of up to kDetStage * G columns are
// staged in LDS and searched there, longer ones in place. Bound by latency:
// what a lane searches is a handful of columns, in rows of W that arrive in one
// coalesced pass each. (Searching every column in global memory made 6 to 8
// dependent gathers per term: 200003 rows, Poisson(8), dA 612 and dB 411 us;
// so 253 and 283 us, near what the lines of B and W that the gathers touch take
// from the last-level cache: about 0.6 and 1.4 GB.)
constexpr int kDetStage = 16;   // columns of W_i per lane
constexpr int kDetAhead = 4;    // terms of a lane searched together

// Four entries from p on, p >= end giving none that is used: one wide load
// (element-aligned) where four more entries of the array follow, else one at a
// time. end: entries of the whole array.
typedef int i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x4u __attribute__((ext_vector_type(4), aligned(8)));

__device__ __forceinline__ void load4(const MLS_G int32_t *a, int64_t p, int64_t end, int (&v)[4])
{
    if (p + 4 <= end) {
        const i32x4u w = *(const MLS_G i32x4u *)(a + p);
        v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p + u < end ? a[p + u] : 0;
    }
}

__device__ __forceinline__ void load4(const MLS_G double *a, int64_t p, int64_t end, double (&v)[4])
{
    if (p + 4 <= end) {
        const f64x4u w = *(const MLS_G f64x4u *)(a + p);
        v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p + u < end ? a[p + u] : 0.0;
    }
}

// first position in the n ascending columns c (in LDS) whose column is >= j,
// for D columns at once; top: the largest power of two <= n
template <int D>
__device__ __forceinline__ void det_lower(const int *c, int n, int top, const int (&j)[D], int (&at)[D])
{
#pragma unroll
    for (int d = 0; d < D; ++d) at[d] = 0;
    for (int step = top; step > 0; step >>= 1) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int x = at[d] + step;
            if (x <= n && c[x - 1] < j[d]) at[d] = x;
        }
    }
}

__device__ __forceinline__ int det_top(int n) { return n > 0 ? 1 << (31 - __clz(n)) : 0; }

template <int G>
__global__ __launch_bounds__(kWG) void k_bwd_det_da(int32_t m, int64_t nnz_b, int64_t nnz_w, const int32_t *arp, const int32_t *aci,
                                                    const int32_t *brp, const int32_t *bci, const double *bval,
                                                    const int32_t *wrp, const int32_t *wci, const double *wval,
                                                    double *dA, uint32_t *err)
{
    constexpr int CAP = kDetStage * G;
    __shared__ __attribute__((aligned(16))) int s_c[kWG / G][CAP];
    const int grp = threadIdx.x / G, l = threadIdx.x % G;
    const int64_t i = (int64_t)blockIdx.x * (kWG / G) + grp;
    const bool row = i < m;
    const int ws = row ? gp(wrp)[i] : 0, wn = row ? gp(wrp)[i + 1] - ws : 0;
    const MLS_G int32_t *wc = gp(wci) + ws;
    const MLS_G double *wv = gp(wval) + ws;
    int *c = s_c[grp];
    const bool staged = wn <= CAP;
    if (staged) {
        for (int x = 4 * l; x < wn; x += 4 * G) {
            int w[4];
            load4(gp(wci), (int64_t)ws + x, nnz_w, w);
            *(int4 *)(c + x) = make_int4(w[0], w[1], w[2], w[3]);
        }
    }
    bwd_sync();
    if (!row) return;
    const int top = det_top(wn);
    bool bad = false;
    // (unsigned positions: the last step may end past the largest int)
    const uint32_t pe = (uint32_t)gp(arp)[i + 1];
    for (uint32_t p = (uint32_t)(gp(arp)[i] + l); p < pe; p += G) {
        const int k = gp(aci)[p];
        const uint32_t qs = (uint32_t)gp(brp)[k], qe = (uint32_t)gp(brp)[k + 1];
        double sum = 0.0;
        if (staged) {
            for (uint32_t q = qs; q < qe; q += kDetAhead) {
                int j[kDetAhead], at[kDetAhead];
                double bv[kDetAhead];
                load4(gp(bci), q, nnz_b, j);
                load4(gp(bval), q, nnz_b, bv);
                det_lower<kDetAhead>(c, wn, top, j, at);
                double w[kDetAhead];
                bool hit[kDetAhead];
#pragma unroll
                for (int u = 0; u < kDetAhead; ++u) {
                    hit[u] = q + u < qe && at[u] < wn && c[at[u]] == j[u];
                    bad |= q + u < qe && !hit[u];
                    w[u] = *(hit[u] ? wv + at[u] : (const MLS_G double *)k_zeros4);
                }
#pragma unroll
                for (int u = 0; u < kDetAhead; ++u)   // terms in ascending j
                    if (hit[u]) sum += w[u] * bv[u];
            }
        } else {
            int lo = 0;   // the columns of B_k ascend, so each search starts past the last hit
            for (uint32_t q = qs; q < qe; ++q) {
                const int j = gp(bci)[q];
                lo = lower_col_w(wc, lo, wn, j);
                if (lo >= wn || wc[lo] != j) { bad = true; break; }
                sum += wv[lo] * gp(bval)[q];
            }
        }
        gpw(dA)[p] = sum;
    }
    if (bad) atomicOr(err, kErrStructure);
}

// A lane holds kDetOwn entries of B_k (one per G), and the group walks the rows
// i of column k of A in ascending order; the next row of W loads while the
// current one is searched.
constexpr int kDetOwn = 2;

template <int G>
__global__ __launch_bounds__(kWG) void k_bwd_det_db(int32_t kb, int64_t nnz_w, const int32_t *trp, const int32_t *tci,
                                                    const double *tv, const int32_t *brp, const int32_t *bci,
                                                    const int32_t *wrp, const int32_t *wci, const double *wval,
                                                    double *dB, uint32_t *err)
{
    constexpr int CAP = kDetStage * G;
    constexpr int NV = kDetStage / 4;   // wide loads of a row of W per lane
    __shared__ __attribute__((aligned(16))) int s_c[kWG / G][CAP];
    const int grp = threadIdx.x / G, l = threadIdx.x % G;
    const int64_t k = (int64_t)blockIdx.x * (kWG / G) + grp;
    if (k >= kb) return;   // whole groups: a group exchanges with itself alone
    int *c = s_c[grp];
    // (unsigned positions: the last step may end past the largest int)
    const uint32_t rs = (uint32_t)gp(trp)[k], re = (uint32_t)gp(trp)[k + 1];
    const uint32_t qs = (uint32_t)gp(brp)[k], qe = (uint32_t)gp(brp)[k + 1];
    bool bad = false;
    for (uint32_t q0 = qs; q0 < qe; q0 += G * kDetOwn) {
        int j[kDetOwn];
        double sum[kDetOwn];
#pragma unroll
        for (int u = 0; u < kDetOwn; ++u) {
            const uint32_t q = q0 + (uint32_t)(u * G + l);
            j[u] = q < qe ? gp(bci)[q] : -1;
            sum[u] = 0.0;
        }
        // the term found last: added once the next row's loads are queued
        double pa = 0.0, pw[kDetOwn];
        bool ph[kDetOwn];
#pragma unroll
        for (int u = 0; u < kDetOwn; ++u) { pw[u] = 0.0; ph[u] = false; }
        for (uint32_t rb = rs; rb < re; rb += G) {   // rows i of column k of A, ascending, G located together
            const bool in = rb + l < re;
            const int i = in ? gp(tci)[rb + l] : 0;
            const double al = in ? gp(tv)[rb + l] : 0.0;
            const int wsl = gp(wrp)[i], wnl = in ? gp(wrp)[i + 1] - wsl : 0;
            const int nr = (int)min((uint32_t)G, re - rb);
            int w[NV][4];
            int w0 = __shfl(wsl, 0, G), n = __shfl(wnl, 0, G);
            auto next_row = [&]() {   // the row's columns x, 4 at a time, lane by lane
#pragma unroll
                for (int x = 0; x < NV; ++x)
                    if (4 * (x * G + l) < n) load4(gp(wci), (int64_t)w0 + 4 * (x * G + l), nnz_w, w[x]);
            };
            next_row();
            for (int y = 0; y < nr; ++y) {
                const double a = __shfl(al, y, G);
                const int cw0 = w0, cn = n;
#pragma unroll
                for (int x = 0; x < NV; ++x)
                    if (4 * (x * G + l) < cn)
                        *(int4 *)(c + 4 * (x * G + l)) = make_int4(w[x][0], w[x][1], w[x][2], w[x][3]);
                bwd_sync();
                w0 = __shfl(wsl, y + 1 < nr ? y + 1 : 0, G);
                n = y + 1 < nr ? __shfl(wnl, y + 1 < nr ? y + 1 : 0, G) : 0;
                next_row();
                int at[kDetOwn];
                if (cn <= CAP) {
                    det_lower<kDetOwn>(c, cn, det_top(cn), j, at);
                } else {
#pragma unroll
                    for (int u = 0; u < kDetOwn; ++u) at[u] = lower_col_w(gp(wci) + cw0, 0, cn, j[u]);
                }
                double v[kDetOwn];
                bool hit[kDetOwn];
#pragma unroll
                for (int u = 0; u < kDetOwn; ++u) {
                    hit[u] = j[u] >= 0 && at[u] < cn && (cn <= CAP ? c[at[u] < CAP ? at[u] : 0] : gp(wci)[cw0 + at[u]]) == j[u];
                    bad |= j[u] >= 0 && !hit[u];
                    v[u] = *(hit[u] ? gp(wval) + cw0 + at[u] : (const MLS_G double *)k_zeros4);
                }
#pragma unroll
                for (int u = 0; u < kDetOwn; ++u) {
                    if (ph[u]) sum[u] += pa * pw[u];
                    ph[u] = hit[u];
                    pw[u] = v[u];
                }
                pa = a;
                bwd_sync();
            }
        }
#pragma unroll
        for (int u = 0; u < kDetOwn; ++u)
            if (ph[u]) sum[u] += pa * pw[u];
#pragma unroll
        for (int u = 0; u < kDetOwn; ++u) {
            const uint32_t q = q0 + (uint32_t)(u * G + l);
            if (q < qe) gpw(dB)[q] = sum[u];
        }
    }
    if (bad) atomicOr(err, kErrStructure);
}

template <int G>
static void launch_det_group(int32_t m, int32_t kb, int64_t nnz_b, int64_t nnz_w, const int32_t *arp, const int32_t *aci, const int32_t *brp,
                             const int32_t *bci, const double *bval, const int32_t *wrp, const int32_t *wci,
                             const double *wval, const int32_t *trp, const int32_t *tci, const double *tv, double *dA,
                             double *dB, uint32_t *err, hipStream_t s)
{
    constexpr int rows = kWG / G;
    if (dA && m > 0) {
        ProfScope ps("bwd_det_dA", s);
        hipLaunchKernelGGL(k_bwd_det_da<G>, dim3((unsigned)((m + rows - 1) / rows)), dim3(kWG), 0, s, m, nnz_b, nnz_w, arp,
                           aci, brp, bci, bval, wrp, wci, wval, dA, err);
    }
    if (dB && kb > 0) {
        ProfScope ps("bwd_det_dB", s);
        hipLaunchKernelGGL(k_bwd_det_db<G>, dim3((unsigned)((kb + rows - 1) / rows)), dim3(kWG), 0, s, kb, nnz_w, trp,
                           tci, tv, brp, bci, wrp, wci, wval, dB, err);
    }
}

void launch_backward_det(int32_t m, int32_t kb, int64_t nnz_b, int64_t nnz_w, const int32_t *arp, const int32_t *aci,
                         const int32_t *brp, const int32_t *bci, const double *bval, const int32_t *wrp,
                         const int32_t *wci, const double *wval, const int32_t *trp, const int32_t *tci,
                         const double *tv, double *dA, double *dB, uint32_t *err, hipStream_t s)
{
    // lanes per row so that most rows of W fit the stage (16 columns per lane):
    // twice their mean length
    const double mean = m > 0 ? (double)nnz_w / m : 0.0;
    if (2.0 * mean <= kDetStage * 8 + 16)
        launch_det_group<8>(m, kb, nnz_b, nnz_w, arp, aci, brp, bci, bval, wrp, wci, wval, trp, tci, tv, dA, dB, err, s);
    else if (2.0 * mean <= kDetStage * 16)
        launch_det_group<16>(m, kb, nnz_b, nnz_w, arp, aci, brp, bci, bval, wrp, wci, wval, trp, tci, tv, dA, dB, err, s);
    else
        launch_det_group<32>(m, kb, nnz_b, nnz_w, arp, aci, brp, bci, bval, wrp, wci, wval, trp, tci, tv, dA, dB, err, s);
}

// ---------------------------------------------------------------------------
// transpose

__global__ void k_tr_count(int64_t nnz, const int32_t *ci, int32_t *cnt)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nnz) atomicAdd(cnt + gp(ci)[p], 1);
}

__global__ void k_tr_rowptr(int32_t n, const int64_t *prefix, int32_t *trp)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n) gpw(trp)[i] = (int32_t)gp(prefix)[i];
}

constexpr int kTrLanes = 8;   // lanes per row of the scatter (their atomics are independent)

// Rows per launch of the kernels with several lanes per row: a launch holds less
// than 2^32 threads.
constexpr int64_t kTrSlice = 1 << 27;

__global__ __launch_bounds__(kWG) void k_tr_scatter(int64_t row0, int32_t nrows, const int32_t *rp, const int32_t *ci,
                                                    const double *v, const int32_t *trp, int32_t *cursor, int32_t *tci,
                                                    double *tv)
{
    const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
    const int64_t i = row0 + t / kTrLanes;
    if (i >= nrows) return;
    const uint32_t e = (uint32_t)gp(rp)[i + 1];   // (unsigned: the last step may end past the largest int)
    for (uint32_t p = (uint32_t)(gp(rp)[i] + (int)(t % kTrLanes)); p < e; p += kTrLanes) {
        const int c = gp(ci)[p];
        const int pos = gp(trp)[c] + atomicAdd(cursor + c, 1);
        gpw(tci)[pos] = (int32_t)i;
        if (v) gpw(tv)[pos] = gp(v)[p];
    }
}

// Rows of the transpose sorted by column (1.6M entries in rows of 8: 83 us with
// an insertion sort per lane in global memory, 16 us so): an entry's place is the number of
// smaller columns in its row (they are distinct). 16 lanes per row rank rows
// of up to 16 entries from each other's registers; the wave takes the longer
// ones of its four rows one at a time, columns in LDS, up to kTrSortMax
// entries; still longer ones are insertion-sorted by one lane.
constexpr int kTrGroup = 16;
constexpr int kTrPer = 8;                       // entries per lane of a wave's row
constexpr int kTrSortMax = kTrPer * kWave;

__global__ __launch_bounds__(kWG) void k_tr_sort(int64_t row0, int32_t n, const int32_t *trp, int32_t *tci, double *tv)
{
    __shared__ int s_c[kWG / kWave][kTrSortMax];
    const int lane = threadIdx.x & 63, l = lane % kTrGroup;
    int *c = s_c[threadIdx.x >> 6];
    const int64_t r = row0 + ((int64_t)blockIdx.x * kWG + threadIdx.x) / kTrGroup;
    const int s = r < n ? gp(trp)[r] : 0, e = r < n ? gp(trp)[r + 1] : 0;
    const int len = e - s;
    const bool mine = len <= kTrGroup && l < len;
    const int col = mine ? gp(tci)[s + l] : 0x7fffffff;
    const double val = mine && tv ? gp(tv)[s + l] : 0.0;
    int rank = 0;
#pragma unroll
    for (int x = 0; x < kTrGroup; ++x) rank += __shfl(col, x, kTrGroup) < col ? 1 : 0;
    if (mine) {
        gpw(tci)[s + rank] = col;
        if (tv) gpw(tv)[s + rank] = val;
    }
    unsigned long long big = __ballot(l == 0 && len > kTrGroup);
    while (big) {
        const int src = __ffsll((long long)big) - 1;
        big &= big - 1ull;
        const int s0 = __builtin_amdgcn_readlane(s, src), nn = __builtin_amdgcn_readlane(len, src);
        MLS_G int32_t *rc = gpw(tci) + s0;
        MLS_G double *rv = gpw(tv) + s0;
        if (nn <= kTrSortMax) {
            int cv[kTrPer];
            double vv[kTrPer];
#pragma unroll
            for (int u = 0; u < kTrPer; ++u) {
                const int x = u * kWave + lane;
                cv[u] = x < nn ? rc[x] : 0x7fffffff;
                vv[u] = x < nn && tv ? rv[x] : 0.0;
                if (x < nn) c[x] = cv[u];
            }
            bwd_sync();
            int at[kTrPer];
#pragma unroll
            for (int u = 0; u < kTrPer; ++u) at[u] = 0;
            for (int x = 0; x < nn; ++x) {
                const int y = c[x];
#pragma unroll
                for (int u = 0; u < kTrPer; ++u) at[u] += y < cv[u] ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < kTrPer; ++u) {
                if (u * kWave + lane >= nn) continue;
                rc[at[u]] = cv[u];
                if (tv) rv[at[u]] = vv[u];
            }
            bwd_sync();
        } else if (lane == 0) {
            for (int a = 1; a < nn; ++a) {
                const int key = rc[a];
                const double kv = tv ? rv[a] : 0.0;
                int b2 = a - 1;
                while (b2 >= 0 && rc[b2] > key) {
                    rc[b2 + 1] = rc[b2];
                    if (tv) rv[b2 + 1] = rv[b2];
                    --b2;
                }
                rc[b2 + 1] = key;
                if (tv) rv[b2 + 1] = kv;
            }
        }
    }
}

void launch_transpose(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t *rp, const int32_t *ci, const double *v,
                      int32_t *trp, int32_t *tci, double *tv, int32_t *cursor, int64_t *tile_sum, int64_t *prefix,
                      int32_t *cnt, hipStream_t s)
{
    ProfScope ps("transpose", s);
    launch_fill_i32(cnt, 0, (cursor - cnt) + ncols, s);   // cursor follows cnt
    if (nnz > 0) hipLaunchKernelGGL(k_tr_count, dim3((unsigned)((nnz + kWG - 1) / kWG)), dim3(kWG), 0, s, nnz, ci, cnt);
    launch_scan(cnt, ncols, tile_sum, prefix, s);
    hipLaunchKernelGGL(k_tr_rowptr, dim3((ncols + kWG) / kWG), dim3(kWG), 0, s, ncols, prefix, trp);
    auto grid = [](int64_t rows, int lanes) {
        const int64_t per = kWG / lanes;
        return dim3((unsigned)((std::min(rows, kTrSlice) + per - 1) / per));
    };
    for (int64_t r = 0; r < nrows; r += kTrSlice)
        hipLaunchKernelGGL(k_tr_scatter, grid(nrows - r, kTrLanes), dim3(kWG), 0, s, r, nrows, rp, ci, v, trp, cursor,
                           tci, tv);
    for (int64_t r = 0; r < ncols; r += kTrSlice)
        hipLaunchKernelGGL(k_tr_sort, grid(ncols - r, kTrGroup), dim3(kWG), 0, s, r, ncols, trp, tci, tv);
}

// out[e] = X(r, c) for the e-th entry (r, c) of pattern P, else 0.0
__global__ void k_mask_gather(int32_t nrows, const int32_t *xrp, const int32_t *xci, const double *xv,
                              const int32_t *prp, const int32_t *pci, double *out)
{
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nrows) return;
    const int xs = gp(xrp)[r], xn = gp(xrp)[r + 1] - xs;
    for (int p = gp(prp)[r]; p < gp(prp)[r + 1]; ++p) {
        int pos = bsearch_w(gp(xci) + xs, xn, gp(pci)[p]);
        gpw(out)[p] = pos >= 0 ? gp(xv)[xs + pos] : 0.0;
    }
}

void launch_mask_gather(int32_t nrows, const int32_t *xrp, const int32_t *xci, const double *xv, const int32_t *prp,
                        const int32_t *pci, double *out, hipStream_t s)
{
    if (nrows <= 0) return;
    ProfScope ps("mask_gather", s);
    hipLaunchKernelGGL(k_mask_gather, dim3((nrows + kWG - 1) / kWG), dim3(kWG), 0, s, nrows, xrp, xci, xv, prp, pci,
                       out);
}

}  // namespace mls
