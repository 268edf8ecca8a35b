// api.hip -- C ABI: workspace layout and the launch sequences of the plain
// and batched two-phase product (Sec. 2.1).
#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/mlspgemm.h"
#include "common.h"
#include "launch.h"
#include "internal.h"

using namespace mls;

namespace mls {

thread_local int g_last_hip_error = 0;
Options g_opt;

spgemm_status hip_fail(hipError_t e)
{
    g_last_hip_error = (int)e;
    return SPGEMM_ERR_HIP;
}

spgemm_status check_launch()
{
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPGEMM_OK : hip_fail(e);
}

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Lanes per row from a mean row length: the next power of two, at least 16. (8
// lanes lose at every mean measured, 3 to 8, on 300000 random rows: a class of
// 256 slots is bound by latency, and wider groups put fewer rows, with less
// LDS, in a wave. Mean 7.9: numeric 429 against 320 us, adjoint 669 against
// 394, symbolic 2449 against 1879; mean 3: 186/168, 274/227, 726/678.)
int pow2_group(double avg)
{
    int g = 16;
    while (g < 64 && g < avg) g <<= 1;
    return g;
}

// Workspace regions for a batch run over na A-rows, nb B-rows, zb B-entries.
Layout make_layout(int64_t nprob, int64_t na, int64_t nb, int64_t zb, int64_t max_ncols, bool need_bw)
{
    Layout L;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align_up(bytes); return o; };
    L.hdr = take(kHdrBytes);
    L.totals = take(sizeof(int64_t) * (size_t)std::max<int64_t>(nprob, 1));
    L.nnz_tab = take(sizeof(int64_t) * 2 * (size_t)std::max<int64_t>(nprob, 1));
    L.probs = take(sizeof(Prob) * (size_t)std::max<int64_t>(nprob, 1));
    L.abase = take(sizeof(int32_t) * (size_t)(nprob + 1));
    L.bbase = take(sizeof(int32_t) * (size_t)(nprob + 1));
    L.val = take(sizeof(int32_t) * (size_t)std::max<int64_t>(na, 1));
    L.cls = take((size_t)std::max<int64_t>(na, 1));
    L.perm = take(sizeof(int32_t) * (size_t)std::max<int64_t>(na, 1));
    L.nblk = (int32_t)((std::max<int64_t>(na, 1) + kBinRowsPerWG - 1) / kBinRowsPerWG);
    L.blk = take(sizeof(int32_t) * (size_t)kNumBins * (size_t)L.nblk);
    L.prefix = take(sizeof(int64_t) * (size_t)(na + 1));
    L.tiles = take(sizeof(int64_t) * (size_t)scan_tiles((int)std::min<int64_t>(na, 0x7fffffff)));
    if (need_bw) {
        L.bw = take(sizeof(uint2) * (size_t)std::max<int64_t>(zb, 1));
        L.bwc = take(sizeof(int32_t) * (size_t)std::max<int64_t>(nb, 1));
        int64_t words = (std::max<int64_t>(max_ncols, 1) + 31) / 32;
        int64_t slots = (int64_t)(256ll << 20) / (words * 4);
        slots = std::max<int64_t>(1, std::min<int64_t>(64, slots));
        L.spill_words = words;
        L.spill_slots = (int)slots;
        L.spill = take(sizeof(uint32_t) * (size_t)(words * slots));
    }
    L.total_min = off;
    if (need_bw) {
        L.scnt = take(sizeof(int32_t) * (size_t)std::max<int64_t>(na, 1));
        L.scr = take(sizeof(uint2) * (size_t)kScratchWords * (size_t)std::max<int64_t>(na, 1));
    }
    L.total = off;
    return L;
}

// The count pass may leave compressed B and the rows' set words in the
// workspace; a fill pass on the same workspace and the same operands uses them
// instead of recomputing. Any other call on that workspace forgets them.
namespace {
std::mutex g_memo_mu;
struct SymMemo {
    const void *ws = nullptr;
    std::vector<uint64_t> key;
    bool valid = false;
    unsigned seen = 0;   // sizes of rows among the kept words (bits kSeen*)
    SymBits bits = kBitsNone;   // what the count pass ran as
} g_memo;
}  // namespace

void memo_forget(const void *ws)
{
    std::lock_guard<std::mutex> lk(g_memo_mu);
    if (g_memo.ws == ws) g_memo.valid = false;
}

Sched make_sched(char *ws, const Layout &L)
{
    Sched sc;
    sc.err = (uint32_t *)(ws + L.hdr + kHdrErr);
    sc.bin_count = (int32_t *)(ws + L.hdr + kHdrBinCount);
    sc.blk_cnt = (int32_t *)(ws + L.blk);
    sc.nblk = L.nblk;
    sc.task_cursor = (int32_t *)(ws + L.hdr + kHdrTaskCursor);
    sc.val = (int32_t *)(ws + L.val);
    sc.cls = (uint8_t *)(ws + L.cls);
    sc.perm = (int32_t *)(ws + L.perm);
    sc.scr = L.has_scratch ? (uint2 *)(ws + L.scr) : nullptr;
    sc.scnt = L.has_scratch ? (int32_t *)(ws + L.scnt) : nullptr;
    sc.seen = (uint32_t *)(ws + L.hdr + kHdrSeen);
    sc.wstart = (int32_t *)(ws + L.prefix);   // the row-pointer scan's array, idle outside the symbolic phase
    return sc;
}

void reset_header(char *ws, const Layout &L, hipStream_t s)
{
    launch_fill_i32((int32_t *)(ws + L.hdr), 0, kHdrBytes / 4, s);
}

// Page-locked landing places for the readbacks: a copy into pageable memory is
// staged by the runtime (20.5 us for 8 to 1032 bytes on an idle stream, 12.6
// us into page-locked memory). One block of kReadSlots slots for the process,
// taken on first use and kept to its end; a call holds a slot only while it
// waits. With every slot taken, or no such memory, the copy goes to the
// caller's own memory.
namespace {
constexpr int kReadSlots = 64;
constexpr size_t kReadSlotBytes = 2048;
std::mutex g_read_mu;
char *g_read_block = nullptr;
bool g_read_tried = false;
uint64_t g_read_free = ~0ull;
static_assert(kReadSlots == 64, "one bit per slot");

struct ReadSlot {
    char *p = nullptr;
    int idx = -1;
    explicit ReadSlot(size_t bytes)
    {
        if (bytes > kReadSlotBytes) return;
        std::lock_guard<std::mutex> lk(g_read_mu);
        if (!g_read_tried) {
            g_read_tried = true;
            void *b = nullptr;
            if (hipHostMalloc(&b, kReadSlots * kReadSlotBytes, hipHostMallocPortable) == hipSuccess)
                g_read_block = (char *)b;
            else
                (void)hipGetLastError();
        }
        if (!g_read_block || !g_read_free) return;
        idx = __builtin_ctzll(g_read_free);
        g_read_free &= g_read_free - 1;
        p = g_read_block + (size_t)idx * kReadSlotBytes;
    }
    ~ReadSlot()
    {
        if (idx < 0) return;
        std::lock_guard<std::mutex> lk(g_read_mu);
        g_read_free |= 1ull << idx;
    }
};
}  // namespace

spgemm_status read_back(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    ReadSlot slot(bytes);
    hipError_t e = hipMemcpyAsync(slot.p ? slot.p : dst, src, bytes, hipMemcpyDeviceToHost, s);
    // (waited for in either case: a copy queued must not outlive the slot)
    const hipError_t e2 = hipStreamSynchronize(s);
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) return hip_fail(e);
    if (slot.p) std::memcpy(dst, slot.p, bytes);
    return SPGEMM_OK;
}

spgemm_status read_errors(char *ws, const Layout &L, hipStream_t s)
{
    uint32_t err = 0;
    const spgemm_status st = read_back(&err, ws + L.hdr + kHdrErr, sizeof(err), s);
    return st == SPGEMM_OK ? err_status(err) : st;
}

spgemm_status err_status(uint32_t err)
{
    if (err & kErrBadCsr) return SPGEMM_ERR_BAD_CSR;
    if (err & kErrOverflow) return SPGEMM_ERR_INDEX_OVERFLOW;
    if (err & kErrStructure) return SPGEMM_ERR_STRUCTURE;
    if (err & kErrTable) return SPGEMM_ERR_STRUCTURE;
    return SPGEMM_OK;
}

// Error word and the header's total in one copy. A refused operand leaves
// *total_host alone.
spgemm_status read_header_total(char *ws, const Layout &L, int64_t *total_host, hipStream_t s)
{
    char hdr[kHdrBytes];
    const spgemm_status st = read_back(hdr, ws + L.hdr, kHdrBytes, s);
    if (st != SPGEMM_OK) return st;
    uint32_t err = 0;
    std::memcpy(&err, hdr + kHdrErr, sizeof(err));
    if (total_host && !(err & kErrBadCsr)) std::memcpy(total_host, hdr + kHdrTotal, sizeof(*total_host));
    return err_status(err);
}

static bool csr_ok(const spgemm_csr *M, bool need_values)
{
    if (!M || M->nrows < 0 || M->ncols < 0 || M->nnz < 0 || M->nnz >= 0x7fffffffLL) return false;
    if (!M->row_ptr) return false;
    if (M->nnz > 0 && !M->col_idx) return false;
    if (need_values && M->nnz > 0 && !M->values) return false;
    return true;
}

// Host-side description of a batch call; uploads the descriptors when
// there is more than one product.
spgemm_status prepare_batch(int32_t nbatch, const spgemm_csr *A, const spgemm_csr *B, const spgemm_csr *C,
                            bool need_values, bool need_bw, char *ws, size_t ws_bytes, hipStream_t s,
                            BatchHost &out, bool upload)
{
    if (nbatch < 1 || !A || !B) return SPGEMM_ERR_INVALID_ARG;
    int64_t na = 0, nb = 0, zb = 0, maxc = 0, za = 0;
    for (int t = 0; t < nbatch; ++t) {
        if (!csr_ok(&A[t], need_values) || !csr_ok(&B[t], need_values)) return SPGEMM_ERR_INVALID_ARG;
        if (A[t].ncols != B[t].nrows) return SPGEMM_ERR_DIM_MISMATCH;
        na += A[t].nrows;
        nb += B[t].nrows;
        zb += B[t].nnz;
        za += A[t].nnz;
        maxc = std::max<int64_t>(maxc, B[t].ncols);
    }
    if (na >= 0x7fffffff || nb >= 0x7fffffff) return SPGEMM_ERR_INDEX_OVERFLOW;
    out.layout = make_layout(nbatch, na, nb, zb, maxc, need_bw);
    if (!ws || ws_bytes < out.layout.total_min) return SPGEMM_ERR_WORKSPACE_TOO_SMALL;
    out.layout.has_scratch = need_bw && ws_bytes >= out.layout.total;
    if (((uintptr_t)ws & 255) != 0) return SPGEMM_ERR_INVALID_ARG;
    out.probs.assign(nbatch, Prob{});
    out.abase.assign(nbatch + 1, 0);
    out.bbase.assign(nbatch + 1, 0);
    out.nnz_tab.assign(2 * (size_t)nbatch, 0);
    int64_t eb = 0;
    for (int t = 0; t < nbatch; ++t) {
        Prob &P = out.probs[t];
        P.arp = A[t].row_ptr; P.aci = A[t].col_idx; P.aval = A[t].values;
        P.brp = B[t].row_ptr; P.bci = B[t].col_idx; P.bval = B[t].values;
        // a step on an empty row of B may read B's first entry (and ignore it):
        // with no entries at all, any device memory serves
        if (B[t].nnz == 0) { P.bci = (const int32_t *)ws; P.bval = (const double *)ws; }
        if (need_bw) {
            P.bw = (uint2 *)(ws + out.layout.bw) + eb;
            P.bwc = (int32_t *)(ws + out.layout.bwc) + out.bbase[t];
        }
        if (C) { P.crp = C[t].row_ptr; P.cci = C[t].col_idx; P.cval = C[t].values; }
        P.nrows = A[t].nrows;
        P.ncols = B[t].ncols;
        P.krows = B[t].nrows;
        P.k_lo = 0;
        P.k_hi = B[t].nrows;
        out.abase[t + 1] = out.abase[t] + A[t].nrows;
        out.bbase[t + 1] = out.bbase[t] + B[t].nrows;
        out.nnz_tab[2 * t] = A[t].nnz;
        out.nnz_tab[2 * t + 1] = B[t].nnz;
        eb += B[t].nnz;
    }
    Batch &bt = out.batch;
    std::memset(&bt, 0, sizeof(bt));
    bt.nprob = nbatch;
    bt.na = (int32_t)na;
    bt.nb = (int32_t)nb;
    // 0 keeps the numeric phase on the wide hash slots
    if (!g_opt.wide_table)
        for (int t = 0; t < nbatch; ++t) bt.max_ncols = std::max(bt.max_ncols, B[t].ncols);
    bt.p0 = out.probs[0];
    bt.probs = (const Prob *)(ws + out.layout.probs);
    bt.abase = (const int32_t *)(ws + out.layout.abase);
    bt.bbase = (const int32_t *)(ws + out.layout.bbase);
    out.zc = 0;
    for (int t = 0; C && t < nbatch; ++t) out.zc += std::max<int64_t>(C[t].nnz, 0);
    out.za = za;
    out.zb = zb;
    out.avg_a = na > 0 ? (double)za / (double)na : 1.0;
    out.avg_b = nb > 0 ? (double)zb / (double)nb : 1.0;
    std::vector<uint64_t> &key = out.key;
    key.clear();
    key.push_back((uint64_t)nbatch);
    key.push_back((uint64_t)ws_bytes);
    for (int t = 0; t < nbatch; ++t) {
        key.push_back((uint64_t)(uintptr_t)A[t].row_ptr);
        key.push_back((uint64_t)(uintptr_t)A[t].col_idx);
        key.push_back((uint64_t)(uintptr_t)B[t].row_ptr);
        key.push_back((uint64_t)(uintptr_t)B[t].col_idx);
        key.push_back((uint64_t)(uint32_t)A[t].nrows);
        key.push_back((uint64_t)(uint32_t)A[t].ncols);
        key.push_back((uint64_t)(uint32_t)B[t].nrows);
        key.push_back((uint64_t)(uint32_t)B[t].ncols);
        key.push_back((uint64_t)A[t].nnz);
        key.push_back((uint64_t)B[t].nnz);
        key.push_back(C ? (uint64_t)(uintptr_t)C[t].row_ptr : 0ull);
    }
    // a single product goes to the kernels by value, its entry counts included
    if (nbatch == 1) return SPGEMM_OK;
    if (!upload) return SPGEMM_ERR_INVALID_ARG;
    hipError_t e = hipSuccess;
    e = hipMemcpyAsync(ws + out.layout.nnz_tab, out.nnz_tab.data(), sizeof(int64_t) * out.nnz_tab.size(),
                       hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        e = hipMemcpyAsync(ws + out.layout.probs, out.probs.data(), sizeof(Prob) * nbatch, hipMemcpyHostToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(ws + out.layout.abase, out.abase.data(), sizeof(int32_t) * (nbatch + 1),
                               hipMemcpyHostToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(ws + out.layout.bbase, out.bbase.data(), sizeof(int32_t) * (nbatch + 1),
                               hipMemcpyHostToDevice, s);
    }
    if (e != hipSuccess) return hip_fail(e);
    return SPGEMM_OK;
}

int choose_group(double avg)
{
    if (g_opt.group_size) return (int)g_opt.group_size;
    return pow2_group(avg);
}

// CSR checks of the operands, queued; the kernels behind them return at once
// when they fail (bad_csr). B is not checked again when every B_t is A_t itself.
static void queue_validate(const BatchHost &bh, char *ws, uint32_t *err, hipStream_t s)
{
    bool same = true;
    for (int t = 0; t < bh.batch.nprob && same; ++t) {
        const Prob &q = bh.probs[t];
        same = q.arp == q.brp && q.aci == q.bci && q.nrows == q.krows && q.ncols == q.krows &&
               q.a_off == q.b_off && bh.nnz_tab[2 * t] == bh.nnz_tab[2 * t + 1];
    }
    const int64_t *tab = bh.batch.nprob > 1 ? (const int64_t *)(ws + bh.layout.nnz_tab) : nullptr;
    launch_validate(bh.batch, same ? 0 : 2, tab, bh.za, bh.zb, err, s);
}

// Waits for a count pass: error word and nnz of every product, in one copy
// (the header, which begins with the error word, and the totals behind it).
static spgemm_status read_counts(BatchHost &bh, char *ws, int64_t *nnz_host, unsigned &seen, hipStream_t s)
{
    const Layout &L = bh.layout;
    const int np = bh.batch.nprob;
    static_assert(kHdrErr == 0 && kHdrBytes % sizeof(int64_t) == 0, "read as one block");
    const size_t words = (L.totals - L.hdr) / sizeof(int64_t);
    std::vector<int64_t> got(words + (size_t)np, 0);
    const spgemm_status st = read_back(got.data(), ws + L.hdr, sizeof(int64_t) * got.size(), s);
    if (st != SPGEMM_OK) return st;
    uint32_t err = 0;
    std::memcpy(&err, got.data(), sizeof(err));
    uint32_t sizes[kNumSeen];
    std::memcpy(sizes, (const char *)got.data() + kHdrSeen, sizeof(sizes));
    seen = 0;
    for (int x = 0; x < kNumSeen; ++x) seen |= sizes[x] ? 1u << x : 0u;
    if (err & kErrBadCsr) return err_status(err);
    int64_t *tot = got.data() + words;
    // products with no rows never write their total
    for (int t = 0; t < np; ++t)
        if (bh.probs[t].nrows == 0) tot[t] = 0;
    if (nnz_host) std::memcpy(nnz_host, tot, sizeof(int64_t) * (size_t)np);
    for (int t = 0; t < np; ++t)
        if (tot[t] >= 0x7fffffffLL) return SPGEMM_ERR_INDEX_OVERFLOW;
    return err_status(err);
}

// Symbolic count or fill over a prepared batch.
spgemm_status run_symbolic(BatchHost &bh, char *ws, int fill, int64_t *nnz_host, hipStream_t s)
{
    Layout &L = bh.layout;
    // few columns: dense bitmaps in place of binning and hash tables, by rule (the
    // test knobs that choose a path or class keep those)
    const SymBits bits = g_opt.force_spill || g_opt.force_class >= 0 ? kBitsNone
                                                                     : symbit_choose(bh.batch, bh.avg_a, bh.avg_b);
    bool reuse = false;
    unsigned seen = 0;
    {
        std::lock_guard<std::mutex> lk(g_memo_mu);
        reuse = fill && g_memo.valid && g_memo.ws == ws && g_memo.bits == bits && g_memo.key == bh.key;
        seen = g_memo.seen;
        if (g_memo.ws == ws) g_memo.valid = false;
    }
    if (fill && !reuse) L.has_scratch = false;   // nothing to expand: recompute every row
    Sched sc = make_sched(ws, L);
    reset_header(ws, L, s);
    if (!fill && g_opt.validate) queue_validate(bh, ws, sc.err, s);
    if (bits != kBitsNone) {
        if (bits == kBitsWords && !reuse) launch_compress(bh.batch, bh.zb, sc.err, s);
        launch_symbit(bh.batch, sc, fill, bits == kBitsWords, s);
    } else {
        if (!reuse) launch_compress(bh.batch, bh.zb, sc.err, s);
        // the fill of a count whose words were all kept has nothing to bin and
        // no row to recompute, and only the sizes of rows seen to expand (an
        // empty launch costs at least 4.5 us of stream time; 20 Galerkin setups
        // 1.75 -> 1.68 ms)
        const bool again = !fill || !reuse || !sc.scr || (seen >> kSeenMore & 1u);
        if (!fill) launch_bin_count(bh.batch, bh.za, sc, bin_force(), s);
        else if (again) launch_bin(bh.batch, kModeFill, sc, bin_force(), nullptr, s);
        if (fill) launch_sym_expand(bh.batch, sc, seen, s);
        if (again) launch_symbolic(bh.batch, sc, fill, choose_group(bh.avg_a), s);
    }
    spgemm_status st = check_launch();
    if (st != SPGEMM_OK) return st;
    if (fill) {
        if (reuse) {   // the words stay valid for another fill pass on the same operands
            std::lock_guard<std::mutex> lk(g_memo_mu);
            g_memo.ws = ws; g_memo.key = bh.key; g_memo.valid = true; g_memo.seen = seen;
            g_memo.bits = bits;
        }
        return SPGEMM_OK;
    }
    for (int t = 0; t < bh.batch.nprob; ++t)
        if (bh.probs[t].nrows == 0) launch_fill_i32(bh.probs[t].crp, 0, 1, s);
    if (bits != kBitsNone && bh.batch.na > 0 && bh.batch.na <= kRowptrSmallRows) {
        launch_rowptr_small(bh.batch, sc.val, (int64_t *)(ws + L.totals), sc.err, s);
    } else {
        int64_t *prefix = (int64_t *)(ws + L.prefix);
        launch_scan(sc.val, bh.batch.na, (int64_t *)(ws + L.tiles), prefix, s);
        launch_write_rowptr(bh.batch, prefix, (int64_t *)(ws + L.totals), sc.err, s);
    }
    st = check_launch();
    if (st != SPGEMM_OK) return st;
    st = read_counts(bh, ws, nnz_host, seen, s);
    if (st == SPGEMM_OK && bits != kBitsColumns) {
        std::lock_guard<std::mutex> lk(g_memo_mu);
        g_memo.ws = ws; g_memo.key = bh.key; g_memo.valid = true; g_memo.seen = seen;
        g_memo.bits = bits;
    }
    return st;
}

spgemm_status run_numeric(BatchHost &bh, char *ws, hipStream_t s)
{
    memo_forget(ws);
    const Layout &L = bh.layout;
    Sched sc = make_sched(ws, L);
    // few rows: two launches in all (the test knobs that choose classes, lanes
    // or table layouts keep the launches by class)
    if (num_small_fit(bh.batch, bh.zc) && bin_force() < 0 && !g_opt.group_size) {
        launch_numeric_small(bh.batch, sc, bh.zc, s);
        return check_launch();
    }
    reset_header(ws, L, s);
    launch_bin(bh.batch, kModeNumeric, sc, bin_force(), nullptr, s);
    launch_numeric(bh.batch, sc, choose_group(bh.avg_b), s);
    return check_launch();
}

}  // namespace mls

// ===========================================================================
// extern "C"

extern "C" {

const char *spgemm_status_string(spgemm_status s)
{
    switch (s) {
    case SPGEMM_OK: return "ok";
    case SPGEMM_ERR_INVALID_ARG: return "invalid argument";
    case SPGEMM_ERR_BAD_CSR: return "invalid CSR matrix";
    case SPGEMM_ERR_DIM_MISMATCH: return "dimension mismatch";
    case SPGEMM_ERR_INDEX_OVERFLOW: return "index overflow (2^31)";
    case SPGEMM_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case SPGEMM_ERR_BUDGET: return "HBM budget too small";
    case SPGEMM_ERR_HIP: return "HIP runtime error";
    case SPGEMM_ERR_UNSUPPORTED: return "unsupported";
    case SPGEMM_ERR_STRUCTURE: return "output structure misses a reached column";
    }
    return "unknown status";
}

int spgemm_last_hip_error(void) { return g_last_hip_error; }

int spgemm_version(void) { return 10000; }

spgemm_status spgemm_set_option(spgemm_option opt, int64_t value)
{
    switch (opt) {
    case SPGEMM_OPT_VALIDATE: g_opt.validate = value != 0; return SPGEMM_OK;
    case SPGEMM_OPT_FORCE_SPILL: g_opt.force_spill = value != 0; return SPGEMM_OK;
    case SPGEMM_OPT_GROUP_SIZE:
        if (value != 0 && value != 8 && value != 16 && value != 32 && value != 64) return SPGEMM_ERR_INVALID_ARG;
        g_opt.group_size = value;
        return SPGEMM_OK;
    case SPGEMM_OPT_FORCE_CLASS:
        if (value < -1 || value >= kNumClasses) return SPGEMM_ERR_INVALID_ARG;
        g_opt.force_class = (int)value;
        return SPGEMM_OK;
    case SPGEMM_OPT_PROFILE: g_opt.profile = value != 0; return SPGEMM_OK;
    case SPGEMM_OPT_WIDE_TABLE: g_opt.wide_table = value != 0; return SPGEMM_OK;
    }
    return SPGEMM_ERR_INVALID_ARG;
}

int64_t spgemm_get_option(spgemm_option opt)
{
    switch (opt) {
    case SPGEMM_OPT_VALIDATE: return g_opt.validate;
    case SPGEMM_OPT_FORCE_SPILL: return g_opt.force_spill;
    case SPGEMM_OPT_GROUP_SIZE: return g_opt.group_size;
    case SPGEMM_OPT_PROFILE: return g_opt.profile;
    case SPGEMM_OPT_WIDE_TABLE: return g_opt.wide_table;
    case SPGEMM_OPT_FORCE_CLASS: return g_opt.force_class;
    default: return 0;
    }
}

spgemm_status spgemm_validate_host(const spgemm_csr *M)
{
    if (!M || M->nrows < 0 || M->ncols < 0 || !M->row_ptr) return SPGEMM_ERR_INVALID_ARG;
    if (M->row_ptr[0] != 0) return SPGEMM_ERR_BAD_CSR;
    for (int32_t i = 0; i < M->nrows; ++i) {
        int32_t s = M->row_ptr[i], e = M->row_ptr[i + 1];
        if (e < s) return SPGEMM_ERR_BAD_CSR;
        for (int32_t p = s; p < e; ++p) {
            int32_t c = M->col_idx[p];
            if (c < 0 || c >= M->ncols) return SPGEMM_ERR_BAD_CSR;
            if (p > s && c <= M->col_idx[p - 1]) return SPGEMM_ERR_BAD_CSR;
        }
    }
    if ((int64_t)M->row_ptr[M->nrows] != M->nnz) return SPGEMM_ERR_BAD_CSR;
    return SPGEMM_OK;
}

spgemm_status spgemm_workspace_size(const spgemm_csr *A, const spgemm_csr *B, size_t *bytes)
{
    return spgemm_batch_workspace_size(1, A, B, bytes);
}

spgemm_status spgemm_batch_workspace_size(int32_t nbatch, const spgemm_csr *A, const spgemm_csr *B, size_t *bytes)
{
    if (nbatch < 1 || !A || !B || !bytes) return SPGEMM_ERR_INVALID_ARG;
    int64_t na = 0, nb = 0, zb = 0, maxc = 0;
    for (int t = 0; t < nbatch; ++t) {
        na += A[t].nrows;
        nb += B[t].nrows;
        zb += B[t].nnz;
        maxc = std::max<int64_t>(maxc, B[t].ncols);
    }
    *bytes = make_layout(nbatch, na, nb, zb, maxc, true).total;
    return SPGEMM_OK;
}

spgemm_status spgemm_row_work(const spgemm_csr *A, const spgemm_csr *B, int32_t *work, int64_t *total_host,
                              void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!work) return SPGEMM_ERR_INVALID_ARG;
    BatchHost bh;
    memo_forget(ws);
    spgemm_status st = prepare_batch(1, A, B, nullptr, false, false, (char *)ws, ws_bytes, stream, bh);
    if (st != SPGEMM_OK) return st;
    char *w = (char *)ws;
    Sched sc = make_sched(w, bh.layout);
    sc.val = work;
    reset_header(w, bh.layout, stream);
    unsigned long long *tot = (unsigned long long *)(w + bh.layout.hdr + kHdrTotal);
    launch_bin(bh.batch, kModeWork, sc, 0, tot, stream);
    st = check_launch();
    if (st != SPGEMM_OK) return st;
    return read_header_total(w, bh.layout, total_host, stream);
}

spgemm_status spgemm_compress(const spgemm_csr *B, uint32_t *words, int32_t *count, void *ws, size_t ws_bytes,
                              hipStream_t stream)
{
    (void)ws; (void)ws_bytes;
    if (!csr_ok(B, false) || !count || (B->nnz > 0 && !words)) return SPGEMM_ERR_INVALID_ARG;
    Batch b;
    std::memset(&b, 0, sizeof(b));
    b.nprob = 1;
    b.nb = B->nrows;
    b.p0.brp = B->row_ptr;
    b.p0.bci = B->col_idx;
    b.p0.bw = (uint2 *)words;
    b.p0.bwc = count;
    b.p0.ncols = B->ncols;
    b.p0.krows = B->nrows;
    launch_compress(b, B->nnz, nullptr, stream);
    return check_launch();
}

spgemm_status spgemm_symbolic(const spgemm_csr *A, const spgemm_csr *B, int32_t *C_row_ptr, int32_t *C_col_idx,
                              int64_t *nnzC_host, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!C_row_ptr) return SPGEMM_ERR_INVALID_ARG;
    spgemm_csr C;
    std::memset(&C, 0, sizeof(C));
    C.nrows = A ? A->nrows : 0;
    C.ncols = B ? B->ncols : 0;
    C.row_ptr = C_row_ptr;
    C.col_idx = C_col_idx;
    return spgemm_batch_symbolic(1, A, B, &C, C_col_idx != nullptr, nnzC_host, ws, ws_bytes, stream);
}

spgemm_status spgemm_batch_symbolic(int32_t nbatch, const spgemm_csr *A, const spgemm_csr *B, spgemm_csr *C,
                                    int32_t fill, int64_t *nnzC_host, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!C) return SPGEMM_ERR_INVALID_ARG;
    for (int t = 0; t < nbatch; ++t) {
        if (!C[t].row_ptr) return SPGEMM_ERR_INVALID_ARG;
        if (fill && !C[t].col_idx) return SPGEMM_ERR_INVALID_ARG;
    }
    BatchHost bh;
    spgemm_status st = prepare_batch(nbatch, A, B, C, false, true, (char *)ws, ws_bytes, stream, bh);
    if (st != SPGEMM_OK) return st;
    return run_symbolic(bh, (char *)ws, fill ? 1 : 0, nnzC_host, stream);
}

spgemm_status spgemm_numeric(const spgemm_csr *A, const spgemm_csr *B, spgemm_csr *C, void *ws, size_t ws_bytes,
                             hipStream_t stream)
{
    return spgemm_batch_numeric(1, A, B, C, ws, ws_bytes, stream);
}

spgemm_status spgemm_batch_numeric(int32_t nbatch, const spgemm_csr *A, const spgemm_csr *B, spgemm_csr *C,
                                   void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!C) return SPGEMM_ERR_INVALID_ARG;
    for (int t = 0; t < nbatch; ++t) {
        if (C[t].nrows != A[t].nrows || C[t].ncols != B[t].ncols) return SPGEMM_ERR_DIM_MISMATCH;
        if (!C[t].row_ptr || (C[t].nnz > 0 && (!C[t].col_idx || !C[t].values))) return SPGEMM_ERR_INVALID_ARG;
    }
    BatchHost bh;
    spgemm_status st = prepare_batch(nbatch, A, B, C, true, false, (char *)ws, ws_bytes, stream, bh);
    if (st != SPGEMM_OK) return st;
    return run_numeric(bh, (char *)ws, stream);
}

spgemm_status spgemm_check_errors(void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!ws || ws_bytes < kHdrBytes) return SPGEMM_ERR_INVALID_ARG;
    Layout L;
    std::memset(&L, 0, sizeof(L));
    L.hdr = 0;
    spgemm_status st = read_errors((char *)ws, L, stream);
    // (a word that is 0 already needs no clearing)
    if (st == SPGEMM_ERR_BAD_CSR || st == SPGEMM_ERR_INDEX_OVERFLOW ||
        st == SPGEMM_ERR_STRUCTURE) {
        launch_fill_i32((int32_t *)((char *)ws + kHdrErr), 0, 1, stream);
        (void)check_launch();   // the word's own verdict is the call's
    }
    return st;
}

}  // extern "C"
