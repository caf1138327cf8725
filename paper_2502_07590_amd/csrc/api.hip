// C ABI of libdsv: argument checks, workspace layout, launch order.  All checks run on the host
// before anything is enqueued; the library never allocates device memory.
#include <algorithm>
#include <cmath>
#include <initializer_list>
#include <mutex>
#include <optional>
#include <vector>

#include "common.h"

namespace dsv {
KernelTimer g_kernel_timer;
namespace {

bool supported_d(int d) { return d == 64 || d == 128; }
bool supported_r(int r) { return r == 16 || r == 32 || r == 64; }
bool supported_dtype(int t) { return t == DSV_F32 || t == DSV_BF16; }
size_t esize(int dtype) { return dtype == DSV_BF16 ? 2 : 4; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// true when every pointer is non-null and 16-byte aligned
bool ok_ptrs(std::initializer_list<const void *> ps)
{
    for (const void *p : ps)
        if (!p || !aligned16(p)) return false;
    return true;
}

dsv_status check_problem(const dsv_problem *p, bool need_r)
{
    if (!p || !p->k_per_head) return DSV_EINVAL;
    if (p->B < 1 || p->H < 1 || p->L < 1) return DSV_EINVAL;
    // (batch, head) pairs index grid.y / grid.x of several kernels (limit 65535)
    if ((int64_t)p->B * p->H > 65535) return DSV_EINVAL;
    if (p->flags & ~DSV_FLAG_SORTED_INDEX) return DSV_EINVAL;
    if (!supported_dtype(p->dtype) || !supported_d(p->d)) return DSV_EUNSUPPORTED;
    if (need_r && !supported_r(p->r)) return DSV_EUNSUPPORTED;
    // the gather kernels address a head's [L, d] matrix with 32-bit byte offsets
    if ((uint64_t)p->L * (uint64_t)p->d * esize(p->dtype) >= (1ull << 32)) return DSV_EUNSUPPORTED;
    for (int h = 0; h < p->H; ++h)
        if (p->k_per_head[h] < 1 || p->k_per_head[h] > p->L) return DSV_EINVAL;
    return DSV_OK;
}

// Launch tables: all (b, h) pairs sorted by descending k (stable), cut into groups of kMaxSlots.
// rows: index rows per head (p.L, or the number of query groups); 0 = p.L.
std::vector<HeadTable> make_tables(const dsv_problem &p, int rows = 0)
{
    const int nbh = p.B * p.H;
    if (rows == 0) rows = p.L;
    std::vector<int64_t> off(nbh + 1, 0);
    for (int bh = 0; bh < nbh; ++bh) off[bh + 1] = off[bh] + (int64_t)rows * p.k_per_head[bh % p.H];
    std::vector<int> order(nbh);
    for (int i = 0; i < nbh; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return p.k_per_head[a % p.H] > p.k_per_head[b % p.H]; });
    std::vector<HeadTable> tabs((nbh + kMaxSlots - 1) / kMaxSlots);
    for (int i = 0; i < nbh; ++i) {
        HeadTable &t = tabs[i / kMaxSlots];
        const int s = i % kMaxSlots;
        t.n = s + 1;
        t.bh[s] = order[i];
        t.k[s] = p.k_per_head[order[i] % p.H];
        t.off[s] = off[order[i]];
    }
    return tabs;
}

size_t total_pairs(const dsv_problem &p)
{
    size_t nnz = 0;
    for (int bh = 0; bh < p.B * p.H; ++bh) nnz += (size_t)p.L * p.k_per_head[bh % p.H];
    return nnz;
}

dsv_status check_workspace(const void *ws, size_t have, size_t need)
{
    if (need == 0) return DSV_OK;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) || have < need) return DSV_EWORKSPACE;
    return DSV_OK;
}

// ---- workspace layouts (byte offsets, every block aligned to 256) ------------------------------
struct Stage1Layout {
    size_t qlr, klr, prefix, krem, win, todo, jcut, cnt, tflag, qc, total;
};

// transposed: also room for jcut and the per-key list lengths of the key-major emission.
// Lq: scored query rows per head (p.L, or one centre query per group: then also room for those rows, qc).
Stage1Layout stage1_layout(const dsv_problem &p, bool transposed, int Lq = 0)
{
    const bool grouped = Lq != 0;
    if (!grouped) Lq = p.L;
    const size_t nbh = (size_t)p.B * p.H;
    const size_t qp = nbh * ((Lq + 31) / 32 * 32);  // per-query state rows are padded to tiles
    Stage1Layout w{};
    size_t o = 0;
    w.qlr = o; o = align_up(o + nbh * Lq * p.r * esize(p.dtype), 256);
    w.klr = o; o = align_up(o + nbh * p.L * p.r * esize(p.dtype), 256);
    w.prefix = o; o = align_up(o + qp * 4, 256);
    w.krem = o; o = align_up(o + qp * 4, 256);
    w.win = o; o = align_up(o + qp * 4, 256);
    w.todo = o; o = align_up(o + (1 + nbh * ((Lq + 31) / 32)) * 4, 256);
    w.jcut = o; if (transposed) o = align_up(o + qp * 4, 256);
    w.cnt = o; if (transposed) o = align_up(o + nbh * p.L * 4, 256);
    w.tflag = o; if (transposed) o = align_up(o + nbh * ((Lq + 31) / 32) * 4, 256);
    w.qc = o; if (grouped) o = align_up(o + nbh * Lq * p.d * esize(p.dtype), 256);
    w.total = o;
    return w;
}

// Cubes must tile the grid, and the grid must be the problem's L tokens.
dsv_status check_grouping(const dsv_problem &p, const dsv_grouping *g)
{
    if (!g) return DSV_EINVAL;
    if (g->F < 1 || g->Hh < 1 || g->Ww < 1 || g->gf < 1 || g->gh < 1 || g->gw < 1) return DSV_EINVAL;
    if ((int64_t)g->F * g->Hh * g->Ww != (int64_t)p.L) return DSV_EINVAL;
    if (g->F % g->gf || g->Hh % g->gh || g->Ww % g->gw) return DSV_EINVAL;
    if ((int64_t)g->gf * g->gh * g->gw > 64) return DSV_EUNSUPPORTED;
    return DSV_OK;
}
int group_size(const dsv_grouping &g) { return g.gf * g.gh * g.gw; }

// Whether the grouped kernels run L2-blocked: sorted indices promised and more than one range.
bool use_split(const dsv_problem &p, const SplitPlan &pl) { return (p.flags & DSV_FLAG_SORTED_INDEX) && pl.S > 1; }

size_t kv_bytes(const dsv_problem &p) { return (size_t)p.L * 2 * p.d * esize(p.dtype); }  // K and V rows of a head
int64_t mean_k(const dsv_problem &p)
{
    int64_t s = 0;
    for (int h = 0; h < p.H; ++h) s += p.k_per_head[h];
    return s / p.H;
}

// Whether the dq step cuts sequences of less than eight full ranges in two or four instead of eight, given blocks enough
// (make_split_plan): every range leaves partial results, segment pointers and a row order, smaller ones stay in the L2 with the
// index that streams past them.  Measured, bf16, d = 128, four heads, eight ranges against four: L = 32768, k = 1092: 3373 : 3163 us;
// 24000, k = 800: 1893 : 1728; k = 2048 no gain.  The forward gains nothing and would share maxima (stage2_core.h); the key-major
// step loses: 32768, k = 327: 1680 : 1882, d = 64, 24000, k = 400: 800 : 1006.
bool few_ranges(const dsv_problem &p) { return mean_k(p) <= 1280; }

// Form of the forward and the dq step for the heads that keep fewer than dense_k keys: a lane group or a wave per row
// (stage2.hip), or key ranges (stage2_split.hip; sorted indices promised).  Their times, estimated in us, each a chain of
// steps -- as long as the longest row -- beside the work of the whole chip:
//   groups   0.1 to 0.3 us per key of a row; least work per pair, until the rows of all heads outgrow the caches
//   waves    a chain 4 to 16 times shorter; every part of a row in whole steps of four keys, the parts meet in exchanges (one
//            per accumulator and halving of the lanes), and no neighbour walks beside, so that a head's rows soon miss
//            the L2.  Chosen where it is 6 % (dq) or 10 % ahead.
//   ranges   seven launches, partial results of every (row, range); rows that stay in the L2
// Measured over 1008 problems (both types and head dimensions, 1 to 12 heads, 500 to 131072 keys, 8 to 5120 kept, lists as
// stage 1 makes them) the form chosen takes 1.012 times the fastest one's time in the mean; of 2016 calls it is more than 5 %
// behind ranges in 2, and behind groups, where only those and waves are open, in 21.  Groups, waves, ranges in us, bf16,
// d = 128: forward, four heads of 3000, k = 20: 12, 34, 56; of 4096, k = 640: 243, 213, 226; one of 8192, k = 320: 120, 78, 119;
// dq, four of 24000, k = 1280: 2656, 4271, 2640; fp32, four of 32768, k = 640: 5522, 7896, 3752.
enum class RowForm { groups, waves, ranges };
struct RowTime {
    RowForm form;
    double us;
};
RowTime row_time(const dsv_problem &p, const SplitPlan &pl, bool dq, int32_t dense_k)
{
    const double row_bytes = (double)p.d * esize(p.dtype), kv = (double)kv_bytes(p) / (1 << 20);
    const int lanes = (int)std::clamp(row_bytes / (dq ? 32 : 64), 4.0, 16.0), parts = 64 / lanes;  // SweepLanes (stage2_core.h)
    double sum = 0, most = 0, whole_steps = 0;
    int n = 0;
    for (int h = 0; h < p.H; ++h) {
        const int32_t k = p.k_per_head[h];
        if (k >= dense_k) continue;
        sum += k;
        most = std::max(most, (double)k);
        whole_steps += 4 * parts * std::ceil(k / (4.0 * parts));
        ++n;
    }
    if (!n) return {RowForm::groups, 0.0};  // nobody asks
    const double heads = (double)p.B * n, rows = heads * p.L, pair = 3.3e-8 * 2 * row_bytes * p.B * p.L;
    auto beside = [](double chain, double all) { return std::sqrt(chain * chain + all * all); };
    auto above = [](double x) { return std::max(0.0, std::log2(x)); };  // doublings past a size
    const double per_key = dq ? 0.19 : p.dtype == DSV_F32 ? 0.17 : p.d == 128 ? 0.31 : 0.1;
    const double groups = 7 + beside(per_key * most, pair * sum * (1.16 + 0.05 * above(kv / 8) + 0.45 * above(kv * std::sqrt(std::min(heads, 4.0)) / 32)));
    const double exchanges = (dq ? 2 * 4e-6 : 9e-6) * (p.d / lanes) * std::log2(parts);
    const double waves = (dq ? 1.06 : 1.1) * (7 + beside(0.008 * most, rows * exchanges + pair * whole_steps * (1 + (dq ? 0.3 : 0.45) * above(kv / 3))));
    const double ranges = 28 + (dq ? 4.4e-6 : 2.5e-6) * p.d * rows * std::max(pl.S_pad, 8) + beside(0.03 * most, pair * sum);
    if (use_split(p, pl) && ranges < std::min(groups, waves)) return {RowForm::ranges, ranges};
    return waves < groups ? RowTime{RowForm::waves, waves} : RowTime{RowForm::groups, groups};
}
RowForm row_form(const dsv_problem &p, const SplitPlan &pl, bool dq, int32_t dense_k) { return row_time(p, pl, dq, dense_k).form; }

// Whether the key-major step runs over query ranges.  Lists differ in length: the blocked form also sorts them by it, the other
// one gives every list a wave.  Blocked against not, us, lists as stage 1 makes them, bf16, d = 128: four heads of 2048 (1 MB),
// k = 160: 91 : 71, k = 640: 158 : 164; 4096, k = 160: 158 : 143, k = 320: 205 : 208; 6000 (3 MB), k = 200: 227 : 239; 12000 (6 MB),
// k = 80: 235 : 211, k = 160: 474 : 522; one head of 2048, k = 640: 85 : 52; d = 64, 12 of 4096 (1 MB), k = 1280: 817 : 994; one of 16384
// (4 MB), k = 160: 195 : 115; fp32, d = 128, four of 6000 (6 MB), k = 80: 186 : 173, k = 160: 259 : 329.
bool split_lists(const dsv_problem &p, const SplitPlan &pl)
{
    const double mb = (double)kv_bytes(p) / (1 << 20);
    return use_split(p, pl) && mb >= 1 && mb * p.B * p.H >= 2 && mb * mean_k(p) * std::sqrt(p.d / 128.0) >= 600;
}

// Whether a whole backward on rows in any order sorts them first, so that the dq step runs L2-blocked: once a head's K and
// V rows no longer share an XCD's 4 MB L2 with everything else.  Measured, bf16, d = 128, k = L / 12, the whole backward
// on rows in any order against ascending ones plus the sort: 4 heads of L = 4096: 450 : 416 + 25 us, 6144: 969 : 760 + 40,
// 8192: 1606 : 1239 + 60; L = 20280: the dq step 7.4 : 3.0 + 0.5 ms.
bool sort_rows_first(const dsv_problem &p)
{
    return !(p.flags & DSV_FLAG_SORTED_INDEX) && can_sort_rows(p) && (size_t)p.L * 2 * p.d * esize(p.dtype) > ((size_t)3 << 20);
}

// Smallest k whose heads run the forward over dense tiles with a mask (dense.hip), INT32_MAX if none should.  (The mask needs
// a workspace, which calls without the flag do not have.)
// Costs measured on bf16, in us.  Gathering: 18.5e-6 per pair at d = 128, 10.4e-6 at d = 64, once the chip is full.  Dense: per
// 64-key tile a round of blocks takes 2.0 (1.45) with at most one block of 128 queries per CU and 2.9 (2.5) when the CUs
// hold two (three), and a last round that is partly empty costs a fifth of a full one.  Estimated and measured, d = 128:
// 12 heads of 2048, 64 : 81; 4 of 4096, 128 : 131; 1 of 8192, 256 : 237; 12 of 8192, 631 : 685; 4 of 16384, 891 : 870; 4 of 32768,
// 3266 : 3402; gathering there with k = L / 16 and L / 30: 91, 56; 102, 59; 100, 72; 933, 526; 1355, 657; 4972, 2924.
// On sparse products, where few pairs are kept (dense_fwd_form in dense.hip), a round's time grows with the share of them, that of the fullest head where
// there are few rounds; a round that is hardly begun costs half of a full one, and one that gives CUs two blocks all of it.  Rounds of 512 blocks and
// their time in full ones of 2.4 us a tile, k = L / 20 or so: 1.00 : 1.04, 1.02 : 1.52, 1.50 : 1.74, 1.52 : 2.11, 1.98 : 2.15, 2.05 : 2.56, 2.89 : 3.03.  Where that
// estimate is the lower one, tiles pay earlier: four of 32768, k = L / 22: 2670, gathering 3610.  (A sixth off all rounds moved heads there that gather
// faster, dense : gathering, us: 24 of 5426, k = L / 26: 530 : 464; two of 33215, k = L / 24: 3144 : 2765.)  Over 1308 calls near the line, with one k or one per head, none
// is more than 2.4 % slower than with the line of dense products alone, and the mean is 11 % faster.  At d = 64 that line holds: gathers of short
// sequences cost less there than the rate above (24 of 5249, k = L / 21, dense : gathering: 307 : 273).
int32_t dense_fwd_min_k(const dsv_problem &p, bool sparse = true)
{
    if (!(p.flags & DSV_FLAG_SORTED_INDEX) || p.dtype != DSV_BF16 || p.L > kBitsMaxKeys || !(p.scale > 0.f)) return INT32_MAX;
    const bool wide = p.d == 128;
    const double pair = wide ? 18.5e-6 : 10.4e-6, light = wide ? 2.0 : 1.45, full = wide ? 2.9 : 2.5, slots = wide ? 512 : 768;
    std::vector<int32_t> ks(p.k_per_head, p.k_per_head + p.H);
    std::sort(ks.begin(), ks.end(), [](int32_t a, int32_t b) { return a > b; });
    int32_t best_k = INT32_MAX;
    double best = 0.0, gathered = 0.0, kept = 0.0;  // us saved by the heads with the largest k
    for (int m = 1; m <= p.H; ++m) {
        gathered += pair * (double)p.B * p.L * ks[m - 1];
        kept += ks[m - 1];
        if (m < p.H && ks[m] == ks[m - 1]) continue;
        const double blocks = (double)p.B * m * ((p.L + 127) / 128), tiles = (p.L + 63) / 64;
        double dense = 1.1 * tiles * (blocks <= 256 ? light : full * std::max(1.0, blocks / slots + 0.2));
        if (sparse && wide && blocks > 256 && kept * 14 <= (double)p.L * m) {  // on sparse products
            const double rounds = blocks / slots, whole = std::floor(rounds), part = rounds - whole;
            const double last = part > 0.5 ? 0.95 + 0.1 * part : part > 0.0 ? 0.5 + 0.5 * part : 0.0;
            const double mean = kept / ((double)p.L * m), share = mean + ((double)ks[0] / p.L - mean) / (0.5 + rounds);
            dense = std::min(dense, 1.05 * tiles * full * (0.74 + 2.9 * share) * std::max(1.0, whole + last));
        }
        if (gathered - dense > best) {
            best = gathered - dense;
            best_k = ks[m - 1];
        }
    }
    return best_k;
}

// Smallest k whose heads run a backward step over dense tiles with a mask (dense_bwd.hip), INT32_MAX if none should.  (As above, the
// mask needs a workspace.)
// Costs in us, bf16.  Gathering, per selected pair, once the chip is full: dq 18.9e-6 at d = 128, 10e-6 at d = 64; dkdv 21.3e-6, 11.3e-6.
// Dense, per pair of the square: a floor, and more where more pairs are kept (groups of four with a third one).  Whole backward
// by gathers against both steps dense: d = 128, three heads of 24000, one key in 24: 3461 : 3774, in 16: 4925 : 4442, in 12: 6199 : 4774,
// in 5: 13724 : 5904; the dkdv step alone, four heads of 6000, one in 16: 238 : 228, in 5: 592 : 283; d = 64, three heads of 24000,
// dq and dkdv, one in 16: 1279, 1239 : 1293, 1548; in 12: 1423, 1627 : 1332, 1663; in 8: 2055, 2407 : 1547, 1852; dq, d = 128, one in 16: one
// head of 65536 5429 : 4739, of 131072 21485 : 19027.
// 40 us are what launches, the mask and a chip that is not full cost small problems.
// The dq step's gathers of short sequences need no partial results, or where few keys are kept those of two or four ranges; dense tiles
// have those of eight to write and to merge (and with fewer ranges blocks that last as much longer, of which few rounds fill the chip
// badly).  Up to 3 MB of K and V rows per head the gathers' own estimate (row_time) decides therefore, unless it is that of eight ranges
// and more; above, rows soon miss the L2 without ranges, and that estimate is as far off as what there is to gain.  Gathers against dense,
// d = 128: 24 heads of 1500, k = 187: 150 : 231; 12 of 3000, k = 250: 185 : 271; 24 of 2048, k = 256: 248 : 341; 12 of 4096, k = 341: 332 : 429;
// but 4 of 2048, k = 512: 85 : 58; 2 of 3000, k = 750: 95 : 61; d = 64, 24 of 3000, k = 375: 292 : 345; 2 of 4096, k = 1024: 90 : 58.  Over 894
// dq steps of 30 us and more (both d, 1 to 24 heads of 1000 to 131072, 1/24 to 3/4 kept) the form chosen takes 1.004 times the faster
// one's time in the mean; dense is chosen where it is more than 5 % slower in 9 (most 14 %), gathers in 14.  Dkdv gathers cost short
// sequences more: of 1008 steps dense is chosen where it is 5 % slower in none, gathers in 241.
// pl, all: ranges of the dq step, and its form and time without dense tiles.
int32_t dense_bwd_min_k(const dsv_problem &p, bool keys, const SplitPlan &pl, const RowTime &all)
{
    // (the key-major tiles start from lse / scale, which has to be a number)
    if (!(p.flags & DSV_FLAG_SORTED_INDEX) || p.dtype != DSV_BF16 || p.L > kBitsMaxKeys || !(p.scale > 1e-30f)) return INT32_MAX;
    const bool wide = p.d == 128;
    const double pair = wide ? (keys ? 21.3e-6 : 18.9e-6) : keys ? 11.3e-6 : 10e-6;
    const double formed = wide ? (keys ? 1.2e-6 : 0.95e-6) : keys ? 0.8e-6 : 0.6e-6, more = wide ? 3e-6 : 2.2e-6;
    const bool flat = keys || (all.form == RowForm::ranges && pl.S_pad >= 8) || kv_bytes(p) > ((size_t)3 << 20);
    std::vector<int32_t> ks(p.k_per_head, p.k_per_head + p.H);
    std::sort(ks.begin(), ks.end(), [](int32_t a, int32_t b) { return a > b; });
    int32_t best_k = INT32_MAX;
    double best = 0.0, rows = 0.0, kept = 0.0;  // us saved by the heads with the largest k; their rows and selected pairs
    for (int m = 1; m <= p.H; ++m) {
        const int32_t k = ks[m - 1];
        rows += (double)p.B * p.L;
        kept += (double)p.B * p.L * k;
        if (m < p.H && ks[m] == k) continue;
        const double dense = formed * rows * p.L + more * kept;
        const double saved = flat ? pair * kept - dense - 40.0
                                  : all.us - row_time(p, pl, true, k).us - (20.0 + dense + 2.4e-6 * p.d * rows * std::max(pl.S_pad, 8));
        if (saved > best) {
            best = saved;
            best_k = k;
        }
    }
    return best_k;
}

// tabs cut in two: heads of at least min_k, and the others
void cut_tables(const std::vector<HeadTable> &tabs, int32_t min_k, std::vector<HeadTable> &yes, std::vector<HeadTable> &no)
{
    for (const HeadTable &t : tabs) {
        HeadTable a{}, b{};
        for (int s = 0; s < t.n; ++s) {
            HeadTable &d = t.k[s] >= min_k ? a : b;
            d.bh[d.n] = t.bh[s];
            d.k[d.n] = t.k[s];
            d.off[d.n++] = t.off[s];
        }
        if (a.n) yes.push_back(a);
        if (b.n) no.push_back(b);
    }
}

// Scratch for masks: all of them, at most 1 GB of bits (of one head 128 rows at least).
size_t mask_bytes(const dsv_problem &p, int heads)
{
    const size_t row = (size_t)bits_pitch(p.L) * 4, rows = std::min((size_t)p.B * heads * p.L, bits_rows(p.L, (size_t)1 << 30));
    return align_up(std::max(rows, (size_t)kDenseMinRows) * row, 256);
}

struct FwdLayout {
    RowForm form;     // of the heads below dense_k
    SplitPlan plan;
    int32_t dense_k;  // heads that keep at least so many keys run over dense tiles
    size_t seg, pm, pl, pacc, hist, order, total;
};

// sparse: whether sparse products count in the rule for heads over tiles with a mask, which needs scratch.
FwdLayout fwd_layout(const dsv_problem &p, bool sparse = true)
{
    FwdLayout w{};
    w.plan = make_split_plan(p, kFwdRangeBytes, false);  // every range brings a maximum of its own (stage2_core.h)
    w.dense_k = dense_fwd_min_k(p, sparse);
    w.form = row_form(p, w.plan, false, w.dense_k);
    int dense = 0;
    for (int h = 0; h < p.H; ++h) dense += p.k_per_head[h] >= w.dense_k;
    if (dense) w.total = mask_bytes(p, dense);
    // with room for the ranges of heads that run over tiles: what callers reserve does not hang on that rule
    if (w.form != RowForm::ranges && row_form(p, w.plan, false, INT32_MAX) != RowForm::ranges) return w;
    const size_t rows = (size_t)p.B * p.H * p.L;
    size_t o = 0;
    w.seg = o; o = align_up(o + rows * (w.plan.S + 1) * 4, 256);
    w.pm = o; o = align_up(o + rows * w.plan.S * 4, 256);
    w.pl = o; o = align_up(o + rows * w.plan.S * 4, 256);
    w.pacc = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
    w.hist = o; o = align_up(o + (size_t)p.B * p.H * w.plan.S * ((size_t)w.plan.range_len + 1) * 4, 256);
    w.order = o; o = align_up(o + rows * w.plan.S * 4, 256);
    w.total = std::max(w.total, o);  // the mask takes the place of the partial results
    return w;
}

// One split backward step (dq or dkdv): segment pointers and two [rows, S, d] partial arrays
// (+ [rows, S] for the dq step's Delta partials; laid out for both so that the steps can share it).
struct StepLayout {
    RowForm form;  // of the dq step
    bool blocked;  // the dkdv step
    SplitPlan plan;
    int32_t dense_k;  // heads that keep at least so many keys run over dense tiles
    size_t seg, pa, pb, pdelta, hist, order, rowstat, mask, mask_bytes, total;
};

void place_step(const dsv_problem &p, StepLayout &w)
{
    const size_t nbh = (size_t)p.B * p.H;
    const size_t rows = nbh * p.L;
    size_t o = 0;
    w.seg = o; o = align_up(o + rows * (w.plan.S + 1) * 4, 256);
    w.pa = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
    w.pb = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
    w.pdelta = o; o = align_up(o + rows * w.plan.S * 4, 256);
    w.hist = o; o = align_up(o + nbh * w.plan.S * ((size_t)w.plan.range_len + 1) * 4, 256);
    w.order = o; o = align_up(o + rows * w.plan.S * 4, 256);
    w.rowstat = o; o = align_up(o + rows * 8, 256);
    w.total = o;
}

// ... and room for the masks of heads that keep at least `least` keys.
void place_masks(const dsv_problem &p, int32_t least, StepLayout &w)
{
    int dense = 0;
    for (int h = 0; h < p.H; ++h) dense += p.k_per_head[h] >= least;
    const size_t row = (size_t)bits_pitch(p.L) * 4, all = (size_t)p.B * dense * p.L;
    w.mask = w.total;
    // whole where they are small beside the partial results; else pieces that fill the chip a few times and that the memory-side
    // cache holds from their making to their use
    const size_t most = bits_rows(p.L, (size_t)256 << 20), piece = bits_rows(p.L, (size_t)96 << 20);
    if (dense) w.mask_bytes = align_up((all <= most ? all : std::max(piece, (size_t)kDenseMinRows)) * row, 256);
    w.total += w.mask_bytes;
}

// Both steps.  Their scratch is never live together: either reserves `bytes`, what the larger one needs.
struct StepLayouts {
    StepLayout dq, dkdv;
    size_t bytes;
    bool spare;  // `bytes` are for dense tiles alone: by gathers the steps need none
};
StepLayouts step_layouts(const dsv_problem &p, bool dense = true)
{
    StepLayouts s{};
    s.dq.plan = make_split_plan(p, kBwdRangeBytes, few_ranges(p));
    s.dkdv.plan = make_split_plan(p, kBwdRangeBytes, false);
    const RowTime all = row_time(p, s.dq.plan, true, INT32_MAX);
    s.dq.dense_k = dense ? dense_bwd_min_k(p, false, s.dq.plan, all) : INT32_MAX;
    s.dkdv.dense_k = dense ? dense_bwd_min_k(p, true, s.dq.plan, all) : INT32_MAX;
    s.dq.form = s.dq.dense_k == INT32_MAX ? all.form : row_form(p, s.dq.plan, true, s.dq.dense_k);
    s.dkdv.blocked = split_lists(p, s.dkdv.plan);
    // masks: where some heads run over dense tiles in either step, so that both steps reserve the same
    const int32_t least = std::min(s.dq.dense_k, s.dkdv.dense_k);
    // with room for the ranges of heads that run over tiles, as the forward has it
    if (all.form == RowForm::ranges || s.dq.form == RowForm::ranges || s.dq.dense_k != INT32_MAX) {
        place_step(p, s.dq);
        place_masks(p, least, s.dq);
    }
    if (s.dkdv.blocked || s.dkdv.dense_k != INT32_MAX) {
        place_step(p, s.dkdv);
        place_masks(p, least, s.dkdv);
    }
    s.bytes = std::max(s.dq.total, s.dkdv.total);
    s.spare = all.form != RowForm::ranges && !s.dkdv.blocked;
    return s;
}
// ... of a call with this workspace: where gathers need none, one without that of dense tiles gathers.
StepLayouts step_layouts(const dsv_problem &p, const void *ws, size_t have)
{
    const StepLayouts s = step_layouts(p);
    return s.spare && check_workspace(ws, have, s.bytes) != DSV_OK ? step_layouts(p, false) : s;
}
size_t step_bytes(const dsv_problem &p) { return step_layouts(p).bytes; }

BwdSplitWorkspace step_buffers(char *ws, const StepLayout &w)
{
    BwdSplitWorkspace b;
    b.seg = reinterpret_cast<int32_t *>(ws + w.seg);
    b.pa = reinterpret_cast<float *>(ws + w.pa);
    b.pb = reinterpret_cast<float *>(ws + w.pb);
    b.pdelta = reinterpret_cast<float *>(ws + w.pdelta);
    b.hist = reinterpret_cast<int32_t *>(ws + w.hist);
    b.order = reinterpret_cast<int32_t *>(ws + w.order);
    b.rowstat = reinterpret_cast<float2 *>(ws + w.rowstat);
    return b;
}

// Whole backward.  own_transpose: the call builds the key-major index itself (dsv_sparse_attn_bwd);
// otherwise the caller brings it (dsv_sparse_attn_bwd_t).
struct BwdLayout {
    size_t delta, cnt, cnt_bytes, col, idxT, step, step_bytes, total;
    size_t least;  // of `total`, what a call cannot do without
};

BwdLayout bwd_layout(const dsv_problem &p, bool own_transpose)
{
    const size_t nbh = (size_t)p.B * p.H;
    const size_t tok = nbh * p.L;
    BwdLayout w{};
    size_t o = 0;
    w.delta = o; o = align_up(o + tok * 4, 256);
    if (own_transpose) {
        w.cnt = o; w.cnt_bytes = idx_transpose_bytes(p); o += w.cnt_bytes;
        w.col = o; o = align_up(o + nbh * ((size_t)p.L + 1) * 8, 256);
        w.idxT = o; o = align_up(o + total_pairs(p) * 4, 256);
    }
    // own_transpose: the lists come out ascending, so the dkdv step runs the L2-blocked kernel whatever p.flags says
    dsv_problem sorted = p;
    sorted.flags |= DSV_FLAG_SORTED_INDEX;
    const StepLayouts steps = step_layouts(own_transpose ? sorted : p);
    w.step = o; w.step_bytes = steps.bytes;
    o += w.step_bytes;
    w.total = o;
    w.least = steps.spare ? w.step : w.total;
    return w;
}

}  // namespace
}  // namespace dsv

using namespace dsv;

// ---- scratch of dsv_lowrank_topk_noalloc ---------------------------------------------------------
// A fixed array in the library's device image: every GPU that loads the library holds its own copy at
// its own address.  In host code the array's NAME is only a handle for hipGetSymbolAddress -- it is not
// a device address and is never passed to a kernel, a copy or a fill; the address is looked up once
// per device (with that device current) and kept here.
constexpr size_t kNoallocBytes = 32u << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's copy of `scratch`; nullptr (and *err set) on failure.
static void *noalloc_scratch(dsv_status *err)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { *err = DSV_EHIP; return nullptr; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { *err = DSV_EHIP; return nullptr; }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

extern "C" {

const char *dsv_version(void) { return "dsv 0.9 (gfx950)"; }

const char *dsv_status_string(dsv_status s)
{
    switch (s) {
    case DSV_OK: return "ok";
    case DSV_EINVAL: return "invalid argument";
    case DSV_EUNSUPPORTED: return "unsupported head dimension, rank or dtype";
    case DSV_EWORKSPACE: return "workspace missing, misaligned or too small";
    case DSV_EHIP: return "HIP runtime error";
    default: return "unknown status";
    }
}

dsv_status dsv_idx_offsets(const dsv_problem *p, int64_t *off)
{
    if (!p || !p->k_per_head || !off || p->B < 1 || p->H < 1 || p->L < 1) return DSV_EINVAL;
    for (int h = 0; h < p->H; ++h)
        if (p->k_per_head[h] < 1 || p->k_per_head[h] > p->L) return DSV_EINVAL;
    off[0] = 0;
    for (int bh = 0; bh < p->B * p->H; ++bh) off[bh + 1] = off[bh] + (int64_t)p->L * p->k_per_head[bh % p->H];
    return DSV_OK;
}

// ------------------------------------------------------------------------------------ stage 1
// grp == nullptr: every query is scored; else only the centre query of every group (idx, idx_t then hold
// one row per group and lists of groups).
static dsv_status lowrank_topk_impl(const dsv_problem *p, const dsv_grouping *grp, const void *Q, const void *K,
                                    const void *Wq, const void *Wk, int32_t *idx, int32_t *idx_t, int64_t *col_ptr,
                                    bool transposed, void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, true);
    if (st != DSV_OK) return st;
    if (grp && (st = check_grouping(*p, grp)) != DSV_OK) return st;
    if (!ok_ptrs({Q, K, Wq, Wk, idx})) return DSV_EINVAL;
    if (transposed && !ok_ptrs({idx_t, col_ptr})) return DSV_EINVAL;
    const int Lq = grp ? p->L / group_size(*grp) : p->L;
    const Stage1Layout w = stage1_layout(*p, transposed, grp ? Lq : 0);
    st = check_workspace(workspace, ws_bytes, w.total);
    if (st != DSV_OK) return st;
    char *ws = static_cast<char *>(workspace);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const void *Qsrc = Q;
    if (grp) {
        st = launch_group_rows(*p, *grp, 0, Q, ws + w.qc, stream);
        if (st != DSV_OK) return st;
        Qsrc = ws + w.qc;
    }
    st = launch_project(*p, Lq, Qsrc, K, Wq, Wk, ws + w.qlr, ws + w.klr, stream);
    if (st != DSV_OK) return st;
    SelectBuffers b;
    b.prefix = reinterpret_cast<uint32_t *>(ws + w.prefix);
    b.krem = reinterpret_cast<int32_t *>(ws + w.krem);
    b.win = reinterpret_cast<uint32_t *>(ws + w.win);
    b.todo = reinterpret_cast<int32_t *>(ws + w.todo);
    b.idx = idx;
    b.jcut = transposed ? reinterpret_cast<int32_t *>(ws + w.jcut) : nullptr;
    b.cnt = transposed ? reinterpret_cast<int32_t *>(ws + w.cnt) : nullptr;
    b.tile_flag = transposed ? reinterpret_cast<int32_t *>(ws + w.tflag) : nullptr;
    b.col = transposed ? col_ptr : nullptr;
    b.idx_t = transposed ? idx_t : nullptr;
    const std::vector<HeadTable> tabs = make_tables(*p, Lq);
    return launch_select(*p, Lq, tabs.data(), (int)tabs.size(), ws + w.qlr, ws + w.klr, b, stream);
}

size_t dsv_lowrank_topk_workspace(const dsv_problem *p)
{
    if (check_problem(p, true) != DSV_OK) return 0;
    return stage1_layout(*p, false).total;
}

dsv_status dsv_lowrank_topk(const dsv_problem *p, const void *Q, const void *K, const void *Wq, const void *Wk,
                            int32_t *idx, void *workspace, size_t ws_bytes, void *hip_stream)
{
    return lowrank_topk_impl(p, nullptr, Q, K, Wq, Wk, idx, nullptr, nullptr, false, workspace, ws_bytes, hip_stream);
}

size_t dsv_lowrank_topk_noalloc_max_bytes(void) { return kNoallocBytes; }

dsv_status dsv_lowrank_topk_noalloc(const dsv_problem *p, const void *Q, const void *K, const void *Wq, const void *Wk,
                                    int32_t *idx, void *hip_stream)
{
    // everything that can be refused is refused before the scratch is looked up
    dsv_status st = check_problem(p, true);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, Wq, Wk, idx})) return DSV_EINVAL;
    const size_t need = stage1_layout(*p, false).total;
    if (need > kNoallocBytes) return DSV_EWORKSPACE;
    void *ws = noalloc_scratch(&st);
    if (!ws) return st;
    // whatever a kernel of this call reads from the layout, a kernel of this call has written before (projections by
    // project_kernel, thresholds and tie budgets by the first radix pass or by the windowed search; the kernel for short
    // sequences writes the thresholds and neither writes nor reads the tie budgets), so what an earlier call left in the
    // array does not matter
    return lowrank_topk_impl(p, nullptr, Q, K, Wq, Wk, idx, nullptr, nullptr, false, ws, kNoallocBytes, hip_stream);
}

size_t dsv_lowrank_topk_t_workspace(const dsv_problem *p)
{
    if (check_problem(p, true) != DSV_OK) return 0;
    return stage1_layout(*p, true).total;
}

dsv_status dsv_lowrank_topk_t(const dsv_problem *p, const void *Q, const void *K, const void *Wq, const void *Wk,
                              int32_t *idx, int32_t *idx_t, int64_t *col_ptr, void *workspace, size_t ws_bytes,
                              void *hip_stream)
{
    return lowrank_topk_impl(p, nullptr, Q, K, Wq, Wk, idx, idx_t, col_ptr, true, workspace, ws_bytes, hip_stream);
}

// ------------------------------------------------------------------------------------ stage 2 forward
size_t dsv_sparse_attn_fwd_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return fwd_layout(*p).total;
}

dsv_status dsv_sparse_attn_fwd(const dsv_problem *p, const void *Q, const void *K, const void *V, const int32_t *idx,
                               void *O, float *lse, void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx, O, lse})) return DSV_EINVAL;
    FwdLayout w = fwd_layout(*p);
    // Heads that only sparse products bring to tiles gather where there is no room for their masks.
    if (check_workspace(workspace, ws_bytes, w.total) != DSV_OK) w = fwd_layout(*p, false);
    st = check_workspace(workspace, ws_bytes, w.total);
    if (st != DSV_OK) return st;
    const std::vector<HeadTable> tabs = make_tables(*p);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    std::vector<HeadTable> dense, rest;
    cut_tables(tabs, w.dense_k, dense, rest);
    std::optional<KernelSpan> span;
    if (!dense.empty()) span.emplace(DSV_KERNEL_FWD_SWEEP, stream);  // both parts together
    for (const HeadTable &t : dense) {
        st = launch_dense_fwd(*p, t, Q, K, V, idx, O, lse, ws, w.total, stream);
        if (st != DSV_OK) return st;
    }
    if (rest.empty()) return DSV_OK;
    if (w.form != RowForm::ranges)
        return launch_sparse_fwd(*p, rest.data(), (int)rest.size(), w.form == RowForm::waves, Q, K, V, idx, O, lse, stream);
    FwdSplitWorkspace b;
    b.seg = reinterpret_cast<int32_t *>(ws + w.seg);
    b.pm = reinterpret_cast<float *>(ws + w.pm);
    b.pl = reinterpret_cast<float *>(ws + w.pl);
    b.pacc = reinterpret_cast<float *>(ws + w.pacc);
    b.hist = reinterpret_cast<int32_t *>(ws + w.hist);
    b.order = reinterpret_cast<int32_t *>(ws + w.order);
    return launch_sparse_fwd_split(*p, rest.data(), (int)rest.size(), Q, K, V, idx, O, lse, w.plan, b, stream);
}

// ------------------------------------------------------------------------------------ stage 2 backward
size_t dsv_sparse_attn_bwd_dq_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return step_bytes(*p);
}

// dense_rows, dense_bits: as in DenseHeads.
static dsv_status bwd_dq_impl(const dsv_problem *p, const StepLayout &w, const void *Q, const void *K, const void *V, const int32_t *idx, const int32_t *dense_rows,
                              const uint32_t *dense_bits, const void *O, const float *lse, const void *dO, void *dQ, float *delta, void *workspace,
                              void *hip_stream)
{
    const std::vector<HeadTable> tabs = make_tables(*p);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    std::vector<HeadTable> dense, rest;
    cut_tables(tabs, w.dense_k, dense, rest);
    const DenseHeads dh{dense.data(), (int)dense.size(), ws + w.mask, w.mask_bytes, dense_rows, dense_bits};
    std::optional<KernelSpan> span;
    if (w.form != RowForm::ranges && !rest.empty()) {
        if (!dense.empty()) span.emplace(DSV_KERNEL_DQ_SWEEP, stream);  // both parts together
        const dsv_status st = launch_bwd_dq(*p, rest.data(), (int)rest.size(), w.form == RowForm::waves, Q, K, V, idx, O, lse, dO, dQ, delta, stream);
        if (st != DSV_OK || dense.empty()) return st;
        rest.clear();
    }
    return launch_bwd_dq_split(*p, rest.data(), (int)rest.size(), dh, Q, K, V, idx, O, lse, dO, dQ, delta, w.plan, step_buffers(ws, w), stream);
}

dsv_status dsv_sparse_attn_bwd_dq(const dsv_problem *p, const void *Q, const void *K, const void *V,
                                  const int32_t *idx, const void *O, const float *lse, const void *dO, void *dQ,
                                  float *delta, void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx, O, lse, dO, dQ, delta})) return DSV_EINVAL;
    const StepLayouts steps = step_layouts(*p, workspace, ws_bytes);
    st = check_workspace(workspace, ws_bytes, steps.bytes);
    if (st != DSV_OK) return st;
    return bwd_dq_impl(p, steps.dq, Q, K, V, idx, nullptr, nullptr, O, lse, dO, dQ, delta, workspace, hip_stream);
}

size_t dsv_idx_transpose_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return idx_transpose_bytes(*p);
}

dsv_status dsv_idx_transpose(const dsv_problem *p, const int32_t *idx, int32_t *idx_t, int64_t *col_ptr,
                             void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({idx, idx_t, col_ptr})) return DSV_EINVAL;
    const size_t need = dsv_idx_transpose_workspace(p);
    st = check_workspace(workspace, ws_bytes, need);
    if (st != DSV_OK) return st;
    const std::vector<HeadTable> tabs = make_tables(*p);
    return launch_idx_transpose(*p, tabs.data(), (int)tabs.size(), idx, false, idx_t, col_ptr,
                                workspace, need, static_cast<hipStream_t>(hip_stream));
}

size_t dsv_sparse_attn_bwd_dkdv_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return step_bytes(*p);
}

dsv_status dsv_sparse_attn_bwd_dkdv(const dsv_problem *p, const void *Q, const void *K, const void *V,
                                    const int32_t *idx_t, const int64_t *col_ptr, const float *lse, const float *delta,
                                    const void *dO, void *dK, void *dV, void *workspace, size_t ws_bytes,
                                    void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx_t, col_ptr, lse, delta, dO, dK, dV})) return DSV_EINVAL;
    const StepLayouts steps = step_layouts(*p, workspace, ws_bytes);
    st = check_workspace(workspace, ws_bytes, steps.bytes);
    if (st != DSV_OK) return st;
    const StepLayout &w = steps.dkdv;
    const std::vector<HeadTable> tabs = make_tables(*p);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *ws = static_cast<char *>(workspace);
    std::vector<HeadTable> dense, rest;
    cut_tables(tabs, w.dense_k, dense, rest);
    const DenseHeads dh{dense.data(), (int)dense.size(), ws + w.mask, w.mask_bytes};
    std::optional<KernelSpan> span;
    if (!w.blocked && !rest.empty()) {
        if (!dense.empty()) span.emplace(DSV_KERNEL_DKDV_SWEEP, stream);  // both parts together
        st = launch_bwd_dkdv(*p, rest.data(), (int)rest.size(), Q, K, V, idx_t, col_ptr, lse, delta, dO, dK, dV, stream);
        if (st != DSV_OK || dense.empty()) return st;
        rest.clear();
    }
    return launch_bwd_dkdv_split(*p, rest.data(), (int)rest.size(), dh, Q, K, V, idx_t, col_ptr, lse, delta, dO, dK, dV, w.plan, step_buffers(ws, w),
                                 stream);
}

size_t dsv_sparse_attn_bwd_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return bwd_layout(*p, true).total;
}

dsv_status dsv_sparse_attn_bwd(const dsv_problem *p, const void *Q, const void *K, const void *V, const int32_t *idx,
                               const void *O, const float *lse, const void *dO, void *dQ, void *dK, void *dV,
                               void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx, O, lse, dO, dQ, dK, dV})) return DSV_EINVAL;
    const BwdLayout w = bwd_layout(*p, true);
    st = check_workspace(workspace, ws_bytes, w.least);
    if (st != DSV_OK) return st;
    const size_t step_have = std::min(w.step_bytes, ws_bytes - w.step);
    char *ws = static_cast<char *>(workspace);
    float *delta = reinterpret_cast<float *>(ws + w.delta);
    int64_t *col = reinterpret_cast<int64_t *>(ws + w.col);
    int32_t *idx_t = reinterpret_cast<int32_t *>(ws + w.idxT);
    // the lists built here are ascending in the query index whatever the order inside the rows of idx is: the dkdv
    // step may run the L2-blocked kernel
    dsv_problem sorted = *p;
    sorted.flags |= DSV_FLAG_SORTED_INDEX;
    const std::vector<HeadTable> tabs = make_tables(*p);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint32_t *bits = nullptr;
    if (sort_rows_first(*p)) {
        // rows in any order: an ascending copy (in the place of the lists, which are built after the dq step) lets the
        // dq step run L2-blocked too; its bitmaps serve the transposition
        // (heads over dense tiles take their rows as they are, through their bitmaps: 20280, keeping 2028 and 4056 keys, the whole
        // backward beside two sparser heads 5220 -> 4809 us)
        bits = transpose_matrix(*p, ws + w.cnt);
        std::vector<HeadTable> dense, rest;
        const StepLayout step = step_layouts(sorted, ws + w.step, step_have).dq;
        cut_tables(tabs, step.dense_k, dense, rest);
        uint32_t *rest_bits = bits;
        if (bits && !dense.empty()) {  // one table, its first heads
            st = launch_bits_build(*p, dense[0], 0, dense[0].n, idx, 0, p->L, bits, stream);
            if (st != DSV_OK) return st;
            rest_bits += (size_t)dense[0].n * p->L * bits_pitch(p->L);
        }
        st = launch_sort_rows(*p, rest.data(), (int)rest.size(), idx, idx_t, rest_bits, stream);
        if (st != DSV_OK) return st;
        st = bwd_dq_impl(&sorted, step, Q, K, V, idx_t, idx, bits, O, lse, dO, dQ, delta, ws + w.step, hip_stream);
    } else {
        st = dsv_sparse_attn_bwd_dq(p, Q, K, V, idx, O, lse, dO, dQ, delta, ws + w.step, step_have, hip_stream);
    }
    if (st != DSV_OK) return st;
    st = launch_idx_transpose(*p, tabs.data(), (int)tabs.size(), idx, bits != nullptr, idx_t, col, ws + w.cnt, w.cnt_bytes, stream);
    if (st != DSV_OK) return st;
    return dsv_sparse_attn_bwd_dkdv(&sorted, Q, K, V, idx_t, col, lse, delta, dO, dK, dV, ws + w.step, step_have, hip_stream);
}

size_t dsv_sparse_attn_bwd_t_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return bwd_layout(*p, false).total;
}

dsv_status dsv_sparse_attn_bwd_t(const dsv_problem *p, const void *Q, const void *K, const void *V,
                                 const int32_t *idx, const int32_t *idx_t, const int64_t *col_ptr, const void *O,
                                 const float *lse, const void *dO, void *dQ, void *dK, void *dV, void *workspace,
                                 size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({O, dQ, dK, dV, idx_t, col_ptr})) return DSV_EINVAL;
    const BwdLayout w = bwd_layout(*p, false);
    st = check_workspace(workspace, ws_bytes, w.least);
    if (st != DSV_OK) return st;
    char *ws = static_cast<char *>(workspace);
    const size_t step_have = std::min(w.step_bytes, ws_bytes - w.step);
    float *delta = reinterpret_cast<float *>(ws + w.delta);
    st = dsv_sparse_attn_bwd_dq(p, Q, K, V, idx, O, lse, dO, dQ, delta, ws + w.step, step_have, hip_stream);
    if (st != DSV_OK) return st;
    return dsv_sparse_attn_bwd_dkdv(p, Q, K, V, idx_t, col_ptr, lse, delta, dO, dK, dV, ws + w.step, step_have,
                                    hip_stream);
}

// ------------------------------------------------------------------------------------ query grouping
size_t dsv_lowrank_topk_grouped_workspace(const dsv_problem *p, const dsv_grouping *g)
{
    if (check_problem(p, true) != DSV_OK || check_grouping(*p, g) != DSV_OK) return 0;
    return stage1_layout(*p, true, p->L / group_size(*g)).total;
}

dsv_status dsv_lowrank_topk_grouped(const dsv_problem *p, const dsv_grouping *g, const void *Q, const void *K,
                                    const void *Wq, const void *Wk, int32_t *idx_g, int32_t *idx_t_g, int64_t *col_ptr,
                                    void *workspace, size_t ws_bytes, void *hip_stream)
{
    if (!g) return DSV_EINVAL;
    if ((idx_t_g == nullptr) != (col_ptr == nullptr)) return DSV_EINVAL;
    return lowrank_topk_impl(p, g, Q, K, Wq, Wk, idx_g, idx_t_g, col_ptr, idx_t_g != nullptr, workspace, ws_bytes,
                             hip_stream);
}

namespace {
// Scratch of one L2-blocked grouped kernel (forward or dq): segment pointers per group row and per-(token row,
// range) partials.  split == false: the plain kernels (rows in any order, or a single range), no scratch.
struct GroupedStepLayout {
    bool split;
    SplitPlan plan;
    size_t seg, pa, pb, pc, total;
};
GroupedStepLayout grouped_step_layout(const dsv_problem &p, const dsv_grouping &g, bool dq)
{
    GroupedStepLayout w{};
    // few: a group's partial results are its members' (four heads of 32768, k = 2048, 2 x 2 x 2, the layer: 8058 -> 7612 us)
    w.plan = make_split_plan(p, kBwdRangeBytes, true);
    w.split = use_split(p, w.plan);
    if (!w.split) return w;
    const size_t nbh = (size_t)p.B * p.H, rows = nbh * p.L, Lq = p.L / group_size(g);
    size_t o = 0;
    w.seg = o; o = align_up(o + nbh * Lq * (w.plan.S + 1) * 4, 256);
    if (dq) {
        w.pa = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
        w.pb = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
        w.pc = o; o = align_up(o + rows * w.plan.S * 4, 256);
    } else {
        w.pa = o; o = align_up(o + rows * w.plan.S * 4, 256);
        w.pb = o; o = align_up(o + rows * w.plan.S * 4, 256);
        w.pc = o; o = align_up(o + rows * w.plan.S * p.d * 4, 256);
    }
    w.total = o;
    return w;
}
GroupedSplit grouped_split(char *ws, const GroupedStepLayout &w)
{
    GroupedSplit s;
    s.plan = w.plan;
    s.seg = reinterpret_cast<int32_t *>(ws + w.seg);
    s.pa = reinterpret_cast<float *>(ws + w.pa);
    s.pb = reinterpret_cast<float *>(ws + w.pb);
    s.pc = reinterpret_cast<float *>(ws + w.pc);
    return s;
}

// The group kernels proper exist for bf16, d = 128 and groups of at most 32 queries.  Every other case (fp32, d = 64,
// larger cubes) runs the per-query kernels on the queries reordered group by group, with the group index expanded to
// one row per query: the same results, without the saving.
bool grouped_native(const dsv_problem &p, const dsv_grouping &g)
{
    return p.dtype == DSV_BF16 && p.d == 128 && group_size(g) <= 32 && (uint64_t)p.L * (uint64_t)group_size(g) < (1ull << 32);
}

struct GroupedFwdGeneral {
    size_t qp, op, lsep, idxx, step, step_bytes, total;
};
GroupedFwdGeneral grouped_fwd_general(const dsv_problem &p)
{
    const size_t nbh = (size_t)p.B * p.H;
    const size_t rows = nbh * p.L * p.d * esize(p.dtype);
    GroupedFwdGeneral w{};
    size_t o = 0;
    w.qp = o; o = align_up(o + rows, 256);
    w.op = o; o = align_up(o + rows, 256);
    w.lsep = o; o = align_up(o + nbh * p.L * 4, 256);
    w.idxx = o; o = align_up(o + total_pairs(p) * 4, 256);
    w.step = o; w.step_bytes = fwd_layout(p).total; o += w.step_bytes;
    w.total = o;
    return w;
}

// The key-major step of the group kernels' cases: by unions or by the per-query sweep on the lists of groups, as the device
// finds (launch_union_prepare), both with the same ranges of queries -- one where 8192 rows hold them all.
struct GroupedKeyLayout {
    StepLayout step;
    size_t use, total;
};
GroupedKeyLayout grouped_key_layout(const dsv_problem &p)
{
    GroupedKeyLayout w{};
    w.step.plan = make_split_plan(p, kBwdRangeBytes, true);
    if ((size_t)p.L <= kMaxRangeRows && row_blocks(p) >= kFewRangesBlocks) {
        w.step.plan.S = w.step.plan.S_pad = 1;
        w.step.plan.range_len = p.L;
    }
    place_step(p, w.step);
    w.use = w.step.total;
    w.total = align_up(w.use + (size_t)p.B * p.H * 4, 256);
    return w;
}

struct GroupedBwdLayout {
    size_t delta, qp, gop, lsep, deltap, idxtx, colx, op, dqp, idxx, step, step_bytes, total;
};
GroupedBwdLayout grouped_bwd_layout(const dsv_problem &p, const dsv_grouping &g)
{
    const size_t nbh = (size_t)p.B * p.H;
    const size_t rows = nbh * p.L * p.d * esize(p.dtype);
    const bool native = grouped_native(p, g);
    dsv_problem sorted = p;
    sorted.flags |= DSV_FLAG_SORTED_INDEX;
    GroupedBwdLayout w{};
    size_t o = 0;
    w.delta = o; o = align_up(o + nbh * p.L * 4, 256);
    w.qp = o; o = align_up(o + rows, 256);
    w.gop = o; o = align_up(o + rows, 256);
    w.lsep = o; o = align_up(o + nbh * p.L * 4, 256);
    w.deltap = o; o = align_up(o + nbh * p.L * 4, 256);
    if (!native) {   // the per-query steps on reordered queries: O and dQ in that order, one index row and list entry per query
        w.idxtx = o; o = align_up(o + total_pairs(p) * 4, 256);
        w.colx = o; o = align_up(o + nbh * ((size_t)p.L + 1) * 8, 256);
        w.op = o; o = align_up(o + rows, 256);
        w.dqp = o; o = align_up(o + rows, 256);
        w.idxx = o; o = align_up(o + total_pairs(p) * 4, 256);
    }
    // the dq step's scratch and the dkdv step's are never live together
    w.step = o;
    w.step_bytes = native ? std::max(grouped_step_layout(p, g, true).total, grouped_key_layout(p).total)
                          : std::max(step_bytes(p), step_bytes(sorted));
    o += w.step_bytes;
    w.total = o;
    return w;
}
}  // namespace

size_t dsv_sparse_attn_fwd_grouped_workspace(const dsv_problem *p, const dsv_grouping *g)
{
    if (check_problem(p, false) != DSV_OK || check_grouping(*p, g) != DSV_OK) return 0;
    return grouped_native(*p, *g) ? grouped_step_layout(*p, *g, false).total : grouped_fwd_general(*p).total;
}

dsv_status dsv_sparse_attn_fwd_grouped(const dsv_problem *p, const dsv_grouping *g, const void *Q, const void *K,
                                       const void *V, const int32_t *idx_g, void *O, float *lse, void *workspace,
                                       size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if ((st = check_grouping(*p, g)) != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx_g, O, lse})) return DSV_EINVAL;
    if (!grouped_native(*p, *g)) {
        const GroupedFwdGeneral w = grouped_fwd_general(*p);
        st = check_workspace(workspace, ws_bytes, w.total);
        if (st != DSV_OK) return st;
        char *ws = static_cast<char *>(workspace);
        hipStream_t stream = static_cast<hipStream_t>(hip_stream);
        const std::vector<HeadTable> tabs = make_tables(*p, p->L / group_size(*g));
        int32_t *idx_x = reinterpret_cast<int32_t *>(ws + w.idxx);
        float *lsep = reinterpret_cast<float *>(ws + w.lsep);
        if ((st = launch_group_rows(*p, *g, 1, Q, ws + w.qp, stream)) != DSV_OK) return st;
        st = launch_group_expand(*p, *g, tabs.data(), (int)tabs.size(), idx_g, nullptr, nullptr, idx_x, nullptr, nullptr, stream);
        if (st != DSV_OK) return st;
        st = dsv_sparse_attn_fwd(p, ws + w.qp, K, V, idx_x, ws + w.op, lsep, w.step_bytes ? ws + w.step : nullptr, w.step_bytes,
                                 hip_stream);
        if (st != DSV_OK) return st;
        if ((st = launch_group_rows(*p, *g, 2, ws + w.op, O, stream)) != DSV_OK) return st;
        return launch_group_scalar(*p, *g, lsep, lse, stream, true);
    }
    const GroupedStepLayout w = grouped_step_layout(*p, *g, false);
    st = check_workspace(workspace, ws_bytes, w.total);
    if (st != DSV_OK) return st;
    const std::vector<HeadTable> tabs = make_tables(*p, p->L / group_size(*g));
    GroupedSplit sp;
    if (w.split) sp = grouped_split(static_cast<char *>(workspace), w);
    return launch_grouped_fwd(*p, *g, tabs.data(), (int)tabs.size(), Q, K, V, idx_g, O, lse, w.split ? &sp : nullptr,
                              static_cast<hipStream_t>(hip_stream));
}

size_t dsv_sparse_attn_bwd_grouped_workspace(const dsv_problem *p, const dsv_grouping *g)
{
    if (check_problem(p, false) != DSV_OK || check_grouping(*p, g) != DSV_OK) return 0;
    return grouped_bwd_layout(*p, *g).total;
}

dsv_status dsv_sparse_attn_bwd_grouped(const dsv_problem *p, const dsv_grouping *g, const void *Q, const void *K,
                                       const void *V, const int32_t *idx_g, const int32_t *idx_t_g,
                                       const int64_t *col_ptr, const void *O, const float *lse, const void *dO, void *dQ,
                                       void *dK, void *dV, void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if ((st = check_grouping(*p, g)) != DSV_OK) return st;
    if (!ok_ptrs({Q, K, V, idx_g, idx_t_g, col_ptr, O, lse, dO, dQ, dK, dV})) return DSV_EINVAL;
    const bool native = grouped_native(*p, *g);
    const GroupedBwdLayout w = grouped_bwd_layout(*p, *g);
    st = check_workspace(workspace, ws_bytes, w.total);
    if (st != DSV_OK) return st;
    char *ws = static_cast<char *>(workspace);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const std::vector<HeadTable> tabs = make_tables(*p, p->L / group_size(*g));
    float *delta = reinterpret_cast<float *>(ws + w.delta);
    float *lsep = reinterpret_cast<float *>(ws + w.lsep), *deltap = reinterpret_cast<float *>(ws + w.deltap);
    // queries reordered group by group: a group's members become neighbours, and the per-query lists that the lists of
    // groups stand for come out ascending
    if ((st = launch_group_rows(*p, *g, 1, Q, ws + w.qp, stream)) != DSV_OK) return st;
    if ((st = launch_group_rows(*p, *g, 1, dO, ws + w.gop, stream)) != DSV_OK) return st;
    if ((st = launch_group_scalar(*p, *g, lse, lsep, stream)) != DSV_OK) return st;
    if (native) {
        // dQ step, group by group (K and V rows gathered once per group)
        const GroupedStepLayout dqw = grouped_step_layout(*p, *g, true);
        GroupedSplit sp;
        if (dqw.split) sp = grouped_split(ws + w.step, dqw);
        st = launch_grouped_dq(*p, *g, tabs.data(), (int)tabs.size(), Q, K, V, idx_g, O, lse, dO, dQ, delta,
                               dqw.split ? &sp : nullptr, stream);
        if (st != DSV_OK) return st;
        if ((st = launch_group_scalar(*p, *g, delta, deltap, stream)) != DSV_OK) return st;
    } else {
        // dQ step by the per-query kernel on the reordered queries, one (expanded) index row per query
        int32_t *idx_x = reinterpret_cast<int32_t *>(ws + w.idxx);
        if ((st = launch_group_rows(*p, *g, 1, O, ws + w.op, stream)) != DSV_OK) return st;
        st = launch_group_expand(*p, *g, tabs.data(), (int)tabs.size(), idx_g, nullptr, nullptr, idx_x, nullptr, nullptr, stream);
        if (st != DSV_OK) return st;
        const size_t dq_bytes = step_bytes(*p);
        st = dsv_sparse_attn_bwd_dq(p, ws + w.qp, K, V, idx_x, ws + w.op, lsep, ws + w.gop, ws + w.dqp, deltap,
                                    dq_bytes ? ws + w.step : nullptr, dq_bytes, hip_stream);
        if (st != DSV_OK) return st;
        if ((st = launch_group_rows(*p, *g, 2, ws + w.dqp, dQ, stream)) != DSV_OK) return st;
    }
    if (native) {
        const int G = group_size(*g);
        const GroupedKeyLayout kw = grouped_key_layout(*p);
        const BwdSplitWorkspace b = step_buffers(ws + w.step, kw.step);
        const bool always = union_limit(*p) >= 16;
        int32_t *use = always ? nullptr : reinterpret_cast<int32_t *>(ws + w.step + kw.use);
        KernelSpan span(DSV_KERNEL_DKDV_SWEEP, stream);  // both forms together
        st = launch_union_prepare(*p, G, tabs.data(), (int)tabs.size(), idx_t_g, col_ptr, lsep, deltap, b.rowstat, use, stream);
        if (st != DSV_OK) return st;
        st = launch_grouped_dkdv(*p, G, tabs.data(), (int)tabs.size(), ws + w.qp, K, V, idx_t_g, col_ptr, ws + w.gop, dK, dV, kw.step.plan, b,
                                 use, stream);
        if (st != DSV_OK) return st;
        if (always) return kw.step.plan.S > 1 ? launch_dkdv_merge_bf16_128(*p, tabs.data(), (int)tabs.size(), dK, dV, kw.step.plan, b, stream) : DSV_OK;
        return launch_bwd_dkdv_split(*p, tabs.data(), (int)tabs.size(), DenseHeads{}, ws + w.qp, K, V, idx_t_g, col_ptr, lsep, deltap, ws + w.gop, dK, dV,
                                     kw.step.plan, b, stream, G, use);
    }
    // dK, dV step: the per-query key-major sweep on the reordered queries
    st = launch_group_expand(*p, *g, tabs.data(), (int)tabs.size(), idx_g, idx_t_g, col_ptr, nullptr,
                             reinterpret_cast<int32_t *>(ws + w.idxtx), reinterpret_cast<int64_t *>(ws + w.colx), stream);
    if (st != DSV_OK) return st;
    dsv_problem sorted = *p;
    sorted.flags |= DSV_FLAG_SORTED_INDEX;
    const size_t dkdv_bytes = step_bytes(sorted);
    return dsv_sparse_attn_bwd_dkdv(&sorted, ws + w.qp, K, V, reinterpret_cast<int32_t *>(ws + w.idxtx),
                                    reinterpret_cast<int64_t *>(ws + w.colx), lsep, deltap, ws + w.gop, dK, dV,
                                    dkdv_bytes ? ws + w.step : nullptr, dkdv_bytes, hip_stream);
}

// ------------------------------------------------------------------------------------ group-size profiling
size_t dsv_group_overlap_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return align_up((size_t)p->B * p->H * 8, 256);
}

dsv_status dsv_group_overlap(const dsv_problem *p, const dsv_grouping *g, const int32_t *idx, float *overlap,
                             void *workspace, size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if ((st = check_grouping(*p, g)) != DSV_OK) return st;
    if (!ok_ptrs({idx, overlap})) return DSV_EINVAL;
    st = check_workspace(workspace, ws_bytes, dsv_group_overlap_workspace(p));
    if (st != DSV_OK) return st;
    const std::vector<HeadTable> tabs = make_tables(*p);
    return launch_group_overlap(*p, *g, tabs.data(), (int)tabs.size(), idx, static_cast<unsigned long long *>(workspace),
                                overlap, static_cast<hipStream_t>(hip_stream));
}

size_t dsv_choose_grouping_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return dsv_group_overlap_workspace(p) + align_up((size_t)p->B * p->H * 4, 256);
}

dsv_status dsv_choose_grouping(const dsv_problem *p, int32_t F, int32_t Hh, int32_t Ww, const int32_t *cubes, int32_t n,
                               const int32_t *idx, float min_overlap, int32_t *chosen, float *overlaps, void *workspace,
                               size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!cubes || !chosen || n < 1 || !ok_ptrs({idx})) return DSV_EINVAL;
    st = check_workspace(workspace, ws_bytes, dsv_choose_grouping_workspace(p));
    if (st != DSV_OK) return st;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int nbh = p->B * p->H;
    float *dev = reinterpret_cast<float *>(static_cast<char *>(workspace) + dsv_group_overlap_workspace(p));
    std::vector<float> host(nbh);
    int best = -1, best_members = 0;
    for (int c = 0; c < n; ++c) {
        const dsv_grouping g{F, Hh, Ww, cubes[3 * c], cubes[3 * c + 1], cubes[3 * c + 2]};
        const dsv_status ok = check_grouping(*p, &g);
        if (ok != DSV_OK) {   // does not tile the grid (or is too large): not a candidate
            if (overlaps) for (int e = 0; e < nbh; ++e) overlaps[(size_t)c * nbh + e] = -1.f;
            continue;
        }
        st = dsv_group_overlap(p, &g, idx, dev, workspace, dsv_group_overlap_workspace(p), hip_stream);
        if (st != DSV_OK) return st;
        DSV_HIP_CHECK(hipMemcpyAsync(host.data(), dev, (size_t)nbh * 4, hipMemcpyDeviceToHost, stream));
        DSV_HIP_CHECK(hipStreamSynchronize(stream));
        bool all = true;
        for (int e = 0; e < nbh; ++e) {
            if (overlaps) overlaps[(size_t)c * nbh + e] = host[e];
            all = all && host[e] >= min_overlap;
        }
        if (all && group_size(g) > best_members) { best = c; best_members = group_size(g); }
    }
    *chosen = best;
    return DSV_OK;
}

// ------------------------------------------------------------------------------------ predictor side
size_t dsv_predictor_loss_workspace(const dsv_problem *p, int32_t n_rows)
{
    if (check_problem(p, true) != DSV_OK || n_rows < 1 || n_rows > p->L) return 0;
    return predictor_layout(*p, n_rows).total;
}

dsv_status dsv_predictor_loss(const dsv_problem *p, const void *Q, const void *K, const void *Wq, const void *Wk,
                              const int32_t *rows, int32_t n_rows, float *loss, float *dWq, float *dWk, void *workspace,
                              size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, true);
    if (st != DSV_OK) return st;
    if (n_rows < 1 || n_rows > p->L) return DSV_EINVAL;
    if (!ok_ptrs({Q, K, Wq, Wk, loss, dWq, dWk}) || !rows) return DSV_EINVAL;
    const PredictorLayout w = predictor_layout(*p, n_rows);
    st = check_workspace(workspace, ws_bytes, w.total);
    if (st != DSV_OK) return st;
    return launch_predictor_loss(*p, Q, K, Wq, Wk, rows, n_rows, loss, dWq, dWk, static_cast<char *>(workspace), w,
                                 static_cast<hipStream_t>(hip_stream));
}

size_t dsv_profile_sparsity_workspace(const dsv_problem *p, int32_t n_rows)
{
    (void)p;
    (void)n_rows;
    return 0;
}

dsv_status dsv_profile_sparsity(const dsv_problem *p, const void *Q, const void *K, const int32_t *rows, int32_t n_rows,
                                float mass, int32_t *counts, float *sparsity, float *ema, float alpha, void *workspace,
                                size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (n_rows < 1 || n_rows > p->L || !(mass > 0.f && mass < 1.f) || !(alpha >= 0.f && alpha <= 1.f)) return DSV_EINVAL;
    if (!ok_ptrs({Q, K}) || !rows || !counts || !sparsity) return DSV_EINVAL;
    (void)workspace;
    (void)ws_bytes;
    return launch_profile_sparsity(*p, Q, K, rows, n_rows, mass, counts, sparsity, ema, alpha, static_cast<hipStream_t>(hip_stream));
}

// ------------------------------------------------------------------------------------ debug validator
size_t dsv_idx_validate_workspace(const dsv_problem *p)
{
    if (check_problem(p, false) != DSV_OK) return 0;
    return 256;
}

dsv_status dsv_idx_validate(const dsv_problem *p, const int32_t *idx, int64_t *report, void *workspace,
                            size_t ws_bytes, void *hip_stream)
{
    dsv_status st = check_problem(p, false);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({idx})) return DSV_EINVAL;
    st = check_workspace(workspace, ws_bytes, 256);
    if (st != DSV_OK) return st;
    const std::vector<HeadTable> tabs = make_tables(*p);
    return launch_idx_validate(*p, tabs.data(), (int)tabs.size(), idx, static_cast<unsigned long long *>(workspace),
                               report, static_cast<hipStream_t>(hip_stream));
}

// ------------------------------------------------------------------------------------ parity exports
dsv_status dsv_lowrank_project(const dsv_problem *p, const void *Q, const void *K, const void *Wq, const void *Wk,
                               void *Qlr, void *Klr, void *hip_stream)
{
    dsv_status st = check_problem(p, true);
    if (st != DSV_OK) return st;
    if (!ok_ptrs({Q, K, Wq, Wk, Qlr, Klr})) return DSV_EINVAL;
    return launch_project(*p, p->L, Q, K, Wq, Wk, Qlr, Klr, static_cast<hipStream_t>(hip_stream));
}

dsv_status dsv_lowrank_scores_rows(const dsv_problem *p, const void *Qlr, const void *Klr, int32_t b, int32_t h,
                                   const int32_t *rows, int32_t n_rows, float *scores, void *hip_stream)
{
    dsv_status st = check_problem(p, true);
    if (st != DSV_OK) return st;
    if (!rows || !scores || n_rows < 1) return DSV_EINVAL;
    if (b < 0 || b >= p->B || h < 0 || h >= p->H) return DSV_EINVAL;
    if (!ok_ptrs({Qlr, Klr})) return DSV_EINVAL;
    return launch_scores_rows(*p, Qlr, Klr, b * p->H + h, rows, n_rows, scores, static_cast<hipStream_t>(hip_stream));
}

// ------------------------------------------------------------------------------------ measurement aid
dsv_status dsv_kernel_timing(int32_t enable)
{
    dsv::KernelTimer &t = dsv::g_kernel_timer;
    if (enable && !t.ev[0][0]) {
        for (int i = 0; i < DSV_KERNEL_COUNT; ++i)
            for (int e = 0; e < 2; ++e)
                if (hipEventCreate(&t.ev[i][e]) != hipSuccess) return DSV_EHIP;
    }
    for (int i = 0; i < DSV_KERNEL_COUNT; ++i) t.recorded[i] = false;
    t.on = enable != 0;
    return DSV_OK;
}

int32_t dsv_threshold_search(int32_t mode)
{
    if (mode < 0 || mode > 2) return -1;
    return dsv::set_threshold_search(mode);
}

int32_t dsv_threshold_sample_keys(int32_t L, int32_t k)
{
    const int mode = dsv::set_threshold_search(-1);
    return mode == 1 ? 0 : dsv::window_sample_keys(L, k, mode == 2);
}

int32_t dsv_dense_min_k(const dsv_problem *p, int32_t step)
{
    if (step < DSV_KERNEL_FWD_SWEEP || step > DSV_KERNEL_DKDV_SWEEP || check_problem(p, false) != DSV_OK) return 0;
    const int32_t k = step == DSV_KERNEL_FWD_SWEEP ? fwd_layout(*p).dense_k : step == DSV_KERNEL_DQ_SWEEP ? step_layouts(*p).dq.dense_k : step_layouts(*p).dkdv.dense_k;
    return k == INT32_MAX ? 0 : k;
}

dsv_status dsv_kernel_ms(int32_t span, float *ms)
{
    dsv::KernelTimer &t = dsv::g_kernel_timer;
    if (!ms || span < 0 || span >= DSV_KERNEL_COUNT || !t.recorded[span]) return DSV_EINVAL;
    if (hipEventSynchronize(t.ev[span][1]) != hipSuccess) return DSV_EHIP;
    if (hipEventElapsedTime(ms, t.ev[span][0], t.ev[span][1]) != hipSuccess) return DSV_EHIP;
    return DSV_OK;
}

}  // extern "C"
