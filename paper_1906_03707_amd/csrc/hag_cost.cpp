// What a pass over the HAG and a pass over the plain lists are expected to cost: the two aggregate the same, and the faster one is taken.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "hag_internal.hpp"

namespace hag {

// Misses are those of one XCD's L2 under the plan's own order, a first-in first-out cache of this many bytes (of the 4 MB, some holds ids and
// results): misses per row read, from a run of at most kSampleReads reads at the start of the plan and one in its middle (in a batch of small graphs
// every stretch is like any other: shorter runs).
constexpr double kCacheBytes = 3e6;
constexpr int64_t kSampleReads = 1 << 20, kSampleReadsBatch = 1 << 14;

static double miss_rate(const Plan &p, const std::vector<int32_t> &col, int64_t n_ids, int lpr, int64_t n_long, double plan_reads, int64_t sample) {
    const int64_t cap = (int64_t)(kCacheBytes / (16 * lpr)), n_all = p.part_begin[1];
    if (n_ids <= cap) return std::min(1., (double)n_ids / std::max(1., plan_reads / kPartitions));   // every row once
    std::vector<int32_t> seen((size_t)n_ids, INT32_MIN);
    // one XCD's items: all of partition 0, or every 8th workgroup's
    const int64_t per = kBlock / item_lanes(lpr, true), step = p.np > 1 ? 1 : kPartitions, n_groups = n_long + (n_all - n_long + per - 1) / per;
    int64_t misses = 0, reads = 0, counted = 0, counted_misses = 0;
    for (const int64_t from : {(int64_t)0, n_groups / 2 / step * step}) {
        // what was cached before a run counts as gone; a run counts from when its cache is full
        const int64_t gone = misses + cap, stop = reads + sample;
        int64_t start_reads = -1, start_misses = 0;
        misses = gone;
        const int64_t first_read = reads;
        for (int64_t g = from; g < n_groups && reads < stop; g += step) {
            const int64_t i0 = g < n_long ? g : n_long + (g - n_long) * per, i1 = g < n_long ? g + 1 : std::min(n_all, i0 + per);
            for (int64_t i = i0; i < i1; ++i) {
                const int32_t *c = col.data() + (p.items[i].beg & ~kItemDependsBit);
                for (int32_t j = 0; j < p.items[i].cnt; ++j) {
                    int32_t &at = seen[c[j]];
                    if (at <= misses - cap || at <= gone - 1) { ++misses; at = (int32_t)misses; }
                }
                reads += p.items[i].cnt;
                if (start_reads < 0 && misses - gone >= cap) { start_reads = reads; start_misses = misses; }
            }
        }
        if (start_reads < 0 || reads - start_reads < 1024) { start_reads = first_read; start_misses = gone; }
        counted += reads - start_reads;
        counted_misses += misses - start_misses;
        if (from == 0 && reads < stop) break;              // the run covered the plan
    }
    return counted > 0 ? (double)counted_misses / (double)counted : 0.;
}

static void add_plan(const hag_handle *h, const Plan &p, const std::vector<int32_t> &col, int w, PassCost &c) {
    if (p.items.empty()) return;
    const int lpr = p.np > 1 ? std::min(4 << w, p.lanes) : 4 << w;
    if (p.np > 1) c.lanes = p.lanes;
    int64_t n_long = 0, long0 = 0;
    for (int k = 0; k < p.np; ++k) {
        const int64_t n = long_items(p, k, block_threshold(h->knobs.sub_max, p, lpr));
        if (k == 0) long0 = n;
        n_long += n;
    }
    const double reads = (double)p.n_reads;
    c.miss[w] += reads * miss_rate(p, col, h->n + h->a, lpr, long0, reads, h->comp.enabled ? kSampleReadsBatch : kSampleReads);
    c.fold[w] += (double)n_long * (kBlock / lpr);
    if (w > 0) return;
    c.launches += p.combine.empty() ? 1 : 2;
    c.reads[p.np > 1] += reads;
    c.slots += (double)p.n_slots;
    c.rows += (double)(p.items.size() - (size_t)p.n_slots + p.combine.size());
}

void estimate_pass(const hag_handle *h, bool lists, bool backward, int w, PassCost &c) {
    if (lists) {
        add_plan(h, backward ? h->p_naive_bwd : h->p_naive_fwd, backward ? h->gt_dcol : h->g_dcol, w, c);
        return;
    }
    for (int32_t st = 0; st < h->stages; ++st) {
        if (backward) {
            add_plan(h, h->p_bwd_stage[st], h->ht_dcol, w, c);
        } else if (!h->stage_single_level[st]) {
            add_plan(h, h->p_fwd_stage[st], h->he.col, w, c);
        } else {
            const double m = h->stage_ptr[st + 1] - h->stage_ptr[st];   // two rows each, which nothing has read before
            c.miss[w] += 2 * m;
            if (w == 0) { c.launches += 1; c.reads[0] += 2 * m; c.rows += m; }
        }
    }
    add_plan(h, backward ? h->p_bwd_src : h->p_fwd, backward ? h->ht_dcol : h->hf_dcol, w, c);
}

void estimate_tiles(const hag_handle *h, Tiles &t, int w, PassCost &c) { add_plan(h, t.plan, t.rest_col, w, c); }

// The prices below were fitted to passes timed on an MI355X: 271 pairs (HAG, plain lists) for each of sum forward, sum transposed and max, over
// 20 graphs of 1e3 to 2.3e5 nodes and 5e4 to 1.1e8 edges (dense groups and overlapping cliques with ids in order and shuffled, community and power-law
// graphs), HAGs of |V| / 16 to |V| nodes that save 1 to 95 % of the row reads, d = 16, 64, 128 and 512.  A pass's time is met within 14 %
// (root mean square; max 17 %).  Taking what they call cheaper costs 0.4 % on average against always knowing (sum: more than 5 % in 9 of 542 cases, the
// worst 17 %; max: 0.5 %, 7 of 271, 33 %); always the lists would cost 13 % on average and up to 3.6 times (max 14 %, 3.8 times), always the HAG
// 13 % and up to 2.2 times (max 20 %, 3.9 times).  Microseconds; bytes and rows.
struct Price { double launch, read, hit, miss, fold, slot, row, item; };
constexpr Price kSumPrice{4.0, 0.9e-6, 1 / 42.5e6, 1 / 12.6e6, 1.4e-5, 1 / 4.5e6, 1 / 7.0e6, 3.8e-5};
constexpr Price kMaxPrice{7.1, 1.6e-6, 1 / 56e6, 1 / 10.3e6, 8.2e-5, 1 / 1.65e6, 1 / 2.5e6, 6.3e-5};

static double gather_us(const PassCost &c, bool max, int64_t d) {
    const Price &p = max ? kMaxPrice : kSumPrice;
    const int lpr = pick_lpr(d), w = lpr == 4 ? 0 : lpr == 8 ? 1 : lpr == 16 ? 2 : lpr == 32 ? 3 : 4;
    const double bytes = 4. * (double)d, all = std::ceil((double)d / (4 * lpr)), cut = std::ceil((double)d / (4 * std::min(lpr, c.lanes)));   // column chunks
    const double reads = c.reads[0] + c.reads[1], chunks = c.reads[1] > c.reads[0] ? cut : all;
    return p.launch * c.launches + p.read * (c.reads[0] * all + c.reads[1] * cut) + bytes * (p.hit * reads + p.miss * c.miss[w] + p.slot * c.slots + p.row * c.rows) +
           p.fold * c.fold[w] * chunks + p.item * (c.slots + c.rows);
}

// The component pass: a workgroup per component, several per compute unit as far as their LDS allows.  Either the compute unit's instructions or, with
// few workgroups side by side, the chains of one of them are what takes the time.  Fitted likewise: 304 pairs over 23 batches of 80 to 5000 graphs
// of 20 to 250 nodes, densities 0.02 to 0.9, d = 8 to 64; the cheaper side costs 0.8 % on average against always knowing (worst 35 %).
static double component_us(const hag_handle *h, bool lists, bool backward, int64_t d, size_t lds) {
    const Components &c = h->comp;
    const double count = (double)c.count, lpr = pick_lpr(d), steps = lists ? 0. : c.steps / (double)c.count;
    const double ids = c.entries[lists][backward] / (double)c.count * lpr / kWave * (lpr == 16 || lpr == 4 ? 1. : 1.85);   // wavefront steps; other widths broadcast ids through LDS
    const double rows = (double)(h->n + (lists ? 0 : h->a)) / (double)c.count * lpr / kWave;
    const double busy = 2.75e-3 * ids + 0.097 * rows;
    const double chain = 6.9e-3 * ids + 0.1445 * rows + (backward && !c.expanded ? 0.81 : 0.07) * steps + 2.64;
    const double per_cu = std::max(1., count / 256), side = std::max(1., std::min({8., std::floor(160. * 1024 / (double)(lds + 256)), per_cu}));
    return 3.24 + per_cu * std::pow(std::pow(busy, 4) + std::pow(chain / side, 4), 0.25);
}

// The dense products: bytes moved, or the steps of the wavefronts and how many rounds of them there are.  23 batches as above, d = 8 to 256: within 6.5 %.
static double dense_us(const hag_handle *h, int64_t d) {
    const double vec = dense_vec(d), tiles = (h->comp.max_nodes + 15) / 16, row_chunks = dense_row_chunks(h->comp.max_nodes);
    const double waves = (double)h->comp.count * row_chunks * std::ceil((double)d / (16 * vec));
    const double wave = std::ceil(h->comp.max_nodes / 32.) * (0.4 + vec * (0.062 + 0.0575 * tiles / row_chunks)) + 0.17 + 0.12 * vec;
    return 4.3 + std::cbrt((1 + std::pow(waves / 1211, 3)) * std::pow(wave, 3) + std::pow(0.153e-6 * 8. * (double)h->n * (double)d, 3));
}

// Passes mostly cut by source, at any width, where they are weighed against tiles.  The prices above were fitted at four widths that fill their column chunks and are too low in between (131072
// nodes, 26 M edges: d = 128 634 us, priced 699, but 132 1203, priced 744): a row is read in whole chunks, and misses are whole lines of 128 bytes.
// Fitted with the tiles below to 17 community and block graphs of 1.2 to 114 M edges (mean degrees 60 to 490), 15 widths from 8 to 512: lists within 7.3 % (root mean square), tiles
// and rest within 8.5 %.  Taking what is called cheaper costs 0.2 % on average against always knowing (more than 5 % in 5 of 255 cases, the worst 9.5 %).
static double row_lines(int64_t d, int64_t chunk) {          // lines a row of d floats touches when it is read in chunks, on average over its rows
    const double unit = (double)std::gcd(4 * d, (int64_t)128);
    const auto lines = [&](int64_t columns) { return columns > 0 ? (4. * (double)columns - unit) / 128 + 1 : 0.; };
    return (double)(d / chunk) * lines(chunk) + lines(d % chunk);
}
static double cut_us(const PassCost &c, int64_t d) {
    if (c.reads[1] <= c.reads[0]) return gather_us(c, false, d);
    const int lpr = pick_lpr(d), w = lpr == 4 ? 0 : lpr == 8 ? 1 : lpr == 16 ? 2 : lpr == 32 ? 3 : 4;
    const int64_t chunk = 4 * std::min(lpr, c.lanes), chunks = (d + chunk - 1) / chunk;
    const double reads = c.reads[0] + c.reads[1], line_bytes = 128 * row_lines(d, chunk);
    return 4.5 + 4. * c.launches + reads * (2.24e-6 * (double)chunks + 2.01e-8 * 4. * (double)(chunks * chunk) + 1.18e-8 * line_bytes) + 2.86e-8 * line_bytes * c.miss[w] +
           4e-6 * (double)d * (0.09 * c.slots + 0.3055 * c.rows);
}

// The tiles of the lists and the rest (us): the launches and the longest unit whatever the size, the steps and the lines their rows touch, the rest's gather.
static double tiles_us(const Tiles &t, int64_t d) {
    const int vec = dense_vec(d);
    const double chunks = std::ceil((double)d / (16 * vec)), steps = (double)t.ptr.back(), step = vec == 1 ? 0. : vec == 2 ? 0.56e-3 : 1.77e-3;
    return 36.9 + steps * (chunks * step + 0.386e-3 * row_lines(d, 16 * vec)) + cut_us(t.cost, d);
}
bool tiles_pay(const hag_handle *h, bool backward, int64_t d) {
    const Tiles &t = h->tiles[backward && !h->symmetric];
    return t.on && (h->knobs.tiles > 1 || tiles_us(t, d) < cut_us(h->cost[1][backward], d));
}

// Predictions this close are taken as equal: the lists then serve graphs below 16 M edges (where the community graphs measured gained from them) and
// the HAG larger ones (114 M edges, 14 to 17 % fewer reads: 2577 against 2704 us for a forward sum at d = 128, 10354 against 10874 us at 512, though the model has the
// two within 8 %).  A max over a HAG carries the winners' ids along: it has to be clearly cheaper.
static bool hag_is_cheaper(const hag_handle *h, bool max, double hag, double lists) {
    return hag < lists * (max ? 0.9 : h->e < 16000000 ? 0.95 : 1.08);
}

int cheapest_form(const hag_handle *h, const FormQuery &q) {
    const bool max = q.max, tiles = q.tiles_allowed && q.lists_allowed && tiles_pay(h, q.backward, q.d);
    const auto list_form = [&](bool lists) {
        const size_t lds = q.component_lds[lists];
        if (lds > 0) return component_us(h, lists, q.backward, q.d, lds);
        if (tiles) return lists ? tiles_us(h->tiles[q.backward && !h->symmetric], q.d) : cut_us(h->cost[0][q.backward], q.d);
        return gather_us(h->cost[lists][q.backward], max, q.d);
    };
    // (without aggregation nodes the pass over the HAG is the one over the lists)
    const bool choose = q.hag_allowed && q.lists_allowed && (h->a > 0 || tiles);
    double hag = 0, lists = 0;
    if (q.hag_allowed && (choose || q.dense_allowed)) hag = list_form(false);
    if (q.lists_allowed && (choose || q.dense_allowed)) lists = list_form(true);
    int form = q.hag_allowed && (!choose || (tiles ? h->knobs.tiles < 2 && hag < 0.95 * lists : hag_is_cheaper(h, max, hag, lists))) ? kFormHag : kFormLists;
    if (q.dense_allowed && dense_us(h, q.d) <= (form == kFormHag ? hag : lists)) form = kFormDense;
    return form;
}

}  // namespace hag
