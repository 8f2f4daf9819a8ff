// Host-side planning for the Adasum tree combiner: layer-table validation, the
// tile table (the bookkeeping of tensor boundaries inside the fused buffer,
// Section 4.4.3 of arXiv 2006.02924), the pass schedule over the binary tree of
// Section 3.4, and the device workspace layout.  Pure C++, no GPU calls.
#include "adasum_host.h"

#include <algorithm>



namespace adasum {

int check_layer_table(const int64_t* layer_offsets, int n_layers) {
    if (n_layers < 0) return ADASUM_ERR_INVALID_ARG;
    if (layer_offsets == nullptr) return ADASUM_ERR_INVALID_ARG;
    if (layer_offsets[0] != 0) return ADASUM_ERR_INVALID_ARG;
    for (int l = 0; l < n_layers; ++l) {
        if (layer_offsets[l + 1] < layer_offsets[l]) return ADASUM_ERR_INVALID_ARG;
    }
    return ADASUM_OK;
}

void build_tiles(const int64_t* layer_offsets, int n_layers, int64_t capacity,
                 std::vector<adasum_tile>& tiles, std::vector<int32_t>& layer_tile_begin) {
    tiles.clear();
    layer_tile_begin.assign(static_cast<size_t>(n_layers) + 1, 0);
    for (int l = 0; l < n_layers; ++l) {
        layer_tile_begin[l] = static_cast<int32_t>(tiles.size());
        int64_t pos = layer_offsets[l];
        const int64_t end = layer_offsets[l + 1];
        while (pos < end) {
            // next global multiple of the capacity strictly above pos, clipped to the layer
            int64_t stop = (pos / capacity + 1) * capacity;
            if (stop > end) stop = end;
            adasum_tile t;
            t.start = pos;
            t.len = static_cast<int32_t>(stop - pos);
            t.layer = l;
            tiles.push_back(t);
            pos = stop;
        }
    }
    layer_tile_begin[n_layers] = static_cast<int32_t>(tiles.size());
}

int build_levels(int K, int radix, std::vector<int>& radices) {
    radices.clear();
    if (K < 1) return ADASUM_ERR_INVALID_ARG;
    if (radix == 0) radix = kDefaultRadix;
    if (radix != 2 && radix != 4 && radix != 8 && radix != 16 && radix != 32 && radix != 64) return ADASUM_ERR_UNSUPPORTED;
    if (K == 1) return ADASUM_OK;
    // the shallowest depth whose sub-trees have at most `radix` leaves
    int depth = 0;
    while ((K + (1 << depth) - 1) / (1 << depth) > radix) ++depth;
    const int widest = (K + (1 << depth) - 1) / (1 << depth);
    int first = 2;
    while (first < widest) first *= 2;
    radices.push_back(first);
    int rest = 1 << depth;
    while (rest > 1) {
        // (only the first pass, over the 16-bit leaves, can be wider than kMaxRadix)
        int r = std::min(rest, std::min(radix, kMaxRadix));
        radices.push_back(r);
        rest /= r;
    }
    return ADASUM_OK;
}

int build_linear_passes(int K, int radix, std::vector<int>& passes) {
    passes.clear();
    if (K < 1) return ADASUM_ERR_INVALID_ARG;
    if (radix == 0) radix = kDefaultRadix;
    if (radix != 2 && radix != 4 && radix != 8 && radix != 16) return ADASUM_ERR_UNSUPPORTED;
    if (K == 1) return ADASUM_OK;
    int first = radix;
    while (first > K) first /= 2;
    passes.push_back(first);
    int rest = K - first;
    while (rest > 0) {
        int r = radix;
        while (r - 1 > rest) r /= 2;
        passes.push_back(r);
        rest -= r - 1;
    }
    return ADASUM_OK;
}

int wide_part_count(int64_t N) {
    int64_t parts = (N + kWidePartAlign - 1) / kWidePartAlign;
    if (parts > kWideParts) parts = kWideParts;
    if (parts < 1) parts = 1;
    // a part is what one wave quarter sums in fp32 before it widens: kept to kWideMaxPart elements, so
    // very long buffers get more parts than the chip holds workgroups (they run in several rounds)
    while (wide_part_elems(N, static_cast<int>(parts)) > kWideMaxPart) parts *= 2;
    return static_cast<int>(parts);
}

int64_t wide_part_elems(int64_t N, int n_parts) {
    const int64_t e = (N + n_parts - 1) / n_parts;
    return (e + kWidePartAlign - 1) / kWidePartAlign * kWidePartAlign;
}

void build_spans(const int64_t* layer_offsets, int n_layers, int n_parts, std::vector<adasum_tile>& spans,
                 std::vector<int32_t>& part_begin, std::vector<int32_t>& layer_begin) {
    // tiles whose capacity is a part: cut at the part boundaries and at the layer boundaries, sorted by
    // start, so the spans of a part are one contiguous run as those of a layer are
    const int64_t E = wide_part_elems(layer_offsets[n_layers], n_parts);
    build_tiles(layer_offsets, n_layers, E, spans, layer_begin);
    part_begin.assign(static_cast<size_t>(n_parts) + 1, 0);
    for (const adasum_tile& t : spans) ++part_begin[static_cast<size_t>(t.start / E) + 1];
    for (int p = 0; p < n_parts; ++p) part_begin[p + 1] += part_begin[p];
}

int64_t count_spans(const int64_t* layer_offsets, int n_layers, int n_parts) {
    const int64_t E = wide_part_elems(layer_offsets[n_layers], n_parts);
    return count_tiles(layer_offsets, n_layers, E);
}

int64_t find_small_layers(const int64_t* layer_offsets, int n_layers, std::vector<SmallLayer>& small) {
    small.clear();
    int64_t total = 0;
    for (int l = 0; l < n_layers; ++l) {
        const int64_t len = layer_offsets[l + 1] - layer_offsets[l];
        if (len < 1 || len > kSmallLayer) continue;
        SmallLayer s;
        s.start = layer_offsets[l];
        s.len = static_cast<int32_t>(len);
        s.layer = l;
        s.coff = static_cast<int32_t>(total);
        s.pad = 0;
        small.push_back(s);
        total += len;
    }
    return total;
}

int64_t count_tiles(const int64_t* layer_offsets, int n_layers, int64_t capacity) {
    int64_t n = 0;
    for (int l = 0; l < n_layers; ++l) {
        const int64_t lo = layer_offsets[l], hi = layer_offsets[l + 1];
        if (hi > lo) n += (hi - 1) / capacity - lo / capacity + 1;
    }
    return n;
}

int gram_tile_capacity(const int64_t* layer_offsets, int n_layers) {
    return count_tiles(layer_offsets, n_layers, kTile) < kFewTiles ? kTileSmall : kTile;
}

int64_t norm_entries_bound(int K, const int64_t* layer_offsets, int n_layers, const std::vector<int>& radices,
                           int node_type) {
    int64_t need = 1;
    int groups = K;
    for (size_t lv = 0; lv < radices.size(); ++lv) {
        groups /= radices[lv];
        // the widest storage type a pass may read gives its finest table
        const int64_t t = count_tiles(layer_offsets, n_layers, combine_tile_capacity(node_type, radices[lv]));
        // (the left-to-right order has one group per pass)
        need = std::max<int64_t>(need, static_cast<int64_t>(std::max(groups, 1)) * t);
    }
    if (radices.empty())
        need = std::max<int64_t>(need, count_tiles(layer_offsets, n_layers, combine_tile_capacity(node_type, 1)));
    return need;
}

int64_t next_entries_bound(int K, const int64_t* layer_offsets, int n_layers, const std::vector<int>& radices,
                           int node_type) {
    int64_t need = 0;
    int groups = K;
    for (size_t lv = 0; lv + 1 < radices.size(); ++lv) {
        groups /= radices[lv];
        if (!pass_feeds_next(radices, lv)) continue;
        const int R2 = radices[lv + 1];
        // the widest storage type a pass may read gives its finest table
        const int64_t t = count_tiles(layer_offsets, n_layers, feed_tile_capacity(node_type, radices[lv]));
        need = std::max<int64_t>(need, static_cast<int64_t>(groups / R2) * t * gram_entries(R2, true));
    }
    return need;
}

int64_t dot_entries_bound(int K, const int64_t* layer_offsets, int n_layers, const std::vector<int>& radices,
                          int node_type) {
    int64_t need = 0;
    int groups = K;
    for (size_t lv = 0; lv + 1 < radices.size(); ++lv) {
        groups /= radices[lv];
        if (radices[lv] != 2) continue;
        const int64_t t = count_tiles(layer_offsets, n_layers, combine_tile_capacity(node_type, 2));
        need = std::max<int64_t>(need, static_cast<int64_t>(groups / 2) * t);
    }
    return need;
}

Layout make_layout(int K, int64_t N, int n_layers, int64_t n_tiles, int64_t norm_entries,
                   const std::vector<int>& radices, int order, int64_t small_rows, int64_t small_elems,
                   int node_type, int64_t dot_entries, int64_t wide_spans) {
    Layout lay;
    lay.N = N;
    lay.n_tiles = n_tiles;
    lay.norm_entries = norm_entries;
    lay.n_layers = n_layers;
    lay.slot_elems = static_cast<int64_t>(align_up(static_cast<size_t>(N), 64));
    lay.node_bytes = elem_bytes(node_type);
    // nodes written by the first pass, unless that pass is already the root
    lay.n_slots = radices.size() > 1 ? K / radices[0] : 0;

    size_t max_partials = 0, max_gram = 0, max_weights = 0, max_nodes = 1;
    int groups = K;
    if (order == ADASUM_ORDER_LINEAR) {
        // one group per pass; slot 0 holds the running result
        lay.n_slots = radices.size() > 1 ? 1 : 0;
    }
    for (size_t lv = 0; lv < radices.size(); ++lv) {
        const int R = radices[lv];
        groups = order == ADASUM_ORDER_LINEAR ? 1 : groups / R;
        // (with the diagonal: a pass fed by the combine below it finds its whole matrix in the partials)
        const size_t np = static_cast<size_t>(gram_partial_entries(R));
        // (a wide pass -- always the first -- leaves its blocks per span, every other pass per Gram tile)
        const size_t rows = wide_radix(R) ? static_cast<size_t>(wide_spans) : static_cast<size_t>(n_tiles);
        max_partials = std::max(max_partials, static_cast<size_t>(groups) * np * rows);
        max_gram = std::max(max_gram, static_cast<size_t>(groups) * n_layers * R * R);
        max_weights = std::max(max_weights, static_cast<size_t>(groups) * n_layers * R);
        max_nodes = std::max(max_nodes, static_cast<size_t>(groups));
    }
    size_t off = 0;
    lay.off_slots = off;
    off = align_up(off + static_cast<size_t>(lay.n_slots) * lay.slot_elems * lay.node_bytes, 256);
    lay.off_partials = off;
    off = align_up(off + max_partials * sizeof(double), 256);
    lay.off_normparts = off;
    off = align_up(off + static_cast<size_t>(norm_entries) * sizeof(double), 256);
    lay.off_normcoarse = off;
    off = align_up(off + max_nodes * static_cast<size_t>(n_tiles) * sizeof(double), 256);
    lay.off_gram = off;
    off = align_up(off + max_gram * sizeof(double), 256);
    lay.off_weights = off;
    off = align_up(off + max_weights * sizeof(double), 256);
    lay.off_leafnorm = off;
    off = align_up(off + static_cast<size_t>(n_layers) * sizeof(double), 256);
    lay.off_small = off;
    lay.small_elems = small_elems;
    off = align_up(off + static_cast<size_t>(small_rows) * static_cast<size_t>(small_elems) * sizeof(double), 256);
    lay.off_dotparts = off;
    lay.dot_entries = dot_entries;
    off = align_up(off + static_cast<size_t>(dot_entries) * sizeof(double), 256);
    lay.base_total = off;
    lay.need = lay.total = off;
    return lay;
}

ResidentPlan plan_resident(int K, const std::vector<int>& radices, int dtype, bool delta, const int64_t* layer_offsets,
                           int n_layers) {
    ResidentPlan p;
    if (radices.size() != 1 || K < 2 || K > kResidentRadix || layer_offsets[n_layers] == 0) return p;
    p.R = resident_operands(K);
    if (p.R > 8 && (delta || dtype == ADASUM_F64)) return p;
    const int64_t N = layer_offsets[n_layers];
    const int64_t step = resident_step_elems(dtype);
    int64_t layers = 0;
    for (int l = 0; l < n_layers; ++l) layers += layer_offsets[l + 1] > layer_offsets[l];
    struct Count {
        int64_t most = 0, all = 0;   // units of the layer that has most, and of all
    };
    auto count = [&](int64_t cap) {
        Count c;
        for (int l = 0; l < n_layers; ++l) {
            const int64_t lo = layer_offsets[l], hi = layer_offsets[l + 1];
            const int64_t n = hi > lo ? (hi - 1) / cap - lo / cap + 1 : 0;
            c.most = std::max(c.most, n);
            c.all += n;
        }
        return c;
    };
    auto take = [&](int form, int64_t cap, const Count& c) {
        p.form = form;
        p.capacity = static_cast<int>(cap);
        p.n_units = c.all;
    };
    const Count one = count(step);
    if (one.all > 0x7fffffff) return p;
    if (one.most <= resident_most(dtype, p.R, 1) && one.all <= resident_slots(dtype, p.R, 1)) {
        take(1, step, one);
        return p;
    }
    for (int form = p.R <= 8 ? 2 : 3; form <= 3; ++form) {
        const int steps = resident_steps(dtype, p.R, delta, form), slots = resident_slots(dtype, p.R, form);
        // What suits the pass is judged by the steps in registers where LDS has one on top: the line is from before there was that one, and
        // refuses tables that fit in all steps.  What that gives away, us for this pass and for the others: BERT-Large / 8 (largest
        // layer 636 units, 477 in all steps), K = 16 bf16 320 and 472 in the tree order (left to right 474 and 469: nothing); 300
        // layers of 40000 elements and ten of 560 units (420 to 448 in all steps), K = 9 317 and 431, K = 12 378 and 522, K = 16
        // 395 and 531.
        const int judged = resident_matrix(dtype, p.R) ? resident_register_steps(dtype, p.R, delta, form) : steps;
        const Count full = count(step * judged);
        if (full.most > resident_most(dtype, p.R, form)) continue;
        // Tables of tiny layers: hardly more units in form 1, which holds more workgroups (K = 2 bf16, 20000 layers of 100 to
        // 300 elements: 43 us, in form 2 95; 600 layers of 1 to 20000: 24 and 28).  (The kernels on the matrix cores hold
        // as many workgroups in either form: with 12 to 16 rows form 1 is still ahead, K = 16 332 us for 542, with 10 it is
        // not, 288 for 277.)
        if (one.all <= 2 * full.all && one.most <= kDirectUnits && !(resident_matrix(dtype, p.R) && p.R < 12)) {
            take(1, step, one);
            return p;
        }
        // As small units as the chip still holds all at once, so that more of it is at work (K = 2 bf16, one layer of 900 000
        // elements in 220 units instead of 25: 15.8 us for 20.3).
        if (layers < slots)
            for (int64_t n = std::max<int64_t>(1, (N + step * (slots - layers) - 1) / (step * (slots - layers))); n < judged; ++n) {
                const Count c = count(step * n);
                if (c.all > slots || c.most > resident_most(dtype, p.R, form)) continue;
                take(form, step * n, c);
                return p;
            }
        // Layers of a little more than half the chip run alone on it, and the rest of it waits with them.  Where such layers
        // hold most of a table, the other passes were faster when this line was drawn (K = 16 fp32 511 and 416, K = 16 bf16 452 and
        // 419, K = 2 bf16 507 and 460; fp32 and fp64 of at most 8 rows stayed ahead: K = 8 fp32 431 and 472).  With the present exchange
        // that still holds for fp32 of 12 and more rows and, by 1 %, for the lower end of some others (K = 4 and 8 bf16); for the rest it
        // gives away up to a third.  20 layers of 270, 300, 340 and 370 units each, us for this pass and for those:
        // K = 16 fp32 413 449 506 538 and 388 422 463 521; K = 12 fp32 322 357 396 417 and 312 349 379 422; K = 10 fp32
        // 305 345 384 407 and 357 394 446 469; K = 16 bf16 274 305 323 453 and 400 434 488 528; K = 12 bf16 287 308 450 472 and
        // 420 452 510 546; K = 8 bf16 454 476 504 555 and 450 485 553 608; K = 4 bf16 465 486 507 532 and 461 513 568 613;
        // K = 2 bf16 308 468 495 539 and 420 470 531 579.  Five layers of 300: K = 16 fp32 117 and 142, K = 16 bf16 86 and
        // 155, K = 2 bf16 126 and 125; two: 52 and 102, 37 and 97, 56 and 58.
        if (form == 3 && (p.R > 8 || dtype == ADASUM_BF16 || dtype == ADASUM_F16)) {
            int64_t alone = 0, units = 0;
            for (int l = 0; l < n_layers; ++l) {
                const int64_t lo = layer_offsets[l], hi = layer_offsets[l + 1], cap = step * judged;
                const int64_t n = hi > lo ? (hi - 1) / cap - lo / cap + 1 : 0;
                if (n <= slots / 2 || n > (dtype == ADASUM_F32 && p.R >= 12 ? slots * 9 / 10 : slots * 7 / 10)) continue;
                ++alone;
                units += n;
            }
            if (alone >= 5 && 2 * units > full.all) return p;
        }
        // (the step in LDS comes after the others: nothing for units that the chip holds at once without it, nor for small layers)
        const Count larger = judged == steps ? full : count(step * steps);
        if (full.all > slots && larger.all * 10 <= full.all * 9) take(form, step * steps, larger);
        else take(form, step * judged, full);
        return p;
    }
    return p;
}

void add_resident(Layout& lay, const ResidentPlan& p) {
    const size_t words = static_cast<size_t>(gram_entries(p.R, true)) * 2;
    size_t off = lay.base_total;
    lay.off_resident = off;
    off = align_up(off + (1 + static_cast<size_t>(p.n_units)) * sizeof(int32_t), 256);
    lay.off_words = off;
    lay.partial_words = static_cast<int64_t>(p.n_units * words);
    off = align_up(off + (static_cast<size_t>(p.n_units) + static_cast<size_t>(lay.n_layers)) * words * sizeof(int64_t), 256);
    lay.need = lay.total = off;
}

void order_layers(const std::vector<int32_t>& layer_begin, int slots, std::vector<int>& layers) {
    // A layer's units wait for each other, so they should be on the chip together: whole layers are packed into runs of
    // half the workgroups that the chip holds (a larger layer into a run of all of them), the largest that still fits
    // next; the runs with the largest layers last.  In element order, units at the seams of such runs waited a whole
    // run's time: K = 8 fp32, ResNet-50 sizes, 271 us; in this order 232.
    const int L = static_cast<int>(layer_begin.size()) - 1;
    auto count = [&](int l) { return layer_begin[l + 1] - layer_begin[l]; };
    std::vector<int> by_size;
    for (int l = 0; l < L; ++l)
        if (count(l) > 0) by_size.push_back(l);
    std::stable_sort(by_size.begin(), by_size.end(), [&](int a, int b) { return count(a) > count(b); });
    struct Run {
        std::vector<int> layers;
        int room;
    };
    std::vector<Run> runs;
    size_t open = 0;   // runs before this one are full
    for (int l : by_size) {
        const int n = count(l);
        while (open < runs.size() && runs[open].room == 0) ++open;
        size_t r = open;
        const size_t last = std::min(runs.size(), open + 64);   // (bounds the search)
        while (r < last && runs[r].room < n) ++r;
        if (r == last) {
            r = runs.size();
            runs.push_back({{}, n > slots / 2 ? slots : slots / 2});
        }
        runs[r].layers.push_back(l);
        runs[r].room -= n;
    }
    layers.clear();
    for (size_t i = runs.size(); i-- > 0;) layers.insert(layers.end(), runs[i].layers.begin(), runs[i].layers.end());
}

void order_units(const std::vector<adasum_tile>& tiles, const std::vector<int32_t>& layer_begin, int slots,
                 std::vector<ResidentUnit>& units) {
    std::vector<int> layers;
    order_layers(layer_begin, slots, layers);
    units.clear();
    units.reserve(tiles.size());
    for (int l : layers) {
        int64_t elems = 0;
        for (int32_t t = layer_begin[l]; t < layer_begin[l + 1]; ++t) elems += tiles[t].len;
        for (int32_t t = layer_begin[l]; t < layer_begin[l + 1]; ++t) {
            ResidentUnit u;
            u.start = tiles[t].start;
            u.len = tiles[t].len;
            u.layer = l;
            u.unit = t;
            u.layer_first = layer_begin[l];
            u.layer_end = layer_begin[l + 1];
            u.small = elems <= kSmallLayer ? static_cast<int32_t>(elems) : 0;
            units.push_back(u);
        }
    }
}

}  // namespace adasum
