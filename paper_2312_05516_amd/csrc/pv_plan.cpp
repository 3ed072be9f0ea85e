// Host-side auxiliary data of a batch: validation, prefix sums and the work lists.
//
// The paper computes the per-batch auxiliary arrays (cumulative sequence lengths, each request's
// region of the concatenated tokens) once on the CPU and reuses them in every layer (Section 6.4;
// Section 4.4.1).  This file is that step, extended with the decomposition of the batch into work
// items for the two attention kernels.  It is pure host code and touches no HIP API.
#include "pv_plan.h"

#include <algorithm>
#include <cmath>
#include <numeric>
#include <cstdlib>
#include <cstring>
#include <new>
#include <unordered_set>

namespace pv {

bool pool_desc_valid(const pv_pool_desc *p, pv_status *why)
{
    pv_status s = PV_OK;
    if (!p || p->num_pages <= 0 || p->num_kv_heads <= 0 || p->page_size <= 0 || p->head_dim <= 0)
        s = PV_ERR_INVALID_ARG;
    else if (p->page_size != 16 || (p->head_dim != 64 && p->head_dim != 128) ||
             (p->dtype != PV_F16 && p->dtype != PV_BF16))
        s = PV_ERR_UNSUPPORTED;
    if (why) *why = s;
    return s == PV_OK;
}

static int32_t env_int(const char *name, int32_t fallback)
{
    const char *v = std::getenv(name);
    if (!v || !*v) return fallback;
    char *end = nullptr;
    long x = std::strtol(v, &end, 10);
    if (end == v || x <= 0 || x > (1 << 24)) return fallback;
    return (int32_t)x;
}

Tuning default_tuning()
{
    Tuning t;
    t.split_target = env_int("PV_SPLIT_TARGET", 0);
    t.split_by_hand = t.split_target > 0;
    if (!t.split_by_hand) t.split_target = kSplitTarget;
    t.min_split_keys = env_int("PV_MIN_SPLIT_KEYS", 256);
    t.wide_min_rows = env_int("PV_WIDE_MIN_ROWS", 33);
    t.xcds = env_int("PV_XCDS", 8);
    t.unify = env_int("PV_UNIFY", 1) == 1 ? 1 : 0;  // any other positive value switches it off
    t.unify_max_steps = env_int("PV_UNIFY_MAX_STEPS", 90000);
    t.even_cus = true;
    {
        const char *v = std::getenv("PV_TILE_MIN_KEYS");
        t.tile_min_keys = (v && *v == '0' && !v[1]) ? 0 : env_int("PV_TILE_MIN_KEYS", 8192);
        t.tile_batch_min_keys = (v && *v) ? 0 : 1536;
    }
    return t;
}

// Whether the full 256-row tiles of a (request, KV head) unit go to the 256-row kernel: that
// kernel exists for head size 128 and pays off when an item streams many 32-key blocks.
static bool use_tile256(const pv_pool_desc *pool, const Tuning &tune, int64_t rows_total,
                        int64_t kv_len)
{
    return tune.tile_min_keys > 0 && pool->head_dim == 128 && rows_total >= kTileRows &&
           kv_len >= tune.tile_min_keys;
}

// an item takes one step per block of keys whatever its row count
static int64_t item_cost(const WorkItem &w) { return w.kv_end - w.kv_begin; }

// A way to cut a list: every item longer than `longest_whole` (and of at least 2 * min_keys keys)
// into parts of about `chunk` keys, evened out and rounded up to whole blocks.
struct Cut {
    int64_t chunk, longest_whole, min_keys;
    int32_t parts(int64_t len) const
    {
        return len <= longest_whole || len < 2 * min_keys ? 1 : ((int32_t)len - 1) / part_len(len) + 1;
    }
    // length of the parts of an item that is cut
    int32_t part_len(int64_t len) const
    {
        const uint32_t keys = (uint32_t)len, n = (keys - 1) / (uint32_t)chunk + 1;
        return (int32_t)(((keys - 1) / n + kKvBlock) / kKvBlock * kKvBlock);
    }
};

// The cut into about `target` equal parts: every item of a list that is shorter than that, only
// items more than twice as long as a target-th of the keys in a longer one.
static Cut target_cut(int64_t total_keys, size_t items, int32_t target, const Tuning &tune)
{
    Cut c;
    c.min_keys = tune.min_split_keys;
    c.chunk = std::max<int64_t>((total_keys + target - 1) / target, c.min_keys);
    c.chunk = (c.chunk + kKvBlock - 1) / kKvBlock * kKvBlock;
    c.longest_whole = (int64_t)items >= target ? 2 * c.chunk : c.chunk;
    return c;
}

// A list of the narrow or the 128-row kernel, and what the rules below need to know of that kernel.
struct CutRule {
    int32_t slots;       // workgroups that the GPU holds at once
    int32_t long_list;   // from this many items on only outliers are cut (0: see target_cut)
    int32_t long_share;  // ... items more than a quarter longer than a long_share-th of the keys
    int32_t stretch_pct; // parts may be longer than a slots-th of the keys by so much, to run at once
    bool always_stretch; // also where they do not run at once even so (else: target_cut)
    int32_t key_ns;      // what a key less in the longest item saves while the GPU is not full
    int32_t always_cut;  // up to this many parts that is not weighed against the merge
    bool level_lists;    // lists of nearly equal items go by how full their last round of CUs is
};

// Cut long items into parts of the KV range.  A cut is not free: every part pays the set-up of an
// item, writes its rows in fp32, and the merge reads them back.  Returns true where an item gets
// fewer parts than the cut into about split_target parts gives it.
//  * Parts that all run at once are best where little more than a slots-th of the keys each does
//    it: one part more than there are slots starts when the others are nearly done.  4 generation
//    steps over 0.7-9 K keys, 64/8 heads, attention alone: 512 parts 19.1 us, 568 parts 21.7, 416
//    20.2.  Lists of 416 to 512 equal items are left whole by that (480 over 2 K keys: 75.5 us,
//    85.9 in 3 parts each; 376, which 1.25 does not reach: 68.5 whole, 63.1 in two, 69.4 in
//    three).
//  * Otherwise the narrow kernel, which is bound by bandwidth, wants about 1024 parts, so that no
//    workgroup walks a long item alone while the others have left: 62 requests over 500 keys and
//    one over 32 K, 64/8 heads, 48.3 us (211 in parts that run at once: the short items take up
//    their slots).  From 640 items on (head size 128) enough run behind one another for cutting
//    outliers alone: 672 items over 0.1-8 K keys 83.3 us against 86.0.  Not so for head size 64,
//    where an item takes half the time per key: 45.8 against 42.2.
//  * With 513 to 1023 items of nearly the same length (the longest a quarter over the average at
//    most) what counts is how many CUs the last round of 256 items leaves idle: whole against two
//    parts, 2.5 K keys on average and +-10 % of that, head size 128: 520 items 121 us / 109, 640 132
//    / 129, 672 136 / 145, 768 146 / 157, 784 170 / 170 (6 K keys: 410 / 394), 896 179 / 184 (426 /
//    421), 928 181 / 197, 1016 193 / 211; head size 64: 640 70 / 67, 672 72 / 75, 768 76 / 79, 800
//    90 / 86, 896 94 / 92, 928 95 / 99.  So whole where it is at least six tenths full.
//  * The 128-row kernel, bound by its arithmetic, with 16 times the rows to merge, takes as few
//    parts as keep the longest within twice a slots-th of the keys: 11 requests of 100 tokens and
//    one over 30 K, 40/40 heads, 163 us against 177 in about 1024 parts, 10 of 128 tokens over
//    1000 whole 53 against 90, 19 (760 items, one over 30 K) 170 against 188.
//  * Nothing is cut where the merge costs more than the shorter longest item gives: about 7 us for
//    one more kernel behind the slowest part (4-5 of its own), and 8 bytes per partial row element
//    at about 4 TB/s.  16 generation steps over 520-640 keys are left whole (10.8-11.2 us; cut
//    11.7), over 900 cut (11.9; whole 14.9); head size 64 up to 1000 (9.0 against 11.7 at 640, 13.4
//    against 11.7 at 1400).  6 requests of 100 tokens over 900 keys, 32/8 heads, 128-row kernel: 19.0
//    whole, 27.6 cut; over 2500 40.6 and 38.8.  Where the cut of all long items does not pay, that
//    of the longest few may.  The 128-row kernel's items (head size 128) are cut in any case while
//    every part has a CU of its own: 80 items in 240 parts 19.8 us, 21.9 whole; 130 in 202 22.1 and
//    23.9; 20 in 56 18.2 and 21.3.
//  * Whatever the list, no part is longer than max_len keys (0 = no such limit).
// No rule (the 256-row kernel), or a target set by hand: target_cut.
static bool split_items(std::vector<WorkItem> &items, std::vector<CombineItem> &combine,
                        int64_t &slots_out, const Tuning &tune, const CutRule *rule,
                        int32_t head_dim, int64_t max_len = 0)
{
    if (items.empty()) return false;
    if (tune.split_by_hand) rule = nullptr;
    // Every KV head has the same items, so lengths are looked at for the first head only, each
    // `heads` times (nothing is cut yet).
    struct Shape { int64_t len, rows; };
    std::vector<Shape> shapes;
    int64_t total_keys = 0, longest = 0;
    for (const WorkItem &w : items) {
        if (w.kv_head != 0) continue;
        const int64_t len = w.kv_end - w.kv_begin;
        shapes.push_back(Shape{len, w.row_count});
        total_keys += len;
        longest = std::max(longest, len);
    }
    const int64_t heads = (int64_t)(items.size() / shapes.size());
    total_keys *= heads;
    const Cut even = target_cut(total_keys, items.size(), tune.split_target, tune);
    Cut cut = even;
    if (rule) {
        auto blocks = [](int64_t keys) { return (keys + kKvBlock - 1) / kKvBlock * kKvBlock; };
        const int64_t n = (int64_t)items.size();
        if (rule->level_lists && n > rule->slots && n < tune.split_target &&
            longest * n * 4 <= total_keys * 5) {
            const int64_t rest = n % kCUs;
            if (rest == 0 || rest * 5 >= kCUs * 3) cut.longest_whole = longest;
        } else if (rule->long_list && n >= rule->long_list) {
            const int64_t share = (total_keys + rule->long_share - 1) / rule->long_share;
            cut.chunk = blocks(std::max<int64_t>(share, tune.min_split_keys));
            cut.longest_whole = cut.chunk + cut.chunk / 4;
        } else if (rule->always_stretch || n <= rule->slots) {
            auto at_once = [&](int64_t chunk) {
                const Cut c = {chunk, chunk, cut.min_keys};
                int64_t parts = 0;
                for (const Shape &s : shapes) parts += c.parts(s.len);
                return parts * heads <= rule->slots;
            };
            const int64_t share = (total_keys + rule->slots - 1) / rule->slots;
            int64_t lo = blocks(std::max<int64_t>(share, tune.min_split_keys));
            int64_t hi = blocks(lo + lo * rule->stretch_pct / 100);
            if (at_once(lo)) {
                hi = lo;
            } else if (at_once(hi)) {
                while (hi - lo > std::max<int64_t>(kKvBlock, lo / 32)) {
                    const int64_t mid = blocks((lo + hi) / 2);
                    (at_once(mid) ? hi : lo) = mid;
                }
            } else if (!rule->always_stretch) {
                hi = 0;
            }
            if (hi) cut.chunk = cut.longest_whole = hi;
        }
        // the cut of all long items, or where that does not pay, of the longest few
        for (bool few = false; cut.longest_whole < longest; few = true) {
            int64_t part_rows = 0, whole = 0, all_parts = 0;
            for (const Shape &s : shapes) {
                const int64_t parts = cut.parts(s.len);
                all_parts += parts * heads;
                if (parts > 1)
                    part_rows += s.rows * parts * heads;
                else
                    whole = std::max(whole, s.len);
            }
            if (cut.parts(longest) > 1) {
                const int64_t part_len = cut.part_len(longest);
                const int64_t after =
                    few || rule->always_stretch ? std::max(whole, part_len) : part_len;
                if ((longest - after) * rule->key_ns >= 7000 + part_rows * head_dim * 8 / 4000 ||
                    all_parts <= rule->always_cut)
                    break;
            }
            cut.chunk = cut.longest_whole = 2 * cut.longest_whole;
        }
    }
    auto too_long = [&](int64_t len) { return max_len > 0 && len > max_len; };
    // items that get fewer parts than the even cut gives them
    bool fewer = false;
    if (longest > even.longest_whole &&
        (cut.chunk > even.chunk || cut.longest_whole > even.longest_whole))
        for (WorkItem &w : items) {
            const int64_t len = w.kv_end - w.kv_begin;
            if (even.parts(len) <= cut.parts(len)) continue;
            fewer = true;
            w.renew_blocks =
                (uint32_t)std::max(even.part_len(len) / (head_dim == 128 ? 32 : 64), 1);
        }
    if (longest <= cut.longest_whole && !too_long(longest))
        return fewer;  // the common case of a long list: nothing is copied
    std::vector<WorkItem> result;
    int64_t all_parts = 0;
    for (const Shape &s : shapes)
        all_parts += std::max<int64_t>(cut.parts(s.len),
                                       too_long(s.len) ? (s.len + max_len - 1) / max_len : 1);
    result.reserve((size_t)(all_parts * heads));
    for (const WorkItem &w : items) {
        const int64_t len = w.kv_end - w.kv_begin;
        int64_t parts = cut.parts(len);
        if (too_long(len)) parts = std::max(parts, (len + max_len - 1) / max_len);
        if (parts <= 1) {
            result.push_back(w);
            continue;
        }
        int64_t part_len = (len + parts - 1) / parts;
        part_len = (part_len + kKvBlock - 1) / kKvBlock * kKvBlock;
        parts = (len + part_len - 1) / part_len;
        if (parts <= 1) {
            result.push_back(w);
            continue;
        }
        CombineItem c;
        c.req = w.req;
        c.kv_head = w.kv_head;
        c.row_begin = w.row_begin;
        c.row_count = w.row_count;
        c.partial_base = (int32_t)slots_out;
        c.split_count = (int32_t)parts;
        c.q_row0 = w.q_row0;
        c.groups = 1;  // set when all rows are known
        combine.push_back(c);
        for (int64_t s = 0; s < parts; ++s) {
            WorkItem part = w;
            part.kv_begin = (int32_t)(w.kv_begin + s * part_len);
            part.kv_end = (int32_t)std::min<int64_t>(w.kv_end, w.kv_begin + (s + 1) * part_len);
            part.split_index = (int32_t)s;
            part.split_count = (int32_t)parts;
            part.partial_base = (int32_t)(slots_out + s * w.row_count);
            result.push_back(part);
        }
        slots_out += parts * w.row_count;
    }
    items.swap(result);
    return fewer;
}

// Order of the XCDs' items where all of them run at once: workgroup k of an XCD goes to CU k % cus, so
// that round after round every CU gets one more.  The longest items are dealt first, each to the CU
// with the least to do, and every CU takes as many as the rounds give it.  In the order of the list
// below some CUs get several long items and others short ones only.  The 128-row kernel over that
// order and over this one, in microseconds: 64 / 8 heads, 2 first prompts of 68-1291 tokens 49.0 /
// 44.1; 32 / 8 heads of size 64, 4 of 392-955 32.1 / 26.9; 11 prompts of 113-459 on contexts of
// 175-923 51.9 / 46.5; geometric mean of 50 batches with 257-1000 tiles 3.1 % less.  Of whole items
// no list was more than 1 % behind.  Parts of cut items are alike already: 272 such lists 1.6 % less
// in the mean, 9 more than 2 % behind (11 requests, half of 35 tokens and half of one over 0.05-1.5
// K, 40/10 heads, 26.4 / 28.1 the worst) and 29 more than 5 % ahead (21 % the best), without a property
// that tells the ones from the others.
// Among CUs with equal loads the last one is taken: dealt from the first CU up, the longest items
// went to the CUs that get one item more, and lists a little over one round (276-352 items) lost
// 2-4 %.  The 16-row kernel reads its items at the rate of memory whatever shares a CU: no difference.
// Lengths are told apart to 1/128 of the longest one, so that one counting pass sorts them:
// 612-760 items take 6-9 us of the host on top of 13-20 for the whole plan, 25-45 with a comparison
// sort for each XCD and a branch for each CU.  That is for a plan that several layers use, and for
// items whose lengths differ (see worth_pairing).
static void pair_up(const std::vector<WorkItem> &items, std::vector<std::vector<uint32_t>> &queues)
{
    const size_t cus = kCUs / queues.size();  // a power of two
    int64_t longest = 1;
    for (const WorkItem &w : items) longest = std::max(longest, item_cost(w));
    int shift = 0;
    while ((longest >> shift) > 255) ++shift;

    const uint32_t set_up = kItemSetUp >> shift;

    struct Dealt { uint32_t pos; uint16_t queue, steps; };
    uint32_t begin[257] = {};
    size_t n = 0, most = 0;
    for (const std::vector<uint32_t> &q : queues)
        if (q.size() > cus) {
            for (uint32_t pos : q) ++begin[256 - (item_cost(items[pos]) >> shift)];
            n += q.size();
            most = std::max(most, q.size());
        }
    for (int b = 0; b < 256; ++b) begin[b + 1] += begin[b];
    std::vector<Dealt> dealt(n);
    for (size_t k = 0; k < most; ++k)  // the XCDs in turn, whose dealing does not depend on each other
        for (size_t q = 0; q < queues.size(); ++q)
            if (k < queues[q].size() && queues[q].size() > cus) {
                const uint32_t pos = queues[q][k];
                const uint16_t steps = (uint16_t)(item_cost(items[pos]) >> shift);
                dealt[begin[255 - steps]++] = Dealt{pos, (uint16_t)q, steps};
            }

    // load * cus + (cus - 1 - CU): the least of them names the CU too, the last one of equals.  Loads
    // are counted in the sorted steps, so that a float (which has a minimum of four in one
    // instruction) holds every key: at most (n + cus) * 351 < 2^24.
    constexpr float kFull = 3e38f;
    const size_t stride = std::max<size_t>(cus, 16);
    std::vector<float> keys(queues.size() * stride, kFull);
    std::vector<uint32_t> taken(queues.size() * cus, 0);
    for (size_t q = 0; q < queues.size(); ++q)
        for (size_t c = 0; c < cus; ++c) keys[q * stride + c] = (float)(cus - 1 - c);
    for (const Dealt &it : dealt) {
        float *key = &keys[it.queue * stride], least[16];
        for (size_t l = 0; l < 16; ++l) least[l] = key[l];
        for (size_t c = 16; c < stride; c += 16)
            for (size_t l = 0; l < 16; ++l) least[l] = key[c + l] < least[l] ? key[c + l] : least[l];
        for (size_t w = 8; w > 0; w /= 2)
            for (size_t l = 0; l < w; ++l) least[l] = least[l + w] < least[l] ? least[l + w] : least[l];
        const uint32_t best = (uint32_t)least[0];
        const size_t c = cus - 1 - (best & (cus - 1));
        std::vector<uint32_t> &queue = queues[it.queue];
        const size_t k = taken[it.queue * cus + c]++ * cus + c;
        queue[k] = it.pos;
        key[c] = k + cus < queue.size() ? (float)(best + (it.steps + set_up) * cus) : kFull;
    }
}

// Items within a 32nd of the longest one's length: any dealing leaves the CUs with as many of them, and
// so as much to do to 3 %.  Five such lists: 0.997-1.004 times the time of the list's own order.
static bool worth_pairing(const std::vector<WorkItem> &items)
{
    int64_t longest = 0, shortest = INT64_MAX;
    for (const WorkItem &w : items) {
        longest = std::max(longest, item_cost(w));
        shortest = std::min(shortest, item_cost(w));
    }
    return (longest - shortest) * 32 > longest;
}

// Order of the work list = order of workgroup dispatch.  Two goals:
//  * longest first, so that in-order dispatch approximates longest-processing-time scheduling;
//  * items that stream the same K/V (the row tiles of one (request, KV head, KV part)) should run
//    at the same time on the same XCD, so that the second and later tiles hit in that XCD's L2.
//    Workgroup i of a launch goes to XCD i % xcds, so a group's items are placed `xcds` positions
//    apart.  Groups are dealt to the XCDs greedily by accumulated cost (longest group first).
// A list of at most `slots` items runs at once, and which items share a CU is all that its order
// decides: see pair_up (0: keep the order of the list).
static void order_items(std::vector<WorkItem> &items, int xcds, size_t slots)
{
    if (items.empty()) return;
    if (xcds < 1) xcds = 1;
    const size_t n = items.size();
    // 1. group by (req, kv_head, split_index); items of a group keep their row order.  The list has
    //    the items of a (req, kv_head) one behind the other, so only a unit with cut items has to
    //    be sorted, by counting (480 items of 72 cut ones: 11.8 us for the whole plan with a
    //    comparison sort over the list and every length looked at, 8.3 now).
    struct Group { uint32_t begin, end; int64_t cost; };
    std::vector<uint32_t> order(n), first;
    std::vector<Group> groups;
    groups.reserve(n);
    for (size_t i = 0; i < n;) {
        size_t j = i;
        int32_t parts = 1;
        for (; j < n && items[j].req == items[i].req && items[j].kv_head == items[i].kv_head; ++j)
            parts = std::max(parts, items[j].split_count);
        const size_t base = groups.size();
        if (parts == 1) {
            int64_t cost = 0;
            for (size_t k = i; k < j; ++k) {
                order[k] = (uint32_t)k;
                cost += item_cost(items[k]);
            }
            groups.push_back(Group{(uint32_t)i, (uint32_t)j, cost});
        } else {
            first.assign((size_t)parts + 1, 0);
            for (size_t k = i; k < j; ++k) ++first[(size_t)items[k].split_index + 1];
            for (int32_t p = 0; p < parts; ++p) {
                first[(size_t)p + 1] += first[(size_t)p];
                groups.push_back(Group{(uint32_t)(i + first[(size_t)p]),
                                       (uint32_t)(i + first[(size_t)p + 1]), 0});
            }
            for (size_t k = i; k < j; ++k) {
                const size_t p = (size_t)items[k].split_index;
                order[i + first[p]++] = (uint32_t)k;
                groups[base + p].cost += item_cost(items[k]);
            }
        }
        i = j;
    }
    // 2. longest group first (per item, so that a long single item is not hidden behind a group of
    //    many short ones), dealt to the least loaded XCD
    std::sort(groups.begin(), groups.end(), [&](const Group &a, const Group &b) {
        const int64_t x = a.cost * (int64_t)(b.end - b.begin);
        const int64_t y = b.cost * (int64_t)(a.end - a.begin);
        return x != y ? x > y : a.begin < b.begin;
    });
    std::vector<std::vector<uint32_t>> queue((size_t)xcds);
    for (auto &qv : queue) qv.reserve(n / (size_t)xcds + 16);
    std::vector<int64_t> load((size_t)xcds, 0);
    for (const Group &g : groups) {
        size_t best = 0;
        for (size_t x = 1; x < (size_t)xcds; ++x)
            if (load[x] < load[best]) best = x;
        for (uint32_t i = g.begin; i < g.end; ++i) queue[best].push_back(order[i]);
        load[best] += g.cost;
    }
    if (n > (size_t)kCUs && n <= slots && kCUs % xcds == 0 && worth_pairing(items))
        pair_up(items, queue);

    // 3. interleave: position k*xcds + x takes the k-th item of XCD x's queue; once a queue is
    //    empty its positions are filled from the queues that still have items
    std::vector<WorkItem> out;
    out.reserve(n);
    std::vector<size_t> at((size_t)xcds, 0);
    size_t x = 0;
    while (out.size() < n) {
        size_t pick = x;
        for (int tries = 0; tries < xcds && at[pick] >= queue[pick].size(); ++tries)
            pick = pick + 1 == (size_t)xcds ? 0 : pick + 1;
        out.push_back(items[queue[pick][at[pick]++]]);
        x = x + 1 == (size_t)xcds ? 0 : x + 1;
    }
    items.swap(out);
}

// One contiguous host image of the arrays the kernels read, each part 256-byte aligned.
static void build_image(pv_plan *plan)
{
    struct Part { const void *src; size_t bytes; };
    const Part parts[9] = {
        {plan->ctx_lens.data(), plan->ctx_lens.size() * sizeof(int32_t)},
        {plan->q_lens.data(), plan->q_lens.size() * sizeof(int32_t)},
        {plan->q_start.data(), plan->q_start.size() * sizeof(int32_t)},
        {plan->combine_chunks.data(), plan->combine_chunks.size() * sizeof(CombineChunk)},
        {plan->narrow.data(), plan->narrow.size() * sizeof(WorkItem)},
        {plan->wide.data(), plan->wide.size() * sizeof(WorkItem)},
        {plan->tile256.data(), plan->tile256.size() * sizeof(WorkItem)},
        {plan->combine.data(), plan->combine.size() * sizeof(CombineItem)},
        {plan->append_groups.data(), plan->append_groups.size() * sizeof(AppendGroup)},
    };
    size_t total = 0;
    for (int i = 0; i < 9; ++i) {
        plan->image_off[i] = total;
        total += (parts[i].bytes + 255) / 256 * 256;
    }
    if (total == 0) total = 256;
    plan->image.assign(total, 0);
    for (int i = 0; i < 9; ++i)
        if (parts[i].bytes)
            std::memcpy(plan->image.data() + plan->image_off[i], parts[i].src, parts[i].bytes);
}

pv_status check_batch(const pv_pool_desc *pool, int32_t num_q_heads, const int32_t *ctx_lens,
                      const int32_t *q_lens, int32_t num_reqs, int32_t max_pages_per_req,
                      int32_t *total_q_out)
{
    pv_status why;
    if (!pool_desc_valid(pool, &why)) return why;
    if (num_q_heads <= 0 || num_q_heads % pool->num_kv_heads != 0) return PV_ERR_INVALID_ARG;
    if (num_reqs < 0 || max_pages_per_req < 0) return PV_ERR_INVALID_ARG;
    if (num_reqs > 0 && (!ctx_lens || !q_lens)) return PV_ERR_INVALID_ARG;
    const int32_t P = pool->page_size;
    const int32_t G = num_q_heads / pool->num_kv_heads;

    int64_t total_q = 0;
    for (int32_t r = 0; r < num_reqs; ++r) {
        if (ctx_lens[r] < 0 || q_lens[r] < 0) return PV_ERR_INVALID_ARG;
        const int64_t len = (int64_t)ctx_lens[r] + q_lens[r];
        if (len > INT32_MAX - 64) return PV_ERR_OUT_OF_RANGE;
        if (q_lens[r] > 0 && (len + P - 1) / P > max_pages_per_req) return PV_ERR_OUT_OF_RANGE;
        if ((int64_t)q_lens[r] * G > INT32_MAX / 2) return PV_ERR_OUT_OF_RANGE;
        total_q += q_lens[r];
    }
    // rows of q/out are indexed with 64-bit arithmetic in the kernels; the row count itself and
    // the workspace slot numbers stay 32-bit
    if (total_q > INT32_MAX / 2) return PV_ERR_OUT_OF_RANGE;
    *total_q_out = (int32_t)total_q;
    return PV_OK;
}

pv_status build_plan(const pv_pool_desc *pool, int32_t num_q_heads, const int32_t *ctx_lens,
                     const int32_t *q_lens, int32_t num_reqs, int32_t max_pages_per_req,
                     const Tuning &tune, pv_plan **out)
{
    if (!out) return PV_ERR_INVALID_ARG;
    *out = nullptr;
    int32_t total_q = 0;
    const pv_status ok = check_batch(pool, num_q_heads, ctx_lens, q_lens, num_reqs,
                                     max_pages_per_req, &total_q);
    if (ok != PV_OK) return ok;
    const int32_t G = num_q_heads / pool->num_kv_heads;

    pv_plan *plan = new (std::nothrow) pv_plan();
    if (!plan) return PV_ERR_INVALID_ARG;
    plan->pool = *pool;
    plan->num_q_heads = num_q_heads;
    plan->group = G;
    plan->num_reqs = num_reqs;
    plan->max_pages_per_req = max_pages_per_req;
    plan->total_q = total_q;
    plan->ctx_lens.assign(ctx_lens, ctx_lens + num_reqs);
    plan->q_lens.assign(q_lens, q_lens + num_reqs);
    plan->q_start.resize(num_reqs);
    plan->partial_slots = 0;
    plan->uploaded = false;
    plan->device = -1;
    plan->d_owned = nullptr;
    std::memset(&plan->dev, 0, sizeof plan->dev);
    plan->timing = false;
    plan->tile_scales_scores = false;
    for (void *&e : plan->events) e = nullptr;
    for (bool &u : plan->event_used) u = false;
    int32_t at = 0;
    for (int32_t r = 0; r < num_reqs; ++r) {
        plan->q_start[r] = at;
        at += q_lens[r];
    }

    // append: runs of new tokens that share an 8-slot group of a page
    for (int32_t r = 0; r < num_reqs; ++r) {
        const int64_t c = ctx_lens[r], end = (int64_t)ctx_lens[r] + q_lens[r];
        for (int64_t t = c; t < end;) {
            const int64_t group_end = (t / 8 + 1) * 8;
            const int64_t stop = std::min(end, group_end);
            AppendGroup g;
            g.req = r;
            g.t_begin = (int32_t)t;
            g.count = (int32_t)(stop - t);
            g.q_row = plan->q_start[r] + (int32_t)(t - c);
            plan->append_groups.push_back(g);
            t = stop;
        }
    }

    // One attention launch instead of two for a mixed batch.  A launch takes at least 2 us of the
    // stream, the two kernels cannot share a CU, and a short bandwidth-oriented launch never gets
    // the GPU up to speed, while its units fit well into the slots the long matrix-core items leave.
    // But an item of the matrix-core kernel holds a workgroup slot for one step per 32 keys whatever
    // its row count, so when the small units (generation steps) are a large amount of work, the
    // bandwidth-oriented kernel is the better place for them.  Measured crossover on mixes of
    // 256-token prompts and generation steps over 2000-token contexts, MHA 40/40 and GQA 64/8 alike:
    // 80-100 K steps of 32 keys summed over the small units and KV heads (~1.5 GB of K/V).
    // The 256-row kernel runs one workgroup per CU and needs a launch of its own, so in a mixed
    // batch it only pays for long KV ranges (tile_min_keys).  A batch that is nearly all long
    // multi-token units of head size 128 is another matter: measured on batches of 256- to 512-token
    // requests it is ahead of the 128-row kernel from about 1.5 K keys up (+5 % there, +7-8 % with
    // mixed lengths of 1-3.5 K or a few generation steps in the batch, +11 % at 4.5 K).  The
    // lower limit applies when at least 90 % of the batch's (row, key) pairs are in full 256-row
    // tiles of units that qualify under it, and those tiles are many enough and even enough that
    // the plan will not cut them (a cut item writes fp32 partial results that a merge pass reads).
    Tuning tune_batch = tune;
    if (tune.tile_batch_min_keys > 0 && tune.tile_min_keys > tune.tile_batch_min_keys &&
        pool->head_dim == 128) {
        int64_t pairs_all = 0, pairs_tile = 0, items = 0, keys = 0, longest = 0;
        // of units that qualify under the usual limit, and of their full tiles
        int64_t pairs_long = 0, pairs_long_tiles = 0, long_items = 0, long_keys = 0;
        int64_t long_min = INT64_MAX, long_max = 0;
        for (int32_t r = 0; r < num_reqs; ++r) {
            const int64_t n = q_lens[r], c = ctx_lens[r];
            if (n == 0) continue;
            const int64_t rows_total = n * G, kv = c + n;
            pairs_all += rows_total * kv;
            if (rows_total >= kTileRows && kv >= tune.tile_batch_min_keys) {
                const int64_t tiles = rows_total / kTileRows;
                pairs_tile += tiles * kTileRows * kv;
                items += tiles * pool->num_kv_heads;
                if (kv >= tune.tile_min_keys) {
                    long_items += tiles * pool->num_kv_heads;
                    long_keys += tiles * pool->num_kv_heads * kv;
                    long_min = std::min(long_min, kv);
                    long_max = std::max(long_max, kv);
                    pairs_long += rows_total * kv;
                    pairs_long_tiles += tiles * kTileRows * kv;
                }
                keys += tiles * pool->num_kv_heads * kv;
                longest = std::max(longest, kv);
            }
        }
        int64_t chunk = (keys + tune.split_target - 1) / std::max(tune.split_target, 1);
        chunk = std::max<int64_t>(chunk, tune.min_split_keys);
        if (items >= tune.split_target && pairs_tile * 10 >= pairs_all * 9 && longest <= 2 * chunk)
            tune_batch.tile_min_keys = tune.tile_batch_min_keys;
        else if (long_items > 0 && long_items < kTileMinItems) {
            const bool minority = pairs_long < pairs_all - pairs_long;
            if (!minority || long_items < kTileMinItemsBeside || long_keys < kTileKeysBeside) {
                // slots that the 128-row kernel's list of the same tiles fills, cut to run at once
                // (where lengths differ the cut finds one that fills them)
                const int64_t wide_parts = kWideSlots / (2 * long_items) * (2 * long_items);
                const bool idle = wide_parts * 8 <= kWideSlots * 7 &&
                                  (long_max - long_min) * 8 <= long_max;
                int64_t limit = kTileKeysMixed;
                if (pairs_long_tiles >= pairs_all - pairs_all / 50)
                    limit = idle ? kTileKeysIdle : kTileKeysAlone;
                if (long_keys < limit)
                    tune_batch.tile_min_keys = 0;
                else
                    plan->tile_scales_scores = true;
            }
        }
    }
    bool all_wide = false;
    if (tune.unify) {
        int64_t wide_steps = 0, small_steps = 0;
        for (int32_t r = 0; r < num_reqs; ++r) {
            const int64_t n = q_lens[r], c = ctx_lens[r];
            if (n == 0) continue;
            const int64_t rows_total = n * G;
            if (rows_total >= tune.wide_min_rows) {
                for (int64_t rb = 0; rb < rows_total; rb += kWideRows) {
                    const int64_t last = (std::min<int64_t>(rows_total, rb + kWideRows) - 1) / G;
                    wide_steps += (c + last + 1 + kKvBlock - 1) / kKvBlock;
                }
            } else {
                small_steps += (c + n + kKvBlock - 1) / kKvBlock;
            }
        }
        all_wide = wide_steps > 0 &&
                   small_steps * (int64_t)pool->num_kv_heads <= (int64_t)tune.unify_max_steps;
    }
    {
        // capacity for the item lists, so that filling them does not reallocate
        size_t n_narrow = 0, n_wide = 0;
        for (int32_t r = 0; r < num_reqs; ++r) {
            const int64_t rows_total = (int64_t)q_lens[r] * G;
            if (rows_total == 0) continue;
            const bool big = rows_total >= tune.wide_min_rows;
            const size_t tiles = (size_t)((rows_total + (big ? kWideRows : kNarrowRows) - 1) /
                                          (big ? kWideRows : kNarrowRows));
            (big || all_wide ? n_wide : n_narrow) += tiles * (size_t)pool->num_kv_heads;
        }
        plan->narrow.reserve(n_narrow);
        plan->wide.reserve(n_wide);
    }
    // K/V of all units, and of the units of a kernel that read theirs once or, in several items,
    // more than once
    int64_t kv_bytes = 0, wide_once = 0, wide_shared = 0, narrow_once = 0, narrow_shared = 0;
    for (int32_t r = 0; r < num_reqs; ++r) {
        const int32_t n = q_lens[r], c = ctx_lens[r];
        if (n == 0) continue;
        const int32_t rows_total = n * G;
        const int64_t unit_bytes = 4 * ((int64_t)c + n) * pool->num_kv_heads * pool->head_dim;
        kv_bytes += unit_bytes;
        // a unit whose rows are all in full tiles of the 256-row kernel has none left for the others
        const bool tiled = use_tile256(pool, tune_batch, rows_total, (int64_t)c + n);
        if (!tiled || rows_total % kTileRows != 0) {
            if (rows_total >= tune.wide_min_rows || all_wide)
                (rows_total <= kWideRows ? wide_once : wide_shared) += unit_bytes;
            else
                (rows_total <= kNarrowRows ? narrow_once : narrow_shared) += unit_bytes;
        }
        for (int32_t hk = 0; hk < pool->num_kv_heads; ++hk) {
            WorkItem w;
            std::memset(&w, 0, sizeof w);
            w.req = r;
            w.kv_head = hk;
            w.kv_begin = 0;
            w.split_index = 0;
            w.split_count = 1;
            w.partial_base = -1;
            w.q_row0 = plan->q_start[r];
            w.ctx = c;
            const bool use_wide = rows_total >= tune.wide_min_rows || all_wide;
            const int32_t tile = use_wide ? kWideRows : kNarrowRows;
            w.alone = rows_total <= kWideRows;
            // long units: their full 256-row tiles go to the 256-row kernel, the rest as usual
            int32_t rb = 0;
            if (tiled) {
                for (; rb + kTileRows <= rows_total; rb += kTileRows) {
                    w.row_begin = rb;
                    w.row_count = kTileRows;
                    w.kv_end = c + (rb + kTileRows - 1) / G + 1;
                    plan->tile256.push_back(w);
                }
            }
            for (; rb < rows_total; rb += tile) {
                w.row_begin = rb;
                w.row_count = std::min(tile, rows_total - rb);
                const int32_t last_token = (rb + w.row_count - 1) / G;
                w.kv_end = c + last_token + 1;  // causal limit of the tile's last row
                (use_wide ? plan->wide : plan->narrow).push_back(w);
            }
        }
    }
    int64_t slots = 0;
    const bool wide_rows = pool->head_dim == 128;
    const CutRule narrow_rule = {
        kNarrowSlots, wide_rows ? kNarrowSlots * 5 / 4 : 0, kNarrowSlots, 25, false,
        wide_rows ? 16 : (int64_t)plan->narrow.size() > kNarrowSlots ? 12 : 9, 0, true};
    const CutRule wide_rule = {kWideSlots, kFewWideItems, kFewWideItems, 100, true,
                               wide_rows ? 31 : 16, wide_rows ? kCUs : 0, false};
    plan->narrow_two_terms =
        split_items(plan->narrow, plan->combine, slots, tune, &narrow_rule, pool->head_dim);
    plan->wide_renews =
        split_items(plan->wide, plan->combine, slots, tune, &wide_rule, pool->head_dim);
    plan->wide_streams = kv_bytes > kStreamKvBytes && wide_once * 3 >= wide_shared;
    plan->narrow_streams = narrow_once > narrow_shared * 4;
    split_items(plan->tile256, plan->combine, slots, tune, nullptr, pool->head_dim,
                kTileMaxKeys);
    if (slots > INT32_MAX / 2) {
        delete plan;
        return PV_ERR_OUT_OF_RANGE;
    }
    order_items(plan->narrow, tune.xcds, 0);
    order_items(plan->wide, tune.xcds, tune.even_cus ? kWideSlots : 0);
    order_items(plan->tile256, tune.xcds, 0);
    plan->partial_slots = slots;
    int64_t merge_rows = 0;
    for (const CombineItem &c : plan->combine) merge_rows += c.row_count;
    size_t chunks = 0;
    for (const CombineItem &c : plan->combine) {
        const int32_t rows = 8 / combine_groups(c.split_count, merge_rows);
        chunks += (size_t)((c.row_count + rows - 1) / rows);
    }
    plan->combine_chunks.reserve(chunks);
    for (size_t i = 0; i < plan->combine.size(); ++i) {
        CombineItem &c = plan->combine[i];
        c.groups = combine_groups(c.split_count, merge_rows);
        for (int32_t r0 = 0; r0 < c.row_count; r0 += 8 / c.groups)
            plan->combine_chunks.push_back(CombineChunk{(int32_t)i, r0});
    }
    // workspace: fp32 partial outputs [slots][D], then (running max, running sum) [slots][2]
    plan->workspace_bytes = (size_t)slots * (size_t)(pool->head_dim + 2) * sizeof(float);
    build_image(plan);
    *out = plan;
    return PV_OK;
}

DeviceLists lists_at(const pv_plan *plan, const void *base)
{
    const unsigned char *b = static_cast<const unsigned char *>(base);
    DeviceLists d;
    d.ctx_lens = reinterpret_cast<const int32_t *>(b + plan->image_off[0]);
    d.q_lens = reinterpret_cast<const int32_t *>(b + plan->image_off[1]);
    d.q_start = reinterpret_cast<const int32_t *>(b + plan->image_off[2]);
    d.combine_chunks = reinterpret_cast<const CombineChunk *>(b + plan->image_off[3]);
    d.narrow = reinterpret_cast<const WorkItem *>(b + plan->image_off[4]);
    d.wide = reinterpret_cast<const WorkItem *>(b + plan->image_off[5]);
    d.tile256 = reinterpret_cast<const WorkItem *>(b + plan->image_off[6]);
    d.combine = reinterpret_cast<const CombineItem *>(b + plan->image_off[7]);
    d.append_groups = reinterpret_cast<const AppendGroup *>(b + plan->image_off[8]);
    return d;
}

}  // namespace pv

// ---------------------------------------------------------------------------------------------
// C ABI: the host-only entry points
// ---------------------------------------------------------------------------------------------
extern "C" {

const char *pv_status_string(pv_status s)
{
    switch (s) {
    case PV_OK: return "ok";
    case PV_ERR_INVALID_ARG: return "invalid argument";
    case PV_ERR_UNSUPPORTED: return "unsupported configuration";
    case PV_ERR_OUT_OF_RANGE: return "length or index out of range";
    case PV_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case PV_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

size_t pv_pool_bytes(const pv_pool_desc *pool)
{
    if (!pv::pool_desc_valid(pool, nullptr)) return 0;
    return (size_t)pool->num_pages * pool->num_kv_heads * pool->page_size * pool->head_dim * 2u;
}

int64_t pv_pool_k_offset(const pv_pool_desc *pool, int32_t page, int32_t head, int32_t slot,
                         int32_t d)
{
    if (!pv::pool_desc_valid(pool, nullptr)) return -1;
    if (page < 0 || page >= pool->num_pages || head < 0 || head >= pool->num_kv_heads ||
        slot < 0 || slot >= pool->page_size || d < 0 || d >= pool->head_dim)
        return -1;
    const int64_t tile = (int64_t)page * pool->num_kv_heads + head;
    const int64_t chunks = pool->head_dim / 8;
    return ((tile * chunks + d / 8) * pool->page_size + slot) * 8 + d % 8;
}

int64_t pv_pool_v_offset(const pv_pool_desc *pool, int32_t page, int32_t head, int32_t slot,
                         int32_t d)
{
    if (!pv::pool_desc_valid(pool, nullptr)) return -1;
    if (page < 0 || page >= pool->num_pages || head < 0 || head >= pool->num_kv_heads ||
        slot < 0 || slot >= pool->page_size || d < 0 || d >= pool->head_dim)
        return -1;
    const int64_t tile = (int64_t)page * pool->num_kv_heads + head;
    const int64_t groups = pool->page_size / 8;
    return ((tile * groups + slot / 8) * pool->head_dim + d) * 8 + slot % 8;
}

pv_status pv_plan_create(const pv_pool_desc *pool, int32_t num_q_heads, const int32_t *ctx_lens,
                         const int32_t *q_lens, int32_t num_reqs, int32_t max_pages_per_req,
                         pv_plan **plan)
{
    return pv::build_plan(pool, num_q_heads, ctx_lens, q_lens, num_reqs, max_pages_per_req,
                          pv::default_tuning(), plan);
}

int32_t pv_plan_total_q(const pv_plan *plan) { return plan ? plan->total_q : -1; }

const int32_t *pv_plan_q_start(const pv_plan *plan)
{
    return plan ? plan->q_start.data() : nullptr;
}

size_t pv_plan_workspace_bytes(const pv_plan *plan) { return plan ? plan->workspace_bytes : 0; }

size_t pv_plan_device_bytes(const pv_plan *plan) { return plan ? plan->image.size() : 0; }

int32_t pv_plan_owns_device_memory(const pv_plan *plan)
{
    return plan ? (plan->d_owned != nullptr ? 1 : 0) : -1;
}

int32_t pv_plan_num_work_items(const pv_plan *plan, int32_t kind)
{
    if (!plan) return -1;
    switch (kind) {
    case 0: return (int32_t)plan->narrow.size();
    case 1: return (int32_t)plan->wide.size();
    case 2: return (int32_t)plan->combine.size();
    case 3: return (int32_t)plan->tile256.size();
    }
    return -1;
}

int32_t pv_plan_kernel_variants(const pv_plan *plan)
{
    if (!plan) return -1;
    return (plan->narrow_two_terms ? 1 : 0) | (plan->narrow_streams ? 2 : 0) |
           (plan->wide_renews ? 4 : 0) | (plan->wide_streams ? 8 : 0) |
           (plan->tile_scales_scores ? 16 : 0);
}

pv_status pv_plan_work_item(const pv_plan *plan, int32_t kind, int32_t index, int32_t out[8])
{
    if (!plan || !out || index < 0) return PV_ERR_INVALID_ARG;
    if (kind == 0 || kind == 1 || kind == 3) {
        const std::vector<pv::WorkItem> &v =
            kind == 0 ? plan->narrow : kind == 1 ? plan->wide : plan->tile256;
        if ((size_t)index >= v.size()) return PV_ERR_INVALID_ARG;
        const pv::WorkItem &w = v[index];
        const int32_t f[8] = {w.req, w.kv_head, w.row_begin, w.row_count,
                              w.kv_begin, w.kv_end, w.split_index, w.split_count};
        std::memcpy(out, f, sizeof f);
        return PV_OK;
    }
    if (kind == 2) {
        if ((size_t)index >= plan->combine.size()) return PV_ERR_INVALID_ARG;
        const pv::CombineItem &c = plan->combine[index];
        const int32_t f[8] = {c.req, c.kv_head, c.row_begin, c.row_count, 0, 0, 0, c.split_count};
        std::memcpy(out, f, sizeof f);
        return PV_OK;
    }
    return PV_ERR_INVALID_ARG;
}

pv_status pv_plan_check_page_table(const pv_plan *plan, const int32_t *page_table,
                                   int32_t check_append_unique)
{
    if (!plan) return PV_ERR_INVALID_ARG;
    if (plan->num_reqs > 0 && !page_table) return PV_ERR_INVALID_ARG;
    const int32_t P = plan->pool.page_size;
    std::unordered_set<int64_t> seen;
    for (int32_t r = 0; r < plan->num_reqs; ++r) {
        const int32_t n = plan->q_lens[r], c = plan->ctx_lens[r];
        if (n == 0) continue;
        const int64_t pages = ((int64_t)c + n + P - 1) / P;
        const int32_t *row = page_table + (int64_t)r * plan->max_pages_per_req;
        for (int64_t lp = 0; lp < pages; ++lp)
            if (row[lp] < 0 || row[lp] >= plan->pool.num_pages) return PV_ERR_OUT_OF_RANGE;
        if (check_append_unique) {
            for (int32_t j = 0; j < n; ++j) {
                const int64_t t = (int64_t)c + j;
                const int64_t key = (int64_t)row[t / P] * P + t % P;
                if (!seen.insert(key).second) return PV_ERR_INVALID_ARG;
            }
        }
    }
    return PV_OK;
}

pv_status pv_rope_table(double base, int32_t head_dim, int32_t max_pos, float *table)
{
    if (!(base > 0.0) || head_dim <= 0 || head_dim % 2 != 0 || max_pos < 0 || !table)
        return PV_ERR_INVALID_ARG;
    const int32_t half = head_dim / 2;
    std::vector<double> theta((size_t)half);
    for (int32_t i = 0; i < half; ++i) theta[(size_t)i] = std::pow(base, -2.0 * i / head_dim);
    for (int64_t t = 0; t < max_pos; ++t) {
        float *row = table + t * head_dim;
        for (int32_t i = 0; i < half; ++i) {
            const double angle = (double)t * theta[(size_t)i];
            row[i] = (float)std::cos(angle);
            row[half + i] = (float)std::sin(angle);
        }
    }
    return PV_OK;
}

double pv_cost_model(const int32_t *ctx_points, const double *attn_cost, int32_t n, double c_other,
                     int32_t l)
{
    if (n <= 0) return c_other;
    if (!ctx_points || !attn_cost) return std::nan("");
    if (n == 1) return attn_cost[0] + c_other;
    // segment whose right end is the first profiled point >= l (clamped to the outer segments)
    const int32_t *hi = std::lower_bound(ctx_points + 1, ctx_points + n - 1, l);
    const int32_t k = (int32_t)(hi - ctx_points) - 1;
    const double t = ((double)l - ctx_points[k]) / ((double)ctx_points[k + 1] - ctx_points[k]);
    return attn_cost[k] + t * (attn_cost[k + 1] - attn_cost[k]) + c_other;
}

pv_status pv_retention_order(const double *cost, const double *idle_time, int32_t n,
                             int32_t *order_out)
{
    if (n < 0 || (n > 0 && (!cost || !idle_time || !order_out))) return PV_ERR_INVALID_ARG;
    for (int32_t i = 0; i < n; ++i)
        if (!(idle_time[i] > 0.0)) return PV_ERR_INVALID_ARG;
    std::iota(order_out, order_out + n, 0);
    std::stable_sort(order_out, order_out + n, [&](int32_t a, int32_t b) {
        return cost[a] / idle_time[a] < cost[b] / idle_time[b];
    });
    return PV_OK;
}

}  // extern "C"
