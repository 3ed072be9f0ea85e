// Internal: host-side batch plan shared by the API file and the kernel launchers.
#pragma once

#include <cstdint>
#include <vector>

#include "pv.h"

namespace pv {

// One unit of kernel work.  A "row" is a (new token, query head within the GQA group) pair of one
// (request, KV head): row = token * G + g, so the rows of one KV head that can share a K/V tile
// are contiguous and ordered by token (which keeps the causal limit monotone in the row index).
struct WorkItem {
    int32_t req;
    int32_t kv_head;
    int32_t row_begin;    // first row of the item
    int32_t row_count;    // rows in the item
    int32_t kv_begin;     // first logical KV position (multiple of 32 unless 0)
    int32_t kv_end;       // one past the last logical KV position any row of the item may see
    int32_t split_index;  // which part of the KV range this is
    int32_t split_count;  // 1 = writes `out` directly, >1 = writes a partial result
    int32_t partial_base; // first workspace row slot of this item (split_count > 1), else -1
    int32_t q_row0;       // q_start[req]
    int32_t ctx;          // ctx_lens[req]
    // 128-row kernel: the reference maximum is renewed every so many blocks (0 = never), where a
    // part would begin if the KV range were cut into about split_target parts.  A probability is
    // rounded to 16 bits unless it is the reference's own, which is exactly 1, so that fewer parts
    // alone would mean results further from those in 64 bits.  Error against that cut's, without
    // and with renewal, and time of the attention call: 10 requests, 128 tokens over 1000, 40/40
    // heads, bf16, whole instead of in three parts +0.77 % / 0.00 %, 51.1 / 51.0 us (the three
    // parts take 85); 6 of 50 tokens over 900, 64/8 heads, whole instead of in four +1.32 % / 0.00
    // %, 28.5 / 30.0 us.
    uint32_t renew_blocks : 31;
    // 128-row kernel: no other item of this (request, KV head) reads this item's K/V (its rows are all
    // of the unit's); whether another request does, only the page table tells
    uint32_t alone : 1;
};
static_assert(sizeof(WorkItem) == 48, "WorkItem is read by the kernels as 12 int32");

// Merge of the partial results of one split item.
struct CombineItem {
    int32_t req;
    int32_t kv_head;
    int32_t row_begin;
    int32_t row_count;
    int32_t partial_base; // slot of split 0, row 0; split s, row i lives at base + s*row_count + i
    int32_t split_count;
    int32_t q_row0;
    int32_t groups;       // thread groups of the merge that share a row (combine_groups)
};
static_assert(sizeof(CombineItem) == 32, "CombineItem is read by the kernels as 8 int32");

// How many of a merge workgroup's eight thread groups share one row, by the number of parts to
// add: with few parts one group reads them all, with many the reads are spread over the groups, so
// that nobody reads more than four parts after one another up to 32 of them.  But only as long as
// that is no more than kMergeGroups workgroups for the rows of the whole merge: more rows than
// that keep the GPU busy by themselves, and every further group of a row reads the row's (max,
// sum) pairs again.  Attention call, with and without that limit: 2 prompts of 256 tokens over 2 K
// and 16 K, 64/8 heads, 210 and 219 us; 128 tokens over 16 K, 40/40 heads, 84.8 and 88.4; 200 over
// 30 K, 32/8 heads, 78.3 and 81.3; 56 generation steps (288 items of 8 rows) 66.7 and 67.2; 4 of
// them (32 items) 19.2 either way, 21.0 with one group a row.  Limits of 1024 and 2048: the same
// within 1 us.
constexpr int kMergeGroups = 512;
constexpr int combine_groups(int split_count, int64_t merge_rows)
{
    int groups = split_count >= 16 ? 8 : split_count >= 8 ? 4 : split_count >= 4 ? 2 : 1;
    while (groups > 1 && merge_rows * groups > 8 * kMergeGroups) groups /= 2;
    return groups;
}

// 8 / CombineItem::groups rows of one combine item: the unit of work of one merge workgroup.
struct CombineChunk {
    int32_t item;  // index into the combine list
    int32_t row0;  // first row (relative to the item) of the chunk
};
static_assert(sizeof(CombineChunk) == 8, "CombineChunk is read by the kernel as 2 int32");

// Up to 8 consecutive new tokens of one request that fall into the same 8-slot group of a page
// (the V pool keeps 8 consecutive slots of one head dimension in one 16-byte run).
struct AppendGroup {
    int32_t req;
    int32_t t_begin;  // logical position of the first token of the group
    int32_t count;    // 1..8 tokens
    int32_t q_row;    // row of that first token in k_new / v_new
};
static_assert(sizeof(AppendGroup) == 16, "AppendGroup is read by the kernel as 4 int32");

// Append and rotary kernels: new rows of more bytes than this, the L2 caches of all XCDs together,
// are read with the streaming hint, because they are read once and what is written (K/V pages,
// rotated queries) is read by the attention that follows: 53 MB (2600 tokens, 40 heads), append
// and attention 187.0 -> 184.7 us (219 -> 217 with the kernel that writes the rows in front); 7 K
// tokens with the rotary embedding see pick_rope.  A smaller batch finds its rows in a cache when
// they come from the kernel before: 14 MB (2736 tokens, 10 heads) 64.5 us, 67.3 with the hint; 4
// generation steps with the rotary embedding 26.0 and 26.3.  Streaming the stores too is slower
// (first prompts 193 -> 204 us).
constexpr int64_t kStreamBytes = 32 << 20;

// Requests with new tokens that the append takes as a kernel argument, and how many one launch
// takes (2 KB of arguments).  Request i of the launch has the append groups group0[i] .. group0[i
// + 1] - 1.
struct AppendReq {
    int32_t req;
    int32_t t_begin;  // logical position of its first new token
    int32_t count;    // new tokens (at least one)
    int32_t q_row;    // row of the first one in k_new / v_new
    int32_t group0;
};
constexpr int kAppendReqs = 96;
struct AppendReqs {
    int32_t n;
    int32_t groups;  // of all n requests
    AppendReq r[kAppendReqs];
};
// append groups (8-slot runs touched) of `count` new tokens from position t_begin on
constexpr int64_t append_group_count(int64_t t_begin, int64_t count)
{
    return count > 0 ? (t_begin + count + 7) / 8 - t_begin / 8 : 0;
}

// 128-row kernel: the K/V of a unit whose rows fit one item is read once.  With the streaming hint
// it does not push out of the L2 caches what the row tiles of larger units read together: 0.4 * n
// prompts of 40-128 tokens and 0.6 * n generation steps over 500-1500, 40/40 heads, whole step
// without and with it 70.2 / 62.5 us (11 requests, 230 MB of K/V), 86.8 / 75.4 (17), 140.4 / 117.8
// (27), 219 / 189 (46); 119 requests, 32/8 heads, head size 64, 61.9 / 56.1.  Not for small batches,
// whose K/V may still be in the last-level cache (256 MB) from the kernels before: of three batches
// in turn 45.1 / 43.3 us at 107 MB each, 20.2 / 20.4 at 43, 23.9 / 26.1 at 58 (40/10 heads).  Not for
// units of more tiles (the hint costs them 17 % at two tiles over 300-900 keys, 10-13 % at four to
// eight), and not where less than a quarter of the bytes is read once: an instance of the kernel
// with both kinds of copies is up to 2 % slower on the others.
// Requests may share pages, whose K/V the hint pushes out between their readers: the kernel looks at
// the page table for that (see attn_wide_kernel), where three quarters of an item's range are shared
// and contexts are long.  Always with the hint, never, and by the table: 24 prompts of 100 tokens over
// a common prefix of 3 K, 40/40 heads, 221.5 / 204.1 / 204.5 us, over two prefixes in turn 236.4 /
// 210.0 / 206.6; 8 such prompts and 20 generation steps 181.5 / 148.5 / 150.8; 40 of 30 over 3 K, 40/10
// heads, 101.3 / 93.7 / 94.1; the same batches over K/V of their own 307.3 / 328.6 / 307.6, 318.6 / 333.0
// / 318.8, 121.1 / 130.8 / 121.4.  Twelve prompts of 100 tokens, always and never: of 3 K keys 60 % shared
// 116.2 / 125.2 us, 75 % 111.3 / 110.4, 85 % 104.4 / 102.5; of 500 keys 83 % 34.3 / 35.4, 93 % 33.4 / 35.4.
constexpr int64_t kStreamKvBytes = 96 << 20;
constexpr int kSharedMinCtx = 640;  // cached tokens from which the kernel looks for shared pages

constexpr int kNarrowRows = 16;  // rows per item of the bandwidth-oriented kernel
constexpr int kWideRows = 128;   // rows per item of the matrix-core kernel (4 waves x 32 rows)
constexpr int kTileRows = 256;   // rows per item of the 256-row matrix-core kernel (4 waves x 64)
// The 256-row kernel takes a batch's long units only if they have this many tiles, or fewer with this
// many keys over all tiles.  Few tiles are cut into about 1024 parts, whose rows, twice as many as
// the 128-row kernel's, the merge has to read: 60-80 us more, whatever the number of keys; in return a
// million tile keys take 100-115 us in place of 120-140.  So what counts is their product, and how well
// the other kernel's list fills its slots.  The few tiles that do go there have their scores scaled in
// fp32 (4 % more time than with scaled queries): 80 parts in 100 of the scaled queries' distance from
// 64 bits, the same as the 128-row kernel's.  Whole step with the 128-row and with the 256-row kernel,
// in microseconds, by million tile keys:
//  * nothing but these tiles: 2.0 (96 tiles) 257 / 301, 2.5 (120) 368 / 384, 3.9 (120) 585 / 547, 5.9
//    (96) 753 / 783, 11.5 (96) 1386 / 1407, 7.7 (120) 1092 / 993.  Where the 128-row kernel's list leaves
//    an eighth of the slots idle the 256-row kernel is ahead sooner: 2.3 (112) 314 / 328, 3.3 (160) 453
//    / 434, 3.6 (112) 483 / 472, 5.2 (160) 703 / 643, 10.3 (160) 1371 / 1200, 19 (160) 2643 / 2224.
//  * remaining rows or other requests beside them, which with the 256-row kernel are a launch of their
//    own: 2.4 (120) 428 / 440, 3.9 (120) 665 / 640, 7.7 (120) 1308 / 1154; with scaled queries 2.8 (170)
//    600 / 693, 4.7 (80) 668 / 689, 4.9 (90) 659 / 694, 5.7 (152) 837 / 797, 7.3 (160) 1146 / 1082, 8.0
//    (80) 1247 / 1274, 9.0 (90) 1537 / 1332, 11.4 (130) 1713 / 1730, 13.2 (150) 2975 / 2440.
//  * at least kTileMinItemsBeside tiles of long units that are less than half of the batch's pairs:
//    1.4 (112) 509 / 582, 1.6 (160) 486 / 560, 2.4 (144) 828 / 881, 2.6 (128) 687 / 757, 3.6 (176) 1417 /
//    1464, 5.3 (120) 1585 / 1540.  The limit is lower than that asks for: one prompt of 512 tokens over
//    20 K keys among shorter ones (the 2.6) has always gone to the kernel for long units.
// From kTileMinItems tiles on the 256-row kernel's list is hardly cut (186 tiles 528 / 536, 192 485 /
// 543, 288 844 / 949, here with the 256-row kernel first); those with many remaining rows would still
// gain by the other kernel (230 with a fifth of them 1004 / 856; 216 with as many 668 / 696 would not).
constexpr int kTileMinItems = 180;
constexpr int64_t kTileKeysAlone = 6000000;
constexpr int64_t kTileKeysIdle = 3500000;
constexpr int64_t kTileKeysMixed = 7000000;
constexpr int kTileMinItemsBeside = 112;
constexpr int64_t kTileKeysBeside = 2500000;
constexpr int kCUs = 256;
// Workgroups that run at once on the CUs: two of the narrow kernel on each (212-216 registers
// a lane; head size 64 has room for three, but 512 parts are ahead of more: 4 generation steps,
// 32/8 heads, 13.4 us with 512 parts, 14.2 with 656), three of the 128-row kernel (161-163
// registers, 48 KiB of LDS).
constexpr int kNarrowSlots = 512;
constexpr int kWideSlots = 768;
constexpr int kItemSetUp = 96;  // keys that take an item as long as its set-up and its result
constexpr int kSplitTarget = 1024;
constexpr int kFewWideItems = 512;  // shorter lists of the 128-row kernel are cut to fill the GPU
constexpr int kKvBlock = 32;     // keys per inner step (two pages)
constexpr float kLazyLog2 = 8.f;  // matrix-core kernels: the reference maximum of a row may lag the
                                  // true one by this many powers of 2
constexpr int kTileMaxPages = 8192;  // page ids an item of the 256-row kernel may span (it keeps
                                     // them in LDS): its KV range is at most 16 times that
constexpr int kTileMaxKeys = kTileMaxPages * 16 - kKvBlock;

// No list has more parts of cut items than this times the target (see split_items): with a chunk
// of a target-th of the keys, `target` parts and one more for each cut item, of which there are no
// more than `target`; the other cuts take a slots-th or a long_share-th of the keys for their
// chunk or more, and no more items are cut than there are in a short list or four fifths of that
// share.
constexpr int kPartsPerTarget = 2;
static_assert(kNarrowSlots * 9 / 5 <= kPartsPerTarget * kSplitTarget &&
                  kFewWideItems * 9 / 5 <= kPartsPerTarget * kSplitTarget &&
                  kWideSlots + kFewWideItems <= kPartsPerTarget * kSplitTarget,
              "pv_attn_workspace_bytes counts on it");

// Where the lists of a plan live on a device: pointers into one buffer laid out as the plan's
// host image (see pv_plan::image).  The launchers take the lists through this, so that the same
// plan can run from its own upload, from a buffer of the caller's, or from the library's static
// scratch array.
struct DeviceLists {
    const int32_t *ctx_lens, *q_lens, *q_start;
    const CombineChunk *combine_chunks;
    const WorkItem *narrow, *wide, *tile256;
    const CombineItem *combine;
    const AppendGroup *append_groups;
};

struct Tuning {
    int32_t split_target;    // cut a list that is shorter into about this many work items
    bool split_by_hand;      // whatever the kernel (see split_items)
    int32_t min_split_keys;  // items are cut from twice this many keys on, by parts of at least this
                             // many before they are evened out (which leaves at least half of it,
                             // and less in an item's last part)
    int32_t wide_min_rows;   // (request, KV head) units with n*G >= this use the matrix-core
                             // kernel; smaller ones are cut into 16-row items of the narrow kernel
    int32_t xcds;            // L2 domains the work list is interleaved over
    int32_t unify;           // 1: a batch with matrix-core work sends its small units to that
                             // kernel too (one attention launch, not two) unless they are many
    int32_t unify_max_steps; // "many": more than this many 32-key steps over all small units and
                             // KV heads (then the bandwidth-oriented kernel is worth its launch)
    int32_t tile_min_keys;   // (request, KV head) units with at least 256 rows and at least this
                             // many keys send their full 256-row tiles to the 256-row kernel
                             // (0 switches that kernel off)
    int32_t tile_batch_min_keys;  // the lower limit that applies instead when nearly all of a
                             // batch's work qualifies under it and its items need no splitting
                             // (0: no such rule; it is off when tile_min_keys is set by hand)
    bool even_cus;           // order lists that run at once by what shares a CU (see pair_up); a plan
                             // for one launch alone does not: 6-9 us of host time for 1-5 us of it
};

}  // namespace pv

struct pv_plan {
    pv_pool_desc pool;
    int32_t num_q_heads;
    int32_t group;  // G
    int32_t num_reqs;
    int32_t max_pages_per_req;
    int32_t total_q;
    std::vector<int32_t> ctx_lens, q_lens, q_start;
    std::vector<pv::WorkItem> narrow, wide, tile256;
    std::vector<pv::CombineItem> combine;
    std::vector<pv::AppendGroup> append_groups;
    std::vector<pv::CombineChunk> combine_chunks;
    int64_t partial_slots;  // workspace row slots
    // Where an item gets fewer parts than the cut into about split_target parts gives it (see
    // split_items): the narrow kernel takes its probabilities in two 16-bit terms, items of the
    // 128-row kernel renew their reference
    bool narrow_two_terms, wide_renews;
    // K/V with the streaming hint: items of the 128-row kernel that are `alone` and share no pages;
    // all of the narrow kernel's
    bool wide_streams, narrow_streams;
    // 256-row kernel: no scaled queries (see kTileMinItems)
    bool tile_scales_scores;
    size_t workspace_bytes;

    // Host image of everything the kernels read from the plan: the nine arrays above, each at a
    // 256-byte aligned offset (image_off, in the order of pv::DeviceLists).  Built with the plan,
    // copied to a device by pv_plan_upload / pv_plan_upload_to / the no-allocation launch.
    std::vector<unsigned char> image;
    size_t image_off[9];

    // device copy (set by pv_plan_upload or pv_plan_upload_to)
    bool uploaded;
    int device;
    void *d_owned;        // device memory the plan allocated itself (pv_plan_upload), else null
    pv::DeviceLists dev;  // valid while `uploaded`

    // optional per-kernel timing: events[2*kind], events[2*kind+1] bracket kernel `kind`
    bool timing;
    void *events[10];
    bool event_used[5];
};

namespace pv {
// the lists of a plan image that was copied to `base`
DeviceLists lists_at(const pv_plan *plan, const void *base);
bool pool_desc_valid(const pv_pool_desc *p, pv_status *why);
Tuning default_tuning();
// what every plan demands of a batch; *total_q = its new tokens
pv_status check_batch(const pv_pool_desc *pool, int32_t num_q_heads, const int32_t *ctx_lens,
                      const int32_t *q_lens, int32_t num_reqs, int32_t max_pages_per_req,
                      int32_t *total_q);
pv_status build_plan(const pv_pool_desc *pool, int32_t num_q_heads, const int32_t *ctx_lens,
                     const int32_t *q_lens, int32_t num_reqs, int32_t max_pages_per_req,
                     const Tuning &tune, pv_plan **out);
}  // namespace pv
