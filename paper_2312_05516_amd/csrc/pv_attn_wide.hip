// Matrix-core attention kernel: work items of up to 128 query rows (new-prompt tokens, times the
// query heads of a GQA group) that share one KV head's K/V stream.
//
// Computes paper Eq. 2-3 with the causal rule of Section 4.4 for the rows of one item over the
// item's KV range, reading K and V through the page table: the pair of matrix products with the
// fused causal mask that Section 4.4 describes, fused flash-style so that the score matrix is
// never materialised.
//
// Mapping to gfx950.  One workgroup = 4 wavefronts = one item; wavefront w owns rows 32w..32w+31.
// The K/V page tiles of a block (two pages; four for head size 64) are copied from HBM straight
// into LDS (global_load_lds, 16 bytes per lane, fully coalesced because a (page, head) tile is
// contiguous in the pool; no register staging, no ds_write) into a ring of three stages, two
// blocks ahead of their use, and every wavefront reads its matrix-core operands from there, so a
// tile is fetched once for all 128 rows.  The pool keeps runs of 8 elements along the contracted
// dimension together, so the plain linear copy already puts the operands where 16 consecutive
// lanes read 256 consecutive bytes (no bank conflicts, no padding, no transposes).  Scores are
// produced transposed, S^T = K Q^T (v_mfma_f32_32x32x16), so each lane owns one query row (softmax
// without cross-lane traffic except one exchange for the maximum) and the probabilities are
// already the B operand of O^T += V^T P^T.  161-163 VGPRs (127-130 for head size 64) and 48 KiB of
// LDS let three workgroups share a CU, whose wavefronts overlap each other's matrix-core,
// vector-ALU and LDS phases.  One raw s_barrier per block, preceded by a wait that leaves only the
// newest loads in flight.  Blocks that touch the causal boundary or the end of the sequence run in a
// second loop, which masks the scores, so the steady-state loop has no branches and the registers
// for one kind of block at a time: room to request all V operands of a block while its scores are
// computed, into the registers that its K operands leave.  Values past the end of the sequence are
// zeroed once in LDS, not by every reader, and a row's token takes one division an item.  The running
// maximum is only moved when a new score exceeds it by more than 2^8 (softmax is shift-invariant),
// which makes rescaling the accumulator rare.
//
// What bounds it: a 32-key block of head size 128 takes 2281 cycles with three workgroups on a CU (1745
// with one or two), of which the matrix cores need 1536 and the LDS reads, by count, 1920; on random
// data the clock is at 1.78 GHz, the chip's power limit.  64 mixed requests, 64/8 heads, whole step
// 254 us, 48 of head size 64 97 us (vector ALU busy half of the time, matrix cores a third); before the
// loops were split and the operands requested ahead 262.7 and 102.7.
#include <type_traits>

#include "pv_device.h"

namespace pv {

// STREAMS: items that are `alone` and whose pages no other request shares copy with the streaming
// hint (see kStreamKvBytes).
// RENEW: some item has renew_blocks.  Lists without any keep an instantiation of their own: with the
// test for it in the loop they take 1 % longer.
template <typename T, int D, bool RENEW, bool STREAMS>
__global__ __launch_bounds__(256, 3) void attn_wide_kernel(
    const WorkItem *__restrict__ items, const uint16_t *__restrict__ q,
    const uint16_t *__restrict__ k_pages, const uint16_t *__restrict__ v_pages,
    const int32_t *__restrict__ page_table, int32_t max_pages, int32_t num_q_heads,
    int32_t num_kv_heads, int32_t group, float scale_log2e, uint32_t q_keep, uint32_t q_sign,
    uint16_t *__restrict__ out, float *__restrict__ ws_o, float *__restrict__ ws_ml,
    int32_t num_reqs)
{
    // Keys per block: 32 for head size 128; 64 for head size 64, where 32 keys are only 8
    // matrix-core instructions of a wavefront against about 70 of the vector ALU, a barrier, a
    // test for the maximum and two LDS round trips.  48 requests over 0.1-3 K tokens, 32/8 heads:
    // 108.8 -> 104.1 us whole step.  (Head size 128 would need 231 registers a lane for 64 keys,
    // two workgroups per CU.)
    constexpr int PAGES = D == 128 ? 2 : 4;
    constexpr int BK = 16 * PAGES;
    constexpr int NT = BK / 32;                 // 32-key score tiles of a block
    constexpr int KS = D / 16;                  // k-steps of S^T = K Q^T
    constexpr int NB = D / 32;                  // 32-wide blocks of d in O^T
    constexpr int TILE_BYTES = 16 * D * 2;      // one (page, head) tile
    constexpr int HALF_BYTES = PAGES * TILE_BYTES;  // K (or V) part of a stage
    constexpr int PASSES = HALF_BYTES / 4096;   // 16-byte copies per lane for K (same for V)
    constexpr int STAGES = 3;
    typedef typename T::vec8 vec8;
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGES][2 * HALF_BYTES];

    const WorkItem it = items[blockIdx.x];
    const int lane = lane_id();
    const int w = wave_id();
    const int q32 = lane & 31;
    const int h = lane >> 5;

    const RowMap rows(it.row_begin, group);
    // wavefront-uniform limits: below unmasked_end nothing is masked for this wavefront's rows
    // (and no slot is past the end); at or beyond wave_end nothing is visible to them
    const int wave_rows = it.row_count - 32 * w;  // may be <= 0
    int unmasked_end = it.ctx + rows.token(32 * w) + 1;
    if (unmasked_end > it.kv_end) unmasked_end = it.kv_end;
    unmasked_end = __builtin_amdgcn_readfirstlane(unmasked_end);
    int wave_end = 0;
    if (wave_rows > 0) {
        wave_end = it.ctx + rows.token(32 * w + (wave_rows < 32 ? wave_rows : 32) - 1) + 1;
        if (wave_end > it.kv_end) wave_end = it.kv_end;
        wave_end = __builtin_amdgcn_readfirstlane(wave_end);
    }

    vec8 qf[KS];
    {
        const bool valid = 32 * w + q32 < it.row_count;
        int tok, head;
        rows.at(valid ? 32 * w + q32 : 0, tok, head);
        const uint16_t *qrow =
            q + ((int64_t)(it.q_row0 + tok) * num_q_heads + it.kv_head * group + head) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // loaded without a condition (a lane without a row reads the item's first one):
            // eight branches less in front of the page ids; 19 first prompts, 64/8 heads 33.0 ->
            // 32.5 us, 8 longer ones, 40/40 heads 181.7 -> 179.6
            const u32x4 got = load16(qrow + 16 * ks + 8 * h);
            u32x4 raw = {0u, 0u, 0u, 0u};
            if (valid) raw = got;
            raw = (raw & q_keep) ^ q_sign;
            qf[ks] = as_vec8<T>(raw);
        }
    }

    // LDS byte offsets of this lane's operands inside a stage.  S^T row i of the K operand is fed
    // with key pi(i) (bits 2 and 3 of i swapped) so that the accumulator registers of S^T, taken in
    // order, are exactly the 8 consecutive keys the P^T operand of the second product needs.
    const int key = (q32 & 0x13) | ((q32 & 4) << 1) | ((q32 & 8) >> 1);
    int k_lds = (key >> 4) * TILE_BYTES + (h * 16 + (key & 15)) * 16;  // + ks * 512
    int v_lds = HALF_BYTES + (h * D + q32) * 16;  // + page * TILE_BYTES + blk * 512
    asm volatile("" : "+v"(k_lds), "+v"(v_lds));  // one register each, not their parts

    const int32_t *pt = page_table + (int64_t)it.req * max_pages;
    const int last_pg = (it.kv_end - 1) >> 4;
    const int pg0 = it.kv_begin >> 4;
    const int nblocks = (it.kv_end - it.kv_begin + BK - 1) / BK;
    // STREAMS: whether somebody else reads an `alone` item's pages.  Looked for where three quarters of
    // them are shared: the page there, in the table rows of the 64 requests around.
    int own_page = 0, other_page = -1;
    if (STREAMS && it.alone && it.ctx >= kSharedMinCtx) {
        const int at = pg0 + (last_pg - pg0) * 3 / 4;
        const int other = max(min(it.req - 32, num_reqs - 64), 0) + lane;
        own_page = pt[at];
        if (other < num_reqs && other != it.req)
            other_page = page_table[(int64_t)other * max_pages + at];
    }
    const uint32_t lane_bytes = (uint32_t)lane * 16u;
    // asynchronous copies move bytes [w*1024, w*1024+1024) of every 4 KiB pass over the K (V) part:
    // ids of the pages that this wavefront's pieces of a block lie in (a page past the end is never
    // used, so any valid id will do)
    static_assert(PASSES == 2, "two pieces of K and two of V per wavefront and block");
    auto page_ids = [&](int b, int &id0, int &id1) {
        const int pg = pg0 + PAGES * b + w * 1024 / TILE_BYTES;
        id0 = pt[pg <= last_pg ? pg : last_pg];
        id1 = pt[pg + PAGES / 2 <= last_pg ? pg + PAGES / 2 : last_pg];
    };
    // the wavefront's pieces of a block into the stage at `stage`, lane l the 16 bytes at 16*l of a
    // piece (scalar base + lane offset); both pieces of K (V) lie at the same place of their page
    const uint64_t piece_off =
        (uint64_t)it.kv_head * TILE_BYTES + (uint32_t)(w * 1024 % TILE_BYTES);
    const unsigned char *k_src = reinterpret_cast<const unsigned char *>(k_pages) + piece_off;
    const unsigned char *v_src = reinterpret_cast<const unsigned char *>(v_pages) + piece_off;
    auto dma_block = [&](unsigned char *stage, int id0, int id1, auto stream_tag) {
        constexpr bool STREAM = decltype(stream_tag)::value;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int off = p * 4096 + w * 1024;  // wavefront-uniform
            // (a page may be larger than 4 GiB)
            const uint64_t page_off =
                (uint64_t)(uint32_t)(p ? id1 : id0) * (uint32_t)num_kv_heads * TILE_BYTES;
            lds_dma16<STREAM>(k_src + page_off, lane_bytes, stage + off);
            lds_dma16<STREAM>(v_src + page_off, lane_bytes, stage + HALF_BYTES + off);
        }
    };
    static_assert(4096 % TILE_BYTES == 0, "a pass covers whole pages");

    f32x16 o[NB];
#pragma unroll
    for (int blk = 0; blk < NB; ++blk)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[blk][v] = 0.f;
    float m_run = -INFINITY;  // reference maximum of the RAW scores (before scaling)
    float m_top = -INFINITY;  // the highest reference so far (RENEW)
    float l_run = 0.f;        // this lane's share of the running sum
    float mc = 0.f;           // m_run in the exp2 domain (0 while there is no reference yet)

    // RENEW: a renewal takes the block's own maximum as the reference also where it is lower, by no
    // more than 2^kRenewLog2 than any reference so far, so that nothing grows by more than that.
    const float renew_margin = (kLazyLog2 + kRenewLog2) / scale_log2e;
    const int renew_blocks = (int)it.renew_blocks;
    int to_renewal = renew_blocks ? renew_blocks + 1 : 0;  // a renewal where it counts to 0
    // one past the last key of the item that the lane's row may see (a part of a KV range need not
    // end at the end of a block), less 8 * h; set in front of the masked loop
    int vis_lane = 0;
    auto compute_block = [&](const unsigned char *sb, int kb0, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        u32x4 kf[NT * KS];  // K operands, requested as soon as the block is published
#pragma unroll
        for (int i = 0; i < NT * KS; ++i)
            kf[i] = *reinterpret_cast<const u32x4 *>(sb + k_lds + (i / KS) * 2 * TILE_BYTES +
                                                     (i % KS) * 512);
        f32x16 s[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) s[t][v] = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                s[t] = T::mfma32(as_vec8<T>(kf[t * KS + ks]), qf[ks], s[t]);
        // all V operands are requested while the matrix cores work on the scores, so that they have
        // arrived when the first exponentials are done
        __builtin_amdgcn_sched_barrier(0);
        u32x4 vf[PAGES * NB];
#pragma unroll
        for (int i = 0; i < PAGES * NB; ++i)
            vf[i] = *reinterpret_cast<const u32x4 *>(sb + v_lds + (i / NB) * TILE_BYTES +
                                                     (i % NB) * 512);
        __builtin_amdgcn_sched_barrier(0);
        // register v = 8*page + j of tile t  <->  key kb0 + 32*t + 16*page + 8*h + j
        if constexpr (MASKED) {
            const int seen = vis_lane - kb0;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (32 * t + 16 * (v >> 3) + (v & 7) >= seen) s[t][v] = -INFINITY;
        }
        float mx = s[0][0];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = t ? 0 : 1; v < 16; ++v) mx = fmaxf(mx, s[t][v]);
        // Lazy rescale: the reference maximum of a row only moves when a new score exceeds it by
        // more than 2^kLazyLog2 in the scaled domain (exact, because softmax is shift-invariant; the
        // probabilities just range up to 2^kLazyLog2 instead of 1).  Each lane tests the keys it
        // holds; only when some lane of the wavefront sees such a score (or has no reference yet)
        // do the two lanes of a row exchange their maxima and the accumulators get rescaled.
        float base = m_run;  // what the test for a new reference compares with: lower for a renewal
        if constexpr (RENEW) base = to_renewal == 0 ? m_top - renew_margin : m_run;
        const bool grow = m_run == -INFINITY || (mx - base) * scale_log2e > kLazyLog2;
        if (__any(grow)) {
            mx = max_halves(mx);
            const float m_new =
                (m_run == -INFINITY || (mx - base) * scale_log2e > kLazyLog2) ? mx : m_run;
            if constexpr (RENEW) {
                m_top = fmaxf(m_top, m_new);
            }
            const float m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float alpha =
                m_run == -INFINITY ? 0.f : fast_exp2((m_run - m_safe) * scale_log2e);
            mc = m_safe * scale_log2e;
            m_run = m_new;
            l_run *= alpha;
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int blk = 0; blk < NB; ++blk) o[blk] *= alpha;
            }
        }
        // page by page: the matrix-core work of a page is issued before the exponentials of the
        // next, so that inside this wavefront the two have something to overlap with
        float psum = 0.f;
#pragma unroll
        for (int pg = 0; pg < PAGES; ++pg) {
            const int t = pg / 2, v0 = 8 * (pg % 2);
            u32x4 praw;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const float p0 = fast_exp2(__builtin_fmaf(s[t][v0 + 2 * jj], scale_log2e, -mc));
                const float p1 = fast_exp2(__builtin_fmaf(s[t][v0 + 2 * jj + 1], scale_log2e, -mc));
                praw[jj] = T::pack2(p0, p1);
                psum = T::add_pair(praw[jj], psum);  // the sum of what the matrix core will see
            }
            const vec8 pf = as_vec8<T>(praw);
#pragma unroll
            for (int blk = 0; blk < NB; ++blk)
                o[blk] = T::mfma32(as_vec8<T>(vf[pg * NB + blk]), pf, o[blk]);
        }
        l_run += psum;
    };

    // prologue: blocks 0 and 1 on their way, block 0 landed and visible to everyone; the page ids of
    // the block after next are always fetched one iteration early
    int id0, id1;
    auto dma_first = [&](unsigned char *stage) {  // nobody waits for the other requests' page ids here
        if (STREAMS && it.alone)
            dma_block(stage, id0, id1, std::bool_constant<STREAMS>{});
        else
            dma_block(stage, id0, id1, std::false_type{});
    };
    page_ids(0, id0, id1);
    dma_first(smem[0]);
    if (nblocks > 1) {
        page_ids(1, id0, id1);
        dma_first(smem[1]);
    }
    page_ids(2, id0, id1);
    asm volatile("" ::: "memory");
    // the queries (loaded first) and block 0 must be there; block 1 may still be on its way
    if (nblocks > 1)
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PASSES, 0));
    else
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" : "+s"(id0), "+s"(id1)::"memory");

    // The item's blocks; `stream`: with the streaming hint on its copies from the third block on.  A
    // flow of its own for either: with both kinds of copies in one loop and a branch between them
    // batches that stream nothing are 2-4 % slower.
    auto run = [&](auto stream) {
        const int tail = it.kv_end - it.kv_begin - BK * (nblocks - 1);  // keys of the last block
        int at = 0, at2 = 2;  // stages of blocks b and b + 2
        // one block: `compute` works on its stage between the copy of the block after next and the
        // barrier that publishes the next one
        auto step = [&](int b, auto compute) {
            const bool more = b + 2 < nblocks;
            if (more) dma_block(smem[at2], id0, id1, stream);  // everyone is done with block b-1
            if constexpr (RENEW) to_renewal = (to_renewal == 0 ? renew_blocks : to_renewal) - 1;
            compute(smem[at], it.kv_begin + BK * b);
            __builtin_amdgcn_sched_barrier(0);
            page_ids(b + 3, id0, id1);
            at = at == STAGES - 1 ? 0 : at + 1;
            at2 = at2 == STAGES - 1 ? 0 : at2 + 1;
            // block b+1 (issued one iteration ago) must have landed before the barrier publishes
            // it; this iteration's own copies may stay in flight.  This wavefront's LDS reads of
            // block b must have returned too: after the barrier the others refill that stage.  They
            // have: the scheduling barrier keeps the block's last matrix-core instructions, which
            // wait for them, in front of this point.
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            if (more)
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * PASSES, 15));
            else
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 15));
            __builtin_amdgcn_s_barrier();
            // the page ids have arrived, too: said here, or the first operand of the next block would
            // be waited for together with them, which means with all other operands
            asm volatile("" : "+s"(id0), "+s"(id1)::"memory");
        };
        // Blocks that nothing is masked in for this wavefront's rows, then those that touch the
        // causal boundary or the end of the sequence: loops of their own with the same barriers
        const int unmasked = wave_end > 0 ? (unmasked_end - it.kv_begin) / BK : 0;
        int b = 0;
        for (; b < unmasked; ++b)
            step(b, [&](const unsigned char *sb, int kb0) {
                compute_block(sb, kb0, std::false_type{});
            });
        // the lane's row is worked out anew: the loop above has no register to keep it in
        int lane_again = (int)(lane_bytes >> 4);
        asm volatile("" : "+v"(lane_again));
        const int own = 32 * w + (lane_again & 31), half = lane_again >> 5;
        vis_lane = it.kv_end - 8 * half;
        if (own < it.row_count)
            vis_lane = min(it.ctx + rows.token(own) + 1, it.kv_end) - 8 * half;
        for (; b < nblocks; ++b) {
            if (b + 1 == nblocks && tail < BK) {
                zero_past_end<D>(smem[at] + HALF_BYTES, tail, 64 * w + lane_again);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            step(b, [&](const unsigned char *sb, int kb0) {
                if (kb0 < wave_end) compute_block(sb, kb0, std::true_type{});
            });
        }
    };
    if (STREAMS && it.alone && !__any(other_page == own_page))
        run(std::bool_constant<STREAMS>{});
    else
        run(std::false_type{});

    // ---- finish: every lane owns one row; the two half-waves hold partial sums ----
    int lane_again = (int)(lane_bytes >> 4);
    asm volatile("" : "+v"(lane_again));
    const int own = 32 * w + (lane_again & 31), half = lane_again >> 5;
    if (q_keep == 0) {  // a scale of zero: an infinity or a NaN among the row's queries makes it NaN
        int tok, head;
        rows.at(own < it.row_count ? own : 0, tok, head);
        const uint16_t *qrow =
            q + ((int64_t)(it.q_row0 + tok) * num_q_heads + it.kv_head * group + head) * D;
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks)
            if (any_not_finite<T>(load16(qrow + 16 * ks + 8 * half))) l_run = NAN;
    }
    const float l_tot = add_halves(l_run);
    if (it.split_count == 1) {
        // The accumulators hold 8 bytes of 32 different rows per register pair: stored from there,
        // every 16 bytes would be a request of their own to L2 (4 million of the 10 million requests
        // of a batch of 8 prompts, 7 K tokens x 40 heads).  The wavefront turns its rows round in
        // its quarter of the ring, which nobody reads any more (last barrier above), and stores
        // whole rows: 120 -> 112 us for that batch, 258 -> 252 us for a mixed batch of 64
        // requests, 64/8 heads.
        // 16 bytes of padding: the 16-byte reads have no bank conflicts; of the 8-byte writes those of
        // rows r and r + 16 meet in the same banks, about 90 cycles a wavefront and item
        constexpr int ROW_BYTES = 2 * D + 16;
        constexpr int PART = STAGES * 2 * HALF_BYTES / 4;
        static_assert(32 * ROW_BYTES + 32 * 8 <= PART, "a wavefront's rows fit its part of the ring");
        unsigned char *part = &smem[0][0] + w * PART;
        int64_t *row_off = reinterpret_cast<int64_t *>(part + 32 * ROW_BYTES);
        const float inv = 1.f / l_tot;
#pragma unroll
        for (int blk = 0; blk < NB; ++blk)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int d = 32 * blk + 8 * a + 4 * half;
                *reinterpret_cast<u32x2 *>(part + (own & 31) * ROW_BYTES + 2 * d) =
                    u32x2{T::pack2(o[blk][4 * a] * inv, o[blk][4 * a + 1] * inv),
                          T::pack2(o[blk][4 * a + 2] * inv, o[blk][4 * a + 3] * inv)};
            }
        int own_again = own < it.row_count ? own : 0, own_tok, own_head;
        asm volatile("" : "+v"(own_again));
        rows.at(own_again, own_tok, own_head);
        if (half == 0)
            row_off[own & 31] = ((int64_t)(it.q_row0 + own_tok) * num_q_heads +
                                 it.kv_head * group + own_head) * D;
        // LDS operations of one wavefront complete in order; the statement keeps the compiler from
        // moving the reads in front of the other lanes' writes
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        constexpr int LPR = D / 8;  // lanes per row, 16 bytes each
        const int c = lane_again % LPR;
#pragma unroll
        for (int r0 = 0; r0 < 32; r0 += 64 / LPR) {
            const int r = r0 + lane_again / LPR;
            if (r < wave_rows)
                *reinterpret_cast<u32x4 *>(out + row_off[r] + 8 * c) =
                    *reinterpret_cast<const u32x4 *>(part + r * ROW_BYTES + 16 * c);
        }
    } else if (own < it.row_count) {
        const int64_t slot = (int64_t)it.partial_base + own;
        float *po = ws_o + slot * D;
#pragma unroll
        for (int blk = 0; blk < NB; ++blk)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int d = 32 * blk + 8 * a + 4 * half;
                *reinterpret_cast<f32x4 *>(po + d) = f32x4{o[blk][4 * a], o[blk][4 * a + 1],
                                                           o[blk][4 * a + 2], o[blk][4 * a + 3]};
            }
        if (half == 0) {
            // the merge works in the log2 domain of the scaled scores
            ws_ml[2 * slot] = m_run == -INFINITY ? -INFINITY : m_run * scale_log2e;
            ws_ml[2 * slot + 1] = l_tot;
        }
    }
}

template <typename T, int D>
static hipError_t launch_wide_t(const pv_plan *plan, const DeviceLists &dl, const void *q, const void *k_pages,
                                const void *v_pages, const int32_t *page_table, float scale,
                                void *out, float *ws_o, float *ws_ml, hipStream_t stream)
{
    const int n = (int)plan->wide.size();
    // A negative scale is applied as |scale| on negated queries, a zero scale as 1 on zeros: so
    // that a masked score, minus infinity, is a probability of zero whatever the scale.  (Zero times
    // an infinity or a NaN among the queries is NaN: the kernel looks for these at its end.)
    float c = (scale < 0.f ? -scale : scale) * kLog2e;
    const uint32_t q_sign = scale < 0.f ? 0x80008000u : 0u;
    const uint32_t q_keep = c == 0.f ? 0u : 0xFFFFFFFFu;
    if (c == 0.f) c = 1.f;
    auto kernel = plan->wide_streams ? (plan->wide_renews ? attn_wide_kernel<T, D, true, true>
                                                          : attn_wide_kernel<T, D, false, true>)
                                     : (plan->wide_renews ? attn_wide_kernel<T, D, true, false>
                                                          : attn_wide_kernel<T, D, false, false>);
    hipLaunchKernelGGL(kernel, dim3(n), dim3(256), 0, stream, dl.wide, (const uint16_t *)q,
                       (const uint16_t *)k_pages, (const uint16_t *)v_pages,
                       page_table, plan->max_pages_per_req, plan->num_q_heads,
                       plan->pool.num_kv_heads, plan->group, c, q_keep, q_sign, (uint16_t *)out,
                       ws_o, ws_ml, plan->num_reqs);
    return hipGetLastError();
}

hipError_t launch_attn_wide(const pv_plan *plan, const DeviceLists &dl, const void *q, const void *k_pages,
                            const void *v_pages, const int32_t *page_table, float scale, void *out,
                            float *ws_o, float *ws_ml, hipStream_t stream)
{
    if (plan->wide.empty()) return hipSuccess;
    const bool f = plan->pool.dtype == PV_F16;
    if (plan->pool.head_dim == 128)
        return f ? launch_wide_t<F16, 128>(plan, dl, q, k_pages, v_pages, page_table, scale, out, ws_o,
                                           ws_ml, stream)
                 : launch_wide_t<BF16, 128>(plan, dl, q, k_pages, v_pages, page_table, scale, out,
                                            ws_o, ws_ml, stream);
    return f ? launch_wide_t<F16, 64>(plan, dl, q, k_pages, v_pages, page_table, scale, out, ws_o,
                                      ws_ml, stream)
             : launch_wide_t<BF16, 64>(plan, dl, q, k_pages, v_pages, page_table, scale, out, ws_o,
                                       ws_ml, stream);
}

}  // namespace pv
