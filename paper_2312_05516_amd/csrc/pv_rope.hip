// Rotary position embedding fused with the KV append: the producer step in front of the hot path
// for the Llama 2 models of the paper (Section 6.1 lists rotary embedding among their features;
// Section 4.4.1: the linear layers produce each token's Q/K/V, the new K/V are stored in their
// slots, then attention runs).  One launch rotates the new K rows and stores them in the pool,
// stores the new V rows, and rotates the Q rows, instead of a rotary pass over Q and K followed by
// the append.
//
// The transform is the published RoFormer one: pair i of a head, for a token at logical position
// t, is rotated by t * theta_i.  cos / sin come from a table [max_pos][D] (D/2 cosines, then D/2
// sines) that the caller computes once (pv_rope_table).  Pairing: style 0 = elements (2i, 2i+1),
// style 1 = elements (i, i + D/2).  The rotation is evaluated in fp32 and rounded to the 16-bit
// type (nearest even); V is moved bit for bit.
//
// Grid: (append groups, head blocks) with D threads; a head block is HB heads of one kind, the KV
// heads first (K rotated + scattered, V scattered as in kv_append_kernel), then the query heads of
// the group's tokens.  The heads of a token share its angles, which are twice the bytes of one
// head's row, so a thread loads them once for all its heads, and then all its rows at once.
#include "pv_device.h"

namespace pv {

template <typename T>
__device__ __forceinline__ void unpack8(u32x4 raw, float (&x)[8])
{
    const typename T::vec8 v = as_vec8<T>(raw);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (float)v[e];
}

template <typename T>
__device__ __forceinline__ u32x4 pack8(const float (&x)[8])
{
    return u32x4{T::pack2(x[0], x[1]), T::pack2(x[2], x[3]), T::pack2(x[4], x[5]),
                 T::pack2(x[6], x[7])};
}

template <typename T, int D, int STYLE, int HB>
__global__ __launch_bounds__(D) void rope_append_kernel(
    const AppendGroup *__restrict__ groups, const uint16_t *q_in,
    uint16_t *q_out /* may be q_in */, const uint16_t *__restrict__ k_new,
    const uint16_t *__restrict__ v_new, const float *__restrict__ cos_sin,
    const int32_t *__restrict__ page_table, int32_t max_pages, int32_t num_q_heads,
    int32_t num_kv_heads, uint16_t *__restrict__ k_pages, uint16_t *__restrict__ v_pages)
{
    constexpr int CH = D / 8;
    const AppendGroup g = groups[blockIdx.x];
    const int kv_blocks = (num_kv_heads + HB - 1) / HB;
    const int y = (int)blockIdx.y;
    const int t = (int)threadIdx.x;
    const bool is_q = y >= kv_blocks;
    const int h0 = (is_q ? y - kv_blocks : y) * HB;
    const int heads = min(HB, (is_q ? num_q_heads : num_kv_heads) - h0);
    const int64_t row_stride = (int64_t)(is_q ? num_q_heads : num_kv_heads) * D;
    const int64_t src_off = (int64_t)g.q_row * row_stride + (int64_t)h0 * D;
    const uint16_t *src = (is_q ? q_in : k_new) + src_off;

    int64_t tile = 0;
    int slot0 = 0;
    if (!is_q) {
        const int64_t page = page_table[(int64_t)g.req * max_pages + (g.t_begin >> 4)];
        slot0 = g.t_begin & 15;
        tile = (page * num_kv_heads + h0) * (int64_t)(16 * D);
    }
    // destination of the 16-byte chunk c8 of token j, head i of the block
    auto store_chunk = [&](int j, int i, int c8, u32x4 val) {
        if (is_q)
            *reinterpret_cast<u32x4 *>(q_out + src_off + j * row_stride + i * D + 8 * c8) = val;
        else
            *reinterpret_cast<u32x4 *>(k_pages + tile + i * (16 * D) + (c8 * 16 + slot0 + j) * 8) =
                val;
    };

    if constexpr (STYLE == 0) {
        // one thread per (token j, chunk c8): 4 pairs inside the chunk, of every head
        const int j = t / CH, c8 = t % CH;
        if (j < g.count) {
            const float *cs = cos_sin + (int64_t)(g.t_begin + j) * D;
            const f32x4 c = *reinterpret_cast<const f32x4 *>(cs + 4 * c8);
            const f32x4 s = *reinterpret_cast<const f32x4 *>(cs + D / 2 + 4 * c8);
            u32x4 raw[HB];
#pragma unroll
            for (int i = 0; i < HB; ++i)
                raw[i] = load16_as<(HB > 1)>(src + j * row_stride + (i < heads ? i : 0) * D + 8 * c8);
#pragma unroll
            for (int i = 0; i < HB; ++i) {
                float x[8], o[8];
                unpack8<T>(raw[i], x);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    o[2 * p] = x[2 * p] * c[p] - x[2 * p + 1] * s[p];
                    o[2 * p + 1] = x[2 * p + 1] * c[p] + x[2 * p] * s[p];
                }
                if (i < heads) store_chunk(j, i, c8, pack8<T>(o));
            }
        }
    } else {
        // one thread per (token j, chunk c8 of the first half): its partner chunk is c8 + CH/2.  A
        // head takes half of the threads; with several heads the other half takes every other one.
        constexpr int LANES = 8 * (CH / 2);
        constexpr int SIDES = HB > 1 ? 2 : 1;
        constexpr int MINE = HB / SIDES;
        const int side = t / LANES, j = t % LANES / (CH / 2), c8 = t % (CH / 2);
        if (side < SIDES && j < g.count) {
            const float *cs = cos_sin + (int64_t)(g.t_begin + j) * D;
            f32x4 c[2], s[2];
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                c[half] = *reinterpret_cast<const f32x4 *>(cs + 8 * c8 + 4 * half);
                s[half] = *reinterpret_cast<const f32x4 *>(cs + D / 2 + 8 * c8 + 4 * half);
            }
            u32x4 ra[MINE], rb[MINE];
#pragma unroll
            for (int m = 0; m < MINE; ++m) {
                const int i = SIDES * m + side;
                const uint16_t *row = src + j * row_stride + (i < heads ? i : 0) * D + 8 * c8;
                ra[m] = load16_as<(HB > 1)>(row);
                rb[m] = load16_as<(HB > 1)>(row + D / 2);
            }
#pragma unroll
            for (int m = 0; m < MINE; ++m) {
                const int i = SIDES * m + side;
                float xa[8], xb[8], oa[8], ob[8];
                unpack8<T>(ra[m], xa);
                unpack8<T>(rb[m], xb);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float ce = c[e / 4][e % 4], se = s[e / 4][e % 4];
                    oa[e] = xa[e] * ce - xb[e] * se;
                    ob[e] = xb[e] * ce + xa[e] * se;
                }
                if (i < heads) {
                    store_chunk(j, i, c8, pack8<T>(oa));
                    store_chunk(j, i, c8 + CH / 2, pack8<T>(ob));
                }
            }
        }
    }

    // V: thread -> head dimension d = t, moved bit for bit
    if (!is_q)
        scatter_v_group<D, HB, (HB > 1)>(v_new + src_off, row_stride, g.count, heads, slot0, t,
                                         v_pages + tile);
}

template <typename T, int D, int STYLE, int HB>
static void launch_rope_t(const pv_plan *plan, const DeviceLists &dl, const void *q_in, void *q_out,
                          const void *k_new, const void *v_new, const float *cos_sin,
                          const int32_t *page_table, void *k_pages, void *v_pages,
                          hipStream_t stream)
{
    const int kv_blocks = (plan->pool.num_kv_heads + HB - 1) / HB;
    const int q_blocks = q_in ? (plan->num_q_heads + HB - 1) / HB : 0;
    const dim3 grid((unsigned)plan->append_groups.size(), (unsigned)(kv_blocks + q_blocks));
    hipLaunchKernelGGL((rope_append_kernel<T, D, STYLE, HB>), grid, dim3(D), 0, stream,
                       dl.append_groups, (const uint16_t *)q_in, (uint16_t *)q_out,
                       (const uint16_t *)k_new, (const uint16_t *)v_new, cos_sin, page_table,
                       plan->max_pages_per_req, plan->num_q_heads, plan->pool.num_kv_heads,
                       (uint16_t *)k_pages, (uint16_t *)v_pages);
}

// A large batch: two rows a thread (two heads a workgroup, four where pairs span the halves of a
// head and half of the threads do a head), and the rows are read with the streaming hint (kStreamBytes).
// 8 prompts, 7 K tokens, whole step: 40/40 heads, interleaved pairs 190 -> 181 us (187 with one head,
// 182 with four; 190 with four and no hint), half pairs 185 -> 177 (185 with two, 178 with eight);
// 64/8 heads, 4 K tokens, half pairs 95 -> 91.  A small batch keeps one head a workgroup, the more of
// them run at once (4 generation steps, 64/8 heads: 24.8 us against 25.5).
template <typename T, int D>
static auto pick_rope(int style, bool many)
{
    if (style == 0) return many ? launch_rope_t<T, D, 0, 2> : launch_rope_t<T, D, 0, 1>;
    return many ? launch_rope_t<T, D, 1, 4> : launch_rope_t<T, D, 1, 1>;
}

hipError_t launch_rope_append(const pv_plan *plan, const DeviceLists &dl, int style, const void *q_in, void *q_out,
                              const void *k_new, const void *v_new, const float *cos_sin,
                              const int32_t *page_table, void *k_pages, void *v_pages,
                              hipStream_t stream)
{
    if (plan->append_groups.empty()) return hipSuccess;
    const bool f = plan->pool.dtype == PV_F16;
    const int64_t rows = 2 * plan->pool.num_kv_heads + (q_in ? plan->num_q_heads : 0);
    const bool many = plan->total_q * rows * plan->pool.head_dim * 2 > kStreamBytes;
    auto go = plan->pool.head_dim == 128
                  ? (f ? pick_rope<F16, 128>(style, many) : pick_rope<BF16, 128>(style, many))
                  : (f ? pick_rope<F16, 64>(style, many) : pick_rope<BF16, 64>(style, many));
    go(plan, dl, q_in, q_out, k_new, v_new, cos_sin, page_table, k_pages, v_pages, stream);
    return hipGetLastError();
}

}  // namespace pv
