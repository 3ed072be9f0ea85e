// KV append: store the new K/V rows of a batch into the slots the page table assigns to them
// (paper Section 4.4.1: the newly generated KV-tokens are stored in their allocated slots before
// the attention runs).  Pure 16-bit moves, so the pool image is bit-exact.
//
// One workgroup of D threads handles one append group (up to 8 consecutive new tokens of a request
// inside one 8-slot group of a page, listed by the host plan) for one KV head.
//   K pool: 8 consecutive head dimensions of a token are one 16-byte run; thread t copies run
//           (token t / (D/8), chunk t % (D/8)).
//   V pool: 8 consecutive slots of one head dimension are one 16-byte run; thread d gathers its
//           dimension from the group's tokens and, when the group is full, writes the run with one
//           16-byte store (otherwise element by element, leaving the other slots untouched).
#include "pv_device.h"

namespace pv {

// KV head h of the tokens of one append group
template <int D, bool STREAM>
__device__ __forceinline__ void append_group(const AppendGroup &g, int h,
                                             const uint16_t *__restrict__ k_new,
                                             const uint16_t *__restrict__ v_new,
                                             const int32_t *__restrict__ page_table,
                                             int32_t max_pages, int32_t num_kv_heads,
                                             uint16_t *__restrict__ k_pages,
                                             uint16_t *__restrict__ v_pages)
{
    constexpr int CH = D / 8;
    const int t = (int)threadIdx.x;
    const int64_t page = page_table[(int64_t)g.req * max_pages + (g.t_begin >> 4)];
    const int slot0 = g.t_begin & 15;  // slot of the group's first token; the group stays in one
                                       // half (8 slots) of the page
    const int64_t tile = (page * num_kv_heads + h) * (int64_t)(16 * D);
    const int64_t row_stride = (int64_t)num_kv_heads * D;
    const uint16_t *ksrc = k_new + (int64_t)g.q_row * row_stride + (int64_t)h * D;
    const uint16_t *vsrc = v_new + (int64_t)g.q_row * row_stride + (int64_t)h * D;

    // K: thread -> (token j, chunk c8)
    {
        const int j = t / CH, c8 = t % CH;
        if (j < g.count) {
            const u32x4 kv = load16_as<STREAM>(ksrc + j * row_stride + 8 * c8);
            *reinterpret_cast<u32x4 *>(k_pages + tile + (c8 * 16 + slot0 + j) * 8) = kv;
        }
    }
    // V: thread -> head dimension d = t
    scatter_v_group<D, 1, STREAM>(vsrc, row_stride, g.count, 1, slot0, t, v_pages + tile);
}

template <int D, bool STREAM>
__global__ __launch_bounds__(D) void kv_append_kernel(
    const AppendGroup *__restrict__ groups, const uint16_t *__restrict__ k_new,
    const uint16_t *__restrict__ v_new, const int32_t *__restrict__ page_table, int32_t max_pages,
    int32_t num_kv_heads, uint16_t *__restrict__ k_pages, uint16_t *__restrict__ v_pages)
{
    const AppendGroup g = groups[blockIdx.x];
    append_group<D, STREAM>(g, (int)blockIdx.y, k_new, v_new, page_table, max_pages, num_kv_heads,
                            k_pages, v_pages);
}

// The same for a batch that has no plan: the requests come with the launch, and a workgroup works out
// its append group from them (a binary search of at most seven steps in the kernel's arguments).
// So the one-shot call needs no device memory for a list, no copy of one and no wait for that copy.
template <int D>
__global__ __launch_bounds__(D) void kv_append_reqs_kernel(
    const AppendReqs reqs, const uint16_t *__restrict__ k_new, const uint16_t *__restrict__ v_new,
    const int32_t *__restrict__ page_table, int32_t max_pages, int32_t num_kv_heads,
    uint16_t *__restrict__ k_pages, uint16_t *__restrict__ v_pages)
{
    const int gi = (int)blockIdx.x;
    int lo = 0, hi = reqs.n - 1;  // the last request whose first group is not behind this one
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (reqs.r[mid].group0 <= gi)
            lo = mid;
        else
            hi = mid - 1;
    }
    const AppendReq r = reqs.r[lo];
    const int run = (r.t_begin >> 3) + gi - r.group0;  // 8-slot run of the request's positions
    const int end = r.t_begin + r.count;
    AppendGroup g;
    g.req = r.req;
    g.t_begin = max(8 * run, r.t_begin);
    g.count = min(8 * run + 8, end) - g.t_begin;
    g.q_row = r.q_row + g.t_begin - r.t_begin;
    append_group<D, false>(g, (int)blockIdx.y, k_new, v_new, page_table, max_pages, num_kv_heads,
                           k_pages, v_pages);
}

hipError_t launch_kv_append_reqs(const pv_pool_desc *pool, const AppendReqs &reqs,
                                 const void *k_new, const void *v_new, const int32_t *page_table,
                                 int32_t max_pages, void *k_pages, void *v_pages,
                                 hipStream_t stream)
{
    if (reqs.n <= 0) return hipSuccess;
    const dim3 grid((unsigned)reqs.groups, (unsigned)pool->num_kv_heads);
    if (pool->head_dim == 128)
        hipLaunchKernelGGL((kv_append_reqs_kernel<128>), grid, dim3(128), 0, stream, reqs,
                           (const uint16_t *)k_new, (const uint16_t *)v_new, page_table, max_pages,
                           pool->num_kv_heads, (uint16_t *)k_pages, (uint16_t *)v_pages);
    else
        hipLaunchKernelGGL((kv_append_reqs_kernel<64>), grid, dim3(64), 0, stream, reqs,
                           (const uint16_t *)k_new, (const uint16_t *)v_new, page_table, max_pages,
                           pool->num_kv_heads, (uint16_t *)k_pages, (uint16_t *)v_pages);
    return hipGetLastError();
}

template <int D, bool STREAM>
static void launch_append_t(const pv_plan *plan, const DeviceLists &dl, const void *k_new,
                            const void *v_new, const int32_t *page_table, void *k_pages,
                            void *v_pages, hipStream_t stream)
{
    const dim3 grid((unsigned)plan->append_groups.size(), (unsigned)plan->pool.num_kv_heads);
    hipLaunchKernelGGL((kv_append_kernel<D, STREAM>), grid, dim3(D), 0, stream, dl.append_groups,
                       (const uint16_t *)k_new, (const uint16_t *)v_new, page_table,
                       plan->max_pages_per_req, plan->pool.num_kv_heads, (uint16_t *)k_pages,
                       (uint16_t *)v_pages);
}

hipError_t launch_kv_append(const pv_plan *plan, const DeviceLists &dl, const void *k_new, const void *v_new,
                            const int32_t *page_table, void *k_pages, void *v_pages,
                            hipStream_t stream)
{
    if (plan->append_groups.empty()) return hipSuccess;
    const bool many = (int64_t)plan->total_q * plan->pool.num_kv_heads * plan->pool.head_dim * 4 >
                      kStreamBytes;
    auto go = plan->pool.head_dim == 128
                  ? (many ? launch_append_t<128, true> : launch_append_t<128, false>)
                  : (many ? launch_append_t<64, true> : launch_append_t<64, false>);
    go(plan, dl, k_new, v_new, page_table, k_pages, v_pages, stream);
    return hipGetLastError();
}

}  // namespace pv
