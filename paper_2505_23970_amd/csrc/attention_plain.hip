// Launchers of the attention kernels over 8-bit pools and of the split merge (the
// kernels are in attention_kernels.h).
#include "attention_kernels.h"

namespace gc {

hipError_t launch_attention_fp8(const AttnArgs& a, int head_dim, int64_t num_items, bool wide, bool three,
                                int resident, hipStream_t s) {
    const dim3 grid((unsigned)(num_items * a.num_kv_heads));
    if (resident > 0 && wide) {
        const int total = (int)(num_items * a.num_kv_heads);
        const dim3 rg((unsigned)resident), rb(kWideWaves * 64);
        if (head_dim == 128)
            hipLaunchKernelGGL((attention_resident_kernel<128, true>), rg, rb, 0, s, a, total);
        else
            hipLaunchKernelGGL((attention_resident_kernel<64, true>), rg, rb, 0, s, a, total);
        return hipGetLastError();
    }
    if (wide) {
        if (head_dim == 128)
            attention_kernel<128, kWideWaves, true><<<grid, kWideWaves * 64, 0, s>>>(a);
        else
            attention_kernel<64, kWideWaves, true><<<grid, kWideWaves * 64, 0, s>>>(a);
    } else {
        if (head_dim == 128)
            attention_kernel<128, kWaves, true><<<grid, kWaves * 64, 0, s>>>(a);
        else if (three)
            attention_kernel<64, kWaves, true, 3><<<grid, kWaves * 64, 0, s>>>(a);
        else
            attention_kernel<64, kWaves, true><<<grid, kWaves * 64, 0, s>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_combine(const CombineArgs& a, int head_dim, int64_t num_combines, int max_splits, hipStream_t s) {
    // Eight thread groups per row save round trips (32 chunks each instead of 8, about
    // 1 us a trip) and cost workgroups (one per row instead of one per eight, about 0.7 ns
    // each to start), so they are for few rows: 16.3 -> 15.1 us (attention and merge) for
    // 128 rows of 17 chunks, but 28.6 -> 31.0 for 4096 rows of 9 and 93 -> 105 for 16384.
    const int64_t all_rows = num_combines * a.num_kv_heads * a.block_m;
    const int trips_saved = ceil_div(max_splits, 8) - ceil_div(max_splits, 32);
    const int groups_of = all_rows <= 1536LL * trips_saved ? 8 : 1;
    const int rows = kCombineThreads / (head_dim / 4 * groups_of);
    const dim3 grid((unsigned)(num_combines * a.num_kv_heads * ceil_div(a.block_m, rows)));
    if (head_dim == 128) {
        if (groups_of > 1)
            combine_kernel<128, 8><<<grid, kCombineThreads, 0, s>>>(a);
        else
            combine_kernel<128, 1><<<grid, kCombineThreads, 0, s>>>(a);
    } else {
        if (groups_of > 1)
            combine_kernel<64, 8><<<grid, kCombineThreads, 0, s>>>(a);
        else
            combine_kernel<64, 1><<<grid, kCombineThreads, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace gc
