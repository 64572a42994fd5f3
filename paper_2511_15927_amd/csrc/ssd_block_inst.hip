// Instantiations and launcher of the one-chunk Mamba-2 call (ssd_block.h).
#include "ssd_block.h"
#include "launch.h"

#include <atomic>

namespace bm {

template <int N, int BLOCKS>
static void prep_one(const SsdBlockArgs& a, hipStream_t st)
{
    static std::atomic<bool> seen[kMaxSeenDevices];
    constexpr size_t lds = ssd_block_prep_lds<N, BLOCKS>();
    auto prep = ssd_block_prep_kernel<N, BLOCKS>;
    if (lds > 64 * 1024 && first_use_on_current_device(seen))
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(prep), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(prep, dim3((unsigned)a.G, 2, (unsigned)a.batch), dim3(1024), lds, st, a);
}

template <int N, int BLOCKS>
static void launch_one(const SsdBlockArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.Dn + 63) / 64), 1, (unsigned)a.batch);
    if (a.h_out) {
        if (a.shared) hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, true, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, true, false>), grid, dim3(256), 0, st, a);
    } else {
        if (a.shared) hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, false, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((ssd_block_kernel<N, BLOCKS, false, false>), grid, dim3(256), 0, st, a);
    }
}

void launch_ssd_block_prep(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) a.L <= 32 ? prep_one<128, 1>(a, st) : prep_one<128, 2>(a, st);
    else a.L <= 32 ? prep_one<64, 1>(a, st) : prep_one<64, 2>(a, st);
}

void launch_ssd_block(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) a.L <= 32 ? launch_one<128, 1>(a, st) : launch_one<128, 2>(a, st);
    else a.L <= 32 ? launch_one<64, 1>(a, st) : launch_one<64, 2>(a, st);
}

}  // namespace bm
