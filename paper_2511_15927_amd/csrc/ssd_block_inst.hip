// Instantiations and launcher of the one-chunk Mamba-2 call (ssd_block.h).
#include "ssd_block.h"
#include "launch.h"

namespace bm {

template <int N, int BLOCKS>
static hipError_t prep_one(const SsdBlockArgs& a, hipStream_t st)
{
    static LdsLimit limit;
    constexpr size_t lds = ssd_block_prep_lds<N, BLOCKS>();
    auto prep = ssd_block_prep_kernel<N, BLOCKS>;
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(prep), lds);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(prep, dim3((unsigned)a.G, 2, (unsigned)a.batch), dim3(1024), lds, st, a);
    return hipSuccess;
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

hipError_t launch_ssd_block_prep(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) return a.L <= 32 ? prep_one<128, 1>(a, st) : prep_one<128, 2>(a, st);
    return a.L <= 32 ? prep_one<64, 1>(a, st) : prep_one<64, 2>(a, st);
}

void launch_ssd_block(int d_state, const SsdBlockArgs& a, hipStream_t st)
{
    if (d_state == 128) a.L <= 32 ? launch_one<128, 1>(a, st) : launch_one<128, 2>(a, st);
    else a.L <= 32 ? launch_one<64, 1>(a, st) : launch_one<64, 2>(a, st);
}

}  // namespace bm
