// Instantiations and launchers of the chunked Mamba-2 kernels (d_state in {64, 128}, head width in {32, 64}).
#include "ssd_kernels.h"
#include "launch.h"

namespace bm {

template <int N, int THREADS>
static hipError_t prep_variant(const SsdPrepPair& pa, int nchunk, int batch, hipStream_t st)
{
    static LdsLimit limit;
    constexpr size_t lds = ssd_prep_lds_bytes<N, THREADS>();
    auto kernel = ssd_prep_kernel<N, THREADS>;
    if (lds > 64 * 1024) {
        const hipError_t err = limit.raise(reinterpret_cast<const void*>(kernel), lds);
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)nchunk, (unsigned)pa.dir[0].G, 2u * (unsigned)batch), dim3(THREADS), lds, st, pa);
    return hipSuccess;
}

bool ssd_supported(int d_state, int headdim) { return (d_state == 64 || d_state == 128) && (headdim == 32 || headdim == 64); }

// Launches that give a CU at most one workgroup take the sixteen-wave form: their duration is one workgroup's chain.
hipError_t launch_ssd_prep(int d_state, const SsdPrepPair& pa, int nchunk, int batch, hipStream_t st)
{
    const bool wide = 2LL * nchunk * pa.dir[0].G * batch <= cu_count();
    if (d_state == 128) return wide ? prep_variant<128, 1024>(pa, nchunk, batch, st) : prep_variant<128, 256>(pa, nchunk, batch, st);
    return wide ? prep_variant<64, 1024>(pa, nchunk, batch, st) : prep_variant<64, 256>(pa, nchunk, batch, st);
}

void launch_ssd_carry(int d_state, const SsdCarryArgs& ca, hipStream_t st)
{
    const long long threads = 2LL * ca.batch * ca.Dn * d_state / 4;
    const dim3 grid((unsigned)((threads + 255) / 256));
    if (d_state == 128) hipLaunchKernelGGL(ssd_carry_kernel<128>, grid, dim3(256), 0, st, ca);
    else hipLaunchKernelGGL(ssd_carry_kernel<64>, grid, dim3(256), 0, st, ca);
}

// Both directions in one launch; nothing to do for the sub-part scanned last (no part starts after it).
void launch_ssd_state(int d_state, int headdim, const SsdStatePair& sp, int subs, int batch, hipStream_t st)
{
    if (subs < 2) return;
    const dim3 grid((unsigned)sp.dir[0].H, (unsigned)(subs - 1), (unsigned)(2 * batch));
    if (d_state == 128 && headdim == 64) hipLaunchKernelGGL((ssd_state_kernel<128, 64>), grid, dim3(256), 0, st, sp);
    else if (d_state == 128 && headdim == 32) hipLaunchKernelGGL((ssd_state_kernel<128, 32>), grid, dim3(256), 0, st, sp);
    else if (d_state == 64 && headdim == 64) hipLaunchKernelGGL((ssd_state_kernel<64, 64>), grid, dim3(256), 0, st, sp);
    else if (d_state == 64 && headdim == 32) hipLaunchKernelGGL((ssd_state_kernel<64, 32>), grid, dim3(256), 0, st, sp);
}

// dirs 1: the direction sp.dir[0]; dirs 2: both in one launch, for calls whose directions write halves of their own.  A
// workgroup holds a CU and a call's time is its longest chain of chunks, so two launches that each leave CUs empty take
// twice as long as one: 120 heads x 32, N 128, 1 x 1024 tokens 72.2 -> 38.1 us a call.
hipError_t launch_ssd_scan(int d_state, int headdim, const SsdStatePair& sp, int dirs, int batch, hipStream_t st)
{
    if (d_state == 128 && headdim == 64) return launch_ssd_wide_n128_p64(sp, dirs, batch, st);
    if (d_state == 128 && headdim == 32) return launch_ssd_wide_n128_p32(sp, dirs, batch, st);
    if (d_state == 64 && headdim == 64) return launch_ssd_wide_n64_p64(sp, dirs, batch, st);
    if (d_state == 64 && headdim == 32) return launch_ssd_wide_n64_p32(sp, dirs, batch, st);
    return hipErrorInvalidValue;
}

}  // namespace bm
