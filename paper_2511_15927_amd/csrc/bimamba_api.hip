// Host side of the C ABI declared in include/bimamba.h: argument validation, workspace carving, kernel dispatch.
#include "bimamba.h"
#include "kernels.h"
#include "launch.h"
#include "bwd_kernels.h"
#include "row_kernels.h"
#include "stack_kernels.h"
#include "ssd_block.h"
#include "ssd_kernels.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <memory>
#include <new>

// Device memory of bimamba_block_fwd_static, the entry point for callers that cannot allocate: one copy per GPU, held
// until the process ends.  In host code this name only identifies the symbol; the address a kernel can use is asked
// from the runtime once per device (static_scratch below).
static __device__ __align__(256) unsigned char scratch[BIMAMBA_STATIC_SCRATCH_BYTES];

namespace {

using namespace bm;

thread_local hipEvent_t g_probe_start = nullptr, g_probe_stop = nullptr;  // one-shot, see bimamba_profile_next_call

}  // namespace

namespace bm {
int cu_count()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
        cus = cached[dev].load(std::memory_order_relaxed);
        if (cus == 0) {
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
            cached[dev].store(cus, std::memory_order_relaxed);
        }
    }
    return cus;   // no device (a host-only query): plan for the 256-CU chip
}
}  // namespace bm

namespace {

// Launch geometry is planned for the SIMDs the device has (four per CU); the thresholds below were measured on MI355X
// (256 CUs, 1024 SIMDs).
inline int simds() { return 4 * cu_count(); }
inline int target_waves() { return 2 * simds(); }   // two waves per SIMD

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Byte range [lo, hi) a tensor view spans (non-negative strides, checked before this is used).
struct Span {
    uintptr_t lo, hi;
};
Span span_of(const bimamba_tensor& t, int channels, size_t elem, const bimamba_desc* d)
{
    const uintptr_t lo = reinterpret_cast<uintptr_t>(t.ptr);
    const int64_t last = (int64_t)(d->batch - 1) * t.stride_batch + (int64_t)(d->seqlen - 1) * t.stride_token + channels;
    return Span{lo, lo + (uintptr_t)last * elem};
}

// Whether writing `out` could touch memory an input view reads.  Views whose byte ranges are apart never do; views
// that interleave inside one buffer (column slices of one projection output, the usual layout) do not either when
// they share both strides, rows tile the batch stride, and their column ranges are apart modulo the row pitch.
bool may_overlap(const bimamba_tensor& out, int out_ch, const bimamba_tensor& in, int in_ch, size_t elem,
                 const bimamba_desc* d)
{
    const Span a = span_of(out, out_ch, elem, d), b = span_of(in, in_ch, elem, d);
    if (a.hi <= b.lo || b.hi <= a.lo) return false;
    if (out.stride_token == in.stride_token && out.stride_batch == in.stride_batch && out.stride_token > 0 &&
        out.stride_batch % out.stride_token == 0) {
        const int64_t pitch = out.stride_token;
        const int64_t delta = ((int64_t)a.lo - (int64_t)b.lo) / (int64_t)elem;
        const int64_t r = ((delta % pitch) + pitch) % pitch;   // out's first column, counted from in's first column
        if (r >= in_ch && r + out_ch <= pitch) return false;
    }
    return true;
}
inline bool is_aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

__global__ __launch_bounds__(256) void zero_fill_kernel(float* p, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// A call's five inputs into buffers of the caller, in one launch: grid (pieces of 256 threads, 1, the tensors).  A thread moves eight
// elements of a row, 16 or 32 bytes at a time where both sides are aligned to that.
struct CopyArgs {
    struct Side {
        char* p;
        long long sb, st;   // bytes
    } from[5], to[5];
    int width[5], vector[5];   // elements of a row
    int batch, L;
};
template <typename T>
__global__ __launch_bounds__(256) void copy_inputs_kernel(const CopyArgs a)
{
    constexpr int kPiece = 8;
    struct __attribute__((aligned(16))) Piece { T v[kPiece]; };
    const int i = blockIdx.z, pieces = (a.width[i] + kPiece - 1) / kPiece;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)a.batch * a.L * pieces) return;
    const long long row = idx / pieces;
    const int first = (int)(idx - row * pieces) * kPiece, b = (int)(row / a.L), t = (int)(row - (long long)b * a.L);
    const T* const from = reinterpret_cast<const T*>(a.from[i].p + b * a.from[i].sb + t * a.from[i].st) + first;
    T* const to = reinterpret_cast<T*>(a.to[i].p + b * a.to[i].sb + t * a.to[i].st) + first;
    if (a.vector[i] && first + kPiece <= a.width[i]) {
        *reinterpret_cast<Piece*>(to) = *reinterpret_cast<const Piece*>(from);
    } else {
        for (int e = 0; e < kPiece && first + e < a.width[i]; e++) to[e] = from[e];
    }
}

bool split_supported(int d_state, int split)
{
    switch (d_state * 8 + split) {
        case 4 * 8 + 1: case 8 * 8 + 1: case 16 * 8 + 1: case 16 * 8 + 2: case 16 * 8 + 4: case 32 * 8 + 1:
        case 32 * 8 + 2: case 32 * 8 + 4: case 64 * 8 + 1: case 64 * 8 + 4: case 128 * 8 + 1: case 128 * 8 + 4:
            return true;
        default: return false;
    }
}

int check_desc(const bimamba_desc* d)
{
    if (!d) return BIMAMBA_ERR_NULL_POINTER;
    if (d->struct_size != sizeof(bimamba_desc)) return BIMAMBA_ERR_BAD_SHAPE;
    if (d->batch < 0 || d->seqlen < 0 || d->d_inner < 1 || d->d_state < 1 || d->n_heads < 1 || d->n_groups < 1 ||
        d->d_conv < 1)
        return BIMAMBA_ERR_BAD_SHAPE;
    if (d->d_inner % d->n_heads || d->n_heads % d->n_groups) return BIMAMBA_ERR_BAD_SHAPE;
    if (d->time_chunks < 0 || d->state_split < 0) return BIMAMBA_ERR_BAD_SHAPE;
    if (d->state_split > 0 && !split_supported(d->d_state, d->state_split)) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->batch > 65535) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->io_dtype != BIMAMBA_F32 && d->io_dtype != BIMAMBA_BF16) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->a_kind != BIMAMBA_A_PER_HEAD_STATE && d->a_kind != BIMAMBA_A_SCALAR_PER_HEAD) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->d_kind != BIMAMBA_D_PER_CHANNEL && d->d_kind != BIMAMBA_D_PER_HEAD) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->combine != BIMAMBA_COMBINE_ADD && d->combine != BIMAMBA_COMBINE_SEPARATE) return BIMAMBA_ERR_UNSUPPORTED;
    if ((d->dt_softplus | 1) != 1 || (d->conv_bc | 1) != 1) return BIMAMBA_ERR_UNSUPPORTED;
    if (d->d_conv > 4) return BIMAMBA_ERR_UNSUPPORTED;
    switch (d->d_state) {
        case 4: case 8: case 16: case 32: case 64: case 128: break;
        default: return BIMAMBA_ERR_UNSUPPORTED;
    }
    if (d->n_groups > 1 && (d->d_inner / d->n_groups) % 64 != 0) return BIMAMBA_ERR_UNSUPPORTED;
    return BIMAMBA_OK;
}

long long waves_of(const bimamba_desc* d, int split)
{
    const int cpw = 64 / split;
    return 2LL * d->batch * ((d->d_inner + cpw - 1) / cpw);
}

// Launch geometry of the lane-per-chain kernels, from measurements on MI355X (1024 SIMDs) with w = the number of waves
// that one lane per chain gives (2 * batch * d_inner / 64), for 32 states (up to 16: pick_geometry below):
//   first       two lanes per chain (each holds half the states), whole sequence, when the 2w waves fill the rounds of
//               resident waves well (two_lanes_fit below).
//   w >= 1920   one lane per chain, whole sequence: close to two waves per SIMD already.
//   else        one lane per chain and the sequence cut into time segments until about 16 waves per SIMD exist: the
//               segment summaries cost a second, cheaper pass, but every SIMD then holds enough waves to issue back
//               to back and to hide the loads, whatever the batch.  Segments stay at 256 tokens or more when that
//               still gives four waves per SIMD, at 128 or more otherwise.
//               If even that leaves fewer than two waves per SIMD (short sequences), two lanes per chain.
// Four lanes per chain cost as many vector instructions per channel and token as two (measured with the tokens dealt:
// 2.36 ms against 1.83 at the headline shape, and twice the HBM fetch because four tiles share a 128-byte line) and
// are not picked below 64 states.  With 64 or 128 states a lane cannot hold a whole chain without starving the SIMD of
// registers, so those shapes split the states first (four lanes per chain) and cut the sequence only as far as two
// waves per SIMD need, in segments of at least 256 tokens.
constexpr int kWavesForSegments = 16384;
constexpr int kMinSegmentTokens = 128;

bool many_states(const bimamba_desc* d) { return d->d_state > 32; }

int segments_for(const bimamba_desc* d, long long waves)
{
    const int L = d->seqlen;
    if (L <= 0 || waves <= 0) return 1;
    const int want = many_states(d) ? target_waves() : kWavesForSegments;
    long long min_tokens = 256;
    if (!many_states(d) && waves * (L / 256) < 4 * simds()) min_tokens = kMinSegmentTokens;
    long long n = (want + waves - 1) / waves;
    const long long max_by_len = L / min_tokens > 0 ? L / min_tokens : 1;
    if (n > max_by_len) n = max_by_len;
    return (int)(n < 1 ? 1 : n);
}

// Two lanes per chain, whole sequence.  Up to 16 states the pair deals its tokens (see run_tiles_dealt) and a SIMD
// holds three such waves at once: measured at d_inner 4096 (L 8192, batch 5 to 32) and d_inner 2048 (L 1024 to 8192,
// batch 16 to 64) against the best of the other geometries, it wins from 1.7 to 5 waves per SIMD (batch 7 to 20 at
// d_inner 4096: -3 to -23 %) and loses outside.
// With 32 states the plain walk keeps three waves on a SIMD: 1.8 to 2, or 2.35 to 3 per SIMD.
bool two_lanes_fit(const bimamba_desc* d, long long w)
{
    const long long per_simd_x100 = 2 * w * 100 / simds();
    if (d->d_state <= 16) return per_simd_x100 >= 170 && per_simd_x100 <= 500;
    return (per_simd_x100 >= 180 && per_simd_x100 <= 200) || (per_simd_x100 >= 235 && per_simd_x100 <= 300);
}

// One lane per chain needs no help from segments or lane splitting.
bool enough_chains(const bimamba_desc* d, long long w) { return many_states(d) ? w >= target_waves() : 8 * w >= 15 * simds(); }

// Whether one lane per chain, the whole call in one launch (short_kernel), is the choice for a call that allows it: up to
// 64 tokens and 16 states, no conv on B and C.  Against the other geometries (bf16, 16 states, 4 / 16 / 32 / 64 tokens, us, other -> one
// launch): 20480 chains (batch * d_inner) 14.4 / 15.0 / 18.8 / 26.1 -> 8.8 / 10.1 / 14.3 / 22.6, 57344 chains 17.6 / 23.9 / 32.1 / 45.4 ->
// 8.5 / 12.7 / 18.2 / 29.8, 262144 chains x 64 118 -> 97; general decays, fp32, halves apart alike.  Only while two lanes per chain make at most
// one wave per SIMD (16384 chains) do more than 32 tokens favour them: 64 tokens 22.3 / 22.0 (one launch / two lanes), fp32 26.4 / 23.7,
// halves apart 23.1 / 20.6.  (Fewer chains yet: the row form.)  And with the directions' halves apart two lanes win more than 48 tokens
// from one to one and a half waves per SIMD, where one lane leaves some SIMDs two waves: 36000 chains x 64 tokens, per-state decays 43.8
// (one launch) / 40.4, a decay per head 35.1 / 35.5; added up 41.7 / 41.4 and 33.1 / 36.3; 57344 chains 46.3 / 53.3.
bool one_launch_fits(const bimamba_desc* d, long long w)
{
    if (d->d_state > 16 || d->conv_bc || d->seqlen > kShortCallTokens) return false;
    if (d->d_state < 16 || d->seqlen <= 32) return true;
    const bool uneven = d->combine == BIMAMBA_COMBINE_SEPARATE && d->seqlen > 48 && w > simds() && 2 * w <= 3 * simds();
    return 2 * w > simds() && !uneven;
}

int pick_split_general(const bimamba_desc* d)
{
    if (d->state_split > 0) return d->state_split;
    const long long w = waves_of(d, 1);
    const bool two = split_supported(d->d_state, 2), four = d->d_state >= 64 && split_supported(d->d_state, 4);
    if (!many_states(d) && two && d->time_chunks <= 1 && !one_launch_fits(d, w) && two_lanes_fit(d, w)) return 2;
    if (enough_chains(d, w)) return 1;
    if (many_states(d)) return w >= target_waves() / 2 && two ? 2 : four ? 4 : two ? 2 : 1;
    if (d->time_chunks == 0 && w * segments_for(d, w) >= target_waves()) return 1;
    return two ? 2 : 1;
}

int pick_chunks_general(const bimamba_desc* d, int split)
{
    const int L = d->seqlen;
    if (L <= 0) return 1;
    int n;
    if (d->time_chunks > 0) {
        n = d->time_chunks;
    } else {
        const long long waves = waves_of(d, split);
        const long long w = waves_of(d, 1);
        const bool whole = d->state_split == 0 && !many_states(d) &&
                           (split == 1 ? enough_chains(d, w) : split == 2 && two_lanes_fit(d, w));
        n = waves >= target_waves() || whole ? 1 : segments_for(d, waves);
    }
    if (n > L) n = L;
    if (n > 4096) n = 4096;
    if (n < 1) n = 1;
    return n;
}

// Up to 16 states, lanes per chain and time segments that are left to the library, for calls that neither fill the chip
// (enough_chains) nor the band of two_lanes_fit.  Either the whole sequence is walked at once, with two lanes per chain
// where 16 states allow it: its time is the tokens' times what a token costs while a SIMD holds at most one wave, or
// up to two; or segments: a price for the two launches more, and a cost that follows the work.  In microseconds, bf16,
// the state's decay general or arithmetic:
//   16 states  whole 8 + 0.165 L (2w <= 1 wave per SIMD) or 8 + 0.25 L;  segments 35 + 0.32 w L
//   8 states   whole 4 + 0.33 L;  segments 35 + 0.21 w L (w >= 1.4 waves per SIMD: always whole)
// Segments fill rounds of resident workgroups (four waves per SIMD with one lane per chain) exactly: one workgroup more than
// a round holds costs a round.  Four rounds while segments keep 128 tokens, else one round of segments of 48 (16 states)
// or 16 tokens; too few tokens for that: two lanes per chain, three waves per SIMD, segments of 24 or more.  The carry folds
// the segments one after the other, so the shortest segment grows with the root of the sequence, and a call too narrow to
// fill one workgroup per CU even with those gets no more of them (1 x 1928 tokens of 256 channels, 8 states: whole 519 us,
// 15 segments 83, 84 segments 36; 1 x 16384 tokens of 64 channels: 1024 segments 128, 128 segments 94, 256 segments 72).
// Over 491 calls (8 and 16 states, 512 to 4096 channels, batch 1 to 48, 64 to 16384 tokens, bf16 and fp32) the choice is on
// average 2.0 % slower than the best of twenty geometries with 16 states and 4.4 % with 8, the general rule 25 % and 31 %.
// Beside the general rule alone, 240 calls of 256 to 4096 channels, decays per state or per head, bf16 or fp32: 24 to 30 %
// less time with 4 states, 24 to 32 % with 8, 14 to 20 % with 16, the worst call 20 % more; 240 calls of 16 to 2048 channels
// at batch 1 to 8: 41 to 46 % less, the worst 1 % more.
struct Geometry {
    int split, nseg;
};
Geometry pick_geometry(const bimamba_desc* d)
{
    const int L = d->seqlen;
    const bool pair = d->d_state == 16;
    const double w = (double)waves_of(d, 1) / simds(), tokens = L;
    if (pair) {
        if (tokens * (2 * w <= 1 ? 0.165 : 0.25) + 8 <= 35 + 0.32 * w * tokens) return {2, 1};
    } else if (w >= 1.4 || tokens * 0.33 + 4 <= 35 + 0.21 * w * tokens) {
        return {1, 1};
    }
    // segments of a launch that holds `layers` workgroups per CU at most
    auto segments = [&](int split, int layers) {
        const int cpw = 64 / split;
        const long long per_segment = (long long)(((d->d_inner + cpw - 1) / cpw + 1) / 2) * d->batch;
        const long long n = (long long)layers * cu_count() / per_segment;
        return (int)(n < 1 ? 1 : n > L ? L : n);
    };
    auto tokens_of = [&](int n) { return L / n; };
    const double root = (pair ? 0.65 : 0.5) * std::sqrt(tokens);
    int n = segments(1, 16);
    if (n > 1 && tokens_of(n) >= 128) return {1, n};
    auto at_most = [&](int n, double shortest) { return std::min(n, std::max(1, (int)(tokens / shortest))); };
    if (pair) {
        n = segments(1, 4);
        if (n > 1 && tokens_of(n) >= std::max(48.0, root)) return {1, n};
        const double shortest = std::max(24.0, root);
        for (int layers = 3; layers > 1; layers--) {
            n = segments(2, layers);
            if (tokens_of(n) >= shortest) return {2, n};
        }
        return {2, at_most(segments(2, 1), std::max(16.0, root))};
    }
    const double shortest = std::max(16.0, root);
    for (int layers = 4; layers > 1; layers--) {
        n = segments(1, layers);
        if (n > 1 && tokens_of(n) >= shortest) return {1, n};
    }
    return {1, at_most(segments(1, 1), shortest)};
}

// coarse: by the general rule whatever the state count (see make_plan).
Geometry geometry_of(const bimamba_desc* d, bool coarse)
{
    const int split = pick_split_general(d);
    const bool open = d->state_split == 0 && d->time_chunks == 0 && d->d_state <= 16 && d->seqlen > 0 && d->batch > 0;
    const long long w = waves_of(d, 1);
    if (open && one_launch_fits(d, w)) return {1, 1};
    if (open && !coarse && !enough_chains(d, w) && !(d->d_state == 16 && two_lanes_fit(d, w))) {
        Geometry g = pick_geometry(d);
        if (g.nseg > 4096) g.nseg = 4096;
        return g;
    }
    return {split, pick_chunks_general(d, split)};
}

struct Plan {
    int split, nseg, seg_len;
    bool two_bc;  // the two directions consume different prepared B|C buffers
    bool ssd;     // Mamba-2 parameterisation on the chunked matrix-core kernels
    int ssd_chunks;
    int ssd_parts, ssd_part_chunks;  // time parts of the matrix-core path (1: every (batch, head) item is one workgroup)
    int ssd_subs, ssd_part_subs, ssd_sub_chunks;  // sub-parts the state pass walks: in all, per part, chunks of each
    bool ssd_meet;  // both directions walk at once and meet in the middle (kSsdMeet), not in time parts, unless rows are far apart
    size_t off_bc[2], off_partial, off_carry, off_sumdt, off_crows[2], off_bt[2], off_score[2], off_pstate[2], off_pdecay[2], total;
};

// The chunked matrix-core path covers bf16 I/O with one decay rate per head, d_state 64 or 128 and heads of 32 or
// 64 channels; forcing time_chunks or state_split selects the lane-per-chain kernels instead.
bool use_ssd(const bimamba_desc* d)
{
    return d->a_kind == BIMAMBA_A_SCALAR_PER_HEAD && d->io_dtype == BIMAMBA_BF16 && d->time_chunks == 0 &&
           d->state_split == 0 && ssd_supported(d->d_state, d->d_inner / d->n_heads) &&
           d->batch <= 32767;   // the preparation kernel's grid holds both directions of every batch element
}

constexpr size_t kScratch = BIMAMBA_STATIC_SCRATCH_BYTES;

// Prepared tiles of the chunked matrix-core path: C (or B^T) and scores of a direction, all of them.
size_t ssd_rows_bytes(const bimamba_desc* d, int chunks) { return align_up((size_t)d->batch * chunks * kQ * d->n_groups * d->d_state * sizeof(__bf16), 256); }
size_t ssd_score_bytes(const bimamba_desc* d, int chunks) { return align_up((size_t)d->batch * chunks * d->n_groups * kScoreOp * sizeof(float), 256); }
size_t ssd_tile_bytes(const bimamba_desc* d, int chunks) { return 2 * (2 * ssd_rows_bytes(d, chunks) + ssd_score_bytes(d, chunks)); }

Plan plan_of(const bimamba_desc* d, bool inputs_shared, bool coarse)
{
    Plan p{};
    // The lane-per-chain geometry is always planned (and its workspace reserved): a call whose x tensors do not meet
    // the matrix-core kernels' alignment needs falls back to it.
    p.ssd = use_ssd(d);
    const Geometry geometry = geometry_of(d, coarse);
    p.split = geometry.split;
    p.nseg = geometry.nseg;
    p.seg_len = d->seqlen > 0 ? (d->seqlen + p.nseg - 1) / p.nseg : 1;
    p.nseg = d->seqlen > 0 ? (d->seqlen + p.seg_len - 1) / p.seg_len : 1;
    p.two_bc = d->conv_bc || !inputs_shared;
    const size_t bc_bytes = align_up((size_t)d->batch * d->seqlen * d->n_groups * 2 * d->d_state * sizeof(float), 256);
    size_t off = 0;
    p.off_bc[0] = off; off += bc_bytes;
    if (p.two_bc) { p.off_bc[1] = off; off += bc_bytes; } else { p.off_bc[1] = p.off_bc[0]; }
    p.off_partial = off;
    if (d->combine == BIMAMBA_COMBINE_ADD) off += align_up((size_t)d->batch * d->seqlen * d->d_inner * sizeof(float), 256);
    p.off_carry = off;
    p.off_sumdt = off;
    if (p.nseg > 1) {
        off += align_up((size_t)2 * d->batch * p.nseg * d->d_inner * d->d_state * sizeof(float), 256);
        p.off_sumdt = off;
        off += align_up((size_t)2 * d->batch * p.nseg * d->d_inner * sizeof(float), 256);
    }
    p.ssd_chunks = (d->seqlen + kQ - 1) / kQ;
    // Time parts: a call whose (batch, head) items would leave at least half of the 256 CUs empty deals each item's
    // chunks to several workgroups (at least 8 chunks each, at most 16 parts); a first, cheaper pass then finds the
    // state entering each part.  That pass runs light workgroups, four to a CU, so it cuts the parts further into
    // sub-parts (at least 4 chunks each) until both directions together bring about that many.
    p.ssd_parts = p.ssd_subs = p.ssd_part_subs = 1;
    p.ssd_part_chunks = p.ssd_sub_chunks = p.ssd_chunks;
    if (p.ssd) {
        // (directions with an output half of their own share a launch: twice the items in flight)
        const long long items = (long long)d->n_heads * d->batch * (d->combine == BIMAMBA_COMBINE_SEPARATE ? 2 : 1);
        const int cus = cu_count();
        long long parts = items > 0 ? cus / items : 1;
        if (parts > p.ssd_chunks / 8) parts = p.ssd_chunks / 8;
        if (parts > 16) parts = 16;
        // Both directions at once, to meet in the middle, where they fit the chip: the walk of two parts an item without the state
        // pass.  More parts, which the state pass lets start anywhere, are ahead when they save more chunks of the walk than that
        // pass, which follows the items, costs.  us, parts / meeting, (heads x channels, states) x tokens, batch 1:
        //   120 x 32, 128   66 18.7/18.0  512 31.8/27.0  1024 56.5/37.1  2048 88.0/55.3  4096 134/91.5  16384 525/387
        //   64 x 64, 128    66 21.2/22.0  130 24.0/24.7  300 29.7/28.0  1024 66.7/45.8  1536 74.5/56.7  2048 83/67.7  4096 124/113  16384 450/513
        //   64 x 32, 64     300 22.6/19.0  1024 45.0/30.2  2048 54.0/46.6  4096 78.0/77.7  16384 248/290
        //   24 x 32, 128    300 24.1/21.0  1024 44.0/32.5  1536 47.7/42.3  2048 50.5/51.4  4096 60.4/84.0;  batch 2, 64 x 64 x 2048 119/77
        p.ssd_meet = d->combine == BIMAMBA_COMBINE_ADD && p.ssd_chunks >= (d->d_inner / d->n_heads > 32 ? 4 : 2) && items > 0 && 2 * items <= cus &&
                     p.ssd_chunks * (parts - 2) <= parts * (4 + items / 2);
        if (p.ssd_meet && parts < 2) {
            // the states it meets with must not take a block call out of the fixed scratch that holds it without them
            // (by the size for separate activations)
            const size_t states = 2 * align_up((size_t)d->batch * d->d_inner * d->d_state * sizeof(float), 256);
            const size_t without = off + (p.two_bc ? 0 : bc_bytes) + ssd_tile_bytes(d, p.ssd_chunks);
            if (without <= kScratch && without + states > kScratch) p.ssd_meet = false;
        }
        if (parts >= 2) {
            const int part_chunks = (int)((p.ssd_chunks + parts - 1) / parts);
            const long long items_both = 2LL * d->n_heads * d->batch;
            const long long subs_wanted = (4LL * cus + items_both - 1) / items_both;
            long long k = (subs_wanted + parts - 1) / parts;
            if (k > part_chunks / 4) k = part_chunks / 4;
            if (k < 1) k = 1;
            p.ssd_part_subs = (int)k;
            p.ssd_sub_chunks = (int)((part_chunks + k - 1) / k);
            p.ssd_part_chunks = p.ssd_part_subs * p.ssd_sub_chunks;
            p.ssd_parts = (p.ssd_chunks + p.ssd_part_chunks - 1) / p.ssd_part_chunks;
            p.ssd_subs = (p.ssd_chunks + p.ssd_sub_chunks - 1) / p.ssd_sub_chunks;
        }
    }
    if (p.ssd) {
        const size_t rows = ssd_rows_bytes(d, p.ssd_chunks), score = ssd_score_bytes(d, p.ssd_chunks);
        for (int s = 0; s < 2; s++) {
            p.off_crows[s] = off; off += rows;
            p.off_bt[s] = off; off += rows;
            p.off_score[s] = off; off += score;
        }
        for (int s = 0; s < 2; s++) {
            p.off_pstate[s] = p.off_pdecay[s] = off;
            // (the states that directions meet with: in the place of those of the parts, of which there are two or more)
            if (p.ssd_meet && p.ssd_parts == 1) off += align_up((size_t)d->batch * d->d_inner * d->d_state * sizeof(float), 256);
            if (p.ssd_parts > 1) {
                off += align_up((size_t)p.ssd_subs * d->batch * d->d_inner * d->d_state * sizeof(float), 256);
                p.off_pdecay[s] = off;
                off += align_up((size_t)p.ssd_subs * d->batch * d->n_heads * sizeof(float), 256);
            }
        }
    }
    p.total = off;
    return p;
}

// The plan of a call that brings `bytes` of workspace.  Segments by cost can be more than the general rule's and so can their
// states.  A block call that fits the fixed scratch of bimamba_block_fwd_static only with the general rule's gets those from
// both block entry points, whose results are bit-identical; bimamba_fwd has no such twin and takes them only where the
// caller's workspace, sized for the block call of the same shape, holds no more.
// (Decided on the size for separate activations: a call must not plan more than bimamba_workspace_bytes said.)
Plan make_plan(const bimamba_desc* d, bool inputs_shared, bool block_variant, size_t bytes)
{
    const Plan fine = plan_of(d, inputs_shared, false);
    if (!block_variant && bytes >= fine.total) return fine;
    const bool fits_coarse_only = plan_of(d, false, false).total > kScratch && plan_of(d, false, true).total <= kScratch;
    return fits_coarse_only ? plan_of(d, inputs_shared, true) : fine;
}

constexpr int64_t kMaxTokenStride = 1 << 26;  // elements

int check_tensor(const bimamba_tensor& t, int channels, size_t elem, const bimamba_desc* d)
{
    const bool empty = d->batch == 0 || d->seqlen == 0;  // nothing is read or written: the pointer may be NULL
    if (!t.ptr && !empty) return BIMAMBA_ERR_NULL_POINTER;
    if (!is_aligned(t.ptr, elem)) return BIMAMBA_ERR_MISALIGNED;
    if (empty) return BIMAMBA_OK;                         // no element exists, so no stride is ever used
    if (t.stride_token < channels) return BIMAMBA_ERR_BAD_SHAPE;
    if (t.stride_token > kMaxTokenStride) return BIMAMBA_ERR_UNSUPPORTED;  // row offsets inside a tile are 32-bit
    if (d->batch > 1 && t.stride_batch < (int64_t)d->seqlen * t.stride_token - (t.stride_token - channels))
        return BIMAMBA_ERR_BAD_SHAPE;
    return BIMAMBA_OK;
}

int check_params(const bimamba_params* p)
{
    if (!p) return BIMAMBA_ERR_NULL_POINTER;
    if (!p->conv_w || !p->A || !p->D) return BIMAMBA_ERR_NULL_POINTER;
    if (!is_aligned(p->conv_w, 4) || !is_aligned(p->A, 4) || !is_aligned(p->D, 4) || !is_aligned(p->conv_b, 4) ||
        !is_aligned(p->dt_bias, 4))
        return BIMAMBA_ERR_MISALIGNED;
    return BIMAMBA_OK;
}

int check_inputs(const bimamba_inputs* in, const bimamba_desc* d, size_t elem)
{
    if (!in) return BIMAMBA_ERR_NULL_POINTER;
    int rc;
    if ((rc = check_tensor(in->x, d->d_inner, elem, d))) return rc;
    if ((rc = check_tensor(in->z, d->d_inner, elem, d))) return rc;
    if ((rc = check_tensor(in->dt, d->n_heads, elem, d))) return rc;
    if ((rc = check_tensor(in->B, d->n_groups * d->d_state, elem, d))) return rc;
    if ((rc = check_tensor(in->C, d->n_groups * d->d_state, elem, d))) return rc;
    return BIMAMBA_OK;
}

bool same_tensor(const bimamba_tensor& a, const bimamba_tensor& b)
{
    return a.ptr == b.ptr && a.stride_batch == b.stride_batch && a.stride_token == b.stride_token;
}

bool same_inputs(const bimamba_inputs* a, const bimamba_inputs* b)
{
    return a == b || (same_tensor(a->x, b->x) && same_tensor(a->z, b->z) && same_tensor(a->dt, b->dt) &&
                      same_tensor(a->B, b->B) && same_tensor(a->C, b->C));
}

bool pairs_readable(const bimamba_tensor& t)
{
    return is_aligned(t.ptr, 4) && t.stride_batch % 2 == 0 && t.stride_token % 2 == 0;
}

TensorArg targ(const bimamba_tensor& t) { return TensorArg{t.ptr, (long long)t.stride_batch, (long long)t.stride_token}; }

// A call of a few dozen tokens with one lane per chain, up to 16 states and no conv on B and C runs as a single
// launch: the scan kernel converts the caller's B and C rows itself instead of reading prepared fp32 rows.
bool short_call(const bimamba_desc* d, const Plan& plan)
{
    return !plan.ssd && plan.split == 1 && plan.nseg == 1 && d->d_state <= 16 && !d->conv_bc &&
           d->seqlen <= kShortCallTokens;
}

// A short call with few chains takes the one-row-per-chain form: everything in one launch.
bool row_call(const bimamba_desc* d, const Plan& plan, RowForm* row)
{
    return !plan.ssd && !d->conv_bc && d->time_chunks == 0 && d->state_split == 0 &&
           row_form(d->batch, d->seqlen, d->d_inner, d->d_state, d->combine == BIMAMBA_COMBINE_SEPARATE, row);
}

// Over how many states the decays of an arithmetic A may be products (SweepArgs::try_progression): no more than in the other forms that
// are the choice for calls of the size.  The row form takes an exponential a state, and so do the calls of its sizes that
// another form runs faster (by products over sixteen states what 13312 chains commit after 16 tokens is 8.1e-7 from 64 bits, this way
// 1.3e-7); lane pairs hold eight states a lane.  One lane a chain is the choice of itself from 1.9 waves per SIMD on.
int decay_run(const bimamba_desc* d)
{
    if (d->d_state > 16 || d->seqlen > kShortCallTokens) return 16;   // (the length matters to the short form only)
    const bool row_size = !d->conv_bc && d->time_chunks == 0 && d->state_split == 0 && row_reach(d->batch, d->seqlen, d->d_inner);
    return row_size ? 0 : enough_chains(d, waves_of(d, 1)) ? 16 : 8;
}

hipError_t launch_scan(const bimamba_desc* d, int split, int short_call, const SweepArgs& sa, const CarryArgs& ca,
                       hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const int scalar_a = d->a_kind == BIMAMBA_A_SCALAR_PER_HEAD, bf16 = d->io_dtype == BIMAMBA_BF16;
#define BM_CASE(n, s) \
    case (n) * 8 + (s): return launch_scan_n##n##_s##s(scalar_a, bf16, sa, ca, d->batch, short_call, st, ev_start, ev_stop);
    switch (d->d_state * 8 + split) {
        BM_CASE(4, 1) BM_CASE(8, 1) BM_CASE(16, 1) BM_CASE(16, 2) BM_CASE(16, 4) BM_CASE(32, 1) BM_CASE(32, 2)
        BM_CASE(32, 4) BM_CASE(64, 1) BM_CASE(64, 4) BM_CASE(128, 1) BM_CASE(128, 4)
        default: return hipErrorInvalidValue;
    }
#undef BM_CASE
}

int run(const bimamba_desc* d, const bimamba_params* pf, const bimamba_params* pb, const bimamba_inputs* in_f,
        const bimamba_inputs* in_b, const float* h_in, const void* tail_in, float* h_out, void* tail_out,
        const bimamba_tensor* out, void* workspace, size_t workspace_bytes, void* hip_stream, bool block_variant)
{
    const hipEvent_t probe_start = g_probe_start, probe_stop = g_probe_stop;
    g_probe_start = g_probe_stop = nullptr;
    int rc = check_desc(d);
    if (rc) return rc;
    const size_t elem = d->io_dtype == BIMAMBA_BF16 ? 2 : 4;
    if ((rc = check_params(pf))) return rc;
    if ((rc = check_params(pb))) return rc;
    if (!in_b) in_b = in_f;
    if ((rc = check_inputs(in_f, d, elem))) return rc;
    if ((rc = check_inputs(in_b, d, elem))) return rc;
    if (!out) return BIMAMBA_ERR_NULL_POINTER;
    const int out_ch = d->combine == BIMAMBA_COMBINE_SEPARATE ? 2 * d->d_inner : d->d_inner;
    if ((rc = check_tensor(*out, out_ch, elem, d))) return rc;
    if (!is_aligned(h_in, 4) || !is_aligned(h_out, 4) || !is_aligned(tail_in, elem) || !is_aligned(tail_out, elem))
        return BIMAMBA_ERR_MISALIGNED;
    const bool shared = same_inputs(in_f, in_b);
    Plan plan = make_plan(d, shared, block_variant, workspace_bytes);
    // the chunked kernels read x two channels at a time and the carried state four states at a time
    if (plan.ssd && !(pairs_readable(in_f->x) && pairs_readable(in_b->x) && is_aligned(h_in, 16) && is_aligned(h_out, 16)))
        plan.ssd = false;
    // the state pass of the time parts addresses a chunk's rows of x with 32-bit byte offsets, the walk its rows of z and out
    // (but in kSsdFarParts)
    constexpr int64_t kMaxNearStride = 1 << 24;
    const bool far = in_f->z.stride_token > kMaxNearStride || in_b->z.stride_token > kMaxNearStride || out->stride_token > kMaxNearStride;
    const bool meet = plan.ssd && plan.ssd_meet && !far;
    if (meet || (plan.ssd && plan.ssd_parts > 1 && (in_f->x.stride_token > kMaxNearStride || in_b->x.stride_token > kMaxNearStride))) {
        plan.ssd_parts = plan.ssd_subs = plan.ssd_part_subs = 1;
        plan.ssd_part_chunks = plan.ssd_sub_chunks = plan.ssd_chunks;
    }
    if (plan.total > 0) {
        if (!workspace) return BIMAMBA_ERR_NULL_POINTER;
        if (!is_aligned(workspace, 16)) return BIMAMBA_ERR_MISALIGNED;
        if (workspace_bytes < plan.total) return BIMAMBA_ERR_WORKSPACE_TOO_SMALL;
    }
    if (d->batch > 0 && d->seqlen > 0) {
        const int gn = d->n_groups * d->d_state;
        for (const bimamba_inputs* in : {in_f, in_b}) {
            if (may_overlap(*out, out_ch, in->x, d->d_inner, elem, d) || may_overlap(*out, out_ch, in->z, d->d_inner, elem, d) ||
                may_overlap(*out, out_ch, in->dt, d->n_heads, elem, d) || may_overlap(*out, out_ch, in->B, gn, elem, d) ||
                may_overlap(*out, out_ch, in->C, gn, elem, d))
                return BIMAMBA_ERR_ALIAS;
        }
    }
    const hipError_t pending = hipPeekAtLastError();   // an error some earlier, unrelated call left behind is not ours to report or clear
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    const int GN = d->n_groups * d->d_state;
    const int tail_ch = d->d_inner + (d->conv_bc ? 2 * GN : 0);
    char* ws = static_cast<char*>(workspace);

    if (d->batch > 0 && d->seqlen > 0) {
        RowForm row;
        if (row_call(d, plan, &row)) {   // the commit of the conv tail is part of the launch too
            RowArgs ra{};
            for (int s = 0; s < 2; s++) {
                const bimamba_inputs* in = s == 0 ? in_f : in_b;
                const bimamba_params* p = s == 0 ? pf : pb;
                DirArgs& da = ra.dir[s];
                da.x = targ(in->x); da.z = targ(in->z); da.dt = targ(in->dt);
                da.Braw = targ(in->B); da.Craw = targ(in->C);
                da.conv_w = p->conv_w; da.conv_b = p->conv_b; da.A = p->A; da.D = p->D; da.dt_bias = p->dt_bias;
            }
            ra.out = out->ptr; ra.out_sb = out->stride_batch; ra.out_st = out->stride_token;
            if (block_variant) {
                ra.h_in = h_in; ra.h_out = h_out;
                ra.tail_in = tail_in; ra.tail_out = d->d_conv > 1 ? tail_out : nullptr;
                tail_out = nullptr;
            }
            ra.L = d->seqlen; ra.Dn = d->d_inner; ra.P = d->d_inner / d->n_heads; ra.HG = d->n_heads / d->n_groups;
            ra.G = d->n_groups; ra.N = d->d_state; ra.K = d->d_conv;
            ra.dt_softplus = d->dt_softplus; ra.d_per_head = d->d_kind == BIMAMBA_D_PER_HEAD;
            ra.a_scalar = d->a_kind == BIMAMBA_A_SCALAR_PER_HEAD; ra.separate = d->combine == BIMAMBA_COMBINE_SEPARATE;
            ra.same_z = same_tensor(in_f->z, in_b->z);
            ra.same_bc = same_tensor(in_f->B, in_b->B) && same_tensor(in_f->C, in_b->C);
            ra.tw = row.tw; ra.tw_log2 = row.tw == 4 ? 2 : row.tw == 2 ? 1 : 0; ra.nseg = row.nseg; ra.seg_len = row.seg_len;
            if (probe_start) (void)hipEventRecord(probe_start, st);
            if (launch_row(d->io_dtype == BIMAMBA_BF16, ra, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
            if (probe_stop) (void)hipEventRecord(probe_stop, st);
        } else {
        // 1. fp32 B|C rows per direction (the chunked path prepares its own operand tiles from the raw rows)
        const bool one_launch = short_call(d, plan);
        const int nbuf = (plan.ssd || one_launch) ? 0 : plan.two_bc ? 2 : 1;
        PrepPair prep{};
        for (int s = 0; s < nbuf; s++) {
            const bimamba_inputs* in = s == 0 ? in_f : in_b;
            const bimamba_params* p = s == 0 ? pf : pb;
            PrepArgs& pa = prep.dir[s];
            pa.B = targ(in->B);
            pa.C = targ(in->C);
            pa.conv_w = p->conv_w;
            pa.conv_b = p->conv_b;
            pa.tail_in = (s == 0 && block_variant) ? tail_in : nullptr;
            pa.dst = reinterpret_cast<float*>(ws + plan.off_bc[s]);
            pa.batch = d->batch; pa.L = d->seqlen; pa.G = d->n_groups; pa.N = d->d_state; pa.K = d->d_conv;
            pa.Dn = d->d_inner; pa.tail_ch = tail_ch; pa.conv_bc = d->conv_bc; pa.dir = s == 0 ? 1 : -1;
        }
        if (nbuf > 0) {
            const long long total = (long long)d->batch * d->seqlen * 2 * GN;
            const dim3 grid((unsigned)((total + 255) / 256), (unsigned)nbuf);
            if (d->io_dtype == BIMAMBA_BF16) hipLaunchKernelGGL(prep_bc_kernel<IoBF16>, grid, dim3(256), 0, st, prep);
            else hipLaunchKernelGGL(prep_bc_kernel<IoF32>, grid, dim3(256), 0, st, prep);
        }
        if (plan.ssd && plan.ssd_chunks == 1) {
            // 2''. one chunk: its operands, then both directions of every (batch, head) item at once
            SsdBlockArgs ba{};
            for (int s = 0; s < 2; s++) {
                const bimamba_inputs* in = s == 0 ? in_f : in_b;
                const bimamba_params* p = s == 0 ? pf : pb;
                SsdBlockDir& bd = ba.dir[s];
                bd.x = targ(in->x); bd.z = targ(in->z); bd.dt = targ(in->dt); bd.B = targ(in->B); bd.C = targ(in->C);
                bd.conv_w = p->conv_w; bd.conv_b = p->conv_b; bd.A = p->A; bd.D = p->D; bd.dt_bias = p->dt_bias;
                ba.score[s] = reinterpret_cast<float*>(ws + plan.off_score[s]);
            }
            ba.c_op = reinterpret_cast<__bf16*>(ws + plan.off_crows[0]);
            ba.b_op = reinterpret_cast<__bf16*>(ws + plan.off_bt[0]);
            ba.out = out->ptr; ba.out_sb = out->stride_batch; ba.out_st = out->stride_token;
            if (block_variant) {
                ba.h_in = h_in; ba.h_out = h_out;
                ba.tail_in = tail_in; ba.tail_out = d->d_conv > 1 ? tail_out : nullptr;
                tail_out = nullptr;
            }
            ba.batch = d->batch; ba.L = d->seqlen; ba.Dn = d->d_inner; ba.H = d->n_heads; ba.P = d->d_inner / d->n_heads;
            ba.HG = d->n_heads / d->n_groups; ba.G = d->n_groups; ba.K = d->d_conv; ba.tail_ch = tail_ch;
            ba.dt_softplus = d->dt_softplus; ba.d_per_head = d->d_kind == BIMAMBA_D_PER_HEAD; ba.conv_bc = d->conv_bc;
            ba.separate = d->combine == BIMAMBA_COMBINE_SEPARATE;
            ba.shared = same_tensor(in_f->x, in_b->x) && same_tensor(in_f->z, in_b->z);
            ba.tiles = ssd_block_tiles(d->d_state, ba);
            if (ba.tiles && ba.conv_bc && ba.tail_out) {
                // every workgroup of a batch element reads B's and C's part of the tail: where it is committed in place, after them.  Where
                // the state is not committed too: the kernel for that writes no such part (with it 16 x 32 tokens of 64 heads x 64 take
                // 16.6 us, 16.1 without)
                const size_t bytes = (size_t)d->batch * (d->d_conv - 1) * tail_ch * sizeof(__bf16);
                const uintptr_t from = reinterpret_cast<uintptr_t>(ba.tail_in), to = reinterpret_cast<uintptr_t>(ba.tail_out);
                if (!ba.h_out || (from && from < to + bytes && to < from + bytes)) {
                    // (the launch for it, 2 us, costs four tiles a workgroup what they save: 16 x 32 tokens of 64 heads x 64 23.8 against
                    // 23.4 us; two tiles or one 11.4 against 13.8, 1 x 32, and 15.8 against 17.0, 32 x 32 of 16 heads)
                    if (ba.tiles == 4) ba.tiles = 0;
                    else {
                        tail_out = ba.tail_out;
                        ba.tail_out = nullptr;
                    }
                }
            }
            if (!ba.tiles && launch_ssd_block_prep(d->d_state, ba, st) != hipSuccess) return BIMAMBA_ERR_HIP;   // (nothing is committed)
            if (probe_start) (void)hipEventRecord(probe_start, st);
            if (launch_ssd_block(d->d_state, ba, st) != hipSuccess) return BIMAMBA_ERR_HIP;
            if (probe_stop) (void)hipEventRecord(probe_stop, st);
        } else if (plan.ssd) {
            // 2'. chunked matrix-core path: per-direction operand tiles, then the reverse scan parks its result and the
            // forward scan adds, gates and stores (or each writes its own half)
            const bool separate = d->combine == BIMAMBA_COMBINE_SEPARATE;
            const bool raw = !separate && same_tensor(in_f->z, in_b->z);
            SsdPrepPair pp{};
            for (int s = 0; s < 2; s++) {
                SsdPrepArgs& pa = pp.dir[s];
                const bimamba_inputs* in = s == 0 ? in_f : in_b;
                const bimamba_params* p = s == 0 ? pf : pb;
                pa.B = targ(in->B); pa.C = targ(in->C);
                pa.conv_w = p->conv_w; pa.conv_b = p->conv_b;
                pa.tail_in = (s == 0 && block_variant) ? tail_in : nullptr;
                pa.K = d->d_conv; pa.Dn = d->d_inner; pa.tail_ch = tail_ch; pa.conv_bc = d->conv_bc;
                pa.c_rows = reinterpret_cast<__bf16*>(ws + plan.off_crows[s]);
                pa.b_t = reinterpret_cast<__bf16*>(ws + plan.off_bt[s]);
                pa.score_op = reinterpret_cast<float*>(ws + plan.off_score[s]);
                pa.L = d->seqlen; pa.G = d->n_groups; pa.dir = s == 0 ? 1 : -1;
                pa.lead = meet && s == 1 ? plan.ssd_chunks * kQ - d->seqlen : 0;
            }
            if (launch_ssd_prep(d->d_state, pp, plan.ssd_chunks, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
            if (probe_start) (void)hipEventRecord(probe_start, st);
            auto scan_args = [&](int s) {
                const bimamba_inputs* in = s == 0 ? in_f : in_b;
                const bimamba_params* p = s == 0 ? pf : pb;
                SsdArgs sa{};
                sa.x = targ(in->x); sa.z = targ(in->z); sa.dt = targ(in->dt);
                sa.conv_w = p->conv_w; sa.conv_b = p->conv_b; sa.A = p->A; sa.D = p->D; sa.dt_bias = p->dt_bias;
                sa.c_rows = reinterpret_cast<const __bf16*>(ws + plan.off_crows[s]);
                sa.b_t = reinterpret_cast<const __bf16*>(ws + plan.off_bt[s]);
                sa.score_op = reinterpret_cast<const float*>(ws + plan.off_score[s]);
                sa.out = out->ptr; sa.out_sb = out->stride_batch; sa.out_st = out->stride_token;
                sa.partial = reinterpret_cast<float*>(ws + plan.off_partial);
                sa.h_in = (s == 0 && block_variant) ? h_in : nullptr;
                sa.h_out = (s == 0 && block_variant) ? h_out : nullptr;
                sa.tail_in = (s == 0 && block_variant) ? tail_in : nullptr;
                sa.L = d->seqlen; sa.Dn = d->d_inner; sa.H = d->n_heads; sa.HG = d->n_heads / d->n_groups;
                sa.G = d->n_groups; sa.K = d->d_conv; sa.tail_ch = tail_ch; sa.nchunk = plan.ssd_chunks;
                sa.parts = plan.ssd_parts; sa.part_chunks = plan.ssd_part_chunks;
                sa.part_subs = plan.ssd_part_subs; sa.sub_chunks = plan.ssd_sub_chunks;
                // (a call in one part enters it with the caller's state)
                sa.part_state = plan.ssd_parts > 1 ? reinterpret_cast<float*>(ws + plan.off_pstate[s]) : const_cast<float*>(sa.h_in);
                sa.part_decay = reinterpret_cast<float*>(ws + plan.off_pdecay[s]);
                sa.dir = s == 0 ? 1 : -1;
                sa.mode = separate ? kSsdFinalOnly
                                   : s == 1 ? (raw ? kSsdPartialRaw : kSsdPartial) : (raw ? kSsdFinalAddRaw : kSsdFinalAdd);
                sa.out_ch_off = separate ? s * d->d_inner : 0;
                sa.dt_softplus = d->dt_softplus; sa.d_per_head = d->d_kind == BIMAMBA_D_PER_HEAD;
                sa.far = far;
                sa.meet = meet; sa.lead = pp.dir[s].lead;
                return sa;
            };
            if (meet) {   // both directions at once: the halves they scan first, then, from the states left, the others' halves
                const int half = (plan.ssd_chunks + 1) / 2;   // the forward direction's chunks of the first launch
                SsdStatePair sp;
                for (int s = 0; s < 2; s++) {
                    sp.dir[s] = scan_args(s);
                    sp.dir[s].mode = raw ? kSsdPartialRaw : kSsdPartial;
                    sp.dir[s].first_chunk = 0;
                    sp.dir[s].part_chunks = s == 0 ? half : plan.ssd_chunks - half;
                    sp.dir[s].h_out = reinterpret_cast<float*>(ws + plan.off_pstate[s]);
                }
                if (launch_ssd_scan(d->d_state, d->d_inner / d->n_heads, sp, 2, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
                for (int s = 0; s < 2; s++) {
                    sp.dir[s] = scan_args(s);
                    sp.dir[s].mode = raw ? kSsdFinalAddRaw : kSsdFinalAdd;
                    sp.dir[s].first_chunk = s == 0 ? half : plan.ssd_chunks - half;
                    sp.dir[s].part_chunks = plan.ssd_chunks - sp.dir[s].first_chunk;
                    sp.dir[s].h_in = reinterpret_cast<const float*>(ws + plan.off_pstate[s]);
                }
                if (launch_ssd_scan(d->d_state, d->d_inner / d->n_heads, sp, 2, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
            }
            if (!meet && plan.ssd_parts > 1) {
                // time parts: every sub-part's end state from a zero start, then the states entering them
                SsdStatePair sp;
                SsdCarryArgs ca{};
                for (int s = 0; s < 2; s++) {
                    sp.dir[s] = scan_args(s);
                    ca.part_state[s] = sp.dir[s].part_state;
                    ca.part_decay[s] = sp.dir[s].part_decay;
                }
                launch_ssd_state(d->d_state, d->d_inner / d->n_heads, sp, plan.ssd_subs, d->batch, st);
                ca.h_in = block_variant ? h_in : nullptr;
                ca.batch = d->batch; ca.Dn = d->d_inner; ca.P = d->d_inner / d->n_heads; ca.H = d->n_heads;
                ca.parts = plan.ssd_subs;
                launch_ssd_carry(d->d_state, ca, st);
            }
            if (!meet) {
                const int head_width = d->d_inner / d->n_heads;
                SsdStatePair sp;
                sp.dir[1] = scan_args(1);
                if (!separate) {   // (the forward direction adds what the reverse one parked)
                    sp.dir[0] = sp.dir[1];
                    if (launch_ssd_scan(d->d_state, head_width, sp, 1, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
                }
                sp.dir[0] = scan_args(0);
                if (launch_ssd_scan(d->d_state, head_width, sp, separate ? 2 : 1, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
            }
            if (probe_stop) (void)hipEventRecord(probe_stop, st);
        } else {
        // 2. scan (summary + carry when the sequence is cut into segments) and combine
        SweepArgs sa{};
        for (int s = 0; s < 2; s++) {
            const bimamba_inputs* in = s == 0 ? in_f : in_b;
            const bimamba_params* p = s == 0 ? pf : pb;
            DirArgs& da = sa.dir[s];
            da.x = targ(in->x); da.z = targ(in->z); da.dt = targ(in->dt);
            da.bc = reinterpret_cast<const float*>(ws + plan.off_bc[s]);
            da.Braw = targ(in->B); da.Craw = targ(in->C);
            da.conv_w = p->conv_w; da.conv_b = p->conv_b; da.A = p->A; da.D = p->D; da.dt_bias = p->dt_bias;
        }
        sa.out = out->ptr; sa.out_sb = out->stride_batch; sa.out_st = out->stride_token;
        sa.partial = reinterpret_cast<float*>(ws + plan.off_partial);
        sa.h_in = block_variant ? h_in : nullptr;
        sa.h_out = block_variant ? h_out : nullptr;
        sa.tail_in = block_variant ? tail_in : nullptr;
        if (block_variant && one_launch && d->d_conv > 1) {
            sa.tail_out = tail_out;   // the forward walk of a short call ends with the tail in registers
            tail_out = nullptr;
        }
        sa.carry = reinterpret_cast<float*>(ws + plan.off_carry);
        sa.sumdt = reinterpret_cast<float*>(ws + plan.off_sumdt);
        sa.L = d->seqlen; sa.Dn = d->d_inner; sa.P = d->d_inner / d->n_heads; sa.HG = d->n_heads / d->n_groups;
        sa.G = d->n_groups; sa.K = d->d_conv; sa.nseg = plan.nseg; sa.seg_len = plan.seg_len; sa.tail_ch = tail_ch;
        sa.dt_softplus = d->dt_softplus; sa.d_per_head = d->d_kind == BIMAMBA_D_PER_HEAD;
        sa.separate = d->combine == BIMAMBA_COMBINE_SEPARATE;
        sa.raw_partial = !sa.separate && same_tensor(in_f->z, in_b->z);
        sa.same_bc = same_tensor(in_f->B, in_b->B) && same_tensor(in_f->C, in_b->C);
        sa.try_progression = decay_run(d);
        CarryArgs ca{};
        ca.carry = sa.carry; ca.sumdt = sa.sumdt; ca.A[0] = pf->A; ca.A[1] = pb->A;
        ca.h_in = sa.h_in; ca.h_out = sa.h_out;
        ca.batch = d->batch; ca.nseg = plan.nseg; ca.Dn = d->d_inner; ca.P = sa.P;
        if (launch_scan(d, plan.split, one_launch, sa, ca, st, probe_start, probe_stop) != hipSuccess) return BIMAMBA_ERR_HIP;
        }
        }
    } else if (block_variant && d->batch > 0 && h_out && h_out != h_in) {
        // empty block: the state passes through unchanged
        const size_t bytes = (size_t)d->batch * d->d_inner * d->d_state * sizeof(float);
        if (h_in) {
            (void)hipMemcpyAsync(h_out, h_in, bytes, hipMemcpyDeviceToDevice, st);
        } else {
            // a kernel rather than a memset node, so the call stays safe to capture into a HIP graph
            const long long n = (long long)d->batch * d->d_inner * d->d_state;
            hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, h_out, n);
        }
    }
    // 3. conv tail for the next block
    if (block_variant && tail_out && d->batch > 0 && d->d_conv > 1) {
        TailArgs ta{};
        ta.x = targ(in_f->x); ta.B = targ(in_f->B); ta.C = targ(in_f->C);
        ta.tail_in = tail_in; ta.tail_out = tail_out;
        ta.batch = d->batch; ta.L = d->seqlen; ta.K = d->d_conv; ta.Dn = d->d_inner; ta.GN = GN; ta.tail_ch = tail_ch;
        const long long total = (long long)d->batch * tail_ch;
        const dim3 grid((unsigned)((total + 255) / 256));
        if (d->io_dtype == BIMAMBA_BF16) hipLaunchKernelGGL(tail_kernel<IoBF16>, grid, dim3(256), 0, st, ta);
        else hipLaunchKernelGGL(tail_kernel<IoF32>, grid, dim3(256), 0, st, ta);
    }
    const hipError_t now = hipPeekAtLastError();
    return now == hipSuccess || now == pending ? BIMAMBA_OK : BIMAMBA_ERR_HIP;
}

// Whether a descriptor can take a stack of layers in one launch, and in which shape.
bool stack_call(const bimamba_desc* d, RowForm* row)
{
    return !use_ssd(d) && !d->conv_bc && d->time_chunks == 0 && d->state_split == 0 && d->combine == BIMAMBA_COMBINE_ADD &&
           d->batch > 0 && stack_form(d->batch, d->seqlen, d->d_inner, d->d_state, row);
}

StackArgs stack_args(const bimamba_desc* d, const RowForm& row, int n_layers, int n_steps)
{
    StackArgs sa{};
    sa.n_layers = n_layers; sa.n_steps = n_steps;
    sa.L = d->seqlen; sa.Dn = d->d_inner; sa.P = d->d_inner / d->n_heads; sa.HG = d->n_heads / d->n_groups;
    sa.G = d->n_groups; sa.N = d->d_state; sa.K = d->d_conv;
    sa.dt_softplus = d->dt_softplus; sa.d_per_head = d->d_kind == BIMAMBA_D_PER_HEAD;
    sa.a_scalar = d->a_kind == BIMAMBA_A_SCALAR_PER_HEAD;
    sa.tw = row.tw; sa.tw_log2 = row.tw == 4 ? 2 : row.tw == 2 ? 1 : 0; sa.nseg = row.nseg; sa.seg_len = row.seg_len;
    return sa;
}

// Buffers of one size, each with its owner: whether no two owners' overlap.
struct Owned {
    uintptr_t at;
    int owner;
};
bool owners_apart(Owned* r, int n, size_t bytes)
{
    std::sort(r, r + n, [](const Owned& x, const Owned& y) { return x.at < y.at; });
    int nearest = -1, other = -1;   // of what lies before: the last buffer, and the last one of another owner than its
    for (int i = 0; i < n; i++) {
        if (nearest >= 0 && r[nearest].owner != r[i].owner) other = nearest;
        nearest = i;
        if (other >= 0 && r[i].at - r[other].at < bytes) return false;
    }
    return true;
}

// Whether a stack's steps may go in any order beside each other: outputs of different steps, and states and tails of different layers,
// lie apart.
bool steps_apart(const bimamba_desc* d, const bimamba_stack_layer* layers, int n_layers, void* const* outs, int n_steps)
{
    const size_t elem = d->io_dtype == BIMAMBA_BF16 ? 2 : 4, channels = (size_t)d->batch * d->d_inner;
    const std::unique_ptr<Owned[]> r(new (std::nothrow) Owned[std::max((size_t)n_layers, (size_t)n_steps * n_layers)]);
    if (!r) return false;
    int n = 0;
    auto take = [&](const void* p, int owner) {
        if (p) r[n++] = Owned{reinterpret_cast<uintptr_t>(p), owner};
    };
    for (int i = 0; i < n_steps * n_layers; i++) take(outs[i], i / n_layers);
    if (!owners_apart(r.get(), n, channels * d->seqlen * elem)) return false;
    n = 0;
    for (int l = 0; l < n_layers; l++) take(layers[l].h, l);
    if (!owners_apart(r.get(), n, channels * d->d_state * sizeof(float))) return false;
    n = 0;
    for (int l = 0; l < n_layers; l++) take(d->d_conv > 1 ? layers[l].tail : nullptr, l);
    return owners_apart(r.get(), n, channels * (d->d_conv - 1) * elem);
}

int run_stack(const bimamba_desc* d, int n_layers, int n_steps, const void* table, const void* table_dev, void* hip_stream)
{
    int rc = check_desc(d);
    if (rc) return rc;
    if (n_layers < 0 || n_steps < 0) return BIMAMBA_ERR_BAD_SHAPE;
    RowForm row;
    if (!stack_call(d, &row)) return BIMAMBA_ERR_UNSUPPORTED;
    if (n_layers == 0 || n_steps == 0) return BIMAMBA_OK;
    if (!table || !table_dev) return BIMAMBA_ERR_NULL_POINTER;
    if (!is_aligned(table, 8) || !is_aligned(table_dev, 8)) return BIMAMBA_ERR_MISALIGNED;
    const size_t elem = d->io_dtype == BIMAMBA_BF16 ? 2 : 4;
    const auto* layers = static_cast<const bimamba_stack_layer*>(table);
    const auto* steps = reinterpret_cast<const bimamba_inputs*>(layers + n_layers);
    const auto* outs = reinterpret_cast<void* const*>(steps + n_steps);
    for (int l = 0; l < n_layers; l++) {
        if ((rc = check_params(&layers[l].f)) || (rc = check_params(&layers[l].b))) return rc;
        if (!is_aligned(layers[l].h, 4) || !is_aligned(layers[l].tail, elem)) return BIMAMBA_ERR_MISALIGNED;
    }
    for (int s = 0; s < n_steps; s++)
        if ((rc = check_inputs(&steps[s], d, elem))) return rc;
    const int gn = d->n_groups * d->d_state;
    for (int i = 0; i < n_steps * n_layers; i++) {
        if (!outs[i]) continue;
        if (!is_aligned(outs[i], elem)) return BIMAMBA_ERR_MISALIGNED;
        const bimamba_tensor o{outs[i], (int64_t)d->seqlen * d->d_inner, d->d_inner};
        for (int s = 0; s < n_steps; s++) {
            const bimamba_inputs& in = steps[s];
            if (may_overlap(o, d->d_inner, in.x, d->d_inner, elem, d) || may_overlap(o, d->d_inner, in.z, d->d_inner, elem, d) ||
                may_overlap(o, d->d_inner, in.dt, d->n_heads, elem, d) || may_overlap(o, d->d_inner, in.B, gn, elem, d) ||
                may_overlap(o, d->d_inner, in.C, gn, elem, d))
                return BIMAMBA_ERR_ALIAS;
        }
    }
    const hipError_t pending = hipPeekAtLastError();
    StackArgs sa = stack_args(d, row, n_layers, n_steps);
    sa.layers = static_cast<const bimamba_stack_layer*>(table_dev);
    sa.steps = reinterpret_cast<const bimamba_inputs*>(sa.layers + n_layers);
    sa.outs = reinterpret_cast<void* const*>(sa.steps + n_steps);
    const bool apart = steps_apart(d, layers, n_layers, outs, n_steps);
    if (launch_stack(d->io_dtype == BIMAMBA_BF16, sa, d->batch, apart, reinterpret_cast<hipStream_t>(hip_stream)) != hipSuccess) return BIMAMBA_ERR_HIP;
    const hipError_t now = hipPeekAtLastError();
    return now == hipSuccess || now == pending ? BIMAMBA_OK : BIMAMBA_ERR_HIP;
}

int copy_inputs(const bimamba_desc* d, const bimamba_inputs* from, const bimamba_inputs* to, void* hip_stream)
{
    int rc = check_desc(d);
    if (rc) return rc;
    const size_t elem = d->io_dtype == BIMAMBA_BF16 ? 2 : 4;
    if ((rc = check_inputs(from, d, elem))) return rc;
    if ((rc = check_inputs(to, d, elem))) return rc;
    if (d->batch == 0 || d->seqlen == 0) return BIMAMBA_OK;
    const int gn = d->n_groups * d->d_state;
    const bimamba_tensor src[5] = {from->x, from->z, from->dt, from->B, from->C}, dst[5] = {to->x, to->z, to->dt, to->B, to->C};
    const int width[5] = {d->d_inner, d->d_inner, d->n_heads, gn, gn};
    CopyArgs a{};
    a.batch = d->batch; a.L = d->seqlen;
    long long most = 0;
    for (int i = 0; i < 5; i++) {
        for (int j = 0; j < 5; j++)
            if (may_overlap(dst[i], width[i], src[j], width[j], elem, d) || (i != j && may_overlap(dst[i], width[i], dst[j], width[j], elem, d)))
                return BIMAMBA_ERR_ALIAS;
        auto side = [&](const bimamba_tensor& t) {
            return CopyArgs::Side{static_cast<char*>(t.ptr), (long long)(t.stride_batch * elem), (long long)(t.stride_token * elem)};
        };
        a.from[i] = side(src[i]);
        a.to[i] = side(dst[i]);
        a.width[i] = width[i];
        auto aligned = [&](const CopyArgs::Side& s) { return is_aligned(s.p, 16) && (s.sb | s.st) % 16 == 0; };
        a.vector[i] = aligned(a.from[i]) && aligned(a.to[i]);
        most = std::max(most, (long long)d->batch * d->seqlen * ((width[i] + 7) / 8));
    }
    const hipError_t pending = hipPeekAtLastError();
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    const dim3 grid((unsigned)((most + 255) / 256), 1, 5);
    if (elem == 2) hipLaunchKernelGGL(copy_inputs_kernel<unsigned short>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(copy_inputs_kernel<float>, grid, dim3(256), 0, st, a);
    const hipError_t now = hipPeekAtLastError();
    return now == hipSuccess || now == pending ? BIMAMBA_OK : BIMAMBA_ERR_HIP;
}

constexpr int kMaxScratchDevices = 64;
std::atomic<void*> g_scratch_addr[kMaxScratchDevices];   // per device: each GPU holds its own copy of the array

// The current device's copy of `scratch`, asked once per device with that device current.
int static_scratch(void** addr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return BIMAMBA_ERR_HIP;
    void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return BIMAMBA_ERR_HIP;
        g_scratch_addr[dev].store(p, std::memory_order_release);
    }
    *addr = p;
    return BIMAMBA_OK;
}

}  // namespace

extern "C" {

int bimamba_fwd(const bimamba_desc* desc, const bimamba_params* pf, const bimamba_params* pb,
                const bimamba_inputs* in_f, const bimamba_inputs* in_b, const bimamba_tensor* out, void* workspace,
                size_t workspace_bytes, void* hip_stream)
{
    return run(desc, pf, pb, in_f, in_b, nullptr, nullptr, nullptr, nullptr, out, workspace, workspace_bytes, hip_stream,
               false);
}

int bimamba_block_fwd(const bimamba_desc* desc, const bimamba_params* pf, const bimamba_params* pb,
                      const bimamba_inputs* in_f, const bimamba_inputs* in_b, const float* h_in, const void* tail_in,
                      float* h_out, void* tail_out, const bimamba_tensor* out, void* workspace, size_t workspace_bytes,
                      void* hip_stream)
{
    return run(desc, pf, pb, in_f, in_b, h_in, tail_in, h_out, tail_out, out, workspace, workspace_bytes, hip_stream,
               true);
}

int bimamba_block_fwd_static(const bimamba_desc* desc, const bimamba_params* pf, const bimamba_params* pb,
                             const bimamba_inputs* in_f, const bimamba_inputs* in_b, const float* h_in,
                             const void* tail_in, float* h_out, void* tail_out, const bimamba_tensor* out,
                             void* hip_stream)
{
    int rc = check_desc(desc);
    if (rc) return rc;
    if (make_plan(desc, false, true, SIZE_MAX).total > (size_t)BIMAMBA_STATIC_SCRATCH_BYTES) return BIMAMBA_ERR_SCRATCH_EXCEEDED;
    void* ws = nullptr;
    if ((rc = static_scratch(&ws))) return rc;
    return run(desc, pf, pb, in_f, in_b, h_in, tail_in, h_out, tail_out, out, ws, BIMAMBA_STATIC_SCRATCH_BYTES, hip_stream,
               true);
}

// ---- gradients -------------------------------------------------------------------------------------------------
namespace {
struct BwdPlan {
    int nseg, seg_len, seg_chunks, tiles;
    int tiles_per_group;
    size_t off_bc[2], off_state, off_state_w, off_seg_h, off_seg_d, off_seg_w, off_params, off_parked, off_part[2], total;
};

int check_bwd_desc(const bimamba_desc* d)
{
    const int rc = check_desc(d);
    if (rc) return rc;
    if (d->n_heads != d->d_inner || d->a_kind != BIMAMBA_A_PER_HEAD_STATE || d->d_kind != BIMAMBA_D_PER_CHANNEL ||
        d->conv_bc || !bm::bwd_supported(d->d_state))
        return BIMAMBA_ERR_UNSUPPORTED;
    return BIMAMBA_OK;
}

BwdPlan make_bwd_plan(const bimamba_desc* d)
{
    BwdPlan p{};
    bm::bwd_segments(d->d_inner, d->batch, d->seqlen, &p.nseg, &p.seg_len, &p.seg_chunks);
    p.tiles = (d->d_inner + 63) / 64;
    const size_t bc = align_up((size_t)d->batch * d->seqlen * d->n_groups * 2 * d->d_state * sizeof(float), 256);
    // (the walk fetches parked rows two tokens ahead, past a sequence's ends: rows to spare on both sides)
    constexpr int kSpareRows = 16;
    const size_t parked = align_up(((size_t)d->batch * d->seqlen + 2 * kSpareRows) * d->d_inner * sizeof(Parked), 256);
    const size_t segs = (size_t)2 * d->batch * p.nseg, row = (size_t)p.tiles * 64 * sizeof(float);   // (one float per chain)
    size_t off = 0;
    p.off_bc[0] = off; off += bc;
    p.off_bc[1] = off; off += bc;    // sized for separate activations
    p.off_state = off; off += segs * p.seg_chunks * row * d->d_state;
    p.off_state_w = off; off += segs * p.seg_chunks * row;
    p.off_seg_h = off; off += segs * row * d->d_state;
    p.off_seg_d = off; off += segs * row * d->d_state;
    p.off_seg_w = off; off += 2 * segs * row;
    p.off_params = off; off += segs * row * (d->d_state + bm::kBwdParams);
    p.off_parked = off + (size_t)kSpareRows * d->d_inner * sizeof(Parked); off += parked;
    // per-wave partial sums of dB | dC: one slot per channel tile of a group and direction
    p.tiles_per_group = (d->d_inner / d->n_groups + 63) / 64;
    const size_t part = align_up((size_t)d->batch * d->seqlen * d->n_groups * p.tiles_per_group * 2 * d->d_state * sizeof(float), 256);
    p.off_part[0] = off; off += part;
    p.off_part[1] = off; off += part;
    p.total = off;
    return p;
}
}  // namespace

int bimamba_bwd(const bimamba_desc* d, const bimamba_params* pf, const bimamba_params* pb, const bimamba_inputs* in_f,
                const bimamba_inputs* in_b, const bimamba_tensor* dout, const bimamba_input_grads* din_f,
                const bimamba_input_grads* din_b, const bimamba_param_grads* dpf, const bimamba_param_grads* dpb,
                void* workspace, size_t workspace_bytes, void* hip_stream)
{
    int rc = check_bwd_desc(d);
    if (rc) return rc;
    const size_t elem = d->io_dtype == BIMAMBA_BF16 ? 2 : 4;
    if ((rc = check_params(pf))) return rc;
    if ((rc = check_params(pb))) return rc;
    if (!in_f || !dout || !din_f || !dpf || !dpb) return BIMAMBA_ERR_NULL_POINTER;
    if (!in_b) in_b = in_f;
    if ((rc = check_inputs(in_f, d, elem))) return rc;
    if ((rc = check_inputs(in_b, d, elem))) return rc;
    const bool shared = same_inputs(in_f, in_b);
    if (shared ? din_b != nullptr && din_b != din_f : din_b == nullptr) return BIMAMBA_ERR_NULL_POINTER;
    if (shared) din_b = nullptr;
    const int out_ch = d->combine == BIMAMBA_COMBINE_SEPARATE ? 2 * d->d_inner : d->d_inner;
    if ((rc = check_tensor(*dout, out_ch, elem, d))) return rc;
    const bool live = d->batch > 0 && d->seqlen > 0;
    for (const bimamba_input_grads* g : {din_f, din_b}) {
        if (!g) continue;
        if ((rc = check_tensor(g->dx, d->d_inner, elem, d))) return rc;
        if ((rc = check_tensor(g->dz, d->d_inner, elem, d))) return rc;
        if ((rc = check_tensor(g->ddt, d->n_heads, elem, d))) return rc;
        if (live && (!g->dB || !g->dC)) return BIMAMBA_ERR_NULL_POINTER;
        if (!is_aligned(g->dB, 4) || !is_aligned(g->dC, 4)) return BIMAMBA_ERR_MISALIGNED;
    }
    if (dpf == dpb) return BIMAMBA_ERR_ALIAS;
    for (const bimamba_param_grads* g : {dpf, dpb}) {
        if (!g->dconv_w || !g->dA || !g->dD) return BIMAMBA_ERR_NULL_POINTER;
        if (!is_aligned(g->dconv_w, 4) || !is_aligned(g->dA, 4) || !is_aligned(g->dD, 4) || !is_aligned(g->dconv_b, 4) ||
            !is_aligned(g->ddt_bias, 4))
            return BIMAMBA_ERR_MISALIGNED;
    }
    const BwdPlan plan = make_bwd_plan(d);
    if (!workspace) return BIMAMBA_ERR_NULL_POINTER;
    if (!is_aligned(workspace, 16)) return BIMAMBA_ERR_MISALIGNED;
    if (workspace_bytes < plan.total) return BIMAMBA_ERR_WORKSPACE_TOO_SMALL;

    const hipError_t pending = hipPeekAtLastError();
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    const int GN = d->n_groups * d->d_state;
    const bool bf16 = d->io_dtype == BIMAMBA_BF16;

    bm::BwdSumArgs sum{};
    sum.N = d->d_state; sum.Dn = d->d_inner; sum.K = d->d_conv;
    for (int s = 0; s < 2; s++) {
        const bimamba_param_grads* g = s == 0 ? dpf : dpb;
        sum.dA[s] = g->dA; sum.dD[s] = g->dD; sum.dconv_w[s] = g->dconv_w; sum.dconv_b[s] = g->dconv_b; sum.ddt_bias[s] = g->ddt_bias;
    }
    if (live) {
        bm::BwdPrepArgs pa{};
        bm::BwdArgs a{};
        for (int s = 0; s < 2; s++) {
            const bimamba_inputs* in = s == 0 ? in_f : in_b;
            const bimamba_params* p = s == 0 ? pf : pb;
            const bimamba_input_grads* gi = (s == 0 || !din_b) ? din_f : din_b;
            const int set = shared ? 0 : s;
            pa.B[set] = targ(in->B); pa.C[set] = targ(in->C);
            pa.dst[set] = reinterpret_cast<float*>(ws + plan.off_bc[set]);
            DirArgs& da = a.dir[s];
            da.x = targ(in->x); da.z = targ(in->z); da.dt = targ(in->dt);
            da.bc = pa.dst[set];
            da.conv_w = p->conv_w; da.conv_b = p->conv_b; da.A = p->A; da.D = p->D; da.dt_bias = p->dt_bias;
            // shared activations: both directions' waves fill slots of one buffer (the two parts are adjacent)
            a.bc_part[s] = reinterpret_cast<float*>(ws + plan.off_part[set]);
            a.gdx[s] = targ(gi->dx); a.gdz[s] = targ(gi->dz); a.gddt[s] = targ(gi->ddt);
            sum.part[set] = a.bc_part[s];
            sum.dB[set] = gi->dB; sum.dC[set] = gi->dC;
        }
        const int sets = shared ? 1 : 2;
        pa.L = d->seqlen; pa.G = d->n_groups; pa.N = d->d_state;
        pa.per_set = (long long)d->batch * d->seqlen * 2 * GN;
        bm::launch_bwd_prep(bf16, pa, sets, st);
        a.dout = targ(*dout);
        a.state = reinterpret_cast<float*>(ws + plan.off_state);
        a.state_w = reinterpret_cast<float*>(ws + plan.off_state_w);
        a.seg_h = reinterpret_cast<float*>(ws + plan.off_seg_h);
        a.seg_d = reinterpret_cast<float*>(ws + plan.off_seg_d);
        a.seg_w = reinterpret_cast<float*>(ws + plan.off_seg_w);
        a.param_part = reinterpret_cast<float*>(ws + plan.off_params);
        a.parked = reinterpret_cast<bm::Parked*>(ws + plan.off_parked);
        a.L = d->seqlen; a.Dn = d->d_inner; a.G = d->n_groups; a.K = d->d_conv;
        a.nseg = plan.nseg; a.seg_len = plan.seg_len; a.seg_chunks = plan.seg_chunks; a.tiles = plan.tiles;
        a.dt_softplus = d->dt_softplus; a.separate = d->combine == BIMAMBA_COMBINE_SEPARATE;
        a.park = shared;
        a.bc_slots = plan.tiles_per_group * (shared ? 2 : 1);
        a.bc_slot_of_rev = shared ? plan.tiles_per_group : 0;
        if (bm::launch_bwd(d->d_state, bf16, a, d->batch, st) != hipSuccess) return BIMAMBA_ERR_HIP;
        sum.sets = sets; sum.slots = a.bc_slots;
        sum.rows = (long long)d->batch * d->seqlen * d->n_groups;
        sum.param_part = a.param_part;
        sum.pitch = (long long)plan.tiles * 64;
        sum.segs = d->batch * plan.nseg;
    }
    bm::launch_bwd_sum(sum, st);   // an empty call's parameter gradients are zero
    const hipError_t now = hipPeekAtLastError();
    return (now == hipSuccess || now == pending) ? BIMAMBA_OK : BIMAMBA_ERR_HIP;
}

size_t bimamba_bwd_workspace_bytes(const bimamba_desc* desc)
{
    if (check_bwd_desc(desc)) return 0;
    return make_bwd_plan(desc).total;
}

size_t bimamba_workspace_bytes(const bimamba_desc* desc, int block_variant)
{
    if (check_desc(desc)) return 0;
    // sized for the larger case (the two directions reading different activations)
    return make_plan(desc, false, block_variant != 0, SIZE_MAX).total;
}

int bimamba_block_stack(const bimamba_desc* desc, int n_layers, int n_steps, const void* table, const void* table_dev, void* hip_stream)
{
    return run_stack(desc, n_layers, n_steps, table, table_dev, hip_stream);
}

int bimamba_block_stack_form(const bimamba_desc* desc)
{
    RowForm row;
    return check_desc(desc) == BIMAMBA_OK && stack_call(desc, &row);
}

int bimamba_block_stack_side_by_side(const bimamba_desc* desc, int n_steps)
{
    RowForm row;
    if (check_desc(desc) != BIMAMBA_OK || n_steps < 1 || !stack_call(desc, &row)) return 0;
    return bm::stack_side_by_side(stack_args(desc, row, 1, n_steps), desc->batch);
}

int bimamba_copy_inputs(const bimamba_desc* desc, const bimamba_inputs* from, const bimamba_inputs* to, void* hip_stream)
{
    return copy_inputs(desc, from, to, hip_stream);
}

int bimamba_time_chunks(const bimamba_desc* desc)
{
    if (check_desc(desc)) return 0;
    const Plan p = make_plan(desc, true, false, SIZE_MAX);
    RowForm row;
    return p.ssd ? (p.ssd_meet ? 1 : p.ssd_parts) : row_call(desc, p, &row) ? 1 : p.nseg;
}

void bimamba_profile_next_call(void* ev_start, void* ev_stop)
{
    g_probe_start = reinterpret_cast<hipEvent_t>(ev_start);
    g_probe_stop = reinterpret_cast<hipEvent_t>(ev_stop);
}

const char* bimamba_status_string(int status)
{
    switch (status) {
        case BIMAMBA_OK: return "ok";
        case BIMAMBA_ERR_NULL_POINTER: return "a required pointer is NULL";
        case BIMAMBA_ERR_BAD_SHAPE: return "bad shape: non-positive or inconsistent dimension or stride";
        case BIMAMBA_ERR_UNSUPPORTED: return "unsupported dtype, d_state, d_conv, grouping or token stride";
        case BIMAMBA_ERR_MISALIGNED: return "misaligned pointer";
        case BIMAMBA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case BIMAMBA_ERR_HIP: return "HIP launch error";
        case BIMAMBA_ERR_ALIAS: return "the output overlaps an input";
        case BIMAMBA_ERR_SCRATCH_EXCEEDED: return "the call needs more scratch than the library's static buffer holds";
        default: return "unknown status";
    }
}

int bimamba_version(void) { return BIMAMBA_VERSION; }

}  // extern "C"
