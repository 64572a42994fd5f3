// Calls of up to 64 tokens with enough chains for one lane each (up to 16 states, no conv on B and C), in one launch.
//
// A block step of many chains is vector work (11 us of the call below) and the waits between its parts: the first loads, the loads
// of the second half of the walk and of what the other direction left for it, the commit.  Here everything a wave needs first is requested
// before any of it is used, the token tiles are requested one ahead also across the meeting of the directions, B|C rows go to LDS as
// fp32 once per workgroup (no copy per wave, no preparation launch), and what one direction leaves for the other stays in LDS.  16 x 32 tokens,
// d_inner 4096, 16 states, committing: 23.9 -> 17.3 us against a walk by the long sweep's token loop with a copy of the rows per
// wave and the partial sums in memory; 64 x 64 tokens 137 -> 93, 32 x 32 with 8 states 33.9 -> 22.5, 32 x 1 token 15.3 -> 12.6.
//
// A workgroup is four waves, the two directions of two adjacent tiles of 64 channels, as in kernels.h; the arithmetic of a token is
// that of token_step there, with the output's dot product in two sums.
#pragma once
#include "kernels.h"

namespace bm {

constexpr int kShortTile = 8;   // tokens whose loads are in flight while the tile before is computed

// What the directions do with a token: kShortAdd parks and adds gated values, kShortAddRaw ungated ones (both directions gate with
// the same z: gated once, at the store), kShortSeparate stores to halves of its own.
constexpr int kShortAdd = 0, kShortAddRaw = 1, kShortSeparate = 2;

// LDS of a workgroup, in floats: B|C rows [pair of waves, if their tiles may lie in two groups][direction, if they differ][L][2N], then
// what the directions leave for each other, [pair][L][64].  (A row to spare in front and one behind: the walk reads one ahead.)
struct ShortLds {
    int rows, pair_rows, dir_rows, park, total;
    __host__ __device__ ShortLds(int L, int N, bool two_sets, bool two_groups, bool separate)
    {
        dir_rows = two_sets ? L * 2 * N : 0;
        const int sets = L * 2 * N + dir_rows;
        pair_rows = two_groups ? sets : 0;
        rows = 2 * N;
        park = rows + sets + pair_rows + 2 * N;
        total = park + (separate ? 0 : 2 * L * 64);
    }
};

// Waits for this wave's LDS traffic, not for the loads it has requested ahead.
__device__ __forceinline__ void short_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int N, int AKIND, int KIND, typename IO, int RUN>
__device__ __forceinline__ void short_walk(const SweepArgs& a, float* lds_all)
{
    using T = typename IO::T;
    // (general decays of 16 states: half a tile, which leaves their factors room in the registers of three waves a SIMD; 64 x 64
    // tokens, d_inner 4096: two waves 129 us, three with a whole tile's spills 131, so 119)
    constexpr int TILE = AKIND == kAPerState && N >= 16 ? kShortTile / 2 : kShortTile;
    constexpr int kRun = RUN > 0 && RUN < N ? RUN : N;
    constexpr bool kSeparate = KIND == kShortSeparate, kRaw = KIND == kShortAddRaw;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int s = w & 1, b = blockIdx.z, L = a.L, last = L - 1;
    const DirArgs& da = a.dir[s];
    const bool two_sets = !a.same_bc, two_groups = a.G > 1;
    const ShortLds lds(L, N, two_sets, two_groups, kSeparate);
    // Lanes past the last channel shadow channel Dn - 1, waves past the last tile the last tile: same inputs, same values, same
    // addresses.
    const int ch = min(tile_of_wave<1>(w, a.Dn) * 64 + lane, a.Dn - 1);
    const int head = ch / a.P;
    const int step = s == 0 ? 1 : -1, tstart = s == 0 ? 0 : last;
    const int n_first = kSeparate ? 0 : s == 0 ? (L + 1) / 2 : L / 2;   // tokens left for the other direction

    // ---- what a wave needs first, all requested before any of it is used
    const T* const xb = (const T*)da.x.p + (size_t)b * da.x.sb + (long long)tstart * da.x.st;
    const T* const zb = (const T*)da.z.p + (size_t)b * da.z.sb + (long long)tstart * da.z.st;
    const T* const db = (const T*)da.dt.p + (size_t)b * da.dt.sb + (long long)tstart * da.dt.st;
    T* const ob = (T*)a.out + (size_t)b * a.out_sb + (long long)tstart * a.out_st + (kSeparate ? s * a.Dn : 0);
    const long long xs = step * da.x.st, zs = step * da.z.st, ds = step * da.dt.st, os = step * a.out_st;
    const unsigned ch_io = (unsigned)ch * (unsigned)sizeof(T), head_io = (unsigned)head * (unsigned)sizeof(T);
    struct Tile {
        T x[TILE], d[TILE], z[TILE];
    };
    Tile next;
#pragma unroll
    for (int i = 0; i < TILE; i++) next.x[i] = next.d[i] = next.z[i] = 0;
    auto request = [&](int j0, bool gated) {
        const TileRows<TILE> tx = tile_rows<TILE>(xb + j0 * xs, xs), td = tile_rows<TILE>(db + j0 * ds, ds);
#pragma unroll
        for (int i = 0; i < TILE; i++) {
            next.x[i] = IO::ld_raw(tx.range, ch_io, tx.row(i));
            next.d[i] = IO::ld_raw(td.range, head_io, td.row(i));
        }
        if (gated) {
            const TileRows<TILE> tz = tile_rows<TILE>(zb + j0 * zs, zs);
#pragma unroll
            for (int i = 0; i < TILE; i++) next.z[i] = IO::ld_raw(tz.range, ch_io, tz.row(i));
        }
    };
    // The walk is two ranges, [0, n_first) and [n_first, L), each of whole tiles and single tokens after them; the request of a
    // tile is made one tile ahead, that of the second range's first tile during the first range.
    const int first_tile = n_first >= TILE ? 0 : n_first;
    if (first_tile + TILE <= L) request(first_tile, !kRaw || first_tile == n_first);
    // B|C rows, each thread one column of every kRows-th token.  The sets (pair of waves, direction) are at most four and uniform.
    constexpr int kRows = 256 / (2 * N), kPer = kShortCallTokens / kRows;
    const int col = tid % (2 * N), row0 = tid / (2 * N);
    auto stage_set = [&](int pair, int set) {
        const int grp = (tile_of_wave<1>(2 * pair, a.Dn) * 64) / a.P / a.HG;   // a tile lies in one group
        const DirArgs& src = a.dir[set];
        const T* const from = (col < N ? (const T*)src.Braw.p + (size_t)b * src.Braw.sb : (const T*)src.Craw.p + (size_t)b * src.Craw.sb) +
                              grp * N + col % N;
        const long long st = col < N ? src.Braw.st : src.Craw.st;
        float* const to = lds_all + lds.rows + pair * lds.pair_rows + set * lds.dir_rows + col;
        T v[kPer];
#pragma unroll
        for (int k = 0; k < kPer; k++)
            v[k] = from[min(k * kRows + row0, last) * st];
#pragma unroll
        for (int k = 0; k < kPer; k++)
            if (k * kRows + row0 < L) to[(k * kRows + row0) * 2 * N] = IO::cvt(v[k]);
    };
    stage_set(0, 0);
    if (two_sets) stage_set(0, 1);
    if (two_groups) {
        stage_set(1, 0);
        if (two_sets) stage_set(1, 1);
    }
    float w4[4], h[N], a2[AKIND == kAPerState ? N : AKIND == kAProgression ? N / kRun : 1], d2 = 0.0f;
    load_taps(da.conv_w + (size_t)ch * a.K, a.K, w4);
    const float cb = da.conv_b ? da.conv_b[ch] : 0.0f;
    const float dval = da.D[a.d_per_head ? head : ch];
    const float dtb = (a.dt_softplus && da.dt_bias) ? da.dt_bias[head] : 0.0f;
    if constexpr (AKIND == kAPerState) {
#pragma unroll
        for (int n = 0; n < N; n++) a2[n] = da.A[(size_t)head * N + n] * kLog2e;
    } else if constexpr (AKIND == kAProgression) {
#pragma unroll
        for (int n = 0; n < N; n += kRun) a2[n / kRun] = da.A[(size_t)head * N + n] * kLog2e;
        d2 = (da.A[(size_t)head * N + 1] - da.A[(size_t)head * N]) * kLog2e;
    } else {
        a2[0] = da.A[head] * kLog2e;
    }
    const size_t h_at = ((size_t)b * a.Dn + ch) * N;
#pragma unroll
    for (int n = 0; n < N; n++) h[n] = 0.0f;
    if (s == 0 && a.h_in) {
#pragma unroll
        for (int n = 0; n < N; n++) h[n] = a.h_in[h_at + n];
    }
    // conv history: the raw tokens before the walk's first one, most recent first (the cached tail, or zeros)
    float xh[3] = {0.0f, 0.0f, 0.0f};
    if (s == 0 && a.tail_in && a.K > 1) {
        T cached[3];
#pragma unroll
        for (int i = 0; i < 3; i++) cached[i] = ((const T*)a.tail_in)[((size_t)b * (a.K - 1) + max(a.K - 2 - i, 0)) * a.tail_ch + ch];
#pragma unroll
        for (int i = 0; i < 3; i++) xh[i] = i < a.K - 1 ? IO::cvt(cached[i]) : 0.0f;
    }
    const bool sp = a.dt_softplus != 0;
    short_barrier();   // B|C rows

    // (places in LDS as running byte offsets of the lane: an addition a token)
    unsigned row_at = (unsigned)(lds.rows + (w >> 1) * lds.pair_rows + s * lds.dir_rows + tstart * 2 * N) * 4u;
    unsigned park_at = (unsigned)(lds.park + ((w >> 1) * L + tstart) * 64 + lane) * 4u;
    keep_narrow(row_at);
    keep_narrow(park_at);
    const unsigned row_step = (unsigned)(step * 2 * N * 4), park_step = (unsigned)(step * 64 * 4);
    auto load_row = [&](BcRow<N>& r) { load_bc_lds<N, 1>(lane_elem((const float*)lds_all, row_at), 0, 0, r); };
    BcRow<N> row;
    load_row(row);
    // One token of the walk: y before the gate.
    auto token = [&](T xraw, float delta) {
        asm volatile("" ::: "memory");   // one row of B|C ahead, not a tile of them: they would not fit the registers
        BcRow<N> row_next;
        row_at += row_step;
        load_row(row_next);
        const float x0 = IO::cvt(xraw);
        const float pre = fmaf(w4[3], x0, fmaf(w4[2], xh[0], fmaf(w4[1], xh[1], fmaf(w4[0], xh[2], cb))));
        xh[2] = xh[1];
        xh[1] = xh[0];
        xh[0] = x0;
        const float xc = silu(pre), u = delta * xc;
        float y[2] = {dval * xc, 0.0f};   // (the second starts with a product)
        float an = 1.0f, ratio = 1.0f;
        if constexpr (AKIND == kAScalar) an = fast_exp2(delta * a2[0]);
        if constexpr (AKIND == kAProgression) ratio = fast_exp2(delta * d2);
#pragma unroll
        for (int n = 0; n < N; n++) {
            if constexpr (AKIND == kAPerState) an = fast_exp2(delta * a2[n]);
            if (AKIND == kAProgression && n % kRun == 0) an = fast_exp2(delta * a2[n / kRun]);
            h[n] = fmaf(an, h[n], u * row.v[n]);
            y[n & 1] = n == 1 ? row.v[N + n] * h[n] : fmaf(row.v[N + n], h[n], y[n & 1]);
            if (AKIND == kAProgression && (n + 1) % kRun != 0) an *= ratio;
        }
        row = row_next;
        return y[0] + y[1];
    };
    auto leave = [&](float y, T zraw) {
        *lane_elem(lds_all, park_at) = kRaw ? y : y * silu(IO::cvt(zraw));
        park_at += park_step;
    };
    auto finish = [&](float y, T zraw) {
        const float zg = silu(IO::cvt(zraw));
        float v = kRaw ? 0.0f : y * zg;
        if constexpr (!kSeparate) {
            const float part = *lane_elem(lds_all, park_at);
            park_at += park_step;
            v = kRaw ? (y + part) * zg : v + part;
        }
        return v;
    };
    auto range = [&](auto final_tag, int j, const int end) {
        constexpr bool kFinal = decltype(final_tag)::value;
        for (; j + TILE <= end; j += TILE) {
            const Tile cur = next;
            if (j + 2 * TILE <= end) request(j + TILE, kFinal || !kRaw);
            else if (!kFinal && end + TILE <= L) request(end, true);
            float delta[TILE];
#pragma unroll
            for (int i = 0; i < TILE; i++) delta[i] = IO::cvt(cur.d[i]);
            if (sp) {
#pragma unroll
                for (int i = 0; i < TILE; i++) delta[i] = softplus(delta[i] + dtb);
            }
            const TileRows<TILE> to = tile_rows<TILE>(ob + j * os, os);
#pragma unroll
            for (int i = 0; i < TILE; i++) {
                const float y = token(cur.x[i], delta[i]);
                if constexpr (kFinal) IO::st_raw(to.range, ch_io, to.row(i), finish(y, cur.z[i]));
                else leave(y, cur.z[i]);
            }
        }
#pragma unroll 1
        for (; j < end; j++) {
            const T xraw = *lane_elem(xb + j * xs, ch_io), draw = *lane_elem(db + j * ds, head_io);
            const T zraw = kFinal || !kRaw ? *lane_elem(zb + j * zs, ch_io) : (T)0;
            float delta = IO::cvt(draw);
            if (sp) delta = softplus(delta + dtb);
            const float y = token(xraw, delta);
            if constexpr (kFinal) IO::st(lane_elem(ob + j * os, ch_io), finish(y, zraw));
            else leave(y, zraw);
        }
    };
    if constexpr (!kSeparate) {
        range(std::false_type{}, 0, n_first);
        short_barrier();   // what the other direction left is there
    }
    range(std::true_type{}, n_first, L);
    // Waves past the last tile shadow it: all have read h_in and tail_in before any of them commits over it (with the halves
    // together the barrier in the middle of the walk came after those reads).
    if (kSeparate && (a.h_out || a.tail_out)) __syncthreads();
    if (s == 0 && a.h_out) {
#pragma unroll
        for (int n = 0; n < N; n++) a.h_out[h_at + n] = h[n];
    }
    // The conv tail is the window the forward walk leaves, raw tokens, so cutting the fp32 form back to the I/O dtype restores
    // their bits.
    if (s == 0 && a.tail_out) {
        T* dst = (T*)a.tail_out + (size_t)b * (a.K - 1) * a.tail_ch + ch;
#pragma unroll
        for (int i = 0; i < 3; i++)
            if (i < a.K - 1) dst[(size_t)(a.K - 2 - i) * a.tail_ch] = io_bits<IO>(xh[i]);
    }
}

// grid (ceil(ceil(Dn / 64) / 2), 1, batch), block 256, dynamic LDS ShortLds::total floats.  Three waves a SIMD: with the nine to twelve
// registers more that the compiler would take, launches of many workgroups hold two (64 x 64 tokens 103 us, 64 x 16 43 -> 38).
//
// RUN: how many states the decays of an arithmetic A are products over before the next exponential; 0: an exponential each, whatever
// A.  The ratio's own rounding grows with the run.  Relative error of the committed state against 64 bits, 20480 chains of 16 states, 16 / 32
// / 64 tokens: runs of sixteen 8.2 / 12.7 / 17.6e-7, of eight 4.6 / 7.6 / 12.0e-7, none 1.3 / 1.8 / 2.8e-7; 16 x 32 tokens, d_inner 4096:
// 17.3, 17.7 and 20.7 us.  A call takes no longer run than the other forms of its size do (decay_run in bimamba_api.hip).
template <int N, int AKIND, int KIND, typename IO, int RUN>
__global__ __launch_bounds__(256, 3) void short_kernel(const SweepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float short_lds[];
    if constexpr (RUN > 0) {   // the progression form if all of a wave's chains qualify, as in sweep_kernel
        const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int ch = min(tile_of_wave<1>(w, a.Dn) * 64 + (int)(threadIdx.x & 63), a.Dn - 1);
        const float* row = a.dir[w & 1].A + (size_t)(ch / a.P) * N;
        const float first = row[0], step = row[1] - row[0];
        bool ok = true;
#pragma unroll
        for (int n = 0; n < N; n++) ok &= row[n] == fmaf((float)n, step, first);
        if (__all(ok)) {
            short_walk<N, kAProgression, KIND, IO, RUN>(a, short_lds);
            return;
        }
    }
    short_walk<N, AKIND, KIND, IO, 0>(a, short_lds);
}

}  // namespace bm
