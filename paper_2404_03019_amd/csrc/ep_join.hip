// The segments that cross block edges of an element-parallel first pass, joined in one launch.
//
// Block c of the pass leaves, in slot 2c ("lo") and slot 2c + 1 ("hi") of a sorted list, the partial
// of a segment that began before it and that of one that goes on behind it (count 0: none). A
// crossing segment is therefore one hi partial and the lo partials of the blocks it reaches into:
// for segments shorter than a block, of exactly one. A row group per block c loads its hi partial
// and the next block's lo partial together with their ids and counts (one trip to memory) and
// stores their combination; a segment that reaches further than kAhead blocks is left to a wave,
// whose groups take its lo partials in turn, and one of more than kTrips such turns to the whole
// thread block. (Left to the block at once, the segments of a power law waited for each other: 56
// against 48 us for the whole call by levels at 2,000,000 rows of 16 columns.)
//
// Bound by latency (a launch and one or two trips to memory), as the partial levels are, but it is
// one launch where they are two or three: 3,908 partials of 16 columns 4.0 us against 7.4 + 3.9,
// 4,688 of 128 columns 4.9 against 6.9 + 4.8 + 4.5. The levels keep the inputs with many partials, or with
// segments that cross many blocks each, which they reduce in logarithmic depth. One segment of half of all
// rows is read by one block here, which makes the call 1 to 20 % slower than by levels.
#include <type_traits>

#include "common.h"

namespace geot {

namespace {

constexpr int kJoinBlock = 512;
constexpr int kAhead = 4;   // lo partials whose ids a group looks at before it leaves a segment to a wave
constexpr int kTrips = 4;   // turns of a wave (4 partials per group each) before it leaves a segment to the block
constexpr int kDeep = 16;   // partials per group and turn there

// (v, i) takes in another partial's maximum and recipient, in any order: the larger value, of
// equal ones the lower row
__device__ __forceinline__ void join_arg(float &v, uint32_t &i, float b, uint32_t ib) {
    const bool take = ib != kNoRecipient && (i == kNoRecipient || b > v || (b == v && ib < i));
    i = take ? ib : i;
    v = __builtin_elementwise_maximum(v, b);
}

template <int RED, int V>
__global__ __launch_bounds__(kJoinBlock) void ep_join_kernel(const EpArgs a, const int64_t chunks, const int64_t nblk,
                                                             const int64_t gap_tw) {
    constexpr bool ARG = RED == RED_MAXARG;
    constexpr int NX = ARG ? V : 1;
    __shared__ float s_v[kJoinBlock * V];
    __shared__ uint32_t s_x[ARG ? kJoinBlock * V : 1];
    __shared__ int64_t s_n[kJoinBlock];
    __shared__ int s_long[kJoinBlock], s_longer[kJoinBlock];
    __shared__ int s_nlong, s_nlonger;
    if ((int64_t)blockIdx.x >= nblk) {   // the extra blocks write the runs of empty segments the pass listed
        gap_fill_rows_body<V>(a.out, a.F, a.ld_out, gap_tw, a.S, a.gaps, (int64_t)blockIdx.x - nblk,
                              (int64_t)gridDim.x - nblk, a.arg_out);
        return;
    }
    const int nvec = (int)((a.F + V - 1) / V);
    int tpr = 1;   // threads per partial
    while (tpr < nvec && tpr < 64) tpr <<= 1;
    const int groups = kJoinBlock / tpr, g = (int)threadIdx.x / tpr, j0 = (int)threadIdx.x % tpr;
    if (threadIdx.x == 0) s_nlong = s_nlonger = 0;
    __syncthreads();
    const float neutral = red_neutral<RED>();
    // vector j's first column; the one that would cross the row's end takes the row's last V columns
    auto column = [&](int j) { return min((int64_t)j * V, a.F - V); };
    auto load = [&](int64_t slot, int j, bool ok, float *x, uint32_t *xi) {
        if (ok) {
            load_vec<V>(a.pv + slot * a.ld_p + column(j), x);
            if constexpr (ARG) {
                float t[V];
                load_vec<V>(reinterpret_cast<const float *>(a.pix + slot * a.ld_p + column(j)), t);
#pragma unroll
                for (int k = 0; k < V; ++k) xi[k] = __float_as_uint(t[k]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < V; ++k) x[k] = neutral;
#pragma unroll
            for (int k = 0; k < NX; ++k) xi[k] = kNoRecipient;
        }
    };
    auto take = [&](float *v, uint32_t *vi, const float *x, const uint32_t *xi) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if constexpr (ARG) join_arg(v[k], vi[k], x[k], xi[k]);
            else v[k] = red_apply<RED>(v[k], x[k]);
        }
    };
    auto store = [&](int32_t seg, int j, float *v, const uint32_t *vi, int64_t n) {
        if (seg < 0 || (int64_t)seg >= a.S) return;   // an id out of range
        if constexpr (ARG) {
            float t[V];
#pragma unroll
            for (int k = 0; k < V; ++k) t[k] = __uint_as_float(v[k] != v[k] ? kNoRecipient : vi[k]);   // NaN has none
            store_vec<V>(reinterpret_cast<float *>(a.arg_out + (int64_t)seg * a.ld_out + column(j)), t);
        }
        if (a.mean) {
            const float fn = (float)n;
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] = v[k] / fn;
        }
        store_vec<V>(a.out + (int64_t)seg * a.ld_out + column(j), v);
    };

    // segment ids are below 2^31 and a block's counts too: their low words
    const int32_t *ids32 = reinterpret_cast<const int32_t *>(a.pseg), *cnt32 = reinterpret_cast<const int32_t *>(a.pcnt);
    auto seg_of = [&](int64_t slot) { return ids32[2 * slot]; };
    auto count_of = [&](int64_t slot) { return cnt32[2 * slot]; };
    const int64_t c = (int64_t)blockIdx.x * groups + g;
    if (c < chunks) {
        const int32_t seg = seg_of(2 * c + 1);
        int64_t n = count_of(2 * c + 1);
        const bool open = n > 0;
        int32_t ids[kAhead], cnt[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t k = min(c + 1 + u, chunks - 1);
            ids[u] = seg_of(2 * k);
            cnt[u] = c + 1 + u < chunks ? count_of(2 * k) : 0;
        }
        // the first vectors load beside the ids: a slot that holds no partial loads what is there
        float v[V], x[V];
        uint32_t vi[NX], xi[NX];
        const bool lane = j0 < nvec;
        load(2 * c + 1, j0, lane, v, vi);
        load(2 * min(c + 1, chunks - 1), j0, lane, x, xi);
        bool on[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) on[u] = cnt[u] > 0 && ids[u] == seg && (u == 0 || on[u - 1]);
        if (open && on[kAhead - 1]) {
            if (j0 == 0) s_long[atomicAdd(&s_nlong, 1)] = g;
        } else if (open) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) n += on[u] ? cnt[u] : 0;
            for (int j = j0; j < nvec; j += tpr) {
                if (j != j0) {
                    load(2 * c + 1, j, true, v, vi);
                    load(2 * min(c + 1, chunks - 1), j, true, x, xi);
                }
                if (on[0]) take(v, vi, x, xi);
#pragma unroll
                for (int u = 1; u < kAhead; ++u) {
                    load(2 * min(c + 1 + u, chunks - 1), j, on[u], x, xi);
                    take(v, vi, x, xi);
                }
                store(seg, j, v, vi, n);
            }
        }
    }
    __syncthreads();
    // this thread's share of the run that starts at block `cl`: the lo partials of blocks k0, k0 + by,
    // ... (kU at a time, at most `trips` times); returns whether the run may go on behind them. A turn's sums
    // are added up by themselves first: no chain of them is longer than a turn's or the turns (maxima join
    // the total directly: 386,951 rows of 8 columns, Zipf lengths, 14.8 us by turns, 14.4 so)
    auto walk = [&](auto ut, int32_t seg, int64_t k0, int64_t by, int trips, int j, bool lane, float *v, uint32_t *vi, int64_t &n) {
        constexpr int kU = decltype(ut)::value;
        bool more = true;
        for (int t = 0; more && t < trips && k0 < chunks; ++t, k0 += kU * by) {
            float x[kU][V];
            uint32_t xi[kU][NX];
            int32_t id[kU], cnt[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t k = k0 + u * by, kk = min(k, chunks - 1);
                id[u] = seg_of(2 * kk);
                cnt[u] = k < chunks ? count_of(2 * kk) : 0;
                load(2 * kk, j, lane, x[u], xi[u]);
            }
            const bool any = cnt[0] > 0 && id[0] == seg;
#pragma unroll
            for (int u = 0; u < kU; ++u) {   // the run is contiguous: past its end nothing matches
                more = more && cnt[u] > 0 && id[u] == seg;
                if (more) {
                    if constexpr (RED != RED_SUM) take(v, vi, x[u], xi[u]);
                    else if (u > 0) take(x[0], xi[0], x[u], xi[u]);
                    n += cnt[u];
                }
            }
            if (RED == RED_SUM && any) take(v, vi, x[0], xi[0]);
        }
        return more && k0 < chunks;
    };
    const int nlong = s_nlong, in_wave = 64 / tpr, gw = g % in_wave, nwaves = kJoinBlock / 64;
    for (int i = (int)threadIdx.x >> 6; i < nlong; i += nwaves) {
        const int64_t cl = (int64_t)blockIdx.x * groups + s_long[i];
        const int32_t seg = seg_of(2 * cl + 1);
        for (int jt = 0; jt < nvec; jt += tpr) {
            const int j = jt + j0;
            float v[V];
            uint32_t vi[NX];
            load(2 * cl + 1, j, j < nvec && gw == 0, v, vi);
            int64_t n = gw == 0 ? count_of(2 * cl + 1) : 0;
            const bool more = walk(std::integral_constant<int, 4>{}, seg, cl + 1 + gw, in_wave, kTrips, j, j < nvec, v, vi, n);
            if (__any(more)) {
                if ((threadIdx.x & 63) == 0) s_longer[atomicAdd(&s_nlonger, 1)] = s_long[i];
                break;   // with all its columns
            }
            for (int d = tpr; d < 64; d <<= 1) {   // the groups' results, pairwise
                float x[V];
                uint32_t xi[NX];
#pragma unroll
                for (int k = 0; k < V; ++k) x[k] = __shfl_xor(v[k], d, 64);
                if constexpr (ARG) {
#pragma unroll
                    for (int k = 0; k < NX; ++k) xi[k] = (uint32_t)__shfl_xor((int)vi[k], d, 64);
                }
                take(v, vi, x, xi);
                n += __shfl_xor((long long)n, d, 64);
            }
            if (gw == 0 && j < nvec) store(seg, j, v, vi, n);
        }
    }
    __syncthreads();
    const int nlonger = s_nlonger;
    for (int i = 0; i < nlonger; ++i) {
        const int64_t cl = (int64_t)blockIdx.x * groups + s_longer[i];
        const int32_t seg = seg_of(2 * cl + 1);
        for (int jt = 0; jt < nvec; jt += tpr) {
            const int j = jt + j0;
            const bool lane = j < nvec;
            float v[V];
            uint32_t vi[NX];
            load(2 * cl + 1, j, lane && g == 0, v, vi);
            int64_t n = g == 0 ? count_of(2 * cl + 1) : 0;
            (void)walk(std::integral_constant<int, kDeep>{}, seg, cl + 1 + g, groups, INT32_MAX, j, lane, v, vi, n);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                s_v[threadIdx.x * V + k] = v[k];
                if constexpr (ARG) s_x[threadIdx.x * V + k] = vi[k];
            }
            s_n[threadIdx.x] = n;
            __syncthreads();
            for (int h = groups >> 1; h > 0; h >>= 1) {   // the groups' results, pairwise
                if (g < h) {
                    const int o = (int)threadIdx.x + h * tpr;
                    float x[V];
                    uint32_t xi[NX];
#pragma unroll
                    for (int k = 0; k < V; ++k) x[k] = s_v[o * V + k];
                    if constexpr (ARG) {
#pragma unroll
                        for (int k = 0; k < V; ++k) xi[k] = s_x[o * V + k];
                    }
                    take(v, vi, x, xi);
                    n += s_n[o];
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        s_v[threadIdx.x * V + k] = v[k];
                        if constexpr (ARG) s_x[threadIdx.x * V + k] = vi[k];
                    }
                    s_n[threadIdx.x] = n;
                }
                __syncthreads();
            }
            if (g == 0 && lane) store(seg, j, v, vi, n);
        }
    }
}

}  // namespace

hipError_t launch_ep_join(const EpArgs &a, int red, int64_t chunks, int gap_blocks, int64_t gap_tw,
                          hipStream_t stream) {
    // 4-float vectors at any 4-byte aligned address; other widths (and pointers) one float at a time
    const int V = a.F >= 4 && (((uintptr_t)a.out | (uintptr_t)a.arg_out) & 3) == 0 ? 4 : 1;
    const int64_t nvec = (a.F + V - 1) / V;
    int tpr = 1;
    while (tpr < nvec && tpr < 64) tpr <<= 1;
    const int64_t groups = kJoinBlock / tpr, nblk = (chunks + groups - 1) / groups;
    if (nblk + gap_blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    auto go = [&](auto rt, auto vt) -> hipError_t {
        hipLaunchKernelGGL((ep_join_kernel<decltype(rt)::value, decltype(vt)::value>), dim3((unsigned)(nblk + gap_blocks)),
                           dim3(kJoinBlock), 0, stream, a, chunks, nblk, gap_tw);
        return hipGetLastError();
    };
    auto by_red = [&](auto vt) -> hipError_t {
        if (red == RED_SUM) return go(std::integral_constant<int, RED_SUM>{}, vt);
        if (red == RED_MAX) return go(std::integral_constant<int, RED_MAX>{}, vt);
        if (red == RED_MAXARG) return go(std::integral_constant<int, RED_MAXARG>{}, vt);
        return hipErrorInvalidValue;
    };
    return V == 4 ? by_red(std::integral_constant<int, 4>{}) : by_red(std::integral_constant<int, 1>{});
}

}  // namespace geot
