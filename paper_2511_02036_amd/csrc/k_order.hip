// Point order for the linearisation.  Within each window the points are sorted by the
// lowest, then the highest, optimisable keyframe that observes them; points that no
// optimisable keyframe observes go last, and ties keep their index order.  The order
// only changes which points the linearisation kernel groups into one chunk: consecutive
// points of this order share most of their keyframes, so a chunk touches few camera
// blocks of the reduced system and each touched block gathers many pairs.  The sums it
// forms are the same (the Schur complement does not depend on the order of the points).
//
// Windows with few optimisable keyframes, whose chunks touch few camera blocks in any order,
// keep the index order (k_order_identity writes it): up to ten where segments follow, since
// any point suits a segment there, up to 20 (kSortMinKopt) in the general form, where the sort
// does not pay below (18 keyframes, 80,000 observations: a solve in index order 1,980 us, sorted
// 2,820).  A problem that turns out not to suit the segments takes the general form's order:
// k_order_keys finds the unsuitable points before anything is sorted, and where the plan finds
// itself over its capacities the index order is written again.  The others use two kernels, run
// once per solve after the input checks:
//   k_order_keys  grid (x, window), one thread per point: key = lowest | highest << 6 (Kopt
//                 for both when no optimisable keyframe observes the point) | observations
//                 << 12, and the set of its optimisable keyframes;
//   k_order       one 1024-thread block per window and lowest keyframe: every block reads the
//                 window's keys once, counts the points and observations of the lower
//                 keyframes (its base), lists its own points in index order and writes them
//                 by highest keyframe, one block scan per highest keyframe that occurs.  Per
//                 position: the point, its first observation, its observation count and the
//                 place of the first observation in the observation order that follows the
//                 points' order.
//   k_order_window  the same order by one 1024-thread block per window.
// A block per lowest keyframe reads a window's keys once each, which pays while the card has
// room for the blocks.  Whole calls without a step, us, a block per lowest keyframe and per
// window: 30 optimisable keyframes, 20,000 points: one window 273 and 348, 8 windows 358 and 435,
// 32 windows 751 and 693, 128 windows 2,458 and 1,832; 22 keyframes, 8,000 points: 209 and 208,
// 270 and 273, 409 and 359, 1,022 and 778; 3,000 points: 182 and 166, 191 and 180, 304 and 254;
// the sort alone, 42 keyframes, 4,000 points: one window 49 and 65, 96 windows 202 and 105.
// The result is deterministic, and the same either way.  k_order_gather (general linearisation)
// or k_seg_gather then copies the observations into that order (once per solve), and the outlier
// flags go there once per round, so that the linearisation reads each chunk's observations as
// one contiguous range.
#include "lba_internal.h"

#include <algorithm>

namespace lba {

constexpr int kOrdThreads = 1024;
constexpr int kOrdWaves = kOrdThreads / kWave;
constexpr int kBuckets = 64;             // digit range: optimisable keyframe index, Kopt = none
constexpr int kOrdLdsPoints = 49152;     // windows up to this many points sort from LDS digits
// a block per lowest keyframe for so many windows at most, if points x optimisable keyframes of
// the largest come to so much
constexpr int kOrdSplitWindows = 8;
constexpr int64_t kOrdSplitWork = 160000;
constexpr int kSortMinKopt = 20;         // the general form sorts windows with more optimisable keyframes

__device__ __forceinline__ bool sorted_window(const OrderArgs &a, const WinInfo &W) {
    const bool segments = a.max_cams > 0 && !a.err[kSegInfoGeneral];
    return a.by_keyframes && W.Kopt > (segments ? a.max_cams : kSortMinKopt);
}
static_assert(kMaxKoptFP64 < kBuckets && kMaxKoptMixed < kBuckets, "keyframe digit range");

__global__ __launch_bounds__(256) void k_order_identity(OrderArgs a) {
    if (*a.err) return;
    const WinInfo W = a.win[blockIdx.y];
    if (sorted_window(a, W)) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < W.M; i += gridDim.x * blockDim.x) {
        const int P = W.pt0 + i;
        const int s = a.pt_start[P];
        a.pinfo[P] = make_int4(P, s, a.pt_start[P + 1] - s, s);
    }
}

__global__ __launch_bounds__(256) void k_order_keys(OrderArgs a) {
    if (*a.err) return;
    const WinInfo W = a.win[blockIdx.y];
    if (a.max_cams == 0 && !sorted_window(a, W)) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < W.M; i += gridDim.x * blockDim.x) {
        const int P = W.pt0 + i;
        const int o0 = a.pt_start[P], o1 = a.pt_start[P + 1];
        unsigned long long set = 0;
        bool dup = false;
        for (int o = o0; o < o1; o += 4) {   // four observations per step: independent loads
            int kf[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) kf[u] = o + u < o1 ? a.obs_kf[o + u] : -1;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = kf[u] >= 0 ? a.opt_map[W.kf0 + kf[u]] : -1;
                if (k < 0) continue;
                dup = dup || ((set >> k) & 1ull);
                set |= 1ull << k;
            }
        }
        const unsigned lo = set ? __builtin_ctzll(set) : W.Kopt, hi = set ? 63 - __builtin_clzll(set) : W.Kopt;
        a.keys[P] = lo | (hi << 6) | ((unsigned)(o1 - o0) << 12);
        if (a.max_cams == 0) continue;
        a.kfmask[P] = set;
        if (dup || __popcll(set) > a.max_cams) a.err[kSegInfoGeneral] = kSegUnsuited;
    }
}

// inclusive scan of one 64-bit value per thread over the block (1024 threads), and the total
__device__ __forceinline__ unsigned long long order_scan(unsigned long long v, unsigned long long *part, int tid,
                                                         unsigned long long &total) {
    const int lane = tid & 63, wave = tid >> 6;
    unsigned long long x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    __syncthreads();   // (the previous scan's parts have been read)
    if (lane == 63) part[wave] = x;
    __syncthreads();
    total = 0;
    unsigned long long add = 0;
#pragma unroll
    for (int w = 0; w < kOrdWaves; ++w) {
        const unsigned long long u = part[w];
        add += w < wave ? u : 0ull;
        total += u;
    }
    return x + add;
}

__global__ __launch_bounds__(kOrdThreads) void k_order(OrderArgs a) {
    __shared__ unsigned long long part[kOrdWaves];
    __shared__ int hist[kBuckets];
    if (*a.err) return;
    const WinInfo W = a.win[blockIdx.y];
    const unsigned lo = blockIdx.x;
    if (!sorted_window(a, W) || (int)lo > W.Kopt) return;
    const int tid = threadIdx.x;
    const uint32_t *key = a.keys + W.pt0;
    if (tid < kBuckets) hist[tid] = 0;
    // points and observations (high word) of the lower keyframes, and this thread's own points
    const int per = (W.M + kOrdThreads - 1) / kOrdThreads;
    const int i0 = min(W.M, tid * per), i1 = min(W.M, i0 + per);
    unsigned long long less = 0;
    int own = 0;
    for (int i = i0; i < i1; ++i) {
        const uint32_t k = key[i];
        if ((k & 63u) < lo) less += 1ull | ((unsigned long long)(k >> 12) << 32);
        own += (k & 63u) == lo;
    }
    unsigned long long before, n;
    order_scan(less, part, tid, before);
    int at = (int)order_scan((unsigned long long)own, part, tid, n) - own;
    const int p0 = (int)(before & 0xffffffffull), count = (int)n;
    if (count == 0) return;
    int32_t *list = a.tmp + W.pt0 + p0;
    for (int i = i0; i < i1; ++i) {
        const uint32_t k = key[i];
        if ((k & 63u) != lo) continue;
        list[at++] = i;
        atomicAdd(&hist[(k >> 6) & 63u], 1);
    }
    __threadfence_block();
    __syncthreads();
    // by highest keyframe, in index order within each
    const int perl = (count + kOrdThreads - 1) / kOrdThreads;
    const int l0 = min(count, tid * perl), l1 = min(count, l0 + perl);
    int pos = W.pt0 + p0;
    int place = W.ob0 + (int)(before >> 32);
    for (unsigned h = lo; (int)h <= W.Kopt; ++h) {
        if (hist[h] == 0) continue;   // (uniform)
        unsigned long long mine = 0;
        for (int l = l0; l < l1; ++l) {
            const uint32_t k = key[list[l]];
            if (((k >> 6) & 63u) == h) mine += 1ull | ((unsigned long long)(k >> 12) << 32);
        }
        unsigned long long tot;
        const unsigned long long ex = order_scan(mine, part, tid, tot) - mine;
        int q = pos + (int)(ex & 0xffffffffull), pl = place + (int)(ex >> 32);
        if (mine)
            for (int l = l0; l < l1; ++l) {
                const int e = list[l];
                const uint32_t k = key[e];
                if (((k >> 6) & 63u) != h) continue;
                const int m = (int)(k >> 12);
                a.pinfo[q++] = make_int4(W.pt0 + e, a.pt_start[W.pt0 + e], m, pl);
                pl += m;
            }
        pos += (int)(tot & 0xffffffffull);
        place += (int)(tot >> 32);
    }
}

// The same order by one block per window, for batches: two stable counting-sort passes over Kopt + 1
// buckets (by the highest keyframe, then by the lowest), each ranking a round of 1024 points with
// one ballot per bucket per wavefront, from digits staged in LDS where they fit.  The second pass
// writes each position's record without its place; a last scan adds that.
//
// One pass: element i of the input order is src[i] (window-local; the identity without src), its
// bucket the 6-bit digit of its key at bit sh.  It goes to place pos of the output: dst[pos], or in
// the last pass pinfo[pos].
template <bool kLast, typename Key>
__device__ void order_pass(const OrderArgs &a, const WinInfo &W, const Key *key, const int32_t *src, int32_t *dst, int sh,
                           int *base, int *wcnt) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, M = W.M;
    const int nb = W.Kopt + 1;
    if (tid < kBuckets) base[tid] = 0;
    __syncthreads();
    for (int i = tid; i < M; i += kOrdThreads) atomicAdd(&base[(key[src ? src[i] : i] >> sh) & (kBuckets - 1)], 1);
    __syncthreads();
    if (tid == 0) {
        int s = 0;
        for (int b = 0; b < nb; ++b) {
            const int c = base[b];
            base[b] = s;
            s += c;
        }
    }
    __syncthreads();
    for (int r = 0; r < M; r += kOrdThreads) {
        const int i = r + tid;
        const bool valid = i < M;
        const int e = valid ? (src ? src[i] : i) : -1;
        const int d = valid ? (int)(key[e] >> sh) & (kBuckets - 1) : -1;
        int ps = 0, pe = 0;
        if (kLast && valid) {   // in flight during the ranking
            ps = a.pt_start[W.pt0 + e];
            pe = a.pt_start[W.pt0 + e + 1];
        }
        int rank = 0, mine = 0;
        for (int b = 0; b < nb; ++b) {
            const unsigned long long bal = __ballot(d == b);
            if (d == b) rank = __popcll(bal & ((1ull << lane) - 1ull));
            if (lane == b) mine = __popcll(bal);
        }
        wcnt[wave * kBuckets + lane] = mine;
        __syncthreads();
        if (valid) {
            int pos = base[d] + rank;
            for (int w = 0; w < wave; ++w) pos += wcnt[w * kBuckets + d];
            if (kLast) a.pinfo[W.pt0 + pos] = make_int4(W.pt0 + e, ps, pe - ps, 0);
            else dst[pos] = e;
        }
        __syncthreads();
        if (tid < kBuckets) {
            int s = 0;
            for (int w = 0; w < kOrdWaves; ++w) s += wcnt[w * kBuckets + tid];
            base[tid] += s;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kOrdThreads) void k_order_window(OrderArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int base[kBuckets];
    __shared__ int wcnt[kOrdWaves * kBuckets];
    if (*a.err) return;
    const WinInfo W = a.win[blockIdx.x];
    if (!sorted_window(a, W)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t *key = a.keys + W.pt0;
    int32_t *tmp = a.tmp + W.pt0;
    if (W.M <= kOrdLdsPoints) {
        uint16_t *lk = reinterpret_cast<uint16_t *>(smem);
        for (int i = tid; i < W.M; i += kOrdThreads) lk[i] = (uint16_t)(key[i] & 0xfffu);
        __syncthreads();
        order_pass<false>(a, W, lk, nullptr, tmp, 6, base, wcnt);   // by the highest keyframe
        __syncthreads();
        order_pass<true>(a, W, lk, tmp, nullptr, 0, base, wcnt);    // then, stably, by the lowest
    } else {
        order_pass<false>(a, W, key, nullptr, tmp, 6, base, wcnt);
        __syncthreads();
        order_pass<true>(a, W, key, tmp, nullptr, 0, base, wcnt);
    }
    __syncthreads();
    // places: the window's first observation plus the exclusive prefix of the counts in this order
    int carry = W.ob0;
    for (int r = 0; r < W.M; r += kOrdThreads) {
        const int i = r + tid;
        const int m = i < W.M ? a.pinfo[W.pt0 + i].z : 0;
        int x = m;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wcnt[wave] = x;
        __syncthreads();
        int add = carry, tot = 0;
        for (int w = 0; w < kOrdWaves; ++w) {
            const int v = wcnt[w];
            add += w < wave ? v : 0;
            tot += v;
        }
        if (i < W.M) a.pinfo[W.pt0 + i].w = add + x - m;
        carry += tot;
        __syncthreads();
    }
}

// Each wavefront takes 64 consecutive positions of the order; their places form one
// contiguous range (a point's observations follow the previous position's, across
// windows too).  The lanes walk that range 64 places at a time (coalesced writes); each
// finds the point of its place by binary lifting over the lanes' inclusive counts.
template <bool kMask>
__global__ __launch_bounds__(256) void k_order_gather(OrderArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t nwv = (int64_t)gridDim.x * (blockDim.x / 64);
    for (int64_t b = ((int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6)) * 64; b < a.n_pt; b += nwv * 64) {
        const int64_t pos = b + lane;
        int4 pi = make_int4(0, 0, 0, 0);
        if (pos < a.n_pt) pi = a.pinfo[pos];
        int incl = pi.z;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        const int total = __shfl(incl, 63, 64);
        const int first = __shfl(pi.w, 0, 64);   // place of the range's first observation
        for (int d0 = 0; d0 < total; d0 += 64) {   // uniform trip count: every lane shuffles
            const int d = d0 + lane;
            int j = 0;   // the first lane whose inclusive count exceeds d (fixed six steps)
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(incl, j + step - 1, 64) <= d) j += step;
            const int excl = __shfl(incl, j, 64) - __shfl(pi.z, j, 64);
            const int o = __shfl(pi.y, j, 64) + (d - excl), dst = first + d;
            if (d >= total) continue;
            if (kMask) {
                a.smask[dst] = a.mask[o];
            } else {
                a.sobs_kf[dst] = a.obs.kf[o];
                a.sobs_type[dst] = a.obs.type[o];
                a.sobs_oct[dst] = a.obs.oct[o];
                if (a.obs.z_f32) {
                    const float *z = static_cast<const float *>(a.obs.z);
                    float *sz = static_cast<float *>(a.sobs_z);
#pragma unroll
                    for (int c = 0; c < 3; ++c) sz[(int64_t)c * a.obs.n_obs + dst] = z[(int64_t)c * a.obs.n_obs + o];
                } else {
                    const double *z = static_cast<const double *>(a.obs.z);
                    double *sz = static_cast<double *>(a.sobs_z);
#pragma unroll
                    for (int c = 0; c < 3; ++c) sz[(int64_t)c * a.obs.n_obs + dst] = z[(int64_t)c * a.obs.n_obs + o];
                }
            }
        }
    }
}

hipError_t launch_order_gather(const OrderArgs &a, bool mask, hipStream_t s) {
    if (a.n_pt <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>(4096, (a.n_pt + 255) / 256);   // 64 positions per wavefront
    if (mask) hipLaunchKernelGGL(k_order_gather<true>, dim3(blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_order_gather<false>, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_order(const OrderArgs &a, int n_windows, int max_points, int max_kopt, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    const int bx = std::max(1, std::min(64, (max_points + 255) / 256));
    const bool sort = a.by_keyframes && max_kopt > (a.max_cams > 0 ? a.max_cams : kSortMinKopt);
    if (sort || a.max_cams > 0) hipLaunchKernelGGL(k_order_keys, dim3(bx, n_windows), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_order_identity, dim3(bx, n_windows), dim3(256), 0, s, a);
    if (sort && n_windows <= kOrdSplitWindows && (int64_t)max_points * max_kopt >= kOrdSplitWork) {
        hipLaunchKernelGGL(k_order, dim3(max_kopt + 1, n_windows), dim3(kOrdThreads), 0, s, a);
    } else if (sort) {
        const size_t lds = sizeof(uint16_t) * (size_t)std::min(max_points, kOrdLdsPoints);
        hipLaunchKernelGGL(k_order_window, dim3(n_windows), dim3(kOrdThreads), lds, s, a);
    }
    return hipGetLastError();
}

// the general form's order after segments were planned in vain: index order again in the windows
// that only the segments have sorted
hipError_t launch_order_general(OrderArgs a, int n_windows, int max_points, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    a.max_cams = 0;
    const int bx = std::max(1, std::min(64, (max_points + 255) / 256));
    hipLaunchKernelGGL(k_order_identity, dim3(bx, n_windows), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace lba
