// Plan of the segment linearisation, formed once per solve (the observation structure is
// fixed for the solve): the points of each window, in the linearisation order, are cut into
// chunks of whole points (at most 64 observations, one per lane, and 32 points) and runs of
// chunks into segments whose points are seen by at most kSegCams optimisable keyframes
// between them.  One wavefront of the linearisation takes one segment, so a segment's share
// of the reduced system is a dense block over its few cameras that stays in registers.
//
//   k_order_keys (k_order) leaves the set of optimisable keyframes of each point;
//   k_seg_count  one wavefront per range of positions: the range's counts and sets are
//                staged in LDS, then cut greedily, 64 positions examined at a time (prefix
//                sums of the counts, prefix unions of the sets); counts of segments, chunks
//                and record doubles;
//   k_seg_scan   one block: exclusive prefix sums over the ranges (so that the plan does not
//                depend on scheduling), capacities checked;
//   k_seg_emit   the same cut again, writing the segments and chunks;
//   k_seg_gather one wavefront per chunk: its observations copied into the order, with a
//                word each: keyframe, type, octave, the camera's place in the segment's set,
//                the point's place in the chunk.
//
// A point seen by more keyframes than a segment holds, a repeated (point, keyframe) pair or
// a plan that exceeds its capacity sets a flag, and the solve takes the general
// linearisation (k_linearize) instead.
#include "lba_internal.h"

#include <algorithm>

namespace lba {

struct SegStage {
    unsigned long long set[kSegRange];   // keyframes of the range's points
    uint8_t cnt[kSegRange];              // and their observations
};

// the chunk that starts at position p: its points' counts and sets by lane
struct SegCand {
    int incl;                  // observations up to and including the lane's position
    unsigned long long uni;    // keyframes of the positions up to and including it
    bool valid;
};

__device__ __forceinline__ SegCand seg_candidates(const SegStage &st, int i, int n, int lane) {
    SegCand c;
    c.valid = i + lane < n;
    c.incl = c.valid ? st.cnt[i + lane] : 0;
    c.uni = c.valid ? st.set[i + lane] : 0ull;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(c.incl, o, 64);
        const unsigned long long u = __shfl_up(c.uni, o, 64);
        if (lane >= o) {
            c.incl += y;
            c.uni |= u;
        }
    }
    return c;
}

// points of a chunk that continues a segment over the keyframes `set`
__device__ __forceinline__ int seg_fit(const SegCand &c, unsigned long long set, int max_cams, int lane) {
    const bool ok = c.valid && lane < kSegPoints && c.incl <= 64 && __popcll(set | c.uni) <= max_cams;
    return __popcll(__ballot(ok));
}

// One range, by one wavefront.  kEmit: write the plan from the range's bases on.
template <bool kEmit>
__device__ void seg_range(const SegPlanArgs &a, int r, int lane, SegStage &st) {
    const Tile rg = a.ranges[r];
    const int n = rg.p1 - rg.p0;
    int nseg = 0, nchunk = 0, flag = 0;
    int64_t rec = 0, seg0 = 0, ch0 = 0, rec0 = 0;
    if (kEmit) {
        seg0 = a.base[3 * (int64_t)r];
        ch0 = a.base[3 * (int64_t)r + 1];
        rec0 = a.base[3 * (int64_t)r + 2];
    }
    int place = n > 0 ? a.pinfo[rg.p0].w : 0;   // places follow the positions without gaps
    for (int i = lane; i < n; i += 64) {
        const int4 pi = a.pinfo[rg.p0 + i];
        st.set[i] = a.kfmask[pi.x];
        st.cnt[i] = (uint8_t)pi.z;
    }
    wave_sync();
    unsigned long long set = 0;
    int open = 0;   // chunks of the open segment
    int4 first = make_int4(0, 0, 0, 0);
    auto close = [&]() {
        if (open == 0) return;
        const int u = __popcll(set);
        if (kEmit && lane == 0) {
            Seg s;
            s.win = rg.win;
            s.chunk0 = (int32_t)(ch0 + nchunk - open);
            s.nchunk = open;
            s.ncam = u;
            s.mask = set;
            s.rec = rec0 + rec;
            s.kf0 = a.win[rg.win].kf0;
            s.K = a.win[rg.win].K;
            s.first = first;
            a.segs[seg0 + nseg] = s;
        }
        ++nseg;
        rec += seg_record(u);
        set = 0;
        open = 0;
    };
    for (int i = 0; i < n;) {
        const SegCand c = seg_candidates(st, i, n, lane);
        const int fresh = seg_fit(c, 0, a.max_cams, lane);
        int np = open > 0 ? seg_fit(c, set, a.max_cams, lane) : fresh;
        // a segment ends when it is full or its keyframes would cut the chunk to less than half
        if (open > 0 && (open >= a.max_chunks || 2 * np < fresh || np == 0)) {
            close();
            np = fresh;
        }
        if (np == 0) {   // (a point beyond the limits: the general path is taken)
            flag = 1;
            np = 1;
        }
        const int nobs = __shfl(c.incl, np - 1, 64);
        set |= __shfl(c.uni, np - 1, 64);
        if (open == 0) first = make_int4(rg.p0 + i, np, place, nobs);
        if (kEmit && lane == 0) {
            a.chunks[ch0 + nchunk] = make_int4(rg.p0 + i, np, place, nobs);
            a.chunk_seg[ch0 + nchunk] = (int32_t)(seg0 + nseg);
        }
        ++open;
        ++nchunk;
        i += np;
        place += nobs;
    }
    close();
    if (!kEmit && lane == 0) {
        a.base[3 * (int64_t)r] = nseg;
        a.base[3 * (int64_t)r + 1] = nchunk;
        a.base[3 * (int64_t)r + 2] = rec;
        if (flag) a.info[kSegInfoGeneral] = kSegOver;
    }
}

__global__ __launch_bounds__(256) void k_seg_count(SegPlanArgs a) {
    __shared__ SegStage st[4];
    if (a.info[0] || a.info[kSegInfoGeneral]) return;
    const int w = threadIdx.x >> 6, r = blockIdx.x * 4 + w;
    if (r < a.n_ranges) seg_range<false>(a, r, threadIdx.x & 63, st[w]);
}

__global__ __launch_bounds__(256) void k_seg_emit(SegPlanArgs a) {
    __shared__ SegStage st[4];
    if (a.info[0] || a.info[kSegInfoGeneral]) return;
    const int w = threadIdx.x >> 6, r = blockIdx.x * 4 + w;
    if (r < a.n_ranges) seg_range<true>(a, r, threadIdx.x & 63, st[w]);
}

__global__ __launch_bounds__(256) void k_seg_gather(SegPlanArgs a) {
    if (a.info[0] || a.info[kSegInfoGeneral]) return;
    const int lane = threadIdx.x & 63, nchunk = a.info[kSegInfoChunks];
    for (int ch = blockIdx.x * 4 + (threadIdx.x >> 6); ch < nchunk; ch += gridDim.x * 4) {
        const int4 ck = a.chunks[ch];
        const Seg S = a.segs[a.chunk_seg[ch]];
        const WinInfo W = a.win[S.win];
        int4 pi = make_int4(0, 0, 0, 0);
        if (lane < ck.y) pi = a.pinfo[ck.x + lane];
        int incl = pi.z;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        int j = 0;   // the first lane whose inclusive count exceeds this lane (six steps)
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
            if (__shfl(incl, j + step - 1, 64) <= lane) j += step;
        j = min(j, 63);
        const int o = __shfl(pi.y, j, 64) + lane - (__shfl(incl, j, 64) - __shfl(pi.z, j, 64));
        const bool has = lane < ck.w;
        const int kf = has ? a.obs.kf[o] : 0;
        const int k = has ? a.opt_map[W.kf0 + kf] : -1;
        const unsigned lc = k >= 0 ? (unsigned)__popcll(S.mask & ((1ull << k) - 1ull)) : (unsigned)kSegNoCam;
        unsigned cams = k >= 0 ? 1u << lc : 0u;   // the chunk's cameras, above its observation count
#pragma unroll
        for (int x = 32; x > 0; x >>= 1) cams |= __shfl_xor(cams, x, 64);
        if (lane == 0) {
            a.chunks[ch].w = ck.w | (int)(cams << 8);
            if (S.chunk0 == ch) a.segs[a.chunk_seg[ch]].first.w = ck.w | (int)(cams << 8);
        }
        if (!has) continue;
        const int64_t dst = ck.z + lane;
        a.words[dst] = (uint32_t)kf | ((uint32_t)a.obs.type[o] << 7) | ((uint32_t)a.obs.oct[o] << 8) | (lc << 13) |
                       ((uint32_t)j << 17);
        if (a.obs.z_f32) {
            const float *z = static_cast<const float *>(a.obs.z);
            float *sz = static_cast<float *>(a.sz);
#pragma unroll
            for (int c = 0; c < 3; ++c) sz[(int64_t)c * a.obs.n_obs + dst] = z[(int64_t)c * a.obs.n_obs + o];
        } else {
            const double *z = static_cast<const double *>(a.obs.z);
            double *sz = static_cast<double *>(a.sz);
#pragma unroll
            for (int c = 0; c < 3; ++c) sz[(int64_t)c * a.obs.n_obs + dst] = z[(int64_t)c * a.obs.n_obs + o];
        }
    }
}

constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void k_seg_scan(SegPlanArgs a) {
    __shared__ long long part[kScanThreads / 64][3];
    if (a.info[0] || a.info[kSegInfoGeneral]) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (a.n_ranges + kScanThreads - 1) / kScanThreads;
    const int r0 = min(a.n_ranges, tid * per), r1 = min(a.n_ranges, r0 + per);
    long long s[3] = {0, 0, 0};
    for (int r = r0; r < r1; ++r)
        for (int q = 0; q < 3; ++q) s[q] += a.base[3 * (int64_t)r + q];
    long long x[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        x[q] = s[q];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(x[q], o, 64);
            if (lane >= o) x[q] += y;
        }
        if (lane == 63) part[wave][q] = x[q];
    }
    __syncthreads();
    long long tot[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        x[q] -= s[q];
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wave) x[q] += part[w][q];
            tot[q] += part[w][q];
        }
    }
    for (int r = r0; r < r1; ++r)
        for (int q = 0; q < 3; ++q) {
            const long long v = a.base[3 * (int64_t)r + q];
            a.base[3 * (int64_t)r + q] = x[q];
            x[q] += v;
        }
    if (tid == 0) {
        a.base[3 * (int64_t)a.n_ranges] = tot[0];   // end of the last range's segments
        a.info[kSegInfoCount] = (int32_t)min(tot[0], (long long)INT32_MAX);
        a.info[kSegInfoChunks] = (int32_t)min(tot[1], (long long)INT32_MAX);
        if (tot[0] > a.seg_cap || tot[1] > a.chunk_cap || tot[2] > a.rec_cap) a.info[kSegInfoGeneral] = kSegOver;
    }
}

hipError_t launch_seg_plan(const SegPlanArgs &a, hipStream_t s) {
    if (a.n_ranges <= 0) return hipSuccess;
    const int br = (a.n_ranges + 3) / 4;
    hipLaunchKernelGGL(k_seg_count, dim3(br), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_seg_scan, dim3(1), dim3(kScanThreads), 0, s, a);
    hipLaunchKernelGGL(k_seg_emit, dim3(br), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_seg_gather, dim3((unsigned)std::min<int64_t>((a.chunk_cap + 3) / 4, 8192)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// the outlier flags of round 2 into the words
__global__ __launch_bounds__(256) void k_seg_mask(SegPlanArgs a) {
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
        const int first = __shfl(pi.w, 0, 64);
        for (int d0 = 0; d0 < total; d0 += 64) {   // uniform trip count: every lane shuffles
            const int d = d0 + lane;
            int j = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(incl, j + step - 1, 64) <= d) j += step;
            const int excl = __shfl(incl, j & 63, 64) - __shfl(pi.z, j & 63, 64);
            const int o = __shfl(pi.y, j & 63, 64) + (d - excl);
            if (d < total) {
                const uint32_t w = a.words[first + d] & ~kSegInactive;
                a.words[first + d] = w | (a.mask[o] ? kSegInactive : 0u);
            }
        }
    }
}

hipError_t launch_seg_mask(const SegPlanArgs &a, hipStream_t s) {
    if (a.n_pt <= 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>(4096, (a.n_pt + 255) / 256);   // 64 positions per wavefront
    hipLaunchKernelGGL(k_seg_mask, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace lba
