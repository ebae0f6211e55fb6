// Per-scale observation counters of keyframe culling (Sections III-D and IV-F).  The
// paper keeps, per map point, a small array of its observation counts per octave, so
// that the redundancy test of an observation -- are there at least min_obs other
// observations of the point at the same or a finer scale? -- is a sum over a few
// counters instead of a walk over the point's observation list.  Here the counters are
// built on the GPU from the window's observations (where the bundle adjustment leaves
// them, outlier flags included).
//
// Observations grouped by ascending point, as the bundle adjustment holds them, take one
// pass (k_cull_grouped): a block owns the points whose first observation lies in its run
// of observations, counts them in LDS, writes their counters once (zeros included) and
// tests its observations against the counts in LDS.  k_cull_order decides that first, from the
// point indices alone: any descent, index out of range, point with kGrpTail or more
// observations past a run's end (and more after it) or run over too many points raises the
// flag, and then three general passes run over zeroed counters (without the flag they return
// at once):
//   1. counters[j][o] += 1 for every active observation (integer atomics: exact, and
//      independent of the order);
//   2. per active observation (k, j, o): others = counters[j][0 .. o + slack] summed,
//      minus itself; redundant if others >= min_obs; per-keyframe totals of observations
//      and redundant observations, summed first in LDS when the block's keyframes span
//      a short range, else with global atomics;
//   3. per keyframe: culled if not protected, it has observations and
//      den * redundant >= num * observations.
// The flag is bit 0 of cull's first byte, which pass 3 writes afterwards: it belongs to the call.
// (Bit 1 keeps protect's first byte, so that protect and cull may be one array.)
#include "lmap_internal.h"

namespace lmap {

// zeroed totals, and the flag
__global__ __launch_bounds__(256) void k_cull_begin(CullArgs a, int general) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < a.n_kf) a.kf_obs[k] = a.kf_red[k] = 0;
    if (k == 0) a.cull[0] = general | (a.protect && a.protect[0] ? 2 : 0);
}

constexpr int kGrpThreads = 256, kGrpRun = 2048, kGrpTail = 256, kGrpCounts = 4096, kGrpTiles = 16, kGrpSpan = 512,
              kGrpCopies = 4, kGrpMinObs = 1 << 20;
constexpr int kGrpOrderBlocks = 4096;

// Whether the single pass can take the observations.  Reads the point indices only, run by
// run, and stops once any block has raised the flag.  Deciding this within the single pass wasted
// the pass where a descent came late: 18 million observations of 2.6 million points 576 us so,
// 390 now, 398 in general passes alone.  Bound by reading the indices: 14.7 us of 210 for those
// in order (5 TB/s; with every index before another loaded rather than taken from the lane below,
// 20.7 us).
__global__ __launch_bounds__(kGrpThreads) void k_cull_order(CullArgs a) {
    const int tid = threadIdx.x, n = a.n_obs;
    const int64_t most = (int64_t)kGrpTiles * (kGrpCounts / a.n_levels);   // points of a run
    for (int64_t r0 = (int64_t)blockIdx.x * kGrpRun; r0 < n; r0 += (int64_t)gridDim.x * kGrpRun) {
        const uint8_t raised = *(volatile uint8_t *)a.cull;
        const int last = n - 1;
        const int first = a.pt[max((int)r0 - 1, 0)], final = a.pt[min((int64_t)last, r0 + kGrpRun - 1)],
                  tail = a.pt[min((int64_t)last, r0 + kGrpRun + kGrpTail - 1)];
        int pt[kGrpRun / kGrpThreads], edge[kGrpRun / kGrpThreads];
        const int w0 = (tid & ~63) - 1;   // before the wavefront's first
#pragma unroll
        for (int u = 0; u < kGrpRun / kGrpThreads; ++u) {   // (past the end: the last one again)
            pt[u] = a.pt[(int)min((int64_t)last, r0 + tid + u * kGrpThreads)];
            edge[u] = a.pt[max(0, (int)min((int64_t)last, r0 + __builtin_amdgcn_readfirstlane(w0) + u * kGrpThreads))];
        }
        if (raised & 1) return;
        bool bad = false;
#pragma unroll
        for (int u = 0; u < kGrpRun / kGrpThreads; ++u) {
            int before = __shfl_up(pt[u], 1, 64);
            if ((tid & 63) == 0) before = edge[u];
            bad = bad || pt[u] < 0 || pt[u] >= a.n_pt || before > pt[u];
        }
        // the run's points, and its last point's tail
        const bool end = r0 + kGrpRun >= n;
        const int64_t p0 = r0 == 0 ? 0 : (int64_t)first + 1, p1 = end ? a.n_pt : (int64_t)final + 1;
        bad = bad || p1 - p0 > most || (r0 + kGrpRun + kGrpTail < n && tail == final);
        if (__any(bad) && (tid & 63) == 0) a.cull[0] = raised | 1;
    }
}

// Bound by the latency of a run's loads, LDS counts and sums, one after the other, with four
// blocks per compute unit: 18 million observations of 2.6 million points take 160 us (1.7 TB/s
// of its bytes), the zeroing and two passes before it 376.  More LDS for the counts, shorter
// runs, or registers for six blocks per unit cost 10 to 60% more; four copies of the totals,
// by lane, are 2% faster than one.  With the flag raised the launch zeroes the counters instead.
__global__ __launch_bounds__(kGrpThreads) void k_cull_grouped(CullArgs a) {
    __shared__ __align__(16) int cnt[kGrpCounts];
    __shared__ int h[kGrpCopies][kGrpSpan];   // observations | redundant << 16, by lane
    __shared__ int s_at[2], s_k[2];
    constexpr int kPer = (kGrpRun + kGrpTail) / kGrpThreads;
    const int tid = threadIdx.x, L = a.n_levels, n = a.n_obs;
    if (a.cull[0] & 1) {   // (uniform) the general passes start from zeros
        const int64_t nc = (int64_t)a.n_pt * L;
        for (int64_t i = blockIdx.x * (int64_t)kGrpThreads + tid; i < nc; i += (int64_t)gridDim.x * kGrpThreads) a.counters[i] = 0;
        return;
    }
    if (blockIdx.x * (int64_t)kGrpRun >= n) return;
    const int i0 = blockIdx.x * kGrpRun, i1 = min(n, i0 + kGrpRun);
    if (tid < 2) {
        s_at[tid] = tid == 0 ? (i0 == 0 ? 0 : n) : n;
        s_k[tid] = tid == 0 ? 0x7fffffff : -1;
    }
    for (int k = tid; k < kGrpCopies * kGrpSpan; k += kGrpThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    // the run and what follows it; the first observations of a point at or after i0 and i1
    // (the run of a point that starts there)
    int pt[kPer], kf[kPer], oc[kPer];
    int lo = n, hi = n;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = i0 + tid + u * kGrpThreads, ic = min(i, n - 1);
        pt[u] = a.pt[ic];
        kf[u] = a.kf[ic];
        oc[u] = a.oct[ic];
        if (a.active && !a.active[ic]) oc[u] = -1;
        const int before = a.pt[max(ic - 1, 0)];
        if (i > 0 && i < n && before != pt[u]) {
            if (i >= i1) hi = min(hi, i);
            lo = min(lo, i);
        }
    }
    if (lo < n) atomicMin(&s_at[0], lo);
    if (hi < n) atomicMin(&s_at[1], hi);
    __syncthreads();
    const int b0 = s_at[0], b1 = s_at[1];   // (none up to the end of the observations: n)
    const int p0 = b0 == 0 ? 0 : a.pt[b0 - 1] + 1, p1 = b1 == n ? a.n_pt : a.pt[b1 - 1] + 1;
    const int tile = kGrpCounts / L;
    int kmin = 0x7fffffff, kmax = -1;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = i0 + tid + u * kGrpThreads;
        if (i < b0 || i >= b1 || oc[u] >= L) oc[u] = -1;   // not this block's, or not counted
        if (oc[u] >= 0 && kf[u] >= 0 && kf[u] < a.n_kf) {
            kmin = min(kmin, kf[u]);
            kmax = max(kmax, kf[u]);
        }
    }
    if (kmax >= 0) {
        atomicMin(&s_k[0], kmin);
        atomicMax(&s_k[1], kmax);
    }
    for (int t0 = p0; t0 < p1; t0 += tile) {
        const int np = min(tile, p1 - t0);
        for (int q = tid; q < np * L; q += kGrpThreads) cnt[q] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (oc[u] >= 0 && pt[u] >= t0 && pt[u] - t0 < np) atomicAdd(&cnt[(pt[u] - t0) * L + oc[u]], 1);
        __syncthreads();
        int32_t *out = a.counters + (size_t)t0 * L;
        for (int q = tid; q < np * L; q += kGrpThreads) out[q] = cnt[q];
        const int k0 = s_k[0];
        const bool local = s_k[1] - k0 < kGrpSpan;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (oc[u] < 0 || pt[u] < t0 || pt[u] - t0 >= np || kf[u] < 0 || kf[u] >= a.n_kf) continue;
            const int top = min(L - 1, oc[u] + a.slack);
            const int *c = cnt + (pt[u] - t0) * L;
            int others = -1;   // the observation itself is one of the counted
            for (int l = 0; l <= top; ++l) others += c[l];
            const bool red = others >= a.min_obs;
            if (local) {
                atomicAdd(&h[tid & (kGrpCopies - 1)][kf[u] - k0], red ? 0x10001 : 1);
            } else {
                atomicAdd(&a.kf_obs[kf[u]], 1);
                if (red) atomicAdd(&a.kf_red[kf[u]], 1);
            }
        }
        __syncthreads();
    }
    const int k0 = s_k[0], span = s_k[1] - k0;
    if (s_k[1] < 0 || span >= kGrpSpan) return;
    for (int k = tid; k <= span; k += kGrpThreads) {
        int t = 0;
#pragma unroll
        for (int q = 0; q < kGrpCopies; ++q) t += h[q][k];
        if (t & 0xffff) atomicAdd(&a.kf_obs[k0 + k], t & 0xffff);
        if (t >> 16) atomicAdd(&a.kf_red[k0 + k], t >> 16);
    }
}

__global__ __launch_bounds__(256) void k_cull_count(CullArgs a) {
    if (!(a.cull[0] & 1)) return;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < a.n_obs; i += gridDim.x * 256) {
        if (a.active && !a.active[i]) continue;
        const int j = a.pt[i], o = a.oct[i];
        if (j < 0 || j >= a.n_pt || o >= a.n_levels) continue;
        atomicAdd(&a.counters[(size_t)j * a.n_levels + o], 1);
    }
}

constexpr int kCullSpan = 1024;   // keyframes per block summed in LDS
// Two observations per thread: more, or a loop over runs, lose the order in which neighbouring
// blocks meet the same points (28 million observations by keyframe: 1,816 us, four per thread
// 1,970, eight 2,040, two runs per block 1,900); 512 threads rather than 256 halve the blocks
// that return at once where the single pass ran.
constexpr int kRedThreads = 512, kRedRun = 2 * kRedThreads;   // observations of a block

__global__ __launch_bounds__(kRedThreads) void k_cull_redundant(CullArgs a) {
    __shared__ int h_obs[kCullSpan], h_red[kCullSpan];
    __shared__ int wmin[kRedThreads / 64], wmax[kRedThreads / 64];
    if (!(a.cull[0] & 1)) return;
    const int64_t i0 = (int64_t)blockIdx.x * kRedRun;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // the block's observations, every load issued before any is used, and their keyframe span
    constexpr int kPer = kRedRun / kRedThreads;
    int kf[kPer], pt[kPer], oc[kPer], on[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t i = min(i0 + threadIdx.x + kRedThreads * u, (int64_t)a.n_obs - 1);   // (past the end: the last one again)
        kf[u] = a.kf[i];
        pt[u] = a.pt[i];
        oc[u] = a.oct[i];
        on[u] = a.active ? a.active[i] : 1;
    }
    int kmin = 0x7fffffff, kmax = -1;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        kmin = min(kmin, kf[u]);
        kmax = max(kmax, kf[u]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        kmin = min(kmin, __shfl_xor(kmin, o, 64));
        kmax = max(kmax, __shfl_xor(kmax, o, 64));
    }
    if (lane == 0) {
        wmin[wv] = kmin;
        wmax[wv] = kmax;
    }
    for (int k = threadIdx.x; k < kCullSpan; k += kRedThreads) h_obs[k] = h_red[k] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kRedThreads / 64; ++w) {
        kmin = min(kmin, wmin[w]);
        kmax = max(kmax, wmax[w]);
    }
    const bool local = kmax >= kmin && kmax - kmin < kCullSpan;
    const int L = a.n_levels;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int k = kf[u], j = pt[u], o = oc[u];
        if (i0 + threadIdx.x + kRedThreads * u >= a.n_obs || !on[u] || k < 0 || k >= a.n_kf || j < 0 || j >= a.n_pt || o >= L) continue;
        const int top = min(L - 1, o + a.slack);
        const int32_t *c = a.counters + (size_t)j * L;
        int others = -1;   // the observation itself is one of the counted
        for (int l = 0; l <= top; ++l) others += c[l];
        const int red = others >= a.min_obs ? 1 : 0;
        if (local) {
            atomicAdd(&h_obs[k - kmin], 1);
            if (red) atomicAdd(&h_red[k - kmin], 1);
        } else {
            atomicAdd(&a.kf_obs[k], 1);
            if (red) atomicAdd(&a.kf_red[k], 1);
        }
    }
    if (!local) return;
    __syncthreads();
    for (int k = threadIdx.x; k <= kmax - kmin; k += kRedThreads) {
        if (h_obs[k]) atomicAdd(&a.kf_obs[kmin + k], h_obs[k]);
        if (h_red[k]) atomicAdd(&a.kf_red[kmin + k], h_red[k]);
    }
}

__global__ __launch_bounds__(256) void k_cull_decide(CullArgs a) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= a.n_kf) return;
    const int no = a.kf_obs[k], nr = a.kf_red[k];
    const bool prot = k == 0 ? a.cull[0] & 2 : a.protect && a.protect[k];
    a.cull[k] = (!prot && no > 0 && (int64_t)a.den * nr >= (int64_t)a.num * no) ? 1 : 0;
}

__global__ __launch_bounds__(256) void k_cull_check(CullArgs a) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < a.n_obs; i += gridDim.x * 256) {
        const int k = a.kf[i], j = a.pt[i], o = a.oct[i];
        if (k < 0 || k >= a.n_kf || j < 0 || j >= a.n_pt || o >= a.n_levels) atomicAdd(&a.err[kErrObs], 1);
    }
}

void launch_cull_check(const CullArgs &a, hipStream_t s) {
    if (a.n_obs <= 0) return;
    prof_begin(LMAP_KCLASS_CHECK, s);
    hipLaunchKernelGGL(k_cull_check, dim3((unsigned)std::min(4096, (a.n_obs + 255) / 256)), dim3(256), 0, s, a);
    prof_end(s);
}

void launch_cull(const CullArgs &a, hipStream_t s) {
    // few observations are bound by the launches, and the single pass takes one more (140,000: 23
    // us in general passes, 26 with it; 2.6 million: 65 and 49); its indices are 32-bit, up to the
    // end of the last run's tail
    const int64_t nc = (int64_t)a.n_pt * a.n_levels;
    const bool grouped = a.n_obs >= kGrpMinObs && a.n_obs <= INT32_MAX - kGrpRun - kGrpTail;
    prof_begin(LMAP_KCLASS_PREP, s);
    hipLaunchKernelGGL(k_cull_begin, dim3((a.n_kf + 255) / 256), dim3(256), 0, s, a, grouped ? 0 : 1);
    prof_end(s);
    if (!grouped) launch_fill_i32(a.counters, nc, 0, s);
    if (a.n_obs > 0) {
        prof_begin(LMAP_KCLASS_CULL_COUNT, s);
        if (grouped) {
            const int runs = (a.n_obs + kGrpRun - 1) / kGrpRun;
            hipLaunchKernelGGL(k_cull_order, dim3(std::min(runs, kGrpOrderBlocks)), dim3(kGrpThreads), 0, s, a);
            const int zero = (int)std::min<int64_t>(4096, (nc + 1023) / 1024);
            hipLaunchKernelGGL(k_cull_grouped, dim3(std::max(runs, zero)), dim3(kGrpThreads), 0, s, a);
        }
        const unsigned blocks = (unsigned)std::min(4096, (a.n_obs + 255) / 256);
        hipLaunchKernelGGL(k_cull_count, dim3(blocks), dim3(256), 0, s, a);
        prof_end(s);
        prof_begin(LMAP_KCLASS_CULL_REDUNDANT, s);
        hipLaunchKernelGGL(k_cull_redundant, dim3((unsigned)(((int64_t)a.n_obs + kRedRun - 1) / kRedRun)), dim3(kRedThreads), 0, s, a);
        prof_end(s);
    }
    prof_begin(LMAP_KCLASS_CULL_DECIDE, s);
    hipLaunchKernelGGL(k_cull_decide, dim3((a.n_kf + 255) / 256), dim3(256), 0, s, a);
    prof_end(s);
}

}  // namespace lmap
