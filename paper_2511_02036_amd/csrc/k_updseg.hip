// Back-substitution, retraction and trial cost by segments (see k_segments for the plan; the
// general form is k_update).
//
// One block per segment, its wavefronts taking the segment's chunks in turn: at most 64
// observations, one per lane, of at most 32 points, one per lane.  Everything the chunk
// reads is contiguous in the linearisation order: the observations' words and measurements,
// the points' positions and the point factors that the linearisation of the same step left.
// The window's poses, trial poses and pose steps (formed once per window by the reduced
// solve) are staged in LDS per block.  Each lane forms W_a^T dp_k(a) = R^T G c in FP64 at
// the current state; lane l sums them for the chunk's point l and back-substitutes with
// V = L L^T, t = L^-1 bl:
//   u = L^-1 q,  y = t - u,  dl = L^-T y,   q = sum_a W_a^T dp_k(a),   X' = X + dl,
// then every lane evaluates its observation's robust cost at (T', X').  The point's part of
// the gain-ratio denominator, dl^T (lambda dl + bl) + q^T V^-1 bl, is
// lambda |dl|^2 + y.t + u.t = lambda |dl|^2 + |t|^2, so bl is not needed.
//
// Bound by the latency of a chunk's loads and its LDS round trips (about 1.5 TB/s of its
// bytes on batches).  Per step against k_update: one window of 64,000
// observations 7 us (10), 48 windows of 1.4 million 44 us (33; the positions that it reads and
// writes in order save that back in k_linseg, whose point loads would be gathers).
#include "lba_internal.h"

#include <algorithm>

namespace lba {

struct UpdSegStage {
    double q[64 * 3];              // per observation: W_a^T dp
    double xs[kSegPoints * 3];     // positions, then trial positions of the chunk's points
    int pst[kSegPoints];           // first observation | observations << 8
};

template <typename ZT>
__global__ __launch_bounds__(256) void k_updseg(UpdSegArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[4][3];
    __shared__ double wt[kMaxLevels + 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = blockDim.x >> 6;
    UpdSegStage &sm = reinterpret_cast<UpdSegStage *>(smem)[wave];
    double *const Tl = reinterpret_cast<double *>(smem + sizeof(UpdSegStage) * waves);
    double *const Tn = Tl + 12 * a.max_k, *const dk = Tn + 12 * a.max_k;
    if (tid < kMaxLevels + 2) wt[tid] = tid < kMaxLevels ? a.c.inv_sigma2[tid] : a.c.huber2[tid - kMaxLevels];
    const int nseg = a.info[kSegInfoCount];
    const ZT *const sz = static_cast<const ZT *>(a.sz);
    const CamParams cam = a.c.cam;
    for (int sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
        const Seg S = a.segs[sg];
        const Ctl *ctl = a.ctl + S.win;
        const int running = ctl->running, state = ctl->cur;
        const double lambda = ctl->lambda;
        if (!running) continue;   // (uniform over the block)
        const double *Xs = state ? a.X1 : a.X0;
        double *Xn = state ? a.X0 : a.X1;
        __syncthreads();          // (the previous segment's poses and sums have been read)
        for (int i = tid; i < 12 * S.K; i += blockDim.x) {
            Tl[i] = a.T[12 * (int64_t)S.kf0 + i];
            Tn[i] = a.Tn[12 * (int64_t)S.kf0 + i];
        }
        for (int i = tid; i < 6 * S.K; i += blockDim.x) dk[i] = a.dk[6 * (int64_t)S.kf0 + i];
        __syncthreads();
        double Ftr = 0.0, den = 0.0;
        for (int ch = wave; ch < S.nchunk; ch += waves) {
            const int4 ck = a.chunks[S.chunk0 + ch];
            const int np = ck.y, nobs = ck.w & 255;
            const int64_t o = min(ck.z + min(lane, max(nobs - 1, 0)), a.n_obs - 1), pos = ck.x + min(lane, np - 1);
            const uint32_t word = a.words[o];
            const ZT z0 = sz[o], z1 = sz[(int64_t)a.n_obs + o], z2 = sz[2 * (int64_t)a.n_obs + o];
            const int4 pin = a.pinfo[pos];
            const double P0 = Xs[3 * pos], P1 = Xs[3 * pos + 1], P2 = Xs[3 * pos + 2];
            double f[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = a.pf[(int64_t)i * a.n_pt + pos];
            if (lane < np) {
                sm.pst[lane] = (pin.w - ck.z) | (pin.z << 8);
                sm.xs[3 * lane] = P0;
                sm.xs[3 * lane + 1] = P1;
                sm.xs[3 * lane + 2] = P2;
            }
            wave_sync();
            const int kf = word & 127u, stereo = (word >> 7) & 1u, oct = (word >> 8) & 31u, pl = (word >> 17) & 31u;
            const bool act = lane < nobs && !(word & kSegInactive);
            const double isg = wt[oct], hub = wt[kMaxLevels + stereo];
            double qv[3] = {0.0, 0.0, 0.0};
            if (act) {
                const double *T = Tl + 12 * kf, *d = dk + 6 * kf;
                double xc, yc, zc, eu, ev, er, rho, w;
                const double e2 = residual(cam, T, sm.xs[3 * pl], sm.xs[3 * pl + 1], sm.xs[3 * pl + 2], (double)z0,
                                           (double)z1, (double)z2, stereo, xc, yc, zc, eu, ev, er);
                huber(e2 * isg, hub, a.robust, rho, w);
                obs_step_q(cam, T, xc, yc, zc, stereo, w * isg, d[1] * zc - d[2] * yc + d[3], d[2] * xc - d[0] * zc + d[4],
                           d[0] * yc - d[1] * xc + d[5], qv);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) sm.q[3 * lane + i] = qv[i];
            wave_sync();
            if (lane < np) {
                const int m0 = pin.w - ck.z, m1 = m0 + pin.z;
                double q0 = 0.0, q1 = 0.0, q2 = 0.0;
                for (int m = m0; m < m1; ++m) {
                    q0 += sm.q[3 * m];
                    q1 += sm.q[3 * m + 1];
                    q2 += sm.q[3 * m + 2];
                }
                // (points without observations have no factor and keep their position)
                double d0 = 0.0, d1 = 0.0, d2 = 0.0;
                if (pin.z > 0) {
                    const double y0 = f[6] - f[0] * q0, y1 = f[7] - (f[1] * q0 + f[2] * q1),
                                 y2 = f[8] - (f[3] * q0 + f[4] * q1 + f[5] * q2);
                    d0 = f[0] * y0 + f[1] * y1 + f[3] * y2;
                    d1 = f[2] * y1 + f[4] * y2;
                    d2 = f[5] * y2;
                    den += lambda * (d0 * d0 + d1 * d1 + d2 * d2) + (f[6] * f[6] + f[7] * f[7] + f[8] * f[8]);
                }
                const double X0 = P0 + d0, X1 = P1 + d1, X2 = P2 + d2;
                Xn[3 * pos] = X0;
                Xn[3 * pos + 1] = X1;
                Xn[3 * pos + 2] = X2;
                sm.xs[3 * lane] = X0;
                sm.xs[3 * lane + 1] = X1;
                sm.xs[3 * lane + 2] = X2;
            }
            wave_sync();
            if (act) {
                double xc, yc, zc, eu, ev, er, rho, w;
                const double e2 = residual(cam, Tn + 12 * kf, sm.xs[3 * pl], sm.xs[3 * pl + 1], sm.xs[3 * pl + 2],
                                           (double)z0, (double)z1, (double)z2, stereo, xc, yc, zc, eu, ev, er);
                huber(e2 * isg, hub, a.robust, rho, w);
                Ftr += rho;
            }
            wave_sync();
        }
        Ftr = wave_sum(Ftr);
        den = wave_sum(den);
        if (lane == 0) {
            red[wave][0] = Ftr;
            red[wave][1] = den;
        }
        __syncthreads();
        if (tid == 0) {
            double F = 0.0, D = 0.0;
            for (int w = 0; w < waves; ++w) {
                F += red[w][0];
                D += red[w][1];
            }
            a.partu[2 * (int64_t)sg] = F;
            a.partu[2 * (int64_t)sg + 1] = D;
        }
    }
}

hipError_t launch_updseg(const UpdSegArgs &a, int64_t seg_cap, int waves, bool z_f32, hipStream_t s) {
    if (seg_cap <= 0) return hipSuccess;
    if (waves < 1 || waves > 4) return hipErrorInvalidValue;
    const size_t lds = sizeof(UpdSegStage) * waves + sizeof(double) * 30 * a.max_k;
    const dim3 grid((unsigned)std::min<int64_t>(seg_cap, 1 << 16)), block(64 * waves);
    if (z_f32) hipLaunchKernelGGL(k_updseg<float>, grid, block, lds, s, a);
    else hipLaunchKernelGGL(k_updseg<double>, grid, block, lds, s, a);
    return hipGetLastError();
}

// positions <-> points: X by position from the points in index order, and back
__global__ __launch_bounds__(256) void k_to_positions(const int4 *pinfo, const double *X, double *Xp, int n) {
    for (int p = blockIdx.x * 256 + threadIdx.x; p < n; p += gridDim.x * 256) {
        const int64_t P = pinfo[p].x;
#pragma unroll
        for (int i = 0; i < 3; ++i) Xp[3 * (int64_t)p + i] = X[3 * P + i];
    }
}

__global__ __launch_bounds__(256) void k_from_positions(UpdSegArgs a, double *X) {
    const WinInfo W = a.win[blockIdx.y];
    const double *Xs = a.ctl[blockIdx.y].cur ? a.X1 : a.X0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < W.M; i += gridDim.x * 256) {
        const int64_t p = W.pt0 + i, P = a.pinfo[p].x;
#pragma unroll
        for (int q = 0; q < 3; ++q) X[3 * P + q] = Xs[3 * p + q];
    }
}

hipError_t launch_to_positions(const int4 *pinfo, const double *X, double *Xp, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_to_positions, dim3(std::min(4096, (n + 255) / 256)), dim3(256), 0, s, pinfo, X, Xp, n);
    return hipGetLastError();
}

hipError_t launch_from_positions(const UpdSegArgs &a, double *X, int n_windows, int max_points, hipStream_t s) {
    if (n_windows <= 0 || max_points <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_from_positions, dim3(std::min(64, (max_points + 255) / 256), n_windows), dim3(256), 0, s, a, X);
    return hipGetLastError();
}

}  // namespace lba
