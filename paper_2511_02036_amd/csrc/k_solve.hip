// Reduced camera system: fixed-order reduction of the per-tile partial sums, FP64 dense
// Cholesky and triangular solves for the pose step, and the per-window Levenberg-
// Marquardt decision (gain ratio, accept / reject, damping update, pose retraction).
#include "lba_internal.h"

#include <algorithm>
#include <type_traits>

namespace lba {

__device__ __forceinline__ void tri_decode(int e, int &ii, int &jj) {
    int r = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > e) --r;
    while ((r + 1) * (r + 2) / 2 <= e) ++r;
    ii = r;
    jj = e - r * (r + 1) / 2;
}

// ------------------------------------------------------------------------------------
// partial sums -> reduced system.  Each block owns 64 entries of one window; its four
// wavefronts sum the tiles t = g, g + 4, ... (g = wavefront) and the four partial sums
// are combined in a fixed order, so the result does not depend on scheduling.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_reduce(ReduceArgs a) {
    __shared__ double acc4[4][64];
    const int w = blockIdx.y;
    const WinInfo W = a.win[w];
    if (!a.ctl[w].running) return;
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;
    const int tot = W.E + W.n;
    if (blockIdx.x == 0 && g == 0) {
        // the window's point-block failure flag (written even when the system is empty)
        double fl = 0.0;
        for (int t = lane; t < W.ntiles; t += 64) fl = fmax(fl, a.partd[4 * (W.tile0 + t) + 2]);
        fl = wave_max(fl);
        if (lane == 0) a.redflag[w] = fl;
    }
    if (blockIdx.x * 64 >= tot) return;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;   // four loads in flight per step
    const double *src = nullptr;
    int64_t stride = 0;
    if (i < W.E) {
        src = a.part + W.part_off + i;
        stride = W.part_stride;
    } else if (i < tot) {
        src = a.partr + W.partr_off + (i - W.E);
        stride = W.n;
    }
    if (src) {
        int t = g;
        for (; t + 12 < W.ntiles; t += 16) {
            s0 += src[(int64_t)t * stride];
            s1 += src[(int64_t)(t + 4) * stride];
            s2 += src[(int64_t)(t + 8) * stride];
            s3 += src[(int64_t)(t + 12) * stride];
        }
        for (; t < W.ntiles; t += 4) s0 += src[(int64_t)t * stride];
    }
    acc4[g][lane] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (g == 0 && i < tot) {
        int64_t o = i;
        if (a.tiled) {
            if (i < W.E) {
                int row, col;
                tri_decode(i, row, col);
                o = red_index(row, col);
            } else {
                o = red_rhs(W.n, true) + (i - W.E);
            }
        }
        a.red[W.red_off + o] = (acc4[0][lane] + acc4[1][lane]) + (acc4[2][lane] + acc4[3][lane]);
    }
}

hipError_t launch_reduce(const ReduceArgs &a, int n_windows, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    dim3 grid((a.max_En + 63) / 64 > 0 ? (a.max_En + 63) / 64 : 1, n_windows), block(256);
    hipLaunchKernelGGL(k_reduce, grid, block, 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Dense FP64 Cholesky of S + lambda I and the two triangular solves for systems too large
// for the matrix-core variant below (more than 216 unknowns): one block of 512 threads
// per window, S held as a packed lower triangle in a per-window copy in HBM, which one
// block keeps hot in its XCD's L2 (kHbm; the template also keeps the LDS-resident form).
// Right-looking with 8-column panels.  Per panel every thread reads the 8x8 diagonal
// block and factors it redundantly in registers, so no lane-to-lane traffic sits on the
// serial path; each thread then solves one row of the panel below the block, and after
// one barrier all threads apply the rank-8 update to the trailing triangle in 4x4
// register tiles.  The forward solve L y = r rides along: every thread also solves the
// panel's 8 entries of y redundantly, and the thread of each row below subtracts its
// share.  The backward solve walks the panels from the last, every thread solving the
// panel's 8 entries from prefetched registers, then all threads updating the rows above.
// The right side, the pivots and the factored diagonal blocks stay in LDS.
// ------------------------------------------------------------------------------------
#ifndef LBA_CHOL_NB
#define LBA_CHOL_NB 8
#endif
constexpr int kNB = LBA_CHOL_NB;
constexpr int kCholThreads = 512;

size_t chol_lds_bytes_hbm(int n) { return sizeof(double) * (4 * (size_t)n + (size_t)kNB * n) + 64; }

// factor the nbk x nbk diagonal block whose top-left entry is (c0, c0) into registers:
// L (lower, row-major kNB x kNB) and its reciprocal diagonal; returns false on a
// non-positive or non-finite pivot
__device__ __forceinline__ bool diag_block_factor(const double *A, int c0, int nbk, double (&L)[kNB][kNB],
                                                  double (&rd)[kNB]) {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < kNB; ++i)
#pragma unroll
        for (int j = 0; j < kNB; ++j) L[i][j] = (i < nbk && j <= i) ? A[packed_lower(c0 + i, c0 + j)] : 0.0;
#pragma unroll
    for (int j = 0; j < kNB; ++j) {
        if (j < nbk) {
            double d = L[j][j];
#pragma unroll
            for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
            if (!(d > 0.0) || !isfinite(d)) ok = false;
            const double r = rsqrt(d);   // one reciprocal square root on the serial path
            L[j][j] = d * r;
            rd[j] = r;
#pragma unroll
            for (int i = j + 1; i < kNB; ++i) {
                double v = L[i][j];
#pragma unroll
                for (int k = 0; k < j; ++k) v -= L[i][k] * L[j][k];
                L[i][j] = v * r;
            }
        } else {
            rd[j] = 0.0;
        }
    }
    return ok;
}

// from the step x (nullptr: none): its pose part in an inertial solve; the pose step per
// keyframe and the trial poses in the segment form
__device__ __forceinline__ void trial_poses(const CholArgs &a, int w, const double *x, int tid, int nth) {
    if (!a.Tn && !a.dpv) return;
    const WinInfo V = a.vis_win[w];
    if (a.dpv)
        for (int i = tid; i < V.n; i += nth) a.dpv[V.dp_off + i] = x ? x[15 * (i / 6) + i % 6] : 0.0;
    if (!a.Tn) return;
    for (int k = tid; k < V.K; k += nth) {
        const int o = a.opt_map[V.kf0 + k];
        double d[6], T[12];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            d[i] = x && o >= 0 ? x[a.stride * o + i] : 0.0;
            a.dk[6 * (int64_t)(V.kf0 + k) + i] = d[i];
        }
#pragma unroll
        for (int i = 0; i < 12; ++i) T[i] = a.T[12 * (int64_t)(V.kf0 + k) + i];
        double *Tn = a.Tn + 12 * (int64_t)(V.kf0 + k);
        if (o >= 0) {
            se3_left_update(d, T, Tn);
        } else {
#pragma unroll
            for (int i = 0; i < 12; ++i) Tn[i] = T[i];
        }
    }
}

template <bool kHbm>
__global__ __launch_bounds__(kCholThreads) void k_cholesky(CholArgs a) {
    extern __shared__ __align__(16) double cs[];
    __shared__ int s_fail;
    const int w = blockIdx.x;
    const WinInfo W = a.win[w];
    Ctl *ctl = a.ctl + w;
    if (!ctl->running) return;
    const int n = W.n, E = W.E;
    const int tid = threadIdx.x, lane = tid & 63;
    const int nth = blockDim.x;
    const double lambda = ctl->lambda;
    double *A = kHbm ? a.fact + W.red_off : cs;   // E, packed lower
    double *y = kHbm ? cs : cs + E;               // n: right side, then the solution
    double *rr = y + n;      // n: copy of the right side (gain-ratio denominator)
    double *rdiag = rr + n;  // n reciprocal pivots
    double *Ld = rdiag + n;  // n x kNB: factored diagonal blocks (row r holds L[r][c0 .. r])
    double *xs = Ld + (size_t)n * kNB;   // n: the solution of L^T x = y
    const double *red = a.red + W.red_off;
    // eight loads in flight per thread (one at a time, each waited on before its store,
    // took a memory round trip per 512 entries)
    for (int i0 = tid; i0 < E + n; i0 += 8 * nth) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * nth;
            v[u] = i < E + n ? red[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * nth;
            if (i < E) {
                A[i] = v[u];
            } else if (i < E + n) {
                y[i - E] = v[u];
                rr[i - E] = v[u];
            }
        }
    }
    if (tid == 0) s_fail = a.redflag[w] != 0.0;
    __syncthreads();
    for (int i = tid; i < n; i += nth) A[packed_lower(i, i)] += lambda;
    __syncthreads();

    // ---- factorisation ----------------------------------------------------------------
    for (int c0 = 0; c0 < n; c0 += kNB) {
        const int nbk = min(kNB, n - c0);
        const int b0 = c0 + nbk;
        double L[kNB][kNB], rd[kNB];
        const bool ok = diag_block_factor(A, c0, nbk, L, rd);
        // the panel's entries of y (forward solve), redundantly in every thread
        double yp[kNB];
#pragma unroll
        for (int j = 0; j < kNB; ++j) {
            double v = j < nbk ? y[c0 + j] : 0.0;
#pragma unroll
            for (int k = 0; k < j; ++k) v -= L[j][k] * yp[k];
            yp[j] = v * rd[j];
        }
        if (!ok) {
            if (tid == 0) s_fail = 1;
        } else {
            // panel rows below the diagonal block: L[r][c0+j] = (A[r][c0+j] - sum_k L[r][c0+k] L[c0+j][c0+k]) / L[c0+j][c0+j]
            for (int r = b0 + tid; r < n; r += nth) {
                double x[kNB];
#pragma unroll
                for (int j = 0; j < kNB; ++j) x[j] = j < nbk ? A[packed_lower(r, c0 + j)] : 0.0;
#pragma unroll
                for (int j = 0; j < kNB; ++j) {
                    double v = x[j];
#pragma unroll
                    for (int k = 0; k < j; ++k) v -= x[k] * L[j][k];
                    x[j] = v * rd[j];
                }
                double dy = 0.0;
#pragma unroll
                for (int j = 0; j < kNB; ++j) {
                    if (j < nbk) A[packed_lower(r, c0 + j)] = x[j];
                    dy += x[j] * yp[j];
                }
                y[r] -= dy;   // this thread owns row r of y in this phase
            }
            // the factored diagonal block goes to Ld (A's copy is still being read by
            // other threads in this phase)
            if (tid < nbk * kNB) {
                const int i = tid / kNB, j = tid % kNB;
                double v = 0.0;
#pragma unroll
                for (int ii = 0; ii < kNB; ++ii)
#pragma unroll
                    for (int jj = 0; jj < kNB; ++jj)
                        if (ii == i && jj == j) v = L[ii][jj];
                Ld[(c0 + i) * kNB + j] = v;
            }
            if (tid < nbk) {
                double v = 0.0;
#pragma unroll
                for (int jj = 0; jj < kNB; ++jj)
                    if (jj == tid) v = rd[jj];
                rdiag[c0 + tid] = v;
            }
        }
        __syncthreads();
        if (s_fail) break;
        // the panel's solved entries of y (every thread has read the unsolved ones)
        if (tid < nbk) {
            double v = 0.0;
#pragma unroll
            for (int jj = 0; jj < kNB; ++jj)
                if (jj == tid) v = yp[jj];
            y[c0 + tid] = v;
        }
        // trailing update A[i][j] -= sum_kk L[i][c0+kk] L[j][c0+kk], b0 <= j <= i < n
        const int m = n - b0;
        const int T4 = (m + 3) / 4;
        const int ntile = T4 * (T4 + 1) / 2;
        for (int t = tid; t < ntile; t += nth) {
            int I, J;
            tri_decode(t, I, J);
            const int i0 = b0 + 4 * I, j0 = b0 + 4 * J;
            double ai[4][kNB], aj[4][kNB];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ri = i0 + u, rj = j0 + u;
#pragma unroll
                for (int kk = 0; kk < kNB; ++kk) {
                    ai[u][kk] = (ri < n && kk < nbk) ? A[packed_lower(ri, c0 + kk)] : 0.0;
                    aj[u][kk] = (rj < n && kk < nbk) ? A[packed_lower(rj, c0 + kk)] : 0.0;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = i0 + u, j = j0 + v;
                    if (i < n && j <= i) {
                        double acc = 0.0;
#pragma unroll
                        for (int kk = 0; kk < kNB; ++kk) acc += ai[u][kk] * aj[v][kk];
                        A[packed_lower(i, j)] -= acc;
                    }
                }
            }
        }
        __syncthreads();
    }
    const int ok = !s_fail;

    // ---- L^T x = y (y was solved with the factorisation; one barrier per panel) ------
    // Each panel's entries of x go to their own array, so the threads still reading the
    // panel's y are not overtaken by its solution; the rows above are updated in the same
    // step.
    if (ok) {
        const int last = n > 0 ? ((n - 1) / kNB) * kNB : 0;
        for (int c0 = last; c0 >= 0 && n > 0; c0 -= kNB) {
            const int nbk = min(kNB, n - c0);
            // the panel's diagonal block and right side, all loads issued before the chain
            double Lb[kNB][kNB], yb[kNB], rb[kNB], xp[kNB];
#pragma unroll
            for (int k = 0; k < kNB; ++k) {
                yb[k] = k < nbk ? y[c0 + k] : 0.0;
                rb[k] = k < nbk ? rdiag[c0 + k] : 0.0;
#pragma unroll
                for (int j = 0; j < k; ++j) Lb[k][j] = k < nbk ? Ld[(c0 + k) * kNB + j] : 0.0;
            }
#pragma unroll
            for (int j = kNB - 1; j >= 0; --j) {
                double v = yb[j];
#pragma unroll
                for (int k = j + 1; k < kNB; ++k) v -= Lb[k][j] * xp[k];
                xp[j] = v * rb[j];
            }
            if (tid < nbk) {
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < kNB; ++j)
                    if (j == tid) v = xp[j];
                xs[c0 + tid] = v;
            }
            for (int j = tid; j < c0; j += nth) {
                double acc = 0.0;
#pragma unroll
                for (int kk = 0; kk < kNB; ++kk)
                    if (kk < nbk) acc += A[packed_lower(c0 + kk, j)] * xp[kk];
                y[j] -= acc;
            }
            __syncthreads();
        }
    }
    double *dp = a.dp + W.dp_off;
    if (tid < 64) {
        double den = 0.0;
        for (int i = lane; i < n; i += 64) {
            const double x = ok ? xs[i] : 0.0;
            dp[i] = x;
            den += x * (lambda * x + rr[i]);   // + point part in the update kernel
        }
        den = wave_sum(den);
        if (lane == 0) {
            ctl->solve_ok = ok;
            ctl->denom_p = den;
        }
    } else {
        trial_poses(a, w, ok ? xs : nullptr, tid - 64, nth - 64);
    }
}


// ------------------------------------------------------------------------------------
// The same factorisation and solves for systems of up to 216 unknowns, on the FP64 matrix
// cores with the matrix in registers: S + lambda I, with the right side appended as row n
// (so that the forward solve L y = r is part of the factorisation) and identity rows up to
// the next multiple of 16, is cut into 16 x 16 tiles of its lower triangle.  Tile (I, J)
// is held transposed in the accumulator layout of v_mfma_f64_16x16x4 (lane l, value v:
// row l % 16 of I, column l / 16 + 4 v of J) by wavefront t % 8, t its place in the
// triangle's columns.  In that layout a tile is a B operand as it stands and the A operand
// of its transpose, so no tile is ever rearranged.  Per panel of 16 columns:
//   1. the tiles below the diagonal are multiplied by the inverse factor of the diagonal
//      tile and published to LDS;
//   2. every trailing tile subtracts the product of its two panel tiles; the owner of the
//      next diagonal tile does that one first and factors it while the others go on.
// The diagonal tile is factored by one wavefront with a row per lane (the four rows of 16
// lanes hold copies): its row and the identity's row, which the same column operations turn
// into the inverse factor; a step's pivot row comes by DPP broadcasts, one reciprocal
// square root per step is on the serial path.  The back solve L^T x = y multiplies by the stored
// inverse factors (no serial chain within a panel), one barrier per panel.  Every sum is
// taken in a fixed order, so solves repeat bit for bit.
// What bounds it: the chain of diagonal tiles (update 0.4k, 16 elimination steps 2.6k of the
// about 6k cycles per panel, panel tiles, two barriers), not the FP64 matrix rate of one
// compute unit (n^3 / 3 flops take 9 us at n = 180).  4 x 4 tiles in registers with 4-column
// panels took four times the barriers and panel steps.  One system, before and now: n = 120
// 61 and 31 us, n = 180 136 and 55 us, n = 216 about 170 and 77 us.
// ------------------------------------------------------------------------------------
constexpr int kTileMaxN = 216;
constexpr int kTileMaxNB = (kTileMaxN + 1 + 15) / 16;               // 14 tile rows
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int tile_slots(int nb) { return (nb * (nb + 1) / 2 + kTileWaves - 1) / kTileWaves; }   // tiles per wavefront

int chol_tile_max_n() { return kTileMaxN; }

typedef double d4 __attribute__((ext_vector_type(4)));

template <int ror>
__device__ __forceinline__ double row_ror(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + ror, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + ror, 0xF, 0xF, false);
    return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

// lane c ^ 1 or c ^ 2
template <int x>
__device__ __forceinline__ double quad_xor(double v) {
    constexpr int perm = x == 1 ? 0xB1 : 0x4E;   // [1, 0, 3, 2] or [2, 3, 0, 1]
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, perm, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), perm, 0xF, 0xF, false);
    return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

__device__ __forceinline__ double join_fp64(unsigned lo, unsigned hi) {
    return __longlong_as_double((long long)lo | ((long long)hi << 32));
}

// sum over the four rows of 16 lanes, in every lane
__device__ __forceinline__ double group_sum(double v) {
    unsigned lo = (unsigned)__double_as_longlong(v), hi = (unsigned)(__double_as_longlong(v) >> 32);
    const auto l2 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h2 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    const double u = join_fp64(l2[0], h2[0]) + join_fp64(l2[1], h2[1]);
    lo = (unsigned)__double_as_longlong(u);
    hi = (unsigned)(__double_as_longlong(u) >> 32);
    const auto l1 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h1 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return join_fp64(l1[0], h1[0]) + join_fp64(l1[1], h1[1]);
}

// lane j of each row of 16 lanes to the whole row
template <int j>
__device__ __forceinline__ double row_bcast(double v) {
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + j, 0xF, 0xF, true));
}

// elimination steps j .. 15 with a row per lane of the tile (A) and of what becomes the
// transposed inverse factor (B); columns from `real` on are padding (pivot 1)
template <int j>
__device__ __forceinline__ void row_steps(double (&A)[16], double (&B)[16], bool &ok, int real) {
    double p = row_bcast<j>(A[j]);
    if (j >= real) p = 1.0;
    ok = ok && p > 0.0 && p < __builtin_huge_val();
    const double rs = rsqrt_fp64(p);
    A[j] *= rs;   // L[i][j]
    B[j] *= rs;
    const double v = -A[j] * rs, u = -B[j] * rs;
#pragma unroll
    for (int c = j + 1; c < 16; ++c) {
        const double q = row_bcast<j>(A[c]);   // A[j][c]
        A[c] = fma(q, v, A[c]);
        B[c] = fma(q, u, B[c]);
        // (B is stored by some lanes only: without this its updates would sink into that
        // branch and keep every q alive)
        asm volatile("" : "+v"(B[c]));
    }
    if constexpr (j < 15) row_steps<j + 1>(A, B, ok, real);
}

// f(constant q) for q = Q .. Q1 - 1 (constants, so that arrays indexed by them stay in
// registers), and the same for the set bits of a uniform mask
template <int Q, int Q1, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (Q < Q1) {
        f(std::integral_constant<int, Q>{});
        static_for<Q + 1, Q1>(f);
    }
}
template <int Q, int Q1, typename F>
__device__ __forceinline__ void masked_for(unsigned m, F &&f) {
    if constexpr (Q < Q1) {
        if ((m >> Q) & 1u) f(std::integral_constant<int, Q>{});
        masked_for<Q + 1, Q1>(m, f);
    }
}
template <int N, typename F>
__device__ __forceinline__ void each_slot(unsigned m, F &&f) {
    constexpr int h = N / 2;
    if (m & ((1u << h) - 1u)) masked_for<0, h>(m, f);
    if (m >> h) masked_for<h, N>(m, f);
}
#define LBA_INLINE __attribute__((always_inline))

template <int kNB>   // tile rows, at most
__global__ __launch_bounds__(kTileThreads) void k_chol_tile(CholArgs a) {
    constexpr int kSlots = tile_slots(kNB);
    __shared__ double Qp[kNB][4][64];   // the panel's tiles
    __shared__ double Lt[kNB][4][64];   // inverse factors of the diagonal tiles, transposed
    __shared__ double Ln[kNB][4][64];   // and as they are (the back solve's operand)
    __shared__ double Dt[16][16];              // the diagonal tile being factored
    __shared__ double y[16 * kNB], xs[16 * kNB], rr[16 * kNB];
    __shared__ int s_fail;
    const int w = blockIdx.x;
    const WinInfo W = a.win[w];
    Ctl *ctl = a.ctl + w;
    if (!ctl->running) return;
    const int n = W.n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, g = lane >> 4;
    const double lambda = ctl->lambda;
    const double *red = a.red + W.red_off, *rhs = red + red_rhs(n, true);
    const int NB = n / 16 + 1;       // rows 0 .. n
    const int In = n / 16, rn = n - 16 * In;   // tile row of the right side, its row there
    const int ntiles = n < 16 * kNB ? NB * (NB + 1) / 2 : 0;
    auto col_start = [&](int J) { return J * NB - J * (J - 1) / 2; };   // place of tile (J, J)
    // this wavefront's slots of the places [t0, t1)
    auto slots = [&](int t0, int t1) {
        auto below = [&](int t) { return (1u << max(0, (t - wave + kTileWaves - 1) / kTileWaves)) - 1u; };
        return below(t1) & ~below(t0);
    };
    if (tid == 0) s_fail = (a.redflag[w] != 0.0) || n >= 16 * kNB;
    // own tiles (slot s: place wave + 8 s of the triangle's columns)
    int tI[kSlots], tJ[kSlots];
    d4 T[kSlots];
    {
        int J = 0, off = wave;       // off: place within column J
        static_for<0, kSlots>([&](auto q) LBA_INLINE {
            constexpr int s = q.value;
            while (J < NB && off >= NB - J) {
                off -= NB - J;
                ++J;
            }
            const bool have = wave + kTileWaves * s < ntiles;
            tI[s] = have ? J + off : -1;
            tJ[s] = have ? J : -1;
            off += kTileWaves;
            // every load is issued before any value is used (tiles that hold only the right
            // side and padding read tile 0 instead)
            const double *t = red + (have && 16 * tI[s] < n ? red_tile(tI[s], tJ[s]) : 0);
            const bool diag = have && tI[s] == tJ[s];
#pragma unroll
            for (int v = 0; v < 4; ++v) T[s][v] = t[diag && g + 4 * v > c ? red_in_tile(g + 4 * v, c) : 64 * v + lane];
        });
        for (int i = tid; i < 16 * kNB; i += kTileThreads) {
            rr[i] = i < n ? rhs[i] : 0.0;
            y[i] = 0.0;
        }
        __syncthreads();
        static_for<0, kSlots>([&](auto q) LBA_INLINE {   // the diagonal, the right side and the padding
            constexpr int s = q.value;
            if (tI[s] < 0 || (tI[s] != tJ[s] && tI[s] != In)) return;
            const int row = 16 * tI[s] + c, col0 = 16 * tJ[s] + g;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int col = col0 + 4 * v, i = min(row, col);
                const bool side = max(row, col) == n && i < n;
                const double b = rr[i];
                double x = row < n && col < n ? T[s][v] : side ? b : 0.0;
                if (row == col) x = row < n ? x + lambda : 1.0;
                T[s][v] = x;
            }
        });
    }
    __syncthreads();
    // (s_fail is read only right after a barrier that follows its last write: a thread
    // that read it while another sets it would leave the panel loop alone)
    const bool failed_before = s_fail != 0;

    // factor the diagonal tile D of panel k: its inverse factor goes to Lt and Ln
    auto factor = [&](d4 D, int k) LBA_INLINE {
        double A[16], B[16];
        // (the lane index is re-derived behind an empty asm statement: what depends on it
        // would otherwise be kept in registers across the panel loop, which has none left)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int c = lane & 15, g = lane >> 4;
#pragma unroll
        for (int v = 0; v < 4; ++v) Dt[g + 4 * v][c] = D[v];
        wave_sync();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            A[q] = Dt[q][c];   // symmetric
            B[q] = q == c ? 1.0 : 0.0;
        }
        bool ok = true;
        row_steps<0>(A, B, ok, n - 16 * k);
        if (g == 0) {   // B: row c of the transposed inverse factor
#pragma unroll
            for (int q = 0; q < 16; ++q) Lt[k][c >> 2][q + 16 * (c & 3)] = B[q];
#pragma unroll
            for (int q = 0; q < 16; ++q) Ln[k][q >> 2][c + 16 * (q & 3)] = B[q];
            if (k == In && c == rn) {
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (q < rn) y[16 * k + q] = A[q];
            }
        }
        if (!ok && lane == 0) s_fail = 1;
    };
    // D - (L_Jk) (L_Ik)^T, the 16 products of an entry summed before they are subtracted: with D
    // as the matrix instructions' accumulator each of them rounds at D's size, and the pose steps'
    // error against 80 bits was 25 to 45% larger (same time)
    auto update = [&](d4 D, int I, int J) LBA_INLINE {
        double qj[4], qi[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            qj[v] = Qp[J][v][lane];
            qi[v] = Qp[I][v][lane];
        }
        d4 P = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) P = __builtin_amdgcn_mfma_f64_16x16x4f64(qj[v], qi[v], P, 0, 0, 0);
        return D - P;
    };

    // ---- factorisation and forward solve ----------------------------------------------
    if (!failed_before) {
        for (int k = -1; k < NB - 1; ++k) {   // (k = -1: the first diagonal tile)
            if (s_fail) break;
            const int off = k < 0 ? 0 : col_start(k), nxt = k < 0 ? 0 : col_start(k + 1);
            // 1. the tiles below the diagonal: (L_Ik)^T = L_kk^-1 (A_Ik)^T
            each_slot<kSlots>(slots(off + 1, nxt), [&](auto q) LBA_INLINE {
                    d4 &t = T[q.value];
                    const int I = tI[q.value];
                    d4 D = {0.0, 0.0, 0.0, 0.0};
                    double li[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) li[v] = Lt[k][v][lane];
#pragma unroll
                    for (int v = 0; v < 4; ++v) D = __builtin_amdgcn_mfma_f64_16x16x4f64(li[v], t[v], D, 0, 0, 0);
                    t = D;
#pragma unroll
                    for (int v = 0; v < 4; ++v) Qp[I][v][lane] = D[v];
                    if (I == In && c == rn) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) y[16 * k + g + 4 * v] = D[v];
                    }
                });
            __syncthreads();
            // 2. trailing tiles, the next diagonal tile first
            if ((nxt & (kTileWaves - 1)) == wave) {
                d4 D = {0.0, 0.0, 0.0, 0.0};
                each_slot<kSlots>(1u << (nxt / kTileWaves), [&](auto q) LBA_INLINE { D = T[q.value]; });
                if (k >= 0) D = update(D, k + 1, k + 1);
                factor(D, k + 1);
            }
            if (k >= 0)
                each_slot<kSlots>(slots(nxt + 1, ntiles),
                          [&](auto q) LBA_INLINE { T[q.value] = update(T[q.value], tI[q.value], tJ[q.value]); });
            __syncthreads();
        }
    }
    __syncthreads();
    const int ok = !s_fail;

    // ---- back solve L^T x = y, one barrier per panel -------------------------------------
    // x_k = L_kk^-T y_k (every wavefront forms it), then the owners of the tiles left of
    // the diagonal subtract their share (L_kJ)^T x_k from y_J
    if (ok) {
        for (int k = NB - 1; k >= 0; --k) {
            double x = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) x = fma(Ln[k][v][lane], y[16 * k + g + 4 * v], x);
            x = group_sum(x);   // x_k[c]
            if (wave == 0 && g == 0) xs[16 * k + c] = x;
            unsigned todo = 0;
            static_for<0, kSlots>([&](auto q) LBA_INLINE { todo |= (tI[q.value] == k && tJ[q.value] < k) ? 1u << q.value : 0u; });
            each_slot<kSlots>(todo, [&](auto slot) LBA_INLINE {
                    const d4 &t = T[slot.value];
                    const int J = tJ[slot.value];
                    double q[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) q[v] = t[v] * x;
                    // sums over the 16 lanes of a row: lane c keeps value c % 4
                    const double u0 = (c & 1 ? q[1] : q[0]) + quad_xor<1>(c & 1 ? q[0] : q[1]);
                    const double u1 = (c & 1 ? q[3] : q[2]) + quad_xor<1>(c & 1 ? q[2] : q[3]);
                    double d = (c & 2 ? u1 : u0) + quad_xor<2>(c & 2 ? u0 : u1);
                    d += row_ror<4>(d);
                    d += row_ror<8>(d);
                    if (c < 4) y[16 * J + g + 4 * c] -= d;
                });
            __syncthreads();
        }
    }
    double *dp = a.dp + W.dp_off;
    if (tid < 64) {
        double den = 0.0;
        for (int i = lane; i < n; i += 64) {
            const double x = ok ? xs[i] : 0.0;
            dp[i] = x;
            den += x * (lambda * x + rr[i]);   // + point part in the update kernel
        }
        den = wave_sum(den);
        if (lane == 0) {
            ctl->solve_ok = ok;
            ctl->denom_p = den;
        }
    } else {
        trial_poses(a, w, ok ? xs : nullptr, tid - 64, kTileThreads - 64);
    }
}

size_t chol_static_lds() { return kernel_static_lds((const void *)k_cholesky<true>); }

hipError_t launch_cholesky(const CholArgs &a, int n_windows, size_t lds, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    if (a.fact) hipLaunchKernelGGL(k_cholesky<true>, dim3(n_windows), dim3(kCholThreads), lds, s, a);
    else if (a.max_n < 16 * 8) hipLaunchKernelGGL(k_chol_tile<8>, dim3(n_windows), dim3(kTileThreads), 0, s, a);
    else if (a.max_n < 16 * 12) hipLaunchKernelGGL(k_chol_tile<12>, dim3(n_windows), dim3(kTileThreads), 0, s, a);
    else hipLaunchKernelGGL(k_chol_tile<kTileMaxNB>, dim3(n_windows), dim3(kTileThreads), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// LM decision per window (one wavefront): gain ratio, accept / reject, damping update
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_decide(DecideArgs a) {
    __shared__ int s_acc;
    const int w = blockIdx.x;
    const WinInfo W = a.win[w];
    Ctl *ctl = a.ctl + w;
    if (!ctl->running) return;
    const int lane = threadIdx.x;
    double Ft = 0.0, den = 0.0, fl = 0.0;
    if (a.part_seg) {   // the window's segments
        const int64_t s0 = a.seg_base[3 * (int64_t)W.rng0];
        const int64_t s1 = a.seg_base[3 * ((int64_t)W.rng0 + (W.M + a.range_pts - 1) / a.range_pts)];
        for (int64_t s = s0 + lane; s < s1; s += 64) {
            Ft += a.part_seg[2 * s];
            den += a.part_seg[2 * s + 1];
        }
    }
    const int64_t u0 = (int64_t)W.tile0 * a.split;   // the update's parts of this window's tiles
    for (int t = lane; t < W.ntiles * a.split && !a.part_seg; t += 64) {
        Ft += a.partu[4 * (u0 + t)];
        den += a.partu[4 * (u0 + t) + 1];
        fl = fmax(fl, a.partu[4 * (u0 + t) + 2]);
    }
    if (a.vi_ed)   // the inertial measurements' costs at the trial state
        for (int e = a.vi_edge_off[w] + lane; e < a.vi_edge_off[w + 1]; e += 64) Ft += a.vi_ed[(int64_t)e * kViEdgeStride + 1];
    Ft = wave_sum(Ft);
    den = wave_sum(den) + ctl->denom_p;
    fl = wave_max(fl);
    if (lane == 0) {
        const int ok = ctl->solve_ok && fl == 0.0;
        const double gain = (ctl->F - Ft) / den;
        const int acc = ok && isfinite(Ft) && isfinite(gain) && gain > 0.0;
        if (a.log && ctl->trials_total < a.log_cap) {
            TrialRec &L = a.log[(int64_t)w * a.log_cap + ctl->trials_total];
            L.round = a.round;
            L.iter = ctl->iter;
            L.trial = ctl->trial;
            L.accepted = acc;
            L.solve_ok = ok;
            L.pad = 0;
            L.lambda = ctl->lambda;
            L.F = ctl->F;
            L.F_trial = Ft;
            L.gain = gain;
        }
        ctl->F_trial = Ft;
        ctl->trials_total += 1;
        const int iters = a.c.iters[a.round - 1];
        if (acc) {
            ctl->F = Ft;
            const double f = 2.0 * gain - 1.0;
            ctl->lambda *= fmax(1.0 / 3.0, 1.0 - f * f * f);
            ctl->nu = 2.0;
            ctl->cur ^= 1;
            ctl->iter += 1;
            ctl->trial = 0;
            if (a.round == 1) ctl->iters_r1 = ctl->iter;
            else ctl->iters_r2 = ctl->iter;
            if (ctl->iter >= iters) ctl->running = 0;
        } else {
            ctl->lambda *= ctl->nu;
            ctl->nu *= 2.0;
            ctl->trial += 1;
            if (ctl->trial >= a.c.max_trials) {
                ctl->running = 0;
                if (a.round == 1) ctl->term_r1 = 1;
                else ctl->term_r2 = 1;
            }
        }
        s_acc = acc;
    }
    __syncthreads();
    if (s_acc) {
        // accepted: T_k <- Exp(dp_k) T_k for the window's optimisable keyframes
        const double *dp = a.dp + W.dp_off;
        for (int k = lane; k < W.K; k += 64) {
            const int ok = a.opt_map[W.kf0 + k];
            if (ok < 0) continue;
            double *T = a.T + 12 * (int64_t)(W.kf0 + k);
            double Tin[12];
#pragma unroll
            for (int i = 0; i < 12; ++i) Tin[i] = T[i];
            if (a.Tn) {
#pragma unroll
                for (int i = 0; i < 12; ++i) T[i] = a.Tn[12 * (int64_t)(W.kf0 + k) + i];
            } else {
                se3_left_update(dp + 6 * ok, Tin, T);
            }
            if (a.vi_state) {   // velocity and biases move additively
                const double *d = a.vi_dp + a.vi_win[w].dp_off + 15 * ok + 6;
                double *st = a.vi_state + 9 * (int64_t)(W.kf0 + k);
#pragma unroll
                for (int q = 0; q < 9; ++q) st[q] += d[q];
            }
        }
    }
}

hipError_t launch_decide(const DecideArgs &a, int n_windows, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_decide, dim3(n_windows), dim3(64), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// damping initialisation of a round: F and lambda0 = tau * max diag(H)
// ------------------------------------------------------------------------------------
constexpr int kInitCols = 384;   // columns of one window's r (n = 6 Kopt <= 360), six per lane
constexpr int kInitRedThreads = 1024;
constexpr int kInitRedWaves = kInitRedThreads / 64;

__global__ __launch_bounds__(kInitRedThreads) void k_init_reduce(InitReduceArgs a) {
    __shared__ double smax[kInitRedWaves];
    __shared__ double colsum[kInitRedWaves][kInitCols];
    const int w = blockIdx.x;
    const WinInfo W = a.win[w];
    Ctl *ctl = a.ctl + w;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // largest diagonal entry of Hpp (per camera, summed over the tiles): wavefront g sums
    // the tiles g, g + G, ... (G wavefronts, four tiles per step), lane l the columns l,
    // l + 64, ... (coalesced rows) ...
    constexpr int G = kInitRedWaves;
    double cs[kInitCols / 64] = {};
    const double *pr = a.partr + W.partr_off;
    for (int t0 = wave; t0 < W.ntiles; t0 += 4 * G) {
#pragma unroll
        for (int c = 0; c < kInitCols / 64; ++c) {
            const int col = lane + 64 * c;
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * G;
                if (col < W.n && t < W.ntiles) v += pr[(int64_t)t * W.n + col];
            }
            cs[c] += v;
        }
    }
#pragma unroll
    for (int c = 0; c < kInitCols / 64; ++c) colsum[wave][lane + 64 * c] = cs[c];
    __syncthreads();
    double md = 0.0;
    if (!a.vi_ed) {
        for (int i = tid; i < W.n; i += blockDim.x) {
            double v = 0.0;
            for (int g = 0; g < G; ++g) v += colsum[g][i];
            md = fmax(md, v);
        }
    } else {
        // the joint diagonal: visual pose entries plus every inertial measurement's
        // diagonal on the 15 unknowns of its two keyframes
        const int e0 = a.vi_edge_off[w], e1 = a.vi_edge_off[w + 1];
        for (int i = tid; i < 15 * W.Kopt; i += blockDim.x) {
            const int o = i / 15, c = i % 15;
            double v = 0.0;
            if (c < 6)
                for (int g = 0; g < G; ++g) v += colsum[g][6 * o + c];
            for (int e = e0; e < e1; ++e) {
                const double *rec = a.vi_ed + (int64_t)e * kViEdgeStride + kViH;
                if (a.opt_map[W.kf0 + a.vi_ei[e]] == o) v += rec[c * (c + 1) / 2 + c];
                if (a.opt_map[W.kf0 + a.vi_ej[e]] == o) v += rec[(15 + c) * (16 + c) / 2 + 15 + c];
            }
            md = fmax(md, v);
        }
    }
    // ... and of the point blocks (per tile), and the cost
    double F = 0.0;
    for (int t = tid; t < W.ntiles; t += blockDim.x) md = fmax(md, a.partd[4 * (W.tile0 + t) + 1]);
    if (wave == 0) {
        for (int t = lane; t < W.ntiles; t += 64) F += a.partd[4 * (W.tile0 + t)];
        if (a.vi_ed)
            for (int e = a.vi_edge_off[w] + lane; e < a.vi_edge_off[w + 1]; e += 64)
                F += a.vi_ed[(int64_t)e * kViEdgeStride];
    }
    md = wave_max(md);
    F = wave_sum(F);
    if (lane == 0) smax[wave] = md;
    __syncthreads();
    if (tid == 0) {
        md = 0.0;
        for (int g = 0; g < kInitRedWaves; ++g) md = fmax(md, smax[g]);
        if (a.round == 1) {
            ctl->F_initial = F;
        } else {
            ctl->F_end_r1 = ctl->F;
            ctl->F_start_r2 = F;
        }
        ctl->F = F;
        ctl->lambda = a.c.tau * md;
        ctl->nu = 2.0;
        ctl->iter = 0;
        ctl->trial = 0;
        ctl->round = a.round;
        ctl->running = a.c.iters[a.round - 1] > 0 ? 1 : 0;
    }
}

static_assert(6 * kMaxKoptFP64 <= kInitCols && 6 * kMaxKoptMixed <= kInitCols, "columns per lane");

hipError_t launch_init_reduce(const InitReduceArgs &a, int n_windows, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_init_reduce, dim3(n_windows), dim3(kInitRedThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace lba
