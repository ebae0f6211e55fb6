// Inertial measurements of the stereo-inertial solve (Section III-C: the local bundle
// adjustment of a visual-inertial system adds inertial residuals to the reprojection
// errors).  Reading: the preintegrated IMU factor of Forster, Carlone, Dellaert and
// Scaramuzza (IEEE T-RO 2017) between keyframes, plus a bias random walk; 15 unknowns per
// optimisable keyframe (camera twist, velocity, gyroscope and accelerometer biases).
//
// Kernels, all FP64:
//   k_vi_eval    one block per measurement: residual, cost and (when linearising) the
//                Jacobian with respect to both keyframes' 15 unknowns, then its Gauss-
//                Newton blocks J^T Info J (packed lower 30 x 30) and -J^T Info r, written
//                to the measurement's record; in trial mode only the cost at the trial
//                state (pose Exp(dp) T, velocity and biases plus the step);
//   k_vi_system  the joint reduced system of 15 Kopt unknowns, the visual reduced system in
//                the pose rows and columns plus the measurements of the window added in
//                measurement order (a fixed order: results do not depend on scheduling);
//   k_vi_setup / k_vi_finish / k_vi_check   state copies and input validation.
// The damping decision adds the measurements' trial costs and applies the velocity and
// bias steps (k_decide); the round's first damping includes their diagonal
// (k_init_reduce).
#include "lba_internal.h"

namespace lba {

// ---- 3x3 helpers, row-major -------------------------------------------------------------
__device__ __forceinline__ void mm3(const double *A, const double *B, double *C) {   // C = A B
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) C[i * 3 + j] = A[i * 3] * B[j] + A[i * 3 + 1] * B[3 + j] + A[i * 3 + 2] * B[6 + j];
}
__device__ __forceinline__ void mtm3(const double *A, const double *B, double *C) {  // C = A^T B
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) C[i * 3 + j] = A[i] * B[j] + A[3 + i] * B[3 + j] + A[6 + i] * B[6 + j];
}
__device__ __forceinline__ void mv3(const double *A, const double *x, double *y) {   // y = A x
#pragma unroll
    for (int i = 0; i < 3; ++i) y[i] = A[i * 3] * x[0] + A[i * 3 + 1] * x[1] + A[i * 3 + 2] * x[2];
}
__device__ __forceinline__ void mtv3(const double *A, const double *x, double *y) {  // y = A^T x
#pragma unroll
    for (int i = 0; i < 3; ++i) y[i] = A[i] * x[0] + A[3 + i] * x[1] + A[6 + i] * x[2];
}
__device__ __forceinline__ void skew3(const double *w, double *W) {
    W[0] = 0.0;   W[1] = -w[2]; W[2] = w[1];
    W[3] = w[2];  W[4] = 0.0;   W[5] = -w[0];
    W[6] = -w[1]; W[7] = w[0];  W[8] = 0.0;
}

// SO(3) exponential through the SE(3) one (zero translation)
__device__ __forceinline__ void rot_exp(const double *w, double *R) {
    const double xi[6] = {w[0], w[1], w[2], 0.0, 0.0, 0.0};
    double t[3];
    se3_exp(xi, R, t);
}

// SO(3) logarithm: angle atan2(|sin|, cos) from the antisymmetric and trace parts; near pi
// the axis is the dominant column of the symmetric part (1 - cos t) a a^T
__device__ void rot_log(const double *R, double *w) {
    const double ax = 0.5 * (R[7] - R[5]), ay = 0.5 * (R[2] - R[6]), az = 0.5 * (R[3] - R[1]);
    const double s = sqrt(ax * ax + ay * ay + az * az);
    const double c = 0.5 * (R[0] + R[4] + R[8] - 1.0);
    const double th = atan2(s, c);
    if (th < 1e-4) {
        const double f = 1.0 + th * th * (1.0 / 6.0);
        w[0] = f * ax; w[1] = f * ay; w[2] = f * az;
        return;
    }
    if (M_PI - th > 1e-4) {
        const double f = th / s;
        w[0] = f * ax; w[1] = f * ay; w[2] = f * az;
        return;
    }
    double S[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) S[i * 3 + j] = 0.5 * (R[i * 3 + j] + R[j * 3 + i]) - (i == j ? c : 0.0);
    int k = 0;
    if (S[4] > S[k * 4]) k = 1;
    if (S[8] > S[k * 4]) k = 2;
    const double v0 = S[k], v1 = S[3 + k], v2 = S[6 + k];
    const double nv = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
    const double sg = (v0 * ax + v1 * ay + v2 * az) < 0.0 ? -1.0 : 1.0;
    w[0] = sg * th * v0 / nv; w[1] = sg * th * v1 / nv; w[2] = sg * th * v2 / nv;
}

// right Jacobian Jr(w) = I - B W + C W^2 and its inverse I + W / 2 + D W^2,
// B = (1 - cos t) / t^2, C = (t - sin t) / t^3, D = 1 / t^2 - (1 + cos t) / (2 t sin t)
__device__ void rot_jr(const double *w, double *J, bool inverse) {
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    const double th = sqrt(th2);
    double W[9], W2[9];
    skew3(w, W);
    mm3(W, W, W2);
    double a, b;
    if (inverse) {
        a = 0.5;
        b = th < 1e-2 ? 1.0 / 12.0 + th2 * (1.0 / 720.0) + th2 * th2 * (1.0 / 30240.0)
                      : 1.0 / th2 - (1.0 + cos(th)) / (2.0 * th * sin(th));
    } else {
        if (th < 1e-2) {
            a = -(0.5 - th2 * (1.0 / 24.0) + th2 * th2 * (1.0 / 720.0));
            b = 1.0 / 6.0 - th2 * (1.0 / 120.0) + th2 * th2 * (1.0 / 5040.0);
        } else {
            const double h = sin(0.5 * th);
            a = -2.0 * h * h / th2;
            b = (th - sin(th)) / (th2 * th);
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) J[i] = (i % 4 == 0 ? 1.0 : 0.0) + a * W[i] + b * W2[i];
}

// ---- per measurement ---------------------------------------------------------------------
// One wavefront per measurement.  Its constants, the two keyframes' states and every 3 x 3
// product are shared out over the lanes (groups of nine per product, one level of products
// after the other); only the rotation's exponential and logarithm run on one lane, and
// that chain bounds it.  Everything on one lane, reading its constants as it went, took 11.3
// us for one window and 17.9 for 64 (mean of linearising and trial cost); 9.6 and 13.9 so.
struct ViShared {
    double dR[9], JRg[9], Jvg[9], Jva[9], Jpg[9], Jpa[9];   // the measurement
    double dv[3], dp[3], bg[3], ba[3], dt;
    double info[81];
    double T[2][12], st[2][9];    // keyframes i and j: pose and (v, bg, ba)
    double Rc[2][9];              // R_cw
    double Rb[2][9], pb[2][3];    // body rotation R_cw^T R_cb and position R_cw^T (t_cb - t_cw)
    double A[9], tx[9];           // -R_cb^T, [t_cb]x
    double Em[9], Hu[9], Hw[9];   // rotation error; [R_i^T u]x, [R_i^T w]x
    double Jr[9], Jri[9];         // right Jacobian of the bias rotation, inverse one of r_R
    double P[15][9];              // products
    double J[15][30], OJ[15][30], r[15], Or[15];
};

// element q of A B or A^T B (3 x 3, row-major)
__device__ __forceinline__ double prod3(const double *A, bool trans, const double *B, int q) {
    const int i = q / 3, j = q - 3 * i, s0 = trans ? 1 : 3, s1 = trans ? 3 : 1;
    return A[i * s0] * B[j] + A[i * s0 + s1] * B[3 + j] + A[i * s0 + 2 * s1] * B[6 + j];
}

// The residual of the measurement in sm, and with jac its Jacobian (15 x 30, columns
// (w, u, v, bg, ba) of keyframe i then of keyframe j).  The left camera twist (w, u) turns
// the body rotation by -R_cb^T w on the right and moves the body position by
// R_cw^T ([t_cb]x w - u).
__device__ __forceinline__ void vi_residual_jacobian(const ViArgs &a, ViShared &sm, int lane, bool jac) {
    const int grp = lane / 9, q = lane - 9 * grp, qi = q / 3, qj = q - 3 * qi;
    if (grp < 2) {
        const double *T = sm.T[grp];
        sm.Rc[grp][q] = T[4 * qi + qj];
        sm.Rb[grp][q] = T[qi] * a.Tcb[qj] + T[4 + qi] * a.Tcb[4 + qj] + T[8 + qi] * a.Tcb[8 + qj];
        if (q < 3) sm.pb[grp][q] = T[q] * (a.Tcb[3] - T[3]) + T[4 + q] * (a.Tcb[7] - T[7]) + T[8 + q] * (a.Tcb[11] - T[11]);
    } else if (grp == 2) {
        sm.A[q] = -a.Tcb[4 * qj + qi];
        const double m = qi == qj ? 0.0 : a.Tcb[4 * (3 - qi - qj) + 3];
        sm.tx[q] = qj - qi == 1 || qj - qi == -2 ? -m : m;
    }
    if (jac)
        for (int i = lane; i < 450; i += 64) (&sm.J[0][0])[i] = 0.0;
    wave_sync();
    const double dt = sm.dt;
    if (lane == 0) {
        const double *si = sm.st[0], *sj = sm.st[1];
        double dbg[3], dba[3], phi[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            dbg[k] = si[3 + k] - sm.bg[k];
            dba[k] = si[6 + k] - sm.ba[k];
        }
        double Eb[9], dRc[9], RiRj[9], Em[9], r[3];
        mv3(sm.JRg, dbg, phi);
        rot_exp(phi, Eb);
        mm3(sm.dR, Eb, dRc);
        mtm3(sm.Rb[0], sm.Rb[1], RiRj);
        mtm3(dRc, RiRj, Em);
        rot_log(Em, r);
        double u[3], wv[3], Ru[3], Rw[3], t1[3], t2[3], t3[3], t4[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            u[k] = sj[k] - si[k] - a.g[k] * dt;
            wv[k] = sm.pb[1][k] - sm.pb[0][k] - si[k] * dt - 0.5 * a.g[k] * dt * dt;
        }
        mtv3(sm.Rb[0], u, Ru);
        mtv3(sm.Rb[0], wv, Rw);
        mv3(sm.Jvg, dbg, t1);
        mv3(sm.Jva, dba, t2);
        mv3(sm.Jpg, dbg, t3);
        mv3(sm.Jpa, dba, t4);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            sm.r[k] = r[k];
            sm.r[3 + k] = Ru[k] - (sm.dv[k] + t1[k] + t2[k]);
            sm.r[6 + k] = Rw[k] - (sm.dp[k] + t3[k] + t4[k]);
            sm.r[9 + k] = sj[3 + k] - si[3 + k];
            sm.r[12 + k] = sj[6 + k] - si[6 + k];
        }
        if (jac) {
            rot_jr(phi, sm.Jr, false);
            rot_jr(r, sm.Jri, true);
            skew3(Ru, sm.Hu);
            skew3(Rw, sm.Hw);
#pragma unroll
            for (int k = 0; k < 9; ++k) sm.Em[k] = Em[k];
        }
    }
    wave_sync();
    if (!jac) return;
    const double *const Ri = sm.Rb[0];
    if (grp < 6) {
        const double *L = grp == 0 ? sm.Rb[1] : grp == 1 ? sm.Em : grp == 2 ? sm.Hu : grp == 3 ? sm.Hw : sm.Rc[grp - 4];
        const double *R = grp == 0 ? Ri : grp == 1 ? sm.Jr : grp < 4 ? sm.A : sm.tx;
        sm.P[grp][q] = prod3(L, grp != 2 && grp != 3, R, q);
    }
    wave_sync();
    if (grp < 7) {   // Jri (Rj^T Ri), Jri (E^T Jr), Jri A, Ri^T (Rc^T [t]x) and Ri^T Rc^T of i and j
        const double *L = grp < 3 ? sm.Jri : grp < 5 ? Ri : sm.Rc[grp - 5];
        const double *R = grp < 2 ? sm.P[grp] : grp == 2 ? sm.A : grp < 5 ? sm.P[grp + 1] : Ri;
        sm.P[6 + grp][grp < 5 ? q : 3 * qj + qi] = prod3(L, grp == 3 || grp == 4, R, q);
    }
    wave_sync();
    if (grp < 2) sm.P[13 + grp][q] = prod3(sm.P[6 + grp], false, grp ? sm.JRg : sm.A, q);
    wave_sync();
    const double rt = Ri[3 * qj + qi];   // Ri^T
#pragma unroll
    for (int ps = 0; ps < 3; ++ps) {
        const int blk = grp + 7 * ps;
        if (grp >= 7 || blk >= 15) continue;
        int row = 0, col = 0;
        double v = 0.0;
        switch (blk) {
        case 0: row = 0; col = 0; v = -sm.P[13][q]; break;
        case 1: row = 0; col = 15; v = sm.P[8][q]; break;
        case 2: row = 0; col = 9; v = -sm.P[14][q]; break;
        case 3: row = 3; col = 0; v = sm.P[2][q]; break;
        case 4: row = 3; col = 6; v = -rt; break;
        case 5: row = 3; col = 21; v = rt; break;
        case 6: row = 3; col = 9; v = -sm.Jvg[q]; break;
        case 7: row = 3; col = 12; v = -sm.Jva[q]; break;
        case 8: row = 6; col = 0; v = sm.P[3][q] - sm.P[9][q]; break;
        case 9: row = 6; col = 3; v = sm.P[11][q]; break;
        case 10: row = 6; col = 15; v = sm.P[10][q]; break;
        case 11: row = 6; col = 18; v = -sm.P[12][q]; break;
        case 12: row = 6; col = 6; v = -dt * rt; break;
        case 13: row = 6; col = 9; v = -sm.Jpg[q]; break;
        case 14: row = 6; col = 12; v = -sm.Jpa[q]; break;
        }
        sm.J[row + qi][col + qj] = v;
    }
    if (lane < 6) {   // bias random walks
        sm.J[9 + lane][9 + lane] = -1.0;
        sm.J[9 + lane][24 + lane] = 1.0;
    }
    wave_sync();
}

__global__ __launch_bounds__(64) void k_vi_eval(ViArgs a) {
    __shared__ ViShared sm;
    const int e = blockIdx.x, lane = threadIdx.x;
    const int w = a.edge_win[e];
    if (a.trial && !a.ctl[w].running) return;
    const WinInfo W = a.win[w];
    const ViEdges &E = a.E;
    const int ki = W.kf0 + E.ei[e], kj = W.kf0 + E.ej[e];
    const int oi = a.opt_map[ki], oj = a.opt_map[kj];
    if (lane < 9) {
        sm.dR[lane] = E.dR[9 * e + lane];
        sm.JRg[lane] = E.JRg[9 * e + lane];
        sm.Jvg[lane] = E.Jvg[9 * e + lane];
        sm.Jva[lane] = E.Jva[9 * e + lane];
        sm.Jpg[lane] = E.Jpg[9 * e + lane];
        sm.Jpa[lane] = E.Jpa[9 * e + lane];
    }
    if (lane < 3) {
        sm.dv[lane] = E.dv[3 * e + lane];
        sm.dp[lane] = E.dp[3 * e + lane];
        sm.bg[lane] = E.bgb[3 * e + lane];
        sm.ba[lane] = E.bab[3 * e + lane];
    }
    if (lane == 0) sm.dt = E.dt[e];
    for (int i = lane; i < 81; i += 64) sm.info[i] = E.info[81 * (int64_t)e + i];
    const double ibg = E.ibg[e], iba = E.iba[e];
    {   // half of the lanes per keyframe
        const int side = lane >> 5, l = lane & 31, k = side ? kj : ki, o = side ? oj : oi;
        if (l < 12) {
            sm.T[side][l] = (a.trial && a.Tn ? a.Tn : a.T)[12 * (int64_t)k + l];
        } else if (l < 21) {
            double v = a.state[9 * (int64_t)k + l - 12];
            if (a.trial && o >= 0) v += a.vdp[a.vwin[w].dp_off + 15 * o + 6 + l - 12];
            sm.st[side][l - 12] = v;
        }
        wave_sync();
        if (a.trial && !a.Tn && l == 0 && o >= 0) {
            double T[12], Tt[12];
#pragma unroll
            for (int q = 0; q < 12; ++q) T[q] = sm.T[side][q];
            se3_left_update(a.dp + W.dp_off + 6 * o, T, Tt);
#pragma unroll
            for (int q = 0; q < 12; ++q) sm.T[side][q] = Tt[q];
        }
        wave_sync();
    }
    vi_residual_jacobian(a, sm, lane, !a.trial);
    // Info r and Info J: the 9 x 9 block, then the two bias blocks (multiples of I)
    if (lane < 15) {
        double v;
        if (lane < 9) {
            v = 0.0;
            for (int k = 0; k < 9; ++k) v += sm.info[lane * 9 + k] * sm.r[k];
        } else {
            v = (lane < 12 ? ibg : iba) * sm.r[lane];
        }
        sm.Or[lane] = v;
    }
    if (!a.trial)
        for (int i = lane; i < 450; i += 64) {
            const int m = i / 30, c = i - 30 * m;
            double v;
            if (m < 9) {
                v = 0.0;
                for (int k = 0; k < 9; ++k) v += sm.info[m * 9 + k] * sm.J[k][c];
            } else {
                v = (m < 12 ? ibg : iba) * sm.J[m][c];
            }
            sm.OJ[m][c] = v;
        }
    wave_sync();
    double *rec = a.ed + (int64_t)e * kViEdgeStride;
    if (lane == 0) {
        double c = 0.0;
        for (int m = 0; m < 15; ++m) c += sm.r[m] * sm.Or[m];
        rec[a.trial ? 1 : 0] = c;
    }
    if (a.trial) return;
    const bool si_opt = oi >= 0, sj_opt = oj >= 0;
    if (lane < 30) {
        double g = 0.0;
        for (int m = 0; m < 15; ++m) g += sm.J[m][lane] * sm.Or[m];
        rec[kViB + lane] = -g;
    }
    for (int idx = lane; idx < 465; idx += 64) {
        int row = (int)((sqrtf(8.0f * idx + 1.0f) - 1.0f) * 0.5f);
        while (row * (row + 1) / 2 > idx) --row;
        while ((row + 1) * (row + 2) / 2 <= idx) ++row;
        const int col = idx - row * (row + 1) / 2;
        const bool need = (row < 15 ? si_opt : sj_opt) && (col < 15 ? si_opt : sj_opt);
        double h = 0.0;
        if (need)
            for (int m = 0; m < 15; ++m) h += sm.J[m][row] * sm.OJ[m][col];
        rec[kViH + idx] = h;
    }
}

// ---- the joint reduced system ---------------------------------------------------------------
// One thread per entry: the visual system's entry, then the measurements that hold it, in
// measurement order.  One block per window that added the measurements one after the other
// was bound by that chain (38 us for one window of 10 optimisable keyframes and 14
// measurements, 44 for 64 windows); an entry belongs to few measurements, whose endpoints
// the block stages in LDS (6 and 11 us).
constexpr int kViSysEdges = 256;   // measurements staged at a time

__global__ __launch_bounds__(256) void k_vi_system(ViArgs a) {
    __shared__ int ends[kViSysEdges];   // optimisable indices of both keyframes, 255 for none
    const int w = blockIdx.y, tid = threadIdx.x;
    if (!a.ctl[w].running) return;
    const WinInfo W = a.win[w], V = a.vwin[w];
    const int n = V.n, E = V.E, idx = blockIdx.x * 256 + tid;
    if ((int)blockIdx.x * 256 >= E + n) return;   // (uniform)
    const double *Sv = a.red + W.red_off;
    const bool live = idx < E + n, side = idx >= E;
    int row = 0, col = 0;
    double v = 0.0;
    if (side) {
        row = live ? idx - E : 0;
        if (live && row % 15 < 6) v = Sv[W.E + 6 * (row / 15) + row % 15];
    } else {
        row = (int)((sqrtf(8.0f * idx + 1.0f) - 1.0f) * 0.5f);
        while (row * (row + 1) / 2 > idx) --row;
        while ((row + 1) * (row + 2) / 2 <= idx) ++row;
        col = idx - row * (row + 1) / 2;
        if (row % 15 < 6 && col % 15 < 6) v = Sv[packed_lower(6 * (row / 15) + row % 15, 6 * (col / 15) + col % 15)];
    }
    const int A = row / 15, B = col / 15, ra = row - 15 * A, cb = col - 15 * B;
    const int e0 = a.edge_off[w], e1 = a.edge_off[w + 1];
    for (int eb = e0; eb < e1; eb += kViSysEdges) {
        const int ne = min(kViSysEdges, e1 - eb);
        __syncthreads();
        for (int q = tid; q < ne; q += 256)
            ends[q] = (a.opt_map[W.kf0 + a.E.ei[eb + q]] & 255) | ((a.opt_map[W.kf0 + a.E.ej[eb + q]] & 255) << 8);
        __syncthreads();
        if (!live) continue;
        for (int q = 0; q < ne; ++q) {
            const int oi = ends[q] & 255, oj = ends[q] >> 8;   // (distinct keyframes)
            int at = -1;   // the entry's place in the measurement's record
            if (side) {
                if (oi == A || oj == A) at = kViB + (oj == A ? 15 : 0) + ra;
            } else if (A == B) {
                if (oi == A || oj == A) {
                    const int s = oj == A ? 15 : 0;
                    at = kViH + (s + ra) * (s + ra + 1) / 2 + s + cb;
                }
            } else if ((oi == A && oj == B) || (oi == B && oj == A)) {
                const int hi = oj == A ? 15 + ra : 15 + cb, lo = oj == A ? cb : ra;
                at = kViH + hi * (hi + 1) / 2 + lo;
            }
            if (at >= 0) v += a.ed[(int64_t)(eb + q) * kViEdgeStride + at];
        }
    }
    // in k_chol_tile's layout
    if (live) a.vred[V.red_off + (side ? red_rhs(n, true) + row : red_index(row, col))] = v;
}

__global__ __launch_bounds__(256) void k_vi_setup(ViArgs a) {
    for (int k = blockIdx.x * 256 + threadIdx.x; k < a.n_kf; k += gridDim.x * 256)
        for (int q = 0; q < 3; ++q) {
            a.state[9 * (int64_t)k + q] = a.v0[3 * (int64_t)k + q];
            a.state[9 * (int64_t)k + 3 + q] = a.bg0[3 * (int64_t)k + q];
            a.state[9 * (int64_t)k + 6 + q] = a.ba0[3 * (int64_t)k + q];
        }
}

__global__ __launch_bounds__(256) void k_vi_finish(ViArgs a) {
    for (int k = blockIdx.x * 256 + threadIdx.x; k < a.n_kf; k += gridDim.x * 256)
        for (int q = 0; q < 3; ++q) {
            a.v_out[3 * (int64_t)k + q] = a.state[9 * (int64_t)k + q];
            a.bg_out[3 * (int64_t)k + q] = a.state[9 * (int64_t)k + 3 + q];
            a.ba_out[3 * (int64_t)k + q] = a.state[9 * (int64_t)k + 6 + q];
        }
}

// Validation: endpoints inside their window and distinct, dt > 0, every value finite.
constexpr int32_t kErrInertial = 1 << 10;

__global__ __launch_bounds__(256) void k_vi_check(ViArgs a) {
    const ViEdges &E = a.E;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < E.n; e += gridDim.x * 256) {
        const WinInfo W = a.win[a.edge_win[e]];
        const int i = E.ei[e], j = E.ej[e];
        bool ok = i >= 0 && i < W.K && j >= 0 && j < W.K && i != j && E.dt[e] > 0.0 && isfinite(E.dt[e]);
        for (int q = 0; q < 9 && ok; ++q)
            ok = isfinite(E.dR[9 * e + q]) && isfinite(E.JRg[9 * e + q]) && isfinite(E.Jvg[9 * e + q]) &&
                 isfinite(E.Jva[9 * e + q]) && isfinite(E.Jpg[9 * e + q]) && isfinite(E.Jpa[9 * e + q]);
        for (int q = 0; q < 3 && ok; ++q)
            ok = isfinite(E.dv[3 * e + q]) && isfinite(E.dp[3 * e + q]) && isfinite(E.bgb[3 * e + q]) &&
                 isfinite(E.bab[3 * e + q]);
        for (int q = 0; q < 81 && ok; ++q) ok = isfinite(E.info[81 * (int64_t)e + q]);
        ok = ok && isfinite(E.ibg[e]) && isfinite(E.iba[e]);
        if (!ok) atomicOr(a.err, kErrInertial);
    }
    for (int k = blockIdx.x * 256 + threadIdx.x; k < a.n_kf; k += gridDim.x * 256) {
        bool ok = true;
        for (int q = 0; q < 3; ++q)
            ok = ok && isfinite(a.v0[3 * (int64_t)k + q]) && isfinite(a.bg0[3 * (int64_t)k + q]) &&
                 isfinite(a.ba0[3 * (int64_t)k + q]);
        if (!ok) atomicOr(a.err, kErrInertial);
    }
}

hipError_t launch_vi_setup(const ViArgs &a, hipStream_t s) {
    if (a.n_kf > 0) hipLaunchKernelGGL(k_vi_setup, dim3((a.n_kf + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_vi_finish(const ViArgs &a, hipStream_t s) {
    if (a.n_kf > 0) hipLaunchKernelGGL(k_vi_finish, dim3((a.n_kf + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_vi_check(const ViArgs &a, hipStream_t s) {
    const int items = std::max(a.E.n, a.n_kf);
    if (items > 0) hipLaunchKernelGGL(k_vi_check, dim3(std::min(1024, (items + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_vi_eval(const ViArgs &a, hipStream_t s) {
    if (a.E.n > 0) hipLaunchKernelGGL(k_vi_eval, dim3(a.E.n), dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_vi_system(const ViArgs &a, int n_windows, int max_n, hipStream_t s) {
    const int items = max_n * (max_n + 1) / 2 + max_n;
    if (n_windows > 0 && items > 0)
        hipLaunchKernelGGL(k_vi_system, dim3((items + 255) / 256, n_windows), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace lba
