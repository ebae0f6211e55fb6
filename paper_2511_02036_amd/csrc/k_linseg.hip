// Linearisation + Schur complement by segments (see k_segments for the plan).
//
// One wavefront takes one segment: a run of points seen by at most kSegCams optimisable
// keyframes between them, in chunks of at most 64 observations (one per lane) and 32
// points.  No wavefront waits for another: all of its staging is its own part of LDS.  Its
// share of the reduced camera system,
//     S = Hpp + lambda I - sum_j sum_{a,b in obs(j)} W_a V_j^-1 W_b^T,
//     r = bp - sum_j sum_{a in obs(j)} W_a V_j^-1 bl_j,
// over its own cameras (60 rows at most) stays in registers for the whole segment.  Per
// chunk:
//   1. each lane forms its observation's residual (FP64), robust weight and FP64 point block
//      Hll_a, bl_a;
//   2. the point sums, one (point, entry) per lane; each lane then factors its point's
//      V = Hll + lambda I = L L^T (reciprocal square roots), and the point's first lane
//      stores the factor for the update;
//   3. Z_a = W_a L^-T goes to LDS, and the observation's own terms Hpp_a - Z_a Z_a^T and
//      r_a = bp_a - Z_a L^-1 bl into FP64 sums per camera (LDS atomics from the lanes of one
//      wavefront only, which the hardware applies in a fixed order; two copies, by the
//      point's parity, halve the lanes that meet at one address);
//   4. the blocks of two cameras of -Z Z^T on the matrix cores (those of one camera come out
//      too and are not read: summed apart from Hpp they would round at the size of what
//      cancels): rows are (camera, component), the contraction runs
//      over (point, component) with four points per step.  A lane finds its row's
//      observation of its point through a byte map (a zero row where the camera does not
//      see the point), so the operands are gathered from LDS and nothing is padded there.
// At the end the segment writes its tiles and camera sums as one record; k_reduce_seg sums a
// window's records in segment order.  Every sum is taken in a fixed order: solves repeat bit
// for bit.
//
// What bounds it: per chunk about 4k cycles of FP64 matrix instructions, 6k of FP64 vector
// work and LDS round trips, and the waits for the next chunk's data, at two wavefronts per
// SIMD (the sums of four row tiles take 80 registers); a small problem is bound by the chain
// of one chunk, about 20k cycles.  Per step, against k_linearize (one block per tile of
// points, pairs of observations listed and summed by the vector units): 11.4 us for one window
// of 12,000 observations (35), 19.4 us for 64,000 (45), 131 us for 48 windows of 1.4 million
// together (362).
// One segment per workgroup: four to a workgroup waited for the longest of them (half as
// slow again on batches).
#include "lba_internal.h"

#include <algorithm>

namespace lba {

constexpr int kSegThreads = 64;    // one segment per workgroup: segments differ in length
constexpr int kSegCopies = 2;      // copies of the camera sums, by point parity

typedef double d4 __attribute__((ext_vector_type(4)));

struct SegLds {
    static constexpr int ZS = 19;   // row stride of Z in values (odd: gathered rows spread over the banks)
    union {
        double hs[9 * 65];          // per entry and observation: Hll (6), bl (3)
        double vs[kSegPoints * 9];  // then the point sums
        double Z[65 * ZS];          // per observation Z_a; row 64 is zero
    };
    double dac[kSegCopies][kSegCams * 27];   // per camera: Hpp (21, lower), r (6)
    double xs[kSegPoints * 3];      // positions of the chunk's points
    uint32_t map[kSegPoints * 4];   // per point, one byte per camera: observation, or 64
    int pst[kSegPoints];            // first observation | observations << 8
};

// 3 x 3 Cholesky V = L L^T and Li = L^-1 by reciprocal square roots (order as chol3_inv)
__device__ __forceinline__ bool chol3_rsqrt(const double *V /*00 01 02 11 12 22*/, double *Li) {
    const double i00 = rsqrt_fp64(V[0]);
    const double l10 = V[1] * i00, l20 = V[2] * i00;
    const double d1 = V[3] - l10 * l10;
    const double i11 = rsqrt_fp64(d1);
    const double l21 = (V[4] - l20 * l10) * i11;
    const double d2 = V[5] - l20 * l20 - l21 * l21;
    const double i22 = rsqrt_fp64(d2);
    const double i10 = -l10 * i00 * i11;
    Li[0] = i00; Li[1] = i10; Li[2] = i11;
    Li[3] = -(l20 * i00 + l21 * i10) * i22;
    Li[4] = -l21 * i11 * i22;
    Li[5] = i22;
    return V[0] > 0.0 && d1 > 0.0 && d2 > 0.0;
}

// value v at byte offset `off` of a buffer; nothing where off is past its end
__device__ __forceinline__ void store_past(__amdgpu_buffer_rsrc_t b, unsigned off, double v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const u2 d = {(unsigned)u, (unsigned)(u >> 32)};
    __builtin_amdgcn_raw_buffer_store_b64(d, b, (int)off, 0, 0);
}

template <typename ZT>
__global__ __launch_bounds__(kSegThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_linseg(LinSegArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int ZS = SegLds::ZS, kCams = kSegCams, kRowTiles = (6 * kCams + 15) / 16, kTiles = kRowTiles * (kRowTiles + 1) / 2;
    double *const wt = reinterpret_cast<double *>(smem);   // 1 / sigma2 per octave, Huber thresholds
    const int lane = threadIdx.x;
    if (lane < kMaxLevels + 2) wt[lane] = lane < kMaxLevels ? a.c.inv_sigma2[lane] : a.c.huber2[lane - kMaxLevels];
    wave_sync();
    SegLds &sm = *reinterpret_cast<SegLds *>(smem + sizeof(double) * (kMaxLevels + 2));
    const int nseg = a.info[kSegInfoCount];
    const ZT *const sz = static_cast<const ZT *>(a.sz);
    const CamParams cam = a.c.cam;

    for (int sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
        // everything the segment's record leads to is loaded at once: its window's control
        // block and poses, its chunks' headers (one per lane) and the first chunk's data
        const Seg S = a.segs[sg];
        const Ctl *ctl = a.ctl + S.win;
        const int running = ctl->running, state = ctl->cur;
        const double lambda = ctl->lambda;
        const double *Tw = a.T + 12 * (int64_t)S.kf0;
        const int4 hdr = a.chunks[S.chunk0 + min(lane, S.nchunk - 1)];
        uint32_t word;
        ZT z0, z1, z2;
        int4 pin;
        double Xp0, Xp1, Xp2;
        // (loads without branches, of the last observation or point where a lane has none: a
        // value merged with an older one would be waited for at once)
        auto load_obs = [&](const int4 &k) {
            const int64_t o = min(k.z + min(lane, max((k.w & 255) - 1, 0)), a.n_obs - 1);
            word = a.words[o];
            z0 = sz[o];
            z1 = sz[(int64_t)a.n_obs + o];
            z2 = sz[2 * (int64_t)a.n_obs + o];
            pin = a.pinfo[k.x + min(lane, k.y - 1)];
        };
        int4 ck = S.first;
        load_obs(ck);
        if (!running) continue;
        const double *Xs = state ? a.X1 : a.X0;
        auto load_points = [&](const int4 &k) {
            const int64_t p = k.x + min(lane, k.y - 1);
            Xp0 = Xs[3 * p];
            Xp1 = Xs[3 * p + 1];
            Xp2 = Xs[3 * p + 2];
        };
        load_points(ck);
        auto chunk = [&](int ch) {
            return make_int4(__builtin_amdgcn_readlane(hdr.x, ch), __builtin_amdgcn_readlane(hdr.y, ch),
                             __builtin_amdgcn_readlane(hdr.z, ch), __builtin_amdgcn_readlane(hdr.w, ch));
        };
        d4 acc[kTiles];
#pragma unroll
        for (int i = 0; i < kTiles; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};
        for (int i = lane; i < kSegCopies * kCams * 27; i += 64) (&sm.dac[0][0])[i] = 0.0;
        int fail = 0;

        for (int ch = 0; ch < S.nchunk; ++ch) {
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));
            const int c = lane & 15, g = lane >> 4;
            const int np = ck.y, nobs = ck.w & 255;
            if (lane < np) {
                sm.pst[lane] = (pin.w - ck.z) | (pin.z << 8);
                sm.xs[3 * lane] = Xp0;
                sm.xs[3 * lane + 1] = Xp1;
                sm.xs[3 * lane + 2] = Xp2;
            }
            sm.map[lane] = 0x40404040u;
            sm.map[64 + lane] = 0x40404040u;
            wave_sync();
            // ---- 1. the observation (lanes without one repeat the chunk's last) ------------
            const int kf = word & 127u, stereo = (word >> 7) & 1u, oct = (word >> 8) & 31u;
            const int lc = (word >> 13) & 15u, pl = (word >> 17) & 31u;
            const bool has = lane < nobs, act = !(word & kSegInactive);
            const bool opt = has && act && lc != kSegNoCam;
            // what phases 3 and 5 need: G = om P^T P (G01 = 0), M = G R, the camera point and bp_a
            double G00, G02, G11, G12, G22, M[9], x, y, z;
            double bp[6];
            {
                double T[12];
                // (from memory: staged in LDS once per segment they cost 1 to 2% of a solve with up to
                // 40 keyframes, and 6% from 48 on, where only seven segments fit a compute unit)
#pragma unroll
                for (int i = 0; i < 12; ++i) T[i] = Tw[12 * kf + i];
                double xc, yc, zc, eu, ev, er;
                const double e2 = residual(cam, T, sm.xs[3 * pl], sm.xs[3 * pl + 1], sm.xs[3 * pl + 2], (double)z0,
                                           (double)z1, (double)z2, stereo, xc, yc, zc, eu, ev, er);
                const double isg = wt[oct];
                double rho, w;
                huber(e2 * isg, wt[kMaxLevels + stereo], a.robust, rho, w);
                const double omd = act ? w * isg : 0.0;
                double Hll[6], bl[3];
                point_block_fp64(cam, T, xc, yc, zc, eu, ev, er, stereo, omd, Hll, bl);
#pragma unroll
                for (int i = 0; i < 6; ++i) sm.hs[i * 65 + lane] = Hll[i];
#pragma unroll
                for (int i = 0; i < 3; ++i) sm.hs[(6 + i) * 65 + lane] = bl[i];
                double gd[3];
                obs_gradient(cam, xc, yc, zc, eu, ev, er, stereo, omd, gd);
                bp[0] = yc * gd[2] - zc * gd[1];
                bp[1] = zc * gd[0] - xc * gd[2];
                bp[2] = xc * gd[1] - yc * gd[0];
                bp[3] = gd[0]; bp[4] = gd[1]; bp[5] = gd[2];
                ObsBlocks<double> B;
                obs_blocks<double>(cam, T, xc, yc, zc, eu, ev, er, stereo, omd, B);
                G00 = B.G[0]; G02 = B.G[2]; G11 = B.G[3]; G12 = B.G[4]; G22 = B.G[5];
#pragma unroll
                for (int i = 0; i < 9; ++i) M[i] = B.M[i];
                x = B.x[0]; y = B.x[1]; z = B.x[2];
            }
            // the next chunk's loads
            const int4 cur = ck;
            if (ch + 1 < S.nchunk) {
                ck = chunk(ch + 1);
                load_obs(ck);
            }
            wave_sync();
            // ---- 2. point sums and factors ----------------------------------------------
            constexpr int kPass = (9 * kSegPoints + 63) / 64;
            double sums[kPass];
#pragma unroll
            for (int ps = 0; ps < kPass; ++ps) {
                const int it = lane + 64 * ps;
                sums[ps] = 0.0;
                if (64 * ps >= 9 * np) continue;
                const int pt = (it * 7282) >> 16, e = it - 9 * pt;   // it / 9, it < 320
                const int st = pt < np ? sm.pst[pt] : 0;
                const double *h = sm.hs + e * 65 + (st & 255);
                const int m = st >> 8;
                double v = 0.0;
                for (int i = 0; i < m; i += 4) {   // four loads in flight; the sum keeps its order
                    double u[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) u[q] = h[min(i + q, m - 1)];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v += i + q < m ? u[q] : 0.0;
                }
                sums[ps] = v;
            }
            wave_sync();   // (every term has been read: the sums take their place)
#pragma unroll
            for (int ps = 0; ps < kPass; ++ps) {
                const int it = lane + 64 * ps;
                if (it < 9 * np) sm.vs[it] = sums[ps];
            }
            wave_sync();
            double Li[6], t0 = 0, t1 = 0, t2 = 0;
            {
                double V[6], bs[3];
#pragma unroll
                for (int i = 0; i < 6; ++i) V[i] = sm.vs[9 * pl + i];
#pragma unroll
                for (int i = 0; i < 3; ++i) bs[i] = sm.vs[9 * pl + 6 + i];
                V[0] += lambda;
                V[3] += lambda;
                V[5] += lambda;
                if (!chol3_rsqrt(V, Li) && has) fail = 1;
                lmul<double>(Li, bs[0], bs[1], bs[2], t0, t1, t2);
                // the point's factor, for this step's back-substitution, by its first lane, plane
                // by plane: buffer stores whose other lanes lie past the plane's end (such lanes
                // store nothing), because a branch here would make the waits for the next chunk's
                // loads wait for these stores too
                const bool first = has && lane == (sm.pst[pl] & 255);
                const unsigned off = first ? 8u * (unsigned)(cur.x + pl) : 0xfffffff0u;
                auto plane = [&](int i, double v) {
                    store_past(__builtin_amdgcn_make_buffer_rsrc(a.pf + (int64_t)i * a.n_pt, (short)0, 8 * a.n_pt, 0x00020000), off, v);
                };
#pragma unroll
                for (int i = 0; i < 6; ++i) plane(i, Li[i]);
                plane(6, t0);
                plane(7, t1);
                plane(8, t2);
            }
            load_points(ck);
            // ---- 3. Z and the camera sums ------------------------------------------------
            wave_sync();   // (Z takes the place of the sums)
            if (lane < 18) sm.Z[64 * ZS + lane] = 0;
            double *const dst = sm.dac[pl & (kSegCopies - 1)] + 27 * lc;
            if (opt) {
                reinterpret_cast<uint8_t *>(sm.map)[16 * pl + lc] = (uint8_t)lane;
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    double w[3];   // row i of W_a = [x]x M ; M
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        w[k] = i == 0 ? y * M[6 + k] - z * M[3 + k]
                             : i == 1 ? z * M[k] - x * M[6 + k]
                             : i == 2 ? x * M[3 + k] - y * M[k] : M[3 * (i - 3) + k];
                    double y0, y1, y2;
                    lmul<double>(Li, w[0], w[1], w[2], y0, y1, y2);
                    sm.Z[lane * ZS + 3 * i] = y0;
                    sm.Z[lane * ZS + 3 * i + 1] = y1;
                    sm.Z[lane * ZS + 3 * i + 2] = y2;
                    bp[i] -= y0 * t0 + y1 * t1 + y2 * t2;   // r_a
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            wave_sync();
            // ---- 4. S -= Z Z^T ---------------------------------------------------------------
            const uint8_t *const map = reinterpret_cast<const uint8_t *>(sm.map);
            // row tiles with a camera of this chunk
            int live = 0;
            {
                const unsigned cams = (unsigned)cur.w >> 8;
#pragma unroll
                for (int t = 0; t < kRowTiles; ++t) {
                    const int c0 = 16 * t / 6, c1 = (16 * t + 15) / 6;   // its first and last camera
                    live |= (cams >> c0) & ((2u << (c1 - c0)) - 1u) ? 1 << t : 0;
                }
            }
            for (int q0 = 0; q0 < cur.y; q0 += 4) {
                double fr[kRowTiles][3];
#pragma unroll
                for (int t = 0; t < kRowTiles; ++t) {
                    if (!((live >> t) & 1)) continue;
                    const int row = 16 * t + c, cm = row / 6;
                    const int slot = map[16 * (q0 + g) + cm];
                    const double *zp = sm.Z + slot * ZS + 3 * (row - 6 * cm);
#pragma unroll
                    for (int k = 0; k < 3; ++k) fr[t][k] = zp[k];
                }
                if (q0 == 0 && opt) {   // (behind the first operands in the LDS queue)
#pragma unroll
                    for (int i = 0; i < 6; ++i) lds_add(dst + 21 + i, bp[i]);
                }
#pragma unroll
                for (int I = 0; I < kRowTiles; ++I) {
#pragma unroll
                    for (int J = 0; J <= I; ++J) {
                        if (!((live >> I) & 1) || !((live >> J) & 1)) continue;
                        const int ti = I * (I + 1) / 2 + J;
#pragma unroll
                        for (int k = 0; k < 3; ++k)
                            acc[ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(-fr[I][k], fr[J][k], acc[ti], 0, 0, 0);
                    }
                }
            }
            // Hpp's entries last: they drain while the next chunk's data arrives
            if (opt) {
                // [x]x G, then the lower triangle of Hpp = [[x]x G [x]x^T, . ; G [x]x^T, G]
                const double C00 = y * G02, C01 = y * G12 - z * G11, C02 = y * G22 - z * G12;
                const double C10 = z * G00 - x * G02, C11 = -x * G12, C12 = z * G02 - x * G22;
                const double C20 = -y * G00, C21 = x * G11, C22 = x * G12 - y * G02;
                const double H[21] = {y * C02 - z * C01,
                                    y * C12 - z * C11, z * C10 - x * C12,
                                    y * C22 - z * C21, z * C20 - x * C22, x * C21 - y * C20,
                                    C00, C10, C20, G00,
                                    C01, C11, C21, 0, G11,
                                    C02, C12, C22, G02, G12, G22};
                // less Z_a Z_a^T, before either is summed: the two nearly cancel where a point has
                // few observations (pose steps' error 5 to 10% larger otherwise; same time)
                double zz[18];
#pragma unroll
                for (int i = 0; i < 18; ++i) zz[i] = sm.Z[lane * ZS + i];
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int j = 0; j <= i; ++j) {
                        const int e = i * (i + 1) / 2 + j;
                        lds_add(dst + e, H[e] - (zz[3 * i] * zz[3 * j] + zz[3 * i + 1] * zz[3 * j + 1] + zz[3 * i + 2] * zz[3 * j + 2]));
                    }
            }
            wave_sync();   // (the next chunk overwrites the staging)
        }

        // ---- the segment's record -----------------------------------------------------------
        // (the lane index is re-derived behind an empty asm statement, here and per chunk: the
        // addresses built from it would otherwise stay in registers, and spill, across the loops)
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int c = lane & 15, g = lane >> 4;
        double *rec = a.rec + S.rec;
        const int nrow = 6 * S.ncam;
#pragma unroll
        for (int I = 0; I < kRowTiles; ++I) {
            if (16 * I >= nrow) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * I + g + 4 * v, ca = row / 6;
                const int len = row < nrow ? 6 * (ca + 1) : 0;   // the row's entries in the record
                double *const out = rec + 3 * ca * (6 * (ca + 1)) + (row - 6 * ca) * len + c;
#pragma unroll
                for (int J = 0; J <= I; ++J)
                    if (16 * J + c < len) out[16 * J] = acc[I * (I + 1) / 2 + J][v];
            }
        }
        for (int i = lane; i < 27 * S.ncam; i += 64) rec[seg_blocks(S.ncam) + i] = sm.dac[0][i] + sm.dac[1][i];
        const int anyfail = __any(fail);
        if (lane == 0) a.segfail[sg] = anyfail;
        wave_sync();
    }
}

hipError_t launch_linseg(const LinSegArgs &a, int64_t seg_cap, bool z_f32, hipStream_t s) {
    if (seg_cap <= 0) return hipSuccess;
    const size_t lds = sizeof(double) * (kMaxLevels + 2) + sizeof(SegLds);
    const dim3 grid((unsigned)std::min<int64_t>(seg_cap, 1 << 16)), block(kSegThreads);   // (a stride beyond)
    if (z_f32) hipLaunchKernelGGL(k_linseg<float>, grid, block, lds, s, a);
    else hipLaunchKernelGGL(k_linseg<double>, grid, block, lds, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// records -> reduced system.  One block per camera block (kA <= kB) of one window: its
// wavefronts share the window's segments and add up those that hold both cameras (lanes: the
// 36 entries, for a diagonal block the 21 lower ones and the 6 of r), and their sums are
// combined in a fixed order.  Bound by the records' bytes on batches (41 us for 48
// windows of 1.4 million observations, k_reduce took 10 for its partial systems), by the chain of loads on one
// window (10 us at 64,000 observations); eight loads in flight, more cost occupancy (16:
// half as slow again on large batches).
// ------------------------------------------------------------------------------------
constexpr int kRedSegWaves = 16;
constexpr int kRedSegFlight = 8;

__global__ __launch_bounds__(64 * kRedSegWaves) void k_reduce_seg(ReduceSegArgs a) {
    __shared__ double part[kRedSegWaves][64];
    const int w = blockIdx.y;
    const WinInfo W = a.win[w];
    if (!a.ctl[w].running) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t s0 = a.base[3 * (int64_t)W.rng0];
    const int64_t s1 = a.base[3 * ((int64_t)W.rng0 + (W.M + a.range_pts - 1) / a.range_pts)];
    if (blockIdx.x == 0 && wave == 0) {   // the window's point-block failure flag
        int fl = 0;
        for (int64_t s = s0 + lane; s < s1; s += 64) fl |= a.segfail[s];
        fl = __any(fl);
        if (lane == 0) a.redflag[w] = fl ? 1.0 : 0.0;
    }
    const int Kopt = W.Kopt;
    if ((int)blockIdx.x >= Kopt * (Kopt + 1) / 2) return;
    // block index -> (kB, kA), row kB of the lower block triangle
    int kB = (int)((sqrtf(8.0f * blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    while (kB * (kB + 1) / 2 > (int)blockIdx.x) --kB;
    while ((kB + 1) * (kB + 2) / 2 <= (int)blockIdx.x) ++kB;
    const int kA = blockIdx.x - kB * (kB + 1) / 2;
    const bool diag = kA == kB;
    const int i = lane / 6, j = lane - 6 * (lane / 6);
    const bool entry = lane < 36 && (!diag || j <= i), rside = diag && lane >= 36 && lane < 42;
    const int hoff = rside ? lane - 15 : i * (i + 1) / 2 + j;   // of a diagonal block's camera sums
    const unsigned long long both = (1ull << kA) | (1ull << kB);
    // this wavefront's share of the segments
    const int64_t per = (s1 - s0 + a.waves - 1) / a.waves;
    const int64_t b1 = min(s1, s0 + per * (wave + 1));
    double sum = 0.0;
    for (int64_t b = s0 + per * wave; b < b1; b += 64) {
        // per segment (one per lane): where this camera block starts in its record
        unsigned long long m = 0;
        int64_t ro = 0, ho = 0;
        int len = 0;
        if (b + lane < b1) {
            const Seg S = a.segs[b + lane];
            m = S.mask;
            const int la = __popcll(m & ((1ull << kA) - 1ull)), lb = __popcll(m & ((1ull << kB) - 1ull));
            len = 6 * (lb + 1);
            ro = S.rec + 3 * lb * len + 6 * la;
            ho = S.rec + seg_blocks(S.ncam) + 27 * la;
        }
        unsigned long long hit = __ballot((m & both) == both);
        while (hit) {   // eight segments at a time: their loads are independent
            double v[kRedSegFlight], h[kRedSegFlight];
#pragma unroll
            for (int u = 0; u < kRedSegFlight; ++u) {
                v[u] = h[u] = 0.0;
                if (!hit) continue;
                const int l = __builtin_ctzll(hit);
                hit &= hit - 1;
                auto uniform = [&](int64_t x) {   // lane l's value
                    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32) |
                                     (uint32_t)__builtin_amdgcn_readlane((int)x, l));
                };
                // (read by every lane: l may have no entry)
                const double *const vb = a.rec + uniform(ro), *const hb = a.rec + uniform(ho);
                const int ln = __builtin_amdgcn_readlane(len, l);
                if (entry && !diag) v[u] = vb[i * ln + j];
                if (diag && (entry || rside)) h[u] = hb[hoff];
            }
#pragma unroll
            for (int u = 0; u < kRedSegFlight; ++u) sum += v[u] + h[u];
        }
    }
    part[wave][lane] = sum;
    __syncthreads();
    if (wave != 0 || !(entry || rside)) return;
    double v = part[0][lane];
    for (int q = 1; q < a.waves; ++q) v += part[q][lane];
    double *red = a.red + W.red_off;
    if (rside) {
        red[red_rhs(W.n, a.tiled) + 6 * kB + lane - 36] = v;
    } else {
        const int row = 6 * kB + i, col = 6 * kA + j;
        red[a.tiled ? red_index(row, col) : packed_lower(row, col)] = v;
    }
}

hipError_t launch_reduce_seg(const ReduceSegArgs &a, int n_windows, hipStream_t s) {
    if (n_windows <= 0) return hipSuccess;
    if (a.waves < 1 || a.waves > kRedSegWaves) return hipErrorInvalidValue;
    const int nb = std::max(1, a.max_kopt * (a.max_kopt + 1) / 2);
    hipLaunchKernelGGL(k_reduce_seg, dim3(nb, n_windows), dim3(64 * a.waves), 0, s, a);
    return hipGetLastError();
}

}  // namespace lba
