// Pair sums of mutual drop pairs (gfx950, FP64): two drops whose nodes are all
// in each other's region 0 (Sec. 2.3), so that the regular rule of Sec. 2.1 on
// the standard grid runs in both directions over the same pairs of nodes. A
// pair's difference, distance and power of 1/r are formed once and serve both:
//   kind 0 (SL): x0 += wW' (f'/r + h (h.f') / r^3),  and the same with the roles
//                exchanged (h -> -h leaves it unchanged);
//   kind 1 (DL): x0 += -6 h (h.u') (h.wN') / r^5,    exchanged: +6 h (h.u) (h.wN) / r^5.
// Per interaction 18.5 FP64 instruction slots against 26 of k_pair (a DL pair:
// 15 shared with v_rsq_f64 as four, 11 per direction).
//
// Block: up to 1024 nodes of one drop (targets; four wavefronts, up to four per
// lane, in registers with their sums) against a run of nodes of the other
// (sources, in chunks of 64 through LDS). In a phase a row of 16 lanes holds 16
// sources, a different one per lane; from step to step lane i goes on to the
// next source and the sums of the sources move one lane down (DPP row
// rotation), so after 16 steps every source of the row has met every target of
// the row's lanes, with no cross-lane reduction and no atomics. Four phases
// pass the chunk's four groups of 16 round the four rows. The sums of a
// chunk's sources are added over the wavefronts in order: everything has a
// fixed order, and results are bit-identical from run to run.
//
// Bound: FP64 issue, at the clock the chip holds under it (counters of a double
// layer of 16 drops of degree 48, 5.0e9 interactions: the CUs issue 94 % of
// their cycles; 6.5e6 cycles in 3.3 ms, 1.95 GHz). Four targets per lane feed
// each LDS read (five 16-byte reads and the six 32-bit moves of the rotation)
// to four pairs; with them a lane holds 48 doubles, which leaves three
// wavefronts per SIMD. That launch: 3.3 ms against 4.1 for the same pairs in
// k_pair; the single layer's 3.1 against 3.9.
#include "gather.hpp"
#include "internal.hpp"

#include <hip/hip_runtime.h>

namespace bim {

constexpr int kMutRec = 10;  // doubles per source in LDS: x, density, weighted normal, pad (80 bytes: the 16
                             // lanes of a row reading consecutive records hit distinct banks)

// v of the next lane (cyclic in rows of 16 lanes)
__device__ inline double row_next(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x12F, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x12F, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// The targets of a lane and their sums.
struct MutTargets {
    double x[3][4], u[3][4], m[3][4], a[3][4];
};

// A chunk's 64 sources (rec, [4 groups][16 + 16 repeated][kMutRec]) against the
// first T targets of each lane; the wavefront's sums of the sources go to rv[64][3].
template <int KIND, int T>
__device__ inline void mutual_chunk(MutTargets &g, const double *rec, double *rv)
{
    const int lane = threadIdx.x & 63, i = lane & 15, row = lane >> 4;
#pragma unroll 1
    for (int ph = 0; ph < 4; ++ph) {
        const int grp = (row + ph) & 3;
        const double *s = rec + (grp * 32 + i) * kMutRec;
        double r0 = 0.0, r1 = 0.0, r2 = 0.0;
#pragma unroll 4
        for (int k = 0; k < 16; ++k, s += kMutRec) {
            const double2 e0 = *reinterpret_cast<const double2 *>(s), e1 = *reinterpret_cast<const double2 *>(s + 2),
                          e2 = *reinterpret_cast<const double2 *>(s + 4);
            double2 e3 = make_double2(0.0, 0.0);
            double e4 = 0.0;
            if (KIND == 1) {
                e3 = *reinterpret_cast<const double2 *>(s + 6);
                e4 = s[8];
            }
#pragma unroll
            for (int q = 0; q < T; ++q) {
                const double hx = g.x[0][q] - e0.x, hy = g.x[1][q] - e0.y, hz = g.x[2][q] - e1.x;
                const double d2 = fma(hz, hz, fma(hy, hy, hx * hx));
                const double y = __builtin_amdgcn_rsq(d2);
                const double hd = fma(hz, e2.y, fma(hy, e2.x, hx * e1.y));
                const double bd = fma(hz, g.u[2][q], fma(hy, g.u[1][q], hx * g.u[0][q]));
                if (KIND == 0) {  // refinements of 1/r as in k_pair
                    const double e = fma(-d2 * y, y, 1.0);
                    const double ri = fma(y * e, 0.5, y), ri2 = ri * ri;
                    const double p = hd * ri2, b = bd * ri2;
                    g.a[0][q] = fma(ri, fma(hx, p, e1.y), g.a[0][q]);
                    g.a[1][q] = fma(ri, fma(hy, p, e2.x), g.a[1][q]);
                    g.a[2][q] = fma(ri, fma(hz, p, e2.y), g.a[2][q]);
                    r0 = fma(ri, fma(hx, b, g.u[0][q]), r0);
                    r1 = fma(ri, fma(hy, b, g.u[1][q]), r1);
                    r2 = fma(ri, fma(hz, b, g.u[2][q]), r2);
                } else {
                    const double z = y * y;
                    const double pw = (z * z) * (y * fma(d2, z, -1.4));  // -0.4 r^-5
                    const double hn = fma(hz, e4, fma(hy, e3.y, hx * e3.x));
                    const double bn = fma(hz, g.m[2][q], fma(hy, g.m[1][q], hx * g.m[0][q]));
                    const double p = (hd * hn) * pw, b = (bd * bn) * pw;
                    g.a[0][q] = fma(p, hx, g.a[0][q]);
                    g.a[1][q] = fma(p, hy, g.a[1][q]);
                    g.a[2][q] = fma(p, hz, g.a[2][q]);
                    r0 = fma(b, hx, r0);
                    r1 = fma(b, hy, r1);
                    r2 = fma(b, hz, r2);
                }
            }
            r0 = row_next(r0);
            r1 = row_next(r1);
            r2 = row_next(r2);
        }
        // 16 rotations: lane i has the sums of source i of the group again
        double *o = rv + (grp * 16 + i) * 3;
        o[0] = ph ? o[0] + r0 : r0;
        o[1] = ph ? o[1] + r1 : r1;
        o[2] = ph ? o[2] + r2 : r2;
    }
}

// Work items blockIdx.x: targets [t0, t0 + nt), nt <= 1024, sources [s0, s0 +
// ns), ns <= R, of the arrays x, d (density), wN, wW (component stride st).
// Partial block of an item, part + item (3 * 1024 + 3 R): the targets' sums
// [3][1024], then the sources' sums [3][R], each times its weight.
template <int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_mutual(
    const MutualWork *__restrict__ work, int R, const double *__restrict__ x, const double *__restrict__ d,
    const double *__restrict__ wN, const double *__restrict__ wW, long st, double *__restrict__ part)
{
    __shared__ double2 srec[2][4 * 32 * kMutRec / 2];
    __shared__ double srv[2][4][64 * 3];
    const MutualWork it = work[blockIdx.x];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // units of 64 targets, as even as they go over the wavefronts
    const int units = (it.nt + 63) / 64, T = units / 4 + (w < units % 4), u0 = w * (units / 4) + min(w, units % 4);
    const int act = min(4, units);
    MutTargets g;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int a = 64 * (u0 + q) + lane;
        const bool in = q < T && a < it.nt;
        const long t = it.t0 + min(a, it.nt - 1);  // surplus lanes repeat the last target with no density
        const double f = in ? (KIND == 0 ? wW[t] : 1.0) : 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            g.x[c][q] = x[c * st + t];
            g.u[c][q] = f * d[c * st + t];
            g.m[c][q] = KIND == 1 ? wN[c * st + t] : 0.0;
            g.a[c][q] = 0.0;
        }
    }
    // a chunk's records: wavefront w loads source `lane` of components w, w + 4, w + 8
    double v[3];
    auto load = [&](int c0) {
        const bool in = c0 + lane < it.ns;
        const long s = it.s0 + min(c0 + lane, it.ns - 1);  // padding: the last source with no density
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int a = w + 4 * q;  // 0..2 position, 3..5 density, 6..8 normal
            v[q] = 0.0;
            if (a < 3)
                v[q] = x[a * st + s];
            else if (a < 6)
                v[q] = in ? (KIND == 0 ? wW[s] : 1.0) * d[(a - 3) * st + s] : 0.0;
            else if (a < 9 && KIND == 1)
                v[q] = in ? wN[(a - 6) * st + s] : 0.0;
        }
    };
    auto store = [&](int b) {
        double *r = reinterpret_cast<double *>(srec[b]) + ((lane >> 4) * 32 + (lane & 15)) * kMutRec;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int a = w + 4 * q;
            if (a < 9) r[a] = r[16 * kMutRec + a] = v[q];
        }
    };
    load(0);
    store(0);
    __syncthreads();
    double *out = part + (long)blockIdx.x * (3 * kMutTargets + 3 * (long)R);
    for (int c0 = 0, b = 0; c0 < it.ns; c0 += 64, b ^= 1) {
        const bool more = c0 + 64 < it.ns;
        if (more) load(c0 + 64);
        const double *rec = reinterpret_cast<const double *>(srec[b]);
        switch (T) {
        case 4: mutual_chunk<KIND, 4>(g, rec, srv[b][w]); break;
        case 3: mutual_chunk<KIND, 3>(g, rec, srv[b][w]); break;
        case 2: mutual_chunk<KIND, 2>(g, rec, srv[b][w]); break;
        case 1: mutual_chunk<KIND, 1>(g, rec, srv[b][w]); break;
        default: break;
        }
        if (more) store(b ^ 1);
        __syncthreads();
        // this chunk's source sums over the wavefronts, in order (the buffers
        // are written again only after the next barrier)
        if (threadIdx.x < 192) {
            const int c = w;
            if (c0 + lane < it.ns) {
                double s = 0.0;
                for (int k = 0; k < act; ++k) s += srv[b][k][3 * lane + c];
                out[3 * kMutTargets + (long)c * R + c0 + lane] = (KIND == 0 ? it.ws : -15.0 * it.ws) * s;
            }
        }
    }
    const double sw = KIND == 0 ? it.wt : 15.0 * it.wt;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q < T)
#pragma unroll
            for (int c = 0; c < 3; ++c) out[c * kMutTargets + 64 * (u0 + q) + lane] = sw * g.a[c][q];
}

// out[c][t] += the sums of the mutual items of target t, in a fixed order: the
// slots of its block of targets, then those of its run of sources (gather.hpp).
// Targets with no slot are left alone.
__global__ __launch_bounds__(256) void k_mutual_gather(int nt, MutualGather mg, const double *__restrict__ part,
                                                       double *__restrict__ out, long ostride)
{
    const int t = blockIdx.x * kGatherTargets + (threadIdx.x & 15), tc = min(t, nt - 1);
    const int a = mg.tb[tc], b = mg.sr[tc];
    const int a0 = mg.toff[a], a1 = mg.toff[a + 1], b0 = mg.soff[b], b1 = mg.soff[b + 1];
    double s[3] = {0.0, 0.0, 0.0};
    gather_slots(s, mg.tent, a0, a1, tc, part, kMutTargets);
    gather_slots(s, mg.sent, b0, b1, tc, part, mg.R);
    const double v = gather_groups(s);
    if (threadIdx.x >= 3 * kGatherTargets || t >= nt || (a0 == a1 && b0 == b1)) return;
    out[(threadIdx.x >> 4) * ostride + t] += v;
}

void launch_mutual_gather(hipStream_t st, int nt, const MutualGather &mg, const double *part, double *out, long ostride)
{
    if (nt <= 0) return;
    hipLaunchKernelGGL(k_mutual_gather, dim3((nt + kGatherTargets - 1) / kGatherTargets), dim3(256), 0, st, nt, mg, part,
                       out, ostride);
}

void launch_mutual(hipStream_t st, int kind, int n, const MutualWork *work, int R, const PairSrc &g, double *part)
{
    if (n <= 0) return;
    if (kind == 0)
        hipLaunchKernelGGL(k_mutual<0>, dim3(n), dim3(256), 0, st, work, R, g.x, g.d, g.wN, g.wW, g.stride, part);
    else
        hipLaunchKernelGGL(k_mutual<1>, dim3(n), dim3(256), 0, st, work, R, g.x, g.d, g.wN, g.wW, g.stride, part);
}

}  // namespace bim
