// Sums of the partial results of pair items per target (gfx950, FP64), shared
// by k_pair_gather and k_mutual_gather.
//
// Block of 256: 16 consecutive targets (a slot's values of neighbouring targets
// are neighbours: 128-byte reads) times 16 groups of list entries, four entries
// in flight per lane. Group g adds entries g, g + 16, .. of the target's lists in
// turn, the groups are added in a fixed order: the sums do not depend on
// scheduling. Bound by the read of the slots; one wavefront per target, which
// reads eight bytes of each line a slot touches, took 72 us for the operator of 64
// drops on the 2x grid and 81 us for the mutual items of 16 drops of degree 48;
// so 17 and 23 (two drops of degree 32, 64 sources an item: 11.5 and 10.0).
#pragma once
#include <hip/hip_runtime.h>

namespace bim {

constexpr int kGatherTargets = 16;

// Adds part[ent[e] + shift + c stride] over this thread's share of e0 <= e < e1.
__device__ inline void gather_slots(double (&s)[3], const int *__restrict__ ent, int e0, int e1, long shift,
                                    const double *__restrict__ part, long stride)
{
    const int g = threadIdx.x >> 4;
    for (int e = e0 + g; e < e1; e += 64) {
        double v[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double *p = part + ((long)ent[min(e + 16 * u, e1 - 1)] + shift);
            v[u][0] = p[0];
            v[u][1] = p[stride];
            v[u][2] = p[2 * stride];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 3; ++c) s[c] += e + 16 * u < e1 ? v[u][c] : 0.0;
    }
}

// The 16 groups' sums: thread 16 c + i (c < 3) returns component c of target i.
__device__ inline double gather_groups(double (&s)[3])
{
    __shared__ double red[4][3][kGatherTargets];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        s[c] += __shfl_xor(s[c], 16, 64);
        s[c] += __shfl_xor(s[c], 32, 64);
        if (lane < 16) red[w][c][lane] = s[c];
    }
    __syncthreads();
    const int c = min((int)threadIdx.x >> 4, 2), i = threadIdx.x & 15;
    return (red[0][c][i] + red[1][c][i]) + (red[2][c][i] + red[3][c][i]);
}

}  // namespace bim
