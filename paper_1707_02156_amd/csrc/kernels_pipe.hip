// Singular self-integral as a batched pipeline over all grid targets of a drop
// (gfx950, FP64). Same quadrature as the fused kernel (Sec. 2.2, Theorem 1,
// Appendix B), reorganised so the Legendre stages are dense contractions on
// the matrix cores:
//
//   R  k_rot_mfma  rotation of x (and the single-layer density) for every
//                  target of a latitude, per degree n (Appendix B, gamma = 0), as
//                  GEMMs on the matrix cores; output by order mu:
//                  B^mu[n - mu][col], col = target*6 + comp*2 + re/im
//   L  k_leg_mfma  G^mu = T^mu B^mu on v_mfma_f64_16x16x4f64, T^mu the Legendre
//                  rows [Ptilde_n^mu(t_j'); dPtilde_n^mu/dtheta(t_j')] of the rotated grid
//   FK k_fk        Fourier sums at the rotated longitudes (symmetries phi -> -phi,
//                  phi -> phi + pi), the pole-rule kernels, per-latitude partial sums;
//                  for the double layer the six stresslet fields and their Fourier
//                  analysis Fa^mu[j'][target*12 + pair*2 + re/im]
//   LA k_leg_mfma  Legendre analysis Bt^mu = (Ptilde^mu)^T Fa^mu (same kernel)
//   AR k_adjrot_mfma adjoint rotation (matrix cores) -> rows of the stored double layer
//                  M[t][pair][2 ncoef(p)] (applied by dl_row, dl_row.hpp)
//
// Layouts: a triangle-ordered operand stores order mu as the rows n = mu..p at
// row offset koff(mu) = mu (p+1) - mu (mu-1)/2, each row NC doubles wide.
#include "internal.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

namespace bim {

typedef double d4_t __attribute__((ext_vector_type(4)));

__host__ __device__ inline long koff(int mu, int P1) { return (long)mu * P1 - (long)mu * (mu - 1) / 2; }

// ----------------------------------------------------------------------------
// R: rotation on the matrix cores. Block (n, latitude j), 256 threads. For the
// 2p targets k of latitude j and the nf fields f (x, then the density):
//   Re f'^mu_n(k, f) = sum_nu A+_{nu mu} Re g^nu,  Im f'^mu_n = sum_nu A-_{nu mu} Im g^nu,
//   g^nu = e^{i nu phi_k} c^nu_{n,f},
// two GEMMs (mu x nu) x (nu x col), col = k nf + f, on v_mfma_f64_16x16x4f64:
// A = A+/- from LDS (zero padded to a multiple of 16), B = g formed in
// registers per lane, one 16-column tile per wavefront at a time.
// Output by order mu: B^mu[koff(mu) + n - mu][t*6 + comp*2 + re/im].
// ----------------------------------------------------------------------------
// Stage the N1 x N1 blocks of A+ and A- at lat into LDS ([nu][mu], NP x NP,
// zero padded, row stride NS), the loads of four rounds issued before their
// stores.
__device__ inline void stage_rot(const double *__restrict__ Ap, const double *__restrict__ Am, size_t lat, int N1,
                                 int NP, int NS, double *sAp, double *sAm)
{
    for (int i0 = threadIdx.x; i0 < NP * NP; i0 += 1024) {
        double a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 256 * u, nu = i / NP, mu = i % NP;
            const bool in = i < NP * NP && nu < N1 && mu < N1;
            a[u] = in ? Ap[lat + nu * N1 + mu] : 0.0;
            b[u] = in ? Am[lat + nu * N1 + mu] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 256 * u;
            if (i < NP * NP) {
                const int nu = i / NP, mu = i % NP;
                sAp[nu * NS + mu] = a[u];
                sAm[nu * NS + mu] = b[u];
            }
        }
    }
}

constexpr int kRotMaxPad = 64;  // degree p <= 63

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_rot_mfma(int p, const double *__restrict__ Ap, const double *__restrict__ Am,
                                                  const double *__restrict__ csp, const double *__restrict__ xc0,
                                                  long xstride, const double *__restrict__ dc0, long dstride,
                                                  PipeDrops pd, int u0, double *__restrict__ Bx,
                                                  double *__restrict__ Bd, long NC)
{
    extern __shared__ double sm[];
    const int ug = u0 + blockIdx.y, dr = ug / (p + 1);
    const int n = blockIdx.x, j = ug % (p + 1);
    const double *xc = xc0 + pd.coff[dr];
    const double *dc = dc0 ? dc0 + pd.coff[dr] : nullptr;
    const int N1 = n + 1, nk = 2 * p, P1 = p + 1;
    const int nf = dc ? 6 : 3;
    const int MT = (N1 + 15) / 16, NP = MT * 16, NS = NP + 1, KS = (N1 + 3) / 4;
    double *sAp = sm;                  // [nu][mu], NP x NP, zero padded, row stride NS
    double *sAm = sAp + NP * NS;
    double *sC = sAm + NP * NS;        // [f][nu][re,im]
    double *sCS = sC + nf * N1 * 2;    // cos, sin of the target longitudes [2][nk]
    const size_t lat = rot_lat_size(p) * j + rot_off(n);
    stage_rot(Ap, Am, lat, N1, NP, NS, sAp, sAm);
    const int b0 = n * (n + 1) / 2;
    for (int i = threadIdx.x; i < nf * N1; i += 256) {
        const int f = i / N1, nu = i % N1;
        const double *c = (f < 3) ? xc + f * xstride : dc + (f - 3) * dstride;
        sC[2 * i] = c[2 * (b0 + nu)];
        sC[2 * i + 1] = c[2 * (b0 + nu) + 1];
    }
    for (int i = threadIdx.x; i < 2 * nk; i += 256) sCS[i] = csp[i];
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r16 = lane & 15, k4 = lane >> 4;
    const int ncol = nk * nf, NT = (ncol + 15) / 16;
    for (int nt = wv; nt < NT; nt += 4) {
        const int col = nt * 16 + r16;
        const bool cok = col < ncol;
        const int k = cok ? col / nf : 0, f = cok ? col % nf : 0;
        const double *cf = sC + 2 * f * N1;
        d4_t ap[4], am[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) ap[m] = am[m] = (d4_t){0, 0, 0, 0};
        // e = nu k mod nk, stepped by 4k as nu advances by 4
        int e = (k4 * k) % nk;
        const int step = (4 * k) % nk;
        for (int ks = 0; ks < KS; ++ks) {
            const int nu = ks * 4 + k4;
            double gr = 0.0, gi = 0.0;
            if (cok && nu < N1) {
                const double cr = cf[2 * nu], ci = cf[2 * nu + 1];
                const double cs = sCS[e], sn = sCS[nk + e];
                gr = cr * cs - ci * sn;
                gi = fma(cr, sn, ci * cs);
            }
            e += step;
            if (e >= nk) e -= nk;
            const double *pa = sAp + nu * NS + r16, *pm = sAm + nu * NS + r16;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (m < MT) {
                    ap[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[m * 16], gr, ap[m], 0, 0, 0);
                    am[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(pm[m * 16], gi, am[m], 0, 0, 0);
                }
        }
        if (!cok) continue;
        const int t = blockIdx.y * nk + k;
        double *dst = (f < 3) ? Bx : Bd;
        const int ff = f < 3 ? f : f - 3;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m < MT)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int mu = m * 16 + 4 * v + k4;
                    if (mu <= n) {
                        double *o = dst + (koff(mu, P1) + (n - mu)) * NC + (long)t * 6 + ff * 2;
                        o[0] = ap[m][v];
                        o[1] = am[m][v];
                    }
                }
    }
}

// ----------------------------------------------------------------------------
// L / LA: batched contraction on the matrix cores.
//   OUT^b[r][col] = sum_k TAB^b[r][k] IN^b[k][col],  b = 0..nb-1,
// with per-batch rows R_b, depth K_b and row offsets; TAB^b row-major R_b x K_b
// at tab_off[b]. Block: all rows of one batch x 64 columns (4 wavefronts x 16).
// ----------------------------------------------------------------------------
struct LegBatch {
    int R, K;          // rows, depth
    long tab_off;      // TAB offset (doubles)
    long in_row;       // first IN row
    long out_row;      // first OUT row
};

template <int MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_leg_mfma(const LegBatch *__restrict__ bt, const double *__restrict__ tab,
                                                  const double *__restrict__ in, double *__restrict__ out, long NC)
{
    __shared__ double sT[MT * 16 * 53];   // rows padded to MT*16, depth padded to 4 (up to 52), odd row stride
    const LegBatch b = bt[blockIdx.y];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long col = (long)blockIdx.x * 64 + wv * 16 + (lane & 15);
    const bool cok = col < NC;
    const int Kp = (b.K + 3) & ~3, Ks = Kp + 1;
    const int kl = lane >> 4;
    // every B value of the lane loaded before the first product (13 depth
    // steps at most): one memory latency per block instead of one per step
    constexpr int KS = 13;
    double bv[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 4 * s + kl;
        bv[s] = (cok && k < b.K) ? in[(b.in_row + k) * NC + col] : 0.0;
    }
    // stage the table block, zero padded: sT[r][k], r < MT*16, k < Kp, row
    // stride Ks; the loads of eight rounds issued before their stores
    for (int i0 = threadIdx.x; i0 < MT * 16 * Kp; i0 += 8 * 256) {
        double tv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + 256 * u, r = i / Kp, k = i % Kp;
            tv[u] = (i < MT * 16 * Kp && r < b.R && k < b.K) ? tab[b.tab_off + (long)r * b.K + k] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + 256 * u;
            if (i < MT * 16 * Kp) sT[(i / Kp) * Ks + i % Kp] = tv[u];
        }
    }
    __syncthreads();
    d4_t acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = (d4_t){0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        if (4 * s >= Kp) break;
        const int k = 4 * s + kl;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const double av = sT[(m * 16 + (lane & 15)) * Ks + k];
            acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[s], acc[m], 0, 0, 0);
        }
    }
    if (!cok) return;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = m * 16 + 4 * v + kl;
            if (r < b.R) out[(b.out_row + r) * NC + col] = acc[m][v];
        }
}

// ----------------------------------------------------------------------------
// FK: Fourier sums and kernels. Item: 16 consecutive targets x one rotated
// latitude j'. Gx rows: j' (Ptilde) and Q1 + j' (d/dtheta); Gd row j'.
// SL: partial[t][j'][3] += omega W (f/r + xh (xh.f)/r^3) summed over the longitudes.
// DL: Fa^mu[j'][t*12 + pair*2 + {cos, sin}] of the six stresslet fields.
//
// The Fourier sums are contractions on v_mfma_f64_4x4x4 (four blocks of 4x4x4:
// 4 rows x 16 columns x depth 4) with the symmetries of the longitudes folded in: with the even and odd
// orders and the cosine and sine sums apart, row kk <= qs/2 gives the points
// kk, kk + qs, -kk and qs - kk, a quarter of the plain product's work. Columns
// are the item's 16 targets, so the three components of x, x_theta, x_phi and
// f at a point meet in one lane, which evaluates the pole rule at its points
// and holds the folded stresslet values as operand rows of the analysis.
//
// A wavefront takes two row tiles, so that rows are padded to eights (9 of degree
// 16 to 16, 17 of degree 32 to 24, 25 of degree 48 to 32: an empty tile runs):
// each LDS read feeds both, and the 48 or 24 independent products of a step cover
// its latency (one tile per wavefront at
// four wavefronts per SIMD read twice as much and waited: 2.26 ms against 2.05
// at the size below). A block (2 to 4 wavefronts, 79 KB of LDS at p = 48, two
// per CU) walks over items; the slab of G that is summed next is on its way
// into the other LDS buffer by 16-byte direct loads meanwhile.
//
// Bound: the FP64 pipe, which the matrix instructions share with the vector
// ones (10000 of some 13500 cycles per wavefront and item are products), then
// HBM. One launch over 15053 targets of degree 48: single layer 3.67 -> 2.05 ms
// (loads alone 1.16 ms, 4.5 TB/s; sums alone 1.55 ms); both layers over 9408
// targets 3.36 -> 2.18 ms; against the thread-per-point recurrences before it.
// ----------------------------------------------------------------------------

// 1/sqrt(x) to full double precision: hardware estimate plus one third-order
// correction (relative error of the estimate e -> O(e^3))
__device__ inline double rsq_full(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

constexpr int kFkT = 16;        // targets per item
constexpr int kFkMaxWaves = 4;  // wavefronts per block (two row tiles each): qs <= 62

__host__ __device__ inline int fk_waves(int qs) { return (qs / 2 + 8) / 8; }      // of two tiles of 4 rows kk = 0..qs/2
__host__ __device__ inline int fk_order_steps(int p) { return (p / 2 + 4) / 4; }  // of 4 even and 4 odd orders

// LDS of a block, in doubles: cos and sin of pi e / qs, two buffers (each a
// slab of G or a third of the analysis operand, whichever is larger), the
// pole values of the item's targets, the single layer's sums per wavefront.
__host__ __device__ inline int fk_buf(int p, int qs, bool dl)
{
    const int slab = (p + 1) * kFkT * 6, third = dl ? fk_waves(qs) * 8 * 2 * kFkT * 4 : 0;
    return slab > third ? slab : third;
}

// threadIdx.x that the compiler takes for a new value at each call: what is
// derived from it is formed again where it is used instead of held in
// registers over the kernel's loop (no register is left at four wavefronts per
// SIMD, and a spill's reload would wait for the direct loads in flight).
__device__ inline int fk_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// x mod n for 0 <= x < 2^12, 4 <= n < 2^7 (rn = 2^20 / n + 1)
__device__ inline int fk_mod(int x, int n, int rn) { return x - (x * rn >> 20) * n; }

// One 16-byte direct load per active lane: lane l's 16 bytes at g go to LDS at
// dst + 16 l. Written out because the compiler would wait for every direct
// load before any later LDS read; it has no result register, and fk_staged
// waits for it.
__device__ inline void fk_load_lds(const double *g, const double *dst)
{
    const unsigned at = __builtin_amdgcn_readfirstlane(
        (unsigned)(unsigned long)(const __attribute__((address_space(3))) double *)dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(g) : "m0", "memory");
}

// Rows src[mu * ld] (mu <= p), the 96 doubles of 16 targets from t0 on
// (targets past the last one repeat it), into the LDS slab [mu][16][6] by
// direct loads: a row is one instruction of 48 lanes.
__device__ inline void fk_stage(const double *__restrict__ src, long ld, int P1, int t0, int nt, int w, int nw,
                                double *slab)
{
    const int lane = fk_tid() & 63;
    if (lane < 48) {
        const double *g = src + (min(t0 + lane / 3, nt - 1) * 6 + lane % 3 * 2) + w * ld;
        for (int mu = w; mu < P1; mu += nw, g += nw * ld) fk_load_lds(g, slab + mu * kFkT * 6);
    }
}

// the direct loads of this wavefront are in LDS, then those of the whole block
__device__ inline void fk_staged()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// all but the last n direct loads of this wavefront are in LDS (0 <= n <= 16),
// then those of the whole block
__device__ inline void fk_staged_but(int n)
{
    switch (n) {
#define FK_WAIT(k) case k: asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory"); break;
        FK_WAIT(1) FK_WAIT(2) FK_WAIT(3) FK_WAIT(4) FK_WAIT(5) FK_WAIT(6) FK_WAIT(7) FK_WAIT(8)
        FK_WAIT(9) FK_WAIT(10) FK_WAIT(11) FK_WAIT(12) FK_WAIT(13) FK_WAIT(14) FK_WAIT(15) FK_WAIT(16)
#undef FK_WAIT
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
}

// Cosine and sine sums over the even and odd orders of three components, for
// the row tiles u = 0, 1 of wavefront w: C[u][c][0], C[u][c][1] the cosine sums
// of the even and odd orders, C[u][c][2], C[u][c][3] the sine sums, at row kk =
// 8w + 4u + lane / 16 and target lane % 16; PHI: also those of the derivative
// in phi, (i mu) g, in D. The table operand (rows 8w + 4u + lane % 4, orders 8s
// + 2 (lane / 16) and the next) starts from the LDS table cs (nk entries) and
// turns by eight orders from step to step.
template <bool PHI>
__device__ inline void fk_sums(int p, int KS, int w, const double2 *cs, int nk, int rn, const double *slab,
                               double (&C)[2][3][4], double (&D)[2][3][4])
{
    const int lane = fk_tid() & 63, t = lane & 15, k4 = lane >> 4;
    double ce[2], se[2], co[2], so[2], c8[2], s8[2], fm = 2.0 * k4;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int ka = 8 * w + 4 * u + (lane & 3);
        const double2 te = cs[fk_mod(2 * k4 * ka, nk, rn)], to = cs[fk_mod((2 * k4 + 1) * ka, nk, rn)],
                      t8 = cs[fk_mod(8 * ka, nk, rn)];
        ce[u] = 2.0 * te.x;
        se[u] = 2.0 * te.y;
        co[u] = 2.0 * to.x;
        so[u] = 2.0 * to.y;
        c8[u] = t8.x;
        s8[u] = t8.y;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                C[u][c][q] = 0.0;
                if (PHI) D[u][c][q] = 0.0;
            }
    }
    // the sums of component c over one step's even (e) and odd (o) orders
    auto add = [&](int c, double2 e, double2 o, const double *ae, const double *be, const double *ao, const double *bo,
                   const double *pae, const double *pbe, const double *pao, const double *pbo, bool odd) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            C[u][c][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(ae[u], e.x, C[u][c][0], 0, 0, 0);
            C[u][c][2] = __builtin_amdgcn_mfma_f64_4x4x4f64(be[u], e.y, C[u][c][2], 0, 0, 0);
            if (PHI) {
                D[u][c][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(pae[u], e.y, D[u][c][0], 0, 0, 0);
                D[u][c][2] = __builtin_amdgcn_mfma_f64_4x4x4f64(pbe[u], e.x, D[u][c][2], 0, 0, 0);
            }
        }
        if (odd)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                C[u][c][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(ao[u], o.x, C[u][c][1], 0, 0, 0);
                C[u][c][3] = __builtin_amdgcn_mfma_f64_4x4x4f64(bo[u], o.y, C[u][c][3], 0, 0, 0);
                if (PHI) {
                    D[u][c][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(pao[u], o.y, D[u][c][1], 0, 0, 0);
                    D[u][c][3] = __builtin_amdgcn_mfma_f64_4x4x4f64(pbo[u], o.x, D[u][c][3], 0, 0, 0);
                }
            }
    };
    const double *g = slab + (2 * k4 * kFkT + t) * 6, *z = slab + t * 6;
    // the last step's orders may lie past p: their table entries are zeroed,
    // their operand is any row of the slab
    const int le = 8 * (KS - 1) + 2 * k4;
    const bool ve = le <= p, vo = le < p;
    // a component's operands of the next step are read as soon as this step's
    // are consumed: a whole step of products covers the LDS latency
    double2 e[3], o[3];
    {
        const double *ge = KS > 1 || ve ? g : z, *go = KS > 1 || vo ? g + kFkT * 6 : z;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            e[c] = *reinterpret_cast<const double2 *>(ge + 2 * c);
            o[c] = *reinterpret_cast<const double2 *>(go + 2 * c);
        }
    }
    double pae[2], pbe[2], pao[2], pbo[2];
#pragma unroll 1
    for (int s = 1; s < KS; ++s) {
        const double *n = g + 8 * kFkT * 6;
        const double *ne = s + 1 < KS || ve ? n : z, *no = s + 1 < KS || vo ? n + kFkT * 6 : z;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            pae[u] = -fm * ce[u];
            pbe[u] = fm * se[u];
            pao[u] = -(fm + 1.0) * co[u];
            pbo[u] = (fm + 1.0) * so[u];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            add(c, e[c], o[c], ce, se, co, so, pae, pbe, pao, pbo, true);
            __builtin_amdgcn_sched_barrier(0);
            e[c] = *reinterpret_cast<const double2 *>(ne + 2 * c);
            o[c] = *reinterpret_cast<const double2 *>(no + 2 * c);
            __builtin_amdgcn_sched_barrier(0);
        }
        g = n;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double xe = fma(ce[u], c8[u], -(se[u] * s8[u])), xo = fma(co[u], c8[u], -(so[u] * s8[u]));
            se[u] = fma(se[u], c8[u], ce[u] * s8[u]);
            so[u] = fma(so[u], c8[u], co[u] * s8[u]);
            ce[u] = xe;
            co[u] = xo;
        }
        if (PHI) fm += 8.0;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ce[u] = ve ? ce[u] : 0.0;
        se[u] = ve ? se[u] : 0.0;
        co[u] = vo ? co[u] : 0.0;
        so[u] = vo ? so[u] : 0.0;
        pae[u] = -fm * ce[u];
        pbe[u] = fm * se[u];
        pao[u] = -(fm + 1.0) * co[u];
        pbo[u] = (fm + 1.0) * so[u];
    }
    const bool odd = 8 * (KS - 1) < p;  // an odd order is left (uniform)
#pragma unroll
    for (int c = 0; c < 3; ++c) add(c, e[c], o[c], ce, se, co, so, pae, pbe, pao, pbo, odd);
    // order 0 counts once
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int u = 0; u < 2; ++u) C[u][c][0] -= z[2 * c];
}

// The sums of one component to its values at the points kk, kk + qs, -kk and
// qs - kk: the odd orders change sign from phi to phi + pi, the sine sums from
// phi to -phi.
__device__ inline void fk_points(double (&C)[4])
{
    const double em = C[0] - C[2], om = C[1] - C[3], ep = C[0] + C[2], op = C[1] + C[3];
    C[0] = em + om;
    C[1] = em - om;
    C[2] = ep + op;
    C[3] = ep - op;
}

template <bool SL, bool DL>
__global__ __launch_bounds__(64 * kFkMaxWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_fk(
    int p, int qs, int nt, int ntb, const double *__restrict__ Gx, const double *__restrict__ Gd, long NC6,
    const double *__restrict__ wsing, const double *__restrict__ cst, const double *__restrict__ X0,
    double *__restrict__ part, double *__restrict__ Fa, long NC12)
{
    extern __shared__ double sm[];
    const int P1 = p + 1, Q1 = qs + 1, nk = 2 * qs, KS = fk_order_steps(p), rn = (1 << 20) / nk + 1;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    double2 *cs = reinterpret_cast<double2 *>(sm);
    double *bA = sm + 2 * nk, *bB = bA + fk_buf(p, qs, DL), *x0 = bB + fk_buf(p, qs, DL), *red = x0 + 3 * kFkT;
    for (int e = threadIdx.x; e < nk; e += blockDim.x) cs[e] = make_double2(cst[e], cst[nk + e]);
    const long ldx = 2L * Q1 * NC6, ldd = (long)Q1 * NC6;
    // pole values of 16 targets from t0 on (3 nt is even; values past the last
    // target are not used)
    auto stage_pole = [&](int t0) {
        const int lane = fk_tid() & 63;
        if (w == 0 && lane < 24) fk_load_lds(X0 + min(t0 * 3 + 2 * lane, 3 * nt - 2), x0);
    };
    int item = blockIdx.x;
    __syncthreads();  // cs (its loads come before the direct loads in the count of fk_staged_but)
    fk_stage(Gx + item / ntb * NC6, ldx, P1, item % ntb * kFkT, nt, w, nw, bA);
    stage_pole(item % ntb * kFkT);
    fk_stage(Gx + (Q1 + item / ntb) * NC6, ldx, P1, item % ntb * kFkT, nt, w, nw, bB);
    const int ntot = ntb * Q1, nrow = (P1 - w + nw - 1) / nw;  // rows of a slab this wavefront loads
    while (true) {
        const int jr = item / ntb, t0 = item % ntb * kFkT;
        const int next = item + gridDim.x, tn = next % ntb * kFkT;
        const bool more = next < ntot;
        // every slab is loaded while the one before it is summed
        fk_staged_but(nrow);  // x in bA (x_theta still on its way to bB)
        double x[2][3][4], N[2][3][4], xt[2][3][4];
        fk_sums<true>(p, KS, w, cs, nk, rn, bA, x, N);
        fk_staged();  // x_theta in bB, every wavefront through with x
        if (SL)
            fk_stage(Gd + jr * NC6, ldd, P1, t0, nt, w, nw, bA);
        else if (more)
            fk_stage(Gx + next / ntb * NC6, ldx, P1, tn, nt, w, nw, bA);
        fk_sums<false>(p, KS, w, cs, nk, rn, bB, xt, xt);
        // the pole rule up to the density: unit vectors h / r (in x), the single
        // layer's weight omega |N| / r (Wr) and the stresslet's -6 omega (h.N) / r^3
        // (sc) at this lane's points kk, kk + qs (which exist once on every row kk
        // <= qs / 2) and -kk, qs - kk (except on the rows of phi = 0 and pi / 2)
        const double om = wsing[jr];
        double Wr[2][4], sc[2][4];
        {
            const int lane = fk_tid() & 63, t = lane & 15;
            const double X[3] = {x0[3 * t], x0[3 * t + 1], x0[3 * t + 2]};
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int kk = 8 * w + 4 * u + (lane >> 4);
                const bool one = kk <= qs / 2, two = one && kk != 0 && 2 * kk != qs;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    fk_points(N[u][c]);
                    fk_points(xt[u][c]);
                    fk_points(x[u][c]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) x[u][c][q] = X[c] - x[u][c][q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool ok = q < 2 ? one : two;
                    double(&h)[3][4] = x[u];
                    const double n0 = xt[u][1][q] * N[u][2][q] - xt[u][2][q] * N[u][1][q];
                    const double n1 = xt[u][2][q] * N[u][0][q] - xt[u][0][q] * N[u][2][q];
                    const double n2 = xt[u][0][q] * N[u][1][q] - xt[u][1][q] * N[u][0][q];
                    const double r2 = h[0][q] * h[0][q] + h[1][q] * h[1][q] + h[2][q] * h[2][q];
                    const double ri = rsq_full(r2);
#pragma unroll
                    for (int c = 0; c < 3; ++c) h[c][q] *= ri;
                    if (SL) {
                        const double nn = n0 * n0 + n1 * n1 + n2 * n2;
                        const double W = om * (nn * rsq_full(nn)) * ri;
                        Wr[u][q] = ok ? W : 0.0;
                    }
                    if (DL) {
                        const double hn = h[0][q] * n0 + h[1][q] * n1 + h[2][q] * n2;
                        const double sv = -6.0 * om * hn * (ri * ri);
                        sc[u][q] = ok ? sv : 0.0;
                    }
                    // formed here, not after the sums of f, so that x_theta and
                    // x_phi are not held over them
#pragma unroll
                    for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(h[c][q]));
                    if (SL) asm volatile("" : "+v"(Wr[u][q]));
                    if (DL) asm volatile("" : "+v"(sc[u][q]));
                }
            }
        }
        if (SL)
            fk_staged();  // f in bA, every wavefront through with x_theta
        else
            __syncthreads();
        if (SL) {
            if (more) fk_stage(Gx + next / ntb * NC6, ldx, P1, tn, nt, w, nw, bB);
            double f[2][3][4];
            fk_sums<false>(p, KS, w, cs, nk, rn, bA, f, f);
            double e0 = 0.0, e1 = 0.0, e2 = 0.0;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int c = 0; c < 3; ++c) fk_points(f[u][c]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double hf = x[u][0][q] * f[u][0][q] + x[u][1][q] * f[u][1][q] + x[u][2][q] * f[u][2][q];
                    e0 = fma(Wr[u][q], fma(x[u][0][q], hf, f[u][0][q]), e0);
                    e1 = fma(Wr[u][q], fma(x[u][1][q], hf, f[u][1][q]), e1);
                    e2 = fma(Wr[u][q], fma(x[u][2][q], hf, f[u][2][q]), e2);
                }
            }
            // sums over the longitudes in a fixed order: the tiles' rows by a
            // butterfly, the wavefronts in turn
            const int lane = fk_tid() & 63, t = lane & 15;
            e0 += __shfl_xor(e0, 16, 64);
            e1 += __shfl_xor(e1, 16, 64);
            e2 += __shfl_xor(e2, 16, 64);
            e0 += __shfl_xor(e0, 32, 64);
            e1 += __shfl_xor(e1, 32, 64);
            e2 += __shfl_xor(e2, 32, 64);
            if (lane < kFkT) {
                red[(w * kFkT + t) * 3] = e0;
                red[(w * kFkT + t) * 3 + 1] = e1;
                red[(w * kFkT + t) * 3 + 2] = e2;
            }
        }
        if (DL) {
            const int lane = fk_tid() & 63, t = lane & 15, k4 = lane >> 4;
            // the analysis operand of two fields at a time, in the buffer that
            // the next item's x_theta (SL: this item's f) leaves free
            double2 *vA = reinterpret_cast<double2 *>(SL ? bA : bB), *vB = vA + nw * 8 * 2 * kFkT;
#pragma unroll
            for (int third = 0; third < 3; ++third) {
                __syncthreads();  // the buffer's last contents are read
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        // pairs (0,0) (0,1) (0,2) (1,1) (1,2) (2,2)
                        constexpr int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
                        const int a = pa[2 * third + f], b = pb[2 * third + f];
                        const double k0 = sc[u][0] * x[u][a][0] * x[u][b][0], k1 = sc[u][1] * x[u][a][1] * x[u][b][1];
                        const double k2 = sc[u][2] * x[u][a][2] * x[u][b][2], k3 = sc[u][3] * x[u][a][3] * x[u][b][3];
                        const int at = ((8 * w + 4 * u + k4) * 2 + f) * kFkT + t;
                        vA[at] = make_double2((k0 + k2) + (k1 + k3), (k0 + k2) - (k1 + k3));  // cosine: even, odd orders
                        vB[at] = make_double2((k0 - k2) + (k1 - k3), (k0 - k2) - (k1 - k3));  // sine
                    }
                __syncthreads();
                if (16 * w <= p) {
                    // table operand: rows the orders 2 ka and 2 ka + 1, ka = 8w + 4u +
                    // lane % 4, depth kk = 4s + lane / 16, turned from step to step
                    double F[2][2][4], ce[2], se[2], co[2], so[2];
                    double2 de[2], dd[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int ka = 8 * w + 4 * u + (lane & 3);
                        const double2 te = cs[fk_mod(2 * ka * k4, nk, rn)], to = cs[fk_mod((2 * ka + 1) * k4, nk, rn)];
                        de[u] = cs[fk_mod(8 * ka, nk, rn)];
                        dd[u] = cs[fk_mod(8 * ka + 4, nk, rn)];
                        ce[u] = te.x;
                        se[u] = te.y;
                        co[u] = to.x;
                        so[u] = to.y;
#pragma unroll
                        for (int f = 0; f < 2; ++f)
#pragma unroll
                            for (int q = 0; q < 4; ++q) F[u][f][q] = 0.0;
                    }
                    const int steps = qs / 8 + 1;  // rows kk <= qs / 2 by fours
                    for (int s = 0; s < steps; ++s) {
#pragma unroll
                        for (int f = 0; f < 2; ++f) {
                            const int at = ((4 * s + k4) * 2 + f) * kFkT + t;
                            const double2 a = vA[at], b = vB[at];
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                F[u][f][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(ce[u], a.x, F[u][f][0], 0, 0, 0);
                                F[u][f][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(co[u], a.y, F[u][f][1], 0, 0, 0);
                                F[u][f][2] = __builtin_amdgcn_mfma_f64_4x4x4f64(se[u], b.x, F[u][f][2], 0, 0, 0);
                                F[u][f][3] = __builtin_amdgcn_mfma_f64_4x4x4f64(so[u], b.y, F[u][f][3], 0, 0, 0);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const double xe = fma(ce[u], de[u].x, -(se[u] * de[u].y));
                            const double xo = fma(co[u], dd[u].x, -(so[u] * dd[u].y));
                            se[u] = fma(se[u], de[u].x, ce[u] * de[u].y);
                            so[u] = fma(so[u], dd[u].x, co[u] * dd[u].y);
                            ce[u] = xe;
                            co[u] = xo;
                        }
                    }
                    if (t0 + t < nt) {
                        double *o = Fa + (long)jr * NC12 + (long)(t0 + t) * 12 + 4 * third;
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int me = 2 * (8 * w + 4 * u + k4), mo = me + 1;
#pragma unroll
                            for (int f = 0; f < 2; ++f) {
                                if (me <= p)
                                    *reinterpret_cast<double2 *>(o + (long)me * Q1 * NC12 + 2 * f) =
                                        make_double2(F[u][f][0], F[u][f][2]);
                                if (mo <= p)
                                    *reinterpret_cast<double2 *>(o + (long)mo * Q1 * NC12 + 2 * f) =
                                        make_double2(F[u][f][1], F[u][f][3]);
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();  // f, or the analysis operand, is read; the sums per wavefront are there
        const int tid = fk_tid();
        if (SL && tid < 3 * kFkT) {
            const int tt = tid / 3, c = tid % 3;
            double s = 0.0;
            for (int v = 0; v < nw; ++v) s += red[(v * kFkT + tt) * 3 + c];
            if (t0 + tt < nt) part[((long)(t0 + tt) * Q1 + jr) * 3 + c] = s;
        }
        if (!more) break;
        stage_pole(tn);
        fk_stage(Gx + (Q1 + next / ntb) * NC6, ldx, P1, tn, nt, w, nw, SL ? bA : bB);
        if (SL) {  // the next item's x is in bB
            double *b = bA;
            bA = bB;
            bB = b;
        }
        item = next;
    }
}

// part[t][j'][3] summed over j' into out (scaled, added); column t belongs to
// unit u0 + t / nk of the pass.
__global__ void k_sum_part(int nt, int Q1, int nk, int P1, const double *__restrict__ part, PipeDrops pd, int u0,
                           double scale, double *__restrict__ out, long ostride)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt * 3) return;
    const int t = i / 3, c = i % 3;
    double s = 0.0;
    for (int j = 0; j < Q1; ++j) s += part[((long)t * Q1 + j) * 3 + c];
    const int ug = u0 + t / nk;
    out[c * ostride + pd.toff[ug / P1] + (long)(ug % P1) * nk + t % nk] += scale * s;
}

// Pole values x0 of every target: sum_n Re x'^0_n sqrt((2n+1)/4pi) from the
// mu = 0 block of the rotated x (col = t*6 + c*2).
__global__ void k_pole(int p, int nt, const double *__restrict__ Bx, long NC, double *__restrict__ X0)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nt * 3) return;
    const int t = i / 3, c = i % 3;
    double s = 0.0;
    for (int n = 0; n <= p; ++n) s += Bx[(long)n * NC + (long)t * 6 + 2 * c] * sqrt((2.0 * n + 1.0) / (4.0 * 3.14159265358979323846));
    X0[3 * t + c] = s;
}

// ----------------------------------------------------------------------------
// AR: adjoint rotation on the matrix cores. Block (n, latitude j), 256 threads.
// a_mu = w_mu Bt^mu[n][.. cos], b_mu = -w_mu Bt^mu[n][.. sin] (w_0 = 1, else 2);
// alpha_nu = sum_mu A+_{nu mu} a_mu, beta_nu = sum_mu A-_{nu mu} b_mu as two GEMMs
// (nu x mu) x (mu x col), col = k*6 + pair over the 2p targets of the latitude;
// both results of one (nu, col) land in the same lane, which writes
// M[t][pair][2 tri(n,nu)] = alpha cos(nu phi_k) + beta sin, [+1] = -alpha sin + beta cos.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_adjrot_mfma(int p, const double *__restrict__ Ap,
                                                     const double *__restrict__ Am, const double *__restrict__ csp,
                                                     const double *__restrict__ Bt, long NC12, PipeDrops pd,
                                                     int u0)
{
    extern __shared__ double sm[];
    const int ug = u0 + blockIdx.y, dr = ug / (p + 1);
    const int n = blockIdx.x, j = ug % (p + 1);
    double *__restrict__ M = pd.M[dr];
    const int N1 = n + 1, nk = 2 * p, P1 = p + 1;
    const int MT = (N1 + 15) / 16, NP = MT * 16, NS = NP + 1, KS = (N1 + 3) / 4;
    double *sAp = sm;                  // [nu][mu], NP x NP, zero padded, row stride NS
    double *sAm = sAp + NP * NS;
    double *sCS = sAm + NP * NS;       // [2][nk]
    const size_t lat = rot_lat_size(p) * j + rot_off(n);
    stage_rot(Ap, Am, lat, N1, NP, NS, sAp, sAm);
    for (int i = threadIdx.x; i < 2 * nk; i += 256) sCS[i] = csp[i];
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r16 = lane & 15, k4 = lane >> 4;
    const int ncol = nk * 6, NT = (ncol + 15) / 16;
    const int nc2 = 2 * ncoef(p);
    for (int nt = wv; nt < NT; nt += 4) {
        const int col = nt * 16 + r16;
        const bool cok = col < ncol;
        const int k = cok ? col / 6 : 0, pr = cok ? col % 6 : 0;
        const long tcol = (long)(blockIdx.y * nk + k) * 12 + pr * 2;
        d4_t al[4], be[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) al[m] = be[m] = (d4_t){0, 0, 0, 0};
        // the next depth step's B operand is loaded while this one's products run
        auto bload = [&](int ks) {
            const int mu = ks * 4 + k4;
            return (cok && mu < N1) ? *reinterpret_cast<const double2 *>(Bt + (koff(mu, P1) + (n - mu)) * NC12 + tcol)
                                    : make_double2(0.0, 0.0);
        };
        double2 vn = bload(0);
        for (int ks = 0; ks < KS; ++ks) {
            const int mu = ks * 4 + k4;
            const double2 v = vn;
            if (ks + 1 < KS) vn = bload(ks + 1);
            const double w = mu ? 2.0 : 1.0;
            const double av = w * v.x, bv = -w * v.y;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (m < MT) {
                    const int nu = m * 16 + r16;
                    al[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(sAp[nu * NS + mu], av, al[m], 0, 0, 0);
                    be[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(sAm[nu * NS + mu], bv, be[m], 0, 0, 0);
                }
        }
        if (!cok) continue;
        const long tg = (long)j * nk + k;  // target index within the drop
        double *Mt = M + (tg * 6 + pr) * nc2 + n * (n + 1);
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (m < MT)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int nu = m * 16 + 4 * v + k4;
                    if (nu <= n) {
                        const int e = (int)(((long)nu * k) % nk);
                        const double cc = sCS[e], ss = sCS[nk + e];
                        const double a_ = al[m][v], b_ = be[m][v];
                        *reinterpret_cast<double2 *>(Mt + 2 * nu) =
                            make_double2(fma(a_, cc, b_ * ss), fma(-a_, ss, b_ * cc));
                    }
                }
    }
}

// ============================================================================
// launchers
// ============================================================================
static inline unsigned cdiv(long a, long b) { return (unsigned)((a + b - 1) / b); }

// allow up to 160 KB of dynamic LDS for the kernels that size it by degree
// (once per process, before any of them is launched: server worker threads
// reach this concurrently, and call_once makes the others wait until it is set)
void pipe_set_lds_limits()
{
    static std::once_flag once;
    std::call_once(once, [] {
        for (const void *fn : {(const void *)k_fk<true, true>, (const void *)k_fk<true, false>,
                               (const void *)k_fk<false, true>})
            (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
    });
}

void launch_rot2(hipStream_t st, int p, const double *Ap, const double *Am, const double *csp, const double *xc,
                 long xstride, const double *dc, long dstride, const PipeDrops &pd, int u0, int nunits,
                 double *Bx, double *Bd, long NC)
{
    const int P1 = p + 1, nk = 2 * p, NP = (P1 + 15) / 16 * 16;
    const int nf = dc ? 6 : 3;
    const size_t lds = (size_t)(2 * NP * (NP + 1) + nf * P1 * 2 + 2 * nk) * sizeof(double);
    hipLaunchKernelGGL(k_rot_mfma, dim3(P1, nunits), dim3(256), lds, st, p, Ap, Am, csp, xc, xstride, dc, dstride,
                       pd, u0, Bx, Bd, NC);
}

size_t rot_lds_bytes(int p)
{
    const int P1 = p + 1, NP = (P1 + 15) / 16 * 16;
    return P1 > kRotMaxPad ? (size_t)1 << 40 : (size_t)(2 * NP * (NP + 1) + 6 * P1 * 2 + 4 * p) * sizeof(double);
}

void launch_leg_mfma(hipStream_t st, int nbatch, int maxrows, const void *batches, const double *tab, const double *in,
                     double *out, long NC)
{
    const dim3 grid(cdiv(NC, 64), nbatch);
    const LegBatch *b = static_cast<const LegBatch *>(batches);
    const int MT = (maxrows + 15) / 16;
    switch (MT) {
    case 1: hipLaunchKernelGGL(k_leg_mfma<1>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    case 2: hipLaunchKernelGGL(k_leg_mfma<2>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    case 3: hipLaunchKernelGGL(k_leg_mfma<3>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    case 4: hipLaunchKernelGGL(k_leg_mfma<4>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    case 5: hipLaunchKernelGGL(k_leg_mfma<5>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    case 6: hipLaunchKernelGGL(k_leg_mfma<6>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    default: hipLaunchKernelGGL(k_leg_mfma<7>, grid, dim3(256), 0, st, b, tab, in, out, NC); break;
    }
}

int leg_mfma_max_rows() { return 7 * 16; }
int leg_mfma_max_depth() { return 52; }

// Blocks of one launch: as many as the device holds at once (by LDS and by two
// wavefronts per SIMD), each taking every gridDim.x-th item, so that an item's
// first loads run under the item before.
void launch_fk(hipStream_t st, bool sl, bool dl, int p, int qs, int nt, const double *Gx, const double *Gd, long NC6,
               const double *wsing, const double *cs, const double *X0, double *part, double *Fa, long NC12)
{
    const int nw = fk_waves(qs), ntb = (nt + kFkT - 1) / kFkT;
    const size_t lds = (4 * (size_t)qs + 2 * fk_buf(p, qs, dl) + 3 * kFkT + (sl ? nw * kFkT * 3 : 0)) * sizeof(double);
    const long items = (long)ntb * (qs + 1), cus = 256, per = std::min<long>(163840 / lds, 8 / nw);
    const dim3 grid((unsigned)std::min(items, cus * per)), block(64 * nw);
    auto go = [&](auto fn) {
        hipLaunchKernelGGL(fn, grid, block, lds, st, p, qs, nt, ntb, Gx, Gd, NC6, wsing, cs, X0, part, Fa, NC12);
    };
    if (sl && dl)
        go(k_fk<true, true>);
    else if (sl)
        go(k_fk<true, false>);
    else
        go(k_fk<false, true>);
}

void launch_sum_part(hipStream_t st, int nt, int Q1, int nk, int P1, const double *part, const PipeDrops &pd, int u0,
                     double scale, double *out, long ostride)
{
    hipLaunchKernelGGL(k_sum_part, dim3(cdiv((long)nt * 3, 256)), dim3(256), 0, st, nt, Q1, nk, P1, part, pd, u0, scale,
                       out, ostride);
}

void launch_pole(hipStream_t st, int p, int nt, const double *Bx, long NC, double *X0)
{
    hipLaunchKernelGGL(k_pole, dim3(cdiv((long)nt * 3, 256)), dim3(256), 0, st, p, nt, Bx, NC, X0);
}

void launch_adjrot(hipStream_t st, int p, const double *Ap, const double *Am, const double *csp, const double *Bt,
                   long NC12, const PipeDrops &pd, int u0, int nunits)
{
    const int P1 = p + 1, nk = 2 * p, NP = (P1 + 15) / 16 * 16;
    const size_t lds = (size_t)(2 * NP * (NP + 1) + 2 * nk) * sizeof(double);
    hipLaunchKernelGGL(k_adjrot_mfma, dim3(P1, nunits), dim3(256), lds, st, p, Ap, Am, csp, Bt, NC12, pd, u0);
}

}  // namespace bim
