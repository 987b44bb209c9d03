#pragma once
// lbm_block.hpp -- the block pass: kDeepSteps time steps of small lattices in
// one launch, one cell per thread.
//
// A lattice of a few thousand cells cannot fill the chip, and a pass that
// walks rows takes the latency of a row (about 0.7 us) once per row of its
// segment and halo: 15 to 20 times per launch.  Here a workgroup holds a
// region of 32 columns by RH rows, a thread per cell, and takes all T steps in
// place: density and psi, psi exchanged through LDS, force and collision, the
// nine post-collision values exchanged through LDS, and so on.  The region
// shrinks by two cells on each side with every step, so 18 x (RH - 14) of its
// cells come out four steps on; the rest is computed again by the
// neighbouring workgroups, on compute units that would be idle.
//
// What bounds it: latency.  A step is two barriers, two LDS exchanges and one
// dependent chain of about 120 instructions, 0.7 us (FP32) to 0.95 us (FP64,
// eight waves), and a launch costs 2 to 3 us besides.  us per step before
// (the deep pass) and after: FP64 64^2 4.0 -> 1.6, 200^2 4.5 -> 2.1, 517 x 301
// 6.1 -> 4.5; FP32 64^2 3.9 -> 1.5, 200^2 4.0 -> 1.6, 512^2 5.6 -> 4.7.  On larger
// lattices the cells computed more than once (1.9 to 6 times as many) cost
// more than the deep pass's start and end; four_shape in the host runtime
// chooses between the two.
//
// The steps call the single step's routines on the same values, rounded to
// the storage type in between: bitwise the results of single steps.
#include "lbm_deep.hpp"

namespace lbmk {

// Arrays of the region's cells, row by row, with a guard that a neighbour
// index past either end stays in.
template <class R, int RH, bool LOC>
struct BlockLds {
    static constexpr int kGuard = kBlockW + 8, kArr = kBlockW * RH + 2 * kGuard;
    R pops[kQ][kArr], psi[kArr];
    float ref[LOC ? kArr : 1];
};

// Waves per SIMD the block pass is compiled for: as many whole workgroups of
// RH / 2 waves as fit a CU's 32 waves, or in FP64, which needs up to 80
// registers, 24 (one workgroup of 32 rows).
template <int ST, int RH>
constexpr int kBlockWaves = (ST == LBM_STORE_F64 ? (RH == 32 ? 16 : 24) : 32) / (RH / 2) * (RH / 2) / 4;

// Block `tile` of nbx x nby that a lattice is cut into, `steps` (1 .. T) steps:
// fewer than T start as if the first T - steps had been taken.
template <int RH, int T, int ST, int COLL>
__device__ __forceinline__ void block_tile(const void *__restrict__ src_v, void *__restrict__ dst_v,
                                           const Coeffs &c, const Phys<typename Store<ST>::R> &P,
                                           int nbx, int nby, int tile, long long t, int steps,
                                           unsigned long long *__restrict__ err)
{
    using E = typename Store<ST>::E;
    using R = typename Store<ST>::R;
    constexpr bool LOC = Store<ST>::local;
    constexpr int H = kHaloT<T>;
    using L = BlockLds<R, RH, LOC>;
    __shared__ L lds;
    const E *src = (const E *)src_v;
    const int by = tile / nbx, bx = tile - by * nbx;
    const int xs = (int)((long long)bx * c.nx / nbx), xe = (int)((long long)(bx + 1) * c.nx / nbx);
    const int ys = (int)((long long)by * c.ny / nby), ye = (int)((long long)(by + 1) * c.ny / nby);
    const int rx = (int)(threadIdx.x & (kBlockW - 1)), ry = (int)(threadIdx.x / kBlockW);
    const int ex = xe - xs + 2 * H, ey = ye - ys + 2 * H;  // the region's cells in use
    auto wrap = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    const int x = wrap(xs - H + rx, c.nx), y = wrap(ys - H + ry, c.ny);
    const int xm = wrap_lo(x - 1, c.nx), xp = wrap_hi(x + 1, c.nx);
    const int ym = wrap_lo(y - 1, c.ny), yp = wrap_hi(y + 1, c.ny);

    // the first step pulls from memory (cells of the region that no step needs
    // read valid cells too)
    R g[kQ];
    R ref = (R)c.rho_ref;
    {
        const size_t p = c.plane;
        const E *r0 = src + (size_t)y * c.pitch, *rm = src + (size_t)ym * c.pitch,
                *rp = src + (size_t)yp * c.pitch;
        g[0] = (R)r0[x];
        g[1] = (R)r0[p + xm];
        g[2] = (R)rm[2 * p + x];
        g[3] = (R)r0[3 * p + xp];
        g[4] = (R)rp[4 * p + x];
        g[5] = (R)rm[5 * p + xm];
        g[6] = (R)rm[6 * p + xp];
        g[7] = (R)rp[7 * p + xp];
        g[8] = (R)rp[8 * p + xm];
        if constexpr (LOC) {
            auto tri = [&](int r) {
                const float *q = ref_row(src, c, r);
                return Tri<R>{(R)q[xm], (R)q[x], (R)q[xp]};
            };
            const Tri<R> C = tri(y);
            reconstruct<R>(g, tri(ym), C, tri(yp));
            ref = C.o;
        }
    }
    const int at = L::kGuard + (int)threadIdx.x;
    unsigned long long bad = ~0ull;
#pragma unroll 1
    for (int j = T - steps; j < T; ++j) {
        // rows whose values this step needs (whole waves leave the others out;
        // columns that are not needed are computed along)
        R rho = R(0), psi = R(0);
        if (ry >= 2 * j && ry < RH - 2 * j) {
            const bool ok = rho_psi<1, R>(g, ref, P, rho, psi);
            if (!ok && rx >= 2 * j && rx < ex - 2 * j && ry < ey - 2 * j)
                bad = min(bad, domain_key(t + (j - (T - steps)), y, x, c.nx));
            lds.psi[at] = psi;
        }
        __syncthreads();
        if (ry > 2 * j && ry < RH - 1 - 2 * j) {
            const R s[kQ] = {psi,
                             lds.psi[at + 1],
                             lds.psi[at + kBlockW],
                             lds.psi[at - 1],
                             lds.psi[at - kBlockW],
                             lds.psi[at + kBlockW + 1],
                             lds.psi[at + kBlockW - 1],
                             lds.psi[at - kBlockW - 1],
                             lds.psi[at - kBlockW + 1]};
            R Fx, Fy, ux, uy, Jx, Jy;
            force<R>(s, P, Fx, Fy);
            velocity<R>(g, rho, Fx, Fy, ux, uy, Jx, Jy);
            if constexpr (COLL == LBM_COLL_MRT)
                collide_mrt<R>(g, rho, ux, uy, Jx, Jy, Fx, Fy, P);
            else
                collide<R>(g, ref, rho, ux, uy, Jx, Jy, Fx, Fy, P);
            // rounded as a single step stores it
            E X[kQ];
            float newref = 0.0f;
            if constexpr (LOC) {
                const R sd =
                    (((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]))) + g[8];
                R e = R(0);
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    const R w = i == 0 ? R(4.0 / 9.0) : (i < 5 ? R(1.0 / 9.0) : R(1.0 / 36.0));
                    const R dev = fma(-w, sd, g[i]);
                    X[i] = (E)dev;
                    e += dev - (R)X[i];
                }
                newref = (float)(ref + (sd + e));
            } else {
#pragma unroll
                for (int i = 0; i < kQ; ++i)
                    X[i] = (E)g[i];
            }
            if (j < T - 1) {
#pragma unroll
                for (int i = 0; i < kQ; ++i)
                    lds.pops[i][at] = (R)X[i];
                if constexpr (LOC) lds.ref[at] = newref;
            } else if (rx >= H && rx < ex - H && ry < ey - H) {
                E *o = (E *)dst_v + (size_t)y * c.pitch + x;
#pragma unroll
                for (int i = 0; i < kQ; ++i)
                    o[i * c.plane] = X[i];
                if constexpr (LOC) ref_row(dst_v, c, y)[x] = newref;
            }
        }
        if (j == T - 1) break;
        __syncthreads();
        if (ry > 2 * j + 1 && ry < RH - 2 - 2 * j) {
            constexpr int W = kBlockW;
            g[0] = lds.pops[0][at];
            g[1] = lds.pops[1][at - 1];
            g[2] = lds.pops[2][at - W];
            g[3] = lds.pops[3][at + 1];
            g[4] = lds.pops[4][at + W];
            g[5] = lds.pops[5][at - W - 1];
            g[6] = lds.pops[6][at - W + 1];
            g[7] = lds.pops[7][at + W + 1];
            g[8] = lds.pops[8][at + W - 1];
            if constexpr (LOC) {
                auto tri = [&](int o) {
                    return Tri<R>{(R)lds.ref[o - 1], (R)lds.ref[o], (R)lds.ref[o + 1]};
                };
                const Tri<R> C = tri(at);
                reconstruct<R>(g, tri(at - W), C, tri(at + W));
                ref = C.o;
            }
        }
    }
    if (bad != ~0ull) atomicMin(err, bad);
}

// What a workgroup of the block pass needs first (tl: nstrips x nseg blocks), on
// one cache line of the arguments: spread over two, each launch waits once more
// for memory, 0.25 us of 3.5 (64^2 FP64, one step).
struct alignas(64) BlockArgs {
    Tiles tl;
    long long t;
    unsigned long long *err;
    int steps;
};

// The block pass over one lattice.
template <int RH, int T, int ST, int COLL>
__global__ __launch_bounds__(kBlockW *RH, (kBlockWaves<ST, RH>)) void block_kernel(
    const void *__restrict__ src, void *__restrict__ dst, Coeffs c,
    Phys<typename Store<ST>::R> P, BlockArgs a)
{
    block_tile<RH, T, ST, COLL>(src, dst, c, P, a.tl.nstrips, a.tl.nseg,
                                xcd_tile(blockIdx.x, a.tl.ntiles), a.t, a.steps, a.err);
}

// The block pass over every lattice of a batch, `done` steps after the table was
// written, from the buffers of this parity.
template <int RH, int T, int ST, int COLL>
__global__ __launch_bounds__(kBlockW *RH, (kBlockWaves<ST, RH>)) void batch_block_kernel(
    const BatchEntry *__restrict__ table, int nlat, long long done, int parity, int steps)
{
    const BatchTile k = batch_tile<&BatchEntry::tile0_4, &BatchEntry::tl4>(
        table, nlat, xcd_tile(blockIdx.x, gridDim.x), done, parity);
    const auto P = in_scalar_registers(Phys<typename Store<ST>::R>(k.c));
    block_tile<RH, T, ST, COLL>(k.src, k.dst, k.c, P, k.tl.nstrips, k.tl.nseg, k.tile, k.t,
                                steps, k.err);
}

#define LBM_BLOCK_ROWS(X) X(16) X(20) X(24) X(32)

template <int ST, int COLL>
hipError_t block_launch_rows(const SweepArgs &a, int steps)
{
    const dim3 grid((unsigned)a.tl.ntiles);
    switch (a.bx) {
#define LBM_CASE(RH)                                                                          \
    case RH:                                                                                  \
        hipLaunchKernelGGL((block_kernel<RH, kDeepSteps, ST, COLL>), grid, dim3(kBlockW *RH), \
                           0, a.stream, a.src, a.dst, a.c,                                    \
                           Phys<typename Store<ST>::R>(a.c),                                  \
                           BlockArgs{a.tl, a.t, a.err, steps});                               \
        break;
        LBM_BLOCK_ROWS(LBM_CASE)
#undef LBM_CASE
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST>
hipError_t launch_block(const SweepArgs &a, int steps)
{
    return a.c.coll == LBM_COLL_MRT ? block_launch_rows<ST, LBM_COLL_MRT>(a, steps)
                                    : block_launch_rows<ST, LBM_COLL_BGK>(a, steps);
}

template <int ST, int COLL>
hipError_t batch_block_launch_rows(const BatchArgs &a, int steps)
{
    switch (a.bx) {
#define LBM_CASE(RH)                                                                          \
    case RH:                                                                                  \
        hipLaunchKernelGGL((batch_block_kernel<RH, kDeepSteps, ST, COLL>), dim3(a.grid),       \
                           dim3(kBlockW *RH), 0, a.stream, a.table, a.nlat, a.steps_add,      \
                           a.launches_add & 1, steps);                                        \
        break;
        LBM_BLOCK_ROWS(LBM_CASE)
#undef LBM_CASE
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST>
hipError_t launch_batch_block(const BatchArgs &a, int steps)
{
    return a.coll == LBM_COLL_MRT ? batch_block_launch_rows<ST, LBM_COLL_MRT>(a, steps)
                                  : batch_block_launch_rows<ST, LBM_COLL_BGK>(a, steps);
}

}  // namespace lbmk
