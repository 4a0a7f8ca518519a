// Several leapfrog steps of a 2D grid (one row in y) per launch.
//
// A 2D step is a few microseconds of launch and memory latency around nanoseconds of
// arithmetic, so the time of a solve is the number of launches: the gradient of 128 x 128 x 500
// steps took 3.45 ms at a launch per step, 1.33 ms at 8 steps per launch (9 to 11 us each);
// 512 x 512 x 200 1.0 ms. Here a work-group takes a core of PL_CZ x PL_CX
// cells with a halo of PL_STEPS cells on each side and advances the whole region up to PL_STEPS
// steps in registers and LDS: a step's results are exact one cell less far into the halo each
// time (a step reaches one cell), so the core is exact after the last one. The halo cells are
// stepped again by their own work-groups (6 times the arithmetic, which is idle otherwise).
// Per step: P to LDS, barrier, faces from P, their W to LDS, barrier, cells from W; everything
// that the steps read from memory (e^k of the history, residuals, source terms) is loaded
// before the first one. The same arithmetic, operation for operation, as stencil.hip's kernel
// for one step, whose equations and modes apply.

#include <algorithm>

#include "wv_internal.h"

namespace wv {

namespace {

constexpr int CZ = PL_CZ, CX = PL_CX, H = PL_STEPS;
constexpr int RZ = CZ + 2 * H, RX = CX + 2 * H;  // the region
constexpr int NT = 256;
constexpr int NC = RZ * RX / NT;                 // cells per thread
static_assert(RZ * RX % NT == 0 && NT % RX == 0, "whole rows per pass of the threads");

template <int MODE, bool EX>
__global__ void __launch_bounds__(NT) plane_steps_kernel(const PlaneArgs a)
{
    // every product that is fused with an addition is written as an fma
#pragma clang fp contract(off)
    constexpr bool ADJ = MODE == MODE_ADJ;
    __shared__ float sP[RZ + 1][RX + 1];       // cell (z, x) at [z + 1][x + 1]: row and column 0 lie outside
    __shared__ float sWz[RZ + 1][RX], sWx[RZ][RX + 1];
    const int tid = threadIdx.x;
    const int tiles_x = (a.nx + CX - 1) / CX;
    const int tile = blockIdx.x, s = blockIdx.y;
    const int z0 = tile / tiles_x * CZ - H, x0 = tile % tiles_x * CX - H;
    const int rx = tid % RX, rz0 = tid / RX;
    constexpr int DZ = NT / RX;  // rows between a thread's cells
    const int N = a.nz * a.nx;
    const int i = x0 + rx;
    const bool in_x = i >= 0 && i < a.nx;

    const float* in = a.in + s * a.sstride;
    float* out = a.out + s * a.sstride;
    float A[NC], Vz[NC], Vx[NC], m[NC], dm[NC], Sc[NC], Sz[NC], Sx[NC];
    bool ins[NC], core[NC];
    int cell[NC];
    const float wyc = a.wyc[0];
    const float wyx_c = wyc * a.wxc[in_x ? i : 0], wyx_x = wyc * a.wxf[in_x ? i : 0];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        const int rz = rz0 + u * DZ, k = z0 + rz;
        ins[u] = in_x && k >= 0 && k < a.nz;
        core[u] = ins[u] && rz >= H && rz < H + CZ && rx >= H && rx < H + CX;
        const int q = ins[u] ? k * a.nx + i : 0, kk = ins[u] ? k : 0;
        cell[u] = q;
        A[u] = in[q];
        Vz[u] = in[N + q];
        Vx[u] = in[3LL * N + q];
        m[u] = a.m[q];
        if (MODE == MODE_INC) dm[u] = a.dm[q];
        Sc[u] = a.wzc[kk] * wyx_c;
        Sz[u] = a.wzf[kk] * wyx_c;
        Sx[u] = a.wzc[kk] * wyx_x;
    }
    // operands of every step, all loaded ahead: e of the history (adjoint, incremental) and the
    // extra term of the v_z face (source, residuals)
    float ev[H][NC], add[H][NC];
#pragma unroll
    for (int t = 0; t < H; ++t)
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            ev[t][u] = 0.f;
            add[t][u] = 0.f;
        }
    if (MODE == MODE_INC || ADJ) {
#pragma unroll
        for (int t = 0; t < H; ++t)
            if (t < a.nsteps && (ADJ || a.en0 || t > 0)) {
                const float* e = a.e + s * a.estride + t * a.elevel;
#pragma unroll
                for (int u = 0; u < NC; ++u) ev[t][u] = e[cell[u]];
            }
    }
    // receivers of the region, ordered by cell, then receiver
    const int r0 = a.rec_ptr[tile], r1 = a.rec_ptr[tile + 1];
    int q0[NC], q1[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        q0[u] = q1[u] = r0;
        if (a.nrec > 0 && r1 > r0 && ins[u]) {
            const int local = (rz0 + u * DZ) * RX + rx;
            int lo = r0, hi = r1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (a.rec_ent[mid].x < local) lo = mid + 1;
                else hi = mid;
            }
            q0[u] = lo;
            while (lo < r1 && a.rec_ent[lo].x == local) ++lo;
            q1[u] = lo;
        }
    }
    if (ADJ) {
#pragma unroll
        for (int u = 0; u < NC; ++u)
            if (q1[u] > q0[u]) {
#pragma unroll
                for (int t = 0; t < H; ++t)
                    if (t < a.nsteps) {
                        const float* row = a.resid + ((long long)s * a.nt + a.tidx - t) * a.nrec;
                        float r = 0.f;
                        for (int q = q0[u]; q < q1[u]; ++q) r += row[a.rec_ent[q].y];
                        add[t][u] = r;
                    }
            }
    }
    if (MODE == MODE_FWD) {
        const int sk = a.src_kji[3 * s], si = a.src_kji[3 * s + 2], R = a.src_radius;
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int k = z0 + rz0 + u * DZ;
            if (ins[u] && abs(k - sk) <= R && abs(i - si) <= R) {
                const float w = a.src_w[(k - sk + R) * (2 * R + 1) + (i - si + R)];
#pragma unroll
                for (int t = 0; t < H; ++t)
                    if (t < a.nsteps) {
                        const float bsrc = a.dt * a.wavelet[(long long)s * a.nt + a.tidx + t];
                        add[t][u] = bsrc * w;
                    }
            }
        }
    }
    float blk[NC], acc[NC], cmp[NC];
    if (ADJ) {
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            acc[u] = a.acc[s * 2LL * N + cell[u]];
            cmp[u] = a.acc[s * 2LL * N + N + cell[u]];
            blk[u] = 0.f;
        }
    }
    // row and column 0 of P, the +1 faces past the region: cells that need them are in the halo
    // or outside the grid, where these values are 0
    for (int q = tid; q < RX + 1; q += NT) sP[0][q] = 0.f;
    for (int q = tid; q < RZ + 1; q += NT) sP[q][0] = 0.f;
    for (int q = tid; q < RX; q += NT) sWz[RZ][q] = 0.f;
    for (int q = tid; q < RZ; q += NT) sWx[q][RX] = 0.f;

#pragma unroll
    for (int t = 0; t < H; ++t) {
        if (t < a.nsteps) {  // the same for the whole grid
            float P[NC];
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                const float p = MODE == MODE_FWD   ? m[u] * A[u]
                                : MODE == MODE_INC ? __builtin_fmaf(m[u], A[u], dm[u] * ev[t][u])
                                                   : Sc[u] * A[u];
                P[u] = ins[u] ? p : 0.f;
                sP[rz0 + u * DZ + 1][rx + 1] = P[u];
            }
            __syncthreads();
            float Wz[NC], Wx[NC];
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                const int rz = rz0 + u * DZ;
                const float dz = P[u] - sP[rz][rx + 1], dx = P[u] - sP[rz + 1][rx];
                if (ADJ) {
                    Vz[u] = __builtin_fmaf(Sz[u], Vz[u], -(a.dtdx * dz)) + add[t][u];
                    Vx[u] = __builtin_fmaf(Sx[u], Vx[u], -(a.dtdx * dx));
                } else {
                    Vz[u] = Sz[u] * (__builtin_fmaf(a.dtdx, dz, Vz[u]) + add[t][u]);
                    Vx[u] = Sx[u] * __builtin_fmaf(a.dtdx, dx, Vx[u]);
                }
                Wz[u] = ins[u] ? (ADJ ? Sz[u] * Vz[u] : Vz[u]) : 0.f;
                Wx[u] = ins[u] ? (ADJ ? Sx[u] * Vx[u] : Vx[u]) : 0.f;
                sWz[rz][rx] = Wz[u];
                sWx[rz][rx] = Wx[u];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                const int rz = rz0 + u * DZ;
                float d = sWz[rz + 1][rx] - Wz[u];
                d += sWx[rz][rx + 1] - Wx[u];
                if (ADJ) {
                    A[u] = __builtin_fmaf(Sc[u], A[u], -((a.dtdx * m[u]) * d));
                    // the block's terms in float32, its sum into the compensated pair at its end
                    const bool first = t == 0, last = t == a.nsteps - 1;
                    float y;
                    if (first && last) {
                        y = __builtin_fmaf(ev[t][u], d, -cmp[u]);
                    } else {
                        blk[u] = first ? ev[t][u] * d : __builtin_fmaf(ev[t][u], d, blk[u]);
                        y = blk[u] - cmp[u];
                    }
                    if (last) {
                        const float sum = acc[u] + y;
                        cmp[u] = (sum - acc[u]) - y;
                        acc[u] = sum;
                    }
                } else {
                    A[u] = Sc[u] * __builtin_fmaf(a.dtdx, d, A[u]);
                    if (EX && core[u] && t < a.nextra)
                        a.e_extra[t * a.xlevel + s * (long long)N + cell[u]] = A[u];
                    if (core[u] && q1[u] > q0[u]) {
                        float* row = a.traces + ((long long)s * a.nt + a.tidx + t) * a.nrec;
                        for (int q = q0[u]; q < q1[u]; ++q) row[a.rec_ent[q].y] = Vz[u];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NC; ++u)
        if (core[u]) {
            out[cell[u]] = A[u];
            out[N + cell[u]] = Vz[u];
            out[3LL * N + cell[u]] = Vx[u];
            if (ADJ) {
                a.acc[s * 2LL * N + cell[u]] = acc[u];
                a.acc[s * 2LL * N + N + cell[u]] = cmp[u];
            }
        }
}

}  // namespace

bool plane_supported(int nz, int ny, int nx, int nsrc)
{
    if (ny != 1) return false;
    const long long wgs = (long long)((nz + CZ - 1) / CZ) * ((nx + CX - 1) / CX) * nsrc;
    return wgs <= PL_MAX_WGS;
}

void launch_plane(int mode, const PlaneArgs& a, int nsrc, hipStream_t st)
{
    WV_REQUIRE(a.nsteps >= 1 && a.nsteps <= H, WV_EINVAL, "steps per launch");
    const dim3 grid(((a.nz + CZ - 1) / CZ) * ((a.nx + CX - 1) / CX), nsrc), block(NT);
    if (mode == MODE_ADJ)
        hipLaunchKernelGGL((plane_steps_kernel<MODE_ADJ, false>), grid, block, 0, st, a);
    else if (mode == MODE_INC)
        hipLaunchKernelGGL((plane_steps_kernel<MODE_INC, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((plane_steps_kernel<MODE_FWD, true>), grid, block, 0, st, a);
    WV_HIP(hipGetLastError());
}

}  // namespace wv
