// HIP kernels of the nodal DG Euler solver for gfx950: the VALU stage (the
// FP64 handles that use_mfma64 leaves to it), sensor, viscous gradient,
// geometry, reductions, prolongation.
//
// Tiling of the VALU stage: one 64-lane wavefront holds EW = floor(64/Np) whole elements, one
// lane per node (lane = element * Np + node); a 256-thread block holds four
// wavefronts.  Elements never straddle wavefronts.  The element's state,
// fluxes and scaled face-flux jumps are staged in LDS; each lane keeps its
// own rows of Dr, Ds and LIFT in registers and forms the contractions
//   rhs_i = -(r_x (Dr F)_i + s_x (Ds F)_i + r_y (Dr G)_i + s_y (Ds G)_i)
//           + sum_q LIFT_iq Fscale_q (n.F(U-) - F*)_q
// (the semi-discrete system in nodal strong form), followed by the
// low-storage Runge-Kutta update in the same kernel.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cstring>

#include "common.hpp"
#include "launch.hpp"

namespace dg {
namespace {

constexpr int kBlock = 256;

template <typename T>
struct StageArgs {
    int K, stage, mode;
    int chunk;     // tiles of an XCD (xcd_tile)
    int riemann;   // numerical flux: RIEMANN_LF or RIEMANN_HLLC
    T g, ra, rb;
    FarField<T> ff;
    const T *__restrict__ Uin;
    T *__restrict__ Uout;
    T *__restrict__ R;
    T *__restrict__ rhs;
    const int *__restrict__ nbr;
    const int *__restrict__ finfo;
    const T *__restrict__ geo;
    const T *__restrict__ fgeo;
    const T *__restrict__ ops;
    const double *__restrict__ dt;
    const T *__restrict__ Q;   // [K][Np][8] sigma Q (viscous handles)
};

// Lane -> (local element, node) map shared by all element-tiled kernels.
template <int P>
struct Tile {
    using O = Order<P>;
    int lane, wave, le, i, el;
    long k;
    bool act;
    // tile `tile` of a mesh of K elements (a single-mesh launch: the block index)
    __device__ Tile(int K, int tile) {
        lane = threadIdx.x & 63;
        wave = threadIdx.x >> 6;
        le = lane / O::Np;
        i = lane - le * O::Np;
        bool lane_ok = le < O::EW;
        el = lane_ok ? wave * O::EW + le : 0;
        k = (long)tile * O::EB + wave * O::EW + le;
        act = lane_ok && k < K;
    }
    __device__ explicit Tile(int K) : Tile(K, blockIdx.x) {}
};

// A block-wide copy of N values into LDS in two halves: load() issues each
// thread's loads back to back (indices clamped, no branches) and store()
// writes them to LDS later, after the kernel has issued its own loads, so
// that the copy's latency overlaps theirs instead of preceding them.
template <typename T, int N>
struct LdsCopy {
    static constexpr int R = (N + kBlock - 1) / kBlock;
    T v[R];
    __device__ void load(const T *__restrict__ src) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = src[min(int(threadIdx.x) + r * kBlock, N - 1)];
    }
    __device__ void store(T *dst) const {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int z = int(threadIdx.x) + r * kBlock;
            if (z < N) dst[z] = v[r];
        }
    }
};

template <typename T, int P, bool AV>
__global__ __launch_bounds__(kBlock) void k_stage(StageArgs<T> a) {
    using O = Order<P>;
    constexpr int Np = O::Np, Nfp = O::Nfp, NF3 = O::Nface, EB = O::EB;
    __shared__ T sU[EB][kFields][Np];
    __shared__ T sF[EB][2 * kFields][Np];
    __shared__ T sJ[EB][kFields][NF3];
    // Dr, Ds and LIFT staged once per block; every thread needs its node's
    // rows of them, which through the caches cost a memory instruction per
    // entry
    constexpr int NOPS = 2 * Np * Np + Np * NF3;
    __shared__ T sOps[NOPS];
    LdsCopy<T, NOPS> opsc;
    opsc.load(a.ops);
    Tile<P> t(a.K, xcd_tile(a.chunk));
    const long k = t.k;
    const int i = t.i, el = t.el;

    T u[kFields] = {};
    if (t.act) {
#pragma unroll
        for (int c = 0; c < kFields; ++c) u[c] = a.Uin[(k * kFields + c) * Np + i];
        T ir = rcp(u[0]);
        T vx = u[1] * ir, vy = u[2] * ir;
        T p = pressure_ir(a.g, u, ir);
        T F[kFields] = {u[1], u[1] * vx + p, u[2] * vx, (u[3] + p) * vx};
        T G[kFields] = {u[2], u[1] * vy, u[2] * vy + p, (u[3] + p) * vy};
        if (AV) {
#pragma unroll
            for (int c = 0; c < kFields; ++c) {
                F[c] -= a.Q[(k * Np + i) * 8 + c];
                G[c] -= a.Q[(k * Np + i) * 8 + 4 + c];
            }
        }
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            sU[el][c][i] = u[c];
            sF[el][c][i] = F[c];
            sF[el][kFields + c][i] = G[c];
        }
    }
    opsc.store(sOps);
    __syncthreads();

    if (t.act) {
        const int info = a.finfo[k];
        for (int q = i; q < NF3; q += Np) {
            const int f = q / Nfp, j = q - f * Nfp;
            const int vm = face_node(P, f, j);
            T um[kFields], up[kFields], d[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) um[c] = sU[el][c][vm];
            const T nx = a.fgeo[(k * 3 + 0) * NF3 + q];
            const T ny = a.fgeo[(k * 3 + 1) * NF3 + q];
            const T fs = a.fgeo[(k * 3 + 2) * NF3 + q];
            const int code = face_bc(info, f);
            long kn = -1;
            int vp = 0;
            if (code == BC_INTERIOR) {
                kn = a.nbr[k * 3 + f];
                vp = face_node(P, face_nbr_face(info, f), Nfp - 1 - j);
#pragma unroll
                for (int c = 0; c < kFields; ++c) up[c] = a.Uin[(kn * kFields + c) * Np + vp];
            } else {
                ghost_state(a.g, code, um, nx, ny, a.ff, up);
            }
            flux_jump(a.riemann, a.g, um, up, nx, ny, d);
            if (AV && code != BC_FARFIELD) {
                // (sigma Q)*.n - (sigma Q)-.n: the central value inside, the
                // mirror closure at a wall (wall_visc_jump), zero at the far
                // field (the element's own value)
                T vmv[kFields], vj[kFields];
#pragma unroll
                for (int c = 0; c < kFields; ++c)
                    vmv[c] = nx * a.Q[(k * Np + vm) * 8 + c] + ny * a.Q[(k * Np + vm) * 8 + 4 + c];
                if (kn >= 0) {
#pragma unroll
                    for (int c = 0; c < kFields; ++c) {
                        T vpv = nx * a.Q[(kn * Np + vp) * 8 + c] + ny * a.Q[(kn * Np + vp) * 8 + 4 + c];
                        vj[c] = T(0.5) * (vmv[c] + vpv) - vmv[c];
                    }
                } else {
                    wall_visc_jump(vmv, nx, ny, vj);
                }
#pragma unroll
                for (int c = 0; c < kFields; ++c) d[c] += vj[c];
            }
#pragma unroll
            for (int c = 0; c < kFields; ++c) sJ[el][c][q] = fs * d[c];
        }
    }
    __syncthreads();
    if (!t.act) return;

    // the node's operator rows: copied into registers up to P = 4; at P = 5
    // (60 values) read from LDS inside the contraction, which leaves the
    // registers for more resident waves (faster there, slower below; the
    // values and the order of operations are the same either way)
    constexpr bool kRowsInRegs = P < 5;
    T rdr[kRowsInRegs ? Np : 1], rds[kRowsInRegs ? Np : 1], rlf[kRowsInRegs ? NF3 : 1];
    if constexpr (kRowsInRegs) {
#pragma unroll
        for (int j = 0; j < Np; ++j) {
            rdr[j] = sOps[i * Np + j];
            rds[j] = sOps[Np * Np + i * Np + j];
        }
#pragma unroll
        for (int q = 0; q < NF3; ++q) rlf[q] = sOps[2 * Np * Np + i * NF3 + q];
    }
    auto dr = [&](int j) -> T {
        if constexpr (kRowsInRegs) return rdr[j]; else return sOps[i * Np + j];
    };
    auto ds = [&](int j) -> T {
        if constexpr (kRowsInRegs) return rds[j]; else return sOps[Np * Np + i * Np + j];
    };
    auto lf = [&](int q) -> T {
        if constexpr (kRowsInRegs) return rlf[q]; else return sOps[2 * Np * Np + i * NF3 + q];
    };
    const T rx = a.geo[(k * 4 + 0) * Np + i], sx = a.geo[(k * 4 + 1) * Np + i];
    const T ry = a.geo[(k * 4 + 2) * Np + i], sy = a.geo[(k * 4 + 3) * Np + i];
    const T dt = a.mode ? T(*a.dt) : T(0);
    // at P = 5 the contractions run node by node across the four fields, so
    // that each operator entry is read from LDS once for all of them (the
    // same sums in the same order as field by field)
    T vol[kRowsInRegs ? 1 : kFields], lift[kRowsInRegs ? 1 : kFields];
    if constexpr (!kRowsInRegs) {
        T drf[kFields] = {}, dsf[kFields] = {}, drg[kFields] = {}, dsg[kFields] = {};
#pragma unroll 3
        for (int j = 0; j < Np; ++j) {
            const T dj = dr(j), sj = ds(j);
#pragma unroll
            for (int c = 0; c < kFields; ++c) {
                const T fv = sF[el][c][j], gv = sF[el][kFields + c][j];
                drf[c] += dj * fv;
                dsf[c] += sj * fv;
                drg[c] += dj * gv;
                dsg[c] += sj * gv;
            }
        }
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            vol[c] = -(rx * drf[c] + sx * dsf[c] + ry * drg[c] + sy * dsg[c]);
            lift[c] = vol[c];
        }
#pragma unroll 3
        for (int q = 0; q < NF3; ++q) {
            const T l = lf(q);
#pragma unroll
            for (int c = 0; c < kFields; ++c) lift[c] += l * sJ[el][c][q];
        }
    }
#pragma unroll
    for (int c = 0; c < kFields; ++c) {
        T val;
        if constexpr (!kRowsInRegs) {
            val = lift[c];
        } else {
            T drf = 0, dsf = 0, drg = 0, dsg = 0;
#pragma unroll
            for (int j = 0; j < Np; ++j) {
                const T fv = sF[el][c][j], gv = sF[el][kFields + c][j];
                drf += dr(j) * fv;
                dsf += ds(j) * fv;
                drg += dr(j) * gv;
                dsg += ds(j) * gv;
            }
            val = -(rx * drf + sx * dsf + ry * drg + sy * dsg);
#pragma unroll
            for (int q = 0; q < NF3; ++q) val += lf(q) * sJ[el][c][q];
        }
        const long idx = (k * kFields + c) * Np + i;
        if (a.mode == 0) {
            a.rhs[idx] = val;
        } else {
            T r = (a.stage == 0) ? dt * val : a.ra * a.R[idx] + dt * val;
            a.R[idx] = r;
            a.Uout[idx] = u[c] + a.rb * r;
        }
    }
}

// ---------------------------------------------------------------------------
// artificial viscosity
// ---------------------------------------------------------------------------

template <typename T>
struct AvArgs {
    int K, P;
    int ngrad, gchunk;   // tiles of the gradient, and of an XCD (xcd_tile)
    T g;
    double gamma;   // the time-step bound is formed in FP64
    FarField<T> ff;
    double s0, kappa;
    const T *__restrict__ U;
    const T *__restrict__ eps_in;
    T *__restrict__ eps_out;
    T *__restrict__ Q;
    const int *__restrict__ nbr;
    const int *__restrict__ finfo;
    const T *__restrict__ geo;
    const T *__restrict__ fgeo;
    const T *__restrict__ ops;
    const T *__restrict__ emax;
    const T *__restrict__ rec;     // [K][16] geometry records (null: per-node geometry for every element)
    const T *__restrict__ opsG;    // matrix-core fragments of Dr, Ds and LIFT
    unsigned long long *__restrict__ vmax;   // CFL-bound slots (gradient with the bound only)
    int *__restrict__ flag;                  // state check (gradient with the bound only)
};

// Persson-Peraire sensor on the density: u_hat = V^{-1} rho, S = (energy of
// the degree-P modes) / (total modal energy), s = log10 S, sine ramp of
// half-width kappa around s0, capped at eps_max,k.  One thread per element:
// the block copies the densities of its kBlock elements into LDS (contiguous
// runs of Np values, all loads issued before the first wait), then each
// thread forms its element's modal energies and viscosity, without block-wide
// phases per element.
template <typename T, int P>
__device__ __forceinline__ void sensor_elem_body(const AvArgs<T> &a, const int tile) {
    using O = Order<P>;
    constexpr int Np = O::Np, Nfp = O::Nfp;
    // an odd row stride puts the threads' rows in distinct LDS banks (Np is
    // even for P = 2, 3 and odd otherwise)
    constexpr int NR = Np | 1;
    __shared__ T sVi[Np * Np];
    __shared__ T sR[kBlock * NR];
    LdsCopy<T, Np * Np> vic;
    vic.load(a.ops + (2 * Np * Np + Np * 3 * Nfp));
    const long k0 = (long)tile * kBlock;
    const int nel = (int)min((long)kBlock, (long)a.K - k0);
    const int nval = nel * Np;
    T rv[Np];
#pragma unroll
    for (int r = 0; r < Np; ++r) {
        const int z = min(int(threadIdx.x) + r * kBlock, nval - 1);
        const int e = z / Np, j = z - e * Np;
        rv[r] = a.U[(k0 + e) * kFields * Np + j];
    }
#pragma unroll
    for (int r = 0; r < Np; ++r) {
        const int z = int(threadIdx.x) + r * kBlock;
        if (z < nval) {
            const int e = z / Np, j = z - e * Np;
            sR[e * NR + j] = rv[r];
        }
    }
    vic.store(sVi);
    __syncthreads();
    if (int(threadIdx.x) >= nel) return;
    const long k = k0 + threadIdx.x;
    const T emax_k = a.emax[k];
    T rho[Np];
#pragma unroll
    for (int j = 0; j < Np; ++j) rho[j] = sR[threadIdx.x * NR + j];
    double num = 0, den = 0;
#pragma unroll
    for (int i = 0; i < Np; ++i) {
        T uh = 0;
#pragma unroll
        for (int j = 0; j < Np; ++j) uh += sVi[i * Np + j] * rho[j];
        const double e2 = double(uh) * double(uh);
        den += e2;
        if (i >= Np - Nfp) num += e2;
    }
    double emax = double(emax_k);
    double e = 0.0;
    if (den > 1e-300 && num > 0.0) {
        double sk = log10(num / den);
        if (sk > a.s0 + a.kappa)
            e = emax;
        else if (sk >= a.s0 - a.kappa)
            e = 0.5 * emax * (1.0 + sin(M_PI * (sk - a.s0) / (2.0 * a.kappa)));
    }
    a.eps_out[k] = T(e);
}

template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_sensor_elem(AvArgs<T> a) {
    sensor_elem_body<T, P>(a, blockIdx.x);
}

// Auxiliary variable of the viscous system, q = sigma grad U (sigma =
// sqrt eps_k), strong form with the central trace (sigma U)*:
//   Q_x = sigma (r_x Dr U + s_x Ds U) + LIFT [Fscale n_x ((sigma U)* - sigma U-)]
// on the matrix cores: a column is one field of one element, 16 columns (4
// elements) a product, and Dr U, Ds U and LIFT applied to the x and y jumps
// are four products whose rows the lane that holds them combines with the
// metric terms (constant on a straight element, per node on a curved one, so
// one path serves both).  Written out as sigma Q, node by node with the x
// and y parts of the four fields adjacent ([K][Np][8]): the stage kernel
// takes a node's or a face node's terms as two 16-byte loads.
template <typename T, int P>
struct GradShape {
    static constexpr int Np = (P + 1) * (P + 2) / 2, Nfp = P + 1, NF3 = 3 * Nfp;
    static constexpr int KSD = (Np + 3) / 4, KSL = (NF3 + 3) / 4, MT = (Np + 15) / 16;
    static constexpr int GW = P == 1 ? 2 : 1;                  // column groups per wavefront
    // Wavefronts that share a column group's row tiles: in FP64 at P = 5 (two
    // tiles) both take one, so a block holds 8 elements instead of 16 and each
    // of its lanes one face node instead of two, whose far-field states (two
    // powers each) followed one another.  Viscous airfoil, ten steps, one
    // wavefront / two: 500 elements 1,468 / 1,286 us, 1,500 1,367 / 1,267,
    // 6,000 1,697 / 1,600, 60,000 6,682 / 6,577 (a kernel on the VALUs: 1,292,
    // 1,339, 1,732 and 7,464).  In FP32 the sharing costs 1% from 60,000 on.
    static constexpr int WG = sizeof(T) == 8 ? MT : 1;
    static constexpr int MW = MT / WG;                         // row tiles of a wavefront
    static constexpr int NT = kBlock / 64 * GW / WG, EB = 4 * NT;   // column groups and elements per block
    static constexpr int NZ = MW * (2 * KSD + KSL);            // A fragments of a wavefront: Dr, Ds, LIFT
    static constexpr int NG = (NZ + 3) / 4;
    static constexpr int SJ = 4 * KSL + 1;                     // LDS stride of a column's jumps
    // LDS stride of a node's result: whole 16-byte vectors, spread over the banks
    static constexpr int SQ = sizeof(T) == 4 ? 12 : 10;
    static constexpr int RG = 32 * SJ > 4 * Np * SQ ? (32 * SJ + 3) / 4 * 4 : 4 * Np * SQ;   // of a group: jumps, then result
    static constexpr int TPT = (EB * NF3 + kBlock - 1) / kBlock;   // face-node tasks per thread
    static constexpr int VW = 16 / int(sizeof(T));
    static constexpr int NV = (EB * kFields * Np / VW + kBlock - 1) / kBlock;   // 16-byte vectors per thread
};

// CFL (a step's first stage): also the time-step bound of the state with its
// viscosity (FP64 per face node, cfl_bound) into the block's slot and the
// state check, from the tile in LDS while the operators are on their way.  A
// sensor that reduced the bound (a thread per node, four block-wide phases)
// took 23 us against the 6 of the sensor alone (120,000 elements, P = 3, ten
// steps: 3,254 us with it, 3,177 with the bound here; 2,000 at P = 5, where
// the chain of a block is what counts, 20 steps: 1,954 and 2,003).
template <typename T, int P, bool CFL>
__device__ __forceinline__ void avgrad_body(const AvArgs<T> &a, const int tile) {
    using S = GradShape<T, P>;
    using V4 = typename VecOf<T>::V4;
    using V16 = typename VecOf<T>::U16;
    constexpr int Np = S::Np, Nfp = S::Nfp, NF3 = S::NF3, KSD = S::KSD, KSL = S::KSL, MW = S::MW, WG = S::WG, GW = S::GW;
    constexpr int EB = S::EB, NG = S::NG, SJ = S::SJ, SQ = S::SQ, RG = S::RG, TPT = S::TPT, VW = S::VW, NV = S::NV;
    __shared__ __attribute__((aligned(16))) T sU[EB * kFields * Np];
    __shared__ __attribute__((aligned(16))) T sW[S::NT * RG];
    __shared__ __attribute__((aligned(16))) T sG[EB][16];
    __shared__ T sSig[EB], sEps[CFL ? EB : 1];
    __shared__ double sRed[kBlock / 64];
    const long k0 = (long)tile * EB;
    const unsigned nel = (unsigned)min((long)EB, (long)a.K - k0);
    const unsigned tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned nflt = nel * kFields * Np, nv = nflt / VW, ntask = nel * NF3;
    // the tile's own data through block-uniform bases and 32-bit offsets
    const T *Ut = a.U + k0 * kFields * Np, *et = a.eps_in + k0, *rt = a.rec ? a.rec + k0 * 16 : nullptr;
    const int *ft = a.finfo + k0, *nt = a.nbr + k0 * 3;
    T *Qt = a.Q + k0 * Np * 8;

    // loads: connectivity, the tile and its geometry, then the neighbours'
    // traces, which stay in flight across the first barrier (a boundary
    // face's neighbour is the element itself)
    int info[TPT], nb[TPT];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const unsigned task = min(tid + t * kBlock, ntask - 1);
        const unsigned e = task / NF3, f = (task - e * NF3) / Nfp;
        info[t] = ft[e];
        nb[t] = nt[e * 3 + f];
    }
    T fsc[TPT];
    if constexpr (CFL)
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
            const unsigned task = min(tid + t * kBlock, ntask - 1), e = task / NF3;
            fsc[t] = a.fgeo[((k0 + e) * 3 + 2) * NF3 + (task - e * NF3)];
        }
    V16 uv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) uv[v] = reinterpret_cast<const V16 *>(Ut)[min(tid + v * kBlock, nv - 1)];
    constexpr int NGV = (EB * 16 / VW + kBlock - 1) / kBlock;
    V16 gv[NGV];
#pragma unroll
    for (int v = 0; v < NGV; ++v) {
#pragma unroll
        for (int e = 0; e < VW; ++e) gv[v][e] = T(1);   // no records: every element takes the per-node tables
        if (rt) gv[v] = reinterpret_cast<const V16 *>(rt)[min(tid + v * kBlock, nel * 16 / VW - 1)];
    }
    const T ev = et[min(tid, nel - 1)];
    T up[TPT][kFields], sp[TPT];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const unsigned task = min(tid + t * kBlock, ntask - 1);
        const unsigned q = task % NF3, f = q / Nfp, j = q - f * Nfp;
        const int vp = face_node(P, face_nbr_face(info[t], f), Nfp - 1 - j);
        const T *src = a.U + (unsigned long)(unsigned)nb[t] * (kFields * Np) + (unsigned)vp;
#pragma unroll
        for (int c = 0; c < kFields; ++c) up[t][c] = src[c * Np];
        sp[t] = a.eps_in[(unsigned)nb[t]];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const unsigned z = tid + v * kBlock;
        if (z < nv) {
#pragma unroll
            for (int e = 0; e < VW; ++e) sU[VW * z + e] = uv[v][e];
        }
    }
#pragma unroll
    for (int v = 0; v < NGV; ++v) {
        const unsigned z = tid + v * kBlock;
        if (z < nel * 16 / VW) {
#pragma unroll
            for (int e = 0; e < VW; ++e) (&sG[0][0])[VW * z + e] = gv[v][e];
        }
    }
    if (tid < nel) {
        sSig[tid] = sqrt(ev);
        if constexpr (CFL) sEps[tid] = ev;
    }
    __syncthreads();

    // jumps Fscale n ((sigma U)* - sigma U-) at the face nodes, column-major
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const unsigned task = tid + t * kBlock;
        if (task < ntask) {
            const unsigned e = task / NF3, q = task - e * NF3, f = q / Nfp;
            const int vm = face_node(P, f, q - f * Nfp);
            T um[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) um[c] = sU[(e * kFields + c) * Np + vm];
            T nx = sG[e][4 + 3 * f], ny = sG[e][5 + 3 * f], fs = sG[e][6 + 3 * f];
            if (sG[e][13] != T(0)) {
                const T *gf = a.fgeo + (k0 + e) * 3 * NF3 + q;
                nx = gf[0];
                ny = gf[NF3];
                fs = gf[2 * NF3];
            }
            const int code = face_bc(info[t], f);
            const T sig = sSig[e];
            T sn = sqrt(sp[t]);
            if (code != BC_INTERIOR) {
                ghost_state(a.g, code, um, nx, ny, a.ff, up[t]);
                sn = sig;
            }
            T *J = sW + (e >> 2) * RG + (e & 3) * kFields * 2 * SJ + q;
            const T fx = fs * nx, fy = fs * ny;
#pragma unroll
            for (int c = 0; c < kFields; ++c) {
                const T d = T(0.5) * (sig * um[c] + sn * up[t][c]) - sig * um[c];
                J[2 * c * SJ] = fx * d;
                J[(2 * c + 1) * SJ] = fy * d;
            }
        }
    }
    V4 ga[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) ga[g] = reinterpret_cast<const V4 *>(a.opsG)[(wave % WG * NG + g) * 64 + lane];
    if constexpr (CFL) {
        double best = 0.0;
        int bad = 0;
        for (unsigned z = tid; z < nel * Np; z += kBlock) {
            const unsigned e = z / Np, i = z - e * Np;
            double u[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) u[c] = double(sU[(e * kFields + c) * Np + i]);
            if (bad_state(a.gamma, u)) bad = 1;
        }
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
            const unsigned task = tid + t * kBlock;
            if (task < ntask) {
                const unsigned e = task / NF3, q = task - e * NF3, f = q / Nfp;
                const int vm = face_node(P, f, q - f * Nfp);
                double u[kFields];
#pragma unroll
                for (int c = 0; c < kFields; ++c) u[c] = double(sU[(e * kFields + c) * Np + vm]);
                const double val = cfl_bound(a.gamma, u, double(fsc[t]), double(sEps[e]), P + 1.0);
                best = val > best ? val : best;
            }
        }
        if (__any(bad) && lane == 0) atomicOr(a.flag, 1);
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(best, off);
            best = o > best ? o : best;
        }
        if (lane == 0) sRed[wave] = best;
    }
    __syncthreads();
    if constexpr (CFL)
        if (tid == 0) {
            double m = sRed[0];
            for (int w = 1; w < kBlock / 64; ++w) m = sRed[w] > m ? sRed[w] : m;
            // non-negative doubles order like their bit patterns
            atomicMax(a.vmax + (blockIdx.x & (kVmaxSlots - 1)), (unsigned long long)__double_as_longlong(m));
        }

    const unsigned col = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int gi = 0; gi < GW; ++gi) {
        const unsigned t = wave / WG * GW + gi, mt0 = wave % WG * MW;
        const V4 zero = {T(0), T(0), T(0), T(0)};
        V4 ar[MW], as[MW], ax[MW], ay[MW];
        if (WG == 1 && 4 * t >= nel) break;   // (of the wavefronts that share a group, none skips the barrier)
        if (WG == 1 || 4 * t < nel) {
            // a column's operand rows beyond its length are zero (the columns of
            // elements past the mesh's end are never written out)
            const T *ub = sU + (t * 16 + col) * Np, *jx = sW + t * RG + col * 2 * SJ, *jy = jx + SJ;
#pragma unroll
            for (int ks = 0; ks < KSD; ++ks) {
                const unsigned row = 4 * ks + kq;
                const T b = 4 * ks + 3 < Np || row < Np ? ub[row] : T(0);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) {
                    const int z = ks * MW + mt, y = KSD * MW + z;
                    ar[mt] = mfma16(ga[z / 4][z % 4], b, ks ? ar[mt] : zero);
                    as[mt] = mfma16(ga[y / 4][y % 4], b, ks ? as[mt] : zero);
                }
            }
#pragma unroll
            for (int ks = 0; ks < KSL; ++ks) {
                const unsigned row = 4 * ks + kq;
                const bool in = 4 * ks + 3 < NF3 || row < NF3;
                const T bx = in ? jx[row] : T(0), by = in ? jy[row] : T(0);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) {
                    const int z = 2 * KSD * MW + ks * MW + mt;
                    ax[mt] = mfma16(ga[z / 4][z % 4], bx, ks ? ax[mt] : zero);
                    ay[mt] = mfma16(ga[z / 4][z % 4], by, ks ? ay[mt] : zero);
                }
            }
        }
        // the result over the group's (consumed) jumps
        if constexpr (WG > 1) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        const unsigned el = t * 4 + (col >> 2), c = col & 3;
        if (el < nel) {
            const T sig = sSig[el];
            const bool curved = sG[el][13] != T(0);
            T rx = sG[el][0], sx = sG[el][1], ry = sG[el][2], sy = sG[el][3];
            T *ob = sW + t * RG + (el & 3) * (Np * SQ) + c;
#pragma unroll
            for (int mt = 0; mt < MW; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // output row of accumulator slot r (consecutive rows per
                    // 16-lane group in FP32, interleaved by 4 in FP64)
                    const unsigned i = 16 * (mt0 + mt) + (sizeof(T) == 4 ? 4 * kq + r : kq + 4 * r);
                    if (i < Np) {
                        if (curved) {
                            const T *gk = a.geo + (k0 + el) * 4 * Np + i;
                            rx = gk[0];
                            sx = gk[Np];
                            ry = gk[2 * Np];
                            sy = gk[3 * Np];
                        }
                        T *o = ob + i * SQ;
                        o[0] = sig * (sig * (rx * ar[mt][r] + sx * as[mt][r]) + ax[mt][r]);
                        o[4] = sig * (sig * (ry * ar[mt][r] + sy * as[mt][r]) + ay[mt][r]);
                    }
                }
        }
    }
    __syncthreads();
    // coalesced copy out, one 16-byte vector per lane
    constexpr int VN = 8 / VW;   // vectors of a node
#pragma unroll
    for (int v = 0; v < (EB * Np * VN + kBlock - 1) / kBlock; ++v) {
        const unsigned z = tid + v * kBlock;
        if (z < nel * Np * VN) {
            const unsigned node = z / VN, h = z - node * VN, g = node / (4 * Np), i = node - g * (4 * Np);
            const T *o = sW + g * RG + i * SQ + h * VW;
            V16 q;
#pragma unroll
            for (int x = 0; x < VW; ++x) q[x] = o[x];
            reinterpret_cast<V16 *>(Qt)[z] = q;
        }
    }
}

// Waves per SIMD of the gradient: what the LDS of its blocks allows, at most 8
// (FP64: its registers allow 4).
template <typename T, int P>
constexpr int grad_waves() {
    using S = GradShape<T, P>;
    constexpr int lds = (S::EB * kFields * S::Np + S::NT * S::RG + S::EB * 17) * int(sizeof(T));
    constexpr int w = 160 * 1024 / lds, cap = sizeof(T) == 4 ? 8 : 4;
    return w < cap ? (w < 1 ? 1 : w) : cap;
}

template <typename T, int P, bool CFL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(grad_waves<T, P>()))) void k_avgrad(AvArgs<T> a) {
    const int tile = xcd_tile(a.gchunk);
    if (tile < a.ngrad) avgrad_body<T, P, CFL>(a, tile);
}

// Batched meshes of one order (FP32 viscous handles): work item = (job,
// tile), a job being one mesh's argument record for this stage (sensor: a tile
// is a block of kBlock elements).
// One work item per block; the grid covers the list's capacity and the
// length is read from device memory (a captured launch stays valid when the
// list changes); surplus blocks exit.
template <int P>
__global__ __launch_bounds__(kBlock) void k_sensor_elem_batch(const AvArgs<float> *__restrict__ jobs,
                                                              const int2 *__restrict__ items,
                                                              const int *__restrict__ nitems_dev) {
    const int w = int(blockIdx.x);
    if (w >= *nitems_dev) return;
    const int2 it = items[w];
    sensor_elem_body<float, P>(jobs[it.x], it.y);
}

template <int P, bool CFL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(grad_waves<float, P>()))) void k_avgrad_batch(const AvArgs<float> *__restrict__ jobs,
                                                         const int2 *__restrict__ items,
                                                         const int *__restrict__ nitems_dev) {
    const int n = *nitems_dev, per = (n + 7) / 8, i = int(blockIdx.x / 8);
    const int w = int(blockIdx.x % 8) * per + i;
    if (i >= per || w >= n) return;
    const int2 it = items[w];
    avgrad_body<float, P, CFL>(jobs[it.x], it.y);
}

// ---------------------------------------------------------------------------
// geometry (FP64, once per mesh)
// ---------------------------------------------------------------------------

template <int P>
__global__ __launch_bounds__(kBlock) void k_geometry(int K, const double *__restrict__ x,
                                                     const double *__restrict__ y,
                                                     const double *__restrict__ ops,
                                                     const double *__restrict__ Mref,
                                                     double *__restrict__ geo,
                                                     double *__restrict__ fgeo,
                                                     double *__restrict__ wmass,
                                                     double *__restrict__ emax, double av_eps0,
                                                     int *__restrict__ count) {
    using O = Order<P>;
    constexpr int Np = O::Np, Nfp = O::Nfp, NF3 = O::Nface, EB = O::EB;
    __shared__ double sX[EB][Np], sY[EB][Np], sJ[EB][Np];
    __shared__ double sM[EB][4][Np];  // xr, xs, yr, ys
    __shared__ double sFs[EB][NF3];
    Tile<P> t(K);
    const long k = t.k;
    const int i = t.i, el = t.el;
    // coordinates relative to the element's first node: Dr and Ds annihilate
    // constants, so the metric terms are the same in exact arithmetic, but
    // the sums no longer cancel the absolute position (on small elements far
    // from the origin that cancellation costs ~|x| / h of the metric terms'
    // precision)
    if (t.act) {
        sX[el][i] = x[k * Np + i] - x[k * Np];
        sY[el][i] = y[k * Np + i] - y[k * Np];
    }
    __syncthreads();
    if (t.act) {
        double xr = 0, xs = 0, yr = 0, ys = 0;
        for (int j = 0; j < Np; ++j) {
            const double dr = ops[i * Np + j], ds = ops[Np * Np + i * Np + j];
            xr += dr * sX[el][j];
            xs += ds * sX[el][j];
            yr += dr * sY[el][j];
            ys += ds * sY[el][j];
        }
        const double J = xr * ys - xs * yr;
        if (!(J > 0.0)) atomicAdd(count, 1);
        geo[(k * 4 + 0) * Np + i] = ys / J;
        geo[(k * 4 + 1) * Np + i] = -yr / J;
        geo[(k * 4 + 2) * Np + i] = -xs / J;
        geo[(k * 4 + 3) * Np + i] = xr / J;
        sJ[el][i] = J;
        sM[el][0][i] = xr;
        sM[el][1][i] = xs;
        sM[el][2][i] = yr;
        sM[el][3][i] = ys;
    }
    __syncthreads();
    if (t.act) {
        for (int q = i; q < NF3; q += Np) {
            const int f = q / Nfp, j = q - f * Nfp;
            const int v = face_node(P, f, j);
            const double xr = sM[el][0][v], xs = sM[el][1][v], yr = sM[el][2][v], ys = sM[el][3][v];
            double ax, ay;
            if (f == 0) {
                ax = yr;
                ay = -xr;
            } else if (f == 1) {
                ax = ys - yr;
                ay = xr - xs;
            } else {
                ax = -ys;
                ay = xs;
            }
            const double len = sqrt(ax * ax + ay * ay);
            fgeo[(k * 3 + 0) * NF3 + q] = ax / len;
            fgeo[(k * 3 + 1) * NF3 + q] = ay / len;
            const double fsc = len / sJ[el][v];
            fgeo[(k * 3 + 2) * NF3 + q] = fsc;
            sFs[el][q] = fsc;
        }
        double w = 0;
        for (int j = 0; j < Np; ++j) w += Mref[i * Np + j] * sJ[el][j];
        wmass[k * Np + i] = w;
    }
    __syncthreads();
    if (t.act && i == 0) {
        double fmax = 0;
        for (int q = 0; q < NF3; ++q) fmax = fmax > sFs[el][q] ? fmax : sFs[el][q];
        emax[k] = av_eps0 * (2.0 / fmax) / P;
    }
}

template <int P>
__global__ void k_check_normals(int K, const int *__restrict__ nbr, const int *__restrict__ finfo,
                                const double *__restrict__ fgeo, int *__restrict__ count) {
    constexpr int Nfp = P + 1, NF3 = 3 * Nfp;
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (long)K * NF3) return;
    const long k = gid / NF3;
    const int q = int(gid - k * NF3);
    const int f = q / Nfp, j = q - f * Nfp;
    const int info = finfo[k];
    if (face_bc(info, f) != BC_INTERIOR) return;
    const long kn = nbr[k * 3 + f];
    const int qn = face_nbr_face(info, f) * Nfp + Nfp - 1 - j;
    const double ex = fgeo[(k * 3 + 0) * NF3 + q] + fgeo[(kn * 3 + 0) * NF3 + qn];
    const double ey = fgeo[(k * 3 + 1) * NF3 + q] + fgeo[(kn * 3 + 1) * NF3 + qn];
    if (!(fabs(ex) <= 1e-10 && fabs(ey) <= 1e-10)) atomicAdd(count + 1, 1);
}

template <int P>
__global__ void k_affine_flags(int K, const double *__restrict__ geo, const double *__restrict__ fgeo,
                               int *__restrict__ flags) {
    constexpr int Np = (P + 1) * (P + 2) / 2, Nfp = P + 1, NF3 = 3 * Nfp;
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    bool affine = true;
    // one scale for the four metric terms: a term that is near zero on this
    // element (an edge nearly parallel to an axis) varies by the rounding of
    // the others, which relative to itself can be large
    double scale = 0;
    for (int m = 0; m < 4; ++m)
        for (int i = 0; i < Np; ++i) scale = fmax(scale, fabs(geo[(k * 4 + m) * Np + i]));
    for (int m = 0; m < 4; ++m) {
        const double *g = geo + (k * 4 + m) * Np;
        for (int i = 1; i < Np; ++i) affine &= fabs(g[i] - g[0]) <= 1e-10 * scale;
    }
    for (int m = 0; m < 3; ++m) {
        const double *g = fgeo + (k * 3 + m) * NF3;
        for (int f = 0; f < 3; ++f) {
            const double ref = g[f * Nfp];
            const double scale = m == 2 ? fabs(ref) : 1.0;
            for (int j = 1; j < Nfp; ++j) affine &= fabs(g[f * Nfp + j] - ref) <= 1e-10 * scale;
        }
    }
    flags[k] = affine ? 1 : 0;
}

template <int P>
__global__ void k_pack_geometry(int K, const double *__restrict__ geo, const double *__restrict__ fgeo,
                                const int *__restrict__ cidx, float *__restrict__ geoA,
                                float *__restrict__ geoC) {
    constexpr int Np = (P + 1) * (P + 2) / 2, Nfp = P + 1, NF3 = 3 * Nfp;
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    float *ga = geoA + k * 16;
    for (int m = 0; m < 4; ++m) ga[m] = float(geo[(k * 4 + m) * Np]);
    for (int f = 0; f < 3; ++f)
        for (int m = 0; m < 3; ++m) ga[4 + 3 * f + m] = float(fgeo[(k * 3 + m) * NF3 + f * Nfp]);
    const int c = cidx[k];
    // slot 13: 1 for a curved element (its per-node record is in geoC)
    ga[13] = c >= 0 ? 1.f : 0.f;
    ga[14] = ga[15] = 0.f;
    if (c >= 0) {
        float *gc = geoC + (long)c * (4 * Np + 9 * Nfp);
        for (int m = 0; m < 4; ++m)
            for (int i = 0; i < Np; ++i) gc[m * Np + i] = float(geo[(k * 4 + m) * Np + i]);
        for (int m = 0; m < 3; ++m)
            for (int q = 0; q < NF3; ++q) gc[4 * Np + m * NF3 + q] = float(fgeo[(k * 3 + m) * NF3 + q]);
    }
}

__global__ void k_cast(const double *__restrict__ src, float *__restrict__ dst, size_t n) {
    const size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n) dst[g] = float(src[g]);
}

template <typename T>
__global__ void k_eps_to_double(const T *__restrict__ src, double *__restrict__ dst, int n) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n) dst[g] = double(src[g]);
}

// ---------------------------------------------------------------------------
// FP64 reductions: time step, totals, residual
// ---------------------------------------------------------------------------

// Fixed-shape tree reduction over the block (deterministic).
template <typename Op>
__device__ double block_reduce(double v, double *sh, Op op) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = op(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

struct MaxOp {
    __device__ double operator()(double a, double b) const { return a > b ? a : b; }
};
struct SumOp {
    __device__ double operator()(double a, double b) const { return a + b; }
};

template <typename T, int P, bool AV>
__global__ __launch_bounds__(kBlock) void k_cfl(int K, double g, const T *__restrict__ U,
                                                const T *__restrict__ eps,
                                                const double *__restrict__ fgeo64,
                                                double *__restrict__ partial,
                                                int *__restrict__ flag) {
    using O = Order<P>;
    constexpr int Np = O::Np, Nfp = O::Nfp, NF3 = O::Nface, EB = O::EB;
    __shared__ double sU[EB][kFields][Np];
    __shared__ double sh[kBlock];
    Tile<P> t(K);
    const long k = t.k;
    const int i = t.i, el = t.el;
    int bad = 0;
    if (t.act) {
        double u[kFields];
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            u[c] = double(U[(k * kFields + c) * Np + i]);
            sU[el][c][i] = u[c];
        }
        if (bad_state(g, u)) bad = 1;
    }
    __syncthreads();
    double vmax = 0.0;
    if (t.act) {
        const double P1 = P + 1.0;
        const double e = AV ? double(eps[k]) : 0.0;
        for (int q = i; q < NF3; q += Np) {
            const int f = q / Nfp, j = q - f * Nfp;
            const int v = face_node(P, f, j);
            double u[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) u[c] = sU[el][c][v];
            const double val = cfl_bound(g, u, fgeo64[(k * 3 + 2) * NF3 + q], e, P1);
            if (val > vmax) vmax = val;
        }
    }
    if (bad) atomicOr(flag, 1);
    const double r = block_reduce(vmax, sh, MaxOp());
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

__global__ __launch_bounds__(kBlock) void k_cfl_finish(int n, const double *__restrict__ partial,
                                                       double cfl, double dt_fixed,
                                                       double *__restrict__ scal) {
    __shared__ double sh[kBlock];
    double v = 0.0;
    // unrolled so that eight loads are in flight per wait (the maximum is
    // exact in any order)
#pragma unroll 8
    for (int b = threadIdx.x; b < n; b += kBlock) v = v > partial[b] ? v : partial[b];
    const double vmax = block_reduce(v, sh, MaxOp());
    if (threadIdx.x == 0) {
        const double dt = dt_fixed > 0.0 ? dt_fixed : cfl * (1.0 / vmax);
        scal[S_DT] = dt;
        scal[S_T] += dt;
        scal[S_DTMIN] = dt < scal[S_DTMIN] ? dt : scal[S_DTMIN];
        scal[S_DTMAX] = dt > scal[S_DTMAX] ? dt : scal[S_DTMAX];
        scal[S_STEPS] += 1.0;
    }
}

__global__ __launch_bounds__(kBlock) void k_cfl_finish_vmax(int n, const double *__restrict__ partial,
                                                            unsigned long long *__restrict__ slot) {
    __shared__ double sh[kBlock];
    double v = 0.0;
#pragma unroll 8
    for (int b = threadIdx.x; b < n; b += kBlock) v = v > partial[b] ? v : partial[b];
    const double vmax = block_reduce(v, sh, MaxOp());
    // the bound in the first slot, zeros in the others
    if (threadIdx.x < kVmaxSlots)
        slot[threadIdx.x] = threadIdx.x == 0 ? (unsigned long long)__double_as_longlong(vmax) : 0ull;
}

// Totals of a state; with a flag also its check.
template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_totals(int K, const T *__restrict__ U,
                                                   const double *__restrict__ wmass,
                                                   double *__restrict__ partial, double g,
                                                   int *__restrict__ flag) {
    using O = Order<P>;
    constexpr int Np = O::Np;
    __shared__ double sh[kBlock];
    Tile<P> t(K);
    double v[kFields] = {0, 0, 0, 0};
    if (t.act) {
        const double w = wmass[t.k * Np + t.i];
        double u[kFields];
#pragma unroll
        for (int c = 0; c < kFields; ++c) u[c] = double(U[(t.k * kFields + c) * Np + t.i]);
        if (flag && bad_state(g, u)) atomicOr(flag, 1);
#pragma unroll
        for (int c = 0; c < kFields; ++c) v[c] = w * u[c];
    }
#pragma unroll
    for (int c = 0; c < kFields; ++c) {
        const double r = block_reduce(v[c], sh, SumOp());
        if (threadIdx.x == 0) partial[blockIdx.x * kFields + c] = r;
    }
}

template <typename T, int P>
__global__ __launch_bounds__(kBlock) void k_absmax(int K, const T *__restrict__ X,
                                                   double *__restrict__ partial) {
    using O = Order<P>;
    constexpr int Np = O::Np;
    __shared__ double sh[kBlock];
    Tile<P> t(K);
    double v[kFields] = {0, 0, 0, 0};
    if (t.act) {
#pragma unroll
        for (int c = 0; c < kFields; ++c) v[c] = fabs(double(X[(t.k * kFields + c) * Np + t.i]));
    }
#pragma unroll
    for (int c = 0; c < kFields; ++c) {
        const double r = block_reduce(v[c], sh, MaxOp());
        if (threadIdx.x == 0) partial[blockIdx.x * kFields + c] = r;
    }
}

template <typename Op>
__global__ __launch_bounds__(kBlock) void k_finish4(int n, const double *__restrict__ partial,
                                                    double *__restrict__ out, Op op) {
    __shared__ double sh[kBlock];
    for (int c = 0; c < kFields; ++c) {
        double v = 0.0;
        for (int b = threadIdx.x; b < n; b += kBlock) v = op(v, partial[b * kFields + c]);
        const double r = block_reduce(v, sh, op);
        if (threadIdx.x == 0) out[c] = r;
    }
}

__global__ void k_reset_scalars(double *scal) {
    if (threadIdx.x == 0) {
        for (int s = 0; s < S_NSCAL; ++s) scal[s] = 0.0;
        scal[S_DTMIN] = DBL_MAX;
    }
}

// ---------------------------------------------------------------------------
// dispatch helpers
// ---------------------------------------------------------------------------

template <int P>
int nblocks(int K) {
    return (K + Order<P>::EB - 1) / Order<P>::EB;
}

int nblocks_rt(int K, int P) {
    switch (P) {
        case 1: return nblocks<1>(K);
        case 2: return nblocks<2>(K);
        case 3: return nblocks<3>(K);
        case 4: return nblocks<4>(K);
        default: return nblocks<5>(K);
    }
}

template <typename F>
hipError_t with_order(int P, F &&f) {
    switch (P) {
        case 1: return f(std::integral_constant<int, 1>());
        case 2: return f(std::integral_constant<int, 2>());
        case 3: return f(std::integral_constant<int, 3>());
        case 4: return f(std::integral_constant<int, 4>());
        case 5: return f(std::integral_constant<int, 5>());
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
const T *tbl_geo(const DevMesh &m);
template <>
const double *tbl_geo<double>(const DevMesh &m) { return m.geo64; }
template <>
const float *tbl_geo<float>(const DevMesh &m) { return m.geo32; }
template <typename T>
const T *tbl_fgeo(const DevMesh &m);
template <>
const double *tbl_fgeo<double>(const DevMesh &m) { return m.fgeo64; }
template <>
const float *tbl_fgeo<float>(const DevMesh &m) { return m.fgeo32; }
template <typename T>
const T *tbl_ops(const DevMesh &m);
template <>
const double *tbl_ops<double>(const DevMesh &m) { return m.ops64; }
template <>
const float *tbl_ops<float>(const DevMesh &m) { return m.ops32; }
template <typename T>
const T *tbl_emax(const DevMesh &m);
template <>
const double *tbl_emax<double>(const DevMesh &m) { return m.emax64; }
template <>
const float *tbl_emax<float>(const DevMesh &m) { return m.emax32; }

template <typename T>
hipError_t stage_t(const DevMesh &m, const void *Uin, void *Uout, void *R, void *rhs, int stage,
                   const void *Q, hipStream_t st) {
    StageArgs<T> a;
    a.riemann = m.riemann;
    a.K = m.K;
    a.stage = stage;
    a.mode = rhs ? 0 : 1;
    a.g = T(m.gamma);
    a.ra = T(rk_a(stage));
    a.rb = T(rk_b(stage));
    a.ff = make_farfield<T>(m.gamma, m.qinf);
    a.Uin = static_cast<const T *>(Uin);
    a.Uout = static_cast<T *>(Uout);
    a.R = static_cast<T *>(R);
    a.rhs = static_cast<T *>(rhs);
    a.nbr = m.nbr;
    a.finfo = m.finfo;
    a.geo = tbl_geo<T>(m);
    a.fgeo = tbl_fgeo<T>(m);
    a.ops = tbl_ops<T>(m);
    a.dt = m.scal + S_DT;
    a.Q = static_cast<const T *>(Q);
    // (the orders and viscosity that use_mfma64 leaves to this kernel)
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        const dim3 grid(xcd_grid(nblocks<P>(m.K)));
        // XCD-contiguous tiles while the states, the register and the per-node
        // geometry stay in the last-level cache; with viscosity always, as
        // the neighbours' sigma Q is twice their state.  Four steps, XCD by
        // XCD / in block order: all curved, P = 2, 230,000 elements 1,419 /
        // 1,475 us, 300,000 2,277 / 2,219, 600,000 4,505 / 4,419; P = 1,
        // 480,000 2,223 / 2,264, 600,000 3,006 / 2,981; viscous, 400,000 at
        // P = 2, a launch 174 / 194 us.
        a.chunk = m.av || in_cache(m.K, (16 * m.Np + 9 * m.Nfp) * sizeof(T)) ? xcd_chunk(nblocks<P>(m.K)) : 0;
        if constexpr (P != 3) {
            if (m.av)
                hipLaunchKernelGGL((k_stage<T, P, true>), grid, dim3(kBlock), 0, st, a);
            else
                hipLaunchKernelGGL((k_stage<T, P, false>), grid, dim3(kBlock), 0, st, a);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    });
}

template <typename T>
AvArgs<T> av_args(const DevMesh &m) {
    AvArgs<T> a;
    a.K = m.K;
    a.P = m.P;
    a.ngrad = grad_tiles(m);
    a.g = T(m.gamma);
    a.gamma = m.gamma;
    a.ff = make_farfield<T>(m.gamma, m.qinf);
    a.s0 = m.av_s0;
    a.kappa = m.av_kappa;
    a.nbr = m.nbr;
    a.finfo = m.finfo;
    a.geo = tbl_geo<T>(m);
    a.fgeo = tbl_fgeo<T>(m);
    a.ops = tbl_ops<T>(m);
    a.emax = tbl_emax<T>(m);
    if constexpr (sizeof(T) == 4) {
        a.rec = m.geoA;
        a.opsG = m.opsG;
    } else {
        a.rec = m.geoA64;
        a.opsG = m.opsG64;
    }
    // XCD-contiguous blocks while what a viscous stage touches (states,
    // register, sigma Q, geometry) stays in the last-level cache.  Four steps
    // of the airfoil, XCD by XCD / in block order: FP64 P = 1, 350,000
    // elements 2,761 / 2,810 us, 450,000 4,069 / 4,001; P = 2, 160,000 2,260 /
    // 2,268, 250,000 4,270 / 4,159; P = 3, 120,000 2,296 / 2,307, 200,000
    // 4,522 / 4,453; FP32 P = 3, 300,000 3,212 / 3,124.
    const size_t geometry = a.rec ? 16 : 4 * m.Np + 9 * m.Nfp;
    a.gchunk = in_cache(m.K, (20 * m.Np + geometry) * sizeof(T)) ? xcd_chunk(a.ngrad) : 0;
    a.vmax = nullptr;
    a.flag = m.flag;
    return a;
}

}  // namespace

int partial_slots(int K, int P) { return nblocks_rt(K, P); }

hipError_t launch_geometry(const DevMesh &m, const double *x, const double *y, double *geo64,
                           double *fgeo64, double *wmass, double *emax64, double av_eps0,
                           hipStream_t st) {
    const double *Mref = m.ops64 + ops_size(m.Np, m.Nfp);
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_geometry<P>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K, x, y,
                           m.ops64, Mref, geo64, fgeo64, wmass, emax64, av_eps0, m.count);
        return hipGetLastError();
    });
}

hipError_t launch_check_normals(const DevMesh &m, hipStream_t st) {
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        const long n = (long)m.K * 3 * (P + 1);
        hipLaunchKernelGGL((k_check_normals<P>), dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st,
                           m.K, m.nbr, m.finfo, m.fgeo64, m.count);
        return hipGetLastError();
    });
}

hipError_t launch_affine_flags(const DevMesh &m, int *flags, hipStream_t st) {
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_affine_flags<P>), dim3((m.K + kBlock - 1) / kBlock), dim3(kBlock), 0, st,
                           m.K, m.geo64, m.fgeo64, flags);
        return hipGetLastError();
    });
}

hipError_t launch_pack_geometry(const DevMesh &m, const int *cidx, float *geoA, float *geoC,
                                hipStream_t st) {
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_pack_geometry<P>), dim3((m.K + kBlock - 1) / kBlock), dim3(kBlock), 0, st,
                           m.K, m.geo64, m.fgeo64, cidx, geoA, geoC);
        return hipGetLastError();
    });
}

hipError_t launch_cast(const double *src, float *dst, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_cast, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_stage(const DevMesh &m, const void *Uin, void *Uout, void *R, void *rhs, int stage,
                        const void *Q, hipStream_t st) {
    // the weak form: its own kernel; FP32 (with or without viscosity): the
    // matrix-core kernel; FP64: the FP64 matrix cores where use_mfma64 says
    // so, else VALU
    if (m.weak) return launch_stage_weak(m, Uin, Uout, R, rhs, stage, false, st);
    if (m.fp32) return launch_stage_mfma(m, Uin, Uout, R, rhs, stage, MfmaStep(), st, Q);
    if (m.opsA64) return launch_stage_mfma64(m, Uin, Uout, R, rhs, stage, false, Q, st);
    return stage_t<double>(m, Uin, Uout, R, rhs, stage, Q, st);
}

template <typename T>
static hipError_t sensor_t(const DevMesh &m, const void *U, void *eps, hipStream_t st) {
    AvArgs<T> a = av_args<T>(m);
    a.U = static_cast<const T *>(U);
    a.eps_out = static_cast<T *>(eps);
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_sensor_elem<T, P>), dim3((m.K + kBlock - 1) / kBlock), dim3(kBlock), 0, st, a);
        return hipGetLastError();
    });
}

hipError_t launch_sensor(const DevMesh &m, const void *U, void *eps, hipStream_t st) {
    return m.fp32 ? sensor_t<float>(m, U, eps, st) : sensor_t<double>(m, U, eps, st);
}

size_t av_args_bytes() { return sizeof(AvArgs<float>); }

void av_fill_args(const DevMesh &m, const void *U, void *eps, void *Q, unsigned long long *vmax, void *out) {
    AvArgs<float> a = av_args<float>(m);
    a.U = static_cast<const float *>(U);
    a.eps_out = static_cast<float *>(eps);
    a.eps_in = static_cast<const float *>(eps);
    a.Q = static_cast<float *>(Q);
    a.vmax = vmax;
    std::memcpy(out, &a, sizeof(a));
}

int sensor_elem_blocks(const DevMesh &m) { return (m.K + kBlock - 1) / kBlock; }

template <typename T>
static int grad_block(int P) {   // elements per block
    int eb = 16;
    (void)with_order(P, [&](auto PC) {
        eb = GradShape<T, decltype(PC)::value>::EB;
        return hipSuccess;
    });
    return eb;
}

int grad_tiles(const DevMesh &m) {
    const int eb = m.fp32 ? grad_block<float>(m.P) : grad_block<double>(m.P);
    return (m.K + eb - 1) / eb;
}

// Fragments of the gradient's products (Dr, Ds, LIFT), for the row tiles of
// each of the wavefronts that share a group: lane l of fragment z = ks MW + mt
// of an operator holds row 16 mt + l % 16, column 4 ks + l / 16 (zero outside
// the matrix), four fragments per group.
size_t grad_opsG_values(int P, bool fp32) {
    size_t n = 0;
    auto values = [&](auto shape) { n = size_t(decltype(shape)::WG) * decltype(shape)::NG * 64 * 4; };
    (void)with_order(P, [&](auto PC) {
        constexpr int PP = decltype(PC)::value;
        if (fp32)
            values(GradShape<float, PP>());
        else
            values(GradShape<double, PP>());
        return hipSuccess;
    });
    return n;
}

template <typename T>
static void fill_opsG(int P, const double *Dr, const double *Ds, const double *LIFT, T *out) {
    (void)with_order(P, [&](auto PC) {
        using S = GradShape<T, decltype(PC)::value>;
        for (int z = 0; z < S::WG * S::NG * 64 * 4; ++z) out[z] = T(0);
        const double *ops[3] = {Dr, Ds, LIFT};
        for (int w = 0; w < S::WG; ++w) {
            int first = 0;
            for (int o = 0; o < 3; ++o) {
                const int cols = o < 2 ? S::Np : S::NF3, nz = (cols + 3) / 4 * S::MW;
                for (int z = 0; z < nz; ++z)
                    for (int l = 0; l < 64; ++l) {
                        const int row = 16 * (w * S::MW + z % S::MW) + (l & 15), c = 4 * (z / S::MW) + (l >> 4);
                        if (row < S::Np && c < cols)
                            out[((w * S::NG + (first + z) / 4) * 64 + l) * 4 + (first + z) % 4] = T(ops[o][row * cols + c]);
                    }
                first += nz;
            }
        }
        return hipSuccess;
    });
}

void grad_fill_opsG(int P, const double *Dr, const double *Ds, const double *LIFT, float *out) {
    fill_opsG<float>(P, Dr, Ds, LIFT, out);
}
void grad_fill_opsG64(int P, const double *Dr, const double *Ds, const double *LIFT, double *out) {
    fill_opsG<double>(P, Dr, Ds, LIFT, out);
}

hipError_t launch_av_batch(int P, bool cfl, const void *jobs, const void *eitems, const int *neitems_dev,
                           int ecapacity, const void *gitems, const int *ngitems_dev, int gcapacity,
                           hipStream_t st) {
    if (ecapacity <= 0 || gcapacity <= 0) return hipSuccess;
    const auto *git = static_cast<const int2 *>(gitems);
    const auto *j = static_cast<const AvArgs<float> *>(jobs);
    const auto *eit = static_cast<const int2 *>(eitems);
    return with_order(P, [&](auto PC) {
        constexpr int PP = decltype(PC)::value;
        hipLaunchKernelGGL((k_sensor_elem_batch<PP>), dim3(ecapacity), dim3(kBlock), 0, st, j, eit, neitems_dev);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const dim3 grid(unsigned((gcapacity + 7) / 8 * 8));
        if (cfl)
            hipLaunchKernelGGL((k_avgrad_batch<PP, true>), grid, dim3(kBlock), 0, st, j, git, ngitems_dev);
        else
            hipLaunchKernelGGL((k_avgrad_batch<PP, false>), grid, dim3(kBlock), 0, st, j, git, ngitems_dev);
        return hipGetLastError();
    });
}

template <typename T, bool CFL>
static hipError_t avgrad_t(const DevMesh &m, const void *U, const void *eps, void *Q, unsigned long long *vmax,
                           hipStream_t st) {
    AvArgs<T> a = av_args<T>(m);
    a.U = static_cast<const T *>(U);
    a.eps_in = static_cast<const T *>(eps);
    a.Q = static_cast<T *>(Q);
    a.vmax = vmax;
    return with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_avgrad<T, P, CFL>), dim3(xcd_grid(grad_tiles(m))), dim3(kBlock), 0, st, a);
        return hipGetLastError();
    });
}

hipError_t launch_avgrad(const DevMesh &m, const void *U, const void *eps, void *Q, hipStream_t st) {
    return m.fp32 ? avgrad_t<float, false>(m, U, eps, Q, nullptr, st)
                  : avgrad_t<double, false>(m, U, eps, Q, nullptr, st);
}

hipError_t launch_avgrad_cfl(const DevMesh &m, const void *U, const void *eps, void *Q, unsigned long long *vmax,
                             hipStream_t st) {
    if (!m.fp32) return hipErrorInvalidValue;
    return avgrad_t<float, true>(m, U, eps, Q, vmax, st);
}

template <typename T>
static hipError_t cfl_t(const DevMesh &m, const void *U, const void *eps, double dt_fixed,
                        hipStream_t st) {
    hipError_t e = with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        if (m.av)
            hipLaunchKernelGGL((k_cfl<T, P, true>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                               m.gamma, static_cast<const T *>(U), static_cast<const T *>(eps),
                               m.fgeo64, m.partial, m.flag);
        else
            hipLaunchKernelGGL((k_cfl<T, P, false>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                               m.gamma, static_cast<const T *>(U), static_cast<const T *>(eps),
                               m.fgeo64, m.partial, m.flag);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cfl_finish, dim3(1), dim3(kBlock), 0, st, nblocks_rt(m.K, m.P), m.partial,
                       m.cfl, dt_fixed, m.scal);
    return hipGetLastError();
}

hipError_t launch_cfl_vmax(const DevMesh &m, const void *U, unsigned long long *slot, hipStream_t st) {
    if (m.fp32 && !m.weak) return launch_cfl_vmax_mfma(m, U, slot, st);
    hipError_t e = with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        if (m.fp32)
            hipLaunchKernelGGL((k_cfl<float, P, false>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                               m.gamma, static_cast<const float *>(U), (const float *)nullptr, m.fgeo64,
                               m.partial, m.flag);
        else
            hipLaunchKernelGGL((k_cfl<double, P, false>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                               m.gamma, static_cast<const double *>(U), (const double *)nullptr, m.fgeo64,
                               m.partial, m.flag);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cfl_finish_vmax, dim3(1), dim3(kBlock), 0, st, nblocks_rt(m.K, m.P), m.partial, slot);
    return hipGetLastError();
}

hipError_t launch_cfl(const DevMesh &m, const void *U, const void *eps, double dt_fixed, hipStream_t st) {
    return m.fp32 ? cfl_t<float>(m, U, eps, dt_fixed, st) : cfl_t<double>(m, U, eps, dt_fixed, st);
}

template <typename T>
static hipError_t totals_t(const DevMesh &m, const void *U, bool check, hipStream_t st) {
    hipError_t e = with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_totals<T, P>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                           static_cast<const T *>(U), m.wmass, m.partial, m.gamma, check ? m.flag : nullptr);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finish4<SumOp>, dim3(1), dim3(kBlock), 0, st, nblocks_rt(m.K, m.P), m.partial,
                       m.scal + S_TOT, SumOp());
    return hipGetLastError();
}

hipError_t launch_totals(const DevMesh &m, const void *U, bool check, hipStream_t st) {
    return m.fp32 ? totals_t<float>(m, U, check, st) : totals_t<double>(m, U, check, st);
}

template <typename T>
static hipError_t residual_t(const DevMesh &m, const void *X, hipStream_t st) {
    hipError_t e = with_order(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_absmax<T, P>), dim3(nblocks<P>(m.K)), dim3(kBlock), 0, st, m.K,
                           static_cast<const T *>(X), m.partial);
        return hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finish4<MaxOp>, dim3(1), dim3(kBlock), 0, st, nblocks_rt(m.K, m.P), m.partial,
                       m.scal + S_RES, MaxOp());
    return hipGetLastError();
}

hipError_t launch_residual(const DevMesh &m, const void *rhs, hipStream_t st) {
    return m.fp32 ? residual_t<float>(m, rhs, st) : residual_t<double>(m, rhs, st);
}

// Prolongation of a state of order P to order Q > P (p-refinement): the
// degree-P polynomial of each element and field evaluated at the order-Q
// nodes, U_Q = I U_P with I = V_Q[:, :Np(P)] V_P^{-1} (the hierarchical modes
// of degree <= P are the first Np(P) of order Q's basis, so this is the
// paper's zero padding of the modal coefficients).  One thread per output
// value; the operator travels in the kernel arguments; sums in FP64.
struct ProlongOp {
    int np_from, np_to;
    double I[kProlongMax];
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_prolong(long n, ProlongOp op, const T *__restrict__ Uf,
                                                    T *__restrict__ Ut) {
    const long idx = (long)blockIdx.x * kBlock + threadIdx.x;
    if (idx >= n) return;
    const long row = idx / op.np_to;          // element * 4 + field
    const int i = int(idx - row * op.np_to);
    const T *src = Uf + row * op.np_from;
    double acc = 0.0;
    for (int j = 0; j < op.np_from; ++j) acc += op.I[i * op.np_from + j] * double(src[j]);
    Ut[idx] = T(acc);
}

hipError_t launch_prolong(int K, int np_from, int np_to, const double *I, bool fp32, const void *Uf, void *Ut,
                          hipStream_t st) {
    if (np_from * np_to > kProlongMax) return hipErrorInvalidValue;
    ProlongOp op;
    op.np_from = np_from;
    op.np_to = np_to;
    for (int z = 0; z < np_from * np_to; ++z) op.I[z] = I[z];
    const long n = long(K) * kFields * np_to;
    const dim3 grid(unsigned((n + kBlock - 1) / kBlock)), block(kBlock);
    if (fp32)
        hipLaunchKernelGGL((k_prolong<float>), grid, block, 0, st, n, op, static_cast<const float *>(Uf),
                           static_cast<float *>(Ut));
    else
        hipLaunchKernelGGL((k_prolong<double>), grid, block, 0, st, n, op, static_cast<const double *>(Uf),
                           static_cast<double *>(Ut));
    return hipGetLastError();
}

hipError_t launch_eps_to_double(const DevMesh &m, const void *eps, double *out, hipStream_t st) {
    const int n = m.K;
    if (m.fp32)
        hipLaunchKernelGGL((k_eps_to_double<float>), dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                           st, static_cast<const float *>(eps), out, n);
    else
        hipLaunchKernelGGL((k_eps_to_double<double>), dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                           st, static_cast<const double *>(eps), out, n);
    return hipGetLastError();
}

hipError_t launch_reset_scalars(const DevMesh &m, hipStream_t st) {
    hipLaunchKernelGGL(k_reset_scalars, dim3(1), dim3(64), 0, st, m.scal);
    return hipGetLastError();
}

}  // namespace dg
