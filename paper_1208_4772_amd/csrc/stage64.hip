// FP64 stage kernel on the matrix cores (v_mfma_f64_16x16x4f64).
//
// With constant metric terms the volume term folds into the fluxes,
//   -(r_x Dr F + s_x Ds F + r_y Dr G + s_y Ds G) = -Dr F' - Ds G',
//   F' = r_x F + r_y G,  G' = s_x F + s_y G,
// and a field's right-hand side is the product
//   [LIFT  -Dr  -Ds] . [Fscale (n.F(U-) - F*); F'; G'],
// formed for column groups of 4 elements x 4 fields in three passes (face
// terms, then F', then G') over one small column-major B buffer in LDS; the
// A operand of each pass is read from the caches into registers.  Each
// element's geometry is one 128-byte FP64 record (k_pack_affine64): the
// metric terms at its first node and the normal and Fscale at each face's
// first node, one value for the whole element or face as the fold assumes
// (the per-node values of a straight element differ by rounding only, which
// Dr and Ds would amplify on small elements).  Boundary faces take the ghost
// states, and either numerical flux.
//
// A tile with a curved element (CURV, a block-uniform test) keeps the fluxes
// unfolded: -Dr F, -Ds F, -Dr G and -Ds G are four products, each scaled row
// by row with the per-node metric term and added up, and the faces take the
// per-face-node normals and Fscale.  Twice the volume products, on the tiles
// along the walls only; their operator fragments come from LDS and the next
// product's metric terms are requested before each product (requested from
// the caches one after the other they were the tile's latency: 60,000 curved
// elements at P = 3, ten steps, 1.75 ms without, 1.64 with; now 1.61, VALU
// kernel 1.71).  Viscous handles (AV) subtract sigma Q from the fluxes and add the
// viscous face terms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace dg {
namespace {

template <int P>
struct Tri64 {
    static constexpr int Np = (P + 1) * (P + 2) / 2;
    static constexpr int Nfp = P + 1;
    static constexpr int NF3 = 3 * Nfp;
    static constexpr int KSD = (Np + 3) / 4;      // k-steps of one direction
    static constexpr int KSL = (NF3 + 3) / 4;     // k-steps of the face pass
    static constexpr int KB = 4 * KSD > 4 * KSL ? 4 * KSD : 4 * KSL;
    static constexpr int KPP = KB % 8 == 4 ? KB : KB + 4;   // column stride (words / 2)
    static constexpr int MT = (Np + 15) / 16;
    static constexpr int NZ = (KSD > KSL ? KSD : KSL) * MT;
    static constexpr int NG = (NZ + 3) / 4;       // A fragments per lane per pass, in groups of 4
    static constexpr int W = 4;
    static constexpr int NTH = 64 * W;
    static constexpr int NT = W;                  // column groups per block, one per wavefront
    static constexpr int EB = 4 * NT;             // elements per block
    static constexpr int TPT = (EB * NF3 + NTH - 1) / NTH;   // face-node tasks per thread
    static constexpr int PPT = (EB * Np + NTH - 1) / NTH;    // pointwise tasks per thread
    static constexpr int NV = (EB * kFields * Np / 2 + NTH - 1) / NTH;   // 16-byte vectors per thread
    static_assert(16 * Np <= 16 * KPP, "a group's result fits in its B block");
};

struct Stage64Args {
    int K, stage, mode, riemann;
    double g, ra, rb;
    FarField<double> ff;
    const double *__restrict__ Uin;
    double *__restrict__ Uout;
    double *__restrict__ R;
    double *__restrict__ rhs;
    const int *__restrict__ nbr;       // [K][3]
    const int *__restrict__ finfo;     // [K] packed neighbour face and bc codes
    int chunk;                         // tiles of an XCD (xcd_tile)
    const double *__restrict__ rec;    // [K][16] r_x s_x r_y s_y | (n_x n_y Fscale) x 3 | curved 0 0
    const double *__restrict__ geo;    // [K][4][Np] per-node metric terms (curved tiles)
    const int *__restrict__ cpre;      // [K + 1] curved elements before element k (meshes with curved elements)
    const f64v16 *__restrict__ Q;      // [K][Np][4] sigma Q, x then y parts of the four fields (viscous handles)
    const f64x4 *__restrict__ opsA;  // [3][NG][64]: LIFT, -Dr, -Ds fragments; lane l of
                                       // fragment z = ks MT + mt: slot z % 4 of group z / 4
    const double *__restrict__ dt;
    // the last stage of a step in a run: also the next step's time-step
    // bound from the new state (as k_cfl: FP64 per face node with the
    // per-face-node Fscale, the state check at every node) into the slots
    int bound;
    const double *__restrict__ fgeo;   // [K][3][3 Nfp] n_x, n_y, Fscale
    unsigned long long *__restrict__ vmax;
    int *__restrict__ flag;
};

// five waves per SIMD (at most 96 registers): 901 us on the 1M-element
// P = 5 mesh, against 1,003 us at the four the default register budget gives
// and 1,151 us at six (which spills), all with the tile's loads one after the
// other (847 us a stage now, the bound of a step's last included).  Viscous
// handles take four (K = 30,000 at P = 3, with those loads: 2.23 ms a run of
// ten steps against 2.25 at five; 2.16 now),
// the curved variant four at P = 5, where five spill.
template <int P, bool AV, bool CURV>
constexpr int waves64() {
    return AV || (P == 5 && CURV) ? 4 : 5;
}

template <int P, bool AV, bool CURV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves64<P, AV, CURV>()))) void k_stage_mfma64(Stage64Args a) {
    using S = Tri64<P>;
    constexpr int Np = S::Np, Nfp = S::Nfp, NF3 = S::NF3, KSD = S::KSD, KSL = S::KSL, KPP = S::KPP;
    constexpr int MT = S::MT, NG = S::NG, W = S::W, NTH = S::NTH, NT = S::NT, EB = S::EB;
    constexpr int TPT = S::TPT, PPT = S::PPT, NV = S::NV;
    __shared__ __attribute__((aligned(16))) double sB[NT][16][KPP];
    __shared__ __attribute__((aligned(16))) double sU[EB * kFields * Np];
    // The first loads' pointers are read with the tile count, not after the exit
    // of the surplus blocks: kernel arguments come from memory, and each round
    // of reads is a part of a small mesh's launch.
    asm volatile("" ::"s"(a.Uin), "s"(a.finfo), "s"(a.nbr), "s"(a.rec), "s"(a.opsA));
    const long k0 = (long)xcd_tile(a.chunk) * EB;
    if (k0 >= a.K) return;
    const int nel = (int)min((long)EB, (long)a.K - k0);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long base = k0 * kFields * Np;
    const int nflt = nel * kFields * Np;
    const int nv = nflt / 2;
    const int ntask = nel * NF3;
    // ---- loads: the tile, then the neighbour traces of this thread's
    // face-node tasks (task = element * 3 Nfp + face node; a boundary task
    // reads its own element and ignores it).  Nothing is stored to LDS before
    // the last is requested, and no load waits for another but the traces for
    // the connectivity: tile vectors loaded one after the other, the
    // neighbour's id after its face code and the curved test first of all were
    // three to five waits more (us a step, before / after: cylinder of 2,100
    // at P = 4 45.8 / 43.0, straight 50,000 at P = 5 256 / 243, 999,698 5,599 /
    // 5,226; ten steps of the viscous airfoil, 30,000 at P = 3, 2,190 / 2,155).
    const f64v16 *Uv = reinterpret_cast<const f64v16 *>(a.Uin + base);
    f64x2 uv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) uv[v] = Uv[min(tid + v * NTH, nv - 1)];
    int infov[TPT];
    double upn[TPT][kFields];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const int task = min(tid + t * NTH, ntask - 1);
        const int e = task / NF3, q = task - e * NF3, f = q / Nfp, j = q - f * Nfp;
        const long k = k0 + e;
        infov[t] = a.finfo[k];
        const long kn = a.nbr[k * 3 + f];   // (k itself at a boundary)
        const int vp = face_node(P, face_nbr_face(infov[t], f), Nfp - 1 - j);
#pragma unroll
        for (int c = 0; c < kFields; ++c) upn[t][c] = a.Uin[(kn * kFields + c) * Np + vp];
    }
    // whether the tile holds a curved element (asked once its loads are on
    // their way: two dependent reads)
    bool curved = false;
    if constexpr (CURV) curved = a.cpre[k0 + nel] != a.cpre[k0];
    // the -Dr and -Ds fragments of a curved tile's four products, staged once
    __shared__ __attribute__((aligned(16))) f64x4 sA[CURV ? 2 * NG * 64 : 1];
    constexpr int NAV = (2 * NG * 64 + NTH - 1) / NTH;
    f64x4 av[CURV ? NAV : 1];
    if (CURV && curved) {
#pragma unroll
        for (int v = 0; v < NAV; ++v) av[CURV ? v : 0] = a.opsA[NG * 64 + min(tid + v * NTH, 2 * NG * 64 - 1)];
    }

#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int z = tid + v * NTH;
        if (z < nv) reinterpret_cast<f64x2 *>(sU)[z] = uv[v];
    }
    if (CURV && curved) {
#pragma unroll
        for (int v = 0; v < NAV; ++v)
            if (tid + v * NTH < 2 * NG * 64) sA[tid + v * NTH] = av[CURV ? v : 0];
    }
    __syncthreads();

    f64x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f64x4{0.0, 0.0, 0.0, 0.0};
    f64x4 ga[NG];
    auto load_A = [&](int pass) {
#pragma unroll
        for (int g = 0; g < NG; ++g) ga[g] = a.opsA[(pass * NG + g) * 64 + lane];
    };
    // one pass of the product over the wavefront's column group: B rows
    // [0, 4 KSN) against the pass's A fragments
    auto product = [&](f64x4(&out)[MT], auto KSC) {
        constexpr int KSN = decltype(KSC)::value;
        const int t = wave;
        if (4 * t < nel) {
#pragma unroll
            for (int ks = 0; ks < KSN; ++ks) {
                const double b = sB[t][lane & 15][4 * ks + (lane >> 4)];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const int z = ks * MT + mt;
                    out[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[z / 4][z % 4], b, out[mt], 0, 0, 0);
                }
            }
        }
    };

    // ---- face terms: rows q < 3 Nfp (rows 3 Nfp .. 4 KSL zero)
    if constexpr (4 * KSL > NF3) {
        constexpr int PADR = 4 * KSL - NF3, PADN = 16 * PADR;
        for (int z = tid; z < NT * PADN; z += NTH) {
            const int t = z / PADN, rem = z - t * PADN;
            sB[t][rem / PADR][NF3 + rem % PADR] = 0.0;
        }
    }
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const int task = tid + t * NTH;
        if (task < ntask) {
            const int e = task / NF3, q = task - e * NF3, f = q / Nfp, j = q - f * Nfp;
            const long k = k0 + e;
            const int vm = face_node(P, f, j);
            double um[kFields], up[kFields], d[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) um[c] = sU[(e * kFields + c) * Np + vm];
            double nx, ny, fs;
            if (CURV && curved) {
                const double *gf = a.fgeo + k * 3 * NF3 + q;
                nx = gf[0];
                ny = gf[NF3];
                fs = gf[2 * NF3];
            } else {
                const double *rc = a.rec + k * 16 + 4 + 3 * f;
                nx = rc[0];
                ny = rc[1];
                fs = rc[2];
            }
            const int code = face_bc(infov[t], f);
            if (code == BC_INTERIOR) {
#pragma unroll
                for (int c = 0; c < kFields; ++c) up[c] = upn[t][c];
            } else {
                ghost_state(a.g, code, um, nx, ny, a.ff, up);
            }
            flux_jump(a.riemann, a.g, um, up, nx, ny, d);
            if constexpr (AV) {
                // (sigma Q)*.n - (sigma Q)-.n: the central value inside, the
                // mirror closure at a wall, zero at the far field
                if (code != BC_FARFIELD) {
                    auto normal = [&](const f64v16 *q8, double(&v)[kFields]) {
#pragma unroll
                        for (int c = 0; c < kFields; ++c) v[c] = nx * q8[c / 2][c % 2] + ny * q8[2 + c / 2][c % 2];
                    };
                    double vm4[kFields], vj[kFields];
                    normal(a.Q + (k * Np + vm) * 4, vm4);
                    if (code == BC_INTERIOR) {
                        const int vp = face_node(P, face_nbr_face(infov[t], f), Nfp - 1 - j);
                        double vp4[kFields];
                        normal(a.Q + ((long)a.nbr[k * 3 + f] * Np + vp) * 4, vp4);
#pragma unroll
                        for (int c = 0; c < kFields; ++c) vj[c] = 0.5 * (vm4[c] + vp4[c]) - vm4[c];
                    } else {
                        wall_visc_jump(vm4, nx, ny, vj);
                    }
#pragma unroll
                    for (int c = 0; c < kFields; ++c) d[c] += vj[c];
                }
            }
            double(*B)[KPP] = sB[e / 4];
            const int col = (e % 4) * kFields;
#pragma unroll
            for (int c = 0; c < kFields; ++c) B[col + c][q] = fs * d[c];
        }
    }
    load_A(0);
    // the pointwise fluxes of this thread's nodes: kept in registers for both
    // directions, or (the curved variant, which needs the registers; with
    // viscosity only at P = 5, as it would read sigma Q again) formed again
    // for each pass
    auto fluxes = [&](int z, double(&F)[kFields], double(&G)[kFields]) {
        const int el = z / Np, i = z - el * Np;
        double u[kFields];
#pragma unroll
        for (int c = 0; c < kFields; ++c) u[c] = sU[(el * kFields + c) * Np + i];
        const double ir = rcp(u[0]);
        const double vx = u[1] * ir, vy = u[2] * ir;
        const double pr = pressure_ir(a.g, u, ir);
        F[0] = u[1];
        F[1] = u[1] * vx + pr;
        F[2] = u[2] * vx;
        F[3] = (u[3] + pr) * vx;
        G[0] = u[2];
        G[1] = u[1] * vy;
        G[2] = u[2] * vy + pr;
        G[3] = (u[3] + pr) * vy;
        if constexpr (AV) {
            const f64v16 *Qe = a.Q + (k0 * Np + z) * 4;
#pragma unroll
            for (int c = 0; c < kFields; ++c) {
                F[c] -= Qe[c / 2][c % 2];
                G[c] -= Qe[2 + c / 2][c % 2];
            }
        }
    };
    constexpr bool kKeep = !CURV || (AV && P < 5);
    double Fv[kKeep ? PPT : 1][kFields], Gv[kKeep ? PPT : 1][kFields];
    if constexpr (kKeep) {
#pragma unroll
        for (int p = 0; p < PPT; ++p) fluxes(min(tid + p * NTH, nel * Np - 1), Fv[p], Gv[p]);
    }
    __syncthreads();
    product(acc, std::integral_constant<int, KSL>());

    // the two volume passes fill rows i < Np of the B buffer (rows Np ..
    // 4 KSD zero)
    auto pad_rows = [&]() {
        if constexpr (4 * KSD > Np) {
            constexpr int PADR = 4 * KSD - Np, PADN = 16 * PADR;
            for (int z = tid; z < NT * PADN; z += NTH) {
                const int t = z / PADN, rem = z - t * PADN;
                sB[t][rem / PADR][Np + rem % PADR] = 0.0;
            }
        }
    };
    if (!(CURV && curved)) {
        // ---- the two directions: F' = r_x F + r_y G, then G' = s_x F + s_y G
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            __syncthreads();
            pad_rows();
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                const int z = tid + p * NTH;
                if (z < nel * Np) {
                    const int el = z / Np, i = z - el * Np;
                    const long k = k0 + el;
                    // r_x, r_y for F'; s_x, s_y for G'
                    const double mf = a.rec[k * 16 + dir], mg = a.rec[k * 16 + 2 + dir];
                    double(*B)[KPP] = sB[el / 4];
                    const int col = (el % 4) * kFields;
                    if constexpr (!kKeep) fluxes(z, Fv[0], Gv[0]);
                    constexpr int one = kKeep ? 1 : 0;
#pragma unroll
                    for (int c = 0; c < kFields; ++c) B[col + c][i] = mf * Fv[one * p][c] + mg * Gv[one * p][c];
                }
            }
            load_A(1 + dir);
            __syncthreads();
            product(acc, std::integral_constant<int, KSD>());
        }
    } else {
        // ---- F, then G: -Dr and -Ds of each, scaled by the metric terms of
        // the rows this lane holds
        const int le = 4 * wave + ((lane & 15) >> 2);
        const double *gk = a.geo + (k0 + min(le, nel - 1)) * 4 * Np;
        auto metrics = [&](double(&g)[MT][4], int m) {   // r_x, s_x, r_y, s_y
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) g[mt][r] = gk[m * Np + min(16 * mt + (lane >> 4) + 4 * r, Np - 1)];
        };
        double g[MT][4], gn[MT][4];
        metrics(g, 0);
#pragma unroll 1
        for (int m = 0; m < 4; ++m) {
            const int flux = m >> 1;
            if (!(m & 1)) {
                __syncthreads();
                pad_rows();
#pragma unroll
                for (int p = 0; p < PPT; ++p) {
                    const int z = tid + p * NTH;
                    if (z < nel * Np) {
                        const int el = z / Np, i = z - el * Np;
                        double(*B)[KPP] = sB[el / 4];
                        const int col = (el % 4) * kFields;
                        if constexpr (!kKeep) fluxes(z, Fv[0], Gv[0]);
                        constexpr int one = kKeep ? 1 : 0;
#pragma unroll
                        for (int c = 0; c < kFields; ++c) B[col + c][i] = flux ? Gv[one * p][c] : Fv[one * p][c];
                    }
                }
                __syncthreads();
            }
            // the next operator's metric terms on their way during the product
            metrics(gn, min(m + 1, 3));
            f64x4 part[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) part[mt] = f64x4{0.0, 0.0, 0.0, 0.0};
            if (4 * wave < nel) {
                const f64x4 *A = sA + (m & 1) * NG * 64 + lane;
                f64x4 a4;
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    const double b = sB[wave][lane & 15][4 * ks + (lane >> 4)];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const int z = ks * MT + mt;
                        if (z % 4 == 0) a4 = A[z / 4 * 64];
                        part[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a4[z % 4], b, part[mt], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[mt][r] += g[mt][r] * part[mt][r];
                    g[mt][r] = gn[mt][r];
                }
        }
    }
    __syncthreads();
    // the result over the wavefront's own B block as [element % 4][field][node]
    // (accumulator slot r of lane l is row 16 mt + l / 16 + 4 r, column l % 16)
    {
        const int t = wave;
        const int col = lane & 15, le = col / kFields, c = col - le * kFields;
        if (4 * t + le < nel) {
            double *res = &sB[t][0][0];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 16 * mt + (lane >> 4) + 4 * r;
                    if (i < Np) res[(le * kFields + c) * Np + i] = acc[mt][r];
                }
        }
    }
    __syncthreads();

    // ---- epilogue: Runge-Kutta update (or the bare rhs) in 16-byte vectors
    const double dt = a.mode ? *a.dt : 0.0;
    const bool rk_read = a.mode && a.stage > 0;
    auto result = [&](int z) -> double {
        const int el = z / (kFields * Np), off = z - el * (kFields * Np);
        return (&sB[el / 4][0][0])[(el % 4) * kFields * Np + off];
    };
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int zv = tid + v * NTH;
        if (zv < nv) {
            const f64x2 rh = {result(2 * zv), result(2 * zv + 1)};
            if (a.mode == 0) {
                reinterpret_cast<f64v16 *>(a.rhs + base)[zv] = rh;
            } else {
                const f64x2 rold = rk_read ? f64x2(reinterpret_cast<const f64v16 *>(a.R + base)[zv]) : f64x2{0.0, 0.0};
                const f64x2 rr = a.stage == 0 ? dt * rh : a.ra * rold + dt * rh;
                const f64x2 un = reinterpret_cast<const f64x2 *>(sU)[zv] + a.rb * rr;
                reinterpret_cast<f64v16 *>(a.R + base)[zv] = rr;
                reinterpret_cast<f64v16 *>(a.Uout + base)[zv] = un;
                if (a.bound) reinterpret_cast<f64x2 *>(sU)[zv] = un;
            }
        }
    }
    for (int z = 2 * nv + tid; z < nflt; z += NTH) {
        const double rh = result(z);
        const long idx = base + z;
        if (a.mode == 0) {
            a.rhs[idx] = rh;
        } else {
            const double rr = a.stage == 0 ? dt * rh : a.ra * a.R[idx] + dt * rh;
            const double un = sU[z] + a.rb * rr;
            a.R[idx] = rr;
            a.Uout[idx] = un;
            if (a.bound) sU[z] = un;
        }
    }
    if (a.bound) {
        __shared__ double sRed[W];
        __syncthreads();
        int bad = 0;
        for (int z = tid; z < nel * Np; z += NTH) {
            const int el = z / Np, i = z - el * Np;
            double u[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) u[c] = sU[(el * kFields + c) * Np + i];
            if (bad_state(a.g, u)) bad = 1;
        }
        double best = 0.0;
        for (int z = tid; z < ntask; z += NTH) {
            const int e = z / NF3, q = z - e * NF3, f = q / Nfp, j = q - f * Nfp;
            const int v = face_node(P, f, j);
            double u[kFields];
#pragma unroll
            for (int c = 0; c < kFields; ++c) u[c] = sU[(e * kFields + c) * Np + v];
            const double b = cfl_bound(a.g, u, a.fgeo[((k0 + e) * 3 + 2) * NF3 + q], 0.0, P + 1.0);
            best = b > best ? b : best;
        }
        if (__any(bad) && lane == 0) atomicOr(a.flag, 1);
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(best, off);
            best = o > best ? o : best;
        }
        if (lane == 0) sRed[wave] = best;
        __syncthreads();
        if (tid == 0) {
            double m = sRed[0];
            for (int w = 1; w < W; ++w) m = sRed[w] > m ? sRed[w] : m;
            atomicMax(a.vmax + (blockIdx.x & (kVmaxSlots - 1)), (unsigned long long)__double_as_longlong(m));
        }
    }
}

// dt = CFL / bound from the slots (or the fixed step), booked into the
// scalars as k_cfl_finish does; clears the slots.  One wavefront of
// kVmaxSlots lanes.
__global__ void k_dt_slots64(double cfl, double dt_fixed, unsigned long long *__restrict__ slots,
                             double *__restrict__ scal) {
    const int l = threadIdx.x;
    unsigned long long v = slots[l];
    for (int off = kVmaxSlots / 2; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    slots[l] = 0ull;
    if (l != 0) return;
    const double vmax = __longlong_as_double((long long)v);
    const double dt = dt_fixed > 0.0 ? dt_fixed : cfl * (1.0 / vmax);
    scal[S_DT] = dt;
    scal[S_T] += dt;
    scal[S_DTMIN] = dt < scal[S_DTMIN] ? dt : scal[S_DTMIN];
    scal[S_DTMAX] = dt > scal[S_DTMAX] ? dt : scal[S_DTMAX];
    scal[S_STEPS] += 1.0;
}

// The 128-byte geometry record of each element: the metric terms at its
// first node, each face's normal and Fscale at its first node, and 1 in slot
// 13 for a curved element (whose per-node tables are used instead).
__global__ void k_pack_affine64(int K, int Np, int Nfp, const double *__restrict__ geo,
                                const double *__restrict__ fgeo, const int *__restrict__ straight,
                                double *__restrict__ rec) {
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const int NF3 = 3 * Nfp;
    double *r = rec + k * 16;
    for (int m = 0; m < 4; ++m) r[m] = geo[(k * 4 + m) * Np];
    for (int f = 0; f < 3; ++f)
        for (int m = 0; m < 3; ++m) r[4 + 3 * f + m] = fgeo[(k * 3 + m) * NF3 + f * Nfp];
    r[13] = straight[k] ? 0.0 : 1.0;
    r[14] = r[15] = 0.0;
}

template <typename F>
auto with_order64(int P, F &&f) {
    switch (P) {
        case 1: return f(std::integral_constant<int, 1>());
        case 2: return f(std::integral_constant<int, 2>());
        case 3: return f(std::integral_constant<int, 3>());
        case 4: return f(std::integral_constant<int, 4>());
        default: return f(std::integral_constant<int, 5>());
    }
}

}  // namespace

size_t mfma64_opsA_values(int P) {
    return with_order64(P, [](auto PC) { return size_t(3) * Tri64<decltype(PC)::value>::NG * 64 * 4; });
}

void mfma64_fill_opsA(int P, const double *Dr, const double *Ds, const double *LIFT, double *out) {
    with_order64(P, [&](auto PC) {
        using S = Tri64<decltype(PC)::value>;
        constexpr int Np = S::Np, NF3 = S::NF3, MT = S::MT, NG = S::NG;
        std::fill(out, out + size_t(3) * NG * 64 * 4, 0.0);
        for (int pass = 0; pass < 3; ++pass) {
            const int ksn = pass == 0 ? S::KSL : S::KSD;
            for (int mt = 0; mt < MT; ++mt)
                for (int l = 0; l < 64; ++l)
                    for (int ks = 0; ks < ksn; ++ks) {
                        const int m = 16 * mt + (l & 15), k = 4 * ks + (l >> 4);
                        double v = 0.0;
                        if (m < Np) {
                            if (pass == 0)
                                v = k < NF3 ? LIFT[m * NF3 + k] : 0.0;
                            else if (k < Np)
                                v = -(pass == 1 ? Dr : Ds)[m * Np + k];
                        }
                        const int z = ks * MT + mt;
                        out[((size_t(pass) * NG + z / 4) * 64 + l) * 4 + z % 4] = v;
                    }
        }
        return 0;
    });
}

hipError_t launch_pack_affine64(const DevMesh &m, const int *straight, double *rec, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_affine64, dim3((m.K + 127) / 128), dim3(128), 0, st, m.K, m.Np, m.Nfp, m.geo64,
                       m.fgeo64, straight, rec);
    return hipGetLastError();
}

hipError_t launch_dt_slots64(const DevMesh &m, double dt_fixed, hipStream_t st) {
    hipLaunchKernelGGL(k_dt_slots64, dim3(1), dim3(kVmaxSlots), 0, st, m.cfl, dt_fixed, m.vmax, m.scal);
    return hipGetLastError();
}

hipError_t launch_stage_mfma64(const DevMesh &m, const void *Uin, void *Uout, void *R, void *rhs, int stage,
                               bool bound, const void *Q, hipStream_t st) {
    if (m.av && !Q) return hipErrorInvalidValue;
    Stage64Args a;
    a.K = m.K;
    a.stage = stage;
    a.mode = rhs ? 0 : 1;
    a.riemann = m.riemann;
    a.g = m.gamma;
    a.ra = rk_a(stage);
    a.rb = rk_b(stage);
    a.ff = make_farfield<double>(m.gamma, m.qinf);
    a.Uin = static_cast<const double *>(Uin);
    a.Uout = static_cast<double *>(Uout);
    a.R = static_cast<double *>(R);
    a.rhs = static_cast<double *>(rhs);
    a.nbr = m.nbr;
    a.finfo = m.finfo;
    a.rec = m.geoA64;
    a.geo = m.geo64;
    a.cpre = m.cpre;
    a.Q = static_cast<const f64v16 *>(Q);
    a.opsA = reinterpret_cast<const f64x4 *>(m.opsA64);
    a.dt = m.scal + S_DT;
    a.bound = bound && !rhs && m.vmax ? 1 : 0;
    a.fgeo = m.fgeo64;
    a.vmax = m.vmax;
    a.flag = m.flag;
    return with_order64(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        using S = Tri64<P>;
        const int blocks = (m.K + S::EB - 1) / S::EB;
        // XCD-contiguous tiles while states, register and geometry records stay
        // in the last-level cache; beyond it consecutive blocks on consecutive
        // tiles stream better.  Five steps of a straight mesh, XCD by XCD / in
        // block order: P = 3, 170,000 elements 1,598 / 1,649 us, 200,000 1,966 /
        // 1,895; P = 4, 115,000 1,422 / 1,524, 130,000 1,633 / 1,607; P = 2,
        // 250,000 1,812 / 1,821, 300,000 2,206 / 2,172.
        a.chunk = in_cache(m.K, 16 * (S::Np + 1) * sizeof(double)) ? xcd_chunk(blocks) : 0;
        const dim3 grid(xcd_grid(blocks)), block(S::NTH);
        if (m.av) {
            // (curved or not: one variant, the tile's test is cheap)
            if constexpr (P >= kMinMatrix64) hipLaunchKernelGGL((k_stage_mfma64<P, true, true>), grid, block, 0, st, a);
        } else if (m.Kc) {
            if constexpr (P >= kMinMatrix64) hipLaunchKernelGGL((k_stage_mfma64<P, false, true>), grid, block, 0, st, a);
        } else {
            hipLaunchKernelGGL((k_stage_mfma64<P, false, false>), grid, block, 0, st, a);
        }
        return hipGetLastError();
    });
}

}  // namespace dg
