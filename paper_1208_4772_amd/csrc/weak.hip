// The paper's over-integrated weak form (Section 2, eqs. stiffness, mass,
// face_mass, semidiscrete) as a selectable variant of the stage kernel:
//
//   M_k dU/dt = V - S,
//   V_i = sum_q w_q J_q [dphi_i/dr (r_x F + r_y G) + dphi_i/ds (s_x F + s_y G)](x_q)
//   S_i = sum_f sum_g w_g sJ_fg phi_i(x_fg) F*(u-, u+)_fg
//
// with the state interpolated to a cubature rule exact for degree 3P and to
// Gauss points on the faces, the fluxes evaluated there, and the per-element
// mass matrix M_k (J M_ref on a straight element, its inverse precomputed by
// Cholesky factorisation on a curved one).  The paper forms S_x and M_k^{-1}
// per curved element (Section 4); here a curved element keeps its metric
// terms per cubature point and its inverse mass matrix, a straight one five
// numbers.  The contractions run on the matrix cores in the handle's precision
// (FP64 or FP32); the setup (metric terms at cubature and face points, mass
// matrices, Cholesky) runs in FP64 on the GPU.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <vector>

#include "common.hpp"
#include "launch.hpp"

namespace dg {
namespace {

template <int P>
struct WShape {
    static constexpr int Np = (P + 1) * (P + 2) / 2, Nfp = P + 1;
    static constexpr int n = (3 * P + 2) / 2;         // points per direction / per face
    static constexpr int NQ = n * n, NG = n;
};

// ---- the stage --------------------------------------------------------------
//
// A wavefront owns a group of four elements, 16 columns (element, field) of
// v_mfma_f32_16x16x4f32 / v_mfma_f64_16x16x4f64, from the state to the
// update, without a block barrier and without LDS between the products:
//   1. a tile of 16 cubature points: Icub . U;
//   2. a lane then holds one field at four points, its quad the four fields:
//      a 4 x 4 transpose within the quad (DPP) gives each lane one point's
//      four fields, it forms that point's fluxes a = w_q J (r_x F + r_y G),
//      b = w_q J (s_x F + s_y G), and transposes them back;
//   3. these registers are the next product's operand as they stand: the
//      accumulator rows a lane holds are taken as that product's k order,
//      and the operator fragments are laid out to match;
//   4. the update's product A2 . [a; b], A2 = M_ref^-1 [Drc^T | Dsc^T | -L]
//      formed in FP64 on the host (straight elements: M_k = J M_ref).
// The face Gauss points take the same steps after the volume: the element's
// own trace and the neighbour's are two products (the neighbour's operand
// gathered straight into registers), each lane forms one point's numerical
// flux.  A curved element's result still wants M_k^-1 M_ref (formed at setup)
// instead of 1 / J: Np x Np per element on the VALUs.
//
// The fragments are the same for every group: a block stages them in LDS and
// its wavefronts walk several groups (read from the caches for every group
// they were 25 to 32 KB of loads per four elements).  A large mesh is bound by
// issue: an FP32 product takes its SIMD 32 cycles and the VALUs' work (fluxes,
// transposes) adds to that, so 999,698 straight elements at P = 5 run a stage
// in 843 us, 49% of it the products and 44% the VALUs (100,000 in 100 us; 132
// with a block barrier between the products and the fluxes in LDS).  A small one is bound
// by the chain of a group's products: 5,000 elements at P = 4 in FP64 take 15
// us a stage (22 us with the contractions on the VALUs, one element per
// block).  Two steps of 100,000 elements, before and after: FP32 P = 4 1,878
// and 875 us, FP64 P = 3 1,511 and 935 us, P = 5 4,579 and 2,190 us.  P = 1
// has a kernel of its own below.
template <typename T, int P>
struct WeakM {
    static constexpr int Np = WShape<P>::Np, Nfp = P + 1, NF3 = 3 * Nfp;
    static constexpr int NQ = WShape<P>::NQ, NG = WShape<P>::NG, NFG = 3 * NG;
    static constexpr int KS1 = (Np + 3) / 4, MT1 = (NQ + 15) / 16;    // volume points
    static constexpr int KSF = (NF3 + 3) / 4, MG = (NFG + 15) / 16;   // face Gauss points
    static constexpr int MT2 = (Np + 15) / 16;                        // update
    // row of accumulator slot r of 16-lane group kq (consecutive rows per
    // group in FP32, interleaved by 4 in FP64)
    static __host__ __device__ constexpr int row(int mt, int kq, int r) {
        return 16 * mt + (sizeof(T) == 4 ? 4 * kq + r : kq + 4 * r);
    }
    // whether slot r of tile mt holds a row below n in any lane
    static __host__ __device__ constexpr bool used(int mt, int r, int n) { return row(mt, 0, r) < n; }
    static constexpr int count_used(int tiles, int n) {
        int c = 0;
        for (int mt = 0; mt < tiles; ++mt)
            for (int r = 0; r < 4; ++r) c += used(mt, r, n) ? 1 : 0;
        return c;
    }
    static constexpr int VF = 16 / int(sizeof(T));   // fragments per 16-byte vector
    // fragments in the order the kernel takes them
    static constexpr int NZ = MT1 * KS1 + 2 * MT2 * count_used(MT1, NQ) + MG * (KS1 + KSF) + MT2 * count_used(MG, NFG);
    static constexpr int NZV = (NZ + VF - 1) / VF;
    static constexpr int TS = 16 * Np + 4;           // LDS values of a group's tile
    static constexpr int NV = (16 * Np / VF + 63) / 64;   // 16-byte vectors of a tile per lane
    // whether the running sums of the tile-by-tile update (PART) wait in LDS:
    // from P = 4 on their registers spill (20,000 elements on the cylinder,
    // five steps, FP32: P = 5 895 us in registers, 785 in LDS; P = 4 556, 544)
    template <bool PART>
    static constexpr bool lds_sum() {
        return PART && P >= 4;
    }
};

template <typename T>
struct WeakArgs {
    int K, stage, mode, riemann;
    int ngroups, per;   // groups of four elements, and of an XCD
    T g, ra, rb;
    FarField<T> ff;
    const T *__restrict__ Uin;
    T *__restrict__ Uout;
    T *__restrict__ R;
    T *__restrict__ rhs;
    const int *__restrict__ nbr;
    const int *__restrict__ finfo;
    const T *__restrict__ ops;     // Icub | Drc | Dsc | wq | If | M_ref^-1
    const T *__restrict__ frag;    // [NZV][64][VF] operator fragments
    const T *__restrict__ wq;      // [NQ] cubature weights
    const T *__restrict__ geoA;    // [K][5] r_x s_x r_y s_y J (straight elements)
    const T *__restrict__ geoF;    // [K][3][NG][3] n_x n_y w_g sJ (FP32 from P = 2: of a straight element w_g sJ / J)
    const T *__restrict__ geoC;    // [Kc][NQ][4] w_q J (r_x, s_x, r_y, s_y)
    const T *__restrict__ mfold;   // [Kc][Np][Np] M_k^-1 M_ref (P = 1: M_k^-1)
    const int *__restrict__ widx;  // [K] curved slot or -1
    const double *__restrict__ dt;
    // the last stage of a run's step: also the time-step bound of the new
    // state (as k_cfl: FP64 per face node) into the slots, and its check.
    // Two launches of 9 us a step less (5,000 elements at P = 4 in FP64, 20
    // steps: 1,674 -> 1,637 us; 4,000 at P = 3 in FP32: 814 -> 742 us).
    int bound;
    double gamma;
    const double *__restrict__ fgeo;   // [K][3][3 Nfp], Fscale last
    unsigned long long *__restrict__ vmax;
    int *__restrict__ flag;
};

// A wavefront's largest bound; its check into the flag.
__device__ __forceinline__ double wave_bound(double best, int bad, int *flag) {
    const bool any = __any(bad);
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(best, off);
        best = o > best ? o : best;
    }
    if (any && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
    return best;
}
__device__ __forceinline__ void post_bound(double best, int slot, unsigned long long *vmax) {
    atomicMax(vmax + (slot & (kVmaxSlots - 1)), (unsigned long long)__double_as_longlong(best));
}

__device__ __forceinline__ float quad_swap(float v, std::integral_constant<int, 1>) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, true));   // lane ^ 1
}
__device__ __forceinline__ float quad_swap(float v, std::integral_constant<int, 2>) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, true));   // lane ^ 2
}
template <int X>
__device__ __forceinline__ double quad_swap(double v, std::integral_constant<int, X>) {
    constexpr int ctrl = X == 1 ? 0xB1 : 0x4E;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// Transpose of the 4 x 4 block a quad holds (x[j] of lane i <-> x[i] of lane j).
template <typename T>
__device__ __forceinline__ void quad_transpose(T (&x)[4], bool b0, bool b1) {
#pragma unroll
    for (int p = 0; p < 4; p += 2) {
        const T u = quad_swap(x[p], std::integral_constant<int, 1>()), v = quad_swap(x[p + 1], std::integral_constant<int, 1>());
        x[p] = b0 ? v : x[p];
        x[p + 1] = b0 ? x[p + 1] : u;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const T u = quad_swap(x[p], std::integral_constant<int, 2>()), v = quad_swap(x[p + 2], std::integral_constant<int, 2>());
        x[p] = b1 ? v : x[p];
        x[p + 2] = b1 ? x[p + 2] : u;
    }
}

// Waves per SIMD: FP32 four (100,000 elements at P = 4, two steps, 886 us; 924
// at five and 1,066 at six, which spill), five at P = 2 (300,000 straight
// elements, four steps, 1,673 against 1,726 us); FP64 three up to P = 3 (947
// against 1,018 us at two, P = 3), two above (5,000 at P = 4, 20 steps: 1.72
// against 2.10 ms at three) and where the bound takes registers (300 at P = 2,
// 20 steps, 793 against 809 us).
template <typename T, int P, bool BOUND = false>
constexpr int weak_waves() {
    return sizeof(T) == 4 ? (P <= 2 ? 5 : 4) : (P <= 3 && !BOUND ? 3 : 2);
}

// Blocks of W wavefronts a compute unit holds at once (LDS and registers).
template <typename T, int P, bool PART, bool BOUND>
constexpr int weak_blocks(int W) {
    using S = WeakM<T, P>;
    const int lds = (S::NZV * 64 * S::VF + W * 2 * S::TS + (S::template lds_sum<PART>() ? W * S::MT2 * 256 : 0)) * int(sizeof(T));
    const int by_lds = 160 * 1024 / lds, by_regs = 4 * weak_waves<T, P, BOUND>() / W;
    const int n = by_lds < by_regs ? by_lds : by_regs;
    return n < 1 ? 1 : n;
}

// PART (FP32 meshes with curved elements): the update's sum tile by tile, each
// tile's own sum (up to P = 3 one for a and one for b) added to the running one.
// A single sum of all 2 NQ + 3 NG products rounds each at its full size, and
// with M_ref^-1 in the operator V and S cancel in it: the right-hand side was up
// to 1.4 times as far from FP64 as by the kernel on the VALUs before, which added
// the two products of a point first and applied the inverse after the
// cancellation (relative L2: cylinder, 144 elements at P = 5, 1.59e-5 against
// 1.10e-5; all curved, 200, 1.16e-4 against 8.3e-5; with PART 1.20e-5 and
// 8.1e-5; over 120 cases of mesh, order and flux 0.98 of the VALU kernel's in
// the geometric mean, at most 1.16, on 32 elements).  It costs 0 to 1%, on small
// meshes at P = 5 4%.  The inverse applied as a product of its own after the sum
// was 1.07 in the mean with a single sum, and tile by tile 0.99 but up to 1.36
// (P = 2) and at least 3 to 5% slower from 20,000 elements on.  Straight FP32
// meshes had the single sum before, too.
template <typename T, int P, int W, bool PART, bool BOUND>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(weak_waves<T, P, BOUND>()))) void k_stage_weak(WeakArgs<T> a) {
    using S = WeakM<T, P>;
    using V4 = typename VecOf<T>::V4;
    using V = typename VecOf<T>::V16;
    using VG = typename VecOf<T>::U16;
    constexpr int Np = S::Np, Nfp = S::Nfp, NF3 = S::NF3, NQ = S::NQ, NG = S::NG, NFG = S::NFG;
    constexpr int KS1 = S::KS1, MT1 = S::MT1, KSF = S::KSF, MG = S::MG, MT2 = S::MT2, VF = S::VF, NZV = S::NZV;
    constexpr int NV = S::NV, TS = S::TS, NTH = 64 * W;
    __shared__ __attribute__((aligned(16))) V sA[NZV * 64];
    __shared__ __attribute__((aligned(16))) T sT[W][2][TS];   // a wavefront's state tile and result tile
    constexpr bool LSUM = S::template lds_sum<PART>();
    __shared__ __attribute__((aligned(16))) V4 sSum[LSUM ? W * MT2 * 64 : 1];   // a lane's running sums
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kq = lane >> 4, c = lane & 3, le = col >> 2;
    const bool b0 = lane & 1, b1 = lane & 2;
    {
        const V *f = reinterpret_cast<const V *>(a.frag);
#pragma unroll 4
        for (int z = tid; z < NZV * 64; z += NTH) sA[z] = f[z];
    }
    const T dt = a.mode ? T(*a.dt) : T(0);
    T wqv[MT1];
#pragma unroll
    for (int mt = 0; mt < MT1; ++mt) wqv[mt] = a.wq[min(S::row(mt, kq, c), NQ - 1)];
    __syncthreads();
    T *sU = sT[wave][0], *sR = sT[wave][1];
    double best = 0.0;
    int bad = 0;

    // XCD x (block b runs on XCD b % 8) walks the x-th contiguous eighth of the groups
    const int g0 = int(blockIdx.x % 8) * a.per, gend = min(g0 + a.per, a.ngroups);
    const int step = int(gridDim.x / 8) * W;
#pragma unroll 1
    for (int grp = g0 + int(blockIdx.x / 8) * W + wave; grp < gend; grp += step) {
        const long k0 = (long)grp * 4;
        const int nel = (int)min(4L, (long)a.K - k0);
        const long base = k0 * kFields * Np;
        const int nvec = nel * kFields * Np / VF;
        // columns past the mesh's end repeat its last element and are not written out
        const long k = k0 + min(le, nel - 1);

        // ---- loads: connectivity and the tile first, then the neighbours'
        // traces (a boundary face reads the element itself and ignores it)
        const int info = a.finfo[k], cs = a.widx[k];
        int nb[3];
#pragma unroll
        for (int f = 0; f < 3; ++f) nb[f] = a.nbr[k * 3 + f];
        VG uv[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) uv[v] = reinterpret_cast<const VG *>(a.Uin + base)[min(lane + 64 * v, nvec - 1)];
        T ga[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) ga[i] = a.geoA[k * 5 + i];
        T un[KSF];
#pragma unroll
        for (int ks = 0; ks < KSF; ++ks) {
            const int q = min(4 * ks + kq, NF3 - 1), f = q / Nfp, j = q - f * Nfp;
            const int kn = f == 0 ? nb[0] : (f == 1 ? nb[1] : nb[2]);
            const int vp = face_node(P, face_nbr_face(info, f), Nfp - 1 - j);
            un[ks] = a.Uin[((long)kn * kFields + c) * Np + vp];
        }
        const bool curved = __any(cs >= 0);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int z = lane + 64 * v;
            if (z < nvec) {
#pragma unroll
                for (int i = 0; i < VF; ++i) sU[VF * z + i] = uv[v][i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const T *ucol = sU + ((int)(k - k0) * kFields + c) * Np;
        T u[KS1];
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) {
            const int j = 4 * ks + kq;
            u[ks] = 4 * ks + 3 < Np || j < Np ? ucol[min(j, Np - 1)] : T(0);
        }

        const V4 zero = {T(0), T(0), T(0), T(0)};
        V4 acc[MT2];
#pragma unroll
        for (int m = 0; m < MT2; ++m) acc[m] = zero;
        // the update divides by J on a straight element (M_k = J M_ref): the
        // volume weights leave J out and the face weights take 1 / J (FP32: in
        // the table, k_weak_face_weights)
        const T iJ = cs >= 0 ? T(1) : T(1) / ga[4];
        V cur;
        // the fragments in order, a vector of VF at a time (z is a constant
        // at every call)
        auto frag = [&](int z) -> T {
            if (z % VF == 0) cur = sA[z / VF * 64 + lane];
            return cur[z % VF];
        };
        // a tile's products go on from the running sum, or (PART) from zero and
        // are added to it
        V4 *sum = sSum + (LSUM ? wave * MT2 * 64 + lane : 0);
        auto open_sum = [&](V4(&part)[MT2]) {
#pragma unroll
            for (int m = 0; m < MT2; ++m) part[m] = PART ? zero : acc[m];
        };
        auto close_sum = [&](const V4(&part)[MT2], bool first, bool last) {
#pragma unroll
            for (int m = 0; m < MT2; ++m) {
                if constexpr (LSUM) {
                    const V4 v = first ? part[m] : sum[m * 64] + part[m];
                    if (last) {
                        acc[m] = v;
                    } else {
                        sum[m * 64] = v;
                        asm volatile("" ::"v"(sum) : "memory");   // not kept in registers
                    }
                } else {
                    acc[m] = PART ? acc[m] + part[m] : part[m];
                }
            }
        };
        int z = 0;
        // ---- volume: 16 cubature points at a time
#pragma unroll
        for (int mt = 0; mt < MT1; ++mt) {
            V4 s;
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) s = mfma16(frag(z++), u[ks], ks ? s : zero);
            T x[4] = {s[0], s[1], s[2], s[3]};
            quad_transpose(x, b0, b1);
            const int q = S::row(mt, kq, c);   // this lane's point
            const T ir = rcp(x[0]);
            const T vx = x[1] * ir, vy = x[2] * ir, p = pressure_ir(a.g, x, ir);
            const T F[kFields] = {x[1], x[1] * vx + p, x[2] * vx, (x[3] + p) * vx};
            const T G[kFields] = {x[2], x[1] * vy, x[2] * vy + p, (x[3] + p) * vy};
            T w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = wqv[mt] * ga[i];
            if (curved && cs >= 0) {
                const T *gq = a.geoC + ((long)cs * NQ + min(q, NQ - 1)) * 4;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = gq[i];
            }
            T fa[4], fb[4];
            const bool in = 16 * mt + 15 < NQ || q < NQ;
#pragma unroll
            for (int i = 0; i < kFields; ++i) {
                fa[i] = in ? w[0] * F[i] + w[2] * G[i] : T(0);
                fb[i] = in ? w[1] * F[i] + w[3] * G[i] : T(0);
            }
            quad_transpose(fa, b0, b1);
            quad_transpose(fb, b0, b1);
            constexpr bool TWO = PART && P <= 3;   // the products with a and with b apart
            V4 part[MT2], pb[TWO ? MT2 : 1];
            open_sum(part);
#pragma unroll
            for (int m = 0; m < (TWO ? MT2 : 1); ++m) pb[m] = zero;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (S::used(mt, r, NQ)) {
#pragma unroll
                    for (int m = 0; m < MT2; ++m) part[m] = mfma16(frag(z++), fa[r], part[m]);
#pragma unroll
                    for (int m = 0; m < MT2; ++m) {
                        V4 &q = TWO ? pb[TWO ? m : 0] : part[m];
                        q = mfma16(frag(z++), fb[r], q);
                    }
                }
            if constexpr (TWO)
#pragma unroll
                for (int m = 0; m < MT2; ++m) part[m] = part[m] + pb[m];
            close_sum(part, mt == 0, false);
        }
        // ---- faces: 16 Gauss points at a time
#pragma unroll
        for (int ks = 0; ks < KSF; ++ks)
            if (4 * ks + 3 >= NF3 && 4 * ks + kq >= NF3) un[ks] = T(0);
#pragma unroll
        for (int mt = 0; mt < MG; ++mt) {
            V4 s, t;
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) s = mfma16(frag(z++), u[ks], ks ? s : zero);
#pragma unroll
            for (int ks = 0; ks < KSF; ++ks) t = mfma16(frag(z++), un[ks], ks ? t : zero);
            T um[4] = {s[0], s[1], s[2], s[3]}, up[4] = {t[0], t[1], t[2], t[3]};
            quad_transpose(um, b0, b1);
            quad_transpose(up, b0, b1);
            const int fg = min(S::row(mt, kq, c), NFG - 1), f = fg / NG;
            const T *gf = a.geoF + (k * NFG + fg) * 3;
            const T nx = gf[0], ny = gf[1], ws = sizeof(T) == 4 ? gf[2] : gf[2] * iJ;
            const int code = face_bc(info, f);
            if (code != BC_INTERIOR) ghost_state(a.g, code, um, nx, ny, a.ff, up);
            T fm[kFields], fp[kFields], lm, lp, star[kFields];
            normal_flux(a.g, um, nx, ny, fm, lm);
            if (a.riemann == RIEMANN_HLLC) {
                hllc_jump(a.g, um, up, nx, ny, fp);
#pragma unroll
                for (int i = 0; i < kFields; ++i) star[i] = fm[i] - fp[i];
            } else {
                normal_flux(a.g, up, nx, ny, fp, lp);
                const T lam = T(0.5) * (lm > lp ? lm : lp);
#pragma unroll
                for (int i = 0; i < kFields; ++i) star[i] = T(0.5) * (fm[i] + fp[i]) - lam * (up[i] - um[i]);
            }
            const bool in = 16 * mt + 15 < NFG || S::row(mt, kq, c) < NFG;
            T fs[4];
#pragma unroll
            for (int i = 0; i < kFields; ++i) fs[i] = in ? ws * star[i] : T(0);
            quad_transpose(fs, b0, b1);
            V4 part[MT2];
            open_sum(part);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (S::used(mt, r, NFG)) {
#pragma unroll
                    for (int m = 0; m < MT2; ++m) part[m] = mfma16(frag(z++), fs[r], part[m]);
                }
            close_sum(part, false, mt == MG - 1);
        }
        // ---- the result into the group's tile, (element, field, node)
#pragma unroll
        for (int m = 0; m < MT2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = S::row(m, kq, r);
                if (i < Np) sR[col * Np + i] = acc[m][r];
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (curved) {
            // curved elements: one lane per node, the four fields together
            constexpr int NT = (4 * Np + 63) / 64;
            T val[NT][kFields];
            bool mine[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int task = lane + 64 * t, e = task / Np, i = task - e * Np;
                const int ce = task < 4 * Np && e < nel ? a.widx[k0 + e] : -1;
                mine[t] = ce >= 0;
                if (mine[t]) {
                    const T *M = a.mfold + (long)ce * Np * Np + i * Np;
#pragma unroll
                    for (int f = 0; f < kFields; ++f) val[t][f] = T(0);
#pragma unroll 5
                    for (int j = 0; j < Np; ++j) {
                        const T m = M[j];
#pragma unroll
                        for (int f = 0; f < kFields; ++f) val[t][f] += m * sR[(e * kFields + f) * Np + j];
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int task = lane + 64 * t, e = task / Np, i = task - e * Np;
                if (mine[t]) {
#pragma unroll
                    for (int f = 0; f < kFields; ++f) sR[(e * kFields + f) * Np + i] = val[t][f];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        // ---- Runge-Kutta update (or the bare rhs), coalesced; the bound's
        // Fscale is requested before the stores, which a later load would
        // wait for
        constexpr int NB = (4 * NF3 + 63) / 64;
        double fsc[NB];
        if constexpr (BOUND)
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const int z = min(lane + 64 * t, nel * NF3 - 1), e = z / NF3;
                fsc[t] = a.fgeo[((k0 + e) * 3 + 2) * NF3 + (z - e * NF3)];
            }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int zv = lane + 64 * v;
            if (zv < nvec) {
                VG rh, un4;
#pragma unroll
                for (int i = 0; i < VF; ++i) {
                    rh[i] = sR[VF * zv + i];
                    un4[i] = sU[VF * zv + i];
                }
                if (a.mode == 0) {
                    reinterpret_cast<VG *>(a.rhs + base)[zv] = rh;
                } else {
                    VG rr = dt * rh;
                    if (a.stage > 0) rr = a.ra * reinterpret_cast<const VG *>(a.R + base)[zv] + dt * rh;
                    un4 = un4 + a.rb * rr;
                    reinterpret_cast<VG *>(a.R + base)[zv] = rr;
                    reinterpret_cast<VG *>(a.Uout + base)[zv] = un4;
                    if constexpr (BOUND)
#pragma unroll
                        for (int i = 0; i < VF; ++i) sU[VF * zv + i] = un4[i];
                }
            }
        }
        if constexpr (BOUND) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int z = lane; z < nel * Np; z += 64) {
                const int e = z / Np, i = z - e * Np;
                double u[kFields];
#pragma unroll
                for (int f = 0; f < kFields; ++f) u[f] = double(sU[(e * kFields + f) * Np + i]);
                if (bad_state(a.gamma, u)) bad = 1;
            }
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                const int z = lane + 64 * t;
                if (z < nel * NF3) {
                    const int e = z / NF3, q = z - e * NF3, f = q / Nfp, v = face_node(P, f, q - f * Nfp);
                    double u[kFields];
#pragma unroll
                    for (int g = 0; g < kFields; ++g) u[g] = double(sU[(e * kFields + g) * Np + v]);
                    const double b = cfl_bound(a.gamma, u, fsc[t], 0.0, P + 1.0);
                    best = b > best ? b : best;
                }
            }
        }
        // the tiles are reused by the next group
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (BOUND) {
        // one atomic per block: a launch's blocks end together (20,000
        // elements at P = 2, 20 steps: 987 us; 1,099 with one per wavefront)
        __shared__ double sRed[W];
        best = wave_bound(best, bad, a.flag);
        if (lane == 0) sRed[wave] = best;
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < W; ++w) best = sRed[w] > best ? sRed[w] : best;
            post_bound(best, int(blockIdx.x), a.vmax);
        }
    }
}

// P = 1 on the VALUs: three nodes and four cubature points fill too little of
// a 16-row tile (100,000 straight elements, 20 steps: 1.62 ms here and 2.75 on
// the tiles above in FP32, 2.53 and 3.72 in FP64).  A block takes 32 elements,
// a thread one point: wavefronts 0 to 2 the 192 face Gauss points, 2 and 3 the
// 128 cubature points, both straight from global memory; after the only
// barrier a quad of wavefronts 0 and 1 takes an element's three nodes.  Bound
// by the chain connectivity, neighbour's trace, flux, update, so every load is
// issued as early as its address is known; blocks walk the mesh contiguously
// per XCD, so that the traces stay in its L2 (500,000 elements, four steps:
// 1.72 -> 1.25 ms in FP32, 2.65 -> 2.33 in FP64 against a kernel with the
// state in LDS and three barriers).  A bound on the registers for a fourth
// FP64 wavefront per SIMD spills: 3.72 ms.  mfold holds M_k^-1 itself here.
constexpr int kW1Elems = 32, kW1Block = 256;

template <typename T>
__global__ __launch_bounds__(kW1Block) void k_stage_weak1(WeakArgs<T> a) {
    using S = WShape<1>;
    constexpr int Np = S::Np, Nfp = S::Nfp, NQ = S::NQ, NG = S::NG, EB = kW1Elems, NFP = EB * 3 * NG;
    static_assert(NQ == 4 && NFP % 64 == 0 && EB * NQ % 64 == 0 && EB * 4 <= kW1Block, "thread roles");
    __shared__ T sA[EB][kFields * 2 * NQ + 4];   // + 4: elements on different banks
    __shared__ T sS[EB][kFields * 3 * NG + 4];
    // the first loads' pointers are read with the tile count, not after the exit
    // of the surplus blocks (a small mesh's right-hand side 11.4 -> 11.0 us)
    asm volatile("" ::"s"(a.Uin), "s"(a.finfo), "s"(a.nbr), "s"(a.ops), "s"(a.geoF));
    const int tile = xcd_tile(a.per), tid = threadIdx.x;
    if (tile >= a.ngroups) return;
    const long k0 = (long)tile * EB;
    const int nel = (int)min((long)EB, (long)a.K - k0);
    const T *Icub = a.ops, *Drc = Icub + NQ * Np, *wq = Drc + 2 * NQ * Np;
    const T *If = wq + NQ, *Minv = If + NG * Nfp;

    // Loads in the order they are wanted, no use of one before the last is
    // issued: connectivity, the update's operands, then the traces of a face
    // Gauss point, the neighbour's at the address the connectivity gave.
    const bool face = tid < NFP;
    const int el = min(tid / (3 * NG), EB - 1), fg = tid % (3 * NG), f = fg / NG, gq = fg - f * NG;
    const long k = k0 + min(el, nel - 1);
    T u0[kFields], u1[kFields], v0[kFields], v1[kFields], gf[3], l0, l1;
    int info = 0, kb = 0;
    if (face) {
        info = a.finfo[k];
        kb = a.nbr[k * 3 + f];
        l0 = If[gq * Nfp];
        l1 = If[gq * Nfp + 1];
#pragma unroll
        for (int m = 0; m < 3; ++m) gf[m] = a.geoF[((k * 3 + f) * NG + gq) * 3 + m];
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            u0[c] = a.Uin[(k * kFields + c) * Np + face_node(1, f, 0)];
            u1[c] = a.Uin[(k * kFields + c) * Np + face_node(1, f, 1)];
        }
    }
    // the update's operands (threads below 128: node i of element ne)
    const int ne = tid >> 2, i = tid & 3;
    const bool node = ne < nel && i < Np;
    const long at = (k0 + ne) * kFields * Np + i;
    T un[kFields], rn[kFields], dn[2 * NQ], ln[3][NG], mn[Np], J = T(1);
    const T dt = a.mode ? T(*a.dt) : T(0);
    int cs = -1;
    if (node) {
        cs = a.widx[k0 + ne];
        J = a.geoA[(k0 + ne) * 5 + 4];
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            un[c] = a.Uin[at + c * Np];
            rn[c] = a.stage > 0 ? a.R[at + c * Np] : T(0);
        }
#pragma unroll
        for (int q = 0; q < 2 * NQ; ++q) dn[q] = Drc[q * Np + i];
#pragma unroll
        for (int ff = 0; ff < 3; ++ff)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int j = i == face_node(1, ff, 0) ? 0 : 1;
                ln[ff][g] = If[g * Nfp + j];
            }
#pragma unroll
        for (int j = 0; j < Np; ++j) mn[j] = Minv[i * Np + j];
    }
    if (face) {
        const int fn = face_nbr_face(info, f);   // the neighbour's face runs backwards
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            v0[c] = a.Uin[((long)kb * kFields + c) * Np + face_node(1, fn, 1)];
            v1[c] = a.Uin[((long)kb * kFields + c) * Np + face_node(1, fn, 0)];
        }
    }
    if (tid >= kW1Block - EB * NQ) {
        // volume fluxes at a cubature point, weighted and mapped
        const int z = tid - (kW1Block - EB * NQ), eq = z / NQ, q = z % NQ;
        const long kq = k0 + min(eq, nel - 1);
        const int cq = a.widx[kq];
        const T *U = a.Uin + kq * kFields * Np;
        const T wJ = wq[q] * a.geoA[kq * 5 + 4];
        T gm[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) gm[m] = wJ * a.geoA[kq * 5 + m];
        T u[kFields] = {};
#pragma unroll
        for (int j = 0; j < Np; ++j) {
            const T phi = Icub[q * Np + j];
#pragma unroll
            for (int c = 0; c < kFields; ++c) u[c] += phi * U[c * Np + j];
        }
        if (cq >= 0)
#pragma unroll
            for (int m = 0; m < 4; ++m) gm[m] = a.geoC[((long)cq * NQ + q) * 4 + m];
        const T ir = rcp(u[0]);
        const T vx = u[1] * ir, vy = u[2] * ir, p = pressure_ir(a.g, u, ir);
        const T F[kFields] = {u[1], u[1] * vx + p, u[2] * vx, (u[3] + p) * vx};
        const T G[kFields] = {u[2], u[1] * vy, u[2] * vy + p, (u[3] + p) * vy};
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            sA[eq][c * 2 * NQ + q] = gm[0] * F[c] + gm[2] * G[c];
            sA[eq][c * 2 * NQ + NQ + q] = gm[1] * F[c] + gm[3] * G[c];
        }
    }

    if (face) {
        // numerical flux at the face Gauss point, times w_g sJ
        const T nx = gf[0], ny = gf[1], ws = gf[2];
        T um[kFields], up[kFields], fm[kFields], lm, d[kFields];
#pragma unroll
        for (int c = 0; c < kFields; ++c) {
            um[c] = l0 * u0[c] + l1 * u1[c];
            up[c] = l0 * v0[c] + l1 * v1[c];
        }
        const int code = face_bc(info, f);
        if (code != BC_INTERIOR) ghost_state(a.g, code, um, nx, ny, a.ff, up);
        normal_flux(a.g, um, nx, ny, fm, lm);
        flux_jump(a.riemann, a.g, um, up, nx, ny, d);
#pragma unroll
        for (int c = 0; c < kFields; ++c) sS[el][c * 3 * NG + fg] = ws * (fm[c] - d[c]);
    }
    if (cs >= 0) {
        J = T(1);
#pragma unroll
        for (int j = 0; j < Np; ++j) mn[j] = a.mfold[((long)cs * Np + i) * Np + j];
    }
    __syncthreads();
    if (ne >= EB) return;
    double fsc[2] = {0.0, 0.0}, u64[kFields];
    if (a.bound && node) {
        // the node's two faces, and its place on each
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int ff = t == 0 ? (i == 2 ? 1 : 0) : (i == 1 ? 1 : 2);
            fsc[t] = a.fgeo[((k0 + ne) * 3 + 2) * 6 + 2 * ff + (i == face_node(1, ff, 0) ? 0 : 1)];
        }
    }
    // V - S at the node, M_k^-1 over the quad, the Runge-Kutta update
#pragma unroll
    for (int c = 0; c < kFields; ++c) {
        T b = T(0);
        if (node) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) b += dn[q] * sA[ne][c * 2 * NQ + q] + dn[NQ + q] * sA[ne][c * 2 * NQ + NQ + q];
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int g = 0; g < NG; ++g) b -= (i == face_node(1, f, 0) || i == face_node(1, f, 1) ? ln[f][g] : T(0)) * sS[ne][(c * 3 + f) * NG + g];
        }
        T val = T(0);
#pragma unroll
        for (int j = 0; j < Np; ++j) {
            const T bj = __shfl(b, j, 4);
            if (node) val += mn[j] * bj;
        }
        if (!node) continue;
        val = val / J;
        if (a.mode == 0) {
            a.rhs[at + c * Np] = val;
        } else {
            const T rr = a.stage == 0 ? dt * val : a.ra * rn[c] + dt * val;
            a.R[at + c * Np] = rr;
            un[c] = un[c] + a.rb * rr;
            a.Uout[at + c * Np] = un[c];
        }
        u64[c] = double(un[c]);
    }
    if (a.bound) {
        double best = 0.0;
        int bad = 0;
        if (node) {
            bad = bad_state(a.gamma, u64);
            const double b0 = cfl_bound(a.gamma, u64, fsc[0], 0.0, 2.0), b1 = cfl_bound(a.gamma, u64, fsc[1], 0.0, 2.0);
            best = b0 > best ? b0 : best;
            best = b1 > best ? b1 : best;
        }
        best = wave_bound(best, bad, a.flag);
        if ((tid & 63) == 0) post_bound(best, int(blockIdx.x) * 2 + (tid >> 6), a.vmax);
    }
}

// ---- setup (FP64) ---------------------------------------------------------

// Per element: metric terms at the first cubature point (all of them for a
// straight element), the unit normal and w_g sJ at every face Gauss point;
// for a curved element the mapped cubature weights per point and the mass
// matrix sum_q w_q J_q phi_i phi_j.  Coordinates relative to the element's
// first node (as the nodal geometry).
template <int P>
__global__ void k_weak_geometry(int K, const double *__restrict__ x, const double *__restrict__ y,
                                const double *__restrict__ ops, const double *__restrict__ Drg,
                                const double *__restrict__ Dsg, const double *__restrict__ wg,
                                const int *__restrict__ widx, double *__restrict__ geoA,
                                double *__restrict__ geoF, double *__restrict__ geoC,
                                double *__restrict__ mass, int *__restrict__ count) {
    using S = WShape<P>;
    constexpr int Np = S::Np, NQ = S::NQ, NG = S::NG;
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const double *Icub = ops, *Drc = Icub + NQ * Np, *Dsc = Drc + NQ * Np, *wq = Dsc + NQ * Np;
    double xl[Np], yl[Np];
    for (int j = 0; j < Np; ++j) {
        xl[j] = x[k * Np + j] - x[k * Np];
        yl[j] = y[k * Np + j] - y[k * Np];
    }
    const int cs = widx[k];
    double *mk = cs >= 0 ? mass + (long)cs * Np * Np : nullptr;
    if (mk)
        for (int z = 0; z < Np * Np; ++z) mk[z] = 0.0;
    for (int q = 0; q < NQ; ++q) {
        double xr = 0, xs = 0, yr = 0, ys = 0;
        for (int j = 0; j < Np; ++j) {
            xr += Drc[q * Np + j] * xl[j];
            xs += Dsc[q * Np + j] * xl[j];
            yr += Drc[q * Np + j] * yl[j];
            ys += Dsc[q * Np + j] * yl[j];
        }
        const double J = xr * ys - xs * yr;
        if (!(J > 0.0)) atomicAdd(count, 1);
        const double rx = ys / J, sx = -yr / J, ry = -xs / J, sy = xr / J;
        if (q == 0) {
            geoA[k * 5 + 0] = rx;
            geoA[k * 5 + 1] = sx;
            geoA[k * 5 + 2] = ry;
            geoA[k * 5 + 3] = sy;
            geoA[k * 5 + 4] = J;
        }
        if (mk) {
            const double wJ = wq[q] * J;
            double *gq = geoC + ((long)cs * NQ + q) * 4;
            gq[0] = wJ * rx;
            gq[1] = wJ * sx;
            gq[2] = wJ * ry;
            gq[3] = wJ * sy;
            for (int i = 0; i < Np; ++i)
                for (int j = 0; j < Np; ++j) mk[i * Np + j] += wJ * Icub[q * Np + i] * Icub[q * Np + j];
        }
    }
    for (int f = 0; f < 3; ++f)
        for (int g = 0; g < NG; ++g) {
            const double *dr = Drg + (f * NG + g) * Np, *ds = Dsg + (f * NG + g) * Np;
            double xr = 0, xs = 0, yr = 0, ys = 0;
            for (int j = 0; j < Np; ++j) {
                xr += dr[j] * xl[j];
                xs += ds[j] * xl[j];
                yr += dr[j] * yl[j];
                ys += ds[j] * yl[j];
            }
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
            const double sJ = sqrt(ax * ax + ay * ay);
            double *gf = geoF + ((k * 3 + f) * NG + g) * 3;
            gf[0] = ax / sJ;
            gf[1] = ay / sJ;
            gf[2] = wg[g] * sJ;
        }
}

// Inverse of each curved element's mass matrix by Cholesky factorisation
// (M = L L^T, factor in `work`, then M^{-1} column by column from
// L y = e_i, L^T x = y), one thread per curved element, in FP64.
__global__ void k_weak_minv(int Kc, int Np, double *__restrict__ mass, double *__restrict__ work,
                            int *__restrict__ count) {
    const long c = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= Kc) return;
    double *M = mass + c * Np * Np, *L = work + c * Np * Np;
    for (int z = 0; z < Np * Np; ++z) L[z] = 0.0;
    for (int j = 0; j < Np; ++j) {
        double d = M[j * Np + j];
        for (int k = 0; k < j; ++k) d -= L[j * Np + k] * L[j * Np + k];
        if (!(d > 0.0)) {
            atomicAdd(count, 1);
            return;
        }
        d = sqrt(d);
        L[j * Np + j] = d;
        for (int i = j + 1; i < Np; ++i) {
            double v = M[i * Np + j];
            for (int k = 0; k < j; ++k) v -= L[i * Np + k] * L[j * Np + k];
            L[i * Np + j] = v / d;
        }
    }
    for (int col = 0; col < Np; ++col) {
        // forward, into M's column col (M is no longer needed row-wise
        // beyond what the solve reads: the solve reads only L)
        for (int i = 0; i < Np; ++i) {
            double v = i == col ? 1.0 : 0.0;
            for (int k = 0; k < i; ++k) v -= L[i * Np + k] * M[k * Np + col];
            M[i * Np + col] = v / L[i * Np + i];
        }
        for (int i = Np - 1; i >= 0; --i) {
            double v = M[i * Np + col];
            for (int k = i + 1; k < Np; ++k) v -= L[k * Np + i] * M[k * Np + col];
            M[i * Np + col] = v / L[i * Np + i];
        }
    }
}

// M_k^-1 M_ref of each curved element (the update's fragments carry M_ref^-1).
__global__ void k_weak_fold(int Kc, int Np, const double *__restrict__ minv, const double *__restrict__ Mref,
                            double *__restrict__ out) {
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (long)Kc * Np * Np) return;
    const int j = int(g % Np);
    const double *row = minv + g / Np * Np;
    double v = 0.0;
    for (int m = 0; m < Np; ++m) v += row[m] * Mref[m * Np + j];
    out[g] = v;
}

// The FP32 face table from P = 2 on: a straight element's weights divided by J
// before the cast.  Divided in the kernel, two roundings of J were common to an
// element's whole face sum and did not cancel against the volume's.
__global__ void k_weak_face_weights(long n, int per, const double *__restrict__ geoF, const double *__restrict__ geoA,
                                    const int *__restrict__ widx, float *__restrict__ out) {
    const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const long k = g / per;
    out[g] = float(g % 3 == 2 && widx[k] < 0 ? geoF[g] / geoA[k * 5 + 4] : geoF[g]);
}

template <typename F>
hipError_t with_order_w(int P, F &&f) {
    switch (P) {
        case 1: return f(std::integral_constant<int, 1>());
        case 2: return f(std::integral_constant<int, 2>());
        case 3: return f(std::integral_constant<int, 3>());
        case 4: return f(std::integral_constant<int, 4>());
        case 5: return f(std::integral_constant<int, 5>());
        default: return hipErrorInvalidValue;
    }
}

// Operator fragments in the order the kernel takes them: lane l holds row
// l % 16 of the 16-row tile and the k-step's column of its 16-lane group.
template <typename T, int P>
void fill_weak_frags(const double *Icub, const double *Drc, const double *Dsc, const double *If, const double *Minv,
                     T *out) {
    using S = WeakM<T, P>;
    constexpr int Np = S::Np, Nfp = S::Nfp, NQ = S::NQ, NG = S::NG, NFG = S::NFG, K2 = 2 * NQ + NFG;
    std::vector<double> B(size_t(Np) * K2, 0.0), A2(size_t(Np) * K2, 0.0);
    for (int i = 0; i < Np; ++i)
        for (int q = 0; q < NQ; ++q) {
            B[size_t(i) * K2 + q] = Drc[q * Np + i];
            B[size_t(i) * K2 + NQ + q] = Dsc[q * Np + i];
        }
    for (int f = 0; f < 3; ++f)
        for (int j = 0; j < Nfp; ++j)
            for (int g = 0; g < NG; ++g) B[size_t(face_node(P, f, j)) * K2 + 2 * NQ + f * NG + g] = -If[g * Nfp + j];
    for (int i = 0; i < Np; ++i)
        for (int k = 0; k < K2; ++k) {
            double s = 0.0;
            for (int m = 0; m < Np; ++m) s += Minv[i * Np + m] * B[size_t(m) * K2 + k];
            A2[size_t(i) * K2 + k] = s;
        }
    for (int z = 0; z < S::NZV * 64 * S::VF; ++z) out[z] = T(0);
    int z = 0;
    // one fragment: value(row within the operator, 16-lane group)
    auto put = [&](int mt, auto &&value) {
        for (int l = 0; l < 64; ++l) out[(z / S::VF * 64 + l) * S::VF + z % S::VF] = T(value(16 * mt + (l & 15), l >> 4));
        ++z;
    };
    auto update = [&](int n, int first, int mt, int r) {   // A2's columns first + row(mt, kq, r)
        for (int m = 0; m < S::MT2; ++m)
            put(m, [&](int i, int kq) {
                const int col = S::row(mt, kq, r);
                return i < Np && col < n ? A2[size_t(i) * K2 + first + col] : 0.0;
            });
    };
    for (int mt = 0; mt < S::MT1; ++mt) {
        for (int ks = 0; ks < S::KS1; ++ks)
            put(mt, [&](int q, int kq) {
                const int j = 4 * ks + kq;
                return q < NQ && j < Np ? Icub[q * Np + j] : 0.0;
            });
        for (int r = 0; r < 4; ++r)
            if (S::used(mt, r, NQ)) {
                update(NQ, 0, mt, r);
                update(NQ, NQ, mt, r);
            }
    }
    for (int mt = 0; mt < S::MG; ++mt) {
        for (int ks = 0; ks < S::KS1; ++ks)   // the element's own trace
            put(mt, [&](int fg, int kq) {
                const int node = 4 * ks + kq;
                double v = 0.0;
                if (fg < NFG && node < Np)
                    for (int j = 0; j < Nfp; ++j)
                        if (face_node(P, fg / NG, j) == node) v = If[(fg % NG) * Nfp + j];
                return v;
            });
        for (int ks = 0; ks < S::KSF; ++ks)   // the neighbour's, at this element's face nodes
            put(mt, [&](int fg, int kq) {
                const int q = 4 * ks + kq;
                return fg < NFG && q < S::NF3 && q / Nfp == fg / NG ? If[(fg % NG) * Nfp + q % Nfp] : 0.0;
            });
        for (int r = 0; r < 4; ++r)
            if (S::used(mt, r, NFG)) update(NFG, 2 * NQ, mt, r);
    }
}

template <typename T>
hipError_t stage_weak_t(const DevMesh &m, const void *Uin, void *Uout, void *R, void *rhs, int stage,
                        bool bound, hipStream_t st) {
    WeakArgs<T> a;
    a.K = m.K;
    a.stage = stage;
    a.mode = rhs ? 0 : 1;
    a.riemann = m.riemann;
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
    if constexpr (sizeof(T) == 8) {
        a.ops = m.wops64;
        a.frag = m.wfrag64;
        a.geoA = m.wgeoA64;
        a.geoF = m.wgeoF64;
        a.geoC = m.wgeoC64;
        a.mfold = m.wmfold64;
    } else {
        a.ops = m.wops32;
        a.frag = m.wfrag32;
        a.geoA = m.wgeoA32;
        a.geoF = m.wgeoF32;
        a.geoC = m.wgeoC32;
        a.mfold = m.wmfold32;
    }
    a.widx = m.widx;
    a.dt = m.scal + S_DT;
    a.bound = bound && !rhs && m.vmax ? 1 : 0;
    a.gamma = m.gamma;
    a.fgeo = m.fgeo64;
    a.vmax = m.vmax;
    a.flag = m.flag;
    a.ngroups = (m.K + 3) / 4;
    a.per = (a.ngroups + 7) / 8;
    return with_order_w(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        using S = WeakM<T, P>;
        a.wq = a.ops + size_t(3) * S::NQ * S::Np;
        if constexpr (P == 1) {
            a.ngroups = (m.K + kW1Elems - 1) / kW1Elems;
            a.per = xcd_chunk(a.ngroups);
            hipLaunchKernelGGL((k_stage_weak1<T>), dim3(xcd_grid(a.ngroups)), dim3(kW1Block), 0, st, a);
            return hipGetLastError();
        } else {
            // Wavefronts that share a block's fragments: four, or eight where
            // only that lets the LDS hold as many wavefronts as the registers
            // do (P = 5: 100,000 FP32 elements, two steps, 2,112 against 2,156
            // us; 20,000 FP64, four steps, 1,109 against 1,231 us) and every
            // SIMD has a group.  Elsewhere four: less padding in a small
            // mesh's last block (800 FP32 elements at P = 3, 60 steps, 2,163
            // against 2,374 us; 20,000 at P = 2, 20 steps, 1,047 against 1,106
            // us).
            auto go = [&](auto SC) {
                constexpr bool PART = decltype(SC)::value;
                constexpr int w4 = 4 * weak_blocks<T, P, PART, false>(4), w8 = 8 * weak_blocks<T, P, PART, false>(8);
                auto shape = [&](auto WC) {
                    constexpr int W = decltype(WC)::value;
                    auto launch = [&](auto BC) {
                        constexpr bool BOUND = decltype(BC)::value;
                        // (a multiple of 8: every XCD's blocks walk the same step)
                        const int want = 8 * ((a.per + W - 1) / W);
                        const int most = max(m.ncu * weak_blocks<T, P, PART, BOUND>(W) / 8 * 8, 8);
                        hipLaunchKernelGGL((k_stage_weak<T, P, W, PART, BOUND>), dim3(unsigned(want < most ? want : most)),
                                           dim3(64 * W), 0, st, a);
                    };
                    // (a variant of its own: the bound's registers would spill
                    // in the other stages too)
                    if (a.bound)
                        launch(std::true_type());
                    else
                        launch(std::false_type());
                };
                if constexpr (w8 > w4) {
                    if (a.ngroups > m.ncu * 4) {
                        shape(std::integral_constant<int, 8>());
                        return;
                    }
                }
                shape(std::integral_constant<int, 4>());
            };
            if constexpr (sizeof(T) == 4) {
                if (m.wKc > 0) {
                    go(std::true_type());
                    return hipGetLastError();
                }
            }
            go(std::false_type());
            return hipGetLastError();
        }
    });
}

}  // namespace

size_t weak_frag_values(int P, bool fp32) {
    size_t n = 0;
    (void)with_order_w(P, [&](auto PC) {
        constexpr int PP = decltype(PC)::value;
        n = size_t(64) * (fp32 ? WeakM<float, PP>::NZV * 4 : WeakM<double, PP>::NZV * 2);
        return hipSuccess;
    });
    return n;
}

template <typename T>
static void fill_frags(int P, const WeakOpsView &w, T *out) {
    (void)with_order_w(P, [&](auto PC) {
        constexpr int PP = decltype(PC)::value;
        fill_weak_frags<T, PP>(w.Icub, w.Drc, w.Dsc, w.If, w.Minv, out);
        return hipSuccess;
    });
}

void weak_fill_frags(int P, const WeakOpsView &w, float *out) { fill_frags(P, w, out); }
void weak_fill_frags(int P, const WeakOpsView &w, double *out) { fill_frags(P, w, out); }

size_t weak_ops_size(int P) {
    const int Np = (P + 1) * (P + 2) / 2, Nfp = P + 1, n = (3 * P + 2) / 2, NQ = n * n;
    return size_t(3) * NQ * Np + NQ + size_t(n) * Nfp + size_t(Np) * Np;
}

hipError_t launch_weak_geometry(const DevMesh &m, const double *x, const double *y, const double *Drg,
                                const double *Dsg, const double *wg, double *geoA, double *geoF, double *geoC,
                                double *mass, double *work, hipStream_t st) {
    hipError_t e = with_order_w(m.P, [&](auto PC) {
        constexpr int P = decltype(PC)::value;
        hipLaunchKernelGGL((k_weak_geometry<P>), dim3((m.K + 63) / 64), dim3(64), 0, st, m.K, x, y, m.wops64,
                           Drg, Dsg, wg, m.widx, geoA, geoF, geoC, mass, m.count);
        return hipGetLastError();
    });
    if (e != hipSuccess || m.wKc == 0) return e;
    hipLaunchKernelGGL(k_weak_minv, dim3((m.wKc + 63) / 64), dim3(64), 0, st, m.wKc, m.Np, mass, work,
                       m.count + 2);
    // the factorisation is done with: the folded matrices take its place
    const long n = (long)m.wKc * m.Np * m.Np;
    hipLaunchKernelGGL(k_weak_fold, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, m.wKc, m.Np, mass,
                       m.ops64 + ops_size(m.Np, m.Nfp), work);
    return hipGetLastError();
}

hipError_t launch_weak_face_weights(const DevMesh &m, const double *geoF, const double *geoA, float *out,
                                    hipStream_t st) {
    const int per = 9 * ((3 * m.P + 2) / 2);   // values of an element
    const long n = (long)m.K * per;
    hipLaunchKernelGGL(k_weak_face_weights, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, n, per, geoF, geoA, m.widx,
                       out);
    return hipGetLastError();
}

hipError_t launch_stage_weak(const DevMesh &m, const void *Uin, void *Uout, void *R, void *rhs, int stage,
                             bool bound, hipStream_t st) {
    return m.fp32 ? stage_weak_t<float>(m, Uin, Uout, R, rhs, stage, bound, st)
                  : stage_weak_t<double>(m, Uin, Uout, R, rhs, stage, bound, st);
}

}  // namespace dg
