// amrmg_kernels.hip -- HIP kernels for gfx950 of the composite AMR multigrid
// path (arXiv:1812.03689): CIC deposit and gather, charge tagging, the FP64
// composite residual with flux matching (Alg. 1; Eqs. lap_flux_differencing,
// coarse_fluxes, flux_differencing), coarse-fine ghost interpolation (Eq.
// 2d_lagrange, Tab. bit_pattern), smoothers, restriction, prolongation and
// coarse-fine residual update of the V-cycle (Alg. 3), the CG bottom solve,
// average down and E = -grad phi (Alg. 2).
//
// Every stencil kernel works on 8^3 bricks (one workgroup per brick, or four
// bricks per workgroup where a thread owns a coarse cell).  The brick a
// workgroup takes is remapped so that each of the chip's eight XCDs (which
// receive workgroups round robin) walks a contiguous run of bricks and keeps
// neighbouring halos in its own L2.  Arithmetic is FP64; the cycle arrays are
// stored in T (float in mixed precision, double otherwise).
#include <hip/hip_ext.h>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <hip/hip_runtime.h>

#include "amrmg_box.hpp"
#include "amrmg_internal.hpp"
#include "amrmg_kernels.hpp"

namespace amrmg {

// step-1 weights of the coarse-fine ghost, already multiplied by the step-2
// weight 8/15 of the coarse node: [pattern 0..13][quadrant 0..3][node 0..8]
__constant__ double c_cfw[14 * 4 * 9];

// optional kernel-execution timestamps for the next launch (profiling)
static thread_local hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;

void set_launch_timing(hipEvent_t start, hipEvent_t stop)
{
    g_ev_start = start;
    g_ev_stop = stop;
}

bool launch_timing_pending() { return g_ev_start != nullptr; }

#define AMRMG_LAUNCH(kernel, grid, block, shmem, stream, ...)                                              \
    do {                                                                                                   \
        if (g_ev_start) {                                                                                  \
            hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, g_ev_start, g_ev_stop, 0, __VA_ARGS__); \
            g_ev_start = g_ev_stop = nullptr;                                                              \
        } else {                                                                                           \
            hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);                           \
        }                                                                                                  \
    } while (0)

hipError_t upload_cf_weights(const double *w)
{
    return hipMemcpyToSymbol(HIP_SYMBOL(c_cfw), w, sizeof(double) * 14 * 4 * 9, 0, hipMemcpyHostToDevice);
}

// workgroup i -> logical index, so that XCD (i mod 8) gets one contiguous run
__device__ __forceinline__ int xcd_remap(int i, int n)
{
    int x = i & 7, q = n >> 3, r = n & 7;
    return x * q + (x < r ? x : r) + (i >> 3);
}

// brick of workgroup i in a range or in an explicit list
__device__ __forceinline__ int pick_brick(int b0, int nb, const int32_t *list, int i)
{
    int k = xcd_remap(i, nb);
    return list ? list[k] : b0 + k;
}

__device__ __forceinline__ void transverse(int d, int &du, int &dv)
{
    du = (d == 0) ? 1 : 0;
    dv = (d == 2) ? 1 : 2;
}

// Two cells adjacent along x in one row of a box: one 16-byte access (8-byte
// alignment is enough for a global access on CDNA).
typedef double dpair __attribute__((ext_vector_type(2)));
typedef dpair dpair_a8 __attribute__((aligned(8)));

// a / h, correctly rounded, from rh = 1/h rounded to nearest: with the
// remainder a - h (a rh) exact in one fma, the corrected quotient is the
// rounded one (Markstein's theorem), in 3 instructions instead of the
// division's dozen.  Only where the quotient, rh and the remainder stay in
// the normal range: not for infinities, an overflowing quotient or a
// subnormal h (dep_level scales the domain's extents for that).
__device__ __forceinline__ double div_by(double a, double h, double rh)
{
    const double q = a * rh;
    return fma(fma(-q, h, a), rh, q);
}

// order the LDS accesses of a wavefront among its lanes
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// accessors: value of local cell l of brick b
// ---------------------------------------------------------------------------
template <class T>
struct BrickAcc {
    const T *u;
    __device__ double operator()(int b, const int *l) const
    {
        return (double)u[(size_t)b * BRICK_CELLS + l[0] + 8 * l[1] + 64 * l[2]];
    }
};

struct OffsetAcc {  // contiguous double slab starting at brick b0
    const double *u;
    int b0;
    __device__ double operator()(int b, const int *l) const
    {
        return u[(size_t)(b - b0) * BRICK_CELLS + l[0] + 8 * l[1] + 64 * l[2]];
    }
};

// The neighbour value that cell l of brick b sees across face (d, s), written
// as a * u_c + bv:
//   same level (in this brick or the face neighbour brick): a = 0, bv = u_nb
//   physical boundary: Dirichlet ghost 2 g - u_c, a = -1, bv = 2 g (g = 0 when
//     !inhom); Robin ghost (central difference of d phi/dn + phi/d = 0),
//     a = (2 d - h)/(2 d + h), bv = 0 (the level's abnd)
//   coarse-fine face, fine side: ghost = cpart + 2/3 u_c - 1/5 u_in, with
//     cpart the coarse part precomputed per ghost (zero when cp == nullptr):
//     a = 2/3, bv = cpart - u_in / 5.
template <class U>
__device__ __forceinline__ void face_nb(const DevMeta &M, int b, const int *lc, int d, int s, const U &u,
                                        const double *cp_d, const float *cp_f, bool inhom, double &a, double &bv)
{
    int l[3] = {lc[0], lc[1], lc[2]};
    int n = l[d] + s;
    if (n >= 0 && n < BRICK) {
        l[d] = n;
        a = 0.0;
        bv = u(b, l);
        return;
    }
    int f = M.nbr[b * 6 + 2 * d + (s > 0)];
    if (f >= 0) {
        l[d] = (s > 0) ? 0 : BRICK - 1;
        a = 0.0;
        bv = u(f, l);
        return;
    }
    int g = -1 - f;
    int du, dv;
    transverse(d, du, dv);
    int t = l[du] + 8 * l[dv];
    if (g < M.nbc) {
        a = M.lc[M.org[b].w].abnd[d];
        bv = inhom ? 2.0 * M.gbc[(size_t)g * 64 + t] : 0.0;
        return;
    }
    size_t cf = (size_t)(g - M.nbc);
    l[d] -= s;  // the fine cell further inside
    double cpv = cp_d ? cp_d[cf * 64 + t] : (cp_f ? (double)cp_f[cf * 64 + t] : 0.0);
    a = 2.0 / 3.0;
    bv = cpv - 0.2 * u(b, l);
}

template <class T>
struct CpPtr;
template <>
struct CpPtr<double> {
    static __device__ const double *d(const double *p) { return p; }
    static __device__ const float *f(const double *) { return nullptr; }
};
template <>
struct CpPtr<float> {
    static __device__ const double *d(const float *) { return nullptr; }
    static __device__ const float *f(const float *p) { return p; }
};

// sum (op 0) or max (op 1) over a workgroup of up to 1024 threads
__device__ double block_reduce(double v, int op)
{
    __shared__ double sh[16];
    for (int o = 32; o > 0; o >>= 1) {
        double w = __shfl_xor(v, o, 64);
        v = op ? fmax(v, w) : v + w;
    }
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double r = sh[0];
    const int nw = blockDim.x >> 6;
    for (int i = 1; i < nw; ++i) r = op ? fmax(r, sh[i]) : r + sh[i];
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------------------
// LDS tile of one brick: the 8^3 cells plus one halo layer on the six faces
// (edges and corners are never read by the 7-point stencil).  A halo cell
// across a same-level face holds the neighbour's value; across a boundary or
// coarse-fine face it holds bv of the ghost a*u_c + bv, and alpha[face] holds
// a, stored as a - 2 on a boundary face so that its sign tells the kinds
// apart (coarse-fine 2/3 > 0, same level 0, boundary a - 2 < -1 since
// |a| < 1 or a = -1; tile_ab takes the 2 back).  All loads of
// a tile are independent and issued before one barrier.
// ---------------------------------------------------------------------------
constexpr int TE = 10;
__device__ __forceinline__ int tix(int x, int y, int z) { return (x + 1) + TE * ((y + 1) + TE * (z + 1)); }

template <class T>
struct SrcB {  // brick-layout array
    const T *u;
    __device__ double operator()(int b, int c) const { return (double)u[(size_t)b * BRICK_CELLS + c]; }
};
struct SrcZ {
    __device__ double operator()(int, int) const { return 0.0; }
};
// coarse parts of coarse-fine ghosts, by face id and face-local cell
struct CpNone {
    __device__ double operator()(size_t, int) const { return 0.0; }
};
template <class T>
struct CpArr {
    const T *cp;
    __device__ double operator()(size_t cf, int fl) const { return cp ? (double)cp[cf * 64 + fl] : 0.0; }
};
// computed on the spot from the coarse level's cycle array (step 1 of the
// two-step interpolation times 8/15), optionally stored for later sweeps
template <class T>
struct CpInline {
    const DevMeta *M;
    const T *ec;
    T *store;
    __device__ double operator()(size_t cf, int fl) const
    {
        int iu = fl & 7, iv = fl >> 3;
        int m = (iu >> 1) + 4 * (iv >> 1), q = (iu & 1) + 2 * (iv & 1);
        size_t e = cf * 16 + m;
        int pat = M->cf_pat[e];
        const double *W = c_cfw + (pat * 4 + q) * 9;
        double v = 0.0;
        for (int w = 0; w < 9; ++w) v += W[w] * (double)ec[M->cf_idx[e * 9 + w]];
        if (store) store[cf * 64 + fl] = (T)v;
        return v;
    }
};

// NT = threads of the workgroup.  Every load of the tile is issued before the
// first LDS store, so a thread waits for memory once.
template <class S, bool ZERO = false, class CP = CpNone, int NT = 256, class V = double>
__device__ void stage_tile(const DevMeta &M, int b, const S &src, const CP &cp, bool inhom, V *tile, V *alpha)
{
    constexpr int NI = BRICK_CELLS / NT, NH = (384 + NT - 1) / NT;
    double vi[NI], vh[NH], ah[NH];
#pragma unroll
    for (int j = 0; j < NI; ++j) vi[j] = ZERO ? 0.0 : src(b, (int)threadIdx.x + NT * j);
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        const int t = threadIdx.x + NT * j;
        vh[j] = 0.0;
        ah[j] = 0.0;
        if (t >= 384) continue;
        const int f = t >> 6, d = f >> 1;
        const bool plus = f & 1;
        const int fl = t & 63;
        const int nb = M.nbr[b * 6 + f];
        if (nb >= 0) {
            if (!ZERO) {
                int du, dv;
                transverse(d, du, dv);
                int m[3];
                m[du] = fl & 7;
                m[dv] = fl >> 3;
                m[d] = plus ? 0 : 7;
                vh[j] = src(nb, m[0] + 8 * m[1] + 64 * m[2]);
            }
        } else {
            const int g = -1 - nb;
            if (g < M.nbc) {
                ah[j] = M.lc[M.org[b].w].abnd[d] - 2.0;
                vh[j] = inhom ? 2.0 * M.gbc[(size_t)g * 64 + fl] : 0.0;
            } else {
                ah[j] = 2.0 / 3.0;
                vh[j] = cp((size_t)(g - M.nbc), fl);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int c = threadIdx.x + NT * j;
        tile[tix(c & 7, (c >> 3) & 7, c >> 6)] = (V)vi[j];
    }
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        const int t = threadIdx.x + NT * j;
        if (t >= 384) continue;
        const int f = t >> 6, d = f >> 1;
        int du, dv;
        transverse(d, du, dv);
        int l[3];
        l[du] = t & 7;
        l[dv] = (t >> 3) & 7;
        l[d] = (f & 1) ? 8 : -1;
        tile[tix(l[0], l[1], l[2])] = (V)vh[j];
        if ((t & 63) == 0) alpha[f] = (V)ah[j];
    }
    __syncthreads();
}

// Ghost form a * u_c + bv of the neighbour of tile cell (x,y,z) across
// (d, s).  A coarse-fine halo slot holds the coarse part; the -u_in/5 term
// uses the current value of the cell further inside.
template <class V>
__device__ __forceinline__ void tile_ab(const V *tile, const V *alpha, int x, int y, int z, int d, int s, V &a, V &bv)
{
    int l[3] = {x, y, z};
    l[d] += s;
    bv = tile[tix(l[0], l[1], l[2])];
    a = (V)0;
    if (l[d] < 0 || l[d] > 7) {
        a = alpha[2 * d + (s > 0)];
        if (a > (V)0) {
            int in[3] = {x, y, z};
            in[d] -= s;
            bv -= (V)0.2 * tile[tix(in[0], in[1], in[2])];
        } else if (a < (V)0) {
            a += (V)2;  // boundary
        }
    }
}

// ---------------------------------------------------------------------------
// FP64 composite residual (Alg. 1) on a range of bricks of the AMR levels
// ---------------------------------------------------------------------------

// Fine part of the flux through a coarse-fine face, per coarse cell of the
// face: over the four fine cells next to the face, sum (u_f/3 + u_in/5 -
// cpart) with u_in the fine cell further inside and cpart the coarse part of
// the fine cell's ghost; the coarse operator gets -1/(2 h_d^2) times it (the
// flux through the coarse face is the mean of the four fine fluxes).  The
// fine side computes these sums (it holds the fine values) into
// ffs[(F * 6 + face) * 16 + m], F the fine brick, face its face towards the
// coarse cell, m = mu + 4 mv the coarse cell's position on that face; the
// coarse side reads them through the children of its brick and of its face
// neighbours, staged in LDS.

// the sum of coarse cell m of face dir of fine brick F from fine values u
// (brick layout) and the coarse parts c[q] of its four fine ghosts (q = the
// fine cell's offsets along the two face axes, first axis fastest)
template <class U>
__device__ __forceinline__ double face_sum(const U &u, int F, int dir, int m, const double *c)
{
    const int d = dir >> 1;
    const bool plus = dir & 1;
    int du, dv;
    transverse(d, du, dv);
    int l[3], li[3];
    l[d] = plus ? 7 : 0;
    li[d] = plus ? 6 : 1;
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        l[du] = li[du] = 2 * (m & 3) + (q & 1);
        l[dv] = li[dv] = 2 * (m >> 2) + (q >> 1);
        sum += (1.0 / 3.0) * u(F, l[0] + 8 * l[1] + 64 * l[2]) + 0.2 * u(F, li[0] + 8 * li[1] + 64 * li[2]) - c[q];
    }
    return sum;
}

// The row layout of the sweep and the outer residual: one wavefront per
// brick.  Lane (y, z) = (lane & 7, lane >> 3) owns the brick's x-row (y, z):
// its 8 cells, their right-hand sides and, for x = 0 and x = 7, the x halo
// slots stay in registers, so x-neighbours need no LDS.  The rows of the
// brick and the y and z halo rows sit in LDS, row (y', z') for y', z' in
// -1..8 at rows[((y' + 1) + 10 (z' + 1)) * 9]: rows are 9 words apart, so the
// 64 lanes reading the same x of their neighbouring rows fall in different
// banks.  Row r of the brick starts at cell 8 r of its slab, so the global
// row loads and stores are whole coalesced vectors.  A workgroup holds BPW
// bricks (one per wavefront).
constexpr int RW = 10, RS = 9;
__device__ __forceinline__ int rrow(int y, int z) { return ((y + 1) + RW * (z + 1)) * RS; }

template <class T>
struct Row8;
template <>
struct Row8<float> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[8])
    {
        const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
        v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    }
    static __device__ __forceinline__ void store(float *p, const float (&v)[8])
    {
        *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
        *(float4 *)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
};
template <>
struct Row8<double> {
    static __device__ __forceinline__ void load(const double *p, double (&v)[8])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double2 a = *(const double2 *)(p + 2 * i);
            v[2 * i] = a.x, v[2 * i + 1] = a.y;
        }
    }
    static __device__ __forceinline__ void store(double *p, const double (&v)[8])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) *(double2 *)(p + 2 * i) = make_double2(v[2 * i], v[2 * i + 1]);
    }
};

// Composite residual r = rho/eps0 - A_comp phi on uncovered cells (zero on
// covered ones) of a range or list of AMR bricks, from FP64 phi and rho in
// brick layout, written as T in brick layout (r_out) and/or FP64 in the
// caller's layout (r_user), with one partial norm per brick (part[b]).  A
// face towards a covered cell takes the mean of the four fine fluxes through
// it (flux matching), from the fine sums ffs of phi.

// One wavefront per brick, lane (y, z) holding the x-row (y, z) of phi and
// rho in registers and the rows of phi with the y and z halo rows in LDS, as
// the sweep kernel does (rrow); the face kinds and the covered-octant masks
// of the brick and of its face neighbours come through scalar loads.  Each
// lane writes its row of r.  BOTH: also the partial norm of the residual of
// phi = 0 (rho/eps0 and the Dirichlet data alone), in part[n_part + b].
//
// On small hierarchies it is bound by its chain of loads.  The fine sums next
// to covered cells come by half rows (four consecutive sums of one child's
// face); loaded cell
// by cell and face by face, each waiting for its own, they made it 15.0 us on 64^3 + 2 levels (now
// 12.3) and 8.5 on 32^3 + 1 (now 6.1).  A direction at a time, not all: on
// large hierarchies it streams, and its registers must leave five wavefronts
// a SIMD.
template <class T, bool BOTH, int BPW>
__global__ void __launch_bounds__(64 * BPW) k_outer_residual(DevMeta M, int b0, int nb, const double *phib,
                                                             const double *rhob, double inv_eps0,
                                                             const double *cp_phi, T *r_out, double *part, int n_part,
                                                             int norm_p, const int32_t *list, double *const *r_user,
                                                             const double *ffs)
{
    __shared__ double rows_all[BPW][RW * RW * RS];
    __shared__ int kids_all[BPW][56];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int k0 = xcd_remap(blockIdx.x, (nb + BPW - 1) / BPW) * BPW + w;
    const bool active = k0 < nb;
    const int kk = active ? k0 : nb - 1;
    const int b = __builtin_amdgcn_readfirstlane(list ? list[kk] : b0 + kk);
    double *rows = rows_all[w];
    int *kids = kids_all[w];
    const int y = lane & 7, z = lane >> 3;
    const int lev = M.org[b].w;
    const LevelConst L = M.lc[lev];
    const uint32_t cm = M.cmask[b];
    int nbf[6], kind[6];
    uint32_t ncm[6];
    bool any_cov = cm != 0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        nbf[f] = M.nbr[b * 6 + f];
        kind[f] = nbf[f] >= 0 ? 0 : ((-1 - nbf[f]) < M.nbc ? 1 : 2);
        ncm[f] = kind[f] == 0 ? (uint32_t)M.cmask[nbf[f]] : 0u;
        any_cov = any_cov || ncm[f] != 0;
    }
    const size_t rb = (size_t)b * BRICK_CELLS + 8 * lane;
    // every cell covered (wavefront-uniform): r = 0, nothing to load; the
    // wavefront still takes part in the workgroup's barrier
    const bool all_cov = cm == 0xffu;
    // the children of the brick and of its face neighbours, for the fine
    // sums of covered faces: kids[8 f + o] of face neighbour f, kids[48 + o]
    // of the brick (-1 where none); read after the barrier below
    if (any_cov && !all_cov && lane < 56) {
        const int nbl = lane < 48 ? M.nbr[b * 6 + (lane >> 3)] : b;
        kids[lane] = nbl >= 0 ? M.child[nbl * 8 + (lane & 7)] : -1;
    }
    double rv[8], u[8], hs[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 8; ++i) rv[i] = u[i] = 0.0;
    if (!all_cov) {
        Row8<double>::load(rhob + rb, rv);
        Row8<double>::load(phib + rb, u);
    }
    // halo slots: the neighbour's phi, 2 g on the boundary (the Dirichlet
    // data enter here), or the coarse part of the coarse-fine ghost
#pragma unroll
    for (int f = 0; f < 6 && !all_cov; ++f) {
        const int d = f >> 1, md = (f & 1) ? 0 : 7;
        const int uu = lane & 7, vv = lane >> 3;
        if (kind[f] == 0) {
            const int c = d == 0 ? md + 8 * uu + 64 * vv : (d == 1 ? uu + 8 * md + 64 * vv : uu + 8 * vv + 64 * md);
            hs[f] = phib[(size_t)nbf[f] * BRICK_CELLS + c];
        } else if (kind[f] == 1) {
            hs[f] = 2.0 * M.gbc[(size_t)(-1 - nbf[f]) * 64 + lane];
        } else {
            hs[f] = cp_phi[(size_t)(-1 - nbf[f] - M.nbc) * 64 + lane];
        }
    }
    const int rym = rrow(y - 1, z), ryp = rrow(y + 1, z), rzm = rrow(y, z - 1), rzp = rrow(y, z + 1), rme = rrow(y, z);
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[rme + i] = u[i];
    rows[rrow(-1, lane >> 3) + (lane & 7)] = hs[2];
    rows[rrow(8, lane >> 3) + (lane & 7)] = hs[3];
    rows[rrow(lane >> 3, -1) + (lane & 7)] = hs[4];
    rows[rrow(lane >> 3, 8) + (lane & 7)] = hs[5];
    // ghost coefficients and the per-row weights (as in the sweep)
    double ag[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) ag[f] = kind[f] == 1 ? L.abnd[f >> 1] : (kind[f] == 2 ? 2.0 / 3.0 : 0.0);
    const double ih2x = L.ih2[0], ih2y = L.ih2[1], ih2z = L.ih2[2];
    const double aym = y == 0 ? ag[2] : 0.0, ayp = y == 7 ? ag[3] : 0.0;
    const double azm = z == 0 ? ag[4] : 0.0, azp = z == 7 ? ag[5] : 0.0;
    const double wyp = (y == 0 && kind[2] == 2) ? 0.8 : 1.0, wym = (y == 7 && kind[3] == 2) ? 0.8 : 1.0;
    const double wzp = (z == 0 && kind[4] == 2) ? 0.8 : 1.0, wzm = (z == 7 && kind[5] == 2) ? 0.8 : 1.0;
    const double wxp0 = kind[0] == 2 ? 0.8 : 1.0, wxm7 = kind[1] == 2 ? 0.8 : 1.0;
    const double den = ih2y * (2.0 - aym - ayp) + ih2z * (2.0 - azm - azp) + 2.0 * ih2x;
    __syncthreads();
    const int ozy = ((y >> 2) << 1) | ((z >> 2) << 2);  // the row's octants: ozy, ozy | 1
    const bool cov[2] = {((cm >> ozy) & 1) != 0, ((cm >> (ozy | 1)) & 1) != 0};
    double r[8], acc = 0.0, acc0 = 0.0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const double uc = u[x];
        const double xm = x == 0 ? hs[0] : u[x - 1], xp = x == 7 ? hs[1] : u[x + 1];
        const double wxm = x == 7 ? wxm7 : 1.0, wxp = x == 0 ? wxp0 : 1.0;
        const double dc = den - (x == 0 ? ih2x * ag[0] : 0.0) - (x == 7 ? ih2x * ag[1] : 0.0);
        const double ym = rows[rym + x], yp = rows[ryp + x], zm = rows[rzm + x], zp = rows[rzp + x];
        r[x] = rv[x] * inv_eps0 - (dc * uc - (ih2x * (wxm * xm + wxp * xp) + ih2y * (wym * ym + wyp * yp) +
                                              ih2z * (wzm * zm + wzp * zp)));
        if (BOTH) {
            // phi = 0: of the operator only the boundary data stay
            double g = 0.0;
            if (x == 0 && kind[0] == 1) g += ih2x * hs[0];
            if (x == 7 && kind[1] == 1) g += ih2x * hs[1];
            if (y == 0 && kind[2] == 1) g += ih2y * ym;
            if (y == 7 && kind[3] == 1) g += ih2y * yp;
            if (z == 0 && kind[4] == 1) g += ih2z * zm;
            if (z == 7 && kind[5] == 1) g += ih2z * zp;
            const double av = cov[x >> 2] ? 0.0 : fabs(rv[x] * inv_eps0 + g);
            acc0 = norm_p == 2 ? acc0 + av * av : norm_p == 1 ? acc0 + av : fmax(acc0, av);
        }
    }
    if (any_cov && !all_cov) {
        // a face towards a covered cell of this level: the flux through it is
        // the mean of the four fine fluxes (the fine sums), in place of the
        // same-level term ih2 (u_c - u_nb).  Along y and z a whole half of the
        // row (one octant) has the covered neighbour or has not.
#pragma unroll 1
        for (int f = 2; f < 6; ++f) {
            const int d = f >> 1, s = f & 1, q = (d == 1 ? y : z) + (s ? 1 : -1), l = q & 7;
            const double ih2 = d == 1 ? ih2y : ih2z;
            const bool inside = q == l;
            const int qo = d == 1 ? ((l >> 2) << 1) | ((z >> 2) << 2) : ((y >> 2) << 1) | ((l >> 2) << 2);
            const uint32_t nm = inside ? cm : (f == 2 ? ncm[2] : f == 3 ? ncm[3] : f == 4 ? ncm[4] : ncm[5]);
            const double *nrow = rows + (d == 1 ? (s ? ryp : rym) : (s ? rzp : rzm));
            bool on[2];
            double2 a[2], c[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                on[h] = !cov[h] && ((nm >> (qo | h)) & 1);
                a[h] = c[h] = make_double2(0.0, 0.0);
                if (on[h]) {
                    // the child covering the neighbours: of this brick, or of the face neighbour
                    const int F = kids[(inside ? 48 : 8 * f) + (qo | h)];
                    const double2 *p = (const double2 *)(ffs + ((size_t)F * 6 + 2 * d + 1 - s) * 16 +
                                                         4 * ((d == 1 ? z : y) & 3));
                    a[h] = p[0], c[h] = p[1];
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (on[h]) {
                    const double fs[4] = {a[h].x, a[h].y, c[h].x, c[h].y};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        r[4 * h + i] += ih2 * (u[4 * h + i] - nrow[4 * h + i]);
                        r[4 * h + i] += 0.5 * ih2 * fs[i];
                    }
                }
        }
        // along x: the cells next to the other half, and the row's ends
        const int m = (y & 3) + 4 * (z & 3);
        const bool in3 = !cov[0] && cov[1], in4 = cov[0] && !cov[1];
        const bool end0 = !cov[0] && ((ncm[0] >> (ozy | 1)) & 1), end7 = !cov[1] && ((ncm[1] >> ozy) & 1);
        double fi = 0.0, f0 = 0.0, f7 = 0.0;
        if (in3) fi = ffs[((size_t)kids[48 + (ozy | 1)] * 6 + 0) * 16 + m];
        if (in4) fi = ffs[((size_t)kids[48 + ozy] * 6 + 1) * 16 + m];
        if (end0) f0 = ffs[((size_t)kids[ozy | 1] * 6 + 1) * 16 + m];
        if (end7) f7 = ffs[((size_t)kids[8 + ozy] * 6 + 0) * 16 + m];
        if (end0) {
            r[0] += ih2x * (u[0] - hs[0]);
            r[0] += 0.5 * ih2x * f0;
        }
        if (in3) {
            r[3] += ih2x * (u[3] - u[4]);
            r[3] += 0.5 * ih2x * fi;
        }
        if (in4) {
            r[4] += ih2x * (u[4] - u[3]);
            r[4] += 0.5 * ih2x * fi;
        }
        if (end7) {
            r[7] += ih2x * (u[7] - hs[1]);
            r[7] += 0.5 * ih2x * f7;
        }
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        if (cov[x >> 2]) r[x] = 0.0;
        const double av = fabs(r[x]);
        acc = norm_p == 2 ? acc + av * av : norm_p == 1 ? acc + av : fmax(acc, av);
    }
    if (active) {
        if (r_out) {
            T rt[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) rt[i] = (T)r[i];
            Row8<T>::store(r_out + rb, rt);
        }
        if (r_user) {
            const int2 us = M.ustr[b];
            double *ru = r_user[lev] + M.ubase[b] + (int64_t)us.x * y + (int64_t)us.y * z;
#pragma unroll
            for (int i = 0; i < 8; ++i) ru[i] = r[i];
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double v = __shfl_xor(acc, o, 64);
        acc = norm_p == 0 ? fmax(acc, v) : acc + v;
        if (BOTH) {
            const double v0 = __shfl_xor(acc0, o, 64);
            acc0 = norm_p == 0 ? fmax(acc0, v0) : acc0 + v0;
        }
    }
    if (active && lane == 0) {
        part[b] = acc;
        if (BOTH) part[n_part + b] = acc0;
    }
}

// Copies between the caller's box-list layout and brick layout on a range or
// list of AMR bricks: to_brick: a -> ab and (when set) b -> bb; else ab -> a.
__global__ void __launch_bounds__(256) k_user_brick(DevMeta M, int b0, int nb, const int32_t *list, int to_brick,
                                                    double *const *a, double *ab, double *const *bu, double *bb)
{
    const int b = pick_brick(b0, nb, list, blockIdx.x);
    const int w = M.org[b].w;
    const int64_t ub = M.ubase[b];
    const int2 us = M.ustr[b];
    for (int c = threadIdx.x; c < BRICK_CELLS; c += 256) {
        int64_t ui = ub + (c & 7) + (int64_t)us.x * ((c >> 3) & 7) + (int64_t)us.y * (c >> 6);
        size_t bi = (size_t)b * BRICK_CELLS + c;
        if (to_brick) {
            ab[bi] = a[w][ui];
            if (bb) bb[bi] = bu[w][ui];
        } else {
            a[w][ui] = ab[bi];
        }
    }
}

// Norms of brick ranges (the AMR levels of each problem) from the bricks'
// partials, in a fixed order.  The ranges are cut into pieces of at most
// NORM_PIECE bricks (x first brick, y bricks, z range); a wavefront sums a
// piece, all its loads in flight, and then one a range adds the piece sums.
// sets = 2: the same for a second set of partials, n_part further on; its
// norms follow the first set's.  Up to NORM_ONE pieces one workgroup does it
// all.  More go to a workgroup per 16; the last to finish (an agent-scope
// count that it sets back) adds the piece sums.
//
// With hout set, the norms are also written to host-visible memory followed
// by a sequence number (the device counter plus one), so that the host can
// poll for them without synchronising the stream.  The host copy goes to hout
// + alt when the counter is odd: two publications in a row land in different
// slots, so the host can still read one while the next is being written.
//
// One workgroup going from range to range took 7.5 us on three ranges of 3000
// bricks, 47 on the 40 of a batch of sixteen and 121 on 4e5 bricks; now 4.9,
// 9.3 and 11.
__global__ void __launch_bounds__(1024) k_level_norms(const int4 *pieces, const int *first, int npiece, int n,
                                                      int sets, const double *part, int n_part, double *psum,
                                                      int *done, int norm_p, double *hout, int alt, unsigned *hseq,
                                                      unsigned *counter)
{
    __shared__ double sh[NORM_ONE], nrm[NORM_ONE];
    __shared__ unsigned sseq;
    __shared__ int slast;
    const bool mx = norm_p == 0, one = gridDim.x == 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (threadIdx.x == 0) sseq = *counter;
    const int np = sets * npiece, p0 = one ? 0 : 16 * (int)blockIdx.x, p1 = one ? np : min(np, p0 + 16);
    for (int p = p0 + wave; p < p1; p += 16) {
        const bool second = p >= npiece;
        const int4 pc = pieces[second ? p - npiece : p];
        const double *v = part + (second ? n_part : 0) + pc.x;
        double a[NORM_PIECE / 64];
#pragma unroll
        for (int j = 0; j < NORM_PIECE / 64; ++j) a[j] = lane + 64 * j < pc.y ? v[lane + 64 * j] : 0.0;
        double s = 0.0;  // (partials are >= 0)
#pragma unroll
        for (int j = 0; j < NORM_PIECE / 64; ++j) s = mx ? fmax(s, a[j]) : s + a[j];
        for (int o = 32; o > 0; o >>= 1) {
            const double t = __shfl_xor(s, o, 64);
            s = mx ? fmax(s, t) : s + t;
        }
        if (lane == 0) {
            if (one) sh[p] = s;
            else __hip_atomic_store(psum + p, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // every wavefront waits for its own sum to arrive: the count below orders
    // (and waits for) the stores of the wavefront that counts alone, and a
    // barrier waits for no store to memory
    if (!one) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (!one) {
        if (threadIdx.x == 0) {
            const int c = __hip_atomic_fetch_add(done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            slast = c == (int)gridDim.x - 1;
            if (slast) __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!slast) return;
    }
    // (ranges NORM_ONE at a time: their sums to LDS, then one wavefront
    // publishes them, with one system-wide fence at the end)
    const unsigned seq = sseq;
    for (int k0 = 0; k0 < sets * n; k0 += NORM_ONE) {
        for (int k = k0 + wave; k < min(sets * n, k0 + NORM_ONE); k += 16) {
            const int j = k >= n ? k - n : k, o = k >= n ? npiece : 0, e = first[j + 1];
            double s = 0.0;
            for (int p = first[j] + lane; p < e; p += 64) {
                const double t = one ? sh[o + p]
                                     : __hip_atomic_load(psum + o + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s = mx ? fmax(s, t) : s + t;
            }
            for (int q = 32; q > 0; q >>= 1) {
                const double t = __shfl_xor(s, q, 64);
                s = mx ? fmax(s, t) : s + t;
            }
            if (lane == 0) nrm[k - k0] = norm_p == 2 ? sqrt(s) : s;
        }
        __syncthreads();
        if (wave == 0 && k0 + lane < sets * n) hout[(seq & 1u) * alt + k0 + lane] = nrm[lane];
        __syncthreads();
    }
    if (wave == 0) {
        __threadfence_system();
        if (lane == 0) {
            *counter = seq + 1;
            *(volatile unsigned *)hseq = seq + 1;
        }
    }
}

// ---------------------------------------------------------------------------
// coarse parts of the coarse-fine ghosts (step 1 of Eq. 2d_lagrange, times
// the step-2 weight 8/15)
// ---------------------------------------------------------------------------
template <class T>
struct SrcBrick {
    const T *u;
    __device__ double operator()(int32_t g) const { return (double)u[g]; }
};

template <class T, class S>
__global__ void __launch_bounds__(256) k_cpart(DevMeta M, int cf0, int ncf, S src, T *cp, const T *fine,
                                               double *ffs)
{
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= ncf * 16) return;
    int cf = cf0 + (i >> 4), m = i & 15;
    size_t e = (size_t)cf * 16 + m;
    const int ow = ffs ? M.gf_owner[M.nbc + cf] : 0;
    int pat = M.cf_pat[e];
    double v[9];
    for (int w = 0; w < 9; ++w) v[w] = src(M.cf_idx[e * 9 + w]);
    int mu = m & 3, mv = m >> 2;
    double c[4];
    for (int q = 0; q < 4; ++q) {
        const double *W = c_cfw + (pat * 4 + q) * 9;
        double s = 0.0;
        for (int w = 0; w < 9; ++w) s += W[w] * v[w];
        int t = (2 * mu + (q & 1)) + 8 * (2 * mv + (q >> 1));
        cp[(size_t)cf * 64 + t] = (T)s;
        c[q] = (double)(T)s;
    }
    // with ffs: the fine sum of this coarse cell from the fine values and these coarse parts
    if (ffs) ffs[((size_t)(ow >> 3) * 6 + (ow & 7)) * 16 + m] = face_sum(SrcB<T>{fine}, ow >> 3, ow & 7, m, c);
}

// fine sums (zero coarse parts) of the coarse-fine faces [cf0, cf0 + ncf) from e
template <class T>
__global__ void __launch_bounds__(256) k_face_sums(DevMeta M, int cf0, int ncf, const T *e, double *ffs)
{
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= ncf * 16) return;
    const int ow = M.gf_owner[M.nbc + cf0 + (i >> 4)], m = i & 15;
    const double c[4] = {0.0, 0.0, 0.0, 0.0};
    ffs[((size_t)(ow >> 3) * 6 + (ow & 7)) * 16 + m] = face_sum(SrcB<T>{e}, ow >> 3, ow & 7, m, c);
}

// ---------------------------------------------------------------------------
// V-cycle kernels on the correction equation (Alg. 3)
// ---------------------------------------------------------------------------

// Gauss-Seidel red-black, one colour: cells with (i+j+k) mod 2 == colour in
// level indices.  Each of the 256 threads owns one cell of that colour.
// init: e is undefined and taken as zero; the other colour is written 0.
template <class T>
__global__ void __launch_bounds__(256) k_gsrb(DevMeta M, int b0, int nb, T *e, const T *r, const T *cp,
                                              int colour, int init)
{
    __shared__ double tile[TE * TE * TE];
    __shared__ double alpha[6];
    int b = b0 + xcd_remap(blockIdx.x, nb);
    int lev = M.org[b].w;
    LevelConst L = M.lc[lev];
    int t = threadIdx.x;
    int z = t >> 5, y = (t >> 2) & 7, xx = (t & 3) << 1;
    int x = xx + (((y + z) & 1) ^ colour);  // brick origins are even
    size_t li = (size_t)b * BRICK_CELLS + x + 8 * y + 64 * z;
    double rv = (double)r[li];
    if (init)
        stage_tile<SrcZ, true>(M, b, SrcZ{}, CpNone{}, false, tile, alpha);
    else
        stage_tile<SrcB<T>, false, CpArr<T>>(M, b, SrcB<T>{e}, CpArr<T>{cp}, false, tile, alpha);
    double num = rv, den = 0.0;
    for (int d = 0; d < 3; ++d)
        for (int s = -1; s <= 1; s += 2) {
            double a, bv;
            tile_ab(tile, alpha, x, y, z, d, s, a, bv);
            num += L.ih2[d] * bv;
            den += L.ih2[d] * (1.0 - a);
        }
    e[li] = (T)(num / den);
    if (init) e[li ^ 1] = (T)0;
}

// damped Jacobi sweep: eout = ein + omega (D^-1 (r - (A - D) ein) - ein)
template <class T>
__global__ void __launch_bounds__(256) k_jacobi(DevMeta M, int b0, int nb, const T *ein, T *eout, const T *r,
                                                const T *cp, double omega, int init)
{
    __shared__ double tile[TE * TE * TE];
    __shared__ double alpha[6];
    int b = b0 + xcd_remap(blockIdx.x, nb);
    int lev = M.org[b].w;
    LevelConst L = M.lc[lev];
    double rv[2];
    for (int k = 0; k < 2; ++k) rv[k] = (double)r[(size_t)b * BRICK_CELLS + threadIdx.x + 256 * k];
    if (init)
        stage_tile<SrcZ, true>(M, b, SrcZ{}, CpNone{}, false, tile, alpha);
    else
        stage_tile<SrcB<T>, false, CpArr<T>>(M, b, SrcB<T>{ein}, CpArr<T>{cp}, false, tile, alpha);
    for (int k = 0; k < 2; ++k) {
        int c = threadIdx.x + 256 * k;
        int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
        double num = rv[k], den = 0.0;
        for (int d = 0; d < 3; ++d)
            for (int s = -1; s <= 1; s += 2) {
                double a, bv;
                tile_ab(tile, alpha, x, y, z, d, s, a, bv);
                num += L.ih2[d] * bv;
                den += L.ih2[d] * (1.0 - a);
            }
        double uc = tile[tix(x, y, z)];
        eout[(size_t)b * BRICK_CELLS + c] = (T)(uc + omega * (num / den - uc));
    }
}

// Brick-hybrid Gauss-Seidel sweep: red then black over the cells of one
// brick in LDS, with the halo taken from the previous sweep (Gauss-Seidel
// inside a brick, Jacobi between bricks, as a parallel Gauss-Seidel works
// inside and between subdomains).  Reads ein, writes eout.
// MODE bits: 1 input is zero; 2 input plus the parent correction (fused
// prolongation); 4 coarse parts of the coarse-fine ghosts computed from the
// coarse level's values in ein and stored into cp (else read from cp);
// 8 phi += result on AMR bricks (fused phi update; phi in brick layout), the
// result itself stored only where the finer level reads it (1.9e8 cells 1050
// -> 891 us, 2.7e7 147 -> 128);
// 16 the fine sums of the result on the brick's coarse-fine faces into ffs.
enum { HG_ZERO = 1, HG_PROL = 2, HG_CPIN = 4, HG_PHI = 8, HG_FFS = 16 };

// face_sum of a brick held in the row layout with zero coarse parts: over the
// four fine cells of coarse cell m of face f, u_f/3 + u_in/5 (u_in the cell
// further inside along the face normal)
template <class T>
__device__ __forceinline__ double row_face_sum(const T *rows, int f, int m)
{
    const int d = f >> 1, at = (f & 1) ? 7 : 0, in = (f & 1) ? 6 : 1;
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = 2 * (m & 3) + (q & 1), v = 2 * (m >> 2) + (q >> 1);
        // (x, y, z) of the face cell and of the cell inside, for the normal d
        // with u, v along the two other axes in x < y < z order
        const int x0 = d == 0 ? at : u, y0 = d == 1 ? at : (d == 0 ? u : v), z0 = d == 2 ? at : v;
        const int x1 = d == 0 ? in : u, y1 = d == 1 ? in : (d == 0 ? u : v), z1 = d == 2 ? in : v;
        sum += (1.0 / 3.0) * (double)rows[rrow(y0, z0) + x0] + 0.2 * (double)rows[rrow(y1, z1) + x1];
    }
    return sum;
}

// parent cell of local cell (x, y, z) of a brick whose parent entry is p
// (parent brick << 3 | octant), as a cell index of the parent's slab
__device__ __forceinline__ size_t parent_cell(int p, int x, int y, int z)
{
    const int oc = p & 7;
    return (size_t)(p >> 3) * BRICK_CELLS + ((oc & 1) * 4 + (x >> 1)) + 8 * (((oc >> 1) & 1) * 4 + (y >> 1)) +
           64 * ((oc >> 2) * 4 + (z >> 1));
}

// Lane-wise choice of a (lane's bit of m clear) or b (set), m a wavefront
// mask from a ballot, as v_cndmask in asm: a choice between two elements of
// a register array written as C++ is rewritten by the compiler into one
// access at a computed index, which moves the array into private memory.
__device__ __forceinline__ float lane_pick(uint64_t m, float a, float b)
{
    float r;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(m));
    return r;
}
__device__ __forceinline__ double lane_pick(uint64_t m, double a, double b)
{
    const uint64_t ia = (uint64_t)__double_as_longlong(a), ib = (uint64_t)__double_as_longlong(b);
    uint32_t lo, hi;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(lo) : "v"((uint32_t)ia), "v"((uint32_t)ib), "s"(m));
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(hi) : "v"((uint32_t)(ia >> 32)), "v"((uint32_t)(ib >> 32)), "s"(m));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <class T, int MODE, int BPW>
__global__ void __launch_bounds__(64 * BPW) k_hgs(DevMeta M, int b0, int nb, const T *ein, T *eout, const T *r,
                                                  T *cp, double *phib, double *ffs)
{
    __shared__ T rows_all[BPW][RW * RW * RS];
    // the wavefront's brick, wavefront-uniform (so its table entries come
    // through scalar loads and the face kinds branch on the scalar unit)
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int k0 = xcd_remap(blockIdx.x, (nb + BPW - 1) / BPW) * BPW + w;
    const bool active = k0 < nb;  // the last workgroup may hold fewer bricks
    const int b = __builtin_amdgcn_readfirstlane(b0 + (active ? k0 : nb - 1));
    T *rows = rows_all[w];
    const int y = lane & 7, z = lane >> 3;
    // face kinds: 0 a brick of the level, 1 the physical boundary (ghost
    // abnd u_c), 2 coarse-fine (ghost 2/3 u_c + cp - u_in/5)
    int nbf[6], kind[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        nbf[f] = M.nbr[b * 6 + f];
        kind[f] = nbf[f] >= 0 ? 0 : ((-1 - nbf[f]) < M.nbc ? 1 : 2);
    }
    // the neighbours' parents (fused prolongation), all in flight together
    int pf[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) pf[f] = (MODE & HG_PROL) ? M.par[nbf[f] >= 0 ? nbf[f] : b] : 0;
    // halo slot of face f at face-local cell fl (first transverse axis
    // fastest): the neighbour's value, 0 on the boundary (homogeneous cycle),
    // or the coarse part of the coarse-fine ghost; with the fused
    // prolongation the neighbour's parent value goes to hp, to be added once
    // every load is out (added here, each face's loads were waited for before
    // the next face's: 1.9e8 cells 545 -> 500 us, 2.7e7 102 -> 93, 64 bricks in
    // FP64 7.6 -> 6.2)
    auto slot = [&](int f, int fl, T &hp) -> T {
        const int d = f >> 1, md = (f & 1) ? 0 : 7;
        hp = (T)0;
        if (kind[f] == 0) {
            if (MODE & HG_ZERO) return (T)0;
            const int u = fl & 7, v = fl >> 3;
            const int c = d == 0 ? md + 8 * u + 64 * v : (d == 1 ? u + 8 * md + 64 * v : u + 8 * v + 64 * md);
            if (MODE & HG_PROL) hp = ein[parent_cell(pf[f], c & 7, (c >> 3) & 7, c >> 6)];
            return ein[(size_t)nbf[f] * BRICK_CELLS + c];
        }
        if (kind[f] == 1 || (MODE & HG_ZERO)) return (T)0;
        const size_t cf = (size_t)(-1 - nbf[f] - M.nbc);
        if (MODE & HG_CPIN) return (T)CpInline<T>{&M, ein, active ? cp : nullptr}(cf, fl);
        return cp ? cp[cf * 64 + fl] : (T)0;
    };
    const LevelConst L = M.lc[M.org[b].w];
    // every load first: right-hand sides, input, halo slots, phi
    const size_t rb = (size_t)b * BRICK_CELLS + 8 * lane;
    T rr[8], er[8], hs[6];
    Row8<T>::load(r + rb, rr);
    if (MODE & HG_ZERO) {
#pragma unroll
        for (int i = 0; i < 8; ++i) er[i] = (T)0;
    } else {
        Row8<T>::load(ein + rb, er);
    }
    T pv[4], hp[6];
    if (MODE & HG_PROL) {
        const size_t pc = parent_cell(M.par[b], 0, y, z);
#pragma unroll
        for (int k = 0; k < 4; ++k) pv[k] = ein[pc + k];
    }
    // x-neighbours held by the previous or the next wavefront of the
    // workgroup (bricks are numbered x-fastest within a box): their starting
    // values are the rows those wavefronts put in LDS, read from there below
    // instead of from memory
    const bool lx_m = BPW > 1 && w > 0 && kind[0] == 0 && nbf[0] == b - 1;
    const bool lx_p = BPW > 1 && w + 1 < BPW && k0 + 1 < nb && kind[1] == 0 && nbf[1] == b + 1;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        hs[f] = hp[f] = (T)0;
        if (!((f == 0 && lx_m) || (f == 1 && lx_p))) hs[f] = slot(f, lane, hp[f]);
    }
    const bool phi = (MODE & HG_PHI) && L.amr >= 0;
    double ph[8];
    if (phi) Row8<double>::load(phib + rb, ph);
    if (MODE & HG_PROL) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            er[2 * k] = (T)((double)er[2 * k] + (double)pv[k]);
            er[2 * k + 1] = (T)((double)er[2 * k + 1] + (double)pv[k]);
        }
#pragma unroll
        for (int f = 0; f < 6; ++f) hs[f] = (T)((double)hs[f] + (double)hp[f]);
    }
    const T ih2x = (T)L.ih2[0], ih2y = (T)L.ih2[1], ih2z = (T)L.ih2[2];
    const int rym = rrow(y - 1, z), ryp = rrow(y + 1, z), rzm = rrow(y, z - 1), rzp = rrow(y, z + 1), rme = rrow(y, z);
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[rme + i] = er[i];
    // y halo rows: face-local cell (x, z); z halo rows: (x, y)
    rows[rrow(-1, lane >> 3) + (lane & 7)] = hs[2];
    rows[rrow(8, lane >> 3) + (lane & 7)] = hs[3];
    rows[rrow(lane >> 3, -1) + (lane & 7)] = hs[4];
    rows[rrow(lane >> 3, 8) + (lane & 7)] = hs[5];
    T hxm = hs[0], hxp = hs[1];
    // ghost coefficients a of the faces, and per row the weights that fold a
    // coarse-fine ghost's -u_in/5 into the neighbour inside
    const T cf5 = (T)0.2;
    T ag[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) ag[f] = kind[f] == 1 ? (T)L.abnd[f >> 1] : (kind[f] == 2 ? (T)(2.0 / 3.0) : (T)0);
    const T aym = y == 0 ? ag[2] : (T)0, ayp = y == 7 ? ag[3] : (T)0;
    const T azm = z == 0 ? ag[4] : (T)0, azp = z == 7 ? ag[5] : (T)0;
    const T wyp = (y == 0 && kind[2] == 2) ? (T)1 - cf5 : (T)1, wym = (y == 7 && kind[3] == 2) ? (T)1 - cf5 : (T)1;
    const T wzp = (z == 0 && kind[4] == 2) ? (T)1 - cf5 : (T)1, wzm = (z == 7 && kind[5] == 2) ? (T)1 - cf5 : (T)1;
    const T wxp0 = kind[0] == 2 ? (T)1 - cf5 : (T)1, wxm7 = kind[1] == 2 ? (T)1 - cf5 : (T)1;
    const T den = ih2y * ((T)2 - aym - ayp) + ih2z * ((T)2 - azm - azp) + (T)2 * ih2x;
    const T inv_mid = (T)1 / den, inv_x0 = (T)1 / (den - ih2x * ag[0]), inv_x7 = (T)1 / (den - ih2x * ag[1]);
    __syncthreads();
    if (BPW > 1) {
        // the neighbours' rows are read before any wavefront starts updating its own
        if (lx_m) hxm = rows_all[w - 1][rme + 7];
        if (lx_p) hxp = rows_all[w + 1][rme];
        __syncthreads();
    }
    // red (colour 0) then black: cell x of row (y, z) has colour (x + y + z)
    // & 1, so in each pair of cells (2k, 2k + 1) of the row exactly one
    // takes part in a pass, the one at x = 2k + p with p = (y + z + pass) &
    // 1.  Its operands are chosen from the row's registers by selects
    // between fixed elements (a lane-dependent register index would be
    // turned into an indexed access to private memory); its LDS neighbours
    // are read at the lane's own offset.
    const int q = (y + z) & 1;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const bool p = ((q + c) & 1) != 0;
        const uint64_t pm = __builtin_amdgcn_ballot_w64(p);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int x = 2 * k + (p ? 1 : 0);
            const T xm = lane_pick(pm, k == 0 ? hxm : er[2 * k - 1], er[2 * k]);
            const T xp = lane_pick(pm, er[2 * k + 1], k == 3 ? hxp : er[2 * k + 2]);
            const T rx = lane_pick(pm, rr[2 * k], rr[2 * k + 1]);
            const T wxm = k == 3 ? lane_pick(pm, (T)1, wxm7) : (T)1;
            const T wxp = k == 0 ? lane_pick(pm, wxp0, (T)1) : (T)1;
            const T inv = k == 0 ? lane_pick(pm, inv_x0, inv_mid) : (k == 3 ? lane_pick(pm, inv_mid, inv_x7) : inv_mid);
            const T num = rx + ih2x * (wxm * xm + wxp * xp) +
                          ih2y * (wym * rows[rym + x] + wyp * rows[ryp + x]) +
                          ih2z * (wzm * rows[rzm + x] + wzp * rows[rzp + x]);
            const T nv = num * inv;
            er[2 * k] = p ? er[2 * k] : nv;
            er[2 * k + 1] = p ? nv : er[2 * k + 1];
            rows[rme + x] = nv;
        }
        __syncthreads();
    }
    if (!active) return;
    // the last sweep's result is read again only where the finer level is
    // (parents and interpolation windows)
    if (!phi || M.eread[b]) Row8<T>::store(eout + rb, er);
    if (phi) {
#pragma unroll
        for (int i = 0; i < 8; ++i) ph[i] += (double)er[i];
        Row8<double>::store(phib + rb, ph);
    }
    // fine sums of the new e on the brick's coarse-fine faces (the coarse
    // correction, and so the ghosts' coarse parts, are zero at the
    // restriction that reads them)
    if (MODE & HG_FFS) {
        for (int t = lane; t < 96; t += 64) {
            const int f = t >> 4;
            if (kind[f] == 2) ffs[((size_t)b * 6 + f) * 16 + (t & 15)] = row_face_sum(rows, f, t & 15);
        }
    }
}

// The first two sweeps of the correction equation in one launch, the first
// from e = 0: r -> the result of both, the same arithmetic as two launches of
// k_hgs (HG_ZERO, then 0 or HG_FFS).  The second sweep wants the halo after
// the first.  Started from zero with a zero halo, the first sweep of a
// neighbour brick needs only that brick's r, and its values on the layer next
// to this brick only r on that layer and on the one behind: red cells r / D,
// black ones from the red cells around them in the neighbour.  Each lane
// recomputes one cell of each of the six layers, so e is never written or
// read between the sweeps.
//
// Against the two launches: 1.9e8 cells of 576^3 425 us (248 + 465), 2.7e7
// cells of 128^3 + 3 levels 70 (39 + 77), 2365 bricks 10.8 (4.7 + 7.0) and in
// FP64 12.8 (8.4 + 9.3), 64 bricks in FP64 7.1 (4.2 + 4.7).
template <class T, bool FFS, int BPW>
__global__ void __launch_bounds__(64 * BPW) k_hgs_first2(DevMeta M, int b0, int nb, T *eout, const T *r, double *ffs)
{
    __shared__ T rows_all[BPW][RW * RW * RS];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int k0 = xcd_remap(blockIdx.x, (nb + BPW - 1) / BPW) * BPW + w;
    const bool active = k0 < nb;  // the last workgroup may hold fewer bricks
    const int b = __builtin_amdgcn_readfirstlane(b0 + (active ? k0 : nb - 1));
    T *rows = rows_all[w];
    const int y = lane & 7, z = lane >> 3;
    int nbf[6], kind[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        nbf[f] = M.nbr[b * 6 + f];
        kind[f] = nbf[f] >= 0 ? 0 : ((-1 - nbf[f]) < M.nbc ? 1 : 2);
    }
    // every load first: the brick's r, and r on two layers of each neighbour
    // (face-local cell (u, v) of the lane, the axes in x < y < z order)
    const size_t rb = (size_t)b * BRICK_CELLS + 8 * lane;
    T rr[8], r0[6], r1[6];
    Row8<T>::load(r + rb, rr);
    const bool lx_m = BPW > 1 && w > 0 && kind[0] == 0 && nbf[0] == b - 1;
    const bool lx_p = BPW > 1 && w + 1 < BPW && k0 + 1 < nb && kind[1] == 0 && nbf[1] == b + 1;
    int nk[6][4];  // kinds of the neighbour's faces at the ends of u and v
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        r0[f] = r1[f] = (T)0;
#pragma unroll
        for (int g = 0; g < 4; ++g) nk[f][g] = 0;
        if (kind[f] != 0 || (f == 0 && lx_m) || (f == 1 && lx_p)) continue;
        const int d = f >> 1, c0 = (f & 1) ? 0 : 7, c1 = (f & 1) ? 1 : 6;
        const T *n = r + (size_t)nbf[f] * BRICK_CELLS;
        const int sd = d == 0 ? 1 : (d == 1 ? 8 : 64), o = d == 0 ? 8 * lane : (d == 1 ? y + 64 * z : lane);
        r0[f] = n[o + sd * c0];
        r1[f] = n[o + sd * c1];
        const int du = d == 0 ? 1 : 0, dv = d == 2 ? 1 : 2;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int q = M.nbr[nbf[f] * 6 + 2 * (g < 2 ? du : dv) + (g & 1)];
            nk[f][g] = q >= 0 ? 0 : ((-1 - q) < M.nbc ? 1 : 2);
        }
    }
    const LevelConst L = M.lc[M.org[b].w];
    const T ih2x = (T)L.ih2[0], ih2y = (T)L.ih2[1], ih2z = (T)L.ih2[2];
    const T cf5 = (T)0.2, two3 = (T)(2.0 / 3.0);
    const T den_in = ih2y * (T)2 + ih2z * (T)2 + (T)2 * ih2x, inv_in = (T)1 / den_in;
    // the neighbours' layers after their first sweep
    T hs[6], inv0[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, du = d == 0 ? 1 : 0, dv = d == 2 ? 1 : 2;
        inv0[f] = inv_in;
        if (nk[f][0] | nk[f][1] | nk[f][2] | nk[f][3]) {
            // ghost coefficients of the neighbour's other faces at this cell
            auto ag = [&](int k, int ax) { return k == 1 ? (T)L.abnd[ax] : (k == 2 ? two3 : (T)0); };
            const T um = y == 0 ? ag(nk[f][0], du) : (T)0, up = y == 7 ? ag(nk[f][1], du) : (T)0;
            const T vm = z == 0 ? ag(nk[f][2], dv) : (T)0, vp = z == 7 ? ag(nk[f][3], dv) : (T)0;
            const T ym = du == 1 ? um : (dv == 1 ? vm : (T)0), yp = du == 1 ? up : (dv == 1 ? vp : (T)0);
            const T zm = dv == 2 ? vm : (T)0, zp = dv == 2 ? vp : (T)0;
            T den = ih2y * ((T)2 - ym - yp) + ih2z * ((T)2 - zm - zp) + (T)2 * ih2x;
            if (du == 0) den = den - ih2x * um - ih2x * up;  // (one of the two at most)
            inv0[f] = (T)1 / den;
        }
        rows[72 * f + y + 9 * z] = r0[f] * inv0[f];  // (the red cells' values)
    }
    wave_fence();
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, c0 = (f & 1) ? 0 : 7;
        const T *pl = rows + 72 * f + y + 9 * z;
        const T um = y > 0 ? pl[-1] : (T)0, up = y < 7 ? pl[1] : (T)0;
        const T vm = z > 0 ? pl[-9] : (T)0, vp = z < 7 ? pl[9] : (T)0;
        const T wup = (y == 0 && nk[f][0] == 2) ? (T)1 - cf5 : (T)1, wum = (y == 7 && nk[f][1] == 2) ? (T)1 - cf5 : (T)1;
        const T wvp = (z == 0 && nk[f][2] == 2) ? (T)1 - cf5 : (T)1, wvm = (z == 7 && nk[f][3] == 2) ? (T)1 - cf5 : (T)1;
        const T iu = d == 0 ? ih2y : ih2x, iv = d == 2 ? ih2y : ih2z, id = d == 0 ? ih2x : (d == 1 ? ih2y : ih2z);
        // (the layer behind has the same D)
        const T in = r1[f] * inv0[f];
        const T black = (r0[f] + id * in + iu * (wum * um + wup * up) + iv * (wvm * vm + wvp * vp)) * inv0[f];
        hs[f] = ((c0 + y + z) & 1) ? black : pl[0];
        if (kind[f] != 0) hs[f] = (T)0;
    }
    wave_fence();
    const int rym = rrow(y - 1, z), ryp = rrow(y + 1, z), rzm = rrow(y, z - 1), rzp = rrow(y, z + 1), rme = rrow(y, z);
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[rme + i] = (T)0;
    rows[rrow(-1, z) + y] = (T)0;
    rows[rrow(8, z) + y] = (T)0;
    rows[rrow(z, -1) + y] = (T)0;
    rows[rrow(z, 8) + y] = (T)0;
    T ag[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) ag[f] = kind[f] == 1 ? (T)L.abnd[f >> 1] : (kind[f] == 2 ? two3 : (T)0);
    const T aym = y == 0 ? ag[2] : (T)0, ayp = y == 7 ? ag[3] : (T)0;
    const T azm = z == 0 ? ag[4] : (T)0, azp = z == 7 ? ag[5] : (T)0;
    const T wyp = (y == 0 && kind[2] == 2) ? (T)1 - cf5 : (T)1, wym = (y == 7 && kind[3] == 2) ? (T)1 - cf5 : (T)1;
    const T wzp = (z == 0 && kind[4] == 2) ? (T)1 - cf5 : (T)1, wzm = (z == 7 && kind[5] == 2) ? (T)1 - cf5 : (T)1;
    const T wxp0 = kind[0] == 2 ? (T)1 - cf5 : (T)1, wxm7 = kind[1] == 2 ? (T)1 - cf5 : (T)1;
    const T den = ih2y * ((T)2 - aym - ayp) + ih2z * ((T)2 - azm - azp) + (T)2 * ih2x;
    const T inv_mid = (T)1 / den, inv_x0 = (T)1 / (den - ih2x * ag[0]), inv_x7 = (T)1 / (den - ih2x * ag[1]);
    T er[8], hxm = (T)0, hxp = (T)0;
#pragma unroll
    for (int i = 0; i < 8; ++i) er[i] = (T)0;
    wave_fence();
    // the colour passes of k_hgs
    const int q = (y + z) & 1;
    auto pass = [&](int c) {
        const bool p = ((q + c) & 1) != 0;
        const uint64_t pm = __builtin_amdgcn_ballot_w64(p);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int x = 2 * k + (p ? 1 : 0);
            const T xm = lane_pick(pm, k == 0 ? hxm : er[2 * k - 1], er[2 * k]);
            const T xp = lane_pick(pm, er[2 * k + 1], k == 3 ? hxp : er[2 * k + 2]);
            const T rx = lane_pick(pm, rr[2 * k], rr[2 * k + 1]);
            const T wxm = k == 3 ? lane_pick(pm, (T)1, wxm7) : (T)1;
            const T wxp = k == 0 ? lane_pick(pm, wxp0, (T)1) : (T)1;
            const T inv = k == 0 ? lane_pick(pm, inv_x0, inv_mid) : (k == 3 ? lane_pick(pm, inv_mid, inv_x7) : inv_mid);
            const T num = rx + ih2x * (wxm * xm + wxp * xp) +
                          ih2y * (wym * rows[rym + x] + wyp * rows[ryp + x]) +
                          ih2z * (wzm * rows[rzm + x] + wzp * rows[rzp + x]);
            const T nv = num * inv;
            er[2 * k] = p ? er[2 * k] : nv;
            er[2 * k + 1] = p ? nv : er[2 * k + 1];
            rows[rme + x] = nv;
        }
        wave_fence();
    };
    pass(0);
    pass(1);
    rows[rrow(-1, z) + y] = hs[2];
    rows[rrow(8, z) + y] = hs[3];
    rows[rrow(z, -1) + y] = hs[4];
    rows[rrow(z, 8) + y] = hs[5];
    hxm = hs[0];
    hxp = hs[1];
    __syncthreads();
    if (BPW > 1) {
        // x-neighbours of the workgroup: their rows after the first sweep,
        // read before any wavefront starts its second
        if (lx_m) hxm = rows_all[w - 1][rme + 7];
        if (lx_p) hxp = rows_all[w + 1][rme];
        __syncthreads();
    }
    pass(0);
    pass(1);
    if (!active) return;
    Row8<T>::store(eout + rb, er);
    if (FFS) {
        for (int t = lane; t < 96; t += 64) {
            const int f = t >> 4;
            if (kind[f] == 2) ffs[((size_t)b * 6 + f) * 16 + (t & 15)] = row_face_sum(rows, f, t & 15);
        }
    }
}

// residual of the homogeneous problem at one cell: r - A e (zero coarse data)
template <class T>
__device__ __forceinline__ double cell_residual(const DevMeta &M, const LevelConst &L, int b, const int *lc,
                                                const T *e, const T *r)
{
    size_t li = (size_t)b * BRICK_CELLS + lc[0] + 8 * lc[1] + 64 * lc[2];
    double uc = (double)e[li], Au = 0.0;
    for (int d = 0; d < 3; ++d)
        for (int s = -1; s <= 1; s += 2) {
            double a, bv;
            face_nb(M, b, lc, d, s, BrickAcc<T>{e}, nullptr, nullptr, false, a, bv);
            Au += L.ih2[d] * ((1.0 - a) * uc - bv);
        }
    return (double)r[li] - Au;
}

// r^{l-1} on covered cells = mean over the 8 children of (r^l - A_nf e^l)
// (Alg. 3, restriction onto the covered domain; e^{l-1} = 0 at that point,
// so the coarse parts of the coarse-fine ghosts are zero).  One wavefront
// per fine brick in the row layout: lane (y, z) computes the residual of its
// row, adds x pairs, then the y and z pairs of the lanes 1 and 8 apart; the
// lanes with even y and z write four coarse cells of their parent's row.
template <class T>
__device__ __forceinline__ void restrict_brick(const DevMeta &M, int b, bool active, const T *e, T *r, T *rows)
{
    const int lane = threadIdx.x & 63, y = lane & 7, z = lane >> 3;
    const LevelConst L = M.lc[M.org[b].w];
    int nbf[6], kind[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        nbf[f] = M.nbr[b * 6 + f];
        kind[f] = nbf[f] >= 0 ? 0 : ((-1 - nbf[f]) < M.nbc ? 1 : 2);
    }
    const size_t rb = (size_t)b * BRICK_CELLS + 8 * lane;
    T rr[8], u[8], hs[6];
    Row8<T>::load(r + rb, rr);
    Row8<T>::load(e + rb, u);
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, md = (f & 1) ? 0 : 7, uu = lane & 7, vv = lane >> 3;
        const int c = d == 0 ? md + 8 * uu + 64 * vv : (d == 1 ? uu + 8 * md + 64 * vv : uu + 8 * vv + 64 * md);
        hs[f] = kind[f] == 0 ? e[(size_t)nbf[f] * BRICK_CELLS + c] : (T)0;
    }
    const int rym = rrow(y - 1, z), ryp = rrow(y + 1, z), rzm = rrow(y, z - 1), rzp = rrow(y, z + 1), rme = rrow(y, z);
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[rme + i] = u[i];
    rows[rrow(-1, lane >> 3) + (lane & 7)] = hs[2];
    rows[rrow(8, lane >> 3) + (lane & 7)] = hs[3];
    rows[rrow(lane >> 3, -1) + (lane & 7)] = hs[4];
    rows[rrow(lane >> 3, 8) + (lane & 7)] = hs[5];
    T ag[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) ag[f] = kind[f] == 1 ? (T)L.abnd[f >> 1] : (kind[f] == 2 ? (T)(2.0 / 3.0) : (T)0);
    const T ih2x = (T)L.ih2[0], ih2y = (T)L.ih2[1], ih2z = (T)L.ih2[2], cf5 = (T)0.2;
    const T aym = y == 0 ? ag[2] : (T)0, ayp = y == 7 ? ag[3] : (T)0;
    const T azm = z == 0 ? ag[4] : (T)0, azp = z == 7 ? ag[5] : (T)0;
    const T wyp = (y == 0 && kind[2] == 2) ? (T)1 - cf5 : (T)1, wym = (y == 7 && kind[3] == 2) ? (T)1 - cf5 : (T)1;
    const T wzp = (z == 0 && kind[4] == 2) ? (T)1 - cf5 : (T)1, wzm = (z == 7 && kind[5] == 2) ? (T)1 - cf5 : (T)1;
    const T wxp0 = kind[0] == 2 ? (T)1 - cf5 : (T)1, wxm7 = kind[1] == 2 ? (T)1 - cf5 : (T)1;
    const T den = ih2y * ((T)2 - aym - ayp) + ih2z * ((T)2 - azm - azp) + (T)2 * ih2x;
    __syncthreads();
    T s4[4];
#pragma unroll
    for (int cx = 0; cx < 4; ++cx) {
        T pair = (T)0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int x = 2 * cx + q;
            const T xm = x == 0 ? hs[0] : u[x - 1], xp = x == 7 ? hs[1] : u[x + 1];
            const T wxm = x == 7 ? wxm7 : (T)1, wxp = x == 0 ? wxp0 : (T)1;
            const T dc = den - (x == 0 ? ih2x * ag[0] : (T)0) - (x == 7 ? ih2x * ag[1] : (T)0);
            const T Au = dc * u[x] - (ih2x * (wxm * xm + wxp * xp) + ih2y * (wym * rows[rym + x] + wyp * rows[ryp + x]) +
                                      ih2z * (wzm * rows[rzm + x] + wzp * rows[rzp + x]));
            pair += rr[x] - Au;
        }
        pair += __shfl_xor(pair, 1, 64);
        pair += __shfl_xor(pair, 8, 64);
        s4[cx] = (T)0.125 * pair;
    }
    if (active && !(y & 1) && !(z & 1)) {
        const int p = M.par[b], oc = p & 7;
        const int Y = ((oc >> 1) & 1) * 4 + (y >> 1), Z = (oc >> 2) * 4 + (z >> 1);
        T *dst = r + (size_t)(p >> 3) * BRICK_CELLS + (oc & 1) * 4 + 8 * Y + 64 * Z;
#pragma unroll
        for (int cx = 0; cx < 4; ++cx) dst[cx] = s4[cx];
    }
}

// Uncovered coarse cells next to covered ones: r -= B_fine e^l, i.e. add
// 1/(2 h_d^2) * sum over the 4 fine faces of (e_f/3 + e_in/5) per coarse-fine
// face (the coarse correction is still zero), from the fine sums ffs of e.
// FP64 arithmetic.  One wavefront per coarse brick, lane (y, z) its row: the
// sums come by half rows, all directions in flight, as far as the row has
// them (see k_outer_residual); only uncovered halves are written, the others
// belong to the restriction.
template <class T>
__device__ __forceinline__ void reflux_brick(const DevMeta &M, int b, bool active, const double *ffs, T *r, int *kids)
{
    const int lane = threadIdx.x & 63, y = lane & 7, z = lane >> 3;
    const LevelConst L = M.lc[M.org[b].w];
    const uint32_t cm = M.cmask[b];
    uint32_t ncm[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int n = M.nbr[b * 6 + f];
        ncm[f] = n >= 0 ? (uint32_t)M.cmask[n] : 0u;
    }
    if (lane < 56) {
        const int nbl = lane < 48 ? M.nbr[b * 6 + (lane >> 3)] : b;
        kids[lane] = nbl >= 0 ? M.child[nbl * 8 + (lane & 7)] : -1;
    }
    T rt[8];
    T *row = r + (size_t)b * BRICK_CELLS + 8 * lane;
    Row8<T>::load(row, rt);
    wave_fence();
    const int ozy = ((y >> 2) << 1) | ((z >> 2) << 2);  // the row's octants: ozy, ozy | 1
    const bool cov[2] = {((cm >> ozy) & 1) != 0, ((cm >> (ozy | 1)) & 1) != 0};
    double add[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) add[i] = 0.0;
    bool on[4][2];
    double2 a[4][2], c[4][2];
#pragma unroll
    for (int f = 2; f < 6; ++f) {
        const int d = f >> 1, s = f & 1, q = (d == 1 ? y : z) + (s ? 1 : -1), l = q & 7;
        const bool inside = q == l;
        const int qo = d == 1 ? ((l >> 2) << 1) | ((z >> 2) << 2) : ((y >> 2) << 1) | ((l >> 2) << 2);
        const uint32_t nm = inside ? cm : ncm[f];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            on[f - 2][h] = !cov[h] && ((nm >> (qo | h)) & 1);
            a[f - 2][h] = c[f - 2][h] = make_double2(0.0, 0.0);
            if (on[f - 2][h]) {
                const int F = kids[(inside ? 48 : 8 * f) + (qo | h)];
                const double2 *p = (const double2 *)(ffs + ((size_t)F * 6 + 2 * d + 1 - s) * 16 +
                                                     4 * ((d == 1 ? z : y) & 3));
                a[f - 2][h] = p[0], c[f - 2][h] = p[1];
            }
        }
    }
    // along x: the cells next to the other half, and the row's ends
    const int m = (y & 3) + 4 * (z & 3);
    const bool in3 = !cov[0] && cov[1], in4 = cov[0] && !cov[1];
    const bool end0 = !cov[0] && ((ncm[0] >> (ozy | 1)) & 1), end7 = !cov[1] && ((ncm[1] >> ozy) & 1);
    double fi = 0.0, f0 = 0.0, f7 = 0.0;
    if (in3) fi = ffs[((size_t)kids[48 + (ozy | 1)] * 6 + 0) * 16 + m];
    if (in4) fi = ffs[((size_t)kids[48 + ozy] * 6 + 1) * 16 + m];
    if (end0) f0 = ffs[((size_t)kids[ozy | 1] * 6 + 1) * 16 + m];
    if (end7) f7 = ffs[((size_t)kids[8 + ozy] * 6 + 0) * 16 + m];
    if (end0) add[0] += 0.5 * L.ih2[0] * f0;
    if (in3) add[3] += 0.5 * L.ih2[0] * fi;
    if (in4) add[4] += 0.5 * L.ih2[0] * fi;
    if (end7) add[7] += 0.5 * L.ih2[0] * f7;
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (on[f][h]) {
                const double ih2 = L.ih2[1 + (f >> 1)];
                add[4 * h] += 0.5 * ih2 * a[f][h].x;
                add[4 * h + 1] += 0.5 * ih2 * a[f][h].y;
                add[4 * h + 2] += 0.5 * ih2 * c[f][h].x;
                add[4 * h + 3] += 0.5 * ih2 * c[f][h].y;
            }
    if (!active) return;
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (!cov[h])
#pragma unroll
            for (int i = 4 * h; i < 4 * h + 4; ++i)
                if (add[i] != 0.0) row[i] = (T)((double)rt[i] + add[i]);
}

// One launch per level step: the restriction of the nb fine bricks from b0
// into their parents (covered coarse cells), then the coarse-fine update of
// the nrf listed coarse bricks (uncovered cells) -- disjoint cells, so the
// two kinds of workgroups run together.
// Workgroups of 128 threads, a wavefront per brick: the first (nrf + 1) / 2
// update two listed coarse bricks each (the longer chain starts first), the
// others restrict two fine bricks each.  64^3 + 2 levels 9.4 and 8.1 us a
// launch -> 6.3 and 5.0, 2.7e7 cells 68 -> 54, a batch of sixteen 13.8 -> 9.7.
template <class T>
__global__ void __launch_bounds__(128) k_restrict(DevMeta M, int b0, int nb, const int32_t *rlist, int nrf,
                                                  const T *e, T *r, const double *ffs)
{
    __shared__ T rows[2][RW * RW * RS];
    __shared__ int kids[2][56];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nwf = (nrf + 1) / 2, nwr = (nb + 1) / 2;
    if ((int)blockIdx.x >= nwf) {
        const int k = xcd_remap(blockIdx.x - nwf, nwr) * 2 + w;
        restrict_brick<T>(M, __builtin_amdgcn_readfirstlane(b0 + (k < nb ? k : nb - 1)), k < nb, e, r, rows[w]);
    } else {
        const int k = xcd_remap(blockIdx.x, nwf) * 2 + w;
        reflux_brick<T>(M, __builtin_amdgcn_readfirstlane(rlist[k < nrf ? k : nrf - 1]), k < nrf, ffs, r, kids[w]);
    }
}

// e^l += I e^{l-1}: piecewise-constant injection of the parent value
template <class T>
__global__ void __launch_bounds__(256) k_prolong(DevMeta M, int b0, int nb, T *e)
{
    int b = b0 + xcd_remap(blockIdx.x, nb);
    int par = M.par[b];
    int pb = par >> 3, oc = par & 7;
    int ox = (oc & 1) * 4, oy = ((oc >> 1) & 1) * 4, oz = (oc >> 2) * 4;
    for (int c = threadIdx.x; c < BRICK_CELLS; c += 256) {
        int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
        size_t li = (size_t)b * BRICK_CELLS + c;
        size_t pi = (size_t)pb * BRICK_CELLS + (ox + (x >> 1)) + 8 * (oy + (y >> 1)) + 64 * (oz + (z >> 1));
        e[li] = (T)((double)e[li] + (double)e[pi]);
    }
}

// phi += e on AMR bricks (FP64 accumulation of the correction; brick layout)
template <class T>
__global__ void __launch_bounds__(256) k_phi_update(DevMeta M, int b0, int nb, double *phib, const T *e,
                                                    const int32_t *list)
{
    int b = pick_brick(b0, nb, list, blockIdx.x);
    for (int c = threadIdx.x; c < BRICK_CELLS; c += 256) {
        size_t i = (size_t)b * BRICK_CELLS + c;
        phib[i] += (double)e[i];
    }
}

// phi^{l} <- U phi^l + R phi^{l+1} for the covered cells under a range of
// fine bricks (Alg. 2, average down; brick layout)
__global__ void __launch_bounds__(256) k_avgdown(DevMeta M, int b0, int nb, double *phib)
{
    int nwg = (nb + 3) >> 2;
    int w = xcd_remap(blockIdx.x, nwg);
    int k = w * 4 + (threadIdx.x >> 6);
    if (k >= nb) return;
    int b = b0 + k;
    int t = threadIdx.x & 63;
    int cx = t & 3, cy = (t >> 2) & 3, cz = t >> 4;
    const double *u = phib + (size_t)b * BRICK_CELLS;
    double s = 0.0;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) s += u[(2 * cx + dx) + 8 * (2 * cy + dy) + 64 * (2 * cz + dz)];
    int par = M.par[b];
    int pb = par >> 3, oc = par & 7;
    int X = (oc & 1) * 4 + cx, Y = ((oc >> 1) & 1) * 4 + cy, Z = (oc >> 2) * 4 + cz;
    phib[(size_t)pb * BRICK_CELLS + X + 8 * Y + 64 * Z] = 0.125 * s;
}

// E_d = -(u_+ - u_-) / (2 h_d) on every cell of a range of AMR bricks (phi in
// brick layout) and phi itself into the caller's layout, in the row layout of
// the outer residual: one wavefront per brick.  Bound by its bytes, 8 read and
// 32 written per cell: 576^3 + 2 levels (2.1e8 cells) 2005 us, 4.2 TB/s; with
// phi in a pass of its own 2045 + 683, and with a lane storing its whole row
// (64 bytes apart from the next lane's) 2900.
template <int BPW>
__global__ void __launch_bounds__(64 * BPW) k_efield(DevMeta M, int b0, int nb, const double *phib,
                                                     const double *cp_phi, double *const *E, double *const *phi,
                                                     const int32_t *list)
{
    __shared__ double rows_all[BPW][RW * RW * RS];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int k0 = xcd_remap(blockIdx.x, (nb + BPW - 1) / BPW) * BPW + w;
    const bool active = k0 < nb;
    const int kk = active ? k0 : nb - 1;
    const int b = __builtin_amdgcn_readfirstlane(list ? list[kk] : b0 + kk);
    double *rows = rows_all[w];
    const int y = lane & 7, z = lane >> 3;
    const int lev = M.org[b].w;
    const LevelConst L = M.lc[lev];
    int nbf[6], kind[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        nbf[f] = M.nbr[b * 6 + f];
        kind[f] = nbf[f] >= 0 ? 0 : ((-1 - nbf[f]) < M.nbc ? 1 : 2);
    }
    double u[8], hs[6];
    Row8<double>::load(phib + (size_t)b * BRICK_CELLS + 8 * lane, u);
    // halo slots: the neighbour's phi, 2 g on the boundary, or the coarse part
    // of the coarse-fine ghost
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, md = (f & 1) ? 0 : 7, uu = lane & 7, vv = lane >> 3;
        const int c = d == 0 ? md + 8 * uu + 64 * vv : (d == 1 ? uu + 8 * md + 64 * vv : uu + 8 * vv + 64 * md);
        hs[f] = kind[f] == 0   ? phib[(size_t)nbf[f] * BRICK_CELLS + c]
                : kind[f] == 1 ? 2.0 * M.gbc[(size_t)(-1 - nbf[f]) * 64 + lane]
                               : cp_phi[(size_t)(-1 - nbf[f] - M.nbc) * 64 + lane];
    }
    const int rym = rrow(y - 1, z), ryp = rrow(y + 1, z), rzm = rrow(y, z - 1), rzp = rrow(y, z + 1), rme = rrow(y, z);
#pragma unroll
    for (int i = 0; i < 8; ++i) rows[rme + i] = u[i];
    rows[rrow(-1, lane >> 3) + (lane & 7)] = hs[2];
    rows[rrow(8, lane >> 3) + (lane & 7)] = hs[3];
    rows[rrow(lane >> 3, -1) + (lane & 7)] = hs[4];
    rows[rrow(lane >> 3, 8) + (lane & 7)] = hs[5];
    const double a0 = L.abnd[0], a1 = L.abnd[1], a2 = L.abnd[2];
    __syncthreads();
    if (!active) return;
    // the neighbour's value across a face of kind k from its halo slot v, the
    // cell uc and the cell further inside
    auto ghost = [](int k, double a, double v, double uc, double in) {
        return k == 0 ? v : (k == 1 ? a * uc + v : (2.0 / 3.0) * uc + (v - 0.2 * in));
    };
    double ex[8], ey[8], ez[8];
    const double h2x = 2.0 * L.h[0], h2y = 2.0 * L.h[1], h2z = 2.0 * L.h[2];
    const int kym = y == 0 ? kind[2] : 0, kyp = y == 7 ? kind[3] : 0;
    const int kzm = z == 0 ? kind[4] : 0, kzp = z == 7 ? kind[5] : 0;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const double um = x == 0 ? ghost(kind[0], a0, hs[0], u[0], u[1]) : u[x - 1];
        const double up = x == 7 ? ghost(kind[1], a0, hs[1], u[7], u[6]) : u[x + 1];
        ex[x] = -(up - um) / h2x;
        const double vm = rows[rym + x], vp = rows[ryp + x], wm = rows[rzm + x], wp = rows[rzp + x];
        ey[x] = -(ghost(kyp, a1, vp, u[x], vm) - ghost(kym, a1, vm, u[x], vp)) / h2y;
        ez[x] = -(ghost(kzp, a2, wp, u[x], wm) - ghost(kzm, a2, wm, u[x], wp)) / h2z;
    }
    // out through the rows in LDS, eight lanes a row, so that each store
    // instruction fills whole 64-byte segments
    const int2 us = M.ustr[b];
    const int64_t ub = M.ubase[b] + (lane & 7) + (int64_t)us.x * (lane >> 3);
    auto store = [&](double *to) {
        wave_fence();
#pragma unroll
        for (int k = 0; k < 8; ++k) to[ub + (int64_t)us.y * k] = rows[rrow(lane >> 3, k) + (lane & 7)];
        wave_fence();
    };
    auto stage = [&](const double (&v)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) rows[rme + i] = v[i];
    };
    store(phi[lev]);
    stage(ex);
    store(E[3 * lev]);
    stage(ey);
    store(E[3 * lev + 1]);
    stage(ez);
    store(E[3 * lev + 2]);
}

// ---------------------------------------------------------------------------
// CG on the coarsest grid, one workgroup of 1024 threads (FP64 vectors and
// dot products).  Homogeneous boundary data, no coarse-fine faces.
// ---------------------------------------------------------------------------
__device__ double block_reduce_1024(double v)
{
    __shared__ double sh[16];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double r = 0.0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) r += sh[i];
    __syncthreads();
    return r;
}

// CG on bricks [b0, b0+nb) of one level with four FP64 work vectors; called
// by a whole workgroup of 1024 threads.  Returns the iteration count.
template <class T>
__device__ int cg_solve(const DevMeta &M, int b0, int nb, const T *rhs, T *e, double *work, double rtol, int maxit)
{
    const int n = nb * BRICK_CELLS;
    double *x = work, *r = x + n, *p = x + 2 * (size_t)n, *q = x + 3 * (size_t)n;
    double rho = 0.0;
    for (int i = threadIdx.x; i < n; i += (int)blockDim.x) {
        double v = (double)rhs[(size_t)b0 * BRICK_CELLS + i];
        x[i] = 0.0;
        r[i] = v;
        p[i] = v;
        rho += v * v;
    }
    rho = block_reduce_1024(rho);
    double stop = rtol * rtol * rho;
    int it = 0;
    OffsetAcc pacc{p, b0};
    const LevelConst L = M.lc[M.org[b0].w];
    while (it < maxit && rho > stop && rho > 0.0) {
        double pq = 0.0;
        for (int i = threadIdx.x; i < n; i += (int)blockDim.x) {
            int b = b0 + (i >> 9), c = i & 511;
            int lc[3] = {c & 7, (c >> 3) & 7, c >> 6};
            double pc = p[i], Ap = 0.0;
            for (int d = 0; d < 3; ++d)
                for (int s = -1; s <= 1; s += 2) {
                    double a, bv;
                    face_nb(M, b, lc, d, s, pacc, nullptr, nullptr, false, a, bv);
                    Ap += L.ih2[d] * ((1.0 - a) * pc - bv);
                }
            q[i] = Ap;
            pq += pc * Ap;
        }
        pq = block_reduce_1024(pq);
        double alpha = rho / pq;
        double rho1 = 0.0;
        for (int i = threadIdx.x; i < n; i += (int)blockDim.x) {
            x[i] += alpha * p[i];
            double rv = r[i] - alpha * q[i];
            r[i] = rv;
            rho1 += rv * rv;
        }
        rho1 = block_reduce_1024(rho1);
        double beta = rho1 / rho;
        for (int i = threadIdx.x; i < n; i += (int)blockDim.x) p[i] = r[i] + beta * p[i];
        rho = rho1;
        ++it;
        __syncthreads();
    }
    for (int i = threadIdx.x; i < n; i += (int)blockDim.x) e[(size_t)b0 * BRICK_CELLS + i] = (T)x[i];
    __syncthreads();
    return it;
}

// CG as above for grids of at most 4096 cells: the search direction lives in
// LDS, each thread keeps its (at most four) cells of x, r and q in registers,
// and a reduction costs one barrier.
constexpr int CG_LDS_MAX = 4096;
constexpr int CG_PER = 8;  // cells per thread: CG_LDS_MAX / CG_PER threads at least

__device__ __forceinline__ double wg_sum_1024(double v, double *red, int slot)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) red[slot * 16 + (threadIdx.x >> 6)] = v;
    __syncthreads();
    double s = 0.0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) s += red[slot * 16 + i];
    return s;
}

template <class T>
__device__ int cg_solve_lds(const DevMeta &M, int b0, int nb, const T *rhs, T *e, double rtol, int maxit, double *p)
{
    __shared__ double red[3 * 16];
    const int n = nb * BRICK_CELLS;
    const LevelConst L = M.lc[M.org[b0].w];
    // neighbours of each owned cell (at most CG_PER per thread), resolved once: LDS index, or -1 for a
    // homogeneous boundary ghost (abnd p_c, in the diagonal); the coarsest
    // grid has no coarse-fine faces
    int nbi[CG_PER][6];
    double diag[CG_PER];
    for (int k = 0; k < CG_PER; ++k) {
        int i = threadIdx.x + (int)blockDim.x * k;
        diag[k] = 0.0;
        for (int f = 0; f < 6; ++f) nbi[k][f] = -1;
        if (i >= n) continue;
        int b = b0 + (i >> 9), c = i & 511;
        int l[3] = {c & 7, (c >> 3) & 7, c >> 6};
        for (int f = 0; f < 6; ++f) {
            int d = f >> 1, s = (f & 1) ? 1 : -1;
            int m[3] = {l[0], l[1], l[2]};
            m[d] += s;
            int bb = b;
            if (m[d] < 0 || m[d] > 7) {
                bb = M.nbr[b * 6 + f];
                m[d] = s > 0 ? 0 : 7;
            }
            if (bb >= 0) {
                nbi[k][f] = (bb - b0) * BRICK_CELLS + m[0] + 8 * m[1] + 64 * m[2];
                diag[k] += L.ih2[d];
            } else {
                diag[k] += (1.0 - L.abnd[d]) * L.ih2[d];
            }
        }
    }
    double x[CG_PER], r[CG_PER];
    double rho = 0.0;
    for (int k = 0; k < CG_PER; ++k) {
        int i = threadIdx.x + (int)blockDim.x * k;
        double v = i < n ? (double)rhs[(size_t)b0 * BRICK_CELLS + i] : 0.0;
        x[k] = 0.0;
        r[k] = v;
        if (i < n) p[i] = v;
        rho += v * v;
    }
    int slot = 0;
    rho = wg_sum_1024(rho, red, slot);
    slot = (slot + 1) % 3;
    double stop = rtol * rtol * rho;
    int it = 0;
    while (it < maxit && rho > stop && rho > 0.0) {
        double q[CG_PER], pk[CG_PER], pq = 0.0;
        for (int k = 0; k < CG_PER; ++k) {
            int i = threadIdx.x + (int)blockDim.x * k;
            q[k] = 0.0;
            pk[k] = 0.0;
            if (i >= n) continue;
            double pc = p[i], off = 0.0;
            for (int f = 0; f < 6; ++f)
                if (nbi[k][f] >= 0) off += L.ih2[f >> 1] * p[nbi[k][f]];
            pk[k] = pc;
            q[k] = diag[k] * pc - off;
            pq += pc * q[k];
        }
        pq = wg_sum_1024(pq, red, slot);
        slot = (slot + 1) % 3;
        double alpha = rho / pq;
        double rho1 = 0.0;
        for (int k = 0; k < CG_PER; ++k) {
            x[k] += alpha * pk[k];
            r[k] -= alpha * q[k];
            rho1 += r[k] * r[k];
        }
        rho1 = wg_sum_1024(rho1, red, slot);
        slot = (slot + 1) % 3;
        double beta = rho1 / rho;
        for (int k = 0; k < CG_PER; ++k) {
            int i = threadIdx.x + (int)blockDim.x * k;
            if (i < n) p[i] = r[k] + beta * pk[k];
        }
        __syncthreads();
        rho = rho1;
        ++it;
    }
    for (int k = 0; k < CG_PER; ++k) {
        int i = threadIdx.x + (int)blockDim.x * k;
        if (i < n) e[(size_t)b0 * BRICK_CELLS + i] = (T)x[k];
    }
    __syncthreads();
    return it;
}

// ---------------------------------------------------------------------------
// Exact solve of the coarsest grid (one box, homogeneous boundary ghosts) by
// its separable eigendecomposition: e = Q diag(1/lambda) Q^T r with Q the
// tensor product of the per-axis orthonormal eigenvector matrices.  Three
// launches over all jobs: forward transforms along x and y per (z plane, block
// of 16 x frequencies); along z per group of 16 columns (forward, division by
// the eigenvalue sum, inverse); inverse along x and y per (plane, block).  The
// work is dense FP64 products, bound by the matrix-core rate, so it is cut
// into 16-wide blocks to occupy every CU (a 64^3 grid gives 256 workgroups per
// launch).  FP64 scratch in natural order (x fastest).
// ---------------------------------------------------------------------------
__device__ __forceinline__ size_t direct_cell(const DirectJob &J, int x, int y, int z)
{
    const int nbx = J.dn[0] >> 3, nby = J.dn[1] >> 3;
    int b = J.b0 + (x >> 3) + nbx * ((y >> 3) + nby * (z >> 3));
    return (size_t)b * BRICK_CELLS + (x & 7) + 8 * (y & 7) + 64 * (z & 7);
}

__device__ __forceinline__ int pad16(int n) { return (n + 15) & ~15; }

typedef double dbl4 __attribute__((ext_vector_type(4)));

// Products on the FP64 matrix cores, one 16 x 16 output tile per wavefront:
// C[r][k] = sum_i Tb[r][i] D[k][i] with the table Tb (K x K, zero-padded, in
// global memory in operand order) and the data D (K values per row).
// v_mfma_f64 16x16x4 takes Tb[r0 + l%16][i] and D[k0 + l%16][i] from lane l,
// each quarter of the wavefront (l/16) its own i, and returns C[r0 + l/16 +
// 4j][k0 + l%16] in element j, so consecutive lanes hold consecutive k.  Which
// i a step takes is free as long as both operands agree: quarter g takes the
// four consecutive i = 16 c + 4 g + q in the four steps q of chunk c, so a
// lane's operands of a chunk are one 32-byte piece of its row, of the table as
// of the data, and the data come straight from global memory (a brick row, a
// row of the scratch) without a detour through LDS.
//
// Bound by the latency of the chain launch, loads, 16 matrix steps (64^3), LDS,
// 16 steps, stores, not by the matrix cores' rate.  With the data staged in
// LDS first (two more barriers, one 87 KB workgroup a CU at 72 x 56 x 88) the
// three launches took 31 us at 64^3, 68 at 72 x 56 x 88, 18 at 32^3 and 62 for
// a batch of sixteen; now 19, 26, 10 and 38.
// threads of the column transform: up to eight 16-row tiles go to as many
// wavefronts (72 cells an axis 16.0 -> 13.2 us; the plane transforms, in more
// workgroups than CUs, lose that way, 11.6 -> 14.4)
constexpr int dst_threads(int NC) { return NC > 4 ? 512 : 256; }
template <int NC>
struct DOp {
    double v[NC][4];
};
// this lane's operands of row block r0 of a table: chunk c, step q
template <int NC>
__device__ __forceinline__ void dst_rows(const double *Tb, int K, int r0, DOp<NC> &t)
{
    const double *p = Tb + (size_t)(r0 >> 4) * (K >> 4) * 256 + 4 * (threadIdx.x & 63);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (16 * c < K)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double2 a = *(const double2 *)(p + 256 * c + 2 * h);
                t.v[c][2 * h] = a.x, t.v[c][2 * h + 1] = a.y;
            }
    }
}
// rows of ld values in LDS: D[k0 + l%16][..]
template <int NC>
__device__ __forceinline__ void dst_lds(const double *D, int ld, int K, DOp<NC> &d)
{
    const double *p = D + (threadIdx.x & 15) * ld + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (16 * c < K)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double2 a = *(const double2 *)(p + 16 * c + 2 * h);
                d.v[c][2 * h] = a.x, d.v[c][2 * h + 1] = a.y;
            }
}
template <int NC>
__device__ __forceinline__ dbl4 dst_mfma(const DOp<NC> &t, const DOp<NC> &d, int K)
{
    dbl4 a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};  // two chains (even and odd steps)
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (16 * c < K)
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(t.v[c][q], d.v[c][q], a0, 0, 0, 0);
                a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(t.v[c][q + 1], d.v[c][q + 1], a1, 0, 0, 0);
            }
    return a0 + a1;
}
// four consecutive values of T as doubles
__device__ __forceinline__ void load4(const float *p, double (&v)[4])
{
    const float4 a = *(const float4 *)p;
    v[0] = (double)a.x, v[1] = (double)a.y, v[2] = (double)a.z, v[3] = (double)a.w;
}
__device__ __forceinline__ void load4(const double *p, double (&v)[4])
{
    const double2 a = *(const double2 *)p, b = *(const double2 *)(p + 2);
    v[0] = a.x, v[1] = a.y, v[2] = b.x, v[3] = b.y;
}

// table pool layout per job: forward and inverse matrices of x, y, z, each
// P_d x P_d with P_d = pad16(n_d), zero-padded, in matrix-core operand order
// (dst_rows); then the eigenvalues of x, y, z (n_d each)
__device__ __forceinline__ const double *dst_table(const DirectJob &J, const double *tab, int d, bool inv)
{
    const int px = pad16(J.dn[0]), py = pad16(J.dn[1]), pz = pad16(J.dn[2]);
    int off = J.tab;
    if (d >= 1) off += 2 * px * px;
    if (d >= 2) off += 2 * py * py;
    const int p = d == 0 ? px : (d == 1 ? py : pz);
    return tab + off + (inv ? p * p : 0);
}

// transforms along x and y of one z plane for one block of 16 x-frequencies
// kx (x positions on the inverse), forward (r -> W) or inverse (W -> e,
// phi += e): the x transform of the whole plane restricted to the block,
// then the y transform of the block.  planes[i] = (job, z | block << 8), or
// with jobs == nullptr the one job J1 and workgroup z * blocks + block.
// NC: chunks of 16 of the longest edge.
template <class T, bool INV, int NC>
__global__ void __launch_bounds__(256) k_dst_plane(const DirectJob *jobs, const int2 *planes, DirectJob J1,
                                                   const double *tab, double *W, const T *r, T *e, double *phib,
                                                   int phi_update)
{
    constexpr int LD = 16 * NC + 2;  // (16-byte rows whose starts fall in different banks)
    __shared__ double Bt[16 * LD];   // x-transformed block [kx - kx0][y]
    // one job (jobs == nullptr): J1, workgroup = z * blocks + block; else from the lists
    int z, kb;
    DirectJob J;
    if (!jobs) {
        J = J1;
        const int nkb = pad16(J.dn[0]) >> 4;
        z = blockIdx.x / nkb;
        kb = blockIdx.x - z * nkb;
    } else {
        const int2 pl = planes[blockIdx.x];
        J = jobs[pl.x];
        z = pl.y & 255;
        kb = pl.y >> 8;
    }
    const int nx = J.dn[0], ny = J.dn[1], kx0 = kb << 4, np = nx * ny;
    const int px = pad16(nx), py = pad16(ny);
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double *w = W + J.w + (size_t)np * z;
    const double *Mx = dst_table(J, tab, 0, INV), *My = dst_table(J, tab, 1, INV);
    DOp<NC> tx, ty;
    dst_rows<NC>(Mx, px, kx0, tx);
    // along x: Bt[kx - kx0][y] = sum_x Mx[kx][x] plane[y][x], 16 rows y a tile
    for (int y0 = wave << 4; y0 < py; y0 += 64) {
        const int y = y0 + lr;
        DOp<NC> d;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int x = 16 * c + 4 * lk;
#pragma unroll
            for (int q = 0; q < 4; ++q) d.v[c][q] = 0.0;
            if (y < ny && x < nx) {
                if (INV) load4(w + y * nx + x, d.v[c]);
                else load4(r + direct_cell(J, x, y, z), d.v[c]);
            }
        }
        if (y0 == (wave << 4)) dst_rows<NC>(My, py, y0, ty);  // in flight with the plane
        const dbl4 s = dst_mfma<NC>(tx, d, px);
#pragma unroll
        for (int j = 0; j < 4; ++j) Bt[(lk + 4 * j) * LD + y] = s[j];
    }
    __syncthreads();
    // along y: out[ky][kx] = sum_y My[ky][y] Bt[kx - kx0][y], 16 rows ky a tile
    DOp<NC> d;
    dst_lds<NC>(Bt, LD, py, d);
    const int x = kx0 + lr;
    for (int y0 = wave << 4; y0 < py; y0 += 64) {
        if (y0 != (wave << 4)) dst_rows<NC>(My, py, y0, ty);
        const dbl4 s = dst_mfma<NC>(ty, d, py);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int y = y0 + lk + 4 * j;
            if (x >= nx || y >= ny) continue;
            if (!INV) {
                w[y * nx + x] = s[j];
            } else {
                const size_t bi = direct_cell(J, x, y, z);
                e[bi] = (T)s[j];
                if (phi_update && J.amr) phib[bi] += s[j];
            }
        }
    }
}

// transform along z of a group of DIRECT_COLS = 16 columns: forward, division
// by the eigenvalue sum, inverse.  groups[i] = (job, first column), or with
// jobs == nullptr the one job J1 and columns from DIRECT_COLS * workgroup.
template <int NC>
__global__ void __launch_bounds__(dst_threads(NC)) k_dst_column(const DirectJob *jobs, const int2 *groups, DirectJob J1,
                                                    const double *tab, double *W)
{
    static_assert(DIRECT_COLS == 16, "one matrix-core tile of columns");
    constexpr int LD = 16 * NC + 2;
    __shared__ double C[16 * LD];  // [column][kz]
    DirectJob J;
    int c0;  // np is a multiple of DIRECT_COLS
    if (!jobs) {  // one job: J1, workgroup = column group
        J = J1;
        c0 = blockIdx.x * DIRECT_COLS;
    } else {
        const int2 gr = groups[blockIdx.x];
        J = jobs[gr.x];
        c0 = gr.y;
    }
    const int nx = J.dn[0], ny = J.dn[1], nz = J.dn[2], np = nx * ny, pz = pad16(nz);
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double *mux = dst_table(J, tab, 2, false) + 2 * pz * pz, *muy = mux + nx, *muz = muy + ny;
    const double *Fz = dst_table(J, tab, 2, false), *Bz = dst_table(J, tab, 2, true);
    const int col = c0 + lr;
    double *w = W + J.w + col;
    DOp<NC> tf, tb, d;
    // (a wavefront without a tile of its own loads nothing)
    if ((wave << 4) < pz) {
        dst_rows<NC>(Fz, pz, wave << 4, tf);
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int zz = 16 * c + 4 * lk + q;
                d.v[c][q] = zz < nz ? w[(size_t)np * zz] : 0.0;
            }
        dst_rows<NC>(Bz, pz, wave << 4, tb);
    }
    const double mxy = mux[col % nx] + muy[col / nx];
    // forward, then the division by the eigenvalue sum of (column, kz)
    for (int z0 = wave << 4; z0 < pz; z0 += dst_threads(NC) / 4) {
        double mz[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) mz[j] = z0 + lk + 4 * j < nz ? muz[z0 + lk + 4 * j] : 1.0;
        if (z0 != (wave << 4)) dst_rows<NC>(Fz, pz, z0, tf);
        const dbl4 s = dst_mfma<NC>(tf, d, pz);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kz = z0 + lk + 4 * j;
            C[lr * LD + kz] = kz < nz ? s[j] / (mxy + mz[j]) : 0.0;
        }
    }
    __syncthreads();
    dst_lds<NC>(C, LD, pz, d);
    for (int z0 = wave << 4; z0 < pz; z0 += dst_threads(NC) / 4) {
        if (z0 != (wave << 4)) dst_rows<NC>(Bz, pz, z0, tb);
        const dbl4 s = dst_mfma<NC>(tb, d, pz);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int zz = z0 + lk + 4 * j;
            if (zz < nz) w[(size_t)np * zz] = s[j];
        }
    }
}

// exact red-black Gauss-Seidel pass over a whole level by one workgroup
template <class T>
__device__ void wg_gs_pass(const DevMeta &M, int b0, int nb, T *e, const T *r, int colour)
{
    const LevelConst L = M.lc[M.org[b0].w];
    for (int i = threadIdx.x; i < nb * 256; i += (int)blockDim.x) {
        int b = b0 + (i >> 8), t = i & 255;
        int z = t >> 5, y = (t >> 2) & 7, xx = (t & 3) << 1;
        int lc[3] = {xx + (((y + z) & 1) ^ colour), y, z};
        size_t li = (size_t)b * BRICK_CELLS + lc[0] + 8 * y + 64 * z;
        double num = (double)r[li], den = 0.0;
        for (int d = 0; d < 3; ++d)
            for (int s = -1; s <= 1; s += 2) {
                double a, bv;
                face_nb(M, b, lc, d, s, BrickAcc<T>{e}, nullptr, nullptr, false, a, bv);
                num += L.ih2[d] * bv;
                den += L.ih2[d] * (1.0 - a);
            }
        e[li] = (T)(num / den);
    }
    __syncthreads();
}

// The part of the V-cycle on the small levels 0..nlev-1 of one problem (no
// coarse-fine faces there) in one workgroup: pre-smoothing and restriction
// down, CG on level 0, prolongation and post-smoothing up, and phi += e on
// AMR levels when phi_update is set.
template <class T>
__global__ void __launch_bounds__(1024) k_coarse_cycle(DevMeta M, const CoarseJob *jobs, T *e, T *r, double *work,
                                                       int nu1, int nu2, double rtol, int maxit, int *iters,
                                                       double *phib, int phi_update)
{
    __shared__ double lds[CG_LDS_MAX];
    const CoarseJob J = jobs[blockIdx.x];
    if (J.direct) return;  // solved by the transform kernels
    for (int k = J.nlev - 1; k >= 1; --k) {
        const int b0 = J.b0[k], nb = J.nb[k];
        for (int i = threadIdx.x; i < nb * BRICK_CELLS; i += (int)blockDim.x) e[(size_t)b0 * BRICK_CELLS + i] = (T)0;
        __syncthreads();
        for (int it = 0; it < nu1; ++it) {
            wg_gs_pass<T>(M, b0, nb, e, r, 0);
            wg_gs_pass<T>(M, b0, nb, e, r, 1);
        }
        const LevelConst L = M.lc[M.org[b0].w];
        for (int i = threadIdx.x; i < nb * 64; i += (int)blockDim.x) {
            int b = b0 + (i >> 6), t = i & 63;
            int cx = t & 3, cy = (t >> 2) & 3, cz = t >> 4;
            double sum = 0.0;
            for (int dz = 0; dz < 2; ++dz)
                for (int dy = 0; dy < 2; ++dy)
                    for (int dx = 0; dx < 2; ++dx) {
                        int lc[3] = {2 * cx + dx, 2 * cy + dy, 2 * cz + dz};
                        sum += cell_residual(M, L, b, lc, e, r);
                    }
            int par = M.par[b];
            int pb = par >> 3, oc = par & 7;
            int X = (oc & 1) * 4 + cx, Y = ((oc >> 1) & 1) * 4 + cy, Z = (oc >> 2) * 4 + cz;
            r[(size_t)pb * BRICK_CELLS + X + 8 * Y + 64 * Z] = (T)(0.125 * sum);
        }
        __syncthreads();
    }
    int it;
    if (J.nb[0] * BRICK_CELLS <= CG_PER * (int)blockDim.x && J.nb[0] * BRICK_CELLS <= CG_LDS_MAX)
        it = cg_solve_lds<T>(M, J.b0[0], J.nb[0], r, e, rtol, maxit, lds);
    else
        it = cg_solve<T>(M, J.b0[0], J.nb[0], r, e, work + J.cg_off, rtol, maxit);
    if (threadIdx.x == 0 && iters) atomicMax(iters, it);
    for (int k = 0; k < J.nlev; ++k) {
        const int b0 = J.b0[k], nb = J.nb[k];
        if (k > 0) {
            for (int i = threadIdx.x; i < nb * BRICK_CELLS; i += (int)blockDim.x) {
                int b = b0 + (i >> 9), c = i & 511;
                int par = M.par[b];
                int pb = par >> 3, oc = par & 7;
                int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
                size_t pi = (size_t)pb * BRICK_CELLS + ((oc & 1) * 4 + (x >> 1)) +
                            8 * (((oc >> 1) & 1) * 4 + (y >> 1)) + 64 * ((oc >> 2) * 4 + (z >> 1));
                size_t li = (size_t)b * BRICK_CELLS + c;
                e[li] = (T)((double)e[li] + (double)e[pi]);
            }
            __syncthreads();
            for (int it2 = 0; it2 < nu2; ++it2) {
                wg_gs_pass<T>(M, b0, nb, e, r, 0);
                wg_gs_pass<T>(M, b0, nb, e, r, 1);
            }
        }
        if (phi_update && M.lc[M.org[b0].w].amr >= 0)
            for (int i = threadIdx.x; i < nb * BRICK_CELLS; i += (int)blockDim.x)
                phib[(size_t)b0 * BRICK_CELLS + i] += (double)e[(size_t)b0 * BRICK_CELLS + i];
    }
}

// ---------------------------------------------------------------------------
// particles
// ---------------------------------------------------------------------------
template <class P>
__device__ __forceinline__ bool cic_stencil(const DepLevel &D, double X, double Y, double Z, int *i0, int *i1,
                                            double *f)
{
    double xs[3] = {X, Y, Z};
    // (the level's numbers in one batch of scalar loads, not one an axis after
    // the axis before)
    bool in = true;
    for (int d = 0; d < 3; ++d) in = in & (xs[d] >= D.lo[d]) & (xs[d] < D.hi[d]);
    if (!in) return false;
    for (int d = 0; d < 3; ++d) {
        double s = div_by((xs[d] - D.lo[d]) * D.sc[d], D.hs[d], D.rh[d]) - 0.5;
        double fl = floor(s);
        int a = (int)fl;
        f[d] = s - fl;
        int b = a + 1;
        a = a < 0 ? 0 : (a > D.n[d] - 1 ? D.n[d] - 1 : a);
        b = b < 0 ? 0 : (b > D.n[d] - 1 ? D.n[d] - 1 : b);
        i0[d] = a;
        i1[d] = b;
    }
    return true;
}

__device__ __forceinline__ int64_t user_index(const DepLevel &D, const int64_t *ubase, const int2 *ustr, int i,
                                              int j, int k)
{
    int g = D.bmap[(i >> 3) + D.nbk[0] * ((j >> 3) + D.nbk[1] * (k >> 3))];
    if (g < 0) return -1;
    int2 s = ustr[g];
    return ubase[g] + (i & 7) + (int64_t)s.x * (j & 7) + (int64_t)s.y * (k & 7);
}

// Deposit every particle on every listed level.  A workgroup takes NT
// consecutive particles of the visiting order (spatially sorted, so they are
// close together) and, per level, accumulates their CIC weights in an LDS
// tile over the bounding box of their stencils, then adds the tile's nonzero
// cells to rho with one FP64 atomic each.  When the box exceeds the tile
// (sparse particles) each wavefront does the same alone, in its own part of
// the tile over the box of its own particles; one whose box exceeds that too
// adds every corner to rho by itself (then hardly any two are shared).
//
// Bounds: reading particles through the order (4e6 particles on 96^3 + 2
// levels: about 305 of 362 us, from four arrays; now 32-byte records, the
// whole deposit 183 us + 43 us to pack them); on dense levels the latency of
// a workgroup's chain, so its registers and LDS are kept to six workgroups a
// CU (9e6 particles on a level of 128^3 + 2, order kept: 209 -> 139 us, 1.5
// us per 1e5); on sparse ones the memory side's atomics, about 12 64-byte
// segments per nanosecond (1e7 particles on the finest level of 128^3 + 3:
// 494 -> 331 us).
// bricks whose layout a tile flush stages in LDS (a workgroup's tile; longer
// boxes look up each cell, a wavefront's go corner by corner)
constexpr int DEP_BRICKS = 64, DEP_WBRICKS = 32;

// minimum over the wavefront, in a scalar register
__device__ __forceinline__ int wave_min(int v)
{
#define AMRMG_DPP_MIN(ctrl, rmask) v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, ctrl, rmask, 0xf, false))
    AMRMG_DPP_MIN(0x111, 0xf);  // row_shr:1, 2, 4, 8: the minimum of each row of 16 lanes in its last lane
    AMRMG_DPP_MIN(0x112, 0xf);
    AMRMG_DPP_MIN(0x114, 0xf);
    AMRMG_DPP_MIN(0x118, 0xf);
    AMRMG_DPP_MIN(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
    AMRMG_DPP_MIN(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef AMRMG_DPP_MIN
    return __builtin_amdgcn_readlane(v, 63);
}

// such a box in LDS
struct DepBox : CellBox {
    // caller's-layout base (-1 outside the level) and strides of brick t of the box
    __device__ __forceinline__ void brick(const DepLevel &D, const int64_t *ubase, const int2 *ustr, int t, int64_t &ub,
                                          int2 &us) const
    {
        const int r = t / nbx, iz = r / nby;
        const int g = D.bmap[(bx0 + t - r * nbx) + D.nbk[0] * ((by0 + r - iz * nby) + D.nbk[1] * (bz0 + iz))];
        ub = -1;
        us = make_int2(0, 0);
        if (g >= 0) {
            ub = ubase[g];
            us = ustr[g];
        }
    }
    // the weights of one stencil into the tile: the 8 corners in an order
    // that the lane number turns (its bits exchange lower and upper along the
    // axes): the particles of a wavefront often share a stencil (the visiting
    // order keeps them together), and the same corner of one cell from every
    // lane at once would serialise the LDS atomics on one address
    __device__ __forceinline__ void add(double *acc, const int *i0, const int *i1, const double *f, double qv) const
    {
        const int st[3] = {1, ex, ex * ey};
        int o[3][2];
        double w[3][2];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const bool sw = (threadIdx.x >> d) & 1;
            const int u = (i1[d] - lo[d]) * st[d], v = (i0[d] - lo[d]) * st[d];
            const double g = 1.0 - f[d];
            o[d][0] = sw ? u : v;
            o[d][1] = sw ? v : u;
            w[d][0] = sw ? f[d] : g;
            w[d][1] = sw ? g : f[d];
        }
#pragma unroll
        for (int yz = 0; yz < 4; ++yz) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const double v = qv * (w[0][x] * w[1][yz & 1] * w[2][yz >> 1]);
                atomicAdd(&acc[o[0][x] + (o[1][yz & 1] + o[2][yz >> 1])], v);
            }
        }
    }
    // the tile's nonzero cells t0, t0 + step, ... to rho; tub, tus: the bricks' table, or tub == nullptr
    __device__ __forceinline__ void flush(const double *acc, int t0, int step, const int64_t *tub, const int2 *tus,
                                          const DepLevel &D, const int64_t *ubase, const int2 *ustr, double *rho) const
    {
        // quotients by ex and ey through the reciprocal (exact: t is below
        // 2^14, so (t + 1/2) / ex lies at least 1/(2 ex) from an integer, far
        // more than the product's rounding)
        const float rex = 1.0f / (float)ex, rey = 1.0f / (float)ey;
        for (int t = t0; t < (int)vol; t += step) {
            const double v = acc[t];
            if (v == 0.0) continue;
            const int r = (int)(((float)t + 0.5f) * rex), rz = (int)(((float)r + 0.5f) * rey);
            const int ii = lo[0] + (t - r * ex), jj = lo[1] + (r - rz * ey), kk = lo[2] + rz;
            int64_t u;
            if (tub) {
                const int k = ((ii >> 3) - bx0) + nbx * (((jj >> 3) - by0) + nby * ((kk >> 3) - bz0));
                const int64_t b = tub[k];
                const int2 s = tus[k];
                u = b < 0 ? -1 : b + (ii & 7) + (int64_t)s.x * (jj & 7) + (int64_t)s.y * (kk & 7);
            } else {
                u = user_index(D, ubase, ustr, ii, jj, kk);
            }
            if (u >= 0) atomicAdd(rho + u, v);
        }
    }
};

// Corner by corner, for a wavefront whose particles lie too far apart for a
// tile: per stencil row (y, z) both x cells of every particle, exchanged
// through LDS so that neighbouring lanes take the two cells of one row -- the
// memory side, which serves atomics by 64-byte segments and bounds this path,
// then sees one request for both.  tab: 64 x 32 bytes of the wavefront's LDS.
struct DepPair {
    int64_t u;
    double v;
};
__device__ __forceinline__ void dep_corners(const DepLevel &D, const int64_t *ubase, const int2 *ustr, DepPair *tab,
                                            bool ok, const int *i0, const int *i1, const double *f, double qv,
                                            double *rho)
{
    const int lane = threadIdx.x & 63;
#pragma unroll 1
    for (int yz = 0; yz < 4; ++yz) {
        const int j = (yz & 1) ? i1[1] : i0[1], k = (yz & 2) ? i1[2] : i0[2];
        const double wy = (yz & 1) ? f[1] : 1.0 - f[1], wz = (yz & 2) ? f[2] : 1.0 - f[2];
        DepPair a, b;
        a.u = b.u = -1;
        if (ok) {
            const int row = D.nbk[0] * ((j >> 3) + D.nbk[1] * (k >> 3));
            const int g0 = D.bmap[(i0[0] >> 3) + row], g1 = D.bmap[(i1[0] >> 3) + row];
            if (g0 >= 0) {
                const int2 s = ustr[g0];
                a.u = ubase[g0] + (i0[0] & 7) + (int64_t)s.x * (j & 7) + (int64_t)s.y * (k & 7);
            }
            if (g1 >= 0) {
                const int2 s = ustr[g1];
                b.u = ubase[g1] + (i1[0] & 7) + (int64_t)s.x * (j & 7) + (int64_t)s.y * (k & 7);
            }
        }
        a.v = qv * ((1.0 - f[0]) * wy * wz);
        b.v = qv * (f[0] * wy * wz);
        tab[2 * lane] = a;
        tab[2 * lane + 1] = b;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        a = tab[lane];
        b = tab[64 + lane];
        __builtin_amdgcn_wave_barrier();
        if (a.u >= 0) atomicAdd(rho + a.u, a.v);
        if (b.u >= 0) atomicAdd(rho + b.u, b.v);
    }
}

// REC: the particles come as records (x, y, z, q) in their own order and are
// read through perm, one 32-byte read each; else as arrays, through perm when
// it is given.  Read through the order from four arrays, a particle cost four
// scattered 8-byte reads, which the memory side serves at the same rate as
// 32-byte ones: first deposit of a build of 9e6 particles 604 -> 238 us (and
// 68 us more for the keys, which write the records).
template <class P, bool REC, int NT, int TILE>
__global__ void __launch_bounds__(NT) k_deposit(int64_t n, const P *x, const P *y, const P *z, const double *q,
                                                const double4 *rec, const uint32_t *perm, DepArgs A,
                                                const int64_t *ubase, const int2 *ustr, unsigned long long *nout,
                                                P *xs, P *ys, P *zs, double *qs)
{
    constexpr int NW = NT / 64, WTILE = TILE / NW;
    __shared__ double acc[TILE];
    __shared__ int box[2][6];  // this level's and the next's
    __shared__ int64_t tub[NW * DEP_WBRICKS];
    __shared__ int2 tus[NW * DEP_WBRICKS];
    static_assert(NW * DEP_WBRICKS >= DEP_BRICKS && WTILE * sizeof(double) >= 128 * sizeof(DepPair), "LDS tables");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    const bool valid = i < n;
    double X = 0.0, Y = 0.0, Z = 0.0, Q = 0.0;
    if (valid) {
        const int64_t p = perm ? (int64_t)perm[i] : i;
        if (REC) {
            const double4 r = rec[p];
            X = r.x, Y = r.y, Z = r.z, Q = r.w;
        } else {
            X = (double)x[p], Y = (double)y[p], Z = (double)z[p], Q = q[p];
        }
        if (xs) {  // the visiting-order copy (exact: P -> double -> P)
            xs[i] = (P)X;
            ys[i] = (P)Y;
            zs[i] = (P)Z;
            qs[i] = Q;
        }
    }
    if (threadIdx.x < 6) box[0][threadIdx.x] = INT_MAX;
    __syncthreads();
    for (int l = 0; l < A.nlev; ++l) {
        const DepLevel &D = A.lev[l];
        int i0[3], i1[3];
        double f[3];
        const bool ok = valid && cic_stencil<P>(D, X, Y, Z, i0, i1, f);
        if (l == 0 && nout) {
            const uint64_t out = __ballot(valid && !ok);
            if (out && lane == 0) atomicAdd(nout, (unsigned long long)__popcll(out));
        }
        const double qv = ok ? Q * D.ivol : 0.0;
        int wv[6];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            wv[d] = wave_min(ok ? i0[d] : INT_MAX);
            wv[3 + d] = wave_min(ok ? ~i1[d] : INT_MAX);
        }
        if (lane < 6) {
            const int v = lane == 0 ? wv[0] : lane == 1 ? wv[1] : lane == 2 ? wv[2] : lane == 3 ? wv[3]
                                                                                : lane == 4 ? wv[4] : wv[5];
            atomicMin(&box[l & 1][lane], v);
        }
        __syncthreads();
        int bv[6];
#pragma unroll
        for (int a = 0; a < 6; ++a) bv[a] = __builtin_amdgcn_readfirstlane(box[l & 1][a]);
        if (threadIdx.x < 6) box[(l + 1) & 1][threadIdx.x] = INT_MAX;  // used after the next barrier
        DepBox B;
        B.set(bv);
        if (B.vol <= TILE && !B.empty()) {
            int64_t ub = -1;
            int2 us = make_int2(0, 0);
            const bool tab = B.nbt <= DEP_BRICKS;
            if (tab && (int)threadIdx.x < B.nbt) B.brick(D, ubase, ustr, threadIdx.x, ub, us);
            for (int t = threadIdx.x; t < (int)B.vol; t += NT) acc[t] = 0.0;
            __syncthreads();
            if (ok) B.add(acc, i0, i1, f, qv);
            if (tab && (int)threadIdx.x < B.nbt) {
                tub[threadIdx.x] = ub;
                tus[threadIdx.x] = us;
            }
            __syncthreads();
            B.flush(acc, threadIdx.x, NT, tab ? tub : nullptr, tus, D, ubase, ustr, A.rho[l]);
        } else if (wv[0] != INT_MAX) {
            B.set(wv);
            double *wacc = acc + wave * WTILE;
            if (B.vol <= WTILE && B.nbt <= DEP_WBRICKS) {
                // the wavefront's own part of the tile and table: no barrier,
                // the LDS accesses of one wavefront keep their order
                int64_t *wub = tub + wave * DEP_WBRICKS, ub = -1;
                int2 *wus = tus + wave * DEP_WBRICKS, us = make_int2(0, 0);
                if (lane < B.nbt) B.brick(D, ubase, ustr, lane, ub, us);
                for (int t = lane; t < (int)B.vol; t += 64) wacc[t] = 0.0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (ok) B.add(wacc, i0, i1, f, qv);
                if (lane < B.nbt) {
                    wub[lane] = ub;
                    wus[lane] = us;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                B.flush(wacc, lane, 64, wub, wus, D, ubase, ustr, A.rho[l]);
            } else {
                dep_corners(D, ubase, ustr, (DepPair *)wacc, ok, i0, i1, f, qv, A.rho[l]);
            }
        }
        __syncthreads();
    }
}

// the particles as records, in their own order
template <class P>
__global__ void __launch_bounds__(256) k_pack_records(int64_t n, const P *x, const P *y, const P *z, const double *q,
                                                      double4 *rec)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) rec[i] = make_double4((double)x[i], (double)y[i], (double)z[i], q ? q[i] : 0.0);
}

// Corners of a CIC stencil: bit d of c selects the upper cell along axis d;
// st[d]: the stencil crosses a brick face along d.  A corner is "fresh"
// when every upper axis of it crosses, so that its brick differs from the
// bricks of the corners below it; spread_corners copies the value of each
// fresh corner to the corners in the same brick (the bits of axes without a
// crossing cleared), with fixed indices only.
__device__ __forceinline__ bool corner_fresh(int c, const bool *st)
{
    return (!(c & 1) || st[0]) && (!(c & 2) || st[1]) && (!(c & 4) || st[2]);
}

template <class V>
__device__ __forceinline__ void spread_corners(const bool *st, V *v)
{
    v[1] = st[0] ? v[1] : v[0];
    v[2] = st[1] ? v[2] : v[0];
    v[3] = st[1] ? (st[0] ? v[3] : v[2]) : v[1];
    v[4] = st[2] ? v[4] : v[0];
    v[5] = st[2] ? (st[0] ? v[5] : v[4]) : v[1];
    v[6] = st[2] ? (st[1] ? v[6] : v[4]) : v[2];
    v[7] = st[2] ? (st[1] ? (st[0] ? v[7] : v[6]) : v[5]) : v[3];
}

// E of one stencil from the caller's arrays E of a level, added to e when all
// its 8 cells are on the level (else false).  Boxes are unions of whole
// bricks, so the cells lie in at most two bricks per axis, each of which is
// looked up once (mostly one in all).  The two x cells of a stencil row are
// read together, also across a brick face (a box stores its rows whole);
// where they are apart, at the face of a box, a lane reads the upper cell by
// itself.  FEW: the rows one after another and every corner's brick looked
// up, in fewer registers.
template <bool FEW>
__device__ __forceinline__ bool gather_cells(const DepLevel &D, const double *const *E, const int64_t *ubase,
                                             const int2 *ustr, const int *i0, const int *i1, const double *f,
                                             double (&e)[3])
{
    // st[d]: the stencil crosses a brick face along d
    const int bstride[3] = {1, D.nbk[0], D.nbk[0] * D.nbk[1]};
    bool st[3];
    int base = 0, off[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        base += (i0[d] >> 3) * bstride[d];
        st[d] = (i1[d] >> 3) != (i0[d] >> 3);
        off[d] = st[d] ? bstride[d] : 0;
    }
    int g[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        g[c] = -1;
        if (FEW || corner_fresh(c, st))
            g[c] = D.bmap[base + ((c & 1) ? off[0] : 0) + ((c & 2) ? off[1] : 0) + ((c & 4) ? off[2] : 0)];
    }
    if (!FEW) spread_corners(st, g);
    bool ok = true;
#pragma unroll
    for (int c = 0; c < 8; ++c) ok = ok && g[c] >= 0;
    if (!ok) return false;
    // rows R at a time: their bases, then the pairs, then the upper cells
    // that lie apart, each step's loads in flight together
    constexpr int R = FEW ? 1 : 4;
#pragma unroll 1
    for (int r0 = 0; r0 < 4; r0 += R) {
        int64_t u0[R], u1[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = r0 + q, j = (r & 1) ? i1[1] : i0[1], k = (r & 2) ? i1[2] : i0[2];
            const int h = r == 0 ? g[0] : r == 1 ? g[2] : r == 2 ? g[4] : g[6];
            const int2 s = ustr[h];
            u0[q] = ubase[h] + (i0[0] & 7) + (int64_t)s.x * (j & 7) + (int64_t)s.y * (k & 7);
            u1[q] = u0[q] + (i1[0] - i0[0]);
        }
        if (st[0])
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int r = r0 + q, j = (r & 1) ? i1[1] : i0[1], k = (r & 2) ? i1[2] : i0[2];
                const int h = r == 0 ? g[1] : r == 1 ? g[3] : r == 2 ? g[5] : g[7];
                const int2 s = ustr[h];
                u1[q] = ubase[h] + (i1[0] & 7) + (int64_t)s.x * (j & 7) + (int64_t)s.y * (k & 7);
            }
        // the pair from the lower cell, or, where the upper is elsewhere, the
        // pair that ends with the lower one (it may be the level's last)
        double lo[R][3], hi[R][3];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int back = u1[q] != u0[q] + 1 && u0[q] > 0 ? 1 : 0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const dpair t = *(const dpair_a8 *)(E[d] + (u0[q] - back));
                lo[q][d] = back ? t.y : t.x;
                hi[q][d] = t.y;
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (u1[q] != u0[q] + 1)
#pragma unroll
                for (int d = 0; d < 3; ++d) hi[q][d] = E[d][u1[q]];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = r0 + q;
            const double wy = (r & 1) ? f[1] : 1.0 - f[1], wz = (r & 2) ? f[2] : 1.0 - f[2];
            const double w0 = (1.0 - f[0]) * wy * wz, w1 = f[0] * wy * wz;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                e[d] += w0 * lo[q][d];
                e[d] += w1 * hi[q][d];
            }
        }
    }
    return true;
}

// cells and bricks of a gather's field tile (one per wavefront)
constexpr int GA_TILE = 256, GA_BRICKS = 32;

// E at every particle from the finest level whose boxes hold all 8 cells of
// its CIC stencil; particles are visited in the given (spatially sorted)
// order so that neighbouring threads read neighbouring field cells.  SRC: the
// positions come as arrays (0, read through perm when it is given), as arrays
// already in the order (1, x[i] is particle perm[i]) or as records in their
// own order (2, read through perm).  E goes to its place directly or, with
// out, to out[i] in the visiting order for k_unpermute.  Same sums in the
// same order whichever way the cells are read.
//
// Read cell by cell it is bound by the vector cache, which returns a
// wavefront's scattered 16-byte loads one or a few lanes at a time (its
// data path 94 % busy on 9e6 particles of 128^3 + 2 levels, 380 us).  TILE:
// where particles are dense, a wavefront loads the box of its stencils into
// LDS once, whole rows at a time, and its lanes read their cells there (250
// us; 4e6 moved particles on 96^3 + 2 levels 280 -> 165 us with the records).
// A box larger than the tile is read cell by cell, in few registers, so that
// the others keep five wavefronts a SIMD.
template <class P, int SRC, bool TILE>
__global__ void __launch_bounds__(256) k_gather(int64_t n, const P *x, const P *y, const P *z, const double4 *rec,
                                                const uint32_t *perm, GatherArgs G, const int64_t *ubase,
                                                const int2 *ustr, double *Ex, double *Ey, double *Ez, double4 *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool valid = i < n;
    int64_t p = i;
    double X = 0.0, Y = 0.0, Z = 0.0;
    if (valid) {
        if (perm) p = (int64_t)perm[i];
        if (SRC == 2) {
            const double4 r = rec[p];
            X = r.x, Y = r.y, Z = r.z;
        } else {
            const int64_t s = SRC == 1 ? i : p;
            X = (double)x[s], Y = (double)y[s], Z = (double)z[s];
        }
    }
    double e[3] = {0.0, 0.0, 0.0};
    bool pend = valid;
    if (!TILE) {
        for (int l = G.nlev - 1; l >= 0 && pend; --l) {
            int i0[3], i1[3];
            double f[3];
            // (outside the domain: on every level)
            pend = cic_stencil<P>(G.lev[l], X, Y, Z, i0, i1, f) &&
                   !gather_cells<false>(G.lev[l], G.E + 3 * l, ubase, ustr, i0, i1, f, e);
        }
    } else {
        __shared__ double field[4][3 * GA_TILE];
        __shared__ int64_t tub[4][GA_BRICKS];
        __shared__ int2 tus[4][GA_BRICKS];
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double *wf = field[wave];
        int64_t *wub = tub[wave];
        int2 *wus = tus[wave];
        for (int l = G.nlev - 1; l >= 0; --l) {
            const DepLevel &D = G.lev[l];
            int i0[3], i1[3];
            double f[3];
            pend = pend && cic_stencil<P>(D, X, Y, Z, i0, i1, f);
            int wv[6];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                wv[d] = wave_min(pend ? i0[d] : INT_MAX);
                wv[3 + d] = wave_min(pend ? ~i1[d] : INT_MAX);
            }
            DepBox B;
            B.set(wv);
            if (B.empty()) break;  // every particle of the wavefront done
            if (B.vol > GA_TILE || B.nbt > GA_BRICKS) {
                if (pend) pend = !gather_cells<true>(D, G.E + 3 * l, ubase, ustr, i0, i1, f, e);
                continue;
            }
            int64_t ub = -1;
            int2 us = make_int2(0, 0);
            if (lane < B.nbt) {
                B.brick(D, ubase, ustr, lane, ub, us);
                wub[lane] = ub;
                wus[lane] = us;
            }
            const uint64_t there = __ballot(ub >= 0);
            wave_fence();
            bool ok = pend && there;
            if (there != ((uint64_t)1 << B.nbt) - 1) {  // some brick of the box is not on the level
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int bx = ((c & 1) ? i1[0] : i0[0]) >> 3, by = ((c & 2) ? i1[1] : i0[1]) >> 3,
                              bz = ((c & 4) ? i1[2] : i0[2]) >> 3;
                    if (ok) ok = (there >> ((bx - B.bx0) + B.nbx * ((by - B.by0) + B.nby * (bz - B.bz0)))) & 1;
                }
            }
            if (!__ballot(ok)) continue;
            // the box of the field into LDS, all loads in flight; quotients by
            // its extents as in the deposit's flush
            const float rex = 1.0f / (float)B.ex, rey = 1.0f / (float)B.ey;
            double v[GA_TILE / 64][3];
#pragma unroll
            for (int j = 0; j < GA_TILE / 64; ++j) {
                const int t = lane + 64 * j;
                v[j][0] = v[j][1] = v[j][2] = 0.0;
                if (t < (int)B.vol) {
                    const int r = (int)(((float)t + 0.5f) * rex), rz = (int)(((float)r + 0.5f) * rey);
                    const int ii = B.lo[0] + (t - r * B.ex), jj = B.lo[1] + (r - rz * B.ey), kk = B.lo[2] + rz;
                    const int k = ((ii >> 3) - B.bx0) + B.nbx * (((jj >> 3) - B.by0) + B.nby * ((kk >> 3) - B.bz0));
                    const int64_t u0 = wub[k];
                    const int2 st = wus[k];
                    if (u0 >= 0) {
                        const int64_t u = u0 + (ii & 7) + (int64_t)st.x * (jj & 7) + (int64_t)st.y * (kk & 7);
#pragma unroll
                        for (int d = 0; d < 3; ++d) v[j][d] = G.E[3 * l + d][u];
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < GA_TILE / 64; ++j)
#pragma unroll
                for (int d = 0; d < 3; ++d) wf[d * GA_TILE + lane + 64 * j] = v[j][d];
            wave_fence();
            if (ok) {
                const int dx = i1[0] - i0[0], dy = B.ex * (i1[1] - i0[1]), dz = B.ex * B.ey * (i1[2] - i0[2]);
                const double *c0 = wf + (i0[0] - B.lo[0]) + B.ex * ((i0[1] - B.lo[1]) + B.ey * (i0[2] - B.lo[2]));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double *c = c0 + ((r & 1) ? dy : 0) + ((r & 2) ? dz : 0);
                    const double wy = (r & 1) ? f[1] : 1.0 - f[1], wz = (r & 2) ? f[2] : 1.0 - f[2];
                    const double w0 = (1.0 - f[0]) * wy * wz, w1 = f[0] * wy * wz;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        e[d] += w0 * c[d * GA_TILE];
                        e[d] += w1 * c[d * GA_TILE + dx];
                    }
                }
                pend = false;
            }
            wave_fence();
        }
    }
    if (!valid) return;
    if (out) {
        out[i] = make_double4(e[0], e[1], e[2], 0.0);
        return;
    }
    Ex[p] = e[0];
    Ey[p] = e[1];
    Ez[p] = e[2];
}

// E of particle p from its record in the visiting order (iperm[p] = its
// place there): one 32-byte read at a scattered place, three coalesced writes
__global__ void __launch_bounds__(256) k_unpermute(int64_t n, const uint32_t *iperm, const double4 *rec, double *Ex,
                                                   double *Ey, double *Ez)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const double4 r = rec[iperm[p]];
    Ex[p] = r.x;
    Ey[p] = r.y;
    Ez[p] = r.z;
}

// max |rho| over a level (per-workgroup partials, then one workgroup)
__global__ void __launch_bounds__(256) k_absmax_part(const double *v, int64_t n, double *part)
{
    double m = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        m = fmax(m, fabs(v[i]));
    m = block_reduce(m, 1);
    if (threadIdx.x == 0) part[blockIdx.x] = m;
}

template <class T>
__global__ void __launch_bounds__(256) k_copy(const T *a, T *b, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) b[i] = a[i];
}

// Tag cells of one level (|rho| > lambda * max|rho|) and mark the blocks of
// the finer level (bf fine cells = half coarse cells per edge) that a tag
// dilated by nbuf cells reaches.  Same value written by every marker.
// max|rho| comes from the partial maxima of k_absmax_part (at most 1024), by
// each workgroup for itself: a launch between the two for one number cost
// more than the reads (2.0 us and a launch, twice a build of three levels).
__global__ void __launch_bounds__(256) k_mark_blocks(const double *rho, const int4 *borg, const int64_t *ubase,
                                                     const int2 *ustr, int nb, const double *part, int parts,
                                                     double lambda, int nbuf, int half, int3 n, int3 g, uint8_t *marks)
{
    int b = xcd_remap(blockIdx.x, nb);
    double vmax = 0.0;
    for (int i = threadIdx.x; i < parts; i += 256) vmax = fmax(vmax, part[i]);
    vmax = block_reduce(vmax, 1);
    int4 o = borg[b];
    int64_t ub = ubase[b];
    int2 us = ustr[b];
    double thr = lambda * vmax;
    for (int c = threadIdx.x; c < BRICK_CELLS; c += 256) {
        int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
        double v = rho[ub + x + (int64_t)us.x * y + (int64_t)us.y * z];
        if (!(fabs(v) > thr)) continue;
        int gi = o.x + x, gj = o.y + y, gk = o.z + z;
        int x0 = max(0, gi - nbuf) / half, x1 = min(n.x - 1, gi + nbuf) / half;
        int y0 = max(0, gj - nbuf) / half, y1 = min(n.y - 1, gj + nbuf) / half;
        int z0 = max(0, gk - nbuf) / half, z1 = min(n.z - 1, gk + nbuf) / half;
        for (int bz = z0; bz <= z1; ++bz)
            for (int by = y0; by <= y1; ++by)
                for (int bx = x0; bx <= x1; ++bx) marks[(size_t)bx + (size_t)g.x * ((size_t)by + (size_t)g.y * bz)] = 1;
    }
}

// Every level's dst from its src, or zero without one, and a counter cleared:
// one launch for all levels (a copy or a fill of a small one is all launch).
__global__ void __launch_bounds__(256) k_set_levels(LevelSet A, unsigned long long *count)
{
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0 && count) *count = 0;
    for (int l = 0; l < A.nlev; ++l) {
        if (i < A.ncell[l]) {
            A.dst[l][i] = A.src[l] ? A.src[l][i] : 0.0;
            return;
        }
        i -= A.ncell[l];
    }
}

// Proper nesting of the marked blocks of the finer level: a block stays
// marked when its footprint on the coarse level (half coarse cells per block
// edge), grown by np cells and clipped to the level's index space cn, lies
// in bricks of the coarse level (cbmap over its brick grid cnbk).  The marks
// are packed into bits in linear block order, word t / 64 holding block t at
// bit t % 64, for the greedy merge on the host.
__global__ void __launch_bounds__(256) k_nest_pack(const uint8_t *marks, int64_t total, int3 g, const int32_t *cbmap,
                                                   int3 cn, int3 cnbk, int half, int np, uint64_t *bits)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool keep = false;
    if (t < total && marks[t]) {
        const int blk[3] = {(int)(t % g.x), (int)((t / g.x) % g.y), (int)(t / ((int64_t)g.x * g.y))};
        const int nn[3] = {cn.x, cn.y, cn.z};
        int b0[3], b1[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int lo = max(0, blk[d] * half - np), hi = min(nn[d], (blk[d] + 1) * half + np);
            b0[d] = lo >> 3;
            b1[d] = (hi - 1) >> 3;
        }
        keep = true;
        for (int bz = b0[2]; bz <= b1[2] && keep; ++bz)
            for (int by = b0[1]; by <= b1[1] && keep; ++by)
                for (int bx = b0[0]; bx <= b1[0] && keep; ++bx)
                    keep = cbmap[bx + (int64_t)cnbk.x * (by + (int64_t)cnbk.y * bz)] >= 0;
    }
    const uint64_t m = __ballot(keep);
    if ((threadIdx.x & 63) == 0 && t < total) bits[t >> 6] = m;
}

// v [n], w [nw] and a counter cleared, in one launch
__global__ void __launch_bounds__(256) k_clear(double *v, int64_t n, uint64_t *w, int64_t nw,
                                               unsigned long long *count)
{
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) v[i] = 0.0;
    if (i < nw) w[i] = 0;
    if (i == 0 && count) *count = 0;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

template <class T>
void launch_outer_residual(hipStream_t st, const DevMeta &M, int b0, int nb, const int32_t *list, const double *phib,
                           const double *rhob, double inv_eps0, const double *cp_phi, T *r_out, double *part,
                           int n_part, int norm_p, bool both, double *const *r_user, const double *ffs)
{
    if (nb <= 0) return;
    // four bricks per workgroup on levels far larger than the chip (the
    // sweep's tuning finds the same), one otherwise
#define AMRMG_RESIDUAL(BOTH, BPW)                                                                                    \
    AMRMG_LAUNCH((k_outer_residual<T, BOTH, BPW>), dim3((nb + BPW - 1) / BPW), dim3(64 * BPW), 0, st, M, b0, nb, phib, \
                 rhob, inv_eps0, cp_phi, r_out, part, n_part, norm_p, list, r_user, ffs)
    if (nb > 16384) {
        if (both) AMRMG_RESIDUAL(true, 4);
        else AMRMG_RESIDUAL(false, 4);
    } else {
        if (both) AMRMG_RESIDUAL(true, 1);
        else AMRMG_RESIDUAL(false, 1);
    }
#undef AMRMG_RESIDUAL
}

void launch_user_brick(hipStream_t st, const DevMeta &M, int b0, int nb, const int32_t *list, bool to_brick,
                       double *const *a, double *ab, double *const *bu, double *bb)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH(k_user_brick, dim3(nb), dim3(256), 0, st, M, b0, nb, list, (int)to_brick, a, ab, bu, bb);
}

void launch_level_norms(hipStream_t st, const NormPlan &N, int sets, const double *part, int n_part, int norm_p,
                        double *hout, int alt, unsigned *hseq, unsigned *counter)
{
    if (N.n <= 0) return;
    const int np = sets * N.npiece;
    AMRMG_LAUNCH(k_level_norms, dim3(np <= NORM_ONE ? 1 : (np + 15) / 16), dim3(1024), 0, st, N.pieces, N.first,
                 N.npiece, N.n, sets, part, n_part, N.psum, N.done, norm_p, hout, alt, hseq, counter);
}

template <class T>
void launch_cpart_brick(hipStream_t st, const DevMeta &M, int cf0, int ncf, const T *src, T *cp, const T *fine,
                        double *ffs)
{
    if (ncf <= 0) return;
    SrcBrick<T> s{src};
    AMRMG_LAUNCH((k_cpart<T, SrcBrick<T>>), dim3(blocks_for((int64_t)ncf * 16, 256)), dim3(256), 0, st, M,
                       cf0, ncf, s, cp, fine, ffs);
}

template <class T>
void launch_face_sums(hipStream_t st, const DevMeta &M, int cf0, int ncf, const T *e, double *ffs)
{
    if (ncf <= 0) return;
    AMRMG_LAUNCH((k_face_sums<T>), dim3(blocks_for((int64_t)ncf * 16, 256)), dim3(256), 0, st, M, cf0, ncf, e,
                 ffs);
}

template <class T>
void launch_gsrb(hipStream_t st, const DevMeta &M, int b0, int nb, T *e, const T *r, const T *cp, int colour,
                 bool init)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH((k_gsrb<T>), dim3(nb), dim3(256), 0, st, M, b0, nb, e, r, cp, colour, (int)init);
}

template <class T>
void launch_jacobi(hipStream_t st, const DevMeta &M, int b0, int nb, const T *ein, T *eout, const T *r, const T *cp,
                   double omega, bool init)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH((k_jacobi<T>), dim3(nb), dim3(256), 0, st, M, b0, nb, ein, eout, r, cp, omega, (int)init);
}

template <class T>
void launch_restrict(hipStream_t st, const DevMeta &M, int b0, int nb, const int32_t *rlist, int nrf, const T *e,
                     T *r, const double *ffs)
{
    if (nb + nrf <= 0) return;
    AMRMG_LAUNCH((k_restrict<T>), dim3((nb + 1) / 2 + (nrf + 1) / 2), dim3(128), 0, st, M, b0, nb, rlist, nrf, e, r,
                 ffs);
}

template <class T>
void launch_prolong(hipStream_t st, const DevMeta &M, int b0, int nb, T *e)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH((k_prolong<T>), dim3(nb), dim3(256), 0, st, M, b0, nb, e);
}

template <class T>
void launch_phi_update(hipStream_t st, const DevMeta &M, int b0, int nb, const int32_t *list, double *phib,
                       const T *e)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH((k_phi_update<T>), dim3(nb), dim3(256), 0, st, M, b0, nb, phib, e, list);
}

void launch_avgdown(hipStream_t st, const DevMeta &M, int b0, int nb, double *phib)
{
    if (nb <= 0) return;
    AMRMG_LAUNCH(k_avgdown, dim3((nb + 3) / 4), dim3(256), 0, st, M, b0, nb, phib);
}

void launch_efield(hipStream_t st, const DevMeta &M, int b0, int nb, const int32_t *list, const double *phib,
                   const double *cp_phi, double *const *E, double *const *phi)
{
    if (nb <= 0) return;
    if (nb > 16384)  // as the outer residual
        AMRMG_LAUNCH((k_efield<4>), dim3((nb + 3) / 4), dim3(256), 0, st, M, b0, nb, phib, cp_phi, E, phi, list);
    else
        AMRMG_LAUNCH((k_efield<1>), dim3(nb), dim3(64), 0, st, M, b0, nb, phib, cp_phi, E, phi, list);
}

template <class P, bool REC, int NT, int TILE>
static void launch_deposit_t(hipStream_t st, int64_t n, const void *x, const void *y, const void *z, const double *q,
                             const double4 *rec, const uint32_t *perm, const DepArgs &A, const int64_t *ubase,
                             const int2 *ustr, unsigned long long *nout, void *xs, void *ys, void *zs, double *qs)
{
    AMRMG_LAUNCH((k_deposit<P, REC, NT, TILE>), dim3(blocks_for(n, NT)), dim3(NT), 0, st, n, (const P *)x,
                 (const P *)y, (const P *)z, q, rec, perm, A, ubase, ustr, nout, (P *)xs, (P *)ys, (P *)zs, qs);
}

void launch_deposit(hipStream_t st, int pos_f32, int64_t n, const void *x, const void *y, const void *z,
                    const double *q, const double4 *rec, const uint32_t *perm, const DepArgs &A, const int64_t *ubase,
                    const int2 *ustr, unsigned long long *nout, void *xs, void *ys, void *zs, double *qs, bool wide)
{
    if (n <= 0 || A.nlev <= 0) return;
    if (!perm) rec = nullptr;
#define AMRMG_DEPOSIT(P, R)                                                                                       \
    do {                                                                                                          \
        if (wide)                                                                                                 \
            launch_deposit_t<P, R, 512, 6144>(st, n, x, y, z, q, rec, perm, A, ubase, ustr, nout, xs, ys, zs, qs); \
        else                                                                                                      \
            launch_deposit_t<P, R, 256, 3072>(st, n, x, y, z, q, rec, perm, A, ubase, ustr, nout, xs, ys, zs, qs); \
    } while (0)
    if (pos_f32) {
        if (rec) AMRMG_DEPOSIT(float, true);
        else AMRMG_DEPOSIT(float, false);
    } else {
        if (rec) AMRMG_DEPOSIT(double, true);
        else AMRMG_DEPOSIT(double, false);
    }
#undef AMRMG_DEPOSIT
}

void launch_pack_records(hipStream_t st, int pos_f32, int64_t n, const void *x, const void *y, const void *z,
                         const double *q, double4 *rec)
{
    if (n <= 0) return;
    const dim3 g(blocks_for(n, 256));
    if (pos_f32)
        AMRMG_LAUNCH((k_pack_records<float>), g, dim3(256), 0, st, n, (const float *)x, (const float *)y,
                     (const float *)z, q, rec);
    else
        AMRMG_LAUNCH((k_pack_records<double>), g, dim3(256), 0, st, n, (const double *)x, (const double *)y,
                     (const double *)z, q, rec);
}

template <class P, int SRC>
static void launch_gather_t(hipStream_t st, int64_t n, const void *x, const void *y, const void *z,
                            const double4 *rec, const uint32_t *perm, const GatherArgs &G, const int64_t *ubase,
                            const int2 *ustr, double *Ex, double *Ey, double *Ez, double4 *out, bool tile)
{
    const dim3 g(blocks_for(n, 256)), blk(256);
    if (tile)
        AMRMG_LAUNCH((k_gather<P, SRC, true>), g, blk, 0, st, n, (const P *)x, (const P *)y, (const P *)z, rec, perm,
                     G, ubase, ustr, Ex, Ey, Ez, out);
    else
        AMRMG_LAUNCH((k_gather<P, SRC, false>), g, blk, 0, st, n, (const P *)x, (const P *)y, (const P *)z, rec, perm,
                     G, ubase, ustr, Ex, Ey, Ez, out);
}

void launch_gather(hipStream_t st, int pos_f32, int64_t n, const void *x, const void *y, const void *z,
                   const double4 *rec, const uint32_t *perm, const uint32_t *iperm, const GatherArgs &G,
                   const int64_t *ubase, const int2 *ustr, double *Ex, double *Ey, double *Ez, double4 *out,
                   bool ordered, bool tile)
{
    if (n <= 0) return;
    if (!perm || !iperm) out = nullptr;
    if (!perm) tile = false;
    if (ordered && perm) {
        if (pos_f32)
            launch_gather_t<float, 1>(st, n, x, y, z, nullptr, perm, G, ubase, ustr, Ex, Ey, Ez, out, tile);
        else
            launch_gather_t<double, 1>(st, n, x, y, z, nullptr, perm, G, ubase, ustr, Ex, Ey, Ez, out, tile);
    } else if (rec && perm) {
        launch_gather_t<double, 2>(st, n, nullptr, nullptr, nullptr, rec, perm, G, ubase, ustr, Ex, Ey, Ez, out, tile);
    } else if (pos_f32) {
        launch_gather_t<float, 0>(st, n, x, y, z, nullptr, perm, G, ubase, ustr, Ex, Ey, Ez, out, tile);
    } else {
        launch_gather_t<double, 0>(st, n, x, y, z, nullptr, perm, G, ubase, ustr, Ex, Ey, Ez, out, tile);
    }
    if (out) AMRMG_LAUNCH(k_unpermute, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, iperm, out, Ex, Ey, Ez);
}

// the size rule: one wavefront (brick) per workgroup
int hgs_rule_threads(int) { return 64; }

template <class T>
void launch_hgs(hipStream_t st, const DevMeta &M, int b0, int nb, const T *ein, T *eout, const T *r, T *cp,
                double *phib, double *ffs, int mode, int nt)
{
    if (nb <= 0) return;
    const int bpw = (nt ? nt : hgs_rule_threads(nb)) / 64;
    const dim3 blk(64 * bpw), grid((nb + bpw - 1) / bpw);
#define AMRMG_HGS_BPW(MD, B)                                                                                     \
    if (bpw == B) {                                                                                              \
        AMRMG_LAUNCH((k_hgs<T, MD, B>), grid, blk, 0, st, M, b0, nb, ein, eout, r, cp, phib, ffs);               \
        return;                                                                                                  \
    }
#define AMRMG_HGS(MD)        \
    case MD:                 \
        AMRMG_HGS_BPW(MD, 1) \
        AMRMG_HGS_BPW(MD, 2) \
        AMRMG_HGS_BPW(MD, 4) \
        break;
    switch (mode) {
        AMRMG_HGS(0)
        AMRMG_HGS(HG_FFS)
        AMRMG_HGS(HG_ZERO | HG_FFS)
        AMRMG_HGS(HG_PHI)
        AMRMG_HGS(HG_PROL | HG_CPIN)
        AMRMG_HGS(HG_PROL | HG_CPIN | HG_PHI)
    default: break;
    }
#undef AMRMG_HGS
#undef AMRMG_HGS_BPW
    fprintf(stderr, "libamrmg: no sweep kernel for mode %d and %d threads per workgroup\n", mode, 64 * bpw);
    abort();
}

template <class T>
void launch_hgs_first2(hipStream_t st, const DevMeta &M, int b0, int nb, T *eout, const T *r, double *ffs,
                       bool face_sums, int nt)
{
    if (nb <= 0) return;
    const int bpw = (nt ? nt : hgs_rule_threads(nb)) / 64;
    const dim3 blk(64 * bpw), grid((nb + bpw - 1) / bpw);
#define AMRMG_FIRST2(F, B) AMRMG_LAUNCH((k_hgs_first2<T, F, B>), grid, blk, 0, st, M, b0, nb, eout, r, ffs)
    if (face_sums) {
        if (bpw == 1) AMRMG_FIRST2(true, 1);
        else if (bpw == 2) AMRMG_FIRST2(true, 2);
        else AMRMG_FIRST2(true, 4);
    } else {
        if (bpw == 1) AMRMG_FIRST2(false, 1);
        else if (bpw == 2) AMRMG_FIRST2(false, 2);
        else AMRMG_FIRST2(false, 4);
    }
#undef AMRMG_FIRST2
}

template <class T>
void launch_coarse_cycle(hipStream_t st, const DevMeta &M, const CoarseJob *jobs, int njobs, T *e, T *r,
                         double *work, int nu1, int nu2, double rtol, int maxit, int *iters, double *phib,
                         bool phi_update, int threads_hint)
{
    if (njobs <= 0) return;
    int threads = threads_hint > 0 ? threads_hint : 1024;
    AMRMG_LAUNCH((k_coarse_cycle<T>), dim3(njobs), dim3(threads), 0, st, M, jobs, e, r, work, nu1, nu2, rtol, maxit,
                 iters, phib, (int)phi_update);
}

template <class T>
void launch_direct(hipStream_t st, const DirectJob *jobs, const int2 *planes, int nplanes, const int2 *groups,
                   int ngroups, const double *tab, double *W, const T *r, T *e, double *phib, bool phi_update,
                   int maxdim, const DirectJob *one)
{
    if (nplanes <= 0) return;
    // one job: its record goes by value and the workgroups' lists are not read
    const DirectJob J1 = one ? *one : DirectJob{};
    const DirectJob *jl = one ? nullptr : jobs;
    const int pu = (int)phi_update;
#define AMRMG_DIRECT(NC)                                                                                           \
    do {                                                                                                           \
        AMRMG_LAUNCH((k_dst_plane<T, false, NC>), dim3(nplanes), dim3(256), 0, st, jl, planes, J1, tab, W, r, e, phib, \
                     pu);                                                                                          \
        AMRMG_LAUNCH((k_dst_column<NC>), dim3(ngroups), dim3(dst_threads(NC)), 0, st, jl, groups, J1, tab, W);                 \
        AMRMG_LAUNCH((k_dst_plane<T, true, NC>), dim3(nplanes), dim3(256), 0, st, jl, planes, J1, tab, W, r, e, phib,  \
                     pu);                                                                                          \
    } while (0)
    // registers for the operands of the longest edge
    if (maxdim <= 32) AMRMG_DIRECT(2);
    else if (maxdim <= 64) AMRMG_DIRECT(4);
    else AMRMG_DIRECT(DIRECT_DIM / 16);
#undef AMRMG_DIRECT
}

template <class T>
void launch_copy(hipStream_t st, const T *a, T *b, int64_t n)
{
    if (n <= 0) return;
    AMRMG_LAUNCH((k_copy<T>), dim3(blocks_for(n, 256)), dim3(256), 0, st, a, b, n);
}

void launch_nest_pack(hipStream_t st, const uint8_t *marks, int64_t total, int3 g, const int32_t *cbmap, int3 cn,
                      int3 cnbk, int half, int np, uint64_t *bits)
{
    if (total <= 0) return;
    AMRMG_LAUNCH(k_nest_pack, dim3(blocks_for(total, 256)), dim3(256), 0, st, marks, total, g, cbmap, cn, cnbk, half, np,
                 bits);
}

void launch_mark_blocks(hipStream_t st, const double *rho, int64_t ncell, const int4 *borg, const int64_t *ubase,
                        const int2 *ustr, int nb, double lambda, int nbuf, int half, int3 n, int3 g, double *scratch,
                        uint8_t *marks)
{
    if (nb <= 0) return;
    int parts = (int)blocks_for(ncell, 256);
    if (parts > 1024) parts = 1024;
    AMRMG_LAUNCH(k_absmax_part, dim3(parts), dim3(256), 0, st, rho, ncell, scratch);
    AMRMG_LAUNCH(k_mark_blocks, dim3(nb), dim3(256), 0, st, rho, borg, ubase, ustr, nb, scratch, parts, lambda, nbuf,
                 half, n, g, marks);
}

void launch_set_levels(hipStream_t st, const LevelSet &A, unsigned long long *count)
{
    int64_t total = 0;
    for (int l = 0; l < A.nlev; ++l) total += A.ncell[l];
    if (total <= 0) total = 1;  // the counter
    hipLaunchKernelGGL(k_set_levels, dim3(blocks_for(total, 256)), dim3(256), 0, st, A, count);
}

void launch_clear(hipStream_t st, double *v, int64_t n, uint64_t *w, int64_t nw, unsigned long long *count)
{
    int64_t total = n > nw ? n : nw;
    if (total <= 0) total = 1;  // the counter
    hipLaunchKernelGGL(k_clear, dim3(blocks_for(total, 256)), dim3(256), 0, st, v, n, w, nw, count);
}

#define AMRMG_INST(T)                                                                                            \
    template void launch_outer_residual<T>(hipStream_t, const DevMeta &, int, int, const int32_t *,               \
                                           const double *, const double *, double, const double *, T *, double *, \
                                           int, int, bool, double *const *, const double *);                      \
    template void launch_cpart_brick<T>(hipStream_t, const DevMeta &, int, int, const T *, T *, const T *,      \
                                        double *);                                                              \
    template void launch_face_sums<T>(hipStream_t, const DevMeta &, int, int, const T *, double *);             \
    template void launch_gsrb<T>(hipStream_t, const DevMeta &, int, int, T *, const T *, const T *, int, bool);  \
    template void launch_jacobi<T>(hipStream_t, const DevMeta &, int, int, const T *, T *, const T *, const T *, \
                                   double, bool);                                                                \
    template void launch_restrict<T>(hipStream_t, const DevMeta &, int, int, const int32_t *, int, const T *,   \
                                     T *, const double *);                                                      \
    template void launch_prolong<T>(hipStream_t, const DevMeta &, int, int, T *);                                \
    template void launch_phi_update<T>(hipStream_t, const DevMeta &, int, int, const int32_t *, double *,         \
                                       const T *);                                                               \
    template void launch_copy<T>(hipStream_t, const T *, T *, int64_t);                                         \
    template void launch_hgs<T>(hipStream_t, const DevMeta &, int, int, const T *, T *, const T *, T *,         \
                                double *, double *, int, int);                                                       \
    template void launch_hgs_first2<T>(hipStream_t, const DevMeta &, int, int, T *, const T *, double *, bool,  \
                                       int);                                                                   \
    template void launch_coarse_cycle<T>(hipStream_t, const DevMeta &, const CoarseJob *, int, T *, T *,        \
                                         double *, int, int, double, int, int *, double *, bool, int);          \
    template void launch_direct<T>(hipStream_t, const DirectJob *, const int2 *, int, const int2 *, int,         \
                                   const double *, double *, const T *, T *, double *, bool, int, const DirectJob *);
AMRMG_INST(float)
AMRMG_INST(double)
#undef AMRMG_INST

}  // namespace amrmg
