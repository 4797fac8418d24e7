// lbm_kernels.hip -- HIP kernels of the TO-LRS lattice Boltzmann LES step for
// gfx950 (MI355X).
//
// Populations are stored in blocks of kPopBlk cells (x-fastest cell order),
// each block holding its Q populations one after another, in two ping-pong
// buffers; the other fields are [component][N].  One step (eqs. LES-1..LES-3
// with the TO correction):
//   k_step     pull-stream with halfway bounce-back (eq. LES-3, Sec. 7.1),
//              moments, effective relaxation time (Sec. 5), BGK relaxation and
//              exact-difference forcing (eq. LES-1/LES-2); writes the
//              predictor populations and rho, v* = v^{p,n*}.
//   k_step_t   the same on 2.5-D tiles, adding during the pull the SGS change
//              the previous step recorded per cell (grids whose populations
//              exceed the Infinity Cache, and smaller ones by lattice and
//              precision: FP64 channels, 2-D from 24 MB).
//   k_chain    binomial closures (Sec. 4.1): from v* the sensitivities
//              R R v* of the E QoIs, U = R R w of the Z QoIs (w = curl v*) and
//              the QoI sums, every power of B on chip.
//   k_chain_pair  2-D closures of at most one E and one Z QoI: the chains,
//              the adjoint curl and the Gram products in one launch.
//   k_kxy, k_kz   kernel filters: the x and y parts of a filter, and its z part.
//   k_fpack, k_fmask, k_funpack  Fourier bands around two hipFFT transforms.
//   k_reduce   sensitivities curl^T U of the Z QoIs (App. A) and the Gram
//              products, reduced per workgroup in FP64.
//   k_sum      fixed-order cross-workgroup sums; the step's LRS draw.
//   k_solve    one workgroup per member: dQ (tracking or LRS, eqs.
//              dQ-from-ref, LRS), Gram solve (eq. O-from-V, eq.
//              orthogonality), gamma (eq. tau-from-dQ-for-tracking).
//   k_apply    dv_SGS = sum_i gamma_i O_i (eq. TO-ansatz), evaluated as
//              sum_i beta_i V_i with beta = G^-1 dQ; its change of the
//              equilibrium is added to the predictor populations in place, or
//              recorded as (rho dv, 2 v* + dv) for the next k_step_t (k_flush
//              applies pending records before the state is read).
//   k_apply_fs the same with the member's solve at its head, in every
//              workgroup (small launches: no k_solve launch).
// Every kernel takes a table of members and a work table mapping each
// workgroup to (member, local block), so one launch serves a whole ensemble.
// All reductions have a fixed order that depends only on the member's own
// geometry, so a member gives bitwise the same result alone or in a batch.
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>
#include <math.h>

#include <type_traits>

#include "lbm_dev.h"
#include "lbm_launch.h"

namespace lbm {

// ---------------------------------------------------------------------------
// Lattices (Sec. 2).  Opposite of i >= 1 is i + 1 for odd i, i - 1 for even i.
// ---------------------------------------------------------------------------
template <int LAT> struct Lat;
template <> struct Lat<LBM_D2Q9> {
    static constexpr int Q = 9, D = 2, NC = 1;
    static constexpr int cx[9] = {0, 1, -1, 0, 0, 1, -1, 1, -1};
    static constexpr int cy[9] = {0, 0, 0, 1, -1, 1, -1, -1, 1};
    static constexpr int cz[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    static constexpr double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                                    1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
};
template <> struct Lat<LBM_D3Q19> {
    static constexpr int Q = 19, D = 3, NC = 3;
    static constexpr int cx[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
    static constexpr int cy[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
    static constexpr int cz[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
    static constexpr double w[19] = {1.0 / 3, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                                     1.0 / 18, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                     1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                     1.0 / 36};
};
__host__ __device__ constexpr int opp(int i) { return i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1); }

__device__ __forceinline__ int wrapi(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }
__device__ __forceinline__ int modi(int a, int n) { int r = a % n; return r < 0 ? r + n : r; }

// ---------------------------------------------------------------------------
// Reductions over the 64-lane wavefront with DPP lane moves (no LDS
// traffic): pairs, quads, half rows and rows of 16 lanes by quad
// permutations and mirrors, then the rows by the two row broadcasts, which
// leaves the sum in lane 63.  The order of the additions is fixed.
// ---------------------------------------------------------------------------
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_add(double v)
{
    const long long b = __double_as_longlong(v);
    int lo, hi;
    if (ROWMASK == 0xf) {   // every lane is written
        lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, false);
        hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, false);
    } else {                // rows outside the mask add zero
        lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWMASK, 0xf, false);
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWMASK, 0xf, false);
    }
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double wave_sum(double v)
{
    v = dpp_add<0xB1, 0xf>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xf>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);   // row_mirror
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum NV values over the workgroup of NW wavefronts; result valid in
// thread 0.  Uses NV * NW doubles of LDS.
template <int NV, int NW = kBlock / 64>
__device__ __forceinline__ void block_sum(double* v, double* lds)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double s = wave_sum(v[k]);
        if (lane == 0) lds[k * NW + wv] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double s = 0;
#pragma unroll
            for (int j = 0; j < NW; ++j) s += lds[k * NW + j];
            v[k] = s;
        }
    }
    __syncthreads();
}

// Global accesses at an element index below 2^32 / sizeof(T) from a
// workgroup-uniform base: the byte offset is formed in 32 bits, so the access
// uses a scalar base plus one 32-bit vector offset (no 64-bit address per
// lane).  The library rejects grids whose fields would not fit.
template <typename T>
__device__ __forceinline__ T ld_at(const T* base, unsigned i)
{
    return *(const T*)((const char*)base + i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void st_at(T* base, unsigned i, T v)
{
    *(T*)((char*)base + i * (unsigned)sizeof(T)) = v;
}

// Element index of population i of cell c in the blocked population layout
// ([block][Q][kPopBlk]): a wavefront's loads of one population stay within
// one block, and the Q arrays a cell touches sit next to each other, which
// the memory system serves faster than Q separate full-length streams.  The
// 32-bit form needs Q * ceil(N / kPopBlk) * kPopBlk elements below 2^32 bytes.
template <int Q>
__device__ __forceinline__ unsigned pop_at(int i, unsigned c)
{
    return (((c >> kPopLog) * Q + (unsigned)i) << kPopLog) | (c & (kPopBlk - 1));
}
template <int Q>
__device__ __forceinline__ size_t pop_at64(int i, size_t c)
{
    return (((c >> kPopLog) * Q + (size_t)i) << kPopLog) | (c & (kPopBlk - 1));
}

// Stores of fields that the next kernel reads.  On small grids (kernels
// instantiated with WT) they are relaxed device-scope atomic stores, written
// through each XCD's L2, so that no dirty lines are left for the L2
// write-back at the end of the kernel, which the next kernel waits for.
// Measured on MI355X (FP32 channel TO-LES): 2427 -> 2592 MLUPS on
// 96 x 48 x 48; no change on 384 x 192 x 192; but 1328 -> 1130 MLUPS for
// the kernel-filter closure on 295 x 47 x 98, whose fields the next kernel
// otherwise finds in the Infinity Cache.  Larger launches store
// non-temporally (5228 -> 5310..5321 MLUPS on 384 x 192 x 192; no change on
// 295 x 47 x 98): the stream-collide itself slows (457 -> 485 us), but its
// populations then no longer push the TO fields out of the Infinity Cache
// (reduce 453 -> 424 us).  Except where a kernel stores row segments of rows
// that are not whole lines (wt = 2, k_step_t): a line's two parts then come
// from two workgroups, non-temporally each goes out by itself, a plain store
// leaves it to the L2 to join them (tiled stream-collide, FP32 230 x 130 x 130
// 344 -> 216 us; FP64 1001 x 1003, whole step 94 -> 84 us).  With 64-bit offsets
// k_step_t always stores plainly: on rows of whole lines that is level with
// non-temporal stores (step, non-temporal and plain: 384 x 192 x 192 1766 and
// 1771 us, 320 x 160 x 160 1033 and 1035, FP64 256 x 128 x 128 991 and 993,
// 2048 x 2048 199 and 195), so one form serves both.
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_fld(T* p, T v, int wt)
{
    if (wt == 1) st_dev(p, v);
    else if (wt == 2) *p = v;
    else __builtin_nontemporal_store(v, p);
}
// Loads of fields whose last reader in the step is the loading kernel: on
// launches without write-through, non-temporal (the apply's chain fields and
// populations: 5325 -> 5448 MLUPS on 384 x 192 x 192; 0.6% slower on
// 96 x 48 x 48, hence plain there).
template <bool WT, typename T>
__device__ __forceinline__ T ld_fld(const T* p)
{
    if constexpr (WT) return *p;
    else return __builtin_nontemporal_load(p);
}
template <typename T>
__device__ __forceinline__ void st_fld_at(T* base, unsigned i, T v, int wt)
{
    st_fld((T*)((char*)base + i * (unsigned)sizeof(T)), v, wt);
}

// Butterfly reduce-scatter over the wavefront: at lane distance D each lane
// keeps one half of its list of L partial sums (the lower half where lane
// bit D is clear, else the upper half, padded with a zero when L is odd)
// and adds its partner's copy of that half.  A level costs ceil(L/2)
// exchanges; after distances 32 .. 1 every lane holds one wave sum.  Returns
// that sum's index in the list (-1 for a lane left holding padding, which
// includes the upper lanes of every level with L = 1).  The order of the
// additions is fixed.
template <int L, int D>
__device__ __forceinline__ int wave_scatter(double* cur, int lane)
{
    constexpr int H = (L + 1) / 2;
    const bool hi = (lane & D) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double lo_v = cur[i];
        const double hi_v = H + i < L ? cur[H + i] : 0.0;
        const double give = hi ? lo_v : hi_v;
        cur[i] = (hi ? hi_v : lo_v) + __shfl_xor(give, D);
    }
    int p = 0;
    if constexpr (D > 1) p = wave_scatter<H, D / 2>(cur, lane);
    if (p < 0) return -1;
    p += hi ? H : 0;
    return p < L ? p : -1;
}

// The sums of block_sum with the result spread over the workgroup: thread
// k < NV returns value k, the waves' sums added in wave order.
template <int NV>
__device__ __forceinline__ double block_sum_spread(const double* v, double* lds)
{
    static_assert(NV <= 64, "one value per lane after the butterfly");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double cur[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) cur[k] = v[k];
    const int idx = wave_scatter<NV, 32>(cur, lane);
    if (idx >= 0) lds[idx * (kBlock / 64) + wv] = cur[0];
    __syncthreads();
    double r = 0;
    if (threadIdx.x < NV) {
#pragma unroll
        for (int j = 0; j < kBlock / 64; ++j) r += lds[threadIdx.x * (kBlock / 64) + j];
    }
    return r;
}

// feq_i(rho, a) - feq_i(rho, b) in difference form (exactly zero when a = b):
// w rho [3 c.(a-b) + 9/2 (c.(a-b))(c.(a+b)) - 3/2 (a-b).(a+b)].
template <typename T>
__device__ __forceinline__ T dfeq(T w, T rho, T cd, T cs, T dd)
{
    return w * rho * (T(3) * cd + T(4.5) * cd * cs - T(1.5) * dd);
}

// ---------------------------------------------------------------------------
// SGS change of the post-collision populations of a cell (eq. LES-2, the
// second difference of the exact-difference form): with a = rho dv,
// b = 2 v* + dv and e = a.b,
//   delta f_i = feq_i(rho, v* + dv) - feq_i(rho, v*)
//             = w_i [3 c_i.a + 9/2 (c_i.a)(c_i.b) - 3/2 e].
// k_apply stores the record (a, b) of every cell; the next stream-collide
// adds delta f of each source cell while it pulls (k_step_t), or k_flush adds
// it in place before the state is read.  Both evaluate it with these
// functions, without contraction and in a fixed order, so a flushed state
// streams to bitwise the populations the deferred pull forms.
// ---------------------------------------------------------------------------
// c_i . a over the nonzero components of c_i (exact signs, no products with
// the constants); A(k) returns component k.
template <int LAT, typename T, typename Get>
__device__ __forceinline__ T cdot(int i, Get A)
{
    // (no contraction: where a component is itself a product, as rho dv in
    // the in-place apply, a fused multiply-add would round differently from
    // the same sum over stored records)
#pragma clang fp contract(off)
    using L = Lat<LAT>;
    const int c[3] = {L::cx[i], L::cy[i], L::D == 3 ? L::cz[i] : 0};
    T s = T(0);
    bool any = false;
#pragma unroll
    for (int k = 0; k < L::D; ++k) {
        if (!c[k]) continue;
        const T v = A(k);
        if (!any) s = c[k] > 0 ? v : -v;
        else s = c[k] > 0 ? s + v : s - v;
        any = true;
    }
    return s;
}

// e = a.b in a fixed order.
template <int D, typename T>
__device__ __forceinline__ T rec_e(const T* a, const T* b)
{
#pragma clang fp contract(off)
    T e = a[0] * b[0];
#pragma unroll
    for (int k = 1; k < D; ++k) e = e + a[k] * b[k];
    return e;
}

// delta f_i from the record (a, b, e) of the cell, with ca = c_i.a and
// cb = c_i.b; opp: delta f of the opposite direction instead, whose c.a and
// c.b are exactly -ca and -cb (rounding is symmetric in sign), so only the
// linear term changes sign.  g + delta f is then one rounded addition.
template <int LAT, typename T>
__device__ __forceinline__ T df_cc(int i, bool opp_dir, T ca, T cb, T e)
{
#pragma clang fp contract(off)
    using L = Lat<LAT>;
    const T lin = T(3) * ca;
    const T s = ((opp_dir ? -lin : lin) + (T(4.5) * ca) * cb) - T(1.5) * e;
    return T(L::w[i]) * s;
}
template <int LAT, typename T, typename GA, typename GB>
__device__ __forceinline__ T df_of(int i, GA A, GB B, T e)
{
    return df_cc<LAT, T>(i, false, cdot<LAT, T>(i, A), cdot<LAT, T>(i, B), e);
}
template <typename T>
__device__ __forceinline__ T add_rn(T g, T d)
{
#pragma clang fp contract(off)
    return g + d;
}
template <int LAT, typename T, typename GA, typename GB>
__device__ __forceinline__ T add_df(T g, int i, GA A, GB B, T e)
{
    return add_rn(g, df_of<LAT, T>(i, A, B, e));
}

// ---------------------------------------------------------------------------
// Pull gather of the post-collision populations of cell (x,y,z).  A32: the
// run keeps 2 N * sizeof(T) below 4 GiB (every TO run does), so each load is
// a 32-bit offset from a scalar base.
// ---------------------------------------------------------------------------
template <int LAT, typename T, bool A32, bool FAST = true>
__device__ __forceinline__ void gather(KMember& m, const T* __restrict__ gs, int x, int y, int z,
                                       int cell, T* f)
{
    using L = Lat<LAT>;
    constexpr int Q = L::Q, D = L::D;
    const int nx = m.nx, ny = m.ny, nz = m.nz;
    // Wavefronts whose cells are all at least one cell from the walls and
    // from the z wrap pull from constant offsets, corrected per cell for the
    // periodic x wrap; the others resolve wrap and bounce-back per population.
    const bool inner = y > 0 && y < ny - 1 && (D == 2 || (z > 0 && z < nz - 1));
    if (FAST && __all(inner)) {
        const int wxm = x == 0 ? nx : 0, wxp = x == nx - 1 ? -nx : 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int off = L::cx[i] + nx * (L::cy[i] + (D == 3 ? ny * L::cz[i] : 0));
            const int src = cell - off + (L::cx[i] == 1 ? wxm : L::cx[i] == -1 ? wxp : 0);
            if (A32)
                f[i] = ld_at(gs, pop_at<Q>(i, (unsigned)src));
            else
                f[i] = gs[pop_at64<Q>(i, (size_t)src)];
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        int sy = y - L::cy[i];
        int src, pi;
        bool bb = m.walls && (sy < 0 || sy >= ny);
        if (bb) {
            src = cell;
            pi = opp(i);
        } else {
            int sx = wrapi(x - L::cx[i], nx);
            sy = wrapi(sy, ny);
            int sz = D == 3 ? wrapi(z - L::cz[i], nz) : 0;
            src = sx + nx * (sy + ny * sz);
            pi = i;
        }
        if (A32)
            f[i] = ld_at(gs, pop_at<Q>(pi, (unsigned)src));
        else
            f[i] = gs[pop_at64<Q>(pi, (size_t)src)];
    }
}

// Moments: rho - 1 and rho u from gathered populations.
template <int LAT, typename T, int PREC>
__device__ __forceinline__ void moments(const T* f, T& drho, T* j)
{
    using L = Lat<LAT>;
    drho = 0;
#pragma unroll
    for (int a = 0; a < L::D; ++a) j[a] = 0;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        drho += f[i];
        if (L::cx[i]) j[0] += T(L::cx[i]) * f[i];
        if (L::cy[i]) j[1] += T(L::cy[i]) * f[i];
        if (L::D == 3 && L::cz[i]) j[2] += T(L::cz[i]) * f[i];
    }
    if (PREC == LBM_FP32_PLAIN) drho -= T(1);
}

// ---------------------------------------------------------------------------
// K1: stream + collide + force.
// MODE 0: plain; 1: plain with statistics and post-streaming velocity;
// 2: TO predictor (statistics, rho, v*).
// ---------------------------------------------------------------------------
// Collision of one cell from its pulled populations f: moments, effective
// relaxation time (Sec. 5), BGK relaxation with the exact-difference force
// (eq. LES-1/LES-2); stores the predictor populations (and in TO mode rho - 1
// and v*), adds the cell's mass and momentum to st and flags instability.
// Shifted storage (FP32 and FP64): the non-equilibrium parts f_i - feq_i have
// zero mass and momentum by definition (u = j / rho), but their rounded
// values do not -- rho u differs from j after rounding, and the equilibria
// are rounded one by one -- and in a quasi-steady flow that rounding repeats
// each step, so relaxation alone would drift the mean flow (measured in FP32
// on the 20 x 24 x 12 channel: +4.5e-5 relative x-momentum after 2500 steps,
// against 3e-8 when only the stored populations are rounded).  The mass and
// momentum the rounding leaves in them are projected out (subtracting
// w_i (s + 3 c_i . sigma) removes a mass s and a momentum sigma), and each
// population is updated as f_i + (force term - omega (f_i - feq_i)), one
// rounding at its own magnitude.  Plain FP32 storage keeps the direct form
// as the baseline.
template <int LAT, typename T, int PREC, int SUB, int MODE, int WT, bool A32 = MODE == 2, bool NT = false>
__device__ __forceinline__ void collide_cell(KMember& m, T* f, int x, int y, int z, int cell, T* __restrict__ gd,
                                             double* st, int& bad)
{
    using L = Lat<LAT>;
    constexpr int Q = L::Q, D = L::D;
    constexpr bool PROJ = PREC != LBM_FP32_PLAIN;
    const int N = m.N, nx = m.nx, ny = m.ny;
    T drho, j[3] = {0, 0, 0};
    moments<LAT, T, PREC>(f, drho, j);
    const T rho = T(1) + drho;
    const T ir = T(1) / rho;
    T u[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < D; ++a) u[a] = j[a] * ir;
    T uu = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) uu += u[a] * u[a];
    if (!(uu <= T(0.25))) bad = 1;

    // non-equilibrium parts fn_i = f_i - feq_i (feq_i - w_i against shifted
    // populations)
    T fn[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T cu = T(L::cx[i]) * u[0] + T(L::cy[i]) * u[1] + (D == 3 ? T(L::cz[i]) * u[2] : T(0));
        const T X = T(3) * cu + T(4.5) * cu * cu - T(1.5) * uu;
        const T geq = PREC == LBM_FP32_PLAIN ? T(L::w[i]) * rho * (T(1) + X) : T(L::w[i]) * (drho + rho * X);
        fn[i] = f[i] - geq;
    }
    if constexpr (PROJ) {
        T sm = 0, sj[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            sm += fn[i];
            if (L::cx[i]) sj[0] += T(L::cx[i]) * fn[i];
            if (L::cy[i]) sj[1] += T(L::cy[i]) * fn[i];
            if (L::D == 3 && L::cz[i]) sj[2] += T(L::cz[i]) * fn[i];
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const T cs = T(L::cx[i]) * sj[0] + T(L::cy[i]) * sj[1] + (D == 3 ? T(L::cz[i]) * sj[2] : T(0));
            fn[i] -= T(L::w[i]) * (sm + T(3) * cs);
        }
    }

    // effective relaxation time (Sec. 5)
    T taue = T(m.tau);
    if constexpr (SUB == LBM_SMAGORINSKY) {
        T P[6] = {0, 0, 0, 0, 0, 0};  // xx yy zz xy xz yz
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const T v = fn[i];
            const int cx = L::cx[i], cy = L::cy[i], cz = L::cz[i];
            if (cx) P[0] += v;
            if (cy) P[1] += v;
            if (cz) P[2] += v;
            if (cx * cy) P[3] += T(cx * cy) * v;
            if (cx * cz) P[4] += T(cx * cz) * v;
            if (cy * cz) P[5] += T(cy * cz) * v;
        }
        const T PP = P[0] * P[0] + P[1] * P[1] + P[2] * P[2] + T(2) * (P[3] * P[3] + P[4] * P[4] + P[5] * P[5]);
        const T nP = sqrt(T(2) * PP);
        const T cm = T(m.cmodel);
        taue = T(0.5) * (taue + sqrt(taue * taue + T(18) * cm * cm * nP * ir));
    } else if constexpr (SUB == LBM_WALE) {
        // velocity gradient g_ab = D_b v_a of the post-streaming field
        const T* __restrict__ vn = (const T*)m.vn;
        T g[3][3];
        const int nz = m.nz;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            int xp = x, xm = x, yp = y, ym = y, zp = z, zm = z;
            if (b == 0) { xp = wrapi(x + 1, nx); xm = wrapi(x - 1, nx); }
            if (b == 1) { yp = y + 1; ym = y - 1; }
            if (b == 2) { zp = wrapi(z + 1, nz); zm = wrapi(z - 1, nz); }
            bool okp = true, okm = true;
            if (b == 1) {
                if (m.walls) { okp = yp < ny; okm = ym >= 0; }
                else { yp = wrapi(yp, ny); ym = wrapi(ym, ny); }
            }
            const int cp = xp + nx * (yp + ny * zp), cm = xm + nx * (ym + ny * zm);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T vp = okp ? vn[(size_t)a * N + cp] : T(0);
                T vm = okm ? vn[(size_t)a * N + cm] : T(0);
                g[a][b] = T(0.5) * (vp - vm);
            }
        }
        T g2[3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) g2[a][b] = g[a][0] * g[0][b] + g[a][1] * g[1][b] + g[a][2] * g[2][b];
        const T tr = g2[0][0] + g2[1][1] + g2[2][2];
        T SS = 0, SdSd = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                T S = T(0.5) * (g[a][b] + g[b][a]);
                T Sd = T(0.5) * (g2[a][b] + g2[b][a]) - (a == b ? tr / T(3) : T(0));
                SS += S * S;
                SdSd += Sd * Sd;
            }
        T den = pow(SS, T(2.5)) + pow(SdSd, T(1.25));
        T cm = T(m.cmodel);
        T nut = den > T(0) ? cm * cm * pow(SdSd, T(1.5)) / den : T(0);
        taue = taue + T(3) * nut;
    }
    const T om = T(1) / taue;

    // body force, F/rho velocity increment, predictor velocity
    T F[3] = {T(m.fprof[y]), 0, 0};
    if (m.drag != 0.0) {
#pragma unroll
        for (int a = 0; a < D; ++a) F[a] -= T(m.drag) * rho * u[a];
    }
    T du[3] = {0, 0, 0}, us[3] = {0, 0, 0};
    T dd = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        du[a] = F[a] * ir;
        us[a] = u[a] + du[a];
        dd += du[a] * (us[a] + u[a]);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const T cd = T(L::cx[i]) * du[0] + T(L::cy[i]) * du[1] + (D == 3 ? T(L::cz[i]) * du[2] : T(0));
        const T cs = T(L::cx[i]) * (us[0] + u[0]) + T(L::cy[i]) * (us[1] + u[1]) +
                     (D == 3 ? T(L::cz[i]) * (us[2] + u[2]) : T(0));
        const T df = dfeq<T>(T(L::w[i]), rho, cd, cs, dd);
        const T out = PROJ ? f[i] + (df - om * fn[i]) : (f[i] - om * fn[i]) + df;
        if (A32 && MODE == 2)
            st_fld_at(gd, pop_at<Q>(i, (unsigned)cell), out, WT);
        else if (A32 && NT)
            __builtin_nontemporal_store(out, (T*)((char*)gd + pop_at<Q>(i, (unsigned)cell) * (unsigned)sizeof(T)));
        else if (A32)
            st_at(gd, pop_at<Q>(i, (unsigned)cell), out);
        else if (NT)
            __builtin_nontemporal_store(out, gd + pop_at64<Q>(i, (size_t)cell));
        else
            gd[pop_at64<Q>(i, (size_t)cell)] = out;
    }
    if (MODE == 2) {
        st_fld_at((T*)m.rho, (unsigned)cell, drho, WT);
#pragma unroll
        for (int a = 0; a < D; ++a) st_fld_at((T*)m.vs + (size_t)a * N, (unsigned)cell, us[a], WT);
    }
    if (MODE == 1 && SUB != LBM_WALE) {  // (with WALE, k_moments wrote v^n)
#pragma unroll
        for (int a = 0; a < D; ++a) ((T*)m.vn)[(size_t)a * N + cell] = u[a];
    }
    if (MODE >= 1) {
        st[0] += (double)drho;
#pragma unroll
        for (int a = 0; a < D; ++a) st[1 + a] += (double)(rho * u[a]);
    }
}

// A32: every population buffer of the launch spans less than 4 GiB, so
// pulls and stores use 32-bit offsets.  NT (plain modes): the populations are
// stored non-temporally, on launches whose populations exceed the Infinity
// Cache.
template <int LAT, typename T, int PREC, int SUB, int MODE, bool WT = false, bool A32 = MODE == 2, bool NT = false>
__global__ __launch_bounds__(kBlock, MODE == 2 ? 1 : 8) void k_step(const DevMember* __restrict__ mems,
                                                 const int2* __restrict__ work, int flip)
{
    using L = Lat<LAT>;
    constexpr int Q = L::Q;
    __shared__ double lds[4 * (kBlock / 64)];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int N = m.N, nx = m.nx, ny = m.ny;
    const int cell = wk.y * kBlock + threadIdx.x;
    const int cur = m.parity ^ flip;
    const T* __restrict__ gs = (const T*)m.g[cur];
    T* __restrict__ gd = (T*)m.g[cur ^ 1];
    double st[4] = {0, 0, 0, 0};
    int bad = 0;
    if (cell < N) {
        const int x = cell % nx, t = cell / nx, y = t % ny, z = t / ny;
        T f[Q];
        gather<LAT, T, A32>(m, gs, x, y, z, cell, f);
        collide_cell<LAT, T, PREC, SUB, MODE, WT, A32, NT>(m, f, x, y, z, cell, gd, st, bad);
    }
    if (MODE >= 1) {
        block_sum<4>(st, lds);
        if (threadIdx.x == 0) {
            double* p = m.part_stats + (size_t)wk.y * 4;
            p[0] = st[0]; p[1] = st[1]; p[2] = st[2]; p[3] = st[3];
        }
    }
    const unsigned long long anybad = __ballot(bad);
    if (anybad && (threadIdx.x & 63) == 0) atomicOr(&m.ctl->flags, 1);
}

// K1t: the TO stream-collide with the previous step's SGS change deferred
// into the pull.  A workgroup owns a TX x TY tile of the xy plane and a chunk
// of zc planes.  For every plane
// of the chunk and one halo plane on each side, the record (a, b) of the tile
// and its one-cell xy halo is staged in LDS together with e = a.b; the pull
// of population i at cell x then reads g*_i(x - c_i) from memory and the
// record of x - c_i from LDS, or for a bounce-back g*_opp(x) and the record of
// x itself.  The records of a step are zero after a flush (nothing pending).
// Statistics are summed per workgroup over its cells in z order.
// (At most 128 VGPRs in FP32: the LDS of a workgroup already limits the
// kernel to four waves per SIMD, and left alone the compiler hoists every
// pull and record read of a cell, 169 VGPRs, two waves.)
#ifndef LBM_STEPT_WAVES
#define LBM_STEPT_WAVES 4
#endif
template <int LAT, typename T, int PREC, int SUB, int TX, int WT, bool A32 = true>
__global__ __launch_bounds__(TX * kBinTY, sizeof(T) == 4 ? LBM_STEPT_WAVES : 2) void k_step_t(const DevMember* __restrict__ mems,
                                                   const int2* __restrict__ work, int flip)
{
    using L = Lat<LAT>;
    constexpr int Q = L::Q, D = L::D;
    constexpr int NT = TX * kBinTY, TY = kBinTY, HX = TX + 2, HY = TY + 2, HXY = HX * HY;
    constexpr int NR = 2 * D;                     // a, b
    constexpr int NSL = D == 3 ? 3 : 1;           // staged planes
    constexpr int NE = (HXY + NT - 1) / NT;
    __shared__ T rs[NSL][NR + 1][HXY];            // a, b, e of the staged cells
    __shared__ double lds[4 * (NT / 64)];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int N = m.N, nx = m.nx, ny = m.ny, nz = m.nz;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    const int zc = m.zc;
    const int tx0 = (wk.y % ntx) * TX;
    const int ty0 = ((wk.y / ntx) % nty) * TY;
    const int tz0 = D == 3 ? (wk.y / (ntx * nty)) * zc : 0;
    const int lx = threadIdx.x % TX, ly = threadIdx.x / TX;
    const int x = tx0 + lx, y = ty0 + ly;
    const bool own = x < nx && y < ny;
    const int cur = m.parity ^ flip;
    const T* __restrict__ gs = (const T*)m.g[cur];
    T* __restrict__ gd = (T*)m.g[cur ^ 1];
    const T* __restrict__ rec = (const T*)m.rec;
    const unsigned sN = (unsigned)N;
    // halo elements staged by this thread, as offsets within a plane; an
    // element beyond a wall loads cell 0 (a bounce-back never reads it)
    int eoff[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = threadIdx.x + k * NT;
        const int hx = e % HX, hy = e / HX;
        const int gx = modi(tx0 + hx - 1, nx);
        int gy = ty0 + hy - 1;
        bool ok = e < HXY;
        if (m.walls) ok = ok && gy >= 0 && gy < ny;
        else gy = modi(gy, ny);
        eoff[k] = ok ? gx + nx * gy : 0;
    }
    const int plane = nx * ny;
    auto fetch = [&](int pz, T (&buf)[NE][NR]) {
        const unsigned zo = (unsigned)(plane * (D == 3 ? modi(pz, nz) : 0));
#pragma unroll
        for (int k = 0; k < NE; ++k)
#pragma unroll
            for (int c = 0; c < NR; ++c) buf[k][c] = ld_at(rec + c * sN, zo + (unsigned)eoff[k]);
    };
    auto stage = [&](int sl, const T (&buf)[NE][NR]) {
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const int e = threadIdx.x + k * NT;
            if (e < HXY) {
#pragma unroll
                for (int c = 0; c < NR; ++c) rs[sl][c][e] = buf[k][c];
                rs[sl][NR][e] = rec_e<D, T>(&buf[k][0], &buf[k][D]);
            }
        }
    };
    double st[4] = {0, 0, 0, 0};
    int bad = 0;
    // the 19 pulls g*_pi(src) of the own cell of plane z (issued before the
    // plane's records are staged, so their latency overlaps the staging)
    // (the general pull only: a constant-offset branch here costs the
    // kernel spills within its 128-VGPR budget)
    auto pull = [&](int z, T (&f)[Q]) { gather<LAT, T, A32, false>(m, gs, x, y, z, x + nx * (y + ny * z), f); };
    // add delta f of each pulled population from the staged records (a
    // bounce-back pulls population opp(i) of the cell itself: its delta f
    // from the own record with the sign of the linear term flipped, so every
    // direction is evaluated with constant c_i) and collide; sl0, sl1, sl2:
    // the staged planes z - 1, z, z + 1
    auto cell_step = [&](int z, int sl0, int sl1, int sl2, T (&f)[Q]) {
        const int cell = x + nx * (y + ny * z);
        const int pown = (ly + 1) * HX + lx + 1;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int sy = y - L::cy[i];
            const bool bb = L::cy[i] != 0 && m.walls && (sy < 0 || sy >= ny);
            const int slz = D == 3 ? (L::cz[i] > 0 ? sl0 : (L::cz[i] < 0 ? sl2 : sl1)) : 0;
            const int pos = bb ? pown : pown - L::cy[i] * HX - L::cx[i];
            const T* r = &rs[bb ? sl1 : slz][0][pos];
            const T ca = cdot<LAT, T>(i, [&](int k) { return r[k * HXY]; });
            const T cb = cdot<LAT, T>(i, [&](int k) { return r[(D + k) * HXY]; });
            f[i] = add_rn(f[i], df_cc<LAT, T>(i, bb, ca, cb, r[NR * HXY]));
        }
        collide_cell<LAT, T, PREC, SUB, 2, WT, A32>(m, f, x, y, z, cell, gd, st, bad);
    };
    if constexpr (D == 2) {
        T buf[NE][NR], f[Q];
        fetch(0, buf);
        if (own) pull(0, f);
        stage(0, buf);
        __syncthreads();
        if (own) cell_step(0, 0, 0, 0, f);
    } else {
        // planes tz0 - 1 .. zend staged in a ring of three; the records of
        // the next plane and the pulls of the current one are in flight
        // while a plane is staged
        const int zend = min(tz0 + zc, nz);
        const int p0 = tz0 - 1, p1 = zend;
        T buf[NE][NR];
        fetch(p0, buf);
        for (int pz = p0; pz <= p1; ++pz) {
            const int sl = (pz - p0) % 3;
            const bool cmp = pz >= tz0 + 1 && own;   // plane pz - 1 once its upper neighbour is staged
            T f[Q];
            if (cmp) pull(pz - 1, f);
            stage(sl, buf);
            __syncthreads();
            if (pz < p1) fetch(pz + 1, buf);
            if (cmp) cell_step(pz - 1, (pz - 2 - p0) % 3, (pz - 1 - p0) % 3, sl, f);
            __syncthreads();
        }
    }
    block_sum<4, NT / 64>(st, lds);
    if (threadIdx.x == 0) {
        double* p = m.part_stats + (size_t)wk.y * 4;
        p[0] = st[0]; p[1] = st[1]; p[2] = st[2]; p[3] = st[3];
    }
    const unsigned long long anybad = __ballot(bad);
    if (anybad && (threadIdx.x & 63) == 0) atomicOr(&m.ctl->flags, 1);
}

// ---------------------------------------------------------------------------
// Post-streaming density and velocity of the current state (stream only,
// the SGS change of the last step included): used for WALE gradients and
// lbm_fields.  rho_out and u_out (nullable): rho [N] and v [D][N] in double.
// ---------------------------------------------------------------------------
template <int LAT, typename T, int PREC, bool TO>
__global__ __launch_bounds__(kBlock) void k_moments(const DevMember* __restrict__ mems,
                                                    const int2* __restrict__ work, int flip,
                                                    double* __restrict__ rho_out, double* __restrict__ u_out)
{
    using L = Lat<LAT>;
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int N = m.N, nx = m.nx, ny = m.ny;
    const int cell = wk.y * kBlock + threadIdx.x;
    if (cell >= N) return;
    const int x = cell % nx, t = cell / nx, y = t % ny, z = t / ny;
    const T* gs = (const T*)m.g[m.parity ^ flip];
    T f[L::Q];
    gather<LAT, T, false>(m, gs, x, y, z, cell, f);
    T drho, j[3] = {0, 0, 0};
    moments<LAT, T, PREC>(f, drho, j);
    const T rho = T(1) + drho;
#pragma unroll
    for (int a = 0; a < L::D; ++a) {
        const T v = j[a] / rho;
        ((T*)m.vn)[(size_t)a * N + cell] = v;
        if (u_out) u_out[(size_t)a * N + cell] = (double)v;
    }
    if (rho_out) rho_out[cell] = (double)rho;
}

// ---------------------------------------------------------------------------
// Helpers for stencils on scalar fields with the filter/derivative boundary
// rule: periodic wrap, zero outside the domain on the wall axis.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T fld(const T* __restrict__ u, int x, int y, int z, int nx, int ny, int nz, int walls)
{
    x = wrapi(x, nx);
    z = wrapi(z, nz);
    if (walls) {
        if (y < 0 || y >= ny) return T(0);
    } else
        y = wrapi(y, ny);
    return u[x + nx * (y + ny * z)];
}

// Central-difference curl of a D-component field at (x,y,z) (2-D: scalar).
template <int D, typename T>
__device__ __forceinline__ void curl_at(const T* __restrict__ v, size_t N, int x, int y, int z, int nx, int ny,
                                        int nz, int walls, T* w)
{
    const T* vx = v;
    const T* vy = v + N;
    if (D == 2) {
        w[0] = T(0.5) * (fld(vy, x + 1, y, z, nx, ny, nz, walls) - fld(vy, x - 1, y, z, nx, ny, nz, walls)) -
               T(0.5) * (fld(vx, x, y + 1, z, nx, ny, nz, walls) - fld(vx, x, y - 1, z, nx, ny, nz, walls));
    } else {
        const T* vz = v + 2 * N;
        T dyvz = T(0.5) * (fld(vz, x, y + 1, z, nx, ny, nz, walls) - fld(vz, x, y - 1, z, nx, ny, nz, walls));
        T dzvy = T(0.5) * (fld(vy, x, y, z + 1, nx, ny, nz, walls) - fld(vy, x, y, z - 1, nx, ny, nz, walls));
        T dzvx = T(0.5) * (fld(vx, x, y, z + 1, nx, ny, nz, walls) - fld(vx, x, y, z - 1, nx, ny, nz, walls));
        T dxvz = T(0.5) * (fld(vz, x + 1, y, z, nx, ny, nz, walls) - fld(vz, x - 1, y, z, nx, ny, nz, walls));
        T dxvy = T(0.5) * (fld(vy, x + 1, y, z, nx, ny, nz, walls) - fld(vy, x - 1, y, z, nx, ny, nz, walls));
        T dyvx = T(0.5) * (fld(vx, x, y + 1, z, nx, ny, nz, walls) - fld(vx, x, y - 1, z, nx, ny, nz, walls));
        w[0] = dyvz - dzvy;
        w[1] = dzvx - dxvz;
        w[2] = dxvy - dyvx;
    }
}

// Neighbour offsets of cell c = (x, y, z) for second-order central
// differences: periodic wrap, and on the wall axis a neighbour beyond a wall
// is the cell itself, counted as zero (ok flags).  Every load of the
// differences below is unconditional, a 32-bit offset from a scalar base (TO
// fields stay below 2^32 bytes), so no branch-joined load stalls the others.
struct Nbr {
    unsigned xm, xp, ym, yp, zm, zp;
    bool okm, okp;
};
__device__ __forceinline__ Nbr nbr_at(unsigned c, int x, int y, int z, int nx, int ny, int nz, int walls, int D)
{
    Nbr n;
    n.xm = c - x + wrapi(x - 1, nx);
    n.xp = c - x + wrapi(x + 1, nx);
    n.okm = true;
    n.okp = true;
    int ym = y - 1, yp = y + 1;
    if (walls) { n.okm = ym >= 0; n.okp = yp < ny; ym = n.okm ? ym : y; yp = n.okp ? yp : y; }
    else { ym = wrapi(ym, ny); yp = wrapi(yp, ny); }
    n.ym = c + (unsigned)((ym - y) * nx);
    n.yp = c + (unsigned)((yp - y) * nx);
    const int plane = nx * ny;
    n.zm = D == 3 ? c + (unsigned)((wrapi(z - 1, nz) - z) * plane) : c;
    n.zp = D == 3 ? c + (unsigned)((wrapi(z + 1, nz) - z) * plane) : c;
    return n;
}

// Central-difference curl of the D-component field u at a cell (2-D: the
// scalar D_x u_y - D_y u_x).  In 3-D the adjoint curl^T is the curl itself.
template <int D, typename T>
__device__ __forceinline__ void curl_nb(const T* __restrict__ u, unsigned sN, unsigned c, const Nbr& n, T* w)
{
    const T* ux = u;
    const T* uy = u + sN;
    auto y0 = [](bool ok, T v) { return ok ? v : T(0); };
    if (D == 2) {
        w[0] = T(0.5) * (ld_at(uy, n.xp) - ld_at(uy, n.xm)) -
               T(0.5) * (y0(n.okp, ld_at(ux, n.yp)) - y0(n.okm, ld_at(ux, n.ym)));
    } else {
        const T* uz = u + 2 * sN;
        const T dyuz = T(0.5) * (y0(n.okp, ld_at(uz, n.yp)) - y0(n.okm, ld_at(uz, n.ym)));
        const T dzuy = T(0.5) * (ld_at(uy, n.zp) - ld_at(uy, n.zm));
        const T dzux = T(0.5) * (ld_at(ux, n.zp) - ld_at(ux, n.zm));
        const T dxuz = T(0.5) * (ld_at(uz, n.xp) - ld_at(uz, n.xm));
        const T dxuy = T(0.5) * (ld_at(uy, n.xp) - ld_at(uy, n.xm));
        const T dyux = T(0.5) * (y0(n.okp, ld_at(ux, n.yp)) - y0(n.okm, ld_at(ux, n.ym)));
        w[0] = dyuz - dzuy;
        w[1] = dzux - dxuz;
        w[2] = dxuy - dyux;
    }
}

// The adjoint curl of a curl field psi (NC components) at a cell, 2-D
// (D_y psi, -D_x psi) (eq. enstrophy-sensitivity-2d), 3-D curl psi
// (eq. enstrophy-sensitivity-3d), in two steps, so that a caller can hold the
// loads and form the curl later: the neighbour values (2-D: psi at y+1, y-1,
// x+1, x-1; 3-D: psi_z, psi_y, psi_x at the pairs of neighbours of D_y psi_z,
// D_z psi_y, D_z psi_x, D_x psi_z, D_x psi_y, D_y psi_x), then central
// differences (zero beyond the walls), without contraction.
template <int D, typename T>
__device__ __forceinline__ void curlT_load(const T* __restrict__ psi, unsigned sN, const Nbr& n, T* r)
{
    if constexpr (D == 2) {
        r[0] = ld_at(psi, n.yp); r[1] = ld_at(psi, n.ym);
        r[2] = ld_at(psi, n.xp); r[3] = ld_at(psi, n.xm);
    } else {
        const T* ux = psi;
        const T* uy = psi + sN;
        const T* uz = psi + 2 * (size_t)sN;
        r[0] = ld_at(uz, n.yp); r[1] = ld_at(uz, n.ym);
        r[2] = ld_at(uy, n.zp); r[3] = ld_at(uy, n.zm);
        r[4] = ld_at(ux, n.zp); r[5] = ld_at(ux, n.zm);
        r[6] = ld_at(uz, n.xp); r[7] = ld_at(uz, n.xm);
        r[8] = ld_at(uy, n.xp); r[9] = ld_at(uy, n.xm);
        r[10] = ld_at(ux, n.yp); r[11] = ld_at(ux, n.ym);
    }
}

template <int D, typename T>
__device__ __forceinline__ void curlT_eval(const T* r, bool okm, bool okp, T* out)
{
#pragma clang fp contract(off)
    auto y0 = [](bool ok, T v) { return ok ? v : T(0); };
    if constexpr (D == 2) {
        out[0] = T(0.5) * (y0(okp, r[0]) - y0(okm, r[1]));
        out[1] = -(T(0.5) * (r[2] - r[3]));
    } else {
        const T dyuz = T(0.5) * (y0(okp, r[0]) - y0(okm, r[1]));
        const T dzuy = T(0.5) * (r[2] - r[3]);
        const T dzux = T(0.5) * (r[4] - r[5]);
        const T dxuz = T(0.5) * (r[6] - r[7]);
        const T dxuy = T(0.5) * (r[8] - r[9]);
        const T dyux = T(0.5) * (y0(okp, r[10]) - y0(okm, r[11]));
        out[0] = dyuz - dzuy;
        out[1] = dzux - dxuz;
        out[2] = dxuy - dyux;
    }
}

// K2a: w = curl v* of kernel-filter and Fourier closures, whose filter passes
// start from w, into the field after the nsa fields U_s.
template <int LAT, typename T, bool WT>
__global__ __launch_bounds__(kBlock) void k_curl(const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    using L = Lat<LAT>;
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    if (!kc(m.prm)->has_z) return;
    const int N = m.N, nx = m.nx, ny = m.ny, nz = m.nz;
    const int cell = wk.y * kBlock + threadIdx.x;
    if (cell >= N) return;
    const int x = cell % nx, t = cell / nx, y = t % ny, z = t / ny;
    const unsigned c = (unsigned)cell;
    const Nbr nb = nbr_at(c, x, y, z, nx, ny, nz, m.walls, L::D);
    T w[3];
    curl_nb<L::D, T>((const T*)m.vs, (unsigned)N, c, nb, w);
    T* W = (T*)m.W + (size_t)kc(m.prm)->nsa * L::NC * N;
#pragma unroll
    for (int a = 0; a < L::NC; ++a) st_fld_at(W + (size_t)a * N, c, w[a], WT);
}

// ---------------------------------------------------------------------------
// K2: the filter chains of the binomial closures, v* to sensitivities in one
// launch.  Filters are polynomials of the binomial operator
// B = (x)_a [1,2,1]/4, so with P_j = B^j v* and W_j = B^j w, w = curl v*:
//   E: V_s = R R v* = sum_j rr_sj P_j        (stored, the final sensitivity);
//   Z: U_s = R R w  = sum_j rr_sj W_j        (stored; k_reduce forms
//      V_s = curl^T U_s from it);
// and the QoI densities 1/2 |R v*|^2, 1/2 |R w|^2 of the tile's cells, summed
// in FP64 per workgroup.  Each component of v* and of w is a chain of its own
// and a workgroup's whole work, so nothing passes between components.
//
// A wavefront's lanes are 64 neighbouring cells in x, of which the inner
// 64 - 2 H are the tile's own (H = NL, a cell for each power); each
// thread holds chain_rows() rows in y.  x neighbours come from DPP lane moves,
// y neighbours from the thread's own rows, except those of its first and last
// row, which pass through LDS between the wavefronts of the workgroup
// (3-D).  In 3-D the workgroup marches in z, two planes at a time (one barrier
// per power and pair): every power keeps the two values its z part needs and
// lags the one before it by a plane, and W_0.. wait in registers until the
// highest power of their plane is known.  [1,2,1] is applied as [1,1] twice
// (two additions per axis, no products); the scale 4^-D per power, exact in
// binary, is in the coefficients.
//
// The powers are never stored: about 100 B of traffic per cell (FP32 channel,
// three QoIs of each kind; counters: 25 in, 76 out) where one launch per power
// moved 260.  Bound by its vector instructions (half of the time; half of
// those form the sensitivities and densities) and by the stores of row
// segments that are not whole lines; measured on MI355X: 31.8 us in four
// launches -> 24 us on 96 x 48 x 48, 781 -> 514 us on 384 x 192 x 192 (352 us
// with the stores left out); on 256 x 256 two launches of 4.6 us -> one of 5.
// The stores are plain ones: neighbouring tiles share lines, which the L2
// merges (non-temporal 624 us, written through 2 us slower on 96 x 48 x 48).
// Without two planes at a time, with the phases of the waiting rings unrolled
// (75 to 100 KB of code), the same march took 660 us.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T fma_(T a, T b, T c);
template <> __device__ __forceinline__ float fma_<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <> __device__ __forceinline__ double fma_<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The value of the previous (next) lane of the wavefront; zero past its ends.
template <int CTRL> __device__ __forceinline__ float lane_shift(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double lane_shift(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <typename T> __device__ __forceinline__ T lane_prev(T v) { return lane_shift<0x138>(v); }   // wave_shr:1
template <typename T> __device__ __forceinline__ T lane_next(T v) { return lane_shift<0x130>(v); }   // wave_shl:1

// Coefficients of the chains in the kernel's arithmetic type.
template <typename T> __device__ __forceinline__ T chain_r(KParam* p, int s, int j);
template <> __device__ __forceinline__ float chain_r<float>(KParam* p, int s, int j) { return p->rf[s][j]; }
template <> __device__ __forceinline__ double chain_r<double>(KParam* p, int s, int j) { return p->r[s][j]; }
template <typename T> __device__ __forceinline__ T chain_rr(KParam* p, int s, int j);
template <> __device__ __forceinline__ float chain_rr<float>(KParam* p, int s, int j) { return p->rrf[s][j]; }
template <> __device__ __forceinline__ double chain_rr<double>(KParam* p, int s, int j) { return p->rr[s][j]; }

// One component's chain on one tile.  CURL < 0: component comp of v*; 0, 1,
// 2: that component of w (2-D: 2, the only one).  edge: LDS of the row
// exchange, [NL][NW + 2][2][2][64], its first and last wavefront slots zero.
template <int LAT, typename T, int NL, int MS, int CURL>
__device__ __forceinline__ void chain_job(KMember& m, KParam* prm, int comp, int tile, T* edge, double* red)
{
    using L = Lat<LAT>;
    constexpr int D = L::D, NC = L::NC, H = NL, R = chain_rows(D, sizeof(T)), NW = chain_waves(D);
    constexpr int KIND = CURL < 0 ? 0 : 1;
    const int nx = m.nx, ny = m.ny, nz = m.nz, walls = m.walls;
    const size_t sN = (size_t)m.N;
    const int nk = prm->nk[KIND];
    const int tx = tile % m.cntx, ty = (tile / m.cntx) % m.cnty, tz = tile / (m.cntx * m.cnty);
    const int lane = threadIdx.x & 63;
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int x0 = tx * m.cvx, xe = min(x0 + m.cvx, nx), y0 = ty * m.cvy, ye = min(y0 + m.cvy, ny);
    // byte offsets of the lane's cell and (for D_x) of its x neighbours
    const int xc = modi(x0 - H + lane, nx);
    const unsigned xb = (unsigned)xc * sizeof(T), xm = (unsigned)wrapi(xc - 1, nx) * sizeof(T),
                   xp = (unsigned)wrapi(xc + 1, nx) * sizeof(T);
    const bool ownx = lane >= H && lane - H < xe - x0;
    // rows -1 .. R of the wavefront: offset in the plane, whether inside the
    // walls (a row beyond them counts as zero and loads row 0), whether own
    const int ys = (walls && ty == 0 ? 0 : y0 - H) + wv * R;
    unsigned yo[R + 2];     // in bytes
    unsigned outm = 0;      // bit r + 1: row r is beyond a wall
    bool any_own = false;
    {
        int yy = modi(ys - 1, ny);
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            const int y = ys - 1 + r;
            const bool ok = !walls || (y >= 0 && y < ny);
            yo[r] = ok ? (unsigned)(yy * nx) * (unsigned)sizeof(T) : 0u;
            outm |= ok ? 0u : 1u << r;
            any_own = any_own || (r >= 1 && r <= R && y >= y0 && y < ye);
            yy = yy + 1 == ny ? 0 : yy + 1;
        }
    }
    double acc[MS];
#pragma unroll
    for (int i = 0; i < MS; ++i) acc[i] = 0;
    const T* vs = (const T*)m.vs;
    // (32-bit byte offsets from scalar bases, the row's part added per use:
    // TO fields stay below 2^32 bytes)
    auto row = [&](const T* base, unsigned zo, int r, unsigned x) {
        return *(const T*)((const char*)base + (zo + yo[r + 1] + x));
    };
    // rows beyond the walls of a field count as zero
    auto mask = [&](T (&a)[R]) {
        if (!outm) return;   // uniform
#pragma unroll
        for (int r = 0; r < R; ++r) a[r] = (outm >> (r + 1)) & 1 ? T(0) : a[r];
    };
    auto mask2 = [&](T (&a)[R + 2]) {
        if (!outm) return;
#pragma unroll
        for (int r = 0; r < R + 2; ++r) a[r] = (outm >> r) & 1 ? T(0) : a[r];
    };
    // x and y parts of one power, [1,2,1] along x and along y, of NP planes
    // at once (one barrier)
    constexpr int NP = D == 3 ? 2 : 1;
    auto filter_xy = [&](int l, T (&a)[NP][R]) {
#pragma unroll
        for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T t = a[u][r] + lane_prev(a[u][r]);
                a[u][r] = t + lane_next(t);
            }
        T lo[NP] = {}, hi[NP] = {};
        if constexpr (NW > 1) {
            T* e = edge + (size_t)l * (NW + 2) * NP * 128 + lane;
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                e[((wv + 1) * NP + u) * 128] = a[u][0];
                e[((wv + 1) * NP + u) * 128 + 64] = a[u][R - 1];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                lo[u] = e[(wv * NP + u) * 128 + 64];
                hi[u] = e[((wv + 2) * NP + u) * 128];
            }
        }
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            T s = lo[u] + a[u][0];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T n = a[u][r] + (r + 1 < R ? a[u][r + 1 < R ? r + 1 : r] : hi[u]);
                a[u][r] = s + n;
                s = n;
            }
        }
    };
    auto own_row = [&](int r) { return ys + r >= y0 && ys + r < ye; };
    T cr[MS][3], crr[MS][NL + 1];
    T* dst[MS];
#pragma unroll
    for (int i = 0; i < MS; ++i) {
        const int s = prm->ks[KIND][i];
#pragma unroll
        for (int j = 0; j < 3; ++j) cr[i][j] = chain_r<T>(prm, s, j);
#pragma unroll
        for (int j = 0; j <= NL; ++j) crr[i][j] = chain_rr<T>(prm, s, j);
        dst[i] = (T*)(KIND == 0 ? m.kV : m.W) + ((size_t)s * (KIND == 0 ? D : NC) + comp) * sN;
    }
    // sensitivities of the own rows from their powers w_0 .. w_NL, stored;
    // densities
    auto emit = [&](unsigned zo, const T (&w)[NL + 1][R]) {
        if (!any_own || !ownx) return;
#pragma unroll
        for (int i = 0; i < MS; ++i) {
            if (i >= nk) break;   // uniform
            T v[R], d[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r] = crr[i][0] * w[0][r];
#pragma unroll
                for (int j = 1; j <= NL; ++j) v[r] = fma_(crr[i][j], w[j][r], v[r]);
                d[r] = fma_(cr[i][2], w[2][r], fma_(cr[i][1], w[1][r], cr[i][0] * w[0][r]));
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!own_row(r)) continue;   // uniform
                acc[i] = __builtin_fma((double)d[r], (double)d[r], acc[i]);
                *(T*)((char*)dst[i] + (zo + yo[r + 1] + xb)) = v[r];
            }
        }
    };
    if constexpr (D == 2) {
        T a[R], b[R + 2];
        if constexpr (CURL < 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = row(vs + comp * sN, 0, r, xb);
        } else {
            T c[R];
#pragma unroll
            for (int r = 0; r < R; ++r) { a[r] = row(vs + sN, 0, r, xp); c[r] = row(vs + sN, 0, r, xm); }
#pragma unroll
            for (int r = -1; r <= R; ++r) b[r + 1] = row(vs, 0, r, xb);
            mask2(b);
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = (a[r] - c[r]) - (b[r + 2] - b[r]);
        }
        mask(a);
        T w[NL + 1][R], f[1][R];
#pragma unroll
        for (int r = 0; r < R; ++r) w[0][r] = f[0][r] = a[r];
#pragma unroll
        for (int j = 1; j <= NL; ++j) {
            filter_xy(j - 1, f);
            mask(f[0]);
#pragma unroll
            for (int r = 0; r < R; ++r) w[j][r] = f[0][r];
        }
        emit(0, w);
    } else {
        const unsigned plane = (unsigned)(nx * ny) * (unsigned)sizeof(T);
        const int z0 = tz * m.czc, z1 = min(z0 + m.czc, nz);
        const T* fa = CURL < 0 ? vs + comp * sN : CURL == 1 ? vs : vs + sN;
        const T* fb = CURL == 2 ? vs : vs + 2 * sN;
        // CURL 0: D_y fb - D_z fa; 1: D_z fa - D_x fb; 2: D_x fa - D_y fb.
        // fa's z difference takes planes p - 1 and p + 1 (am, an); D_y takes
        // fb's rows -1 .. R, D_x the rows at x + 1 and x - 1.
        constexpr bool ZD = CURL == 0 || CURL == 1;
        constexpr int NB = CURL < 0 ? 1 : (CURL == 1 ? 2 * R : R + 2);
        T am[R], ac[R], an[2][R], ax[2][CURL == 2 ? R : 1], bn[2][NB];
        T px[NL][R], pt[NL][R];             // per power: last plane's xy part; sum of the last two
        T d[NL][NL][R];                     // w_j waiting for the highest power of their plane: d[j][0 .. NL - j - 1]
#pragma unroll
        for (int r = 0; r < R; ++r) {
            am[r] = ac[r] = T(0);
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                px[l][r] = 0;
                pt[l][r] = 0;
#pragma unroll
                for (int k = 0; k < NL - l; ++k) d[l][k][r] = 0;
            }
        }
        // planes of w_0: [pa, pb), two at a time (a plane past pb is loaded
        // and filtered to no effect)
        const int pa = z0 - NL, pb = z1 + NL;
        const unsigned zlast = (unsigned)(nz - 1) * plane;
        auto next = [&](unsigned z) { return z == zlast ? 0u : z + plane; };
        unsigned za = (unsigned)modi(ZD ? pa - 1 : pa, nz) * plane;   // planes of the fa and fb rows fetched next
        unsigned zb = (unsigned)modi(pa, nz) * plane;
        auto fetch = [&] {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    an[u][r] = row(fa, za, r, CURL == 2 ? xp : xb);
                    if constexpr (CURL == 2) ax[u][r] = row(fa, za, r, xm);
                }
                za = next(za);
                if constexpr (CURL == 1) {
#pragma unroll
                    for (int r = 0; r < R; ++r) { bn[u][r] = row(fb, zb, r, xp); bn[u][R + r] = row(fb, zb, r, xm); }
                } else if constexpr (CURL >= 0) {
#pragma unroll
                    for (int k = 0; k < NB; ++k) bn[u][k] = row(fb, zb, k - 1, xb);
                }
                zb = next(zb);
            }
        };
        if constexpr (ZD) {
#pragma unroll
            for (int r = 0; r < R; ++r) am[r] = row(fa, za, r, xb);
            za = next(za);
#pragma unroll
            for (int r = 0; r < R; ++r) ac[r] = row(fa, za, r, xb);
            za = next(za);
        }
        // w_0 of the two planes fetched last
        auto form = [&](T (&a)[2][R]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if constexpr (CURL == 0 || CURL == 2) mask2(bn[u]);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if constexpr (CURL < 0) a[u][r] = an[u][r];
                    const T below = u == 0 ? am[r] : ac[r];
                    if constexpr (CURL == 0) a[u][r] = (bn[u][r + 2] - bn[u][r]) - (an[u][r] - below);    // D_y v_z - D_z v_y
                    if constexpr (CURL == 1) a[u][r] = (an[u][r] - below) - (bn[u][r] - bn[u][R + r]);    // D_z v_x - D_x v_z
                    if constexpr (CURL == 2) a[u][r] = (an[u][r] - ax[u][r]) - (bn[u][r + 2] - bn[u][r]); // D_x v_y - D_y v_x
                }
            }
            if constexpr (ZD) {
#pragma unroll
                for (int r = 0; r < R; ++r) { am[r] = an[0][r]; ac[r] = an[1][r]; }
            }
            mask(a[0]);
            mask(a[1]);
        };
        fetch();
        T a[2][R];
        form(a);
        unsigned zo = (unsigned)z0 * plane;   // output plane
#pragma unroll 1
        for (int p = pa; p < pb; p += 2) {
            T w[2][NL + 1][R];
            fetch();   // the next planes, in flight during this pair's filtering
            // w_j of planes p - NL and p + 1 - NL: waiting ones first; the
            // new ones take their places
            auto queue = [&](int j) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int L = NL - j;   // planes w_j waits
                    if (L == 0) { w[0][j][r] = a[0][r]; w[1][j][r] = a[1][r];}
                    else if (L == 1) { w[0][j][r] = d[j][0][r]; w[1][j][r] = a[0][r]; d[j][0][r] = a[1][r]; }
                    else {
                        w[0][j][r] = d[j][0][r];
                        w[1][j][r] = d[j][1][r];
#pragma unroll
                        for (int k = 0; k + 2 < L; ++k) d[j][k][r] = d[j][k + 2][r];
                        d[j][L - 2][r] = a[0][r];
                        d[j][L - 1][r] = a[1][r];
                    }
                }
            };
            queue(0);
#pragma unroll
            for (int j = 1; j <= NL; ++j) {
                filter_xy(j - 1, a);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const T t0 = px[j - 1][r] + a[0][r], t1 = a[0][r] + a[1][r];
                    px[j - 1][r] = a[1][r];
                    a[0][r] = pt[j - 1][r] + t0;
                    a[1][r] = t0 + t1;
                    pt[j - 1][r] = t1;
                }
                mask(a[0]);
                mask(a[1]);
                queue(j);
            }
            // the next pair's w_0, formed ahead of this pair's stores: loads
            // and stores complete in one order, so a wait for the loads at the
            // head of the next pair would wait for the stores as well
            form(a);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) asm volatile("" : "+v"(a[u][r]) : : "memory");
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (p + u < z0 + NL || p + u >= pb) continue;   // uniform
                emit(zo, w[u]);
                zo += plane;
            }
        }
    }
    if constexpr (NW > 1) __syncthreads();
    block_sum<MS, NW>(acc, red);
    if (threadIdx.x == 0) {
        const int ncw = m.cnt * D;   // row length of part_q
#pragma unroll
        for (int i = 0; i < MS; ++i)
            if (i < nk) m.part_q[(size_t)prm->ks[KIND][i] * ncw + tile * (KIND == 0 ? D : NC) + comp] = 0.5 * acc[i];
    }
}

template <int LAT, typename T, int NL, int MS>
__global__ __launch_bounds__(64 * chain_waves(Lat<LAT>::D), Lat<LAT>::D == 2 ? 1 : 2) void k_chain(
    const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    using L = Lat<LAT>;
    constexpr int D = L::D, NC = L::NC, NW = chain_waves(D);
    __shared__ T edge[NW > 1 ? NL * (NW + 2) * 256 : 1];
    __shared__ double red[MS * NW];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    KParam* prm = kc(m.prm);
    const int tile = wk.y / (D + NC), job = wk.y % (D + NC);
    if constexpr (NW > 1) {
        for (int k = threadIdx.x; k < NL * 512; k += 64 * NW) {   // the slots beyond the first and last wavefront
            const int l = k / 512, e = k % 512;
            edge[(size_t)l * (NW + 2) * 256 + (e < 256 ? e : (NW + 1) * 256 + e - 256)] = T(0);
        }
        __syncthreads();
    }
    if (job < D) chain_job<LAT, T, NL, MS, -1>(m, prm, job, tile, edge, red);
    else if (D == 2) chain_job<LAT, T, NL, MS, 2>(m, prm, 0, tile, edge, red);
    else if (job == D) chain_job<LAT, T, NL, MS, D == 3 ? 0 : 2>(m, prm, 0, tile, edge, red);
    else if (job == D + 1) chain_job<LAT, T, NL, MS, D == 3 ? 1 : 2>(m, prm, 1, tile, edge, red);
    else chain_job<LAT, T, NL, MS, 2>(m, prm, 2, tile, edge, red);
}

// K2 and K2c of 2-D closures of at most one E and one Z QoI and no
// mean-profile QoIs (the paper's 2-D set): chains, adjoint curl and Gram sums
// in one launch, one wavefront per tile.  v* of the tile and its halo lies in
// registers (16 rows, lanes in x); powers as in k_chain, the curls from
// neighbouring lanes and rows, so the halo is NL + 2 cells in x and NL + 1 in y.
// Bound by its launch and one load latency: measured on MI355X, 256 x 256, FP32,
// k_chain and k_reduce 5.0 and 4.9 us -> one launch of 5.5 us; 16 members of
// 128 to 208 cells squared, 7 and 11 -> 7.2 us.
// EZ: bit 0 an E QoI, bit 1 a Z QoI; MASK: the tile has rows beyond a wall.
// (Template parameters, so that the chains of a tile are one block of code
// that the compiler can interleave.)
template <typename T, int NL, bool WT, int EZ, bool MASK>
__device__ __forceinline__ void chain_pair(KMember& m, KParam* prm, int tile)
{
    constexpr int HX = NL + 2, HY = NL + 1, R = kPairRows;
    constexpr int ne = EZ & 1, nz = EZ >> 1;
    const int nx = m.nx, ny = m.ny, walls = m.walls;
    const unsigned sN = (unsigned)m.N;
    const int tx = tile % m.pntx, ty = tile / m.pntx, lane = threadIdx.x;
    const int x0 = tx * m.pvx, xe = min(x0 + m.pvx, nx), y0 = ty * m.pvy, ye = min(y0 + m.pvy, ny);
    const int xc = modi(x0 - HX + lane, nx);
    const bool ownx = lane >= HX && lane - HX < xe - x0;
    const int ys = walls && ty == 0 ? 0 : y0 - HY;
    unsigned yo[R + 2], outm = 0;   // rows -1 .. R; bit r + 1: row r is beyond a wall
    {
        int yy = modi(ys - 1, ny);
#pragma unroll
        for (int r = 0; r < R + 2; ++r) {
            const int y = ys - 1 + r;
            const bool ok = !walls || (y >= 0 && y < ny);
            yo[r] = ok ? (unsigned)(yy * nx) : 0u;
            outm |= ok ? 0u : 1u << r;
            yy = yy + 1 == ny ? 0 : yy + 1;
        }
    }
    const T* vs = (const T*)m.vs;
    T a[R + 2], b[R];   // v_x of rows -1 .. R, v_y
#pragma unroll
    for (int r = 0; r < R + 2; ++r) a[r] = ld_at(vs, yo[r] + (unsigned)xc);
#pragma unroll
    for (int r = 0; r < R; ++r) b[r] = ld_at(vs + sN, yo[r + 1] + (unsigned)xc);
    // rows beyond the walls count as zero
    auto mask = [&](T* f, int first, int n) {
        if constexpr (MASK) {
#pragma unroll
            for (int r = 0; r < n; ++r) f[r] = (outm >> (first + r)) & 1 ? T(0) : f[r];
        }
    };
    mask(a, 0, R + 2);
    mask(b, 1, R);
    T w[R];
#pragma unroll
    for (int r = 0; r < R; ++r) w[r] = (lane_next(b[r]) - lane_prev(b[r])) - (a[r + 2] - a[r]);
    mask(w, 1, R);
    auto filter = [&](T (&f)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T t = f[r] + lane_prev(f[r]);
            f[r] = t + lane_next(t);
        }
        T s = f[0];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const T n = r + 1 < R ? f[r] + f[r + 1 < R ? r + 1 : r] : f[r];
            f[r] = s + n;
            s = n;
        }
        mask(f, 1, R);
    };
    // f -> R R f in place, its QoI density |R f|^2 summed over the own cells
    auto own_row = [&](int r) { return ys + r >= y0 && ys + r < ye; };
    auto chain = [&](T (&f)[R], int s, double& q) {
        T cr[3], crr[NL + 1], v[R], d[R];
#pragma unroll
        for (int j = 0; j < 3; ++j) cr[j] = chain_r<T>(prm, s, j);
#pragma unroll
        for (int j = 0; j <= NL; ++j) crr[j] = chain_rr<T>(prm, s, j);
#pragma unroll
        for (int r = 0; r < R; ++r) { v[r] = crr[0] * f[r]; d[r] = cr[0] * f[r]; }
#pragma unroll
        for (int j = 1; j <= NL; ++j) {
            filter(f);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[r] = fma_(crr[j], f[r], v[r]);
                if (j < 3) d[r] = fma_(cr[j < 3 ? j : 0], f[r], d[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f[r] = v[r];
            if (own_row(r) && ownx) q = __builtin_fma((double)d[r], (double)d[r], q);
        }
    };
    T* kV = (T*)m.kV;
    T ve[2][R];
#pragma unroll
    for (int r = 0; r < R; ++r) { ve[0][r] = a[r + 1]; ve[1][r] = b[r]; }
    double acc[5] = {0, 0, 0, 0, 0};   // q_E, q_Z, G_EE, G_EZ, G_ZZ
    if (ne) {   // uniform
        chain(ve[0], 0, acc[0]);
        chain(ve[1], 0, acc[0]);
    }
    if (nz) chain(w, ne, acc[1]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!own_row(r)) continue;   // uniform; an own row has its neighbours among the thread's rows
        const T wn = lane_next(w[r]), wp = lane_prev(w[r]);
        const T up = r + 1 < R ? w[r + 1 < R ? r + 1 : r] : T(0), dn = r > 0 ? w[r > 0 ? r - 1 : 0] : T(0);
        const T z0 = T(0.5) * (up - dn), z1 = -(T(0.5) * (wn - wp));
        if (!ownx) continue;
        const unsigned c = yo[r + 1] + (unsigned)xc;
        if (ne) {
            st_fld_at(kV, c, ve[0][r], WT);
            st_fld_at(kV + sN, c, ve[1][r], WT);
            acc[2] += (double)fma_(ve[0][r], ve[0][r], ve[1][r] * ve[1][r]);
        }
        if (nz) {
            st_fld_at(kV + (size_t)(2 * ne) * sN, c, z0, WT);
            st_fld_at(kV + (size_t)(2 * ne + 1) * sN, c, z1, WT);
            acc[4] += (double)fma_(z0, z0, z1 * z1);
        }
        if (ne && nz) acc[3] += (double)fma_(ve[0][r], z0, ve[1][r] * z1);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k] = wave_sum(acc[k]);
    if (lane == 0) {
        double* out = m.part_to + tile;
        const size_t n = (size_t)m.pnt;
        if (ne) out[0] = 0.5 * acc[0];
        if (nz) out[ne * n] = 0.5 * acc[1];
        const int g = ne + nz;
        if (ne) out[g * n] = acc[2];
        if (ne && nz) out[(g + 1) * n] = acc[3];
        if (nz) out[(ne ? g + 2 : g) * n] = acc[4];
    }
}

template <typename T, int NL, bool WT>
__global__ __launch_bounds__(64) void k_chain_pair(const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    KParam* prm = kc(m.prm);
    const int ez = prm->nk[0] + 2 * prm->nk[1];
#define LBM_EZ(MASK)                                                        \
    do {                                                                    \
        if (ez == 3) chain_pair<T, NL, WT, 3, MASK>(m, prm, wk.y);          \
        else if (ez == 2) chain_pair<T, NL, WT, 2, MASK>(m, prm, wk.y);     \
        else chain_pair<T, NL, WT, 1, MASK>(m, prm, wk.y);                  \
    } while (0)
    if (m.walls) LBM_EZ(true); else LBM_EZ(false);
#undef LBM_EZ
}

// ---------------------------------------------------------------------------
// K2c: per-cell sensitivities and Gram products, FP64 partial sums per
// workgroup.  Workgroups cover one y row (2-D) or one y plane (3-D) each, so
// the mean-profile partial sums stay separated by y.  V_s of an E QoI is read,
// that of a Z QoI formed as curl^T U_s and stored for the apply.  The QoI sums
// of binomial closures come from k_chain; KF, kernel-filter and Fourier
// closures: the QoIs are formed here as 1/2 <v*, V_s>.
// Partial layout: q_sa[nsa] (KF), G_sa[nsa(nsa+1)/2], then (with MP QoIs)
// U = sum v*_x and P_s = sum V_s,x.
// FP32, 3-D, three QoIs of each kind: 76 B in and 36 B out per cell; measured
// on MI355X 392 us on 384 x 192 x 192 (counters: 114 B in, the curl's
// neighbours missing the L2; 5.5 TB/s) and 11 us on 96 x 48 x 48 (436 and 14.5
// us with the powers of B as input).
// ---------------------------------------------------------------------------
// Waves per SIMD asked of the compiler (FP32): what a variant fits without
// spills.
template <typename T, int ME, int MZ, bool KF> constexpr int reduce_waves()
{
    if (sizeof(T) == 8 || (ME + MZ == 8 && MZ > 0)) return 1;
    return KF && (ME > 3 || MZ > 3) ? 3 : 4;
}
// ME, MZ: most E and Z QoIs of a member (its E QoIs come first, so that the
// loads of each kind have their own registers); ME = 0: MZ of either kind
// (uneven closures).
template <int LAT, typename T, int ME, int MZ, bool KF, bool WT>
__global__ __launch_bounds__(kBlock, (reduce_waves<T, ME, MZ, KF>())) void k_reduce(
    const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    using L = Lat<LAT>;
    constexpr int D = L::D, NC = L::NC;
    constexpr int MAXSA = ME + MZ, NG = MAXSA * (MAXSA + 1) / 2;
    constexpr int NQ = KF ? MAXSA : 0;
    constexpr int NV = NQ + NG + 1 + MAXSA;
    constexpr int NLD = D == 2 ? 4 : 12;                                  // loads of a curl
    constexpr int ZG = D == 3 && MZ == 6 ? 3 : (MZ == 0 ? 1 : MZ);       // Z positions loaded at a time
    __shared__ double lds[NV * (kBlock / 64)];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    KParam* prm = kc(m.prm);
    const int nx = m.nx, ny = m.ny, nz = m.nz;
    const int y = wk.y / m.nbx2, bx = wk.y % m.nbx2;
    const int plane = nx * nz;
    const int nsa = prm->nsa, ne = prm->nk[0];
    const bool hasmp = prm->nmp > 0;
    const unsigned sN = (unsigned)m.N;
    T* kV = (T*)m.kV;
    const int nz0 = ME > 0 ? ne : 0;   // QoI of the first Z position
    // QoI of position k of the accumulators; nsa or more: none
    auto qoi = [&](int k) { return k < ME ? (k < ne ? k : nsa) : nz0 + k - ME; };
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0;
    // one cell at a time, all its loads in flight before it is evaluated
    for (int c = 0; c < m.cpt2; ++c) {
        const int p = (bx * m.cpt2 + c) * kBlock + threadIdx.x;
        if (p >= plane) break;
        const int x = p % nx, z = p / nx;
        const unsigned cell = (unsigned)(x + nx * (y + ny * z));
        const Nbr n = nbr_at(cell, x, y, z, nx, ny, nz, m.walls, D);
        T V[MAXSA][D], v0[D], ld[ZG][NLD];
        if (KF) {
#pragma unroll
            for (int a = 0; a < D; ++a) v0[a] = ld_at((const T*)m.vs + (size_t)a * sN, cell);
        } else {
            v0[0] = hasmp ? ld_at((const T*)m.vs, cell) : T(0);
        }
        if constexpr (MZ <= ZG) {
#pragma unroll
            for (int s = 0; s < MZ; ++s) {
#pragma unroll
                for (int k = 0; k < NLD; ++k) ld[s][k] = 0;
                const int q = nz0 + s;   // (the branches are uniform)
                if (ME == 0 && q < ne) {
#pragma unroll
                    for (int a = 0; a < D; ++a) ld[s][a] = ld_at(kV + (size_t)(q * D + a) * sN, cell);
                } else if (q < nsa) {
                    curlT_load<D, T>((const T*)m.W + (size_t)q * NC * sN, sN, n, ld[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < ME; ++s)
#pragma unroll
                for (int a = 0; a < D; ++a) V[s][a] = s < ne ? ld_at(kV + (size_t)(s * D + a) * sN, cell) : T(0);
#pragma unroll
            for (int s = 0; s < MZ; ++s) {
                const int q = nz0 + s;
                if (ME == 0 && q < ne) {
#pragma unroll
                    for (int a = 0; a < D; ++a) V[s][a] = ld[s][a];
                    continue;
                }
                curlT_eval<D, T>(ld[s], n.okm, n.okp, V[ME + s]);
                if (q < nsa) {
#pragma unroll
                    for (int a = 0; a < D; ++a) st_fld_at(kV + (size_t)(q * D + a) * sN, cell, V[ME + s][a], WT);
                }
            }
        } else {
            // ZG positions at a time, within the registers of ld
            static_assert(ME == 0, "grouped positions hold either kind");
#pragma unroll
            for (int s0 = 0; s0 < MZ; s0 += ZG) {
#pragma unroll
                for (int k = 0; k < ZG; ++k) {
                    const int q = s0 + k;
                    if (q >= MZ) continue;
#pragma unroll
                    for (int j = 0; j < NLD; ++j) ld[k][j] = 0;
                    if (q < ne) {
#pragma unroll
                        for (int a = 0; a < D; ++a) ld[k][a] = ld_at(kV + (size_t)(q * D + a) * sN, cell);
                    } else if (q < nsa) {
                        curlT_load<D, T>((const T*)m.W + (size_t)q * NC * sN, sN, n, ld[k]);
                    }
                }
#pragma unroll
                for (int k = 0; k < ZG; ++k) {
                    const int q = s0 + k;
                    if (q >= MZ) continue;
                    if (q < ne) {
#pragma unroll
                        for (int a = 0; a < D; ++a) V[q][a] = ld[k][a];
                        continue;
                    }
                    curlT_eval<D, T>(ld[k], n.okm, n.okp, V[q]);
                    if (q < nsa) {
#pragma unroll
                        for (int a = 0; a < D; ++a) st_fld_at(kV + (size_t)(q * D + a) * sN, cell, V[q][a], WT);
                    }
                }
            }
        }
        if constexpr (KF) {
#pragma unroll
            for (int s = 0; s < MAXSA; ++s) {
                double qd = 0;
#pragma unroll
                for (int a = 0; a < D; ++a) qd += 0.5 * (double)(v0[a] * V[s][a]);
                acc[s] += qd;
            }
        }
        // (multiply-adds by hand, so that every variant rounds alike: a batch may
        // take another one than a member alone)
        int g = 0;
#pragma unroll
        for (int s = 0; s < MAXSA; ++s) {
            T d = fma_(V[s][0], V[s][0], V[s][1] * V[s][1]);
            if (D == 3) d = fma_(V[s][D - 1], V[s][D - 1], d);
            acc[NQ + g++] += (double)d;
#pragma unroll
            for (int t2 = s + 1; t2 < MAXSA; ++t2, ++g) {
                d = V[s][0] * V[t2][0];
#pragma unroll
                for (int a = 1; a < D; ++a) d = fma_(V[s][a], V[t2][a], d);
                acc[NQ + g] += (double)d;
            }
        }
        if (hasmp) {
            acc[NQ + NG] += (double)v0[0];
#pragma unroll
            for (int s = 0; s < MAXSA; ++s) acc[NQ + NG + 1 + s] += (double)V[s][0];
        }
    }
    // band weights w_j(y) of this row (workgroup-uniform: scalar loads,
    // issued before the reduction so that their latency is hidden)
    double wb[kMaxQ];
    const int nmp = prm->nmp;
    if (hasmp) {
        const LBM_K double* bw = kc(m.bandw);
#pragma unroll
        for (int jm = 0; jm < kMaxQ; ++jm) wb[jm] = bw[(size_t)prm->mp_band[jm < nmp ? jm : nmp - 1] * ny + y];
    }
    // partials are stored value-major, [npart][ny * nbx2], so that the
    // cross-block sums read them contiguously; thread t writes value t
    const double r = block_sum_spread<NV>(acc, lds);
    const int t = threadIdx.x;
    const size_t nblk = (size_t)ny * m.nbx2;
    double* out = m.part_to + wk.y;
    if (t < NQ) {
        const int q = qoi(t);
        if (q < nsa) out[q * nblk] = r;
    } else if (t < NQ + NG) {
        int g = t - NQ, k = 0;   // positions (k, k + g), in the order of acc
        while (g >= MAXSA - k) { g -= MAXSA - k; ++k; }
        const int sa = qoi(k), t2 = qoi(k + g);
        if (sa < nsa && t2 < nsa) out[(nsa + sa * nsa - sa * (sa - 1) / 2 + (t2 - sa)) * nblk] = r;
    } else if (hasmp && t < NV) {
        // mean-profile terms, weighted by the band weights of this row:
        // w_j(y) sum v*_x (column 0) and w_j(y) sum V_s,x (column 1 + s)
        const int k = t - (NQ + NG), col = k == 0 ? 0 : 1 + qoi(k - 1);
        if (col <= nsa) {
            const int o = nsa + nsa * (nsa + 1) / 2;
#pragma unroll
            for (int jm = 0; jm < kMaxQ; ++jm)
                if (jm < nmp) out[(o + jm * (1 + nsa) + col) * nblk] = wb[jm] * r;
        }
    }
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and Box-Muller normals.
// Counter (block, step_lo, step_hi, "LRS1"), key (seed_lo, seed_hi).
// ---------------------------------------------------------------------------
__device__ inline void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
        const uint32_t lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// The four normals of Philox block blk of a step: Box-Muller on the block's
// two pairs of uniforms.
__device__ inline void lrs_block_normals(unsigned long long seed, long long step, int blk, double* zz)
{
    uint32_t c[4] = {(uint32_t)blk, (uint32_t)(unsigned long long)step,
                     (uint32_t)((unsigned long long)step >> 32), 0x4C525331u};
    philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    for (int p = 0; p < 2; ++p) {
        const double u1 = ((double)c[2 * p] + 0.5) * 2.3283064365386963e-10;
        const double u2 = ((double)c[2 * p + 1] + 0.5) * 2.3283064365386963e-10;
        const double rad = sqrt(-2.0 * log(u1));
        double sn, cs;
        sincospi(2.0 * u2, &sn, &cs);
        zz[2 * p] = rad * cs;
        zz[2 * p + 1] = rad * sn;
    }
}

__device__ inline void lrs_normals(unsigned long long seed, long long step, int n, double* z)
{
    for (int blk = 0; 4 * blk < n; ++blk) {
        double zz[4];
        lrs_block_normals(seed, step, blk, zz);
        for (int k = 0; k < 4; ++k)
            if (4 * blk + k < n) z[4 * blk + k] = zz[k];
    }
}

static __global__ void k_philox_test(const uint32_t* in, uint32_t* out, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c[4] = {in[6 * i], in[6 * i + 1], in[6 * i + 2], in[6 * i + 3]};
    philox4x32_10(c, in[6 * i + 4], in[6 * i + 5]);
    for (int k = 0; k < 4; ++k) out[4 * i + k] = c[k];
}

static __global__ void k_normals_test(unsigned long long seed, long long step0, int nsteps, int n, double* out)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsteps) return;
    double z[kMaxQ];
    lrs_normals(seed, step0 + s, n, z);
    for (int k = 0; k < n; ++k) out[(size_t)s * n + k] = z[k];
}

// ---------------------------------------------------------------------------
// K2d: cross-block sums, one workgroup per (member, value slot).  Slots 0..3
// sum the statistics of the stream-collide workgroups, slots 4.. the TO
// partials of the reduce workgroups; the order is fixed by the member's own
// block counts.  Slot -1 makes the member's LRS draw of the step, slots
// -2 - c chunk c of the product of the LRS history with its rows of C.
// ---------------------------------------------------------------------------
static __global__ __launch_bounds__(kBlock) void k_sum(const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    __shared__ double red[kBlock / 64];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int slot = wk.y;
    if (slot == -1) {
        // the member's LRS draw for this step, off the solve's critical
        // path: normals xi (four per Philox block), then e = mu + L xi
        __shared__ double z[kMaxQ];
        KParam* prm = kc(m.prm);
        DevCtl* ctl = m.ctl;
        const long long step = ctl->step;
        if (prm->mode != LBM_CLOSURE_LRS || step < prm->spinup) return;   // uniform
        const int nq = prm->nq, tid = threadIdx.x;
        if (tid < (nq + 3) / 4) {
            double zz[4];
            lrs_block_normals(prm->seed, step, tid, zz);
            for (int k = 0; k < 4; ++k)
                if (4 * tid + k < nq) z[4 * tid + k] = zz[k];
        }
        __syncthreads();
        if (tid < nq) {
            double e = prm->mu[tid];
            for (int j = 0; j <= tid; ++j) e += prm->L[tid * kMaxQ + j] * z[j];
            ctl->lrs_e[tid] = e;
        }
        return;
    }
    if (slot < -1) {
        // history chunk c of the LRS product: sum over the x entries r in
        // [c kHistRows, (c+1) kHistRows) of x_r C[r][k], where x runs over
        // z^{n-1..n-h} then z*^{n-1..n-h} (z = q / s) from the record ring
        __shared__ double lds[kMaxQ * (kBlock / 64)];
        KParam* prm = kc(m.prm);
        DevCtl* ctl = m.ctl;
        const long long step = ctl->step;
        const int c = -2 - slot;
        if (prm->mode != LBM_CLOSURE_LRS || prm->h == 0 || c >= prm->nhc || step < prm->spinup) return;   // uniform
        const int nq = prm->nq, h = prm->h, rows = 2 * h * nq;
        double acc[kMaxQ];
#pragma unroll
        for (int k = 0; k < kMaxQ; ++k) acc[k] = 0.0;
#pragma unroll
        for (int u = 0; u < kHistRows / kBlock; ++u) {
            const int r = c * kHistRows + u * kBlock + threadIdx.x;
            if (r < rows) {
                const int b = r / nq, i = r % nq;
                const bool corr = b < h;                       // z^{n-1-b}, else z*^{n-1-(b-h)}
                const long long mstep = step - 1 - (corr ? b : b - h);
                const lbm_qoi_rec* rec = m.recs + (size_t)(mstep % m.rec_cap);
                double qv = rec->q[i];
                if (corr && !(rec->flags & 2)) qv += rec->dq[i];
                const double x = qv / prm->scale[i];
                const double* crow = prm->chist + (size_t)r * nq;
#pragma unroll
                for (int k = 0; k < kMaxQ; ++k)
                    if (k < nq) acc[k] += x * crow[k];
            }
        }
        const double v = block_sum_spread<kMaxQ>(acc, lds);
        if (threadIdx.x < nq) m.hpart[c * kMaxQ + threadIdx.x] = v;
        return;
    }
    if (slot >= 4 + m.npart) return;
    if (slot == 0 && threadIdx.x == 0) {
        // the step this launch belongs to, for a fused apply, and a first LRS
        // scale that the last fused apply left pending
        DevCtl* ctl = m.ctl;
        ctl->step_snap = ctl->step;
        if (ctl->s_pend) {
            for (int k = 0; k < kMaxQ; ++k) ctl->s[k] = ctl->s_next[k];
            ctl->s_set = 1;
            ctl->s_pend = 0;
        }
    }
    double v[1] = {0};
    if (slot < 4) {
#pragma unroll 8
        for (int b = threadIdx.x; b < m.nst; b += kBlock) v[0] += m.part_stats[(size_t)b * 4 + slot];
    } else {
        // the QoI sums of binomial closures are k_chain's, the others k_reduce's
        KParam* prm = kc(m.prm);
        const int s = slot - 4;
        const bool chain = s < prm->nsa && !prm->kf && !m.pair;
        const int nblk = chain ? m.cnt * (prm->sa_kind[s] == 0 ? m.cd : m.cnc) : m.pair ? m.pnt : m.ny * m.nbx2;
        const double* p = chain ? m.part_q + (size_t)s * m.cnt * m.cd : m.part_to + (size_t)s * nblk;
#pragma unroll 8
        for (int b = threadIdx.x; b < nblk; b += kBlock) v[0] += p[b];
    }
    block_sum<1>(v, red);
    if (threadIdx.x == 0) m.sums[slot] = v[0];
}

// ---------------------------------------------------------------------------
// K3: the member's solve.  The QoI vector and Gram matrix from the
// fixed-order sums (k_sum), dQ, beta = G^-1 dQ and gamma_k = dQ_k (G^-1)_kk,
// the per-step record and the coefficients of the dv build.  Every input is
// first staged into LDS in one parallel pass, and all small matrices live
// there.  G is symmetric positive semi-definite, so Gauss-Jordan elimination
// needs no pivoting; its pivots are the squared Cholesky pivots, and G counts
// as singular when one of them is not above 1e-14 times the largest diagonal
// entry.  The elimination takes four pivots per barrier, ping-ponging between
// two copies of [G | I].
//
// It runs in one of two places.  k_solve: one workgroup per member, writing
// the coefficients, the record and the control state for k_apply.  Or in
// every workgroup of the apply k_apply_fs (small launches), with
// the apply's own field loads in flight meanwhile, each workgroup forming
// the same coefficients from the same sums with the same arithmetic; there
// the member's first workgroup alone writes the record, advances the step
// counter and leaves a first LRS scale to be committed by the next step's
// k_sum, and every workgroup takes the step from the snapshot k_sum made of
// it, so no workgroup reads a value another one of the launch writes.
// ---------------------------------------------------------------------------
constexpr int kMaxSums = 4 + kMaxSA + kMaxSA * (kMaxSA + 1) / 2 + kMaxQ * (1 + kMaxSA);

struct SolveLds {
    double M[2][kMaxQ][2 * kMaxQ];
    double sf[kMaxSums];
    double Cs[(kMaxQ + 1) * kMaxQ], es[kMaxQ], hps[kMaxHistChunks * kMaxQ];
    double q[kMaxQ], dq[kMaxQ], beta[kMaxQ], gam[kMaxQ], sc[kMaxQ], qs[kMaxQ];
    double gmps[kMaxQ * kMaxQ];
    int saslot[kMaxSA], mpslot[kMaxQ], mpband[kMaxQ];
    long long step;
    int sset, flags;
};

// ROLE 0: k_solve (every output, the step counter from ctl->step); 1: the
// leader of a fused apply (the record, the step counter, a pending scale);
// 2: another workgroup of a fused apply (LDS outputs only).  Every thread of
// the workgroup calls it; pre() issues the caller's loads right after the
// solve's own; S.beta holds the result.
template <int NTH, int ROLE, typename Pre>
__device__ void solve_member(KMember& m, SolveLds& S, Pre&& pre)
{
    static_assert(NTH == kBlock, "the solve runs on a whole workgroup");
    KParam* prm = kc(m.prm);
    DevCtl* ctl = m.ctl;
    const int tid = threadIdx.x;
    const int nq = prm->nq, nsa = prm->nsa, nmp = prm->nmp;
    const int ny = m.ny;
    const int nflat = nsa + nsa * (nsa + 1) / 2;
    const bool lrs = prm->mode == LBM_CLOSURE_LRS;

    // (a) stage the sums, the LRS model and the control state; clear M.
    // Every load's address and count come from the member record itself or
    // are fixed, none from a value loaded from the closure parameters, so
    // all of them are in flight after one dependent load.  They are issued
    // first, then the caller's own loads (pre), then stored to LDS: a wave's
    // loads complete in order, so the stores wait only for the solve's own.
    // (Measured on MI355X: the caller's loads issued after the staging
    // barrier instead are no faster.)
    static_assert(kMaxSums <= kBlock && kMaxQ * kMaxQ <= kBlock &&
                  (kMaxQ + 1) * kMaxQ <= 2 * kBlock, "one or two staged values per thread");
    const double r_sf = tid < 4 + m.npart ? m.sums[tid] : 0.0;   // 4 + npart sums
    const double r_c0 = prm->C[tid];
    const double r_c1 = tid < (kMaxQ + 1) * kMaxQ - kBlock ? prm->C[kBlock + tid] : 0.0;
    const double r_g = prm->gmp[tid];
    double r_es = 0, r_s = 0;
    int r_sas = 0, r_mps = 0, r_mpb = 0;
    if (tid < kMaxQ) {
        r_es = ctl->lrs_e[tid];
        r_s = ctl->s[tid];
        r_mps = prm->mp_slot[tid];
        r_mpb = prm->mp_band[tid];
    }
    if (tid < kMaxSA) r_sas = prm->sa_slot[tid];
    long long r_step = 0;
    int r_sset = 0, r_flags = 0;
    if (tid == 0) {
        r_step = ROLE == 0 ? ctl->step : ctl->step_snap;
        r_sset = ctl->s_set;
        r_flags = ctl->flags;
    }
    pre();
    if (tid < 4 + m.npart) S.sf[tid] = r_sf;
    S.Cs[tid] = r_c0;
    if (tid < (kMaxQ + 1) * kMaxQ - kBlock) S.Cs[kBlock + tid] = r_c1;
    S.gmps[tid] = r_g;
    if (tid < kMaxQ) {
        S.es[tid] = r_es;
        S.sc[tid] = r_s;
        S.mpslot[tid] = r_mps;
        S.mpband[tid] = r_mpb;
        S.q[tid] = 0; S.dq[tid] = 0; S.beta[tid] = 0; S.gam[tid] = 0;
    }
    if (tid < kMaxSA) S.saslot[tid] = r_sas;
    if (tid == 0) {
        S.step = r_step;
        S.sset = r_sset;
        S.flags = r_flags;
    }
    if (lrs)
        for (int k = tid; k < prm->nhc * kMaxQ; k += NTH) S.hps[k] = m.hpart[k];
    for (int k = tid; k < 2 * kMaxQ * 2 * kMaxQ; k += NTH) (&S.M[0][0][0])[k] = 0.0;
    // band weights of row y = tid, used at the end (clamped index; loaded now
    // so that their latency overlaps the solve)
    double wv0[kMaxQ];
    if (ROLE == 0 && nmp > 0 && tid < ny) {
#pragma unroll
        for (int jm = 0; jm < kMaxQ; ++jm) wv0[jm] = m.bandw[(size_t)prm->mp_band[jm < nmp ? jm : nmp - 1] * ny + tid];
    }
    __syncthreads();
    const long long step = S.step;
    const bool active = step >= prm->spinup;
    // (b) assemble q and G (left half of M), the mean-profile entries and
    // the identity (right half)
    const double* sfp = S.sf + 4;
    if (tid < nsa) {
        const int s = tid;
        S.q[S.saslot[s]] = sfp[s];
        int g = nsa + s * nsa - s * (s - 1) / 2;
        for (int t = s; t < nsa; ++t, ++g) {
            S.M[0][S.saslot[s]][S.saslot[t]] = sfp[g];
            S.M[0][S.saslot[t]][S.saslot[s]] = sfp[g];
        }
    }
    for (int pr = tid; pr < nmp * (1 + nsa); pr += NTH) {
        const int jm = pr / (1 + nsa), c = pr % (1 + nsa);
        const double v = sfp[nflat + pr];
        const int uj = S.mpslot[jm];
        if (c == 0)
            S.q[uj] = v;
        else {
            const int us = S.saslot[c - 1];
            S.M[0][uj][us] = v;
            S.M[0][us][uj] = v;
        }
    }
    for (int pr = tid; pr < nmp * nmp; pr += NTH) {
        const int a = pr / nmp, b = pr % nmp;
        S.M[0][S.mpslot[a]][S.mpslot[b]] = S.gmps[a * kMaxQ + b];
    }
    if (tid < nq) S.M[0][tid][kMaxQ + tid] = 1.0;
    __syncthreads();
    // (c) dQ for tracking; the LRS scale (fixed at the first active step)
    if (active && tid < nq) {
        const int k = tid;
        if (prm->mode == LBM_CLOSURE_TRACK) {
            if (step < prm->nref) S.dq[k] = prm->qref[(size_t)step * nq + k] - S.q[k];
        } else if (lrs) {
            if (!S.sset) {
                S.sc[k] = prm->have_scale ? prm->scale[k] : (S.q[k] != 0.0 ? fabs(S.q[k]) : 1.0);
                if (ROLE == 0) ctl->s[k] = S.sc[k];
                if (ROLE == 1) ctl->s_next[k] = S.sc[k];
            }
            S.qs[k] = S.q[k] / S.sc[k];
        }
    }
    __syncthreads();
    // (d) the LRS draw: dQ = s (x C + e) - q*, with e = mu + L xi and the
    // history part of x C formed ahead of this kernel (k_sum); terms past nq
    // add exact zeros
    if (active && lrs && tid < nq) {
        const int k = tid;
        double zh = S.es[k];
        for (int c = 0; c < prm->nhc; ++c) zh += S.hps[c * kMaxQ + k];
#pragma unroll
        for (int i = 0; i < kMaxQ; ++i) {
            const int ic = i < nq ? i : 0;
            const double t = S.qs[ic] * S.Cs[ic * kMaxQ + k];
            zh += i < nq ? t : 0.0;
        }
        zh += S.Cs[nq * kMaxQ + k];
        S.dq[k] = S.sc[k] * zh - S.q[k];
    }
    // (e) Gauss-Jordan on [G | I] (only columns 0..nq-1 and kMaxQ..kMaxQ+nq-1
    // are nonzero), four pivots per barrier.  For pivot rows j0..j0+3 every
    // thread eliminates the 4x4 pivot block P in registers, applied to its
    // column's pivot-row entries r (t = P^-1 r, pivots in order, each checked
    // against the singular threshold; the block is identity-padded past nq),
    // then row i of its column becomes t_(i-j0) inside the block and
    // M[i][c] - sum_a M[i][j0+a] t_a outside it.  Every thread computes the
    // same pivots from the same values, so the singular flag is uniform.
    // The four eliminations of a block are those of four consecutive pivots.
    double mx = 0;
    for (int k = 0; k < nq; ++k) mx = fmax(mx, S.M[0][k][k]);
    int sing = mx > 0 ? 0 : 1;
    int cur = 0;
    // thread layout: one column of [G | I] each, rows split over the
    // NTH / (2 nq) groups of threads
    const int ncol = 2 * nq, ngrp = NTH / ncol;
    const int gcol = tid % ncol, grow = tid / ncol;
    const int cc = gcol < nq ? gcol : kMaxQ + gcol - nq;
    __syncthreads();
    for (int j0 = 0; j0 < nq && !sing; j0 += 4) {
        const int bs = min(4, nq - j0);   // rows j0..j0+3 stay inside M (nq <= kMaxQ)
        double P[4][4], t[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int b2 = 0; b2 < 4; ++b2) P[a][b2] = a < bs && b2 < bs ? S.M[cur][j0 + a][j0 + b2] : (a == b2 ? 1.0 : 0.0);
            t[a] = a < bs ? S.M[cur][j0 + a][cc] : 0.0;
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const double piv = P[a][a];
            if (a < bs && !(piv > 1e-14 * mx)) sing = 1;
            const double rp = 1.0 / piv;
#pragma unroll
            for (int b2 = a + 1; b2 < 4; ++b2) P[a][b2] *= rp;
            t[a] *= rp;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (e == a) continue;
                const double f = P[e][a];
#pragma unroll
                for (int b2 = a + 1; b2 < 4; ++b2) P[e][b2] -= f * P[a][b2];
                t[e] -= f * t[a];
            }
        }
        if (sing) break;   // uniform
        if (grow < ngrp) {
            for (int i = grow; i < nq; i += ngrp) {
                const int d = i - j0;
                double v;
                if (d >= 0 && d < bs) {
                    v = d == 0 ? t[0] : d == 1 ? t[1] : d == 2 ? t[2] : t[3];
                } else {
                    // past nq the block columns of M are zero and t is zero
                    v = S.M[cur][i][cc];
#pragma unroll
                    for (int a = 0; a < 4; ++a) v -= S.M[cur][i][j0 + a] * t[a];
                }
                S.M[cur ^ 1][i][cc] = v;
            }
        }
        cur ^= 1;
        __syncthreads();
    }
    // (f) beta = G^-1 dQ, gamma_k = dQ_k (G^-1)_kk
    if (!sing && tid < nq) {
        double b = 0;
        for (int j = 0; j < nq; ++j) b += S.M[cur][tid][kMaxQ + j] * S.dq[j];
        S.beta[tid] = b;
        S.gam[tid] = S.dq[tid] * S.M[cur][tid][kMaxQ + tid];
    }
    __syncthreads();
    // (g) beta of the sensitivities, record, counters
    if (ROLE == 0 && tid < kMaxSA) {
        const double b = tid < nsa ? S.beta[S.saslot[tid]] : 0.0;
        ctl->bsa[tid] = b;
        ctl->bsaf[tid] = (float)b;
    }
    if (ROLE <= 1) {
        lbm_qoi_rec* rec = m.recs + (size_t)(step % m.rec_cap);
        if (tid < kMaxQ) {
            rec->q[tid] = tid < nq ? S.q[tid] : 0.0;
            rec->dq[tid] = tid < nq ? S.dq[tid] : 0.0;
            rec->gamma[tid] = tid < nq ? S.gam[tid] : 0.0;
        }
        if (tid == 0) {
            rec->step = step;
            rec->flags = (S.flags & 1) | (sing ? 2 : 0);
            rec->nq = nq;
            rec->mass = (double)m.N + S.sf[0];
            rec->mom[0] = S.sf[1];
            rec->mom[1] = S.sf[2];
            rec->mom[2] = S.sf[3];
            rec->diag_e = 0;
            rec->diag_z = 0;
            if (active && lrs && !S.sset) {
                if (ROLE == 0) ctl->s_set = 1;
                else ctl->s_pend = 1;
            }
            ctl->step = step + 1;
        }
    }
    // (h) mean-profile part of dv: cmp(y) = sum_j beta_mp_j w_j(y) (in a
    // fused apply every cell forms its own row's value)
    if (ROLE == 0) {
        if (nmp > 0) {
            for (int yy = tid; yy < ny; yy += NTH) {
                // all band-weight loads first (clamped index; terms past nmp add exact zeros)
                double wv[kMaxQ];
#pragma unroll
                for (int jm = 0; jm < kMaxQ; ++jm)
                    wv[jm] = yy == tid ? wv0[jm] : m.bandw[(size_t)S.mpband[jm < nmp ? jm : nmp - 1] * ny + yy];
                double c = 0;
#pragma unroll
                for (int jm = 0; jm < kMaxQ; ++jm) c += jm < nmp ? S.beta[S.mpslot[jm]] * wv[jm] : 0.0;
                m.cmp[yy] = c;
            }
        } else {
            for (int yy = tid; yy < ny; yy += NTH) m.cmp[yy] = 0.0;
        }
    }
}

static __global__ __launch_bounds__(kBlock) void k_solve(const DevMember* __restrict__ mems, const int* __restrict__ work)
{
    __shared__ SolveLds S;
    KMember& m = *kc(mems + work[blockIdx.x]);
    solve_member<kBlock, 0>(m, S, [] {});
}

// K4: dv = sum_s beta_s V_s + e_x cmp(y) (eq. TO-ansatz as sum_i beta_i V_i),
// and the SGS change of the cell's predictor populations
// delta f_i = feq_i(rho, v* + dv) - feq_i(rho, v*): DEF, the record
// (a, b) = (rho dv, 2 v* + dv) that the next stream-collide applies during
// its pull; otherwise added in place to the populations the stream-collide of
// this step wrote (small grids, and the WALE substrate, whose velocity
// gradients need the complete post-streaming state).
template <typename T> __device__ __forceinline__ T coef_bsa(KCtl* c, int s);
template <> __device__ __forceinline__ float coef_bsa<float>(KCtl* c, int s) { return c->bsaf[s]; }
template <> __device__ __forceinline__ double coef_bsa<double>(KCtl* c, int s) { return c->bsa[s]; }

// One cell of the apply: its fields (the sensitivities of QoIs past nsa are
// zero) and, in place, the populations the stream-collide of this step wrote.
template <int LAT, typename T, int MAXSA, bool DEF>
struct ApplyIn {
    T vs[Lat<LAT>::D], V[MAXSA][Lat<LAT>::D];
    T rho1;                            // rho - 1
    T gi[DEF ? 1 : Lat<LAT>::Q];
};

template <int LAT, typename T, int MAXSA, bool WT, bool DEF>
__device__ __forceinline__ void apply_load(KMember& m, KParam* prm, int flip, int cell, ApplyIn<LAT, T, MAXSA, DEF>& in)
{
    using L = Lat<LAT>;
    constexpr int D = L::D;
    const size_t sN = (size_t)m.N;
    const int nsa = prm->nsa;
    const T* __restrict__ kV = (const T*)m.kV;
    if constexpr (!DEF) {
        const T* g = (const T*)m.g[m.parity ^ flip ^ 1];
#pragma unroll
        for (int i = 0; i < L::Q; ++i) in.gi[i] = ld_fld<WT>(g + pop_at64<L::Q>(i, (size_t)cell));
    }
#pragma unroll
    for (int a = 0; a < D; ++a) in.vs[a] = ld_fld<WT>((const T*)m.vs + a * sN + cell);
#pragma unroll
    for (int s = 0; s < MAXSA; ++s)
#pragma unroll
        for (int a = 0; a < D; ++a) in.V[s][a] = s < nsa ? ld_fld<WT>(kV + (size_t)(s * D + a) * sN + cell) : T(0);
    in.rho1 = ((const T*)m.rho)[cell];
}

// The rest of the cell: dv from the coefficients beta, and the SGS change
// (rho dv, 2 v* + dv), stored as the record (DEF) or added in place to the
// populations.
template <int LAT, typename T, int MAXSA, bool WT, bool DEF>
__device__ __forceinline__ void apply_finish(KMember& m, int flip, int cell, const ApplyIn<LAT, T, MAXSA, DEF>& in,
                                             const T (&beta)[MAXSA], bool hasmp, double cmp)
{
    using L = Lat<LAT>;
    constexpr int D = L::D;
    const size_t sN = (size_t)m.N;
    T out[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        T acc = 0;
#pragma unroll
        for (int s = 0; s < MAXSA; ++s) acc = fma_(beta[s], in.V[s][a], acc);
        out[a] = acc;
    }
    if (hasmp) out[0] += T(cmp);
    const T rho = T(1) + in.rho1;
    T ra[D], rb[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        ra[a] = rho * out[a];
        rb[a] = T(2) * in.vs[a] + out[a];
    }
    // (TO fields stay below 2^32 bytes: 32-bit offsets from scalar bases)
    if constexpr (DEF) {
        T* rec = (T*)m.rec;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            st_fld_at(rec + (size_t)a * sN, (unsigned)cell, ra[a], WT);
            st_fld_at(rec + (size_t)(D + a) * sN, (unsigned)cell, rb[a], WT);
        }
    } else {
        T* g = (T*)m.g[m.parity ^ flip ^ 1];
        const T e = rec_e<D, T>(ra, rb);
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
            st_fld(g + pop_at64<L::Q>(i, (size_t)cell),
                   add_df<LAT, T>(in.gi[i], i, [&](int k) { return ra[k]; }, [&](int k) { return rb[k]; }, e), WT);
    }
}

template <int LAT, typename T, int MAXSA, bool WT, bool DEF>
__global__ __launch_bounds__(kBlock) void k_apply(const DevMember* __restrict__ mems, const int2* __restrict__ work,
                                                  int flip)
{
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    KParam* prm = kc(m.prm);
    const int cell = wk.y * kBlock + threadIdx.x;
    if (cell >= m.N) return;
    KCtl* ctl = kc(m.ctl);
    ApplyIn<LAT, T, MAXSA, DEF> in;
    apply_load<LAT, T, MAXSA, WT, DEF>(m, prm, flip, cell, in);
    T beta[MAXSA];
#pragma unroll
    for (int s = 0; s < MAXSA; ++s) beta[s] = coef_bsa<T>(ctl, s);   // zero past nsa
    const bool hasmp = prm->nmp > 0;
    apply_finish<LAT, T, MAXSA, WT, DEF>(m, flip, cell, in, beta, hasmp, hasmp ? m.cmp[(cell / m.nx) % m.ny] : 0.0);
}

// The apply with the member's solve at its head (launches of at most
// kFusedApplyPairs workgroups).  A workgroup takes a pair of
// blocks of one member (work entry (member, p): blocks 2p and 2p + 1), issues
// the loads of both cells of every thread, then solves on all its threads
// while they are in flight (two waves per SIMD: every workgroup of the launch
// is resident at once), and finishes both cells with the solve's
// coefficients; cmp(y) = sum_j beta_mp_j w_j(y) is formed per cell in the
// order and precision k_solve forms it.  Pair 0 is the member's leader.
template <int LAT, typename T, int MAXSA, bool WT, bool DEF>
__global__ __launch_bounds__(kBlock, 2) void k_apply_fs(const DevMember* __restrict__ mems,
                                                         const int2* __restrict__ work, int flip)
{
    __shared__ SolveLds S;
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    KParam* prm = kc(m.prm);
    const int N = m.N, nx = m.nx, ny = m.ny;
    const int nmp = prm->nmp, nsa = prm->nsa;
    int cells[2];
    bool own[2];
    ApplyIn<LAT, T, MAXSA, DEF> in[2];
    double wv[2][kMaxQ];
    // the cells' loads, issued right after the solve's own
    auto load = [&] {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = (2 * wk.y + u) * kBlock + threadIdx.x;
            own[u] = c < N;
            cells[u] = own[u] ? c : 0;   // a thread past the grid loads cell 0 and stores nothing
            apply_load<LAT, T, MAXSA, WT, DEF>(m, prm, flip, cells[u], in[u]);
            const int y = (cells[u] / nx) % ny;
            if (nmp > 0) {
#pragma unroll
                for (int jm = 0; jm < kMaxQ; ++jm)
                    wv[u][jm] = jm < nmp ? m.bandw[(size_t)prm->mp_band[jm] * ny + y] : 0.0;
            }
        }
    };
    if (wk.y == 0) solve_member<kBlock, 1>(m, S, load);
    else solve_member<kBlock, 2>(m, S, load);
    T beta[MAXSA];   // (S.beta is complete at the solve's last barrier)
#pragma unroll
    for (int s = 0; s < MAXSA; ++s) beta[s] = s < nsa ? T(S.beta[S.saslot[s]]) : T(0);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (!own[u]) continue;
        double cmp = 0;
        if (nmp > 0) {
#pragma unroll
            for (int jm = 0; jm < kMaxQ; ++jm) cmp += jm < nmp ? S.beta[S.mpslot[jm]] * wv[u][jm] : 0.0;
        }
        apply_finish<LAT, T, MAXSA, WT, DEF>(m, flip, cells[u], in[u], beta, nmp > 0, cmp);
    }
}

// A pending SGS change (the records of the last step) added in place to the
// current populations g[parity ^ flip], and the records cleared, so the state
// can be read or replaced (checkpoints, fields, a closure change).
template <int LAT, typename T>
__global__ __launch_bounds__(kBlock) void k_flush(const DevMember* __restrict__ mems, const int2* __restrict__ work,
                                                  int flip)
{
    using L = Lat<LAT>;
    constexpr int D = L::D;
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int N = m.N;
    const int cell = wk.y * kBlock + threadIdx.x;
    if (cell >= N) return;
    const size_t sN = (size_t)N;
    T* rec = (T*)m.rec;
    T ra[D], rb[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        ra[a] = rec[a * sN + cell];
        rb[a] = rec[(D + a) * sN + cell];
    }
    const T e = rec_e<D, T>(ra, rb);
    T* g = (T*)m.g[m.parity ^ flip];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        g[pop_at64<L::Q>(i, (size_t)cell)] = add_df<LAT, T>(g[pop_at64<L::Q>(i, (size_t)cell)], i,
                                                             [&](int k) { return ra[k]; },
                                                             [&](int k) { return rb[k]; }, e);
#pragma unroll
    for (int a = 0; a < 2 * D; ++a) rec[a * sN + cell] = T(0);
}

// ---------------------------------------------------------------------------
// Kernel filters (Sec. 4.1, eq. gaussian and eq. laplace) as separable
// passes: G_s = g (x) g (x) g; L_s = sum over the axes a of the dilated
// biharmonic l along a and boxes b of width s across a, gathered by the z part:
//   L_s f = b_z (b_y l_x f + l_y b_x f) + l_z (b_y b_x f)        (2-D: the
//   first bracket alone).
// k_kxy forms the x and y parts of one QoI's filter on 64 x 16 tiles staged in
// LDS with the filter's halo, k_kz the z parts and the sum, each thread eight
// planes of a cell column from one window in registers; R R takes the pair
// twice.  One launch of each per application serves all QoIs and components
// (job blockIdx.y).  Periodic wrap, zero padding on the wall axis at every
// pass.  Radii are template parameters (a branch on the job's, uniform), so
// the windows live in registers and the taps in scalar registers; outputs are
// formed four (k_kxy) and eight (k_kz) at a time, which divides the loads per
// output by as many.  Bound by the traffic of the intermediates, 830 B per
// cell for the paper's 3-D set where one 1-D pass per launch level and term
// moved 1900; measured on MI355X, 295 x 47 x 98, FP32: seven launches of 129 us ->
// 98 (k_kxy, half of it vector instructions) and 53 us (k_kz, 4.9 TB/s), twice
// each.  (A wavefront staging whole rows, without the index divisions, has
// fewer loads in flight: 109 us.)
// ---------------------------------------------------------------------------
constexpr int kFilTX = 64, kFilTY = 16, kFilZ = 8;

// c-weighted symmetric sum: t_0 w_c + sum_k t_k (w_(c-k) + w_(c+k)).
template <int R, typename T>
__device__ __forceinline__ T sym_taps(const T (&t)[R + 1], const T* w)
{
    T s = t[0] * w[R];
#pragma unroll
    for (int k = 1; k <= R; ++k) s = fma_(t[k], w[R - k] + w[R + k], s);
    return s;
}
template <int R, typename T>
__device__ __forceinline__ T box_sum(const T* w)
{
    T s = w[R];
#pragma unroll
    for (int k = 1; k <= R; ++k) s += w[R - k] + w[R + k];
    return s;
}

// GAUSS: y1 = g_y g_x f.  LAPL: y1 = b_y l_x f + l_y b_x f, y2 = b_y b_x f (RB
// > 0; for RB = 0 b is the identity).  D = 2: the filter itself into dst.
template <int D, typename T, int KIND, int RA, int RB>
__device__ __forceinline__ void kfil_xy(KMember& m, const LBM_K KFil& j, int tile, int comp, T* sm)
{
    constexpr int TX = kFilTX, TY = kFilTY, HX = TX + 2 * RA, HY = TY + 2 * RA, SX = (HX + 3) / 4 * 4;
    constexpr bool GA = KIND == LBM_FILT_GAUSS;
    constexpr int RY = GA ? RA : RB;         // rows of A_x f beyond the tile
    T* f = sm;                               // [HY][SX]
    T* ax = f + HY * SX;                     // A_x f, rows -RY .. TY + RY
    T* bx = ax + (TY + 2 * RY) * TX;         // b_x f, all rows (RB > 0)
    const int nx = m.nx, ny = m.ny, tid = threadIdx.x;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    const int x0 = tile % ntx * TX, y0 = tile / ntx % nty * TY, z = tile / (ntx * nty);
    const size_t sN = (size_t)m.N;
    const unsigned zo = (unsigned)z * (unsigned)(nx * ny);
    const T* src = (const T*)j.src + comp * sN;
    const LBM_K T* tp = kc((const T*)j.taps);
    T t[RA + 1];
#pragma unroll
    for (int k = 0; k <= RA; ++k) t[k] = tp[k];
    for (int e = tid; e < HY * HX; e += kBlock) {
        const int hx = e % HX, hy = e / HX;
        int gx = wrapi(x0 + hx - RA, nx), gy = y0 + hy - RA;
        if ((unsigned)gx >= (unsigned)nx) gx = modi(gx, nx);
        bool ok = true;
        if (m.walls) ok = gy >= 0 && gy < ny;
        else {
            gy = wrapi(gy, ny);
            if ((unsigned)gy >= (unsigned)ny) gy = modi(gy, ny);
        }
        f[hy * SX + hx] = ok ? ld_at(src, zo + (unsigned)(gx + nx * gy)) : T(0);
    }
    __syncthreads();
    for (int q = tid; q < HY * (TX / 4); q += kBlock) {
        const int r = q / (TX / 4), c = q % (TX / 4) * 4;
        const bool a_row = GA || (r >= RA - RY && r < RA + TY + RY);
        if (!a_row && RB == 0) continue;
        T w[4 + 2 * RA];
#pragma unroll
        for (int k = 0; k < 4 + 2 * RA; ++k) w[k] = f[r * SX + c + k];
        if (a_row) {
#pragma unroll
            for (int k = 0; k < 4; ++k) ax[(r - (RA - RY)) * TX + c + k] = sym_taps<RA, T>(t, w + k);
        }
        if constexpr (RB > 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) bx[r * TX + c + k] = box_sum<RB, T>(w + k + RA - RB);
        }
    }
    __syncthreads();
    const int lx = tid % TX, yq = tid / TX * 4, x = x0 + lx;
    if (x >= nx) return;
    T o1[4], o2[4];
    if constexpr (GA) {
        T w[4 + 2 * RA];
#pragma unroll
        for (int k = 0; k < 4 + 2 * RA; ++k) w[k] = ax[(yq + k) * TX + lx];
#pragma unroll
        for (int k = 0; k < 4; ++k) o1[k] = sym_taps<RA, T>(t, w + k);
    } else {
        T w[4 + 2 * RA], u[4 + 2 * RB];
#pragma unroll
        for (int k = 0; k < 4 + 2 * RA; ++k) w[k] = RB > 0 ? bx[(yq + k) * TX + lx] : f[(yq + k) * SX + lx + RA];
#pragma unroll
        for (int k = 0; k < 4 + 2 * RB; ++k) u[k] = ax[(yq + k) * TX + lx];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            o1[k] = box_sum<RB, T>(u + k) + sym_taps<RA, T>(t, w + k);
            o2[k] = box_sum<RB, T>(w + k + RA - RB);
        }
    }
    T* d1 = (T*)(D == 2 ? j.dst : j.y1) + comp * sN;
    T* d2 = (T*)j.y2 + comp * sN;
    const T cf = T(j.coef);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int y = y0 + yq + k;
        if (y >= ny) break;
        const unsigned c = zo + (unsigned)(x + nx * y);
        st_at(d1, c, D == 2 ? cf * o1[k] : o1[k]);
        if (D == 3 && !GA && RB > 0) st_at(d2, c, o2[k]);
    }
}

// GAUSS: dst = g_z y1.  LAPL: dst = coef (b_z y1 + l_z y2), y2 the source for
// RB = 0.
template <typename T, int KIND, int RA, int RB>
__device__ __forceinline__ void kfil_z(KMember& m, const LBM_K KFil& j, int blk, int comp)
{
    constexpr int NO = kFilZ;
    constexpr bool GA = KIND == LBM_FILT_GAUSS;
    const unsigned plane = (unsigned)(m.nx * m.ny);
    const int nz = m.nz, nb = (int)((plane + kBlock - 1) / kBlock);
    const unsigned c = (unsigned)(blk % nb) * kBlock + threadIdx.x;
    const int z0 = blk / nb * NO;
    if (c >= plane) return;
    const size_t sN = (size_t)m.N;
    const T* a = (const T*)(GA ? j.y1 : (RB > 0 ? j.y2 : j.src)) + comp * sN;
    const T* b = (const T*)j.y1 + comp * sN;
    const LBM_K T* tp = kc((const T*)j.taps);
    T t[RA + 1];
#pragma unroll
    for (int k = 0; k <= RA; ++k) t[k] = tp[k];
    T w[NO + 2 * RA], u[GA ? 1 : NO + 2 * RB];
    unsigned zo = (unsigned)modi(z0 - RA, nz) * plane;   // (uniform)
    const unsigned zl = (unsigned)(nz - 1) * plane;
#pragma unroll
    for (int k = 0; k < NO + 2 * RA; ++k) {
        w[k] = ld_at(a, zo + c);
        if constexpr (!GA) {
            if (k >= RA - RB && k < RA + RB + NO) u[k - (RA - RB)] = ld_at(b, zo + c);
        }
        zo = zo == zl ? 0u : zo + plane;
    }
    T* dst = (T*)j.dst + comp * sN;
    const T cf = T(j.coef);
#pragma unroll
    for (int k = 0; k < NO; ++k) {
        if (z0 + k >= nz) break;
        T o;
        if constexpr (GA) o = sym_taps<RA, T>(t, w + k);
        else o = cf * (box_sum<RB, T>(u + k) + sym_taps<RA, T>(t, w + k));
        st_at(dst, (unsigned)(z0 + k) * plane + c, o);
    }
}

// The variants: GAUSS radii 2 (also the identity), 4, .., 12; LAPL radius 2, 7
// and 12 (s = 1, 3, 5; boxes of radius 0, 1, 2).
#define LBM_KFIL_SWITCH(CALL)                                  \
    switch (j.kind * 16 + j.ra) {                              \
    case LBM_FILT_GAUSS * 16 + 2: CALL(LBM_FILT_GAUSS, 2, 0); break;   \
    case LBM_FILT_GAUSS * 16 + 4: CALL(LBM_FILT_GAUSS, 4, 0); break;   \
    case LBM_FILT_GAUSS * 16 + 6: CALL(LBM_FILT_GAUSS, 6, 0); break;   \
    case LBM_FILT_GAUSS * 16 + 8: CALL(LBM_FILT_GAUSS, 8, 0); break;   \
    case LBM_FILT_GAUSS * 16 + 10: CALL(LBM_FILT_GAUSS, 10, 0); break; \
    case LBM_FILT_GAUSS * 16 + 12: CALL(LBM_FILT_GAUSS, 12, 0); break; \
    case LBM_FILT_LAPL * 16 + 2: CALL(LBM_FILT_LAPL, 2, 0); break;     \
    case LBM_FILT_LAPL * 16 + 7: CALL(LBM_FILT_LAPL, 7, 1); break;     \
    case LBM_FILT_LAPL * 16 + 12: CALL(LBM_FILT_LAPL, 12, 2); break;   \
    }

// Work of a filter launch in the XCDs' order: workgroup b runs on XCD b mod 8
// and takes item (b mod 8) q + b / 8 of each XCD's q; none past n.
__device__ __forceinline__ int xcd_item(int n)
{
    const int q = (n + 7) / 8, b = (int)blockIdx.x;
    return (b & 7) * q + (b >> 3) < n && (b >> 3) < q ? (b & 7) * q + (b >> 3) : -1;
}

template <int LAT, typename T>
__global__ __launch_bounds__(kBlock) void k_kxy(const DevMember* __restrict__ mems, int mem,
                                               const KFil* __restrict__ jobs, int n)
{
    extern __shared__ __align__(16) unsigned char kfil_lds[];
    constexpr int D = Lat<LAT>::D;
    const LBM_K KFil& j = *kc(jobs + blockIdx.y / D);
    const int comp = blockIdx.y % D, item = xcd_item(n);
    if (item < 0 || comp >= j.ncomp) return;   // uniform
    KMember& m = *kc(mems + mem);
    T* sm = (T*)kfil_lds;
#define LBM_KXY(KIND, RA, RB) kfil_xy<D, T, KIND, RA, RB>(m, j, item, comp, sm)
    LBM_KFIL_SWITCH(LBM_KXY)
#undef LBM_KXY
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_kz(const DevMember* __restrict__ mems, int mem,
                                               const KFil* __restrict__ jobs, int n)
{
    const LBM_K KFil& j = *kc(jobs + blockIdx.y / 3);
    const int comp = blockIdx.y % 3, item = xcd_item(n);
    if (item < 0 || comp >= j.ncomp) return;
    KMember& m = *kc(mems + mem);
#define LBM_KZ(KIND, RA, RB) kfil_z<T, KIND, RA, RB>(m, j, item, comp)
    LBM_KFIL_SWITCH(LBM_KZ)
#undef LBM_KZ
}

// LDS of k_kxy for jobs of radius up to ra (the larger of the two kinds).
constexpr size_t kfil_lds_bytes(int ra, size_t esz)
{
    const int hx = (kFilTX + 2 * ra + 3) / 4 * 4, hy = kFilTY + 2 * ra, rb = ra / 5;
    return esz * (size_t)(hy * hx + (kFilTY + 2 * rb + hy) * kFilTX);
}

// ---------------------------------------------------------------------------
// Sharp Fourier band filters (eq. scale-aware-energy-fourier) through hipFFT.
// k_fpack forms w = curl v* and writes the components of v* (with E QoIs) and of
// w (with Z QoIs) as complex fields; one forward transform of all of them;
// k_fmask writes, per QoI and component, the masked spectrum (l - 1/2 <= |k| < m
// + 1/2, integer mode indices; with the 1/N of the inverse transform); one
// inverse transform of all of them; k_funpack takes the real parts to V_s = R v*
// (E) and U_s = R w (Z).  256 x 256, FP32, three bands of each kind, MI355X:
// fourteen launches per step -> seven, the step 73 -> 53 us (with the solve in
// the apply).  Every component keeps a complex field of its own: two of them as
// the real and imaginary part of one halve the transforms (47 us), but a
// transform rounds relative to the larger part (FP32, smooth field, w_z beside
// v_z, bands 0 to 3: error 1.5e-7 -> 4.0e-7 on 64^3, 1.8e-7 -> 1.3e-6 on 192^3).
// ---------------------------------------------------------------------------
// nv components of v*, then nw of w
template <int LAT, typename T, typename CT>
__global__ __launch_bounds__(kBlock) void k_fpack(const T* __restrict__ vs, CT* __restrict__ dst, int nv, int nw, int nx,
                                                  int ny, int nz)
{
    using L = Lat<LAT>;
    constexpr int D = L::D, NC = L::NC;
    const unsigned N = (unsigned)nx * ny * nz, i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= N) return;
    CT o;
    o.y = T(0);
    if (nv) {   // uniform
#pragma unroll
        for (int a = 0; a < D; ++a) {
            o.x = ld_at(vs + (size_t)a * N, i);
            dst[(size_t)a * N + i] = o;
        }
    }
    if (nw) {
        const int x = (int)(i % nx), t = (int)(i / nx), y = t % ny, z = t / ny;
        const Nbr n = nbr_at(i, x, y, z, nx, ny, nz, 0, D);
        T w[3];
        curl_nb<D, T>(vs, N, i, n, w);
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            o.x = w[a];
            dst[(size_t)(nv + a) * N + i] = o;
        }
    }
}

// the masked spectrum of every slot, out[slot][cell]
template <typename T, typename CT>
__global__ __launch_bounds__(kBlock) void k_fmask(const CT* __restrict__ spec, CT* __restrict__ out, FSlots sl, int nx,
                                                  int ny, int nz)
{
    const size_t N = (size_t)nx * ny * nz;
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= N) return;
    const int jx = (int)(i % nx), jy = (int)((i / nx) % ny), jz = (int)(i / ((size_t)nx * ny));
    const int kx = jx <= nx / 2 ? jx : jx - nx, ky = jy <= ny / 2 ? jy : jy - ny, kz = jz <= nz / 2 ? jz : jz - nz;
    const double kn = sqrt((double)kx * kx + (double)ky * ky + (double)kz * kz);
    const T s = T(1.0 / (double)N);
    for (int b = 0; b < sl.n; ++b) {
        const bool keep = kn >= sl.l[b] - 0.5 && kn < sl.m[b] + 0.5;
        CT o;
        o.x = o.y = T(0);
        if (keep) {
            const CT c = spec[(size_t)sl.field[b] * N + i];
            o.x = c.x * s;
            o.y = c.y * s;
        }
        out[(size_t)b * N + i] = o;
    }
}

// the real parts of the inverse transforms into their destinations
template <typename T, typename CT>
__global__ __launch_bounds__(kBlock) void k_funpack(const CT* __restrict__ src, FSlots sl, size_t N)
{
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= N) return;
    const int b = blockIdx.y;
    ((T*)sl.dst[b])[i] = src[(size_t)b * N + i].x;
}

template <int LAT, typename T>
static void launch_fourier(const FourierProg& f, hipStream_t st)
{
    using CT = typename std::conditional<std::is_same<T, float>::value, float2, double2>::type;
    const size_t N = (size_t)f.nx * f.ny * f.nz;
    const dim3 blk(kBlock), grd((unsigned)((N + kBlock - 1) / kBlock));
    auto exec = [&](void* plan, void* data, int dir) {
        hipfftHandle h = (hipfftHandle)plan;
        hipfftResult r = hipfftSetStream(h, st);
        if (r == HIPFFT_SUCCESS) {
            if constexpr (std::is_same<T, float>::value)
                r = hipfftExecC2C(h, (hipfftComplex*)data, (hipfftComplex*)data, dir);
            else
                r = hipfftExecZ2Z(h, (hipfftDoubleComplex*)data, (hipfftDoubleComplex*)data, dir);
        }
        if (r != HIPFFT_SUCCESS) f.failed = 1;
    };
    hipLaunchKernelGGL((k_fpack<LAT, T, CT>), grd, blk, 0, st, (const T*)f.vs, (CT*)f.spec, f.nv, f.nw, f.nx, f.ny, f.nz);
    exec(f.plan[0], f.spec, HIPFFT_FORWARD);
    hipLaunchKernelGGL((k_fmask<T, CT>), grd, blk, 0, st, (const CT*)f.spec, (CT*)f.band, f.slots, f.nx, f.ny, f.nz);
    exec(f.plan[1], f.band, HIPFFT_BACKWARD);
    hipLaunchKernelGGL((k_funpack<T, CT>), dim3(grd.x, f.slots.n), blk, 0, st, (const CT*)f.band, f.slots, N);
}

// ---------------------------------------------------------------------------
// Diagnostics of plain runs: E and Z of the post-streaming velocity.
// ---------------------------------------------------------------------------
template <int LAT, typename T>
__global__ __launch_bounds__(kBlock) void k_diag(const DevMember* __restrict__ mems, const int2* __restrict__ work)
{
    using L = Lat<LAT>;
    constexpr int D = L::D;
    __shared__ double lds[2 * (kBlock / 64)];
    const int2 wk = work[blockIdx.x];
    KMember& m = *kc(mems + wk.x);
    const int N = m.N, nx = m.nx, ny = m.ny, nz = m.nz;
    const int cell = wk.y * kBlock + threadIdx.x;
    double v[2] = {0, 0};
    if (cell < N) {
        const int x = cell % nx, t = cell / nx, y = t % ny, z = t / ny;
        const T* vn = (const T*)m.vn;
        double e = 0;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const double u = (double)vn[(size_t)a * N + cell];
            e += 0.5 * u * u;
        }
        T w[3];
        curl_at<D, T>(vn, (size_t)N, x, y, z, nx, ny, nz, m.walls, w);
        double zz = 0;
#pragma unroll
        for (int a = 0; a < L::NC; ++a) zz += 0.5 * (double)w[a] * (double)w[a];
        v[0] = e;
        v[1] = zz;
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        m.part_diag[(size_t)wk.y * 2] = v[0];
        m.part_diag[(size_t)wk.y * 2 + 1] = v[1];
    }
}

static __global__ __launch_bounds__(kBlock) void k_fin_diag(const DevMember* __restrict__ mems, const int* __restrict__ work)
{
    __shared__ double red[6 * (kBlock / 64)];
    KMember& m = *kc(mems + work[blockIdx.x]);
    double v[6] = {0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < m.nb1; b += kBlock) {
        for (int k = 0; k < 4; ++k) v[k] += m.part_stats[(size_t)b * 4 + k];
        v[4] += m.part_diag[(size_t)b * 2];
        v[5] += m.part_diag[(size_t)b * 2 + 1];
    }
    block_sum<6>(v, red);
    if (threadIdx.x == 0) {
        DevCtl* ctl = m.ctl;
        const long long step = ctl->step;
        lbm_qoi_rec* rec = m.recs + (size_t)(step % m.rec_cap);
        rec->step = step;
        rec->flags = ctl->flags & 1;
        rec->nq = 0;
        rec->mass = (double)m.N + v[0];
        rec->mom[0] = v[1];
        rec->mom[1] = v[2];
        rec->mom[2] = v[3];
        rec->diag_e = v[4];
        rec->diag_z = v[5];
        for (int k = 0; k < kMaxQ; ++k) { rec->q[k] = 0; rec->dq[k] = 0; rec->gamma[k] = 0; }
        ctl->step = step + 1;
    }
}

#ifndef LBM_PART
// ---------------------------------------------------------------------------
// State access kernels.
// ---------------------------------------------------------------------------
template <int LAT, typename T, int PREC>
__global__ void k_init(const DevMember* __restrict__ mems, int flip, const double* __restrict__ rho0,
                       const double* __restrict__ u0)
{
    using L = Lat<LAT>;
    KMember& m = *kc(mems);
    const int N = m.N;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= N) return;
    T* g = (T*)m.g[m.parity ^ flip];
    const double r = rho0 ? rho0[cell] : 1.0;
    double u[3] = {0, 0, 0}, uu = 0;
    for (int a = 0; a < L::D; ++a) { u[a] = u0 ? u0[(size_t)a * N + cell] : 0.0; uu += u[a] * u[a]; }
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const double cu = L::cx[i] * u[0] + L::cy[i] * u[1] + L::cz[i] * u[2];
        const double X = 3.0 * cu + 4.5 * cu * cu - 1.5 * uu;
        const double feq = L::w[i] * r * (1.0 + X);
        g[pop_at64<L::Q>(i, (size_t)cell)] = PREC == LBM_FP32_PLAIN ? (T)feq : (T)(L::w[i] * ((r - 1.0) + r * X));
    }
    if (m.has_to) {
        ((T*)m.rho)[cell] = 0;
        for (int a = 0; a < L::D; ++a) ((T*)m.vs)[(size_t)a * N + cell] = 0;
    }
}

template <int LAT, typename T, int PREC>
__global__ void k_get_pop(const DevMember* __restrict__ mems, int flip, double* __restrict__ f)
{
    using L = Lat<LAT>;
    KMember& m = *kc(mems);
    const int N = m.N;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= N) return;
    const T* g = (const T*)m.g[m.parity ^ flip];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        f[(size_t)i * N + cell] = (double)g[pop_at64<L::Q>(i, (size_t)cell)] + (PREC == LBM_FP32_PLAIN ? 0.0 : L::w[i]);
}

template <int LAT, typename T, int PREC>
__global__ void k_set_pop(const DevMember* __restrict__ mems, int flip, const double* __restrict__ f)
{
    using L = Lat<LAT>;
    KMember& m = *kc(mems);
    const int N = m.N;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= N) return;
    T* g = (T*)m.g[m.parity ^ flip];
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        g[pop_at64<L::Q>(i, (size_t)cell)] = (T)(f[(size_t)i * N + cell] - (PREC == LBM_FP32_PLAIN ? 0.0 : L::w[i]));
    if (m.has_to) {
        ((T*)m.rho)[cell] = 0;
        for (int a = 0; a < L::D; ++a) ((T*)m.vs)[(size_t)a * N + cell] = 0;
    }
}

// Wall-anchored stride-m projection (Sec. 3, the projection phi_m; Sec. 7.1
// for the channel): coarse cell (i, j, k) takes the fine cell
// (m i + o, m j + o, m k + o), o = (m - 1) / 2, so the coarse walls, half a
// coarse cell beyond the first and last coarse rows, coincide with the fine
// ones.  Writes the full populations (nullable fpop [Q][Nc]) and the velocity
// sum c f / sum f of the post-collision state (nullable vout [D][Nc]).
template <int LAT, typename T, int PREC>
__global__ __launch_bounds__(kBlock) void k_project(const DevMember* __restrict__ fine, int flip, int m, int ncx,
                                                    int ncy, int ncz, double* __restrict__ fpop,
                                                    void* __restrict__ vout, int vout_fp64, int kind)
{
    using L = Lat<LAT>;
    KMember& F = *kc(fine);
    const int Nc = ncx * ncy * ncz;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= Nc) return;
    const int i = cell % ncx, t = cell / ncx, j = t % ncy, k = t / ncy;
    const int o = (m - 1) / 2;
    if (L::D == 2 && kind == LBM_PROJ_BICUBIC) {
        // bicubic (2-D, doubly periodic): the weighted mean over fine cells
        // (m i + o + rx, m j + o + ry), |rx|, |ry| < 2 m, with weights
        // K(rx / m) K(ry / m) / S^2, K the Keys cubic (a = -1/2), S the sum
        // of K(r / m) over the window; of the populations, and of the
        // velocity of each fine cell
        const int R = 2 * m - 1;
        auto keys = [](double x) {
            x = fabs(x);
            return x <= 1.0 ? (1.5 * x - 2.5) * x * x + 1.0 : (x < 2.0 ? ((-0.5 * x + 2.5) * x - 4.0) * x + 2.0 : 0.0);
        };
        double S = 0;
        for (int r = -R; r <= R; ++r) S += keys((double)r / m);
        const double rS = 1.0 / S;
        const T* g = (const T*)F.g[F.parity ^ flip];
        double acc[L::Q], uacc[2] = {0, 0};
#pragma unroll
        for (int q = 0; q < L::Q; ++q) acc[q] = 0;
        for (int ry = -R; ry <= R; ++ry) {
            const double wy = keys((double)ry / m) * rS;
            const int yf = modi(m * j + o + ry, F.ny);
            for (int rx = -R; rx <= R; ++rx) {
                const double w = wy * keys((double)rx / m) * rS;
                const size_t fc = (size_t)yf * F.nx + (size_t)modi(m * i + o + rx, F.nx);
                double drho = 0, jx = 0, jy = 0;
#pragma unroll
                for (int q = 0; q < L::Q; ++q) {
                    const double gq = (double)g[pop_at64<L::Q>(q, fc)];
                    acc[q] += w * gq;
                    drho += gq;
                    jx += L::cx[q] * gq;
                    jy += L::cy[q] * gq;
                }
                const double rho = PREC == LBM_FP32_PLAIN ? drho : 1.0 + drho;
                uacc[0] += w * (jx / rho);
                uacc[1] += w * (jy / rho);
            }
        }
        if (fpop) {
#pragma unroll
            for (int q = 0; q < L::Q; ++q) fpop[(size_t)q * Nc + cell] = acc[q] + (PREC == LBM_FP32_PLAIN ? 0.0 : L::w[q]);
        }
        if (vout) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (vout_fp64) ((double*)vout)[(size_t)a * Nc + cell] = uacc[a];
                else ((float*)vout)[(size_t)a * Nc + cell] = (float)uacc[a];
            }
        }
        return;
    }
    const int zf = L::D == 3 ? m * k + o : 0;
    const size_t fc = ((size_t)zf * F.ny + (size_t)(m * j + o)) * F.nx + (size_t)(m * i + o);
    const T* g = (const T*)F.g[F.parity ^ flip];
    double drho = 0, jm[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < L::Q; ++q) {
        const double gq = (double)g[pop_at64<L::Q>(q, fc)];
        if (fpop) fpop[(size_t)q * Nc + cell] = gq + (PREC == LBM_FP32_PLAIN ? 0.0 : L::w[q]);
        drho += gq;
        jm[0] += L::cx[q] * gq;
        jm[1] += L::cy[q] * gq;
        jm[2] += L::cz[q] * gq;
    }
    if (vout) {
        // shifted storage: rho - 1 = sum g and rho v = sum c g (sum c w = 0)
        const double rho = PREC == LBM_FP32_PLAIN ? drho : 1.0 + drho;
#pragma unroll
        for (int a = 0; a < L::D; ++a) {
            const double u = jm[a] / rho;
            if (vout_fp64) ((double*)vout)[(size_t)a * Nc + cell] = u;
            else ((float*)vout)[(size_t)a * Nc + cell] = (float)u;
        }
    }
}

// The bicubic velocity projection in two separable passes (the reference
// QoIs of the Kolmogorov case): x, for every fine row yf and coarse column
// i, the weighted sum over the fine columns of the fine-cell velocities
// into tmp [2][fny][ncx]; then y, for every coarse cell, the weighted sum
// of tmp over the fine rows.  Weights as in k_project.
__device__ __forceinline__ double keys_w(int r, int m, double rS)
{
    const double x = fabs((double)r / m);
    return (x <= 1.0 ? (1.5 * x - 2.5) * x * x + 1.0 : (x < 2.0 ? ((-0.5 * x + 2.5) * x - 4.0) * x + 2.0 : 0.0)) * rS;
}

template <typename T, int PREC>
__global__ __launch_bounds__(kBlock) void k_proj_bx(const DevMember* __restrict__ fine, int flip, int m, int ncx,
                                                    double rS, double* __restrict__ tmp)
{
    using L = Lat<LBM_D2Q9>;
    KMember& F = *kc(fine);
    const int n = F.ny * ncx;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int i = idx % ncx, yf = idx / ncx;
    const int o = (m - 1) / 2, R = 2 * m - 1;
    const T* g = (const T*)F.g[F.parity ^ flip];
    double ux = 0, uy = 0;
    for (int rx = -R; rx <= R; ++rx) {
        const size_t fc = (size_t)yf * F.nx + (size_t)modi(m * i + o + rx, F.nx);
        double drho = 0, jx = 0, jy = 0;
#pragma unroll
        for (int q = 0; q < L::Q; ++q) {
            const double gq = (double)g[pop_at64<L::Q>(q, fc)];
            drho += gq;
            jx += L::cx[q] * gq;
            jy += L::cy[q] * gq;
        }
        const double rho = PREC == LBM_FP32_PLAIN ? drho : 1.0 + drho;
        const double w = keys_w(rx, m, rS);
        ux += w * (jx / rho);
        uy += w * (jy / rho);
    }
    tmp[idx] = ux;
    tmp[(size_t)n + idx] = uy;
}

static __global__ __launch_bounds__(kBlock) void k_proj_by(int m, int ncx, int ncy, int fny, double rS,
                                                    const double* __restrict__ tmp, void* __restrict__ vout,
                                                    int vout_fp64)
{
    const int Nc = ncx * ncy;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= Nc) return;
    const int i = cell % ncx, j = cell / ncx;
    const int o = (m - 1) / 2, R = 2 * m - 1;
    const size_t n = (size_t)fny * ncx;
    double v[2] = {0, 0};
    for (int ry = -R; ry <= R; ++ry) {
        const size_t t = (size_t)modi(m * j + o + ry, fny) * ncx + i;
        const double w = keys_w(ry, m, rS);
        v[0] += w * tmp[t];
        v[1] += w * tmp[n + t];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (vout_fp64) ((double*)vout)[(size_t)a * Nc + cell] = v[a];
        else ((float*)vout)[(size_t)a * Nc + cell] = (float)v[a];
    }
}

void launch_project(int lattice, int precision, const DevMember* fine, int flip, int m, int ncx, int ncy, int ncz,
                    double* fpop, void* vout, int vout_fp64, int kind, hipStream_t st, double* tmp)
{
    const int Nc = ncx * ncy * ncz;
    const dim3 blk(kBlock), grd((Nc + kBlock - 1) / kBlock);
    if (kind == LBM_PROJ_BICUBIC && !fpop && tmp && lattice == LBM_D2Q9) {
        double S = 0;   // the sum of the window's kernel values (host copy of k_project's)
        for (int r = -(2 * m - 1); r <= 2 * m - 1; ++r) {
            const double x = std::fabs((double)r / m);
            S += x <= 1.0 ? (1.5 * x - 2.5) * x * x + 1.0 : (x < 2.0 ? ((-0.5 * x + 2.5) * x - 4.0) * x + 2.0 : 0.0);
        }
        const int fny = ncy * m, nx1 = fny * ncx;
        const dim3 g1((nx1 + kBlock - 1) / kBlock);
        if (precision == LBM_FP64)
            hipLaunchKernelGGL((k_proj_bx<double, LBM_FP64>), g1, blk, 0, st, fine, flip, m, ncx, 1.0 / S, tmp);
        else if (precision == LBM_FP32_PLAIN)
            hipLaunchKernelGGL((k_proj_bx<float, LBM_FP32_PLAIN>), g1, blk, 0, st, fine, flip, m, ncx, 1.0 / S, tmp);
        else
            hipLaunchKernelGGL((k_proj_bx<float, LBM_FP32_SHIFTED>), g1, blk, 0, st, fine, flip, m, ncx, 1.0 / S, tmp);
        hipLaunchKernelGGL(k_proj_by, grd, blk, 0, st, m, ncx, ncy, fny, 1.0 / S, (const double*)tmp, vout, vout_fp64);
        return;
    }
#define LBM_PROJ(LAT, T, PREC)                                                                                    \
    hipLaunchKernelGGL((k_project<LAT, T, PREC>), grd, blk, 0, st, fine, flip, m, ncx, ncy, ncz, fpop, vout, vout_fp64, \
                       kind)
    switch (lattice * 3 + precision) {
    case LBM_D2Q9 * 3 + LBM_FP32_SHIFTED: LBM_PROJ(LBM_D2Q9, float, LBM_FP32_SHIFTED); break;
    case LBM_D2Q9 * 3 + LBM_FP64: LBM_PROJ(LBM_D2Q9, double, LBM_FP64); break;
    case LBM_D2Q9 * 3 + LBM_FP32_PLAIN: LBM_PROJ(LBM_D2Q9, float, LBM_FP32_PLAIN); break;
    case LBM_D3Q19 * 3 + LBM_FP32_SHIFTED: LBM_PROJ(LBM_D3Q19, float, LBM_FP32_SHIFTED); break;
    case LBM_D3Q19 * 3 + LBM_FP64: LBM_PROJ(LBM_D3Q19, double, LBM_FP64); break;
    case LBM_D3Q19 * 3 + LBM_FP32_PLAIN: LBM_PROJ(LBM_D3Q19, float, LBM_FP32_PLAIN); break;
    }
#undef LBM_PROJ
}

// Pure streaming (no collision) into the other buffer.
template <int LAT, typename T, bool TO>
__global__ void k_stream_only(const DevMember* __restrict__ mems, int flip)
{
    using L = Lat<LAT>;
    KMember& m = *kc(mems);
    const int N = m.N, nx = m.nx, ny = m.ny;
    const int cell = blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= N) return;
    const int x = cell % nx, t = cell / nx, y = t % ny, z = t / ny;
    T f[L::Q];
    gather<LAT, T, false>(m, (const T*)m.g[m.parity ^ flip], x, y, z, cell, f);
    T* gd = (T*)m.g[m.parity ^ flip ^ 1];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) gd[pop_at64<L::Q>(i, (size_t)cell)] = f[i];
}

#endif  // LBM_PART

// ---------------------------------------------------------------------------
// Launch wrappers (host side), one instantiation per lattice/precision/kind.
// ---------------------------------------------------------------------------
// The TO step after the stream-collide: sensitivities, reduction, solve and
// apply.
template <int LAT, typename T>
void launch_to(const LaunchGroup& g, hipStream_t st, int flip, hipEvent_t* ev)
{
    const dim3 blk(kBlock);
    auto mark = [&](int k) {
        if (ev) (void)hipEventRecord(ev[k], st);
    };
    if (g.nkfil > 0 && g.any_z) {   // (the binomial chains and the Fourier bands form w themselves)
        if (g.wt) hipLaunchKernelGGL((k_curl<LAT, T, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1);
        else hipLaunchKernelGGL((k_curl<LAT, T, false>), dim3(g.nb1), blk, 0, st, g.mems, g.work1);
    }
    mark(2);
    if (g.kf) {
        if (g.fprog) launch_fourier<LAT, T>(*g.fprog, st);
        // R twice: the x and y parts, then (3-D) the z parts with the sum
        const int ntile = (g.kdim[0] + kFilTX - 1) / kFilTX * ((g.kdim[1] + kFilTY - 1) / kFilTY) * g.kdim[2];
        const int nzb = (g.kdim[0] * g.kdim[1] + kBlock - 1) / kBlock * ((g.kdim[2] + kFilZ - 1) / kFilZ);
        for (int app = 0; app < (g.nkfil > 0 ? 2 : 0); ++app) {
            const KFil* jobs = g.kfil + app * g.nkfil;
            hipLaunchKernelGGL((k_kxy<LAT, T>), dim3((ntile + 7) / 8 * 8, g.nkfil * Lat<LAT>::D), blk,
                               kfil_lds_bytes(g.krad, sizeof(T)), st, g.mems, g.kmem, jobs, ntile);
            if constexpr (Lat<LAT>::D == 3)
                hipLaunchKernelGGL((k_kz<T>), dim3((nzb + 7) / 8 * 8, g.nkfil * 3), blk, 0, st, g.mems, g.kmem, jobs, nzb);
        }
    }
    if (g.pair) {
        if constexpr (Lat<LAT>::D == 2) {
#define LBM_PAIR(NLV)                                                                                          \
    do {                                                                                                       \
        if (g.wt) hipLaunchKernelGGL((k_chain_pair<T, NLV, true>), dim3(g.nbq), dim3(64), 0, st, g.mems, g.workq); \
        else hipLaunchKernelGGL((k_chain_pair<T, NLV, false>), dim3(g.nbq), dim3(64), 0, st, g.mems, g.workq); \
    } while (0)
            if (g.cnl == 2) LBM_PAIR(2); else LBM_PAIR(4);
#undef LBM_PAIR
        }
    } else if (g.nbc > 0) {
#define LBM_CHAIN(NLV, MSV)                                                                                    \
    hipLaunchKernelGGL((k_chain<LAT, T, NLV, MSV>), dim3(g.nbc), dim3(64 * chain_waves(Lat<LAT>::D)), 0, st, g.mems, g.workc)
        if (g.cnl == 2) { if (g.maxe <= 4 && g.maxz <= 4) LBM_CHAIN(2, 4); else LBM_CHAIN(2, 8); }
        else { if (g.maxe <= 4 && g.maxz <= 4) LBM_CHAIN(4, 4); else LBM_CHAIN(4, 8); }
#undef LBM_CHAIN
    }
    mark(3);
#define LBM_REDUCE(MEV, MZV, KFV)                                                                            \
    do {                                                                                                     \
        if (g.wt) hipLaunchKernelGGL((k_reduce<LAT, T, MEV, MZV, KFV, true>), dim3(g.nbr), blk, 0, st, g.mems, g.workr); \
        else hipLaunchKernelGGL((k_reduce<LAT, T, MEV, MZV, KFV, false>), dim3(g.nbr), blk, 0, st, g.mems, g.workr); \
    } while (0)
    // The variant of most positions a member fills.  MI355X, FP32, 256 x 128 x 128
    // and 96 x 48 x 48, us: two E QoIs <3, 0> 22 and 7.4, <3, 3> 37 and 10; five
    // E <8, 0> 49 and 12, <0, 6> 58 and 11, <0, 8> 92 and 14; two Z <3, 3> 43 and
    // 10, the same with no E positions; five E and a Z <0, 6> 84 and 12.5, <0, 8>
    // 125 and 16; an E and five Z 164 and 16, 202 and 20; two E and four Z <4, 4>
    // 141 and 14, <0, 6> 142 and 15.
#define LBM_REDUCE_KIND(KFV)                                               \
    do {                                                                   \
        if (g.maxe <= 1 && g.maxz <= 1) LBM_REDUCE(1, 1, KFV);             \
        else if (g.maxz == 0 && g.maxe <= 3) LBM_REDUCE(3, 0, KFV);        \
        else if (g.maxz == 0) LBM_REDUCE(8, 0, KFV);                       \
        else if (g.maxe <= 3 && g.maxz <= 3) LBM_REDUCE(3, 3, KFV);        \
        else if (g.maxe <= 4 && g.maxz <= 4) LBM_REDUCE(4, 4, KFV);        \
        else if (g.maxsa <= 6) LBM_REDUCE(0, 6, KFV);                      \
        else LBM_REDUCE(0, 8, KFV);                                        \
    } while (0)
    if (g.kf) LBM_REDUCE_KIND(true); else if (!g.pair) LBM_REDUCE_KIND(false);
#undef LBM_REDUCE_KIND
#undef LBM_REDUCE
    mark(4);
    hipLaunchKernelGGL(k_sum, dim3(g.nbs), blk, 0, st, g.mems, g.works);
    // the apply forms the solve itself on small launches (one launch less per step)
    const bool fused = fused_solve(g);
    if (!fused) hipLaunchKernelGGL(k_solve, dim3(g.nmem), blk, 0, st, g.mems, g.workm);
    mark(5);
    if (!g.probe) {
#define LBM_APPLY(SAV, DEFV)                                                                                 \
    do {                                                                                                     \
    if (fused && g.wt) hipLaunchKernelGGL((k_apply_fs<LAT, T, SAV, true, DEFV>), dim3(g.nbp), blk, 0, st, g.mems, g.workp, flip); \
    else if (fused) hipLaunchKernelGGL((k_apply_fs<LAT, T, SAV, false, DEFV>), dim3(g.nbp), blk, 0, st, g.mems, g.workp, flip); \
    else if (g.wt) hipLaunchKernelGGL((k_apply<LAT, T, SAV, true, DEFV>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
    else hipLaunchKernelGGL((k_apply<LAT, T, SAV, false, DEFV>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
    } while (0)
        if (g.defer && g.substrate != LBM_WALE) {
            if (g.maxsa <= 2) LBM_APPLY(2, true); else if (g.maxsa <= 6) LBM_APPLY(6, true); else LBM_APPLY(kMaxSA, true);
        } else {
            if (g.maxsa <= 2) LBM_APPLY(2, false); else if (g.maxsa <= 6) LBM_APPLY(6, false); else LBM_APPLY(kMaxSA, false);
        }
#undef LBM_APPLY
    }
}
#ifdef LBM_PART
#if LBM_PART != 0
extern template void launch_to<LBM_D2Q9, float>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#endif
#if LBM_PART != 3
extern template void launch_to<LBM_D3Q19, float>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#endif
#endif

template <int LAT, typename T, int PREC>
void launch_step_group(const LaunchGroup& g, hipStream_t st, int flip, hipEvent_t* ev)
{
    const dim3 blk(kBlock);
    if (g.nb1 == 0) return;
    auto mark = [&](int k) {
        if (ev) (void)hipEventRecord(ev[k], st);
    };
    mark(0);
    if (g.probe) goto to_chain;
    if (g.substrate == LBM_WALE) {
        if (g.mode == 2)
            hipLaunchKernelGGL((k_moments<LAT, T, PREC, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip,
                               (double*)nullptr, (double*)nullptr);
        else
            hipLaunchKernelGGL((k_moments<LAT, T, PREC, false>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip,
                               (double*)nullptr, (double*)nullptr);
    }
#define LBM_STEP_TK(SUB, TXV, ...)                                                                         \
    hipLaunchKernelGGL((k_step_t<LAT, T, PREC, SUB, TXV, __VA_ARGS__>), dim3(g.nbb), dim3(TXV * kBinTY), 0, st, g.mems, \
                       g.workb, flip)
#define LBM_STEP_T(SUB, TXV)                                                                               \
    do {                                                                                                   \
        if (!g.a32) LBM_STEP_TK(SUB, TXV, 2, false);                                                       \
        else if (g.wt) LBM_STEP_TK(SUB, TXV, 1);                                                           \
        else if (g.rag) LBM_STEP_TK(SUB, TXV, 2);                                                          \
        else LBM_STEP_TK(SUB, TXV, 0);                                                                     \
    } while (0)
#define LBM_STEP_SUB(SUB)                                                                                  \
    do {                                                                                                   \
        if constexpr (SUB != LBM_WALE) {                                                                   \
            if (g.mode == 2 && g.defer) {                                                                  \
                if (Lat<LAT>::D == 3 && g.btx == kBinTXW)                                                  \
                    LBM_STEP_T(SUB, (Lat<LAT>::D == 3 ? kBinTXW : kBinTX));                                \
                else                                                                                       \
                    LBM_STEP_T(SUB, kBinTX);                                                               \
                break;                                                                                     \
            }                                                                                              \
        }                                                                                                  \
        if (g.mode == 2 && !g.a32)                                                                         \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 2, false, false>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.mode == 2 && g.wt)                                                                      \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 2, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.mode == 2)                                                                              \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 2>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.mode == 1 && g.a32)                                                                     \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 1, false, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.mode == 1)                                                                              \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 1>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.a32 && g.nt)                                                                            \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 0, false, true, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.a32)                                                                                    \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 0, false, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else if (g.nt)                                                                                     \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 0, false, false, true>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
        else                                                                                               \
            hipLaunchKernelGGL((k_step<LAT, T, PREC, SUB, 0>), dim3(g.nb1), blk, 0, st, g.mems, g.work1, flip); \
    } while (0)
    if (g.substrate == LBM_SMAGORINSKY)
        LBM_STEP_SUB(LBM_SMAGORINSKY);
    else if (g.substrate == LBM_WALE)
        LBM_STEP_SUB(LBM_WALE);
    else
        LBM_STEP_SUB(LBM_BGK);
#undef LBM_STEP_SUB
#undef LBM_STEP_T
#undef LBM_STEP_TK
to_chain:
    mark(1);
    if (g.mode == 2) {
        launch_to<LAT, T>(g, st, flip, ev);
        mark(6);
    } else if (g.mode == 1) {
        hipLaunchKernelGGL((k_diag<LAT, T>), dim3(g.nb1), blk, 0, st, g.mems, g.work1);
        hipLaunchKernelGGL(k_fin_diag, dim3(g.nmem), blk, 0, st, g.mems, g.workm);
        mark(2); mark(3); mark(4); mark(5); mark(6);
    } else {
        mark(2); mark(3); mark(4); mark(5); mark(6);
    }
}

// The step kernels of one lattice and precision are compiled in a translation
// unit of their own (LBM_PART = 3 lattice + precision, built in parallel; the
// two FP32 forms share the TO kernels of the shifted one), everything else in
// the one without LBM_PART.
#ifdef LBM_PART
#if LBM_PART == 0
template void launch_step_group<LBM_D2Q9, float, LBM_FP32_SHIFTED>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#elif LBM_PART == 1
template void launch_step_group<LBM_D2Q9, double, LBM_FP64>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#elif LBM_PART == 2
template void launch_step_group<LBM_D2Q9, float, LBM_FP32_PLAIN>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#elif LBM_PART == 3
template void launch_step_group<LBM_D3Q19, float, LBM_FP32_SHIFTED>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#elif LBM_PART == 4
template void launch_step_group<LBM_D3Q19, double, LBM_FP64>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#else
template void launch_step_group<LBM_D3Q19, float, LBM_FP32_PLAIN>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
#endif
}  // namespace lbm
#else
extern template void launch_step_group<LBM_D2Q9, float, LBM_FP32_SHIFTED>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
extern template void launch_step_group<LBM_D2Q9, double, LBM_FP64>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
extern template void launch_step_group<LBM_D2Q9, float, LBM_FP32_PLAIN>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
extern template void launch_step_group<LBM_D3Q19, float, LBM_FP32_SHIFTED>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
extern template void launch_step_group<LBM_D3Q19, double, LBM_FP64>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);
extern template void launch_step_group<LBM_D3Q19, float, LBM_FP32_PLAIN>(const LaunchGroup&, hipStream_t, int, hipEvent_t*);

void launch_step(const LaunchGroup& g, hipStream_t st, int flip, hipEvent_t* ev)
{
    const int key = g.lattice * 3 + g.precision;
    switch (key) {
    case LBM_D2Q9 * 3 + LBM_FP32_SHIFTED: launch_step_group<LBM_D2Q9, float, LBM_FP32_SHIFTED>(g, st, flip, ev); break;
    case LBM_D2Q9 * 3 + LBM_FP64: launch_step_group<LBM_D2Q9, double, LBM_FP64>(g, st, flip, ev); break;
    case LBM_D2Q9 * 3 + LBM_FP32_PLAIN: launch_step_group<LBM_D2Q9, float, LBM_FP32_PLAIN>(g, st, flip, ev); break;
    case LBM_D3Q19 * 3 + LBM_FP32_SHIFTED: launch_step_group<LBM_D3Q19, float, LBM_FP32_SHIFTED>(g, st, flip, ev); break;
    case LBM_D3Q19 * 3 + LBM_FP64: launch_step_group<LBM_D3Q19, double, LBM_FP64>(g, st, flip, ev); break;
    case LBM_D3Q19 * 3 + LBM_FP32_PLAIN: launch_step_group<LBM_D3Q19, float, LBM_FP32_PLAIN>(g, st, flip, ev); break;
    }
}

template <int LAT, typename T, int PREC>
static void launch_state_t(int op, const DevMember* dm, int N, bool has_to, int flip, hipStream_t st,
                           const double* a, double* b)
{
    const dim3 blk(kBlock), grd((N + kBlock - 1) / kBlock);
    switch (op) {
    case OP_INIT: hipLaunchKernelGGL((k_init<LAT, T, PREC>), grd, blk, 0, st, dm, flip, a, (const double*)b); break;
    case OP_GET_POP: hipLaunchKernelGGL((k_get_pop<LAT, T, PREC>), grd, blk, 0, st, dm, flip, b); break;
    case OP_SET_POP: hipLaunchKernelGGL((k_set_pop<LAT, T, PREC>), grd, blk, 0, st, dm, flip, a); break;
    case OP_STREAM:
        if (has_to) hipLaunchKernelGGL((k_stream_only<LAT, T, true>), grd, blk, 0, st, dm, flip);
        else hipLaunchKernelGGL((k_stream_only<LAT, T, false>), grd, blk, 0, st, dm, flip);
        break;
    }
}

void launch_state(int op, int lattice, int precision, const DevMember* dm, int N, bool has_to, int flip,
                  hipStream_t st, const double* a, double* b)
{
    const int key = lattice * 3 + precision;
    switch (key) {
    case LBM_D2Q9 * 3 + LBM_FP32_SHIFTED: launch_state_t<LBM_D2Q9, float, LBM_FP32_SHIFTED>(op, dm, N, has_to, flip, st, a, b); break;
    case LBM_D2Q9 * 3 + LBM_FP64: launch_state_t<LBM_D2Q9, double, LBM_FP64>(op, dm, N, has_to, flip, st, a, b); break;
    case LBM_D2Q9 * 3 + LBM_FP32_PLAIN: launch_state_t<LBM_D2Q9, float, LBM_FP32_PLAIN>(op, dm, N, has_to, flip, st, a, b); break;
    case LBM_D3Q19 * 3 + LBM_FP32_SHIFTED: launch_state_t<LBM_D3Q19, float, LBM_FP32_SHIFTED>(op, dm, N, has_to, flip, st, a, b); break;
    case LBM_D3Q19 * 3 + LBM_FP64: launch_state_t<LBM_D3Q19, double, LBM_FP64>(op, dm, N, has_to, flip, st, a, b); break;
    case LBM_D3Q19 * 3 + LBM_FP32_PLAIN: launch_state_t<LBM_D3Q19, float, LBM_FP32_PLAIN>(op, dm, N, has_to, flip, st, a, b); break;
    }
}

void launch_fields(int lattice, int precision, const DevMember* dm, const int2* work1, int nb1, bool has_to,
                   int flip, hipStream_t st, double* rho_out, double* u_out)
{
    const int key = lattice * 3 + precision;
    const dim3 blk(kBlock), grd(nb1);
#define LBM_MOM(LAT, T, PREC)                                                                                  \
    do {                                                                                                       \
        if (has_to) hipLaunchKernelGGL((k_moments<LAT, T, PREC, true>), grd, blk, 0, st, dm, work1, flip, rho_out, \
                                       u_out);                                                                   \
        else hipLaunchKernelGGL((k_moments<LAT, T, PREC, false>), grd, blk, 0, st, dm, work1, flip, rho_out, u_out); \
    } while (0)
    switch (key) {
    case LBM_D2Q9 * 3 + LBM_FP32_SHIFTED: LBM_MOM(LBM_D2Q9, float, LBM_FP32_SHIFTED); break;
    case LBM_D2Q9 * 3 + LBM_FP64: LBM_MOM(LBM_D2Q9, double, LBM_FP64); break;
    case LBM_D2Q9 * 3 + LBM_FP32_PLAIN: LBM_MOM(LBM_D2Q9, float, LBM_FP32_PLAIN); break;
    case LBM_D3Q19 * 3 + LBM_FP32_SHIFTED: LBM_MOM(LBM_D3Q19, float, LBM_FP32_SHIFTED); break;
    case LBM_D3Q19 * 3 + LBM_FP64: LBM_MOM(LBM_D3Q19, double, LBM_FP64); break;
    case LBM_D3Q19 * 3 + LBM_FP32_PLAIN: LBM_MOM(LBM_D3Q19, float, LBM_FP32_PLAIN); break;
    }
#undef LBM_MOM
}

void launch_flush(int lattice, int precision, const DevMember* dm, const int2* work1, int nb1, int flip,
                  hipStream_t st)
{
    const dim3 blk(kBlock), grd(nb1);
    if (lattice == LBM_D2Q9) {
        if (precision == LBM_FP64) hipLaunchKernelGGL((k_flush<LBM_D2Q9, double>), grd, blk, 0, st, dm, work1, flip);
        else hipLaunchKernelGGL((k_flush<LBM_D2Q9, float>), grd, blk, 0, st, dm, work1, flip);
    } else {
        if (precision == LBM_FP64) hipLaunchKernelGGL((k_flush<LBM_D3Q19, double>), grd, blk, 0, st, dm, work1, flip);
        else hipLaunchKernelGGL((k_flush<LBM_D3Q19, float>), grd, blk, 0, st, dm, work1, flip);
    }
}

void launch_philox_test(const uint32_t* in, uint32_t* out, int n, hipStream_t st)
{
    hipLaunchKernelGGL(k_philox_test, dim3((n + 63) / 64), dim3(64), 0, st, in, out, n);
}

void launch_normals_test(unsigned long long seed, long long step0, int nsteps, int n, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_normals_test, dim3((nsteps + 63) / 64), dim3(64), 0, st, seed, step0, nsteps, n, out);
}

int lattice_table(int lattice, int* c, double* w)
{
    if (lattice == LBM_D2Q9) {
        using L = Lat<LBM_D2Q9>;
        for (int i = 0; i < L::Q; ++i) { c[3 * i] = L::cx[i]; c[3 * i + 1] = L::cy[i]; c[3 * i + 2] = L::cz[i]; w[i] = L::w[i]; }
        return L::Q;
    }
    using L = Lat<LBM_D3Q19>;
    for (int i = 0; i < L::Q; ++i) { c[3 * i] = L::cx[i]; c[3 * i + 1] = L::cy[i]; c[3 * i + 2] = L::cz[i]; w[i] = L::w[i]; }
    return L::Q;
}

}  // namespace lbm
#endif
