// lbm_launch.h -- launch interface between the host library and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <vector>

#include "lbm_dev.h"

namespace lbm {

// One application of a QoI's kernel filter R (in device memory, one job per
// blockIdx.y and component): dst = R src through the intermediates y1 and y2
// (k_kxy, k_kz).  kind LBM_FILT_GAUSS: taps g_0 .. g_ra; LBM_FILT_LAPL: the
// dilated biharmonic l_0 .. l_ra, boxes of radius rb, times coef.  Pointers are
// device addresses in the member's arena.
struct KFil {
    int kind, ra, rb, ncomp;
    double coef;
    const void* taps;      // element type of the run
    const void* src;
    void* y1;
    void* y2;
    void* dst;
};

// Fourier band QoIs of a member (host side): the complex fields (nv components
// of v*, then nw of w) and their spectra; per slot of the inverse transform (a
// component of a QoI) its field, band and destination.  Plans are hipfftHandle
// values.
constexpr int kMaxSlots = 3 * kMaxSA;   // at most three components per QoI
struct FourierQ { int e, l, m; void* dst; };
struct FSlots {
    int n, field[kMaxSlots], l[kMaxSlots], m[kMaxSlots];
    void* dst[kMaxSlots];
};
struct FourierProg {
    void* plan[2];        // forward: the fields; inverse: the slots
    void* spec;           // [nv + nw][N] complex
    void* band;           // [slots][N] complex
    const void* vs;       // v* [D][N]
    int nx, ny, nz, nv, nw;
    FSlots slots;
    mutable int failed = 0;         // set when a hipFFT call of a launch fails
};

// One launch per kernel phase covers every member of a group: members share
// lattice, precision, substrate and mode, and are mapped to workgroups by
// the work tables.
struct LaunchGroup {
    int lattice, precision, substrate, mode;  // mode 0 plain, 1 plain + records, 2 TO
    int any_z, maxsa, maxe, maxz;   // most E/Z, E and Z QoIs of a member
    int cnl;            // binomial closures: powers of the chains (2 or 4)
    int btx;            // stream-collide tile width of every member (kBinTX or kBinTXW)
    const DevMember* mems;
    const int2* work1;  // cell kernels: (member, block of kBlock cells)
    int nb1;
    const int2* workp;  // the apply with the solve: (member, pair p of blocks 2p and 2p + 1)
    int nbp;
    const int2* workr;  // reduce: (member, y * nbx2 + bx)
    int nbr;
    const int2* workb;  // tiled stream-collide: (member, xyz tile)
    int nbb;
    const int2* workc;  // filter chains: (member, tile * (D + NC) + chain)
    int nbc;
    int pair;           // 2-D closures of at most one E and one Z QoI: k_chain_pair
    const int2* workq;  // its tiles: (member, tile)
    int nbq;
    const int2* works;  // cross-block sums: (member, value slot)
    int nbs;
    const int* workm;   // one workgroup per member
    int nmem;
    int probe;          // TO mode only: the QoI chain of the field already in v* (no
                        // stream-collide, no apply); see lbm_project_qoi
    int kf;             // kernel-filter or Fourier closure (one member per group)
    const KFil* kfil;   // kernel filters: nkfil jobs of the first application of R, then of
    int nkfil, krad;    // the second (device memory); their largest radius
    int kmem, kdim[3];  // the member and its grid
    const FourierProg* fprog;   // Fourier band QoIs (host memory; null if none)
    int wt;             // store the fields the next kernel reads through the L2 (small launches)
    int defer;          // TO mode: the SGS change is recorded and applied by the next step's pull (k_step_t)
    int a32;            // every member's population buffer spans less than 4 GiB (32-bit offsets)
    int nt;             // plain runs: the launch's populations exceed the Infinity Cache (non-temporal stores)
    int rag;            // rows of some member are not whole 128-byte lines (k_step_t: plain stores)
    int sep_solve;      // TO mode: the solve in its own launch (k_solve) even where k_apply could form it
};

// TO mode: the apply forms the solve itself (no k_solve launch): not for
// probe steps (no apply) or a forced own launch, and only where the apply's
// workgroups are all resident at once.
inline bool fused_solve(const LaunchGroup& g)
{
    return !g.probe && !g.sep_solve && g.nbp <= kFusedApplyPairs;
}

enum { OP_INIT = 0, OP_GET_POP = 1, OP_SET_POP = 2, OP_STREAM = 3 };

// ev (nullable): 7 events recorded at the phase boundaries of the step
// (start, after stream-collide, after the curl of kernel-filter closures,
// after the filters, after the reduce, after the cross-block sums and
// solve, after the apply).
constexpr int kNumPhases = 6;
void launch_step(const LaunchGroup& g, hipStream_t st, int flip, hipEvent_t* ev = nullptr);
void launch_state(int op, int lattice, int precision, const DevMember* dm, int N, bool has_to, int flip,
                  hipStream_t st, const double* a, double* b);
// Moments of the current state into vn, and (nullable) rho [N] and v [D][N]
// in double into rho_out and u_out.
void launch_fields(int lattice, int precision, const DevMember* dm, const int2* work1, int nb1, bool has_to,
                   int flip, hipStream_t st, double* rho_out, double* u_out = nullptr);
// The pending SGS change of deferring members added to their current
// populations g[parity ^ flip] and their records cleared (k_flush).
void launch_flush(int lattice, int precision, const DevMember* dm, const int2* work1, int nb1, int flip,
                  hipStream_t st);
void launch_philox_test(const uint32_t* in, uint32_t* out, int n, hipStream_t st);
void launch_normals_test(unsigned long long seed, long long step0, int nsteps, int n, double* out, hipStream_t st);
int lattice_table(int lattice, int* c, double* w);
// Projection of a fine member's state (coarse grid ncx x ncy x ncz; kind
// LBM_PROJ_STRIDE: the wall-anchored stride-m subsampling; LBM_PROJ_BICUBIC:
// the bicubic mean of a doubly periodic 2-D grid): full populations into
// fpop [Q][Nc] (nullable) and the post-collision velocity into vout [D][Nc]
// (nullable; double if vout_fp64).  tmp (nullable): device scratch of
// 2 * (ncy m) * ncx doubles, with which the bicubic velocity projection runs
// as two separable passes.
void launch_project(int lattice, int precision, const DevMember* fine, int flip, int m, int ncx, int ncy, int ncz,
                    double* fpop, void* vout, int vout_fp64, int kind, hipStream_t st, double* tmp = nullptr);

}  // namespace lbm
