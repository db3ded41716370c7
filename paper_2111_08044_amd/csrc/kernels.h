// Launch wrappers of the HIP kernels (kernels.hip).  dtype: 0 = complex64,
// 1 = complex128.  All launches are asynchronous on stream s.
#pragma once
#include <hip/hip_runtime.h>

#include "fl_common.h"

namespace fl {

// pd's gates; chains in one workgroup (g.W = 0) apply them reps times in one
// launch, others take reps = 1 (also launch_adjoint)
hipError_t launch_sweep(int dtype, const fl_geom& g, void* psi, const void* gates, const fl_pass& pd, int reps,
                        hipStream_t s);
// bond reductions of shorter chains, one tile
hipError_t launch_rdm(int dtype, const fl_geom& g, const void* psi, const fl_pass& pd, double* partials, int nslot,
                      hipStream_t s);
// one pass of the bond reductions of chains from FL_RDM_MIN_WINDOWS sites on
hipError_t launch_rdm_windows(int dtype, const fl_geom& g, const void* psi, const rdm_desc& pd, double* partials,
                              int grid, int nslot, hipStream_t s);
hipError_t launch_finalize(const double* partials, int nblocks, int nvals, double* out, hipStream_t s);
// <H0> and the norm from finalized bond sums red[L*16] and FP64 bond terms h64[(L-1)*32]:
// out[0] = <H0>, out[1] = <psi|psi>; rdm (may be NULL) = [L-1][4][4] complex
hipError_t launch_energy_contract(const double* red, const double* h64, int L, double* out, double* rdm, hipStream_t s);
hipError_t launch_init(int dtype, void* psi, int L, const void* tabs, int a, int b, hipStream_t s);
hipError_t launch_overlap(int dta, const void* a, int dtb, const void* b, uint64_t n, double* partials, int grid,
                          hipStream_t s);
// one cover pass of H0 psi bond by bond, every entry of the terms as given:
// single-tile chains, and terms that are not Hermitian to rounding
hipError_t launch_apply_h(int dtype, const fl_geom& g, const void* psi, void* lam, const void* hmat, const fl_pass& pd,
                          int first, hipStream_t s);
// one cover pass of H0 psi on full tiles: `first` writes lambda, the others add to it
#define FL_HWIN_MAX 8       // windows per pass
#define FL_HWIN_REALS 52    // reals per window: the summed Hamiltonian of its bonds (layout: apply_h_window)
struct apply_h_desc {
    int32_t h, nwin, first;
    int32_t u0[FL_HWIN_MAX];   // first tile bit of each window; the last one >= 4
};
// tab: the pass's windows; dots: NULL, or per-workgroup sums [grid][4] of Re <psi|lambda>, 0, <psi|psi>,
// <lambda|lambda> (of the final lambda: the last pass)
hipError_t launch_apply_h_tiles(int dtype, const fl_geom& g, const void* psi, void* lam, const void* tab,
                                const apply_h_desc& pd, double* dots, int grid, hipStream_t s);
hipError_t launch_adjoint(int dtype, const fl_geom& g, void* psi, void* lam, const void* gates, const fl_pass& pd,
                          int reps, double* Mpart, int grid, hipStream_t s);
// reverse pass of the 4-qubit-window form (complex64, full 13-bit tiles) on
// the matrix cores: mats = the pass's window fragments (4 KiB per group, the
// transposes of the forward's), Qpart [grid][FL_WIN4_MAX_GROUPS][512]
// per-workgroup scratch, Qsum [pass groups][512] += the pass's window
// overlaps (Re, Im of 16x16)
hipError_t launch_adjoint_win4(const fl_geom& g, void* psi, void* lam, const void* mats, const fl_pass& pd,
                               double* Qpart, int grid, double* Qsum, hipStream_t s);
hipError_t launch_zero(double* p, uint64_t n, hipStream_t s);
// 4-qubit windows on FP32 MFMA; full tiles only (C + W = 13); mats: 4 KiB of fragments per window
hipError_t launch_dense4(const fl_geom& g, void* psi, const void* mats, const fl_pass& pd, hipStream_t s);
// mode 0: FP32 MFMA, 1: split-BF16x3 MFMA; mats: pre-arranged window matrices of the plan
hipError_t launch_dense6(int mode, const fl_geom& g, void* psi, const void* mats, const fl_pass& pd, hipStream_t s);

}  // namespace fl
