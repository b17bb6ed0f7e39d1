// Mode-space COCG iteration (modal.hip): argument blocks and launchers.
#pragma once

#include "internal.h"

// Residuals kept per right-hand side between two replacements: a ring of as
// many vectors as fit the workspaces of the other iteration paths.
template <typename T> struct ModalRing;
template <> struct ModalRing<float> { static constexpr int n = 6; };
template <> struct ModalRing<double> { static constexpr int n = 5; };

// Planes per chunk of the mode pass (a power of two).
constexpr int kModalChunk = 8;

enum { MODAL_PART = 5 };  // values per block partial of the mode pass: rho, sigma, |r|^2

// Scalars of one right-hand side.  The plane pass of a step advances them
// from the last mode pass's partials; the mode pass reads them.
struct ModalScal {
  zd rho, sigma;          // r^T z and z^T q_old of the current residual
  zd rho_old, alpha_old;  // of the last step
  zd alpha;               // written by the mode pass of the step
  int step;               // index of the current residual since the last replacement
  int base;               // residuals before this one are folded into S and T
  int flag;               // breakdown
  int pad_;
};

// The nonlocal term as the plane pass adds it (kb.hip).
template <typename T>
struct KBPlane {
  int nu = 0, npad = 0;
  const int* uvox = nullptr;
  const int* uplane = nullptr;  // [nz + 1] first union voxel of each plane
  const int* prange = nullptr;
  const T* Bt = nullptr;        // [nproj][nu]
  const double* W = nullptr;    // [slot][2 npad] (h^3 D) B^T z
};

template <typename T>
struct PlaneArgs {
  int nz, nplanes, nmb, ndp;
  cplx<T>* vec;
  const int* active;
  const double* Vd;
  const float* Vf;
  ModalScal* sc;
  const double* part;
  double* dpart;
  zd* x = nullptr;
  const int* xset = nullptr;
  KBPlane<T> kb;
  bool pair = false;
};

template <typename T>
struct ModeArgsZ {
  int nz, nx, nxy, nmb, ndp;
  cplx<T>* ring[ModalRing<T>::n];
  cplx<T>* w;
  const cplx<T>* ft;
  const int* e_rhs;
  const int* active;
  ModalScal* sc;
  double* part;         // [rhs][nmb][MODAL_PART]
  const double* dpart;  // [rhs][ndp][2] z^T V z
  zd *ha, *hb;          // [rhs][ring] alpha and beta of the steps in the ring
  cplx<T>*fold_s, *fold_t;
  long long fold_stride;
  bool pair;
};

// Device state of a batch.
template <typename T>
struct Modal {
  int nE = 0;              // mode-table entries
  int nmb = 0;             // mode blocks of the mode pass (modal_mode_blocks)
  int ndp = 0;             // partials of z^T V z per rhs (planes, nonlocal term)
  cplx<T>* ring[ModalRing<T>::n];
  cplx<T>* w = nullptr;    // Z and W, in turn
  cplx<T>* ft = nullptr;   // filter table [nE][3 nf + nf^2][mode]
  const int* e_rhs = nullptr;
  ModalScal* sc = nullptr;
  double* part = nullptr;
  double* dpart = nullptr;
  zd *ha = nullptr, *hb = nullptr;
  cplx<T>*fold_s = nullptr, *fold_t = nullptr;  // folded direction and correction, per rhs at fold_stride
  long long fold_stride = 0;
  // pairs at a lateral Bloch vector (complex64, square register-FFT planes):
  // right-hand sides 2k (primary) and 2k + 1 (shadow), listed together
  bool pair = false;
};

int modal_mode_blocks(iobm_ctx c);
// the filter table for the context's current mode table
template <typename T>
hipError_t modal_setup(iobm_ctx c, Modal<T>& M);
// (re)start the listed rhs from the real-space residual in ring slot 0
template <typename T>
hipError_t modal_start(iobm_ctx c, const Modal<T>& M, int nact, const int* active);
// one iteration of the listed rhs; fold: the ring of some may be full after it
// (the kernels check which, so that true is always right)
template <typename T>
hipError_t modal_step(iobm_ctx c, const Modal<T>& M, int nact, const int* active, bool fold);
// x += d (x written without being read where xset = 0); ring_reads and nfirst
// are for the timing hook's byte count
template <typename T>
hipError_t modal_correct(iobm_ctx c, const Modal<T>& M, zd* x, const int* xset, int nact, const int* active,
                         double ring_reads, int nfirst);
// forget the steps of the listed rhs since the last replacement (their
// correction is then zero)
template <typename T>
hipError_t modal_drop(iobm_ctx c, const Modal<T>& M, int nact, const int* active);
// |r|^2 and breakdown flags of the listed rhs
template <typename T>
hipError_t modal_check(iobm_ctx c, const Modal<T>& M, int nact, const int* active, double* rn2, int* flag);

// kb.hip: projector sums of x, W = (h^3 D) B^T x, and C^T W to dz[rhs dzs]
template <typename T>
hipError_t launch_kb_coeffs(iobm_ctx c, const cplx<T>* x, int nrhs, const int* active, double* dz, long long dzs,
                            KBPlane<T>* out);
