// ktmi_spectra.hpp -- arguments and launcher of the smooth Cooper-Frye spectra
// kernels (ktmi_spectra.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "ktmi_device.hpp"
#include "ktmi_surface.hpp"

namespace ktmi {

// element slices summed by the fold kernel: at least 256 elements each up to
// kMinSlicesCap slices, and more where that leaves the chip idle
constexpr int kMinSlicesCap = 64, kMaxSlices = 512;

struct SpectraArgs {
  const double* elements;  // n surface records of kSurfRec doubles
  long n;
  double T, eps_plus_P;    // freeze-out temperature; e + P for delta f (0: none)
  int ns, nY, npt, nphi;
  long nbins;              // ns nY npt nphi
  const double* tables;    // mass, dof, stat, mu (ns each), Y, pT, cos phi, sin phi
  double far2;             // (u~^tau)^2 from which on an element's factors are not used
  double* partial;         // slices x nbins
  double* out;             // nbins
};

int spectra_min_slices(long n);           // fewest slices a call runs with
int spectra_slices(long n, long nbins);  // slices a workspace of the asked size holds
int launch_spectra(const SpectraArgs& a, int nslice, hipStream_t s);

}  // namespace ktmi
