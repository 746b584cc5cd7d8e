// kernels3.hpp -- host-side launchers of the D3Q27 kernels (gfx950).
//
// Storage convention (as on D2Q9): plane i of a buffer holds the
// post-collision, not yet streamed populations g_i, so the observable state
// is f_i(x, t) = g_i(x - c_i) (periodic); a sweep pulls g_i(x - c_i) from one
// buffer, collides and stores g_i(x) into the other.  Shifted storage keeps
// g_i - w_i rho0.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "d3q27.hpp"
#include "plan3.hpp"

namespace oreg {

struct Geometry3 {
  int nx, ny, nz;
  int64_t cells;  // nx * ny * nz
};

// Workgroups of the diagnostics reduction (fixed, so the FP64 sums depend
// only on the box size).
constexpr int kDiag3Blocks = 1024;

// Wavefront tasks of one sweep: 64-node segments of every x-row.
int64_t sweep3_tasks(const Geometry3& g);

// One time step src -> dst.
hipError_t launch_sweep3(int eq, int coll, int st, const void* src, void* dst, const Geometry3& g,
                         const Coef64& c, hipStream_t s);

// OReg boxes whose buffers hold populations or ten numbers per node
// (march3.hip); *fmt says which (0: populations, 1: ten numbers).
// One time step src -> dst (ten numbers; sets *fmt_dst).
hipError_t launch_march3(int eq, int st, const void* src, void* dst, const unsigned int* fmt_src,
                         unsigned int* fmt_dst, const Geometry3& g, const Coef64& c,
                         const MarchShape& s, hipStream_t q);
// rho, ux, uy, uz into out[4][cells].
hipError_t launch_march3_moments(int eq, int st, const void* src, double* out,
                                 const unsigned int* fmt, const Geometry3& g, const Coef64& c,
                                 const MarchShape& s, hipStream_t q);
// The seven sums of lb3_diagnostics by workgroup, s.ntx s.nty s.nzc of them, into
// partials[][7].
hipError_t launch_march3_sums(int eq, int st, const void* src, double* partials,
                              const unsigned int* fmt, const Geometry3& g, const Coef64& c,
                              double theta_energy, const MarchShape& s, hipStream_t q);
// The populations of src into alt, if src holds ten numbers per node.
hipError_t launch_expand3(int eq, int st, const void* src, void* alt, const unsigned int* fmt,
                          const Geometry3& g, const Coef64& c, hipStream_t s);

// g from device FP64 fields [nz][ny][nx]; invalid nodes are counted in *bad.
// fmt (also below): the buffer's format flag, or null where a box always holds
// populations; alt holds the expanded populations when the flag is set.
hipError_t launch_init3(int eq, int st, const double* rho, const double* ux, const double* uy,
                        const double* uz, void* dst, const Geometry3& g, const Coef64& c,
                        unsigned int* bad, unsigned int* fmt, hipStream_t s);

// Plane i of pre-collision FP64 populations into a buffer.  Called in plane order
// for all 27, it counts invalid populations and nodes (a value that is not
// finite, a sum that is not positive) into *bad; sum[cells] is its workspace.
hipError_t launch_import3(int st, int i, const double* fin, void* dst, double* sum,
                          unsigned int* bad, const Geometry3& g, const Coef64& c, hipStream_t s);
// Plane i of them from a buffer.
hipError_t launch_export3(int st, int i, const void* src, const void* alt,
                          const unsigned int* fmt, double* fout, const Geometry3& g,
                          const Coef64& c, hipStream_t s);

// rho, ux, uy, uz into out[4][cells].
hipError_t launch_moments3(int st, const void* src, double* out, const Geometry3& g,
                           const Coef64& c, hipStream_t s);

// The seven FP64 sums of lb3_diagnostics into out[7]; partials holds
// kDiag3Blocks * 7 doubles.
hipError_t launch_diagnostics3(int st, const void* src, double* partials, double* out,
                               const Geometry3& g, const Coef64& c, double theta_energy,
                               hipStream_t s);
// Its second half: the sum of partials[n][7].
hipError_t launch_diagnostics3_final(const double* partials, int n, double* out, hipStream_t s);

}  // namespace oreg
