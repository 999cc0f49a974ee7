// Internal declarations of the PM library: context, workspace layout and the
// launchers of the HIP kernels.  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "batch.h"
#include "layout.h"
#include "pm.h"

namespace pmk {

// A real N^3 mesh in the x-blocked layout (layout.h), stored so that its
// r2c transform fits in place:
//   real view    r[N/8][N][N][8]       (float)
//   complex view c[N/8][N][N/2][8]     (float2, same bytes, kz = 0 .. N/2-1)
//   Nyquist plane q[N/8][N][8]         (float2, kz = N/2)
struct Field {
  float* r = nullptr;
  float2* q = nullptr;
  float2* c() const { return reinterpret_cast<float2*>(r); }
};

// Device tables of one FFT size N.
struct FftTables {
  int n = 0;
  float2* tw_n = nullptr;   // exp(-2 pi i k / N), k in [0, N)
  float2* tw_h = nullptr;   // exp(-2 pi i k / (N/2)), k in [0, N/2)
  // FD kernel tables (float32 from float64):  x/y axes use the signed
  // frequency of numpy's fftfreq, the z axis k in [0, N/2].
  float* dxy = nullptr;     // D(w)  = (8 sin w - sin 2w) / 6
  float* kxy = nullptr;     // K1(w) = (2 sin(w/2))^2
  float* wxy = nullptr;     // sinc^2(w/2)  (CIC window per axis)
  float* sxy = nullptr;     // exp(-w^2 rs^2) (split filter per axis)
  float* dz = nullptr;
  float* kz = nullptr;
  float* wz = nullptr;
  float* sz = nullptr;
};

// Spectral multiplication applied between the forward and the inverse x
// transforms of the fused x pass.
// Fan-out kinds read one input spectrum and write n_out outputs; fan-in
// kinds (the transposes, used by the adjoint) read n_in inputs and write the
// sum of their conjugate-multiplied spectra to one output; they overwrite
// their inputs.
enum SpecOpKind : int {
  OP_IDENTITY = 0,   // 1 output: X (round trip, scaled)
  OP_FORCE = 1,      // 3 outputs: i D_d g X with g = scale W^-n S / K^2
  OP_LPT1 = 2,       // 9 outputs from delta_L = X * pk[n^2]: s1 (3), phi_ij (6)
  OP_LPT2 = 3,       // 3 outputs: -i D_d / K^2 X * scale
  OP_LINEAR = 4,     // 1 output: X * pk[n^2]
  OP_LPT_PHI = 5,    // 6 outputs: phi_ij of delta_L = X * pk[n^2] (xx, yy, zz, xy, xz, yz)
  OP_FORCE_XS = 6,   // 2 outputs after the x pass, g = scale W^-n S / K^2: i D_x g X (F_x) and i g X,
                     // the factor F_y and F_z share until their y and z passes
  OP_FORCE_T = 16,   // fan-in 3: sum_d conj(i D_d g) X_d
  OP_LPT2_T = 17,    // fan-in 3: sum_d conj(-i D_d scale / K^2) X_d
  OP_LPT1_T = 18,    // fan-in 9: pk[n^2] (sum_d conj(i D_d / K^2) X_d + sum_ij D_i D_j / K^2 X_ij)
};

inline bool op_fan_in(int kind) { return kind >= 16; }

constexpr int kMaxOut = 9;

struct SpecOp {
  int kind = OP_IDENTITY;
  int n_out = 1;
  int n_in = 1;
  float scale = 1.f;
  int deconv = 0;
  int split = 0;
  const float* pk = nullptr;  // table indexed by integer |n|^2
  float2* out_c[kMaxOut] = {};
  float2* out_q[kMaxOut] = {};
  // fan-in inputs (forward y transformed); the op consumes them: the first
  // input of the lowest D(w_x) power holds partial sums between launches
  float2* in_c[kMaxOut] = {};
  float2* in_q[kMaxOut] = {};
};

// ---- FFT launchers (fft.hip) ---------------------------------------------
// Forward r2c: z pass (real -> complex + Nyquist plane), then y pass.
// (gate: a BatchArg whose one descriptor, of member 0 or skipped, lets the
// launches run or return at once)
void fft_r2c_zy(const FftTables& t, Field* f, int nf, hipStream_t s, const BatchArg& gate = BatchArg());
// Fused x pass: forward x transform of `in`, spectral op, inverse x
// transforms written to op.out_*.  `in` may alias out[0].
void fft_x_fused(const FftTables& t, const Field& in, const SpecOp& op, hipStream_t s);
// The force's x pass in one launch: forward x transform of `in`, times the
// Green's function, inverse x transforms into op.out_* (OP_FORCE_XS: out[0] =
// F_x, which may alias `in`, out[1] = the factor F_y and F_z share).
// Batched launches (bat.d != null) cover every member of a plan, as do the
// batched forms of the passes below.
void fft_x_force(const FftTables& t, const Field& in, const SpecOp& op, hipStream_t s,
                 const BatchArg& bat = BatchArg());
// Inverse y pass of the three force meshes after an OP_FORCE_XS x pass:
// f[0] holds F_x, f[2] the shared factor i g X.  f[2] becomes F_z times
// D(w_z) in place and f[1] receives F_y = transform of D(w_y) i g X; one
// read of the shared factor feeds both.
// (64^3 and larger meshes; up to kPlaneMax the plane passes below take its
// place and that of the z passes)
void fft_y_force(const FftTables& t, Field* f, hipStream_t s, const BatchArg& bat = BatchArg());
// x pass of the transposed force (OP_FORCE_T: op.scale, deconv, split) over
// the forward-(z, y) spectra f[0..2] of its x, y, z inputs; the result (the
// fan-in, inverse-x transformed) replaces f[0].
void fft_x_force_t(const FftTables& t, Field* f, const SpecOp& op, hipStream_t s, const BatchArg& gate = BatchArg());
// Single passes (the composites above call these).
void fft_z_r2c(const FftTables& t, Field* f, int nf, hipStream_t s, const BatchArg& bat = BatchArg());
void fft_y(const FftTables& t, Field* f, int nf, int dir, hipStream_t s, const BatchArg& bat = BatchArg());
void fft_z_c2r(const FftTables& t, Field* f, int nf, hipStream_t s);
// z pass of three fields written as one interleaved real mesh
// out[x/8][y][z][x%8][3] (the force meshes the particle readout gathers from).
// The three fields must be equally spaced in memory (f[2] - f[1] == f[1] - f[0]
// for both the arrays and the Nyquist planes), as the workspace meshes are.
void fft_z_c2r_interleaved3(const FftTables& t, const Field* f, float* out, hipStream_t s,
                            const BatchArg& bat = BatchArg());

// Force passes of meshes up to kPlaneMax cells per side: in.r to the spectrum
// after z and y in `out` (another field), and F_x in f[0], the shared factor
// in f[2] (after fft_x_force) to the interleaved mesh.
constexpr int kPlaneMax = 32;
void fft_plane_forward(const FftTables& t, const Field& in, const Field& out, hipStream_t s,
                       const BatchArg& bat = BatchArg());
void fft_plane_force(const FftTables& t, const Field* f, float* out, hipStream_t s, const BatchArg& bat = BatchArg());
// Inverse: y pass then z pass (complex + Nyquist plane -> real), unnormalised.
void fft_c2r_yz(const FftTables& t, Field* f, int nf, hipStream_t s, const BatchArg& gate = BatchArg());

// z stages of the LPT initial conditions, fused with what they feed: the six
// z spectra of the potential's second derivatives (xx yy zz xy xz yz) to the
// z spectrum of delta2, and the displacements' z spectra to particles
struct LptParticleArgs;
void launch_lpt_delta2(const FftTables& t, const Field* phi, const Field& out, hipStream_t s);
void launch_lpt_particles(const FftTables& t, const LptParticleArgs& a, hipStream_t s);
// z passes whose real side is a caller's plain [x][y][z] mesh (16-byte aligned).
void fft_z_r2c_std(const FftTables& t, const float* in, const Field& f, hipStream_t s);
void fft_z_c2r_std(const FftTables& t, const Field& f, float* out, hipStream_t s);
// x passes whose spectral side is a caller's numpy-layout half spectrum
// [kx][ky][kz], kz = 0 .. N/2: forward to it, inverse of scale times it.
void fft_x_forward_np(const FftTables& t, const Field& f, float2* spec, hipStream_t s);
void fft_x_inverse_np(const FftTables& t, const float2* spec, const Field& f, float scale, hipStream_t s);

// Binned power spectrum of a field whose z and y transforms are done: forward
// x transform and binning in one pass.  out holds per bin j = 1 .. n_bins the
// number of modes, the sum of |n| and the sum of |X|^2, n_bins values each.
struct PowerArgs {
  int n_bins = 0;
  int n_max = 0;                 // > 0: only modes with every |n_d| < n_max
  int deconv = 0;                // divide |X|^2 by the CIC window squared
  const float2* c = nullptr;
  const float2* q = nullptr;
  const float* wxy = nullptr;
  const float* wz = nullptr;
  double* partial = nullptr;     // power_partial_doubles(n_bins) of scratch
  double* out = nullptr;
};
long power_partial_doubles(int n_bins);
void launch_power(const FftTables& t, const PowerArgs& a, hipStream_t s);

}  // namespace pmk
