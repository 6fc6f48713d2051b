// Assembly, support masking, loads and the block-Jacobi preconditioner.
//
// Sec. 2.2.1: K is the sum of all element matrices placed by their index maps; supports enter
// through Lagrange multipliers with V u = b.  The same displacement follows from masking: a
// constrained DOF d gets K[d, :] = K[:, d] = 0, K[d, d] = 1 and f[d] = 0, and with prescribed
// values b a free row's load loses K(row, d) b[d] (lifting; u = b is written on d after the
// solve), which keeps K symmetric positive definite and its pattern unchanged.
//
// Assembly is gather-based and deterministic: a thread per two entries (slot, a, b) of a 6x6
// block sums the slot's element contributions in ascending contribution id (= ascending element, then
// ascending scalar index), with no atomics, so K is bitwise reproducible.  An entry below the
// diagonal (block (I, J) with J < I, or a > b in a diagonal block) sums the contributions of its
// transposed entry, (b, a) of block (J, I), in the same order: the element matrices are
// symmetric only up to rounding, and this makes K bitwise symmetric, which lets the PCG
// products read a lower block as the transpose of its mirror.
#include "sso_internal.h"

namespace sso {
namespace {

inline unsigned nblk(int64_t n, int tpb) { return (unsigned)((n + tpb - 1) / tpb); }


// K block values, row-major inside each 6x6 block, blocks in slot order: entries (a, b) and (a,
// b + 1), b even, a thread.  Contributions are taken four at a time, their loads in flight together
// (an inner block's corner has one, two or four): a thread an entry and one contribution after the
// other took 347 us for a 300 x 300 shell, 0.65 GB, and 16 for a 60 x 60 one, waiting for memory in
// a chain of up to eleven loads; this takes 225 and 12 (two at a time 209 and 14).
__global__ void __launch_bounds__(256)
k_assemble(Mesh m, int64_t n_blocks, const int32_t* __restrict__ bsrow,
           const int32_t* __restrict__ bcol, const int32_t* __restrict__ bseg,
           const int32_t* __restrict__ bperm, const int32_t* __restrict__ bsym,
           const double* __restrict__ coo, double* __restrict__ K) {
  constexpr int AT_ONCE = 4;
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= 18 * n_blocks) return;
  const int64_t s = t / 18;
  const int q = (int)(t - 18 * s), a = q / 3, b = 2 * (q - 3 * a);
  const int I = bsrow[s], J = bcol[s];
  // the upper triangle's entries whose values these take: themselves, or their transposes (in the
  // value slot: block (J, I) for J < I, the slot itself otherwise)
  const int64_t su = bsym[2 * s + 1];
  const int p0 = bseg[su], p1 = bseg[su + 1];
  const bool fa = m.fixed[6 * (int64_t)I + a] != 0;
  const bool f0 = fa || m.fixed[6 * (int64_t)J + b], f1 = fa || m.fixed[6 * (int64_t)J + b + 1];
  const bool low0 = J < I || (J == I && a > b), low1 = J < I || (J == I && a > b + 1);
  double v0 = 0.0, v1 = 0.0;
  for (int p = p0; p < p1; p += AT_ONCE) {
    int32_t c[AT_ONCE];
    double x0[AT_ONCE], x1[AT_ONCE];
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) c[k] = bperm[p + k < p1 ? p + k : p1 - 1];
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) {
      const BlockRef r = decode_block(c[k], m.n_beams);
      x0[k] = coo[low0 ? coo_index(r, b, a, m.n_beams) : coo_index(r, a, b, m.n_beams)];
      x1[k] = coo[low1 ? coo_index(r, b + 1, a, m.n_beams) : coo_index(r, a, b + 1, m.n_beams)];
    }
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k)
      if (p + k < p1) {
        v0 += x0[k];
        v1 += x1[k];
      }
  }
  if (f0) v0 = (I == J && a == b) ? 1.0 : 0.0;
  if (f1) v1 = (I == J && a == b + 1) ? 1.0 : 0.0;
  *reinterpret_cast<double2*>(K + 36 * s + 6 * a + b) = double2{v0, v1};
}

// f = f_nodal + sum over incident quads (ascending element) of -(gamma t + q) A / 4 on uz,
// masked.  The diagonal block slot of node I lists its incident elements in that order.
__global__ void k_loads(Mesh m, const int32_t* bdiag, const int32_t* bseg, const int32_t* bperm,
                        const double* qarea, double* f) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= 6 * (int64_t)m.n_nodes) return;
  int I = (int)(t / 6), c = (int)(t % 6);
  double v = m.f_nodal[t];
  if (c == 2 && (m.unit_weight != 0.0 || m.surface_load != 0.0)) {
    int s = bdiag[I];
    for (int p = bseg[s]; p < bseg[s + 1]; ++p) {
      BlockRef r = decode_block(bperm[p], m.n_beams);
      if (!r.quad) continue;
      double te = m.quad_prop[5 * (int64_t)r.e];
      v += -(m.unit_weight * te + m.surface_load) * qarea[r.e] / 4.0;
    }
  }
  f[t] = m.fixed[t] ? 0.0 : v;
}

// Prescribed support displacements b (Eq. 3 with b != 0) by lifting: the solve runs on
// u - b (b extended by 0 to the free DOFs), so f[t] = 0 on a constrained DOF (the masked row
// is the identity) and, on a free DOF t = 6 I + a, f[t] = fm[t] - sum over the slots of block
// row I (ascending) and components c of a constrained (J, c) of K(t, 6 J + c) b[6 J + c], with
// the unmasked entry summed from the element contributions in the assembly's order.  The
// solve keeps the constrained components at exactly 0 and solves K_ff u_f = f_f - K_fc b_c;
// k_apply_prescribed then writes u_c = b_c.
__global__ void k_lift(Mesh m, const int32_t* brow_ptr, const int32_t* bcol, const int32_t* bseg,
                       const int32_t* bperm, const double* coo, const double* fm, double* f) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= 6 * (int64_t)m.n_nodes) return;
  if (m.fixed[t]) {
    f[t] = 0.0;
    return;
  }
  const int I = (int)(t / 6), a = (int)(t % 6);
  double acc = 0.0;
  for (int s = brow_ptr[I]; s < brow_ptr[I + 1]; ++s) {
    const int64_t J = bcol[s];
    for (int c = 0; c < 6; ++c) {
      const int64_t d = 6 * J + c;
      if (!m.fixed[d] || m.u_presc[d] == 0.0) continue;
      double kv = 0.0;
      for (int p = bseg[s]; p < bseg[s + 1]; ++p) {
        const BlockRef r = decode_block(bperm[p], m.n_beams);
        kv += coo[coo_index(r, a, c, m.n_beams)];
      }
      acc += kv * m.u_presc[d];
    }
  }
  f[t] = fm[t] - acc;
}

__global__ void k_apply_prescribed(int64_t n, const uint8_t* fixed, const double* b, double* u) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < n && fixed[t]) u[t] = b[t];
}

__global__ void k_mask_vector(int64_t n, const uint8_t* fixed, const double* in, double* out) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= n) return;
  out[t] = fixed[t] ? 0.0 : in[t];
}

// Dinv_I = (K_II)^{-1} by Cholesky of the (masked, SPD) diagonal block, stored packed (upper
// triangle, dinv_index); entries (i, j) and (j, i) of W^T W are the same sum in the same order.
__global__ void k_block_jacobi(int n_nodes, const int32_t* bdiag, const double* K, double* Dinv,
                               float* Dinv32, unsigned* err) {
  int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= n_nodes) return;
  const double* A = K + 36 * (int64_t)bdiag[I];
  double L[6][6];
  bool ok = true;
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) L[i][j] = 0.0;
  for (int j = 0; j < 6; ++j) {
    double d = A[6 * j + j];
    for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
    if (!(d > 0.0)) {
      ok = false;
      d = 1.0;
    }
    L[j][j] = sqrt(d);
    for (int i = j + 1; i < 6; ++i) {
      double v = A[6 * i + j];
      for (int k = 0; k < j; ++k) v -= L[i][k] * L[j][k];
      L[i][j] = v / L[j][j];
    }
  }
  if (!ok) atomicOr(err, ERR_DIAG);
  // W = L^{-1} (lower triangular), then Dinv = W^T W
  double W[6][6];
  for (int i = 0; i < 6; ++i)
    for (int j = 0; j < 6; ++j) W[i][j] = 0.0;
  for (int j = 0; j < 6; ++j) {
    W[j][j] = 1.0 / L[j][j];
    for (int i = j + 1; i < 6; ++i) {
      double v = 0.0;
      for (int k = j; k < i; ++k) v -= L[i][k] * W[k][j];
      W[i][j] = v / L[i][i];
    }
  }
  double* out = Dinv + DINV_PACKED * (int64_t)I;
  for (int i = 0; i < 6; ++i)
    for (int j = i; j < 6; ++j) {
      double v = 0.0;
      for (int k = j; k < 6; ++k) v += W[k][i] * W[k][j];
      out[dinv_index(i, j)] = v;
      if (Dinv32) Dinv32[DINV_PACKED * (int64_t)I + dinv_index(i, j)] = (float)v;
    }
}

// Scalar CSR order of the block values (for read-back and parity checks).
__global__ void k_scalar_values(int n_nodes, const int32_t* brow_ptr, const double* K,
                                double* vals) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= 6 * (int64_t)n_nodes) return;
  int I = (int)(t / 6), a = (int)(t % 6);
  int rb = brow_ptr[I], nbc = brow_ptr[I + 1] - rb;
  int64_t rp = 36 * (int64_t)rb + 6 * (int64_t)a * nbc;
  for (int k = 0; k < nbc; ++k)
    for (int b = 0; b < 6; ++b) vals[rp + 6 * k + b] = K[36 * (int64_t)(rb + k) + 6 * a + b];
}

}  // namespace

hipError_t launch_assemble(const Mesh& m, const Pattern& pat, const double* coo, double* K,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_assemble, dim3(nblk(18 * pat.n_blocks, 256)), dim3(256), 0, s, m,
                     pat.n_blocks, pat.bsrow, pat.bcol, pat.bseg, pat.bperm, pat.bsym, coo,
                     K);
  return hipGetLastError();
}

hipError_t launch_loads(const Mesh& m, const Pattern& pat, const double* qarea, double* f,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_loads, dim3(nblk(6 * (int64_t)m.n_nodes, 256)), dim3(256), 0, s, m,
                     pat.bdiag, pat.bseg, pat.bperm, qarea, f);
  return hipGetLastError();
}

hipError_t launch_lift(const Mesh& m, const Pattern& pat, const double* coo, const double* fm,
                       double* f, hipStream_t s) {
  hipLaunchKernelGGL(k_lift, dim3(nblk(6 * (int64_t)m.n_nodes, 256)), dim3(256), 0, s, m,
                     pat.brow_ptr, pat.bcol, pat.bseg, pat.bperm, coo, fm, f);
  return hipGetLastError();
}

hipError_t launch_apply_prescribed(const Mesh& m, double* u, hipStream_t s) {
  const int64_t n = 6 * (int64_t)m.n_nodes;
  hipLaunchKernelGGL(k_apply_prescribed, dim3(nblk(n, 256)), dim3(256), 0, s, n, m.fixed,
                     m.u_presc, u);
  return hipGetLastError();
}

hipError_t launch_mask_vector(const Mesh& m, const double* in, double* out, hipStream_t s) {
  int64_t n = 6 * (int64_t)m.n_nodes;
  hipLaunchKernelGGL(k_mask_vector, dim3(nblk(n, 256)), dim3(256), 0, s, n, m.fixed, in, out);
  return hipGetLastError();
}

hipError_t launch_block_jacobi(const Mesh& m, const Pattern& pat, const double* K, double* Dinv,
                               float* Dinv32, unsigned* d_err, hipStream_t s) {
  hipLaunchKernelGGL(k_block_jacobi, dim3(nblk(m.n_nodes, 128)), dim3(128), 0, s, m.n_nodes,
                     pat.bdiag, K, Dinv, Dinv32, d_err);
  return hipGetLastError();
}

hipError_t launch_scalar_values(const Mesh& m, const Pattern& pat, const double* K, double* vals,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_scalar_values, dim3(nblk(6 * (int64_t)m.n_nodes, 256)), dim3(256), 0, s,
                     m.n_nodes, pat.brow_ptr, K, vals);
  return hipGetLastError();
}

}  // namespace sso
