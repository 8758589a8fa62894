// The update of one cell, shared by every kernel that collides cells
// (collide.hip: one step over the lattice; pair.hip: two steps in one pass and
// the cells around the foils between them): the IBM velocity correction, Guo
// forcing and BGK relaxation, and the force reduction of a step with foils.
#pragma once

#include "lattice_dev.h"

namespace ibmk {

// True if (x, y) lies in the node box of foil w.
__device__ __forceinline__ bool in_box(const FoilBox& b, int x, int y) {
  return y >= b.y0 && y < b.y0 + b.h && x >= b.x0 && x < b.x0 + b.w;
}

// The IBM correction at a cell.
struct Correction {
  float x = 0.f, y = 0.f, z = 0.f;
  bool hit = false;                                    // a support node (else zero)
};

// Whether (x, y) is a support node of foil b's markers, from the step's bitmap
// over its node box.
__device__ __forceinline__ bool support_node(const FoilBox& b, int x, int y) {
  if (!in_box(b, x, y)) return false;
  const int lx = x - b.x0, ly = y - b.y0;
  return (gmem(b.bits)[ly * b.words + (lx >> 5)] >> (lx & 31)) & 1u;
}

// du(x) of one foil (Eq. 15) from the 4 span layers within reach of the layer
// images `img` written by the spread kernel: their records, and their sum
// added to c.
typedef float f4 __attribute__((ext_vector_type(4)));   // one 16-byte load per record
__device__ __forceinline__ void correction_load(const Geo& g, const FoilBox& b, const float4* img, int x, int y, int z,
                                                f4 v[4]) {
  const auto* p = gmem(reinterpret_cast<const f4*>(img));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int s = z - 2 + k;
    s = s < 0 ? s + g.nz : (s >= g.nz ? s - g.nz : s);
    s = s < 0 ? s + g.nz : s;                          // a span of one layer wraps twice
    v[k] = p[((long long)s * b.side + (y - b.y0)) * b.side + (x - b.x0)];
  }
}
__device__ __forceinline__ void correction_add(const float wz[4], const f4 v[4], Correction& c) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c.x = __builtin_fmaf(wz[k], v[k].x, c.x);
    c.y = __builtin_fmaf(wz[k], v[k].y, c.y);
    c.z = __builtin_fmaf(wz[k], v[k].z, c.z);
  }
  c.hit = true;
}

// Sum over the foils at cell (x, y, z) of step `a`'s correction.
__device__ __forceinline__ Correction correction(const Geo& g, const CollideArgs& a, int x, int y, int z) {
  Correction c;
  for (int w = 0; w < a.nw; ++w) {
    const FoilBox& b = a.box[w];
    if (y < b.y0 || y >= b.y0 + b.h) continue;         // wave-uniform: most rows miss
    if (!support_node(b, x, y)) continue;              // zero there
    f4 v[4];
    correction_load(g, b, b.corr, x, y, z, v);
    correction_add(a.wz, v, c);
  }
  return c;
}

// Post-collision values of cell (x, y, z) from its pulled ones, in place: the
// Zou-He rebuild at the x faces (ZH: the solve has Zou-He faces), moments,
// IBM velocity correction and Guo forcing, BGK relaxation.  Returns the
// density deviation of the pre-collision state.
// `g` and `ph` are the solve's (the same at every step), `a` the step's arguments.
// Everything is computed in stored units
// (kS f~): the moments, the equilibrium (Eq. 4, with rho scaled) and the
// Guo term (Eq. 8, with F scaled) are linear in the distributions, and kS is
// a power of two, so the result is the same as in units of f~.
// Every operation and every fused multiply-add is written out and the
// compiler's own contraction is off: a cell gets the same bits in whatever
// kernel updates it, which a solve stepped in other portions, in a group or
// from a checkpoint relies on.
//
// The IBM correction is fetched here after the moments, or, EARLY, by the
// caller (`c`) while the pull is in flight.
template <class St, bool IBM, bool FORCE, bool ZH, bool EARLY>
__device__ __forceinline__ float update_cell(const Geo& g, const Phys& ph, const CollideArgs& a, int x, int y, int z,
                                             float f[kQ], Correction c = Correction()) {
#pragma clang fp contract(off)
  constexpr float kS = St::kS, kInv = St::kInv;
  if constexpr (ZH) {
    // Zou-He x faces: rebuild the entering populations at the face lanes
    // (the rule of zou_he, each face's branch on its own so the rest of
    // the row keeps f in registers)
    if ((g.yper || (y > 0 && y < g.ny - 1)) && (g.zper || (z > 0 && z < g.nz - 1))) {
      if (x == 0 && g.bclo >= BC_ZH_VELOCITY) zou_he_face<St, true, 1>(ph, g.bclo, f);
      if (x == g.nx - 1 && x != 0 && g.bchi >= BC_ZH_VELOCITY) zou_he_face<St, true, -1>(ph, g.bchi, f);
    }
  }
  float dr, jx, jy, jz;                            // kS drho, kS j
  moments19(f, dr, jx, jy, jz);
  const float drho = dr * kInv;
  const float rho = 1.0f + drho;
  const float srho = kS * rho;
  const float inv = 1.0f / srho;
  float Fx = 0.f, Fy = 0.f, Fz = 0.f;                // kS F
  if (FORCE) {
    Fx = kS * ph.fb[0]; Fy = kS * ph.fb[1]; Fz = kS * ph.fb[2];
    jx += 0.5f * Fx; jy += 0.5f * Fy; jz += 0.5f * Fz;   // (the halves are exact)
  }
  float ux = jx * inv, uy = jy * inv, uz = jz * inv;
  bool forced = FORCE;
  if (IBM) {
    if (!EARLY) c = correction(g, a, x, y, z);
    if (c.hit) {
      ux += c.x; uy += c.y; uz += c.z;                 // Eq. 16
      const float r2 = 2.0f * srho;                    // Eq. 11 / Eq. 26
      Fx = __builtin_fmaf(r2, c.x, Fx);
      Fy = __builtin_fmaf(r2, c.y, Fy);
      Fz = __builtin_fmaf(r2, c.z, Fz);
      forced = true;
    }
  }
  // (which of two products is rounded on its own follows the kernels' first
  // form, here and below, so that results stay those of earlier builds)
  const float usq = __builtin_fmaf(uz, uz, IBM ? __builtin_fmaf(uy, uy, ux * ux) : __builtin_fmaf(ux, ux, uy * uy));
  const float om = ph.omega;
  // Equilibrium (Eq. 4) by opposite pairs: with cu_opp = -cu, the even part
  // w (drho + rho (4.5 cu^2 - 1.5 u^2)) is shared and the odd part 3 w rho cu
  // changes sign, so each pair costs one evaluation
  const float c15 = 1.5f * usq;
  const float k1[2] = {wq(1) * srho, wq(7) * srho}, k3[2] = {3.0f * wq(1) * srho, 3.0f * wq(7) * srho},
              kd[2] = {wq(1) * dr, wq(7) * dr};
  const float e0 = __builtin_fmaf(wq(0), dr, -(wq(0) * srho * c15));
  f[0] = __builtin_fmaf(-om, f[0] - e0, f[0]);
  // c_i . u of a diagonal, without the rounding of one of its two products
  // j inv where the velocity is just that (no IBM correction)
  auto diagonal_cu = [&](int i) {
    if (IBM || i < 7) return cdot(i, ux, uy, uz);
    switch (i) {
      case 7: return FORCE ? __builtin_fmaf(jx, inv, uy) : __builtin_fmaf(jy, inv, ux);
      case 9: return FORCE ? __builtin_fmaf(jx, inv, -uy) : __builtin_fmaf(-jy, inv, ux);
      case 11: return __builtin_fmaf(jz, inv, ux);
      case 13: return FORCE ? __builtin_fmaf(-jz, inv, ux) : __builtin_fmaf(jx, inv, -uz);
      case 15: return FORCE ? __builtin_fmaf(jz, inv, uy) : __builtin_fmaf(jy, inv, uz);
      default: return FORCE ? __builtin_fmaf(-jz, inv, uy) : __builtin_fmaf(jy, inv, -uz);
    }
  };
#pragma unroll
  for (int i = 1; i < kQ; ++i) {
    if (oppq(i) < i) continue;
    const int c = i < 7 ? 0 : 1;                       // axis or diagonal weight
    const float cu = diagonal_cu(i);
    const float A = __builtin_fmaf(k1[c], __builtin_fmaf(cu, 4.5f * cu, -c15), kd[c]);
    const float fp = __builtin_fmaf(k3[c], cu, A);     // feq of i and of opp(i)
    const float fm = __builtin_fmaf(-k3[c], cu, A);
    f[i] = __builtin_fmaf(-om, f[i] - fp, f[i]);
    f[oppq(i)] = __builtin_fmaf(-om, f[oppq(i)] - fm, f[oppq(i)]);
  }
  if (forced) {                                        // Eq. 8
    const float k = ph.guo_k;
    const float uF = __builtin_fmaf(uz, Fz, IBM ? __builtin_fmaf(uy, Fy, ux * Fx) : __builtin_fmaf(ux, Fx, uy * Fy));
    f[0] = __builtin_fmaf(k * wq(0), 3.0f * (0.f - uF), f[0]);
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
      const float cF = cdot(i, Fx, Fy, Fz);
      float gi;
      if (i < 7) {
        gi = __builtin_fmaf(3.0f, cF - uF, 9.0f * cdot(i, ux, uy, uz) * cF);
      } else {
        const float cu = IBM || oppq(i) > i ? diagonal_cu(i) : (i == 10 ? __builtin_fmaf(jy, inv, -ux) : -diagonal_cu(oppq(i)));
        gi = __builtin_fmaf(9.0f * cu, cF, 3.0f * (cF - uF));
      }
      f[i] = __builtin_fmaf(k * wq(i), gi, f[i]);
    }
  }
  return drho;
}

// Pre-collision values of cell (x, y, z) on a wave-uniform row, in stored
// units: the scalar-base pull where no y or z wall reflects into the row.
template <class St>
__device__ __forceinline__ void pull_row(const typename St::T* __restrict__ S, const Geo& g, int x, int y,
                                         int z, float f[kQ]) {
  if (pull_rows_inside(g, y, z))
    pull19_rows<St>(S, g, x, y, z, f);
  else
    pull19<St, true>(S, g, x, y, z, f);
}

// Streaming store of a cell's post-collision values (stored units) and, at
// x = 0 / nx-1, the ghost layer of the state being written.
template <class St>
__device__ __forceinline__ void store_cell(typename St::T* __restrict__ D, const Geo& g, const Phys& p, int x,
                                           int y, int z, float o[kQ]) {
  using T = typename St::T;
  T* own = D + rowbase(g, y, z);
  if constexpr (sizeof(T) == 2) {
    // 16-bit storage: one buffer descriptor over the cell row's 19
    // population rows, so each store takes its row as a scalar offset and
    // the lane's x as the vector offset, with no per-store address
    // arithmetic (FP32 measured faster with plain stores)
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(own, 0, (int)(kQ * g.ps * (long long)sizeof(T)), kRawBufferWord3);
    const int bo = x * (int)sizeof(T);
#pragma unroll
    for (int i = 0; i < kQ; ++i) St::stb(rs, bo, (int)(i * g.ps * (long long)sizeof(T)), o[i]);
  } else {
#pragma unroll
    for (int i = 0; i < kQ; ++i) St::stnr(own + (long long)i * g.ps + x, o[i]);
  }
  if (x == 0 || x == g.nx - 1) {
#pragma unroll
    for (int i = 0; i < kQ; ++i) o[i] *= St::kInv;
    write_ghosts<St>(D, g, p, x, y, z, o);
  }
}

// After the marker kernels of step `a`, one wave per foil w: the sum over span
// layers of the layer forces and moments, the coefficients (Sec. 3.6-3.7: lift
// is the lateral component, counted outward for a mirrored pair; thrust is
// -F_x; drag = -thrust) and the history row.  The order is fixed: 256 partial
// sums over the layers t, t + 256, ..., of which a lane holds four, then halves
// added to halves.  In registers and lane shuffles, as a block of 256 threads
// with the partial sums in LDS took 4 us, most of it barriers: the smallest
// solves waited for it (collide 64x48x8 with two foils 9.4 -> 7.7 us).  (A
// block of its own for it, no faster, made the 16-bit collide of 160x128x128
// 5% slower.)
__device__ __forceinline__ void reduce_forces(const CollideArgs& a, int w, int lane) {
  const auto* fp = gmem(a.fpart) + 4 * (size_t)w * a.g.nz;
  double F[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int q = 0; q < 2; ++q) {                        // partial sums q and q + 2 of the lane
    double v[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[j][k] = 0.0;
      for (int l = lane + 64 * q + 128 * j; l < a.g.nz; l += 256)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[j][k] += fp[4 * l + k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) F[k] = q == 0 ? v[0][k] + v[1][k] : F[k] + (v[0][k] + v[1][k]);
  }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) F[k] += __shfl_down(F[k], h);
  if (lane == 0) {
    double* h = a.hist + ((size_t)a.hist_row * a.nw + w) * 8;
    h[0] = F[0];
    h[1] = F[1];
    h[2] = F[2];
    h[3] = F[3];
    h[4] = -a.sense[w] * F[1] / a.qS;
    h[5] = -F[0] / a.qS;
    h[6] = F[0] / a.qS;
    h[7] = F[3] / (a.qS * a.chord[w]);
  }
}

}  // namespace ibmk
