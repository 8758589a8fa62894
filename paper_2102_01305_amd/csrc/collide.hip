// gfx950 lattice kernels of the D3Q19 BGK + implicit-IBM time step.
//
//  collide   fused pull-streaming, moments, IBM velocity correction, Guo
//            forcing and BGK relaxation over every cell (Eqs. 1-11, 16, 26);
//            rebuilds the entering populations of Zou-He face cells where a
//            solve has such faces; writes the x-face ghost layer of the next
//            state; on steps with foils, block 0 makes the fixed-order force
//            sum and the coefficients.
//  ghost     the same ghost rule for a freshly initialised state.
//  init_eq   equilibrium initial state from rho, u.
//  moments   rho and velocity of every cell (read-back).
//  mass      fixed-order sum of the per-block mass partials.
//
// Distributions are stored as deviations from the lattice weights,
// f~_i = f_i - w_i, so FP32 (and 16-bit) storage keeps the small velocity
// signal out of the rounding of the O(w_i) rest value.
#include "update_dev.h"

namespace ibmk {

// ---------------------------------------------------------------- collide --

// One cell update: pull-streaming, the update of the cell, streaming store of
// the post-collision values and, at x = 0 / nx-1, the ghost layer of the next
// state.  Returns the density deviation of the pre-collision state.
template <class St, bool IBM, bool FORCE, bool ZH>
__device__ __forceinline__ float collide_cell(const CollideArgs& a, const typename St::T* __restrict__ S,
                                              typename St::T* __restrict__ D, int x, int y, int z) {
  float f[kQ];
  pull_row<St>(S, a.g, x, y, z, f);
  // IBM correction: with Zou-He faces it is fetched while the pull is in
  // flight (measured faster there), else after the moments
  Correction c;
  if (IBM && ZH) c = correction(a.g, a, x, y, z);
  const float drho = update_cell<St, IBM, FORCE, ZH, ZH>(a.g, a.p, a, x, y, z, f, c);
  store_cell<St>(D, a.g, a.p, x, y, z, f);
  return drho;
}

// Every cell, one row per wave, 64 cells along x per wave, 4 waves per block.
template <class St, bool IBM, bool FORCE, bool CHECK, bool ZH>
__device__ __forceinline__ void collide_block(const CollideArgs& __restrict__ a, int lb,
                                              const void* src, void* dst) {
  using T = typename St::T;
  const Geo& g = a.g;
  const T* __restrict__ S = static_cast<const T*>(src);
  T* __restrict__ D = static_cast<T*>(dst);
  // the first block reduces the step's forces on its way, a wave per foil
  if (IBM && lb == 0)
    for (int w = (int)threadIdx.y; w < a.nw; w += kBlockRows) reduce_forces(a, w, (int)threadIdx.x);
  // Waves to (64-cell chunk, row).  FP32: a block is one chunk of 4
  // consecutive rows (tiles in XCD runs, below).  16-bit storage: waves run along x first, so the
  // chunks of a row sit in one block and the cache line each chunk shares
  // with its neighbour (the x -/+ 1 pulls) is fetched from memory once; at
  // 2 bytes a wave reads a single line per population row, so these shared
  // lines are a large part of its reads.
  int xc, row;
  if (sizeof(T) == 2) {
    const int gw = __builtin_amdgcn_readfirstlane(lb * kBlockRows + (int)threadIdx.y);
    row = a.nxc_mul ? (int)__umulhi((unsigned)gw, a.nxc_mul) : gw / a.nxc;
    xc = gw - row * a.nxc;
  } else {
    // Workgroups are dealt to the 8 XCDs in turn; a single solve's tiles are
    // reordered so that each XCD takes runs of 4 block rows (all chunks of
    // 16 lattice rows; 8 block rows where a row has 8 or more chunks,
    // measured faster there: 512x384x384 -1.1%, 256-cell rows +0.3%), and
    // the cache lines two chunks of a row share are fetched by one L2.
    // Bijective on the tiles; grouped launches keep the plain order.
    int lt = lb;
    const int G = (a.nxc >= 8 ? 8 : 4) * a.nxc;
    // (M from gridDim, which loads beside the arguments' address: from nblocks,
    // its load came behind a branch, 0.2 us more a launch)
    const int M = (int)(gridDim.x / (8 * G)) * 8 * G;
    if (lt < M && (int)gridDim.x == a.nblocks) {
      const int xcd = lt & 7, k = lt >> 3;
      lt = ((k / G) * 8 + xcd) * G + k % G;
    }
    xc = lt % a.nxc;
    row = (lt / a.nxc) * kBlockRows + (int)threadIdx.y;
  }
  const int x = xc * kBlockX + threadIdx.x;
  // one row per wave: make the row index wave-uniform for the compiler
  row = __builtin_amdgcn_readfirstlane(row);
  const bool active = x < g.nx && row < g.ny * g.nz;
  double dm = 0.0;
  bool bad = false;
  if (active) {
    const int z = __builtin_amdgcn_readfirstlane(
        sizeof(T) == 2 && a.ny_mul ? (int)__umulhi((unsigned)row, a.ny_mul) : row / g.ny);
    const int y = __builtin_amdgcn_readfirstlane(row - z * g.ny);
    const float drho = collide_cell<St, IBM, FORCE, ZH>(a, S, D, x, y, z);
    if (CHECK) {
      dm = (double)drho;
      bad = !isfinite(drho);
    }
  }
  if (CHECK) {
    // wave reduction, then 4 waves through LDS, fixed order
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dm += __shfl_xor(dm, off);
    __shared__ double part[kBlockRows];
    if (threadIdx.x == 0) part[threadIdx.y] = dm;
    if (bad) atomicOr(a.flags, 1);
    __syncthreads();
    if (threadIdx.x == 0 && threadIdx.y == 0) {
      double s = 0.0;
      for (int r = 0; r < kBlockRows; ++r) s += part[r];
      a.mass_part[lb] = s;
    }
  }
}

// A grouped collide launch also carries each solve's state buffers as
// kernel arguments, so the compiler knows they are global memory.
struct CollideGroup {
  Group g;
  const void* src[kMaxGroup];
  void* dst[kMaxGroup];
};

template <class St, bool IBM, bool FORCE, bool CHECK, bool ZH>
__global__ void __launch_bounds__(kBlockX * kBlockRows)
k_collide(CollideGroup gr) {
  int lb;
  const int k = group_index(gr.g, lb);
  const CollideArgs* a = static_cast<const CollideArgs*>(gr.g.args[k]);
  collide_block<St, IBM, FORCE, CHECK, ZH>(*a, lb, gr.src[k], gr.dst[k]);
}

// One instantiation per (foils, body force, check step, Zou-He faces): the
// solves without Zou-He faces run a kernel without the rebuild.
template <class St, bool IBM, bool FORCE>
static hipError_t launch_collide_c(bool check, bool zh, const CollideGroup& g, int blocks, hipStream_t s) {
  const dim3 b(kBlockX, kBlockRows);
  switch ((check ? 2 : 0) | (zh ? 1 : 0)) {
    case 0: k_collide<St, IBM, FORCE, false, false><<<blocks, b, 0, s>>>(g); break;
    case 1: k_collide<St, IBM, FORCE, false, true><<<blocks, b, 0, s>>>(g); break;
    case 2: k_collide<St, IBM, FORCE, true, false><<<blocks, b, 0, s>>>(g); break;
    default: k_collide<St, IBM, FORCE, true, true><<<blocks, b, 0, s>>>(g); break;
  }
  return hipGetLastError();
}

template <class St>
static hipError_t launch_collide_s(bool ibm, bool force, bool check, bool zh, const CollideGroup& g,
                                   int blocks, hipStream_t s) {
  switch ((ibm ? 2 : 0) | (force ? 1 : 0)) {
    case 0: return launch_collide_c<St, false, false>(check, zh, g, blocks, s);
    case 1: return launch_collide_c<St, false, true>(check, zh, g, blocks, s);
    case 2: return launch_collide_c<St, true, false>(check, zh, g, blocks, s);
    default: return launch_collide_c<St, true, true>(check, zh, g, blocks, s);
  }
}

hipError_t launch_collide(int storage, bool ibm, bool force, bool check, bool zh,
                          const CollideArgs* const* host, const void* const* dev, const void* const* src,
                          void* const* dst, int n, hipStream_t s) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  CollideGroup g;
  int blocks[kMaxGroup];
  for (int k = 0; k < n; ++k) {
    blocks[k] = host[k]->nblocks;
    g.src[k] = src[k];
    g.dst[k] = dst[k];
  }
  const int total = group_fill(g.g, dev, blocks, n);
  if (total == 0) return hipSuccess;
  switch (storage) {
    case ST_F32: return launch_collide_s<StF32>(ibm, force, check, zh, g, total, s);
    case ST_F16: return launch_collide_s<StF16>(ibm, force, check, zh, g, total, s);
    default: return launch_collide_s<StBF16>(ibm, force, check, zh, g, total, s);
  }
}

// ------------------------------------------------------------ ghost, init --
template <class St>
__global__ void k_ghost(Geo g, Phys p, typename St::T* buf) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= g.ny * g.nz) return;
  const int z = row / g.ny, y = row - z * g.ny;
  const long long rb = rowbase(g, y, z);
  float o[kQ];
  for (int side = 0; side < 2; ++side) {
    const int x = side == 0 ? 0 : g.nx - 1;
#pragma unroll
    for (int i = 0; i < kQ; ++i) o[i] = St::ld(buf + (long long)i * g.ps + rb + x);
    write_ghosts<St>(buf, g, p, x, y, z, o);
    if (g.nx == 1) break;
  }
}

hipError_t launch_ghost(int storage, const Geo& g, const Phys& p, void* buf, hipStream_t s) {
  const int rows = g.ny * g.nz;
  const int nb = (rows + 255) / 256;
  switch (storage) {
    case ST_F32: k_ghost<StF32><<<nb, 256, 0, s>>>(g, p, static_cast<float*>(buf)); break;
    case ST_F16: k_ghost<StF16><<<nb, 256, 0, s>>>(g, p, static_cast<__half*>(buf)); break;
    default: k_ghost<StBF16><<<nb, 256, 0, s>>>(g, p, static_cast<unsigned short*>(buf)); break;
  }
  return hipGetLastError();
}

// Equilibrium (Eq. 4) of FP64 rho, u (dense, x fastest; NULL = 1 / 0),
// evaluated in FP64 and rounded once to the storage type.
template <class St>
__global__ void k_init_eq(Geo g, const double* rho, const double* u, typename St::T* D) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= N) return;
  const int x = (int)(cell % g.nx);
  const size_t r = cell / g.nx;
  const int y = (int)(r % g.ny), z = (int)(r / g.ny);
  const double rh = rho ? rho[cell] : 1.0;
  const double ux = u ? u[cell] : 0.0, uy = u ? u[N + cell] : 0.0, uz = u ? u[2 * N + cell] : 0.0;
  const double usq = ux * ux + uy * uy + uz * uz;
  const long long own = rowbase(g, y, z) + x;
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const double cu = cxq(i) * ux + cyq(i) * uy + czq(i) * uz;
    const double v = wqd(i) * ((rh - 1.0) + rh * (3.0 * cu + 4.5 * cu * cu - 1.5 * usq));
    St::st(D + (long long)i * g.ps + own, (float)v);
  }
}

hipError_t launch_init_eq(int storage, const Geo& g, const double* rho, const double* u,
                          void* dst, hipStream_t s) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const unsigned nb = (unsigned)((N + 255) / 256);
  switch (storage) {
    case ST_F32: k_init_eq<StF32><<<nb, 256, 0, s>>>(g, rho, u, static_cast<float*>(dst)); break;
    case ST_F16: k_init_eq<StF16><<<nb, 256, 0, s>>>(g, rho, u, static_cast<__half*>(dst)); break;
    default: k_init_eq<StBF16><<<nb, 256, 0, s>>>(g, rho, u, static_cast<unsigned short*>(dst)); break;
  }
  return hipGetLastError();
}

// rho and u* = (sum c f + F_body/2)/rho of the pre-collision state, as
// 4 dense float planes (rho, ux, uy, uz).
template <class St>
__global__ void k_moments(Geo g, Phys p, const typename St::T* S, float* out) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= N) return;
  const int x = (int)(cell % g.nx);
  const size_t r = cell / g.nx;
  const int y = (int)(r % g.ny), z = (int)(r / g.ny);
  float f[kQ];
  pull19<St>(S, g, x, y, z, f);
  zou_he<St, false>(g, p, x, y, z, f);
  float drho = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    drho += f[i];
    jx += cxq(i) * f[i];
    jy += cyq(i) * f[i];
    jz += czq(i) * f[i];
  }
  const float rho = 1.0f + drho;
  out[cell] = rho;
  out[N + cell] = (jx + 0.5f * p.fb[0]) / rho;
  out[2 * N + cell] = (jy + 0.5f * p.fb[1]) / rho;
  out[3 * N + cell] = (jz + 0.5f * p.fb[2]) / rho;
}

hipError_t launch_moments(int storage, const Geo& g, const Phys& p, const void* src,
                          float* out, hipStream_t s) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const unsigned nb = (unsigned)((N + 255) / 256);
  switch (storage) {
    case ST_F32: k_moments<StF32><<<nb, 256, 0, s>>>(g, p, static_cast<const float*>(src), out); break;
    case ST_F16: k_moments<StF16><<<nb, 256, 0, s>>>(g, p, static_cast<const __half*>(src), out); break;
    default: k_moments<StBF16><<<nb, 256, 0, s>>>(g, p, static_cast<const unsigned short*>(src), out); break;
  }
  return hipGetLastError();
}

// Checkpoints: the stored populations as dense float planes of f - w, and
// back, one thread per cell (reads and writes run along x in both).  All its
// reads are issued together: for a small field `dense` is host memory.
template <class St, bool PACK>
__global__ void k_dense(Geo g, float* dense, int q0, int nq, typename St::T* state) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= N) return;
  const int x = (int)(cell % g.nx);
  const size_t r = cell / g.nx;
  const int y = (int)(r % g.ny), z = (int)(r / g.ny);
  typename St::T* own = state + rowbase(g, y, z) + x;
  float v[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q)
    if (q < nq) v[q] = PACK ? dense[q * N + cell] : St::ld(own + (long long)(q0 + q) * g.ps);
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    if (q >= nq) continue;
    if (PACK)
      St::st(own + (long long)(q0 + q) * g.ps, v[q]);
    else
      dense[q * N + cell] = v[q];
  }
}

// (hipLaunchKernel returns the launch's own status: hipGetLastError would also
// give an error that some earlier call of the thread left, and the read-backs
// are answered whatever that was)
template <bool PACK>
static hipError_t launch_dense(int storage, Geo g, float* dense, int q0, int nq, void* state, hipStream_t s) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  void* args[] = {&g, &dense, &q0, &nq, &state};
  const void* fn = storage == ST_F32   ? reinterpret_cast<const void*>(k_dense<StF32, PACK>)
                   : storage == ST_F16 ? reinterpret_cast<const void*>(k_dense<StF16, PACK>)
                                       : reinterpret_cast<const void*>(k_dense<StBF16, PACK>);
  return hipLaunchKernel(fn, dim3((unsigned)((N + 255) / 256)), dim3(256), args, 0, s);
}

hipError_t launch_pack(int storage, const Geo& g, const float* dense, int q0, int nq, void* state, hipStream_t s) {
  return launch_dense<true>(storage, g, const_cast<float*>(dense), q0, nq, state, s);
}

hipError_t launch_unpack(int storage, const Geo& g, const void* state, int q0, int nq, float* dense,
                         hipStream_t s) {
  return launch_dense<false>(storage, g, dense, q0, nq, const_cast<void*>(state), s);
}

__global__ void k_export(const double* hist, long long first, long long ring, int n, int row, const int* flags,
                         double* out) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) out[i] = hist[((first + i / row) % ring) * row + i % row];
  if (threadIdx.x == 0) *reinterpret_cast<int*>(out + kExportDoubles) = *flags;
}

hipError_t launch_export(const double* hist, long long first, long long ring, int n, int row, const int* flags,
                         double* out, hipStream_t s) {
  void* args[] = {&hist, &first, &ring, &n, &row, &flags, &out};
  return hipLaunchKernel(reinterpret_cast<const void*>(k_export), dim3(1), dim3(256), args, 0, s);
}

__global__ void k_mass_reduce(const double* part, int n, double ncells, double* out, long long step) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += part[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = ncells + sh[0];
    out[1] = (double)step;
  }
}

hipError_t launch_mass_reduce(const double* part, int n, double ncells, double* out,
                              long long step, hipStream_t s) {
  k_mass_reduce<<<1, 256, 0, s>>>(part, n, ncells, out, step);
  return hipGetLastError();
}

}  // namespace ibmk
