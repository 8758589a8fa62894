// Internal declarations shared by the host API (api.cpp) and the gfx950
// kernels (collide.hip, markers.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace ibmk {

constexpr int kQ = 19;
constexpr int kMaxWings = 8;
constexpr int kMaxPerim = 128;     // perimeter markers per foil (LDS of the inversion)
constexpr int kBlockX = 64;        // collide block: 64 cells along x ...
constexpr int kBlockRows = 4;      // ... times 4 rows, one row per wave
constexpr int kPairRows = 12;       // two-step pass: rows along z of a block's column ...
constexpr int kPairThreads = (kPairRows + 3) * 64;   // ... a wave each, two beside them, one for the x sides
constexpr int kPairPlanes = 64;     // most planes along y of such a column
constexpr int kCUs = 256;           // compute units of the device
constexpr int kFactorWindow = 64;  // steps whose perimeter factors (and launch arguments) are made at once
constexpr int kMaxGroup = 64;      // solves in one grouped launch

enum Bc { BC_PERIODIC = 0, BC_WALL = 1, BC_VELOCITY = 2, BC_PRESSURE = 3, BC_ZH_VELOCITY = 4,
          BC_ZH_PRESSURE = 5 };
enum Storage { ST_F32 = 0, ST_F16 = 1, ST_BF16 = 2 };

// FP16 storage keeps 2^12 (f_i - w_i): a power of two, so the scaling is
// exact, and it lifts the deviations of a slow background flow (~1e-5) out
// of the FP16 subnormal range while |f_i - w_i| up to 16 stays finite.
constexpr float kF16Scale = 4096.0f;
constexpr float kF16Unscale = 1.0f / 4096.0f;

// Padded distribution layout, row-major slabs: population q of row
// r = z*ny + y, cell x, lives at element ((r+1)*19 + q)*px + x; px >= nx + 2
// and px*elem is a multiple of 128 bytes so every population row starts on a
// cache line.  The first slab is padding.  After the slabs, at byte offset
// goff, each state keeps its x-face ghost records: 32 bytes per row and side.
struct Geo {
  int nx, ny, nz, px;
  long long ps;        // population stride within a slab (= px)
  long long goff;      // byte offset of a state's ghost records from its base
  int yper, zper;      // periodic y / z
  int bclo, bchi;      // kinds of the -x / +x faces
};

struct Phys {
  float omega;         // 1/tau
  float guo_k;         // 1 - 1/(2 tau)
  float fb[3];         // body force density
  float u_in[3];       // velocity of VELOCITY faces
  float rho_out;       // density of PRESSURE faces
};

// Per foil and step: the xy box of lattice nodes that its markers' kernel
// supports can reach (identical for every span layer of an extruded foil).
// Band moments and the spread correction are stored over this box, with a
// fixed pitch `side` (the largest box the motion can produce).
struct FoilBox {
  int x0, y0, w, h;    // box origin and size for this step
  int side;            // pitch of the per-layer images
  int words;           // 32-bit words per row of `bits`
  // per-layer images over the box, written and read at this step's support
  // nodes only (below)
  const float4* band;  // [nz][side][side] rho, u*x, u*y, u*z
  const float4* corr;  // [nz][side][side] du_x, du_y, du_z, 0 (spread result)
  // this step's support nodes of the foil's markers, bit (lx, ly) relative
  // to the box origin: the only cells the spread can reach, so the cells
  // of the box outside it have a zero correction
  const unsigned* bits;
};

// Of whole cache lines, so that every step's arguments start on one: they are
// cold when its kernel starts, and each further line that the first waves wait
// for costs a launch 0.1 us.  (By its size, not by alignas: loads that the
// compiler knows to be aligned get wider and want longer runs of scalar
// registers, and the two-step kernels with a body force kept 5 to 170 more of
// them in lanes: 257x97x65 with a force 42.6 -> 43.3 us a step.)
struct CollideArgs {
  Geo g;
  Phys p;
  int nw;                    // foils whose correction the kernel applies
  FoilBox box[kMaxWings];
  float wz[4];               // span weights delta(1.5), delta(0.5), delta(0.5), delta(1.5)
  int nxc;                   // 64-wide chunks along x
  int nblocks;               // row groups of 4 rows x 64 cells
  // n / nxc and n / ny as umulhi(n, m) for the wave indices the kernel
  // divides (m = floor(2^32 / d) + 1, exact when n d < 2^32; 0: divide)
  unsigned nxc_mul, ny_mul;
  double* mass_part;         // per-block partial sums (check steps); face blocks after nblocks
  int* flags;                // bit 0: non-finite density seen
  // force reduction on steps with foils
  const double* fpart;       // [nw][nz][4] layer forces and moments
  double* hist;              // [H][nw][8]
  long long hist_row;
  double qS;                 // 0.5 u_ref^2 area_ref
  double sense[kMaxWings], chord[kMaxWings];
  double pad[3];
};
static_assert(sizeof(CollideArgs) % 64 == 0, "a step's arguments start on a cache line");

// Cells around a foil that step s + 1's marker kernels pull from: its node box
// of that step, which reaches past every neighbour of a support node by a
// spare cell, and one cell more; clipped to the box.
__host__ __device__ inline void near_region(const FoilBox& b, const Geo& g, int& x0, int& y0, int& w, int& h) {
  x0 = b.x0 > 0 ? b.x0 - 1 : 0;
  y0 = b.y0 > 0 ? b.y0 - 1 : 0;
  w = (b.x0 + b.w + 1 < g.nx ? b.x0 + b.w + 1 : g.nx) - x0;
  h = (b.y0 + b.h + 1 < g.ny ? b.y0 + b.h + 1 : g.ny) - y0;
}

// A grouped launch: the blocks of solve k are start[k] .. start[k+1]-1 and
// read that solve's arguments from device memory at args[k].  One solve is a
// group of one, so a solve runs the same code alone and in a group.
struct Group {
  int n;
  int start[kMaxGroup + 1];
  const void* args[kMaxGroup];
};

// launch wrappers of collide.hip and pair.hip (the marker kernels' are in
// marker_args.h); all enqueue on `s` and return hipError_t.  `host[k]` is the
// host copy of the arguments that `dev[k]` holds on the device (used for grid
// and LDS sizing only); `src[k]`, `dst[k]` are the solve's states.
hipError_t launch_collide(int storage, bool ibm, bool force, bool check, bool zh,
                          const CollideArgs* const* host, const void* const* dev, const void* const* src,
                          void* const* dst, int n, hipStream_t s);
// Two steps of FP32 states in one pass: dev[k] is the first step's arguments, followed by
// the second's; ylen[k] planes per block.
hipError_t launch_pair(bool ibm, bool force, bool zh, const CollideArgs* const* host,
                       const void* const* dev, const void* const* src, void* const* dst, const int* ylen,
                       int n, hipStream_t s);
// The first of two steps on the cells that the marker kernels of the second
// read (arguments as launch_pair), and that step's force reduction.
hipError_t launch_near(bool force, bool zh, const CollideArgs* const* host, const void* const* dev,
                       const void* const* src, void* const* dst, int n, hipStream_t s);
// Blocks of a solve's pair pass with columns of `ylen` planes.
int pair_blocks(const Geo& g, int ylen);
hipError_t launch_ghost(int storage, const Geo& g, const Phys& p, void* buf, hipStream_t s);
hipError_t launch_init_eq(int storage, const Geo& g, const double* rho, const double* u,
                          void* dst, hipStream_t s);
hipError_t launch_moments(int storage, const Geo& g, const Phys& p, const void* src,
                          float* out, hipStream_t s);
hipError_t launch_mass_reduce(const double* part, int n, double ncells, double* out,
                              long long step, hipStream_t s);
constexpr size_t kMaxLds = 160 * 1024;  // LDS per block on gfx950

// Populations q0 .. q0 + nq - 1 between a state and dense float planes of
// f - w ([population][cell], x fastest), as the checkpoint calls move them.
hipError_t launch_pack(int storage, const Geo& g, const float* dense, int q0, int nq, void* state, hipStream_t s);
hipError_t launch_unpack(int storage, const Geo& g, const void* state, int q0, int nq, float* dense,
                         hipStream_t s);
// n values of the force-history ring from row `first` on and the status flags
// into pinned host memory (the flags after kExportDoubles values).
hipError_t launch_export(const double* hist, long long first, long long ring, int n, int row, const int* flags,
                         double* out, hipStream_t s);
constexpr size_t kExportDoubles = 4096;

// Static scratch of ibmlbm_create_noalloc (scratch.hip): its size, and the
// device address of a device's copy (looked up once per device).
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;
hipError_t scratch_address(int device, void** out);

}  // namespace ibmk
