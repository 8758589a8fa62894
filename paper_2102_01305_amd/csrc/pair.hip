// gfx950 lattice kernels that take two time steps in one pass over the lattice.
//
//  pair   steps s and s+1 of every cell: the state after step s lives in LDS
//         and registers only, so two steps read the lattice once and write it
//         once.
//  near   step s of the cells around the foils alone, from which the marker
//         kernels of step s+1 take their band moments before `pair` runs.
#include "update_dev.h"

namespace ibmk {

// Slot in LDS of the 16 populations that move in x or z (0, 3 and 4 stay on
// their lane).
__host__ __device__ constexpr int lslot(int i) { return i < 3 ? i - 1 : i - 3; }

// What an open x face presents to the cells beside it in place of the boundary
// cell's values o: the ghost layer's equilibrium, in the populations with
// c_x = dir (the others are not pulled from there).
__device__ __forceinline__ void face_values(const Phys& p, int kind, int dir, float o[kQ]) {
#pragma clang fp contract(off)
  float drho, jx, jy, jz, rg, ux, uy, uz;
  moments19(o, drho, jx, jy, jz);
  open_face(p, kind, 1.0f + drho, jx, jy, jz, rg, ux, uy, uz);
  const float usq = ux * ux + uy * uy + uz * uz;
#pragma unroll
  for (int i = 0; i < kQ; ++i)
    if (cxq(i) == dir) o[i] = feq_dev_strict(i, rg - 1.0f, rg, ux, uy, uz, usq);
}

// Buffer descriptor over the rows of one z (n_y slabs from `base` on): every
// population row of every y is then a 32-bit scalar offset and the lane's x a
// 32-bit vector offset, with no 64-bit address arithmetic per load or store.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t span_rsrc(char* base) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, kRawBufferWord3);
}

// Pre-collision values (stored units) of one cell per lane in plane y of a
// column, with the sources of pull19.  Every population is read at its upwind
// neighbour first, all 19 loads together: of a row of lanes (ROW: z uniform in
// the wave) through the descriptors of its three z, of the cells beside the
// column (z varies) by address; the few lanes at an x face and beside a wall
// then take the ghost record or their own opposite population instead.
template <bool ROW>
__device__ __forceinline__ void pull_plane(const char* __restrict__ S, const Geo& g, const __amdgpu_buffer_rsrc_t rz[3],
                                           __amdgpu_buffer_rsrc_t rg, unsigned popb, bool edge, int x, int y, int z, float f[kQ]) {
  constexpr int es = sizeof(float);
  const unsigned rowb = (unsigned)kQ * popb;
  const int ys[3] = {y == 0 ? g.ny - 1 : y - 1, y, y == g.ny - 1 ? 0 : y + 1};   // y - c_y
  const int zs[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};   // z - c_z
  const unsigned xo = (unsigned)x * es;
  const unsigned yo[3] = {ys[0] * rowb, ys[1] * rowb, ys[2] * rowb};
  if (ROW) {
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      f[i] = StF32::ldb(rz[1 - czq(i)], (int)xo, (int)(yo[1 - cyq(i)] + (unsigned)i * popb - (unsigned)(cxq(i) * es)));
  } else {
    const char* lane[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) lane[k] = S + (unsigned long long)(unsigned)(zs[k] * g.ny + 1) * rowb + xo;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      f[i] = *(reinterpret_cast<const float*>(lane[1 - czq(i)] +
                                                (yo[1 - cyq(i)] + (unsigned)i * popb - (unsigned)(cxq(i) * es))));
      __builtin_amdgcn_sched_barrier(0);               // (no 19 addresses held at once)
    }
  }
  if (edge && (x == 0 || x == g.nx - 1)) {
    // (a row's ghost records by its scalar offset: a record's address made in
    // each lane took 40 vector operations a face)
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      if (cxq(i) == 0) continue;
      const int gr = zs[1 - czq(i)] * g.ny + ys[1 - cyq(i)] + (cxq(i) == 1 ? 0 : g.ny * g.nz);
      if (cxq(i) == 1 ? x == 0 : x == g.nx - 1)
        f[i] = ROW ? StF32::ldb(rg, 0, gr * 32 + xslot(i) * es) : StF32::ldb(rg, gr * 32 + xslot(i) * es, 0);
    }
  }
  const int wy = g.yper ? 0 : (y == 0 ? 1 : (y == g.ny - 1 ? -1 : 0));
  const int wz = g.zper ? 0 : (z == 0 ? 1 : (z == g.nz - 1 ? -1 : 0));
  if (wy != 0 || wz != 0) {
    const char* own = S + (unsigned long long)(unsigned)(z * g.ny + y + 1) * rowb + xo;
#pragma unroll
    for (int i = 1; i < kQ; ++i)
      if ((cyq(i) != 0 && cyq(i) == wy) || (czq(i) != 0 && czq(i) == wz))
        f[i] = *(reinterpret_cast<const float*>(own + (unsigned)oppq(i) * popb));
  }
}

// Support nodes of the foils in a block's column, per foil, step of the pair
// and plane: one bit per cell of the row from x0 - 1 on.
struct ColumnBits {
  unsigned w[kMaxWings][2][kPairPlanes + 2][3];
};

// Fill `cb` for the planes from p0 on (all threads of the block).
__device__ __forceinline__ void column_bits(const CollideArgs& a, const CollideArgs& b, int x0, int p0, int planes,
                                            ColumnBits& cb) {
  for (int e = (int)threadIdx.x; e < a.nw * 2 * planes * 3; e += (int)blockDim.x) {
    const int q = e % 3, p = (e / 3) % planes, s = (e / (3 * planes)) & 1, k = e / (6 * planes);
    const FoilBox& f = s ? b.box[k] : a.box[k];
    const int ly = p0 + p - f.y0, lx = x0 - 1 + 32 * q - f.x0;   // of the word's first bit
    unsigned v = 0;
    if (ly >= 0 && ly < f.h && lx > -32 && lx < f.w) {
      const auto* row = gmem(f.bits) + ly * f.words;
      const int i = lx >> 5, sh = lx & 31;                        // (rounded down: -1 for lx < 0)
      const unsigned lo = i >= 0 ? row[i] : 0u, hi = i + 1 < f.words ? row[i + 1] : 0u;
      v = sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
    }
    cb.w[k][s][p][q] = v;
  }
}

// The corrections of both steps together, so that their loads share one wait:
// step s (`a`) at plane p, step s + 1 (`b`, whose images are in `band`) at
// plane p - 1; a lane asks for either with ina, inb.
__device__ __forceinline__ void correction2(const Geo& g, const CollideArgs& a, const CollideArgs& b,
                                            const ColumnBits& cb, int p0, int col, int x, int p, bool ina, bool inb,
                                            int z, Correction& ca, Correction& cc) {
  for (int k = 0; k < a.nw; ++k) {
    const bool ha = ina && ((cb.w[k][0][p - p0][col >> 5] >> (col & 31)) & 1u);
    const bool hb = inb && ((cb.w[k][1][p - 1 - p0][col >> 5] >> (col & 31)) & 1u);
    f4 va[4], vb[4];
    if (ha) correction_load(g, a.box[k], a.box[k].corr, x, p, z, va);
    if (hb) correction_load(g, b.box[k], b.box[k].band, x, p - 1, z, vb);
    if (ha) correction_add(a.wz, va, ca);
    if (hb) correction_add(b.wz, vb, cc);
  }
}

// A block takes a column of the lattice, 64 cells along x times R = 12 rows
// along z, and marches along y over `ylen` planes.  At plane p its 15 waves (one
// row each, two of them the rows beside the column, and one wave of lanes for
// the cells beside it in x) have step s's pull of that plane in registers,
// update it and exchange the result through LDS; the R rows then have every
// value that step s+1 of plane p-1 pulls: from plane p just exchanged, and from
// planes p-1 and p-2 in the registers of the lane that uses them.
//
// Bound: memory, as for one step at a time, but the lattice is read and
// written once for two steps: per launch 1.12 x the 76 B a cell that a read
// takes (the rows and lines columns share, as far as one L2 does not serve
// both) and 76 B written, 5.0 TB/s at 512x384x384 (periodic), with the vector
// units busy 41% of the time.  Two steps of the collide kernel against one
// launch here: 256x192x192 483 -> 317 us, 256x256x256 864 -> 592,
// 512x384x384 3926 -> 2415; clap & fling 256x192x192 335 us (a plane that meets
// a foil takes 2.4 us longer), whole step 275 -> 207 us.  Where memory does not
// bind, a plane takes 3.8 us of issue, to which scalar pressure adds: 127 to 312
// scalar registers are kept in lanes of vector registers, and most of the lane
// reads that bring them back (553 of 564 with foils) lie in the march.
// Why this shape: one block per compute unit, so R near what 16 waves and
// 160 KB of LDS allow (halo work 1 + 3/R); the same with R = 7 or 8 and two
// blocks per unit 1262-1281 us a step at 512x384x384 (1228 with R = 12), R = 5
// at 128 registers 1328.  R = 13, with all 16 waves, is slower by 3% where 12
// divides the span (256x192x192 160.6 -> 165.9 us a step, 512x384x384 1228 ->
// 1269) and faster where its tiles are fewer (257x97x65 42.6 -> 38.1,
// 256x192x101 92.7 -> 91.5, 256x192x193 180.7 -> 166.6, 256x192x199 183.7 ->
// 169.2): 12 is not the better one everywhere.
// What the march needed: descriptors per z in place of per-lane addresses, no
// row offsets kept over the loop (168 vector registers and spills with them,
// 103-128 now and none in memory; a reload in the march waits for the pull), the
// next plane's pull in flight over the exchange and step s+1 (1427 -> 1284 us a
// step), and LDS by plane parity, one barrier a plane instead of two (-> 1254).
template <bool IBM, bool FORCE, bool ZH>
__device__ __forceinline__ void pair_block(const CollideArgs& __restrict__ a, const CollideArgs& __restrict__ b,
                                           int lb, int nblocks, int ylen, const void* src, void* dst) {
  constexpr int R = kPairRows, LX = kBlockX + 2;
  __shared__ float shm[2][16][R + 2][LX];                  // by the parity of the plane
  const Geo g = a.g;                                   // (by value: no reload after a store)
  const Phys ph = a.p;
  const char* __restrict__ S = static_cast<const char*>(src);
  float* __restrict__ D = static_cast<float*>(dst);
  __shared__ ColumnBits cb;
  __shared__ float face[2][2][R][kQ + 1];              // by parity: step s+1 at the x faces, per side and row
  // each XCD takes one run of consecutive columns: neighbours share their
  // halo rows and lines through one L2
  const int per = nblocks >> 3;
  const int lt = lb < 8 * per ? (lb & 7) * per + (lb >> 3) : lb;
  const int nzt = (g.nz + R - 1) / R;
  const int xc = lt % a.nxc, zt = (lt / a.nxc) % nzt, yc = lt / (a.nxc * nzt);
  const int x0 = xc * kBlockX, xe = x0 + kBlockX < g.nx ? x0 + kBlockX : g.nx;
  const int z0 = zt * R, cnt = g.nz - z0 < R ? g.nz - z0 : R;
  const int ya = yc * ylen, yb = ya + ylen < g.ny ? ya + ylen : g.ny;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)threadIdx.x & 63;
  // rows z0-1 .. z0+cnt of the column (0 .. cnt+1); outside a wall: none
  const bool halo = w == R + 2;
  int x, r, z, col, kind = BC_PERIODIC, dir = 0;
  bool act;
  if (!halo) {
    r = w;
    x = x0 + lane;
    col = lane + 1;
    act = x < g.nx;
  } else {
    // lanes 0..31: the cells at x0 - 1, lanes 32..63: those at xe
    r = lane & 31;
    const bool hi = lane >= 32;
    x = hi ? xe : x0 - 1;
    col = hi ? xe - x0 + 1 : 0;
    act = true;
    if (x < 0 || x == g.nx) {
      kind = hi ? g.bchi : g.bclo;
      dir = hi ? -1 : 1;
      act = kind != BC_WALL;
      // a periodic image, or the boundary cell an open face's ghost is made from
      x = (x < 0) == (kind == BC_PERIODIC) ? g.nx - 1 : 0;
    }
  }
  z = z0 - 1 + r;
  act = act && r <= cnt + 1 && (g.zper || (z >= 0 && z < g.nz));
  z = z < 0 ? z + g.nz : (z >= g.nz ? z - g.nz : z);
  const int zu = __builtin_amdgcn_readfirstlane(z);    // the row's z, for the compiler wave-uniform
  // what the wave's row is, in one scalar (a flag each would take two)
  enum : int { kHalo = 1, kInner = 2, kXw0 = 4, kXw1 = 8, kZw0 = 16, kZw1 = 32, kWalls = 60, kEdge = 64 };
  const bool takes2 = !halo && w >= 1 && w <= cnt;     // rows that take step s+1
  int is = (halo ? kHalo : 0) | (x0 == 0 || xe >= g.nx - 1 ? kEdge : 0);   // (lanes lie at an x face)
  if (takes2)
    is |= kInner | (g.bclo == BC_WALL && x0 == 0 ? kXw0 : 0) | (g.bchi == BC_WALL && xe == g.nx ? kXw1 : 0) |
          (!g.zper && zu == 0 ? kZw0 : 0) | (!g.zper && zu == g.nz - 1 ? kZw1 : 0);
  is = __builtin_amdgcn_readfirstlane(is);
  const unsigned popb0 = (unsigned)g.px * (unsigned)sizeof(float);
  // descriptors of the three z that a row of lanes pulls from, and of the row
  // it writes
  __amdgpu_buffer_rsrc_t rz[3], rd;
  const __amdgpu_buffer_rsrc_t rg = span_rsrc(const_cast<char*>(S) + g.goff);   // x-face ghost records
  {
    const unsigned long long slab = (unsigned long long)(kQ * popb0);
    const int zl = zu == 0 ? g.nz - 1 : zu - 1, zh = zu == g.nz - 1 ? 0 : zu + 1;
    rz[0] = span_rsrc(const_cast<char*>(S) + (unsigned)(zl * g.ny + 1) * slab);
    rz[1] = span_rsrc(const_cast<char*>(S) + (unsigned)(zu * g.ny + 1) * slab);
    rz[2] = span_rsrc(const_cast<char*>(S) + (unsigned)(zh * g.ny + 1) * slab);
    rd = span_rsrc(reinterpret_cast<char*>(D) + (unsigned)(zu * g.ny + 1) * slab);
  }

  // planes whose cells in this column may have a correction (a foil's node
  // boxes of both steps, and the plane after for step s+1; a periodic y axis
  // wraps none of them: see pair_ok)
  int fy0 = 0x7fffffff, fy1 = -1;
  if (IBM) {
    for (int k = 0; k < a.nw; ++k) {
      const FoilBox& ba = a.box[k];
      const FoilBox& bb = b.box[k];
      const int xa = ba.x0 < bb.x0 ? ba.x0 : bb.x0, xb = ba.x0 + ba.w > bb.x0 + bb.w ? ba.x0 + ba.w : bb.x0 + bb.w;
      if (xb < x0 || xa > xe) continue;
      const int y0 = ba.y0 < bb.y0 ? ba.y0 : bb.y0, y1 = ba.y0 + ba.h > bb.y0 + bb.h ? ba.y0 + ba.h : bb.y0 + bb.h;
      fy0 = y0 < fy0 ? y0 : fy0;
      fy1 = y1 > fy1 ? y1 : fy1;
    }
    if (fy0 <= yb && fy1 >= ya - 1) {
      column_bits(a, b, x0, ya - 1, yb - ya + 2, cb);
      __syncthreads();
    } else {
      fy1 = -1;
    }
  }

  // cy = 0 values of the plane before (the cells step s+1 takes next), and
  // cy = +1 values of the plane before and the one before that
  float h0[9], pa[5], pb[5], hx = 0.f, hz = 0.f;
  constexpr int i0[9] = {0, 1, 2, 5, 6, 11, 12, 13, 14}, ip[5] = {3, 7, 10, 15, 17}, im[5] = {4, 8, 9, 16, 18};
#pragma unroll
  for (int k = 0; k < 9; ++k) h0[k] = 0.f;
#pragma unroll
  for (int k = 0; k < 5; ++k) pa[k] = pb[k] = 0.f;

  // value of population i at the inner lane's upwind neighbour in the plane
  // in LDS, and the lane's own
  auto from = [&](int p, int i) { return shm[p & 1][lslot(i)][w - czq(i)][lane + 1 - cxq(i)]; };
  auto own = [&](int p, int i) { return shm[p & 1][lslot(i)][w][lane + 1]; };

  // step s's values of a plane: pulled while the plane before is still worked
  // on, updated in place, exchanged
  float nf[kQ];
  auto inside = [&](int p) { return g.yper || (p >= 0 && p < g.ny); };
  auto pull = [&](int p) {
    // made anew for each plane: the 19 row offsets derived from it, kept
    // over the loop, would take the registers of two more waves per SIMD
    unsigned popb = popb0;
    asm volatile("" : "+s"(popb));
    const int y = p < 0 ? p + g.ny : (p >= g.ny ? p - g.ny : p);
    if (!(is & kHalo))
      pull_plane<true>(S, g, rz, rg, popb, is & kEdge, x, y, zu, nf);
    else
      pull_plane<false>(S, g, rz, rg, popb, is & kEdge, x, y, z, nf);
  };
  // The ghost records of plane q - 1, whose cells at the x faces were exchanged
  // in iteration q: by a wave that takes no step s+1, a lane per side and row
  // (in the waves of the rows, one lane of 64 took them a third of their time).
  auto ghosts = [&](int q) {
    // With foils and a body force, what follows is made anew for each plane:
    // kept over the loop it spilled two vector registers to memory, whose
    // reloads in the march wait for the pull in flight (clap & fling 256 x 192 x 192 with a body
    // force 222 -> 212 us a step; the other instantiations, which do not spill,
    // 0.5% slower by it).
    int ln = lane;
    if (IBM && FORCE) asm volatile("" : "+v"(ln));
    const int side = ln >> 5, row = ln & 31;
    const int fx = side ? g.nx - 1 : 0;
    if (row < cnt && (side ? xe == g.nx : x0 == 0)) {
      float v[kQ];
#pragma unroll
      for (int i = 0; i < kQ; ++i) v[i] = face[q & 1][side][row][i];
      write_ghosts<StF32>(D, g, ph, fx, q - 1, z0 + row, v);
    }
  };
  const int first = inside(ya - 1) ? ya - 1 : 0;
  if (act) pull(first);
  for (int p = first; p <= yb; ++p) {
    const bool real = inside(p);                       // else: beyond a y wall (the last plane only)
    float o[3] = {0.f, 0.f, 0.f};                      // own values of populations 0, 3, 4
    Correction c2;                                     // of step s+1 at plane p-1
    if (real) {
      if (act) {
        const int y = p < 0 ? p + g.ny : (p >= g.ny ? p - g.ny : p);
        // both steps' corrections, while the pull is in flight
        Correction c;
        if (IBM && p >= fy0 && p <= fy1) correction2(g, a, b, cb, ya - 1, col, x, p, true, (is & kInner) && p > ya, z, c, c2);
        update_cell<StF32, IBM, FORCE, ZH, true>(g, ph, a, x, y, z, nf, c);
        if ((is & kHalo) && kind != BC_PERIODIC) face_values(ph, kind, dir, nf);
#pragma unroll
        for (int i = 1; i < kQ; ++i)
          if (i != 3 && i != 4) shm[p & 1][lslot(i)][r][col] = nf[i];
        o[0] = nf[0];
        o[1] = nf[3];
        o[2] = nf[4];
        if (p < yb && inside(p + 1)) pull(p + 1);
      }
    }
    // one barrier a plane: what was read of this parity's buffer two planes
    // ago was read before the last one
    __syncthreads();
    if ((is & kEdge) && w == 0 && p > ya + 1) ghosts(p - 1);
    if (!(is & kInner)) continue;
    if (p > ya) {
      float f[kQ];
#pragma unroll
      for (int k = 0; k < 9; ++k) f[i0[k]] = h0[k];
#pragma unroll
      for (int k = 0; k < 5; ++k) f[ip[k]] = pb[k];
      // cy = -1: from plane p, or, where that lies beyond a y wall, reflected
      // from the cell's own values of plane p-1, which LDS still holds
      f[4] = real ? o[2] : pa[0];
      const float* sp = &shm[(real ? p : p - 1) & 1][0][w][lane + 1];
#pragma unroll
      for (int k = 1; k < 5; ++k) {
        const int i = im[k];
        f[i] = sp[real ? (lslot(i) * (R + 2) - czq(i)) * LX - cxq(i) : lslot(oppq(i)) * (R + 2) * LX];
      }
      if ((is & kWalls) && real) {
        // reflected at the cell itself, from its own values of plane p-1
        if ((is & kXw0) && x == 0) f[9] = hx;
        if ((is & kXw1) && x == g.nx - 1) f[8] = hx;
        if (is & kZw0) f[18] = hz;
        if (is & kZw1) f[16] = hz;
      }
      if (IBM && !real && p >= fy0 && p <= fy1) {
        Correction c;
        correction2(g, a, b, cb, ya - 1, col, x, p, false, act, zu, c, c2);
      }
      update_cell<StF32, IBM, FORCE, ZH, true>(g, ph, b, x, p - 1, zu, f, c2);
      if (act) {
        unsigned popb = popb0;
        asm volatile("" : "+s"(popb));
#pragma unroll
        for (int i = 0; i < kQ; ++i)
          StF32::stb(rd, x * (int)sizeof(float), (int)((unsigned)((p - 1) * kQ + i) * popb), f[i]);
        if ((is & kEdge) && (x == 0 || x == g.nx - 1)) {
#pragma unroll
          for (int i = 0; i < kQ; ++i) face[p & 1][x != 0][w - 1][i] = f[i];
        }
      }
    }
    // the values of plane p that the next two planes' updates pull
#pragma unroll
    for (int k = 0; k < 5; ++k) pb[k] = pa[k];
    if (p == 0 && !g.yper) {                           // a y wall reflects those below the first plane
      pb[0] = o[2];
#pragma unroll
      for (int k = 1; k < 5; ++k) pb[k] = own(p, oppq(ip[k]));
    }
    h0[0] = o[0];
    pa[0] = o[1];
#pragma unroll
    for (int k = 1; k < 9; ++k) h0[k] = from(p, i0[k]);
#pragma unroll
    for (int k = 1; k < 5; ++k) pa[k] = from(p, ip[k]);
    if (is & kWalls) {
      const bool l0 = (is & kXw0) && x == 0, l1 = (is & kXw1) && x == g.nx - 1;
      const bool zw0 = is & kZw0, zw1 = is & kZw1;
#pragma unroll
      for (int k = 1; k < 9; ++k) {
        const int i = i0[k];
        if ((cxq(i) == 1 && l0) || (cxq(i) == -1 && l1) || (czq(i) == 1 && zw0) || (czq(i) == -1 && zw1))
          h0[k] = own(p, oppq(i));
      }
#pragma unroll
      for (int k = 1; k < 5; ++k) {
        const int i = ip[k];
        if ((cxq(i) == 1 && l0) || (cxq(i) == -1 && l1) || (czq(i) == 1 && zw0) || (czq(i) == -1 && zw1))
          pb[k] = own(p, oppq(i));
      }
      hx = x == 0 ? own(p, 10) : own(p, 7);
      hz = zw0 ? own(p, 17) : own(p, 15);
    }
  }
  if (is & kEdge) {
    __syncthreads();
    if (w == 0) ghosts(yb);
  }
  // step s+1's forces, by a wave that has had no step s+1 to take
  if (IBM && lb == 0 && w == 0)
    for (int k = 0; k < a.nw; ++k) reduce_forces(b, k, lane);
}

struct PairGroup {
  Group g;
  const void* src[kMaxGroup];
  void* dst[kMaxGroup];
  int ylen[kMaxGroup];
};

template <bool IBM, bool FORCE, bool ZH>
__global__ void __launch_bounds__(kPairThreads, 4) k_pair(PairGroup gr) {
  int lb;
  const int k = group_index(gr.g, lb);
  const CollideArgs* a = static_cast<const CollideArgs*>(gr.g.args[k]);
  pair_block<IBM, FORCE, ZH>(a[0], a[1], lb, gr.g.start[k + 1] - gr.g.start[k], gr.ylen[k], gr.src[k], gr.dst[k]);
}

// Blocks of one solve's pair launch with columns of `ylen` planes.
int pair_blocks(const Geo& g, int ylen) {
  return ((g.nx + kBlockX - 1) / kBlockX) * ((g.nz + kPairRows - 1) / kPairRows) * ((g.ny + ylen - 1) / ylen);
}

hipError_t launch_pair(bool ibm, bool force, bool zh, const CollideArgs* const* host,
                       const void* const* dev, const void* const* src, void* const* dst, const int* ylen, int n,
                       hipStream_t s) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  PairGroup g;
  int blocks[kMaxGroup];
  for (int k = 0; k < n; ++k) {
    blocks[k] = pair_blocks(host[k]->g, ylen[k]);
    g.src[k] = src[k];
    g.dst[k] = dst[k];
    g.ylen[k] = ylen[k];
  }
  const int total = group_fill(g.g, dev, blocks, n);
  switch ((ibm ? 4 : 0) | (force ? 2 : 0) | (zh ? 1 : 0)) {
    case 0: k_pair<false, false, false><<<total, kPairThreads, 0, s>>>(g); break;
    case 1: k_pair<false, false, true><<<total, kPairThreads, 0, s>>>(g); break;
    case 2: k_pair<false, true, false><<<total, kPairThreads, 0, s>>>(g); break;
    case 3: k_pair<false, true, true><<<total, kPairThreads, 0, s>>>(g); break;
    case 4: k_pair<true, false, false><<<total, kPairThreads, 0, s>>>(g); break;
    case 5: k_pair<true, false, true><<<total, kPairThreads, 0, s>>>(g); break;
    case 6: k_pair<true, true, false><<<total, kPairThreads, 0, s>>>(g); break;
    default: k_pair<true, true, true><<<total, kPairThreads, 0, s>>>(g); break;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------- near --

// Does a support node of foil box f lie at (x, y) or beside it?
__device__ __forceinline__ bool near_support(const FoilBox& f, int x, int y) {
  const int lx = x - 1 - f.x0, ly = y - f.y0, i = lx >> 5, sh = lx & 31;   // (i is -1 left of the box)
  unsigned any = 0u;
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    const int r = ly + d;
    if (r < 0 || r >= f.h) continue;
    const auto* row = gmem(f.bits) + r * f.words;
    const unsigned lo = i >= 0 && i < f.words ? row[i] : 0u, hi = i + 1 < f.words ? row[i + 1] : 0u;
    any |= sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
  }
  return any & 7u;
}

// Step s of the cells that step s + 1's marker kernels pull from: the support
// nodes of that step and the cells beside them (k_pair overwrites every cell
// afterwards).  A wave takes 64 cells of a foil's region (near_region of step
// s + 1) of one layer, row after row: a row is some 25 to 50 cells long, so
// that a wave per row left half of its lanes idle, and a third to a half of
// the region lies inside the foil or in the corners, where no marker reads.
// The stores are plain ones: the marker kernels read them next.  Bound by the
// latency of its three rounds of dependent loads (bits, pull, correction).
// Against a wave per row over the whole region with streaming stores: clap &
// fling 256 x 192 x 192 21.0 -> 15.0 us (17.4 with streaming stores),
// 512 x 384 x 384 50.8 -> 36.7, cylinder 256 x 192 x 192 15.6 -> 14.5; a step
// of 16 solves of a sweep 523 -> 505.  The corrections' loads issued together
// with the pull's gave nothing.
template <bool FORCE, bool ZH>
__device__ __forceinline__ void near_block(const CollideArgs& __restrict__ a, const CollideArgs& __restrict__ b,
                                           int lb, const void* src, void* dst) {
  const Geo g = a.g;
  const Phys& ph = a.p;
  if (lb == 0) {                                       // (the first block: step s's forces)
    for (int k = (int)threadIdx.y; k < a.nw; k += kBlockRows) reduce_forces(a, k, (int)threadIdx.x);
    return;
  }
  int u = __builtin_amdgcn_readfirstlane((lb - 1) * kBlockRows + (int)threadIdx.y);
  for (int k = 0; k < a.nw; ++k) {
    int x0, y0, w, h;
    near_region(b.box[k], g, x0, y0, w, h);
    const int nc = (w * h + kBlockX - 1) / kBlockX, units = nc * g.nz;
    if (u >= units) {
      u -= units;
      continue;
    }
    const int z = __builtin_amdgcn_readfirstlane(u / nc);
    const unsigned e = (unsigned)((u - z * nc) * kBlockX) + threadIdx.x;
    const int row = (int)(e / (unsigned)w), x = x0 + (int)e - row * w, y = y0 + row;
    if (row >= h || !near_support(b.box[k], x, y)) return;
    const float* S = static_cast<const float*>(src);
    float* D = static_cast<float*>(dst);
    float f[kQ];
    const unsigned popb = (unsigned)(g.px * sizeof(float)), slab = kQ * popb;
    // beside a y wall or an x face, and where the region's rows pass a
    // descriptor's 31 bits: source by source (z is periodic where there are foils)
    if ((unsigned long long)(h + 3) * slab >= (1ull << 31) ||
        !__all(x > 0 && x < g.nx - 1 && y > 0 && y < g.ny - 1)) {
      pull19<StF32, true>(S, g, x, y, z, f);
      update_cell<StF32, true, FORCE, ZH, false>(g, ph, a, x, y, z, f);
      store_cell<StF32>(D, g, ph, x, y, z, f);
      return;
    }
    // every source lies in the region's rows of three layers: one descriptor
    // per layer (from the row before the region on), the lane's cell as its
    // offset
    const int zs[3] = {z == 0 ? g.nz - 1 : z - 1, z, z == g.nz - 1 ? 0 : z + 1};   // z - c_z
    __amdgpu_buffer_rsrc_t rz[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
      rz[j] = span_rsrc(reinterpret_cast<char*>(const_cast<float*>(S)) +
                        (unsigned long long)(unsigned)(zs[j] * g.ny + y0) * slab);
    const __amdgpu_buffer_rsrc_t rd =
        span_rsrc(reinterpret_cast<char*>(D) + (unsigned long long)(unsigned)(z * g.ny + y0) * slab);
    const int vo = (int)((unsigned)row * slab + (unsigned)x * 4u);
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      f[i] = StF32::ldb(rz[1 - czq(i)], vo, (int)((unsigned)(1 - cyq(i)) * slab + (unsigned)i * popb) - cxq(i) * 4);
    update_cell<StF32, true, FORCE, ZH, false>(g, ph, a, x, y, z, f);
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f[i]), rd, vo, (int)(slab + (unsigned)i * popb), 0);
    return;
  }
}

struct NearGroup {
  Group g;
  const void* src[kMaxGroup];
  void* dst[kMaxGroup];
};

template <bool FORCE, bool ZH>
__global__ void __launch_bounds__(kBlockX * kBlockRows) k_near(NearGroup gr) {
  int lb;
  const int k = group_index(gr.g, lb);
  const CollideArgs* a = static_cast<const CollideArgs*>(gr.g.args[k]);
  near_block<FORCE, ZH>(a[0], a[1], lb, gr.src[k], gr.dst[k]);
}

hipError_t launch_near(bool force, bool zh, const CollideArgs* const* host, const void* const* dev,
                       const void* const* src, void* const* dst, int n, hipStream_t s) {
  if (n < 1 || n > kMaxGroup) return hipErrorInvalidValue;
  NearGroup g;
  int blocks[kMaxGroup];
  for (int k = 0; k < n; ++k) {
    long long waves = 0;
    for (int j = 0; j < host[k]->nw; ++j) {
      int x0, y0, w, h;
      near_region(host[k][1].box[j], host[k]->g, x0, y0, w, h);
      waves += (long long)((w * h + kBlockX - 1) / kBlockX) * host[k]->g.nz;
    }
    blocks[k] = (int)((waves + kBlockRows - 1) / kBlockRows) + 1;
    g.src[k] = src[k];
    g.dst[k] = dst[k];
  }
  const int total = group_fill(g.g, dev, blocks, n);
  const dim3 b(kBlockX, kBlockRows);
  switch ((force ? 2 : 0) | (zh ? 1 : 0)) {
    case 0: k_near<false, false><<<total, b, 0, s>>>(g); break;
    case 1: k_near<false, true><<<total, b, 0, s>>>(g); break;
    case 2: k_near<true, false><<<total, b, 0, s>>>(g); break;
    default: k_near<true, true><<<total, b, 0, s>>>(g); break;
  }
  return hipGetLastError();
}

}  // namespace ibmk
