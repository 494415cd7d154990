// Geometric multigrid V-cycle, FP32, used as the preconditioner of the FP64
// flexible CG for the implicit-Euler systems of Eqs. (oxygen) and (chemo).
// (The paper preconditions the same SPD systems with algebraic multigrid.)
//
// Hierarchy: voxel-centred 2:1 coarsening per axis, n_{k+1} = ceil(n_k / 2); a
// level-k cell I covers the fine cells [I 2^k, min((I+1) 2^k, n0)) per axis
// (ragged at odd edges).  The level-k operator is
//     (A_k u)_I = c_I u_I + sum_faces g_IJ (u_I - u_J),
// c_I the sum of the fine reaction coefficients over the cell, and g_IJ the
// finite-volume coupling of the two aggregates: D/h^2 times the shared face
// area over the centre distance, both in fine-voxel units,
//     g = a * area / ((e_I + e_J) / 2),   e = extents along the face normal.
// Restriction sums fine residuals over the aggregate; prolongation is
// cell-centred linear interpolation (about a third fewer CG iterations than
// piecewise-constant for the diffusion-dominated drug operator); smoothing is
// weighted Jacobi (two sweeps before and two after the coarse-grid
// correction).  Levels above `mg_coarse_max` cells run as multi-workgroup
// kernels; the remaining levels of each system are one workgroup working in
// LDS down to a single cell (solved exactly), the same cycle.
//
// Fused kernels per global level k:
//   pre      u1 = w Dinv r (first sweep from zero, formed on the fly at the
//            neighbours), u2 = (1-w) u1 + w Dinv (r + sum g u1_J)
//   restrict r_{k+1}(I) = sum over children of (r - A u2)
//   post1    u3 = u2 + P e_{k+1} (formed on the fly; P the cell-centred
//            linear interpolation, restriction stays the aggregate sum), u4 =
//            Jacobi(u3)
//   post2    u5 = Jacobi(u4); at level 0 u5 is the CG's z, and the same kernel
//            reduces r.z and finishes beta of the flexible CG.
#include <type_traits>

#include "dev_util.h"

namespace hca {

template <bool UNI>
struct Geo {
  int nx, ny, nz, k, n0x, n0y, n0z;
  float a;

  __device__ inline int ext(int I, int n0) const {
    if (UNI) return 1;
    const int lo = I << k;
    const int hi = min((I + 1) << k, n0);
    return hi - lo;
  }
  // couplings of the faces (x,y,z)-(x+1,y,z), (x,y,z)-(x,y+1,z), (x,y,z)-(x,y,z+1)
  __device__ inline float gx(int x, int y, int z) const {
    if (UNI) return a;
    return 2.f * a * (float)(ext(y, n0y) * ext(z, n0z)) / (float)(ext(x, n0x) + ext(x + 1, n0x));
  }
  __device__ inline float gy(int x, int y, int z) const {
    if (UNI) return a;
    return 2.f * a * (float)(ext(x, n0x) * ext(z, n0z)) / (float)(ext(y, n0y) + ext(y + 1, n0y));
  }
  __device__ inline float gz(int x, int y, int z) const {
    if (UNI) return a;
    return 2.f * a * (float)(ext(x, n0x) * ext(y, n0y)) / (float)(ext(z, n0z) + ext(z + 1, n0z));
  }
  // sum of the couplings of the existing faces of (x,y,z)
  __device__ inline float gsum(int x, int y, int z) const {
    float s = 0.f;
    if (x > 0) s += gx(x - 1, y, z);
    if (x + 1 < nx) s += gx(x, y, z);
    if (y > 0) s += gy(x, y - 1, z);
    if (y + 1 < ny) s += gy(x, y, z);
    if (z > 0) s += gz(x, y, z - 1);
    if (z + 1 < nz) s += gz(x, y, z);
    return s;
  }
};

template <bool UNI>
__device__ inline Geo<UNI> geo_of(const MgRep& m) {
  const float a = m.a;
  Geo<UNI> g;
  g.nx = m.nx;
  g.ny = m.ny;
  g.nz = m.nz;
  g.k = m.k;
  g.n0x = m.n0x;
  g.n0y = m.n0y;
  g.n0z = m.n0z;
  g.a = a;
  return g;
}

// LDS plane of one tile with a one-cell frame: (tx + 2) (256/tx + 2) values.
constexpr int kPlaneMaxF = 400;

// Marches a tile over [t.z0, t.z1) and calls f(z, i, v_i, sum_J g_IJ v_J, ctr)
// for the tile's cells inside the level, v = op.value(op.load(x, y, z, j))
// possibly formed on the fly and ctr = op.ctr(i) the cell's own further
// operands (D^-1, r).  Each plane of v with its x/y frame is formed once into
// LDS (double buffered), so v is evaluated about once per cell instead of at
// every neighbour; the neighbour terms are added in the order -x, +x, -y, +y,
// -z, +z.  Software pipelined: the loads of plane z+2 and the centre
// operands of plane z+1 are issued before plane z is computed.  Called by the
// whole workgroup (it synchronises).
template <bool UNI, typename OP, typename F, typename E>
__device__ inline void mg_plane(const Geo<UNI>& G, const Tile& t, int tx, long long base,
                                float (*lds)[kPlaneMaxF], const OP& op, F f, E epilogue) {
  using Raw = typename OP::Raw;
  using Ctr = typename OP::Ctr;
  const int ty = kBlock / tx;
  const int lx = (int)(threadIdx.x % tx), ly = (int)(threadIdx.x / tx);
  const int x = t.x0 + lx, y = t.y0 + ly;
  const bool valid = x < G.nx && y < G.ny;
  const int W = tx + 2;
  const int o = (ly + 1) * W + lx + 1;
  const int nframe = 2 * W + 2 * ty;
  const long long plane = (long long)G.nx * G.ny;
  // this thread's frame cell (at most one: nframe <= 256)
  const int k = threadIdx.x;
  const bool has_frame = k < nframe;
  int hx = 0, hy = 0;
  if (k < W) {
    hx = k;
    hy = 0;
  } else if (k < 2 * W) {
    hx = k - W;
    hy = ty + 1;
  } else if (k < 2 * W + ty) {
    hx = 0;
    hy = 1 + k - 2 * W;
  } else {
    hx = W - 1;
    hy = 1 + k - 2 * W - ty;
  }
  const int gx = t.x0 + hx - 1, gy = t.y0 + hy - 1;
  const bool fin = has_frame && gx >= 0 && gx < G.nx && gy >= 0 && gy < G.ny;
  const int fo = hy * W + hx;
  const long long fidx = fin ? gx + (long long)G.nx * gy : 0;
  const long long iidx = x + (long long)G.nx * y;
  Raw ri = op.zero(), rf = op.zero();
  auto load_plane = [&](int z) {
    const long long pz = base + plane * z;
    if (valid) ri = op.load(x, y, z, pz + iidx);
    if (fin) rf = op.load(gx, gy, z, pz + fidx);
  };
  auto store_plane = [&](float* buf) {
    buf[o] = valid ? op.value(ri) : 0.f;
    if (has_frame) buf[fo] = fin ? op.value(rf) : 0.f;
  };
  const int z0 = t.z0, z1 = t.z1;
  long long i = base + iidx + plane * z0;
  float* cur = lds[0];
  float* nxt = lds[1];
  __syncthreads();   // the previous tile's readers are done with both buffers
  load_plane(z0);
  float vm = (valid && z0 > 0) ? op.value(op.load(x, y, z0 - 1, i - plane)) : 0.f;
  Ctr cc = op.ctr_zero();
  if (valid) {
    if constexpr (OP::kCtrInRaw)
      cc = op.ctr_of(ri);
    else
      cc = op.ctr(i);
  }
  store_plane(cur);
  if (z0 + 1 < G.nz) load_plane(z0 + 1);
  __syncthreads();
  float vc = cur[o];
  for (int z = z0; z < z1; ++z) {
    const bool zr = z + 1 < G.nz;
    const bool more = z + 1 < z1;
    Ctr cn = op.ctr_zero();
    if constexpr (OP::kCtrInRaw) {   // plane z+1's raw operands are its centre operands
      if (more && valid) cn = op.ctr_of(ri);
    }
    if (zr) store_plane(nxt);
    if (more && z + 2 < G.nz) load_plane(z + 2);
    if constexpr (!OP::kCtrInRaw) cn = (more && valid) ? op.ctr(i + plane) : op.ctr_zero();
    float s = 0.f;
    if (valid) {
      if (x > 0) s += G.gx(x - 1, y, z) * cur[o - 1];
      if (x + 1 < G.nx) s += G.gx(x, y, z) * cur[o + 1];
      if (y > 0) s += G.gy(x, y - 1, z) * cur[o - W];
      if (y + 1 < G.ny) s += G.gy(x, y, z) * cur[o + W];
    }
    __syncthreads();
    const float vp = zr ? nxt[o] : 0.f;
    if (valid) {
      if (z > 0) s += G.gz(x, y, z - 1) * vm;
      if (zr) s += G.gz(x, y, z) * vp;
      f(z, i, vc, s, cc);
    }
    epilogue(z);   // every thread, every plane
    vm = vc;
    vc = vp;
    cc = cn;
    float* tmp = cur;
    cur = nxt;
    nxt = tmp;
    i += plane;
  }
}

template <bool UNI, typename OP, typename F>
__device__ inline void mg_plane(const Geo<UNI>& G, const Tile& t, int tx, long long base,
                                float (*lds)[kPlaneMaxF], const OP& op, F f) {
  mg_plane(G, t, tx, base, lds, op, f, [](int) {});
}

// Centre operands of the smoothers: D^-1 and r of the cell.
template <typename RT>
struct CtrDR {
  float dinv;
  RT r;
};

struct TileXY {
  int rep, x, y, z0, z1;
  bool valid;
};

__device__ inline TileXY tile_xy(const Tile* tiles, const MgRep* reps, int ti) {
  const Tile t = tiles[ti];
  const MgRep& m = reps[t.rep];
  TileXY c;
  c.rep = t.rep;
  c.x = t.x0 + (int)(threadIdx.x % m.tx);
  c.y = t.y0 + (int)(threadIdx.x / m.tx);
  c.z0 = t.z0;
  c.z1 = t.z1;
  c.valid = c.x < m.nx && c.y < m.ny;
  return c;
}

// Every kernel below loops over its workgroup's contiguous run of tiles.
#define FOR_MY_TILES(ntiles)   \
  int tile_b_, tile_e_;        \
  tile_range((ntiles), tile_b_, tile_e_); \
  for (int ti = tile_b_; ti < tile_e_; ++ti)

// ---- setup per solve -------------------------------------------------------

// Level 0: Dinv = 1 / (c + a deg).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_mg_prep0(MgLevel L0, const T* __restrict__ c) {
  FOR_MY_TILES(L0.ntiles) {
    const TileXY t = tile_xy(L0.tiles, L0.reps, ti);
    if (!t.valid) continue;
    const MgRep m = L0.reps[t.rep];
    const Geo<true> G = geo_of<true>(m);
    long long i = m.off + t.x + (long long)m.nx * (t.y + (long long)m.ny * t.z0);
    const long long plane = (long long)m.nx * m.ny;
    for (int z = t.z0; z < t.z1; ++z, i += plane)
      L0.dinv[i] = (float)(1.0 / ((double)c[i] + (double)G.gsum(t.x, t.y, z)));
  }
}

// Level k+1 from level k: c_{k+1} = sum of the children's c, Dinv_{k+1}.
// From level 0 (FROM0) the same pass also writes level 0's Dinv = 1 / (c +
// a deg) of every child (each level-0 cell is the child of exactly one
// level-1 cell), so level 0's c is read once.
template <bool FROM0, typename T>
__global__ void __launch_bounds__(kBlock) k_mg_coarsen(MgLevel Lf, MgLevel Lc,
                                                       const T* __restrict__ c0) {
  FOR_MY_TILES(Lc.nrtiles) {
    const TileXY t = tile_xy(Lc.rtiles, Lc.reps, ti);
    if (!t.valid) continue;
    const MgRep mc = Lc.reps[t.rep];
    const MgRep mf = Lf.reps[t.rep];
    const Geo<false> G = geo_of<false>(mc);
    const Geo<true> Gf = geo_of<true>(mf);
    for (int Z = t.z0; Z < t.z1; ++Z) {
      float s = 0.f;
      for (int dz = 0; dz < 2; ++dz) {
        const int z = 2 * Z + dz;
        if (z >= mf.nz) break;
        for (int dy = 0; dy < 2; ++dy) {
          const int y = 2 * t.y + dy;
          if (y >= mf.ny) break;
          for (int dx = 0; dx < 2; ++dx) {
            const int x = 2 * t.x + dx;
            if (x >= mf.nx) break;
            const long long j = mf.off + x + (long long)mf.nx * (y + (long long)mf.ny * z);
            if (FROM0) {
              const double cj = (double)c0[j];
              Lf.dinv[j] = (float)(1.0 / (cj + (double)Gf.gsum(x, y, z)));
              s += (float)cj;
            } else {
              s += Lf.c[j];
            }
          }
        }
      }
      const long long I = mc.off + t.x + (long long)mc.nx * (t.y + (long long)mc.ny * Z);
      Lc.c[I] = s;
      Lc.dinv[I] = 1.f / (s + G.gsum(t.x, t.y, Z));
    }
  }
}

// ---- V-cycle, global levels ------------------------------------------------

// First sweep from zero, formed on the fly at the neighbours: u1 = w D^-1 r.
template <typename RT>
struct OpPre {
  struct Raw {
    float dinv;
    RT r;
  };
  using Ctr = CtrDR<RT>;
  static constexpr bool kCtrInRaw = true;   // ctr_of(raw) instead of a second load
  const float* __restrict__ dinv;
  const RT* __restrict__ r;
  float omega;
  __device__ inline Raw zero() const { return Raw{0.f, (RT)0}; }
  __device__ inline Raw load(int, int, int, long long j) const { return Raw{dinv[j], r[j]}; }
  __device__ inline float value(const Raw& v) const { return omega * v.dinv * (float)v.r; }
  __device__ inline Ctr ctr_zero() const { return Ctr{0.f, (RT)0}; }
  __device__ inline Ctr ctr(long long i) const { return Ctr{dinv[i], r[i]}; }
  __device__ inline Ctr ctr_of(const Raw& v) const { return Ctr{v.dinv, v.r}; }
};

template <bool L0, typename RT>
__global__ void __launch_bounds__(kBlock) k_mg_pre(MgLevel Lk, float wa, float wb,
                                                   const RT* __restrict__ r, float* __restrict__ u,
                                                   const SolveScal* ss) {
  __shared__ float lds[2][kPlaneMaxF];
  FOR_MY_TILES(Lk.ntiles) {
    const Tile t = Lk.tiles[ti];
    if (ss[t.rep].done) continue;
    const MgRep m = Lk.reps[t.rep];
    const Geo<L0> G = geo_of<L0>(m);
    const OpPre<RT> op{Lk.dinv, r, wa};
    mg_plane(G, t, m.tx, m.off, lds, op,
             [&](int, long long i, float u1, float s, const CtrDR<RT>& c) {
               u[i] = (1.f - wb) * u1 + wb * c.dinv * ((float)c.r + s);
             });
  }
}
// Plain operand v = u with the cell's (D^-1, r) (second post-sweep, and the
// residual of the restriction).
template <typename RT>
struct OpU {
  struct Raw {
    float u;
  };
  using Ctr = CtrDR<RT>;
  static constexpr bool kCtrInRaw = false;
  const float* __restrict__ u;
  const float* __restrict__ dinv;
  const RT* __restrict__ r;
  __device__ inline Raw zero() const { return Raw{0.f}; }
  __device__ inline Raw load(int, int, int, long long j) const { return Raw{u[j]}; }
  __device__ inline float value(const Raw& v) const { return v.u; }
  __device__ inline Ctr ctr_zero() const { return Ctr{0.f, (RT)0}; }
  __device__ inline Ctr ctr(long long i) const { return Ctr{dinv[i], r[i]}; }
};

// Restriction r_{k+1}(I) = sum over the children of (r - A u), marched over
// the fine level's tiles: each cell's residual from the LDS plane of u, the
// 2 x 2 children of a coarse cell summed across lanes (tiles are 16 or 32
// columns wide, so a cell's x-neighbour is lane ^ 1 and its y-neighbour
// lane ^ tx, both in the same wavefront), the two child planes in a register.
// Tile origins are even in x, y and z.
template <bool L0, typename RT>
__global__ void __launch_bounds__(kBlock) k_mg_restrict(MgLevel Lf, MgLevel Lc,
                                                        const RT* __restrict__ r,
                                                        const SolveScal* ss) {
  __shared__ float lds[2][kPlaneMaxF];
  FOR_MY_TILES(Lf.ntiles) {
    const Tile t = Lf.tiles[ti];
    if (ss[t.rep].done) continue;
    const MgRep mf = Lf.reps[t.rep];
    const MgRep mc = Lc.reps[t.rep];
    const Geo<L0> G = geo_of<L0>(mf);
    const int tx = mf.tx;
    const int lx = (int)(threadIdx.x % tx), ly = (int)(threadIdx.x / tx);
    const int x = t.x0 + lx, y = t.y0 + ly;
    const bool lead = ((lx | ly) & 1) == 0 && x < mf.nx && y < mf.ny;
    float res = 0.f, acc = 0.f;
    const OpU<RT> op{Lf.u, Lf.dinv, r};
    mg_plane(G, t, tx, mf.off, lds, op,
             [&](int, long long, float uc, float s, const CtrDR<RT>& c) {
               res = (float)c.r - uc / c.dinv + s;
             },
             [&](int z) {
               float q = res + __shfl_xor(res, 1, 64);
               q = q + __shfl_xor(q, tx, 64);
               acc += q;
               res = 0.f;
               if ((z & 1) || z + 1 == mf.nz) {
                 if (lead)
                   Lc.r[mc.off + (x >> 1) + (long long)mc.nx * ((y >> 1) + (long long)mc.ny * (z >> 1))] = acc;
                 acc = 0.f;
               }
             });
  }
}

// Cell-centred linear prolongation, per axis: fine cell i of a level with nf
// cells takes 3/4 of its own aggregate I = i/2 and 1/4 of the neighbouring
// aggregate J on its side; at the lattice boundary, and inside or next to the
// single-cell aggregate of an odd edge, it takes its own aggregate alone.
__device__ inline void lin_axis(int i, int nf, int nc, int& I, int& J, float& wJ) {
  I = i >> 1;
  J = (i & 1) ? I + 1 : I - 1;
  wJ = 0.25f;
  const bool ragged = (nf & 1) != 0;
  if (J < 0 || J >= nc || (ragged && (I == nc - 1 || J == nc - 1))) {
    J = I;
    wJ = 0.f;
  }
}


// Post-smoothing after the coarse-grid correction: u3 = u2 + P e, then one
// weighted-Jacobi sweep of u3 into ualt.  P e is separable: a coarse plane Z
// interpolated in x and y to one of this thread's fine columns,
//     E_Z = (1 - wy) ((1 - wx) e[Z,Iy,Ix] + wx e[Z,Iy,Jx])
//           + wy ((1 - wx) e[Z,Jy,Ix] + wx e[Z,Jy,Jx]),
// serves every fine plane whose z interpolation takes Z (four of them), and a
// fine plane takes (1 - wz) E_Iz + wz E_Jz.  Each thread owns two columns (its
// interior cell and at most one frame cell of the tile) and keeps E of the
// coarse planes I - 1, I, I + 1 around the current fine plane's I = z / 2 in
// registers, the four coarse values of plane I + 2 in flight: four coarse
// loads per column per two fine planes instead of eight per cell.  The
// marching (one plane of u3 with its frame in LDS, double buffered, the
// loads of plane z + 2 issued before plane z is computed, neighbour terms in
// the order -x, +x, -y, +y, -z, +z) is that of mg_plane.
struct PCol {
  int o[4];    // offsets of (Iy,Ix), (Iy,Jx), (Jy,Ix), (Jy,Jx) within a coarse plane
  float wx, wy;
};

__device__ inline PCol pcol(int x, int y, int nfx, int nfy, const MgRep& mc) {
  int Ix, Jx, Iy, Jy;
  PCol c;
  lin_axis(x, nfx, mc.nx, Ix, Jx, c.wx);
  lin_axis(y, nfy, mc.ny, Iy, Jy, c.wy);
  c.o[0] = Iy * mc.nx + Ix;
  c.o[1] = Iy * mc.nx + Jx;
  c.o[2] = Jy * mc.nx + Ix;
  c.o[3] = Jy * mc.nx + Jx;
  return c;
}

// E of coarse plane Z (x first along each coarse row, then y)
__device__ inline float pcol_interp(const PCol& c, const float (&g)[4]) {
  const float r0 = (1.f - c.wx) * g[0] + c.wx * g[1];
  const float r1 = (1.f - c.wx) * g[2] + c.wx * g[3];
  return (1.f - c.wy) * r0 + c.wy * r1;
}

// The coarse-plane window of one column: E of planes I-1, I, I+1 and the raw
// values of plane I+2 (planes outside the level read as 0; they only ever
// enter with weight 0).
struct PWin {
  float em, e0, ep;
  float g[4];
};

template <bool L0, typename RT>
__global__ void __launch_bounds__(kBlock) k_mg_post1(MgLevel Lk, MgLevel Lc, const float* __restrict__ e,
                                                     float omega, const RT* __restrict__ r,
                                                     const SolveScal* ss) {
  __shared__ float lds[2][kPlaneMaxF];
  float* __restrict__ out = Lk.ualt;
  const float* __restrict__ u = Lk.u;
  const float* __restrict__ dinv = Lk.dinv;
  FOR_MY_TILES(Lk.ntiles) {
    const Tile t = Lk.tiles[ti];
    if (ss[t.rep].done) continue;
    const MgRep m = Lk.reps[t.rep];
    const MgRep mc = Lc.reps[t.rep];
    const Geo<L0> G = geo_of<L0>(m);
    const int tx = m.tx, ty = kBlock / tx;
    const int lx = (int)(threadIdx.x % tx), ly = (int)(threadIdx.x / tx);
    const int x = t.x0 + lx, y = t.y0 + ly;
    const bool valid = x < G.nx && y < G.ny;
    const int W = tx + 2;
    const int o = (ly + 1) * W + lx + 1;
    const int nframe = 2 * W + 2 * ty;
    const int k = threadIdx.x;
    const bool has_frame = k < nframe;
    int hx = 0, hy = 0;
    if (k < W) {
      hx = k;
      hy = 0;
    } else if (k < 2 * W) {
      hx = k - W;
      hy = ty + 1;
    } else if (k < 2 * W + ty) {
      hx = 0;
      hy = 1 + k - 2 * W;
    } else {
      hx = W - 1;
      hy = 1 + k - 2 * W - ty;
    }
    const int fx = t.x0 + hx - 1, fy = t.y0 + hy - 1;
    const bool fin = has_frame && fx >= 0 && fx < G.nx && fy >= 0 && fy < G.ny;
    const int fo = hy * W + hx;
    const long long plane = (long long)G.nx * G.ny;
    const long long fidx = fin ? fx + (long long)G.nx * fy : 0;
    const long long iidx = x + (long long)G.nx * y;
    const PCol ci = pcol(valid ? x : 0, valid ? y : 0, G.nx, G.ny, mc);
    const PCol cf = pcol(fin ? fx : 0, fin ? fy : 0, G.nx, G.ny, mc);
    const float* __restrict__ eb = e + mc.off;
    const long long csz = (long long)mc.nx * mc.ny;
    auto gather = [&](const PCol& c, bool on, int Z, float (&g)[4]) {
      if (on && Z >= 0 && Z < mc.nz) {
        const float* b = eb + csz * Z;
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = b[c.o[q]];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = 0.f;
      }
    };
    PWin wi, wf;
    int Iw;
    // window centred on coarse plane I (prologue: E of I-1, I, I+1 directly)
    auto win_start = [&](int I) {
      Iw = I;
      float g[4];
      gather(ci, valid, I - 1, g);
      wi.em = pcol_interp(ci, g);
      gather(ci, valid, I, g);
      wi.e0 = pcol_interp(ci, g);
      gather(ci, valid, I + 1, g);
      wi.ep = pcol_interp(ci, g);
      gather(ci, valid, I + 2, wi.g);
      gather(cf, fin, I - 1, g);
      wf.em = pcol_interp(cf, g);
      gather(cf, fin, I, g);
      wf.e0 = pcol_interp(cf, g);
      gather(cf, fin, I + 1, g);
      wf.ep = pcol_interp(cf, g);
      gather(cf, fin, I + 2, wf.g);
    };
    auto win_step = [&](PWin& w, const PCol& c, bool on) {
      w.em = w.e0;
      w.e0 = w.ep;
      w.ep = pcol_interp(c, w.g);
      gather(c, on, Iw + 2, w.g);
    };
    // P e of fine plane z at a column (the window moved to z / 2 first)
    auto pe = [&](const PWin& w, int z) {
      int Iz, Jz;
      float wz;
      lin_axis(z, G.nz, mc.nz, Iz, Jz, wz);
      if (Jz == Iz) return w.e0;
      return (1.f - wz) * w.e0 + wz * (Jz < Iz ? w.em : w.ep);
    };
    auto win_to = [&](int z) {
      if ((z >> 1) != Iw) {   // planes are formed in increasing z: one step
        ++Iw;
        win_step(wi, ci, valid);
        win_step(wf, cf, fin);
      }
    };
    float ui = 0.f, uf = 0.f;   // raw u of the next plane to form
    auto load_plane = [&](int z) {
      const long long pz = m.off + plane * z;
      if (valid) ui = u[pz + iidx];
      if (fin) uf = u[pz + fidx];
    };
    auto store_plane = [&](float* buf, int z) {
      win_to(z);
      buf[o] = valid ? ui + pe(wi, z) : 0.f;
      if (has_frame) buf[fo] = fin ? uf + pe(wf, z) : 0.f;
    };
    const int z0 = t.z0, z1 = t.z1;
    long long i = m.off + iidx + plane * z0;
    float* cur = lds[0];
    float* nxt = lds[1];
    __syncthreads();   // the previous tile's readers are done with both buffers
    win_start((z0 > 0 ? z0 - 1 : z0) >> 1);
    load_plane(z0);
    float vm = 0.f;
    if (z0 > 0) {
      const float um = valid ? u[i - plane] : 0.f;
      win_to(z0 - 1);
      vm = valid ? um + pe(wi, z0 - 1) : 0.f;
    }
    float cd = 0.f;
    RT cr = (RT)0;
    if (valid) {
      cd = dinv[i];
      cr = r[i];
    }
    store_plane(cur, z0);
    if (z0 + 1 < G.nz) load_plane(z0 + 1);
    __syncthreads();
    float vc = cur[o];
    for (int z = z0; z < z1; ++z) {
      const bool zr = z + 1 < G.nz;
      const bool more = z + 1 < z1;
      if (zr) store_plane(nxt, z + 1);
      if (more && z + 2 < G.nz) load_plane(z + 2);
      float nd = 0.f;
      RT nr = (RT)0;
      if (more && valid) {
        nd = dinv[i + plane];
        nr = r[i + plane];
      }
      float s = 0.f;
      if (valid) {
        if (x > 0) s += G.gx(x - 1, y, z) * cur[o - 1];
        if (x + 1 < G.nx) s += G.gx(x, y, z) * cur[o + 1];
        if (y > 0) s += G.gy(x, y - 1, z) * cur[o - W];
        if (y + 1 < G.ny) s += G.gy(x, y, z) * cur[o + W];
      }
      __syncthreads();
      const float vp = zr ? nxt[o] : 0.f;
      if (valid) {
        if (z > 0) s += G.gz(x, y, z - 1) * vm;
        if (zr) s += G.gz(x, y, z) * vp;
        out[i] = (1.f - omega) * vc + omega * cd * ((float)cr + s);
      }
      vm = vc;
      vc = vp;
      cd = nd;
      cr = nr;
      float* tmp = cur;
      cur = nxt;
      nxt = tmp;
      i += plane;
    }
  }
}
// One weighted-Jacobi sweep out = in + omega D^-1 (r - A in) (level 0's third
// pre- and post-sweep).
template <bool L0, typename RT>
__global__ void __launch_bounds__(kBlock) k_mg_sweep(MgLevel Lk, float omega, const float* __restrict__ in,
                                                     float* __restrict__ out, const RT* __restrict__ r,
                                                     const SolveScal* ss) {
  __shared__ float lds[2][kPlaneMaxF];
  FOR_MY_TILES(Lk.ntiles) {
    const Tile t = Lk.tiles[ti];
    if (ss[t.rep].done) continue;
    const MgRep m = Lk.reps[t.rep];
    const Geo<L0> G = geo_of<L0>(m);
    const OpU<RT> op{in, Lk.dinv, r};
    mg_plane(G, t, m.tx, m.off, lds, op,
             [&](int, long long i, float v, float s, const CtrDR<RT>& c) {
               out[i] = (1.f - omega) * v + omega * c.dinv * ((float)c.r + s);
             });
  }
}

template <bool L0, typename RT, typename ST>
__global__ void __launch_bounds__(kBlock) k_mg_post2(MgLevel Lk, float omega, const float* __restrict__ in,
                                                     const RT* __restrict__ r, SolverBufsT<ST> sb) {
  __shared__ double lds4[4];
  __shared__ float lds[2][kPlaneMaxF];
  FOR_MY_TILES(Lk.ntiles) {
    const Tile t = Lk.tiles[ti];
    if (sb.ss[t.rep].done) continue;
    const MgRep m = Lk.reps[t.rep];
    const Geo<L0> G = geo_of<L0>(m);
    double rz = 0.0;
    // level 0 reads the FP64 residual (for r.z): the cycle works on r sc
    const double sc = L0 ? sb.ss[t.rep].sc : 1.0, isc = L0 ? sb.ss[t.rep].isc : 1.0;
    float* const zo = cg_z(sb, sb.ss[t.rep].it);
    {
      const OpU<RT> op{in, Lk.dinv, r};
      mg_plane(G, t, m.tx, m.off, lds, op,
               [&](int, long long i, float u4, float s, const CtrDR<RT>& c) {
                 const float rs = L0 ? (float)((double)c.r * sc) : (float)c.r;
                 const float u5 = (1.f - omega) * u4 + omega * c.dinv * (rs + s);
                 if (L0) {
                   zo[i] = u5;
                   rz += (double)c.r * ((double)u5 * isc);
                 } else {
                   Lk.u[i] = u5;
                 }
               });
    }
    if (L0) {
      // level 0: partial r.z of this tile (finished by the RED_RZ reduce)
      rz = block_sum(rz, lds4);
      store_partials(sb.partial + (size_t)ti * 3, rz, 0.0, 0.0);
    }
  }
}

// ---- fused smoothing passes (temporal blocking) --------------------------------
//
// A pass makes S dependent Jacobi sweeps over a tile without leaving the
// workgroup (S = 3 on level 0, 2 below):
//   pre:  stage 0 u1 = w0 D^-1 r; stages 1 .. S-1 sweeps, the last written to
//         the level's u; stage S the residual r - A u, summed over the 2 x 2 x 2
//         children into the next level's r.
//   post: stage 0 u + P e; stages 1 .. S sweeps; on level 0 the last one is the
//         CG's z (FP32, scaled) and feeds its r.z partial.
//
// Layout.  A thread owns a strip of four cells in x, so that a stage's
// neighbours in x are its own registers and, at the strip's ends, the adjacent
// lanes' (one DPP move each); only the two neighbour rows go through LDS, as
// 16-byte reads.  A wavefront holds frpw rows of fe strips, a workgroup the rows of
// its wavefronts (up to kF3Block / 64; as many as the level's largest tile needs,
// MgLevel::fthreads): the tile's columns extended by one strip on either side in
// x and by S rows in y.  Stage s is valid on the rings up to
// S - s; the lanes beyond compute values that no valid cell reads, so no stage
// is masked.  D^-1, r and u are 0 outside the lattice, which keeps every
// stage's value there 0 and makes the neighbour sum the sum over the existing
// faces.  The tile marches through z: in the step for plane z the stages work
// on the planes z + S, ..., z.  A stage reads its neighbours' rows of the plane
// that the stage before wrote one step earlier, so one barrier per step orders
// everything; a cell's own values in z, and r and D^-1 of the S + 1 planes in
// flight, stay in registers, in slots that are compile-time constants since
// the march is unrolled by four planes (indexed by the plane number mod 4).
// The next plane's operands are loaded one step ahead.
//
// What bounds it: on large lattices HBM (halo rows mostly meet in the L2: the
// pre pass fetches 10.1 B per cell of its 8, the post pass 28 of 20.5), on
// small ones the latency of a step (LDS read, S dependent stages, barrier) at
// 12 wavefronts per CU.  Measured on one 384^3 lattice's three systems, all
// iterating: pre 705 -> 643 us, post 1475 -> 1051 us per V-cycle against one
// cell per thread with the ring columns dealt to a second slot, which was bound
// by its vector and scalar instructions (2.3 and 2.2 per cell and plane; now
// 0.8 and 0.4).  Workgroups of 384 threads, two per CU, took 705 and 1064 us
// (more halo); at four wavefronts per SIMD (128 registers) the post pass spills.
constexpr int kF3MaxStrips = 32;   // strips per row of the extended tile
// Strips of a plane in LDS for `threads` threads: the tile's rows, a row above
// and below, and slots that the lanes without a strip write to (with their
// neighbours' slots).  The 2 S stage planes are interleaved by strip
// (kF3Stride 16-byte values: 6, or 5 of which 4 are used, both free of bank
// conflicts), so that their offsets are constants at any workgroup size.
__host__ __device__ constexpr int f3_idle(int threads) { return threads + 2 * kF3MaxStrips; }
__host__ __device__ constexpr int f3_strips(int threads) { return f3_idle(threads) + 64 + kF3MaxStrips; }
template <int S>
struct F3Lds {
  static constexpr int kStride = S == 3 ? 6 : 5;
  static constexpr int kPlane = 16 * kStride;
};
template <int S>
int f3_lds_pre(int threads) { return f3_strips(threads) * (F3Lds<S>::kPlane + 16); }
template <int S>
int f3_lds_post(int threads) { return f3_strips(threads) * F3Lds<S>::kPlane + threads * 32; }

// Weights of a fused pass's sweeps, in stage order.
struct F3W {
  float w[3];
};

// Strip accesses are buffer instructions on the extended tile's part of a plane:
// a lane without a strip has the offset kNoLane, whose loads the hardware's
// range check turns into 0 and whose stores it drops, and a plane past the
// lattice's last has a range of 0.  So every step issues the same memory
// instructions with no branch around them, and the compiler's waits for a
// load count exactly the instructions issued after it (with branches it
// assumes the shortest path and waits for younger loads too, which undoes
// the loads' lead of two planes).  A strip is read whole at any alignment;
// cells past the lattice's end are zeroed by the reader.
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNoLane = 0x80000000u;

__device__ inline __amdgpu_buffer_rsrc_t strip_buf(const void* p, bool in) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, in ? 0x7fffffff : 0, 0x00020000);
}
__device__ inline f4 strip_load(__amdgpu_buffer_rsrc_t b, unsigned off) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, 0));
}
template <typename T>
struct StripVal;   // four stored values of r
template <>
struct StripVal<float> {
  f4 v;
  __device__ inline void load(__amdgpu_buffer_rsrc_t b, unsigned off) { v = strip_load(b, off); }
  __device__ inline float operator[](int i) const { return v[i]; }
  __device__ inline void clear(int i) { v[i] = 0.f; }
};
template <>
struct StripVal<double> {
  d2 a, b;
  __device__ inline void load(__amdgpu_buffer_rsrc_t buf, unsigned off) {
    a = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)off, 0, 0));
    b = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)(off + 16u), 0, 0));
  }
  __device__ inline double operator[](int i) const { return i < 2 ? a[i & 1] : b[i & 1]; }
  __device__ inline void clear(int i) {
    if (i < 2)
      a[i & 1] = 0.0;
    else
      b[i & 1] = 0.0;
  }
};
// Stores a strip (off: kNoLane on lanes that hold none); nv: its cells inside
// the lattice, read only where a strip of the wavefront is ragged.
__device__ inline void strip_store(__amdgpu_buffer_rsrc_t b, unsigned off, const float (&v)[4], int nv, bool ragged) {
  if (!ragged) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, f4{v[0], v[1], v[2], v[3]}), b, (int)off, 0, 0);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[i]), b, (int)(i < nv ? off + 4u * i : kNoLane), 0, 0);
  }
}

// The value of the lane below / above (0 at the wavefront's ends).
__device__ inline float lane_below(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));   // wave_shr:1
}
__device__ inline float lane_above(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));   // wave_shl:1
}

// A thread's place in its extended tile.
struct F3Own {
  int p;          // LDS strip index (one pad row above the first)
  unsigned vo;    // first cell, from the extended tile's first cell within a plane
  int x, y;       // first cell
  int nv;         // cells of the strip inside the lattice (0: none)
  bool active;    // the lane holds a strip
  bool inner;     // the strip belongs to the tile proper and to the lattice
};

__device__ inline F3Own f3_own(const Tile& t, const MgRep& m, int S) {
  F3Own f;
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int rw = lane / m.fe, e = lane - rw * m.fe;
  const int row = wave * m.frpw + rw;
  f.active = rw < m.frpw && row < m.fty + 2 * S;
  f.x = t.x0 + 4 * (e - 1);
  f.y = t.y0 + row - S;
  f.p = f.active ? (row + 1) * m.fe + e : f3_idle((int)blockDim.x) + lane;
  f.vo = (unsigned)(4 * e + m.nx * row);
  const bool in = f.active && f.x >= 0 && f.x < m.nx && f.y >= 0 && f.y < m.ny;
  f.nv = in ? min(4, m.nx - f.x) : 0;
  f.inner = in && e > 0 && e + 1 < m.fe && row >= S && row < S + m.fty;
  return f;
}

// Face couplings of a strip.  UNI: every cell is a full 2^k-cube, so a face
// couples with a 2^k (folded into `a`).  Otherwise the finite-volume coupling
// a (area / centre distance) of the cells' extents (ragged last cells),
// separable per axis; on full cubes the two agree bit for bit (every factor is
// a power of two).
template <bool UNI>
struct F3Geo {
  float a;
  __device__ inline void init(const Geo<false>&, const F3Own&, float a_) { a = a_; }
  __device__ inline void plane(const Geo<false>&, int) {}
  __device__ inline float nb(int, float xm, float xp, float ym, float yp, float zm, float zp) const {
    return ((xm + xp) + (ym + yp)) + (zm + zp);
  }
};
template <>
struct F3Geo<false> {
  float a;
  float ex[4], X[5], ey, Ym, Yp;   // extents; inverse centre distances (X[i]: between x - 1 + i and x + i)
  float ez, Zm, Zp;
  __device__ static inline float ext(int I, int n, int k, int n0) {
    return (I >= 0 && I < n) ? (float)(min((I + 1) << k, n0) - (I << k)) : (float)(1 << k);
  }
  __device__ inline void init(const Geo<false>& G, const F3Own& f, float a_) {
    a = a_;
    float e[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) e[i] = ext(f.x - 1 + i, G.nx, G.k, G.n0x);
#pragma unroll
    for (int i = 0; i < 4; ++i) ex[i] = e[i + 1];
#pragma unroll
    for (int i = 0; i < 5; ++i) X[i] = 2.f / (e[i] + e[i + 1]);
    ey = ext(f.y, G.ny, G.k, G.n0y);
    Ym = 2.f / (ext(f.y - 1, G.ny, G.k, G.n0y) + ey);
    Yp = 2.f / (ey + ext(f.y + 1, G.ny, G.k, G.n0y));
  }
  // factors of the plane z that a stage works on
  __device__ inline void plane(const Geo<false>& G, int z) {
    ez = ext(z, G.nz, G.k, G.n0z);
    Zm = 2.f / (ext(z - 1, G.nz, G.k, G.n0z) + ez);
    Zp = 2.f / (ez + ext(z + 1, G.nz, G.k, G.n0z));
  }
  __device__ inline float nb(int i, float xm, float xp, float ym, float yp, float zm, float zp) const {
    const float sx = fmaf(X[i + 1], xp, X[i] * xm);
    const float sy = fmaf(Yp, yp, Ym * ym);
    const float sz = fmaf(Zp, zp, Zm * zm);
    return fmaf(ex[i] * ey, sz, fmaf(ex[i] * ez, sy, (ey * ez) * sx));
  }
};

// The first plane a tile [z0, z1) marches from: S below it (0 at least), where
// S = 2 (z0 is even); S = 3's r.z groups want a multiple of four.
template <int S>
__device__ inline int f3_first_plane(int z0) {
  return S == 2 ? max(z0 - 2, 0) : max(z0 - 4, 0) & ~3;
}

// The marching of both passes over a tile: stage 0's planes in groups
// of four, each plane's step specialised for its number in the group.  From
// f3_first_plane (the planes below the lattice are 0) to the S above the tile.
// A stage skips the planes that the tile does not depend on (a quarter of the
// sweeps of a 16-plane tile; three sweeps in four of a lattice of one plane:
// level 0 of 117 x 103 x 91 with five systems, post 39.4 -> 35.7 us; 128^3, pre 27.4
// -> 24.9).
template <int S, typename STEP>
__device__ inline void f3_march(int z0, int z1, bool active, STEP step) {
  const int zf = f3_first_plane<S>(z0);
  if (active) {
    for (int z = zf; z < z1 + S; z += 4) {
      step(z, std::integral_constant<int, 0>());
      step(z + 1, std::integral_constant<int, 1>());
      step(z + 2, std::integral_constant<int, 2>());
      step(z + 3, std::integral_constant<int, 3>());
    }
  } else {
    for (int z = zf; z < z1 + S; z += 4)
#pragma unroll
      for (int k = 0; k < 4; ++k) __syncthreads();
  }
}

// Sum of the six neighbours' stage values of cell i: `u` the strip's own
// values in the plane, rows from LDS, z neighbours below and above.
#define F3_NB(i, u, lo, hi, ym, yp, zm, zp)                                                             \
  geo.nb(i, (i) == 0 ? (lo) : (u)[(i) == 0 ? 0 : (i)-1], (i) == 3 ? (hi) : (u)[(i) == 3 ? 3 : (i) + 1], \
         (ym)[i], (yp)[i], (zm)[i], (zp)[i])

// One weighted-Jacobi sweep of a cell: u + w (D^-1 (r + a nb) - u).  P32
// (precision 32): in the form (1 - w) u + (w D^-1) (r + a nb) and with the
// roundings of one kernel per cell, which the stored fields' last bits follow.
template <bool P32>
__device__ inline float f3_sweep(float w, float d, float r, float a, float nb, float u) {
  const float t = fmaf(a, nb, r);
  return P32 ? fmaf(1.f - w, u, (w * d) * t) : fmaf(w, fmaf(d, t, -u), u);
}

// The first sweep from zero, w D^-1 r, rounded (not contracted into the sums
// that take it).
__device__ inline float f3_first(float w, float d, float r) {
#pragma clang fp contract(off)
  return w * d * r;
}

// Pre-smoothing and restriction of one level.  On level 0 in precision 32
// (whose r is FP32 already) r is scaled by the system's power of two here;
// otherwise it is the scaled FP32 copy or a coarser level's r.
template <int S, bool UNI, bool P32>
__global__ void __launch_bounds__(kF3Block, 3) k_mg_prefused(MgLevel Lk, MgLevel Lc, F3W w, float ascale,
                                                             const float* __restrict__ r, const SolveScal* ss) {
  extern __shared__ __attribute__((aligned(16))) float4 lds_f3[];
  constexpr int kSt = F3Lds<S>::kStride;
  constexpr bool kDiv = S == 2 && !P32;   // the residual's u / D^-1 rounded as one kernel per sweep rounds it
  float4* const sV = lds_f3;   // [strip][stage][parity]
  const int nstrips = f3_strips((int)blockDim.x);
  float2* const sQ = reinterpret_cast<float2*>(lds_f3 + nstrips * kSt);   // [strip][parity]: residual sums over x
                                                                          // pairs of the odd rows
  const Tile t = Lk.ftiles[blockIdx.x];
  if (t.rep < 0 || ss[t.rep].done) return;
  const MgRep m = Lk.reps[t.rep];
  const MgRep mc = Lc.reps[t.rep];
  const F3Own f = f3_own(t, m, S);
  const int fe = m.fe, nz = m.nz;
  const Geo<false> G = geo_of<false>(m);
  F3Geo<UNI> geo;
  geo.init(G, f, UNI ? m.a * ascale : m.a);
  const long long plane = (long long)m.nx * m.ny;
  // the extended tile's first cell in the plane that is loaded next (uniform,
  // and kept opaque to the compiler, which would otherwise carry one pointer
  // per array and unrolled plane), and the strip's byte offsets from it
  long long at = m.off + t.x0 - 4 + (long long)m.nx * (t.y0 - S) + plane * f3_first_plane<S>(t.z0);
  const unsigned vo = f.nv > 0 ? 4u * f.vo : kNoLane;
  const unsigned io = f.inner ? 4u * f.vo : kNoLane;
  const int sce = P32 && S == 3 ? ilogb(ss[t.rep].sc) : 0;
  const int z0 = t.z0, z1 = t.z1;
  for (int k = threadIdx.x; k < nstrips * (kSt + 1); k += blockDim.x) lds_f3[k] = float4{0.f, 0.f, 0.f, 0.f};
  const bool wact = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) * m.frpw < m.fty + 2 * S);
  const bool ragged = __ballot(f.nv > 0 && f.nv < 4) != 0;   // a strip of the wavefront straddles the lattice's end
  const bool lead = f.inner && ((f.y & 1) == 0), odd = f.inner && ((f.y & 1) != 0);
  float h[S][2][4];        // a stage's values at the two newest planes, by plane parity
  float rh[4][4], dh[4][4];   // r, D^-1 by step mod 4
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int s = 0; s < S; ++s) h[s][0][i] = h[s][1][i] = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) rh[k][i] = dh[k][i] = 0.f;
  }
  // operands of the next two planes, by plane parity
  f4 nr[2], nd[2];
  const int zlim = min(nz, z1 + S);   // the tile depends on the planes below
  auto fetch = [&](int z, int q) {   // plane z, at `at`, into slot q
    const bool in = z < zlim;
    nr[q] = strip_load(strip_buf(r + at, in), vo);
    nd[q] = strip_load(strip_buf(Lk.dinv + at, in), vo);
  };
  float q0 = 0.f, q1 = 0.f, acc0 = 0.f, acc1 = 0.f;
  // the residual sums of plane z, complete once the odd rows' are in LDS; the
  // coarse cells' after their second plane
  const unsigned c0 = lead ? 4u * (unsigned)(((f.x - t.x0) >> 1) + mc.nx * ((f.y - t.y0) >> 1)) : kNoLane;
  const unsigned c1 = lead && f.x + 2 < m.nx ? c0 + 4u : kNoLane;
  const long long cat = mc.off + (t.x0 >> 1) + (long long)mc.nx * (t.y0 >> 1);
  auto take_pair = [&](int z, int q, bool last) {
    const float2 o = sQ[2 * (f.p + fe) + q];
    acc0 += q0 + o.x;
    acc1 += q1 + o.y;
    if (last) {
      const auto b = strip_buf(Lc.r + (cat + (long long)mc.nx * mc.ny * (z >> 1)), true);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc0), b, (int)c0, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc1), b, (int)c1, 0, 0);
      acc0 = acc1 = 0.f;
    }
  };
  {
    const int zf = f3_first_plane<S>(z0);
    fetch(zf, 0);
    at += plane;
    fetch(zf + 1, 1);
  }
  __syncthreads();
  auto step = [&](int z, auto K) {   // z: stage 0's plane
    constexpr int k = decltype(K)::value, wb = k & 1, rb = wb ^ 1;
    {
      float nv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        rh[k][i] = P32 && S == 3 ? ldexpf(nr[wb][i], sce) : nr[wb][i];
        dh[k][i] = nd[wb][i];
      }
      if (ragged) {
#pragma unroll
        for (int i = 1; i < 4; ++i)
          if (i >= f.nv) rh[k][i] = dh[k][i] = 0.f;
      }
      at += plane;
      asm volatile("" : "+s"(at));
      fetch(z + 2, wb);
#pragma unroll
      for (int i = 0; i < 4; ++i) nv[i] = f3_first(w.w[0], dh[k][i], rh[k][i]);
#pragma unroll
      for (int s = 1; s <= S; ++s) {   // stage s at plane z - s, from stage s - 1
        constexpr int kk[4] = {k, (k + 3) & 3, (k + 2) & 3, (k + 1) & 3};
        const int zs = z - s;
        float out[4] = {0.f, 0.f, 0.f, 0.f};
        if (zs >= max(z0 - (S - s), 0) && zs < min(z1 + (S - s), nz)) {   // a plane the tile depends on
          const float4 ym4 = sV[(f.p - fe) * kSt + 2 * (s - 1) + rb], yp4 = sV[(f.p + fe) * kSt + 2 * (s - 1) + rb];
          const float ym[4] = {ym4.x, ym4.y, ym4.z, ym4.w}, yp[4] = {yp4.x, yp4.y, yp4.z, yp4.w};
          const float* u = h[s - 1][rb];
          const float lo = lane_below(u[3]), hi = lane_above(u[0]);
          geo.plane(G, zs);
          if (s < S) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              out[i] = f3_sweep<P32>(w.w[s], dh[kk[s]][i], rh[kk[s]][i], geo.a,
                                     F3_NB(i, u, lo, hi, ym, yp, h[s - 1][wb], nv), u[i]);
            if (s == S - 1)
              strip_store(strip_buf(Lk.u + (at - (s + 2) * plane), zs >= z0 && zs < z1), io, out, f.nv, ragged);
          } else if (zs >= z0 && zs < z1) {   // residual, summed over x pairs
            if (zs > z0) take_pair(zs - 1, rb, ((k - S) & 1) == 0);   // zs - 1 odd
            float res[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float d = dh[kk[s]][i];
              const float rcp = __builtin_amdgcn_rcpf(d);
              float c;
              if (kDiv) {
                const float q = u[i] * rcp;
                c = rh[kk[s]][i] - fmaf(fmaf(-q, d, u[i]), rcp, q);
              } else {
                c = fmaf(-u[i], rcp, rh[kk[s]][i]);
              }
              res[i] = fmaf(geo.a, F3_NB(i, u, lo, hi, ym, yp, h[s - 1][wb], nv), c);
            }
            if (ragged) {
#pragma unroll
              for (int i = 1; i < 4; ++i)
                if (i >= f.nv) res[i] = 0.f;
            }
            q0 = res[0] + res[1];
            q1 = res[2] + res[3];
            if (odd) sQ[2 * f.p + wb] = float2{q0, q1};
          }
        }
        // stage s - 1's new plane: registers and LDS
#pragma unroll
        for (int i = 0; i < 4; ++i) h[s - 1][wb][i] = nv[i];
        sV[f.p * kSt + 2 * (s - 1) + wb] = float4{nv[0], nv[1], nv[2], nv[3]};
#pragma unroll
        for (int i = 0; i < 4; ++i) nv[i] = out[i];
      }
    }
    __syncthreads();
  };
  f3_march<S>(z0, z1, wact, step);
  if (wact) take_pair(z1 - 1, (z1 + S - 1) & 1, true);
}

// Prolongation and post-smoothing of one level; e the next level's
// correction.  The prolongation is the cell-centred linear interpolation of
// lin_axis: where an axis takes its own aggregate alone, the other
// aggregate's value is replaced by it.
template <int S, bool UNI, bool ZOUT, bool P32, typename ST>
__global__ void __launch_bounds__(kF3Block, 3) k_mg_postfused(MgLevel Lk, MgLevel Lc, const float* __restrict__ e,
                                                              F3W w, float ascale, const float* __restrict__ r,
                                                              float* __restrict__ out, SolverBufsT<ST> sb,
                                                              double* __restrict__ colsum) {
  __shared__ double sRz[kF3Block / 64];
  extern __shared__ __attribute__((aligned(16))) float4 lds_f3[];
  constexpr int kSt = F3Lds<S>::kStride;
  float4* const sV = lds_f3;   // [strip][stage][parity]
  const int nstrips = f3_strips((int)blockDim.x);
  float4* const sE = lds_f3 + nstrips * kSt + 2 * threadIdx.x;   // the strip's correction on its two coarse planes
                                                                  // (by plane parity; its owner's alone)
  const Tile t = Lk.ftiles[blockIdx.x];
  if (t.rep < 0 || sb.ss[t.rep].done) return;
  float* const zo = ZOUT ? cg_z(sb, sb.ss[t.rep].it) : out;
  const MgRep m = Lk.reps[t.rep];
  const MgRep mc = Lc.reps[t.rep];
  const F3Own f = f3_own(t, m, S);
  const int fe = m.fe, nz = m.nz;
  const Geo<false> G = geo_of<false>(m);
  F3Geo<UNI> geo;
  geo.init(G, f, UNI ? m.a * ascale : m.a);
  const long long plane = (long long)m.nx * m.ny;
  // the extended tile's first cell in the plane that is loaded next (uniform,
  // and kept opaque to the compiler, which would otherwise carry one pointer
  // per array and unrolled plane), and the strip's byte offsets from it
  long long at = m.off + t.x0 - 4 + (long long)m.nx * (t.y0 - S) + plane * f3_first_plane<S>(t.z0);
  const unsigned vo = f.nv > 0 ? 4u * f.vo : kNoLane;
  const unsigned io = f.inner ? 4u * f.vo : kNoLane;
  const int sce = P32 && S == 3 ? ilogb(sb.ss[t.rep].sc) : 0;
  const int z0 = t.z0, z1 = t.z1;
  for (int k = threadIdx.x; k < nstrips * kSt; k += blockDim.x) lds_f3[k] = float4{0.f, 0.f, 0.f, 0.f};
  if (ZOUT && threadIdx.x < kF3Block / 64) sRz[threadIdx.x] = 0.0;
  const bool wact = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) * m.frpw < m.fty + 2 * S);
  const bool ragged = __ballot(f.nv > 0 && f.nv < 4) != 0;
  // the strip's coarse cells: x / 2 - 1 .. x / 2 + 2 of the rows Iy and Jy
  const int I0 = f.x >> 1;
  bool own[4], owny = true;   // the cell takes its own aggregate alone in x, in y
  // byte offsets of the rows from the first aggregate of the extended tile
  // in a coarse plane, which is at `eat` in the plane to load next
  const int X0 = t.x0 / 2 - 3, Y0 = max(0, (t.y0 - S) / 2 - 1);
  unsigned e0 = kNoLane, e1 = kNoLane;
  long long eat = mc.off + X0 + (long long)mc.nx * Y0;
  {
    int I, J;
    float wj;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      lin_axis(f.x + i, m.nx, mc.nx, I, J, wj);
      own[i] = J == I;
    }
    if (f.nv > 0) {
      lin_axis(f.y, m.ny, mc.ny, I, J, wj);
      owny = J == I;
      e0 = 4u * (unsigned)(mc.nx * (I - Y0) + I0 - 1 - X0);
      e1 = 4u * (unsigned)(mc.nx * (J - Y0) + I0 - 1 - X0);
    }
  }
  const long long cplane = (long long)mc.nx * mc.ny;
  const int ncz = mc.nz;
  f4 g0, g1;   // coarse values in flight (one coarse plane)
  auto fetch_e = [&](int Z) {   // at `eat` (planes past the last are never taken)
    const auto b = strip_buf(e + eat, Z < ncz);
    g0 = strip_load(b, e0);
    g1 = strip_load(b, e1);
  };
  auto make_e = [&](int q) {   // the correction interpolated in x and y

    auto line = [&](const f4& g, float (&v)[4]) {
      v[0] = own[0] ? g[1] : fmaf(0.75f, g[1], 0.25f * g[0]);
      v[1] = own[1] ? g[1] : fmaf(0.75f, g[1], 0.25f * g[2]);
      v[2] = own[2] ? g[2] : fmaf(0.75f, g[2], 0.25f * g[1]);
      v[3] = own[3] ? g[2] : fmaf(0.75f, g[2], 0.25f * g[3]);
    };
    float a[4], b[4];
    line(g0, a);
    line(g1, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = owny ? a[i] : fmaf(0.75f, a[i], 0.25f * b[i]);
    const float4 o{a[0], a[1], a[2], a[3]};
    sE[q] = o;
  };
  float h[S][2][4];
  f4 rh[4], dh[4];   // by step mod 4; a plane's are loaded when the plane four below is done with
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int s = 0; s < S; ++s) h[s][0][i] = h[s][1][i] = 0.f;
  }
  // u of the next two planes, by plane parity; the stored r of the tile's own
  // cells for r.z, one plane ahead
  f4 nu[2];
  StripVal<ST> rq;
  const int zlim = min(nz, z1 + S);   // the tile depends on the planes below
  auto fetch_u = [&](int z, int q) { nu[q] = strip_load(strip_buf(Lk.u + at, z < zlim), vo); };   // plane z is at `at`
  auto fetch_rd = [&](int z, int q) {   // plane z is one below `at`
    rh[q] = strip_load(strip_buf(r + (at - plane), z < zlim), vo);
    dh[q] = strip_load(strip_buf(Lk.dinv + (at - plane), z < zlim), vo);
  };
#pragma unroll
  for (int k = 0; k < 4; ++k) rh[k] = dh[k] = 0.f;
  const unsigned ir = f.inner ? (unsigned)sizeof(ST) * f.vo : kNoLane;
  if constexpr (ZOUT) rq.load(strip_buf(sb.r + at, false), ir);
  double rz = 0.0;
  double rzc[4] = {0.0, 0.0, 0.0, 0.0};   // precision 32: per column
  const int zf = f3_first_plane<S>(z0);
  const bool zrag = (nz & 1) != 0;
  // E of zf's own coarse plane and of the one below
  if (zf > 0) {
    eat += cplane * ((zf >> 1) - 1);
    fetch_e((zf >> 1) - 1);
    make_e(1);
    eat += cplane;
  } else {
    sE[1] = float4{0.f, 0.f, 0.f, 0.f};
  }
  fetch_e(zf >> 1);
  make_e(0);
  eat += cplane;
  fetch_e((zf >> 1) + 1);   // for the first odd plane's step
  fetch_u(zf, 0);
  at += plane;
  fetch_rd(zf, 0);
  fetch_u(zf + 1, 1);
  __syncthreads();
  const int gmask = m.fgroup - 1;
  // r.z of the group of planes that ends with z: one partial per gmask + 1
  // planes of a tile column, whatever the tile's depth, so that the sum does
  // not depend on how the batch's lattices are cut in z
  auto put_rz = [&](int z) {
    if (threadIdx.x == 0) {
      double tsum = 0.0;
      for (int k = 0; k < kF3Block / 64; ++k) tsum += sRz[k];
      store_partials(sb.partial + (size_t)(t.part + (z - z0) / (gmask + 1)) * 3, tsum * sb.ss[t.rep].isc, 0.0, 0.0);
    }
  };
  auto step = [&](int z, auto K) {
    constexpr int k = decltype(K)::value, wb = k & 1, rb = wb ^ 1;
    {
      constexpr int eI = k >> 1, eJ = eI ^ 1;   // E of plane z / 2 and of the other one z takes
      const int Z = z >> 1;
      if (k & 1) {   // plane Z + 1, loaded two steps before
        make_e(eJ);
        eat += cplane;
        asm volatile("" : "+s"(eat));
        fetch_e(Z + 2);
      }
      float nv[4];
      {
        const int J = (k & 1) ? Z + 1 : Z - 1;
        const bool alone = J < 0 || J >= ncz || (zrag && (Z == ncz - 1 || J == ncz - 1));
        // weights of E (0 past the last plane; lanes without a strip have E = 0)
        const float wJ = z >= nz || alone ? 0.f : 0.25f, wI = z >= nz ? 0.f : 1.f - wJ;
        const float4 eI4 = sE[eI], eJ4 = sE[eJ];
        const float E[2][4] = {{eI4.x, eI4.y, eI4.z, eI4.w}, {eJ4.x, eJ4.y, eJ4.z, eJ4.w}};
        constexpr int k1 = (k + 3) & 3;   // the plane below, whose r and D^-1 stage 1 takes now
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (P32 && S == 3) rh[k1][i] = ldexpf(rh[k1][i], sce);
          nv[i] = nu[wb][i] + fmaf(wI, E[0][i], wJ * E[1][i]);
        }
        if (ragged) {
#pragma unroll
          for (int i = 1; i < 4; ++i)
            if (i >= f.nv) rh[k1][i] = dh[k1][i] = nv[i] = 0.f;
        }
      }
      at += plane;
      asm volatile("" : "+s"(at));
      fetch_u(z + 2, wb);
#pragma unroll
      for (int s = 1; s <= S; ++s) {
        constexpr int kk[4] = {k, (k + 3) & 3, (k + 2) & 3, (k + 1) & 3};
        const int zs = z - s;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (zs >= max(z0 - (S - s), 0) && zs < min(z1 + (S - s), nz)) {   // a plane the tile depends on
          const float4 ym4 = sV[(f.p - fe) * kSt + 2 * (s - 1) + rb], yp4 = sV[(f.p + fe) * kSt + 2 * (s - 1) + rb];
          const float ym[4] = {ym4.x, ym4.y, ym4.z, ym4.w}, yp[4] = {yp4.x, yp4.y, yp4.z, yp4.w};
          const float* u = h[s - 1][rb];
          const float lo = lane_below(u[3]), hi = lane_above(u[0]);
          geo.plane(G, zs);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            v[i] = f3_sweep<P32>(w.w[s - 1], dh[kk[s]][i], rh[kk[s]][i], geo.a,
                                 F3_NB(i, u, lo, hi, ym, yp, h[s - 1][wb], nv), u[i]);
          if (s == S) {
            const bool mine = zs >= z0 && zs < z1;
            strip_store(strip_buf(zo + (at - (S + 2) * plane), mine), io, v, f.nv, ragged);
            if constexpr (ZOUT) {
              // (lanes and planes that are not the tile's have r = 0 here)
              if (ragged) {
#pragma unroll
                for (int i = 1; i < 4; ++i)
                  if (i >= f.nv) rq.clear(i);
              }
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                if (P32)
                  rzc[i] = fma((double)rq[i], (double)v[i], rzc[i]);
                else
                  rz = fma((double)rq[i], (double)v[i], rz);
              }
            }
          }
          if constexpr (ZOUT && !P32) {
            // zs is the last plane of a group in one step of four at most
            if (s == S && ((k - S) & 3) == 3 && (zs & gmask) == gmask && zs >= z0 && zs < z1) {
              rz = wave_sum(rz);
              if ((threadIdx.x & 63) == 0) sRz[threadIdx.x >> 6] = rz;
              rz = 0.0;
            }
            if (s == S && ((k - S) & 3) == 0 && (zs & gmask) == 0 && zs > z0 && zs < z1) put_rz(zs - 1);
          }
        }
        if (s == S) {
          fetch_rd(z + 1, (k + 1) & 3);
          if constexpr (ZOUT)
            rq.load(strip_buf(sb.r + (at - (S + 1) * plane), zs + 1 >= z0 && zs + 1 < z1), ir);   // the next plane's
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) h[s - 1][wb][i] = nv[i];
        sV[f.p * kSt + 2 * (s - 1) + wb] = float4{nv[0], nv[1], nv[2], nv[3]};
#pragma unroll
        for (int i = 0; i < 4; ++i) nv[i] = v[i];
      }
    }
    __syncthreads();
  };
  f3_march<S>(z0, z1, wact, step);
  if constexpr (ZOUT && P32) {
    if (f.inner) {
      double* o = colsum + m.col_off + t.part * plane + f.x + (long long)m.nx * f.y;
      const double isc = sb.ss[t.rep].isc;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < f.nv) o[i] = rzc[i] * isc;
    }
  }
  if constexpr (ZOUT && !P32) {
    if ((z1 & gmask) != 0) {   // the lattice's last, shorter group
      rz = wave_sum(rz);
      if ((threadIdx.x & 63) == 0) sRz[threadIdx.x >> 6] = rz;
      __syncthreads();
    }
    put_rz(z1 - 1);
  }
}

// Precision 32: r.z summed from the post pass's column sums (over the depth of
// its tiles) per tile of tx x 512 / tx columns, wavefront butterfly, then the
// wavefronts in turn.  Its rounding reaches the stored fields: FP32 storage
// turns the last bit of beta into flipped last bits of a field, which the
// fitted guess of the next solves spreads over the lattice, so this order is
// kept whatever the smoothing tiles are.
__global__ void __launch_bounds__(kRzBlock) k_mg_rz32(MgLevel L0, const double* __restrict__ colsum,
                                                      double* __restrict__ partial, const SolveScal* ss) {
  __shared__ double sum[kRzBlock / 64];
  const Tile t = L0.rztiles[blockIdx.x];
  if (ss[t.rep].done) return;
  const MgRep m = L0.reps[t.rep];
  const int x = t.x0 + (int)threadIdx.x % m.tx, y = t.y0 + (int)threadIdx.x / m.tx;
  double rz = x < m.nx && y < m.ny ? colsum[m.col_off + x + (long long)m.nx * (y + (long long)m.ny * t.part)] : 0.0;
  rz = wave_sum(rz);
  if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = rz;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tsum = 0.0;
    for (int k = 0; k < kRzBlock / 64; ++k) tsum += sum[k];
    store_partials(partial + (size_t)blockIdx.x * 3, tsum, 0.0, 0.0);
  }
}

#undef F3_NB

// ---- coarse levels: one workgroup per system, in LDS --------------------------

// A level of a system's coarse solve: dims (those of level kc halved j times,
// rounded up) and the cells of the levels kc+1 .. before it, by which its
// blocks lie in LDS and in the precomputed block.
struct CoarseLevel {
  int nx, ny, nz, n, plane, before;
};

__device__ inline CoarseLevel coarse_level(const MgCoarseRep& cr, int j, int before) {
  CoarseLevel L;
  const int up = (1 << j) - 1;
  L.nx = (cr.dims[0] + up) >> j;
  L.ny = (cr.dims[1] + up) >> j;
  L.nz = (cr.dims[2] + up) >> j;
  L.plane = L.nx * L.ny;
  L.n = L.plane * L.nz;
  L.before = before;
  return L;
}

// Coordinates of cell t (t < 2^13): the float quotient (t + 1/2) / nx is at
// least 1/(2 nx) from an integer and its error below 2^-21 of it, far less.
__device__ inline void cell_xyz(const CoarseLevel& L, int t, int& x, int& y, int& z) {
  const int q = (int)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)L.nx));
  x = t - __mul24(q, L.nx);
  z = (int)(((float)q + 0.5f) * __builtin_amdgcn_rcpf((float)L.ny));
  y = q - __mul24(z, L.ny);
}

// One cell of a level as its thread holds it: D^-1, the residual and the
// couplings to the neighbours -x, +x, -y, +y, -z, +z (0 at a missing face).
struct CoarseCell {
  float d, r, g[6];
};

// sum_J g_IJ v(J) over the neighbours of cell t, in the order -x, +x, -y, +y,
// -z, +z (FLAT: a level of one plane).  No coordinates and no bounds: a missing
// face has the coupling 0, and v lies in LDS between finite numbers, a
// neighbour's place being at most a level's cells away.
template <bool FLAT>
__device__ inline float coarse_nbsum(const CoarseLevel& L, const CoarseCell& c, const float* v, int t) {
  const float* w = v + t;
  float s = c.g[0] * w[-1];
  s += c.g[1] * w[1];
  s += c.g[2] * w[-L.nx];
  s += c.g[3] * w[L.nx];
  if (!FLAT) {
    s += c.g[4] * w[-L.plane];
    s += c.g[5] * w[L.plane];
  }
  return s;
}

// D^-1 and the couplings of cell t from a level's block [gz | gy | gx | D^-1]
// (couplings to +x, +y, +z, 0 at the upper edges; those of the cells before
// t are the ones to its lower neighbours: 0 again at the lower edges, where
// they are an upper edge's of the row, the plane or the array before).
template <bool FLAT>
__device__ inline void coarse_cell(const CoarseLevel& L, const float* blk, int t, CoarseCell& c) {
  const float *gz = blk + t, *gy = gz + L.n, *gx = gy + L.n;
  c.d = gx[L.n];
  c.g[0] = gx[-1];
  c.g[1] = gx[0];
  c.g[2] = gy[-L.nx];
  c.g[3] = gy[0];
  if (!FLAT) {
    const float gzm = blk[max(t - L.plane, 0)];
    c.g[4] = t >= L.plane ? gzm : 0.f;
    c.g[5] = gz[0];
  }
}

// The couplings of cell (x, y, z) of a level whose cells are all alike: g along each axis.
template <bool FLAT>
__device__ inline void coarse_alike(const CoarseLevel& L, const float (&g)[3], int x, int y, int z, CoarseCell& c) {
  c.g[0] = x > 0 ? g[0] : 0.f;
  c.g[1] = x + 1 < L.nx ? g[0] : 0.f;
  c.g[2] = y > 0 ? g[1] : 0.f;
  c.g[3] = y + 1 < L.ny ? g[1] : 0.f;
  if (!FLAT) {
    c.g[4] = z > 0 ? g[2] : 0.f;
    c.g[5] = z + 1 < L.nz ? g[2] : 0.f;
  }
}

// u2 of the two sweeps from zero (dr: D^-1 r of the level)
template <bool FLAT>
__device__ inline float coarse_pre(const CoarseLevel& L, const CoarseCell& c, const float* dr, int t, float wa,
                                   float wb) {
  const float s = coarse_nbsum<FLAT>(L, c, dr, t);
  const float u1 = wa * c.d * c.r;
  return (1.f - wb) * u1 + wb * c.d * (c.r + wa * s);
}

// (r - A u) of cell t, its own u given
template <bool FLAT>
__device__ inline float coarse_res(const CoarseLevel& L, const CoarseCell& c, const float* v, int t, float u) {
  return c.r - u / c.d + coarse_nbsum<FLAT>(L, c, v, t);
}

// One weighted-Jacobi sweep of cell t, its own u given
template <bool FLAT>
__device__ inline float coarse_sweep(const CoarseLevel& L, const CoarseCell& c, const float* v, int t, float u,
                                     float omega) {
  return (1.f - omega) * u + omega * c.d * (c.r + coarse_nbsum<FLAT>(L, c, v, t));
}

// Cell t of level C: the sum of its up to eight children's residuals (level
// L), every one read (for an absent one some number nearby) and weighted 0 or
// 1, in the order x, then y, then z.
template <bool FLAT>
__device__ inline float coarse_sum8(const CoarseLevel& L, const CoarseLevel& C, const float* res, int t) {
  int X, Y, Z;
  cell_xyz(C, t, X, Y, Z);
  const float* f = res + 2 * (X + __mul24(L.nx, Y) + __mul24(L.plane, Z));
  const bool x1 = 2 * X + 1 < L.nx, y1 = 2 * Y + 1 < L.ny, z1 = 2 * Z + 1 < L.nz;
  float s = f[0];
  s += x1 ? f[1] : 0.f;
  s += y1 ? f[L.nx] : 0.f;
  s += (x1 & y1) ? f[L.nx + 1] : 0.f;
  if (!FLAT) {
    const float* h = f + L.plane;
    s += z1 ? h[0] : 0.f;
    s += (x1 & z1) ? h[1] : 0.f;
    s += (y1 & z1) ? h[L.nx] : 0.f;
    s += (x1 & y1 & z1) ? h[L.nx + 1] : 0.f;
  }
  return s;
}

// Where cell (x, y, z) of level L takes its correction from in level C: the
// cell with the larger weight and the distances to the other one of each axis (0:
// none, weight 0 instead of 1/4).
struct CoarseParent {
  int at, dx, dy, dz;
};

// lin_axis's coarse cells of fine cell i, without branches: the nearer one and the distance to the other
__device__ inline void coarse_axis(int i, int nf, int nc, int& I, int& d) {
  I = i >> 1;
  d = (i & 1) ? 1 : -1;
  const int J = I + d;
  const bool none = (J < 0) | (J >= nc) | (((nf & 1) != 0) & ((I == nc - 1) | (J == nc - 1)));
  d = none ? 0 : d;
}

template <bool FLAT>
__device__ inline CoarseParent coarse_parent(const CoarseLevel& L, const CoarseLevel& C, int x, int y, int z) {
  int Ix, Iy, Iz = 0, dx, dy, dz = 0;
  coarse_axis(x, L.nx, C.nx, Ix, dx);
  coarse_axis(y, L.ny, C.ny, Iy, dy);
  if (!FLAT) coarse_axis(z, L.nz, C.nz, Iz, dz);
  return {Ix + __mul24(Iy, C.nx) + __mul24(Iz, C.plane), dx, __mul24(dy, C.nx), __mul24(dz, C.plane)};
}

// u3 = u2 + P e of a cell (e: level C's correction): x first along each
// coarse row, then y, then z (the global levels' order).
template <bool FLAT>
__device__ inline float coarse_prolong(const CoarseParent& P, const float* e, float u) {
  const float wx = P.dx ? 0.25f : 0.f, wy = P.dy ? 0.25f : 0.f, wz = P.dz ? 0.25f : 0.f;
  const float* e0 = e + P.at;
  const float r00 = (1.f - wx) * e0[0] + wx * e0[P.dx];
  const float r01 = (1.f - wx) * e0[P.dy] + wx * e0[P.dy + P.dx];
  const float p0 = (1.f - wy) * r00 + wy * r01;
  if (FLAT) return u + p0;
  const float* e1 = e0 + P.dz;
  const float r10 = (1.f - wx) * e1[0] + wx * e1[P.dx];
  const float r11 = (1.f - wx) * e1[P.dy] + wx * e1[P.dy + P.dx];
  const float p1 = (1.f - wy) * r10 + wy * r11;
  return u + ((1.f - wz) * p0 + wz * p1);
}

// Between two phases: of the workgroup, or of one wavefront (whose LDS
// accesses are made in their order; only the compiler has to keep it).
template <bool WAVE>
__device__ inline void coarse_sync() {
  if (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Once per solve, one workgroup per system: coarse reaction terms of the
// one-workgroup levels (summed from level kc, in LDS), then each level's
// couplings and D^-1 into the system's precomputed block.  Each face's coupling
// (a division) is formed once and shared through LDS, none of a level kc whose
// cells are alike (k_mg_coarse does not read them); a level's couplings and the
// next one's reaction terms are formed side by side, every D^-1 at the end
// (50 x 50 cells 13.4 -> 9.9 us, 16^3 13.0 -> 8.1).
__global__ void __launch_bounds__(kCoarseThreads) k_mg_coarse_prep(const MgCoarseRep* coarse,
                                                                   const float* const* lev_c,
                                                                   float* __restrict__ pre) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int rep = blockIdx.x;
  const MgCoarseRep& cr = coarse[rep];
  const int J = cr.nlev, alike = cr.alike;
  const int n0 = cr.dims[0] * cr.dims[1] * cr.dims[2], all = n0 + cr.rest;
  // LDS: the couplings [gz | gy | gx] of level kc, then of each other one; the
  // reaction terms in the same order of levels
  float* sc = lds + 3 * all;
  {
    const float* gc = lev_c[cr.kc] + cr.off_kc;
    for (int t = threadIdx.x; t < n0; t += kCoarseThreads) sc[t] = gc[t];
  }
  __syncthreads();
  for (int j = 0, at = 0; j < J; ++j) {   // at: cells of the levels before, kc's included
    const CoarseLevel L = coarse_level(cr, j, 0);
    if (j > 0 || !alike) {
      Geo<false> G;
      G.nx = L.nx;
      G.ny = L.ny;
      G.nz = L.nz;
      G.k = cr.kc + j;
      G.n0x = cr.n0[0];
      G.n0y = cr.n0[1];
      G.n0z = cr.n0[2];
      G.a = cr.a;
      float *lz = lds + 3 * at, *ly = lz + L.n, *lx = ly + L.n;
      float* g = pre + cr.pre_off + 4 * at;
      // from the last thread down: the first ones form the next level's terms
      for (int t = kCoarseThreads - 1 - (int)threadIdx.x; t < L.n; t += kCoarseThreads) {
        int x, y, z;
        cell_xyz(L, t, x, y, z);
        g[t] = lz[t] = z + 1 < L.nz ? G.gz(x, y, z) : 0.f;
        g[L.n + t] = ly[t] = y + 1 < L.ny ? G.gy(x, y, z) : 0.f;
        g[2 * L.n + t] = lx[t] = x + 1 < L.nx ? G.gx(x, y, z) : 0.f;
      }
    }
    if (j + 1 < J) {
      const CoarseLevel C = coarse_level(cr, j + 1, 0);
      for (int t = threadIdx.x; t < C.n; t += kCoarseThreads)
        sc[at + L.n + t] = coarse_sum8<false>(L, C, sc + at, t);
    }
    __syncthreads();
    at += L.n;
  }
  // D^-1: c and the couplings in the order of Geo::gsum (a missing face adds 0)
  for (int j = 0, at = 0; j < J; ++j) {
    const CoarseLevel L = coarse_level(cr, j, 0);
    const float *lz = lds + 3 * at, *ly = lz + L.n, *lx = ly + L.n;
    float* d = pre + cr.pre_off + 4 * at + 3 * L.n;
    for (int t = threadIdx.x; t < L.n; t += kCoarseThreads) {
      float s;
      if (j == 0 && alike) {
        int x, y, z;
        cell_xyz(L, t, x, y, z);
        s = x > 0 ? cr.g[0] : 0.f;
        s += x + 1 < L.nx ? cr.g[0] : 0.f;
        s += y > 0 ? cr.g[1] : 0.f;
        s += y + 1 < L.ny ? cr.g[1] : 0.f;
        s += z > 0 ? cr.g[2] : 0.f;
        s += z + 1 < L.nz ? cr.g[2] : 0.f;
      } else {
        s = t >= 1 ? lx[t - 1] : 0.f;
        s += lx[t];
        s += t >= L.nx ? ly[t - L.nx] : 0.f;
        s += ly[t];
        s += t >= L.plane ? lz[t - L.plane] : 0.f;
        s += lz[t];
      }
      d[t] = 1.f / (sc[at + t] + s);
    }
    at += L.n;
  }
}

// LDS of a coarse solve: the blocks [gz | gy | gx | D^-1] of the levels after
// kc (`rest` cells); level kc's [ub] and [ua], each between two guards of
// zeros; [ua | ub | r] of the others, zeros at first.
struct CoarseLds {
  float *blocks, *levels;
  __device__ inline float* blk(const CoarseLevel& L) const { return blocks + 4 * L.before; }
  __device__ inline float* ua(const CoarseLevel& L) const { return levels + 3 * L.before; }
};

// The levels from L (its index j) down while one has more than `stop` cells,
// each with at most K cells a thread; on entry level L's residual (r) and
// D^-1 r (ub) are in LDS, on return those of the level that L has become.
template <bool FLAT, bool WAVE, int K>
__device__ inline void coarse_down(const MgCoarseRep& cr, const CoarseLds& M, CoarseLevel& L, int& j, int stop,
                                   float wa, float wb) {
  constexpr int T = WAVE ? 64 : kCoarseThreads;
  while (L.n > stop) {
    const CoarseLevel C = coarse_level(cr, j + 1, L.before + L.n);
    float *ua = M.ua(L), *ub = ua + L.n, *r = ub + L.n;
    CoarseCell c[K];
    float u[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = (int)threadIdx.x + k * T;
      if (t >= L.n) break;
      coarse_cell<FLAT>(L, M.blk(L), t, c[k]);
      c[k].r = r[t];
      u[k] = coarse_pre<FLAT>(L, c[k], ub, t, wa, wb);
      ua[t] = u[k];
    }
    coarse_sync<WAVE>();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = (int)threadIdx.x + k * T;
      if (t >= L.n) break;
      ub[t] = coarse_res<FLAT>(L, c[k], ua, t, u[k]);
    }
    coarse_sync<WAVE>();
    for (int t = threadIdx.x; t < C.n; t += T) {
      const float s = coarse_sum8<FLAT>(L, C, ub, t);
      M.ua(C)[2 * C.n + t] = s;
      M.ua(C)[C.n + t] = M.blk(C)[3 * C.n + t] * s;
    }
    coarse_sync<WAVE>();
    L = C;
    ++j;
  }
}

// From level j's corrected u (C's ua) up to level `to`'s.
template <bool FLAT, bool WAVE, int K>
__device__ inline void coarse_up(const MgCoarseRep& cr, const CoarseLds& M, CoarseLevel& C, int& j, int to,
                                 float wa, float wb) {
  constexpr int T = WAVE ? 64 : kCoarseThreads;
  while (j > to) {
    --j;
    CoarseLevel L = coarse_level(cr, j, 0);
    L.before = C.before - L.n;
    float *ua = M.ua(L), *ub = ua + L.n, *r = ub + L.n;
    CoarseCell c[K];
    float u[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = (int)threadIdx.x + k * T;
      if (t >= L.n) break;
      coarse_cell<FLAT>(L, M.blk(L), t, c[k]);
      c[k].r = r[t];
      int x, y, z;
      cell_xyz(L, t, x, y, z);
      u[k] = coarse_prolong<FLAT>(coarse_parent<FLAT>(L, C, x, y, z), M.ua(C), ua[t]);
      ua[t] = u[k];
    }
    coarse_sync<WAVE>();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = (int)threadIdx.x + k * T;
      if (t >= L.n) break;
      u[k] = coarse_sweep<FLAT>(L, c[k], ua, t, u[k], wb);
      ub[t] = u[k];
    }
    coarse_sync<WAVE>();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = (int)threadIdx.x + k * T;
      if (t >= L.n) break;
      ua[t] = coarse_sweep<FLAT>(L, c[k], ub, t, u[k], wa);
    }
    coarse_sync<WAVE>();
    C = L;
  }
}

// The V-cycle of levels kc.. of one system in LDS (one workgroup per system),
// the same cycle as the multi-workgroup levels: two sweeps, restriction by
// aggregate sums, ..., the one-cell level solved exactly (no faces: u = D^-1 r),
// cell-centred linear prolongation, two sweeps; the correction of level kc is
// written to that level's global u.
//
// A serial chain of phases on one CU: its time is LDS accesses, latencies and
// barriers, not bandwidth.  So level kc's cells (M a thread) keep D^-1, r, u and
// their couplings in registers from the first phase to the last and share
// only what neighbours read; every cell's residual is formed once, by its own
// thread, and then summed; neighbours are read without coordinates or
// bounds, between zeros; and levels of at most 64 cells are the first
// wavefront's alone, without barriers.  Measured, the mean of a solve's calls:
// 50 x 50 cells 10.0 us and 16^3 cells 10.9 us, against 22 and 19 us where every
// phase took each cell's coordinates, couplings and D^-1 from LDS again.
template <int M, bool FLAT>
__global__ void __launch_bounds__(kCoarseThreads) k_mg_coarse(const MgCoarseRep* __restrict__ coarse,
                                                              float wa, float wb,
                                                              const float* __restrict__ pre,
                                                              const SolveScal* __restrict__ ss) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int rep = blockIdx.x;
  const MgCoarseRep cr = coarse[rep];
  const int done = ss[rep].done;
  asm volatile("" ::"s"(cr.r_kc), "s"(cr.pre_off), "s"(cr.rest));   // with `done`, not after it
  if (done) return;
  const int J = cr.nlev, tid = (int)threadIdx.x;
  const CoarseLevel L0 = coarse_level(cr, 0, 0);
  const float* blk = pre + cr.pre_off;
  const float* gr = cr.r_kc;
  float* gu = cr.u_kc;
  if (J == 1) {   // level kc is the one-cell level itself
    if (tid == 0) gu[0] = blk[3] * gr[0];
    return;
  }
  CoarseLevel L = coarse_level(cr, 1, 0);
  const int rest = cr.rest, guard = FLAT ? L0.nx : L0.plane;
  float *ub = lds + 4 * rest + guard, *ua = ub + L0.n + guard;
  const CoarseLds S{lds, ua + L0.n + guard};
  CoarseCell c[M];
  CoarseParent P[M];
  float u[M];
  // Slots beyond the level's cells repeat its last one, stores included.  The
  // thread's number is hidden from the compiler in each phase, which otherwise
  // keeps every index of every cell in registers from the first to the last.
#define FOR_MY_CELLS(BODY)                                    \
  {                                                           \
    int t0 = tid;                                             \
    asm volatile("" : "+v"(t0));                              \
    _Pragma("unroll") for (int m = 0; m < M; ++m) {           \
      const int t = min(t0 + m * kCoarseThreads, L0.n - 1);   \
      BODY;                                                   \
    }                                                         \
  }
  FOR_MY_CELLS(c[m].r = gr[t])
  if (cr.alike) {
    FOR_MY_CELLS(c[m].d = blk[3 * L0.n + t])
  } else {
    FOR_MY_CELLS(coarse_cell<FLAT>(L0, blk, t, c[m]))
  }
  {
    const float4* src = reinterpret_cast<const float4*>(blk + 4 * L0.n);
    float4* dst = reinterpret_cast<float4*>(lds);
    for (int i = tid; i < rest; i += kCoarseThreads) dst[i] = src[i];
  }
  for (int i = tid; i < guard; i += kCoarseThreads) ub[i - guard] = ub[L0.n + i] = ua[L0.n + i] = 0.f;
  for (int i = tid; i < 3 * rest; i += kCoarseThreads) S.levels[i] = 0.f;
  // (the loads under way) what else a cell needs from its coordinates
  FOR_MY_CELLS({
    int x; int y; int z;
    cell_xyz(L0, t, x, y, z);
    if (cr.alike) coarse_alike<FLAT>(L0, cr.g, x, y, z, c[m]);
    P[m] = coarse_parent<FLAT>(L0, L, x, y, z);
    asm volatile("" : "+v"(P[m].at), "+v"(P[m].dx), "+v"(P[m].dy), "+v"(P[m].dz));
  })
  FOR_MY_CELLS(ub[t] = c[m].d * c[m].r)
  __syncthreads();
  FOR_MY_CELLS(u[m] = coarse_pre<FLAT>(L0, c[m], ub, t, wa, wb))
  FOR_MY_CELLS(ua[t] = u[m])
  __syncthreads();
  float v[M];
  FOR_MY_CELLS(v[m] = coarse_res<FLAT>(L0, c[m], ua, t, u[m]))
  FOR_MY_CELLS(ub[t] = v[m])
  __syncthreads();
  for (int t = tid; t < L.n; t += kCoarseThreads) {
    const float s = coarse_sum8<FLAT>(L0, L, ub, t);
    S.ua(L)[2 * L.n + t] = s;
    S.ua(L)[L.n + t] = S.blk(L)[3 * L.n + t] * s;
  }
  __syncthreads();
  int j = 1;
  const bool two = L.n > kCoarseThreads;   // at most twice as many: more do not fit LDS
  if (two) coarse_down<FLAT, false, 2>(cr, S, L, j, kCoarseThreads, wa, wb);
  const int j2 = j;
  coarse_down<FLAT, false, 1>(cr, S, L, j, 64, wa, wb);
  const int jw = j;
  if (tid < 64) {
    CoarseLevel W = L;
    coarse_down<FLAT, true, 1>(cr, S, W, j, 1, wa, wb);
    if (tid == 0) S.ua(W)[0] = S.ua(W)[1];   // u = D^-1 r
    coarse_sync<true>();
    coarse_up<FLAT, true, 1>(cr, S, W, j, jw, wa, wb);
  }
  __syncthreads();
  j = jw;
  coarse_up<FLAT, false, 1>(cr, S, L, j, j2, wa, wb);
  if (two) coarse_up<FLAT, false, 2>(cr, S, L, j, 1, wa, wb);
  FOR_MY_CELLS(ua[t] = u[m] = coarse_prolong<FLAT>(P[m], S.ua(L), u[m]))
  __syncthreads();
  FOR_MY_CELLS(u[m] = coarse_sweep<FLAT>(L0, c[m], ua, t, u[m], wb))
  FOR_MY_CELLS(ub[t] = u[m])
  __syncthreads();
  FOR_MY_CELLS(u[m] = coarse_sweep<FLAT>(L0, c[m], ub, t, u[m], wa))
  FOR_MY_CELLS(gu[t] = u[m])
#undef FOR_MY_CELLS
}

// ---- launchers -------------------------------------------------------------

hipError_t mg_set_fused_lds() {
  const void* pre3[] = {(const void*)k_mg_prefused<3, true, false>, (const void*)k_mg_prefused<3, true, true>};
  const void* pre2[] = {(const void*)k_mg_prefused<2, true, false>, (const void*)k_mg_prefused<2, false, false>,
                        (const void*)k_mg_prefused<2, true, true>};
  const void* post3[] = {(const void*)k_mg_postfused<3, true, true, false, double>,
                         (const void*)k_mg_postfused<3, true, true, true, float>};
  const void* post2[] = {(const void*)k_mg_postfused<2, true, false, false, double>,
                         (const void*)k_mg_postfused<2, false, false, false, double>,
                         (const void*)k_mg_postfused<2, true, false, true, float>};
  hipError_t e = hipSuccess;
  auto set = [&](const void* f, int bytes) {
    if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
  for (const void* f : pre3) set(f, f3_lds_pre<3>(kF3Block));
  for (const void* f : pre2) set(f, f3_lds_pre<2>(kF3Block));
  for (const void* f : post3) set(f, f3_lds_post<3>(kF3Block));
  for (const void* f : post2) set(f, f3_lds_post<2>(kF3Block));
  return e;
}

// The coarse solve for level kc of up to `cells` cells: the fewest cells a
// thread that take them (the slots of a thread are worked on together, those
// beyond a system's cells for nothing).  Level kc is chosen with no more than the last
// one's; today's bound is lower, 5814 cells by a level's 28 bytes a cell in 160 KiB.
// flat: every system has one plane.
typedef void (*CoarseKernel)(const MgCoarseRep*, float, float, const float*, const SolveScal*);
template <bool FLAT>
static CoarseKernel coarse_kernel_of(int cells) {
  if (cells <= kCoarseThreads) return k_mg_coarse<1, FLAT>;
  if (cells <= 2 * kCoarseThreads) return k_mg_coarse<2, FLAT>;
  if (cells <= 3 * kCoarseThreads) return k_mg_coarse<3, FLAT>;
  if (cells <= 4 * kCoarseThreads) return k_mg_coarse<4, FLAT>;
  return k_mg_coarse<kCoarseMaxCellsPerThread, FLAT>;
}
static CoarseKernel coarse_kernel(int cells, int flat) {
  return flat ? coarse_kernel_of<true>(cells) : coarse_kernel_of<false>(cells);
}

hipError_t mg_set_coarse_lds(int cells, int flat, int bytes) {
  hipError_t e =
      hipFuncSetAttribute((const void*)coarse_kernel(cells, flat), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_mg_coarse_prep, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <typename T>
void launch_mg_prepare(hipStream_t s, const Work& w, const MgBufs& mg, const T* c) {
  // level 0's D^-1 comes with level 1's c (k_mg_coarsen<true>); a level 1 with
  // no restriction tiles would leave it to k_mg_prep0
  if (mg.lev[0].ntiles && !mg.lev[1].nrtiles)
    hca_launch(k_mg_prep0<T>, dim3(grid_tiles(mg.lev[0].ntiles, w.max_blocks)), dim3(kBlock), 0, s, mg.lev[0], c);
  for (int k = 0; k < mg.nlev_glob; ++k) {
    const MgLevel& Lc = mg.lev[k + 1];
    if (!Lc.nrtiles) continue;
    if (k == 0)
      hca_launch(k_mg_coarsen<true, T>, dim3(grid_tiles(Lc.nrtiles, w.max_blocks)), dim3(kBlock), 0, s, mg.lev[k], Lc, c);
    else
      hca_launch(k_mg_coarsen<false, T>, dim3(grid_tiles(Lc.nrtiles, w.max_blocks)), dim3(kBlock), 0, s, mg.lev[k], Lc, c);
  }
  hca_launch(k_mg_coarse_prep, dim3(w.nreps), dim3(kCoarseThreads), mg.coarse_lds_bytes, s, mg.coarse,
             (const float* const*)mg.lev_c, mg.coarse_pre);
}

template <typename T>
void launch_mg_vcycle(hipStream_t s, const Work& w, const MgBufs& mg, const SolverBufsT<T>& sb,
                      MgHook hook, void* hctx) {
  // levels >= 1: pre-sweeps with weights (wa, wb), post-sweeps with (wb, wa);
  // level 0: three sweeps (w0[0], w0[1], w0[2]) before, reversed after
  const float wa = mg.w_a, wb = mg.w_b;
  const float* w0 = mg.w0;
  const SolveScal* ss = sb.ss;
  // level 0's residual for the fused passes: the scaled FP32 copy, or (stored
  // in FP32 anyway) r itself, scaled as it is read
  constexpr bool kP32 = sizeof(T) == 4;
  const float* r0 = kP32 ? (const float*)sb.r : sb.r32;
  auto H = [&](int seg, int begin) {
    if (hook) hook(hctx, seg, begin);
  };
  // a level's correction: its u, or its ualt where its post-smoothing ran fused
  auto corr = [&](int k) -> const float* {
    return (mg.fused && k < mg.nlev_glob && mg.lev[k].nftiles) ? mg.lev[k].ualt : mg.lev[k].u;
  };
  if (mg.fused) {
    const MgLevel& L = mg.lev[0];
    const MgLevel& C = mg.lev[1];
    H(MG_PRE3_0, 1);
    hca_launch((k_mg_prefused<3, true, kP32>), dim3(L.nftiles), dim3(L.fthreads), f3_lds_pre<3>(L.fthreads), s, L, C,
               F3W{{w0[0], w0[1], w0[2]}}, 1.f, r0, ss);
    H(MG_PRE3_0, 0);
  } else {
    const MgLevel& L = mg.lev[0];
    const MgLevel& C = mg.lev[1];
    H(MG_PRE0, 1);
    hca_launch((k_mg_pre<true, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, w0[0],
               w0[1], (const float*)sb.r32, L.ualt, ss);
    H(MG_PRE0, 0);
    H(MG_SWEEP0, 1);
    hca_launch((k_mg_sweep<true, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, w0[2],
               (const float*)L.ualt, L.u, (const float*)sb.r32, ss);
    H(MG_SWEEP0, 0);
    H(MG_RESTRICT0, 1);
    hca_launch((k_mg_restrict<true, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, C,
                       (const float*)sb.r32, ss);
    H(MG_RESTRICT0, 0);
  }
  if (mg.nlev_glob > 1) {
    H(MG_DOWN, 1);
    for (int k = 1; k < mg.nlev_glob; ++k) {
      const MgLevel& L = mg.lev[k];
      const MgLevel& C = mg.lev[k + 1];
      if (!L.ntiles) continue;
      if (mg.fused && L.nftiles) {
        auto pre = k_mg_prefused<2, true, kP32>;
        if constexpr (!kP32)   // (precision 32 fuses uniform levels alone)
          if (!L.uniform) pre = k_mg_prefused<2, false, kP32>;
        hca_launch(pre, dim3(L.nftiles), dim3(L.fthreads), f3_lds_pre<2>(L.fthreads), s, L, C, F3W{{wa, wb, 0.f}},
                   (float)(1 << k), (const float*)L.r, ss);
        continue;
      }
      hca_launch((k_mg_pre<false, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, wa, wb,
                 (const float*)L.r, L.u, ss);
      hca_launch((k_mg_restrict<false, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, C,
                 (const float*)L.r, ss);
    }
    H(MG_DOWN, 0);
  }
  H(MG_COARSE, 1);
  hca_launch(coarse_kernel(mg.coarse_cells, mg.coarse_flat), dim3(w.nreps), dim3(kCoarseThreads), mg.coarse_lds_bytes, s,
             (const MgCoarseRep*)mg.coarse, wa, wb, (const float*)mg.coarse_pre, ss);
  H(MG_COARSE, 0);
  if (mg.nlev_glob > 1) {
    H(MG_UP, 1);
    for (int k = mg.nlev_glob - 1; k >= 1; --k) {
      const MgLevel& L = mg.lev[k];
      const MgLevel& C = mg.lev[k + 1];
      if (!L.ntiles) continue;
      if (mg.fused && L.nftiles) {
        auto post = k_mg_postfused<2, true, false, kP32, T>;
        if constexpr (!kP32)
          if (!L.uniform) post = k_mg_postfused<2, false, false, kP32, T>;
        hca_launch(post, dim3(L.nftiles), dim3(L.fthreads), f3_lds_post<2>(L.fthreads), s, L, C, corr(k + 1),
                   F3W{{wb, wa, 0.f}}, (float)(1 << k), (const float*)L.r, L.ualt, sb, (double*)nullptr);
        continue;
      }
      hca_launch((k_mg_post1<false, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, C,
                 corr(k + 1), wb, (const float*)L.r, ss);
      hca_launch((k_mg_post2<false, float, T>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, wa,
                 (const float*)L.ualt, (const float*)L.r, sb);
    }
    H(MG_UP, 0);
  }
  if (mg.fused) {
    const MgLevel& L = mg.lev[0];
    const MgLevel& C = mg.lev[1];
    H(MG_POST3_0, 1);
    hca_launch((k_mg_postfused<3, true, true, kP32, T>), dim3(L.nftiles), dim3(L.fthreads),
               f3_lds_post<3>(L.fthreads), s, L, C, corr(1),
               F3W{{w0[2], w0[1], w0[0]}}, 1.f, r0, (float*)nullptr, sb, mg.colsum);
    if (kP32)
      hca_launch(k_mg_rz32, dim3(L.nrztiles), dim3(kRzBlock), 0, s, L, (const double*)mg.colsum, sb.partial, ss);
    H(MG_POST3_0, 0);
    launch_cg_reduce(s, w, sb, RED_RZF, 0.0, 0);
  } else {
    const MgLevel& L = mg.lev[0];
    const MgLevel& C = mg.lev[1];
    H(MG_POST1_0, 1);
    hca_launch((k_mg_post1<true, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, C,
               corr(1), w0[2], (const float*)sb.r32, ss);
    H(MG_POST1_0, 0);
    H(MG_SWEEP0, 1);
    hca_launch((k_mg_sweep<true, float>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, w0[1],
               (const float*)L.ualt, L.u, (const float*)sb.r32, ss);
    H(MG_SWEEP0, 0);
    H(MG_POST2_0, 1);
    hca_launch((k_mg_post2<true, T, T>), dim3(grid_tiles(L.ntiles, w.max_blocks)), dim3(kBlock), 0, s, L, w0[0],
               (const float*)L.u, (const T*)sb.r, sb);
    H(MG_POST2_0, 0);
    launch_cg_reduce(s, w, sb, RED_RZ, 0.0, 0);
  }
}

template void launch_mg_prepare<double>(hipStream_t, const Work&, const MgBufs&, const double*);
template void launch_mg_prepare<float>(hipStream_t, const Work&, const MgBufs&, const float*);
template void launch_mg_vcycle<double>(hipStream_t, const Work&, const MgBufs&,
                                       const SolverBufsT<double>&, MgHook, void*);
template void launch_mg_vcycle<float>(hipStream_t, const Work&, const MgBufs&,
                                      const SolverBufsT<float>&, MgHook, void*);

}  // namespace hca
