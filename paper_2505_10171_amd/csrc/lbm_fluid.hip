// lbm_fluid.hip -- lattice kernels of liblbm for gfx950.
//
// Storage: the 19 total populations f of each node, in blocks of 64 nodes (19
// runs of 64 values; see pidx).  The colour is carried by the per-node order
// parameter; the colour populations are rebuilt by the moments pass (see
// rebuild_moments).
// FP32 storage keeps the deviation d_i = f_i - w_i rho0 (so that the small
// velocity survives FP32 rounding); FP16 storage keeps
// h_i = (f_i - w_i R) / (w_i rho0) with R the node's density of the previous
// state.  All arithmetic is FP32; momentum exchange sums are FP64.
//
// A step of the fluid runs k_interface (interface normal, curvature and CSF
// coefficient from phi, in one z-march), k_fused (collision, force, streaming and
// bounce-back of f, one thread per node, reading and writing every population
// exactly once), k_links (moving-wall terms and momentum exchange at particle
// links, and the particles' capillary forces) and k_moments (density and order
// parameter of the post-stream state).
#include <algorithm>

#include "launch_rules.h"
#include "lbm_device.h"

namespace lbm {

// ------------------------------------------------------------ wetting rotation
// Geometric wetting (n_pm equation): at a fluid node with a solid neighbour the
// colour gradient is rotated to make the angle theta (through fluid a) with the
// solid's outward normal n_s, keeping |G|: G <- |G| (-cos(theta) n_s + sin(theta) t^),
// t = n* - (n*.n_s) n_s.  The solid is the lowest-index neighbouring particle,
// else the wall.  Applied inside the diffuse interface (|G| > EPS_G); left
// unchanged if the tangential part |G - (G.n_s) n_s| <= EPS_GT (axis undefined).
// Between those thresholds and twice their value the rotated vector is blended
// in with weight w = min(1, |t|/EPS_GT - 1) min(1, |G|/EPS_G - 1), so that G is
// continuous in phi (no last-bit difference can switch the rotation on or off).
// GEO: the geometries compiled in (Geometry).
template <int GEO>
__device__ __forceinline__ void wetting_rotate(const SimDev& s, int gx, int gy, int gz, int minp,
                                               bool wall_nb, float& Gx, float& Gy, float& Gz) {
  float g = sqrtf(Gx * Gx + Gy * Gy + Gz * Gz);
  if (!(g > EPS_G)) return;
  float nsx, nsy, nsz, nc, ns;
  if (minp >= 0) {
    // in FP64, rounded once to FP32 (the wetting direction next to a particle
    // moves the velocity there at the 1e-5 level)
    const DevParticle& P = s.P[minp];
    const double dx = wrapd((double)gx - P.x[0], (double)s.nx);
    const double dy = wrapd((double)gy - P.x[1], (double)s.ny);
    const double dz = wrapd((double)gz - P.x[2], (double)s.nz);
    const double idn = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
    nsx = (float)(dx * idn);
    nsy = (float)(dy * idn);
    nsz = (float)(dz * idn);
    nc = P.neg_cos_t;
    ns = P.sin_t;
  } else if (wall_nb && (GEO == GEO_PLAIN || s.has_wall == 1)) {
    nsx = 0.f;
    nsy = 0.f;
    nsz = (gz == 1) ? 1.f : -1.f;
    nc = s.wall_neg_cos;
    ns = s.wall_sin;
  } else if (GEO == GEO_ANY && wall_nb && s.has_wall == 3) {
    // textured wall: the normal of the nearest point of the solid surface (the
    // plane's top face z = 1/2, or its underside z = nz - 1/2 through the
    // periodic z direction; the boxes grown by half a node), from it to the
    // node; on ties the plane, then the lowest box index
    // (in half nodes all coordinates are whole numbers: distances are compared
    // squared and exact, in integers; one square root, for the winner)
    const int hx = 2 * gx, hy = 2 * gy, hz = 2 * gz;
    const int dt = hz - 1, du = (2 * s.nz - 1) - hz;
    const int dp = min(dt, du);
    long long best2 = (long long)dp * dp;
    int b0 = 0, b1 = 0, b2 = 0;
    const int n_boxes = s.n_boxes;
    for (int b = 0; b < n_boxes; ++b) {
      const int* B = s.boxes[b];
      // beyond the upper face, before the lower one, or 0 between them
      const int d0 = max(hx - (2 * B[3] + 1), 0) + min(hx - (2 * B[0] - 1), 0);
      const int d1 = max(hy - (2 * B[4] + 1), 0) + min(hy - (2 * B[1] - 1), 0);
      const int d2 = max(hz - (2 * B[5] + 1), 0) + min(hz - (2 * B[2] - 1), 0);
      const long long dd = (long long)d0 * d0 + (long long)d1 * d1 + (long long)d2 * d2;
      if (dd > 0 && dd < best2) {
        best2 = dd;
        b0 = d0;
        b1 = d1;
        b2 = d2;
      }
    }
    double bx = 0.0, by = 0.0, bz = dt <= du ? 1.0 : -1.0;
    if ((b0 | b1 | b2) != 0) {
      const double idn = 1.0 / sqrt(0.25 * (double)best2);
      bx = 0.5 * (double)b0 * idn;
      by = 0.5 * (double)b1 * idn;
      bz = 0.5 * (double)b2 * idn;
    }
    nsx = (float)bx;
    nsy = (float)by;
    nsz = (float)bz;
    nc = s.wall_neg_cos;
    ns = s.wall_sin;
  } else if (wall_nb) {
    // tube: the wall's outward normal points from the node to the axis
    const double dy = (double)gy - s.tube_yc, dz = (double)gz - s.tube_zc;
    const double r = sqrt(dy * dy + dz * dz);
    if (!(r > 0.0)) return;
    nsx = 0.f;
    nsy = (float)(-dy / r);
    nsz = (float)(-dz / r);
    nc = s.wall_neg_cos;
    ns = s.wall_sin;
  } else {
    return;
  }
  float a = Gx * nsx + Gy * nsy + Gz * nsz;
  float tx = Gx - a * nsx, ty = Gy - a * nsy, tz = Gz - a * nsz;
  float tn = sqrtf(tx * tx + ty * ty + tz * tz);
  if (!(tn > EPS_GT)) return;
  float it = 1.0f / tn;
  const float rx = g * (nc * nsx + ns * tx * it);
  const float ry = g * (nc * nsy + ns * ty * it);
  const float rz = g * (nc * nsz + ns * tz * it);
  const float w = fminf(1.0f, tn / EPS_GT - 1.0f) * fminf(1.0f, g / EPS_G - 1.0f);
  if (w >= 1.0f) {
    Gx = rx;
    Gy = ry;
    Gz = rz;
  } else {
    Gx += w * (rx - Gx);
    Gy += w * (ry - Gy);
    Gz += w * (rz - Gz);
  }
}

// One direction of each opposite pair: +x, +y, +z, (1,1,0), (1,-1,0), (1,0,1),
// (1,0,-1), (0,1,1), (0,1,-1).
__host__ __device__ constexpr int pair_dir(int k) {
  constexpr int t[9] = {1, 3, 5, 7, 8, 11, 12, 15, 16};
  return t[k];
}

// index of halo record j of thread t
__device__ __forceinline__ int k_of(int t, int j) { return t + 256 * j; }

// XCD-aware block order: consecutive dispatches go round-robin over the 8 XCDs;
// give each XCD a contiguous range of blocks so that data shared by neighbouring
// blocks (halo reads, pushed populations) meets in the same L2.
__device__ __forceinline__ int xcd_tile(int lin, int nblk) {
  if ((nblk & 7) == 0) {
    const int per = nblk >> 3;
    return (lin & 7) * per + (lin >> 3);
  }
  return lin;
}

// ---------------------------------------------------------------- refill
// Refilling (refilling eqs.): f_a, f_b of a fresh node = equilibria of the mean
// neighbour densities (fluid, not fresh, D3Q19 neighbours; rho0/2 each if none)
// at the surface velocity of the particle that uncovered it.  Stored are the
// total f and the node's moments (rho, phi) in rp[rd ^ 1].  The neighbour
// densities are those of the post-stream state: in a step (REFILL_STEP) rebuilt
// from the state that collided, as the moments pass does; between steps
// (REFILL_BOUNDARY) the current moments rp[rd ^ 1].  In a step the refill's blocks
// run in the launch of the moments pass: neither reads what the other writes (the
// moments pass leaves fresh nodes alone), and the refill's dependent loads hide
// behind it (500 spheres 23 us, 20 spheres 9 to 12, one 2 to 4).
enum { REFILL_STEP = 0, REFILL_BOUNDARY = 1 };
constexpr int REFILL_PER = 14;  // fresh nodes per block: a thread per neighbour direction
struct RefillLds {
  float a[REFILL_PER][18], b[REFILL_PER][18];
  int c[REFILL_PER][18];
};
// block `block` of the `blocks` that refill simulation s
template <int STORE, int MODE>
__device__ __forceinline__ void refill_block(const Batch& bt, const SimDev& s, int block,
                                             int blocks, RefillLds& lds) {
  using IO = Codec<STORE>;
  using T = typename IO::T;
  if (s.np == 0) return;
  T* b = (T*)s.pops[bt.cur];
  const GLB float* RO = gp((const float*)s.rp[bt.rd]);
  float* RN = s.rp[bt.rd ^ 1];
  constexpr int PER = REFILL_PER;
  auto &sh_a = lds.a, &sh_b = lds.b;
  auto& sh_c = lds.c;
  const uint32_t cnt = min(s.counters[bt.fc], s.fresh_cap);
  const int N = (int)s.N;
  const int slot = threadIdx.x / 18, dir = threadIdx.x % 18 + 1;
  for (uint32_t base = (uint32_t)block * PER; base < cnt; base += (uint32_t)blocks * PER) {
    const uint32_t k = base + slot;
    if (slot < PER) {
      float ra = 0.f, rb = 0.f;
      int c = 0;
      if (k < cnt) {
        const int n = (int)s.fresh[k];
        const int x = n % s.nx, y = (n / s.nx) % s.ny, z = n / (s.nx * s.ny);
        const int mx = wrapi(x + cx(dir), s.nx), my = wrapi(y + cy(dir), s.ny),
                  mz = wrapi(z + cz(dir), s.nz);
        const int m = mx + s.nx * (my + s.ny * mz);
        // a fluid node that is not fresh: in a step, one that was fluid in the
        // state that collided (the moments pass beside it clears the marks)
        const uint16_t mk = s.mask[m];
        if (MODE == REFILL_STEP ? (mk & ~FRESH_BIT) == 0 && !(RO[N + m] > PHI_SOLID_TEST)
                                : mk == 0) {
          float rho, sg;
          if (MODE == REFILL_STEP) {
            const Nbr nbm(mx, my, mz, s.nx, s.ny, s.nz);
            rebuild_moments<STORE>(gp((const T*)b), RO, gp((const float*)s.nrm), N, m, nbm,
                                   s.rho0, 0.5f * s.beta, STORE ? RO[m] : 0.f, rho, sg);
          } else {
            // FP32 keeps no density where phi is +-1
            const float ph = RN[N + m];
            rho = STORE == 0 && phi_pure(ph)
                      ? node_density<STORE>(gp((const T*)b), N, m, s.rho0, 0.f)
                      : RN[m];
            sg = rho * ph;
          }
          ra = 0.5f * (rho + sg);
          rb = 0.5f * (rho - sg);
          c = 1;
        }
      }
      sh_a[slot][dir - 1] = ra;
      sh_b[slot][dir - 1] = rb;
      sh_c[slot][dir - 1] = c;
    }
    __syncthreads();
    if ((int)threadIdx.x < PER && base + threadIdx.x < cnt) {
      const uint32_t kk = base + threadIdx.x;
      float sa = 0.f, sb = 0.f;
      int c = 0;
      for (int i = 0; i < 18; ++i) {
        sa += sh_a[threadIdx.x][i];
        sb += sh_b[threadIdx.x][i];
        c += sh_c[threadIdx.x][i];
      }
      const int n = (int)s.fresh[kk];
      const int p = (int)s.fresh_own[kk];
      const int x = n % s.nx, y = (n / s.nx) % s.ny, z = n / (s.nx * s.ny);
      const float ra = c ? sa / c : 0.5f * s.rho0;
      const float rb = c ? sb / c : 0.5f * s.rho0;
      const DevParticle& P = s.P[p];
      const double rx = wrapd((double)x - P.x[0], (double)s.nx);
      const double ry = wrapd((double)y - P.x[1], (double)s.ny);
      const double rz = wrapd((double)z - P.x[2], (double)s.nz);
      const float ux = (float)(P.v[0] + P.w[1] * rz - P.w[2] * ry);
      const float uy = (float)(P.v[1] + P.w[2] * rx - P.w[0] * rz);
      const float uz = (float)(P.v[2] + P.w[0] * ry - P.w[1] * rx);
      const float uu = ux * ux + uy * uy + uz * uz;
      const float rho = ra + rb;
      // FP16: encoded with the reference the decoders of this state use
      const float Rn = STORE ? RO[n] : 0.f;
      for (int q = 0; q < Q; ++q) {
        const float cu = cx(q) * ux + cy(q) * uy + cz(q) * uz;
        const float poly = 3.0f * cu + 4.5f * cu * cu - 1.5f * uu;
        const float dq = wq(q) * ((rho - s.rho0) + rho * poly);
        IO::st(b + pidx(q, N, n), wq(q) * s.rho0, 1.0f / (wq(q) * s.rho0), wq(q) * Rn, dq);
      }
      // f^a - f^b = (ra - rb) / rho f: the order parameter of the node
      RN[n] = rho;
      RN[N + n] = (ra - rb) / rho;
    }
    __syncthreads();
  }
}

template <int STORE>
__global__ __launch_bounds__(256) void k_refill_boundary(Batch bt) {
  __shared__ RefillLds lds;
  refill_block<STORE, REFILL_BOUNDARY>(bt, bt.tab[blockIdx.y], blockIdx.x, gridDim.x, lds);
}

// ------------------------------------------------------------- moments kernel
// Density and order parameter phi = sum g / rho (order-parameter eq.) of every
// fluid node of the post-stream state into rp[rd ^ 1], the colour populations
// rebuilt from the state that collided (the colour source (phi, r n) of each
// node, formed from its moments and normal).  The refill writes the moments of
// the fresh nodes; this pass clears their FRESH mark.  Solid nodes get (rho0, solid_phi(mask)), so that stencils can tell solids
// from phi alone.
//
// A block takes an x-y tile of the simulation's moments tiling and marches up
// s.mkz planes.  The colour sources of three planes of the tile grown by one
// node sit in an LDS ring; each plane adds the sources of the plane above.
// A pure tile plane (TileKind) takes no sources and, in FP32, no populations:
// its phi stays, and its density is not kept.
constexpr int MOM_HALO = 66 * 6;  // largest tile plane grown by one: (64 + 2)(4 + 2)
// LX: log2 of the tiles' x width (the tile's LDS offsets are then immediates)
struct MomLds {
  v4f ring[3][MOM_HALO];
  uint8_t kinds[258];
};
template <int STORE, int LX>
__device__ __forceinline__ void moments_block(const Batch& bt, const SimDev& s, const int2 sb,
                                              MomLds& lds) {
  using IO = Codec<STORE>;
  using T = typename IO::T;
  auto& ring = lds.ring;
  auto& kinds = lds.kinds;
  const int N = (int)s.N;
  const int nx = s.nx, ny = s.ny, nz = s.nz, P = nx * ny;
  const GLB float* __restrict__ NX = gp((const float*)s.nrm);
  const float hb = 0.5f * s.beta;
  const GLB T* __restrict__ pops = gp((const T*)s.pops[bt.cur]);
  const GLB float* __restrict__ RO = gp((const float*)s.rp[bt.rd]);
  GLB float* __restrict__ RN = gp(s.rp[bt.rd ^ 1]);
  GLB uint16_t* __restrict__ MASK = gp(s.mask);
  constexpr int tlx = LX, tx = 1 << tlx, ty = 256 >> tlx, HX = tx + 2, HY = ty + 2;
  const int bx = sb.y % s.mtiles_x, r = sb.y / s.mtiles_x;
  const int mkz = bt.mkz > 0 ? bt.mkz : s.mkz;
  const int by = r % s.mtiles_y, z0 = (r / s.mtiles_y) * mkz;
  const int kz = min(mkz, nz - z0);
  const int t = (int)threadIdx.x;
  const int lx = t & (tx - 1), ly = t >> tlx;
  const int gx = bx * tx + lx, gy = by * ty + ly;
  const bool in = gx < nx && gy < ny;
  // this thread's halo records of a plane: t and t + 256 (a plane has at
  // most 396); past a partial tile's end they are only kept in bounds
  // (-1: beyond an open x end; its record is all NaN, the mark of a
  // population that entered through the pressure boundary)
  int hoff[2];
  bool hon[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int k = t + 256 * j;
    hon[j] = k < HX * HY;
    const int hy = k / HX, hx = k - hy * HX;
    int x = bx * tx - 1 + hx, y = by * ty - 1 + hy;
    const bool out = s.open_x && (x < 0 || x >= nx);
    x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
    hoff[j] = !hon[j] ? 0 : out ? -1 : min(x, nx - 1) + nx * min(y, ny - 1);
  }
  const float qnan = __int_as_float(0x7fc00000);
  const v4f open_rec = v4f{qnan, qnan, qnan, qnan};
  auto zwrap = [&](int z) { return z < 0 ? z + nz : (z >= nz ? z - nz : z); };
  // the kinds of the block's tile planes (entry zz + 1; mixed ones bound by
  // pure ones below and above)
  {
    const GLB uint8_t* __restrict__ KIND = gp((const uint8_t*)s.kind);
    if (t < 2) kinds[t * (kz + 1)] = KIND_PURE_A;
    if (t < kz) kinds[t + 1] = KIND[((z0 + t) * s.mtiles_y + by) * s.mtiles_x + bx];
  }
  __syncthreads();
  auto kind_of = [&](int zz) { return __builtin_amdgcn_readfirstlane((int)kinds[zz + 1]); };
  int k0 = kind_of(0), k1 = kz > 1 ? kind_of(1) : KIND_PURE_A;
  // planes z0 - 1 and z0 into the ring, if a mixed plane reads them
#pragma unroll
  for (int dz = 0; dz < 2; ++dz) {
    if (k0 != KIND_MIXED && (dz == 0 || k1 != KIND_MIXED)) continue;
    const int zp = zwrap(z0 - 1 + dz);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (hon[j])
        ring[(z0 + 2 + dz) % 3][k_of(t, j)] =
            hoff[j] < 0 ? open_rec : colour_source(RO, NX, N, hoff[j] + P * zp, hb);
  }
  // Each plane takes one round of global loads: the node's populations and
  // the raw moments and normal of the next plane's halo records, all issued
  // before the first wait (indices clamped in bounds instead of branches, which
  // would wait inside them); the records are formed once the loads are in.
  float sr[2][5];
  auto fetch_raw = [&](int z) {
    const int zp = zwrap(z + 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int m = max(hoff[j], 0) + P * zp;
      sr[j][0] = RO[m];
      sr[j][1] = RO[N + m];
      sr[j][2] = NX[m];
      sr[j][3] = NX[N + m];
      sr[j][4] = NX[2 * N + m];
    }
  };
  const int gxc = min(gx, nx - 1), gyc = min(gy, ny - 1);
  const float rho0 = s.rho0;  // kept in a register: the stores below may alias s
  // a pure tile plane: phi of its fluid nodes stays what it is (every source
  // of the colour is the same pure fluid).  FP16 needs the density as the
  // next state's reference; FP32 keeps none there, so that the populations of
  // the pure fluids are not read at all
  auto pure_plane = [&](int z, float phi) {
    if (!in) return;
    const int n = gx + nx * (gy + ny * z);
    const uint16_t m = MASK[n];
    if (m & FRESH_BIT) {
      MASK[n] = (uint16_t)(m & ~FRESH_BIT);
      return;
    }
    if (m != 0) {
      RN[n] = rho0;
      RN[N + n] = solid_phi(m);
      return;
    }
    if (STORE) RN[n] = node_density<STORE>(pops, N, n, rho0, RO[n]);
    RN[N + n] = phi;
  };
  // a plane's results are stored once the next plane's loads are in, so that
  // they are in flight during the sums instead of ahead of the next loads
  int pn = -1;
  uint16_t pm = 0;
  float prabs = 0.f, psg = 0.f;
  auto store_pending = [&]() {
    if (pn < 0) return;
    if (pm & FRESH_BIT) {  // refilled node: moments written by the refill
      MASK[pn] = (uint16_t)(pm & ~FRESH_BIT);
    } else if (pm != 0) {
      RN[pn] = rho0;
      RN[N + pn] = solid_phi(pm);
    } else {
      RN[pn] = prabs;
      RN[N + pn] = psg / prabs;
    }
  };
  for (int zz = 0; zz < kz; ++zz) {
    const int z = z0 + zz;
    const int kind = k0, above = k1;
    k0 = k1;
    k1 = zz + 2 < kz ? kind_of(zz + 2) : KIND_PURE_A;
    if (kind != KIND_MIXED) {
      // its plane above is read by the mixed planes z + 1 and z + 2
      if (above == KIND_MIXED || k1 == KIND_MIXED) {
        fetch_raw(z);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          if (hon[j])
            ring[(z + 1) % 3][k_of(t, j)] =
                hoff[j] < 0 ? open_rec
                            : colour_record(sr[j][0], sr[j][1], sr[j][2], sr[j][3], sr[j][4], hb);
      }
      pure_plane(z, pure_sign(kind));
      continue;
    }
    const int n = gxc + nx * (gyc + ny * z);
    float d[Q];
    const uint16_t m = MASK[n];
    load_pops<STORE>(pops, N, n, rho0, STORE ? RO[n] : 0.f, d);
    fetch_raw(z);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (hon[j])
        ring[(z + 1) % 3][k_of(t, j)] =
            hoff[j] < 0 ? open_rec
                        : colour_record(sr[j][0], sr[j][1], sr[j][2], sr[j][3], sr[j][4], hb);
    store_pending();
    __syncthreads();
    if (in) {
      const int c0 = (lx + 1) + HX * (ly + 1);
      colour_sums(
          d, [&](int i) { return ring[(z + 3 - cz(i)) % 3][c0 - cx(i) - HX * cy(i)]; },
          ring[z % 3][c0], rho0, prabs, psg);
      pn = n;
      pm = m;
    }
    __syncthreads();
  }
  store_pending();
}

// W64: every simulation of the launch has 64-wide tiles; else the tile width
// is the block's simulation's (an ensemble mixes them: one uniform branch per
// block, against offsets computed from a width in a register, see k_interface)
// The first nsim x nref blocks refill (the longest chains start first).
template <int STORE, bool W64>
// four waves per SIMD (128 VGPRs): the refill's loads alone would take 141
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_moments(
    Batch bt, int nref) {
  __shared__ union {
    MomLds mom;
    RefillLds ref;
  } u;
  const int first = bt.nsim * nref;
  if ((int)blockIdx.x < first) {
    const int si = (int)blockIdx.x / nref;
    refill_block<STORE, REFILL_STEP>(bt, bt.tab[si], (int)blockIdx.x - si * nref, nref, u.ref);
    return;
  }
  MomLds& lds = u.mom;
  const int2 sb = batch_block_in(bt, bt.mblk, (int)blockIdx.x - first);
  const SimDev& s = bt.tab[sb.x];
  if (W64 || s.mtile_lx == 6)
    moments_block<STORE, 6>(bt, s, sb, lds);
  else if (s.mtile_lx == 5)
    moments_block<STORE, 5>(bt, s, sb, lds);
  else
    moments_block<STORE, 4>(bt, s, sb, lds);
}

// Between steps, after the mask changed with the populations in place (and
// the refill of fresh nodes): solid nodes get (rho0, solid_phi(mask)), fresh nodes
// lose their mark, fluid nodes keep their moments.
__global__ __launch_bounds__(256) void k_moments_boundary(Batch bt) {
  const int2 sb = batch_block(bt, blockIdx.x);
  const SimDev& s = bt.tab[sb.x];
  int n, gx, gy, gz;
  if (sb.y == 0 && threadIdx.x == 0) s.counters[bt.fc] = 0u;  // fresh list consumed
  if (!tile_node(s, sb.y, n, gx, gy, gz)) return;
  const uint16_t m = s.mask[n];
  if (m & FRESH_BIT) {
    s.mask[n] = (uint16_t)(m & ~FRESH_BIT);
  } else if (m != 0) {
    float* RN = s.rp[bt.rd ^ 1];
    RN[n] = s.rho0;
    RN[s.N + n] = solid_phi(m);
  }
}

// ------------------------------------------------------------ init kernels
__global__ void k_init_mask(SimDev s) {
  long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= s.N) return;
  int z = (int)(n / ((long long)s.nx * s.ny));
  const int x = (int)(n % s.nx), y = (int)((n / s.nx) % s.ny);
  s.mask[n] = static_wall(s, x, y, z) ? 1 : 0;
  s.claim[n] = 0xFFFFFFFFu;
}

// fluid at rest: f = w rho0 (d = 0), moments (rho0, phi0) in both moment
// buffers (phi0 staged in the phi plane of rp[0]; (rho0, solid_phi(mask)) at solids)
template <int STORE>
__global__ void k_init_pops(SimDev s, void* pops) {
  using IO = Codec<STORE>;
  using T = typename IO::T;
  long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= s.N) return;
  T* b = (T*)pops;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const float wr0 = wq(i) * s.rho0;
    IO::st(b + pidx(i, (int)s.N, (int)n), wr0, 1.0f / wr0, wr0, 0.f);
  }
  const uint16_t m0 = s.mask[n];
  const float p0 = (m0 == 0) ? s.rp[0][s.N + n] : solid_phi(m0);
  for (int k = 0; k < 2; ++k) {
    s.rp[k][n] = s.rho0;
    s.rp[k][s.N + n] = p0;
  }
}

// --------------------------------------------------------- global mass (FP64)
// masses of fluids a and b, sum of rho (1 +- phi) / 2 over fluid nodes, from
// the moments rp (rho plane, phi plane) of the current state, added into
// acc[0], acc[1] (cleared by the caller).  FP32 keeps no density where phi is
// +-1: it is summed from the populations there
template <int STORE>
__global__ __launch_bounds__(256) void k_mass(SimDev s, const float* __restrict__ rp,
                                              const void* __restrict__ pops,
                                              double* __restrict__ acc) {
  using T = typename Codec<STORE>::T;
  __shared__ double sh[2][256];
  double a = 0.0, b = 0.0;
  for (long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x; n < s.N;
       n += (long long)gridDim.x * blockDim.x) {
    if (s.mask[n] != 0) continue;
    const float phi = rp[s.N + n];
    const double rho = STORE == 0 && phi_pure(phi)
                           ? (double)node_density<STORE>(gp((const T*)pops), (int)s.N, (int)n,
                                                         s.rho0, 0.f)
                           : (double)rp[n];
    const double sg = rho * (double)phi;
    a += 0.5 * (rho + sg);
    b += 0.5 * (rho - sg);
  }
  sh[0][threadIdx.x] = a;
  sh[1][threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + o];
      sh[1][threadIdx.x] += sh[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    atomicAdd(&acc[0], sh[0][0]);
    atomicAdd(&acc[1], sh[1][0]);
  }
}

// n doubles set to zero (a kernel, not a memset: safe inside a captured graph)
__global__ void k_zero_f64(double* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

enum { MODE_STEP = 0, MODE_FIELDS = 1 };

// ------------------------------------------------------ interface kernels
// Colour gradient G = 3 sum_i w_i c_i phi(x + c_i) (isotropic stencil, the value
// at x for solid neighbours), the geometric wetting rotation next to solids,
// the normal n = G / max(|G|, EPS_G); then the curvature kappa = div n (same
// stencil and closure), the CSF coefficient c = -sigma kappa max(|G|, EPS_G) / 2
// (the surface-tension force is c n) and the set of directions whose neighbour
// is solid (bit i, bit 31 = node solid).  Written: the normal planes (n_x, n_y,
// n_z, |G|; NaN and -1 at a solid node) and the curvature word.
//
// One kernel: a block takes an x-y tile of the moments tiling and marches up
// its s.mkz planes.  phi of the tile grown by two nodes sits in an LDS ring of
// four planes, the normals of the tile grown by one node in a ring of three;
// per plane z the block loads phi of plane z + 2, forms the normals of plane
// z + 1 on the grown tile (a node's normal is formed once per block that needs
// it: 1.55 times per node for 64 x 4 tiles) and the curvature of plane z.  The
// normals never travel to HBM and back between the two stencils.
constexpr int IF_PHI = 68 * 8;          // largest tile plane grown by two: (64 + 4)(4 + 4)
constexpr int IF_NRM = MOM_HALO;  // grown by one: (64 + 2)(4 + 2)
// GEO: the geometries of the batch, so that the periodic box on a plane carries
// none of the others' bookkeeping and a tube without surface tension no queue of
// rotations (below) and nothing of a textured wall's.
// LX: as for the moments pass
struct IfLds {
  float fring[4][IF_PHI];
  // normals of three planes, one array per component (the curvature reads
  // only the components its stencil direction needs); |G| only where the
  // curvature needs it, at the tile's own nodes
  float nrx[3][IF_NRM], nry[3][IF_NRM], nrz[3][IF_NRM], nrg[2][256];
  uint32_t wcls[2][4];
  // entries that the wetting rotation is still to turn: 2 planes at most
  uint16_t wet[2 * IF_NRM];
  uint32_t n_wet;
};
static_assert(6 * sizeof(IfLds) <= 160 * 1024, "six blocks per CU");
template <int GEO, int LX>
__device__ __forceinline__ void interface_block(const Batch& bt, const SimDev& s, const int2 sb,
                                                IfLds& lds) {
  constexpr bool OPEN = GEO != GEO_PLAIN;
  auto& fring = lds.fring;
  auto &nrx = lds.nrx, &nry = lds.nry, &nrz = lds.nrz;
  auto& nrg = lds.nrg;
  auto& wcls = lds.wcls;
  const int N = (int)s.N;
  const GLB float* __restrict__ PHI = gp((const float*)s.rp[bt.rd ^ 1]) + s.N;
  GLB float* __restrict__ NX = gp(s.nrm);
  GLB float* __restrict__ CUR = gp((float*)s.curv);
  const int nx = s.nx, ny = s.ny, nz = s.nz, P = nx * ny;
  constexpr int tlx = LX, tx = 1 << tlx, ty = 256 >> tlx;
  constexpr int FX = tx + 4, FY = ty + 4, HX = tx + 2, HY = ty + 2;
  const int bx = sb.y % s.mtiles_x, r = sb.y / s.mtiles_x;
  const int mkz = bt.mkz > 0 ? bt.mkz : s.mkz;
  const int by = r % s.mtiles_y, z0 = (r / s.mtiles_y) * mkz;
  const int kz = min(mkz, nz - z0);
  const int t = (int)threadIdx.x;
  const int lx = t & (tx - 1), ly = t >> tlx;
  const int gx = bx * tx + lx, gy = by * ty + ly;
  const bool in = gx < nx && gy < ny;
  const int x0 = bx * tx, y0 = by * ty;
  // this thread's phi region entries (t, t + 256, t + 512): plane offsets
  // (-1: beyond an open x end, where phi reads as a solid's: the gradient and
  // curvature take the node's own value there and the direction is flagged)
  int foff[3];
  bool fon[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int k = t + 256 * j;
    fon[j] = k < FX * FY;
    const int fy = k / FX, fx = k - fy * FX;
    const int ax = x0 - 2 + fx;
    foff[j] = !fon[j] ? 0
              : (OPEN && s.open_x && (ax < 0 || ax >= nx)) ? -1
                                                   : wrapi(ax, nx) + nx * wrapi(y0 - 2 + fy, ny);
  }
  // this thread's normal region entries: first its own column and row of the
  // region's first tx x ty entries, then the region's two top rows and its
  // two right columns (2 tx + 2 ty + 4 <= 256 entries for the tiles used), so
  // that a wave's entries lie in whole rows: its phi reads are consecutive
  // LDS words (taken in region order, a wave's 64 entries crossed a row end,
  // and two of them met in one LDS bank)
  int hx_[2], hy_[2];
  bool hon[2];
  hx_[0] = lx;
  hy_[0] = ly;
  hon[0] = true;
  {
    const int u = t - 2 * tx;
    hon[1] = u < 2 * HY;
    hx_[1] = u < 0 ? lx : tx + (u & 1);
    hy_[1] = u < 0 ? ty + (t >> tlx) : (u >> 1);
  }
  auto zw = [&](int z) { return wrapi(z, nz); };
  auto fslot = [&](int z) { return (z + 8) & 3; };  // z >= -2
  auto nslot = [&](int z) { return (z + 3) % 3; };   // z >= -1
  auto gslot = [&](int z) { return (z + 2) & 1; };   // z >= -1
  auto load_phi = [&](int z, float* v) {
    const int zp = zw(z);
#pragma unroll
    for (int j = 0; j < 3; ++j)
      v[j] = !fon[j] ? 0.f : (OPEN && foff[j] < 0) ? PHI_SOLID : PHI[foff[j] + P * zp];
  };
  auto store_phi = [&](int z, const float* v) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (fon[j]) fring[fslot(z)][t + 256 * j] = v[j];
  };
  const float qnan = __int_as_float(0x7fc00000);
  // G as a unit vector (or less, below EPS_G) and |G|
  auto unit = [](float Gx, float Gy, float Gz) -> v4f {
    const float g = sqrtf(Gx * Gx + Gy * Gy + Gz * Gz);
    // 1 / max(g, EPS_G): the hardware reciprocal (within 1 ulp) and one Newton
    // step, which leaves it within a hair of half an ulp (the divisor lies in
    // [1e-4, 4], far from denormals and overflow); three instructions where the
    // full division takes twelve
    const float m = fmaxf(g, EPS_G);
    const float r0 = __builtin_amdgcn_rcpf(m);
    const float ig = __fmaf_rn(__fmaf_rn(-m, r0, 1.0f), r0, r0);
    return v4f{Gx * ig, Gy * ig, Gz * ig, g};
  };
  // normal of region entry (hx, hy) of plane z from the phi ring
  // SOL: a solid (or open-end) node may lie in the three phi planes read;
  // without, the per-neighbour tests are left out (a block-uniform choice)
  // (an entry inside the interface with a solid neighbour: `wet`, G itself)
  auto normal = [&](int hx, int hy, int z, bool& wet, auto SOL) -> v4f {
    const int c = (hx + 1) + FX * (hy + 1);
    const float* fm = fring[fslot(z - 1)];
    const float* f0 = fring[fslot(z)];
    const float* fp = fring[fslot(z + 1)];
    const float p0 = f0[c];
    if (decltype(SOL)::value && !(p0 < PHI_SOLID_TEST)) return v4f{qnan, qnan, qnan, -1.0f};
    float Gx = 0.f, Gy = 0.f, Gz = 0.f;
    bool solid = false;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int i = pair_dir(q);
      const float* sp_ = cz(i) > 0 ? fp : (cz(i) < 0 ? fm : f0);
      const float* sm_ = cz(i) > 0 ? fm : (cz(i) < 0 ? fp : f0);
      float vp = sp_[c + cx(i) + FX * cy(i)];
      float vm = sm_[c - cx(i) - FX * cy(i)];
      if constexpr (decltype(SOL)::value) {
        const bool spd = vp > PHI_SOLID_TEST, smd = vm > PHI_SOLID_TEST;
        solid |= spd | smd;
        vp = spd ? p0 : vp;
        vm = smd ? p0 : vm;
      }
      // G += 3 w_i c_i (phi(x + c_i) - phi(x - c_i)), each term one fused
      // multiply-add; terms with a zero lattice coefficient add nothing and are
      // left out (the compiler keeps 0 * d, which IEEE arithmetic does not fold)
      const float k = 3.0f * wq(i), df = vp - vm;
      if (cx(i) != 0) Gx = __fmaf_rn((float)cx(i) * k, df, Gx);
      if (cy(i) != 0) Gy = __fmaf_rn((float)cy(i) * k, df, Gy);
      if (cz(i) != 0) Gz = __fmaf_rn((float)cz(i) * k, df, Gz);
    }
    v4f v = unit(Gx, Gy, Gz);
    wet = decltype(SOL)::value && solid && v.w > EPS_G;
    if (wet) v = v4f{Gx, Gy, Gz, v.w};
    return v;
  };
  auto put_normal = [&](int hx, int hy, int z, v4f v) {
    const int sl = nslot(z), k = hx + HX * hy;
    nrx[sl][k] = v.x;
    nry[sl][k] = v.y;
    nrz[sl][k] = v.z;
    // a tile node: its |G| kept for the curvature
    const int tlx = hx - 1, tly = hy - 1;
    if (tlx >= 0 && tlx < tx && tly >= 0 && tly < ty) nrg[gslot(z)][tlx + tx * tly] = v.w;
  };
  // The wetting rotation applies only inside the interface (|G| > EPS_G, its own
  // first test); only there the solid is identified, from the phi codes of the
  // neighbours in the ring: the lowest-index particle, else the wall (an open end
  // is neither).
  auto rotated = [&](int hx, int hy, int z, float Gx, float Gy, float Gz) -> v4f {
    const int c = (hx + 1) + FX * (hy + 1);
    const float* fm = fring[fslot(z - 1)];
    const float* f0 = fring[fslot(z)];
    const float* fp = fring[fslot(z + 1)];
    float pmin = 3.0e38f;
    bool wall = false;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int i = pair_dir(q);
      const float* sp_ = cz(i) > 0 ? fp : (cz(i) < 0 ? fm : f0);
      const float* sm_ = cz(i) > 0 ? fm : (cz(i) < 0 ? fp : f0);
      const float vp = sp_[c + cx(i) + FX * cy(i)];
      const float vm = sm_[c - cx(i) - FX * cy(i)];
      wall |= vp == solid_phi(1) || vm == solid_phi(1);
      if (vp >= solid_phi(2)) pmin = fminf(pmin, vp);
      if (vm >= solid_phi(2)) pmin = fminf(pmin, vm);
    }
    if (wall || pmin < 3.0e38f) {
      const int ax = wrapi(x0 - 1 + hx, nx), ay = wrapi(y0 - 1 + hy, ny), az = zw(z);
      const int minp = pmin < 3.0e38f ? (int)(pmin - solid_phi(2)) : -1;
      wetting_rotate<GEO>(s, ax, ay, az, minp, wall, Gx, Gy, Gz);
    }
    return unit(Gx, Gy, Gz);
  };
  // A few entries of a plane are rotated, and the chain is long (the scan, the
  // particle's record from memory, square roots and divisions in FP64): they are
  // queued, and all of up to two planes take it at once, a thread each.  Each
  // thread for its own two entries as they came, a block passed the chain twice
  // per plane (sphere of radius 10 in 32x32x52: 19.6 -> 14.7 us, a drop on pillars
  // in 256x128x64 66 -> 43, a layer along the axis of a 320x83x83 tube 60.6 -> 42.3, a
  // plug in it 40.9 -> 42.5, a drop 34.2 -> 34.4).  One fluid alone has none to turn, and
  // the queue's registers cost it a wave per SIMD (28.2 us against 25.8): the tube
  // without surface tension goes without.
  constexpr bool QUEUE = GEO != GEO_TUBE;
  // up: 1 for the upper of two planes that are formed before rotate_wet
  auto normals = [&](int z, int up, auto SOL) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      bool wet = false;
      if (hon[j]) {
        v4f v = normal(hx_[j], hy_[j], z, wet, SOL);
        if (decltype(SOL)::value && !QUEUE && wet) v = rotated(hx_[j], hy_[j], z, v.x, v.y, v.z);
        put_normal(hx_[j], hy_[j], z, v);
      }
      if constexpr (decltype(SOL)::value && QUEUE) {
        // (the order is free; the compiler takes a wave's places at once)
        if (wet)
          lds.wet[atomicAdd(&lds.n_wet, 1u)] = (uint16_t)((hx_[j] + HX * hy_[j]) | (up << 15));
      }
    }
  };
  // the queued entries of plane z (and, marked up, z + 1), between the barrier
  // behind the normals and the one that this ends with
  auto rotate_wet = [&](int z) {
    if constexpr (QUEUE) {
      const uint32_t n_wet = __builtin_amdgcn_readfirstlane(lds.n_wet);
      if (n_wet == 0u) return;
      for (uint32_t w = t; w < n_wet; w += 256) {
        const uint32_t code = lds.wet[w];
        const int k = (int)(code & 0x7fffu), hy = k / HX, hx = k - HX * hy;
        const int zn = z + (int)(code >> 15), sl = nslot(zn);
        put_normal(hx, hy, zn, rotated(hx, hy, zn, nrx[sl][k], nry[sl][k], nrz[sl][k]));
      }
      __syncthreads();
      if (t == 0) lds.n_wet = 0u;
    }
  };
  const std::integral_constant<bool, true> with_solids;
  const std::integral_constant<bool, false> no_solids;
  // the normals of a plane whose phi planes hold one pure fluid: zero (NaN
  // at its solid nodes, if it may have any)
  auto zero_normals = [&](int z, bool solids) {
    const int sl = nslot(z);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (hon[j]) {
        const bool sd =
            solids && fring[fslot(z)][(hx_[j] + 1) + FX * (hy_[j] + 1)] > PHI_SOLID_TEST;
        const float v = sd ? qnan : 0.f;
        const int k = hx_[j] + HX * hy_[j];
        nrx[sl][k] = v;
        nry[sl][k] = v;
        nrz[sl][k] = v;
        const int tlx = hx_[j] - 1, tly = hy_[j] - 1;
        if (tlx >= 0 && tlx < tx && tly >= 0 && tly < ty)
          nrg[gslot(z)][tlx + tx * tly] = sd ? -1.f : 0.f;
      }
  };
  // what a phi plane of the grown tile holds: 1 phi = +1, 2 phi = -1, 4 a fluid
  // node of any other phi, 8 a solid (or open-end) node; each wave's word into
  // wcls, to be combined behind a barrier (two buffers in turn: a pure plane
  // passes one barrier only)
  auto classify = [&](const float* v, int shift) -> uint32_t {
    bool sd = false;
#pragma unroll
    for (int j = 0; j < 3; ++j) sd |= fon[j] && v[j] > PHI_SOLID_TEST;
    uint32_t c = __ballot(sd) ? 8u : 0u;
    // in the interface one value per lane tells (entry 0 always holds a node)
    if (__ballot(phi_mixed(v[0]))) {
      c |= 4u;
    } else {
      bool a = false, b = false, o = false;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a |= fon[j] && v[j] == 1.0f;
        b |= fon[j] && v[j] == -1.0f;
        o |= fon[j] && phi_mixed(v[j]);
      }
      c |= (__ballot(a) ? 1u : 0u) | (__ballot(b) ? 2u : 0u) | (__ballot(o) ? 4u : 0u);
    }
    return c << shift;
  };
  auto block_class = [&](int b) -> uint32_t {
    return __builtin_amdgcn_readfirstlane(wcls[b][0] | wcls[b][1] | wcls[b][2] | wcls[b][3]);
  };
  // one pure fluid (or only solids) in planes of the given classes
  auto pure_class = [](uint32_t c) { return (c & 4u) == 0u && (c & 3u) != 3u; };
  // prologue: phi of planes z0 - 2 .. z0 + 1, normals of planes z0 - 1, z0
  uint32_t pcls = 0;
  {
    float v[3];
    for (int dz = -2; dz <= 1; ++dz) {
      load_phi(z0 + dz, v);
      store_phi(z0 + dz, v);
      pcls |= classify(v, 4 * (1 - dz));
    }
  }
  float nxt[3];
  load_phi(z0 + 2, nxt);
  if ((t & 63) == 0) wcls[1][t >> 6] = pcls;
  if (t == 0) lds.n_wet = 0u;
  __syncthreads();
  // four bits for each of the phi planes z + 2 - k (k = 0 .. 4) of the current
  // plane z, once the loop has shifted in plane z + 2
  uint32_t hist = block_class(1);
  {
    // planes z0 - 2 .. z0 and z0 - 1 .. z0 + 1
    const uint32_t lo = (hist >> 4) | (hist >> 8) | (hist >> 12), hi = hist | (hist >> 4) | (hist >> 8);
    if (pure_class(lo & 15u))
      zero_normals(z0 - 1, (lo & 8u) != 0u);
    else if (lo & 8u)
      normals(z0 - 1, 0, with_solids);
    else
      normals(z0 - 1, 0, no_solids);
    if (pure_class(hi & 15u))
      zero_normals(z0, (hi & 8u) != 0u);
    else if (hi & 8u)
      normals(z0, 1, with_solids);
    else
      normals(z0, 1, no_solids);
  }
  __syncthreads();  // the loop's first phi store reuses the slot of plane z0 - 2
  if (hist & 0x8888u) rotate_wet(z0 - 1);
  // kept in a register: read from s after the stores below, it would be a
  // load behind them (they may alias s) and its wait would wait for them too
  const float csf = -0.5f * s.sigma;
  const int s_mtx = s.mtiles_x, s_mty = s.mtiles_y;
  // (not compiled in: instances per storage are slower, 512x256x192 192 -> 204 us
  // in FP32, 233 -> 247 in FP16)
  const bool fp16 = s.storage != 0;
  GLB uint8_t* __restrict__ KIND = gp(s.kind);
  for (int zz = 0; zz < kz; ++zz) {
    const int z = z0 + zz;
    store_phi(z + 2, nxt);
    {
      const uint32_t c = classify(nxt, 0);
      if ((t & 63) == 0) wcls[zz & 1][t >> 6] = c;
    }
    __syncthreads();
    hist = (hist << 4) | block_class(zz & 1);
    if (zz + 1 < kz) load_phi(z + 3, nxt);
    const uint32_t near = hist | (hist >> 4) | (hist >> 8);  // planes z .. z + 2
    const uint32_t all = near | (hist >> 12) | (hist >> 16);  // planes z - 2 .. z + 2
    const bool pure = pure_class(all & 15u);
    if (t == 0)
      KIND[(z * s_mty + by) * s_mtx + bx] =
          (hist & 0x700u) == 0u ? KIND_SOLID
          : !pure ? KIND_MIXED
                  : (uint8_t)(((all & 2u) ? KIND_PURE_B : KIND_PURE_A) + ((all & 8u) ? 2 : 0));
    if (pure_class(near & 15u))
      zero_normals(z + 1, (near & 8u) != 0u);
    else if (near & 8u)
      normals(z + 1, 0, with_solids);
    else
      normals(z + 1, 0, no_solids);
    if (pure) {
      // no normal, curvature or |G|; the solid-neighbour bits where there are
      // solids, from phi.  Without solids nothing of the rings is read here, and the
      // next plane's barrier orders the zeros just written
      uint32_t bits = 0u;
      if (all & 8u) {
        if (in) {
          const int n = gx + nx * (gy + ny * z);
          // (the index is hidden from the compiler, which would form the eighteen
          // addresses outside the march and spill the curvature's registers)
          int c = (lx + 2) + FX * (ly + 2);
          asm volatile("" : "+v"(c));
          bits = 0x80000000u;
          if (!(fring[fslot(z)][c] > PHI_SOLID_TEST)) {
            bits = 0u;
#pragma unroll
            for (int i = 1; i < Q; ++i)
              bits |= fring[fslot(z + cz(i))][c + cx(i) + FX * cy(i)] > PHI_SOLID_TEST ? (1u << i) : 0u;
          }
          if (!fp16) CUR[2 * n + 1] = __uint_as_float(bits);
        }
        __syncthreads();
      }
      if (fp16 && in) {
        const int n = gx + nx * (gy + ny * z);
        const bool sd = bits >> 31;
        const float v = sd ? qnan : 0.f;
        NX[n] = v;
        NX[N + n] = v;
        NX[2 * N + n] = v;
        NX[3 * N + n] = sd ? -1.f : 0.f;
        CUR[2 * n] = 0.f;
        CUR[2 * n + 1] = __uint_as_float(bits);
      }
      continue;
    }
    __syncthreads();
    if (near & 8u) rotate_wet(z + 1);
    // the curvature reads the normals of planes z - 1 .. z + 1
    const bool csol = (hist & 0x8880u) != 0u;
    if (in && !csol) {
      const int c0 = (lx + 1) + HX * (ly + 1);
      const int n = gx + nx * (gy + ny * z);
      const int s0 = nslot(z);
      const v4f own = v4f{nrx[s0][c0], nry[s0][c0], nrz[s0][c0], nrg[gslot(z)][t]};
      float kappa = 0.f;
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int i = pair_dir(q);
        const int sp_ = nslot(z + cz(i)), sm_ = nslot(z - cz(i));
        const int cp = c0 + cx(i) + HX * cy(i), cm = c0 - cx(i) - HX * cy(i);
        float dn = 0.f;
        if (cx(i) != 0) dn += (float)cx(i) * (nrx[sp_][cp] - nrx[sm_][cm]);
        if (cy(i) != 0) dn += (float)cy(i) * (nry[sp_][cp] - nry[sm_][cm]);
        if (cz(i) != 0) dn += (float)cz(i) * (nrz[sp_][cp] - nrz[sm_][cm]);
        kappa += 3.0f * wq(i) * dn;
      }
      NX[n] = own.x;
      NX[N + n] = own.y;
      NX[2 * N + n] = own.z;
      NX[3 * N + n] = own.w;
      CUR[2 * n] = csf * kappa * fmaxf(own.w, EPS_G);
      CUR[2 * n + 1] = __uint_as_float(0u);
    } else if (in) {
      const int c0 = (lx + 1) + HX * (ly + 1);
      const int n = gx + nx * (gy + ny * z);
      const int s0 = nslot(z);
      const v4f own = v4f{nrx[s0][c0], nry[s0][c0], nrz[s0][c0], nrg[gslot(z)][t]};
      float c = 0.f;
      uint32_t bits = 0x80000000u;
      if (own.w >= 0.f) {
        // pair by pair: the components c_i selects, of both neighbours (a
        // NaN marks a solid neighbour: its value is replaced by the node's own)
        float kappa = 0.f;
        bits = 0u;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          const int i = pair_dir(q), o = opp(i);
          const int sp_ = nslot(z + cz(i)), sm_ = nslot(z - cz(i));
          const int cp = c0 + cx(i) + HX * cy(i), cm = c0 - cx(i) - HX * cy(i);
          float px = cx(i) != 0 ? nrx[sp_][cp] : 0.f;
          float mx = cx(i) != 0 ? nrx[sm_][cm] : 0.f;
          float py = cy(i) != 0 ? nry[sp_][cp] : 0.f;
          float my = cy(i) != 0 ? nry[sm_][cm] : 0.f;
          float pz = cz(i) != 0 ? nrz[sp_][cp] : 0.f;
          float mz = cz(i) != 0 ? nrz[sm_][cm] : 0.f;
          const bool sp = (px != px) | (py != py) | (pz != pz);
          const bool sm = (mx != mx) | (my != my) | (mz != mz);
          if (sp) {
            px = own.x;
            py = own.y;
            pz = own.z;
          }
          if (sm) {
            mx = own.x;
            my = own.y;
            mz = own.z;
          }
          kappa += 3.0f * wq(i) * cdot(i, px - mx, py - my, pz - mz);
          bits |= (sp ? (1u << i) : 0u) | (sm ? (1u << o) : 0u);
        }
        c = csf * kappa * fmaxf(own.w, EPS_G);
      }
      NX[n] = own.x;
      NX[N + n] = own.y;
      NX[2 * N + n] = own.z;
      NX[3 * N + n] = own.w;
      CUR[2 * n] = c;
      CUR[2 * n + 1] = __uint_as_float(bits);
    }
  }
}

// W64: as for the moments pass
template <int GEO, bool W64>
// six waves per SIMD and blocks per CU; with all geometries five, as the rotation would
// spill (a layer in a tube 47.4 -> 42.3 us, a plug 45.6 -> 42.5)
__global__ __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(GEO == GEO_ANY ? 5 : 6, 8))) void k_interface(Batch bt) {
  __shared__ IfLds lds;
  const int2 sb = batch_block_in(bt, bt.mblk, blockIdx.x);
  const SimDev& s = bt.tab[sb.x];
  if (W64 || s.mtile_lx == 6)
    interface_block<GEO, 6>(bt, s, sb, lds);
  else if (s.mtile_lx == 5)
    interface_block<GEO, 5>(bt, s, sb, lds);
  else
    interface_block<GEO, 4>(bt, s, sb, lds);
}

// per-particle box of (phi, G) at the nodes the Lagrangian points interpolate
// (G after the wetting rotation, from the step's normal field): of a box of the
// simulation's side B the nodes from floor(x - R) to floor(x + R) + 1 per axis, the
// largest sphere's being the whole (one sphere of radius 20 beside 400 of radius 3, with
// the fused step: 425 us with whole boxes for all, 391 as a launch of their own, 154 so).
// block `block` of the `blocks` of particle p
__device__ __forceinline__ void capillary_box(const Batch& bt, const SimDev& s, int p, int block,
                                              int blocks) {
  DevParticle& P = s.P[p];
  const int B = s.cap_B;
  int org[3], w[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    org[k] = (int)floor(P.x[k] - P.R);
    w[k] = min((int)floor(P.x[k] + P.R) + 2 - org[k], B);
  }
  const int vol = w[0] * w[1] * w[2];
  // (no surface tension: no capillary force)
  if (s.cap_pref == 0.0 || block * 256 >= vol) return;
  float4* box = s.capbox + (long long)p * B * B * B;
  // the record's fields held in registers (the box stores may alias the record)
  const int nx = s.nx, ny = s.ny, nz = s.nz, N = (int)s.N;
  const GLB float* __restrict__ PHI = gp((const float*)s.rp[bt.rd ^ 1]) + N;
  const GLB float* __restrict__ NRM = gp((const float*)s.nrm);
  const GLB uint8_t* __restrict__ KIND = gp((const uint8_t*)s.kind);
  // a particle whose box holds no fluid node with |G| near EPS_G or above gets
  // no force: every point's G is a convex combination of corner values, so it
  // would fail the |G| > EPS_G test of the force kernel (the 0.99 margin covers
  // rounding); the box's nodes say so here, once, for that kernel
  bool iface = false;
  for (int k = block * 256 + (int)threadIdx.x; k < vol; k += blocks * 256) {
    const int ix = k % w[0], iy = (k / w[0]) % w[1], iz = k / (w[0] * w[1]);
    const int x = wrapi(org[0] + ix, nx), y = wrapi(org[1] + iy, ny), z = wrapi(org[2] + iz, nz);
    const unsigned n = (unsigned)(x + nx * (y + ny * z));
    // every plane read at once and the solid case taken by selects (a load
    // used only inside a branch is made there, a second round trip)
    const float gw = at(NRM + 3 * N, n), ph = at(PHI, n);
    const float n0 = at(NRM, n), n1 = at(NRM + N, n), n2 = at(NRM + 2 * N, n);
    const uint8_t kind = KIND[kind_index(s, x, y, z)];
    // G = n max(|G|, EPS_G): the colour gradient after the wetting rotation;
    // phi = 2 marks a solid node; on a pure tile plane G is zero and its
    // normal planes are not looked at
    const bool fl = !(ph > PHI_SOLID_TEST), mixed = fl && kind == KIND_MIXED;
    const float gm = fmaxf(gw, EPS_G);
    const float4 v = make_float4(fl ? ph : 2.f, mixed ? n0 * gm : 0.f, mixed ? n1 * gm : 0.f,
                                 mixed ? n2 * gm : 0.f);
    box[ix + B * (iy + B * iz)] = v;
    iface |= v.x <= 1.5f && v.y * v.y + v.z * v.z + v.w * v.w > (0.99f * EPS_G) * (0.99f * EPS_G);
  }
  if (__syncthreads_or(iface) && threadIdx.x == 0) P.cap_on = 1;
}

// ------------------------------------------------------------- fused kernel
// Per fluid node (one thread, x-fastest): populations in, the paper's collision
// on the total f (MRT + Guo forcing; the printed relaxation vector gives omega
// to every even and omega' = 8(2-omega)/(8-omega) to every odd non-conserved
// moment -- the two-relaxation-time operator computed here), the force c n +
// body force on fluid a, push streaming, and half-way bounce-back at every
// solid link.  The recolouring of f* into the two colours is not stored: the
// next moments pass rebuilds it from phi, rho and n of this state.  At
// particle links the moving-wall term and the momentum exchange are added by
// k_links.
// OPEN: the batch has simulations with open x ends (their anti-bounce-back is
// compiled into this instance only).
// FP32: cap_rows x cap_blocks blocks in front fill the particles' capillary boxes,
// which read the normals as this kernel does and are summed beside k_links.
template <int STORE, int MODE, bool OPEN>
// six waves per SIMD: the FP16 instance fits 80 VGPRs without spills (it took
// 85 and five waves; eight waves spill and nearly double its time); the FP32
// instances need fewer anyway
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_fused(Batch bt, int cap_rows,
                                              int cap_blocks, float* __restrict__ out_rho,
                                              float* __restrict__ out_u,
                                              float* __restrict__ out_phi,
                                              float* __restrict__ out_F) {
  using IO = Codec<STORE>;
  using T = typename IO::T;
  // (in FP16 zero, but by its arguments: as a constant the instance spills)
  const int first = MODE == MODE_STEP ? cap_rows * cap_blocks : 0;
  if (STORE == 0 && (int)blockIdx.x < first) {
    const int row = (int)blockIdx.x / cap_blocks;
    const int2 cp = batch_particle(bt, row);
    capillary_box(bt, bt.tab[cp.x], cp.y, (int)blockIdx.x - row * cap_blocks, cap_blocks);
    return;
  }
  const int2 sb = batch_block(bt, xcd_tile((int)blockIdx.x - first, (int)gridDim.x - first));
  const SimDev& s = bt.tab[sb.x];
  const GLB T* __restrict__ sp_ = gp((const T*)s.pops[bt.cur]);
  GLB T* __restrict__ dp_ = gp((T*)s.pops[bt.cur ^ 1]);
  const GLB float* __restrict__ NX = gp((const float*)s.nrm);
  // moments of this state (rho, phi planes) and of the one before it; FP16
  // decodes with the latter's density and encodes with the former's
  const GLB float* __restrict__ RM = gp((const float*)s.rp[bt.rd ^ 1]);
  const GLB float* __restrict__ RP = gp((const float*)s.rp[bt.rd]);
  const int nx = s.nx, ny = s.ny, nz = s.nz;
  const int N = (int)s.N;
  int n, gx, gy, gz;
  if (!tile_node(s, sb.y, n, gx, gy, gz)) return;
  const float rho0 = s.rho0;
  const float inv_rho0 = 1.0f / rho0;
  // on a pure tile plane the normal and the CSF coefficient are zero, phi is
  // known, and without solids near so are the neighbour bits: none is loaded
  const GLB float* __restrict__ cur = gp((const float*)s.curv);
  const int kind =
      STORE ? KIND_MIXED : gp((const uint8_t*)s.kind)[kind_index(s, gx, gy, gz)];
  uint32_t bits = 0u;
  if (kind == KIND_SOLID)
    bits = 0x80000000u;
  else if (kind >= KIND_PURE_A_SOLID)
    bits = __float_as_uint(at(cur, 2u * (unsigned)n + 1u));
  // MODE_FIELDS: the fields that are asked for
  auto put = [&](float r, float ph, float ux, float uy, float uz, float fx, float fy, float fz) {
    if (out_rho) out_rho[n] = r;
    if (out_phi) out_phi[n] = ph;
    if (out_u) {
      out_u[n] = ux;
      out_u[N + n] = uy;
      out_u[2 * N + n] = uz;
    }
    if (out_F) {
      out_F[n] = fx;
      out_F[N + n] = fy;
      out_F[2 * N + n] = fz;
    }
  };
  auto solid_node = [&]() {
    if (MODE == MODE_FIELDS) {
      const uint16_t m0 = s.mask[n];
      float ux = 0.f, uy = 0.f, uz = 0.f;
      if (m0 >= 2) {
        const DevParticle& P = s.P[m0 - 2];
        double rx = wrapd((double)gx - P.x[0], (double)nx);
        double ry = wrapd((double)gy - P.x[1], (double)ny);
        double rz = wrapd((double)gz - P.x[2], (double)nz);
        ux = (float)(P.v[0] + P.w[1] * rz - P.w[2] * ry);
        uy = (float)(P.v[1] + P.w[2] * rx - P.w[0] * rz);
        uz = (float)(P.v[2] + P.w[0] * ry - P.w[1] * rx);
      }
      put(0.f, 0.f, ux, uy, uz, 0.f, 0.f, 0.f);
    }
  };
  if (bits & 0x80000000u) {
    solid_node();
    return;
  }
  const Nbr nb(gx, gy, gz, nx, ny, nz);
  float d[Q];
  const float Rn = STORE ? at(RP, (unsigned)n) : 0.f;
  const auto pb = pop_base(sp_, n);
#pragma unroll
  for (int i = 0; i < Q; ++i) d[i] = IO::ld(pb + i * POP_BLOCK, wq(i) * rho0, wq(i) * Rn);
  // FP16: the densities of this state at the node and at its 18 neighbours,
  // the references the pushed populations are encoded with.  Loaded here with
  // the populations (neighbour indices wrap, so every load is in bounds): a
  // load at the push, behind the stores before it, would wait for those too.
  float Rd[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) Rd[i] = STORE ? at(RM, (unsigned)(i == 0 ? n : nb(i))) : 0.f;
  float3 nc = make_float3(0.f, 0.f, 0.f);
  float phi = pure_sign(kind), cb = 0.f;
  if (kind == KIND_MIXED) {
    nc = make_float3(at(NX, (unsigned)n), at(NX + N, (unsigned)n), at(NX + 2 * N, (unsigned)n));
    phi = at(RM + N, (unsigned)n);
    cb = at(cur, 2u * (unsigned)n);
    // here with the populations, not before them: few nodes of a mixed tile
    // plane are solid, and the wait would come before every load
    bits = __float_as_uint(at(cur, 2u * (unsigned)n + 1u));
    if (bits & 0x80000000u) {
      solid_node();
      return;
    }
  }
  float drho = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    drho += d[i];
    if (cx(i) != 0) jx += (float)cx(i) * d[i];
    if (cy(i) != 0) jy += (float)cy(i) * d[i];
    if (cz(i) != 0) jz += (float)cz(i) * d[i];
  }
  const float rho = rho0 + drho;
  // force: CSF surface tension c n + body force on fluid a (weight (1+phi)/2)
  const float fa = 0.5f * (1.0f + phi);
  const float Fx = cb * nc.x + s.body[0] * fa;
  const float Fy = cb * nc.y + s.body[1] * fa;
  const float Fz = cb * nc.z + s.body[2] * fa;
  const float irho = 1.0f / rho;
  const float ux = (jx + 0.5f * Fx) * irho;
  const float uy = (jy + 0.5f * Fy) * irho;
  const float uz = (jz + 0.5f * Fz) * irho;
  const float uu = ux * ux + uy * uy + uz * uz;

  if (MODE == MODE_FIELDS) {
    put(rho, phi, ux, uy, uz, Fx, Fy, Fz);
    return;
  }
  if (!(rho > 0.f) || !(uu <= 0.09f)) atomicOr(&s.counters[1], (uint32_t)ST_UNSTABLE);
  // next to a solid the density of the colliding state for the link kernel: the
  // moments pass keeps none on a pure tile plane (one that is mixed now may
  // have been pure then, but not around a node of another phi than +-1)
  if (STORE == 0 && bits != 0u && phi_pure(phi)) gp(s.rp[bt.rd ^ 1])[n] = rho;
  // local relaxation: harmonic mean of the kinematic viscosities
  const float inv_nu = (1.0f + phi) * s.inv2nua + (1.0f - phi) * s.inv2nub;
  const float om = 1.0f / (0.5f + 3.0f / inv_nu);
  const float om2 = 8.0f * (2.0f - om) / (8.0f - om);
  const float cfs = 1.0f - 0.5f * om, cfa = 1.0f - 0.5f * om2;
  const float uF = ux * Fx + uy * Fy + uz * Fz;

  // FP16: each population is encoded with the density of the node that
  // stores it
  auto st_pop = [&](int i, int node, float R, float dv) {
    IO::st(dp_ + pidx(i, N, node), wq(i) * rho0, inv_rho0 * (1.0f / wq(i)), wq(i) * R, dv);
  };
  // push to the neighbour in direction i, or bounce back into direction opp(i);
  // through an open x end the anti-bounce-back of the pressure boundary
  // (pressure inlet/outlet eq.): f_opp = -f*_i + 2 w_i rho_w (1 + 9/2 (c_i.u)^2
  // - 3/2 u^2), u the node's velocity, p_w = rho_w / 3
  auto emit = [&](int i, float dv) {
    if (bits & (1u << i)) {
      if (OPEN && s.open_x && ((cx(i) < 0 && gx == 0) || (cx(i) > 0 && gx == nx - 1))) {
        const float drw = cx(i) < 0 ? s.drho_in : s.drho_out;
        const float cu = cdot(i, ux, uy, uz);
        const float w = wq(i);
        // as deviations from w rho0: -d*_i + 2 w (drho_w + rho_w (9/2 cu^2 - 3/2 u^2))
        st_pop(opp(i), n, Rd[0], -dv + 2.0f * w * (drw + (rho0 + drw) * (4.5f * cu * cu - 1.5f * uu)));
      } else {
        st_pop(opp(i), n, Rd[0], dv);
      }
    } else {
      st_pop(i, nb(i), Rd[i], dv);
    }
  };

  {
    const float w0 = wq(0);
    const float deq = w0 * (drho - 1.5f * rho * uu);
    const float fb = w0 * (-3.0f * uF);
    st_pop(0, n, Rd[0], d[0] - om * (d[0] - deq) + cfs * fb);
  }
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int i = pair_dir(q);
    const int o = opp(i);
    const float w = wq(i);
    const float cu = cdot(i, ux, uy, uz);
    const float cF = cdot(i, Fx, Fy, Fz);
    const float eqs = w * (drho + rho * (4.5f * cu * cu - 1.5f * uu));
    const float eqa = w * rho * 3.0f * cu;
    const float fs = w * (9.0f * cu * cF - 3.0f * uF);
    const float fa2 = w * 3.0f * cF;
    const float sy = 0.5f * (d[i] + d[o]) - eqs;
    const float an = 0.5f * (d[i] - d[o]) - eqa;
    const float common = -om * sy + cfs * fs;
    const float anti = -om2 * an + cfa * fa2;
    emit(i, d[i] + common + anti);
    emit(o, d[o] + common - anti);
  }
}

// The capillary boxes of a batch in FP16: in the launch of k_fused their code costs
// that instance, which fills its 80 VGPRs, a spill per node (582 -> 605 us in
// 512x256x192 with 500 spheres, against 19 for this launch; with one sphere 4).
__global__ __launch_bounds__(256) void k_capbox(Batch bt) {
  const int2 cp = batch_particle(bt, (int)blockIdx.y);
  capillary_box(bt, bt.tab[cp.x], cp.y, (int)blockIdx.x, (int)gridDim.x);
}

// Six sums over the threads of a block of 256: true, with the sum in v, for
// thread c < 6 of component c.
__device__ __forceinline__ bool block_sum6(double* acc, double (*red)[6], double& v) {
#pragma unroll
  for (int c = 0; c < 6; ++c)
    for (int off = 32; off > 0; off >>= 1) acc[c] += __shfl_xor(acc[c], off, 64);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    for (int c = 0; c < 6; ++c) red[wave][c] = acc[c];
  __syncthreads();
  if (threadIdx.x >= 6) return false;
  v = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
  return true;
}

// Capillary force (capillary-force eq.): sum over the polar/azimuthal grid of
// sigma 9/2 k beta max(0, 1 - phi^2) dA sin(theta_p) m^, m^ = normalise(n_s - (n.n_s) n),
// torque arm R n_s; phi and G trilinear over fluid corners, from the box that
// k_fused's launch filled.  Block `block` of the `blocks` of a particle, FP64 block
// reductions combined with FP64 atomics (the accumulators are consumed and cleared
// by the DEM).
constexpr int CAP_TAB = 512;
struct CapLds {
  double tab[4][CAP_TAB];
  double red[4][6];
};
__device__ __forceinline__ void capillary_block(const SimDev& s, int p, int block, int blocks,
                                                CapLds& lds) {
  DevParticle& P = s.P[p];
  if (s.cap_pref == 0.0) return;  // no surface tension: no capillary force
  const int B = s.cap_B;
  const GLB v4f* box = gp((const v4f*)s.capbox) + (long long)p * B * B * B;
  const int org0 = (int)floor(P.x[0] - P.R), org1 = (int)floor(P.x[1] - P.R),
            org2 = (int)floor(P.x[2] - P.R);
  const double R = P.R, da = s.cap_dang;
  const double pref = s.cap_pref * (double)P.sin_t;
  const int na = s.cap_na, nph = s.cap_nphi;
  // the polar and azimuthal grids are fixed: their sines and cosines once per
  // workgroup (same arguments, same values as per point)
  // no fluid node of the box near the interface (the box kernel's flag): no force
  if (!P.cap_on) return;
  constexpr int TAB = CAP_TAB;
  double *t_sa = lds.tab[0], *t_ca = lds.tab[1], *t_sp = lds.tab[2], *t_cp = lds.tab[3];
  const bool tab = na <= TAB && nph <= TAB;
  if (tab) {
    for (int j = threadIdx.x; j < na; j += blockDim.x) sincos((j + 0.5) * da, &t_sa[j], &t_ca[j]);
    for (int k = threadIdx.x; k < nph; k += blockDim.x) sincos(k * da, &t_sp[k], &t_cp[k]);
  }
  __syncthreads();
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int idx = block * 256 + (int)threadIdx.x; idx < na * nph; idx += blocks * 256) {
    const int j = idx / nph, k = idx % nph;
    double sa, ca, sp, cp;
    if (tab) {
      sa = t_sa[j];
      ca = t_ca[j];
      sp = t_sp[k];
      cp = t_cp[k];
    } else {
      sincos((j + 0.5) * da, &sa, &ca);
      sincos(k * da, &sp, &cp);
    }
    const double sh[3] = {sa * cp, sa * sp, ca};
    const double xp[3] = {P.x[0] + R * sh[0], P.x[1] + R * sh[1], P.x[2] + R * sh[2]};
    const double f0 = floor(xp[0]), f1 = floor(xp[1]), f2 = floor(xp[2]);
    const double fr0 = xp[0] - f0, fr1 = xp[1] - f1, fr2 = xp[2] - f2;
    const int i0 = (int)f0 - org0, i1 = (int)f1 - org1, i2 = (int)f2 - org2;
    // per-point arithmetic in FP64: the torque is a small residual of large,
    // cancelling per-point moments
    double W = 0.0, phi = 0.0, Gx = 0.0, Gy = 0.0, Gz = 0.0;
    // the eight corners loaded at once; a solid corner (phi = 2) takes weight
    // 0, which adds exact zeros (the box holds finite values): the same sums as
    // leaving it out, without a load round trip per corner
    v4f cv[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int ox = c & 1, oy = (c >> 1) & 1, oz = c >> 2;
      cv[c] = box[(i0 + ox) + B * ((i1 + oy) + B * (i2 + oz))];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int ox = c & 1, oy = (c >> 1) & 1, oz = c >> 2;
      const v4f v = cv[c];
      const double w = (ox ? fr0 : 1.0 - fr0) * (oy ? fr1 : 1.0 - fr1) * (oz ? fr2 : 1.0 - fr2);
      const double wf = v.x > 1.5f ? 0.0 : w;
      W += wf;
      phi += wf * (double)v.x;
      Gx += wf * (double)v.y;
      Gy += wf * (double)v.z;
      Gz += wf * (double)v.w;
    }
    // the three tests at once, after the values they need (W = 0 gives NaN,
    // which fails them): a test on W and phi alone before G is formed would let
    // the compiler load the corners' G only after it, a second round trip
    const double iW = 1.0 / W;
    phi *= iW;
    Gx *= iW;
    Gy *= iW;
    Gz *= iW;
    const double wgt = 1.0 - phi * phi;
    const double g = sqrt(Gx * Gx + Gy * Gy + Gz * Gz);
    if (!(W > 0.0) || !(wgt > 0.0) || !(g > (double)EPS_G)) continue;
    const double ig = 1.0 / g;
    const double nx_ = Gx * ig, ny_ = Gy * ig, nz_ = Gz * ig;
    const double a = nx_ * sh[0] + ny_ * sh[1] + nz_ * sh[2];
    const double mx = sh[0] - a * nx_, my = sh[1] - a * ny_, mz = sh[2] - a * nz_;
    const double mn = sqrt(mx * mx + my * my + mz * mz);
    if (!(mn > (double)EPS_T)) continue;
    const double dA = R * R * sa * da * da;
    const double coef = pref * wgt * dA / mn;
    const double dF[3] = {coef * mx, coef * my, coef * mz};
    const double arm[3] = {R * sh[0], R * sh[1], R * sh[2]};
    acc[0] += dF[0];
    acc[1] += dF[1];
    acc[2] += dF[2];
    acc[3] += arm[1] * dF[2] - arm[2] * dF[1];
    acc[4] += arm[2] * dF[0] - arm[0] * dF[2];
    acc[5] += arm[0] * dF[1] - arm[1] * dF[0];
  }
  double v;
  if (block_sum6(acc, lds.red, v)) {
    if (threadIdx.x < 3)
      atomicAdd(&P.Fca[threadIdx.x], v);
    else
      atomicAdd(&P.Tca[threadIdx.x - 3], v);
  }
}

// Moving-wall correction and momentum exchange on particle links, after
// k_fused has bounced f*_i back into direction opp(i) at the fluid node x:
// f_opp(x) += 6 w_i rho(x) (c_opp . u_w) (its colour share phi(x) is added by
// the moments pass, as for every bounced population), with
// u_w = V + Omega x (x + c_i/2 - X) (half-way bounce-back eqs.), and the
// momentum given to the particle dP = (c_i - u_w) f*_i - (c_opp - u_w) f_opp
// (hydrodynamic force eqs.), summed in FP64 per particle.  One grid row per
// particle over the nodes of its bounding box grown by one; with capillary
// forces the row's blocks from link_blocks on sum those, which need nothing of the
// others (the dependent chains of both hide each other's: one sphere 11.5 + 8 -> 11 us, 20
// spheres 14 + 5 -> 15.7, 500 spheres 77 + 25 -> 81).
// The grid is sized by the largest sphere; a block past its particle's box leaves at once
// (one sphere of radius 20 beside 400 of radius 3: 230 -> 136 us.  Blocks that take
// several turns instead need 196 VGPRs for 116: 79 us there, but 1,000 spheres of radius 8
// 314 -> 473).
template <int STORE>
__global__ __launch_bounds__(256) void k_links(Batch bt, int link_blocks) {
  __shared__ union {
    double red[4][6];
    CapLds cap;
  } u;
  // one thread per node of the particle's box; runs after k_fused, before the
  // buffers swap: src holds the state it read, dst the state it wrote
  using IO = Codec<STORE>;
  using T = typename IO::T;
  const int2 sp = batch_particle(bt, blockIdx.y);
  const SimDev& s = bt.tab[sp.x];
  const int p = sp.y;
  if ((int)blockIdx.x >= link_blocks) {
    capillary_block(s, p, (int)blockIdx.x - link_blocks, (int)gridDim.x - link_blocks, u.cap);
    return;
  }
  GLB T* __restrict__ dp_ = gp((T*)s.pops[bt.cur ^ 1]);
  // moments of the state that collided: rho(x), and the FP16 reference of the
  // populations k_fused wrote
  const GLB float* __restrict__ RM = gp((const float*)s.rp[bt.rd ^ 1]);
  const GLB uint16_t* __restrict__ MASK = gp((const uint16_t*)s.mask);
  // the record's fields in registers: read from it behind the population stores
  // they were loaded again in every direction (one sphere 13 -> 9.7 us, 20 spheres
  // 19 -> 14.8, 500 spheres 82 -> 68, with the half-way coordinates formed once)
  const DevParticle& P = s.P[p];
  const double X0 = P.x[0], X1 = P.x[1], X2 = P.x[2], R = P.R;
  const double V0 = P.v[0], V1 = P.v[1], V2 = P.v[2];
  const double W0 = P.w[0], W1 = P.w[1], W2 = P.w[2];
  const int nx = s.nx, ny = s.ny, nz = s.nz, N = (int)s.N;
  const float rho0 = s.rho0;
  int lo[3], w[3];
  const int L[3] = {nx, ny, nz};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double X = k == 0 ? X0 : (k == 1 ? X1 : X2);
    lo[k] = (int)floor(X - R) - 2;
    w[k] = (int)floor(X + R) + 2 - lo[k] + 1;
    if (w[k] > L[k]) {
      lo[k] = 0;
      w[k] = L[k];
    }
  }
  const int vol = w[0] * w[1] * w[2];
  if ((int)(blockIdx.x * blockDim.x) >= vol) return;
  double acc[6] = {0, 0, 0, 0, 0, 0};
  bool any = false;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < vol) {
    const int gx = wrapi(lo[0] + k % w[0], nx);
    const int gy = wrapi(lo[1] + (k / w[0]) % w[1], ny);
    const int gz = wrapi(lo[2] + k / (w[0] * w[1]), nz);
    // a fluid node with a link to p lies within R + sqrt(2) of its centre and
    // not inside (R - 0.5 leaves room for rounding): others load nothing
    const double dx = wrapd((double)gx - X0, (double)nx);
    const double dy = wrapd((double)gy - X1, (double)ny);
    const double dz = wrapd((double)gz - X2, (double)nz);
    const double d2 = dx * dx + dy * dy + dz * dz;
    const double rlo = R - 0.5, rhi = R + 1.5;
    const int n = gx + nx * (gy + ny * gz);
    if (d2 < rhi * rhi && (rlo <= 0.0 || d2 >= rlo * rlo)) {
      // the node's and its neighbours' masks, its density and the 18
      // populations that bounce-back may have written, all in one round trip
      // (reading the populations only after the masks, in the link directions,
      // moves less data but adds a round trip: C2 16 -> 20 us)
      const Nbr nb(gx, gy, gz, nx, ny, nz);
      const uint16_t me = (uint16_t)(2 + p);
      const uint16_t m0 = at(MASK, (unsigned)n);
      uint32_t lm = 0;  // bit i: the neighbour in direction i is a solid node of p
#pragma unroll
      for (int i = 1; i < Q; ++i) lm |= (at(MASK, (unsigned)nb(i)) == me) ? (1u << i) : 0u;
      const float rho = at(RM, (unsigned)n);
      const float Re = STORE ? rho : 0.f;
      const auto pb = pop_base(dp_, n);
      float ds[Q];
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const int o = opp(i);
        ds[i] = IO::ld(pb + o * POP_BLOCK, wq(o) * rho0, wq(o) * Re);
      }
      if (m0 != 0) lm = 0;
      if (lm) {
        any = true;
        // the half-way points' coordinates from the centre, three per axis
        double rxs[3], rys[3], rzs[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          rxs[c] = wrapd((double)gx + 0.5 * (c - 1) - X0, (double)nx);
          rys[c] = wrapd((double)gy + 0.5 * (c - 1) - X1, (double)ny);
          rzs[c] = wrapd((double)gz + 0.5 * (c - 1) - X2, (double)nz);
        }
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          if (!(lm & (1u << i))) continue;
          const int o = opp(i);
          const float wr0 = wq(o) * rho0;
          const double rx = rxs[1 + cx(i)], ry = rys[1 + cy(i)], rz = rzs[1 + cz(i)];
          const double uwx = V0 + (W1 * rz - W2 * ry);
          const double uwy = V1 + (W2 * rx - W0 * rz);
          const double uwz = V2 + (W0 * ry - W1 * rx);
          const float cu = (float)(-(cx(i) * uwx + cy(i) * uwy + cz(i) * uwz));  // c_opp . u_w
          const float corr = 6.0f * wq(i) * rho * cu;
          const float dso = ds[i] + corr;
          IO::st(pb + o * POP_BLOCK, wr0, 1.0f / wr0, wq(o) * Re, dso);
          const double wr = wqd(i) * (double)rho0;
          const double fin = (double)ds[i] + wr;
          const double fout = (double)dso + wr;
          // (c_i - u_w) f*_i - (c_opp - u_w) f_opp
          const double sum = fin + fout, dif = fin - fout;
          const double dPx = cx(i) * sum - uwx * dif;
          const double dPy = cy(i) * sum - uwy * dif;
          const double dPz = cz(i) * sum - uwz * dif;
          acc[0] += dPx;
          acc[1] += dPy;
          acc[2] += dPz;
          acc[3] += ry * dPz - rz * dPy;
          acc[4] += rz * dPx - rx * dPz;
          acc[5] += rx * dPy - ry * dPx;
        }
      }
    }
  }
  if (!__syncthreads_or(any)) return;  // no link in this block
  double v;
  if (block_sum6(acc, u.red, v) && v != 0.0) {
    DevParticle* Pw = s.P + p;
    if (threadIdx.x < 3)
      atomicAdd(&Pw->Fh[threadIdx.x], v);
    else
      atomicAdd(&Pw->Th[threadIdx.x - 3], v);
  }
}

// ------------------------------------------------------------ host launchers
static inline unsigned nblocks(long long n, int b) { return (unsigned)((n + b - 1) / b); }

// Batched launchers: one launch over every simulation of the batch.
// nblk: total 256-node blocks; np_rows: total particle rows; Bmax: the largest
// mask-box side of the batch.
// mnblk: blocks of the moments tiling
template <int GEO>
static hipError_t launch_interface_geo(const Batch& b, unsigned mnblk, hipStream_t st) {
  if (b.mlx == 6)
    hipLaunchKernelGGL((k_interface<GEO, true>), dim3(mnblk), dim3(256), 0, st, b);
  else
    hipLaunchKernelGGL((k_interface<GEO, false>), dim3(mnblk), dim3(256), 0, st, b);
  return hipGetLastError();
}
hipError_t launch_interface(const Batch& b, unsigned mnblk, hipStream_t st) {
  if (b.geometry == GEO_PLAIN) return launch_interface_geo<GEO_PLAIN>(b, mnblk, st);
  if (b.geometry == GEO_TUBE) return launch_interface_geo<GEO_TUBE>(b, mnblk, st);
  return launch_interface_geo<GEO_ANY>(b, mnblk, st);
}

// cap_rows particle rows (0: none) fill their capillary boxes of at most Bcap nodes
// a side, in a step; own: blocks that the particles' own boxes take
hipError_t launch_fused(const Batch& b, int storage, unsigned nblk, int cap_rows, int Bcap,
                        long long own, hipStream_t st) {
  const dim3 t(256);
  float* const no = nullptr;
  if (storage == 0) {
    const int cap_blocks = particle_blocks_flat(nblk, cap_rows, Bcap, own);
    const dim3 grid(nblk + (unsigned)cap_rows * (unsigned)cap_blocks);
    if (b.open)
      hipLaunchKernelGGL((k_fused<0, MODE_STEP, true>), grid, t, 0, st, b, cap_rows, cap_blocks, no,
                         no, no, no);
    else
      hipLaunchKernelGGL((k_fused<0, MODE_STEP, false>), grid, t, 0, st, b, cap_rows, cap_blocks,
                         no, no, no, no);
  } else {
    if (cap_rows > 0)
      hipLaunchKernelGGL(k_capbox, dim3(particle_blocks(cap_rows, Bcap, own), cap_rows), t, 0, st, b);
    if (b.open)
      hipLaunchKernelGGL((k_fused<1, MODE_STEP, true>), dim3(nblk), t, 0, st, b, 0, 0, no, no, no,
                         no);
    else
      hipLaunchKernelGGL((k_fused<1, MODE_STEP, false>), dim3(nblk), t, 0, st, b, 0, 0, no, no, no,
                         no);
  }
  return hipGetLastError();
}

// the fields of the current state, written where a pointer is given; it writes no
// populations and needs no open-end instance
hipError_t launch_fields(const Batch& b, int storage, unsigned nblk, float* orho, float* ou,
                         float* ophi, float* oF, hipStream_t st) {
  const dim3 grid(nblk), t(256);
  if (storage == 0)
    hipLaunchKernelGGL((k_fused<0, MODE_FIELDS, false>), grid, t, 0, st, b, 0, 0, orho, ou, ophi,
                       oF);
  else
    hipLaunchKernelGGL((k_fused<1, MODE_FIELDS, false>), grid, t, 0, st, b, 0, 0, orho, ou, ophi,
                       oF);
  return hipGetLastError();
}

// npts: Lagrangian points per particle, 0: no capillary forces
hipError_t launch_links(const Batch& b, int storage, int np_rows, int Bmax, int npts,
                        hipStream_t st) {
  if (np_rows == 0) return hipSuccess;
  // the box of k_links spans at most 2 R + 6 nodes per axis, R <= (Bmask - 5) / 2
  const long long B = Bmax + 1;
  const unsigned nl = nblocks(B * B * B, 256);
  // workgroups per particle: four points per thread, or down to one where
  // few particles leave the GPU idle (about 2,048 workgroups in all)
  const int wide = std::min(npts / 256, (2048 + np_rows - 1) / np_rows);
  const int many = std::max(1, (4096 + np_rows - 1) / np_rows);
  const int split = std::max(1, std::min(64, std::max(std::min(npts / (256 * 4), many), wide)));
  const dim3 grid(nl + (npts > 0 ? split : 0), np_rows);
  if (storage == 0)
    hipLaunchKernelGGL(k_links<0>, grid, dim3(256), 0, st, b, (int)nl);
  else
    hipLaunchKernelGGL(k_links<1>, grid, dim3(256), 0, st, b, (int)nl);
  return hipGetLastError();
}

// Blocks of 14 fresh nodes per simulation that refill: two per particle of the
// busiest simulation (128 to 1,024 in all for one simulation; at least four for
// each of a batch).  The fresh nodes of a step scale with the moving particles,
// and a block that must take a second round of them doubles the dependent chain
// (500 spheres: 196 -> 185 us for the particle phase with 1,000 blocks instead of
// 128); a batch's idle blocks cost too (64 boxes with 128 each: 16 us).
static int refill_blocks(size_t fresh_cap_max, int np_max, int nsim) {
  if (fresh_cap_max == 0) return 0;
  const size_t all = (fresh_cap_max + REFILL_PER - 1) / REFILL_PER;
  const int least = nsim == 1 ? 128 : 4;
  return (int)std::min<size_t>(all, (size_t)std::min(1024, std::max(least, 2 * np_max)));
}

// in a step: the refill of the fresh nodes and the moments of all others; mnblk
// blocks of the moments tiling, fresh_cap_max: the largest fresh-list capacity of
// the batch (0: no refill), np_max: the most particles of one simulation
hipError_t launch_moments(const Batch& b, int storage, unsigned mnblk, size_t fresh_cap_max,
                          int np_max, hipStream_t st) {
  const int nref = refill_blocks(fresh_cap_max, np_max, b.nsim);
  const dim3 g(mnblk + (unsigned)(b.nsim * nref)), t(256);
  if (storage == 0) {
    if (b.mlx == 6)
      hipLaunchKernelGGL((k_moments<0, true>), g, t, 0, st, b, nref);
    else
      hipLaunchKernelGGL((k_moments<0, false>), g, t, 0, st, b, nref);
  } else {
    if (b.mlx == 6)
      hipLaunchKernelGGL((k_moments<1, true>), g, t, 0, st, b, nref);
    else
      hipLaunchKernelGGL((k_moments<1, false>), g, t, 0, st, b, nref);
  }
  return hipGetLastError();
}

// between steps, after the mask changed (one simulation; nblk per-node blocks)
hipError_t launch_boundary(const Batch& b, int storage, unsigned nblk, size_t fresh_cap_max,
                           int np_max, hipStream_t st) {
  const int nref = refill_blocks(fresh_cap_max, np_max, b.nsim);
  if (nref > 0 && storage == 0)
    hipLaunchKernelGGL(k_refill_boundary<0>, dim3(nref, b.nsim), dim3(256), 0, st, b);
  else if (nref > 0)
    hipLaunchKernelGGL(k_refill_boundary<1>, dim3(nref, b.nsim), dim3(256), 0, st, b);
  hipLaunchKernelGGL(k_moments_boundary, dim3(nblk), dim3(256), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_init_mask(const SimDev& s, hipStream_t st) {
  hipLaunchKernelGGL(k_init_mask, dim3(nblocks(s.N, 256)), dim3(256), 0, st, s);
  return hipGetLastError();
}

hipError_t launch_init_pops(const SimDev& s, void* pops, hipStream_t st) {
  if (s.storage == 0)
    hipLaunchKernelGGL(k_init_pops<0>, dim3(nblocks(s.N, 256)), dim3(256), 0, st, s, pops);
  else
    hipLaunchKernelGGL(k_init_pops<1>, dim3(nblocks(s.N, 256)), dim3(256), 0, st, s, pops);
  return hipGetLastError();
}

// rp: moments (rho plane, phi plane) of the current state, pops its
// populations; acc: 2 doubles, cleared before
hipError_t launch_mass(const SimDev& s, const float* rp, const void* pops, double* acc,
                       hipStream_t st) {
  unsigned nb = nblocks(s.N, 256);
  if (nb > 4096) nb = 4096;
  if (s.storage == 0)
    hipLaunchKernelGGL(k_mass<0>, dim3(nb), dim3(256), 0, st, s, rp, pops, acc);
  else
    hipLaunchKernelGGL(k_mass<1>, dim3(nb), dim3(256), 0, st, s, rp, pops, acc);
  return hipGetLastError();
}

hipError_t launch_zero_f64(double* p, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_f64, dim3(nblocks(n, 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

}  // namespace lbm
