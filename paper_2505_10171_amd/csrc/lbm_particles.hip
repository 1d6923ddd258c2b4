// lbm_particles.hip -- particle kernels of liblbm for gfx950: solid mask update
// and the DEM (contacts with sliding and rolling friction, velocity Verlet).  The
// refilling of fresh nodes, the links and the capillary force are in lbm_fluid.hip,
// whose launches they share.
#include <algorithm>

#include "launch_rules.h"
#include "lbm_device.h"

namespace lbm {

// ------------------------------------------------------------------ masks
// Particle bounding box: every node inside the sphere lies in it.
struct Box {
  int lo[3], w[3];
};
__device__ __forceinline__ Box particle_box(const SimDev& s, const double* X, double R) {
  Box b;
  const int L[3] = {s.nx, s.ny, s.nz};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = (int)floor(X[k] - R) - 1;
    b.w[k] = (int)floor(X[k] + R) + 1 - b.lo[k] + 1;
    if (b.w[k] > L[k]) {
      b.lo[k] = 0;
      b.w[k] = L[k];
    }
  }
  return b;
}

// Inside test: ((dx*dx)+(dy*dy))+(dz*dz) < R*R in FP64, rounded operation by
// operation (no contraction), d wrapped once into (-L/2, L/2].
__device__ __attribute__((noinline)) bool inside_sphere(int x, int y, int z, const double* X,
                                                        double R, int nx, int ny, int nz) {
#pragma clang fp contract(off)
  double dx = wrapd((double)x - X[0], (double)nx);
  double dy = wrapd((double)y - X[1], (double)ny);
  double dz = wrapd((double)z - X[2], (double)nz);
  double a = dx * dx;
  double b = dy * dy;
  double c = dz * dz;
  double d2 = (a + b) + c;
  return d2 < R * R;
}

// Pushed particles: the heads of their records, staged in the view buffer,
// into the records, whose present centre and radius the mask update releases.  A
// simulation that has failed (status flags) keeps its records; the mask update then
// finds every node as it is.
static_assert(2 * sizeof(DemView) >= sizeof(DevParticleHead), "the views hold the heads");
__global__ void k_push(SimDev s) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= s.np || s.counters[1] != 0u) return;
  DevParticle& P = s.P[p];
  const DevParticleHead h = ((const DevParticleHead*)s.view)[p];
  for (int d = 0; d < 3; ++d) P.xo[d] = P.x[d];
  P.Ro = P.R;
  *(DevParticleHead*)&P = h;
}

// Mask of the new positions, one grid row of blocks per particle p.  A node's new
// owner is the lowest particle inside which it lies.  With RELEASE, the nodes
// that belonged to p (old box) pass to their new owner or become fluid (fresh);
// the fluid nodes of the new box whose owner is p become p's.  Every node is
// written by one block only: by its old owner's, or, if it was fluid, by its new
// owner's; what another block may read there meanwhile (the new code, or the
// fresh mark) leaves that block's part unchanged, so the pass needs no claims in
// memory and no second and third kernel (one launch for three: 12 -> 5 us
// with one sphere of radius 4, 14 -> 6.6 with 20 of radius 5, 40 -> 34 with 500
// of radius 4).  But each block looks through all particles, so that boxes of many
// take the claims below; and the grid is sized by the largest sphere, so it is bounded
// (particle_blocks) and a block past both boxes of its own leaves before that (one
// sphere of radius 20 beside 400 of radius 3: 437 us without, 60 with).
constexpr int MASK_NEAR = 64;  // overlapping particles listed; more: all are tested
// STRIDE: the grid is bounded, the blocks take several turns (that loop takes 24 VGPRs
// and three waves per SIMD more: 97 -> 106 us with 500 spheres of radius 8)
template <bool RELEASE, bool STRIDE>
__global__ __launch_bounds__(256) void k_mask(Batch bt) {
  const int2 sp = batch_particle(bt, blockIdx.y);
  const SimDev& s = bt.tab[sp.x];
  const int p = sp.y, np = s.np;
  const DevParticle* PP = s.P;
  // the record's fields held in registers (the stores below may alias it)
  const int nx = s.nx, ny = s.ny, nz = s.nz;
  const double X[3] = {PP[p].x[0], PP[p].x[1], PP[p].x[2]}, R = PP[p].R;
  const double Xo[3] = {PP[p].xo[0], PP[p].xo[1], PP[p].xo[2]}, Ro = PP[p].Ro;
  GLB uint16_t* __restrict__ MASK = gp(s.mask);
  // this block's nodes of both boxes, 256 of each at a time
  const Box b = particle_box(s, X, R), bo = particle_box(s, Xo, Ro);
  auto vol = [](const Box& q) { return q.w[0] * q.w[1] * q.w[2]; };
  const int nodes = max(vol(b), RELEASE ? vol(bo) : 0);
  int k0 = (int)(blockIdx.x * blockDim.x);
  if (k0 >= nodes) return;
  auto node = [&](const Box& q, int& x, int& y, int& z) -> bool {
    const int k = k0 + (int)threadIdx.x;
    if (k >= vol(q)) return false;
    x = wrapi(q.lo[0] + k % q.w[0], nx);
    y = wrapi(q.lo[1] + (k / q.w[0]) % q.w[1], ny);
    z = wrapi(q.lo[2] + k / (q.w[0] * q.w[1]), nz);
    return true;
  };
  int x = 0, y = 0, z = 0, xo = 0, yo = 0, zo = 0;
  unsigned n = 0, no = 0;
  bool in = false, ino = false;
  uint16_t m = 0, mo = 0;
  // their mask codes: the first with the candidates' positions in flight
  auto load = [&]() {
    in = node(b, x, y, z);
    ino = RELEASE && node(bo, xo, yo, zo);
    n = in ? (unsigned)(x + nx * (y + ny * z)) : 0u;
    no = ino ? (unsigned)(xo + nx * (yo + ny * zo)) : 0u;
    m = at((const GLB uint16_t*)MASK, n);
    if (RELEASE) mo = at((const GLB uint16_t*)MASK, no);
  };
  load();
  // particles whose new sphere meets p's new or old one: a node inside both
  // spheres is nearer than both radii to both centres (the margin covers rounding)
  __shared__ int near[MASK_NEAR], n_near;
  if (threadIdx.x == 0) n_near = 0;
  __syncthreads();
  for (int q = threadIdx.x; q < np; q += blockDim.x) {
    if (q == p) continue;
    const double Xq[3] = {PP[q].x[0], PP[q].x[1], PP[q].x[2]}, Rq = PP[q].R;
    auto meets = [&](const double* C, double Rc) {
      const double dx = wrapd(Xq[0] - C[0], (double)nx), dy = wrapd(Xq[1] - C[1], (double)ny),
                   dz = wrapd(Xq[2] - C[2], (double)nz);
      const double lim = Rq + Rc + 1e-3;
      return dx * dx + dy * dy + dz * dz < lim * lim;
    };
    if (meets(X, R) || (RELEASE && meets(Xo, Ro))) {
      const int slot = atomicAdd(&n_near, 1);
      if (slot < MASK_NEAR) near[slot] = q;
    }
  }
  __syncthreads();
  const bool listed = n_near <= MASK_NEAR;
  const int tests = listed ? n_near : np;
  // the lowest particle that holds node (x, y, z), np if none
  auto owner = [&](int x, int y, int z) {
    int c = inside_sphere(x, y, z, X, R, nx, ny, nz) ? p : np;
    for (int u = 0; u < tests; ++u) {
      const int q = listed ? near[u] : u;
      if (q < c && q != p) {
        const double Xq[3] = {PP[q].x[0], PP[q].x[1], PP[q].x[2]};
        if (inside_sphere(x, y, z, Xq, PP[q].R, nx, ny, nz)) c = q;
      }
    }
    return c;
  };
  for (;;) {
    if (RELEASE) {
      const bool mine = ino && mo == (uint16_t)(2 + p);
      const int c = mine ? owner(xo, yo, zo) : p;
      const bool fresh = c == np;
      // the wave's fresh nodes take consecutive slots of the fresh list: one
      // atomic per wave (the list's order does not matter to the refill)
      const unsigned long long want = __ballot(fresh);
      if (want) {
        const int lane = (int)(threadIdx.x & 63), first = __ffsll((long long)want) - 1;
        uint32_t base0 = 0;
        if (lane == first) base0 = atomicAdd(&s.counters[bt.fc], (uint32_t)__popcll(want));
        base0 = (uint32_t)__shfl((int)base0, first, 64);
        if (fresh) {
          MASK[no] = FRESH_BIT;
          const uint32_t slot = base0 + (uint32_t)__popcll(want & ((1ull << lane) - 1ull));
          if (slot < s.fresh_cap) {
            s.fresh[slot] = no;
            s.fresh_own[slot] = (uint32_t)p;
          } else {
            atomicOr(&s.counters[1], (uint32_t)ST_FRESH_FULL);
          }
        }
      }
      if (mine && !fresh && c != p) MASK[no] = (uint16_t)(2 + c);
    }
    if (in && m == 0 && owner(x, y, z) == p) MASK[n] = (uint16_t)(2 + p);
    k0 += (int)(gridDim.x * blockDim.x);
    if (!STRIDE || k0 >= nodes) return;
    load();
  }
}

// The same by claims in memory, three kernels whose time does not grow with the number
// of particles per block: for boxes of many (mask_by_search).
// claim: lowest particle index inside which a node lies (new positions)
__global__ void k_claim(Batch bt) {
  const int2 sp = batch_particle(bt, blockIdx.y);
  const SimDev& s = bt.tab[sp.x];
  const int p = sp.y;
  const DevParticle& P = s.P[p];
  const Box b = particle_box(s, P.x, P.R);
  const int vol = b.w[0] * b.w[1] * b.w[2];
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < vol; k += gridDim.x * blockDim.x) {
    const int ix = k % b.w[0], iy = (k / b.w[0]) % b.w[1], iz = k / (b.w[0] * b.w[1]);
    const int x = wrapi(b.lo[0] + ix, s.nx), y = wrapi(b.lo[1] + iy, s.ny),
              z = wrapi(b.lo[2] + iz, s.nz);
    if (static_wall(s, x, y, z)) continue;
    if (inside_sphere(x, y, z, P.x, P.R, s.nx, s.ny, s.nz)) {
      const long long n = (long long)x + (long long)s.nx * ((long long)y + (long long)s.ny * z);
      atomicMin(&s.claim[n], (uint32_t)p);
    }
  }
}

// release: nodes that belonged to p (old box) become fluid (fresh) or pass to
// the particle that claims them now.  Each such node is visited once (by p).
__global__ void k_release(Batch bt) {
  const int2 sp = batch_particle(bt, blockIdx.y);
  const SimDev& s = bt.tab[sp.x];
  const int p = sp.y;
  const DevParticle& P = s.P[p];
  double Xo[3] = {P.xo[0], P.xo[1], P.xo[2]};
  const Box b = particle_box(s, Xo, P.Ro);
  const int vol = b.w[0] * b.w[1] * b.w[2];
  // the record's fields held in registers (the stores below may alias it)
  const int nx = s.nx, ny = s.ny, nz = s.nz;
  GLB uint16_t* __restrict__ MASK = gp(s.mask);
  const GLB uint32_t* __restrict__ CLAIM = gp((const uint32_t*)s.claim);
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < vol; k += gridDim.x * blockDim.x) {
    const int ix = k % b.w[0], iy = (k / b.w[0]) % b.w[1], iz = k / (b.w[0] * b.w[1]);
    const int x = wrapi(b.lo[0] + ix, nx), y = wrapi(b.lo[1] + iy, ny), z = wrapi(b.lo[2] + iz, nz);
    const unsigned n = (unsigned)(x + nx * (y + ny * z));
    // mask and claim in one round trip
    const uint16_t m = at((const GLB uint16_t*)MASK, n);
    const uint32_t c = at(CLAIM, n);
    const bool mine = m == (uint16_t)(2 + p);
    const bool fresh = mine && c == 0xFFFFFFFFu;
    // the wave's fresh nodes take consecutive slots of the fresh list: one
    // atomic per wave (the list's order does not matter to the refill)
    const unsigned long long want = __ballot(fresh);
    uint32_t base0 = 0;
    const int lane = (int)(threadIdx.x & 63);
    const int first = want ? __ffsll((long long)want) - 1 : 0;
    if (want && lane == first) base0 = atomicAdd(&s.counters[bt.fc], (uint32_t)__popcll(want));
    base0 = (uint32_t)__shfl((int)base0, first, 64);
    if (!mine) continue;
    if (fresh) {
      MASK[n] = FRESH_BIT;
      const uint32_t slot = base0 + (uint32_t)__popcll(want & ((1ull << lane) - 1ull));
      if (slot < s.fresh_cap) {
        s.fresh[slot] = n;
        s.fresh_own[slot] = (uint32_t)p;
      } else {
        atomicOr(&s.counters[1], (uint32_t)ST_FRESH_FULL);
      }
    } else if (c != (uint32_t)p) {
      MASK[n] = (uint16_t)(2 + c);
    }
  }
}

// cover: nodes claimed by p become p's solid nodes; claims are cleared
__global__ void k_cover(Batch bt) {
  const int2 sp = batch_particle(bt, blockIdx.y);
  const SimDev& s = bt.tab[sp.x];
  const int p = sp.y;
  const DevParticle& P = s.P[p];
  const Box b = particle_box(s, P.x, P.R);
  const int vol = b.w[0] * b.w[1] * b.w[2];
  // the record's fields held in registers (the stores below may alias it)
  const int nx = s.nx, ny = s.ny, nz = s.nz;
  GLB uint16_t* __restrict__ MASK = gp(s.mask);
  GLB uint32_t* __restrict__ CLAIM = gp(s.claim);
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < vol; k += gridDim.x * blockDim.x) {
    const int ix = k % b.w[0], iy = (k / b.w[0]) % b.w[1], iz = k / (b.w[0] * b.w[1]);
    const int x = wrapi(b.lo[0] + ix, nx), y = wrapi(b.lo[1] + iy, ny), z = wrapi(b.lo[2] + iz, nz);
    const unsigned n = (unsigned)(x + nx * (y + ny * z));
    if (at((const GLB uint32_t*)CLAIM, n) == (uint32_t)p) {
      MASK[n] = (uint16_t)(2 + p);
      CLAIM[n] = 0xFFFFFFFFu;
    }
  }
}

// -------------------------------------------------------------------- DEM
__device__ inline void cross3(const double* a, const double* b, double* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ inline double dot3(const double* a, const double* b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// spring with a Coulomb cap (sliding friction eqs.; rolling uses the same rule)
__device__ inline void capped_spring(double k, double gam, double cap, double* xi, const double* v,
                                     double dt, double* F) {
  double F0[3];
  for (int d = 0; d < 3; ++d) F0[d] = -k * xi[d] - gam * v[d];
  const double f0 = sqrt(dot3(F0, F0));
  if (f0 <= cap) {
    for (int d = 0; d < 3; ++d) {
      F[d] = F0[d];
      xi[d] += v[d] * dt;
    }
  } else {
    for (int d = 0; d < 3; ++d) F[d] = cap * F0[d] / f0;
    for (int d = 0; d < 3; ++d) xi[d] = (k > 0.0) ? -(F[d] + gam * v[d]) / k : 0.0;
  }
}

__device__ inline void rel_vec(const SimDev& s, const double* a, const double* b, double* d) {
  d[0] = wrapd(a[0] - b[0], (double)s.nx);
  d[1] = wrapd(a[1] - b[1], (double)s.ny);
  d[2] = wrapd(a[2] - b[2], (double)s.nz);
}

// The unit quaternion of the rotation vector th; false for no rotation.
__device__ __forceinline__ bool quat_of(const double* th, double* dq) {
  const double a = sqrt(dot3(th, th));
  if (!(a > 0.0)) return false;
  const double h = 0.5 * a, sh = sin(h) / a;
  dq[0] = cos(h);
  for (int k = 0; k < 3; ++k) dq[1 + k] = th[k] * sh;
  return true;
}
// q <- dq q, normalised
__device__ __forceinline__ void quat_turn(double* q, const double* dq) {
  double r[4] = {dq[0] * q[0] - dq[1] * q[1] - dq[2] * q[2] - dq[3] * q[3],
                 dq[0] * q[1] + dq[1] * q[0] + dq[2] * q[3] - dq[3] * q[2],
                 dq[0] * q[2] - dq[1] * q[3] + dq[2] * q[0] + dq[3] * q[1],
                 dq[0] * q[3] + dq[1] * q[2] - dq[2] * q[1] + dq[3] * q[0]};
  const double nq = sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + r[3] * r[3]);
  for (int k = 0; k < 4; ++k) q[k] = r[k] / nq;
}
__device__ void quat_rotate(double* q, const double* th) {
  double dq[4];
  if (quat_of(th, dq)) quat_turn(q, dq);
}

// Contact geometry of a particle at x with the static wall: partner -1 is the
// plane's top face (normal +z, surface z = 1/2) or the tube (the cylinder
// r = R_t, normal from the wall to the centre, towards the axis), -2 the
// plane's underside seen through the periodic z direction (normal -z, surface
// z = nz - 1/2).  delta is the overlap with the mechanical radius Rc; false if
// the simulation has no such wall face.
__device__ __forceinline__ bool wall_geom(const SimDev& s, const double* x, double Rc, int partner,
                                          double& delta, double* nh) {
  nh[0] = nh[1] = nh[2] = 0.0;
  if (s.has_wall == 3 && partner <= -3) {
    // box -3 - b of a textured wall: its nearest surface point; no contact
    // while the centre is inside the box
    const int b = -3 - partner;
    if (b >= s.n_boxes) return false;
    const int* B = s.boxes[b];
    double d[3];
    for (int k = 0; k < 3; ++k) {
      const double lo = B[k] - 0.5, hi = B[3 + k] + 0.5;
      d[k] = x[k] - (x[k] < lo ? lo : (x[k] > hi ? hi : x[k]));
    }
    const double dn = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    if (!(dn > 0.0)) {
      delta = -1.0;
      return true;
    }
    for (int k = 0; k < 3; ++k) nh[k] = d[k] / dn;
    delta = Rc - dn;
    return true;
  }
  if (s.has_wall == 1 || s.has_wall == 3) {
    if (partner == -1) {
      delta = Rc - (x[2] - 0.5);
      nh[2] = 1.0;
    } else {
      delta = Rc - (((double)s.nz - 0.5) - x[2]);
      nh[2] = -1.0;
    }
    return true;
  }
  if (s.has_wall == 2 && partner == -1) {
    const double dy = x[1] - s.tube_yc, dz = x[2] - s.tube_zc;
    const double r = sqrt(dy * dy + dz * dz);
    if (r > 0.0) {
      nh[1] = -dy / r;
      nh[2] = -dz / r;
    }
    delta = Rc - (sqrt(s.tube_R2) - r);
    return true;
  }
  return false;
}

// The pair tests of the DEM's candidate search spread over the GPU (boxes with
// up to 32 MAXNB particles): the tests of particle i against partners
// 32 w .. 32 w + 31 (centre distance, minimum image, below Rc_i + Rc_j + skin)
// form the hit mask stored as word w of row i of the candidate-list buffer
// (MAXNB words per particle), which k_dem_setup turns into the candidate list.
// Positions and contact radii are those the step starts from.  Grid
// (ceil(32 np_max ceil(np_max / 32) / 256), nsim).
__global__ __launch_bounds__(256) void k_dem_search(Batch bt) {
  // one thread per (particle i, partner j): half a wave takes the 32 partners
  // of one hit word and a ballot forms the word (one round of loads)
  const SimDev& s = bt.tab[blockIdx.y];
  const int np = s.np;
  const int nw = (np + 31) / 32;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long r = t / 32;  // word index (i, w)
  const int u = (int)(t & 31);
  const bool inr = r < (long long)np * nw;
  const int i = inr ? (int)(r / nw) : 0, w = inr ? (int)(r % nw) : 0;
  const int j = 32 * w + u;
  bool hit = false;
  if (inr && j < np && j != i) {
    const DevParticle* PP = s.P;
    const double skin = 1.5;
    const double xi[3] = {PP[i].x[0], PP[i].x[1], PP[i].x[2]};
    const double xj[3] = {PP[j].x[0], PP[j].x[1], PP[j].x[2]};
    double dx[3];
    rel_vec(s, xi, xj, dx);
    const double lim = PP[i].Rc + PP[j].Rc + skin;
    hit = dot3(dx, dx) < lim * lim;
  }
  const unsigned long long b = __ballot(hit);
  const uint32_t word = (uint32_t)(b >> (threadIdx.x & 32));
  if (inr && u == 0) ((uint32_t*)s.nb)[(long long)i * MAXNB + w] = word;
}

// ---------------------------------------------- DEM over the whole GPU
// Boxes with more particles than the LDS variants hold well: each lattice step
// runs k_dem_setup (one thread per particle: fluid force mean, candidate list,
// predictor of the first sub-step), then per DEM sub-step one launch of
// k_dem_sub with a wave per particle: lane q < MAXNB evaluates the contact
// with candidate q, lanes MAXNB and MAXNB + 1 the wall and its underside; the
// contact forces are summed over the wave, and lane 0 applies the corrector and
// the predictor of the next sub-step.  The positions and predicted velocities
// the contacts read are the view of the sub-step (two buffers, so that a
// sub-step's predictor does not overwrite what its contacts still read), and
// a particle's contact table is written only by its own wave.

// Predictor of a sub-step (velocity Verlet, held fluid force, contact force of
// the last sub-step): new centre, orientation and predicted velocities, into
// the record and the view.
__device__ void dem_predict(const SimDev& s, DevParticle& P, DemView& v, double dt) {
  // every field read before the first store (a load behind a store to the
  // record would wait for it)
  const int kin = P.kin;
  const double mass = P.mass, inertia = P.inertia;
  const int nx = s.nx, ny = s.ny, nz = s.nz, has_wall = s.has_wall, open_x = s.open_x;
  double Ff[3], Fcp[3], Tf[3], Tcp[3], X[3], V[3], W[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    Ff[d] = P.Ff[d];
    Fcp[d] = P.Fcp[d];
    Tf[d] = P.Tf[d];
    Tcp[d] = P.Tcp[d];
    X[d] = P.x[d];
    V[d] = P.v[d];
    W[d] = P.w[d];
  }
  double th[3], ao[3], bo[3], vp[3], wp[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (kin) {
      ao[d] = 0.0;
      bo[d] = 0.0;
    } else {
      ao[d] = (Ff[d] + Fcp[d]) / mass;
      bo[d] = (Tf[d] + Tcp[d]) / inertia;
    }
    X[d] += V[d] * dt + 0.5 * ao[d] * dt * dt;
    th[d] = W[d] * dt + 0.5 * bo[d] * dt * dt;
    vp[d] = V[d] + ao[d] * dt;
    wp[d] = W[d] + bo[d] * dt;
  }
  const double L[3] = {(double)nx, (double)ny, (double)nz};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if ((d == 2 && has_wall) || (d == 0 && open_x)) continue;
    if (X[d] >= L[d])
      X[d] -= L[d];
    else if (X[d] < 0.0)
      X[d] += L[d];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    P.ao[d] = ao[d];
    P.bo[d] = bo[d];
    P.x[d] = X[d];
    P.vp[d] = vp[d];
    P.wp[d] = wp[d];
    v.x[d] = X[d];
    v.vp[d] = vp[d];
    v.wp[d] = wp[d];
  }
  quat_rotate(P.q, th);
}

// Pair candidates of every particle within Rc_i + Rc_j + skin by a full loop
// (boxes too large for the hit masks of k_dem_search), ascending, as lists
// of the candidate-list buffer (-1 after the last).
__global__ __launch_bounds__(64) void k_dem_lists(Batch bt, int np_rows) {
  const int r = blockIdx.x * 64 + threadIdx.x;
  if (r >= np_rows) return;
  const int2 sp = batch_particle(bt, r);
  const SimDev& s = bt.tab[sp.x];
  const int i = sp.y, np = s.np;
  const DevParticle* PP = s.P;
  const double skin = 1.5;
  const double xi[3] = {PP[i].x[0], PP[i].x[1], PP[i].x[2]};
  const double Rci = PP[i].Rc;
  int* nb = s.nb + (long long)i * MAXNB;
  int c = 0;
  for (int j = 0; j < np; ++j) {
    if (j == i) continue;
    const double xj[3] = {PP[j].x[0], PP[j].x[1], PP[j].x[2]};
    double dx[3];
    rel_vec(s, xi, xj, dx);
    const double lim = Rci + PP[j].Rc + skin;
    if (dot3(dx, dx) < lim * lim) {
      if (c < MAXNB)
        nb[c++] = j;
      else
        atomicOr(&s.counters[1], (uint32_t)ST_CONTACT_FULL);
    }
  }
  if (c < MAXNB) nb[c] = -1;
}

// Per-step set-up of one particle (thread): held fluid force and torque (mean
// of this and the previous lattice step) and gravity, its candidate list (from
// k_dem_search's hit masks when `masks`, else the lists of k_dem_lists), the
// springs of partners that left it freed, the predictor of the first
// sub-step into view 0, and the constant view fields in both views.
__global__ __launch_bounds__(64) void k_dem_setup(Batch bt, int np_rows, int masks) {
  const int r = blockIdx.x * 64 + threadIdx.x;
  if (r >= np_rows) return;
  const int2 sp = batch_particle(bt, r);
  const SimDev& s = bt.tab[sp.x];
  const int i = sp.y, np = s.np;
  DevParticle& P = s.P[i];
  // every field read before the first store (a load behind a store to the
  // record waits for it: one round trip per component otherwise)
  double Fca[3], Tca[3], Fh[3], Th[3], Ffp[3], Tfp[3], X[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    Fca[d] = P.Fca[d];
    Tca[d] = P.Tca[d];
    Fh[d] = P.Fh[d];
    Th[d] = P.Th[d];
    Ffp[d] = P.Ffp[d];
    Tfp[d] = P.Tfp[d];
    X[d] = P.x[d];
  }
  const int havep = P.havep;
  const double g_p = P.g_p, R = P.R;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    P.Fcap[d] = Fca[d];
    P.Tcap[d] = Tca[d];
    P.Fca[d] = 0.0;
    P.Tca[d] = 0.0;
    const double fc = Fh[d] + Fca[d], tc = Th[d] + Tca[d];
    const double fp = havep ? Ffp[d] : fc, tp = havep ? Tfp[d] : tc;
    P.Ff[d] = 0.5 * (fc + fp) - (d == 2 ? g_p : 0.0);
    P.Tf[d] = 0.5 * (tc + tp);
    P.Ffp[d] = fc;
    P.Tfp[d] = tc;
    P.Fh_last[d] = Fh[d];
    P.Th_last[d] = Th[d];
    P.Fh[d] = 0.0;
    P.Th[d] = 0.0;
    P.xo[d] = X[d];
    P.Facc[d] = 0.0;
    P.Tacc[d] = 0.0;
  }
  P.Ro = R;
  P.havep = 1;
  P.cap_on = 0;
  // the step counter advances here (the sub-steps' history record takes the
  // value before it)
  if (i == 0) {
    *s.step_counter += 1;
    s.counters[0] = 0u;  // the fresh list, which the mask update fills again
  }
  int* nb = s.nb + (long long)i * MAXNB;
  int c = 0;
  // membership of a partner in this step's candidate list, from registers (a
  // re-read of the list just written would wait for its stores, per slot)
  uint32_t words[MAXNB];
  int lst[MAXNB];
  int jlast = -1;  // masks: the last partner the list took (it is capped at MAXNB)
  if (masks) {
    // row i holds one hit mask per 32 partners: all words read before the
    // list overwrites them
    const int nw = (np + 31) / 32;
#pragma unroll
    for (int w = 0; w < MAXNB; ++w) words[w] = w < nw ? ((const uint32_t*)nb)[w] : 0u;
#pragma unroll
    for (int w = 0; w < MAXNB; ++w) {
      uint32_t hit = words[w];
      while (hit) {
        const int j = 32 * w + __builtin_ctz(hit);
        hit &= hit - 1;
        if (c < MAXNB) {
          nb[c++] = j;
          jlast = j;
        } else {
          atomicOr(&s.counters[1], (uint32_t)ST_CONTACT_FULL);
        }
      }
    }
    if (c < MAXNB) nb[c] = -1;
  } else {
    // the list as k_dem_lists wrote it: entries up to the first negative one
    bool end = false;
#pragma unroll
    for (int w = 0; w < MAXNB; ++w) {
      lst[w] = nb[w];
      end |= lst[w] < 0;
      c += end ? 0 : 1;
    }
  }
  auto listed = [&](int pt) {
    bool r = false;
    if (masks) {
      // the list holds the set bits in increasing order up to jlast
#pragma unroll
      for (int w = 0; w < MAXNB; ++w) r |= (w == (pt >> 5)) && ((words[w] >> (pt & 31)) & 1u);
      return r && pt <= jlast;
    }
#pragma unroll
    for (int w = 0; w < MAXNB; ++w) r |= w < c && lst[w] == pt;
    return r;
  };
  // free pair springs whose partner is out of range
  Contact* tab = s.ct + (long long)i * MAXC;
  for (int k = 0; k < MAXC; ++k) {
    const int pt = tab[k].partner;
    if (pt < 0) continue;
    if (!listed(pt)) tab[k].partner = -100;
  }
  DemView* V0 = s.view;
  DemView* V1 = s.view + np;
  V0[i].Rc = V1[i].Rc = P.Rc;
  V0[i].mu_s = V1[i].mu_s = P.mu_s;
  V0[i].mu_r = V1[i].mu_r = P.mu_r;
  dem_predict(s, P, V0[i], 1.0 / s.n_sub);
}

// The contact force of one active contact whose spring slot sl is known
// (normal spring-dashpot, sliding and rolling friction after Luding's model as
// the paper describes it).
__device__ __forceinline__ void contact_force(const SimDev& s, Contact* sl, double delta,
                                              const double* nh, const double* vi,
                                              const double* wi, const double* vj,
                                              const double* wj, double Rci, double Rcj,
                                              const double* armj, double mu, double mur,
                                              double dt, double* Fo, double* To) {
  double vrel[3];
  for (int d = 0; d < 3; ++d) vrel[d] = vi[d] - vj[d];
  const double ddot = -dot3(vrel, nh);
  const double Fn = s.kn * delta + s.gn * ddot;
  double ri[3], rj[3], t1[3], t2[3], vc[3];
  for (int d = 0; d < 3; ++d) ri[d] = -(Rci - 0.5 * delta) * nh[d];
  for (int d = 0; d < 3; ++d) rj[d] = ri[d] + armj[d];
  cross3(wi, ri, t1);
  cross3(wj, rj, t2);
  for (int d = 0; d < 3; ++d) vc[d] = vrel[d] + t1[d] - t2[d];
  const double vn = dot3(vc, nh);
  double vt[3];
  for (int d = 0; d < 3; ++d) vt[d] = vc[d] - vn * nh[d];
  double xt[3], xr[3];
  for (int d = 0; d < 3; ++d) {
    xt[d] = sl->xt[d];
    xr[d] = sl->xr[d];
  }
  double xn = dot3(xt, nh);
  for (int d = 0; d < 3; ++d) xt[d] -= xn * nh[d];
  xn = dot3(xr, nh);
  for (int d = 0; d < 3; ++d) xr[d] -= xn * nh[d];
  const double Fcap = mu * (Fn > 0.0 ? Fn : 0.0);
  double Ft[3];
  capped_spring(s.kt, s.gt, Fcap, xt, vt, dt, Ft);
  const double ap = (Rcj > 0.0) ? Rci * Rcj / (Rci + Rcj) : Rci;
  double nwi[3], nwj[3], vr[3], Fr[3];
  cross3(nh, wi, nwi);
  cross3(nh, wj, nwj);
  for (int d = 0; d < 3; ++d) vr[d] = -ap * (nwi[d] - nwj[d]);
  const double Rcap = mur * (Fn > 0.0 ? Fn : 0.0);
  capped_spring(s.kr, s.gr, Rcap, xr, vr, dt, Fr);
  for (int d = 0; d < 3; ++d) {
    sl->xt[d] = xt[d];
    sl->xr[d] = xr[d];
  }
  double Tt[3], Tr[3];
  cross3(ri, Ft, Tt);
  cross3(nh, Fr, Tr);
  for (int d = 0; d < 3; ++d) {
    Fo[d] = Fn * nh[d] + Ft[d];
    To[d] = Tt[d] + ap * Tr[d];
  }
}

// One DEM sub-step of every particle: a wave per particle (four per block).
__global__ __launch_bounds__(256) void k_dem_sub(Batch bt, int np_rows, int sub) {
  // the particle row is the same for the whole wave; declared uniform, it lets
  // the simulation record and the particle's own data be read by scalar loads
  const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + ((int)threadIdx.x >> 6));
  const int lane = (int)threadIdx.x & 63;
  if (r >= np_rows) return;  // the whole wave
  const int2 sp = batch_particle(bt, r);
  const SimDev& s = bt.tab[sp.x];
  if (sub >= s.n_sub) return;
  const int i = sp.y, np = s.np;
  const double dt = 1.0 / s.n_sub;
  const DemView* V = s.view + (sub & 1) * np;
  const DemView& me = V[i];
  Contact* tab = s.ct + (long long)i * MAXC;
  int ids[MAXC];
#pragma unroll
  for (int k = 0; k < MAXC; ++k) ids[k] = tab[k].partner;
  // this lane's partner: candidate `lane`, or the wall (-1) or its underside (-2)
  int partner = -100;
  // lanes past the list's end stay idle (a list shorter than MAXNB ends at -1):
  // a lane is past it when a lower lane holds a negative entry (one ballot)
  const int j = lane < MAXNB ? s.nb[(long long)i * MAXNB + lane] : 0;
  const unsigned long long neg = __ballot(j < 0);
  if (lane < MAXNB) {
    partner = (j >= 0 && (neg & ((1ull << lane) - 1ull)) == 0ull) ? j : -100;
  } else if (lane == MAXNB && s.has_wall) {
    partner = -1;
  } else if (lane == MAXNB + 1 && s.has_wall) {
    partner = -2;
  } else if (lane >= MAXNB + 2 && s.has_wall == 3 && lane - (MAXNB + 2) < s.n_boxes) {
    partner = -3 - (lane - (MAXNB + 2));  // a box of the textured wall
  }
  // the partner's velocities by value (a pointer that may also point at a
  // local array of zeros puts that array in scratch and makes the loads generic)
  double delta = 0.0, nh[3] = {0.0, 0.0, 0.0}, arm[3] = {0.0, 0.0, 0.0};
  double vj[3] = {0.0, 0.0, 0.0}, wj[3] = {0.0, 0.0, 0.0};
  double Rcj = 0.0, mu = me.mu_s, mur = me.mu_r;
  if (partner >= 0) {
    const DemView& pj = V[partner];
    rel_vec(s, me.x, pj.x, arm);  // X_i - X_j, min image
    const double dist = sqrt(dot3(arm, arm));
    Rcj = pj.Rc;
    delta = me.Rc + Rcj - dist;
    if (dist > 0.0)
      for (int d = 0; d < 3; ++d) nh[d] = arm[d] / dist;
    for (int d = 0; d < 3; ++d) {
      vj[d] = pj.vp[d];
      wj[d] = pj.wp[d];
    }
    mu = 0.5 * (me.mu_s + pj.mu_s);
    mur = 0.5 * (me.mu_r + pj.mu_r);
  } else if (partner != -100) {
    if (!wall_geom(s, me.x, me.Rc, partner, delta, nh)) partner = -100;
  }
  const bool has = partner != -100;
  const bool active = has && delta > 0.0;
  int found = -1, nfree = 0;
#pragma unroll
  for (int k = MAXC - 1; k >= 0; --k)
    if (has && ids[k] == partner) found = k;
  // new contacts take the free slots in lane order (free before this pass)
  const unsigned long long need = __ballot(active && found < 0);
  const int rank = __popcll(need & ((1ull << lane) - 1ull));
  int slot = found;
  if (active && found < 0) {
    slot = -1;
#pragma unroll
    for (int k = 0; k < MAXC; ++k)
      if (ids[k] == -100) {
        if (nfree == rank) slot = k;
        ++nfree;
      }
    if (slot < 0) {
      atomicOr(&s.counters[1], (uint32_t)ST_CONTACT_FULL);
    } else {
      tab[slot].partner = partner;
      for (int d = 0; d < 3; ++d) tab[slot].xt[d] = tab[slot].xr[d] = 0.0;
    }
  }
  double acc[6] = {0, 0, 0, 0, 0, 0};
  if (active && slot >= 0) {
    double Fo[3], To[3];
    contact_force(s, &tab[slot], delta, nh, me.vp, me.wp, vj, wj, me.Rc, Rcj, arm, mu, mur, dt,
                  Fo, To);
    for (int d = 0; d < 3; ++d) {
      acc[d] = Fo[d];
      acc[3 + d] = To[d];
    }
  } else if (has && !active && found >= 0) {
    tab[found].partner = -100;  // the contact ended: its springs are released
  }
#pragma unroll
  for (int c = 0; c < 6; ++c)
    for (int off = 32; off > 0; off >>= 1) acc[c] += __shfl_xor(acc[c], off, 64);
  if (lane != 0) return;
  DevParticle& P = s.P[i];
  // every field read before the first store (a load behind a store to the
  // record would wait for it)
  const int kin = P.kin;
  const double mass = P.mass, inertia = P.inertia;
  double Ff[3], Tf[3], ao[3], bo[3], Vv[3], Ww[3], Fa[3], Ta[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    Ff[d] = P.Ff[d];
    Tf[d] = P.Tf[d];
    ao[d] = P.ao[d];
    bo[d] = P.bo[d];
    Vv[d] = P.v[d];
    Ww[d] = P.w[d];
    Fa[d] = P.Facc[d];
    Ta[d] = P.Tacc[d];
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (!kin) {
      const double an = (Ff[d] + acc[d]) / mass;
      const double bn = (Tf[d] + acc[3 + d]) / inertia;
      P.v[d] = Vv[d] + 0.5 * (ao[d] + an) * dt;
      P.w[d] = Ww[d] + 0.5 * (bo[d] + bn) * dt;
    }
    P.Fcp[d] = acc[d];
    P.Tcp[d] = acc[3 + d];
    P.Facc[d] = Fa[d] + acc[d];
    P.Tacc[d] = Ta[d] + acc[3 + d];
  }
  if (sub + 1 < s.n_sub) {
    dem_predict(s, P, s.view[((sub + 1) & 1) * np + i], dt);
    return;
  }
  // the last sub-step: contact means and the history record
  for (int d = 0; d < 3; ++d) {
    P.Fcon[d] = P.Facc[d] / s.n_sub;
    P.Tcon[d] = P.Tacc[d] / s.n_sub;
  }
  if (near_open_end(s, P.x[0], P.R)) atomicOr(&s.counters[1], (uint32_t)ST_OPEN_END);
  if (s.hist_cap > 0) {
    const unsigned long long step = *s.step_counter - 1;  // advanced by k_dem_setup
    double* h = s.hist + ((long long)(step % (unsigned long long)s.hist_cap) * np + i) *
                             LBM_HIST_DOUBLES_DEV;
    for (int d = 0; d < 3; ++d) {
      h[d] = P.Fh_last[d];
      h[3 + d] = P.Th_last[d];
      h[6 + d] = P.Fcap[d];
      h[9 + d] = P.Tcap[d];
      h[12 + d] = P.Fcon[d];
      h[15 + d] = P.Tcon[d];
      h[18 + d] = P.x[d];
      h[21 + d] = P.v[d];
      h[24 + d] = P.w[d];
    }
  }
}

// Boxes with few particles: one workgroup per simulation, 16 lanes per
// particle, the whole lattice step in one launch.  Fluid forces (momentum
// exchange + capillary) are held over n_sub velocity-Verlet sub-steps; contacts
// are evaluated at the new positions with the predicted velocities; gravity is
// the downward g_p.
//
// The step is a serial chain of FP64 arithmetic, so its length is instructions,
// not data: lanes 0-2 integrate the three components of the translation and
// lanes 3-5 those of the rotation (a division each, not six), a lane takes one
// wall face or candidate (ten wall partners of a textured wall at once), and
// the state stays in registers over the sub-steps.  LDS holds what others read:
// the views (two, so that a sub-step takes one barrier), the spring table and
// the candidate lists.  With a thread per particle and everything in LDS it took
// 22 us for one sphere, 33 for 20 and 67 for six on a wall of eight boxes.
constexpr int DEM_LANES = 16;   // per particle; as many as contact slots
constexpr int DEM_SMALL = 48;   // particles of a box that take this kernel (768 threads)
constexpr int DEM_ITEMS = 2 + 8 + MAXNB;  // wall faces, boxes, candidates
static_assert(DEM_LANES == MAXC, "a lane per contact slot");
struct DemRow {
  DemView view[2];
  Contact ct[MAXC];
  int nb[MAXNB];
  int8_t slot[(DEM_ITEMS + 7) / 8 * 8];  // spring slot of each item, -1 none
};
__global__ __launch_bounds__(DEM_SMALL * DEM_LANES) void k_dem(Batch bt) {
  const SimDev& s = bt.tab[blockIdx.x];
  if (s.np == 0) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char dem_lds[];
  DemRow* const rows = (DemRow*)dem_lds;
  const int np = s.np;
  const int i = (int)threadIdx.x / DEM_LANES, l = (int)threadIdx.x % DEM_LANES;
  const bool on = i < np;  // the same for a particle's 16 lanes
  const unsigned below = (1u << l) - 1u;
  // the 16 lanes' bits of a ballot (every lane of the wave calls it)
  auto group = [&](bool p) {
    return (unsigned)(__ballot(p) >> (threadIdx.x & 48u)) & 0xffffu;
  };
  const int n_sub = s.n_sub, has_wall = s.has_wall, open_x = s.open_x;
  const double dt = 1.0 / n_sub;
  DevParticle& P = s.P[on ? i : 0];
  DemRow& me = rows[on ? i : 0];
  // ---- loads: this lane's component (translation 0-2, rotation 3-5; the
  // record keeps each pair of vectors side by side) and its contact slot
  const int c = l < 6 ? l : 0, d = c % 3;
  const bool rot = c >= 3;
  const int kin = P.kin, havep = P.havep;
  const double M = rot ? P.inertia : P.mass;
  double X = P.x[d], V = (&P.v[0])[c], C = (&P.Fcp[0])[c];
  const double Fh = (&P.Fh[0])[c], Fca = (&P.Fca[0])[c], Fp = (&P.Ffp[0])[c];
  const double g_p = P.g_p, R = P.R, Rc = P.Rc, mu_s = P.mu_s, mu_r = P.mu_r;
  double q[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = P.q[k];
  const Contact mine = s.ct[(long long)(on ? i : 0) * MAXC + l];
  const unsigned long long step = *s.step_counter;
  const double X0 = X;
  // fluid force or torque: the mean of this and the previous lattice step (the
  // averaging of the Verlet update over the previous and current step)
  const double fc = Fh + Fca;
  double F = 0.5 * (fc + (havep ? Fp : fc));
  if (c == 2) F -= g_p;
  if (on) {
    me.ct[l] = mine;
    for (int k = l; k < DEM_ITEMS; k += DEM_LANES) me.slot[k] = -1;
    if (l < 3) me.view[0].x[l] = X;
    if (l < 2) {
      me.view[l].Rc = Rc;
      me.view[l].mu_s = mu_s;
      me.view[l].mu_r = mu_r;
    }
  }
  __syncthreads();
  // ---- pair candidates within Rc_i + Rc_j + skin (ascending index)
  const double skin = 1.5;
  int cnt = 0;
  for (int j0 = 0; j0 < np; j0 += DEM_LANES) {
    const int j = j0 + l;
    bool hit = false;
    if (on && j < np && j != i) {
      double dx[3];
      rel_vec(s, me.view[0].x, rows[j].view[0].x, dx);
      const double lim = Rc + rows[j].view[0].Rc + skin;
      hit = dot3(dx, dx) < lim * lim;
    }
    const unsigned hits = group(hit);
    const int pos = cnt + __popc(hits & below);
    if (hit) {
      if (pos < MAXNB)
        me.nb[pos] = j;
      else
        atomicOr(&s.counters[1], (uint32_t)ST_CONTACT_FULL);
    }
    cnt += __popc(hits);
  }
  cnt = min(cnt, MAXNB);
  __syncthreads();
  // ---- items: the wall faces and boxes, then the candidates.  Each spring finds
  // its item; pair springs whose partner is out of range are freed
  const int nw = has_wall == 0 ? 0 : has_wall == 2 ? 1 : 2 + (has_wall == 3 ? s.n_boxes : 0);
  const int items = on ? nw + cnt : 0;
  bool held = on && mine.partner != -100;
  if (held) {
    int it = -1;
    if (mine.partner < 0) {
      it = -1 - mine.partner;
    } else {
      for (int k = 0; k < cnt; ++k)
        if (me.nb[k] == mine.partner) it = nw + k;
    }
    if (it >= 0) {
      me.slot[it] = (int8_t)l;
    } else {
      me.ct[l].partner = -100;
      held = false;
    }
  }
  unsigned used = group(held);
  __syncthreads();
  double acc_mean = 0.0, A = 0.0, th[3] = {0.0, 0.0, 0.0};
  for (int sub = 0; sub < n_sub; ++sub) {
    // predictor: new centre, orientation and predicted velocities
    DemView& vw = me.view[sub & 1];
    {
      A = kin ? 0.0 : (F + C) / M;
      const double move = V * dt + 0.5 * A * dt * dt;
      const double vp = V + A * dt;
      X += move;
      const double Ld = d == 0 ? (double)s.nx : d == 1 ? (double)s.ny : (double)s.nz;
      if (!((d == 2 && has_wall) || (d == 0 && open_x))) {
        if (X >= Ld)
          X -= Ld;
        else if (X < 0.0)
          X += Ld;
      }
      if (on && l < 3) vw.x[l] = X;
      if (on && l < 3) vw.vp[l] = vp;
      if (on && l >= 3 && l < 6) vw.wp[l - 3] = vp;
      // the orientation, which no contact reads: lane k keeps the rotation of
      // every 16th sub-step from the k-th, and its sine, cosine and root are
      // taken once per 16 sub-steps
      const int k = sub & (DEM_LANES - 1);
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double v = __shfl(move, 3 + e, DEM_LANES);
        th[e] = l == k ? v : th[e];
      }
      if (k == DEM_LANES - 1 || sub + 1 == n_sub) {
        double dq[4] = {0.0, 0.0, 0.0, 0.0};
        const unsigned turns = group(l <= k && quat_of(th, dq));
        for (int u = 0; u <= k; ++u) {
          double w[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = __shfl(dq[e], u, DEM_LANES);
          if ((turns >> u) & 1u) quat_turn(q, w);
        }
      }
    }
    __syncthreads();
    // contacts: a lane per item
    double acc[6] = {0, 0, 0, 0, 0, 0};
    bool any = false;
    for (int base = 0; __any(base < items); base += DEM_LANES) {
      const int it = base + l;
      const bool has0 = it < items;
      int partner = -100;
      if (has0) partner = it < nw ? -1 - it : me.nb[it - nw];
      double delta = 0.0, nh[3] = {0.0, 0.0, 0.0}, arm[3] = {0.0, 0.0, 0.0};
      double vj[3] = {0.0, 0.0, 0.0}, wj[3] = {0.0, 0.0, 0.0};
      double Rcj = 0.0, mu = mu_s, mur = mu_r;
      bool has = has0;
      if (partner >= 0) {
        const DemView& pj = rows[partner].view[sub & 1];
        rel_vec(s, vw.x, pj.x, arm);  // X_i - X_j, min image
        const double dist = sqrt(dot3(arm, arm));
        Rcj = pj.Rc;
        delta = Rc + Rcj - dist;
        if (dist > 0.0)
          for (int k = 0; k < 3; ++k) nh[k] = arm[k] / dist;
        for (int k = 0; k < 3; ++k) {
          vj[k] = pj.vp[k];
          wj[k] = pj.wp[k];
        }
        mu = 0.5 * (mu_s + pj.mu_s);
        mur = 0.5 * (mu_r + pj.mu_r);
      } else if (has0) {
        has = wall_geom(s, vw.x, Rc, partner, delta, nh);
      }
      const bool active = has && delta > 0.0;
      int slot = has ? (int)me.slot[it] : -1;
      const bool ended = has && !active && slot >= 0, fresh = active && slot < 0;
      if (__any(ended || fresh)) {
        const unsigned out = group(ended), need = group(fresh);
        unsigned freed = 0u;
        for (unsigned m = out; m; m &= m - 1u)
          freed |= 1u << __shfl(slot, __ffs((int)m) - 1, DEM_LANES);
        if (ended) {  // its springs are released
          me.ct[slot].partner = -100;
          me.slot[it] = -1;
        }
        // (another lane may take the slot below: not moved past that)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // new contacts take the free slots in item order: as many as there are once
        // the lower items whose contacts end in this pass have given up theirs
        unsigned open = (~used | freed) & 0xffffu;
        if (fresh) {
          const int rank = __popc(need & below);
          unsigned m = open;
          for (int k = rank; k > 0; --k) m &= m - 1u;
          if (rank < __popc(~used & 0xffffu) + __popc(out & below)) {
            slot = __ffs((int)m) - 1;
            me.ct[slot].partner = partner;
            for (int k = 0; k < 3; ++k) me.ct[slot].xt[k] = me.ct[slot].xr[k] = 0.0;
            me.slot[it] = (int8_t)slot;
          } else {
            atomicOr(&s.counters[1], (uint32_t)ST_CONTACT_FULL);
          }
        }
        for (unsigned m = need; m; m &= m - 1u) open &= open - 1u;
        used = ~open & 0xffffu;
      }
      if (active && slot >= 0) {
        double Fo[3], To[3];
        contact_force(s, &me.ct[slot], delta, nh, vw.vp, vw.wp, vj, wj, Rc, Rcj, arm, mu, mur, dt,
                      Fo, To);
        for (int k = 0; k < 3; ++k) {
          acc[k] += Fo[k];
          acc[3 + k] += To[k];
        }
        any = true;
      }
    }
    // sums over the particle's lanes (a butterfly: every lane gets the same bits)
    if (__any(any)) {
#pragma unroll
      for (int k = 0; k < 6; ++k)
        for (int o = DEM_LANES / 2; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, DEM_LANES);
    }
    // corrector
    C = c == 0 ? acc[0] : c == 1 ? acc[1] : c == 2 ? acc[2] : c == 3 ? acc[3] : c == 4 ? acc[4]
                                                                                       : acc[5];
    if (!kin) V += 0.5 * (A + (F + C) / M) * dt;
    acc_mean += C;
  }
  // ---- the record, the springs and the history
  __syncthreads();
  if (on) {
    if (l < 6) {
      (&P.v[0])[c] = V;
      (&P.Fcap[0])[c] = Fca;
      (&P.Fca[0])[c] = 0.0;
      (&P.Ffp[0])[c] = fc;
      (&P.Fh_last[0])[c] = Fh;
      (&P.Fh[0])[c] = 0.0;
      (&P.Fcp[0])[c] = C;
      (&P.Fcon[0])[c] = acc_mean / n_sub;
      if (c < 3) {
        P.x[c] = X;
        P.xo[c] = X0;
      }
    }
    if (l == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) P.q[k] = q[k];
      P.Ro = R;
      P.havep = 1;
      P.cap_on = 0;
      if (near_open_end(s, X, R)) atomicOr(&s.counters[1], (uint32_t)ST_OPEN_END);
    }
    s.ct[(long long)i * MAXC + l] = me.ct[l];
    if (s.hist_cap > 0 && l < 6) {
      double* h = s.hist + ((long long)(step % (unsigned long long)s.hist_cap) * np + i) *
                               LBM_HIST_DOUBLES_DEV;
      h[c] = Fh;
      h[6 + c] = Fca;
      h[12 + c] = acc_mean / n_sub;
      if (c < 3) h[18 + c] = X;
      h[21 + c] = V;
    }
  }
  if (threadIdx.x == 0) {
    *s.step_counter = step + 1;
    s.counters[0] = 0u;  // the fresh list, which the mask update fills again
  }
}

// ------------------------------------------------------------ host launchers

hipError_t launch_push(const SimDev& s, hipStream_t st) {
  hipLaunchKernelGGL(k_push, dim3((unsigned)((s.np + 63) / 64)), dim3(64), 0, st, s);
  return hipGetLastError();
}

// np_max: the most particles of one simulation of the batch; own: blocks that the
// particles' own boxes take
hipError_t launch_mask_update(const Batch& b, int np_rows, int np_max, int Bmax, long long own,
                              bool with_release, hipStream_t st) {
  if (np_rows == 0) return hipSuccess;
  dim3 grid(particle_blocks(np_rows, Bmax, own), np_rows);
  if (!mask_by_search(np_max, b.fc == 2)) {
    hipLaunchKernelGGL(k_claim, grid, dim3(256), 0, st, b);
    if (with_release) hipLaunchKernelGGL(k_release, grid, dim3(256), 0, st, b);
    hipLaunchKernelGGL(k_cover, grid, dim3(256), 0, st, b);
    return hipGetLastError();
  }
  const bool stride = (long long)grid.x * 256 < (long long)Bmax * Bmax * Bmax;
  auto* k = with_release ? (stride ? k_mask<true, true> : k_mask<true, false>)
                         : (stride ? k_mask<false, true> : k_mask<false, false>);
  hipLaunchKernelGGL(k, grid, dim3(256), 0, st, b);
  return hipGetLastError();
}

// np_max: the most particles of one simulation in the batch; np_rows: particle
// rows of the batch; n_sub_max: the most DEM sub-steps of one simulation
hipError_t launch_dem(const Batch& b, int np_max, int np_rows, int n_sub_max, hipStream_t st) {
  if (np_max == 0) return hipSuccess;
  if (np_max <= DEM_SMALL) {
    const unsigned threads = (unsigned)((np_max * DEM_LANES + 63) / 64 * 64);
    hipLaunchKernelGGL(k_dem, dim3(b.nsim), dim3(threads), np_max * sizeof(DemRow), st, b);
    return hipGetLastError();
  }
  // many particles: set-up, then a launch per sub-step with a wave per particle
  const unsigned g64 = (unsigned)((np_rows + 63) / 64);
  if (np_max <= 32 * MAXNB) {
    // the pair tests on many CUs; the hit masks fit the list buffer
    const long long nw = (np_max + 31) / 32;
    const unsigned gx = (unsigned)(((long long)np_max * nw * 32 + 255) / 256);
    hipLaunchKernelGGL(k_dem_search, dim3(gx, b.nsim), dim3(256), 0, st, b);
    hipLaunchKernelGGL(k_dem_setup, dim3(g64), dim3(64), 0, st, b, np_rows, 1);
  } else {
    hipLaunchKernelGGL(k_dem_lists, dim3(g64), dim3(64), 0, st, b, np_rows);
    hipLaunchKernelGGL(k_dem_setup, dim3(g64), dim3(64), 0, st, b, np_rows, 0);
  }
  const unsigned g4 = (unsigned)((np_rows + 3) / 4);
  for (int sub = 0; sub < n_sub_max; ++sub)
    hipLaunchKernelGGL(k_dem_sub, dim3(g4), dim3(256), 0, st, b, np_rows, sub);
  return hipGetLastError();
}

}  // namespace lbm
