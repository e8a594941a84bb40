// Articulated rigid bodies on a fixed base (Appendix D.1): the batched forward
// substeps (composite rigid body algorithm for the mass matrix, recursive
// Newton-Euler for the bias forces, a sparse solve, semi-implicit Euler) and
// their reverse-mode adjoint.
//
// One environment per group of G lanes of a wave (G: the link count rounded up
// to 8, 16, 32 or 64), lane i working on link i; a block is one wave, so its
// barriers are cheap. Every spatial quantity is a world-frame Plucker vector
// about one fixed origin (motion: angular velocity, velocity of the body point
// at the origin; force: moment about the origin, force). In that frame the
// tree recursions need no coordinate transforms:
//  - poses and root-path sums (velocities, accelerations) are taken by pointer
//    doubling: round k combines a lane's partial result with that of its 2^k-th
//    ancestor through a lane permute, ceil(log2 D) rounds for a tree D deep;
//  - subtree sums (forces, composite inertias) go children first over the tree's
//    height levels through LDS, a lane's running sum staying in registers;
//  - the joint-space mass matrix M_ij = S_j . (Ic_i S_i), j on i's root path,
//    is kept as one row per link with its ancestors in order of depth, so the
//    ancestors that two links of a path share have the same places in both rows.
//    Eliminated leaves first (M = L^T P L, L unit triangular) it keeps its sparsity, and
//    eliminating link k from its ancestor i's row is one dense multiply-add
//    of the leading part of row k, 128 bits at a time. The right-hand side is
//    eliminated along with the rows; the solve with L goes down one depth at a
//    time, each lane taking its one ancestor there through a lane permute.
// A substep touches HBM only for the torques and the tape. The adjoint reads
// the recorded joint accelerations and so needs one elimination, with the
// cotangent as right-hand side, and no bias forces.
//
// Bound by instruction issue once the chip is full (65536 hands of 13 links: the
// vector ALUs were busy 81% of the time), by their chain when it is not. Walking
// root paths and subtrees by 64-bit link masks, with a factorisation and solves
// over them, 16 substeps of those hands took 951 us forward and 1809 us back;
// 595 and 990 now. 256 hands: 146 and 263 us; 91 and 138 now.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "mpm_device.h"
#include "rb_kernels.h"

namespace mpmx {

namespace rb {

constexpr int kBlock = 64;   // one wave per block

struct V6 {
  float c[6];   // [0..2] angular part (or moment), [3..5] linear part (or force)
};

MD V6 zero6() {
  V6 r;
#pragma unroll
  for (int k = 0; k < 6; ++k) r.c[k] = 0.f;
  return r;
}
MD V6 add6(const V6& a, const V6& b) {
  V6 r;
#pragma unroll
  for (int k = 0; k < 6; ++k) r.c[k] = a.c[k] + b.c[k];
  return r;
}
MD V6 sub6(const V6& a, const V6& b) {
  V6 r;
#pragma unroll
  for (int k = 0; k < 6; ++k) r.c[k] = a.c[k] - b.c[k];
  return r;
}
MD V6 scale6(const V6& a, float s) {
  V6 r;
#pragma unroll
  for (int k = 0; k < 6; ++k) r.c[k] = a.c[k] * s;
  return r;
}
MD float dot6(const V6& a, const V6& b) {
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < 6; ++k) s = fmaf(a.c[k], b.c[k], s);
  return s;
}
MD void cross3(const float* a, const float* b, float* r) {
  r[0] = a[1] * b[2] - a[2] * b[1];
  r[1] = a[2] * b[0] - a[0] * b[2];
  r[2] = a[0] * b[1] - a[1] * b[0];
}
// motion x motion: (w_a x w_b, w_a x v_b + v_a x w_b)
MD V6 crm(const V6& a, const V6& b) {
  V6 r;
  float t[3];
  cross3(a.c, b.c, r.c);
  cross3(a.c, b.c + 3, r.c + 3);
  cross3(a.c + 3, b.c, t);
  r.c[3] += t[0]; r.c[4] += t[1]; r.c[5] += t[2];
  return r;
}
// motion x* force: (w x n + v x f, w x f)
MD V6 crf(const V6& a, const V6& f) {
  V6 r;
  float t[3];
  cross3(a.c, f.c, r.c);
  cross3(a.c + 3, f.c + 3, t);
  r.c[0] += t[0]; r.c[1] += t[1]; r.c[2] += t[2];
  cross3(a.c, f.c + 3, r.c + 3);
  return r;
}

// spatial inertia about the origin: mass, first moment h = m c, rotational inertia J about the origin
// (symmetric: xx yy zz xy xz yz)
struct Inertia {
  float m, h[3], J[6];
};
MD V6 iapply(const Inertia& I, const V6& a) {
  const float* w = a.c;
  const float* v = a.c + 3;
  V6 r;
  float t[3];
  cross3(I.h, v, t);
  r.c[0] = I.J[0] * w[0] + I.J[3] * w[1] + I.J[4] * w[2] + t[0];
  r.c[1] = I.J[3] * w[0] + I.J[1] * w[1] + I.J[5] * w[2] + t[1];
  r.c[2] = I.J[4] * w[0] + I.J[5] * w[1] + I.J[2] * w[2] + t[2];
  cross3(I.h, w, t);
  r.c[3] = I.m * v[0] - t[0];
  r.c[4] = I.m * v[1] - t[1];
  r.c[5] = I.m * v[2] - t[2];
  return r;
}

// link sets as bit masks: 32 bits where they suffice (a 64-bit set costs its walk
// about five more instructions per link)
template <int G>
using Mask = std::conditional_t<(G <= 32), uint32_t, uint64_t>;
MD int first_bit(uint32_t m) { return __builtin_ctz(m); }
MD int first_bit(uint64_t m) { return __builtin_ctzll(m); }
MD int last_bit(uint32_t m) { return 31 - __builtin_clz(m); }
MD int last_bit(uint64_t m) { return 63 - __builtin_clzll(m); }

MD float lane_read(float x, int addr) {   // x of the lane at byte address `addr` (lane * 4); every lane takes part
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, x)));
}

constexpr int rounds_max(int G) { return G == 8 ? 3 : G == 16 ? 4 : G == 32 ? 5 : 6; }

// a lane's own link
template <int G>
struct Link {
  float Rt[9], pt[3], ax[3], m, com[3], In[6];
  float ct[4];                 // its first contact sphere
  Mask<G> anc, desc, kids;
  int up[rounds_max(G)];       // byte address of the lane of the 2^k-th ancestor, the lane's own where there is none
  int nup;                     // how many of them there are: depth >= 2^k for k < nup
  int c0;                      // first lane of the environment
  int cb, ce;
  int height, depth;   // levels: longest path down to a leaf, joints above
  bool prism;          // the joint slides along its axis instead of turning about it
};
template <int G>
MD Link<G> load_link(const RbModel& M, int i, int c0, bool live) {
  Link<G> l;
  l.c0 = c0;
  const float* s = M.link + (size_t)(live ? i : 0) * kRbLinkF;
#pragma unroll
  for (int k = 0; k < 9; ++k) l.Rt[k] = s[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    l.pt[k] = s[9 + k];
    l.ax[k] = s[12 + k];
    l.com[k] = s[16 + k];
  }
  l.m = s[15];
#pragma unroll
  for (int k = 0; k < 6; ++k) l.In[k] = s[19 + k];
  l.anc = live ? (Mask<G>)M.anc[i] : 0;
  l.desc = live ? (Mask<G>)M.desc[i] & ~((Mask<G>)1 << i) : 0;
  l.kids = live ? (Mask<G>)M.kids[i] : 0;
  l.cb = live ? M.cbeg[i] : 0;
  l.ce = live ? M.cbeg[i + 1] : 0;
  l.height = live ? (M.level[i] & 0xffff) : -1;
  l.depth = live ? (M.level[i] >> 16) : -1;
  l.prism = s[25] != 0.f;
#pragma unroll
  for (int k = 0; k < 4; ++k) l.ct[k] = l.cb < l.ce ? M.contact[(size_t)l.cb * 4 + k] : 0.f;
  // 2^k-th ancestors: the parent is the last link above i on its root path (parents come first)
  const Mask<G> above = l.anc & ~((Mask<G>)1 << i);
  l.nup = 0;
#pragma unroll
  for (int k = 0; k < rounds_max(G); ++k) {
    if (k == 0)
      l.up[0] = (c0 + (above ? last_bit(above) : i)) * 4;
    else
      l.up[k] = __builtin_amdgcn_ds_bpermute(l.up[k - 1], l.up[k - 1]);
    if (l.depth >= (1 << k)) {
      l.nup = k + 1;
    } else {
      l.up[k] = (c0 + i) * 4;
    }
  }
  return l;
}

struct Prm {
  float damp, ke, kd, kf, zg;   // zg relative to the spatial origin
};
MD Prm load_prm(const RbModel& M, int e) {
  Prm p{0.f, 0.f, 0.f, 0.f, -INFINITY};
  if (e < M.E) {
    const float* r = M.prm + (size_t)e * kRbPrm;
    p.damp = r[0]; p.ke = r[1]; p.kd = r[2]; p.kf = r[3]; p.zg = r[4] - M.zref;
  }
  return p;
}

// LDS of a block. A column per lane: rows of vectors being summed over subtrees
// (quads of rows side by side, so that a lane moves 128 bits at a time), joint
// motions, mass-matrix rows. The sums are finished before the mass matrix
// is written and it is used up before the next ones, so the two share their space.
typedef float f4 __attribute__((ext_vector_type(4), may_alias));
typedef float f2 __attribute__((ext_vector_type(2), may_alias));
template <int G>
struct BlockLds {
  static constexpr int kRow = G + 4;   // a multiple of four, spread over the banks
  union {
    f4 sum[4 * kBlock];
    f4 row[kBlock * kRow / 4];
  };
  f4 S[6 * kBlock / 4];
  f2 piv[kBlock];   // 1 / pivot and eliminated right-hand side of a link
};

// NR values of a lane (an even number) as a column
template <int NR>
MD void put_rows(f4* A, int col, const float (&a)[NR]) {
#pragma unroll
  for (int q = 0; q < NR / 4; ++q) A[q * kBlock + col] = f4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
  if constexpr (NR % 4 == 2) reinterpret_cast<f2*>(A + NR / 4 * kBlock)[col] = f2{a[NR - 2], a[NR - 1]};
}
template <int NR>
MD void get_rows(const f4* A, int col, float (&a)[NR]) {
#pragma unroll
  for (int q = 0; q < NR / 4; ++q) {
    const f4 v = A[q * kBlock + col];
#pragma unroll
    for (int k = 0; k < 4; ++k) a[4 * q + k] = v[k];
  }
  if constexpr (NR % 4 == 2) {
    const f2 v = reinterpret_cast<const f2*>(A + NR / 4 * kBlock)[col];
    a[NR - 2] = v[0];
    a[NR - 1] = v[1];
  }
}

// Subtree sums: a lane's own values on entry, the sums over its subtree on
// return. One height level at a time a link adds its children's finished
// columns, so a level costs the most children of any of its links (not the size
// of the largest subtree).
template <int G, int NR>
MD void subtree_sums(const RbModel& M, const Link<G>& l, int col, bool live, f4* A, float (&a)[NR]) {
  if (live) put_rows(A, col, a);
  __syncthreads();
  for (int h = 1; h < M.H; ++h) {
    if (l.height == h) {
      Mask<G> mk = l.kids;
      while (mk) {
        const int c = first_bit(mk);
        mk &= mk - 1;
        float v[NR];
        get_rows(A, l.c0 + c, v);
#pragma unroll
        for (int k = 0; k < NR; ++k) a[k] += v[k];
      }
      put_rows(A, col, a);
    }
    __syncthreads();
  }
}

// sum of x over the links of the root path
template <int G>
MD void path_sum(const RbModel& M, const Link<G>& l, V6& x) {
#pragma unroll
  for (int k = 0; k < rounds_max(G); ++k) {
    if ((1 << k) >= M.D) break;
    float t[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) t[c] = lane_read(x.c[c], l.up[k]);
    if (k < l.nup) {
#pragma unroll
      for (int c = 0; c < 6; ++c) x.c[c] += t[c];
    }
  }
}

// what the adjoint needs of one substep's forward, per lane
struct Frame {
  float R[9], p[3];
  V6 S, V, u, A;
  Inertia I;
};

template <int G>
MD void contact_point(const RbModel& M, const Link<G>& l, const Frame& F, int c, float* cw, float* x) {
  float s[4] = {l.ct[0], l.ct[1], l.ct[2], l.ct[3]};
  if (c > l.cb) {
    const f4 v = reinterpret_cast<const f4*>(M.contact)[c];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = v[k];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) cw[a] = F.p[a] + F.R[3 * a] * s[0] + F.R[3 * a + 1] * s[1] + F.R[3 * a + 2] * s[2];
  x[0] = cw[0];
  x[1] = cw[1];
  x[2] = cw[2] - s[3];
}

// Solves M x = b for the mass matrix M_ij = S_j . (Ic_i S_i); L.S holds every
// lane's S. Row i has the ancestors' entries by depth, its own at l.depth.
// Leaves first, one height level at a time: the level's links invert their
// pivots, then every link above them eliminates them from its row and
// right-hand side (row_i -= (M_ki / M_kk) row_k over i's root path). Rows a
// level reads are never written in that level. Every lane of the block calls it.
template <int G>
MD float solve(const RbModel& M, const Link<G>& l, BlockLds<G>& L, int col, bool live, const Inertia& Ic,
               const V6& S, float b) {
  constexpr int kRow = BlockLds<G>::kRow;
  float* row = reinterpret_cast<float*>(L.row) + col * kRow;
  {
    const V6 Fc = iapply(Ic, S);
    Mask<G> mk = l.anc;
    for (int d = 0; mk; ++d) {
      const int j = first_bit(mk);
      mk &= mk - 1;
      float Sj[6];
      get_rows(L.S, l.c0 + j, Sj);
      float t = 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) t = fmaf(Sj[k], Fc.c[k], t);
      row[d] = t;
    }
  }
  __syncthreads();
  float inv = 0.f;
  for (int h = 0; h < M.H; ++h) {
    if (l.height == h) {
      const float p = row[l.depth];
      inv = p > 0.f ? 1.f / p : __builtin_nanf("");   // a non-positive pivot: the env is flagged non-finite
      L.piv[col] = f2{inv, b};
    }
    __syncthreads();
    // the links of height h (the same in every environment of the block)
    Mask<G> mk = l.desc & (Mask<G>)__ballot(l.height == h);
    while (mk) {
      const int k = l.c0 + first_bit(mk);
      mk &= mk - 1;
      const f2 pk = L.piv[k];
      const float* rk = reinterpret_cast<const float*>(L.row) + k * kRow;
      const float lki = rk[l.depth] * pk[0];
      b = fmaf(-lki, pk[1], b);
      for (int d = 0; d <= l.depth; d += 4) {   // past l.depth: places that row i does not use
        const f4 vk = *reinterpret_cast<const f4*>(rk + d);
        f4 vi = *reinterpret_cast<f4*>(row + d);
#pragma unroll
        for (int c = 0; c < 4; ++c) vi[c] = fmaf(-lki, vk[c], vi[c]);
        *reinterpret_cast<f4*>(row + d) = vi;
      }
    }
    __syncthreads();
  }
  // x_k = (b_k - sum over the ancestors j of M_kj x_j) / M_kk: a lane has its x once the depths above are done
  Mask<G> rem = l.anc;
  for (int d = 0; d + 1 < M.D; ++d) {
    const float xj = lane_read(b * inv, (l.c0 + (rem ? first_bit(rem) : 0)) * 4);
    if (l.depth > d) b = fmaf(-row[d], xj, b);
    rem &= rem - 1;
  }
  __syncthreads();   // the rows' space is free
  return live ? b * inv : 0.f;
}

// Poses, joint motions, inertias, velocities and accelerations of an environment's links at (q, qd) with joint
// accelerations qdd (a sum over the root path of S_j qdd_j + V_j x S_j qd_j, and -g).
template <int G>
MD void kinematics(const RbModel& M, const Link<G>& l, float q, float qd, float qdd, Frame& F) {
  // own joint: R = joint_rot Rot(axis, q) (Rodrigues: c I + s [a]x + (1 - c) a a^T) and p = joint_pos; a
  // prismatic joint turns nothing (Rot = I) and shifts joint_pos by q joint_rot axis
  {
    float sn = 0.f, cs = 1.f;
    if (!l.prism) sincosf(q, &sn, &cs);
    const float* a = l.ax;
    const float oc = 1.f - cs;
    const float Rq[9] = {cs + oc * a[0] * a[0], oc * a[0] * a[1] - sn * a[2], oc * a[0] * a[2] + sn * a[1],
                         oc * a[1] * a[0] + sn * a[2], cs + oc * a[1] * a[1], oc * a[1] * a[2] - sn * a[0],
                         oc * a[2] * a[0] - sn * a[1], oc * a[2] * a[1] + sn * a[0], cs + oc * a[2] * a[2]};
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c)
        F.R[3 * r + c] = l.Rt[3 * r] * Rq[c] + l.Rt[3 * r + 1] * Rq[3 + c] + l.Rt[3 * r + 2] * Rq[6 + c];
    const float qs = l.prism ? q : 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      F.p[k] = fmaf(qs, l.Rt[3 * k] * a[0] + l.Rt[3 * k + 1] * a[1] + l.Rt[3 * k + 2] * a[2], l.pt[k]);
  }
  // world pose: after round k a lane's pose is relative to its 2^(k+1)-th ancestor (or the world)
#pragma unroll
  for (int k = 0; k < rounds_max(G); ++k) {
    if ((1 << k) >= M.D) break;
    float R[9], p[3];
#pragma unroll
    for (int c = 0; c < 9; ++c) R[c] = lane_read(F.R[c], l.up[k]);
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = lane_read(F.p[c], l.up[k]);
    if (k < l.nup) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
        p[r] += R[3 * r] * F.p[0] + R[3 * r + 1] * F.p[1] + R[3 * r + 2] * F.p[2];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float b0 = F.R[c], b1 = F.R[3 + c], b2 = F.R[6 + c];
#pragma unroll
        for (int r = 0; r < 3; ++r) F.R[3 * r + c] = R[3 * r] * b0 + R[3 * r + 1] * b1 + R[3 * r + 2] * b2;
        F.p[c] = p[c];
      }
    }
  }
  // joint motion S = (s, p x s) for a revolute joint, (0, s) for a prismatic one, s = R axis; body inertia
  // about the origin
  {
    const float* R = F.R;
    float s[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) s[r] = R[3 * r] * l.ax[0] + R[3 * r + 1] * l.ax[1] + R[3 * r + 2] * l.ax[2];
    if (l.prism) {
      F.S.c[0] = 0.f; F.S.c[1] = 0.f; F.S.c[2] = 0.f;
      F.S.c[3] = s[0]; F.S.c[4] = s[1]; F.S.c[5] = s[2];
    } else {
      F.S.c[0] = s[0]; F.S.c[1] = s[1]; F.S.c[2] = s[2];
      cross3(F.p, s, F.S.c + 3);
    }
    float c[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) c[r] = F.p[r] + R[3 * r] * l.com[0] + R[3 * r + 1] * l.com[1] + R[3 * r + 2] * l.com[2];
    // R Ib R^T
    const float Ib[9] = {l.In[0], l.In[3], l.In[4], l.In[3], l.In[1], l.In[5], l.In[4], l.In[5], l.In[2]};
    float T[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) T[3 * r + k] = R[3 * r] * Ib[k] + R[3 * r + 1] * Ib[3 + k] + R[3 * r + 2] * Ib[6 + k];
    float W[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) W[3 * r + k] = T[3 * r] * R[3 * k] + T[3 * r + 1] * R[3 * k + 1] + T[3 * r + 2] * R[3 * k + 2];
    const float m = l.m;
    const float cc = c[0] * c[0] + c[1] * c[1] + c[2] * c[2];
    F.I.m = m;
    F.I.h[0] = m * c[0]; F.I.h[1] = m * c[1]; F.I.h[2] = m * c[2];
    F.I.J[0] = W[0] + m * (cc - c[0] * c[0]);
    F.I.J[1] = W[4] + m * (cc - c[1] * c[1]);
    F.I.J[2] = W[8] + m * (cc - c[2] * c[2]);
    F.I.J[3] = W[1] - m * c[0] * c[1];
    F.I.J[4] = W[2] - m * c[0] * c[2];
    F.I.J[5] = W[5] - m * c[1] * c[2];
  }
  F.u = scale6(F.S, qd);
  F.V = F.u;
  path_sum(M, l, F.V);
  F.A = crm(F.V, F.u);
#pragma unroll
  for (int k = 0; k < 6; ++k) F.A.c[k] = fmaf(F.S.c[k], qdd, F.A.c[k]);
  path_sum(M, l, F.A);
  F.A.c[3] -= M.g[0];
  F.A.c[4] -= M.g[1];
  F.A.c[5] -= M.g[2];
}

MD void inertia_rows(const Inertia& I, float* a) {
  a[0] = I.m;
#pragma unroll
  for (int k = 0; k < 3; ++k) a[1 + k] = I.h[k];
#pragma unroll
  for (int k = 0; k < 6; ++k) a[4 + k] = I.J[k];
}
MD Inertia inertia_of(const float* a) {
  Inertia I;
  I.m = a[0];
#pragma unroll
  for (int k = 0; k < 3; ++k) I.h[k] = a[1 + k];
#pragma unroll
  for (int k = 0; k < 6; ++k) I.J[k] = a[4 + k];
  return I;
}

// One substep's dynamics of an environment: qdd of the lane's joint. Every lane of the block calls it (barriers
// and lane permutes inside).
template <int G>
MD float dynamics(const RbModel& M, const Link<G>& l, BlockLds<G>& L, int col, bool live, float q, float qd,
                  float tau, const Prm& P) {
  Frame F;
  kinematics(M, l, q, qd, 0.f, F);
  // force of the link at qdd = 0, less the ground contact on its spheres
  V6 f = add6(iapply(F.I, F.A), crf(F.V, iapply(F.I, F.V)));
  for (int c = l.cb; c < l.ce; ++c) {
    float cw[3], x[3], xd[3];
    contact_point(M, l, F, c, cw, x);
    cross3(F.V.c, x, xd);
    xd[0] += F.V.c[3]; xd[1] += F.V.c[4]; xd[2] += F.V.c[5];
    const float depth = P.zg - x[2];
    if (depth > 0.f) {
      const float fc[3] = {-P.kf * xd[0], -P.kf * xd[1], P.ke * depth - P.kd * xd[2]};
      float n[3];
      cross3(x, fc, n);
      f.c[0] -= n[0]; f.c[1] -= n[1]; f.c[2] -= n[2];
      f.c[3] -= fc[0]; f.c[4] -= fc[1]; f.c[5] -= fc[2];
    }
  }
  // subtree sums: force (bias torque S_i . F_i) and composite inertia
  float a[16];
#pragma unroll
  for (int k = 0; k < 6; ++k) a[k] = f.c[k];
  inertia_rows(F.I, a + 6);
  if (live) put_rows(L.S, col, F.S.c);
  subtree_sums(M, l, col, live, L.sum, a);
  float rhs = fmaf(-P.damp, qd, tau);
#pragma unroll
  for (int k = 0; k < 6; ++k) rhs = fmaf(-F.S.c[k], a[k], rhs);
  return solve(M, l, L, col, live, inertia_of(a + 6), F.S, rhs);
}

template <int G>
__global__ __launch_bounds__(kBlock) void k_rb_forward(RbModel M, int S, float* __restrict__ q,
                                                       float* __restrict__ qd, const float* __restrict__ tau,
                                                       float* __restrict__ tape, float* __restrict__ tape_qdd,
                                                       int32_t* __restrict__ errs) {
  constexpr int EPB = kBlock / G;
  __shared__ BlockLds<G> lds;
  const int lane = threadIdx.x % G, grp = threadIdx.x / G;
  const int e = blockIdx.x * EPB + grp;
  const int N = M.N, E = M.E;
  const bool live = e < E && lane < N;
  const Link<G> l = load_link<G>(M, lane, grp * G, live);
  const Prm P = load_prm(M, e);
  const size_t at = (size_t)e * N + lane;
  float qi = live ? q[at] : 0.f, qdi = live ? qd[at] : 0.f;
  if (tape && live) {
    tape[(size_t)e * 2 * N + lane] = qi;
    tape[(size_t)e * 2 * N + N + lane] = qdi;
  }
  for (int s = 0; s < S; ++s) {
    const float ti = (tau && live) ? tau[(size_t)s * E * N + at] : 0.f;
    const float qdd = dynamics<G>(M, l, lds, threadIdx.x, live, qi, qdi, ti, P);
    qdi = fmaf(M.dt, qdd, qdi);
    qi = fmaf(M.dt, qdi, qi);
    if (tape && live) {
      float* t = tape + ((size_t)(s + 1) * E + e) * 2 * N;
      t[lane] = qi;
      t[N + lane] = qdi;
      tape_qdd[(size_t)s * E * N + at] = qdd;
    }
  }
  if (live) {
    q[at] = qi;
    qd[at] = qdi;
    if (!isfinite(qi) || !isfinite(qdi)) atomicOr(&errs[e], 1);
  }
}

// Three waves per SIMD (168 VGPRs, a few spilled): 65536 hands of 13 links take 990 us for 16 substeps, against
// 1275 at two waves without spills and 1144 at four.
template <int G>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_rb_backward(RbModel M, int S, const float* __restrict__ tape,
                                                        const float* __restrict__ tape_qdd,
                                                        const float* __restrict__ gq, const float* __restrict__ gqd,
                                                        float* __restrict__ dq0, float* __restrict__ dqd0,
                                                        float* __restrict__ dtau, double* __restrict__ dprm) {
  constexpr int EPB = kBlock / G;
  __shared__ BlockLds<G> lds;
  BlockLds<G>& L = lds;
  const int lane = threadIdx.x % G, grp = threadIdx.x / G, col = threadIdx.x;
  const int e = blockIdx.x * EPB + grp;
  const int N = M.N, E = M.E;
  const bool live = e < E && lane < N;
  const Link<G> l = load_link<G>(M, lane, grp * G, live);
  const Prm P = load_prm(M, e);
  const size_t at = (size_t)e * N + lane;
  // cotangents of the current (q, qd)
  float a = (gq && live) ? gq[at] : 0.f;
  float b = (gqd && live) ? gqd[at] : 0.f;
  float acc[kRbPrm] = {0.f, 0.f, 0.f, 0.f, 0.f};
  // the record of the next substep to reverse, read one ahead
  float qn = 0.f, qdn = 0.f, qddn = 0.f;
  auto prefetch = [&](int s) {
    if (s < 0 || !live) return;
    const float* t = tape + ((size_t)s * E + e) * 2 * N;
    qn = t[lane];
    qdn = t[N + lane];
    qddn = tape_qdd[(size_t)s * E * N + at];
  };
  prefetch(S - 1);
  for (int s = S - 1; s >= 0; --s) {
    const float qi = qn, qdi = qdn, qdd = qddn;
    prefetch(s - 1);
    Frame F;
    kinematics(M, l, qi, qdi, qdd, F);
    // qd' = qd + dt qdd, q' = q + dt qd': the cotangent of qd' is b + dt a, that of qdd dt (b + dt a)
    const float gtot = fmaf(M.dt, a, b);
    float lam;   // torque cotangent M^-1 qdd_bar
    {
      float ic[10];
      inertia_rows(F.I, ic);
      if (live) put_rows(L.S, col, F.S.c);
      subtree_sums(M, l, col, live, L.sum, ic);
      lam = solve(M, l, L, col, live, inertia_of(ic), F.S, M.dt * gtot);
    }
    if (dtau && live) dtau[(size_t)s * E * N + at] = lam;
    acc[0] -= lam * qdi;
    // phi = lambda . ID(q, qd, qdd): Lambda_k = sum over k's root path of lambda_i S_i
    V6 Lam = scale6(F.S, lam);
    path_sum(M, l, Lam);
    const V6 IV = iapply(F.I, F.V);
    const V6 IA = iapply(F.I, F.A);
    V6 f = add6(IA, crf(F.V, IV));   // less the contact forces below
    // phi = sum_k Lambda_k . f_k: f_bar = Lambda; A_bar = I Lambda; V_bar from V x* (I V)
    const V6 Abar = iapply(F.I, Lam);
    const V6 VL = crm(F.V, Lam);
    const V6 IVL = iapply(F.I, VL);
    V6 Vbar = scale6(add6(crf(Lam, IV), IVL), -1.f);
    // geometric wrench of the body: the body's inertia turned with it, a . (I b) over the pairs
    // (Lambda, A) and (-V x Lambda, V) gives -(a x* I b + b x* I a)
    V6 W = sub6(add6(crf(VL, IV), crf(F.V, IVL)), add6(crf(Lam, IA), crf(F.A, Abar)));
    for (int c = l.cb; c < l.ce; ++c) {
      float cw[3], x[3], xd[3];
      contact_point(M, l, F, c, cw, x);
      cross3(F.V.c, x, xd);
      xd[0] += F.V.c[3]; xd[1] += F.V.c[4]; xd[2] += F.V.c[5];
      const float depth = P.zg - x[2];
      if (depth > 0.f) {
        const float fc[3] = {-P.kf * xd[0], -P.kf * xd[1], P.ke * depth - P.kd * xd[2]};
        float t0[3];
        cross3(x, fc, t0);
        f.c[0] -= t0[0]; f.c[1] -= t0[1]; f.c[2] -= t0[2];
        f.c[3] -= fc[0]; f.c[4] -= fc[1]; f.c[5] -= fc[2];
        // phi_c = -f . lh, lh = Lambda_v + Lambda_w x x (the point's velocity under Lambda)
        float lh[3];
        cross3(Lam.c, x, lh);
        lh[0] += Lam.c[3]; lh[1] += Lam.c[4]; lh[2] += Lam.c[5];
        const float xdb[3] = {P.kf * lh[0], P.kf * lh[1], P.kd * lh[2]};
        float xb[3], t1[3], t2[3];
        cross3(Lam.c, fc, t1);
        cross3(xdb, F.V.c, t2);
        xb[0] = t1[0] + t2[0];
        xb[1] = t1[1] + t2[1];
        xb[2] = t1[2] + t2[2] + P.ke * lh[2];
        // xd = v + w x x
        cross3(x, xdb, t1);
        Vbar.c[0] += t1[0]; Vbar.c[1] += t1[1]; Vbar.c[2] += t1[2];
        Vbar.c[3] += xdb[0]; Vbar.c[4] += xdb[1]; Vbar.c[5] += xdb[2];
        // the sphere centre moves with the body
        cross3(cw, xb, t1);
        W.c[0] += t1[0]; W.c[1] += t1[1]; W.c[2] += t1[2];
        W.c[3] += xb[0]; W.c[4] += xb[1]; W.c[5] += xb[2];
        // parameters (cotangent -dphi/dp)
        acc[1] += lh[2] * depth;
        acc[2] -= lh[2] * xd[2];
        acc[3] -= lh[0] * xd[0] + lh[1] * xd[1];
        acc[4] += P.ke * lh[2];
      }
    }
    // phi = sum_i lambda_i S_i . F_i (F_i the subtree force) and A_i = A_0 + sum over the root path of
    // (S_j qdd_j + V_j x S_j qd_j): subtree sums of f and of A_bar
    float t12[12];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      t12[k] = f.c[k];
      t12[6 + k] = Abar.c[k];
    }
    subtree_sums(M, l, col, live, L.sum, t12);
    V6 DA, Sbar;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      DA.c[k] = t12[6 + k];
      Sbar.c[k] = fmaf(t12[k], lam, DA.c[k] * qdd);
    }
    Vbar = add6(Vbar, crf(F.u, DA));
    // V_i = sum over the root path of u_j, u_j = S_j qd_j
    subtree_sums(M, l, col, live, L.sum, Vbar.c);
    const V6 ubar = sub6(Vbar, crf(F.V, DA));
    Sbar = add6(Sbar, scale6(ubar, qdi));
    const float dphi_qd = dot6(F.S, ubar);
    W = add6(W, crf(F.S, Sbar));
    // turning joint j moves its whole subtree: dphi/dq_j = S_j . (subtree sum of the wrenches)
    subtree_sums(M, l, col, live, L.sum, W.c);
    const float dphi_q = dot6(F.S, W);
    a = a - dphi_q;
    b = gtot - P.damp * lam - dphi_qd;
  }
  if (live) {
    dq0[at] = a;
    dqd0[at] = b;
  }
  if (dprm) {
    float* part = reinterpret_cast<float*>(L.sum);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kRbPrm; ++c) part[c * kBlock + col] = live ? acc[c] : 0.f;
    __syncthreads();
    if (lane < kRbPrm && e < E) {
      double s = 0.0;
      for (int k = 0; k < N; ++k) s += (double)part[lane * kBlock + grp * G + k];
      dprm[(size_t)e * kRbPrm + lane] = s;
    }
  }
}

}  // namespace rb

int rb_group(int N) { return N <= 8 ? 8 : N <= 16 ? 16 : N <= 32 ? 32 : 64; }

void launch_rb_forward(const RbModel& m, int S, float* q, float* qd, const float* tau, float* tape, float* tape_qdd,
                       int32_t* errs, hipStream_t s) {
  const int G = rb_group(m.N), epb = rb::kBlock / G;
  const dim3 grid((m.E + epb - 1) / epb), block(rb::kBlock);
  switch (G) {
    case 8: rb::k_rb_forward<8><<<grid, block, 0, s>>>(m, S, q, qd, tau, tape, tape_qdd, errs); break;
    case 16: rb::k_rb_forward<16><<<grid, block, 0, s>>>(m, S, q, qd, tau, tape, tape_qdd, errs); break;
    case 32: rb::k_rb_forward<32><<<grid, block, 0, s>>>(m, S, q, qd, tau, tape, tape_qdd, errs); break;
    default: rb::k_rb_forward<64><<<grid, block, 0, s>>>(m, S, q, qd, tau, tape, tape_qdd, errs); break;
  }
}

void launch_rb_backward(const RbModel& m, int S, const float* tape, const float* tape_qdd, const float* gq,
                        const float* gqd, float* dq0, float* dqd0, float* dtau, double* dprm, hipStream_t s) {
  const int G = rb_group(m.N), epb = rb::kBlock / G;
  const dim3 grid((m.E + epb - 1) / epb), block(rb::kBlock);
  switch (G) {
    case 8: rb::k_rb_backward<8><<<grid, block, 0, s>>>(m, S, tape, tape_qdd, gq, gqd, dq0, dqd0, dtau, dprm); break;
    case 16: rb::k_rb_backward<16><<<grid, block, 0, s>>>(m, S, tape, tape_qdd, gq, gqd, dq0, dqd0, dtau, dprm); break;
    case 32: rb::k_rb_backward<32><<<grid, block, 0, s>>>(m, S, tape, tape_qdd, gq, gqd, dq0, dqd0, dtau, dprm); break;
    default: rb::k_rb_backward<64><<<grid, block, 0, s>>>(m, S, tape, tape_qdd, gq, gqd, dq0, dqd0, dtau, dprm); break;
  }
}

}  // namespace mpmx
