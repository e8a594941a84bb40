// Tetrahedral FEM with activations (Appendix D.2): rest data, the batched
// forward substeps and their reverse-mode adjoint.
//
// One block per environment. Each substep is an element pass (stress and the
// element's node forces, written to LDS) and a node pass that sums them -- no
// atomics, so the result does not depend on the schedule. A thread keeps its
// elements' rest data and its nodes' state in registers; LDS holds the nodes'
// values for the elements (128-bit entries) and the element forces for the
// nodes. A substep touches HBM only for the activations and the tape.
//
// Nodes are taken in order of their element count (a wave's lanes run equally
// long), and an element writes each corner's force into that node's own row
// of slots: the node adds up one contiguous row in incidence order, with
// nothing to look up. Rows have an odd pitch, so rows of neighbouring lanes
// with the same element count never share a bank: for the 199-node, 480-element
// jumper the node sums' LDS reads go through in 86 bank cycles per component where rows
// in node order without padding took 388, over 46 wave iterations instead of 80.
//
// Bound by instruction issue (the ALUs busy 82% of the time in the forward
// pass, 68% in the adjoint, whose 165 registers leave three blocks per CU; its LDS is busy
// 51%). 4096 jumpers, 80 substeps, forward / adjoint: 2433 / 5200 us when the
// nodes looked up their incidences (ALUs 74% and LDS 72% busy in the forward pass, a third of that
// bank conflicts), 1251 / 2620 now; 48 jumpers: 474 / 860 us, then 173 / 307. With
// 512 threads per block and one element each the batch takes 1561 / 2939 us, with
// registers held to five and four blocks per CU 1621 / 3786. (K = B B^T in place of
// B would spare a third of the products, but rounds the elastic forces, a
// difference of nearly equal terms, more coarsely.)
#include <hip/hip_runtime.h>

#include "fem_kernels.h"
#include "mpm_device.h"

namespace mpmx {

namespace fem {

MD float3 ld3(const float* p) { return make_float3(p[0], p[1], p[2]); }
MD float3 sub3(float3 a, float3 b) { return make_float3(a.x - b.x, a.y - b.y, a.z - b.z); }
MD float3 cross3f(float3 a, float3 b) {
  return make_float3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
MD float dot3f(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// matrix with columns a, b, c
MD M3 from_cols(float3 a, float3 b, float3 c) {
  M3 r;
  r.m[0][0] = a.x; r.m[1][0] = a.y; r.m[2][0] = a.z;
  r.m[0][1] = b.x; r.m[1][1] = b.y; r.m[2][1] = b.z;
  r.m[0][2] = c.x; r.m[1][2] = c.y; r.m[2][2] = c.z;
  return r;
}
MD float3 col(const M3& A, int j) { return make_float3(A.m[0][j], A.m[1][j], A.m[2][j]); }
MD float ddot(const M3& A, const M3& B) {
  float s = 0.f;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) s = fmaf(A.m[i][j], B.m[i][j], s);
  return s;
}
// cof(F) = dJ/dF: column j is the cross product of the next two columns of F (cyclically)
MD M3 cofactor(const M3& F) {
  const float3 f0 = col(F, 0), f1 = col(F, 1), f2 = col(F, 2);
  return from_cols(cross3f(f1, f2), cross3f(f2, f0), cross3f(f0, f1));
}
// directional derivative of cof at F along G
MD M3 dcofactor(const M3& F, const M3& G) {
  const float3 f0 = col(F, 0), f1 = col(F, 1), f2 = col(F, 2);
  const float3 g0 = col(G, 0), g1 = col(G, 1), g2 = col(G, 2);
  const float3 a = cross3f(g1, f2), b = cross3f(f1, g2);
  const float3 c = cross3f(g2, f0), d = cross3f(f2, g0);
  const float3 p = cross3f(g0, f1), q = cross3f(f0, g1);
  return from_cols(make_float3(a.x + b.x, a.y + b.y, a.z + b.z), make_float3(c.x + d.x, c.y + d.y, c.z + d.z),
                   make_float3(p.x + q.x, p.y + q.y, p.z + q.z));
}

MD float3 add3(float3 a, float3 b) { return make_float3(a.x + b.x, a.y + b.y, a.z + b.z); }

struct Prm {
  float mu, lam, rho, damp, ke, kd, kf, zg, alpha;
};
MD Prm load_prm(const float* p) {
  Prm r;
  r.mu = p[0]; r.lam = p[1]; r.rho = p[2]; r.damp = p[3];
  r.ke = p[4]; r.kd = p[5]; r.kf = p[6]; r.zg = p[7];
  r.alpha = 1.f + 0.75f * r.mu / r.lam;
  return r;
}

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

// LDS of the blocks (n nodes, P slots): the forward block's nodes are {x, y, z, v_x} [n] and {v_y, v_z} [n],
// the backward block's {x, y, z, u_x} [n], {v, u_y} [n] and u_z [n] (u: the force cotangent dt/m vbar_tot);
// then 3 floats per slot
struct FwdLds {
  f4* a;
  f2* b;
  float* slot;
};
MD FwdLds fwd_lds(f4* base, int n) {
  FwdLds L;
  L.a = base;
  L.b = reinterpret_cast<f2*>(base + n);
  L.slot = reinterpret_cast<float*>(L.b + n);
  return L;
}
struct BwdLds {
  f4 *a, *b;
  float *uz, *slot;
};
MD BwdLds bwd_lds(f4* base, int n) {
  BwdLds L;
  L.a = base;
  L.b = base + n;
  L.uz = reinterpret_cast<float*>(base + 2 * n);
  L.slot = L.uz + n;
  return L;
}

// element data a thread keeps for the whole launch: corners' nodes and slots, B, volume
template <int TPT>
struct OwnTets {
  ushort4 t[TPT], s[TPT];
  M3 B[TPT];
  float W[TPT];
};
template <int TPT>
MD void load_own_tets(const FemMesh& m, int e, OwnTets<TPT>& o) {
#pragma unroll
  for (int q = 0; q < TPT; ++q) {
    const int t = threadIdx.x + q * kFemThreads;
    if (t >= m.T) continue;   // never used
    o.t[q] = m.ptets[t];
    o.s[q] = m.slots[t];
    const float* b = m.Bm + ((int64_t)e * m.T + t) * 9;
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) o.B[q].m[i][j] = b[3 * i + j];
    o.W[q] = m.W[(int64_t)e * m.T + t];
  }
}

// a thread's nodes (places threadIdx.x + q * kFemThreads in the kernels' order)
template <int NPT>
struct OwnNodes {
  int id[NPT], row[NPT], deg[NPT];   // the mesh's node, its first slot and how many it has
  float w[NPT];                      // lumped volume
};
template <int NPT>
MD void load_own_nodes(const FemMesh& m, int e, OwnNodes<NPT>& o) {
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int p = threadIdx.x + q * kFemThreads;
    o.id[q] = o.row[q] = o.deg[q] = 0;
    o.w[q] = 1.f;
    if (p >= m.n) continue;
    const int4 r = m.rows[p];
    o.id[q] = r.x;
    o.row[q] = 3 * r.y;
    o.deg[q] = r.z;
    o.w[q] = m.wm[(int64_t)e * m.n + r.x];
  }
}

MD void put_slot(float* slot, int s, float3 f) {
  slot[3 * s] = f.x;
  slot[3 * s + 1] = f.y;
  slot[3 * s + 2] = f.z;
}
// the columns of an element go to corners 1..3, minus their sum to corner 0 (of the columns as they are
// rounded, so no part of the sum may be fused with what made them)
MD void put_corners(float* slot, ushort4 s, float3 h0, float3 h1, float3 h2) {
#pragma clang fp contract(off)
  put_slot(slot, s.x, make_float3(-(h0.x + h1.x + h2.x), -(h0.y + h1.y + h2.y), -(h0.z + h1.z + h2.z)));
  put_slot(slot, s.y, h0);
  put_slot(slot, s.z, h1);
  put_slot(slot, s.w, h2);
}
// sum of a node's slots in incidence order, two reads in flight
MD float3 sum_row(const float* h, int deg) {
  float3 s = make_float3(0.f, 0.f, 0.f);
  int k = 0;
  for (; k + 1 < deg; k += 2, h += 6) {
    const float3 a = ld3(h), b = ld3(h + 3);
    s.x += a.x; s.y += a.y; s.z += a.z;
    s.x += b.x; s.y += b.y; s.z += b.z;
  }
  if (k < deg) s = add3(s, ld3(h));
  return s;
}

// ----------------------------------------------------------------------------
// rest data
// ----------------------------------------------------------------------------
__global__ void k_fem_rest(FemMesh m, const float* __restrict__ X, float* __restrict__ Bm, float* __restrict__ W,
                           int32_t* __restrict__ bad) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)m.E * m.T) return;
  const int e = (int)(id / m.T), t = (int)(id - (int64_t)e * m.T);
  const int4 tt = m.tets[t];
  const float* Xe = X + (int64_t)e * m.n * 3;
  const float3 x0 = ld3(Xe + 3 * tt.x);
  const float3 d0 = sub3(ld3(Xe + 3 * tt.y), x0), d1 = sub3(ld3(Xe + 3 * tt.z), x0), d2 = sub3(ld3(Xe + 3 * tt.w), x0);
  const float3 c12 = cross3f(d1, d2), c20 = cross3f(d2, d0), c01 = cross3f(d0, d1);
  const float det = dot3f(d0, c12);
  // longest edge: the three from node 0 and the three between the others
  float L2 = fmaxf(fmaxf(dot3f(d0, d0), dot3f(d1, d1)), dot3f(d2, d2));
  const float3 e01 = sub3(d1, d0), e02 = sub3(d2, d0), e12 = sub3(d2, d1);
  L2 = fmaxf(L2, fmaxf(fmaxf(dot3f(e01, e01), dot3f(e02, e02)), dot3f(e12, e12)));
  const float L3 = L2 * sqrtf(L2);
  if (!(fabsf(det) >= 1e-9f * L3) || !isfinite(det)) {
    atomicOr(bad, 1);
    return;
  }
  // rows of D^-1 are the cross products of the other two columns over det
  const float inv = 1.f / det;
  float* b = Bm + id * 9;
  b[0] = c12.x * inv; b[1] = c12.y * inv; b[2] = c12.z * inv;
  b[3] = c20.x * inv; b[4] = c20.y * inv; b[5] = c20.z * inv;
  b[6] = c01.x * inv; b[7] = c01.y * inv; b[8] = c01.z * inv;
  W[id] = fabsf(det) * (1.f / 6.f);
}

__global__ void k_fem_lumped(FemMesh m, const float* __restrict__ W, float* __restrict__ wm) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)m.E * m.n) return;
  const int e = (int)(id / m.n), i = (int)(id - (int64_t)e * m.n);
  float s = 0.f;
  for (int q = m.inc_off[i]; q < m.inc_off[i + 1]; ++q) s += W[(int64_t)e * m.T + (m.inc[q] >> 2)];
  wm[id] = 0.25f * s;
}

// ----------------------------------------------------------------------------
// forward
// ----------------------------------------------------------------------------
template <int TPT, int NPT>
__global__ void __launch_bounds__(kFemThreads) k_fem_forward(FemMesh m, int S, float* __restrict__ x,
                                                             float* __restrict__ v, const float* __restrict__ act,
                                                             float* __restrict__ tape,
                                                             float* __restrict__ tape_act, int32_t* __restrict__ errs) {
  extern __shared__ f4 fem_lds[];
  const int e = blockIdx.x, n = m.n, T = m.T, E = m.E;
  const FwdLds L = fwd_lds(fem_lds, n);
  const Prm p = load_prm(m.prm + (int64_t)e * kFemPrm);
  OwnTets<TPT> own;
  load_own_tets<TPT>(m, e, own);
  OwnNodes<NPT> nod;
  load_own_nodes<NPT>(m, e, nod);
  float3 xs[NPT], vs[NPT];
  float im[NPT];
  // state of the thread's nodes to LDS, and to the tape as substep k's (six planes of n per env)
  auto publish = [&](int q, int k) {
    const int i = threadIdx.x + q * kFemThreads;
    L.a[i] = f4{xs[q].x, xs[q].y, xs[q].z, vs[q].x};
    L.b[i] = f2{vs[q].y, vs[q].z};
    if (tape) {
      float* o = tape + ((int64_t)k * E + e) * 6 * n + i;
      o[0] = xs[q].x; o[n] = xs[q].y; o[2 * n] = xs[q].z;
      o[3 * n] = vs[q].x; o[4 * n] = vs[q].y; o[5 * n] = vs[q].z;
    }
  };
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    if ((int)threadIdx.x + q * kFemThreads >= n) continue;
    const int64_t at = ((int64_t)e * n + nod.id[q]) * 3;
    xs[q] = ld3(x + at);
    vs[q] = ld3(v + at);
    im[q] = 1.f / (p.rho * nod.w[q]);
    publish(q, 0);
  }
  float an[TPT];   // activations of the next substep, read one ahead
  auto prefetch = [&](int k) {
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * kFemThreads;
      an[q] = act && k < S && t < T ? act[((int64_t)k * E + e) * T + t] : 0.f;
    }
  };
  prefetch(0);
  __syncthreads();
  for (int k = 0; k < S; ++k) {
    float ak[TPT];
#pragma unroll
    for (int q = 0; q < TPT; ++q) ak[q] = an[q];
    prefetch(k + 1);
    // element pass: the forces -W P B^T on corners 1..3
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * kFemThreads;
      if (t >= T) continue;
      const float a = ak[q];
      if (tape_act) tape_act[((int64_t)k * E + e) * T + t] = a;
      const f4 a0 = L.a[own.t[q].x], a1 = L.a[own.t[q].y], a2 = L.a[own.t[q].z], a3 = L.a[own.t[q].w];
      const f2 b0 = L.b[own.t[q].x], b1 = L.b[own.t[q].y], b2 = L.b[own.t[q].z], b3 = L.b[own.t[q].w];
      const float3 x0 = make_float3(a0[0], a0[1], a0[2]), v0 = make_float3(a0[3], b0[0], b0[1]);
      const M3 D = from_cols(sub3(make_float3(a1[0], a1[1], a1[2]), x0), sub3(make_float3(a2[0], a2[1], a2[2]), x0),
                             sub3(make_float3(a3[0], a3[1], a3[2]), x0));
      const M3 V = from_cols(sub3(make_float3(a1[3], b1[0], b1[1]), v0), sub3(make_float3(a2[3], b2[0], b2[1]), v0),
                             sub3(make_float3(a3[3], b3[0], b3[1]), v0));
      const M3 F = m3_mul(D, own.B[q]);
      const M3 Fd = m3_mul(V, own.B[q]);
      const float Ic = ddot(F, F);
      const float J = m3_det(F);
      const float s = p.mu * (1.f - 1.f / (Ic + 1.f));
      const float r = p.lam * (J - p.alpha - a);
      const M3 cof = cofactor(F);
      M3 P;
      for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) P.m[i][j] = fmaf(s, F.m[i][j], fmaf(r, cof.m[i][j], p.damp * Fd.m[i][j]));
      const M3 H = m3_mul_abt(P, own.B[q]);   // P B_m^T
      float3 h[3];
      for (int c = 0; c < 3; ++c)
        h[c] = make_float3(-own.W[q] * H.m[0][c], -own.W[q] * H.m[1][c], -own.W[q] * H.m[2][c]);
      put_corners(L.slot, own.s[q], h[0], h[1], h[2]);
    }
    __syncthreads();
    // node pass: sum, ground contact, semi-implicit Euler
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      if ((int)threadIdx.x + q * kFemThreads >= n) continue;
      float3 f = sum_row(L.slot + nod.row[q], nod.deg[q]);
      const float3 xi = xs[q], vi = vs[q];
      if (xi.z < p.zg) {
        f.x -= p.kf * vi.x;
        f.y -= p.kf * vi.y;
        f.z += p.ke * (p.zg - xi.z) - p.kd * vi.z;
      }
      const float3 vn = make_float3(vi.x + m.dt * (f.x * im[q] + m.g[0]), vi.y + m.dt * (f.y * im[q] + m.g[1]),
                                    vi.z + m.dt * (f.z * im[q] + m.g[2]));
      vs[q] = vn;
      xs[q] = make_float3(xi.x + m.dt * vn.x, xi.y + m.dt * vn.y, xi.z + m.dt * vn.z);
      publish(q, k + 1);
    }
    __syncthreads();
  }
  bool finite = true;
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    if ((int)threadIdx.x + q * kFemThreads >= n) continue;
    const int64_t at = ((int64_t)e * n + nod.id[q]) * 3;
    x[at] = xs[q].x; x[at + 1] = xs[q].y; x[at + 2] = xs[q].z;
    v[at] = vs[q].x; v[at + 1] = vs[q].y; v[at + 2] = vs[q].z;
    finite = finite && isfinite(xs[q].x) && isfinite(xs[q].y) && isfinite(xs[q].z) && isfinite(vs[q].x) &&
             isfinite(vs[q].y) && isfinite(vs[q].z);
  }
  if (!finite) atomicOr(&errs[e], 1);
}

// ----------------------------------------------------------------------------
// backward
// ----------------------------------------------------------------------------
template <int TPT, int NPT>
__global__ void __launch_bounds__(kFemThreads) k_fem_backward(FemMesh m, int S, const float* __restrict__ tape,
                                                              const float* __restrict__ tape_act,
                                                              const float* __restrict__ gx,
                                                              const float* __restrict__ gv, float* __restrict__ dx0,
                                                              float* __restrict__ dv0, float* __restrict__ dact,
                                                              double* __restrict__ dprm) {
  extern __shared__ f4 fem_lds[];
  __shared__ double red[kFemThreads / 64][8];
  const int e = blockIdx.x, n = m.n, T = m.T, E = m.E;
  const BwdLds L = bwd_lds(fem_lds, n);
  const Prm p = load_prm(m.prm + (int64_t)e * kFemPrm);
  OwnTets<TPT> own;
  load_own_tets<TPT>(m, e, own);
  OwnNodes<NPT> nod;
  load_own_nodes<NPT>(m, e, nod);
  // cotangents of the thread's nodes
  float3 xb[NPT], vb[NPT];
  float cm[NPT];
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    xb[q] = vb[q] = make_float3(0.f, 0.f, 0.f);
    cm[q] = m.dt / (p.rho * nod.w[q]);
    if ((int)threadIdx.x + q * kFemThreads >= n) continue;
    const int64_t at = ((int64_t)e * n + nod.id[q]) * 3;
    if (gx) xb[q] = ld3(gx + at);
    if (gv) vb[q] = ld3(gv + at);
  }
  // per-thread parameter cotangents: mu, lam, damp, k_e, k_d, k_f, z_g
  float pmu = 0.f, plam = 0.f, pdamp = 0.f, pke = 0.f, pkd = 0.f, pkf = 0.f, pzg = 0.f;
  // the tape rows of this thread's nodes and elements for the next substep, read one substep ahead
  float pf[NPT][6], an[TPT];
  auto prefetch = [&](int k) {
    if (k < 0) return;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int i = threadIdx.x + q * kFemThreads;
      if (i < n) {
        const float* st = tape + ((int64_t)k * E + e) * 6 * n + i;
        for (int c = 0; c < 6; ++c) pf[q][c] = st[c * n];
      }
    }
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * kFemThreads;
      if (t < T) an[q] = tape_act[((int64_t)k * E + e) * T + t];
    }
  };
  prefetch(S - 1);
  for (int k = S - 1; k >= 0; --k) {
    // node pass 1: state k from the tape; vbar_tot = vbar' + dt xbar'; u = dt/m vbar_tot (the force
    // cotangent); ground-contact terms
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      const int i = threadIdx.x + q * kFemThreads;
      if (i >= n) continue;
      const float3 xi = make_float3(pf[q][0], pf[q][1], pf[q][2]);
      const float3 vi = make_float3(pf[q][3], pf[q][4], pf[q][5]);
      vb[q] = make_float3(fmaf(m.dt, xb[q].x, vb[q].x), fmaf(m.dt, xb[q].y, vb[q].y), fmaf(m.dt, xb[q].z, vb[q].z));
      const float3 u = make_float3(cm[q] * vb[q].x, cm[q] * vb[q].y, cm[q] * vb[q].z);
      L.a[i] = f4{xi.x, xi.y, xi.z, u.x};
      L.b[i] = f4{vi.x, vi.y, vi.z, u.y};
      L.uz[i] = u.z;
      if (xi.z < p.zg) {
        xb[q].z -= p.ke * u.z;
        vb[q].z -= p.kd * u.z;
        vb[q].x -= p.kf * u.x;
        vb[q].y -= p.kf * u.y;
        pke = fmaf(p.zg - xi.z, u.z, pke);
        pkd = fmaf(-vi.z, u.z, pkd);
        pkf -= vi.x * u.x + vi.y * u.y;
        pzg = fmaf(p.ke, u.z, pzg);
      }
    }
    float ak[TPT];
#pragma unroll
    for (int q = 0; q < TPT; ++q) ak[q] = an[q];
    prefetch(k - 1);   // in flight during the element pass
    __syncthreads();
    // element pass: with G = U B, the element's share of the loss is -W P : G; its cotangents are
    // Fbar = -W dP[G] (the energy Hessian is symmetric), Fdot_bar = -W damp G, and the activation's
    // W lam cof(F) : G
    M3 dvb[TPT];   // the V cotangent columns wait in registers for the second sum
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * kFemThreads;
      if (t >= T) continue;
      const float a = ak[q];
      M3 D, V, U;
      {
        const ushort4 tt = own.t[q];
        const f4 a0 = L.a[tt.x], b0 = L.b[tt.x];
        const float z0 = L.uz[tt.x];
        const int ids[3] = {tt.y, tt.z, tt.w};
        for (int c = 0; c < 3; ++c) {
          const f4 ac = L.a[ids[c]] - a0, bc = L.b[ids[c]] - b0;
          for (int i = 0; i < 3; ++i) {
            D.m[i][c] = ac[i];
            V.m[i][c] = bc[i];
          }
          U.m[0][c] = ac[3];
          U.m[1][c] = bc[3];
          U.m[2][c] = L.uz[ids[c]] - z0;
        }
      }
      const M3 B = own.B[q];
      const float Wt = own.W[q];
      const M3 F = m3_mul(D, B);
      const M3 G = m3_mul(U, B);
      const float Ic = ddot(F, F);
      const float J = m3_det(F);
      const float ic1 = 1.f / (Ic + 1.f);
      const float s = p.mu * (1.f - ic1);
      const float r = p.lam * (J - p.alpha - a);
      const M3 cof = cofactor(F);
      const M3 dcof = dcofactor(F, G);
      const float FG = ddot(F, G), cG = ddot(cof, G);
      const float c2 = 2.f * p.mu * ic1 * ic1 * FG;
      M3 Fb;
      for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
          const float dP = fmaf(s, G.m[i][j], fmaf(c2, F.m[i][j], fmaf(p.lam * cG, cof.m[i][j], r * dcof.m[i][j])));
          Fb.m[i][j] = -Wt * dP;
        }
      const M3 Dsb = m3_mul_abt(Fb, B), Q = m3_mul_abt(G, B);
      dvb[q] = m3_scale(Q, -Wt * p.damp);
      put_corners(L.slot, own.s[q], col(Dsb, 0), col(Dsb, 1), col(Dsb, 2));
      if (dact) dact[((int64_t)k * E + e) * T + t] = Wt * p.lam * cG;
      pmu -= Wt * ((1.f - ic1) * FG - 0.75f * cG);
      plam -= Wt * (J - p.alpha - a + 0.75f * p.mu / p.lam) * cG;
      pdamp -= Wt * ddot(V, Q);   // F' : G = V : G B^T
    }
    __syncthreads();
    // node pass 2: the element cotangents summed onto the nodes give the cotangent of state k, the
    // D columns first, then (through the same slots) the V columns
#pragma unroll
    for (int q = 0; q < NPT; ++q)
      if ((int)threadIdx.x + q * kFemThreads < n) xb[q] = add3(xb[q], sum_row(L.slot + nod.row[q], nod.deg[q]));
    __syncthreads();
#pragma unroll
    for (int q = 0; q < TPT; ++q)
      if ((int)threadIdx.x + q * kFemThreads < T) put_corners(L.slot, own.s[q], col(dvb[q], 0), col(dvb[q], 1), col(dvb[q], 2));
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NPT; ++q)
      if ((int)threadIdx.x + q * kFemThreads < n) vb[q] = add3(vb[q], sum_row(L.slot + nod.row[q], nod.deg[q]));
    // the next iteration's node pass 1 writes what the elements read before the last two barriers, and its
    // element pass, which writes the slots, starts after another, so no barrier is needed here
  }
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    if ((int)threadIdx.x + q * kFemThreads >= n) continue;
    const int64_t at = ((int64_t)e * n + nod.id[q]) * 3;
    dx0[at] = xb[q].x; dx0[at + 1] = xb[q].y; dx0[at + 2] = xb[q].z;
    dv0[at] = vb[q].x; dv0[at + 1] = vb[q].y; dv0[at + 2] = vb[q].z;
  }
  if (!dprm) return;
  // block sums of the parameter cotangents in FP64
  double part[7] = {pmu, plam, pdamp, pke, pkd, pkf, pzg};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c = 0; c < 7; ++c) {
    double vsum = part[c];
    for (int off = 32; off > 0; off >>= 1) vsum += __shfl_down(vsum, off);
    if (lane == 0) red[wave][c] = vsum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot[7];
    for (int c = 0; c < 7; ++c) {
      tot[c] = 0.0;
      for (int w = 0; w < kFemThreads / 64; ++w) tot[c] += red[w][c];
    }
    const float* pr = m.prm + (int64_t)e * kFemPrm;
    // rho dL/drho = -(mu dL/dmu + lam dL/dlam + damp dL/ddamp + k_e dL/dk_e + k_d dL/dk_d + k_f dL/dk_f)
    const double scaled = (double)pr[0] * tot[0] + (double)pr[1] * tot[1] + (double)pr[3] * tot[2] +
                          (double)pr[4] * tot[3] + (double)pr[5] * tot[4] + (double)pr[6] * tot[5];
    double* o = dprm + (int64_t)e * kFemPrm;
    o[0] = tot[0];
    o[1] = tot[1];
    o[2] = -scaled / (double)pr[2];
    o[3] = tot[2];
    o[4] = tot[3];
    o[5] = tot[4];
    o[6] = tot[5];
    o[7] = tot[6];
  }
}

// dynamic LDS above 64 KiB has to be allowed per kernel
template <typename K>
void allow_lds(K kernel, size_t bytes) {
  if (bytes > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace fem

using namespace fem;

size_t fem_forward_lds(int n, int P) { return sizeof(float) * (size_t)(6 * n + 3 * P); }
size_t fem_backward_lds(int n, int P) { return sizeof(float) * (size_t)(9 * n + 3 * P); }

void launch_fem_rest(const FemMesh& m, const float* X, float* Bm, float* W, float* wm, int32_t* bad,
                     hipStream_t s) {
  const int64_t nt = (int64_t)m.E * m.T, nn = (int64_t)m.E * m.n;
  hipLaunchKernelGGL(k_fem_rest, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, m, X, Bm, W, bad);
  hipLaunchKernelGGL(k_fem_lumped, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, m, W, wm);
}

// the instance whose threads hold 1, 2 or 4 elements and 1 or 2 nodes
#define MPMX_FEM_BY_SIZE(L)                             \
  if (m.n <= kFemThreads) {                             \
    if (m.T <= kFemThreads) { L(1, 1); }                \
    else if (m.T <= 2 * kFemThreads) { L(2, 1); }       \
    else { L(4, 1); }                                   \
  } else {                                              \
    if (m.T <= kFemThreads) { L(1, 2); }                \
    else if (m.T <= 2 * kFemThreads) { L(2, 2); }       \
    else { L(4, 2); }                                   \
  }

void launch_fem_forward(const FemMesh& m, int S, float* x, float* v, const float* act, float* tape,
                        float* tape_act, int32_t* errs, hipStream_t s) {
  const size_t lds = fem_forward_lds(m.n, m.P);
#define L(T, N)                               \
  allow_lds(k_fem_forward<T, N>, lds);        \
  hipLaunchKernelGGL((k_fem_forward<T, N>), dim3(m.E), dim3(kFemThreads), lds, s, m, S, x, v, act, tape, tape_act, errs)
  MPMX_FEM_BY_SIZE(L)
#undef L
}

void launch_fem_backward(const FemMesh& m, int S, const float* tape, const float* tape_act, const float* gx,
                         const float* gv, float* dx0, float* dv0, float* dact, double* dprm, hipStream_t s) {
  const size_t lds = fem_backward_lds(m.n, m.P);
#define L(T, N)                               \
  allow_lds(k_fem_backward<T, N>, lds);       \
  hipLaunchKernelGGL((k_fem_backward<T, N>), dim3(m.E), dim3(kFemThreads), lds, s, m, S, tape, tape_act, gx, gv, dx0, dv0, dact, dprm)
  MPMX_FEM_BY_SIZE(L)
#undef L
}

}  // namespace mpmx
