// Particle kernels of the batched mode: gathers straight from the grid, and
// scatters summed per column of base cells in LDS.
//
// A block takes one work item, up to 256 particles of one environment that are
// contiguous in (tile, cell) order, thread t <-> particle t. Both scatters of
// the method (P2G, and the grid-velocity cotangents of the G2P adjoint) add to
// node base + o the value W(o) (g + A (o - f)) of the particle, and W(o) times
// the mass for the P2G. No float atomics touch LDS: ds_add_f32 runs at 193
// cycles per wave instruction here whether or not lanes collide (an integer
// add takes 5, a 128-bit read 6 to 15), so a block of 256 particles that pushed
// one cell's 27 x 4 sums with them spent 13,000 cycles on it. Instead
//  1. the block finds the tile rows its particles lie in and their boxes of
//     nodes, and counting-sorts its particles by current stencil base (integer atomics);
//  2. each particle stores a 17-float payload at its sorted position;
//  3. a thread owns a (column of base cells, z node) and sums the particles of
//     the column's three cells that reach the node, one contiguous range of
//     the sorted payloads, for the column's nine (x, y) node offsets at once.
//     These tasks are taken in order of their length, so that a wave's lanes
//     run equally long: at one particle per cell a task has 2.7 particles on
//     average but the longest of 64 unsorted ones has 7;
//  4. the nine sums are added to the block's box of nodes in LDS in nine phases
//     of one (x, y) offset each: within a phase no two threads share a node, so
//     plain 128-bit reads and writes do;
//  5. each box node goes to the grid once, four lanes per node.
//
// Measured, us per launch, on 3.2 M water particles (16 envs, 96^3, 0.9 per cell, large
// box), 640,000 corotated (32 envs, 48^3, 8 per cell, small box) and 320,000 von Mises
// (128 envs, 48^3, 8 per cell, small box); before: a scatter per box node or per cell,
// with LDS copies of the grid for the gathers, over a grid stored one channel at a time:
//                 water          corotated      von Mises
//   P2G           353 -> 241     63 -> 52.5     53 -> 34
//   G2P           222 -> 133     25 -> 21.5     20 -> 18.5
//   G2P + P2G     462 -> 289     71 -> 60       63 -> 45
//   G2P adjoint   514 -> 356     71 -> 61       68 -> 48
//   P2G adjoint   326 -> 208     65 -> 43       50 -> 34
//   adjoint pair  749 -> 453     114 -> 88      100 -> 72.5
// What bounds them now: at 8 per cell instruction issue (the vector ALUs are busy 72%
// of a G2P + P2G and 78% of a pair, the rest is the scatter's chain of barriers); at
// one per cell the box flush, 2.75 million 64-byte lines of global atomics per
// launch at the chip's 20 per ns, 137 us, which the rest overlaps in part.
#include "mpm_kernels.h"

namespace mpmx {

constexpr int kItem = kItemSize;
constexpr int kMaxRuns = 8;        // tile rows per block that get their own box
constexpr int kWaveRows = 8;       // candidates a wave may list for them
constexpr int kBins = 8;           // task lengths told apart
// Box budgets in nodes (a block with more takes several passes over slabs of z)
// and room for base cells (a block with more adds to the grid directly). The
// larger pair leaves four blocks per CU (LDS) and holds a box of 28 z nodes
// across a whole tile row. The smaller one with its 96 VGPRs leaves five (32,000
// bytes of LDS is the most for that) to all but the adjoint pair, whose 128 VGPRs
// allow four: the scatter's barriers and LDS chains want the fifth where the boxes
// fit. From large to small, us: P2G and G2P + P2G of 640,000 corotated particles (32
// envs, 48^3, 8 per cell) 56 -> 52.5 and 64 -> 60, of 320,000 von Mises (128 envs,
// 48^3, 8 per cell) 41 -> 34 and 51 -> 45; where they do not fit, at one particle per
// cell, the second pass costs more: 3.2 M water particles (16 envs, 96^3) 241 -> 258
// and 288 -> 294. The G2P adjoint follows its registers too: water 357 -> 336,
// corotated 65 -> 62, but a batch of three materials 252 -> 267 (its von Mises form
// spills). The pair differs by spills and passes alone: water 449 -> 467, the others
// within 1%. (384 nodes with six blocks lost to one of the two at each of these.)
// The autotuner measures both and takes one for all four kernels.
constexpr int kBoxLarge = 1024;
constexpr int kBoxSmall = 640;
template <int BOXN>
constexpr int col_cells() { return BOXN; }
template <int BOXN>
constexpr int waves_per_simd() { return BOXN == kBoxLarge ? 4 : 5; }

// whole-wavefront sum (DPP, device library)
extern "C" __device__ __attribute__((const)) float __ockl_wfred_add_f32(float);

// smallest of each 16-bit half over the wavefront
typedef short short2v __attribute__((ext_vector_type(2)));
template <int CTRL, int ROWS>
MD int pk_min_dpp(int x) {
  const int y = __builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xf, false);
  const short2v m = __builtin_elementwise_min(__builtin_bit_cast(short2v, x), __builtin_bit_cast(short2v, y));
  return __builtin_bit_cast(int, m);
}
MD int wave_pk_min(int x) {
  x = pk_min_dpp<0xB1, 0xf>(x);    // quad_perm [1, 0, 3, 2]
  x = pk_min_dpp<0x4E, 0xf>(x);    // quad_perm [2, 3, 0, 1]
  x = pk_min_dpp<0x124, 0xf>(x);   // row_ror 4 and 8: all 16 lanes of a row
  x = pk_min_dpp<0x128, 0xf>(x);
  x = pk_min_dpp<0x142, 0xa>(x);   // row_bcast 15: rows 1 and 3 take in rows 0 and 2
  x = pk_min_dpp<0x143, 0xc>(x);   // row_bcast 31: rows 2 and 3 take in row 1
  return __builtin_amdgcn_readlane(x, 63);
}

// the block's runs (distinct tile rows): boxes of nodes, base cells and (base
// column, z node) tasks, each concatenated over the runs. A run lies in one tile
// row, so it has at most 4 x 4 columns of base cells and 6 x 6 of nodes.
struct Runs {
  int last[4], wsum[4];               // per wave: its last particle's tile row; row changes in it
  int rows[4][kWaveRows];             // per wave: the tile row after each change
  int cols[kMaxRuns], zmin[kMaxRuns], zmax[kMaxRuns];   // base columns in use (x bits 0-3, y 4-7), base z bounds
  int lo[kMaxRuns][3], hi[kMaxRuns][3];   // node bounds (inclusive)
  int ext[kMaxRuns][3];
  int node[kMaxRuns + 1], cell[kMaxRuns + 1], task[kMaxRuns + 1];   // first of each run, then the total
  float inv_z[kMaxRuns], inv_cy[kMaxRuns];   // 1 / ext z, 1 / columns in y
  int n;                              // runs in use
  int occupied;                       // base cells that hold a particle
  int bin[kBins];                     // tasks of each length in this pass
};

template <int BOXN>
struct ColShared {
  float4 box[BOXN];                   // sums of this pass's nodes
  float4 pay[4 * kItem];              // payload row r of sorted position q at pay[r * 256 + q]
  float fz[kItem];                    // f on z of sorted position q
  int start[col_cells<BOXN>() + 1];   // first sorted position of each base cell
  uint16_t list[BOXN * 4 / 9 + 1];    // this pass's tasks that have particles, the longest first
  int wtot[4];
  Runs r;
};

// quotient of 0 <= a < 2^21 by d >= 1 from a float reciprocal of d: (a + 1/2) / d
// lies at least 1/(2d) inside (q, q + 1), and the two roundings (of 1/d and of
// the product) move it by less than (a + 1/2) / d * 2^-23 < 1/(2d)
MD int small_div(int a, float inv_d) { return (int)(((float)a + 0.5f) * inv_d); }

// State and cotangent rows of a block's particles: `base` points at the block's
// first particle (uniform over the block), t is the thread's particle in the
// block, so that each access is one scalar base and the same 32-bit lane offset.
MD void load_x3(const float* __restrict__ base, int64_t N, uint32_t t, float x[3]) {
  x[0] = base[t]; x[1] = (base + N)[t]; x[2] = (base + 2 * N)[t];
}
MD M3 ld_m3(const float* __restrict__ base, int64_t N, uint32_t t, int c0) {
  M3 m;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) m.m[i][j] = (base + (c0 + 3 * i + j) * N)[t];
  return m;
}
MD void st_m3(float* __restrict__ base, int64_t N, uint32_t t, int c0, const M3& m) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) (base + (c0 + 3 * i + j) * N)[t] = m.m[i][j];
}
MD void ld_v3(const float* __restrict__ base, int64_t N, uint32_t t, int c0, float v[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) v[a] = (base + (c0 + a) * N)[t];
}
MD void st_v3(float* __restrict__ base, int64_t N, uint32_t t, int c0, const float v[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) (base + (c0 + a) * N)[t] = v[a];
}
MD void copy_rows(const float* __restrict__ src, float* __restrict__ dst, int64_t N, uint32_t t) {
  for (int c = 0; c < 24; ++c) (dst + c * N)[t] = (src + c * N)[t];
}

// quadratic B-spline weight of node offset o (0, 1, 2) at f = x n - base, and
// its f-derivative: each piece is w = k (f - s)^2 + m, dw/df = 2 k (f - s). For
// a wave-uniform o the constants are scalars and the weight costs three
// instructions, so loops can recompute it instead of holding a table
MD void spline_piece(int o, float f, float& w, float& dw) {
  const float k = o == 1 ? -1.f : 0.5f, sft = o == 0 ? 1.5f : (o == 1 ? 1.f : 0.5f), m = o == 1 ? 0.75f : 0.f;
  const float u = f - sft;
  w = fmaf(k * u, u, m);
  dw = 2.f * k * u;
}

// per-env parameter cotangents of a block: each wave sums its 64 FP32 terms
// with a DPP reduction (a parameter none of its lanes touched costs one
// ballot), the block and the grid accumulate in FP64
MD void block_reduce_params(float pb[PB_COUNT], double* __restrict__ acc) {
  __shared__ double red[PB_COUNT][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < PB_COUNT; ++k) {
    float v = 0.f;
    if (__ballot(pb[k] != 0.f) != 0ull) v = __ockl_wfred_add_f32(pb[k]);
    if (lane == 0) red[k][wave] = (double)v;
  }
  __syncthreads();
  if (threadIdx.x < PB_COUNT) {
    double s = 0.0;
    for (int w = 0; w < 4; ++w) s += red[threadIdx.x][w];
    if (s != 0.0) atomicAdd(&acc[threadIdx.x], s);
  }
}

// ----------------------------------------------------------------------------
// the column scatter
// ----------------------------------------------------------------------------
// Runs, boxes and the counting sort for the block's particles with stencil
// bases b (every thread calls it): pos = this thread's sorted position. False,
// for every thread, if the block's particles lie in more than kMaxRuns tile
// rows or their boxes hold more base cells than there is room for (the caller
// then adds to the grid directly).
template <int BOXN>
MD bool col_index(const EnvDev& e, const int b[3], bool valid, ColShared<BOXN>& S, int& pos) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  Runs& R = S.r;
  for (int i = t; i <= col_cells<BOXN>(); i += kItem) S.start[i] = 0;
  if (t == 0) R.occupied = 0;
  if (t < kMaxRuns) { R.cols[t] = 0; R.zmin[t] = 0x7fff; R.zmax[t] = 0; }
  const int row = valid ? (b[0] >> 2) * e.T + (b[1] >> 2) : -1;
  int prev = __shfl_up(row, 1);
  if (lane == 63) R.last[wave] = row;
  __syncthreads();
  if (lane == 0) prev = wave ? R.last[wave - 1] : -1;
  const bool first = valid && row != prev;   // rows are >= 0
  const uint64_t bal = __ballot(first);
  const int at = __popcll(bal & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
  if (first && at < kWaveRows) R.rows[wave][at] = row;
  if (lane == 0) R.wsum[wave] = __popcll(bal);
  __syncthreads();
  // the distinct rows among the waves' candidates, in the same order in every wave: a particle that left its
  // tile row since the sort makes two changes but at most one more run
  int cand = -1;
  bool over = false;
  if (lane < 4 * kWaveRows) {
    const int c = R.wsum[lane / kWaveRows];
    if (lane % kWaveRows < c) cand = R.rows[lane / kWaveRows][lane % kWaveRows];
    over = c > kWaveRows;
  }
  uint64_t rest = __ballot(cand >= 0);
  int run = -1, nr = 0;
  while (rest != 0ull && nr < kMaxRuns) {
    const int rr = __builtin_amdgcn_readlane(cand, __ffsll((unsigned long long)rest) - 1);
    if (row == rr) run = nr;
    rest &= ~__ballot(cand == rr);
    ++nr;
  }
  if (__ballot(over) != 0ull || rest != 0ull) nr = 0;   // too many: the caller adds to the grid directly
  // bounds of each run: which of its tile row's four columns in x and in y are in use (ballots), and base z
  // (one packed reduction); then integer atomics per wave
  for (int k = 0; k < nr; ++k) {
    const bool mine = run == k;
    const uint64_t of_k = __ballot(mine);
    if (of_k == 0ull) continue;
    int cols = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cols |= __ballot(mine && (b[0] & 3) == j) != 0ull ? 1 << j : 0;
      cols |= __ballot(mine && (b[1] & 3) == j) != 0ull ? 16 << j : 0;
    }
    const int z = wave_pk_min(mine ? (b[2] & 0xffff) | (int)((uint32_t)-b[2] << 16) : 0x7fff7fff);
    const int first_of_k = __ffsll((unsigned long long)of_k) - 1;
    const int tx = __builtin_amdgcn_readlane(b[0], first_of_k) & ~3, ty = __builtin_amdgcn_readlane(b[1], first_of_k) & ~3;
    if (lane == 0) {
      atomicOr(&R.cols[k], cols);
      atomicMin(&R.zmin[k], (int)(short)(z & 0xffff));
      atomicMax(&R.zmax[k], -(z >> 16));
      R.lo[k][0] = tx;   // the same value from every wave: the row's first node; the tight bound follows
      R.lo[k][1] = ty;
    }
  }
  __syncthreads();
  // every thread derives the tables; thread 0 keeps them for the scatter
  int node = 0, cell = 0, task = 0, cid = 0;
  for (int k = 0; k < nr; ++k) {
    const int cols = R.cols[k], cx = cols & 15, cy = (cols >> 4) & 15;
    const int lo[3] = {R.lo[k][0] + __ffs(cx) - 1, R.lo[k][1] + __ffs(cy) - 1, R.zmin[k]};
    const int ext[3] = {32 - __clz(cx) - __ffs(cx) + 3, 32 - __clz(cy) - __ffs(cy) + 3, R.zmax[k] - lo[2] + 3};
    if (run == k) cid = cell + ((b[0] - lo[0]) * (ext[1] - 2) + (b[1] - lo[1])) * (ext[2] - 2) + (b[2] - lo[2]);
    if (t == 0) {
      R.node[k] = node; R.cell[k] = cell; R.task[k] = task;
      for (int a = 0; a < 3; ++a) { R.ext[k][a] = ext[a]; R.hi[k][a] = lo[a] + ext[a] - 1; }
      R.inv_z[k] = 1.f / (float)ext[2];
      R.inv_cy[k] = 1.f / (float)(ext[1] - 2);
    }
    const int columns = (ext[0] - 2) * (ext[1] - 2);
    node += ext[0] * ext[1] * ext[2];
    cell += columns * (ext[2] - 2);
    task += columns * ext[2];
  }
  if (t == 0) { R.node[nr] = node; R.cell[nr] = cell; R.task[nr] = task; R.n = nr; }
  if (nr == 0 || cell > col_cells<BOXN>()) return false;
  int rank = 0;
  if (valid) rank = atomicAdd(&S.start[cid + 1], 1);   // counts one cell up: the inclusive scan makes start[] exclusive
  const uint64_t firsts = __ballot(valid && rank == 0);
  if (lane == 0) atomicAdd(&R.occupied, (int)__popcll(firsts));
  __syncthreads();
  if (t < kMaxRuns * 3 && t / 3 < nr) R.lo[t / 3][t % 3] = R.hi[t / 3][t % 3] - R.ext[t / 3][t % 3] + 1;   // the tight bounds
  // block-wide inclusive prefix sum of start[0, cell]
  const int n = cell + 1, per = (n + kItem - 1) / kItem;
  const int i0 = min(t * per, n), i1 = min(i0 + per, n);
  int s = 0;
  for (int i = i0; i < i1; ++i) { s += S.start[i]; S.start[i] = s; }
  int x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) S.wtot[wave] = x;
  __syncthreads();
  int off = x - s;
  for (int w = 0; w < wave; ++w) off += S.wtot[w];
  for (int i = i0; i < i1; ++i) S.start[i] += off;
  __syncthreads();
  pos = valid ? S.start[cid] + rank : 0;
  return true;
}

// payload of a particle with value g + A (o - f) at node offset o: the first and
// last x and y weights, the value at (1, 1, f_z), the columns of A, and f_z; in
// rows strided by 256 particles so that lanes reading different particles' rows
// spread over the LDS banks
template <int BOXN>
MD void col_store(ColShared<BOXN>& S, int q, const Stencil& sc, const float g[3], const float A[3][3]) {
  const float d0 = 1.f - sc.f[0], d1 = 1.f - sc.f[1];
  float c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) c[a] = fmaf(A[a][0], d0, fmaf(A[a][1], d1, g[a]));
  S.pay[q] = make_float4(sc.w[0][0], sc.w[0][2], sc.w[1][0], sc.w[1][2]);
  S.pay[kItem + q] = make_float4(c[0], c[1], c[2], A[0][0]);
  S.pay[2 * kItem + q] = make_float4(A[1][0], A[2][0], A[0][1], A[1][1]);
  S.pay[3 * kItem + q] = make_float4(A[2][1], A[0][2], A[1][2], A[2][2]);
  S.fz[q] = sc.f[2];
}

// x of another lane, 0 where the DPP control CTRL has none
template <int CTRL>
MD float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;   // quad_perm [1, 0, 3, 2], [2, 3, 0, 1]

// flags the tiles the runs' boxes touch: a run's nodes span at most two tiles in x and y
MD void mark_run_tiles(const EnvDev& e, const Runs& R, uint32_t* __restrict__ flags) {
  for (int r = threadIdx.x >> 6; r < R.n; r += kItem / 64) {   // a wave per run
    const int lane = threadIdx.x & 63;
    const int tx = (R.lo[r][0] >> 2) + (lane & 1), ty = (R.lo[r][1] >> 2) + ((lane >> 1) & 1);
    const bool in = tx <= R.hi[r][0] >> 2 && ty <= R.hi[r][1] >> 2;
    const int tz1 = R.hi[r][2] >> 2;
    for (int tz = (R.lo[r][2] >> 2) + (lane >> 2); tz <= tz1; tz += 16)
      if (in) flags[e.tile_off + (tx * e.T + ty) * e.T + tz] = 1u;
  }
}

MD void mark_particle_tiles(const EnvDev& e, const int b[3], uint32_t* __restrict__ flags) {
  for (int a = 0; a < 2; ++a)
    for (int c = 0; c < 2; ++c)
      for (int d = 0; d < 2; ++d) {
        const int tx = (b[0] + 2 * a) >> 2, ty = (b[1] + 2 * c) >> 2, tz = (b[2] + 2 * d) >> 2;
        flags[e.tile_off + (tx * e.T + ty) * e.T + tz] = 1u;
      }
}

// Sums the stored payloads into group 0 of the grid (every thread calls it,
// after col_index returned true and the payloads are written). Channels: with
// MASS (mass sum W, the affine value), else the affine value alone. A pass
// takes runs together while their boxes fit, or a slab of z of one that does
// not fit alone.
template <bool MASS, int BOXN>
MD void col_scatter(const EnvDev& e, ColShared<BOXN>& S, float mass, float* __restrict__ grid) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  Runs& R = S.r;
  const int nr = R.n;
  // 1, 2 or 4 lanes share a task's particles: about eight each
  const int count = S.start[R.cell[nr]];
  const int split = count >= 4 * R.occupied ? 2 : (count >= 2 * R.occupied ? 1 : 0);
  for (int r0 = 0, z0 = 0; r0 < nr;) {
    const int layer = R.ext[r0][0] * R.ext[r0][1], zall = R.ext[r0][2];
    const bool slab = layer * zall > BOXN;
    const int zn = slab ? min(BOXN / layer, zall - z0) : zall;   // z nodes of the slab
    const int n0 = R.node[r0];
    int r1 = r0 + 1;
    if (!slab)
      while (r1 < nr && R.node[r1 + 1] - n0 <= BOXN) ++r1;
    const int nodes = slab ? layer * zn : R.node[r1] - n0;
    for (int i = t; i < nodes; i += kItem) S.box[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (t < kBins) R.bin[t] = 0;
    __syncthreads();
    // the pass's tasks (run, base column, z node), counted by length: a task's order within its length does
    // not matter. Columns are at most 16 of a run's 36 node columns, so 4/9 of the nodes bounds the tasks.
    constexpr int kMine = (BOXN * 4 / 9 + kItem - 1) / kItem;
    int code[kMine], slot[kMine];
    const int task0 = R.task[r0], task1 = slab ? (R.ext[r0][0] - 2) * (R.ext[r0][1] - 2) * zn : R.task[r1] - task0;
    const float inv_slab = slab ? 1.f / (float)zn : 0.f;
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
      const int i = t + m * kItem;
      code[m] = -1;
      slot[m] = 0;
      if (i < task1) {
        int r = r0;
        while (r + 1 < r1 && R.task[r + 1] - task0 <= i) ++r;
        const int loc = i - (R.task[r] - task0), cz = R.ext[r][2] - 2;
        const int col = small_div(loc, slab ? inv_slab : R.inv_z[r]), zl = loc - col * (slab ? zn : cz + 2), z = z0 + zl;
        const int* start = S.start + R.cell[r] + col * cz;
        const int n = start[min(z, cz - 1) + 1] - start[max(z - 2, 0)];
        if (n > 0) {
          const int jx = small_div(col, R.inv_cy[r]), jy = col - jx * (R.ext[r][1] - 2);
          const int len = min((n + (1 << split) - 1) >> split, kBins) - 1;
          slot[m] = (len << 16) | atomicAdd(&R.bin[len], 1);
          code[m] = (r << 13) | (jx << 11) | (jy << 9) | zl;
        }
      }
    }
    __syncthreads();
    // first entry of each length: lane k of every wave sums the longer ones
    int longer = 0;
    const int mine = lane < kBins ? R.bin[lane] : 0;
#pragma unroll
    for (int k = kBins - 1; k > 0; --k) {
      const int of_k = __builtin_amdgcn_readlane(mine, k);   // by every lane: the lane read may not be masked off
      longer += lane < k ? of_k : 0;
    }
    const int tasks = __builtin_amdgcn_readlane(longer + mine, 0);
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
      const int at = (slot[m] & 0xffff) + __shfl(longer, slot[m] >> 16);
      if (code[m] >= 0) S.list[at] = (uint16_t)code[m];
    }
    __syncthreads();
    for (int u0 = 0; u0 < tasks << split; u0 += kItem) {
      const int ti = (u0 + t) >> split, part = t & ((1 << split) - 1);
      const bool live = ti < tasks;
      float acc[9][4];
#pragma unroll
      for (int o = 0; o < 9; ++o)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[o][c] = 0.f;
      int node = 0, sy = 0, sx = 0;
      if (live) {
        const int g = S.list[ti], r = g >> 13, jx = (g >> 11) & 3, jy = (g >> 9) & 3, zl = g & 511;
        const int cz = R.ext[r][2] - 2, cy = R.ext[r][1] - 2, z = z0 + zl;
        sy = slab ? zn : cz + 2;
        sx = (cy + 2) * sy;
        node = (slab ? 0 : R.node[r] - n0) + jx * sx + jy * sy + zl;
        const int* start = S.start + R.cell[r] + (jx * cy + jy) * cz;
        const int q1 = start[min(z, cz - 1) + 1];
        // particles before s1 have base z - 2, those before s2 z - 1, the rest z
        const int s1 = start[min(max(z - 1, 0), cz)], s2 = start[min(z, cz)];
#pragma unroll 1
        for (int q = start[max(z - 2, 0)] + part; q < q1; q += 1 << split) {
          const float4 p0 = S.pay[q], p1 = S.pay[kItem + q], p2 = S.pay[2 * kItem + q], p3 = S.pay[3 * kItem + q];
          const float fz = S.fz[q];
          const bool mid = q >= s1 && q < s2;
          const float oz = q < s1 ? 2.f : (mid ? 1.f : 0.f);
          // the z weight k (f - s)^2 + m of the piece at offset oz
          const float uz = fz - fmaf(-0.5f, oz, 1.5f);
          const float wz = fmaf((mid ? -1.f : 0.5f) * uz, uz, mid ? 0.75f : 0.f);
          const float wx[3] = {p0.x, 1.f - p0.x - p0.y, p0.y}, wy[3] = {p0.z, 1.f - p0.z - p0.w, p0.w};
          // the value at offsets (1, 1, oz), then +- a column of A per step in x and y
          const float ax[3] = {p1.w, p2.x, p2.y}, ay[3] = {p2.z, p2.w, p3.x}, az[3] = {p3.y, p3.z, p3.w};
          const float d2 = oz - fz;
          const float v[3] = {fmaf(az[0], d2, p1.x), fmaf(az[1], d2, p1.y), fmaf(az[2], d2, p1.z)};
#pragma unroll
          for (int ox = 0; ox < 3; ++ox) {
            const float wxz = wx[ox] * wz;
            float vx[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) vx[a] = ox == 0 ? v[a] - ax[a] : (ox == 1 ? v[a] : v[a] + ax[a]);
#pragma unroll
            for (int oy = 0; oy < 3; ++oy) {
              const float W = wxz * wy[oy];
              float* s = acc[3 * ox + oy];
              if (MASS) s[0] += W;
#pragma unroll
              for (int a = 0; a < 3; ++a) {
                const float va = oy == 0 ? vx[a] - ay[a] : (oy == 1 ? vx[a] : vx[a] + ay[a]);
                s[MASS + a] = fmaf(W, va, s[MASS + a]);
              }
            }
          }
        }
      }
      if (split >= 1)
#pragma unroll
        for (int o = 0; o < 9; ++o)
#pragma unroll
          for (int c = 0; c < 3 + MASS; ++c) acc[o][c] += dpp_mov<kQuadXor1>(acc[o][c]);
      if (split == 2)
#pragma unroll
        for (int o = 0; o < 9; ++o)
#pragma unroll
          for (int c = 0; c < 3 + MASS; ++c) acc[o][c] += dpp_mov<kQuadXor2>(acc[o][c]);
      const bool adds = live && part == 0;
#pragma unroll
      for (int o = 0; o < 9; ++o) {
        if (adds) {
          float4& at = S.box[node + (o / 3) * sx + (o % 3) * sy];
          float4 d = at;
          d.x += acc[o][0]; d.y += acc[o][1]; d.z += acc[o][2];
          if (MASS) d.w += acc[o][3];
          at = d;
        }
        __syncthreads();
      }
    }
    // the box to the grid, four lanes per node, 16 z nodes of one (x, y) column per wave and step. What depends
    // on the column is wave-uniform (scalar), what depends on the lane does not change with the column.
    const int w = __builtin_amdgcn_readfirstlane(wave), c = lane & 3;
    const float scale = MASS && c == 0 ? mass : 1.f;
    for (int r = r0; r < r1; ++r) {
      const int ey = __builtin_amdgcn_readfirstlane(R.ext[r][1]), columns = __builtin_amdgcn_readfirstlane(R.ext[r][0]) * ey;
      const int zr = __builtin_amdgcn_readfirstlane(slab ? zn : R.ext[r][2]);
      const int x0 = __builtin_amdgcn_readfirstlane(R.lo[r][0]), y0 = __builtin_amdgcn_readfirstlane(R.lo[r][1]);
      const float* sums = reinterpret_cast<const float*>(S.box) + 4 * (slab ? 0 : R.node[r] - n0) + c;
      const int per = (65536 + ey - 1) / ey;   // col / ey = col per >> 16 for col < 36
      for (int z = lane >> 2; z < zr; z += 16) {
        const int k = R.lo[r][2] + z0 + z;
        const uint32_t off = (k >> 2) * 512 + (k & 3) * 4 + c;
#pragma unroll 3
        for (int col = w; col < columns; col += 4) {
          const int jx = (col * per) >> 16, jy = col - jx * ey;
          const float v = sums[4 * (col * zr + z)];
          if (v != 0.f)   // else no particle weight reached the node
            atomicAdd(grid + node_base(e, x0 + jx, y0 + jy, 0) + off, scale * v);
        }
      }
    }
    if (slab && z0 + zn < zall) z0 += zn;
    else { r0 = r1; z0 = 0; }
    if (r0 < nr) __syncthreads();
  }
}

// the block's particles' 27 nodes added to the grid directly (boxes that do not
// fit): the payload rows, which hold nothing then, carry the particles
template <bool MASS, int BOXN>
MD void direct_scatter(const EnvDev& e, int count, ColShared<BOXN>& S, const Stencil& sc, const float g[3],
                       const float A[3][3], float mass, float* __restrict__ grid) {
  float row[3][4];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    row[a][0] = g[a];
#pragma unroll
    for (int c = 0; c < 3; ++c) row[a][1 + c] = A[a][c];
  }
  quad_scatter<MASS>(e, count, sc, row, mass, 1.f, [](const float r[4], const float d[3]) {
    return r[0] + r[1] * d[0] + r[2] * d[1] + r[3] * d[2];
  }, S.pay, grid);
}

// ----------------------------------------------------------------------------
// pieces of the substep for one particle
// ----------------------------------------------------------------------------
// G2P gather: v = sum W v_i, C = 4 n^2 sum W v_i d^T at position x.
// The solids take the sums axis by axis (z, then y, then x), which weighs a
// partial sum once instead of each node.
MD void gather_v_nested(const EnvDev& e, const float* __restrict__ grid, const float x[3], float vn[3], M3& Cn) {
  const Stencil sc = make_stencil(x, e.n, e.fn);
  const StencilAddr sa = stencil_addr(e, sc.b);
  const float4* genv = env_group1(e, grid);
  Cn = m3_zero();
  vn[0] = vn[1] = vn[2] = 0.f;
  float wdz[3], wdy[3];
  for (int o = 0; o < 3; ++o) {
    wdz[o] = sc.w[2][o] * ((float)o - sc.f[2]);
    wdy[o] = sc.w[1][o] * ((float)o - sc.f[1]);
  }
#pragma unroll 1
  for (int ox = 0; ox < 3; ++ox) {
    const uint32_t ax = ox == 0 ? sa.x[0] : (ox == 1 ? sa.x[1] : sa.x[2]);
    float sy[3] = {0.f, 0.f, 0.f}, syd[3] = {0.f, 0.f, 0.f}, syz[3] = {0.f, 0.f, 0.f};   // sums of v, v d_y, v d_z
#pragma unroll
    for (int oy = 0; oy < 3; ++oy) {
      float col[3] = {0.f, 0.f, 0.f}, colz[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int oz = 0; oz < 3; ++oz) {
        const float4 v4 = genv[ax + sa.y[oy] + sa.z[oz]];
        const float vi[3] = {v4.x, v4.y, v4.z};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          col[a] = fmaf(sc.w[2][oz], vi[a], col[a]);
          colz[a] = fmaf(wdz[oz], vi[a], colz[a]);
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        sy[a] = fmaf(sc.w[1][oy], col[a], sy[a]);
        syd[a] = fmaf(wdy[oy], col[a], syd[a]);
        syz[a] = fmaf(sc.w[1][oy], colz[a], syz[a]);
      }
    }
    float wx, dwx;
    spline_piece(ox, sc.f[0], wx, dwx);
    const float wdx = wx * ((float)ox - sc.f[0]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      vn[a] = fmaf(wx, sy[a], vn[a]);
      Cn.m[a][0] = fmaf(wdx, sy[a], Cn.m[a][0]);
      Cn.m[a][1] = fmaf(wx, syd[a], Cn.m[a][1]);
      Cn.m[a][2] = fmaf(wx, syz[a], Cn.m[a][2]);
    }
  }
  Cn = m3_scale(Cn, 4.f * e.fn);   // 4 n^2 dx
}

// The fluids weigh each node, with offsets in metres, as k_g2p_direct does. Their
// F is a product of (1 + dt tr C)^(1/3) along the path, which keeps the rounding
// of tr C (it repeats while a particle stays near one place in its cell), and the
// cotangents of rho, K and gamma are sums over all particles and substeps that
// nearly cancel. On 3.2 M water particles (16 envs, 96^3, 100 substeps, eight
// seeds) two runs of one build differ there by 1.2e-5 to 2.5e-5; against the
// kernels that staged boxes in LDS, which summed in this order, the nested sums
// differed by 3.1 times that (4.4 in the worst seed) and these differ by 1.7 times
// (2.2). The fluid's scatter hides the products: G2P + P2G 287.5 -> 288.7 us, the
// whole pass 121 ms either way (k_g2p alone 128 -> 133 us).
MD void gather_v_flat(const EnvDev& e, const float* __restrict__ grid, const float x[3], float vn[3], M3& Cn) {
  const Stencil sc = make_stencil(x, e.n, e.fn);
  const StencilAddr sa = stencil_addr(e, sc.b);
  const float4* genv = env_group1(e, grid);
  Cn = m3_zero();
  vn[0] = vn[1] = vn[2] = 0.f;
  float wdz[3];
  for (int o = 0; o < 3; ++o) wdz[o] = sc.w[2][o] * (((float)o - sc.f[2]) * e.dx);
#pragma unroll 1
  for (int ox = 0; ox < 3; ++ox) {
    const uint32_t ax = ox == 0 ? sa.x[0] : (ox == 1 ? sa.x[1] : sa.x[2]);
    const float wx = sel3(sc.w[0], ox), d0 = ((float)ox - sc.f[0]) * e.dx;
#pragma unroll
    for (int oy = 0; oy < 3; ++oy) {
      const float wxy = wx * sc.w[1][oy], d1 = ((float)oy - sc.f[1]) * e.dx;
      float col[3] = {0.f, 0.f, 0.f}, colz[3] = {0.f, 0.f, 0.f};   // sums of W v, W v d_z over the column
#pragma unroll
      for (int oz = 0; oz < 3; ++oz) {
        const float4 v4 = genv[ax + sa.y[oy] + sa.z[oz]];
        const float vi[3] = {v4.x, v4.y, v4.z};
        const float W = wxy * sc.w[2][oz], Wd = wxy * wdz[oz];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          col[a] = fmaf(W, vi[a], col[a]);
          colz[a] = fmaf(Wd, vi[a], colz[a]);
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        vn[a] += col[a];
        Cn.m[a][0] = fmaf(col[a], d0, Cn.m[a][0]);
        Cn.m[a][1] = fmaf(col[a], d1, Cn.m[a][1]);
        Cn.m[a][2] += colz[a];
      }
    }
  }
  Cn = m3_scale(Cn, 4.f * e.fn * e.fn);
}

MD void gather_v(const EnvDev& e, int mat, const float* __restrict__ grid, const float x[3], float vn[3], M3& Cn) {
  if (mat == MAT_FLUID_TAIT || mat == MAT_FLUID_PAPER)
    gather_v_flat(e, grid, x, vn, Cn);
  else
    gather_v_nested(e, grid, x, vn, Cn);
}

// writes a particle's new state and reports a non-finite one
MD void store_new_state(float* __restrict__ out, int64_t N, uint32_t t, const float xn[3], const float vn[3],
                        const M3& Cn, const M3& Hn, int32_t* err) {
  st_v3(out, N, t, 0, xn);
  st_v3(out, N, t, 3, vn);
  st_m3(out, N, t, 6, Cn);
  st_m3(out, N, t, 15, Hn);
  bool fin = true;
  for (int a = 0; a < 3; ++a) fin = fin && isfinite(xn[a]) && isfinite(vn[a]);
  for (int i = 0; i < 3; ++i) for (int j = 0; j < 3; ++j) fin = fin && isfinite(Hn.m[i][j]);
  if (!fin) atomicOr(err, ERR_NONFINITE);
}

// P2G of the block's particles at positions x (every thread calls it);
// load_rest(v, C, H) supplies the rest of a particle's state
template <int BOXN, typename LoadRest>
MD void p2g_col_body(const EnvDev& e, int mat, int count, const float x[3], LoadRest load_rest,
                     float* __restrict__ grid, uint32_t* __restrict__ flags, int32_t* err, ColShared<BOXN>& S) {
  const bool valid = (int)threadIdx.x < count;
  const Stencil sc = make_stencil(x, e.n, e.fn);
  if (valid && sc.oob) atomicOr(err, ERR_OUT_OF_DOMAIN);
  int pos = 0;
  const bool fits = col_index<BOXN>(e, sc.b, valid, S, pos);
  float mv[3], Ad[3][3];
  if (valid) {
    float v[3];
    M3 Cm, H;
    load_rest(v, Cm, H);
    const M3 A = m3_axpy(m3_scale(Cm, e.mp), -e.dt * e.vp * 4.f * e.fn * e.fn, stress(e, H, mat));
    for (int a = 0; a < 3; ++a) {
      mv[a] = e.mp * v[a];
      for (int c = 0; c < 3; ++c) Ad[a][c] = A.m[a][c] * e.dx;
    }
    if (fits)
      col_store(S, pos, sc, mv, Ad);
    else
      mark_particle_tiles(e, sc.b, flags);
  }
  if (!fits) {
    direct_scatter<true>(e, count, S, sc, mv, Ad, e.mp, grid);
    return;
  }
  col_scatter<true, BOXN>(e, S, e.mp, grid);
  mark_run_tiles(e, S.r, flags);
}

// P2G adjoint of one particle: gathers (mbar, Pbar), adds the G2P part
// (x rows 0-2 and F rows 3-11 of part) and returns the state cotangent.
// st, part: the block's first particle's rows. eig: 12 floats per thread that
// keep the eigen-decomposition of B across the stencil loop (only A and v stay
// live through it). The node sums are taken per (x, y) column; with
// gw = m_p mbar + Pbar (m_p v + A d) per node, a column needs sums of w_z gw and
// w_z' gw for the position, of w_z mbar, w_z Pbar and w_z d_z Pbar for the rest.
template <int MAT>
MD void p2g_adjoint_particle(const EnvDev& e, int mat, const float* __restrict__ st, const float* part, int64_t N,
                             uint32_t t, const float* gcot, float (*eig)[kItem], float pb[PB_COUNT], float cx[3],
                             float cv[3], M3& cC, M3& cF) {
  constexpr bool kEig = MAT == MAT_COROTATED || MAT == MAT_VONMISES || MAT < 0;
  const bool use_eig = kEig && (mat == MAT_COROTATED || mat == MAT_VONMISES);
  float x[3], v[3];
  load_x3(st, N, t, x);
  ld_v3(st, N, t, 3, v);
  const Stencil sc = make_stencil(x, e.n, e.fn);
  const StencilAddr sa = stencil_addr(e, sc.b);
  const float4* genv = env_group1(e, gcot);
  const float kf = -e.dt * e.vp * 4.f * e.fn * e.fn;
  M3 A;   // times dx: offsets d in grid units below
  {
    const M3 Cm = ld_m3(st, N, t, 6);
    const M3 H = ld_m3(st, N, t, 15);
    const StressPrep spr = stress_prep(e, H, mat);
    A = m3_scale(m3_axpy(m3_scale(Cm, e.mp), kf, stress_from(e, spr, mat)), e.dx);
    if (use_eig)
      for (int i = 0; i < 3; ++i) {
        eig[9 + i][t] = spr.l[i];
        for (int j = 0; j < 3; ++j) eig[3 * i + j][t] = spr.U.m[i][j];
      }
  }
  float gx[3] = {0.f, 0.f, 0.f};   // sum of grad W gw, grid units
  float sP[3] = {0.f, 0.f, 0.f};   // sum of W Pbar
  float sm = 0.f;                  // sum of W mbar
  M3 Ab = m3_zero();               // sum of W Pbar d^T, grid units
#pragma unroll 1
  for (int ox = 0; ox < 3; ++ox)
#pragma unroll 1
    for (int oy = 0; oy < 3; ++oy) {
      const uint32_t axy = (ox == 0 ? sa.x[0] : (ox == 1 ? sa.x[1] : sa.x[2])) +
                           (oy == 0 ? sa.y[0] : (oy == 1 ? sa.y[1] : sa.y[2]));
      float4 mP[3];
#pragma unroll
      for (int oz = 0; oz < 3; ++oz) mP[oz] = genv[axy + sa.z[oz]];
      float wx, wy, dwx, dwy;
      spline_piece(ox, sc.f[0], wx, dwx);
      spline_piece(oy, sc.f[1], wy, dwy);
      const float d0 = (float)ox - sc.f[0], d1 = (float)oy - sc.f[1], wxy = wx * wy;
      float uc[3], cP[3] = {0.f, 0.f, 0.f}, cPz[3] = {0.f, 0.f, 0.f}, cm = 0.f, s0 = 0.f, s1 = 0.f;
      for (int a = 0; a < 3; ++a) uc[a] = fmaf(A.m[a][0], d0, fmaf(A.m[a][1], d1, e.mp * v[a]));
#pragma unroll
      for (int oz = 0; oz < 3; ++oz) {
        const float wz = sc.w[2][oz], dz = (float)oz - sc.f[2], wzd = wz * dz;
        const float Pb[3] = {mP[oz].y, mP[oz].z, mP[oz].w};
        float gw = e.mp * mP[oz].x;
        for (int a = 0; a < 3; ++a) gw = fmaf(Pb[a], fmaf(A.m[a][2], dz, uc[a]), gw);
        s0 = fmaf(wz, gw, s0);
        s1 = fmaf(sc.dw[2][oz], gw, s1);
        cm = fmaf(wz, mP[oz].x, cm);
        for (int a = 0; a < 3; ++a) {
          cP[a] = fmaf(wz, Pb[a], cP[a]);
          cPz[a] = fmaf(wzd, Pb[a], cPz[a]);
        }
      }
      gx[0] = fmaf(dwx * wy, s0, gx[0]);
      gx[1] = fmaf(wx * dwy, s0, gx[1]);
      gx[2] = fmaf(wxy, s1, gx[2]);
      sm = fmaf(wxy, cm, sm);
      const float w0 = wxy * d0, w1 = wxy * d1;
      for (int a = 0; a < 3; ++a) {
        sP[a] = fmaf(wxy, cP[a], sP[a]);
        Ab.m[a][0] = fmaf(w0, cP[a], Ab.m[a][0]);
        Ab.m[a][1] = fmaf(w1, cP[a], Ab.m[a][1]);
        Ab.m[a][2] = fmaf(wxy, cPz[a], Ab.m[a][2]);
      }
    }
  // x: grad W = n dw, and the stencil sum of -W A^T Pbar is -A^T sP (A / dx = n A here)
  for (int a = 0; a < 3; ++a)
    cx[a] = fmaf(e.fn, gx[a] - (A.m[0][a] * sP[0] + A.m[1][a] * sP[1] + A.m[2][a] * sP[2]), (part + a * N)[t]);
  Ab = m3_scale(Ab, e.dx);
  const M3 Cm = ld_m3(st, N, t, 6);
  const M3 H = ld_m3(st, N, t, 15);
  StressPrep spr;
  if (use_eig) {
    M3 U;
    float l[3];
    for (int i = 0; i < 3; ++i) {
      l[i] = eig[9 + i][t];
      for (int j = 0; j < 3; ++j) U.m[i][j] = eig[3 * i + j][t];
    }
    spr = stress_prep_with_eig(H, U, l, mat);
  } else {
    spr = stress_prep(e, H, mat);
  }
  const M3 tau = stress_from(e, spr, mat);
  // m_p enters m_i (weight W) and P_i through m_p (v + C d): the C d part
  // summed over the nodes is <C, sum W Pbar d^T>
  const float mpb = sm + v[0] * sP[0] + v[1] * sP[1] + v[2] * sP[2] + m3_ddot(Cm, Ab);
  for (int a = 0; a < 3; ++a) cv[a] = e.mp * sP[a];
  cC = m3_scale(Ab, e.mp);
  pb[PB_VP] += (-e.dt * 4.f * e.fn * e.fn) * m3_ddot(Ab, tau);
  pb[PB_MP] += mpb;
  cF = ld_m3(part, N, t, 3);
  stress_vjp_from(e, H, spr, m3_scale(Ab, kf), cF, pb, mat);
}

// G2P adjoint of the block's particles (every thread calls it): the cotangent
// (cx, cv, cC, cF) of the substep's output state -> the particle's partial
// cotangent (part rows 0-2: x, 3-11: F), the node-velocity cotangents added to
// group 0 of gcot. st: the substep's input state, st_next: its output (the
// tape's C' is the forward's own value); both and part: the block's first
// particle's rows.
template <int BOXN>
MD void g2p_adjoint_body(const EnvDev& e, int mat, int count, uint32_t t, const float* __restrict__ st,
                         const float* __restrict__ st_next, int64_t N, const float cx[3], const float cv[3],
                         const M3& cC, const M3& cF, float* part, const float* __restrict__ grid, float* gcot,
                         float pb[PB_COUNT], ColShared<BOXN>& S) {
  const bool valid = (int)threadIdx.x < count;
  float x[3];
  load_x3(st, N, t, x);
  const Stencil sc = make_stencil(x, e.n, e.fn);
  int pos = 0;
  const bool fits = col_index<BOXN>(e, sc.b, valid, S, pos);
  float vb[3], Ad[3][3];   // Ad: 4 n^2 dx Cbar
  if (valid) {
    for (int a = 0; a < 3; ++a) vb[a] = fmaf(e.dt, cx[a], cv[a]);
    {
      const M3 H = ld_m3(st, N, t, 15);
      const M3 Cn = ld_m3(st_next, N, t, 6);
      const M3 Ftrb = project_vjp(e, trial_h(e, Cn, H), cF, pb, mat);
      const M3 Cb = m3_axpy(cC, e.dt, m3_mul_abt(Ftrb, f_of(H)));
      st_m3(part, N, t, 3, m3_mul_atb(m3_axpy(m3_eye(), e.dt, Cn), Ftrb));
      for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) Ad[a][c] = 4.f * e.fn * Cb.m[a][c];
    }
    if (fits) col_store(S, pos, sc, vb, Ad);
    // x: with vg = v_i (vbar + Ad d) per node, sums of grad W vg and of W v_i, axis by axis as in gather_v
    const StencilAddr sa = stencil_addr(e, sc.b);
    const float4* genv = env_group1(e, grid);
    float gx[3] = {0.f, 0.f, 0.f}, sv[3] = {0.f, 0.f, 0.f};
#pragma unroll 1
    for (int ox = 0; ox < 3; ++ox) {
      const uint32_t ax = ox == 0 ? sa.x[0] : (ox == 1 ? sa.x[1] : sa.x[2]);
      float wx, dwx;
      spline_piece(ox, sc.f[0], wx, dwx);
      const float d0 = (float)ox - sc.f[0];
      float g0[3], yv[3] = {0.f, 0.f, 0.f}, yx = 0.f, yy = 0.f, yz = 0.f;
      for (int a = 0; a < 3; ++a) g0[a] = fmaf(Ad[a][0], d0, vb[a]);
#pragma unroll 1
      for (int oy = 0; oy < 3; ++oy) {
        const uint32_t axy = ax + (oy == 0 ? sa.y[0] : (oy == 1 ? sa.y[1] : sa.y[2]));
        float4 v4[3];
#pragma unroll
        for (int oz = 0; oz < 3; ++oz) v4[oz] = genv[axy + sa.z[oz]];
        float wy, dwy;
        spline_piece(oy, sc.f[1], wy, dwy);
        const float d1 = (float)oy - sc.f[1];
        float gc[3], cs[3] = {0.f, 0.f, 0.f}, s0 = 0.f, s1 = 0.f;
        for (int a = 0; a < 3; ++a) gc[a] = fmaf(Ad[a][1], d1, g0[a]);
#pragma unroll
        for (int oz = 0; oz < 3; ++oz) {
          const float vi[3] = {v4[oz].x, v4[oz].y, v4[oz].z};
          const float dz = (float)oz - sc.f[2];
          float vg = vi[0] * fmaf(Ad[0][2], dz, gc[0]);
          vg = fmaf(vi[1], fmaf(Ad[1][2], dz, gc[1]), vg);
          vg = fmaf(vi[2], fmaf(Ad[2][2], dz, gc[2]), vg);
          s0 = fmaf(sc.w[2][oz], vg, s0);
          s1 = fmaf(sc.dw[2][oz], vg, s1);
          for (int a = 0; a < 3; ++a) cs[a] = fmaf(sc.w[2][oz], vi[a], cs[a]);
        }
        yx = fmaf(wy, s0, yx);
        yy = fmaf(dwy, s0, yy);
        yz = fmaf(wy, s1, yz);
        for (int a = 0; a < 3; ++a) yv[a] = fmaf(wy, cs[a], yv[a]);
      }
      gx[0] = fmaf(dwx, yx, gx[0]);
      gx[1] = fmaf(wx, yy, gx[1]);
      gx[2] = fmaf(wx, yz, gx[2]);
      for (int a = 0; a < 3; ++a) sv[a] = fmaf(wx, yv[a], sv[a]);
    }
    // grad W = n dw, and the stencil sum of -4 n^2 W Cbar^T v_i is -n Ad^T sv
    float xb[3];
    for (int a = 0; a < 3; ++a)
      xb[a] = fmaf(e.fn, gx[a] - (Ad[0][a] * sv[0] + Ad[1][a] * sv[1] + Ad[2][a] * sv[2]), cx[a]);
    st_v3(part, N, t, 0, xb);
  }
  if (fits)
    col_scatter<false, BOXN>(e, S, 0.f, gcot);
  else
    direct_scatter<false>(e, count, S, sc, vb, Ad, 0.f, gcot);
}

// ----------------------------------------------------------------------------
// kernels: one block per work item (figures: top of this file). MAT < 0 reads the material at run time.
// An env past its substep count (k_call >= nsub) is frozen: its state and
// cotangent pass through.
// ----------------------------------------------------------------------------
template <int BOXN, int MAT>
__global__ void __launch_bounds__(256, waves_per_simd<BOXN>())
k_p2g_col(const float* __restrict__ st, int64_t N, const EnvDev* __restrict__ envs,
          const WorkItem* __restrict__ items, float* __restrict__ grid, uint32_t* __restrict__ flags,
          int32_t* __restrict__ errs, int k_call) {
  __shared__ ColShared<BOXN> S;
  const WorkItem it = items[blockIdx.x];
  const EnvDev& e = envs[it.env];
  if (k_call >= e.nsub) return;
  const bool valid = (int)threadIdx.x < it.count;
  const uint32_t t = valid ? threadIdx.x : 0;
  st += it.start;
  float x[3];
  load_x3(st, N, t, x);
  p2g_col_body<BOXN>(e, MAT >= 0 ? MAT : e.material, it.count, x, [&](float v[3], M3& Cm, M3& H) {
    ld_v3(st, N, t, 3, v);
    Cm = ld_m3(st, N, t, 6);
    H = ld_m3(st, N, t, 15);
  }, grid, flags, errs + it.env, S);
}

// G2P: 27 128-bit node reads per particle straight from the grid. Neighbouring
// lanes read the same lines, which the L1 serves: staging boxes in LDS first took
// 222 us where this takes 133 (3.2 M water particles; 3.5 TB/s of state alone).
template <int MAT>
__global__ void __launch_bounds__(256) k_g2p(const float* __restrict__ st, float* __restrict__ out, int64_t N,
                                             const EnvDev* __restrict__ envs, const WorkItem* __restrict__ items,
                                             const float* __restrict__ grid, int32_t* __restrict__ errs, int k_call) {
  const WorkItem it = items[blockIdx.x];
  if ((int)threadIdx.x >= it.count) return;
  const EnvDev& e = envs[it.env];
  const uint32_t t = threadIdx.x;
  st += it.start;
  out += it.start;
  if (k_call >= e.nsub) {
    copy_rows(st, out, N, t);
    return;
  }
  float x[3], xn[3], vn[3];
  load_x3(st, N, t, x);
  const M3 H = ld_m3(st, N, t, 15);
  M3 Cn;
  const int mat = MAT >= 0 ? MAT : e.material;
  gather_v(e, mat, grid, x, vn, Cn);
  for (int a = 0; a < 3; ++a) xn[a] = fmaf(e.dt, vn[a], x[a]);
  store_new_state(out, N, t, xn, vn, Cn, project(e, trial_h(e, Cn, H), mat), errs + it.env);
}

// G2P of substep k fused with P2G of substep k + 1: the new state goes to the
// tape once and is scattered from registers. k_call is substep k's call index;
// an env frozen at k copies its state, one frozen at k + 1 only takes the G2P.
template <int BOXN, int MAT>
__global__ void __launch_bounds__(256, waves_per_simd<BOXN>())
k_g2p2g_col(const float* __restrict__ st, float* __restrict__ out, int64_t N, const EnvDev* __restrict__ envs,
            const WorkItem* __restrict__ items, const float* __restrict__ grid_in, float* __restrict__ grid_out,
            uint32_t* __restrict__ flags_out, int32_t* __restrict__ errs, int k_call) {
  __shared__ ColShared<BOXN> S;
  const WorkItem it = items[blockIdx.x];
  const EnvDev& e = envs[it.env];
  const int mat = MAT >= 0 ? MAT : e.material;
  const bool valid = (int)threadIdx.x < it.count;
  const uint32_t t = valid ? threadIdx.x : 0;
  st += it.start;
  out += it.start;
  if (k_call >= e.nsub) {
    if (valid) copy_rows(st, out, N, t);
    return;
  }
  float x[3], xn[3], vn[3] = {0.f, 0.f, 0.f};
  M3 Cn = m3_zero(), Hn = m3_zero();
  load_x3(st, N, t, x);
  if (valid) {
    const M3 H = ld_m3(st, N, t, 15);
    gather_v(e, mat, grid_in, x, vn, Cn);
    Hn = project(e, trial_h(e, Cn, H), mat);
  }
  for (int a = 0; a < 3; ++a) xn[a] = fmaf(e.dt, vn[a], x[a]);
  if (valid) store_new_state(out, N, t, xn, vn, Cn, Hn, errs + it.env);
  if (k_call + 1 >= e.nsub) return;   // the env stops after this substep (uniform over the block)
  p2g_col_body<BOXN>(e, mat, it.count, xn, [&](float v[3], M3& Cm, M3& H) {
    for (int a = 0; a < 3; ++a) v[a] = vn[a];
    Cm = Cn;
    H = Hn;
  }, grid_out, flags_out, errs + it.env, S);
}

// G2P adjoint. Its gather of v and its payload share the particle's registers, so
// the von Mises form spills a little at five blocks per CU and is still faster there
// on equal envs (50 -> 47 us, 320,000 particles; corotated, without spills, 65 -> 62).
template <int BOXN, int MAT>
__global__ void __launch_bounds__(256, waves_per_simd<BOXN>())
k_g2p_adjoint_col(const float* __restrict__ st, const float* __restrict__ st_next,
                  const float* __restrict__ cot, float* __restrict__ part, int64_t N,
                  const EnvDev* __restrict__ envs, const WorkItem* __restrict__ items,
                  const float* __restrict__ grid, float* __restrict__ gcot, double* __restrict__ pacc,
                  int k_call) {
  __shared__ ColShared<BOXN> S;
  const WorkItem it = items[blockIdx.x];
  const EnvDev& e = envs[it.env];
  if (k_call >= e.nsub) return;
  const bool valid = (int)threadIdx.x < it.count;
  const uint32_t t = valid ? threadIdx.x : 0;
  cot += it.start;
  float pb[PB_COUNT] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float cx[3], cv[3];
  ld_v3(cot, N, t, 0, cx);
  ld_v3(cot, N, t, 3, cv);
  g2p_adjoint_body<BOXN>(e, MAT >= 0 ? MAT : e.material, it.count, t, st + it.start, st_next + it.start, N, cx, cv,
                         ld_m3(cot, N, t, 6), ld_m3(cot, N, t, 15), part + it.start, grid, gcot, pb, S);
  block_reduce_params(pb, pacc + (int64_t)it.env * 8);
}

// P2G adjoint: a gather of (mbar, Pbar) and the stress VJP; issue-bound. Four waves per
// SIMD; the nodes are summed flat per (x, y) column, since sums nested per axis keep
// more registers live and spill (640,000 corotated particles: 54 us nested, 43 flat).
template <int MAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_p2g_adjoint(const float* __restrict__ st, const float* __restrict__ part, float* __restrict__ cot_out, int64_t N,
              const EnvDev* __restrict__ envs, const WorkItem* __restrict__ items, const float* __restrict__ gcot,
              double* __restrict__ pacc, int k_call, const float* __restrict__ cot_in) {
  constexpr bool kEig = MAT == MAT_COROTATED || MAT == MAT_VONMISES || MAT < 0;
  __shared__ float eig[kEig ? 12 : 1][kItem];
  const WorkItem it = items[blockIdx.x];
  const EnvDev& e = envs[it.env];
  const bool valid = (int)threadIdx.x < it.count;
  const uint32_t t = valid ? threadIdx.x : 0;
  cot_out += it.start;
  if (k_call >= e.nsub) {
    if (valid) copy_rows(cot_in + it.start, cot_out, N, t);
    return;
  }
  float pb[PB_COUNT] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (valid) {
    float cx[3], cv[3];
    M3 cC, cF;
    p2g_adjoint_particle<MAT>(e, MAT >= 0 ? MAT : e.material, st + it.start, part + it.start, N, t, gcot, eig, pb, cx,
                              cv, cC, cF);
    st_v3(cot_out, N, t, 0, cx);
    st_v3(cot_out, N, t, 3, cv);
    st_m3(cot_out, N, t, 6, cC);
    st_m3(cot_out, N, t, 15, cF);
  }
  block_reduce_params(pb, pacc + (int64_t)it.env * 8);
}

// P2G adjoint of substep k fused with the G2P adjoint of substep k - 1: the
// cotangent of state k stays in registers between the gather of (mbar, Pbar)
// (group 1 of gcot, written by substep k's grid adjoint) and the scatter of
// substep k - 1's node-velocity cotangents into group 0, which that grid
// adjoint cleared. An env frozen at k takes its state-k cotangent from cot_end,
// the cotangent that entered the segment; one frozen at k - 1 as well has
// nothing to do. `part` holds substep k's partials on entry and substep k - 1's
// on exit (each thread reads its own particle's before it writes them).
template <int BOXN, int MAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_adj_pair_col(const float* __restrict__ st_prev, const float* __restrict__ st, float* part,
               const float* __restrict__ cot_end, int64_t N, const EnvDev* __restrict__ envs,
               const WorkItem* __restrict__ items, const float* __restrict__ grid_prev, float* gcot,
               double* __restrict__ pacc, int k_call) {
  __shared__ ColShared<BOXN> S;
  const WorkItem it = items[blockIdx.x];
  const EnvDev& e = envs[it.env];
  const int mat = MAT >= 0 ? MAT : e.material;
  if (k_call - 1 >= e.nsub) return;
  const bool valid = (int)threadIdx.x < it.count;
  const uint32_t t = valid ? threadIdx.x : 0;
  st_prev += it.start;
  st += it.start;
  part += it.start;
  cot_end += it.start;
  float pb[PB_COUNT] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float cx[3] = {0.f, 0.f, 0.f}, cv[3] = {0.f, 0.f, 0.f};
  M3 cC = m3_zero(), cF = m3_zero();
  if (valid) {
    if (k_call >= e.nsub) {
      ld_v3(cot_end, N, t, 0, cx);
      ld_v3(cot_end, N, t, 3, cv);
      cC = ld_m3(cot_end, N, t, 6);
      cF = ld_m3(cot_end, N, t, 15);
    } else {
      // the eigen-decomposition waits in the payload rows, which are written only after col_index's barriers
      static_assert(sizeof(S.pay) >= 12 * kItem * sizeof(float), "eigen stash exceeds the payload rows");
      p2g_adjoint_particle<MAT>(e, mat, st, part, N, t, gcot, reinterpret_cast<float(*)[kItem]>(S.pay), pb, cx, cv, cC,
                                cF);
    }
  }
  g2p_adjoint_body<BOXN>(e, mat, it.count, t, st_prev, st, N, cx, cv, cC, cF, part, grid_prev, gcot, pb, S);
  block_reduce_params(pb, pacc + (int64_t)it.env * 8);
}

// ----------------------------------------------------------------------------
// launchers: one launch per material range
// ----------------------------------------------------------------------------
#define MPMX_BY_MAT(mat, LAUNCH)                          \
  switch (mat) {                                          \
    case MAT_NEOHOOKEAN: LAUNCH(MAT_NEOHOOKEAN); break;   \
    case MAT_COROTATED: LAUNCH(MAT_COROTATED); break;     \
    case MAT_VONMISES: LAUNCH(MAT_VONMISES); break;       \
    case MAT_FLUID_TAIT: LAUNCH(MAT_FLUID_TAIT); break;   \
    case MAT_FLUID_PAPER: LAUNCH(MAT_FLUID_PAPER); break; \
    case -1: LAUNCH(-1); break;                           \
    default: break;                                       \
  }

void launch_p2g_col(const float* st, int64_t N, const EnvDev* envs, const WorkItem* items, int n_items, float* grid,
                    uint32_t* flags, int32_t* errs, int k_call, int box, int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) hipLaunchKernelGGL((k_p2g_col<BOX, M>), dim3(n_items), dim3(kItem), 0, s, st, N, envs, items, grid, flags, errs, k_call)
  if (box) {
    constexpr int BOX = kBoxSmall;
    MPMX_BY_MAT(mat, L)
  } else {
    constexpr int BOX = kBoxLarge;
    MPMX_BY_MAT(mat, L)
  }
#undef L
}

void launch_g2p(const float* st, float* out, int64_t N, const EnvDev* envs, const WorkItem* items, int n_items,
                const float* grid, int32_t* errs, int k_call, int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) hipLaunchKernelGGL((k_g2p<M>), dim3(n_items), dim3(kItem), 0, s, st, out, N, envs, items, grid, errs, k_call)
  MPMX_BY_MAT(mat, L)
#undef L
}

void launch_g2p2g_col(const float* st, float* out, int64_t N, const EnvDev* envs, const WorkItem* items, int n_items,
                      const float* grid_in, float* grid_out, uint32_t* flags_out, int32_t* errs, int k_call, int box,
                      int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) \
  hipLaunchKernelGGL((k_g2p2g_col<BOX, M>), dim3(n_items), dim3(kItem), 0, s, st, out, N, envs, items, grid_in, grid_out, flags_out, errs, k_call)
  if (box) {
    constexpr int BOX = kBoxSmall;
    MPMX_BY_MAT(mat, L)
  } else {
    constexpr int BOX = kBoxLarge;
    MPMX_BY_MAT(mat, L)
  }
#undef L
}

void launch_g2p_adjoint_col(const float* st, const float* st_next, const float* cot, float* part, int64_t N,
                            const EnvDev* envs, const WorkItem* items, int n_items, const float* grid, float* gcot,
                            double* pacc, int k_call, int box, int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) \
  hipLaunchKernelGGL((k_g2p_adjoint_col<BOX, M>), dim3(n_items), dim3(kItem), 0, s, st, st_next, cot, part, N, envs, items, grid, gcot, pacc, k_call)
  if (box) {
    constexpr int BOX = kBoxSmall;
    MPMX_BY_MAT(mat, L)
  } else {
    constexpr int BOX = kBoxLarge;
    MPMX_BY_MAT(mat, L)
  }
#undef L
}

void launch_p2g_adjoint(const float* st, const float* part, float* cot_out, int64_t N, const EnvDev* envs,
                        const WorkItem* items, int n_items, const float* gcot, double* pacc, int k_call,
                        const float* cot_in, int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) \
  hipLaunchKernelGGL((k_p2g_adjoint<M>), dim3(n_items), dim3(kItem), 0, s, st, part, cot_out, N, envs, items, gcot, pacc, k_call, cot_in)
  MPMX_BY_MAT(mat, L)
#undef L
}

void launch_adj_pair_col(const float* st_prev, const float* st, float* part, const float* cot_end, int64_t N,
                         const EnvDev* envs, const WorkItem* items, int n_items, const float* grid_prev, float* gcot,
                         double* pacc, int k_call, int box, int mat, hipStream_t s) {
  if (n_items == 0) return;
#define L(M) \
  hipLaunchKernelGGL((k_adj_pair_col<BOX, M>), dim3(n_items), dim3(kItem), 0, s, st_prev, st, part, cot_end, N, envs, items, grid_prev, gcot, pacc, k_call)
  if (box) {
    constexpr int BOX = kBoxSmall;
    MPMX_BY_MAT(mat, L)
  } else {
    constexpr int BOX = kBoxLarge;
    MPMX_BY_MAT(mat, L)
  }
#undef L
}

}  // namespace mpmx
