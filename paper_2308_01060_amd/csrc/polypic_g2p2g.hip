// G2P of one step fused with the P2G of the next, for gfx950.
//
// G2P reads no coefficients: the new ones come from the grid velocity alone
// (Eq. 6-8, section 3.3), and the next step's P2G (Eq. 1, 4, 13) is their only
// reader.  One thread per output slot i (particle perm[i]) therefore does:
//
//   * G2P at the particle's position: gather the 27 node velocities per
//     component, project them onto the first n_modes modes, write the new
//     coefficients, the advected position x' (and F', mass) at slot i;
//   * P2G at x' with the coefficients still in registers: the stencil of x',
//     the weighted mode rows, and the nodal mass and momentum streamed node by
//     node into FP64 LDS bricks around 4^3-node tiles (lane groups that share a
//     base node add across lanes first), then one float atomic per brick node
//     and channel into the next grid.
//
// The coefficient array is written once and never read back, instead of being
// written by G2P and read again by the next step's P2G: the particle stream
// drops from 40 + 24 n_modes to 28 + 12 n_modes bytes per particle.  The result
// is the G2P call followed by the P2G call on its outputs, up to the order of
// the floating-point sums.
#include <type_traits>

#include "polypic_internal.hpp"

namespace polypic {

namespace {

// Slot of a thread: lane groups of 2^lg consecutive slots (which in cell order
// usually share a cell, hence a base node), the groups of a wavefront spread over
// the workgroup's chunk so that they sit in different cells and their brick
// atomics do not collide.
// Output rows are staged in LDS, one float per slot, and 64 lanes of a wavefront must
// write 64 distinct banks.  kRotate (rows that leave in whole lines, from a stage in slot
// order): the wavefronts' places rotate from one 64 slots to the next, so that the
// slots of a wavefront differ modulo 64.  Where a place steps back, two groups of a
// wavefront come close to each other and may share a cell, so rows that leave slot by
// slot keep the places and permute the stage instead (stage_pos; measured, at rest, 4.19 M
// particles, rotated and permuted: 1, 4 and 8 modes 174, 187 and 198 us, 171, 184 and 195).
template <int NW, bool kRotate>
__device__ __forceinline__ int fused_slot(int tid, int lg) {
  static_assert(NW == 4, "four wavefronts' groups of 2 or 4 lanes: 64 slots per 16 >> lg groups");
  const int lane = tid & (kWave - 1);
  const int wv = tid / kWave;
  const int group = lane >> lg;
  const int place = kRotate ? (wv + (group >> (4 - lg))) & (NW - 1) : wv;
  return ((group * NW + place) << lg) | (lane & ((1 << lg) - 1));
}

// Position of slot s in a staging row (a permutation of each 32 slots) where the places do
// not rotate.  The 64 slots one wavefront writes agree in their wavefront-index bits (lg,
// lg + 1) and differ in bits 5-7, which a plain index drops from the bank number.  XORing bit
// 6, and bits 5 ^ 7, into the wavefront-index bits puts the writes of each half wavefront on
// 32 distinct banks and those of the whole wavefront on 64, while a read of 64 consecutive
// slots only permutes each half.
__device__ __forceinline__ int stage_pos(int s, int lg) {
  return s ^ (((s >> 6) & 1) << lg) ^ ((((s >> 7) ^ (s >> 5)) & 1) << (lg + 1));
}

// Bricks of the scatter.  A workgroup's slots are in the order of the positions before
// the advection, so the 4^3-node tiles of those positions are runs of consecutive slots,
// and one step moves a particle by less than a cell: a brick covers its tile's cells and
// one cell around them (8^3 nodes).  A particle that crossed into a neighbouring tile
// then stays in its own tile's brick.  With bricks of the tile alone (6^3 nodes), given to
// the tiles of the new positions, such particles take a chunk past its bricks and go to
// HBM, 27 atomics per channel each, and the call slows with the speed of the flow
// (measured, 4.19 M particles, 4 modes, 0.1, 1.3 and 2.6 % of a cell per step and axis: 237,
// 507 and 860 us; with these bricks 208, 234 and 258; at rest 188 and 185).  The z stride
// spreads a half wavefront's cells over the banks, as in the tile-only bricks.
constexpr int kFuseN = kBrickN + 2;  // nodes per brick edge
constexpr int kFuseSY = 8;
constexpr int kFuseSZ = 68;
constexpr int kFuseV = (kFuseN - 1) * (1 + kFuseSY + kFuseSZ) + 1;  // doubles per channel
constexpr int kFuseNodes = kFuseN * kFuseN * kFuseN;
// A round of the scatter fills two channels: two rounds let three bricks fit where all four
// channels at once would leave two, and a chunk of a block's edge or of a small scene touches
// three or four tiles (of a 16^3-cell block's slots, 4.5 % lie in the
// third tile of their chunk or later, 0.9 % in the fourth or later).
constexpr int kFuseK = 3;  // bricks per workgroup
// All four channels of one brick fit in two rounds' space of three: a chunk of one brick (a
// dense block at rest is mostly such chunks) takes one round (measured, at rest, 4.19 M
// particles, two rounds and one: 1, 4 and 8 modes 180, 193 and 206 us, 175, 188 and 201).
constexpr int kFusePool = 2 * kFuseK;  // channels of bricks that the LDS holds
constexpr int kFuseOneRound = kFusePool / 4;  // bricks that fit with all four channels
constexpr int kFuseBrickF = (2 * kFusePool * kFuseV + 63) / 64 * 64;  // in floats
// Coefficients of the last component that the second half reads back from the LDS rows
// they were staged in, instead of holding them in registers across the scatter of the
// other channels: at 27 modes the 128 registers of 4 waves per SIMD otherwise spill, and
// the spills' scratch traffic costs more than these reads (measured, 27 modes: 414 us at
// 11 spilled registers, 385 at none; 776 and 718 for a batch of 6 M particles).  (The instance
// of one scene that writes slot by slot spills one register for the permuted stage: 377 us
// rotated and without it, 374 so.)
template <int NR>
constexpr int kFuseKept = NR > 8 ? 12 : 0;
constexpr uint32_t kNoCell = 0xFFFFFFFFu;
// first node of the 4^3 tile of a packed base node (10 bits an axis)
__device__ __forceinline__ uint32_t tile_bits(uint32_t cell) { return cell & 0x3FCFF3FCu; }
constexpr int kQuadCell = 10;  // particles per cell of a chunk from which quads fold

// LDS (about 40 KB per 256-thread workgroup at 27 modes) allows 4 waves per SIMD; the
// launch bound holds the registers to the 128 that allow them too (measured, 4.19 M
// particles: 0.40 ms at 3 waves per SIMD, 0.38 ms at 4).  With at most 8 modes 28 KB and, for
// one scene, fewer registers allow 5 (a whole step at 4 modes 291 us, 309 where LDS holds it
// to 4); the batch's instances at 4 and 8 modes need the registers of 4.
// Lane groups: a group whose particles share brick and base node adds its node values
// across lanes first, and one lane does the atomics.  A pair adds in 32 bits, a quad's two
// pairs in 64, as the bricks (their sums then hold the bits that pairs leave; measured, 32 and
// 64 bits for the second sum, 4.19 M particles at 16 per cell: 4 modes 240 and 233 us, 27 modes
// 387 and 398).  Pairs do best while the 32 pairs of a wavefront fall in different cells (one
// DPP fold per node value instead of two); in chunks whose cells hold more particles two pairs
// of a wavefront share a cell and its LDS addresses, and quads do better.  By default
// (lane_group 2) the kernel counts the cells of each chunk and takes quads from kQuadCell
// particles per cell on (measured, pairs and quads, 27 modes: 195 and 207 us at 8 per cell, 301
// and 299 at 12, 405 and 382 at 16; 4 modes: 120 and 134 at 8, 219 and 186 at 12, 308 and 230
// at 16).
// kRowMode: how the output rows are written.
constexpr int kBySlot = 0;       // every thread its slot of each row
constexpr int kLinesCached = 1;  // in whole lines, the rows' ends through the caches
constexpr int kLinesStream = 2;  // in whole lines, the ends streamed as well
template <int NR, int BS, class Scenes, int kRowMode>
__global__ __launch_bounds__(BS, 4) void g2p2g_kernel(G2P2GArgs a, Scenes sc) {
  constexpr int NW = BS / kWave;
  constexpr int K = kFuseK;
  constexpr int kKept = kFuseKept<NR>;
  constexpr bool kRotate = kRowMode != kBySlot;
  static_assert(!Scenes::kMany, "a workgroup's slots lie in one scene (OneScene, SceneChunks)");
  constexpr int kRows = NR + 1 > 10 ? NR + 1 : 10;  // staged: a component, or F and the mass
  constexpr int kStage0 =  // floats
      kFuseBrickF + kKept * BS > kRows * BS ? kFuseBrickF + kKept * BS - kRows * BS : 0;
  __shared__ alignas(16) double lds_all[(kStage0 + kRows * BS) / 2];
  static_assert(kStage0 % 4 == 0 && sizeof(lds_all) >= kFuseBrickF * sizeof(float), "layout");
  double* const brick = lds_all;  // [brick][channel of the round][node]
  __shared__ uint32_t cell_of[BS];  // by slot: base node before the advection, 10 bits an axis
  __shared__ int16_t run_of[BS];    // by slot: its run of equal tiles
  __shared__ int wave_heads[NW];    // heads of runs, and of cells << 16
  __shared__ uint32_t run_tile[K];  // tiles of the first runs
  __shared__ int16_t run_head[K];   // first slot of those runs
  __shared__ int origin[K][3];      // first base node of the bricks
  __shared__ int n_astray;          // slots without a brick in place
  constexpr int kCand = 8 + K;      // candidates for a brick placed anew
  __shared__ uint32_t cand_at[16];
  __shared__ int votes[K][16];      // of the brick, for a candidate
  static_assert(kCand <= 16, "candidates");

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wv = tid / kWave;
  const size_t Ps = (size_t)a.P;
  // this workgroup's chunk (in launch order, or XCD-contiguous), its slots
  // [i0, i0 + n_slots) and the scene of the first
  const Chunk ck = sc.template chunk<BS>(a.P, block_chunks(a.sched, gridDim.x).begin);
  if (ck.n <= 0) return;  // (whole workgroup: past the last chunk of a scene-chunked launch)
  const int64_t i0 = ck.i0;
  const int n_slots = ck.n;
  const SceneGrid g = sc.grid(ck.s);  // uniform over the workgroup
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int nxny = nx * ny;

  // ---------------------------------------------------------------- G2P
  // Lane pairs to begin with; the chunk's cells may turn out to call for quads.
  int lg = a.lane_group == 4 ? 2 : 1;
  int slot = fused_slot<NW, kRotate>(tid, lg);
  bool in = slot < n_slots;
  // a caller permutation is clamped into [0, P): a bad one gives wrong results, never a fault
  int p = in ? (a.perm ? min(max(a.perm[i0 + slot], 0), (int)(a.P - 1)) : (int)(i0 + slot)) : 0;
  float xp[3] = {0.f, 0.f, 0.f};
  if (in) {
    xp[0] = a.x_in[p];
    xp[1] = a.x_in[Ps + p];
    xp[2] = a.x_in[2 * Ps + p];
  }
  int b0, b1, b2;
  float t0, t1, t2;
  bool ok = stencil_axis_apart(xp[0], g.ox, g.inv_dx, nx, b0, t0);
  ok &= stencil_axis_apart(xp[1], g.oy, g.inv_dx, ny, b1, t1);
  ok &= stencil_axis_apart(xp[2], g.oz, g.inv_dx, nz, b2, t2);
  if (in && !ok) raise_flag(a.status, kFlagRange);
  if (tid == 0) n_astray = 0;
  bool gather = in && ok;
  cell_of[slot] = gather ? (uint32_t)b0 | ((uint32_t)b1 << 10) | ((uint32_t)b2 << 20) : kNoCell;
  float* const stage = reinterpret_cast<float*>(lds_all) + kStage0;
  // every lane's stencil lies in the grid (a flagged or idle lane has base node
  // 0 and the grid at least 3 nodes per axis), so the gathers need no branch;
  // such lanes are zeroed afterwards, only in the wavefronts that hold one
  int64_t vbase = g.node_off + (int64_t)(b2 * ny + b1) * nx + b0;
  auto gather_nodes = [&](int ax, float(&v)[27]) {
    const float* vg = a.gv + (size_t)ax * a.gstride + vbase;
#pragma unroll
    for (int jz = 0; jz < 3; ++jz)
#pragma unroll
      for (int jy = 0; jy < 3; ++jy)
#pragma unroll
        for (int jx = 0; jx < 3; ++jx) v[jx + 3 * jy + 9 * jz] = vg[jz * nxny + jy * nx + jx];
  };
  float v[27];
  gather_nodes(0, v);

  // While the first gathers are in flight: the chunk's runs of equal tiles in slot order
  // (thread t looks at slot t), and its cells.
  int n_runs = 0, cells = 0;
  __syncthreads();
  {
    const uint32_t cell = cell_of[tid], before = tid > 0 ? cell_of[tid - 1] : kNoCell;
    const bool some = cell != kNoCell;
    const bool head = some && (before == kNoCell || tile_bits(before) != tile_bits(cell));
    const unsigned long long hb = __ballot(head), cb = __ballot(some && before != cell);
    if (lane == 0) wave_heads[wv] = __popcll(hb) | (__popcll(cb) << 16);
    __syncthreads();
    int pre = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int h = wave_heads[w];
      pre += w < wv ? h & 0xFFFF : 0;
      n_runs += h & 0xFFFF;
      cells += h >> 16;
    }
    n_runs = __builtin_amdgcn_readfirstlane(n_runs);
    cells = __builtin_amdgcn_readfirstlane(cells);
    const int run = pre + lanes_below(hb) + (head ? 1 : 0) - 1;
    run_of[tid] = (int16_t)run;  // (-1 before the first valid slot)
    if (head && run < K) {
      run_tile[run] = tile_bits(cell);
      run_head[run] = (int16_t)tid;
    }
  }
  if (lg == 1 && n_slots >= kQuadCell * cells) {  // (uniform)
    lg = 2;
    stage[slot] = xp[0];
    stage[BS + slot] = xp[1];
    stage[2 * BS + slot] = xp[2];
    stage[3 * BS + slot] = __int_as_float(p);
    __syncthreads();
    slot = fused_slot<NW, kRotate>(tid, lg);
    in = slot < n_slots;
    xp[0] = stage[slot];
    xp[1] = stage[BS + slot];
    xp[2] = stage[2 * BS + slot];
    p = __float_as_int(stage[3 * BS + slot]);
    gather = cell_of[slot] != kNoCell;
    stencil_axis_apart(xp[0], g.ox, g.inv_dx, nx, b0, t0);
    stencil_axis_apart(xp[1], g.oy, g.inv_dx, ny, b1, t1);
    stencil_axis_apart(xp[2], g.oz, g.inv_dx, nz, b2, t2);
    vbase = g.node_off + (int64_t)(b2 * ny + b1) * nx + b0;
    gather_nodes(0, v);
    __syncthreads();  // the stage is read
  }
  const bool quads = lg == 2;  // (uniform)
  const int put_at = kRotate ? slot : stage_pos(slot, lg);  // of its slot in a staging row
  float c[3][27];  // the new coefficients, kept for the P2G half
  float xn[3];     // the advected position
  // Output rows go through LDS (the bricks are not in use yet) so that every
  // wavefront writes 64 consecutive slots (measured, 27 modes, 4.19 M particles:
  // 2.0 ms with the rows written from the spread slots, 0.47 ms staged).  The last kKept
  // rows lie past the bricks.
  auto row_at = [&](int k) { return stage + k * BS; };
  // `rows` staged rows out, row k from row_at(k0 + k) to dst(k): every thread its slot, or
  // in whole lines, a quarter of the rows per wavefront
  const int wave = __builtin_amdgcn_readfirstlane(wv);
  auto write_rows = [&](auto rows, int k0, auto dst) {
    if constexpr (kRowMode == kBySlot) {
      const int get_at = kRotate ? tid : stage_pos(tid, lg);
#pragma unroll
      for (int k = 0; k < rows; ++k)
        row_store_nt(row_at(k0 + k)[get_at], dst(k), n_slots, tid * (int)sizeof(float));
    } else {
      const int body = rows_body(n_slots);  // (uniform)
      auto each = [&](auto&& put) {
#pragma unroll
        for (int k = 0; k < rows; k += NW)
          if (k + NW <= rows || k + wave < rows) put(row_at(k0 + k + wave), dst(k + wave));
      };
      if (4 * lane < body) each([&](const float* s, float* row) { row_store_body(s, row, lane); });
      each([&](const float* s, float* row) {
        row_store_ends<kRowMode == kLinesStream>(s, row, n_slots, body, lane);
      });
    }
  };
  {
    const Proj1D px = proj_g2p(t0);
    const Proj1D py = proj_g2p(t1);
    const Proj1D pz = proj_g2p(t2);
    const bool any_idle = __ballot(!gather) != 0ull;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
      project_modes<NR>(v, px, py, pz, c[ax]);
      // the next component's gathers go out now, ahead of this component's
      // staging barriers and stores (v is free once projected)
      if (ax < 2) gather_nodes(ax + 1, v);
      if (any_idle) {
#pragma unroll
        for (int r = 0; r < NR; ++r) c[ax][r] = gather ? c[ax][r] : 0.0f;
      }
#pragma unroll
      for (int r = NR; r < 27; ++r) c[ax][r] = 0.0f;
      float x1 = fmaf(a.dt, c[ax][0], xp[ax]);
      x1 = fmaxf(x1, g.lo[ax]);
      xn[ax] = fminf(x1, g.hi[ax]);
      // rows of this component: x', then the NR coefficients; written once, never re-read
      // here, so streamed past the caches the gathers use
      row_at(0)[put_at] = xn[ax];
#pragma unroll
      for (int r = 0; r < NR; ++r) row_at(1 + r)[put_at] = c[ax][r];
      __syncthreads();
      // (this workgroup's slots)
      float* const co = a.coeff_out + (size_t)ax * NR * Ps + i0;
      float* const xo = a.x_out + (size_t)ax * Ps + i0;
      write_rows(std::integral_constant<int, NR + 1>{}, 0,
                 [&](int k) { return k == 0 ? xo : co + (size_t)(k - 1) * Ps; });
      __syncthreads();  // the next component overwrites the stage
    }
  }
  float m = 0.0f;
  if (in) m = a.mass_in ? a.mass_in[p] : a.uniform_mass;
  if (a.F_in || a.mass_out) {  // (uniform: kernel arguments)
    // F' = F + dt C F with C_ab = c[a][1 + b] / dx; rows 0-8 F', row 9 the mass
    float Fn[9];
    if (in && a.F_in) {
      float F[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) F[e] = a.F_in[(size_t)e * Ps + p];
      const float sdt = a.dt / g.dx;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int col = 0; col < 3; ++col) {
          float acc = 0.0f;
          if constexpr (NR >= 4) {
#pragma unroll
            for (int k = 0; k < 3; ++k) acc = fmaf(c[r][1 + k], F[3 * k + col], acc);
          }
          Fn[3 * r + col] = fmaf(sdt, acc, F[3 * r + col]);
        }
    } else {
#pragma unroll
      for (int e = 0; e < 9; ++e) Fn[e] = 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) row_at(e)[put_at] = Fn[e];
    row_at(9)[put_at] = m;
    __syncthreads();
    if (a.F_out)
      write_rows(std::integral_constant<int, 9>{}, 0,
                 [&](int k) { return a.F_out + (size_t)k * Ps + i0; });
    if (a.mass_out)
      write_rows(std::integral_constant<int, 1>{}, 9, [&](int) { return a.mass_out + i0; });
    __syncthreads();  // the bricks are cleared next
  }

  // ---------------------------------------------------------------- P2G of x'
  bool valid = in;
  int c0 = 0, c1 = 0, c2 = 0;
  float u0 = 0.f, u1 = 0.f, u2 = 0.f;
  if (valid) {
    bool ok2 = stencil_axis_joint(xn[0], g.ox, g.inv_dx, nx, c0, u0);
    ok2 &= stencil_axis_joint(xn[1], g.oy, g.inv_dx, ny, c1, u1);
    ok2 &= stencil_axis_joint(xn[2], g.oz, g.inv_dx, nz, c2, u2);
    if (!ok2) {  // (x' is clamped into the grid: only for a grid too small for a stencil)
      raise_flag(a.status, kFlagRange);
      valid = false;
    }
  }
  if (!valid) m = 0.0f;
  // the first K runs of equal tiles (in sorted order every tile is one run) take a brick each
  const int seg = run_of[slot];
  int nb = min(n_runs, K);
  // this thread's nodes of every brick (it clears and flushes them)
  constexpr int kOwn = kFuseNodes / BS;
  static_assert(kOwn * BS == kFuseNodes, "whole nodes per thread");
  const int own_x = tid & 7, own_y = (tid >> 3) & 7, own_z = tid >> 6;  // z: + q * BS / 64
  const int own_lds = own_x + kFuseSY * own_y + kFuseSZ * own_z;
  auto clear_bricks = [&](int k0, int k1) {
    for (int k = k0; k < k1; ++k)
#pragma unroll
      for (int q = 0; q < kOwn; ++q) brick[k * kFuseV + own_lds + q * (BS / 64) * kFuseSZ] = 0.0;
  };
  clear_bricks(0, nb <= kFuseOneRound ? 4 * nb : 2 * nb);
  // in place, a brick's first base node is one below its tile
  const uint32_t cell = cell_of[slot], tl = tile_bits(cell);
  int w0 = (int)(tl & 1023u) - 1, w1 = (int)((tl >> 10) & 1023u) - 1, w2 = (int)(tl >> 20) - 1;
  auto inside = [&](int o0, int o1, int o2) {
    return max(max((unsigned)(c0 - o0), (unsigned)(c1 - o1)), (unsigned)(c2 - o2)) <
           (unsigned)(kFuseN - 2);
  };
  int my_brick = gather && seg >= 0 && seg < K && inside(w0, w1, w2) ? seg : -1;
  const bool heads = gather && seg >= 0 && seg < K && slot == run_head[seg];
  if (heads) {
    origin[seg][0] = w0;
    origin[seg][1] = w1;
    origin[seg][2] = w2;
  }
  const unsigned long long miss = __ballot(gather && my_brick < 0);
  if (miss != 0ull && lane == 0) atomicAdd(&n_astray, __popcll(miss));
  __syncthreads();  // the bricks are clear and placed
  // (a launch whose workgroups all run at once takes as long as its longest, and to place the
  // bricks anew takes 1.5 us of it: there up to a quarter of the slots go to HBM first;
  // measured, 4,096 particles at 27 modes 16.9 us without that and 15.1)
  const int few = gridDim.x <= 256 ? BS / 4 : 0;
  const bool astray = __builtin_amdgcn_readfirstlane(n_astray) > few;  // (uniform)
  if (astray) {
    // Slots left their bricks, or are past the bricks.  The bricks are then placed anew, one
    // after the other, each on the candidate that holds most of the slots left: the bricks in
    // place, and the tiles of eight slots of the chunk moved as those slots moved.  A flow of
    // several cells per step moves a tile's particles alike; a splash or a jet moves a few of
    // them, and the others are to stay in their brick (measured, 4.19 M particles, 4 modes, 185
    // us at rest: a smooth flow of 1.3 and 3.8 cells per step and axis 451 and 789 us; the first
    // cell of every tile moved 3 and 6 cells 249 and 301, all others moved so 260 and 286.  With
    // bricks moved by their tile's first slot 1686 and 4631; 1389 and 2884, 1578 and 2572.  With
    // bricks on the tiles of the new positions 6575 and 7536; 277 and 650, 641 and 928).
    constexpr int kSample = BS / 8;
    auto pack = [](int o0, int o1, int o2) {  // (a brick that starts below the grid starts on it)
      return (uint32_t)max(o0, 0) | (uint32_t)max(o1, 0) << 10 | (uint32_t)max(o2, 0) << 20;
    };
    if (slot % kSample == 0)
      cand_at[slot / kSample] =
          gather ? pack(c0 - 1 - (int)(cell & 3u), c1 - 1 - (int)((cell >> 10) & 3u),
                        c2 - 1 - (int)((cell >> 20) & 3u))
                 : kNoCell;
    if (heads) cand_at[8 + seg] = pack(w0, w1, w2);
    if (tid >= nb && tid < K) cand_at[8 + tid] = kNoCell;
    if (tid < 16 * K) votes[tid / 16][tid % 16] = 0;
    clear_bricks(nb <= kFuseOneRound ? 4 * nb : 2 * nb, kFusePool);
    __syncthreads();
    const int cand = (int)cand_at[lane & 15];
    uint32_t fits = 0;  // candidates that hold this slot
#pragma unroll
    for (int j = 0; j < kCand; ++j) {
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(cand, j);
      if (o != kNoCell && inside((int)(o & 1023u), (int)((o >> 10) & 1023u), (int)(o >> 20)))
        fits |= 1u << j;
    }
    if (!gather) fits = 0;
    my_brick = -1;
    for (nb = 0; nb < K; ++nb) {
      const uint32_t left = my_brick < 0 ? fits : 0u;
      int mine = 0;  // votes of this wavefront, for candidate `lane`
#pragma unroll
      for (int j = 0; j < kCand; ++j) {
        const int n = __popcll(__ballot((left >> j) & 1u));
        mine = lane == j ? n : mine;
      }
      if (mine != 0) atomicAdd(&votes[nb][lane], mine);
      __syncthreads();
      int most = votes[nb][lane & 15] << 4 | (15 - (lane & 15));
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0x128, 0xF, 0xF, false));  // row_ror 8
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0x124, 0xF, 0xF, false));
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0x122, 0xF, 0xF, false));
      most = max(most, __builtin_amdgcn_mov_dpp(most, 0x121, 0xF, 0xF, false));
      most = __builtin_amdgcn_readfirstlane(most);
      if (most >> 4 == 0) break;  // (uniform) none left that a candidate holds
      const int best = 15 - (most & 15);
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(cand, best);
      if ((left >> best) & 1u) {
        my_brick = nb;
        w0 = (int)(o & 1023u);
        w1 = (int)((o >> 10) & 1023u);
        w2 = (int)(o >> 20);
      }
      if (tid == 0) {
        origin[nb][0] = (int)(o & 1023u);
        origin[nb][1] = (int)((o >> 10) & 1023u);
        origin[nb][2] = (int)(o >> 20);
      }
    }
  }
  const int chn = nb <= kFuseOneRound ? 4 : 2;  // (uniform) channels of a round
  const bool lds = my_brick >= 0;  // (a slot without a brick goes to HBM)
  if (a.regions) {
    // the regions the scatter lands in: the 6^3 nodes of each brick's tile, and those of
    // the new tile of every slot that left its tile or went to HBM (a box holding its
    // stencil), of every slot when bricks were placed anew; before the scatter holds its node
    // values (plain stores)
    if (!astray && tid < 8 * nb) {
      const uint32_t tc = run_tile[tid >> 3];
      flag_box_corner(a.regions, g.region_off, (uint32_t)ck.s, nx, ny, nz,
                      (int)(tc & 1023u), (int)((tc >> 10) & 1023u),
                      (int)(tc >> 20), kBrickN, tid & 7);
    }
    if (valid && (astray || !lds ||
                  tile_bits((uint32_t)c0 | ((uint32_t)c1 << 10) | ((uint32_t)c2 << 20)) != tl)) {
#pragma unroll
      for (int corner = 0; corner < 8; ++corner)
        flag_box_corner(a.regions, g.region_off, (uint32_t)ck.s, nx, ny, nz, c0 & ~(kBrickT - 1),
                        c1 & ~(kBrickT - 1), c2 & ~(kBrickT - 1), kBrickN, corner);
    }
  }
  // the lane pair (lane ^ 1), and with quads the other pair of the quad, share this
  // lane's base node (which its brick holds as well): every lane runs the exchanges (an
  // invalid one with zero mass), since a DPP read from a lane that did not execute it is
  // undefined
  const int mykey = valid ? ((c2 * 1024 + c1) * 1024 + c0) : -1 - lane;
  const bool pair = mykey == pair_swap_i(mykey);
  bool quad = false;
  if (quads) {
    const int quad_pair = quad_swap_i((int)pair), quad_key = quad_swap_i(mykey);
    quad = pair && quad_pair != 0 && mykey == quad_key;
  }
  const bool emit = valid && (quad ? (lane & 3) == 0 : (!pair || (lane & 1) == 0));
  const float pair_f = pair ? 1.0f : 0.0f;
  const int quad_m = quad ? ~0 : 0;
  {
    const Rows Rx = p2g_rows_scaled(basis_p2g(u0), m);
    const Rows Ry = p2g_rows_scaled(basis_p2g(u1), 1.0f);
    const Rows Rz = p2g_rows_scaled(basis_p2g(u2), 1.0f);
    const int lbase = (c0 - w0) + kFuseSY * (c1 - w1) + kFuseSZ * (c2 - w2);
    const int64_t gbase = g.node_off + (int64_t)(c2 * ny + c1) * nx + c0;
    double* const lb = brick + (lds ? my_brick * chn * kFuseV + lbase : 0);
    // one plane of 9 node values at a time: the folds run on every lane, then a
    // single predicated block per plane does the atomics
    auto emitter = [&](int ch) {
      double* const lbc = lb + (ch & (chn - 1)) * kFuseV;
      // (the HBM base is formed only on that rare path, to keep registers free)
      float* const gc = ch == 0 ? a.gm : ch == 1 ? a.gp0 : ch == 2 ? a.gp1 : a.gp2;
      return [=](int jz, float (&v)[9]) {
        float w[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) w[k] = pair_fold(v[k], pair_f);
        // rows [j0, j1) of the plane to the brick, or to HBM
        auto put = [&](int j0, int j1, auto&& value) {
          if (!emit) return;
          if (lds) {
#pragma unroll
            for (int jy = j0; jy < j1; ++jy)
#pragma unroll
              for (int jx = 0; jx < 3; ++jx)
                atomicAdd(lbc + jx + kFuseSY * jy + kFuseSZ * jz, value(jx + 3 * jy));
          } else {
#pragma unroll
            for (int jy = j0; jy < j1; ++jy)
#pragma unroll
              for (int jx = 0; jx < 3; ++jx)
                atomicAdd(gc + gbase + (jz * nxny + jy * nx + jx), (float)value(jx + 3 * jy));
          }
        };
        if (quads) {
          // two pairs are added in 64 bits, as the bricks add; a row at a time, for the registers
#pragma unroll
          for (int jy = 0; jy < 3; ++jy) {
            float other[3];  // (every lane)
#pragma unroll
            for (int jx = 0; jx < 3; ++jx) other[jx] = quad_other(w[jx + 3 * jy], quad_m);
            put(jy, jy + 1, [&](int k) { return (double)w[k] + (double)other[k - 3 * jy]; });
          }
        } else {
          put(0, 3, [&](int k) { return (double)w[k]; });
        }
      };
    };
    // Flush of two channels of a round: one global float atomic per channel per non-zero brick
    // node, by the node's owner thread, which clears it for the next round.
    auto flush = [&](int ch0, bool clear) {
      float* const dst[4] = {a.gm, a.gp0, a.gp1, a.gp2};
      const int own_node = own_x + nx * own_y + nxny * own_z;  // from the brick's corner
      for (int sb = 0; sb < nb; ++sb) {
        // the brick's corner is uniform, so that a node's address is a scalar base and this
        // thread's offset from the corner
        const int ox = __builtin_amdgcn_readfirstlane(origin[sb][0]);
        const int oy = __builtin_amdgcn_readfirstlane(origin[sb][1]);
        const int oz = __builtin_amdgcn_readfirstlane(origin[sb][2]);
        const int64_t corner = g.node_off + ((int64_t)oz * ny + oy) * nx + ox;
        const bool in_xy = (unsigned)(ox + own_x) < (unsigned)nx && (unsigned)(oy + own_y) < (unsigned)ny;
        double* const src = brick + (sb * chn + (ch0 & (chn - 1))) * kFuseV + own_lds;
#pragma unroll
        for (int q = 0; q < kOwn; ++q) {
          double* const at = src + q * (BS / 64) * kFuseSZ;
          float v[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) v[k] = (float)at[k * kFuseV];
          if (clear) {
#pragma unroll
            for (int k = 0; k < 2; ++k) at[k * kFuseV] = 0.0;
          }
          if (!in_xy || (unsigned)(oz + own_z + q * (BS / 64)) >= (unsigned)nz) continue;
#pragma unroll
          for (int k = 0; k < 2; ++k)
            if (v[k] != 0.0f)
              atomicAdd(dst[ch0 + k] + corner + (unsigned)(own_node + q * (BS / 64) * nxny), v[k]);
        }
      }
    };
    {  // mass: m W_ip
      float one[27];
#pragma unroll
      for (int r = 0; r < 27; ++r) one[r] = r == 0 ? 1.0f : 0.0f;
      stream_modes_planes<1>(one, Rx, Ry, Rz, emitter(0));
    }
    stream_modes_planes<NR>(c[0], Rx, Ry, Rz, emitter(1));
    if (chn == 2) {
      __syncthreads();
      flush(0, true);
      __syncthreads();
    }
    stream_modes_planes<NR>(c[1], Rx, Ry, Rz, emitter(2));
#pragma unroll
    for (int r = NR - kKept; r < NR; ++r) c[2][r] = row_at(1 + r)[put_at];  // (this thread's own)
    stream_modes_planes<NR>(c[2], Rx, Ry, Rz, emitter(3));
    __syncthreads();
    if (chn == 4) flush(0, false);
    flush(2, false);
  }
}

template <int NR, class Scenes>
hipError_t launch_nr(const G2P2GArgs& a, const Scenes& sc, unsigned blocks, hipStream_t stream) {
  constexpr int BS = kSceneChunk;
  // Whole lines cost more instructions per row than a slot per thread, and pay at 27 modes
  // when the rows start off the 32-byte sectors (measured, a slot per thread and whole
  // lines: P = 1234567 173 and 131 us, 2500007 305 and 240, 4000037 484 and 409; P = 2500008
  // 260 and 265, 4000040 406 and 450; at 4 modes, P = 2500007, 153 and 168).  The rows' ends
  // go through the caches while those still hold a line when the neighbouring workgroup's
  // part of it comes: up to about 4 M particles (through the caches and streamed: 2500007 257
  // and 274 us, 3400007 339 and 380, 3900003 414 and 419, 4000037 435 and 431, 4100009 470 and
  // 447, 4194303 460 and 463, 5500001 629 and 581).
  // A batch's workgroups neighbour each other on one XCD, whose L2 joins the parts of a
  // line: 718 us a slot per thread, 745 in lines.
  if constexpr (NR == 27 && std::is_same_v<Scenes, OneScene>) {
    if (rows_want_lines(NR, 32, a.P, {a.coeff_out, a.x_out})) {
      if (a.P < 4000000)
        g2p2g_kernel<NR, BS, Scenes, kLinesCached><<<blocks, BS, 0, stream>>>(a, sc);
      else
        g2p2g_kernel<NR, BS, Scenes, kLinesStream><<<blocks, BS, 0, stream>>>(a, sc);
      return hipGetLastError();
    }
  }
  g2p2g_kernel<NR, BS, Scenes, kBySlot><<<blocks, BS, 0, stream>>>(a, sc);
  return hipGetLastError();
}

// blocks: workgroups of kSceneChunk threads that cover every chunk
template <class Scenes>
hipError_t launch_modes(const G2P2GArgs& a, const Scenes& sc, int n_modes, int64_t n_nodes,
                        unsigned blocks, hipStream_t stream) {
  if (!a.accumulate) {
    hipError_t e = launch_grid_clear(a.gm, a.gp0, n_nodes, nullptr, stream);
    if (e != hipSuccess) return e;
  }
  if (a.P == 0) return hipSuccess;
  switch (n_modes) {
    case 1: return launch_nr<1>(a, sc, blocks, stream);
    case 4: return launch_nr<4>(a, sc, blocks, stream);
    case 8: return launch_nr<8>(a, sc, blocks, stream);
    case 27: return launch_nr<27>(a, sc, blocks, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_g2p2g(const G2P2GArgs& a, int n_modes, hipStream_t stream) {
  OneScene one;
  one.sg.nx = a.g.nx;
  one.sg.ny = a.g.ny;
  one.sg.nz = a.g.nz;
  one.sg.inv_dx = a.g.inv_dx;
  one.sg.ox = a.g.ox;
  one.sg.oy = a.g.oy;
  one.sg.oz = a.g.oz;
  one.sg.dx = a.dx;
  for (int k = 0; k < 3; ++k) {
    one.sg.lo[k] = a.lo[k];
    one.sg.hi[k] = a.hi[k];
  }
  one.sg.node_off = 0;
  one.sg.region_off = 0;
  const unsigned blocks = (unsigned)((a.P + kSceneChunk - 1) / kSceneChunk);
  return launch_modes(a, one, n_modes, (int64_t)a.g.nx * a.g.ny * a.g.nz, blocks, stream);
}

hipError_t launch_g2p2g_batch(const G2P2GArgs& a, const SceneDev* table, int n_scenes,
                              int n_modes, hipStream_t stream) {
  // each scene in chunks of its own: at most one partial chunk per scene
  SceneChunks sc{table, n_scenes};
  const unsigned blocks = (unsigned)(a.P / kSceneChunk + n_scenes + 1);
  return launch_modes(a, sc, n_modes, a.gstride, blocks, stream);
}

}  // namespace polypic
