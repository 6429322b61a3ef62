// G2P gather + projection (Eq. 6-8 and section 3.3) with advection and the
// optional F update, for gfx950.
//
// One thread per output slot i, reading particle perm[i].  Per velocity
// component the 27 node values are gathered and projected onto the first
// n_modes modes by the separable product of 1-D projection rows
// (x, then y, then z); rows and modes beyond n_modes are skipped at compile
// time.  All outputs are written at slot i, so with a sort permutation the
// particle arrays come out in cell order.
#include "polypic_internal.hpp"

namespace polypic {

namespace {

// kLines: the rows are staged in LDS and written in whole lines (rows_out_lines).
template <int NR, int BS, class Scenes, bool kLines>
__global__ __launch_bounds__(BS) void g2p_kernel(G2PArgs a, Scenes sc) {
  constexpr int NW = BS / kWave;
  constexpr int kRows = NR + 1 > 9 ? NR + 1 : 9;  // a component, or F
  __shared__ alignas(16) float stage[kLines ? kRows * BS : 1];
  const ChunkRange cr = block_chunks(a.sched, (a.P + BS - 1) / BS);  // one chunk
  const int64_t i0 = cr.begin * BS;
  const int tid = threadIdx.x;
  const int n_slots = (int)min((int64_t)BS, a.P - i0);
  // (a thread past the slots repeats the last one and writes nothing)
  const bool in = tid < n_slots;
  if (!kLines && !in) return;
  const int64_t i = i0 + min(tid, n_slots - 1);
  const int s0 = sc.first(i0);  // uniform over the workgroup
  const int s = sc.of(i, s0);
  // one wave-uniform lookup unless the wavefront straddles a scene boundary
  SceneGrid sg = sc.grid(s0);
  if constexpr (Scenes::kMany) {
    if (__ballot(s != s0) != 0ull) sg = sc.grid(s);
  }
  const size_t Ps = (size_t)a.P;
  const int nx = sg.nx, ny = sg.ny;
  // a caller permutation is clamped into [0, P): a bad one gives wrong results, never a fault
  const int p = a.perm ? min(max(a.perm[i], 0), (int)(a.P - 1)) : (int)i;
  const float xp[3] = {a.x_in[p], a.x_in[Ps + p], a.x_in[2 * Ps + p]};
  int b0, b1, b2;
  float t0, t1, t2;
  bool ok = stencil_axis(xp[0], sg.ox, sg.inv_dx, nx, b0, t0);
  ok &= stencil_axis(xp[1], sg.oy, sg.inv_dx, ny, b1, t1);
  ok &= stencil_axis(xp[2], sg.oz, sg.inv_dx, sg.nz, b2, t2);
  if (in && !ok) raise_flag(a.status, kFlagRange);

  const Proj1D px = proj_g2p(t0);
  const Proj1D py = proj_g2p(t1);
  const Proj1D pz = proj_g2p(t2);
  const size_t N = (size_t)a.gstride;
  const int nxny = nx * ny;
  const int64_t gbase = sg.node_off + (int64_t)(b2 * ny + b1) * nx + b0;

  float lin[3][3];  // lin[a][b] = coefficient of mode 1 + b for component a
  float F[9];
  if (a.F_in) {
#pragma unroll
    for (int e = 0; e < 9; ++e) F[e] = a.F_in[(size_t)e * Ps + p];
  }
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    float c[27];
    if (ok) {
      const float* vg = a.gv + (size_t)ax * N + gbase;
      float v[27];
#pragma unroll
      for (int jz = 0; jz < 3; ++jz)
#pragma unroll
        for (int jy = 0; jy < 3; ++jy)
#pragma unroll
          for (int jx = 0; jx < 3; ++jx) v[jx + 3 * jy + 9 * jz] = vg[jz * nxny + jy * nx + jx];
      project_modes<NR>(v, px, py, pz, c);
    } else {
#pragma unroll
      for (int r = 0; r < 27; ++r) c[r] = 0.0f;
    }
    // Outputs are streamed with non-temporal stores: written once, never re-read by this
    // kernel, they would otherwise displace the grid lines the gathers reuse from L2
    // (measured: 0.40 -> 0.27 ms at 27 modes, 4.19 M particles).
    float xn = fmaf(a.dt, c[0], xp[ax]);
    xn = fmaxf(xn, sg.lo[ax]);
    xn = fminf(xn, sg.hi[ax]);
    if constexpr (kLines) {
      float* const row = stage + tid;
      row[0] = xn;
#pragma unroll
      for (int r = 0; r < NR; ++r) row[(1 + r) * BS] = c[r];
      __syncthreads();
      rows_out_lines<NW, NR>(stage + BS, a.coeff_out + (size_t)ax * NR * Ps + i0, Ps, n_slots, tid);
      if (a.x_out)
        rows_out_lines<NW, 1>(stage, a.x_out + (size_t)ax * Ps + i0, Ps, n_slots, tid, 3);
      __syncthreads();  // the next component overwrites the stage
    } else {
      float* co = a.coeff_out + (size_t)ax * NR * Ps + i;
#pragma unroll
      for (int r = 0; r < NR; ++r) __builtin_nontemporal_store(c[r], co + (size_t)r * Ps);
      if (a.x_out) __builtin_nontemporal_store(xn, a.x_out + (size_t)ax * Ps + i);
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) lin[ax][b] = (NR >= 4) ? c[1 + b] : 0.0f;
  }
  if (a.F_out) {
    // F' = F + dt C F with C_ab = lin[a][b] / dx
    const float s = a.dt / sg.dx;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int col = 0; col < 3; ++col) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) acc = fmaf(lin[r][k], F[3 * k + col], acc);
        const float f = fmaf(s, acc, F[3 * r + col]);
        if constexpr (kLines)
          stage[(3 * r + col) * BS + tid] = f;
        else
          __builtin_nontemporal_store(f, a.F_out + (size_t)(3 * r + col) * Ps + i);
      }
    if constexpr (kLines) {
      __syncthreads();
      rows_out_lines<NW, 9>(stage, a.F_out + i0, Ps, n_slots, tid);
    }
  }
  if (!in) return;
  if (a.mass_out) __builtin_nontemporal_store(a.mass_in[p], a.mass_out + i);
}

template <int NR, class Scenes>
hipError_t launch_nr(const G2PArgs& a, const Scenes& sc, hipStream_t stream) {
  if constexpr (NR == 27) {
    // (measured, 27 modes: 229 -> 115 us at P = 1500003, 110 at 1500032; 512 threads against
    // 256: 128 and 138 at 1769471)
    if (rows_want_lines(NR, 64, a.P, {a.coeff_out, a.x_out})) {
      constexpr int BS = 512;
      const unsigned blocks = (unsigned)((a.P + BS - 1) / BS);
      g2p_kernel<NR, BS, Scenes, true><<<blocks, BS, 0, stream>>>(a, sc);
      return hipGetLastError();
    }
  }
  // 512 particles per workgroup: each output row is then written in 2 KB runs per
  // workgroup (measured in the step, 27 modes, 4.19 M particles: 0.37 ms at 256
  // threads, 0.27 ms at 512, 0.32 ms at 1024)
  constexpr int BS = 512;
  const unsigned blocks = (unsigned)((a.P + BS - 1) / BS);
  g2p_kernel<NR, BS, Scenes, false><<<blocks, BS, 0, stream>>>(a, sc);
  return hipGetLastError();
}

template <class Scenes>
hipError_t launch_modes(const G2PArgs& a, const Scenes& sc, int n_modes, hipStream_t stream) {
  if (a.P == 0) return hipSuccess;
  if (a.sched != kSchedLinear && a.sched != kSchedXcd) return hipErrorInvalidValue;
  switch (n_modes) {
    case 1: return launch_nr<1>(a, sc, stream);
    case 4: return launch_nr<4>(a, sc, stream);
    case 8: return launch_nr<8>(a, sc, stream);
    case 27: return launch_nr<27>(a, sc, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_g2p(const G2PArgs& a0, int n_modes, hipStream_t stream) {
  G2PArgs a = a0;
  a.gstride = (int64_t)a.g.nx * a.g.ny * a.g.nz;
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
  return launch_modes(a, one, n_modes, stream);
}

hipError_t launch_g2p_batch(const G2PArgs& a, const SceneDev* table, int n_scenes, int n_modes,
                            hipStream_t stream) {
  SceneTable st{table, n_scenes};
  return launch_modes(a, st, n_modes, stream);
}

}  // namespace polypic
