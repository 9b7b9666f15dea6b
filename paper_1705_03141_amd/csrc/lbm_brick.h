// lbm_brick.h -- the fused step for small lattices: one brick of BX x BY x BZ cells per
// workgroup, one thread per cell of the brick and of the 1-cell shell around it.
//
// A column of the marching kernel (lbm_step.h) pulls two planes before it collides its first one,
// so a lattice too small to fill the device with long columns spends most of a step in that
// serial prologue: three dependent pulls of 6 us each for columns of one plane.  Here every cell
// the brick needs is pulled at once, each by its own thread, and the brick is collided after one
// barrier: 2.5 or 2.8 pulls per cell instead of 1.5 (1 + 2 / planes), but one latency instead of
// several, and no padding of rows to 32 or 64 cells.  Results are bitwise those of the
// marching kernel: both complete a pull with finish_pull and collide with collide_cell.
//
// The scalars of the brick with a 2-cell halo are staged once (mirror images beyond lateral
// walls); the pull modes of the z faces differ per lane, and only workgroups on such a face
// execute more than one of them.  What bounds a step is its latency (launch, one round of loads
// from another XCD's writes, pull, collision) while every compute unit has one workgroup, and the
// 2.5 pulls per cell beyond that.  Measured per step, FP32, against the marching kernel: 32^3 9.8
// against 19.2 us, 41^3 21 against 23, 48^3 19.4 against 27.4; 64^3 40 against 30.
#pragma once

#include "lbm_step.h"

namespace lbm {

template <int BX_, int BY_, int BZ_>
struct Brick {
  static constexpr int BX = BX_, BY = BY_, BZ = BZ_;
  static constexpr int NC = BX * BY * BZ;                           // cells of the brick
  static constexpr int DX = BX + 2, DY = BY + 2, DZ = BZ + 2, ND = DX * DY * DZ;  // with its shell
  static constexpr int NT = (ND + 63) / 64 * 64;
  static constexpr int SX = BX + 4, SY = BY + 4, SZ = BZ + 4, NS = SX * SY * SZ;  // staged cells
  static constexpr int KS = (NS + NT - 1) / NT;
  static constexpr int WAVES = 3;  // per SIMD
  static_assert(NC % 64 == 0, "the brick's cells are whole waves");
};

// Position of shell cell r (0 <= r < ND - NC) relative to the brick's origin: the planes below and
// above, then the rings of the planes between.
template <int BX, int BY, int BZ>
__device__ __forceinline__ void shell_cell(int r, int& x, int& y, int& z) {
  constexpr int P = (BX + 2) * (BY + 2), RING = 2 * (BX + 2) + 2 * BY;
  if (r < 2 * P) {
    const int q = r < P ? r : r - P;
    z = r < P ? -1 : BZ;
    y = q / (BX + 2) - 1;
    x = q % (BX + 2) - 1;
  } else {
    const int q = r - 2 * P;
    z = q / RING;
    ring_cell<BX, BY>(q % RING, x, y);
  }
}

template <typename T, typename B, bool INIT, bool WALLS>
__global__ void __launch_bounds__(B::NT, B::WAVES) brick_kernel(const StepArgs A) {
  constexpr int BX = B::BX, BY = B::BY, BZ = B::BZ, NC = B::NC, ND = B::ND, NT = B::NT, SX = B::SX, SXY = B::SX * B::SY, NS = B::NS, KS = B::KS,
                DX = B::DX, DXY = B::DX * B::DY;
  __shared__ float4 sS[INIT ? 1 : NS];  // staged scalars (e, a, b, w_x)
  __shared__ float2 sW[INIT ? 1 : NS];  // (w_y, w_z)
  __shared__ float2 sD[2][ND];          // (rho_r/rho, rho) and (rho_b/rho, rho) of time t
  const Geo& G = A.geo;
  const bool zper = G.face_lo == FACE_PERIODIC, outflow = G.face_hi == FACE_OUTFLOW;
  const int plane = G.plane, pb = plane * (int)sizeof(T);

  // block -> brick; the grid is padded to a multiple of 8 so that the blocks of one XCD (ids
  // congruent modulo 8) take neighbouring bricks
  const int nb = (int)gridDim.x, L = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
  const int bxn = (G.nx + BX - 1) / BX, byn = (G.ny + BY - 1) / BY, bzn = (G.nz + BZ - 1) / BZ;
  if (L >= bxn * byn * bzn) return;  // the whole block, before any barrier
  const int bz = L / (bxn * byn), by = (L / bxn) % byn, bx = L % bxn;
  const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;

  // this thread's cell: the brick's cells first, in whole waves
  const int tid = threadIdx.x;
  const bool own = tid < NC, active = tid < ND;
  int lx = tid % BX, ly = (tid / BX) % BY, lz = tid / (BX * BY);
  if (!own) shell_cell<BX, BY, BZ>(min(tid, ND - 1) - NC, lx, ly, lz);
  const bool live = own && x0 + lx < G.nx && y0 + ly < G.ny && z0 + lz < G.nz;
  auto zsrc = [&](int q) { return zper ? wrap(q, G.nz) : min(max(q, 0), G.nz - 1); };
  const int gx = wrap(x0 + lx, G.nx), gy = wrap(y0 + ly, G.ny), gz = zsrc(z0 + lz), col = gy * G.nx + gx;
  const int wf = WALLS ? wall_flags(G, gx, gy) : 0;

  PlaneState st;
  st.clear();
  if constexpr (INIT) {
    if (own)
      init_cell<true>(A.init, A.pc, G.n, (long long)gz * plane + col, st.rho, st.rho_r, st.rho_b, st.e, st.df);
    else if (active)
      init_cell<false>(A.init, A.pc, G.n, (long long)gz * plane + col, st.rho, st.rho_r, st.rho_b, st.e, st.df);
  } else {
    // the loads of the staged scalars, then those of the populations
    float sv[KS][5];
    unsigned flip = 0;
    const rsrc_t rsc = buffer_of(A.sc_in, (unsigned)(5 * G.nz * plane * 4));
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int idx = min(tid + k * NT, NS - 1);
      const int ux = x0 + idx % SX - 2, uy = y0 + (idx / SX) % B::SY - 2, uz = z0 + idx / SXY - 2;
      int sx, sy;
      if (WALLS && G.wall_x) {
        sx = mirror(ux, G.nx);
        if (ux < 0 || ux >= G.nx) flip |= 1u << (2 * k);
      } else {
        sx = wrap(ux, G.nx);
      }
      if (WALLS && G.wall_y) {
        sy = mirror(uy, G.ny);
        if (uy < 0 || uy >= G.ny) flip |= 2u << (2 * k);
      } else {
        sy = wrap(uy, G.ny);
      }
      const unsigned o = (unsigned)((zsrc(uz) * 5 * plane + sy * G.nx + sx) * 4);
#pragma unroll
      for (int c = 0; c < 5; ++c) sv[k][c] = load_f32(rsc, o, c * plane * 4);
    }
    const bool outlet_c = outflow && gz == G.nz - 1;
    const int mode = plane_mode(G, gz);
    typename Word<T>::W ld[Q];
    // (the descriptor starts early enough for the corrections of mirrored populations)
    const int early = WALLS ? kMirrorSpan * pb : 0;
    const rsrc_t rg = buffer_of(static_cast<const char*>(A.g_in) - early, (unsigned)(Q * G.nz * pb + early));
    if (active && !outlet_c) {
      unsigned o[3][3];
      column_offsets<T, WALLS>(G, gx, gy, early, o);
      const unsigned zo[3] = {(unsigned)(zsrc(gz - 1) * Q * pb), (unsigned)(gz * Q * pb), (unsigned)(zsrc(gz + 1) * Q * pb)};
      const unsigned at[2][2] = {{0u - (wf & 1), 0u - ((wf >> 1) & 1)}, {0u - ((wf >> 2) & 1), 0u - ((wf >> 3) & 1)}};
      with_mode(mode, [&](auto M) {
        static_for<0, Q>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          constexpr Src s = resolve<i, decltype(M)::value>();
          unsigned v = zo[s.dz + 1] + o[s.dy + 1][s.dx + 1];
          if constexpr (WALLS) v += mirror_shift<s.j, s.dx, s.dy>(at, pb);
          ld[i] = Word<T>::load(rg, v, s.j * pb);
        });
      });
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KS; ++k)
      if (tid + k * NT < NS) {
        const float psi = sv[k][1];
        const float wx = __uint_as_float(__float_as_uint(sv[k][2]) ^ ((flip << (31 - 2 * k)) & 0x80000000u));
        const float wy = __uint_as_float(__float_as_uint(sv[k][3]) ^ ((flip << (30 - 2 * k)) & 0x80000000u));
        sS[tid + k * NT] = make_float4(sv[k][0], psi_a(psi), psi_b(psi), wx);
        sW[tid + k * NT] = make_float2(wy, sv[k][4]);
      }
    __syncthreads();
    if (active) {
      const int idx0 = (lz + 1) * SXY + (ly + 1) * SX + lx + 1;  // the cell's corner (-1, -1, -1)
      const float4* const S[3] = {sS, sS + SXY, sS + 2 * SXY};
      const float2* const W[3] = {sW, sW + SXY, sW + 2 * SXY};
      if (outlet_c) {
        outlet_cell<true>(A.outlet, A.pc, plane, col, st.rho, st.rho_r, st.rho_b, st.e, st.df);
      } else {
        with_mode(mode, [&](auto M) {
          int b0 = idx0;
          asm volatile("" : "+v"(b0));
          if (own)
            finish_pull<T, decltype(M)::value, true, SX, 4>(ld, S, W, b0, A.pc, st.rho, st.rho_r, st.rho_b, st.e, st.df,
                                                            st.shift, st.drho);
          else
            finish_pull<T, decltype(M)::value, false, SX, 4>(ld, S, W, b0, A.pc, st.rho, st.rho_r, st.rho_b, st.e,
                                                             st.df, st.shift, st.drho);
        });
      }
    }
  }
  if (active) {
    if (is_inflow(G, gx, gy, gz)) {  // R10: inflow sites are pure red at rho_r0
      st.rho = st.rho_r = G.rho_r0;
      st.rho_b = 0.0f;
    }
    const int d = (lz + 1) * DXY + (ly + 1) * DX + lx + 1;
    const float inv = rcp(st.rho);
    sD[0][d] = make_float2(st.rho_r * inv, st.rho);
    sD[1][d] = make_float2(st.rho_b * inv, st.rho);
  }
  __syncthreads();
  if (!live) return;

  // the gradients, from the cell's minority colour fraction (as in the marching kernel)
  const bool red_minor = st.rho_r <= st.rho_b;
  float gp[3], gr[3];
  {
    float vp[3][3][3], vr[3][3][3];
    const float2* D2 = sD[red_minor ? 0 : 1];
    // beyond a wall the stencil sees the boundary cell (reading R9)
    const int xo[3] = {(wf & 1) ? 0 : -1, 0, (wf & 2) ? 0 : 1};
    const int yo[3] = {(wf & 4) ? 0 : -DX, 0, (wf & 8) ? 0 : DX};
    const int zo[3] = {!zper && gz == 0 ? 0 : -DXY, 0, !zper && gz == G.nz - 1 ? 0 : DXY};
    const int d = (lz + 1) * DXY + (ly + 1) * DX + lx + 1;
#pragma unroll
    for (int dz = 0; dz < 3; ++dz) {
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
          const float2 v = D2[d + zo[dz] + yo[dy] + xo[dx]];
          vp[dz][dy][dx] = v.x;
          vr[dz][dy][dx] = v.y;
        }
      __builtin_amdgcn_sched_barrier(0);  // one plane of reads at a time
    }
    gradient27(vp, gp);
    gradient27(vr, gr);
    const float two = red_minor ? 2.0f : -2.0f;
    gp[0] *= two;
    gp[1] *= two;
    gp[2] *= two;
  }
  if (!(st.rho > 0.0f && st.rho < 3.0e38f)) *A.unstable = 1;
  CellOut o;
  collide_cell<Word<T>::kOutShift>(A.cp, A.rates, st.df, st.shift, st.drho, st.rho, st.rho_r, st.rho_b, gp, gr, o);
  const rsrc_t go = buffer_of(A.g_out, (unsigned)(Q * G.nz * pb));
  const rsrc_t so = buffer_of(A.sc_out, (unsigned)(5 * G.nz * plane * 4));
  const unsigned og = (unsigned)(gz * Q * pb + col * (int)sizeof(T)), os = (unsigned)((gz * 5 * plane + col) * 4);
#pragma unroll
  for (int i = 0; i < Q; ++i) Word<T>::store(Word<T>::enc_scaled(o.g[i]), go, og, i * pb);
  store_f32(st.e, so, os, 0);
  store_f32(psi_encode(st.rho_r, st.rho_b, st.rho), so, os, plane * 4);
  store_f32(o.wx, so, os, 2 * plane * 4);
  store_f32(o.wy, so, os, 3 * plane * 4);
  store_f32(o.wz, so, os, 4 * plane * 4);
}

template <typename T, typename B>
hipError_t launch_brick(const StepArgs& a, hipStream_t s) {
  const Geo& g = a.geo;
  const unsigned n = (unsigned)(((g.nx + B::BX - 1) / B::BX) * ((g.ny + B::BY - 1) / B::BY) * ((g.nz + B::BZ - 1) / B::BZ));
  const dim3 grid((n + 7) / 8 * 8), block(B::NT);
  const bool walls = g.wall_x || g.wall_y;
  if (a.init_mode && walls)
    hipLaunchKernelGGL((brick_kernel<T, B, true, true>), grid, block, 0, s, a);
  else if (a.init_mode)
    hipLaunchKernelGGL((brick_kernel<T, B, true, false>), grid, block, 0, s, a);
  else if (walls)
    hipLaunchKernelGGL((brick_kernel<T, B, false, true>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((brick_kernel<T, B, false, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_bricks_T(const StepArgs& a, hipStream_t s) {
  return small_bricks(a.geo) ? launch_brick<T, Brick<8, 4, 4>>(a, s) : launch_brick<T, Brick<16, 4, 4>>(a, s);
}

#define LBM_INSTANTIATE_BRICK(T) template hipError_t launch_bricks_T<T>(const StepArgs&, hipStream_t);

}  // namespace lbm
