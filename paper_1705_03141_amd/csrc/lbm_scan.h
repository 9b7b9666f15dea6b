// lbm_scan.h -- one pass over a lattice that forms the macroscopic state of every cell (densities
// and momentum of time t) and hands it to a consumer: block means on the device (coarse
// state) or the FP64 reductions of the diagnostics.
//
// It is the step kernel's pull without the ring and the collision: a workgroup of 64 x 4
// threads owns a column of cells and marches through a chunk of z planes, with the scalars of
// three source planes (and the next one) staged in LDS with a 1-cell halo, so that a cell costs
// its 27 population loads and about 1.5 x 5 scalar loads.  Bound by the read of the state, 128
// B per FP32 cell.  The kernel it replaces loaded the scalars of all 26 neighbours from global
// memory, about 150 loads per cell.  Measured, coarse state with factor 1 of the FP32 jet
// 256x256x1024 (128 B read and 16 B written per cell): 2.37 ms, 4.1 TB/s, against 11.3 ms; with
// factor 4 of an FP16 jet 112x112x448, where one thread walked the 64 cells of a block:
// 0.16 ms against 1.8 ms; diagnostics of an FP32 85^3 lattice 30 us against 79 us.
#pragma once

#include "lbm_step.h"

namespace lbm {

struct ScanTile {
  static constexpr int TX = 64, TY = 4, NT = TX * TY;
  static constexpr int SX = TX + 2, SY = TY + 2, NS = SX * SY;  // staged cells of a plane
  static constexpr int KS = (NS + NT - 1) / NT;                 // per thread
};

// (Four waves per SIMD leave 128 registers: the diagnostics between lateral walls spill some 24 of them, 96 B
// per lane, and the coarse state keeps its block sums, whose factor is a run-time value, in 32 B of scratch.)
template <typename T, bool WALLS, int KIND>
__global__ void __launch_bounds__(ScanTile::NT, 4) scan_kernel(const AuxArgs A, const ScanArgs R) {
  constexpr int TX = ScanTile::TX, TY = ScanTile::TY, NT = ScanTile::NT, SX = ScanTile::SX, NS = ScanTile::NS,
                KS = ScanTile::KS;
  // four slots: planes p - 1, p, p + 1 are read while p + 2 is written (its slot held p - 2, last
  // read before the previous barrier)
  __shared__ float4 sS[4][NS];  // e, a, b, w_x
  __shared__ float2 sW[4][NS];  // w_y, w_z
  const Geo& G = A.geo;
  const int plane = G.plane;
  const bool zper = G.face_lo == FACE_PERIODIC;
  const int pb = plane * (int)sizeof(T);
  const unsigned slab_bytes = (unsigned)(Q * pb), sc_bytes = (unsigned)(5 * plane * 4);
  const char* gin = static_cast<const char*>(A.g_in);

  // the grid is padded to a multiple of 8: the blocks of one XCD cover a contiguous range
  const int nb = (int)gridDim.x, L = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
  const int ntiles = R.tiles_x * R.tiles_y, chunk = L / ntiles, tile = L - chunk * ntiles;
  if (chunk >= R.nchunks) return;  // the whole block, before any barrier
  const int tyi = tile / R.tiles_x, txi = tile - tyi * R.tiles_x;
  const int x0 = txi * TX, y0 = tyi * TY, z0 = chunk * R.zchunk, z1 = min(z0 + R.zchunk, G.nz);

  const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
  const bool live = x0 + lx < G.nx && y0 + ly < G.ny;
  const int gx = wrap(x0 + lx, G.nx), gy = wrap(y0 + ly, G.ny), col = gy * G.nx + gx;
  // beyond lateral walls the staged cells are mirror images (as in the step kernel)
  unsigned stOff[KS];
  int walls = WALLS ? wall_flags(G, gx, gy) : 0;
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const int idx = min(tid + k * NT, NS - 1);
    const int ux = x0 + idx % SX - 1, uy = y0 + idx / SX - 1;
    const bool mx = WALLS && G.wall_x, my = WALLS && G.wall_y;
    if (mx && (ux < 0 || ux >= G.nx)) walls |= 256 << (2 * k);
    if (my && (uy < 0 || uy >= G.ny)) walls |= 512 << (2 * k);
    const int sx = mx ? mirror(ux, G.nx) : wrap(ux, G.nx), sy = my ? mirror(uy, G.ny) : wrap(uy, G.ny);
    stOff[k] = (unsigned)((sy * G.nx + sx) * 4);
  }
  auto zsrc = [&](int q) { return zper ? wrap(q, G.nz) : min(max(q, 0), G.nz - 1); };

  auto stage_load = [&](int q, float(&st)[KS][5]) {
    const rsrc_t r = buffer_of(A.sc_in + (size_t)zsrc(q) * 5 * (size_t)plane, sc_bytes);
#pragma unroll
    for (int k = 0; k < KS; ++k)
      if (k < KS - 1 || tid + k * NT < NS)
#pragma unroll
        for (int c = 0; c < 5; ++c) st[k][c] = load_f32(r, stOff[k], c * plane * 4);
  };
  auto stage_store = [&](int q, const float(&st)[KS][5]) {
#pragma unroll
    for (int k = 0; k < KS; ++k)
      if (k < KS - 1 || tid + k * NT < NS) {
        const float psi = st[k][1];
        float wx = st[k][2], wy = st[k][3];
        if constexpr (WALLS) {
          wx = __uint_as_float(__float_as_uint(wx) ^ (((unsigned)walls << (23 - 2 * k)) & 0x80000000u));
          wy = __uint_as_float(__float_as_uint(wy) ^ (((unsigned)walls << (22 - 2 * k)) & 0x80000000u));
        }
        sS[q & 3][tid + k * NT] = make_float4(st[k][0], psi_a(psi), psi_b(psi), wx);
        sW[q & 3][tid + k * NT] = make_float2(wy, st[k][4]);
      }
  };

  // consumers' state
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // block sums of phi and u / u_scale
  __shared__ float4 red[KIND == kScanCoarse ? NT / 2 : 1];  // row sums, one per pair of columns
  double v[8] = {};
  auto coarse_add = [&](int z, float rho, float rho_r, float rho_b, const float(&j)[3], const float(&F)[3]) {
    const float inv = 1.0f / rho;
    const float c[4] = {(rho_r - rho_b) * inv, (j[0] + 0.5f * F[0]) * inv * R.inv_u,
                        (j[1] + 0.5f * F[1]) * inv * R.inv_u, (j[2] + 0.5f * F[2]) * inv * R.inv_u};
    if (R.factor == 1) {
      if (live)
        reinterpret_cast<float4*>(R.out)[((long long)z * R.ph + gy) * R.pw + gx] = make_float4(c[0], c[1], c[2], c[3]);
      return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] += c[k];
    if ((z + 1) % R.factor != 0) return;
    for (int off = 1; off < R.factor; off *= 2)
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] += __shfl_xor(s[k], off, 64);
    if (lx % R.factor == 0) red[tid / 2] = make_float4(s[0], s[1], s[2], s[3]);
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = 0.0f;
  };
  // after the barrier that follows the last plane of a block of planes: its rows together
  auto coarse_put = [&](int z) {
    const int f = R.factor;
    if (f == 1 || (z + 1) % f != 0 || !live || lx % f != 0 || ly % f != 0) return;
    float4 t = red[tid / 2];
    for (int r = 1; r < f; ++r) {
      const float4 o = red[(tid + r * TX) / 2];
      t = make_float4(t.x + o.x, t.y + o.y, t.z + o.z, t.w + o.w);
    }
    const float w = 1.0f / (float)(f * f * f);
    reinterpret_cast<float4*>(R.out)[((long long)(z / f) * R.ph + gy / f) * R.pw + gx / f] =
        make_float4(t.x * w, t.y * w, t.z * w, t.w * w);
  };
  auto diag_add = [&](int z, float rho, float rho_r, float rho_b, const float(&j)[3], const float(&F)[3]) {
    if (!live) return;
    const double rr = rho_r, rb = rho_b;
    const double ux = ((double)j[0] + 0.5 * F[0]) / rho, uy = ((double)j[1] + 0.5 * F[1]) / rho,
                 uz = ((double)j[2] + 0.5 * F[2]) / rho;
    const double p = rr * 9.0 * (1.0 - (double)A.pc.alpha_r) / 19.0 + rb * 9.0 * (1.0 - (double)A.pc.alpha_b) / 19.0;
    const double dx = gx - R.q.xc, dy = gy - R.q.yc, dz = z - R.q.zc;
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    const bool bad = !(rho > 0.0f) || isnan(rho_r) || isnan(rho_b) || isnan(j[0]) || isnan(j[1]) || isnan(j[2]);
    v[0] += rr;
    v[1] += rb;
    if (r <= R.q.r_in) {
      v[2] += p;
      v[3] += 1.0;
    }
    if (r >= R.q.r_out) {
      v[4] += p;
      v[5] += 1.0;
    }
    v[6] += bad ? 1.0 : 0.0;
    v[7] = fmax(v[7], bad ? 0.0 : sqrt(ux * ux + uy * uy + uz * uz));
  };
  auto consume = [&](int z, float rho, float rho_r, float rho_b, const float(&j)[3], bool inflow) {
    float F[3];
    body_force(A, rho, F);
    if (inflow) F[0] = F[1] = F[2] = 0.0f;  // read-back reports the set velocity (no F/2 shift)
    if constexpr (KIND == kScanCoarse)
      coarse_add(z, rho, rho_r, rho_b, j, F);
    else
      diag_add(z, rho, rho_r, rho_b, j, F);
  };

  if (!A.init_mode) {
    float st[3][KS][5];  // the first three planes at once
#pragma unroll
    for (int k = 0; k < 3; ++k) stage_load(z0 - 1 + k, st[k]);
#pragma unroll
    for (int k = 0; k < 3; ++k) stage_store(z0 - 1 + k, st[k]);
    __syncthreads();
  }
  const bool outflow = G.face_hi == FACE_OUTFLOW && !A.init_mode;
  const int sI = ly * SX + lx;  // the cell's corner (-1, -1) in a staged plane
  // the cell below, of which the outlet plane is formed (no chunk begins on that plane)
  float below_rho = 1.0f, below_r = 0.0f, below_b = 1.0f, below_e = 0.0f, below_j[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll 1
  for (int z = z0; z < z1; ++z) {
    float rho, rho_r, rho_b, e, j[3];
    bool inflow = false;
    if (A.init_mode) {
      const long long c = (long long)z * plane + col;
      float df[Q];
      init_cell<false>(A.init, A.pc, G.n, c, rho, rho_r, rho_b, e, df);
#pragma unroll
      for (int d = 0; d < 3; ++d) j[d] = rho * A.init[(2 + d) * G.n + c];
    } else {
      const bool outlet_z = outflow && z == G.nz - 1;
      float st[KS][5];
      stage_load(z + 2, st);
      if (!outlet_z) {
        typename Word<T>::W ld[Q];
        int ax = gx, ay = gy, wf = walls;
        asm volatile("" : "+v"(ax), "+v"(ay), "+v"(wf));  // offsets are formed per plane
        unsigned o[3][3];
        const int from = WALLS ? kMirrorSpan * pb : 0;
        column_offsets<T, WALLS>(G, ax, ay, from, o);
        const unsigned early = (unsigned)from;
        const rsrc_t slab[3] = {buffer_of(gin + (size_t)zsrc(z - 1) * slab_bytes - early, slab_bytes + early),
                                buffer_of(gin + (size_t)z * slab_bytes - early, slab_bytes + early),
                                buffer_of(gin + (size_t)zsrc(z + 1) * slab_bytes - early, slab_bytes + early)};
        const float4* const S[3] = {sS[(z - 1) & 3], sS[z & 3], sS[(z + 1) & 3]};
        const float2* const W[3] = {sW[(z - 1) & 3], sW[z & 3], sW[(z + 1) & 3]};
        with_mode(plane_mode(G, z), [&](auto M) {
          if constexpr (WALLS)
            issue_pull_walls<T, decltype(M)::value>(slab, pb, o, wf, ld);
          else
            issue_pull<T, decltype(M)::value>(slab, pb, o, ld);
          float df[Q], shift, drho;
          int b0 = sI;
          asm volatile("" : "+v"(b0));  // the modes' LDS reads are not merged above the switch
          finish_pull<T, decltype(M)::value, true, SX, 4>(ld, S, W, b0, A.pc, rho, rho_r, rho_b, e, df, shift, drho);
          // (the shift to the present rest equilibrium is isotropic and carries no momentum)
          j[0] = j[1] = j[2] = 0.0f;
#pragma unroll
          for (int i = 1; i < Q; i += 2) {  // populations i and i + 1 are opposite
            const float d = df[i] - df[i + 1];
            if (CX[i] != 0) j[0] += (float)CX[i] * d;
            if (CY[i] != 0) j[1] += (float)CY[i] * d;
            if (CZ[i] != 0) j[2] += (float)CZ[i] * d;
          }
        });
        below_rho = rho, below_r = rho_r, below_b = rho_b, below_e = e;
        below_j[0] = j[0], below_j[1] = j[1], below_j[2] = j[2];
      } else {
        // R11 on the totals: (previous record + lambda x the cell below) / (1 + lambda)
        int oc = col;
        asm volatile("" : "+v"(oc));  // the record's loads stay in this branch of the plane loop
        const float* rec = A.outlet_in + oc;
        float Fz = 0.0f;
        if (A.cp.force) Fz = (below_rho - A.cp.rho_ref) * A.cp.gz;
        float lam = (below_j[2] + 0.5f * Fz) / below_rho;
        lam = lam > 0.0f ? lam : 0.0f;
        const float inv = 1.0f / (1.0f + lam);
        j[0] = j[1] = j[2] = 0.0f;
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const float d = rec[i * plane] + rec[(Q + i) * plane];
          if (CX[i] != 0) j[0] += (float)CX[i] * d;
          if (CY[i] != 0) j[1] += (float)CY[i] * d;
          if (CZ[i] != 0) j[2] += (float)CZ[i] * d;
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) j[d] = (j[d] + lam * below_j[d]) * inv;
        const float e_prev = rec[54 * plane], psi_prev = rec[55 * plane];
        const float rho_prev = rho_of_psi(A.pc, e_prev, psi_prev);
        const float rr = (psi_a(psi_prev) * rho_prev + lam * below_r) * inv;
        const float rb = (psi_b(psi_prev) * rho_prev + lam * below_b) * inv;
        const float psi = psi_encode(rr, rb, rr + rb);
        rho = rho_of_psi(A.pc, (e_prev + lam * below_e) * inv, psi);
        rho_r = psi_a(psi) * rho;
        rho_b = psi_b(psi) * rho;
      }
      stage_store(z + 2, st);
    }
    if (is_inflow(G, gx, gy, z)) {
      inflow = true;
      rho = rho_r = G.rho_r0;
      rho_b = 0.0f;
      j[0] = j[1] = 0.0f;
      j[2] = G.rho_r0 * inflow_speed(G, col, A.step);
    }
    consume(z, rho, rho_r, rho_b, j, inflow);
    __syncthreads();
    if constexpr (KIND == kScanCoarse) coarse_put(z);
  }

  if constexpr (KIND == kScanDiag) {
    // part[block] = {mass_r, mass_b, p_in, n_in, p_out, n_out, bad cells, umax}: wave64 butterfly,
    // then across the 4 waves through LDS, in a fixed order
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        const double o = __shfl_xor(v[k], off, 64);
        v[k] = (k == 7) ? fmax(v[k], o) : v[k] + o;
      }
    }
    __shared__ double dred[4][8];
    if (lx == 0)
#pragma unroll
      for (int k = 0; k < 8; ++k) dred[ly][k] = v[k];
    __syncthreads();
    if (tid < 8) {
      double t = dred[0][tid];
      for (int w = 1; w < 4; ++w) t = (tid == 7) ? fmax(t, dred[w][tid]) : t + dred[w][tid];
      R.part[(long long)L * 8 + tid] = t;
    }
  }
}

template <typename T, int KIND>
hipError_t launch_scan(const AuxArgs& a, const ScanArgs& r, hipStream_t s) {
  const unsigned nb = (unsigned)((scan_blocks(r) + 7) / 8 * 8);
  if (a.geo.wall_x || a.geo.wall_y)
    hipLaunchKernelGGL((scan_kernel<T, true, KIND>), dim3(nb), dim3(ScanTile::NT), 0, s, a, r);
  else
    hipLaunchKernelGGL((scan_kernel<T, false, KIND>), dim3(nb), dim3(ScanTile::NT), 0, s, a, r);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse_T(const AuxArgs& a, int f, float inv_u, float* out, int ph, int pw, hipStream_t s) {
  if ((f == 1 && !scan_idle(a.geo)) || f == 2 || f == 4) {  // the factors that divide the tile
    ScanArgs r = scan_plan(a.geo, f, kScanCoarse);
    r.factor = f;
    r.inv_u = inv_u;
    r.out = out;
    r.ph = ph;
    r.pw = pw;
    return launch_scan<T, kScanCoarse>(a, r, s);
  }
  const long long nb = (long long)(a.geo.nx / f) * (a.geo.ny / f) * (a.geo.nz / f);
  hipLaunchKernelGGL(coarse_kernel<T>, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, s, a, f, inv_u, out, ph, pw);
  return hipGetLastError();
}

// part: 8 doubles for each of the diag_blocks(geo) blocks
template <typename T>
hipError_t launch_diag_T(const AuxArgs& a, const DiagQuery& q, double* part, double* out, hipStream_t s) {
  hipError_t e;
  if (scan_idle(a.geo)) {
    hipLaunchKernelGGL(diag_kernel<T>, dim3((unsigned)diag_blocks(a.geo)), dim3(256), 0, s, a, q, part);
    e = hipGetLastError();
  } else {
    ScanArgs r = scan_plan(a.geo, 1, kScanDiag);
    r.q = q;
    r.part = part;
    e = launch_scan<T, kScanDiag>(a, r, s);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(256), 0, s, part, diag_blocks(a.geo), out);
  return hipGetLastError();
}

#define LBM_INSTANTIATE_SCAN(T)                                                                       \
  template hipError_t launch_coarse_T<T>(const AuxArgs&, int, float, float*, int, int, hipStream_t); \
  template hipError_t launch_diag_T<T>(const AuxArgs&, const DiagQuery&, double*, double*, hipStream_t);

}  // namespace lbm
