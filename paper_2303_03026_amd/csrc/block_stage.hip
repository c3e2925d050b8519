// FP64 stage of the per-kernel path for blocks of any size (4 .. 16 cells a
// side) and the limiters of two ghost layers: conserved -> primitive, limited
// reconstruction, interface fluxes in every direction, flux difference, psi
// damping and the SSPRK combination of one block in one workgroup.
//
// It replaces launches that passed primitives and face fluxes through memory
// (a padded state written and read once per direction, three face arrays
// written and read: about 15 times the state, where this reads it once, with
// its neighbours' rims, and writes it once).  Van Leer + HLL, a captured
// SSPRK(2,2) step, before -> now: 512 blocks of 8^3 255 -> 101 us, of 16^3
// 1648 -> 427 us, 8 blocks of 16^3 103 -> 52; 1024 2D blocks of 8^2 (cada3 +
// HLLC) 98 -> 47 us; an SSPRK(3,3) step of 2309 blocks of 8^3 on three levels
// 2030 -> 560 us.
//
// What bounds it, by counters: memory traffic.  256^3 in blocks of 16^3 moves
// 7.1 (w = 1) and 8.8 GB (w < 1) a launch at 4.9 and 5.3 TB/s, where a device
// copy reaches 4.7, with 1478 and 1489 VALU instructions a cell, 37 to 43% of
// the issue peak; 2309 blocks of 8^3 move 0.9 GB at 4.9 TB/s, with 1900 VALU
// instructions a cell (halo cells and far faces of short lines), 31% of the
// peak, in 2309 waves on the 2048 places of two waves per SIMD (the 3D
// instances take 249 to 256 registers).
//
// Thread t of a workgroup owns the column (i, j) = (t % nx, t / nx) and
// marches through its planes; the z stencil is a register queue (as in the
// fused stage) and the x and y stencils read one LDS plane with its two-deep
// halo, filled from same-level neighbours in place and from the block's ghost
// cells on its other faces.  A thread evaluates the left
// x face and the lower y face of its cell; rows and waves do not coincide
// here, so the neighbours' faces come through LDS.  The far faces of the lines
// are evaluated once per plane, x and y in one pass (a y face is an x face
// with x and y exchanged).  Short blocks leave lanes idle (4^2 columns are a
// quarter of a wave); sharing a wave among blocks cost the scalar block
// address and spilled 18 to 120 registers, and gave nothing on 4096 blocks of
// 4^3 (791 us either way, with filled ghost cells).
#include "fused_lanes.h"
#include "kernels.h"

namespace amrvac {
namespace {

struct BlockShape {
  int nx;       // cells a side
  int cols;     // nx * nx (2D: nx * nx, one plane)
  int row;      // LDS row stride of a plane, in cells
  int nseg;     // workgroups per block, each marching its share of the planes (3D)
};

// Cells and faces lie in LDS with their
// nine variables together: the block size is a run-time value, and with one
// array per variable every access would need an address register of its own
// (the 3D instances spilled 150 to 260 registers).
template <int NDIM, int LIM, int FLX>
__global__ void __launch_bounds__(256, 2) k_stage_block(GridConst G, Tables T, JobScalars J, BlockShape S,
                                                        const double* __restrict__ in, const double* base, double* out,
                                                        double wgt, PhysConst P, DevStatus* st,
                                                        double* __restrict__ freg) {
  extern __shared__ double lds[];
  const int nx = S.nx, pn = G.pn, ng = G.ng, row = S.row * NV;
  const long PC = G.pcells;
  const int tc = threadIdx.x, blk = blockIdx.x / S.nseg, seg = blockIdx.x - blk * S.nseg;
  const bool live = tc < S.cols;  // (the other threads only take part in the barriers)
  const int b = T.order[blk];
  // the planes of this workgroup
  const int k0 = NDIM == 3 ? seg * nx / S.nseg : 0, k1 = NDIM == 3 ? (seg + 1) * nx / S.nseg : 1;
  // LDS: the plane, the x and y faces of its columns, the far faces of its
  // lines (x at l, y at nx + l)
  double* const Wp = lds;
  double* const Fx = Wp + NV * S.row * (nx + 4);
  double* const Fy = Fx + NV * S.cols;
  double* const Xf = Fy + NV * S.cols;
  const double* const U = in + (long)b * NV * PC;
  // from U to the values outside each face: the ghost cells, or the cells
  // themselves of a same-level neighbour
  long* const out_of = reinterpret_cast<long*>(Xf + 2 * NV * nx);
  auto outside = [&](int f) -> long {
    const int* L = T.link + ((long)b * 6 + f) * LINK_INTS;
    if (L[0] != LINK_SAME) return 0;
    const int step = f < 2 ? 1 : (f < 4 ? pn : pn * pn);
    return (long)(L[1] - b) * NV * PC + (f & 1 ? -nx : nx) * step;
  };
  if (tc < 4) out_of[tc] = outside(tc);
  const long below = NDIM == 3 ? outside(4) : 0, above = NDIM == 3 ? outside(5) : 0;
  auto cell = [&](int x, int y, int z) { return ((NDIM == 3 ? z + ng : 0) * pn + y + ng) * pn + x + ng; };
  auto at = [&](int x, int y) { return (y + 2) * row + (x + 2) * NV; };
  int bad = 0;
  unsigned nfix = 0;
  auto convert = [&](const double u[NV], double w[NV], bool count) {
    const int f = cons_to_prim(u, w, P);
    if (f && count) {
      bad |= f;
      if (P.fix) ++nfix;
    }
  };
  // whether plane z, which two marches may convert, counts as this one's
  auto owns = [&](int z) { return (z >= k0 || k0 == 0) && (z < k1 || k1 == nx); };
  auto load = [&](const double* s, int c, double u[NV]) {
#pragma unroll
    for (int q = 0; q < NV; ++q) u[q] = s[q * PC + c];
  };
  auto load_z = [&](int i, int j, int z, double u[NV]) {
    load(U + (z < 0 ? below : z >= nx ? above : 0), cell(i, j, z), u);
  };
  // flux registers of the faces towards finer or coarser leaves
  const int nfc = NDIM == 3 ? nx * nx : nx;
  unsigned regs = 0;
  if (freg && live) {
#pragma unroll
    for (int f = 0; f < 2 * NDIM; ++f) {
      const int kd = T.link[((long)b * 6 + f) * LINK_INTS];
      if (kd == LINK_FINE || kd == LINK_COARSE) regs |= 1u << f;
    }
  }
  auto put_reg = [&](int f, int c, const double F[NV], int swap) {
    double* p = freg + ((long)b * 6 + f) * NV * nfc + c;
#pragma unroll
    for (int q = 0; q < NV; ++q) p[swap_xy(q, swap) * nfc] = F[q];
  };
  const int job = T.job[b];
  const double dt = J.dt_scale * J.dt[job], kappa = J.kappa[job], ch = J.ch[job], hic = 0.5 / ch;
  const double idx = T.inv_dx[3 * b], idy = T.inv_dx[3 * b + 1], idz = T.inv_dx[3 * b + 2];
  // a plane's 8 nx halo cells (two layers on four sides) into LDS; of a third
  // ghost layer only the check of its values
  auto halo = [&](int z, int tc) {
    for (int h = tc; h < 4 * ng * nx; h += S.cols) {
      int r = h, a = 0;  // layer outwards, then side, then position
      for (; r >= 4 * nx; r -= 4 * nx) ++a;
      const int side = r / nx, n = r - side * nx;
      const int o = side & 1 ? nx + a : -1 - a;
      const int x = side < 2 ? o : n, y = side < 2 ? n : o;
      double u[NV], w[NV];
      load(U + out_of[side], cell(x, y, z), u);
      convert(u, w, true);
      if (a < 2) {
#pragma unroll
        for (int q = 0; q < NV; ++q) Wp[at(x, y) + q] = w[q];
      }
    }
  };
  // flux of the face between the plane's cells c + s and c + 2 s of the line
  // c, c + s, c + 2 s, c + 3 s, in the frame of direction DIR
  auto face = [&](auto dir, int c, int s, int swap, double F[NV]) {
    constexpr int DIR = decltype(dir)::value;
    double wl[NV], wr[NV];
    for_increments<LIM, double>(
        [&](int q, double& m, double& w, double& p) {
          const double* v = Wp + c + swap_xy(q, swap);
          m = v[0];
          w = v[s];
          p = v[2 * s];
        },
        [&](int q, double w, double r, double) { wl[q] = w + r; });
    for_increments<LIM, double>(
        [&](int q, double& m, double& w, double& p) {
          const double* v = Wp + c + swap_xy(q, swap);
          m = v[s];
          w = v[2 * s];
          p = v[3 * s];
        },
        [&](int q, double w, double, double l) { wr[q] = w - l; });
    const bool low = !((wl[I_RHO] > 0.0) && (wl[4] > 0.0) && (wr[I_RHO] > 0.0) && (wr[4] > 0.0));
    if (__any(low)) {
      asm volatile("");  // keeps the branch wave-uniform
      if (low) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          wl[q] = Wp[c + s + swap_xy(q, swap)];
          wr[q] = Wp[c + 2 * s + swap_xy(q, swap)];
        }
      }
    }
    face_flux<FLX, DIR, double>(wl, wr, ch, hic, P.gamma, P.inv_gm1, F);
  };
  using DX = std::integral_constant<int, 0>;
  using DY = std::integral_constant<int, 1>;

  // z queue: W(k+1), the left state of face k+1/2 and the flux differences,
  // which enter plane k holding -F_z(k-1/2)/dz
  lds_barrier();  // out_of is there
  double wb[NV], wla[NV], acc[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) acc[q] = 0.0;
  if (live) {
    const int i = tc % nx, j = tc / nx;
    double u[NV], wa[NV];
    load(U, cell(i, j, k0), u);
    convert(u, wa, true);
#pragma unroll
    for (int q = 0; q < NV; ++q) Wp[at(i, j) + q] = wa[q];
    if (NDIM == 3) {
      double wm2[NV], wm1[NV], wl[NV], wr[NV];
      load_z(i, j, k0 - 2, u);
      convert(u, wm2, k0 == 0);
      load_z(i, j, k0 - 1, u);
      convert(u, wm1, k0 == 0);
      load_z(i, j, k0 + 1, u);
      convert(u, wb, owns(k0 + 1));
      for_increments<LIM, double>([&](int q, double& m, double& w, double& p) { m = wm2[q]; w = wm1[q]; p = wa[q]; },
                                  [&](int q, double w, double r, double) { wl[q] = w + r; });
      for_increments<LIM, double>([&](int q, double& m, double& w, double& p) { m = wm1[q]; w = wa[q]; p = wb[q]; },
                                  [&](int q, double w, double r, double l) {
                                    wr[q] = w - l;
                                    wla[q] = w + r;
                                  });
      positivity_fallback(wl, wr, wm1, wa);
      face_flux<FLX, 2, double>(wl, wr, ch, hic, P.gamma, P.inv_gm1, acc);
      if ((regs & 16u) && k0 == 0) put_reg(4, j * nx + i, acc, 0);
#pragma unroll
      for (int q = 0; q < NV; ++q) acc[q] = -(acc[q] * idz);
    }
    if (NDIM == 3 && ng > 2) {
      if (k0 == 0) {
        load_z(i, j, -3, u);
        convert(u, wa, true);
      }
      if (k1 == nx) {
        load_z(i, j, nx + 2, u);
        convert(u, wa, true);
      }
    }
    halo(k0, tc);
  }
  const int tcol = tc;
  for (int k = k0; k < k1; ++k) {
    // the column again, for this plane's addresses (see the fused stage)
    int tc = tcol;
    if (NDIM == 3) asm volatile("" : "+v"(tc));
    const int i = tc % nx, j = tc / nx;
    const int kofs = NDIM == 3 ? k * nx : 0;
    lds_barrier();  // the plane is complete
    if (live) {
      for (int l = tc; l < 2 * nx; l += S.cols) {  // far faces: x lines, then y lines
        const int y = l >= nx ? 1 : 0, n = l - y * nx;
        double F[NV];
        face(DX{}, y ? at(n, nx - 2) : at(nx - 2, n), y ? row : NV, y, F);
#pragma unroll
        for (int q = 0; q < NV; ++q) Xf[l * NV + swap_xy(q, y)] = F[q];
        if ((regs >> (y ? 3 : 1)) & 1u) put_reg(y ? 3 : 1, kofs + n, F, y);
      }
      double F[NV];
      face(DX{}, at(i - 2, j), NV, 0, F);
#pragma unroll
      for (int q = 0; q < NV; ++q) Fx[tc * NV + q] = F[q];
      if ((regs & 1u) && i == 0) put_reg(0, kofs + j, F, 0);
      face(DY{}, at(i, j - 2), row, 0, F);
#pragma unroll
      for (int q = 0; q < NV; ++q) Fy[tc * NV + q] = F[q];
      if ((regs & 4u) && j == 0) put_reg(2, kofs + i, F, 0);
    }
    lds_barrier();  // every face of the plane is there
    if (live) {
      const double* xn = i + 1 < nx ? Fx + (tc + 1) * NV : Xf + j * NV;
      const double* yn = j + 1 < nx ? Fy + (tc + nx) * NV : Xf + (nx + i) * NV;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        acc[q] = acc[q] + (xn[q] - Fx[tc * NV + q]) * idx;
        acc[q] = acc[q] + (yn[q] - Fy[tc * NV + q]) * idy;
      }
      const int c = cell(i, j, k);
      double fz[NV];
      if (NDIM == 3) {
        // (plane k+2 loaded here, not a plane's faces ahead: no registers are
        // left for it, and the spills took 512 blocks of 8^3 108 against 101 us)
        double uc[NV], wa[NV], wc[NV], wl[NV], wr[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) wa[q] = Wp[at(i, j) + q];
        load_z(i, j, k + 2, uc);
        convert(uc, wc, owns(k + 2));
        for_increments<LIM, double>([&](int q, double& m, double& w, double& p) { m = wa[q]; w = wb[q]; p = wc[q]; },
                                    [&](int q, double w, double r, double l) {
                                      wl[q] = wla[q];
                                      wr[q] = w - l;
                                      wla[q] = w + r;
                                    });
        positivity_fallback(wl, wr, wa, wb);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          Wp[at(i, j) + q] = wb[q];  // W(k+1): the next plane's own cell
          wb[q] = wc[q];
        }
        face_flux<FLX, 2, double>(wl, wr, ch, hic, P.gamma, P.inv_gm1, fz);
        if ((regs & 32u) && k == nx - 1) put_reg(5, j * nx + i, fz, 0);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          fz[q] = fz[q] * idz;
          acc[q] = acc[q] + fz[q];
        }
      }
      double u[NV], ub[NV];
      load(U, c, u);
      if (wgt != 1.0) load(base + (long)b * NV * PC, c, ub);
      double* const ob = out + (long)b * NV * PC;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        double lq = -acc[q];
        if (q == I_PSI) lq = lq - kappa * u[I_PSI];
        const double tq = u[q] + dt * lq;
        const double r = wgt == 1.0 ? tq : ub[q] + wgt * (tq - ub[q]);
        ob[q * PC + c] = r;
        if (NDIM == 3) acc[q] = -fz[q];
      }
      if (NDIM == 3 && k + 1 < k1) halo(k + 1, tc);
    }
  }
  if (bad) atomicOr(&st->flags, (unsigned)bad);
  if (nfix) atomicAdd(&st->nfix, (unsigned long long)nfix);
}

template <int NDIM, int LIM>
hipError_t launch_flux_of(hipStream_t s, const GridConst& G, const Tables& T, const JobScalars& J, const BlockShape& S,
                          const double* in, const double* base, double* out, double w, const PhysConst& P,
                          DevStatus* st, double* freg) {
  const unsigned grid = (unsigned)(T.nactive * S.nseg);
  const unsigned threads = (unsigned)((S.cols + 63) / 64 * 64);
  const size_t bytes = (size_t)NV * (S.row * (S.nx + 4) + 2 * S.cols + 2 * S.nx) * sizeof(double) + 4 * sizeof(long);
#define AMRVAC_BLOCK_LAUNCH(FX) \
  k_stage_block<NDIM, LIM, FX><<<grid, threads, bytes, s>>>(G, T, J, S, in, base, out, w, P, st, freg)
  if (P.flux == FLUX_HLLD)
    AMRVAC_BLOCK_LAUNCH(FLUX_HLLD);
  else if (P.flux == FLUX_HLLC)
    AMRVAC_BLOCK_LAUNCH(FLUX_HLLC);
  else
    AMRVAC_BLOCK_LAUNCH(FLUX_HLL);
#undef AMRVAC_BLOCK_LAUNCH
  return hipGetLastError();
}

}  // namespace

hipError_t launch_block_stage(hipStream_t s, const GridConst& G, const Tables& T, const JobScalars& J, const void* in,
                              const void* base, void* out, double w, const PhysConst& P, DevStatus* st,
                              double* freg) {
  if (G.ng < 2 || G.nx < 4 || G.nx > 16 || G.precision != 0 || P.limiter >= LIM_WENO5) return hipErrorInvalidValue;
  if (T.nactive <= 0) return hipSuccess;
  BlockShape S;
  S.nx = G.nx;
  S.cols = G.nx * G.nx;
  S.row = G.nx + 5;  // odd for even nx: columns fall on distinct banks
  // Small grids: more, shorter marches, until there is a wave per SIMD (each
  // march converts four planes before its first face, so no further: 512
  // blocks of 8^3 took 311 us per step with 2 marches, 327 with 4; 8 blocks
  // of 16^3 took 103 us with 4, 62 with 16, and 120 before; ghost cells of
  // same-level faces filled).
  const long waves = (long)T.nactive * ((S.cols + 63) / 64);
  S.nseg = 1;
  while (G.ndim == 3 && S.nseg < G.nx && waves * S.nseg < 1024) ++S.nseg;
  const double *pi = static_cast<const double*>(in), *pb = static_cast<const double*>(base);
  double* po = static_cast<double*>(out);
#define AMRVAC_BLOCK_LIM(ND)                                                                              \
  (P.limiter == LIM_KOREN   ? launch_flux_of<ND, LIM_KOREN>(s, G, T, J, S, pi, pb, po, w, P, st, freg)    \
   : P.limiter == LIM_CADA3 ? launch_flux_of<ND, LIM_CADA3>(s, G, T, J, S, pi, pb, po, w, P, st, freg)    \
                            : launch_flux_of<ND, LIM_VANLEER>(s, G, T, J, S, pi, pb, po, w, P, st, freg))
  return G.ndim == 3 ? AMRVAC_BLOCK_LIM(3) : AMRVAC_BLOCK_LIM(2);
#undef AMRVAC_BLOCK_LIM
}

}  // namespace amrvac
