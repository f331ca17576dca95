// HIP kernels (gfx950) of the library other than collide-and-stream:
// reductions, initial data, read-out and state access, the adjoint sweep and
// the plain copy kernel used as the bandwidth reference.
#include <algorithm>

#include "lbm_device.h"

namespace mclbm {
namespace {

// Records from the block partials, in two stages where a sample has more than
// kRecordChunk blocks: each block of the first adds up kRecordChunk rows in place,
// into the first of them (which no other block touches), and the second stage
// takes one block per segment over those rows. One block over the 65536 rows of
// a 256^3 sample took 96 us; the two stages take 9.
constexpr int kRecordChunk = 1024;

__device__ __forceinline__ void add_record_rows(const double* rows, int count, size_t stride, double (&res)[kRecord]) {
  double v[kRecord] = {0, 0, 0, 0, 0, 0, 1e300, -1e300};
  for (int k = threadIdx.x; k < count; k += 256) {
    const double* p = rows + size_t(k) * stride * kRecord;
#pragma unroll
    for (int q = 0; q < 6; ++q) v[q] += p[q];
    v[6] = fmin(v[6], p[6]);
    v[7] = fmax(v[7], p[7]);
  }
  block_record<256>(v, res);
}

__global__ void __launch_bounds__(256)
    record_chunk_kernel(double* partials, const Seg* segs, int nseg, int total_blocks) {
  const BlockChunk c = chunk_in_window(segs, nseg, total_blocks, kRecordChunk, blockIdx.x);
  if (c.count == 0) return;
  double* rows = partials + size_t(c.first) * kRecord;
  double res[kRecord];
  add_record_rows(rows, c.count, 1, res);
  if (threadIdx.x == 0) {  // after the barrier of the reduction: every row is read
#pragma unroll
    for (int q = 0; q < kRecord; ++q) rows[q] = res[q];
  }
}

__global__ void __launch_bounds__(256)
    record_finalize_kernel(const double* partials, const Seg* segs, const DevSample* samples, double* out) {
  const Seg sg = segs[blockIdx.x];
  const bool chunked = sg.nblocks > kRecordChunk;
  double res[kRecord];
  add_record_rows(partials + size_t(sg.first_block) * kRecord,
                  chunked ? (sg.nblocks + kRecordChunk - 1) / kRecordChunk : sg.nblocks, chunked ? kRecordChunk : 1, res);
  if (threadIdx.x == 0) {
    const DevSample& sp = samples[sg.sample];
    const double ncell = double(uint64_t(1) << (3 * sp.log2n));
    double* o = out + size_t(sg.sample) * kRecord;
    o[0] = ncell + res[0];
    o[1] = res[1];
    o[2] = res[2];
    o[3] = res[3];
    o[4] = res[4] / ncell;
    o[5] = res[6];
    o[6] = res[7];
    o[7] = res[5] / ncell;
  }
}

// ---------------------------------------------------------------- initial data
// u0(x) = u0 [TGV(x) + amp * s(x)] with s from the (projected) coefficients yc[24].
// The kernels of the initial data take groups of 256 consecutive nodes, `per` of
// them per block, and look sin and cos up in a table of the block: 11 of them
// per node in double cost more than the rest of the node's work (init of
// 1000 x 32^3 D3Q19 in float 613 -> 432 us).
constexpr int kMaxN = 1024;

// sc[k] = (sin, cos) of 2 pi k / n; sin(2 x_k) is the entry of 2 k
__device__ __forceinline__ void make_axis_table(double2* sc, int n) {
  for (int k = threadIdx.x; k < n; k += 256) sc[k] = make_double2(sinpi(2.0 * k / n), cospi(2.0 * k / n));
}

__device__ __forceinline__ void initial_velocity(const double2& x1, const double2& x2, const double2& y1,
                                                 const double2& y2, const double2& z1, const double2& z2, double u0,
                                                 double amp, const double* yc, double (&u)[3]) {
  const double a[3][2] = {{x2.x, x2.y}, {y2.x, y2.y}, {z2.x, z2.y}};  // sin(2 x_axis), cos(2 x_axis)
  double s[3] = {0.0, 0.0, 0.0};
  for (int al = 0; al < 3; ++al)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j)
        for (int k = 0; k < 2; ++k) s[al] += yc[8 * al + 4 * i + 2 * j + k] * a[0][i] * a[1][j] * a[2][k];
  u[0] = u0 * (x1.x * y1.y * z1.y + amp * 0.125 * s[0]);
  u[1] = u0 * (-x1.y * y1.x * z1.y + amp * 0.125 * s[1]);
  u[2] = u0 * (amp * 0.125 * s[2]);
}

template <int QN, typename T>
__global__ void __launch_bounds__(256)
    init_kernel(T* __restrict__ pop, const DevSample* __restrict__ samples, const Seg* __restrict__ segs, int nseg, int per,
                const double* __restrict__ ycoef) {
  __shared__ double2 sc[kMaxN];
  const Seg sg = segs[find_segment(segs, nseg, int(blockIdx.x) * per)];
  const int first = int(blockIdx.x) * per - sg.first_block, last = first + per;
  const DevSample& sp = samples[sg.sample];
  const int l = sp.log2n, n = 1 << l, msk = n - 1;
  make_axis_table(sc, n);
  __syncthreads();
  const double* yc = ycoef + size_t(sg.sample) * 24;
  T* base = pop + sp.offset;
  for (int b = first; b < last; ++b) {
    const uint32_t cell = uint32_t(b) * 256u + threadIdx.x;
    const int x = int(cell) & msk, y = int(cell >> l) & msk, z = int(cell >> (2 * l));
    double u[3];
    initial_velocity(sc[x], sc[(2 * x) & msk], sc[y], sc[(2 * y) & msk], sc[z], sc[(2 * z) & msk], sp.u0, sp.amp, yc, u);
    const double usq15 = 1.5 * (u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const double cu = double(cx(i)) * u[0] + double(cy(i)) * u[1] + double(cz(i)) * u[2];
      const double gi = weight<QN>(i) * (3.0 * cu + 4.5 * cu * cu - usq15);
      st(base + size_t(plane_of<QN>(i)) * sp.pstride, cell, T(gi));
    });
  }
}

// ---------------------------------------------------------------- read-out and state access
template <int QN, typename T>
__global__ void __launch_bounds__(256)
    moments_kernel(const T* pop, const DevSample* samples, int sample, int parity, double* rho, double* u) {
  const DevSample& sp = samples[sample];
  const int l = sp.log2n;
  const uint32_t ncell = 1u << (3 * l);
  const Cell c = make_cell(blockIdx.x * 256u + threadIdx.x, l);
  T g[Q];
  load_state<QN>(pop + sp.offset, sp.pstride, c, parity & 1, g);
  double d = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double v = double(g[i]);
    d += v;
    if constexpr (cx(i) != 0) jx += cx(i) * v;
    if constexpr (cy(i) != 0) jy += cy(i) * v;
    if constexpr (cz(i) != 0) jz += cz(i) * v;
  });
  const double r = 1.0 + d;
  if (rho) rho[c.cell] = r;
  if (u) {
    u[c.cell] = jx / r;
    u[size_t(ncell) + c.cell] = jy / r;
    u[2 * size_t(ncell) + c.cell] = jz / r;
  }
}

template <int QN, typename T>
__global__ void __launch_bounds__(256)
    get_state_kernel(const T* pop, const DevSample* samples, int sample, int parity, double* f) {
  const DevSample& sp = samples[sample];
  const int l = sp.log2n;
  const uint32_t ncell = 1u << (3 * l);
  const Cell c = make_cell(blockIdx.x * 256u + threadIdx.x, l);
  T g[Q];
  load_state<QN>(pop + sp.offset, sp.pstride, c, parity & 1, g);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    f[size_t(plane_of<QN>(i)) * ncell + c.cell] = weight<QN>(i) + double(g[i]);
  });
}

template <int QN, typename T>
__global__ void __launch_bounds__(256)
    set_state_kernel(T* pop, const DevSample* samples, int sample, int parity, const double* f) {
  const DevSample& sp = samples[sample];
  const int l = sp.log2n;
  const uint32_t ncell = 1u << (3 * l);
  const Cell c = make_cell(blockIdx.x * 256u + threadIdx.x, l);
  T g[Q];
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    g[i] = T(f[size_t(plane_of<QN>(i)) * ncell + c.cell] - weight<QN>(i));
  });
  write_state<QN>(pop + sp.offset, sp.pstride, c, parity & 1, g);
}

// Populations (unshifted, double) of selected cells of one sample: f[k][27].
template <int QN, typename T>
__global__ void __launch_bounds__(64)
    gather_cells_kernel(const T* pop, const DevSample* samples, int sample, int parity, const int64_t* cells,
                        int count, double* f) {
  const int k = blockIdx.x * 64 + threadIdx.x;
  if (k >= count) return;
  const DevSample& sp = samples[sample];
  const int l = sp.log2n;
  const Cell c = make_cell(uint32_t(cells[k]), l);
  T g[Q];
  load_state<QN>(pop + sp.offset, sp.pstride, c, parity & 1, g);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    f[size_t(k) * QN + plane_of<QN>(i)] = weight<QN>(i) + double(g[i]);
  });
}

template <int QN, typename T>
__global__ void poison_kernel(T* pop, const DevSample* samples, int sample, int parity, uint32_t cell, int k) {
  const DevSample& sp = samples[sample];
  const int l = sp.log2n;
  const Cell c = make_cell(cell, l);
  T* base = pop + sp.offset;
  const T nan = T(__builtin_nan(""));
  const int i = velocity_of_plane<QN>(k);
  // slot of population i of this node (see load_state)
  if (!(parity & 1)) {
    base[size_t(k) * sp.pstride + cell] = nan;
  } else {
    const uint32_t nb = c.oz[1 - cz(i)] + c.oy[1 - cy(i)] + c.ox[1 - cx(i)];
    base[size_t(plane_of<QN>(opposite(i))) * sp.pstride + nb] = nan;
  }
}

template <int QN, typename T>
__global__ void __launch_bounds__(256)
    canonical_copy_kernel(const T* pop, T* dst, const DevSample* samples, const Seg* segs, int nseg) {
  const int b = blockIdx.x;
  const Seg sg = segs[find_segment(segs, nseg, b)];
  const DevSample& sp = samples[sg.sample];
  const int l = sp.log2n;
  const Cell c = make_cell(uint32_t(b - sg.first_block) * 256u + threadIdx.x, l);
  T g[Q];
  load_state<QN>(pop + sp.offset, sp.pstride, c, sg.parity & 1, g);
  write_state<QN>(dst + sp.offset, sp.pstride, c, false, g);
}

// Adjoint vectors lam[q][n^3] (double, the population order of get_state)
// into or out of the natural layout of the storage type. No shift: an
// adjoint is a derivative, which the constant weights do not enter.
template <int QN, typename T>
__global__ void __launch_bounds__(256) put_adjoint_kernel(T* dst, const DevSample* samples, int sample,
                                                          const double* lam) {
  const DevSample& sp = samples[sample];
  const uint32_t ncell = 1u << (3 * sp.log2n);
  const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
  for_vel<QN>([&](auto ic) {
    constexpr int k = plane_of<QN>(decltype(ic)::value);
    dst[sp.offset + size_t(k) * sp.pstride + cell] = T(lam[size_t(k) * ncell + cell]);
  });
}

template <int QN, typename T>
__global__ void __launch_bounds__(256) get_adjoint_kernel(const T* src, const DevSample* samples, int sample,
                                                          double* lam) {
  const DevSample& sp = samples[sample];
  const uint32_t ncell = 1u << (3 * sp.log2n);
  const uint32_t cell = blockIdx.x * 256u + threadIdx.x;
  for_vel<QN>([&](auto ic) {
    constexpr int k = plane_of<QN>(decltype(ic)::value);
    lam[size_t(k) * ncell + cell] = double(src[sp.offset + size_t(k) * sp.pstride + cell]);
  });
}

// ---------------------------------------------------------------- adjoint
// Seed: J = (1/M) sum_m KE_m with KE = (1/n^3) sum_x |u|^2 / 2, u = j / rho:
// dJ/dg_i(x) = (1 / (M n^3)) (c_i . u - |u|^2) / rho.
template <int QN, typename T>
__global__ void __launch_bounds__(256) adjoint_seed_kernel(const T* pop, T* lam, const DevSample* samples,
                                                           const Seg* segs, int nseg, double inv_m) {
  const int b = blockIdx.x;
  const Seg sg = segs[find_segment(segs, nseg, b)];
  const DevSample& sp = samples[sg.sample];
  const int l = sp.log2n;
  const uint32_t ncell = 1u << (3 * l);
  const Cell c = make_cell(uint32_t(b - sg.first_block) * 256u + threadIdx.x, l);
  T g[Q];
  load_state<QN>(pop + sp.offset, sp.pstride, c, sg.parity & 1, g);
  double d = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double v = double(g[i]);
    d += v;
    if constexpr (cx(i) != 0) jx += cx(i) * v;
    if constexpr (cy(i) != 0) jy += cy(i) * v;
    if constexpr (cz(i) != 0) jz += cz(i) * v;
  });
  const double rho = 1.0 + d;
  const double ux = jx / rho, uy = jy / rho, uz = jz / rho;
  const double usq = ux * ux + uy * uy + uz * uz;
  const double coef = inv_m / double(ncell) / rho;
  T* lb = lam + sp.offset;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double cu = double(cx(i)) * ux + double(cy(i)) * uy + double(cz(i)) * uz;
    st(lb + size_t(plane_of<QN>(i)) * sp.pstride, c.cell, T(coef * (cu - usq)));
  });
}

// One reverse step: lambda_n(x) = (d collide / d g_n(x))^T [lambda_{n+1, i}(x + c_i)]_i,
// the transpose of "collide at x, then move population i to x + c_i".
// EXACT: the collision with the exact stabiliser of eq. (kbc_entropy), whose
// t = omega gamma / 2 is the root of F(t) = sum_i dh_i ln(f*_i / w_i) with
// f*_i = w_i + g_i - omega ds_i - t dh_i; by the implicit function theorem
// dt = (dF at fixed t) / D, D = sum_i dh_i^2 / f*_i, so the adjoint of t
// reaches F's inputs (dh, ds and g directly) with weight tbar / D.
// ARGS: the launch table comes as kernel arguments, as in the step kernels.
template <int QN, typename T, int BLOCK, bool BUF, bool EXACT, bool ARGS>
__global__ void __launch_bounds__(BLOCK) adjoint_step_kernel(const T* state, const T* lam_in, T* lam_out,
                                                           const DevSample* samples, const Seg* segs,
                                                           UniformSegs uniform, int nseg) {
  const BlockSite site = ARGS ? block_site(uniform, blockIdx.x) : block_site(segs, nseg, samples, blockIdx.x);
  const int l = site.log2n;
  const Cell c = make_cell(site.local_block * uint32_t(BLOCK) + threadIdx.x, l);
  const Relax<T> rp = relax_of<T>(samples[site.sample]);
  // every array is streamed once per reverse step: non-temporal accesses
  using Planes = typename std::conditional<BUF, BufPlanes<T, true, QN>, PtrPlanes<T, true, QN>>::type;
  const Planes st_in(const_cast<T*>(state) + site.offset, site.pstride);
  const Planes lam_src(const_cast<T*>(lam_in) + site.offset, site.pstride);
  const Planes lam_dst(lam_out + site.offset, site.pstride);

  // lambda is pulled from x + c_i; rows longer than a wave (and held whole by
  // the block) are read at the node's own x and shifted by lane exchange
  const uint32_t n = 1u << l;
  const bool rows = n > 64u && n <= uint32_t(BLOCK);
  __shared__ EdgeLds<T, BLOCK> edge;
  T g[Q], nu[Q];
  if (rows) {
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      g[i] = st_in.load(i, c.cell);
      nu[i] = lam_src.load(i, neighbour_yz<i, +1>(c));
    });
    row_shift<QN, -1, BLOCK>(nu, edge, n);
  } else {
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      g[i] = st_in.load(i, c.cell);
      nu[i] = lam_src.load(i, neighbour<i, +1>(c));
    });
  }

  // forward intermediates, as in kbc_collide
  const Macro<T> m = macroscopic<QN>(g);
  T fneq[Q];
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    fneq[i] = g[i] - geq<QN, i>(m);
  });
  const Shear<T> s = shear_coefficients<QN>(fneq);
  T A = T(0), B = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const T r = recip(T(weight<QN>(i)) + geq<QN, i>(m));
    if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) {
      const T ds = shear_part<i>(s);
      const T dh = fneq[i] - ds;
      A += ds * dh * r;
      B += dh * dh * r;
    } else {
      B += fneq[i] * fneq[i] * r;
    }
  });
  const bool active = B > equilibrium_threshold<T>(m);  // as in the forward collision
  T gamma = T(2);
  if (active) gamma = rp.two_over_omega - rp.kappa * (A / B);
  T t = T(0.5) * rp.omega * gamma;
  if constexpr (EXACT) {
    // the forward collision's t, from the same start and with the same steps
    if (active) {
      T ge[Q], dh[Q], bs[Q];
      for_vel<QN>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        ge[i] = geq<QN, i>(m);
      });
      exact_terms<QN>(ge, fneq, s, rp.eps, dh, bs);
      t = exact_entropic_t<QN>(dh, bs, m, t);
    }
  }

  // reverse sweep (the direct path of g* = g - omega ds - t dh hands nu to g
  // unchanged; tbar is the adjoint of t)
  T tbar = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) tbar -= nu[i] * (fneq[i] - shear_part<i>(s));
    else tbar -= nu[i] * fneq[i];
  });
  T Abar = T(0), Bbar = T(0), Fbar = T(0);
  if (active) {
    if constexpr (EXACT) {
      T d = T(0);
      for_vel<QN>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        T ds = T(0);
        if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) ds = shear_part<i>(s);
        const T dh = fneq[i] - ds;
        const T gs = (((geq<QN, i>(m) - ds) + rp.eps * ds) + dh) - t * dh;  // f*_i - w_i
        d += dh * dh * recip(T(weight<QN>(i)) + gs);
      });
      Fbar = tbar / d;
    } else {
      const T gbar = T(0.5) * rp.omega * tbar;
      Abar = -rp.kappa * gbar / B;
      Bbar = rp.kappa * gbar * (A / B) / B;  // B * B would underflow in float
    }
  }
  // adjoints of fneq (through dh and the weights) and of the shear coefficients
  T fbar[Q], geqbar[Q];
  T dsxb = T(0), dsyb = T(0), dszb = T(0), exyb = T(0), exzb = T(0), eyzb = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    T dsb, dhb;
    if constexpr (EXACT) {
      // dF = sum_i [ln(f*_i / w_i) - t dh_i / f*_i] d(dh_i) - omega dh_i / f*_i d(ds_i)
      //      + dh_i / f*_i d(g_i), with g_i = g^eq_i + fneq_i
      T ds = T(0);
      if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) ds = shear_part<i>(s);
      const T dh = fneq[i] - ds;
      T x = T(0), lg = T(0);
      if (active) {
        constexpr double w = weight<QN>(i);
        const T gs = geq<QN, i>(m) + (fneq[i] - rp.omega * ds) - t * dh;
        x = Fbar * dh * recip(T(w) + gs);
        lg = Fbar * log1p_acc(gs * T(1.0 / w));
      }
      if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) dsb = -rp.omega * nu[i] - rp.omega * x;
      else dsb = T(0);
      dhb = -t * nu[i] + lg - t * x;
      geqbar[i] = x;
      fbar[i] = dhb + x;
    } else {
      const T r = recip(T(weight<QN>(i)) + geq<QN, i>(m));
      T rbar;
      T ds = T(0), dh;
      if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) {
        ds = shear_part<i>(s);
        dh = fneq[i] - ds;
        dsb = -rp.omega * nu[i] + Abar * dh * r;
        dhb = -t * nu[i] + Abar * ds * r + T(2) * Bbar * dh * r;
        rbar = Abar * ds * dh + Bbar * dh * dh;
      } else {
        dh = fneq[i];
        dsb = T(0);
        dhb = -t * nu[i] + T(2) * Bbar * dh * r;
        rbar = Bbar * dh * dh;
      }
      geqbar[i] = -rbar * r * r;  // through f^eq = w + g^eq
      fbar[i] = dhb;              // dh = fneq - ds
    }
    dsb -= dhb;
    if constexpr (nonzeros(i) == 1) {
      if constexpr (cx(i) != 0) dsxb += dsb;
      else if constexpr (cy(i) != 0) dsyb += dsb;
      else dszb += dsb;
    } else if constexpr (nonzeros(i) == 2) {
      if constexpr (cz(i) == 0) exyb += signed_term<cx(i) * cy(i)>(dsb);
      else if constexpr (cy(i) == 0) exzb += signed_term<cx(i) * cz(i)>(dsb);
      else eyzb += signed_term<cy(i) * cz(i)>(dsb);
    }
  });
  // dsz = -(dsx + dsy); dsx = (2 Nxz - Nyz)/6; dsy = (2 Nyz - Nxz)/6
  const T dsxt = dsxb - dszb, dsyt = dsyb - dszb;
  const T sixth = T(1) / T(6);
  const T nxzb = (T(2) * dsxt - dsyt) * sixth;
  const T nyzb = (T(2) * dsyt - dsxt) * sixth;
  const T pxxb = nxzb, pyyb = nyzb, pzzb = -(nxzb + nyzb);
  const T pxyb = T(0.25) * exyb, pxzb = T(0.25) * exzb, pyzb = T(0.25) * eyzb;
  // second moments of fneq
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    T acc = fbar[i];
    if constexpr (cx(i) != 0) acc += pxxb;
    if constexpr (cy(i) != 0) acc += pyyb;
    if constexpr (cz(i) != 0) acc += pzzb;
    if constexpr (cx(i) * cy(i) != 0) acc += signed_term<cx(i) * cy(i)>(pxyb);
    if constexpr (cx(i) * cz(i) != 0) acc += signed_term<cx(i) * cz(i)>(pxzb);
    if constexpr (cy(i) * cz(i) != 0) acc += signed_term<cy(i) * cz(i)>(pyzb);
    fbar[i] = acc;
    geqbar[i] -= acc;  // fneq = g - geq
  });
  // g^eq_i = w_i [drho + 3 c.j + inv (4.5 (c.j)^2 - 1.5 |j|^2)], inv = 1 / (1 + drho)
  T S = T(0), jxb = T(0), jyb = T(0), jzb = T(0), invb = T(0);
  const T jsq15 = T(1.5) * (m.jx * m.jx + m.jy * m.jy + m.jz * m.jz);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const T si = T(weight<QN>(i)) * geqbar[i];
    S += si;
    if constexpr (nonzeros(i) == 0) {
      invb -= si * jsq15;
    } else {
      const T cj = cdot<i>(m.jx, m.jy, m.jz);
      invb += si * (T(4.5) * cj * cj - jsq15);
      const T coef = si * (T(3) + T(9) * m.inv * cj);
      if constexpr (cx(i) != 0) jxb += signed_term<cx(i)>(coef);
      if constexpr (cy(i) != 0) jyb += signed_term<cy(i)>(coef);
      if constexpr (cz(i) != 0) jzb += signed_term<cz(i)>(coef);
    }
  });
  jxb -= T(3) * m.inv * S * m.jx;
  jyb -= T(3) * m.inv * S * m.jy;
  jzb -= T(3) * m.inv * S * m.jz;
  const T drhob = S - m.inv * m.inv * invb;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    T v = nu[i] + fbar[i] + drhob;
    if constexpr (cx(i) != 0) v += signed_term<cx(i)>(jxb);
    if constexpr (cy(i) != 0) v += signed_term<cy(i)>(jyb);
    if constexpr (cz(i) != 0) v += signed_term<cz(i)>(jzb);
    lam_dst.store(i, c.cell, v);
  });
}

// dJ/du0(x) = sum_i lambda_0,i w_i [3 c_i + 9 (c_i.u0) c_i - 3 u0]; projected on the
// 24 basis products with factor amp * u0 / 8 (before the projection matrix).
// A block takes `per` groups of 256 nodes. Its sums over the nodes factor per
// axis, sum_x a_i(x) sum_(y,z) a_j(y) a_k(z) ubar(x, y, z): groups that start at the
// same place of a row give a thread the same x, so it adds the 12 inner sums of
// its nodes and only then multiplies by its a_i(x); one reduction per block
// follows (node by node, with 24 wave reductions and 11 sines each, 2 x 128^3 in
// float took 435 us; this takes 112, of which the reads at the card's rate are
// 75).
template <int QN, typename T>
__global__ void __launch_bounds__(256) init_adjoint_kernel(const T* __restrict__ lam, const DevSample* __restrict__ samples, const Seg* __restrict__ segs,
                                                           int nseg, int per, const double* __restrict__ ycoef, double* __restrict__ partials) {
  __shared__ double2 sc[kMaxN];
  __shared__ double sh[4][24];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Seg sg = segs[find_segment(segs, nseg, int(blockIdx.x) * per)];
  const int first = int(blockIdx.x) * per - sg.first_block, last = first + per;
  const DevSample& sp = samples[sg.sample];
  const int l = sp.log2n, n = 1 << l, msk = n - 1;
  make_axis_table(sc, n);
  __syncthreads();
  const double* yc = ycoef + size_t(sg.sample) * 24;
  const T* lb = lam + sp.offset;
  double acc[24];
#pragma unroll
  for (int p = 0; p < 24; ++p) acc[p] = 0.0;
  const int phases = n > 256 ? n / 256 : 1;  // groups per row
  for (int phase = 0; phase < phases; ++phase) {
    double in[3][4];
#pragma unroll
    for (int q = 0; q < 12; ++q) in[q >> 2][q & 3] = 0.0;
    const int b0 = first + ((phase - first) & (phases - 1));
    const int x = int(uint32_t(b0) * 256u + threadIdx.x) & msk;
    const double2 x1 = sc[x], x2 = sc[(2 * x) & msk];
    for (int b = b0; b < last; b += phases) {
      const uint32_t cell = uint32_t(b) * 256u + threadIdx.x;
      T g[Q];  // all loads in flight before the first is used
      for_vel<QN>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        g[i] = ld(lb + size_t(plane_of<QN>(i)) * sp.pstride, cell);
      });
      __builtin_amdgcn_sched_barrier(0);
      const int y = int(cell >> l) & msk, z = int(cell >> (2 * l));
      const double2 y2 = sc[(2 * y) & msk], z2 = sc[(2 * z) & msk];
      double u[3];
      initial_velocity(x1, x2, sc[y], y2, sc[z], z2, sp.u0, sp.amp, yc, u);
      // ub = sum_i li (3 c_i + 9 (c_i.u) c_i - 3 u), li = w_i lambda_i
      double sum = 0.0, l1[3] = {0.0, 0.0, 0.0}, l2[3] = {0.0, 0.0, 0.0};
      for_vel<QN>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const double li = double(g[i]) * weight<QN>(i);
        sum += li;
        if constexpr (nonzeros(i) > 0) {
          const double lcu = li * cdot<i>(u[0], u[1], u[2]);
          if constexpr (cx(i) != 0) { l1[0] += cx(i) * li; l2[0] += cx(i) * lcu; }
          if constexpr (cy(i) != 0) { l1[1] += cy(i) * li; l2[1] += cy(i) * lcu; }
          if constexpr (cz(i) != 0) { l1[2] += cz(i) * li; l2[2] += cz(i) * lcu; }
        }
      });
      const double jk[4] = {y2.x * z2.x, y2.x * z2.y, y2.y * z2.x, y2.y * z2.y};
#pragma unroll
      for (int al = 0; al < 3; ++al) {
        const double ub = 3.0 * l1[al] + 9.0 * l2[al] - 3.0 * u[al] * sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) in[al][q] += ub * jk[q];
      }
    }
#pragma unroll
    for (int al = 0; al < 3; ++al)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc[8 * al + q] += x2.x * in[al][q];
        acc[8 * al + 4 + q] += x2.y * in[al][q];
      }
  }
  const double scale = sp.amp * sp.u0 * 0.125;
#pragma unroll
  for (int p = 0; p < 24; ++p) {
    const double v = wave_sum(acc[p]);
    if (lane == 0) sh[wave][p] = scale * v;
  }
  __syncthreads();
  if (threadIdx.x < 24) {
    const int p = threadIdx.x;
    partials[size_t(sg.first_block + first) * 24 + p] = ((sh[0][p] + sh[1][p]) + sh[2][p]) + sh[3][p];
  }
}

// The rows of a sample's blocks (one in `per`), added by 40 threads per
// parameter in fixed order (one parameter after the other, over the partials of
// every 256 nodes: 184 us at 2 x 128^3, this 8).
constexpr int kInitParts = 40;

__global__ void __launch_bounds__(24 * kInitParts) init_adjoint_finalize_kernel(const double* partials,
                                                                                const Seg* segs, int per,
                                                                                const DevSample* samples,
                                                                                const double* pmat, double* dJdY) {
  const Seg sg = segs[blockIdx.x];
  __shared__ double red[kInitParts][24];
  __shared__ double dprime[24];
  const int p = threadIdx.x % 24, part = threadIdx.x / 24;
  {
    double acc = 0.0;
    const int rows = (sg.nblocks + per - 1) / per;
#pragma unroll 4
    for (int k = part; k < rows; k += kInitParts)
      acc += partials[(size_t(sg.first_block) + size_t(k) * per) * 24 + p];
    red[part][p] = acc;
  }
  __syncthreads();
  if (threadIdx.x < 24) {
    double acc = 0.0;
    for (int k = 0; k < kInitParts; ++k) acc += red[k][threadIdx.x];
    dprime[threadIdx.x] = acc;
  }
  __syncthreads();
  if (threadIdx.x < 24) {
    const int q = threadIdx.x;
    double v = dprime[q];
    if (samples[sg.sample].project) {
      // Y' = P Y, so dJ/dY = P^T dJ/dY'
      v = 0.0;
      for (int r = 0; r < 24; ++r) v += pmat[r * 24 + q] * dprime[r];
    }
    dJdY[size_t(sg.sample) * 24 + q] = v;
  }
}

__global__ void extract_kernel(const double* records, int m, int field, double* out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < m) out[s] = records[size_t(s) * kRecord + field];
}

// Energy per unit volume of sample s at record k, in lattice units: the
// kinetic energy of a record of the step kernel (field 4, the mean of |u|^2/2
// over the nodes), or the shell spectrum of eq. (energySpecDisc) summed over
// kappa = 0..n/2. LANES threads share one sample: each takes every LANES-th
// term and they add up in a fixed tree, after which all of them hold the sum.
struct RecordEnergy {
  static constexpr int LANES = 1;
  const double* rec;
  int m;
  __device__ double operator()(int k, int s, int) const { return rec[(size_t(k) * m + s) * kRecord + 4]; }
};
struct SpectrumEnergy {
  static constexpr int LANES = 16;
  const double* ek;
  int count, len;
  __device__ double operator()(int k, int s, int lane) const {
    const double* e = ek + (size_t(k) * count + s) * len;
    double sum = 0.0;
    for (int j = lane; j < len; j += LANES) sum += e[j];
#pragma unroll
    for (int o = LANES / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    return sum;
  }
};

// Dissipation rate per sample and record, d = -dE/dt in physical units (E /
// u0^2 against t = steps * (2 pi / n) * u0): centred differences inside the
// series, one-sided at its ends. Block (sample group, record); the sums of a
// spectrum's row run across LANES threads, so a wave reads whole lines of it.
// Latency of one load chain is all there is to it: one thread per record took
// 3570 us for the spectra of 1000 samples at 61 times and 394 us for their
// records; this takes 9 and 5, and 4 for the mean.
template <class Energy>
__global__ void __launch_bounds__(256) dissipation_kernel(Energy energy, const DissSample* smp, int m, int nrec,
                                                          int64_t first_tick, int record_every, double* diss) {
  constexpr int LANES = Energy::LANES, PER_BLOCK = 256 / LANES;
  const int s = blockIdx.x * PER_BLOCK + threadIdx.x / LANES, lane = threadIdx.x % LANES;
  if (s >= m) return;  // all lanes of a sample together
  const DissSample d = smp[s];
  for (int k = blockIdx.y; k < nrec; k += gridDim.y) {
    const int k0 = k > 0 ? k - 1 : 0, k1 = k + 1 < nrec ? k + 1 : nrec - 1;
    const double e0 = energy(k0, s, lane) * d.inv_u0sq;
    const double e1 = energy(k1, s, lane) * d.inv_u0sq;
    const double t0 = double((first_tick + int64_t(k0) * record_every) / d.stride) * d.dt;
    const double t1 = double((first_tick + int64_t(k1) * record_every) / d.stride) * d.dt;
    if (lane == 0) diss[size_t(k) * m + s] = -(e1 - e0) / (t1 - t0);
  }
}

// eta = (eps^3 / mean_s d)^(1/4), one block per record.
__global__ void __launch_bounds__(256) kolmogorov_kernel(const double* diss, int m, double eps, double* eta) {
  __shared__ double red[256];
  const double* d = diss + size_t(blockIdx.x) * m;
  double acc = 0.0;
  for (int s = threadIdx.x; s < m; s += 256) acc += d[s];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) eta[blockIdx.x] = sqrt(sqrt(eps * eps * eps / (red[0] / m)));
}

template <class Energy>
hipError_t launch_dissipation_of(Energy energy, const DissSample* smp, int m, int nrec, int64_t first_tick,
                                 int record_every, double eps, double* diss, double* eta, hipStream_t s) {
  constexpr int PER_BLOCK = 256 / Energy::LANES;
  const dim3 grid(unsigned((m + PER_BLOCK - 1) / PER_BLOCK), unsigned(nrec < 65535 ? nrec : 65535));
  hipLaunchKernelGGL(dissipation_kernel<Energy>, grid, dim3(256), 0, s, energy, smp, m, nrec, first_tick, record_every,
                     diss);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !eta) return e;
  hipLaunchKernelGGL(kolmogorov_kernel, dim3(unsigned(nrec)), dim3(256), 0, s, diss, m, eps, eta);
  return hipGetLastError();
}

// One 16-byte element per thread with non-temporal loads and stores (the
// fastest plain copy measured on gfx950: 6.5-6.6 TB/s on 4 GiB, against
// 6.1-6.2 TB/s with ordinary accesses and 5.1-5.3 TB/s with grid-stride
// loops).
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(256) stream_copy_kernel(const f32x4* __restrict__ src, f32x4* __restrict__ dst,
                                                          size_t n4) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < n4) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// f(lattice, value of the storage type) for a run-time lattice and precision
template <typename F>
hipError_t dispatch(int q, int precision, F&& f) {
  using Q27 = std::integral_constant<int, 27>;
  using Q19 = std::integral_constant<int, 19>;
  if (q == 27) return precision == 0 ? f(Q27{}, double{}) : f(Q27{}, float{});
  if (q == 19) return precision == 0 ? f(Q19{}, double{}) : f(Q19{}, float{});
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_step(int q, int precision, StepKind kind, const StepLaunch& L, hipStream_t s) {
  if (q == 27) return precision == 0 ? launch_step_d3q27_f64(kind, L, s) : launch_step_d3q27_f32(kind, L, s);
  if (q == 19) return precision == 0 ? launch_step_d3q19_f64(kind, L, s) : launch_step_d3q19_f32(kind, L, s);
  return hipErrorInvalidValue;
}

hipError_t launch_step2(int q, int precision, const Step2Launch& L, hipStream_t s) {
  if (q == 27) return precision == 0 ? launch_step2_d3q27_f64(L, s) : launch_step2_d3q27_f32(L, s);
  if (q == 19) return precision == 0 ? launch_step2_d3q19_f64(L, s) : launch_step2_d3q19_f32(L, s);
  return hipErrorInvalidValue;
}

hipError_t launch_record_finalize(double* partials, const Seg* segs, int32_t nseg, int32_t total_blocks,
                                  int32_t most_blocks, const DevSample* samples, double* out, hipStream_t s) {
  if (most_blocks > kRecordChunk) {
    const dim3 grid(unsigned((total_blocks + kRecordChunk - 1) / kRecordChunk));
    hipLaunchKernelGGL(record_chunk_kernel, grid, dim3(256), 0, s, partials, segs, nseg, total_blocks);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(record_finalize_kernel, dim3(nseg), dim3(256), 0, s, partials, segs, samples, out);
  return hipGetLastError();
}

namespace {
// Groups of 256 nodes per block of the kernels of the initial data: enough blocks
// to fill the card first, then up to 16 groups, which share a block's table of
// sines and its reduction; a power of two that divides every sample's groups, so
// that a block's groups are of one sample.
int groups_per_block(int32_t total_blocks, int32_t least_blocks) {
  int per = 1;
  while (2 * per <= std::min(16, std::min(least_blocks, total_blocks / 2048))) per *= 2;
  return per;
}
}  // namespace

hipError_t launch_init(int q, int precision, void* pop, const DevSample* samples, const Seg* segs, int32_t nseg,
                       int32_t total_blocks, int32_t least_blocks, const double* ycoef, hipStream_t s) {
  const int per = groups_per_block(total_blocks, least_blocks);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((init_kernel<decltype(qc)::value, T>), dim3(total_blocks / per), dim3(256), 0, s,
                       static_cast<T*>(pop), samples, segs, nseg, per, ycoef);
    return hipGetLastError();
  });
}

hipError_t launch_moments(int q, int precision, const void* pop, const DevSample* samples, int32_t sample, int32_t n,
                          int32_t parity, double* rho, double* u, hipStream_t s) {
  const unsigned blocks = unsigned((uint64_t(n) * n * n) / 256);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((moments_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(256), 0, s,
                       static_cast<const T*>(pop), samples, sample, parity, rho, u);
    return hipGetLastError();
  });
}

hipError_t launch_get_state(int q, int precision, const void* pop, const DevSample* samples, int32_t sample,
                            int32_t n, int32_t parity, double* f, hipStream_t s) {
  const unsigned blocks = unsigned((uint64_t(n) * n * n) / 256);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((get_state_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(256), 0, s,
                       static_cast<const T*>(pop), samples, sample, parity, f);
    return hipGetLastError();
  });
}

hipError_t launch_set_state(int q, int precision, void* pop, const DevSample* samples, int32_t sample, int32_t n,
                            int32_t parity, const double* f, hipStream_t s) {
  const unsigned blocks = unsigned((uint64_t(n) * n * n) / 256);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((set_state_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(256), 0, s,
                       static_cast<T*>(pop), samples, sample, parity, f);
    return hipGetLastError();
  });
}

hipError_t launch_gather_cells(int q, int precision, const void* pop, const DevSample* samples, int32_t sample,
                               int32_t parity, const int64_t* cells, int32_t count, double* f, hipStream_t s) {
  const unsigned blocks = unsigned((count + 63) / 64);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((gather_cells_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(64), 0, s,
                       static_cast<const T*>(pop), samples, sample, parity, cells, count, f);
    return hipGetLastError();
  });
}

hipError_t launch_poison(int q, int precision, void* pop, const DevSample* samples, int32_t sample, int32_t parity,
                         int64_t cell, int32_t k, hipStream_t s) {
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((poison_kernel<decltype(qc)::value, T>), dim3(1), dim3(1), 0, s, static_cast<T*>(pop),
                       samples, sample, parity, uint32_t(cell), k);
    return hipGetLastError();
  });
}

hipError_t launch_canonical_copy(int q, int precision, const void* pop, void* dst, const DevSample* samples,
                                 const Seg* segs, int32_t nseg, int32_t total_blocks, hipStream_t s) {
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((canonical_copy_kernel<decltype(qc)::value, T>), dim3(total_blocks), dim3(256), 0, s,
                       static_cast<const T*>(pop), static_cast<T*>(dst), samples, segs, nseg);
    return hipGetLastError();
  });
}

hipError_t launch_put_adjoint(int q, int precision, void* dst, const DevSample* samples, int32_t sample, int32_t n,
                              const double* lam, hipStream_t s) {
  const unsigned blocks = unsigned((uint64_t(n) * n * n) / 256);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((put_adjoint_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(256), 0, s,
                       static_cast<T*>(dst), samples, sample, lam);
    return hipGetLastError();
  });
}

hipError_t launch_get_adjoint(int q, int precision, const void* src, const DevSample* samples, int32_t sample,
                              int32_t n, double* lam, hipStream_t s) {
  const unsigned blocks = unsigned((uint64_t(n) * n * n) / 256);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((get_adjoint_kernel<decltype(qc)::value, T>), dim3(blocks), dim3(256), 0, s,
                       static_cast<const T*>(src), samples, sample, lam);
    return hipGetLastError();
  });
}

hipError_t launch_adjoint_seed(int q, int precision, const void* pop, void* lam, const DevSample* samples,
                               const Seg* segs, int32_t nseg, int32_t total_blocks, double inv_m, hipStream_t s) {
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((adjoint_seed_kernel<decltype(qc)::value, T>), dim3(total_blocks), dim3(256), 0, s,
                       static_cast<const T*>(pop), static_cast<T*>(lam), samples, segs, nseg, inv_m);
    return hipGetLastError();
  });
}

namespace {
template <int QN, typename T, int BLOCK, bool ARGS>
hipError_t launch_adjoint_step_t(const T* a, const T* b, T* o, const DevSample* samples, const Seg* segs,
                                 const UniformSegs& uniform, int32_t nseg, int32_t total_blocks, int32_t buffer_ok,
                                 int32_t exact_gamma, hipStream_t s) {
  const dim3 grid(total_blocks), blk(BLOCK);
  if (exact_gamma) {
    // FP64 only (the host refuses FP32): see mclbm_backward
    if constexpr (!std::is_same<T, double>::value) return hipErrorInvalidValue;
    else if (buffer_ok)
      hipLaunchKernelGGL((adjoint_step_kernel<QN, T, BLOCK, true, true, ARGS>), grid, blk, 0, s, a, b, o, samples,
                         segs, uniform, nseg);
    else
      hipLaunchKernelGGL((adjoint_step_kernel<QN, T, BLOCK, false, true, ARGS>), grid, blk, 0, s, a, b, o, samples,
                         segs, uniform, nseg);
  } else if (buffer_ok) {
    hipLaunchKernelGGL((adjoint_step_kernel<QN, T, BLOCK, true, false, ARGS>), grid, blk, 0, s, a, b, o, samples, segs,
                       uniform, nseg);
  } else {
    hipLaunchKernelGGL((adjoint_step_kernel<QN, T, BLOCK, false, false, ARGS>), grid, blk, 0, s, a, b, o, samples,
                       segs, uniform, nseg);
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_adjoint_step(int q, int precision, const void* state, const void* lam_in, void* lam_out,
                               const DevSample* samples, const Seg* segs, const UniformSegs& uniform, int32_t nseg,
                               int32_t total_blocks, int32_t block, int32_t buffer_ok, int32_t exact_gamma,
                               hipStream_t s) {
  return dispatch(q, precision, [&](auto qc, auto tc) {
    constexpr int QN = decltype(qc)::value;
    using T = decltype(tc);
    const T* a = static_cast<const T*>(state);
    const T* b = static_cast<const T*>(lam_in);
    T* o = static_cast<T*>(lam_out);
    if (block == kSmallBlock && uniform.on)
      return launch_adjoint_step_t<QN, T, kSmallBlock, true>(a, b, o, samples, segs, uniform, nseg, total_blocks,
                                                             buffer_ok, exact_gamma, s);
    if (block == kSmallBlock)
      return launch_adjoint_step_t<QN, T, kSmallBlock, false>(a, b, o, samples, segs, uniform, nseg, total_blocks,
                                                              buffer_ok, exact_gamma, s);
    if (block == 256)
      return launch_adjoint_step_t<QN, T, 256, false>(a, b, o, samples, segs, uniform, nseg, total_blocks, buffer_ok,
                                                      exact_gamma, s);
    return hipErrorInvalidValue;
  });
}

hipError_t launch_init_adjoint(int q, int precision, const void* lam, const DevSample* samples, const Seg* segs,
                               int32_t nseg, int32_t total_blocks, int32_t least_blocks, const double* ycoef,
                               double* partials, hipStream_t s) {
  const int per = groups_per_block(total_blocks, least_blocks);
  return dispatch(q, precision, [&](auto qc, auto tc) {
    using T = decltype(tc);
    hipLaunchKernelGGL((init_adjoint_kernel<decltype(qc)::value, T>), dim3(total_blocks / per), dim3(256), 0, s,
                       static_cast<const T*>(lam), samples, segs, nseg, per, ycoef, partials);
    return hipGetLastError();
  });
}

hipError_t launch_init_adjoint_finalize(const double* partials, const Seg* segs, int32_t nseg, int32_t total_blocks,
                                        int32_t least_blocks, const DevSample* samples, const double* pmat, double* dJdY,
                                        hipStream_t s) {
  hipLaunchKernelGGL(init_adjoint_finalize_kernel, dim3(nseg), dim3(24 * kInitParts), 0, s, partials, segs,
                     groups_per_block(total_blocks, least_blocks), samples, pmat, dJdY);
  return hipGetLastError();
}

hipError_t launch_extract(const double* records, int32_t m, int32_t field, double* out, hipStream_t s) {
  hipLaunchKernelGGL(extract_kernel, dim3((m + 255) / 256), dim3(256), 0, s, records, m, field, out);
  return hipGetLastError();
}

hipError_t launch_dissipation(const double* records, const DissSample* smp, int32_t m, int32_t nrec,
                              int64_t first_tick, int32_t record_every, double eps, double* diss, double* eta,
                              hipStream_t s) {
  return launch_dissipation_of(RecordEnergy{records, m}, smp, m, nrec, first_tick, record_every, eps, diss, eta, s);
}

hipError_t launch_dissipation_spectra(const double* ek, int32_t n, const DissSample* smp, int32_t count,
                                      int32_t nrec, int64_t first_tick, int32_t record_every, double eps,
                                      double* diss, double* eta, hipStream_t s) {
  return launch_dissipation_of(SpectrumEnergy{ek, count, n / 2 + 1}, smp, count, nrec, first_tick, record_every, eps,
                               diss, eta, s);
}

hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n4 = bytes / 16;
  const size_t blocks = (n4 + 255) / 256;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(stream_copy_kernel, dim3(unsigned(blocks)), dim3(256), 0, s, static_cast<const f32x4*>(src),
                     static_cast<f32x4*>(dst), n4);
  return hipGetLastError();
}

}  // namespace mclbm
