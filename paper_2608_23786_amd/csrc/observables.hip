// FP64 observables of one sample's velocity field (gfx950):
//   * the power spectral density Psi(k) = sum_a |F(u_a)(k)|^2 of the
//     three velocity components (unnormalised forward transform);
//   * the shell energy spectrum E(kappa) = 4 pi / |S_kappa| sum_{S_kappa}
//     |k|^2 / 2 * Psi(k) / N^6 (eqs. (dftCoeff), (energySpecDisc));
//   * the autocorrelation R_h = N^-6 F^-1(Psi)_h with an unnormalised inverse
//     and the structure function S2(r) = 1/|C_r| sum_{h in C_r} 2 (R_0 - R_h)
//     (Lemma (structureFunctionSpectral), eq. (SF_single_spec2));
//   * point values of all samples at the q^3 nodes common to every
//     resolution, and the 1-point Wasserstein distance between two such
//     ensembles by sorting (Algorithm 2, eq. (wassersteinPermutations)).
//
// The velocity is real, so its transform is stored for kx = 0..N/2 only
// (the rest follows by conjugate symmetry), fields [z][y][kx]. A shell C_r
// is closed under a change of sign of any lag component, so S2 needs R only
// summed over the lags that fold to f = (|hx|, |hy|, |hz|), f_a = 0..N/2:
// X(f) = sum_{h -> f} R_h = N^-6 sum_k Psi(k) prod_a mu(f_a) cos(2 pi k_a f_a / N)
// with mu(0) = mu(N/2) = 1 and mu = 2 otherwise (the lags behind f_a). The
// inverse transforms therefore run as cosine sums that keep f_a = 0..N/2,
// which shrinks each axis' output to about half. The pipeline is five
// passes over HBM:
//   1. x: velocities from the populations (either AA parity), or from the
//      velocity a record tick captured, and the forward transform along x
//      of the three components, per row in LDS (two real components share
//      one complex transform);
//   2. y: forward transforms along y of the three fields;
//   3. per z-line: the forward transforms along z of the three fields,
//      Psi, its shell sums for the spectrum, its total (R_0), and the
//      folded inverse along z, G[ky][kx][f_z] (real);
//   4. y: the folded inverse along y of G, H[f_y][kx][f_z] (two real lines
//      per complex transform);
//   5. per row (f_y, f_z): the folded inverse along x (H is even in kx once
//      y and z are folded, so its transform is real; two rows per complex
//      transform), X(f), and the shell sums for S2.
// Transforms of whole lines in two factors (three at 512) held in registers,
// with exchanges through LDS between them, twiddles by sincospi;
// each launch hands every XCD a contiguous run of blocks, so that blocks sharing cache lines share an
// L2. Shells hold the integer vectors (minimum image, components in
// {-N/2+1, ..., N/2}) whose length rounds to the shell index. Every shell sum
// is taken per line (the line folded by the magnitude of its own
// coordinate, the lengths of a shell forming an interval of it), then over
// the lines of a block, then over blocks, each in a fixed order: results do
// not depend on scheduling. The number of vectors in a shell depends on N
// only and is counted exactly in the last stage. A half-spectrum mode
// 0 < kx < N/2 stands for itself and its conjugate partner at -k, which has
// the same length: weight 2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "lbm_device.h"

namespace mclbm {
namespace {

// Elements of a line that a thread holds in the transforms, and the threads per line
constexpr int fft_elems(int n) { return n >= 512 ? 8 : (n >= 128 ? 16 : (n >= 32 ? 8 : 4)); }
constexpr int fft_threads(int n) { return n / fft_elems(n); }

// Lines per block of the transforms along y: 128 threads (256 from 256 on; at
// 256 16 lines take 284 us of two samples, 8 take 299), and 128 bytes or more of
// consecutive lines per access; it divides n, so it divides the n (n/2 + 1)
// lines of a field.
constexpr int y_lines(int n) { return n >= 512 ? 4 : (n == 32 ? 32 : (n >= 16 ? 16 : 8)); }

// Lines per block of the z pass: its phases (loads, exchanges, shell sums) are
// kept apart by barriers, so more and smaller blocks overlap better (us of two
// 256^3 with 4 / 8 / 16 lines 276 / 277 / 300, of twelve 128^3 198 / 189 / 223).
constexpr int z_lines(int n) { return n == 128 || n == 256 ? 8 : y_lines(n); }

// Threads per block of the passes that end in shell sums. The transforms of a block
// take 16 to 128 threads, too few for its shell sums, which are as long a chain of
// instructions: the block has 256, all of which take (line, shell) pairs, in the z
// pass up to 64 (from 128 on the pairs' LDS would cost it blocks) and in the last
// pass up to 256 (us with the transforms' threads alone / with 256: z pass of four
// samples of 32^3 19.7 / 9.0, of two of 64^3 16.2 / 10.2; last pass 8.8 / 5.2, 9.4 /
// 6.5, of twelve 128^3 38.0 / 30.5, of two 256^3 55.3 / 38.9).
constexpr int sum_threads(int n, int transform_threads) { return n <= 64 ? 256 : transform_threads; }
constexpr int last_threads(int n, int transform_threads) { return n <= 256 ? 256 : transform_threads; }

// Pairs of real lines per block of the folded inverse passes along y and x
// (one complex transform per pair)
constexpr int cos_pairs(int n) { return n >= 512 ? 4 : (n >= 128 ? 8 : 16); }

// Lines of the folded passes: (N/2 + 1)^2 per value of the other index
constexpr size_t folded_lines(int n) { return size_t(n / 2 + 1) * (n / 2 + 1); }

// rows of the spectrum's and the structure function's shell tables: one
// per block of the pass that writes them
constexpr size_t spectrum_bin_rows(int n) { return size_t(n) * (n / 2 + 1) / z_lines(n); }
constexpr size_t sf_bin_rows(int n) { return (folded_lines(n) + 2 * cos_pairs(n) - 1) / (2 * cos_pairs(n)); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

constexpr int log2_of(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Transforms of whole lines, in registers but for the exchanges between their
// factors. A line of N elements belongs to fft_threads(N) threads; thread t
// holds elements t + m N/E, m < E = fft_elems(N), before and after (the same
// set, so Psi can stay in registers between a forward and an inverse
// transform). N = A B with A = E: thread t transforms its A elements
// (n = t + B m to k1), multiplies by W_N^{t k1}, and after one exchange through
// LDS transforms the B elements of each k1 = t + B j to k = k1 + A k2. 512 is
// 8 x 8 x 8 with two exchanges. Against radix-4 steps of a thread's quartet,
// with a pass over LDS after each, a 256-element line goes through LDS once
// instead of three times: us of two samples of 256^3,
// y 318 -> 284, z 327 -> 275; at 512 6660 -> 6020 for one sample from its
// populations, 4650 -> 3830 from its velocity; to 128 within 2 %.

// LDS slots of a line: rows of B + 1 for the exchange (or N in natural
// order), an odd number of 16-byte slots, so that lanes that touch the same
// element of consecutive lines fall on different banks, as do those of one line.
template <int N>
constexpr int lds_line() {
  return N >= 512 ? 585 : ((fft_elems(N) * (N / fft_elems(N) + 1)) | 1);
}

// The same in 8-byte slots, for exchanges of one part of the values at a time
// (half the LDS, which doubles the blocks of a CU) by LINES lines whose lanes
// are neighbours: the lines of 32 lanes are 32 / LINES banks of 8 bytes apart,
// and the lanes of one line take the banks between.
template <int N, int LINES>
constexpr int lds_half_line() {
  const int least = N >= 512 ? 584 : fft_elems(N) * (N / fft_elems(N) + 1), step = LINES >= 32 ? 1 : 32 / LINES;
  return (least + 31 - step) / 32 * 32 + step;
}

// e^{-2 pi i k / N}, k < N; the first quadrant computed, the others its rotations
template <int N>
__device__ __forceinline__ void make_twiddles(double2* tw) {
  for (int k = threadIdx.x; k < N / 4; k += blockDim.x) {
    double s, c;
    sincospi(2.0 * k / N, &s, &c);
    tw[k] = make_double2(c, -s);
    tw[k + N / 4] = make_double2(-s, -c);
    tw[k + N / 2] = make_double2(-c, s);
    tw[k + 3 * N / 4] = make_double2(s, c);
  }
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// a times w (SIGN -1) or its conjugate (SIGN +1)
template <int SIGN>
__device__ __forceinline__ double2 cmul_dir(double2 a, double2 w) {
  return cmul(a, make_double2(w.x, SIGN < 0 ? w.y : -w.y));
}

// a times e^{SIGN i pi / 2}
template <int SIGN>
__device__ __forceinline__ double2 quarter_turn(double2 a) {
  return SIGN < 0 ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}

// Transforms of R elements in registers, natural order in and out
template <int R, int SIGN>
__device__ __forceinline__ void dft(double2* x) {
  if constexpr (R == 2) {
    const double2 a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const double2 s0 = cadd(x[0], x[2]), d0 = csub(x[0], x[2]);
    const double2 s1 = cadd(x[1], x[3]), d1 = quarter_turn<SIGN>(csub(x[1], x[3]));
    x[0] = cadd(s0, s1);
    x[1] = cadd(d0, d1);
    x[2] = csub(s0, s1);
    x[3] = csub(d0, d1);
  } else if constexpr (R == 8) {
    constexpr double h = 0.70710678118654752440;
    double2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
    dft<4, SIGN>(e);
    dft<4, SIGN>(o);
    const double2 t1 = quarter_turn<SIGN>(o[1]), t3 = quarter_turn<SIGN>(o[3]);
    o[1] = make_double2(h * (o[1].x + t1.x), h * (o[1].y + t1.y));
    o[2] = quarter_turn<SIGN>(o[2]);
    o[3] = make_double2(h * (t3.x - o[3].x), h * (t3.y - o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = cadd(e[k], o[k]);
      x[k + 4] = csub(e[k], o[k]);
    }
  } else {
    static_assert(R == 16, "radix");
    constexpr double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
    // e^{-i pi j / 8} for the products j = 0, 1, 2, 3, 4, 6, 9 of two digits
    double2 y[4][4];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < 4; ++n1) y[n2][n1] = x[n2 + 4 * n1];
      dft<4, SIGN>(y[n2]);
    }
    const double2 w1 = make_double2(c1, -s1), w2 = make_double2(h, -h), w3 = make_double2(s1, -c1);
    y[1][1] = cmul_dir<SIGN>(y[1][1], w1);
    y[1][2] = cmul_dir<SIGN>(y[1][2], w2);
    y[1][3] = cmul_dir<SIGN>(y[1][3], w3);
    y[2][1] = cmul_dir<SIGN>(y[2][1], w2);
    y[2][2] = quarter_turn<SIGN>(y[2][2]);
    y[2][3] = quarter_turn<SIGN>(cmul_dir<SIGN>(y[2][3], w2));
    y[3][1] = cmul_dir<SIGN>(y[3][1], w3);
    y[3][2] = quarter_turn<SIGN>(cmul_dir<SIGN>(y[3][2], w2));
    y[3][3] = cmul_dir<SIGN>(y[3][3], make_double2(-c1, s1));
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      double2 z[4] = {y[0][k1], y[1][k1], y[2][k1], y[3][k1]};
      dft<4, SIGN>(z);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) x[k1 + 4 * k2] = z[k2];
    }
  }
}

// R values of a thread through LDS: x[k] to at(k), then from from(k). V double2
// moves them in one go, V double the real parts, then the imaginary parts.
template <int R, typename V, typename To, typename From>
__device__ __forceinline__ void exchange(double2 (&x)[R], V* ln, bool active, To&& to, From&& from) {
  if constexpr (std::is_same<V, double2>::value) {
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) ln[to(k)] = x[k];
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) x[k] = ln[from(k)];
    }
  } else {
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) ln[to(k)] = x[k].x;
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) x[k].x = ln[from(k)];
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) ln[to(k)] = x[k].y;
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int k = 0; k < R; ++k) x[k].y = ln[from(k)];
    }
  }
}

// The transform of the line that the calling thread shares (its LDS at ln), its
// elements in x; every thread of the block calls it, those without a line with
// active = false. The line's LDS must be free on entry, and is read until the
// next barrier after the return.
template <int N, int SIGN, typename V>
__device__ __forceinline__ void fft_line(double2 (&x)[fft_elems(N)], int t, V* ln, const double2* tw,
                                         bool active = true) {
  constexpr int E = fft_elems(N);
  if (active) {
    dft<E, SIGN>(x);
#pragma unroll
    for (int k1 = 1; k1 < E; ++k1) x[k1] = cmul_dir<SIGN>(x[k1], tw[k1 * t]);
  }
  if constexpr (N < 512) {
    constexpr int B = N / E, PER = E / B;
    exchange(x, ln, active, [&](int k1) { return k1 * (B + 1) + t; },
             [&](int k) { return (t + B * (k / B)) * (B + 1) + k % B; });
    if (active) {
      double2 y[E];
#pragma unroll
      for (int j = 0; j < PER; ++j) dft<B, SIGN>(x + j * B);
#pragma unroll
      for (int k = 0; k < E; ++k) y[k / B + PER * (k % B)] = x[k];
#pragma unroll
      for (int k = 0; k < E; ++k) x[k] = y[k];
    }
  } else {
    static_assert(N == 512 && E == 8, "three factors of 8");
    const int k1 = t & 7, hi = t >> 3;
    exchange(x, ln, active, [&](int k) { return k * 65 + t; }, [&](int m) { return k1 * 65 + hi + 8 * m; });
    if (active) {
      dft<8, SIGN>(x);
#pragma unroll
      for (int q = 1; q < 8; ++q) x[q] = cmul_dir<SIGN>(x[q], tw[8 * hi * q]);
    }
    __syncthreads();
    exchange(x, ln, active, [&](int q) { return k1 * 73 + q * 9 + hi; },
             [&](int m) { return k1 * 73 + hi * 9 + m; });
    if (active) dft<8, SIGN>(x);
  }
}

// A batch of samples shares one launch: blockIdx.z is the sample's place in
// the batch, and its work area starts wstride bytes after the previous one.
template <typename P>
__device__ __forceinline__ P* in_batch(P* p, size_t wstride) {
  using B = typename std::conditional<std::is_const<P>::value, const char, char>::type;
  return reinterpret_cast<P*>(reinterpret_cast<B*>(p) + size_t(blockIdx.z) * wstride);
}

// floor(sqrt(v)) for 0 <= v < 2^24, which holds for every value the shell
// ranges meet (n <= 1024): the hardware's square root is within 2^-12 of the
// true one there, so its floor is off by one at most, and one step back or
// forward corrects it.
__device__ __forceinline__ int isqrt_floor(int v) {
  if (v <= 0) return 0;
  int r = int(__builtin_amdgcn_sqrtf(float(v)));
  r -= r * r > v ? 1 : 0;
  r += (r + 1) * (r + 1) <= v ? 1 : 0;
  return r;
}

// The m in [0, half] with round(sqrt(s + m^2)) == r form the interval
// [a, b] (empty when a > b): m^2 in [ceil(((2r-1)^2 - 4s)/4),
// floor(((2r+1)^2 - 1 - 4s)/4)].
__device__ __forceinline__ void shell_range(int half, int s, int r, int& a, int& b) {
  a = 1;
  b = 0;
  const int lo2 = r == 0 ? 0 : (2 * r - 1) * (2 * r - 1);
  const int top = (2 * r + 1) * (2 * r + 1) - 1 - 4 * s;
  if (top < 0) return;
  const int m2max = top / 4;
  const int bot = lo2 - 4 * s;
  const int m2min = bot <= 0 ? 0 : (bot + 3) / 4;
  if (m2min > m2max) return;
  int lo = isqrt_floor(m2min);
  if (lo * lo < m2min) ++lo;
  int hi = isqrt_floor(m2max);
  if (hi > half) hi = half;
  a = lo;
  b = hi;
}

// Lattice vectors a folded index m stands for: m and -m, except m = 0 and
// m = half (the Nyquist value is present once).
__device__ __forceinline__ double fold_weight(int m, int half) { return (m == 0 || m == half) ? 1.0 : 2.0; }

// Lattice vectors standing behind the folded indices a..b
__device__ __forceinline__ double range_count(int half, int a, int b) {
  if (a > b) return 0.0;
  return 2.0 * (b - a + 1) - (a == 0 ? 1.0 : 0.0) - (b == half ? 1.0 : 0.0);
}

// x-rows per block of the forward transform along x: two nodes per thread,
// and an even number of rows (two rows share one transform of uz)
constexpr int fwd_rows(int n) { return n >= 256 ? 2 : 512 / n; }

// Pass 1: ROWS rows (z, y) per block. Velocities of the rows' nodes from the
// populations (the parity selects the AA slots; consecutive threads take
// consecutive nodes of a row, so every population plane is read in
// contiguous runs), or, with FROM_U, read from the velocity a record tick
// captured (u + voffset, three planes of N^3; pop and parity unused), and
// the forward transform along x of the three
// components, kx = 0..N/2 written to h[c][(z N + y) NH + kx]. The components
// are real, so two share one complex transform: ux + i uy of each row, and
// uz of a pair of rows, by way of LDS; the two
// spectra of a line are separated afterwards from Z(k) and Z(N - k):
// A(k) = (Z(k) + conj Z(N - k)) / 2, B(k) = (Z(k) - conj Z(N - k)) / 2i.
template <int QN, typename T, int N, bool FROM_U>
__global__ void __launch_bounds__(256) fwd_x_kernel(const T* pop, const double* u, const DevSample* samples,
                                                    int sample0, int parity, double2* h0, size_t wstride) {
  constexpr int ROWS = fwd_rows(N), PAIRS = ROWS / 2, LINES = ROWS + PAIRS;
  constexpr int NH = N / 2 + 1, E = fft_elems(N), TPL = fft_threads(N);
  constexpr int LS = lds_line<N>();
  static_assert(LINES * TPL <= 256, "one line element set per thread");
  __shared__ double2 sh[LINES * LS];
  __shared__ double2 tw[N];
  const DevSample& sp = samples[sample0 + blockIdx.z];
  double2* h = in_batch(h0, wstride);
  const size_t row0 = size_t(remap_block(blockIdx.x, gridDim.x, 1)) * ROWS;
  make_twiddles<N>(tw);
  double* shd = reinterpret_cast<double*>(sh);
  for (int e = threadIdx.x; e < ROWS * N; e += 256) {
    const int r = e / N, x = e % N;
    const uint32_t cell = uint32_t((row0 + r) * N + x);
    double ux, uy, uz;
    if constexpr (FROM_U) {
      constexpr size_t plane = size_t(N) * N * N;
      const double* ub = u + sp.voffset;
      ux = ub[cell];
      uy = ub[plane + cell];
      uz = ub[2 * plane + cell];
    } else {
      T g[Q];
      load_state<QN>(pop + sp.offset, sp.pstride, make_cell(cell, sp.log2n), parity & 1, g);
      node_velocity<QN>(g, ux, uy, uz);
    }
    sh[r * LS + x] = make_double2(ux, uy);
    shd[2 * ((ROWS + r / 2) * LS + x) + (r & 1)] = uz;
  }
  __syncthreads();
  const int t = threadIdx.x % TPL;
  const bool active = threadIdx.x < LINES * TPL;
  double2* ln = sh + (active ? threadIdx.x / TPL : 0) * LS;
  double2 x[E];
  if (active) {
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = ln[t + m * TPL];
  }
  __syncthreads();
  fft_line<N, -1>(x, t, ln, tw, active);
  __syncthreads();
  if (active) {
#pragma unroll
    for (int m = 0; m < E; ++m) ln[t + m * TPL] = x[m];
  }
  __syncthreads();
  const size_t field = size_t(N) * N * NH;
  for (int e = threadIdx.x; e < LINES * NH; e += 256) {
    const int l = e / NH, k = e % NH;
    const double2 z = sh[l * LS + k];
    const double2 zn = sh[l * LS + ((N - k) & (N - 1))];
    const double2 a = make_double2(0.5 * (z.x + zn.x), 0.5 * (z.y - zn.y));  // (Z(k) + conj Z(N-k)) / 2
    const double2 b = make_double2(0.5 * (z.y + zn.y), 0.5 * (zn.x - z.x));  // (Z(k) - conj Z(N-k)) / 2i
    if (l < ROWS) {
      h[(row0 + l) * NH + k] = a;
      h[field + (row0 + l) * NH + k] = b;
    } else {
      const int p = l - ROWS;
      h[2 * field + (row0 + 2 * p) * NH + k] = a;
      h[2 * field + (row0 + 2 * p + 1) * NH + k] = b;
    }
  }
}

// Pass 2: forward transform along y of the fields h + c * N N NH,
// c = blockIdx.y; LINES lines (z, kx) per block, consecutive kx (consecutive
// threads take consecutive lines, so their global accesses are contiguous).
template <int N, int LINES>
__global__ void __launch_bounds__(LINES * fft_threads(N)) fft_y_kernel(double2* h0, size_t wstride) {
  constexpr int NH = N / 2 + 1, LS = lds_line<N>(), E = fft_elems(N), TPL = fft_threads(N);
  __shared__ double2 sh[LINES * LS];
  __shared__ double2 tw[N];
  const int l = threadIdx.x % LINES, t = threadIdx.x / LINES;
  const int line = remap_block(blockIdx.x, gridDim.x, 1) * LINES + l, z = line / NH, kx = line % NH;
  double2* d = in_batch(h0, wstride) + size_t(blockIdx.y) * N * N * NH + (size_t(z) * N + t) * NH + kx;
  double2 x[E];
#pragma unroll
  for (int m = 0; m < E; ++m) x[m] = d[size_t(m * TPL) * NH];
  make_twiddles<N>(tw);
  __syncthreads();
  fft_line<N, -1>(x, t, sh + l * LS, tw);
#pragma unroll
  for (int m = 0; m < E; ++m) d[size_t(m * TPL) * NH] = x[m];
}

// Pass 3: LINES z-lines (y, kx) per block (consecutive threads on consecutive
// lines). The forward transform along z
// of each of the three fields (already transformed along x and y), one
// field at a time in LDS, with Psi, the sum of |.|^2 over the fields, kept in
// registers (a thread's elements are the same for every field, and the
// inverse transform takes the same). |k|^2 Psi then goes to
// the transform's LDS in natural order for the shell sums of |k|^2/2 Psi
// over the block's lines (each line folded by |kz| and weighted by its kx
// weight, the lines added in order) into sbins[block][kappa] and the sum of
// Psi into sbins[block][N/2 + 1] (rows of N/2 + 2 values); last, the folded
// inverse transform of Psi along z, G(f_z) = mu(f_z) Re F^-1(Psi)(f_z) for
// f_z = 0..N/2 (Psi is real, so that real part is even), written to
// g[(ky NH + kx)(N/2 + 1) + f_z]: the block's lines are consecutive (ky, kx),
// so it writes one contiguous run. One LDS area serves all three, which
// keeps a block at the transform's LDS.
template <int N, int LINES>
__global__ void __launch_bounds__(sum_threads(N, LINES * fft_threads(N))) z_psd_kernel(const double2* h0, double* g0, double* sbins0,
                                                                       size_t wstride) {
  constexpr int NH = N / 2 + 1, HALF = N / 2, LS = lds_half_line<N, LINES>(), E = fft_elems(N), TPL = fft_threads(N);
  constexpr int THREADS = sum_threads(N, LINES * TPL);
  constexpr bool PAIRWISE = THREADS > LINES * TPL;  // a thread per (line, shell), beyond those of the transforms
  // Psi of every line (an odd number of doubles apart) lives in the transform's LDS
  // between the forward and the inverse transforms, then the folded lines
  constexpr int PS = N + 1, HP = HALF + 1;
  constexpr int USED = PS + (PAIRWISE ? HP : 0), SH = LS > USED ? LS : USED;
  __shared__ double sh[LINES * SH];
  __shared__ double tot[(THREADS + 63) / 64], last[LINES];
  __shared__ double2 tw[N];
  double* const psi = sh;
  const size_t field = size_t(N) * N * NH;
  double* g = in_batch(g0, wstride);
  double* sbins = in_batch(sbins0, wstride);
  const int line0 = remap_block(blockIdx.x, gridDim.x, 1) * LINES;
  const int l = threadIdx.x % LINES, t = threadIdx.x / LINES;
  const bool active = !PAIRWISE || t < TPL;
  double* const ln = sh + l * LS;
  const double2* d = in_batch(h0, wstride) + size_t(t) * field / N + line0 + l;   // lines are (y, kx), kx fastest
  make_twiddles<N>(tw);
  double ps[E];
#pragma unroll
  for (int m = 0; m < E; ++m) ps[m] = 0.0;
  for (int c = 0; c < 3; ++c) {
    double2 x[E];
    if (active) {
#pragma unroll
      for (int m = 0; m < E; ++m) x[m] = d[m * (TPL * field / N)];
    }
    d += field;
    __syncthreads();  // the twiddles are there; the field before is read
    fft_line<N, -1>(x, t, ln, tw, active);
    if (active) {
#pragma unroll
      for (int m = 0; m < E; ++m) ps[m] += x[m].x * x[m].x + x[m].y * x[m].y;
    }
  }
  __syncthreads();  // Psi overwrites sh
  // Psi folded by |kz| with the weight |k|^2 of its mode, in two halves that are
  // added when read: element m and element N - m (zero behind m = 0; the
  // Nyquist value is its own partner, a half in either)
  const int myline = line0 + l, myx = myline % NH, myy = myline / NH;
  const double s_xy = double(myx) * myx + double(myy <= HALF ? myy : N - myy) * (myy <= HALF ? myy : N - myy);
  if (active) {
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int k = t + m * TPL, kf = k <= HALF ? k : N - k;
      const double w = fma(double(kf), double(kf), s_xy) * ps[m];
      psi[l * PS + k] = k == HALF ? 0.5 * w : w;
    }
  }
  if (t == 0) psi[l * PS + N] = 0.0;
  double total = 0.0;
#pragma unroll
  for (int m = 0; m < E; ++m) total += ps[m];
  total *= fold_weight(myx, HALF);
  constexpr int LANES = THREADS >= 64 ? 64 : THREADS;
#pragma unroll
  for (int o = LANES / 2; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
  if (threadIdx.x % LANES == 0) tot[threadIdx.x / LANES] = total;
  __syncthreads();
  // the shell sums, the block's lines added in order
  const size_t blk = size_t(line0 / LINES);
  // of one line, times half of the mode's weight in |k|^2 / 2
  auto line_sum = [&](int k, int r) {
    const int line = line0 + k, y = line / NH, kx = line % NH;
    const int ky = y <= HALF ? y : y - N;
    const double* pl = psi + k * PS;
    int a, b;
    shell_range(HALF, kx * kx + ky * ky, r, a, b);
    double part = 0.0;
    for (int m = a; m <= b; ++m) part += pl[m] + pl[N - m];
    return (kx == 0 || kx == HALF ? 0.5 : 1.0) * part;
  };
  if constexpr (PAIRWISE) {
    double* const part = sh + LINES * PS;  // [LINES][HP]
    for (int e = threadIdx.x; e < LINES * HP; e += THREADS) part[e] = line_sum(e / HP, e % HP);
    __syncthreads();
    for (int r = threadIdx.x; r <= HALF; r += THREADS) {
      double sum = 0.0;
      for (int k = 0; k < LINES; ++k) sum += part[k * HP + r];
      sbins[blk * (HALF + 2) + r] = sum;
    }
  } else {
    // a shell per thread; the last shell, one too many for the threads at 128 and
    // 256, takes a thread per line
    for (int e = threadIdx.x; e < HALF + LINES; e += THREADS) {
      const int r = e < HALF ? e : HALF, k0 = e < HALF ? 0 : e - HALF, k1 = e < HALF ? LINES : k0 + 1;
      double sum = 0.0;
      for (int k = k0; k < k1; ++k) sum += line_sum(k, r);
      if (e < HALF)
        sbins[blk * (HALF + 2) + r] = sum;
      else
        last[k0] = sum;
    }
  }
  if (threadIdx.x == 0) {
    double sum = 0.0;
    for (int k = 0; k < (THREADS + 63) / 64; ++k) sum += tot[k];
    sbins[blk * (HALF + 2) + HALF + 1] = sum;
  }
  __syncthreads();  // Psi and the sums are read; the inverse overwrites sh
  if (!PAIRWISE && threadIdx.x == 0) {
    double sum = 0.0;
    for (int k = 0; k < LINES; ++k) sum += last[k];
    sbins[blk * (HALF + 2) + HALF] = sum;
  }
  double2 x[E];
#pragma unroll
  for (int m = 0; m < E; ++m) x[m] = make_double2(ps[m], 0.0);
  fft_line<N, +1>(x, t, ln, tw, active);
  __syncthreads();  // the transform's reads are done; sh stages the output
  // outputs 0..N/2; mu is 2 except at 0 and N/2
  double* const stage = sh;
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int f = t + m * TPL;
    if (active && f <= HALF) stage[l * HP + f] = fold_weight(f, HALF) * x[m].x;
  }
  __syncthreads();
  double* out = g + size_t(line0) * HP;
  for (int i = threadIdx.x; i < LINES * HP; i += THREADS) out[i] = stage[i];
}

// Pass 4: the folded inverse transform along y. Lines j = kx (N/2 + 1) + f_z
// of G[ky][j] (J = (N/2 + 1)^2 of them), 2 PAIRS consecutive lines per block
// (consecutive threads take consecutive lines, so each ky is read in one
// contiguous run); two real lines share one complex transform,
// Z = G_a + i G_b, and H[f_y][j] = mu(f_y) sum_ky G[ky][j] cos(2 pi ky f_y / N)
// is mu(f_y) Re of their transforms: Re A(f) = (Re Z(f) + Re Z(N - f)) / 2,
// Re B(f) = (Im Z(f) + Im Z(N - f)) / 2, for f_y = 0..N/2. Lines past J
// transform zeros and are not written.
template <int N, int PAIRS>
__global__ void __launch_bounds__(PAIRS * fft_threads(N)) cos_y_kernel(const double* g0, double* hout0,
                                                                       size_t wstride) {
  constexpr int HALF = N / 2, HP = HALF + 1, J = HP * HP, LS = lds_line<N>(), E = fft_elems(N), TPL = fft_threads(N);
  constexpr int THREADS = PAIRS * TPL;
  __shared__ double2 sh[PAIRS * LS];
  __shared__ double2 tw[N];
  const double* g = in_batch(g0, wstride);
  double* ho = in_batch(hout0, wstride);
  const int j0 = remap_block(blockIdx.x, gridDim.x, 1) * 2 * PAIRS;
  const int p = threadIdx.x % PAIRS, t = threadIdx.x / PAIRS;
  const int ja = j0 + 2 * p, jb = ja + 1;
  double2 x[E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const size_t row = size_t(t + m * TPL) * J;
    x[m] = make_double2(ja < J ? g[row + ja] : 0.0, jb < J ? g[row + jb] : 0.0);
  }
  make_twiddles<N>(tw);
  __syncthreads();
  fft_line<N, +1>(x, t, sh + p * LS, tw);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < E; ++m) sh[p * LS + t + m * TPL] = x[m];
  __syncthreads();
  for (int e = threadIdx.x; e < HP * PAIRS; e += THREADS) {
    const int f = e / PAIRS, pe = e % PAIRS;
    const int j = j0 + 2 * pe;
    if (j >= J) continue;
    const double2 z = sh[pe * LS + f], zn = sh[pe * LS + ((N - f) & (N - 1))];
    const bool edge = f == 0 || f == HALF;  // mu = 1 and Z(N - f) = Z(f)
    ho[size_t(f) * J + j] = edge ? z.x : z.x + zn.x;
    if (j + 1 < J) ho[size_t(f) * J + j + 1] = edge ? z.y : z.y + zn.y;
  }
}

// Pass 5: the folded inverse transform along x and the shell sums of S2.
// Rows q = f_y (N/2 + 1) + f_z of H[f_y][kx][f_z] (lines along kx =
// 0..N/2), 2 PAIRS consecutive rows per block. With y and z folded, H is
// even in kx (a mode at -kx is the conjugate partner of one at kx with ky,
// kz negated, and the folds are even in those), so the transform of its
// even extension is real: two rows share one complex transform, Z = E_a +
// i E_b giving x_a + i x_b, and X(f) = mu(f_x) x(f_x) is N^6 times the sum
// of R_h over the lags that fold to f. The shell sums of
// 2 (mu(f) R_0 - X(f)) (mu(f) the number of those lags) over the block's
// rows (each row folded by f_x, the rows added in order) go to
// rbins[block][r] (rows of N/2 + 2 values, the last one 0). r0: R_0 times
// N^6 (the sum of Psi). Rows past (N/2 + 1)^2 transform zeros and add
// nothing.
template <int N, int PAIRS>
__global__ void __launch_bounds__(last_threads(N, PAIRS * fft_threads(N)))
    cos_x_kernel(const double* hin0, const double* r00, double* rbins0, size_t wstride) {
  constexpr int HALF = N / 2, HP = HALF + 1, J = HP * HP, LS = lds_line<N>(), ROWS = 2 * PAIRS;
  constexpr int E = fft_elems(N), TPL = fft_threads(N), THREADS = last_threads(N, PAIRS * TPL);
  // the transforms, then (as doubles) the rows' X values and their shell sums
  constexpr int SH = PAIRS * LS > ROWS * HP ? PAIRS * LS : ROWS * HP;
  __shared__ double2 sh[SH];
  __shared__ double2 tw[N];
  const double* hin = in_batch(hin0, wstride);
  const double* r0 = in_batch(r00, wstride);
  double* rbins = in_batch(rbins0, wstride);
  const int q0 = remap_block(blockIdx.x, gridDim.x, 1) * ROWS;
  const int p = threadIdx.x % PAIRS, t = threadIdx.x / PAIRS;
  const bool active = t < TPL;
  const int qa = q0 + 2 * p, qb = qa + 1;
  const size_t ba = size_t(qa / HP) * J + qa % HP, bb = size_t(qb / HP) * J + qb % HP;
  double2 x[E];
  if (active) {
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int kx = t + m * TPL, kf = kx <= HALF ? kx : N - kx;  // the even extension
      x[m] = make_double2(qa < J ? hin[ba + size_t(kf) * HP] : 0.0, qb < J ? hin[bb + size_t(kf) * HP] : 0.0);
    }
  }
  make_twiddles<N>(tw);
  __syncthreads();
  fft_line<N, +1>(x, t, sh + p * LS, tw, active);
  __syncthreads();  // the transform's reads are done; sh holds the rows next
  double* xr = reinterpret_cast<double*>(sh);  // [ROWS][HP]
  double* part = xr + ROWS * HP;                // [ROWS][HP]
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const int f = t + m * TPL;
    if (active && f <= HALF) {
      xr[(2 * p) * HP + f] = fold_weight(f, HALF) * x[m].x;
      xr[(2 * p + 1) * HP + f] = fold_weight(f, HALF) * x[m].y;
    }
  }
  __syncthreads();
  const double R0 = *r0;
  for (int e = threadIdx.x; e < ROWS * HP; e += THREADS) {
    const int rho = e / HP, c = e % HP;
    const int q = q0 + rho;
    double sum = 0.0;
    if (q < J) {
      const int fy = q / HP, fz = q % HP;
      const double myz = fold_weight(fy, HALF) * fold_weight(fz, HALF);
      int a, b;
      shell_range(HALF, fy * fy + fz * fz, c, a, b);
      const double* row = xr + rho * HP;
      for (int m = a; m <= b; ++m) sum += 2.0 * (myz * fold_weight(m, HALF) * R0 - row[m]);
    }
    part[e] = sum;
  }
  __syncthreads();
  const size_t blk = size_t(q0 / ROWS);
  for (int c = threadIdx.x; c <= HALF + 1; c += THREADS) {
    double sum = 0.0;
    for (int r = 0; r < ROWS && c <= HALF; ++r) sum += part[r * HP + c];
    rbins[blk * (HALF + 2) + c] = sum;
  }
}

// Shell reduction, stage 1: block b sums rows [b CHUNK, (b+1) CHUNK) of the
// row-major table bins (width values per row) column by column, in row
// order, into psum[b][col].
constexpr int kShellChunk = 32;

__global__ void __launch_bounds__(256) shell_partial_kernel(const double* bins0, int rows, int width, double* psum0,
                                                            size_t wstride) {
  const double* bins = in_batch(bins0, wstride);
  double* psum = in_batch(psum0, wstride);
  const int r0 = blockIdx.x * kShellChunk;
  const int r1 = r0 + kShellChunk < rows ? r0 + kShellChunk : rows;
  for (int col = threadIdx.x; col < width; col += 256) {
    double a = 0.0;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) a += bins[size_t(r) * width + col];
    psum[size_t(blockIdx.x) * width + col] = a;
  }
}

// Number of lattice vectors of each shell, one block per shell r = 0..N/2:
// the vectors with components in {-N/2+1, ..., N/2} whose length rounds to
// r, counted over (p, q, m) folded to p, q, m >= 0 (whole numbers, exact in
// any order). They depend on n only; the spectrum and the structure
// function of every sample of a call share them.
__global__ void __launch_bounds__(256) shell_count_kernel(int n, double* cnt) {
  __shared__ double sc[256];
  const int col = blockIdx.x, half = n / 2;
  double c = 0.0;
  for (int e = threadIdx.x; e < (half + 1) * (half + 1); e += 256) {
    const int p = e / (half + 1), q = e % (half + 1);
    int lo, hi;
    shell_range(half, p * p + q * q, col, lo, hi);
    c += fold_weight(p, half) * fold_weight(q, half) * range_count(half, lo, hi);
  }
  sc[threadIdx.x] = c;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) sc[threadIdx.x] += sc[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) cnt[col] = sc[0];
}

// Stage 2, one block per column: the partials summed over the chunks (thread
// t takes chunks t, t + 256, ..., then a fixed tree), divided by the shell's
// number of vectors cnt[col] (shell_count_kernel). mode 0 (spectrum):
// out[kappa] = 4 pi / count * sum / N^6 for kappa = 0..N/2 (out may be NULL),
// and column N/2 + 1 (the sum of Psi, R_0 times N^6) into *r0. mode 1
// (structure function): out[r - 1] = sum / count / N^6 for r = 1..N/2.
__global__ void __launch_bounds__(256) shell_final_kernel(const double* psum0, const double* cnt, int chunks,
                                                          int width, int n, int mode, double* out0, double* r00,
                                                          size_t wstride) {
  __shared__ double sa[256];
  const double* psum = in_batch(psum0, wstride);
  double* out = out0 ? out0 + size_t(blockIdx.z) * (mode == 0 ? n / 2 + 1 : n / 2) : nullptr;
  double* r0 = r00 ? in_batch(r00, wstride) : nullptr;
  const int col = blockIdx.x, half = n / 2;
  double a = 0.0;
  for (int b = threadIdx.x; b < chunks; b += 256) a += psum[size_t(b) * width + col];
  sa[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) sa[threadIdx.x] += sa[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double norm = 1.0 / (double(n) * n * n) / (double(n) * n * n);
    const double sum = sa[0], cnt_c = col <= half ? cnt[col] : 0.0;
    if (mode == 0) {
      if (col <= half && out) out[col] = cnt_c > 0 ? 4.0 * M_PI / cnt_c * sum * norm : 0.0;
      if (col == half + 1 && r0) *r0 = sum;
    } else if (col >= 1 && col <= half) {
      out[col - 1] = cnt_c > 0 ? sum * norm / cnt_c : 0.0;
    }
  }
}

// Velocity of every sample at the q^3 nodes x = (n/q) * j: out[s][3][q^3].
template <int QN, typename T>
__global__ void __launch_bounds__(64) point_values_kernel(const T* pop, const DevSample* samples, const Seg* segs,
                                                          int q, int physical, double* out) {
  const Seg sg = segs[blockIdx.y];
  const DevSample& sp = samples[sg.sample];
  const int l = sp.log2n;
  const int n = 1 << l;
  const int q3 = q * q * q;
  const int j = blockIdx.x * 64 + threadIdx.x;
  if (j >= q3) return;
  const int step = n / q;
  const int jx = j % q, jy = (j / q) % q, jz = j / (q * q);
  const uint32_t msk = uint32_t(n - 1);
  const uint32_t x = uint32_t(jx * step), y = uint32_t(jy * step), z = uint32_t(jz * step);
  const T* base = pop + sp.offset;
  const bool odd = sg.parity & 1;
  double d = 0.0, jxs = 0.0, jys = 0.0, jzs = 0.0;
  for (int i = 0; i < Q; ++i) {
    if (!in_lattice<QN>(i)) continue;
    size_t idx;
    int slot;
    if (!odd) {
      idx = (size_t(z) << (2 * l)) + (size_t(y) << l) + x;
      slot = plane_of<QN>(i);
    } else {
      const uint32_t xs = (x - uint32_t(cx(i))) & msk, ys = (y - uint32_t(cy(i))) & msk,
                     zs = (z - uint32_t(cz(i))) & msk;
      idx = (size_t(zs) << (2 * l)) + (size_t(ys) << l) + xs;
      slot = plane_of<QN>(opposite(i));
    }
    const double v = double(base[size_t(slot) * sp.pstride + idx]);
    d += v;
    jxs += cx(i) * v;
    jys += cy(i) * v;
    jzs += cz(i) * v;
  }
  const double rho = physical ? (1.0 + d) * sp.u0 : 1.0 + d;   // u / u0 or u
  double* o = out + size_t(sg.sample) * 3 * q3;
  o[j] = jxs / rho;
  o[q3 + j] = jys / rho;
  o[2 * q3 + j] = jzs / rho;
}

__device__ __forceinline__ double flip_sign(double v, uint32_t sign) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  return __builtin_bit_cast(double, u ^ (uint64_t(sign) << 32));
}

// Sorting a column of 64 E values in the registers of one wave (bitonic):
// position i of the sorted order is element i % E of lane i / E. Steps of the
// network whose partner lies E or more positions away exchange between lanes,
// the others inside a lane, both without barriers. Merges that run downwards in
// a lane run upwards on the negated values, so that the direction costs one
// sign flip per value and merge instead of selects in every step.
template <int E>
__device__ __forceinline__ void wave_sort(double (&v)[E], int lane) {
  static_for<1, log2_of(64 * E) + 1>([&](auto kc) {
    constexpr int k = 1 << decltype(kc)::value;
    const uint32_t sign = k >= E && ((lane * E) & k) != 0 ? 0x80000000u : 0u;
    if constexpr (k >= E) {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = flip_sign(v[e], sign);
    }
    static_for<0, decltype(kc)::value>([&](auto jc) {
      constexpr int j = k >> (decltype(jc)::value + 1);
      if constexpr (j >= E) {
        const bool low = ((lane * E) & j) == 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const double o = __shfl_xor(v[e], j / E, 64);
          const double lo = fmin(v[e], o), hi = fmax(v[e], o);
          v[e] = low ? lo : hi;
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          if ((e & j) == 0) {
            const bool up = k >= E || (e & k) == 0;
            const double lo = fmin(v[e], v[e | j]), hi = fmax(v[e], v[e | j]);
            v[e] = up ? lo : hi;
            v[e | j] = up ? hi : lo;
          }
        }
      }
    });
    if constexpr (k >= E) {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = flip_sign(v[e], sign);
    }
  });
}

// Columns of one block of w1_wave_kernel, one wave each: neighbouring columns
// share the 64-byte segments that the rows are read in.
constexpr int kW1Columns = 4;

// One wave per (component, node), for m <= 64 E: sort the m values of both
// ensembles in registers and average |a_(i) - b_(i)|. The values come through
// LDS so that the block reads each row's neighbouring columns together. A NaN
// (which minima drop) makes the column NaN. Bound by the network's
// instructions: 1000 values of 1536 columns 163 us in LDS with a barrier per
// step, one block per column, against 52.
template <int E>
__global__ void __launch_bounds__(64 * kW1Columns)
    w1_wave_kernel(const double* a, const double* b, int m, int q3, double* col) {
  __shared__ double tile[kW1Columns][64 + 1];
  const int c0 = blockIdx.x * kW1Columns, columns = 3 * q3;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int tr = threadIdx.x / kW1Columns, tc = threadIdx.x % kW1Columns;
  double v[2][E];
  bool nan = false;
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const double* x = side ? b : a;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int row = 64 * e + tr;
      tile[tc][tr] = row < m && c0 + tc < columns ? x[size_t(row) * columns + c0 + tc] : 1.0e308;
      __syncthreads();
      v[side][e] = tile[w][lane];
      nan = nan || v[side][e] != v[side][e];
      __syncthreads();
    }
    wave_sort<E>(v[side], lane);
  }
  double acc = 0.0;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (lane * E + e < m) acc += fabs(v[0][e] - v[1][e]);
  acc = wave_sum(acc);
  if (__any(nan)) acc = __builtin_nan("");
  if (lane == 0 && c0 + w < columns) col[c0 + w] = acc / m;
}

// The same with one block per column for 1024 < m <= 4096, more values than a
// wave's registers hold in a network of bounded code size: bitonic sort in LDS
// (whose comparisons would carry a NaN to any place; the column becomes NaN here too).
__global__ void __launch_bounds__(256) w1_column_kernel(const double* a, const double* b, int m, int q3, int p2,
                                                        double* col) {
  __shared__ double sa[4096], sb[4096];
  const int c = blockIdx.x;  // column = comp * q3 + node
  bool nan = false;
  for (int i = threadIdx.x; i < p2; i += 256) {
    sa[i] = i < m ? a[size_t(i) * 3 * q3 + c] : 1.0e308;
    sb[i] = i < m ? b[size_t(i) * 3 * q3 + c] : 1.0e308;
    nan = nan || sa[i] != sa[i] || sb[i] != sb[i];
  }
  nan = __syncthreads_or(nan);
  for (int k = 2; k <= p2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < p2; i += 256) {
        const int ixj = i ^ j;
        if (ixj > i) {
          const bool up = (i & k) == 0;
          double x = sa[i], y = sa[ixj];
          if ((x > y) == up) {
            sa[i] = y;
            sa[ixj] = x;
          }
          x = sb[i];
          y = sb[ixj];
          if ((x > y) == up) {
            sb[i] = y;
            sb[ixj] = x;
          }
        }
      }
      __syncthreads();
    }
  }
  __shared__ double red[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) acc += fabs(sa[i] - sb[i]);
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) col[c] = nan ? __builtin_nan("") : red[0] / m;
}

// out[c] = (1/q^3) sum over nodes of the column distances of component c.
__global__ void __launch_bounds__(256) w1_reduce_kernel(const double* col, int q3, double* out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < q3; i += 256) acc += col[size_t(blockIdx.x) * q3 + i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] / q3;
}

// One block per sample: the eight sums of the relative L1 sample error
// (numerator and denominator for the three components and for the Euclidean
// length of the vector) over the q^3 nodes, then their four ratios.
__global__ void __launch_bounds__(256) sample_error_kernel(const double* a, const double* b, int q3, double* ratio) {
  const size_t base = size_t(blockIdx.x) * 3 * q3;
  double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int j = threadIdx.x; j < q3; j += 256) {
    double d2 = 0.0, r2 = 0.0;
    for (int c = 0; c < 3; ++c) {
      const double x = a[base + size_t(c) * q3 + j], r = b[base + size_t(c) * q3 + j];
      acc[2 * c] += fabs(x - r);
      acc[2 * c + 1] += fabs(r);
      d2 += (x - r) * (x - r);
      r2 += r * r;
    }
    acc[6] += sqrt(d2);
    acc[7] += sqrt(r2);
  }
  __shared__ double red[8][256];
  for (int k = 0; k < 8; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st)
      for (int k = 0; k < 8; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 4) ratio[size_t(blockIdx.x) * 4 + threadIdx.x] = red[2 * threadIdx.x][0] / red[2 * threadIdx.x + 1][0];
}

// out[k] = mean over the m samples of ratio[m][k], one block per k.
__global__ void __launch_bounds__(256) sample_mean_kernel(const double* ratio, int m, double* out) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) acc += ratio[size_t(i) * 4 + blockIdx.x];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0] / m;
}

// Column statistics of x[m][ld] over its m rows, one block per column: the
// mean by a fixed-order sum, then the spread about it (second pass) with the
// 1/(m - 1) normalisation of the empirical variance.
__global__ void __launch_bounds__(256) ensemble_moments_kernel(const double* x, int m, int64_t ld, double* mean,
                                                               double* sd) {
  __shared__ double red[256];
  const int c = blockIdx.x;
  double acc = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) acc += x[size_t(i) * ld + c];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  const double mu = red[0] / m;
  if (threadIdx.x == 0) mean[c] = mu;
  if (!sd) return;
  __syncthreads();  // every thread has read red[0]
  acc = 0.0;
  for (int i = threadIdx.x; i < m; i += 256) {
    const double v = x[size_t(i) * ld + c] - mu;
    acc += v * v;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) sd[c] = sqrt(red[0] / (m - 1));
}

// Sample-wise compensation of the spectra and structure functions of the
// samples sample0.. (one n): element j of a row of width n + 1 is kappa = j
// of the spectrum for j <= n/2, else lag r = j - n/2 of the structure
// function. Velocities in units of the sample's u0; lags in physical units.
__global__ void __launch_bounds__(256) compensate_kernel(const DevSample* samples, int sample0, int count, int n,
                                                         const double* d, const double* s2, const double* ek,
                                                         double* s2c, double* ekc) {
  constexpr double kKolmogorov = 1.5;
  const int half = n / 2, width = n + 1;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= count * width) return;
  const int s = e / width, j = e % width;
  const double u0 = samples[sample0 + s].u0;
  const double ds = d[s];
  if (j <= half) {
    if (ek) {
      const size_t o = size_t(s) * (half + 1) + j;
      ekc[o] = pow(double(j), 5.0 / 3.0) * (ek[o] / (u0 * u0)) / (kKolmogorov * cbrt(ds * ds));
    }
  } else if (s2) {
    const int r = j - half;
    const size_t o = size_t(s) * half + (r - 1);
    const double dr = ds * (r * 2.0 * M_PI / n);
    s2c[o] = (s2[o] / (u0 * u0)) / cbrt(dr * dr);
  }
}


struct ObsWork {
  double2* h;       // 3 fields of N * N * NH complex; after pass 3, H
  double* g;        // N (N/2 + 1)^2: the folded z-transform G
  double* sbins;    // spectrum_bin_rows(N) rows of N/2 + 2
  double* rbins;    // sf_bin_rows(N) rows of N/2 + 2
  double* psum;     // one row of N/2 + 2 per chunk of either table
  double* r0;       // 1
  double* cnt;      // N/2 + 1 shell sizes (used in the first sample's area)
};

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

size_t chunks_of(size_t rows) { return (rows + kShellChunk - 1) / kShellChunk; }

// Byte sizes of the parts of one sample's work area (each a multiple of 256)
struct WorkSizes {
  size_t h, g, sbins, rbins, psum, r0, cnt;
  size_t total() const { return h + g + sbins + rbins + psum + r0 + cnt; }
};

WorkSizes work_sizes(int n) {
  const size_t nh = size_t(n / 2 + 1), width = size_t(n / 2 + 2);
  const size_t srows = spectrum_bin_rows(n), rrows = sf_bin_rows(n);
  WorkSizes z;
  z.h = align256(3 * size_t(n) * n * nh * sizeof(double2));
  z.g = align256(size_t(n) * folded_lines(n) * sizeof(double));
  z.sbins = align256(srows * width * sizeof(double));
  z.rbins = align256(rrows * width * sizeof(double));
  z.psum = align256(chunks_of(std::max(srows, rrows)) * width * sizeof(double));
  z.r0 = align256(sizeof(double));
  z.cnt = align256(width * sizeof(double));
  return z;
}

// bytes of one sample's work area (a multiple of 256)
size_t sample_work_bytes(int n) { return work_sizes(n).total(); }

ObsWork carve(void* work, int n) {
  const WorkSizes z = work_sizes(n);
  char* p = static_cast<char*>(work);
  ObsWork w;
  w.h = reinterpret_cast<double2*>(p);
  w.g = reinterpret_cast<double*>(p += z.h);
  w.sbins = reinterpret_cast<double*>(p += z.g);
  w.rbins = reinterpret_cast<double*>(p += z.sbins);
  w.psum = reinterpret_cast<double*>(p += z.rbins);
  w.r0 = reinterpret_cast<double*>(p += z.psum);
  w.cnt = reinterpret_cast<double*>(p += z.r0);
  return w;
}

template <int QN, typename T, int N, bool FROM_U>
hipError_t observables_t(const T* pop, const double* u, const DevSample* samples, int sample0, int count, int parity,
                         void* work, double* s2, double* ek, hipStream_t s) {
  constexpr int NH = N / 2 + 1, LY = y_lines(N), LZ = z_lines(N);
  constexpr int ROWS_X = fwd_rows(N);
  constexpr int PC = cos_pairs(N);
  constexpr int W = N / 2 + 2;
  static_assert(N % LY == 0 && N % LZ == 0 && (N * N) % ROWS_X == 0, "launch shapes must tile the field");
  const ObsWork w = carve(work, N);
  const size_t ws = sample_work_bytes(N);
  const unsigned z = unsigned(count);
  const int lines = N * NH;
  const int srows = int(spectrum_bin_rows(N)), rrows = int(sf_bin_rows(N));
  const int lchunks = int(chunks_of(srows)), rchunks = int(chunks_of(rrows));
  hipLaunchKernelGGL((fwd_x_kernel<QN, T, N, FROM_U>), dim3(N * N / ROWS_X, 1, z), dim3(256), 0, s, pop, u, samples,
                     sample0, parity, w.h, ws);
  constexpr int TPL = fft_threads(N);
  hipLaunchKernelGGL((fft_y_kernel<N, LY>), dim3(lines / LY, 3, z), dim3(LY * TPL), 0, s, w.h, ws);
  hipLaunchKernelGGL((z_psd_kernel<N, LZ>), dim3(lines / LZ, 1, z), dim3(sum_threads(N, LZ * TPL)), 0, s, w.h, w.g, w.sbins, ws);
  hipLaunchKernelGGL(shell_partial_kernel, dim3(lchunks, 1, z), dim3(256), 0, s, w.sbins, srows, W, w.psum, ws);
  hipLaunchKernelGGL(shell_count_kernel, dim3(NH), dim3(256), 0, s, N, w.cnt);
  hipLaunchKernelGGL(shell_final_kernel, dim3(W, 1, z), dim3(256), 0, s, w.psum, w.cnt, lchunks, W, N, 0, ek, w.r0,
                     ws);
  if (s2) {
    double* hr = reinterpret_cast<double*>(w.h);
    hipLaunchKernelGGL((cos_y_kernel<N, PC>), dim3(rrows, 1, z), dim3(PC * TPL), 0, s, w.g, hr, ws);
    hipLaunchKernelGGL((cos_x_kernel<N, PC>), dim3(rrows, 1, z), dim3(last_threads(N, PC * TPL)), 0, s, hr, w.r0, w.rbins, ws);
    hipLaunchKernelGGL(shell_partial_kernel, dim3(rchunks, 1, z), dim3(256), 0, s, w.rbins, rrows, W, w.psum, ws);
    hipLaunchKernelGGL(shell_final_kernel, dim3(W, 1, z), dim3(256), 0, s, w.psum, w.cnt, rchunks, W, N, 1, s2,
                       nullptr, ws);
  }
  return hipGetLastError();
}

template <int QN, typename T, bool FROM_U>
hipError_t observables_n(int n, const void* pop, const double* u, const DevSample* samples, int sample0, int count,
                         int parity, void* work, double* s2, double* ek, hipStream_t s) {
  const T* p = static_cast<const T*>(pop);
  switch (n) {
    case 8: return observables_t<QN, T, 8, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 16: return observables_t<QN, T, 16, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 32: return observables_t<QN, T, 32, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 64: return observables_t<QN, T, 64, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 128: return observables_t<QN, T, 128, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 256: return observables_t<QN, T, 256, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    case 512: return observables_t<QN, T, 512, FROM_U>(p, u, samples, sample0, count, parity, work, s2, ek, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

size_t observables_work_bytes(int n, int count) { return sample_work_bytes(n) * size_t(count); }

hipError_t launch_observables(int q, int precision, const void* pop, const DevSample* samples, int32_t sample0,
                              int32_t count, int32_t n, int32_t parity, void* work, double* s2, double* ek,
                              hipStream_t s) {
  if (q == 27) {
    return precision == 0
               ? observables_n<27, double, false>(n, pop, nullptr, samples, sample0, count, parity, work, s2, ek, s)
               : observables_n<27, float, false>(n, pop, nullptr, samples, sample0, count, parity, work, s2, ek, s);
  }
  if (q == 19) {
    return precision == 0
               ? observables_n<19, double, false>(n, pop, nullptr, samples, sample0, count, parity, work, s2, ek, s)
               : observables_n<19, float, false>(n, pop, nullptr, samples, sample0, count, parity, work, s2, ek, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_observables_velocity(const double* u, const DevSample* samples, int32_t sample0, int32_t count,
                                       int32_t n, void* work, double* s2, double* ek, hipStream_t s) {
  return observables_n<27, double, true>(n, nullptr, u, samples, sample0, count, 0, work, s2, ek, s);
}

hipError_t launch_point_values(int lattice, int precision, const void* pop, const DevSample* samples,
                               const Seg* segs, int32_t nseg, int q, int physical, double* out, hipStream_t s) {
  const dim3 grid(unsigned((q * q * q + 63) / 64), unsigned(nseg));
  if (lattice == 27 && precision == 0)
    hipLaunchKernelGGL((point_values_kernel<27, double>), grid, dim3(64), 0, s, static_cast<const double*>(pop),
                       samples, segs, q, physical, out);
  else if (lattice == 27)
    hipLaunchKernelGGL((point_values_kernel<27, float>), grid, dim3(64), 0, s, static_cast<const float*>(pop),
                       samples, segs, q, physical, out);
  else if (lattice == 19 && precision == 0)
    hipLaunchKernelGGL((point_values_kernel<19, double>), grid, dim3(64), 0, s, static_cast<const double*>(pop),
                       samples, segs, q, physical, out);
  else if (lattice == 19)
    hipLaunchKernelGGL((point_values_kernel<19, float>), grid, dim3(64), 0, s, static_cast<const float*>(pop),
                       samples, segs, q, physical, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_w1(const double* a, const double* b, int m, int q, double* col, double* out, hipStream_t s) {
  const int q3 = q * q * q;
  int p2 = 1;
  while (p2 < m) p2 <<= 1;
  const dim3 waves(unsigned((3 * q3 + kW1Columns - 1) / kW1Columns)), block(64 * kW1Columns);
  if (p2 <= 64) hipLaunchKernelGGL(w1_wave_kernel<1>, waves, block, 0, s, a, b, m, q3, col);
  else if (p2 == 128) hipLaunchKernelGGL(w1_wave_kernel<2>, waves, block, 0, s, a, b, m, q3, col);
  else if (p2 == 256) hipLaunchKernelGGL(w1_wave_kernel<4>, waves, block, 0, s, a, b, m, q3, col);
  else if (p2 == 512) hipLaunchKernelGGL(w1_wave_kernel<8>, waves, block, 0, s, a, b, m, q3, col);
  else if (p2 == 1024) hipLaunchKernelGGL(w1_wave_kernel<16>, waves, block, 0, s, a, b, m, q3, col);
  else hipLaunchKernelGGL(w1_column_kernel, dim3(unsigned(3 * q3)), dim3(256), 0, s, a, b, m, q3, p2, col);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(w1_reduce_kernel, dim3(3), dim3(256), 0, s, col, q3, out);
  return hipGetLastError();
}

// Device scratch of the sample error for callers that cannot allocate: the
// per-sample ratios, 4 doubles per sample. Each GPU holds its own copy for the
// life of the process; its address is looked up once per device
// (hipGetSymbolAddress with that device current) and kept, and kernels
// receive that address, never the array's name, which in host code is only
// a stand-in.
static __device__ __align__(256) double scratch[4 * kNoAllocMaxSamples];

static std::mutex g_scratch_mutex;
static std::vector<double*> g_scratch_ptr;  // per device; nullptr until looked up

hipError_t sample_error_scratch(double** ratio) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (size_t(dev) >= g_scratch_ptr.size()) g_scratch_ptr.resize(size_t(dev) + 1, nullptr);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *ratio = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_sample_error(const double* a, const double* b, int m, int q, double* ratio, double* out,
                               hipStream_t s) {
  hipLaunchKernelGGL(sample_error_kernel, dim3(unsigned(m)), dim3(256), 0, s, a, b, q * q * q, ratio);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sample_mean_kernel, dim3(4), dim3(256), 0, s, ratio, m, out);
  return hipGetLastError();
}

hipError_t launch_ensemble_moments(const double* x, int m, int k, int64_t ld, double* mean, double* sd,
                                   hipStream_t s) {
  hipLaunchKernelGGL(ensemble_moments_kernel, dim3(unsigned(k)), dim3(256), 0, s, x, m, ld, mean, sd);
  return hipGetLastError();
}

hipError_t launch_compensate(const DevSample* samples, int sample0, int count, int n, const double* d,
                             const double* s2, const double* ek, double* s2c, double* ekc, hipStream_t s) {
  const int total = count * (n + 1);
  hipLaunchKernelGGL(compensate_kernel, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, samples, sample0, count,
                     n, d, s2, ek, s2c, ekc);
  return hipGetLastError();
}

}  // namespace mclbm
