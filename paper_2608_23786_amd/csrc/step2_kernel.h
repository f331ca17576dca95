// Two collide-and-stream steps in one pass over memory.
//
// One step moves 2 q values per node through HBM and runs at the copy rate of
// the card, so the only way to go faster is to move less: this kernel reads
// the populations of a state once, takes two steps, and writes them once.
// Source and destination are different buffers in the same layout; a pair of
// launches, there and back, advances the in-place state by four steps. Either
// layout of the in-place scheme serves. After an even number of steps slot i of
// a node holds population i before its collision: the loads are to the node's own
// place and the stores stream. After an odd number slot -i holds population i
// after its collision: the loads stream (population i of node x from x - c_i) and
// the stores are to the node's own place. Rows that lie whole in a tile stay in
// whole lines either way and take the even layout; 64-node tiles of longer rows
// take the odd one, since stores off their lines by one node write them in parts
// (1.12 x the bytes at 256^3). us a pass in the even / odd layout, taken with a
// cheaper collision: 64 x 64^3 794 / 839, one 256^3 1028 / 891, 8 x 128^3 1050 / 887.
//
// us a pass / two single steps, FP32: 64 x 64^3 842 / 1162, 512 x 32^3 777 / 1180,
// 8 x 128^3 1077 / 1240, one 256^3 961 / 1252, one 512^3 8078 / 11720; 64 x 64^3 of
// D3Q19 598 / 811; FP64 64 x 64^3 1617 / 2386. Bound by arithmetic in FP32 (two
// collisions of 700 issue slots and the rim's share per node), by what it reads
// and writes, rims included, in FP64.
//
// A block owns a tile of nodes in the x-y plane and marches along z. Per plane
// it loads the 27 populations of its nodes, takes the first collision, and
// keeps the results on chip until the planes around them are there: a node's
// second collision needs the first-step results of its 26 neighbours. Values
// that stay in their row (c_y = 0) move by one lane and wait in registers;
// values that change row (c_y != 0) wait in LDS, those with c_z = -1, 0, +1 for
// the second collision of the same, the next and the next but one iteration,
// so 1, 2 and 3 planes of them are held: (6 + 12 + 18) values per node for
// D3Q27, 147 KB of the CU's 160 KB for 1024 nodes.
//
// The first collision is taken in the tile's rim as well (redundantly in the
// neighbouring tiles): one row on each side in y unless the tile spans the
// axis, one lane on each side in x where rows are longer than the tile, and
// one plane on each end of the z range. Loads of the next plane are issued
// before the second collision, which hides them.
#pragma once

#include "lbm_device.h"

namespace mclbm {
namespace {

// A run of samples of one resolution, tiled alike. The z planes of all its
// samples form one list; `teams` teams of blocks take equal contiguous parts of
// it (whatever samples such a part cuts), the blocks of a team one tile each,
// so that neighbouring tiles, which share the lines of their rims, march
// through the same planes at the same time.
template <typename T>
struct Step2Args {
  const T* src;
  T* dst;
  int64_t src_shift, dst_shift;  // element offset of a sample's populations: DevSample::offset + shift
  const DevSample* samples;
  int32_t sample0;
  int32_t log2n;
  int32_t tiles_x, tiles_y;
  int32_t teams;
  int32_t planes;                // samples * n
  int32_t* flags;
};

template <typename T>
__device__ __forceinline__ T uniform_value(T v) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
  else
    return __builtin_bit_cast(T, uniform64(__builtin_bit_cast(uint64_t, v)));
}

// Population planes through buffer resources: a lane gives a 32-bit byte
// offset, the plane, row and z offsets stay in scalar registers. WIDE: for
// samples of 2 GiB and more the resource is built per plane on a 64-bit base,
// which walks from plane to plane (one such walk per set of loads or stores:
// 27 resources kept through the loop would not fit the scalar registers).
template <typename T, int QN, bool WIDE>
struct Slabs {
  char* base;
  uint64_t plane_bytes;
  __device__ __forceinline__ Slabs(T* b, uint32_t pstride)
      : base(reinterpret_cast<char*>(uniform64(reinterpret_cast<uint64_t>(b)))),
        plane_bytes(uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(pstride)))) * sizeof(T)) {}

  // f(resource, scalar plane offset, velocity) for every velocity, planes ascending
  template <typename F>
  __device__ __forceinline__ void for_planes(F&& f) const {
    if constexpr (WIDE) {
      uint64_t p = reinterpret_cast<uint64_t>(base);
      asm volatile("" : "+s"(p));
      for_vel<QN>([&](auto ic) {
        f(__builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(p), 0, int(0xFFFFFFFFu), kBufferFlags), 0u, ic);
        p += plane_bytes;
      });
    } else {
      const __amdgpu_buffer_rsrc_t r =
          __builtin_amdgcn_make_buffer_rsrc(base, 0, int(uint32_t(QN) * uint32_t(plane_bytes)), kBufferFlags);
      for_vel<QN>([&](auto ic) { f(r, uint32_t(plane_of<QN>(decltype(ic)::value)) * uint32_t(plane_bytes), ic); });
    }
  }
};

// Loads through the caches (a neighbouring tile of the same XCD reads the rim's
// lines again), stores marked non-temporal (the other setting of either was
// 0 to 4 % slower at 64^3 and up to 28 % at 128^3 and up, measured).
template <typename T>
__device__ __forceinline__ T slab_load(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, int(off), int(soff), 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, int(off), int(soff), 0));
}
template <typename T>
__device__ __forceinline__ void slab_store(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff, T v) {
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, int(off), int(soff), kAuxNontemporal);
  else
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), v), r, int(off), int(soff),
        kAuxNontemporal);
}

// Rank of velocity i among those of its c_z that change row (c_y != 0), and
// their number: the value's place in its LDS plane.
template <int QN>
__host__ __device__ constexpr int row_rank(int i) {
  int r = 0;
  for (int k = 0; k < i; ++k)
    if (in_lattice<QN>(k) && cy(k) != 0 && cz(k) == cz(i)) ++r;
  return r;
}
template <int QN>
__host__ __device__ constexpr int row_count(int c) {
  int r = 0;
  for (int k = 0; k < Q; ++k)
    if (in_lattice<QN>(k) && cy(k) != 0 && cz(k) == c) ++r;
  return r;
}
// LDS planes: c_z = -1 at 0, two of c_z = 0, three of c_z = +1
template <int QN>
__host__ __device__ constexpr int lds_planes() {
  return row_count<QN>(-1) + 2 * row_count<QN>(0) + 3 * row_count<QN>(1);
}

// Tile shape: rows of LX nodes, R rows per block (one wave per row where LX is
// 64). HY: the tile has a rim of one row on each side in y (0 where it spans
// the axis). SIDE: it also has a rim of one column on each side in x, where
// rows are longer than a wave: one more wave takes the first collision of the
// 2 R rim nodes, so that the rows keep whole, aligned lines.
template <int QN, typename T, int LX, int R, int HY, bool SIDE, bool WIDE>
__global__ void __launch_bounds__((R + SIDE) * LX) kbc_step2_kernel(Step2Args<T> a) {
  static_assert((R + SIDE) * LX <= 1024 && ((R + SIDE) * LX) % 64 == 0, "whole waves");
  static_assert(!SIDE || (HY == 1 && LX == 64 && 2 * R <= 64), "the rim columns fit one wave");
  constexpr int STRIDE = LX + 2 * SIDE, NODES = R * STRIDE;      // LDS elements per row and per plane of values
  constexpr bool UNIFORM_ROW = LX == 64;                         // a wave lies in one row (or in the rim columns)
  constexpr int RPW = 64 / LX;                                   // rows per wave
  constexpr bool PULL = SIDE;                                    // the layout of odd parity
  constexpr uint32_t S = uint32_t(sizeof(T));
  constexpr int NM = row_count<QN>(-1), N0 = row_count<QN>(0), NP = row_count<QN>(1);
  __shared__ T lds[lds_planes<QN>() * NODES];
  __shared__ T edge[SIDE ? R : 1][6];  // c_y = 0 values entering a row: from the right rim (c_x = -1), from the left

  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const bool side_wave = SIDE && wave == R;

  // LDS column and row of this thread's node (a rim column left of 0 where
  // there is one). Addresses are formed from them where they are used, about
  // 20 instructions per plane: kept through the loop they would push the
  // collision's values out of the 128 registers that 16 waves per CU leave.
  auto row_thread = [&](int& col, int& row) {
    int t = int(threadIdx.x);
    asm volatile("" : "+v"(t));
    col = t % LX + (SIDE ? 1 : 0);
    row = UNIFORM_ROW ? wave : t / LX;
  };
  auto thread = [&](int& col, int& row) {
    row_thread(col, row);
    if constexpr (SIDE) {
      const int k = col - 1, pair = k >> 1;  // lanes past the rim repeat a node
      row = side_wave ? (pair < R ? pair : R - 1) : row;
      col = side_wave ? (k & 1) * (LX + 1) : col;
    }
  };

  // a value that stays in its row moves one lane along x
  auto lane_shift = [&](T v, int c) {
    if constexpr (LX >= 64) {
      return c > 0 ? rotate_lanes<true>(v) : rotate_lanes<false>(v);
    } else {
      int t = int(threadIdx.x);
      asm volatile("" : "+v"(t));
      const int p = ((t & 63 & ~(LX - 1)) + ((t + (c > 0 ? -1 : 1)) & (LX - 1))) * 4;
      if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_ds_bpermute(p, __builtin_bit_cast(int, v)));
      } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(p, int(uint32_t(u))));
        const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(p, int(uint32_t(u >> 32))));
        return __builtin_bit_cast(T, (uint64_t(hi) << 32) | lo);
      }
    }
  };

  const int b = remap_block(blockIdx.x, gridDim.x, 1);
  const int tiles = a.tiles_x * a.tiles_y, team = b / tiles, tile = b - team * tiles;
  const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
  const int l = a.log2n, n = 1 << l;
  const uint32_t msk = uint32_t(n - 1);
  int at = int((int64_t(a.planes) * team) / a.teams);
  const int end = int((int64_t(a.planes) * (team + 1)) / a.teams);
  while (at < end) {
    // the next run of planes of one sample
    const int z0 = at & (n - 1), z1 = end - at < n - z0 ? z0 + (end - at) : n;
    const int sample = a.sample0 + (at >> l);
    at += z1 - z0;
    const DevSample& sp = a.samples[sample];
    const int y0 = (ty * n) / a.tiles_y, ny = ((ty + 1) * n) / a.tiles_y - y0;
    const int x0 = tx * LX;
    // whether this wave takes the first collision, and the second
    const bool first = HY == 0 || side_wave || wave * RPW < ny + 2;
    const bool second = HY == 0 || (!side_wave && wave * RPW + RPW > 1 && wave * RPW <= ny);

    const uint32_t zbytes = S << (2 * l);
    const Slabs<T, QN, WIDE> src(const_cast<T*>(a.src) + (int64_t(sp.offset) + a.src_shift), sp.pstride);
    const Slabs<T, QN, WIDE> dst(a.dst + (int64_t(sp.offset) + a.dst_shift), sp.pstride);
    // in scalar registers
    Relax<T> rp = relax_of<T>(sp);
    rp.omega = uniform_value(rp.omega);
    rp.two_over_omega = uniform_value(rp.two_over_omega);
    rp.kappa = uniform_value(rp.kappa);
    rp.eps = uniform_value(rp.eps);

    T hold0[3] = {T(0), T(0), T(0)}, holdp1[3] = {T(0), T(0), T(0)}, holdp2[3] = {T(0), T(0), T(0)};  // by c_x + 1
    int w0 = NM * NODES, r0 = (NM + N0) * NODES;                  // c_z = 0: written / read plane
    int wp = (NM + 2 * N0) * NODES, mp = wp + NP * NODES, rp0 = mp + NP * NODES;  // c_z = +1: written, waiting, read
    bool bad = false;

    T g[Q];
    // byte offsets of the nodes around (x, y, z) against (SIGN -1) or along (+1)
    // the velocities, by c + 1 per axis
    auto around = [&](auto sign, int col, int row, int z, uint32_t (&xb)[3], uint32_t (&yb)[3], uint32_t (&zb)[3]) {
      constexpr int SIGN = decltype(sign)::value;
      const uint32_t x = uint32_t(x0 + col - SIDE), y = uint32_t(y0 + row - HY);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const uint32_t d = uint32_t(SIGN * (c - 1));
        xb[c] = ((x + d) & msk) * S;
        yb[c] = (((y + d) & msk) << l) * S;
        zb[c] = ((uint32_t(z) + d) & msk) * zbytes;
      }
    };
    auto load_plane = [&](int zz) {
      int col, row;
      thread(col, row);
      uint32_t xb[3], yb[3], zb[3];
      around(std::integral_constant<int, -1>{}, col, row, zz, xb, yb, zb);
      src.for_planes([&](__amdgpu_buffer_rsrc_t rs, uint32_t plane, auto ic) {
        constexpr int i = PULL ? opposite(decltype(ic)::value) : decltype(ic)::value;
        if constexpr (PULL) g[i] = slab_load<T>(rs, xb[cx(i) + 1] + yb[cy(i) + 1], plane + zb[cz(i) + 1]);
        else g[i] = slab_load<T>(rs, xb[1] + yb[1], plane + zb[1]);
      });
    };

    // the values of g are not needed any more: without this the compiler keeps
    // them for a last iteration that loads no further plane
    auto release = [&]() {
      for_vel<QN>([&](auto ic) {
        T undefined;
        asm volatile("" : "=v"(undefined));
        g[decltype(ic)::value] = undefined;
      });
    };

    T now[9];  // c_y = 0, by 3 (c_x + 1) + c_z + 1
    // first collision of a plane; its values to LDS and, shifted along x, to now
    auto first_collision = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      const CellResult<T> res = kbc_collide<QN>(g, rp);
      __builtin_amdgcn_sched_barrier(0);
      bad = bad || res.bad;
      int col, row;
      thread(col, row);
      const int me = row * STRIDE + col;
      for_vel<QN>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (cy(i) != 0) {
          constexpr int k = row_rank<QN>(i);
          const int plane = cz(i) < 0 ? 0 : cz(i) == 0 ? w0 : wp;
          lds[plane + k * NODES + me] = g[i];
        } else {
          constexpr int k = 3 * (cx(i) + 1) + cz(i) + 1;
          if constexpr (cx(i) == 0) now[k] = g[i];
          else now[k] = lane_shift(g[i], cx(i));
        }
      });
      if constexpr (SIDE) {
        if (side_wave) {
          for_vel<QN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (cy(i) == 0 && cx(i) != 0) {
              if ((col == 0) == (cx(i) > 0)) edge[row][(cx(i) > 0 ? 3 : 0) + cz(i) + 1] = g[i];
            }
          });
        }
      }
    };
    // the values that entered this row from the rim columns
    auto take_edges = [&]() {
      if constexpr (SIDE) {
        if (!side_wave) {
          const int lane = int(threadIdx.x) & 63;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const T right = edge[wave][c], left = edge[wave][3 + c];
            now[c] = lane == 63 ? right : now[c];
            now[6 + c] = lane == 0 ? left : now[6 + c];
          }
        }
      }
    };
    auto next_plane = [&]() {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        hold0[c] = now[3 * c + 1];
        holdp2[c] = holdp1[c];
        holdp1[c] = now[3 * c + 2];
      }
      const int t0 = w0;
      w0 = r0;
      r0 = t0;
      const int tp = rp0;
      rp0 = mp;
      mp = wp;
      wp = tp;
    };

    if (!first) {
      // a wave of a row beyond the tile keeps the others' barriers
      for (int zz = z0 - 1; zz <= z1; ++zz) {
        __syncthreads();
        __syncthreads();
      }
      __syncthreads();
      continue;
    }
    load_plane(z0 - 1);
#pragma unroll 1
    for (int zz = z0 - 1; zz <= z0; ++zz) {  // the planes below the first second collision
      first_collision();
      load_plane(zz + 1);
      __syncthreads();
      take_edges();
      __syncthreads();
      next_plane();
    }
#pragma unroll 1
    for (int zz = z0 + 1; zz <= z1; ++zz) {
      first_collision();
      __syncthreads();
      take_edges();
      if (second) {
        T f[Q];
        {
          // LDS element of the node a value comes from, (x - c_x, y - c_y)
          int col, row;
          row_thread(col, row);
          const int from_x[3] = {SIDE ? col + 1 : (col + 1) & (LX - 1), col, SIDE ? col - 1 : (col - 1) & (LX - 1)};
          // (a rim row in a wave of several rows computes values that are not used)
          const int up = !HY ? (row + 1) & (R - 1) : RPW > 1 && row == R - 1 ? row : row + 1;
          const int down = !HY ? (row - 1) & (R - 1) : RPW > 1 && row == 0 ? row : row - 1;
          const int from_y[3] = {up * STRIDE, row * STRIDE, down * STRIDE};
          for_vel<QN>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (cy(i) != 0) {
              constexpr int k = row_rank<QN>(i);
              const int plane = cz(i) < 0 ? 0 : cz(i) == 0 ? r0 : rp0;
              f[i] = lds[plane + k * NODES + from_y[cy(i) + 1] + from_x[cx(i) + 1]];
            } else {
              if constexpr (cz(i) < 0) f[i] = now[3 * (cx(i) + 1)];
              else if constexpr (cz(i) == 0) f[i] = hold0[cx(i) + 1];
              else f[i] = holdp2[cx(i) + 1];
            }
          });
        }
        __syncthreads();  // the planes read here are written in the next iteration
        release();
        if (zz < z1) load_plane(zz + 1);
        __builtin_amdgcn_sched_barrier(0);
        const CellResult<T> res = kbc_collide<QN>(f, rp);
        __builtin_amdgcn_sched_barrier(0);
        int col, row;
        row_thread(col, row);
        const bool out = !(HY && RPW > 1) || (row >= 1 && row <= ny);
        bad = bad || (out && res.bad);
        if (out) {
          uint32_t xb[3], yb[3], zb[3];
          around(std::integral_constant<int, 1>{}, col, row, zz - 1, xb, yb, zb);
          dst.for_planes([&](__amdgpu_buffer_rsrc_t rs, uint32_t plane, auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (PULL)
              slab_store<T>(rs, xb[1] + yb[1], plane + zb[1], f[opposite(i)]);
            else if constexpr (UNIFORM_ROW)
              slab_store<T>(rs, xb[cx(i) + 1], plane + zb[cz(i) + 1] + yb[cy(i) + 1], f[i]);
            else
              slab_store<T>(rs, yb[cy(i) + 1] + xb[cx(i) + 1], plane + zb[cz(i) + 1], f[i]);
          });
        }
      } else {
        __syncthreads();
        release();
        if (zz < z1) load_plane(zz + 1);
      }
      next_plane();
    }
    if (bad) a.flags[sample] = 1;
    __syncthreads();  // the next run writes the LDS planes that this one still reads
  }
}

template <int QN, typename T, int LX, int R, int HY, bool SIDE>
hipError_t launch_step2_tile(const Step2Launch& L, hipStream_t s) {
  Step2Args<T> a;
  a.src = static_cast<const T*>(L.src);
  a.dst = static_cast<T*>(L.dst);
  a.src_shift = L.src_shift;
  a.dst_shift = L.dst_shift;
  a.samples = L.samples;
  a.sample0 = L.sample0;
  a.log2n = L.log2n;
  a.tiles_x = L.tiles.x;
  a.tiles_y = L.tiles.y;
  a.teams = L.teams;
  a.planes = L.count << L.log2n;
  a.flags = L.flags;
  const dim3 grid(unsigned(L.teams * L.tiles.x * L.tiles.y)), blk((R + SIDE) * LX);
  if constexpr (SIDE) {
    if (L.wide) {
      hipLaunchKernelGGL((kbc_step2_kernel<QN, T, LX, R, HY, SIDE, true>), grid, blk, 0, s, a);
      return hipGetLastError();
    }
  }
  if (L.wide) return hipErrorInvalidValue;
  hipLaunchKernelGGL((kbc_step2_kernel<QN, T, LX, R, HY, SIDE, false>), grid, blk, 0, s, a);
  return hipGetLastError();
}

// The tile of a resolution (step2_tiles gives its counts to the host): whole
// planes up to 32 x 32 in float and 16 x 16 in double, then bands of rows of
// one wave, then 64-node tiles of longer rows with rim columns.
template <int QN, typename T>
hipError_t launch_step2_t(const Step2Launch& L, hipStream_t s) {
  constexpr bool f32 = std::is_same<T, float>::value;
  switch (L.log2n) {
    case 3: return launch_step2_tile<QN, T, 8, 8, 0, false>(L, s);
    case 4: return launch_step2_tile<QN, T, 16, 16, 0, false>(L, s);
    case 5:
      if constexpr (QN == 27 && !f32) return hipErrorInvalidValue;   // stays with single steps
      else return launch_step2_tile<QN, T, 32, f32 ? 32 : 16, f32 ? 0 : 1, false>(L, s);
    case 6: return launch_step2_tile<QN, T, 64, f32 ? 16 : 8, 1, false>(L, s);
    case 7:
    case 8:
    case 9: return launch_step2_tile<QN, T, 64, f32 ? 15 : 7, 1, true>(L, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace mclbm
