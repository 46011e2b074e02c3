// fam_strip.h - the marching-strip machinery shared by the stage, OE and
// adjoint kernels: a 64-lane wave owns a strip of columns and marches up a tile
// of rows, keeping three state rows in an LDS ring.
#pragma once

#include "fam_device.h"
#include "fam_kernels.h"

namespace fam {

constexpr int LANES = 64;

// ---------------------------------------------------------------------------
// LDS row window: lane l holds LDS column l = grid column i0 - 2 + l.  Lanes 0
// and 63 only load; lanes 1 and 62 are ring columns; lanes 2..61 write output.
// ---------------------------------------------------------------------------
template <int NPLU, int SLOTS = 3>
struct alignas(16) Window {
  // two values before and after the rows: the load-only lanes 0 and 63 read their
  // missing neighbour column there or in the next plane, and nothing uses what
  // they compute from it (two, not one, so that the rows start on 16 bytes)
  double f[SLOTS * NPLU * LANES + 4];
  __device__ __forceinline__ double& at(int slot, int plane, int col) {
    return f[2 + (slot * NPLU + plane) * LANES + col];
  }
  __device__ __forceinline__ double at(int slot, int plane, int col) const {
    return f[2 + (slot * NPLU + plane) * LANES + col];
  }
};

// three row slots used as a ring: row r+2 is fetched into the slot of row r-1
// once every read of row r-1 in the current iteration is done
__device__ __forceinline__ int slot_of(int r) { return ((r % 3) + 3) % 3; }

// row r, column ci of the double Mach reflection at boundary time tb (mesh or ghost
// cells; see fam_config.dmr), for all lanes at once
template <int NPLU>
__device__ __forceinline__ void dmr_cells(const double* __restrict__ U, const Inst& in, int r, int ci, double tb,
                                          double (&reg)[NPLU], long long moff) {
  const double xc = in.x0 + (ci + 0.5) * in.dx;
  // top: the exact shock line at the upper boundary; bottom inflow part, left inflow
  const bool top = r >= in.ny;
  const bool behind = xc < 1.0 / 6.0 + (in.ytop + 20.0 * tb) * 0.57735026918962576451;
  const bool post = top ? behind : r < 0 ? xc < 1.0 / 6.0 : ci < 0;
  // (rho, u, v, p) = (8, 8.25 cos 30deg, -8.25 sin 30deg, 116.5) behind the shock,
  // (1.4, 0, 0, 1) ahead; conservative, with 1/(gamma - 1) = in.dmr_einv
  constexpr double rl = 8.0, ul = 8.25 * 0.86602540378443864676, vl = -8.25 * 0.5, pl = 116.5;
  const double qpost[4] = {rl, rl * ul, rl * vl, pl * in.dmr_einv + 0.5 * rl * (ul * ul + vl * vl)};
  const double qpre[4] = {1.4, 0.0, 0.0, in.dmr_einv};
  // the others: the mesh cell itself, right outflow (copy of the last column) and,
  // below the mesh, the reflecting wall: mirror image of row -1 - r with rho v and
  // the y-moments of the other components negated
  const int gi = min(max(ci, 0), in.nx - 1);
  const int gj = min(r < 0 ? -1 - r : r, in.ny - 1);
  const size_t base = (size_t)gj * in.nx + gi;
#pragma unroll
  for (int p = 0; p < NPLU; ++p) {
    const double v = U[p * in.plane + base + (p % 3 == 0 ? 0 : moff)];
    const bool neg = r < 0 && ((p / 3 == 2) ? (p % 3 != 2) : (p % 3 == 2));
    const double ahead = p % 3 == 0 ? qpre[p / 3] : 0.0, back = p % 3 == 0 ? qpost[p / 3] : 0.0;
    reg[p] = post ? back : top ? ahead : neg ? -v : v;
  }
}

// b - a in doubles for two arrays of doubles that may be separate allocations
// (integer addresses: a pointer difference is defined only within one array;
// both are 8-byte aligned, so the byte difference shifts exactly)
__device__ __forceinline__ long long elem_offset(const double* a, const double* b) {
  return ((long long)(uintptr_t)b - (long long)(uintptr_t)a) >> 3;
}

// Row r of the state U; its moment planes (m = 1, 2) lie moff elements after
// the places U's own would have (0: a plain state).  DMR: the instance uses the
// double Mach reflection boundaries (a separate instantiation, so the plain
// kernels carry none of its registers)
template <int NPLU, bool DMR>
__device__ __forceinline__ void fetch_row(const double* __restrict__ U, const Inst& in, int i0, int r,
                                          int lane, double (&reg)[NPLU], double tb, long long moff = 0) {
  const int ci = i0 - 2 + lane;
  if constexpr (DMR) {
    if (r < 0 || r >= in.ny || i0 < 2 || i0 + LANES - 2 > in.nx) {
      dmr_cells<NPLU>(U, in, r, ci, tb, reg, moff);
      return;
    }
  }
  const int gj = ghost(r, in.ny, in.bcy);
  const int gi = ghost(ci, in.nx, in.bcx);
  const size_t base = (size_t)gj * in.nx + gi;
#pragma unroll
  for (int p = 0; p < NPLU; ++p) reg[p] = U[p * in.plane + base + (p % 3 == 0 ? 0 : moff)];
}

// Row gj of the state U, columns i0 - 2 .. i0 + 61 (ghost columns mapped), straight
// into LDS at dst (NPLU planes of 64 values), past the vector registers, which are
// what the stage kernel is short of.  Asynchronous: dma_wait() before its data is
// read, dma_reads_done() before it may overwrite what was read.  A strip with
// rows_aligned() moves 16 bytes per lane, two planes with one instruction (6 for the 12
// planes of the Euler equations; pc: pair_column()); the others take 4 bytes per lane,
// which any width and column map allows (24 instructions).
using GlobalWord = const __attribute__((address_space(1))) unsigned;
using LdsWord = __attribute__((address_space(3))) unsigned;

// Both waits are explicit.  The compiler's own tracking takes an instruction's LDS
// target for the bytes of one lane and would let reads of other lanes' data pass.
// (A wave waits for itself: a workgroup is one wave.)
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void dma_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// whether the rows of every plane of U can be loaded 16 bytes a lane in this strip: rows
// that start on 16 bytes, and ghost columns, if any, that are periodic images (i0 and nx
// are even, so that a pair of columns has adjacent images)
__device__ __forceinline__ bool rows_aligned(const double* U, const Inst& in, int i0) {
  return ((i0 >= 2 && i0 + LANES - 2 <= in.nx) || in.bcx == 0) &&
         (((uintptr_t)U | (uintptr_t)(8 * (size_t)in.nx)) & 15) == 0;
}
// the column of this lane's pair of such a row
__device__ __forceinline__ int pair_column(const Inst& in, int i0, int lane) {
  return ghost(i0 - 2 + 2 * (lane & 31), in.nx, in.bcx);
}

template <int NPLU>
__device__ __forceinline__ void dma_row(const double* __restrict__ U, const Inst& in, size_t plane, int i0, int gj,
                                        int lane, double* dst, bool aligned, int pc) {
  LdsWord* l = (LdsWord*)dst;
  if (aligned) {
    const double* row = U + (size_t)gj * in.nx + ((lane >> 5) * plane + pc);
#pragma unroll
    for (int p = 0; p < NPLU; p += 2) {
      if (p + 1 < NPLU || lane < 32)
        __builtin_amdgcn_global_load_lds((GlobalWord*)row, l + p * 2 * LANES, 16, 0, 0);
      row += 2 * plane;
    }
  } else {
    const double* row = U + (size_t)gj * in.nx;
    const int c0 = i0 - 2 + (lane >> 1);
    GlobalWord* g0 = (GlobalWord*)(row + ghost(c0, in.nx, in.bcx)) + (lane & 1);
    GlobalWord* g1 = (GlobalWord*)(row + ghost(c0 + LANES / 2, in.nx, in.bcx)) + (lane & 1);
#pragma unroll
    for (int p = 0; p < NPLU; ++p) {
      __builtin_amdgcn_global_load_lds(g0, l + p * 2 * LANES, 4, 0, 0);
      __builtin_amdgcn_global_load_lds(g1, l + p * 2 * LANES + LANES, 4, 0, 0);
      g0 += 2 * plane;
      g1 += 2 * plane;
    }
  }
}

// The same for a state whose moment planes lie moff elements after the places that U's
// own would have (aligned: moff even too)
template <int NPLU>
__device__ __forceinline__ void dma_row_split(const double* __restrict__ U, long long moff, const Inst& in, int i0,
                                              int gj, int lane, double* dst, bool aligned, int pc) {
  LdsWord* l = (LdsWord*)dst;
  const size_t plane = in.plane;
  auto off = [&](int p) { return (long long)(p * plane) + (p % 3 == 0 ? 0 : moff); };
  if (aligned) {
    const double* row = U + (size_t)gj * in.nx + pc;
#pragma unroll
    for (int p = 0; p < NPLU; p += 2)
      if (p + 1 < NPLU || lane < 32)
        __builtin_amdgcn_global_load_lds((GlobalWord*)(row + (lane < 32 ? off(p) : off(p + 1))), l + p * 2 * LANES, 16,
                                         0, 0);
  } else {
    const double* row = U + (size_t)gj * in.nx;
    const int c0 = i0 - 2 + (lane >> 1);
    GlobalWord* g0 = (GlobalWord*)(row + ghost(c0, in.nx, in.bcx)) + (lane & 1);
    GlobalWord* g1 = (GlobalWord*)(row + ghost(c0 + LANES / 2, in.nx, in.bcx)) + (lane & 1);
#pragma unroll
    for (int p = 0; p < NPLU; ++p) {
      __builtin_amdgcn_global_load_lds(g0 + 2 * off(p), l + p * 2 * LANES, 4, 0, 0);
      __builtin_amdgcn_global_load_lds(g1 + 2 * off(p), l + p * 2 * LANES + LANES, 4, 0, 0);
    }
  }
}

template <int NPLU, int SLOTS>
__device__ __forceinline__ void store_row(Window<NPLU, SLOTS>& W, int slot, int lane, const double (&reg)[NPLU]) {
#pragma unroll
  for (int p = 0; p < NPLU; ++p) W.at(slot, p, lane) = reg[p];
}

// stencil of component c around LDS column col
template <int K, class WIN>
__device__ __forceinline__ void gather(const WIN& W, int c, int col, int sl, int sm, int sh,
                                       double (&u0)[9], double (&u1)[9], double (&u2)[9]) {
  const int sr[3] = {sl, sm, sh};
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int l = b * 3 + a;
      u0[l] = W.at(sr[b], c * 3 + 0, col + a - 1);
      const bool x_used = (K >= 5) ? (l != 1 && l != 7) : (l == 4);
      const bool y_used = (K >= 5) ? (l != 3 && l != 5) : (l == 4);
      u1[l] = x_used ? W.at(sr[b], c * 3 + 1, col + a - 1) : 0.0;
      u2[l] = y_used ? W.at(sr[b], c * 3 + 2, col + a - 1) : 0.0;
    }
}

// neighbour-lane values by DPP whole-wave shifts (GFX9 wave_shr:1 / wave_shl:1):
// from_left(x) in lane l is x of lane l - 1, from_right(x) is x of lane l + 1;
// lane 0 (resp. 63) keeps its own value
__device__ __forceinline__ double from_left(double x) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(x), __double2loint(x), 0x138, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(x), __double2hiint(x), 0x138, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double from_right(double x) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(x), __double2loint(x), 0x130, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(x), __double2hiint(x), 0x130, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

}  // namespace fam
