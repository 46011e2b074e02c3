// fam_kernels.h - argument blocks and launchers shared by the host library and
// the HIP kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include <algorithm>

namespace fam {

constexpr int STRIP = 60;   // output columns per 2D strip (one wavefront)
// waves of the RK stage kernel per SIMD that its registers and LDS allow (order k,
// nc components, reconstruction in characteristic variables)
__host__ __device__ constexpr int stage_waves(int k, int nc, bool charv) {
  return nc == 1 ? 4 : (k >= 6 || charv) ? 1 : 2;
}

constexpr int SIMDS = 1024;   // 256 CUs x 4

// Whether the tiles (or work-list items) of a launch all start at once: a workgroup of
// one wave each, and a wave slot for every workgroup.  Then their order does not matter
// and is not renewed (6 us; six meshes 5 % faster).  A grid of fewer workgroups than
// items takes them in turns, in that order.
inline bool starts_at_once(int nblocks, int nitems, int waves) {
  return nblocks == nitems && nitems <= SIMDS * waves;
}

// Rows per strip tile from a model of a launch of tiles(H) waves.  A tile of H rows
// costs H + 2 row times (it also reconstructs a ring row on either side); w waves
// on a SIMD take 1 + share (w - 1) times as long as one, up to `waves` of them,
// and further tiles follow in rounds.  On small meshes the rows' latency decides:
// one-row tiles on every SIMD; from about a million cells it is the ring rows and
// the last round.  Measured (us a stage launch at the model's height / with 8 rows):
// 40x40 k=4 10.7 / 37.6; 96x80 k=5, limiter 23.5 / 64.8; 203x131 k=5 14.3 / 47.6;
// 256x256 k=6 22.8 / 58.2; 512x512 k=5 37.7 / 52.2 (5 rows); 700x700 k=5 56.9 / 79.8
// (5 rows); 1024x1024 k=5 110.7 / 129.9 (10 rows); 1201x1000 k=6 167.5 / 180.9 (24).
template <class F>
inline int model_rows(F tiles, int ny, int waves, double share) {
  int best = 1;
  double least = 1e300;
  for (int H = 1; H <= std::min(ny, 128); ++H) {
    const long long w = ((long long)tiles(H) + SIMDS - 1) / SIMDS;   // waves of the fullest SIMD
    const long long rounds = w / waves, rest = w % waves;
    const double cost =
        (H + 2) * ((double)rounds * (1.0 + share * (waves - 1)) + (rest > 0 ? 1.0 + share * (rest - 1) : 0.0));
    if (cost < least) {
      least = cost;
      best = H;
    }
  }
  return best;
}

// The slowdown of a further wave on a SIMD, from launches of 1, 2, 3 ... waves on
// each (512x512 and 700x555, 1 to 32 rows): stage 0.45 with two waves of nc = 4, 0.3
// with four of nc = 1; OE kernel 0.3
inline int stage_rows(int nx, int ny, int k, int nc, bool charv) {
  const int strips = (nx + STRIP - 1) / STRIP;
  return model_rows([&](int H) { return (long long)strips * ((ny + H - 1) / H); }, ny, stage_waves(k, nc, charv),
                    nc == 1 ? 0.3 : 0.45);
}
inline int oe_rows(int nx, int ny, int nc) {
  const int strips = (nx + STRIP - 1) / STRIP;
  return model_rows([&](int H) { return (long long)strips * ((ny + H - 1) / H); }, ny, nc == 1 ? 4 : 2, 0.3);
}

struct PhysParams {
  double gamma, ax, ay;
};

// one mesh instance (a batched context holds many)
struct Inst {
  int id;
  int nx, ny;
  size_t plane;            // nx * ny
  size_t offset;           // start of the instance in a batched state (doubles)
  double dx, dy;
  int bcx, bcy;            // 0 periodic, 1 transmissive
  const double* alpha_in;  // a set: wave speeds of the stage input state
  double* alpha_out;       // a set: max-accumulators for the stage output state
  const double* dt;        // time step of the current step
  const int* done;         // instance finished (fam_run), may be null
  // double Mach reflection boundaries (dmr != 0): the boundary time of a launch is
  // *t_end - t_ofs * dt (t_end: the step's end time; t_ofs 1, 0, 1/2 for the RK
  // stages, 0 for OE); x0, ytop: domain; dmr_einv = 1 / (gamma - 1)
  int dmr;
  const double* t_end;
  double t_ofs;
  double x0, ytop, dmr_einv;
  // stage reconstruction in local characteristic variables (Euler, k = 5)
  int charv;
};

struct StageArgs {
  PhysParams phys;
  const double* Us;
  const double* U0;
  double* Uout;
  // moment planes (m = 1, 2) of the output; NULL: those of Uout.  With Uout the
  // state and Uout_mom a stage buffer, the last stage of a step writes its
  // averages in place (each output cell reads only its own U0 value) and leaves
  // its moments for the OE, which then writes only moment planes
  double* Uout_mom;
  // Shu-Osher stage ca U0 + (1 - ca) L with L = Us + dt R(Us), evaluated as
  // L + ca (U0 - L): the rounded 1/3 and 2/3 of the last stage sum to 1 - 2^-54,
  // which as separate weights would shrink every value by that much each step
  double ca;
  int* flag;
  const int* done;
  int pp;                  // positivity limiter on the stage reconstruction (2D Euler)
  // single-instance limiter launches: tiles run in the order tile_perm (cells
  // that needed the exact test in the previous launch first); each tile writes
  // its count of such cells to tile_work
  const int* tile_perm;
  int* tile_work;
  // single-instance limiter launches over a segment list: the cost of each row of
  // each strip in rows without limiter work, row_cost[strip * ny + row] (NULL: not
  // recorded)
  float* row_cost;
};

struct OEArgs {
  PhysParams phys;
  const double* Un;
  // average planes (m = 0) of the input; NULL: those of Un.  When they are
  // Uout's own (avg_in_place = 1) the OE leaves them unwritten: it changes no
  // average, so it then moves 8 planes per cell to HBM instead of 12
  const double* Ua;
  int avg_in_place;
  double* Uout;
  double gamma_k;
  int type;                // 1 or 2
  int k6_table;
  const double2* stats;    // Type I: [block*4 + c] of type1_blocks(cells) blocks: max |u - mean|, max |u|
  int* flag;
  const int* done;
  double* delta_out;       // single instance, test export: delta per cell (NULL: not written)
};

// A wave-speed maximum (x, y) is accumulated by atomics in ALPHA_SLOTS slots, one
// cache line apart; its readers take the largest.  Device atomics are executed at
// the memory side, one cache line at a time: a wave's two cost 24 ns on a shared
// pair, which bounded launches of many short waves (1024 waves: 24.5 us, on 32
// slots a line apart 3.0 us of which 2.6 are the launch; 16 slots 3.0, and 4.9
// against 2.9 at 2048 waves; 32 slots packed in 4 lines 6.2).
constexpr int ALPHA_SLOTS = 32;
constexpr int ALPHA_STRIDE = 16;                          // doubles: 128 B
constexpr int ALPHA_SET = ALPHA_SLOTS * ALPHA_STRIDE;     // one maximum (x, y)
// Batches keep one slot per set: their atomics go to as many lines as there are
// instances, and with slots a small instance would hold as much memory for them as for
// its state (16x16 Euler: 24 KB).  An instance has two lines: a launch reads one set and
// accumulates the next, and reads of the line that the atomics go to wait for them (two
// meshes of 2000^2, a step 2960 us with all sets in one line, 2470 with two).
// Offset of set 3 parity + (stage input 0..2) of an instance, and an instance's doubles
__host__ __device__ constexpr size_t alpha_set(bool spread, int set) {
  return spread ? (size_t)set * ALPHA_SET : (set % 2) * ALPHA_STRIDE + (set / 2) * 2;
}
__host__ __device__ constexpr size_t alpha_inst(bool spread) { return spread ? 6 * ALPHA_SET : 2 * ALPHA_STRIDE; }

// per-instance step bookkeeping (device)
struct StepState {
  double* alpha;           // wave-speed maxima: alpha_inst doubles
  double dt;               // time step of the current step
  double t;                // time reached: the context clock (0 at set-up, advanced by every step)
  double t_final;          // <= 0: none
  double dt_fixed;         // > 0: use instead of the CFL rule
  double cfl;
  double hx, hy;           // lengths of the time-step rule: dx, dy or dx^{k/3}, dy^{k/3}
  int dim;
  int done;
  int steps;
  int pad_;
};

void launch_stage2d(int k, int sys, const StageArgs& A, const Inst& in, int H, hipStream_t s);
// tile_perm := tiles with tile_work > 0 first, then the others (both in index order)
void launch_tile_order(const int* tile_work, int* tile_perm, int ntiles, hipStream_t s);
void launch_tile_identity(int* tile_perm, int* tile_work, int ntiles, hipStream_t s);
// limiter-on stage launch over a list of strip segments (x unused, y = first
// column, z = first row, w = rows; w <= 0: empty), one wave per entry; then the
// list for the next launch: each strip cut into segments of equal recorded cost,
// at most `budget` segments in all
void launch_stage2d_list(int k, int sys, const StageArgs& A, const Inst& in, const int4* seg, const int* nseg,
                         int budget, hipStream_t s);
// state: partition_state_bytes() of device memory
size_t partition_state_bytes();
void launch_partition(const float* row_cost, float* pref, void* state, int strips, int ny, int budget, int4* seg,
                      int* nseg, hipStream_t s);
void launch_fill(float* p, float v, size_t n, hipStream_t s);
constexpr int PART_MAX_STRIPS = 1024;
// point values of the stage reconstruction at every cell's flux points (test export)
void launch_dbg_recon(int dim, int k, int nc, const double* U, const Inst& in, double* vals, hipStream_t s);
void launch_oe2d(int k, int sys, const OEArgs& A, const Inst& in, int H, hipStream_t s);
void launch_stage2d_batched(int k, int sys, const StageArgs& A, const Inst* insts, const int4* work, int nwork,
                            int nblocks, hipStream_t s);
void launch_oe2d_batched(int k, int sys, const OEArgs& A, const Inst* insts, const int4* work, int nwork,
                         int nblocks, hipStream_t s);
void launch_alpha2d(int sys, const PhysParams& pp, const double* U, const Inst* insts, int ninst,
                    size_t max_cells, int* flag, hipStream_t s);
// Type I reference quantities of one instance (nmom = moments per component)
// Type I statistics: partial (TYPE1_BLOCKS * 4 sums) and stats (TYPE1_BLOCKS * 4 pairs of maxima) of one entry
// per block and component, which the OE kernels reduce themselves.  256 cells a block up to one block per CU
constexpr int TYPE1_BLOCKS = 256;
__host__ __device__ inline int type1_blocks(size_t cells) {
  return cells >= (size_t)TYPE1_BLOCKS * 256 ? TYPE1_BLOCKS : (int)((cells + 255) / 256);
}
void launch_type1_stats(const double* U, const Inst& in, int nc, int nmom, double* partial, double2* stats,
                        hipStream_t s);

// 1D
void launch_stage1d(int k, int sys, const StageArgs& A, const Inst& in, hipStream_t s);
// largest 1D mesh that runs in one workgroup: a lane per cell and per ghost on either
// side; the 1D Euler kernel needs more than the 128 registers a lane of 1024 may have
__host__ __device__ constexpr int run1d_max(int nc) { return nc == 1 ? 1022 : 510; }
void launch_run1d(int k, int sys, const PhysParams& pp, double* U, const Inst& in, StepState* st, int* flag,
                  int nsteps, int test, bool more, bool fresh, double dt_fixed, double t_final, int oe,
                  double gamma_k, hipStream_t s);
// A run to an end time starts with RUN_FIRST steps; each later chunk holds the steps
// still needed at the last step's dt, at most 64, rounded up to even, so that few steps
// past the end time are no-ops.  After each chunk it tests for non-physical states.
constexpr int RUN_FIRST = 2;
__host__ __device__ inline int run_chunk(double t_left, double dt) {
  const double need = ceil(t_left / dt);
  const int want = need > 62.0 ? 64 : need > 2.0 ? (int)need : 2;
  return want + (want & 1);
}
void launch_oe1d(int k, int sys, const OEArgs& A, const Inst& in, hipStream_t s);
void launch_alpha1d(int sys, const PhysParams& pp, const double* U, const Inst& in, int* flag, hipStream_t s);

// step bookkeeping: dt, clipping, termination, zeroing of the accumulators
void launch_step_begin(StepState* st, int ninst, int parity, double dt_fixed, double t_final, hipStream_t s);
// per run: wave-speed slots, dt, step count and termination back to zero; the
// time (the context clock) is kept
void launch_reset_steps(StepState* st, int ninst, double t_final, double dt_fixed, hipStream_t s);
void launch_set_time(StepState* st, int ninst, double t, hipStream_t s);

}  // namespace fam
