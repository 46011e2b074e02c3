// fam_kernels2d.hip - the 2D kernels of one mesh (tiles in fam_tiles2d.h): stage and OE
// launches, the limiter's tile order and segment list, reductions over the averages.
#include "fam_tiles2d.h"

namespace fam {

template <int K, class P, bool PP, bool DMR, bool CHAR = false>
__global__ void FAM_STAGE_ATTR(K, CHAR) stage2d_kernel(StageArgs A, Inst in, int H) {
  FAM_STAGE_SHARED(K, P::NC, CHAR);
  if (*A.done) return;
  const P phys = make_phys<P>(A.phys);
  double amx = 0.0, amy = 0.0;
  bool bad = false;
  int i0, j0, tile = 0;
  if constexpr (PP) {
    // 1D grid: tiles in the order of the previous launch's limiter work, if any
    const int strips = (in.nx + STRIP - 1) / STRIP;
    // tiles with limiter work first (spread over the XCDs in turn), then the
    // others in the XCD-aware order of their row-major index
    const int N = gridDim.x;
    tile = A.tile_perm
               ? __builtin_amdgcn_readfirstlane(A.tile_perm[heavy_first_slot(blockIdx.x, N, A.tile_perm[N])])
               : xcd_tile(blockIdx.x, N);
    i0 = (tile % strips) * STRIP;
    j0 = (tile / strips) * H;
    S.nwork = 0;
  } else {
    const int T = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    i0 = (T % gridDim.x) * STRIP;
    j0 = (T / gridDim.x) * H;
  }
  stage_tile<K, P, PP, DMR, CHAR>(phys, A, in, i0, j0, H, S, amx, amy, bad);
  flush_wave_results(amx, amy, bad, in.alpha_out, A.flag);
  if constexpr (PP) {
    if (threadIdx.x == 0 && A.tile_perm) A.tile_work[tile] = S.nwork;
  }
}

// tile_perm := tiles with tile_work > 0 first, then the others, each group in
// index order (one block; each thread owns a contiguous chunk)
__global__ void __launch_bounds__(1024) tile_order_kernel(const int* __restrict__ work, int* __restrict__ perm,
                                                          int n) {
  __shared__ int cnt[1024];
  const int t = threadIdx.x, nt = blockDim.x;
  const int per = (n + nt - 1) / nt;
  const int lo = min(n, t * per), hi = min(n, lo + per);
  int heavy = 0;
  for (int k = lo; k < hi; ++k) heavy += work[k] > 0;
  cnt[t] = heavy;
  __syncthreads();
  // inclusive scan of the per-thread counts (Hillis-Steele)
  for (int off = 1; off < nt; off <<= 1) {
    const int v = t >= off ? cnt[t - off] : 0;
    __syncthreads();
    cnt[t] += v;
    __syncthreads();
  }
  const int total = cnt[nt - 1];
  if (t == 0) perm[n] = total;         // heavy tiles: read by the stage kernel
  int h = cnt[t] - heavy;              // heavy tiles before this chunk
  int l = total + (lo - h);            // light tiles go after all heavy ones
  for (int k = lo; k < hi; ++k) {
    if (work[k] > 0) perm[h++] = k;
    else perm[l++] = k;
  }
}

void launch_tile_order(const int* tile_work, int* tile_perm, int ntiles, hipStream_t s) {
  hipLaunchKernelGGL(tile_order_kernel, dim3(1), dim3(1024), 0, s, tile_work, tile_perm, ntiles);
}

__global__ void tile_identity_kernel(int* __restrict__ perm, int* __restrict__ work, int n) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k <= n; k += gridDim.x * blockDim.x) {
    perm[k] = k < n ? k : 0;   // perm[n]: no tile with limiter work yet
    if (k < n) work[k] = 0;
  }
}

template <int K, class P, bool DMR, bool CHAR = false>
__global__ void FAM_STAGE_ATTR(K, CHAR) stage2d_list_kernel(StageArgs A, Inst in, const int4* __restrict__ seg,
                                                    const int* __restrict__ nseg) {
  FAM_STAGE_SHARED(K, P::NC, CHAR);
  if (*A.done) return;
  const int n = *nseg;
  if ((int)blockIdx.x >= n) return;
  // the list is ordered by row band: each XCD takes a contiguous share
  const int4 it = seg[xcd_tile(blockIdx.x, n)];
  if (it.w <= 0) return;
  const P phys = make_phys<P>(A.phys);
  double amx = 0.0, amy = 0.0;
  bool bad = false;
  S.nwork = 0;
  stage_tile<K, P, true, DMR, CHAR>(phys, A, in, it.y, it.z, it.w, S, amx, amy, bad);
  flush_wave_results(amx, amy, bad, in.alpha_out, A.flag);
}

// Segment list for the next limiter-on launch.  Each strip's rows are cut into
// n_s segments of equal recorded cost; n_s = ceil(C_s / (tau - R)) with C_s the
// strip's cost, R the cost of a segment's three extra ring rows (three mean
// rows) and tau the smallest per-segment bound (bisection) for which the
// segments fit the budget (one wave slot each).  Two launches:
//   part_scan_kernel (one block per strip): inclusive prefix sums of the row
//     costs and C_s;
//   part_cut_kernel (one block per strip): every block repeats the bisection
//     (same inputs, same operations, same result), takes its strip's n_s and
//     first list index, and starts segment k at the first row whose inclusive
//     prefix exceeds k C_s / n_s.
constexpr int PART_T = 1024;

// strip costs of the partition (device)
struct PartState {
  float Cs[PART_MAX_STRIPS];
};

__global__ void __launch_bounds__(PART_T) part_scan_kernel(const float* __restrict__ cost, float* __restrict__ pref,
                                                          int ny, PartState* __restrict__ ps) {
  __shared__ float sh[PART_T / 64];
  const int t = threadIdx.x, s = blockIdx.x, lane = t & 63, wv = t >> 6;
  const float* __restrict__ C = cost + (size_t)s * ny;
  float* __restrict__ P = pref + (size_t)s * ny;
  // thread t owns rows [t * per, (t + 1) * per)
  const int per = (ny + PART_T - 1) / PART_T;
  const int r0 = min(ny, t * per), r1 = min(ny, r0 + per);
  float own = 0.0f;
  for (int r = r0; r < r1; ++r) own += C[r];
  // inclusive scan of the thread sums: waves, then the wave totals
  float v = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const float u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  if (lane == 63) sh[wv] = v;
  __syncthreads();
  if (wv == 0) {
    float w = lane < PART_T / 64 ? sh[lane] : 0.0f;
#pragma unroll
    for (int off = 1; off < PART_T / 64; off <<= 1) {
      const float u = __shfl_up(w, off);
      if (lane >= off) w += u;
    }
    if (lane < PART_T / 64) sh[lane] = w;
  }
  __syncthreads();
  const float incl = v + (wv > 0 ? sh[wv - 1] : 0.0f);
  float run = incl - own;
  for (int r = r0; r < r1; ++r) {
    run += C[r];
    P[r] = run;
  }
  if (t == PART_T - 1) ps->Cs[s] = incl;
}

// Segment counts of all strips for the bound tau (lane-strided over the strips,
// summed across the wave): every lane returns the same total.
__device__ __forceinline__ int part_count(const float* sC, int strips, int budget, float R, float tau, int lane) {
  const float inv = 1.0f / (tau - R);
  int c = 0;
  for (int q = lane; q < strips; q += 64) {
    const float x = sC[q] * inv;
    c += x > (float)budget ? budget + 1 : max(1, (int)ceilf(x));
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) c += __shfl_xor(c, m);
  return c;
}

constexpr int PART_CUT_T = 256;
constexpr int PART_LDS_ROWS = 8192;   // strips up to this height search an LDS copy

__global__ void __launch_bounds__(PART_CUT_T) part_cut_kernel(const float* __restrict__ pref, int strips, int ny,
                                                              int budget, const PartState* __restrict__ ps,
                                                              int4* __restrict__ seg, int* __restrict__ nseg) {
  __shared__ float sC[PART_MAX_STRIPS];
  __shared__ int sn[PART_MAX_STRIPS];   // segments per strip
  __shared__ float sp[PART_LDS_ROWS];
  __shared__ int s_all;
  __shared__ float s_Cs;
  const int t = threadIdx.x, s = blockIdx.x, lane = t & 63;
  const float* __restrict__ P = pref + (size_t)s * ny;
  const bool in_lds = ny <= PART_LDS_ROWS;
  if (in_lds)
    for (int r = t; r < ny; r += PART_CUT_T) sp[r] = P[r];
  for (int q = t; q < strips; q += PART_CUT_T) sC[q] = ps->Cs[q];
  __syncthreads();
  if (t < 64) {
    // every block repeats the same bisection (same inputs, same operations)
    float total = 0.0f, cmax = 0.0f;
    for (int q = lane; q < strips; q += 64) {
      total += sC[q];
      cmax = fmaxf(cmax, sC[q]);
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {   // butterfly: every lane ends with the same sums
      total += __shfl_xor(total, m);
      cmax = fmaxf(cmax, __shfl_xor(cmax, m));
    }
    const float R = 3.0f * total / ((float)strips * (float)ny);
    // lo: below any fit (fewer than budget segments cannot hold the total).
    // hi: a bound that fits -- total / (budget - strips) + R fits in exact
    // arithmetic (the ceilings add at most one per strip); if rounding spoils
    // it, one segment per strip (strips <= budget) always fits.
    float lo = total / (float)budget, hi = 2.0f * cmax + R + 1.0f;
    if (strips < budget) {
      const float h1 = 1.001f * total / (float)(budget - strips) + R;
      if (h1 < hi && part_count(sC, strips, budget, R, h1, lane) <= budget) hi = h1;
    }
    for (int it = 0; it < 14; ++it) {
      const float tau = 0.5f * (lo + hi);
      const bool fits = tau > R && part_count(sC, strips, budget, R, tau, lane) <= budget;
      if (fits) hi = tau;
      else lo = tau;
    }
    // every strip's count (<= budget at a bound that fits) and their sum
    const float inv = 1.0f / (hi - R);
    int all = 0;
    for (int q = lane; q < strips; q += 64) {
      const int n = max(1, (int)ceilf(sC[q] * inv));
      sn[q] = n;
      all += n;
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) all += __shfl_xor(all, m);
    if (lane == 0) {
      s_all = all;
      s_Cs = sC[s];
    }
  }
  __syncthreads();
  const int n = sn[s];
  const float Cs = s_Cs;
  if (s == 0 && t == 0) *nseg = s_all;
  for (int k = t; k < n; k += PART_CUT_T) {
    // list position: segments ordered by their index within the strip, then by
    // strip (the k-th segments of all strips cover similar rows, so each XCD's
    // contiguous share of the list is a band of rows across the strips)
    int pos = 0;
    for (int q = 0; q < strips; ++q) pos += min(sn[q], k) + (q < s && sn[q] > k ? 1 : 0);
    int st[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int kk = k + e;
      if (kk == 0) { st[e] = 0; continue; }
      if (kk == n) { st[e] = ny; continue; }
      const float target = Cs * (float)kk / (float)n;
      int x = 0, y = ny;   // first row with P > target
      while (x < y) {
        const int m = (x + y) >> 1;
        if ((in_lds ? sp[m] : P[m]) <= target) x = m + 1;
        else y = m;
      }
      st[e] = x;
    }
    seg[pos] = make_int4(0, s * STRIP, st[0], st[1] - st[0]);
  }
}

__global__ void fill_kernel(float* __restrict__ p, float v, size_t n) {
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) p[k] = v;
}

template <int K, class P, bool DMR, int SLOTS>
__global__ void FAM_OE_ATTR oe2d_kernel(OEArgs A, Inst in, int H) {
  __shared__ Window<3 * P::NC, SLOTS> W;
  __shared__ double t1s[8];
  if (*A.done) return;
  const P phys = make_phys<P>(A.phys);
  bool bad = false;
  const int T = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int i0 = (T % gridDim.x) * STRIP, j0 = (T / gridDim.x) * H;
  if (K == 6 && A.k6_table)
    oe_tile<K, P, true, DMR, SLOTS>(phys, A, in, i0, j0, H, W, t1s, bad);
  else
    oe_tile<K, P, false, DMR, SLOTS>(phys, A, in, i0, j0, H, W, t1s, bad);
  if (__any(bad) && threadIdx.x == 0) atomicOr(A.flag, 1);
}

// ---------------------------------------------------------------------------
// reductions over cell averages
// ---------------------------------------------------------------------------
// alpha_out[inst] = max over cells of the spectral radii at the averages.  SPREAD (one
// mesh): every wave adds to one of the slots; a batch: every block to the one there is,
// which takes 24 ns a block, so a mesh has up to 256 blocks (a single step of 40 meshes
// of 64^2 to 512^2, us with 256 / 512 / 1024: 1155 / 1170 / 1198; two of 2000^2 2461 /
// 2459 / 2475).
template <class P, bool SPREAD>
__global__ void __launch_bounds__(256) alpha2d_kernel(PhysParams pp, const double* __restrict__ U,
                                                      const Inst* __restrict__ insts, int ninst, int* flag) {
  const P phys = make_phys<P>(pp);
  constexpr int NC = P::NC;
  bool bad = false;
  for (int inst = blockIdx.y; inst < ninst; inst += gridDim.y) {
    const Inst in = insts[inst];
    const size_t n = (size_t)in.nx * in.ny;
    if ((size_t)blockIdx.x * blockDim.x >= n) continue;
    double mx = 0.0, my = 0.0;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
      double avg[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) avg[c] = U[in.offset + (c * 3) * in.plane + idx];
      mx = fmax(mx, phys.speed(0, avg, bad));
      my = fmax(my, phys.speed(1, avg, bad));
    }
    mx = wave_max(mx);
    my = wave_max(my);
    if constexpr (SPREAD) {
      if ((threadIdx.x & 63) == 0) {
        double* slot = alpha_slot(in.alpha_out, blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64);
        atomic_max_nonneg(&slot[0], mx);
        atomic_max_nonneg(&slot[1], my);
      }
    } else {
      __shared__ double2 red[4];
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_double2(mx, my);
      __syncthreads();
      if (threadIdx.x == 0) {
        atomic_max_nonneg(&in.alpha_out[0], fmax(fmax(red[0].x, red[1].x), fmax(red[2].x, red[3].x)));
        atomic_max_nonneg(&in.alpha_out[1], fmax(fmax(red[0].y, red[1].y), fmax(red[2].y, red[3].y)));
      }
      __syncthreads();
    }
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// Type I statistics, pass 1: per-block partial sums and max |u| of each component
__global__ void __launch_bounds__(256) type1_pass1_kernel(const double* __restrict__ U, Inst in, int nc,
                                                          int nmom, double* __restrict__ partial) {
  __shared__ double red[4][4];
  const size_t n = (size_t)in.nx * in.ny;
  for (int c = 0; c < nc; ++c) {
    double s = 0.0;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x)
      s += U[in.offset + (c * nmom) * in.plane + idx];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = s;
  }
  __syncthreads();
  if ((int)threadIdx.x < nc) {
    const int c = threadIdx.x;
    partial[blockIdx.x * 4 + c] = ((red[c][0] + red[c][1]) + red[c][2]) + red[c][3];
  }
}

// Pass 2: every wave adds the partial sums to the mean (the same order in each), then
// per block max |u - mean| and max |u|.  The OE kernels take the largest over the
// blocks.  700x555, one component: both passes 9.6 us, against 62.9 us with the mean
// added by one thread (28), the maxima by atomics on one address (25) and a launch
// that read them back (5).
__global__ void __launch_bounds__(256) type1_pass2_kernel(const double* __restrict__ U, Inst in, int nc,
                                                          int nmom, const double* __restrict__ partial,
                                                          double2* __restrict__ stats) {
  __shared__ double2 red[4][4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const size_t n = (size_t)in.nx * in.ny;
  for (int c = 0; c < nc; ++c) {
    double s = 0.0;
    for (int b = lane; b < (int)gridDim.x; b += 64) s += partial[b * 4 + c];
    const double mu = wave_sum(s) / ((double)in.nx * in.ny);
    double d = 0.0, a = 0.0;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
      const double v = U[in.offset + (c * nmom) * in.plane + idx];
      d = fmax(d, fabs(v - mu));
      a = fmax(a, fabs(v));
    }
    d = wave_max(d);
    a = wave_max(a);
    if (lane == 0) red[c][wv] = make_double2(d, a);
  }
  __syncthreads();
  if ((int)threadIdx.x < nc) {
    const double2* r = red[threadIdx.x];
    stats[blockIdx.x * 4 + threadIdx.x] = make_double2(fmax(fmax(r[0].x, r[1].x), fmax(r[2].x, r[3].x)),
                                                       fmax(fmax(r[0].y, r[1].y), fmax(r[2].y, r[3].y)));
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// the double Mach reflection boundaries are an Euler 2D option; other systems
// compile only the plain instantiation
template <class P>
static bool dmr_of(const Inst& in) {
  if constexpr (std::is_same_v<P, Euler<2>>)
    return in.dmr != 0;
  else
    return false;
}
template <int K, class P, bool DMR, bool CHAR = false>
static void launch_stage2d_d(StageArgs A, const Inst& in, int H, hipStream_t s) {
  dim3 grid((in.nx + STRIP - 1) / STRIP, (in.ny + H - 1) / H);
  if (A.pp) {
    const int ntiles = grid.x * grid.y;
    if (starts_at_once(ntiles, ntiles, stage_waves(K, P::NC, CHAR))) A.tile_perm = nullptr;
    hipLaunchKernelGGL((stage2d_kernel<K, P, true, DMR, CHAR>), dim3(ntiles), dim3(LANES), 0, s, A, in, H);
    if (A.tile_perm) launch_tile_order(A.tile_work, const_cast<int*>(A.tile_perm), ntiles, s);
  } else {
    hipLaunchKernelGGL((stage2d_kernel<K, P, false, DMR, CHAR>), grid, dim3(LANES), 0, s, A, in, H);
  }
}
template <int K, class P>
static void launch_stage2d_t(const StageArgs& A, const Inst& in, int H, hipStream_t s) {
  if constexpr (std::is_same_v<P, Euler<2>>) {
    // characteristic variables: FAM5 only (the variant the paper times)
    if constexpr (K == 5) {
      if (in.charv) {
        if (dmr_of<P>(in)) return launch_stage2d_d<K, P, true, true>(A, in, H, s);
        return launch_stage2d_d<K, P, false, true>(A, in, H, s);
      }
    }
    if (dmr_of<P>(in)) return launch_stage2d_d<K, P, true>(A, in, H, s);
  }
  launch_stage2d_d<K, P, false>(A, in, H, s);
}
template <int K, class P>
static void launch_oe2d_t(const OEArgs& A, const Inst& in, int H, hipStream_t s) {
  dim3 grid((in.nx + STRIP - 1) / STRIP, (in.ny + H - 1) / H);
  if constexpr (std::is_same_v<P, Euler<2>>) {
    if (dmr_of<P>(in)) {
      hipLaunchKernelGGL((oe2d_kernel<K, P, true, 3>), grid, dim3(LANES), 0, s, A, in, H);
      return;
    }
    if (grid.x * grid.y > SIMDS) {
      hipLaunchKernelGGL((oe2d_kernel<K, P, false, 3>), grid, dim3(LANES), 0, s, A, in, H);
      return;
    }
  }
  hipLaunchKernelGGL((oe2d_kernel<K, P, false, 4>), grid, dim3(LANES), 0, s, A, in, H);
}
void launch_stage2d(int k, int sys, const StageArgs& A, const Inst& in, int H, hipStream_t s) {
  FAM_DISPATCH_P(sys, FAM_DISPATCH_K(k, (launch_stage2d_t<KK, PP>(A, in, H, s))));
}
template <int K, class P>
static void launch_stage2d_list_t(const StageArgs& A, const Inst& in, const int4* seg, const int* nseg, int budget,
                                  hipStream_t s) {
  if constexpr (std::is_same_v<P, Euler<2>> && K == 5) {
    if (in.charv) {
      if (dmr_of<P>(in))
        hipLaunchKernelGGL((stage2d_list_kernel<K, P, true, true>), dim3(budget), dim3(LANES), 0, s, A, in, seg,
                           nseg);
      else
        hipLaunchKernelGGL((stage2d_list_kernel<K, P, false, true>), dim3(budget), dim3(LANES), 0, s, A, in, seg,
                           nseg);
      return;
    }
  }
  if constexpr (std::is_same_v<P, Euler<2>>) {
    if (dmr_of<P>(in)) {
      hipLaunchKernelGGL((stage2d_list_kernel<K, P, true>), dim3(budget), dim3(LANES), 0, s, A, in, seg, nseg);
      return;
    }
  }
  hipLaunchKernelGGL((stage2d_list_kernel<K, P, false>), dim3(budget), dim3(LANES), 0, s, A, in, seg, nseg);
}
void launch_stage2d_list(int k, int sys, const StageArgs& A, const Inst& in, const int4* seg, const int* nseg,
                         int budget, hipStream_t s) {
  // the limiter is a 2D Euler option
  (void)sys;
  switch (k) {
    case 3: launch_stage2d_list_t<3, Euler<2>>(A, in, seg, nseg, budget, s); break;
    case 4: launch_stage2d_list_t<4, Euler<2>>(A, in, seg, nseg, budget, s); break;
    case 5: launch_stage2d_list_t<5, Euler<2>>(A, in, seg, nseg, budget, s); break;
    default: launch_stage2d_list_t<6, Euler<2>>(A, in, seg, nseg, budget, s); break;
  }
}
size_t partition_state_bytes() { return sizeof(PartState); }
void launch_partition(const float* row_cost, float* pref, void* state, int strips, int ny, int budget, int4* seg,
                      int* nseg, hipStream_t s) {
  PartState* ps = static_cast<PartState*>(state);
  hipLaunchKernelGGL(part_scan_kernel, dim3(strips), dim3(PART_T), 0, s, row_cost, pref, ny, ps);
  hipLaunchKernelGGL(part_cut_kernel, dim3(strips), dim3(PART_CUT_T), 0, s, pref, strips, ny, budget, ps, seg, nseg);
}
void launch_fill(float* p, float v, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)std::min<size_t>(1024, (n + 255) / 256)), dim3(256), 0, s, p, v, n);
}
void launch_tile_identity(int* tile_perm, int* tile_work, int ntiles, hipStream_t s) {
  hipLaunchKernelGGL(tile_identity_kernel, dim3(std::min(1024, (ntiles + 255) / 256)), dim3(256), 0, s, tile_perm,
                     tile_work, ntiles);
}
void launch_oe2d(int k, int sys, const OEArgs& A, const Inst& in, int H, hipStream_t s) {
  FAM_DISPATCH_P(sys, FAM_DISPATCH_K(k, (launch_oe2d_t<KK, PP>(A, in, H, s))));
}
void launch_alpha2d(int sys, const PhysParams& pp, const double* U, const Inst* insts, int ninst,
                    size_t max_cells, int* flag, hipStream_t s) {
  const int bx = (int)std::min<size_t>((max_cells + 255) / 256, ninst == 1 ? 1024 : 256);
  const dim3 grid(bx < 1 ? 1 : bx, std::min(ninst, 65535));
  if (ninst == 1) {
    FAM_DISPATCH_P(sys, hipLaunchKernelGGL((alpha2d_kernel<PP, true>), grid, dim3(256), 0, s, pp, U, insts, ninst, flag));
  } else {
    FAM_DISPATCH_P(sys, hipLaunchKernelGGL((alpha2d_kernel<PP, false>), grid, dim3(256), 0, s, pp, U, insts, ninst, flag));
  }
}
void launch_type1_stats(const double* U, const Inst& in, int nc, int nmom, double* partial, double2* stats,
                        hipStream_t s) {
  const int nb = type1_blocks((size_t)in.nx * in.ny);
  hipLaunchKernelGGL(type1_pass1_kernel, dim3(nb), dim3(256), 0, s, U, in, nc, nmom, partial);
  hipLaunchKernelGGL(type1_pass2_kernel, dim3(nb), dim3(256), 0, s, U, in, nc, nmom, partial, stats);
}

}  // namespace fam
