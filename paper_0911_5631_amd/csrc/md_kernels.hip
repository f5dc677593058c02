// md_kernels.hip -- gfx950 kernels of the soft-sphere MD hot path.
//
// A time step k of every replica of an engine is two launches:
//   k_sort  (b) when the displacement rule fires (always with the plain cell
//           method): wrap, and a stable counting sort of the atoms by cell
//           (Secs. 3.4, 3.5) -- cell_start from the occupancy counts, ranks
//           from the cell-layer rows, scatter into the other buffer variant.
//           Replicas that do not rebuild leave at once.
//   k_step  (b) the neighbour matrix W from the contiguous cell ranges of
//           the sorted atoms when rebuilding; (c) forces from W (or from the
//           cells); (d), (e) second half kick, kinetic energy, maximum speed;
//           (a) of the next step: half kick and drift, and the binning of the
//           new positions into the next cell-layer set.
// Nothing waits for other workgroups inside these launches: the rebuild
// decision of step k is recomputed by every workgroup of k_sort from the
// maximum speed of step k-1 (one atomicMax per workgroup into a spread ring
// slot) and the displacement committed by step k-1, and committed for k_step by
// the workgroup of the replica's first cell tile, so no device-scope fence or
// "last block" finalisation is needed (on gfx950 a device-scope release writes
// back the whole L2).
// Replicas whose tiles the chip holds at once take many steps per launch
//   k_run   the same parts in one kernel, with barriers over the replica's
//           workgroups between them.
// Either leaves a replica so that the other can go on with it.  Properties are
// reduced on demand (k_props) in a fixed order.
//
// Floating point: compiled with -ffp-contract=off, so every FP64 expression
// rounds as written (no fused multiply-add); cell indices and neighbour
// decisions are then the ones an FP64 CPU evaluation of the same expressions
// makes.
#include <hip/hip_runtime.h>

#include <limits.h>

#include <type_traits>

#include "md_device.h"
#include "md_kernels.h"

namespace md {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

// Global-address-space view of a pointer read from a descriptor: the loads
// and stores through it are global_* instructions instead of flat_* ones
// (which also count against the LDS wait counter).
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gp(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}
typedef const __attribute__((address_space(1))) double *gcdouble;
typedef const __attribute__((address_space(1))) int32_t *gcint;

// The thread's index, worked out here and not before: what depends on it only
// (lane masks, offsets) would otherwise be hoisted out of the loops over tiles
// and steps, held across them and spilled.
__device__ __forceinline__ int tid_here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  __builtin_assume(t >= 0 && t < TILE);
  return t;
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ bool uniform(bool b) {
  return __builtin_amdgcn_readfirstlane(b ? 1 : 0) != 0;
}
__device__ __forceinline__ double uniform(double v) {
  const long long b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Loads and stores of data that other workgroups of the same launch write or
// read (k_run; COH): device-scope, so they neither stay in nor come from an
// XCD's own L2.  In the other kernels a launch only reads what earlier
// launches wrote, and they are plain.
template <bool COH, class T>
__device__ __forceinline__ T ld(const __attribute__((address_space(1))) T *p) {
  if constexpr (COH) return __hip_atomic_load((const T *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool COH, class T>
__device__ __forceinline__ void st(__attribute__((address_space(1))) T *p, T v) {
  if constexpr (COH)
    __hip_atomic_store((T *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

// Replica descriptors are written by the host only, between launches: read
// through the constant address space their fields are scalar loads held in
// SGPRs (a wave-uniform descriptor) instead of vector loads into VGPRs.
typedef const __attribute__((address_space(4))) SlotDev SlotC;
__device__ __forceinline__ SlotC &slot(const Tables &T, int idx) {
  return *(SlotC *)(T.slots + idx);
}
// The same view of other host-written tables, and of control words that a
// kernel reads while no workgroup of the same launch writes them.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *cview(const T *p) {
  return (const __attribute__((address_space(4))) T *)p;
}

// Workgroups go to the 8 XCDs round-robin; renumber them so that each XCD
// walks a contiguous range of tiles and neighbouring atoms share an L2.
__device__ __forceinline__ int xcd_block(int b, int g) {
  if ((g & 7) == 0) return (b & 7) * (g >> 3) + (b >> 3);
  return b;
}

// The tiles workgroup b of g takes in a launch over n tiles (t = first;
// t < end; t += step).  ORDER_PASSES: in pass p the 8 XCDs take consecutive
// runs of g/8 tiles, XCD x the x-th run of the pass.  ORDER_SLABS: XCD x
// takes the x-th eighth of all tiles and its workgroups walk it together,
// g/8 tiles at a time, so the neighbour rows of a tile in z (the halo of its
// window) are staged by the same XCD shortly before or after it, while its
// L2 still holds them.  Both visit every tile exactly once.
struct TileWalk {
  int t, step, end;
  __device__ __forceinline__ TileWalk(int b, int g, int n, int order) {
    if ((g & 7) != 0) {
      t = b;
      step = g;
      end = n;
    } else if (order == ORDER_SLABS) {
      const int per = (n + 7) >> 3;
      t = (b & 7) * per + (b >> 3);
      step = g >> 3;
      end = min(n, ((b & 7) + 1) * per);
    } else {
      t = (b & 7) * (g >> 3) + (b >> 3);
      step = g;
      end = n;
    }
  }
};

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// Maximum over the wave of a 64-bit unsigned value, in every lane: DPP row
// shifts within rows of 16 lanes, then row broadcasts (ALU only, no LDS
// round trips); lanes that have no source keep their own value.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_max_step(unsigned long long v) {
  const int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
  const uint32_t slo = (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
  const uint32_t shi = (uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
  const unsigned long long o = ((unsigned long long)shi << 32) | slo;
  return o > v ? o : v;
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) {
  v = dpp_max_step<0x111, 0xF>(v);  // row_shr:1
  v = dpp_max_step<0x112, 0xF>(v);  // row_shr:2
  v = dpp_max_step<0x114, 0xF>(v);  // row_shr:4
  v = dpp_max_step<0x118, 0xF>(v);  // row_shr:8: lane 15 of a row holds the row maximum
  v = dpp_max_step<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_max_step<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3: lane 63 holds all
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}

// Compensated FP32 pair (value, error) and exact TwoSum combination.
struct F2 {
  float hi, lo;
};
__device__ __forceinline__ F2 f2_add(F2 a, F2 b) {
  float s = a.hi + b.hi;
  float bp = s - a.hi;
  float e = (a.hi - (s - bp)) + (b.hi - bp);
  return F2{s, (a.lo + b.lo) + e};
}
__device__ __forceinline__ F2 wave_sum_f2(F2 v) {
  for (int o = 32; o > 0; o >>= 1) {
    F2 w{__shfl_xor(v.hi, o, 64), __shfl_xor(v.lo, o, 64)};
    v = f2_add(v, w);
  }
  return v;
}

// k mod 3 for k >= -3, from its 32-bit halves (2^32 = 1 mod 3): a step's state
// is picked by it some ten times, and a 64-bit remainder is ~50 instructions.
__device__ __forceinline__ int64_t mod3(int64_t k) {
  const uint64_t u = (uint64_t)(k + 3);
  const uint32_t s = (uint32_t)u % 3u + (uint32_t)(u >> 32) % 3u;
  return s >= 3u ? s - 3u : s;
}

// Periodic wrap into [-L/2, L/2) (exact: Sterbenz) -- idempotent.
__device__ __forceinline__ double wrap1(double x, double L, double halfL) {
  if (x >= halfL) return x - L;
  if (x < -halfL) return x + L;
  return x;
}

// (int)((x + L/2) * invW) clamped to [0, G-1]; the clamp is applied before the
// conversion (same result for every finite x, no out-of-range conversion).
__device__ __forceinline__ int cell_coord(double x, double halfL, double invW, int G) {
  const double q = (x + halfL) * invW;
  return (int)fmin(fmax(q, 0.0), (double)(G - 1));
}

__device__ __forceinline__ int cell_of(SlotC &S, double x, double y, double z) {
  const int G = S.G;
  return (cell_coord(z, S.halfL, S.invW, G) * G + cell_coord(y, S.halfL, S.invW, G)) * G +
         cell_coord(x, S.halfL, S.invW, G);
}

// Descriptor of the state a replica holds between launches (r(done), or the
// drifted r(done+1), which lives in the same variant).
__device__ __forceinline__ SlotC &slot_held(const Tables &T, int r) {
  const CtlDev &C = T.ctl[r];
  return slot(T, 2 * r + C.var_ring[mod3(C.done)]);
}

// State index held by a replica between launches.
__device__ __forceinline__ int64_t cur_state(const CtlDev &C) {
  return C.clean ? C.done : C.done + 1;
}

__device__ __forceinline__ void latch_error(CtlDev &C, int bits, int64_t step) {
  atomicOr(&C.err, bits);
  atomicMin((unsigned long long *)&C.err_step, (unsigned long long)step);
}

// A new position of step `step`: latch an error for a non-finite coordinate
// or one outside [-3L/2, 3L/2) (the wrap at the next rebuild could not bring
// it back); returns its bit, or 0.
__device__ __forceinline__ int check_atom(SlotC &S, CtlDev &C, double x, double y, double z,
                                          int64_t step) {
  int bad = 0;
  if (!(isfinite(x) && isfinite(y) && isfinite(z))) {
    bad = ERR_NONFINITE;
  } else if (fabs(x) >= 3.0 * S.halfL || fabs(y) >= 3.0 * S.halfL || fabs(z) >= 3.0 * S.halfL) {
    bad = ERR_ESCAPED;
  }
  if (bad) latch_error(C, bad, step);
  return bad;
}

// Cell and layer assignment of one atom (Secs. 3.2, 3.4): the atom's cell
// from its wrapped coordinates, a layer slot from the cell's occupancy
// counter (atomic), the row entry, or the set's overflow list beyond hcap.
// The sort of a rebuild step reads the rows; the cell each atom lands in
// there is written by the sort itself.  Returns the error latched for this
// atom, or 0.
template <bool COH>
__device__ __forceinline__ int bin_atom(SlotC &S, CtlDev &C, int set, int i, double x, double y,
                                        double z, int64_t step) {
  // Called by a prefix of the lanes of a wave (the active atoms of a tile).
  int bad = check_atom(S, C, x, y, z, step);
  if (bad == ERR_NONFINITE) x = y = z = 0.0;
  const int c = cell_of(S, wrap1(x, S.L, S.halfL), wrap1(y, S.L, S.halfL), wrap1(z, S.L, S.halfL));
  // Consecutive lanes with the same cell take their layer slots with one
  // atomic: atoms are stored in cell order, so most of a cell's atoms are
  // neighbours in a wave.
  // (the empty asm keeps the lane masks below from being hoisted out of the
  // tile loop, where they would be held across it and spilled)
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const unsigned long long active = __ballot(1);
  const int na = __popcll(active);
  const int cp = __shfl_up(c, 1, 64);
  const bool leader = lane == 0 || cp != c;
  const unsigned long long lmask = __ballot(leader) & active;
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);
  const int lead = 63 - __clzll(lmask & upto);
  const unsigned long long after = lmask & ~upto;
  const int next = after ? __ffsll((long long)after) - 1 : na;
  int base = 0;
  if (leader) base = atomicAdd(&S.cnt[set][c], next - lane);
  const int slot = __shfl(base, lead, 64) + (lane - lead);
  // the occupancy of the cell's tile, one atomic per run of lanes in one tile
  // (the shuffle runs on every active lane: a lane reading from an inactive
  // one gets 0)
  const int ct = c / CTILE;
  const int ctp = __shfl_up(ct, 1, 64);
  const bool tlead = lane == 0 || ctp != ct;
  const unsigned long long tmask = __ballot(tlead) & active;
  const unsigned long long tafter = tmask & ~upto;
  const int tnext = tafter ? __ffsll((long long)tafter) - 1 : na;
  if (tlead) atomicAdd(&S.tcnt[set][ct], tnext - lane);
  if (slot < S.hcap) {
    st<COH>(&gp(S.H[set])[(size_t)c * S.hcap + slot], i);
  } else {
    const int o = atomicAdd(&S.ovf_n[set], 1);
    if (o < OVF_CAP) {
      st<COH>(&gp(S.ovf[set])[2 * o], c);
      st<COH>(&gp(S.ovf[set])[2 * o + 1], i);
    } else {
      latch_error(C, ERR_CELL, step);
      bad |= ERR_CELL;
    }
  }
  return bad;
}

#define MD_CX(p, q)                             \
  {                                             \
    const int lo_ = min(p, q), hi_ = max(p, q); \
    p = lo_;                                    \
    q = hi_;                                    \
  }
// Compare-exchange network ordering eight values (Batcher odd-even merge).
__device__ __forceinline__ void sort8(int (&v)[8]) {
  MD_CX(v[0], v[1]) MD_CX(v[2], v[3]) MD_CX(v[4], v[5]) MD_CX(v[6], v[7])
  MD_CX(v[0], v[2]) MD_CX(v[1], v[3]) MD_CX(v[4], v[6]) MD_CX(v[5], v[7])
  MD_CX(v[1], v[2]) MD_CX(v[5], v[6])
  MD_CX(v[0], v[4]) MD_CX(v[1], v[5]) MD_CX(v[2], v[6]) MD_CX(v[3], v[7])
  MD_CX(v[2], v[4]) MD_CX(v[3], v[5])
  MD_CX(v[1], v[2]) MD_CX(v[3], v[4]) MD_CX(v[5], v[6])
}
#undef MD_CX

// Visit the atoms of cell c (occupancy cnt) of a set in ascending storage
// index, passing each one's rank (the order of the row entries themselves
// depends on atomic timing, so it is not used).  Up to eight atoms held in
// the row are ordered with a sorting network; larger or overflowing cells
// take repeated minimum searches over the row and the set's overflow list.
template <bool COH, class Visit>
__device__ __forceinline__ void visit_cell(SlotC &S, int set, int c, int cnt,
                                           Visit &&visit) {
  const int32_t *__restrict__ row = S.H[set] + (size_t)c * S.hcap;
  const int inrow = min(cnt, S.hcap);
  if (cnt <= 8 && inrow == cnt) {
    int v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = e < cnt ? ld<COH>(&gp(row)[e]) : INT_MAX;
    sort8(v);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < cnt) visit(v[e], e);
    return;
  }
  int last = -1;
  for (int r = 0; r < cnt; ++r) {
    int best = INT_MAX;
    for (int e = 0; e < inrow; ++e) {
      const int v = ld<COH>(&gp(row)[e]);
      best = (v > last && v < best) ? v : best;
    }
    if (cnt > inrow) {
      const int no = min(ld<COH>(&gp((const int32_t *)S.ovf_n)[set]), OVF_CAP);
      const gcint ov = gp((const int32_t *)S.ovf[set]);
      for (int e = 0; e < no; ++e)
        if (ld<COH>(&ov[2 * e]) == c) {
          const int v = ld<COH>(&ov[2 * e + 1]);
          best = (v > last && v < best) ? v : best;
        }
    }
    if (best == INT_MAX) break;
    last = best;
    visit(best, r);
  }
}

// Maximum of the spread slots of ring entry e (each wave reads all slots;
// every lane loads, the upper half the same slots again, and those copies
// count as zero: no lane-dependent branch for the loads to wait behind).  A
// slot without a replica has no ring and reads as zero.
static_assert((VSPREAD & (VSPREAD - 1)) == 0 && VSPREAD <= 64, "VSPREAD: a power of two");
__device__ __forceinline__ double ring_max(SlotC &S, int64_t e) {
  const int l = threadIdx.x & 63;
  double v = 0.0;
  if (S.vring != nullptr)
    v = __longlong_as_double((long long)S.vring[(e * VSPREAD + (l & (VSPREAD - 1))) * 16]);
  return wave_max(l < VSPREAD ? v : 0.0);
}

// The same for all three ring entries at once: the loads do not wait for the
// step number that selects an entry.  A slot without a replica has no ring
// and reads as zero.
__device__ __forceinline__ void ring_max3(SlotC &S, double (&v)[3]) {
  const int l = threadIdx.x & 63;
  double a[3] = {0.0, 0.0, 0.0};
  if (l < VSPREAD && S.vring != nullptr)
    for (int e = 0; e < 3; ++e)
      a[e] = __longlong_as_double((long long)S.vring[(e * VSPREAD + l) * 16]);
  for (int e = 0; e < 3; ++e) v[e] = wave_max(a[e]);
}

// Entry e (0, 1 or 2) of three values held in registers.
template <class X>
__device__ __forceinline__ X pick3(X a0, X a1, X a2, int64_t e) {
  return e == 0 ? a0 : e == 1 ? a1 : a2;
}

// Whether r(k) is binned during step k-1, so that a sort at step k finds its
// rows (binning every step would cost a step's worth of atomics and row
// writes where a rebuild comes about one step in ten).  Always with the cell
// method and at a forced rebuild; otherwise when the displacement rule of
// rebuild_rule, accumulated with BIN_AHEAD times the maximum speed of step
// k-2 (that of step k-1 is not known while step k-1 runs), would fire at
// step k.  The sort of step k-1, which holds every input of the rule, takes
// this decision for the step kernel of step k-1 and records it
// (CtlDev::bin_ring); the sort of step k reads there whether the rows exist
// (k_run, which takes the same replicas, bins only when the rule has fired, so
// the rule itself does not tell).  When the rule fires
// without them (the maximum speed grew by more than BIN_AHEAD in one step)
// it latches ERR_UNBINNED and the host bins r(k) and resumes, so the
// trajectory does not depend on the guess.  Called by whole waves.
// bins_rule takes the words already read: D2 the committed displacement
// after step k-2, V2 the maximum v^2 of step k-2.
__device__ __forceinline__ bool bins_rule(const SlotC &S, int64_t force_step, int64_t k,
                                          double D2, double V2) {
  if (S.cell_only || k == force_step) return true;
  const bool rb1 = (k - 1 == force_step) || D2 > S.half_shell;
  const double D1 = (rb1 ? 0.0 : D2) + BIN_AHEAD * sqrt(V2) * S.dt;
  return D1 > S.half_shell;
}
template <class Ctl>
__device__ __forceinline__ bool bins_due(SlotC &S, const Ctl &C, int64_t k) {
  const double D2 = C.disp_ring[mod3(k - 2)];
  const double V2 = ring_max(S, mod3(k - 2));
  return bins_rule(S, C.force_step, k, D2, V2);
}

// Rebuild decision for step k (Sec. 3.1): rebuilt when the accumulated sum
// of vmax*dt exceeds delta/2.  disp after step k-1 is recomputed from the
// committed disp after step k-2 (D2) and vmax^2 of step k-1 (V1); *disp1
// receives it.
__device__ __forceinline__ bool rebuild_rule(const SlotC &S, int64_t force_step, int64_t k,
                                             double D2, double V1, double *disp1) {
  const bool rb1 = (k - 1 == force_step) || D2 > S.half_shell;
  const double D1 = (rb1 ? 0.0 : D2) + sqrt(V1) * S.dt;
  *disp1 = D1;
  return (k == force_step) || D1 > S.half_shell;
}

// ---------------------------------------------------------------------------
// (a): first half kick and drift of a clean replica, and binning of r(k+1)
// ---------------------------------------------------------------------------
// One tile of a clean replica at state k; bin: r(k+1) into its set.  Returns
// the error latched for the thread's atom, or 0.
template <bool COH>
__device__ __forceinline__ int kick_tile(SlotC &S, CtlDev &C, int lt, int64_t k, bool bin) {
  const int i = lt * TILE + threadIdx.x;
  if (i >= S.n) return 0;
  const int pb = (int)(k & 1), vb = (int)((k + 1) & 1);
  double f[3];
  for (int a = 0; a < 3; ++a)
    f[a] = S.fp64 ? gp((const double *)S.F)[a * S.npad + i]
                  : (double)gp((const float *)S.F)[a * S.npad + i];
  double xn[3];
  for (int a = 0; a < 3; ++a) {
    const double v = gp(S.V[vb][a])[i] + S.hdt * f[a];
    st<COH>(&gp(S.V[vb][a])[i], v);
    xn[a] = gp(S.P[pb][a])[i] + S.dt * v;
    st<COH>(&gp(S.P[pb ^ 1][a])[i], xn[a]);
  }
  return bin ? bin_atom<COH>(S, C, (int)mod3(k + 1), i, xn[0], xn[1], xn[2], k + 1)
             : check_atom(S, C, xn[0], xn[1], xn[2], k + 1);
}
__global__ __launch_bounds__(TILE) void k_kick(Tables T) {
  const int nt = T.hdr[HDR_NTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nt; t += gridDim.x) {
    const int r = T.tile_rep[t];
    if (slot(T, 2 * r).n <= 0) continue;
    SlotC &S = slot_held(T, r);
    CtlDev &C = T.ctl[r];
    // errors latched by this launch (err_step = done + 1) do not stop it
    if ((C.err != 0 && C.err_step <= C.done) || !C.clean || C.done >= C.target) continue;
    const int64_t k = C.done;
    const bool bin = bins_due(slot(T, 2 * r), C, k + 1);
    // (nobody reads this word in this launch)
    if (t == S.tile_off && threadIdx.x == 0) C.bin_ring[mod3(k)] = bin ? 1 : 0;
    kick_tile<false>(S, C, t - S.tile_off, k, bin);
  }
}

// After k_kick: the kicked replicas hold a drifted state (one thread per
// replica; same gate as the kick).
__global__ void k_kick_end(Tables T) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= T.nslots) return;
  CtlDev &C = T.ctl[r];
  if (slot(T, 2 * r).n <= 0) return;
  if ((C.err != 0 && C.err_step <= C.done) || !C.clean || C.done >= C.target) return;
  C.clean = 0;
}

// Positions of the sorted atoms in 16 bits per coordinate (units of L / 2^16
// from the box's lower corner; x and y in the low word, z in the high one's
// low half), written by the sort for the traversal of the same step.  They
// live in the cell-layer rows of set (k + 2) % 3, which nobody holds during
// step k: the rows of state k are in set k % 3, those of state k + 1 (binned
// ahead during step k) in set (k + 1) % 3.  SlotDev::pk_lim is 0 where the
// rows are too few to hold them.
typedef unsigned long long pk_t;
typedef const __attribute__((address_space(1))) pk_t *gcpk;
typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ pk_t *pk_array(SlotC &S, int64_t k) {
  return (pk_t *)S.H[(int)mod3(k + 2)];
}
__device__ __forceinline__ pk_t pk_of(SlotC &S, double x, double y, double z) {
  const double q = S.pk_scale, h = S.halfL;
  const uint32_t ux = (uint32_t)(int)((x + h) * q) & 0xffffu;
  const uint32_t uy = (uint32_t)(int)((y + h) * q) & 0xffffu;
  const uint32_t uz = (uint32_t)(int)((z + h) * q) & 0xffffu;
  return ((pk_t)uz << 32) | (uy << 16) | ux;
}
// Squared distance of two packed positions; the 16-bit differences wrap, so
// it is the distance of the nearest images.  Each coordinate is within one
// unit of the true one, so a pair within r_n passes s <= (r_n + sqrt 3
// units)^2 (SlotDev::pk_lim); the exact test follows for those that pass.
__device__ __forceinline__ uint32_t pk_dist2(pk_t a, pk_t b) {
  const short2v dxy = __builtin_bit_cast(short2v, (uint32_t)a) -
                      __builtin_bit_cast(short2v, (uint32_t)b);
  const short2v dz = __builtin_bit_cast(short2v, (uint32_t)(a >> 32)) -
                     __builtin_bit_cast(short2v, (uint32_t)(b >> 32));
  return (uint32_t)__builtin_amdgcn_sdot2(dz, dz, __builtin_amdgcn_sdot2(dxy, dxy, 0, false),
                                          false);
}

// ---------------------------------------------------------------------------
// (b): the counting sort by cell
// ---------------------------------------------------------------------------
// Positions listed at a time, and the LDS of the sort.
constexpr int SORT_CAP = 1024;
struct SortLds {
  int s_red[4], s_wsum[4], s_bsum[4], s_any[4];
  int s_bc[TILE], s_bb[TILE], s_bp[TILE];
  int src[SORT_CAP];
  uint8_t lc[SORT_CAP];
};
// The atoms in replica rep's tiles before tile upto, kept by a workgroup from
// one of its units to the next.
struct SortRun {
  int rep = -1, upto = 0, pre = 0;
};

// Share sp of nsp of cell tile t of replica r at step k (the sorts of a step:
// mode MODE_STEP, v(k-1/2) is carried; of the held state: v(k)): from
// descriptor S into D, or in place without reordering (!reo).
template <bool COH>
__device__ __forceinline__ void sort_unit(SlotC &S, SlotC &D, CtlDev &C, int64_t k, int mode,
                                          bool reo, int t, int sp, int nsp, int r, SortRun &run,
                                          SortLds &lds) {
  const int tid = tid_here();
  const int set = (int)mod3(k);
  const int pb = (int)(k & 1);
  const int vb = mode == MODE_STEP ? pb : pb ^ 1;
  const int lt = t - S.ctile_off;
  const int w = tid >> 6, l = tid & 63;

  // atoms in the earlier tiles: a workgroup takes its units in increasing
  // order, so the sum kept from its previous unit of the same replica only
  // grows by the tiles in between (about the grid's size; O(tiles) loads
  // per workgroup instead of every earlier tile at every unit).  Eight
  // loads in flight per thread: integer sums, so the grouping does not
  // change the result.
  const auto TC = gp((const int32_t *)S.tcnt[set]);
  if (run.rep != r || run.upto > lt) {
    run.rep = r;
    run.upto = 0;
    run.pre = 0;
  }
  int pre = 0;
  {
    int q = run.upto + (int)tid;
    for (; q + 7 * TILE < lt; q += 8 * TILE) {
      int p8[8];
#pragma unroll
      for (int u8 = 0; u8 < 8; ++u8) p8[u8] = ld<COH>(&TC[q + u8 * TILE]);
#pragma unroll
      for (int u8 = 0; u8 < 8; ++u8) pre += p8[u8];
    }
    for (; q < lt; q += TILE) pre += ld<COH>(&TC[q]);
  }
  for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o, 64);
  if (l == 0) lds.s_red[w] = pre;

  // workgroup exclusive scan of one cell count per thread
  const int c = lt * CTILE + tid;
  const int cnt = c < S.ncell ? ld<COH>(&gp((const int32_t *)S.cnt[set])[c]) : 0;
  int incl = cnt;
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (l >= o) incl += y;
  }
  if (l == 63) lds.s_wsum[w] = incl;
  const int wmax = wave_max_i(cnt);
  __syncthreads();
  run.pre += ((lds.s_red[0] + lds.s_red[1]) + lds.s_red[2]) + lds.s_red[3];
  run.upto = lt;
  int before = run.pre;
  for (int q = 0; q < w; ++q) before += lds.s_wsum[q];
  const int base = before + incl - cnt;
  if (sp == 0) {
    if (l == 0 && wmax > C.max_h) atomicMax(&C.max_h, wmax);
    if (c <= S.ncell) st<COH>(&gp(S.cs)[c], base);  // c == ncell: the total, n
  }

  // Every atom goes to base of its cell + its rank by current index.  This
  // share takes the tile's positions [s0, s1) in cell order, SORT_CAP at a
  // time: first the storage index of the atom that belongs at each is listed
  // in LDS, then the atoms are moved, consecutive threads to consecutive
  // positions, so the stores are whole lines and all of a thread's loads are
  // in flight together.  (Moved by the thread that holds their cell, four at
  // a time, every store instruction wrote 8 bytes to each of 64 cells: sorting
  // took 176 us at 4 x 10^6, now 134.)
  const int n = S.n;
  const double L = S.L, halfL = S.halfL;
  const bool mixsp = S.nsp > 0;  // a mixture: the species move with the atoms
  const bool packed = S.pk_lim != 0;  // and their packed positions (near_rows)
  const auto PK = gp(pk_array(S, k));
  const int base0 = run.pre;
  const int total = ((lds.s_wsum[0] + lds.s_wsum[1]) + lds.s_wsum[2]) + lds.s_wsum[3];
  const int s1 = base0 + (int)((int64_t)total * (sp + 1) / nsp);
  const bool big = c < S.ncell && cnt > 8 && cnt <= min(S.hcap, 8191);
  for (int s0 = base0 + (int)((int64_t)total * sp / nsp); s0 < s1; s0 += SORT_CAP) {
    const int se = min(s1, s0 + SORT_CAP);
    auto list = [&](int p, int atom, int lc) {
      if (p < s0 || p >= se) return;
      lds.src[p - s0] = atom;
      lds.lc[p - s0] = (uint8_t)lc;
    };
    const bool here = c < S.ncell && cnt > 0 && base < se && base + cnt > s0;
    // cells of up to eight atoms (the usual ones): a sorting network
    if (here && !big) {
      if (cnt <= 8 && cnt <= S.hcap) {
        const int32_t *row = S.H[set] + (size_t)c * S.hcap;
        int v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = e < cnt ? ld<COH>(&gp(row)[e]) : INT_MAX;
        sort8(v);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e < cnt) list(base + e, v[e], tid);
      } else {
        // a cell that spilled into the overflow list: repeated minimum searches
        visit_cell<COH>(S, set, c, cnt, [&](int atom, int q) { list(base + q, atom, tid); });
      }
    }
    // larger cells whose members all sit in their rows, by the whole
    // workgroup: their atoms are listed (big cell j holds entries s_bp[j] ...
    // of the list), and each atom's rank is the number of smaller indices in
    // its row
    const bool bigh = here && big;
    const bool anybig = __ballot(bigh) != 0;
    if (l == 0) lds.s_any[w] = anybig ? 1 : 0;
    __syncthreads();
    if ((lds.s_any[0] | lds.s_any[1]) | (lds.s_any[2] | lds.s_any[3])) {
      const int bv = bigh ? ((1 << 21) | cnt) : 0;  // (cell count, atom count)
      int binc = bv;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(binc, o, 64);
        if (l >= o) binc += y;
      }
      if (l == 63) lds.s_bsum[w] = binc;
      __syncthreads();
      int bbefore = 0;
      for (int q = 0; q < w; ++q) bbefore += lds.s_bsum[q];
      const int bex = bbefore + binc - bv;
      if (bigh) {
        const int j = bex >> 21;
        lds.s_bc[j] = c;
        lds.s_bb[j] = base;
        lds.s_bp[j] = bex & ((1 << 21) - 1);
      }
      const int btot = ((lds.s_bsum[0] + lds.s_bsum[1]) + lds.s_bsum[2]) + lds.s_bsum[3];
      const int nb = btot >> 21, B = btot & ((1 << 21) - 1);
      __syncthreads();
      for (int q = tid; q < B; q += TILE) {
        int lo = 0, hi = nb - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (lds.s_bp[mid] <= q) lo = mid;
          else hi = mid - 1;
        }
        const int cj = lds.s_bc[lo];
        const int cntj = (lo + 1 < nb ? lds.s_bp[lo + 1] : B) - lds.s_bp[lo];
        const auto row = gp((const int32_t *)S.H[set]) + (size_t)cj * S.hcap;
        const int v = ld<COH>(&row[q - lds.s_bp[lo]]);
        int rank = 0;
        for (int f = 0; f < cntj; ++f) rank += ld<COH>(&row[f]) < v ? 1 : 0;
        list(lds.s_bb[lo] + rank, v, cj - lt * CTILE);
      }
      __syncthreads();
    }
    for (int p0 = s0 + tid; p0 < se; p0 += 4 * TILE) {
      int at[4], cc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int p = p0 + u * TILE;
        at[u] = p < se ? lds.src[p - s0] : -1;
        cc[u] = p < se ? lt * CTILE + lds.lc[p - s0] : 0;
        if (p >= n || at[u] >= n) at[u] = -1;  // inconsistent counts: never expected
      }
      if (!reo) {
        // no reordering: position p of cell order refers to the atom where it
        // is; it is wrapped in place (read and written by this thread only)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = at[u];
          if (q < 0) continue;
          st<COH>(&gp(S.perm)[p0 + u * TILE], q);
          st<COH>(&gp(S.cell)[q], cc[u]);
#pragma unroll
          for (int d = 0; d < 3; ++d) st<COH>(&gp(S.P[pb][d])[q], wrap1(ld<COH>(&gp((const double *)S.P[pb][d])[q]), L, halfL));
        }
        continue;
      }
      double pv[4][6];
      int idv[4], spv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = max(at[u], 0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          pv[u][d] = ld<COH>(&gp((const double *)S.P[pb][d])[q]);
          pv[u][3 + d] = ld<COH>(&gp((const double *)S.V[vb][d])[q]);
        }
        idv[u] = ld<COH>(&gp((const int32_t *)S.id)[q]);
        spv[u] = mixsp ? ld<COH>(&gp((const int32_t *)S.sp)[q]) : 0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (at[u] < 0) continue;
        const int p = p0 + u * TILE;
        double x[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          x[d] = wrap1(pv[u][d], L, halfL);
          st<COH>(&gp(D.P[pb][d])[p], x[d]);
          st<COH>(&gp(D.V[vb][d])[p], pv[u][3 + d]);
        }
        if (packed) st<COH>(&PK[p], pk_of(S, x[0], x[1], x[2]));
        st<COH>(&gp(D.id)[p], idv[u]);
        st<COH>(&gp(D.cell)[p], cc[u]);
        if (mixsp) st<COH>(&gp(D.sp)[p], spv[u]);
      }
    }
    __syncthreads();
  }
  __syncthreads();
}

// Workgroup t of a replica takes cell tile t (CTILE cells, one per thread):
// cell_start of the tile's first cell is the sum of the occupancies of the
// earlier tiles (counted while binning), cell_start of its cells follows
// from a workgroup scan, and every atom goes to cell_start of its cell plus
// its rank among the cell's atoms by current storage index -- the sequential
// layer assignment of Sec. 3.4 read in cell order (Sec. 3.5), i.e. a stable
// counting sort.  Positions are wrapped on the way (Sec. 3.1, step (b)).
// Workgroups depend on nobody.
//   mode == MODE_STEP: step k = base + s + 1 of a run; replicas whose rule
//   does not fire leave; v(k-1/2) is carried.
//   otherwise: the held clean state (k = done); v(k) is carried; k_flip
//   switches the variant afterwards.
__global__ __launch_bounds__(TILE, 4) void k_sort(Tables T, int s, int mode, int only) {
  __shared__ SortLds lds;
  // the decision for a replica is launch-invariant: a workgroup works it out
  // once for a run of consecutive cell tiles of one replica
  int rc = -1, var = 0;
  int64_t k = 0;
  bool skip = true, rebuild = false, unbinned = false, reo = true;
  double d1 = 0.0;
  SortRun run;
  // one replica: every unit is replica 0's
  const bool solo = T.nslots == 1;
  // last reordering before step k, and whether step k bins r(k+1) (MODE_STEP)
  int64_t reo1 = 0;
  bool bin1 = false;
  // works out the decision for replica r; leaves skip set when the launch
  // has nothing to do for it
  auto decide = [&](int r) {
    CtlDev &C = T.ctl[r];
    SlotC &S0 = slot(T, 2 * r);
    rc = r;
    skip = true;
    if (only >= 0 && r != only) return;
    if (mode == MODE_STEP) {
      // every word the rule reads is loaded before any is tested: an idle
      // launch is this evaluation, and tested one after another the words
      // were a chain of dependent loads
      const int64_t base = C.base, target = C.target, err_step = C.err_step;
      const int64_t force_step = C.force_step, bins_step = C.bins_step;
      const int32_t err = C.err;
      const int64_t ro0 = C.reo_ring[0], ro1 = C.reo_ring[1], ro2 = C.reo_ring[2];
      const double dp0 = C.disp_ring[0], dp1 = C.disp_ring[1], dp2 = C.disp_ring[2];
      const int32_t vr0 = C.var_ring[0], vr1 = C.var_ring[1], vr2 = C.var_ring[2];
      const int32_t bn0 = C.bin_ring[0], bn1 = C.bin_ring[1], bn2 = C.bin_ring[2];
      double vm[3];
      ring_max3(S0, vm);
      k = base + s + 1;
      const int64_t e1 = mod3(k - 1), e2 = mod3(k - 2);
      const double D2 = pick3(dp0, dp1, dp2, e2);
      var = pick3(vr0, vr1, vr2, e1);
      reo1 = pick3(ro0, ro1, ro2, e1);
      rebuild = true;
      d1 = 0.0;
      const double V1 = pick3(vm[0], vm[1], vm[2], e1);
      if (!S0.cell_only) rebuild = rebuild_rule(S0, force_step, k, D2, V1, &d1);
      unbinned = rebuild && pick3(bn0, bn1, bn2, e1) == 0 && k != bins_step;
      // the step kernel's binning ahead for step k + 1 (see bins_due): the
      // rule of step k + 1 from the displacement after step k-1 (d1, which
      // this launch commits) and the maximum speed of step k-1
      bin1 = k != target && bins_rule(S0, force_step, k + 1, d1, V1);
      // reorder at this rebuild, or keep the storage order (Table 7: the
      // reordering is done at the first rebuild N_R steps after the last)
      reo = !S0.noreo && (S0.nr <= 0 || k - reo1 >= S0.nr);
      if (k > target || (err != 0 && err_step <= k)) return;
    } else {
      if (!C.clean) return;
      k = C.done;
      if (C.err != 0 && C.err_step <= k) return;
      var = C.var_ring[mod3(k)];
      rebuild = true;
      unbinned = false;
      reo = !S0.noreo;  // a sort of the held state reorders (k_flip records it)
    }
    skip = false;
  };
  if (solo) {
    // (needs no table read, so it overlaps the header's loads) with nothing
    // to sort in this launch only the workgroup of unit 0 has work: it
    // records the decision
    decide(0);
    if (skip || (mode == MODE_STEP && (!rebuild || unbinned) &&
                 xcd_block(blockIdx.x, gridDim.x) != 0))
      return;
  }
  const int nct = cview(T.hdr)[HDR_NCTILES];
  // a cell tile is shared by nsp workgroups (dense systems, whose cells hold
  // many atoms); unit u = (tile u / nsp, share u % nsp)
  const int nsp = max(cview(T.hdr)[HDR_SPLIT], 1);
  const int nunits = nct * nsp;
  for (int u = xcd_block(blockIdx.x, gridDim.x); u < nunits; u += gridDim.x) {
    const int t = u / nsp, sp = u - t * nsp;
    const int r = solo ? 0 : cview(T.ctile_rep)[t];
    CtlDev &C = T.ctl[r];
    SlotC &S0 = slot(T, 2 * r);
    if (r != rc) decide(r);
    // one replica: its units are all the launch has, so a workgroup with
    // nothing to do for it stops instead of visiting its other units (an
    // idle launch then costs one unit per workgroup)
    if (skip) {
      if (solo) break;
      continue;
    }
    if (mode == MODE_STEP) {
      if (t == S0.ctile_off && sp == 0 && threadIdx.x == 0) {
        // the one writer of these ring slots for step k (with one replica
        // that is unit 0, the first unit of its workgroup, so no workgroup
        // stops before it); a step whose rows are missing is stopped here
        // and done again once the host has binned it
        if (unbinned) {
          latch_error(C, ERR_UNBINNED, k);
        } else {
          C.rb_ring[mod3(k)] = rebuild ? (reo ? RB_REORDER : RB_PERM) : RB_NONE;
          C.bin_ring[mod3(k)] = bin1 ? 1 : 0;
          C.reo_ring[mod3(k)] = rebuild && reo ? k : reo1;
          if (!S0.cell_only) {
            C.disp_ring[mod3(k - 1)] = d1;
            if (rebuild && k != C.force_step) C.n_rebuilds += 1;
          }
        }
      }
      if (!rebuild || unbinned) {
        if (solo) break;
        continue;
      }
    }
    sort_unit<false>(slot(T, 2 * r + var), slot(T, 2 * r + (var ^ 1)), C, k, mode, reo, t, sp, nsp, r,
              run, lds);
  }
}

// After a sort of the held states (mode != MODE_STEP): switch the replicas
// that were sorted to their other variant (same gate as k_sort).
__global__ void k_flip(Tables T, int only) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= T.nslots || (only >= 0 && r != only)) return;
  if (slot(T, 2 * r).n <= 0) return;
  CtlDev &C = T.ctl[r];
  if (!C.clean || slot(T, 2 * r).noreo) return;  // no reordering: nothing moved
  const int64_t k = C.done;
  if (C.err != 0 && C.err_step <= k) return;
  C.var_ring[mod3(k)] ^= 1;
  C.ord_ring[mod3(k)] = 0;  // the held state is in cell order again
  C.reo_ring[mod3(k)] = k;
}

// ---------------------------------------------------------------------------
// (b)-(e) and the next (a): the step kernel
// ---------------------------------------------------------------------------
template <typename R>
struct Acc {
  R fx, fy, fz, u, w;
};

// FP32 1/s: the hardware reciprocal (within 1 ulp) refined by one Newton step
// (two explicit FMAs), which brings it to about half an ulp.  The refinement
// matters where every pair has the same separation (a lattice): a reciprocal
// 1 ulp off then shifts every pair's virial term by ~2e-6 relative through
// the cancellation in r^-6 - 1/2, and the shift does not average out.
__device__ __forceinline__ float recip(float s) {
  const float r = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(r, __builtin_fmaf(-s, r, 1.0f), r);
}
__device__ __forceinline__ double recip(double s) { return 1.0 / s; }

// Pair force and energy of Eq. (1) with the soft-sphere shift: for r^2 = s,
// f = 48 r^-8 (r^-6 - 1/2) (force on i is f d), u = 4 r^-6 (r^-6 - 1) + shift.
// FP32 uses the refined hardware reciprocal above.
// The energy and virial terms are summed only when `energy` is set (a
// wave-uniform flag: the steps whose per-atom sums somebody reads); the
// force arithmetic is the same either way.  The list loops pass a constant: with a
// run-time flag the compiler works the terms out for every pair of every step
// and selects (9 of the 37 VALU instructions a list entry costs, VALU issue
// being half of a list step), and a branch over them at every pair costs as
// much as it saves.  200 steps of 864 atoms: selects 2 250 us, a branch a pair
// 2 323, a constant 2 209; 1 000 of 4e6: 340.9, 340.3, 337.1 ms; 200 of 32 000
// in FP64: 2 975, 3 056, 2 902 us.
template <typename R>
__device__ __forceinline__ void pair_accum(Acc<R> &a, double dx, double dy, double dz, double s,
                                           R ushift, bool energy) {
  const R sr = (R)s;
  const R rri = recip(sr);
  const R rri3 = rri * rri * rri;
  const R f = (R)48 * rri3 * (rri3 - (R)0.5) * rri;
  a.fx += f * (R)dx;
  a.fy += f * (R)dy;
  a.fz += f * (R)dz;
  if (energy) {
    a.u += (R)4 * rri3 * (rri3 - (R)1) + ushift;
    a.w += f * sr;
  }
}

// The same for species pair k of a mixture: Eq. (1) in units of sigma_ab and
// epsilon_ab, r^-2 scaled by sigma^2 (with sigma = epsilon = 1 every product
// is the one-species arithmetic above).
template <typename R>
__device__ __forceinline__ void pair_accum_mix(Acc<R> &a, double dx, double dy, double dz,
                                               double s, const PairTab *t, int k, bool energy) {
  const R sr = (R)s;
  const R rinv = recip(sr);
  const R rri = (R)t->sig2[k] * rinv;
  const R rri3 = rri * rri * rri;
  const R f = (R)t->eps48[k] * rri3 * (rri3 - (R)0.5) * rinv;
  a.fx += f * (R)dx;
  a.fy += f * (R)dy;
  a.fz += f * (R)dz;
  if (energy) {
    a.u += (R)t->eps4[k] * rri3 * (rri3 - (R)1) + (R)t->shift[k];
    a.w += f * sr;
  }
}

// Image shift code: 2 bits per dimension, a two's-complement multiple of L
// (0 -> 0, 1 -> +L, 3 -> -L).
__device__ __forceinline__ double img_shift(uint32_t code, double L) {
  return code == 0 ? 0.0 : (code == 1 ? L : -L);
}

// Cell coordinate c (one of the 27 offsets, so -1..G) wrapped into [0, G),
// and the image code of the atoms found there.
__device__ __forceinline__ int wrap_cell(int c, int G, uint32_t *code) {
  if (c >= G) {
    *code = 3;
    return c - G;
  }
  if (c < 0) {
    *code = 1;
    return c + G;
  }
  *code = 0;
  return c;
}

// ---------------------------------------------------------------------------
// LDS window of a tile
// ---------------------------------------------------------------------------
// Shared state of a tile's window while the tile is evaluated.
struct Window {
  int wt[WSTRIDE];       // staging intervals: count (-1: none), then (start, len, slot)
  int dl[NROWS * 3];     // per (source row, dz, dy): slot - storage index for the
                         // target row's main piece, its cell 0 and its cell G-1
  int rf;                // first source row (cz G + cy) of the tile
  int whole;             // 1: the window is the whole system, slot = storage index
};

// At a sort: the candidates of the tile's atoms (sorted, so the tile is a run
// of cells spanning source rows rf..rl) lie in the 9 target rows (dz, dy) of
// every source row, in the x-range of that source row widened by one cell
// (with the periodic wrap).  Wave 0 lists (target row, x-range) for every
// (source row, dz, dy), sorts the list by target row (bitonic, across the
// lanes), unites the x-ranges of equal rows, and turns each row into 1-3 cell
// pieces (cell 0 | main | cell G-1 when the x-range wraps, else one piece),
// i.e. storage-index intervals via cell_start.  Wave 0 then gives the pieces
// LDS slots in list order while they fit in WCAP (from the first that does
// not, pieces stay in global memory), merging storage-adjacent ones into
// staging intervals, with wave prefix sums.  The staging table also goes to
// S.win for the list steps until the next sort.
__device__ __forceinline__ void make_window(SlotC &S, int lt, Window &w, int *scratch) {
  const int tid = tid_here();
  __shared__ int s_np;
  int *piece = scratch;              // [2 * 192] start, end
  int *pdelta = scratch + 2 * 192;   // [192] slot - storage index, or NOSLOT
  const int n = S.n;
  const int lane = tid;
  int T = INT_MAX, xa = 0, xb = 0, ell = 0, pos = 0, np = 0;
  bool full = false, w0 = false, wg = false;
  if (tid < 64) {
    const int G = S.G;
    const int i_f = lt * TILE, i_l = min(n, i_f + TILE) - 1;
    const auto CL = gp((const int32_t *)S.cell);
    const int c_f = CL[i_f], c_l = CL[i_l];
    const int rf = c_f / G, rl = c_l / G, ns = rl - rf + 1;
    const bool whole = n <= WCAP && !S.nowin;
    if (lane == 0) {
      w.rf = rf;
      w.whole = whole;
    }
    if (whole || ns * 9 > NROWS || S.nowin) {
      if (lane == 0) s_np = whole ? -2 : -1;  // whole system / no window
    } else {
      if (lane < ns * 9) {
        const int sr = lane / 9, q = lane % 9;
        const int rho = rf + sr, cz = rho / G, cy = rho % G;
        uint32_t im;
        const int tz = wrap_cell(cz + q / 3 - 1, G, &im);
        const int ty = wrap_cell(cy + q % 3 - 1, G, &im);
        T = tz * G + ty;
        xa = (sr == 0 ? c_f % G : 0) - 1;
        xb = (sr == ns - 1 ? c_l % G : G - 1) + 1;
        ell = lane;
      }
      {
        // sort the ns * 9 entries by row: each entry's rank is the number
        // of entries before it (smaller row, or the same row and a lower
        // lane), read lane by lane through scalar registers; the entries
        // then move to their ranks through LDS (lanes without an entry keep
        // theirs, past every rank)
        const int ne9 = ns * 9;
        int rank = lane;
        if (lane < ne9) {
          rank = 0;
          for (int j = 0; j < ne9; ++j) {
            const int Tj = __builtin_amdgcn_readlane(T, j);
            rank += (Tj < T || (Tj == T && j < lane)) ? 1 : 0;
          }
        }
        int *srt = scratch + 3 * 192;  // [4][64], after the pieces
        srt[rank] = T;
        srt[64 + rank] = xa;
        srt[128 + rank] = xb;
        srt[192 + rank] = ell;
        T = srt[lane];
        xa = srt[64 + lane];
        xb = srt[128 + lane];
        ell = srt[192 + lane];
      }
      const int Tp = __shfl_up(T, 1, 64);
      const bool lead = T != INT_MAX && (lane == 0 || Tp != T);
      int ua = xa, ub = xb;
      for (int d = 1; d < 64; ++d) {
        const int T2 = __shfl_down(T, d, 64), a2 = __shfl_down(xa, d, 64),
                  b2 = __shfl_down(xb, d, 64);
        const bool same = lane + d < 64 && T2 == T && T != INT_MAX;
        if (same) {
          ua = min(ua, a2);
          ub = max(ub, b2);
        }
        if (__ballot(same) == 0) break;
      }
      int c0[3] = {0, 0, 0}, c1[3] = {0, 0, 0};
      if (lead) {
        const int rb = T * G;
        full = ub - ua + 1 >= G;
        if (full) {
          c0[0] = rb;
          c1[0] = rb + G;
          np = 1;
        } else {
          w0 = ub >= G;  // x = G is cell 0 of the row
          wg = ua < 0;   // x = -1 is cell G-1 of the row
          if (w0) {
            c0[np] = rb;
            c1[np] = rb + 1;
            ++np;
          }
          c0[np] = rb + max(ua, 0);
          c1[np] = rb + min(ub, G - 1) + 1;
          ++np;
          if (wg) {
            c0[np] = rb + G - 1;
            c1[np] = rb + G;
            ++np;
          }
        }
      }
      pos = np;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(pos, o, 64);
        if (lane >= o) pos += y;
      }
      const int total = __shfl(pos, 63, 64);
      pos -= np;
      const auto CS = gp((const int32_t *)S.cs);
      for (int e = 0; e < np; ++e) {
        piece[2 * (pos + e)] = CS[c0[e]];
        piece[2 * (pos + e) + 1] = CS[c1[e]];
      }
      // every lane of a run takes its leader's pieces
      const unsigned long long lmask = __ballot(lead);
      const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);
      const int ll = 63 - __clzll(lmask & upto);
      pos = __shfl(pos, ll, 64);
      np = __shfl(np, ll, 64);
      full = __shfl((int)full, ll, 64);
      w0 = __shfl((int)w0, ll, 64);
      wg = __shfl((int)wg, ll, 64);
      if (lane == 0) s_np = total;
    }
  }
  __syncthreads();
  if (tid < 64) {
    const int npc = s_np;
    if (npc == -2) {
      if (lane == 0) {
        w.wt[0] = 1;
        w.wt[1] = 0;
        w.wt[2] = n;
        w.wt[3] = 0;
      }
    } else if (npc < 0) {
      if (lane == 0) w.wt[0] = -1;
    } else {
      // Pieces take slots in list order while they fit (from the first that
      // does not, the rest stay in global memory).  A non-empty piece that
      // continues the previous non-empty one in storage extends its staging
      // interval, else it opens one (at most NWIN).  Lane l holds pieces
      // 3l .. 3l+2; offsets and interval numbers are wave prefix sums.
      int ps[3], pe[3], ln[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int p = 3 * lane + e;
        ps[e] = p < npc ? piece[2 * p] : 0;
        pe[e] = p < npc ? piece[2 * p + 1] : 0;
        ln[e] = p < npc ? max(pe[e] - ps[e], 0) : 0;
      }
      auto scan = [&](int v) {  // inclusive prefix sum over the wave
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(v, o, 64);
          if (lane >= o) v += y;
        }
        return v;
      };
      const int lsum = (ln[0] + ln[1]) + ln[2];
      int off[3];
      off[0] = scan(lsum) - lsum;
      off[1] = off[0] + ln[0];
      off[2] = off[1] + ln[1];
      const int pe_prev = __shfl_up(pe[2], 1, 64), ln_prev = __shfl_up(ln[2], 1, 64);
      bool fit[3], st[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int p = 3 * lane + e;
        const int prev_end = e == 0 ? pe_prev : pe[e - 1];
        const bool prev_full = e == 0 ? (lane > 0 && ln_prev > 0) : ln[e - 1] > 0;
        fit[e] = p < npc && ln[e] > 0 && off[e] + ln[e] <= WCAP;
        st[e] = fit[e] && !(prev_full && ps[e] == prev_end);
      }
      const int nst = (int)st[0] + (int)st[1] + (int)st[2];
      const int kincl = scan(nst), nstarts = __shfl(kincl, 63, 64);
      int k[3];
      k[0] = kincl - nst + (int)st[0] - 1;
      k[1] = k[0] + (int)st[1];
      k[2] = k[1] + (int)st[2];
      bool ok[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) ok[e] = fit[e] && k[e] < NWIN;
      // the piece after e continues e's interval?
      const bool ok_next0 = __shfl_down((int)ok[0], 1, 64) != 0,
                 st_next0 = __shfl_down((int)st[0], 1, 64) != 0;
      const bool cont[3] = {ok[1] && !st[1], ok[2] && !st[2],
                            lane < 63 && ok_next0 && !st_next0};
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int p = 3 * lane + e;
        if (p < npc) pdelta[p] = ln[e] == 0 ? 0 : (ok[e] ? off[e] - ps[e] : NOSLOT);
        if (ok[e] && st[e]) {
          w.wt[3 * k[e] + 1] = ps[e];
          w.wt[3 * k[e] + 3] = off[e];
        }
        if (ok[e] && !cont[e]) w.wt[3 * k[e] + 2] = off[e] + ln[e];  // end slot
      }
      // (same wave, later instructions: the end slots are written) length =
      // end - first slot
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (ok[e] && st[e]) w.wt[3 * k[e] + 2] -= off[e];
      if (lane == 0) w.wt[0] = min(nstarts, NWIN);
    }
  }
  __syncthreads();
  if (tid < 64 && T != INT_MAX) {
    const int dm = pdelta[pos + (w0 ? 1 : 0)];
    w.dl[3 * ell] = dm;
    w.dl[3 * ell + 1] = full ? dm : (w0 ? pdelta[pos] : NOSLOT);
    w.dl[3 * ell + 2] = full ? dm : (wg ? pdelta[pos + np - 1] : NOSLOT);
  }
  // the staging table for the list steps until the next sort
  auto WG = gp(S.win) + (size_t)lt * WSTRIDE;
  const int nint = w.wt[0];
  if ((int)tid < 1 + 3 * max(nint, 0)) WG[tid] = w.wt[tid];
  __syncthreads();
}

template <bool COH>
__device__ __forceinline__ void stage_species(const int *wt, gcint SP, int8_t *ssp) {
  const int tid = tid_here(), nint = wt[0];
  if (nint <= 0) return;
  const int total = wt[3 * nint] + wt[3 * nint - 1];
  int q = 0, end = wt[2];
  for (int sl = tid; sl < total; sl += TILE) {
    while (sl >= end) {
      ++q;
      end = wt[3 * q + 3] + wt[3 * q + 2];
    }
    ssp[sl] = (int8_t)ld<COH>(&SP[wt[3 * q + 1] + (sl - wt[3 * q + 3])]);
  }
}

// Stage the window's atoms (positions of the current step) into LDS.
// MIX: the species of the window's atoms go to ssp beside the coordinates.
template <bool MIX, bool COH>
__device__ __forceinline__ void stage_window(const int *wt, gcdouble X, gcdouble Y, gcdouble Z,
                                             double *sx, double *sy, double *sz, gcint SP,
                                             int8_t *ssp) {
  const int tid = tid_here();
  // The intervals fill slots 0 .. total-1 in order.  The coordinates go
  // straight from global memory into LDS (loads that write LDS, not
  // registers): wave w fills chunks of 32 slots c = w, w + 4, ..., lane l
  // the low (l even) or high (l odd) word of slot 32c + l/2, whose source it
  // finds by walking the interval table forward.  Nothing waits for the
  // data here, so all of a wave's loads are in flight together; the barrier
  // after the staging waits for them.
  const int nint = wt[0];
  if (nint <= 0) return;
  constexpr int AUX = COH ? 16 : 0;  // 16: device scope (sc1), see ld<COH>
  const int total = wt[3 * nint] + wt[3 * nint - 1];
  typedef __attribute__((address_space(1))) const char *gcchar;
  typedef __attribute__((address_space(3))) void *lvoid;
  const int l = tid & 63;
  const int c0 = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const int nch = (total + 31) >> 5;
  int q = 0, end = wt[2];
  for (int c = c0; c < nch; c += TILE / 64) {
    const int sl = 32 * c + (l >> 1);
    if (sl < total) {
      while (sl >= end) {
        ++q;
        end = wt[3 * q + 3] + wt[3 * q + 2];
      }
      const size_t off = (size_t)(wt[3 * q + 1] + (sl - wt[3 * q + 3])) * 8 + 4 * (l & 1);
      __builtin_amdgcn_global_load_lds((gcchar)X + off, (lvoid)((char *)sx + 256 * c), 4, 0, AUX);
      __builtin_amdgcn_global_load_lds((gcchar)Y + off, (lvoid)((char *)sy + 256 * c), 4, 0, AUX);
      __builtin_amdgcn_global_load_lds((gcchar)Z + off, (lvoid)((char *)sz + 256 * c), 4, 0, AUX);
    }
  }
  // the species bytes through registers (after the coordinates' loads have
  // gone out)
  if constexpr (MIX) stage_species<COH>(wt, SP, ssp);
}

// Storage bounds of neighbour row q (dz = q / 3 - 1, dy = q % 3 - 1) of an
// atom in cell (cx, cy, cz): the x-neighbours that do not wrap (one
// contiguous range, b[0] .. b[1]) and the one wrapped cell (b[2] .. b[3]).
template <class CSP>
__device__ __forceinline__ void row_bounds(CSP CS, int G, int cx, int cy, int cz, int q,
                                           int (&b)[4]) {
  const int xm0 = max(cx - 1, 0), xm1 = min(cx + 2, G);
  const int xe = cx == 0 ? G - 1 : 0;
  const int nz = cz + q / 3 - 1, ny = cy + q % 3 - 1;
  const int row = ((nz < 0 ? nz + G : nz >= G ? nz - G : nz) * G +
                   (ny < 0 ? ny + G : ny >= G ? ny - G : ny)) * G;
  b[0] = CS[row + xm0];
  b[1] = CS[row + xm1];
  b[2] = CS[row + xe];
  b[3] = CS[row + xe + 1];
}

// The general 27-cell traversal (offsets z-major, x fastest; ascending
// storage index within a cell, which is ascending index before the sort):
// atoms that are not stored in cell order, atoms whose list overflowed, and
// systems without room for the packed positions (near_rows is the usual
// traversal).  The three cells of an x-row are one contiguous range of storage
// indices unless the row wraps, where it is two.  Candidates are read from
// the LDS window (slot = storage index + the row piece's offset), or from
// global memory for a piece the window could not hold.  Accepts r^2 < r_n^2
// into W when building (window slot, or storage index with GFLAG), and
// accumulates the forces of pairs with r^2 < r_c^2.  Positions were wrapped
// by the sort, so they are read as stored.
// MIX: a mixture; the candidates' species come from ssp (LDS) or SP, atom
// i's is spi, and each pair takes its own cutoff and parameters from tab.
template <typename R, bool MIX, bool COH>
__device__ __forceinline__ int traverse_sorted(SlotC &S, int i, int ci, gcdouble X,
                                               gcdouble Y, gcdouble Z, const Window &w,
                                               const double *sx, const double *sy,
                                               const double *sz, double xi, double yi,
                                               double zi, bool build, bool force, bool energy,
                                               Acc<R> &a, const int8_t *ssp, gcint SP, int spi,
                                               const PairTab *tab, bool unord,
                                               bool global_only = false,
                                               const int *pre0 = nullptr) {
  const int G = S.G;
  const double L = S.L, rn2 = S.rn2, rc2 = S.rc2;
  const R ushift = (R)S.ushift;
  const int mcap = S.mcap;
  // the next list entry's address: row min(m, mcap - 1) of W (an atom whose
  // list overflows keeps overwriting its last row; its list is not used)
  auto wp = gp(S.W) + i;
  const size_t np = (size_t)S.npad;
  const auto CS = gp((const int32_t *)S.cs);
  const int cx = ci % G, cy = (ci / G) % G, cz = ci / (G * G);
  // global_only: candidates from global memory (the window's row table is
  // not at hand)
  const bool whole = !global_only && w.whole, rows = !global_only && !whole && w.wt[0] >= 0;
  const int sr = rows ? ci / G - w.rf : 0;  // source row of the atom within the tile
  int m = 0;
  // without reordering, position j of cell order is the atom stored at perm[j]
  const bool noreo = unord;
  const gcint PERM = gp((const int32_t *)S.perm);
  // A lane at an x-edge of the box (cx = 0 or G-1) has two ranges per row,
  // the wrapped cell and the row's own cells: it visits both in x order (cell
  // G-1 first when cx = 0, cell 0 last when cx = G-1), each candidate with
  // its own window offset and x image shift.
  const bool wlo = cx == 0, whi = cx == G - 1 && cx != 0;
  const bool edge = wlo || whi;
  const bool anyedge = __ballot(edge) != 0;
  // One row, in two passes over at most 32 candidates at a time: the first
  // only tests (r^2 < r_n^2, one acceptance bit per candidate and lane), the
  // second takes each lane's accepted candidates in order, lists them and
  // adds their forces.  EDGE: some lane has two ranges.  own: the row may hold
  // atom i itself (the 27 cells are distinct for G >= 3, so only q = 4 does).
  auto row = [&](auto edg, bool own, int loM, int hiM, int dM, int loW, int hiW, int dW,
                 uint32_t cyz, double by, double bz) {
    constexpr bool EDGE = decltype(edg)::value;
    // candidate k: k < lenF of the first range, then the second
    int loF = loM, lenF = hiM - loM, tot = lenF, loS = 0;
    if (EDGE) {
      const int lenW = edge ? hiW - loW : 0;
      lenF = wlo ? lenW : tot;
      loF = wlo ? loW : loM;
      loS = (wlo ? loM : loW) - lenF;
      tot += lenW;
    }
    const double bw = wlo ? L : -L;
    const uint32_t cw = cyz | ((wlo ? 1u : 3u) << J_BITS);
    // position j in cell order, window offset and whether the x image applies
    auto where = [&](int k, int &j, int &d, bool &isw) {
      isw = false;
      j = loF + k;
      d = dM;
      if (EDGE) {
        const bool inF = k < lenF;
        j = (inF ? loF : loS) + k;
        isw = edge && inF == wlo;
        d = isw ? dW : dM;
      }
    };
    auto coords = [&](int j, int d, double &x, double &y, double &z, int &js, int &sj) {
      js = j;
      if (d != NOSLOT) {
        x = sx[j + d];
        y = sy[j + d];
        z = sz[j + d];
        if (MIX) sj = ssp[j + d];
      } else {
        if (noreo) js = ld<COH>(&PERM[j]);
        x = ld<COH>(&X[js]);
        y = ld<COH>(&Y[js]);
        z = ld<COH>(&Z[js]);
        if (MIX) sj = ld<COH>(&SP[js]);
      }
    };
    auto separation = [&](double x, double y, double z, bool isw, double &dx, double &dy,
                          double &dz) {
      dx = xi - x;
      dy = yi - y;
      dz = zi - z;
      if (EDGE) dx = dx + (isw ? bw : 0.0);
      dy = dy + by;
      dz = dz + bz;
      return (dx * dx + dy * dy) + dz * dz;
    };
    for (int c0 = 0; __ballot(c0 < tot) != 0; c0 += 32) {
      const int end = min(tot - c0, 32);
      uint32_t acc = 0;
      int g = 0;
      for (; g < end; g += 4) {
        double x[4], y[4], z[4];
        bool isw[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = min(c0 + g + u, tot - 1);  // (past the last: cleared below)
          int j, d, js, sj;
          where(k, j, d, isw[u]);
          coords(j, d, x[u], y[u], z[u], js, sj);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          double dx, dy, dz;
          acc = (acc << 1) | (separation(x[u], y[u], z[u], isw[u], dx, dy, dz) < rn2 ? 1u : 0u);
        }
      }
      // candidate c0 in the highest bit, those past the last cleared
      acc = end > 0 ? (acc >> (g - end)) << (32 - end) : 0u;
      while (acc != 0) {
        const int b = __clz((int)acc);
        acc &= ~(0x80000000u >> b);
        int j, d, js, sj;
        bool isw;
        double x, y, z, dx, dy, dz;
        where(c0 + b, j, d, isw);
        coords(j, d, x, y, z, js, sj);
        if (own && js == i) continue;
        const double s = separation(x, y, z, isw, dx, dy, dz);
        if (build) {
          const uint32_t idx =
              d != NOSLOT ? (uint32_t)(j + d) : ((uint32_t)js | GFLAG);
          *wp = (int32_t)(idx | (isw ? cw : cyz));
          ++m;
          wp += m < mcap ? np : (size_t)0;
        }
        if (MIX) {
          const int kk = (spi * MAXSP + sj) & (MAXSP * MAXSP - 1);
          if (force && s < tab->rc2[kk]) pair_accum_mix<R>(a, dx, dy, dz, s, tab, kk, energy);
        } else if (force && s < rc2) {
          pair_accum<R>(a, dx, dy, dz, s, ushift, energy);
        }
      }
    }
  };
  auto bounds = [&](int q, int (&b)[4]) { row_bounds(CS, G, cx, cy, cz, q, b); };
  // (row 0's bounds may have been loaded by the caller, ahead of the window)
  int cur[4], nxt[4];
  if (pre0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = pre0[u];
  } else {
    bounds(0, cur);
  }
#pragma unroll 1
  for (int q = 0; q < 9; ++q) {
    if (q < 8) bounds(q + 1, nxt);
    uint32_t iz, iy;
    wrap_cell(cz + q / 3 - 1, G, &iz);
    wrap_cell(cy + q % 3 - 1, G, &iy);
    const double by = img_shift(iy, L), bz = img_shift(iz, L);
    const uint32_t cyz = ((iy << 2) | (iz << 4)) << J_BITS;
    int dm = NOSLOT, d0 = NOSLOT, dg = NOSLOT;
    if (whole) {
      dm = d0 = dg = 0;
    } else if (rows) {
      const int e = 3 * (sr * 9 + q);
      dm = w.dl[e];
      d0 = w.dl[e + 1];
      dg = w.dl[e + 2];
    }
    const int dw = wlo ? dg : d0;
    if (anyedge)
      row(std::true_type{}, q == 4, cur[0], cur[1], dm, cur[2], cur[3], dw, cyz, by, bz);
    else
      row(std::false_type{}, q == 4, cur[0], cur[1], dm, 0, 0, 0, cyz, by, bz);
#pragma unroll
    for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
  }
  return m;
}

// 27-cell traversal over the sorted atoms, first half (offsets z-major, x
// fastest; ascending storage index within a cell, which is ascending index
// before the sort): emit(entry) for every candidate whose packed position is
// near enough to atom i's, in order, entry being its list entry (window slot
// of its row piece, or storage index with GFLAG; image code).  The three
// cells of an x-row are one contiguous range of storage indices unless the
// row wraps (a lane at an x-edge of the box), where it is two, taken in x
// order.
// What bounds a rebuild step is VALU issue and the waits of its dependent
// chains: the full test is 9 FP64 operations on three 8-byte coordinates, a
// wave runs ~135 of them per lane for the ~77 candidates a lane has, and the
// accept path (list store, pair arithmetic) ran for every candidate that any
// lane accepted.  Packed, a candidate is one 8-byte load, four operations and
// a compare, without image shifts or a choice of where its piece lives; the
// exact test runs for the ~12 per lane that pass, together with the pair
// arithmetic, over the finished list.  Evaluation with a build, N = 256 000:
// 63.0 -> 54.5 us, VALU instructions per wave 6 143 -> 4 325; the FP64 cell
// method at N = 2 048 41.5 -> 35.0 us per step.  Eight loads at a time instead
// of four (and the shorter mod3): 200 steps of 864 atoms 2 334 -> 2 250 us,
// 1 000 of 4e6 345.7 -> 340.9 ms, 200 of 110 592 LJ atoms 15.14 -> 14.95 ms.
// EDGE: some lane of the wave is at an x-edge of the box; the other waves skip
// the choice between the two ranges.
template <bool EDGE, class Emit>
__device__ __forceinline__ void near_rows(SlotC &S, int i, int ci, const Window &w, const pk_t *pk,
                                          const int (&pre0)[4], Emit &&emit) {
  const int G = S.G;
  const uint32_t lim = S.pk_lim;
  // 32-bit byte offsets from uniform bases
  typedef const __attribute__((address_space(1))) char *gcchar;
  const gcchar CS = (gcchar)gp((const int32_t *)S.cs), PK = (gcchar)gp(pk);
  auto cs_at = [&](int c) { return *(gcint)(CS + (uint32_t)(4 * c)); };
  const int cx = ci % G, cy = (ci / G) % G, cz = ci / (G * G);
  const bool whole = w.whole, rows = !whole && w.wt[0] >= 0;
  const int sr = rows ? ci / G - w.rf : 0;  // source row of the atom within the tile
  const pk_t me = *(gcpk)(PK + (uint32_t)(8 * i));
  // a lane at an x-edge visits the wrapped cell first when cx = 0 (cell G-1),
  // last when cx = G-1 (cell 0)
  const bool wlo = EDGE && cx == 0, edge = EDGE && (cx == 0 || cx == G - 1);
  const uint32_t cxw = (wlo ? 1u : 3u) << J_BITS;
  const int xm0 = max(cx - 1, 0), xm1 = min(cx + 2, G), xe = cx == 0 ? G - 1 : 0;
  // the cells of a row start at plane + yrow[dy + 1]
  int yrow[3];
  uint32_t ycode[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    yrow[d] = wrap_cell(cy + d - 1, G, &ycode[d]) * G;
    ycode[d] <<= J_BITS + 2;
  }
  uint32_t zc;
  int plane = wrap_cell(cz - 1, G, &zc) * G * G;
  int cur[4], nxt[4] = {0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < 4; ++u) cur[u] = pre0[u];
#pragma unroll 1
  for (int pz = 0; pz < 3; ++pz) {
    const uint32_t zcode = zc << (J_BITS + 4);
    const int next_plane = wrap_cell(cz + pz, G, &zc) * G * G;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      // the next row's bounds are loaded before this one is visited
      if (d < 2 || pz < 2) {
        const int row = d < 2 ? plane + yrow[d < 2 ? d + 1 : 0] : next_plane + yrow[0];
        nxt[0] = cs_at(row + xm0);
        nxt[1] = cs_at(row + xm1);
        if (EDGE) {
          nxt[2] = cs_at(row + xe);
          nxt[3] = cs_at(row + xe + 1);
        }
      }
      const uint32_t cyz = ycode[d] | zcode;
      int dm = NOSLOT, dw = NOSLOT;
      if (whole) {
        dm = dw = 0;
      } else if (rows) {
        const int e = 3 * (sr * 9 + 3 * pz + d);
        dm = w.dl[e];
        if (EDGE) dw = w.dl[e + (wlo ? 2 : 1)];
      }
      // candidates k = 0 .. tot-1: the first range (k < lenF), then the
      // second; candidate k of a range is atom lo + k, its entry e + k
      int loF = cur[0], lenF = cur[1] - cur[0], tot = lenF, loS = 0;
      uint32_t eF = (dm == NOSLOT ? (uint32_t)cur[0] | GFLAG : (uint32_t)(cur[0] + dm)) | cyz,
               eS = 0;
      int self = pz == 1 && d == 1 ? i - cur[0] : -1;
      if (EDGE) {
        const int lenM = lenF, lenW = edge ? cur[3] - cur[2] : 0;
        const uint32_t eM = eF, eW = (dw == NOSLOT ? (uint32_t)cur[2] | GFLAG
                                                   : (uint32_t)(cur[2] + dw)) | cyz | cxw;
        tot += lenW;
        lenF = wlo ? lenW : lenM;
        loF = wlo ? cur[2] : cur[0];
        loS = (wlo ? cur[0] : cur[2]) - lenF;
        eF = wlo ? eW : eM;
        eS = (wlo ? eM : eW) - (uint32_t)lenF;
        if (self >= 0 && wlo) self += lenW;
      }
      for (int c0 = 0; __ballot(c0 < tot) != 0; c0 += 32) {
        // one bit per candidate c0 .. c0+31, the first in the highest (a
        // group may read past its range: the array has the room, and the
        // extra bits are dropped)
        auto test = [&](int lo, int k, int end) {
          uint32_t acc = 0;
          const int cnt = end - k;
          uint32_t off = 8u * (uint32_t)(lo + k);
          for (int g = 0; g < cnt; g += PK_GROUP, off += 8 * PK_GROUP) {
            pk_t c[PK_GROUP];
#pragma unroll
            for (int u = 0; u < PK_GROUP; ++u) c[u] = *(gcpk)(PK + off + 8 * u);
#pragma unroll
            for (int u = 0; u < PK_GROUP; ++u)
              acc = (acc << 1) | (pk_dist2(me, c[u]) <= lim ? 1u : 0u);
          }
          return cnt > 0 ? acc >> (-cnt & (PK_GROUP - 1)) : 0u;
        };
        const int end = min(tot, c0 + 32);
        uint32_t acc = test(loF, c0, EDGE ? min(lenF, end) : end);
        if (EDGE) {
          const int k2 = max(lenF, c0);
          const uint32_t acc2 = test(loS, k2, end);
          if (k2 < end) acc = (acc << ((end - k2) & 31)) | acc2;  // (32 only after none)
        }
        if (end <= c0) continue;
        // candidate c0 + b in bit b
        acc = __brev(acc << (32 - (end - c0)));
        if (pz == 1 && d == 1 && self >= c0 && self < c0 + 32) acc &= ~(1u << (self - c0));
        while (acc != 0) {
          const int k = c0 + __ffs((int)acc) - 1;
          acc &= acc - 1;
          emit((EDGE && k >= lenF ? eS : eF) + (uint32_t)k);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) cur[u] = nxt[u];
    }
    plane = next_plane;
  }
}
template <class Emit>
__device__ __forceinline__ void near_atoms(SlotC &S, int i, int ci, const Window &w,
                                           const pk_t *pk, const int (&pre0)[4], Emit &&emit) {
  const int cx = ci % S.G;
  if (__ballot(cx == 0 || cx == S.G - 1) != 0)
    near_rows<true>(S, i, ci, w, pk, pre0, emit);
  else
    near_rows<false>(S, i, ci, w, pk, pre0, emit);
}

// Coordinates of neighbour-list entry e: from the LDS window, or from
// global memory when the entry carries a storage index.
template <bool MIX, bool COH>
__device__ __forceinline__ void entry_pos(uint32_t e, gcdouble X, gcdouble Y, gcdouble Z,
                                          const double *sx, const double *sy, const double *sz,
                                          double &xj, double &yj, double &zj, gcint SP,
                                          const int8_t *ssp, int &sj) {
  const uint32_t idx = e & IDX_MASK;
  if (e & GFLAG) {
    xj = ld<COH>(&X[idx]);
    yj = ld<COH>(&Y[idx]);
    zj = ld<COH>(&Z[idx]);
    if (MIX) sj = ld<COH>(&SP[idx]);
  } else {
    xj = sx[idx];
    yj = sy[idx];
    zj = sz[idx];
    if (MIX) sj = ssp[idx];
  }
}

// One neighbour-list entry e (index + image code) of atom i, counted when ok.
// SHIFT = false when no entry of the wave's current group carries an image
// code.
// MIX: kk = the species pair (masked into the table: a masked-off entry may
// carry any species byte).
template <typename R, bool SHIFT, bool MIX>
__device__ __forceinline__ void list_pair(Acc<R> &a, bool ok, uint32_t e, double xi, double yi,
                                          double zi, double xj, double yj, double zj, double L,
                                          double rc2, R ushift, bool energy, int kk,
                                          const PairTab *tab) {
  double dx = xi - xj, dy = yi - yj, dz = zi - zj;
  if (SHIFT) {
    // each 2-bit field sign-extended is the multiple of L (exact products)
    dx = dx + (double)((int32_t)(e << (32 - J_BITS - 2)) >> 30) * L;
    dy = dy + (double)((int32_t)(e << (32 - J_BITS - 4)) >> 30) * L;
    dz = dz + (double)((int32_t)e >> 30) * L;
  }
  const double s = (dx * dx + dy * dy) + dz * dz;
  if (MIX) {
    if (ok && s < tab->rc2[kk]) pair_accum_mix<R>(a, dx, dy, dz, s, tab, kk, energy);
  } else if (ok && s < rc2) {
    pair_accum<R>(a, dx, dy, dz, s, ushift, energy);
  }
}

// Four entries q0 .. q0+3 of an atom's list of m (their coordinate reads
// together).  A group without image codes anywhere in the wave skips the
// shifts.
// PRE: they are among the first NP, whose coordinates outside the window have
// been gathered into g*.
struct Four {
  uint32_t e[4];
};
template <typename R, bool MIX, bool COH, bool PRE, int NP>
__device__ __forceinline__ void list_group(Acc<R> &a, int q0, int m, Four f, gcdouble X,
                                           gcdouble Y, gcdouble Z, const double *sx,
                                           const double *sy, const double *sz, double xi, double yi,
                                           double zi, double L, double rc2, R ushift, bool energy,
                                           const PairTab *tab, int spi, gcint SP,
                                           const int8_t *ssp, const double *gx, const double *gy,
                                           const double *gz, const int *gs) {
  bool ok[4];
  uint32_t eg[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    ok[u] = q0 + u < m;
    eg[u] = ok[u] ? f.e[u] : 0u;
  }
  const uint32_t any = (eg[0] | eg[1]) | (eg[2] | eg[3]);
  double xj[4], yj[4], zj[4];
  int sj[4] = {0, 0, 0, 0};
  if (__ballot((any & GFLAG) != 0) == 0) {
    // the usual case: every entry of the wave is a window slot
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t sl = eg[u] & IDX_MASK;
      xj[u] = sx[sl];
      yj[u] = sy[sl];
      zj[u] = sz[sl];
      if (MIX) sj[u] = ssp[sl];
    }
  } else if constexpr (PRE) {
    // window slots from LDS (slot 0 for an entry outside it), the others from
    // the gathered coordinates
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool g = (eg[u] & GFLAG) != 0;
      const uint32_t sl = g ? 0u : eg[u] & IDX_MASK;
      const int qu = q0 + u < NP ? q0 + u : NP - 1;
      xj[u] = g ? gx[qu] : sx[sl];
      yj[u] = g ? gy[qu] : sy[sl];
      zj[u] = g ? gz[qu] : sz[sl];
      if (MIX) sj[u] = g ? gs[qu] : ssp[sl];
    }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      entry_pos<MIX, COH>(eg[u], X, Y, Z, sx, sy, sz, xj[u], yj[u], zj[u], SP, ssp, sj[u]);
  }
  auto kk = [&](int u) { return (spi * MAXSP + sj[u]) & (MAXSP * MAXSP - 1); };
  if (__ballot((any >> J_BITS) != 0) == 0) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      list_pair<R, false, MIX>(a, ok[u], eg[u], xi, yi, zi, xj[u], yj[u], zj[u], L, rc2, ushift,
                               energy, kk(u), tab);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      list_pair<R, true, MIX>(a, ok[u], eg[u], xi, yi, zi, xj[u], yj[u], zj[u], L, rc2, ushift,
                              energy, kk(u), tab);
  }
}

// Whether the storage of the state that step k (or a host evaluation at
// the held state k) works on is not the cell order of the last sort: always
// without reordering, else after a rebuild that kept the storage order
// (CtlDev::rb_ring) and until the next reordering (CtlDev::ord_ring).  The
// words are read through the constant view (written by earlier launches), so
// the test can be made again wherever it is needed instead of held.
template <class Ctl>
__device__ __forceinline__ bool unordered(SlotC &S, const Ctl &C, int64_t k, int mode) {
  if (S.noreo) return true;
  if (mode != MODE_STEP) return C.ord_ring[mod3(k)] != 0;
  const int rb = C.rb_ring[mod3(k)];
  return rb != RB_NONE ? rb == RB_PERM : C.ord_ring[mod3(k - 1)] != 0;
}

// ACC: the steps of a block, which sum their properties and add them to the
// block sums.  MIX: a mixture (species staged with the window, pair
// parameters in LDS).
// pub: thread TILE - 64 stores pubv there before the tile's last barrier
// (the step kernel's next tile, published to the workgroup without a
// barrier of its own).
// COH: a cell step of k_run (other workgroups of this launch wrote r(k); see
// ld).
// unord(): whether the atoms are not in cell order (asked again where needed
// instead of held).  si: index of the step in the replay.
// A counter of arrivals at barriers of k_run carries this bit once one of the
// workgroups that count there has latched an error; set before the workgroup's
// next arrival.
constexpr int RUN_BAD = 1 << 29;
__device__ __forceinline__ void bring_error(int32_t *counter) {
  __hip_atomic_fetch_or(counter, RUN_BAD, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool MIX>
struct StepLds {
  // 4 slots of padding: a group of candidates may read up to 3 slots past the
  // window's last
  double sx[WCAP + 4], sy[WCAP + 4], sz[WCAP + 4];
  Window win;
  // a mixture: the pair table and the window's species
  typename std::conditional<MIX, PairTab, char>::type tab;
  int8_t ssp[MIX ? WCAP + 4 : 1];
  unsigned long long sv[4];
  double sh[4][8];
  int32_t *call;  // k_run: this workgroup's counter of arrivals at barriers
};
// The end of a tile's step: (d), (e) and the next (a) -- x and v become those
// of the next step -- the binning of r(k+1) where bin_next, the clearing of
// the set after next (clear), and the tile's maximum speed and properties.
// put_v: v goes to memory (k_run keeps it in registers from step to step).
template <typename R, bool ACC, bool COH, class Lds>
__device__ __forceinline__ void finish_tile(SlotC &S, CtlDev &C, Lds &lds, int lt, int64_t k,
                                            int mode, bool last, bool bin_next, bool clear,
                                            bool put_v, double (&x)[3], double (&v)[3],
                                            const Acc<R> &a, int m, int si, int *pub, int pubv) {
  const int tid = tid_here();
  // (d), (e) and the next (a)
  const int i = lt * TILE + tid;
  const bool act = i < S.n, force = mode != MODE_BUILD;
  const int pb = (int)(k & 1);
  double vv = 0.0;
  if (act && force) {
    const double f[3] = {(double)a.fx, (double)a.fy, (double)a.fz};
    if (mode == MODE_STEP)
      for (int q = 0; q < 3; ++q) v[q] = v[q] + S.hdt * f[q];  // (d)
    vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];            // (e)
    if (mode == MODE_STEP) {
      if (!last) {
        double xn[3];
        for (int q = 0; q < 3; ++q) {
          v[q] = v[q] + S.hdt * f[q];  // (a) of step k+1
          xn[q] = x[q] + S.dt * v[q];
          // streaming stores: the next step's kernels read these from
          // any XCD, so they are not kept in this XCD's L2 (less for its
          // write-back when the kernel ends)
          x[q] = xn[q];
          if (COH)
            st<true>(&gp(S.P[pb ^ 1][q])[i], xn[q]);
          else
            __builtin_nontemporal_store(xn[q], &gp(S.P[pb ^ 1][q])[i]);
        }
        const int bad =
            bin_next ? bin_atom<COH>(S, C, (int)mod3(k + 1), i, xn[0], xn[1], xn[2], k + 1)
                     : check_atom(S, C, xn[0], xn[1], xn[2], k + 1);
        if (COH && bad) bring_error(lds.call);
      }
      if (put_v)
        for (int q = 0; q < 3; ++q) {
          if (COH)
            st<true>(&gp(S.V[pb ^ 1][q])[i], v[q]);
          else
            __builtin_nontemporal_store(v[q], &gp(S.V[pb ^ 1][q])[i]);
        }
    }
    if (mode != MODE_STEP || last) {
      auto F = gp((R *)S.F);
      F[i] = a.fx;
      F[S.npad + i] = a.fy;
      F[2 * S.npad + i] = a.fz;
      auto U = gp((R *)S.UA);
      U[i] = a.u;
      U[S.npad + i] = a.w;
    }
  }

  // the set after next is cleared for the binning of step k+2
  if (mode == MODE_STEP && clear) {
    const int zs = (int)mod3(k + 2);
    const int c0 = lt * S.cpt, c1 = min(c0 + S.cpt, S.ncell);
    for (int c = c0 + tid; c < c1; c += TILE) st<COH>(&gp(S.cnt[zs])[c], 0);
    for (int q = lt * TILE + tid; q < S.nctiles; q += S.ntiles * TILE)
      st<COH>(&gp(S.tcnt[zs])[q], 0);
    if (lt == 0 && tid == 0) st<COH>(&gp(S.ovf_n)[zs], 0);
  }

  // the maximum speed of the step (the rebuild rule needs it every step):
  // v^2 >= 0, so its bit pattern orders like the value
  auto &sv = lds.sv;
  const int w = tid >> 6, l = tid & 63;
  const unsigned long long vbits = wave_max_u64((unsigned long long)__double_as_longlong(vv));
  if (l == 0) sv[w] = vbits;
  // the other properties only where somebody reads them: the last step of a
  // run, evaluations of a held state, and the steps of a block
  const bool full = mode != MODE_STEP || last || ACC;
  auto &sh = lds.sh;
  if (full) {
    const int mm = act && !S.cell_only ? m : 0;
    const double ke = wave_sum(vv);
    const double sm = wave_sum((double)mm);
    const int mmax = wave_max_i(mm);
    double pe_hi, pe_lo, vr_hi, vr_lo;
    if (sizeof(R) == 8) {
      pe_hi = wave_sum((double)a.u);
      vr_hi = wave_sum((double)a.w);
      pe_lo = vr_lo = 0.0;
    } else {
      F2 pe = wave_sum_f2(F2{(float)a.u, 0.0f});
      F2 vr = wave_sum_f2(F2{(float)a.w, 0.0f});
      pe_hi = pe.hi;
      pe_lo = pe.lo;
      vr_hi = vr.hi;
      vr_lo = vr.lo;
    }
    if (l == 0) {
      sh[w][0] = ke;
      sh[w][2] = pe_hi;
      sh[w][3] = pe_lo;
      sh[w][4] = vr_hi;
      sh[w][5] = vr_lo;
      sh[w][6] = sm;
      sh[w][7] = (double)mmax;
    }
  }
  __syncthreads();
  if (tid == 0) {
    const unsigned long long b01 = sv[0] > sv[1] ? sv[0] : sv[1];
    const unsigned long long b23 = sv[2] > sv[3] ? sv[2] : sv[3];
    const unsigned long long vmb = b01 > b23 ? b01 : b23;
    // one atomic per workgroup, spread over VSPREAD cache lines
    if (force) atomicMax(&S.vring[(mod3(k) * VSPREAD + (lt & (VSPREAD - 1))) * 16], vmb);
    if (full) {
      auto q = gp(S.part) + (size_t)lt * NPART;
      if (force) {
        q[0] = ((sh[0][0] + sh[1][0]) + sh[2][0]) + sh[3][0];
        q[1] = __longlong_as_double((long long)vmb);
        if (sizeof(R) == 8) {
          q[2] = ((sh[0][2] + sh[1][2]) + sh[2][2]) + sh[3][2];
          q[3] = 0.0;
          q[4] = ((sh[0][4] + sh[1][4]) + sh[2][4]) + sh[3][4];
          q[5] = 0.0;
        } else {
          F2 e{(float)sh[0][2], (float)sh[0][3]}, v2{(float)sh[0][4], (float)sh[0][5]};
          for (int k2 = 1; k2 < 4; ++k2) {
            e = f2_add(e, F2{(float)sh[k2][2], (float)sh[k2][3]});
            v2 = f2_add(v2, F2{(float)sh[k2][4], (float)sh[k2][5]});
          }
          q[2] = e.hi;
          q[3] = e.lo;
          q[4] = v2.hi;
          q[5] = v2.lo;
        }
      }
      q[6] = ((sh[0][6] + sh[1][6]) + sh[2][6]) + sh[3][6];
      q[7] = fmax(fmax(sh[0][7], sh[1][7]), fmax(sh[2][7], sh[3][7]));
      if (ACC && mode == MODE_STEP) {
        // this tile's part of the block sums (the tile's atoms change at a
        // sort, the total over tiles does not)
        auto A = gp(S.acc) + (size_t)lt * NACC;
        A[0] = A[0] + q[0];
        A[1] = A[1] + (q[2] + q[3]);
        A[2] = A[2] + (q[4] + q[5]);
        A[3] = A[3] + q[6];
        if (S.tpart) {
          // a traced replica: this step's tile partials, reduced by k_trace
          // at the end of the replay
          auto Q = gp(S.tpart) + ((size_t)si * S.ntiles + lt) * 4;
          Q[0] = q[0];
          Q[1] = q[2] + q[3];
          Q[2] = q[4] + q[5];
          Q[3] = q[1];
        }
      }
    }
  }
  if (pub != nullptr && tid == TILE - 64) *pub = pubv;
  __syncthreads();
}

template <typename R, bool ACC, bool MIX, bool COH, class Unord>
__device__ __forceinline__ void step_tile(SlotC &S, CtlDev &C, StepLds<MIX> &lds, int lt, int64_t k,
                                          int mode, bool cells, bool build, bool last,
                                          bool bin_next, bool clear, Unord unord, int si, int *pub,
                                          int pubv) {
  const int tid = tid_here();
  double *const sx = lds.sx, *const sy = lds.sy, *const sz = lds.sz;
  Window &win = lds.win;
  const int i = lt * TILE + tid;
  const bool act = i < S.n;
  const int pb = (int)(k & 1);
  const int vb = mode == MODE_STEP ? pb : pb ^ 1;  // v(k-1/2) during a run, v(k) when clean
  const gcdouble X = gp((const double *)S.P[pb][0]);
  const gcdouble Y = gp((const double *)S.P[pb][1]);
  const gcdouble Z = gp((const double *)S.P[pb][2]);
  const bool force = mode != MODE_BUILD;
  const double L = S.L;

  // loads that do not wait for the window: own position and velocity, list
  // length and the first NE list entries (or the own cell when sorted).
  // Velocities, list lengths and these entries are read once a step:
  // streaming (non-temporal) loads, so they do not displace the window data
  // that neighbouring tiles read again from the caches.  (Entries past the
  // first NE, the bulk of a long list such as LJ r_c = 3's, are read plainly:
  // such lists stay in the last-level cache from step to step.)
  constexpr int NE = sizeof(R) == 8 ? 8 : 12;
  if constexpr (COH) cells = true;  // (k_run's list steps are own_step's)
  const bool list = !COH && !cells && force;
  const auto Wc = gp((const int32_t *)S.W) + i;
  const size_t np = (size_t)S.npad;
  double xi = 0, yi = 0, zi = 0, v[3] = {0.0, 0.0, 0.0};
  int m = 0, ci = 0;
  uint32_t e[NE];
  // the window table first: the staging waits for it, not for the rest
  int wtv = 0;
  if (list && tid < WSTRIDE) wtv = gp((const int32_t *)S.win)[lt * WSTRIDE + tid];
  if (act) {
    xi = ld<COH>(&X[i]);
    yi = ld<COH>(&Y[i]);
    zi = ld<COH>(&Z[i]);
    if (force)
      for (int q = 0; q < 3; ++q)
        v[q] = COH ? ld<COH>(&gp((const double *)S.V[vb][q])[i])
                   : __builtin_nontemporal_load(&gp(S.V[vb][q])[i]);
    if (list) {
      m = __builtin_nontemporal_load(&gp(S.m)[i]);
#pragma unroll
      for (int u = 0; u < NE; ++u)
        e[u] = u < S.mcap ? (uint32_t)__builtin_nontemporal_load(&Wc[(size_t)u * np]) : 0u;
    } else if (cells) {
      ci = ld<COH>(&gp((const int32_t *)S.cell)[i]);
    }
  }

  const PairTab *tab = nullptr;
  int8_t *ssp = nullptr;
  const gcint SP = gp((const int32_t *)S.sp);
  int spi = 0;
  if constexpr (MIX) {
    tab = &lds.tab;
    ssp = lds.ssp;
    constexpr int NT = (int)(sizeof(PairTab) / sizeof(double));
    if (tid < NT)
      ((double *)&lds.tab)[tid] = gp((const double *)S.tab)[tid];
    if (act) spi = ld<COH>(&SP[i]);
  }
  // a cell step: the bounds of the first neighbour row of the traversal go
  // out before the window is built (wave 0 builds it; the others wait)
  int b0[4] = {0, 0, 0, 0};
  if (cells && act) {
    const int G = S.G;
    row_bounds(gp((const int32_t *)S.cs), G, ci % G, (ci / G) % G, ci / (G * G), 0, b0);
  }
  if (cells && unord()) {
    // no reordering: the tile's atoms are not a run of cells, so there is no
    // window; candidates are read from global memory through perm, and the
    // list steps until the next sort stage nothing
    if (tid == 0) {
      win.wt[0] = -1;
      win.whole = 0;
      win.rf = 0;
      gp(S.win)[(size_t)lt * WSTRIDE] = -1;
    }
    __syncthreads();
  } else if (cells) {
    make_window(S, lt, win, (int *)sx);
  } else if (list) {
    if (tid < WSTRIDE) win.wt[tid] = wtv;
    __syncthreads();
  }
  // a cell step over atoms in cell order: which candidates are near comes from
  // their packed positions, while the window's loads are in flight
  const bool near = cells && S.pk_lim != 0 && !unord();
  if (cells) stage_window<MIX, COH>(win.wt, X, Y, Z, sx, sy, sz, SP, ssp);
  int mr = 0;
  if (near && build && act) {
    // the list with its few entries that are only nearly near; an atom with
    // more than mcap of them (its list may overflow) is done again below
    const int mcap = S.mcap;
    auto wp = gp(S.W) + i;
    near_atoms(S, i, ci, win, pk_array(S, k), b0, [&](uint32_t e1) {
      *wp = (int32_t)e1;
      ++mr;
      wp += mr < mcap ? np : (size_t)0;
    });
  }
  // The first NP entries that live outside the window: their coordinates
  // are gathered now, while the window is staged, instead of inside the
  // pair loop (by the waves that have such entries; only a group holding
  // one reads them).
  constexpr int NP = 8;  // (all NE = 12 of FP32 forces: more registers, spills)
  double gx[NP], gy[NP], gz[NP];
  int gs[NP];
  uint32_t gor = 0;
  if (list && act && m <= S.mcap)
    for (int u = 0; u < NP; ++u) gor |= u < m ? e[u] : 0u;
  if (__ballot((gor & GFLAG) != 0) != 0) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      gx[u] = gy[u] = gz[u] = 0.0;
      gs[u] = 0;
      if (u < m && (e[u] & GFLAG) && m <= S.mcap && act) {
        const uint32_t idx = e[u] & IDX_MASK;
        gx[u] = ld<COH>(&X[idx]);
        gy[u] = ld<COH>(&Y[idx]);
        gz[u] = ld<COH>(&Z[idx]);
        if (MIX) gs[u] = ld<COH>(&SP[idx]);
      }
    }
  }
  if (list) stage_window<MIX, COH>(win.wt, X, Y, Z, sx, sy, sz, SP, ssp);
  if (cells || list) __syncthreads();

  Acc<R> a{(R)0, (R)0, (R)0, (R)0, (R)0};
  if (act) {
    if (near && (!build || mr <= S.mcap)) {
      // exact test, force, and the list closed up over the entries that fail
      const double rn2 = S.rn2, rc2 = S.rc2;
      const R ushift = (R)S.ushift;
      const bool energy = mode != MODE_STEP || last || ACC;
      auto pair = [&](uint32_t e1, double xj, double yj, double zj, int sj) {
        // each 2-bit field sign-extended is the multiple of L (exact products)
        const double dx = xi - xj + (double)((int32_t)(e1 << (32 - J_BITS - 2)) >> 30) * L;
        const double dy = yi - yj + (double)((int32_t)(e1 << (32 - J_BITS - 4)) >> 30) * L;
        const double dz = zi - zj + (double)((int32_t)e1 >> 30) * L;
        const double s2 = (dx * dx + dy * dy) + dz * dz;
        if (!(s2 < rn2)) return false;
        if (MIX) {
          const int kk = (spi * MAXSP + sj) & (MAXSP * MAXSP - 1);
          if (force && s2 < tab->rc2[kk]) pair_accum_mix<R>(a, dx, dy, dz, s2, tab, kk, energy);
        } else if (force && s2 < rc2) {
          pair_accum<R>(a, dx, dy, dz, s2, ushift, energy);
        }
        return true;
      };
      if (build) {
        const auto Wb = gp(S.W) + i;
        uint32_t en[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) en[u] = u < mr ? (uint32_t)Wb[(size_t)u * np] : 0u;
        for (int q = 0; __ballot(q < mr) != 0; q += 4) {
          uint32_t eg[4];
          double xj[4], yj[4], zj[4];
          int sj[4] = {0, 0, 0, 0};
#pragma unroll
          for (int u = 0; u < 4; ++u) eg[u] = en[u];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            en[u] = q + 4 + u < mr ? (uint32_t)Wb[(size_t)(q + 4 + u) * np] : 0u;
          if (__ballot((((eg[0] | eg[1]) | (eg[2] | eg[3])) & GFLAG) != 0) == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t sl = eg[u] & IDX_MASK;
              xj[u] = sx[sl];
              yj[u] = sy[sl];
              zj[u] = sz[sl];
              if (MIX) sj[u] = ssp[sl];
            }
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              entry_pos<MIX, COH>(eg[u], X, Y, Z, sx, sy, sz, xj[u], yj[u], zj[u], SP, ssp, sj[u]);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (q + u < mr && pair(eg[u], xj[u], yj[u], zj[u], sj[u])) {
              if (m != q + u) Wb[(size_t)m * np] = (int32_t)eg[u];
              ++m;
            }
        }
        gp(S.m)[i] = m;
      } else {
        near_atoms(S, i, ci, win, pk_array(S, k), b0, [&](uint32_t e1) {
          double xj, yj, zj;
          int sj = 0;
          entry_pos<MIX, COH>(e1, X, Y, Z, sx, sy, sz, xj, yj, zj, SP, ssp, sj);
          (void)pair(e1, xj, yj, zj, sj);
        });
      }
    } else if (cells) {
      m = traverse_sorted<R, MIX, COH>(S, i, ci, X, Y, Z, win, sx, sy, sz, xi, yi, zi, build, force,
                                  mode != MODE_STEP || last || ACC, a, ssp, SP, spi, tab,
                                  unord(), false, b0);
      if (build) gp(S.m)[i] = m;
    } else if (list) {
      if (m <= S.mcap) {
        const double rc2 = S.rc2;
        const R ushift = (R)S.ushift;
        // entries in order, four at a time, for as long as any lane of the wave
        // has some left: a lane past its length takes the group with no effect,
        // so the wave runs max(m)/4 groups whatever the spread of m
        auto group = [&](auto pre, auto en, int q0, uint32_t e0, uint32_t e1, uint32_t e2,
                         uint32_t e3) {
          list_group<R, MIX, COH, decltype(pre)::value, NP>(
              a, q0, m, {e0, e1, e2, e3}, X, Y, Z, sx, sy, sz, xi, yi, zi, L, rc2, ushift,
              decltype(en)::value, tab, spi, SP, ssp, gx, gy, gz, gs);
        };
        auto rest = [&](auto en, int q) {
          for (; __ballot(q < m) != 0; q += 4) {
            uint32_t ew[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
              ew[u] = q + u < m ? (uint32_t)Wc[(size_t)(q + u) * np] : 0u;
            group(std::false_type{}, en, q, ew[0], ew[1], ew[2], ew[3]);
          }
        };
        // (outside a block few steps sum energies: they read their entries
        // again, so that the loaded ones need one loop)
        if (!ACC && (mode != MODE_STEP || last)) {
          rest(std::true_type{}, 0);
        } else {
          constexpr std::bool_constant<ACC> en{};
#pragma unroll
          for (int g = 0; g < NP / 4; ++g)
            if (__ballot(4 * g < m) != 0)
              group(std::true_type{}, en, 4 * g, e[4 * g], e[4 * g + 1], e[4 * g + 2],
                    e[4 * g + 3]);
#pragma unroll
          for (int g = NP / 4; g < NE / 4; ++g)
            if (__ballot(4 * g < m) != 0)
              group(std::false_type{}, en, 4 * g, e[4 * g], e[4 * g + 1], e[4 * g + 2],
                    e[4 * g + 3]);
          rest(en, NE);
        }
      } else {
        // the list overflowed its capacity at the last build: evaluate this
        // atom over the 27 cells of its cell at that sort, with the positions
        // of now (exact: an atom within r_c now was within r_n then, since
        // neither moved more than delta/2), reading them from global memory
        traverse_sorted<R, MIX, COH>(S, i, gp(S.cell)[i], X, Y, Z, win, sx, sy, sz, xi, yi, zi,
                                false, true, mode != MODE_STEP || last || ACC, a, ssp, SP, spi,
                                tab, unord(), true);
      }
    }
  }

  double x[3] = {xi, yi, zi};
  finish_tile<R, ACC, COH>(S, C, lds, lt, k, mode, last, bin_next, clear, true, x, v, a, m, si, pub,
                           pubv);
}

// A tile that stays with its workgroup from step to step (k_run with one tile
// per workgroup): an atom's position, velocity, list length and first NR list
// entries are held in registers, the window's intervals (and a mixture's
// species and pair table) in LDS, so a list step only reads its window.
template <typename R>
struct Own {
  static constexpr int NR = sizeof(R) == 8 ? 12 : 20;
  double x[3], v[3];
  int m, sp;
  uint32_t e[NR];
};
// State k of tile lt after a build (or at the start of a launch).
template <typename R, bool MIX>
__device__ __forceinline__ void own_load(SlotC &S, StepLds<MIX> &lds, int lt, int64_t k,
                                         Own<R> &o) {
  const int tid = tid_here(), i = lt * TILE + tid, pb = (int)(k & 1);
  const auto W = gp((const int32_t *)S.W) + i;
  const size_t np = (size_t)S.npad;
  if (tid < WSTRIDE) lds.win.wt[tid] = gp((const int32_t *)S.win)[lt * WSTRIDE + tid];
  if constexpr (MIX) {
    constexpr int NT = (int)(sizeof(PairTab) / sizeof(double));
    if (tid < NT) ((double *)&lds.tab)[tid] = gp((const double *)S.tab)[tid];
  }
  o.m = o.sp = 0;
#pragma unroll
  for (int q = 0; q < 3; ++q) o.x[q] = o.v[q] = 0.0;
#pragma unroll
  for (int u = 0; u < Own<R>::NR; ++u) o.e[u] = 0u;
  if (i < S.n) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      o.x[q] = ld<true>(&gp((const double *)S.P[pb][q])[i]);
      o.v[q] = ld<true>(&gp((const double *)S.V[pb][q])[i]);
    }
    o.m = gp((const int32_t *)S.m)[i];
    if (MIX) o.sp = ld<true>(&gp((const int32_t *)S.sp)[i]);
#pragma unroll
    for (int u = 0; u < Own<R>::NR; ++u) o.e[u] = u < S.mcap ? (uint32_t)W[(size_t)u * np] : 0u;
  }
  __syncthreads();
  if constexpr (MIX) stage_species<true>(lds.win.wt, gp((const int32_t *)S.sp), lds.ssp);
}
// A list step of the held tile (the list path of step_tile, entry for entry).
template <typename R, bool ACC, bool MIX>
__device__ __forceinline__ void own_step(SlotC &S, CtlDev &C, StepLds<MIX> &lds, int lt, int64_t k,
                                         bool last, bool clear, bool unord, int si, Own<R> &o) {
  constexpr int NR = Own<R>::NR;
  const int tid = tid_here(), i = lt * TILE + tid, pb = (int)(k & 1);
  const gcdouble X = gp((const double *)S.P[pb][0]);
  const gcdouble Y = gp((const double *)S.P[pb][1]);
  const gcdouble Z = gp((const double *)S.P[pb][2]);
  const double *const sx = lds.sx, *const sy = lds.sy, *const sz = lds.sz;
  const gcint SP = gp((const int32_t *)S.sp);
  const int8_t *ssp = MIX ? lds.ssp : nullptr;
  const PairTab *tab = nullptr;
  if constexpr (MIX) tab = &lds.tab;
  // (the list stays the same from step to step: what is decoded from it would
  // be hoisted out of the step loop, 12 registers an entry, and spilled)
  asm volatile("" : "+v"(o.m), "+v"(o.sp));
#pragma unroll
  for (int u = 0; u < NR; ++u) asm volatile("" : "+v"(o.e[u]));
  stage_window<false, true>(lds.win.wt, X, Y, Z, lds.sx, lds.sy, lds.sz, SP, nullptr);
  __syncthreads();
  Acc<R> a{(R)0, (R)0, (R)0, (R)0, (R)0};
  const bool energy = last || ACC;
  if (i < S.n) {
    const double L = S.L, rc2 = S.rc2;
    const R ushift = (R)S.ushift;
    const int m = o.m;
    if (m <= S.mcap) {
      const auto W = gp((const int32_t *)S.W) + i;
      const size_t np = (size_t)S.npad;
      auto group = [&](auto en, int q0, Four f) {
        list_group<R, MIX, true, false, 4>(a, q0, m, f, X, Y, Z, sx, sy, sz, o.x[0], o.x[1], o.x[2],
                                           L, rc2, ushift, decltype(en)::value, tab, o.sp, SP, ssp,
                                           nullptr, nullptr, nullptr, nullptr);
      };
      auto rest = [&](auto en, int q) {
        for (; __ballot(q < m) != 0; q += 4) {
          Four f;
#pragma unroll
          for (int u = 0; u < 4; ++u) f.e[u] = q + u < m ? (uint32_t)W[(size_t)(q + u) * np] : 0u;
          group(en, q, f);
        }
      };
      // (only a run's last step sums energies outside a block: its entries
      // are read again, so that the held ones need one loop)
      if (!ACC && last) {
        rest(std::true_type{}, 0);
      } else {
        constexpr std::bool_constant<ACC> en{};
#pragma unroll
        for (int g = 0; g < NR / 4; ++g)
          if (__ballot(4 * g < m) != 0)
            group(en, 4 * g, {o.e[4 * g], o.e[4 * g + 1], o.e[4 * g + 2], o.e[4 * g + 3]});
        rest(en, NR);
      }
    } else {
      // its list overflowed: over the 27 cells of its cell at the last sort
      traverse_sorted<R, MIX, true>(S, i, ld<true>(&gp((const int32_t *)S.cell)[i]), X, Y, Z, lds.win, sx, sy, sz, o.x[0],
                                    o.x[1], o.x[2], false, true, energy, a, ssp, SP, o.sp, tab,
                                    unord, true);
    }
  }
  finish_tile<R, ACC, true>(S, C, lds, lt, k, MODE_STEP, last, false, clear, false, o.x, o.v, a,
                            o.m, si, nullptr, 0);
}
// v(k-1/2) of the held tile to memory, where state k keeps it.
template <typename R>
__device__ __forceinline__ void own_store(SlotC &S, int lt, int64_t k, const Own<R> &o) {
  const int i = lt * TILE + tid_here();
  if (i < S.n)
#pragma unroll
    for (int q = 0; q < 3; ++q) st<true>(&gp(S.V[k & 1][q])[i], o.v[q]);
}

// ACC: every step of this launch also adds its properties to the block sums
// (a separate instantiation, so steps outside a block run the plain kernel).
// MIX: the replicas are mixtures (more LDS: three workgroups per CU).
template <typename R, bool ACC, bool MIX>
__global__ __launch_bounds__(TILE, MIX ? 3 : 4) void k_step(Tables T, int s, int mode,
                                                          int force_build, int only) {
  // what a workgroup decides per replica is launch-invariant: it is worked
  // out once for a run of consecutive tiles of one replica (every tile, for
  // a single system).  The control words used here are written by earlier
  // launches only (this launch writes other ring slots, read alongside but
  // not used, and err_step > k).
  int rc = -1, var = 0;
  int64_t k = 0;
  bool skip = true, last = false, cells = false, build = false, bin_next = false;
  // the header's words, lane l holding word l % 8: a vector load that goes
  // out with the decision's loads and is waited for only where the tile
  // loop needs it
  const int hdr_l = cview(T.hdr)[threadIdx.x & 7];
  // works out the decision for replica r; leaves skip set when the launch
  // has nothing to do for it
  auto decide = [&](int r) {
    rc = r;
    skip = true;
    SlotC &S0 = slot(T, 2 * r);
    auto &C = *cview(T.ctl + r);
    if (only >= 0 && r != only) return;
    last = false;
    if (mode == MODE_STEP) {
      // every word is read before any is tested: one round of loads where
      // tests one after another made a chain of them
      const int64_t base = C.base, target = C.target, err_step = C.err_step;
      const int32_t err = C.err, fp64 = S0.fp64, cell_only = S0.cell_only;
      const int32_t vr0 = C.var_ring[0], vr1 = C.var_ring[1], vr2 = C.var_ring[2];
      const int32_t rb0 = C.rb_ring[0], rb1 = C.rb_ring[1], rb2 = C.rb_ring[2];
      const int32_t bn0 = C.bin_ring[0], bn1 = C.bin_ring[1], bn2 = C.bin_ring[2];
      // (the empty asm takes these words at one point: left to itself the
      // compiler issued the descriptor's loads only after waiting for the
      // control words)
      asm volatile("" ::"s"(base), "s"(fp64), "s"(cell_only));
      k = base + s + 1;
      const int64_t e0 = mod3(k), e1 = mod3(k - 1);
      last = k == target;
      var = pick3(vr0, vr1, vr2, e1);
      // k_sort of this step decided, and if so gathered r(k) into the other
      // variant (or, without reordering, found the cell order in place)
      const int rb = pick3(rb0, rb1, rb2, e0);
      cells = rb != RB_NONE;
      build = cells && !cell_only;
      if (rb == RB_REORDER) var ^= 1;
      // r(k+1) is binned here if a sort at step k+1 may need its rows (the
      // rule of bins_due, evaluated by k_sort of this step)
      bin_next = pick3(bn0, bn1, bn2, e0) != 0;
      // stop at an error of an earlier step; one latched by this launch
      // (while binning r(k+1), err_step = k + 1) must not stop the others
      skip = fp64 != (sizeof(R) == 8) || k > target || (err != 0 && err_step <= k);
    } else {
      if (S0.fp64 != (sizeof(R) == 8) || !C.clean) return;
      k = C.done;
      var = C.var_ring[mod3(k)];
      build = !S0.cell_only && (force_build || mode == MODE_BUILD);
      cells = build || S0.cell_only;
      skip = C.err != 0 && C.err_step <= k;
    }
  };
  const int x = blockIdx.x & 7, nwg = gridDim.x >> 3;
  constexpr int CLAIMER = TILE - 64;
  int32_t *cnt = T.walk + 64 * x, *fin = T.walk + 64 * (8 + x);
  // one replica: decided before the tile loop (the decision needs no tile
  // table, so its loads go out with the header's); a launch with nothing to
  // step for it ends here, counting every workgroup finished if it takes
  // its tiles on demand (below)
  const bool solo = T.nslots == 1;
  if (solo) {
    decide(0);
    if (skip) {
      const int nt = __builtin_amdgcn_readlane(hdr_l, HDR_NTILES);
      if ((gridDim.x & 7) == 0 && nt > (int)gridDim.x && threadIdx.x == CLAIMER &&
          atomicAdd(fin, 1) == nwg - 1) {
        atomicExch(cnt, 0);
        atomicExch(fin, 0);
      }
      return;
    }
  }
  const int nt = __builtin_amdgcn_readlane(hdr_l, HDR_NTILES);
  const int order = __builtin_amdgcn_readlane(hdr_l, HDR_ORDER);
  const TileWalk tw(blockIdx.x, gridDim.x, nt, order);
  // A launch with more tiles than workgroups takes them on demand; the
  // others walk them statically.  On demand: workgroup group x = block & 7
  // (the XCD the block is dispatched to) owns the tiles of the static
  // walk's share of x (TileWalk); a workgroup does the first tile of its
  // static walk, then claims the next ones from the group's counter, so one
  // whose tiles ran long does fewer of them.  The claim for the next tile
  // goes out from the last wave as a tile starts (that wave waits for the
  // window build anyway, so the claim's latency hides) and is published to
  // the workgroup before the tile's last barrier.  Every workgroup counts
  // itself finished once a claim finds no tile left; the last of the group
  // resets the group's counters for the next launch.
  const bool dyn = (gridDim.x & 7) == 0 && nt > (int)gridDim.x;
  const bool slabs = order == ORDER_SLABS;
  __shared__ int s_claim[2];
  __shared__ StepLds<MIX> lds;
  // the tile after this one: the static walk's, or the claimed one (double-
  // buffered: a slot is written again only after the last barrier of the
  // next tile, which every thread passes after reading it)
  int it = 0, claim = 0;
  bool stepped = false;
  auto next = [&](int t) {
    if (!dyn) return t + tw.step;
    const int b = it & 1;
    ++it;
    if (!stepped) {
      if (threadIdx.x == CLAIMER) s_claim[b] = claim;
      __syncthreads();
    }
    const int q = nwg + s_claim[b];  // the q-th tile of group x in the walk's order
    const int u = slabs ? tw.t - (int)(blockIdx.x >> 3) + q
                        : x * nwg + q % nwg + (q / nwg) * (int)gridDim.x;
    return u < tw.end ? u : nt;
  };
  for (int t = tw.t; t < tw.end; t = next(t)) {
    stepped = false;
    if (dyn && threadIdx.x == CLAIMER) claim = atomicAdd(cnt, 1);
    const int r = solo ? 0 : cview(T.tile_rep)[t];
    if (r != rc) decide(r);
    if (skip) continue;
    CtlDev &C = T.ctl[r];
    SlotC &S = slot(T, 2 * r + var);
    const int lt = t - S.tile_off;
    if (mode == MODE_STEP && lt == 0 && threadIdx.x == 0) {
      // the one writer of these ring slots in this launch (nobody reads them
      // before the next launch)
      C.var_ring[mod3(k)] = var;
      C.ord_ring[mod3(k)] = unordered(S, *cview(&C), k, mode) ? 1 : 0;
    }
    step_tile<R, ACC, MIX, false>(
        S, C, lds, lt, k, mode, cells, build, last, bin_next, true,
        [&] { return unordered(S, *cview(&C), k, mode); }, s, dyn ? &s_claim[it & 1] : nullptr,
        claim);
    stepped = true;
    if (mode == MODE_STEP && lt == 0 && threadIdx.x < VSPREAD)
      S.vring[(mod3(k + 1) * VSPREAD + threadIdx.x) * 16] = 0ull;
  }
  if (dyn && threadIdx.x == CLAIMER && atomicAdd(fin, 1) == nwg - 1) {
    atomicExch(cnt, 0);
    atomicExch(fin, 0);
  }
}

// The step counters after K steps of a run from `base`.
__device__ __forceinline__ void end_run(CtlDev &C, int K, int64_t base, int64_t target, int err,
                                        int64_t err_step) {
  int64_t done = base + K < target ? base + K : target;
  if (err != 0) done = err_step - 1 < done ? err_step - 1 : done;
  if (done < C.done) done = C.done;
  C.done = done;
  C.base = done;
  // a replica that ran holds a drifted state unless it finished
  C.clean = (done == target && err == 0) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// several steps in one launch
// ---------------------------------------------------------------------------
// A system whose tiles all fit on the chip at once (1 024 of them, 262 144
// atoms) spends most of a step between kernels: at N = 110 592 a step of two
// launches took 25 us, 10 of them tile work.  k_run keeps its workgroups, one
// per tile, through `steps` steps and separates the steps by a barrier over
// the grid (1.5-2.4 us at 8-1 000 workgroups, against ~4 us for a kernel
// boundary and ~4.5 us for a sort launch that finds nothing to sort); the
// sort runs between two barriers of a rebuild step.
//
// Who takes part: a barrier over workgroups needs all of them running, and
// what else the GPU does is not known here (another stream, another process).
// So each launch begins with a roll call: a workgroup counts itself in, and
// the launch is committed to the workgroups present, to all of them once the
// last has come, or to those that have come when one has waited long enough
// (roll_wait).  The others find the launch committed without them and leave.
// Everybody
// who takes part is running and stays so, so every barrier completes, and
// with fewer participants than tiles each steps several.  (The spin bound of
// the barriers is a backstop: it latches ERR_STALL, and none of the launch's
// steps is counted.)
//
// What is shared: everything that another workgroup may read in the same
// launch is stored device-scope (st) and read so (ld), past the caches that
// only one XCD or CU sees.  The exceptions are the packed positions and
// cell_start, which a build reads again and again, and the cells that
// make_window reads: they are read plainly, behind a barrier that invalidates
// the caches.  A tile's list, window and sums are only touched by its own
// workgroup, the same for the whole launch.  (Plain stores with one write-back per
// XCD, by the last workgroup to arrive there, missed stores of other waves
// once in some 10^5 rebuilds.)
//
// The longest wait for the others, in ticks of the 100 MHz clock, where `here`
// of `size` have come for `steps` steps.  A system alone waits half as long as
// the launch would lose by going on with those (a step is 12 us or more and
// takes size / here times as long), and 50 us, as long as the workgroups take
// to be dispatched: what fills the chip now is mostly another such launch, and
// when that ends the rest come.  With a wait of 100 us for whoever had come,
// and launches of 256 steps, the second of two systems of 256 000 atoms on two
// streams went on with the 24 workgroups that found room: 1 000 steps each
// took 131 and 31 ms, 600 steps of three systems up to 995 ms; now 46 and 47,
// and 28 to 43 (in launches of a step 47 and 47, and 47).
// In a batch a replica's last workgroup may come when another's replica is
// through, 64 steps of 13-60 us.
constexpr long long ROLL_TICKS = 5000, ROLL_TICKS_BATCH = 500000, ROLL_TICKS_STEP = 600;
__device__ __forceinline__ bool roll_wait(long long waited, int here, int size, int steps,
                                          bool solo) {
  return waited * here <
         size * (solo ? ROLL_TICKS : ROLL_TICKS_BATCH) + (long long)(size - here) * steps * ROLL_TICKS_STEP;
}
constexpr int RUN_SPINS = 1 << 22;
// A replica's lines of Tables::run, 256 bytes each; zero between launches.
// Whatever all workgroups count is counted in 32 groups, then over the groups:
// 1 000 workgroups on one counter take 12.7 us, in 32 groups 2.0.  A group's
// line and the root's hold the words RUN_BAR (arrivals at barriers), RUN_CALL
// (at the roll call; ROLL_CLOSED: it is over), RUN_GONE (workgroups through)
// and RUN_BASE (rank of the group's first, of a roll call that was closed).
enum { RUN_GROUPS = 32, RUN_ROOT = 32, RUN_EPOCH = 33, RUN_STATE = 34, RUN_END = 35 };
enum { RUN_BAR = 0, RUN_CALL = 1, RUN_GONE = 2, RUN_BASE = 3, RUN_WORDS = 4 };
static_assert(RUN_END <= RUN_LINES, "Tables::run");
constexpr int ROLL_CLOSED = 1 << 30;
// Member q of n counts itself at a word of its group (`word` of its line):
// true for the last of all.
__device__ __forceinline__ int group_size(int g, int n) {
  return (n - g + RUN_GROUPS - 1) / RUN_GROUPS;
}
__device__ __forceinline__ bool count_in(int32_t *w, int word, int q, int n, int *index) {
  constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;
  const int g = q & (RUN_GROUPS - 1);
  *index = __hip_atomic_fetch_add(&w[64 * g + word], 1, __ATOMIC_RELAXED, AG);
  return *index == group_size(g, n) - 1 &&
         __hip_atomic_fetch_add(&w[64 * RUN_ROOT + word], 1, __ATOMIC_RELAXED, AG) ==
             min(n, (int)RUN_GROUPS) - 1;
}

// A participant's place among n (epoch: barriers passed).
struct RunSeat {
  int32_t *w;
  int rank, n, epoch;
};
// The maximum speed of a ring entry as of a barrier, and whether the run stops
// there.
struct RunOut {
  unsigned long long vbits;
  int stop;
};
// In the epoch word: the run stops at this barrier.
constexpr int RUN_STOP = 1 << 30;
// The epoch word once it has reached epoch v, or -1.
__device__ __forceinline__ int run_wait(int32_t *f, int v) {
#pragma unroll 1
  for (int it = 0; it < RUN_SPINS; ++it) {
    const int e = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if ((e & (RUN_STOP - 1)) >= v) return e;
    __builtin_amdgcn_s_sleep(1);
  }
  return -1;
}

// The grid barrier.
// drop: plain loads after it see what was stored (device-scope) before it:
// the caches of the CU and of its XCD are invalidated, by one wave for its
// workgroup.
// ring: the maximum speed of that ring entry (< 0: none) is left in `out`,
// read by one wave.
// Whether the run stops is one decision for all: it goes with the epoch, from
// what every workgroup brought (bring_error).  (The error word itself may
// already hold an error of the next phase, which a workgroup that was quicker
// is in: one that acted on it would leave the others waiting.)  A workgroup
// whose barrier gives up stops, and brings that to the next one it comes to.
__device__ __forceinline__ void run_barrier(RunSeat &p, bool drop, int ring, SlotC &S0, CtlDev &C,
                                            RunOut &out) {
  constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;
  __builtin_amdgcn_s_waitcnt(0);  // this wave's device-scope stores have arrived
  __syncthreads();
  ++p.epoch;
  if (threadIdx.x < 64) {
    int e = 0;
    if (threadIdx.x == 0) {
      // (both worked out here: left to itself the compiler holds them across
      // the step, spilled, and the reloads are in the barrier's chain)
      auto wg = gp(p.w);
      int one;
      asm volatile("v_mov_b32 %0, 1" : "=v"(one));
      asm volatile("" : "+v"(wg));
      int32_t *w = (int32_t *)wg;
      const int g = p.rank & (RUN_GROUPS - 1), in = group_size(g, p.n);
      const int ng = p.n < RUN_GROUPS ? p.n : RUN_GROUPS;
      const int got = __hip_atomic_fetch_add(&w[64 * g], one, __ATOMIC_RELAXED, AG) + 1;
      if ((got & (RUN_BAD - 1)) == p.epoch * in) {
        if (got >= RUN_BAD) {
          bring_error(&w[64 * RUN_ROOT]);
          __builtin_amdgcn_s_waitcnt(0);  // before the arrival below
        }
        const int all = __hip_atomic_fetch_add(&w[64 * RUN_ROOT], one, __ATOMIC_RELAXED, AG) + 1;
        if ((all & (RUN_BAD - 1)) == p.epoch * ng)
          __hip_atomic_store(&w[64 * RUN_EPOCH], p.epoch | (all >= RUN_BAD ? RUN_STOP : 0),
                             __ATOMIC_RELAXED, AG);
      }
      e = run_wait(&w[64 * RUN_EPOCH], p.epoch);
      if (e < 0) {
        latch_error(C, ERR_STALL, C.done + 1);
        bring_error(&w[64 * g]);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    // (the loads below come back after the invalidation)
    if (drop) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    unsigned long long v = 0;
    if (ring >= 0 && threadIdx.x < VSPREAD)
      v = __hip_atomic_load(&S0.vring[(ring * VSPREAD + threadIdx.x) * 16], __ATOMIC_RELAXED, AG);
    v = wave_max_u64(v);
    if (threadIdx.x == 0) {
      out.vbits = v;
      out.stop = e < 0 || (e & RUN_STOP) != 0 ? 1 : 0;
    }
  }
  __syncthreads();
}

// The roll call's result, once: all `size` (everybody has come), or those that
// have come when it is closed, at most `limit`.  A workgroup counts itself in
// its group before the group is closed, or finds it closed.
__device__ __forceinline__ void roll_close(int32_t *w, int size, int limit, int all) {
  constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;
  int zero = 0;
  const int claim = all <= limit && all > 0 ? all : -1;
  if (!__hip_atomic_compare_exchange_strong(&w[64 * RUN_STATE], &zero, claim, __ATOMIC_RELAXED,
                                            __ATOMIC_RELAXED, AG) || claim > 0)
    return;
  int n = 0;
  for (int g = 0; g < min(size, (int)RUN_GROUPS); ++g) {
    __hip_atomic_store(&w[64 * g + RUN_BASE], n, __ATOMIC_RELAXED, AG);
    n += __hip_atomic_fetch_or(&w[64 * g + RUN_CALL], ROLL_CLOSED, __ATOMIC_RELAXED, AG);
  }
  __builtin_amdgcn_s_waitcnt(0);  // the bases have arrived
  __hip_atomic_store(&w[64 * RUN_STATE], min(n, limit), __ATOMIC_RELAXED, AG);
}
__device__ __forceinline__ int roll_here(const int32_t *w, int size) {
  int n = 0;
  for (int g = 0; g < min(size, (int)RUN_GROUPS); ++g)
    n += __hip_atomic_load(&w[64 * g + RUN_CALL], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
         (ROLL_CLOSED - 1);
  return n;
}

// One workgroup's part in steps done + 1 .. min(done + steps, target) of
// replica r, which `size` workgroups (this one `seat` of them) come to take.
// A target below zero: the one in the control block.  commit: also the step
// counters (a traced replica's are advanced after its trace has been
// reduced).  solo: the launch is this replica's alone.
template <typename R, bool ACC, bool MIX>
__device__ __forceinline__ void run_replica(const Tables &T, StepLds<MIX> &lds, int r, int seat,
                                            int size, bool solo, int steps, long long to,
                                            int commit) {
  constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;
  // (every thread has read `out` and the roll call before a tile's first
  // barrier, after which the tile writes these words)
  RunOut &out = *(RunOut *)lds.sh;
  int &s_rank = ((int *)lds.sv)[0], &s_n = ((int *)lds.sv)[1];
  static_assert(sizeof(SortLds) <= sizeof(lds.sx), "the sort's LDS shares the window's");
  SortLds &slds = *(SortLds *)lds.sx;
  int32_t *w = T.run + 64 * (RUN_HEAD + RUN_LINES * r);
  CtlDev &C = T.ctl[r];
  SlotC &S0 = slot(T, 2 * r);
  // the control words as earlier launches left them (this launch writes them
  // only after the roll call)
  const auto &C0 = *cview(T.ctl + r);
  const int64_t target = to < 0 ? C0.target : (int64_t)to;
  const int64_t done = C0.done, force_step = C0.force_step, bins_step = C0.bins_step;
  const bool ahead = C0.bin_ring[mod3(done)] != 0;
  const int64_t end = done + steps < target ? done + steps : target;
  const bool clean = C0.clean != 0, cell_only = S0.cell_only != 0;
  int64_t k = done + 1;
  double D2 = C0.disp_ring[mod3(k - 2)];
  double V1 = uniform(ring_max(S0, mod3(k - 1))), V2 = uniform(ring_max(S0, mod3(k - 2)));
  int var = C0.var_ring[mod3(k - 1)];
  int64_t reo1 = C0.reo_ring[mod3(k - 1)];
  bool ord = C0.ord_ring[mod3(k - 1)] != 0;
  const bool idle = C0.err != 0 || done >= end;
  // (read here, every word: a workgroup that comes after the others have gone
  // on may find other words, and takes no part)
  asm volatile("" ::"s"(done), "s"(target), "s"(reo1), "s"(var), "s"((int)ord), "s"((int)clean),
               "s"((int)ahead), "s"((int)idle), "s"(__double_as_longlong(D2)));
  // roll call
  RunSeat me;
  me.w = w;
  me.epoch = 0;
  if (threadIdx.x == 0) {
    int index;
    if (count_in(w, RUN_CALL, seat, size, &index)) roll_close(w, size, T.run_max, size);
    int n = 0;
    const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
    while ((n = __hip_atomic_load(&w[64 * RUN_STATE], __ATOMIC_RELAXED, AG)) <= 0) {
      // (the first of a group looks after the others)
      const long long t = (long long)__builtin_amdgcn_s_memrealtime() - t0;
      if (n == 0 && index == 0 && t >= (solo ? ROLL_TICKS : ROLL_TICKS_BATCH)) {
        const int here = roll_here(w, size);
        if (!roll_wait(t, here, size, idle ? 0 : (int)(end - done), solo))
          roll_close(w, size, T.run_max, 0);
      }
      __builtin_amdgcn_s_sleep(1);
    }
    // (the workgroups of a roll call that was closed are numbered by their
    // groups; one that came later takes no part)
    s_rank = n == size ? seat
             : (index & ROLL_CLOSED) != 0
                 ? size
                 : __hip_atomic_load(&w[64 * (seat & (RUN_GROUPS - 1)) + RUN_BASE],
                                     __ATOMIC_RELAXED, AG) + index;
    s_n = n;
    lds.call = &w[64 * (s_rank & (RUN_GROUPS - 1)) + RUN_BAR];
  }
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(s_n);
  const bool all = n == size;
  // with everybody present a workgroup's place goes by its number, so that
  // each XCD has a contiguous eighth of the tiles of a system that is alone
  const int rank = __builtin_amdgcn_readfirstlane(s_rank);
  if (rank < n) {
    me.rank = rank;
    me.n = n;
    const int nt = S0.ntiles, per = (nt + 7) >> 3;
    // one: a tile each (and none for some workgroups of a system alone, whose
    // `size` is 8 per)
    const bool one = all && nt <= n, slab = solo && all;
    const int first = slab ? (rank & 7) * per + (rank >> 3) : rank;
    const int tend = slab ? min(nt, ((rank & 7) + 1) * per) : nt,
              tstep = one ? nt : slab ? n >> 3 : n;
    // shares of a cell tile: as many units as participants where that leaves a
    // share an atom or so per thread
    const int nsp = max(1, min(8, n / S0.nctiles)), nunits = S0.nctiles * nsp;
    const bool lead = rank == 0 && threadIdx.x == 0;
    int stop = idle ? 1 : 0;  // nothing to do: the loop below is not entered
    auto barrier = [&](bool drop, bool ring) {
      run_barrier(me, drop, ring ? (int)mod3(k) : -1, S0, C, out);
      stop = __builtin_amdgcn_readfirstlane(out.stop);
    };
    if (lead) {
      C.target = target;
      C.base = done;
      if (clean && !idle) C.bin_ring[mod3(done)] = cell_only ? 1 : 0;
    }
    // With a list, a sort's positions are binned when the rule has fired: here
    // that is a barrier more, where binning ahead (see bins_rule) costs a step
    // its atomics and a full barrier about one and a half times per rebuild.
    // With the cell method every step bins the next one's.  (A replica of a
    // batch that the two launches left in mid-run holds r(k) binned where
    // bin_ring says so.)
    bool binned = (clean ? cell_only : ahead) || k == bins_step;
    int dirty = 7;  // cell-layer sets to be cleared (as far as is known)
    if (clean && !idle) {
      for (int t = first; t < tend; t += tstep)
        if (kick_tile<true>(slot(T, 2 * r + var), C, t, done, binned)) bring_error(lds.call);
      barrier(false, false);
    }
    // the decisions of k_sort for step k
    double d1 = 0.0;
    bool rebuild = true, reo = true;
    // (the loop's state is the same in every lane, but the compiler loses that
    // through the barriers' one-lane branches: without this it held the step
    // number and the descriptors in vector registers and spilled them)
    auto scalars = [&] {
      k = uniform(k);
      var = uniform(var);
      reo1 = uniform(reo1);
      ord = uniform(ord);
      dirty = uniform(dirty);
      D2 = uniform(D2);
      V1 = uniform(V1);
      V2 = uniform(V2);
      binned = uniform(binned);
    };
    auto decide = [&] {
      scalars();
      d1 = 0.0;
      rebuild = true;
      if (!cell_only) rebuild = uniform(rebuild_rule(S0, force_step, k, D2, V1, &d1));
      d1 = uniform(d1);
      reo = !S0.noreo && (S0.nr <= 0 || k - reo1 >= S0.nr);
    };
    auto record = [&] {
      if (!lead) return;
      C.rb_ring[mod3(k)] = rebuild ? (reo ? RB_REORDER : RB_PERM) : RB_NONE;
      C.bin_ring[mod3(k)] = cell_only && k != target ? 1 : 0;
      C.reo_ring[mod3(k)] = reo1;
      if (!cell_only) {
        C.disp_ring[mod3(k - 1)] = d1;
        if (rebuild && k != force_step) C.n_rebuilds += 1;
      }
      C.var_ring[mod3(k)] = var;
      C.ord_ring[mod3(k)] = ord ? 1 : 0;
    };
    auto to_clear = [&] {
      const int set = (int)mod3(k + 2);
      const bool c = (dirty >> set & 1) != 0;
      dirty &= ~(1 << set);
      return c;
    };
    // the end of step k, with its barrier
    auto next = [&] {
      if (first == 0 && threadIdx.x < VSPREAD)
        st<true>(&gp(S0.vring)[(mod3(k + 1) * VSPREAD + threadIdx.x) * 16], 0ull);
      barrier(false, true);
      D2 = d1;
      V2 = V1;
      V1 = uniform(__longlong_as_double((long long)out.vbits));
      binned = cell_only;
      ++k;
    };
    while (k <= end && stop == 0) {
      decide();
      if (!rebuild) {
        // the list steps up to the next rebuild; with one tile per workgroup it
        // is held from step to step
        const bool unord = ord || S0.noreo;
        Own<R> own;
        bool held = false;
        do {
          SlotC &S = slot(T, 2 * r + var);
          record();
          const bool clear = to_clear();
          for (int t = first; t < tend; t += tstep) {
            if (!held) own_load<R, MIX>(S, lds, t, k, own);
            own_step<R, ACC, MIX>(S, C, lds, t, k, k == target, clear, unord, (int)(k - done - 1),
                                  own);
            if (!one) own_store(S, t, k + 1, own);
          }
          held = one;
          next();
          if (k > end || stop != 0) break;
          decide();
        } while (!rebuild);
        if (one && first < tend) own_store(slot(T, 2 * r + var), first, k, own);
        if (k > end || stop != 0) break;
      }
      scalars();
      const int set = (int)mod3(k);
      if (!binned) {
        SlotC &S = slot(T, 2 * r + var);
        const int pb = (int)(k & 1);
        for (int t = first; t < tend; t += tstep) {
          const int i = t * TILE + tid_here();
          if (i < S.n && bin_atom<true>(S, C, set, i, ld<true>(&gp((const double *)S.P[pb][0])[i]),
                                        ld<true>(&gp((const double *)S.P[pb][1])[i]),
                                        ld<true>(&gp((const double *)S.P[pb][2])[i]), k))
            bring_error(lds.call);
        }
        // (counted where binning ahead would have missed it)
        if (lead && !uniform(bins_rule(S0, force_step, k, D2, V2))) C.late_bins += 1;
        barrier(false, false);
        if (stop != 0) break;
      }
      scalars();
      SortRun sr;
      for (int u = rank; u < nunits; u += n) {
        const int t = u / nsp;
        sort_unit<true>(slot(T, 2 * r + var), slot(T, 2 * r + (var ^ 1)), C, k, MODE_STEP, reo,
                  S0.ctile_off + t, u - t * nsp, nsp, r, sr, slds);
      }
      barrier(true, false);
      // (an exit of its own here costs the loop's state a score of registers)
      const int tdone = stop != 0 ? 0 : tend;
      if (reo) var ^= 1;
      ord = !reo;
      if (reo) reo1 = k;
      dirty |= 1 << set;
      scalars();
      record();
      const bool unord = ord || S0.noreo, clear = to_clear(), bin1 = cell_only && k != target;
      for (int t = first; t < tdone; t += tstep)
        step_tile<R, ACC, MIX, true>(slot(T, 2 * r + var), C, lds, t, k, MODE_STEP, true, !cell_only,
                                     k == target, bin1, clear,
                                     [&] { return unord; }, (int)(k - done - 1), nullptr, 0);
      next();
    }
    if (lead && commit && !idle) {
      const int64_t es = (int64_t)__hip_atomic_load((unsigned long long *)&C.err_step,
                                                   __ATOMIC_RELAXED, AG);
      end_run(C, (int)(end - done), done, target,
              __hip_atomic_load(&C.err, __ATOMIC_RELAXED, AG), es);
    }
  }
  // the last to leave clears the words for the next launch
  int index;
  if (threadIdx.x == 0 && count_in(w, RUN_GONE, seat, size, &index))
    for (int q = 0; q < RUN_END; ++q)
      for (int u = 0; u < RUN_WORDS; u += 2)
        __hip_atomic_store((unsigned long long *)&w[64 * q + u], 0ull, __ATOMIC_RELAXED, AG);
}

// A system alone: one workgroup per tile.  A batch: a workgroup takes the next
// of the seats of its replicas (SlotDev::run_n each, one after the other) and
// ends with it, so every replica goes through its steps at its own pace, none
// waits for another's rebuild, and the chip is shared with other streams at
// every seat's end (with 1 024 workgroups that went from seat to seat, another
// stream's kernel waited 16 ms beside 256 replicas).  The launch has more
// workgroups than seats, since each XCD is dealt an eighth of them, and one
// that is through with its seats sooner takes more.  Seats are handed out in order and a replica's are
// never more than the chip holds at once, so the first replica that is not
// through gets all of its workgroups as the chip empties, or goes on with
// those that have come when it has waited long enough.
template <typename R, bool ACC, bool MIX>
__global__ __launch_bounds__(TILE, MIX ? 3 : 4) void k_run(Tables T, int steps, long long target,
                                                         int commit, int seats) {
  constexpr int AG = __HIP_MEMORY_SCOPE_AGENT;
  __shared__ StepLds<MIX> lds;
  const bool solo = seats == 0;  // a system alone: its workgroups are its seats
  int q = blockIdx.x, r = 0;
  if (!solo) {
    int &s_seat = ((int *)lds.sv)[2];
    if (threadIdx.x == 0) s_seat = __hip_atomic_fetch_add(&T.run[0], 1, __ATOMIC_RELAXED, AG);
    __syncthreads();
    q = __builtin_amdgcn_readfirstlane(s_seat);
    r = q < seats ? cview(T.run_rep)[q] : -1;
  }
  SlotC &S0 = slot(T, 2 * max(r, 0));
  if (r >= 0 && S0.fp64 == (sizeof(R) == 8))
    run_replica<R, ACC, MIX>(T, lds, r, solo ? q : q - S0.run_off, solo ? (int)gridDim.x : S0.run_n,
                             solo, steps, target, commit);
  if (!solo && threadIdx.x == 0 &&
      __hip_atomic_fetch_add(&T.run[64], 1, __ATOMIC_RELAXED, AG) == (int)gridDim.x - 1) {
    __hip_atomic_store(&T.run[0], 0, __ATOMIC_RELAXED, AG);
    __hip_atomic_store(&T.run[64], 0, __ATOMIC_RELAXED, AG);
  }
}

// End of a graph replay of K steps, before k_replay_end: for every traced
// replica (workgroup (s, r)) the properties of step base + s + 1, reduced
// from the tile partials in a fixed order (as k_props), into its trace ring.
__global__ __launch_bounds__(TILE) void k_trace(Tables T, int K) {
  const int s = blockIdx.x, r = blockIdx.y;
  if (s >= K || r >= T.nslots) return;
  SlotC &S = slot(T, 2 * r);
  if (S.n <= 0 || S.tpart == nullptr) return;
  const CtlDev &C = T.ctl[r];
  const int64_t k = C.base + s + 1;
  if (k > C.target || (C.err != 0 && C.err_step <= k)) return;
  __shared__ double sh[TILE][4];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int t = threadIdx.x; t < S.ntiles; t += TILE) {
    const double *q = S.tpart + ((size_t)s * S.ntiles + t) * 4;
    v[0] += q[0];
    v[1] += q[1];
    v[2] += q[2];
    v[3] = fmax(v[3], q[3]);
  }
  for (int j = 0; j < 4; ++j) sh[threadIdx.x][j] = v[j];
  __syncthreads();
  for (int h = TILE / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h)
      for (int j = 0; j < 4; ++j) {
        const double o = sh[threadIdx.x + h][j];
        sh[threadIdx.x][j] = j == 3 ? fmax(sh[threadIdx.x][j], o) : sh[threadIdx.x][j] + o;
      }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double *row = S.trace + (size_t)(k % TRACE_RING) * TRACE_W;
    row[0] = (double)k;
    row[1] = 0.5 * sh[0][0];
    row[2] = 0.5 * sh[0][1];
    row[3] = 0.5 * sh[0][2];
    row[4] = sh[0][3];
  }
}

// End of a graph replay of K steps: advance the step counters (one thread
// per replica; no other kernel of the replay reads what is written here).
__global__ void k_replay_end(Tables T, int K) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= T.nslots) return;
  CtlDev &C = T.ctl[r];
  if (slot(T, 2 * r).n <= 0) return;
  if (C.base >= C.target && C.done >= C.target) return;
  end_run(C, K, C.base, C.target, C.err, C.err_step);
}

// Host-ordered update of a replica's target (single thread).
__global__ void k_set_target(Tables T, int slot, long long target) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    CtlDev &C = T.ctl[slot];
    C.target = target;
    C.base = C.done;
  }
}

// Fixed-order reduction of the per-tile partials of each replica (one
// workgroup per replica): thread t takes tiles t, t+256, ... in sequence, then
// a fixed tree.
__global__ __launch_bounds__(TILE) void k_props(Tables T, int only, CtlDev *ctl_out) {
  const int r = blockIdx.x;
  if (r >= T.nslots || (only >= 0 && r != only)) return;
  if (slot(T, 2 * r).n <= 0) return;
  SlotC &S = slot_held(T, r);
  CtlDev &C = T.ctl[r];
  constexpr int NV = 6 + NACC;
  __shared__ double sh[TILE][NV];
  double v[NV] = {};
  for (int t = threadIdx.x; t < S.ntiles; t += TILE) {
    const double *q = S.part + (size_t)t * NPART;
    v[0] += q[0];
    v[1] = fmax(v[1], q[1]);
    v[2] += q[2] + q[3];
    v[3] += q[4] + q[5];
    v[4] += q[6];
    v[5] = fmax(v[5], q[7]);
    const double *A = S.acc + (size_t)t * NACC;
    for (int j = 0; j < NACC; ++j) v[6 + j] += A[j];
  }
  for (int j = 0; j < NV; ++j) sh[threadIdx.x][j] = v[j];
  __syncthreads();
  for (int h = TILE / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      for (int j = 0; j < NV; ++j) {
        const double o = sh[threadIdx.x + h][j];
        sh[threadIdx.x][j] = (j == 1 || j == 5) ? fmax(sh[threadIdx.x][j], o)
                                                : sh[threadIdx.x][j] + o;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 3) {
    double vm = 0.0;
    for (int q = 0; q < VSPREAD; ++q)
      vm = fmax(vm, __longlong_as_double((long long)S.vring[(threadIdx.x * VSPREAD + q) * 16]));
    C.vmax_ring[threadIdx.x] = (uint64_t)__double_as_longlong(vm);
  }
  if (threadIdx.x == 0) {
    C.ke = 0.5 * sh[0][0];
    C.vmax2 = sh[0][1];
    C.pe = 0.5 * sh[0][2];
    C.vir = 0.5 * sh[0][3];
    C.sum_m = (int64_t)sh[0][4];
    C.max_m = (int)sh[0][5];
    for (int j = 0; j < NACC; ++j) C.acc_sum[j] = sh[0][6 + j];
  }
  if (ctl_out != nullptr) {
    // the control block, to where the host reads it
    __syncthreads();
    if (threadIdx.x < sizeof(CtlDev) / 4)
      ((int32_t *)(ctl_out + r))[threadIdx.x] = ((const int32_t *)&C)[threadIdx.x];
  }
}
static_assert(sizeof(CtlDev) / 4 <= TILE && sizeof(CtlDev) % 4 == 0, "one word per thread");

// Step (f) during equilibration (Secs. 3.1 and 5.1): scale the velocities of a
// held clean state by one factor so that sum v^2 = 3 (N - 1) T (the centre of
// mass is at rest, leaving 3 (N - 1) degrees of freedom), from the kinetic
// energy k_props reduced just before.  The tile's kinetic-energy and max-v^2
// partials are recomputed from the scaled velocities, in the step kernel's
// order; the rebuild rule keeps the maximum speed of (e), taken before (f).
__global__ __launch_bounds__(TILE) void k_adjust(Tables T, int only, double temperature) {
  __shared__ double sk[4];
  __shared__ unsigned long long sv[4];
  const int nt = cview(T.hdr)[HDR_NTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nt; t += gridDim.x) {
    const int r = cview(T.tile_rep)[t];
    if (only >= 0 && r != only) continue;
    if (slot(T, 2 * r).n <= 0) continue;
    SlotC &S = slot_held(T, r);
    const CtlDev &C = T.ctl[r];
    const double ke = C.ke;
    if (!C.clean || C.err != 0 || S.n < 2 || !(ke > 0.0)) continue;
    const double fac = sqrt((1.5 * (double)(S.n - 1) * temperature) / ke);
    const int lt = t - S.tile_off;
    const int i = lt * TILE + threadIdx.x;
    const int vb = (int)((C.done + 1) & 1);
    double vv = 0.0;
    if (i < S.n) {
      double v[3];
      for (int a = 0; a < 3; ++a) {
        v[a] = gp(S.V[vb][a])[i] * fac;
        gp(S.V[vb][a])[i] = v[a];
      }
      vv = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const double ks = wave_sum(vv);
    const unsigned long long vb2 = wave_max_u64((unsigned long long)__double_as_longlong(vv));
    if (l == 0) {
      sk[w] = ks;
      sv[w] = vb2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      auto q = gp(S.part) + (size_t)lt * NPART;
      q[0] = ((sk[0] + sk[1]) + sk[2]) + sk[3];
      const unsigned long long b01 = sv[0] > sv[1] ? sv[0] : sv[1];
      const unsigned long long b23 = sv[2] > sv[3] ? sv[2] : sv[3];
      q[1] = __longlong_as_double((long long)(b01 > b23 ? b01 : b23));
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// binning of the held state outside a step (creation, host-side sorts)
// ---------------------------------------------------------------------------
// A batch goes on from k_run in two launches a step: its replicas in mid-run
// hold r(done + 1) unbinned, where those launches would have binned it ahead
// if bins_due.  k_due (one wave per replica) finds the replicas to be binned
// and records it, k_bin_due bins them; without it every one whose rule fires
// at once would wait for the host.
__global__ __launch_bounds__(64) void k_due(Tables T) {
  const int r = blockIdx.x;
  SlotC &S0 = slot(T, 2 * r);
  if (S0.n <= 0) return;
  CtlDev &C = T.ctl[r];
  const int64_t k = C.done + 1;
  const bool due = C.err == 0 && !C.clean && k <= C.target && k != C.bins_step &&
                   C.bin_ring[mod3(C.done)] == 0 && bins_due(S0, C, k);
  if (threadIdx.x == 0) {
    C.bin_due = due ? 1 : 0;
    if (due) C.bin_ring[mod3(k - 1)] = 1;
  }
}
__global__ __launch_bounds__(TILE) void k_bin_due(Tables T) {
  const int nt = T.hdr[HDR_NTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nt; t += gridDim.x) {
    const int r = T.tile_rep[t];
    CtlDev &C = T.ctl[r];
    if (slot(T, 2 * r).n <= 0 || C.bin_due == 0) continue;
    SlotC &S = slot_held(T, r);
    const int i = (t - S.tile_off) * TILE + threadIdx.x;
    if (i >= S.n) continue;
    const int64_t k = C.done + 1;
    const int pb = (int)(k & 1);
    bin_atom<false>(S, C, (int)mod3(k), i, S.P[pb][0][i], S.P[pb][1][i], S.P[pb][2][i], k);
  }
}
__global__ __launch_bounds__(TILE) void k_insert(Tables T, int wrap_store, int only) {
  const int nt = T.hdr[HDR_NTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nt; t += gridDim.x) {
    const int r = T.tile_rep[t];
    if (only >= 0 && r != only) continue;
    if (slot(T, 2 * r).n <= 0) continue;
    SlotC &S = slot_held(T, r);
    CtlDev &C = T.ctl[r];
    const int i = (t - S.tile_off) * TILE + threadIdx.x;
    if (i >= S.n) continue;
    const int64_t k = cur_state(C);
    const int pb = (int)(k & 1);
    const double x = S.P[pb][0][i], y = S.P[pb][1][i], z = S.P[pb][2][i];
    bin_atom<false>(S, C, (int)mod3(k), i, x, y, z, k);  // checks the unwrapped coordinates
    if (wrap_store && isfinite(x) && isfinite(y) && isfinite(z)) {
      S.P[pb][0][i] = wrap1(x, S.L, S.halfL);
      S.P[pb][1][i] = wrap1(y, S.L, S.halfL);
      S.P[pb][2][i] = wrap1(z, S.L, S.halfL);
    }
  }
}

// Cell index of the held position of every atom of replica `only`, storage
// order, into out (md_get_cells): the cell of bin_atom without binning.
__global__ __launch_bounds__(TILE) void k_cells(Tables T, int only, int32_t *out) {
  const int nt = T.hdr[HDR_NTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nt; t += gridDim.x) {
    const int r = T.tile_rep[t];
    if (r != only || slot(T, 2 * r).n <= 0) continue;
    SlotC &S = slot_held(T, r);
    const CtlDev &C = T.ctl[r];
    const int i = (t - S.tile_off) * TILE + threadIdx.x;
    if (i >= S.n) continue;
    const int pb = (int)(cur_state(C) & 1);
    double x = S.P[pb][0][i], y = S.P[pb][1][i], z = S.P[pb][2][i];
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) x = y = z = 0.0;
    out[i] = cell_of(S, wrap1(x, S.L, S.halfL), wrap1(y, S.L, S.halfL), wrap1(z, S.L, S.halfL));
  }
}

// ---------------------------------------------------------------------------
// state to and from the host
// ---------------------------------------------------------------------------
// The storage position of every atom of replica r by original index, into the
// cell array of the descriptor variant not in use (the next sort overwrites
// it anyway).
__device__ __forceinline__ int32_t *inverse_of(const Tables &T, int r) {
  const CtlDev &C = T.ctl[r];
  return slot(T, 2 * r + (C.var_ring[mod3(C.done)] ^ 1)).cell;
}
__global__ __launch_bounds__(TILE) void k_invert(Tables T, int r, CtlDev *ctl_out) {
  SlotC &S = slot_held(T, r);
  const auto inv = gp(inverse_of(T, r));
  const auto id = gp((const int32_t *)S.id);
  for (int p = blockIdx.x * TILE + threadIdx.x; p < S.n; p += gridDim.x * TILE)
    if ((uint32_t)id[p] < (uint32_t)S.n) inv[id[p]] = p;
  // the control block, to where the host reads it
  if (blockIdx.x == 0 && threadIdx.x < sizeof(CtlDev) / 4)
    ((int32_t *)ctl_out)[threadIdx.x] = ((const int32_t *)&T.ctl[r])[threadIdx.x];
}
// Atoms c0 .. c0+cnt-1 (original indices) of the arrays in `what` (EXP_*), in
// the caller's layout, one array after the other, into host memory: the
// stores are consecutive, so they cross the bus as whole lines, and no copy
// of the state is made on the device.
__global__ __launch_bounds__(TILE) void k_export(Tables T, int r, int what, int c0, int cnt,
                                                 double *out) {
  SlotC &S = slot_held(T, r);
  const CtlDev &C = T.ctl[r];
  const int64_t k = cur_state(C);
  const int pb = (int)(k & 1), vb = (int)((C.clean ? k + 1 : k) & 1);
  const auto inv = gp((const int32_t *)inverse_of(T, r));
  const size_t np = S.npad;
  const bool f64 = S.fp64 != 0;
  auto real = [&](const void *a, size_t q) {
    return f64 ? gp((const double *)a)[q] : (double)gp((const float *)a)[q];
  };
  const int n3 = 3 * cnt;
  for (int kind = 0; kind < 5; ++kind) {
    if (!(what >> kind & 1)) continue;
    const bool vec = kind < 3;
    const int len = vec ? n3 : cnt;
    for (int e = blockIdx.x * TILE + threadIdx.x; e < len; e += gridDim.x * TILE) {
      const int j = vec ? e / 3 : e, d = vec ? e - 3 * j : 0;
      const int p = inv[c0 + j];
      double v;
      if (kind == 0) v = gp((const double *)S.P[pb][d])[p];
      else if (kind == 1) v = gp((const double *)S.V[vb][d])[p];
      else if (kind == 2) v = real(S.F, d * np + p);
      else v = real(S.UA, (kind - 3) * np + p);
      out[e] = v;
    }
    out += len;
  }
}
// The reverse for a state at step `step` in descriptor variant `variant`:
// atoms c0 .. c0+cnt-1 of positions and velocities (host memory, one after
// the other) in storage order of the original indices.
__global__ __launch_bounds__(TILE) void k_import(SlotDev S, int step, int c0, int cnt,
                                                 const double *in) {
  const int pb = step & 1, vb = pb ^ 1;
  for (int e = blockIdx.x * TILE + threadIdx.x; e < 3 * cnt; e += gridDim.x * TILE) {
    const int j = e / 3, d = e - 3 * j;
    gp(S.P[pb][d])[c0 + j] = in[e];
    gp(S.V[vb][d])[c0 + j] = in[3 * cnt + e];
    if (d == 0) gp(S.id)[c0 + j] = c0 + j;
  }
}

// Clear the cell-layer set of the held state (before re-binning it).
__global__ __launch_bounds__(TILE) void k_clear_set(Tables T, int only) {
  const int nct = T.hdr[HDR_NCTILES];
  for (int t = xcd_block(blockIdx.x, gridDim.x); t < nct; t += gridDim.x) {
    const int r = T.ctile_rep[t];
    if (only >= 0 && r != only) continue;
    SlotC &S = slot(T, 2 * r);
    const CtlDev &C = T.ctl[r];
    const int set = (int)mod3(cur_state(C));
    const int lt = t - S.ctile_off;
    const int c = lt * CTILE + threadIdx.x;
    if (c < S.ncell) S.cnt[set][c] = 0;
    if (threadIdx.x == 0) S.tcnt[set][lt] = 0;
    if (lt == 0 && threadIdx.x == 0) S.ovf_n[set] = 0;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_kick(const Tables &T, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_kick, dim3(grid), dim3(TILE), 0, s, T);
  hipLaunchKernelGGL(k_kick_end, dim3((T.nslots + TILE - 1) / TILE), dim3(TILE), 0, s, T);
}
void launch_sort(const Tables &T, int cgrid, int step_in_replay, int mode, int only,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_sort, dim3(cgrid), dim3(TILE), 0, s, T, step_in_replay, mode, only);
}
template <typename R, bool ACC, bool MIX>
static void launch_k_step(const Tables &T, int grid, int step_in_replay, int mode,
                          int force_build, int only, hipStream_t s) {
  hipLaunchKernelGGL((k_step<R, ACC, MIX>), dim3(grid), dim3(TILE), 0, s, T, step_in_replay, mode,
                     force_build, only);
}
template <typename R>
static void launch_k_step_r(const Tables &T, int grid, int step_in_replay, int mode,
                            int force_build, int only, hipStream_t s, bool accum, bool mix) {
  if (accum) {
    if (mix) launch_k_step<R, true, true>(T, grid, step_in_replay, mode, force_build, only, s);
    else launch_k_step<R, true, false>(T, grid, step_in_replay, mode, force_build, only, s);
  } else {
    if (mix) launch_k_step<R, false, true>(T, grid, step_in_replay, mode, force_build, only, s);
    else launch_k_step<R, false, false>(T, grid, step_in_replay, mode, force_build, only, s);
  }
}
void launch_step(const Tables &T, int grid, int step_in_replay, int mode, int force_build,
                 int only, int precisions, hipStream_t s, bool accum, bool mix) {
  if (precisions & PREC_FP32)
    launch_k_step_r<float>(T, grid, step_in_replay, mode, force_build, only, s, accum, mix);
  if (precisions & PREC_FP64)
    launch_k_step_r<double>(T, grid, step_in_replay, mode, force_build, only, s, accum, mix);
}
template <typename R>
static void *run_kernel(bool accum, bool mix) {
  if (accum) return mix ? (void *)k_run<R, true, true> : (void *)k_run<R, true, false>;
  return mix ? (void *)k_run<R, false, true> : (void *)k_run<R, false, false>;
}
static void *run_kernel(int precision, bool accum, bool mix) {
  return precision == PREC_FP64 ? run_kernel<double>(accum, mix) : run_kernel<float>(accum, mix);
}
int run_capacity(int precision, bool accum, bool mix, int cus) {
  int per = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, run_kernel(precision, accum, mix), TILE,
                                                   0) != hipSuccess)
    return 0;
  return per * cus;
}
hipError_t launch_run(const Tables &T, int grid, int steps, long long target, bool commit,
                      int seats, int precision, bool accum, bool mix, hipStream_t s) {
  int c = commit ? 1 : 0;
  Tables t = T;
  void *args[] = {&t, &steps, &target, &c, &seats};
  return hipLaunchKernel(run_kernel(precision, accum, mix), dim3(grid), dim3(TILE), args, 0, s);
}
void launch_trace(const Tables &T, int K, hipStream_t s) {
  hipLaunchKernelGGL(k_trace, dim3(K, T.nslots), dim3(TILE), 0, s, T, K);
}
void launch_replay_end(const Tables &T, int K, hipStream_t s) {
  hipLaunchKernelGGL(k_replay_end, dim3((T.nslots + TILE - 1) / TILE), dim3(TILE), 0, s, T, K);
}
void launch_set_target(const Tables &T, int slot, long long target, hipStream_t s) {
  hipLaunchKernelGGL(k_set_target, dim3(1), dim3(64), 0, s, T, slot, target);
}
void launch_props(const Tables &T, int only, CtlDev *ctl_out, hipStream_t s) {
  hipLaunchKernelGGL(k_props, dim3(T.nslots), dim3(TILE), 0, s, T, only, ctl_out);
}
void launch_adjust(const Tables &T, int grid, int only, double temperature, hipStream_t s) {
  hipLaunchKernelGGL(k_adjust, dim3(grid), dim3(TILE), 0, s, T, only, temperature);
}
void launch_insert(const Tables &T, int grid, int wrap_store, int only, hipStream_t s) {
  hipLaunchKernelGGL(k_insert, dim3(grid), dim3(TILE), 0, s, T, wrap_store, only);
}
void launch_bin_due(const Tables &T, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_due, dim3(T.nslots), dim3(64), 0, s, T);
  hipLaunchKernelGGL(k_bin_due, dim3(grid), dim3(TILE), 0, s, T);
}
void launch_cells(const Tables &T, int grid, int only, int32_t *out, hipStream_t s) {
  hipLaunchKernelGGL(k_cells, dim3(grid), dim3(TILE), 0, s, T, only, out);
}
void launch_invert(const Tables &T, int r, int n, CtlDev *ctl_out, hipStream_t s) {
  const int g = (n + TILE - 1) / TILE;
  hipLaunchKernelGGL(k_invert, dim3(g < 2048 ? g : 2048), dim3(TILE), 0, s, T, r, ctl_out);
}
void launch_export(const Tables &T, int r, int what, int c0, int cnt, double *out,
                   hipStream_t s) {
  const int g = (3 * cnt + TILE - 1) / TILE;
  hipLaunchKernelGGL(k_export, dim3(g < 1024 ? g : 1024), dim3(TILE), 0, s, T, r, what, c0, cnt,
                     out);
}
void launch_import(const SlotDev &S, int64_t step, int c0, int cnt, const double *in,
                   hipStream_t s) {
  const int g = (3 * cnt + TILE - 1) / TILE;
  hipLaunchKernelGGL(k_import, dim3(g < 1024 ? g : 1024), dim3(TILE), 0, s, S, (int)(step & 1), c0,
                     cnt, in);
}
void launch_flip(const Tables &T, int only, hipStream_t s) {
  hipLaunchKernelGGL(k_flip, dim3((T.nslots + TILE - 1) / TILE), dim3(TILE), 0, s, T, only);
}
void launch_clear_set(const Tables &T, int cgrid, int only, hipStream_t s) {
  hipLaunchKernelGGL(k_clear_set, dim3(cgrid), dim3(TILE), 0, s, T, only);
}

}  // namespace md
