// kernels.hip -- HIP kernels of the reaction step for gfx950 (CDNA4, wave64).
//
// One reaction step is two kernels (sweep and resolve) where the sweep bins the
// next step's A's, up to four elsewhere (Table I of the paper, steps 1-9, on
// one GPU; the communication steps 4, 6 and 8 have nothing to exchange):
//   k_prep     closes the previous step (counters, bond rows), bins the
//              A-role particles into coarse cells of width >= 2 rc (record:
//              jittered position, id, slot, adjacency row) and re-jitters every
//              particle (the MD stand-in between steps; positions ping-pong
//              between two buffers)
//   k_sweep    every particle streams once with coalesced SoA loads (in brick
//              order once the storage is sorted, the A records of the brick and
//              its halo staged in LDS); candidates go to an LDS queue so that
//              the exact distance test (step 1) and the keyed Philox draws
//              (step 2) run on full wavefronts; each retained pair lowers its A's key (w1, id_T) by
//              a 64-bit atomicMin (steps 3-5) and joins the workgroup's list
//   k_resolve  per sweep workgroup (one wavefront each), the listed pairs
//              whose A chose their T; of those the smallest (w2, id_A) per T
//              is bonded, states and adjacency updated (steps 6-9); the nearest
//              selection and several rules have resolves of their own
// plus the counting sort of the storage by brick (within a brick its A's,
// then the rest by dual cell), the synthetic generator and the helpers of the
// runtime.
//
// Arithmetic follows the contract of include/polyreact.h: FP32 min-image
// distance with explicitly rounded operations (no contraction), Philox4x32-10
// per pair keyed by (step, id_A, id_T), integer threshold on word 0.  Every
// selection is a minimum over 64-bit keys, so no result depends on thread or
// atomic order, nor on the storage order of the particles.
#include <hip/hip_ext.h>
#include <algorithm>
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "../../include/polyreact.h"

namespace pr {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32
// multiplies (hi/lo) and xors, the 64-bit key bumped by the Weyl increments
// after each round.
// ---------------------------------------------------------------------------
struct W4 {
  uint32_t w0, w1, w2, w3;
};

// d behind a pointer that the compiler cannot see through, in read-only memory
// (the kernel's arguments, or a batch's device array): what is read through it
// comes in by scalar loads where it is used.  Read directly, the fields that a
// long kernel uses anywhere are loaded ahead of it and kept, and what the
// scalar registers do not hold is spilled into lanes of vector registers,
// whose reads are vector instructions: in the sweep 88 spilled registers, 40
// this way (1,048,576 particles, 256 steps with load and read-out: 7.80 -> 7.55 ms).
__device__ __forceinline__ const Dev& fresh(const Dev& d) {
  typedef const __attribute__((address_space(4))) Dev* cptr;
  cptr p = (cptr)&d;
  asm volatile("" : "+s"(p));
  return *(const Dev*)p;
}

// a ^ b ^ c in one instruction (gfx950's three-input bitwise op; 0x96 is the
// truth table of the three-way exclusive or)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ W4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     unsigned long long key) {
  // the key (the seed) is uniform in every caller
  uint32_t k0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)key);
  uint32_t k1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(key >> 32));
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one 32x32 -> 64-bit product each (a single v_mad_u64_u32)
    const unsigned long long p0 = 0xD2511F53ull * c0, p1 = 0xCD9E8D57ull * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = xor3(hi1, c1, k0);
    const uint32_t n2 = xor3(hi0, c3, k1);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    // the round keys are bumped on the scalar unit each round rather than
    // precomputed: twenty live key registers would spill to vector lanes
    asm volatile("" : "+s"(k0), "+s"(k1));
  }
  return W4{c0, c1, c2, c3};
}

__device__ __forceinline__ uint32_t byte_sum(uint32_t v, uint32_t acc) {
  return __builtin_amdgcn_sad_u8(v, 0u, acc);  // |bytes - 0| summed, plus acc
}

// Irwin-Hall(12) offsets of the synthetic initial configuration:
// S_d = (12 bytes) - 1530, bytes of words 3d..3d+2 of the blocks
// (step, id, 0..2, tag).
__device__ __forceinline__ void ih12(uint32_t step, uint32_t id, uint32_t tag,
                                     unsigned long long key, int32_t S[3]) {
  const W4 a = philox(step, id, 0u, tag, key);
  const W4 b = philox(step, id, 1u, tag, key);
  const W4 c = philox(step, id, 2u, tag, key);
  S[0] = (int32_t)byte_sum(a.w2, byte_sum(a.w1, byte_sum(a.w0, 0u))) - 1530;
  S[1] = (int32_t)byte_sum(b.w1, byte_sum(b.w0, byte_sum(a.w3, 0u))) - 1530;
  S[2] = (int32_t)byte_sum(c.w0, byte_sum(b.w3, byte_sum(b.w2, 0u))) - 1530;
}

// Irwin-Hall(4) offsets of the re-jitter between reaction steps (the stand-in
// for the MD): S_d = (the 4 bytes of word d) - 510, block (step, id, 0, tag).
__device__ __forceinline__ void ih4(uint32_t step, uint32_t id, uint32_t tag,
                                    unsigned long long key, int32_t S[3]) {
  const W4 a = philox(step, id, 0u, tag, key);
  // the -510 rides in the accumulator (32-bit wrap: the sum is in [0, 1020])
  constexpr uint32_t kMinus510 = 0u - 510u;
  S[0] = (int32_t)byte_sum(a.w0, kMinus510);
  S[1] = (int32_t)byte_sum(a.w1, kMinus510);
  S[2] = (int32_t)byte_sum(a.w2, kMinus510);
}

// Correctly rounded FP32 square root of a positive normal x: the hardware
// estimate (within one ulp) is moved one ulp down or up when x lies beyond
// the midpoint to that neighbour; the residuals x - s_dn * s and x - s_up * s
// are each rounded once by the fused multiply-add, and their signs decide
// exactly (s_dn * s and s_up * s are the midpoints' squares up to a term below
// the rounding of x).
__device__ __forceinline__ float sqrt_rn(float x) {
  float s = __builtin_amdgcn_sqrtf(x);
  const float s_dn = __uint_as_float(__float_as_uint(s) - 1u);
  const float s_up = __uint_as_float(__float_as_uint(s) + 1u);
  const float v_dn = __builtin_fmaf(-s_dn, s, x);
  const float v_up = __builtin_fmaf(-s_up, s, x);
  s = v_dn <= 0.0f ? s_dn : s;
  s = v_up > 0.0f ? s_up : s;
  return s;
}

__device__ __forceinline__ float wrap_box(float v, float L) {
  if (v < 0.0f) v = __fadd_rn(v, L);
  if (v >= L) v = __fsub_rn(v, L);
  return v;
}

// Single conditional wrap of a difference (selects, no branches).
__device__ __forceinline__ float min_image(float d, float L, float halfL) {
  const float dn = __fsub_rn(d, L), up = __fadd_rn(d, L);
  return d > halfL ? dn : (d < -halfL ? up : d);
}

__device__ __forceinline__ bool in_window(int32_t t, int32_t s, int32_t type, int32_t lo,
                                          int32_t hi) {
  return t == type && s >= lo && s <= hi;
}

__device__ __forceinline__ bool is_a(const Dev& d, int32_t t, int32_t s) {
  return in_window(t, s, d.rule.type_a, d.rule.a_min, d.rule.a_max);
}

__device__ __forceinline__ bool is_t(const Dev& d, int32_t t, int32_t s) {
  return in_window(t, s, d.rule.type_t, d.rule.t_min, d.rule.t_max);
}

__device__ __forceinline__ uint8_t role_of(const Dev& d, int32_t t, int32_t s) {
  if (d.nrules > 1) {  // a mask over the rules: T bits 0-3, A bits 4-7
    uint32_t m = 0;
    for (int r = 0; r < d.nrules; ++r) {
      const RuleD& q = d.mr[r].r;
      if (in_window(t, s, q.type_t, q.t_min, q.t_max)) m |= 1u << r;
      if (in_window(t, s, q.type_a, q.a_min, q.a_max)) m |= 16u << r;
    }
    return (uint8_t)m;
  }
  return is_t(d, t, s) ? kRoleT : (is_a(d, t, s) ? kRoleA : kRoleNone);
}

// Whether a role byte makes its particle an A (of some rule).
__device__ __forceinline__ bool role_is_a(uint32_t b, bool multi) {
  return multi ? (b & kMaskA) != 0u : b == kRoleA;
}

__device__ __forceinline__ int cell1(float u, int nc) {
  int c = (int)floorf(u);
  return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__device__ __forceinline__ int cell_of(const Dev& d, float x, float y, float z) {
  const int nc = d.nc;
  const int cx = cell1(__fmul_rn(x, d.inv_w), nc);
  const int cy = cell1(__fmul_rn(y, d.inv_w), nc);
  const int cz = cell1(__fmul_rn(z, d.inv_w), nc);
  return (cz * nc + cy) * nc + cx;
}

// Record r of cell c in the buckets: rank by rank (all cells' first records,
// then all second ones, ..), so that x-adjacent cells' records share cache
// lines; a cell holds 0.5 records on average, and with kCellCap consecutive
// records per cell every one of them had a 128-byte line to itself (1,048,576
// particles, 256 steps with load and read-out 8.39 -> 8.28 ms; the unsorted
// sweep of 1,000,003 particles 55 -> 47 us).
__device__ __forceinline__ size_t rec_at(const Dev& d, int c, uint32_t r) {
  return (size_t)r * (size_t)d.ncell + (size_t)c;
}

__device__ __forceinline__ void set_err(Ctl* c, int code) { atomicCAS(&c->err, 0, code); }

// A flag that any number of workgroups may set for the next kernel: a store that
// stays in the chiplet's L2 to the end of this one, as atomics (and stores) of
// thousands of workgroups that go to one address of the device's memory are served
// one after another (a stateless step of 1,000,003 particles that retains every
// pair, most lists overflowing: the sweep 325 us with an atomic count, 50 with
// this).
__device__ __forceinline__ void set_flag(uint32_t* f) {
  __hip_atomic_store(f, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int32_t read_err(const Ctl* c) {
  return __hip_atomic_load(&c->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Element p (0 or 1) of a two-element array held in the kernel argument:
// both pointers are read and one selected, without dynamic indexing (which
// would copy the argument to scratch); the select keeps the pointers in the
// global address space.
template <typename T>
__device__ __forceinline__ T* pick(T* const (&v)[2], uint32_t p) {
  T* const a = v[0];
  T* const b = v[1];
  return (p & 1u) ? b : a;
}

// Storage set s, member by member (a select of the whole aggregate would be
// built in scratch memory).
__device__ __forceinline__ Arr pick_set(const Dev& d, uint32_t s) {
  // s is uniform: a scalar select keeps the pointers in scalar registers
  s = (uint32_t)__builtin_amdgcn_readfirstlane((int)s);
  const Arr &u = d.set[0], &v = d.set[1];
  Arr r;
  for (int q = 0; q < 2; ++q) {
    r.x[q] = pick({u.x[q], v.x[q]}, s);
    r.y[q] = pick({u.y[q], v.y[q]}, s);
    r.z[q] = pick({u.z[q], v.z[q]}, s);
  }
  r.typ = pick({u.typ, v.typ}, s);
  r.st = pick({u.st, v.st}, s);
  r.adj = pick({u.adj, v.adj}, s);
  r.id = pick({u.id, v.id}, s);
  r.role = pick({u.role, v.role}, s);
  r.vx = pick({u.vx, v.vx}, s);
  r.vy = pick({u.vy, v.vy}, s);
  r.vz = pick({u.vz, v.vz}, s);
  return r;
}

// Step k of the current block: reaction step number and buffer parity.
struct StepInfo {
  uint32_t step, par;
};

__device__ __forceinline__ StepInfo step_info(const Ctl* c, int k) {
  // uniform over the launch (scalar registers, scalar selects of buffers)
  const uint32_t s0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c->step0);
  const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c->par0);
  return StepInfo{s0 + (uint32_t)k, (p0 + (uint32_t)k) & 1u};
}

// Buffers kept by step mod 3 (fused binning).
__device__ __forceinline__ uint32_t mod3(uint32_t step) { return step % 3u; }

// Inclusive prefix sum over the wavefront with DPP: shifts by 1, 2, 4 and 8
// lanes within each row of 16, then the row broadcasts of lanes 15 and 31
// (lanes without a source add 0).  Every lane of the wavefront must be
// active.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return x;
}

// The number of lanes below this one set in b.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long b) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
}

// Orders a wavefront's LDS accesses before and after it (its lanes exchange
// data through LDS without a workgroup barrier).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Exclusive prefix sum over the workgroup (wavefront scans, then the
// wavefront totals through LDS, read by every thread).  Every thread of the
// block must call it, with every lane active.
template <int kT = kThreads, bool kReuse = true>
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* s_wave,
                                                    uint32_t& total) {
  constexpr int nw = kT / 64;
  const int lane = __lane_id(), w = threadIdx.x / 64;
  const uint32_t x = wave_scan_incl(v);
  if (lane == 63) s_wave[w] = x;
  __syncthreads();
  uint32_t below = 0, all = 0;
#pragma unroll
  for (int i = 0; i < nw; ++i) {
    const uint32_t t = s_wave[i];
    below += i < w ? t : 0u;
    all += t;
  }
  total = all;
  if (kReuse) __syncthreads();  // s_wave is free for the next call
  return below + x - v;
}

// Adds v of every lane to *dst with one LDS atomic per wavefront (every lane
// of the wave must call it, with every lane active).
__device__ __forceinline__ void wave_add(int* dst, int v) {
  const int t = (int)wave_scan_incl((uint32_t)v);  // lane 63: the wavefront's sum
  if (__lane_id() == 63 && t) atomicAdd(dst, t);
}

// ---------------------------------------------------------------------------
// Control block set-up (a kernel rather than a memset/memcpy so that a
// captured graph may hold it).  A full reset selects storage set 0 and
// parity 0 (the caller clears both cell-count buffers with it).
// ---------------------------------------------------------------------------
__global__ void k_ctl_reset(Ctl* c, uint32_t step, int full) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    c->step0 = step;
    if (full) {
      c->par0 = 0;
      c->err = 0;
      c->set = 0;
      for (int p = 0; p < 2; ++p) {
        c->ovf_n[p] = 0;
        c->ret_ovf[p] = 0;
        c->nwin_ovf[p] = 0;
      }
      c->stats_n0 = 0;
      c->log_n = 0;
    }
  }
}

// Position validation and the roles after a load.
__global__ __launch_bounds__(kThreads) void k_classify(Dev d) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.n) return;
  const Arr a = pick_set(d, 0);
  const float x = pick(a.x, 0)[k], y = pick(a.y, 0)[k], z = pick(a.z, 0)[k];
  const bool ok = (x >= 0.0f && x < d.L) && (y >= 0.0f && y < d.L) && (z >= 0.0f && z < d.L);
  if (!ok) set_err(d.ctl, PR_EINVAL);
  a.role[k] = role_of(d, a.typ[k], a.st[k]);
}

// Identity storage order after a load (slot == id), cleared T flags.
__global__ __launch_bounds__(kThreads) void k_identity(Dev d) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.n) return;
  if (pick_set(d, 0).id) pick_set(d, 0).id[k] = k;
  if (d.slot_of) d.slot_of[k] = k;
  d.tflag[k] = 0;
}

// ---------------------------------------------------------------------------
// Synthetic jittered-lattice initial configuration (storage set 0, parity 0,
// slot == id).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_generate(Dev d, int kind, unsigned long long gseed,
                                                       float c0, float a, int nl,
                                                       unsigned long long thr_x) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.n) return;
  const Arr o = pick_set(d, 0);
  const unsigned long long n3 = (unsigned long long)nl * nl * nl;
  const unsigned long long s = ((unsigned long long)k * 2147483647ull) % n3;
  const int ix = (int)(s % nl), iy = (int)((s / nl) % nl),
            iz = (int)(s / ((unsigned long long)nl * nl));
  int32_t S[3];
  ih12(0u, (uint32_t)k, 2u, gseed, S);
  const float px = __fmul_rn(__fadd_rn((float)ix, 0.5f), a);
  const float py = __fmul_rn(__fadd_rn((float)iy, 0.5f), a);
  const float pz = __fmul_rn(__fadd_rn((float)iz, 0.5f), a);
  pick(o.x, 0)[k] = wrap_box(__fadd_rn(px, __fmul_rn((float)S[0], c0)), d.L);
  pick(o.y, 0)[k] = wrap_box(__fadd_rn(py, __fmul_rn((float)S[1], c0)), d.L);
  pick(o.z, 0)[k] = wrap_box(__fadd_rn(pz, __fmul_rn((float)S[2], c0)), d.L);
  const W4 w = philox(0u, (uint32_t)k, 0u, 3u, gseed);
  const bool pick = (unsigned long long)w.w0 < thr_x;
  if (kind == 0) {
    o.typ[k] = pick ? 1 : 0;
    o.st[k] = pick ? 4 : 2;
  } else {
    o.typ[k] = 0;
    o.st[k] = pick ? 2 : 0;
  }
  for (int b = 0; b < d.B; ++b) o.adj[(size_t)k * d.B + b] = -1;
}

// ---------------------------------------------------------------------------
// Closing a step, group g (one workgroup of kThreads): the counters of sweep
// workgroups g*kGroup .. +kGroup summed into the step's partial record and
// their staged bonds appended to the bond log (one reservation per group; rows
// of a step end up in group order and readers order them by id_A).  Group 0
// also takes the bonds beyond the staging windows and resets the step's
// per-parity counters.
// ---------------------------------------------------------------------------
static_assert(kWinCap >= 2, "the closing reads two staged bonds ahead");
__device__ void close_group(const Dev& d, uint32_t par, uint32_t step, uint32_t sidx, int g,
                            uint32_t* s_wave) {
  __shared__ int s_sum[kPart];
  __shared__ uint64_t s_row;
  Ctl* c = d.ctl;
  const int tid = threadIdx.x;
  if (tid < kPart) s_sum[tid] = 0;
  const int w = g * kGroup + tid;
  const int2* staged = pick(d.wgw, par) + w * kWinCap;
  int o[kWgOut] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  // a workgroup stages 0.3 bonds per step on average: its first two are read
  // with its counters, before their number is known (a window holds
  // kWinCap >= 2), which saves a dependent round trip in the common case
  int2 pre[2] = {make_int2(0, 0), make_int2(0, 0)};
  if (w < d.nwg_sweep) {
    const int32_t* src = pick(d.wgo, par) + w * kWgOut;
#pragma unroll
    for (int q = 0; q < kWgOut; ++q) o[q] = src[q];
    pre[0] = staged[0];
    pre[1] = staged[1];
  }
  // the A's of the step: counted by the sweep workgroups (fused binning), else
  // by the binning workgroups (strided over the groups)
  int a_elig = d.fuse ? o[kOutAElig] : 0;
  for (int q = w; !d.fuse && q < d.nwg_prep; q += d.ngroups * kGroup)
    a_elig += pick(d.abst, par)[q];
  const uint32_t nw = (uint32_t)min(o[kOutBonds], kWinCap);
  uint32_t tot = 0;
  const uint32_t off = block_scan_excl(nw, s_wave, tot);
  const uint32_t nwov = g == 0 ? c->nwin_ovf[par] : 0u;
  if (tid == 0 && tot + nwov > 0) s_row = atomicAdd((unsigned long long*)&c->log_n,
                                                    (unsigned long long)(tot + nwov));
  // partial layout: a_elig, t_elig, in_rc, drawn, excluded, proposals, bonds, lost
  const int v[kPart] = {a_elig,         o[kOutTElig], o[kOutInRc], o[kOutDrawn],
                        o[kOutExcl],    o[kOutProp],  o[kOutBonds], o[kOutLost]};
#pragma unroll
  for (int q = 0; q < kPart; ++q) wave_add(&s_sum[q], v[q]);
  __syncthreads();
  const uint64_t row0 = s_row;
  for (uint32_t e = 0; e < nw; ++e) {
    const uint64_t row = row0 + off + e;
    const int2 b = e < 2 ? pre[e] : staged[e];
    if ((int64_t)row < d.log_cap) {
      d.log[3 * row] = (int32_t)step;
      d.log[3 * row + 1] = b.x;
      d.log[3 * row + 2] = b.y;
    }
  }
  if (g == 0) {
    for (uint32_t e = tid; e < nwov; e += blockDim.x) {
      const uint64_t row = row0 + tot + e;
      const int2 b = pick(d.wov, par)[e];
      if ((int64_t)row < d.log_cap) {
        d.log[3 * row] = (int32_t)step;
        d.log[3 * row + 1] = b.x;
        d.log[3 * row + 2] = b.y;
      }
    }
  }
  __syncthreads();
  if (tid < kPart && (int64_t)sidx < d.part_cap)
    d.part[((size_t)sidx * d.ngroups + g) * kPart + tid] = s_sum[tid];
  if (g == 0 && tid == 0) {
    c->ovf_n[par] = 0;
    c->ret_ovf[par] = 0;
    c->nwin_ovf[par] = 0;
  }
}

// ---------------------------------------------------------------------------
// k_prep: [closing groups of step k - 1 when k > 0][binning of the A-role
// particles, kThreads * kPrepRoles slots per block].
// ---------------------------------------------------------------------------
__device__ __forceinline__ void prep_body(const Dev& d, int k, int blk) {
  __shared__ int s_na;
  __shared__ uint32_t s_wave[kThreads / 64 + 1];
  const StepInfo si = step_info(d.ctl, k);
  const Arr a = pick_set(d, d.ctl->set & 1u);
  const int ncl = k > 0 ? d.ngroups : 0;
  int b = blk;
  if (b < ncl) {  // closing groups of the previous step of the block
    close_group(d, si.par ^ 1u, si.step - 1u, d.ctl->stats_n0 + (uint32_t)k - 1u, b, s_wave);
    return;
  }
  b -= ncl;
  // binning of the A's: each lane scans kPrepRoles role bytes, the slots of
  // the wavefront's A's are compacted into LDS (ballot-free: a wave prefix
  // sum of the per-lane counts) and handled one per lane.  An A's record
  // holds its re-jittered position (the same draws as the sweep's), id, slot
  // and adjacency row.
  __shared__ int32_t s_list[kThreads / 64][kPrepRoles * 64];
  if (threadIdx.x == 0) s_na = 0;
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  const int i0 = (b * kThreads + threadIdx.x) * kPrepRoles;
  const bool ok = read_err(d.ctl) == 0;
  uint32_t rw[kPrepRoles / 4] = {0u, 0u, 0u, 0u};
  if (ok && i0 + kPrepRoles <= d.n) {
    const uint4 v = *(const uint4*)(a.role + i0);
    rw[0] = v.x;
    rw[1] = v.y;
    rw[2] = v.z;
    rw[3] = v.w;
  } else if (ok && i0 < d.n) {
#pragma unroll
    for (int q = 0; q < kPrepRoles / 4; ++q)
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + 4 * q + e;
        if (i < d.n) rw[q] |= (uint32_t)a.role[i] << (8 * e);
      }
  }
  int na = 0;
  const bool multi = d.nrules > 1;
#pragma unroll
  for (int q = 0; q < kPrepRoles / 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) na += role_is_a((rw[q] >> (8 * e)) & 0xFFu, multi);
  const uint32_t incl = wave_scan_incl((uint32_t)na);
  const int wtot = __builtin_amdgcn_readlane((int)incl, 63);
  int at = (int)incl - na;
#pragma unroll
  for (int q = 0; q < kPrepRoles / 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (role_is_a((rw[q] >> (8 * e)) & 0xFFu, multi)) s_list[wv][at++] = i0 + 4 * q + e;
  __syncthreads();
  for (int e = lane; e < wtot; e += 64) {
    const int i = s_list[wv][e];
    float x = pick(a.x, si.par)[i], y = pick(a.y, si.par)[i], z = pick(a.z, si.par)[i];
    const int id = a.id ? a.id[i] : i;
    int4 q4 = make_int4(-1, -1, -1, -1);
    if (d.adj_staged) {
      const int32_t* row = a.adj + (size_t)i * d.B;
      q4.x = row[0];
      if (d.B > 1) q4.y = row[1];
      if (d.B > 2) q4.z = row[2];
      if (d.B > 3) q4.w = row[3];
    }
    if (d.jitter && d.jit_c != 0.0f) {
      int32_t S[3];
      ih4(si.step, (uint32_t)id, 1u, d.seed, S);
      x = wrap_box(__fadd_rn(x, __fmul_rn((float)S[0], d.jit_c)), d.L);
      y = wrap_box(__fadd_rn(y, __fmul_rn((float)S[1], d.jit_c)), d.L);
      z = wrap_box(__fadd_rn(z, __fmul_rn((float)S[2], d.jit_c)), d.L);
    }
    const int c = cell_of(d, x, y, z);
    const uint32_t r = atomicAdd(&pick(d.cnt, si.par)[c], 1u);
    const float4 rec = make_float4(x, y, z, __int_as_float(id));
    if (r < (uint32_t)kCellCap) {
      const size_t ri = rec_at(d, c, r);
      d.rec[ri] = rec;
      d.rsa[ri] = i;
      if (d.adj_staged) d.radj[ri] = q4;
    } else {
      const uint32_t o = atomicAdd(&d.ctl->ovf_n[si.par], 1u);
      pick(d.ovf, si.par)[o] = rec;
      pick(d.ovf_sa, si.par)[o] = i;
    }
  }
  if (lane == 0 && wtot) atomicAdd(&s_na, wtot);
  __syncthreads();
  if (threadIdx.x == 0) pick(d.abst, si.par)[b] = s_na;
}

// Closes step k of the block (one workgroup per closing group).
__device__ __forceinline__ void close_body(const Dev& d, int k, int g) {
  __shared__ uint32_t s_wave[kThreads / 64 + 1];
  const StepInfo si = step_info(d.ctl, k);
  close_group(d, si.par, si.step, d.ctl->stats_n0 + (uint32_t)k, g, s_wave);
}

// Advances the block origin by K steps (after the block's last step closed).
__device__ __forceinline__ void advance_ctl(Ctl* c, int K) {
  c->step0 += (uint32_t)K;
  c->par0 = (c->par0 + (uint32_t)K) & 1u;
  c->stats_n0 += (uint32_t)K;
}

// ---------------------------------------------------------------------------
// Pair tests shared by the sweep and the resolution.
// ---------------------------------------------------------------------------
// The 2x2x2 block of coarse cells around a particle: per dimension the cells
// floor(u - 1/2) and floor(u - 1/2) + 1 (periodic), u = x / cell width.
__device__ __forceinline__ void lo_hi(float v, float inv_w, int nc, int& c0, int& c1) {
  const int l = (int)floorf(__fsub_rn(__fmul_rn(v, inv_w), 0.5f));
  c0 = l < 0 ? l + nc : l;
  c1 = l + 1 >= nc ? l + 1 - nc : l + 1;
  if (nc == 1) c0 = c1 = 0;
}

// floor(v) as an integer in one instruction (v is a finite coordinate in
// cell units, far inside the int range): identical to (int)floorf(v)
__device__ __forceinline__ int floor_int(float v) {
  int r;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(v));
  return r;
}

// Local coordinate, in a staged region whose first cell is `base`, of the
// lower cell floor(u - 1/2) of a particle's 2x2x2 block (u = v / width; the
// cell index, in [-1, nc - 1], is taken mod nc): in [0, nc - 1].
__device__ __forceinline__ int local_lo(float v, float inv_w, int base, int nc) {
  const int l = floor_int(__fsub_rn(__fmul_rn(v, inv_w), 0.5f)) - base;
  return l < 0 ? l + nc : l;
}

__device__ __forceinline__ float dist2(const Dev& d, float xj, float yj, float zj, float4 a) {
  const float dx = min_image(__fsub_rn(xj, a.x), d.L, d.halfL);
  const float dy = min_image(__fsub_rn(yj, a.y), d.L, d.halfL);
  const float dz = min_image(__fsub_rn(zj, a.z), d.L, d.halfL);
  return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
}

// dist2 of two positions whose difference is known to lie within
// (-L/2, L/2) in every component (the minimum image is the identity there).
__device__ __forceinline__ float dist2_plain(float xj, float yj, float zj, float4 a) {
  const float dx = __fsub_rn(xj, a.x), dy = __fsub_rn(yj, a.y), dz = __fsub_rn(zj, a.z);
  return __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
}

__device__ __forceinline__ bool row_has(const int32_t* row, int B, int32_t v) {
  for (int b = 0; b < B; ++b)
    if (row[b] == v) return true;
  return false;
}

// The A records of a step: per-cell counts and bucket records with the A's
// slots, then the overflow list.
struct Buckets {
  const uint32_t* cnt;
  const float4* rec;
  const int32_t* sa;
  const float4* ovf;
  const int32_t* osa;
  uint32_t novf;
};

// Those of step `step` (parity par): filled by the binning kernel (kF =
// false), or with fused binning by the previous step's sweep.
template <bool kF>
__device__ __forceinline__ Buckets step_buckets(const Dev& d, uint32_t par, uint32_t step) {
  if (kF) {
    const uint32_t q = mod3(step);
    return Buckets{d.fcnt[q], pick(d.frec, par), pick(d.fsa, par), pick(d.fovf, par),
                   pick(d.fovf_sa, par), d.ctl->fovf_n[q]};
  }
  return Buckets{pick(d.cnt, par), d.rec, d.rsa, pick(d.ovf, par), pick(d.ovf_sa, par),
                 d.ctl->ovf_n[par]};
}

// Visits the A records (record, slot of the A) of the 2x2x2 cell block around
// (x, y, z) in the buckets, then the overflow list.
template <typename F>
__device__ __forceinline__ void for_global_records(const Dev& d, const Buckets& bk, float x,
                                                   float y, float z, F f) {
  const int nc = d.nc;
  int cx0, cx1, cy0, cy1, cz0, cz1;
  lo_hi(x, d.inv_w, nc, cx0, cx1);
  lo_hi(y, d.inv_w, nc, cy0, cy1);
  lo_hi(z, d.inv_w, nc, cz0, cz1);
  const int m = nc > 1 ? 2 : 1;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int ia = q >> 2, ib = (q >> 1) & 1, ie = q & 1;
    if (ia >= m || ib >= m || ie >= m) continue;
    const int c = ((ia ? cz1 : cz0) * nc + (ib ? cy1 : cy0)) * nc + (ie ? cx1 : cx0);
    uint32_t nr = bk.cnt[c];
    nr = nr < (uint32_t)kCellCap ? nr : (uint32_t)kCellCap;
    for (uint32_t r = 0; r < nr; ++r) f(bk.rec[rec_at(d, c, r)], bk.sa[rec_at(d, c, r)]);
  }
  for (uint32_t r = 0; r < bk.novf; ++r) f(bk.ovf[r], bk.osa[r]);
}

// Staged region of a brick along one dimension: the brick's cells plus one
// halo cell per side (the whole grid in single-brick mode).
__device__ __forceinline__ void region_dim(const Dev& d, int bc, int& base, int& ext) {
  if (d.nbricks == 1) {
    base = 0;
    ext = d.nc;
  } else {
    const int lo = bc * d.bs;
    const int sz = min(d.bs, d.nc - lo);
    base = lo == 0 ? d.nc - 1 : lo - 1;
    ext = sz + 2;
  }
}

// q = w / nb and r = w mod nb for a brick index: a high multiply by
// floor(2^32 / nb) is below the quotient by at most one.
__device__ __forceinline__ int div_nb(const Dev& d, int w, int& r) {
  uint32_t q = __umulhi((uint32_t)w, d.nb_m);
  int rr = w - (int)q * d.nb;
  if (rr >= d.nb) {
    q++;
    rr -= d.nb;
  }
  r = rr;
  return (int)q;
}

// x / d for the small operands of a staged region (x < 1024, d <= 64) as
// (x * m) >> 16 with m = ceil(2^16 / d): exact there, and two instructions
// instead of an integer division.
__device__ __forceinline__ uint32_t recip16(uint32_t d) { return (65536u + d - 1u) / d; }
__device__ __forceinline__ int div_small(int x, uint32_t m) { return (int)(((uint32_t)x * m) >> 16); }

// ---------------------------------------------------------------------------
// Fused binning.  The sweep of step k writes the A records of step k + 1 into
// cell buckets of their own (counts by step mod 3, records by step parity):
// each A's own sweep workgroup re-jitters it once more and appends it to the
// bucket of its cell.  The resolve of step k then drops the record of an A
// whose bond ends its A role (its x becomes NaN: no distance test with it
// passes) and appends a T that takes the A role.
// ---------------------------------------------------------------------------
// Appends the record of A (slot, id) at (x, y, z) to the buckets of step
// `step` (parity par) and notes where it went.
__device__ __forceinline__ void fuse_bin(const Dev& d, uint32_t par, uint32_t step, int slot,
                                         uint32_t id, float x, float y, float z) {
  const int c = cell_of(d, x, y, z);
  const uint32_t r = atomicAdd(&d.fcnt[mod3(step)][c], 1u);
  const float4 rec = make_float4(x, y, z, __uint_as_float(id));
  if (r < (uint32_t)kCellCap) {
    const int q = (int)rec_at(d, c, r);
    pick(d.frec, par)[q] = rec;
    pick(d.fsa, par)[q] = slot;
    d.apos[slot] = q;
  } else {
    const uint32_t o = atomicAdd(&d.ctl->fovf_n[mod3(step)], 1u);
    pick(d.fovf, par)[o] = rec;
    pick(d.fovf_sa, par)[o] = slot;
    d.apos[slot] = -1 - (int)o;
  }
}

// Drops the record of the next step (parity par) at q (a bucket record, or
// overflow entry -1 - q), or that of the A in `slot`.
__device__ __forceinline__ void fuse_drop_at(const Dev& d, uint32_t par, int q) {
  float* x = q >= 0 ? &pick(d.frec, par)[q].x : &pick(d.fovf, par)[-1 - q].x;
  *x = __int_as_float(0x7FC00000);  // quiet NaN
}
__device__ __forceinline__ void fuse_drop(const Dev& d, uint32_t par, int slot) {
  fuse_drop_at(d, par, d.apos[slot]);
}

// The brick of sweep workgroup w (1 << wshift workgroups share one).
__device__ __forceinline__ int brick_of(const Dev& d, int w) { return w >> d.wshift; }

// Slot range of sweep/resolve workgroup w.
template <bool kBrick>
__device__ __forceinline__ void range_of(const Dev& d, int w, int& s0, int& s1) {
  if (kBrick) {
    const int b = brick_of(d, w);
    s0 = d.bstart[b];
    s1 = d.bstart[b + 1];
    // its share of the brick's slots
    const int per = (s1 - s0 + (1 << d.wshift) - 1) >> d.wshift;
    s0 = min(s1, s0 + (w - (b << d.wshift)) * per);
    s1 = min(s1, s0 + per);
  } else {
    s0 = w * kThreads;
    s1 = min(d.n, s0 + kThreads);
  }
}

// Acceptance, exclusion and A-side choice of an in-range pair with draws r
// (steps 2-5).  A retained pair lowers the A's key (w1, id_T) with a 64-bit atomicMin whose
// result is not needed, flags its T and is handed to the resolve in the
// workgroup's list.  arow: the A's adjacency row staged with its record
// (nullptr: the row is read from the particle arrays).
// The sweep counts in LDS (cnt: the workgroup's counters by WgOut), one atomic
// per wavefront and event: per-lane counters would hold registers through the
// scan and need a wavefront sum each at the end.
__device__ __forceinline__ void count_one(int* c) { atomicAdd(c, 1); }

struct RetList {
  int* n;
  int4* ent;
  uint32_t *w1, *w2;  // w1: several rules only
};

// The adjacency row of width B <= kAdjStage at `row`, every entry loaded at once.
__device__ __forceinline__ int4 row_load(const int32_t* row, int B) {
  int4 r = make_int4(-1, -1, -1, -1);
  r.x = row[0];
  if (B > 1) r.y = row[1];
  if (B > 2) r.z = row[2];
  if (B > 3) r.w = row[3];
  return r;
}

// Whether v is in the adjacency row of width B at `row`.
__device__ __forceinline__ bool row_has_wide(const int32_t* row, int B, int32_t v) {
  if (B > kAdjStage) return row_has(row, B, v);
  const int4 r = row_load(row, B);
  return r.x == v || r.y == v || r.z == v || r.w == v;
}

// Whether idj is bonded to the A in slot sa (arow: the A's row staged with its
// record, nullptr: the row is read from the particle arrays).
__device__ __forceinline__ bool pair_bonded(const Dev& d, const Arr& a, int sa, uint32_t idj,
                                            const int4* arow) {
  const int v = (int)idj;
  if (!arow) return row_has_wide(a.adj + (size_t)sa * d.B, d.B, v);
  const int4 q = *arow;
  return q.x == v || q.y == v || q.z == v || q.w == v;
}

__device__ __forceinline__ void retain(const Dev& d, const Arr& a, W4 r, int ida, int sa,
                                       uint32_t idj, int sj, const int4* arow, int* cnt,
                                       const RetList& l) {
  if (!((unsigned long long)r.w0 < d.thresh)) return;
  count_one(&cnt[kOutDrawn]);
  if (d.rule.exclude && pair_bonded(d, a, sa, idj, arow)) {
    count_one(&cnt[kOutExcl]);
    return;
  }
  d.tflag[sj] = 1;
  atomicMin(&d.slotA[ida], ((unsigned long long)r.w1 << 32) | (unsigned long long)idj);
  const int p = atomicAdd(l.n, 1);
  if (p < kRetCap) {
    l.ent[p] = make_int4(ida, sa, sj, (int)idj);
    l.w2[p] = r.w2;
  }
}

// The nearest selection (LAMMPS fix bond/create, Sec. IV A of the paper): an
// in-range pair that is not excluded as bonded lowers the A's key (r2 bits,
// id_T) and its T's (r2 bits, id_A), the T's in LDS (r2 >= 0 orders like its
// bits, equal distances go to the lower id).
__device__ __forceinline__ void near_pair(int ida, uint32_t idj, float r2, bool excluded, int* cnt,
                                          unsigned long long* best_a,
                                          unsigned long long* best_t) {
  if (excluded) {
    count_one(&cnt[kOutExcl]);
    return;
  }
  const unsigned long long rb = (unsigned long long)__float_as_uint(r2) << 32;
  atomicMin(best_a, rb | idj);
  atomicMin(best_t, rb | (uint32_t)ida);
}

// The A's of a nearest sweep's workgroup, (id, slot) of the first kNearList of
// them in the place of its retained pairs, for the resolve.
constexpr int kNearList = kRetCap * (int)(sizeof(int4) / sizeof(int2));
static_assert(kNearList == 64, "one wavefront reads the list");
__device__ __forceinline__ void near_list(bool is_src, int id, int slot, int2* list, int* n) {
  const unsigned long long m = __ballot(is_src);
  if (!m) return;
  int at = 0;
  if (__lane_id() == 0) at = atomicAdd(n, (int)__popcll(m));
  at = __builtin_amdgcn_readlane(at, 0) + (int)lanes_below(m);
  if (is_src && at < kNearList) list[at] = make_int2(id, slot);
}

// ---------------------------------------------------------------------------
// Several concurrent rules (nrules > 1): Table I generalised over the rules.
// Every rule contributes candidates with its own draw (counter word 3 = the
// rule's tag); each A picks among its accepted candidates of all rules the
// smallest (w1, id_T), the lower rule on a tie; each T keeps the smallest
// (w2, id_A) of the pairs that picked it; a particle that wins both as an A
// and as a T keeps the pair with the smaller (w3, partner id, rule) and a
// pair is bonded only if both of its particles keep it.  Three kernels after
// the binning: the sweep (draws, A-side picks by 64-bit atomicMin, the
// retained pairs in the workgroup's list), the T-side choice and the final
// choice with the bonds.
// ---------------------------------------------------------------------------
// (each rule's word is read as a scalar before the selection, so that the
// kernel argument is not indexed dynamically, which would copy it to scratch)
__device__ __forceinline__ uint32_t rule_tag(const Dev& d, int r) {
  uint32_t t = 0;
#pragma unroll
  for (int q = 0; q < kMaxRules; ++q) {
    const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)d.mr[q].tag);
    t = r == q ? v : t;
  }
  return t;
}

__device__ __forceinline__ void rule_deltas(const Dev& d, int r, int32_t& da, int32_t& dt) {
  da = 0;
  dt = 0;
#pragma unroll
  for (int q = 0; q < kMaxRules; ++q) {
    const int32_t va = __builtin_amdgcn_readfirstlane(d.mr[q].r.d_a),
                  vt = __builtin_amdgcn_readfirstlane(d.mr[q].r.d_t);
    da = r == q ? va : da;
    dt = r == q ? vt : dt;
  }
}

__device__ __forceinline__ bool key_less(unsigned long long k1, int r1, unsigned long long k2,
                                         int r2) {
  return k1 < k2 || (k1 == k2 && r1 < r2);
}

// Visits the rules r under which the pair (A record at slot sa, T of role
// mask rt) is a candidate at squared distance r2, in increasing r:
// f(r, draw words, drawn but excluded as bonded, drawn).
template <typename F>
__device__ __forceinline__ void multi_candidates(const Dev& d, const Arr& a, uint32_t step,
                                                 uint32_t rt, int sa, int ida, uint32_t idj,
                                                 float r2, F f, const int4* arow = nullptr) {
  const uint32_t both = rt & ((uint32_t)a.role[sa] >> 4);
  if (!both) return;
  // not unrolled: four copies of the generator took the sweep beyond the 72
  // registers of seven waves per SIMD, and at six the 1728 bricks of 1,048,576
  // particles need a second round of workgroups (40.5 us per step; 33.9 now)
#pragma unroll 1
  for (int r = 0; r < d.nrules; ++r) {
    const RuleX& q = d.mr[r];
    if (!((both >> r) & 1u) || !(r2 < q.rc2)) continue;
    const W4 w = philox(step, (uint32_t)ida, idj, q.tag, d.seed);
    const bool acc = w.w0 < q.thresh;
    f(r, w, acc && q.r.exclude && pair_bonded(d, a, sa, idj, arow), acc);
  }
}

// The candidates of an in-range pair (within the largest cutoff) under every
// rule both roles allow: draws, exclusion, A-side pick, and the retained ones
// into the list with their rule in bits 30-31 of id_T (ids are below 2^30).
__device__ __forceinline__ void multi_pair(const Dev& d, const Arr& a, uint32_t step, uint32_t rt,
                                           int ida, int sa, uint32_t idj, int sj, float r2,
                                           const int4* arow, int* cnt, const RetList& l) {
  if ((uint32_t)ida == idj) return;  // a particle with both roles is no partner of itself
  multi_candidates(d, a, step, rt, sa, ida, idj, r2, [&](int r, W4 w, bool ex, bool acc) {
    count_one(&cnt[kOutInRc]);
    if (!acc) return;
    count_one(&cnt[kOutDrawn]);
    if (ex) {
      count_one(&cnt[kOutExcl]);
      return;
    }
    d.tflag[sj] = 1;
    atomicMin(&d.slotA[ida], ((unsigned long long)w.w1 << 32) | idj);
    const int p = atomicAdd(l.n, 1);
    if (p < kRetCap) {
      l.ent[p] = make_int4(ida, sa, sj, (int)(idj | ((uint32_t)r << 30)));
      l.w1[p] = w.w1;
      l.w2[p] = w.w2;
    }
  }, arow);
}

// ---------------------------------------------------------------------------
// The scan of a T's block in the staged records, the sweep's inner loop.  It
// looks for candidates, not for in-range pairs: positions are taken as 16-bit
// integers in units of L / 2^m (Dev::qscale, m >= 16, so that the integers wrap
// around exactly where the box does and their differences need no minimum
// image), two packed subtractions and two dot products give the squared
// distance in those units, and every pair within the cutoff passes (Dev::qthr
// allows for the rounding, scan_units).  The few others that pass (about 0.5%)
// fall at the exact FP32 test, which every candidate takes on full wavefronts
// from the queue.  The four runs of two x-adjacent cells are one sequence: a
// word D counts down in each of its bytes to the ends of the runs, the sign
// bits of the bytes say which runs are not yet done, and their dot product with
// the (byte) steps between the runs moves the index.  These words are the same
// for every T of a block: the staging writes them once per block (s_blk, while
// the records are on their way), instead of each T from eight cell offsets.
// Bound: VALU issue, of the trips of a wavefront's longest block (14 instructions
// each instead of 24 with one compare and select per run and FP32 distance, 30
// in a region that wraps in one axis and 42 beyond) and of what comes before
// them.  1,048,576 particles, 256 steps with load and read-out: 7.90 -> 7.80 ms
// by the integer test, 7.54 -> 7.42 by the words of the block and a bit per
// place for the hits; 4,194,304 (chain growth, blocks nearly empty), 128 steps:
// 8.28 -> 8.09 by the latter.
// ---------------------------------------------------------------------------
typedef short short2_t __attribute__((ext_vector_type(2)));

// A position in the scan's units: (x | y << 16, z).
__device__ __forceinline__ uint2 quant(const Dev& d, float x, float y, float z) {
  const uint32_t qx = (uint32_t)(int)__fmul_rn(x, d.qscale), qy = (uint32_t)(int)__fmul_rn(y, d.qscale),
                 qz = (uint32_t)(int)__fmul_rn(z, d.qscale);
  return make_uint2(__builtin_amdgcn_perm(qy, qx, 0x05040100u), qz & 0xFFFFu);
}

// Squared distance in the scan's units (32-bit wrap; every component difference
// is below 2^15 in magnitude).
__device__ __forceinline__ uint32_t quant_d2(uint2 a, uint2 b) {
  const short2_t dxy = __builtin_bit_cast(short2_t, a.x) - __builtin_bit_cast(short2_t, b.x);
  const short2_t dz = __builtin_bit_cast(short2_t, a.y) - __builtin_bit_cast(short2_t, b.y);
  return (uint32_t)__builtin_amdgcn_sdot2(dz, dz, __builtin_amdgcn_sdot2(dxy, dxy, 0, false), false);
}

// A block (first region cell l, ex cells per row, exy per layer; s_off: first
// record of each region cell) as the scan takes it: x the word D, y the steps
// between its runs (dy, dz) = (0,0), (1,0), (0,1), (1,1) of two cells each, and in
// the last byte minus what the index starts from.
__device__ __forceinline__ uint2 scan_entry(const uint16_t* s_off, int l, int ex, int exy) {
  static_assert(8 * kCellCap <= 127, "no borrow from byte to byte of D");
  const int l1 = l + ex, l2 = l + exy, l3 = l2 + ex;
  const int b0 = (int)s_off[l], b1 = (int)s_off[l1], b2 = (int)s_off[l2], b3 = (int)s_off[l3];
  const int p1 = (int)s_off[l + 2] - b0;
  const int p2 = p1 + (int)s_off[l1 + 2] - b1;
  const int p3 = p2 + (int)s_off[l2 + 2] - b2;
  const int tot = p3 + (int)s_off[l3 + 2] - b3;
  // record of place q: q + o3, plus (o2 - o3) while q < p3, (o1 - o2) while q
  // < p2 and (o0 - o1) while q < p1 (o: the run's first record less its place)
  const int o1 = b1 - p1, o2 = b2 - p2, o3 = b3 - p3;
  const uint32_t D =
      ((uint32_t)p1 | ((uint32_t)p2 << 8) | ((uint32_t)p3 << 16) | ((uint32_t)tot << 24)) +
      0x7F7F7F7Fu;
  // bytes -(step) mod 256: a set sign byte counts -128
  const uint32_t step = ((uint32_t)(o1 - b0) & 0xFFu) | (((uint32_t)(o2 - o1) & 0xFFu) << 8) |
                        (((uint32_t)(o3 - o2) & 0xFFu) << 16) | ((uint32_t)-o3 << 24);
  return make_uint2(D, step);
}
constexpr uint32_t kScanMax = 32;  // records of a block the scan's mask holds

// The staged record of place q (a block's word less q in every byte, q << 7).
__device__ __forceinline__ uint32_t scan_index(uint32_t D, uint32_t step, uint32_t q7) {
  return ((uint32_t)__builtin_amdgcn_sdot4((int)(D & 0x80808080u), (int)step, (int)q7, false) >>
          7) & 0xFFu;
}

// Candidates of the T at t among the staged records (s_qr) of block e (at most
// kScanMax records): a bit each, the last place's the lowest.
__device__ __forceinline__ uint32_t scan_block(const uint2* s_qr, uint2 e, uint2 t, uint32_t thr) {
  uint32_t m = 0, q7 = 0;
  while ((int32_t)e.x < 0) {  // the last byte: places left
    const uint32_t r = scan_index(e.x, e.y, q7);
    m = m + m + (quant_d2(s_qr[r], t) < thr ? 1u : 0u);
    e.x -= 0x01010101u;
    q7 += 128u;
  }
  return m;
}

// The staged record of a bit of scan_block's mask.
__device__ __forceinline__ uint32_t scan_record(uint2 e, uint32_t bit) {
  const uint32_t q = (e.x >> 24) - 0x80u - bit;
  return scan_index(e.x - q * 0x01010101u, e.y, q << 7);
}

// The selection a sweep is compiled for.
enum Policy { kRandom = 0, kNearest = 1, kMulti = 2 };

// Whether a role byte makes its particle a T / an A under the sweep's policy.
template <int kPol>
__device__ __forceinline__ bool pol_t(int role) {
  return kPol == kMulti ? (role & kMaskT) != 0 : role == kRoleT;
}

// ---------------------------------------------------------------------------
// k_sweep: every particle is re-jittered (resident systems) and written to
// the other position buffer; T's test the step's A records at their new
// positions.  Sorted storage: one workgroup per brick (or share of one), the A
// records of the brick and its halo (positions, ids, slots, adjacency rows)
// staged in LDS, each region cell's by the thread that read its count, and the
// brick's particles handled kTPass at a time.  A T whose 2x2x2 cell block lies in
// the staged region scans it for candidates (scan_block); the wavefront then
// reserves queue slots for all of them at once (ballot and mbcnt over the
// per-lane counts), and the queue takes the exact test and the draws on full
// wavefronts after the pass.  Every other T is deferred to a list and scanned
// again after the queue: T's with more than four candidates, of a block with
// more records than the scan's mask holds, or whose pairs find the queue
// full, in the staged records; in the global buckets particles that drifted
// out of the staged region since the last sort, bricks whose region holds
// more than kStageRecs records and steps with bucket overflow.  A deferred T
// enters the queue with none of its pairs, so every pair is drawn exactly
// once.  (Unsorted storage: dense_sweep_body.)
// ---------------------------------------------------------------------------
// One particle of a sweep pass, loaded with coalesced SoA reads.
struct Part {
  int role, id;
  float x, y, z;
};

__device__ __forceinline__ Part load_part(const Arr& a, const float* X, const float* Y,
                                          const float* Z, int slot, int s1) {
  Part q{kRoleNone, 0, 0.0f, 0.0f, 0.0f};
  if (slot < s1) {
    // 32-bit byte offsets (n < 2^30): the loads take the array base from
    // scalar registers and need no 64-bit address arithmetic
    const uint32_t bo = (uint32_t)slot * 4u;
    q.role = a.role[(uint32_t)slot];
    q.x = *(const float*)((const char*)X + bo);
    q.y = *(const float*)((const char*)Y + bo);
    q.z = *(const float*)((const char*)Z + bo);
    q.id = *(const int32_t*)((const char*)a.id + bo);
  }
  return q;
}

// The re-jittered position (identical arithmetic in k_prep and k_sweep).
__device__ __forceinline__ void rejitter(const Dev& d, uint32_t step, uint32_t id, float& x,
                                         float& y, float& z) {
  int32_t S[3];
  ih4(step, id, 1u, d.seed, S);
  x = wrap_box(__fadd_rn(x, __fmul_rn((float)S[0], d.jit_c)), d.L);
  y = wrap_box(__fadd_rn(y, __fmul_rn((float)S[1], d.jit_c)), d.L);
  z = wrap_box(__fadd_rn(z, __fmul_rn((float)S[2], d.jit_c)), d.L);
}

// kTwo: two region cells per thread while staging (brick edges above
// kOneCellBrick); else one, with the smaller tables.
// kF: fused binning (the sweep bins the next step's A records; sorted storage).
// kNt: the re-jittered positions stored non-temporally (Dev::nt_pos; random
// selection only).
// kPol: the selection (Policy).  The nearest selection and several rules need
// a queued pair's distance: it is computed again from the T's position, just
// written by this workgroup.  (Their pairs on full wavefronts from the queue
// and the next step's A's binned here, against sweeps of their own that took
// each pair where the scan met it, after a binning kernel: 1,048,576
// particles, nearest 39.1 + 8.4 -> 31.3 us, two rules 28.8 + 5.4 -> 28.0.)
template <int kPol, bool kTwo, bool kF = false, bool kNt = false>
__device__ __forceinline__ void sweep_body(const Dev& d0, int k, int w, int nwg) {
  const Dev& d = d0;
  constexpr int kCells = kTwo ? kStageCells : kStageCells1;  // region cells at most
  constexpr int kPer = kTPass / kThreads;
  constexpr int kTP = kPer * kThreads;
  constexpr uint32_t kQEmpty = 0xFFFFFFFFu;
  __shared__ float4 s_rec[kStageRecs];
  __shared__ uint2 s_qr[kStageRecs];      // the records' positions in the scan's units
  __shared__ int4 s_radj[kStageRecs];
  __shared__ int32_t s_rsa[kStageRecs];
  __shared__ uint16_t s_off[kCells + 1];  // first record of a region cell
  // the 2x2x2 block from each region cell on that has one (scan_entry)
  constexpr int kEdge = kTwo ? kMaxBrick + 2 : kOneCellBrick + 2;
  __shared__ uint2 s_blk[(kEdge - 1) * kEdge * kEdge - kEdge - 1];
  // queued candidate: local T | its block << 10 | bit of the scan's mask << 20
  __shared__ uint32_t s_q[kQueue];
  static_assert(kTP <= 1024 && kCells <= 1024 && kScanMax <= 32, "fields of a queued candidate");
  // ids of the pass's T's (nearest selection: read again with the position)
  __shared__ int32_t s_tid[kPol == kNearest ? 1 : kTP];
  __shared__ uint16_t s_def[kTP];            // deferred T's (local index in the pass)
  __shared__ int4 s_ent[kRetCap];  // retained pairs; nearest selection: the A's as (id, slot)
  __shared__ uint32_t s_ew1[kPol == kMulti ? kRetCap : 1], s_ew2[kPol == kNearest ? 1 : kRetCap];
  // nearest selection: the best key of each T of the pass, of each staged A
  __shared__ unsigned long long s_best[kPol == kNearest ? kTP : 1];
  __shared__ unsigned long long s_best_a[kPol == kNearest ? kStageRecs : 1];
  __shared__ uint32_t s_wave[kThreads / 64 + 1];
  __shared__ int s_cnt[5];
  __shared__ int s_qn, s_ndef, s_ne, s_dead;
  const int tid = threadIdx.x;
  if (tid < 5) s_cnt[tid] = 0;
  if (kPol == kNearest) {
    for (int q = tid; q < kTP; q += kThreads) s_best[q] = kEmpty;
    for (int q = tid; q < kStageRecs; q += kThreads) s_best_a[q] = kEmpty;
  }
  if (tid == 0) {
    s_qn = 0;
    s_ndef = 0;
    s_ne = 0;
    s_dead = read_err(d.ctl) != 0;
  }
  // staging at the top wave priority: the workgroups dispatched last stage
  // while the compute units already run the pass loops of the others, and
  // below those waves' priority their staging waits for issue slots
  __builtin_amdgcn_s_setprio(3);
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = si.par, step = si.step;
  const Arr a = pick_set(d, c->set & 1u);
  // positions of the previous step (parity par); the re-jittered ones are
  // written to parity par ^ 1
  const float *X = pick(a.x, par), *Y = pick(a.y, par), *Z = pick(a.z, par);
  float *XW = pick(a.x, par ^ 1u), *YW = pick(a.y, par ^ 1u), *ZW = pick(a.z, par ^ 1u);
  const bool jit = d.jitter && d.jit_c != 0.0f;
  const Buckets bk = step_buckets<kF>(d, par, step);
  const RetList rl{&s_ne, s_ent, s_ew1, s_ew2};
  int s0, s1;
  range_of<true>(d, w, s0, s1);
  int bx = 0, ex = 0, by = 0, ey = 0, bz = 0, ez = 0;
  bool staged = false;
  const int nc = d.nc;
  int ncs = 0;
  uint32_t mine = 0, mine2 = 0, m_exy = 0, m_ex = 0;
  int gc = 0, gc2 = 0;  // global cells of this thread's region cells
  auto put_rec = [&](uint32_t r, const float4& v) {
    s_rec[r] = v;
    // a dropped record's x is NaN, which has no integer: any position will do,
    // the exact test lets no pair with it pass
    s_qr[r] = quant(d, v.x == v.x ? v.x : 0.0f, v.y, v.z);
  };
  // global cell of region cell cl (region cells in z, y, x order)
  auto region_cell = [&](int cl) {
    const int lz = div_small(cl, m_exy), rem = cl - lz * ex * ey;
    const int ly = div_small(rem, m_ex), lx = rem - ly * ex;
    int cx = bx + lx, cy = by + ly, cz = bz + lz;
    cx -= cx >= nc ? nc : 0;
    cy -= cy >= nc ? nc : 0;
    cz -= cz >= nc ? nc : 0;
    return (cz * nc + cy) * nc + cx;
  };
  int bxc, byc;
  const int bzc = div_nb(d, div_nb(d, brick_of(d, w), bxc), byc);
  region_dim(d, bxc, bx, ex);
  region_dim(d, byc, by, ey);
  region_dim(d, bzc, bz, ez);
  ncs = ex * ey * ez;
  m_exy = recip16((uint32_t)(ex * ey));
  m_ex = recip16((uint32_t)ex);
  // the record counts of this thread's region cells (2 tid and 2 tid + 1,
  // or tid), issued first
#pragma unroll
  for (int h = 0; h < (kTwo ? 2 : 1); ++h) {
    const int cl = kTwo ? 2 * tid + h : tid;
    if (cl < ncs) {
      const int gcl = region_cell(cl);
      (h ? gc2 : gc) = gcl;
      (h ? mine2 : mine) = bk.cnt[gcl];
    }
  }
  // the first particle of the first pass, issued behind the record counts
  // (memory operations complete in issue order)
  Part cur = load_part(a, X, Y, Z, s0 + tid, s1);
  mine = mine < (uint32_t)kCellCap ? mine : (uint32_t)kCellCap;
  mine2 = mine2 < (uint32_t)kCellCap ? mine2 : (uint32_t)kCellCap;
  uint32_t total = 0;
  const uint32_t off = block_scan_excl<kThreads, false>(mine + mine2, s_wave, total);
  staged = total <= (uint32_t)kStageRecs && bk.novf == 0;
  // each thread stages the records of its own region cells: the first
  // kFirst of a cell loaded together, the rare rest one after another
  constexpr int kFirst = kTwo ? 2 : 4;
  const int cl0 = kTwo ? 2 * tid : tid;
  const size_t nn = (size_t)d.ncell;  // rank r of a cell lies r * ncell records further
  // the first records in registers (named, so that none of them lives in
  // scratch), loaded together, then written to LDS
  float4 rv0 = make_float4(0.f, 0.f, 0.f, 0.f), rv1 = rv0, rv2 = rv0, rv3 = rv0;
  int32_t sv0 = 0, sv1 = 0, sv2 = 0, sv3 = 0;
  auto rec_load = [&](size_t r0, uint32_t m) {
    if (m > 0u) { rv0 = bk.rec[r0]; sv0 = bk.sa[r0]; }
    if (m > 1u) { rv1 = bk.rec[r0 + nn]; sv1 = bk.sa[r0 + nn]; }
    if (kFirst > 2 && m > 2u) { rv2 = bk.rec[r0 + 2 * nn]; sv2 = bk.sa[r0 + 2 * nn]; }
    if (kFirst > 3 && m > 3u) { rv3 = bk.rec[r0 + 3 * nn]; sv3 = bk.sa[r0 + 3 * nn]; }
  };
  auto rec_put = [&](size_t r0, uint32_t o, uint32_t m) {
    if (m > 0u) { put_rec(o, rv0); s_rsa[o] = sv0; }
    if (m > 1u) { put_rec(o + 1, rv1); s_rsa[o + 1] = sv1; }
    if (kFirst > 2 && m > 2u) { put_rec(o + 2, rv2); s_rsa[o + 2] = sv2; }
    if (kFirst > 3 && m > 3u) { put_rec(o + 3, rv3); s_rsa[o + 3] = sv3; }
    if (!kF && d.adj_staged)
      for (uint32_t j = 0; j < m && j < (uint32_t)kFirst; ++j) s_radj[o + j] = d.radj[r0 + j * nn];
    for (uint32_t j = kFirst; j < m; ++j) {
      put_rec(o + j, bk.rec[r0 + j * nn]);
      s_rsa[o + j] = bk.sa[r0 + j * nn];
      if (!kF && d.adj_staged) s_radj[o + j] = d.radj[r0 + j * nn];
    }
  };
  if (cl0 < ncs) s_off[cl0] = (uint16_t)off;
  if (kTwo && cl0 + 1 < ncs) s_off[cl0 + 1] = (uint16_t)(off + mine);
  if (tid == 0) s_off[ncs] = (uint16_t)total;
  if (!staged) mine = mine2 = 0;
  rec_load((size_t)gc, mine);
  if (kTwo) {
    rec_put((size_t)gc, off, mine);
    rec_load((size_t)gc2, mine2);
  }
  __syncthreads();
  // the blocks (the last one's far corner is the region's last cell)
#pragma unroll
  for (int h = 0; h < (kTwo ? 2 : 1); ++h)
    if (cl0 + h + ex * ey + ex + 2 <= ncs) s_blk[cl0 + h] = scan_entry(s_off, cl0 + h, ex, ex * ey);
  if (kTwo) rec_put((size_t)gc2, off + mine, mine2);
  else rec_put((size_t)gc, off, mine);
  __syncthreads();
  const bool dead = s_dead != 0;
  // the workgroup-uniform switches of the pass loop, one scalar register
  // whose bits are tested where they are used (kept as separate booleans
  // they would each occupy a 64-bit lane mask)
  constexpr uint32_t kFJit = 1u, kFMove = 2u, kFStaged = 4u;
  const uint32_t flags0 = (uint32_t)__builtin_amdgcn_readfirstlane(
      (jit ? kFJit : 0u) | (d.jitter ? kFMove : 0u) | (staged ? kFStaged : 0u));
  int t_elig = 0, a_elig = 0;  // of the wavefront
  for (int base = s0; base < s1 && !dead; base += kTP) {
    if (base != s0) cur = load_part(a, X, Y, Z, base + tid, s1);
    int id_0 = 0, id_1 = 0, id_2 = 0;  // nearest selection: ids of the thread's particles
    static_assert(kPer == 3, "id_0, id_1, id_2");
#pragma unroll 1
    for (int u = 0; u < kPer; ++u) {
      const Dev& d = fresh(d0);
      const int lt = u * kThreads + tid;
      const int slot = base + lt;
      uint32_t fl = flags0;
      asm volatile("" : "+s"(fl));
      // wave priority by progress: the arbiter otherwise favours the oldest
      // waves, so the workgroups dispatched first race ahead and the last
      // ones end up running nearly alone on their compute units at the end
      if (u == 0) __builtin_amdgcn_s_setprio(3);
      else if (u == 1) __builtin_amdgcn_s_setprio(2);
      else __builtin_amdgcn_s_setprio(1);
      t_elig += (int)__popcll(__ballot(slot < s1 && pol_t<kPol>(cur.role)));
      if (kF)
        a_elig += (int)__popcll(__ballot(slot < s1 && role_is_a((uint32_t)cur.role, kPol == kMulti)));
      // the next particle's loads are in flight while this one is handled
      Part nxt = cur;
      if (u + 1 < kPer) nxt = load_part(a, X, Y, Z, slot + kThreads, s1);
      const uint32_t idj = (uint32_t)cur.id;
      if (kPol == kNearest) {
        id_0 = id_1;
        id_1 = id_2;
        id_2 = cur.id;
      }
      if (slot < s1 && (fl & kFMove)) {  // the re-jitter (stand-in for the MD between steps)
        if (fl & kFJit) rejitter(d, step, idj, cur.x, cur.y, cur.z);
        const uint32_t bo = (uint32_t)slot * 4u;  // 32-bit byte offsets: scalar-base stores
        if (kNt) {
          __builtin_nontemporal_store(cur.x, (float*)((char*)XW + bo));
          __builtin_nontemporal_store(cur.y, (float*)((char*)YW + bo));
          __builtin_nontemporal_store(cur.z, (float*)((char*)ZW + bo));
        } else {
          *(float*)((char*)XW + bo) = cur.x;
          *(float*)((char*)YW + bo) = cur.y;
          *(float*)((char*)ZW + bo) = cur.z;
        }
      }
      if (kPol == kMulti && slot < s1) {  // the flags of the T-side choice
        d.wfa[slot] = 0;
        d.wft[slot] = 0;
      }
      if (kF && slot < s1 && role_is_a((uint32_t)cur.role, kPol == kMulti)) {
        // fused binning: the A's record of the next step, re-jittered once
        // more (its bucket's returning atomic completes behind the rest of
        // the pass)
        float nx = cur.x, ny = cur.y, nz = cur.z;
        if (fl & kFJit) rejitter(d, step + 1u, idj, nx, ny, nz);
        fuse_bin(d, par ^ 1u, step + 1u, slot, idj, nx, ny, nz);
      }
      if (kPol == kNearest)
        near_list(slot < s1 && cur.role == kRoleA, cur.id, slot, (int2*)s_ent, &s_ne);
      // candidates among the staged records (a T with more than four is deferred)
      uint32_t hits = 0, blk = 0;
      bool defer = false;
      if (slot < s1 && pol_t<kPol>(cur.role)) {
        defer = true;
        if (fl & kFStaged) {
          if (kPol != kNearest) s_tid[lt] = (int)idj;
          const float px = cur.x, py = cur.y, pz = cur.z;
          // local coordinates (in the staged region) of the lower corner of
          // the T's 2x2x2 cell block: floor(u - 1/2) - base, taken mod nc
          const int lx0 = local_lo(px, d.inv_w, bx, nc), ly0 = local_lo(py, d.inv_w, by, nc),
                    lz0 = local_lo(pz, d.inv_w, bz, nc);
          if ((uint32_t)lx0 < (uint32_t)(ex - 1) && (uint32_t)ly0 < (uint32_t)(ey - 1) &&
              (uint32_t)lz0 < (uint32_t)(ez - 1)) {
            const int l0 = (int)__umul24(__umul24(lz0, ey) + ly0, ex) + lx0;  // small operands
            const uint2 e = s_blk[l0];
            if (e.x < (0x80u + kScanMax) << 24) {
              hits = scan_block(s_qr, e, quant(d, px, py, pz), d.qthr);
              blk = (uint32_t)l0;
              defer = __popc(hits) > 4;
            }
          }
        }
      }
      const int nh = defer ? 0 : __popc(hits);
      // queue slots for the wavefront's held pairs: lane j's pairs go after
      // those of the lower lanes (counts from four ballots)
      const unsigned long long g1 = __ballot(nh >= 1);
      if (g1) {
        const unsigned long long g2 = __ballot(nh >= 2), g3 = __ballot(nh >= 3),
                                 g4 = __ballot(nh >= 4);
        const uint32_t wtot =
            (uint32_t)(__popcll(g1) + __popcll(g2) + __popcll(g3) + __popcll(g4));
        uint32_t qb = 0;
        if (__lane_id() == 0) qb = (uint32_t)atomicAdd(&s_qn, (int)wtot);
        qb = (uint32_t)__builtin_amdgcn_readlane((int)qb, 0);
        const uint32_t p =
            qb + lanes_below(g1) + lanes_below(g2) + lanes_below(g3) + lanes_below(g4);
        if (nh > 0) {
          if (p + (uint32_t)nh <= (uint32_t)kQueue) {
            for (int j = 0; j < nh; ++j) {
              s_q[p + j] = (uint32_t)lt | (blk << 10) | ((uint32_t)(__ffs((int)hits) - 1) << 20);
              hits &= hits - 1u;
            }
          } else {
            // the pairs do not all fit: the T is deferred and the slots it
            // reserved below kQueue are marked empty
            for (int j = 0; j < nh; ++j)
              if (p + j < (uint32_t)kQueue) s_q[p + j] = kQEmpty;
            defer = true;
          }
        }
      }
      if (defer) s_def[atomicAdd(&s_ndef, 1)] = (uint16_t)lt;
      cur = nxt;
    }
    __syncthreads();
    const Dev& d = fresh(d0);
    // nearest selection, whole bricks: the pairs of a staged A (about five) are
    // merged in LDS before the device-wide minimum, which is served beyond the
    // chiplet's cache and bounds the queue of a full chip (64 steps at
    // 1,048,576 particles with load and read-out 2.57 -> 2.48 ms).  Where bricks
    // are shared among workgroups the chip is not full, and the minimum comes
    // sooner without (137,899 particles, 218 steps: 4.27 ms, merged 4.31).
    const bool merge_a = kPol == kNearest && d.wshift == 0;
    // the pass's queued pairs: draws (or keys) on full wavefronts
    const int qn = min(s_qn, kQueue);
    for (int e = tid; e < qn; e += kThreads) {
      const uint32_t q = s_q[e];
      if (q == kQEmpty) continue;
      const uint32_t lt = q & 1023u, r = scan_record(s_blk[(q >> 10) & 1023u], q >> 20);
      const int sj = base + (int)lt;
      const uint32_t idj = (uint32_t)(kPol == kNearest ? a.id[sj] : s_tid[lt]);
      const int4* arow = d.adj_staged && !kF ? &s_radj[r] : nullptr;
      // the exact test, on the T's position as this workgroup has just written
      // it (the draws meanwhile: few candidates fail it)
      const float4 A = s_rec[r];
      const int ida = __float_as_int(A.w), sa = s_rsa[r];
      const float tx = d.jitter ? XW[sj] : X[sj], ty = d.jitter ? YW[sj] : Y[sj],
                  tz = d.jitter ? ZW[sj] : Z[sj];
      // the nearest selection tests every pair's exclusion, several rules its T's
      // role: what they read is under way with the position
      const bool row_ahead = kPol == kNearest && d.rule.exclude && !arow && d.B <= kAdjStage;
      int4 row = make_int4(-1, -1, -1, -1);
      if (row_ahead) row = row_load(a.adj + (size_t)sa * d.B, d.B);
      const uint32_t rt = kPol == kMulti ? a.role[sj] & kMaskT : 0u;
      W4 w4{0u, 0u, 0u, 0u};
      if (kPol == kRandom) w4 = philox(step, (uint32_t)ida, idj, 0u, d.seed);
      const float r2 = dist2(d, tx, ty, tz, A);
      if (!(r2 < d.rc2)) continue;
      if (kPol != kMulti) count_one(&s_cnt[kOutInRc]);  // several rules: counted per rule
      if (kPol == kRandom)
        retain(d, a, w4, ida, sa, idj, sj, arow, s_cnt, rl);
      else if (kPol == kNearest) {
        const bool excl = row_ahead ? row.x == (int)idj || row.y == (int)idj ||
                                          row.z == (int)idj || row.w == (int)idj
                                    : d.rule.exclude && pair_bonded(d, a, sa, idj, arow);
        if (merge_a) near_pair(ida, idj, r2, excl, s_cnt, &s_best_a[r], &s_best[lt]);
        else near_pair(ida, idj, r2, excl, s_cnt, &d.slotA[ida], &s_best[lt]);
      } else
        multi_pair(d, a, step, rt, ida, sa, idj, sj, r2, arow, s_cnt, rl);
    }
    // the deferred T's, eight lanes each, one cell of the block per lane: from
    // the staged records when the block lies in a staged region, else from the
    // buckets and the overflow list.  They are few, and what bounds them is
    // latency, at the end of the last workgroups with nothing left to hide it:
    // one lane each walked the cells one after another, up to 5 us (1,048,576
    // particles, 256 steps with load and read-out 7.45 ms, this 7.07).  A lane
    // reads its count and first record together; what not every lane needs (a
    // second record, the slots of pairs in range) is read when it does, as each
    // is a request of its own: where nearly every T is deferred (particles that
    // move a cutoff per step, 1,048,576 of them) these requests bound the sweep,
    // 70 us per step, with two records and slots ahead 91, with one lane each
    // and a cell's records in one line 75.  From the last thread down: the first
    // wavefronts have the queue.
    const int ndef = s_ndef;
    for (int e = (kThreads - 1 - tid) >> 3; e < ndef; e += kThreads / 8) {
      const int lt = (int)s_def[e], slot = base + lt, sub = tid & 7;
      const float px = d.jitter ? XW[slot] : X[slot], py = d.jitter ? YW[slot] : Y[slot],
                  pz = d.jitter ? ZW[slot] : Z[slot];
      const uint32_t idj = (uint32_t)a.id[slot];
      const uint32_t rt = kPol == kMulti ? a.role[slot] & kMaskT : 0u;
      int lx0 = 0, ly0 = 0, lz0 = 0;
      bool in = staged;
      if (staged) {
        lx0 = local_lo(px, d.inv_w, bx, nc);
        ly0 = local_lo(py, d.inv_w, by, nc);
        lz0 = local_lo(pz, d.inv_w, bz, nc);
        in = (uint32_t)lx0 < (uint32_t)(ex - 1) && (uint32_t)ly0 < (uint32_t)(ey - 1) &&
             (uint32_t)lz0 < (uint32_t)(ez - 1);
      }
      // a pair within the cutoff
      auto take = [&](const float4& A, int sa, float r2, const int4* arow)
                      __attribute__((always_inline)) {
        const int ida = __float_as_int(A.w);
        if (kPol != kMulti) count_one(&s_cnt[kOutInRc]);
        if (kPol == kRandom)
          retain(d, a, philox(step, (uint32_t)ida, idj, 0u, d.seed), ida, sa, idj, slot, arow,
                 s_cnt, rl);
        else if (kPol == kNearest)
          near_pair(ida, idj, r2, d.rule.exclude && pair_bonded(d, a, sa, idj, arow), s_cnt,
                    &d.slotA[ida], &s_best[lt]);
        else
          multi_pair(d, a, step, rt, ida, sa, idj, slot, r2, arow, s_cnt, rl);
      };
      int q = 0;  // the lane's cell: its first staged record, or the cell
      uint32_t nr = 0;
      float4 A0 = make_float4(0.f, 0.f, 0.f, 0.f);
      const size_t nn = (size_t)d.ncell;
      if (in) {
        const int lr = ((lz0 + (sub >> 2)) * ey + ly0 + ((sub >> 1) & 1)) * ex + lx0 + (sub & 1);
        q = (int)s_off[lr];
        nr = (uint32_t)s_off[lr + 1] - (uint32_t)q;
      } else {
        int cx0, cx1, cy0, cy1, cz0, cz1;
        lo_hi(px, d.inv_w, nc, cx0, cx1);
        lo_hi(py, d.inv_w, nc, cy0, cy1);
        lo_hi(pz, d.inv_w, nc, cz0, cz1);
        q = (((sub & 4) ? cz1 : cz0) * nc + ((sub & 2) ? cy1 : cy0)) * nc + ((sub & 1) ? cx1 : cx0);
        nr = bk.cnt[q];
        A0 = bk.rec[q];
        nr = nr < (uint32_t)kCellCap ? nr : (uint32_t)kCellCap;
        if (nc == 1 && sub) nr = 0;  // one cell, not eight
      }
      for (uint32_t r = 0; r < nr; ++r) {
        float4 A = A0;
        if (in) A = s_rec[q + r];
        else if (r > 0u) A = bk.rec[q + r * nn];
        const float r2 = dist2(d, px, py, pz, A);
        if (!(r2 < d.rc2)) continue;
        int32_t sa;
        if (in) sa = s_rsa[q + r];
        else sa = bk.sa[q + r * nn];
        take(A, sa, r2, in && d.adj_staged && !kF ? &s_radj[q + r] : nullptr);
      }
      // the overflow list (no brick is staged then), kOvfAhead records of the
      // lane's eighth in flight: the long lists of crowded steps are walked at
      // the latency of their reads (262,144 particles, half of them A's: 410 us
      // per step, with one record and its slot at a time 560; one million, 15-20%
      // A's, no list and no brick staged: within 4% of one lane per T)
      constexpr uint32_t kOvfAhead = 4;
      for (uint32_t r0 = (uint32_t)sub; r0 < bk.novf; r0 += 8u * kOvfAhead) {
        float4 V[kOvfAhead];
#pragma unroll
        for (uint32_t u = 0; u < kOvfAhead; ++u) V[u] = bk.ovf[min(r0 + 8u * u, bk.novf - 1u)];
        uint32_t hit = 0;
#pragma unroll
        for (uint32_t u = 0; u < kOvfAhead; ++u)
          hit |= r0 + 8u * u < bk.novf && dist2(d, px, py, pz, V[u]) < d.rc2 ? 1u << u : 0u;
        while (hit) {
          const uint32_t r = r0 + 8u * (uint32_t)(__ffs((int)hit) - 1);
          hit &= hit - 1u;
          const float4 A = bk.ovf[r];
          take(A, bk.osa[r], dist2(d, px, py, pz, A), nullptr);
        }
      }
    }
    __syncthreads();
    if (kPol == kNearest) {
      // the staged A's with a candidate: one global minimum each
      for (int q = tid; merge_a && q < kStageRecs; q += kThreads) {
        const unsigned long long b = s_best_a[q];
        if (b == kEmpty) continue;
        atomicMin(&d.slotA[__float_as_int(s_rec[q].w)], b);
        s_best_a[q] = kEmpty;
      }
      // every T of the pass with a candidate: its closest A, its slot
      unsigned long long b[kPer];
      const int t[kPer] = {id_0, id_1, id_2};
#pragma unroll
      for (int u = 0; u < kPer; ++u) b[u] = s_best[u * kThreads + tid];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        if (b[u] == kEmpty) continue;
        d.tnear[t[u]] = make_int2((int)(uint32_t)b[u], base + u * kThreads + tid);
        s_best[u * kThreads + tid] = kEmpty;
      }
    }
    if (tid == 0) {
      s_qn = 0;
      s_ndef = 0;
    }
    __syncthreads();
  }
  if (kF && !dead) {
    // fused binning: the counts two steps ahead (last read in the previous
    // step) are cleared for the next step's sweep
    for (int q = w * kThreads + tid; q < d.ncell; q += nwg * kThreads) d.fcnt[mod3(step + 2u)][q] = 0u;
    if (w == 0 && tid == 0) d.ctl->fovf_n[mod3(step + 2u)] = 0u;
  }
  // clear the bucket counts of the next step's parity (no workgroup of this
  // step reads them; with fused binning too, so that they are clear whenever
  // a step with the binning kernel follows)
  for (int q = w * kThreads + tid; q < d.ncell; q += nwg * kThreads)
    pick(d.cnt, par ^ 1u)[q] = 0u;
  if (__lane_id() == 0) {
    atomicAdd(&s_cnt[kOutTElig], t_elig);
    if (kF) atomicAdd(&s_cnt[4], a_elig);
  }
  __syncthreads();
  const int ne = s_ne;
  const int nk = kPol == kNearest ? ne : (ne < kRetCap ? ne : kRetCap);
  if (tid < min(nk, kRetCap)) {
    pick(d.wge, par)[w * kRetCap + tid] = s_ent[tid];
    if (kPol != kNearest) pick(d.wgk, par)[w * kRetCap + tid] = s_ew2[tid];
    if (kPol == kMulti) d.wgk1[w * kRetCap + tid] = s_ew1[tid];
  }
  int32_t* out = pick(d.wgo, par) + w * kWgOut;
  if (tid < 4) out[tid] = s_cnt[tid];
  if (tid == 0) {
    out[kOutRet] = nk;
    if (kF) out[kOutAElig] = s_cnt[4];
    if (kPol != kNearest && ne > kRetCap) set_flag(&d.ctl->ret_ovf[par]);
  }
}

// ---------------------------------------------------------------------------
// The sweep on unsorted storage, any selection (the single step on the
// caller's arrays, and resident systems that never sort): workgroup w takes
// slots w * kThreads .. + kThreads - 1, one per thread.  The particles are in
// any order, so a T's eight cells and their records are reads of lines no
// neighbouring lane shares: their latency and the caches' request rate bound
// the kernel.  A T issues its eight counts together, keeps them as nibbles of
// one word (a bucket holds at most eight records) and then takes its records
// four at a time, with four loads in flight; in-range pairs go to an LDS queue
// so that the draws run on full wavefronts.  1,000,003 particles in random
// order, 5% A's: walking the cells one after another with the draw in the
// loop 74 us, this 47 us; 4,000 particles 16.3 and 10.1 us.
// ---------------------------------------------------------------------------
template <int kPol>
__device__ __forceinline__ void dense_sweep_body(const Dev& d, int k, int w, int nwg) {
  constexpr int kDenseQ = 512;
  static_assert(kCellCap <= 8, "a cell's record count fits a nibble");
  __shared__ uint2 s_q[kDenseQ];  // cell (or overflow index), local T | record << 8 | overflow << 31
  __shared__ int32_t s_tid[kThreads];
  __shared__ float s_pos[kPol == kRandom ? 1 : 3][kPol == kRandom ? 1 : kThreads];
  __shared__ unsigned long long s_best[kPol == kNearest ? kThreads : 1];
  __shared__ int4 s_ent[kRetCap];
  __shared__ uint32_t s_ew1[kPol == kMulti ? kRetCap : 1], s_ew2[kRetCap];
  __shared__ int s_cnt[4], s_qn, s_ne;
  const int tid = threadIdx.x;
  if (tid < 4) s_cnt[tid] = 0;
  if (tid == 0) {
    s_qn = 0;
    s_ne = 0;
  }
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = si.par, step = si.step;
  const Arr a = pick_set(d, c->set & 1u);
  const bool dead = read_err(c) != 0;
  const Buckets bk = step_buckets<false>(d, par, step);
  const RetList rl{&s_ne, s_ent, s_ew1, s_ew2};
  const int slot = w * kThreads + tid;
  float x = 0.0f, y = 0.0f, z = 0.0f;
  uint32_t id = (uint32_t)slot;
  bool is_target = false;
  if (kPol == kNearest) s_best[tid] = kEmpty;
  if (slot < d.n && !dead) {
    x = pick(a.x, par)[slot];
    y = pick(a.y, par)[slot];
    z = pick(a.z, par)[slot];
    if (a.id) id = (uint32_t)a.id[slot];
    is_target = pol_t<kPol>(a.role[slot]);
    if (d.jitter) {
      if (d.jit_c != 0.0f) rejitter(d, step, id, x, y, z);
      pick(a.x, par ^ 1u)[slot] = x;
      pick(a.y, par ^ 1u)[slot] = y;
      pick(a.z, par ^ 1u)[slot] = z;
    }
  }
  if (kPol == kMulti && slot < d.n && !dead) {  // the flags of the T-side choice
    d.wfa[slot] = 0;
    d.wft[slot] = 0;
  }
  __syncthreads();
  if (kPol == kNearest)
    near_list(slot < d.n && !dead && a.role[slot] == kRoleA, (int)id, slot, (int2*)s_ent, &s_ne);
  // an in-range pair: draw or keys; lt: the T's thread, whose position is in
  // LDS when the distance is needed again
  auto pair = [&](int lt, uint32_t idj, const float4& A, int sa) __attribute__((always_inline)) {
    const int sj = w * kThreads + lt;
    if (kPol == kRandom) {
      retain(d, a, philox(step, (uint32_t)__float_as_int(A.w), idj, 0u, d.seed),
             __float_as_int(A.w), sa, idj, sj, nullptr, s_cnt, rl);
      return;
    }
    const float r2 = dist2(d, s_pos[0][lt], s_pos[1][lt], s_pos[2][lt], A);
    if (kPol == kNearest)
      near_pair(__float_as_int(A.w), idj, r2,
                d.rule.exclude && pair_bonded(d, a, sa, idj, nullptr), s_cnt,
                &d.slotA[__float_as_int(A.w)], &s_best[lt]);
    else
      multi_pair(d, a, step, a.role[sj] & kMaskT, __float_as_int(A.w), sa, idj, sj, r2, nullptr, s_cnt,
                 rl);
  };
  if (is_target) {
    count_one(&s_cnt[kOutTElig]);
    s_tid[tid] = (int32_t)id;
    if (kPol != kRandom) {
      s_pos[0][tid] = x;
      s_pos[1][tid] = y;
      s_pos[2][tid] = z;
    }
    const int nc = d.nc;
    int cx0, cx1, cy0, cy1, cz0, cz1;
    lo_hi(x, d.inv_w, nc, cx0, cx1);
    lo_hi(y, d.inv_w, nc, cy0, cy1);
    lo_hi(z, d.inv_w, nc, cz0, cz1);
    // rows (y, z) of the block; one cell per side: the block is that cell
    const int r00 = (cz0 * nc + cy0) * nc, r01 = (cz0 * nc + cy1) * nc,
              r10 = (cz1 * nc + cy0) * nc, r11 = (cz1 * nc + cy1) * nc;
    uint32_t cnt[8];
    cnt[0] = bk.cnt[r00 + cx0];
    cnt[1] = bk.cnt[r00 + cx1];
    cnt[2] = bk.cnt[r01 + cx0];
    cnt[3] = bk.cnt[r01 + cx1];
    cnt[4] = bk.cnt[r10 + cx0];
    cnt[5] = bk.cnt[r10 + cx1];
    cnt[6] = bk.cnt[r11 + cx0];
    cnt[7] = bk.cnt[r11 + cx1];
    uint32_t left = 0;  // records not taken yet, a nibble per cell
#pragma unroll
    for (int q = 0; q < 8; ++q)
      left |= (cnt[q] < (uint32_t)kCellCap ? cnt[q] : (uint32_t)kCellCap) << (4 * q);
    if (nc == 1) left &= 15u;
    auto hit = [&](const float4& A, uint32_t cell, uint32_t what) {
      if (!(dist2(d, x, y, z, A) < d.rc2)) return;
      if (kPol != kMulti) count_one(&s_cnt[kOutInRc]);
      const int p = atomicAdd(&s_qn, 1);
      if (p < kDenseQ) {
        s_q[p] = make_uint2(cell, (uint32_t)tid | what);
      } else {  // the queue is full: drawn at once
        const bool o = what >> 31;
        const size_t r = o ? (size_t)cell : rec_at(d, (int)cell, what >> 8);
        pair(tid, id, A, (o ? bk.osa : bk.sa)[r]);
      }
    };
    while (left) {
      float4 A[4];
      uint32_t cell[4], rec[4];
      bool have[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        have[u] = left != 0u;
        const int sh = have[u] ? __builtin_ctz(left) & 28 : 0;
        const int row = sh & 16 ? (sh & 8 ? r11 : r10) : (sh & 8 ? r01 : r00);
        cell[u] = (uint32_t)(row + (sh & 4 ? cx1 : cx0));
        rec[u] = ((left >> sh) & 15u) - 1u;
        if (have[u]) {
          left -= 1u << sh;
          A[u] = bk.rec[rec_at(d, (int)cell[u], rec[u])];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (have[u]) hit(A[u], cell[u], rec[u] << 8);
    }
    for (uint32_t r = 0; r < bk.novf; ++r) hit(bk.ovf[r], r, 1u << 31);
  }
  __syncthreads();
  const int qn = min(s_qn, kDenseQ);
  for (int e = tid; e < qn; e += kThreads) {
    const uint2 q = s_q[e];
    const int lt = (int)(q.y & 0xFFu);
    const bool o = q.y >> 31;
    const size_t r = o ? (size_t)q.x : rec_at(d, (int)q.x, q.y >> 8);
    pair(lt, (uint32_t)s_tid[lt], (o ? bk.ovf : bk.rec)[r], (o ? bk.osa : bk.sa)[r]);
  }
  if (kPol == kNearest) {  // a T with a candidate: its closest A, its slot
    __syncthreads();
    if (s_best[tid] != kEmpty) d.tnear[id] = make_int2((int)(uint32_t)s_best[tid], slot);
  }
  // clear the bucket counts of the next step's parity (as the other sweep)
  for (int q = w * kThreads + tid; q < d.ncell_clear; q += nwg * kThreads)
    pick(d.cnt, par ^ 1u)[q] = 0u;
  __syncthreads();
  const int ne = s_ne;
  const int nk = kPol == kNearest ? ne : (ne < kRetCap ? ne : kRetCap);
  if (tid < min(nk, kRetCap)) {
    pick(d.wge, par)[w * kRetCap + tid] = s_ent[tid];
    if (kPol != kNearest) pick(d.wgk, par)[w * kRetCap + tid] = s_ew2[tid];
    if (kPol == kMulti) d.wgk1[w * kRetCap + tid] = s_ew1[tid];
  }
  int32_t* out = pick(d.wgo, par) + w * kWgOut;
  if (tid < 4) out[tid] = s_cnt[tid];
  if (tid == 0) {
    out[kOutRet] = nk;
    if (kPol != kNearest && ne > kRetCap) set_flag(&d.ctl->ret_ovf[par]);
  }
}

// ---------------------------------------------------------------------------
// k_resolve: the T side (steps 6-7) and the bonds (step 9).  Every retained
// pair belongs to the workgroup that owns its T's slot.  Normally the pairs
// come from the sweep workgroup's list: a pair whose A's final key names its
// T is a proposal (the A's key is emptied for the next step), and of the
// proposals to one T the smallest (w2, id_A) is bonded.  If any list
// overflowed in this step, every flagged T enumerates its pairs again (same
// cells, same draws) instead.  An A chose exactly one T and a T bonds at most
// one A, so every state and adjacency row has one writer.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool adj_append(int32_t* row, int B, int32_t v) {
  for (int b = 0; b < B; ++b)
    if (row[b] < 0) {
      row[b] = v;
      return true;
    }
  return false;
}

struct BondCtx {
  int* nw;
  int* lost;
  uint32_t step;
};

// Fused binning after a bond of step `step`: the A's record of the next step
// is dropped when the bond ends its A role, and a T that takes the A role
// (chain growth) is binned for the next step at its re-jittered position.
__device__ void fuse_after_bond(const Dev& d, const Arr& a, uint32_t par, uint32_t step, int sa,
                                int sj, uint32_t idj, uint8_t ra, uint8_t rt) {
  if (ra != kRoleA) fuse_drop(d, par ^ 1u, sa);
  if (rt != kRoleA) return;
  float x = pick(a.x, par ^ 1u)[sj], y = pick(a.y, par ^ 1u)[sj], z = pick(a.z, par ^ 1u)[sj];
  if (d.jitter && d.jit_c != 0.0f) rejitter(d, step + 1u, idj, x, y, z);
  fuse_bin(d, par ^ 1u, step + 1u, sj, idj, x, y, z);
}

// The same for one particle of a bond of several rules, whose role mask went
// from `was` to `now`.
__device__ void fuse_role_change(const Dev& d, const Arr& a, uint32_t par, uint32_t step, int slot,
                                 uint32_t id, uint8_t was, uint8_t now) {
  const bool had = role_is_a(was, true), has = role_is_a(now, true);
  if (had && !has) fuse_drop(d, par ^ 1u, slot);
  if (had || !has) return;
  float x = pick(a.x, par ^ 1u)[slot], y = pick(a.y, par ^ 1u)[slot], z = pick(a.z, par ^ 1u)[slot];
  if (d.jitter && d.jit_c != 0.0f) rejitter(d, step + 1u, id, x, y, z);
  fuse_bin(d, par ^ 1u, step + 1u, slot, id, x, y, z);
}

__device__ __forceinline__ void make_bond(const Dev& d, const Arr& a, uint32_t par, int w,
                                          int ida, int sa, int sj, int idj, const BondCtx& b) {
  const int32_t na = a.st[sa] + d.rule.d_a, nt = a.st[sj] + d.rule.d_t;
  a.st[sa] = na;
  a.st[sj] = nt;
  const uint8_t ra = role_of(d, a.typ[sa], na), rt = role_of(d, a.typ[sj], nt);
  a.role[sa] = ra;
  a.role[sj] = rt;
  if (d.fuse) fuse_after_bond(d, a, par, b.step, sa, sj, (uint32_t)idj, ra, rt);
  int lost = 0;
  if (!adj_append(a.adj + (size_t)sa * d.B, d.B, (int32_t)idj)) lost++;
  if (!adj_append(a.adj + (size_t)sj * d.B, d.B, (int32_t)ida)) lost++;
  if (lost) atomicAdd(b.lost, lost);
  const int p = atomicAdd(b.nw, 1);
  if (p < kWinCap) {
    pick(d.wgw, par)[w * kWinCap + p] = make_int2(ida, idj);
  } else {
    const uint32_t o = atomicAdd(&d.ctl->nwin_ovf[par], 1u);
    pick(d.wov, par)[o] = make_int2(ida, idj);
  }
}

// The operands of a bond read ahead of the decision, together with the A's
// key: both states and types and (rows of width B <= kAdjStage) both
// adjacency rows.  Every particle takes at most one bond per step, and only
// that bond writes its state and row (and, with fused binning, the bucket
// position of an A's record or a T's binned record; positions are final after
// the sweep), so values read ahead are the ones a bond made after the
// decision would read.
struct BondOps {
  int32_t sta, stt, tya, tyt;
  int4 rowa, rowt;
  // fused binning: where the A's next-step record is, and the T's position
  // of this step (binned if the bond gives the T the A role)
  int32_t apa;
  float tx, ty, tz;
};

// The slot adj_append would fill in a row read ahead (B when it is full).
__device__ __forceinline__ int first_empty(int4 r, int B) {
  if (r.x < 0) return 0;
  if (B > 1 && r.y < 0) return 1;
  if (B > 2 && r.z < 0) return 2;
  if (B > 3 && r.w < 0) return 3;
  return B;
}

// make_bond with its operands read ahead (rows of width B <= kAdjStage).
__device__ __forceinline__ void make_bond_ahead(const Dev& d, const Arr& a, uint32_t par, int w,
                                                int ida, int sa, int sj, int idj,
                                                const BondOps& o, const BondCtx& b) {
  const int32_t na = o.sta + d.rule.d_a, nt = o.stt + d.rule.d_t;
  a.st[sa] = na;
  a.st[sj] = nt;
  const uint8_t ra = role_of(d, o.tya, na), rt = role_of(d, o.tyt, nt);
  a.role[sa] = ra;
  a.role[sj] = rt;
  if (d.fuse) {  // fuse_after_bond with the operands read ahead
    if (ra != kRoleA) fuse_drop_at(d, par ^ 1u, o.apa);
    if (rt == kRoleA) {
      float x = o.tx, y = o.ty, z = o.tz;
      if (d.jitter && d.jit_c != 0.0f) rejitter(d, b.step + 1u, (uint32_t)idj, x, y, z);
      fuse_bin(d, par ^ 1u, b.step + 1u, sj, (uint32_t)idj, x, y, z);
    }
  }
  int lost = 0;
  const int fa = first_empty(o.rowa, d.B), ft = first_empty(o.rowt, d.B);
  if (fa < d.B) a.adj[(size_t)sa * d.B + fa] = (int32_t)idj;
  else lost++;
  if (ft < d.B) a.adj[(size_t)sj * d.B + ft] = (int32_t)ida;
  else lost++;
  if (lost) atomicAdd(b.lost, lost);
  const int p = atomicAdd(b.nw, 1);
  if (p < kWinCap) {
    pick(d.wgw, par)[w * kWinCap + p] = make_int2(ida, idj);
  } else {
    const uint32_t q = atomicAdd(&d.ctl->nwin_ovf[par], 1u);
    pick(d.wov, par)[q] = make_int2(ida, idj);
  }
}

// One wavefront per unit (four units per workgroup).  Every barrier is taken by
// the whole workgroup (mode is the same for all its units).
// kHostPar: the step's parity from Dev::kpar0 (resident systems), else from
// the control block.
template <bool kBrick, bool kHostPar = false>
__device__ __forceinline__ void resolve_body(const Dev& d, int k, int wg, int nunits) {
  constexpr int kG = kThreads / 64;  // units per workgroup
  __shared__ int s_nw[kG], s_lost[kG], s_prop[kG];
  __shared__ int s_mode;
  __shared__ unsigned long long s_key[kG][kRetCap];
  __shared__ int32_t s_sj[kG][kRetCap];
  const int g = (int)(threadIdx.x >> 6), tid = (int)__lane_id();
  const int w = wg * kG + g;
  const bool live = w < nunits;  // the last workgroup's spare wavefronts
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = kHostPar ? (d.kpar0 + (uint32_t)k) & 1u : si.par, step = si.step;
  if (tid == 0) {
    s_nw[g] = 0;
    s_lost[g] = 0;
    s_prop[g] = 0;
  }
  if (threadIdx.x == 0) s_mode = read_err(c) ? 0 : (c->ret_ovf[par] ? 2 : 1);
  // the list's length and its entries in one round trip, issued before the
  // mode is known (read but not used in the other modes, as are entries past
  // the length), then the A keys with the bonds' operands in a second one
  int ne = 0;
  int4 e = make_int4(0, 0, 0, 0);
  uint32_t w2 = 0;
  if (live) {
    ne = pick(d.wgo, par)[w * kWgOut + kOutRet];
    if (tid < kRetCap) {
      e = pick(d.wge, par)[w * kRetCap + tid];
      w2 = pick(d.wgk, par)[w * kRetCap + tid];
    }
  }
  __syncthreads();
  const int mode = s_mode;
  const Arr a = pick_set(d, c->set & 1u);
  const BondCtx bc{&s_nw[g], &s_lost[g], step};
  if (mode == 1) {
    const bool ahead = d.adj_staged != 0;
    bool chosen = false;
    unsigned long long key = kEmpty;
    BondOps ops{0, 0, 0, 0, make_int4(0, 0, 0, 0), make_int4(0, 0, 0, 0), 0, 0.0f, 0.0f, 0.0f};
    if (tid < ne) {
      const unsigned long long ka = d.slotA[e.x];
      if (ahead) {
        ops.sta = a.st[e.y];
        ops.stt = a.st[e.z];
        ops.tya = a.typ[e.y];
        ops.tyt = a.typ[e.z];
        ops.rowa = row_load(a.adj + (size_t)e.y * d.B, d.B);
        ops.rowt = row_load(a.adj + (size_t)e.z * d.B, d.B);
        if (d.fuse) {
          ops.apa = d.apos[e.y];
          ops.tx = pick(a.x, par ^ 1u)[e.z];
          ops.ty = pick(a.y, par ^ 1u)[e.z];
          ops.tz = pick(a.z, par ^ 1u)[e.z];
        }
      }
      d.tflag[e.z] = 0;
      chosen = (uint32_t)ka == (uint32_t)e.w;
      if (chosen) {
        d.slotA[e.x] = kEmpty;
        key = ((unsigned long long)w2 << 32) | (uint32_t)e.x;
        atomicAdd(&s_prop[g], 1);
      }
      s_key[g][tid] = key;
      s_sj[g][tid] = e.z;
    }
    __syncthreads();
    if (chosen) {
      bool win = true;
      for (int f = 0; f < ne; ++f)
        if (s_sj[g][f] == e.z && s_key[g][f] < key) win = false;
      if (win) {
        if (ahead) make_bond_ahead(d, a, par, w, e.x, e.y, e.z, e.w, ops, bc);
        else make_bond(d, a, par, w, e.x, e.y, e.z, e.w, bc);
      }
    }
  } else if (mode == 2 && live) {
    const float *X = pick(a.x, par ^ 1u), *Y = pick(a.y, par ^ 1u), *Z = pick(a.z, par ^ 1u);
    const Buckets bk = d.fuse ? step_buckets<true>(d, par, step) : step_buckets<false>(d, par, step);
    int s0, s1;
    range_of<kBrick>(d, w, s0, s1);
    for (int base = s0; base < s1; base += 64) {
      const int slot = base + tid;
      if (slot < s1 && d.tflag[slot]) {
        d.tflag[slot] = 0;
        const float xj = X[slot], yj = Y[slot], zj = Z[slot];
        const uint32_t idj = a.id ? (uint32_t)a.id[slot] : (uint32_t)slot;
        unsigned long long best = kEmpty;
        int best_sa = 0, np = 0;
        for_global_records(d, bk, xj, yj, zj, [&](float4 A, int sa) {
          if (!(dist2(d, xj, yj, zj, A) < d.rc2)) return;
          const int ida = __float_as_int(A.w);
          if ((uint32_t)d.slotA[ida] != idj) return;  // not retained, or the A chose another T
          const W4 r = philox(step, (uint32_t)ida, idj, 0u, d.seed);
          d.slotA[ida] = kEmpty;
          np++;
          const unsigned long long bid = ((unsigned long long)r.w2 << 32) | (uint32_t)ida;
          if (bid < best) {
            best = bid;
            best_sa = sa;
          }
        });
        if (np) atomicAdd(&s_prop[g], np);
        if (best != kEmpty) make_bond(d, a, par, w, (int)(uint32_t)best, best_sa, slot, (int)idj, bc);
      }
    }
  }
  __syncthreads();
  if (tid == 0 && live) {
    int32_t* out = pick(d.wgo, par) + w * kWgOut;
    out[kOutProp] = s_prop[g];
    out[kOutBonds] = s_nw[g];
    out[kOutLost] = s_lost[g];
  }
}

// The brick of sweep workgroup g.  Workgroups are dispatched to the eight
// XCDs in turn (g mod 8), each XCD with an L2 of its own; XCD x takes the
// contiguous run of bricks x * q + min(x, r) .. (q or q + 1 of them, q =
// nbricks / 8, r = nbricks mod 8), a slab of neighbouring bricks, so that
// the A records a brick's neighbours stage again are in the same L2.
__device__ __forceinline__ int xcd_brick(int g, int nbricks) {
  constexpr int kXcd = 8;
  const int q = nbricks / kXcd, r = nbricks - q * kXcd;
  const int x = g % kXcd, i = g / kXcd;
  return x * q + min(x, r) + i;
}

// The A records of a brick's region staged in LDS (sorted storage, brick
// edges up to kOneCellBrick: one region cell per thread), as the random
// selection's sweep stages them, for the kinetics counters.  A T whose 2x2x2
// block leaves the staged region, and every T of a brick whose region holds
// more than kStageRecs records or of a step with bucket overflow, scans the
// global buckets instead; either way a T visits the same pairs.
struct StagedRegion {
  float4* rec;    // records (x, y, z, id_A)
  int4* radj;     // the A's adjacency rows (rows of width <= kAdjStage)
  int32_t* rsa;   // the A's slots
  uint16_t* off;  // first record of each region cell (one more entry: the total)
  int bx, ex, by, ey, bz, ez;
  bool staged, nowrap;
};

__device__ __forceinline__ void stage_region(const Dev& d, const Buckets& bk, int w,
                                             StagedRegion& g, uint32_t* s_wave) {
  const int tid = threadIdx.x, nc = d.nc;
  int bxc, byc;
  const int bzc = div_nb(d, div_nb(d, w, bxc), byc);
  region_dim(d, bxc, g.bx, g.ex);
  region_dim(d, byc, g.by, g.ey);
  region_dim(d, bzc, g.bz, g.ez);
  const int ex = g.ex, ey = g.ey, ncs = ex * ey * g.ez;
  // a region that does not wrap around the box and spans less than half of
  // it: the minimum image leaves every difference in it unchanged
  g.nowrap = d.nbricks > 1 && g.bx + ex <= nc && 2 * ex + 1 <= nc && g.by + ey <= nc &&
             2 * ey + 1 <= nc && g.bz + g.ez <= nc && 2 * g.ez + 1 <= nc;
  uint32_t mine = 0;
  int gc = 0;
  if (tid < ncs) {
    const int lz = div_small(tid, recip16((uint32_t)(ex * ey))), rem = tid - lz * ex * ey;
    const int ly = div_small(rem, recip16((uint32_t)ex)), lx = rem - ly * ex;
    int cx = g.bx + lx, cy = g.by + ly, cz = g.bz + lz;
    cx -= cx >= nc ? nc : 0;
    cy -= cy >= nc ? nc : 0;
    cz -= cz >= nc ? nc : 0;
    gc = (cz * nc + cy) * nc + cx;
    mine = bk.cnt[gc];
    mine = mine < (uint32_t)kCellCap ? mine : (uint32_t)kCellCap;
  }
  uint32_t total = 0;
  const uint32_t off = block_scan_excl(mine, s_wave, total);
  g.staged = total <= (uint32_t)kStageRecs && bk.novf == 0;
  if (tid < ncs) {
    g.off[tid] = (uint16_t)off;
    if (g.staged) {
      const size_t r0 = (size_t)gc, nn = (size_t)d.ncell;
      // the first two records loaded together, the rare rest one by one
      float4 rv0 = make_float4(0.f, 0.f, 0.f, 0.f), rv1 = rv0;
      int32_t sv0 = 0, sv1 = 0;
      int4 av0 = make_int4(-1, -1, -1, -1), av1 = av0;
      if (mine > 0u) {
        rv0 = bk.rec[r0];
        sv0 = bk.sa[r0];
        if (d.adj_staged) av0 = d.radj[r0];
      }
      if (mine > 1u) {
        rv1 = bk.rec[r0 + nn];
        sv1 = bk.sa[r0 + nn];
        if (d.adj_staged) av1 = d.radj[r0 + nn];
      }
      if (mine > 0u) {
        g.rec[off] = rv0;
        g.rsa[off] = sv0;
        g.radj[off] = av0;
      }
      if (mine > 1u) {
        g.rec[off + 1] = rv1;
        g.rsa[off + 1] = sv1;
        g.radj[off + 1] = av1;
      }
      for (uint32_t j = 2; j < mine; ++j) {
        g.rec[off + j] = bk.rec[r0 + j * nn];
        g.rsa[off + j] = bk.sa[r0 + j * nn];
        if (d.adj_staged) g.radj[off + j] = d.radj[r0 + j * nn];
      }
    }
  }
  if (tid == 0) g.off[ncs] = (uint16_t)total;
  __syncthreads();
}

// The A side of the nearest selection and the bonds.  A T with a candidate
// left (its closest A, its slot) in tnear[id_T]; each A whose closest T keeps
// it in return is tested once, with the pair's draw (word 0 of the counter
// (step, id_A, id_T, 0)), and bonds when it passes.  One wavefront per sweep
// workgroup (four per workgroup) takes the A's of its list, or, when it has
// more than kNearList, finds them by the role bytes of its slots.  Every A is
// read, and its key emptied, by one thread; a T that takes the A role here has
// no key.  Bound by latency (the list with its length, key, tnear).  1,048,576
// particles, 5% A's: by the cells' buckets 14.0 us, by the role bytes 11.0, by
// the list 8.3 us.
template <bool kBrick>
__device__ __forceinline__ void near_resolve_body(const Dev& d, int k, int wg, int nunits) {
  constexpr int kG = kThreads / 64;
  __shared__ int s_nw[kG], s_lost[kG];
  const int g = (int)(threadIdx.x >> 6), lane = (int)__lane_id();
  const int w = wg * kG + g;
  if (lane == 0) {
    s_nw[g] = 0;
    s_lost[g] = 0;
  }
  wave_sync();
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = si.par, step = si.step;
  const Arr a = pick_set(d, c->set & 1u);
  const BondCtx bc{&s_nw[g], &s_lost[g], step};
  int prop = 0, mutual = 0;
  auto visit = [&](int ida, int sa) __attribute__((always_inline)) {
    const unsigned long long key = d.slotA[ida];
    if (key == kEmpty) return;
    d.slotA[ida] = kEmpty;
    prop++;
    const uint32_t idj = (uint32_t)key;
    const int2 t = d.tnear[idj];
    if (t.x != ida) return;  // the T's closest A is another one
    mutual++;
    const W4 r = philox(step, (uint32_t)ida, idj, 0u, d.seed);
    if ((unsigned long long)r.w0 < d.thresh) make_bond(d, a, par, w, ida, sa, t.y, (int)idj, bc);
  };
  const bool live = w < nunits && read_err(c) == 0;
  int na = 0;
  int2 e = make_int2(0, 0);
  if (live) {
    na = pick(d.wgo, par)[w * kWgOut + kOutRet];
    e = ((const int2*)(pick(d.wge, par) + (size_t)w * kRetCap))[lane];
  }
  // one pass over the list, or over the slots (uniform over the wavefront)
  int s0 = 0, s1 = na <= kNearList ? 64 : 0;
  if (na > kNearList) range_of<kBrick>(d, w, s0, s1);
  for (int i = s0 + lane; i < s1 && live; i += 64) {
    int sa = e.y, ida = e.x;
    bool is_src = lane < na;
    if (na > kNearList) {
      is_src = a.role[i] == kRoleA;
      sa = i;
      ida = is_src && a.id ? a.id[i] : i;
    }
    if (is_src) visit(ida, sa);
  }
  const int np = (int)wave_scan_incl((uint32_t)prop), nm = (int)wave_scan_incl((uint32_t)mutual);
  wave_sync();
  if (lane == 63 && w < nunits) {
    int32_t* out = pick(d.wgo, par) + w * kWgOut;
    out[kOutDrawn] = nm;
    out[kOutProp] = np;
    out[kOutBonds] = s_nw[g];
    out[kOutLost] = s_lost[g];
  }
}

// The winning pair of a T, recorded at both slots for the final choice (one
// writer each: the A picked one T).
__device__ __forceinline__ void multi_win(const Dev& d, int ida, int sa, uint32_t idj, int sj,
                                          int rule) {
  d.wint[sj] = make_int4(ida, sa, rule, 0);
  d.wina[sa] = make_int4((int)idj, sj, rule, 0);
  d.wft[sj] = 1;
  d.wfa[sa] = 1;
}

// The T side of several rules, one wavefront per sweep workgroup (four per
// workgroup).  Normally from the sweep's lists: a listed pair whose A's final
// key is its (w1, id_T) is a proposal -- the lower rule when two rules of one
// pair share the key -- and the smallest (w2, id_A) of a T's proposals wins;
// the winners' entries are marked (bit 31 of id_A) for the final choice.  When
// a list overflowed in this step, every T with an accepted candidate
// enumerates its pairs again (same cells, same draws).  Bound by latency.
// 1,048,576 particles, two rules: enumerating 15.2 us, this 4.9 us.
template <bool kBrick>
__device__ __forceinline__ void multi_resolve_body(const Dev& d, int k, int wg, int nunits) {
  constexpr int kG = kThreads / 64;
  __shared__ int s_prop[kG];
  __shared__ unsigned long long s_key[kG][kRetCap], s_a[kG][kRetCap];
  __shared__ int32_t s_sj[kG][kRetCap];
  const int g = (int)(threadIdx.x >> 6), lane = (int)__lane_id();
  const int w = wg * kG + g;
  const bool live = w < nunits;
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = si.par, step = si.step;
  const Arr a = pick_set(d, c->set & 1u);
  const int mode = read_err(c) ? 0 : (c->ret_ovf[par] ? 2 : 1);
  if (lane == 0) s_prop[g] = 0;
  __syncthreads();
  if (mode == 1 && live) {
    const int ne = pick(d.wgo, par)[w * kWgOut + kOutRet];
    int4 e = make_int4(0, 0, 0, 0);
    uint32_t w1 = 0, w2 = 0;
    bool chosen = false;
    if (lane < kRetCap) {  // entries past the length are read and not used
      e = pick(d.wge, par)[w * kRetCap + lane];
      w1 = d.wgk1[w * kRetCap + lane];
      w2 = pick(d.wgk, par)[w * kRetCap + lane];
    }
    const uint32_t idj = (uint32_t)e.w & 0x3FFFFFFFu;
    const int rule = (int)((uint32_t)e.w >> 30);
    if (lane < ne) {
      d.tflag[e.z] = 0;
      chosen = d.slotA[e.x] == (((unsigned long long)w1 << 32) | idj);
      s_a[g][lane] = chosen ? ((unsigned long long)(uint32_t)e.x << 32) | (uint32_t)e.z : kEmpty;
      s_sj[g][lane] = rule;
    }
    wave_sync();
    if (chosen) {  // two rules of the same pair with the same key: the lower rule
      const unsigned long long me = s_a[g][lane];
      for (int f = 0; f < ne; ++f)
        if (s_a[g][f] == me && s_sj[g][f] < rule) chosen = false;
    }
    wave_sync();
    if (lane < ne) {
      s_key[g][lane] = chosen ? ((unsigned long long)w2 << 32) | (uint32_t)e.x : kEmpty;
      s_sj[g][lane] = e.z;
    }
    wave_sync();
    if (chosen) {
      d.slotA[e.x] = kEmpty;  // only this T's wavefront reads the key that names it
      atomicAdd(&s_prop[g], 1);
      const unsigned long long key = s_key[g][lane];
      bool win = true;
      for (int f = 0; f < ne; ++f)
        if (s_sj[g][f] == e.z && s_key[g][f] < key) win = false;
      if (win) {
        multi_win(d, e.x, e.y, idj, e.z, rule);
        pick(d.wge, par)[w * kRetCap + lane].x = (int)((uint32_t)e.x | 0x80000000u);
      }
    }
  } else if (mode == 2 && live) {
    const float *X = pick(a.x, par ^ 1u), *Y = pick(a.y, par ^ 1u), *Z = pick(a.z, par ^ 1u);
    const Buckets bk =
        d.fuse ? step_buckets<true>(d, par, step) : step_buckets<false>(d, par, step);
    int s0, s1;
    range_of<kBrick>(d, w, s0, s1);
    for (int slot = s0 + lane; slot < s1; slot += 64) {
      if (d.tflag[slot] != 1) continue;
      d.tflag[slot] = 0;
      const float x = X[slot], y = Y[slot], z = Z[slot];
      const uint32_t id = a.id ? (uint32_t)a.id[slot] : (uint32_t)slot;
      const uint32_t rt = a.role[slot] & kMaskT;
      unsigned long long best = kEmpty;
      int best_sa = 0, best_r = 0, prop = 0;
      for_global_records(d, bk, x, y, z, [&](float4 A, int sa) {
        const int ida = __float_as_int(A.w);
        if ((uint32_t)ida == id) return;
        const float r2 = dist2(d, x, y, z, A);
        if (!(r2 < d.rc2)) return;
        const unsigned long long key = d.slotA[ida];
        if (key == kEmpty || (uint32_t)key != id) return;  // the A picked another T
        int got = -1;
        W4 wg{0, 0, 0, 0};
        multi_candidates(d, a, step, rt, sa, ida, id, r2, [&](int r, W4 wd, bool ex, bool acc) {
          if (got < 0 && acc && !ex && wd.w1 == (uint32_t)(key >> 32)) {
            got = r;
            wg = wd;
          }
        });
        if (got < 0) return;
        d.slotA[ida] = kEmpty;  // only this T's thread reads the key that names it
        prop++;
        const unsigned long long k2 = ((unsigned long long)wg.w2 << 32) | (uint32_t)ida;
        if (k2 < best) {
          best = k2;
          best_sa = sa;
          best_r = got;
        }
      });
      if (prop) atomicAdd(&s_prop[g], prop);
      if (best != kEmpty) multi_win(d, (int)(uint32_t)best, best_sa, id, slot, best_r);
    }
  }
  __syncthreads();
  if (lane == 0 && live) pick(d.wgo, par)[w * kWgOut + kOutProp] = s_prop[g];
}

// A bond of several rules (step 9) with its operands read ahead (rows only for
// B <= kAdjStage): states, roles, adjacency rows, and the staged (id_A, id_T)
// row for the log, with the rule in bits 30-31 of id_T.
__device__ __forceinline__ void make_bond_multi(const Dev& d, const Arr& a, uint32_t par, int w,
                                                int ida, int sa, int sj, int idj, int rule,
                                                const BondOps& o, const BondCtx& b) {
  int32_t da, dt;
  rule_deltas(d, rule, da, dt);
  const int32_t na = o.sta + da, nt = o.stt + dt;
  const uint8_t ra = role_of(d, o.tya, na), rt = role_of(d, o.tyt, nt);
  a.st[sa] = na;
  a.st[sj] = nt;
  a.role[sa] = ra;
  a.role[sj] = rt;
  if (d.fuse) {  // either particle may leave or take an A role (of any rule)
    fuse_role_change(d, a, par, b.step, sa, (uint32_t)ida, role_of(d, o.tya, o.sta), ra);
    fuse_role_change(d, a, par, b.step, sj, (uint32_t)idj, role_of(d, o.tyt, o.stt), rt);
  }
  int lost = 0;
  int32_t *rowa = a.adj + (size_t)sa * d.B, *rowt = a.adj + (size_t)sj * d.B;
  if (d.adj_staged) {
    const int fa = first_empty(o.rowa, d.B), ft = first_empty(o.rowt, d.B);
    if (fa < d.B) rowa[fa] = (int32_t)idj;
    else lost++;
    if (ft < d.B) rowt[ft] = (int32_t)ida;
    else lost++;
  } else {
    if (!adj_append(rowa, d.B, (int32_t)idj)) lost++;
    if (!adj_append(rowt, d.B, (int32_t)ida)) lost++;
  }
  if (lost) atomicAdd(b.lost, lost);
  const int2 row = make_int2(ida, (int)((uint32_t)idj | ((uint32_t)rule << 30)));
  const int p = atomicAdd(b.nw, 1);
  if (p < kWinCap) {
    pick(d.wgw, par)[w * kWinCap + p] = row;
  } else {
    const uint32_t q = atomicAdd(&d.ctl->nwin_ovf[par], 1u);
    pick(d.wov, par)[q] = row;
  }
}

// Step 8 and the bonds, from the T of every winning pair: one wavefront per
// sweep workgroup, the marked entries of its list (or, when a list overflowed,
// the flagged T's of its slots).  1,048,576 particles: scanning every slot's
// flag 8.4 us, this 7.3 us (it also maintains the next step's bins).
template <bool kBrick>
__device__ __forceinline__ void multi_final_body(const Dev& d, int k, int wg, int nunits) {
  constexpr int kG = kThreads / 64;
  __shared__ int s_nw[kG], s_lost[kG];
  const int g = (int)(threadIdx.x >> 6), lane = (int)__lane_id();
  const int w = wg * kG + g;
  const bool live = w < nunits;
  if (lane == 0) {
    s_nw[g] = 0;
    s_lost[g] = 0;
  }
  __syncthreads();
  const Ctl* c = d.ctl;
  const StepInfo si = step_info(c, k);
  const uint32_t par = si.par, step = si.step;
  const Arr a = pick_set(d, c->set & 1u);
  const BondCtx bc{&s_nw[g], &s_lost[g], step};
  // the pair (A ida in slot sa, T id in slot) of rule r, the T's winner
  auto decide = [&](int slot, uint32_t id, int ida, int sa, int r) __attribute__((always_inline)) {
    const uint8_t also_a = d.wfa[slot], also_t = d.wft[sa];
    // a particle takes at most one bond per step: what is read here is what a
    // bond made after the decision would read
    BondOps o{a.st[sa], a.st[slot], a.typ[sa], a.typ[slot], make_int4(0, 0, 0, 0),
              make_int4(0, 0, 0, 0), 0, 0.0f, 0.0f, 0.0f};
    if (d.adj_staged) {
      o.rowa = row_load(a.adj + (size_t)sa * d.B, d.B);
      o.rowt = row_load(a.adj + (size_t)slot * d.B, d.B);
    }
    const W4 wd = philox(step, (uint32_t)ida, id, rule_tag(d, r), d.seed);
    bool keep = true;
    if (also_a) {  // this T also won as the A of another pair
      const int4 q = d.wina[slot];
      const W4 wo = philox(step, id, (uint32_t)q.x, rule_tag(d, q.z), d.seed);
      keep = key_less(((unsigned long long)wd.w3 << 32) | (uint32_t)ida, r,
                      ((unsigned long long)wo.w3 << 32) | (uint32_t)q.x, q.z);
    }
    if (keep && also_t) {  // the A also won as the T of another pair
      const int4 q = d.wint[sa];
      const W4 wo = philox(step, (uint32_t)q.x, (uint32_t)ida, rule_tag(d, q.z), d.seed);
      keep = key_less(((unsigned long long)wd.w3 << 32) | id, r,
                      ((unsigned long long)wo.w3 << 32) | (uint32_t)q.x, q.z);
    }
    if (keep) make_bond_multi(d, a, par, w, ida, sa, slot, (int)id, r, o, bc);
  };
  int ne = 0;
  int4 e = make_int4(0, 0, 0, 0);
  if (live) {  // the list's length and its entries in one round trip
    ne = pick(d.wgo, par)[w * kWgOut + kOutRet];
    if (lane < kRetCap) e = pick(d.wge, par)[w * kRetCap + lane];
  }
  const int mode = read_err(c) ? 0 : (c->ret_ovf[par] ? 2 : 1);
  if (mode == 1 && live) {
    if (lane < ne && e.x < 0)
      decide(e.z, (uint32_t)e.w & 0x3FFFFFFFu, e.x & 0x7FFFFFFF, e.y, (int)((uint32_t)e.w >> 30));
  } else if (mode == 2 && live) {
    int s0, s1;
    range_of<kBrick>(d, w, s0, s1);
    for (int slot = s0 + lane; slot < s1; slot += 64) {
      if (!d.wft[slot]) continue;
      const int4 t = d.wint[slot];
      decide(slot, a.id ? (uint32_t)a.id[slot] : (uint32_t)slot, t.x, t.y, t.z);
    }
  }
  __syncthreads();
  if (lane == 0 && live) {
    int32_t* out = pick(d.wgo, par) + w * kWgOut;
    out[kOutBonds] = s_nw[g];
    out[kOutLost] = s_lost[g];
  }
}

// ---------------------------------------------------------------------------
// Bonded-force coupling: velocity Verlet with the mirror-LJ bond force over
// the adjacency table (Sec. II D, Eq. (mirror LJ)), md_theta steps before each
// reaction step.  Every operation is FP32, rounded on its own, in the order
// the oracle uses.  Only bonded particles feel a force, so
//   k_md_free  takes a particle without bonds through all md_theta drifts in
//              registers (one read and one write of its state instead of
//              md_theta) and gathers the bonded ones into compact arrays, each
//              workgroup's kThreads * kMdPer particles into their own range:
//              position, velocity with the slot, and slot -> compact index.
//              (One list for all, reserved by a global counter, serialised at
//              its address: 116 us with one reservation per wavefront, 24-27
//              with one per workgroup);
//   k_md_sub   sub-step m = 0 .. theta over the compact arrays alone, one
//              workgroup per range: m = 0 kicks half a step and drifts, 0 < m <
//              theta completes the previous step's second half kick, kicks and
//              drifts, m = theta completes the last one and writes the state
//              back.  Sub-step 0 also turns the adjacency rows (ids) into rows
//              of compact indices, so that a bond costs one 16-byte gather.
// The compact positions ping-pong between the overflow record arrays and the
// index map is the sort's rank array (both idle between the reaction steps).
// The positions are read from and written back to the parity of the reaction
// step.  Bound: k_md_free by HBM (64 bytes per particle at B = 4), k_md_sub by
// its launch while few particles are bonded.  1,048,576 particles, ten MD
// steps per reaction step, the first 32 reaction steps (up to 6% bonded): one
// kernel over all particles per MD step took 11 x 15.5 us; k_md_free 18 us
// and 11 x 4.5-4.8 us.  Over 320 reaction steps k_md_sub takes 7.4 us on
// average, 17 at most; with every particle bonded (1,030,301 in chains) a run of
// 8 reaction steps takes 2.4 ms, 4.4 by the one kernel.
// ---------------------------------------------------------------------------
// Whether the MD left a particle in the box: a drift of a box length or more is
// not undone by the single wrap, and a position outside has no cell.
__device__ __forceinline__ bool in_box(const Dev& d, float x, float y, float z) {
  return x >= 0.0f && x < d.L && y >= 0.0f && y < d.L && z >= 0.0f && z < d.L;
}

__global__ __launch_bounds__(kThreads) void k_md_free(Dev d, int k) {
  __shared__ int32_t s_slot[kThreads * kMdPer];  // the workgroup's bonded slots
  __shared__ int s_n;
  const Ctl* c = d.ctl;
  const uint32_t par = (c->par0 + (uint32_t)k) & 1u;
  const Arr a = pick_set(d, c->set & 1u);
  float *X = pick(a.x, par), *Y = pick(a.y, par), *Z = pick(a.z, par);
  if (read_err(c)) return;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  const int i0 = blockIdx.x * (kThreads * kMdPer) + threadIdx.x;
  float x[kMdPer], y[kMdPer], z[kMdPer], vx[kMdPer], vy[kMdPer], vz[kMdPer];
  bool bonded[kMdPer];
#pragma unroll
  for (int u = 0; u < kMdPer; ++u) {
    const int i = i0 + u * kThreads;
    bonded[u] = false;
    if (i < d.n) {
      if (d.md_all) {
        bonded[u] = true;
      } else if (d.md_vec) {
        const int4 r = ((const int4*)a.adj)[i];
        bonded[u] = r.x >= 0 || r.y >= 0 || r.z >= 0 || r.w >= 0;
      } else {
        const int32_t* row = a.adj + (size_t)i * d.B;
        for (int b = 0; b < d.B; ++b) bonded[u] |= row[b] >= 0;
      }
      x[u] = X[i];
      y[u] = Y[i];
      z[u] = Z[i];
      vx[u] = a.vx[i];
      vy[u] = a.vy[i];
      vz[u] = a.vz[i];
    }
  }
#pragma unroll
  for (int u = 0; u < kMdPer; ++u) {
    const unsigned long long m = __ballot(bonded[u]);
    if (m) {  // the wavefront's bonded lanes, in lane order
      int at = 0;
      if (__lane_id() == 0) at = atomicAdd(&s_n, (int)__popcll(m));
      at = __builtin_amdgcn_readlane(at, 0);
      if (bonded[u]) s_slot[at + (int)lanes_below(m)] = i0 + u * kThreads;
    }
  }
  bool inside = true;
#pragma unroll
  for (int u = 0; u < kMdPer; ++u) {
    const int i = i0 + u * kThreads;
    if (i >= d.n || bonded[u]) continue;
    // the half kicks of a force-free particle add +0 (which turns -0 into +0)
    const float wx = __fadd_rn(vx[u], 0.0f), wy = __fadd_rn(vy[u], 0.0f),
                wz = __fadd_rn(vz[u], 0.0f);
    const float sx = __fmul_rn(d.md_dt, wx), sy = __fmul_rn(d.md_dt, wy),
                sz = __fmul_rn(d.md_dt, wz);
    float px = x[u], py = y[u], pz = z[u];
    for (int t = 0; t < d.md_theta; ++t) {
      px = wrap_box(__fadd_rn(px, sx), d.L);
      py = wrap_box(__fadd_rn(py, sy), d.L);
      pz = wrap_box(__fadd_rn(pz, sz), d.L);
    }
    inside &= in_box(d, px, py, pz);
    X[i] = px;
    Y[i] = py;
    Z[i] = pz;
    a.vx[i] = wx;
    a.vy[i] = wy;
    a.vz[i] = wz;
  }
  if (!inside) set_err(d.ctl, PR_EINVAL);
  __syncthreads();
  const int nb = s_n, q0 = blockIdx.x * (kThreads * kMdPer);
  if (threadIdx.x == 0) d.md_n[blockIdx.x] = nb;
  for (int e = threadIdx.x; e < nb; e += kThreads) {
    const int i = s_slot[e], q = q0 + e;
    d.rank[i] = q;
    d.ovf[0][q] = make_float4(X[i], Y[i], Z[i], 0.0f);
    d.md_vel[q] = make_float4(a.vx[i], a.vy[i], a.vz[i], __int_as_float(i));
  }
}

// The mirror-LJ force of the partner at o on the particle at p, added to f;
// false when the bond is stretched to 2 sigma_c or beyond.
__device__ __forceinline__ bool md_bond(const Dev& d, float4 p, float4 o, float& fx, float& fy,
                                        float& fz) {
  const float dx = min_image(__fsub_rn(o.x, p.x), d.L, d.halfL);
  const float dy = min_image(__fsub_rn(o.y, p.y), d.L, d.halfL);
  const float dz = min_image(__fsub_rn(o.z, p.z), d.L, d.halfL);
  const float r2 = __fadd_rn(__fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy)), __fmul_rn(dz, dz));
  if (!(r2 > d.md_sc2)) return true;  // no force up to sigma_c
  const float r = sqrt_rn(r2);
  const float sgap = __fsub_rn(d.md_two_sc, r);
  if (!(sgap > 0.0f)) return false;
  const float q = __fdiv_rn(d.md_sig, sgap);
  const float q2 = __fmul_rn(q, q);
  const float q6 = __fmul_rn(__fmul_rn(q2, q2), q2);
  const float q12 = __fmul_rn(q6, q6);
  const float cf =
      __fdiv_rn(__fdiv_rn(__fmul_rn(d.md_e24, __fsub_rn(__fadd_rn(q12, q12), q6)), sgap), r);
  fx = __fadd_rn(fx, __fmul_rn(cf, dx));
  fy = __fadd_rn(fy, __fmul_rn(cf, dy));
  fz = __fadd_rn(fz, __fmul_rn(cf, dz));
  return true;
}

// The compact index of partner id j (-1: none; an entry that names no particle,
// which a loaded row may hold, is no bond).
__device__ __forceinline__ int32_t md_index(const Dev& d, int32_t j) {
  return (uint32_t)j < (uint32_t)d.n ? d.rank[d.slot_of[j]] : -1;
}

__global__ __launch_bounds__(kThreads) void k_md_sub(Dev d, int k, int m) {
  const Ctl* c = d.ctl;
  const uint32_t par = (c->par0 + (uint32_t)k) & 1u;
  const int nb = d.md_n[blockIdx.x], q0 = blockIdx.x * (kThreads * kMdPer), B = d.B;
  if (read_err(c)) return;
  const Arr a = pick_set(d, c->set & 1u);
  const float4* P = pick(d.ovf, (uint32_t)m);
  float4* PW = pick(d.ovf, (uint32_t)m ^ 1u);
  const float h = d.md_h;
  for (int e = threadIdx.x; e < nb; e += kThreads) {
    const int q = q0 + e;
    const float4 p = P[q], v4 = d.md_vel[q];
    const int slot = __float_as_int(v4.w);
    float fx = 0.0f, fy = 0.0f, fz = 0.0f;
    bool ok = true;
    if (d.md_vec) {  // the four partners gathered together, then taken in row order
      int4 j;
      if (m == 0) {
        j = ((const int4*)a.adj)[slot];
        j = make_int4(md_index(d, j.x), md_index(d, j.y), md_index(d, j.z), md_index(d, j.w));
        ((int4*)d.md_row)[q] = j;
      } else {
        j = ((const int4*)d.md_row)[q];
      }
      float4 o0 = p, o1 = p, o2 = p, o3 = p;  // at distance 0: no force
      if (j.x >= 0) o0 = P[j.x];
      if (j.y >= 0) o1 = P[j.y];
      if (j.z >= 0) o2 = P[j.z];
      if (j.w >= 0) o3 = P[j.w];
      ok = md_bond(d, p, o0, fx, fy, fz);
      ok = md_bond(d, p, o1, fx, fy, fz) && ok;
      ok = md_bond(d, p, o2, fx, fy, fz) && ok;
      ok = md_bond(d, p, o3, fx, fy, fz) && ok;
    } else {
      int32_t* row = d.md_row + (size_t)q * B;
      for (int b = 0; b < B; ++b) {
        int32_t j;
        if (m == 0) {
          j = md_index(d, a.adj[(size_t)slot * B + b]);
          row[b] = j;
        } else {
          j = row[b];
        }
        if (j >= 0) ok = md_bond(d, p, P[j], fx, fy, fz) && ok;
      }
    }
    if (!ok) set_err(d.ctl, PR_EINVAL);
    float vx = v4.x, vy = v4.y, vz = v4.z;
    if (m > 0) {  // the second half kick of the previous MD step
      vx = __fadd_rn(vx, __fmul_rn(h, fx));
      vy = __fadd_rn(vy, __fmul_rn(h, fy));
      vz = __fadd_rn(vz, __fmul_rn(h, fz));
    }
    if (m < d.md_theta) {  // the first half kick and the drift of MD step m
      vx = __fadd_rn(vx, __fmul_rn(h, fx));
      vy = __fadd_rn(vy, __fmul_rn(h, fy));
      vz = __fadd_rn(vz, __fmul_rn(h, fz));
      PW[q] = make_float4(wrap_box(__fadd_rn(p.x, __fmul_rn(d.md_dt, vx)), d.L),
                          wrap_box(__fadd_rn(p.y, __fmul_rn(d.md_dt, vy)), d.L),
                          wrap_box(__fadd_rn(p.z, __fmul_rn(d.md_dt, vz)), d.L), 0.0f);
      d.md_vel[q] = make_float4(vx, vy, vz, v4.w);
    } else {
      if (!in_box(d, p.x, p.y, p.z)) set_err(d.ctl, PR_EINVAL);
      pick(a.x, par)[slot] = p.x;
      pick(a.y, par)[slot] = p.y;
      pick(a.z, par)[slot] = p.z;
      a.vx[slot] = vx;
      a.vy[slot] = vy;
      a.vz[slot] = vz;
    }
  }
}

// Whether some row names a particle whose own row is empty (only a loaded
// configuration can: a bond fills both rows, or finds one of them full): then
// ctl->md_lone is set, and every particle is taken as bonded (Dev::md_all).
__global__ __launch_bounds__(kThreads) void k_md_check(Dev d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const int32_t* adj = pick_set(d, d.ctl->set & 1u).adj;
  for (int b = 0; b < d.B; ++b) {
    const int32_t j = adj[(size_t)i * d.B + b];
    if ((uint32_t)j >= (uint32_t)d.n) continue;  // names no particle
    const int32_t* row = adj + (size_t)d.slot_of[j] * d.B;
    bool empty = true;
    for (int e = 0; e < d.B; ++e) empty &= row[e] < 0;
    if (empty) d.ctl->md_lone = 1u;
  }
}

// Initial velocities: per component the Irwin-Hall(4) offset of the bytes of
// word d of the Philox block (0, id, 0, 6) times cv = fl32(sqrt(T / 21845)).
__global__ __launch_bounds__(kThreads) void k_md_init(Dev d, unsigned long long vseed, float cv) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  int32_t S[3];
  ih4(0u, a.id ? (uint32_t)a.id[i] : (uint32_t)i, 6u, vseed, S);
  a.vx[i] = __fmul_rn((float)S[0], cv);
  a.vy[i] = __fmul_rn((float)S[1], cv);
  a.vz[i] = __fmul_rn((float)S[2], cv);
}

// The id -> slot map of the current storage set.
__global__ __launch_bounds__(kThreads) void k_slot_of(Dev d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  d.slot_of[a.id ? a.id[i] : i] = i;
}

// Velocities in particle-id order.
__global__ __launch_bounds__(kThreads) void k_gather_v(Dev d, float* ox, float* oy, float* oz) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  const int id = a.id ? a.id[i] : i;
  ox[id] = a.vx[i];
  oy[id] = a.vy[i];
  oz[id] = a.vz[i];
}

// ---------------------------------------------------------------------------
// Kinetics counters of the current configuration (the quantities of the
// paper's rate equations, Sec. II B-C): populations of the A type by state,
// and, per state of the A-eligible particles, their T-eligible partners
// within the cutoff (not bonded to them when the rule excludes bonded pairs)
// with a histogram of those pairs by distance.  Three kernels: the binning of
// the A's at the current positions (k_prep without re-jitter), the counting
// (each pair found once, from its T, as in the sweep; counts to LDS, then one
// global atomic per workgroup and counter into one of kKinSlices slices) and
// k_kin_end.
// ---------------------------------------------------------------------------
// The distance bin of an in-range pair: the b with e2[b] <= r2 < e2[b + 1]
// (the last bin ends at the cutoff), found from a guess by the uniform bin
// width in r and moved by the exact edges, so that no pair walks every bin.
__device__ __forceinline__ int kin_bin(float r2, const float* e2, int nbins, float scale) {
  int b = (int)(__fsqrt_rn(r2) * scale);
  b = b < 0 ? 0 : (b > nbins - 1 ? nbins - 1 : b);
  while (b > 0 && r2 < e2[b]) --b;
  while (b + 1 < nbins && !(r2 < e2[b + 1])) ++b;
  return b;
}

// A workgroup's counters in LDS.
struct KinLds {
  uint32_t pop[kKinMaxState], pairs[kKinMaxState], hist[kKinMaxBins];
  float e2[kKinMaxBins + 1];
};

// Cleared, with the bin edges e2[b] = fl32((rc b / nbins)^2), the product in
// double.
__device__ __forceinline__ void kin_init(KinLds& s, int nstate, int nbins, double rc) {
  for (int q = threadIdx.x; q < nstate; q += kThreads) s.pop[q] = s.pairs[q] = 0u;
  for (int q = threadIdx.x; q <= nbins; q += kThreads) {
    if (q < nbins) s.hist[q] = 0u;
    const double r = rc * (double)q / (double)nbins;
    s.e2[q] = (float)(r * r);
  }
}

__device__ __forceinline__ void kin_count_pop(const Dev& d, KinLds& s, int nstate, int32_t typ,
                                              int32_t st) {
  if (typ == d.rule.type_a && st >= 0 && st < nstate) atomicAdd(&s.pop[st], 1u);
}

// A pair of the A in slot sa (row of it staged, or nullptr) and the T id.
__device__ __forceinline__ void kin_pair(const Dev& d, const Arr& a, KinLds& s, int nstate,
                                         int nbins, float scale, int sa, uint32_t id, float r2,
                                         const int4* arow) {
  const int32_t st = a.st[sa];
  if (d.rule.exclude && pair_bonded(d, a, sa, id, arow)) return;
  if (st >= 0 && st < nstate) atomicAdd(&s.pairs[st], 1u);
  if (nbins > 0) atomicAdd(&s.hist[kin_bin(r2, s.e2, nbins, scale)], 1u);
}

// The workgroup's sums into its slice (few workgroups share an address).
__device__ __forceinline__ void kin_flush(const KinLds& s, int nstate, int nbins,
                                          unsigned long long* kin) {
  unsigned long long* v = kin + (size_t)(blockIdx.x % kKinSlices) * kKinStride;
  for (int q = threadIdx.x; q < nstate; q += kThreads) {
    if (s.pop[q]) atomicAdd(&v[q], (unsigned long long)s.pop[q]);
    if (s.pairs[q]) atomicAdd(&v[kKinMaxState + q], (unsigned long long)s.pairs[q]);
  }
  for (int q = threadIdx.x; q < nbins; q += kThreads)
    if (s.hist[q]) atomicAdd(&v[2 * kKinMaxState + q], (unsigned long long)s.hist[q]);
}

__device__ __forceinline__ Buckets kin_buckets(const Dev& d, const Ctl* c, uint32_t par) {
  return Buckets{pick(d.cnt, par), d.rec, d.rsa, pick(d.ovf, par), pick(d.ovf_sa, par),
                 c->ovf_n[par]};
}

__global__ __launch_bounds__(kThreads) void k_kin_pairs(Dev d, int nstate, int nbins, double rc,
                                                        unsigned long long* __restrict__ kin) {
  __shared__ KinLds s_kin;
  const Ctl* c = d.ctl;
  // after an error positions may be outside the box: nothing is counted, and the
  // end reports it
  const bool dead = read_err(c) != 0;
  kin_init(s_kin, nstate, nbins, rc);
  __syncthreads();
  const float scale = nbins > 0 ? (float)nbins / __fsqrt_rn(d.rc2) : 0.0f;
  const uint32_t par = c->par0;
  const Arr a = pick_set(d, c->set & 1u);
  const float *X = pick(a.x, par), *Y = pick(a.y, par), *Z = pick(a.z, par);
  const Buckets bk = kin_buckets(d, c, par);
  for (int slot = blockIdx.x * blockDim.x + threadIdx.x; slot < d.n && !dead;
       slot += gridDim.x * blockDim.x) {
    kin_count_pop(d, s_kin, nstate, a.typ[slot], a.st[slot]);
    if (a.role[slot] != kRoleT) continue;
    const float x = X[slot], y = Y[slot], z = Z[slot];
    const uint32_t id = (uint32_t)(a.id ? a.id[slot] : slot);
    for_global_records(d, bk, x, y, z, [&](float4 A, int sa) {
      const float r2 = dist2(d, x, y, z, A);
      if (r2 < d.rc2) kin_pair(d, a, s_kin, nstate, nbins, scale, sa, id, r2, nullptr);
    });
  }
  __syncthreads();
  kin_flush(s_kin, nstate, nbins, kin);
}

// k_kin_pairs on sorted storage (brick edges up to kOneCellBrick), one
// workgroup per brick with its region's A records staged (StagedRegion): the
// same pairs, the same counts.  As in the sweep a T scans its block as one
// sequence of four runs, keeps up to four in-range records in a register and
// queues them, so that the rows, states and bins are handled on full
// wavefronts after the pass; T's with more, and T's outside the staged region,
// are handled one by one then.  1,048,576 particles: every pair handled where
// the scan met it 44.7 us (and 4.5 for the populations), this 30.1 us with them.
__global__ __launch_bounds__(kThreads) void k_kin_pairs_staged(
    Dev d, int nstate, int nbins, double rc, unsigned long long* __restrict__ kin) {
  __shared__ KinLds s_kin;
  __shared__ float4 s_rec[kStageRecs];
  __shared__ int4 s_radj[kStageRecs];
  __shared__ int32_t s_rsa[kStageRecs];
  __shared__ uint16_t s_off[kStageCells1 + 1];
  __shared__ uint32_t s_wave[kThreads / 64 + 1];
  __shared__ uint32_t s_q[kQueue];    // local T | staged record << 16
  __shared__ uint16_t s_def[kTPass];  // T's handled one by one
  __shared__ int s_qn, s_ndef;
  const int tid = threadIdx.x;
  const Ctl* c = d.ctl;
  const bool dead = read_err(c) != 0;  // as above
  kin_init(s_kin, nstate, nbins, rc);
  if (tid == 0) s_qn = s_ndef = 0;
  const float scale = nbins > 0 ? (float)nbins / __fsqrt_rn(d.rc2) : 0.0f;
  const uint32_t par = c->par0;
  const Arr a = pick_set(d, c->set & 1u);
  const float *X = pick(a.x, par), *Y = pick(a.y, par), *Z = pick(a.z, par);
  const Buckets bk = kin_buckets(d, c, par);
  const int w = xcd_brick(blockIdx.x, gridDim.x), nc = d.nc;
  int s0, s1;
  range_of<true>(d, w, s0, s1);
  StagedRegion g;
  g.rec = s_rec;
  g.radj = s_radj;
  g.rsa = s_rsa;
  g.off = s_off;
  stage_region(d, bk, w, g, s_wave);  // ends with a barrier (the tables above too)
  const bool rows = d.adj_staged != 0;
  for (int base = s0; base < s1 && !dead; base += kTPass) {
    Part cur = load_part(a, X, Y, Z, base + tid, s1);
    int32_t typ = base + tid < s1 ? a.typ[base + tid] : 0, st = base + tid < s1 ? a.st[base + tid] : -1;
#pragma unroll 1
    for (int u = 0; u < kTPass / kThreads; ++u) {
      const int lt = u * kThreads + tid, next = base + lt + kThreads;
      Part nxt = cur;
      int32_t ntyp = 0, nst = -1;
      if (u + 1 < kTPass / kThreads) {  // in flight while this one is handled
        nxt = load_part(a, X, Y, Z, next, s1);
        if (next < s1) {
          ntyp = a.typ[next];
          nst = a.st[next];
        }
      }
      if (base + lt < s1) kin_count_pop(d, s_kin, nstate, typ, st);
      if (base + lt < s1 && cur.role == kRoleT) {
        int nh = 0;
        uint32_t hits = 0;
        bool one_by_one = true;
        const int lx0 = local_lo(cur.x, d.inv_w, g.bx, nc), ly0 = local_lo(cur.y, d.inv_w, g.by, nc),
                  lz0 = local_lo(cur.z, d.inv_w, g.bz, nc);
        if (g.staged && (uint32_t)lx0 < (uint32_t)(g.ex - 1) &&
            (uint32_t)ly0 < (uint32_t)(g.ey - 1) && (uint32_t)lz0 < (uint32_t)(g.ez - 1)) {
          const int l0 = (lz0 * g.ey + ly0) * g.ex + lx0;
          const int l1 = l0 + g.ex, l2 = l0 + g.ex * g.ey, l3 = l2 + g.ex;
          const int b0 = (int)s_off[l0], b1 = (int)s_off[l1], b2 = (int)s_off[l2],
                    b3 = (int)s_off[l3];
          const int p1 = (int)s_off[l0 + 2] - b0;
          const int p2 = p1 + (int)s_off[l1 + 2] - b1;
          const int p3 = p2 + (int)s_off[l2 + 2] - b2;
          const int tot = p3 + (int)s_off[l3 + 2] - b3;
          const int o1 = b1 - p1, o2 = b2 - p2, o3 = b3 - p3;
          auto scan = [&](auto dist) {
            for (int q = 0; q < tot; ++q) {
              const int r = q + (q < p1 ? b0 : (q < p2 ? o1 : (q < p3 ? o2 : o3)));
              if (dist(s_rec[r]) < d.rc2) {
                hits |= (uint32_t)r << ((8 * nh) & 31);
                nh++;
              }
            }
          };
          if (g.nowrap) scan([&](float4 A) { return dist2_plain(cur.x, cur.y, cur.z, A); });
          else scan([&](float4 A) { return dist2(d, cur.x, cur.y, cur.z, A); });
          one_by_one = nh > 4;
          if (nh > 0 && !one_by_one) {
            const int p = atomicAdd(&s_qn, nh);
            one_by_one = p + nh > kQueue;  // the slots below kQueue are marked empty
            for (int e = 0; e < nh && p + e < kQueue; ++e)
              s_q[p + e] = one_by_one ? 0xFFFFFFFFu
                                      : (uint32_t)lt | (((hits >> (8 * e)) & 0xFFu) << 16);
          }
        }
        if (one_by_one) s_def[atomicAdd(&s_ndef, 1)] = (uint16_t)lt;
      }
      cur = nxt;
      typ = ntyp;
      st = nst;
    }
    __syncthreads();
    const int qn = min(s_qn, kQueue), nd = s_ndef;
    for (int e = tid; e < qn; e += kThreads) {
      const uint32_t q = s_q[e];
      if (q == 0xFFFFFFFFu) continue;
      const int slot = base + (int)(q & 0xFFFFu), r = (int)(q >> 16);
      kin_pair(d, a, s_kin, nstate, nbins, scale, s_rsa[r], (uint32_t)a.id[slot],
               dist2(d, X[slot], Y[slot], Z[slot], s_rec[r]), rows ? &s_radj[r] : nullptr);
    }
    for (int e = tid; e < nd; e += kThreads) {
      const int slot = base + (int)s_def[e];
      const float x = X[slot], y = Y[slot], z = Z[slot];
      const uint32_t id = (uint32_t)a.id[slot];
      for_global_records(d, bk, x, y, z, [&](float4 A, int sa) {
        const float r2 = dist2(d, x, y, z, A);
        if (r2 < d.rc2) kin_pair(d, a, s_kin, nstate, nbins, scale, sa, id, r2, nullptr);
      });
    }
    __syncthreads();
    if (tid == 0) s_qn = s_ndef = 0;
    __syncthreads();
  }
  kin_flush(s_kin, nstate, nbins, kin);
}

// The end of a read-out: workgroup 0 sums the slices of every counter in use
// (one wavefront per counter, one lane per slice) into *out, which the host
// reads after the stream, and clears them for the next read-out; the others
// leave the A grid of the current parity as a step expects to find it (no
// records; workgroup 0: no overflow).
__global__ __launch_bounds__(kFinThreads) void k_kin_end(Dev d, int nstate, int nbins,
                                                      unsigned long long* kin, KinOut* out) {
  static_assert(kKinSlices == 64, "one lane per slice");
  const uint32_t par = d.ctl->par0;
  if (blockIdx.x > 0) {
    for (int q = (blockIdx.x - 1) * kFinThreads + threadIdx.x; q < d.ncell;
         q += (gridDim.x - 1) * kFinThreads)
      pick(d.cnt, par)[q] = 0u;
    return;
  }
  const int lane = (int)__lane_id();
  for (int e = (int)(threadIdx.x >> 6); e < 2 * nstate + nbins; e += kFinThreads / 64) {
    const int q = e < nstate ? e : (e < 2 * nstate ? kKinMaxState + e - nstate
                                                   : 2 * (kKinMaxState - nstate) + e);
    unsigned long long* v = &kin[(size_t)lane * kKinStride + q];
    unsigned long long t = *v;
    *v = 0ull;
    for (int j = 32; j > 0; j >>= 1) t += __shfl_xor(t, j);
    if (lane == 0) out->v[q] = (int64_t)t;
  }
  if (threadIdx.x == 0) {
    out->err = read_err(d.ctl);
    d.ctl->ovf_n[par] = 0u;
  }
}

// ---------------------------------------------------------------------------
// Stateless single step: the first kernel (position check, roles, binning of
// the A's) and the last one (counters, the step's bonds sorted by id_A into
// the caller's buffer).  Four launches make a step: the first kernel also sets
// the control block up, the sweep clears the cell counts of the previous call
// (the calls alternate between the two count buffers), and the last one leaves
// the per-call words as the next call expects them.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_single_prep(Dev d, uint32_t step, uint32_t par) {
  __shared__ int s_na;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (threadIdx.x == 0) s_na = 0;
  if (i == 0) {  // err, ovf_n, ret_ovf and nwin_ovf are zero between calls
    d.ctl->step0 = step;
    d.ctl->par0 = par;
    d.ctl->set = 0;
  }
  __syncthreads();
  bool is_src = false;
  if (i < d.n) {
    const Arr a = pick_set(d, 0);
    const float x = a.x[0][i], y = a.y[0][i], z = a.z[0][i];
    const bool ok = (x >= 0.0f && x < d.L) && (y >= 0.0f && y < d.L) && (z >= 0.0f && z < d.L);
    if (!ok) set_err(d.ctl, PR_EINVAL);
    const uint8_t role = role_of(d, a.typ[i], a.st[i]);
    a.role[i] = role;
    is_src = role_is_a(role, d.nrules > 1);
    if (is_src && ok) {  // the unsorted sweeps read no staged adjacency rows
      const int c = cell_of(d, x, y, z);
      const uint32_t r = atomicAdd(&pick(d.cnt, par)[c], 1u);
      const float4 rec = make_float4(x, y, z, __int_as_float(i));
      if (r < (uint32_t)kCellCap) {
        const size_t ri = rec_at(d, c, r);
        d.rec[ri] = rec;
        d.rsa[ri] = i;
      } else {
        const uint32_t o = atomicAdd(&d.ctl->ovf_n[par], 1u);
        pick(d.ovf, par)[o] = rec;
        pick(d.ovf_sa, par)[o] = i;
      }
    }
  }
  const unsigned long long m = __ballot(is_src);
  if (__lane_id() == 0 && m) atomicAdd(&s_na, (int)__popcll(m));
  __syncthreads();
  if (threadIdx.x == 0) pick(d.abst, par)[blockIdx.x] = s_na;
}

__device__ void bitonic_sort(unsigned long long* buf, int n2) {
  for (int k = 2; k <= n2; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int t = threadIdx.x; t < n2; t += blockDim.x) {
        const int ixj = t ^ j;
        if (ixj > t) {
          const unsigned long long a = buf[t], b = buf[ixj];
          const bool up = (t & k) == 0;
          if ((a > b) == up) {
            buf[t] = b;
            buf[ixj] = a;
          }
        }
      }
      __threadfence_block();
      __syncthreads();
    }
}

// The first n2 keys (a power of two up to 1024), one per thread of a
// 1024-thread workgroup, sorted ascending: the bitonic network with the
// exchanges inside a wavefront as lane shuffles (45 of the 55 steps of 1024
// keys) and only those across wavefronts through LDS and barriers.  buf: 1024
// keys of LDS.
__device__ __forceinline__ unsigned long long sort_1024(unsigned long long key, int n2,
                                                        unsigned long long* buf) {
  const int t = threadIdx.x;
  for (int k = 2; k <= n2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      unsigned long long other;
      if (j >= 64) {
        __syncthreads();
        buf[t] = key;
        __syncthreads();
        other = buf[t ^ j];
      } else {
        other = __shfl_xor(key, j);
      }
      // the lower place of a pair keeps the smaller key in an ascending run
      const bool keep_min = ((t & j) == 0) == ((t & k) == 0);
      key = keep_min == (key < other) ? key : other;
    }
  }
  return key;
}

// A bond key (id_A << 32 | id_T) as row t of the caller's buffer; with several
// rules the rule rides in bits 30-31 of id_T.
__device__ __forceinline__ void put_bond(const Dev& d, int64_t t, unsigned long long key) {
  if (t >= d.bonds_cap) return;
  const uint32_t tt = (uint32_t)key;
  if (d.bonds_rule) {
    d.bonds[3 * t] = (int32_t)(key >> 32);
    d.bonds[3 * t + 1] = (int32_t)(d.nrules > 1 ? tt & 0x3FFFFFFFu : tt);
    d.bonds[3 * t + 2] = (int32_t)(d.nrules > 1 ? tt >> 30 : 0u);
  } else {
    d.bonds[2 * t] = (int32_t)(key >> 32);
    d.bonds[2 * t + 1] = (int32_t)tt;
  }
}

// The last kernel: one workgroup sums the counters of the sweep workgroups and
// collects their staged bonds (keys to LDS, beyond kSortLds to sortbuf), sorts
// them and reports to *out, which the host reads after the stream.  Bound by
// its round trips: the counters of 4 sweep workgroups per thread at 1M
// particles are loaded together.  It replaces the closing, block-end and sort
// kernels and two copies: 36 us of kernels at 1,000,003 particles (950 bonds),
// now 17.4-19.9 us; 9 us at 4,000, now 5.
__global__ __launch_bounds__(kFinThreads) void k_single_finish(Dev d, uint32_t par, SingleOut* out) {
  __shared__ unsigned long long s_b[kSortLds];
  __shared__ unsigned long long s_sum[kPart];
  __shared__ int s_nb;
  const int tid = threadIdx.x;
  Ctl* c = d.ctl;
  if (tid < kPart) s_sum[tid] = 0ull;
  if (tid == 0) s_nb = 0;
  __syncthreads();
  const int32_t err = read_err(c);
  const int nwov = err ? 0 : (int)c->nwin_ovf[par];
  auto keep = [&](int2 b) {
    const int p = atomicAdd(&s_nb, 1);
    const unsigned long long key = ((unsigned long long)(uint32_t)b.x << 32) | (uint32_t)b.y;
    if (p < kSortLds) s_b[p] = key;
    d.sortbuf[p] = key;
  };
  // in 64 bits: a wavefront adds up a sixteenth of all workgroups' counters
  long long v[kPart] = {0, 0, 0, 0, 0, 0, 0, 0};
  constexpr int kAt = 4;  // sweep workgroups per thread and round, loaded together
  for (int w0 = tid; w0 < d.nwg_sweep; w0 += kAt * kFinThreads) {
    int nb[kAt];
#pragma unroll
    for (int u = 0; u < kAt; ++u) {
      const int w = w0 + u * kFinThreads;
      nb[u] = 0;
      if (w < d.nwg_sweep) {
        const int32_t* o = pick(d.wgo, par) + (size_t)w * kWgOut;
        v[0] += pick(d.abst, par)[w];
        v[1] += o[kOutTElig];
        v[2] += o[kOutInRc];
        v[3] += o[kOutDrawn];
        v[4] += o[kOutExcl];
        v[5] += o[kOutProp];
        v[7] += o[kOutLost];
        nb[u] = err ? 0 : o[kOutBonds];
        v[6] += nb[u];
      }
    }
#pragma unroll
    for (int u = 0; u < kAt; ++u)
      for (int e = 0; e < min(nb[u], kWinCap); ++e)
        keep((pick(d.wgw, par) + (size_t)(w0 + u * kFinThreads) * kWinCap)[e]);
  }
#pragma unroll
  for (int q = 0; q < kPart; ++q) {
    // 24 bits and (if any) the rest, so that neither sum of 64 lanes wraps
    const uint32_t high = (uint32_t)(v[q] >> 24);
    unsigned long long t = wave_scan_incl((uint32_t)v[q] & 0xFFFFFFu);
    if (__ballot(high != 0u)) t += (unsigned long long)wave_scan_incl(high) << 24;
    if (__lane_id() == 63 && t) atomicAdd(&s_sum[q], t);
  }
  for (int e = tid; e < nwov; e += kFinThreads) keep(pick(d.wov, par)[e]);
  __syncthreads();
  const int m = s_nb;
  int n2 = 1;
  while (n2 < m) n2 <<= 1;
  if (n2 <= kFinThreads) {
    const unsigned long long key = sort_1024(tid < m ? s_b[tid] : kEmpty, n2, s_b);
    if (tid < m) put_bond(d, tid, key);
  } else {
    unsigned long long* buf = n2 <= kSortLds ? s_b : d.sortbuf;
    for (int t = tid; t < n2; t += kFinThreads)
      if (t >= m) buf[t] = kEmpty;
    __threadfence_block();
    __syncthreads();
    bitonic_sort(buf, n2);
    for (int t = tid; t < m; t += kFinThreads) put_bond(d, t, buf[t]);
  }
  if (tid < kPart) out->sum[tid] = (int64_t)s_sum[tid];
  if (tid == 0) {
    out->err = err;
    out->n_bonds = m;
    c->err = 0;
    c->ovf_n[par] = 0;
    c->ret_ovf[par] = 0;
    c->nwin_ovf[par] = 0;
  }
}

// ---------------------------------------------------------------------------
// Order of a resident system's bond log by (step, id_A) when the steps were
// run in increasing order and no row was dropped: the rows of each step then lie
// together, as many as its counters say, and only need their order by id_A.
// k_log_segs finds the first row of each of the K steps from k0 on (seg[0 .. K],
// step k0's is row0) from the counter log and leaves the most rows of a step
// and the rows of all in ctl->log_most and log_rows; k_log_steps sorts the rows
// of step blockIdx.x of these in LDS, in place.  Bound by latency (two
// launches; the steps are sorted beside each other).  It replaces a radix sort
// of the whole log (eight passes over 64-bit keys) for logs of up to kLogLds
// rows per step: 13 launches; a system of 4,000 particles after 200 steps read
// its bonds in 80 us, now 54.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kFinThreads) void k_log_segs(Dev d, int k0, int K, uint32_t row0,
                                                           uint32_t* seg) {
  __shared__ uint32_t s_wave[kFinThreads / 64 + 1];
  __shared__ uint32_t s_most;
  if (threadIdx.x == 0) s_most = 0;
  uint32_t carry = 0;
  for (int base = 0; base < K; base += kFinThreads) {
    const int k = base + (int)threadIdx.x;
    uint32_t v = 0;
    if (k < K) {
      // the bonds of each group
      const int32_t* p = d.part + (size_t)(k0 + k) * d.ngroups * kPart + 6;
      for (int g = 0; g < d.ngroups; ++g) v += (uint32_t)p[g * kPart];
    }
    uint32_t total = 0;
    const uint32_t ex = block_scan_excl<kFinThreads>(v, s_wave, total);
    if (k < K) seg[k] = row0 + carry + ex;
    carry += total;
    if (v) atomicMax(&s_most, v);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    seg[K] = row0 + carry;
    d.ctl->log_most = s_most;
    d.ctl->log_rows = carry;
  }
}

__global__ __launch_bounds__(kThreads) void k_log_steps(Dev d, const uint32_t* seg) {
  __shared__ unsigned long long s_b[kLogLds];
  const uint32_t r0 = seg[blockIdx.x], r1 = seg[blockIdx.x + 1];
  const int m = (int)(r1 - r0);
  if (m < 2 || m > kLogLds) return;
  int32_t* row = d.log + 3 * (size_t)r0;
  int n2 = 2;
  while (n2 < m) n2 <<= 1;
  for (int t = threadIdx.x; t < n2; t += kThreads)
    s_b[t] = t < m ? ((unsigned long long)(uint32_t)row[3 * t + 1] << 32) | (uint32_t)row[3 * t + 2]
                   : kEmpty;
  __syncthreads();
  bitonic_sort(s_b, n2);
  for (int t = threadIdx.x; t < m; t += kThreads) {  // the step number stays
    row[3 * t + 1] = (int32_t)(s_b[t] >> 32);
    row[3 * t + 2] = (int32_t)(uint32_t)s_b[t];
  }
}

// ---------------------------------------------------------------------------
// Spatial sort of the storage by brick, within a brick its A's first and the
// rest by dual cell (counting sort: count, per-brick scan, scan over bricks,
// scatter).  Results never depend on the storage order; the sort only gives
// each sweep workgroup a compact region and its wavefronts similar blocks.
// ---------------------------------------------------------------------------
// The sort bin of a particle: its brick b and, within it, bin 0 for an A
// (the brick's few A's then share a handful of cache lines, which the binning
// of every step reads), else 1 + its dual cell floor(u - 1/2) (u = position /
// cell width; bs + 1 values per dimension from the brick's first cell - 1).
// All T's of one dual cell have the same 2x2x2 partner block, so a wavefront
// of them scans runs of equal length.
__device__ __forceinline__ int sort_bin(const Dev& d, float x, float y, float z, uint8_t role,
                                        int& b) {
  const float ux = __fmul_rn(x, d.inv_w), uy = __fmul_rn(y, d.inv_w), uz = __fmul_rn(z, d.inv_w);
  const int nc = d.nc, bs = d.bs, e = bs + 1;
  int bx = 0, by = 0, bz = 0;
  if (d.nbricks > 1) {
    bx = cell1(ux, nc) / bs;
    by = cell1(uy, nc) / bs;
    bz = cell1(uz, nc) / bs;
  }
  b = (bz * d.nb + by) * d.nb + bx;
  const int lx = min(max((int)floorf(__fsub_rn(ux, 0.5f)) - (bx * bs - 1), 0), bs);
  const int ly = min(max((int)floorf(__fsub_rn(uy, 0.5f)) - (by * bs - 1), 0), bs);
  const int lz = min(max((int)floorf(__fsub_rn(uz, 0.5f)) - (bz * bs - 1), 0), bs);
  return b * d.nd + (role_is_a(role, d.nrules > 1) ? 0 : 1 + (lz * e + ly) * e + lx);
}

// Ranks within sort bins.  The storage is in bin order from the previous
// sort, so the 64 particles of a wavefront fall into few bins: the lowest lane
// of each bin reserves the ranks of all its lanes with one returning atomic.
// kFresh: storage in another order (the first sort after a load), a wavefront
// holds as many bins as lanes: one atomic per lane.
template <bool kFresh = false>
__device__ __forceinline__ void sort_count_body(const Dev& d, int k) {
  const bool valid = k < d.n;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  const uint32_t par = d.ctl->par0;
  int b, bin = -1;
  if (valid)
    bin = sort_bin(d, pick(a.x, par)[k], pick(a.y, par)[k], pick(a.z, par)[k], a.role[k], b);
  if (kFresh) {
    if (valid) d.rank[k] = (int32_t)atomicAdd(&d.dcnt[bin], 1u);
    return;
  }
  // group the lanes by bin: each round takes the lowest ungrouped lane's bin
  int leader = 0;
  unsigned long long peers = 0ull;
  unsigned long long todo = __ballot(valid);
  while (todo) {
    const int ld = (int)__builtin_ctzll(todo);
    const int lb = __builtin_amdgcn_readlane(bin, ld);
    const bool mine = valid && bin == lb;
    const unsigned long long m = __ballot(mine);
    if (mine) {
      leader = ld;
      peers = m;
    }
    todo &= ~m;
  }
  uint32_t r = 0u;
  if (valid && __lane_id() == (unsigned)leader)
    r = atomicAdd(&d.dcnt[bin], (uint32_t)__popcll(peers));
  r = (uint32_t)__shfl((int)r, leader);
  if (valid) d.rank[k] = (int32_t)(r + lanes_below(peers));
}

// Offsets of the bins within brick b (one wavefront, up to six consecutive
// bins per lane: nd = (bs + 1)^3 + 1 <= 344), the brick's total for the scan
// over bricks; the counts are cleared for the next sort.
__device__ __forceinline__ void sort_local_body(const Dev& d, int b) {
  if (b >= d.nbricks) return;
  constexpr int kPerLane = 6;
  const int lane = __lane_id(), nd = d.nd, per = (nd + 63) / 64;
  uint32_t* c = d.dcnt + (size_t)b * nd;
  uint32_t* o = d.dloc + (size_t)b * nd;
  const int j0 = lane * per;
  uint32_t v[kPerLane], sum = 0u;
#pragma unroll
  for (int q = 0; q < kPerLane; ++q) {
    v[q] = q < per && j0 + q < nd ? c[j0 + q] : 0u;
    sum += v[q];
  }
  const uint32_t x = wave_scan_incl(sum);
  uint32_t run = x - sum;
#pragma unroll
  for (int q = 0; q < kPerLane; ++q) {
    if (q < per && j0 + q < nd) {
      o[j0 + q] = run;
      c[j0 + q] = 0u;
    }
    run += v[q];
  }
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  if (lane == 0) d.bcnt[b] = total;
}

__device__ __forceinline__ void sort_scan_body(const Dev& d) {
  __shared__ uint32_t s_wave[kFinThreads / 64 + 1];
  uint32_t carry = 0;
  for (int base = 0; base < d.nbricks; base += blockDim.x) {
    const int b = base + threadIdx.x;
    const uint32_t v = b < d.nbricks ? d.bcnt[b] : 0u;
    uint32_t total = 0;
    const uint32_t ex = block_scan_excl<kFinThreads>(v, s_wave, total);
    if (b < d.nbricks) {
      d.bstart[b] = (int32_t)(carry + ex);
      d.bcnt[b] = 0u;
    }
    carry += total;
  }
  if (threadIdx.x == 0) {
    d.bstart[d.nbricks] = (int32_t)carry;
    if (d.fuse) {  // overflow of the first two steps after the sort
      const uint32_t s0 = d.ctl->step0;
      d.ctl->fovf_n[mod3(s0)] = 0u;
      d.ctl->fovf_n[mod3(s0 + 1u)] = 0u;
    }
  }
}

// Row k of adj moved to row ns of o: rows of width 4 or 2 as one vector when
// both arrays are aligned.
__device__ __forceinline__ void move_row(const Dev& d, const int32_t* adj, int k, int32_t* o,
                                         int ns) {
  const bool vec = (((uintptr_t)adj | (uintptr_t)o) & 15u) == 0u;
  if (vec && d.B == 4) {
    ((int4*)o)[ns] = ((const int4*)adj)[k];
  } else if (vec && d.B == 2) {
    ((int2*)o)[ns] = ((const int2*)adj)[k];
  } else {
    for (int q = 0; q < d.B; ++q) o[(size_t)ns * d.B + q] = adj[(size_t)k * d.B + q];
  }
}

// With fused binning, the record of an A (slot ns after the sort) of the first
// step after the sort.
__device__ __forceinline__ void sort_bin_first(const Dev& d, uint32_t par, int ns, int id,
                                               uint8_t role, float x, float y, float z) {
  if (!d.fuse || !role_is_a(role, d.nrules > 1)) return;
  if (d.jitter && d.jit_c != 0.0f) rejitter(d, d.ctl->step0, (uint32_t)id, x, y, z);
  fuse_bin(d, par, d.ctl->step0, ns, (uint32_t)id, x, y, z);
}

__device__ __forceinline__ void sort_scatter_body(const Dev& d, int k) {
  if (k >= d.n) return;
  const uint32_t s = d.ctl->set & 1u, par = d.ctl->par0;
  const Arr a = pick_set(d, s), o = pick_set(d, s ^ 1u);
  const float x = pick(a.x, par)[k], y = pick(a.y, par)[k], z = pick(a.z, par)[k];
  const uint8_t role = a.role[k];
  int b;
  const int bin = sort_bin(d, x, y, z, role, b);
  const int ns = d.bstart[b] + (int)d.dloc[bin] + d.rank[k];
  pick(o.x, par)[ns] = x;
  pick(o.y, par)[ns] = y;
  pick(o.z, par)[ns] = z;
  o.typ[ns] = a.typ[k];
  o.st[ns] = a.st[k];
  o.role[ns] = role;
  const int id = a.id[k];
  o.id[ns] = id;
  if (a.vx) {
    o.vx[ns] = a.vx[k];
    o.vy[ns] = a.vy[k];
    o.vz[ns] = a.vz[k];
  }
  if (d.slot_of) d.slot_of[id] = ns;
  sort_bin_first(d, par, ns, id, role, x, y, z);
  move_row(d, a.adj, k, o.adj, ns);
}

// The scatter of a fresh sort (storage in the caller's order, so every
// particle's slot is on a line of its own): one 16-byte record (position, id)
// and one 8-byte one (type, state) per particle instead of seven 4- and 1-byte
// stores, into the overflow arrays (idle at a sort), and the rows in place;
// sort_unpack then writes the arrays in slot order.  Bound by the number of
// scattered stores: 1,048,576 particles, rows of four, 113 us, now 51 and 12 us
// for the unpacking (rows of two, two rules: 70 and 13); 4,194,304: 750 us, now
// 348 and 35.
__device__ __forceinline__ void sort_scatter_fresh_body(const Dev& d, int k) {
  if (k >= d.n) return;
  const uint32_t s = d.ctl->set & 1u, par = d.ctl->par0;
  const Arr a = pick_set(d, s), o = pick_set(d, s ^ 1u);
  const float x = pick(a.x, par)[k], y = pick(a.y, par)[k], z = pick(a.z, par)[k];
  int b;
  const int bin = sort_bin(d, x, y, z, a.role[k], b);
  const int ns = d.bstart[b] + (int)d.dloc[bin] + d.rank[k];
  const int id = a.id[k];
  d.ovf[0][ns] = make_float4(x, y, z, __int_as_float(id));
  ((int2*)d.ovf[1])[ns] = make_int2(a.typ[k], a.st[k]);
  if (a.vx) d.md_vel[ns] = make_float4(a.vx[k], a.vy[k], a.vz[k], 0.0f);
  if (d.slot_of) d.slot_of[id] = ns;
  move_row(d, a.adj, k, o.adj, ns);
}
__device__ __forceinline__ void sort_unpack_body(const Dev& d, int ns) {
  if (ns >= d.n) return;
  const uint32_t s = d.ctl->set & 1u, par = d.ctl->par0;
  const Arr o = pick_set(d, s ^ 1u);
  const float4 r = d.ovf[0][ns];
  const int2 ts = ((const int2*)d.ovf[1])[ns];
  const int id = __float_as_int(r.w);
  const uint8_t role = role_of(d, ts.x, ts.y);
  pick(o.x, par)[ns] = r.x;
  pick(o.y, par)[ns] = r.y;
  pick(o.z, par)[ns] = r.z;
  o.id[ns] = id;
  o.typ[ns] = ts.x;
  o.st[ns] = ts.y;
  o.role[ns] = role;
  if (o.vx) {
    const float4 v = d.md_vel[ns];
    o.vx[ns] = v.x;
    o.vy[ns] = v.y;
    o.vz[ns] = v.z;
  }
  sort_bin_first(d, par, ns, id, role, r.x, r.y, r.z);
}

// ---------------------------------------------------------------------------
// Entry points.  One system: the kernel argument is its Dev and the grid is
// its own.  A batch of systems (independent replicas stepping in lockstep):
// the Devs live in device memory and map[blockIdx.x] = (replica, local block,
// blocks of that replica) spreads one grid over all of them.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_prep(Dev d, int k) { prep_body(d, k, blockIdx.x); }
__global__ __launch_bounds__(kThreads) void k_close(Dev d, int k) { close_body(d, k, blockIdx.x); }
__global__ void k_advance(Ctl* c, int K) {
  if (threadIdx.x == 0 && blockIdx.x == 0) advance_ctl(c, K);
}

// The Dev argument (a kernel's first), see fresh.
__device__ __forceinline__ const Dev& kernarg_dev() {
  return fresh(*(const Dev*)__builtin_amdgcn_kernarg_segment_ptr());
}

// With fused binning there is no prep kernel: the closing groups of step
// k - 1 trail the sweep of step k (workgroups nwg_sweep and up when k > 0).
// Nothing the sweep reads or writes is theirs (the counters, staged bonds and
// overflow words of step k - 1's parity, the log), and they are dispatched
// with the sweep's workgroups, so their chain of round trips (with the
// returning atomic that reserves log rows) runs beside the sweep instead of
// lengthening the resolve.
template <int kPol, bool kTwo, bool kF, bool kNt = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    kPol == kNearest ? (kF ? (kTwo ? 6 : 7) : (kTwo ? 5 : 6)) : 7))) void k_sweep(Dev d, int k) {
  if (kF && (int)blockIdx.x >= d.nwg_sweep) {
    __shared__ uint32_t s_wave[kThreads / 64 + 1];
    const StepInfo si = step_info(d.ctl, k);
    close_group(d, si.par ^ 1u, si.step - 1u, d.ctl->stats_n0 + (uint32_t)k - 1u,
                (int)blockIdx.x - d.nwg_sweep, s_wave);
    return;
  }
  sweep_body<kPol, kTwo, kF, kNt>(kernarg_dev(), k, xcd_brick(blockIdx.x, d.nwg_sweep), d.nwg_sweep);
}
template <int kPol>
__global__ __launch_bounds__(kThreads) void k_dense_sweep(Dev d, int k) {
  dense_sweep_body<kPol>(d, k, blockIdx.x, gridDim.x);
}
template <bool kBrick>
__global__ __launch_bounds__(kThreads) void k_resolve(Dev d, int k) {
  resolve_body<kBrick, true>(d, k, blockIdx.x, d.nwg_sweep);
}
template <bool kBrick>
__global__ __launch_bounds__(kThreads) void k_near_resolve(Dev d, int k) {
  near_resolve_body<kBrick>(d, k, blockIdx.x, d.nwg_sweep);
}
template <bool kBrick>
__global__ __launch_bounds__(kThreads) void k_multi_resolve(Dev d, int k) {
  multi_resolve_body<kBrick>(d, k, blockIdx.x, d.nwg_sweep);
}
template <bool kBrick>
__global__ __launch_bounds__(kThreads) void k_multi_final(Dev d, int k) {
  multi_final_body<kBrick>(d, k, blockIdx.x, d.nwg_sweep);
}
template <bool kFresh>
__global__ __launch_bounds__(kThreads) void k_sort_count(Dev d) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  sort_count_body<kFresh>(d, k);
  if (d.fuse) {  // fused binning: the scatter bins the first step after the sort
    const uint32_t s0 = d.ctl->step0;
    for (int q = k; q < d.ncell; q += gridDim.x * blockDim.x) {
      d.fcnt[mod3(s0)][q] = 0u;
      d.fcnt[mod3(s0 + 1u)][q] = 0u;
    }
  }
}
__global__ __launch_bounds__(kThreads) void k_sort_local(Dev d) {
  sort_local_body(d, blockIdx.x * (kThreads / 64) + (int)(threadIdx.x / 64));
}
__global__ __launch_bounds__(kFinThreads) void k_sort_scan(Dev d) { sort_scan_body(d); }
__global__ __launch_bounds__(kThreads) void k_sort_scatter(Dev d) {
  sort_scatter_body(d, blockIdx.x * blockDim.x + threadIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_sort_scatter_fresh(Dev d) {
  sort_scatter_fresh_body(d, blockIdx.x * blockDim.x + threadIdx.x);
}
__global__ __launch_bounds__(kThreads) void k_sort_unpack(Dev d) {
  sort_unpack_body(d, blockIdx.x * blockDim.x + threadIdx.x);
}
__global__ void k_sort_flip(Ctl* c) {
  if (threadIdx.x == 0 && blockIdx.x == 0) c->set ^= 1u;
}

// The block's map entry, made wavefront-uniform (scalar registers) so that
// the replica's Dev is read with scalar loads.
__device__ __forceinline__ int4 uniform_map(const int4* __restrict__ map) {
  const int4 m = map[blockIdx.x];
  return make_int4(__builtin_amdgcn_readfirstlane(m.x), __builtin_amdgcn_readfirstlane(m.y),
                   __builtin_amdgcn_readfirstlane(m.z), 0);
}

// A replica takes part in steps k < k_limit of a block; its workgroups of
// later steps return at once (uniformly: the whole block belongs to it).
__global__ __launch_bounds__(kThreads) void k_prep_b(const Dev* __restrict__ ds,
                                                     const int4* __restrict__ map, int k) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (k >= d.k_limit) return;
  prep_body(d, k, m.y);
}
template <bool kTwo, bool kF>
// With fused binning, workgroups nsw and up close step k - 1 of each replica
// (closing map cmap), as the trailing workgroups of k_sweep do.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7))) void k_sweep_b(
    const Dev* __restrict__ ds, const int4* __restrict__ map, int nsw,
    const int4* __restrict__ cmap, int k) {
  if (kF && (int)blockIdx.x >= nsw) {
    const int4 c = cmap[__builtin_amdgcn_readfirstlane((int)blockIdx.x - nsw)];
    const Dev& d = ds[__builtin_amdgcn_readfirstlane(c.x)];
    if (k >= d.k_limit) return;  // the block end closes the replica's last step
    __shared__ uint32_t s_wave[kThreads / 64 + 1];
    const StepInfo si = step_info(d.ctl, k);
    close_group(d, si.par ^ 1u, si.step - 1u, d.ctl->stats_n0 + (uint32_t)k - 1u,
                __builtin_amdgcn_readfirstlane(c.y), s_wave);
    return;
  }
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (k >= d.k_limit || d.rule.policy != PR_POLICY_RANDOM) return;
  sweep_body<kRandom, kTwo, kF>(fresh(d), k, m.y, m.z);
}
template <bool kTwo>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    kTwo ? 5 : 6))) void k_near_sweep_b(const Dev* __restrict__ ds,
                                                 const int4* __restrict__ map, int k) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (k >= d.k_limit || d.rule.policy != PR_POLICY_NEAREST) return;
  sweep_body<kNearest, kTwo>(fresh(d), k, m.y, m.z);
}
// four sweep workgroups' slots per workgroup (the resolve's map)
__global__ __launch_bounds__(kThreads) void k_near_resolve_b(const Dev* __restrict__ ds,
                                                             const int4* __restrict__ map, int k) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (k >= d.k_limit || d.rule.policy != PR_POLICY_NEAREST) return;
  near_resolve_body<true>(d, k, m.y, m.z);
}
__global__ __launch_bounds__(kThreads) void k_resolve_b(const Dev* __restrict__ ds,
                                                        const int4* __restrict__ map, int k) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (k >= d.k_limit || d.rule.policy != PR_POLICY_RANDOM) return;
  resolve_body<true>(d, k, m.y, m.z);
}
__global__ __launch_bounds__(kThreads) void k_close_b(const Dev* __restrict__ ds,
                                                      const int4* __restrict__ map, int k) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  if (d.k_limit < 1) return;
  close_body(d, k < d.k_limit - 1 ? k : d.k_limit - 1, m.y);  // the replica's last step
}
// one thread per replica
__global__ void k_ctl_b(const Dev* __restrict__ ds, int nrep, int op, uint32_t arg) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrep) return;
  const Dev& d = ds[r];
  Ctl* c = d.ctl;
  if (op == 0) {
    c->step0 = d.first_step;                 // start of a block
  } else if (op == 1) {                      // end of a block of arg steps
    const int kk = d.k_limit < (int)arg ? d.k_limit : (int)arg;
    if (kk > 0) advance_ctl(c, kk);
  } else {
    c->set ^= 1u;                            // after a sort
  }
}
__global__ __launch_bounds__(kThreads) void k_sort_count_b(const Dev* __restrict__ ds,
                                                           const int4* __restrict__ map) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  sort_count_body(d, m.y * kThreads + threadIdx.x);
  if (d.fuse) {  // fused binning: the scatter bins the block's first step
    const uint32_t s0 = d.ctl->step0;
    for (int q = m.y * kThreads + threadIdx.x; q < d.ncell; q += m.z * kThreads) {
      d.fcnt[mod3(s0)][q] = 0u;
      d.fcnt[mod3(s0 + 1u)][q] = 0u;
    }
  }
}
// ngrp blocks per replica (the brick groups of the largest one)
__global__ __launch_bounds__(kThreads) void k_sort_local_b(const Dev* __restrict__ ds, int ngrp) {
  const int r = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)ngrp));
  const int g = (int)blockIdx.x - r * ngrp;
  sort_local_body(ds[r], g * (kThreads / 64) + (int)(threadIdx.x / 64));
}
__global__ __launch_bounds__(kFinThreads) void k_sort_scan_b(const Dev* __restrict__ ds) {
  const Dev& d = ds[__builtin_amdgcn_readfirstlane((int)blockIdx.x)];
  sort_scan_body(d);
}
__global__ __launch_bounds__(kThreads) void k_sort_scatter_b(const Dev* __restrict__ ds,
                                                             const int4* __restrict__ map) {
  const int4 m = uniform_map(map);
  const Dev& d = ds[m.x];
  sort_scatter_body(d, m.y * kThreads + threadIdx.x);
}

// Storage order -> particle-id order (positions of the current parity).
__global__ __launch_bounds__(kThreads) void k_gather_out(Dev d, float* ox, float* oy, float* oz,
                                                         int32_t* otyp, int32_t* ost,
                                                         int32_t* oadj) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.n) return;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  const uint32_t par = d.ctl->par0;
  const int id = a.id[k];
  if (ox) ox[id] = pick(a.x, par)[k];
  if (oy) oy[id] = pick(a.y, par)[k];
  if (oz) oz[id] = pick(a.z, par)[k];
  if (otyp) otyp[id] = a.typ[k];
  if (ost) ost[id] = a.st[k];
  if (oadj)
    for (int b = 0; b < d.B; ++b) oadj[(size_t)id * d.B + b] = a.adj[(size_t)k * d.B + b];
}

// The same for large systems on sorted storage in two kernels: one 16-byte
// record (position, state) per particle scattered by id into an overflow array
// (idle between runs) and the row as one vector, then the records unpacked in
// id order.  1,048,576 particles, rows of four: eight scattered stores per
// particle 148 us, now 50 us; 4,194,304, rows of two: 506 and
// 200.
__global__ __launch_bounds__(kThreads) void k_gather_rec(Dev d, int32_t* otyp, int32_t* oadj) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= d.n) return;
  const Arr a = pick_set(d, d.ctl->set & 1u);
  const uint32_t par = d.ctl->par0;
  const int id = a.id[k];
  d.ovf[0][id] = make_float4(pick(a.x, par)[k], pick(a.y, par)[k], pick(a.z, par)[k],
                             __int_as_float(a.st[k]));
  if (otyp) otyp[id] = a.typ[k];
  if (oadj) move_row(d, a.adj, k, oadj, id);
}
__global__ __launch_bounds__(kThreads) void k_gather_unpack(Dev d, float* ox, float* oy, float* oz,
                                                            int32_t* ost) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d.n) return;
  const float4 r = d.ovf[0][i];
  if (ox) ox[i] = r.x;
  if (oy) oy[i] = r.y;
  if (oz) oz[i] = r.z;
  if (ost) ost[i] = __float_as_int(r.w);
}

// The re-jitter alone (the stand-in for the MD between reaction steps),
// step k of a block: every particle's position of parity par moves by the
// step's offsets into parity par ^ 1, exactly as the sweep of a reaction
// step moves it, and the cell counts of the next parity are cleared as the
// sweep clears them.  No reaction happens.
template <bool kNt>
__global__ __launch_bounds__(kThreads) void k_jitter_only(Dev d, int k) {
  const Ctl* c = d.ctl;
  const uint32_t par = (c->par0 + (uint32_t)k) & 1u, step = c->step0 + (uint32_t)k;
  const Arr a = pick_set(d, c->set & 1u);
  const float *X = pick(a.x, par), *Y = pick(a.y, par), *Z = pick(a.z, par);
  float *XW = pick(a.x, par ^ 1u), *YW = pick(a.y, par ^ 1u), *ZW = pick(a.z, par ^ 1u);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < d.n) {
    float x = X[i], y = Y[i], z = Z[i];
    if (d.jit_c != 0.0f) rejitter(d, step, a.id ? (uint32_t)a.id[i] : (uint32_t)i, x, y, z);
    if (kNt) {  // the sweep's store policy
      __builtin_nontemporal_store(x, &XW[i]);
      __builtin_nontemporal_store(y, &YW[i]);
      __builtin_nontemporal_store(z, &ZW[i]);
    } else {
      XW[i] = x;
      YW[i] = y;
      ZW[i] = z;
    }
  }
  for (int q = i; q < d.ncell; q += gridDim.x * blockDim.x) pick(d.cnt, par ^ 1u)[q] = 0u;
}

// Moves the block origin by K steps of the re-jitter alone: the draw step
// and the position parity advance, the counter log does not (nothing was
// logged).
__global__ void k_advance_jitter(Ctl* c, int K) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    c->step0 += (uint32_t)K;
    c->par0 = (c->par0 + (uint32_t)K) & 1u;
  }
}

// Plain device copy of n elements of T (one element per lane and
// iteration, grid-stride): the project's own bandwidth probe, with a known
// request shape per wavefront (64 lanes x sizeof(T) contiguous bytes).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_stream_copy(const T* __restrict__ src,
                                                          T* __restrict__ dst, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

// Fills n 32-bit words with v (clears scratch inside code a caller may
// capture into a graph, where memset nodes are avoided).
__global__ __launch_bounds__(kThreads) void k_fill_u32(uint32_t* __restrict__ p, long long n,
                                                       uint32_t v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}

// The bonded-force kernel's square root on caller data (n values > 0, normal).
__global__ __launch_bounds__(kThreads) void k_sqrt_rn(const float* __restrict__ in,
                                                      float* __restrict__ out, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sqrt_rn(in[i]);
}

// The generator's words for caller counters (4 uint32 per counter).
__global__ __launch_bounds__(kThreads) void k_draws(const uint4* __restrict__ ctr, long long n,
                                                    unsigned long long key, uint4* out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint4 c = ctr[i];
  const W4 w = philox(c.x, c.y, c.z, c.w, key);
  out[i] = make_uint4(w.w0, w.w1, w.w2, w.w3);
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
static inline int blocks_for(long long n, int t) { return (int)((n + t - 1) / t); }

hipError_t launch_ctl_reset(Ctl* c, uint32_t step, int full, hipStream_t s) {
  k_ctl_reset<<<1, 64, 0, s>>>(c, step, full);
  return hipGetLastError();
}

hipError_t launch_classify(const Dev& d, hipStream_t s) {
  if (d.n > 0) k_classify<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d);
  return hipGetLastError();
}

hipError_t launch_identity(const Dev& d, hipStream_t s) {
  if (d.n > 0) k_identity<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d);
  return hipGetLastError();
}

hipError_t launch_generate(const Dev& d, int kind, unsigned long long gseed, float c0, float a,
                           int nl, unsigned long long thr, hipStream_t s) {
  if (d.n > 0)
    k_generate<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d, kind, gseed, c0, a, nl, thr);
  return hipGetLastError();
}

// The kernels of step k after the binning: sweep, resolve (and the final choice
// of several rules).
static hipError_t launch_selection(const Dev& d, int k, hipStream_t s, hipEvent_t ev_sweep0,
                                   hipEvent_t ev_sweep1) {
  // with fused binning, closing groups of step k - 1 trail the sweep
  const dim3 g(d.nwg_sweep + (d.fuse && k > 0 ? d.ngroups : 0)), b(kThreads);
  const int gr = (d.nwg_sweep + 3) / 4;  // one wavefront per sweep workgroup
  const int pol = d.nrules > 1 ? kMulti : (d.rule.policy == PR_POLICY_NEAREST ? kNearest : kRandom);
  const bool two = d.bs > kOneCellBrick;  // two region cells per staging thread
  void (*kern)(Dev, int);
  if (!d.sorted)
    kern = pol == kRandom ? k_dense_sweep<kRandom>
                          : (pol == kNearest ? k_dense_sweep<kNearest> : k_dense_sweep<kMulti>);
  else if (pol == kMulti && !d.fuse)
    kern = two ? k_sweep<kMulti, true, false> : k_sweep<kMulti, false, false>;
  else if (pol == kMulti)
    kern = two ? k_sweep<kMulti, true, true> : k_sweep<kMulti, false, true>;
  else if (!d.fuse)
    kern = pol == kRandom ? (two ? k_sweep<kRandom, true, false> : k_sweep<kRandom, false, false>)
                          : (two ? k_sweep<kNearest, true, false> : k_sweep<kNearest, false, false>);
  else if (pol == kRandom)
    kern = two ? (d.nt_pos ? k_sweep<kRandom, true, true, true> : k_sweep<kRandom, true, true>)
               : (d.nt_pos ? k_sweep<kRandom, false, true, true> : k_sweep<kRandom, false, true>);
  else
    kern = two ? k_sweep<kNearest, true, true> : k_sweep<kNearest, false, true>;
  if (ev_sweep0) hipExtLaunchKernelGGL(kern, g, b, 0, s, ev_sweep0, ev_sweep1, 0, d, k);
  else kern<<<g, b, 0, s>>>(d, k);
  if (pol == kMulti) {
    auto res = d.sorted ? k_multi_resolve<true> : k_multi_resolve<false>;
    auto fin = d.sorted ? k_multi_final<true> : k_multi_final<false>;
    res<<<gr, kThreads, 0, s>>>(d, k);
    fin<<<gr, kThreads, 0, s>>>(d, k);
  } else {
    auto res = pol == kRandom ? (d.sorted ? k_resolve<true> : k_resolve<false>)
                              : (d.sorted ? k_near_resolve<true> : k_near_resolve<false>);
    res<<<gr, kThreads, 0, s>>>(d, k);
  }
  return hipGetLastError();
}

// Step k of a block: prep (with the closing of step k - 1), sweep, resolve.
// ev_sweep0/1 (timed runs): the sweep is launched with hipExtLaunchKernel,
// which stamps the two events at the kernel's own start and end.
hipError_t launch_step(const Dev& d, int k, hipStream_t s, hipEvent_t ev_sweep0,
                       hipEvent_t ev_sweep1) {
  if (d.md_theta > 0) {
    const int g = blocks_for(d.n, kThreads * kMdPer);
    k_md_free<<<g, kThreads, 0, s>>>(d, k);
    for (int m = 0; m <= d.md_theta; ++m) k_md_sub<<<g, kThreads, 0, s>>>(d, k, m);
  }
  if (!d.fuse) {  // with fused binning the previous sweep has binned the A's
    const int prep_blocks = d.nwg_prep + (k > 0 ? d.ngroups : 0);
    k_prep<<<prep_blocks, kThreads, 0, s>>>(d, k);
  }
  return launch_selection(d, k, s, ev_sweep0, ev_sweep1);
}

hipError_t launch_block_end(const Dev& d, int K, hipStream_t s) {
  k_close<<<d.ngroups, kThreads, 0, s>>>(d, K - 1);
  k_advance<<<1, 64, 0, s>>>(d.ctl, K);
  return hipGetLastError();
}

// The stateless step: four launches (five with several rules).
hipError_t launch_single(const Dev& d, uint32_t step, uint32_t par, SingleOut* out,
                         hipStream_t s) {
  k_single_prep<<<d.nwg_sweep, kThreads, 0, s>>>(d, step, par);
  const hipError_t e = launch_selection(d, 0, s, nullptr, nullptr);
  if (e != hipSuccess) return e;
  k_single_finish<<<1, kFinThreads, 0, s>>>(d, par, out);
  return hipGetLastError();
}

// fresh: the storage is in the caller's order (the first sort after a load).
// Small systems' arrays stay in the L2s, where the plain kernels' scattered
// stores merge: kFreshMin particles is where the record scatter with its second
// kernel starts to win (load, one step and read-out: 262,144 particles 149 us
// with the plain kernels and 146 with the records, 524,288 271 and 207).
hipError_t launch_sort(const Dev& d, bool fresh, hipStream_t s) {
  const int g = blocks_for(d.n, kThreads);
  fresh = fresh && d.n >= kFreshMin;
  if (fresh) k_sort_count<true><<<g, kThreads, 0, s>>>(d);
  else k_sort_count<false><<<g, kThreads, 0, s>>>(d);
  k_sort_local<<<blocks_for(d.nbricks, kThreads / 64), kThreads, 0, s>>>(d);
  k_sort_scan<<<1, kFinThreads, 0, s>>>(d);
  if (fresh) {
    k_sort_scatter_fresh<<<g, kThreads, 0, s>>>(d);
    k_sort_unpack<<<g, kThreads, 0, s>>>(d);
  } else {
    k_sort_scatter<<<g, kThreads, 0, s>>>(d);
  }
  k_sort_flip<<<1, 64, 0, s>>>(d.ctl);
  return hipGetLastError();
}

// Batched launches (every replica in one grid per kernel).
static inline int ctl_blocks(int nrep) { return (nrep + 63) / 64; }

hipError_t launch_ctl_b(const BatchLaunch& b, int op, uint32_t arg, hipStream_t s) {
  k_ctl_b<<<ctl_blocks(b.nrep), 64, 0, s>>>(b.ds, b.nrep, op, arg);
  return hipGetLastError();
}

hipError_t launch_step_b(const BatchLaunch& b, int k, hipStream_t s) {
  if (b.fuse) {  // every replica random and fused: sweep with the closing, then resolve
    const int ncl = k > 0 ? b.n_close : 0;
    if (b.two)
      k_sweep_b<true, true><<<b.n_sweep + ncl, kThreads, 0, s>>>(b.ds, b.sweep, b.n_sweep,
                                                                  b.close, k);
    else
      k_sweep_b<false, true><<<b.n_sweep + ncl, kThreads, 0, s>>>(b.ds, b.sweep, b.n_sweep,
                                                                   b.close, k);
    k_resolve_b<<<b.n_res, kThreads, 0, s>>>(b.ds, b.res, k);
    return hipGetLastError();
  }
  if (k > 0)
    k_prep_b<<<b.n_prepk, kThreads, 0, s>>>(b.ds, b.prepk, k);
  else
    k_prep_b<<<b.n_prep0, kThreads, 0, s>>>(b.ds, b.prep0, k);
  if (b.any_random) {
    if (b.two)
      k_sweep_b<true, false><<<b.n_sweep, kThreads, 0, s>>>(b.ds, b.sweep, b.n_sweep, b.close, k);
    else
      k_sweep_b<false, false><<<b.n_sweep, kThreads, 0, s>>>(b.ds, b.sweep, b.n_sweep, b.close,
                                                             k);
    k_resolve_b<<<b.n_res, kThreads, 0, s>>>(b.ds, b.res, k);
  }
  if (b.any_nearest) {
    if (b.two)
      k_near_sweep_b<true><<<b.n_sweep, kThreads, 0, s>>>(b.ds, b.sweep, k);
    else
      k_near_sweep_b<false><<<b.n_sweep, kThreads, 0, s>>>(b.ds, b.sweep, k);
    k_near_resolve_b<<<b.n_res, kThreads, 0, s>>>(b.ds, b.res, k);
  }
  return hipGetLastError();
}

hipError_t launch_block_end_b(const BatchLaunch& b, int K, hipStream_t s) {
  k_close_b<<<b.n_close, kThreads, 0, s>>>(b.ds, b.close, K - 1);
  return launch_ctl_b(b, 1, (uint32_t)K, s);
}

hipError_t launch_sort_b(const BatchLaunch& b, hipStream_t s) {
  k_sort_count_b<<<b.n_part, kThreads, 0, s>>>(b.ds, b.part);
  k_sort_local_b<<<b.n_sortl * b.nrep, kThreads, 0, s>>>(b.ds, b.n_sortl);
  k_sort_scan_b<<<b.nrep, kFinThreads, 0, s>>>(b.ds);
  k_sort_scatter_b<<<b.n_part, kThreads, 0, s>>>(b.ds, b.part);
  return launch_ctl_b(b, 2, 0u, s);
}

hipError_t launch_gather_out(const Dev& d, float* ox, float* oy, float* oz, int32_t* otyp,
                             int32_t* ost, int32_t* oadj, hipStream_t s) {
  const int g = blocks_for(d.n, kThreads);
  if (d.sorted && d.n >= kFreshMin) {  // the fresh sort's line, for the same reason
    k_gather_rec<<<g, kThreads, 0, s>>>(d, otyp, oadj);
    if (ox || oy || oz || ost) k_gather_unpack<<<g, kThreads, 0, s>>>(d, ox, oy, oz, ost);
    return hipGetLastError();
  }
  k_gather_out<<<g, kThreads, 0, s>>>(d, ox, oy, oz, otyp, ost, oadj);
  return hipGetLastError();
}

hipError_t launch_log_segs(const Dev& d, int k0, int K, uint32_t row0, uint32_t* seg,
                           hipStream_t s) {
  k_log_segs<<<1, kFinThreads, 0, s>>>(d, k0, K, row0, seg);
  return hipGetLastError();
}

hipError_t launch_log_steps(const Dev& d, int K, const uint32_t* seg, hipStream_t s) {
  if (K > 0) k_log_steps<<<K, kThreads, 0, s>>>(d, seg);
  return hipGetLastError();
}

// n_steps of the re-jitter alone, then the block origin moved by them.
// ev0/ev1 (may be null): stamped at the start and end of each step's kernel.
hipError_t launch_jitter_only(const Dev& d, int n_steps, hipStream_t s, hipEvent_t ev0,
                              hipEvent_t ev1) {
  const dim3 g(blocks_for(d.n, kThreads)), b(kThreads);
  for (int k = 0; k < n_steps; ++k) {
    auto kern = d.nt_pos ? k_jitter_only<true> : k_jitter_only<false>;
    if (ev0) hipExtLaunchKernelGGL(kern, g, b, 0, s, ev0, ev1, 0, d, k);
    else kern<<<g, b, 0, s>>>(d, k);
  }
  k_advance_jitter<<<1, 64, 0, s>>>(d.ctl, n_steps);
  return hipGetLastError();
}

// bytes must be a multiple of width; width 4, 8 or 16.  The grid holds
// 2048 workgroups (8 per compute unit) and strides over the buffer.
hipError_t launch_stream_copy(const void* src, void* dst, long long bytes, int width,
                              hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const dim3 g(2048), b(kThreads);
  if (width == 16)
    hipExtLaunchKernelGGL(k_stream_copy<uint4>, g, b, 0, s, ev0, ev1, 0, (const uint4*)src,
                          (uint4*)dst, bytes / 16);
  else if (width == 8)
    hipExtLaunchKernelGGL(k_stream_copy<uint2>, g, b, 0, s, ev0, ev1, 0, (const uint2*)src,
                          (uint2*)dst, bytes / 8);
  else
    hipExtLaunchKernelGGL(k_stream_copy<uint32_t>, g, b, 0, s, ev0, ev1, 0, (const uint32_t*)src,
                          (uint32_t*)dst, bytes / 4);
  return hipGetLastError();
}

// Kinetics counters (the slices are zero): the A binning of the current
// positions (a copy of d without re-jitter), the counting, the end.
hipError_t launch_kinetics(const Dev& d, int nstate, int nbins, double rc, unsigned long long* kin,
                           KinOut* out, hipStream_t s) {
  Dev dn = d;
  dn.jit_c = 0.0f;
  dn.fuse = 0;  // binned into the plain buckets here, whatever the steps use
  dn.wshift = 0;  // one workgroup per brick
  k_prep<<<d.nwg_prep, kThreads, 0, s>>>(dn, 0);
  if (d.sorted && d.bs <= kOneCellBrick)
    k_kin_pairs_staged<<<d.nbricks, kThreads, 0, s>>>(dn, nstate, nbins, rc, kin);
  else
    k_kin_pairs<<<std::min(blocks_for(d.n, kThreads), 2048), kThreads, 0, s>>>(dn, nstate, nbins,
                                                                               rc, kin);
  k_kin_end<<<1 + std::min(blocks_for(d.ncell, kFinThreads), 256), kFinThreads, 0, s>>>(
      dn, nstate, nbins, kin, out);
  return hipGetLastError();
}

// ctl->md_lone of the current configuration (k_md_check); slot_of is valid.
hipError_t launch_md_check(const Dev& d, hipStream_t s) {
  k_fill_u32<<<1, kThreads, 0, s>>>(&d.ctl->md_lone, 1, 0u);
  if (d.n > 0) k_md_check<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d);
  return hipGetLastError();
}

hipError_t launch_md_init(const Dev& d, unsigned long long vseed, float cv, hipStream_t s) {
  if (d.n > 0) {
    k_slot_of<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d);
    if (cv >= 0.0f) k_md_init<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d, vseed, cv);
  }
  return hipGetLastError();
}

hipError_t launch_gather_v(const Dev& d, float* ox, float* oy, float* oz, hipStream_t s) {
  if (d.n > 0) k_gather_v<<<blocks_for(d.n, kThreads), kThreads, 0, s>>>(d, ox, oy, oz);
  return hipGetLastError();
}

hipError_t launch_sqrt_rn(const float* in, float* out, long long n, hipStream_t s) {
  if (n > 0) k_sqrt_rn<<<blocks_for(n, kThreads), kThreads, 0, s>>>(in, out, n);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, long long n, uint32_t v, hipStream_t s) {
  if (n > 0) k_fill_u32<<<(int)std::min<long long>(blocks_for(n, kThreads), 4096), kThreads, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_draws(const uint32_t* ctr, long long n, unsigned long long key, uint32_t* out,
                        hipStream_t s) {
  k_draws<<<blocks_for(n, kThreads), kThreads, 0, s>>>((const uint4*)ctr, n, key, (uint4*)out);
  return hipGetLastError();
}

}  // namespace pr
