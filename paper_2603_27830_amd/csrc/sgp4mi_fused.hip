// Elements to states in one launch: initialisation fused into propagation.
//
// jaxsgp4 traces initialisation and propagation into one function and maps it
// over satellites and times (paper sections 2.2 and 3.1); the two-stage path
// of this library instead writes a 512-byte record per satellite and reads it
// back.  For short time lists (a catalogue propagated to one or a few epochs)
// the record round trip and the second launch dominate, so this kernel keeps
// the constants on chip: the first kFusedSats lanes of a workgroup initialise a
// satellite each and leave the constants that their precision reads in LDS;
// then all lanes take the workgroup's points in output order, so that stores
// are contiguous whatever the number of times.  Batches of few satellites spread
// their times over the grid's y extent, each workgroup repeating the
// initialisation (compute units would otherwise idle).
#include "sgp4mi_initcore.h"
#include "sgp4mi_out.h"

#include <algorithm>

namespace sgp4mi {

// Satellites of a workgroup: one wavefront initialises while the others wait, and
// several workgroups on a compute unit fill the gaps.  128 lanes up to kFusedNarrow
// times of a workgroup, 256 beyond: 1M x 8 FP64 164 us with 128 and 182 with 256,
// 300,000 x 2 mixed 17 and 20, but 300,007 x 19 mixed 57 and 51, 20,000 x 200 FP64
// 103 and 88.  (128 satellites on 256 lanes 66 us where 64 on 128 took 65, 256 on
// 256 72.)  Grids of up to two workgroups per compute unit take 256 lanes from four
// times on (their points then need one pass: 4,096 deep-space satellites x 32 FP64 39
// -> 25 us, near-Earth ones the same 12).
constexpr int kFusedSats = 64;
constexpr int kFusedNarrow = 8;
constexpr int32_t kFusedLdsNarrow = 20416;  // an eighth of a compute unit's LDS

struct FusedArgs {
  int64_t n, T;
  const double* elem;   // [8][n]
  const double* t;      // [T]
  uint8_t* user_flags;  // nullable
  GravIn grav;
  double vkms;
  double ref_day;       // reference instant of the epoch row, days after JD 2415020.0
  int64_t per;          // times per workgroup
  int32_t round;        // deep-space members that LDS holds
};

// The satellite's constants as the two-stage path reads them from its slot:
// the double values, and their float roundings for the float types.
template <class TS, class TP>
__device__ __forceinline__ SatC<TS, TP> sat_of(const double* x, uint32_t info, const double* deep) {
  SatC<TS, TP> c;
  c.M0 = TS(x[kM0]); c.Mdot = TS(x[kMdot]); c.argp0 = TS(x[kArgp0]); c.argpdot = TS(x[kArgpdot]);
  c.node0 = TS(x[kNode0]); c.nodedot = TS(x[kNodedot]); c.nodecf = TS(x[kNodecf]); c.C1 = TS(x[kC1]);
  c.bC4 = TS(x[kBC4]); c.t2cof = TS(x[kT2cof]); c.argpcof = TS(x[kArgpcof]); c.Mcof = TS(x[kMcof]);
  c.D2 = TS(x[kD2]); c.D3 = TS(x[kD3]); c.D4 = TS(x[kD4]); c.bC5 = TS(x[kBC5]); c.t3cof = TS(x[kT3cof]);
  c.t4cof = TS(x[kT4cof]); c.t5cof = TS(x[kT5cof]); c.n0pp = TS(x[kN0pp]); c.a0pp = TS(x[kA0pp]);
  c.e0 = TS(x[kE0]);
  c.epoch_min = x[kEpochMin];
  c.eta = TP(x[kEta]); c.dM0 = TP(x[kDM0]); c.sinM0 = TP(x[kSinM0]); c.aycof = TP(x[kAycof]);
  c.Lcof = TP(x[kLcof]); c.c41 = TP(x[kC41]); c.x1 = TP(x[kX1]); c.x7 = TP(x[kX7]); c.cosi = TP(x[kCosi]);
  c.sini = TP(x[kSini]); c.i0 = TP(x[kI0]);
  c.spA1 = TP(x[kSpA1]); c.spX1h = TP(x[kSpX1h]); c.spX1k = TP(x[kSpX1k]); c.spX7q = TP(x[kSpX7q]);
  c.spCN = TP(x[kSpCN]); c.spCI = TP(x[kSpCI]);
  c.pC1 = TP(x[kC1]); c.pbC4 = TP(x[kBC4]); c.pD2 = TP(x[kD2]); c.pD3 = TP(x[kD3]); c.pD4 = TP(x[kD4]);
  c.pbC5 = TP(x[kBC5]); c.pMcof = TP(x[kMcof]); c.pArgpcof = TP(x[kArgpcof]); c.pA0pp = TP(x[kA0pp]);
  c.pE0 = TP(x[kE0]);
  c.info = info;
  c.deep = deep;
  return c;
}

// Gravity scalars as the initialisation kernel writes them to the record
// header.
__device__ __forceinline__ Grav grav_of(const FusedArgs& a) {
  Grav g;
  g.ke = a.grav.ke;
  g.radius = a.grav.radius;
  g.vkms = a.vkms;
  g.k2 = 0.5 * a.grav.j2;
  g.j3oj2 = a.grav.j3oj2;
  g.radius_f = float(a.grav.radius);
  g.vkms_f = float(a.vkms);
  g.k2_f = float(0.5 * a.grav.j2);
  return g;
}

// Initialisation of satellite i into rec (kNRec doubles); returns the info word
// and, with it, the elements and the epoch for a deep-space satellite's terms.
__device__ __forceinline__ uint32_t init_sat(const FusedArgs& a, int64_t i, double* rec, double* el, double* epoch,
                                             bool near_only) {
#pragma unroll
  for (int k = 0; k < 7; ++k) el[k] = a.elem[k * a.n + i];
  *epoch = a.elem[7 * a.n + i];
  uint32_t code;
  bool isimp, dsp;
  init_record<double>(a.grav, el, rec, &code, &isimp, &dsp, near_only);
  rec[kEpochMin] = 1440.0 * *epoch;
  return code | (isimp ? kInfoIsimp : 0u) | (dsp ? kInfoDeep : 0u);
}

__device__ __forceinline__ void put_flags(const FusedArgs& a, int64_t i, uint32_t info, bool resonant) {
  if (!a.user_flags || blockIdx.y != 0) return;
  const uint32_t code = info & kInfoCodeMask;
  uint8_t f = 0;
  if (info & kInfoDeep) f |= 1;
  if (info & kInfoIsimp) f |= 2;
  if (code == 1 || code == 2) f |= 4;
  if (resonant) f |= 8;
  a.user_flags[i] = f;
}

// One time: each lane initialises and propagates its own satellite.  Bound by
// VALU issue: 1M satellites FP64 43 -> 33 us with the reciprocals and roots of
// init_record; four wavefronts per SIMD (128 registers) spill and take 42.  Both
// kinds of satellite share the initialisation (repeated for deep-space ones behind
// the near-Earth ones, 100,000 with 2 % of them took 30 us, 20.5 so).
template <class TS, class TP, bool kOff32>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
    fused_one_kernel(FusedArgs a, Out<TP, kOff32> out) {
  const int64_t i = int64_t(blockIdx.x) * 64 + threadIdx.x;
  if (i >= a.n) return;
  const Grav g = grav_of(a);
  double rec[kNRec], el[7], epoch;
  const uint32_t info = init_sat(a, i, rec, el, &epoch, false);
  PointState<TP> s;
  uint32_t code;
  if (info & kInfoDeep) {
    double deep[kNDeep];
    init_deep(el, rec, g.ke, a.ref_day + epoch, deep, false);
    put_flags(a, i, info, deep[kDRes] != 0.0);
    code = deep_point<TS, TP>(sat_of<TS, TP>(rec, info, deep), g, a.t[0], s);
  } else {
    put_flags(a, i, info, false);
    code = sgp4_point<TS, TP>(sat_of<TS, TP>(rec, info, nullptr), g, a.t[0], s);
  }
  out.put(i, code, s);
}

// The constants of one satellite as the near-Earth terms of each precision read
// them (the entries of the record in its order; accessor of load_from).  The
// sizes are odd multiples of 16 bytes, so that neighbouring satellites' entries
// lie in different banks.
template <class TS, class TP>
struct LdsSat;
template <>
struct LdsSat<double, float> {  // as the mixed path: double secular terms, float periodic and drag terms
  double d[kEpochMin + 1];
  float f[kNRec - kEta];
  uint32_t info;
  __device__ __forceinline__ void put(const double* rec) {
#pragma unroll
    for (int k = 0; k <= kEpochMin; ++k) d[k] = rec[k];
#pragma unroll
    for (int k = kEta; k < kNRec; ++k) f[k - kEta] = float(rec[k]);
  }
  __device__ __forceinline__ double dbl(int k) const { return k <= kEpochMin ? d[k] : 0.0; }
  __device__ __forceinline__ float flt(int k) const { return k >= kEta ? f[k - kEta] : 0.0f; }
};
template <>
struct LdsSat<double, double> {  // all but the unfolded inclination functions
  double d[kNRec - 3];
  uint32_t info;
  uint32_t pad;
  __device__ __forceinline__ void put(const double* rec) {
#pragma unroll
    for (int k = 0; k < kNRec; ++k)
      if (k < kC41 || k > kX7) d[k < kC41 ? k : k - 3] = rec[k];
  }
  __device__ __forceinline__ double dbl(int k) const { return k < kC41 ? d[k] : k > kX7 ? d[k - 3] : 0.0; }
  __device__ __forceinline__ float flt(int) const { return 0.0f; }
};
template <>
struct LdsSat<float, float> {  // floats, the epoch in double
  double epoch;
  float f[kNRec];
  uint32_t info;
  __device__ __forceinline__ void put(const double* rec) {
    epoch = rec[kEpochMin];
#pragma unroll
    for (int k = 0; k < kNRec; ++k) f[k] = float(rec[k]);
  }
  __device__ __forceinline__ double dbl(int) const { return epoch; }
  __device__ __forceinline__ float flt(int k) const { return f[k]; }
};
static_assert(sizeof(LdsSat<double, float>) == 13 * 16 && sizeof(LdsSat<double, double>) == 19 * 16 &&
                  sizeof(LdsSat<float, float>) == 11 * 16,
              "odd multiples of 16 bytes");
static_assert(kX7 == kC41 + 2, "three unfolded functions");
#define SGP4MI_LDS_REC(TS, TP)                                                                                 \
  template <> __device__ __forceinline__ double rec_val<double, const LdsSat<TS, TP>*>(const LdsSat<TS, TP>* s, int k) { \
    return s->dbl(k);                                                                                          \
  }                                                                                                            \
  template <> __device__ __forceinline__ float rec_val<float, const LdsSat<TS, TP>*>(const LdsSat<TS, TP>* s, int k) {   \
    return s->flt(k);                                                                                          \
  }
SGP4MI_LDS_REC(double, float)
SGP4MI_LDS_REC(double, double)
SGP4MI_LDS_REC(float, float)
#undef SGP4MI_LDS_REC

// The kernel's arguments as a function of its own reads them: through the
// segment they are passed in (as references they would go to the stack).
template <class TP, bool kOff32>
struct FusedCall {
  FusedArgs a;  // first
  Out<TP, kOff32> out;
};
typedef const __attribute__((address_space(4))) uint32_t* KernArgs;
template <class T>
__device__ __forceinline__ T kernel_arguments(KernArgs p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);  // the same in every lane
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v)), hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
  p = reinterpret_cast<KernArgs>(uint64_t(hi) << 32 | lo);
  static_assert(sizeof(T) % 4 == 0 && alignof(T) <= 8, "whole words at the segment's start");
  uint32_t w[sizeof(T) / 4];
#pragma unroll
  for (size_t k = 0; k < sizeof(T) / 4; ++k) w[k] = p[k];
  T t;
  __builtin_memcpy(&t, w, sizeof t);
  return t;
}

// A deep-space member's constants and terms, as all of its points read them.
struct LdsDeep {
  static constexpr int kFew = 5;
  double d[kEpochMin + 1], few[kFew], deep[kNDeep];  // few: kI0, kC1, kBC4, kA0pp, kE0
  uint32_t info;
  int32_t sat;  // of the workgroup
  __device__ __forceinline__ void put(const double* rec) {
#pragma unroll
    for (int k = 0; k <= kEpochMin; ++k) d[k] = rec[k];
    few[0] = rec[kI0]; few[1] = rec[kC1]; few[2] = rec[kBC4]; few[3] = rec[kA0pp]; few[4] = rec[kE0];
  }
  // what deep_point reads
  template <class TS, class TP>
  __device__ __forceinline__ SatC<TS, TP> sat_c() const {
    SatC<TS, TP> c;
    c.M0 = TS(d[kM0]); c.Mdot = TS(d[kMdot]); c.argp0 = TS(d[kArgp0]); c.argpdot = TS(d[kArgpdot]);
    c.node0 = TS(d[kNode0]); c.nodedot = TS(d[kNodedot]); c.nodecf = TS(d[kNodecf]); c.t2cof = TS(d[kT2cof]);
    c.n0pp = TS(d[kN0pp]); c.epoch_min = d[kEpochMin];
    c.i0 = TP(few[0]); c.C1 = TS(few[1]); c.bC4 = TS(few[2]); c.a0pp = TS(few[3]); c.e0 = TS(few[4]);
    c.info = info;
    c.deep = deep;
    return c;
  }
};

// A deep-space member's initialisation into LDS, and one of its points.  Functions
// of their own, without loops around them: the near-Earth loop does not share its
// registers with the terms (inlined, 300,007 x 19 mixed without a deep-space member
// took 58 us, 50 so), and no loop carries the hundred or so constants of their
// series in scalar registers (one function with both loops: 278 us instead of 153 at
// 100,000 deep-space satellites x 32 FP64).
typedef __attribute__((address_space(3))) LdsDeep* LDeep;
static __device__ __attribute__((noinline)) void fused_deep_init(KernArgs args, int64_t i, int32_t sat, LDeep to) {
  const FusedArgs a = kernel_arguments<FusedArgs>(args);
  LdsDeep& d = *(LdsDeep*)to;
  double rec[kNRec], el[7], epoch;
  const uint32_t info = init_sat(a, i, rec, el, &epoch, false);
  d.info = info;
  d.sat = sat;
  d.put(rec);
  init_deep(el, rec, a.grav.ke, a.ref_day + epoch, d.deep, false);
  put_flags(a, i, info, d.deep[kDRes] != 0.0);
}
template <class TS, class TP, bool kOff32>
__device__ __attribute__((noinline)) void fused_deep_point(KernArgs args, int64_t p, double t, LDeep from) {
  const FusedCall<TP, kOff32> call = kernel_arguments<FusedCall<TP, kOff32>>(args);
  const LdsDeep& d = *(const LdsDeep*)from;
  PointState<TP> s;
  const uint32_t code = deep_point<TS, TP>(d.sat_c<TS, TP>(), grav_of(call.a), t, s);
  call.out.put(p, code, s);
}

// kFusedSats satellites, times [y per, (y + 1) per) of the list.  Bound by VALU
// issue.  One wavefront of sixteen initialising for 64 satellites, in runs of 16
// times, took 204 us at 300,007 x 19 mixed, this 51; a lane per satellite walking
// its times in registers, outputs regrouped through LDS by eight times, 107
// (pieces of cache lines); 1M x 8 FP64 240 -> 164, 300,000 x 2 mixed 32 -> 17.
// Deep-space members: every point a lane, as for the others.  100,000 of them x 32
// FP64 153 us, where walking the times on the lane that met the satellite took 1,022
// and sixteen wavefronts behind one initialising 273; 15 % of them among near-Earth
// ones 98, 793 and 230.
template <class TS, class TP, bool kOff32, int kBlock>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
    fused_kernel(FusedCall<TP, kOff32> call) {
  const FusedArgs& a = call.a;
  const Out<TP, kOff32>& out = call.out;
  // the near-Earth members' constants, then rounds of deep-space members
  extern __shared__ __align__(16) unsigned char lds[];
  LdsSat<TS, TP>* const sats = reinterpret_cast<LdsSat<TS, TP>*>(lds);
  __shared__ unsigned long long deep_lanes;
  const int64_t i0 = int64_t(blockIdx.x) * kFusedSats;
  const int32_t ns = int32_t(a.n - i0 < kFusedSats ? a.n - i0 : kFusedSats);
  const Grav g = grav_of(a);
  if (threadIdx.x < kFusedSats) {
    bool deep = false;
    if (int32_t(threadIdx.x) < ns) {
      double rec[kNRec], el[7], epoch;
      const uint32_t info = init_sat(a, i0 + threadIdx.x, rec, el, &epoch, true);
      deep = (info & kInfoDeep) != 0;
      if (!deep) {
        put_flags(a, i0 + threadIdx.x, info, false);
        sats[threadIdx.x].put(rec);
      }
      sats[threadIdx.x].info = info;
    }
    const unsigned long long m = __ballot(deep);
    if (threadIdx.x == 0) deep_lanes = m;
  }
  __syncthreads();
  const int64_t t0 = int64_t(blockIdx.y) * a.per;
  const int32_t nt = int32_t(t0 + a.per < a.T ? a.per : a.T - t0);
  const int32_t step_s = kBlock / nt, step_j = kBlock - step_s * nt;  // one pass further: satellites, times
  int32_t s = int32_t(threadIdx.x) / nt, j = int32_t(threadIdx.x) - s * nt;
  while (s < ns) {
    const LdsSat<TS, TP>* const p = &sats[s];
    asm volatile("" ::: "memory");
    SatC<TS, TP> c = load_from<TS, TP, const LdsSat<TS, TP>*, const LdsSat<TS, TP>*>(p, p);
    if (!(c.info & kInfoDeep)) {
      PointState<TP> st;
      const uint32_t code = sgp4_point<TS, TP>(c, g, a.t[t0 + j], st);
      // kOff32: every point index is below 2^30 and fits 32-bit arithmetic
      out.put(kOff32 ? int64_t(uint32_t(i0 + s) * uint32_t(a.T) + uint32_t(t0 + j)) : (i0 + s) * a.T + t0 + j, code, st);
    }
    s += step_s;
    j += step_j;
    if (j >= nt) {
      j -= nt;
      ++s;
    }
  }
  // Deep-space members, a round of as many as LDS holds at a time: the lanes that met
  // them initialise one each, then all lanes take the round's points in output order.
  const unsigned long long members = deep_lanes;
  if (members == 0) return;
  const KernArgs args = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
  const LDeep deeps = (LDeep)(LdsDeep*)lds;
  const bool mine = threadIdx.x < kFusedSats && (members >> threadIdx.x & 1ull);
  const int32_t rank = mine ? __popcll(members & ((1ull << threadIdx.x) - 1ull)) : -1;
  const int32_t nd = __popcll(members);
  for (int32_t d0 = 0; d0 < nd; d0 += a.round) {
    const int32_t m = nd - d0 < a.round ? nd - d0 : a.round;
    __syncthreads();  // the near-Earth constants, the last round's
    if (rank >= d0 && rank < d0 + m)
      fused_deep_init(args, i0 + threadIdx.x, threadIdx.x, deeps + (rank - d0));
    __syncthreads();
    for (int32_t q = threadIdx.x; q < m * nt; q += kBlock) {
      const int32_t e = q / nt, jd = q - e * nt;
      fused_deep_point<TS, TP, kOff32>(args, (i0 + deeps[e].sat) * a.T + t0 + jd, a.t[t0 + jd], deeps + e);
    }
  }
}

template <class TP>
static bool fused_fits32(int64_t P) {
  return P >= 0 && uint64_t(P) * sizeof(TP) < (uint64_t(1) << 32);
}

template <class TS, class TP, bool kOff32>
static void fused_go(const FusedArgs& a, void* r, void* v, uint8_t* err, hipStream_t s) {
  const int64_t P = a.n * a.T;
  Out<TP, kOff32> o{static_cast<TP*>(r), static_cast<TP*>(v), err, P};
  if (a.T == 1) {
    hipLaunchKernelGGL((fused_one_kernel<TS, TP, kOff32>), dim3(unsigned((a.n + 63) / 64)), dim3(64), 0, s, a, o);
    return;
  }
  const dim3 grid(unsigned((a.n + kFusedSats - 1) / kFusedSats), unsigned((a.T + a.per - 1) / a.per));
  // LDS for all members' deep-space terms where that leaves as many workgroups on
  // a compute unit: four of 256 lanes (sixteen wavefronts, as many as their
  // registers allow), or grids of up to four workgroups each; else an eighth of
  // the unit's
  const bool wide = a.per > kFusedNarrow || (a.per >= 4 && int64_t(grid.x) * grid.y <= 512);
  FusedArgs b = a;
  b.round = wide || int64_t(grid.x) * grid.y <= 1024 ? kFusedSats : kFusedLdsNarrow / int32_t(sizeof(LdsDeep));
  const size_t lds = std::max(sizeof(LdsDeep) * size_t(b.round), sizeof(LdsSat<TS, TP>) * kFusedSats);
  static_assert(sizeof(LdsDeep) * kFusedSats <= 40000 && sizeof(LdsSat<TS, TP>) * kFusedSats <= kFusedLdsNarrow,
                "four and eight workgroups on a compute unit");
  if (wide)
    hipLaunchKernelGGL((fused_kernel<TS, TP, kOff32, 256>), grid, dim3(256), lds, s, FusedCall<TP, kOff32>{b, o});
  else
    hipLaunchKernelGGL((fused_kernel<TS, TP, kOff32, 128>), grid, dim3(128), lds, s, FusedCall<TP, kOff32>{b, o});
}

template <class TS, class TP>
static void fused_t(const FusedArgs& a, void* r, void* v, uint8_t* err, hipStream_t s) {
  if (fused_fits32<TP>(a.n * a.T)) fused_go<TS, TP, true>(a, r, v, err, s);
  else fused_go<TS, TP, false>(a, r, v, err, s);
}

// Largest T and n of a fused launch, as the interface states them: 65,535 runs of 16
// times, and 2^32 lanes at 64 per satellite group and run time (the grid itself is
// smaller: at most 512 groups of times in y).
constexpr int64_t kFusedRun = 16;
int64_t fused_max_T() { return 65535 * kFusedRun; }
bool fused_fits(int64_t n, int64_t T) {
  return grid_fits(uint64_t((n + 63) / 64), 64 * uint64_t(std::max<int64_t>(1, std::min(T, kFusedRun))));
}

hipError_t launch_fused(int precision, const double g[5], double ref_day, int64_t n, const double* elem,
                        const double* t, int64_t T, void* r, void* v, uint8_t* err, uint8_t* user_flags,
                        hipStream_t s) {
  FusedArgs a;
  a.n = n;
  a.T = T;
  a.elem = elem;
  a.t = t;
  a.user_flags = user_flags;
  a.grav = grav_in(g);
  a.vkms = a.grav.radius * a.grav.ke / 60.0;
  a.ref_day = ref_day;
  // Two workgroups per CU, as far as there are times: every further split of the
  // times initialises the satellites once more (60,000 x 4 FP64: 17.4 us at four
  // per CU, 15.7 at two; 20,000 x 64 30 us at two, 38 at one).
  const int64_t wgs = (n + kFusedSats - 1) / kFusedSats, groups = std::min<int64_t>(T, (512 + wgs - 1) / wgs);
  a.per = (T + groups - 1) / groups;
  switch (precision) {
    case 0: fused_t<double, double>(a, r, v, err, s); break;
    case 1: fused_t<float, float>(a, r, v, err, s); break;
    case 2: fused_t<double, float>(a, r, v, err, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace sgp4mi
