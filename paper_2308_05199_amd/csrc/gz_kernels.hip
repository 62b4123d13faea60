// gz_kernels.hip -- gfx950 kernels of the GZ1 codec.
//
// Layout of the work: a lane owns a 32-element segment (L/32 consecutive
// lanes own one block), a workgroup of TPB lanes owns a strip of TPB*32
// elements (a whole number of 4096-element superblocks).  Workgroups are
// persistent: they take strips in ticket order, so every strip a strip waits
// for is already running.  Strip payload offsets come from one decoupled
// look-back pass over agent-scope status words (a single read of the input,
// a single write of the output), tagged with a launch epoch so they never
// need clearing.  No MFMA: the path is bound by HBM, not by arithmetic.
// Short streams, fp64, tiles, most batches and short fused steps are encoded by
// units (2048 elements, a wave each, section "unit encode"), long fused steps by
// waves that code superblocks, and most of the decoding runs by waves that need
// no scan.  Strips serve long fp32 compressions, the explicit thread counts, the
// tuner, decode-and-accumulate and fp32 scatter compression.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "gz_common.h"
#include "gz_kernels.h"
#include "gz_ring.h"

namespace gzk {

// ------------------------------------------------------------------ utils
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr uint32_t SPIN_LIMIT = 1u << 22;
constexpr uint64_t VMASK = (1ull << 34) - 1;

// Look-back words and control counters are read and written at system
// scope (sc0 sc1): such accesses are not served from an XCD's own L2, so a
// word published by a workgroup on another XCD is seen on the next poll.
__device__ __forceinline__ void st_agent(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint32_t ld_agent32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint64_t sw_pack(uint64_t flag, uint32_t ep, uint64_t v) {
  return (flag << 62) | ((uint64_t)(ep & 0x0FFFFFFFu) << 34) | (v & VMASK);
}

// Cross-lane moves by DPP: VALU operations, where __shfl goes through the LDS
// crossbar (its latency, six times in series for a scan, sat on every
// superblock's critical path: 1 GiB compression 409 -> 396 us, decompression
// 272 -> 267 us, a mixed batch of 512 requests 319 -> 299 us, a single fused
// step of 2 M elements 24.0 -> 22.7 us).  Lanes without a source read 0.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E;     // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int DPP_SHR = 0x110;                      // row_shr:n is DPP_SHR + n
constexpr int DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;

// The value of the lane below (the lanes of a block, tile or group of up to
// 16 lanes that starts on a multiple of its size; a row's first lane reads 0).
__device__ __forceinline__ uint32_t lane_below(uint32_t v) { return dpp<DPP_SHR + 1>(v); }

__device__ __forceinline__ uint32_t read_lane(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp<DPP_SHR + 1>(v);
  v += dpp<DPP_SHR + 2>(v);
  v += dpp<DPP_SHR + 4>(v);
  v += dpp<DPP_SHR + 8>(v);
  v += dpp<DPP_BCAST15, 0xA>(v);
  v += dpp<DPP_BCAST31, 0xC>(v);
  return v;
}

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long v) {
  return ((unsigned long long)dpp<CTRL, ROWS>((uint32_t)(v >> 32)) << 32) |
         dpp<CTRL, ROWS>((uint32_t)v);
}

// Sum over the wave (every lane active), the same in every lane.
__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
  v += dpp64<DPP_SHR + 1>(v);
  v += dpp64<DPP_SHR + 2>(v);
  v += dpp64<DPP_SHR + 4>(v);
  v += dpp64<DPP_SHR + 8>(v);
  v += dpp64<DPP_BCAST15, 0xA>(v);
  v += dpp64<DPP_BCAST31, 0xC>(v);
  return ((unsigned long long)read_lane((uint32_t)(v >> 32), 63) << 32) |
         read_lane((uint32_t)v, 63);
}

// OR / carry over the LPB lanes that own one block.
template <int LPB>
__device__ __forceinline__ uint32_t grp_or(uint32_t v) {
  if (LPB >= 2) v |= dpp<DPP_XOR1>(v);
  if (LPB >= 4) v |= dpp<DPP_XOR2>(v);
  return v;
}

template <int LPB>
__device__ __forceinline__ uint32_t grp_excl_sum(uint32_t v, uint32_t w) {
  uint32_t incl = v;
  if (LPB >= 2) {
    const uint32_t t = dpp<DPP_SHR + 1>(incl);
    if (w >= 1) incl += t;
  }
  if (LPB >= 4) {
    const uint32_t t = dpp<DPP_SHR + 2>(incl);
    if (w >= 2) incl += t;
  }
  return incl - v;
}

// ----------------------------------------------------------- quantisation
// fp32: r = x/t is formed as fl32((double)x * (1/(double)t)).  The double
// product is within 2^-52 (relative) of x/t, while x/t never lies within
// 2^-49 of a float rounding boundary in the normal range (x, t have 24-bit
// significands and a boundary needs 25), so the rounding to float equals
// the IEEE quotient; below the normal range both give q = 0.  x - xh is
// exact (Sterbenz), so |x - xh| <= eb is tested in float against the largest
// float not above eb.
// Saturating conversions (the hardware instructions are defined for every
// input; the C++ casts are not).
__device__ __forceinline__ int32_t cvt_sat(float f) {
  int32_t r;
  asm("v_cvt_i32_f32 %0, %1" : "=v"(r) : "v"(f));
  return r;
}
__device__ __forceinline__ int32_t cvt_sat(double f) {
  int32_t r;
  asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(f));
  return r;
}

// FAIL over a run of elements.  fp32: the largest |rr| and |x - xh| seen, with
// NaN kept (v_maximum3_f32 takes two elements an instruction), tested once at
// the end; a compare per condition and element would issue two compares and
// two or three scalar mask operations instead of one instruction.  fp64 has no
// such maximum and keeps the compares.
template <typename T>
struct QBad;
template <>
struct QBad<float> {
  float r = 0.0f, d = 0.0f;
  // |rr| < 2^29 exactly when |r| < 2^29 (floats from 2^23 up are integers,
  // which rint leaves alone; below, both hold)
  __device__ __forceinline__ bool any(float eblo) const {
    return !(r < 536870912.0f) || !(d <= eblo);
  }
};
template <>
struct QBad<double> {
  bool bad = false;
  __device__ __forceinline__ bool any(double) const { return bad; }
};

// When |r| < 2^29 the rounded value rr is an integer held exactly, so
// (T)q == rr and xh is formed from rr directly.
__device__ __forceinline__ int32_t quant(float x, double rinv, float t, QBad<float>& b) {
  const float r = (float)((double)x * rinv);
  const float rr = __builtin_rintf(r);
  const float d = x - rr * t;
  b.r = __builtin_elementwise_maximum(b.r, fabsf(rr));
  b.d = __builtin_elementwise_maximum(b.d, fabsf(d));
  return cvt_sat(rr);
}

// fp64: r = x/t correctly rounded.  With y = 1/t correctly rounded (rinv), q0
// = x y is within 2 ulp of x/t; one correction with the remainder brings it
// within 1 ulp, and a second one from there gives the correctly rounded
// quotient (Markstein: y correctly rounded, q faithful, remainder exact).
// The host sets rinv only for steps t in [2^-900, 2^900]: then remainders of
// quotients of 2^-2 and more are normal, smaller quotients round to q = 0
// whatever their last bits, and overflowing ones end as NaN or infinity, which
// fail.  For other steps x and t are scaled by 2^600 or 2^-600 first (exactly, or
// to an infinity whose quotient fails, or below a quotient of 2^-1000), or
// divided.
__device__ __forceinline__ double quot(double x, double t, double y) {
  const double q0 = x * y;
  const double q1 = __builtin_fma(__builtin_fma(-q0, t, x), y, q0);
  return __builtin_fma(__builtin_fma(-q1, t, x), y, q1);
}

__device__ __forceinline__ int32_t quant(double x, double r, double t, double eb,
                                         QBad<double>& b) {
  double rr = __builtin_rint(r);
  bool inr = fabs(r) <= 536870911.0;
  int32_t q = cvt_sat(rr);
  double d = x - rr * t;
  b.bad |= !inr || !(fabs(d) <= eb);
  return q;
}

// Quantises v[0..N) into q (!FULL: elements past vcnt give 0 and never fail).
template <int N, bool FULL>
__device__ __forceinline__ void quant_run(const float* v, const Job& J, uint32_t vcnt, uint32_t* q,
                                          QBad<float>& b) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float x = FULL || i < (int)vcnt ? v[i] : 0.0f;
    q[i] = (uint32_t)quant(x, J.rinv, J.t32, b);
    // four elements at a time: interleaving more of them costs registers
    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  }
}
template <int N, bool FULL>
__device__ __forceinline__ void quant_run(const double* v, const Job& J, uint32_t vcnt,
                                          uint32_t* q, QBad<double>& b) {
  if (J.rinv != 0.0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double x = FULL || i < (int)vcnt ? v[i] : 0.0;
      q[i] = (uint32_t)quant(x, quot(x, J.t64, J.rinv), J.t64, J.eb, b);
    }
  } else if constexpr (N == 32) {
    // strips: steps out of the reciprocal's range, brought into it by a power of
    // two (2^24 values with 256 threads: 140 us by a rolled loop of divisions,
    // 73.5 so)
    const double s = J.t64 < 1.0 ? 0x1p600 : 0x1p-600, ts = J.t64 * s, y = 1.0 / ts;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double x = FULL || i < (int)vcnt ? v[i] : 0.0;
      q[i] = (uint32_t)quant(x, quot(x * s, ts, y), J.t64, J.eb, b);
    }
  } else {
    // units, short of registers (unrolled, mixed batches lost 5%, 132 -> 136 us)
#pragma unroll 1
    for (int i = 0; i < N; ++i) {
      // (a rolled loop over registers would put them in memory)
      double x = 0.0;
#pragma unroll
      for (int k = 0; k < N; ++k) x = k == i && (FULL || k < (int)vcnt) ? v[k] : x;
      const uint32_t z = (uint32_t)quant(x, x / J.t64, J.t64, J.eb, b);
#pragma unroll
      for (int k = 0; k < N; ++k) q[k] = k == i ? z : q[k];
    }
  }
}
template <typename T>
__device__ __forceinline__ T bad_bound(const Job& J);
template <>
__device__ __forceinline__ float bad_bound<float>(const Job& J) { return J.eblo; }
template <>
__device__ __forceinline__ double bad_bound<double>(const Job& J) { return J.eb; }

// bits of element i as u32 words (1 for float, 2 for double)
__device__ __forceinline__ void raw_words(float v, uint32_t* dst) {
  dst[0] = __float_as_uint(v);
}
__device__ __forceinline__ void raw_words(double v, uint32_t* dst) {
  unsigned long long b = (unsigned long long)__double_as_longlong(v);
  dst[0] = (uint32_t)b;
  dst[1] = (uint32_t)(b >> 32);
}
__device__ __forceinline__ float from_raw(const uint32_t* src, float) {
  return __uint_as_float(src[0]);
}
__device__ __forceinline__ double from_raw(const uint32_t* src, double) {
  unsigned long long b = (unsigned long long)src[0] | ((unsigned long long)src[1] << 32);
  return __longlong_as_double((long long)b);
}

// ------------------------------------------------------------- LDS state
struct Smem {
  uint32_t cur;                  // strip being processed
  uint32_t epoch;
  uint32_t tp_key;               // decode: 1 + ticket whose table words follow
  uint32_t tp_t0, tp_t1;
  uint32_t flag;                 // strip error flags
  uint32_t hdr_ok;
  uint32_t hdr_job;              // 1 + job whose stream header was checked
  uint32_t wtot[MAX_TPB / 64];
  unsigned long long excl;       // strip exclusive prefix (dwords, chain-wide)
  unsigned long long pj;         // chain prefix at the job's first strip
  unsigned long long paydw;      // decode: payload size of the incoming stream (dwords)
  float t32;                     // decode: step of the incoming stream
  double t64;
  uint32_t hb[MAX_TPB / 4];      // header bytes of the strip's blocks
  uint32_t wts[192];             // selector weights (tile mode)
};

// Staging buffer for one strip's payload (dynamic LDS): 16 bytes of headroom
// for realigning the copy-in, TPB*32*sizeof(T) bytes, 16 bytes of tail.
extern __shared__ __attribute__((aligned(16))) uint32_t g_stage[];

__device__ __forceinline__ uint32_t first_ticket(const Ctl& C, Smem& sm) {
  if (threadIdx.x == 0) {
    sm.epoch = ld_agent32(&C.ctrl->epoch);
    sm.hdr_job = 0;
    sm.tp_key = 0;
    sm.cur = atomicAdd(&C.ctrl->ticket, 1u);
  }
  __syncthreads();
  return sm.cur;
}

__device__ __forceinline__ void epilogue(const Ctl& C) {
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t d = atomicAdd(&C.ctrl->done, 1u);
    if (d == gridDim.x - 1) {  // last workgroup: reset for the next launch
      atomicExch(&C.ctrl->ticket, 0u);
      atomicExch(&C.ctrl->done, 0u);
      atomicAdd(&C.ctrl->epoch, 1u);
    }
  }
}

__device__ __forceinline__ bool aborted(const Ctl& C) {
  return (ld_agent32(&C.ctrl->err) & ERRF_TIMEOUT) != 0;
}

// Bound of every inter-workgroup wait: C.wait_ticks of the constant-rate
// clock from the 64th unsuccessful poll (or SPIN_LIMIT polls), or another
// workgroup's timeout.  Checked every 64 polls; the clock (a scalar memory
// read) is not touched by waits that end within the first 63 polls.
__device__ __forceinline__ bool wait_over(const Ctl& C, uint32_t spins, uint64_t& t0) {
  if ((spins & 63u) != 0) return false;
  if (spins == 64) {
    t0 = (uint64_t)wall_clock64();
    return false;
  }
  return spins > SPIN_LIMIT || (uint64_t)wall_clock64() - t0 > C.wait_ticks || aborted(C);
}

// Publishes the strip aggregate (or, at the head of a chain, its prefix).
__device__ __forceinline__ void publish_agg(const Ctl& C, uint64_t gs, uint64_t chain0,
                                            uint32_t ep, uint64_t agg) {
  st_agent(C.status + gs, sw_pack(gs == chain0 ? 2 : 1, ep, agg));
}

// Decoupled look-back run by one wave after publish_agg: returns the
// exclusive prefix (dwords) of strip gs within its chain and publishes its
// inclusive prefix.  One probe reads SUB x 64 predecessors (SUB independent
// loads per lane); sub-windows resolved before a not-yet-published word are
// added in before the probe is retried from there.  Strips and units probe 256 words;
// the per-wave fused kernel, with more and smaller chain elements, probes 64
// (its status-word reads would otherwise rival its payload traffic).
constexpr int LB_SUB = 4;

template <int SUB = LB_SUB, bool PUBLISH = true>
__device__ uint64_t lookback(const Ctl& C, uint64_t gs, uint64_t chain0, uint32_t ep,
                             uint64_t agg, bool& timeout) {
  const int lane = __lane_id();
  if (gs == chain0) return 0;
  uint64_t excl = 0;
  int64_t top = (int64_t)gs - 1;
  uint32_t spins = 0;
  uint64_t t0 = 0;
  for (;;) {
    uint32_t flag[SUB];
    uint64_t val[SUB];
    // every load is issued before any is used: lanes before the chain's
    // start read its first word (a load under a divergent branch is merged
    // by register copies that wait for it at once, one round trip per load)
    uint64_t w[SUB];
#pragma unroll
    for (int m = 0; m < SUB; ++m) {
      const int64_t idx = top - 64 * m - lane;
      w[m] = ld_agent(C.status + (idx >= (int64_t)chain0 ? idx : (int64_t)chain0));
    }
#pragma unroll
    for (int m = 0; m < SUB; ++m) {
      const int64_t idx = top - 64 * m - lane;
      const bool cur = (uint32_t)((w[m] >> 34) & 0x0FFFFFFFu) == (ep & 0x0FFFFFFFu);
      const bool in_chain = idx >= (int64_t)chain0;
      flag[m] = in_chain ? (cur ? (uint32_t)(w[m] >> 62) : 0u) : 2u;
      val[m] = in_chain ? (w[m] & VMASK) : 0ull;
    }
    uint64_t part = 0;  // this lane's share of the resolved sub-windows
    int resolved = 0;   // sub-windows fully added in
    bool done = false, wait = false;
#pragma unroll
    for (int m = 0; m < SUB; ++m) {
      if (!done && !wait) {
        const uint64_t pm = __ballot(flag[m] == 2);
        const uint64_t zm = __ballot(flag[m] == 0);
        const int p = pm ? (int)__builtin_ctzll(pm) : 64;
        const uint64_t upto = p >= 63 ? ~0ull : ((2ull << p) - 1);
        if (zm & upto) {
          wait = true;
        } else {
          part += lane <= p ? val[m] : 0ull;
          ++resolved;
          done = p < 64;
        }
      }
    }
    excl += wave_sum64(part);
    if (done) break;
    top -= 64 * resolved;
    if (wait) {
      ++spins;
      if (wait_over(C, spins, t0)) {
        timeout = true;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  if (PUBLISH && lane == 0) st_agent(C.status + gs, sw_pack(2, ep, timeout ? 0 : excl + agg));
  return excl;
}

// Chain prefix at the first strip of job j (packed Scatter output).
__device__ uint64_t job_base_wait(const Ctl& C, uint32_t j, uint32_t ep, bool& timeout) {
  uint32_t spins = 0;
  uint64_t t0 = 0;
  for (;;) {
    uint64_t w = ld_agent(C.jobbase + j);
    if ((uint32_t)((w >> 34) & 0x0FFFFFFFu) == (ep & 0x0FFFFFFFu) && (w >> 62) == 2)
      return w & VMASK;
    ++spins;
    if (wait_over(C, spins, t0)) {
      timeout = true;
      return 0;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// Strip-level exclusive scan of per-lane sizes; returns the lane's exclusive
// prefix and the strip total.
__device__ __forceinline__ uint32_t strip_scan(uint32_t contrib, Smem& sm, uint32_t& total) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int nw = blockDim.x >> 6;
  uint32_t incl = wave_incl_scan(contrib);
  if (lane == 63) sm.wtot[wid] = incl;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int k = 0; k < nw; ++k) {
    uint32_t t = sm.wtot[k];
    pre += (k < wid) ? t : 0u;
    tot += t;
  }
  total = tot;
  return pre + incl - contrib;
}

// Magnitude plane j of a segment: bit i = bit j of a[i].
// ---- bit planes.  Plane j of a lane's 32 magnitudes a[i] is the word whose
// bit i is bit j of a[i].  Planes are moved 8 at a time: the bytes 8g..8g+7
// of eight magnitudes form an 8x8 bit matrix (one byte per element) that a
// three-stage delta swap transposes into one byte per plane.

// v_perm_b32: byte k of the result is byte sel.k of the 8-byte value
// (hi:lo); selector 0x0C yields a zero byte.
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  return __builtin_amdgcn_perm(hi, lo, sel);
}
// Selector taking byte b of x0..x3 (as lo, hi pairs (x0, x1), (x2, x3)).
__device__ __forceinline__ uint32_t sel_lo(uint32_t b) { return 0x0C0C0000u | ((4u + b) << 8) | b; }
__device__ __forceinline__ uint32_t sel_hi(uint32_t b) { return ((4u + b) << 24) | (b << 16) | 0x0C0Cu; }
// Byte b of four words, gathered into one word (x0's byte lowest).
__device__ __forceinline__ uint32_t gather4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                            uint32_t b) {
  return perm(x1, x0, sel_lo(b)) | perm(x3, x2, sel_hi(b));
}

// 8x8 bit transpose of the 64-bit value hi:lo (bit c of byte r <-> bit r of
// byte c).
__device__ __forceinline__ void tr8x8(uint32_t& lo, uint32_t& hi) {
  uint32_t t;
  t = ((lo >> 7) ^ lo) & 0x00AA00AAu;
  lo ^= t | (t << 7);
  t = ((hi >> 7) ^ hi) & 0x00AA00AAu;
  hi ^= t | (t << 7);
  t = ((lo >> 14) ^ lo) & 0x0000CCCCu;
  lo ^= t | (t << 14);
  t = ((hi >> 14) ^ hi) & 0x0000CCCCu;
  hi ^= t | (t << 14);
  const uint32_t nl = (lo & 0x0F0F0F0Fu) | ((hi << 4) & 0xF0F0F0F0u);
  const uint32_t nh = (hi & 0xF0F0F0F0u) | ((lo >> 4) & 0x0F0F0F0Fu);
  lo = nl;
  hi = nh;
}

// Writes planes 0..F-1 of a[] to dst[j * stride].
__device__ __forceinline__ void put_planes(const uint32_t (&a)[32], uint32_t F, uint32_t* dst,
                                           uint32_t stride) {
  for (uint32_t g = 0; 8 * g < F; ++g) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo[k] = gather4(a[8 * k], a[8 * k + 1], a[8 * k + 2], a[8 * k + 3], g);
      hi[k] = gather4(a[8 * k + 4], a[8 * k + 5], a[8 * k + 6], a[8 * k + 7], g);
      tr8x8(lo[k], hi[k]);
    }
    const uint32_t nj = min(F - 8 * g, 8u);
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      if (j < nj) {
        const uint32_t b = j & 3;
        const uint32_t word = j < 4 ? gather4(lo[0], lo[1], lo[2], lo[3], b)
                                    : gather4(hi[0], hi[1], hi[2], hi[3], b);
        dst[(8 * g + j) * stride] = word;
      }
    }
  }
}

// Magnitudes a[] from planes src[j * stride], j < F (planes >= F are zero).
__device__ __forceinline__ void get_planes(const uint32_t* src, uint32_t stride, uint32_t F,
                                           uint32_t (&a)[32]) {
  if (F == 0) {
#pragma unroll
    for (int i = 0; i < 32; ++i) a[i] = 0;
    return;
  }
  {  // planes 0..7 set byte 0 and clear the rest (no separate clearing pass)
    const uint32_t nj = min(F, 8u);
    uint32_t P[8];
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) P[j] = j < nj ? src[j * stride] : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t lo = gather4(P[0], P[1], P[2], P[3], (uint32_t)k);
      uint32_t hi = gather4(P[4], P[5], P[6], P[7], (uint32_t)k);
      tr8x8(lo, hi);
#pragma unroll
      for (int m = 0; m < 8; ++m) a[8 * k + m] = perm(m < 4 ? lo : hi, 0u, 0x0C0C0C04u + (m & 3));
    }
  }
  for (uint32_t g = 1; 8 * g < F; ++g) {
    const uint32_t nj = min(F - 8 * g, 8u);
    uint32_t P[8];
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) P[j] = j < nj ? src[(8 * g + j) * stride] : 0u;
    // a[8k+m] takes byte m of (lo, hi) of group k as its byte g
    uint32_t sel[4];
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b)
      sel[b] = (0x03020100u & ~(0xFFu << (8 * g))) | ((4u + b) << (8 * g));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t lo = gather4(P[0], P[1], P[2], P[3], (uint32_t)k);
      uint32_t hi = gather4(P[4], P[5], P[6], P[7], (uint32_t)k);
      tr8x8(lo, hi);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        a[8 * k + m] = perm(m < 4 ? lo : hi, a[8 * k + m], sel[m & 3]);
      }
    }
  }
}

// ---- coalesced strip transfers through LDS.  A strip's raw values sit in
// LDS segment by segment with 4 dwords of padding after each 32-element
// segment, so 16-byte global accesses stay contiguous across lanes and the
// per-lane 16-byte LDS accesses hit distinct banks.
template <typename T>
__device__ __forceinline__ constexpr uint32_t seg_stride() {
  return 32 * (sizeof(T) / 4) + 4;
}

// Loads strip values src[0 .. TPB*32) (nvalid of them valid, the rest 0)
// into the LDS segment layout.
template <typename T>
__device__ __forceinline__ void strip_to_lds(const T* __restrict__ src, uint64_t nvalid) {
  constexpr uint32_t SEGW = 32 * (sizeof(T) / 4), STR = seg_stride<T>();
  const uint32_t tid = threadIdx.x, TPB = blockDim.x;
  const uint32_t nch = TPB * SEGW / 4;  // 16-byte chunks
  const uint32_t* s32 = (const uint32_t*)src;
  const uint64_t vdw = nvalid * (sizeof(T) / 4);
  uint32_t* buf = g_stage + 4;
  for (uint32_t k0 = 0; k0 < nch; k0 += 4 * TPB) {
    u4u r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t k = k0 + u * TPB + tid;
      const uint64_t dw = 4ull * k;
      if (k < nch && dw + 4 <= vdw) {
        r[u] = *(const u4u*)(s32 + dw);
      } else {
        r[u].x = (k < nch && dw + 0 < vdw) ? s32[dw + 0] : 0u;
        r[u].y = (k < nch && dw + 1 < vdw) ? s32[dw + 1] : 0u;
        r[u].z = (k < nch && dw + 2 < vdw) ? s32[dw + 2] : 0u;
        r[u].w = 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t k = k0 + u * TPB + tid;
      if (k < nch) {
        const uint32_t dw = 4 * k;
        *(u4u*)(buf + (dw / SEGW) * STR + dw % SEGW) = r[u];
      }
    }
  }
}

// A whole input strip into the padded LDS layout with eight unconditional
// 16-byte loads in flight per lane, in straight-line code (the general copy
// above waits for every outstanding memory operation, the previous strip's
// stores included, at the top of each pass, and after each load of a
// branch that has a partial-chunk side).  Used by the fp32 encoder, whose
// registers are free at this point.
template <typename T>
__device__ __forceinline__ void strip_to_lds_whole(const T* __restrict__ src) {
  constexpr uint32_t SEGW = 32 * (sizeof(T) / 4), STR = seg_stride<T>();
  const uint32_t tid = threadIdx.x, TPB = blockDim.x;
  const uint32_t* s32 = (const uint32_t*)src;
  uint32_t* buf = g_stage + 4;
#pragma unroll
  for (uint32_t h = 0; h < SEGW / 4; h += 8) {
    u4u r[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) r[u] = *(const u4u*)(s32 + 4 * ((h + u) * TPB + tid));
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) {
      const uint32_t dw = 4 * ((h + u) * TPB + tid);
      *(u4u*)(buf + (dw / SEGW) * STR + dw % SEGW) = r[u];
    }
  }
}

// The lane index as a value the compiler cannot see through: addresses
// derived from it are formed where they are used, not hoisted out of the
// persistent loop into registers held across a whole strip.
__device__ __forceinline__ uint32_t opaque_tid() {
  uint32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Stores the LDS segment layout to dst[0 .. nvalid) with 16-byte stores.
template <typename T>
__device__ __forceinline__ void lds_to_strip(T* __restrict__ dst, uint64_t nvalid) {
  constexpr uint32_t SEGW = 32 * (sizeof(T) / 4), STR = seg_stride<T>();
  const uint32_t tid = threadIdx.x, TPB = blockDim.x;
  const uint64_t vdw = nvalid * (sizeof(T) / 4);
  const uint32_t nch = (uint32_t)min((uint64_t)TPB * SEGW / 4, (vdw + 3) / 4);
  uint32_t* d32 = (uint32_t*)dst;
  const uint32_t* buf = g_stage + 4;
  if (nvalid == (uint64_t)TPB * SEG) {  // a whole strip: 8 reads in flight, then 8 stores
    const uint32_t t = opaque_tid();
#pragma unroll
    for (uint32_t h = 0; h < SEGW / 4; h += 8) {
      u4u r[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) {
        const uint32_t dw = 4 * ((h + u) * TPB + t);
        r[u] = *(const u4u*)(buf + (dw / SEGW) * STR + dw % SEGW);
      }
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) ((u4u*)(d32 + 4ull * (h + u) * TPB))[t] = r[u];
    }
    return;
  }
  for (uint32_t k = tid; k < nch; k += TPB) {
    const uint32_t dw = 4 * k;
    const u4u r = *(const u4u*)(buf + (dw / SEGW) * STR + dw % SEGW);
    if (dw + 4 <= vdw) {
      *(u4u*)(d32 + dw) = r;
    } else {
      if (dw + 0 < vdw) d32[dw + 0] = r.x;
      if (dw + 1 < vdw) d32[dw + 1] = r.y;
      if (dw + 2 < vdw) d32[dw + 2] = r.z;
    }
  }
}

// The lane's own segment in the LDS layout.
template <typename T>
__device__ __forceinline__ void lane_from_lds(T (&v)[32]);
template <>
__device__ __forceinline__ void lane_from_lds<float>(float (&v)[32]) {
  const f4u* p = (const f4u*)(g_stage + 4 + threadIdx.x * seg_stride<float>());
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const f4u r = p[k];
    v[4 * k] = r.x; v[4 * k + 1] = r.y; v[4 * k + 2] = r.z; v[4 * k + 3] = r.w;
  }
}
template <>
__device__ __forceinline__ void lane_from_lds<double>(double (&v)[32]) {
  const d2u* p = (const d2u*)(g_stage + 4 + threadIdx.x * seg_stride<double>());
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const d2u r = p[k];
    v[2 * k] = r.x; v[2 * k + 1] = r.y;
  }
}
template <typename T>
__device__ __forceinline__ void lane_to_lds(const T (&v)[32]);
template <>
__device__ __forceinline__ void lane_to_lds<float>(const float (&v)[32]) {
  f4u* p = (f4u*)(g_stage + 4 + threadIdx.x * seg_stride<float>());
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    f4u r;
    r.x = v[4 * k]; r.y = v[4 * k + 1]; r.z = v[4 * k + 2]; r.w = v[4 * k + 3];
    p[k] = r;
  }
}
template <>
__device__ __forceinline__ void lane_to_lds<double>(const double (&v)[32]) {
  d2u* p = (d2u*)(g_stage + 4 + threadIdx.x * seg_stride<double>());
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    d2u r;
    r.x = v[2 * k]; r.y = v[2 * k + 1];
    p[k] = r;
  }
}

// Where the lane's block sits in the incoming payload (dwords from the
// payload start) and how it is coded; lets the fused step re-read a block.
struct DecInfo {
  uint32_t off_dw, kind, F;
};

// Rebuilds the lane's 32 values from its block's words at pw (LDS or global).
template <typename T, int LPB, bool FULL>
__device__ __forceinline__ void unpack_seg(const uint32_t* pw, uint32_t kind, uint32_t F,
                                           uint32_t w, uint32_t vcnt, bool exists, T t,
                                           T (&v)[32]) {
  constexpr uint32_t EW = sizeof(T) / 4;
  if (kind == K_RAW) {
#pragma unroll
    for (int i = 0; i < 32; ++i)
      v[i] = (FULL || i < (int)vcnt) ? from_raw(pw + (w * 32 + i) * EW, T()) : (T)0;
    return;
  }
  // L1D; a ZERO block (or a lane past the end) is an L1D block with base 0
  // and no planes, which decodes to +0 without a separate clearing pass
  const bool z = kind == K_ZERO || !exists;
  const int32_t base = z ? 0 : (int32_t)pw[0];
  const uint32_t Fz = z ? 0u : F;
  uint32_t a[32];
  get_planes(pw + 1 + LPB + w, LPB, Fz, a);
  const uint32_t sg = Fz ? pw[1 + w] : 0u;
  uint32_t acc = 0;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int32_t)sg, i, 1);  // 0 or ~0
    uint32_t d = (a[i] ^ neg) - neg;
    if (i == 0 && w == 0) d = 0;
    acc += d;
    a[i] = acc;  // local prefix
  }
  const uint32_t carry = grp_excl_sum<LPB>(acc, w) + (uint32_t)base;
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = (T)(int32_t)(carry + a[i]) * t;
}

// --------------------------------------------------------------- encode
// Per-lane result of analysing a segment: the block's kind, width and size
// (identical on the LPB lanes of a block) and this lane's share of the
// payload (base, sign word, residual magnitudes).
struct LaneCode {
  uint32_t a[32];   // |d| of the lane's 32 elements (rawregs: their fp32 bits)
  uint32_t rawregs; // RAW block whose fp32 values sit in a[]
  uint32_t sg;      // sign bits
  int32_t base;     // q of the block's first element (lane w == 0)
  uint32_t kind, F, size_dw;
  bool exists;
};

// Mode 0: 1D blocks of L consecutive elements, L1D prediction, from the
// quantised values in lc.a (bad: one of the lane's failed).  KEEP (fp32
// fused step): a block whose quantisation fails puts its values' bits in a[]
// for the RAW payload, from the lane's LDS segment, where the fused step
// stored them (they are not in global memory); keep_row: that segment, if
// not the strip layout's.
template <uint32_t EW, int L, bool FULL, bool KEEP = false>
__device__ __forceinline__ void analyze_q(const Job& J, uint64_t seg, uint32_t w, bool bad,
                                          uint32_t vcnt, LaneCode& lc,
                                          const uint32_t* keep_row = nullptr) {
  constexpr int LPB = L / 32;
  const uint64_t b = seg / LPB;
  uint32_t (&a)[32] = lc.a;
  const int32_t base = (int32_t)a[0];
  const int32_t prev = (int32_t)lane_below(a[31]);
  const uint32_t badb = grp_or<LPB>(bad ? 1u : 0u);
  const bool rawregs = KEEP && EW == 1 && badb;
  uint32_t sg = 0, orv = 0;
  if (rawregs) {
    // a RAW block stores the values themselves: the fused step left them in
    // the lane's own LDS segment (so v[] need not outlive the quantisation)
    float u[32];
    if (keep_row) {
      const f4u* p = (const f4u*)keep_row;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const f4u r = p[k];
        u[4 * k] = r.x; u[4 * k + 1] = r.y; u[4 * k + 2] = r.z; u[4 * k + 3] = r.w;
      }
    } else {
      lane_from_lds<float>(u);
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) a[i] = (FULL || i < (int)vcnt) ? __float_as_uint(u[i]) : 0u;
  } else {
    // residual magnitudes in place (downwards, so a[i-1] still holds q)
#pragma unroll
    for (int i = 31; i >= 0; --i) {
      const int32_t pq = i ? (int32_t)a[i - 1] : prev;
      int32_t d = (int32_t)(a[i] - (uint32_t)pq);
      if (i == 0 && w == 0) d = 0;
      if (!FULL && i >= (int)vcnt) d = 0;
      const uint32_t ad = (uint32_t)(d < 0 ? -d : d);
      a[i] = ad;
      orv |= ad;
      sg = __builtin_amdgcn_alignbit(sg, (uint32_t)d, 31);
    }
  }
  const uint32_t nzb = grp_or<LPB>((base != 0 ? 1u : 0u) | orv);
  orv = grp_or<LPB>(orv);

  const bool exists = FULL || b < J.B;
  const uint32_t m = FULL ? (uint32_t)L
                          : (exists ? (uint32_t)min((uint64_t)L, J.n - b * (uint64_t)L) : 0u);
  uint32_t F = orv ? 32u - (uint32_t)__clz(orv) : 0u;
  uint32_t kind, size_dw;
  const uint32_t raw_dw = m * EW;
  if (!exists) {
    kind = K_ZERO; size_dw = 0; F = 0;
  } else if (badb) {
    kind = K_RAW; size_dw = raw_dw; F = 0;
  } else if (!nzb) {
    kind = K_ZERO; size_dw = 0; F = 0;
  } else {
    kind = K_L1D;
    size_dw = 1u + (F ? (F + 1u) * LPB : 0u);
    if (size_dw > raw_dw) { kind = K_RAW; size_dw = raw_dw; F = 0; }
  }
  lc.rawregs = (exists && rawregs) ? 1u : 0u;
  lc.sg = sg;
  lc.base = base;
  lc.kind = kind;
  lc.F = F;
  lc.size_dw = size_dw;
  lc.exists = exists;
}

// The same from the lane's values v.
template <typename T, int L, bool FULL, bool KEEP = false>
__device__ __forceinline__ void analyze_1d(const Job& J, uint64_t seg, uint32_t w,
                                           const T (&v)[32], uint32_t vcnt, LaneCode& lc,
                                           const uint32_t* keep_row = nullptr) {
  QBad<T> qb;
  quant_run<32, FULL>(v, J, vcnt, lc.a, qb);
  analyze_q<sizeof(T) / 4, L, FULL, KEEP>(J, seg, w, qb.any(bad_bound<T>(J)), vcnt, lc, keep_row);
}

// ---- mode 1: 8x8 tiles, two lanes per tile (lane w owns rows 4w..4w+3).
__device__ __forceinline__ uint32_t bitlen(int32_t v) {
  const uint32_t a = (uint32_t)(v < 0 ? -v : v);
  return a ? 32u - (uint32_t)__clz(a) : 0u;
}

// Tile features (16 int8 bit lengths of sampled values and residuals) as
// four packed words, identical on both lanes of the tile.
__device__ __forceinline__ void tile_features(const int32_t (&q)[32], uint32_t w,
                                              uint32_t (&f)[4]) {
  // each lane computes 8 features in pairs (g0: f0 f1 | f2 f3, g1: f4 f5 |
  // f6 f7, g2: f8 f9 | f10 f11, g3: f12 f13 | f14 f15)
  uint32_t p0, p1, p2, p3;
  if (w == 0) {  // rows 0..3
    p0 = bitlen(q[0]) | bitlen(q[21]) << 8;
    p1 = bitlen(q[9] - q[8]) | bitlen(q[30] - q[29]) << 8;
    p2 = bitlen(q[11] - q[3]) | bitlen(q[25] - q[17]) << 8;
    p3 = bitlen(q[13] - q[12] - q[5] + q[4]) | bitlen(q[18] - q[17] - q[10] + q[9]) << 8;
  } else {       // rows 4..7
    p0 = bitlen(q[10]) | bitlen(q[31]) << 8;
    p1 = bitlen(q[3] - q[2]) | bitlen(q[23] - q[22]) << 8;
    p2 = bitlen(q[14] - q[6]) | bitlen(q[28] - q[20]) << 8;
    p3 = bitlen(q[13] - q[12] - q[5] + q[4]) | bitlen(q[17] - q[16] - q[9] + q[8]) << 8;
  }
  const uint32_t x0 = p0 | p1 << 16, x1 = p2 | p3 << 16;
  const uint32_t y0 = dpp<DPP_XOR1>(x0), y1 = dpp<DPP_XOR1>(x1);
  const uint32_t l0 = w ? y0 : x0, l1 = w ? y1 : x1;  // lane 0's pairs
  const uint32_t h0 = w ? x0 : y0, h1 = w ? x1 : y1;  // lane 1's pairs
  f[0] = (l0 & 0xFFFFu) | (h0 << 16);
  f[1] = (l0 >> 16) | (h0 & 0xFFFF0000u);
  f[2] = (l1 & 0xFFFFu) | (h1 << 16);
  f[3] = (l1 >> 16) | (h1 & 0xFFFF0000u);
}

// int8 MLP 16 -> 32 -> 3 on the tile's features; the two lanes of a tile
// each evaluate 16 hidden units.  Weights come from LDS (blob layout).
// Returns 0 NONE, 1 L1D, 2 L2D (argmax, lowest index on ties).
__device__ __forceinline__ uint32_t mlp_choose(const uint32_t (&f)[4], uint32_t w,
                                               const uint32_t* wts) {
  const int s = (int)wts[1];
  const int32_t rnd = s ? (1 << (s - 1)) : 0;
  const uint32_t* W1 = wts + 2;           // 32 rows x 4 words
  const int32_t* b1 = (const int32_t*)(wts + 2 + 128);
  const uint32_t* W2 = wts + 2 + 128 + 32;  // 3 rows x 8 words
  const int32_t* b2 = (const int32_t*)(wts + 2 + 128 + 32 + 24);
  uint32_t hp[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    uint32_t packed = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = 16 * (int)w + 4 * g + u;
      int32_t acc = b1[k];
      acc = __builtin_amdgcn_sdot4((int)W1[4 * k + 0], (int)f[0], acc, false);
      acc = __builtin_amdgcn_sdot4((int)W1[4 * k + 1], (int)f[1], acc, false);
      acc = __builtin_amdgcn_sdot4((int)W1[4 * k + 2], (int)f[2], acc, false);
      acc = __builtin_amdgcn_sdot4((int)W1[4 * k + 3], (int)f[3], acc, false);
      int32_t h = (acc + rnd) >> s;
      h = h < 0 ? 0 : (h > 127 ? 127 : h);
      packed |= (uint32_t)h << (8 * u);
    }
    hp[g] = packed;
  }
  int32_t lg[3];
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    int32_t acc = 0;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      acc = __builtin_amdgcn_sdot4((int)W2[8 * o + 4 * w + g], (int)hp[g], acc, false);
    lg[o] = acc + (int32_t)dpp<DPP_XOR1>((uint32_t)acc) + b2[o];
  }
  uint32_t best = 0;
  int32_t bv = lg[0];
  if (lg[1] > bv) { best = 1; bv = lg[1]; }
  if (lg[2] > bv) { best = 2; }
  return best;
}

// Residual of element i of the lane for predictor k (0 NONE, 1 L1D, 2 L2D).
// up[c] is q of the row above the lane's first row (lane 1 only).
template <int K>
__device__ __forceinline__ int32_t tile_res(const int32_t (&q)[32], const int32_t (&up)[8],
                                            uint32_t w, int i) {
  const int r = i / 8, c = i % 8;
  const int32_t x = q[i];
  if (K == 0) return x;
  const bool top = (r == 0 && w == 0);  // first row of the tile
  const int32_t left = c ? q[i - 1] : 0;
  const int32_t above = r ? q[i - 8] : up[c];
  if (K == 1) {
    if (c) return (int32_t)((uint32_t)x - (uint32_t)left);
    return top ? 0 : (int32_t)((uint32_t)x - (uint32_t)above);
  }
  if (top) return c ? (int32_t)((uint32_t)x - (uint32_t)left) : 0;
  if (!c) return (int32_t)((uint32_t)x - (uint32_t)above);
  const int32_t diag = r ? q[i - 9] : up[c - 1];
  return (int32_t)((uint32_t)x - (uint32_t)left - (uint32_t)above + (uint32_t)diag);
}

template <int K>
__device__ __forceinline__ uint32_t tile_or(const int32_t (&q)[32], const int32_t (&up)[8],
                                            uint32_t w) {
  uint32_t o = 0;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int32_t d = tile_res<K>(q, up, w, i);
    o |= (uint32_t)(d < 0 ? -d : d);
  }
  return grp_or<2>(o);
}

template <int K>
__device__ __forceinline__ void tile_mag(int32_t (&q)[32], const int32_t (&up)[8], uint32_t w,
                                         uint32_t& sg) {
  sg = 0;
#pragma unroll
  for (int i = 31; i >= 0; --i) {  // in place, downwards
    const int32_t d = tile_res<K>(q, up, w, i);
    q[i] = d < 0 ? -d : d;
    sg = __builtin_amdgcn_alignbit(sg, (uint32_t)d, 31);
  }
}

__device__ __forceinline__ uint32_t size_of(uint32_t kind, uint32_t F) {
  const uint32_t planes = F ? (F + 1u) * 2u : 0u;  // L = 64: two words per plane
  return kind == K_NONE ? planes : 1u + planes;
}

// Quantised tile values of the lane (used by the trial kernel and mode 1).
__device__ __forceinline__ void tile_quant(const Job& J, const float (&v)[32], int32_t (&q)[32],
                                           bool& bad) {
  QBad<float> qb;
  quant_run<32, true>(v, J, 32, (uint32_t*)q, qb);
  bad = grp_or<2>(qb.any(J.eblo) ? 1u : 0u) != 0;
}

// Mode 1 analysis: exhaustive trial (select 1), MLP (select 0) or L1D only.
__device__ __forceinline__ void analyze_tile(const Job& J, uint32_t w, const float (&v)[32],
                                             bool exists, const uint32_t* wts, LaneCode& lc) {
  int32_t (&q)[32] = *reinterpret_cast<int32_t(*)[32]>(lc.a);
  bool bad;
  tile_quant(J, v, q, bad);
  int32_t up[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) up[c] = (int32_t)lane_below((uint32_t)q[24 + c]);
  const int32_t base = q[0];
  uint32_t pk;  // 0 NONE, 1 L1D, 2 L2D
  uint32_t orv;
  if (J.select == 1) {
    const uint32_t o0 = tile_or<0>(q, up, w), o1 = tile_or<1>(q, up, w), o2 = tile_or<2>(q, up, w);
    const uint32_t F0 = o0 ? 32u - __clz(o0) : 0u, F1 = o1 ? 32u - __clz(o1) : 0u,
                   F2 = o2 ? 32u - __clz(o2) : 0u;
    const uint32_t s0 = size_of(K_NONE, F0), s1 = size_of(K_L1D, F1), s2 = size_of(K_L2D, F2);
    pk = 0; orv = o0;
    uint32_t bs = s0;
    if (s1 < bs) { pk = 1; bs = s1; orv = o1; }
    if (s2 < bs) { pk = 2; orv = o2; }
  } else if (J.select == 0) {
    uint32_t f[4];
    tile_features(q, w, f);
    pk = mlp_choose(f, w, wts);
    orv = pk == 0 ? tile_or<0>(q, up, w) : pk == 1 ? tile_or<1>(q, up, w) : tile_or<2>(q, up, w);
  } else {
    pk = 1;
    orv = tile_or<1>(q, up, w);
  }
  uint32_t sg;
  if (pk == 0) tile_mag<0>(q, up, w, sg);
  else if (pk == 1) tile_mag<1>(q, up, w, sg);
  else tile_mag<2>(q, up, w, sg);
  const uint32_t nzb = grp_or<2>(base != 0 ? 1u : 0u) | orv;
  uint32_t F = orv ? 32u - (uint32_t)__clz(orv) : 0u;
  uint32_t kind = pk == 0 ? K_NONE : pk == 1 ? K_L1D : K_L2D;
  uint32_t size_dw = size_of(kind, F);
  if (!exists) {
    kind = K_ZERO; F = 0; size_dw = 0;
  } else if (bad) {
    kind = K_RAW; F = 0; size_dw = 64;
  } else if (!nzb) {
    kind = K_ZERO; F = 0; size_dw = 0;
  } else if (size_dw > 64) {
    kind = K_RAW; F = 0; size_dw = 64;
  }
  lc.rawregs = 0;  // RAW tiles re-read their values from the input
  lc.sg = sg;
  lc.base = base;
  lc.kind = kind;
  lc.F = F;
  lc.size_dw = size_dw;
  lc.exists = exists;
}

// Element i of a lane segment: its offset from the segment's first element.
template <int MODE>
__device__ __forceinline__ uint64_t seg_off(const Job& J, int i) {
  return MODE == 0 ? (uint64_t)i : (uint64_t)(i / 8) * J.nx + (i % 8);
}
// First element of segment seg (mode 1: row 4w of tile seg/2).
template <int MODE>
__device__ __forceinline__ uint64_t seg_first(const Job& J, uint64_t seg) {
  if (MODE == 0) return seg * SEG;
  const uint32_t b = (uint32_t)(seg >> 1), tpr = J.nx / 8;  // fewer than 2^26 tiles: n < 2^32
  const uint32_t R = b / tpr, Cc = b - R * tpr;
  return (8 * (uint64_t)R + 4 * (seg & 1)) * J.nx + 8 * Cc;
}

// Scan, publish, stage, look back and write one strip (any mode).  KEEPV:
// v stays valid for RAW blocks; otherwise RAW blocks re-read J.in.
// Recomputes the fused step's sums y = x' + local of a lane (RAW blocks).
struct FusedSrc {
  const uint32_t* pay;  // incoming payload (global)
  DecInfo di;
  float t;
};

// Residual i of a lane read straight from its block's planes.
template <int LPB>
__device__ __forceinline__ uint32_t plane_res(const uint32_t* pw, uint32_t F, uint32_t sg,
                                              uint32_t w, int i) {
  uint32_t a = 0;
  for (uint32_t j = 0; j < F; ++j) a |= ((pw[1 + (j + 1) * LPB + w] >> i) & 1u) << j;
  const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int32_t)sg, i, 1);
  return (i == 0 && w == 0) ? 0u : (a ^ neg) - neg;
}

// Stages the fused step's sums y = x' + local of a RAW block bit for bit,
// re-deriving x' from the incoming block one element at a time (rare path,
// kept rolled so it adds no register pressure).
template <int LPB>
__device__ __forceinline__ void fused_raw_stage(const Job& J, const FusedSrc& fs, uint64_t seg,
                                             uint32_t w, uint32_t vcnt, uint32_t* st) {
  const uint32_t* pw = fs.pay + fs.di.off_dw;
  const uint32_t kind = fs.di.kind, F = fs.di.F;
  uint32_t carry = 0, sg = 0;
  if (kind == K_L1D) {
    sg = F ? pw[1 + w] : 0u;
    uint32_t tot = 0;
    for (int i = 0; i < 32; ++i) tot += plane_res<LPB>(pw, F, sg, w, i);
    carry = grp_excl_sum<LPB>(tot, w) + pw[0];
  }
  const float* loc = J.local + seg * SEG;
  uint32_t acc = 0;
  for (int i = 0; i < (int)vcnt; ++i) {
    float xp = 0.0f;
    if (kind == K_L1D) {
      acc += plane_res<LPB>(pw, F, sg, w, i);
      xp = (float)(int32_t)(carry + acc) * fs.t;
    } else if (kind == K_RAW) {
      xp = __uint_as_float(pw[w * 32 + i]);
    }
    st[w * 32 + i] = __float_as_uint(xp + loc[i]);
  }
}

// Word i (0..15) of the stream header for a payload of `payload` bytes.
__device__ __forceinline__ uint32_t hdr_word(const Job& J, uint32_t i, uint64_t payload) {
  const unsigned long long ebits = (unsigned long long)__double_as_longlong(J.eb);
  switch (i) {
    case 0: return 0x31435A47u;
    case 1: return 1u | (J.dtype << 16) | (J.log2L << 24);
    case 2: return (uint32_t)J.n;
    case 3: return (uint32_t)(J.n >> 32);
    case 4: return (uint32_t)ebits;
    case 5: return (uint32_t)(ebits >> 32);
    case 6: return (uint32_t)payload;
    case 7: return (uint32_t)(payload >> 32);
    case 8: return J.mode;
    case 9: return J.nx;
    case 10: return SUPER;
    default: return 0u;
  }
}

template <typename T, int L, int MODE, bool FUSED, bool FULL>
__device__ void emit_strip(const Job& J, uint64_t s, uint64_t gs, const Ctl& C, Smem& sm,
                           uint32_t vcnt, const LaneCode& lc, const FusedSrc* fs, bool skip,
                           uint32_t& tk) {
  constexpr int LPB = L / 32;
  constexpr uint32_t EW = sizeof(T) / 4;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint32_t TPB = blockDim.x;
  const uint64_t seg = s * TPB + tid;
  const uint32_t w = tid & (LPB - 1);
  uint32_t* stage = g_stage + 4;
  const uint32_t kind = lc.kind, F = lc.F, size_dw = lc.size_dw;

  uint32_t total;
  const uint32_t excl_lane = strip_scan(w == 0 ? size_dw : 0u, sm, total);
  const uint32_t boff = (w == 0) ? excl_lane : excl_lane - size_dw;
  if (tid == 0) publish_agg(C, gs, J.chain0, sm.epoch, total);
  if (w == 0) ((uint8_t*)sm.hb)[tid / LPB] = (uint8_t)(lc.exists ? ((kind << 5) | F) : 0u);

  // pack the payload into LDS while the predecessors resolve
  uint32_t* st = stage + boff;
  if (kind == K_L1D || kind == K_L2D || kind == K_NONE) {
    uint32_t o = 0;
    if (kind != K_NONE) {
      if (w == 0) st[0] = (uint32_t)lc.base;
      o = 1;
    }
    if (F) {
      st[o + w] = lc.sg;
      put_planes(lc.a, F, st + o + LPB + w, LPB);
    }
  }
  // a separate (not else) branch: the magnitudes are dead before it runs
  if (FUSED && kind == K_RAW && lc.rawregs) {
#pragma unroll
    for (int i = 0; i < 32; ++i)  // unrolled: a[] stays in registers
      if ((FULL && MODE == 0) || i < (int)vcnt) st[w * 32 + i] = lc.a[i];
  } else if (kind == K_RAW) {  // blocks too wide to code (rare): re-derive
    if (FUSED) {
      fused_raw_stage<L / 32>(J, *fs, seg, w, vcnt, st);
    } else {
      const T* src = (const T*)J.in + seg_first<MODE>(J, seg);
      for (int i = 0; i < (int)vcnt; ++i) {  // rolled: a rare path, kept small
        uint32_t wd[2];
        raw_words(src[seg_off<MODE>(J, i)], wd);
        st[(w * 32 + i) * EW] = wd[0];
        if (EW == 2) st[(w * 32 + i) * EW + 1] = wd[1];
      }
    }
  }

  if (wid == 0) {
    bool to = false;
    uint64_t ex = lookback(C, gs, J.chain0, sm.epoch, total, to);
    uint64_t pj = 0;
    if (J.chain0 != J.strip0) {
      if (s == 0) {
        if (lane == 0 && !to) st_agent(C.jobbase + J.job, sw_pack(2, sm.epoch, ex));
        pj = ex;
      } else if (!to) {
        pj = job_base_wait(C, J.job, sm.epoch, to);
      }
    }
    if (lane == 0) {
      sm.excl = ex;
      sm.pj = pj;
      sm.flag = to ? ERRF_TIMEOUT : 0u;
      if (to) atomicOr(&C.ctrl->err, ERRF_TIMEOUT);
    }
  }
  __syncthreads();
  // The workgroup's next strip is ticketed only now, once this strip's
  // offset is known: a ticket held by a workgroup that has not started it
  // would stall the look-back of every later strip.
  if (tid == 0) tk = atomicAdd(&C.ctrl->ticket, 1u);
  if (sm.flag || skip) return;

  const uint64_t pj = sm.pj;
  const uint64_t erel = sm.excl - pj;  // strip offset inside this job's payload
  uint8_t* base8 = (uint8_t*)J.out + J.fixed_off + 4 * pj;
  uint32_t* dst = (uint32_t*)(base8 + J.pay_off) + erel;
  for (uint32_t k = tid; k < total; k += TPB) dst[k] = stage[k];

  if (lc.exists && (seg & (SUPER / SEG - 1)) == 0)
    ((uint32_t*)(base8 + HDR))[seg / (SUPER / SEG)] = (uint32_t)(erel + boff);
  // header bytes as whole words (the strip starts on a 4-block boundary)
  const uint32_t nblk = TPB / LPB;
  const uint64_t blk0 = s * (uint64_t)nblk;
  for (uint32_t i = tid; i < nblk / 4; i += TPB) {
    if (blk0 + 4 * i < J.B) *(uint32_t*)(base8 + J.hdr_off + blk0 + 4 * i) = sm.hb[i];
  }
  // the last strip completes the header and the size outputs
  if (s == J.nstrips - 1 && tid < 16) {
    const uint64_t payload = 4 * (sm.excl + total - pj);
    ((uint32_t*)base8)[tid] = hdr_word(J, tid, payload);
    if (tid == 0) {
      if (J.out_bytes) *J.out_bytes = J.pay_off + payload;
      if (J.chunk_off) *J.chunk_off = J.fixed_off + 4 * pj;
    }
  }
}

// Mode 0 strip encode (FULL: the strip lies entirely inside n).  fs: the
// fused step's incoming stream, to re-derive the sums of RAW blocks.
template <typename T, int L, bool FULL, bool FUSED>
__device__ __forceinline__ void encode_strip(const Job& J, uint64_t s, uint64_t gs, const Ctl& C,
                                             Smem& sm, const T (&v)[32], uint32_t vcnt,
                                             const FusedSrc* fs, bool skip, uint32_t& tk) {
  const uint64_t seg = s * blockDim.x + threadIdx.x;
  LaneCode lc;
  analyze_1d<T, L, FULL, FUSED>(J, seg, threadIdx.x & (L / 32 - 1), v, vcnt, lc);
  emit_strip<T, L, 0, FUSED, FULL>(J, s, gs, C, sm, vcnt, lc, fs, skip, tk);
}

// --------------------------------------------------------------- decode
// Checks the stream header against the job; sets sm.hdr_ok, sm.paydw, sm.t*.
__device__ void check_header(const Job& J, const uint8_t* in, uint64_t in_bytes, Smem& sm) {
  const int tid = threadIdx.x;
  if (tid < 64) {
    const bool readable = in_bytes >= HDR;
    uint32_t wv = (tid < 16 && readable) ? ((const uint32_t*)in)[tid] : 0u;
    bool ok = true;
    switch (tid) {
      case 0: ok = wv == 0x31435A47u; break;
      case 1: ok = wv == (1u | (J.dtype << 16) | (J.log2L << 24)); break;
      case 2: ok = wv == (uint32_t)J.n; break;
      case 3: ok = wv == (uint32_t)(J.n >> 32); break;
      case 8: ok = wv == J.mode; break;
      case 9: ok = wv == J.nx; break;
      case 10: ok = wv == SUPER; break;
      case 4: case 5: case 6: case 7: ok = true; break;
      default: ok = wv == 0u; break;
    }
    uint64_t okm = __ballot(ok);
    const uint32_t e0 = read_lane(wv, 4), e1 = read_lane(wv, 5);
    const uint32_t p0 = read_lane(wv, 6), p1 = read_lane(wv, 7);
    if (tid == 0) {
      double eb = __longlong_as_double((long long)(((uint64_t)e1 << 32) | e0));
      uint64_t payload = ((uint64_t)p1 << 32) | p0;
      bool good = readable && okm == ~0ull;
      good = good && (eb > 0.0) && isfinite(eb);
      float t32 = (float)(2.0 * eb);
      double t64 = 2.0 * eb;
      if (J.dtype == 0) good = good && isfinite(t32) && t32 != 0.0f;
      else good = good && isfinite(t64) && t64 != 0.0;
      good = good && (payload % 4 == 0) && payload <= in_bytes &&
             J.pay_off <= in_bytes - payload;
      sm.hdr_ok = good ? 1u : 0u;
      sm.t32 = t32;
      sm.t64 = t64;
      sm.paydw = payload / 4;
    }
  }
  __syncthreads();
  // Marked checked only after the barrier: every wave has then read the old
  // mark and entered this function, so all of them take the same barriers.
  if (tid == 0) sm.hdr_job = J.job + 1;
}

template <typename T>
__device__ __forceinline__ T step_of(const Smem& sm);
template <>
__device__ __forceinline__ float step_of<float>(const Smem& sm) { return sm.t32; }
template <>
__device__ __forceinline__ double step_of<double>(const Smem& sm) { return sm.t64; }

// Copies payload dwords [src, src + P) into LDS with 16-byte loads; returns
// the LDS address of src[0].  Only bytes inside [lo, src + 4P) are read,
// where lo <= src is readable stream memory.
__device__ __forceinline__ const uint32_t* copy_in(const uint32_t* src, uint32_t P) {
  const uint32_t tid = threadIdx.x, TPB = blockDim.x;
  // realigned by pointer arithmetic (an integer round trip would lose the
  // pointer's global address space)
  const uint32_t delta = (uint32_t)(((uintptr_t)src & 15u) >> 2);
  const u4u* al = (const u4u*)(src - delta);
  const uint32_t nch = (delta + P + 3) / 4;  // 16-byte chunks touched
  const uint32_t full = (delta + P) / 4;     // chunks entirely inside
  u4u* dstc = (u4u*)g_stage;
  // whole chunks, four independent loads in flight per lane.  The first
  // 8 TPB chunks (all of an fp32 strip: a payload never exceeds the raw
  // size) are straight-line code: in a loop, the next pass's loads into the
  // same registers make the compiler wait for every outstanding memory
  // operation before each load.  fp64 strips may need the loop after it.
  // Lanes past the end re-read the last whole chunk instead of branching
  // around the load (a conditional load leaves a merge of registers that the
  // compiler resolves with copies, which wait for the load at once).
#pragma unroll
  for (uint32_t h = 0; h < 2; ++h) {
    const uint32_t k0 = h * 4 * TPB;
    if (full <= k0) break;
    u4u r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = al[min(k0 + u * TPB + tid, full - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t k = k0 + u * TPB + tid;
      if (k < full) dstc[k] = r[u];
    }
  }
  for (uint32_t k = 8 * TPB + tid; k < full; k += TPB) dstc[k] = al[k];
  // the range ends inside the last chunk: dword loads, so that nothing past
  // it is read
  if (full < nch && tid == 0) {
    const uint32_t* p = (const uint32_t*)(al + full);
    const uint32_t lim = delta + P - 4 * full;  // 1..3 valid dwords
    u4u r;
    r.x = p[0];
    r.y = lim > 1 ? p[1] : 0u;
    r.z = lim > 2 ? p[2] : 0u;
    r.w = 0u;
    dstc[full] = r;
  }
  return g_stage + delta;
}

// Rebuilds the lane's 4 tile rows (mode 1) from its block's words at pw.
// Each lane first sums its own rows as if the row above were zero; lane 1
// then adds lane 0's last row (L2D) or its first-column value (L1D).
template <typename T>
__device__ __forceinline__ void unpack_tile(const uint32_t* pw, uint32_t kind, uint32_t F,
                                            uint32_t w, bool exists, T t, T (&v)[32]) {
  if (kind == K_RAW) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = from_raw(pw + (w * 32 + i) * (sizeof(T) / 4), T());
    return;
  }
  if (kind == K_ZERO || !exists) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = (T)0;
    return;
  }
  const uint32_t o = kind == K_NONE ? 0u : 1u;
  const uint32_t base = o ? pw[0] : 0u;
  uint32_t q[32];
  get_planes(pw + o + 2 + w, 2, F, q);
  const uint32_t sg = F ? pw[o + w] : 0u;
#pragma unroll
  for (int i = 0; i < 32; ++i) {  // signed residuals
    const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int32_t)sg, i, 1);
    q[i] = (q[i] ^ neg) - neg;
  }
  if (kind == K_L1D) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int i = 8 * r + c;
        if (c) q[i] = q[i - 1] + q[i];
        else if (r) q[i] = q[i - 8] + q[i];
        else q[i] = w == 0 ? base : q[i];  // (0,0) holds the base
      }
    }
    const uint32_t carry = lane_below(q[24]);  // lane 0's q(3,0)
    if (w) {
#pragma unroll
      for (int i = 0; i < 32; ++i) q[i] += carry;
    }
  } else if (kind == K_L2D) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint32_t acc = 0;  // v(r,c): the row prefix of d
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int i = 8 * r + c;
        if (r == 0 && w == 0) {
          q[i] = c ? q[i - 1] + q[i] : base;  // first row: L1D along the row
        } else {
          acc += q[i];
          q[i] = (r ? q[i - 8] : 0u) + acc;
        }
      }
    }
    uint32_t up[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) up[c] = lane_below(q[24 + c]);  // lane 0's row 3
    if (w) {
#pragma unroll
      for (int i = 0; i < 32; ++i) q[i] += up[i % 8];
    }
  }
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = (T)(int32_t)q[i] * t;
}

// Decodes the lane's segment of strip s of the stream at `in` into v[];
// returns false (and flags the context) if the strip is malformed.
// Superblock-table words bounding strip s's payload (0 where the table is
// absent or the superblock lies past the end).
__device__ __forceinline__ void table_words(const Job& J, const uint8_t* in, uint64_t in_bytes,
                                            uint64_t s, uint32_t& T0, uint32_t& T1) {
  const uint32_t* table = (const uint32_t*)(in + HDR);
  const uint64_t sb0 = s * (uint64_t)(blockDim.x * SEG / SUPER);
  const uint64_t sbn = sb0 + blockDim.x * SEG / SUPER;
  T0 = 0;
  T1 = 0;
  if (in_bytes >= J.pay_off && J.NS) {
    // both loads issued before either is used (clamped indices, not
    // conditional loads, which the compiler waits for one at a time)
    const uint32_t a = table[min(sb0, J.NS - 1)];
    const uint32_t b = table[min(sbn, J.NS - 1)];
    T0 = sb0 < J.NS ? a : 0u;
    T1 = sbn < J.NS ? b : 0u;
  }
}

// pkey (nonzero): the strip's table words may already sit in sm.tp_t0/t1,
// fetched by thread 0 during the previous strip (when sm.tp_key == pkey).
template <typename T, int L, bool FULL, int MODE = 0>
__device__ bool decode_strip(const Job& J, const uint8_t* in, uint64_t in_bytes, uint64_t s,
                             const Ctl& C, Smem& sm, T (&v)[32], uint32_t vcnt, DecInfo& di,
                             uint32_t pkey = 0) {
  constexpr int LPB = L / 32;
  constexpr uint32_t EW = sizeof(T) / 4;
  const int tid = threadIdx.x;
  const uint32_t TPB = blockDim.x;
  const uint64_t seg = s * TPB + tid;
  const uint32_t w = tid & (LPB - 1);
  const uint64_t b = seg / LPB;

  // strip payload range from the superblock table; the table words are
  // read together with the header (both lie in the stream's fixed part,
  // readable when in_bytes reaches the payload)
  const uint32_t* table = (const uint32_t*)(in + HDR);
  const uint64_t sb0 = s * (uint64_t)(TPB * SEG / SUPER);
  const uint64_t sbn = sb0 + TPB * SEG / SUPER;
  uint32_t T0, T1;
  if (pkey && sm.tp_key == pkey) {
    T0 = sm.tp_t0;
    T1 = sm.tp_t1;
  } else {
    table_words(J, in, in_bytes, s, T0, T1);
  }
  // a lane that starts a superblock checks its table entry below; the word
  // is read now, with the others, not after the scan
  const bool exists = FULL || b < J.B;
  const bool sb_lane = exists && (seg & (SUPER / SEG - 1)) == 0;
  uint32_t Tsb = 0;
  if (in_bytes >= J.pay_off && J.NS) {  // every lane loads (clamped): no wait per load
    const uint32_t x = table[min(seg / (SUPER / SEG), J.NS - 1)];
    Tsb = sb_lane ? x : 0u;
  }
  if (sm.hdr_job != J.job + 1) check_header(J, in, in_bytes, sm);
  const bool ok = sm.hdr_ok != 0;  // implies in_bytes >= J.pay_off
  const uint64_t pay_dw = sm.paydw;
  uint64_t E = 0, En = 0;
  if (ok) {
    E = sb0 < J.NS ? T0 : pay_dw;
    En = sbn < J.NS ? T1 : pay_dw;
  }
  const bool rng = ok && E <= En && En <= pay_dw && En - E <= (uint64_t)TPB * SEG * EW;
  const uint32_t P = rng ? (uint32_t)(En - E) : 0u;
  // the header byte is loaded before the payload copy, in the same round
  // trip (after it, it would cost a second one)
  const uint32_t hb = (rng && exists) ? (uint32_t)in[J.hdr_off + b] : 0u;
  const uint32_t* S = g_stage + 4;
  if (rng) S = copy_in((const uint32_t*)(in + J.pay_off) + E, P);

  const uint32_t m = FULL ? (uint32_t)L
                          : (exists ? (uint32_t)min((uint64_t)L, J.n - b * (uint64_t)L) : 0u);
  const uint32_t kind = hb >> 5, F = hb & 31u;
  uint32_t size_dw = 0;
  bool hv = true;
  if (kind == K_ZERO) hv = F == 0;
  else if (kind == K_RAW) { hv = F == 0; size_dw = m * EW; }
  else if (kind == K_L1D || (MODE == 1 && kind == K_L2D)) size_dw = 1u + (F ? (F + 1u) * LPB : 0u);
  else if (MODE == 1 && kind == K_NONE) { hv = F > 0; size_dw = (F + 1u) * LPB; }
  else hv = false;
  if (!hv) size_dw = 0;

  uint32_t total;
  const uint32_t excl_lane = strip_scan(w == 0 ? size_dw : 0u, sm, total);
  const uint32_t boff = (w == 0) ? excl_lane : excl_lane - size_dw;
  bool good = rng && hv && total == P;
  if (good && sb_lane) good = (uint64_t)Tsb == E + boff;
  if (s == 0) good = good && E == 0;
  if (rng && s == J.nstrips - 1 && tid < 4) {
    const uint64_t pb = J.B + tid;
    if (pb < ((J.B + 3) & ~3ull)) good = good && in[J.hdr_off + pb] == 0;
  }
  good = __syncthreads_and(good ? 1 : 0) != 0;  // also completes the copy-in
  if (!good) {
    if (tid == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = (T)0;
    return false;
  }

  di.off_dw = (uint32_t)E + boff;
  di.kind = kind;
  di.F = F;
  if (MODE == 0) unpack_seg<T, LPB, FULL>(S + boff, kind, F, w, vcnt, exists, step_of<T>(sm), v);
  else unpack_tile<T>(S + boff, kind, F, w, exists, step_of<T>(sm), v);
  return true;
}

// ---------------------------------------------------------------- kernels
template <typename T, int L, bool FULL>
__device__ __forceinline__ void compress_body(const Job& J, uint64_t s, uint64_t gs,
                                              const Ctl& C, Smem& sm, uint32_t& tk) {
  const uint64_t seg = s * blockDim.x + threadIdx.x;
  const uint64_t e0 = seg * SEG;
  const uint32_t vcnt = FULL ? 32u : (e0 >= J.n ? 0u : (uint32_t)min((uint64_t)SEG, J.n - e0));
  const uint64_t s0 = s * blockDim.x * (uint64_t)SEG;
  if (FULL && sizeof(T) == 4) strip_to_lds_whole<T>((const T*)J.in + s0);
  else strip_to_lds<T>((const T*)J.in + s0, FULL ? (uint64_t)blockDim.x * SEG : J.n - s0);
  __syncthreads();
  T v[32];
  lane_from_lds<T>(v);
  encode_strip<T, L, FULL, false>(J, s, gs, C, sm, v, vcnt, nullptr, false, tk);
}

template <typename T, int L>
__device__ __forceinline__ void compress_one(const Job& J, uint64_t s, uint64_t gs,
                                             const Ctl& C, Smem& sm, uint32_t& tk) {
  if ((s + 1) * blockDim.x * SEG <= J.n) compress_body<T, L, true>(J, s, gs, C, sm, tk);
  else compress_body<T, L, false>(J, s, gs, C, sm, tk);
}

template <typename T, int L, bool FULL>
__device__ __forceinline__ void decompress_body(const Job& J, uint64_t s, const Ctl& C,
                                                Smem& sm) {
  const uint64_t off = J.in_off ? J.in_off[J.job] : 0ull;
  const uint8_t* in = (const uint8_t*)J.in + off;
  const uint64_t avail = off <= J.in_bytes ? J.in_bytes - off : 0ull;
  const uint64_t e0 = (s * blockDim.x + threadIdx.x) * SEG;
  const uint32_t vcnt = FULL ? 32u : (e0 >= J.n ? 0u : (uint32_t)min((uint64_t)SEG, J.n - e0));
  T v[32];
  DecInfo di;
  if (decode_strip<T, L, FULL>(J, in, avail, s, C, sm, v, vcnt, di)) {
    __syncthreads();  // every lane has read its payload words
    lane_to_lds<T>(v);
    __syncthreads();
    const uint64_t s0 = s * blockDim.x * (uint64_t)SEG;
    lds_to_strip<T>((T*)J.out + s0, FULL ? (uint64_t)blockDim.x * SEG : J.n - s0);
  }
}

template <typename T, int L>
__device__ __forceinline__ void decompress_one(const Job& J, uint64_t s, const Ctl& C,
                                               Smem& sm) {
  if ((s + 1) * blockDim.x * SEG <= J.n) decompress_body<T, L, true>(J, s, C, sm);
  else decompress_body<T, L, false>(J, s, C, sm);
}

// Decode-and-accumulate (fp32): acc[i] = fl32(decoded[i] + acc[i]), the
// reduction that follows each receive in recursive-doubling Allreduce
// (Sec. 3.3.4), without writing the decoded values to memory.  A whole
// strip's accumulator is read with coalesced loads issued before the decode,
// so they are in flight while it runs.  A malformed stream leaves acc as it
// was (and flags the context).
template <int L, bool FULL>
__device__ __forceinline__ void accum_body(const Job& J, uint64_t s, const Ctl& C, Smem& sm) {
  constexpr uint32_t STR = seg_stride<float>();
  const uint32_t TPB = blockDim.x;
  const uint64_t e0 = (s * TPB + threadIdx.x) * SEG;
  const uint32_t vcnt = FULL ? 32u : (e0 >= J.n ? 0u : (uint32_t)min((uint64_t)SEG, J.n - e0));
  const uint64_t s0 = s * TPB * (uint64_t)SEG;
  uint32_t* acc = (uint32_t*)((float*)J.out + s0);
  u4u old[8];
  if (FULL) {  // chunk u*TPB + tid of the strip
    const uint32_t tid = opaque_tid();
#pragma unroll
    for (int u = 0; u < 8; ++u) old[u] = ((const u4u*)(acc + 4ull * u * TPB))[tid];
  }
  float v[32];
  DecInfo di;
  if (!decode_strip<float, L, FULL>(J, (const uint8_t*)J.in, J.in_bytes, s, C, sm, v, vcnt, di))
    return;
  __syncthreads();  // every lane has read its payload words
  lane_to_lds<float>(v);
  __syncthreads();
  const uint32_t* buf = g_stage + 4;
  if (FULL) {
    const uint32_t tid = opaque_tid();
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t k = u * TPB + tid;  // chunk k = segment k/8, words 4*(k%8)..
      const u4u d = *(const u4u*)(buf + (k / 8) * STR + 4 * (k % 8));
      u4u y;
      y.x = __float_as_uint(__uint_as_float(d.x) + __uint_as_float(old[u].x));
      y.y = __float_as_uint(__uint_as_float(d.y) + __uint_as_float(old[u].y));
      y.z = __float_as_uint(__uint_as_float(d.z) + __uint_as_float(old[u].z));
      y.w = __float_as_uint(__uint_as_float(d.w) + __uint_as_float(old[u].w));
      ((u4u*)(acc + 4ull * u * TPB))[tid] = y;
    }
  } else {  // the tail strip: element by element
    const uint64_t nv = J.n - s0;
    for (uint32_t i = threadIdx.x; i < nv; i += TPB) {
      const float d = __uint_as_float(buf[(i / 32) * STR + i % 32]);
      acc[i] = __float_as_uint(d + __uint_as_float(acc[i]));
    }
  }
}

template <int L>
__device__ __forceinline__ void accum_one(const Job& J, uint64_t s, const Ctl& C, Smem& sm) {
  if ((s + 1) * blockDim.x * SEG <= J.n) accum_body<L, true>(J, s, C, sm);
  else accum_body<L, false>(J, s, C, sm);
}

// Single-stream decoding that fetches the next strip's table words (thread 0
// holds the next ticket, nxt) while this strip unpacks and stores, so that
// the next strip's payload copy starts at once: one dependent memory round
// trip per strip instead of two.
template <typename T, int L, bool FULL>
__device__ __forceinline__ void decompress_tp_body(const Job& J, uint64_t s, const Ctl& C,
                                                   Smem& sm, uint32_t nxt) {
  const uint8_t* in = (const uint8_t*)J.in;
  const uint64_t e0 = (s * blockDim.x + threadIdx.x) * SEG;
  const uint32_t vcnt = FULL ? 32u : (e0 >= J.n ? 0u : (uint32_t)min((uint64_t)SEG, J.n - e0));
  T v[32];
  DecInfo di;
  if (decode_strip<T, L, FULL>(J, in, J.in_bytes, s, C, sm, v, vcnt, di, (uint32_t)s + 1u)) {
    uint32_t p0 = 0, p1 = 0;
    if (threadIdx.x == 0 && nxt < J.nstrips) table_words(J, in, J.in_bytes, nxt, p0, p1);
    __syncthreads();  // every lane has read its payload words
    lane_to_lds<T>(v);
    __syncthreads();
    // read by the next strip after the loop's barrier; written before the
    // stores are issued, so that waiting for the table words does not also
    // wait for this strip's stores (the wait counter is in order)
    if (threadIdx.x == 0) {
      sm.tp_t0 = p0;
      sm.tp_t1 = p1;
      sm.tp_key = nxt + 1u;
    }
    const uint64_t s0 = s * blockDim.x * (uint64_t)SEG;
    lds_to_strip<T>((T*)J.out + s0, FULL ? (uint64_t)blockDim.x * SEG : J.n - s0);
  }
}

template <typename T, int L>
__device__ __forceinline__ void decompress_tp_one(const Job& J, uint64_t s, const Ctl& C,
                                                  Smem& sm, uint32_t nxt) {
  if ((s + 1) * blockDim.x * SEG <= J.n) decompress_tp_body<T, L, true>(J, s, C, sm, nxt);
  else decompress_tp_body<T, L, false>(J, s, C, sm, nxt);
}

// ---------------------------------------------------------- per-wave decode
// A wave decodes whole 4096-element superblocks on its own: a superblock's
// payload offset is its table entry, so waves need no scan across each
// other, no ticket and no workgroup barrier, and the phases of different
// waves (loads, unpacking, stores) overlap freely.  Superblock i goes to
// wave i mod W (W waves in the grid): decoding has no dependency between
// superblocks, so this static assignment needs no co-residency.  A wave's
// LDS region holds the superblock's payload, then its decoded values in the
// padded segment layout for coalesced stores.  Lane l decodes segments l and
// 64 + l of the superblock.  For fp32 streams of more than 2^24 elements,
// shorter than 2^19, and batches of them (the unit decoder takes the rest).
struct WaveDec {
  static constexpr uint32_t WAVES = 8;  // per workgroup
  static_assert(WAVES == DEC_WAVES_F32, "host's job shares assume this");
  static constexpr uint32_t REGION = 2 * 64 * seg_stride<float>() + 8;  // dwords per wave
};

// LDS written by some lanes of the wave is read by others: the wave's LDS
// operations complete in order, and the compiler may not move memory
// accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// The lane's word of the stream header (lanes 0..15; 0 if unreadable).
__device__ __forceinline__ uint32_t wave_header_load(const Job& J, const uint8_t* in) {
  const uint32_t lane = __lane_id();
  return (lane < 16 && J.in_bytes >= HDR) ? ((const uint32_t*)in)[lane] : 0u;
}

// A lane's value in every lane: as a scalar, or (VEC) in a vector register.  The
// job-share decoder has vector registers to spare and spills scalar ones (23 and
// 6): 64 chunks of 2^21, ring data, 137 and 136 us a launch, 6 ranks of 4 M
// elements 31.4 and 29.7, 64 chunks of 2^20 at ratio 2 84.5 and 81.3; the fused
// kernels lose 2 to 6% by it.
template <bool VEC>
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {
  return VEC ? __shfl(v, lane) : read_lane(v, lane);
}

// The stream header (the lanes' words wv) against the job, by one wave: ok,
// payload dwords and step.
template <typename T, bool VEC = false>
__device__ __forceinline__ bool wave_header_eval(const Job& J, uint32_t wv, uint64_t& paydw,
                                                 T& t) {
  const uint32_t lane = __lane_id();
  const bool readable = J.in_bytes >= HDR;
  bool ok = true;
  switch (lane) {
    case 0: ok = wv == 0x31435A47u; break;
    case 1: ok = wv == (1u | (J.dtype << 16) | (J.log2L << 24)); break;
    case 2: ok = wv == (uint32_t)J.n; break;
    case 3: ok = wv == (uint32_t)(J.n >> 32); break;
    case 8: ok = wv == J.mode; break;
    case 9: ok = wv == J.nx; break;
    case 10: ok = wv == SUPER; break;
    case 4: case 5: case 6: case 7: ok = true; break;
    default: ok = lane < 16 ? wv == 0u : true; break;
  }
  const bool allok = __ballot(ok) == ~0ull;
  const uint32_t e0 = lane_value<VEC>(wv, 4), e1 = lane_value<VEC>(wv, 5),
                 p0 = lane_value<VEC>(wv, 6), p1 = lane_value<VEC>(wv, 7);
  const double eb = __longlong_as_double((long long)(((uint64_t)e1 << 32) | e0));
  const uint64_t payload = ((uint64_t)p1 << 32) | p0;
  bool good = readable && allok && (eb > 0.0) && isfinite(eb);
  const float t32 = (float)(2.0 * eb);
  const double t64 = 2.0 * eb;
  if (sizeof(T) == 4) good = good && isfinite(t32) && t32 != 0.0f;
  else good = good && isfinite(t64) && t64 != 0.0;
  good = good && (payload % 4 == 0) && payload <= J.in_bytes && J.pay_off <= J.in_bytes - payload;
  paydw = payload / 4;
  t = sizeof(T) == 4 ? (T)t32 : (T)t64;
  return good;
}

template <typename T, bool VEC = false>
__device__ __forceinline__ bool wave_header(const Job& J, const uint8_t* in, uint64_t& paydw,
                                            T& t) {
  return wave_header_eval<T, VEC>(J, wave_header_load(J, in), paydw, t);
}

// Block layout of superblock sb of an incoming stream, read by one wave:
// its payload range [E, En) in dwords from the payload start and, for
// segment 64h + lane (h = 0, 1), its block's kind, width, existence and
// payload offset from E; half0 = the payload dwords of the first 64
// segments' blocks.
struct WaveBlocks {
  uint64_t E, En;
  uint32_t kind[2], F[2], boff[2], half0;
  bool ex[2];
};

// The words wave_blocks_eval needs (table entries of sb and sb + 1, the
// lane's word of header bytes), read together.  SPEC: the stream header
// has not been checked yet, so offsets are clamped to the readable bytes
// (a stream that fails the check never has these words used); otherwise
// the checked header puts them inside the stream.
template <int L, bool SPEC>
__device__ __forceinline__ void wave_blocks_load(const Job& J, const uint8_t* in, uint64_t sb,
                                                 uint32_t (&raw)[3]) {
  constexpr uint32_t BPS = SUPER / L;
  const uint32_t lane = __lane_id();
  const uint64_t hb_end = (J.B + 3) & ~3ull;
  const uint64_t hidx = min(sb * BPS + 4ull * (lane & (BPS / 4 - 1)), hb_end - 4);
  const uint64_t o[3] = {HDR + 4 * sb, HDR + 4 * min(sb + 1, J.NS - 1), J.hdr_off + hidx};
  if (!SPEC) {
#pragma unroll
    for (int i = 0; i < 3; ++i) raw[i] = *(const uint32_t*)(in + o[i]);
    return;
  }
  if (J.in_bytes < 4) {  // nothing readable (the header check fails too)
    raw[0] = raw[1] = raw[2] = 0u;
    return;
  }
  const uint64_t lim = (J.in_bytes - 4) & ~3ull;
#pragma unroll
  for (int i = 0; i < 3; ++i) raw[i] = *(const uint32_t*)(in + min(o[i], lim));
}

// False if the table entries, header bytes or block sizes are inconsistent
// (the same checks as the strip decoder's); raw from wave_blocks_load, of a
// stream whose header passed.
template <typename T, int L, int MODE = 0, bool VEC = false>
__device__ bool wave_blocks_eval(const Job& J, uint64_t sb, uint64_t paydw, uint32_t nval,
                                 const uint32_t (&raw)[3], WaveBlocks& wb) {
  constexpr uint32_t EW = sizeof(T) / 4, LPB = L / 32, BPS = SUPER / L;
  const uint32_t lane = __lane_id();
  const uint32_t ta = raw[0], tb = raw[1], hraw = raw[2];
  const uint64_t b0 = sb * BPS;
  const uint64_t hb_end = (J.B + 3) & ~3ull;
  const uint32_t hw = (lane < BPS / 4 && b0 + 4ull * lane < hb_end) ? hraw : 0u;
  const uint64_t E = ta;
  const uint64_t En = sb + 1 < J.NS ? (uint64_t)tb : paydw;
  bool good = (sb != 0 || E == 0) && E <= En && En <= paydw && En - E <= (uint64_t)SUPER * EW;
  // header bytes past the last block (zero padding of the last word)
  if (lane < BPS / 4) {
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint64_t bb = b0 + 4ull * lane + k;
      if (bb >= J.B && bb < hb_end && ((hw >> (8 * k)) & 0xFFu)) good = false;
    }
  }
  // kinds, widths and sizes of the lane's two blocks; exclusive offsets
  uint32_t tot = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t seg = 64 * h + lane, lb = seg / LPB, w = seg % LPB;
    const uint32_t hb = (__shfl(hw, (int)(lb / 4)) >> (8 * (lb % 4))) & 0xFFu;
    const bool ex = lb * (uint32_t)L < nval;
    const uint32_t m = ex ? min((uint32_t)L, nval - lb * (uint32_t)L) : 0u;
    const uint32_t kd = ex ? hb >> 5 : 0u, f = ex ? hb & 31u : 0u;
    uint32_t size_dw = 0;
    bool hv = true;
    if (kd == K_ZERO) hv = f == 0;
    else if (kd == K_RAW) { hv = f == 0; size_dw = m * EW; }
    else if (kd == K_L1D || (MODE == 1 && kd == K_L2D)) size_dw = 1u + (f ? (f + 1u) * LPB : 0u);
    else if (MODE == 1 && kd == K_NONE) { hv = f > 0; size_dw = (f + 1u) * LPB; }
    else hv = false;
    if (!hv) size_dw = 0;
    good = good && hv;
    const uint32_t contrib = w == 0 ? size_dw : 0u;
    const uint32_t incl = wave_incl_scan(contrib);
    const uint32_t excl = tot + incl - contrib;
    wb.boff[h] = w == 0 ? excl : excl - size_dw;  // later lanes of a block contribute 0
    tot += lane_value<VEC>(incl, 63);
    if (h == 0) wb.half0 = tot;
    wb.kind[h] = kd;
    wb.F[h] = f;
    wb.ex[h] = ex;
  }
  good = good && (uint64_t)tot == En - E;
  wb.E = E;
  wb.En = En;
  return __ballot(good) == ~0ull;
}


// Copies P payload dwords from src (global) into dst (LDS, 16-byte aligned),
// realigned so that every load is a whole 16-byte chunk: only bytes inside
// [16-byte floor of src, src + P) are read, and src lies past the stream's
// fixed part.  Returns where src[0] landed (dst + 0..3).  MAXW bounds P.
// UNROLL: straight-line code with uniform guards (a loop makes the compiler
// wait for every outstanding memory operation at its head, the previous
// stores included; the decoder gains, the fused step, short of registers,
// does not).
template <uint32_t MAXW, bool UNROLL>
__device__ __forceinline__ const uint32_t* wave_stage_payload(const uint32_t* src, uint32_t P,
                                                              uint32_t* dst) {
  const uint32_t lane = __lane_id();
  const uint32_t delta = (uint32_t)(((uintptr_t)src & 15u) >> 2);
  const u4u* al = (const u4u*)(src - delta);
  const uint32_t full = (delta + P) / 4, nch = (delta + P + 3) / 4;
  u4u* d4 = (u4u*)dst;
  constexpr uint32_t MAXCH = (MAXW + 3) / 4 + 1;
  if (UNROLL) {
#pragma unroll
    for (uint32_t k0 = 0; k0 < MAXCH; k0 += 8 * 64) {
      if (k0 < full) {
        u4u r[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) r[u] = al[min(k0 + u * 64 + lane, full - 1)];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u)
          if (k0 + u * 64 + lane < full) d4[k0 + u * 64 + lane] = r[u];
      }
    }
  } else {
    for (uint32_t k0 = 0; k0 < MAXCH && k0 < full; k0 += 8 * 64) {
      u4u r[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) r[u] = al[min(k0 + u * 64 + lane, full - 1)];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u)
        if (k0 + u * 64 + lane < full) d4[k0 + u * 64 + lane] = r[u];
    }
  }
  if (full < nch && lane == 0) {
    const uint32_t* q = (const uint32_t*)(al + full);
    const uint32_t lim = delta + P - 4 * full;  // 1..3 valid dwords
    u4u r;
    r.x = q[0];
    r.y = lim > 1 ? q[1] : 0u;
    r.z = lim > 2 ? q[2] : 0u;
    r.w = 0u;
    d4[full] = r;
  }
  return dst + delta;
}

// The stream header's first 16-byte aligned chunk (always readable once the
// header has been checked).
__device__ __forceinline__ const uint32_t* hdr_chunk(const uint8_t* in) {
  return (const uint32_t*)(in + ((0u - (uint32_t)(uintptr_t)in) & 15u));  // keeps in's address space
}

// wave_stage_payload in two parts, so that a superblock's payload is in
// flight while the wave decodes the previous one.  Issue: the first
// PAY_CPL * 64 chunks (PAY_CPL per lane: payloads up to 2048 dwords, ratio
// 2 and up; 12 per lane measured no faster on ratio-1.7 data) and the
// partial last chunk's dwords into registers, every
// load issued whatever the size (clamped to the readable bytes [16-byte
// floor of src, src + P), or to the stream header's first aligned chunk if
// that range is empty), so that each path issues the same memory
// operations.  Commit: those into dst, and any chunks past them copied
// there and then.
constexpr uint32_t PAY_CPL = 8;
struct PayRegs {
  u4u r[PAY_CPL];
  uint32_t t[3];
  const u4u* al;
  uint32_t delta, full, nch, P;
};

__device__ __forceinline__ void wave_pay_issue(const uint32_t* src, uint32_t P, const uint8_t* in,
                                               PayRegs& pr) {
  const uint32_t lane = __lane_id();
  pr.delta = (uint32_t)(((uintptr_t)src & 15u) >> 2);
  pr.al = (const u4u*)(src - pr.delta);
  pr.P = P;
  pr.full = (pr.delta + P) / 4;
  pr.nch = (pr.delta + P + 3) / 4;
  const u4u* safe = (const u4u*)hdr_chunk(in);
  const u4u* base = pr.full ? pr.al : safe;
  const uint32_t last = pr.full ? pr.full - 1 : 0u;
#pragma unroll
  for (uint32_t u = 0; u < PAY_CPL; ++u) pr.r[u] = base[min(u * 64 + lane, last)];
  const uint32_t nd = pr.delta + P;  // readable dwords from al
  const uint32_t* b32 = nd ? (const uint32_t*)pr.al : (const uint32_t*)safe;
  const uint32_t lastd = nd ? nd - 1 : 0u;
#pragma unroll
  for (uint32_t j = 0; j < 3; ++j) pr.t[j] = b32[min(4 * pr.full + j, lastd)];
}

// Returns where src[0] landed in dst (16-byte aligned LDS).
__device__ __forceinline__ const uint32_t* wave_pay_commit(const PayRegs& pr, uint32_t* dst) {
  const uint32_t lane = __lane_id();
  u4u* d4 = (u4u*)dst;
#pragma unroll
  for (uint32_t u = 0; u < PAY_CPL; ++u)
    if (u * 64 + lane < pr.full) d4[u * 64 + lane] = pr.r[u];
  if (pr.full < pr.nch && lane == 0) {
    const uint32_t lim = pr.delta + pr.P - 4 * pr.full;  // 1..3 valid dwords
    u4u r;
    r.x = pr.t[0];
    r.y = lim > 1 ? pr.t[1] : 0u;
    r.z = lim > 2 ? pr.t[2] : 0u;
    r.w = 0u;
    d4[pr.full] = r;
  }
  for (uint32_t k0 = PAY_CPL * 64; k0 < pr.full; k0 += 8 * 64) {
    u4u r[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) r[u] = pr.al[min(k0 + u * 64 + lane, pr.full - 1)];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u)
      if (k0 + u * 64 + lane < pr.full) d4[k0 + u * 64 + lane] = r[u];
  }
  return dst + pr.delta;
}

template <int L, uint32_t OP, uint32_t NOLD>
__device__ __forceinline__ void wave_unpack_store(const Job& J, uint64_t sb, uint32_t nval, float t,
                                                  uint32_t* R, const uint32_t* S,
                                                  const WaveBlocks& wb, const u4u (&old)[NOLD]);

// Decodes superblock sb into J.out (OP 1), or adds it to the fp32 values
// there (OP 3, decode-and-accumulate); false (nothing written) if it is
// malformed.  raw: sb's table and header-byte words (wave_blocks_load), on
// return those of the wave's next superblock nsb (if it exists), whose
// loads go out with this superblock's payload copy.
template <int L, uint32_t OP = 1>
__device__ bool wave_decode_super(const Job& J, const uint8_t* in, uint64_t sb, uint64_t paydw,
                                  float t, uint32_t* R, uint32_t (&raw)[3], uint64_t nsb) {
  constexpr uint32_t CPL = SUPER / 4 / 64;  // 16-byte chunks per lane of a superblock
  const uint32_t lane = __lane_id();
  const uint64_t e0 = sb * SUPER;
  const uint32_t nval = (uint32_t)min((uint64_t)SUPER, J.n - e0);
  uint32_t* d32 = (uint32_t*)((float*)J.out + e0);
  // OP 3: the accumulator of a whole superblock is in flight during the decode
  u4u old[OP == 3 ? CPL : 1];
  if (OP == 3 && nval == SUPER) {
#pragma unroll
    for (uint32_t u = 0; u < CPL; ++u) old[u] = ((const u4u*)d32)[u * 64 + lane];
  }
  WaveBlocks wb;
  const bool ok = wave_blocks_eval<float, L>(J, sb, paydw, nval, raw, wb);
  const uint32_t* S = R;
  if (ok)
    S = wave_stage_payload<SUPER, true>((const uint32_t*)(in + J.pay_off) + wb.E,
                                        (uint32_t)(wb.En - wb.E), R);
  // the next superblock's words are in flight during this one's unpacking
  if (nsb < J.NS) wave_blocks_load<L, false>(J, in, nsb, raw);
  if (!ok) return false;
  wave_unpack_store<L, OP>(J, sb, nval, t, R, S, wb, old);
  return true;
}

// Decodes superblock sb (layout wb, payload staged at S in the wave's
// region R) into J.out (OP 1), or adds it to the fp32 values there (OP 3,
// old: the accumulator's superblock if whole).
template <int L, uint32_t OP, uint32_t NOLD>
__device__ __forceinline__ void wave_unpack_store(const Job& J, uint64_t sb, uint32_t nval, float t,
                                                  uint32_t* R, const uint32_t* S,
                                                  const WaveBlocks& wb, const u4u (&old)[NOLD]) {
  constexpr uint32_t LPB = L / 32, STR = seg_stride<float>();
  constexpr uint32_t CPL = SUPER / 4 / 64;  // 16-byte chunks per lane of a superblock
  const uint32_t lane = __lane_id();
  const uint64_t e0 = sb * SUPER;
  uint32_t* d32 = (uint32_t*)((float*)J.out + e0);
  wave_lds_sync();
  const uint32_t* boff = wb.boff;
  const uint32_t* kind = wb.kind;
  const uint32_t* F = wb.F;
  const bool* ex = wb.ex;
  float v0[32], v1[32];
  {
    const uint32_t seg = lane, w = seg % LPB;
    const uint32_t vc = (uint32_t)min(32, max(0, (int)nval - (int)(seg * 32)));
    if (nval == SUPER) unpack_seg<float, LPB, true>(S + boff[0], kind[0], F[0], w, vc, ex[0], t, v0);
    else unpack_seg<float, LPB, false>(S + boff[0], kind[0], F[0], w, vc, ex[0], t, v0);
  }
  {
    const uint32_t seg = 64 + lane, w = seg % LPB;
    const uint32_t vc = (uint32_t)min(32, max(0, (int)nval - (int)(seg * 32)));
    if (nval == SUPER) unpack_seg<float, LPB, true>(S + boff[1], kind[1], F[1], w, vc, ex[1], t, v1);
    else unpack_seg<float, LPB, false>(S + boff[1], kind[1], F[1], w, vc, ex[1], t, v1);
  }
  wave_lds_sync();  // every lane has read its payload words
  // values into the padded segment layout, then coalesced 16-byte stores
  {
    uint32_t* p0 = R + lane * STR;
    uint32_t* p1 = R + (64 + lane) * STR;
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      p0[i] = __float_as_uint(v0[i]);
      p1[i] = __float_as_uint(v1[i]);
    }
  }
  wave_lds_sync();
  // decoded + old, in fp32 (OP 3)
  auto addf = [](uint32_t a, uint32_t b) { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); };
  if (nval == SUPER) {
#pragma unroll
    for (uint32_t u = 0; u < CPL; ++u) {
      const uint32_t k = u * 64 + lane, dw = 4 * k;
      u4u r = *(const u4u*)(R + (dw / SEG) * STR + dw % SEG);
      if (OP == 3) {
        r.x = addf(r.x, old[u].x);
        r.y = addf(r.y, old[u].y);
        r.z = addf(r.z, old[u].z);
        r.w = addf(r.w, old[u].w);
      }
      ((u4u*)d32)[k] = r;
    }
  } else {
    for (uint32_t k = lane; 4 * k < nval; k += 64) {
      const uint32_t dw = 4 * k;
      u4u r = *(const u4u*)(R + (dw / SEG) * STR + dw % SEG);
      if (dw + 4 <= nval) {
        if (OP == 3) {
          const u4u a = ((const u4u*)d32)[k];
          r.x = addf(r.x, a.x);
          r.y = addf(r.y, a.y);
          r.z = addf(r.z, a.z);
          r.w = addf(r.w, a.w);
        }
        ((u4u*)d32)[k] = r;
      } else {
        if (dw + 0 < nval) d32[dw + 0] = OP == 3 ? addf(r.x, d32[dw + 0]) : r.x;
        if (dw + 1 < nval) d32[dw + 1] = OP == 3 ? addf(r.y, d32[dw + 1]) : r.y;
        if (dw + 2 < nval) d32[dw + 2] = OP == 3 ? addf(r.z, d32[dw + 2]) : r.z;
      }
    }
  }
  wave_lds_sync();  // the region is read before the next superblock's copy-in
}

// One step of wave_decode_whole: commits superblock sb's payload (issued a
// step earlier), evaluates the layout of the next one (its words loaded a
// step earlier), issues that payload and the words after it, then decodes
// and stores sb.
template <int L, bool VEC>
__device__ __forceinline__ void wave_whole_step(const Job& J, const uint8_t* in, uint64_t paydw,
                                                float t, uint32_t* R, uint64_t W, uint64_t NF,
                                                uint64_t sb, const WaveBlocks& wb, PayRegs& pr,
                                                uint32_t (&raw)[3], WaveBlocks& wbn, bool& okn) {
  const uint32_t* pay = (const uint32_t*)(in + J.pay_off);
  const uint32_t* S = wave_pay_commit(pr, R);
  const uint64_t nx = min(sb + W, NF - 1);  // past the end: a whole superblock again, unused
  okn = wave_blocks_eval<float, L, 0, VEC>(J, nx, paydw, SUPER, raw, wbn);
  wave_pay_issue(okn ? pay + wbn.E : hdr_chunk(in), okn ? (uint32_t)(wbn.En - wbn.E) : 0u, in, pr);
  wave_blocks_load<L, false>(J, in, min(nx + W, NF - 1), raw);
  const u4u none[1] = {};
  wave_unpack_store<L, 1>(J, sb, SUPER, t, R, S, wb, none);
}

// The whole superblocks sb, sb + W, ... of an fp32 stream, each one's
// payload in flight while the wave decodes the one before (the first step
// is written out once, so that at the loop's head the same memory
// operations are outstanding on every path: the compiler then waits only
// for the payload, not for the previous superblock's stores).  On return sb
// is the wave's first superblock not decoded; bad is set (and decoding
// stops) at a malformed one.
template <int L, bool VEC = false>
__device__ __forceinline__ void wave_decode_whole(const Job& J, const uint8_t* in, uint64_t paydw,
                                                  float t, uint32_t* R, uint64_t W, uint64_t& sb,
                                                  bool& bad) {
  const uint64_t NF = J.n / SUPER;
  if (sb >= NF) return;
  const uint32_t* pay = (const uint32_t*)(in + J.pay_off);
  uint32_t raw[3];
  wave_blocks_load<L, false>(J, in, sb, raw);
  WaveBlocks wb, wbn;
  bool ok = wave_blocks_eval<float, L, 0, VEC>(J, sb, paydw, SUPER, raw, wb), okn;
  PayRegs pr;
  wave_pay_issue(ok ? pay + wb.E : hdr_chunk(in), ok ? (uint32_t)(wb.En - wb.E) : 0u, in, pr);
  wave_blocks_load<L, false>(J, in, min(sb + W, NF - 1), raw);
  if (!ok) {
    bad = true;
    return;
  }
  wave_whole_step<L, VEC>(J, in, paydw, t, R, W, NF, sb, wb, pr, raw, wbn, okn);
  for (sb += W; sb < NF; sb += W) {
    if (!okn) {
      bad = true;
      return;
    }
    wb = wbn;
    wave_whole_step<L, VEC>(J, in, paydw, t, R, W, NF, sb, wb, pr, raw, wbn, okn);
  }
}

template <int L>
__global__ __launch_bounds__(WaveDec::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_decompress_w(Job J, Ctl C) {
  const uint32_t wid = threadIdx.x >> 6;
  uint32_t* R = g_stage + wid * WaveDec::REGION;
  const uint8_t* in = (const uint8_t*)J.in;
  uint64_t paydw = 0;
  float t = 0;
  bool bad = !wave_header<float>(J, in, paydw, t);
  if (!bad) {
    const uint64_t W = (uint64_t)gridDim.x * (blockDim.x >> 6);
    uint64_t sb = (uint64_t)blockIdx.x * (blockDim.x >> 6) + wid;
    wave_decode_whole<L>(J, in, paydw, t, R, W, sb, bad);
    if (!bad) {  // the partial last superblock
      uint32_t raw[3] = {0u, 0u, 0u};
      if (sb < J.NS) wave_blocks_load<L, false>(J, in, sb, raw);
      for (; sb < J.NS; sb += W)
        if (!wave_decode_super<L>(J, in, sb, paydw, t, R, raw, sb + W)) bad = true;
    }
  }
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

// Single-stream decode-and-accumulate by waves (fp32): as k_decompress_w,
// each superblock added to the accumulator J.out.
template <int L>
__global__ __launch_bounds__(WaveDec::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_accum_w(Job J, Ctl C) {
  const uint32_t wid = threadIdx.x >> 6;
  uint32_t* R = g_stage + wid * WaveDec::REGION;
  const uint8_t* in = (const uint8_t*)J.in;
  uint64_t paydw = 0;
  float t = 0;
  bool bad = !wave_header<float>(J, in, paydw, t);
  if (!bad) {
    const uint64_t W = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const uint64_t sb0 = (uint64_t)blockIdx.x * (blockDim.x >> 6) + wid;
    uint32_t raw[3] = {0u, 0u, 0u};
    if (sb0 < J.NS) wave_blocks_load<L, false>(J, in, sb0, raw);
    for (uint64_t sb = sb0; sb < J.NS; sb += W)
      if (!wave_decode_super<L, 3>(J, in, sb, paydw, t, R, raw, sb + W)) bad = true;
  }
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

// One superblock of a batch job: the job's stream is checked and the superblock
// added to the accumulator.
template <int L>
__device__ __forceinline__ bool wave_accum_super(const Job& J, uint64_t sb, uint32_t* R) {
  const uint64_t off = J.in_off ? J.in_off[J.job] : 0ull;
  Job Jl = J;
  Jl.in_bytes = off <= J.in_bytes ? J.in_bytes - off : 0ull;
  const uint8_t* in = (const uint8_t*)J.in + off;
  uint32_t raw[3];
  wave_blocks_load<L, true>(Jl, in, sb, raw);  // in flight with the header's words
  uint64_t paydw = 0;
  float t = 0;
  if (!wave_header<float>(Jl, in, paydw, t)) return false;
  return wave_decode_super<L, 3>(Jl, in, sb, paydw, t, R, raw, ~0ull);
}

// Superblocks first, first + stride, ... of one fp32 stream (job J, its
// stream at in) by one wave, whole ones pipelined as in k_decompress_w.
template <int L>
__device__ __forceinline__ void wave_job_decode(const Job& J, const uint8_t* in, uint64_t first,
                                                uint64_t stride, uint32_t* R, bool& bad) {
  uint64_t paydw = 0;
  float t = 0;
  if (!wave_header<float, true>(J, in, paydw, t)) {
    bad = true;
    return;
  }
  uint64_t sb = first;
  wave_decode_whole<L, true>(J, in, paydw, t, R, stride, sb, bad);
  if (bad) return;
  uint32_t raw[3] = {0u, 0u, 0u};
  if (sb < J.NS) wave_blocks_load<L, false>(J, in, sb, raw);
  for (; sb < J.NS; sb += stride)
    if (!wave_decode_super<L>(J, in, sb, paydw, t, R, raw, sb + stride)) bad = true;
}

// Batched decoding of fp32 1D jobs by shares: the map holds jw (job, first
// superblock, stride) triples, one per wave's share (waves take them
// statically); each wave decodes superblocks first, first + stride, ... of its
// job with the pipelined single-stream decoder.
__global__ __launch_bounds__(WaveDec::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_batch_decode_w(
    const Job* __restrict__ jobs, const uint32_t* __restrict__ map, uint32_t jw, Ctl C) {
  constexpr uint32_t WAVES = WaveDec::WAVES;
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* R = g_stage + wid * WaveDec::REGION;
  bool bad = false;
  for (uint32_t w = blockIdx.x * WAVES + wid; w < jw; w += gridDim.x * WAVES) {
    Job J = jobs[map[3 * (uint64_t)w]];
    const uint64_t first = map[3 * (uint64_t)w + 1], stride = map[3 * (uint64_t)w + 2];
    const uint64_t off = J.in_off ? J.in_off[J.job] : 0ull;
    J.in_bytes = off <= J.in_bytes ? J.in_bytes - off : 0ull;
    const uint8_t* in = (const uint8_t*)J.in + off;
    bool jb = false;  // this share's job only
    switch (J.log2L) {
      case 5: wave_job_decode<32>(J, in, first, stride, R, jb); break;
      case 6: wave_job_decode<64>(J, in, first, stride, R, jb); break;
      case 7: wave_job_decode<128>(J, in, first, stride, R, jb); break;
      default: jb = true; break;
    }
    bad = bad || jb;
  }
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

// Batched decode-and-accumulate (fp32) by waves: batch superblock i is
// superblock map[2i + 1] of job map[2i], or, without a map (jobs of equal
// superblock counts), superblock i / njobs of job i % njobs; waves take them
// statically.
__global__ __launch_bounds__(WaveDec::WAVES * 64)
__attribute__((amdgpu_waves_per_eu(2, 2))) void k_batch_accum_w(
    const Job* __restrict__ jobs, const uint32_t* __restrict__ map, uint32_t njobs,
    uint32_t total, Ctl C) {
  constexpr uint32_t WAVES = WaveDec::WAVES;
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* R = g_stage + wid * WaveDec::REGION;
  bool bad = false;
  const uint32_t W = gridDim.x * WAVES;
  for (uint32_t i = blockIdx.x * WAVES + wid; i < total; i += W) {
    const uint32_t j = map ? map[2 * (uint64_t)i] : i % njobs;
    const uint64_t sb = map ? map[2 * (uint64_t)i + 1] : i / njobs;
    const Job J = jobs[j];
    bool ok = false;
    switch ((J.dtype << 3) | J.log2L) {
      case 5: ok = wave_accum_super<32>(J, sb, R); break;
      case 6: ok = wave_accum_super<64>(J, sb, R); break;
      case 7: ok = wave_accum_super<128>(J, sb, R); break;
      default: break;
    }
    if (!ok) bad = true;
  }
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

// ---- shared by the per-wave encoders
__device__ __forceinline__ uint32_t lds_load_acq(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store_rel(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Bounded wait until *p >= want (lane 0 polls); false on timeout.
__device__ __forceinline__ bool lds_wait_ge(const Ctl& C, const uint32_t* p, uint32_t want) {
  uint32_t ok = 1;
  if (__lane_id() == 0) {
    uint32_t spins = 0;
    uint64_t t0 = 0;
    while (lds_load_acq(p) < want) {
      if (wait_over(C, ++spins, t0)) {
        atomicOr(&C.ctrl->err, ERRF_TIMEOUT);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return read_lane(ok, 0) != 0;
}

// The lane's share of its block's payload at st (the block's first word):
// base, sign word and planes of an L1D block, or the values of a RAW block
// (from registers, re-derived by the fused step, or re-read from J.in).
template <typename T, int L, bool FUSED, bool FULL, int MODE = 0>
__device__ __forceinline__ void wave_pack(const Job& J, uint64_t seg, uint32_t w, uint32_t vcnt,
                                          const LaneCode& lc, const FusedSrc& fs, uint32_t* st) {
  constexpr uint32_t LPB = L / 32, EW = sizeof(T) / 4;
  if (lc.kind == K_L1D || (MODE == 1 && (lc.kind == K_L2D || lc.kind == K_NONE))) {
    const uint32_t o = MODE == 1 && lc.kind == K_NONE ? 0u : 1u;  // NONE stores no base
    if (o && w == 0) st[0] = (uint32_t)lc.base;
    if (lc.F) {
      st[o + w] = lc.sg;
      put_planes(lc.a, lc.F, st + o + LPB + w, LPB);
    }
  }
  if (FUSED && lc.kind == K_RAW && lc.rawregs) {
#pragma unroll
    for (int i = 0; i < 32; ++i)  // unrolled: a[] stays in registers
      if (FULL || i < (int)vcnt) st[w * 32 + i] = lc.a[i];
  } else if (lc.kind == K_RAW) {  // blocks too wide to code (rare)
    if (FUSED) {
      fused_raw_stage<LPB>(J, fs, seg, w, vcnt, st);
    } else {
      const T* src = (const T*)J.in + seg_first<MODE>(J, seg);
      for (int i = 0; i < (int)vcnt; ++i) {
        uint32_t wd[2];
        raw_words(src[seg_off<MODE>(J, i)], wd);
        st[(w * 32 + i) * EW] = wd[0];
        if (EW == 2) st[(w * 32 + i) * EW + 1] = wd[1];
      }
    }
  }
}

// Mode 1 (fp32, 8x8 tiles, L = 64): lane w of tile seg/2 owns its rows
// 4w..4w+3, loaded/stored as 4 rows of 8 floats.
__device__ __forceinline__ void load_tile(const Job& J, const float* __restrict__ p, bool ex,
                                          float (&v)[32]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f4u t = ex ? *(const f4u*)(p + r * (uint64_t)J.nx + 4 * h) : f4u{0, 0, 0, 0};
      v[8 * r + 4 * h] = t.x; v[8 * r + 4 * h + 1] = t.y;
      v[8 * r + 4 * h + 2] = t.z; v[8 * r + 4 * h + 3] = t.w;
    }
  }
}
__device__ __forceinline__ void store_tile(const Job& J, float* __restrict__ p,
                                           const float (&v)[32]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f4u t;
      t.x = v[8 * r + 4 * h]; t.y = v[8 * r + 4 * h + 1];
      t.z = v[8 * r + 4 * h + 2]; t.w = v[8 * r + 4 * h + 3];
      *(f4u*)(p + r * (uint64_t)J.nx + 4 * h) = t;
    }
  }
}

// ---------------------------------------------------- per-wave fused step
// The fused step of long fp32 streams and large uniform batches (more units than
// one pass of the unit kernel below codes) by single waves, a whole superblock each: eight
// waves a CU with two units' work per claim.  On an 8-rank ring of 256^3 (2048
// waves, two superblocks each) 376 us against 407 us by units, whose 2816
// workers pass over the 8192 units three times; from one pass down the unit
// kernel is the faster (6 ranks of 4 M elements: 166 against 211 us).
// A wave claims a superblock, builds its payload in LDS in two halves of 64
// segments (lane l codes segment 64h + l), learns its offset and writes
// payload, table word and header bytes, with no workgroup barrier.  Offsets
// come from a two-level scan: a workgroup claims rounds of WAVES consecutive
// superblocks with one global ticket; inside a round the waves combine their
// sizes through LDS, and the round is one element of the decoupled look-back.
// Wave region (dwords): X and A, each 64 padded segments, and HB, the
// superblock's header bytes.  The incoming payload is staged in X (whole, or
// half by half if it does not fit); each lane loads its own addend row; the
// first half's sums (kept for RAW blocks) and then payload in A, the second
// half's sums and payload in X.
struct WaveEnc {
  static constexpr uint32_t WAVES = 8;  // per workgroup
  static constexpr uint32_t STR = 36;   // seg_stride<float>()
  static constexpr uint32_t XW = 64 * STR, AW = 64 * STR, HBW = SUPER / 32 / 4;
  static constexpr uint32_t REGION = XW + AW + HBW + 4;
};

// The lane's own row of 32 values at src (vcnt valid, the rest 0): eight
// 16-byte loads, each instruction touching a line per lane, nearly all L1
// hits after the first.
template <bool FULL>
__device__ __forceinline__ void wave_row_load(const uint32_t* src, uint32_t vcnt, u4u (&r)[8]) {
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) {
    if (FULL) {
      r[k] = ((const u4u*)src)[k];
    } else {
      const uint32_t dw = 4 * k;
      if (dw + 4 <= vcnt) {
        r[k] = *(const u4u*)(src + dw);
      } else {
        r[k].x = dw + 0 < vcnt ? src[dw + 0] : 0u;
        r[k].y = dw + 1 < vcnt ? src[dw + 1] : 0u;
        r[k].z = dw + 2 < vcnt ? src[dw + 2] : 0u;
        r[k].w = 0u;
      }
    }
  }
}

__device__ __forceinline__ void wave_row_put(uint32_t* X, const float (&v)[32]) {
  f4u* p = (f4u*)(X + __lane_id() * WaveEnc::STR);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    f4u r;
    r.x = v[4 * k]; r.y = v[4 * k + 1]; r.z = v[4 * k + 2]; r.w = v[4 * k + 3];
    p[k] = r;
  }
}

// The fused step's first words of a superblock (the incoming stream's
// header word of the lane, table and header-byte words), loaded ahead.
struct UnitPre {
  uint32_t wv, raw[3];
  bool valid;
};

template <int L>
__device__ __forceinline__ void wave_unit_preload(const Job& J, uint64_t u, UnitPre& p) {
  const uint8_t* in = (const uint8_t*)J.in;
  wave_blocks_load<L, true>(J, in, u, p.raw);
  p.wv = wave_header_load(J, in);
  p.valid = true;
}

// Encodes superblock u of job J into the wave's region (fused: incoming
// stream J.in plus addend J.local; ahead: its first words if loaded ahead):
// tot[0] payload dwords in A, tot[1] in X, header bytes in HB; good is false
// for a malformed incoming superblock.  pub(size) is called with the whole
// size as soon as it is known, before the second half is packed.
template <int L, bool FULL, class Pub>
__device__ __forceinline__ void wave_encode_unit(const Job& J, uint64_t u, uint32_t* R,
                                                 uint32_t (&tot)[2], bool& good,
                                                 const UnitPre& ahead, const Pub& pub) {
  constexpr uint32_t LPB = L / 32, BPS = SUPER / L, HALF = 64 * SEG;
  const uint32_t lane = __lane_id();
  const uint32_t w = lane & (LPB - 1);
  uint32_t* X = R;
  uint32_t* A = R + WaveEnc::XW;
  uint32_t* HB = A + WaveEnc::AW;
  const uint64_t e0 = u * SUPER;
  const uint32_t nval = FULL ? SUPER : (uint32_t)min((uint64_t)SUPER, J.n - e0);
  const uint8_t* in = (const uint8_t*)J.in;
  // the incoming superblock's layout (fused step)
  good = true;
  WaveBlocks wb = {};
  FusedSrc fs;
  fs.pay = (const uint32_t*)(in + J.pay_off);
  fs.t = 0.0f;
  {
    uint64_t paydw = 0;
    UnitPre p = ahead;
    if (!p.valid) wave_unit_preload<L>(J, u, p);  // table words with the header's
    good = wave_header_eval<float>(J, p.wv, paydw, fs.t);
    if (good) good = wave_blocks_eval<float, L>(J, u, paydw, nval, p.raw, wb);
  }
  // the whole incoming payload is staged at once when its realigned copy
  // fits X (always, at any ratio above about 1.8)
  const uint32_t Ptot = good ? (uint32_t)(wb.En - wb.E) : 0u;
  const bool whole = Ptot + 8 <= WaveEnc::XW;
  const uint32_t* S = X;

#pragma unroll
  for (uint32_t h = 0; h < 2; ++h) {
    const uint32_t hval =
        FULL ? HALF : (uint32_t)min((int)HALF, max(0, (int)nval - (int)(h * HALF)));
    const uint64_t seg = e0 / SEG + 64 * h + lane;
    const uint32_t vcnt = FULL ? 32u : (uint32_t)min(32, max(0, (int)hval - 32 * (int)lane));
    float v[32];
    uint32_t* AD = h ? X : A;  // the sums' rows
    const uint32_t hoff = (h && !whole) ? wb.half0 : 0u;
    if (good && (h == 0 || !whole)) {
      const uint32_t P = whole ? Ptot : (h ? Ptot - wb.half0 : wb.half0);
      S = wave_stage_payload<SUPER, false>(fs.pay + wb.E + hoff, P, X);
    }
    // the lane's own 32 addend values, in flight during the decode (a
    // coalesced load transposed through LDS measured slower here)
    u4u lr[8];
    wave_row_load<FULL>((const uint32_t*)(J.local + e0 + h * HALF) + 32 * lane, vcnt, lr);
    if (good) {
      wave_lds_sync();
      unpack_seg<float, LPB, FULL>(S + (wb.boff[h] - hoff), wb.kind[h], wb.F[h], w, vcnt,
                                   wb.ex[h], fs.t, v);
      fs.di.off_dw = (uint32_t)wb.E + wb.boff[h];
      fs.di.kind = wb.kind[h];
      fs.di.F = wb.F[h];
    } else {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = 0.0f;
      fs.di.off_dw = 0;
      fs.di.kind = K_ZERO;
      fs.di.F = 0;
    }
    wave_lds_sync();  // payload words read before X takes the sums
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // incoming + local, fp32
      v[4 * k] = v[4 * k] + __uint_as_float(lr[k].x);
      v[4 * k + 1] = v[4 * k + 1] + __uint_as_float(lr[k].y);
      v[4 * k + 2] = v[4 * k + 2] + __uint_as_float(lr[k].z);
      v[4 * k + 3] = v[4 * k + 3] + __uint_as_float(lr[k].w);
    }
    wave_row_put(AD, v);  // the sums, for a RAW block (own row)
    LaneCode lc;
    analyze_1d<float, L, FULL, true>(J, seg, w, v, vcnt, lc, AD + lane * WaveEnc::STR);
    const uint32_t contrib = w == 0 ? lc.size_dw : 0u;
    const uint32_t incl = wave_incl_scan(contrib);
    const uint32_t boff = w == 0 ? incl - contrib : incl - lc.size_dw;
    tot[h] = read_lane(incl, 63);
    if (h == 1) pub(tot[0] + tot[1]);
    if (w == 0)
      ((uint8_t*)HB)[(64 * h + lane) / LPB] =
          (uint8_t)(lc.exists ? ((lc.kind << 5) | lc.F) : 0u);
    wave_lds_sync();  // every row of X is read before the second half's payload goes there
    wave_pack<float, L, true, FULL>(J, seg, w, vcnt, lc, fs, (h ? X : A) + boff);
  }
  wave_lds_sync();  // A, X and HB are complete
}

// Writes superblock u's payload (tot[0] dwords from A, tot[1] from X) at
// dword offset ex of the job's payload, its table word and header bytes;
// the job's last superblock also writes the stream header and size.
template <int L>
__device__ __forceinline__ void wave_write_unit(const Job& J, uint64_t u, uint64_t ex,
                                                const uint32_t (&tot)[2], const uint32_t* R) {
  constexpr uint32_t BPS = SUPER / L;
  const uint32_t lane = __lane_id();
  const uint32_t* X = R;
  const uint32_t* A = R + WaveEnc::XW;
  const uint32_t* HB = A + WaveEnc::AW;
  uint8_t* base8 = (uint8_t*)J.out;
  uint32_t* dst = (uint32_t*)(base8 + J.pay_off) + ex;
  for (uint32_t k = lane; k < tot[0]; k += 64) dst[k] = A[k];
  for (uint32_t k = lane; k < tot[1]; k += 64) dst[tot[0] + k] = X[k];
  if (lane == 0) ((uint32_t*)(base8 + HDR))[u] = (uint32_t)ex;
  const uint64_t b0 = u * BPS;
  if (lane < BPS / 4 && b0 + 4 * lane < J.B)
    *(uint32_t*)(base8 + J.hdr_off + b0 + 4 * lane) = HB[lane];
  if (u == J.NS - 1 && lane < 16) {
    const uint64_t payload = 4 * (ex + tot[0] + tot[1]);
    ((uint32_t*)base8)[lane] = hdr_word(J, lane, payload);
    if (lane == 0 && J.out_bytes) *J.out_bytes = J.pay_off + payload;
  }
  wave_lds_sync();  // the region is read before the next superblock reuses it
}

// ---- rounds.  A workgroup's waves claim slots of rounds through an LDS
// counter (claim k: round k / WAVES, slot k % WAVES).  A round's global
// ticket T is taken by the wave that fetched the previous round's prefix,
// right after: the previous round's waves are then about to write and
// claim again, so the ticket is held for about one write-out and the
// round's first claimer need not wait for the atomic (a round past the end
// hands on a ticket past the end; round 0's first claimer takes its own).
// Slot s of the round is superblock WAVES * (T's round within its job) + s.  Per round (a ring of WRING
// entries in LDS): the slots' sizes, a count of them, and the round's
// exclusive prefix, fetched by one elected wave with the look-back over
// rounds.  The wave that completes the count publishes the round's
// aggregate (or its inclusive prefix, if the prefix is known); the fetcher
// publishes the inclusive prefix if the count is complete.  Either way the
// round's status word is published, and an inclusive word is not left
// overwritten by an aggregate (the completer re-checks for the prefix once
// its aggregate store has completed).
// Deadlock freedom: every wait is on earlier rounds (tickets handed to
// running workgroups) or on earlier slots of the same round (claimed
// before, by waves of the same workgroup); the first claimer of a round
// waits for the round WRING earlier in the same entry to be released by all
// its claimers, each of which releases it once.  Nothing assumes that the
// grid's workgroups are resident together, and every wait is bounded.
constexpr uint32_t WRING = 4;
constexpr uint32_t SIZE_NONE = 0xFFFFFFFFu;

struct RoundState {
  unsigned long long prefix;  // exclusive prefix of the round (dwords)
  uint32_t pticket;   // this entry's next round's ticket, taken ahead ...
  uint32_t pflag;     // ... by the previous round: 1 + the round it is for
  uint32_t ticket;
  uint32_t ready;     // 1 + round number once ticket (and the reset) is done
  uint32_t cnt;       // sizes written
  uint32_t fetch;     // 1 once a wave has been elected to fetch the prefix
  uint32_t pready;    // 1 + round number once prefix is set
  uint32_t released;  // claimers done with this entry
  uint32_t size[WaveEnc::WAVES];
};
struct WaveSched {
  uint32_t claim;
  RoundState rs[WRING];
};

// Clears the schedule (before the workgroup's first barrier).
__device__ __forceinline__ void wave_sched_init(WaveSched& ws) {
  if (threadIdx.x == 0) {
    ws.claim = 0;
#pragma unroll
    for (uint32_t i = 0; i < WRING; ++i) {
      ws.rs[i].ready = 0;
      ws.rs[i].pflag = 0;
      ws.rs[i].released = WaveEnc::WAVES;
    }
  }
  __syncthreads();
}

struct Claim {
  uint32_t round, slot, ticket;  // ticket 0xFFFFFFFF: timed out
  bool done;                     // ticket known
};

// A round's first claimer opens it: resets the entry, takes the round's
// ticket (handed on, or, for round 0, from the counter) and marks it ready.
__device__ __forceinline__ uint32_t wave_round_open(const Ctl& C, RoundState& rs,
                                                    uint32_t round) {
  uint32_t t = 0;
  if (__lane_id() == 0) {
    rs.cnt = 0;
    rs.fetch = 0;
    rs.pready = 0;
    rs.released = 0;
#pragma unroll
    for (uint32_t i = 0; i < WaveEnc::WAVES; ++i) rs.size[i] = SIZE_NONE;
    t = round > 0 ? rs.pticket : atomicAdd(&C.ctrl->ticket, 1u);
    rs.ticket = t;
    lds_store_rel(&rs.ready, round + 1);
  }
  return read_lane(t, 0);
}

// Takes the wave's next slot and, if that needs no wait, its round's ticket
// (done); wave_claim_finish completes it otherwise.  A wave may try this
// before releasing its current slot (it waits for nothing), but finishes
// only after the release, so the claim protocol's waits are unchanged.
__device__ __forceinline__ Claim wave_claim_try(const Ctl& C, WaveSched& ws) {
  const uint32_t lane = __lane_id();
  uint32_t k = 0;
  if (lane == 0) k = atomicAdd(&ws.claim, 1u);
  k = read_lane(k, 0);
  Claim c;
  c.round = k / WaveEnc::WAVES;
  c.slot = k % WaveEnc::WAVES;
  c.ticket = 0xFFFFFFFFu;
  c.done = false;
  RoundState& rs = ws.rs[c.round % WRING];
  uint32_t ok = 0;
  if (lane == 0)
    ok = c.slot == 0
             ? (lds_load_acq(&rs.released) >= WaveEnc::WAVES &&
                (c.round == 0 || lds_load_acq(&rs.pflag) >= c.round + 1))
             : lds_load_acq(&rs.ready) >= c.round + 1;
  if (read_lane(ok, 0)) {
    c.ticket = c.slot == 0 ? wave_round_open(C, rs, c.round)
                           : __builtin_amdgcn_readfirstlane(rs.ticket);
    c.done = true;
  }
  return c;
}

__device__ __forceinline__ void wave_claim_finish(const Ctl& C, WaveSched& ws, Claim& c) {
  if (c.done) return;
  c.done = true;
  RoundState& rs = ws.rs[c.round % WRING];
  if (c.slot == 0) {
    // the entry's previous round has been released by all its claimers, and
    // the round's ticket has been handed on by the previous round
    if (!lds_wait_ge(C, &rs.released, WaveEnc::WAVES) ||
        (c.round > 0 && !lds_wait_ge(C, &rs.pflag, c.round + 1)))
      return;  // timed out: ticket stays past the end
    c.ticket = wave_round_open(C, rs, c.round);
    return;
  }
  if (!lds_wait_ge(C, &rs.ready, c.round + 1)) return;
  c.ticket = __builtin_amdgcn_readfirstlane(rs.ticket);
}

__device__ __forceinline__ Claim wave_claim(const Ctl& C, WaveSched& ws) {
  Claim c = wave_claim_try(C, ws);
  wave_claim_finish(C, ws, c);
  return c;
}

// Hands round r + 1 its ticket (lane 0): a fresh one, or t past the end.
__device__ __forceinline__ void wave_hand_on(const Ctl& C, WaveSched& ws, uint32_t r,
                                             uint32_t t, bool fresh) {
  RoundState& nx = ws.rs[(r + 1) % WRING];
  nx.pticket = fresh ? atomicAdd(&C.ctrl->ticket, 1u) : t;
  lds_store_rel(&nx.pflag, r + 2);
}

// The claimer is done with its round's entry.
__device__ __forceinline__ void wave_release(RoundState& rs) {
  if (__lane_id() == 0)
    __hip_atomic_fetch_add(&rs.released, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint32_t round_sum(const RoundState& rs) {
  uint32_t a = 0;
#pragma unroll
  for (uint32_t i = 0; i < WaveEnc::WAVES; ++i) a += rs.size[i];
  return a;
}

// Superblock u (slot cl.slot of round entry rs; u >= J.NS: an empty slot
// past the job's end) of round gs of the chain that starts at chain0:
// encodes it into the wave's region and finds its offset (off, dwords).
// True if the unit is to be written out (wave_write_unit); the caller then
// releases the slot.
template <int L>
__device__ __forceinline__ bool wave_round_begin(const Job& J, uint64_t u, const Claim& cl,
                                                 WaveSched& ws, uint64_t gs, uint64_t chain0,
                                                 const Ctl& C, uint32_t ep, uint32_t* R,
                                                 const UnitPre& pre, uint32_t (&tot)[2],
                                                 uint64_t& off) {
  RoundState& rs = ws.rs[cl.round % WRING];
  const uint32_t lane = __lane_id();
  const bool live = u < J.NS;
  tot[0] = tot[1] = 0u;
  bool good = true;
  // the size into the round; the wave completing the count publishes
  auto pub = [&](uint32_t size) {
    if (lane != 0) return;
    __hip_atomic_store(&rs.size[cl.slot], size, __ATOMIC_RELEASE,
                       __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint32_t c =
        __hip_atomic_fetch_add(&rs.cnt, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) + 1;
    if (c == WaveEnc::WAVES) {
      const uint32_t agg = round_sum(rs);
      if (lds_load_acq(&rs.pready) >= cl.round + 1) {
        st_agent(C.status + gs, sw_pack(2, ep, rs.prefix + agg));
      } else {
        publish_agg(C, gs, chain0, ep, agg);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): that store has completed
        if (lds_load_acq(&rs.pready) >= cl.round + 1)
          st_agent(C.status + gs, sw_pack(2, ep, rs.prefix + agg));
      }
    }
  };
  if (live) {
    if ((u + 1) * SUPER <= J.n) wave_encode_unit<L, true>(J, u, R, tot, good, pre, pub);
    else wave_encode_unit<L, false>(J, u, R, tot, good, pre, pub);
  } else {
    pub(0u);
    return false;
  }
  // the round's prefix: fetched by one wave, read by the others
  uint32_t fetcher = 0;
  if (lane == 0) fetcher = atomicCAS(&rs.fetch, 0u, 1u) == 0u ? 1u : 0u;
  fetcher = read_lane(fetcher, 0);
  bool to = false;
  uint64_t prefix = 0;
  if (fetcher) {
    prefix = lookback<1, false>(C, gs, chain0, ep, 0, to);
    if (lane == 0) {
      rs.prefix = prefix;
      lds_store_rel(&rs.pready, cl.round + 1);
      if (lds_load_acq(&rs.cnt) == WaveEnc::WAVES && !to)
        st_agent(C.status + gs, sw_pack(2, ep, prefix + round_sum(rs)));
      wave_hand_on(C, ws, cl.round, 0, true);
    }
  } else {
    to = !lds_wait_ge(C, &rs.pready, cl.round + 1);
    prefix = rs.prefix;
  }
  // plus the sizes of the round's earlier slots
  uint32_t below = 0;
  if (lane < cl.slot) {
    uint32_t spins = 0;
    uint64_t t0 = 0;
    uint32_t v;
    while ((v = lds_load_acq(&rs.size[lane])) == SIZE_NONE) {
      if (wait_over(C, ++spins, t0)) {
        to = true;
        v = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    below = v;
  }
  to = __ballot(to) != 0;
  below = (uint32_t)wave_sum64(below);
  if (lane == 0) {
    if (to) atomicOr(&C.ctrl->err, ERRF_TIMEOUT);
    if (!good) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
  }
  off = prefix + below;
  return !to && good;
}

#define GZ_WAVE_ATTR __launch_bounds__(WaveEnc::WAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
// Rounds of a job of NS superblocks.
__device__ __forceinline__ uint64_t rounds_of(uint64_t NS) {
  return (NS + WaveEnc::WAVES - 1) / WaveEnc::WAVES;
}

// One stream: round ticket T covers superblocks WAVES * T + slot, look-back
// word T.  Longer streams than one pass of the unit kernel's workers: 2^23, 2^24
// and 2^26 elements 38, 58 and 170 us, by units 45, 61 and 183.
template <int L>
__global__ GZ_WAVE_ATTR void k_fused_w(Job J, Ctl C) {
  __shared__ WaveSched ws;
  wave_sched_init(ws);
  uint32_t* R = g_stage + (threadIdx.x >> 6) * WaveEnc::REGION;
  const uint32_t ep = ld_agent32(&C.ctrl->epoch);
  const uint64_t NR = rounds_of(J.NS);
  Claim cl = wave_claim(C, ws);
  UnitPre pre;
  pre.valid = false;
  for (;;) {
    RoundState& rs = ws.rs[cl.round % WRING];
    if (cl.ticket >= NR) {  // past the end (or timed out)
      if (cl.slot == 0 && __lane_id() == 0) wave_hand_on(C, ws, cl.round, cl.ticket, false);
      wave_release(rs);
      break;
    }
    const uint64_t u = (uint64_t)cl.ticket * WaveEnc::WAVES + cl.slot;
    uint32_t tot[2];
    uint64_t off = 0;
    const bool wr = wave_round_begin<L>(J, u, cl, ws, cl.ticket, 0, C, ep, R, pre, tot, off);
    // the next slot, and its first words ahead of this unit's stores
    Claim nx = wave_claim_try(C, ws);
    pre.valid = false;
    if (nx.done && nx.ticket < NR) {
      const uint64_t v = (uint64_t)nx.ticket * WaveEnc::WAVES + nx.slot;
      if (v < J.NS) wave_unit_preload<L>(J, v, pre);
    }
    if (wr) wave_write_unit<L>(J, u, off, tot, R);
    wave_release(rs);
    wave_claim_finish(C, ws, nx);
    cl = nx;
  }
  epilogue(C);
}

// njobs streams of NS superblocks each (total = njobs x rounds per job),
// every one its own chain: round ticket T is round T / njobs of job
// T % njobs, look-back word j x rounds + round.
template <int L>
__global__ GZ_WAVE_ATTR void k_batch_fused_w(const Job* __restrict__ jobs, uint32_t njobs,
                                              uint32_t total, Ctl C) {
  __shared__ WaveSched ws;
  wave_sched_init(ws);
  uint32_t* R = g_stage + (threadIdx.x >> 6) * WaveEnc::REGION;
  const uint32_t ep = ld_agent32(&C.ctrl->epoch);
  Claim cl = wave_claim(C, ws);
  UnitPre pre;
  pre.valid = false;
  for (;;) {
    RoundState& rs = ws.rs[cl.round % WRING];
    if (cl.ticket >= total) {  // past the end (or timed out)
      if (cl.slot == 0 && __lane_id() == 0) wave_hand_on(C, ws, cl.round, cl.ticket, false);
      wave_release(rs);
      break;
    }
    const uint32_t j = cl.ticket % njobs;
    const Job J = jobs[j];
    const uint64_t NR = rounds_of(J.NS), r = cl.ticket / njobs;
    const uint64_t u = r * WaveEnc::WAVES + cl.slot;
    uint32_t tot[2];
    uint64_t off = 0;
    const bool wr =
        wave_round_begin<L>(J, u, cl, ws, j * NR + r, j * NR, C, ep, R, pre, tot, off);
    // the next slot, and its first words ahead of this unit's stores
    Claim nx = wave_claim_try(C, ws);
    pre.valid = false;
    if (nx.done && nx.ticket < total) {
      const Job& K = jobs[nx.ticket % njobs];
      const uint64_t v = (uint64_t)(nx.ticket / njobs) * WaveEnc::WAVES + nx.slot;
      if (v < K.NS) wave_unit_preload<L>(K, v, pre);
    }
    if (wr) wave_write_unit<L>(J, u, off, tot, R);
    wave_release(rs);
    wave_claim_finish(C, ws, nx);
    cl = nx;
  }
  epilogue(C);
}

// ------------------------------------------------------------ unit encode
// 1D encoding (compression of either type, and the fp32 fused step) by
// single waves.  A wave codes a unit of 64 segments (2048 elements, half a
// superblock; lane l owns segment l): it builds the unit's payload in LDS,
// and writes it, its table word (first half of a superblock) and its header
// bytes once its offset is known.  There is no workgroup barrier, so the waves
// of a CU are in different phases (loads, arithmetic, stores) at once, and a
// short stream spreads over many CUs.
//
// Offsets come from a two-level scan: the W working waves of a workgroup
// code W consecutive units, a round (unit_slot); inside a round
// sizes are combined through LDS, and the round is one element of the
// decoupled look-back, which the workgroup's last wave, the scheduler, runs.
// A worker does not wait for its offset: small payloads are held in LDS, up
// to two of them, while the wave analyses its next units, and written later.
// (A prefix is known once the slowest of the ~4000 units in flight before it
// has published: 4-9 us after a round's own sizes, more than the 6 us a unit
// takes.)  Payloads too large to be held twice are written at once, after a
// wait: holding one of them made the next wait as long and delayed the next
// ticket (2^27 fp32 values at ratio 2: 246 us held, 229 written at once).
//
// Bound by VALU and scalar issue behind the latency of loads and stores, not
// by the prefix: a copy that did not wait for offsets took the same time.
// Before (strips; the fused step by superblocks) and now: 2^14 fp32 values
// 13.9 -> 9.4 us, 20 M fp64 values 85 -> 55.8 us, a batch of 512 mixed requests
// compressed and decompressed 317 -> 228 us, one fused step of 2 M values 24.1 ->
// 16.9 us, a ring Allreduce of 6 x 4 M 215 -> 171 us.  Long fp32 streams are left
// to strips (1 GiB 380 us) and long fused steps to the waves above.
template <bool FUSED>
struct UnitEnc {
  static constexpr uint32_t SEGS = 64;
  // rows of 32 dwords (the fused step's incoming payload, then its addend and
  // sums); compression stages half rows of 16 at a time
  static constexpr uint32_t STR = FUSED ? 36 : 20;
  static constexpr uint32_t XW = SEGS * STR;            // staging (dwords)
  static constexpr uint32_t HBW = SEGS / 4;             // header bytes
  // payloads held, each behind its header bytes
  static constexpr uint32_t QW = FUSED ? 1344 : 1392;
  static constexpr uint32_t HELD = (FUSED ? QW : QW / 2) - HBW;  // largest payload held
  static constexpr uint32_t PACKW = FUSED ? XW : XW + QW;  // payloads not held
  static constexpr uint32_t REGION = XW + QW + HBW;     // per worker
  static constexpr uint32_t MAXW = FUSED ? UNIT_WORKERS_FUSED : UNIT_WORKERS;
};

// 16-byte chunk i = 64 k + lane, k < 8, of 64 rows of 32 dwords that lie
// stride dwords apart at src: row i / 8, chunk i % 8.  vdw: valid dwords from
// src; the rest read as 0.
template <uint32_t STRIDE, bool FULL>
__device__ __forceinline__ void unit_rows_load(const uint32_t* src, uint32_t vdw, u4u (&r)[8]) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) {
    const uint32_t i = 64 * k + lane;
    const uint32_t dw = STRIDE == 32 ? 4 * i : (i / 8) * STRIDE + 4 * (i % 8);
    if (FULL || dw + 4 <= vdw) {
      r[k] = *(const u4u*)(src + dw);
    } else {
      r[k].x = dw + 0 < vdw ? src[dw + 0] : 0u;
      r[k].y = dw + 1 < vdw ? src[dw + 1] : 0u;
      r[k].z = dw + 2 < vdw ? src[dw + 2] : 0u;
      r[k].w = 0u;
    }
  }
}

// Those chunks into rows STR dwords apart in LDS: the whole rows, or half h
// of each (by the lanes that hold it).
template <uint32_t STR>
__device__ __forceinline__ void unit_rows_put(const u4u (&r)[8], uint32_t* X) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) *(u4u*)(X + (8 * k + lane / 8) * STR + 4 * (lane % 8)) = r[k];
}
template <uint32_t STR>
__device__ __forceinline__ void unit_halves_put(const u4u (&r)[8], uint32_t h, uint32_t* X) {
  const uint32_t lane = __lane_id();
  if (((lane >> 2) & 1) == h) {
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) *(u4u*)(X + (8 * k + lane / 8) * STR + 4 * (lane % 4)) = r[k];
  }
}

// The lane's block of unit 2 sb + h of an incoming stream: kind, width and
// offset inside the unit's payload, P dwords at off0 from the payload's start.
// False if superblock sb is malformed.
struct UnitIn {
  uint32_t off0, P, kind, F, boff;
  bool ex;
};

template <typename T, int L, int MODE = 0>
__device__ __forceinline__ bool unit_in_eval(const Job& J, uint64_t sb, uint32_t h,
                                             uint64_t paydw, uint32_t nval,
                                             const uint32_t (&raw)[3], UnitIn& ui) {
  WaveBlocks wb;
  const bool good = wave_blocks_eval<T, L, MODE>(J, sb, paydw, nval, raw, wb);
  ui.kind = h ? wb.kind[1] : wb.kind[0];
  ui.F = h ? wb.F[1] : wb.F[0];
  ui.ex = h ? wb.ex[1] : wb.ex[0];
  ui.boff = h ? wb.boff[1] - wb.half0 : wb.boff[0];
  ui.off0 = (uint32_t)wb.E + (h ? wb.half0 : 0u);
  ui.P = h ? (uint32_t)(wb.En - wb.E) - wb.half0 : wb.half0;
  return good;
}

// Loads and analyses unit u of job J (fused: incoming stream J.in plus
// addend J.local): the lane's code lc and, for RAW blocks of the fused step,
// its source fs.  X is free for the payload afterwards.
template <typename T, int L, bool FUSED, bool FULL, int MODE>
__device__ __forceinline__ void unit_analyse(const Job& J, uint64_t u, uint32_t w, uint32_t vcnt,
                                             uint32_t* X, LaneCode& lc, FusedSrc& fs,
                                             bool& good, const uint32_t* wts) {
  constexpr uint32_t LPB = L / 32, EW = sizeof(T) / 4, STR = UnitEnc<FUSED>::STR;
  const uint32_t lane = __lane_id();
  const uint64_t e0 = u * (uint32_t)UNIT_ELEMS, seg = u * 64 + lane;
  const uint32_t hval = FULL ? (uint32_t)UNIT_ELEMS : (uint32_t)min((uint64_t)(uint32_t)UNIT_ELEMS, J.n - e0);
  good = true;
  if constexpr (MODE == 1) {
    const bool ex = FULL || (seg >> 1) < J.B;
    float v[32];
    load_tile(J, (const float*)J.in + (ex ? seg_first<1>(J, seg) : 0), ex, v);
    analyze_tile(J, w, v, ex, wts, lc);
  } else if constexpr (FUSED) {
    const uint8_t* in = (const uint8_t*)J.in;
    const uint64_t sb = u >> 1;
    // an empty stream (n = 0) is its header: it has no table entry or header
    // byte to read, and what lies behind it in the buffer is not looked at
    const bool some = FULL || J.NS != 0;
    uint32_t raw[3];
    const uint32_t hdr = wave_header_load(J, in);
    if (some) wave_blocks_load<L, true>(J, in, sb, raw);  // table words with the header's
    u4u lr[8];  // the unit's addend, in flight until the add
    unit_rows_load<32, FULL>((const uint32_t*)(J.local + e0), hval, lr);
    uint64_t paydw = 0;
    good = wave_header_eval<float>(J, hdr, paydw, fs.t);
    UnitIn ui = {0u, 0u, K_ZERO, 0u, 0u, false};
    if (good && some)
      good = unit_in_eval<float, L>(J, sb, (uint32_t)(u & 1), paydw,
                             (uint32_t)min((uint64_t)SUPER, J.n - sb * SUPER), raw, ui);
    fs.pay = (const uint32_t*)(in + J.pay_off);
    float v[32];
    if (good) {
      const uint32_t* S = wave_stage_payload<(uint32_t)UNIT_ELEMS, false>(fs.pay + ui.off0, ui.P, X);
      wave_lds_sync();
      unpack_seg<float, LPB, FULL>(S + ui.boff, ui.kind, ui.F, w, vcnt, ui.ex, fs.t, v);
      fs.di.off_dw = ui.off0 + ui.boff;
      fs.di.kind = ui.kind;
      fs.di.F = ui.F;
    } else {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = 0.0f;
      fs.di.off_dw = 0;
      fs.di.kind = K_ZERO;
      fs.di.F = 0;
    }
    // the addend through X (each lane reading its own row from memory touches
    // 64 lines per load, and at 12 waves a CU the L1 does not hold them until
    // the row's last load: a ring step 62 -> 51 us)
    wave_lds_sync();  // payload words read before X takes the addend
    unit_rows_put<STR>(lr, X);
    wave_lds_sync();
    {
      f4u* p = (f4u*)(X + lane * STR);
#pragma unroll
      for (int k = 0; k < 8; ++k) {  // incoming + local, fp32; the sum stays for RAW blocks
        f4u r = p[k];
        r.x = v[4 * k] = v[4 * k] + r.x;
        r.y = v[4 * k + 1] = v[4 * k + 1] + r.y;
        r.z = v[4 * k + 2] = v[4 * k + 2] + r.z;
        r.w = v[4 * k + 3] = v[4 * k + 3] + r.w;
        p[k] = r;
      }
    }
    analyze_1d<float, L, FULL, true>(J, seg, w, v, vcnt, lc, X + lane * STR);
  } else {
    // half rows of 16 dwords at a time through LDS (16 fp32 or 8 fp64 values),
    // so that payloads of earlier units can be held there; fp64's second 32
    // dwords of each row are loaded while the first are quantised
    const uint32_t* src = (const uint32_t*)((const T*)J.in + e0);
    const uint32_t vdw = hval * EW;
    u4u r[8];
    unit_rows_load<32 * EW, FULL>(src, vdw, r);
    QBad<T> qb;
#pragma unroll
    for (uint32_t p = 0; p < 2 * EW; ++p) {
      constexpr uint32_t HV = 16 / EW;  // values per half row
      unit_halves_put<STR>(r, p & 1, X);
      if (EW == 2 && p == 1) unit_rows_load<32 * EW, FULL>(src + 32, vdw > 32 ? vdw - 32 : 0u, r);
      wave_lds_sync();
      T val[HV];
      const u4u* row = (const u4u*)(X + lane * STR);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u4u d = row[k];
        const uint32_t wd[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (uint32_t i = 0; i < 4 / EW; ++i) val[4 / EW * k + i] = from_raw(wd + EW * i, T());
      }
      wave_lds_sync();  // read before the next half rows go there
      quant_run<HV, FULL>(val, J, vcnt > HV * p ? vcnt - HV * p : 0u, lc.a + HV * p, qb);
    }
    analyze_q<EW, L, FULL, false>(J, seg, w, qb.any(bad_bound<T>(J)), vcnt, lc);
  }
}

// ---- rounds.  A workgroup's state: a ring of RING rounds in LDS and the
// launch's epoch.  Round k of the workgroup (k = 0, 1, ...) sits in entry
// k % RING.  From the moment that the ticket of round k + 1 is taken, every later
// round's prefix waits for round k + 1's sizes; so it is taken when no worker of
// the workgroup has a wait for a prefix before its next size: by the worker that
// publishes last in round k (in flight while it packs), if all sizes are small
// enough to be held, else by the scheduler once it has the round's prefix.  Taken
// at the first publication, tickets were held through such waits where large and
// small payloads alternate, and each of them delayed the whole chain (2^28 fp32
// values, half of the units large: 6058 us, now 447; a thousandth large: 1095,
// now 394; 2^27 of ratio 2.8: 1815, now 233; all small or all large: the same).
// Launches that give no workgroup a second round, and batches of short chains
// until a workgroup meets a large payload (unit_early), take the ticket at the
// first publication all the same, unless that payload is large.  Whoever takes it opens the round's entry.  The worker
// that publishes last also publishes the round's sum; the scheduler then runs the
// look-back and puts the round's prefix into the entry.
// Round k + 1 is opened once every worker has published round k - 1 and the
// scheduler is done with round k + 1 - RING (ring_need).
// Deadlock freedom: a worker waits for the offset of a round only after
// publishing it, and prefixes depend on earlier tickets only; tickets are
// handed only to running workgroups, nothing assumes that the grid's
// workgroups are resident together, and every wait is bounded.  Opening round
// k + 1 with its ticket in hand waits for the scheduler's look-back of an
// earlier round, on earlier tickets only.
// Every workgroup takes exactly one ticket past the end, so the last of them
// (total + workgroups - 1) ends the launch's use of the counter: its taker
// resets counter and epoch for the next launch.
constexpr uint32_t UNIT_PUB = 256;

struct URound {
  unsigned long long prefix;  // exclusive prefix of the round (dwords)
  unsigned long long pj;      // the chain's prefix at the job's first round
  uint32_t ticket;
  uint32_t ready;   // 1 + round number once ticket (and the reset) is done
  uint32_t cnt;     // UNIT_PUB for each size written, and 1 for each of them too large to be held
  uint32_t pready;  // 1 + round number once prefix is set: the scheduler's mark
  uint32_t bad;     // 1: the prefix is not to be used (a wait expired)
  uint32_t claim;   // 1 once a worker has claimed the next round's ticket
  uint32_t agg;     // 1 + round number once its aggregate's store has completed
  uint32_t size[16];
};
struct USched {
  uint32_t epoch;
  uint32_t early; // batches: 1 while a round's first worker takes the next ticket
  uint32_t over;  // 1 once this workgroup has taken a ticket past the end
  URound rs[RING];
};

// Ticket t has been taken (lane 0): the launch's last one resets the counter.
__device__ __forceinline__ void unit_taken(const Ctl& C, USched& us, uint32_t t, uint32_t total) {
  if (t < total) return;
  us.over = 1;
  if (t == total + gridDim.x - 1) {
    atomicExch(&C.ctrl->ticket, 0u);
    atomicAdd(&C.ctrl->epoch, 1u);
  }
}

// Opens round k with ticket t (lane 0).
__device__ __forceinline__ void unit_open(const Ctl& C, USched& us, uint32_t k, uint32_t t,
                                          uint32_t total) {
  unit_taken(C, us, t, total);
  URound& e = us.rs[k % RING];
  e.cnt = 0;
  e.bad = 0;
  e.claim = 0;
  e.ticket = t;
  lds_store_rel(&e.ready, k + 1);
}

__device__ __forceinline__ void unit_begin(const Ctl& C, USched& us, uint32_t total) {
  if (threadIdx.x == 0) {
    us.epoch = ld_agent32(&C.ctrl->epoch);  // in hand before this workgroup's last ticket
    us.over = 0;
#pragma unroll
    for (uint32_t i = 0; i < RING; ++i) us.rs[i].ready = us.rs[i].pready = us.rs[i].agg = 0;
    unit_open(C, us, 0, atomicAdd(&C.ctrl->ticket, 1u), total);
  }
  __syncthreads();
}

__device__ __forceinline__ void unit_end(const Ctl& C, USched& us, uint32_t total) {
  __syncthreads();
  if (threadIdx.x == 0)
    while (!us.over) unit_taken(C, us, atomicAdd(&C.ctrl->ticket, 1u), total);  // after a timeout
}

// True for one of those who ask for the next ticket in round entry e.
__device__ __forceinline__ bool unit_claim(URound& e) {
  uint32_t won = 0;
  if (__lane_id() == 0) won = atomicCAS(&e.claim, 0u, 1u) == 0u ? 1u : 0u;
  return read_lane(won, 0) != 0;
}

// A round's place in its chain.
struct UChain {
  uint64_t gs, chain0;  // look-back words of the round and the chain's start
  uint64_t r;           // round of the job
  uint32_t job;
  bool packed;          // the chain runs through several jobs
};

// The scheduler's step for round k: sizes, look-back, prefix.  False once a
// wait expired.
__device__ __forceinline__ bool unit_sched(const Ctl& C, USched& us, uint32_t k, uint32_t W,
                                           uint32_t total, const UChain& ch) {
  URound& e = us.rs[k % RING];
  const uint32_t lane = __lane_id(), ep = us.epoch;
  if (!lds_wait_ge(C, &e.cnt, W * UNIT_PUB)) return false;
  const uint32_t cnt = __builtin_amdgcn_readfirstlane(e.cnt);
  const uint64_t agg = wave_sum64(lane < W ? e.size[lane] : 0u);
  bool to = false;
  const uint64_t prefix = lookback<LB_SUB, false>(C, ch.gs, ch.chain0, ep, agg, to);
  uint64_t pj = 0;
  if (ch.packed) {
    if (ch.r == 0) {
      if (lane == 0 && !to) st_agent(C.jobbase + ch.job, sw_pack(2, ep, prefix));
      pj = prefix;
    } else if (!to) {
      pj = job_base_wait(C, ch.job, ep, to);
    }
  }
  if (lane == 0) {
    if (to) atomicOr(&C.ctrl->err, ERRF_TIMEOUT);
    e.bad = to ? 1u : 0u;
    e.prefix = prefix;
    e.pj = pj;
    lds_store_rel(&e.pready, k + 1);
  }
  // a round with a payload too large to be held: the next ticket, unless its
  // first worker has it
  const bool taker = (cnt % UNIT_PUB) != 0 && unit_claim(e);
  uint32_t tk = 0;
  if (taker && lane == 0) tk = atomicAdd(&C.ctrl->ticket, 1u);
  // the inclusive prefix, once the aggregate cannot land after it (the head
  // of a chain publishes its inclusive prefix as its aggregate)
  if (ch.gs != ch.chain0 && !to && lds_wait_ge(C, &e.agg, k + 1) && lane == 0)
    st_agent(C.status + ch.gs, sw_pack(2, ep, prefix + agg));
  if (taker && lane == 0) unit_open(C, us, k + 1, tk, total);
  return true;
}

// A coded unit that is held until its offset is known: its header bytes at Q +
// at, then size dwords of payload.
struct UnitHeld {
  uint32_t at, size, k, job;    // k: round of the workgroup
  uint64_t u;                   // unit of the job
};
// Up to two of them, h0 the older.
struct UnitQueue {
  UnitHeld h0, h1;
  uint32_t n;
};

// The worker's unit of round k: in turn from either end, so that the units of
// consecutive rounds of short jobs (one live unit or a few) go to different
// workers, which code two rounds at once (4096 jobs of 200 values: fp32 108 -> 88
// us, fp64 141 -> 102; of 6000 values 110 -> 93 and 137 -> 106).
__device__ __forceinline__ uint32_t unit_slot(uint32_t wid, uint32_t k, uint32_t W) {
  return k & 1 ? W - 1 - wid : wid;
}

// Unit u's offset in its job's payload (dwords); pj: the chain's prefix at
// the job's first round.  False if a wait expired.
__device__ __forceinline__ bool unit_offset(const Ctl& C, USched& us, uint32_t k, uint32_t slot,
                                            uint64_t& off, uint64_t& pj) {
  URound& e = us.rs[k % RING];
  const uint32_t lane = __lane_id();
  if (!lds_wait_ge(C, &e.pready, k + 1) || e.bad) return false;
  pj = e.pj;
  // plus the round's earlier units (all sizes are there once the prefix is)
  off = e.prefix - pj + wave_sum64(lane < slot ? e.size[lane] : 0u);
  return true;
}

// Table word, header bytes and, for the job's last unit, stream header and
// size outputs of unit u (size dwords at off); returns where its payload goes.
template <int L>
__device__ __forceinline__ uint32_t* unit_meta(const Job& J, uint64_t u, uint64_t off, uint64_t pj,
                                               uint32_t size, uint32_t hb) {
  constexpr uint32_t BPU = UNIT_ELEMS / L;
  const uint32_t lane = __lane_id();
  uint8_t* base8 = (uint8_t*)J.out + J.fixed_off + 4 * pj;
  if (lane == 0 && !(u & 1) && (u >> 1) < J.NS) ((uint32_t*)(base8 + HDR))[u >> 1] = (uint32_t)off;
  const uint64_t b0 = u * BPU;
  if (lane < BPU / 4 && b0 + 4 * lane < J.B)
    *(uint32_t*)(base8 + J.hdr_off + b0 + 4 * lane) = hb;
  if ((u + 1) * UNIT_ELEMS >= J.n && lane < 16) {  // the last unit
    const uint64_t payload = 4 * (off + size);
    ((uint32_t*)base8)[lane] = hdr_word(J, lane, payload);
    if (lane == 0) {
      if (J.out_bytes) *J.out_bytes = J.pay_off + payload;
      if (J.chunk_off) *J.chunk_off = J.fixed_off + 4 * pj;
    }
  }
  return (uint32_t*)(base8 + J.pay_off) + off;
}

// Writes the oldest held unit (of job J).
__device__ __forceinline__ void unit_flush(const Job& J, const Ctl& C, USched& us, uint32_t wid,
                                           uint32_t W, const uint32_t* Q, UnitQueue& q) {
  const UnitHeld h = q.h0;
  q.h0 = q.h1;
  --q.n;
  uint64_t off, pj;
  if (!unit_offset(C, us, h.k, unit_slot(wid, h.k, W), off, pj)) return;
  const uint32_t hb = Q[h.at + (__lane_id() & 15)];
  const uint32_t* pay = Q + h.at + 16;
  uint32_t* dst = J.log2L == 5   ? unit_meta<32>(J, h.u, off, pj, h.size, hb)
                  : J.log2L == 6 ? unit_meta<64>(J, h.u, off, pj, h.size, hb)
                                 : unit_meta<128>(J, h.u, off, pj, h.size, hb);
  for (uint32_t i = __lane_id(); i < h.size; i += 64) dst[i] = pay[i];
}

// One unit: round k of the workgroup is round r of job J (index job); worker
// wid codes its slot's unit W r + slot (past the job's end: an empty slot).  flush(q)
// writes the oldest unit held.
template <typename T, int L, bool FUSED, bool FULL, int MODE, class Flush>
__device__ __forceinline__ void unit_code(const Job& J, uint32_t job, uint64_t gs, uint64_t u,
                                          bool live, uint32_t k, uint32_t slot, uint32_t W,
                                          uint32_t total, bool batch, USched& us, const Ctl& C,
                                          uint32_t* X, UnitQueue& q, const Flush& flush,
                                          const uint32_t* wts) {
  using U = UnitEnc<FUSED>;
  constexpr uint32_t LPB = L / 32;
  const uint32_t lane = __lane_id(), w = lane & (LPB - 1);
  uint32_t* Q = X + U::XW;
  uint32_t* HB = Q + U::QW;
  const uint64_t e0 = u * UNIT_ELEMS, seg = u * U::SEGS + lane;
  LaneCode lc;
  FusedSrc fs;
  uint32_t size = 0, boff = 0, vcnt = 32;
  bool good = true;
  // a unit's size is on every later round's way: it goes before packing and
  // writing on the same SIMD (ring Reduce_scatter by units 423 -> 402 us)
  __builtin_amdgcn_s_setprio(2);
  if (live) {
    if (!FULL)
      vcnt = (uint32_t)min((int64_t)32, max((int64_t)0, (int64_t)(J.n - e0) - 32 * (int64_t)lane));
    unit_analyse<T, L, FUSED, FULL, MODE>(J, u, w, vcnt, X, lc, fs, good, wts);
    const uint32_t contrib = w == 0 ? lc.size_dw : 0u;
    const uint32_t incl = wave_incl_scan(contrib);
    boff = w == 0 ? incl - contrib : incl - lc.size_dw;
    size = read_lane(incl, 63);
  }
  __builtin_amdgcn_s_setprio(0);
  URound& e = us.rs[k % RING];
  uint32_t c = 0;
  if (lane == 0) {
    e.size[slot] = size;
    const uint32_t add = UNIT_PUB + (size > U::HELD ? 1u : 0u);
    c = add + __hip_atomic_fetch_add(&e.cnt, add, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // the round's last size: publish their sum at once (the scheduler may still
  // be in the look-back of the round before, which must not hold it up)
  c = read_lane(c, 0);
  const bool held = size <= U::HELD;
  // (workers of a round may see us.early before and after a change: if both the
  // first and the last ask, the claim settles it; if neither does, the change
  // came from a payload of this round, and the scheduler asks)
  const bool early = total <= gridDim.x ||
                     (batch && __builtin_amdgcn_readfirstlane(us.early) != 0);
  if (batch && !held && lane == 0) us.early = 0;
  auto open = [&](uint32_t t) {  // once the next round's entry is free
    const RingNeed n = ring_need(k + 1);
    const bool free = (!n.published || lds_wait_ge(C, &us.rs[n.pub].cnt, W * UNIT_PUB)) &&
                      (!n.scheduled || lds_wait_ge(C, &us.rs[n.sched].pready, n.mark));
    if (lane == 0) {
      if (free) unit_open(C, us, k + 1, t, total);
      else unit_taken(C, us, t, total);
    }
  };
  if (c / UNIT_PUB == W) {
    const uint64_t agg = wave_sum64(lane < W ? e.size[lane] : 0u);
    if (lane == 0) {
      publish_agg(C, gs, J.chain0, us.epoch, agg);
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): that store has completed
      lds_store_rel(&e.agg, k + 1);
    }
  }
  // the next ticket is this worker's to take: the first one's (early) or the
  // last one's, while no size so far is too large to be held
  const bool taker = c == (early ? UNIT_PUB : W * UNIT_PUB) && unit_claim(e);
  // room for this unit's payload: held ones lie at the two ends of Q, so that
  // two fit whenever their sizes' sum does (laid one behind the other, a third
  // often fitted neither before nor behind the second, which then had to be
  // waited for: 2^27 fp32 values of ratio 3.6 458 us, now 212).  Units of two
  // rounds ago and older are written whatever the room (a worker may be past the
  // end of many short jobs in a row, and their rounds' entries are reused)
  uint32_t at = 0;
  if (!held) {
    while (q.n) flush(q);
  } else {
    while (q.n && (q.n == 2 || q.h0.k + 1 < k)) flush(q);
    if (q.n) {
      if (q.h0.size + size + 2 * U::HBW <= U::QW) at = q.h0.at ? 0u : U::QW - U::HBW - size;
      else flush(q);
    }
  }
  uint32_t tk = 0;
  if (taker) {
    if (lane == 0) tk = atomicAdd(&C.ctrl->ticket, 1u);  // in flight while packing
    if (!live) open(tk);
  }
  if (!live) return;
  if (!good && lane == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
  wave_lds_sync();  // every row of X is read before the payload goes there
  if (w == 0)
    ((uint8_t*)(held ? Q + at : HB))[lane / LPB] =
        (uint8_t)(lc.exists ? ((lc.kind << 5) | lc.F) : 0u);
  if (held) {
    wave_pack<T, L, FUSED, FULL, MODE>(J, seg, w, vcnt, lc, fs, Q + at + U::HBW + boff);
    if (taker) open(tk);
    wave_lds_sync();  // payload and header bytes are complete
    if (good) {
      const UnitHeld h = {at, size, k, job, u};
      if (q.n) q.h1 = h;  // (not an indexed array: that would live in memory)
      else q.h0 = h;
      ++q.n;
    }
    return;
  }
  // too large to hold: written at once.  An fp64 payload may exceed X: then
  // it is packed in two halves of 32 lanes (no block crosses them).
  const uint32_t lo = sizeof(T) == 8 ? read_lane(boff, 32) : 0u;
  const bool two = sizeof(T) == 8 && size > U::PACKW;
  if (!two) wave_pack<T, L, FUSED, FULL, MODE>(J, seg, w, vcnt, lc, fs, X + boff);
  wave_lds_sync();
  uint64_t off, pj;
  const bool known = unit_offset(C, us, k, slot, off, pj);
  if (!known || !good) return;
  uint32_t* dst = unit_meta<L>(J, u, off, pj, size, HB[lane & (U::HBW - 1)]);
  if (!two) {
    for (uint32_t i = lane; i < size; i += 64) dst[i] = X[i];
  } else {
#pragma unroll 1
    for (uint32_t p = 0; p < 2; ++p) {
      const uint32_t o = p ? lo : 0u, m = p ? size - lo : lo;
      if ((lane >> 5) == p) wave_pack<T, L, FUSED, FULL, MODE>(J, seg, w, vcnt, lc, fs, X + boff - o);
      wave_lds_sync();
      for (uint32_t i = lane; i < m; i += 64) dst[o + i] = X[i];
      wave_lds_sync();
    }
  }
  wave_lds_sync();  // the region is read before the next unit reuses it
}

template <typename T, int L, bool FUSED, int MODE = 0, class Flush>
__device__ __forceinline__ void unit_one(const Job& J, uint32_t job, uint64_t r, uint32_t k,
                                         uint32_t wid, uint32_t W, uint32_t total, bool early, USched& us,
                                         const Ctl& C, uint32_t* X, UnitQueue& q,
                                         const Flush& flush,
                                         const uint32_t* wts = nullptr) {
  const uint32_t slot = unit_slot(wid, k, W);
  const uint64_t u = r * W + slot;
  // an empty stream is one unit of no values
  const bool live = u == 0 || u * UNIT_ELEMS < J.n;
  if ((u + 1) * UNIT_ELEMS <= J.n)
    unit_code<T, L, FUSED, true, MODE>(J, job, J.strip0 + r, u, live, k, slot, W, total, early, us, C, X, q, flush, wts);
  else
    unit_code<T, L, FUSED, false, MODE>(J, job, J.strip0 + r, u, live, k, slot, W, total, early, us, C, X, q, flush, wts);
}

// Registers for four waves per SIMD (the fused step: three), as the LDS allows.
#define GZ_UNIT_ATTR(FUSED)                                        \
  __launch_bounds__((UnitEnc<FUSED>::MAXW + 1) * 64)               \
      __attribute__((amdgpu_waves_per_eu((FUSED) ? 3 : 4, (FUSED) ? 3 : 4)))

// One stream: round ticket t is round t of the job.
template <typename T, int L, bool FUSED>
__global__ GZ_UNIT_ATTR(FUSED) void k_unit(Job J, Ctl C) {
  __shared__ USched us;
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t W = (blockDim.x >> 6) - 1, total = J.nstrips;
  unit_begin(C, us, total);
  if (wid == W) {
    __builtin_amdgcn_s_setprio(3);
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      if (!unit_sched(C, us, k, W, total, UChain{t, 0, t, 0, false})) break;
    }
  } else {
    uint32_t* X = g_stage + wid * UnitEnc<FUSED>::REGION;
    UnitQueue q;
    q.n = 0;
    auto flush = [&](UnitQueue& x) { unit_flush(J, C, us, wid, W, X + UnitEnc<FUSED>::XW, x); };
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      unit_one<T, L, FUSED>(J, 0, t, k, wid, W, total, false, us, C, X, q, flush);
    }
    while (q.n) flush(q);
  }
  unit_end(C, us, total);
}

// One field of 8x8 tiles: a unit's lanes load their rows straight from the
// field.  Bound by VALU issue (the selector's features and network, or three
// predictors).  33 M values with the learned selector: compressed 108 -> 82 us
// against 256-thread strips (both ways 189 -> 124; 128-131 us with 11 workers).
__global__ GZ_UNIT_ATTR(false) void k_unit_tiles(Job J, Ctl C) {
  __shared__ USched us;
  __shared__ uint32_t wts[192];
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t W = (blockDim.x >> 6) - 1, total = J.nstrips;
  for (uint32_t k = threadIdx.x; k < 189; k += blockDim.x) wts[k] = ((const uint32_t*)C.blob)[k];
  unit_begin(C, us, total);  // ends with a barrier
  if (wid == W) {
    __builtin_amdgcn_s_setprio(3);
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      if (!unit_sched(C, us, k, W, total, UChain{t, 0, t, 0, false})) break;
    }
  } else {
    uint32_t* X = g_stage + wid * UnitEnc<false>::REGION;
    UnitQueue q;
    q.n = 0;
    auto flush = [&](UnitQueue& x) { unit_flush(J, C, us, wid, W, X + UnitEnc<false>::XW, x); };
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      unit_one<float, 64, false, 1>(J, 0, t, k, wid, W, total, false, us, C, X, q, flush, wts);
    }
    while (q.n) flush(q);
  }
  unit_end(C, us, total);
}

// A batch: ticket t is round map[2t + 1] of job map[2t], or, for jobs of the
// same number of rounds (njobs > 0), round t / njobs of job t % njobs.
template <uint32_t OP, bool WIDE>
__global__ GZ_UNIT_ATTR(OP == 2) void k_batch_unit(const Job* __restrict__ jobs,
                                                   const uint32_t* __restrict__ map,
                                                   uint32_t njobs, uint32_t total,
                                                   uint32_t early, Ctl C) {
  constexpr bool FUSED = OP == 2;
  __shared__ USched us;
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t W = (blockDim.x >> 6) - 1;
  if (threadIdx.x == 0) us.early = early;
  unit_begin(C, us, total);
  if (wid == W) {
    __builtin_amdgcn_s_setprio(3);
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      const uint32_t j = njobs ? t % njobs : map[2 * (uint64_t)t];
      const uint64_t r = njobs ? t / njobs : map[2 * (uint64_t)t + 1];
      const Job& J = jobs[j];
      if (!unit_sched(C, us, k, W, total,
                      UChain{J.strip0 + r, J.chain0, r, j, J.chain0 != J.strip0}))
        break;
    }
  } else {
    uint32_t* X = g_stage + wid * UnitEnc<FUSED>::REGION;
    UnitQueue q;
    q.n = 0;
    auto flush = [&](UnitQueue& x) {
      unit_flush(jobs[x.h0.job], C, us, wid, W, X + UnitEnc<FUSED>::XW, x);
    };
    for (uint32_t k = 0;; ++k) {
      if (!lds_wait_ge(C, &us.rs[k % RING].ready, k + 1)) break;
      const uint32_t t = __builtin_amdgcn_readfirstlane(us.rs[k % RING].ticket);
      if (t >= total) break;
      const uint32_t j = njobs ? t % njobs : map[2 * (uint64_t)t];
      const uint64_t r = njobs ? t / njobs : map[2 * (uint64_t)t + 1];
      const Job J = jobs[j];
      switch ((J.dtype << 3) | J.log2L) {
        case 5: unit_one<float, 32, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        case 6: unit_one<float, 64, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        case 7: unit_one<float, 128, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        case 13: if constexpr (WIDE) unit_one<double, 32, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        case 14: if constexpr (WIDE) unit_one<double, 64, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        case 15: if constexpr (WIDE) unit_one<double, 128, FUSED>(J, j, r, k, wid, W, total, true, us, C, X, q, flush); break;
        default: break;
      }
    }
    while (q.n) flush(q);
  }
  unit_end(C, us, total);
}

// ------------------------------------------------------------ unit decode
// Decoding by single waves, a unit of 2048 elements each: 8x8 tiles, batches
// that hold fp64 jobs, and medium streams.  Units are independent (a
// superblock's offset is its table entry, its second unit's follows from the
// header bytes, which both units check whole), so waves take them statically.
// A unit needs 9 KB of LDS (payload, then rows of values for coalesced stores;
// fp64 rows 16 values at a time) and 128 registers: four waves per SIMD, where
// the superblock decoder above has two (fp64, before, one; tiles, before, three
// in 256-thread strips with barriers).  Bound by HBM for long fp64 streams,
// by the two dependent loads of a unit for short ones.  20 M fp64 values 46 ->
// 37.4 us, 8 M tile values 50.5 -> 20.8 us, 4096 mixed requests 55 -> 34 us;
// fp32 streams of 2^20 / 2^22 / 2^24 / 2^26 / 2^28 elements 10.1 / 11.2 / 19.5 / 68 /
// 266 us by superblocks, 9.3 / 10.1 / 18.4 / 75 / 283 us by units.
struct UnitDec {
  static constexpr uint32_t STR = 36, XW = 64 * STR, WAVES = 4;  // region (dwords), per workgroup
};

// The lane's quantised values of a block that is not RAW, from its words at pw.
template <int LPB>
__device__ __forceinline__ void unpack_q(const uint32_t* pw, uint32_t kind, uint32_t F, uint32_t w,
                                         bool exists, uint32_t (&a)[32]) {
  const bool z = kind == K_ZERO || kind == K_RAW || !exists;
  const uint32_t base = z ? 0u : pw[0], Fz = z ? 0u : F;
  get_planes(pw + 1 + LPB + w, LPB, Fz, a);
  const uint32_t sg = Fz ? pw[1 + w] : 0u;
  uint32_t acc = 0;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const uint32_t neg = (uint32_t)__builtin_amdgcn_sbfe((int32_t)sg, i, 1);  // 0 or ~0
    uint32_t d = (a[i] ^ neg) - neg;
    if (i == 0 && w == 0) d = 0;
    acc += d;
    a[i] = acc;
  }
  const uint32_t carry = grp_excl_sum<LPB>(acc, w) + base;
#pragma unroll
  for (int i = 0; i < 32; ++i) a[i] += carry;
}

// Rows of 32 dwords in X to rows STRIDE dwords apart at dst, with 16-byte
// stores (vdw: valid dwords from dst).
template <uint32_t STRIDE, bool FULL>
__device__ __forceinline__ void unit_rows_store(uint32_t* dst, uint32_t vdw, const uint32_t* X) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) {
    const uint32_t row = 8 * k + lane / 8, c = 4 * (lane % 8), dw = row * STRIDE + c;
    const u4u r = *(const u4u*)(X + row * UnitDec::STR + c);
    if (FULL || dw + 4 <= vdw) {
      *(u4u*)(dst + dw) = r;
    } else {
      if (dw + 0 < vdw) dst[dw + 0] = r.x;
      if (dw + 1 < vdw) dst[dw + 1] = r.y;
      if (dw + 2 < vdw) dst[dw + 2] = r.z;
    }
  }
}

template <typename T, int L, int MODE, bool FULL>
__device__ __forceinline__ void unit_decode_put(const Job& J, uint64_t u, T t, const UnitIn& ui,
                                                const uint32_t* pay, uint32_t* X) {
  constexpr uint32_t LPB = L / 32, EW = sizeof(T) / 4;
  const uint32_t lane = __lane_id(), w = lane & (LPB - 1);
  const uint64_t e0 = u * UNIT_ELEMS;
  const uint32_t hval = FULL ? (uint32_t)UNIT_ELEMS : (uint32_t)min((uint64_t)UNIT_ELEMS, J.n - e0);
  const uint32_t vc = FULL ? 32u : (uint32_t)min(32, max(0, (int)hval - 32 * (int)lane));
  const uint32_t* gp = pay + ui.off0;  // the unit's payload (global)
  // fp64 payloads may exceed the region: those are read where they are
  const bool fits = EW == 1 || ui.P + 4 <= UnitDec::XW;
  const uint32_t* S = X;
  if (fits) S = wave_stage_payload<UnitDec::XW - 4, true>(gp, ui.P, X);
  wave_lds_sync();
  if constexpr (MODE == 1) {
    float v[32];
    unpack_tile<float>(S + ui.boff, ui.kind, ui.F, w, ui.ex, t, v);
    if (ui.ex) store_tile(J, (float*)J.out + seg_first<1>(J, u * 64 + lane), v);
    wave_lds_sync();  // read before the next unit's payload goes there
  } else if constexpr (EW == 1) {
    float v[32];
    unpack_seg<float, LPB, FULL>(S + ui.boff, ui.kind, ui.F, w, vc, ui.ex, t, v);
    wave_lds_sync();  // every lane has read its payload words
    f4u* p = (f4u*)(X + lane * UnitDec::STR);
#pragma unroll
    for (int k = 0; k < 8; ++k) p[k] = f4u{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
    wave_lds_sync();
    unit_rows_store<32, FULL>((uint32_t*)((float*)J.out + e0), hval, X);
    wave_lds_sync();
  } else {
    uint32_t q[32];
    if (fits) unpack_q<LPB>(S + ui.boff, ui.kind, ui.F, w, ui.ex, q);
    else unpack_q<LPB>(gp + ui.boff, ui.kind, ui.F, w, ui.ex, q);
    const uint32_t* rw = gp + ui.boff + w * 64;  // a RAW block's words of this lane
    uint32_t* dst = (uint32_t*)((double*)J.out + e0);
#pragma unroll
    for (uint32_t p = 0; p < 2; ++p) {
      wave_lds_sync();  // payload words (or the first half's rows) have been read
      d2u* row = (d2u*)(X + lane * UnitDec::STR);
      if (ui.kind == K_RAW && ui.ex) {
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i) {
          const uint32_t e = 16 * p + i;
          if (FULL || e < vc) ((double*)row)[i] = from_raw(rw + 2 * e, 0.0);
        }
      } else {
#pragma unroll
        for (uint32_t i = 0; i < 16; i += 2)
          row[i / 2] = d2u{(double)(int32_t)q[16 * p + i] * t, (double)(int32_t)q[16 * p + i + 1] * t};
      }
      wave_lds_sync();
      const uint32_t vdw = 2 * hval > 32 * p ? 2 * hval - 32 * p : 0u;
      unit_rows_store<64, FULL>(dst + 32 * p, vdw, X);
    }
    wave_lds_sync();
  }
}

// Decodes unit u of the stream at `in` (job J, in_bytes readable); false
// (nothing written) if its superblock is malformed.
template <typename T, int L, int MODE>
__device__ __forceinline__ bool unit_decode(const Job& J, const uint8_t* in, uint64_t u,
                                            uint32_t* X) {
  const uint64_t sb = u >> 1;
  uint32_t raw[3];
  const uint32_t hdr = wave_header_load(J, in);
  wave_blocks_load<L, true>(J, in, sb, raw);  // in flight with the header's words
  uint64_t paydw = 0;
  T t = 0;
  if (!wave_header_eval<T>(J, hdr, paydw, t)) return false;
  UnitIn ui;
  if (!unit_in_eval<T, L, MODE>(J, sb, (uint32_t)(u & 1), paydw,
                                (uint32_t)min((uint64_t)SUPER, J.n - sb * SUPER), raw, ui))
    return false;
  const uint32_t* pay = (const uint32_t*)(in + J.pay_off);
  if ((u + 1) * UNIT_ELEMS <= J.n) unit_decode_put<T, L, MODE, true>(J, u, t, ui, pay, X);
  else if (u * UNIT_ELEMS < J.n) unit_decode_put<T, L, MODE, false>(J, u, t, ui, pay, X);
  return true;
}

#define GZ_UNIT_DEC_ATTR \
  __launch_bounds__(UnitDec::WAVES * 64) __attribute__((amdgpu_waves_per_eu(4, 4)))

template <typename T, int L, int MODE>
__global__ GZ_UNIT_DEC_ATTR void k_unit_decode(Job J, Ctl C) {
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = blockDim.x >> 6;
  uint32_t* X = g_stage + wid * UnitDec::XW;
  bool bad = false;
  if (J.NS == 0) {  // an empty stream: its header only
    uint64_t paydw;
    T t;
    bad = !wave_header<T>(J, (const uint8_t*)J.in, paydw, t);
  }
  for (uint64_t u = (uint64_t)blockIdx.x * wn + wid; u < 2 * J.NS; u += (uint64_t)gridDim.x * wn)
    bad |= !unit_decode<T, L, MODE>(J, (const uint8_t*)J.in, u, X);
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

// A batch's superblocks as k_batch_accum_w takes them, two units each.
__global__ GZ_UNIT_DEC_ATTR void k_batch_unit_decode(const Job* __restrict__ jobs,
                                                     const uint32_t* __restrict__ map,
                                                     uint32_t njobs, uint32_t total, Ctl C) {
  const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wn = blockDim.x >> 6;
  uint32_t* X = g_stage + wid * UnitDec::XW;
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * wn + wid; i < 2ull * total;
       i += (uint64_t)gridDim.x * wn) {
    const uint64_t s = i >> 1;
    const uint32_t j = map ? map[2 * s] : (uint32_t)s % njobs;
    const uint64_t u = 2 * (uint64_t)(map ? map[2 * s + 1] : (uint32_t)s / njobs) + (i & 1);
    Job J = jobs[j];
    const uint64_t off = J.in_off ? J.in_off[J.job] : 0ull;
    J.in_bytes = off <= J.in_bytes ? J.in_bytes - off : 0ull;
    const uint8_t* in = (const uint8_t*)J.in + off;
    bool ok = false;
    switch ((J.dtype << 3) | J.log2L) {
      case 5: ok = unit_decode<float, 32, 0>(J, in, u, X); break;
      case 6: ok = unit_decode<float, 64, 0>(J, in, u, X); break;
      case 7: ok = unit_decode<float, 128, 0>(J, in, u, X); break;
      case 13: ok = unit_decode<double, 32, 0>(J, in, u, X); break;
      case 14: ok = unit_decode<double, 64, 0>(J, in, u, X); break;
      case 15: ok = unit_decode<double, 128, 0>(J, in, u, X); break;
      default: break;
    }
    bad |= !ok;
  }
  if (bad && __lane_id() == 0) atomicOr(&C.ctrl->err, ERRF_CORRUPT);
}

template <int L, bool FULL>
__device__ __forceinline__ void fused_body(const Job& J, uint64_t s, uint64_t gs, const Ctl& C,
                                           Smem& sm, uint32_t& tk) {
  const uint64_t e0 = (s * blockDim.x + threadIdx.x) * SEG;
  const uint32_t vcnt = FULL ? 32u : (e0 >= J.n ? 0u : (uint32_t)min((uint64_t)SEG, J.n - e0));
  const uint64_t s0 = s * blockDim.x * (uint64_t)SEG;
  float v[32];
  FusedSrc fs;
  const bool ok = decode_strip<float, L, FULL>(J, (const uint8_t*)J.in, J.in_bytes, s, C, sm,
                                               v, vcnt, fs.di);
  fs.pay = (const uint32_t*)((const uint8_t*)J.in + J.pay_off);
  fs.t = sm.t32;
  // The local addend moves through LDS with coalesced loads once the decode
  // is done with the LDS.  (Each lane reading its own 32 values would touch
  // a different 128-byte line in every lane of every load; loading it before
  // the decode holds 32 more registers across it: both measured slower.)
  __syncthreads();  // every lane has read its payload words from LDS
  strip_to_lds<float>(J.local + s0, FULL ? (uint64_t)blockDim.x * SEG : J.n - s0);
  __syncthreads();
  float a[32];
  lane_from_lds<float>(a);
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = v[i] + a[i];  // incoming + local, fp32
  lane_to_lds<float>(v);  // the sums, for a RAW block (own segment: no barrier)
  encode_strip<float, L, FULL, true>(J, s, gs, C, sm, v, vcnt, &fs, !ok, tk);
}

template <int L>
__device__ __forceinline__ void fused_one(const Job& J, uint64_t s, uint64_t gs, const Ctl& C,
                                          Smem& sm, uint32_t& tk) {
  if ((s + 1) * blockDim.x * SEG <= J.n) fused_body<L, true>(J, s, gs, C, sm, tk);
  else fused_body<L, false>(J, s, gs, C, sm, tk);
}

// Persistent loop: the next ticket is requested while the current strip is
// processed, so the atomic's latency is hidden.
#define GZ_STRIP_LOOP(TOTAL, BODY)                                      \
  __shared__ Smem sm;                                                   \
  uint32_t t = first_ticket(C, sm);                                     \
  while (t < (TOTAL)) {                                                 \
    uint32_t nxt = 0;                                                   \
    if (threadIdx.x == 0) nxt = atomicAdd(&C.ctrl->ticket, 1u);         \
    BODY;                                                               \
    __syncthreads();                                                    \
    if (threadIdx.x == 0) sm.cur = nxt;                                 \
    __syncthreads();                                                    \
    t = sm.cur;                                                         \
  }                                                                     \
  epilogue(C);

// Persistent loop of the chained (encoding) operations: BODY sets `nxt`
// (in thread 0) to the next ticket right after its strip's look-back; a
// body that never reaches it leaves the exit value.
#define GZ_CHAIN_LOOP(TOTAL, BODY)                                      \
  __shared__ Smem sm;                                                   \
  uint32_t t = first_ticket(C, sm);                                     \
  while (t < (TOTAL)) {                                                 \
    uint32_t nxt = 0xFFFFFFFFu;                                         \
    BODY;                                                               \
    __syncthreads();                                                    \
    if (threadIdx.x == 0) sm.cur = nxt;                                 \
    __syncthreads();                                                    \
    t = sm.cur;                                                         \
  }                                                                     \
  epilogue(C);

// The fused step is built for four waves per SIMD (a few registers spill):
// that fits one 1024-thread workgroup per CU, which measured faster than
// two of 512 or three 256-thread ones without spills.
#define GZ_FUSED_ATTR __launch_bounds__(MAX_TPB) __attribute__((amdgpu_waves_per_eu(4, 8)))
// tile encoding (selector and three predictors) needs more registers
#define GZ_TILE_ATTR __launch_bounds__(MAX_TPB_WIDE) __attribute__((amdgpu_waves_per_eu(3, 8)))

template <typename T, int L>
__global__ __launch_bounds__(sizeof(T) == 4 ? MAX_TPB : MAX_TPB_WIDE)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 4, 8))) void k_compress(Job J, Ctl C) {
  GZ_CHAIN_LOOP(J.nstrips, (compress_one<T, L>(J, t, t, C, sm, nxt)))
}

template <typename T, int L>
__global__ __launch_bounds__(sizeof(T) == 4 ? MAX_TPB : MAX_TPB_WIDE)
__attribute__((amdgpu_waves_per_eu(4, 8))) void k_decompress(Job J, Ctl C) {
  GZ_STRIP_LOOP(J.nstrips, (decompress_tp_one<T, L>(J, t, C, sm, nxt)))
}

template <int L>
__global__ __launch_bounds__(MAX_TPB) __attribute__((amdgpu_waves_per_eu(4, 8)))
void k_accum(Job J, Ctl C) {
  GZ_STRIP_LOOP(J.nstrips, (accum_one<L>(J, t, C, sm)))
}

template <int L>
__global__ GZ_FUSED_ATTR void k_fused(Job J, Ctl C) {
  GZ_CHAIN_LOOP(J.nstrips, (fused_one<L>(J, t, t, C, sm, nxt)))
}

// Batched: ticket t processes strip strip_job[2t + 1] of job strip_job[2t]
// or, when every job has the same strip count (njobs > 0, jobs interleaved
// round-robin), strip t / njobs of job t % njobs; its look-back word is
// J.strip0 + that strip.  One kernel per operation; WIDE admits fp64 jobs
// (fp32-only batches avoid the register pressure of the fp64 paths).
template <uint32_t OP, bool WIDE>
__device__ __forceinline__ void batch_body(const Job* __restrict__ jobs,
                                           const uint32_t* __restrict__ strip_job, uint32_t njobs,
                                           uint32_t t, const Ctl& C, Smem& sm, uint32_t& tk) {
  const uint32_t j = njobs ? t % njobs : strip_job[2 * (uint64_t)t];
  const uint64_t s = njobs ? t / njobs : strip_job[2 * (uint64_t)t + 1];
  const Job J = jobs[j];
  const uint64_t gs = J.strip0 + s;
  const uint32_t key = (J.dtype << 3) | J.log2L;
  if (OP == 0) {
    switch (key) {
      case 5: compress_one<float, 32>(J, s, gs, C, sm, tk); break;
      case 6: compress_one<float, 64>(J, s, gs, C, sm, tk); break;
      case 7: compress_one<float, 128>(J, s, gs, C, sm, tk); break;
      case 13: if (WIDE) compress_one<double, 32>(J, s, gs, C, sm, tk); break;
      case 14: if (WIDE) compress_one<double, 64>(J, s, gs, C, sm, tk); break;
      case 15: if (WIDE) compress_one<double, 128>(J, s, gs, C, sm, tk); break;
      default: break;
    }
  } else if (OP == 1) {
    switch (key) {
      case 5: decompress_one<float, 32>(J, s, C, sm); break;
      case 6: decompress_one<float, 64>(J, s, C, sm); break;
      case 7: decompress_one<float, 128>(J, s, C, sm); break;
      case 13: if (WIDE) decompress_one<double, 32>(J, s, C, sm); break;
      case 14: if (WIDE) decompress_one<double, 64>(J, s, C, sm); break;
      case 15: if (WIDE) decompress_one<double, 128>(J, s, C, sm); break;
      default: break;
    }
  } else if (OP == 2) {
    switch (key) {
      case 5: fused_one<32>(J, s, gs, C, sm, tk); break;
      case 6: fused_one<64>(J, s, gs, C, sm, tk); break;
      case 7: fused_one<128>(J, s, gs, C, sm, tk); break;
      default: break;
    }
  } else {
    switch (key) {
      case 5: accum_one<32>(J, s, C, sm); break;
      case 6: accum_one<64>(J, s, C, sm); break;
      case 7: accum_one<128>(J, s, C, sm); break;
      default: break;
    }
  }
}

template <uint32_t OP, bool WIDE>
__global__ __launch_bounds__(WIDE ? MAX_TPB_WIDE : MAX_TPB)
__attribute__((amdgpu_waves_per_eu((OP == 0 && WIDE) ? 3 : 4, 8))) void k_batch(const Job* __restrict__ jobs,
                                       const uint32_t* __restrict__ strip_job, uint32_t njobs,
                                       uint32_t total, Ctl C) {
  if constexpr (OP == 1 || OP == 3) {
    GZ_STRIP_LOOP(total, (batch_body<OP, WIDE>(jobs, strip_job, njobs, t, C, sm, nxt)))
  } else {
    GZ_CHAIN_LOOP(total, (batch_body<OP, WIDE>(jobs, strip_job, njobs, t, C, sm, nxt)))
  }
}

// ------------------------------------------------------------ tile mode
template <bool FULL>
__device__ __forceinline__ void compress_tiles_body(const Job& J, uint64_t s, uint64_t gs,
                                                    const Ctl& C, Smem& sm, uint32_t& tk) {
  const uint64_t seg = s * blockDim.x + threadIdx.x;
  const bool ex = FULL || (seg >> 1) < J.B;
  float v[32];
  load_tile(J, (const float*)J.in + (ex ? seg_first<1>(J, seg) : 0), ex, v);
  LaneCode lc;
  analyze_tile(J, threadIdx.x & 1u, v, ex, sm.wts, lc);
  emit_strip<float, 64, 1, false, FULL>(J, s, gs, C, sm, ex ? 32u : 0u, lc, nullptr, false, tk);
}

__device__ __forceinline__ void load_weights(const Ctl& C, Smem& sm) {
  for (uint32_t k = threadIdx.x; k < 189; k += blockDim.x) sm.wts[k] = ((const uint32_t*)C.blob)[k];
  __syncthreads();
}

__global__ GZ_TILE_ATTR void k_compress_tiles(Job J, Ctl C) {
  __shared__ Smem sm;
  load_weights(C, sm);
  uint32_t t = first_ticket(C, sm);
  while (t < J.nstrips) {
    uint32_t nxt = 0xFFFFFFFFu;  // the next ticket, taken after the look-back
    if ((t + 1) * (uint64_t)blockDim.x <= 2 * J.B) compress_tiles_body<true>(J, t, t, C, sm, nxt);
    else compress_tiles_body<false>(J, t, t, C, sm, nxt);
    __syncthreads();
    if (threadIdx.x == 0) sm.cur = nxt;
    __syncthreads();
    t = sm.cur;
  }
  epilogue(C);
}

__global__ __launch_bounds__(MAX_TPB_WIDE)
__attribute__((amdgpu_waves_per_eu(4, 8))) void k_decompress_tiles(Job J, Ctl C) {
  __shared__ Smem sm;
  uint32_t t = first_ticket(C, sm);
  while (t < J.nstrips) {
    uint32_t nxt = 0;
    if (threadIdx.x == 0) nxt = atomicAdd(&C.ctrl->ticket, 1u);
    const uint64_t seg = t * (uint64_t)blockDim.x + threadIdx.x;
    const bool ex = (seg >> 1) < J.B;
    float v[32];
    DecInfo di;
    if (decode_strip<float, 64, false, 1>(J, (const uint8_t*)J.in, J.in_bytes, t, C, sm, v,
                                          ex ? 32u : 0u, di) && ex)
      store_tile(J, (float*)J.out + seg_first<1>(J, seg), v);
    __syncthreads();
    if (threadIdx.x == 0) sm.cur = nxt;
    __syncthreads();
    t = sm.cur;
  }
  epilogue(C);
}

// Training data of the selector: per tile the 16 features, the sizes of the
// three encodings and the exhaustive-trial label (255: RAW or ZERO tile).
__global__ __launch_bounds__(256) void k_tile_trial(Job J, int8_t* __restrict__ feat,
                                                   uint32_t* __restrict__ sizes,
                                                   uint8_t* __restrict__ label) {
  const uint64_t nseg = 2 * J.B;
  for (uint64_t seg = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
       seg - threadIdx.x < nseg; seg += (uint64_t)gridDim.x * blockDim.x) {
    // whole waves iterate together (the tile's two lanes shuffle)
    const bool ex = seg < nseg;
    const uint32_t w = threadIdx.x & 1u;
    float v[32];
    load_tile(J, (const float*)J.in + (ex ? seg_first<1>(J, seg) : 0), ex, v);
    int32_t q[32];
    bool bad;
    tile_quant(J, v, q, bad);
    int32_t up[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) up[c] = (int32_t)lane_below((uint32_t)q[24 + c]);
    uint32_t f[4];
    tile_features(q, w, f);
    const uint32_t o0 = tile_or<0>(q, up, w), o1 = tile_or<1>(q, up, w), o2 = tile_or<2>(q, up, w);
    const uint32_t s0 = size_of(K_NONE, o0 ? 32u - __clz(o0) : 0u);
    const uint32_t s1 = size_of(K_L1D, o1 ? 32u - __clz(o1) : 0u);
    const uint32_t s2 = size_of(K_L2D, o2 ? 32u - __clz(o2) : 0u);
    uint32_t best = 0, bs = s0;
    if (s1 < bs) { best = 1; bs = s1; }
    if (s2 < bs) best = 2;
    const bool zero = (grp_or<2>(q[0] != 0 ? 1u : 0u) | o0) == 0;
    if (ex && w == 0) {
      const uint64_t b = seg >> 1;
      ((uint32_t*)feat)[4 * b + 0] = f[0];
      ((uint32_t*)feat)[4 * b + 1] = f[1];
      ((uint32_t*)feat)[4 * b + 2] = f[2];
      ((uint32_t*)feat)[4 * b + 3] = f[3];
      sizes[3 * b + 0] = 4 * s0;
      sizes[3 * b + 1] = 4 * s1;
      sizes[3 * b + 2] = 4 * s2;
      label[b] = (bad || zero) ? 255 : (uint8_t)best;
    }
  }
}

// Elementwise quantisation (verification entry point).
template <typename T>
__global__ void k_quantize(const T* __restrict__ x, uint64_t n, Job J, int32_t* __restrict__ q,
                           uint8_t* __restrict__ fail) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    QBad<T> qb;
    uint32_t qi;
    quant_run<1, true>(x + i, J, 1, &qi, qb);
    const bool bad = qb.any(bad_bound<T>(J));
    q[i] = bad ? 0 : (int32_t)qi;
    fail[i] = bad ? 1 : 0;
  }
}

// Clears the control block (after a device error) without a memset node.
__global__ void k_reset(Ctl C) {
  if (threadIdx.x == 0) {
    C.ctrl->ticket = 0;
    C.ctrl->done = 0;
    C.ctrl->epoch = C.ctrl->epoch + 1;
  }
}

// Reports the sticky device status of a launch (GZ_OK 0, GZ_ECORRUPT 3,
// GZ_ETIMEOUT 7) into *out (when given) and clears it, so that the next
// launch on the same workspace starts clean.
__global__ void k_finish(Ctl C, uint32_t* out) {
  if (threadIdx.x == 0) {
    const uint32_t e = ld_agent32(&C.ctrl->err);
    if (out) *out = (e & ERRF_CORRUPT) ? 3u : (e & ERRF_TIMEOUT) ? 7u : 0u;
    if (e) atomicAnd(&C.ctrl->err, 0u);
  }
}

// ------------------------------------------------------------ launchers
// Dynamic LDS: the strip staging buffer (largest strip payload + headroom).
static size_t stage_bytes(uint32_t dtype, uint32_t tpb) {
  return 32 + (size_t)tpb * (SEG * (dtype == 0 ? 1 : 2) + 4) * 4;  // padded segment layout
}

size_t lds_bytes(uint32_t wide, uint32_t tpb) { return stage_bytes(wide, tpb) + sizeof(Smem); }

template <typename T, int L>
static hipError_t launch_c(const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_compress<T, L>), dim3(grid), dim3(tpb), stage_bytes(J.dtype, tpb), st, J,
                     C);
  return hipGetLastError();
}
template <typename T, int L>
static hipError_t launch_d(const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_decompress<T, L>), dim3(grid), dim3(tpb), stage_bytes(J.dtype, tpb), st,
                     J, C);
  return hipGetLastError();
}
template <int L>
static hipError_t launch_dw(const Job& J, const Ctl& C, uint32_t grid, hipStream_t st) {
  hipLaunchKernelGGL((k_decompress_w<L>), dim3(grid), dim3(WaveDec::WAVES * 64),
                     wave_decode_lds(), st, J, C);
  return hipGetLastError();
}

hipError_t launch_decompress_wave(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st) {
  const uint64_t need = (J.NS + WaveDec::WAVES - 1) / WaveDec::WAVES;
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, need));
  switch (J.log2L) {
    case 5: return launch_dw<32>(J, C, grid, st);
    case 6: return launch_dw<64>(J, C, grid, st);
    case 7: return launch_dw<128>(J, C, grid, st);
  }
  return hipErrorInvalidValue;
}

size_t wave_fused_lds() {
  return (size_t)WaveEnc::WAVES * WaveEnc::REGION * 4 + sizeof(WaveSched);
}

template <int L>
static hipError_t launch_fw(const Job* d_jobs, uint32_t njobs, uint32_t total, const Ctl& C,
                            uint32_t cus, hipStream_t st) {
  // one workgroup per round in flight, at most one per CU (the LDS allows one)
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, total));
  hipLaunchKernelGGL((k_batch_fused_w<L>), dim3(grid), dim3(WaveEnc::WAVES * 64),
                     (size_t)WaveEnc::WAVES * WaveEnc::REGION * 4, st, d_jobs, njobs, total, C);
  return hipGetLastError();
}

template <int L>
static hipError_t launch_fw1(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st) {
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, wave_rounds(J.NS)));
  hipLaunchKernelGGL((k_fused_w<L>), dim3(grid), dim3(WaveEnc::WAVES * 64),
                     (size_t)WaveEnc::WAVES * WaveEnc::REGION * 4, st, J, C);
  return hipGetLastError();
}

hipError_t launch_fused_wave_single(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st) {
  switch (J.log2L) {
    case 5: return launch_fw1<32>(J, C, cus, st);
    case 6: return launch_fw1<64>(J, C, cus, st);
    case 7: return launch_fw1<128>(J, C, cus, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_fused_wave(const Job* d_jobs, uint32_t njobs, uint32_t total, uint32_t log2L,
                             const Ctl& C, uint32_t cus, hipStream_t st) {
  switch (log2L) {
    case 5: return launch_fw<32>(d_jobs, njobs, total, C, cus, st);
    case 6: return launch_fw<64>(d_jobs, njobs, total, C, cus, st);
    case 7: return launch_fw<128>(d_jobs, njobs, total, C, cus, st);
  }
  return hipErrorInvalidValue;
}

size_t unit_lds(bool fused, uint32_t workers) {
  return (size_t)workers * (fused ? UnitEnc<true>::REGION : UnitEnc<false>::REGION) * 4 +
         sizeof(USched);
}

template <typename T, int L, bool FUSED>
static hipError_t launch_u(const Job& J, const Ctl& C, uint32_t workers, uint32_t grid,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_unit<T, L, FUSED>), dim3(grid), dim3((workers + 1) * 64),
                     (size_t)workers * UnitEnc<FUSED>::REGION * 4, st, J, C);
  return hipGetLastError();
}

template <uint32_t OP, bool WIDE>
static hipError_t launch_bu(const Job* d_jobs, const uint32_t* d_map, uint32_t njobs,
                            uint32_t total, const Ctl& C, uint32_t workers, uint32_t early,
                            uint32_t grid, hipStream_t st) {
  hipLaunchKernelGGL((k_batch_unit<OP, WIDE>), dim3(grid), dim3((workers + 1) * 64),
                     (size_t)workers * UnitEnc<OP == 2>::REGION * 4, st, d_jobs, d_map, njobs,
                     total, early, C);
  return hipGetLastError();
}

// Workgroups in flight: as many as the CUs hold, at most one per round.
static uint32_t unit_grid(bool fused, uint32_t cus, uint32_t workers, uint32_t total) {
  return (uint32_t)std::max<uint64_t>(
      1, std::min<uint64_t>((uint64_t)cus * unit_per_cu(fused, workers), total));
}

// Whether a batch's workgroups take tickets at a round's first publication until
// they meet a payload too large to be held (longest: rounds of its longest
// chain).  It lets a workgroup whose round is part empty go on to the next job's
// (512 requests of 1 K to 1 M values 115 us, early 107; 64 jobs of 2^20 110 and
// 98), but the first large payload of each workgroup then delays a chain: with
// one unit in a hundred large, chains of 137 rounds lost nothing to it (32 jobs of
// 2^22 206 us, 210 by strips), 547 rounds 314 against 196 (8 of 2^24).  Not given
// up at a large payload, it cost chains of 35 rounds of ratio 3 122 against 109.
static uint32_t unit_early(uint32_t longest) { return longest <= 192 ? 1u : 0u; }

hipError_t launch_unit(uint32_t op, const Job& J, const Ctl& C, uint32_t workers, uint32_t cus,
                       hipStream_t st) {
  const bool fused = op == 2;
  const uint32_t grid = unit_grid(fused, cus, workers, J.nstrips);
  if (J.mode == 1) {
    hipLaunchKernelGGL(k_unit_tiles, dim3(grid), dim3((workers + 1) * 64),
                       (size_t)workers * UnitEnc<false>::REGION * 4, st, J, C);
    return hipGetLastError();
  }
  switch ((J.dtype << 3) | J.log2L) {
    case 5: return fused ? launch_u<float, 32, true>(J, C, workers, grid, st)
                         : launch_u<float, 32, false>(J, C, workers, grid, st);
    case 6: return fused ? launch_u<float, 64, true>(J, C, workers, grid, st)
                         : launch_u<float, 64, false>(J, C, workers, grid, st);
    case 7: return fused ? launch_u<float, 128, true>(J, C, workers, grid, st)
                         : launch_u<float, 128, false>(J, C, workers, grid, st);
    case 13: return fused ? hipErrorInvalidValue
                          : launch_u<double, 32, false>(J, C, workers, grid, st);
    case 14: return fused ? hipErrorInvalidValue
                          : launch_u<double, 64, false>(J, C, workers, grid, st);
    case 15: return fused ? hipErrorInvalidValue
                          : launch_u<double, 128, false>(J, C, workers, grid, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_batch_unit(uint32_t op, const Job* d_jobs, const uint32_t* d_map,
                             uint32_t njobs, uint32_t total, bool wide, const Ctl& C,
                             uint32_t workers, uint32_t longest, uint32_t cus,
                             hipStream_t st) {
  const uint32_t grid = unit_grid(op == 2, cus, workers, total);
  const uint32_t early = unit_early(longest);
  if (op == 0)
    return wide ? launch_bu<0, true>(d_jobs, d_map, njobs, total, C, workers, early, grid, st)
                : launch_bu<0, false>(d_jobs, d_map, njobs, total, C, workers, early, grid, st);
  if (op == 2 && !wide)
    return launch_bu<2, false>(d_jobs, d_map, njobs, total, C, workers, early, grid, st);
  return hipErrorInvalidValue;
}

template <typename T, int L, int MODE>
static hipError_t launch_ud(const Job& J, const Ctl& C, uint32_t grid, uint32_t waves,
                            hipStream_t st) {
  hipLaunchKernelGGL((k_unit_decode<T, L, MODE>), dim3(grid), dim3(waves * 64),
                     (size_t)waves * UnitDec::XW * 4, st, J, C);
  return hipGetLastError();
}

hipError_t launch_unit_decode(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st) {
  // short streams: a wave a workgroup, so that they spread over the CUs
  const uint64_t units = std::max<uint64_t>(1, 2 * J.NS);
  const uint32_t waves = units <= 2ull * cus ? 1 : UnitDec::WAVES;
  const uint32_t grid =
      (uint32_t)std::min<uint64_t>((uint64_t)cus * 16 / waves, (units + waves - 1) / waves);
  if (J.mode == 1) return launch_ud<float, 64, 1>(J, C, grid, waves, st);
  switch ((J.dtype << 3) | J.log2L) {
    case 5: return launch_ud<float, 32, 0>(J, C, grid, waves, st);
    case 6: return launch_ud<float, 64, 0>(J, C, grid, waves, st);
    case 7: return launch_ud<float, 128, 0>(J, C, grid, waves, st);
    case 13: return launch_ud<double, 32, 0>(J, C, grid, waves, st);
    case 14: return launch_ud<double, 64, 0>(J, C, grid, waves, st);
    case 15: return launch_ud<double, 128, 0>(J, C, grid, waves, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_batch_unit_decode(const Job* d_jobs, const uint32_t* d_map, uint32_t njobs,
                                    uint32_t total, uint32_t cus, const Ctl& C, hipStream_t st) {
  const uint64_t units = std::max<uint64_t>(1, 2ull * total);
  const uint32_t grid = (uint32_t)std::min<uint64_t>(
      (uint64_t)cus * 16 / UnitDec::WAVES, (units + UnitDec::WAVES - 1) / UnitDec::WAVES);
  hipLaunchKernelGGL(k_batch_unit_decode, dim3(grid), dim3(UnitDec::WAVES * 64),
                     (size_t)UnitDec::WAVES * UnitDec::XW * 4, st, d_jobs, d_map, njobs, total, C);
  return hipGetLastError();
}

template <int L>
static hipError_t launch_aw(const Job& J, const Ctl& C, uint32_t grid, hipStream_t st) {
  const size_t lds = (size_t)WaveDec::WAVES * WaveDec::REGION * 4;
  hipLaunchKernelGGL((k_accum_w<L>), dim3(grid), dim3(WaveDec::WAVES * 64), lds, st, J, C);
  return hipGetLastError();
}

hipError_t launch_accum_wave(const Job& J, const Ctl& C, uint32_t cus, hipStream_t st) {
  const uint64_t need = (J.NS + WaveDec::WAVES - 1) / WaveDec::WAVES;
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, need));
  switch (J.log2L) {
    case 5: return launch_aw<32>(J, C, grid, st);
    case 6: return launch_aw<64>(J, C, grid, st);
    case 7: return launch_aw<128>(J, C, grid, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_decode_shares(const Job* d_jobs, const uint32_t* d_map, uint32_t jw,
                                uint32_t cus, const Ctl& C, hipStream_t st) {
  constexpr uint32_t WAVES = WaveDec::WAVES;
  const uint32_t grid =
      (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, (jw + WAVES - 1) / WAVES));
  hipLaunchKernelGGL(k_batch_decode_w, dim3(grid), dim3(WAVES * 64), wave_decode_lds(), st, d_jobs,
                     d_map, jw, C);
  return hipGetLastError();
}

hipError_t launch_accum_wave_batch(const Job* d_jobs, const uint32_t* d_map, uint32_t njobs,
                                   uint32_t total, uint32_t cus, const Ctl& C, hipStream_t st) {
  constexpr uint32_t WAVES = WaveDec::WAVES;
  const uint64_t need = ((uint64_t)total + WAVES - 1) / WAVES;
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cus, need));
  hipLaunchKernelGGL(k_batch_accum_w, dim3(grid), dim3(WAVES * 64), wave_decode_lds(), st, d_jobs,
                     d_map, njobs, total, C);
  return hipGetLastError();
}

size_t wave_decode_lds() { return (size_t)WaveDec::WAVES * WaveDec::REGION * 4; }

size_t unit_decode_lds() { return (size_t)UnitDec::WAVES * UnitDec::XW * 4; }

template <int L>
static hipError_t launch_a(const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_accum<L>), dim3(grid), dim3(tpb), stage_bytes(0, tpb), st, J, C);
  return hipGetLastError();
}
template <int L>
static hipError_t launch_f(const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                           hipStream_t st) {
  hipLaunchKernelGGL((k_fused<L>), dim3(grid), dim3(tpb), stage_bytes(0, tpb), st, J, C);
  return hipGetLastError();
}

hipError_t launch_single(uint32_t op, const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                         hipStream_t st) {
  const uint32_t key = (J.dtype << 3) | J.log2L;
  if (op == 0) {
    switch (key) {
      case 5: return launch_c<float, 32>(J, C, tpb, grid, st);
      case 6: return launch_c<float, 64>(J, C, tpb, grid, st);
      case 7: return launch_c<float, 128>(J, C, tpb, grid, st);
      case 13: return launch_c<double, 32>(J, C, tpb, grid, st);
      case 14: return launch_c<double, 64>(J, C, tpb, grid, st);
      case 15: return launch_c<double, 128>(J, C, tpb, grid, st);
    }
  } else if (op == 1) {
    switch (key) {
      case 5: return launch_d<float, 32>(J, C, tpb, grid, st);
      case 6: return launch_d<float, 64>(J, C, tpb, grid, st);
      case 7: return launch_d<float, 128>(J, C, tpb, grid, st);
      case 13: return launch_d<double, 32>(J, C, tpb, grid, st);
      case 14: return launch_d<double, 64>(J, C, tpb, grid, st);
      case 15: return launch_d<double, 128>(J, C, tpb, grid, st);
    }
  } else if (op == 2) {
    switch (key) {
      case 5: return launch_f<32>(J, C, tpb, grid, st);
      case 6: return launch_f<64>(J, C, tpb, grid, st);
      case 7: return launch_f<128>(J, C, tpb, grid, st);
    }
  } else if (op == 3) {
    switch (key) {
      case 5: return launch_a<32>(J, C, tpb, grid, st);
      case 6: return launch_a<64>(J, C, tpb, grid, st);
      case 7: return launch_a<128>(J, C, tpb, grid, st);
    }
  }
  return hipErrorInvalidValue;
}

static const void* batch_kernel(uint32_t op, bool wide) {
  switch (op * 2 + (wide ? 1 : 0)) {
    case 0: return (const void*)k_batch<0, false>;
    case 1: return (const void*)k_batch<0, true>;
    case 2: return (const void*)k_batch<1, false>;
    case 3: return (const void*)k_batch<1, true>;
    case 4: return (const void*)k_batch<2, false>;
    default: return (const void*)k_batch<3, false>;
  }
}

hipError_t launch_batch(uint32_t op, const Job* d_jobs, const uint32_t* d_strip_job,
                        uint32_t njobs, uint32_t total, const Ctl& C, uint32_t tpb, uint32_t grid, bool wide,
                        hipStream_t st) {
  const size_t lds = stage_bytes(wide ? 1 : 0, tpb);
  if (op == 0 && !wide)
    hipLaunchKernelGGL((k_batch<0, false>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else if (op == 0)
    hipLaunchKernelGGL((k_batch<0, true>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else if (op == 1 && !wide)
    hipLaunchKernelGGL((k_batch<1, false>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else if (op == 1)
    hipLaunchKernelGGL((k_batch<1, true>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else if (op == 2)
    hipLaunchKernelGGL((k_batch<2, false>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else if (op == 3 && !wide)
    hipLaunchKernelGGL((k_batch<3, false>), dim3(grid), dim3(tpb), lds, st, d_jobs, d_strip_job,
                       njobs, total, C);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_quantize(const void* x, uint64_t n, const Job& J, int32_t* q, uint8_t* fail,
                           hipStream_t st) {
  uint64_t blocks = (n + 255) / 256;
  uint32_t grid = (uint32_t)(blocks < 65536 ? (blocks ? blocks : 1) : 65536);
  if (J.dtype == 0)
    hipLaunchKernelGGL(k_quantize<float>, dim3(grid), dim3(256), 0, st, (const float*)x, n, J, q,
                       fail);
  else
    hipLaunchKernelGGL(k_quantize<double>, dim3(grid), dim3(256), 0, st, (const double*)x, n, J,
                       q, fail);
  return hipGetLastError();
}

hipError_t launch_tiles(uint32_t op, const Job& J, const Ctl& C, uint32_t tpb, uint32_t grid,
                        hipStream_t st) {
  if (op == 0)
    hipLaunchKernelGGL(k_compress_tiles, dim3(grid), dim3(tpb), stage_bytes(0, tpb), st, J, C);
  else
    hipLaunchKernelGGL(k_decompress_tiles, dim3(grid), dim3(tpb), stage_bytes(0, tpb), st, J, C);
  return hipGetLastError();
}

hipError_t launch_tile_trial(const Job& J, int8_t* feat, uint32_t* sizes, uint8_t* label,
                             hipStream_t st) {
  // every tile is read from J.in and written to the three outputs
  if (J.B && (!J.in || !feat || !sizes || !label || J.nx == 0 || J.nx % 8 != 0 ||
              J.n != 64 * J.B || J.n % (8ull * J.nx) != 0))
    return hipErrorInvalidValue;
  const uint64_t segs = 2 * J.B;
  uint64_t blocks = (segs + 255) / 256;
  const uint32_t grid = (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
  hipLaunchKernelGGL(k_tile_trial, dim3(grid), dim3(256), 0, st, J, feat, sizes, label);
  return hipGetLastError();
}

hipError_t launch_finish(const Ctl& C, uint32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(64), 0, st, C, status);
  return hipGetLastError();
}

hipError_t launch_reset(const Ctl& C, hipStream_t st) {
  hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, st, C);
  return hipGetLastError();
}

int occupancy_blocks(uint32_t op, uint32_t dtype, uint32_t log2L, uint32_t tpb) {
  int nb = 0;
  const void* f = nullptr;
  const uint32_t key = (dtype << 3) | log2L;
  if (op == 0) {
    switch (key) {
      case 5: f = (const void*)k_compress<float, 32>; break;
      case 6: f = (const void*)k_compress<float, 64>; break;
      case 7: f = (const void*)k_compress<float, 128>; break;
      case 13: f = (const void*)k_compress<double, 32>; break;
      case 14: f = (const void*)k_compress<double, 64>; break;
      case 15: f = (const void*)k_compress<double, 128>; break;
    }
  } else if (op == 1) {
    switch (key) {
      case 5: f = (const void*)k_decompress<float, 32>; break;
      case 6: f = (const void*)k_decompress<float, 64>; break;
      case 7: f = (const void*)k_decompress<float, 128>; break;
      case 13: f = (const void*)k_decompress<double, 32>; break;
      case 14: f = (const void*)k_decompress<double, 64>; break;
      case 15: f = (const void*)k_decompress<double, 128>; break;
    }
  } else if (op == 2) {
    switch (key) {
      case 5: f = (const void*)k_fused<32>; break;
      case 6: f = (const void*)k_fused<64>; break;
      case 7: f = (const void*)k_fused<128>; break;
    }
  } else if (op == OCC_TILE_C) {
    f = (const void*)k_compress_tiles;
  } else if (op == OCC_TILE_D) {
    f = (const void*)k_decompress_tiles;
  } else if (op == OCC_ACCUM) {
    switch (log2L) {
      case 5: f = (const void*)k_accum<32>; break;
      case 6: f = (const void*)k_accum<64>; break;
      case 7: f = (const void*)k_accum<128>; break;
    }
  } else {
    f = batch_kernel(op - OCC_BATCH, dtype != 0);  // batched op (op - OCC_BATCH)
  }
  if (!f) return 1;
  const bool f32_only = op == 2 || op >= OCC_BATCH + 2;  // fused, accumulate, tiles
  const size_t lds = stage_bytes(f32_only ? 0 : dtype, tpb);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, (int)tpb, lds) != hipSuccess || nb < 1)
    nb = 1;
  return nb;
}

}  // namespace gzk
