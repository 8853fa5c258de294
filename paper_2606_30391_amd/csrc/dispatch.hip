// dispatch.hip -- MI355X (gfx950) kernels and C-ABI host dispatch of the paper's own
// request dispatcher (Festina, Sec. 3.3 as the paper runs it): one operating point per GPU
// (its current frequency and the SMs free when the request's memory is available), the
// 2% stability tie-break, the F_max fallback ordered by availability, and a new GPU's
// least-energy level.
//
// k_dsp_hosts  one block per model: list of the GPUs hosting it (wavefront ballots), in the
//                caller's workspace; with at most 4 profile steps, also a
//                64-byte record per (model, host) with everything Phase One reads, so that
//                the 16 lanes of a request load their hosts with coalesced 16-byte loads.
// k_dispatch   16 lanes per request (four per wavefront; 32 lanes in a launch of at most
//                8,192 requests, 64 in one of at most 2,048, a block of 512 for a few requests on a
//                large fleet) stride over the model's hosts.  Per host:
//                the first free-memory profile step that holds Req_mem gives T_avail and
//                SM_free; the point (SM_free, F_curr) is feasible when T_avail + TTFT and
//                TBT meet the SLOs; E = P * (TTFT + Lout * TBT) in float64.  One pass
//                evaluates every host (a lane's first four hosts stay in registers) and
//                the group takes E_min; among hosts with E <= E_min + 0.02 |E_min| the largest
//                stability key (most memory, most SMs, lowest id packed in 64 bits) wins,
//                and the lane holding it writes the result.  With no
//                candidate: the hosts feasible at the top level, earliest T_avail (then
//                lowest id).  Else lane k scores a new GPU at level k and the least energy
//                (lowest k on ties) wins.
// Over arrival waves (festina_dispatch_waves), profiles of at most 4 steps: k_wave4_init packs every
//                GPU's profile and state into 16-byte words; one k_dispatch4 per wave reads, for
//                kBatch hosts of a lane at once, the id list, then state, previous commits and
//                profile, then the table entries (four memory round trips per wave, where a
//                loop over the hosts takes five per host); commits and state as below.
// Longer profiles: k_wave_init copies the caller's state into a
//                workspace buffer; one k_dispatch per wave reads the state with the previous
//                wave's commits applied, stores that state for the next wave, and commits its
//                own placements (batch, memory from the admitting step on, F_max boost) with
//                atomics; k_wave_final writes the last state back.
//
// Exactness: the energies are float64 in the same order of operations as any float64
// evaluation of P0 + k*s*f^3*u and P * (TTFT + Lout*TBT) without contraction, so the 2%
// test and every comparison are decided on identical values; the SLO tests add or compare
// float32 inputs exactly.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstddef>
#include <cstdint>

#include "festina.h"

namespace {

constexpr int kRows = FESTINA_N_ROWS;
constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kHostBlock = 256;
constexpr int kMaxSteps = 8;                 // profile steps loaded at once
constexpr double kStability = 0.02;          // energies within 2% of the least tie

// Wave-by-wave calls keep two kinds of buffers in the workspace, each one allocation:
//   state   int32 [G][2] (current level, batch) then int32 [G][S] free MiB per profile step;
//   commits uint64 [G] (requests placed in the low 32 bits, bit 32 set by an F_max
//           placement) then uint64 [G][S] MiB taken per step (a request admitted at step s
//           counts at s and at every later step).
__device__ __forceinline__ int2 *state_fb(int32_t *st) { return reinterpret_cast<int2 *>(st); }
__device__ __forceinline__ int32_t *state_mem(int32_t *st, int G) { return st + 2 * (size_t)G; }
__device__ __forceinline__ unsigned long long *commit_taken(unsigned long long *c, int G) { return c + G; }

struct DspArgs {
  int32_t M, NS, NF, C, words;
  const float *sm_level, *freq_level, *pf, *dc;
  double p0;
  int32_t G, S;
  const int32_t *freq_cur, *batch;
  const float *kdyn;
  const uint32_t *resident;
  const float *t_avail;
  const int32_t *mem_free, *sm_free, *kv;
  double k_new;
  int32_t R;
  const int32_t *model, *prompt, *pred;
  const float *slo_ttft, *slo_tbt;
  int32_t *out_gpu, *out_freq, *out_sm;
  uint8_t *out_phase;
  float *out_energy;
  int32_t *host_cnt, *host_list;     // workspace: [M], [M][G]
  int4 *hrec;                        // workspace: [M][G][4] host records when S <= 4
  int32_t packed;
  int32_t r0;                        // first request of the launch (a.R: one past the last)
  // Wave-by-wave calls only (the kWaves kernels): the state this wave sees is `wstate` with
  // the previous wave's commits `wprev` applied (freq_cur, batch and mem_free are unused).
  // The launch also writes that state to `wfold` (the next wave's state), commits this
  // wave's placements to `wcur`, and clears `wnext` (the commits of the wave after).
  int32_t *wstate, *wfold;
  unsigned long long *wprev, *wcur, *wnext;
};

typedef int v4i __attribute__((ext_vector_type(4)));

// Energy on one operating point: P = p0 + k*s*f^3*u, E = P * (ttft + lout*tbt), each
// operation rounded separately (no fused multiply-add).
__device__ __forceinline__ double point_energy(double p0, double kg, double s, double f, double u, double ttft,
                                            double lout, double tbt) {
#pragma clang fp contract(off)
  const double f3 = f * f * f;
  const double P = p0 + kg * s * f3 * u;
  return P * (ttft + lout * tbt);
}

// One block per model, kListGpus GPUs at a time: the hosting GPUs' ids are collected in LDS in any
// order (every use of the list is a reduction whose result does not depend on it), all residency
// words of a thread in flight together, then each thread takes one host at a time.  With one
// workgroup-wide scan per 256 GPUs instead, 10,000 GPUs took 68 us.
constexpr int kListThreads = 1024, kListPer = 16, kListGpus = kListThreads * kListPer;

__global__ void __launch_bounds__(kListThreads) k_dsp_hosts(DspArgs a) {
  __shared__ int ids[kListGpus];
  __shared__ int cnt;
  const int m = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  int base = 0;
  for (int G0 = 0; G0 < a.G; G0 += kListGpus) {
    if (threadIdx.x == 0) cnt = 0;
    uint32_t word[kListPer];
#pragma unroll
    for (int u = 0; u < kListPer; ++u) {
      const int g = G0 + u * kListThreads + threadIdx.x;
      word[u] = g < a.G ? a.resident[(size_t)g * a.words + (m >> 5)] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kListPer; ++u) {
      const bool has = (word[u] >> (m & 31)) & 1u;
      const unsigned long long bal = __ballot(has);
      if (bal == 0ull) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&cnt, __popcll(bal));
      at = __builtin_amdgcn_readfirstlane(at);
      if (has) ids[at + __popcll(bal & ((1ull << lane) - 1ull))] = G0 + u * kListThreads + threadIdx.x;
    }
    __syncthreads();
    const int n = cnt;
    for (int i = threadIdx.x; i < n; i += kListThreads) {
      const int g = ids[i];
      const size_t at = (size_t)m * a.G + base + i;
      a.host_list[at] = g;
      if (a.packed) {
        // one 64-byte record per (model, host): id, batch row + 1 (-1: no candidate),
        // current level, k; the profile's free memory, times and SM levels
        const int B = a.batch[g];
        int4 r0 = make_int4(g, B < 0 ? -1 : min(B, kRows - 1) + 1, a.freq_cur[g], __float_as_int(a.kdyn[g]));
        int mem[4] = {0, 0, 0, 0}, tt[4] = {0, 0, 0, 0}, sm[4] = {-1, -1, -1, -1};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (s < a.S) {
            mem[s] = a.mem_free[(size_t)g * a.S + s];
            tt[s] = __float_as_int(a.t_avail[(size_t)g * a.S + s]);
            sm[s] = a.sm_free[(size_t)g * a.S + s];
          }
        int4 *rec = a.hrec + at * 4;
        rec[0] = r0;
        rec[1] = make_int4(mem[0], mem[1], mem[2], mem[3]);
        rec[2] = make_int4(tt[0], tt[1], tt[2], tt[3]);
        rec[3] = make_int4(sm[0], sm[1], sm[2], sm[3]);
      }
    }
    base += n;
    __syncthreads();                              // ids and cnt are rewritten
  }
  if (threadIdx.x == 0) a.host_cnt[m] = base;
}

struct Point {
  int ok;                        // the host has a profile step holding the memory
  double ta;                     // T_avail
  int sm, mem, b;
};

// GPU g's state as the launch sees it: the stored one, and in a wave-by-wave call with
// the previous wave's commits applied (batch grown, level boosted, memory taken; a step
// left short of memory reads -1 MiB).
template <bool kWaves>
__device__ __forceinline__ int view_batch(const DspArgs &a, int g) {
  if (!kWaves) return a.batch[g];
  return state_fb(a.wstate)[g].y + (int)(uint32_t)a.wprev[g];
}
template <bool kWaves>
__device__ __forceinline__ int view_freq(const DspArgs &a, int g) {
  if (!kWaves) return a.freq_cur[g];
  return (a.wprev[g] >> 32) ? a.NF - 1 : state_fb(a.wstate)[g].x;
}
template <bool kWaves>
__device__ __forceinline__ int view_mem(const DspArgs &a, int g, int s) {
  if (!kWaves) return a.mem_free[(size_t)g * a.S + s];
  const long long v = (long long)state_mem(a.wstate, a.G)[(size_t)g * a.S + s] - (long long)commit_taken(a.wprev, a.G)[(size_t)g * a.S + s];
  return v < -1 ? -1 : (int)v;
}

// Phase One for host g: first profile step whose free memory holds `need` KiB.
template <bool kWaves>
__device__ __forceinline__ Point host_point(const DspArgs &a, int g, long long need) {
  Point p{0, 0.0, -1, 0, 1};
  const int B = view_batch<kWaves>(a, g);
  if (B < 0) return p;
  p.b = min(B, kRows - 1) + 1;
  const size_t base = (size_t)g * a.S;
  if (a.S <= kMaxSteps) {
    int mem[kMaxSteps];
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s) mem[s] = s < a.S ? view_mem<kWaves>(a, g, s) : 0;
    int st = -1;
#pragma unroll
    for (int s = kMaxSteps - 1; s >= 0; --s)
      if (s < a.S && (long long)mem[s] * 1024 >= need) st = s;
    if (st < 0) return p;
    p.ok = 1;
    p.ta = (double)a.t_avail[base + st];
    p.sm = a.sm_free[base + st];
#pragma unroll
    for (int s = 0; s < kMaxSteps; ++s)
      if (s == st) p.mem = mem[s];
    return p;
  }
  for (int s = 0; s < a.S; ++s) {
    const int mem = view_mem<kWaves>(a, g, s);
    if ((long long)mem * 1024 >= need) {
      p.ok = 1;
      p.ta = (double)a.t_avail[base + s];
      p.sm = a.sm_free[base + s];
      p.mem = mem;
      return p;
    }
  }
  return p;
}

struct Host {
  int g, kcur;
  double kd;
  Point p;
};

// Phase One inputs of host number h of model m: from the packed record, or gathered.
template <bool kWaves>
__device__ __forceinline__ Host load_host(const DspArgs &a, int m, int h, const int *hl, long long need) {
  Host o;
  if (!kWaves && a.packed) {
    const v4i *rec = reinterpret_cast<const v4i *>(a.hrec + ((size_t)m * a.G + h) * 4);
    const v4i r0 = rec[0], mem = rec[1], tt = rec[2], sm = rec[3];
    __builtin_amdgcn_sched_barrier(0);   // the four loads in flight together, before any test
    o.g = r0.x;
    o.kcur = r0.z;
    o.kd = (double)__int_as_float(r0.w);
    o.p = Point{0, 0.0, -1, 0, r0.y};
    if (r0.y < 0) return o;
    int st = -1;
#pragma unroll
    for (int s = 3; s >= 0; --s)
      if (s < a.S && (long long)mem[s] * 1024 >= need) st = s;
    if (st < 0) return o;
    o.p.ok = 1;
    o.p.ta = (double)__int_as_float(st == 0 ? tt.x : st == 1 ? tt.y : st == 2 ? tt.z : tt.w);
    o.p.sm = st == 0 ? sm.x : st == 1 ? sm.y : st == 2 ? sm.z : sm.w;
    o.p.mem = st == 0 ? mem.x : st == 1 ? mem.y : st == 2 ? mem.z : mem.w;
    return o;
  }
  o.g = hl[h];
  o.kcur = view_freq<kWaves>(a, o.g);
  o.kd = (double)a.kdyn[o.g];
  o.p = host_point<kWaves>(a, o.g, need);
  return o;
}

// The SLO test and energy of one operating point from its gathered values: does the request
// (SLOs slo_ttft, slo_tbt) meet both starting at ta with batch b?  Energy if so.
__device__ __forceinline__ bool point_test(const DspArgs &a, float ttft, float tbt, float s, float f, int b, double ta,
                                           double kg, double lout, float slo_ttft, float slo_tbt, double &e) {
  if (!(ta + (double)ttft < (double)slo_ttft && tbt < slo_tbt)) return false;
  e = point_energy(a.p0, kg, (double)s, (double)f, (double)b / 32.0, (double)ttft, lout, (double)tbt);
  return (float)e < __builtin_huge_valf();
}

// Does the request meet its SLOs on (j, k) starting at ta with batch b?  Energy if so.
__device__ __forceinline__ bool point_ok(const DspArgs &a, int m, int prow, int b, int j, int k, double ta,
                                         double kg, double lout, float slo_ttft, float slo_tbt, double &e) {
  if (j < 0 || j >= a.NS || k < 0 || k >= a.NF) return false;
  const size_t cell = (size_t)j * a.NF + k;
  const float ttft = a.pf[((size_t)m * kRows + (prow >= 0 ? prow : b - 1)) * a.C + cell];
  const float tbt = a.dc[((size_t)m * kRows + (b - 1)) * a.C + cell];
  return point_test(a, ttft, tbt, a.sm_level[j], a.freq_level[k], b, ta, kg, lout, slo_ttft, slo_tbt, e);
}

// Stability order as one integer: more free memory, then more free SMs, then a lower GPU id
// is a larger key (memory biased to unsigned; SM level < 256; id < 2^24); 0 = no candidate.
__device__ __forceinline__ unsigned long long stability_key(int mem, int sm, int g) {
  return ((unsigned long long)((unsigned)mem ^ 0x80000000u) << 32) | ((unsigned long long)(sm & 0xff) << 24) |
         (unsigned long long)(0xffffffu - (unsigned)g);
}

// Lanes per request: 16 (four requests per wavefront) when a launch holds enough requests
// to fill the GPU, else 32 or 64, so that a request's hosts take fewer rounds of loads.
constexpr int kWideRequests = 2048;              // at most this many requests: 64 lanes each
constexpr int kMidRequests = 8192;               // at most this many: 32 lanes each
// At most kFewRequests requests on a fleet of at least kBlockGpus GPUs: a whole block each, so that
// its hosts take one round of loads (one request on 10,000 GPUs, 781 hosts: 64 lanes take 13).
constexpr int kFewRequests = 256, kBlockGpus = 2048;
constexpr int kCached = 4;                       // hosts per lane whose Phase One result stays in registers

// Reductions over the kGroup lanes of a request: shuffles inside a wavefront; a request of a
// whole block (kBlockLanes lanes) meets in LDS, and every thread of the block takes part.
constexpr int kBlockLanes = 512;
template <int kGroup>
__device__ __forceinline__ double group_min(double v) {
  constexpr int W = kGroup <= kWave ? kGroup : kWave;
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off, W));
  if constexpr (kGroup > kWave) {
    __shared__ double part[kGroup / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kGroup / kWave; ++i) v = fmin(v, part[i]);
  }
  return v;
}

template <int kGroup>
__device__ __forceinline__ unsigned long long group_max(unsigned long long v) {
  constexpr int W = kGroup <= kWave ? kGroup : kWave;
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) {
    const unsigned lo = __shfl_xor((unsigned)v, off, W), hi = __shfl_xor((unsigned)(v >> 32), off, W);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    v = o > v ? o : v;
  }
  if constexpr (kGroup > kWave) {
    __shared__ unsigned long long part[kGroup / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kGroup / kWave; ++i) v = part[i] > v ? part[i] : v;
  }
  return v;
}

// The pick of least (v, id): earliest time (F_max) or least energy (scale-out), then the lowest
// index; e and x travel with it.
__device__ __forceinline__ void pick_min(double &v, double &e, int &id, int &x, double ov, double oe, int oid, int ox) {
  if (ov < v || (ov == v && oid < id)) {
    v = ov;
    e = oe;
    id = oid;
    x = ox;
  }
}
template <int kGroup, int kUse>                   // kUse: one LDS array set per call site
__device__ __forceinline__ void group_pick(double &v, double &e, int &id, int &x) {
  constexpr int W = kGroup <= kWave ? kGroup : kWave;
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1)
    pick_min(v, e, id, x, __shfl_xor(v, off, W), __shfl_xor(e, off, W), __shfl_xor(id, off, W), __shfl_xor(x, off, W));
  if constexpr (kGroup > kWave) {
    __shared__ double pv[kGroup / kWave], pe[kGroup / kWave];
    __shared__ int pi[kGroup / kWave], px[kGroup / kWave];
    if ((threadIdx.x & (kWave - 1)) == 0) {
      const int i = threadIdx.x >> 6;
      pv[i] = v;
      pe[i] = e;
      pi[i] = id;
      px[i] = x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kGroup / kWave; ++i) pick_min(v, e, id, x, pv[i], pe[i], pi[i], px[i]);
  }
}

// kGroup lanes per request (64 / kGroup requests per wavefront, or one per block); lane s of a
// request strides over its model's hosts (s, s + kGroup, ...), all reductions stay inside the
// group.
template <int kGroup, bool kWaves>
__global__ void __launch_bounds__(kGroup <= kWave ? kWavesPerBlock * kWave : kGroup) k_dispatch(DspArgs a) {
#pragma clang fp contract(off)
  constexpr int kReqPerBlock = kGroup <= kWave ? kWavesPerBlock * kWave / kGroup : 1;
  if (kWaves) {
    // the state this wave sees, stored for the next wave; the commits after that cleared
    for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < a.G; g += gridDim.x * blockDim.x) {
      state_fb(a.wfold)[g] = make_int2(view_freq<true>(a, g), view_batch<true>(a, g));
      a.wnext[g] = 0ull;
      for (int s = 0; s < a.S; ++s) {
        const size_t at = (size_t)g * a.S + s;
        state_mem(a.wfold, a.G)[at] = view_mem<true>(a, g, s);
        commit_taken(a.wnext, a.G)[at] = 0ull;
      }
    }
  }
  const int sub = threadIdx.x & (kGroup - 1);
  const int r = a.r0 + blockIdx.x * kReqPerBlock + threadIdx.x / kGroup;
  if (r >= a.R) return;
  const double inf = __builtin_huge_val();
  const int m = a.model[r];
  const int pt = a.prompt[r], pd = a.pred[r];
  const float slo_ttft = a.slo_ttft[r], slo_tbt = a.slo_tbt[r];
  int gsel = -1, ksel = -1, jsel = -1, phase = 0;
  double esel = inf;
  bool writer = sub == 0;
  long long need = 0;
  if (m >= 0 && m < a.M && pd >= 0 && pt >= 0) {
    const int prow = pt == 0 ? -1 : (min((int)(((unsigned)pt + 255u) >> 8), kRows) - 1);
    const long long lout_i = ((long long)pd * 105 + 99) / 100;
    const double lout = (double)lout_i;
    need = (long long)a.kv[m] * ((long long)pt + lout_i);
    const int nh = a.host_cnt[m];
    const int *hl = a.host_list + (size_t)m * a.G;
    // Phase One at every host, least energy; the first kCached hosts of a lane are kept
    double emin = inf;
    double ec[kCached];
    unsigned long long kc[kCached];
#pragma unroll
    for (int i = 0; i < kCached; ++i) {
      ec[i] = inf;
      kc[i] = 0ull;
    }
    for (int i = 0, h = sub; h < nh; ++i, h += kGroup) {
      const Host H = load_host<kWaves>(a, m, h, hl, need);
      const int g = H.g;
      const Point &p = H.p;
      double e;
      if (!(p.ok && point_ok(a, m, prow, p.b, p.sm, H.kcur, p.ta, H.kd, lout, slo_ttft, slo_tbt, e))) continue;
      emin = fmin(emin, e);
#pragma unroll
      for (int c = 0; c < kCached; ++c)
        if (i == c) {
          ec[c] = e;
          kc[c] = stability_key(p.mem, p.sm, g);
        }
    }
    emin = group_min<kGroup>(emin);
    if (emin < inf) {
      // Phase Two: the largest stability key among the hosts within 2% of the least energy
      const double bound = emin + kStability * fabs(emin);
      unsigned long long best = 0ull;
      double ebest = inf;
#pragma unroll
      for (int c = 0; c < kCached; ++c)
        if (kc[c] > best && ec[c] <= bound) {
          best = kc[c];
          ebest = ec[c];
        }
      for (int h = sub + kCached * kGroup; h < nh; h += kGroup) {   // hosts past the cached ones
        const Host H = load_host<kWaves>(a, m, h, hl, need);
        const int g = H.g;
        const Point &p = H.p;
        double e;
        if (!(p.ok && point_ok(a, m, prow, p.b, p.sm, H.kcur, p.ta, H.kd, lout, slo_ttft, slo_tbt, e))) continue;
        const unsigned long long key = stability_key(p.mem, p.sm, g);
        if (e <= bound && key > best) {
          best = key;
          ebest = e;
        }
      }
      const unsigned long long wbest = group_max<kGroup>(best);
      if (wbest != 0ull) {                 // the least-energy host is within the bound, unless E_min = -inf
        writer = best == wbest;            // exactly one lane of the group holds the winning key
        gsel = (int)(0xffffffu - (unsigned)(wbest & 0xffffffull));
        jsel = (int)((wbest >> 24) & 0xffull);
        ksel = view_freq<kWaves>(a, gsel);   // the winner's current level
        phase = 1;
        esel = ebest;
      }
    } else {
      // Phase Three: the earliest available host that meets the SLOs at the top level
      const int kmax = a.NF - 1;
      int bg = INT_MAX, bsm = -1;
      double bt = inf, be = inf;
      for (int h = sub; h < nh; h += kGroup) {
        const Host H = load_host<kWaves>(a, m, h, hl, need);
        const int g = H.g;
        const Point &p = H.p;
        double e;
        if (!(p.ok && point_ok(a, m, prow, p.b, p.sm, kmax, p.ta, H.kd, lout, slo_ttft, slo_tbt, e))) continue;
        pick_min(bt, be, bg, bsm, p.ta, e, g, p.sm);
      }
      group_pick<kGroup, 0>(bt, be, bg, bsm);
      if (bg != INT_MAX) {
        gsel = bg;
        ksel = kmax;
        jsel = bsm;
        phase = 2;
        esel = be;
      } else {
        // scale out: a new GPU (batch 1, every SM, available now), lane s scores levels s, s + kGroup, ...
        int bk = INT_MAX, none = 0;
        double bke = inf, same = inf;
        for (int k = sub; k < a.NF; k += kGroup) {
          double e;
          if (point_ok(a, m, prow, 1, a.NS - 1, k, 0.0, a.k_new, lout, slo_ttft, slo_tbt, e)) pick_min(bke, same, bk, none, e, e, k, 0);
        }
        group_pick<kGroup, 1>(bke, same, bk, none);
        if (bk != INT_MAX) {
          ksel = bk;
          jsel = a.NS - 1;
          phase = 3;
          esel = bke;
        }
      }
    }
  }
  if (writer) {
    a.out_gpu[r] = gsel;
    a.out_freq[r] = ksel;
    a.out_sm[r] = jsel;
    a.out_phase[r] = (uint8_t)phase;
    a.out_energy[r] = (float)esel;
    if (kWaves && (phase == 1 || phase == 2)) {
      // commit to the chosen GPU: one more request in its batch, and ceil(Req_mem / 1024)
      // MiB from the step that admitted it (the first whose free memory holds Req_mem) on
      const size_t base = (size_t)gsel * a.S;
      int st = 0;
      while (st < a.S - 1 && (long long)view_mem<true>(a, gsel, st) * 1024 < need) ++st;
      const unsigned long long q = (unsigned long long)((need + 1023) / 1024);
      atomicAdd(&a.wcur[gsel], phase == 2 ? (1ull << 32) | 1ull : 1ull);
      for (int s = st; s < a.S; ++s) atomicAdd(&commit_taken(a.wcur, a.G)[base + s], q);
    }
  }
}

// Start of a wave-by-wave call: the caller's state copied into the first state buffer, the
// three commit buffers cleared.
__global__ void __launch_bounds__(kHostBlock) k_wave_init(int32_t G, int32_t S, int32_t *st0, unsigned long long *c0,
                                                          unsigned long long *c1, unsigned long long *c2,
                                                          const int32_t *freq0, const int32_t *batch0,
                                                          const int32_t *mem0) {
  const int g = blockIdx.x * kHostBlock + threadIdx.x;
  if (g >= G) return;
  state_fb(st0)[g] = make_int2(freq0[g], batch0[g]);
  c0[g] = c1[g] = c2[g] = 0ull;
  for (int s = 0; s < S; ++s) {
    const size_t at = (size_t)g * S + s;
    state_mem(st0, G)[at] = mem0[at];
    commit_taken(c0, G)[at] = commit_taken(c1, G)[at] = commit_taken(c2, G)[at] = 0ull;
  }
}

// End of a wave-by-wave call: the last state with the last wave's commits applied, into
// the caller's arrays.
__global__ void __launch_bounds__(kHostBlock) k_wave_final(DspArgs a, int32_t *freq, int32_t *batch, int32_t *mem) {
  const int g = blockIdx.x * kHostBlock + threadIdx.x;
  if (g >= a.G) return;
  batch[g] = view_batch<true>(a, g);
  freq[g] = view_freq<true>(a, g);
  for (int s = 0; s < a.S; ++s) mem[(size_t)g * a.S + s] = view_mem<true>(a, g, s);
}

// ------------------------------------------------------------------ waves, at most 4 profile steps
// Per GPU, 16-byte words: profile (as given, read-only) {k, 0, 0, 0}, {T_avail[4]}, {SM_free[4]};
// state {level, batch, 0, 0}, {free MiB[4]}; commits {requests placed | F_max << 32, 0}, {MiB
// taken at step 0, 1}, {at 2, 3}, counted at the admitting step only (a view adds them up).
constexpr int kProf4 = 3, kState4 = 2, kCommit4 = 3;

struct Wave4 {
  const v4i *prof, *state;
  const v4i *prev;
  v4i *next_state, *next;        // the next wave's state; the commits of the wave after (cleared)
  unsigned long long *cur;       // this wave's commits
};

struct View4 {
  int freq, batch, mem[4];
};

// A GPU's state with the previous wave's commits applied.
__device__ __forceinline__ View4 view4(const DspArgs &a, v4i s0, v4i s1, v4i c0, v4i c1, v4i c2) {
  View4 v;
  v.freq = c0.y ? a.NF - 1 : s0.x;
  v.batch = s0.y + c0.x;
  const long long t[4] = {(long long)((unsigned long long)(unsigned)c1.x | ((unsigned long long)(unsigned)c1.y << 32)),
                          (long long)((unsigned long long)(unsigned)c1.z | ((unsigned long long)(unsigned)c1.w << 32)),
                          (long long)((unsigned long long)(unsigned)c2.x | ((unsigned long long)(unsigned)c2.y << 32)),
                          (long long)((unsigned long long)(unsigned)c2.z | ((unsigned long long)(unsigned)c2.w << 32))};
  long long sum = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    sum += t[s];
    const long long m = (long long)s1[s] - sum;
    v.mem[s] = m < -1 ? -1 : (int)m;
  }
  return v;
}

// One host of a lane: its point for the request (Phase One) and what committing to it needs.
struct Host4 {
  int g, b, sm, mem, step, freq;
  float kd, ta;
};

// Hosts i, i + stride, ... (kBatch of them, those below n) of model m, each group of loads in
// flight together.  step < 0: no candidate.
template <int kBatch>
__device__ __forceinline__ void load_hosts4(const DspArgs &a, const Wave4 &w, const int *hl, int n, int i, int stride,
                                            long long need, Host4 (&o)[kBatch]) {
  // mem * 1024 >= need as mem >= ceil(need / 1024), in 32 bits (a need beyond them: no host)
  const long long up = (need + 1023) >> 10;
  const int mib = up < INT_MIN ? INT_MIN : (int)(up > INT_MAX ? INT_MAX : up);
  const bool fits = up <= INT_MAX;
  int g[kBatch];
#pragma unroll
  for (int c = 0; c < kBatch; ++c) g[c] = hl[min(i + c * stride, a.G - 1)];
#pragma unroll
  for (int c = 0; c < kBatch; ++c) g[c] = i + c * stride < n ? g[c] : 0;   // past the list: any GPU
  v4i p0[kBatch], p1[kBatch], p2[kBatch], s0[kBatch], s1[kBatch], c0[kBatch], c1[kBatch], c2[kBatch];
#pragma unroll
  for (int c = 0; c < kBatch; ++c) {
    const v4i *p = w.prof + (size_t)g[c] * kProf4, *s = w.state + (size_t)g[c] * kState4,
              *q = w.prev + (size_t)g[c] * kCommit4;
    p0[c] = p[0];
    p1[c] = p[1];
    p2[c] = p[2];
    s0[c] = s[0];
    s1[c] = s[1];
    c0[c] = q[0];
    c1[c] = q[1];
    c2[c] = q[2];
  }
  __builtin_amdgcn_sched_barrier(0);             // every load is issued before the first use
#pragma unroll
  for (int c = 0; c < kBatch; ++c) {
    const View4 v = view4(a, s0[c], s1[c], c0[c], c1[c], c2[c]);
    int st = -1;
#pragma unroll
    for (int s = 3; s >= 0; --s)
      if (s < a.S && v.mem[s] >= mib) st = s;
    if (v.batch < 0 || i + c * stride >= n || !fits) st = -1;
    o[c].g = g[c];
    o[c].b = min(v.batch, kRows - 1) + 1;
    o[c].freq = v.freq;
    o[c].kd = __int_as_float(p0[c].x);
    o[c].step = st;
    o[c].ta = __int_as_float(st <= 0 ? p1[c].x : st == 1 ? p1[c].y : st == 2 ? p1[c].z : p1[c].w);
    o[c].sm = st <= 0 ? p2[c].x : st == 1 ? p2[c].y : st == 2 ? p2[c].z : p2[c].w;
    o[c].mem = st <= 0 ? v.mem[0] : st == 1 ? v.mem[1] : st == 2 ? v.mem[2] : v.mem[3];
  }
}

// Energies of kBatch points at their own level (k < 0) or level k; inf where the request's SLOs
// are missed.  The table entries of all points are loaded together.
template <int kBatch>
__device__ __forceinline__ void points4(const DspArgs &a, const float *s_sm, const float *s_f, int m, int prow, int k,
                                        double lout, float slo_ttft, float slo_tbt, const Host4 (&h)[kBatch],
                                        double (&e)[kBatch]) {
  float ttft[kBatch], tbt[kBatch];
  bool ok[kBatch];
  int kk[kBatch], jj[kBatch];
#pragma unroll
  for (int c = 0; c < kBatch; ++c) {
    kk[c] = k < 0 ? h[c].freq : k;
    jj[c] = h[c].sm;
    ok[c] = h[c].step >= 0 && jj[c] >= 0 && jj[c] < a.NS && kk[c] >= 0 && kk[c] < a.NF;
    if (!ok[c]) kk[c] = jj[c] = 0;
    const int b = ok[c] ? h[c].b : 1;
    const size_t cell = (size_t)jj[c] * a.NF + kk[c];
    ttft[c] = a.pf[((size_t)m * kRows + (prow >= 0 ? prow : b - 1)) * a.C + cell];
    tbt[c] = a.dc[((size_t)m * kRows + (b - 1)) * a.C + cell];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < kBatch; ++c) {
    double x;
    const bool in = ok[c] && point_test(a, ttft[c], tbt[c], s_sm[jj[c]], s_f[kk[c]], h[c].b, (double)h[c].ta,
                                        (double)h[c].kd, lout, slo_ttft, slo_tbt, x);
    e[c] = in ? x : __builtin_huge_val();
  }
}

// One wave: k_dispatch's phases over hosts in batches; a lane's first batch stays in registers.
template <int kGroup, int kBatch>
__global__ void __launch_bounds__(kWavesPerBlock * kWave) k_dispatch4(DspArgs a, Wave4 w) {
#pragma clang fp contract(off)
  __shared__ float s_sm[FESTINA_MAX_CELLS], s_f[FESTINA_MAX_CELLS];
  for (int i = threadIdx.x; i < a.NS; i += blockDim.x) s_sm[i] = a.sm_level[i];
  for (int i = threadIdx.x; i < a.NF; i += blockDim.x) s_f[i] = a.freq_level[i];
  const int sub = threadIdx.x & (kGroup - 1);
  const int r = a.r0 + blockIdx.x * (kWavesPerBlock * kWave / kGroup) + threadIdx.x / kGroup;
  const int rc = min(r, a.R - 1);
  const int m = a.model[rc], pt = a.prompt[rc], pd = a.pred[rc];
  const float slo_ttft = a.slo_ttft[rc], slo_tbt = a.slo_tbt[rc];
  // the state this wave sees, stored for the next wave; the commits after that cleared
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < a.G; g += gridDim.x * blockDim.x) {
    const v4i *s = w.state + (size_t)g * kState4, *q = w.prev + (size_t)g * kCommit4;
    const View4 v = view4(a, s[0], s[1], q[0], q[1], q[2]);
    w.next_state[(size_t)g * kState4] = v4i{v.freq, v.batch, 0, 0};
    w.next_state[(size_t)g * kState4 + 1] = v4i{v.mem[0], v.mem[1], v.mem[2], v.mem[3]};
#pragma unroll
    for (int i = 0; i < kCommit4; ++i) w.next[(size_t)g * kCommit4 + i] = v4i{0, 0, 0, 0};
  }
  __syncthreads();
  if (r >= a.R) return;
  const double inf = __builtin_huge_val();
  int gsel = -1, ksel = -1, jsel = -1, phase = 0, step = 0;
  double esel = inf;
  bool writer = sub == 0;
  long long need = 0;
  if (m >= 0 && m < a.M && pd >= 0 && pt >= 0) {
    const int prow = pt == 0 ? -1 : (min((int)(((unsigned)pt + 255u) >> 8), kRows) - 1);
    const long long lout_i = ((long long)pd * 105 + 99) / 100;
    const double lout = (double)lout_i;
    const int *hl = a.host_list + (size_t)m * a.G;
    const int nh = a.host_cnt[m];
    need = (long long)a.kv[m] * ((long long)pt + lout_i);
    Host4 first[kBatch];
    double ef[kBatch];
    load_hosts4<kBatch>(a, w, hl, nh, sub, kGroup, need, first);
    points4<kBatch>(a, s_sm, s_f, m, prow, -1, lout, slo_ttft, slo_tbt, first, ef);
    double emin = inf;
#pragma unroll
    for (int c = 0; c < kBatch; ++c) emin = fmin(emin, ef[c]);
    for (int h = sub + kBatch * kGroup; h < nh; h += kBatch * kGroup) {
      Host4 o[kBatch];
      double e[kBatch];
      load_hosts4<kBatch>(a, w, hl, nh, h, kGroup, need, o);
      points4<kBatch>(a, s_sm, s_f, m, prow, -1, lout, slo_ttft, slo_tbt, o, e);
#pragma unroll
      for (int c = 0; c < kBatch; ++c) emin = fmin(emin, e[c]);
    }
    emin = group_min<kGroup>(emin);
    if (emin < inf) {
      // Phase Two: the largest stability key among the hosts within 2% of the least energy
      const double bound = emin + kStability * fabs(emin);
      unsigned long long best = 0ull;
      const auto offer = [&](const Host4 &o, double e) {
        const unsigned long long key = stability_key(o.mem, o.sm, o.g);
        if (e < inf && e <= bound && key > best) {
          best = key;
          esel = e;
          ksel = o.freq;
          step = o.step;
        }
      };
#pragma unroll
      for (int c = 0; c < kBatch; ++c) offer(first[c], ef[c]);
      for (int h = sub + kBatch * kGroup; h < nh; h += kBatch * kGroup) {
        Host4 o[kBatch];
        double e[kBatch];
        load_hosts4<kBatch>(a, w, hl, nh, h, kGroup, need, o);
        points4<kBatch>(a, s_sm, s_f, m, prow, -1, lout, slo_ttft, slo_tbt, o, e);
#pragma unroll
        for (int c = 0; c < kBatch; ++c) offer(o[c], e[c]);
      }
      const unsigned long long wbest = group_max<kGroup>(best);
      // (no key: E_min = -inf, of a -inf input, makes the bound NaN and no host is offered)
      if (wbest != 0ull) {
        writer = best == wbest;            // exactly one lane of the group holds the winning key
        gsel = (int)(0xffffffu - (unsigned)(wbest & 0xffffffull));
        jsel = (int)((wbest >> 24) & 0xffull);
        phase = 1;
      }
    } else {
      // Phase Three: the earliest available host that meets the SLOs at the top level
      int bg = INT_MAX, bsm = -1;
      double bt = inf, be = inf;
      const auto take = [&](const Host4 &o, double e) {
        if (e < inf) pick_min(bt, be, bg, bsm, (double)o.ta, e, o.g, o.sm | (o.step << 16));
      };
      points4<kBatch>(a, s_sm, s_f, m, prow, a.NF - 1, lout, slo_ttft, slo_tbt, first, ef);
#pragma unroll
      for (int c = 0; c < kBatch; ++c) take(first[c], ef[c]);
      for (int h = sub + kBatch * kGroup; h < nh; h += kBatch * kGroup) {
        Host4 o[kBatch];
        double e[kBatch];
        load_hosts4<kBatch>(a, w, hl, nh, h, kGroup, need, o);
        points4<kBatch>(a, s_sm, s_f, m, prow, a.NF - 1, lout, slo_ttft, slo_tbt, o, e);
#pragma unroll
        for (int c = 0; c < kBatch; ++c) take(o[c], e[c]);
      }
      group_pick<kGroup, 0>(bt, be, bg, bsm);
      if (bg != INT_MAX) {
        gsel = bg;
        ksel = a.NF - 1;
        jsel = bsm & 0xffff;
        step = bsm >> 16;
        phase = 2;
        esel = be;
      } else {
        // scale out: a new GPU (batch 1, every SM, available now), lane s scores levels s, s + kGroup, ...
        int bk = INT_MAX, none = 0;
        double bke = inf, same = inf;
        for (int k = sub; k < a.NF; k += kGroup) {
          double e;
          if (point_ok(a, m, prow, 1, a.NS - 1, k, 0.0, a.k_new, lout, slo_ttft, slo_tbt, e)) pick_min(bke, same, bk, none, e, e, k, 0);
        }
        group_pick<kGroup, 1>(bke, same, bk, none);
        if (bk != INT_MAX) {
          ksel = bk;
          jsel = a.NS - 1;
          phase = 3;
          esel = bke;
        }
      }
    }
  }
  if (writer) {
    a.out_gpu[r] = gsel;
    a.out_freq[r] = ksel;
    a.out_sm[r] = jsel;
    a.out_phase[r] = (uint8_t)phase;
    a.out_energy[r] = (float)esel;
    if (phase == 1 || phase == 2) {
      // commit: one more request in the GPU's batch, ceil(Req_mem / 1024) MiB from `step` on
      unsigned long long *q = w.cur + (size_t)gsel * 2 * kCommit4;
      atomicAdd(q, phase == 2 ? (1ull << 32) | 1ull : 1ull);
      atomicAdd(q + 2 + step, (unsigned long long)((need + 1023) / 1024));
    }
  }
}

// Start of a wave-by-wave call: profiles and state packed, the commit buffers cleared.
__global__ void __launch_bounds__(kHostBlock) k_wave4_init(DspArgs a, v4i *prof, v4i *state, v4i *c0, v4i *c1, v4i *c2) {
  const int g = blockIdx.x * kHostBlock + threadIdx.x;
  if (g >= a.G) return;
  v4i mem{0, 0, 0, 0}, tt{0, 0, 0, 0}, sm{-1, -1, -1, -1};
#pragma unroll
  for (int s = 0; s < 4; ++s)
    if (s < a.S) {
      mem[s] = a.mem_free[(size_t)g * a.S + s];
      tt[s] = __float_as_int(a.t_avail[(size_t)g * a.S + s]);
      sm[s] = a.sm_free[(size_t)g * a.S + s];
    }
  prof[(size_t)g * kProf4] = v4i{__float_as_int(a.kdyn[g]), 0, 0, 0};
  prof[(size_t)g * kProf4 + 1] = tt;
  prof[(size_t)g * kProf4 + 2] = sm;
  state[(size_t)g * kState4] = v4i{a.freq_cur[g], a.batch[g], 0, 0};
  state[(size_t)g * kState4 + 1] = mem;
#pragma unroll
  for (int i = 0; i < kCommit4; ++i) c0[(size_t)g * kCommit4 + i] = c1[(size_t)g * kCommit4 + i] = c2[(size_t)g * kCommit4 + i] = v4i{0, 0, 0, 0};
}

// End of a wave-by-wave call: the last state with the last wave's commits applied, into the
// caller's arrays.
__global__ void __launch_bounds__(kHostBlock) k_wave4_final(DspArgs a, Wave4 w, int32_t *freq, int32_t *batch, int32_t *mem) {
  const int g = blockIdx.x * kHostBlock + threadIdx.x;
  if (g >= a.G) return;
  const v4i *s = w.state + (size_t)g * kState4, *q = w.prev + (size_t)g * kCommit4;
  const View4 v = view4(a, s[0], s[1], q[0], q[1], q[2]);
  freq[g] = v.freq;
  batch[g] = v.batch;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < a.S) mem[(size_t)g * a.S + i] = v.mem[i];
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

bool dsp_shapes_ok(const festina_lut *L, const festina_gpu_avail *A) {
  if (!L || !A) return false;
  if (L->n_models < 1 || L->n_rows != kRows || L->n_sm < 1 || L->n_freq < 1) return false;
  if (A->n_gpus < 1 || A->n_steps < 1) return false;
  if ((long long)L->n_models * A->n_gpus > INT_MAX) return false;
  if (A->n_gpus > 0xffffff) return false;       // GPU ids are packed in 24 bits
  return true;
}

}  // namespace

extern "C" size_t festina_dispatch_workspace_bytes(const festina_lut *L, const festina_gpu_avail *A) {
  if (!dsp_shapes_ok(L, A)) return 0;
  size_t bytes = align256(sizeof(int32_t) * L->n_models) + align256(sizeof(int32_t) * (size_t)L->n_models * A->n_gpus);
  if (A->n_steps <= 4) bytes += align256((size_t)64 * L->n_models * A->n_gpus);     // host records
  return bytes;
}

// k_dispatch over requests lo .. hi-1, with the group width their number calls for.
template <bool kWaves>
static festina_status launch_dispatch(DspArgs a, int32_t lo, int32_t hi, hipStream_t st) {
  a.r0 = lo;
  a.R = hi;
  const long long n = (long long)hi - lo;
  if (n <= kFewRequests && a.G >= kBlockGpus) {
    k_dispatch<kBlockLanes, kWaves><<<(unsigned)n, kBlockLanes, 0, st>>>(a);
  } else if (n <= kWideRequests) {
    const long long per_block = (long long)kWavesPerBlock * (kWave / 64);
    k_dispatch<64, kWaves><<<(unsigned)((n + per_block - 1) / per_block), kWavesPerBlock * kWave, 0, st>>>(a);
  } else if (n <= kMidRequests) {
    const long long per_block = (long long)kWavesPerBlock * (kWave / 32);
    k_dispatch<32, kWaves><<<(unsigned)((n + per_block - 1) / per_block), kWavesPerBlock * kWave, 0, st>>>(a);
  } else {
    const long long per_block = (long long)kWavesPerBlock * (kWave / 16);
    k_dispatch<16, kWaves><<<(unsigned)((n + per_block - 1) / per_block), kWavesPerBlock * kWave, 0, st>>>(a);
  }
  return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
}

// Checks the arguments common to both dispatch calls; fills everything but the workspace.
static festina_status dsp_args(const festina_lut *L, const festina_gpu_avail *A, const festina_requests *Q,
                               festina_dispatches *out, DspArgs &a) {
  if (!dsp_shapes_ok(L, A) || !Q || !out || Q->n_requests < 0) return FESTINA_ERR_INVALID;
  const long long C = (long long)L->n_sm * L->n_freq;
  if (C > FESTINA_MAX_CELLS) return FESTINA_ERR_UNSUPPORTED;
  if (!L->sm_level || !L->freq_level || !L->pf || !L->dc) return FESTINA_ERR_INVALID;
  if (!A->freq_cur || !A->batch || !A->k_dyn_w || !A->resident || !A->t_avail_ms || !A->mem_free_mib ||
      !A->sm_free || !A->kv_kib_per_token)
    return FESTINA_ERR_INVALID;
  if (Q->n_requests > 0) {
    if (!Q->model || !Q->prompt_tokens || !Q->pred_out_tokens || !Q->slo_ttft_ms || !Q->slo_tbt_ms)
      return FESTINA_ERR_INVALID;
    if (!out->gpu || !out->freq_level || !out->sm_level || !out->phase || !out->energy_mj) return FESTINA_ERR_INVALID;
  }
  a.M = L->n_models;
  a.NS = L->n_sm;
  a.NF = L->n_freq;
  a.C = (int32_t)C;
  a.words = (L->n_models + 31) / 32;
  a.sm_level = L->sm_level;
  a.freq_level = L->freq_level;
  a.pf = L->pf;
  a.dc = L->dc;
  a.p0 = (double)L->p0_w;
  a.G = A->n_gpus;
  a.S = A->n_steps;
  a.freq_cur = A->freq_cur;
  a.batch = A->batch;
  a.kdyn = A->k_dyn_w;
  a.resident = A->resident;
  a.t_avail = A->t_avail_ms;
  a.mem_free = A->mem_free_mib;
  a.sm_free = A->sm_free;
  a.kv = A->kv_kib_per_token;
  a.k_new = (double)A->k_new_w;
  a.R = Q->n_requests;
  a.model = Q->model;
  a.prompt = Q->prompt_tokens;
  a.pred = Q->pred_out_tokens;
  a.slo_ttft = Q->slo_ttft_ms;
  a.slo_tbt = Q->slo_tbt_ms;
  a.out_gpu = out->gpu;
  a.out_freq = out->freq_level;
  a.out_sm = out->sm_level;
  a.out_phase = out->phase;
  a.out_energy = out->energy_mj;
  a.r0 = 0;
  a.wstate = a.wfold = nullptr;
  a.wprev = a.wcur = a.wnext = nullptr;
  a.packed = 0;
  a.hrec = nullptr;
  return FESTINA_OK;
}

extern "C" festina_status festina_dispatch_requests(const festina_lut *L, const festina_gpu_avail *A,
                                                    const festina_requests *Q, festina_dispatches *out,
                                                    void *workspace, size_t workspace_bytes, void *stream) {
  DspArgs a;
  const festina_status chk = dsp_args(L, A, Q, out, a);
  if (chk != FESTINA_OK) return chk;
  const size_t need = festina_dispatch_workspace_bytes(L, A);
  if (!workspace || workspace_bytes < need || (((uintptr_t)workspace) & 255) != 0) return FESTINA_ERR_INVALID;
  if (Q->n_requests == 0) return FESTINA_OK;
  char *ws = static_cast<char *>(workspace);
  a.host_cnt = reinterpret_cast<int32_t *>(ws);
  a.host_list = reinterpret_cast<int32_t *>(ws + align256(sizeof(int32_t) * L->n_models));
  a.packed = A->n_steps <= 4 ? 1 : 0;
  a.hrec = reinterpret_cast<int4 *>(ws + align256(sizeof(int32_t) * L->n_models) +
                                    align256(sizeof(int32_t) * (size_t)L->n_models * A->n_gpus));
  hipStream_t st = static_cast<hipStream_t>(stream);
  k_dsp_hosts<<<a.M, kListThreads, 0, st>>>(a);
  if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  return launch_dispatch<false>(a, 0, a.R, st);
}

// Workspace of a wave-by-wave call: host counts and lists, two state buffers (the state
// each wave sees alternates between them) and three commit buffers (the previous wave's,
// read; the current wave's, written; the next wave's, cleared); the packed profiles when they
// have at most 4 steps.
constexpr int kSteps4 = 4;
static size_t state_bytes(size_t G, size_t S) {
  return align256(S <= kSteps4 ? sizeof(v4i) * kState4 * G : sizeof(int32_t) * (2 * G + G * S));
}
static size_t commit_bytes(size_t G, size_t S) {
  return align256(S <= kSteps4 ? sizeof(v4i) * kCommit4 * G : sizeof(unsigned long long) * (G + G * S));
}
static size_t profile_bytes(size_t G, size_t S) { return S <= kSteps4 ? align256(sizeof(v4i) * kProf4 * G) : 0; }

extern "C" size_t festina_dispatch_waves_workspace_bytes(const festina_lut *L, const festina_gpu_avail *A) {
  if (!dsp_shapes_ok(L, A)) return 0;
  const size_t G = (size_t)A->n_gpus, S = (size_t)A->n_steps;
  return align256(sizeof(int32_t) * L->n_models) + align256(sizeof(int32_t) * (size_t)L->n_models * G) +
         2 * state_bytes(G, S) + 3 * commit_bytes(G, S) + profile_bytes(G, S);
}

// k_dispatch4 over requests lo .. hi-1.  A wave's kernel is a chain of memory round trips (the
// previous wave's state comes from beyond the L2s): 64 lanes x 2 hosts take 128 hosts in one
// chain.  Waves of 256 / 4,096 / 32,768 requests on 1,024 GPUs (80 hosts each) take 7.1 / 11.7 / 67 us
// each; when the split was chosen 7.8 / 14.9 / 65, against 10.4 / 14.7 / 71 with 32 lanes x 4, 17.5 /
// 18.8 / 76 with 16 x 4 and 12.2 / 25.4 / 129 with k_dispatch's loop over single hosts.  On a small fleet most of 64 lanes would
// have no host: 4,096 requests on 128 GPUs take 10.9 us with 64 lanes, 9.9 with 16.  A launch holds
// fewer than 2^32 threads, so waves of 2^26 requests or more take 16 lanes whatever the fleet.
constexpr int kSmallFleet = 256, kNarrowRequests = 2048, kWidestRequests = (1 << 26) - 1;
static festina_status launch_dispatch4(DspArgs a, const Wave4 &w, int32_t lo, int32_t hi, hipStream_t st) {
  a.r0 = lo;
  a.R = hi;
  const long long n = (long long)hi - lo;
  constexpr int T = kWavesPerBlock * kWave;
  const auto blocks = [&](int group) { return (unsigned)((n * group + T - 1) / T); };
  if ((a.G <= kSmallFleet && n > kNarrowRequests) || n > kWidestRequests)
    k_dispatch4<16, 4><<<blocks(16), T, 0, st>>>(a, w);
  else
    k_dispatch4<64, 2><<<blocks(64), T, 0, st>>>(a, w);
  return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
}

extern "C" festina_status festina_dispatch_waves(const festina_lut *L, const festina_gpu_avail *A,
                                                 const festina_requests *Q, int32_t n_waves,
                                                 const int32_t *wave_start, festina_gpu_state *state,
                                                 festina_dispatches *out, void *workspace, size_t workspace_bytes,
                                                 void *stream) {
  DspArgs a;
  const festina_status chk = dsp_args(L, A, Q, out, a);
  if (chk != FESTINA_OK) return chk;
  if (!state || !state->freq_cur || !state->batch || !state->mem_free_mib || n_waves < 0) return FESTINA_ERR_INVALID;
  if (n_waves == 0) {
    if (Q->n_requests != 0) return FESTINA_ERR_INVALID;
  } else {
    if (!wave_start || wave_start[0] != 0 || wave_start[n_waves] != Q->n_requests) return FESTINA_ERR_INVALID;
    for (int32_t w = 0; w < n_waves; ++w)
      if (wave_start[w + 1] < wave_start[w]) return FESTINA_ERR_INVALID;
  }
  const size_t need = festina_dispatch_waves_workspace_bytes(L, A);
  if (!workspace || workspace_bytes < need || (((uintptr_t)workspace) & 255) != 0) return FESTINA_ERR_INVALID;
  const size_t G = (size_t)A->n_gpus, S = (size_t)A->n_steps;
  char *ws = static_cast<char *>(workspace);
  size_t at = 0;
  auto take = [&](size_t bytes) {
    char *p = ws + at;
    at += align256(bytes);
    return p;
  };
  a.host_cnt = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * L->n_models));
  a.host_list = reinterpret_cast<int32_t *>(take(sizeof(int32_t) * (size_t)L->n_models * G));
  char *sb[2], *db[3];
  for (char *&x : sb) x = take(state_bytes(G, S));
  for (char *&x : db) x = take(commit_bytes(G, S));
  v4i *prof = reinterpret_cast<v4i *>(take(profile_bytes(G, S)));
  const bool packed = S <= kSteps4;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const unsigned gblocks = (unsigned)((G + kHostBlock - 1) / kHostBlock);
  const auto i32 = [](char *p) { return reinterpret_cast<int32_t *>(p); };
  const auto u64 = [](char *p) { return reinterpret_cast<unsigned long long *>(p); };
  const auto w16 = [](char *p) { return reinterpret_cast<v4i *>(p); };
  if (packed)
    k_wave4_init<<<gblocks, kHostBlock, 0, st>>>(a, prof, w16(sb[0]), w16(db[0]), w16(db[1]), w16(db[2]));
  else
    k_wave_init<<<gblocks, kHostBlock, 0, st>>>(A->n_gpus, A->n_steps, i32(sb[0]), u64(db[0]), u64(db[1]), u64(db[2]),
                                                A->freq_cur, A->batch, A->mem_free_mib);
  if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  if (Q->n_requests > 0) {
    k_dsp_hosts<<<a.M, kListThreads, 0, st>>>(a);
    if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  }
  // Launch v (of the non-empty waves) sees sb[v % 2] with db[(v + 2) % 3] applied, stores
  // that in sb[(v + 1) % 2], commits to db[v % 3] and clears db[(v + 1) % 3].
  a.freq_cur = a.batch = a.mem_free = nullptr;
  int v = 0;
  for (int32_t w = 0; w < n_waves; ++w) {
    const int32_t lo = wave_start[w], hi = wave_start[w + 1];
    if (hi == lo) continue;
    char *seen = sb[v % 2], *fold = sb[(v + 1) % 2], *prev = db[(v + 2) % 3], *cur = db[v % 3], *next = db[(v + 1) % 3];
    festina_status s;
    if (packed) {
      s = launch_dispatch4(a, Wave4{prof, w16(seen), w16(prev), w16(fold), w16(next), u64(cur)}, lo, hi, st);
    } else {
      a.wstate = i32(seen);
      a.wfold = i32(fold);
      a.wprev = u64(prev);
      a.wcur = u64(cur);
      a.wnext = u64(next);
      s = launch_dispatch<true>(a, lo, hi, st);
    }
    if (s != FESTINA_OK) return FESTINA_ERR_DEVICE;
    ++v;
  }
  if (packed) {
    const Wave4 w{prof, w16(sb[v % 2]), w16(db[(v + 2) % 3]), nullptr, nullptr, nullptr};
    k_wave4_final<<<gblocks, kHostBlock, 0, st>>>(a, w, state->freq_cur, state->batch, state->mem_free_mib);
  } else {
    a.wstate = i32(sb[v % 2]);
    a.wprev = u64(db[(v + 2) % 3]);
    k_wave_final<<<gblocks, kHostBlock, 0, st>>>(a, state->freq_cur, state->batch, state->mem_free_mib);
  }
  return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
}
