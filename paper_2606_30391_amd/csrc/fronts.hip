// fronts.hip -- MI355X (gfx950) kernels of the placement search over candidate fronts
// (Festina, Sec. 3.3, Phases One and Two), for tables of 8 SM x 16 frequency levels.
//
// For one (arrival wave, model) and one prefill cell (SM level jp, frequency level k) every
// candidate (GPU, decode SM level jd) is a line in the request's term x = TTFT / Lout:
//   key = Pp * x + Y,  Pp = P0 + k_g u_g s_jp f_k^3,  Y = (P0 + k_g u_g s_jd f_k^3) * TBT,
// key = energy / Lout (Eq. energy).  With x >= 0 a candidate whose Pp, Y and TBT are all at
// least another's can never be chosen over it, whatever the request's prompt, output length
// and SLOs.  Lightly loaded GPUs dominate loaded ones in almost every cell, so the candidates
// left (the cell's front) average 1.1 per cell where 40 to 80 GPUs host the model: a request
// scores about 140 candidates instead of 5,000 to 6,300.
//
//   k_models   per model: its hosting GPUs in chunks of kChunkHosts, each chunk grouped by
//              SM-cap class; for each pair of batch rows whether the decode latencies of one
//              are nowhere above the other's; flags of unusual table values
//   k_fronts   per (wave, model): drops hosts dominated by one host of their class on every
//              cell, then builds each cell's front from the others
//   k_choose   a workgroup takes a run of consecutive requests, groups them by (wave, model)
//              in LDS, and each wavefront scores 16 requests of one group against its front:
//              lanes are cells, the argmin with the lowest-index tie-break is fused
//
// Measured per call against the kernels of festina.hip, which score every candidate: 262,144 requests
// in 64 waves on 1,024 capped GPUs 142 -> 50 us, 65,536 on 512 GPUs 43.9 -> 25, 20,011 in 64 waves on
// 333 capped GPUs 47.7 -> 35.6.  Those are bound by VALU issue, 1.5 instructions a candidate.  Of
// these, k_models and k_fronts (5 and 18 us of the 50) are chains of memory round trips, k_fronts'
// VALU issue taking 31% of its time; k_choose (27 us) issues VALU instructions 60% of its time, the
// rest being its sort and the loads that one workgroup per CU does not hide.
//
// Exactness: keys are evaluated with the same float32 operations for every candidate, so the
// least key over the fronts is the least over all candidates: rounding is monotone, and a
// dropped candidate's key is never below its dominator's.  Equal keys go to the lowest index:
// a candidate is dropped in favour of a higher-indexed one only where its key is strictly
// larger after rounding (margins in both Pp and Y).  Requests without a prompt, with a padded
// output outside [1, 2^40], or whose prompt row holds negative or tiny entries, and buckets whose
// front does not fit, are scored against every hosting GPU instead (choose_all).  A negative decode
// latency only keeps its hosts from the comparison of whole hosts (it turns the order of their Y).
#include "fronts.h"

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <type_traits>

namespace {

constexpr int kRows = FESTINA_N_ROWS;
constexpr int kWave = 64;
constexpr int kNS = 8, kNF = 16, kCells = kNS * kNF;
constexpr int kR = 16;                           // requests scored together by one wavefront
constexpr int kChunkHosts = 128;                 // hosts pruned together by k_fronts
constexpr int kStage = 16;                       // hosts whose decode rows are staged together
constexpr int kSlots = 1024;                     // groups of a workgroup's requests
constexpr int kChooseThreads = 1024;
constexpr int kXcds = 8;                         // MI355X: 8 XCDs, each with its own L2
constexpr float kInf = __builtin_huge_valf();
// Value of a masked (SLO-missing) latency: a quiet NaN stays NaN through every multiply and
// FMA, v_min ignores it and no comparison matches it.
constexpr float kMask = __builtin_nanf("");
// A prompt latency at least this large keeps a normal value when divided by any Lout up to
// 2^40 (2^-86 * 2^-40 = 2^-126, the least normal float).
constexpr float kTinyLatency = 0x1p-86f;
// Relative gaps that make a key strictly larger after rounding: a key is one fused
// multiply-add of Pp and Y (kGapCell, of the largest key); Pp and Y are themselves within 3
// roundings of the exact terms when the GPUs' power coefficients are compared (kGapHost).
constexpr float kGapCell = 0x1p-21f;
constexpr float kGapHost = 0x1p-19f;
// Power factors s_j f_k^3 and power coefficients up to this size cannot make a power infinite.
constexpr float kMaxFactor = 0x1p60f;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

// row_max of a prefill row with a negative entry, and of one with a tiny entry
constexpr float kRowNegative = -1.f, kRowTiny = -2.f;
constexpr int kOddRows = 1 << 24;                // in a bucket's info: its model has such rows
// How k_choose decides a request: by its bucket's front, or against every hosting GPU: without a
// prompt, on energies (Lout or its prompt row do not allow keys), or on keys (negative prompt row).
enum Kind { kByFront = 0, kNoPrompt = 1, kByEnergy = 2, kByKey = 3 };

struct FrontArgs {
  int32_t M, G, W, words, R, cap, chunk, n_chunks;
  const float *sm_level, *freq_level, *pf, *dc;
  float p0;
  const int32_t *batch;
  const float *kdyn;
  const uint32_t *resident;
  const int8_t *cap_pf, *cap_dc;
  const int32_t *model, *wave, *prompt, *pred;
  const float *slo_ttft, *slo_tbt;
  int32_t *choice;
  uint8_t *feasible;
  float *energy;
  // workspace
  int32_t *host_cnt;             // [M]
  int2 *hosts;                   // [M][G] {GPU, cap_pf | cap_dc << 3 | first << 6 | end << 14}: the
                                 // host's class segment [first, end) within its chunk
  uint32_t *rowle;               // [M][32] bit b of word a: row a's decode latencies <= row b's (0: row
                                 // a holds a negative entry)
  int32_t *dc_positive;          // [M] whether every decode entry is large enough for the host-level
                                 // margin (or never feasible)
  float *row_max;                // [M][32] largest finite prefill entry of the row, or kRowNegative,
                                 // kRowTiny
  int2 *info;                    // [W * M] {nA | nB << 8 | span << 16 | kOddRows, first step}, or
                                 // {-1, }: no front
  v4f *front;                    // steps of 64 {Pp, Y, TBT, id = GPU * 8 + SM level}: `cap` per bucket,
                                 // then a pool for longer fronts; in a bucket's span the nA steps of
                                 // range A (SM levels 0-3) from the start, nB of range B from the end
  int32_t *pool_used;            // [1] steps taken from the pool
  int32_t pool_steps;
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniformf(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ float lane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ float cube(float f) { return f * f * f; }

// Read-only view in the constant address space: scalar loads where the address is uniform.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *ro(const T *p) {
  return (const __attribute__((address_space(4))) T *)(p);
}

// Prompt bucket of a token count: min(ceil(tokens / 256), 32) - 1.
__device__ __forceinline__ int prompt_row(int pt) { return min((int)(((unsigned)pt + 255u) >> 8), kRows) - 1; }

// A fresh copy of the lane id: a test made on it is made where it is used, not kept as a lane
// mask in scalar registers across a loop.
__device__ __forceinline__ int lane_fresh() {
  int l = __lane_id();
  asm volatile("" : "+v"(l));
  return l;
}

// Wave-level LDS barrier: stores by any lane of the wavefront are visible to its loads after.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sum over the wavefront's 64 lanes with DPP moves: shifts by 1, 2, 4 and 8
// lanes within each row of 16, then row broadcasts.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
  return v;
}

// ------------------------------------------------------------------ per model
constexpr int kModelBlock = 256;
constexpr int kClasses = kNS * kNS;              // (cap_pf, cap_dc) pairs
static_assert(kClasses == kWave, "one lane per class in the chunk sort");

// Adds bit b to `bits` when every lane is set in m (scalar instructions in a row: computed apart,
// the masks of all rows would be held in scalar registers at once).
__device__ __forceinline__ void add_all(unsigned long long m, uint32_t bit, uint32_t &bits) {
  uint32_t s;
  asm volatile("s_cmp_eq_u64 %2, -1\n\t"
               "s_cselect_b32 %0, %3, 0\n\t"
               "s_or_b32 %1, %1, %0"
               : "=&s"(s), "+s"(bits)
               : "s"(m), "i"(bit)
               : "scc");
}

// Whether row x of model m's decode table is nowhere above row y, for all y and the rows x of
// `part`: a wavefront compares kRowsPerWave rows with all 32 (2 cells per lane, in registers);
// entries that are never feasible (NaN, inf) count as inf.
constexpr int kRowsPerWave = 2, kRowParts = kRows / (4 * kRowsPerWave);

__device__ __forceinline__ void model_rows(const FrontArgs &a, int m, int part) {
  const int lane = threadIdx.x & (kWave - 1), wv = uniform(threadIdx.x >> 6);
  const float *p = a.dc + (size_t)m * kRows * kCells;
  float t0[kRows], t1[kRows], u0[kRowsPerWave], u1[kRowsPerWave];
  const int x0 = (part * 4 + wv) * kRowsPerWave;
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    u0[i] = p[(x0 + i) * kCells + lane];
    u1[i] = p[(x0 + i) * kCells + 64 + lane];
  }
#pragma unroll
  for (int b = 0; b < kRows; ++b) {
    t0[b] = p[b * kCells + lane];
    t1[b] = p[b * kCells + 64 + lane];
  }
  float mn = kInf;
#pragma unroll
  for (int b = 0; b < kRows; ++b) {
    t0[b] = t0[b] < kInf ? t0[b] : kInf;
    t1[b] = t1[b] < kInf ? t1[b] : kInf;
    mn = fminf(mn, fminf(t0[b], t1[b]));
  }
#pragma unroll
  for (int i = 0; i < kRowsPerWave; ++i) {
    const float v0 = u0[i] < kInf ? u0[i] : kInf, v1 = u1[i] < kInf ? u1[i] : kInf;
    uint32_t bits = 0;
#pragma unroll
    for (int b = 0; b < kRows; ++b) {
      add_all(__ballot((v0 <= t0[b]) & (v1 <= t1[b])), 1u << b, bits);
      __builtin_amdgcn_sched_barrier(0);
    }
    // a row with a negative entry takes no part in the comparison of hosts: not even itself is above it
    const bool neg = __ballot((u0[i] < 0.f) | (u1[i] < 0.f)) != 0ull;
    if (lane == 0) a.rowle[m * kRows + x0 + i] = neg ? 0u : bits;
  }
  if (x0 == 0) {
    const bool small = __ballot(mn < 0x1p-60f) != 0ull;
    if (lane == 0) a.dc_positive[m] = small ? 0 : 1;
  }
}

// Blocks [0, M): the hosting GPUs of one model.  Blocks [M, 5M): a part of its decode rows.
// Blocks [5M, 13M): four prefill rows each, one per wavefront.
__global__ void __launch_bounds__(kModelBlock) k_models(FrontArgs a) {
  const int lane = threadIdx.x & (kWave - 1), wv = uniform(threadIdx.x >> 6);
  if ((int)blockIdx.x >= (1 + kRowParts) * a.M) {
    const int row = (blockIdx.x - (1 + kRowParts) * a.M) * 4 + wv;
    const float *p = a.pf + (size_t)row * kCells;
    const float v0 = p[lane], v1 = p[64 + lane];
    const float a0 = fabsf(v0), a1 = fabsf(v1);
    const bool neg = __ballot(v0 < 0.f || v1 < 0.f) != 0ull;
    const bool tiny = __ballot((a0 > 0.f && a0 < kTinyLatency) || (a1 > 0.f && a1 < kTinyLatency)) != 0ull;
    float mx = fmaxf(v0 < kInf ? v0 : 0.f, v1 < kInf ? v1 : 0.f);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
    if (lane == 0) a.row_max[row] = tiny ? kRowTiny : (neg ? kRowNegative : mx);
    return;
  }
  if ((int)blockIdx.x >= a.M) {
    model_rows(a, (blockIdx.x - a.M) / kRowParts, (blockIdx.x - a.M) % kRowParts);
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *a.pool_used = 0;
  // hosting GPUs with SM caps inside the table, 4 per thread and round, all loads of a round
  // together; a full chunk (or the last one) is grouped by class and written out
  const int m = blockIdx.x;
  __shared__ int wsum[4][4], s_cls[kClasses], s_end[kClasses];
  int2 *list = a.hosts + (size_t)m * a.G;
  int n = 0;
  for (int G0 = 0; G0 < a.G; G0 += 4 * kModelBlock) {
    bool has[4];
    int caps[4], before[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int g = G0 + u * kModelBlock + threadIdx.x, gc = min(g, a.G - 1);
      const uint32_t word = a.resident[(size_t)gc * a.words + (m >> 5)];
      const int cp = a.cap_pf ? (int)a.cap_pf[gc] : kNS - 1, cd = a.cap_dc ? (int)a.cap_dc[gc] : kNS - 1;
      has[u] = g < a.G && ((word >> (m & 31)) & 1u) && cp >= 0 && cp < kNS && cd >= 0 && cd < kNS;
      caps[u] = cp | (cd << 3);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned long long bal = __ballot(has[u]);
      before[u] = __popcll(bal & ((1ull << lane) - 1ull));
      if (lane == 0) wsum[u][wv] = __popcll(bal);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      int mine = n;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int s = wsum[u][i];
        mine += i < wv ? s : 0;
        n += s;
      }
      if (has[u]) list[mine + before[u]] = make_int2(G0 + u * kModelBlock + threadIdx.x, caps[u]);
    }
    __syncthreads();                              // wsum is rewritten; the list is written
  }
  if (threadIdx.x == 0) a.host_cnt[m] = n;
  for (int c0 = 0; c0 < n; c0 += kChunkHosts) {
    const int nc = min(kChunkHosts, n - c0), t = threadIdx.x;
    if (t < kClasses) s_cls[t] = 0;
    __syncthreads();
    int2 h = make_int2(0, 0);
    int rank = 0;
    if (t < nc) {
      h = list[c0 + t];
      rank = atomicAdd(&s_cls[h.y], 1);
    }
    __syncthreads();
    if (t < kWave) {
      const int c = s_cls[t], inc = wave_scan(c);
      s_cls[t] = inc - c;
      s_end[t] = inc;
    }
    __syncthreads();
    if (t < nc) {
      const int lo = s_cls[h.y], hi = s_end[h.y];
      list[c0 + lo + rank] = make_int2(h.x, h.y | (lo << 6) | (hi << 14));
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ per (wave, model)
constexpr int kNegativeHost = 64;                // beside a host's caps: its powers or latencies may be
                                                 // negative
constexpr int kFrontBlock = 128;                 // one wavefront per range of SM levels
static_assert(kFrontBlock == kChunkHosts && kFrontBlock == kCells, "one thread per chunk host and per cell");

struct Line {
  float y, t;
  int id;
};

// Whether candidate (y, t, id) can be dropped for h, whose Pp is no larger: h's key is at most the
// candidate's for every request, and h has the lower index or the strictly smaller key (Y
// below `strict`, see k_fronts).
__device__ __forceinline__ bool dominates(const Line &h, float y, float t, int id, float strict) {
  return (h.y <= y) & (h.t <= t) & ((h.id < id) | (h.y < strict));
}

__global__ void __launch_bounds__(kFrontBlock) k_fronts(FrontArgs a) {
  __shared__ v4i s_h[kChunkHosts];               // {kappa, GPU, row, rowle word} of the chunk's hosts
  __shared__ v4i s_s[kChunkHosts];               // undominated hosts {kappa, GPU, row, caps | kNegativeHost}, then
  __shared__ v4i s_o[kChunkHosts];               // by ascending kappa
  __shared__ float s_row[kStage][kCells];        // their decode rows
  __shared__ float s_pd[kCells];                 // s_j * f_k^3
  __shared__ uint32_t s_rl[kRows];
  __shared__ float s_pmin[2];
  __shared__ int s_bad[2], s_n[2], s_cnt[2], s_long;
  const int bucket = blockIdx.x;
  const int w = bucket / a.M, m = bucket - w * a.M;
  const int t = threadIdx.x, lane = t & (kWave - 1), r = uniform(t >> 6);
  const int n = ro(a.host_cnt)[m];
  const int positive = ro(a.dc_positive)[m];
  const float p0 = a.p0;
  const float pd = a.sm_level[t >> 4] * cube(a.freq_level[t & 15]);
  if (t < kRows) s_rl[t] = a.rowle[m * kRows + t];
  s_pd[t] = pd;
  if (t == 0) s_long = 0;
  {
    float mn = pd;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mn = fminf(mn, __shfl_xor(mn, off, kWave));
    const bool odd = __ballot(!(pd >= 0.f && pd <= kMaxFactor)) != 0ull;
    if (lane == 0) {
      s_pmin[r] = mn;
      s_bad[r] = odd;
    }
  }
  __syncthreads();
  const float pmin = fminf(s_pmin[0], s_pmin[1]);
  bool bad = s_bad[0] || s_bad[1] || !(p0 >= 0.f && p0 < kInf);
  const bool margin = p0 >= 0x1p-20f && positive != 0;
  // the largest request term of the rows that the front serves (1 / Lout <= 1)
  float xmax = a.row_max[m * kRows + (lane & (kRows - 1))];
  const bool odd_rows = __ballot(xmax < 0.f) != 0ull;
  xmax = fmaxf(xmax, 0.f);
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) xmax = fmaxf(xmax, __shfl_xor(xmax, off, kWave));

  v4f *front = a.front + (size_t)bucket * a.cap * kWave;
  int first = bucket * a.cap, span = a.cap;
  const int jp = r * 4 + (lane >> 4), k = lane & 15;
  const float pdp = s_pd[jp * 16 + k];
  const v4f none = v4f{kMask, kMask, kMask, __int_as_float(INT_MAX)};
  int total = 0, mx = 0;
  for (;;) {                                     // once; again for a front longer than cap
  // the undropped candidates of least TBT and of least Y so far, and the largest Pp among them
  Line h1{kInf, kInf, INT_MAX}, h2 = h1;
  float hp = 0.f;
  int cnt = 0;
  // one candidate of this lane's cell (where `on`), of Pp at least hp, read at byte offset at
  // of its host's decode row; kp is the host's kappa
  const auto consider = [&](bool on, float kp, float Pp, const float *row, unsigned at, int id, float xm) {
    const float tb = row[at], y = fmaf(kp, s_pd[at], p0) * tb;
    // a Y this far below y leaves a strictly smaller key after the one rounding of the FMA,
    // whatever the request: keys are at most Pp * xmax + Y.  (An infinite or NaN TBT makes Y
    // infinite or NaN.  xm is xmax, or NaN where the host's powers or latencies may be negative:
    // so is strict then, and nothing compares below it.)
    const float strict = fmaf(-kGapCell, fmaf(Pp, xm, y), y);
    if (on & (y < kInf) & !dominates(h1, y, tb, id, strict) & !dominates(h2, y, tb, id, strict)) {
      if (cnt < span) front[(unsigned)((r == 0 ? cnt : span - 1 - cnt) * kWave + lane)] = v4f{Pp, y, tb, __int_as_float(id)};
      ++cnt;
      hp = Pp;
      if (tb < h1.t) h1 = Line{y, tb, id};
      if (y < h2.y) h2 = Line{y, tb, id};
    }
  };
  for (int c0 = 0; c0 < n; c0 += kChunkHosts) {
    const int nc = min(kChunkHosts, n - c0);
    // this thread's host
    float kap = kMask;
    int g = 0, row = 0, pack = 0;
    if (t < nc) {
      const int2 e = a.hosts[(size_t)m * a.G + c0 + t];
      g = e.x;
      pack = e.y;
      const int B = a.batch[(size_t)w * a.G + g];
      const float kd = a.kdyn[g];
      const int bb = min(B, kRows - 1) + 1;
      row = max(bb - 1, 0);
      kap = B >= 0 ? kd * ((float)bb * 0.03125f) : kMask;   // NaN: no candidate
    }
    bad = bad || kap < -kMaxFactor;
    const uint32_t rl = kap >= 0.f ? s_rl[row] : 0u;   // (negative powers turn the order of Y, too)
    s_h[t] = v4i{__float_as_int(kap), g, row, (int)rl};
    if (c0 > 0 && cnt > 255) s_long = 1;
    __syncthreads();
    if (c0 > 0 && s_long) {                        // too long to keep: scored against every host
      bad = true;
      break;
    }
    // dropped where one host of its class is no worse on every cell
    bool keep = kap == kap;
    if (t < nc && rl != 0u) {
      const int lo = (pack >> 6) & 0xff, hi = (pack >> 14) & 0xff;
      const float gap = kGapHost * fmaf(kap, pmin, p0);
#pragma unroll 4
      for (int i = lo; i < hi; ++i) {
        const v4i o = s_h[i];
        const float ok = __int_as_float(o.x);
        const bool le = ok <= kap && ((((uint32_t)o.w) >> row) & 1u);
        const bool strict = margin && (kap - ok) * pmin > gap;
        if (le && i != t && (o.y < g || strict)) keep = false;
      }
    }
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) s_n[r] = __popcll(bal);
    __syncthreads();
    const int ns = s_n[0] + s_n[1];
    const v4i mine = v4i{__float_as_int(kap), g, row, (pack & 63) | (rl == 0u ? kNegativeHost : 0)};
    if (keep) s_s[(r ? s_n[0] : 0) + __popcll(bal & ((1ull << lane) - 1ull))] = mine;
    __syncthreads();
    if (t < ns) {
      const v4i o = s_s[t];
      const float ok = __int_as_float(o.x);
      int rank = 0;
#pragma unroll 4
      for (int i = 0; i < ns; ++i) {
        const v4i x = s_s[i];
        const float xk = __int_as_float(x.x);
        rank += xk < ok || (xk == ok && x.y < o.y);
      }
      s_o[rank] = o;
    }
    __syncthreads();
    if (ns > 0 && fmaf(__int_as_float(s_o[0].x), pdp, p0) < hp) {   // (a later chunk only: kappa
      h1 = h2 = Line{kInf, kInf, INT_MAX};                            // ascends within a chunk)
      hp = 0.f;
    }
    for (int s0 = 0; s0 < ns; s0 += kStage) {
      const int nb = min(kStage, ns - s0);
      {
        float v[kStage];
        const int rows = s_o[min(s0 + (lane & (kStage - 1)), ns - 1)].z;
        const float *dcm = a.dc + (size_t)m * kRows * kCells;
#pragma unroll
        for (int i = 0; i < kStage; ++i)
          v[i] = dcm[__builtin_amdgcn_readlane(rows, i) * kCells + t];
#pragma unroll
        for (int i = 0; i < kStage; ++i) s_row[i][t] = v[i];
      }
      __syncthreads();
      v4i next = s_o[s0];
      for (int i = 0; i < nb; ++i) {
        const v4i o = next;
        next = s_o[min(s0 + i + 1, ns - 1)];
        const int caps = uniform(o.w), cp = caps & 7, cd = (caps >> 3) & 7;
        if (cp < r * 4) continue;                // no cell of this range
        const float xm = caps & kNegativeHost ? kMask : xmax;
        const float kp = uniformf(__int_as_float(o.x));
        const int gid = uniform(o.y) * kNS;
        const float Pp = fmaf(kp, pdp, p0);
        // the prefill-capped candidates (decode levels above cp, the highest first: lower TBT
        // first gives shorter fronts), then the GPU's own level
        if ((cp >> 2) == r)
          for (int jx = cd; jx > cp; --jx) consider((jp == cp) & (Pp < kInf), kp, Pp, s_row[i], jx * 16 + k, gid + jx, xm);
        consider((jp <= cp) & (Pp < kInf), kp, Pp, s_row[i], min(jp, cd) * 16 + k, gid + jp, xm);
      }
      __syncthreads();
    }
  }
  mx = cnt;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mx = max(mx, __shfl_xor(mx, off, kWave));
  const bool any = __ballot(bad) != 0ull;
  if (lane == 0) {
    s_cnt[r] = mx;
    s_bad[r] = any;
  }
  __syncthreads();
  total = s_cnt[0] + s_cnt[1];
  bad = s_bad[0] || s_bad[1] || total > 255;
  if (bad || total <= span) {
    for (int s = cnt; s < mx && !bad; ++s) front[(unsigned)((r == 0 ? s : span - 1 - s) * kWave + lane)] = none;
    break;
  }
  // a front longer than the bucket's steps is built again in the pool, if it has room
  if (t == 0) s_n[0] = atomicAdd(a.pool_used, total);
  __syncthreads();
  const int at = s_n[0];
  if (at > a.pool_steps - total) {
    bad = true;
    break;
  }
  first = gridDim.x * a.cap + at;
  span = total;
  front = a.front + (size_t)first * kWave;
  __syncthreads();                               // s_n is rewritten
  }
  if (t == 0) a.info[bucket] = bad ? make_int2(-1, 0) : make_int2(s_cnt[0] | (s_cnt[1] << 8) | (span << 16) | (odd_rows ? kOddRows : 0), first);
}

// ------------------------------------------------------------------ choosing
// v_min_f32 / v_min3_f32 as single instructions: a quiet-NaN operand yields the other operands,
// which is the masking rule; fminf would add a canonicalising v_max_f32 per operand.
__device__ __forceinline__ float vmin(float x, float y) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
__device__ __forceinline__ float vmin3(float x, float y, float z) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
  return r;
}
template <int CTRL>
__device__ __forceinline__ float dppf(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
constexpr int kDppRor8 = 0x128;        // row_ror:8: lane i reads lane i ^ 8 of its row
constexpr int kDppHalfMirror = 0x141;  // lane i reads lane 7 - i of its group of 8
constexpr int kDppQuad2301 = 0x4E;     // lane i reads lane i ^ 2 of its quad
constexpr int kDppQuad1032 = 0xB1;     // lane i reads lane i ^ 1 of its quad

// The least value over the wavefront's lanes of v[q], for N requests at once, returned in lane l
// for request l / (64 / N): each exchange halves the values a lane holds (permlane32, then
// permlane16, then a row rotation by 8 and, for 16 requests, the row half mirror pair up the
// requests), and the rest is reduced inside the request's lanes.
template <int N>
__device__ __forceinline__ float wave_min(const float (&v)[N]) {
  float u[N / 2], w[N / 4];
#pragma unroll
  for (int p = 0; p < N / 2; ++p) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[p]), __float_as_uint(v[p + N / 2]), false, false);
    u[p] = vmin(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
#pragma unroll
  for (int p = 0; p < N / 4; ++p) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u[p]), __float_as_uint(u[p + N / 4]), false, false);
    w[p] = vmin(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  const int lane = __lane_id();
  const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0;
  float d;
  if constexpr (N == 16) {
    float c[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) c[p] = vmin(b3 ? w[p + 2] : w[p], dppf<kDppRor8>(b3 ? w[p] : w[p + 2]));
    d = vmin(b2 ? c[1] : c[0], dppf<kDppHalfMirror>(b2 ? c[0] : c[1]));
  } else {
    static_assert(N == 8, "16 or 8 requests");
    d = vmin(b3 ? w[1] : w[0], dppf<kDppRor8>(b3 ? w[0] : w[1]));
    d = vmin(d, dppf<kDppHalfMirror>(d));
  }
  d = vmin(d, dppf<kDppQuad2301>(d));
  d = vmin(d, dppf<kDppQuad1032>(d));
  return d;
}

__device__ __forceinline__ int wave_min_int(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
  return v;
}

// A wave-uniform pointer into global memory kept in scalar registers, so that loads through it
// take a scalar base and a 32-bit lane offset.
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> scalar_ptr(gptr<T> p) {
  asm volatile("" : "+s"(p));
  return p;
}
template <typename T>
__device__ __forceinline__ gptr<T> scalar_ptr(const T *p) {
  return scalar_ptr((gptr<T>)p);
}

// A candidate's Y where its TBT meets the SLO, else NaN; opaque, since the compiler would
// otherwise mask every key instead.
__device__ __forceinline__ float masked_y(v4f c, float sb) {
  float y = c.z < sb ? c.y : kMask;
  asm volatile("" : "+v"(y));
  return y;
}

// The keys of one range's steps [e, n) at this lane's cell, into the least keys: two steps at a
// time, an odd last one by itself.  dir = -1: the steps lie before f.
template <int N>
__device__ __forceinline__ void more_keys(gptr<v4f> f, int dir, int e, int n, const float (&x)[N], float sb,
                                          float (&acc)[N]) {
  const unsigned lane = threadIdx.x & (kWave - 1);
  for (; e + 1 < n; e += 2) {
    const v4f c = scalar_ptr(f + dir * e * kWave)[lane], d = scalar_ptr(f + dir * (e + 1) * kWave)[lane];
    const float cy = masked_y(c, sb), dy = masked_y(d, sb);
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = vmin3(acc[q], fmaf(c.x, x[q], cy), fmaf(d.x, x[q], dy));
  }
  if (e < n) {
    const v4f c = scalar_ptr(f + dir * e * kWave)[lane];
    const float cy = masked_y(c, sb);
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = vmin(acc[q], fmaf(c.x, x[q], cy));
  }
}

// The first set bit of m, or -1; its set bits are added to `count` (scalar instructions in a
// row, see add_all).
__device__ __forceinline__ unsigned first_lane(unsigned long long m, int &count) {
  unsigned c, s;
  asm volatile("s_ff1_i32_b64 %0, %3\n\t"
               "s_bcnt1_i32_b64 %1, %3\n\t"
               "s_add_i32 %2, %2, %1"
               : "=&s"(c), "=&s"(s), "+s"(count)
               : "s"(m)
               : "scc");
  return c;
}

// A request as the wavefront sees it: the 64 / N lanes of request q hold its fields.
struct Req {
  int r;                         // request index
  int off;                       // offset of its prefill row, -1: no prompt
  float st, sb, rl, lout;        // SLOs, 1 / Lout (0: not decided on keys), Lout
};

__device__ __forceinline__ void put_result(const FrontArgs &a, int r, bool found, int index, float e) {
  a.choice[r] = found ? index : -1;
  a.feasible[r] = found ? 1 : 0;
  a.energy[r] = found ? e : kInf;
}

// The selected requests (of up to N; all of one bucket and TBT SLO sb) against its front.
template <int N>
__device__ __forceinline__ void choose_front(const FrontArgs &a, int2 info, bool sel, float sb, const Req &rq, v2f *Q) {
  constexpr int L = kWave / N;                   // lanes per request
  const int lane = threadIdx.x & (kWave - 1);
  const int nA = info.x & 0xff, nB = (info.x >> 8) & 0xff, last = ((info.x >> 16) & 0xff) - 1;
  const gptr<v4f> f = scalar_ptr(a.front + (size_t)info.y * kWave);
  const gptr<v4f> fB = scalar_ptr(f + last * kWave);
  const int off = sel ? rq.off : 0;              // an unselected request reads the first row
  const unsigned ul = (unsigned)lane;
  // request terms and SLOs for the lanes' broadcast reads; an unselected request is masked
  if (lane % L == 0) Q[lane / L] = v2f{sel ? rq.st : -kInf, rq.rl};
  wave_sync();
  float xA[N], xB[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const gptr<float> p = scalar_ptr(a.pf + (unsigned)__builtin_amdgcn_readlane(off, L * q));
    xA[q] = p[ul];
    xB[q] = p[64u + ul];
  }
  v4f cA = f[ul], cB = fB[ul];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const float st = Q[q].x, rl = Q[q].y;
    xA[q] = xA[q] < st ? xA[q] * rl : kMask;
    xB[q] = xB[q] < st ? xB[q] * rl : kMask;
    if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // four requests' terms at a time
  }
  // the least key of each request at this lane's two cells: the steps that both ranges have,
  // one of each at a time, then the longer range's others two at a time (a candidate whose TBT
  // misses the SLO is masked)
  float acc[N];
  const int both = min(nA, nB), nmax = max(nA, nB);
#pragma unroll
  for (int q = 0; q < N; ++q) acc[q] = kInf;
  for (int e = 0; e < both; ++e) {
    const float ay = masked_y(cA, sb), by = masked_y(cB, sb);
#pragma unroll
    for (int q = 0; q < N; ++q) acc[q] = vmin3(acc[q], fmaf(cA.x, xA[q], ay), fmaf(cB.x, xB[q], by));
    cA = scalar_ptr(f + min(e + 1, last) * kWave)[ul];
    cB = scalar_ptr(fB - min(e + 1, last) * kWave)[ul];
  }
  if (nA > both) more_keys<N>(f, 1, both, nA, xA, sb, acc);
  if (nB > both) more_keys<N>(fB, -1, both, nB, xB, sb, acc);
  __builtin_amdgcn_sched_barrier(0);
  const float Kl = wave_min<N>(acc);             // request lane / L
  const float Ks = sel && Kl < kInf && rq.lout * Kl < kInf ? Kl : kMask;   // NaN: infeasible
  // the lane that attains K*, per request (a byte each)
  unsigned lanes[N / 4] = {};
  int hits = 0;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const float K = lane_f(Ks, L * q);
    const unsigned c = first_lane(__ballot(acc[q] == K), hits);
    lanes[q >> 2] |= (c & 0xffu) << (8 * (q & 3));
    __builtin_amdgcn_sched_barrier(0);           // one request's lane mask at a time
  }
  const int ln = lane_fresh();
  unsigned word;
  if constexpr (N == 16)
    word = ln < 32 ? (ln < 16 ? lanes[0] : lanes[1]) : (ln < 48 ? lanes[2] : lanes[3]);
  else
    word = ln < 32 ? lanes[0] : lanes[1];
  const int at = (int)((word >> ((ln / L & 3) * 8)) & 0xffu);
  // the L lanes of a request walk that lane's cells for the lowest id with that key, L / 2 steps
  // of each range at a time: the lower half of the lanes range A, the upper half range B
  int best = INT_MAX;
  {
    const bool inB = (ln & (L / 2)) != 0;
    const int c = at & (kWave - 1);
    const int ne = at < kWave ? (inB ? nB : nA) : 0;
    const float v = a.pf[(unsigned)(off + (inB ? kWave : 0) + c)];
    const float x = v < rq.st ? v * rq.rl : kMask;
    for (int e0 = 0; e0 < nmax; e0 += L / 2) {
      const int e = e0 + (ln & (L / 2 - 1)), ec = max(min(e, ne - 1), 0);
      const v4f o = f[(unsigned)((inB ? last - ec : ec) * kWave + c)];
      const bool hit = e < ne && fmaf(o.x, x, o.y) == Ks && o.z < sb;
      best = hit ? min(best, __float_as_int(o.w) * kNF + (c & 15)) : best;
    }
  }
  if (L == 8) best = min(best, __builtin_amdgcn_update_dpp(0, best, kDppHalfMirror, 0xf, 0xf, false));
  best = min(best, __builtin_amdgcn_update_dpp(0, best, kDppQuad2301, 0xf, 0xf, false));
  best = min(best, __builtin_amdgcn_update_dpp(0, best, kDppQuad1032, 0xf, 0xf, false));
  // some request attains its least key in several lanes: every request's front is searched for
  // the lowest id with its key
  if (hits > __popcll(__ballot(Ks == Ks)) / L) {
    for (int q = 0; q < N; ++q) {
      const float K = lane_f(Ks, L * q);
      const float st = Q[q].x, rl = Q[q].y;
      const float *p = a.pf + (unsigned)__builtin_amdgcn_readlane(off, L * q);
      const float v0 = p[ul], v1 = p[64u + ul];
      const float x0 = v0 < st ? v0 * rl : kMask, x1 = v1 < st ? v1 * rl : kMask;
      int id = INT_MAX;
      for (int e = 0; e < nA + nB; ++e) {
        const bool ra = e < nA;
        const v4f o = f[(ra ? e : last - (e - nA)) * kWave + lane];
        if (fmaf(o.x, ra ? x0 : x1, o.y) == K && o.z < sb) id = min(id, __float_as_int(o.w) * kNF + (lane & 15));
      }
      id = wave_min_int(id);
      best = lane / L == q ? id : best;
    }
  }
  if (sel && lane % L == 0) put_result(a, rq.r, best != INT_MAX, best, rq.lout * Kl);
}

// ------------------------------------------------------------------ against every hosting GPU
// A candidate's key (kByKey: x = TTFT / Lout) or energy (kByEnergy: x = TTFT; kNoPrompt: x = Pp * TTFT,
// TTFT being the GPU's): both passes evaluate exactly these operations, and the one-launch kernel too.
template <int KIND>
__device__ __forceinline__ float all_value(float Pp, float Y, float x, float lout) {
  if constexpr (KIND == kByKey) return fmaf(Pp, x, Y);
  return fmaf(lout, Y, KIND == kNoPrompt ? x : Pp * x);
}

// Up to 64 hosts of one (wave, model), one per lane.
struct Hosts {
  int n, g, caps, row;           // row: offset of the host's batch row
  float kap;                     // a host without candidates: NaN, so that no value on it compares
};

__device__ __forceinline__ Hosts load_hosts(const FrontArgs &a, int m, int w, int c0, int n) {
  const int lane = threadIdx.x & (kWave - 1);
  Hosts o;
  o.n = min(kWave, n - c0);
  const int2 h = a.hosts[(size_t)m * a.G + c0 + min(lane, o.n - 1)];
  const int B = a.batch[(size_t)w * a.G + h.x];
  const int bb = min(B, kRows - 1) + 1;
  o.g = h.x;
  o.caps = h.y & 63;
  o.kap = B >= 0 ? a.kdyn[h.x] * ((float)bb * 0.03125f) : kMask;
  o.row = max(bb - 1, 0) * kCells;
  return o;
}

// The SLOs and Lout of a wavefront's N requests: st0, sb0 where the selected ones share theirs (one),
// else lane 64 / N * q holds those of request q (read where they are used: as scalars, all of them
// would leave k_choose short of registers).
template <int N>
struct AllSlos {
  bool one;
  float st0, sb0, st, sb, lout[N];
};

// This lane's cells under one pair of SM caps, remade where the caps change (hosts are grouped by them).
struct Cells {
  int caps = -1;
  unsigned p[2], d[2];           // cells of the prefill and of the decode latency
  float pdp[2], pdd[2];          // their power factors

  __device__ __forceinline__ void set(int c, const float *s_pd) {
    if (c == caps) return;
    caps = c;
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int j = (lane >> 4) + 4 * r;
      p[r] = min(j, c & 7) * 16 + (lane & 15);
      d[r] = min(j, c >> 3) * 16 + (lane & 15);
      pdp[r] = s_pd[p[r]];
      pdd[r] = s_pd[d[r]];
    }
  }
};

// U hosts (from i0 on) at this lane's two cells: powers, and the table entries, all requested together.
template <int U, int KIND>
struct Entries {
  int caps[U];
  float Pp[U][2], Pd[U][2], tb[U][2], tt[U][2];

  __device__ __forceinline__ void load(const Hosts &h, gptr<float> dcm, gptr<float> pfm, const float *s_pd, float p0,
                                       Cells &c, int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u, h.n - 1);
      const int row = __builtin_amdgcn_readlane(h.row, i);
      caps[u] = __builtin_amdgcn_readlane(h.caps, i);
      // (a host past the last repeats it without power: no value on it compares)
      const float kap = i0 + u < h.n ? lane_f(h.kap, i) : kMask;
      c.set(caps[u], s_pd);
      const gptr<float> d = scalar_ptr(dcm + row), p = scalar_ptr(pfm + row);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        tb[u][r] = d[c.d[r]];
        if (KIND == kNoPrompt) tt[u][r] = p[c.p[r]];
        Pp[u][r] = fmaf(kap, c.pdp[r], p0);
        Pd[u][r] = fmaf(kap, c.pdd[r], p0);
      }
    }
  }
};

// The least values over the chunk's hosts at this lane's two cells, into acc: the table entries of four
// hosts are requested together (four wavefronts per SIMD hide the trip), two hosts scored at a time.
// The prompt terms under a host's caps are fetched from their lanes where the caps change.
template <int N, int KIND>
__device__ __forceinline__ void all_hosts(const Hosts &h, gptr<float> dcm, gptr<float> pfm, const float *s_pd, float p0,
                                          const AllSlos<N> &slo, const float (&xA)[N], const float (&xB)[N],
                                          float (&acc)[N]) {
  constexpr int U = 4;
  const int lane = threadIdx.x & (kWave - 1);
  float x[2][N];
  int now = -1;
  Cells cells;
  Entries<U, KIND> e;
  // hosts [u, u + two] at cell r; those of a pair have the same caps if requests have prompts
  const auto score = [&](int u, auto two, int r) {
    constexpr int T = decltype(two)::value;
    float Y[T], X[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float tb = e.tb[u + t][r], tt = KIND == kNoPrompt ? e.tt[u + t][r] : 0.f;
      X[t] = e.Pp[u + t][r] * tt;
      Y[t] = e.Pd[u + t][r] * tb;
      if (slo.one) {
        Y[t] = tb < slo.sb0 && (KIND != kNoPrompt || tt < slo.st0) ? Y[t] : kMask;
        asm volatile("" : "+v"(Y[t]));             // (else every value would be masked, not this one)
      }
    }
    const auto value = [&](int t, int q, float y) {
      return all_value<KIND>(e.Pp[u + t][r], y, KIND == kNoPrompt ? X[t] : x[r][q], slo.lout[q]);
    };
    const auto masked = [&](int t, int q) {
      if (slo.one) return Y[t];
      constexpr int L = kWave / N;
      const bool in = e.tb[u + t][r] < lane_f(slo.sb, L * q) &&
                      (KIND != kNoPrompt || e.tt[u + t][r] < lane_f(slo.st, L * q));
      return in ? Y[t] : kMask;
    };
    if (slo.one) {
#pragma unroll
      for (int q = 0; q < N; ++q)
        acc[q] = T == 2 ? vmin3(acc[q], value(0, q, Y[0]), value(T - 1, q, Y[T - 1])) : vmin(acc[q], value(0, q, Y[0]));
    } else {
#pragma unroll
      for (int q = 0; q < N; ++q)
        acc[q] = T == 2 ? vmin3(acc[q], value(0, q, masked(0, q)), value(T - 1, q, masked(T - 1, q)))
                        : vmin(acc[q], value(0, q, masked(0, q)));
    }
  };
  const auto upper = [](int caps) { return max(caps & 7, caps >> 3) >= 4; };   // else cell 1 repeats a lower level's
  const auto terms = [&](int caps) {
    if (KIND == kNoPrompt || caps == now) return;
    now = caps;
    const int cp = caps & 7;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int from = ((min((lane >> 4) + 4 * r, cp) & 3) * 16 + (lane & 15)) << 2;
#pragma unroll
      for (int q = 0; q < N; ++q)
        x[r][q] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(r == 0 || cp < 4 ? xA[q] : xB[q])));
    }
  };
  for (int i0 = 0; i0 < h.n; i0 += U) {
    e.load(h, dcm, pfm, s_pd, p0, cells, i0);
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      if (KIND == kNoPrompt || e.caps[u] == e.caps[u + 1]) {
        terms(e.caps[u]);
        score(u, std::integral_constant<int, 2>{}, 0);
        if (upper(e.caps[u]) || upper(e.caps[u + 1])) score(u, std::integral_constant<int, 2>{}, 1);
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          terms(e.caps[u + t]);
          score(u + t, std::integral_constant<int, 1>{}, 0);
          if (upper(e.caps[u + t])) score(u + t, std::integral_constant<int, 1>{}, 1);
        }
      }
    }
  }
}

// The selected requests (of up to N; all of one bucket and kind) against every GPU hosting the model:
// for requests that the fronts do not serve.  Bound by VALU issue (69% of k_choose's time for 262,144
// requests without prompts, 10 instructions per (request, host) of 128 cells).  us per call without
// prompts, against four requests at a time and against festina.hip's kernels: 65,536 requests on 512 GPUs 136 / 398 / 159, 262,144 on
// 1,024 578 / 1,684 / 951, 16,384 on 256 69 / 349 / 85, 20,011 on 333 88 / 173 / 74 (groups of four here).
// Every request with SLOs of its own, read from its lane for each candidate: 168, 853 and (20,011) 129.
// (A variant of four requests beside this one took 98 us for the first, and 0.5% of every call that
// has none: it left the registers of k_choose's other path fewer.)
// A request is decided on keys where its bucket's front would decide it so, by its own fields only, so
// that its result does not depend on whether there is a front.  Lanes are cells (levels 0-3, then 4-7); then lanes are hosts, and each request's tied cells
// are evaluated on all of them for the lowest index.
template <int N, int KIND>
__device__ __forceinline__ void choose_all(const FrontArgs &a, int bucket, bool sel, const Req &rq, v2f *Q,
                                           const float *s_pd) {
  constexpr int L = kWave / N;                     // lanes per request
  const int lane = threadIdx.x & (kWave - 1);
  const int w = bucket / a.M, m = bucket - w * a.M;
  const int n = ro(a.host_cnt)[m];
  const float p0 = a.p0;
  const gptr<float> dcm = scalar_ptr(a.dc + (size_t)m * kRows * kCells), pfm = scalar_ptr(a.pf + (size_t)m * kRows * kCells);
  const float st = sel ? rq.st : -kInf;            // an unselected request is masked
  AllSlos<N> slo;
  {
    const int l0 = __builtin_ctzll(__ballot(sel));
    slo.st = st;
    slo.sb = rq.sb;
    slo.st0 = lane_f(st, l0);
    slo.sb0 = lane_f(rq.sb, l0);
    const bool other = __float_as_int(rq.sb) != __float_as_int(slo.sb0) ||
                       (KIND == kNoPrompt && __float_as_int(st) != __float_as_int(slo.st0));
    slo.one = __ballot(sel && other) == 0ull;
#pragma unroll
    for (int q = 0; q < N; ++q) slo.lout[q] = lane_f(rq.lout, L * q);
  }
  float xA[N], xB[N], acc[N];
#pragma unroll
  for (int q = 0; q < N; ++q) acc[q] = kInf;
  if constexpr (KIND != kNoPrompt) {
    if (lane % L == 0) Q[lane / L] = v2f{st, rq.rl};
    wave_sync();
    const int off = sel ? rq.off : 0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const gptr<float> p = scalar_ptr(a.pf + (unsigned)__builtin_amdgcn_readlane(off, L * q));
      xA[q] = p[(unsigned)lane];
      xB[q] = p[64u + (unsigned)lane];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const float sq = Q[q].x, rl = KIND == kByKey ? Q[q].y : 1.f;
      xA[q] = xA[q] < sq ? xA[q] * rl : kMask;
      xB[q] = xB[q] < sq ? xB[q] * rl : kMask;
      if ((q & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (n == 0) {
    if (sel && lane % L == 0) put_result(a, rq.r, false, -1, kInf);
    return;
  }
  const int last = (n - 1) & ~(kWave - 1);         // the last chunk of 64 hosts
  Hosts h;
  for (int c0 = 0; c0 <= last; c0 += kWave) {
    h = load_hosts(a, m, w, c0, n);
    all_hosts<N, KIND>(h, dcm, pfm, s_pd, p0, slo, xA, xB, acc);
  }
  const float Kl = wave_min<N>(acc);               // request lane / L
  const float energy = KIND == kByKey ? rq.lout * Kl : Kl;
  const float Ks = sel && Kl < kInf && energy < kInf ? Kl : kMask;   // NaN: infeasible
#pragma unroll
  for (int q = 0; q < N; ++q) {                    // the lanes that attain a request's least value
    const unsigned long long tied = __ballot(acc[q] == lane_f(Ks, L * q));
    if (lane == 0) Q[q] = v2f{__uint_as_float((unsigned)tied), __uint_as_float((unsigned)(tied >> 32))};
    __builtin_amdgcn_sched_barrier(0);
  }
  wave_sync();
  int best = INT_MAX;
  for (int c0 = last; c0 >= 0; c0 -= kWave) {      // (the last chunk's hosts are at hand)
    if (c0 != last) h = load_hosts(a, m, w, c0, n);
    const int cp = h.caps & 7, cd = h.caps >> 3;
    constexpr int U = 4;                           // requests whose table entries are requested together
#pragma unroll
    for (int q0 = 0; q0 < N; q0 += U) {
      unsigned long long tied[U];
      unsigned long long any = 0ull;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const v2f t = Q[q0 + u];
        tied[u] = ((unsigned long long)(unsigned)uniform(__float_as_int(t.y)) << 32) | (unsigned)uniform(__float_as_int(t.x));
        any |= tied[u];
      }
      while (any) {                                // once, unless a request attains its value in several lanes
        float tb[U][2], tt[U][2];
        any = 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c = tied[u] ? __builtin_ctzll(tied[u]) : 0;
          const int off = __builtin_amdgcn_readlane(rq.off, L * (q0 + u));
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int cP = min((c >> 4) + 4 * r, cp) * 16 + (c & 15), cD = min((c >> 4) + 4 * r, cd) * 16 + (c & 15);
            tb[u][r] = dcm[(unsigned)(h.row + cD)];
            tt[u][r] = KIND == kNoPrompt ? pfm[(unsigned)(h.row + cP)] : a.pf[(unsigned)(max(off, 0) + cP)];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = q0 + u, c = tied[u] ? __builtin_ctzll(tied[u]) : 0;
          const float K = tied[u] ? lane_f(Ks, L * q) : kMask, lout = lane_f(rq.lout, L * q);
          const float sq = lane_f(rq.st, L * q), sb = lane_f(rq.sb, L * q), rl = KIND == kByKey ? lane_f(rq.rl, L * q) : 1.f;
          int id = INT_MAX;
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int cell = c + kWave * r;
            const int cP = min(cell >> 4, cp) * 16 + (c & 15), cD = min(cell >> 4, cd) * 16 + (c & 15);
            const float Pp = fmaf(h.kap, s_pd[cP], p0), Y = fmaf(h.kap, s_pd[cD], p0) * tb[u][r];
            const float x = KIND == kNoPrompt ? Pp * tt[u][r] : (KIND == kByKey ? tt[u][r] * rl : tt[u][r]);
            const bool hit = lane < h.n && tt[u][r] < sq && tb[u][r] < sb && all_value<KIND>(Pp, Y, x, lout) == K;
            for (unsigned long long b = __ballot(hit); b; b &= b - 1)
              id = min(id, __builtin_amdgcn_readlane(h.g, __builtin_ctzll(b)) * kCells + cell);
          }
          best = lane / L == q ? min(best, id) : best;
          tied[u] &= tied[u] - 1;
          any |= tied[u];
        }
      }
    }
  }
  if (sel && lane % L == 0) put_result(a, rq.r, best != INT_MAX, best, energy);
}

__device__ __forceinline__ void choose_all(const FrontArgs &a, int bucket, int kind, bool sel, const Req &rq, v2f *Q,
                                           const float *s_pd) {
  if (kind == kNoPrompt)
    choose_all<8, kNoPrompt>(a, bucket, sel, rq, Q, s_pd);
  else if (kind == kByEnergy)
    choose_all<8, kByEnergy>(a, bucket, sel, rq, Q, s_pd);
  else
    choose_all<8, kByKey>(a, bucket, sel, rq, Q, s_pd);
}

// The kernel's arguments (its only parameter) read again from the kernel-argument segment where
// they are needed: a rare path's pointers do not stay in scalar registers through the others.
__device__ __forceinline__ FrontArgs fresh_args() {
  auto p = (const __attribute__((address_space(4))) FrontArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const FrontArgs *)p;
}

// Workgroup c takes requests [c * chunk, (c + 1) * chunk): consecutive chunks (requests that
// arrive together, hence share fronts) go to one XCD's L2.  The requests are grouped by a hash
// of their bucket with a counting sort in LDS; a tile is up to 16 requests of one group, and
// the requests of one tile that share a bucket are scored together.
__global__ void __launch_bounds__(kChooseThreads) k_choose(FrontArgs a) {
  __shared__ v4i s_rec[kChooseThreads];          // {row offset, TTFT SLO, TBT SLO, 1 / Lout}
  __shared__ float s_lout[kChooseThreads];
  __shared__ int s_bkt[kChooseThreads];          // bucket * 4 + kind
  __shared__ int2 s_info[kChooseThreads];        // its bucket's front
  __shared__ uint16_t s_ord[kChooseThreads];     // request of each sorted position
  __shared__ int s_cnt[kSlots];                  // requests per slot, then the slot's start
  __shared__ unsigned s_tile[kSlots];            // first position | requests << 16
  __shared__ v2f s_q[kChooseThreads / kWave][kR];
  __shared__ float s_pd[kCells];
  __shared__ int s_sum[kChooseThreads / kWave];
  __shared__ int s_next, s_again, s_rest;
  const int per = (a.n_chunks + kXcds - 1) / kXcds;
  const int ck = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  if ((int)blockIdx.x / kXcds >= per || ck >= a.n_chunks) return;
  const int t = threadIdx.x, lane = t & (kWave - 1), wv = uniform(t >> 6);
  const int first = ck * a.chunk;
  const int nreq = min(a.chunk, a.R - first);
  s_cnt[t] = 0;
  if (t < kCells) s_pd[t] = a.sm_level[t >> 4] * cube(a.freq_level[t & 15]);
  if (t == 0) s_next = s_again = s_rest = 0;
  int slot = -1, pos = 0;
  int2 info = make_int2(-1, 0);
  int m = -1, w = 0, pt = 0, pr = 0;
  float st = 0.f, sb = 0.f;
  if (t < nreq) {
    const int r = first + t;
    m = a.model[r];
    w = a.wave ? a.wave[r] : 0;
    pt = a.prompt[r];
    pr = a.pred[r];
    st = a.slo_ttft[r];
    sb = a.slo_tbt[r];
  }
  __syncthreads();
  if (t < nreq) {
    if (m >= 0 && m < a.M && w >= 0 && w < a.W && pt >= 0 && pr >= 0) {
      const int bucket = w * a.M + m;
      const int row = pt > 0 ? m * kRows + prompt_row(pt) : 0;
      const float lout = (float)(((long long)pr * 105 + 99) / 100);
      const float rl = pt > 0 && lout >= 1.f && lout <= 0x1p40f ? 1.f / lout : 0.f;
      const int kind = pt == 0 ? kNoPrompt : (rl == 0.f ? kByEnergy : kByFront);
      if (kind == kByFront) info = a.info[bucket];
      s_rec[t] = v4i{pt > 0 ? row * kCells : -1, __float_as_int(st), __float_as_int(sb), __float_as_int(rl)};
      s_lout[t] = lout;
      s_bkt[t] = bucket * 4 + kind;
      // requests of one bucket and TBT SLO share a slot, those without a front of one bucket and kind;
      // others may too
      const unsigned h = kind == kByFront ? (unsigned)__float_as_int(sb) * 0x9E3779B1u >> 29 : (unsigned)kind;
      slot = (((unsigned)bucket * 8u + h) & (kSlots / 2 - 1)) << 1 | (kind != kByFront ? 1 : 0);
      pos = atomicAdd(&s_cnt[slot], 1);
    } else {
      put_result(a, first + t, false, -1, kInf);
    }
  }
  __syncthreads();
  // starts and tiles of the slots, one slot per thread: counts in the low half, tiles in the high
  const int n = s_cnt[t];
  const int mine = n | (((n + kR - 1) / kR) << 16);
  const int inc = wave_scan(mine);
  if (lane == kWave - 1) s_sum[wv] = inc;
  __syncthreads();
  int ex = inc - mine, tiles = 0;
#pragma unroll
  for (int i = 0; i < kChooseThreads / kWave; ++i) {
    const int s = s_sum[i];
    ex += i < wv ? s : 0;
    tiles += s >> 16;
  }
  s_cnt[t] = ex & 0xffff;
  if (slot >= 0 && (info.x & kOddRows)) {         // (info is used first here: nothing waits for it before)
    if (s_rec[t].w != 0) {                         // decided on keys, unless its prompt row is an odd one
      const float top = a.row_max[m * kRows + prompt_row(pt)];
      if (top < 0.f) info.x = -1;
      if (top == kRowTiny) s_rec[t].w = 0;
      if (top < 0.f) s_bkt[t] += top == kRowTiny ? kByEnergy : kByKey;
    }
    if (info.x < 0) s_rest = 1;
  }
  s_info[t] = info;
  for (int i = 0; i * kR < n; ++i)
    s_tile[(ex >> 16) + i] = (unsigned)((ex & 0xffff) + i * kR) | ((unsigned)min(kR, n - i * kR) << 16);
  __syncthreads();
  if (slot >= 0) s_ord[s_cnt[slot] + pos] = (uint16_t)t;
  __syncthreads();
  const bool rest = uniform(s_rest) != 0;
  // Requests with a front first; the others in a second round over the tiles, so that their path (which
  // most calls never take) shares no registers with this one.
  for (;;) {
    int ti = 0;
    if (lane == 0) ti = atomicAdd(&s_next, 1);
    ti = uniform(ti);
    if (ti >= tiles) break;
    const unsigned tile = (unsigned)uniform((int)s_tile[ti]);
    const int nt = (int)(tile >> 16);
    const int q = nt > 8 ? lane >> 2 : lane >> 3;  // 4 or 8 lanes per request: tiles of up to 16 or 8
    const bool has = q < nt;
    const int i = s_ord[(tile & 0xffffu) + (has ? q : 0)];
    const v4i rec = s_rec[i];
    const Req rq{first + i, rec.x, __int_as_float(rec.y), __int_as_float(rec.z), __int_as_float(rec.w), s_lout[i]};
    const int bkt = s_bkt[i];
    const int2 in = s_info[i];
    unsigned long long todo = __ballot(has && in.x >= 0);
    while (todo) {
      const int ld = __builtin_ctzll(todo);
      const int b = __builtin_amdgcn_readlane(bkt, ld), sbi = __builtin_amdgcn_readlane(rec.z, ld);
      const bool sel = has && bkt == b && rec.z == sbi;      // as bits: a NaN SLO matches itself
      todo &= ~__ballot(sel);
      const int2 fr = make_int2(__builtin_amdgcn_readlane(in.x, ld), __builtin_amdgcn_readlane(in.y, ld));
      if (nt > 8)
        choose_front<16>(a, fr, sel, __int_as_float(sbi), rq, s_q[wv]);
      else
        choose_front<8>(a, fr, sel, __int_as_float(sbi), rq, s_q[wv]);
    }
  }
  if (!rest) return;
  for (;;) {
    int ti = 0;
    if (lane == 0) ti = atomicAdd(&s_again, 1);
    ti = uniform(ti);
    if (ti >= 2 * tiles) break;
    // half a tile: with sixteen requests, as choose_front takes, the prompt terms under a host's caps
    // would not fit the registers
    const unsigned tile = (unsigned)uniform((int)s_tile[ti >> 1]);
    const int nt = (int)(tile >> 16), q0 = (ti & 1) * 8;
    if (q0 >= nt) continue;
    const int q = q0 + (lane >> 3);
    const bool has = q < nt;
    const int i = s_ord[(tile & 0xffffu) + (has ? q : 0)];
    const v4i rec = s_rec[i];
    const Req rq{first + i, rec.x, __int_as_float(rec.y), __int_as_float(rec.z), __int_as_float(rec.w), s_lout[i]};
    const int bkt = s_bkt[i];
    unsigned long long todo = __ballot(has && s_info[i].x < 0);
    while (todo) {
      const int b = __builtin_amdgcn_readlane(bkt, __builtin_ctzll(todo));
      const bool sel = has && bkt == b;
      todo &= ~__ballot(sel);
      choose_all(fresh_args(), b >> 2, b & 3, sel, rq, s_q[wv], s_pd);
    }
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

hipError_t mark(void *ev, hipStream_t st) {
  return ev ? hipEventRecord(static_cast<hipEvent_t>(ev), st) : hipSuccess;
}

}  // namespace

namespace festina_fronts {

// Fronts are built for every (wave, model), whether or not requests ask for it.
bool sparse(long long buckets, long long R) { return buckets > 1024 + R / 4; }

bool layout(const festina_lut *L, const festina_gpus *G, const festina_requests *Q, Layout *o) {
  const long long M = L->n_models, Gn = G->n_gpus, W = G->n_waves, R = Q->n_requests;
  if (L->n_sm != kNS || L->n_freq != kNF || M > INT_MAX / (2 * kRows * kCells) || Gn > (1 << 24)) return false;
  const long long buckets = W * M;
  if (sparse(buckets, R)) return false;
  // steps per bucket: 16 (fronts of the capped, 1,024-GPU fleets take 4.6 on average and 8 at the
  // 99th percentile), up to 255 for few buckets (with many hosts some fronts are longer, and were built
  // twice: 32 models of 1,024 hosts each 112 -> 68 us, of 3,900 588 -> 344), less where the buckets
  // do not leave room beside the host lists
  const long long step = kWave * (long long)sizeof(v4f);
  const long long room = (31LL << 20) - (long long)sizeof(int2) * M * Gn - 16 * buckets - 512 * M;
  const long long fit = room / (buckets * step);
  const long long want = buckets > 1024 ? 16 : (buckets <= 64 ? 255 : 16384 / buckets);
  const int cap = (int)(fit <= want ? fit - 1 : want);   // the rest is the pool of longer fronts
  if (room <= 0 || cap < 8) return false;
  const long long left = room / step - cap * buckets;
  const long long pool = left < 4096 ? left : 4096;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align256(off + bytes);
    return at;
  };
  o->host_cnt = take(sizeof(int32_t) * M);
  o->hosts = take(sizeof(int2) * M * Gn);
  o->rowle = take(sizeof(uint32_t) * M * kRows);
  o->dc_positive = take(sizeof(int32_t) * M);
  o->row_max = take(sizeof(float) * M * kRows);
  o->info = take(sizeof(int2) * buckets);
  o->pool_used = take(sizeof(int32_t));
  o->front = take((size_t)step * (cap * buckets + pool));
  o->total = off;
  if (off > FESTINA_NOALLOC_WORKSPACE_BYTES) return false;
  o->buckets = (int32_t)buckets;
  o->cap = cap;
  o->pool_steps = (int32_t)pool;
  // (with many hosts per model, requests without a front take long: few requests go to more workgroups)
  const long long c = ((R + 255) / 256 + 63) & ~63LL, least = (M <= 4 ? Gn : 4 * Gn / M) > 384 ? 16 : 128;
  o->chunk = (int32_t)(R <= 256 * least ? least : (c > kChooseThreads ? kChooseThreads : (c < 64 ? 64 : c)));
  return true;
}

festina_status launch(const festina_lut *L, const festina_gpus *G, const festina_requests *Q,
                      const festina_placements *out, const Layout &lay, char *ws, void *stream, void *ev_begin,
                      void *ev_end) {
  FrontArgs a;
  a.M = L->n_models;
  a.G = G->n_gpus;
  a.W = G->n_waves;
  a.words = (L->n_models + 31) / 32;
  a.R = Q->n_requests;
  a.cap = lay.cap;
  a.chunk = lay.chunk;
  a.n_chunks = (int32_t)(((long long)a.R + a.chunk - 1) / a.chunk);
  a.sm_level = L->sm_level;
  a.freq_level = L->freq_level;
  a.pf = L->pf;
  a.dc = L->dc;
  a.p0 = L->p0_w;
  a.batch = G->batch;
  a.kdyn = G->k_dyn_w;
  a.resident = G->resident;
  a.cap_pf = G->cap_pf;
  a.cap_dc = G->cap_dc;
  a.model = Q->model;
  a.wave = Q->wave;
  a.prompt = Q->prompt_tokens;
  a.pred = Q->pred_out_tokens;
  a.slo_ttft = Q->slo_ttft_ms;
  a.slo_tbt = Q->slo_tbt_ms;
  a.choice = out->choice;
  a.feasible = out->feasible;
  a.energy = out->energy_mj;
  a.host_cnt = reinterpret_cast<int32_t *>(ws + lay.host_cnt);
  a.hosts = reinterpret_cast<int2 *>(ws + lay.hosts);
  a.rowle = reinterpret_cast<uint32_t *>(ws + lay.rowle);
  a.dc_positive = reinterpret_cast<int32_t *>(ws + lay.dc_positive);
  a.row_max = reinterpret_cast<float *>(ws + lay.row_max);
  a.info = reinterpret_cast<int2 *>(ws + lay.info);
  a.pool_used = reinterpret_cast<int32_t *>(ws + lay.pool_used);
  a.pool_steps = lay.pool_steps;
  a.front = reinterpret_cast<v4f *>(ws + lay.front);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (mark(ev_begin, st) != hipSuccess) return FESTINA_ERR_DEVICE;
  k_models<<<(1 + kRowParts + kRows / 4) * a.M, kModelBlock, 0, st>>>(a);
  if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  k_fronts<<<lay.buckets, kFrontBlock, 0, st>>>(a);
  if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  const int grid = (a.n_chunks + kXcds - 1) / kXcds * kXcds;
  k_choose<<<grid, kChooseThreads, 0, st>>>(a);
  if (hipGetLastError() != hipSuccess || mark(ev_end, st) != hipSuccess) return FESTINA_ERR_DEVICE;
  return FESTINA_OK;
}

}  // namespace festina_fronts
