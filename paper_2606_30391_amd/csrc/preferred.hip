// preferred.hip -- MI355X (gfx950) kernels and C-ABI host dispatch of the preferred
// configuration of every active LLM (Festina, App. E, Eq. preferred_sm and
// Eq. preferred_frequency) and of the fleet's energy waste ratio (Sec. 3.5.1,
// Eq. energy_waste, energy_optimal, energy_waste_ratio).
//
// k_preferred: 16 lanes per LLM instance slot.  For each phase the lanes span the
//   (SM level, frequency level) cells of the model's table row (prefill: the average
//   prompt's 256-token bucket, duration TTFT; decode: the batch row, duration
//   avg_out x TBT), mask cells whose latency is not strictly below the SLO, and reduce
//   (energy, cell) to the least-energy cell, lowest cell on exact ties, carrying its
//   duration and power.  Lane 0 then forms the time-weighted SM share and the
//   energy-weighted frequency.  Power is the placement model P = P0 + k*s*f^3*u with
//   u = min(B + 1, 32) / 32.
// k_ewr_single (fleets up to 16,384 GPUs, one launch) or k_ewr_gpu + k_ewr_total: a
//   thread per GPU takes F_g = the highest preferred frequency of its instances and its
//   waste sum t (F_g^3 - F_l^3) in float64; one block (or per-block partials in the
//   workspace, then one block) adds waste and optimal energy in a fixed order, so the
//   totals are deterministic.
//
// Exactness: SLO tests compare float32 table entries with float32 SLOs; the per-phase
// energies and the averages are float32 (P = fma(k*u*f^3, s, P0), E = P * duration); the
// EWR sums are float64 from float32 inputs.
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "festina.h"

namespace {

constexpr int kRows = FESTINA_N_ROWS;
constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kEwrBlock = 256;
constexpr float kInf = __builtin_huge_valf();

struct PrefArgs {
  int32_t M, NS, NF, C;
  const float *sm_level, *freq_level, *pf, *dc;
  float p0;
  int32_t G, K;
  const int32_t *n_inst, *model, *avg_in, *avg_out, *batch;
  const float *slo_ttft, *slo_tbt, *kdyn;
  festina_preferred out;
};

struct Best {
  float e, t, p;
  int cell;
};

// One instance slot's results from its two phases' cells.
__device__ __forceinline__ void put_preferred(const PrefArgs &a, long long slot, const Best &bp, const Best &bd) {
  const bool hp = bp.cell != INT_MAX, hd = bd.cell != INT_MAX;
  const int cp = hp ? bp.cell : 0, cd = hd ? bd.cell : 0;
  const int jp = cp / a.NF, kp = cp - jp * a.NF, jd = cd / a.NF, kd = cd - jd * a.NF;
  const festina_preferred &o = a.out;
  o.sm_p[slot] = hp ? jp : -1;
  o.f_p[slot] = hp ? kp : -1;
  o.sm_d[slot] = hd ? jd : -1;
  o.f_d[slot] = hd ? kd : -1;
  o.t_p_ms[slot] = hp ? bp.t : 0.f;
  o.p_p_w[slot] = hp ? bp.p : 0.f;
  o.t_d_ms[slot] = hd ? bd.t : 0.f;
  o.p_d_w[slot] = hd ? bd.p : 0.f;
  o.t_ms[slot] = (hp ? bp.t : 0.f) + (hd ? bd.t : 0.f);
  o.feasible[slot] = (hp && hd) ? 1 : 0;
  float smp = __builtin_nanf(""), fpr = __builtin_nanf("");
  if (hp && hd) {
    const float sp = a.sm_level[jp], sd = a.sm_level[jd];
    const float fp = a.freq_level[kp], fd = a.freq_level[kd];
    smp = fmaf(sp, bp.t, sd * bd.t) / (bp.t + bd.t);
    const float ep = bp.p * bp.t, ed = bd.p * bd.t;
    fpr = fmaf(ep, fp, ed * fd) / fmaf(bd.p, bd.t, ep);
  }
  o.sm_pref[slot] = smp;
  o.f_pref[slot] = fpr;
}

// 16 lanes per instance slot (a row of 16 lanes is one slot, so the reductions are DPP moves):
// lane l holds the cells 16 q + l of both phases, CPL per phase, and all table entries of a slot
// are loaded together.  Bound by its three dependent loads (slot, table rows, chosen cells).
// 2,048 GPUs x 4 slots of 8 x 16 tables: 6.1 us; a wavefront per slot spent some 380 VALU
// instructions on each, most of them in the 64-lane reductions of four values, and took 9.9.
constexpr int kSlotLanes = 16;

// The candidate at DPP source lane CTRL against this lane's: the lesser energy, then the lower cell.
template <int CTRL>
__device__ __forceinline__ void best_dpp(float &e, int &c) {
  const float oe = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(e), CTRL, 0xf, 0xf, false));
  const int oc = __builtin_amdgcn_update_dpp(0, c, CTRL, 0xf, 0xf, false);
  const bool t = oe < e || (oe == e && oc < c);
  e = t ? oe : e;
  c = t ? oc : c;
}

// The least-energy feasible cell of one phase over the slot's 16 lanes (lowest cell on ties), in
// every lane; lat[q]: this lane's latency at cell 16 q + l.
template <int CPL>
__device__ __forceinline__ Best slot_best(const PrefArgs &a, const float (&lat)[CPL], const float (&sj)[CPL],
                                          const float (&f3)[CPL], int l, float slo, float dur_scale, float ku) {
  float e = kInf;
  int c = INT_MAX;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const float P = fmaf(ku * f3[q], sj[q], a.p0);
    const float x = P * (dur_scale * lat[q]);
    const bool in = lat[q] < slo && x < e;       // cells ascend with q: the first least one
    e = in ? x : e;
    c = in ? q * kSlotLanes + l : c;
  }
  best_dpp<0x128>(e, c);                         // row_ror:8
  best_dpp<0x141>(e, c);                         // row_half_mirror
  best_dpp<0x4E>(e, c);                          // quad_perm [2,3,0,1]
  best_dpp<0xB1>(e, c);                          // quad_perm [1,0,3,2]
  return Best{e, 0.f, 0.f, c};
}

template <int CPL>
__global__ void __launch_bounds__(kWavesPerBlock * kWave) k_preferred(PrefArgs a) {
  constexpr int kPerBlock = kWavesPerBlock * kWave / kSlotLanes;
  const int l = threadIdx.x & (kSlotLanes - 1);
  const long long n_slots = (long long)a.G * a.K;
  const long long slot0 = (long long)blockIdx.x * kPerBlock + (threadIdx.x / kSlotLanes);
  const long long slot = slot0 < n_slots ? slot0 : n_slots - 1;
  const int g = (int)(slot / a.K), i = (int)(slot - (long long)g * a.K);
  const int n = a.n_inst[g];
  const int m = a.model[slot];
  const int B = a.batch[slot];
  const int tin = a.avg_in[slot], tout = a.avg_out[slot];
  const float st = a.slo_ttft[slot], sb = a.slo_tbt[slot], kd = a.kdyn[g];
  float sj[CPL], f3[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int c = q * kSlotLanes + l, cc = c < a.C ? c : 0;
    const int j = cc / a.NF;
    const float f = a.freq_level[cc - j * a.NF];
    sj[q] = a.sm_level[j];
    f3[q] = f * f * f;
  }
  const bool ok = n >= 0 && n <= a.K && i < n && m >= 0 && m < a.M && B >= 0 && tin >= 1 && tout >= 0;
  const int bb = ok ? (B >= kRows ? kRows : B + 1) : 1;
  const int prow = ok ? min((int)(((unsigned)tin + 255u) >> 8), kRows) - 1 : 0;
  const size_t base = (size_t)(ok ? m : 0) * kRows * a.C;
  const float *rp = a.pf + base + (size_t)prow * a.C, *rd = a.dc + base + (size_t)(bb - 1) * a.C;
  float lp[CPL], ld[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const int c = q * kSlotLanes + l, cc = c < a.C ? c : 0;
    lp[q] = rp[cc];
    ld[q] = rd[cc];
  }
  __builtin_amdgcn_sched_barrier(0);             // every load of the slot is issued before the first use
#pragma unroll
  for (int q = 0; q < CPL; ++q)
    if (!ok || q * kSlotLanes + l >= a.C) lp[q] = ld[q] = kInf;   // never below an SLO
  const float ku = kd * ((float)bb * 0.03125f);
  Best bp = slot_best<CPL>(a, lp, sj, f3, l, st, 1.f, ku);
  Best bd = slot_best<CPL>(a, ld, sj, f3, l, sb, (float)tout, ku);
  if (l != 0 || slot0 >= n_slots) return;
  // the chosen cells' duration and power, with the operations of slot_best (fewer values in
  // the reduction than carrying them along)
  const auto fill = [&](Best &b, const float *row, float scale) {
    if (b.cell == INT_MAX) return;
    const int j = b.cell / a.NF;
    const float f = a.freq_level[b.cell - j * a.NF];
    b.p = fmaf(ku * (f * f * f), a.sm_level[j], a.p0);
    b.t = scale * row[b.cell];
  };
  fill(bp, rp, 1.f);
  fill(bd, rd, (float)tout);
  put_preferred(a, slot, bp, bd);
}

struct EwrArgs {
  int32_t G, K;
  const int32_t *n_inst;
  const float *f_pref, *t_ms;
  float *f_gpu;
  double *waste_gpu;
  double *totals;
  double *partial;               // [blocks][2] waste, optimal
  bool quads;                    // four slots per load: K a multiple of 4, both arrays 16-byte aligned
};

__device__ __forceinline__ double cube64(double x) { return x * x * x; }

__device__ double block_sum(double v, double *s) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  __syncthreads();
  if (lane == 0) s[wv] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += s[w];
  return t;
}

// GPU g: F_g, its waste (written) and its optimal-energy share (returned in og).  With at
// most kEwrSlots slots per GPU every slot is loaded at once (one memory round trip) and
// masked by the instance count afterwards.
constexpr int kEwrSlots = 8;

struct EwrIn {
  int n;
  float f[kEwrSlots], t[kEwrSlots];
};

__device__ __forceinline__ EwrIn ewr_load(const EwrArgs &a, int g) {
  EwrIn in;
  in.n = a.n_inst[g];
  const size_t base = (size_t)g * a.K;
  if (a.quads) {
#pragma unroll
    for (int i = 0; i < kEwrSlots; i += 4) {
      float4 f = {0.f, 0.f, 0.f, 0.f}, t = f;
      if (i < a.K) {
        f = *reinterpret_cast<const float4 *>(a.f_pref + base + i);
        t = *reinterpret_cast<const float4 *>(a.t_ms + base + i);
      }
      in.f[i] = f.x, in.f[i + 1] = f.y, in.f[i + 2] = f.z, in.f[i + 3] = f.w;
      in.t[i] = t.x, in.t[i + 1] = t.y, in.t[i + 2] = t.z, in.t[i + 3] = t.w;
    }
    return in;
  }
#pragma unroll
  for (int i = 0; i < kEwrSlots; ++i) {
    in.f[i] = i < a.K ? a.f_pref[base + i] : 0.f;
    in.t[i] = i < a.K ? a.t_ms[base + i] : 0.f;
  }
  return in;
}

// The waste of GPU g (written, with F_g) from its slots; its optimal-energy share in og.
__device__ __forceinline__ double ewr_sum(const EwrArgs &a, int g, const EwrIn &in, double &og) {
  const int nn = (in.n >= 0 && in.n <= a.K) ? in.n : 0;
  float fg = 0.f;
  double wg = 0.0;
  og = 0.0;
#pragma unroll
  for (int i = 0; i < kEwrSlots; ++i)
    if (i < nn && isfinite(in.f[i]) && isfinite(in.t[i]) && in.f[i] > fg) fg = in.f[i];
  const double fg3 = cube64((double)fg);
#pragma unroll
  for (int i = 0; i < kEwrSlots; ++i)
    if (i < nn && isfinite(in.f[i]) && isfinite(in.t[i])) {
      const double fl3 = cube64((double)in.f[i]);
      wg += (double)in.t[i] * (fg3 - fl3);
      og += (double)in.t[i] * fl3;
    }
  a.f_gpu[g] = fg;
  a.waste_gpu[g] = wg;
  return wg;
}

__device__ __forceinline__ double ewr_one_gpu(const EwrArgs &a, int g, double &og) {
  if (a.K <= kEwrSlots) return ewr_sum(a, g, ewr_load(a, g), og);
  const int n = a.n_inst[g];
  const int nn = (n >= 0 && n <= a.K) ? n : 0;
  const size_t base = (size_t)g * a.K;
  float fg = 0.f;
  double wg = 0.0;
  og = 0.0;
  for (int i = 0; i < nn; ++i) {
    const float f = a.f_pref[base + i], t = a.t_ms[base + i];
    if (isfinite(f) && isfinite(t) && f > fg) fg = f;
  }
  const double fg3 = cube64((double)fg);
  for (int i = 0; i < nn; ++i) {
    const float f = a.f_pref[base + i], t = a.t_ms[base + i];
    if (!(isfinite(f) && isfinite(t))) continue;
    const double fl3 = cube64((double)f);
    wg += (double)t * (fg3 - fl3);
    og += (double)t * fl3;
  }
  a.f_gpu[g] = fg;
  a.waste_gpu[g] = wg;
  return wg;
}

__global__ void __launch_bounds__(kEwrBlock) k_ewr_gpu(EwrArgs a) {
  __shared__ double s[kEwrBlock / kWave];
  const int g = blockIdx.x * kEwrBlock + threadIdx.x;
  double wg = 0.0, og = 0.0;
  if (g < a.G) wg = ewr_one_gpu(a, g, og);
  const double bw = block_sum(wg, s);
  const double bo = block_sum(og, s);
  if (threadIdx.x == 0) {
    a.partial[2 * blockIdx.x] = bw;
    a.partial[2 * blockIdx.x + 1] = bo;
  }
}

__global__ void __launch_bounds__(kEwrBlock) k_ewr_total(EwrArgs a, int32_t nblocks) {
  __shared__ double s[kEwrBlock / kWave];
  double w = 0.0, o = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += kEwrBlock) {
    w += a.partial[2 * b];
    o += a.partial[2 * b + 1];
  }
  const double tw = block_sum(w, s);
  const double to = block_sum(o, s);
  if (threadIdx.x == 0) {
    a.totals[0] = tw;
    a.totals[1] = to;
    a.totals[2] = tw / to;
  }
}

// Fleets of at most kEwrSingle GPUs: one block of 1024 threads does everything in one
// launch (each thread a fixed stride of GPUs, then one block reduction: deterministic).
constexpr int kEwrSingleBlock = 1024;
constexpr int kEwrSingle = 16 * kEwrSingleBlock;

__global__ void __launch_bounds__(kEwrSingleBlock) k_ewr_single(EwrArgs a) {
  __shared__ double s[2][kEwrSingleBlock / kWave];
  double w = 0.0, o = 0.0;
  if (a.K <= kEwrSlots) {
    // the slots of two GPUs in flight per thread, four slots per load where they allow it
    // (the single block is bound by its loads' latency and lines): 2,048 GPUs of 4 slots
    // 4.7 us; one GPU at a time, a load per slot and two reductions took 8.2
    for (int g0 = threadIdx.x; g0 < a.G; g0 += 2 * kEwrSingleBlock) {
      EwrIn in[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) in[u] = ewr_load(a, min(g0 + u * kEwrSingleBlock, a.G - 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int g = g0 + u * kEwrSingleBlock;
        if (g < a.G) {
          double og;
          w += ewr_sum(a, g, in[u], og);
          o += og;
        }
      }
    }
  } else {
    for (int g = threadIdx.x; g < a.G; g += kEwrSingleBlock) {
      double og;
      w += ewr_one_gpu(a, g, og);
      o += og;
    }
  }
  for (int off = 32; off >= 1; off >>= 1) {
    w += __shfl_xor(w, off, kWave);
    o += __shfl_xor(o, off, kWave);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    s[0][wv] = w;
    s[1][wv] = o;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double tw = 0.0, to = 0.0;
    for (int i = 0; i < kEwrSingleBlock / kWave; ++i) {
      tw += s[0][i];
      to += s[1][i];
    }
    a.totals[0] = tw;
    a.totals[1] = to;
    a.totals[2] = tw / to;
  }
}

}  // namespace

extern "C" festina_status festina_preferred_configs(const festina_lut *L, const festina_llms *Q,
                                                    festina_preferred *out, void *stream) {
  if (!L || !Q || !out) return FESTINA_ERR_INVALID;
  if (L->n_models < 1 || L->n_rows != kRows || L->n_sm < 1 || L->n_freq < 1) return FESTINA_ERR_INVALID;
  if (Q->n_gpus < 0 || Q->max_inst < 1) return FESTINA_ERR_INVALID;
  const long long C = (long long)L->n_sm * L->n_freq;
  if (C > FESTINA_MAX_CELLS) return FESTINA_ERR_UNSUPPORTED;
  if (!L->sm_level || !L->freq_level || !L->pf || !L->dc) return FESTINA_ERR_INVALID;
  if (Q->n_gpus == 0) return FESTINA_OK;
  if (!Q->n_inst || !Q->model || !Q->avg_in_tokens || !Q->avg_out_tokens || !Q->batch || !Q->slo_ttft_ms ||
      !Q->slo_tbt_ms || !Q->k_dyn_w)
    return FESTINA_ERR_INVALID;
  if (!out->sm_p || !out->f_p || !out->sm_d || !out->f_d || !out->t_p_ms || !out->t_d_ms || !out->p_p_w ||
      !out->p_d_w || !out->t_ms || !out->sm_pref || !out->f_pref || !out->feasible)
    return FESTINA_ERR_INVALID;
  const long long slots = (long long)Q->n_gpus * Q->max_inst;
  if ((slots + kWavesPerBlock - 1) / kWavesPerBlock > INT_MAX) return FESTINA_ERR_INVALID;
  const long long per = kWavesPerBlock * kWave / kSlotLanes, blocks = (slots + per - 1) / per;
  PrefArgs a;
  a.M = L->n_models;
  a.NS = L->n_sm;
  a.NF = L->n_freq;
  a.C = (int32_t)C;
  a.sm_level = L->sm_level;
  a.freq_level = L->freq_level;
  a.pf = L->pf;
  a.dc = L->dc;
  a.p0 = L->p0_w;
  a.G = Q->n_gpus;
  a.K = Q->max_inst;
  a.n_inst = Q->n_inst;
  a.model = Q->model;
  a.avg_in = Q->avg_in_tokens;
  a.avg_out = Q->avg_out_tokens;
  a.batch = Q->batch;
  a.slo_ttft = Q->slo_ttft_ms;
  a.slo_tbt = Q->slo_tbt_ms;
  a.kdyn = Q->k_dyn_w;
  a.out = *out;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const dim3 grid((unsigned)blocks), block(kWavesPerBlock * kWave);
  if (C <= 4 * kSlotLanes)
    k_preferred<4><<<grid, block, 0, st>>>(a);
  else if (C <= 8 * kSlotLanes)
    k_preferred<8><<<grid, block, 0, st>>>(a);
  else
    k_preferred<FESTINA_MAX_CELLS / kSlotLanes><<<grid, block, 0, st>>>(a);
  return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
}

extern "C" size_t festina_ewr_workspace_bytes(int32_t n_gpus) {
  if (n_gpus < 1) return 0;
  const size_t blocks = ((size_t)n_gpus + kEwrBlock - 1) / kEwrBlock;
  return (blocks * 2 * sizeof(double) + 255) & ~(size_t)255;
}

extern "C" festina_status festina_fleet_ewr(int32_t n_gpus, int32_t max_inst, const int32_t *n_inst,
                                            const float *f_pref, const float *t_ms, festina_ewr *out,
                                            void *workspace, size_t workspace_bytes, void *stream) {
  if (n_gpus < 1 || max_inst < 1 || !n_inst || !f_pref || !t_ms || !out) return FESTINA_ERR_INVALID;
  if (!out->f_gpu || !out->waste_gpu || !out->totals) return FESTINA_ERR_INVALID;
  const size_t need = festina_ewr_workspace_bytes(n_gpus);
  if (!workspace || workspace_bytes < need || (((uintptr_t)workspace) & 255) != 0) return FESTINA_ERR_INVALID;
  EwrArgs a;
  a.G = n_gpus;
  a.K = max_inst;
  a.n_inst = n_inst;
  a.f_pref = f_pref;
  a.t_ms = t_ms;
  a.f_gpu = out->f_gpu;
  a.waste_gpu = out->waste_gpu;
  a.totals = out->totals;
  a.partial = static_cast<double *>(workspace);
  a.quads = max_inst % 4 == 0 && (((uintptr_t)f_pref | (uintptr_t)t_ms) & 15) == 0;
  const int blocks = (int)(((long long)n_gpus + kEwrBlock - 1) / kEwrBlock);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (n_gpus <= kEwrSingle) {
    k_ewr_single<<<1, kEwrSingleBlock, 0, st>>>(a);
    return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
  }
  k_ewr_gpu<<<blocks, kEwrBlock, 0, st>>>(a);
  if (hipGetLastError() != hipSuccess) return FESTINA_ERR_DEVICE;
  k_ewr_total<<<1, kEwrBlock, 0, st>>>(a, blocks);
  return hipGetLastError() == hipSuccess ? FESTINA_OK : FESTINA_ERR_DEVICE;
}
