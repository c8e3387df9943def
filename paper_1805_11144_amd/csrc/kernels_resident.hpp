// The resident kernel: every step of a small model in one launch, one workgroup
// per batch column.
//
// Such a model is bound by latency: a step of one 100-neuron ensemble is seven
// merged groups of a few rows, and an interpreter that fetches each group's
// descriptor, indices and parameters from L2 (k_persistent) spends 12,000
// cycles a step on it, a hipGraph of one launch per group about 2 us a group.
// Here every neuron's state, encoder and bias are loaded into registers once a
// run (with 40 slots the form with lookups spills 8 of 256 registers, read back
// from scratch each step), all other rows, the decoders and the items of work are
// in LDS.  Each wavefront runs its own list of entries, held in its lanes, and
// fetches the next entry's items while it works on the current one.
// Every sum is taken in the order of the driver that would otherwise run the
// model, so the results are the same bits.  Measured a step: one recurrent ensemble of
// 100 neurons 2.2 us (k_persistent 4.9), 320 ensembles of 50 neurons in 14
// groups 15.8 us (launches 32).  By shader counters the first is bound by its
// serial chain: of its one wavefront's 5,160 cycles a step it issues in 51% (340
// VALU, 180 scalar, 40 LDS instructions) and waits for LDS and barriers in the
// rest.  The second is bound by VALU issue on the four SIMDs of its CU, busy 65%
// of the time; its wavefronts wait 42% of theirs.
//
// Neurons: lane r of slot s of a wavefront holds neuron r of a 64-neuron chunk of
// one ensemble; consecutive slots hold an ensemble's chunks.
#pragma once

#include "kernels.hpp"

struct ResArgs {
  const int32_t* row_of;
  const int32_t *sched, *sched_n, *items, *entries, *units, *slot_rec;
  const float *slot_par, *slot_dec, *weights;
  const int32_t* probe_at;
  int32_t nrow, nitem, nunit, nent, nprobe, waves, split, spikes, probe_barrier;
  float tau_rc, tau_ref, amp, full, inv_tau;
};

typedef int res_i4 __attribute__((ext_vector_type(4)));

// neuron_update for spiking neurons with dt <= tau_rc / 16: the same values by
// the same operations, selected instead of branched to, so that several neurons'
// updates overlap.  The partial step's exponent is at least -1/16, so expm1's
// polynomial is the branch taken.  An overshoot ratio q above 1/16 (voltages that
// a caller set above threshold, or V and J within a few ulp of 1) crosses before
// the step began: tau_rc (-ln(1 - q)), tau_rc times the polynomial (no less than
// q) and the q >= 1 case all end at `integ`, which is at most tau_rc / 16.
__device__ __forceinline__ float res_neuron(float j, float& v, float& rf, const ResArgs& A, float amp_dt, float dt) {
  const float integ = __builtin_amdgcn_fmed3f(dt - rf, 0.0f, dt);
  const float ep = expm1_small(-integ * A.inv_tau);
  const float e = rf > 0.0f ? ep : A.full;
  const float vn = v - (j - v) * e;
  float rn = __builtin_amdgcn_fmed3f(rf - dt, 0.0f, __builtin_inff());
  const float drive = j - 1.0f;
  const float q = (vn - 1.0f) * __builtin_amdgcn_rcpf(drive);
  const float since = fminf(A.tau_rc * neg_log1m_small(q), integ);
  float rs = A.tau_ref - (drive > 0.0f ? since : 0.0f);
  __asm__ volatile("" : "+v"(rn), "+v"(rs));   // computed on every lane (see lif_update_bf)
  const bool spk = vn > 1.0f;
  v = spk ? 0.0f : __builtin_amdgcn_fmed3f(vn, 0.0f, __builtin_inff());
  rf = spk ? rs : rn;
  return spk ? amp_dt : 0.0f;
}

template <int CTRL>
__device__ __forceinline__ float res_dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

// The sums over the wavefront's lanes of NB (8 or 4) registers, in wave_sum's
// order: lane l of each row of 16 returns the sum of register l % NB.  Each
// level adds a pair of registers at once, one in the lanes whose bit is clear
// and one in the others; the rows of 16 are then added in order.  About four
// instructions per sum, eleven with wave_sum.
template <int NB>
__device__ __forceinline__ float res_sums(const float (&p)[NB], int lane) {
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
  float q[NB / 2], r[NB / 4], x;
#pragma unroll
  for (int i = 0; i < NB / 2; ++i) q[i] = (b0 ? p[2 * i + 1] : p[2 * i]) + res_dpp<0xB1>(b0 ? p[2 * i] : p[2 * i + 1]);
#pragma unroll
  for (int i = 0; i < NB / 4; ++i) r[i] = (b1 ? q[2 * i + 1] : q[2 * i]) + res_dpp<0x4E>(b1 ? q[2 * i] : q[2 * i + 1]);
  // lanes l and l ^ 4: row_ror 12 reads lane l + 4, row_ror 4 lane l - 4
  const float& hi = r[NB / 4 - 1];
  // (both formed on every lane: in a branch the other lanes would read as zero)
  const float xh = hi + res_dpp<0x124>(hi), xl = r[0] + res_dpp<0x12C>(r[0]);
  x = b2 ? xh : xl;
  x += res_dpp<0x128>(x);   // lanes l and l ^ 8
  // rows of 16 in order: ((r0 + r1) + r2) + r3 in row 0
  const int xi = __builtin_bit_cast(int, x);
  const auto s = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);   // {r0, r0, r2, r2}, {r1, r1, r3, r3}
  const auto e = __builtin_amdgcn_permlane32_swap(s[0], s[0], false, false);
  const auto o = __builtin_amdgcn_permlane32_swap(s[1], s[1], false, false);
  const int s0 = s[0], s1 = s[1], e1 = e[1], o1 = o[1];
  return ((__builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1)) + __builtin_bit_cast(float, e1)) +
         __builtin_bit_cast(float, o1);
}

// The sums of eight registers over the lanes in the order of a shuffle-down sum
// (lane l + 32, then + 16, .. + 1): the sum of register i in lane 8 i.. of a row
// pair, see res_tree's use.  Registers are paired level by level as above.
__device__ __forceinline__ float res_tree8(const float (&p)[8], int lane) {
  float q[4], r[2], x;
#pragma unroll
  for (int i = 0; i < 4; ++i) {   // + 32: p[2i] in the lower half, p[2i + 1] in the upper
    const auto s = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, p[2 * i]), __builtin_bit_cast(int, p[2 * i + 1]),
                                                    false, false);
    const int a = s[0], b = s[1];
    q[i] = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {   // + 16: q[2i] in even rows, q[2i + 1] in odd rows
    const auto s = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, q[2 * i]), __builtin_bit_cast(int, q[2 * i + 1]),
                                                    false, false);
    const int a = s[0], b = s[1];
    r[i] = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
  }
  const bool b3 = lane & 8;
  x = (b3 ? r[1] : r[0]) + res_dpp<0x128>(b3 ? r[0] : r[1]);   // + 8
  x += res_dpp<0x12C>(x);                                      // + 4 (lane l + 4, lanes l % 8 < 4)
  x += res_dpp<0x12E>(x);                                      // + 2
  x += res_dpp<0x12F>(x);                                      // + 1
  return x;   // register 2 (2 b + a) + c at lane 32 c + 16 a + 8 b
}

// PLAIN: every ensemble has at most 64 neurons and stores its decoded output
// only.  Without that, a slot's place in its ensemble and its spikes' place are
// looked up.
template <int D, int ND, int S, bool PLAIN>
__global__ void __launch_bounds__(512) k_resident(float* state, int64_t rows, int32_t B, ResArgs A, int64_t n_steps,
                                                  float dt, const float* stage, int32_t feed_rows, float* probe_buf,
                                                  int64_t t0) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  constexpr int NB = S < 8 ? 4 : 8;   // slots whose decoded sums are taken together
  const int64_t col = blockIdx.x;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  float* g = state + col * rows;
  const int nslot = A.waves * S;
  float* st = lds;
  float* fbuf = st + A.nrow;                // two steps of feed rows
  float* part = fbuf + 2 * feed_rows;       // per slot: the chunk's decoded sums
  res_i4* items = (res_i4*)(lds + (A.nrow + 2 * feed_rows + nslot * ND + 3) / 4 * 4);
  res_i4* units = items + A.nitem;
  int32_t* rec = (int32_t*)(units + A.nunit);
  float* decl = (float*)(rec + 8 * nslot);
  int32_t* entries = (int32_t*)(decl + nslot * ND * 64);
  auto copy = [&](int32_t* to, const int32_t* from, int n) {
    for (int r = tid; r < n; r += nt) to[r] = G(from)[r];
  };
  for (int r = tid; r < A.nrow; r += nt) st[r] = r == 0 ? 1.0f : r == 1 ? 0.0f : g[G(A.row_of)[r]];
  copy((int32_t*)items, A.items, 4 * A.nitem);
  copy((int32_t*)units, A.units, 4 * A.nunit);
  copy(rec, A.slot_rec, 8 * nslot);
  copy((int32_t*)decl, (const int32_t*)A.slot_dec, nslot * ND * 64);
  copy(entries, A.entries, A.nent);
  const res_i4 mine = *(const __attribute__((address_space(1))) res_i4*)(G(A.sched) + 4 * (64 * wave + lane));
  const int32_t nent = __builtin_amdgcn_readfirstlane(G(A.sched_n)[wave]);
  const int32_t m0 = mine[0], m1 = mine[1], m2 = mine[2], m3 = mine[3];
  // this wavefront's neurons
  float V[S], R[S], bias[S], enc[S][D];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int64_t i = (int64_t)wave * S + s;
    gptr<float> p = G(A.slot_par) + i * (D + 1) * 64 + lane;
#pragma unroll
    for (int q = 0; q < D; ++q) enc[s][q] = p[64 * q];
    bias[s] = p[64 * D];
    gptr<int32_t> sr = G(A.slot_rec) + 8 * i;
    const bool live = lane < sr[3];
    V[s] = live ? g[sr[5] + lane] : 0.0f;
    R[s] = live ? g[sr[6] + lane] : 0.0f;
  }
  const float amp_dt = A.amp / dt;
  // feed rows are fetched two steps ahead into registers, and stored to LDS one
  // step ahead; the first step's go to LDS here
  float fr[2] = {0.0f, 0.0f};
  auto fetch = [&](int64_t k) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (k < n_steps && tid + i * nt < feed_rows) fr[i] = stage[(k * feed_rows + tid + i * nt) * B + col];
  };
  auto put = [&](int64_t k) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (tid + i * nt < feed_rows) fbuf[(k & 1) * feed_rows + tid + i * nt] = fr[i];
  };
  fetch(0);
  put(0);
  fetch(1);
  int32_t pa[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) pa[i] = tid + i * nt < A.nprobe ? G(A.probe_at)[tid + i * nt] : 0;
  __syncthreads();
  const int32_t* myrec = rec + 8 * wave * S;
  const float* mydec = decl + (int64_t)wave * S * ND * 64 + lane;
  float* mypart = part + wave * S * ND;
  // the slots' input places, uniform, and the output place and flags of slot
  // NB i + lane; with 40 slots the registers are all taken and LDS serves both
  constexpr bool kHeld = S < 40;
  int32_t xat[kHeld ? S : 1], oat[kHeld ? (S + NB - 1) / NB : 1], ofl[kHeld ? (S + NB - 1) / NB : 1];
  if constexpr (kHeld) {
#pragma unroll
    for (int s = 0; s < S; ++s) xat[s] = __builtin_amdgcn_readfirstlane(G(A.slot_rec)[8 * (wave * S + s)]);
#pragma unroll
    for (int i = 0; i < (S + NB - 1) / NB; ++i) {
      const bool in = lane < NB && NB * i + lane < S;
      oat[i] = in ? G(A.slot_rec)[8 * (wave * S + NB * i + lane) + 1] : 0;
      ofl[i] = in ? G(A.slot_rec)[8 * (wave * S + NB * i + lane) + 4] : 0;
    }
  }
  const float* feed = fbuf;   // this step's feed rows
  float* pb = probe_buf + t0 * A.nprobe * B + col;
  for (int64_t k = 0; k < n_steps; ++k) {
    feed = fbuf + (k & 1) * feed_rows;
    res_i4 item = items[__builtin_amdgcn_readlane(m1, 0) + lane];
    for (int pos = 0; pos < nent; ++pos) {
      const int32_t word = __builtin_amdgcn_readlane(m0, pos), a = __builtin_amdgcn_readlane(m2, pos);
      const int32_t b = __builtin_amdgcn_readlane(m3, pos), type = word & 15;
      const res_i4 cur = item;
      item = items[__builtin_amdgcn_readlane(m1, pos + 1) + lane];   // entries past the last are empty
      const int32_t i0 = cur[0], i1 = cur[1], i2 = cur[2], i3 = cur[3];
      const float f2 = __builtin_bit_cast(float, i2), f3 = __builtin_bit_cast(float, i3);
      // Neurons.  Outside the branches on the type below, where the compiler would
      // keep a second copy of every V and R and move them over at each entry.
      const int lo = type == ms::RES_ENS ? a : 0, hi = type == ms::RES_ENS ? b : 0;
      float acc[ND];
#pragma unroll
      for (int q = 0; q < ND; ++q) acc[q] = 0.0f;
#pragma unroll
      for (int s0 = 0; s0 < S; s0 += NB) {
        if (s0 >= hi || s0 + NB <= lo) continue;
        float x[NB][D], p[ND][NB];
        int32_t xr[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) xr[u] = kHeld ? xat[kHeld ? s0 + u : 0] : myrec[8 * (s0 + u)];
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
          for (int q = 0; q < D; ++q)
            x[u][q] = D == 1 || q == 0 ? st[xr[u]] : ((myrec[8 * (s0 + u) + 4] >> 8) & 15) > q ? st[xr[u] + q] : 0.0f;
        float sp[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          const int s = s0 + u;
          float j = bias[s];
#pragma unroll
          for (int q = 0; q < D; ++q) j += enc[s][q] * x[u][q];
          float v = V[s], rf = R[s];
          sp[u] = res_neuron(j, v, rf, A, amp_dt, dt);
          const bool in = s >= lo && s < hi;   // slots of other ensemble groups keep their state
          V[s] = in ? v : V[s];
          R[s] = in ? rf : R[s];
          const bool fresh = PLAIN || A.split || (myrec[8 * s + 4] & 1);
#pragma unroll
          for (int q = 0; q < ND; ++q) {
            const float d = mydec[(s * ND + q) * 64];
            acc[q] = fresh ? d * sp[u] : fmaf(d, sp[u], acc[q]);
            p[q][u] = acc[q];
          }
        }
        if (!PLAIN && A.spikes) {
#pragma unroll
          for (int u = 0; u < NB; ++u) {
            const int s = s0 + u, sr = myrec[8 * s + 2];
            if (s >= lo && s < hi && sr >= 0 && lane < myrec[8 * s + 3]) st[sr + lane] = sp[u];
          }
        }
        // lane l < NB: slot s0 + l
#pragma unroll
        for (int q = 0; q < ND; ++q) {
          float t = res_sums<NB>(p[q], lane);
          const int s = s0 + lane;
          if (lane < NB && s >= lo && s < hi) {
            const int32_t fl = kHeld ? ofl[kHeld ? s0 / NB : 0] : myrec[8 * s + 4];
            const int32_t at = kHeld ? oat[kHeld ? s0 / NB : 0] : myrec[8 * s + 1];
            if (!PLAIN && A.split) {   // a sum per chunk; the last chunk adds them in order
              mypart[s * ND + q] = t;
              // other lanes read it: the fence keeps the order of store and loads,
              // which are at different addresses for every single lane
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
              const int32_t c = fl >> 12;
              if (c > 0 && (fl & 2)) {
                t = mypart[(s - c) * ND + q];
                for (int i = 1; i <= c; ++i) t += mypart[(s - c + i) * ND + q];
              }
            }
            if ((PLAIN || (fl & 2)) && q < (ND == 1 ? 1 : (fl >> 2) & 63)) st[at + q] = t;
          }
        }
      }
      if (type == ms::RES_SIMPLE) {
        if (lane < a) {
          float* d = st + i0;
          const float x = ((i1 & ms::kResFeed) ? feed : st)[i1 & 0xffff], old = *d;
          const bool lp = i1 & ms::kResLowpass;
          *d = fmaf(f2, lp ? old : x, lp ? f3 * x : (i1 & ms::kResInit) ? f3 : old);
        }
      } else if (type == ms::RES_SUM4) {
        if (lane < a) {
          const float s0 = st[i1 & 0xffff], s1 = st[(uint32_t)i1 >> 16], s2 = st[i2 & 0xffff], s3 = st[(uint32_t)i2 >> 16];
          st[i0] = (((0.0f + s0) + s1) + s2) + s3;
        }
      } else if (type == ms::RES_TREE) {
        // units a .. a + b - 1: up to 8 rows of a product each, rows of W across
        // the lanes (K <= 128, zero past it and past the rows); the next unit's
        // record and weights are fetched while this one's sums are formed
        res_i4 u = units[a];
        float w0[8], w1[8];
        auto load = [&](float (&w)[8], int32_t off) {
          gptr<float> p = G(A.weights) + off + lane;
#pragma unroll
          for (int i = 0; i < 8; ++i) w[i] = p[128 * i];
        };
        load(w0, __builtin_amdgcn_readfirstlane(u[3]));
        load(w1, __builtin_amdgcn_readfirstlane(u[3]) + 64);
        for (int c = 0; c < b; ++c) {
          const res_i4 un = units[c + 1 < b ? a + c + 1 : a];
          const int32_t next = __builtin_amdgcn_readfirstlane(un[3]), d0 = u[0], K = u[2], n = (d0 >> 20) & 15;
          const float* x = st + u[1];
          const float x0 = x[lane];   // K >= 64
          const float x1 = lane + 64 < K ? x[lane + 64] : 0.0f;
          float p[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) p[i] = w0[i] * x0;
          load(w0, next);
#pragma unroll
          for (int i = 0; i < 8; ++i) p[i] = lane + 64 < K ? fmaf(w1[i], x1, p[i]) : p[i];
          load(w1, next + 64);
          const float t = res_tree8(p, lane);
          const int i = 2 * (2 * ((lane >> 3) & 1) + ((lane >> 4) & 1)) + (lane >> 5);
          if (lane % 8 == 0 && i < n) {
            float* d = st + (d0 & 0xfffff) + i;
            *d = ((d0 >> 28) & 1 ? 0.0f : *d) + t;
          }
          u = un;
        }
      } else if (type == ms::RES_INC) {
        if (lane < a) {
          float acc = i2 & ms::kResInit ? f3 : st[i0];
#pragma unroll 1
          for (int32_t e = i1; e < i1 + (i2 & 0xffffff); ++e) {
            const int32_t s = entries[2 * e];
            acc = fmaf(__builtin_bit_cast(float, entries[2 * e + 1]), ((s & ms::kResFeed) ? feed : st)[s & 0xffff], acc);
          }
          st[i0] = acc;
        }
      } else if (type == ms::RES_DOT) {
        const int32_t M = b & 0xffffff, parts = b >> 24, n = lane < a ? i2 : 0;
        gptr<float> w = G(A.weights) + i3;
        const float* x = st + i1;
        float s = 0.0f;
#pragma unroll 1
        for (int32_t q0 = 0; q0 < n; q0 += 8) {   // eight loads in flight
          float wv[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) wv[i] = w[(int64_t)min(q0 + i, n - 1) * M];
#pragma unroll
          for (int i = 0; i < 8; ++i) s = q0 + i < n ? fmaf(wv[i], x[q0 + i], s) : s;
        }
        float acc = s;
        if (parts > 1) {
          acc = 0.0f;
#pragma unroll 1
          for (int32_t p = 0; p < parts; ++p) acc += __shfl(s, lane + p);
        }
        if (lane < a && lane % parts == 0) {
          float* d = st + (i0 & 0xffff);
          *d = (i0 & ms::kResInit ? 0.0f : *d) + acc;
        }
      }
      if (word & ms::kResBar) {
        if (word & ms::kResPut) put(k + 1);
        __syncthreads();
      }
    }
    fetch(k + 2);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (tid + i * nt < A.nprobe) pb[(int64_t)(tid + i * nt) * B] = st[pa[i]];
    for (int32_t r = tid + 2 * nt; r < A.nprobe; r += nt) pb[(int64_t)r * B] = st[G(A.probe_at)[r]];
    pb += (int64_t)A.nprobe * B;
    if (A.probe_barrier) __syncthreads();
  }
  for (int r = tid; r < A.nrow; r += nt)
    if (r > 1) g[G(A.row_of)[r]] = st[r];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int32_t* sr = myrec + 8 * s;
    if (lane < sr[3]) {
      g[sr[5] + lane] = V[s];
      g[sr[6] + lane] = R[s];
    }
  }
}
