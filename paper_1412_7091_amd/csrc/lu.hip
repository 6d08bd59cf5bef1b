// Pivoted LU factorisation and row solves for the solve-from-scratch step
// (section 3.5, last paragraph): instead of carrying U^{-T} from step to step
// through the Woodbury identity, factor A = U_new^T every step and solve
// A z_i = h_i for the m examples of the minibatch, O(d^3) + O(m d^2) work.
//
// Both halves are chains: d pivots one after another, then twice d / 16 blocks
// of unknowns, so what counts is the time of one link and not the flops.
//
// Factorisation (right-looking, partial pivoting, P A = L R), panels of 32
// columns, one launch per panel.  Rows are never interchanged: piv[k] names
// the row of A chosen at step k, act lists the rows not chosen yet (ascending),
// and every access to a row goes through one of the two.  Launch p applies
// panel p - 1 to everything on its right and factors panel p:
//   block 0        the columns of panel p: U12 by substitution, the rank-32
//                  update on MFMA into LDS, then the panel itself;
//   blocks 1 ..    32 columns each of the panels after p: U12 and the update;
//   last block     inverses of the 16 x 16 diagonal blocks of panel p - 1 for
//                  the row solves.
// Factoring a panel is a chain of 32 links.  Up to 512 active rows four waves
// take eight columns each, all rows in the registers of each (WavePanel): a
// link is then one wave's arg-max by DPP, its row by v_readlane and the rank-1
// update, without a barrier, and the waves on its right catch up meanwhile.
// Above, a row per thread on all waves (panel_links), because eight columns of
// 1024 rows do not fit a wave's registers: a link is the largest |a| per wave,
// its row published in LDS, one barrier, the wave holding the largest found by
// every wave for itself, the row read back, the update.  In both the column in
// hand is always register 0 (the update shifts the row by one register), so a
// link is one loop body.
//
// Row solves, P A = L R: A z = h is z = R^{-1} L^{-1} P h.  A workgroup solves
// for 16 examples; its waves hold the right-hand sides as MFMA accumulators
// (16 unknowns x 16 examples a block) and go through the blocks once forward
// and once back.  A link: the owner multiplies its block by the inverse of the
// diagonal block (an accumulator has the layout of an MFMA's B operand, so no
// data moves between lanes), publishes it in LDS, one barrier, and every wave
// subtracts the block's part from the blocks it owns, the factor's fragments
// loaded several links ahead.
//
// At d = 500, m = 128: 440 us for the factorisation and 47 us for the solves
// (1.4 ms when a link was three barriers and ten shuffles and the interchanges
// and the update were launches of their own; 0.5 ms for the solves with a
// launch per 64 unknowns on m / 16 workgroups).  The 16 panel launches take 34
// us (468 rows; the first, whose columns are cold, 42) down to 17 (52 rows and
// the last): the update's loads, substitution and products 8 to 4 us, the links
// 20 to 11 us, which is 0.63 us each at 468 rows (7 columns of 8 rows per lane to
// update, in one wave) and 0.33 at 52, the write-back 4 to 1 us, about 1.5 us
// outside the kernel's body.  The last launch has 20 links (7 us) and the
// inverses of its own diagonal blocks (6 us), which the others leave to the next
// launch.  With panel_links for all sizes a link was 0.75 us and the step 585 us
// instead of 553 (d = 256: 304 instead of 279; d = 1024, whose first half keeps
// them at 1.1 us a link, write-back included: 1506 and 1459).
#include <hip/hip_runtime.h>
#include <math.h>

#include "gemm_tile.h"
#include "lst_internal.h"

namespace lst {

namespace {

constexpr int kNB = 32;        // panel width
constexpr int kSub = 16;       // diagonal blocks of the row solves
constexpr int kLdT = 36;       // row stride of the 32 x 32 blocks in LDS (16-byte rows)
constexpr int kRB = 4;         // 16-row blocks of a wave in the rank-32 update

// LDS of a panel launch of nt threads: the panel, column by column (the
// updated columns on their way from MFMA layout to a row per thread, then the
// multipliers), and the small blocks.
struct PanelSmall {
  float L11[kNB][kLdT];        // multipliers of pivot rows, by column: L11[k][i] = l_ik
  float U12T[kNB][kLdT];       // U12, a row per column
  float slot[2][16][kLdT];     // each wave's candidate row (by parity of the link)
  unsigned skey[2][16];
  int prow[kNB];               // rows of the previous panel's pivots
  int wcnt[16];
  // panels of up to 512 rows
  float U[kNB][kNB];           // rows of R right of the pivot's eight columns
  float Ud[kNB][8];            // and within them, from the pivot on
  int pslot[kNB];              // active row chosen at each link
  volatile int done;           // links whose multipliers are in T
  int rowid[512];              // the active rows
  short step[512];             // link that chose each active row (kNB: none)
  int bad;                     // a pivot was zero or not finite
};
__host__ __device__ inline size_t panel_lds_bytes(int nt) {
  return (size_t)kNB * (nt + 4) * sizeof(float) + sizeof(PanelSmall);
}

__device__ __forceinline__ unsigned dpp_max(unsigned v, unsigned o) { return v > o ? v : o; }
// Largest v of each row of 16 lanes, in all of them.
__device__ __forceinline__ unsigned row_max16(unsigned v) {
  v = dpp_max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));
  v = dpp_max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
  v = dpp_max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
  v = dpp_max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
  return v;
}
__device__ __forceinline__ unsigned wave_max(unsigned v) {
  v = row_max16(v);
  const unsigned a = (unsigned)__builtin_amdgcn_readlane((int)v, 0);
  const unsigned b = (unsigned)__builtin_amdgcn_readlane((int)v, 16);
  const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)v, 32);
  const unsigned e = (unsigned)__builtin_amdgcn_readlane((int)v, 48);
  return dpp_max(dpp_max(a, b), dpp_max(c, e));
}

// Four floats at p (16-byte aligned when VEC).
template <bool VEC>
__device__ __forceinline__ floatx4 load4(const float* p) {
  if (VEC) return *reinterpret_cast<const floatx4*>(p);
  return floatx4{p[0], p[1], p[2], p[3]};
}

// What one launch works on (the panel at column j0 has R = d - j0 active rows).
struct LuArgs {
  float* A;
  int d, j0;
  int* piv;         // d: row chosen at step k
  const int* act;   // R: the active rows, ascending
  int* act_next;    // R - 32 of them after this panel
  float* dinv;      // per 16-block: L_kk^{-1}, then R_kk^{-1} (256 floats each)
  int* flags;
};

// Inverses of the two 16 x 16 diagonal blocks of L and of R at column q0, by
// one wave: lane 16 b + n holds column n of inverse b (L, L, R, R).  R is
// taken from its last row up, which makes it a lower triangle too.  Rows past
// d are those of the identity.
__device__ void diag_inverses(const LuArgs& a, int q0, PanelSmall& sm) {
  const int lane = threadIdx.x & 63, n = lane & 15, sub = (lane >> 4) & 1;
  const bool low = lane < 32;
  const int nv2 = min(kNB, a.d - q0);  // rows of the panel
  {
    // the panel's 32 x 32 block in pivot order (a wave's LDS accesses complete
    // in order), the identity past its end
    const int c = lane & 31;
    for (int i = lane >> 5; i < kNB; i += 2) {
      const float v = a.A[(size_t)a.piv[q0 + min(i, nv2 - 1)] * a.d + q0 + min(c, nv2 - 1)];
      sm.L11[i][c] = (i < nv2 && c < nv2) ? v : (i == c ? 1.f : 0.f);
    }
    asm volatile("" ::: "memory");
  }
  if (kSub * sub >= nv2) return;
  const int o = kSub * sub;
  float x[kSub];
#pragma unroll
  for (int i = 0; i < kSub; ++i) {
    const int fi = o + (low ? i : kSub - 1 - i);
    float s = (i == n) ? 1.f : 0.f;
#pragma unroll
    for (int k = 0; k < i; ++k) s -= sm.L11[fi][o + (low ? k : kSub - 1 - k)] * x[k];
    x[i] = low ? s : s / sm.L11[fi][fi];
  }
  float* out = a.dinv + (size_t)(2 * ((q0 + o) / kSub) + (low ? 0 : 1)) * (kSub * kSub);
#pragma unroll
  for (int i = 0; i < kSub; ++i) {
    const int r = low ? i : kSub - 1 - i, c = low ? n : kSub - 1 - n;
    out[r * kSub + c] = x[i];
  }
}

// y <- L^{-1} y (16 entries at yp, a lane's own) for the unit lower triangle
// with column k at Lc + kLdT k: each entry is subtracted from all later ones as
// it becomes final, so that the only chain is one multiply-add an entry (a dot
// product per entry is a chain of them).
__device__ __forceinline__ void substitute16(const float* Lc, float* yp) {
  float y[16];
#pragma unroll
  for (int i = 0; i < 16; i += 4) {
    const floatx4 v = *reinterpret_cast<const floatx4*>(yp + i);
    y[i] = v[0]; y[i + 1] = v[1]; y[i + 2] = v[2]; y[i + 3] = v[3];
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) {
#pragma unroll
    for (int i = (k + 1) / 4 * 4; i < 16; i += 4) {
      const floatx4 l = *reinterpret_cast<const floatx4*>(Lc + k * kLdT + i);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (i + q > k) y[i + q] -= l[q] * y[k];
    }
    // (or all of L is read into registers first)
    if (k % 4 == 3) asm volatile("" ::: "memory");
  }
#pragma unroll
  for (int i = 0; i < 16; i += 4)
    *reinterpret_cast<floatx4*>(yp + i) = floatx4{y[i], y[i + 1], y[i + 2], y[i + 3]};
}

// The same for 32 entries: the first 16, their part in the others, the others.
__device__ __forceinline__ void substitute32(const float (*L)[kLdT], float* yp) {
  substitute16(&L[0][0], yp);
  floatx4 y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = *reinterpret_cast<const floatx4*>(yp + 16 + 4 * i);
#pragma unroll 4
  for (int k = 0; k < 16; ++k) {
    const float yk = yp[k];
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] -= *reinterpret_cast<const floatx4*>(&L[k][16 + 4 * i]) * yk;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) *reinterpret_cast<floatx4*>(yp + 16 + 4 * i) = y[i];
  substitute16(&L[16][16], yp + 16);
}

// Columns s0 .. s0 + 31 (as far as they go): U12 = L11^{-1} A[pivots] of the
// panel at column q0 = j0 - 32, written back, then A[active] -= L21 U12.  The
// result stays in LDS (T[column][active row]) or goes back to memory.
template <int NT, bool VEC, bool TO_LDS>
__device__ __forceinline__ void update_columns(const LuArgs& a, int s0, float* T, PanelSmall& sm) {
  constexpr int NW = NT / 64, TLD = NT + 4;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int d = a.d, q0 = a.j0 - kNB, R = d - a.j0, nc = min(kNB, d - s0);
  const int g = lane >> 4, l16 = lane & 15;
  if (tid < kNB) sm.prow[tid] = a.piv[q0 + tid];
  // The wave's rows: 16-row blocks w, w + NW, ...; rows and columns past the
  // end are read at a clamped place and never stored.
  int crow[kRB][4], lrow[kRB];
#pragma unroll
  for (int t = 0; t < kRB; ++t) {
    const int b = kSub * (w + NW * t);
    lrow[t] = a.act[min(b + l16, R - 1)];
#pragma unroll
    for (int r = 0; r < 4; ++r) crow[t][r] = a.act[min(b + 4 * g + r, R - 1)];
  }
  __syncthreads();
  // L11 and the slab's pivot rows: thread (i, c) of 32 x 32, NT / 32 rows at a
  // time, every load issued before the first is used
  constexpr int kPer = kNB * kNB / NT;
  float lv[kPer], uv[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const float* row = a.A + (size_t)sm.prow[(tid >> 5) + u * (NT / 32)] * d;
    lv[u] = row[q0 + (tid & 31)];
    uv[u] = row[s0 + min(tid & 31, nc - 1)];
  }
  // The update's operands are requested before the substitution and used after
  // it, except by 1024 threads, whose 128 registers do not hold them so long.
  floatx4 fl[kRB][2], acc[kRB][2];
  auto operands = [&](int t) {
    if (kSub * (w + NW * t) >= R) return;
    const float* lp = a.A + (size_t)lrow[t] * d + q0 + 4 * g;
    fl[t][0] = load4<VEC>(lp);
    fl[t][1] = load4<VEC>(lp + 16);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* cp = a.A + (size_t)crow[t][r] * d + s0;
      acc[t][0][r] = cp[min(l16, nc - 1)];
      acc[t][1][r] = cp[min(16 + l16, nc - 1)];
    }
  };
  if (NT < 1024)
#pragma unroll
    for (int t = 0; t < kRB; ++t) operands(t);
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int i = (tid >> 5) + u * (NT / 32), c = tid & 31;
    sm.L11[c][i] = lv[u];
    sm.U12T[c][i] = uv[u];
  }
  __syncthreads();
  if (tid < kNB) substitute32(sm.L11, sm.U12T[tid]);  // a column per lane
  __syncthreads();
  {
    const int c = tid & 31;
    if (c < nc)
      for (int i = tid >> 5; i < kNB; i += NT / 32)
        a.A[(size_t)sm.prow[i] * d + s0 + c] = sm.U12T[c][i];
  }
  if (NT == 1024)
#pragma unroll
    for (int t = 0; t < kRB; ++t) operands(t);
  floatx4 fu[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int s = 0; s < 2; ++s)
      fu[h][s] = -*reinterpret_cast<const floatx4*>(&sm.U12T[16 * h + l16][16 * s + 4 * g]);
#pragma unroll
  for (int t = 0; t < kRB; ++t) {
    const int b = kSub * (w + NW * t);
    if (b >= R) continue;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          acc[t][h] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(fl[t][s][q], fu[h][s][q], acc[t][h], 0, 0, 0);
    if (TO_LDS) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<floatx4*>(T + (16 * h + l16) * TLD + b + 4 * g) = acc[t][h];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (b + 4 * g + r >= R) continue;
        float* cp = a.A + (size_t)crow[t][r] * d + s0;
        if (l16 < nc) cp[l16] = acc[t][0][r];
        if (16 + l16 < nc) cp[16 + l16] = acc[t][1][r];
      }
    }
  }
}

// Links c0 .. c0 + 7 of a panel whose rows have W columns left (a[0 .. W), the
// column of the link in a[0]).
template <int NT, int W>
__device__ __forceinline__ void panel_links(float (&x)[kNB], int c0, int nc, bool& active,
                                            int& step, int row, const LuArgs& a, float* T,
                                            PanelSmall& sm) {
  constexpr int NW = NT / 64, TLD = NT + 4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int s = 0; s < 8; ++s) {
    const int c = c0 + s, par = s & 1;
    if (c >= nc) return;
    // |a| as an integer orders like |a| (a NaN above infinity); 0: not active
    const unsigned key = active ? (__float_as_uint(x[0]) & 0x7fffffffu) + 1u : 0u;
    const unsigned wm = wave_max(key);
    const int src = __ffsll((unsigned long long)__ballot(key == wm)) - 1;
    if (lane == src) {
#pragma unroll
      for (int i = 0; i < W; i += 4)
        *reinterpret_cast<floatx4*>(&sm.slot[par][w][i]) =
            floatx4{x[i], x[i + 1], x[i + 2], x[i + 3]};
      sm.skey[par][w] = wm;
    }
    lds_barrier();
    // the first wave with the largest key: ties go to the lower row
    const unsigned k = sm.skey[par][lane & (NW - 1)];
    const unsigned km = (unsigned)__builtin_amdgcn_readfirstlane((int)row_max16(k));
    const int ww = __ffsll((unsigned long long)__ballot(k == km)) - 1;
    float p[W];
#pragma unroll
    for (int i = 0; i < W; i += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(&sm.slot[par][ww][i]);
      p[i] = v[0]; p[i + 1] = v[1]; p[i + 2] = v[2]; p[i + 3] = v[3];
    }
    const float prc = 1.f / p[0];
    if (w == ww && lane == src) {
      active = false;
      step = c;
    }
    const float l = active ? x[0] * prc : 0.f;
    T[c * TLD + tid] = l;
#pragma unroll
    for (int i = 0; i + 1 < W; ++i) x[i] = x[i + 1] - l * p[i + 1];
    if (w == ww) {
      // the row of R, as published; its multipliers are in T
      const int pr = __builtin_amdgcn_readlane(row, src);
      if (lane < W && c + lane < nc)
        a.A[(size_t)pr * a.d + a.j0 + c + lane] = sm.slot[par][ww][lane];
      if (lane == 0) {
        a.piv[a.j0 + c] = pr;
        if (!(fabsf(p[0]) > 0.f) || !isfinite(p[0])) atomicCAS(a.flags + F_ERR, 0, LST_ESINGULAR);
      }
    }
  }
}

// ------------------------------------------------ panels of up to 512 rows
// Four waves, eight columns each, with rows 64 r + lane in their registers.  A
// wave first follows: as a link's multipliers appear in T it takes its own part
// of the pivot row by v_readlane and applies the rank-1 update.  When all
// earlier links are done it leads: largest |a| by DPP, its row by ballots, the
// multipliers into T, one link after another with no barrier and no LDS round
// trip between them.  The update of a link thus runs on four SIMDs, and only
// the leader's eight columns of it lie in the chain.
template <int RPL>
struct WavePanel {
  float x[RPL][8];
  int ret[RPL];   // 0x80000000 once the row is chosen (or does not exist), else 0
  int step[RPL];  // the link that chose it
  float p[8];     // the pivot row

  // Active row 64 r + src is the pivot of link c: its entries into p and to
  // out, and retired.
  template <int r>
  __device__ __forceinline__ void retire(int src, int c, float* out) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      p[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[r][i]), src));
    if ((int)(threadIdx.x & 63) == src) {
      ret[r] = (int)0x80000000;
      step[r] = c;
#pragma unroll
      for (int i = 0; i < 8; i += 4)
        *reinterpret_cast<floatx4*>(out + i) =
            floatx4{x[r][i], x[r][i + 1], x[r][i + 2], x[r][i + 3]};
    }
    // keeps the branches of different r apart (merged, they would index the
    // registers by r)
    asm volatile("; row %0" ::"n"(r));
  }
  // Row r or a later one holds the largest key.
  template <int r>
  __device__ __forceinline__ void choose(const int (&key)[RPL], int wm, int c, PanelSmall& sm) {
    if constexpr (r < RPL) {
      const unsigned long long mk = __ballot(key[r] == wm);
      if (mk != 0ull || r == RPL - 1) {
        const int src = mk != 0ull ? __ffsll((unsigned long long)mk) - 1 : 0;
        retire<r>(src, c, sm.Ud[c]);
        if ((threadIdx.x & 63) == 0) sm.pslot[c] = 64 * r + src;
      } else {
        choose<r + 1>(key, wm, c, sm);
      }
    }
  }
  template <int r>
  __device__ __forceinline__ void take(int slot, int c, float* out) {
    if constexpr (r < RPL) {
      if ((slot >> 6) == r || r == RPL - 1)
        retire<r>(slot & 63, c, out);
      else
        take<r + 1>(slot, c, out);
    }
  }

  __device__ __forceinline__ void run(int w, int R, int nc, float* T, int tld, PanelSmall& sm) {
    const int lane = threadIdx.x & 63, cb = 8 * w;
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      ret[r] = 64 * r + lane < R ? 0 : (int)0x80000000;
      step[r] = kNB;
#pragma unroll
      for (int i = 0; i < 8; ++i) x[r][i] = T[(cb + i) * tld + 64 * r + lane];
    }
    for (int c = 0; c < cb; ++c) {
      while (sm.done <= c) __builtin_amdgcn_s_sleep(1);  // a leader always gets there
      asm volatile("" ::: "memory");
      const int slot = __builtin_amdgcn_readfirstlane(sm.pslot[c]);
      float l[RPL];
#pragma unroll
      for (int r = 0; r < RPL; ++r) l[r] = T[c * tld + 64 * r + lane];
      take<0>(slot, c, &sm.U[c][cb]);
#pragma unroll
      for (int r = 0; r < RPL; ++r)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[r][i] -= l[r] * p[i];
    }
    // lead: the column of the link is x[.][0], the rows shift as they are updated
    for (int s = 0; s < 8; ++s) {
      const int c = cb + s;
      if (c >= nc) break;
      // |a| as an integer orders like |a| (a NaN above infinity); chosen rows
      // are negative
      int key[RPL], km = (int)0x80000000;
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        key[r] = (__float_as_int(x[r][0]) & 0x7fffffff) | ret[r];
        km = max(km, key[r]);
      }
      km = max(km, __builtin_amdgcn_update_dpp(0, km, 0x128, 0xf, 0xf, false));
      km = max(km, __builtin_amdgcn_update_dpp(0, km, 0x124, 0xf, 0xf, false));
      km = max(km, __builtin_amdgcn_update_dpp(0, km, 0x122, 0xf, 0xf, false));
      km = max(km, __builtin_amdgcn_update_dpp(0, km, 0x121, 0xf, 0xf, false));
      const int wm = max(max(__builtin_amdgcn_readlane(km, 0), __builtin_amdgcn_readlane(km, 16)),
                         max(__builtin_amdgcn_readlane(km, 32), __builtin_amdgcn_readlane(km, 48)));
      choose<0>(key, wm, c, sm);
      if (lane == 0 && (!(fabsf(p[0]) > 0.f) || !isfinite(p[0]))) sm.bad = 1;
      const float rc = 1.f / p[0];
      float l[RPL];
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        l[r] = ret[r] == 0 ? x[r][0] * rc : 0.f;
        T[c * tld + 64 * r + lane] = l[r];
      }
      // published after the multipliers and pslot (a wave's LDS accesses
      // complete in order)
      asm volatile("" ::: "memory");
      if (lane == 0) sm.done = c + 1;
#pragma unroll
      for (int r = 0; r < RPL; ++r)
#pragma unroll
        for (int i = 0; i < 7; ++i) x[r][i] = x[r][i + 1] - l[r] * p[i + 1];
    }
    if (w == (nc - 1) / 8) {  // it has seen every link
#pragma unroll
      for (int r = 0; r < RPL; ++r) sm.step[64 * r + lane] = (short)step[r];
    }
  }
};

// The panel's columns in T, active rows 0 .. R - 1 (R <= 64 RPL).
template <int RPL>
__device__ __forceinline__ void factor_by_waves(float* T, int tld, int R, int nc, PanelSmall& sm) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (8 * w < nc) {  // waves 0 .. 3
    WavePanel<RPL> wp;
    wp.run(w, R, nc, T, tld, sm);
  }
}

// Links of a panel of more than 512 rows: a row per thread, all waves.
template <int NT>
__device__ __forceinline__ void factor_by_block(const LuArgs& a, float* T, int R, int nc, int row,
                                                bool& active, PanelSmall& sm) {
  constexpr int TLD = NT + 4;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  float x[kNB];
  // (threads past the rows and columns past the panel hold values that are
  // never used: a row that is not active takes no part, a column past the end
  // is not reached)
#pragma unroll
  for (int c = 0; c < kNB; ++c) x[c] = T[c * TLD + tid];
  int step = kNB;  // the link that chose this row
  // a wave writes T only at its own rows, which only it has read
  panel_links<NT, 32>(x, 0, nc, active, step, row, a, T, sm);
  panel_links<NT, 24>(x, 8, nc, active, step, row, a, T, sm);
  panel_links<NT, 16>(x, 16, nc, active, step, row, a, T, sm);
  panel_links<NT, 8>(x, 24, nc, active, step, row, a, T, sm);
  // the multipliers go back: 32 lanes a row, each up to the link that chose it
  for (int r0 = 0; r0 < 64; r0 += 2) {
    const int src = r0 + (lane >> 5), c = lane & 31;
    const int rr = __shfl(row, src), st = __shfl(step, src);
    const int t = 64 * w + src;
    if (t < R && c < nc && c < st) a.A[(size_t)rr * a.d + a.j0 + c] = T[c * TLD + t];
  }
}

template <int NT, bool VEC>
__global__ __launch_bounds__(NT) void lu_panel_kernel(LuArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  constexpr int NW = NT / 64, TLD = NT + 4;
  float* T = reinterpret_cast<float*>(lds_raw);
  PanelSmall& sm = *reinterpret_cast<PanelSmall*>(lds_raw + (size_t)kNB * TLD * sizeof(float));
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = a.d, R = d - a.j0, nc = min(kNB, R);
  if (blockIdx.x > 0) {
    const int s0 = a.j0 + kNB * (int)blockIdx.x;
    if (s0 < d)
      update_columns<NT, VEC, false>(a, s0, T, sm);
    else if (w == 0)
      diag_inverses(a, a.j0 - kNB, sm);
    return;
  }
  bool active = tid < R;
  const int row = a.act[min(tid, R - 1)];
  if (NT < 1024) sm.rowid[tid & 511] = row;
  if (tid == 0) {
    sm.done = 0;
    sm.bad = 0;
  }
  if (a.j0 > 0) {
    update_columns<NT, VEC, true>(a, a.j0, T, sm);
  } else {
    // 32 lanes a row
    for (int t = tid >> 5; t < R; t += NT / 32)
      T[(tid & 31) * TLD + t] = a.A[(size_t)a.act[t] * d + min(tid & 31, nc - 1)];
  }
  __syncthreads();
  if constexpr (NT == 1024) {
    factor_by_block<NT>(a, T, R, nc, row, active, sm);
  } else {
    const int rpl = (R + 63) / 64;  // 1 .. NT / 64
    switch (rpl) {
      case 1: factor_by_waves<1>(T, TLD, R, nc, sm); break;
      case 2: factor_by_waves<2>(T, TLD, R, nc, sm); break;
      case 3: factor_by_waves<3>(T, TLD, R, nc, sm); break;
      case 4: factor_by_waves<4>(T, TLD, R, nc, sm); break;
      default:
        if constexpr (NT == 512) {
          if (rpl == 5) factor_by_waves<5>(T, TLD, R, nc, sm);
          else if (rpl == 6) factor_by_waves<6>(T, TLD, R, nc, sm);
          else if (rpl == 7) factor_by_waves<7>(T, TLD, R, nc, sm);
          else factor_by_waves<8>(T, TLD, R, nc, sm);
        }
        break;
    }
    __syncthreads();
    // everything goes back: multipliers before the link that chose the row,
    // the row of R from there on
    {
      const int c = tid & 31;
#pragma unroll 4
      for (int t = tid >> 5; t < R; t += NT / 32) {
        const int st = sm.step[t];
        const float* src = c < st                  ? T + c * TLD + t
                           : (c >> 3) == (st >> 3) ? &sm.Ud[st][c - st]
                                                   : &sm.U[st][c];
        const float v = *src;
        if (c < nc) a.A[(size_t)sm.rowid[t] * d + a.j0 + c] = v;
      }
    }
    if (tid < R) {
      const int st = sm.step[tid];
      active = st == kNB;
      if (!active) a.piv[a.j0 + st] = row;
    }
    if (tid == 0 && sm.bad) atomicCAS(a.flags + F_ERR, 0, LST_ESINGULAR);
  }
  // the rows that stay active, in order
  const unsigned long long on = __ballot(active);
  if (lane == 0) sm.wcnt[w] = __popcll(on);
  __syncthreads();
  int off = __popcll(on & ((1ull << lane) - 1ull));
  for (int v = 0; v < w; ++v) off += sm.wcnt[v];
  if (active) a.act_next[off] = row;
  // the last panel's own diagonal blocks (after the barrier above, which
  // follows the block's stores to A and piv)
  if (R <= kNB && w == 0) diag_inverses(a, a.j0, sm);
}

__global__ __launch_bounds__(256) void lu_iota_kernel(int* act, int d) {
  for (int j = blockIdx.x * 256 + threadIdx.x; j < d; j += gridDim.x * 256) act[j] = j;
}

// X_i = -lr a_i z_i with P A = L R and A z_i = h_i, 16 examples a workgroup.
// Wave w owns the 16-blocks w, w + NW, ... of the unknowns (RB of them); the
// accumulator of a block holds unknowns 4 g + r (g = lane / 16) of example
// lane % 16.
template <int RB, bool VEC>
__global__ __launch_bounds__(1024) void lu_rows_kernel(const float* __restrict__ F,
                                                       const int* __restrict__ piv,
                                                       const float* __restrict__ dinv, int d,
                                                       const float* __restrict__ H, int m,
                                                       float* __restrict__ Xout,
                                                       const float* __restrict__ acoef, float lr) {
  constexpr int NW = 16;
  constexpr int PF = RB <= 2 ? 4 : 2;  // links whose fragments are in flight
  __shared__ floatx4 xs[2][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const int nb = (d + kSub - 1) / kSub;
  const int ex = blockIdx.x * kSub + l16;
  const float* hr = H + (size_t)min(ex, m - 1) * d;
  floatx4 acc[RB];
  const float* rp[RB];
#pragma unroll
  for (int t = 0; t < RB; ++t) {
    const int b = kSub * (w + NW * t);
    rp[t] = F + (size_t)piv[min(b + l16, d - 1)] * d;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = b + 4 * g + r;
      const float h = hr[piv[min(j, d - 1)]];
      acc[t][r] = j < d ? h : 0.f;
    }
  }
  // Block J's columns of the rows of slot t.  Past the matrix's end they are
  // read at a clamped place: unknowns past it are published as zeros, and
  // accumulators of rows past it reach nothing else.  No branch, so that the
  // loads of several links stay in flight.
  auto frag = [&](int t, int J) {
    const int k = kSub * J + 4 * g;
    if (VEC) return *reinterpret_cast<const floatx4*>(rp[t] + min(k, d - 4));
    return floatx4{rp[t][min(k, d - 1)], rp[t][min(k + 1, d - 1)], rp[t][min(k + 2, d - 1)],
                   rp[t][min(k + 3, d - 1)]};
  };
  auto diag = [&](int J, int up) {
    return *reinterpret_cast<const floatx4*>(dinv + (size_t)(2 * min(J, nb - 1) + up) *
                                                        (kSub * kSub) +
                                             l16 * kSub + 4 * g);
  };
  floatx4 dv[RB];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const bool up = pass == 1;
#pragma unroll
    for (int t = 0; t < RB; ++t) dv[t] = diag(w + NW * t, pass);
    // links in order of slots: while slot S is solved, the slots after it (up:
    // before it) take every block, slot S the blocks before (after) its own
#pragma unroll
    for (int SS = 0; SS < RB; ++SS) {
      const int S = up ? RB - 1 - SS : SS;
      floatx4 f[PF][RB];
      auto block_of = [&](int i) { return NW * S + (up ? NW - 1 - i : i); };
      auto load = [&](floatx4(&fr)[RB], int i) {
        const int J = block_of(min(i, NW - 1));
#pragma unroll
        for (int t = 0; t < RB; ++t)
          if (up ? t <= S : t >= S) fr[t] = frag(t, min(J, nb - 1));
      };
#pragma unroll
      for (int i = 0; i + 1 < PF; ++i) load(f[i], i);
#pragma unroll 1
      for (int i0 = 0; i0 < NW; i0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          const int i = i0 + u, J = block_of(i), par = u & 1;
          load(f[(u + PF - 1) % PF], i + PF - 1);
          if (J < nb) {  // uniform
            const bool own = w == J - NW * S;
            if (own) {
              floatx4 xv = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int q = 0; q < 4; ++q)
                xv = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[S][q], acc[S][q], xv, 0, 0, 0);
#pragma unroll
              for (int r = 0; r < 4; ++r) xv[r] = kSub * J + 4 * g + r < d ? xv[r] : 0.f;
              acc[S] = xv;
              xs[par][lane] = xv;
            }
            lds_barrier();
            const floatx4 xb = -xs[par][lane];
#pragma unroll
            for (int tt = 0; tt < RB; ++tt) {
              const int t = up ? RB - 1 - tt : tt;
              const bool take = t == S ? (up ? w < J - NW * S : w > J - NW * S)
                                       : (up ? t < S : t > S);
              if (take) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                  acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[u][t][q], xb[q], acc[t], 0, 0, 0);
              }
            }
          }
        }
      }
    }
  }
  if (ex >= m) return;
  const float sc = -lr * acoef[ex];
  float* out = Xout + (size_t)ex * d;
#pragma unroll
  for (int t = 0; t < RB; ++t) {
    const int j = kSub * (w + NW * t) + 4 * g;
    if (VEC) {
      if (j < d) *reinterpret_cast<floatx4*>(out + j) = acc[t] * sc;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j + r < d) out[j + r] = acc[t][r] * sc;
    }
  }
}

template <int NT>
hipError_t panel_launch(const LuArgs& a, int blocks, bool vec, hipStream_t s) {
  const size_t lds = panel_lds_bytes(NT);
  if (vec)
    hipLaunchKernelGGL((lu_panel_kernel<NT, true>), dim3(blocks), dim3(NT), lds, s, a);
  else
    hipLaunchKernelGGL((lu_panel_kernel<NT, false>), dim3(blocks), dim3(NT), lds, s, a);
  return hipGetLastError();
}

template <int NT>
hipError_t panel_configure() {
  const void* k[2] = {reinterpret_cast<const void*>(&lu_panel_kernel<NT, true>),
                      reinterpret_cast<const void*>(&lu_panel_kernel<NT, false>)};
  for (const void* f : k) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)panel_lds_bytes(NT));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int RB>
hipError_t rows_launch(const float* F, const int* piv, const float* dinv, int d, const float* H,
                       int m, float* Xout, const float* acoef, float lr, bool vec, hipStream_t s) {
  const dim3 grid((m + kSub - 1) / kSub);
  if (vec)
    hipLaunchKernelGGL((lu_rows_kernel<RB, true>), grid, dim3(1024), 0, s, F, piv, dinv, d, H, m,
                       Xout, acoef, lr);
  else
    hipLaunchKernelGGL((lu_rows_kernel<RB, false>), grid, dim3(1024), 0, s, F, piv, dinv, d, H, m,
                       Xout, acoef, lr);
  return hipGetLastError();
}

}  // namespace

size_t lu_dinv_floats(int d) { return (size_t)2 * ((d + kNB - 1) / kNB * 2) * kSub * kSub; }

hipError_t lu_configure() {
  hipError_t e = panel_configure<256>();
  if (e == hipSuccess) e = panel_configure<512>();
  if (e == hipSuccess) e = panel_configure<1024>();
  return e;
}

hipError_t lu_factor(float* A, int d, int* piv, int* act, float* dinv, int* flags,
                     hipStream_t s) {
  if (d < 1 || d > kLuMaxD) return hipErrorInvalidValue;
  hipLaunchKernelGGL(lu_iota_kernel, dim3((d + 255) / 256), dim3(256), 0, s, act, d);
  const bool vec = d % 4 == 0;  // A comes from the device allocator: its rows are then aligned
  for (int j0 = 0, p = 0; j0 < d; j0 += kNB, ++p) {
    const int R = d - j0;
    const LuArgs a{A, d, j0, piv, act + (p & 1) * d, act + ((p & 1) ^ 1) * d, dinv, flags};
    // the columns right of the panel, and the previous panel's diagonal blocks
    const int blocks = j0 == 0 ? 1 : 1 + (R > kNB ? (R - kNB + kNB - 1) / kNB : 0) + 1;
    // a thread per active row, in the update's products and the write-back (above
    // 512 rows also in the links, whose barriers are shorter with fewer waves)
    const hipError_t e = R <= 256   ? panel_launch<256>(a, blocks, vec, s)
                         : R <= 512 ? panel_launch<512>(a, blocks, vec, s)
                                    : panel_launch<1024>(a, blocks, vec, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t lu_solve_rows(const float* F, const int* piv, const float* dinv, int d, const float* H,
                         int m, float* Xout, const float* acoef, float lr, hipStream_t s) {
  if (d < 1 || d > kLuMaxD || m < 1) return hipErrorInvalidValue;
  const bool vec = d % 4 == 0;  // F and Xout come from the device allocator
  if (d <= 256) return rows_launch<1>(F, piv, dinv, d, H, m, Xout, acoef, lr, vec, s);
  if (d <= 512) return rows_launch<2>(F, piv, dinv, d, H, m, Xout, acoef, lr, vec, s);
  return rows_launch<4>(F, piv, dinv, d, H, m, Xout, acoef, lr, vec, s);
}

}  // namespace lst
