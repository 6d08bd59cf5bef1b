// fp32 MFMA GEMM for the large products outside the step: the naive
// explicit-W baseline, W = V U, the initial W^T W.  (The step's own small
// products run as panel tiles inside the step kernel; see gemm_tile.h.)
#include "gemm_tile.h"

namespace lst {

// ---------------------------------------------------------------------------
// Large products (the naive explicit-W baseline, V U, the initial W^T W): TM x
// 128 output tiles, K in slices of 32 that LDS-DMA (BigRegs for rows that are not
// aligned) brings into one of two LDS stages while the other is multiplied, four
// waves of 32 x 32 blocks on
// v_mfma_f32_32x32x2f32.  Bound by the fp32 MFMA rate from m = 128 on, by
// memory below about m = 64 (TM follows M, so that padding is not multiplied).
//   - 64 KB of LDS (TM = 128): two workgroups share a compute unit, and one
//     multiplies while the other waits for its first slice or stores its tile.
//   - An operand whose k is contiguous lands as rows of 32 floats, one whose
//     output index is contiguous as 32 rows of T floats, both as they lie in
//     memory; 16-byte slots are XOR-swizzled so that fragment reads are free of
//     bank conflicts.  (Transposing through registers cost W -= lr R^T H 720 us
//     at D = 200 000, d = 500, m = 128.)
//   - The product is computed transposed (MFMA rows are output columns), so a
//     lane holds four consecutive columns of an output row: 16-byte loads and
//     stores, the old C in flight during the last slice.
// At D = 200 000, d = 500, m = 128 (25.6 GFLOP each): O = H^T W^T 265 us (303
// before), grad_H 230 (291), W -= lr R^T H 322 (724); the MFMA units are busy 61,
// 70 and 50 % of the time.  Tiles of 64 columns, a raised wave priority while
// multiplying and 64-row tiles for the last product changed less than 2 %.
// ---------------------------------------------------------------------------
constexpr int GB_BK = 32;

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Place of a 16-byte piece of an operand's slice: pieces e = 0 .. 8 T - 1, in the
// order of S and, up to the swizzle, of memory.  k-contiguous: rows [o0, o0 + T) x
// k in [k0, k0 + 32) as S[row][slot ^ (row & 7)].  Otherwise k in [k0, k0 + 32) x
// columns [o0, o0 + T) as S[k][slot ^ (8 if k & 4)] (the two halves of a wave read
// rows k and k + 4 together).  slot: the memory's slot that piece e of S holds.
template <int T, int KC>
struct BigPiece {
  static constexpr int SLOTS = KC ? GB_BK / 4 : T / 4;
  static constexpr int SW = T / 4 >= 16 ? 8 : 4;  // T = 32: 8 slots a row
  int row, slot;
  __device__ __forceinline__ explicit BigPiece(int e)
      : row(e / SLOTS), slot((e % SLOTS) ^ (KC ? row & 7 : (row & 4) ? SW : 0)) {}
};

// A slice by LDS-DMA, zeros outside [0, nout) x [0, kend): rows of both operands
// 16-byte aligned; k-contiguous: kend % 4 == 0; otherwise the last piece of a row
// may carry columns >= nout, which reach only outputs that are not stored.
template <int T, int KC>
__device__ __forceinline__ void big_fill(const VMat& v, int o0, int nout, int k0, int kend,
                                         float* S, int part, int parts) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned base = lds_u32(S);
  constexpr int NI = T * GB_BK / 256 / 4;
#pragma unroll
  for (int u = 0; u < NI; ++u) {
    if (u * parts / NI != part) continue;
    const int j = wave + 4 * u;
    const BigPiece<T, KC> p(64 * j + lane);
    const int o = o0 + (KC ? p.row : 4 * p.slot), k = k0 + (KC ? 4 * p.slot : p.row);
    const float* gp =
        o < nout && k < kend ? vm_row(v, KC ? o : k) + (KC ? k : o) : g_dma_zero;
    dma16(gp, base + 1024u * j);
  }
}

// A slice through registers, for rows that are not aligned: loads of 16 bytes at
// 4-byte addresses, element by element where a piece crosses the operand's end.
// An LDS-DMA lane takes only 4 bytes an instruction there: V U at D = 50 000, d =
// 126: 47 us against 39 so, d = 301: 192 and 153; a step of the explicit layer at
// D = 20 000, d = 514, m = 500: 689 and 534.
typedef float floatx4_a4 __attribute__((ext_vector_type(4), aligned(4)));

template <int T, int KC>
struct BigRegs {
  static constexpr int NI = T * GB_BK / 4 / 256;
  floatx4 x[NI];
  __device__ __forceinline__ void load(const VMat& v, int o0, int nout, int k0, int kend) {
#pragma unroll
    for (int u = 0; u < NI; ++u) {
      const BigPiece<T, KC> p(threadIdx.x + 256 * u);
      const int o = o0 + (KC ? p.row : 4 * p.slot), k = k0 + (KC ? 4 * p.slot : p.row);
      const int left = o < nout && k < kend ? (KC ? kend - k : nout - o) : 0;
      x[u] = floatx4{0.f, 0.f, 0.f, 0.f};
      if (left > 0) {
        const float* gp = vm_row(v, KC ? o : k) + (KC ? k : o);
        if (left >= 4) {
          x[u] = *reinterpret_cast<const floatx4_a4*>(gp);
        } else {
          x[u][0] = gp[0];
          if (left > 1) x[u][1] = gp[1];
          if (left > 2) x[u][2] = gp[2];
        }
      }
    }
  }
  __device__ __forceinline__ void store(float* S) const {
#pragma unroll
    for (int u = 0; u < NI; ++u)
      *reinterpret_cast<floatx4*>(S + 4 * (threadIdx.x + 256 * u)) = x[u];
  }
};

// The MFMA operand of row r (of T) for the k of an 8-wide slice at kk: register
// q of half h = lane / 32 holds k = kk + 4 h + q.
template <int T, int KC>
__device__ __forceinline__ floatx4 big_frag(const float* S, int r, int kk) {
  const int h = (threadIdx.x >> 5) & 1;
  if (KC) {
    return *reinterpret_cast<const floatx4*>(S + r * GB_BK + 4 * (((kk >> 2) + h) ^ (r & 7)));
  } else {
    constexpr int SW = T / 4 >= 16 ? 8 : 4;
    floatx4 f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = kk + 4 * h + q;
      f[q] = S[k * T + 4 * ((r >> 2) ^ (h ? SW : 0)) + (r & 3)];
    }
    return f;
  }
}

template <int TM, int TN, bool DMA, int A_KC, int B_KC>
__global__ __launch_bounds__(256, 2) void gemm_big_kernel(GemmProblem P, int total,
                                                          const int* skip_if, const int* run_if,
                                                          int pad) {
  if (skip_if && *skip_if) return;
  if (run_if && !*run_if) return;
  constexpr int WM = TM == 32 ? 1 : 2, WN = 4 / WM;           // waves
  constexpr int IM = TM / WM / 32, IN = TN / WN / 32;       // 32 x 32 blocks of a wave
  constexpr int AF = TM * GB_BK, STAGE = (TM + TN) * GB_BK; // floats
  __shared__ __attribute__((aligned(16))) float smem[2][STAGE];
  // consecutive tiles of an XCD share the rows of A
  int lt = xcd_tile(blockIdx.x, total);
  const int per = P.tiles_m * P.tiles_n;
  const int z = lt / per;
  lt -= z * per;
  const int tm = lt / P.tiles_n, tn = lt - tm * P.tiles_n;
  int kb = 0, ke = P.K;
  if (P.ksplit > 1) {
    const int kc = ((P.K + P.ksplit - 1) / P.ksplit + GB_BK - 1) / GB_BK * GB_BK;
    kb = min(P.K, z * kc);
    ke = min(P.K, kb + kc);
  }
  const int m0 = tm * TM, n0 = tn * TN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave - wm * WN;
  const int l32 = lane & 31, h = lane >> 5;
  floatx16 acc[IM][IN];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < IN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const VMat A = P.A, B = P.B;
  // part p (of parts) of slice c; parts and p are constants where it is called
  auto fill = [&](int c, int p, int parts) __attribute__((always_inline)) {
    float* S = smem[c & 1];
    const int k0 = kb + c * GB_BK;
    big_fill<TM, A_KC>(A, m0, P.M, k0, ke, S, p, parts);
    big_fill<TN, B_KC>(B, n0, P.N, k0, ke, S + AF, p, parts);
  };
  const int nch = (ke - kb + GB_BK - 1) / GB_BK;
  // output row of block i, first of the four output columns of group q of block j
  auto row_of = [&](int i) { return m0 + (wm * IM + i) * 32 + l32; };
  auto col_of = [&](int j, int q) { return n0 + (wn * IN + j) * 32 + 8 * q + 4 * h; };
  const bool keep = P.epi == EPI_STORE && P.beta != 0.f;
  float* C = P.epi == EPI_PARTIAL ? P.C + (size_t)z * P.M * P.N : P.C;
  const int ldc = P.epi == EPI_PARTIAL ? P.N : P.ldc;
  // (with PAD_C a last piece carries zeros past column N, as B's rows there are
  // zero; NaN in a row of A that is not finite)
  const bool vecc = (P.N % 4 == 0 || (pad & PAD_C)) && ldc % 4 == 0 && ((uintptr_t)C & 15) == 0;
  // Multiplies slice c; with next, slice c + 1 is requested a part at a time
  // between the MFMAs (all of it at once holds the wave for as long as the
  // memory pipeline takes to accept it).
  auto multiply = [&](int c, bool next) __attribute__((always_inline)) {
    const float* Sa = smem[c & 1];
    const float* Sb = Sa + AF;
    auto frags = [&](int kk, floatx4(&fa)[IM], floatx4(&fb)[IN]) {
#pragma unroll
      for (int i = 0; i < IM; ++i)
        fa[i] = big_frag<TM, A_KC>(Sa, (wm * IM + i) * 32 + l32, kk);
#pragma unroll
      for (int j = 0; j < IN; ++j)
        fb[j] = big_frag<TN, B_KC>(Sb, (wn * IN + j) * 32 + l32, kk);
    };
    floatx4 fa[2][IM], fb[2][IN];
    frags(0, fa[0], fb[0]);
#pragma unroll
    for (int s = 0; s < GB_BK / 8; ++s) {
      if (s + 1 < GB_BK / 8) frags(8 * (s + 1), fa[(s + 1) & 1], fb[(s + 1) & 1]);
      if (next) fill(c + 1, s, GB_BK / 8);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int j = 0; j < IN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[s & 1][j][q], fa[s & 1][i][q],
                                                             acc[i][j], 0, 0, 0);
    }
  };
  if constexpr (DMA) {
    if (nch > 0) fill(0, 0, 1);
    for (int c = 0; c + 1 < nch; ++c) {
      wait_vm_le(0);
      lds_barrier();  // slice c has landed; every wave is done with slice c - 1
      multiply(c, true);
    }
    wait_vm_le(0);
  } else {
    BigRegs<TM, A_KC> ra;
    BigRegs<TN, B_KC> rb;
    auto load = [&](int c) __attribute__((always_inline)) {
      ra.load(A, m0, P.M, kb + c * GB_BK, ke);
      rb.load(B, n0, P.N, kb + c * GB_BK, ke);
    };
    auto store = [&](int c) __attribute__((always_inline)) {
      ra.store(smem[c & 1]);
      rb.store(smem[c & 1] + AF);
    };
    if (nch > 0) {
      load(0);
      store(0);
    }
    for (int c = 0; c + 1 < nch; ++c) {
      lds_barrier();  // as above
      load(c + 1);
      multiply(c, false);
      store(c + 1);
    }
  }
  lds_barrier();
  floatx4 old[IM][IN][4];
  if (keep) {
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < IN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = min(row_of(i), P.M - 1), col = col_of(j, q);
          const float* cp = C + (size_t)row * ldc;
          if (vecc) {
            old[i][j][q] = *reinterpret_cast<const floatx4*>(cp + min(col, P.N - 4));
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) old[i][j][q][r] = cp[min(col + r, P.N - 1)];
          }
        }
  }
  if (nch > 0) multiply(nch - 1, false);
  const float alpha = P.epi == EPI_PARTIAL ? 1.f : P.alpha, beta = P.beta;
#pragma unroll
  for (int i = 0; i < IM; ++i) {
    const int row = row_of(i);
    if (row >= P.M) continue;
#pragma unroll
    for (int j = 0; j < IN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = col_of(j, q);
        floatx4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = alpha * acc[i][j][4 * q + r];
        if (keep) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] += beta * old[i][j][q][r];
        }
        float* cp = C + (size_t)row * ldc;
        if (vecc) {
          if (col < P.N) *reinterpret_cast<floatx4*>(cp + col) = v;
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (col + r < P.N) cp[col + r] = v[r];
        }
      }
  }
}

namespace {

template <int TM, int TN, bool DMA>
void big_dispatch(const GemmProblem& p, int total, const int* skip_if, const int* run_if, int pad,
                  hipStream_t s) {
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(total), dim3(256), 0, s, p, total, skip_if, run_if,
                       pad);
  };
  if (p.a_kc && p.b_kc) run(gemm_big_kernel<TM, TN, DMA, 1, 1>);
  else if (p.a_kc) run(gemm_big_kernel<TM, TN, DMA, 1, 0>);
  else run(gemm_big_kernel<TM, TN, DMA, 0, 0>);
}

}  // namespace

hipError_t gemm_big_launch(GemmProblem p, hipStream_t s, const int* skip_if, const int* run_if,
                           int pad) {
  if (p.epi != EPI_STORE && p.epi != EPI_PARTIAL) return hipErrorInvalidValue;
  if (!p.a_kc && p.b_kc) return hipErrorInvalidValue;
  if ((pad & PAD_K) && (!p.a_kc || p.b_kc)) return hipErrorInvalidValue;
  if ((pad & PAD_C) && (p.epi != EPI_STORE || p.beta != 0.f || !p.b_kc)) return hipErrorInvalidValue;
  if (p.ksplit < 1) p.ksplit = 1;
  constexpr int kTN = 128;
  // the tile's rows: for M >= 16 at most half of them padding (M is the minibatch
  // or D or d)
  const int tmr = p.M <= 32 ? 32 : p.M <= 64 ? 64 : 128;
  p.tiles_m = (p.M + tmr - 1) / tmr;
  p.tiles_n = (p.N + kTN - 1) / kTN;
  const int total = p.tiles_m * p.tiles_n * (p.epi == EPI_PARTIAL ? p.ksplit : 1);
  if (total == 0) return hipSuccess;
  // LDS-DMA takes pieces of 16 bytes: aligned rows, and whole pieces of a contiguous
  // k (PAD_K: the last piece's zeros meet the zeros of B's rows past K)
  const bool v16 = p.A.vec && p.B.vec &&
                   ((!p.a_kc && !p.b_kc) || p.K % 4 == 0 || (pad & PAD_K));
  if (v16) {
    if (tmr == 32) big_dispatch<32, kTN, true>(p, total, skip_if, run_if, pad, s);
    else if (tmr == 64) big_dispatch<64, kTN, true>(p, total, skip_if, run_if, pad, s);
    else big_dispatch<128, kTN, true>(p, total, skip_if, run_if, pad, s);
  } else {
    if (tmr == 32) big_dispatch<32, kTN, false>(p, total, skip_if, run_if, pad, s);
    else if (tmr == 64) big_dispatch<64, kTN, false>(p, total, skip_if, run_if, pad, s);
    else big_dispatch<128, kTN, false>(p, total, skip_if, run_if, pad, s);
  }
  return hipGetLastError();
}

// C = alpha * sum_z ws[z] + beta * C, the slices added in order within each
// quarter of them (a wave each), then the quarters (split-K partials of grad_H
// at m = 128, d = 500, 128 slices: 6.5 us; 32 with a thread per entry and
// all slices one after another).
constexpr int kRedBatch = 8;

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* ws, int splits, int M,
                                                            int N, float* C, int ldc, float alpha,
                                                            float beta, int sym,
                                                            const int* skip_if) {
  if (skip_if && *skip_if) return;
  __shared__ float part[3][64];
  const size_t total = (size_t)M * N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int per = (splits + 3) / 4, zb = w * per, ze = min(splits, zb + per);
  for (size_t e0 = (size_t)blockIdx.x * 64; e0 < total; e0 += (size_t)gridDim.x * 64) {
    const size_t e = e0 + lane, ec = e < total ? e : total - 1;
    float s = 0.f;
    for (int z0 = zb; z0 < ze; z0 += kRedBatch) {
      float v[kRedBatch];
#pragma unroll
      for (int u = 0; u < kRedBatch; ++u) v[u] = ws[(size_t)min(z0 + u, ze - 1) * total + ec];
#pragma unroll
      for (int u = 0; u < kRedBatch; ++u) s += z0 + u < ze ? v[u] : 0.f;
    }
    if (w > 0) part[w - 1][lane] = s;
    __syncthreads();
    if (w == 0 && e < total) {
      const int r = (int)(e / N), c = (int)(e - (size_t)r * N);
      s = ((s + part[0][lane]) + part[1][lane]) + part[2][lane];
      if (!(sym && r > c)) {
        float o = alpha * s;
        if (beta != 0.f) o += beta * C[(size_t)r * ldc + c];
        C[(size_t)r * ldc + c] = o;
        if (sym) C[(size_t)c * ldc + r] = o;
      }
    }
    __syncthreads();
  }
}

static int aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

VMat vmat(const float* p, int ld, int rows) {
  VMat v{};
  v.p[0] = p;
  v.ld[0] = ld;
  v.r1 = rows;
  v.nb = 1;
  v.vec = (ld % 4 == 0) && aligned16(p);
  return v;
}

VMat vmat2(const float* p0, int ld0, int rows0, const float* p1, int ld1, int rows1) {
  VMat v{};
  v.p[0] = p0;
  v.ld[0] = ld0;
  v.p[1] = p1;
  v.ld[1] = ld1;
  v.r1 = rows0;  // block 1 holds rows [rows0, rows0 + rows1)
  (void)rows1;
  v.nb = 2;
  v.vec = (ld0 % 4 == 0) && (ld1 % 4 == 0) && aligned16(p0) && aligned16(p1);
  return v;
}

GemmProblem gemm_problem(int layout, int M, int N, int K, const VMat& A, const VMat& B, float* C,
                         int ldc, float alpha, float beta, int epi) {
  GemmProblem p{};
  p.M = M; p.N = N; p.K = K;
  p.a_kc = (layout != L_TN);
  p.b_kc = (layout == L_NT);
  p.A = A; p.B = B;
  p.C = C; p.ldc = ldc;
  p.alpha = alpha; p.beta = beta;
  p.epi = epi;
  p.ksplit = 1;
  return p;
}

hipError_t gemm_splitk_reduce(const float* ws, int splits, int M, int N, float* C, int ldc,
                              float alpha, float beta, int sym, const int* skip_if,
                              hipStream_t s) {
  const size_t total = (size_t)M * N;
  int blocks = (int)((total + 63) / 64);
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks), dim3(256), 0, s, ws, splits, M, N, C,
                     ldc, alpha, beta, sym, skip_if);
  return hipGetLastError();
}

}  // namespace lst
