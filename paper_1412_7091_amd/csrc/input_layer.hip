// The sparse input layer of section 2.2 ("the easy part"): a K-sparse input
// x (K (index, value) pairs per example; index -1 unused) enters the first
// hidden layer through a D_in x d matrix W_in, so that
//   forward: A[i, :] = sum_k v_ik W_in[u_ik, :]           (O(K d) per example)
//   update:  W_in[r, :] -= lr * sum_{(i,k): u_ik = r} v_ik dA[i, :]
// touch only the rows the minibatch refers to.  The update writes each row
// once and adds its pairs in (example, pair) order (long lists in fixed parts):
// deterministic, with no atomics on W_in.  A slot is a pair's position i K + k.
//
// Up to kInputSmall slots the update is one launch, a wave per slot: every
// wave reads all the indices (8 KB at most, in flight together) and so checks
// them, and finds its row's slots and whether it is the first, without any
// table.  Larger calls are grouped first (four launches):
//   group   blocks of 256 or 1024 slots sort theirs by (row, slot); the first
//           slot of each run counts the run in an open-addressing table of the
//           rows: atomics per block and row, however often the block names it;
//   update  rows that one block names: the wave of the run sums its slots.  Rows
//           that several blocks name are listed as their second run arrives and
//           taken in turn by other waves, whose lane b looks for block b's run
//           (they are the frequent rows, next to each other in sorted order).
//           Whoever updates a row empties its table entry, so the table needs
//           no pass of its own;
//   hot     rows of kInputHotSlots slots or more: a block per kPartSlots slots of
//           the row, 64 to a wave; the sums of rows of several parts are added
//           in part order by one more launch.
// Measured at d = 512, m K = 65 536, Zipf 1.1 (the four launches): 15 + 28 + 13
// + 5 us; uniform rows at d = 500: 95 us.  A table of slots took one atomic per
// slot, 8600 of them at the most frequent row (178 us), and the owner of a
// repeated row read the later indices to find its slots (398 us), hot rows
// another 126 us; uniform rows 870 us, but 18 at 2049 slots, where this form took
// 24 with blocks of 1024 slots (now 17).  m K = 1280, d = 500: 6.6 us (a table of
// slots in four launches, 21 us).
#include <math.h>
#include <stdlib.h>

#include <algorithm>
#include <new>
#include <type_traits>

#include "lst_internal.h"

struct lst_input {
  int64_t D = 0;
  int d = 0;
  int device = 0;
  hipStream_t stream = nullptr;
  float* W = nullptr;
  int* flags = nullptr;  // [0]: sticky status
  // workspace of one large update (InputWs)
  unsigned char* ws = nullptr;
  unsigned char* sorted = nullptr;
  float* psum = nullptr;
};

namespace lst {
namespace {

// Slots (and table entries) of the row table: twice the largest number of
// slots, so that the table is at most half full.
constexpr int kInputMaxSlots = 65536;
constexpr int kInputHashBits = 17;
constexpr int kInputHashSize = 1 << kInputHashBits;
static_assert(kInputHashSize >= 2 * kInputMaxSlots, "the row table must stay half empty");
// Slots up to which the update is one launch: each wave then reads 8 KB of
// indices.  2048 slots at d = 512: uniform rows 5.7 us (17 grouped), Zipf 1.1 11.8
// (27), sixteen rows 10.4 (22).  Only where nearly all of more than 768 slots name
// one row is the grouped form faster (2048 slots: 52 and 22 us), which the host
// cannot see.
constexpr int kInputSmall = 2048;
// Slots sorted by one block: 256, 512 or 1024, the fewest that give at most a block
// per lane of a wave.  The sort is a chain of exchanges, 36, 45 or 55 stages, whose
// waves share a compute unit: 2049 slots at d = 500, the whole update, 17 us with
// blocks of 256 and 24 with 1024; 16 384 slots 31 and 40; 16 385 slots of 200 rows,
// d = 32: 21 with 512 and 23 with 1024.
constexpr int kMaxSorted = 64;  // sorted blocks
static_assert(kInputMaxSlots <= kMaxSorted * 1024, "a lane of a wave per sorted block");
// Rows of this many slots or more are not left to one wave.
constexpr int kInputHotSlots = 64;
constexpr int kPartSlots = 256;  // slots of a hot row that one block sums
constexpr int kMaxParts = kInputMaxSlots / kInputHotSlots + kInputMaxSlots / kPartSlots;
constexpr int kMaxSplit = kInputMaxSlots / kPartSlots;     // rows of several parts
constexpr int kMaxSums = 2 * kInputMaxSlots / kPartSlots;  // their parts

// The workspace of one large update, in three allocations: three pointers are what
// its launches pass (the host spends time on every byte of kernel arguments: with
// every array by itself, the update of 2049 slots at d = 500 took 17 us, 13 to 16
// so), and allocations below 2 MB are the cheap ones (one of 2.5 MB made
// lst_input_init 8 us longer).
struct InputWs {
  unsigned char* p;
  // open-addressing table of the rows (empty between calls): row in the upper,
  // number of runs in the lower 32 bits
  static constexpr size_t kTable = 0;
  // parts of the rows of at least kInputHotSlots slots: [0] = (parts, rows of
  // several parts, sums taken of psum), then (row, part, slots of the row, the
  // row's first sum in psum); and the rows of several parts
  static constexpr size_t kPart = kTable + kInputHashSize * sizeof(unsigned long long);
  static constexpr size_t kSplit = kPart + (1 + kMaxParts) * sizeof(int4);
  // the last sorted row of each 64 positions, then of each 16
  static constexpr size_t kPiv = kSplit + kMaxSplit * sizeof(int4);
  // table entries of the rows several blocks name ([0]: count)
  static constexpr size_t kMulti = kPiv + (kInputMaxSlots / 64 + kInputMaxSlots / 16) * sizeof(int);
  static constexpr size_t kBytes = kMulti + (1 + kInputMaxSlots / 2) * sizeof(int);

  unsigned char* sorted;
  // per sorted position: pair (offset of the example's row of dA, value), row,
  // length of the run that starts there (0: none does) and the run's table entry
  static constexpr size_t kPair = 0;
  static constexpr size_t kRow = kPair + kInputMaxSlots * sizeof(uint2);
  static constexpr size_t kLen = kRow + kInputMaxSlots * sizeof(int);
  static constexpr size_t kEnt = kLen + kInputMaxSlots * sizeof(int);
  static constexpr size_t kSortedBytes = kEnt + kInputMaxSlots * sizeof(int);

  float* psum;  // the sums of the rows of several parts, kMaxSums rows of d

  template <class T>
  __device__ __forceinline__ static T* at(unsigned char* base, size_t off) {
    return reinterpret_cast<T*>(base + off);
  }
  __device__ __forceinline__ unsigned long long* table() const {
    return at<unsigned long long>(p, kTable);
  }
  __device__ __forceinline__ int4* part() const { return at<int4>(p, kPart); }
  __device__ __forceinline__ int4* split() const { return at<int4>(p, kSplit); }
  __device__ __forceinline__ int* piv() const { return at<int>(p, kPiv); }
  __device__ __forceinline__ int* multi() const { return at<int>(p, kMulti); }
  __device__ __forceinline__ uint2* spair() const { return at<uint2>(sorted, kPair); }
  __device__ __forceinline__ int* srow() const { return at<int>(sorted, kRow); }
  __device__ __forceinline__ int* rlen() const { return at<int>(sorted, kLen); }
  __device__ __forceinline__ int* rent() const { return at<int>(sorted, kEnt); }
};
static_assert(InputWs::kPart % 16 == 0 && InputWs::kPiv % 16 == 0 && InputWs::kRow % 16 == 0,
              "read in pieces of 16 bytes");

__device__ __forceinline__ unsigned input_hash(int r) {
  return ((unsigned)r * 2654435761u) >> (32 - kInputHashBits);
}

// An empty table entry (no row is 0x7fffffff or above).
constexpr unsigned long long kNoEntry = ~0ull;

__global__ void input_table_init_kernel(InputWs ws) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e == 0) ws.multi()[0] = 0;
  if (e < kInputHashSize) ws.table()[e] = kNoEntry;
}

// The wave's number in its block, in a scalar register: what depends on it
// alone (an example's pairs) is then loaded once per wave.
__device__ __forceinline__ int wave_index() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Four columns of a row from col on (columns past d read as zero and are not
// written) in one access of 16 bytes, at a 4-byte address unless VEC (65 536
// uniform slots at d = 301: update 138 -> 79 us against an access a float).
typedef float floatx4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC>
__device__ __forceinline__ float4 row_load4(const float* row, int col, int d) {
  float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
  if (VEC) {
    if (col < d) w = *reinterpret_cast<const float4*>(row + col);
  } else if (col + 3 < d) {
    const floatx4_a4 v = *reinterpret_cast<const floatx4_a4*>(row + col);
    w = make_float4(v[0], v[1], v[2], v[3]);
  } else {
    if (col < d) w.x = row[col];
    if (col + 1 < d) w.y = row[col + 1];
    if (col + 2 < d) w.z = row[col + 2];
  }
  return w;
}
template <bool VEC>
__device__ __forceinline__ void row_store4(float* row, int col, int d, float4 w) {
  if (VEC) {
    if (col < d) *reinterpret_cast<float4*>(row + col) = w;
  } else if (col + 3 < d) {
    *reinterpret_cast<floatx4_a4*>(row + col) = floatx4_a4{w.x, w.y, w.z, w.w};
  } else {
    if (col < d) row[col] = w.x;
    if (col + 1 < d) row[col + 1] = w.y;
    if (col + 2 < d) row[col + 2] = w.z;
  }
}
__device__ __forceinline__ void add4(float4& a, float v, const float4& w) {
  a.x += v * w.x; a.y += v * w.y; a.z += v * w.z; a.w += v * w.w;
}

// Inputs of up to kInputSplitK pairs: a wave per (example, 256 columns), the
// example's rows all in flight together, added in pair order, its indices checked
// on the way (m = 128, K = 10, d = 500: 3.9 us; 11.0 and a 1.7 us launch for the
// check with a wave per example and two rounds of rows).  Longer inputs: below.
constexpr int kInputSplitK = 16;

template <bool VEC>
__global__ __launch_bounds__(256) void input_forward_kernel(const float* __restrict__ W,
                                                            int64_t D, int d,
                                                            const int32_t* __restrict__ idx,
                                                            const float* __restrict__ val, int m,
                                                            int K, float* __restrict__ A,
                                                            int* flags) {
  const int nch = (d + 255) / 256;
  const int w = blockIdx.x * 4 + wave_index(), lane = threadIdx.x & 63;
  if (w >= m * nch) return;
  const int i = w / nch, col = (w - i * nch) * 256 + 4 * lane;
  const int32_t* ip = idx + (size_t)i * K;
  const float* vp = val + (size_t)i * K;
  int r[kInputSplitK];
  float v[kInputSplitK];
#pragma unroll
  for (int u = 0; u < kInputSplitK; ++u) {
    r[u] = ip[min(u, K - 1)];
    v[u] = vp[min(u, K - 1)];
  }
  float4 g[kInputSplitK];
  bool bad = false;
#pragma unroll
  for (int u = 0; u < kInputSplitK; ++u) {
    // padding, a bad index and pairs past K add nothing
    const bool on = u < K && r[u] >= 0 && (int64_t)r[u] < D;
    bad |= u < K && (r[u] < -1 || (int64_t)r[u] >= D);
    if (!on) r[u] = -1;
    g[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (on) g[u] = row_load4<VEC>(W + (size_t)r[u] * d, col, d);
  }
  if (bad && lane == 0) atomicCAS(flags, 0, LST_EINDEX);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int u = 0; u < kInputSplitK; ++u)
    if (r[u] >= 0) add4(acc, v[u], g[u]);
  row_store4<VEC>(A + (size_t)i * d, col, d, acc);
}

// Pairs handled per round by the longer inputs: their loads are all issued
// before the first result is used.
constexpr int kInputBatch = 8;

// Long inputs (K > kInputSplitK): one block per (example, 256-column chunk);
// wave w sums the pairs of the w-th quarter of the example's list in order,
// and the four partial sums are added in wave order, so the result does not
// depend on timing.  Rows that repeat come from the caches, and the instructions
// for each pair are then the bound: its index and value are handed out by
// v_readlane (m = 1024, K = 20, d = 4096, sixteen rows: 19 us; 29 with scalar loads
// and branches for every pair, 24 with vector ones), and a long list's indices
// arrive 64 at a time (m = 64, K = 1024, d = 512: 33 us, 52 in batches of eight).
template <bool VEC>
__global__ __launch_bounds__(256) void input_forward_split_kernel(
    const float* __restrict__ W, int64_t D, int d, const int32_t* __restrict__ idx,
    const float* __restrict__ val, int m, int K, float* __restrict__ A, int* flags) {
  __shared__ float4 part[3][64];
  const int nch = (d + 255) / 256;
  const int i = blockIdx.x / nch, c0 = (blockIdx.x % nch) * 256;
  const int wave = wave_index(), lane = threadIdx.x & 63;
  const int col = c0 + 4 * lane;
  const int q = (K + 3) / 4, kb = wave * q, ke = min(K, kb + q);
  const int32_t* ip = idx + (size_t)i * K;
  const float* vp = val + (size_t)i * K;
  // 64 pairs at a time, one a lane, the next 64 on their way
  int rn = -1;
  float vn = 0.f;
  auto next_pairs = [&](int k) {
    rn = -1;
    if (k < ke) {
      rn = ip[k];
      vn = vp[k];
    }
  };
  next_pairs(kb + lane);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  bool bad = false;
  for (int k0 = kb; k0 < ke; k0 += 64) {
    // (D fits 31 bits) padding, a bad index and pairs past ke add nothing
    bad |= (unsigned)rn + 1u > (unsigned)D;
    const int rl = (unsigned)rn < (unsigned)D ? rn : -1;
    const float vl = vn;
    next_pairs(k0 + 64 + lane);
    for (int b = 0; b < min(64, ke - k0); b += kInputBatch) {
      int r[kInputBatch];
      float4 w[kInputBatch];
#pragma unroll
      for (int u = 0; u < kInputBatch; ++u) {
        r[u] = __builtin_amdgcn_readlane(rl, b + u);
        w[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r[u] >= 0) w[u] = row_load4<VEC>(W + (size_t)r[u] * d, col, d);
      }
#pragma unroll
      for (int u = 0; u < kInputBatch; ++u)
        if (r[u] >= 0)
          add4(acc, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vl), b + u)), w[u]);
    }
  }
  if (bad) atomicCAS(flags, 0, LST_EINDEX);
  if (wave > 0) part[wave - 1][lane] = acc;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const float4 o = part[p][lane];
    acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
  }
  row_store4<VEC>(A + (size_t)i * d, col, d, acc);
}

// ------------------------------------------------------------------- update
// Rows of dA in flight in a wave that sums a list, two 256-column chunks each.
constexpr int kListRows = 8;

// acc += sum over the list's slots t0 .. t0 + cnt - 1 (cnt <= 64; lane l holds
// slot l's value v and the offset o of its row of dA) of v dA[row], in order,
// columns cg + 256 c + 4 lane (c < 2).
template <bool VEC>
__device__ __forceinline__ void sum_list(const float* gA, int d, int cg, int cnt, float v,
                                         unsigned o, float4 (&acc)[2]) {
  const int lane = threadIdx.x & 63;
  for (int t0 = 0; t0 < cnt; t0 += kListRows) {
    float4 g[kListRows][2];
#pragma unroll
    for (int u = 0; u < kListRows; ++u) {
      // slots past the list re-read its last row
      const float* gr = gA + (unsigned)__builtin_amdgcn_readlane((int)o, min(t0 + u, cnt - 1));
#pragma unroll
      for (int c = 0; c < 2; ++c) g[u][c] = row_load4<VEC>(gr, cg + 256 * c + 4 * lane, d);
    }
#pragma unroll
    for (int u = 0; u < kListRows; ++u) {
      if (t0 + u >= cnt) break;
      const float vu = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t0 + u));
#pragma unroll
      for (int c = 0; c < 2; ++c) add4(acc[c], vu, g[u][c]);
    }
  }
}

// The sum for one column a lane (col; offset in bounds for every lane), cnt <= 64,
// all loads in flight together (a row of 2048 slots: 52 us, with 32 at a time 79).
__device__ __forceinline__ float sum_list_col(const float* gA, int col, int cnt, float v,
                                              unsigned o) {
  float g[64];
#pragma unroll
  for (int u = 0; u < 64; ++u)
    g[u] = gA[(unsigned)__builtin_amdgcn_readlane((int)o, min(u, cnt - 1)) + (unsigned)col];
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 64; ++u) {
    const float vu = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), u));
    if (u < cnt) acc += vu * g[u];
  }
  return acc;
}

// Row r -= lr (sum over the wave's list of cnt slots, lane l holding v and o).
template <bool VEC>
__device__ __forceinline__ void update_row(float* W, const float* gA, int d, int r, int cnt,
                                           float v, unsigned o, float lr) {
  const int lane = threadIdx.x & 63;
  float* row = W + (size_t)r * d;
  for (int cg = 0; cg < d; cg += 512) {
    float4 old[2], acc[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      old[c] = row_load4<VEC>(row, cg + 256 * c + 4 * lane, d);
      acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    sum_list<VEC>(gA, d, cg, cnt, v, o, acc);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      old[c].x -= lr * acc[c].x; old[c].y -= lr * acc[c].y;
      old[c].z -= lr * acc[c].z; old[c].w -= lr * acc[c].w;
      row_store4<VEC>(row, cg + 256 * c + 4 * lane, d, old[c]);
    }
  }
}

// Up to 64 NU slots, a wave per slot.  Every wave holds all the indices, so
// each finds any bad one (and then nothing is written).  The wave of a row's
// first slot updates the row; a row of kInputHotSlots slots or more is shared
// out by columns, 64 to each of its first waves (d <= 4096 = 64 x 64).
template <int NU, bool VEC>
__global__ __launch_bounds__(256) void input_update_small_kernel(
    float* __restrict__ W, int64_t D, int d, const int32_t* __restrict__ idx,
    const float* __restrict__ val, const float* __restrict__ gA, int n, int K, float lr,
    int* flags) {
  __shared__ unsigned short list[4][64 * NU];
  const int w = wave_index(), lane = threadIdx.x & 63;
  const int e = blockIdx.x * 4 + w;
  if (e >= n) return;
  int x[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) x[u] = idx[min(64 * u + lane, n - 1)];
  const int r = idx[e];
  const int pending = *flags;
  bool bad = false;
#pragma unroll
  for (int u = 0; u < NU; ++u) bad |= x[u] < -1 || (int64_t)x[u] >= D;
  if (__ballot(bad) != 0ull) {
    if (lane == 0) atomicCAS(flags, 0, LST_EINDEX);
    return;
  }
  if (r < 0 || pending != 0) return;
  int cnt = 0, first = n, before = 0;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const unsigned long long hb = __ballot(x[u] == r && 64 * u + lane < n);
    if (hb != 0ull) {
      if (x[u] == r && 64 * u + lane < n)
        list[w][cnt + __popcll(hb & ((1ull << lane) - 1ull))] = (unsigned short)(64 * u + lane);
      if (cnt == 0) first = 64 * u + __ffsll((unsigned long long)hb) - 1;
      if (e >= 64 * u + 64)
        before += __popcll(hb);
      else if (e >= 64 * u)
        before += __popcll(hb & ((1ull << (e - 64 * u)) - 1ull));
      cnt += __popcll(hb);
    }
  }
  // the list is read back by other lanes of this wave (its LDS accesses
  // complete in order)
  asm volatile("" ::: "memory");
  if (cnt < kInputHotSlots) {
    if (first != e) return;
    const int s = list[w][min(lane, cnt - 1)];
    update_row<VEC>(W, gA, d, r, cnt, val[s], (unsigned)(s / K) * (unsigned)d, lr);
    return;
  }
  if (64 * before >= d) return;
  const int col = 64 * before + lane, colc = min(col, d - 1);
  const float old = W[(size_t)r * d + colc];
  // in the order of the grouped form: 64 slots, then parts of kPartSlots, then the
  // parts
  float acc = 0.f;
  for (int p0 = 0; p0 < cnt; p0 += kPartSlots) {
    float part = 0.f;
    for (int t0 = p0; t0 < min(cnt, p0 + kPartSlots); t0 += 64) {
      const int s = list[w][min(t0 + lane, cnt - 1)];
      part += sum_list_col(gA, colc, min(64, cnt - t0), val[s], (unsigned)(s / K) * (unsigned)d);
    }
    acc += part;
  }
  if (col < d) W[(size_t)r * d + col] = old - lr * acc;
}

// The value of lane (lane ^ J).
template <int J>
__device__ __forceinline__ unsigned lane_xor(unsigned v) {
  if constexpr (J == 1) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
  } else if constexpr (J == 2) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);
  } else if constexpr (J == 4) {  // 7 - x within eight lanes, then 3 - x within four
    const int m = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);
    return (unsigned)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xf, 0xf, true);
  } else if constexpr (J == 8) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);
  } else if constexpr (J == 16) {  // [0]: the even rows twice, [1]: the odd ones
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (threadIdx.x & 16) ? p[0] : p[1];
  } else {
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (threadIdx.x & 32) ? p[0] : p[1];
  }
}

// Ascending order of one key per thread over a block of SB threads (bitonic;
// strides below 64 between lanes, by DPP and lane swaps, which do not go through
// the LDS unit as shuffles do; the others through LDS).
template <int SB, int KK, int J, int P>
__device__ __forceinline__ void sort_stages(unsigned long long& x, unsigned long long (*sh)[SB]) {
  const int t = threadIdx.x;
  unsigned long long o;
  if constexpr (J >= 64) {  // (two buffers in turn: one barrier a stage)
    sh[P][t] = x;
    __syncthreads();
    o = sh[P][t ^ J];
  } else {
    o = ((unsigned long long)lane_xor<J>((unsigned)(x >> 32)) << 32) | lane_xor<J>((unsigned)x);
  }
  const bool up = (t & KK) == 0, low = (t & J) == 0;
  x = (low == up) == (o < x) ? o : x;  // (keys are distinct)
  constexpr int Q = J >= 64 ? P ^ 1 : P;
  if constexpr (J > 1)
    sort_stages<SB, KK, J / 2, Q>(x, sh);
  else if constexpr (KK < SB)
    sort_stages<SB, 2 * KK, KK, Q>(x, sh);
}

// Block b sorts slots [SB b, +SB) by (row, slot) and counts each run in the
// table; a row is listed as its second run arrives.
template <int SB>
__global__ __launch_bounds__(SB) void input_group_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ val, int n, int K, int d, int64_t D,
    InputWs ws, int* flags) {
  __shared__ unsigned long long bufs[2][SB];
  __shared__ unsigned long long heads[SB / 64];
  __shared__ float vals[SB];
  const int t = threadIdx.x, e = blockIdx.x * SB + t;
  unsigned long long* table = ws.table();
  int *piv = ws.piv(), *multi = ws.multi();
  if (e == 0) ws.part()[0] = make_int4(0, 0, 0, 0);
  const int r = e < n ? idx[e] : -1;
  vals[t] = e < n ? val[e] : 0.f;
  if (r < -1 || (int64_t)r >= D) atomicCAS(flags, 0, LST_EINDEX);
  const bool valid = r >= 0 && (int64_t)r < D;
  const unsigned row = valid ? (unsigned)r : 0xffffffffu;  // the others last
  unsigned long long x = ((unsigned long long)row << 32) | (unsigned)e;
  sort_stages<SB, 2, 1, 0>(x, bufs);
  __syncthreads();
  unsigned long long* sh = bufs[0];
  sh[t] = x;
  __syncthreads();
  const unsigned my = (unsigned)(x >> 32);
  const int slot = (int)(unsigned)x;
  const float v = vals[slot & (SB - 1)];
  const bool head = my != 0xffffffffu && (t == 0 || (unsigned)(sh[t - 1] >> 32) != my);
  const bool end = my == 0xffffffffu;  // no run: ends the one before
  const unsigned long long stop = __ballot(head || end);
  if ((t & 63) == 0) heads[t >> 6] = stop;
  __syncthreads();
  int len = 0, ent = -1;
  if (head) {
    // up to the next head (or the end of the valid slots)
    int nx = SB;
    unsigned long long m = heads[t >> 6] & (~0ull << (t & 63)) & ~(1ull << (t & 63));
    for (int q = t >> 6; q < SB / 64; ++q) {
      if (q > (t >> 6)) m = heads[q];
      if (m != 0ull) {
        nx = 64 * q + __ffsll((unsigned long long)m) - 1;
        break;
      }
    }
    len = nx - t;
  }
  // the position's arrays are whole blocks (kInputMaxSlots is a multiple of SB)
  const int row_out = end ? 0x7fffffff : (int)my;
  ws.srow()[e] = row_out;
  ws.spair()[e] = make_uint2((unsigned)(slot / K) * (unsigned)d, __float_as_uint(v));
  ws.rlen()[e] = len;
  if ((t & 63) == 63) piv[e >> 6] = row_out;
  if ((t & 15) == 15) piv[kInputMaxSlots / 64 + (e >> 4)] = row_out;
  if (head) {
    // a new row: one atomic; a row that another block has entered: one more
    unsigned h = input_hash((int)my);
    const unsigned long long mine = ((unsigned long long)my << 32) | 1ull;
    for (int probe = 0; probe < kInputHashSize; ++probe) {
      const unsigned long long prev = atomicCAS(table + h, kNoEntry, mine);
      if (prev == kNoEntry || (unsigned)(prev >> 32) == my) {
        ent = (int)h;
        if (prev != kNoEntry && (unsigned)atomicAdd(table + h, 1ull) == 1u)
          multi[1 + atomicAdd(multi, 1)] = (int)h;
        break;
      }
      h = (h + 1) & (kInputHashSize - 1);
    }
  }
  ws.rent()[e] = ent;
}

// Block b's run of row r: its first position in q, its length returned (0:
// none).  Four dependent loads: the block's groups of 64 by their last rows, the group's four of 16, the sixteen rows, the length.
__device__ __forceinline__ int below(const int4& x, int r) {
  return (x.x < r) + (x.y < r) + (x.z < r) + (x.w < r);
}
template <int SB>
__device__ __forceinline__ int find_run(const InputWs& ws, int b, int nb, int r, int& q) {
  q = 0;
  if (b >= nb) return 0;
  constexpr int kGroups = SB / 64;
  const int* piv = ws.piv();
  const int4* p64 = reinterpret_cast<const int4*>(piv + b * kGroups);
  int grp = 0;
#pragma unroll
  for (int u = 0; u < kGroups / 4; ++u) grp += below(p64[u], r);
  if (grp == kGroups) return 0;
  grp += b * kGroups;
  const int sub =
      4 * grp + below(reinterpret_cast<const int4*>(piv + kInputMaxSlots / 64)[grp], r);
  const int4* sr = reinterpret_cast<const int4*>(ws.srow() + 16 * sub);
  int lt = 0;
  bool eq = false;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int4 x = sr[u];
    lt += below(x, r);
    eq |= x.x == r || x.y == r || x.z == r || x.w == r;
  }
  if (!eq) return 0;
  q = 16 * sub + lt;
  return ws.rlen()[q];
}

// Exclusive prefix sum over the wave (every lane takes part); total in all lanes.
__device__ __forceinline__ int wave_prefix(int v, int& total) {
  const int lane = threadIdx.x & 63;
  int s = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(s, off);
    if (lane >= off) s += o;
  }
  total = __builtin_amdgcn_readlane(s, 63);
  return s - v;
}

// Sorted positions of one wave: their runs are looked up together, one a lane.  4
// for large calls (the largest Zipf 1.1 call, update and forward pass: 81 us, 92 at
// 16, with too few waves for the rows of one slot; uniform rows 126, 155 at 1); 1 up
// to 16 384 slots, whose runs are too few to fill the chip (4096 slots in pairs, d =
// 2048: 22 us, 24 at 4; 16 384 at d = 500: 22, 21).
template <int SB>
constexpr int kRunsPerWave = SB == 256 ? 1 : 4;
// Blocks (of four waves) for the rows that several blocks name, at most (and no
// more than a wave per such row).
constexpr int kMultiBlocks = 1024;
static_assert(kInputMaxSlots / 2 <= 4 * kMultiBlocks * 64, "a lane for each of a wave's rows");

// Lists the parts of a row of total (>= kInputHotSlots) slots; every lane of
// the wave takes part.
__device__ __forceinline__ void list_parts(const InputWs& ws, int row, int total) {
  int4 *part = ws.part(), *split = ws.split();
  const int lane = threadIdx.x & 63;
  const int np = (total + kPartSlots - 1) / kPartSlots;
  int at = 0, sum = 0;
  if (lane == 0) {
    at = 1 + atomicAdd(&part->x, np);
    if (np > 1) {
      sum = atomicAdd(&part->z, np);
      split[atomicAdd(&part->y, 1)] = make_int4(row, sum, np, 0);
    }
  }
  at = __builtin_amdgcn_readlane(at, 0);
  sum = __builtin_amdgcn_readlane(sum, 0);
  for (int j = lane; j < np; j += 64) part[at + j] = make_int4(row, j, total, sum);
}

// Positions [p0, p0 + R): the runs whose row no other block names.
template <int R, bool VEC>
__device__ __forceinline__ void update_runs(float* W, const float* gA, int d, float lr, int p0,
                                            const InputWs& ws, int pending) {
  unsigned long long* table = ws.table();
  const uint2* spair = ws.spair();
  const int lane = threadIdx.x & 63;
  const int p = p0 + min(lane, R - 1);
  int len = ws.rlen()[p];
  const int r = ws.srow()[p], h = ws.rent()[p];
  const uint2 pr = spair[p];
  bool mine = false;
  if (lane < R && len > 0 && h >= 0) {
    if ((unsigned)table[h] == 1u) {
      mine = true;
      table[h] = kNoEntry;
    }
  }
  if (pending != 0) return;
  unsigned long long many = __ballot(mine && len >= kInputHotSlots);
  while (many != 0ull) {
    const int l = __ffsll((unsigned long long)many) - 1;
    many &= many - 1;
    list_parts(ws, __builtin_amdgcn_readlane(r, l), __builtin_amdgcn_readlane(len, l));
  }
  // rows of one slot, kListRows / 2 at a time
  unsigned long long todo = __ballot(mine && len == 1);
  constexpr int kS = kListRows / 2;
  while (todo != 0ull) {
    int rr[kS];
    float vv[kS];
    unsigned oo[kS];
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < kS; ++u) {
      const bool on = todo != 0ull;
      const int l = on ? __ffsll((unsigned long long)todo) - 1 : 0;
      if (on) {
        rr[u] = __builtin_amdgcn_readlane(r, l);
        vv[u] = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)pr.y, l));
        oo[u] = (unsigned)__builtin_amdgcn_readlane((int)pr.x, l);
        ++cnt;
      } else {  // the first one again (never stored)
        rr[u] = rr[0];
        vv[u] = 0.f;
        oo[u] = oo[0];
      }
      todo &= todo - 1;
    }
    for (int cg = 0; cg < d; cg += 512) {
      float4 old[kS][2], g[kS][2];
#pragma unroll
      for (int u = 0; u < kS; ++u)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int col = cg + 256 * c + 4 * lane;
          old[u][c] = row_load4<VEC>(W + (size_t)rr[u] * d, col, d);
          g[u][c] = row_load4<VEC>(gA + oo[u], col, d);
        }
#pragma unroll
      for (int u = 0; u < kS; ++u) {
        if (u >= cnt) break;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          old[u][c].x -= lr * (vv[u] * g[u][c].x); old[u][c].y -= lr * (vv[u] * g[u][c].y);
          old[u][c].z -= lr * (vv[u] * g[u][c].z); old[u][c].w -= lr * (vv[u] * g[u][c].w);
          row_store4<VEC>(W + (size_t)rr[u] * d, cg + 256 * c + 4 * lane, d, old[u][c]);
        }
      }
    }
  }
  // rows of several slots, one after another (the run's slots are in order)
  unsigned long long more = __ballot(mine && len > 1 && len < kInputHotSlots);
  while (more != 0ull) {
    const int l = __ffsll((unsigned long long)more) - 1;
    more &= more - 1;
    const int cnt = __builtin_amdgcn_readlane(len, l);
    const uint2 x = spair[p0 + l + min(lane, cnt - 1)];
    update_row<VEC>(W, gA, d, __builtin_amdgcn_readlane(r, l), cnt, __uint_as_float(x.y), x.x, lr);
  }
}

template <int SB, bool VEC>
__global__ __launch_bounds__(256) void input_update_kernel(float* __restrict__ W, int d,
                                                           const float* __restrict__ gA, int n,
                                                           float lr, InputWs ws, const int* flags,
                                                           int multi_blocks) {
  __shared__ uint2 list[4][kInputHotSlots];
  const int w = wave_index(), lane = threadIdx.x & 63;
  const int nb = (n + SB - 1) / SB;
  const int pending = *flags;
  if ((int)blockIdx.x >= multi_blocks) {
    const int p0 = (((int)blockIdx.x - multi_blocks) * 4 + w) * kRunsPerWave<SB>;
    if (p0 >= nb * SB) return;
    update_runs<kRunsPerWave<SB>, VEC>(W, gA, d, lr, p0, ws, pending);
    return;
  }
  // The listed rows wv, wv + nw, ...: one a lane, then one after another.
  const int wv = (int)blockIdx.x * 4 + w, nw = 4 * multi_blocks;
  unsigned long long* table = ws.table();
  const uint2* spair = ws.spair();
  const int* multi = ws.multi();
  const int count = multi[0];
  const int at = wv + nw * lane;
  int row = -1;
  if (at < count) {
    const int h = multi[1 + at];
    row = (int)(table[h] >> 32);
    table[h] = kNoEntry;
  }
  if (pending != 0) return;
  for (int l = 0; wv + nw * l < count; ++l) {
    const int r = __builtin_amdgcn_readlane(row, l);
    int q, total;
    const int mine = find_run<SB>(ws, lane, nb, r, q);
    const int off = wave_prefix(mine, total);
    if (total >= kInputHotSlots) {
      list_parts(ws, r, total);
      continue;
    }
    for (int u = 0; u < mine; ++u) list[w][off + u] = spair[q + u];
    // the list is read back by other lanes of this wave (its LDS accesses
    // complete in order)
    asm volatile("" ::: "memory");
    const uint2 x = list[w][min(lane, total - 1)];
    update_row<VEC>(W, gA, d, r, total, __uint_as_float(x.y), x.x, lr);
    asm volatile("" ::: "memory");
  }
}

// Blocks of the hot rows' launches; they take the parts (the rows) in turn.
constexpr int kHotBlocks = 1024;
// Parts times 64-column chunks up to which the parts are taken chunk by chunk: what
// the blocks take in one turn.  At d = 500, 64 parts (16 384 slots on one row): 26
// us for the update, 36 with 512 columns a block; 157 parts (40 000 slots): 44, 39.
constexpr int kHotNarrow = kHotBlocks;

// One part: kPartSlots slots of a hot row, in order, 64 to each wave; the four
// sums are added in wave order.  The row itself is updated if this is all of it.
// A block takes 512 columns of it, eight rows of dA in flight, or, when the parts
// are too few to fill the chip so, 64 columns with all of a wave's 64 rows in
// flight: the same sums.  (2049 slots on 16 rows, the whole update: 18 us at d =
// 2048, 48 when a block took all columns of a part; d = 500: 18, 23.)
template <int SB, bool VEC>
__global__ __launch_bounds__(256) void input_hot_kernel(float* __restrict__ W, int d,
                                                        const float* __restrict__ gA, int n,
                                                        float lr, InputWs ws, const int* flags) {
  __shared__ float4 sums[3][2][64];
  __shared__ float sums1[3][64];
  __shared__ int s_off[64], s_q[64];
  const int nb = (n + SB - 1) / SB;
  const int w = wave_index(), lane = threadIdx.x & 63;
  const int4* part = ws.part();
  const uint2* spair = ws.spair();
  if (blockIdx.x == 0 && threadIdx.x == 0) ws.multi()[0] = 0;  // its rows are done
  const int count = *flags != 0 ? 0 : part[0].x;
  const bool narrow = count * ((d + 63) / 64) <= kHotNarrow;
  const int cw = narrow ? 64 : 512, nch = (d + cw - 1) / cw;
  for (int b = blockIdx.x; b < count * nch; b += gridDim.x) {
    const int4 pt = part[1 + b / nch];
    const int cg = b % nch * cw;
    const int r = __builtin_amdgcn_readfirstlane(pt.x), j = __builtin_amdgcn_readfirstlane(pt.y),
              total = __builtin_amdgcn_readfirstlane(pt.z),
              sum0 = __builtin_amdgcn_readfirstlane(pt.w);
    if (w == 0) {
      int q, all;
      const int mine = find_run<SB>(ws, lane, nb, r, q);
      s_off[lane] = wave_prefix(mine, all);
      s_q[lane] = q;
    }
    const bool whole = total <= kPartSlots;
    float* out = whole ? W + (size_t)r * d : ws.psum + (size_t)(sum0 + j) * d;
    const int col = cg + lane, colc = min(col, d - 1);  // narrow
    float old1 = 0.f;
    float4 old[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      old[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (!narrow && w == 0 && whole) old[c] = row_load4<VEC>(out, cg + 256 * c + 4 * lane, d);
    }
    if (narrow && w == 0 && whole) old1 = out[colc];
    __syncthreads();
    const int tb = j * kPartSlots + 64 * w, te = min(total, tb + 64);
    uint2 x = make_uint2(0u, 0u);
    if (tb < te) {
      const int t = min(tb + lane, te - 1);
      int lo = 0;  // the last block whose first slot is not after t
#pragma unroll
      for (int s = 32; s > 0; s >>= 1)
        if (s_off[lo + s] <= t) lo += s;
      x = spair[s_q[lo] + t - s_off[lo]];
    }
    if (narrow) {
      float acc = 0.f;
      if (tb < te) acc = sum_list_col(gA, colc, te - tb, __uint_as_float(x.y), x.x);
      if (w > 0) sums1[w - 1][lane] = acc;
      __syncthreads();
      if (w == 0) {
#pragma unroll
        for (int v = 0; v < 3; ++v) acc += sums1[v][lane];
        if (col < d) out[col] = whole ? old1 - lr * acc : acc;
      }
    } else {
      float4 acc[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (tb < te) sum_list<VEC>(gA, d, cg, te - tb, __uint_as_float(x.y), x.x, acc);
      if (w > 0) {
        sums[w - 1][0][lane] = acc[0];
        sums[w - 1][1][lane] = acc[1];
      }
      __syncthreads();
      if (w == 0) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
          for (int v = 0; v < 3; ++v) {
            const float4 o = sums[v][c][lane];
            acc[c].x += o.x; acc[c].y += o.y; acc[c].z += o.z; acc[c].w += o.w;
          }
          if (whole) {
            acc[c].x = old[c].x - lr * acc[c].x; acc[c].y = old[c].y - lr * acc[c].y;
            acc[c].z = old[c].z - lr * acc[c].z; acc[c].w = old[c].w - lr * acc[c].w;
          }
          row_store4<VEC>(out, cg + 256 * c + 4 * lane, d, acc[c]);
        }
      }
    }
    __syncthreads();
  }
}

// Rows of several parts: a wave per (row, 64 columns) adds the parts' sums in
// order, sixteen in flight, and updates the row.
__global__ __launch_bounds__(256) void input_split_kernel(float* __restrict__ W, int d, float lr,
                                                          InputWs ws, const int* flags) {
  const int nch = (d + 63) / 64;
  const int w = wave_index(), lane = threadIdx.x & 63;
  const int count = *flags != 0 ? 0 : ws.part()[0].y;
  for (int b = (int)blockIdx.x * 4 + w; b < count * nch; b += 4 * gridDim.x) {
    const int4 sp = ws.split()[b / nch];
    const int col = (b % nch) * 64 + lane, colc = min(col, d - 1), np = sp.z;
    float* out = W + (size_t)sp.x * d + colc;
    const float old = *out;
    const float* ps = ws.psum + (size_t)sp.y * d + colc;
    float acc = 0.f;
    for (int j0 = 0; j0 < np; j0 += 16) {
      float g[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) g[u] = ps[(size_t)min(j0 + u, np - 1) * d];
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += j0 + u < np ? g[u] : 0.f;
    }
    if (col < d) *out = old - lr * acc;
  }
}

int check_batch(lst_input* s, int32_t m, int32_t K, const int32_t* idx, const float* val) {
  if (!s || m < 1 || K < 1 || !idx || !val) return LST_EINVAL;
  if ((int64_t)m * K > kInputMaxSlots) return LST_EINVAL;
  return LST_OK;
}

struct DeviceScope {
  int prev = -1;
  explicit DeviceScope(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) (void)hipSetDevice(dev);
  }
  ~DeviceScope() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

}  // namespace
}  // namespace lst

using namespace lst;

extern "C" {

int lst_input_init(lst_input** out, int64_t D_in, int32_t d, const float* W_in,
                   void* hip_stream) {
  if (!out || !W_in || D_in < 1 || d < 1 || d > 4096 || D_in > (int64_t)0x7fffffff)
    return LST_EINVAL;
  lst_input* s = new (std::nothrow) lst_input();
  if (!s) return LST_ENOMEM;
  s->D = D_in;
  s->d = d;
  s->stream = static_cast<hipStream_t>(hip_stream);
  auto fail = [&](int code) {
    (void)hipStreamSynchronize(s->stream);
    for (void* p : {(void*)s->W, (void*)s->flags, (void*)s->ws, (void*)s->sorted,
                    (void*)s->psum})
      if (p) (void)hipFree(p);
    delete s;
    return code;
  };
  if (hipGetDevice(&s->device) != hipSuccess) return fail(LST_EHIP);
  if (hipMalloc((void**)&s->W, (size_t)D_in * d * sizeof(float)) != hipSuccess ||
      hipMalloc((void**)&s->flags, sizeof(int)) != hipSuccess ||
      hipMalloc((void**)&s->ws, InputWs::kBytes) != hipSuccess ||
      hipMalloc((void**)&s->sorted, InputWs::kSortedBytes) != hipSuccess ||
      hipMalloc((void**)&s->psum, (size_t)kMaxSums * d * sizeof(float)) != hipSuccess)
    return fail(LST_ENOMEM);
  hipLaunchKernelGGL(input_table_init_kernel, dim3(kInputHashSize / 256), dim3(256), 0, s->stream,
                     InputWs{s->ws, s->sorted, s->psum});
  if (hipMemsetAsync(s->flags, 0, sizeof(int), s->stream) != hipSuccess ||
      hipMemcpyAsync(s->W, W_in, (size_t)D_in * d * sizeof(float), hipMemcpyDeviceToDevice,
                     s->stream) != hipSuccess ||
      hipStreamSynchronize(s->stream) != hipSuccess)
    return fail(LST_EHIP);
  *out = s;
  return LST_OK;
}

int lst_input_forward(lst_input* s, int32_t m, int32_t K, const int32_t* idx, const float* val,
                      float* A) {
  int rc = check_batch(s, m, K, idx, val);
  if (rc != LST_OK) return rc;
  if (!A) return LST_EINVAL;
  DeviceScope g(s->device);
  const int nch = (s->d + 255) / 256;
  const bool vec = (s->d % 4 == 0) && (((uintptr_t)A & 15) == 0);
  if (K > kInputSplitK) {
    const dim3 grid((unsigned)(m * nch));
    if (vec)
      hipLaunchKernelGGL(input_forward_split_kernel<true>, grid, dim3(256), 0, s->stream, s->W,
                         s->D, s->d, idx, val, m, K, A, s->flags);
    else
      hipLaunchKernelGGL(input_forward_split_kernel<false>, grid, dim3(256), 0, s->stream, s->W,
                         s->D, s->d, idx, val, m, K, A, s->flags);
  } else {
    const dim3 grid((unsigned)((m * nch + 3) / 4));
    if (vec)
      hipLaunchKernelGGL(input_forward_kernel<true>, grid, dim3(256), 0, s->stream, s->W, s->D,
                         s->d, idx, val, m, K, A, s->flags);
    else
      hipLaunchKernelGGL(input_forward_kernel<false>, grid, dim3(256), 0, s->stream, s->W, s->D,
                         s->d, idx, val, m, K, A, s->flags);
  }
  return hipGetLastError() == hipSuccess ? LST_OK : LST_EHIP;
}

int lst_input_update(lst_input* s, int32_t m, int32_t K, const int32_t* idx, const float* val,
                     const float* grad_A, float lr) {
  int rc = check_batch(s, m, K, idx, val);
  if (rc != LST_OK) return rc;
  if (!grad_A || !(lr > 0.f) || !isfinite(lr)) return LST_EINVAL;
  DeviceScope g(s->device);
  const int n = m * K;
  const bool vec = (s->d % 4 == 0) && (((uintptr_t)grad_A & 15) == 0);
  if (n <= kInputSmall) {
    const dim3 grid((unsigned)((n + 3) / 4));
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s->stream, s->W, s->D, s->d, idx, val, grad_A,
                         n, K, lr, s->flags);
    };
    if (n <= 64 * 4)
      vec ? run(input_update_small_kernel<4, true>) : run(input_update_small_kernel<4, false>);
    else
      vec ? run(input_update_small_kernel<kInputSmall / 64, true>)
          : run(input_update_small_kernel<kInputSmall / 64, false>);
    return hipGetLastError() == hipSuccess ? LST_OK : LST_EHIP;
  }
  const int parts = n / kInputHotSlots + n / kPartSlots;  // at most
  const InputWs ws{s->ws, s->sorted, s->psum};
  auto grouped = [&](auto block, auto vec16) {
    constexpr int SB = decltype(block)::value;
    constexpr bool VEC = decltype(vec16)::value;
    const int nb = (n + SB - 1) / SB;
    hipLaunchKernelGGL(input_group_kernel<SB>, dim3(nb), dim3(SB), 0, s->stream, idx, val, n, K,
                       s->d, s->D, ws, s->flags);
    const int multi_blocks = std::min(kMultiBlocks, (n / 2 + 3) / 4);
    hipLaunchKernelGGL((input_update_kernel<SB, VEC>),
                       dim3((unsigned)(multi_blocks + nb * SB / (4 * kRunsPerWave<SB>))),
                       dim3(256), 0, s->stream, s->W, s->d, grad_A, n, lr, ws, s->flags,
                       multi_blocks);
    hipLaunchKernelGGL((input_hot_kernel<SB, VEC>),
                       dim3((unsigned)std::min(parts * ((s->d + 63) / 64), kHotBlocks)), dim3(256),
                       0, s->stream, s->W, s->d, grad_A, n, lr, ws, s->flags);
  };
  auto blocks_of = [&](auto block) {
    vec ? grouped(block, std::true_type{}) : grouped(block, std::false_type{});
  };
  if (n <= 256 * kMaxSorted) blocks_of(std::integral_constant<int, 256>{});
  else if (n <= 512 * kMaxSorted) blocks_of(std::integral_constant<int, 512>{});
  else blocks_of(std::integral_constant<int, 1024>{});
  const int most = (n / kPartSlots) * ((s->d + 63) / 64);
  hipLaunchKernelGGL(input_split_kernel, dim3((unsigned)std::min((most + 3) / 4, kHotBlocks)),
                     dim3(256), 0, s->stream, s->W, s->d, lr, ws, s->flags);
  return hipGetLastError() == hipSuccess ? LST_OK : LST_EHIP;
}

int lst_input_get_W(lst_input* s, float* W) {
  if (!s || !W) return LST_EINVAL;
  DeviceScope g(s->device);
  return hipMemcpyAsync(W, s->W, (size_t)s->D * s->d * sizeof(float), hipMemcpyDeviceToDevice,
                        s->stream) == hipSuccess
             ? LST_OK
             : LST_EHIP;
}

int lst_input_sync(lst_input* s) {
  if (!s) return LST_EINVAL;
  DeviceScope g(s->device);
  int err = 0;
  if (hipStreamSynchronize(s->stream) != hipSuccess ||
      hipMemcpy(&err, s->flags, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
    return LST_EHIP;
  if (err) {
    const int zero = 0;
    if (hipMemcpy(s->flags, &zero, sizeof(int), hipMemcpyHostToDevice) != hipSuccess)
      return LST_EHIP;
  }
  return err;
}

void lst_input_free(lst_input* s) {
  if (!s) return;
  DeviceScope g(s->device);
  (void)hipStreamSynchronize(s->stream);
  for (void* p : {(void*)s->W, (void*)s->flags, (void*)s->ws, (void*)s->sorted,
                  (void*)s->psum})
    (void)hipFree(p);
  delete s;
}

}  // extern "C"
