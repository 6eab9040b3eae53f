// MFMA GEMM for gfx950 with fused epilogues, used where the decoder's work is a
// dense contraction: prompt prefill (M = prompt rows) and lockstep multi-stream
// decode (M = streams).  C[M, N] = A[M, K] * W[N, K]^T with fp32 accumulation.
//
// Operands are of type TM: _Float16 for bf16 models (the bf16 weights are
// repacked at load time to fp16 times a power-of-two scale, exact for this
// weight range, and activations are rounded to fp16 once), float for fp32
// models (v_mfma_f32_16x16x4_f32).  The finished tile is staged in LDS so the
// epilogue can use any column pairing (rotary pairs i / i + 32 of a head,
// gate / up columns) without shuffles.
#include "hh_kernels.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

namespace hh {

enum class GemmKind { QKV = 0, Resid = 1, GateUp = 2, Logits = 3 };

typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- epilogues
//
// The GEMM works on logical columns n; epi.b_row(n) names the weight row of
// column n (-1: none).  A tile covers logical columns [n0, n0 + BN) and the
// epilogue receives the finished fp32 tile Cs[BM][ldc] in LDS.

// Columns = rows of [Wq; Wk; Wv]; a tile holds whole heads (BN % 64 == 0).
// Rotates query heads into q (and qM), key heads into the KV page slot of
// each row; copies value heads.
template <typename TKV>
struct EpiQKV {
  int hq, hkv;
  float scale;
  const int* row_stream;
  const int* row_pos;
  const float2* rope;
  float* q;
  TKV* qM;  // nullptr, or rotated queries again in the MFMA operand type
  TKV* kv;
  KvLayout L;
  int layer;
  const int* page_table;
  __device__ int b_row(int n) const { return n < (hq + 2 * hkv) * 64 ? n : -1; }
  // Rotary pair (i, i + 32) of head `head` in row `row`, unscaled.
  __device__ void head_pair(int row, int head, int i, float y0, float y1) const {
    const int p = row_pos[row];
    head_pair_at(row, head, i, y0, y1, p, page_table[(size_t)row_stream[row] * L.max_pages + p / kPage]);
  }
  // The same with the row's position p and the KV page holding it given.
  __device__ void head_pair_at(int row, int head, int i, float y0, float y1, int p, int page) const {
    head_pair_cs(row, head, i, y0, y1, p, page, head < hq + hkv ? rope[(size_t)p * 32 + i] : make_float2(1.f, 0.f));
  }
  // ... and with the rotation's (cos, sin) at (p, i) given.
  __device__ void head_pair_cs(int row, int head, int i, float y0, float y1, int p, int page, float2 cs) const {
    y0 *= scale;
    y1 *= scale;
    if (head < hq + hkv) {
      const float r0 = y0 * cs.x - y1 * cs.y, r1 = y1 * cs.x + y0 * cs.y;
      if (head < hq) {
        if (q) {
          q[((size_t)row * hq + head) * 64 + i] = r0;
          q[((size_t)row * hq + head) * 64 + i + 32] = r1;
        }
        if (qM) {
          qM[((size_t)row * hq + head) * 64 + i] = (TKV)r0;
          qM[((size_t)row * hq + head) * 64 + i + 32] = (TKV)r1;
        }
      } else {
        TKV* dst = kv + L.head_tile(layer, page, 0, head - hq) + (p % kPage) * 64;
        dst[i] = (TKV)r0;
        dst[i + 32] = (TKV)r1;
      }
    } else {
      TKV* dst = kv + L.head_tile(layer, page, 1, head - hq - hkv) + (p % kPage) * 64;
      dst[i] = (TKV)y0;
      dst[i + 32] = (TKV)y1;
    }
  }
  // Register epilogue of the tile kernel (see k_gemm_tile): the lane's rows
  // row0 + 16 i < M, columns cb + 8 h .. + 8 and the same + 32 of the group of
  // 64 at cb (one head, its kind the same for the whole wave).  A row's
  // lookups are loaded before the previous row's stores: the stores may alias
  // the tables as far as the compiler can tell, and would serialise one round
  // trip per row.
  template <int FM>
  __device__ void tile(int row0, int cb, int h, int M, const f32x4 (&acc)[FM][4]) const {
    const int head = cb / 64;
    if (head >= hq + 2 * hkv) return;
    const bool isq = head < hq, isk = !isq && head < hq + hkv;
    const int kvh = isq ? 0 : isk ? head - hq : head - hq - hkv;
    int p[FM], pg[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) p[i] = row_pos[min(row0 + 16 * i, M - 1)];
    if (!isq) {
#pragma unroll
      for (int i = 0; i < FM; ++i) pg[i] = row_stream[min(row0 + 16 * i, M - 1)];
#pragma unroll
      for (int i = 0; i < FM; ++i) pg[i] = page_table[(size_t)pg[i] * L.max_pages + p[i] / kPage];
    }
    f32x4 cs[2][4];  // (cos, sin) of pairs 8 h .. + 8
    auto look = [&](f32x4* c, int pos) {
      const f32x4* src = reinterpret_cast<const f32x4*>(rope + (size_t)pos * 32 + 8 * h);
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = src[e];
    };
    if (isq || isk) look(cs[0], p[0]);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if (i + 1 < FM && (isq || isk)) look(cs[(i + 1) & 1], p[i + 1]);
      f32x4 lo[2], hi[2];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float y0 = acc[i][e >> 2][e & 3] * scale, y1 = acc[i][2 + (e >> 2)][e & 3] * scale;
        if (isq || isk) {
          const float c = cs[i & 1][e >> 1][2 * (e & 1)], sn = cs[i & 1][e >> 1][2 * (e & 1) + 1];
          const float r0 = y0 * c - y1 * sn, r1 = y1 * c + y0 * sn;
          y0 = r0;
          y1 = r1;
        }
        lo[e >> 2][e & 3] = y0;
        hi[e >> 2][e & 3] = y1;
      }
      const int row = row0 + 16 * i;
      // (Every loaded value is used before the branch: one left pending on the
      // path around it would be waited for in every step of the main loop.)
      const size_t ko = isq ? 0 : L.head_tile(layer, pg[i], isk ? 0 : 1, kvh) + (p[i] % kPage) * 64 + 8 * h;
      asm volatile("" ::"v"(ko), "v"(lo[0]), "v"(lo[1]), "v"(hi[0]), "v"(hi[1]));
      if (row >= M) continue;
      auto store = [&](TKV* dst) {
        if constexpr (sizeof(TKV) == 2) {
          f16x8 a, b;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            a[e] = (_Float16)lo[e >> 2][e & 3];
            b[e] = (_Float16)hi[e >> 2][e & 3];
          }
          *reinterpret_cast<f16x8*>(dst) = a;
          *reinterpret_cast<f16x8*>(dst + 32) = b;
        }
      };
      if (isq) {
        const size_t o = ((size_t)row * hq + head) * 64 + 8 * h;
        if (q) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            *reinterpret_cast<f32x4*>(q + o + 4 * e) = lo[e];
            *reinterpret_cast<f32x4*>(q + o + 32 + 4 * e) = hi[e];
          }
        }
        if (qM) store(qM + o);
      } else {
        store(kv + ko);
      }
    }
  }
  __device__ void operator()(const float* Cs, int ldc, int m0, int M, int n0, int BM, int BN) const {
    // Each row's position and KV page are looked up once per tile and kept
    // in the row's padding of the tile (ldc >= BN + 2): the element loop
    // then has no chain of dependent global loads per element.
    int* info = const_cast<int*>(reinterpret_cast<const int*>(Cs));
    for (int r = threadIdx.x; r < BM; r += blockDim.x) {
      const int row = m0 + r;
      if (row < M) {
        const int p = row_pos[row];
        info[r * ldc + BN] = p;
        info[r * ldc + BN + 1] = page_table[(size_t)row_stream[row] * L.max_pages + p / kPage];
      }
    }
    __syncthreads();
    // U pairs per thread at a time: their rotations are loaded before any
    // of their stores.
    constexpr int U = 8;
    const int nh = BN / 64, total = BM * 32 * nh;
    for (int base = threadIdx.x; base < total; base += U * (int)blockDim.x) {
      float2 cs[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int idx = base + u * (int)blockDim.x;
        const int r = idx / (32 * nh), head = n0 / 64 + (idx / 32) % nh;
        cs[u] = make_float2(1.f, 0.f);
        if (idx < total && m0 + r < M && head < hq + hkv) cs[u] = rope[(size_t)info[r * ldc + BN] * 32 + (idx & 31)];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int idx = base + u * (int)blockDim.x;
        const int r = idx / (32 * nh), hh = (idx / 32) % nh, i = idx & 31, row = m0 + r;
        const int head = n0 / 64 + hh;
        if (idx >= total || row >= M || head >= hq + 2 * hkv) continue;
        head_pair_cs(row, head, i, Cs[r * ldc + hh * 64 + i], Cs[r * ldc + hh * 64 + i + 32], info[r * ldc + BN],
                     info[r * ldc + BN + 1], cs[u]);
      }
    }
  }
};

// x[row, col] += C (residual add of the O and down projections).
struct EpiResid {
  int N;
  float scale;
  float* x;
  __device__ int b_row(int n) const { return n < N ? n : -1; }
  // The next row's x is loaded before this row's stores.  N % 64 == 0.
  template <int FM>
  __device__ void tile(int row0, int cb, int h, int M, const f32x4 (&acc)[FM][4]) const {
    if (cb >= N) return;
    f32x4 v[2][4];
    auto at = [&](int i, int j) {
      return reinterpret_cast<f32x4*>(x + (size_t)min(row0 + 16 * i, M - 1) * N + cb + 32 * (j >> 1) + 8 * h + 4 * (j & 1));
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) v[0][j] = *at(0, j);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if (i + 1 < FM) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[(i + 1) & 1][j] = *at(i + 1, j);
      }
      // The sums before the branch: a load left pending on a path around its
      // use would be waited for in every step of the main loop.
      f32x4 t[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[j][e] = v[i & 1][j][e] + acc[i][j][e] * scale;
      asm volatile("" ::"v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]));
      if (row0 + 16 * i < M) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *at(i, j) = t[j];
      }
    }
  }
  __device__ void operator()(const float* Cs, int ldc, int m0, int M, int n0, int BM, int BN) const {
    for (int idx = threadIdx.x; idx < BM * BN; idx += blockDim.x) {
      const int r = idx / BN, c = idx % BN, row = m0 + r, col = n0 + c;
      if (row < M && col < N) x[(size_t)row * N + col] += Cs[r * ldc + c] * scale;
    }
  }
};

// Logical columns come in groups of 2 * half: gate columns j = group * half + c
// (c < half), then the matching up columns (rows F + j of [Wg; Wu]);
// m[row, j] = silu(gate) * up.
template <typename TM>
struct EpiGateUp {
  int F, half;
  float scale;
  TM* m;
  __device__ int b_row(int n) const {
    const int c = n % (2 * half), j = (n / (2 * half)) * half + (c < half ? c : c - half);
    return j < F ? (c < half ? j : F + j) : -1;
  }
  // Register epilogue (half == 32): gate columns cb + 8 h .. + 8, their up
  // columns 32 later.
  template <int FM>
  __device__ void tile(int row0, int cb, int h, int M, const f32x4 (&acc)[FM][4]) const {
    const int col = (cb / 64) * 32 + 8 * h;
    if (col >= F) return;  // F % 8 == 0
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      f16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float gt = acc[i][e >> 2][e & 3] * scale;
        o[e] = (_Float16)(silu_rcp(gt) * (acc[i][2 + (e >> 2)][e & 3] * scale));
      }
      const int row = row0 + 16 * i;
      if (row < M) *reinterpret_cast<f16x8*>(m + (size_t)row * F + col) = o;
    }
  }
  __device__ void operator()(const float* Cs, int ldc, int m0, int M, int n0, int BM, int BN) const {
    const int j0 = (n0 / (2 * half)) * half, nc = BN / 2;
    for (int idx = threadIdx.x; idx < BM * nc; idx += blockDim.x) {
      const int r = idx / nc, c = idx % nc, row = m0 + r, col = j0 + c;
      if (row >= M || col >= F) continue;
      const int cg = (c / half) * 2 * half + c % half;  // gate column in the tile; up is half later
      const float g = Cs[r * ldc + cg] * scale, u = Cs[r * ldc + cg + half] * scale;
      m[(size_t)row * F + col] = (TM)(silu(g) * u);
    }
  }
};

// s += a, and what the addition rounds off goes to rest (exactly where |s| is
// the larger, else to the rounding of the difference).
__device__ __forceinline__ void add_rest(f32x4& s, const f32x4& a, f32x4& rest) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float t = s[e] + a[e];
    rest[e] += a[e] - (t - s[e]);
    s[e] = t;
  }
}

// LM head rows: optional fp32 logits, and the packed argmax of row slot_row (-1:
// of every row) into the row's stream slot.  PAIR (tile kernel only): blocks
// of 32 rows of A hold 16 rows' fp16 high parts and then their low parts,
// scaled per row (k_norm_rows): the two products are added and scaled back.
// Each K step's high products are added up apart from the running sum
// (kPairSums, add_rest): 2,048 products in one chain of MFMA accumulations have
// twice the error of the one-row head's 64 chains.
template <bool PAIR>
struct EpiLogits {
  int V;
  float scale;
  float* logits;
  unsigned long long* slot;
  const int* row_stream;
  int slot_row;
  const float* row_scale;  // PAIR: one factor per logical row
  int rows;                // PAIR: logical rows
  __device__ int b_row(int n) const { return n < V ? n : -1; }
  template <int FM>
  __device__ void tile(int row0, int cb, int h, int M, const f32x4 (&acc)[FM][4]) const {
    constexpr int STEP = PAIR ? 2 : 1;
    const int l15 = threadIdx.x & 15;
    const int nrows = PAIR ? rows : M;
    const bool vec = V % 4 == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0;
#pragma unroll
    for (int i = 0; i < FM; i += STEP) {
      // Every wave's block starts at a multiple of 32 rows of A.
      const int row = PAIR ? ((row0 - l15) >> 1) + 8 * i + l15 : row0 + 16 * i;
      const bool in = row < nrows;
      const float f = PAIR ? scale * row_scale[in ? row : 0] : scale;
      unsigned long long best = 0ull;
      const bool keyed = slot && (slot_row < 0 || row == slot_row) && in;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = cb + 32 * (j >> 1) + 8 * h + 4 * (j & 1);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (PAIR ? acc[i][j][e] + acc[i + STEP - 1][j][e] : acc[i][j][e]) * f;
        if (logits && in) {
          float* dst = logits + (size_t)row * V + col;
          if (vec) {
            if (col < V) *reinterpret_cast<f32x4*>(dst) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < V) dst[e] = v[e];
          }
        }
        if (keyed) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const unsigned long long k = argmax_key(v[e], (uint32_t)(col + e));
            if (col + e < V && k > best) best = k;
          }
        }
      }
      if (keyed) {
        // The four lanes of a row are all in here together.
        unsigned long long o = __shfl_xor(best, 16);
        best = o > best ? o : best;
        o = __shfl_xor(best, 32);
        best = o > best ? o : best;
        if (h == 0) atomicMax(slot + row_stream[row], best);
      }
    }
  }
  // One 32 x 64 block of a workgroup of 512 threads that walks column blocks:
  // thread t takes four columns of row t / 16 and keeps the best key it has
  // seen; finish() gives each row's to its slot, one atomic per workgroup
  // and row (2,004 blocks' atomics on the same few words were half of the
  // 4-bit head's time at 6 rows).
  __device__ void block(const float* Cs, int ldc, int M, int n0, unsigned long long& best) const {
    const int row = threadIdx.x >> 4, col = n0 + 4 * (threadIdx.x & 15);
    if (row >= M) return;
    const f32x4 c = *reinterpret_cast<const f32x4*>(Cs + row * ldc + col - n0);
    float* dst = logits ? logits + (size_t)row * V + col : nullptr;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (col + e >= V) continue;
      const float v = c[e] * scale;
      if (dst) dst[e] = v;
      const unsigned long long k = argmax_key(v, (uint32_t)(col + e));
      best = k > best ? k : best;
    }
  }
  __device__ void finish(int M, unsigned long long best) const {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      const unsigned long long k = __shfl_xor(best, o);
      best = k > best ? k : best;
    }
    const int row = threadIdx.x >> 4;
    if (slot && (threadIdx.x & 15) == 0 && row < M && (slot_row < 0 || row == slot_row))
      atomicMax(slot + row_stream[row], best);
  }
  __device__ void operator()(const float* Cs, int ldc, int m0, int M, int n0, int BM, int BN) const {
    if (logits)
      for (int idx = threadIdx.x; idx < BM * BN; idx += blockDim.x) {
        const int r = idx / BN, c = idx % BN, row = m0 + r, col = n0 + c;
        if (row < M && col < V) logits[(size_t)row * V + col] = Cs[r * ldc + c] * scale;
      }
    if (slot && (int)threadIdx.x < BM && m0 + (int)threadIdx.x < M &&
        (slot_row < 0 || m0 + (int)threadIdx.x == slot_row)) {
      const int r = threadIdx.x;
      unsigned long long best = 0ull;
      for (int c = 0; c < BN && n0 + c < V; ++c) {
        const unsigned long long k = argmax_key(Cs[r * ldc + c] * scale, (uint32_t)(n0 + c));
        best = k > best ? k : best;
      }
      atomicMax(slot + row_stream[m0 + r], best);
    }
  }
};
template <class Epi>
constexpr bool kPairSums = false;
template <>
constexpr bool kPairSums<EpiLogits<true>> = true;

// ---------------------------------------------------------------- generic kernel (64 x 64)

// Any operand type and any K % 8 == 0 (fp32 models, odd shapes): 64x64 tile,
// four waves of 32x32 as 16x16 MFMA fragments, K in steps of 32 through LDS.
constexpr int GBM = 64, GBN = 64, GBK = 32;
constexpr int GLDC = GBN + 4;

// SUMS (fp32 operands): products of 16 k at a time are added to sums that keep
// their roundings apart, for rows whose sums must be as good as those of the
// one-row head (64 chains a row).
template <typename TM, typename Epi, bool SUMS = false>
__global__ __launch_bounds__(256) void k_gemm(const TM* __restrict__ A, int M, const TM* __restrict__ W, int K,
                                              Epi epi) {
  constexpr int V = Vec16<TM>::n;  // elements per 16-byte chunk
  constexpr int CPR = GBK / V;     // chunks per tile row
  constexpr int LDK = GBK + V;     // padded LDS row (elements)
  __shared__ __attribute__((aligned(16))) TM As[GBM * LDK];
  __shared__ __attribute__((aligned(16))) TM Bs[GBN * LDK];
  __shared__ float Cs[GBM * GLDC];
  const int n0 = blockIdx.x * GBN, m0 = blockIdx.y * GBM;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int wm = wv >> 1, wn = wv & 1;
  const int lr = lane & 15, lk = lane >> 4;
  f32x4 acc[2][2], sum[SUMS ? 2 : 1][2], rest[SUMS ? 2 : 1][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (SUMS) sum[i][j] = rest[i][j] = acc[i][j];
    }

  for (int k0 = 0; k0 < K; k0 += GBK) {
    for (int c = tid; c < GBM * CPR; c += 256) {
      const int r = c / CPR, kc = (c % CPR) * V;
      u32x4 va = {0u, 0u, 0u, 0u}, vb = {0u, 0u, 0u, 0u};
      if (m0 + r < M && k0 + kc < K) va = *reinterpret_cast<const u32x4*>(A + (size_t)(m0 + r) * K + k0 + kc);
      const int br = epi.b_row(n0 + r);
      if (br >= 0 && k0 + kc < K) vb = *reinterpret_cast<const u32x4*>(W + (size_t)br * K + k0 + kc);
      *reinterpret_cast<u32x4*>(As + r * LDK + kc) = va;
      *reinterpret_cast<u32x4*>(Bs + r * LDK + kc) = vb;
    }
    __syncthreads();
    if constexpr (sizeof(TM) == 2) {
      // 16x16x32 f16: lane supplies A[lr][8lk..8lk+8) and W[lr][8lk..8lk+8).
      f16x8 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[i] = *reinterpret_cast<const f16x8*>(As + (wm * 32 + i * 16 + lr) * LDK + 8 * lk);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        b[j] = *reinterpret_cast<const f16x8*>(Bs + (wn * 32 + j * 16 + lr) * LDK + 8 * lk);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[j], acc[i][j], 0, 0, 0);
    } else {
      // 16x16x4 f32: lane supplies A[lr][kk + lk] and W[lr][kk + lk].
#pragma unroll
      for (int kk = 0; kk < GBK; kk += 4) {
        float a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = As[(wm * 32 + i * 16 + lr) * LDK + kk + lk];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = Bs[(wn * 32 + j * 16 + lr) * LDK + kk + lk];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        if constexpr (SUMS) {
          if (kk % 16 == 12)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                add_rest(sum[i][j], acc[i][j], rest[i][j]);
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
              }
        }
      }
    }
    __syncthreads();
  }
  if constexpr (SUMS) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)  // (an overflowed sum stays infinite)
          acc[i][j][e] = sum[i][j][e] + (fabsf(rest[i][j][e]) < INFINITY ? rest[i][j][e] : 0.f);
  }
  // Output fragment layout: lane holds C[4 * lk + e][lr] of its 16x16 fragment.
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        Cs[(wm * 32 + i * 16 + 4 * lk + e) * GLDC + wn * 32 + j * 16 + lr] = acc[i][j][e];
  __syncthreads();
  epi(Cs, GLDC, m0, M, n0, GBM, GBN);
}

// ---------------------------------------------------------------- fp16 kernel (BM x 128 x 64)

// fp16 operands, K % 64 == 0.  Tile BM x 128 (BM = 128, 64 or 32), K step 64;
// four waves (2 x 2 for BM >= 64, else 1 x 4), each a block of 32x32x16
// MFMAs.  Operands go global -> LDS with direct 16-byte loads, a wave
// instruction moving 8 whole rows of the step (8 cache lines) into an
// XOR-swizzled row-major stage, so every MFMA fragment read is a
// conflict-free 16-byte read.
// NSTAGE stages: the loads of the next NSTAGE-1 steps are in flight while a
// step computes; two workgroups per CU hide the rest of the latency.  Split-K
// workgroups write fp32 partial tiles that k_splitk_finalize sums in a fixed
// order (bitwise reproducible) before applying the epilogue.  Tiles are
// numbered with the column index fastest, so (with workgroups dealt
// round-robin to the 8 XCDs) row blocks that share a weight tile run on the
// same XCD and reuse it from its L2.
template <int BM>
struct F16Tile {
  static constexpr int BN = 128, BK = 64;
  // Four waves; two workgroups per CU fit in LDS (two independent
  // workgroups hide each other's barrier and load stalls better than one
  // workgroup of eight waves with a deeper pipeline).
  static constexpr int NW = 4;
  static constexpr int THREADS = 64 * NW;
  static constexpr int OCC = 2;
  static constexpr int NSTAGE = BM == 128 ? 2 : 3;
  static constexpr int WGM = BM >= 64 ? 2 : 1, WGN = NW / WGM;  // wave grid
  static constexpr int FM = BM / WGM / 32, FN = BN / WGN / 32;  // 32x32 blocks per wave
  static constexpr int GROUPS = (BM + BN) / 8;        // 1 KiB row groups (8 rows x 64 k) per stage
  static constexpr int NI = GROUPS / NW;               // loads per wave per stage
  static constexpr int STAGE = GROUPS * 1024;
  static constexpr int LDC = BN + 4;
  static constexpr int CS = BM * LDC * 4;
  static constexpr int LDS = (NSTAGE * STAGE > CS ? NSTAGE * STAGE : CS);
  static_assert(GROUPS % NW == 0, "row groups split evenly over the waves");
};


// Workgroup barrier without the memory fence __syncthreads() adds (waits are
// explicit in the caller).
__device__ __forceinline__ void bare_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One 16-byte direct global -> LDS load per lane (wave-uniform LDS base).
// Kept in a device function: the builtin written directly in a kernel body
// makes the host pass drop the kernel's launch stub without a diagnostic.
__device__ __forceinline__ void load_lds16(const _Float16* src, char* dst) {
  __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
}

template <int NI, int NW>
__device__ __forceinline__ void issue_stage(const _Float16* const* src, int koff, char* dst, int wave) {
#pragma unroll
  for (int q = 0; q < NI; ++q)
    __builtin_amdgcn_global_load_lds(src[q] + koff, dst + (wave + NW * q) * 1024, 16, 0, 0);
}

// Wait until at most n * NI of this wave's loads are outstanding (n <= 3).
template <int NI>
__device__ __forceinline__ void wait_stages(int n) {
#define HH_VMWAIT(c) __builtin_amdgcn_s_waitcnt(((c) & 15) | (0x7 << 4) | (0xF << 8) | (((c) >> 4) << 14))
  switch (n) {
    case 0: HH_VMWAIT(0); break;
    case 1: HH_VMWAIT(NI); break;
    case 2: HH_VMWAIT(2 * NI); break;
    default: HH_VMWAIT(3 * NI); break;
  }
#undef HH_VMWAIT
}

template <int BM, class Epi>
__global__ __launch_bounds__(F16Tile<BM>::THREADS, F16Tile<BM>::OCC) void k_gemm_f16(const _Float16* __restrict__ A, int M,
                                                  const _Float16* __restrict__ W, int K, int ntn, int ntiles,
                                                  int steps_per_split, float* __restrict__ partial, int ncols,
                                                  Epi epi) {
  using T = F16Tile<BM>;
  static_assert((T::NSTAGE - 1) * T::NI <= 63, "in-flight loads exceed the vmcnt range");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tile = blockIdx.x % ntiles, split = blockIdx.x / ntiles;
  const int tn = tile % ntn, tm = tile / ntn;
  const int m0 = tm * BM, n0 = tn * T::BN;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  const int nk_all = K / T::BK;
  const int s0 = split * steps_per_split;
  const int nk = min(nk_all, s0 + steps_per_split) - s0;

  // Per-lane source addresses of the row groups this wave loads (fixed over
  // K).  A stage holds the BM rows of A then the BN rows of W, 128 bytes (the
  // step's 64 k) each; instruction q of wave w fills row group g = w + 4q
  // (rows 8g .. 8g + 7, 1 KiB; g = w + NW q): lane l takes row r = 8g + l/8 and stores it
  // in slot l%8, which holds the row's k chunk (l%8) ^ swz(r), swz(r) =
  // (r/2)%8.  Each instruction thus reads 8 whole cache lines, and an MFMA
  // fragment read (16 consecutive rows, one chunk, per 64-bank cycle) hits
  // 16 distinct bank quads.
  const _Float16* src[T::NI];
#pragma unroll
  for (int q = 0; q < T::NI; ++q) {
    const int rr = 8 * (wave + T::NW * q) + (lane >> 3);  // row within the stage
    const int chunk = (lane & 7) ^ ((rr >> 1) & 7);
    if (rr < BM) {
      const int row = min(m0 + rr, M - 1);  // rows past M: computed, never stored
      src[q] = A + (size_t)row * K + (size_t)s0 * T::BK + chunk * 8;
    } else {
      const int br = epi.b_row(n0 + rr - BM);
      src[q] = W + (size_t)(br < 0 ? 0 : br) * K + (size_t)s0 * T::BK + chunk * 8;
    }
  }

  f32x16 acc[T::FM][T::FN];
#pragma unroll
  for (int i = 0; i < T::FM; ++i)
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // Waits are explicit: __syncthreads() would add a workgroup release fence,
  // i.e. vmcnt(0), and stall on the later steps' loads as well.
  constexpr int kWaitLds = 0xF | (0x7 << 4) | (0x3 << 14);  // lgkmcnt(0)
  for (int i = 0; i < T::NSTAGE - 1 && i < nk; ++i)
    issue_stage<T::NI, T::NW>(src, i * T::BK, smem + i * T::STAGE, wave);
  for (int step = 0; step < nk; ++step) {
    const int ahead = step + T::NSTAGE - 1;
    if (ahead < nk) issue_stage<T::NI, T::NW>(src, ahead * T::BK, smem + (ahead % T::NSTAGE) * T::STAGE, wave);
    const int later = min(T::NSTAGE - 1, nk - 1 - step);  // stages after `step` in flight
    wait_stages<T::NI>(later);   // this wave's loads of `step` have landed
    bare_barrier();              // ... and every other wave's
    const char* sb = smem + (step % T::NSTAGE) * T::STAGE;
    // Fragment of rows r0 .. r0 + 31, k 16 kb .. + 16: lane l reads row
    // r0 + l%32, chunk 2 kb + l/32, from its swizzled slot.
    auto frag = [&](int r0, int kb) {
      const int r = r0 + (lane & 31), c = 2 * kb + (lane >> 5);
      return *reinterpret_cast<const f16x8*>(sb + r * 128 + 16 * (c ^ ((r >> 1) & 7)));
    };
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      f16x8 a[T::FM], b[T::FN];
#pragma unroll
      for (int i = 0; i < T::FM; ++i) a[i] = frag((wm * T::FM + i) * 32, kb);
#pragma unroll
      for (int j = 0; j < T::FN; ++j) b[j] = frag(BM + (wn * T::FN + j) * 32, kb);
#pragma unroll
      for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(kWaitLds);  // this wave's reads of the stage are done ...
    bare_barrier();                         // ... and every wave's, before it is refilled
  }
  // Result element e of lane l in a 32x32 block: row 8(e/4) + 4(l/32) + e%4, column l%32.
  if (partial) {
    float* dst = partial + (size_t)split * M * ncols;
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
      for (int j = 0; j < T::FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = m0 + (wm * T::FM + i) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          const int c = n0 + (wn * T::FN + j) * 32 + (lane & 31);
          if (r < M && c < ncols) dst[(size_t)r * ncols + c] = acc[i][j][e];
        }
    return;
  }
  float* Cs = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < T::FM; ++i)
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = (wm * T::FM + i) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        const int c = (wn * T::FN + j) * 32 + (lane & 31);
        Cs[r * T::LDC + c] = acc[i][j][e];
      }
  __syncthreads();
  epi(Cs, T::LDC, m0, M, n0, BM, T::BN);
}

// Sum the split-K partials of a 2-row block in split order and apply the
// epilogue (small blocks give the reduction enough workgroups; each thread
// sums one element's partials with independent loads).
constexpr int kFinRows = 2;
template <class Epi>
__global__ __launch_bounds__(256) void k_splitk_finalize(const float* __restrict__ partial, int splits, int M,
                                                         int ncols, int ntn, Epi epi) {
  constexpr int BN = 128, LDC = BN + 4;
  __shared__ float Cs[kFinRows * LDC];
  const int tn = blockIdx.x % ntn, tm = blockIdx.x / ntn;
  const int m0 = tm * kFinRows, n0 = tn * BN;
  for (int idx = threadIdx.x; idx < kFinRows * BN; idx += 256) {
    const int r = idx / BN, c = idx % BN;
    float v = 0.f;
    if (m0 + r < M && n0 + c < ncols) {
      const float* pp = partial + (size_t)(m0 + r) * ncols + n0 + c;
      const size_t stride = (size_t)M * ncols;
      int sp = 0;
      for (; sp + 4 <= splits; sp += 4) {
        const float a = pp[sp * stride], b = pp[(sp + 1) * stride], c2 = pp[(sp + 2) * stride], d = pp[(sp + 3) * stride];
        v += a;  // split order, as in the loop below
        v += b;
        v += c2;
        v += d;
      }
      for (; sp < splits; ++sp) v += pp[sp * stride];
    }
    Cs[r * LDC + c] = v;
  }
  __syncthreads();
  epi(Cs, LDC, m0, M, n0, kFinRows, BN);
}

// ---------------------------------------------------------------- tile kernel (prompt prefill)

// Prompt-sized GEMMs (M >= 128, and the head of every row from two rows on, which
// are 32 rows of fp16 terms): BM x BN x 64 tiles, eight waves, each a block of WM
// x 64 outputs as 16x16x32 MFMAs with the weights as the first operand: a lane's
// four results are then four consecutive columns of one row, and with the weight
// rows of a fragment taken in the order 8(r/4) + 4(j%2) + r%4 of each 32, two
// fragments give it eight, so every store is 16 bytes.
//
// What bounds it (counters, gate/up at 8192 rows, 256 x 256): the matrix cores are
// busy for 55 % of the cycles.  A K step reads 192 KiB of fragments from the LDS
// and writes 64 KiB into it, 2,048 cycles at 128 bytes each, as many as its MFMAs
// take, and the two overlap in part.  On weights of real spread the clock is also
// about 9 % lower than on zeros (448 against 410 us).  Against the kernel before
// (32x32x16 MFMAs, a workgroup per tile): 16x16x32 forms move half the accumulator
// registers per product (gate/up at 8192 rows 525 -> 505 us); one workgroup per CU
// walks the tiles of its XCD, and its loads run on into the next tile (the load
// cursor below is NST steps ahead of the MFMAs and knows nothing of tile ends), so
// neither the pipeline's fill nor the epilogue's stores leave the matrix cores idle
// (505 -> 448 us, 1,230 TFLOP/s; a library product of that shape without the
// epilogue 500 us).
//
// K steps go global -> LDS with direct 16-byte loads through NST stages, the
// addresses in scalar registers (a row group's offset and the step's) but
// for one lane offset per operand.  The fragments of a step's second half are
// read under the first half's MFMAs, the next step's first half under the
// second's; the one barrier per step stands where every wave holds its last
// fragments of the stage that the loads behind the barrier refill.
//
// LDS holds 128-byte rows (64 k) of eight 16-byte chunks; row r's chunk c lies
// at c ^ swz(r): the 16 rows of a fragment fall on 16 distinct quads of banks
// with swz = (r/2) % 8 for the activations' 16 consecutive rows, and with
// (r/2) % 2 + 2 ((r/8) % 4) for the weights' order above.
//
// XCDs: workgroups are dealt round-robin to the eight, and an XCD takes a run
// of consecutive tiles, numbered down bands of 1,024 rows, so that its 32
// workgroups share a few row and column tiles in its L2 (but see kDealSplits).
template <int BM_, int BN_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, NW = 8, THREADS = 64 * NW;
  static constexpr int WGN = BN / 64, WGM = NW / WGN, WM = BM / WGM;  // wave grid, rows per wave
  static constexpr int FM = WM / 16, FN = 4;                          // 16 x 16 blocks per wave
  static constexpr int NA = BM / 64, NB = BN / 64, NI = NA + NB;      // 8-row groups per wave and stage
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr int NST = (160 * 1024) / STAGE >= 3 ? 3 : 2;
  static constexpr int LDS = NST * STAGE;
  static_assert(WM % 32 == 0 && LDS <= 160 * 1024 && (NST - 1) * NI <= 63, "tile");
};

// One 16-byte direct buffer -> LDS load per lane (a device function for the
// reason given at load_lds16).
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ void buffer_lds16(__amdgpu_buffer_rsrc_t r, lds_char* dst, int voff, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

// Split products of one round whose units are dealt to the XCDs in turn, down the
// rows first: QKV (us at 256 / 384 / 448 rows, with the splits of tile_choice, in
// runs 14.6 / 15.3 / 16.5, dealt 12.4 / 13.7 / 15.6; along the columns first 13.3 /
// 14.0 / 15.3).  Their partials take as long to write back as the K steps take.
// The down projection is no faster dealt (256 rows 17.9 / 18.0, 512 18.6 / 19.0).
template <class Epi>
constexpr bool kDealSplits = false;
template <typename TKV>
constexpr bool kDealSplits<EpiQKV<TKV>> = true;

template <int BM, int BN, class Epi>
__global__ __launch_bounds__(512, 2) void k_gemm_tile(const _Float16* __restrict__ A, int M,
                                                      const _Float16* __restrict__ W, int K, int ntm, int ntn,
                                                      int splits, int steps_per_split, float* __restrict__ partial,
                                                      int ncols, Epi epi) {
  using T = Tile<BM, BN>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef __attribute__((address_space(3))) const f16x8 lds_f16x8;
  const int tiles = ntm * ntn, units = tiles * splits;
  const int per = (units + 7) / 8, hop = gridDim.x / 8, xcd = blockIdx.x & 7;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int wm = wave / T::WGN, wn = wave % T::WGN, l15 = lane & 15, h = lane >> 4;
  const int nk_all = K / 64;
  const unsigned rowb = (unsigned)K * 2;

  // The unit'th piece of work of this workgroup: a tile and a K split.
  struct Unit {
    int m0, n0, split, s0, nk;
  };
  auto unit_at = [&](int idx, Unit& u) {
    const bool deal = kDealSplits<Epi> && splits > 1;
    const int o = deal ? 8 * idx + xcd : xcd * per + idx;
    if (idx >= per || o >= units) return false;
    u.split = o / tiles;
    const int t = o - u.split * tiles;
    if (deal) {
      u.n0 = (t / ntm) * BN;
      u.m0 = (t % ntm) * BM;
    } else {
      constexpr int GM = 1024 / BM;
      const int band = t / (GM * ntn), r = t - band * GM * ntn, gm = min(GM, ntm - band * GM);
      u.n0 = (r / gm) * BN;
      u.m0 = (band * GM + r % gm) * BM;
    }
    u.s0 = u.split * steps_per_split;
    u.nk = min(nk_all, u.s0 + steps_per_split) - u.s0;
    return true;
  };
  int idx = blockIdx.x >> 3;
  Unit u;
  if (!unit_at(idx, u)) return;

  // Load cursor: the next K step to load, on the tile it belongs to.  Wave w's
  // instruction q fills row group g = w + 8 q (rows 8g .. 8g + 7, 1 KiB) of an
  // operand.  Rows past M in a group that starts before M are outside the
  // buffer's range (zeros); a group wholly past M, or past the columns, loads
  // the tile's first rows instead.  Neither is ever stored.
  int cidx = idx, ck = 0;
  bool alive = true;
  Unit cu = u;
  const char *pa, *pw;
  unsigned reca, oa[T::NA], ow[T::NB];
  auto cursor_tile = [&]() {
    pa = reinterpret_cast<const char*>(A) + ((size_t)cu.m0 * K + (size_t)cu.s0 * 64) * 2;
    const int rows = min(M - cu.m0, BM);
    reca = (unsigned)rows * rowb - (unsigned)cu.s0 * 128;
#pragma unroll
    for (int q = 0; q < T::NA; ++q) oa[q] = 8 * (wave + 8 * q) < rows ? (unsigned)(8 * (wave + 8 * q)) * rowb : 0u;
    const int b0 = epi.b_row(cu.n0);
    pw = reinterpret_cast<const char*>(W) + ((size_t)b0 * K + (size_t)cu.s0 * 64) * 2;
#pragma unroll
    for (int q = 0; q < T::NB; ++q) {
      const int br = epi.b_row(cu.n0 + 8 * (wave + 8 * q));
      ow[q] = br < 0 ? 0u : (unsigned)(br - b0) * rowb;
    }
    ck = cu.nk;
  };
  auto cursor_next = [&]() {
    if (!alive) return;
    if (--ck > 0) {
      pa += 128;
      pw += 128;
      reca -= 128;
      return;
    }
    cidx += hop;
    alive = unit_at(cidx, cu);  // past the last unit: the last step again, into stages nobody reads
    if (alive) cursor_tile();
  };
  cursor_tile();
  const int va = (lane >> 3) * (int)rowb + 16 * ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7));
  const int vb = (lane >> 3) * (int)rowb + 16 * ((lane & 7) ^ (((lane >> 4) & 1) | ((wave & 3) << 1)));
  auto issue = [&](unsigned so) {
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)pa, (short)0, (int)reca, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)pw, (short)0, -1, 0x00020000);
    lds_char* dst = (lds_char*)smem + so + wave * 1024;
#pragma unroll
    for (int q = 0; q < T::NA; ++q) buffer_lds16(ra, dst + 8192 * q, va, oa[q]);
#pragma unroll
    for (int q = 0; q < T::NB; ++q) buffer_lds16(rw, dst + BM * 128 + 8192 * q, vb, ow[q]);
  };

  // Fragment addresses of the two 32-wide halves of a step.
  int fa[2], fw[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    fa[kb] = (wm * T::WM + l15) * 128 + 16 * ((4 * kb + h) ^ (l15 >> 1));
    fw[kb] = (BM + wn * 64 + 8 * (l15 >> 2) + (l15 & 3)) * 128 +
             16 * ((4 * kb + h) ^ (((l15 >> 1) & 1) | ((l15 >> 2) << 1)));
  }
  f32x4 acc[T::FM][T::FN];
  // kPairSums: the high parts' sums over the steps so far (their roundings go
  // to the low parts' accumulators); acc holds one step's.
  constexpr bool SUMS = kPairSums<Epi>;
  f32x4 sum[SUMS ? T::FM / 2 : 1][T::FN];
  f16x8 a[2][T::FM], b[2][T::FN];
  auto frags = [&](int kb, unsigned so) {
    const lds_char* base = (const lds_char*)smem + so;
#pragma unroll
    for (int j = 0; j < T::FN; ++j) b[kb][j] = *(lds_f16x8*)(base + fw[kb] + (j >> 1) * 4096 + (j & 1) * 512);
#pragma unroll
    for (int i = 0; i < T::FM; ++i) a[kb][i] = *(lds_f16x8*)(base + fa[kb] + i * 2048);
  };
  auto mma = [&](int kb) {
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
      for (int j = 0; j < T::FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
            b[kb][j], a[kb][i], SUMS && kb == 0 && i % 2 == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i][j], 0, 0, 0);
  };
  constexpr int NRD = T::FM + T::FN;
  constexpr int kWaitLds = 0xF | (0x7 << 4) | (0x3 << 14);  // lgkmcnt(0)
#pragma unroll
  for (int s = 0; s < T::NST; ++s) {
    issue(s * T::STAGE);
    cursor_next();
  }
  unsigned so = 0;
  wait_stages<T::NI>(T::NST - 1);
  bare_barrier();
  frags(0, 0);
  while (true) {
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
      for (int j = 0; j < T::FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (SUMS) {
#pragma unroll
      for (int i = 0; i < T::FM / 2; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int step = 0; step < u.nk; ++step) {
      const unsigned sn = so + T::STAGE == T::LDS ? 0u : so + T::STAGE;
      __builtin_amdgcn_sched_barrier(0);
      frags(1, so);
      mma(0);
#pragma unroll
      for (int k = 0; k < NRD; ++k) {  // MFMA, read, MFMA, read, ...
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(kWaitLds);  // this wave has its last fragments of the stage
      wait_stages<T::NI>(T::NST - 2);        // and its loads of the next step have landed
      bare_barrier();
      __builtin_amdgcn_sched_barrier(0);
      frags(0, sn);
      issue(so);
      mma(1);
#pragma unroll
      for (int k = 0; k < (T::NI > NRD ? T::NI : NRD); ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (k < T::NI) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        if (k < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (SUMS) {
#pragma unroll
        for (int i = 0; i < T::FM / 2; ++i)
#pragma unroll
          for (int j = 0; j < T::FN; ++j) add_rest(sum[i][j], acc[2 * i][j], acc[2 * i + 1][j]);
      }
      cursor_next();
      so = sn;
    }
    if constexpr (SUMS) {
#pragma unroll
      for (int i = 0; i < T::FM / 2; ++i)
#pragma unroll
        for (int j = 0; j < T::FN; ++j) acc[2 * i][j] = sum[i][j];
    }
    const int row0 = u.m0 + wm * T::WM + l15, cb = u.n0 + wn * 64;
    if (partial) {
      float* dst = partial + (size_t)u.split * M * ncols;
      if (cb < ncols) {  // ncols % 64 == 0
#pragma unroll
        for (int i = 0; i < T::FM; ++i)
          if (row0 + 16 * i < M) {
#pragma unroll
            for (int j = 0; j < T::FN; ++j)
              *reinterpret_cast<f32x4*>(dst + (size_t)(row0 + 16 * i) * ncols + cb + 32 * (j >> 1) + 8 * h + 4 * (j & 1)) =
                  acc[i][j];
          }
      }
    } else {
      epi.template tile<T::FM>(row0, cb, h, M, acc);
    }
    idx += hop;
    if (!unit_at(idx, u)) break;
  }
  wait_stages<T::NI>(0);  // no direct-to-LDS load outlives the workgroup
}

// ---------------------------------------------------------------- mid kernel (at most 128 rows)

// Short prompts and lockstep decoding past 32 streams: C[M <= 128, N] = A W^T is
// bound by bringing operands into the CUs, so a workgroup owns 64 logical
// columns over one K range and takes each operand in once, through a ring of
// DEPTH 64-wide K steps in LDS with DEPTH - 2 of them in flight (direct loads of
// whole 128-byte lines; the 16-row pattern of an MFMA operand loaded straight
// to registers reaches a quarter of their rate: 38 against 150 GB/s a CU from
// the L2).  The small-tile kernel, which has two steps in flight and reads
// the weights once per 64 rows, is slower where launch_mid says so (gate/up at
// 64 rows 24.1 -> 18.1 us; what is left there is ~5 us of start and end, and
// 0.4 us a step at ~13 TB/s into the CUs).
// Eight waves: wave w has columns 16 (w % 4) .. + 16 and the 32-wide half w / 4
// of each step, for all MT * 16 rows; the halves are added in LDS.
template <int MT_>
struct Mid {
  static constexpr int MT = MT_, ROWS = 16 * MT, STAGE = (ROWS + 64) * 128, DEPTH = MT == 8 ? 6 : 8;
  static constexpr int XI = MT == 8 ? 2 : 1, NI = XI + 1;  // a wave's loads per step
  static constexpr int LDS = DEPTH * STAGE, LDC = 68;
  static_assert(ROWS * LDC * 4 <= LDS && LDS <= 160 * 1024, "ring, and the finished tile in it");
};

template <int MT, class Epi>
__global__ __launch_bounds__(512, 2) void k_gemm_mid(const _Float16* __restrict__ A, int M,
                                                     const _Float16* __restrict__ W, int K, int nb,
                                                     int steps_per_split, float* __restrict__ partial, int ncols,
                                                     Epi epi) {
  using T = Mid<MT>;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  typedef __attribute__((address_space(3))) const f16x8 lds_f16x8;
  const int cbk = blockIdx.x % nb, split = blockIdx.x / nb, n0 = cbk * 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int cw = wave & 3, kh = wave >> 2, l15 = lane & 15, h = lane >> 4;
  const int s0 = split * steps_per_split, nk = min(K / 64, s0 + steps_per_split) - s0;
  const unsigned rowb = (unsigned)K * 2;

  // Activations: wave w's instruction q fills row group w + 8 q (8 rows, 1 KiB;
  // with 32 rows waves 4 .. 7 repeat waves 0 .. 3).  Groups past M load the first
  // rows again, rows past M in a group are outside the buffer's range; no
  // such row is stored.  Weights: wave w fills row group w of the 64 columns.
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(A) + (size_t)s0 * 128), (short)0, (int)((unsigned)M * rowb - (unsigned)s0 * 128),
      0x00020000);
  const int b0 = epi.b_row(n0), br = epi.b_row(n0 + 8 * wave);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(reinterpret_cast<const char*>(W) + ((size_t)b0 * K + (size_t)s0 * 64) * 2), (short)0, -1, 0x00020000);
  const int xw = MT == 2 ? wave & 3 : wave;
  const int va = (lane >> 3) * (int)rowb + 16 * ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7));
  unsigned oa[T::XI];
#pragma unroll
  for (int q = 0; q < T::XI; ++q) oa[q] = 8 * (xw + 8 * q) < M ? (unsigned)(8 * (xw + 8 * q)) * rowb : 0u;
  const unsigned ow = br < 0 ? 0u : (unsigned)(br - b0) * rowb;
  // Steps past the range load its last one again, into slots nobody reads.
  auto issue = [&](int s, unsigned so) {
    const unsigned koff = (unsigned)min(s, nk - 1) * 128;
    lds_char* dst = (lds_char*)smem + so;
#pragma unroll
    for (int q = 0; q < T::XI; ++q) buffer_lds16(ra, dst + (xw + 8 * q) * 1024, va, oa[q] + koff);
    buffer_lds16(rw, dst + T::ROWS * 128 + wave * 1024, va, ow + koff);
  };
  f32x4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fx = l15 * 128 + 16 * ((4 * kh + h) ^ (l15 >> 1)), fw = fx + (T::ROWS + 16 * cw) * 128;
  f16x8 x[2][MT], w[2];
  auto frags = [&](int set, unsigned so) {
    const lds_char* base = (const lds_char*)smem + so;
    w[set] = *(lds_f16x8*)(base + fw);
#pragma unroll
    for (int m = 0; m < MT; ++m) x[set][m] = *(lds_f16x8*)(base + fx + m * 2048);
  };
#define HH_MID_WAIT(steps)                                                                            \
  __builtin_amdgcn_s_waitcnt(((T::NI * (steps)) & 15) | (0x7 << 4) | (0xF << 8) | (((T::NI * (steps)) >> 4) << 14))
#pragma unroll
  for (int s = 0; s + 1 < T::DEPTH; ++s) issue(s, s * T::STAGE);
  HH_MID_WAIT(T::DEPTH - 2);
  bare_barrier();
  frags(0, 0);
  unsigned so = 0, sp = (T::DEPTH - 1) * T::STAGE;  // this step's slot and the one before it
  // Step s + 1 has landed (this wave's loads, then every wave's), and every
  // wave is done with step s - 1, whose slot is refilled.  The next step's
  // fragments are read under this one's products.
  auto step = [&](int s, int set) {
    HH_MID_WAIT(T::DEPTH - 3);
    bare_barrier();
    issue(s + T::DEPTH - 1, sp);
    const unsigned sn = so + T::STAGE == T::LDS ? 0u : so + T::STAGE;
    frags(set ^ 1, sn);
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[set], x[set][m], acc[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < MT + 1; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    sp = so;
    so = sn;
  };
  int s = 0;
  for (; s + 1 < nk; s += 2) {
    step(s, 0);
    step(s + 1, 1);
  }
  if (s < nk) step(s, 0);
#undef HH_MID_WAIT
  __builtin_amdgcn_s_waitcnt(0);  // no direct-to-LDS load is left
  __syncthreads();
  float* Cs = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    if (kh == g) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        f32x4* c = reinterpret_cast<f32x4*>(Cs + (16 * m + l15) * T::LDC + 16 * cw + 4 * h);
        *c = g ? *c + acc[m] : acc[m];
      }
    }
    __syncthreads();
  }
  if (partial) {  // ncols % 64 == 0
    float* dst = partial + (size_t)split * M * ncols + n0;
    for (int i = threadIdx.x; i < M * 16; i += 512)
      *reinterpret_cast<f32x4*>(dst + (size_t)(i >> 4) * ncols + 4 * (i & 15)) =
          *reinterpret_cast<const f32x4*>(Cs + (i >> 4) * T::LDC + 4 * (i & 15));
    return;
  }
  epi(Cs, T::LDC, 0, M, n0, T::ROWS, 64);
}

// ---------------------------------------------------------------- launchers

// Launchers return the number of K splits used.  With defer set, split
// partials are left in the workspace for the caller to reduce (1: the
// epilogue already ran).
template <int BM, class Epi>
static int launch_f16(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const _Float16* W, int K, int n_cols,
                      const Epi& e, bool defer) {
  using T = F16Tile<BM>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_f16<BM, Epi>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
    attr = true;
  }
  const int ntn = (n_cols + T::BN - 1) / T::BN;
  const int ntiles = ((M + BM - 1) / BM) * ntn;
  const int nk = K / T::BK;
  // Split K only when tiles alone leave most CUs idle: then aim at 256
  // workgroups, at least 4 K steps each, with partials that fit the workspace.
  int splits = ntiles < 128 ? (256 + ntiles - 1) / ntiles : 1;
  splits = std::min(splits, std::max(1, nk / 4));
  while (splits > 1 && (size_t)splits * M * n_cols * sizeof(float) > ws.bytes) --splits;
  const int per = (nk + splits - 1) / splits;
  splits = (nk + per - 1) / per;
  float* part = splits > 1 ? ws.ptr : nullptr;
  k_gemm_f16<BM, Epi><<<ntiles * splits, T::THREADS, T::LDS, st>>>(A, M, W, K, ntn, ntiles, per, part, n_cols, e);
  if (splits > 1 && !defer)
    k_splitk_finalize<Epi><<<((M + kFinRows - 1) / kFinRows) * ntn, 256, 0, st>>>(part, splits, M, n_cols, ntn, e);
  return splits;
}

template <int BM, int BN, class Epi>
static int launch_tile(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const _Float16* W, int K, int n_cols,
                       int splits, const Epi& e, bool defer) {
  using T = Tile<BM, BN>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_tile<BM, BN, Epi>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
    attr = true;
  }
  const int ntn = (n_cols + BN - 1) / BN, ntm = (M + BM - 1) / BM;
  const int nk = K / 64;
  splits = std::max(1, std::min(splits, nk / 4));
  while (splits > 1 && (size_t)splits * M * n_cols * sizeof(float) > ws.bytes) --splits;
  const int per = (nk + splits - 1) / splits;
  splits = (nk + per - 1) / per;
  float* part = splits > 1 ? ws.ptr : nullptr;
  // One workgroup per CU, the same number on each XCD.
  const int grid = 8 * std::min((ntm * ntn * splits + 7) / 8, 256 / 8);
  k_gemm_tile<BM, BN, Epi><<<grid, T::THREADS, T::LDS, st>>>(A, M, W, K, ntm, ntn, splits, per, part, n_cols, e);
  if (splits > 1 && !defer) {
    const int nf = (n_cols + 127) / 128;
    k_splitk_finalize<Epi><<<((M + kFinRows - 1) / kFinRows) * nf, 256, 0, st>>>(part, splits, M, n_cols, nf, e);
  }
  return splits;
}

// Returns the K splits, 0 where the small-tile kernel is the better one.  us a
// layer of the 1B model, this kernel / small tiles: gate/up at 24 rows 17.8 /
// 20.3, 40 rows 17.5 / 22.2, 64 rows 18.1 / 24.1, 99 rows 21.9 / 25.0, 128 rows
// 23.6 / 25.4; O and down together at 24 rows 14.4 / 13.7, 40 rows 15.2 / 16.1,
// 64 rows 16.6 / 17.8, 99 rows 21.6 / 19.4; QKV at 24 rows 6.2 / 5.8, 40 rows
// 6.7 / 7.0, 64 rows 7.4 / 8.0, 99 rows 9.6 / 9.6; the LM head at 64 rows 145 /
// 115.  So: gate/up at any of these row counts, O, down and QKV from 33 to 64.
template <int MT, class Epi>
static int launch_mid(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const _Float16* W, int K, int n_cols,
                      const Epi& e, bool defer) {
  using T = Mid<MT>;
  const int nb = (n_cols + 63) / 64, nk = K / 64;
  int splits = std::max(1, std::min((256 + nb / 2) / nb, nk / 4));
  while (splits > 1 && (size_t)splits * M * n_cols * sizeof(float) > ws.bytes) --splits;
  const int per = (nk + splits - 1) / splits;
  splits = (nk + per - 1) / per;
  if (nb * splits < 64) return 0;  // a quarter of the CUs
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_mid<MT, Epi>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
    attr = true;
  }
  float* part = splits > 1 ? ws.ptr : nullptr;
  k_gemm_mid<MT, Epi><<<nb * splits, 512, T::LDS, st>>>(A, M, W, K, nb, per, part, n_cols, e);
  if (splits > 1 && !defer) {
    const int nf = (n_cols + 127) / 128;
    k_splitk_finalize<Epi><<<((M + kFinRows - 1) / kFinRows) * nf, 256, 0, st>>>(part, splits, M, n_cols, nf, e);
  }
  return splits;
}

template <class Epi>
static int run_mid(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const _Float16* W, int K, int n_cols,
                   const Epi& e, GemmKind kind, bool defer) {
  if constexpr (std::is_same<Epi, EpiLogits<false>>::value) {
    return 0;
  } else {
    if (M > 128 || n_cols % 64) return 0;
    if (M > 32 && M <= 64) return launch_mid<4>(st, ws, A, M, W, K, n_cols, e, defer);
    if constexpr (std::is_same<Epi, EpiGateUp<_Float16>>::value)
      return M <= 32 ? launch_mid<2>(st, ws, A, M, W, K, n_cols, e, defer)
                     : launch_mid<8>(st, ws, A, M, W, K, n_cols, e, defer);
    return 0;
  }
}

// ---------------------------------------------------------------- skinny kernel (<= 32 rows)

// Lockstep multi-stream decode: C[M <= 32, N] = A W^T is weight streaming, not
// arithmetic.  A workgroup owns 64 logical columns (one QKV head, 32 gate + 32
// up columns, or 64 residual columns) and one K range; each group of four
// waves takes 16 weight rows per wave (KW groups split the K range).  Weights
// go from HBM straight into registers as the A operand of 16x16x32 MFMAs (lane
// l: row l%16, k 8(l/16) .. + 8), from a copy laid out as 16 x 32 operand
// tiles, in batches of eight K blocks with the next batch loading while one
// computes; the activations (at most 32 rows) of each batch are loaded once per
// K group, coalesced, into double-buffered LDS (16-byte row padding keeps the
// B fragment reads conflict-free).  The finished 64-column tile goes through
// LDS into the usual epilogue, or into split partials when K is split to give
// every CU work.
// RowNorm consumer of the 32-row kernels: thread t < 256 loads float4 t % 8
// of row t / 8's block sums (nss <= 32, a multiple of 4; eight consecutive
// lanes read one row's 128 bytes) first thing, so that the tail finds them
// landed (zeros past M rows or nss sums).
__device__ __forceinline__ void row_norm_loads(float4& ssv, const RowNorm& rn, int M) {
  if (!rn.ss_in || threadIdx.x >= 256) return;
  const __amdgpu_buffer_rsrc_t res =
      __builtin_amdgcn_make_buffer_rsrc((void*)rn.ss_in, (short)0, (int)((size_t)M * rn.nss * 4), 0x00020000);
  const int r = threadIdx.x >> 3, q = threadIdx.x & 7;
  ssv = __builtin_bit_cast(
      float4, __builtin_amdgcn_raw_buffer_load_b128(
                  res, r < M && 4 * q < rn.nss ? (unsigned)((r * rn.nss + 4 * q) * 4) : 0x80000000u, 0, 0));
}

// acc0[j] of lane l: column 16 rw + 4 (l / 16) + j, row l % 16 (acc1: row
// + 16).  K groups add into the LDS tile Cs (32 x 68 floats) in group order;
// rows are scaled by their norm factors (RowNorm consumer; rs: 32 floats of LDS).
template <int KW>
__device__ __forceinline__ void skinny_tile(float* Cs, const f32x4& acc0, const f32x4& acc1, int rw, int kg, int lane,
                                            const RowNorm& rn, const float4& ssv, float* rs) {
  constexpr int LDC = 68;
  const int col = 16 * rw + 4 * (lane >> 4), r = lane & 15;
  float f0 = 1.f, f1 = 1.f;  // norm factors of rows r and r + 16
  if (rn.ss_in) {
    if (threadIdx.x < 256) {
      float v = (ssv.x + ssv.y) + (ssv.z + ssv.w);
      v += __shfl_xor(v, 1);
      v += __shfl_xor(v, 2);
      v += __shfl_xor(v, 4);
      if ((threadIdx.x & 7) == 0) rs[threadIdx.x >> 3] = rsqrtf(v / rn.n + rn.eps);
    }
    __syncthreads();
    f0 = rs[r];
    f1 = rs[r + 16];
  }
#pragma unroll
  for (int g = 0; g < KW; ++g) {
    if (kg == g) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        Cs[r * LDC + col + j] = (g ? Cs[r * LDC + col + j] : 0.f) + acc0[j] * f0;
        Cs[(r + 16) * LDC + col + j] = (g ? Cs[(r + 16) * LDC + col + j] : 0.f) + acc1[j] * f1;
      }
    }
    __syncthreads();
  }
}

// The finished tile (Cs: the caller's activation buffer, once every wave is done
// with it) goes to the split partials or through the epilogue.  A RowNorm
// producer's last split of the column block then finishes the residual (flag:
// LDS scratch of one int).
template <class Epi, int KW>
__device__ __forceinline__ void skinny_tail(float* Cs, const f32x4& acc0, const f32x4& acc1, int rw, int kg, int lane,
                                            float* __restrict__ partial, int split, int splits, int cb, int M,
                                            int ncols, int n0, const Epi& epi, const RowNorm& rn,
                                            const float4& ssv, float* rs, int* flag) {
  constexpr int LDC = 68;
  skinny_tile<KW>(Cs, acc0, acc1, rw, kg, lane, rn, ssv, rs);
  if (partial) {
    bool producer = false;
    if constexpr (std::is_same<Epi, EpiResid>::value) producer = rn.cnt != nullptr;
    if (!producer) {
      float* dst = partial + (size_t)split * M * ncols;
      for (int i = threadIdx.x; i < M * 64; i += blockDim.x) {
        const int rr = i / 64, c = i % 64;
        if (n0 + c < ncols) dst[(size_t)rr * ncols + n0 + c] = Cs[rr * LDC + c];
      }
      return;
    }
    if constexpr (std::is_same<Epi, EpiResid>::value) {
      // RowNorm producer.  The partials go out and come back with the
      // agent-coherent cache policy, so that no fence (and no writeback or
      // invalidation of a whole L2) is needed: a split's stores have
      // completed before it counts itself in, and the last split to arrive
      // reads every split's partials from the coherent level.
      constexpr int kSc1 = 16;
      const int N = epi.N;
      const __amdgpu_buffer_rsrc_t pres = __builtin_amdgcn_make_buffer_rsrc(
          (void*)partial, (short)0, (int)((size_t)splits * M * ncols * 4), 0x00020000);
      const unsigned sstride = (unsigned)M * ncols * 4;  // bytes of one split's partials
      // Items: row rr = it / 16, four columns n0 + 4 (it % 16); a row's 16
      // items are 16 aligned lanes of one wave (M * 16 <= 512 <= 2 blockDim).
      // Every split loads its items' x and gains before counting itself in,
      // so the last one does not wait for them afterwards.
      float4 xa[2], ga[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int it = threadIdx.x + blockDim.x * k, rr = it >> 4, c = n0 + 4 * (it & 15);
        if (it < M * 16 && c < N) {
          xa[k] = *reinterpret_cast<const float4*>(epi.x + (size_t)rr * N + c);
          ga[k] = *reinterpret_cast<const float4*>(rn.gain + c);
        }
      }
      for (int it = threadIdx.x; it < M * 16; it += blockDim.x) {
        const int rr = it >> 4, c = n0 + 4 * (it & 15);
        if (c < ncols) {
          const float4 v = *reinterpret_cast<const float4*>(Cs + rr * LDC + 4 * (it & 15));
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), pres,
                                                 (unsigned)split * sstride + (unsigned)(rr * ncols + c) * 4, 0, kSc1);
        }
      }
      __builtin_amdgcn_s_waitcnt(0);  // every store of this thread acknowledged
      __syncthreads();
      if (threadIdx.x == 0) *flag = atomicAdd(rn.cnt + cb, 1) == splits - 1;
      __syncthreads();
      if (!*flag) return;
      // Up to 8 splits: both items' partials are loaded at once; more splits
      // go 8 at a time.  Either way they are summed in split order.
      float4 t[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) t[k] = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int s0 = 0; s0 < splits; s0 += 8) {
        float4 u[2][8];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int it = threadIdx.x + blockDim.x * k, rr = it >> 4, c = n0 + 4 * (it & 15);
          const bool ok = it < M * 16 && c < N;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            u[k][j] = __builtin_bit_cast(
                float4, __builtin_amdgcn_raw_buffer_load_b128(
                            pres, ok && s0 + j < splits ? (unsigned)(s0 + j) * sstride + (unsigned)(rr * ncols + c) * 4
                                                        : 0x80000000u,
                            0, kSc1));
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (s0 + j < splits) {
              t[k].x += u[k][j].x;
              t[k].y += u[k][j].y;
              t[k].z += u[k][j].z;
              t[k].w += u[k][j].w;
            }
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int it = threadIdx.x + blockDim.x * k, rr = it >> 4, c = n0 + 4 * (it & 15);
        float sq = 0.f;
        if (it < M * 16 && c < N) {
          float4 a = xa[k];
          a.x += t[k].x * epi.scale;
          a.y += t[k].y * epi.scale;
          a.z += t[k].z * epi.scale;
          a.w += t[k].w * epi.scale;
          *reinterpret_cast<float4*>(epi.x + (size_t)rr * N + c) = a;
          const float4 g = ga[k];
          typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
          const f16x4 o = {(_Float16)(a.x * g.x), (_Float16)(a.y * g.y), (_Float16)(a.z * g.z), (_Float16)(a.w * g.w)};
          *reinterpret_cast<f16x4*>(rn.y + (size_t)rr * N + c) = o;
          sq = a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        }
        sq += __shfl_xor(sq, 8);
        sq += __shfl_xor(sq, 4);
        sq += __shfl_xor(sq, 2);
        sq += __shfl_xor(sq, 1);
        if (it < M * 16 && (it & 15) == 0) rn.ss_out[(size_t)rr * ((N + 63) / 64) + cb] = sq;
      }
      if (threadIdx.x == 0) __hip_atomic_store(rn.cnt + cb, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  epi(Cs, LDC, 0, M, n0, 32, 64);
}
constexpr int kSkinnyTileBytes = 32 * 68 * 4;
// LDS row pitch (halfs) of the activation-resident skinny kernel: a K group's
// largest block count rounded up to 4 blocks (256 bytes), plus 16 bytes.
__host__ __device__ constexpr int skinny_res_pitch(int steps_per_split, int kw) {
  return 32 * ((((steps_per_split + kw - 1) / kw) + 3) & ~3) + 8;
}

template <class Epi, int U, int KW>
__global__ __launch_bounds__(256 * KW) void k_gemm_skinny(const _Float16* __restrict__ A, int M,
                                                          const _Float16* __restrict__ Wt, int K, int nb,
                                                          int steps_per_split, float* __restrict__ partial, int ncols,
                                                          Epi epi, RowNorm rn) {
  constexpr int XP = 32 * U + 8;              // LDS row pitch of an activation chunk (halfs; 16 bytes of padding)
  constexpr int XCH = 32 * (32 * U / 8);      // 16-byte chunks per activation batch (32 rows)
  static_assert(XCH % 256 == 0, "activation chunks split evenly over a group's threads");
  __shared__ __attribute__((aligned(16))) _Float16 xs[KW][2][32 * XP];
  static_assert(sizeof(xs) >= kSkinnyTileBytes, "the tile fits the activation buffers");
  __shared__ float rs[32];
  __shared__ int flag;
  float4 ssv = make_float4(0.f, 0.f, 0.f, 0.f);
  row_norm_loads(ssv, rn, M);
  const int cb = blockIdx.x % nb, split = blockIdx.x / nb;
  const int n0 = cb * 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rw = wave & 3, kg = wave >> 2;  // 16-row group, K group
  const int gt = threadIdx.x & 255;         // thread index within the K group
  const int k0 = split * steps_per_split * 32;
  const int nkb_all = min(K - k0, steps_per_split * 32) / 32;  // K blocks of 32 in this range
  // K group kg takes blocks [kb_lo, kb_lo + nkb) of the range.
  const int kb_lo = (nkb_all * kg) / KW, nkb = (nkb_all * (kg + 1)) / KW - kb_lo;
  const int kbase = k0 + 32 * kb_lo;

  // Weights (16 x 32 operand tiles, 1 KiB each in lane order, so a load
  // instruction reads one contiguous KiB) and activations both come through
  // range-checked buffer loads: the batches need no clamping (blocks past this
  // range read further on, or zeros past the matrix, and are never used), and
  // activation rows past M read zeros.
  const int nkbt = K / 32;  // tiles per 16-row block
  const int rb = 4 * cb + rw;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)Wt, (short)0, (int)((size_t)((ncols + 15) / 16) * 16 * K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t xres =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)((size_t)M * K * 2), 0x00020000);
  const unsigned wvoff = (unsigned)((((size_t)rb * nkbt + kbase / 32) * 64 + lane) * 16);
  // Activation batch: group thread t loads chunks t + 256 j (row c / (4 U), 8
  // halfs at 8 (c % (4 U))), consecutive threads reading consecutive 16 bytes.
  constexpr int XJ = XCH / 256;
  auto xload = [&](f16x8* v, int kb0) {
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
      const int c = gt + 256 * j, r = c / (4 * U), kc = c % (4 * U);
      v[j] = __builtin_bit_cast(
          f16x8, __builtin_amdgcn_raw_buffer_load_b128(xres, (unsigned)((r * K + kbase + 32 * kb0 + 8 * kc) * 2), 0, 0));
    }
  };
  auto xstore = [&](const f16x8* v, int buf) {
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
      const int c = gt + 256 * j, r = c / (4 * U), kc = c % (4 * U);
      *reinterpret_cast<f16x8*>(&xs[kg][buf][r * XP + 8 * kc]) = v[j];
    }
  };
  // Weights are read once per step: non-temporal loads (streaming policy in
  // the caches) measured 15.9 -> 15.1 us for gate/up and 98 -> 93 us for the
  // LM head at 32 rows.
  constexpr int kNt = 2;
  auto wload = [&](f16x8* w, int kb0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      w[u] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, wvoff + 1024u * (kb0 + u), 0, kNt));
  };
  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const f16x8* w, int buf, int kb0) {
    const _Float16* xb = &xs[kg][buf][(lane & 15) * XP + 8 * (lane >> 4)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kb0 + u < nkb) {
        const f16x8 b0 = *reinterpret_cast<const f16x8*>(xb + 32 * u);
        const f16x8 b1 = *reinterpret_cast<const f16x8*>(xb + 16 * XP + 32 * u);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u], b0, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u], b1, acc1, 0, 0, 0);
      }
    }
  };
  // Batch i computes from xs[kg][i & 1] and registers wa / wb while batch
  // i + 1's activations and weights load; one barrier per batch (the same
  // count in every K group) orders the LDS reuse.
  const int nbatch = ((nkb_all + KW - 1) / KW + U - 1) / U;
  f16x8 wa[U], wb[U], xv[XJ];
  xload(xv, 0);
  wload(wa, 0);
  xstore(xv, 0);
  __syncthreads();
  for (int bt = 0; bt < nbatch; bt += 2) {
    if (bt + 1 < nbatch) {
      xload(xv, (bt + 1) * U);  // issued before the weights, so waiting for it leaves them in flight
      wload(wb, (bt + 1) * U);
    }
    compute(wa, 0, bt * U);
    if (bt + 1 >= nbatch) break;
    xstore(xv, 1);
    __syncthreads();
    if (bt + 2 < nbatch) {
      xload(xv, (bt + 2) * U);
      wload(wa, (bt + 2) * U);
    }
    compute(wb, 1, (bt + 1) * U);
    if (bt + 2 >= nbatch) break;
    xstore(xv, 0);
    __syncthreads();
  }

  __syncthreads();  // every wave is done with the activations
  skinny_tail<Epi, KW>(reinterpret_cast<float*>(&xs[0][0][0]), acc0, acc1, rw, kg, lane, partial, split, gridDim.x / nb,
                       cb, M, ncols, n0, epi, rn, ssv, rs, &flag);
}

// Activation-resident variant, for grids of at most two workgroups per CU:
// every wave issues its first weight loads with the activations and the rest
// (at most 32 K blocks, 32 KiB per wave, in all) once those have landed, the workgroup's activation range (32 rows x at most 1024 K
// per K group) goes into LDS once, and each block's MFMAs wait only for that
// block's weights.  The batched kernel above pays an L2 round trip and a
// barrier per 256 K of activations, and keeps two batches in flight: at 32
// rows its gate/up launch took 7.3 us with no weight loads at all.  Loads a
// wave does not need (blocks past its range, chunks past the group's K) take
// an offset past the buffer's range, which returns zeros without a memory
// access, so the issue order stays branch-free.  Wave rw of a K group loads
// rows rw, rw + 4, ... (16-byte chunks lane + 64 q along the row); the LDS row
// pitch is 16 bytes past a multiple of 256 bytes, as in the batched kernel,
// so the B fragment reads stay conflict-free.
template <class Epi, int NB, int KW>
__global__ __launch_bounds__(256 * KW) void k_gemm_skinny_res(const _Float16* __restrict__ A, int M,
                                                              const _Float16* __restrict__ Wt, int K, int nb,
                                                              int steps_per_split, float* __restrict__ partial,
                                                              int ncols, Epi epi, RowNorm rn) {
  constexpr int XQ = (4 * NB + 63) / 64;  // activation chunks per lane and row
  constexpr unsigned kOob = 0x80000000u;  // past every buffer range here (ranges stay below 2^31 bytes)
  extern __shared__ __attribute__((aligned(16))) _Float16 xsd[];
  __shared__ float rs[32];
  __shared__ int flag;
  float4 ssv = make_float4(0.f, 0.f, 0.f, 0.f);
  row_norm_loads(ssv, rn, M);  // first, so that no later wait covers them
  const int cb = blockIdx.x % nb, split = blockIdx.x / nb;
  const int n0 = cb * 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rw = wave & 3, kg = wave >> 2;
  const int k0 = split * steps_per_split * 32;
  const int nkb_all = min(K - k0, steps_per_split * 32) / 32;
  const int kb_lo = (nkb_all * kg) / KW, nkb = (nkb_all * (kg + 1)) / KW - kb_lo;
  const int kbase = k0 + 32 * kb_lo;
  const int pitch = skinny_res_pitch(steps_per_split, KW);
  _Float16* xs = xsd + (size_t)kg * 32 * pitch;
  // Chunks past the group's K are stored to a 16-byte slot past the tiles.
  _Float16* sink = xsd + (size_t)KW * 32 * pitch;

  const int nkbt = K / 32;
  const int rb = 4 * cb + rw;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)Wt, (short)0, (int)((size_t)((ncols + 15) / 16) * 16 * K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t xres =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)((size_t)M * K * 2), 0x00020000);
  const unsigned wvoff = (unsigned)((((size_t)rb * nkbt + kbase / 32) * 64 + lane) * 16);
  constexpr int kNt = 2;  // weights are read once per step: streaming policy
  // Activations first, so that the wait before their LDS stores leaves the
  // weights in flight.  Rows past M read zeros.
  f16x8 xv[8][XQ];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int kc = lane + 64 * q;
      const unsigned off = kc < 4 * nkb ? (unsigned)(((rw + 4 * i) * K + kbase + 8 * kc) * 2) : kOob;
      xv[i][q] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(xres, off, 0, 0));
    }
  // The scheduler would otherwise start the LDS stores (and so wait for the
  // activations) before issuing the first weight loads.
  __builtin_amdgcn_sched_barrier(0);
  // Wave (rb, kg) starts its tiles at block `rot` of its range and wraps
  // around, so that the waves' first requests do not all fall on 32 KiB
  // boundaries (every range starts on one).
  const int rot = nkb > 0 ? (rb * 13 + kg * 7) % nkb : 0;
  auto blk = [&](int u) { return u + rot < nkb ? u + rot : u + rot - nkb; };
  // Only the first W0 weight blocks go out with the activations: with every
  // block issued at once, the activations (a shared 128 KiB per workgroup,
  // from memory after the producing launch) came back behind the weight
  // stream, ~10 us into a 13.5 us gate/up launch, and every MFMA waited for
  // them.  The rest of the weights follow once the activations have landed
  // (the 32-row step 0.957 -> 0.947 ms; 4, 12 and 16 blocks first measured
  // 0.948, 0.951 and 0.954).
  constexpr int W0 = NB < 8 ? NB : 8;
  f16x8 w[NB];
#pragma unroll
  for (int u = 0; u < W0; ++u)
    w[u] = __builtin_bit_cast(
        f16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, u < nkb ? wvoff + 1024u * blk(u) : kOob, 0, kNt));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int kc = lane + 64 * q;
      _Float16* dst = kc < 4 * nkb ? xs + (rw + 4 * i) * pitch + 8 * kc : sink;
      *reinterpret_cast<f16x8*>(dst) = xv[i][q];
    }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = W0; u < NB; ++u)
    w[u] = __builtin_bit_cast(
        f16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, u < nkb ? wvoff + 1024u * blk(u) : kOob, 0, kNt));
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();

  f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
  const _Float16* xb = xs + (lane & 15) * pitch + 8 * (lane >> 4);
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    if (u < nkb) {
      const int kb = blk(u);
      const f16x8 b0 = *reinterpret_cast<const f16x8*>(xb + 32 * kb);
      const f16x8 b1 = *reinterpret_cast<const f16x8*>(xb + 16 * pitch + 32 * kb);
      acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u], b0, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u], b1, acc1, 0, 0, 0);
    }
  }

  __syncthreads();  // every wave is done with the activations
  skinny_tail<Epi, KW>(reinterpret_cast<float*>(xsd), acc0, acc1, rw, kg, lane, partial, split, gridDim.x / nb, cb, M,
                       ncols, n0, epi, rn, ssv, rs, &flag);
}

constexpr int kSkinnyResLds = 159 * 1024;  // dynamic LDS limit of the resident kernel

template <class Epi, int NB, int KW>
static bool skinny_res_go(hipStream_t st, unsigned bytes, const _Float16* A, int M, const _Float16* Wt, int K, int nb,
                          int splits, int per, float* part, int n_cols, const Epi& e, const RowNorm& rn) {
  // Once per instantiation, to the largest size the launcher allows (the
  // kernel's static LDS takes the rest of the 160 KiB).
  static const hipError_t attr = [] {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_skinny_res<Epi, NB, KW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kSkinnyResLds);
    if (e != hipSuccess) (void)hipGetLastError();  // the batched kernel runs instead
    return e;
  }();
  if (attr != hipSuccess) return false;
  k_gemm_skinny_res<Epi, NB, KW><<<nb * splits, 256 * KW, bytes, st>>>(A, M, Wt, K, nb, per, part, n_cols, e, rn);
  return true;
}

// The activation-resident kernel takes grids of at most two workgroups per CU
// whose K groups hold at most 32 K blocks (1024 K) each (HH_SKINNY_RES=0 turns
// it off, for comparison); returns false when the batched kernel is to run.
template <class Epi>
static bool launch_skinny_res(hipStream_t st, const _Float16* A, int M, const _Float16* Wt, int K, int nb, int splits,
                              int per, float* part, int n_cols, int kw, const Epi& e, const RowNorm& rn) {
  if constexpr (std::is_same<Epi, EpiLogits<false>>::value) {
    return false;
  } else {
    const char* v = getenv("HH_SKINNY_RES");
    const bool on = !(v && v[0] == '0');
    const int gmax = (per + kw - 1) / kw;
    // K-group tiles plus the 16-byte sink for unused chunks.
    const size_t lds = (size_t)kw * 32 * skinny_res_pitch(per, kw) * 2 + 16;
    if (!on || (long long)nb * splits > 2 * 256 || gmax > 32 || lds > (size_t)kSkinnyResLds) return false;
    const unsigned bytes = (unsigned)std::max<size_t>(lds, kSkinnyTileBytes);
    auto go = [&](auto nbc, auto kwc) {
      return skinny_res_go<Epi, decltype(nbc)::value, decltype(kwc)::value>(st, bytes, A, M, Wt, K, nb, splits, per,
                                                                            part, n_cols, e, rn);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    if (kw == 2) {
      if (gmax <= 8) return go(std::integral_constant<int, 8>(), I2());
      if (gmax <= 16) return go(std::integral_constant<int, 16>(), I2());
      return go(std::integral_constant<int, 32>(), I2());
    }
    if (gmax <= 8) return go(std::integral_constant<int, 8>(), I1());
    if (gmax <= 16) return go(std::integral_constant<int, 16>(), I1());
    return go(std::integral_constant<int, 32>(), I1());
  }
}

// ---------------------------------------------------------------- skinny kernel on 4-bit codes

// The activation-resident product on a 4-bit model's stored codes: lockstep
// decoding streamed the fp16 copies of the dequantized values, 3.6 times the
// bytes.  A lane's 16-byte load holds its operand rows' codes of four K
// blocks; a block's eight codes become fp16 values of exactly q / 16 (nibbles in
// the mantissa of 64, then minus 64.5) times the group's scale (times 16: at most
// 16 2^14 / 7).  Both factors are exact and the product is rounded once, so it is
// the copy's operand, down to scales of 2^-21 (2^-35 of the model's largest
// weight; below, the scale is rounded too).  us at 6 rows of the 1B model, fp16
// tiles / codes: gate/up 14.5 / 8.8, down 11.4 / 9.0, O 7.2 / 7.1, QKV 5.0 / 4.6, LM
// head 86 / 35; what is left is a launch's start and end and the activations'
// round trip, and in the head the unpacking (15 instructions per 8 codes and
// lane).
// Waves, K groups, activations and the tail are k_gemm_skinny_res's.  BY_K:
// scales belong to k (W_down, grouped along its output rows) and go through
// LDS.  LOOP (LM head): a workgroup walks the column blocks with its
// activations resident and the next block's codes in flight.
// mask and magic: 0x000F000F and 0x54005400, in registers (q4_constants), so that
// each pair takes one and-or instruction, which has no room for literals.
__device__ __forceinline__ void q4_constants(unsigned& mask, unsigned& magic) {
  asm("s_mov_b32 %0, 0x000f000f" : "=s"(mask));
  asm("v_mov_b32 %0, 0x54005400" : "=v"(magic));
}
__device__ __forceinline__ f16x8 q4_values(unsigned w, unsigned mask, unsigned magic) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  const h2 off = {(_Float16)64.5f, (_Float16)64.5f};
  f16x8 r;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const unsigned t = ((w >> (4 * p)) & mask) | magic;
    const h2 v = __builtin_bit_cast(h2, t) - off;
    r[2 * p] = v[0];
    r[2 * p + 1] = v[1];
  }
  return r;
}

constexpr int q4_pitch(int nb4) { return 128 * nb4 + 8; }  // LDS row of a K group's activations (halfs)

template <class Epi, int NB4, int KW, bool BY_K, bool LOOP, bool TWO>
__global__ __launch_bounds__(256 * KW) void k_gemm_skinny_q4(const _Float16* __restrict__ A, int M, WTiles wt, int K,
                                                             int nb, int blocks_per_split,
                                                             float* __restrict__ partial, int ncols, Epi epi,
                                                             RowNorm rn) {
  constexpr int XQ = (16 * NB4 + 63) / 64, PITCH = q4_pitch(NB4);
  constexpr unsigned kOob = 0x80000000u;  // past every buffer range here
  constexpr int kNt = 2;                  // codes are read once per step: streaming policy
  extern __shared__ __attribute__((aligned(16))) _Float16 xsd[];
  __shared__ float rs[32];
  __shared__ int flag;
  float4 ssv = make_float4(0.f, 0.f, 0.f, 0.f);
  row_norm_loads(ssv, rn, M);
  int cb = blockIdx.x % nb;
  const int split = LOOP ? 0 : blockIdx.x / nb;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rw = wave & 3, kg = wave >> 2;
  const int kb0 = split * blocks_per_split;  // 128-wide K blocks
  const int n_all = min(K / 128 - kb0, blocks_per_split);
  const int lo = (n_all * kg) / KW, n4 = (n_all * (kg + 1)) / KW - lo;  // this K group's, at most NB4
  const int kbase = 128 * (kb0 + lo), nk4 = K / 128;
  _Float16* xs = xsd + (size_t)kg * 32 * PITCH;
  _Float16* after = xsd + (size_t)KW * 32 * PITCH;
  _Float16* sk = after + (size_t)kg * 2 * 128 * NB4;  // BY_K: scales of the two 32-column groups
  float* tail = reinterpret_cast<float*>(LOOP ? after : xsd);

  const size_t rb16 = (size_t)((ncols + 15) / 16);
  const __amdgpu_buffer_rsrc_t xres =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)((size_t)M * K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t cres =
      __builtin_amdgcn_make_buffer_rsrc((void*)wt.q, (short)0, (int)(rb16 * 16 * K / 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t sres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)wt.s, (short)0, (int)(BY_K ? (size_t)(ncols / 32) * K * 2 : rb16 * 16 * (K / 32) * 2), 0x00020000);
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x4 w[NB4], wn[LOOP ? NB4 : 1];
  u32x2 sc[NB4], sn[LOOP ? NB4 : 1];
  auto load = [&](u32x4* cw, u32x2* cs, int c) {
    const unsigned b0 = (unsigned)((4 * c + rw) * nk4 + kb0 + lo);
#pragma unroll
    for (int u = 0; u < NB4; ++u) {
      const bool ok = u < n4 && c < nb;
      cw[u] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(cres, ok ? ((b0 + u) * 64 + lane) * 16 : kOob, 0, kNt));
      if (!BY_K)
        cs[u] = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_raw_buffer_load_b64(sres, ok ? ((b0 + u) * 16 + (lane & 15)) * 8 : kOob, 0, kNt));
    }
  };
  // Activations (rows past M and K past the group's read zeros, and a K
  // group's missing blocks have zero scales: no branch below) and, with scales
  // by k, the workgroup's scales first; then the codes.
  static_assert(XQ * 64 == 16 * NB4, "whole waves of chunks");
  f16x8 xv[8][XQ];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int kc = lane + 64 * q;
      xv[i][q] = __builtin_bit_cast(
          f16x8, __builtin_amdgcn_raw_buffer_load_b128(
                     xres, kc < 16 * n4 ? (unsigned)(((rw + 4 * i) * K + kbase + 8 * kc) * 2) : kOob, 0, 0));
    }
  constexpr int SJ = (32 * NB4 + 255) / 256;
  f16x8 sv[BY_K ? SJ : 1];
  if constexpr (BY_K) {
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
      const int c = (threadIdx.x & 255) + 256 * j, g = c / (16 * NB4), kc = c % (16 * NB4);
      sv[j] = __builtin_bit_cast(
          f16x8, __builtin_amdgcn_raw_buffer_load_b128(
                     sres, g < 2 && kc < 16 * n4 ? (unsigned)(((2 * cb + g) * K + kbase + 8 * kc) * 2) : kOob, 0, 0));
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  load(w, sc, cb);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int kc = lane + 64 * q;
      *reinterpret_cast<f16x8*>(xs + (rw + 4 * i) * PITCH + 8 * kc) = xv[i][q];
    }
  if constexpr (BY_K) {
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
      const int c = (threadIdx.x & 255) + 256 * j, g = c / (16 * NB4), kc = c % (16 * NB4);
      if (g < 2) *reinterpret_cast<f16x8*>(sk + g * 128 * NB4 + 8 * kc) = sv[j];
    }
  }
  __syncthreads();
  const _Float16* xb = xs + (lane & 15) * PITCH + 8 * (lane >> 4);
  const _Float16* sb = sk + (rw >> 1) * 128 * NB4 + 8 * (lane >> 4);
  unsigned long long best = 0ull;
  unsigned mask, magic;
  q4_constants(mask, magic);
  while (true) {
    if constexpr (LOOP) load(wn, sn, cb + (int)gridDim.x);  // past the last block: zeros, no access
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NB4; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const _Float16* xp = xb + 128 * u + 32 * j;
        const f16x8 x0 = *reinterpret_cast<const f16x8*>(xp);
        f16x8 a = q4_values(w[u][j], mask, magic);
        if constexpr (BY_K) {
          a = a * *reinterpret_cast<const f16x8*>(sb + 128 * u + 32 * j);
        } else {
          const _Float16 f = __builtin_bit_cast(_Float16, (unsigned short)(sc[u][j >> 1] >> (16 * (j & 1))));
          a = a * f16x8{f, f, f, f, f, f, f, f};
        }
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, x0, acc0, 0, 0, 0);
        if constexpr (TWO)
          acc1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, *reinterpret_cast<const f16x8*>(xp + 16 * PITCH), acc1, 0, 0, 0);
      }
    if (!LOOP) __syncthreads();  // every wave is done with the activations
    if constexpr (!LOOP) {
      skinny_tail<Epi, KW>(tail, acc0, acc1, rw, kg, lane, partial, split, (int)gridDim.x / nb, cb, M, ncols, cb * 64,
                           epi, rn, ssv, rs, &flag);
      break;
    } else {
      skinny_tile<KW>(tail, acc0, acc1, rw, kg, lane, rn, ssv, rs);
      epi.block(tail, 68, M, cb * 64, best);
    }
    cb += gridDim.x;
    if (cb >= nb) break;
    __syncthreads();  // the tile is read out
#pragma unroll
    for (int u = 0; u < NB4; ++u) {
      w[u] = wn[LOOP ? u : 0];
      sc[u] = sn[LOOP ? u : 0];
    }
  }
  if constexpr (LOOP) epi.finish(M, best);
}

template <class Epi, int NB4, int KW, bool BY_K, bool LOOP, bool TWO>
static bool skinny_q4_run(hipStream_t st, int grid, const _Float16* A, int M, const WTiles& wt, int K, int nb, int per,
                         float* part, int n_cols, const Epi& e, const RowNorm& rn) {
  const size_t need = ((size_t)KW * 32 * q4_pitch(NB4) + (BY_K ? (size_t)KW * 2 * 128 * NB4 : 0)) * 2 +
                      (LOOP ? kSkinnyTileBytes : 0);
  constexpr size_t kLds = 159 * 1024;  // the kernel's static LDS takes the rest
  if (need > kLds) return false;
  static const hipError_t attr = [] {
    const hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_skinny_q4<Epi, NB4, KW, BY_K, LOOP, TWO>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (r != hipSuccess) (void)hipGetLastError();  // the fp16 tiles are used instead
    return r;
  }();
  if (attr != hipSuccess) return false;
  k_gemm_skinny_q4<Epi, NB4, KW, BY_K, LOOP, TWO>
      <<<grid, 256 * KW, std::max<size_t>(need, kSkinnyTileBytes), st>>>(A, M, wt, K, nb, per, part, n_cols, e, rn);
  return true;
}

template <class Epi, int NB4, int KW, bool BY_K, bool LOOP>
static bool skinny_q4_go(hipStream_t st, int grid, const _Float16* A, int M, const WTiles& wt, int K, int nb, int per,
                         float* part, int n_cols, const Epi& e, const RowNorm& rn) {
  return M > 16 ? skinny_q4_run<Epi, NB4, KW, BY_K, LOOP, true>(st, grid, A, M, wt, K, nb, per, part, n_cols, e, rn)
                : skinny_q4_run<Epi, NB4, KW, BY_K, LOOP, false>(st, grid, A, M, wt, K, nb, per, part, n_cols, e, rn);
}

// K splits of the <= 32-row kernels, 32-wide K blocks per split, and K groups
// per workgroup.
struct SkinnyPlan {
  int splits, per, kw;
};
static SkinnyPlan skinny_plan(int M, int K, int n_cols, size_t ws_bytes, bool codes) {
  const int nb = (n_cols + 63) / 64, nk = K / 32;
  // Split K only to give about 256 workgroups, with at least 16 K blocks
  // (512 K) per split: at 32 rows the O and QKV products (64 K blocks) run
  // 4 splits, not 8 and 6 (step 1.002 -> 0.978 ms; the down projection keeps
  // 8, which 4 slowed).
  int splits = std::max(1, std::min((256 + nb - 1) / nb, nk / 16));
  while (splits > 1 && (size_t)splits * M * n_cols * sizeof(float) > ws_bytes) --splits;
  int per = (nk + splits - 1) / splits;
  if (codes) per = (per + 3) & ~3;  // whole 128-wide blocks of codes
  splits = (nk + per - 1) / per;
  // Unsplit (long) K ranges take two K groups per workgroup: eight waves per
  // CU keep more weight loads in flight (gate/up 17.0 -> 15.9 us at 32 rows).
  return SkinnyPlan{splits, per, splits == 1 ? 2 : 1};
}

// Shapes of the kernel on codes: K a multiple of 128, at most 1,024 of it per K
// group, one workgroup per (64 columns, split) up to two per CU, or the LM head,
// which loops and does not split.  (31-bit byte offsets as in launch_skinny.)
static bool skinny_q4_fits(const SkinnyPlan& p, int K, int n_cols, bool head, bool by_k) {
  const int nb = (n_cols + 63) / 64;
  if (K % 128 || p.per % 4 || (p.per / 4 + p.kw - 1) / p.kw > 8) return false;
  if ((size_t)((n_cols + 15) / 16) * 16 * K * 2 >= ((size_t)1 << 31) || (by_k && n_cols % 64)) return false;
  return head ? p.splits == 1 && !by_k : (long long)nb * p.splits <= 2 * 256;
}
bool skinny_codes_serve(int K, int n_cols, bool head, bool by_k, size_t ws_bytes, int max_rows) {
  for (int M = 1; M <= std::min(32, max_rows); ++M)
    if (!skinny_q4_fits(skinny_plan(M, K, n_cols, ws_bytes, true), K, n_cols, head, by_k)) return false;
  return true;
}

template <class Epi>
static bool launch_skinny_q4(hipStream_t st, const _Float16* A, int M, const WTiles& wt, int K, int nb, int splits,
                             int per32, float* part, int n_cols, int kw, const Epi& e, const RowNorm& rn) {
  constexpr bool head = std::is_same<Epi, EpiLogits<false>>::value;
  if (!wt.q || !skinny_q4_fits(SkinnyPlan{splits, per32, kw}, K, n_cols, head, wt.by_k)) return false;
  const int per = per32 / 4, g = (per + kw - 1) / kw;
  if constexpr (head) {
    return skinny_q4_go<Epi, 8, 2, false, true>(st, std::min(nb, 256), A, M, wt, K, nb, per, part, n_cols, e, rn);
  } else {
    auto go = [&](auto n, auto k, auto by) {
      return skinny_q4_go<Epi, decltype(n)::value, decltype(k)::value, decltype(by)::value, false>(
          st, nb * splits, A, M, wt, K, nb, per, part, n_cols, e, rn);
    };
    using std::integral_constant;
    using I1 = integral_constant<int, 1>;
    using I2 = integral_constant<int, 2>;
    using I4 = integral_constant<int, 4>;
    using I8 = integral_constant<int, 8>;
    using No = std::false_type;
    if constexpr (std::is_same<Epi, EpiResid>::value) {
      using Yes = std::true_type;
      if (wt.by_k) return kw == 2 ? go(I8(), I2(), Yes()) : g <= 4 ? go(I4(), I1(), Yes()) : go(I8(), I1(), Yes());
    }
    if (wt.by_k) return false;
    if (kw == 2) return g <= 4 ? go(I4(), I2(), No()) : go(I8(), I2(), No());
    return g <= 4 ? go(I4(), I1(), No()) : go(I8(), I1(), No());
  }
}

// Returns the K splits, 0 when the shape does not fit the 32-row kernels.
// rn: see RowNorm; its producer half runs only in the activation-resident
// kernel of a split residual product (*fused = 1 then, and the partials are
// consumed in the kernel).
template <class Epi>
static int launch_skinny(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const WTiles& wt, int K,
                         int n_cols, const Epi& e, bool defer, RowNorm rn, int* fused) {
  if (fused) *fused = 0;
  // Buffer ranges take 31-bit byte offsets.
  if ((size_t)((n_cols + 15) / 16) * 16 * K * 2 >= ((size_t)1 << 31) || (size_t)32 * K * 2 >= ((size_t)1 << 31)) return 0;
  // The consumer half reads at most 32 block sums per row (a multiple of 4).
  if (rn.ss_in && (rn.nss > 32 || rn.nss % 4)) return 0;
  const int nb = (n_cols + 63) / 64;
  const SkinnyPlan plan = skinny_plan(M, K, n_cols, ws.bytes, wt.q != nullptr);
  const int splits = plan.splits, per = plan.per, kw = plan.kw;
  const _Float16* Wt = wt.h;
  float* part = splits > 1 ? ws.ptr : nullptr;
  if (!(std::is_same<Epi, EpiResid>::value && splits > 1 && n_cols % 64 == 0 && nb <= rn.ncnt)) rn.cnt = nullptr;
  if (!launch_skinny_q4<Epi>(st, A, M, wt, K, nb, splits, per, part, n_cols, kw, e, rn)) {
    if (!Wt) return 0;
    if (!launch_skinny_res<Epi>(st, A, M, Wt, K, nb, splits, per, part, n_cols, kw, e, rn)) {
      rn.cnt = nullptr;
      if (kw == 2)
        k_gemm_skinny<Epi, 8, 2><<<nb * splits, 512, 0, st>>>(A, M, Wt, K, nb, per, part, n_cols, e, rn);
      else
        k_gemm_skinny<Epi, 8, 1><<<nb * splits, 256, 0, st>>>(A, M, Wt, K, nb, per, part, n_cols, e, rn);
    }
  }
  if (rn.cnt) {
    if (fused) *fused = 1;
    return splits;
  }
  if (splits > 1 && !defer)
    k_splitk_finalize<Epi><<<((M + kFinRows - 1) / kFinRows) * ((n_cols + 127) / 128), 256, 0, st>>>(
        part, splits, M, n_cols, (n_cols + 127) / 128, e);
  return splits;
}

// RowNorm consumer fallback for products that no 32-row kernel takes: scale
// the rows of A (x * gain as fp16) in place by their norm factors.
__global__ __launch_bounds__(256) void k_rownorm_apply(_Float16* __restrict__ A, int K, RowNorm rn) {
  __shared__ float red[4];
  const int row = blockIdx.x;
  float v = 0.f;
  if (threadIdx.x == 0)
    for (int j = 0; j < rn.nss; ++j) v += rn.ss_in[(size_t)row * rn.nss + j];
  const float inv = rsqrtf(block_sum256(v, red) / rn.n + rn.eps);
  for (int k = threadIdx.x; k < K; k += 256) A[(size_t)row * K + k] = (_Float16)((float)A[(size_t)row * K + k] * inv);
}

// Tile choice of a prompt-sized GEMM: {BM, BN, splits}, BM == 0 for the
// small-tile kernel.  HH_GEMM_QKV / _RESID (O projection) / _DOWN / _GATEUP =
// "BMxBNxS" (or "0") overrides it, for tuning.
struct TileCfg {
  int bm, bn, splits;
};

// The tile and K splits (a power of two up to max_splits) of least estimated
// time: rounds x (steps x step + tail), where a round is a unit (tile, K split)
// on each of the 256 CUs, plus writing and reading back the partials of a
// split.  step and tail (us) are fits to the products of the 1B layer at 512 ..
// 8,192 rows, and the choices they give are the fastest measured there or
// within 3 %: gate/up 256 x 256 from 1,024 rows (8,192 rows: 256 x 256 448, 256
// x 128 509 us; 1,024: 65 and 69) and 256 x 128 at 512 (37.5; 256 x 256 on half
// the CUs 56); QKV 128 x 128 to 1,024 rows and 256 x 128 above (8,192: 114, 256
// x 256 132, 128 x 128 134); down 8,192 rows 256 x 256 236 (128 x 128 302),
// 1,024 rows 128 x 128 in two splits 47.
static TileCfg fit_tile(GemmKind kind, int M, int n_cols, int K, int max_splits, double* us = nullptr) {
  struct Cand {
    int bm, bn;
    double step, tail, tail_qkv;
  };
  static const Cand cands[3] = {{256, 256, 1.60, 4.7, 16.0}, {256, 128, 0.95, 2.3, 7.0}, {128, 128, 0.58, 1.4, 4.0}};
  TileCfg best{0, 0, 1};
  double least = 1e30;
  for (const Cand& c : cands)
    for (int splits = 1; splits <= max_splits; splits *= 2) {
      const int nk = K / 64;
      if (splits > 1 && nk / splits < 4) break;
      const long long units = (long long)((M + c.bm - 1) / c.bm) * ((n_cols + c.bn - 1) / c.bn) * splits;
      const double t = (double)((units + 255) / 256) *
                           ((double)((nk + splits - 1) / splits) * c.step + (kind == GemmKind::QKV ? c.tail_qkv : c.tail)) +
                       (splits > 1 ? 0.37e-6 * 4.0 * splits * (double)M * n_cols : 0.0);
      if (t < least) {
        least = t;
        best = TileCfg{c.bm, c.bn, splits};
      }
    }
  if (us) *us = least;
  return best;
}

// Gate/up rows that go to a first launch of full rounds (0: one launch for
// all).  A last round that holds a few row tiles costs as much as a full one
// (3,168 rows: 832 tiles of 256 x 256 on 256 CUs, 3.25 rounds, take four), so
// the last rows go to a launch of their own where its estimate and ~5 us
// between the two come to less.  Up to 128 rows that launch is the mid
// kernel's (~0.55 us a step and ~5 us, one round of 256 blocks of 64 columns).
// Whole 1B prefills, one launch / two: 1,100 rows 4.05 / 3.92 ms, 1,230 4.15 /
// 4.00, 2,100 6.74 / 6.33, 2,500 7.18 / 7.09, 32 prompts of 99 10.56 / 10.40.
static int gateup_first_rows(int M, int n_cols, int K) {
  if (getenv("HH_GEMM_GATEUP")) return 0;
  double whole = 0.0;
  fit_tile(GemmKind::GateUp, M, n_cols, K, 1, &whole);
  int first = 0;
  double least = 0.95 * whole;
  for (int k = 0; k < 4; ++k) {
    const int m1 = (M - 1) / 256 * 256 - 256 * k, rest = M - m1;
    if (m1 < 512) break;
    double t = 0.0, t2 = 0.0;
    fit_tile(GemmKind::GateUp, m1, n_cols, K, 1, &t);
    if (rest > 128) fit_tile(GemmKind::GateUp, rest, n_cols, K, 1, &t2);
    else t2 = (double)((n_cols / 64 + 255) / 256) * (K / 64 * 0.55 + 5.0);
    if (t + t2 + 5.0 < least) {
      least = t + t2 + 5.0;
      first = m1;
    }
  }
  return first;
}

static TileCfg tile_choice(GemmKind kind, int M, int n_cols, int K) {
  static const char* names[4] = {"HH_GEMM_QKV", "HH_GEMM_RESID", "HH_GEMM_GATEUP", "HH_GEMM_LOGITS"};
  // The down projection (K > N) has a knob of its own.
  const char* env = getenv(kind == GemmKind::Resid && K > n_cols ? "HH_GEMM_DOWN" : names[(int)kind]);
  if (env) {
    TileCfg c{0, 0, 1};
    if (sscanf(env, "%dx%dx%d", &c.bm, &c.bn, &c.splits) < 2) return TileCfg{0, 0, 1};
    if (kind == GemmKind::Logits) c.splits = 1;  // partials have whole groups of 64 columns
    return c;
  }
  // Below 512 rows (1B shapes; us a layer at 256 rows, tiles / the small-tile
  // kernel): two or more row tiles of gate/up 26.9 / 33.6; the down
  // projection with K split over 256 workgroups 18.6 / 20.8; QKV from 256 rows
  // with the K splits, up to four, that fill one round (its reduction applies the
  // epilogue): 256 rows, four, 12.4 + 6.3 / 12.8 + 7.0; 384 rows, three, 13.7 +
  // 8.9 / 24.0 (four, two rounds, 17.7 + 8.2); 448 rows, two, 15.6 + 8.9 (four
  // 18.0 + 9.0); O stays with the small tiles (13.4 / 8.7: few steps, and two
  // workgroups a CU hide each other's start).
  if (kind == GemmKind::GateUp && (n_cols < 8192 || M <= 128)) return TileCfg{0, 0, 1};
  if (kind == GemmKind::QKV && M < 512) {
    if (M < 256) return TileCfg{0, 0, 1};
    const int tiles = (M + 127) / 128 * ((n_cols + 127) / 128);
    return TileCfg{128, 128, std::max(1, std::min(4, 256 / tiles))};
  }
  if (kind == GemmKind::Resid && M < 512 && (K < 4096 || M <= 128)) return TileCfg{0, 0, 1};
  return fit_tile(kind, M, n_cols, K, kind == GemmKind::Resid ? 8 : 1);
}

// Returns the splits used, 0 when the shape is left to the small-tile kernel.
template <class Epi>
static int run_tile(hipStream_t st, GemmWorkspace ws, const _Float16* A, int M, const _Float16* W, int K, int n_cols,
                    const Epi& e, GemmKind kind, bool defer) {
  if (M < 128) return 0;
  const TileCfg c = tile_choice(kind, M, n_cols, K);
  if (c.bm == 256 && c.bn == 256) return launch_tile<256, 256>(st, ws, A, M, W, K, n_cols, c.splits, e, defer);
  if (c.bm == 256 && c.bn == 128) return launch_tile<256, 128>(st, ws, A, M, W, K, n_cols, c.splits, e, defer);
  if (c.bm == 128 && c.bn == 128) return launch_tile<128, 128>(st, ws, A, M, W, K, n_cols, c.splits, e, defer);
  return 0;
}

// Run C = A W^T over n_cols logical columns with epilogue e; returns the K
// splits used (with defer, partials of a split run are left in ws.ptr).
// rn (fp16 operands only): RowNorm's consumer and producer halves, honoured
// by the 32-row kernels; a consumer request that no 32-row kernel takes
// scales A's rows first, and *fused says whether the producer half ran.
template <typename TM, class Epi>
static int run_gemm(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int K, int n_cols, const Epi& e,
                    GemmKind kind, bool defer = false, const WTiles& Wt = WTiles(), const RowNorm& rn = RowNorm(),
                    int* fused = nullptr) {
  if (fused) *fused = 0;
  if constexpr (sizeof(TM) == 2) {
    if (M <= 32 && (Wt.h || Wt.q) && K % 64 == 0) {
      const int sp = launch_skinny(st, ws, reinterpret_cast<const _Float16*>(A), M, Wt, K, n_cols, e, defer, rn, fused);
      if (sp > 0) return sp;
    }
    if (rn.ss_in)
      k_rownorm_apply<<<M, 256, 0, st>>>(reinterpret_cast<_Float16*>(const_cast<TM*>(A)), K, rn);
    if (K % 64 == 0) {
      const _Float16* Ah = reinterpret_cast<const _Float16*>(A);
      const _Float16* Wh = reinterpret_cast<const _Float16*>(W);
      const int spm = run_mid(st, ws, Ah, M, Wh, K, n_cols, e, kind, defer);
      if (spm > 0) return spm;
      const int sp = run_tile(st, ws, Ah, M, Wh, K, n_cols, e, kind, defer);
      if (sp > 0) return sp;
      const long long ntn = (n_cols + 127) / 128;
      if (M <= 32) return launch_f16<32>(st, ws, Ah, M, Wh, K, n_cols, e, defer);
      if (M <= 64 || ((M + 127) / 128) * ntn < 256) return launch_f16<64>(st, ws, Ah, M, Wh, K, n_cols, e, defer);
      return launch_f16<128>(st, ws, Ah, M, Wh, K, n_cols, e, defer);
    }
  }
  k_gemm<TM, Epi><<<dim3((n_cols + GBN - 1) / GBN, (M + GBM - 1) / GBM), 256, 0, st>>>(A, M, W, K, e);
  return 1;
}

// ---------------------------------------------------------------- residual + RMSNorm

// One row per workgroup: x[row] += (sum of the split partials, in split
// order) * scale when splits > 0, then h[row] = x[row] * rsqrt(mean(x^2) +
// eps) * gain in the MFMA operand type.  The row (N % 4 == 0, N <= 4096) stays
// in registers between the two halves.
constexpr int kNormMaxChunks = 4;  // float4 chunks per thread: N <= 4096
constexpr int kNormSplitBatch = 8;  // split partials in flight per chunk
template <typename TM>
__global__ __launch_bounds__(256) void k_resid_norm(const float* __restrict__ partial, int splits, int M, int N, float scale,
                                                    float* __restrict__ x, const float* __restrict__ gain, float eps,
                                                    TM* __restrict__ h, const int* __restrict__ rows) {
  __shared__ float red[4];
  const int row = blockIdx.x, nc = N >> 2;
  float4* xr = reinterpret_cast<float4*>(x + (size_t)(rows ? rows[row] : row) * N);
  float4 v[kNormMaxChunks], g[kNormMaxChunks];
  // The gains load with the row, so the second half waits on no global load.
#pragma unroll
  for (int k = 0; k < kNormMaxChunks; ++k) {
    const int ch = threadIdx.x + 256 * k;
    if (ch < nc) g[k] = reinterpret_cast<const float4*>(gain)[ch];
  }
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < kNormMaxChunks; ++k) {
    const int ch = threadIdx.x + 256 * k;
    if (ch < nc) {
      float4 a = xr[ch];
      if (splits > 0) {
        const float4* pp = reinterpret_cast<const float4*>(partial + (size_t)row * N) + ch;
        const size_t stride = (size_t)M * nc;  // one split's partials, in float4
        // Up to kNormSplitBatch partials are loaded at once (clamped indices,
        // unused ones dropped), then summed in split order.
        float4 t = pp[0];
        for (int s0 = 1; s0 < splits; s0 += kNormSplitBatch) {
          float4 u[kNormSplitBatch];
#pragma unroll
          for (int j = 0; j < kNormSplitBatch; ++j) u[j] = pp[min(s0 + j, splits - 1) * stride];
#pragma unroll
          for (int j = 0; j < kNormSplitBatch; ++j)
            if (s0 + j < splits) {
              t.x += u[j].x;
              t.y += u[j].y;
              t.z += u[j].z;
              t.w += u[j].w;
            }
        }
        a.x += t.x * scale;
        a.y += t.y * scale;
        a.z += t.z * scale;
        a.w += t.w * scale;
        xr[ch] = a;
      }
      v[k] = a;
      ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
    }
  }
  const float inv = rsqrtf(block_sum256(ss, red) / (float)N + eps);
#pragma unroll
  for (int k = 0; k < kNormMaxChunks; ++k) {
    const int ch = threadIdx.x + 256 * k;
    if (ch < nc) {
      const float4 gk = g[k];
      TM* hr = h + (size_t)row * N + 4 * ch;
      if constexpr (sizeof(TM) == 2) {
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        const f16x4 o = {(_Float16)(v[k].x * inv * gk.x), (_Float16)(v[k].y * inv * gk.y),
                         (_Float16)(v[k].z * inv * gk.z), (_Float16)(v[k].w * inv * gk.w)};
        *reinterpret_cast<f16x4*>(hr) = o;
      } else {
        *reinterpret_cast<float4*>(hr) = make_float4(v[k].x * inv * gk.x, v[k].y * inv * gk.y, v[k].z * inv * gk.z,
                                                     v[k].w * inv * gk.w);
      }
    }
  }
}

template <typename TM, typename TKV>
void GemmKernels<TM, TKV>::qkv(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int d, int hq, int hkv, float scale,
                               const int* row_stream, const int* row_pos, const float2* rope, float* q, TM* qM,
                               TKV* kv, KvLayout L, int layer, const int* page_table, const WTiles& Wt) {
  EpiQKV<TKV> e{hq, hkv, scale, row_stream, row_pos, rope, q, reinterpret_cast<TKV*>(qM), kv, L, layer, page_table};
  run_gemm<TM>(st, ws, A, M, W, d, (hq + 2 * hkv) * 64, e, GemmKind::QKV, false, Wt);
}

template <typename TM, typename TKV>
int GemmKernels<TM, TKV>::qkv_deferred(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int d, int hq,
                                       int hkv, float scale, const int* row_stream, const int* row_pos,
                                       const float2* rope, float* q, TKV* kv, KvLayout L, int layer,
                                       const int* page_table, const WTiles& Wt, const RowNorm& rn) {
  EpiQKV<TKV> e{hq, hkv, scale, row_stream, row_pos, rope, q, nullptr, kv, L, layer, page_table};
  return run_gemm<TM>(st, ws, A, M, W, d, (hq + 2 * hkv) * 64, e, GemmKind::QKV, true, Wt, rn);
}

template <typename TM, typename TKV>
bool GemmKernels<TM, TKV>::norm_fusable(int N) {
  return N % 4 == 0 && N <= 4 * 256 * kNormMaxChunks;
}

template <typename TM, typename TKV>
bool GemmKernels<TM, TKV>::resid(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int K, int N,
                                 float scale, float* x, const float* gain, float eps, TM* h, const WTiles& Wt, float* ss,
                                 int* cnt, int ncnt) {
  EpiResid e{N, scale, x};
  const bool norm = gain != nullptr;
  RowNorm rn;
  if constexpr (sizeof(TM) == 2) {
    if (norm && ss && cnt) {
      rn.cnt = cnt;
      rn.ncnt = ncnt;
      rn.gain = gain;
      rn.y = reinterpret_cast<_Float16*>(h);
      rn.ss_out = ss;
    }
  }
  int fused = 0;
  const int sp = run_gemm<TM>(st, ws, A, M, W, K, N, e, GemmKind::Resid, norm, Wt, rn, &fused);
  if (norm && !fused) k_resid_norm<TM><<<M, 256, 0, st>>>(ws.ptr, sp > 1 ? sp : 0, M, N, scale, x, gain, eps, h, nullptr);
  return fused != 0;
}

template <typename TM, typename TKV>
void GemmKernels<TM, TKV>::rmsnorm(hipStream_t st, int M, float* x, int N, const float* gain, float eps, TM* h,
                                   const int* rows) {
  k_resid_norm<TM><<<M, 256, 0, st>>>(nullptr, 0, M, N, 1.f, x, gain, eps, h, rows);
}

template <typename TM, typename TKV>
void GemmKernels<TM, TKV>::gateup(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int d, int F, float scale,
                                  TM* m, const WTiles& Wt, const RowNorm& rn) {
  // Groups of 32 gate + 32 up columns: every tile width here is a multiple of 64.
  EpiGateUp<TM> e{F, 32, scale, m};
  const int n_cols = ((F + 31) / 32) * 64;
  if constexpr (sizeof(TM) == 2) {
    // (run_gemm scales all of A's rows for a RowNorm request: one launch then.)
    const int first = M > 512 && n_cols >= 8192 && d % 64 == 0 && !rn.ss_in ? gateup_first_rows(M, n_cols, d) : 0;
    if (first > 0) {
      run_gemm<TM>(st, ws, A, first, W, d, n_cols, e, GemmKind::GateUp, false, Wt, rn);
      A += (size_t)first * d;
      e.m += (size_t)first * F;
      M -= first;
    }
  }
  run_gemm<TM>(st, ws, A, M, W, d, n_cols, e, GemmKind::GateUp, false, Wt, rn);
}

template <typename TM, typename TKV>
void GemmKernels<TM, TKV>::logits(hipStream_t st, GemmWorkspace ws, const TM* A, int M, const TM* W, int d, int V, float scale,
                                  float* logits, unsigned long long* slot, const int* row_stream, const WTiles& Wt,
                                  const RowNorm& rn, int slot_row) {
  EpiLogits<false> e{V, scale, logits, slot, row_stream, slot_row, nullptr, 0};
  run_gemm<TM>(st, ws, A, M, W, d, V, e, GemmKind::Logits, false, Wt, rn);
}

// ---------------------------------------------------------------- LM head of many rows

// Final RMSNorm of one row per workgroup, in 64 bits up to the stored value.
// SPLIT: into fp16 high and low parts: row r of x goes to rows 32 (r / 16) +
// r % 16 and + 16 of out, times the power of two that puts its largest value
// in [2^13, 2^14) (row_scale[r]: the inverse); the parts hold a value to 2^-23
// of itself or 2^-38 of the row's largest.  Else into fp32 rows.
template <bool SPLIT, typename TO>
__global__ __launch_bounds__(256) void k_norm_rows(const float* __restrict__ x, int N, const float* __restrict__ gain,
                                                   float eps, TO* __restrict__ out, float* __restrict__ row_scale) {
  __shared__ double red[4];
  __shared__ float redm[4];
  const int row = blockIdx.x;
  const float* xr = x + (size_t)row * N;
  double ss = 0.0;
  for (int k = threadIdx.x; k < N; k += 256) ss += (double)xr[k] * xr[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const double inv = 1.0 / sqrt((red[0] + red[1] + red[2] + red[3]) / N + eps);
  if constexpr (!SPLIT) {
    for (int k = threadIdx.x; k < N; k += 256) out[(size_t)row * N + k] = (TO)(xr[k] * inv * gain[k]);
  } else {
    float mx = 0.f;
    for (int k = threadIdx.x; k < N; k += 256) mx = fmaxf(mx, fabsf((float)(xr[k] * inv * gain[k])));
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) redm[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(redm[0], redm[1]), fmaxf(redm[2], redm[3]));
    int e = 0;  // mx = f 2^e, f in [0.5, 1)
    if (mx > 0.f && mx < INFINITY) (void)frexpf(mx, &e);
    const float up = ldexpf(1.f, min(14 - e, 126));
    if (threadIdx.x == 0) row_scale[row] = 1.f / up;
    TO* hi = out + (size_t)(32 * (row >> 4) + (row & 15)) * N;
    TO* lo = hi + (size_t)16 * N;
    for (int k = threadIdx.x; k < N; k += 256) {
      const double v = xr[k] * inv * gain[k] * up;
      const TO a = (TO)(float)v;
      hi[k] = a;
      lo[k] = (TO)(float)(v - (double)(float)a);
    }
  }
}

// A row's logits were 32-bit products of the row with the weights, one pass
// over the LM head per row (84 us each on the 1B model).  Two fp16 terms per
// value keep that precision on the matrix cores, and the rows share the pass.
// Relative error (2-norm) against 64 bits, one-row head / one MFMA chain per
// sum / sums kept apart from their roundings: bf16 d 2,048 1.21 / 2.82 / 0.66
// 1e-7, d 256 0.94 / 1.25 / 0.71; fp32 d 2,048 0.99 / 7.8 / 0.75, d 256 0.90 /
// 2.9 / 0.81.  200 rows of the 1B head (with the call's ~110 us of other work)
// 16,340 / 319 / 398 us, fp32 31,020 / 1,686 / 1,848 us.
template <typename TM, typename TKV>
void GemmKernels<TM, TKV>::logits_rows(hipStream_t st, const float* x, int M, const float* gain, float eps, TM* rows,
                                       float* row_scale, const TM* W, int d, int V, float scale, float* logits,
                                       unsigned long long* slot, const int* row_stream, int slot_row) {
  if constexpr (sizeof(TM) == 2) {
    _Float16* split = reinterpret_cast<_Float16*>(rows);
    k_norm_rows<true, _Float16><<<M, 256, 0, st>>>(x, d, gain, eps, split, row_scale);
    EpiLogits<true> e{V, scale, logits, slot, row_stream, slot_row, row_scale, M};
    const int n = 32 * ((M + 15) / 16);
    const TileCfg c = fit_tile(GemmKind::Logits, n, V, d, 1);
    const GemmWorkspace none{nullptr, 0};
    const _Float16* Wh = reinterpret_cast<const _Float16*>(W);
    // (256 x 256 tiles leave no registers for the sums.)
    if (c.bm == 256) launch_tile<256, 128>(st, none, split, n, Wh, d, V, 1, e, true);
    else launch_tile<128, 128>(st, none, split, n, Wh, d, V, 1, e, true);
  } else {
    k_norm_rows<false, TM><<<M, 256, 0, st>>>(x, d, gain, eps, rows, nullptr);
    EpiLogits<false> e{V, scale, logits, slot, row_stream, slot_row, nullptr, 0};
    k_gemm<TM, EpiLogits<false>, true><<<dim3((V + GBN - 1) / GBN, (M + GBM - 1) / GBM), 256, 0, st>>>(rows, M, W, d, e);
  }
}

template struct GemmKernels<float, float>;
template struct GemmKernels<_Float16, _Float16>;

}  // namespace hh
