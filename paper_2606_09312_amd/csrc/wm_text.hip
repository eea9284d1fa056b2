// Chunked transformer state encoder (Sec. 3.3): sliding-window chunks of
// each program's token sequence, a post-LayerNorm transformer backbone of the
// CodeBERT (RoBERTa) shape on every chunk, masked mean pooling per chunk, the
// mean over a program's chunks, and a linear projection head to the latent.
//
// All chunks of all programs are one batch of rows, one row per (chunk,
// position).  Head widths 32 and 64 (bf16: windows up to 512) take the packed
// paths: the rows are the chunks' tokens and nothing else, attention is fused
// per (chunk, head), and dense products run on bf16 operands, in float32 as
// six products of three bf16 planes per operand.  Other shapes take the general
// path: every chunk takes `window` rows (positions past its tokens are
// padding: never pooled, masked as attention keys), products in an LDS-tiled
// matrix-core kernel (128 x 128 output tiles, 32-deep stages), attention by the
// same kernel batched over (chunk, head) for the scores and for probabilities
// x values, with a row softmax in between.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "wm_device.h"
#include "wm_internal.h"

using namespace wm;

struct wm_text_model {
  wm_text_dims dims;
  uint8_t* base;
  const float *tok_emb, *pos_emb, *ln0_g, *ln0_b;
  const float *wqkv, *bqkv, *wo, *bo, *ln1_g, *ln1_b, *w1, *b1, *w2, *b2, *ln2_g, *ln2_b;
  const float *wp, *bp;
  // packed paths: the layer matrices as bf16 (WM_FP32: three planes) in the place of the
  // float32 ones, which are then null
  const __bf16 *wqkv16, *wo16, *w116, *w216;
};

namespace wm {
namespace text {

constexpr float LN_EPS = 1e-5f;

// Matrix-core products of the two precisions (32 x 32 output, 16 or 2 deep).
struct BF {
  static constexpr int KF = 16, SL = 8;
  using Elem = __bf16;
  using Frag = bf16x8;
  static __device__ __forceinline__ f32x16 mfma(Frag a, Frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
struct FP {
  static constexpr int KF = 2, SL = 1;
  using Elem = float;
  using Frag = float;
  static __device__ __forceinline__ f32x16 mfma(Frag a, Frag b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m));
  return x;
}

// x as three bf16 planes, x = hi + mid + lo to 2^-24 |x| (each remainder is
// exact in float32): the operand form of the float32 products below.  Past the
// largest bf16 (3.39e38, below the largest float32) hi stays there: rounding to
// infinity would leave no remainder.  NaN and infinities give NaN.
__device__ __forceinline__ void split3(float x, __bf16& hi, __bf16& mid, __bf16& lo) {
  hi = (__bf16)__builtin_amdgcn_fmed3f(x, -0x1.fep127f, 0x1.fep127f);
  const float r = x - (float)hi;
  mid = (__bf16)r;
  lo = (__bf16)(r - (float)mid);
}

// Where element (r, k) of a product operand of `rows` rows lies: slices of 32
// columns, each [rows][32], so that the 32-deep slice of a tile is one
// contiguous range.  In row-major order a slice took 64 bytes from every row:
// half of each cache line, and rows whose pitch is a multiple of 2 KiB (3072
// columns) all in one L2 channel.  Whole batches, ms: float32, 3 programs 5.22 ->
// 4.76 (128 x 64 tiles), bf16, 32 programs 16.19 -> 15.98.
__device__ __forceinline__ size_t op_at(size_t r, int k, size_t rows) {
  return ((size_t)(k >> 5) * rows + r) * 32 + (k & 31);
}

// One LayerNorm output (the same value wherever it is recomputed).
__device__ __forceinline__ float ln_value(float x, float mean, float rs, float g, float b) {
  return fmaf((x - mean) * rs, g, b);
}

// Programs and their chunks (host-built, passed by value).
struct TTable {
  int32_t S;
  int32_t chunk_off[WM_TEXT_MAX_PROGRAMS + 1];   // first chunk of each program
  int32_t tok_off[WM_TEXT_MAX_PROGRAMS + 1];     // first token of each program
  int32_t row_off[WM_TEXT_MAX_PROGRAMS + 1];     // first row of each program
};

__device__ __forceinline__ int program_of(const TTable& tt, int c) {
  int lo = 0, hi = tt.S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tt.chunk_off[mid] <= c) lo = mid; else hi = mid - 1;
  }
  return lo;
}
// First token, token count and first row of chunk c.  A program's chunks are
// `window` rows apart; only its last chunk can hold fewer tokens, and on the
// packed paths the next program's rows follow them directly.
__device__ __forceinline__ void chunk_span(const TTable& tt, int c, int window, int stride,
                                           int& first, int& len, int& row) {
  const int s = program_of(tt, c), k = c - tt.chunk_off[s];
  first = tt.tok_off[s] + k * stride;
  len = min(window, tt.tok_off[s + 1] - first);
  row = tt.row_off[s] + k * window;
}
// Position of row r in its chunk, the chunk's first token and token count.
__device__ __forceinline__ void row_span(const TTable& tt, int r, int window, int stride, int& p, int& first, int& len) {
  int lo = 0, hi = tt.S - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tt.row_off[mid] <= r) lo = mid; else hi = mid - 1;
  }
  const int k = min((r - tt.row_off[lo]) / window, tt.chunk_off[lo + 1] - tt.chunk_off[lo] - 1);
  p = r - tt.row_off[lo] - k * window;
  first = tt.tok_off[lo] + k * stride;
  len = min(window, tt.tok_off[lo + 1] - first);
}

// ---------------------------------------------------------------------------
// Row sums before LayerNorm.  y[r] = tok_emb[id] + pos_emb[p] (padding rows
// zero), then as ln_kernel.  One wavefront per row, lanes over the features.
constexpr int LN_MAX_PER_LANE = 16;               // hidden <= 1024

// LayerNorm of one row held as x[i] = feature lane + 64 i.  Packed paths: writes
// the normalised row as the next product's operand (hb; plane > 0: its three
// planes) and its mean and 1/deviation (stats); the residual path and the pooling recompute the float32
// values from y and those two, so they are never stored (10 -> 6 bytes per
// feature; 68,608 rows of 768: 85 -> 60 us).  General path: writes h.
__device__ __forceinline__ void ln_row(const float (&x)[LN_MAX_PER_LANE], float s, int H, const float* g,
                                       const float* b, size_t r, int rows, float* h, __bf16* hb, size_t plane,
                                       float2* stats) {
  const int lane = threadIdx.x & 63;
  const float mean = wave_sum(s) / (float)H;
  float v = 0.0f;
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i)
    if (lane + 64 * i < H) v = fmaf(x[i] - mean, x[i] - mean, v);
  const float rs = rsqrtf(wave_sum(v) / (float)H + LN_EPS);
  if (stats && lane == 0) stats[r] = make_float2(mean, rs);
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int f = lane + 64 * i;
    if (f < H) {
      const float o = ln_value(x[i], mean, rs, g[f], b[f]);
      const size_t at = op_at(r, f, rows);
      if (plane) split3(o, hb[at], hb[plane + at], hb[2 * plane + at]);
      else if (hb) hb[at] = (__bf16)o;
      else h[r * H + f] = o;
    }
  }
}

__global__ __launch_bounds__(256) void embed_ln_kernel(const int32_t* __restrict__ tokens,
                                                       const TTable tt, int window, int stride,
                                                       const float* __restrict__ tok_emb,
                                                       const float* __restrict__ pos_emb,
                                                       const float* __restrict__ g,
                                                       const float* __restrict__ b, int H, int vocab,
                                                       int rows, float* __restrict__ y, float* __restrict__ h,
                                                       __bf16* __restrict__ hb, size_t plane,
                                                       float2* __restrict__ stats, int32_t* err) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: scalar search
  if (r >= rows) return;
  int p, first, len;
  row_span(tt, r, window, stride, p, first, len);
  if (p >= len) {                                 // general path only: padding
    for (int f = lane; f < H; f += 64) h[(size_t)r * H + f] = 0.0f;
    return;
  }
  int id = tokens[first + p];
  if (id < 0 || id >= vocab) {
    if (lane == 0) atomicOr(err, ERRBIT_TOKEN);
    id = 0;
  }
  float x[LN_MAX_PER_LANE];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int f = lane + 64 * i;
    x[i] = f < H ? tok_emb[(size_t)id * H + f] + pos_emb[(size_t)p * H + f] : 0.0f;
    if (hb && f < H) y[(size_t)r * H + f] = x[i];
    s += x[i];
  }
  ln_row(x, s, H, g, b, r, rows, h, hb, plane, stats);
}

// LN(y[r]) (the residual sum is formed by the product's epilogue).
__global__ __launch_bounds__(256) void ln_kernel(const float* __restrict__ y,
                                                 const float* __restrict__ g,
                                                 const float* __restrict__ b, int H, int rows,
                                                 float* __restrict__ h, __bf16* __restrict__ hb, size_t plane,
                                                 float2* __restrict__ stats) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const float* in = y + (size_t)r * H;
  float x[LN_MAX_PER_LANE];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < LN_MAX_PER_LANE; ++i) {
    const int f = lane + 64 * i;
    x[i] = f < H ? in[f] : 0.0f;
    s += x[i];
  }
  ln_row(x, s, H, g, b, r, rows, h, hb, plane, stats);
}

// ---------------------------------------------------------------------------
// Batched product  C[b] = epi(alpha * A[b] . op(B[b])^T)  with
//   A[b](m, k) = A[offA(b) + m lda + k]
//   B[b](n, k) = B[offB(b) + n ldb + k]          (BT = false)
//              = B[offB(b) + k ldb + n]          (BT = true: stored k-major)
//   off(b) = (b / bdiv) s1 + (b % bdiv) s2
//   epi: + bias[n], then GELU, then + R[offC(b) + m ldr + n] (each optional)
// Workgroup = 4 wavefronts on a 128 x 128 output tile (2 x 2 matrix-core
// tiles each); 32-deep stages staged in LDS with rows of the contraction
// contiguous (one 16-byte LDS read per operand fragment); the next stage's
// loads are in flight during the current stage's products.
struct GemmArgs {
  const float* A;
  const float* B;
  float* C;
  const float* bias;
  const float* res;
  int M, N, K, lda, ldb, ldc, ldr, bdiv, tiles_n;
  long long sA1, sA2, sB1, sB2, sC1, sC2;
  float alpha;
  int gelu;
};
constexpr int GT = 128, GK = 32;

template <class PR, bool BT>
__global__ __launch_bounds__(256) void gemm_kernel(const GemmArgs g) {
  using Elem = typename PR::Elem;
  using Frag = typename PR::Frag;
  constexpr bool BFM = std::is_same<PR, BF>::value;
  constexpr int KF = PR::KF, SL = PR::SL;
  constexpr int LDW = GK + (BFM ? 8 : 4);
  __shared__ __attribute__((aligned(16))) Elem As[GT * LDW];
  __shared__ __attribute__((aligned(16))) Elem Bs[GT * LDW];
  const int bidx = blockIdx.y;
  const long long offA = (long long)(bidx / g.bdiv) * g.sA1 + (long long)(bidx % g.bdiv) * g.sA2;
  const long long offB = (long long)(bidx / g.bdiv) * g.sB1 + (long long)(bidx % g.bdiv) * g.sB2;
  const long long offC = (long long)(bidx / g.bdiv) * g.sC1 + (long long)(bidx % g.bdiv) * g.sC2;
  const float* A = g.A + offA;
  const float* B = g.B + offB;
  const int m0 = (blockIdx.x / g.tiles_n) * GT, n0 = (blockIdx.x % g.tiles_n) * GT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // loaders: row-major operands by (row, 16-deep half), k-major B by (column, 16-deep half)
  const int lr = tid >> 1, lk = (tid & 1) * 16;
  const int bc = tid & (GT - 1), bk = (tid >> 7) * 16;
  float va[16], vb[16];
  auto load = [&](int k0) {
    const bool okA = m0 + lr < g.M;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 x = okA ? *reinterpret_cast<const f32x4*>(A + (size_t)(m0 + lr) * g.lda + k0 + lk + 4 * q)
                          : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < 4; ++i) va[4 * q + i] = x[i];
    }
    if constexpr (!BT) {
      const bool okB = n0 + lr < g.N;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 x = okB ? *reinterpret_cast<const f32x4*>(B + (size_t)(n0 + lr) * g.ldb + k0 + lk + 4 * q)
                            : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < 4; ++i) vb[4 * q + i] = x[i];
      }
    } else {
      const bool okB = n0 + bc < g.N;
#pragma unroll
      for (int j = 0; j < 16; ++j) vb[j] = okB ? B[(size_t)(k0 + bk + j) * g.ldb + n0 + bc] : 0.0f;
    }
  };
  auto store = [&]() {
    Elem* da = As + lr * LDW + lk;
    Elem* db = BT ? Bs + bc * LDW + bk : Bs + lr * LDW + lk;
    if constexpr (BFM) {
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        bf16x8 ea, eb;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          ea[j] = (__bf16)va[8 * h2 + j];
          eb[j] = (__bf16)vb[8 * h2 + j];
        }
        *reinterpret_cast<bf16x8*>(da + 8 * h2) = ea;
        *reinterpret_cast<bf16x8*>(db + 8 * h2) = eb;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<f32x4*>(da + 4 * q) = f32x4{va[4 * q], va[4 * q + 1], va[4 * q + 2], va[4 * q + 3]};
        *reinterpret_cast<f32x4*>(db + 4 * q) = f32x4{vb[4 * q], vb[4 * q + 1], vb[4 * q + 2], vb[4 * q + 3]};
      }
    }
  };

  const int wm = wave & 1, wn = wave >> 1;
  const int cl = lane & 31, h = lane >> 5;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{};
  load(0);
  for (int k0 = 0; k0 < g.K; k0 += GK) {
    __syncthreads();
    store();
    __syncthreads();
    if (k0 + GK < g.K) load(k0 + GK);
#pragma unroll
    for (int ks = 0; ks < GK / KF; ++ks) {
      Frag fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const Elem* pa = As + (wm * 64 + i * 32 + cl) * LDW + ks * KF + h * SL;
        const Elem* pb = Bs + (wn * 64 + i * 32 + cl) * LDW + ks * KF + h * SL;
        fa[i] = *reinterpret_cast<const Frag*>(pa);
        fb[i] = *reinterpret_cast<const Frag*>(pb);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = PR::mfma(fa[i], fb[j], acc[i][j]);
    }
  }
  float* C = g.C + offC;
  const float* R = g.res ? g.res + offC : nullptr;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn * 64 + j * 32 + cl;
      if (n >= g.N) continue;
      const float bn = g.bias ? g.bias[n] : 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + wm * 64 + i * 32 + acc_row(h, r);
        if (m >= g.M) continue;
        float v = fmaf(acc[i][j][r], g.alpha, bn);
        if (g.gelu) v = gelu(v);
        if (R) v += R[(size_t)m * g.ldr + n];
        C[(size_t)m * g.ldc + n] = v;
      }
    }
}

// bf16 dense product with operands stored as bf16 (the product-operand
// values themselves):  C = epi(A . W^T), A [M][K] and W [N][K] in slices
// (op_at), epilogue + bias[n], GELU, + LN(y)[m][n] (the residual, recomputed
// from the previous row sums y, their mean and 1/deviation), C fp32 or bf16
// row-major, or (slices) the bf16 operand of the next product.  With a
// residual C is y itself: each element is read and then written by one lane.
//
// Both kernels stage 32-deep slices of A and W in a ring of four LDS buffers
// by loads straight to LDS, three slices ahead.  A slice row is 64 bytes (four
// 16-byte units); unit u of row r holds contraction unit u ^ ((r >> 2) & 3),
// so that the 16 lanes that the LDS serves together read 16 different bank
// groups.  LDS row 32 j + c of a wavefront's 32 TN columns holds column
// TN c + j: a lane then owns TN neighbouring columns of C and stores them
// together.
struct Gemm16Args {
  const __bf16* A;
  const __bf16* W;
  void* C;
  const float* bias;
  const float* res;        // y, or null
  const float2* stats;     // [M] mean, 1/deviation of y
  const float *ln_g, *ln_b;
  int M, N, K, tiles_n, gelu, slices;
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

// Buffer resource of `bytes` bytes at p (wave-uniform).
__device__ __forceinline__ u32x4 buffer_of(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a),
               (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)),
               (uint32_t)__builtin_amdgcn_readfirstlane(bytes), 0x00020000u};
}
// 16 bytes per lane from byte vo (per lane) of a buffer into LDS at d + lane *
// 16.  Inline assembly, because the compiler otherwise waits
// for every outstanding copy before an LDS read of another slice of the ring;
// the kernels wait for the copies themselves (the instruction has no register
// output, so nothing can be overwritten while it is in flight).  s_nop 4 covers the
// wait of a load on a scalar register that a vector instruction wrote, which the
// compiler does not see here.  m0 is listed
// as clobbered for the compiler's own uses of it; the warning that it is a
// reserved register does not apply to a value nobody keeps there.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy16(u32x4 r, __bf16* d, uint32_t vo) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void*)d);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(l), "v"(vo), "s"(r) : "memory", "m0");
}
#pragma clang diagnostic pop
// Wait until at most VM vector-memory operations are outstanding, and (LGKM)
// for every LDS read.
template <int VM, bool LGKM>
__device__ __forceinline__ void wait_counts() {
  __builtin_amdgcn_s_waitcnt((VM & 15) | (7 << 4) | ((LGKM ? 0 : 15) << 8) | ((VM >> 4) << 14));
}
// Barrier without the waits of __syncthreads; nothing moves across it.
__device__ __forceinline__ void raw_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }
template <int P>
__device__ __forceinline__ void wave_priority() { __builtin_amdgcn_s_setprio(P); }

// Tile of a workgroup: workgroups go to the 8 XCDs in turn, so XCD x takes a
// contiguous run of tiles (columns fastest) and its L2 holds one A panel and W.
__device__ __forceinline__ int xcd_tile(int bid, int total) {
  const int per = total >> 3, rem = total & 7, x = bid & 7, i = bid >> 3;
  return x * per + min(x, rem) + i;
}

// Slice s of a tile's `rows` rows from row r0 of an operand of M rows.
__device__ __forceinline__ u32x4 slice_of(const __bf16* p, int r0, int rows, int M, int s) {
  return buffer_of(p + ((size_t)s * M + r0) * GK, (uint32_t)rows * (GK * 2));
}
// Where thread t's 16-byte unit i of a slice comes from (bytes from the tile's
// first row), rows past the last one clamped to it (their results are dropped).
template <int TN>
__device__ __forceinline__ uint32_t slice_offset(int u, int rows) {
  const int r = u >> 2, s = (u ^ (r >> 2)) & 3;
  const int c = r % (32 * TN), row = TN > 1 ? r - c + TN * (c & 31) + (c >> 5) : r;
  return (uint32_t)min(row, rows - 1) * (GK * 2) + s * 16;
}

// Epilogue of one wavefront: TM x TN tiles at rows m0 + mw, columns n ..
// n + TN - 1 of this lane.  Loads and stores go through buffers that end at
// row M, so rows past it read zero and are not written; the residual of the
// next rows is read while these are written.
template <int TM, int TN, bool OUT16>
__device__ __forceinline__ void gemm16_epilogue(const Gemm16Args& g, const f32x16 (&acc)[TM][TN], int m0, int rows,
                                                int mw, int n, int h) {
  typedef float fv __attribute__((ext_vector_type(TN)));
  constexpr int ES = OUT16 ? 2 : 4;
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(static_cast<uint8_t*>(g.C) + (size_t)m0 * g.N * ES), (short)0, (uint32_t)rows * g.N * ES, 0x00020000);
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(g.res + (g.res ? (size_t)m0 * g.N : 0)), (short)0, g.res ? (uint32_t)rows * g.N * 4 : 0u, 0x00020000);
  if (n >= g.N) return;
  const uint32_t base = (uint32_t)(mw + 4 * h) * g.N + n;
  float bias[TN], lg[TN], lb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    bias[j] = g.bias[n + j];
    if constexpr (!OUT16) {
      lg[j] = g.ln_g[n + j];
      lb[j] = g.ln_b[n + j];
    }
  }
  fv res[2][8];
  u32x2 st[2][8];
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(g.stats + (g.stats ? m0 : 0)), (short)0, g.stats ? (uint32_t)rows * 8u : 0u, 0x00020000);
  // half a tile (8 of a lane's 16 rows) at a time
#pragma unroll
  for (int i = -1; i < 2 * TM; ++i) {
    if constexpr (!OUT16) {
      if (i + 1 < 2 * TM) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const uint32_t row = ((i + 1) >> 1) * 32 + acc_row(0, 8 * ((i + 1) & 1) + r);
          const uint32_t o = (base + row * g.N) * 4;
          if constexpr (TN == 2) res[(i + 1) & 1][r] = __builtin_bit_cast(fv, __builtin_amdgcn_raw_buffer_load_b64(rr, o, 0, 0));
          else res[(i + 1) & 1][r][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rr, o, 0, 0));
          st[(i + 1) & 1][r] = __builtin_amdgcn_raw_buffer_load_b64(rs, (uint32_t)(mw + 4 * h + row) * 8, 0, 0);
        }
      }
    }
    if (i < 0) continue;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t row = (i >> 1) * 32 + acc_row(0, 8 * (i & 1) + r);
      const uint32_t o = base + row * g.N;
      fv v;
#pragma unroll
      for (int j = 0; j < TN; ++j) v[j] = acc[i < 0 ? 0 : i >> 1][j][8 * (i & 1) + r] + bias[j];
      if (g.gelu) {
#pragma unroll
        for (int j = 0; j < TN; ++j) v[j] = gelu_as<OUT16>(v[j]);
      }
      if constexpr (OUT16) {
        typedef __bf16 bv __attribute__((ext_vector_type(TN)));
        bv q;
#pragma unroll
        for (int j = 0; j < TN; ++j) q[j] = (__bf16)v[j];
        if (g.slices) {
          if (mw + 4 * h + (int)row < rows)
            *reinterpret_cast<bv*>(static_cast<__bf16*>(g.C) + op_at((size_t)m0 + mw + 4 * h + row, n, g.M)) = q;
        } else if constexpr (TN == 2) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, q), rc, o * 2, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, q), rc, o * 2, 0, 0);
      } else {
        const float mean = __uint_as_float(st[i & 1][r][0]), inv = __uint_as_float(st[i & 1][r][1]);
#pragma unroll
        for (int j = 0; j < TN; ++j) v[j] += ln_value(res[i & 1][r][j], mean, inv, lg[j], lb[j]);
        if constexpr (TN == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rc, o * 4, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v[0]), rc, o * 4, 0, 0);
      }
    }
  }
}

// Large products: 256 x 256 tiles, 8 wavefronts of 128 x 64, one workgroup per
// compute unit (a 256 x 256 tile is what its registers hold; per product it
// needs the fewest bytes from L2).  The wavefronts are two groups, one of each
// per SIMD, half a step apart: while one group's matrix instructions run, the
// other reads the fragments of its next 16-deep step and issues copies.  Each
// phase ends at a barrier, the second group is one barrier behind.
//
// Slice s + 3 goes into the buffer of slice s - 1 while slice s is read: the
// second group's last reads of slice s - 1 complete one barrier before the
// first group's copies begin.  Slice s + 1 has landed, for all wavefronts,
// before the barrier that ends the second group's last reads of slice s.
//
// Main loop alone 990-1110 TFLOP/s (a register-only loop of these products on
// random operands runs 1870: power); with the epilogue, which HBM bounds,
// M = 64512: N 2304, K 768 (bf16 out) 289 us, 768/768 (fp32 + residual) 141,
// 3072/768 (GELU) 456, 768/3072 377, against 404, 271, 560 and 565 us for one
// 32-deep buffer, two barriers per slice and a register-staged copy.
template <bool OUT16>
__global__ __launch_bounds__(512, 2) void gemm16_large_kernel(const Gemm16Args g) {
  constexpr int TM = 4, TN = 2, BM = 256, BN = 256;
  constexpr int SLICE = (BM + BN) * GK;
  __shared__ __attribute__((aligned(16))) __bf16 S[4 * SLICE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, h = lane >> 5;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  // uniform, so that the slices' buffers are formed by scalar instructions
  const int m0 = __builtin_amdgcn_readfirstlane((t / g.tiles_n) * BM);
  const int n0 = __builtin_amdgcn_readfirstlane((t % g.tiles_n) * BN);
  const int rows = min(BM, g.M - m0), cols = min(BN, g.N - n0);
  const int grp = wave >> 2, wn = wave & 3;
  const int nk = g.K / GK;
  uint32_t oa[2], ob[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    oa[i] = slice_offset<1>(i * 512 + tid, rows);
    ob[i] = slice_offset<TN>(i * 512 + tid, cols);
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x16{};
  bf16x8 fa[TM], fb[TN];
  const int sw = (cl >> 2) & 3;
  auto frags = [&](int s, int ks) {
    const __bf16* a = S + (s & 3) * SLICE + cl * GK + ((2 * ks + h) ^ sw) * 8;
#pragma unroll
    for (int j = 0; j < TN; ++j)
      fb[j] = *reinterpret_cast<const bf16x8*>(a + (BM + (wn * TN + j) * 32) * GK);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(a + (grp * TM + i) * 32 * GK);
  };
  auto products = [&]() {
    wave_priority<1>();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = BF::mfma(fa[i], fb[j], acc[i][j]);
    wave_priority<0>();
  };
  auto copyA = [&](int s) {
    __bf16* d = S + (s & 3) * SLICE + wave * 512;
    const u32x4 ra = slice_of(g.A, m0, rows, g.M, s);
    copy16(ra, d, oa[0]);
    copy16(ra, d + 4096, oa[1]);
  };
  auto copyB = [&](int s) {
    __bf16* d = S + (s & 3) * SLICE + BM * GK + wave * 512;
    const u32x4 rb = slice_of(g.W, n0, cols, g.N, s);
    copy16(rb, d, ob[0]);
    copy16(rb, d + 4096, ob[1]);
  };
  for (int s = 0; s < 3 && s < nk; ++s) { copyA(s); copyB(s); }
  if (nk >= 3) wait_counts<8, false>(); else wait_counts<0, false>();
  raw_barrier();
  if (grp) raw_barrier();
  for (int s = 0; s < nk; ++s) {
    const bool more = s + 3 < nk;
    frags(s, 0);
    if (more) copyA(s + 3);
    wait_counts<63, true>();
    raw_barrier();
    products();
    raw_barrier();
    frags(s, 1);
    if (more) { copyB(s + 3); wait_counts<8, true>(); } else wait_counts<0, true>();
    raw_barrier();
    products();
    raw_barrier();
  }
  if (!grp) raw_barrier();
  gemm16_epilogue<TM, TN, OUT16>(g, acc, m0, rows, grp * 128, n0 + wn * 64 + TN * cl, h);
}

// Products with too few 256 x 256 tiles to fill the chip: tiles of 64 WM x
// 64 rows and columns (WM = 2: 128 x 64, WM = 1: 64 x 64), 4 wavefronts of
// 32 WM x 32, several workgroups per compute unit.  One barrier per slice:
// slice s has landed and every wavefront has consumed slice s - 1, whose
// buffer is then filled with slice s + 3.
template <int WM, bool OUT16>
__global__ __launch_bounds__(256, 2) void gemm16_small_kernel(const Gemm16Args g) {
  constexpr int BM = 64 * WM, BN = 64, UA = WM, ND = UA + 1;
  constexpr int SLICE = (BM + BN) * GK;
  __shared__ __attribute__((aligned(16))) __bf16 S[4 * SLICE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, h = lane >> 5;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  // uniform, so that the slices' buffers are formed by scalar instructions
  const int m0 = __builtin_amdgcn_readfirstlane((t / g.tiles_n) * BM);
  const int n0 = __builtin_amdgcn_readfirstlane((t % g.tiles_n) * BN);
  const int rows = min(BM, g.M - m0), cols = min(BN, g.N - n0);
  const int wm = wave & 1, wn = wave >> 1;
  const int nk = g.K / GK;
  uint32_t oa[UA];
#pragma unroll
  for (int i = 0; i < UA; ++i) oa[i] = slice_offset<1>(i * 256 + tid, rows);
  const uint32_t ob = slice_offset<1>(tid, cols);
  f32x16 acc[WM][1];
#pragma unroll
  for (int i = 0; i < WM; ++i) acc[i][0] = f32x16{};
  const int sw = (cl >> 2) & 3;
  auto copy = [&](int s) {
    __bf16* d = S + (s & 3) * SLICE + wave * 512;
    const u32x4 ra = slice_of(g.A, m0, rows, g.M, s), rb = slice_of(g.W, n0, cols, g.N, s);
#pragma unroll
    for (int i = 0; i < UA; ++i) copy16(ra, d + i * 2048, oa[i]);
    copy16(rb, d + BM * GK, ob);
  };
  for (int s = 0; s < 3 && s < nk; ++s) copy(s);
  for (int s = 0; s < nk; ++s) {
    if (s + 2 < nk) wait_counts<2 * ND, true>(); else wait_counts<0, true>();
    raw_barrier();
    if (s + 3 < nk) copy(s + 3);
    const __bf16* base = S + (s & 3) * SLICE + cl * GK;
    bf16x8 fa[2][WM], fb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const __bf16* a = base + ((2 * ks + h) ^ sw) * 8;
      fb[ks] = *reinterpret_cast<const bf16x8*>(a + (BM + wn * 32) * GK);
#pragma unroll
      for (int i = 0; i < WM; ++i) fa[ks][i] = *reinterpret_cast<const bf16x8*>(a + (wm * WM + i) * 32 * GK);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < WM; ++i) acc[i][0] = BF::mfma(fa[ks][i], fb[ks], acc[i][0]);
  }
  gemm16_epilogue<WM, 1, OUT16>(g, acc, m0, rows, wm * 32 * WM, n0 + wn * 32 + cl, h);
}

// Row softmax of the attention scores, keys past the chunk's tokens masked.
// One wavefront per row (chunk c, head, query); in place.
constexpr int SM_MAX_PER_LANE = 16;               // window <= 1024
__global__ __launch_bounds__(256) void softmax_kernel(float* __restrict__ s, const TTable tt,
                                                      int window, int stride, int heads,
                                                      long long rows) {
  const int lane = threadIdx.x & 63;
  const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int c = (int)(r / ((long long)heads * window));
  int first, len, row0;
  chunk_span(tt, c, window, stride, first, len, row0);
  float* row = s + r * window;
  float x[SM_MAX_PER_LANE];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < SM_MAX_PER_LANE; ++i) {
    const int k = lane + 64 * i;
    x[i] = (k < window && k < len) ? row[k] : -INFINITY;
    mx = fmaxf(mx, x[i]);
  }
  mx = wave_max(mx);
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < SM_MAX_PER_LANE; ++i) {
    x[i] = x[i] == -INFINITY ? 0.0f : __expf(x[i] - mx);
    sum += x[i];
  }
  const float inv = 1.0f / wave_sum(sum);
#pragma unroll
  for (int i = 0; i < SM_MAX_PER_LANE; ++i) {
    const int k = lane + 64 * i;
    if (k < window) row[k] = x[i] * inv;
  }
}

// Fused attention of one (chunk, head) per workgroup, bf16: wavefront w
// takes queries [32 w, 32 w + 32).  K and V of the chunk are staged in LDS
// once (K row-major, V transposed with its keys permuted into accumulator
// order); the scores are computed transposed, S^T = K . Q^T, so a query is a
// lane's column and its softmax statistics are per-lane values completed across
// the lane pair (L, L^32).  Pass 1 finds the row maximum; pass 2 recomputes the
// scores (matrix instructions have room: the vector unit is what bounds this
// kernel), forms p = exp(s - max), rounds it as the product operand,
// accumulates O^T = V^T . P with P straight from the accumulators (its key
// order is the one V was permuted into) and sums p; O is divided by the sum
// at the end.  One exponential per score instead of two, and keys are masked
// in the last 32-key block only: 68,608 rows, 12 heads of 64: 324 -> 184 us.
__device__ __forceinline__ float exp2_of(float x) { return __builtin_amdgcn_exp2f(x); }
template <int DH>
__global__ __launch_bounds__(1024) void attention_kernel(const __bf16* __restrict__ qkv,
                                                         __bf16* __restrict__ ctx, const TTable tt,
                                                         int window, int stride, int heads, int H, int rows,
                                                         float scale) {
  constexpr int KS = DH / 16;                 // 16-deep steps over the head width
  constexpr int DB = DH / 32;                 // 32-row blocks of the head width
  constexpr int KW = DH + 8;                  // padded K row (bf16)
  extern __shared__ __attribute__((aligned(16))) __bf16 lds_att[];
  const int VW = window + 8;                  // padded V^T row (bf16)
  __bf16* Ks = lds_att;                       // [window][KW]
  __bf16* Vt = lds_att + (size_t)window * KW; // [DH][VW]
  const int c = blockIdx.x / heads, head = blockIdx.x % heads;
  int first, len, row0;
  chunk_span(tt, c, window, stride, first, len, row0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nt = blockDim.x;
  const int cl = lane & 31, h = lane >> 5;
  const __bf16* base = qkv + (size_t)row0 * 3 * H + head * DH;
  const int nkb = (len + 31) / 32;

  // stage K (row-major) and V (transposed, keys in accumulator order per block)
  for (int u = tid; u < nkb * 32 * (DH / 8); u += nt) {
    const int key = u / (DH / 8), d8 = (u % (DH / 8)) * 8;
    bf16x8 kv = {}, vv = {};
    if (key < len) {
      kv = *reinterpret_cast<const bf16x8*>(base + (size_t)key * 3 * H + H + d8);
      vv = *reinterpret_cast<const bf16x8*>(base + (size_t)key * 3 * H + 2 * H + d8);
    }
    *reinterpret_cast<bf16x8*>(Ks + key * KW + d8) = kv;
    // key = 32 kb + acc_row(hh, 8 f + j)  ->  position 32 kb + 16 f + 8 hh + j
    const int kb = key >> 5, kr = key & 31;
    const int hh = (kr >> 2) & 1, rr = ((kr >> 3) << 2) | (kr & 3);
    const int pos = kb * 32 + (rr >> 3) * 16 + hh * 8 + (rr & 7);
#pragma unroll
    for (int i = 0; i < 8; ++i) Vt[(d8 + i) * VW + pos] = vv[i];
  }
  // this wavefront's queries as B operands: Q[q][16 kk + 8 h + j]
  const int q = wave * 32 + cl;
  bf16x8 qf[KS];
  {
    const __bf16* qrow = base + (size_t)min(q, len - 1) * 3 * H;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + 16 * kk + 8 * h);
  }
  __syncthreads();
  if (wave * 32 >= len) return;               // no valid query in this wavefront

  auto scores = [&](int kb) -> f32x16 {
    f32x16 sacc = {};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const bf16x8 kfrag = *reinterpret_cast<const bf16x8*>(Ks + (kb * 32 + cl) * KW + 16 * kk + 8 * h);
      sacc = BF::mfma(kfrag, qf[kk], sacc);
    }
    return sacc;
  };
  // pass 1: the maximum score over the valid keys (the chunk's last block may
  // hold fewer than 32)
  const int nfull = len / 32;
  float mx = -INFINITY;
  for (int kb = 0; kb < nfull; ++kb) {
    const f32x16 sacc = scores(kb);
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
  }
  if (nfull < nkb) {
    const f32x16 sacc = scores(nfull);
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (nfull * 32 + acc_row(h, r) < len) mx = fmaxf(mx, sacc[r]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  // pass 2: p = exp((s - max) scale) as 2^(s c - max c), O^T += V^T . P, sum of p
  const float c2 = scale * 1.4426950408889634f, mc = mx * c2;
  float sum = 0.0f;
  f32x16 oacc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) oacc[b] = f32x16{};
  auto block = [&](int kb, bool last) {
    const f32x16 sacc = scores(kb);
    bf16x8 pf[2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = 8 * f + j;
        float pv = exp2_of(fmaf(sacc[r], c2, -mc));
        if (last) pv = kb * 32 + acc_row(h, r) < len ? pv : 0.0f;
        sum += pv;
        pf[f][j] = (__bf16)pv;
      }
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const bf16x8 vfrag = *reinterpret_cast<const bf16x8*>(Vt + (b * 32 + cl) * VW + kb * 32 + 16 * f + 8 * h);
        oacc[b] = BF::mfma(vfrag, pf[f], oacc[b]);
      }
  };
  for (int kb = 0; kb < nfull; ++kb) block(kb, false);
  if (nfull < nkb) block(nfull, true);
  const float inv = 1.0f / (sum + __shfl_xor(sum, 32));
  if (q < len) {                // the output as the next product's operand
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const size_t orow = (size_t)row0 + q;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (__bf16)(oacc[b][4 * r4 + i] * inv);
        *reinterpret_cast<bf16x4*>(ctx + op_at(orow, head * DH + 32 * b + 8 * r4 + 4 * h, rows)) = o;
      }
  }
}

// float32 dense product on the bf16 matrix cores: both operands as three bf16
// planes (split3), C = sum of the six plane products that matter
// (hi hi; hi mid, mid hi, hi lo, mid mid, lo hi: what is left out is below
// 2^-25 of |a||b|), the five small ones in an accumulator of their own.  Six
// bf16 products take 96 cycles per 16x16x32 where float32 ones take 256.  Its
// distance from float64 over the encoder equals that of the float32 products
// (5e-7).
//
// Tiles are 64 x 64, slices of 32 in a ring of three, and 8 wavefronts in two
// groups: group kg takes the 16-deep half kg of every slice, and the groups' sums
// are added through LDS at the end, each group finishing half of the rows.  With
// two workgroups per compute unit that is four wavefronts per SIMD.  A slice's
// fragments are read while the products of the slice before run.  Copies from
// L2 bound it (64,263 rows: matrix cores 44% of the SIMD cycles, 29 bytes per clock
// and compute unit from L2, the rest of the time waiting): operands in slices (op_at)
// took the products of 2400 rows of 768 columns from 3.74 to 3.37 ms over 12 layers.
// 128 x 64 tiles, which read a quarter fewer bytes from LDS but leave two
// wavefronts per SIMD, are slower (encoder calls, 64 / 128 rows, ms: 300 rows 1.83
// / 1.91, 1200 2.69 / 2.76, 1600 3.33 / 3.61, 2000 3.79 / 4.12).  A call of 2400 rows, with
// 4 wavefronts on 64 x 64 tiles of row-major operands, then this kernel: 5.22, 4.65
// ms.
struct Gemm3Args {
  const __bf16 *A, *W;      // planes a_plane, w_plane elements apart
  void* C;                  // float32, or planes c_plane elements apart
  const float* bias;
  const float* res;         // y (then C is y), or null
  const float2* stats;
  const float *ln_g, *ln_b;
  size_t a_plane, w_plane, c_plane;
  int M, N, K, tiles_n, gelu;
};
template <bool SPLIT_OUT>
__global__ __launch_bounds__(512, 4) void gemm16x3_kernel(const Gemm3Args g) {
  constexpr int BM = 64, BN = 64, PL = BM * GK, SLICE = 6 * PL;   // planes: A hi, mid, lo, W hi, mid, lo
  constexpr int NR = 8;                         // rows that a lane finishes
  __shared__ __attribute__((aligned(16))) __bf16 S[3 * SLICE];
  static_assert(4 * NR * 256 * 4 <= sizeof(S), "the groups' exchange takes the ring's place");
  const int tid = threadIdx.x, lane = tid & 63, q = tid & 255;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, h = lane >> 5;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  // uniform, so that the slices' buffers are formed by scalar instructions
  const int m0 = __builtin_amdgcn_readfirstlane((t / g.tiles_n) * BM);
  const int n0 = __builtin_amdgcn_readfirstlane((t % g.tiles_n) * BN);
  const int rows = min(BM, g.M - m0), cols = min(BN, g.N - n0);
  const int kg = wave >> 2, wm = wave & 1, wn = (wave >> 1) & 1;
  const int nk = g.K / GK;
  const uint32_t oa = slice_offset<1>(q, rows), ob = slice_offset<1>(q, cols);
  // a plane is 256 units: group 0 copies A, group 1 W
  auto copy = [&](int s, int b) {
    __bf16* d = S + b * SLICE + (wave & 3) * 512;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (kg == 0) copy16(slice_of(g.A + p * g.a_plane, m0, rows, g.M, s), d + p * PL, oa);
      else copy16(slice_of(g.W + p * g.w_plane, n0, cols, g.N, s), d + (3 + p) * PL, ob);
    }
  };
  // at most `slices` slices' copies of this wavefront outstanding, LDS reads done
  auto wait = [&](int slices) {
    if (slices == 0) wait_counts<0, true>();
    else if (slices == 1) wait_counts<3, true>();
    else wait_counts<6, true>();
  };
  const int fo = cl * GK + (((2 * kg + h) ^ (cl >> 2)) & 3) * 8;
  struct Frags { bf16x8 a[3], b[3]; };
  auto read = [&](int b, Frags& f) {
    const __bf16* base = S + b * SLICE + fo;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      f.a[p] = *reinterpret_cast<const bf16x8*>(base + p * PL + wm * 32 * GK);
      f.b[p] = *reinterpret_cast<const bf16x8*>(base + (3 + p) * PL + wn * 32 * GK);
    }
  };
  f32x16 hi = {}, lo = {};
  auto products = [&](const Frags& f) {
    hi = BF::mfma(f.a[0], f.b[0], hi);
    lo = BF::mfma(f.a[2], f.b[0], lo);
    lo = BF::mfma(f.a[1], f.b[1], lo);
    lo = BF::mfma(f.a[0], f.b[2], lo);
    lo = BF::mfma(f.a[1], f.b[0], lo);
    lo = BF::mfma(f.a[0], f.b[1], lo);
  };
  // Step s multiplies slice s from registers, reads slice s + 1 and copies slice
  // s + 3 into slice s's buffer, which every wavefront has read by the barrier;
  // slice s + 1 has landed by then, slice s + 2 may be in flight.
  int cur = 0;                                   // buffer of slice s
  auto step = [&](int s, const Frags& now, Frags& next) {
    wait(s + 2 < nk ? 1 : 0);
    raw_barrier();
    if (s + 3 < nk) copy(s + 3, cur);
    cur = cur == 2 ? 0 : cur + 1;
    if (s + 1 < nk) read(cur, next);
    sched_fence();
    products(now);
  };
  Frags f0, f1;
  copy(0, 0);
  if (nk > 1) copy(1, 1);
  if (nk > 2) copy(2, 2);
  wait(nk > 2 ? 2 : nk > 1 ? 1 : 0);
  raw_barrier();
  read(0, f0);
  for (int s = 0; s < nk; s += 2) {
    step(s, f0, f1);
    if (s + 1 < nk) step(s + 1, f1, f0);
  }
  // the groups' sums: each hands over the half of the lane's 16 rows that the other
  // finishes (group kg: half kg)
  float* x = reinterpret_cast<float*>(S);        // [group][hi, lo][NR][256]
  __syncthreads();                               // the ring has been read
  float vh[NR], vl[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float h0 = hi[r], h1 = hi[8 + r], l0 = lo[r], l1 = lo[8 + r];
    vh[r] = kg ? h1 : h0;
    vl[r] = kg ? l1 : l0;
    x[((kg * 2 + 0) * NR + r) * 256 + q] = kg ? h0 : h1;
    x[((kg * 2 + 1) * NR + r) * 256 + q] = kg ? l0 : l1;
  }
  __syncthreads();
  const int n = n0 + wn * 32 + cl;
  if (n >= g.N) return;
  const float bias = g.bias[n];
  const float lg = g.res ? g.ln_g[n] : 0.0f, lb = g.res ? g.ln_b[n] : 0.0f;
  const int mt = m0 + wm * 32 + kg * 16 + 4 * h;
  float y[NR];
  float2 st[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int m = min(mt + acc_row(0, r), g.M - 1);
    y[r] = g.res ? g.res[(size_t)m * g.N + n] : 0.0f;
    st[r] = g.res ? g.stats[m] : make_float2(0.0f, 0.0f);
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int m = mt + acc_row(0, r);
    if (m >= g.M) continue;
    const float sh = vh[r] + x[(((kg ^ 1) * 2 + 0) * NR + r) * 256 + q];
    const float sl = vl[r] + x[(((kg ^ 1) * 2 + 1) * NR + r) * 256 + q];
    float v = (sh + sl) + bias;
    if (g.gelu) v = gelu(v);
    if (g.res) v += ln_value(y[r], st[r].x, st[r].y, lg, lb);
    if constexpr (SPLIT_OUT) {
      __bf16* c = static_cast<__bf16*>(g.C) + op_at(m, n, g.M);
      split3(v, c[0], c[g.c_plane], c[2 * g.c_plane]);
    } else {
      static_cast<float*>(g.C)[(size_t)m * g.N + n] = v;
    }
  }
}

// n float32 values, matrices [N][K] one after another, as `planes` bf16 planes
// (1: rounded; 3: split3), n apart, every matrix in slices.
__global__ __launch_bounds__(256) void split_planes_kernel(const float* __restrict__ src, size_t n, int N, int K,
                                                           int planes, __bf16* __restrict__ dst) {
  for (size_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const size_t row = i / K, l = row / N;
    const size_t o = l * N * K + op_at(row - l * N, (int)(i - row * K), N);
    if (planes == 1) dst[o] = (__bf16)src[i];
    else split3(src[i], dst[o], dst[n + o], dst[2 * n + o]);
  }
}

// Fused float32 attention of one (chunk, head) and 128 queries: wavefront w
// takes queries 32 w .. of the block; keys in blocks of 64, staged in LDS (K and
// V row-major), softmax online.  S^T = K . Q^T on the float32 matrix cores with
// the contraction enumerated half by half (a lane half reads its 32 features
// in 16-byte pieces), so a query is a lane's column; P stays in the
// accumulators, whose key order V's rows are read in.  Row strides keep both
// reads off shared banks.  Replaces score matrices in memory, a softmax pass
// and two batched products (150 us per layer at 2400 rows).
template <int DH>
__global__ __launch_bounds__(256, 2) void attention32_kernel(const float* __restrict__ qkv,
                                                             __bf16* __restrict__ ctx, size_t plane,
                                                             const TTable tt, int window, int stride, int heads,
                                                             int H, int rows, float scale) {
  constexpr int KB = 64, DB = DH / 32, HS = DH / 2;     // keys per block, 32-feature blocks, features per lane half
  constexpr int KW = DH + 4, VW = DH + 8;
  __shared__ __attribute__((aligned(16))) float Ks[KB * KW];
  __shared__ __attribute__((aligned(16))) float Vs[KB * VW];
  const int c = blockIdx.x / heads, head = blockIdx.x % heads;
  int first, len, row0;
  chunk_span(tt, c, window, stride, first, len, row0);
  const int q0 = blockIdx.y * 128;
  if (q0 >= len) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cl = lane & 31, h = lane >> 5;
  const float* base = qkv + (size_t)row0 * 3 * H + head * DH;
  const int q = q0 + wave * 32 + cl;
  // scores in units of log2: exp(s scale) = 2^(s scale log2 e)
  const float c2 = scale * 1.4426950408889634f;
  float qf[HS];
  {
    const float* qrow = base + (size_t)min(q, len - 1) * 3 * H + h * HS;
#pragma unroll
    for (int i = 0; i < HS; i += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(qrow + i);
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[i + j] = v[j];
    }
  }
  f32x16 oacc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) oacc[b] = f32x16{};
  float mx = -INFINITY, sum = 0.0f;
  constexpr int NU = KB * (DH / 4) / 256;              // 16-byte units per thread and matrix
  f32x4 kn[NU], vn[NU];                                // the next block, loaded under this one's products
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const int u = tid + 256 * i, key = u / (DH / 4), d4 = (u % (DH / 4)) * 4;
      const float* src = base + (size_t)min(k0 + key, len - 1) * 3 * H + d4;   // keys past the end are masked
      kn[i] = *reinterpret_cast<const f32x4*>(src + H);
      vn[i] = *reinterpret_cast<const f32x4*>(src + 2 * H);
    }
  };
  load(0);
  for (int k0 = 0; k0 < len; k0 += KB) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NU; ++i) {
      const int u = tid + 256 * i, key = u / (DH / 4), d4 = (u % (DH / 4)) * 4;
      *reinterpret_cast<f32x4*>(Ks + key * KW + d4) = kn[i];
      *reinterpret_cast<f32x4*>(Vs + key * VW + d4) = vn[i];
    }
    __syncthreads();
    if (k0 + KB < len) load(k0 + KB);
#pragma unroll
    for (int kb = 0; kb < KB / 32; ++kb) {
      const int kbase = k0 + 32 * kb;
      if (kbase >= len) break;
      f32x16 s = {};
#pragma unroll
      for (int i = 0; i < HS; i += 4) {
        const f32x4 kf = *reinterpret_cast<const f32x4*>(Ks + (32 * kb + cl) * KW + h * HS + i);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float a = kf[j];
          s = FP::mfma(a, qf[i + j], s);
        }
      }
      float bm = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = kbase + acc_row(h, r) < len ? s[r] * c2 : -INFINITY;
        bm = fmaxf(bm, s[r]);
      }
      bm = fmaxf(bm, __shfl_xor(bm, 32));
      const float nm = fmaxf(mx, bm);
      const float at = nm == -INFINITY ? 0.0f : nm;   // only keys of weight 0 so far (scores that overflowed)
      const float f = exp2_of(mx - at);        // 0 at the first block
      float bs = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = exp2_of(s[r] - at);
        bs += s[r];
      }
      sum = fmaf(sum, f, bs);
      mx = nm;
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] *= f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = s[r];
#pragma unroll
        for (int b = 0; b < DB; ++b)
          oacc[b] = FP::mfma(Vs[(32 * kb + acc_row(h, r)) * VW + 32 * b + cl], p, oacc[b]);
      }
    }
  }
  const float inv = 1.0f / (sum + __shfl_xor(sum, 32));
  if (q < len) {
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        __bf16* o = ctx + op_at((size_t)row0 + q, head * DH + 32 * b, rows);
        const int d = acc_row(h, r);
        split3(oacc[b][r] * inv, o[d], o[plane + d], o[2 * plane + d]);
      }
  }
}

// Masked mean over a chunk's tokens: one workgroup per chunk; thread t sums
// the feature quad t % (H/4) over the tokens p = t / (H/4) + k G (G token
// groups, 16-byte loads), then the G partial sums are added in group order.
// Packed paths (stats given): the rows are LN(y), recomputed as they are read.
constexpr int POOL_THREADS = 1024;
__global__ __launch_bounds__(POOL_THREADS) void pool_kernel(const float* __restrict__ h, const float2* __restrict__ stats,
                                                            const float* __restrict__ ln_g,
                                                            const float* __restrict__ ln_b, const TTable tt,
                                                            int window, int stride, int H,
                                                            float* __restrict__ pooled) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  __shared__ f4 part[POOL_THREADS];
  const int c = blockIdx.x, tid = threadIdx.x;
  int first, len, row0;
  chunk_span(tt, c, window, stride, first, len, row0);
  const float inv = 1.0f / (float)len;
  const int nq = H / 4, groups = POOL_THREADS / nq;        // H <= 1024: at least 4 groups
  const int q = tid % nq, grp = tid / nq;
  f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  if (grp < groups) {
    const f4* base = reinterpret_cast<const f4*>(h + (size_t)row0 * H) + q;
    if (stats) {
      const f4 g = reinterpret_cast<const f4*>(ln_g)[q], b = reinterpret_cast<const f4*>(ln_b)[q];
      for (int p = grp; p < len; p += groups) {
        const f4 x = base[(size_t)p * nq];
        const float2 st = stats[row0 + p];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += ln_value(x[i], st.x, st.y, g[i], b[i]);
      }
    } else {
      for (int p = grp; p < len; p += groups) acc += base[(size_t)p * nq];
    }
  }
  part[tid] = acc;
  __syncthreads();
  if (tid < nq) {
    f4 t = part[tid];
    for (int g2 = 1; g2 < groups; ++g2) t += part[g2 * nq + tid];
    *reinterpret_cast<f4*>(pooled + (size_t)c * H + 4 * tid) = t * inv;
  }
}

// Program vector (mean of its chunk vectors; zero for an empty program, as
// a product operand) and z = Wp v + bp.  One workgroup per program.
__global__ __launch_bounds__(256) void project_kernel(const float* __restrict__ pooled,
                                                      const TTable tt, int H, int d,
                                                      const float* __restrict__ wp,
                                                      const float* __restrict__ bp, int bf16,
                                                      float* __restrict__ z) {
  extern __shared__ float v[];
  const int s = blockIdx.x;
  const int c0 = tt.chunk_off[s], c1 = tt.chunk_off[s + 1];
  const float inv = c1 > c0 ? 1.0f / (float)(c1 - c0) : 0.0f;
  for (int f = threadIdx.x; f < H; f += blockDim.x) {
    float a = 0.0f;
    for (int c = c0; c < c1; ++c) a += pooled[(size_t)c * H + f];
    a *= inv;
    v[f] = bf16 ? (float)(__bf16)a : a;
  }
  __syncthreads();
  for (int o = threadIdx.x; o < d; o += blockDim.x) {
    float a = bp[o];
    for (int f = 0; f < H; ++f) a = fmaf(wp[(size_t)o * H + f], v[f], a);
    z[(size_t)s * d + o] = a;
  }
}

}  // namespace text
}  // namespace wm

using namespace wm::text;

namespace {

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

int n_chunks_of(int n_tokens, int window, int stride) {
  if (n_tokens <= 0) return 0;
  if (n_tokens <= window) return 1;
  return 1 + (n_tokens - window + stride - 1) / stride;
}

// Packed paths: rows of tokens only, products on bf16 operands (float32: three
// planes of them) and fused attention, whose head widths and (bf16) window
// these are.  Everything else takes the general path.
bool packed_path(const wm_text_dims& d) {
  const int dh = d.hidden / d.heads;
  return (dh == 32 || dh == 64) && (d.precision == WM_FP32 || d.window <= 512);
}

struct TextLayout {
  size_t err, h, qkv, sc, ctx, y, f, pooled, hb, qkvb, ctxb, fb, stats, total;
};

TextLayout text_layout(const wm_text_dims& dm, int n_chunks) {
  const size_t rows = (size_t)n_chunks * dm.window, H = dm.hidden;
  const bool bf = packed_path(dm), f32 = bf && dm.precision == WM_FP32;
  const size_t pb = f32 ? 6 : 2;             // bytes of a product operand
  TextLayout L;
  size_t o = 0;
  L.err = o; o += 256;
  L.h = o; o = al256(o + (bf ? 0 : rows * H * 4));
  L.qkv = o; o = al256(o + (bf && !f32 ? 0 : rows * 3 * H * 4));
  L.sc = o; o = al256(o + (bf ? 0 : (size_t)n_chunks * dm.heads * dm.window * dm.window * 4));
  L.ctx = o; o = al256(o + (bf ? 0 : rows * H * 4));
  L.y = o; o = al256(o + rows * H * 4);
  L.f = o; o = al256(o + (bf ? 0 : rows * (size_t)dm.ffn * 4));
  L.pooled = o; o = al256(o + (size_t)n_chunks * H * 4);
  // packed paths: the product operands and the rows' LayerNorm statistics (the
  // float32 h, scores, context and hidden buffers above, and in bf16 qkv, are
  // then unused and sized zero)
  L.hb = o; o = al256(o + (bf ? rows * H * pb : 0));
  L.qkvb = o; o = al256(o + (bf && !f32 ? rows * 3 * H * 2 : 0));
  L.ctxb = o; o = al256(o + (bf ? rows * H * pb : 0));
  L.fb = o; o = al256(o + (bf ? rows * (size_t)dm.ffn * pb : 0));
  L.stats = o; o = al256(o + (bf ? rows * 8 : 0));
  L.total = o;
  return L;
}

template <class PR>
hipError_t launch_gemm(const GemmArgs& g0, int batch, bool bt, hipStream_t st) {
  GemmArgs g = g0;
  g.tiles_n = (g.N + GT - 1) / GT;
  const dim3 grid(((g.M + GT - 1) / GT) * g.tiles_n, batch);
  if (bt) hipLaunchKernelGGL((gemm_kernel<PR, true>), grid, dim3(256), 0, st, g);
  else hipLaunchKernelGGL((gemm_kernel<PR, false>), grid, dim3(256), 0, st, g);
  return hipGetLastError();
}

GemmArgs dense(const float* A, int M, int K, const float* W, int N, float* C, const float* bias,
               const float* res, int gelu) {
  GemmArgs g{};
  g.A = A; g.B = W; g.C = C; g.bias = bias; g.res = res;
  g.M = M; g.N = N; g.K = K; g.lda = K; g.ldb = K; g.ldc = N; g.ldr = N; g.bdiv = 1;
  g.alpha = 1.0f; g.gelu = gelu;
  return g;
}

}  // namespace

extern "C" {

wm_status wm_text_model_create(const wm_text_dims* dims, const wm_text_weights* w, wm_text_model** out) {
  if (!dims || !w || !out) return set_error(WM_ERR_INVALID_ARGUMENT, "null argument");
  *out = nullptr;
  const wm_text_dims& d = *dims;
  if (d.vocab < 1 || d.hidden < 1 || d.heads < 1 || d.ffn < 1 || d.layers < 0 || d.window < 1 ||
      d.stride < 1 || d.stride > d.window || d.d < 1)
    return set_error(WM_ERR_INVALID_ARGUMENT, "dims must be positive with 1 <= stride <= window");
  if (d.precision != WM_FP32 && d.precision != WM_BF16)
    return set_error(WM_ERR_INVALID_ARGUMENT, "unknown precision");
  if (d.hidden % d.heads || (d.hidden / d.heads) % 32 || d.hidden % 32 || d.ffn % 32 || d.window % 32 ||
      d.hidden > 64 * LN_MAX_PER_LANE || d.window > 64 * SM_MAX_PER_LANE)
    return set_error(WM_ERR_UNSUPPORTED,
                     "need hidden, ffn, window and the head width multiples of 32, hidden <= 1024, window <= 1024");
  const float* req[] = {w->tok_emb, w->pos_emb, w->ln0_g, w->ln0_b, w->wp, w->bp};
  for (const float* p : req)
    if (!p) return set_error(WM_ERR_INVALID_ARGUMENT, "null weight pointer");
  if (d.layers > 0) {
    const float* lreq[] = {w->wqkv, w->bqkv, w->wo, w->bo, w->ln1_g, w->ln1_b, w->w1, w->b1, w->w2,
                           w->b2, w->ln2_g, w->ln2_b};
    for (const float* p : lreq)
      if (!p) return set_error(WM_ERR_INVALID_ARGUMENT, "null layer weight pointer");
  }
  const size_t H = d.hidden, F = d.ffn, L = d.layers;
  const bool bf = d.precision == WM_BF16;
  auto rnd = [&](float v) {
    if (!bf) return v;
    return (float)(__bf16)v;
  };
  struct Part { const float* src; size_t n; bool matrix; size_t off; };
  std::vector<Part> parts = {
      {w->tok_emb, (size_t)d.vocab * H, false, 0}, {w->pos_emb, (size_t)d.window * H, false, 0},
      {w->ln0_g, H, false, 0}, {w->ln0_b, H, false, 0},
      {w->wqkv, L * 3 * H * H, true, 0}, {w->bqkv, L * 3 * H, false, 0},
      {w->wo, L * H * H, true, 0}, {w->bo, L * H, false, 0},
      {w->ln1_g, L * H, false, 0}, {w->ln1_b, L * H, false, 0},
      {w->w1, L * F * H, true, 0}, {w->b1, L * F, false, 0},
      {w->w2, L * H * F, true, 0}, {w->b2, L * H, false, 0},
      {w->ln2_g, L * H, false, 0}, {w->ln2_b, L * H, false, 0},
      {w->wp, (size_t)d.d * H, true, 0}, {w->bp, (size_t)d.d, false, 0}};
  // Packed paths hold wqkv, wo, w1, w2 (parts 4, 6, 10, 12) as bf16, in float32 as three
  // planes: 2 or 6 bytes per weight.  They are formed on the device from float32 copies
  // that are held one at a time.
  const int mats[4] = {4, 6, 10, 12};
  const int mat_n[4] = {3 * d.hidden, d.hidden, d.ffn, d.hidden}, mat_k[4] = {d.hidden, d.hidden, d.hidden, d.ffn};
  const bool packed = packed_path(d);
  const size_t planes = bf ? 1 : 3;
  auto staged = [&](size_t i) { return packed && (i == 4 || i == 6 || i == 10 || i == 12); };
  size_t total = 0, stage = 0;
  for (size_t i = 0; i < parts.size(); ++i) {
    Part& p = parts[i];
    p.off = total;
    total = al256(total + p.n * (staged(i) ? 2 * planes : 4));
    if (staged(i) && p.n * 4 > stage) stage = p.n * 4;
  }
  void *dev = nullptr, *tmp_dev = nullptr;
  if (hipMalloc(&dev, total) != hipSuccess || (stage > 0 && hipMalloc(&tmp_dev, stage) != hipSuccess)) {
    (void)hipGetLastError();
    (void)hipFree(dev);
    return set_error(WM_ERR_OUT_OF_MEMORY, "hipMalloc of the encoder failed");
  }
  uint8_t* base = static_cast<uint8_t*>(dev);
  std::vector<float> tmp;
  hipError_t e = hipSuccess;
  for (size_t i = 0; i < parts.size() && e == hipSuccess; ++i) {
    const Part& p = parts[i];
    if (p.n == 0) continue;
    tmp.assign(p.src, p.src + p.n);
    if (p.matrix)
      for (auto& v : tmp) v = rnd(v);
    e = hipMemcpy(staged(i) ? tmp_dev : base + p.off, tmp.data(), p.n * 4, hipMemcpyHostToDevice);
    if (!staged(i) || e != hipSuccess) continue;
    const int q = i == 4 ? 0 : i == 6 ? 1 : i == 10 ? 2 : 3;
    hipLaunchKernelGGL(split_planes_kernel, dim3(2048), dim3(256), 0, nullptr, static_cast<const float*>(tmp_dev), p.n,
                       mat_n[q], mat_k[q], (int)planes, reinterpret_cast<__bf16*>(base + p.off));
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  }
  (void)hipFree(tmp_dev);
  if (e != hipSuccess) {
    (void)hipFree(dev);
    return set_error(WM_ERR_DEVICE, std::string("copying the encoder weights: ") + hipGetErrorString(e));
  }
  wm_text_model* m = new (std::nothrow) wm_text_model;
  if (!m) {
    (void)hipFree(dev);
    return set_error(WM_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  m->dims = d;
  m->base = base;
  const float** dst[] = {&m->tok_emb, &m->pos_emb, &m->ln0_g, &m->ln0_b, &m->wqkv, &m->bqkv, &m->wo,
                         &m->bo, &m->ln1_g, &m->ln1_b, &m->w1, &m->b1, &m->w2, &m->b2, &m->ln2_g,
                         &m->ln2_b, &m->wp, &m->bp};
  for (size_t i = 0; i < parts.size(); ++i)
    *dst[i] = staged(i) ? nullptr : reinterpret_cast<const float*>(base + parts[i].off);
  const __bf16** dst16[] = {&m->wqkv16, &m->wo16, &m->w116, &m->w216};
  for (int i = 0; i < 4; ++i)
    *dst16[i] = packed ? reinterpret_cast<const __bf16*>(base + parts[mats[i]].off) : nullptr;
  *out = m;
  return clear_error();
}

void wm_text_model_destroy(wm_text_model* m) {
  if (!m) return;
  (void)hipFree(m->base);
  delete m;
}

int32_t wm_text_chunks(const wm_text_model* m, const int32_t* tok_off, int32_t S) {
  if (!m || !tok_off || S < 1 || S > WM_TEXT_MAX_PROGRAMS || tok_off[0] != 0) return -1;
  long long n = 0;
  for (int s = 0; s < S; ++s) {
    if (tok_off[s + 1] < tok_off[s]) return -1;
    n += n_chunks_of(tok_off[s + 1] - tok_off[s], m->dims.window, m->dims.stride);
  }
  return n > (1LL << 30) / m->dims.window ? -1 : (int32_t)n;
}

size_t wm_text_workspace_bytes(const wm_text_model* m, int32_t n_chunks) {
  if (!m || n_chunks < 0) return 0;
  return text_layout(m->dims, n_chunks).total;
}

wm_status wm_encode_text(const wm_text_model* m, const int32_t* tokens, const int32_t* tok_off,
                         int32_t S, float* z0, void* ws, size_t ws_bytes, void* stream) {
  if (!m) return set_error(WM_ERR_INVALID_ARGUMENT, "model is NULL");
  if (!tok_off || S < 1 || S > WM_TEXT_MAX_PROGRAMS)
    return set_error(WM_ERR_INVALID_ARGUMENT, "need tok_off and 1 <= S <= " + std::to_string(WM_TEXT_MAX_PROGRAMS));
  const int32_t n_chunks = wm_text_chunks(m, tok_off, S);
  if (n_chunks < 0) return set_error(WM_ERR_INVALID_ARGUMENT, "tok_off must start at 0 and be non-decreasing");
  if (!z0 || (tok_off[S] > 0 && !tokens)) return set_error(WM_ERR_INVALID_ARGUMENT, "null tokens/z0");
  if (!ws) return set_error(WM_ERR_INVALID_ARGUMENT, "workspace is NULL");
  const wm_text_dims& d = m->dims;
  const TextLayout L = text_layout(d, n_chunks);
  if (ws_bytes < L.total) return set_error(WM_ERR_INVALID_ARGUMENT, "workspace too small");

  TTable tt;
  tt.S = S;
  tt.chunk_off[0] = 0;
  tt.row_off[0] = 0;
  for (int s = 0; s < S; ++s) {
    tt.tok_off[s] = tok_off[s];
    const int n = tok_off[s + 1] - tok_off[s], nc = n_chunks_of(n, d.window, d.stride);
    tt.chunk_off[s + 1] = tt.chunk_off[s] + nc;
    // the packed paths' rows are the chunks' tokens alone; the general path's
    // batched products take every chunk at `window` rows
    tt.row_off[s + 1] = tt.row_off[s] + (nc == 0 ? 0 : !packed_path(d) ? nc * d.window
                                         : (nc - 1) * d.window + (n - (nc - 1) * d.stride));
  }
  tt.tok_off[S] = tok_off[S];

  hipStream_t st = static_cast<hipStream_t>(stream);
  uint8_t* w8 = static_cast<uint8_t*>(ws);
  auto fp = [&](size_t o) { return reinterpret_cast<float*>(w8 + o); };
  int32_t* err = reinterpret_cast<int32_t*>(w8 + L.err);
  float *h = fp(L.h), *qkv = fp(L.qkv), *sc = fp(L.sc), *ctx = fp(L.ctx), *y = fp(L.y), *f = fp(L.f);
  float* pooled = fp(L.pooled);
  const int H = d.hidden, F = d.ffn, W = d.window, nh = d.heads, dh = H / nh;
  const int rows = tt.row_off[S];
  const bool bf = d.precision == WM_BF16;
  const bool fused = packed_path(d), f32 = fused && !bf;
  auto gemm = [&](const GemmArgs& g, int batch, bool bt) {
    return bf ? launch_gemm<BF>(g, batch, bt, st) : launch_gemm<FP>(g, batch, bt, st);
  };
#define WM_TT(K, CALL)                                                                     \
  do {                                                                                     \
    timing_begin(K, st);                                                                   \
    hipError_t e_ = (CALL);                                                                \
    timing_end(K, st);                                                                     \
    if (e_ != hipSuccess) return set_error(WM_ERR_DEVICE, std::string("kernel launch: ") + hipGetErrorString(e_)); \
  } while (0)

  float2* stats = fused ? reinterpret_cast<float2*>(w8 + L.stats) : nullptr;
  auto g16 = [&](const __bf16* A, int M, int K, const __bf16* Wm, int N, void* C, const float* bias,
                 const float* res, const float* lng, const float* lnb, int gelu, bool out16) {
    Gemm16Args g;
    g.A = A; g.W = Wm; g.C = C; g.bias = bias; g.res = res; g.stats = res ? stats : nullptr;
    g.ln_g = lng; g.ln_b = lnb; g.M = M; g.N = N; g.K = K; g.gelu = gelu; g.slices = gelu;   // the hidden layer: operand of the next product
    auto tiles = [&](int bm, int bn) { g.tiles_n = (N + bn - 1) / bn; return dim3(((M + bm - 1) / bm) * g.tiles_n); };
    auto go = [&](auto kern, dim3 grid, int threads) { hipLaunchKernelGGL(kern, grid, dim3(threads), 0, st, g); };
    // Which tile: a 256 x 256 tile keeps a compute unit busy for about four
    // times as long as a 128 x 64 tile does with its share, so it needs at
    // least 64 tiles (a quarter of the compute units) to win; 64 x 64 tiles
    // only where 128 x 64 ones leave half of the chip idle.  Measured (us,
    // large / 128 x 64 / 64 x 64): N 768, K 3072 at M = 300: 56 / 32 / 25; 2400
    // (30 large tiles): 61 / 36 / 53; 4800 (57): 63 / 69 / 103; 9600: 68 / 138 /
    // 204.  N 2304, K 768 at M = 300: 18 / 12 / 14; 2400 (90): 21 / 25 / 26; 4800:
    // 24 / 43 / 44.
    const long long large = (long long)((M + 255) / 256) * ((N + 255) / 256);
    const long long small = (long long)((M + 127) / 128) * ((N + 63) / 64);
    if (large >= 64) {
      const dim3 grid = tiles(256, 256);
      if (out16) go(gemm16_large_kernel<true>, grid, 512); else go(gemm16_large_kernel<false>, grid, 512);
    } else if (small >= 128) {
      const dim3 grid = tiles(128, 64);
      if (out16) go(gemm16_small_kernel<2, true>, grid, 256); else go(gemm16_small_kernel<2, false>, grid, 256);
    } else {
      const dim3 grid = tiles(64, 64);
      if (out16) go(gemm16_small_kernel<1, true>, grid, 256); else go(gemm16_small_kernel<1, false>, grid, 256);
    }
    return hipGetLastError();
  };
  auto g3 = [&](const __bf16* A, int K, const __bf16* Wm, size_t w_plane, int N, void* C, const float* bias,
                const float* res, const float* lng, const float* lnb, int gelu, bool split) {
    Gemm3Args g;
    g.A = A; g.W = Wm; g.C = C; g.bias = bias; g.res = res; g.stats = stats; g.ln_g = lng; g.ln_b = lnb;
    g.a_plane = (size_t)rows * K; g.w_plane = w_plane; g.c_plane = (size_t)rows * N;
    g.M = rows; g.N = N; g.K = K; g.gelu = gelu;
    g.tiles_n = (N + 63) / 64;
    const dim3 grid(((rows + 63) / 64) * g.tiles_n);
    if (split) hipLaunchKernelGGL(gemm16x3_kernel<true>, grid, dim3(512), 0, st, g);
    else hipLaunchKernelGGL(gemm16x3_kernel<false>, grid, dim3(512), 0, st, g);
    return hipGetLastError();
  };
  auto ln = [&](const float* yin, const float* gm, const float* bt, __bf16* hbo) {
    hipLaunchKernelGGL(ln_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, yin, gm, bt, H, rows, h, hbo, f32 ? (size_t)rows * H : 0, stats);
    return hipGetLastError();
  };
  __bf16* hb = reinterpret_cast<__bf16*>(w8 + L.hb);
  __bf16* qkvb = reinterpret_cast<__bf16*>(w8 + L.qkvb);
  __bf16* ctxb = reinterpret_cast<__bf16*>(w8 + L.ctxb);
  __bf16* fb = reinterpret_cast<__bf16*>(w8 + L.fb);

  if (n_chunks > 0) {
    WM_TT(TK_TEXT_OTHER, [&]() { hipLaunchKernelGGL(embed_ln_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, tokens,
                                             tt, W, d.stride, m->tok_emb, m->pos_emb, m->ln0_g, m->ln0_b,
                                             H, d.vocab, rows, y, h, fused ? hb : nullptr, f32 ? (size_t)rows * H : 0, stats, err); return hipGetLastError(); }());
    for (int l = 0; l < d.layers; ++l) {
      const size_t lH = (size_t)l * H;
      const float* g0 = l ? m->ln2_g + lH - H : m->ln0_g;       // the LayerNorm before this layer
      const float* b0 = l ? m->ln2_b + lH - H : m->ln0_b;
      if (f32) {
        const size_t Lw = (size_t)d.layers * H;
        WM_TT(TK_TEXT_GEMM, g3(hb, H, m->wqkv16 + lH * 3 * H, Lw * 3 * H, 3 * H, qkv, m->bqkv + 3 * lH, nullptr,
                               nullptr, nullptr, 0, false));
        WM_TT(TK_TEXT_ATTN, [&]() {
          hipLaunchKernelGGL(dh == 64 ? attention32_kernel<64> : attention32_kernel<32>,
                             dim3(n_chunks * nh, (W + 127) / 128), dim3(256), 0, st, qkv, ctxb, (size_t)rows * H, tt, W,
                             d.stride, nh, H, rows, 1.0f / std::sqrt((float)dh));
          return hipGetLastError();
        }());
        WM_TT(TK_TEXT_GEMM, g3(ctxb, H, m->wo16 + lH * H, Lw * H, H, y, m->bo + lH, y, g0, b0, 0, false));
        WM_TT(TK_TEXT_OTHER, ln(y, m->ln1_g + lH, m->ln1_b + lH, hb));
        WM_TT(TK_TEXT_GEMM, g3(hb, H, m->w116 + lH * F, Lw * F, F, fb, m->b1 + (size_t)l * F, nullptr, nullptr,
                               nullptr, 1, true));
        WM_TT(TK_TEXT_GEMM, g3(fb, F, m->w216 + lH * F, Lw * F, H, y, m->b2 + lH, y, m->ln1_g + lH, m->ln1_b + lH, 0,
                               false));
        WM_TT(TK_TEXT_OTHER, ln(y, m->ln2_g + lH, m->ln2_b + lH, hb));
        continue;
      }
      if (fused) {
        // bf16: every product operand is stored as bf16
        WM_TT(TK_TEXT_GEMM, g16(hb, rows, H, m->wqkv16 + lH * 3 * H, 3 * H, qkvb, m->bqkv + 3 * lH,
                                nullptr, nullptr, nullptr, 0, true));
        const int lds = (W * (dh + 8) + dh * (W + 8)) * 2;
        auto kern = dh == 64 ? attention_kernel<64> : attention_kernel<32>;
        WM_TT(TK_TEXT_ATTN, [&]() {
          hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
          if (e != hipSuccess) { (void)hipGetLastError(); return e; }
          hipLaunchKernelGGL(kern, dim3(n_chunks * nh), dim3(64 * (W / 32)), lds, st, qkvb, ctxb, tt, W,
                             d.stride, nh, H, rows, 1.0f / std::sqrt((float)dh));
          return hipGetLastError();
        }());
        WM_TT(TK_TEXT_GEMM, g16(ctxb, rows, H, m->wo16 + lH * H, H, y, m->bo + lH, y, g0, b0, 0, false));
        WM_TT(TK_TEXT_OTHER, ln(y, m->ln1_g + lH, m->ln1_b + lH, hb));
        WM_TT(TK_TEXT_GEMM, g16(hb, rows, H, m->w116 + (size_t)l * F * H, F, fb, m->b1 + (size_t)l * F,
                                nullptr, nullptr, nullptr, 1, true));
        WM_TT(TK_TEXT_GEMM, g16(fb, rows, F, m->w216 + (size_t)l * H * F, H, y, m->b2 + lH, y, m->ln1_g + lH,
                                m->ln1_b + lH, 0, false));
        WM_TT(TK_TEXT_OTHER, ln(y, m->ln2_g + lH, m->ln2_b + lH, hb));
        continue;
      }
      // q, k, v
      WM_TT(TK_TEXT_GEMM, gemm(dense(h, rows, H, m->wqkv + lH * 3 * H, 3 * H, qkv, m->bqkv + 3 * lH,
                                     nullptr, 0), 1, false));
      // scores per (chunk, head): q k^T / sqrt(dh)
      GemmArgs s{};
      s.A = qkv; s.B = qkv + H; s.C = sc; s.M = W; s.N = W; s.K = dh;
      s.lda = 3 * H; s.ldb = 3 * H; s.ldc = W; s.bdiv = nh;
      s.sA1 = (long long)W * 3 * H; s.sA2 = dh; s.sB1 = s.sA1; s.sB2 = dh;
      s.sC1 = (long long)nh * W * W; s.sC2 = (long long)W * W;
      s.alpha = 1.0f / std::sqrt((float)dh);
      WM_TT(TK_TEXT_ATTN, gemm(s, n_chunks * nh, false));
      WM_TT(TK_TEXT_ATTN, [&]() { hipLaunchKernelGGL(softmax_kernel, dim3((unsigned)(((long long)n_chunks * nh * W + 3) / 4)),
                                              dim3(256), 0, st, sc, tt, W, d.stride, nh,
                                              (long long)n_chunks * nh * W); return hipGetLastError(); }());
      // context = P v per (chunk, head), into the head's columns
      GemmArgs pv{};
      pv.A = sc; pv.B = qkv + 2 * H; pv.C = ctx; pv.M = W; pv.N = dh; pv.K = W;
      pv.lda = W; pv.ldb = 3 * H; pv.ldc = H; pv.bdiv = nh;
      pv.sA1 = (long long)nh * W * W; pv.sA2 = (long long)W * W;
      pv.sB1 = (long long)W * 3 * H; pv.sB2 = dh;
      pv.sC1 = (long long)W * H; pv.sC2 = dh;
      pv.alpha = 1.0f;
      WM_TT(TK_TEXT_ATTN, gemm(pv, n_chunks * nh, true));
      // h = LN(h + ctx Wo^T + bo)
      WM_TT(TK_TEXT_GEMM, gemm(dense(ctx, rows, H, m->wo + lH * H, H, y, m->bo + lH, h, 0), 1, false));
      WM_TT(TK_TEXT_OTHER, ln(y, m->ln1_g + lH, m->ln1_b + lH, nullptr));
      // h = LN(h + GELU(h W1^T + b1) W2^T + b2)
      WM_TT(TK_TEXT_GEMM, gemm(dense(h, rows, H, m->w1 + (size_t)l * F * H, F, f, m->b1 + (size_t)l * F,
                                     nullptr, 1), 1, false));
      WM_TT(TK_TEXT_GEMM, gemm(dense(f, rows, F, m->w2 + (size_t)l * H * F, H, y, m->b2 + lH, h, 0), 1, false));
      WM_TT(TK_TEXT_OTHER, ln(y, m->ln2_g + lH, m->ln2_b + lH, nullptr));
    }
    const size_t lastH = d.layers > 0 ? (size_t)(d.layers - 1) * H : 0;
    const float* last_g = d.layers > 0 ? m->ln2_g + lastH : m->ln0_g;
    const float* last_b = d.layers > 0 ? m->ln2_b + lastH : m->ln0_b;
    WM_TT(TK_TEXT_OTHER, [&]() { hipLaunchKernelGGL(pool_kernel, dim3(n_chunks), dim3(POOL_THREADS), 0, st, fused ? y : h,
                                             stats, last_g, last_b, tt, W, d.stride, H, pooled); return hipGetLastError(); }());
  }
  WM_TT(TK_TEXT_OTHER, [&]() { hipLaunchKernelGGL(project_kernel, dim3(S), dim3(256), H * (int)sizeof(float), st,
                                           pooled, tt, H, d.d, m->wp, m->bp, bf ? 1 : 0, z0); return hipGetLastError(); }());
#undef WM_TT
  return clear_error();
}

}  // extern "C"
