// Surrogate network kernels: a multilayer perceptron with BF16 matrix-core
// GEMMs (v_mfma_f32_16x16x32_bf16, FP32 accumulation), fused bias + SiLU
// epilogue, SiLU backward, column sums, mean-squared-error loss and Adam with
// FP32 master weights and a BF16 working copy.
//
// Layer l: Z_l = H_l W_l^T + b_l (W_l stored [out][in]), H_{l+1} = SiLU(Z_l)
// for hidden layers, the last layer linear.  Backward with G = dL/dZ_l:
//   dW_l = G^T H_l,  db_l = sum over the batch of G,  dH_l = G W_l,
//   dL/dZ_{l-1} = dH_l * SiLU'(Z_{l-1}).
#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "semx_internal.hpp"

struct semx_mlp {
  int nl = 0;
  std::vector<int> w;
  int max_batch = 0;
  hipStream_t stream = nullptr;
  std::string err;
  int64_t nparam = 0;
  std::vector<int64_t> woff, boff;
  semx::DevBuf theta, theta_bf, grad, m, v;
  std::vector<semx::DevBuf> Z, H;  // Z[l] [B][w[l+1]], H[l] (l >= 1) [B][w[l]], both FP32
  semx::DevBuf Hb[2];              // BF16 copies of a layer's H: the next product's operand, layers in turn
  semx::DevBuf g0, g1;             // backward work [B][max width]
  semx::DevBuf scratch;
  semx::DevBuf splitk;             // split-K partial sums
  char* stage = nullptr;           // pinned, kStageSlots pieces of kStageBytes (download)
  hipEvent_t staged[2] = {nullptr, nullptr};
  std::mutex stage_use;            // one download through them at a time
  const float* x_saved = nullptr;
  int batch_saved = 0;
  int device = 0;                  // device current at creation (allocation-free forward)
};

namespace semx {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 32;
// LDS place of element (r, k) of a tile.  SWZ (both operands contiguous along
// k): rows of 64 bytes, whose four 16-byte pieces are permuted by the row so
// that neither the writes nor the reads of a wave meet on a bank (with rows
// padded to 80 bytes half the LDS cycles of the output layer were conflicts).
// Otherwise rows of 80 bytes, which suit the pieces that Tile's turned form
// writes (training at batch 128 is 3 % slower with permuted rows).
template <bool SWZ>
constexpr int kPitch = SWZ ? BK : BK + 8;
template <bool SWZ>
__device__ __forceinline__ int lds_at(int r, int k) {
  return r * kPitch<SWZ> + (SWZ ? (((k >> 3) ^ (r >> 1)) & 3) * 8 + (k & 7) : k);
}
// columns of tiles that share an XCD's L2 (gemm_kernel)
constexpr int kGroup = 16;
constexpr int64_t kSplitWs = 2 << 20;  // floats of split-K partial sums per network (8 MB)

// Workspace of semx_mlp_forward_noalloc: two activation buffers of
// kNoAllocFloats / 2 floats each, in the code object's own device memory (each
// GPU the library runs on holds one copy until the process ends).  Host code
// never passes `scratch` itself to a kernel: its name is a host-side handle;
// the device address comes from hipGetSymbolAddress, once per device.
constexpr int64_t kNoAllocFloats = 4 << 20;  // 16 MB
__device__ __align__(256) float scratch[kNoAllocFloats];
constexpr int kMaxDevices = 64;
float* g_scratch_dev[kMaxDevices] = {};  // device address of `scratch`, per device
hipError_t g_scratch_err[kMaxDevices] = {};
std::once_flag g_scratch_once[kMaxDevices];

// Resolve `scratch` on the current device (once per device).
hipError_t noalloc_setup(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(g_scratch_once[dev], [dev]() {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    g_scratch_err[dev] = e;
    g_scratch_dev[dev] = e == hipSuccess ? static_cast<float*>(ptr) : nullptr;
  });
  return g_scratch_err[dev];
}

// Eight elements of an operand as they lie in memory: a request that stays in
// flight until the values are converted into LDS.
template <class T>
struct Raw8;
template <>
struct Raw8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float* p) {
    a = *reinterpret_cast<const float4*>(p);
    b = *reinterpret_cast<const float4*>(p + 4);
  }
  __device__ __forceinline__ void set(int e, float x) {
    if (e == 0) a.x = x; else if (e == 1) a.y = x; else if (e == 2) a.z = x; else if (e == 3) a.w = x;
    else if (e == 4) b.x = x; else if (e == 5) b.y = x; else if (e == 6) b.z = x; else b.w = x;
  }
  __device__ __forceinline__ bf16x8 bf16() const {
    return bf16x8{(__bf16)a.x, (__bf16)a.y, (__bf16)a.z, (__bf16)a.w, (__bf16)b.x, (__bf16)b.y, (__bf16)b.z, (__bf16)b.w};
  }
};
template <>
struct Raw8<__bf16> {
  bf16x8 v;
  __device__ __forceinline__ void load(const __bf16* p) { v = *reinterpret_cast<const bf16x8*>(p); }
  __device__ __forceinline__ void set(int e, __bf16 x) { v[e] = x; }
  __device__ __forceinline__ bf16x8 bf16() const { return v; }
};

// A thread's share of one operand tile T[r][k] (ROWS rows x BK, 256 threads) of
// X(r, k) = X[r * sr + k * sk], rows r0 .. r0+ROWS-1, k in [k0, kend).
// KC: X is contiguous along k (sk = 1), a thread takes ROWS / 64 chunks of 8
// consecutive k of one row.
// How the chunks are loaded (the launch decides by the operands' sizes):
//   kWhole    every chunk lies wholly inside or wholly outside the operand and
//             is 16-byte aligned: one vector load at an address that is clamped
//             into the operand, zeroed on the way into LDS where it lies past
//             kend (rows past R give sums that are not stored);
//   kJudged   by vectors where the operand is aligned (`wide`) and the chunk lies
//             inside, else element by element with bounds (64-516-516-24564 at
//             batch 128: forward 77 -> 58 us, training step 385 -> 262);
//   kElement  element by element (neither operand is aligned: 12-129-257-515 at
//             batch 128 33 against 41 us).
enum class Loads { kElement, kJudged, kWhole };
template <class T, bool KC, int ROWS, Loads LD>
struct Tile {
  static constexpr bool VEC = LD == Loads::kWhole;
  static constexpr int C = ROWS / 64;
  Raw8<T> raw[C];

  __device__ __forceinline__ void load(const T* __restrict__ X, int64_t sr, int64_t sk, int R, int r0, int k0, int kend,
                                       int t, int wide) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int r = r0 + (t >> 2) + 64 * c, k = k0 + (t & 3) * 8;
      if constexpr (VEC) {
        raw[c].load(X + (int64_t)min(r, R - 1) * sr + min(k, kend - 8));
      } else if (LD == Loads::kJudged && wide && r < R && k + 8 <= kend) {
        raw[c].load(X + (int64_t)r * sr + k);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          raw[c].set(e, (r < R && k + e < kend) ? X[(int64_t)r * sr + (int64_t)(k + e) * sk] : (T)0.0f);
      }
    }
  }
  template <bool TAIL, bool SWZ>
  __device__ __forceinline__ void store(__bf16* Ts, int k0, int kend, int t) const {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int kk = (t & 3) * 8;
      bf16x8 w = raw[c].bf16();
      if (VEC && TAIL && k0 + kk >= kend) w = bf16x8{};
      *reinterpret_cast<bf16x8*>(Ts + lds_at<SWZ>((t >> 2) + 64 * c, kk)) = w;
    }
  }
};

// X contiguous along r (sr = 1): a thread takes a block of 4 rows x KQ
// consecutive k, turns it in its registers and writes KQ elements of a row at a
// time.  The lanes of a wave run over k first, so that their writes (rows 80
// bytes apart) fall on different banks; with eight rows of one k a thread,
// written element by element, up to 16 lanes met on a bank: the weight gradient
// of 24576 outputs at batch 128 took 34.5 us, now 26 (its 50 MB of output alone 10),
// the input gradient 28, now 23.
template <class T, int ROWS, Loads LD>
struct Tile<T, false, ROWS, LD> {
  static constexpr bool VEC = LD == Loads::kWhole;
  static constexpr int KQ = ROWS / 32;  // 4 or 2
  typedef T T4 __attribute__((ext_vector_type(4)));
  typedef __bf16 BK4 __attribute__((ext_vector_type(KQ)));
  T4 raw[KQ];

  __device__ static __forceinline__ int kof(int t) { return t % (BK / KQ) * KQ; }
  __device__ static __forceinline__ int row(int t) { return t / (BK / KQ) * 4; }

  __device__ __forceinline__ void load(const T* __restrict__ X, int64_t sr, int64_t sk, int R, int r0, int k0, int kend,
                                       int t, int wide) {
    const int r = r0 + row(t), k = k0 + kof(t);
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      if constexpr (VEC) {
        raw[j] = *reinterpret_cast<const T4*>(X + min(r, R - 4) + (int64_t)min(k + j, kend - 1) * sk);
      } else if (LD == Loads::kJudged && wide && r + 4 <= R && k + j < kend) {
        raw[j] = *reinterpret_cast<const T4*>(X + r + (int64_t)(k + j) * sk);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          raw[j][e] = (r + e < R && k + j < kend) ? X[(int64_t)(r + e) * sr + (int64_t)(k + j) * sk] : (T)0.0f;
      }
    }
  }
  template <bool TAIL, bool SWZ>
  __device__ __forceinline__ void store(__bf16* Ts, int k0, int kend, int t) const {
    const int r = row(t), k = kof(t);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      BK4 w;
#pragma unroll
      for (int j = 0; j < KQ; ++j) w[j] = VEC && TAIL && k0 + k + j >= kend ? (__bf16)0.0f : (__bf16)raw[j][e];
      *reinterpret_cast<BK4*>(Ts + lds_at<SWZ>(r + e, k)) = w;
    }
  }
};

__device__ __forceinline__ float silu(float v) { return v / (1.0f + expf(-v)); }
__device__ __forceinline__ float silu_grad(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// What a GEMM does with its sums.
constexpr int kBias = 1;      // C = sum + bias[n]
constexpr int kSiluKeep = 2;  // C = sum + bias[n] (the pre-activation), H = SiLU(C), Hb the same in BF16 (the next product's operand)
constexpr int kSilu = 3;      // H = SiLU(sum + bias[n]) (inference: the pre-activation is not kept)
constexpr int kGradZ = 4;     // C = sum * SiLU'(Z[m][n]); split-K slices store their partial sums (the reduction applies Z)
constexpr int kBiasStream = 6;  // kBias, the output past the caches
constexpr int kGradW = 5;     // C = sum; db[m] = sum of A over k

// C[m][n] = sum_k A(m,k) B(k,n), A(m,k) = A[m*sam + k*sak], B(k,n) = B[k*sbk + n*sbn].
// Split-K (gridDim.z > 1): slice z covers k in [z kchunk, (z+1) kchunk) and
// stores its partial sums to C + z M N (row stride N).
//
// One workgroup of four waves per tile of 32 WT x 32 WT outputs, a wave WT x WT
// matrix-core tiles; k in steps of 32 through two LDS buffers (one barrier a
// step).  The network's products are short in k and often small: what bounds
// them is the latency of the operand loads, a round trip per step when a step
// waits for its own.  The loads of PF steps are therefore in flight at a time,
// held as they came from memory and converted on the way into LDS (64 x 64
// tiles that waited for each step: the hidden layers' products at batch 128 18
// us, now 6.8).  WT = 2 (64 x 64) where few tiles would leave compute units idle,
// WT = 4 (128 x 128: half the operand traffic and LDS reads per product) from
// 512 tiles: the 4096 x 24576 x 512 output layer 344 -> 172 us, with permuted
// LDS rows, whole-line stores and tile order below (L2 misses 8.7 -> 3.8
// million lines) 164, 630 TFLOP/s.  Its products alone take 115 us, its 402 MB
// of stores alone 74: the two hardly overlap.  The order of the sum over k is
// the same in both.
template <class TA, class TB, int EPI, bool AKC, bool BKC, int WT, Loads LD>
__global__ __launch_bounds__(256, WT == 2 ? 4 : 2) void gemm_kernel(int M, int N, int K, int kchunk,
                                                                    const TA* __restrict__ A, int64_t sam, int64_t sak,
                                                                    const TB* __restrict__ B, int64_t sbk, int64_t sbn,
                                                                    float* __restrict__ C, int64_t ldc,
                                                                    const float* __restrict__ bias,
                                                                    float* __restrict__ H,
                                                                    __bf16* __restrict__ Hb,
                                                                    const float* __restrict__ Z,
                                                                    float* __restrict__ db, int outv, int wa, int wb) {
  constexpr bool SWZ = AKC && BKC;
  constexpr int ROWS = 32 * WT, PF = LD != Loads::kWhole ? 1 : WT == 2 ? 4 : 2;
  __shared__ __attribute__((aligned(16))) __bf16 As[2][ROWS * kPitch<SWZ>];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[2][ROWS * kPitch<SWZ>];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // A split-K slice on one XCD (consecutive blocks go to the eight XCDs in
  // turn), so that its tiles meet the operands' slices in one L2: the input
  // gradient of 24576 outputs at batch 128 23.1 -> 18.8 us
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (EPI == kGradZ && gridDim.z % kNumXcd == 0) {
    const int tiles = gridDim.x * gridDim.y, L = bx + gridDim.x * (by + gridDim.y * bz);
    const int tile = L / kNumXcd % tiles;
    bz = L % kNumXcd + kNumXcd * (L / kNumXcd / tiles);
    bx = tile % gridDim.x;
    by = tile / gridDim.x;
  }
  // Many tiles: columns of tiles in groups of kGroup, row by row inside a group,
  // an eighth of that order to each XCD, so that what its L2 holds of B is used
  // by all of A before the next group
  if (WT == 4 && gridDim.z == 1 && EPI != kGradW) {
    const int nx = gridDim.x, ny = gridDim.y, n = nx * ny, L = bx + nx * by;
    if (n % kNumXcd == 0) {
      const int T = L % kNumXcd * (n / kNumXcd) + L / kNumXcd, g = T / (kGroup * ny), r = T - g * kGroup * ny;
      const int w = min(kGroup, nx - g * kGroup);
      bx = g * kGroup + r % w;
      by = r / w;
    }
  }
  const int bm = by * ROWS, bn = bx * ROWS;
  const int wu = __builtin_amdgcn_readfirstlane(wv), wm = wu >> 1, wn = wu & 1;
  const bool split = gridDim.z > 1;
  const int kbeg = bz * kchunk;
  const int kend = min(K, kbeg + kchunk);
  const int steps = (kend - kbeg + BK - 1) / BK;
  f32x4 acc[WT][WT];
#pragma unroll
  for (int a = 0; a < WT; ++a)
#pragma unroll
    for (int b = 0; b < WT; ++b) acc[a][b] = (f32x4){0.f, 0.f, 0.f, 0.f};
  Tile<TA, AKC, ROWS, LD> ta[PF];
  Tile<TB, BKC, ROWS, LD> tb[PF];
#pragma unroll
  for (int p = 0; p < PF; ++p) {
    ta[p].load(A, sam, sak, M, bm, kbeg + p * BK, kend, t, wa);
    tb[p].load(B, sbn, sbk, N, bn, kbeg + p * BK, kend, t, wb);
  }
  if constexpr (EPI == kGradW) {
    // the blocks of the first column also sum their rows of A over k, in order
    if (bx == 0 && bz == 0 && t < ROWS && bm + t < M) {
      const TA* p = A + (int64_t)(bm + t) * sam;
      float s = 0.0f;
      int k = 0;
      for (; k + 32 <= K; k += 32) {
        float v[32];
#pragma unroll
        for (int e = 0; e < 32; ++e) v[e] = (float)p[(int64_t)(k + e) * sak];
#pragma unroll
        for (int e = 0; e < 32; ++e) s += v[e];
      }
      for (; k < K; ++k) s += (float)p[(int64_t)k * sak];
      db[bm + t] = s;
    }
  }
  // One step: tile p to LDS, the tile PF steps ahead requested in its place
  // (LOAD), products.  The loop's loads are unconditional, so that the compiler
  // counts them and a step waits for its own tile alone; the last PF steps
  // request nothing, and only there can a tile end inside.
  auto step = [&](auto load, auto p_, int s) {
    constexpr bool LOAD = decltype(load)::value;
    constexpr int p = decltype(p_)::value;
    // buffer s & 1 was last read in step s - 2, before the barrier of step s - 1
    __bf16* as = As[s & 1];
    __bf16* bs = Bs[s & 1];
    ta[p].template store<!LOAD, SWZ>(as, kbeg + s * BK, kend, t);
    tb[p].template store<!LOAD, SWZ>(bs, kbeg + s * BK, kend, t);
    if constexpr (LOAD) {
      ta[p].load(A, sam, sak, M, bm, kbeg + (s + PF) * BK, kend, t, wa);
      tb[p].load(B, sbn, sbk, N, bn, kbeg + (s + PF) * BK, kend, t, wb);
    }
    __syncthreads();
    bf16x8 av[WT], bv[WT];
#pragma unroll
    for (int a = 0; a < WT; ++a)
      av[a] = *reinterpret_cast<const bf16x8*>(as + lds_at<SWZ>(wm * 16 * WT + a * 16 + (lane & 15), 8 * (lane >> 4)));
#pragma unroll
    for (int b = 0; b < WT; ++b)
      bv[b] = *reinterpret_cast<const bf16x8*>(bs + lds_at<SWZ>(wn * 16 * WT + b * 16 + (lane & 15), 8 * (lane >> 4)));
#pragma unroll
    for (int a = 0; a < WT; ++a)
#pragma unroll
      for (int b = 0; b < WT; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[b], av[a], acc[a][b], 0, 0, 0);
  };
  auto group = [&](auto load, int s0) {
    constexpr bool LOAD = decltype(load)::value;
    step(load, std::integral_constant<int, 0>{}, s0);
    if constexpr (PF > 1)
      if (LOAD || s0 + 1 < steps) step(load, std::integral_constant<int, 1>{}, s0 + 1);
    if constexpr (PF > 2) {
      if (LOAD || s0 + 2 < steps) step(load, std::integral_constant<int, 2>{}, s0 + 2);
      if (LOAD || s0 + 3 < steps) step(load, std::integral_constant<int, 3>{}, s0 + 3);
    }
  };
  int s0 = 0;
  for (; s0 + PF < steps; s0 += PF) group(std::true_type{}, s0);
  group(std::false_type{}, s0);
  // The product is taken transposed (B's columns as the rows of the matrix-core
  // tile): a lane holds four consecutive n of one m, one 16-byte store.
  // Outputs of 64 MB and more go past the caches (402 MB at batch 4096: 257 ->
  // 210 us for the network, 202 with the 16-byte stores).
  const int64_t ldz = split ? N : ldc;
  float* Cz = split ? C + (int64_t)bz * M * N : C;
  const int m0 = bm + wm * 16 * WT + (lane & 15), n0 = bn + wn * 16 * WT + 4 * (lane >> 4);
  constexpr bool BIAS = EPI == kBias || EPI == kBiasStream || EPI == kSiluKeep || EPI == kSilu;
  if constexpr (EPI == kBias || EPI == kBiasStream) {
    // Whole 128-byte lines: a store of one tile holds 64 bytes of 16 rows; lanes
    // eight rows apart exchange halves of a pair of tiles, so that a store holds
    // the 128 bytes of both in 8 rows.
    if (outv) {
      const bool hi = lane & 8;
      const int mr = bm + wm * 16 * WT + (lane & 7);
#pragma unroll
      for (int b = 0; b < WT; b += 2) {
        const int n = n0 + 16 * (b + (hi ? 1 : 0));
        f32x4 add0, add1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          add0[r] = bias[min(n0 + 16 * b + r, N - 1)];
          add1[r] = bias[min(n0 + 16 * (b + 1) + r, N - 1)];
        }
#pragma unroll
        for (int a = 0; a < WT; ++a) {
          f32x4 lo = acc[a][b] + add0, up = acc[a][b + 1] + add1;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x = hi ? lo[r] : up[r];
            // row_ror:8, the lane eight away in its row of sixteen
            const float y = __builtin_bit_cast(
                float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
            if (hi) lo[r] = y;
            else up[r] = y;
          }
          const int m = n < N ? mr + 16 * a : M;
          f32x4* o = reinterpret_cast<f32x4*>(Cz + (int64_t)m * ldz + n);
          f32x4* o8 = reinterpret_cast<f32x4*>(Cz + (int64_t)(m + 8) * ldz + n);
          if constexpr (EPI == kBiasStream) {
            if (m < M) __builtin_nontemporal_store(lo, o);
            if (m + 8 < M) __builtin_nontemporal_store(up, o8);
          } else {
            if (m < M) *o = lo;
            if (m + 8 < M) *o8 = up;
          }
        }
      }
      return;
    }
  }
#pragma unroll
  for (int b = 0; b < WT; ++b) {
    const int n = n0 + 16 * b;
    if (n >= N) continue;
    float add[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (BIAS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) add[r] = n + r < N ? bias[n + r] : 0.0f;
    }
#pragma unroll
    for (int a = 0; a < WT; ++a) {
      const int m = m0 + 16 * a;
      if (m >= M) continue;
      const int64_t o = (int64_t)m * ldz + n;
      f32x4 v = acc[a][b];
      if constexpr (BIAS) v += (f32x4){add[0], add[1], add[2], add[3]};
      if (outv) {
        if constexpr (EPI == kGradZ)
          if (!split) {
            const f32x4 z = *reinterpret_cast<const f32x4*>(Z + o);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] *= silu_grad(z[r]);
          }
        if constexpr (EPI == kBiasStream) __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(Cz + o));
        else if constexpr (EPI != kSilu) *reinterpret_cast<f32x4*>(Cz + o) = v;
        if constexpr (EPI == kSiluKeep || EPI == kSilu) {
          f32x4 h;
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = silu(v[r]);
          *reinterpret_cast<f32x4*>(H + o) = h;
          if constexpr (EPI == kSiluKeep)
            if (Hb) *reinterpret_cast<bf16x4*>(Hb + o) = bf16x4{(__bf16)h[0], (__bf16)h[1], (__bf16)h[2], (__bf16)h[3]};
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (n + r >= N) continue;
          float x = v[r];
          if (EPI == kGradZ && !split) x *= silu_grad(Z[o + r]);
          if (EPI != kSilu) Cz[o + r] = x;
          if (EPI == kSiluKeep || EPI == kSilu) H[o + r] = silu(x);
          if (EPI == kSiluKeep && Hb) Hb[o + r] = (__bf16)silu(x);
        }
      }
    }
  }
}

// C[m][n] = sum over the nz slices of P (fixed order: deterministic), times
// SiLU'(Z) when Z is given.
__global__ void splitk_reduce_kernel(int M, int N, int nz, const float* __restrict__ P, const float* __restrict__ Z,
                                     float* __restrict__ C, int64_t ldc) {
  const int64_t MN = (int64_t)M * N;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < MN; t += (int64_t)gridDim.x * blockDim.x) {
    float s = 0.0f;
    int z = 0;
    for (; z + 8 <= nz; z += 8) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = P[(z + e) * MN + t];
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e];
    }
    for (; z < nz; ++z) s += P[z * MN + t];
    const int64_t o = (t / N) * ldc + t % N;
    if (Z) s *= silu_grad(Z[o]);
    C[o] = s;
  }
}

template <class T>
bool aligned16(const T* p, int64_t stride) {
  return (reinterpret_cast<uintptr_t>(p) % 16 == 0) && ((stride * (int64_t)sizeof(T)) % 16 == 0);
}

// The outputs a GEMM may write and what its epilogue reads.
struct GemmOut {
  float* C = nullptr;
  int64_t ldc = 0;
  const float* bias = nullptr;
  float* H = nullptr;
  __bf16* Hb = nullptr;
  const float* Z = nullptr;
  float* db = nullptr;
  float* ws = nullptr;  // split-K partial sums
};

template <class TA, class TB, int EPI, bool AKC, bool BKC>
hipError_t gemm_launch(hipStream_t s, int M, int N, int K, const TA* A, int64_t sam, int64_t sak, const TB* B,
                       int64_t sbk, int64_t sbn, const GemmOut& O) {
  // whole vectors: 16-byte alignment and, for both operands, eights along the
  // contiguous direction
  const int wa = aligned16(A, AKC ? sam : sak) && (AKC ? sak : sam) == 1;
  const int wb = aligned16(B, BKC ? sbn : sbk) && (BKC ? sbk : sbn) == 1;
  const bool vec = wa && wb && (AKC ? K : M) % 8 == 0 && (BKC ? K : N) % 8 == 0;
  const int tiles = ((N + 63) / 64) * ((M + 63) / 64);
  int nz = 1, kchunk = K;
  if ((EPI == kGradZ || EPI == kGradW) && O.ws && tiles < 128 && K >= 1024) {
    nz = std::min<int>(32, (512 + tiles - 1) / tiles);
    kchunk = (((K + nz - 1) / nz + BK - 1) / BK) * BK;
    nz = (K + kchunk - 1) / kchunk;
    while (nz > 1 && (int64_t)nz * M * N > kSplitWs) {
      kchunk *= 2;
      nz = (K + kchunk - 1) / kchunk;
    }
  }
  const bool wide = vec && (int64_t)((N + 127) / 128) * ((M + 127) / 128) >= 512;
  const int rows = wide ? 128 : 64;
  const dim3 grid((N + rows - 1) / rows, (M + rows - 1) / rows, nz), block(256);
  float* C = nz > 1 ? O.ws : O.C;
  // outputs in fours along n
  const int outv = (nz > 1 ? N : O.ldc) % 4 == 0 && N % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(O.H) % 16 == 0 && reinterpret_cast<uintptr_t>(O.Hb) % 8 == 0 && reinterpret_cast<uintptr_t>(O.Z) % 16 == 0;
  auto go = [&](auto kernel) {
    kernel<<<grid, block, 0, s>>>(M, N, K, kchunk, A, sam, sak, B, sbk, sbn, C, O.ldc, O.bias, O.H, O.Hb, O.Z, O.db, outv, wa, wb);
  };
  if (wide) go(gemm_kernel<TA, TB, EPI, AKC, BKC, 4, Loads::kWhole>);
  else if (vec) go(gemm_kernel<TA, TB, EPI, AKC, BKC, 2, Loads::kWhole>);
  else if (wa || wb) go(gemm_kernel<TA, TB, EPI, AKC, BKC, 2, Loads::kJudged>);
  else go(gemm_kernel<TA, TB, EPI, AKC, BKC, 2, Loads::kElement>);
  if (nz > 1) {
    const int64_t MN = (int64_t)M * N;
    const unsigned nb = (unsigned)std::min<int64_t>((MN + 255) / 256, 4096);
    splitk_reduce_kernel<<<nb, 256, 0, s>>>(M, N, nz, O.ws, EPI == kGradZ ? O.Z : nullptr, O.C, O.ldc);
  }
  return hipGetLastError();
}

// dy = 2 (y - t) / n and, when `loss` is given, loss += sum (y - t)^2 / n (FP64)
__global__ __launch_bounds__(256) void mse_kernel(int64_t n, const float* __restrict__ y, const float* __restrict__ t,
                                                  float* __restrict__ dy, double* __restrict__ loss) {
  __shared__ double red[256];
  double s = 0.0;
  const float inv = 1.0f / (float)n;
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  const bool vec = (reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(t) | reinterpret_cast<uintptr_t>(dy)) % 16 == 0;
  const int64_t nv = vec ? n / 4 : 0;
  for (int64_t i = i0; i < nv; i += stride) {
    const f32x4 d = reinterpret_cast<const f32x4*>(y)[i] - reinterpret_cast<const f32x4*>(t)[i];
    if (dy) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = 2.0f * d[e] * inv;
      reinterpret_cast<f32x4*>(dy)[i] = o;
    }
    if (loss)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += (double)d[e] * (double)d[e];
  }
  for (int64_t i = 4 * nv + i0; i < n; i += stride) {
    const float d = y[i] - t[i];
    if (dy) dy[i] = 2.0f * d * inv;
    if (loss) s += (double)d * (double)d;
  }
  if (!loss) return;
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(loss, red[0] / (double)n);
}

// y[r][c] = a[c] x[r][c] + b[c] (column-wise affine map; x and y may alias)
__global__ void affine_cols_kernel(int64_t n, int cols, const float* x, const float* __restrict__ a,
                                   const float* __restrict__ b, float* y) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(t % cols);
    y[t] = a[c] * x[t] + b[c];
  }
}

// Ensemble statistics of one row per block: members' predictions P[k][r][c]
// (normalised units), mean over members mapped back through a[c] m + b[c],
// and the spread indicator || a * std || / || mean (physical) || with the
// unbiased standard deviation over the members (zero for one member); the
// two norms are FP64 block reductions in a fixed order.
__global__ void ensemble_kernel(int members, int64_t rows, int cols, const float* __restrict__ P,
                                const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ mean,
                                float* __restrict__ ind) {
  __shared__ double red[2][256];
  const int64_t r = blockIdx.x;
  if (r >= rows) return;
  double s_sp = 0.0, s_mn = 0.0;
  const float inv_m = 1.0f / (float)members;
  const float inv_m1 = members > 1 ? 1.0f / (float)(members - 1) : 0.0f;
  for (int c = threadIdx.x; c < cols; c += blockDim.x) {
    float sum = 0.0f;
    for (int k = 0; k < members; ++k) sum += P[((int64_t)k * rows + r) * cols + c];
    const float mu = sum * inv_m;
    float ss = 0.0f;
    for (int k = 0; k < members; ++k) {
      const float d = P[((int64_t)k * rows + r) * cols + c] - mu;
      ss += d * d;
    }
    const float sd = a[c] * sqrtf(ss * inv_m1);
    const float mp = a[c] * mu + b[c];
    mean[r * cols + c] = mp;
    s_sp += (double)sd * sd;
    s_mn += (double)mp * mp;
  }
  red[0][threadIdx.x] = s_sp;
  red[1][threadIdx.x] = s_mn;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      red[0][threadIdx.x] += red[0][threadIdx.x + st];
      red[1][threadIdx.x] += red[1][threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) ind[r] = (float)(sqrt(red[0][0]) / fmax(sqrt(red[1][0]), 1e-30));
}

__global__ void adam_kernel(int64_t n, float lr, float b1, float b2, float eps, float c1, float c2,
                            const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                            float* __restrict__ th, __bf16* __restrict__ thb) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float t = th[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    th[i] = t;
    thb[i] = (__bf16)t;
  }
}

__global__ void to_bf16_kernel(int64_t n, const float* __restrict__ x, __bf16* __restrict__ y) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (__bf16)x[i];
}

// Layer l of the forward pass: A(m,k) = h[m*in + k] (FP32, rounded to BF16 on its
// way into LDS, or already BF16), B(k,n) = W[n*in + k].
template <int EPI, class TA>
hipError_t layer(semx_mlp* p, int l, int batch, const TA* h, GemmOut& O) {
  const int in = p->w[l], out = p->w[l + 1];
  const __bf16* W = p->theta_bf.as<__bf16>() + p->woff[l];
  O.ldc = out;
  O.bias = p->theta.as<float>() + p->boff[l];
  return gemm_launch<TA, __bf16, EPI, true, true>(p->stream, batch, out, in, h, in, 1, W, 1, in, O);
}

// Whether the product after a hidden layer of this width reads its BF16 copy: half
// the bytes where whole rows of it are 16-byte aligned (512 wide, 4096 x 24576
// outputs: 185 us against 202), else the FP32 activations load faster (516 wide:
// 1000 us against 1365).
bool bf16_rows(int width) { return width % 8 == 0; }

// The network's output, past the caches where they would not hold it until its
// reader comes.
template <class TA>
hipError_t output_layer(semx_mlp* p, int l, int batch, const TA* h, GemmOut& O) {
  return (int64_t)batch * p->w[l + 1] * 4 >= (int64_t(64) << 20) ? layer<kBiasStream>(p, l, batch, h, O)
                                                                  : layer<kBias>(p, l, batch, h, O);
}

unsigned g1(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

int mfail(semx_mlp* p, int code, const std::string& m) {
  if (p) p->err = m;
  return code;
}

int mhip(semx_mlp* p, hipError_t e, const char* what) {
  return mfail(p, SEMX_EHIP, std::string("HIP error ") + hipGetErrorName(e) + " in " + what);
}

int malloc_buf(semx_mlp* p, DevBuf& b, size_t bytes) {
  if (b.p) (void)hipFree(b.p);
  b.p = nullptr;
  b.bytes = 0;
  if (!bytes) return SEMX_OK;
  if (hipMalloc(&b.p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    b.p = nullptr;
    return mfail(p, SEMX_ENOMEM, "hipMalloc failed");
  }
  b.bytes = bytes;
  return SEMX_OK;
}

// Device to host copy of a whole parameter vector, complete on return.  Copied
// straight into pageable memory, 53 MB took 3.1 ms, and 2 ms more where the
// pages were new; the device's share is 0.9.  So the destination's pages are
// made present first, while the kernels queued on the stream still run, and the
// data comes through two pinned pieces, one on its way while the other is
// copied out.  Anything unusual (small, pinned or device memory, a stream under
// capture, pages that cannot be written, the pieces in use by another thread)
// goes the direct way.
constexpr int kStageSlots = 2;
constexpr int64_t kStageBytes = 4 << 20;

int download(semx_mlp* p, float* dst, const float* src) {
  const int64_t bytes = sizeof(float) * p->nparam;
  char* d = reinterpret_cast<char*>(dst);
  const char* s = reinterpret_cast<const char*>(src);
  std::unique_lock<std::mutex> use(p->stage_use, std::defer_lock);
  bool staged = p->stage && bytes >= kStageBytes && use.try_lock();
  if (staged) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    hipPointerAttribute_t at{};
    staged = hipStreamIsCapturing(p->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
    if (staged && hipPointerGetAttributes(&at, dst) == hipSuccess) staged = at.type == hipMemoryTypeUnregistered;
    (void)hipGetLastError();  // an ordinary host pointer may be reported as an invalid value
  }
  if (staged) {
    const uintptr_t page = (uintptr_t)sysconf(_SC_PAGESIZE);
    const uintptr_t beg = reinterpret_cast<uintptr_t>(d) / page * page;
    const uintptr_t end = (reinterpret_cast<uintptr_t>(d) + bytes + page - 1) / page * page;
    staged = madvise(reinterpret_cast<void*>(beg), end - beg, MADV_POPULATE_WRITE) == 0;
  }
  if (!staged) {
    if (use.owns_lock()) use.unlock();
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, p->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    return e == hipSuccess ? SEMX_OK : mhip(p, e, "parameter download");
  }
  const int64_t pieces = (bytes + kStageBytes - 1) / kStageBytes;
  hipError_t e = hipSuccess;
  for (int64_t k = 0; k < pieces + kStageSlots - 1 && e == hipSuccess; ++k) {
    if (k < pieces) {
      const int64_t n = std::min(kStageBytes, bytes - k * kStageBytes);
      e = hipMemcpyAsync(p->stage + k % kStageSlots * kStageBytes, s + k * kStageBytes, n, hipMemcpyDeviceToHost, p->stream);
      if (e == hipSuccess) e = hipEventRecord(p->staged[k % kStageSlots], p->stream);
    }
    const int64_t o = k - (kStageSlots - 1);  // the piece to copy out
    if (o < 0 || e != hipSuccess) continue;
    e = hipEventSynchronize(p->staged[o % kStageSlots]);
    if (e == hipSuccess)
      std::memcpy(d + o * kStageBytes, p->stage + o % kStageSlots * kStageBytes, std::min(kStageBytes, bytes - o * kStageBytes));
  }
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(p->stream);  // nothing of this call is on its way on return
    return mhip(p, e, "parameter download");
  }
  return SEMX_OK;
}

}  // namespace
}  // namespace semx

using namespace semx;

#define MLP_HIP(p, call)                          \
  do {                                            \
    hipError_t e_ = (call);                       \
    if (e_ != hipSuccess) return mhip(p, e_, #call); \
  } while (0)

extern "C" {

int semx_mlp_create(semx_mlp** out, int nlayers, const int* widths, int max_batch, void* hip_stream) {
  if (!out) return SEMX_EINVAL;
  *out = nullptr;
  if (nlayers < 1 || nlayers > 16 || !widths || max_batch < 1) return SEMX_EINVAL;
  for (int l = 0; l <= nlayers; ++l)
    if (widths[l] < 1 || widths[l] > (1 << 20)) return SEMX_EINVAL;
  semx_mlp* p = new semx_mlp();
  if (hipGetDevice(&p->device) != hipSuccess) {
    delete p;
    return SEMX_EHIP;
  }
  // the allocation-free forward's workspace on this device (resolved once per device)
  if (noalloc_setup(p->device) != hipSuccess) {
    delete p;
    return SEMX_EHIP;
  }
  p->nl = nlayers;
  p->w.assign(widths, widths + nlayers + 1);
  p->max_batch = max_batch;
  p->stream = static_cast<hipStream_t>(hip_stream);
  int64_t off = 0, maxw = 0;
  for (int l = 0; l < nlayers; ++l) {
    p->woff.push_back(off);
    off += (int64_t)p->w[l + 1] * p->w[l];
    p->boff.push_back(off);
    off += p->w[l + 1];
  }
  for (int x : p->w) maxw = std::max<int64_t>(maxw, x);
  p->nparam = off;
  int rc = malloc_buf(p, p->theta, sizeof(float) * off);
  if (!rc) rc = malloc_buf(p, p->theta_bf, sizeof(__bf16) * off);
  if (!rc) rc = malloc_buf(p, p->grad, sizeof(float) * off);
  if (!rc) rc = malloc_buf(p, p->m, sizeof(float) * off);
  if (!rc) rc = malloc_buf(p, p->v, sizeof(float) * off);
  if (!rc) rc = malloc_buf(p, p->g0, sizeof(float) * max_batch * maxw);
  if (!rc) rc = malloc_buf(p, p->g1, sizeof(float) * max_batch * maxw);
  if (!rc) rc = malloc_buf(p, p->scratch, 64);
  if (!rc) rc = malloc_buf(p, p->splitk, sizeof(float) * semx::kSplitWs);
  p->Z.resize(nlayers);
  p->H.resize(nlayers + 1);
  for (int l = 0; l < nlayers && !rc; ++l) {
    rc = malloc_buf(p, p->Z[l], sizeof(float) * max_batch * p->w[l + 1]);
    if (!rc && l + 1 < nlayers) rc = malloc_buf(p, p->H[l + 1], sizeof(float) * max_batch * p->w[l + 1]);
  }
  int widest = 0;  // hidden layer
  for (int l = 1; l < nlayers; ++l) widest = std::max(widest, p->w[l]);
  for (int k = 0; k < 2 && k + 1 < nlayers && !rc; ++k) rc = malloc_buf(p, p->Hb[k], sizeof(__bf16) * max_batch * widest);
  if (rc) {
    semx_mlp_destroy(p);
    return rc;
  }
  // without the pinned pieces downloads go the direct way
  if (sizeof(float) * off >= kStageBytes) {
    void* st = nullptr;
    bool ok = hipHostMalloc(&st, kStageSlots * kStageBytes, hipHostMallocDefault) == hipSuccess;
    for (int k = 0; k < kStageSlots && ok; ++k)
      ok = hipEventCreateWithFlags(&p->staged[k], hipEventDisableTiming) == hipSuccess;
    if (ok) p->stage = static_cast<char*>(st);
    else if (st) (void)hipHostFree(st);
    (void)hipGetLastError();
  }
  *out = p;
  return SEMX_OK;
}

int semx_mlp_destroy(semx_mlp* p) {
  if (!p) return SEMX_OK;
  (void)hipStreamSynchronize(p->stream);
  for (DevBuf* b : {&p->theta, &p->theta_bf, &p->grad, &p->m, &p->v, &p->g0, &p->g1, &p->scratch, &p->splitk,
                    &p->Hb[0], &p->Hb[1]})
    dev_free(*b);
  if (p->stage) (void)hipHostFree(p->stage);
  for (hipEvent_t ev : p->staged)
    if (ev) (void)hipEventDestroy(ev);
  for (auto& b : p->Z) dev_free(b);
  for (auto& b : p->H) dev_free(b);
  delete p;
  return SEMX_OK;
}

const char* semx_mlp_last_error(const semx_mlp* p) { return p ? p->err.c_str() : "null network"; }

int semx_mlp_num_params(semx_mlp* p, int64_t* n) {
  if (!p || !n) return SEMX_EINVAL;
  *n = p->nparam;
  return SEMX_OK;
}

int semx_mlp_set_params(semx_mlp* p, const float* params) {
  if (!p || !params) return SEMX_EINVAL;
  MLP_HIP(p, hipMemcpyAsync(p->theta.p, params, sizeof(float) * p->nparam, hipMemcpyHostToDevice, p->stream));
  to_bf16_kernel<<<g1(p->nparam), 256, 0, p->stream>>>(p->nparam, p->theta.as<float>(), p->theta_bf.as<__bf16>());
  MLP_HIP(p, hipMemsetAsync(p->m.p, 0, sizeof(float) * p->nparam, p->stream));
  MLP_HIP(p, hipMemsetAsync(p->v.p, 0, sizeof(float) * p->nparam, p->stream));
  MLP_HIP(p, hipStreamSynchronize(p->stream));
  return SEMX_OK;
}

int semx_mlp_get_params(semx_mlp* p, float* params) {
  if (!p || !params) return SEMX_EINVAL;
  return download(p, params, p->theta.as<float>());
}

int semx_mlp_get_grads(semx_mlp* p, float* grads) {
  if (!p || !grads) return SEMX_EINVAL;
  return download(p, grads, p->grad.as<float>());
}

int semx_mlp_forward(semx_mlp* p, const float* x_dev, int batch, float* y_dev) {
  if (!p || !x_dev || !y_dev) return SEMX_EINVAL;
  if (batch < 1 || batch > p->max_batch) return mfail(p, SEMX_EINVAL, "forward: batch outside [1, max_batch]");
  for (int l = 0; l < p->nl; ++l) {
    const bool last = l + 1 == p->nl;
    GemmOut O;
    O.C = last ? y_dev : p->Z[l].as<float>();
    if (!last) {
      O.H = p->H[l + 1].as<float>();
      if (bf16_rows(p->w[l + 1])) O.Hb = p->Hb[l & 1].as<__bf16>();
    }
    hipError_t e;
    if (l > 0 && bf16_rows(p->w[l])) {
      const __bf16* h = p->Hb[(l + 1) & 1].as<__bf16>();  // the layer before wrote it
      e = last ? output_layer(p, l, batch, h, O) : layer<kSiluKeep>(p, l, batch, h, O);
    } else {
      const float* h = l > 0 ? p->H[l].as<float>() : x_dev;
      e = last ? output_layer(p, l, batch, h, O) : layer<kSiluKeep>(p, l, batch, h, O);
    }
    if (e != hipSuccess) return mhip(p, e, "mlp forward gemm");
  }
  // the output layer's pre-activation is y itself; keep a copy for backward bookkeeping
  p->x_saved = x_dev;
  p->batch_saved = batch;
  return SEMX_OK;
}

int semx_mlp_forward_noalloc(semx_mlp* p, const float* x_dev, int batch, float* y_dev) {
  if (!p || !x_dev || !y_dev) return SEMX_EINVAL;
  if (batch < 1) return mfail(p, SEMX_EINVAL, "forward_noalloc: batch must be >= 1");
  int hmax = 0;
  for (int l = 1; l < p->nl; ++l) hmax = std::max(hmax, p->w[l]);
  if ((int64_t)batch * hmax > kNoAllocFloats / 2)
    return mfail(p, SEMX_EINVAL, "forward_noalloc: batch x widest hidden layer above " +
                                     std::to_string(kNoAllocFloats / 2) + " floats");
  float* ws = (p->device >= 0 && p->device < kMaxDevices) ? g_scratch_dev[p->device] : nullptr;
  if (!ws) return mfail(p, SEMX_ESTATE, "forward_noalloc: workspace address not resolved on this device");
  float* buf[2] = {ws, ws + kNoAllocFloats / 2};
  const float* h = x_dev;
  for (int l = 0; l < p->nl; ++l) {
    const bool last = l + 1 == p->nl;
    GemmOut O;
    O.C = y_dev;
    O.H = buf[l & 1];
    const hipError_t e = last ? output_layer(p, l, batch, h, O) : layer<kSilu>(p, l, batch, h, O);
    if (e != hipSuccess) return mhip(p, e, "mlp forward_noalloc gemm");
    h = O.H;
  }
  return SEMX_OK;
}

int semx_mlp_backward(semx_mlp* p, const float* dy_dev, int batch) {
  if (!p || !dy_dev) return SEMX_EINVAL;
  if (!p->x_saved || batch != p->batch_saved)
    return mfail(p, SEMX_ESTATE, "backward: call forward with the same batch first (its input must stay alive)");
  const __bf16* W = p->theta_bf.as<__bf16>();
  float* gr = p->grad.as<float>();
  const float* g = dy_dev;
  float* bufs[2] = {p->g0.as<float>(), p->g1.as<float>()};
  int cur = 0;
  for (int l = p->nl - 1; l >= 0; --l) {
    const int in = p->w[l], out = p->w[l + 1];
    // dW = G^T H : C[n_out][k_in] = sum_b G[b][n_out] H[b][k_in]; db = sum_b G
    GemmOut O;
    O.C = gr + p->woff[l];
    O.ldc = in;
    O.db = gr + p->boff[l];
    O.ws = p->splitk.as<float>();
    const float* h = l == 0 ? p->x_saved : p->H[l].as<float>();
    hipError_t e = gemm_launch<float, float, kGradW, false, false>(p->stream, out, in, batch, g, 1, out, h, in, 1, O);
    if (e != hipSuccess) return mhip(p, e, "mlp wgrad gemm");
    if (l == 0) break;
    // dL/dZ = (G W) SiLU'(Z) : C[b][k_in] = sum_o G[b][o] W[o][k_in]
    GemmOut D;
    D.C = bufs[cur];
    D.ldc = in;
    D.Z = p->Z[l - 1].as<float>();
    D.ws = p->splitk.as<float>();
    e = gemm_launch<float, __bf16, kGradZ, true, false>(p->stream, batch, in, out, g, out, 1, W + p->woff[l], in, 1, D);
    if (e != hipSuccess) return mhip(p, e, "mlp dgrad gemm");
    g = bufs[cur];
    cur ^= 1;
  }
  MLP_HIP(p, hipGetLastError());
  return SEMX_OK;
}

int semx_mlp_mse(semx_mlp* p, const float* y_dev, const float* t_dev, int64_t n, float* dy_dev, double* loss) {
  if (!p || !y_dev || !t_dev || n < 1) return SEMX_EINVAL;
  if (!dy_dev && !loss) return SEMX_OK;
  double* d = loss ? p->scratch.as<double>() : nullptr;
  if (d) MLP_HIP(p, hipMemsetAsync(d, 0, sizeof(double), p->stream));
  // the FP64 sum ends in one atomic a block: few blocks; dy alone: all
  const unsigned top = d ? 1024 : 8192;
  mse_kernel<<<std::min(g1(n), top), 256, 0, p->stream>>>(n, y_dev, t_dev, dy_dev, d);
  MLP_HIP(p, hipGetLastError());
  if (loss) {
    MLP_HIP(p, hipMemcpyAsync(loss, d, sizeof(double), hipMemcpyDeviceToHost, p->stream));
    MLP_HIP(p, hipStreamSynchronize(p->stream));
  }
  return SEMX_OK;
}

int semx_mlp_adam(semx_mlp* p, float lr, float beta1, float beta2, float eps, int64_t step) {
  if (!p || step < 1 || !(lr >= 0.0f)) return SEMX_EINVAL;
  const float c1 = 1.0f - std::pow(beta1, (float)step), c2 = 1.0f - std::pow(beta2, (float)step);
  adam_kernel<<<g1(p->nparam), 256, 0, p->stream>>>(p->nparam, lr, beta1, beta2, eps, c1, c2, p->grad.as<float>(),
                                                    p->m.as<float>(), p->v.as<float>(), p->theta.as<float>(),
                                                    p->theta_bf.as<__bf16>());
  MLP_HIP(p, hipGetLastError());
  return SEMX_OK;
}

int semx_mlp_affine(semx_mlp* p, const float* x_dev, int64_t rows, int cols, const float* scale_dev,
                    const float* shift_dev, float* y_dev) {
  if (!p || !x_dev || !y_dev || !scale_dev || !shift_dev || rows < 0 || cols < 1) return SEMX_EINVAL;
  if (rows == 0) return SEMX_OK;
  const int64_t n = rows * (int64_t)cols;
  affine_cols_kernel<<<g1(n) > 8192 ? 8192 : g1(n), 256, 0, p->stream>>>(n, cols, x_dev, scale_dev, shift_dev, y_dev);
  MLP_HIP(p, hipGetLastError());
  return SEMX_OK;
}

int semx_mlp_ensemble(semx_mlp* p, const float* preds_dev, int members, int64_t rows, int cols,
                      const float* scale_dev, const float* shift_dev, float* mean_dev, float* indicator_dev) {
  if (!p || !preds_dev || !scale_dev || !shift_dev || !mean_dev || !indicator_dev || members < 1 || rows < 0 ||
      cols < 1)
    return SEMX_EINVAL;
  if (rows == 0) return SEMX_OK;
  if (rows > INT32_MAX) return mfail(p, SEMX_EINVAL, "ensemble: too many rows");
  ensemble_kernel<<<(unsigned)rows, 256, 0, p->stream>>>(members, rows, cols, preds_dev, scale_dev, shift_dev,
                                                         mean_dev, indicator_dev);
  MLP_HIP(p, hipGetLastError());
  return SEMX_OK;
}

}  // extern "C"
