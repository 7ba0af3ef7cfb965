// MLP policy phase for gfx950: a rendered frame per env in, actions out.
//
// The paper's RL rollouts run an MLP policy beside physics and rendering on
// the same GPU (Evaluation, RL Training, MLP-based RL).  The observation of an
// env is its camera 0 frame as K = 4 W H integers 0..255: the RGB bytes in
// memory order, then the top byte of each 24-bit depth.  Layers:
//   h1 = relu(x W1 + b1)   W1 bfloat16 [K][H], held as panels [K / 32][H][32]
//   h2 = relu(h1 W2 + b2)  float32
//   y  = h2 W3 + b3        float32, A = 3 B outputs
//   a  = a_max clamp(y, -1, 1): the force on body b is a[3b .. 3b+2]
// Layer 1 is the one dense contraction of the step loop (K = 65,536 at
// 128x128); it runs on MFMA (v_mfma_f32_16x16x32_bf16): every observation
// value is an 8-bit integer, exact in bfloat16, so each product is exact and
// only the float32 accumulation rounds.  K is split over workgroups (partial
// sums in float32, added in a fixed order by the head), so that a batch of a
// few hundred envs still fills 256 CUs.  Up to H = 1024, layers 2 and 3 are
// small (H^2 and H A per env) and run on the VALU in one head kernel, one
// workgroup per env.  Wider policies (H = 4096: 16.8 M multiply-adds per env
// in layer 2) run layers 2 and 3 as batched products over all envs on
// float32 MFMA (v_mfma_f32_16x16x4_f32), each split over K like layer 1,
// with small kernels that add the splits in order and apply the bias and the
// activation.
#include "vuda_internal.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace vuda {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 64;      // envs per layer-1 workgroup
constexpr int kCols = 256;     // hidden units per layer-1 workgroup (64 per wave)
constexpr int kKStep = 32;     // k per MFMA
constexpr int kLdsPad = 8;     // bfloat16 between staged rows (the 16 rows of a fragment read then meet every bank)

constexpr int kXcds = 8;        // accelerator complex dies, each with its own L2

// Position of this workgroup in the grid's logical order (x fastest, then
// y, then z).  The dispatcher deals workgroups to the XCDs round-robin in
// launch order; renumbered like this, each XCD takes one contiguous run of
// the logical order, so that the row tiles that share a weight slice (and
// the column tiles that share rows) meet in one L2 instead of eight.
__device__ __forceinline__ int3 xcd_tile() {
  const int total = gridDim.x * gridDim.y * gridDim.z;
  int b = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  if (total % kXcds == 0) b = (b % kXcds) * (total / kXcds) + b / kXcds;
  return make_int3(b % gridDim.x, (b / gridDim.x) % gridDim.y, b / (gridDim.x * gridDim.y));
}

// bfloat16 bits of the integers in the four bytes of w (exact: 8-bit values)
__device__ __forceinline__ uint2 bytes_to_bf16(uint32_t w) {
  // (the compiler turns these into v_cvt_f32_ubyte0..3)
  const uint32_t f0 = __float_as_uint((float)(w & 0xFFu));
  const uint32_t f1 = __float_as_uint((float)((w >> 8) & 0xFFu));
  const uint32_t f2 = __float_as_uint((float)((w >> 16) & 0xFFu));
  const uint32_t f3 = __float_as_uint((float)(w >> 24));
  // the upper halves of (f1, f0) and (f3, f2)
  return make_uint2(__builtin_amdgcn_perm(f1, f0, 0x07060302u), __builtin_amdgcn_perm(f3, f2, 0x07060302u));
}

// One thread's share of the kStage (64 or 32) observation values that a stage
// takes of a frame: kStage / 4 of them, a run (RGB part: bytes in a row) or
// fours (depth part: words 16 i + 4 q, so that the threads of a row read whole
// sectors).  The RGB part ends at 3 W H, a multiple of kStage, so a stage is on
// one side; only the members of that side are loaded and read.  They are
// loaded a stage ahead and converted only after that stage's MFMAs, so that
// the wait for them does not come before the MFMAs.
struct __attribute__((packed, aligned(8))) Bytes16 {  // a frame starts on a multiple of 8 bytes
  uint32_t w[4];
};
template <int kStage>
union ObsRaw {
  Bytes16 c;                // kStage 64
  uint2 c2;                 // kStage 32
  uint4 d[kStage / 16];
};

// q of 4: the thread's place in its row of kStage values at k
template <bool kRgb, int kStage>
__device__ __forceinline__ void obs_load(ObsRaw<kStage>& r, const uint8_t* rgb, const uint32_t* depth, int k, int q,
                                         int krgb) {
  if constexpr (kRgb) {
    if constexpr (kStage == 64) r.c = *(const Bytes16*)(rgb + k + 16 * q);
    else r.c2 = *(const uint2*)(rgb + k + 8 * q);
  } else {
    // (a load for a stage still in the RGB part reads depth words 0 on)
    const uint32_t* p = depth + max(k - krgb, 0) + 4 * q;
#pragma unroll
    for (int i = 0; i < kStage / 16; ++i) r.d[i] = *(const uint4*)(p + 16 * i);
  }
}

// the values as bfloat16 into the staged row
template <bool kRgb, int kStage>
__device__ __forceinline__ void obs_stage(const ObsRaw<kStage>& r, uint16_t* row, int q) {
  if constexpr (kRgb) {
    const uint32_t w[4] = {kStage == 64 ? r.c.w[0] : r.c2.x, kStage == 64 ? r.c.w[1] : r.c2.y,
                           kStage == 64 ? r.c.w[2] : 0u, kStage == 64 ? r.c.w[3] : 0u};
#pragma unroll
    for (int i = 0; i < kStage / 32; ++i) {
      const uint2 lo = bytes_to_bf16(w[2 * i]), hi = bytes_to_bf16(w[2 * i + 1]);
      *(uint4*)(row + kStage / 4 * q + 8 * i) = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kStage / 16; ++i) {
      // byte 2 of each depth word: its top byte (background 0xFFFFFFFF gives 255)
      const uint32_t w = __builtin_amdgcn_perm(r.d[i].y, r.d[i].x, 0x0c0c0602u) |
                         (__builtin_amdgcn_perm(r.d[i].w, r.d[i].z, 0x0c0c0602u) << 16);
      *(uint2*)(row + 16 * i + 4 * q) = bytes_to_bf16(w);
    }
  }
}

// Layer 1: partial sums over k in [s Kc, (s+1) Kc) for kRows envs and kCols
// hidden units.  Wave w owns units n0 + 64 w .. + 63 of all kRows envs: 4 x 4
// blocks of 16 x 16, one MFMA each per 32 k.  kStage k are staged between two
// barriers.  At 1,024 envs of 128x128 the reads of W1 bound it (each tile of 64
// envs reads its columns' weights from L2, 8.6 GB at hidden 4096): 707 us at
// hidden 4096 (778 TFLOP/s), which took 887 in stages of 32 with a branch
// around each load.  Tiles of 128 envs in the same splits were slower (one wave
// per SIMD: 1,101 us for the launch against 1,006), and so were fragments a
// stage ahead (two waves per SIMD in place of three: 1,077).
template <int kStage>
__global__ __launch_bounds__(256, 2) void policy_l1_kernel(WorldDev W, PolicyLaunch L) {
  constexpr int kRb = kRows / 16;
  constexpr int kLdsRow = kStage + kLdsPad;
  __shared__ __align__(16) uint16_t sA[2][kRows * kLdsRow];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int3 tile = xcd_tile();
  const int m0 = tile.x * kRows;
  const int n0 = tile.y * kCols + 64 * wave;
  const int s = tile.z;
  const int krgb = L.krgb, Kc = L.kchunk;
  const int kbeg = s * Kc, kend = kbeg + Kc;
  const int nstages = Kc / kStage;
  // staging role: row r, place q4 of each stage
  const int r = tid >> 2, q4 = tid & 3;
  // rows past M (a ragged last tile) read row M - 1's frame: a row of A only
  // reaches the same row of the product, and those rows are not stored
  const int64_t off = W.cams[W.envs[L.envs[min(m0 + r, L.M - 1)]].cam_off].pix_off;
  const uint8_t* rgb = W.rgb + 3 * off;
  const uint32_t* dep = W.depth + off;
  // B fragments: lane (column n0 + 16 cb + lane % 16, k + 8 (lane / 16) .. + 7),
  // in the panel of step k at (k / 32) 32 H
  const int64_t panel = (int64_t)kKStep * L.H;
  const uint16_t* bpan = L.w1t + (kbeg / kKStep) * panel;  // uniform: the panel in bn
  uint32_t bcol[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
    bcol[cb] = (uint32_t)(min(n0 + 16 * cb + (lane & 15), L.H - 1) * kKStep + 8 * (lane >> 4));
  f32x4 acc[kRb][4];
#pragma unroll
  for (int i = 0; i < kRb; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  ObsRaw<kStage> raw;
  // W1 fragments run one step of 32 k ahead of the MFMAs that use them (those
  // loaded by the last step of a chunk are the next chunk's, or the padding
  // panel's, and unused)
  uint4 bn[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) bn[cb] = *(const uint4*)(bpan + bcol[cb]);
  if (kbeg < krgb) {
    obs_load<true, kStage>(raw, rgb, dep, kbeg, q4, krgb);
    obs_stage<true, kStage>(raw, &sA[0][r * kLdsRow], q4);
  } else {
    obs_load<false, kStage>(raw, rgb, dep, kbeg, q4, krgb);
    obs_stage<false, kStage>(raw, &sA[0][r * kLdsRow], q4);
  }
  __syncthreads();
  // One stage: the next stage's observation bytes (of the kind the template
  // argument names) go out, this stage's MFMAs run, then the bytes are
  // converted and staged.  No branch surrounds a load, so no register copy of
  // a loaded value (and no wait for it) lands before the MFMAs.  The last
  // stage reloads itself (in bounds, unused).
  const auto step = [&](auto next, int t) {
    constexpr bool kNextRgb = decltype(next)::value;
    const int buf = t & 1;
    const int knext = min(kbeg + (t + 1) * kStage, kend - kStage);
    obs_load<kNextRgb, kStage>(raw, rgb, dep, knext, q4, krgb);
    // First of all, so that the wait for them leaves the W1 loads of the step under
    // way (put after those, layer 1 of 100 envs of 104x100 at hidden 300 took 227
    // us, like this 198; stages of two steps are ordered so by themselves).
    if constexpr (kStage == kKStep) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kStage / kKStep; ++q) {
      uint4 b[4];
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) b[cb] = bn[cb];
      bpan += panel;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) bn[cb] = *(const uint4*)(bpan + bcol[cb]);
      // the loads go out before the MFMAs
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rb = 0; rb < kRb; ++rb) {
        const bf16x8 a = __builtin_bit_cast(
            bf16x8, *(const uint4*)&sA[buf][(16 * rb + (lane & 15)) * kLdsRow + kKStep * q + 8 * (lane >> 4)]);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
          acc[rb][cb] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b[cb]), acc[rb][cb], 0, 0, 0);
      }
      // nothing below moves above the MFMAs
      __builtin_amdgcn_sched_barrier(0);
    }
    obs_stage<kNextRgb, kStage>(raw, &sA[buf ^ 1][r * kLdsRow], q4);
    __syncthreads();
  };
  // stages whose successor is in the RGB part, then the rest
  const int t_rgb = min(max((krgb - kbeg) / kStage, 0), nstages);  // stages in the RGB part
  int t = 0;
  for (; t < t_rgb - 1; ++t) step(std::true_type{}, t);
  for (; t < nstages; ++t) step(std::false_type{}, t);
  // D layout: lane holds rows 4 (lane / 16) + i of a block, column lane % 16
  float* P = L.partial + (int64_t)s * L.M * L.H;
#pragma unroll
  for (int rb = 0; rb < kRb; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const int n = n0 + 16 * cb + (lane & 15);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + 16 * rb + 4 * (lane >> 4) + i;
        if (m < L.M && n < L.H) P[(int64_t)m * L.H + n] = acc[rb][cb][i];
      }
    }
}

// sum_{s < n} p[s * stride], in s order; the loads go out kBatch at a time
// (independent, so their latencies overlap), the additions stay in order
template <int kBatch>
__device__ __forceinline__ float ordered_strided_sum(const float* p, int64_t stride, int n) {
  float acc = 0.0f;
  int s = 0;
  for (; s + kBatch <= n; s += kBatch) {
    float v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) v[u] = p[(s + u) * stride];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) acc = acc + v[u];
  }
  for (; s < n; ++s) acc = acc + p[s * stride];
  return acc;
}

// acc[e] = sum_{i < n} x[e pitch + i] w[i * stride] in i order (x in LDS, rows
// on 16 bytes), loads kBatch at a time
template <int kBatch, int kEnvs>
__device__ __forceinline__ void ordered_dots(const float* x, int pitch, const float* w, int64_t stride, int n,
                                             float (&acc)[kEnvs]) {
#pragma unroll
  for (int e = 0; e < kEnvs; ++e) acc[e] = 0.0f;
  int i = 0;
  // (one copy of the batch: the kernel runs each line a few times per launch,
  // and unrolled further it waits for its instructions)
#pragma unroll 1
  for (; i + kBatch <= n; i += kBatch) {
    float v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) v[u] = w[(i + u) * stride];
#pragma unroll
    for (int u = 0; u < kBatch; u += 4)
#pragma unroll
      for (int e = 0; e < kEnvs; ++e) {
        const float4 q = *(const float4*)(x + e * pitch + i + u);
        acc[e] = acc[e] + q.x * v[u];
        acc[e] = acc[e] + q.y * v[u + 1];
        acc[e] = acc[e] + q.z * v[u + 2];
        acc[e] = acc[e] + q.w * v[u + 3];
      }
  }
#pragma unroll 1
  for (; i < n; ++i) {
    const float v = w[i * stride];
#pragma unroll
    for (int e = 0; e < kEnvs; ++e) acc[e] = acc[e] + x[e * pitch + i] * v;
  }
}

__device__ __forceinline__ float relu(float v) { return v > 0.0f ? v : 0.0f; }

// a_max clamp(y, -1, 1) for a finite y
__device__ __forceinline__ float action_of(float y, float a_max) {
  return a_max * __builtin_amdgcn_fmed3f(y, -1.0f, 1.0f);
}

// Layers 2 and 3 of kEnvs envs per workgroup (blockDim = H rounded up to 64,
// at most 1024): the split-K partials added in split order, then every unit
// on its own lane, its dot products in index order.  The reads bound it: W2
// from L2 by each workgroup (268 MB a launch at 1,024 envs of H = 256 and one
// env each, 4.3 GB at H = 1,024: layer 1 and head 237 us, 167 with two), the
// partials (33 MB at 250 envs in 128 splits) from memory.  Batches of 64 loads
// or of two in flight were slower (the head alone 20 us where it takes 16).
// (Splitting each sum over more lanes was slower too, and would reorder it.)
template <int kEnvs>
__global__ __launch_bounds__(1024) void policy_head_kernel(WorldDev W, PolicyLaunch L) {
  extern __shared__ __align__(16) float sh[];  // h1, h2 [kEnvs][pitch]
  const int m0 = blockIdx.x * kEnvs;
  if (m0 >= L.M) return;
  const int j = threadIdx.x, H = L.H, pitch = (H + 3) & ~3;
  float* h1 = sh;
  float* h2 = sh + kEnvs * pitch;
  // (rows past M, in a ragged last workgroup, repeat the last one and are not
  // written)
  if (j < H) {
#pragma unroll
    for (int e = 0; e < kEnvs; ++e) {
      const int m = min(m0 + e, L.M - 1);
      const float s1 = ordered_strided_sum<16>(L.partial + (int64_t)m * H + j, (int64_t)L.M * H, L.splits);
      h1[e * pitch + j] = relu(s1 + L.b1[j]);
    }
  }
  __syncthreads();
  if (j < H) {
    float acc[kEnvs];
    ordered_dots<32, kEnvs>(h1, pitch, L.w2 + j, H, H, acc);
#pragma unroll
    for (int e = 0; e < kEnvs; ++e) h2[e * pitch + j] = relu(acc[e] + L.b2[j]);
  }
  __syncthreads();
  // one (env, action) pair per lane
  for (int i = j; i < kEnvs * L.A; i += blockDim.x) {
    const int e = kEnvs == 1 ? 0 : i / L.A, q = i - e * L.A;
    float acc[1];
    ordered_dots<32, 1>(h2 + e * pitch, pitch, L.w3 + q, L.A, H, acc);
    if (kEnvs == 1 || m0 + e < L.M)
      W.actions[(int64_t)L.envs[m0 + e] * L.A + q] = action_of(acc[0] + L.b3[q], L.a_max);
  }
  if (j < kEnvs && m0 + j < L.M) W.act_on[L.envs[m0 + j]] = 1;
}

// ---- layers 2 and 3 as batched products (H > 1024) ----

// out[m][j] = relu(sum_s P[s][m][j] + b[j]) for j < N, P with row stride N
__global__ __launch_bounds__(256) void policy_hidden_kernel(const float* P, int splits, int M, int N, const float* b,
                                                            float* out) {
  const int m = blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (m >= M || j >= N) return;
  const int64_t at = (int64_t)m * N + j;
  out[at] = relu(ordered_strided_sum<16>(P + at, (int64_t)M * N, splits) + b[j]);
}

// actions of row m: a_max clamp(sum_s P[s][m][q] + b3[q]) for q < A, P with
// row stride ldp; and the env's force flag
__global__ __launch_bounds__(256) void policy_act_kernel(WorldDev W, PolicyLaunch L, const float* P, int splits,
                                                         int ldp) {
  const int m = blockIdx.x;
  if (m >= L.M) return;
  const int env = L.envs[m];
  for (int q = threadIdx.x; q < L.A; q += blockDim.x) {
    const float y = ordered_strided_sum<16>(P + (int64_t)m * ldp + q, (int64_t)L.M * ldp, splits);
    W.actions[(int64_t)env * L.A + q] = action_of(y + L.b3[q], L.a_max);
  }
  if (threadIdx.x == 0) W.act_on[env] = 1;
}

constexpr int kDTile = 64;   // rows and columns of a dense-product workgroup tile
constexpr int kDStep = 16;   // k per staged step
constexpr int kAPitch = 20;  // floats per staged A row (16 + 4: lanes of one read hit distinct banks)
constexpr int kBPitch = 80;  // floats per staged B row (64 + 16)

// P[s][m][n] = sum_{k in chunk s} X[m][k] B[k][n] for m < M, n < ldb: X is
// [M][K] and B [K][ldb] row-major float32, K and ldb multiples of 64, chunk
// a multiple of kDStep.  Workgroup: a 64 x 64 tile of one chunk; wave w
// owns the 32 x 32 quadrant (w & 1, w >> 1), 2 x 2 blocks of 16 x 16.
__global__ __launch_bounds__(256) void policy_dense_kernel(const float* X, const float* B, int M, int K, int ldb,
                                                           int kchunk, float* P) {
  __shared__ __align__(16) float sA[2][kDTile * kAPitch];
  __shared__ __align__(16) float sB[2][kDStep * kBPitch];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int3 tile = xcd_tile();
  const int m0 = tile.x * kDTile, n0 = tile.y * kDTile, s = tile.z;
  const int wm = 32 * (wave & 1), wn = 32 * (wave >> 1);
  const int kbeg = s * kchunk, nsteps = kchunk / kDStep;
  // staging roles: X row ar, columns ac .. ac+3; B row br, columns bc .. bc+3
  const int ar = tid >> 2, ac = 4 * (tid & 3);
  const int br = tid >> 4, bc = 4 * (tid & 15);
  // rows past M read row M - 1: a row of X only reaches the same row of
  // the product, and those rows are not stored
  const float* xa = X + (int64_t)min(m0 + ar, M - 1) * K + ac;
  const float* bb = B + (int64_t)br * ldb + n0 + bc;
  float4 ra = *(const float4*)(xa + kbeg);
  float4 rb = *(const float4*)(bb + (int64_t)kbeg * ldb);
  *(float4*)&sA[0][ar * kAPitch + ac] = ra;
  *(float4*)&sB[0][br * kBPitch + bc] = rb;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  __syncthreads();
  for (int t = 0; t < nsteps; ++t) {
    const int buf = t & 1;
    if (t + 1 < nsteps) {
      const int k = kbeg + (t + 1) * kDStep;
      ra = *(const float4*)(xa + k);
      rb = *(const float4*)(bb + (int64_t)k * ldb);
    }
    // operands of v_mfma_f32_16x16x4_f32: lane l holds A[l % 16][l / 16]
    // and B[l / 16][l % 16] of the 16 x 4 and 4 x 16 blocks
#pragma unroll
    for (int kk = 0; kk < kDStep; kk += 4) {
      float a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = sA[buf][(wm + 16 * i + (lane & 15)) * kAPitch + kk + (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = sB[buf][(kk + (lane >> 4)) * kBPitch + wn + 16 * j + (lane & 15)];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    if (t + 1 < nsteps) {
      *(float4*)&sA[buf ^ 1][ar * kAPitch + ac] = ra;
      *(float4*)&sB[buf ^ 1][br * kBPitch + bc] = rb;
    }
    __syncthreads();
  }
  // D layout: lane holds rows 4 (lane / 16) + r of a block, column lane % 16
  float* Ps = P + (int64_t)s * M * ldb;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn + 16 * j + (lane & 15);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        if (m < M) Ps[(int64_t)m * ldb + n] = acc[i][j][r];
      }
    }
}

}  // namespace

hipError_t launch_policy(const WorldDev& w, const PolicyLaunch& l, hipStream_t s, LaunchEvents* ev) {
  if (l.M <= 0) return hipSuccess;
  const dim3 g1((l.M + kRows - 1) / kRows, (l.H + kCols - 1) / kCols, l.splits);
  // Stages of 64 values where the RGB part and each chunk are whole stages;
  // frames of an odd multiple of 32 pixels and chunks of an odd number of steps
  // take stages of 32 (a barrier per 16 MFMAs).
  const bool whole = l.krgb % 64 == 0 && l.kchunk % 64 == 0;
  if (whole) timed_launch(ev, true, false, policy_l1_kernel<64>, g1, dim3(256), 0, s, w, l);
  else timed_launch(ev, true, false, policy_l1_kernel<32>, g1, dim3(256), 0, s, w, l);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!l.layered) {
    const int threads = (l.H + 63) / 64 * 64;
    // Two envs per workgroup, which halve the reads of the weights, from 2^18 hidden
    // units over the batch on.  Layer 1 and head in us, one env and two (frames of
    // 64x64 up to hidden 512, of 8x8 above): 1,024 at H = 256 40.7 and 36.8, 600 at
    // 512 68.6 and 60.0, 410 at 640 48.9 and 38.0, 300 at 1,024 101 and 67, 4,096 at
    // 64 15.8 and 15.3; from there on two were faster at every size measured.  Below
    // it one is ahead while it gives each CU a workgroup or each SIMD two waves at
    // most (256 at 256 31.5 and 35.0, 512 at 256 32.4 and 32.6, 256 at 512 41.0 and
    // 42.0, 192 at 1,024 66.1 and 67.2), two once it gives them more (1,000 at 256
    // 41.0 and 36.8, 800 at 256 46.6 and 43.1, 300 at 512 51.9 and 45.0): the line
    // leaves those to one.  Four envs were slower everywhere.
    const int envs = (int64_t)l.M * l.H >= 1 << 18 ? 2 : 1;
    const dim3 g((l.M + envs - 1) / envs), b(threads);
    const uint32_t lds = (uint32_t)(2 * envs * ((l.H + 3) & ~3) * sizeof(float));
    if (envs == 2) timed_launch(ev, false, true, policy_head_kernel<2>, g, b, lds, s, w, l);
    else timed_launch(ev, false, true, policy_head_kernel<1>, g, b, lds, s, w, l);
    return hipGetLastError();
  }
  // h1, then layer 2 into the partials (free again once h1 is made), h2,
  // layer 3, the actions
  const int mt = (l.M + kDTile - 1) / kDTile;
  const dim3 gh((l.H + 255) / 256, l.M);
  hipLaunchKernelGGL(policy_hidden_kernel, gh, dim3(256), 0, s, l.partial, l.splits, l.M, l.H, l.b1, l.h1);
  hipLaunchKernelGGL(policy_dense_kernel, dim3(mt, l.H / kDTile, l.s2), dim3(256), 0, s, l.h1, l.w2, l.M, l.H, l.H,
                     l.H / l.s2, l.partial);
  hipLaunchKernelGGL(policy_hidden_kernel, gh, dim3(256), 0, s, l.partial, l.s2, l.M, l.H, l.b2, l.h2);
  hipLaunchKernelGGL(policy_dense_kernel, dim3(mt, l.Ap / kDTile, l.s3), dim3(256), 0, s, l.h2, l.w3p, l.M, l.H,
                     l.Ap, l.H / l.s3, l.partial);
  timed_launch(ev, false, true, policy_act_kernel, dim3(l.M), dim3(256), 0, s, w, l, (const float*)l.partial, l.s3, l.Ap);
  return hipGetLastError();
}

}  // namespace vuda
