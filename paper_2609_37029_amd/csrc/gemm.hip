// Weight-streaming GEMMs of the drafter: C[M][N] = A[M][K] . W[N][K]^T with
// fp32 accumulation, for the boundary fusion, the QKV / O / gate-up / down
// projections of every layer and the vocabulary head (Sec. 2.3, App. B.1).
//
// These GEMMs stream each weight once from HBM and reuse it across all M =
// batch x B rows: loader waves stage the weights through LDS by DMA while
// compute waves read the activation rows straight into MFMA fragments
// (frag_gemm below, tiles of 16 to 256 rows); the vocabulary head above 64 rows
// has a kernel of its own (gemm_tiled_kernel). fp32 (gemm_f32_kernel): fp32 MFMA
// on operands loaded straight into registers, with the same epilogues.
//
// Epilogues: EPI_STORE writes fp32 (split-K partials); EPI_LOGITS writes the
// fp32 logits; EPI_SWIGLU reads the gate and up rows of w_gate_up interleaved
// in 16-row blocks (each wave's n-tile pairs are matching gate / up columns)
// and writes silu(gate) * up in the activation dtype. The vocabulary head's
// epilogue can also take each row's first argmax (greedy sampling) or form
// the 16-token chunk log-masses of the two-level draw (Eq. 8).
#include "ldr_internal.h"

#include <type_traits>
#include <utility>

namespace ldr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16 bytes as a native vector (HIP's uint4 is a struct whose copies become
// memcpys that keep arrays of them in scratch).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;   // K step: one LDS stage, two MFMA k-steps
// Interleaved N index of the SwiGLU GEMM -> row of w_gate_up.
__device__ inline int swiglu_row(int c, int mlp) {
  const int blk = c >> 4, out = ((blk >> 1) << 4) | (c & 15);
  return (blk & 1) ? mlp + out : out;
}

__device__ inline float silu(float x) { return x / (1.f + expf(-x)); }
// silu of the bf16 GEMMs, whose result is rounded to bf16: the hardware
// exp2 and reciprocal (about 1 ulp each in fp32) instead of expf and an IEEE
// division, a few VALU operations in place of some thirty.
__device__ inline float silu_bf16(float x) {
  return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x * -1.44269504088896341f));
}

// One 16 x 16 x 32 MFMA of an activation fragment and a weight fragment.
// TRANS (the SwiGLU GEMMs) takes the weight fragment first, so the
// accumulator tile is transposed: lane l holds columns 4 (l / 16) .. + 3 of
// row l % 16, 4 consecutive outputs of one row. Otherwise lane l holds rows
// 4 (l / 16) .. + 3 of column l % 16. The products and sums are the same
// either way. (The SwiGLU epilogue writes 4 consecutive bf16 at a time; the
// fp32 split-K stores of 4 consecutive columns per lane measured 1 us slower
// for the QKV projection, whose rows lie 24 KB apart, and no faster for the
// others.)
template <bool TRANS>
__device__ __forceinline__ void mma_tile(const bf16x8& a, const bf16x8& w, f32x4& acc) {
  acc = TRANS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, acc, 0, 0, 0)
              : __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w, acc, 0, 0, 0);
}

// Stores one tile's accumulators: EPI_STORE / EPI_LOGITS fp32 (split z at
// z * split_stride), EPI_SWIGLU silu(gate) * up in the activation dtype,
// row-major or in the fragment layout of [M][mlp] (a.out_frag). The fp32
// tiles are in the MFMA's own layout (lane l: rows 4 (l / 16) .. + 3 of column
// l % 16); the SwiGLU tiles are transposed (mma_tile), so a lane writes 4
// consecutive bf16 of one row (8 bytes in either layout). SwiGLU waves whose
// tile lies inside the matrix skip the per-element tests (a wave-uniform
// branch).
template <int MTW, int NTW, int WM, int WN, int EPI>
__device__ __forceinline__ void store_tile(const GemmArgs& a, int n0, int m0, int z,
                                           const f32x4 (&acc)[MTW][NTW]) {
  constexpr int TM = MTW * 16, TN = NTW * 16;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  if constexpr (EPI == EPI_STORE || EPI == EPI_LOGITS) {
    const int crow = (lane >> 4) * 4, ccol = lane & 15;
    const int rb = m0 + wm * TM + crow, cb = n0 + wn * TN + ccol;
    float* out = static_cast<float*>(a.out) + (long)z * a.split_stride + (long)rb * a.ldo + cb;
    if (m0 + wm * TM + TM <= a.M && n0 + wn * TN + TN <= a.N) {
      // the wave's tile lies inside the matrix: no per-element tests
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float* o = out + (long)(i * 16 + v) * a.ldo;
#pragma unroll
          for (int j = 0; j < NTW; ++j) o[j * 16] = acc[i][j][v];
        }
    } else {
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int j = 0; j < NTW; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (rb + i * 16 + v < a.M && cb + j * 16 < a.N)
              out[(long)(i * 16 + v) * a.ldo + j * 16] = acc[i][j][v];
    }
  } else {
    const int r0 = m0 + wm * TM + (lane & 15), c4 = (lane >> 4) * 4;
    uint16_t* out = static_cast<uint16_t*>(a.out);
    // n-tiles j (gate) and j + 1 (up) hold the same 16 output columns
    const int ob = (n0 + wn * TN) / 2 + c4;
    const bool full = m0 + wm * TM + TM <= a.M && (n0 + wn * TN + TN) / 2 <= a.mlp &&
                      (a.out_frag || ((a.ldo & 3) == 0 &&
                                      (reinterpret_cast<uintptr_t>(a.out) & 7) == 0));
    auto put = [&](auto full_t) {
      constexpr bool FULL = decltype(full_t)::value;
#pragma unroll
      for (int j = 0; j < NTW; j += 2) {
        const int col = ob + j * 8;
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
          const int row = r0 + i * 16;
          if (!FULL && (row >= a.M || col >= a.mlp)) continue;
          // col % 8 is 0 or 4: the 4 elements stay inside one 8-element run
          // of the fragment layout
          const long off = a.out_frag ? ((long)(row >> 4) * (a.mlp >> 5) + (col >> 5)) * 512 +
                                            ((((col >> 3) & 3) << 4) | (row & 15)) * 8 + (col & 7)
                                      : (long)row * a.ldo + col;
          uint16_t h[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) h[v] = f32_to_bf16(silu_bf16(acc[i][j][v]) * acc[i][j + 1][v]);
          if (FULL) {
            *reinterpret_cast<uint2*>(out + off) =
                uint2{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (col + v < a.mlp) out[off + v] = h[v];
          }
        }
      }
    };
    if (full) put(std::true_type{});
    else put(std::false_type{});
  }
}

// The tile (x, y) and K split z of this workgroup. Workgroups go to the 8
// XCDs in turn by linear id (id mod 8), and each XCD has its own L2: the
// linear ids are renumbered so that XCD c takes the c-th eighth of the tiles
// in (z, x, y) order. A K split's activation columns are then read into one
// or two XCDs' L2 instead of all eight, and the row tiles of one column tile
// (M above one tile) share their weight columns in one L2. Returns l, the tile's
// place in that order.
__device__ __forceinline__ int xcd_tile(int& x, int& y, int& z) {
  const int gx = gridDim.x, gy = gridDim.y;
  const int total = gx * gy * gridDim.z;
  const int lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int q = total >> 3, r = total & 7, c = lin & 7, slot = lin >> 3;
  const int l = c < r ? c * (q + 1) + slot : r * (q + 1) + (c - r) * q + slot;
  y = l % gy;
  x = (l / gy) % gx;
  z = l / (gx * gy);
  return l;
}

// fp32 on v_mfma_f32_16x16x4_f32 (full fp32 products and sums). A workgroup
// owns MT x NT tiles of 16 x 16 outputs; its 8 waves take the 16-deep K chunks
// in turn and add their tiles up in LDS, in wave order. A lane loads 16 bytes of
// a row's chunk (4 lanes a row), its four elements serving four MFMAs: the order
// of the contraction index is free as long as both operands share it. No LDS
// staging: these models are small, a launch is one load latency, U chunks of
// loads in flight a wave, and the reduction. What bounds it is that latency: a
// SIMT kernel that staged 16-deep steps through LDS, one round trip each, took
// 24.4 us for the Tiny model's SwiGLU GEMM (8 x 2048 x 256) and 5.2 now.
constexpr int kF32Waves = 8;
template <int MT, int NT, int EPI>
__global__ void __launch_bounds__(kF32Waves * 64) gemm_f32_kernel(GemmArgs a) {
  static_assert(EPI != EPI_SWIGLU || NT % 2 == 0, "swiglu pairs");
  constexpr int U = 4;
  __shared__ float red[kF32Waves][MT * NT * 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.x * NT * 16, m0 = blockIdx.y * MT * 16, z = blockIdx.z;
  const int kper = a.K / a.splits, kbeg = z * kper, chunks = kper / 16;
  const int lr = lane & 15, kq = (lane >> 4) * 4;
  const float* ap[MT];
  const float* wp[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)   // rows past M repeat the last one (not stored)
    ap[i] = static_cast<const float*>(a.A) + (long)min(m0 + i * 16 + lr, a.M - 1) * a.lda + kbeg + kq;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int gn = min(n0 + j * 16 + lr, a.N - 1);
    const int row = EPI == EPI_SWIGLU ? swiglu_row(gn, a.mlp) : gn;
    wp[j] = static_cast<const float*>(a.W) + (long)row * a.ldw + kbeg + kq;
  }
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = wave; c0 < chunks; c0 += U * kF32Waves) {
    f32x4 av[U][MT], wv[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {   // chunks past the end repeat the last one (not used)
      const int k = min(c0 + u * kF32Waves, chunks - 1) * 16;
#pragma unroll
      for (int i = 0; i < MT; ++i) av[u][i] = *reinterpret_cast<const f32x4*>(ap[i] + k);
#pragma unroll
      for (int j = 0; j < NT; ++j) wv[u][j] = *reinterpret_cast<const f32x4*>(wp[j] + k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c0 + u * kF32Waves < chunks)   // wave-uniform
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][i][e], wv[u][j][e], acc[i][j],
                                                               0, 0, 0);
  }
  // tile (i, j): element (row (lane / 16) * 4 + v, column lane % 16) at v * 64 + lane
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][(i * NT + j) * 256 + v * 64 + lane] = acc[i][j][v];
  __syncthreads();
  auto total = [&](int e) {
    float s = red[0][e];
#pragma unroll
    for (int w = 1; w < kF32Waves; ++w) s += red[w][e];
    return s;
  };
  constexpr int NP = EPI == EPI_SWIGLU ? NT / 2 : NT;   // output column tiles
  for (int o = tid; o < MT * NP * 256; o += kF32Waves * 64) {
    const int t = o >> 8, i = t / NP, j = t % NP, l = o & 63, v = (o >> 6) & 3;
    const int row = m0 + i * 16 + (l >> 4) * 4 + v;
    if (row >= a.M) continue;
    if constexpr (EPI == EPI_SWIGLU) {   // column tiles 2 j (gate) and 2 j + 1 (up)
      const int col = (n0 >> 1) + j * 16 + (l & 15);
      const int e = (i * NT + 2 * j) * 256 + v * 64 + l;
      if (col < a.mlp)
        static_cast<float*>(a.out)[(long)row * a.ldo + col] = silu(total(e)) * total(e + 256);
    } else {
      const int col = n0 + j * 16 + (l & 15);
      if (col < a.N)
        static_cast<float*>(a.out)[(long)z * a.split_stride + (long)row * a.ldo + col] =
            total((i * NT + j) * 256 + v * 64 + l);
    }
  }
}

template <int N> __device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ inline void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14)); }
__device__ inline void sched_fence() { __builtin_amdgcn_sched_barrier(0); }
__device__ inline void group_barrier() {
  sched_fence();
  __builtin_amdgcn_s_barrier();
  sched_fence();
}

#define LDR_GP(p) ((__attribute__((address_space(1))) void*)(p))
#define LDR_LP(p) ((__attribute__((address_space(3))) void*)(p))

// ---------------------------------------------------------------------------
// GEMM with the activation rows in the fragment layout.
//
// In the fragment layout of a [M][K] bf16 matrix (rows padded to 16), the
// 16 x 32 block of rows 16 r .. and columns 32 c .. is 1 KB at element
// (r * (K / 32) + c) * 512, its 16-byte chunk l holding row 16 r + (l & 15),
// columns 32 c + (l >> 4) * 8 .. + 8: the A operand of v_mfma_f32_16x16x32_bf16
// for lane l, so a wave loads an A fragment from global memory with one fully
// coalesced 16-byte load per lane. That is, element (m, k) sits at
// ((m >> 4) * (K >> 5) + (k >> 5)) * 512 + ((((k >> 3) & 3) << 4) | (m & 15)) * 8
// + (k & 7). The residual norms, the attention output and the SwiGLU GEMM write
// their rows in that layout for the GEMM that reads them.
//
// A workgroup owns BM rows x BN columns of the output and a 1/splits share of
// K, in steps of 64. NW compute waves own MTW 16-row tiles each: their A
// fragments go straight to registers, FRA steps ahead (private, so no LDS),
// and they read all BN weight rows of a step from LDS. NL loader waves only
// stage the weights by DMA (global_load_lds, 8 rows of 128 bytes per
// instruction, 16-byte chunk c of row r at c ^ (r & 7)) into a ring of NB
// stages, NB - 1 steps ahead. A wave that issued the weight DMA itself
// between its MFMAs ran them at about half their rate; with the DMA in waves
// of its own the compute waves keep most of it.
// BM follows M (16, 32, 64, 128 or 256 rows): below 256 the GEMM is the weight
// stream alone, and the activation rows' loads share its path into the CU, so
// a tile reads no more of them than it has rows. (64 rows, Qwen3-8B, against
// 256-column tiles of a kernel that staged both operands through registers and
// LDS: gate/up 64.7 -> 47.2 us, the step 1100 -> 899 us; 80 rows, against 256-row
// tiles: the step 1021 -> 939 us.) A may also be row-major (ROWA: the boundary states in the
// arena; every GEMM of at most 16 rows).
// Ordering: at step kt every wave waits for its own share of what the step
// needs (a loader: its DMA of stage kt, with the NB - 2 later stages still in
// flight; a compute wave: its A loads of stage kt and its LDS reads of step
// kt - 1), then the step's barrier. After it the loaders refill the buffer of
// stage kt - 1, whose readers are past the barrier, with stage kt + NB - 1,
// and the compute waves read stage kt. Both roles meet the same nk barriers.
template <class F, int... P>
__device__ __forceinline__ void for_phases(F&& f, std::integer_sequence<int, P...>) {
  (f(std::integral_constant<int, P>{}), ...);
}

template <int N> __device__ inline void wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

constexpr int kFragLoaders = 4;   // loader waves

// NW compute waves of MTW 16-row tiles each; ROWA: activations row-major
// (row stride lda) instead of the fragment layout.
template <int MTW, int NTW, int EPI, int FRA, int NL, int NB, int NW, bool ROWA>
__device__ __forceinline__ void frag_gemm(const GemmArgs& a) {
  constexpr int WM = NW, WN = 1, TM = MTW * 16, TN = NTW * 16;
  constexpr int BM = WM * TM, BN = WN * TN;
  constexpr int STAGE = BN * 128;             // W bytes per stage (BN rows x 64 k)
  constexpr int GROUPS = BN / 8;              // DMA instructions per stage (8 rows each)
  static_assert(GROUPS % NL == 0, "loaders share the stage evenly");
  constexpr int GPL = GROUPS / NL;            // DMA instructions per loader and stage
  constexpr int AV = MTW * 2;                 // A loads per stage per compute lane
  constexpr int WAIT_W = GPL * (NB - 2);
  constexpr int WAIT_A = AV * (FRA - 1);
  static_assert(WAIT_W < 64 && WAIT_A < 64, "vmcnt range");
  static_assert(NB % FRA == 0, "the unrolled loop cycles both rings");
  static_assert(EPI != EPI_SWIGLU || NTW % 2 == 0, "swiglu pairs");
  __shared__ __attribute__((aligned(1024))) uint8_t Wsm[NB * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int bx, by, z;
  const int l = xcd_tile(bx, by, z);
  const int n0 = bx * BN, m0 = by * BM;
  const int kper = a.K / a.splits, kbeg = z * kper, nk = kper / BK;
  // Workgroups start their K range at different steps and wrap around: weight
  // rows lie a power of two apart, so workgroups that walk K in step keep asking
  // for the same 128 bytes of every row, which sit on few of the memory
  // channels. Up to 64 rows, coarse phases by groups of 8 tiles and finer ones
  // inside (the batch-1 SwiGLU GEMM 45 -> 35 us, 4.5 -> 5.7 TB/s; steps of 16 and
  // 64 rows 825 -> 770 and 925 -> 858 us); above, coarse phases by XCD, finer ones
  // inside it, so that the workgroups of one L2 stay near the same activation
  // columns (256 rows 1211 -> 1175 us, 1024 rows unchanged; the first rule costs
  // those 3%).
  // All row tiles of a column tile start at the same step, whatever their number,
  // by the place and the XCD of the first of them: they read the same weights side
  // by side, and a sequence's logits do not depend on the row tile it falls in.
  // (The XCD of an earlier place by steps back over the XCDs' first places: a
  // division cost every launch of a step 0.2 to 0.4 us. Up to 64 rows there is one
  // row tile.)
  int phase;
  if constexpr (BM <= 64) {
    phase = ((l >> 3) & 7) * 8 + (l & 7);
  } else {
    const int total = gridDim.x * gridDim.y * gridDim.z, q = total >> 3, r = total & 7;
    const int l0 = l - by;
    int xcd = (blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) & 7;
    while (l0 < xcd * q + min(xcd, r)) --xcd;
    phase = xcd * 8 + ((l0 >> 3) & 7);
  }
  const int rot = phase * nk / 64;
  auto kstep = [&](int st) {   // the K step of stage st (past the end: the last one's)
    const int q = min(st, nk - 1) + rot;
    return q >= nk ? q - nk : q;
  };
  if (wave >= NW) {
    // loader l: groups l * GPL .. + GPL of every stage; lane -> row g * 8 +
    // lane / 8, physical chunk lane % 8 <- logical chunk (lane % 8) ^ (row & 7);
    // weight rows past N repeat the last one (their columns are not stored)
    const int l = wave - NW;
    const uint16_t* W = static_cast<const uint16_t*>(a.W);
    const uint16_t* wsrc[GPL];
    int wdst[GPL];
#pragma unroll
    for (int q = 0; q < GPL; ++q) {
      const int g = l * GPL + q;
      const int r = g * 8 + (lane >> 3);
      const int c = (lane & 7) ^ (r & 7);
      const int gn = min(n0 + r, a.N - 1);
      const int wrow = EPI == EPI_SWIGLU ? swiglu_row(gn, a.mlp) : gn;
      wsrc[q] = W + (long)wrow * a.ldw + kbeg + c * 8;
      wdst[q] = g * 1024;
    }
    auto issue_w = [&](int buf, int stage) {   // stages past the end reload the last one
      const int off = kstep(stage) * BK;
      uint8_t* dst = Wsm + buf * STAGE;
#pragma unroll
      for (int q = 0; q < GPL; ++q)
        __builtin_amdgcn_global_load_lds(LDR_GP(wsrc[q] + off), LDR_LP(dst + wdst[q]), 16, 0, 0);
    };
#pragma unroll
    for (int st = 0; st < NB - 1; ++st) issue_w(st, st);
    int buf = NB - 1;
    for (int kt = 0; kt < nk; ++kt) {
      wait_vmcnt<WAIT_W>();
      group_barrier();
      issue_w(buf, kt + NB - 1);
      buf = buf == NB - 1 ? 0 : buf + 1;
    }
    wait_vmcnt<0>();   // no DMA outlives the workgroup
    return;
  }
  const int wm = wave;
  const uint16_t* A = static_cast<const uint16_t*>(a.A);
  // A fragments of m-tile i and k half kk of a step: in the fragment layout
  // one 1 KB block each (row blocks past the padded row count repeat the
  // last one); row-major, lane l reads row l % 16 (rows past M repeat the
  // last one), 8 columns from (l / 16) * 8. Those rows are never stored.
  const uint16_t* asrc[MTW];
  if constexpr (ROWA) {
#pragma unroll
    for (int i = 0; i < MTW; ++i) {
      const int r = min(m0 + wm * TM + i * 16 + (lane & 15), a.M - 1);
      asrc[i] = A + (long)r * a.lda + kbeg + (lane >> 4) * 8;
    }
  } else {
    const int mpad = (a.M + 15) & ~15;
#pragma unroll
    for (int i = 0; i < MTW; ++i) {
      const int rg = min(m0 + wm * TM + i * 16, mpad - 16) >> 4;
      asrc[i] = A + ((long)rg * (a.K >> 5) + (kbeg >> 5)) * 512 + lane * 8;
    }
  }
  constexpr int KKA = ROWA ? 32 : 512;       // elements between the two k halves
  constexpr long STA = ROWA ? BK : 1024;     // elements between steps
  u32x4 aq[FRA][MTW][2];
  auto load_a = [&](u32x4 (&dst)[MTW][2], int stage) {   // past the end: the last stage again
    const long off = (long)kstep(stage) * STA;
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        dst[i][kk] = *reinterpret_cast<const u32x4*>(asrc[i] + off + kk * KKA);
  };
  // W fragment offsets in a stage: row j * 16 + lane % 16, logical chunk
  // kk * 4 + lane / 16
  int woff[NTW][2];
#pragma unroll
  for (int j = 0; j < NTW; ++j)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int r = j * 16 + (lane & 15);
      woff[j][kk] = r * 128 + (((kk * 4 + (lane >> 4)) ^ (r & 7)) * 16);
    }
  f32x4 acc[MTW][NTW];
#pragma unroll
  for (int i = 0; i < MTW; ++i)
#pragma unroll
    for (int j = 0; j < NTW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < FRA; ++st) load_a(aq[st], st);
  // step kt in phase p = kt mod NB: W stage kt in buffer p, A stage kt in
  // register slot p mod FRA, refilled with stage kt + FRA after the MFMAs
  auto step = [&](int kt, auto pc) {
    constexpr int p = decltype(pc)::value;
    sched_fence();
    wait_vm_lgkm0<WAIT_A>();
    __builtin_amdgcn_s_barrier();
    sched_fence();
    const uint8_t* cur = Wsm + p * STAGE;
    bf16x8 bfr[2][NTW];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int j = 0; j < NTW; ++j)
        bfr[kk][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(cur + woff[j][kk]));
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int j = 0; j < NTW; ++j)
          mma_tile<EPI == EPI_SWIGLU>(__builtin_bit_cast(bf16x8, aq[p % FRA][i][kk]), bfr[kk][j],
                                      acc[i][j]);
    load_a(aq[p % FRA], kt + FRA);
    sched_fence();
  };
  const int full = nk / NB * NB;
  int kt = 0;
  for (; kt < full; kt += NB)
    for_phases([&](auto pc) { step(kt + decltype(pc)::value, pc); },
               std::make_integer_sequence<int, NB>{});
  const int rem = nk - full;   // uniform: every wave takes the same steps
  for_phases([&](auto pc) { if (decltype(pc)::value < rem) step(kt + decltype(pc)::value, pc); },
             std::make_integer_sequence<int, NB - 1>{});
  wait_vm_lgkm0<0>();
  store_tile<MTW, NTW, WM, WN, EPI>(a, n0, m0, z, acc);
}

// NW x MTW row tiles of 16, BN = 16 NTW columns.
template <int NW, int MTW, int NTW, int EPI, bool ROWA>
__global__ void __launch_bounds__(64 * (NW + kFragLoaders), 1) gemm_frag_kernel(GemmArgs a) {
  frag_gemm<MTW, NTW, EPI, 2, kFragLoaders, 6, NW, ROWA>(a);
}

// ---------------------------------------------------------------------------
// GEMM on tiled operands (the vocabulary head).
//
// The activation rows arrive tiled in blocks of TR = 256 rows by TK = 32
// columns, block (r / TR, k / TK) at ((r / TR) * (K / TK) + k / TK) * TR * TK,
// its rows contiguous (TK elements each); the weight [N][K] in column blocks:
// element (n, k) at (k / TK) * R * TK + n * TK + k % TK, R = N rounded up to
// 256 (the layout ldr_tile_matrix writes). One K block of any run of weight
// rows, and of one activation row tile, is then consecutive memory that HBM
// streams at full rate; the same rows read in row-major order are 64-byte
// pieces 8 KB apart, which it serves at about half.
//
// A workgroup of 8 waves owns a 256 x HB output tile, HB = 304 = 19 x 16
// columns: the vocabulary of 151936 then makes 500 tiles, under two rounds
// over the 256 CUs (256-column tiles would make 594: a third round of 82
// tiles that runs nearly as long as a full one, at one CU's streaming rate).
// The waves compute 128 x 80 each (8 x 5 MFMA tiles), so the tile computes
// HW = 320 columns; the last 16 belong to the next tile: their weight rows
// are not staged and their columns are dropped.
// Waves 0-3 and 4-7 form two groups that share the four SIMDs pairwise and take
// turns, one barrier apart: while one group issues its 40 MFMAs for the current
// K block, the other reads its fragments of that block from LDS and starts the
// DMA (global_load_lds) of its part of the block D steps ahead: group 0 the
// 256 A rows (16 KB), group 1 the 304 W rows (19 KB). Each SIMD's matrix unit
// is thus fed by one wave or the other most of the time. Stages of 576 rows x
// 64 B live in NB = 4 LDS buffers; the 16-byte chunk c of stage row r sits at
// chunk c ^ ((r >> 2) & 3), so the 16 lanes of a fragment read hit 64 distinct
// banks.
//
// Ordering (t = K block, barriers numbered from the start of the loop):
//  * group 0 reads block t between barriers 2t and 2t + 1, group 1 between
//    2t + 1 and 2t + 2; each waits for its own LDS reads before the barrier that
//    ends its memory phase, so a buffer's last reader is done two barriers
//    before the DMA that refills it (D = NB - 1) is issued;
//  * every wave waits for its own DMA of block t + 1 (vmcnt) before barrier
//    2t + 2, after which block t + 1 is whole in LDS for both groups.
constexpr int TR = 256, TK = 32;
constexpr long TBLK = (long)TR * TK;
constexpr int HB = 304, HW = 320;

__device__ inline int tile_swz(int r) { return (r >> 2) & 3; }
// The 16 rows of wave wq's DMA issue q past the tile's HB columns.
__device__ inline bool lr_overlap(int wq, int q) { return wq * 80 + q * 16 >= HB; }

// Greedy partial of the fused head: the largest logit of a column range and
// its first token.
struct HeadPart { float key; int idx; };

__device__ inline void head_combine(HeadPart& a, const HeadPart& b) {
  if (b.key > a.key || (b.key == a.key && b.idx < a.idx)) a = b;
}

// Epilogues of the vocabulary head: logits only; the greedy partials (logits
// optional); the logits and the chunk log-masses at T > 0 (T = 1 without the
// division).
constexpr int kHeadLogits = 0, kHeadArgmax = 1, kHeadChunks = 2, kHeadChunksUnitT = 3;

template <int HS>
__global__ void __launch_bounds__(512, 1) gemm_tiled_kernel(GemmArgs a, HeadSampleArgs hs) {
  constexpr int NB = 4, D = NB - 1;
  constexpr int STAGE = (TR + HW) * TK * 2;   // bytes: A rows 0..255, W rows 256..575
  constexpr int MT = 8, NT = 5;               // 16 x 16 MFMA tiles per wave: 128 x 80
  constexpr int QA = TR / 64, QW = HW / 64;   // DMA issues per lane: 4 (A), 5 (W)
  __shared__ __attribute__((aligned(1024))) uint8_t S0[STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t S1[STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t S2[STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t S3[STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = wave >> 2, wq = wave & 3;
  const int wm = grp, wn = wq;   // output rows wm * 128 .., columns wn * 80 ..
  const int nkb = a.K / TK;
  int ct, rt, z_;
  xcd_tile(ct, rt, z_);   // column tile, row tile: the row tiles of a column tile share its
                          // weight columns in one L2
  const int n0 = ct * HB;
  // DMA: wave wq of group 0 moves A rows wq * 64 + q * 16 + lane / 4, of group 1
  // W rows wq * 80 + q * 16 + lane / 4 (4 lanes per 64-byte row, lane & 3 = the
  // destination chunk); W rows past the padded matrix read its last row.
  const uint16_t* src[QW];
  int dst[QW];
  long kstride;
  if (grp == 0) {
    const uint16_t* tile = static_cast<const uint16_t*>(a.A) + (long)rt * nkb * TBLK;
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      const int r = wq * 64 + (q < QA ? q : 0) * 16 + (lane >> 2);
      src[q] = tile + r * TK + (((lane & 3) ^ tile_swz(r)) * 8);
      dst[q] = (wq * 64 + (q < QA ? q : 0) * 16) * 64;
    }
    kstride = TBLK;
  } else {
    // The last 16 of the 320 rows belong to the next tile; their output
    // columns are dropped. Their DMA (wave 3, q = 4) re-reads the 16 rows
    // before them, which the same wave has just requested (a cache hit, with
    // the same chunk swizzle), instead of fetching 16 more rows from memory:
    // every wave still issues QW DMAs per block.
    const long R = a.ldw;   // padded weight rows of one column block
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      const int lr = wq * 80 + q * 16 + (lane >> 2) - (lr_overlap(wq, q) ? 16 : 0);
      const long gr = min((long)n0 + lr, R - 1);
      src[q] = static_cast<const uint16_t*>(a.W) + gr * TK +
               (((lane & 3) ^ tile_swz(TR + lr)) * 8);
      dst[q] = (TR + wq * 80 + q * 16) * 64;
    }
    kstride = R * TK;
  }
  // Blocks past the end reload the last one (never read).
  auto issue_a = [&](uint8_t* buf, int t) {
    const long off = (long)min(t, nkb - 1) * kstride;
#pragma unroll
    for (int q = 0; q < QA; ++q)
      __builtin_amdgcn_global_load_lds(LDR_GP(src[q] + off), LDR_LP(buf + dst[q]), 16, 0, 0);
  };
  auto issue_w = [&](uint8_t* buf, int t) {
    const long off = (long)min(t, nkb - 1) * kstride;
#pragma unroll
    for (int q = 0; q < QW; ++q)
      __builtin_amdgcn_global_load_lds(LDR_GP(src[q] + off), LDR_LP(buf + dst[q]), 16, 0, 0);
  };
  int aoff[MT], woff[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int r = wm * 128 + i * 16 + (lane & 15);
    aoff[i] = r * 64 + (((lane >> 4) ^ tile_swz(r)) * 16);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int r = TR + wn * 80 + j * 16 + (lane & 15);
    woff[j] = r * 64 + (((lane >> 4) ^ tile_swz(r)) * 16);
  }
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 af[MT], bfr[NT];

#define LDR_MEM(t, cur, nxt, ISSUE)                                                            \
  {                                                                                            \
    sched_fence();                                                                             \
    _Pragma("unroll") for (int i = 0; i < MT; ++i) af[i] =                                     \
        __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(cur + aoff[i]));            \
    _Pragma("unroll") for (int j = 0; j < NT; ++j) bfr[j] =                                    \
        __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(cur + woff[j]));            \
    ISSUE(nxt, (t) + D);                                                                       \
    sched_fence();                                                                             \
    wait_lgkmcnt0();                                                                           \
  }
#define LDR_MMA()                                                                              \
  {                                                                                            \
    sched_fence();                                                                             \
    __builtin_amdgcn_s_setprio(1);                                                             \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                             \
      _Pragma("unroll") for (int j = 0; j < NT; ++j) acc[i][j] =                               \
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);          \
    __builtin_amdgcn_s_setprio(0);                                                             \
    sched_fence();                                                                             \
  }
#define LDR_G0(t, cur, nxt) { LDR_MEM(t, cur, nxt, issue_a) group_barrier(); LDR_MMA() wait_vmcnt<QA * (D - 1)>(); group_barrier(); }
#define LDR_G1(t, cur, nxt) { LDR_MEM(t, cur, nxt, issue_w) wait_vmcnt<QW * (D - 1)>(); group_barrier(); LDR_MMA() group_barrier(); }
  if (grp == 0) { issue_a(S0, 0); issue_a(S1, 1); issue_a(S2, 2); }
  else { issue_w(S0, 0); issue_w(S1, 1); issue_w(S2, 2); }
  wait_vmcnt<0>();
  group_barrier();
  if (grp == 0) {
    for (int t = 0; t < nkb; t += NB) {
      LDR_G0(t, S0, S3) LDR_G0(t + 1, S1, S0) LDR_G0(t + 2, S2, S1) LDR_G0(t + 3, S3, S2)
    }
    group_barrier();   // pairs with group 1's offset barrier
  } else {
    group_barrier();   // offset: group 1 starts one barrier later
    for (int t = 0; t < nkb; t += NB) {
      LDR_G1(t, S0, S3) LDR_G1(t + 1, S1, S0) LDR_G1(t + 2, S2, S1) LDR_G1(t + 3, S3, S2)
    }
  }
#undef LDR_G1
#undef LDR_G0
#undef LDR_MMA
#undef LDR_MEM
  wait_vmcnt<0>();   // no DMA outlives the workgroup
  // The MFMAs take the weight fragments as their first operand, so each
  // 16 x 16 accumulator tile is (token, row): lane l holds 4 consecutive
  // tokens g * 4 .. + 3 (g = l / 16) of row l % 16, one float4 of logits, and
  // the 4 lanes g = 0 .. 3 of a row hold one 16-token chunk.
  const int g = lane >> 4, rl = lane & 15;
  const int r0 = rt * TR + wm * 128, c0 = n0 + wn * 80;
  const int cend = min(a.N, n0 + HB);   // the tile's own columns
  // Most waves hold no token past the vocabulary and write rows that start
  // on 16 bytes: their epilogues skip the per-token tests (wave-uniform).
  const bool full = c0 + NT * 16 <= a.N && (a.ldo & 3) == 0;
  if (HS != kHeadArgmax || hs.store_logits) {
    float* out = static_cast<float*>(a.out);
    auto store = [&](auto full_t) {
      constexpr bool FULL = decltype(full_t)::value;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int row = r0 + i * 16 + rl;
        if (row >= a.M) continue;
        float* orow = out + (long)row * a.ldo + c0 + g * 4;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int col = c0 + j * 16 + g * 4;
          float* o = orow + j * 16;
          if (FULL) {
            if (c0 + j * 16 < cend) *reinterpret_cast<f32x4*>(o) = acc[i][j];
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (col + v < cend) o[v] = acc[i][j][v];
          }
        }
      }
    };
    if (full) store(std::true_type{});
    else store(std::false_type{});
  }
  // Lane exchanges across the row groups: xor 16 (a swizzle inside each half
  // wave) and xor 32 (a permute).
  auto x16 = [](float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x),
                                                                 0x401F));
  };
  const int perm32 = (lane ^ 32) << 2;
  auto x32 = [perm32](float x) {
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_ds_bpermute(perm32, __builtin_bit_cast(int, x)));
  };
  if constexpr (HS == kHeadChunks || HS == kHeadChunksUnitT) {
    // Chunk log-masses (the first level of the two-level draw of Eq. 8 at
    // T > 0): each lane's max and sum of exp(z/T - max) over its 4 tokens,
    // (t0 + t1) + (t2 + t3), then over the chunk's 4 lanes (xor 16, then
    // xor 32) -- the order and operations of the log-mass pass over stored
    // logits, so L_c has the same bits. Tokens past the vocabulary count as
    // -inf; chunks past the tile's own columns belong to the next tile and
    // are not written. Lane group g keeps chunk g (group 0 also chunk 4).
    const float T = hs.T;
    auto chunks = [&](auto full_t) {
      constexpr bool FULL = decltype(full_t)::value;
      // IP row blocks of NT chunks side by side, one phase at a time, so that
      // each lane exchange waits once for all of them
      constexpr int IP = 2;
#pragma unroll
      for (int i0 = 0; i0 < MT; i0 += IP) {
        float zt[IP][NT][4], m[IP][NT], sum[IP][NT], o16[IP][NT], o32[IP][NT];
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int col = c0 + j * 16 + g * 4;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const float x = acc[i0 + ii][j][v];
              zt[ii][j][v] = FULL || col + v < a.N ? (HS == kHeadChunksUnitT ? x : x / T)
                                                   : -INFINITY;
            }
            m[ii][j] = fmaxf(fmaxf(zt[ii][j][0], zt[ii][j][1]), fmaxf(zt[ii][j][2], zt[ii][j][3]));
          }
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) o16[ii][j] = x16(m[ii][j]);
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) m[ii][j] = fmaxf(m[ii][j], o16[ii][j]);
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) o32[ii][j] = x32(m[ii][j]);
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            m[ii][j] = fmaxf(m[ii][j], o32[ii][j]);
            float e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) e[v] = chunk_term(zt[ii][j][v], m[ii][j]);
            sum[ii][j] = (e[0] + e[1]) + (e[2] + e[3]);
          }
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) o16[ii][j] = x16(sum[ii][j]);
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) sum[ii][j] += o16[ii][j];
#pragma unroll
        for (int ii = 0; ii < IP; ++ii)
#pragma unroll
          for (int j = 0; j < NT; ++j) o32[ii][j] = x32(sum[ii][j]);
#pragma unroll
        for (int ii = 0; ii < IP; ++ii) {
          float keep = 0.f, keep4 = 0.f;
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            sum[ii][j] += o32[ii][j];
            const float L = chunk_log_mass(m[ii][j], sum[ii][j]);
            if (j == 4) keep4 = L;
            else keep = g == j ? L : keep;
          }
          const int row = r0 + (i0 + ii) * 16 + rl;
          if (row < a.M) {
            float* Lr = hs.L + (long)row * hs.ldL + c0 / 16;
            if (c0 + g * 16 < cend) Lr[g] = keep;
            if (NT > 4 && g == 0 && c0 + 64 < cend) Lr[4] = keep4;
          }
        }
      }
    };
    if (full) chunks(std::true_type{});
    else chunks(std::false_type{});
  }
  if constexpr (HS == kHeadArgmax) {
    // Greedy epilogue (Eq. 8 at T = 0: the first argmax of each row). Per row
    // of the tile: each lane's best of its 20 tokens, the 4 lanes of the row
    // (its 80 columns of this wave) by lane exchanges, the 4 waves of the row
    // through LDS, one partial per (row, column tile).
    __shared__ HeadPart tab[TR][4];
    HeadPart* parts = static_cast<HeadPart*>(hs.parts);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      HeadPart p{-INFINITY, 0x7fffffff};
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int col = c0 + j * 16 + g * 4 + v;
          if (col < cend) head_combine(p, HeadPart{acc[i][j][v], col});
        }
      HeadPart o;
      o.key = x16(p.key);
      o.idx = __builtin_amdgcn_ds_swizzle(p.idx, 0x401F);
      head_combine(p, o);
      o.key = x32(p.key);
      o.idx = __builtin_amdgcn_ds_bpermute(perm32, p.idx);
      head_combine(p, o);
      if (g == 0) tab[wm * 128 + i * 16 + rl][wn] = p;
    }
    __syncthreads();
    if (tid < TR) {
      const int row = rt * TR + tid;
      HeadPart p = tab[tid][0];
#pragma unroll
      for (int q = 1; q < 4; ++q) head_combine(p, tab[tid][q]);
      if (row < a.M) parts[(long)row * hs.nparts + ct] = p;
    }
  }
}

// One wave per row: the column tiles' partials, then the first argmax, its
// logit as lse and log q = 0, as the separate sampler reports them at T = 0.
__global__ void __launch_bounds__(64) head_argmax_merge_kernel(const HeadPart* parts, int nparts,
                                                               int32_t* tokens, float* lse,
                                                               float* logq) {
  const int r = blockIdx.x;
  HeadPart p{-INFINITY, 0x7fffffff};
  for (int s = threadIdx.x; s < nparts; s += 64) head_combine(p, parts[(long)r * nparts + s]);
  for (int off = 32; off >= 1; off >>= 1)
    head_combine(p, HeadPart{__shfl_xor(p.key, off), __shfl_xor(p.idx, off)});
  if (threadIdx.x == 0) {
    tokens[r] = p.idx;
    lse[r] = p.key;
    logq[r] = 0.f;
  }
}

// Column-block copy of a row-major [rows][cols] 2-byte matrix (the weight
// layout of the vocabulary head): one thread per 16-byte chunk of the
// destination, whose column block kb holds R = rows rounded up to 256 rows
// of TK elements; padding rows are zero.
__global__ void __launch_bounds__(256) tile_matrix_kernel(const uint16_t* src, long ld, int rows,
                                                          long R, uint16_t* dst, long chunks) {
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < chunks;
       e += (long)gridDim.x * blockDim.x) {
    const long kb = e / (R * (TK / 8));
    const long in = e % (R * (TK / 8));
    const long row = in / (TK / 8);
    const int col = (int)(kb * TK + (in % (TK / 8)) * 8);
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (row < rows) v = *reinterpret_cast<const u32x4*>(src + row * ld + col);
    *reinterpret_cast<u32x4*>(dst + e * 8) = v;
  }
}

// Launches gemm_frag_kernel for the plan's BM x BN tile. EPI_SWIGLU rows are in
// the fragment layout or, for at most 16 rows, row-major.
template <int EPI, bool ROWA, int NW, int MTW>
hipError_t launch_bn(const GemmPlan& p, dim3 grid, const GemmArgs& a, hipStream_t st) {
  const dim3 block(64 * (NW + kFragLoaders));
  if (p.bn == 128)
    hipLaunchKernelGGL((gemm_frag_kernel<NW, MTW, 8, EPI, ROWA>), grid, block, 0, st, a);
  else if (p.bn == 96)
    hipLaunchKernelGGL((gemm_frag_kernel<NW, MTW, 6, EPI, ROWA>), grid, block, 0, st, a);
  else if constexpr (NW * MTW > 4)   // 64 columns: above 64 rows only
    hipLaunchKernelGGL((gemm_frag_kernel<NW, MTW, 4, EPI, ROWA>), grid, block, 0, st, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_frag(const GemmPlan& p, dim3 grid, const GemmArgs& a, hipStream_t st) {
  if (p.bm == 16) return launch_bn<EPI, true, 1, 1>(p, grid, a, st);
  if constexpr (EPI == EPI_STORE) {
    if (!p.frag) {
      switch (p.bm) {
        case 32: return launch_bn<EPI, true, 2, 1>(p, grid, a, st);
        case 64: return launch_bn<EPI, true, 4, 1>(p, grid, a, st);
        case 128: return launch_bn<EPI, true, 8, 1>(p, grid, a, st);
        default: return launch_bn<EPI, true, 8, 2>(p, grid, a, st);
      }
    }
  }
  switch (p.bm) {
    case 32: return launch_bn<EPI, false, 2, 1>(p, grid, a, st);
    case 64: return launch_bn<EPI, false, 4, 1>(p, grid, a, st);
    case 128: return launch_bn<EPI, false, 8, 1>(p, grid, a, st);
    default: return launch_bn<EPI, false, 8, 2>(p, grid, a, st);
  }
}

}  // namespace

// bf16: BM is the smallest of 16, 32, 64, 128 and 256 that covers M (several
// row tiles past 256); BN and the K split (1, 2, 4, 8; only where allowed) are
// chosen among 128, 96 and 64 columns.
GemmPlan plan_gemm(int dtype, int M, int N, int K, bool allow_split, bool swiglu, bool frag,
                   int max_splits) {
  GemmPlan p{};
  constexpr int kCUs = 256;
  p.splits = 1;
  if (!allow_split) max_splits = 1;
  if (dtype == LDR_F32) {
    // 16 or 32 rows; 16 columns, or 32 for SwiGLU pairs and where 16-column tiles
    // would put more than four workgroups on a CU; K is split only while the
    // tiles leave half of the CUs idle and a split keeps 512 (4 chunks a wave)
    p.bm = M <= 16 ? 16 : 32;
    p.grid_y = (M + p.bm - 1) / p.bm;
    p.bn = swiglu || (long)((N + 15) / 16) * p.grid_y > 4 * kCUs ? 32 : 16;
    p.grid_x = (N + p.bn - 1) / p.bn;
    const long tiles = (long)p.grid_x * p.grid_y;
    while (p.splits < max_splits && tiles * p.splits * 2 <= kCUs && K % (2 * p.splits * 16) == 0 &&
           K / (2 * p.splits) >= 512)
      p.splits *= 2;
    return p;
  }
  p.bm = M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : M <= 128 ? 128 : 256;
  p.frag = p.bm > 16 && (swiglu || frag);
  p.grid_y = (M + p.bm - 1) / p.bm;
  const int widths[3] = {128, 96, 64};
  if (p.bm <= 64) {
    // Few rows: the weight stream. 128 columns, or 96 where they fill more of
    // the workgroups' last round over the CUs (the batch-1 QKV projection 48 x 4
    // workgroups against 64 x 4: 14.6 -> 13.2 us; the SwiGLU GEMM 47.6 and 47.7
    // us either way), and the K split that brings them to about one per CU, an
    // even number of at least 4 K steps each.
    double best = -1.0;
    for (int w = 0; w < 2; ++w) {
      const long tiles = (long)((N + widths[w] - 1) / widths[w]) * p.grid_y;
      int sp = 1;
      while (sp < max_splits && tiles * sp * 2 <= kCUs && K % (2 * sp * 2 * BK) == 0 &&
             K / (2 * sp) >= 4 * BK)
        sp *= 2;
      const long wg = tiles * sp;
      const double fill = (double)wg / (double)(((wg + kCUs - 1) / kCUs) * kCUs);
      if (fill > best + 1e-9) { best = fill; p.bn = widths[w]; p.splits = sp; }
    }
  } else if (swiglu) {
    // no split-K: the column width whose rounds over the CUs times the bytes a
    // tile streams (all its activation rows plus its weight columns) is least
    double best = 0.0;
    const int order[3] = {96, 128, 64};
    for (const int w : order) {
      const long tiles = (long)p.grid_y * ((N + w - 1) / w);
      const double cost = (double)((tiles + kCUs - 1) / kCUs) * (p.bm + w) * K;
      if (best == 0.0 || cost < best) { best = cost; p.bn = w; }
    }
  } else {
    // 128, 96 or 64 columns and a K split that keeps the workgroups within one
    // round over the CUs (no split where the tiles alone take more): the least
    // rounds over the CUs times the bytes a workgroup moves, its activation rows
    // and weight columns over its K range, and four times its output tile (fp32
    // partials are written in a burst at the end and read back by the next
    // kernel; the four is a fit to the plans measured best at 256 and 1024 rows of
    // the Qwen3-8B shape). At 1024 rows the down projection then runs on 128 columns split
    // in two instead of 64 unsplit, with as many workgroups (120 -> 84 us); at 256
    // rows QKV, O and down keep 96 x 4, 64 x 4 and 128 x 8 (O at 128 x 8, the next
    // by this cost, makes its own time up in the norm that reads the partials).
    double best = 0.0;
    for (const int w : widths) {
      const long tiles = (long)((N + w - 1) / w) * p.grid_y;
      for (int sp = 1; sp <= max_splits; sp *= 2) {
        if (K % (sp * BK) != 0 || K / sp < 2 * BK) break;
        const long wg = tiles * sp;
        if (sp > 1 && wg > kCUs) break;
        const double rounds = (double)((wg + kCUs - 1) / kCUs);
        const double cost =
            rounds * (((double)p.bm + w) * (K / sp) * 2.0 + 4.0 * p.bm * w * 4.0 * (sp > 1 ? 2 : 1));
        if (best == 0.0 || cost < best) { best = cost; p.bn = w; p.splits = sp; }
      }
    }
  }
  p.grid_x = (N + p.bn - 1) / p.bn;
  return p;
}

hipError_t launch_gemm(int dtype, int epi, const GemmPlan& p, const GemmArgs& a,
                       hipStream_t st) {
  if (dtype == LDR_F32) {
    const dim3 grid(p.grid_x, p.grid_y, p.splits), block(kF32Waves * 64);
#define LDR_F32K(MT, NT, EPI) \
  hipLaunchKernelGGL((gemm_f32_kernel<MT, NT, EPI>), grid, block, 0, st, a)
    if (epi == EPI_SWIGLU) {
      if (p.bm == 16) LDR_F32K(1, 2, EPI_SWIGLU); else LDR_F32K(2, 2, EPI_SWIGLU);
    } else if (p.bn == 16) {   // EPI_STORE and EPI_LOGITS share the fp32 store
      if (p.bm == 16) LDR_F32K(1, 1, EPI_STORE); else LDR_F32K(2, 1, EPI_STORE);
    } else {
      if (p.bm == 16) LDR_F32K(1, 2, EPI_STORE); else LDR_F32K(2, 2, EPI_STORE);
    }
#undef LDR_F32K
    return hipGetLastError();
  }
  const dim3 grid(p.grid_x, p.grid_y, p.splits);
  if (epi == EPI_SWIGLU) return launch_frag<EPI_SWIGLU>(p, grid, a, st);
  return launch_frag<EPI_STORE>(p, grid, a, st);   // EPI_LOGITS: the same store, never split
}

bool gemm_tiled_supported(int M, int N, int K) {
  return M > 0 && N > 0 && K % (TK * 4) == 0;
}

hipError_t launch_gemm_tiled(const GemmArgs& a0, hipStream_t st) {
  if (!gemm_tiled_supported(a0.M, a0.N, a0.K) || a0.splits != 1) return hipErrorInvalidValue;
  GemmArgs a = a0;
  a.ldw = (a.N + TR - 1) / TR * TR;   // padded rows of a weight column block
  const dim3 grid((a.N + HB - 1) / HB, (a.M + TR - 1) / TR, 1);
  hipLaunchKernelGGL((gemm_tiled_kernel<kHeadLogits>), grid, dim3(512), 0, st, a,
                     HeadSampleArgs{});
  return hipGetLastError();
}

size_t head_sample_part_bytes(int rows, int vocab) {
  return (size_t)rows * ((vocab + HB - 1) / HB) * sizeof(HeadPart);
}

hipError_t launch_gemm_tiled_argmax(const GemmArgs& a0, const HeadSampleArgs& hs0, int32_t* tokens,
                                    float* lse, float* logq, hipStream_t st) {
  if (!gemm_tiled_supported(a0.M, a0.N, a0.K) || a0.splits != 1) return hipErrorInvalidValue;
  GemmArgs a = a0;
  a.ldw = (a.N + TR - 1) / TR * TR;
  HeadSampleArgs hs = hs0;
  hs.nparts = (a.N + HB - 1) / HB;
  const dim3 grid(hs.nparts, (a.M + TR - 1) / TR, 1);
  hipLaunchKernelGGL((gemm_tiled_kernel<kHeadArgmax>), grid, dim3(512), 0, st, a, hs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_argmax_merge_kernel, dim3(a.M), dim3(64), 0, st,
                     static_cast<const HeadPart*>(hs.parts), hs.nparts, tokens, lse, logq);
  return hipGetLastError();
}

hipError_t launch_gemm_tiled_chunks(const GemmArgs& a0, const HeadSampleArgs& hs0,
                                    hipStream_t st) {
  if (!gemm_tiled_supported(a0.M, a0.N, a0.K) || a0.splits != 1 || !a0.out || !hs0.L ||
      !(hs0.T > 0.f) || hs0.ldL < (a0.N + 15) / 16)
    return hipErrorInvalidValue;
  GemmArgs a = a0;
  a.ldw = (a.N + TR - 1) / TR * TR;
  HeadSampleArgs hs = hs0;
  hs.store_logits = 1;
  const dim3 grid((a.N + HB - 1) / HB, (a.M + TR - 1) / TR, 1);
  if (hs.T == 1.f)
    hipLaunchKernelGGL((gemm_tiled_kernel<kHeadChunksUnitT>), grid, dim3(512), 0, st, a, hs);
  else
    hipLaunchKernelGGL((gemm_tiled_kernel<kHeadChunks>), grid, dim3(512), 0, st, a, hs);
  return hipGetLastError();
}

size_t tiled_elems(long rows, long cols) { return (size_t)((rows + TR - 1) / TR) * TR * cols; }

hipError_t launch_tile_matrix(const void* src, long ld, int rows, int cols, void* dst,
                              hipStream_t st) {
  const long chunks = (long)tiled_elems(rows, cols) / 8;
  const long want = (chunks + 255) / 256, blocks = want < 8192 ? want : 8192;
  const long R = (rows + TR - 1) / TR * TR;
  hipLaunchKernelGGL(tile_matrix_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                     static_cast<const uint16_t*>(src), ld, rows, R,
                     static_cast<uint16_t*>(dst), chunks);
  return hipGetLastError();
}

}  // namespace ldr
