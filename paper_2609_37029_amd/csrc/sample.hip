// Per-position sampling of the factorised proposal (Eq. 8).
//
// T > 0: a two-level Gumbel-max, an exact draw from q = softmax(z/T) over the
// support. The vocabulary is cut into chunks of 16 consecutive tokens; chunk c
// has log-mass L_c = log sum_{v in c} exp(z_v/T). The chunk is the first
// argmax of L_c + h_c (h_c Gumbel noise of stream 3), the token the first
// argmax of z_v/T + g_v over that chunk (g_v Gumbel noise of stream 0):
//  * chunk_lse_kernel streams the logits once (16-byte loads, four sweeps in
//    flight per lane) and writes L_c: a lane holds 4 tokens of a chunk, the
//    chunk's max and sum of exp(z/T - max) are reduced over its 4 lanes with
//    DPP, in the balanced pairwise order (t0 + t1) + (t2 + t3), ... over the
//    chunk's tokens;
//  * chunk_draw_kernel, one workgroup per row, runs the Gumbel-max over the
//    row's L_c like a one-level sampler over V/16 entries: per lane the
//    running max / sum of exp(L_c) for the log-normaliser and the best key,
//    exact keys computed only for entries that a cheap upper bound of the
//    noise cannot rule out; it combines the lanes' results (lower index wins
//    ties), then draws the token inside the winning chunk, one lane per
//    token, and writes the token, lse and log q(y).
// T = 0 is the first argmax of the logits (sample_partial_kernel + merge).
//
// The noise is a pure function of (seed, step, stream, row, entry):
// Philox4x32-10 (Salmon et al., SC 2011; key = the seed, counter (entry / 4,
// row, step, stream)); one Philox block serves 4 consecutive entries, 32 bits
// each. The uniform u = (2 (bits >> 9) + 1) 2^-24 is exact, and
// g = -log(-log u) uses a log made of IEEE fp32 operations only (no
// contraction, correctly rounded division), so every key fl(x + g) is
// reproducible bit for bit.
#include <mutex>
#include <type_traits>

#include "ldr_internal.h"
#include "noise.h"

namespace ldr {
namespace {

constexpr int kThreads = 256;

struct Partial { float m, s, key; int idx; };  // max z/T, sum exp(z/T - m), best key, token

__device__ inline bool better(float k1, int i1, float k2, int i2) {
  return k1 > k2 || (k1 == k2 && i1 < i2);
}

__device__ inline void combine(Partial& a, const Partial& b) {
  if (better(b.key, b.idx, a.key, a.idx)) { a.key = b.key; a.idx = b.idx; }
  const float m = fmaxf(a.m, b.m);
  if (m == -INFINITY) return;
  a.s = a.s * __expf(a.m - m) + b.s * __expf(b.m - m);
  a.m = m;
}

// Reductions over the 64 lanes of a wave: DPP inside each row of 16, then two
// lane exchanges. Every lane ends with the same value.
__device__ inline float wave_max64(float v) {
  v = max16(v);
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}
__device__ inline float wave_sum64(float v) {
  v = sum16(v);
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}
__device__ inline int min16(int v) {
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false));
  return min(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false));
}

// The lanes' partials combined over rows of 16 lanes (W = 16) or the whole wave
// (W = 64), every lane with the result: the max first, then each sum rescaled
// once, the best key and the lowest index among its equals.
template <int W> __device__ inline Partial lanes_combine(const Partial& p) {
  Partial o;
  o.m = W == 64 ? wave_max64(p.m) : max16(p.m);
  const float s = o.m == -INFINITY ? 0.f : p.s * __expf(p.m - o.m);
  o.s = W == 64 ? wave_sum64(s) : sum16(s);
  o.key = W == 64 ? wave_max64(p.key) : max16(p.key);
  o.idx = min16(p.key == o.key ? p.idx : 0x7fffffff);
  if (W == 64) {
    o.idx = min(o.idx, __shfl_xor(o.idx, 16));
    o.idx = min(o.idx, __shfl_xor(o.idx, 32));
  }
  return o;
}

struct SampleArgs {
  const float* logits; int rows, vocab, chunk, splits;
  float T; uint64_t seed, step;
  Partial* part;
  const TopK* sel;  // top-k support per row, or null for the full vocabulary
  int row_mul, row_add;  // row r of the launch is logits row (and noise row) r * mul + add
  int vec;               // rows start on 16 bytes (V % 4 == 0, aligned logits): 16-byte loads
  float* L;              // chunk log-masses [rows][ldL] (T > 0)
  int ldL, nch;          // row stride of L (a multiple of 4) and chunks per row
};

constexpr int kChunk = 16;        // tokens per vocabulary chunk of the two-level draw
constexpr uint32_t kChunkStream = 3;

// Exact k-th largest logit of a row by radix selection on order_key (four
// 8-bit digits, most significant first, LDS histograms), then the index cut
// among the tokens equal to it. One workgroup per row.
constexpr int kSelThreads = 1024;
__device__ TopK radix_select(const float* z, int vocab, int k) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t s_digit, s_above;
  __shared__ int wcount[kSelThreads / 64];
  __shared__ int s_base, s_cut;
  uint32_t prefix = 0u, mask = 0u, count_eq = 0u;
  int remaining = k;  // rank of the wanted value among the keys matching prefix
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    for (int i = threadIdx.x; i < 256; i += kSelThreads) hist[i] = 0u;
    __syncthreads();
    for (int v = threadIdx.x; v < vocab; v += kSelThreads) {
      const uint32_t u = order_key(z[v]);
      if ((u & mask) == prefix) atomicAdd(&hist[(u >> shift) & 0xFFu], 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {  // the digit where the count from the top reaches `remaining`
      uint32_t cum = 0u;
      int d = 255;
      for (; d > 0; --d) {
        if (cum + hist[d] >= (uint32_t)remaining) break;
        cum += hist[d];
      }
      s_digit = (uint32_t)d;
      s_above = cum;
    }
    __syncthreads();
    const uint32_t d = s_digit;
    remaining -= (int)s_above;
    prefix |= d << shift;
    mask |= 0xFFu << shift;
    count_eq = hist[d];
    __syncthreads();
  }
  // `remaining` of the count_eq tokens equal to the k-th value are inside:
  // the lowest indices first
  int v_cut = vocab;
  if (remaining < (int)count_eq) {
    if (threadIdx.x == 0) { s_base = 0; s_cut = -1; }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int v0 = 0; v0 < vocab; v0 += kSelThreads) {
      const int v = v0 + (int)threadIdx.x;
      const bool eq = v < vocab && order_key(z[v]) == prefix;
      const uint64_t ball = __ballot(eq);
      if (lane == 0) wcount[w] = __popcll(ball);
      __syncthreads();
      int rank = s_base + __popcll(ball & ((1ull << lane) - 1ull)) + 1;
      for (int i = 0; i < w; ++i) rank += wcount[i];
      if (eq && rank == remaining) s_cut = v;
      __syncthreads();
      if (threadIdx.x == 0)
        for (int i = 0; i < kSelThreads / 64; ++i) s_base += wcount[i];
      __syncthreads();
      if (s_cut >= 0) break;  // uniform: read after the barrier
    }
    v_cut = s_cut;
  }
  return TopK{prefix, v_cut};
}

__global__ void __launch_bounds__(kSelThreads) topk_select_kernel(const float* logits, int vocab,
                                                                  int k, TopK* sel, int row_mul,
                                                                  int row_add) {
  const TopK t =
      radix_select(logits + ((long)blockIdx.x * row_mul + row_add) * vocab, vocab, k);
  if (threadIdx.x == 0) sel[blockIdx.x] = t;
}

// Log-mass of the support tokens of a chunk, whose 16 tokens sit 4 each on 4
// consecutive lanes (x: the lane's, at v; tokens at or past v1 are outside), in
// the balanced pairwise order; every lane returns it.
template <bool UNIT_T, bool TOPK>
__device__ inline float chunk_mass(const TopK& sel, const float (&x)[4], int v, int v1, float T) {
  float zt[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bool in = v + i < v1;
    if constexpr (TOPK) in = in && in_support(sel, x[i], v + i);
    zt[i] = in ? (UNIT_T ? x[i] : x[i] / T) : -INFINITY;  // IEEE division
  }
  float m = fmaxf(fmaxf(zt[0], zt[1]), fmaxf(zt[2], zt[3]));
  m = fmaxf(m, dpp<0xB1>(m));   // the chunk's 4 lanes
  m = fmaxf(m, dpp<0x4E>(m));
  float e[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) e[i] = chunk_term(zt[i], m);
  float sum = (e[0] + e[1]) + (e[2] + e[3]);
  sum += dpp<0xB1>(sum);
  sum += dpp<0x4E>(sum);
  return chunk_log_mass(m, sum);
}
__device__ inline float support_chunk_mass(const TopK& sel, const float (&x)[4], int v, int v1,
                                           float T) {
  return T == 1.f ? chunk_mass<true, true>(sel, x, v, v1, T)
                  : chunk_mass<false, true>(sel, x, v, v1, T);
}

// The top-k support of a row and its chunk log-masses in one launch, one
// workgroup per row, for k <= kSelMaxK and at most kSelMaxChunks chunks:
//  1. one pass over the row keeps every 16-token chunk's largest order_key in
//     LDS (16-byte loads, four sweeps in flight per lane);
//  2. a value t0 such that at least k chunks reach it, by bitwise search over
//     those maxima: at least k tokens reach t0, so the support lies in the
//     chunks that do, and the search stops once they are few;
//  3. the exact k-th largest key among those chunks' tokens, held in registers,
//     and the index cut among its equals, by the same bitwise search;
//  4. the log-masses of those chunks (the operations of chunk_lse_kernel, so the
//     same bits); every other chunk has no support token and takes -inf, so the
//     log-mass pass over the logits is not needed.
// Where ties put more than kSelCap chunks at t0, the row falls back to the radix
// selection and a pass for the log-masses. The radix kernel reads the row five
// times with 4-byte loads and one LDS atomic per token, most of them on a few
// bins. 256 rows of 151936, k = 50: 244 us and 29 us for the log-mass pass then,
// 49 us for this launch (3.2 TB/s; half of it the pass over the row).
// Beyond k = 256 the candidate chunks outgrow the registers; the radix kernel
// stays for those.
// More rows than CUs, each of at most kSelCap chunks (8192 tokens), go to
// workgroups of 256 threads that take every chunk as a candidate: 3. and 4. alone.
// Of 1024 threads, whose registers and counts are sized for long rows, two rows
// fit a CU at a time and a step of the search is mostly its barrier (2048 rows of
// 5003 tokens, k = 20: the call 216 us with 1024 threads, 201 with the radix
// kernel, 110 with 256). Up to 256 rows the two differ by less than 2 us.
constexpr int kSelMaxK = 256, kSelMaxChunks = 14336, kSelCap = 512;

template <bool VEC, int NT>   // NT: kSelThreads, or 256 for at most kSelCap chunks
__global__ void __launch_bounds__(NT) topk_chunks_kernel(SampleArgs a, int k, TopK* sel) {
  constexpr bool ALL = NT < kSelThreads;   // every chunk is a candidate
  constexpr int KPT = kSelMaxChunks / kSelThreads, EPT = kSelCap * kChunk / NT;
  extern __shared__ uint32_t mx[];   // [nch] chunk maxima, then the candidate chunks
  __shared__ int cnt[3], s_nc;
  const int tid = threadIdx.x, lane = tid & 63;
  const int r = blockIdx.x, V = a.vocab, nch = a.nch;
  const float* z = a.logits + ((long)r * a.row_mul + a.row_add) * V;
  float* L = a.L ? a.L + (long)r * a.ldL : nullptr;
  int* cand = reinterpret_cast<int*>(mx + nch);
  if (tid < 3) cnt[tid] = 0;
  if (tid == 3) s_nc = 0;

  if constexpr (!ALL) {  // 1. chunk maxima: 4 lanes hold a chunk, 4 tokens each
    constexpr int U = 4, kSweep = kSelThreads * 4;
    auto load = [&](int v, float (&x)[4]) {
      if constexpr (VEC) {   // V % 4 == 0, v at most V - 4
        const float4 t = *reinterpret_cast<const float4*>(z + v);
        x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = z[min(v + i, V - 1)];   // repeats: the same maximum
      }
    };
    for (int vb = 4 * tid; vb < (V + 15) / 16 * 16; vb += U * kSweep) {
      float x[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) load(min(vb + u * kSweep, (V - 1) / 4 * 4), x[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int v = vb + u * kSweep;
        uint32_t m = max(max(order_key(x[u][0]), order_key(x[u][1])),
                         max(order_key(x[u][2]), order_key(x[u][3])));
        if (v >= V) m = 0u;   // lanes of the last chunk past the row
        m = max(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0xB1, 0xF, 0xF, false));
        m = max(m, (uint32_t)__builtin_amdgcn_mov_dpp((int)m, 0x4E, 0xF, 0xF, false));
        if ((tid & 3) == 0 && v < V) mx[v / kChunk] = m;
      }
    }
  }
  __syncthreads();
  // workgroup-wide count of pred over N values a thread; uniform, one barrier
  int turn = 0;
  auto count = [&](auto n_tag, auto&& pred) -> int {
    int c = 0;
#pragma unroll
    for (int i = 0; i < decltype(n_tag)::value; ++i) c += __popcll(__ballot(pred(i)));
    if (tid == 0) cnt[turn == 2 ? 0 : turn + 1] = 0;
    if (lane == 0 && c) atomicAdd(&cnt[turn], c);
    __syncthreads();
    c = cnt[turn];
    turn = turn == 2 ? 0 : turn + 1;
    return c;
  };
  using NK = std::integral_constant<int, KPT>;
  using NE = std::integral_constant<int, EPT>;

  int nc = nch;
  if constexpr (!ALL) {
    uint32_t key[KPT];
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int c = tid + i * kSelThreads;
      key[i] = c < nch ? mx[c] : 0u;
    }
    // 2. t0: chunks with a maximum >= t0 hold the support
    uint32_t t0 = 0u;
    const int enough = 64 + 2 * k < kSelCap ? 64 + 2 * k : kSelCap;
    for (int bit = 31; bit >= 0 && nc > enough; --bit) {
      const uint32_t t = t0 | (1u << bit);
      const int c = count(NK{}, [&](int i) { return key[i] >= t; });
      if (c >= k) { t0 = t; nc = c; }
    }

    if (nc > kSelCap) {   // ties: the general selection, then every chunk's log-mass
      const TopK t = radix_select(z, V, k);
      if (tid == 0) sel[r] = t;
      if (L)
        for (int vb = 4 * tid; vb < (V + 15) / 16 * 16; vb += 4 * kSelThreads) {
          float x[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = vb + i < V ? z[vb + i] : -INFINITY;
          const float l = support_chunk_mass(t, x, vb, V, a.T);
          if ((tid & 3) == 0) L[vb / kChunk] = l;
        }
      return;
    }

    // the candidate chunks, in any order; the others have no support token
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      const int c = tid + i * kSelThreads;
      const bool in = c < nch && key[i] >= t0;
      const uint64_t m = __ballot(in);
      int at = 0;
      if (lane == 0 && m) at = atomicAdd(&s_nc, __popcll(m));
      at = __shfl(at, 0);
      if (in) cand[at + __popcll(m & ((1ull << lane) - 1ull))] = c;
      else if (L && c < nch) L[c] = -INFINITY;
    }
    __syncthreads();
  }
  auto chunk_of = [&](int ci) { return ALL ? ci : cand[ci]; };

  // 3. the k-th largest key of their tokens
  uint32_t ek[EPT];
  int ev[EPT];   // token, -1: none
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = tid + i * NT, ci = e / kChunk;
    int v = -1;
    if (ci < nc) v = chunk_of(ci) * kChunk + (e & (kChunk - 1));
    if (v >= V) v = -1;
    ev[i] = v;
    ek[i] = v >= 0 ? order_key(z[v]) : 0u;
  }
  uint32_t tau = 0u;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t t = tau | (1u << bit);
    if (count(NE{}, [&](int i) { return ek[i] >= t; }) >= k) tau = t;
  }
  const int above = count(NE{}, [&](int i) { return ev[i] >= 0 && ek[i] > tau; });
  const int equal = count(NE{}, [&](int i) { return ev[i] >= 0 && ek[i] == tau; });
  // the lowest k - above of the equal tokens are inside
  int v_cut = V;
  if (k - above < equal) {
    v_cut = 0;   // the largest index with fewer than k - above equal tokens before it
    for (int bit = 30; bit >= 0; --bit) {
      const int t = v_cut | (1 << bit);
      if (t >= V) continue;
      if (count(NE{}, [&](int i) { return ev[i] >= 0 && ek[i] == tau && ev[i] < t; }) < k - above)
        v_cut = t;
    }
  }
  const TopK t{tau, v_cut};
  if (tid == 0) sel[r] = t;
  // 4. log-masses of the candidate chunks
  if (L)
    for (int i = tid; i < nc * 4; i += NT) {
      const int c = chunk_of(i >> 2), v = c * kChunk + (i & 3) * 4;
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = v + q < V ? z[v + q] : -INFINITY;
      const float l = support_chunk_mass(t, x, v, V, a.T);
      if ((i & 3) == 0) L[c] = l;
    }
}

// The lane's G values of a sweep at v (G a multiple of 4): 16-byte loads
// inside the range [.., v1) when vec, else one load per entry (-inf past v1).
template <int G>
__device__ inline void load_group(const float* z, int v, int v1, bool vec, float (&zz)[G]) {
  if (vec && v + G <= v1) {
#pragma unroll
    for (int b = 0; b < G / 4; ++b) {
      const float4 x = *reinterpret_cast<const float4*>(z + v + 4 * b);
      zz[4 * b] = x.x; zz[4 * b + 1] = x.y; zz[4 * b + 2] = x.z; zz[4 * b + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < G; ++i) zz[i] = v + i < v1 ? z[v + i] : -INFINITY;
  }
}

// Greedy steps (T = 0): the first argmax of the chunk, its logits streamed in
// the sampling sweeps' pattern (the next sweep's loads in flight).
__device__ void argmax_tokens(const SampleArgs& a, const float* z, int v0, int v1, Partial& p) {
  constexpr int kSweep = kThreads * kGroup;
  const int lane_off = (int)threadIdx.x * kGroup;
  float znext[kGroup];
  load_group(z, v0 + lane_off, v1, a.vec, znext);
  for (int vb = v0; vb < v1; vb += kSweep) {
    const int v = vb + lane_off;
    float zcur[kGroup];
#pragma unroll
    for (int i = 0; i < kGroup; ++i) zcur[i] = znext[i];
    if (vb + kSweep < v1) load_group(z, v + kSweep, v1, a.vec, znext);
#pragma unroll
    for (int i = 0; i < kGroup; ++i)
      if (v + i < v1 && better(zcur[i], v + i, p.key, p.idx)) { p.key = zcur[i]; p.idx = v + i; }
  }
}

// Gumbel-max over the chunk log-masses L_c of row r, entries [c0, c1). Every
// lane keeps the max / sum of exp(L_c) of its entries (so the row's lse is
// log sum_c exp(L_c)) and the best (key, chunk) of the entries it evaluated
// exactly. Per sweep of G entries a lane evaluates first the exact key of
// its entry with the largest upper bound L_c + bound(h_c); the largest key of
// the wave so far is then a lower bound of the row's best, and any other
// entry is a candidate only unless L_c + bound(h_c) + margin < that bound,
// which proves that its exact key loses (the margin, 1e-3 plus 1e-6
// relative, covers the rounding of the test and of the fixed-sequence log,
// whose error is below 1e-5 here). Chunks without support tokens
// (L_c = -inf) take no part. The bound is within 0.06 of the exact key and the
// lanes' best entries are settled by then, so few waves meet a candidate: its
// key is computed on the spot (collecting candidates in an LDS queue for full
// waves cost twelve ballots and their branches a sweep, more than it saved).
// G entries per lane and sweep (a multiple of 4, the noise words of G / 4 Philox
// blocks): with 12, one sweep of 1024 lanes covers 12288 chunks, a 196K-token
// vocabulary.
template <int NT, int G = kGroup>
__device__ void chunk_keys(const SampleArgs& a, const float* Lr, int r, int c0, int c1,
                           Partial& p) {
  constexpr int kSweep = NT * G;
  const int lane_off = (int)threadIdx.x * G;
  const uint64_t nrow = (uint64_t)r * a.row_mul + a.row_add;
  float znext[G];
  load_group(Lr, c0 + lane_off, c1, true, znext);
  for (int vb = c0; vb < c1; vb += kSweep) {
    const int v = vb + lane_off;
    float zt[G];
#pragma unroll
    for (int i = 0; i < G; ++i) zt[i] = znext[i];
    if (vb + kSweep < c1) load_group(Lr, v + kSweep, c1, true, znext);
    uint32_t bits[G];
    noise_group(a.seed, a.step, nrow, kChunkStream, (uint64_t)(v / G), bits);
    float gm = -INFINITY, ub[G];
    bool in[G];
    int top = -1;
    float top_ub = -INFINITY, zsel = 0.f;
    uint32_t bsel = 0u;
#pragma unroll
    for (int i = 0; i < G; ++i) {
      in[i] = v + i < c1 && zt[i] > -INFINITY;
      gm = fmaxf(gm, in[i] ? zt[i] : -INFINITY);
      ub[i] = zt[i] + gumbel_upper(bits[i]);
      if (in[i] && (top < 0 || ub[i] > top_ub)) {
        top = i; top_ub = ub[i]; zsel = zt[i]; bsel = bits[i];
      }
    }
    if (gm > p.m) { p.s *= __expf(p.m - gm); p.m = gm; }
    // the lane's most promising entry, exactly; then the wave's best key
    if (top >= 0) {
      const float key = __fadd_rn(zsel, gumbel_from_bits(bsel));
      if (better(key, v + top, p.key, p.idx)) { p.key = key; p.idx = v + top; }
    }
    const float bound = wave_max64(p.key);
#pragma unroll
    for (int i = 0; i < G; ++i) {
      if (in[i]) p.s += __expf(zt[i] - p.m);
      const float margin = 1e-3f + 1e-6f * (fabsf(zt[i]) + fabsf(bound));
      if (in[i] && i != top && !(ub[i] + margin < bound)) {
        const float key = __fadd_rn(zt[i], gumbel_from_bits(bits[i]));
        if (better(key, v + i, p.key, p.idx)) { p.key = key; p.idx = v + i; }
      }
    }
  }
}

// Chunk log-masses of one row, `slice` tokens (a multiple of 16) a workgroup: each
// lane takes 4 consecutive tokens, so 4 lanes hold a chunk. Whole groups of U
// sweeps of kThreads * 4 tokens load without bounds checks (U loads in flight
// per lane), the rest one guarded sweep at a time. Writes L_c for the chunks
// it covers.
template <bool UNIT_T, bool TOPK, bool VEC>
__global__ void __launch_bounds__(kThreads) chunk_lse_kernel(SampleArgs a, int slice) {
  constexpr int U = 4, kSweep = kThreads * 4;
  const int r = blockIdx.y;
  const int v0 = blockIdx.x * slice, v1 = min(a.vocab, v0 + slice);
  const float* z = a.logits + ((long)r * a.row_mul + a.row_add) * a.vocab;
  float* L = a.L + (long)r * a.ldL;
  const TopK sel = TOPK ? a.sel[r] : TopK{0u, 0};
  const float T = a.T;
  const int t4 = 4 * (int)threadIdx.x;
  auto chunk = [&](int v, const float (&x)[4]) {
    const float l = chunk_mass<UNIT_T, TOPK>(sel, x, v, v1, T);
    if ((threadIdx.x & 3) == 0 && v < v1) L[v / kChunk] = l;
  };
  int vb = v0;
  for (; vb + U * kSweep <= v1; vb += U * kSweep) {
    float x[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* zp = z + vb + u * kSweep + t4;
      if constexpr (VEC) {
        const float4 t = *reinterpret_cast<const float4*>(zp);
        x[u][0] = t.x; x[u][1] = t.y; x[u][2] = t.z; x[u][3] = t.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[u][i] = zp[i];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) chunk(vb + u * kSweep + t4, x[u]);
  }
  for (; vb < v1; vb += kSweep) {
    const int v = vb + t4;
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = v + i < v1 ? z[v + i] : -INFINITY;
    chunk(v, x);
  }
}

// The chunk keys and the in-chunk draw of one row (T > 0), one workgroup of
// kDrawThreads threads per row: the Gumbel-max over all its chunk log-masses
// (12 entries a lane and sweep), the lanes' partials combined (max / sum of exp(L)
// for lse, best key and chunk), then lanes 0 .. 15 of the first wave take the 16
// tokens of the winning chunk c (support members only), their exact keys
// fl(fl(z_v/T) + g_v), and the first maximum is the token.
constexpr int kDrawThreads = 1024;
__global__ void __launch_bounds__(kDrawThreads) chunk_draw_kernel(SampleArgs a, int32_t* tokens,
                                                                  float* lse, float* logq) {
  const int r = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Partial p{-INFINITY, 0.f, -INFINITY, 0x7fffffff};
  chunk_keys<kDrawThreads, 12>(a, a.L + (long)r * a.ldL, r, 0, a.nch, p);
  p = lanes_combine<64>(p);
  __shared__ Partial red[kDrawThreads / 64];
  static_assert(kDrawThreads / 64 == 16, "one row of lanes holds the waves' partials");
  if (lane == 0) red[wave] = p;
  __syncthreads();
  if (wave != 0) return;
  p = lanes_combine<16>(red[lane & 15]);
  const long g = (long)r * a.row_mul + a.row_add;
  const float* z = a.logits + g * a.vocab;
  // the chunk's tokens: lane i < 16 takes token 16 c + i (no chunk: none)
  const int v = p.idx < a.nch ? p.idx * kChunk + lane : a.vocab;
  float key = -INFINITY, zt = -INFINITY;
  if (lane < kChunk && v < a.vocab) {
    const float zv = z[v];
    const bool in = !a.sel || in_support(a.sel[r], zv, v);
    if (in) {
      zt = a.T == 1.f ? zv : zv / a.T;
      uint32_t w[4];
      noise_block(noise_key(a.seed, a.step, 0), (uint32_t)g, (uint32_t)(v >> 2), w);
      key = __fadd_rn(zt, gumbel_from_bits(w[v & 3]));
    }
  }
  int best = key > -INFINITY ? v : 0x7fffffff;
  for (int off = 8; off >= 1; off >>= 1) {   // lanes 0 .. 15: first maximum
    const float k2 = __shfl_xor(key, off);
    const int b2 = __shfl_xor(best, off);
    const float z2 = __shfl_xor(zt, off);
    if (better(k2, b2, key, best)) { key = k2; best = b2; zt = z2; }
  }
  if (lane == 0) {
    const float l = p.m + logf(p.s);
    tokens[g] = best;
    lse[g] = l;
    logq[g] = zt - l;
  }
}

// Eq. 7 for position i of every sequence: z[b][i][v] += (W_c E_c(y))[v] with
// y = y_{i-1}(b), y_0 the anchor (an anchor outside [0, V) reads row 0). A
// workgroup takes 64 VT vocabulary entries, VT per lane, and its four waves the
// rows in turn, kMkPer of every 16 at a time. (Two entries a lane at rank 64 and
// below: the real vocabulary's workgroups are then all resident at once; with one
// a last eighth of them started when the others were done.) The entries' W_c rows reach
// LDS through coalesced 16-byte loads (rows padded by 16 bytes, so the lanes'
// row reads spread over the banks). The rank vectors E_c(y) are the same for
// all lanes: they come by scalar loads and enter the products from scalar
// registers, their conversion from bf16 on the scalar unit (as fp32 in LDS, two
// 16-byte reads for every eight products made the reads, beside the products,
// what bounds the kernel). Each entry's sum runs over the rank index in order
// with separate fp32 multiplies and adds (no fused multiply-add), so the
// corrected logits are a fixed sequence of IEEE operations that the sampler then
// reads like any other logits; at rank 64, 16 sequences and V = 151936 these 311 M
// products and sums a position are 8 to 9 us of vector issue, the floor here.
// LM: also write the chunk log-masses L_c (1: T = 1, 2: divide by T): a chunk's
// 16 tokens sit on 16 lanes, reduced in the log-mass pass's order and with its
// operations, so with its bits, and that pass (a launch and a read of the logits
// for every position) is not needed. Per position 16.9 + 4.6 us of the two
// launches -> 15.8 (8 positions at rank 128, whose staging registers left two
// waves a SIMD: 561 -> 291 us the call).
constexpr int kMkRows = 16, kMkThreads = 256, kMkPer = kMkRows / (kMkThreads / 64);
// 16 bytes as a native vector (arrays of HIP's struct uint4 end up in scratch)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 8 consecutive rank entries at a wave-uniform address, through the scalar cache.
template <typename T> __device__ inline void scalar_rank8(const T* p, float (&e)[8]);
template <> __device__ inline void scalar_rank8<uint16_t>(const uint16_t* p, float (&e)[8]) {
  const u32x4 x = *(const __attribute__((address_space(4))) u32x4*)(uintptr_t)p;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    e[2 * i] = __uint_as_float(x[i] << 16);
    e[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u);
  }
}
template <> __device__ inline void scalar_rank8<float>(const float* p, float (&e)[8]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const u32x4 x = *(const __attribute__((address_space(4))) u32x4*)(uintptr_t)(p + 4 * h);
#pragma unroll
    for (int i = 0; i < 4; ++i) e[4 * h + i] = __uint_as_float(x[i]);
  }
}

struct MarkovArgs {
  float* logits; int batch, B, vocab, i;
  const int32_t* anchor; const int32_t* tokens;
  const void* E; const void* W; int rank;
  float* L; int ldL; float T;   // LM
};

template <typename T, int VT, int LM>
__global__ void __launch_bounds__(kMkThreads) markov_correct_kernel(MarkovArgs a) {
#pragma clang fp contract(off)   // products and sums rounded separately, as the oracle states
  extern __shared__ __attribute__((aligned(16))) uint8_t w_raw[];
  T* w_lds = reinterpret_cast<T*>(w_raw);
  constexpr int EPV = 16 / sizeof(T);   // elements per 16-byte piece (8 or 4)
  const int rank = a.rank, vocab = a.vocab, wld = rank + EPV;   // padded W row in LDS (elements)
  const T* E = static_cast<const T*>(a.E);
  const T* W = static_cast<const T*>(a.W);
  const int v0 = blockIdx.x * 64 * VT, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // the W_c rows of the tile, 4 pieces a thread in flight (rows past V repeat the last one)
  const int per_row = rank / EPV, pieces = 64 * VT * per_row;
  const uint32_t inv = ((1u << 20) + per_row - 1) / per_row;   // exact quotients below 8192
  u32x4 wreg[4];
  auto w_at = [&](int c, int& r, int& k) {
    r = (int)((uint32_t)c * inv >> 20);
    k = (c - r * per_row) * EPV;
  };
  auto w_load = [&](int c0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int r, k;
      w_at(min(c0 + (int)threadIdx.x + q * kMkThreads, pieces - 1), r, k);
      wreg[q] = *reinterpret_cast<const u32x4*>(W + (long)min(v0 + r, vocab - 1) * rank + k);
    }
  };
  auto w_store = [&](int c0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = c0 + (int)threadIdx.x + q * kMkThreads;
      int r, k;
      w_at(c, r, k);
      if (c < pieces) *reinterpret_cast<u32x4*>(w_lds + r * wld + k) = wreg[q];
    }
  };
  w_load(0);
  for (int b0 = 0; b0 < a.batch; b0 += kMkRows) {
    // this wave's sequences b0 + wave, + 4, + 8, + 12 (past the batch: the last one, not stored)
    float zold[kMkPer][VT];
    const T* er[kMkPer];
#pragma unroll
    for (int r = 0; r < kMkPer; ++r) {
      const int b = min(b0 + wave + r * 4, a.batch - 1);
      int y = a.i == 0 ? a.anchor[b] : a.tokens[(long)b * a.B + a.i - 1];
      y = __builtin_amdgcn_readfirstlane(y);
      if (y < 0 || y >= vocab) y = 0;
      er[r] = E + (long)y * rank;
#pragma unroll
      for (int t = 0; t < VT; ++t)
        zold[r][t] = a.logits[((long)b * a.B + a.i) * vocab + min(v0 + t * 64 + lane, vocab - 1)];
    }
    if (b0 == 0) {
      w_store(0);
      for (int c0 = 4 * kMkThreads; c0 < pieces; c0 += 4 * kMkThreads) { w_load(c0); w_store(c0); }
      __syncthreads();
    }
    float c[kMkPer][VT];
#pragma unroll
    for (int r = 0; r < kMkPer; ++r)
#pragma unroll
      for (int t = 0; t < VT; ++t) c[r][t] = 0.f;
    for (int k0 = 0; k0 < rank; k0 += 8) {
      float w[VT][8];
#pragma unroll
      for (int t = 0; t < VT; ++t)
#pragma unroll
        for (int h = 0; h < 8 / EPV; ++h) {
          const u32x4 raw =
              *reinterpret_cast<const u32x4*>(w_lds + (t * 64 + lane) * wld + k0 + h * EPV);
          const T* wv = reinterpret_cast<const T*>(&raw);
#pragma unroll
          for (int e = 0; e < EPV; ++e) w[t][h * EPV + e] = Elem<T>::load(wv + e);
        }
#pragma unroll
      for (int r = 0; r < kMkPer; ++r) {
        float e[8];
        scalar_rank8<T>(er[r] + k0, e);
#pragma unroll
        for (int t = 0; t < VT; ++t) {
          float x = c[r][t];
#pragma unroll
          for (int k = 0; k < 8; ++k) x = x + w[t][k] * e[k];
          c[r][t] = x;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kMkPer; ++r) {
      const int b = b0 + wave + r * 4;
      if (b >= a.batch) break;   // wave-uniform
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        const int v = v0 + t * 64 + lane;
        const float z = zold[r][t] + c[r][t];
        if (v < vocab) a.logits[((long)b * a.B + a.i) * vocab + v] = z;
        if constexpr (LM != 0) {
          const float zt = v < vocab ? (LM == 1 ? z : z / a.T) : -INFINITY;   // IEEE division
          const float m = max16(zt);
          const float l = chunk_log_mass(m, sum16(chunk_term(zt, m)));
          if ((lane & (kChunk - 1)) == 0 && v < vocab) a.L[(long)b * a.ldL + v / kChunk] = l;
        }
      }
    }
  }
}

// Greedy partial: the first argmax of chunk [sp * chunk, ..) of the row; a row
// of one chunk is then done (its token, its logit as lse, log q = 0).
__global__ void __launch_bounds__(kThreads) sample_partial_kernel(SampleArgs a, int32_t* tokens,
                                                                  float* lse, float* logq) {
  const int sp = blockIdx.x, r = blockIdx.y;
  const int v0 = sp * a.chunk, v1 = min(a.vocab, v0 + a.chunk);
  const float* z = a.logits + ((long)r * a.row_mul + a.row_add) * a.vocab;
  Partial p{-INFINITY, 0.f, -INFINITY, 0x7fffffff};
  argmax_tokens(a, z, v0, v1, p);
  for (int off = 32; off >= 1; off >>= 1) {
    Partial o{__shfl_xor(p.m, off), __shfl_xor(p.s, off), __shfl_xor(p.key, off),
              __shfl_xor(p.idx, off)};
    combine(p, o);
  }
  __shared__ Partial red[kThreads / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = p;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kThreads / 64; ++w) combine(p, red[w]);
    if (a.splits > 1) {
      a.part[(long)r * a.splits + sp] = p;
    } else {
      const long g = (long)r * a.row_mul + a.row_add;
      tokens[g] = p.idx;
      lse[g] = p.key;
      logq[g] = 0.f;
    }
  }
}

// One wave per row (T = 0): the greedy partials in order, the first argmax,
// its logit as lse and log q = 0.
__global__ void __launch_bounds__(64) sample_merge_kernel(SampleArgs a, int32_t* tokens,
                                                          float* lse, float* logq) {
  const int r = blockIdx.x, lane = threadIdx.x;
  Partial p{-INFINITY, 0.f, -INFINITY, 0x7fffffff};
  for (int sp = lane; sp < a.splits; sp += 64) combine(p, a.part[(long)r * a.splits + sp]);
  for (int off = 32; off >= 1; off >>= 1) {
    Partial o{__shfl_xor(p.m, off), __shfl_xor(p.s, off), __shfl_xor(p.key, off),
              __shfl_xor(p.idx, off)};
    combine(p, o);
  }
  if (lane == 0) {
    const long g = (long)r * a.row_mul + a.row_add;
    tokens[g] = p.idx;
    lse[g] = p.key;
    logq[g] = 0.f;
  }
}

__global__ void __launch_bounds__(kThreads) gumbel_fill_kernel(uint64_t seed, uint64_t step,
                                                               uint32_t stream, int rows,
                                                               int vocab, float* out) {
  const int groups = (vocab + kGroup - 1) / kGroup;
  const long total = (long)rows * groups;
  for (long i = blockIdx.x * (long)kThreads + threadIdx.x; i < total;
       i += (long)gridDim.x * kThreads) {
    const int r = (int)(i / groups), c = (int)(i % groups);
    uint32_t bits[kGroup];
    noise_group(seed, step, (uint64_t)r, stream, (uint64_t)c, bits);
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      const int v = c * kGroup + k;
      if (v < vocab) out[(long)r * vocab + v] = gumbel_from_bits(bits[k]);
    }
  }
}

}  // namespace

SamplePlan sample_plan(int rows, int vocab) {
  SamplePlan p;
  // T = 0: a chunk of one sweep times the largest power of two that keeps
  // at least 2048 / rows chunks per row (about 2048 workgroups; 4096 measured
  // no faster), one chunk per row from 2048 rows on
  constexpr int sweep = kThreads * kGroup;
  const long target = ((long)vocab * rows + 2047) / 2048;
  int chunk = sweep;
  while (chunk * 2L <= target && chunk < 32 * sweep) chunk *= 2;
  // (and for a vocabulary of at most four sweeps, where the merge's launch
  // costs more than walking them)
  if (rows >= 2048 || vocab <= 4 * sweep) chunk = (vocab + sweep - 1) / sweep * sweep;
  p.greedy_chunk = chunk;
  p.greedy_splits = (vocab + chunk - 1) / chunk;
  // T > 0: 16-token chunks, their log-masses in rows padded to 4 floats
  p.nch = (vocab + kChunk - 1) / kChunk;
  p.ldL = (p.nch + 3) / 4 * 4;
  return p;
}

size_t sample_part_bytes(int rows, int vocab) {
  const SamplePlan p = sample_plan(rows, vocab);
  const size_t L = ((size_t)rows * p.ldL * sizeof(float) + 255) / 256 * 256;
  return L + (size_t)rows * p.greedy_splits * sizeof(Partial);
}

// Static scratch of ldr_sample_noalloc: the sampler's partials and top-k
// supports for callers that cannot allocate. Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the symbol);
// it uses the device address hipGetSymbolAddress returns for the current GPU.
static __device__ __align__(256) uint8_t scratch[LDR_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::once_flag g_scratch_once[kMaxDevices];
void* g_scratch_ptr[kMaxDevices];
hipError_t g_scratch_err[kMaxDevices];
}  // namespace

hipError_t noalloc_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  // once per device, with that device current (the calling thread's)
  std::call_once(g_scratch_once[dev], [dev] {
    void* p = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = g_scratch_err[dev] == hipSuccess ? p : nullptr;
  });
  if (g_scratch_err[dev] != hipSuccess) return g_scratch_err[dev];
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

namespace {
// Arguments of the sampler's kernels for `rows` rows, workspace ws (the
// chunk log-masses, then the partials).
SampleArgs sample_args(const float* logits, int rows, int vocab, float temperature,
                       uint64_t seed, uint64_t step, void* ws, int row_mul, int row_add) {
  const SamplePlan pl = sample_plan(rows, vocab);
  SampleArgs a;
  a.logits = logits; a.rows = rows; a.vocab = vocab; a.T = temperature;
  a.seed = seed; a.step = step;
  a.sel = nullptr; a.row_mul = row_mul; a.row_add = row_add;
  a.vec = vocab % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0;
  a.L = static_cast<float*>(ws);
  a.ldL = pl.ldL; a.nch = pl.nch;
  a.part = reinterpret_cast<Partial*>(static_cast<uint8_t*>(ws) +
                                      ((size_t)rows * pl.ldL * sizeof(float) + 255) / 256 * 256);
  a.chunk = pl.greedy_chunk; a.splits = pl.greedy_splits;
  return a;
}

// The row split evenly over max(1, 2048 / rows) workgroups (about 2048 in all: one
// round of resident workgroups), rounded up to whole sweeps of 1024 tokens.
hipError_t chunk_lse(const SampleArgs& a, hipStream_t st) {
  const int per_row = a.rows >= 2048 ? 1 : 2048 / a.rows;
  const long even = ((long)a.vocab + per_row - 1) / per_row;
  const int slice = (int)((even + 1023) / 1024 * 1024);
  const dim3 grid((unsigned)(((long)a.vocab + slice - 1) / slice), (unsigned)a.rows);
  const bool unit = a.T == 1.f, topk = a.sel != nullptr;
#define LDR_CL(U, K, V) \
  hipLaunchKernelGGL((chunk_lse_kernel<U, K, V>), grid, dim3(kThreads), 0, st, a, slice)
  if (a.vec) {
    if (unit) { if (topk) LDR_CL(true, true, true); else LDR_CL(true, false, true); }
    else { if (topk) LDR_CL(false, true, true); else LDR_CL(false, false, true); }
  } else {
    if (unit) { if (topk) LDR_CL(true, true, false); else LDR_CL(true, false, false); }
    else { if (topk) LDR_CL(false, true, false); else LDR_CL(false, false, false); }
  }
#undef LDR_CL
  return hipGetLastError();
}

bool topk_in_chunks(const SampleArgs& a, int k) {
  return k <= kSelMaxK && a.nch <= kSelMaxChunks;
}

// The rows' top-k supports; with topk_in_chunks also their log-masses (a.L).
hipError_t topk_support(const SampleArgs& a, int k, TopK* sel, hipStream_t st) {
  if (!topk_in_chunks(a, k)) {
    hipLaunchKernelGGL(topk_select_kernel, dim3(a.rows), dim3(kSelThreads), 0, st, a.logits,
                       a.vocab, k, sel, a.row_mul, a.row_add);
    return hipGetLastError();
  }
  if (a.rows > 256 && a.nch <= kSelCap) {   // 4-byte loads at any alignment
    hipLaunchKernelGGL((topk_chunks_kernel<false, 256>), dim3(a.rows), dim3(256), 0, st, a, k, sel);
    return hipGetLastError();
  }
  const size_t lds = (size_t)(a.nch + kSelCap) * 4;   // at most 58 KB: two workgroups a CU
  if (a.vec)
    hipLaunchKernelGGL((topk_chunks_kernel<true, kSelThreads>), dim3(a.rows), dim3(kSelThreads), lds,
                       st, a, k, sel);
  else
    hipLaunchKernelGGL((topk_chunks_kernel<false, kSelThreads>), dim3(a.rows), dim3(kSelThreads),
                       lds, st, a, k, sel);
  return hipGetLastError();
}

hipError_t sample_finish(const SampleArgs& a, int32_t* tokens, float* lse, float* logq,
                         hipStream_t st) {
  if (a.T > 0.f) {
    hipLaunchKernelGGL(chunk_draw_kernel, dim3(a.rows), dim3(kDrawThreads), 0, st, a, tokens,
                       lse, logq);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(sample_partial_kernel, dim3(a.splits, a.rows), dim3(kThreads), 0, st, a,
                     tokens, lse, logq);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return e;
  hipLaunchKernelGGL(sample_merge_kernel, dim3(a.rows), dim3(64), 0, st, a, tokens, lse, logq);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_topk_select(const float* logits, int rows, int vocab, int k, TopK* sel,
                              hipStream_t st) {
  SampleArgs a = sample_args(logits, rows, vocab, 1.f, 0, 0, nullptr, 1, 0);
  a.L = nullptr;   // the supports alone
  return topk_support(a, k, sel, st);
}

hipError_t launch_sample(const float* logits, int rows, int vocab, float temperature,
                         int top_k, uint64_t seed, uint64_t step, int32_t* tokens, float* lse,
                         float* logq, void* ws, size_t sel_off, hipStream_t st, int row_mul,
                         int row_add) {
  SampleArgs a = sample_args(logits, rows, vocab, temperature, seed, step, ws, row_mul, row_add);
  if (temperature > 0.f) {
    if (top_k > 0 && top_k < vocab) {  // T = 0 is the argmax either way
      TopK* sel = reinterpret_cast<TopK*>(static_cast<uint8_t*>(ws) + sel_off);
      const hipError_t e = topk_support(a, top_k, sel, st);   // with the log-masses, if it can
      if (e != hipSuccess) return e;
      a.sel = sel;
      if (topk_in_chunks(a, top_k)) return sample_finish(a, tokens, lse, logq, st);
    }
    const hipError_t e = chunk_lse(a, st);
    if (e != hipSuccess) return e;
  }
  return sample_finish(a, tokens, lse, logq, st);
}

hipError_t launch_sample_finish(const float* logits, int rows, int vocab, float temperature,
                                uint64_t seed, uint64_t step, void* ws, int32_t* tokens,
                                float* lse, float* logq, hipStream_t st) {
  return sample_finish(sample_args(logits, rows, vocab, temperature, seed, step, ws, 1, 0),
                       tokens, lse, logq, st);
}

hipError_t launch_gumbel_fill(uint64_t seed, uint64_t step, int stream, int rows, int vocab,
                              float* out, hipStream_t st) {
  const long groups = (long)rows * ((vocab + kGroup - 1) / kGroup);
  long blocks = (groups + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(gumbel_fill_kernel, dim3((int)(blocks > 0 ? blocks : 1)), dim3(kThreads),
                     0, st, seed, step, (uint32_t)stream, rows, vocab, out);
  return hipGetLastError();
}

hipError_t launch_sample_markov(float* logits, int batch, int B, int vocab, const int32_t* anchor,
                                const void* E, const void* W, int rank, int dtype,
                                float temperature, int top_k, uint64_t seed, uint64_t step,
                                int32_t* tokens, float* lse, float* logq, void* ws,
                                size_t sel_off, hipStream_t st) {
  const int esz = dtype == LDR_BF16 ? 2 : 4;
  const int vt = rank <= 64 ? 2 : 1;   // vocabulary entries per lane
  const size_t lds = (size_t)64 * vt * (rank + 16 / esz) * esz;
  const dim3 grid((unsigned)((vocab + 64 * vt - 1) / (64 * vt)));
  // full-vocabulary draws take the chunk log-masses from the correction
  const bool lm = temperature > 0.f && (top_k == 0 || top_k >= vocab);
  for (int i = 0; i < B; ++i) {
    const SampleArgs sa = sample_args(logits, batch, vocab, temperature, seed, step, ws, B, i);
    MarkovArgs a{logits, batch, B, vocab, i, anchor, tokens, E, W, rank, sa.L, sa.ldL, temperature};
#define LDR_MK(T, VT, LM) \
  hipLaunchKernelGGL((markov_correct_kernel<T, VT, LM>), grid, dim3(kMkThreads), lds, st, a)
#define LDR_MKL(T, VT)                                                    \
  if (!lm) LDR_MK(T, VT, 0); else if (temperature == 1.f) LDR_MK(T, VT, 1); \
  else LDR_MK(T, VT, 2)
    if (dtype == LDR_BF16) {
      if (vt == 2) { LDR_MKL(uint16_t, 2); } else { LDR_MKL(uint16_t, 1); }
    } else {
      if (vt == 2) { LDR_MKL(float, 2); } else { LDR_MKL(float, 1); }
    }
#undef LDR_MKL
#undef LDR_MK
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = lm ? sample_finish(sa, tokens, lse, logq, st)
           : launch_sample(logits, batch, vocab, temperature, top_k, seed, step, tokens, lse, logq,
                           ws, sel_off, st, B, i);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ldr
