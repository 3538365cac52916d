// Fixed-size context views on the GPU (Sec. 2.2; App. A.2, Eq. 10-11).
//
// One workgroup per (kv group g, layer j, sequence b) ingests the new rows of
// that sequence for that head group, reading each new row once:
//  * ring write of the last min(n, W) rows into window slots (t + r) mod W;
//    K rows as they come ([W][d]), V transposed ([d][W]) so that attention
//    reads V with the key index contiguous, as its P.V contraction needs;
//  * for the rep * R summary queries of the group's query heads, the
//    statistics of the new set N (Eq. 10) by a tiled online log-sum-exp over
//    the rows, then the two-way merge with the stored (eta, m) (Eq. 11);
//  * a slice of the boundary-state copy.
// The commit then advances t (or raises the sticky range flag): in the last
// kernel that reads t, the last workgroup of a sequence does it, once every
// other workgroup of that sequence has counted itself done on the sequence's
// device counter (each counts after its own reads of t), so every workgroup
// reads the old t and no separate launch is needed; without new rows a
// one-thread-per-sequence commit kernel does it.
#include "ldr_internal.h"

namespace ldr {
namespace {

constexpr int kThreads = 256;
constexpr int kTileRows = 32;   // rows of N staged in LDS per step

__global__ void __launch_bounds__(kThreads)
views_reset_kernel(uint8_t* arena, size_t stride, size_t eta_off, size_t eta_bytes,
                   int batch, int64_t* pos) {
  const size_t words = stride / 4;
  const size_t total = words * (size_t)batch;
  uint32_t* w = reinterpret_cast<uint32_t*>(arena);
  for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < total;
       i += (size_t)gridDim.x * kThreads) {
    const size_t off = (i % words) * 4;
    const bool is_eta = off >= eta_off && off < eta_off + eta_bytes;
    w[i] = is_eta ? 0xff800000u : 0u;  // -inf log-normalizer, zero elsewhere
  }
  if (blockIdx.x == 0)
    for (int b = threadIdx.x; b < batch; b += kThreads) pos[b] = 0;
}

// The commit of a sequence by the last of its workgroups in a launch (done ==
// null: not this launch). Each sequence has a counter on a line of its own: one
// counter for the whole launch takes an atomic of every workgroup in turn, which
// cost 9 us of the pooled update of 17 rows (1280 workgroups, 24.2 -> 15.6 us).
struct CommitTail {
  int32_t* done;      // device counters, kCommitStride words apart, 0 between launches
  int total;          // workgroups of the launch per sequence
  int64_t* pos; const int32_t* n_new; int max_new; int32_t* status;
};

__device__ inline void commit(const CommitTail& c, int b) {
  const int n = c.n_new[b];
  if (n < 0 || n > c.max_new)
    atomicOr(c.status, kFlagRange);
  else
    c.pos[b] += n;
}

__device__ void commit_tail(const CommitTail& c, int b) {
  if (!c.done) return;
  __syncthreads();   // every thread of the workgroup is past its reads of t
  if (threadIdx.x != 0) return;
  int32_t* done = c.done + b * kCommitStride;
  if (atomicAdd(done, 1) != c.total - 1) return;
  commit(c, b);
  atomicExch(done, 0);   // ready for the next launch
}

struct UpdateArgs {
  uint8_t* arena; size_t stride; size_t kw, vw, m, eta, h;
  const int64_t* pos; const void* G; const int32_t* n_new; int max_new;
  const void* K_new; const void* V_new; const void* h_new;
  int D, hq, hkv, d, W, R, rep, hb_elems;  // hb_elems = L_b * hidden
  int keep_win, keep_sum, keep_bnd;         // views kept (ablation variants drop some)
  int Wx;                                   // rows per (layer, group) region (window first)
  float inv_sqrt_d;
  int splits;                // row ranges per (group, layer, sequence) (bf16 kernel)
  float* part; float* part_ml;   // splits > 1: the ranges' O [unit][split][query][d] and (m, l)
  CommitTail ct;
};

// Sum over aligned groups of tpq lanes (tpq a power of two): DPP lane swaps
// inside rows of 16 (after each step every lane of a group holds the same
// value), cross-row shuffles beyond.
__device__ inline float group_sum(float v, int tpq) {
  if (tpq >= 2) v += dpp<0xB1>(v);
  if (tpq >= 4) v += dpp<0x4E>(v);
  if (tpq >= 8) v += dpp<0x141>(v);
  if (tpq >= 16) v += dpp<0x140>(v);
  for (int off = 16; off < tpq; off <<= 1) v += __shfl_xor(v, off);
  return v;
}

// 16-byte copy of `n16` chunks.
__device__ inline void copy16(void* dst, const void* src, int idx) {
  reinterpret_cast<uint4*>(dst)[idx] = reinterpret_cast<const uint4*>(src)[idx];
}

// This workgroup's slice of the boundary-state copy (the D * H_kv workgroups
// of a sequence share it).
template <typename T>
__device__ inline void boundary_slice(const UpdateArgs& a, uint8_t* seq, int j, int g, int b,
                                      int nthreads) {
  const int chunks = a.hb_elems * (int)sizeof(T) / 16;
  const int wgs = a.D * a.hkv, wid = j * a.hkv + g;
  const int per = (chunks + wgs - 1) / wgs;
  const int c0 = wid * per, c1 = min(chunks, c0 + per);
  T* hdst = reinterpret_cast<T*>(seq + a.h);
  const T* hsrc = reinterpret_cast<const T*>(a.h_new) + (size_t)b * a.hb_elems;
  for (int c = c0 + (int)threadIdx.x; c < c1; c += nthreads) copy16(hdst, hsrc, c);
}

// The same slice in two parts, for a kernel that has other work while the
// loads are in flight: the first chunk of every thread is held in a register.
struct BoundaryCopy { const uint4* src; uint4* dst; int c0, c1; uint4 first; };
template <typename T>
__device__ inline BoundaryCopy boundary_load(const UpdateArgs& a, uint8_t* seq, int j, int g,
                                             int b) {
  const int chunks = a.hb_elems * (int)sizeof(T) / 16;
  const int wgs = a.D * a.hkv, wid = j * a.hkv + g, per = (chunks + wgs - 1) / wgs;
  BoundaryCopy c;
  c.dst = reinterpret_cast<uint4*>(seq + a.h);
  c.src = reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.h_new) +
                                         (size_t)b * a.hb_elems);
  c.c0 = wid * per + (int)threadIdx.x;
  c.c1 = min(chunks, wid * per + per);
  if (c.c0 < c.c1) c.first = c.src[c.c0];
  return c;
}
__device__ inline void boundary_store(const BoundaryCopy& c, int nthreads) {
  if (c.c0 < c.c1) c.dst[c.c0] = c.first;
  for (int i = c.c0 + nthreads; i < c.c1; i += nthreads) c.dst[i] = c.src[i];
}

// DPT: dims of the head each thread owns; TPQ = d / DPT threads share one
// summary query, Q = rep * R queries per workgroup, Q * TPQ = kThreads.
template <typename T, int DPT>
__device__ __forceinline__ void views_update_body(const UpdateArgs& a) {
  const int g = blockIdx.x, j = blockIdx.y, b = blockIdx.z;
  const int n = a.n_new[b];
  if (n <= 0 || n > a.max_new) return;  // empty set: identity; bad count: commit flags it
  const int64_t t = a.pos[b];
  const int d = a.d;
  uint8_t* seq = a.arena + (size_t)b * a.stride;

  // Summary query q of the group is (head g*rep + q / R, summary row q % R);
  // the group's queries are contiguous in G, M and eta. TPQ = d / DPT threads
  // share a query; thread `part` owns dims (c * TPQ + part) * 4 + e.
  constexpr int NV = DPT / 4;         // float4 chunks per thread
  const int tpq = d / DPT;
  const int q = threadIdx.x / tpq;
  const int part = threadIdx.x % tpq;
  const size_t qrow = ((size_t)j * a.hq + g * a.rep) * a.R + q;
  float* Mq = reinterpret_cast<float*>(seq + a.m) + qrow * d;
  float* etaq = reinterpret_cast<float*>(seq + a.eta) + qrow;

  // The stored (eta, m) and the query are loaded first: the stores below go
  // to the same arena, so these loads could not be moved ahead of them.
  const bool sum = a.keep_sum, win = a.keep_win;
  const float eta_a = sum ? *etaq : -INFINITY;
  float4 ma[NV];
  float gq[DPT], acc[DPT];
#pragma unroll
  for (int i = 0; i < DPT; ++i) gq[i] = acc[i] = 0.f;
#pragma unroll
  for (int c = 0; c < NV; ++c) ma[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  if (sum) {
    const T* Gp = reinterpret_cast<const T*>(a.G) + qrow * d;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const int dim = (c * tpq + part) * 4;
      ma[c] = *reinterpret_cast<const float4*>(Mq + dim);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        gq[c * 4 + e] = Elem<T>::load(Gp + dim + e) * a.inv_sqrt_d;
        acc[c * 4 + e] = 0.f;
      }
    }
  }

  if (a.keep_bnd) boundary_slice<T>(a, seq, j, g, b, kThreads);

  // ---- rows of the new set N, tile by tile: window ring write of the last
  // min(n, W) rows (slot (t + r) mod W) and the tiled online log-sum-exp ----
  __shared__ float Ks[kTileRows][256 + 4];
  __shared__ float Vs[kTileRows][256 + 4];
  constexpr int EPC = 16 / sizeof(T);  // elements per 16-byte chunk
  T* Kw = reinterpret_cast<T*>(seq + a.kw) + ((size_t)(j * a.hkv + g) * a.Wx) * d;
  T* Vw = reinterpret_cast<T*>(seq + a.vw) + ((size_t)(j * a.hkv + g) * a.Wx) * d;
  float mx = -INFINITY, l = 0.f;
  for (int r0 = 0; r0 < ((win || sum) ? n : 0); r0 += kTileRows) {
    const int nr = min(kTileRows, n - r0);
    __syncthreads();
    const int cpr = d / EPC;
    for (int i = threadIdx.x; i < nr * cpr; i += kThreads) {
      const int r = i / cpr, e0 = (i % cpr) * EPC;
      const size_t src = ((((size_t)b * a.max_new + r0 + r) * a.D + j) * a.hkv + g) * d + e0;
      const uint4 kv = *reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.K_new) + src);
      const uint4 vv = *reinterpret_cast<const uint4*>(reinterpret_cast<const T*>(a.V_new) + src);
      if (win && r0 + r >= n - a.W) {  // only the last W rows can survive in the ring
        const size_t slot = (size_t)((t + r0 + r) % a.W);
        *reinterpret_cast<uint4*>(Kw + slot * d + e0) = kv;
      }
      const T* kp = reinterpret_cast<const T*>(&kv);
      const T* vp = reinterpret_cast<const T*>(&vv);
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        Ks[r][e0 + e] = Elem<T>::load(kp + e);
        Vs[r][e0 + e] = Elem<T>::load(vp + e);
      }
    }
    __syncthreads();
    {  // window V, transposed: lanes take consecutive rows of one dim, whose
       // slots are contiguous (apart from the wrap of the ring)
      const int rs = max(0, n - a.W - r0);  // first row of the tile that survives
      const int r = threadIdx.x % kTileRows;
      if (win && r >= rs && r < nr) {
        const size_t slot = (size_t)((t + r0 + r) % a.W);
        for (int e = threadIdx.x / kTileRows; e < d; e += kThreads / kTileRows)
          Elem<T>::store(Vw + (size_t)e * a.Wx + slot, Vs[r][e]);
      }
    }
    if (!sum) continue;   // window only: no statistics
    float s[kTileRows];
    float tmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < kTileRows; ++r) {
      s[r] = -INFINITY;
      if (r < nr) {   // uniform: a step's few rows skip the rest of the tile (9: 8.5 -> 7.1 us)
        float p = 0.f;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          const float4 k4 = *reinterpret_cast<const float4*>(&Ks[r][(c * tpq + part) * 4]);
          p += gq[c * 4 + 0] * k4.x + gq[c * 4 + 1] * k4.y + gq[c * 4 + 2] * k4.z +
               gq[c * 4 + 3] * k4.w;
        }
        s[r] = group_sum(p, tpq);
      }
      tmax = fmaxf(tmax, s[r]);
    }
    const float nm = fmaxf(mx, tmax);
    const float alpha = expf(mx - nm);  // mx = -inf on the first tile: 0
    l *= alpha;
#pragma unroll
    for (int i = 0; i < DPT; ++i) acc[i] *= alpha;
#pragma unroll
    for (int r = 0; r < kTileRows; ++r) {
      if (r < nr) {
        const float p = expf(s[r] - nm);
        l += p;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
          const float4 v4 = *reinterpret_cast<const float4*>(&Vs[r][(c * tpq + part) * 4]);
          acc[c * 4 + 0] += p * v4.x;
          acc[c * 4 + 1] += p * v4.y;
          acc[c * 4 + 2] += p * v4.z;
          acc[c * 4 + 3] += p * v4.w;
        }
      }
    }
    mx = nm;
  }
  if (!sum) return;
  // eta_N = log sum exp(s), m_N = sum exp(s - eta_N) v, merged with (eta_A, m_A)
  const float eta_n = mx + logf(l);
  const float inv_l = 1.f / l;
  float wa, wn, eta;
  if (eta_a == -INFINITY) {  // empty A: the merge returns N
    wa = 0.f; wn = inv_l; eta = eta_n;
  } else {
    const float mu = fmaxf(eta_a, eta_n);
    eta = mu + logf(expf(eta_a - mu) + expf(eta_n - mu));
    wa = expf(eta_a - eta);
    wn = expf(eta_n - eta) * inv_l;
  }
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const int dim = (c * tpq + part) * 4;
    const float4 m_a = wa != 0.f ? ma[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 r;
    r.x = wa * m_a.x + wn * acc[c * 4 + 0];
    r.y = wa * m_a.y + wn * acc[c * 4 + 1];
    r.z = wa * m_a.z + wn * acc[c * 4 + 2];
    r.w = wa * m_a.w + wn * acc[c * 4 + 3];
    *reinterpret_cast<float4*>(Mq + dim) = r;
  }
  if (part == 0) *etaq = eta;
}

template <typename T, int DPT>
__global__ void __launch_bounds__(kThreads) views_update_kernel(UpdateArgs a) {
  views_update_body<T, DPT>(a);
  commit_tail(a.ct, blockIdx.z);
}

// bf16 path on the matrix cores (v_mfma_f32_16x16x32_bf16).
//
// One compute wave per 16 summary queries of the group (NW = rep * R / 16) and
// one loader wave, which only stages the new rows, 32 at a time, by DMA
// (global_load_lds) into a ring of NB stages, K rows then V rows, both as they
// lie in memory. (The one or two tiles of a short update are staged by the compute
// waves themselves, all at once: NB = 1 or 2.) The scores are formed transposed, S^T = K G^T, so that a lane
// holds 8 keys of one query and its probabilities are already the B operand of
// O^T = V^T P^T (the order of the contraction index is free as long as both
// operands share it); the V^T operand comes from the row-major V tile by
// transposing LDS reads (ds_read_b64_tr_b16). No operand is transposed through
// LDS stores and no probability passes through LDS.
//  * bf16 products are exact in fp32 and the sums are fp32, as on the vector
//    path; P enters as two bf16 terms, hi = bf16(P) and lo = bf16(P - hi), so
//    its relative error is near 2^-17 rather than bf16's 2^-9 (two MFMAs per
//    tile instead of one);
//  * the online log-sum-exp keeps, per query, a reference m (in log2 units)
//    that moves only when a tile's largest score passes it by more than 8:
//    l and O share it, so a stale reference changes nothing but their scale,
//    and below that no lane exchange and no rescale is needed;
//  * then the merge of Eq. 11 with the stored (eta, m), as on the vector path.
// 16-byte chunk c of row r sits at chunk c ^ row_swz(r) (the DMA permutes its
// source addresses), so that the 16-row fragment reads of K and the 8-row half
// waves of the transposing reads of V each hit 64 distinct banks.
//
// Long updates of few sequences (prefill) leave most CUs without work at one
// workgroup per (group, layer, sequence), so the rows are then also cut into
// `splits` ranges of whole tiles: each workgroup writes its (m, l, O) to the
// caller's workspace and views_commit_merge_kernel combines them in order.
//
// What bounds it: the rows' stream from HBM once the loads run ahead of the
// tiles. Qwen3-8B shape, a 4096-row chunk of one sequence 350 -> 34 us (one
// workgroup per group and layer before; 85 us unsplit), of 16 sequences 661 ->
// 319 us (4.6 TB/s; the loads alone, without any arithmetic, take about as long),
// 17 rows of 16 sequences 20.4 -> 14.8 us.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ inline bf16x8 frag8(const void* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}
template <int N> __device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Chunk permutation of LDS row r (rows of DH bf16, DH / 8 chunks of 16 bytes).
template <int DH> __device__ inline int row_swz(int r) {
  return DH == 128 ? ((r & 7) << 1) | ((r >> 3) & 1) : (((r >> 1) & 3) << 1) | ((r >> 3) & 1);
}

// Weights of the merge of (eta_a, m_a) with a new set of log-normaliser eta_n
// (Eq. 11): m = wa m_a + wn m_n, and the merged eta. An empty A returns N.
__device__ inline void merge_weights(float eta_a, float eta_n, float& wa, float& wn, float& eta) {
  if (eta_a == -INFINITY) {
    wa = 0.f; wn = 1.f; eta = eta_n;
    return;
  }
  const float mu = fmaxf(eta_a, eta_n);
  eta = mu + logf(expf(eta_a - mu) + expf(eta_n - mu));
  wa = expf(eta_a - eta);
  wn = expf(eta_n - eta);
}

constexpr float kLn2 = 0.693147180559945309f, kLog2e = 1.44269504088896341f;

// SUM: the learned summary is kept (otherwise only the ring and the boundary
// are written, from the first tile that holds a surviving row on). NB = 1, 2: the
// update has at most so many tiles (a decode step: one). With the loader wave and
// its four stages two workgroups fit a CU, and each loads its stored (eta, m)
// after the tiles: 33 rows of 64 sequences, on new inputs, 113 us against 91.
template <int DH, int NW, int NB, bool SUM>
__device__ __forceinline__ void views_rows_body(const UpdateArgs& a) {
  constexpr bool SELF = NB <= 2;   // no loader wave
  constexpr int KT = kTileRows, KS = DH / 32, NT = DH / 16, NTH = NW * 64;
  constexpr int CPR = DH / 8, ROWB = DH * 2;      // 16-byte chunks and bytes of a row
  constexpr int MAT = KT * ROWB, STAGE = 2 * MAT; // bytes of a K or V tile, of a stage
  constexpr int QI = MAT / 1024, RPI = 1024 / ROWB;   // DMA instructions a tile, rows each
  __shared__ __attribute__((aligned(1024))) uint8_t sm[NB * STAGE];
  const int g = blockIdx.x, j = blockIdx.y;
  const int b = blockIdx.z / a.splits, sp = blockIdx.z - b * a.splits;
  const int n = a.n_new[b];
  if (n <= 0 || n > a.max_new) return;  // empty set: identity; bad count: commit flags it
  const int64_t t = a.pos[b];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  // this workgroup's tiles
  const int tiles = (n + KT - 1) / KT, per = (tiles + a.splits - 1) / a.splits;
  const int t1 = min(tiles, (sp + 1) * per);
  int t0 = sp * per;
  if (!SUM) t0 = a.keep_win ? max(t0, max(0, n - a.W) / KT) : t1;
  const int nt = t1 - t0;
  const int nr_last = n - (tiles - 1) * KT;
  const bool ragged = t1 == tiles && nr_last < KT;   // the last tile has padding rows

  const size_t rstride = (size_t)a.D * a.hkv * DH;
  const size_t base = (size_t)b * a.max_new * rstride + (size_t)(j * a.hkv + g) * DH;
  const uint16_t* Kn = static_cast<const uint16_t*>(a.K_new) + base;
  const uint16_t* Vn = static_cast<const uint16_t*>(a.V_new) + base;
  // DMA instructions [qa, qb) of a tile's K and V rows; in the ragged tile, rows
  // past n repeat row n - 1
  auto issue = [&](int buf, int tile, int qa, int qb) {
    const int r0 = min(tile, t1 - 1) * KT;
    const bool whole = r0 + KT <= n;
    uint8_t* dst = sm + buf * STAGE;
    const uint16_t* kb = Kn + (size_t)r0 * rstride;
    const uint16_t* vb = Vn + (size_t)r0 * rstride;
#pragma unroll
    for (int q = qa; q < qb; ++q) {
      const int r = q * RPI + lane / CPR;
      const uint32_t row = whole ? r : min(r, n - 1 - r0);
      const uint32_t off = row * (uint32_t)rstride + ((lane % CPR) ^ row_swz<DH>(r)) * 8;
      __builtin_amdgcn_global_load_lds(
          (__attribute__((address_space(1))) void*)(kb + off),
          (__attribute__((address_space(3))) void*)(dst + q * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds(
          (__attribute__((address_space(1))) void*)(vb + off),
          (__attribute__((address_space(3))) void*)(dst + MAT + q * 1024), 16, 0, 0);
    }
  };
  if (!SELF && wave == NW) {   // the loader
    if (nt <= 0) return;
#pragma unroll
    for (int st = 0; st < NB - 1; ++st) issue(st, t0 + st, 0, QI);
    int buf = NB - 1;
    for (int kt = 0; kt < nt; ++kt) {
      wait_vmcnt<2 * QI * (SELF ? 0 : NB - 2)>();   // stage kt has landed
      __builtin_amdgcn_s_barrier();                   // and stage kt - 1 has been read
      if (ragged && kt == nt - 1) __builtin_amdgcn_s_barrier();
      issue(buf, t0 + kt + NB - 1, 0, QI);
      buf = buf == NB - 1 ? 0 : buf + 1;
    }
    wait_vmcnt<0>();   // no DMA outlives the workgroup
    return;
  }
  // every wave stages its share of every tile (none: neither summary nor window)
  if constexpr (SELF) {
#pragma unroll
    for (int st = 0; st < NB; ++st) {
      if (st >= nt) break;
      if constexpr (QI >= NW) {
        issue(st, t0 + st, wave * (QI / NW), (wave + 1) * (QI / NW));
      } else if (wave < QI) {
        issue(st, t0 + st, wave, wave + 1);
      }
    }
  }

  uint8_t* seq = a.arena + (size_t)b * a.stride;
  // the wave's queries: rows q0 .. q0 + 15 of G, M and eta (this lane: query
  // q0 + lr, dims dt * 16 + lg * 4 .. + 3)
  const size_t q0 = ((size_t)j * a.hq + (size_t)g * a.rep) * a.R + (size_t)wave * 16;
  bf16x8 gf[KS];   // B layout: query lr, dims ks * 32 + lg * 8 ..
  if constexpr (SUM) {
    const uint16_t* Gq = static_cast<const uint16_t*>(a.G) + (q0 + lr) * DH + lg * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) gf[ks] = frag8(Gq + ks * 32);
  }
  // the stored (eta, m): ahead of the tiles in a short update, whose time is this
  // latency; after them otherwise
  float* Mq = reinterpret_cast<float*>(seq + a.m) + (q0 + lr) * DH + lg * 4;
  float* etaq = reinterpret_cast<float*>(seq + a.eta) + q0 + lr;
  f32x4 ma[NT];
  float eta_a = -INFINITY;
  auto load_stored = [&]() {
    eta_a = *etaq;
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) ma[dt] = *reinterpret_cast<const f32x4*>(Mq + dt * 16);
  };
  if constexpr (SUM && SELF) load_stored();
  BoundaryCopy bc{};
  if (SELF && a.keep_bnd) bc = boundary_load<uint16_t>(a, seq, j, g, b);

  uint16_t* Kw = reinterpret_cast<uint16_t*>(seq + a.kw) + ((size_t)(j * a.hkv + g) * a.Wx) * DH;
  uint16_t* Vw = reinterpret_cast<uint16_t*>(seq + a.vw) + ((size_t)(j * a.hkv + g) * a.Wx) * DH;
  const uint32_t tm = a.keep_win ? (uint32_t)(t % a.W) : 0u;
  const float c2 = a.inv_sqrt_d * kLog2e;
  const int krow = lr * ROWB, ksz = row_swz<DH>(lr);
  const int vr = lg * 4 + (lr >> 2);
  const int vrow = vr * ROWB + (lr & 1) * 8, vsz = ((lr >> 1) & 1) ^ row_swz<DH>(vr);
  f32x4 o[NT];
#pragma unroll
  for (int dt = 0; dt < NT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;   // of query lr; l: this lane's keys only

  int buf = 0;
  for (int kt = 0; kt < nt; ++kt) {
    const int r0 = (t0 + kt) * KT, nr = min(KT, n - r0);
    if constexpr (SELF) { if (kt == 0) wait_vmcnt<0>(); }   // own share of the tiles
    else __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));   // own LDS reads of stage kt - 1
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");   // the tile's LDS reads stay behind the barrier
    __builtin_amdgcn_sched_barrier(0);
    uint8_t* Kt = sm + buf * STAGE;
    uint8_t* Vt = Kt + MAT;
    if (ragged && kt == nt - 1) {   // padding rows of V are 0 (their probability is)
      for (int i = tid; i < (KT - nr) * CPR; i += NTH)
        *reinterpret_cast<u32x4*>(Vt + nr * ROWB + i * 16) = u32x4{0u, 0u, 0u, 0u};
      lds_barrier();
    }
    if (a.keep_win && r0 + nr > n - a.W) {   // rows that survive in the ring
      const int rs = max(0, n - a.W - r0);
      for (int i = rs * CPR + tid; i < nr * CPR; i += NTH) {
        const int r = i / CPR, c = i % CPR;
        const size_t slot = (tm + (uint32_t)(r0 + r)) % (uint32_t)a.W;
        *reinterpret_cast<u32x4*>(Kw + slot * DH + c * 8) =
            *reinterpret_cast<const u32x4*>(Kt + r * ROWB + ((c ^ row_swz<DH>(r)) * 16));
      }
      const int r = tid % KT;   // V^T: lanes take consecutive rows of one dim
      if (r >= rs && r < nr) {
        const size_t slot = (tm + (uint32_t)(r0 + r)) % (uint32_t)a.W;
        for (int e = tid / KT; e < DH; e += NTH / KT)
          Vw[(size_t)e * a.Wx + slot] = *reinterpret_cast<const uint16_t*>(
              Vt + r * ROWB + (((e >> 3) ^ row_swz<DH>(r)) * 16) + (e & 7) * 2);
      }
    }
    if constexpr (SUM) {
      // raw scores of query lr with keys h * 16 + lg * 4 + v
      f32x4 sc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        sc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          sc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              frag8(Kt + h * 16 * ROWB + krow + (((ks * 4 + lg) ^ ksz) * 16)), gf[ks], sc[h], 0, 0,
              0);
      }
      if (nr < KT) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (h * 16 + lg * 4 + v >= nr) sc[h][v] = -INFINITY;
      }
      float cm = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                       fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3]))) * c2;
      if (__ballot(cm > m + 8.f) != 0) {
        cm = fmaxf(cm, __shfl_xor(cm, 16));
        cm = fmaxf(cm, __shfl_xor(cm, 32));
        const float mn = cm > m + 8.f ? cm : m;
        const float alpha = mn == m ? 1.f : __builtin_amdgcn_exp2f(m - mn);   // first tile: 0
        m = mn;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt) o[dt] *= alpha;
      }
      bf16x8 phi, plo;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sc[i >> 2][i & 3], c2, -m));
        l += p;
        phi[i] = (__bf16)p;
        plo[i] = (__bf16)(p - (float)phi[i]);
      }
#pragma unroll
      for (int dt = 0; dt < NT; ++dt) {
        uint8_t* vp = Vt + vrow + ((vsz ^ (dt * 2)) * 16);
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)vp);
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(vp + 16 * ROWB));
        const bf16x8 vf = __builtin_bit_cast(
            bf16x8, (s16x8)__builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, phi, o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, plo, o[dt], 0, 0, 0);
      }
    }
    buf = buf == NB - 1 ? 0 : buf + 1;
  }
  if (!SELF && a.keep_bnd && sp == 0) bc = boundary_load<uint16_t>(a, seq, j, g, b);
  boundary_store(bc, NTH);
  if constexpr (SUM) {
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (a.splits > 1) {   // (m, l, O) of this range, 0 weight if it is empty
      const size_t row = ((((size_t)b * a.D + j) * a.hkv + g) * a.splits + sp) * (NW * 16) +
                         wave * 16 + lr;
      float* po = a.part + row * DH + lg * 4;
#pragma unroll
      for (int dt = 0; dt < NT; ++dt) *reinterpret_cast<f32x4*>(po + dt * 16) = o[dt];
      if (lg == 0)
        *reinterpret_cast<float2*>(a.part_ml + row * 2) = make_float2(m, l);
      return;
    }
    // eta_N = m + log l, m_N = O / l, merged with (eta_A, m_A) (Eq. 11)
    if constexpr (!SELF) load_stored();
    float wa, wn, e;
    merge_weights(eta_a, m * kLn2 + logf(l), wa, wn, e);
    wn *= 1.f / l;
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) {
      f32x4 r;
#pragma unroll
      for (int v = 0; v < 4; ++v) r[v] = (wa != 0.f ? wa * ma[dt][v] : 0.f) + wn * o[dt][v];
      *reinterpret_cast<f32x4*>(Mq + dt * 16) = r;
    }
    if (lg == 0) *etaq = e;
  }
}

template <int DH, int NW, int NB, bool SUM>
__global__ void __launch_bounds__((NB > 2 ? NW + 1 : NW) * 64)
    __attribute__((amdgpu_waves_per_eu(NB > 2 ? 4 : 3)))
views_update_rows_kernel(UpdateArgs a) {
  views_rows_body<DH, NW, NB, SUM>(a);
  commit_tail(a.ct, blockIdx.z / a.splits);
}

// Combines the row ranges' (m, l, O) of 8 (d 128) or 16 (d 64) queries in range
// order and merges them with the stored (eta, m) (Eq. 11). Grid (group and
// layer, query tile, sequence); a thread owns 4 dims of one query, the threads
// of a query in one wave (so every one of them has read eta before one of them writes it).
template <int DH>
__global__ void __launch_bounds__(256) views_commit_merge_kernel(UpdateArgs a) {
  constexpr int C4 = DH / 4, QP = 256 / C4, U = 8;   // float4s a query, queries, ranges in flight
  const int g = blockIdx.x % a.hkv, j = blockIdx.x / a.hkv, b = blockIdx.z;
  const int n = a.n_new[b], nq = a.rep * a.R;
  if (n > 0 && n <= a.max_new) {
    uint8_t* seq = a.arena + (size_t)b * a.stride;
    const size_t unit = ((size_t)b * a.D + j) * a.hkv + g;
    const int q = blockIdx.y * QP + (int)threadIdx.x / C4, c = (int)threadIdx.x % C4;
    const size_t row0 = unit * a.splits * nq + q;
    const size_t qrow = ((size_t)j * a.hq + (size_t)g * a.rep) * a.R + q;
    float* Mq = reinterpret_cast<float*>(seq + a.m) + qrow * DH + c * 4;
    float* etaq = reinterpret_cast<float*>(seq + a.eta) + qrow;
    const float eta_a = *etaq;
    const f32x4 ma = *reinterpret_cast<const f32x4*>(Mq);
    float m = -INFINITY, l = 0.f;
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < a.splits; s0 += U) {
      float2 ml[U];
      f32x4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {   // ranges past the last one repeat it (weight 0)
        const size_t row = row0 + (size_t)min(s0 + u, a.splits - 1) * nq;
        ml[u] = *reinterpret_cast<const float2*>(a.part_ml + row * 2);
        x[u] = *reinterpret_cast<const f32x4*>(a.part + row * DH + c * 4);
      }
      float mn = m;
#pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, ml[u].x);
      const float alpha = mn == m ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      l *= alpha;
      o *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= a.splits) break;
        const float w = __builtin_amdgcn_exp2f(ml[u].x - m);   // an empty range: 0
        l += w * ml[u].y;
        o += w * x[u];
      }
    }
    float wa, wn, e;
    merge_weights(eta_a, m * kLn2 + logf(l), wa, wn, e);
    wn *= 1.f / l;
    f32x4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = (wa != 0.f ? wa * ma[v] : 0.f) + wn * o[v];
    *reinterpret_cast<f32x4*>(Mq) = r;
    if (c == 0) *etaq = e;
  }
  // t was read by the launch before this one, and is not read here
  if (a.ct.done && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) commit(a.ct, b);
}

// Mean-pooled summary (the views as the configurations word them): for each
// of two strides S, slot c mod P of the bank holds the mean K and V row of
// chunk c = rows [cS, (c+1)S). The chunks the new rows touch are summed in fp32
// in row order, the open chunk continuing from its stored sums, and each slot
// takes sum / rows so far; only the last P chunks are written (older ones would
// be recycled by the same update). Slots are the bank rows after the window
// rows of the (layer, group) region: K row-major, V transposed, like the window.
//
// The chunks of a bank are independent: a team of d / EPC threads (EPC elements of
// K and of V each) sums one chunk, and the teams of a workgroup take runs of
// consecutive chunks, whose V means go through LDS so that the slots of a
// dimension are written side by side (each team writing its own column, 2 bytes
// a line, took 268 us for 1000 rows of 16 sequences, 178 now). EPC is 16 bytes,
// or 2 elements where the launch leaves room for the two to four times as many
// threads (a decode step of few sequences): a thread's chain of conversions, sums
// and divisions is then that much shorter (17 rows of one sequence 7.4 -> 5.1 us,
// of 16 sequences the whole update 21.4 -> 16.9). The first and the last chunk of
// a bank are in one run: the first may continue from the stored sums of the open
// chunk, which the last replaces after the barrier.
struct PoolArgs {
  uint8_t* arena; size_t stride, kw, vw, ps;
  const int64_t* pos; const int32_t* n_new; int max_new;
  const void* K_new; const void* V_new;
  int D, hkv, d, Wr, Wx, P, S0, S1, zc;
  CommitTail ct;
};

// x / y and x % y for x >= 0, in 32 bits where x allows it (a 64-bit division
// is some hundred instructions).
__device__ inline int64_t div_pos(int64_t x, int y) {
  return x <= 0x7fffffff ? (int64_t)((uint32_t)x / (uint32_t)y) : x / y;
}
__device__ inline int mod_pos(int64_t x, int y) { return (int)(x - div_pos(x, y) * y); }

template <int BYTES> struct Piece;   // so many bytes as a native vector
template <> struct Piece<16> { typedef u32x4 type; };
template <> struct Piece<8> { typedef uint32_t type __attribute__((ext_vector_type(2))); };
template <> struct Piece<4> { typedef uint32_t type; };

template <typename T, int EPC>   // EPC: elements a thread
__device__ __forceinline__ void views_pool_body(const PoolArgs& a) {
  typedef typename Piece<EPC * sizeof(T)>::type P;
  constexpr int U = 8;   // rows in flight
  constexpr int kMaxTeams = kThreads / (64 / EPC);
  // [team][d], rows padded by EPC: a column's reads spread over the banks
  __shared__ __attribute__((aligned(16))) T Vs[(kThreads + kMaxTeams) * EPC];
  __shared__ int slots[kMaxTeams];
  const int g = blockIdx.x, j = blockIdx.y, b = blockIdx.z / a.zc, z = blockIdx.z - b * a.zc;
  const int n = a.n_new[b];
  if (n <= 0 || n > a.max_new) return;   // empty set: identity; bad count: commit flags it
  // threads of a team and teams, both powers of two (d is 64 or 128): shifts,
  // since a division by a value known only at run time is some thirty instructions
  // and there were two for every V element written
  const int d = a.d, tw = d / EPC, lw = __builtin_ctz(tw);
  const int lt = __builtin_ctz(kThreads) - lw, teams = 1 << lt;
  const int team = (int)threadIdx.x >> lw, e = ((int)threadIdx.x & (tw - 1)) * EPC;
  const int64_t t = a.pos[b];
  uint8_t* seq = a.arena + (size_t)b * a.stride;
  const size_t grp = (size_t)j * a.hkv + g;
  T* Kw = reinterpret_cast<T*>(seq + a.kw) + grp * a.Wx * d;
  T* Vw = reinterpret_cast<T*>(seq + a.vw) + grp * a.Wx * d;
  const size_t rstride = (size_t)a.D * a.hkv * d;
  const size_t base = (size_t)b * a.max_new * rstride + grp * d + e;
  const T* Kn = static_cast<const T*>(a.K_new) + base;
  const T* Vn = static_cast<const T*>(a.V_new) + base;
  // runs of `teams` chunks, the bank with the longer chunks first, dealt out to
  // the zc workgroups in turn
  int run = z;
  for (int k = 0; k < 2; ++k) {
    const int bank = (a.S0 >= a.S1) == (k == 0) ? 0 : 1;
    const int S = bank ? a.S1 : a.S0;
    const int64_t c0 = div_pos(t, S), c1 = div_pos(t + n - 1, S);
    const int64_t cfirst = c0 > c1 - a.P + 1 ? c0 : c1 - a.P + 1;
    const int items = (int)(c1 - cfirst) + 1, runs = (items + teams - 1) >> lt;
    float* ps = reinterpret_cast<float*>(seq + a.ps) + (grp * 2 + bank) * 2 * d + e;   // K, V sums
    for (; run < runs; run += a.zc) {
      // items: the first chunk, the last, then the ones between
      const int item = run * teams + team;
      const int64_t c = item == 0 ? cfirst : item == 1 ? c1 : cfirst + item - 1;
      const bool live = item < items;
      float sk[EPC], sv[EPC];
      if (live) {
        const int64_t r0 = t > c * S ? t : c * S, r1 = t + n < (c + 1) * S ? t + n : (c + 1) * S;
        const bool carry = c == c0 && c0 * S != t;   // the chunk was opened by an earlier update
        const int f0 = (int)(r0 - t), f1 = (int)(r1 - t);
#pragma unroll
        for (int i = 0; i < EPC; ++i) { sk[i] = carry ? ps[i] : 0.f; sv[i] = carry ? ps[d + i] : 0.f; }
        for (int p0 = f0; p0 < f1; p0 += U) {
          P kx[U], vx[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {   // rows past the chunk repeat its last one (not added)
            const size_t row = (size_t)min(p0 + u, f1 - 1) * rstride;
            kx[u] = *reinterpret_cast<const P*>(Kn + row);
            vx[u] = *reinterpret_cast<const P*>(Vn + row);
          }
          __builtin_amdgcn_sched_barrier(0);   // all loads of the round are in flight
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const bool in = p0 + u < f1;
            const T* kp = reinterpret_cast<const T*>(&kx[u]);
            const T* vp = reinterpret_cast<const T*>(&vx[u]);
#pragma unroll
            for (int i = 0; i < EPC; ++i) {
              const float nk = sk[i] + Elem<T>::load(kp + i), nv = sv[i] + Elem<T>::load(vp + i);
              sk[i] = in ? nk : sk[i];
              sv[i] = in ? nv : sv[i];
            }
          }
        }
        const float cnt = (float)(r1 - c * S);
        const int slot = a.Wr + bank * a.P + mod_pos(c, a.P);
        P ko, vo;
        T* kq = reinterpret_cast<T*>(&ko);
        T* vq = reinterpret_cast<T*>(&vo);
#pragma unroll
        for (int i = 0; i < EPC; ++i) {
          Elem<T>::store(kq + i, sk[i] / cnt);
          Elem<T>::store(vq + i, sv[i] / cnt);
        }
        *reinterpret_cast<P*>(Kw + (size_t)slot * d + e) = ko;
        *reinterpret_cast<P*>(&Vs[team * (d + EPC) + e]) = vo;
        if (e == 0) slots[team] = slot;
      } else if (e == 0) {
        slots[team] = -1;
      }
      __syncthreads();
      if (live && c == c1) {   // the last chunk's sums (used next time only if it is still open)
#pragma unroll
        for (int i = 0; i < EPC; ++i) { ps[i] = sk[i]; ps[d + i] = sv[i]; }
      }
      const int col = (int)threadIdx.x & (teams - 1), vslot = slots[col];
      if (vslot >= 0)   // lanes take the run's slots
        for (int k = (int)threadIdx.x >> lt; k < d; k += tw)
          Vw[(size_t)k * a.Wx + vslot] = Vs[col * (d + EPC) + k];
      __syncthreads();
    }
    run -= runs;
  }
}

// 4 waves a SIMD: one register more than they allow costs up to 4% of 17 to 64
// rows of many sequences (64 of 64 rows: 129.0 us at 3)
template <typename T, int EPC>
__global__ void __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(EPC == 2 ? 6 : 4))) views_pool_kernel(PoolArgs a) {
  views_pool_body<T, EPC>(a);
  commit_tail(a.ct, blockIdx.z / a.zc);
}

__global__ void views_commit_kernel(int batch, int64_t* pos, const int32_t* n_new,
                                    int max_new, int32_t* status) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  const int n = n_new[b];
  if (n < 0 || n > max_new)
    atomicOr(status, kFlagRange);
  else
    pos[b] += n;
}

constexpr int kMaxSplits = 32;   // row ranges of one (group, layer, sequence)

// Compute waves of the bf16 kernel for this shape; 0: the vector kernel.
int views_rows_waves(const Shape& s) {
  if (s.dtype != LDR_BF16 || (s.d != 64 && s.d != 128)) return 0;
  if (!s.learned) return 4;   // ring writes and boundary only
  const int q = s.rep * s.R;
  return q == 32 || q == 64 || q == 128 ? q / 16 : 0;
}

template <typename T>
hipError_t launch_update_t(const UpdateArgs& a, int dpt, dim3 grid, hipStream_t st) {
  switch (dpt) {
    case 4: hipLaunchKernelGGL((views_update_kernel<T, 4>), grid, dim3(kThreads), 0, st, a); break;
    case 8: hipLaunchKernelGGL((views_update_kernel<T, 8>), grid, dim3(kThreads), 0, st, a); break;
    case 16: hipLaunchKernelGGL((views_update_kernel<T, 16>), grid, dim3(kThreads), 0, st, a); break;
    case 32: hipLaunchKernelGGL((views_update_kernel<T, 32>), grid, dim3(kThreads), 0, st, a); break;
    case 64: hipLaunchKernelGGL((views_update_kernel<T, 64>), grid, dim3(kThreads), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The bf16 kernel for NB stages; NW = 4 waves where there are no summary queries.
template <int NB, bool SUM>
hipError_t launch_rows(const Shape& s, const UpdateArgs& a, dim3 grid, hipStream_t st) {
#define LDR_VU(DH, NW)                                                                        \
  if (s.d == DH && views_rows_waves(s) == NW) {                                               \
    hipLaunchKernelGGL((views_update_rows_kernel<DH, NW, NB, SUM>), grid,                     \
                       dim3((NB > 2 ? NW + 1 : NW) * 64), 0, st, a);                          \
    return hipGetLastError();                                                                 \
  }
  LDR_VU(128, 4) LDR_VU(64, 4)
  if constexpr (SUM) { LDR_VU(128, 2) LDR_VU(64, 2) }
  if constexpr (SUM && NB != 2) { LDR_VU(128, 8) LDR_VU(64, 8) }
#undef LDR_VU
  return hipErrorInvalidValue;
}

}  // namespace

// Row ranges of an update with a learned summary: as many as keep the launch
// within the two workgroups per CU that are resident at once (a 4096-row chunk
// of one Qwen3-8B sequence, 40 units: 6 ranges 44.6 us with the merge, 10 41.1,
// 13 -- 520 workgroups, a second round -- 47.8), each of at least 4 tiles (128
// rows; shorter ranges only add partials to write and merge). 1: no split.
int views_splits(const Shape& s, int batch, int max_new) {
  const long units = (long)s.hkv * s.D * batch;
  long sp = 512 / units;
  sp = sp < kMaxSplits ? sp : kMaxSplits;
  const long by_rows = max_new / (4 * kTileRows);
  sp = sp < by_rows ? sp : by_rows;
  return sp > 1 ? (int)sp : 1;
}

size_t views_update_ws_bytes(const Shape& s, int batch, int max_new) {
  if (!s.learned || !views_rows_waves(s)) return 0;
  const int sp = views_splits(s, batch, max_new);
  return sp > 1 ? (size_t)s.hkv * s.D * batch * sp * s.rep * s.R * (s.d + 2) * sizeof(float) : 0;
}

// Threads per summary query: Q = rep * R queries share 256 threads.
int views_dims_per_thread(const Shape& s) {
  if (s.R == 0) return s.d % 16 == 0 ? 16 : 0;   // no learned queries: ring writes only
  const int q = s.rep * s.R;
  if (q <= 0 || q > kThreads || kThreads % q) return 0;
  const int tpq = kThreads / q;
  if (tpq > 64 || s.d % tpq || s.d > 256) return 0;
  const int dpt = s.d / tpq;
  return (dpt == 4 || dpt == 8 || dpt == 16 || dpt == 32 || dpt == 64) ? dpt : 0;
}

hipError_t launch_views_reset(const Shape& s, const Layout& L, int batch, void* arena,
                              int64_t* pos, hipStream_t st) {
  const size_t words = L.stride / 4 * (size_t)batch;
  const int blocks = (int)((words + kThreads - 1) / kThreads < 4096
                               ? (words + kThreads - 1) / kThreads : 4096);
  const size_t eta_bytes = s.learned ? (size_t)s.D * s.hq * s.R * 4 : 0;
  hipLaunchKernelGGL(views_reset_kernel, dim3(blocks > 0 ? blocks : 1), dim3(kThreads), 0, st,
                     static_cast<uint8_t*>(arena), L.stride, L.eta, eta_bytes, batch, pos);
  return hipGetLastError();
}

hipError_t launch_views_update(const Shape& s, const Layout& L, int batch, void* arena,
                               int64_t* pos, const void* G, const int32_t* n_new,
                               int max_new, const void* K_new, const void* V_new,
                               const void* h_new, hipStream_t st, int32_t* status,
                               int32_t* done, void* ws) {
  UpdateArgs a;
  a.arena = static_cast<uint8_t*>(arena); a.stride = L.stride;
  a.kw = L.kw; a.vw = L.vw; a.m = L.m; a.eta = L.eta; a.h = L.h;
  a.pos = pos; a.G = G; a.n_new = n_new; a.max_new = max_new;
  a.K_new = K_new; a.V_new = V_new; a.h_new = h_new;
  a.D = s.D; a.hq = s.hq; a.hkv = s.hkv; a.d = s.d; a.W = s.W; a.R = s.R; a.rep = s.rep;
  a.hb_elems = s.Lb * s.hidden;
  a.keep_win = s.keep_win; a.keep_sum = s.learned; a.keep_bnd = s.keep_bnd;
  a.Wx = s.Wx;
  a.inv_sqrt_d = 1.0f / sqrtf((float)s.d);
  const dim3 grid(s.hkv, s.D, batch);
  a.splits = 1; a.part = nullptr; a.part_ml = nullptr;
  a.ct = CommitTail{done, (int)(grid.x * grid.y), pos, n_new, max_new, status};
  const int q = s.rep * s.R;
  const bool rows_kernel = views_rows_waves(s) > 0;
  // Two tiles without a loader wave where that lets more workgroups onto the CUs
  // and there are more than the two per CU of the four-stage ring (Qwen3-8B
  // shape, 33 rows: 16 sequences 24.0 -> 19.2 us, but 1 sequence 8.8 -> 10.4); the
  // eight waves of 128 queries fill the CUs either way (Qwen3-32B shape, 64
  // sequences: 126 us with the ring, 138 without).
  const bool two_tiles = rows_kernel && views_rows_waves(s) <= 4 && max_new <= 2 * kTileRows &&
                         (long)grid.x * grid.y * grid.z > 512;
  if (rows_kernel && s.learned && max_new <= kTileRows) {
    return launch_rows<1, true>(s, a, grid, st);
  } else if (two_tiles && s.learned) {
    return launch_rows<2, true>(s, a, grid, st);
  } else if (rows_kernel && s.learned) {
    const int sp = ws ? views_splits(s, batch, max_new) : 1;
    const dim3 sgrid(s.hkv, s.D, batch * sp);
    a.splits = sp;
    if (sp == 1) {
      return launch_rows<4, true>(s, a, grid, st);
    } else {
      const size_t rows = (size_t)s.hkv * s.D * batch * sp * q;
      a.part = static_cast<float*>(ws); a.part_ml = a.part + rows * s.d;
      const CommitTail ct = a.ct;
      a.ct.done = nullptr;   // the merge commits
      hipError_t e = launch_rows<4, true>(s, a, sgrid, st);
      if (e != hipSuccess) return e;
      a.ct = ct;
      const dim3 mgrid(s.hkv * s.D, q / (1024 / s.d), batch);
      if (s.d == 128) hipLaunchKernelGGL(views_commit_merge_kernel<128>, mgrid, dim3(256), 0, st, a);
      else hipLaunchKernelGGL(views_commit_merge_kernel<64>, mgrid, dim3(256), 0, st, a);
      return hipGetLastError();
    }
  } else if (rows_kernel) {
    return max_new <= kTileRows       ? launch_rows<1, false>(s, a, grid, st)
           : two_tiles                ? launch_rows<2, false>(s, a, grid, st)
                                      : launch_rows<4, false>(s, a, grid, st);
  }
  const int dpt = views_dims_per_thread(s);
  return s.dtype == LDR_BF16 ? launch_update_t<uint16_t>(a, dpt, grid, st)
                             : launch_update_t<float>(a, dpt, grid, st);
}

hipError_t launch_views_pool(const Shape& s, const Layout& L, int batch, void* arena,
                             int64_t* pos, const int32_t* n_new, int max_new,
                             const void* K_new, const void* V_new, hipStream_t st,
                             int32_t* status, int32_t* done) {
  PoolArgs a;
  a.arena = static_cast<uint8_t*>(arena); a.stride = L.stride; a.kw = L.kw; a.vw = L.vw;
  a.ps = L.ps; a.pos = pos; a.n_new = n_new; a.max_new = max_new; a.K_new = K_new;
  a.V_new = V_new; a.D = s.D; a.hkv = s.hkv; a.d = s.d; a.Wr = s.Wr; a.Wx = s.Wx; a.P = s.P;
  a.S0 = s.S0; a.S1 = s.S1;
  // workgroups per (group, layer, sequence): one per run of chunks the rows can
  // touch, at most about 8 workgroups per CU in all. 2 elements a thread while
  // the runs of those smaller teams stay within that and the rows are few (300
  // rows of one sequence, chunks of 64: 27.3 us against 26.8)
  const int c0 = max_new / s.S0 + 1, c1 = max_new / s.S1 + 1;
  auto runs_of = [&](int epc) -> long {
    const int teams = kThreads / (s.d / epc);
    return ((c0 < s.P ? c0 : s.P) + teams - 1) / teams + ((c1 < s.P ? c1 : s.P) + teams - 1) / teams;
  };
  const long units = (long)s.hkv * s.D * batch, cap = 2048 / units;
  const bool narrow = max_new <= 2 * kTileRows && units * runs_of(2) <= 2048;
  const long runs = runs_of(narrow ? 2 : 16 / (int)s.el);
  const long zc = runs < cap ? runs : cap;
  a.zc = zc > 1 ? (int)zc : 1;
  const dim3 grid(s.hkv, s.D, batch * a.zc), block(kThreads);
  a.ct = CommitTail{done, (int)(grid.x * grid.y) * a.zc, pos, n_new, max_new, status};
  if (s.dtype == LDR_BF16) {
    if (narrow) hipLaunchKernelGGL((views_pool_kernel<uint16_t, 2>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((views_pool_kernel<uint16_t, 8>), grid, block, 0, st, a);
  } else {
    if (narrow) hipLaunchKernelGGL((views_pool_kernel<float, 2>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((views_pool_kernel<float, 4>), grid, block, 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_views_commit(int batch, int64_t* pos, const int32_t* n_new, int max_new,
                               int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(views_commit_kernel, dim3((batch + 255) / 256), dim3(256), 0, st, batch,
                     pos, n_new, max_new, status);
  return hipGetLastError();
}

}  // namespace ldr
