// Weight-streaming linear kernels (MFMA skinny GEMM) with fused RMSNorm scale, RoPE + paged-KV
// write, residual, SwiGLU and LM-head argmax epilogues.
//
//  * k_linear_lds    M <= 16 rows: the activation rows are staged once per workgroup in LDS as MFMA
//                    B-operand slots, so the vector-memory path carries weight tiles only.
//  * k_linear_mfma   any M (prefill, large batches): activation fragments are read from global
//                    memory next to each weight tile.
//
// Both compute every output with the same arithmetic: wave ks of the KS K-splits accumulates its
// k-range in k order on MFMA, and the KS partial sums are added in S consecutive groups
// (y = sum_s (sum_{k in group s} p_k), each sum left to right, starting from 0). The split (KS, S)
// depends only on the weight shape (N, K), so a row's output is bit-identical whatever kernel
// runs it and however many rows share the pass: verifying d drafts gives the same logits, row by
// row, as plain greedy decoding (d = 0). (k_linear_lds supports S == 1 only.)
#include "device_common.h"

#include <algorithm>

namespace seedk {

// n-group of pass j of this workgroup: g0 + j * gs
struct Grp {
  int g0, gs;
};

// ---------------------------------------------------------------------------------------------
// Epilogues. Y(lt, m, c) is the finished fp32 output (column c of local tile lt = j*NT + nl, row
// m). Element e of the (lt, m, c) space is handled by thread e mod blockDim; the global values an
// element needs (residual, gain, KV block, RoPE angles) are loaded for the thread's first element
// at kernel start, before the weight stream, so the epilogue itself costs no extra round trip.
// ---------------------------------------------------------------------------------------------
struct EpiPre {
  float h, g;        // EPI_RESID: residual value and next-norm gain
  int pos, blk;      // EPI_QKV: position and KV block of the row
  float cs, sn;      // EPI_QKV: RoPE cos/sin for the element's rotary pair
};

__device__ __forceinline__ void epi_coords(const LinArgs& a, Grp gr, int e, int& lt, int& m, int& c, int& nt) {
  const int per = a.M * 16;
  lt = e / per;
  const int r = e - lt * per;
  m = r >> 4;
  c = r & 15;
  const int j = lt / a.NT, nl = lt - j * a.NT;
  nt = (gr.g0 + j * gr.gs) * a.NT + nl;
}

template <int EPI>
__device__ __forceinline__ void epi_load(const LinArgs& a, Grp gr, int e, EpiPre& p) {
  int lt, m, c, nt;
  epi_coords(a, gr, e, lt, m, c, nt);
  if (e >= a.NJ * a.NT * a.M * 16 || nt >= (a.N >> 4)) return;
  if constexpr (EPI == EPI_RESID) {
    p.h = a.h[(size_t)m * a.N + nt * 16 + c];
    p.g = a.gain_next[nt * 16 + c];
  } else if constexpr (EPI == EPI_QKV) {
    int sec, head, j;
    qkv_tile(a, nt, sec, head, j);
    p.pos = a.row_slot[m];   // the cache slot (the rotary position enters through row_rope)
    p.blk = a.row_blk[m];
    const int fi = 8 * j + (c & 7);
    p.cs = a.row_rope[(size_t)m * a.head_dim + fi];
    p.sn = a.row_rope[(size_t)m * a.head_dim + (a.head_dim >> 1) + fi];
  }
}

template <typename T, int EPI>
__device__ void linear_epilogue(const LinArgs& a, Grp gr, const float* Y, int y_lt_stride, const EpiPre& pre) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int n_tiles = a.N >> 4;
  const int M = a.M;
  const int total = a.NJ * a.NT * M * 16;
#define YV(lt_, m_, c_) Y[(lt_) * y_lt_stride + (m_) * 16 + (c_)]
  if constexpr (EPI == EPI_RESID || EPI == EPI_QKV) {
    // nthr is a multiple of 64 and total of 16, so the 16 columns of one (lt, m) are 16 aligned
    // lanes of one wave in the same iteration (the ssq butterfly below stays inside them)
    for (int e = tid; e < total; e += nthr) {
      int lt, m, c, nt;
      epi_coords(a, gr, e, lt, m, c, nt);
      if (nt >= n_tiles) continue;
      EpiPre p = pre;
      if (e != tid) epi_load<EPI>(a, gr, e, p);
      if constexpr (EPI == EPI_RESID) {
        const float v = p.h + YV(lt, m, c);
        const size_t off = (size_t)m * a.N + nt * 16 + c;
        a.h[off] = v;
        act_put1<T>(a.xg, a.N >> 5, m, nt * 16 + c, v * p.g);
        float s = v * v;
        s += __shfl_xor(s, 8);
        s += __shfl_xor(s, 4);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 1);
        if (c == 0) a.ssq_out[(size_t)m * n_tiles + nt] = s;
      } else {
        const int HD = a.head_dim, half = HD >> 1;
        int sec, head, j;
        qkv_tile(a, nt, sec, head, j);
        const int d = (c < 8) ? 8 * j + c : half + 8 * j + (c - 8);
        float y = YV(lt, m, c);
        if (sec < 2) {
          const float partner = YV(lt, m, c ^ 8);
          y = (c < 8) ? (y * p.cs - partner * p.sn) : (y * p.cs + partner * p.sn);
        }
        if (sec == 0) {
          a.q[(size_t)m * a.n_heads * HD + head * HD + d] = y;
        } else {
          T* kvp = reinterpret_cast<T*>(a.kv);
          const size_t base = ((size_t)(a.layer * a.n_blocks + p.blk) * 2 + (sec - 1)) * a.n_kv + head;
          if (sec == 1) kvp[base * 16 * HD + (p.pos & 15) * HD + d] = ET<T>::from_f32(y);
          else kvp[base * HD * 16 + d * 16 + (p.pos & 15)] = ET<T>::from_f32(y);
        }
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    const int F = a.N >> 1;
    for (int e = tid; e < a.NJ * a.NT * M * 8; e += nthr) {
      const int lt = e / (M * 8), r = e - lt * M * 8, m = r >> 3, c = r & 7;
      const int j = lt / a.NT, nt = (gr.g0 + j * gr.gs) * a.NT + (lt - j * a.NT);
      if (nt >= n_tiles) continue;
      const float g = YV(lt, m, c), u = YV(lt, m, c + 8);
      act_put1<T>(a.act, F >> 5, m, nt * 8 + c, g / (1.f + __expf(-g)) * u);
    }
  } else {  // EPI_HEAD
    if (a.logits) {
      for (int e = tid; e < total; e += nthr) {
        int lt, m, c, nt;
        epi_coords(a, gr, e, lt, m, c, nt);
        if (nt >= n_tiles) continue;
        a.logits[(long long)m * a.ld_logits + nt * 16 + c] = YV(lt, m, c);
      }
    }
    // argmax of each row over each pass's n-group (lowest token id among equal maxima): one wave
    // per (pass, row), lane-strided candidates, then a butterfly; the partial of n-group g goes to
    // slot g and k_argmax_finalize reduces the slots (none when the caller wants the logits only)
    const int lane = tid & 63, wave = tid >> 6, nw = nthr >> 6;
    for (int q = wave; a.amax_val && q < a.NJ * M; q += nw) {
      const int j = q / M, m = q - j * M;
      const int grp = gr.g0 + j * gr.gs;
      if (grp * a.NT >= n_tiles) continue;
      const int n_cand = min(a.NT, n_tiles - grp * a.NT) * 16;
      const int id0 = grp * a.NT * 16;
      float best = NEG_INF;
      int bi = -1;
      for (int jc = lane; jc < n_cand; jc += 64) {
        const float v = YV(j * a.NT + (jc >> 4), m, jc & 15);
        if (bi < 0 || v > best) { best = v; bi = id0 + jc; }
      }
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(bi, o);
        if (oi >= 0 && (bi < 0 || ov > best || (ov == best && oi < bi))) { best = ov; bi = oi; }
      }
      if (lane == 0) {
        a.amax_val[(size_t)m * a.amax_stride + grp] = best;
        a.amax_idx[(size_t)m * a.amax_stride + grp] = bi;
      }
    }
  }
#undef YV
}

// RMSNorm scale of row m from its per-16-feature sums of squares. Lane partials (lane-strided,
// pre-loaded in ssv when available) are combined by a fixed xor tree, so the value does not
// depend on which wave computes it or on how many rows share the pass.
__device__ __forceinline__ float wave_row_scale(const LinArgs& a, int m, const float* ssv, bool pre) {
  const int lane = threadIdx.x & 63;
  float s;
  if (pre) {
    s = ((ssv[0] + ssv[1]) + ssv[2]) + ssv[3];
  } else {
    s = 0.f;
    for (int j = lane; j < a.nssq; j += 64) s += a.ssq[(size_t)m * a.nssq + j];
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  return rsqrtf(s / (float)a.K + a.eps);
}

__device__ __forceinline__ bool preload_row_ssq(const LinArgs& a, int m, float ssv[4]) {
  const int lane = threadIdx.x & 63;
  if (m >= a.M || a.nssq > 256) return false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = lane + 64 * i;
    ssv[i] = j < a.nssq ? a.ssq[(size_t)m * a.nssq + j] : 0.f;
  }
  return true;
}

// sum of n consecutive wave partials (stride `per` floats), left to right from 0
__device__ __forceinline__ float sum_partials(const float* p, int n, int per) {
  float t = 0.f;
  for (int k = 0; k < n; ++k) t += p[(size_t)k * per];
  return t;
}

// A staged B-operand slot: 32 bytes of LDS holding one row's 8 values of k-group kg of k-tile kt
// (rest = kt * 4 + kg), the two 16-byte halves of the packed activation slot side by side.
struct Slot {
  uint4 p0, p1;
};
__device__ __forceinline__ Slot load_slot(const void* X, int KT, int row, int rest) {
  const char* p = reinterpret_cast<const char*>(X) + ((size_t)(row >> 4) * KT + (rest >> 2)) * ACT_TILE +
                  (row & 15) * ACT_ROW + (rest & 3) * 16;
  return Slot{*reinterpret_cast<const uint4*>(p), *reinterpret_cast<const uint4*>(p + ACT_PLANE)};
}
__device__ __forceinline__ void store_slot(char* p, const Slot& v) {
  reinterpret_cast<uint4*>(p)[0] = v.p0;
  reinterpret_cast<uint4*>(p)[1] = v.p1;
}
template <typename T>
__device__ __forceinline__ typename ET<T>::B lds_slot(const char* p) {
  return ET<T>::join(reinterpret_cast<const uint4*>(p)[0], reinterpret_cast<const uint4*>(p)[1]);
}

__host__ __device__ inline size_t lds_x_bytes(int M, int nkt) { return (size_t)nkt * 4 * M * 32 + 32; }

// ---------------------------------------------------------------------------------------------
// Skinny GEMM with the activation rows in LDS: Y[M, N] = X[M, K] W^T, M <= 16 (one MFMA tile).
//
// The workgroup (NT * KS/S waves) issues its first weight tiles, then stages the X columns of its
// K-slice into LDS as MFMA B-operand slots: slot (kt, kg, r) = 32 bytes holding
// x[r][32kt + 8kg .. +7] (bf16 hi/lo pair for bf16 weights, fp32 otherwise), plus one zero slot
// for the token columns r >= M. Waves then stream weight tiles with P in flight, reading their B
// operands from LDS.
//
// Work: the workgroup makes NJ passes over n-groups blockIdx.x + j*gridDim.x (NT n-tiles each);
// wave (nl, ks) covers k-range ks of n-tile nl of every pass, as one continuous stream. All KS
// K-splits of an n-tile run in one workgroup (the runtime uses this kernel only with S == 1).
// ---------------------------------------------------------------------------------------------
template <typename T, int PRO, int EPI, bool ALIAS>
__global__ void __launch_bounds__(1024) k_linear_lds(LinArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int P = 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NW = a.NT * a.KS;
  const int KT = a.K >> 5, n_tiles = a.N >> 4, M = a.M;
  const int nl = wave / a.KS, ks = wave - nl * a.KS;
  const int tl = lane & 15, kg = lane >> 4;
  const Grp gr{(int)blockIdx.x, (int)gridDim.x};
  const int kt0 = (ks * KT) / a.KS, nk = ((ks + 1) * KT) / a.KS - kt0;
  int nj = 0;
  while (nj < a.NJ && (gr.g0 + nj * gr.gs) * a.NT + nl < n_tiles) ++nj;
  const int Sw = nj * nk;  // weight tiles this wave streams
  const T* w0 = reinterpret_cast<const T*>(a.W) + ((size_t)(gr.g0 * a.NT + nl) * KT + kt0) * 512 + lane * 8;
  const size_t wj = (size_t)gr.gs * a.NT * KT * 512;  // elements from one pass's n-tile to the next

  // ---- weight prefetch ----
  typename ET<T>::A wb[P];
  int jI = 0, iI = 0;  // pass / k-tile of the next tile to issue
  auto issue = [&](int slot) {
    wb[slot] = ET<T>::load_nt(w0 + jI * wj + (size_t)iI * 512);
    if (++iI == nk) { iI = 0; ++jI; }
  };
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (p < Sw) issue(p);

  EpiPre epre{};
  epi_load<EPI>(a, gr, tid, epre);
  float ssv[4] = {0.f, 0.f, 0.f, 0.f};
  bool pre = false;
  if constexpr (PRO == PRO_NORM) pre = preload_row_ssq(a, wave, ssv);

  // ---- stage X into LDS (loads first, then the LDS writes) ----
  const size_t zero_off = (size_t)KT * 4 * M * 32;
  // partials [NJ][NW][M][16] and the row scales: after the staged rows, or (when both do not fit)
  // over them once the stream is done
  constexpr bool alias = ALIAS;
  float* part = reinterpret_cast<float*>(alias ? lds : lds + lds_x_bytes(M, KT));
  float* s_rs = part + (size_t)a.NJ * NW * M * 16;
  {
    // two batches of 2 slots per thread per round trip: both batches' loads are issued before
    // either is written, so a workgroup whose rows take several batches (O at 5 rows, the LM head
    // at more than 3) pays half the round trips. Loads are branch-free (slots past the end reload
    // the last one and are not written) and none is issued after a wait: a load under a branch
    // makes the compiler wait for every load in flight before each write, and a surplus load
    // issued after the first wait would add a round trip to the one-batch case.
    const int items = KT * 4 * M, bs = 2 * (int)blockDim.x;
    Slot xa[2], xb[2];
    auto ld = [&](Slot (&xv)[2], int q0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = min(q0 + u * (int)blockDim.x + tid, items - 1);
        xv[u] = load_slot(a.X, KT, q % M, q / M);
      }
    };
    auto st = [&](const Slot (&xv)[2], int q0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = q0 + u * (int)blockDim.x + tid;
        if (q < items) store_slot(lds + (size_t)q * 32, xv[u]);
      }
    };
    if constexpr (!ALIAS) {
      if (items <= bs) {   // one batch (both paths finish their loads before they merge)
        ld(xa, 0);
        st(xa, 0);
      } else {
        for (int q0 = 0; q0 < items; q0 += 2 * bs) {
          ld(xa, q0);
          ld(xb, q0 + bs);
          st(xa, q0);
          st(xb, q0 + bs);
        }
      }
    } else {
      // one batch per round trip, loads under the item bound: with this variant's pass registers
      // the forms above make the compiler wait for every weight tile of the ring below
      for (int q0 = 0; q0 < items; q0 += bs) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int q = q0 + u * (int)blockDim.x + tid;
          if (q < items) xa[u] = load_slot(a.X, KT, q % M, q / M);
        }
        st(xa, q0);
      }
    }
    if (tid < 2) *reinterpret_cast<float4*>(lds + zero_off + tid * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();

  // ---- stream ----
  const bool live_col = tl < M;
  const char* xa = lds + (live_col ? ((size_t)kt0 * 4 * M + (size_t)kg * M + tl) * 32 : zero_off);
  const size_t xs = live_col ? (size_t)4 * M * 32 : 0;  // bytes per k-tile
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  f32x4 done[ALIAS ? LDS_MAX_PASSES : 1];   // finished passes, kept until the staged rows are no longer read
  int jC = 0, iC = 0;  // pass / k-tile of the next tile to consume
  auto consume = [&](int slot) {
    ET<T>::mma(acc, wb[slot], lds_slot<T>(xa + iC * xs));
    if (++iC == nk) {
      if constexpr (!ALIAS) {
        if (live_col) {
          float* dst = part + ((size_t)(jC * NW + wave) * M + tl) * 16 + 4 * kg;
          dst[0] = acc[0]; dst[1] = acc[1]; dst[2] = acc[2]; dst[3] = acc[3];
        }
      } else {
#pragma unroll
        for (int q = 0; q < (ALIAS ? LDS_MAX_PASSES : 1); ++q)
          if (q == jC) done[q] = acc;
      }
      acc = f32x4{0.f, 0.f, 0.f, 0.f};
      iC = 0;
      ++jC;
    }
  };
  int s0 = 0;
  for (; s0 + 2 * P <= Sw; s0 += P) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      consume(p);
      issue(p);
      // keep each refill next to its consumption (the scheduler would otherwise sink all refills
      // below the last MFMA and drain the pipeline once per P tiles)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (s0 + p < Sw) {
      consume(p);
      if (s0 + p + P < Sw) issue(p);
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (s0 + P + p < Sw) consume(p);

  if constexpr (ALIAS) {
    __syncthreads();   // every wave is done with the staged rows
    if (live_col) {
#pragma unroll
      for (int q = 0; q < (ALIAS ? LDS_MAX_PASSES : 1); ++q)
        if (q < nj) {
          float* dst = part + ((size_t)(q * NW + wave) * M + tl) * 16 + 4 * kg;
          dst[0] = done[q][0]; dst[1] = done[q][1]; dst[2] = done[q][2]; dst[3] = done[q][3];
        }
    }
  }

  // ---- sums over the K-splits (in ks order), RMSNorm row scale, epilogue ----
  if constexpr (PRO == PRO_NORM) {
    for (int m = wave; m < M; m += NW) {
      const float r = wave_row_scale(a, m, ssv, pre && m == wave);
      if (lane == 0) s_rs[m] = r;
    }
  }
  __syncthreads();
  const int per = M * 16;
  for (int e = tid; e < a.NJ * a.NT * per; e += blockDim.x) {
    const int lt = e / per, r = e - lt * per;
    const int j = lt / a.NT, nl2 = lt - j * a.NT;
    float* src = part + (size_t)(j * NW + nl2 * a.KS) * per + r;
    float y = sum_partials(src, a.KS, per);
    if constexpr (PRO == PRO_NORM) y *= s_rs[r >> 4];
    *src = y;
  }
  __syncthreads();
  linear_epilogue<T, EPI>(a, gr, part, a.KS * per, epre);
}

// ---------------------------------------------------------------------------------------------
// Skinny GEMM with activation fragments from global memory: Y[M, N] = X[M, K] W^T, M <= 16*TT.
// Workgroup = NT*KS waves; wave (nl, ks) streams n-tile blockIdx.x*NT+nl over the ks-th
// contiguous range of k-tiles; each wave keeps P weight tiles in flight together with the
// matching activation fragments, refilling a slot right after taking its data (vector memory
// returns in issue order, so every wait is for the oldest slot only). Lanes past the last row
// read row 0 (branch-free issue) and are zeroed when consumed.
// ---------------------------------------------------------------------------------------------
template <typename T, int PRO, int EPI, int TT>
__global__ void __launch_bounds__(1024) k_linear_mfma(LinArgs a) {
  extern __shared__ float smem[];
  __shared__ float s_rs[64];
  float* s_red = smem;         // [NW][M][16]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NW = a.NT * a.KS;
  const int KT = a.K >> 5, n_tiles = a.N >> 4;
  const int M = a.M;
  const int nl = wave / a.KS, ks = wave - nl * a.KS;
  const int nt = blockIdx.x * a.NT + nl;
  const int tl = lane & 15, kg = lane >> 4;
  const Grp gr{(int)blockIdx.x, (int)gridDim.x};
  EpiPre epre{};
  epi_load<EPI>(a, gr, tid, epre);
  float ssv[4] = {0.f, 0.f, 0.f, 0.f};
  bool pre = false;
  if constexpr (PRO == PRO_NORM) pre = preload_row_ssq(a, wave, ssv);
  f32x4 acc[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (nt < n_tiles) {
    const int kt0 = (ks * KT) / a.KS, kt1 = ((ks + 1) * KT) / a.KS;
    const int nk = kt1 - kt0;
    const T* wp = reinterpret_cast<const T*>(a.W) + ((size_t)nt * KT + kt0) * 512 + lane * 8;
    const char* xp[TT];
    bool ok[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int tok = tt * 16 + tl;
      ok[tt] = tok < M;
      xp[tt] = reinterpret_cast<const char*>(a.X) + ((size_t)(ok[tt] ? tt : 0) * KT + kt0) * ACT_TILE +
               (ok[tt] ? tl : 0) * ACT_ROW + kg * 16;
    }
    constexpr int P = (TT <= 1) ? 4 : (TT == 2 ? 3 : 2);
    typename ET<T>::A wb[P];
    Slot xb[P][TT];
    auto issue = [&](int slot, int j) {
      wb[slot] = ET<T>::load_nt(wp + (size_t)j * 512);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        const char* p = xp[tt] + (size_t)j * ACT_TILE;
        xb[slot][tt] = Slot{*reinterpret_cast<const uint4*>(p), *reinterpret_cast<const uint4*>(p + ACT_PLANE)};
      }
    };
    auto consume = [&](int slot) {
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        const uint4 z = make_uint4(0, 0, 0, 0);
        ET<T>::mma(acc[tt], wb[slot], ET<T>::join(ok[tt] ? xb[slot][tt].p0 : z, ok[tt] ? xb[slot][tt].p1 : z));
      }
    };
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (i < nk) issue(i, i);
    int base = 0;
    for (; base + 2 * P <= nk; base += P) {
#pragma unroll
      for (int i = 0; i < P; ++i) {
        consume(i);
        issue(i, base + i + P);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (base + i < nk) {
        consume(i);
        if (base + i + P < nk) issue(i, base + i + P);
      }
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (base + P + i < nk) consume(i);
  }
  // lane (tl, kg) holds rows 4*kg+i of the n-tile for token tt*16+tl
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int tok = tt * 16 + tl;
    if (tok < M) {
      float* dst = s_red + ((size_t)wave * M + tok) * 16 + 4 * kg;
      dst[0] = acc[tt][0]; dst[1] = acc[tt][1]; dst[2] = acc[tt][2]; dst[3] = acc[tt][3];
    }
  }
  if constexpr (PRO == PRO_NORM) {
    for (int m = wave; m < M; m += NW) {
      const float r = wave_row_scale(a, m, ssv, pre && m == wave);
      if (lane == 0) s_rs[m] = r;
    }
  }
  __syncthreads();
  const int per = M * 16, KSs = a.KS / a.S;
  for (int e = tid; e < a.NT * per; e += blockDim.x) {
    const int nl2 = e / per, r = e - nl2 * per;
    float* src = s_red + (size_t)(nl2 * a.KS) * per + r;
    float y = 0.f;
    for (int s2 = 0; s2 < a.S; ++s2) y += sum_partials(src + (size_t)s2 * KSs * per, KSs, per);
    if constexpr (PRO == PRO_NORM) y *= s_rs[r >> 4];
    *src = y;
  }
  __syncthreads();
  linear_epilogue<T, EPI>(a, gr, s_red, a.KS * per, epre);
}

// ---------------------------------------------------------------------------------------------
// Wide passes (16 < M <= 64 rows: batched verification, prefill, the drafting objective's pass):
// the K split runs across workgroups. Workgroup (n-group g, k-range ks) stages the activation
// columns of its k-range only (they fit LDS where the whole K of M rows does not) and its NT
// waves stream one n-tile each over that range, exactly as wave (nl, ks) of the narrow kernels
// does (same tiles, same order, same B slots), for TT token tiles of 16 rows. The range partials
// go to global memory; k_splitk_reduce adds them in k-range order from 0 and runs the epilogue,
// so every row gets the bit-identical output of the narrow kernels.
// ---------------------------------------------------------------------------------------------
template <typename T, int TT, int XI, int PRO>
__global__ void __launch_bounds__(512) k_linear_splitk(LinArgs a, float* part) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int P = 8;
  const int tid = threadIdx.x, lane = tid & 63, nl = tid >> 6;
  const int KT = a.K >> 5, n_tiles = a.N >> 4, M = a.M;
  const int tl = lane & 15, kg = lane >> 4;
  const int ks = blockIdx.y;
  const int kt0 = (ks * KT) / a.KS, nk = ((ks + 1) * KT) / a.KS - kt0;
  const int nt = blockIdx.x * a.NT + nl;
  const bool live = nt < n_tiles;
  const T* w0 = reinterpret_cast<const T*>(a.W) + ((size_t)(live ? nt : 0) * KT + kt0) * 512 + lane * 8;

  // ---- the k-range's activations first (cache hits: issued ahead of the weight tiles they do
  // not queue behind the weights' HBM round trip), XI items per thread, branch-free: item
  // q = (i*4 + kg)*M + r is slot q = x[r][32(kt0+i) + 8kg .. +7]; items past the end load item 0
  // and go to a dummy slot ----
  const int items = nk * 4 * M;
  Slot xv[XI];
#pragma unroll
  for (int u = 0; u < XI; ++u) {
    const int q = u * (int)blockDim.x + tid, qc = q < items ? q : 0;
    xv[u] = load_slot(a.X, KT, qc % M, kt0 * 4 + qc / M);
  }

  // ---- weight prefetch (slots past the range re-read its last tile, never consumed) ----
  typename ET<T>::A wb[P];
#pragma unroll
  for (int p = 0; p < P; ++p) wb[p] = ET<T>::load_nt(w0 + (size_t)min(p, nk - 1) * 512);

  const size_t zero_off = (size_t)items * 32;
#pragma unroll
  for (int u = 0; u < XI; ++u) {
    const int q = u * (int)blockDim.x + tid;
    store_slot(lds + (q < items ? (size_t)q * 32 : zero_off + 32), xv[u]);
  }
  // items beyond XI per thread (shapes the launcher could not cover up front)
  for (int q = XI * (int)blockDim.x + tid; q < items; q += blockDim.x) {
    store_slot(lds + (size_t)q * 32, load_slot(a.X, KT, q % M, kt0 * 4 + q / M));
  }
  if (tid < 2) *reinterpret_cast<float4*>(lds + zero_off + tid * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();

  // ---- stream the range: TT token tiles per weight tile ----
  const char* xa[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int m = tt * 16 + tl;
    xa[tt] = lds + (m < M ? ((size_t)kg * M + m) * 32 : zero_off);
  }
  const size_t xs = (size_t)4 * M * 32;   // bytes per k-tile
  f32x4 acc[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto consume = [&](int slot, int i) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int m = tt * 16 + tl;
      ET<T>::mma(acc[tt], wb[slot], lds_slot<T>(xa[tt] + (m < M ? i * xs : 0)));
    }
  };
  int s0 = 0;
  for (; s0 + 2 * P <= nk; s0 += P) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      consume(p, s0 + p);
      wb[p] = ET<T>::load_nt(w0 + (size_t)(s0 + p + P) * 512);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    if (s0 + p < nk) {
      consume(p, s0 + p);
      if (s0 + p + P < nk) wb[p] = ET<T>::load_nt(w0 + (size_t)(s0 + p + P) * 512);
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (s0 + P + p < nk) consume(p, s0 + P + p);

  // ---- the RMSNorm row scales, once per launch (workgroup (0, 0)), for the reduction ----
  if constexpr (PRO == PRO_NORM) {
    if (blockIdx.x == 0 && blockIdx.y == 0) {
      const float ssv[4] = {0.f, 0.f, 0.f, 0.f};
      for (int m = nl; m < M; m += a.NT) {
        const float r = wave_row_scale(a, m, ssv, false);
        if (lane == 0) a.part_rs[m] = r;
      }
    }
  }
  // ---- range partial: part[ks][m][n], lane (tl, kg) holds features 4kg..4kg+3 of token tt*16+tl ----
  if (live) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int m = tt * 16 + tl;
      if (m < M)
        *reinterpret_cast<float4*>(part + ((size_t)ks * M + m) * a.N + nt * 16 + 4 * kg) =
            make_float4(acc[tt][0], acc[tt][1], acc[tt][2], acc[tt][3]);
    }
  }
}

// Sum of the k-range partials (k-range order, from 0), RMSNorm row scale, epilogue. Workgroup g
// handles n-tiles g*NT .. g*NT+NT-1 of all M rows (a.NT, a.NJ = 1 describe that layout to the
// shared epilogue); the launcher gives it one thread per output element.
template <typename T, int PRO, int EPI>
__global__ void __launch_bounds__(1024) k_splitk_reduce(LinArgs a, const float* part) {
  extern __shared__ float Y[];   // [NT][M][16]
  const int tid = threadIdx.x;
  const int M = a.M, n_tiles = a.N >> 4;
  const Grp gr{(int)blockIdx.x, (int)gridDim.x};
  EpiPre epre{};
  epi_load<EPI>(a, gr, tid, epre);
  const int per = M * 16;
  for (int e = tid; e < a.NT * per; e += blockDim.x) {
    const int lt = e / per, r = e - lt * per, m = r >> 4, c = r & 15;
    const int nt = blockIdx.x * a.NT + lt;
    // all k-range partials in flight at once, then added in k-range order from 0 (the order of
    // sum_partials)
    const float* pp = part + (size_t)m * a.N + min(nt, n_tiles - 1) * 16 + c;
    const size_t stride = (size_t)M * a.N;
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = k < a.KS ? pp[k * stride] : 0.f;
    float y = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (k < a.KS) y += v[k];
    for (int k = 16; k < a.KS; ++k) y += pp[k * stride];
    if constexpr (PRO == PRO_NORM) y *= a.part_rs[m];   // row scale from the split-K launch
    Y[e] = nt < n_tiles ? y : 0.f;
  }
  __syncthreads();
  linear_epilogue<T, EPI>(a, gr, Y, per, epre);
}

// Reduce per-n-group argmax partials of one row; lowest token id wins among equal maxima.
__global__ void __launch_bounds__(256) k_argmax_finalize(const float* val, const int* idx, int stride, int n_parts,
                                                         int* tok_out, int tok_stride) {
  const int m = blockIdx.x, tid = threadIdx.x;
  __shared__ float s_v[256];
  __shared__ int s_i[256];
  float best = NEG_INF;
  int bi = -1;
  for (int j = tid; j < n_parts; j += blockDim.x) {
    const float v = val[(size_t)m * stride + j];
    const int i = idx[(size_t)m * stride + j];
    if (i >= 0 && (bi < 0 || v > best || (v == best && i < bi))) { best = v; bi = i; }
  }
  s_v[tid] = best;
  s_i[tid] = bi;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if (tid < o) {
      const float v = s_v[tid + o];
      const int i = s_i[tid + o];
      if (i >= 0 && (s_i[tid] < 0 || v > s_v[tid] || (v == s_v[tid] && i < s_i[tid]))) { s_v[tid] = v; s_i[tid] = i; }
    }
    __syncthreads();
  }
  if (tid == 0) tok_out[m * tok_stride] = s_i[0] < 0 ? 0 : s_i[0];
}

// ---------------------------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------------------------
// Waves (n-tiles) per workgroup of the split-K kernel: 8, or fewer (down to 4) where that gives
// the busiest CU at least 30% fewer weight tiles with the grid's workgroups spread evenly over the
// 256 CUs: the 2560-wide projections (down: 160 n-tiles x 16 k-ranges make 320 workgroups of 8,
// so 64 CUs stream two, against 512 of 5, two on every CU; O: 160 workgroups of 8 leave 96 CUs
// idle, 256 of 5 fill them). Measured: verify down 17.9 -> 16.0 us at 5 rows, O 16.4 -> 15.4 us at
// 40 rows; QKV (384 n-tiles, 25% by this count) was slower with 6. Each wave's work and summation
// order are the same for any choice.
static int splitk_nt(int n_tiles, int ks) {
  constexpr int CUS = 256;
  auto cost = [&](int nt) {   // weight tiles per k-range on the busiest CU
    const long long wgs = (long long)((n_tiles + nt - 1) / nt) * ks;
    return (wgs + CUS - 1) / CUS * nt;
  };
  int best = 8;
  for (int nt = 7; nt >= 4; --nt)
    if (cost(nt) < cost(best)) best = nt;
  return 10 * cost(best) <= 7 * cost(8) ? best : 8;
}

size_t linear_lds_bytes(int M, int K, int NT, int KS, int S, int NJ, int kind) {
  (void)S;
  if (kind == LIN_LDS) {
    const size_t x = lds_x_bytes(M, K >> 5), part = (size_t)(NJ * NT * KS * M + 1) * 16 * sizeof(float);
    return x + part <= linear_lds_limit() ? x + part : std::max(x, part);
  }
  if (kind == LIN_SPLITK) {
    const int nk_max = ((K >> 5) + KS - 1) / KS;
    return (size_t)nk_max * 4 * M * 32 + 64;
  }
  return (size_t)(NT * KS * M * 16) * sizeof(float);
}

// ---------------------------------------------------------------------------------------------
// LM head for 16 < M <= 64 rows (batched verification, draft trees of more than 16 nodes): the
// activation rows of all M tokens do not fit LDS whole (4 bytes per element as MFMA B slots), so
// they are staged in chunks of HEAD_CK k-tiles, double-buffered: the loads of chunk c+1 are issued
// before chunk c is consumed and written to the other buffer after it. Each of the 8 waves
// streams one n-tile over all of K in k order (KS = 1, as the narrow kernel does for any M), for TT
// token tiles of 16 rows, so every row's logits are bit-identical to a pass of fewer rows. A
// workgroup has HEAD_WIDE_NT = 16 waves (n-tiles), so the 40 staged rows of a batch-8 verification
// are read by 594 workgroups instead of 1187 (the argmax partials are per 16-n-tile group; the
// maximum over them is the same).
// ---------------------------------------------------------------------------------------------
constexpr int HEAD_CK = 8;   // k-tiles per staged chunk (= the weight ring depth)
static size_t g_lds_limit = 65536;   // dynamic LDS one workgroup may use (set by configure_kernels)

template <typename T, int TT, int NW>
__global__ void __launch_bounds__(NW * 64) k_linear_head_chunked(LinArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ float s_rs[64];
  constexpr int P = HEAD_CK;
  constexpr int NTH = NW * 64;
  constexpr int XI = (HEAD_CK * 4 * 16 * TT + NTH - 1) / NTH;   // staged items per thread and chunk
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int KT = a.K >> 5, n_tiles = a.N >> 4, M = a.M;
  const int tl = lane & 15, kg = lane >> 4;
  const Grp gr{(int)blockIdx.x, (int)gridDim.x};
  const int nt = blockIdx.x * a.NT + wave;
  const T* w0 = reinterpret_cast<const T*>(a.W) + (size_t)(nt < n_tiles ? nt : 0) * KT * 512 + lane * 8;
  const size_t chunk_bytes = (size_t)HEAD_CK * 4 * M * 32;
  const size_t zero_off = 2 * chunk_bytes;
  const int NC = (KT + HEAD_CK - 1) / HEAD_CK;

  EpiPre epre{};
  epi_load<EPI_HEAD>(a, gr, tid, epre);
  float ssv[4] = {0.f, 0.f, 0.f, 0.f};
  const bool pre = preload_row_ssq(a, wave, ssv);

  // chunk c's items q = (ktl*4 + kg)*M + r hold x[r][32(c*CK + ktl) + 8kg .. +7]; loaded branch-free
  // (items past the chunk reload item 0 and are not written)
  Slot xv[XI];
  auto stage_load = [&](int c) {
    const int nkc = min(HEAD_CK, KT - c * HEAD_CK), items = nkc * 4 * M;
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      const int q = u * NTH + tid, qc = q < items ? q : 0;
      xv[u] = load_slot(a.X, KT, qc % M, c * HEAD_CK * 4 + qc / M);
    }
  };
  auto stage_store = [&](int c) {
    const int nkc = min(HEAD_CK, KT - c * HEAD_CK), items = nkc * 4 * M;
    char* buf = lds + (c & 1) * chunk_bytes;
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      const int q = u * NTH + tid;
      if (q < items) store_slot(buf + (size_t)q * 32, xv[u]);
    }
  };

  stage_load(0);
  typename ET<T>::A wb[P];
#pragma unroll
  for (int p = 0; p < P; ++p) wb[p] = ET<T>::load_nt(w0 + (size_t)min(p, KT - 1) * 512);
  stage_store(0);
  if (tid < 2) *reinterpret_cast<float4*>(lds + zero_off + tid * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();

  f32x4 acc[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // every load below is issued unconditionally (the last chunk is reloaded past the end, weight
  // tiles past K re-read the last one, neither is consumed): a load under a data-dependent branch
  // makes the compiler's wait counts assume the path without it, and every refill would then wait
  // for the whole ring
  for (int c = 0; c < NC; ++c) {
    stage_load(min(c + 1, NC - 1));
    const char* buf = lds + (c & 1) * chunk_bytes;
    const int nkc = min(HEAD_CK, KT - c * HEAD_CK);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (p < nkc) {
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const int m = tt * 16 + tl;
          const char* xb = m < M ? buf + ((size_t)(p * 4 + kg) * M + m) * 32 : lds + zero_off;
          ET<T>::mma(acc[tt], wb[p], lds_slot<T>(xb));
        }
      }
      const int nxt = c * HEAD_CK + p + P;
      wb[p] = ET<T>::load_nt(w0 + (size_t)min(nxt, KT - 1) * 512);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (c + 1 < NC) stage_store(c + 1);
    __syncthreads();
  }

  // lane (tl, kg) holds features 4kg..4kg+3 of token tt*16+tl: Y[wave][m][16] over the buffers
  float* Y = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int m = tt * 16 + tl;
    if (m < M) {
      float* dst = Y + ((size_t)wave * M + m) * 16 + 4 * kg;
      dst[0] = acc[tt][0]; dst[1] = acc[tt][1]; dst[2] = acc[tt][2]; dst[3] = acc[tt][3];
    }
  }
  for (int m = wave; m < M; m += a.NT) {
    const float r = wave_row_scale(a, m, ssv, pre && m == wave);
    if (lane == 0) s_rs[m] = r;
  }
  __syncthreads();
  const int per = M * 16;
  for (int e = tid; e < a.NT * per; e += blockDim.x) {
    float y = sum_partials(Y + e, 1, per);   // the one k-range, as the narrow kernel adds it
    y *= s_rs[(e % per) >> 4];
    Y[e] = y;
  }
  __syncthreads();
  linear_epilogue<T, EPI_HEAD>(a, gr, Y, per, epre);
}

size_t head_chunked_lds(int M) { return 2 * (size_t)HEAD_CK * 4 * M * 32 + 32; }

template <typename T, int PRO, int EPI>
static void launch_linear_pe(const LinArgs& a0, int kind, hipStream_t s, const LaunchEvents* ev) {
  LinArgs a = a0;
  const int n_tiles = a.N >> 4;
  const int n_groups = (n_tiles + a.NT - 1) / a.NT;
  if (kind == LIN_LDS) {
    const dim3 grid((n_groups + a.NJ - 1) / a.NJ);
    const dim3 block(64 * a.NT * a.KS);
    const size_t lds = linear_lds_bytes(a.M, a.K, a.NT, a.KS, a.S, a.NJ, kind);
    const bool alias = lds < lds_x_bytes(a.M, a.K >> 5) + (size_t)(a.NJ * a.NT * a.KS * a.M + 1) * 16 * sizeof(float);
    if (alias) launch(k_linear_lds<T, PRO, EPI, true>, grid, block, lds, s, ev, a);
    else launch(k_linear_lds<T, PRO, EPI, false>, grid, block, lds, s, ev, a);
    return;
  }
  if (kind == LIN_SPLITK) {
    const int nk_max = ((a.K >> 5) + a.KS - 1) / a.KS;
    LinArgs b = a;
    b.NT = splitk_nt(n_tiles, a.KS);
    b.NJ = 1;
    const dim3 grid((n_tiles + b.NT - 1) / b.NT, a.KS), block(64 * b.NT);
    const size_t lds = (size_t)nk_max * 4 * a.M * 32 + 64;   // + zero slot + dummy slot
    const LaunchEvents e0{ev ? ev->start : nullptr, nullptr}, e1{nullptr, ev ? ev->stop : nullptr};
    const int xi = (nk_max * 4 * a.M + (int)block.x - 1) / (int)block.x <= 4 ? 4 : 8;
    const LaunchEvents* e = ev ? &e0 : nullptr;
    switch ((a.M + 15) / 16 * 16 + xi) {
      case 20: launch(k_linear_splitk<T, 1, 4, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 24: launch(k_linear_splitk<T, 1, 8, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 36: launch(k_linear_splitk<T, 2, 4, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 40: launch(k_linear_splitk<T, 2, 8, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 52: launch(k_linear_splitk<T, 3, 4, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 56: launch(k_linear_splitk<T, 3, 8, PRO>, grid, block, lds, s, e, b, a.part); break;
      case 68: launch(k_linear_splitk<T, 4, 4, PRO>, grid, block, lds, s, e, b, a.part); break;
      default: launch(k_linear_splitk<T, 4, 8, PRO>, grid, block, lds, s, e, b, a.part); break;
    }
    // one output element per thread (the epilogue loads each thread's row data up front)
    LinArgs r = a;
    r.NT = 1;
    r.NJ = 1;
    const int rthreads = (a.M * 16 + 63) / 64 * 64;
    launch(k_splitk_reduce<T, PRO, EPI>, dim3(n_tiles), dim3(rthreads), (size_t)a.M * 16 * sizeof(float), s,
           ev ? &e1 : nullptr, r, (const float*)a.part);
    return;
  }
  a.NJ = 1;
  const dim3 grid(n_groups), block(64 * a.NT * a.KS);
  const int TT = (a.M + 15) / 16;
  if constexpr (EPI == EPI_HEAD) {
    if (a.M > 16 && a.KS == 1 && a.NT == HEAD_WIDE_NT && a.S == 1 && head_chunked_lds(a.M) <= g_lds_limit) {
      const size_t lds_h = head_chunked_lds(a.M);
      switch (TT) {
        case 2: launch(k_linear_head_chunked<T, 2, HEAD_WIDE_NT>, grid, block, lds_h, s, ev, a); break;
        case 3: launch(k_linear_head_chunked<T, 3, HEAD_WIDE_NT>, grid, block, lds_h, s, ev, a); break;
        default: launch(k_linear_head_chunked<T, 4, HEAD_WIDE_NT>, grid, block, lds_h, s, ev, a); break;
      }
      return;
    }
  }
  const size_t lds = linear_lds_bytes(a.M, a.K, a.NT, a.KS, a.S, 1, kind);
  switch (TT) {
    case 1: launch(k_linear_mfma<T, PRO, EPI, 1>, grid, block, lds, s, ev, a); break;
    case 2: launch(k_linear_mfma<T, PRO, EPI, 2>, grid, block, lds, s, ev, a); break;
    case 3: launch(k_linear_mfma<T, PRO, EPI, 3>, grid, block, lds, s, ev, a); break;
    default: launch(k_linear_mfma<T, PRO, EPI, 4>, grid, block, lds, s, ev, a); break;
  }
}

template <typename T>
void launch_linear(const LinArgs& a, int prologue, int epilogue, int kind, hipStream_t s, const LaunchEvents* ev) {
  if (kind == LIN_WIDE) {
    launch_linear_wide<T>(a, epilogue, s, ev);
    return;
  }
  if (prologue == PRO_NORM) {
    switch (epilogue) {
      case EPI_QKV: launch_linear_pe<T, PRO_NORM, EPI_QKV>(a, kind, s, ev); break;
      case EPI_SWIGLU: launch_linear_pe<T, PRO_NORM, EPI_SWIGLU>(a, kind, s, ev); break;
      default: launch_linear_pe<T, PRO_NORM, EPI_HEAD>(a, kind, s, ev); break;
    }
  } else {
    launch_linear_pe<T, PRO_PLAIN, EPI_RESID>(a, kind, s, ev);
  }
}

void launch_argmax_finalize(const float* val, const int* idx, int stride, int n_parts, int M, int* tok_out,
                            int tok_stride, hipStream_t s) {
  hipLaunchKernelGGL(k_argmax_finalize, dim3(M), dim3(256), 0, s, val, idx, stride, n_parts, tok_out, tok_stride);
}

template <typename T, int PRO, int EPI>
static bool allow_big_lds(int bytes) {
  const void* fns[] = {reinterpret_cast<const void*>(&k_linear_lds<T, PRO, EPI, false>),
                       reinterpret_cast<const void*>(&k_linear_lds<T, PRO, EPI, true>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 1, 4, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 1, 8, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 2, 4, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 2, 8, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 3, 4, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 3, 8, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 4, 4, PRO>),
                       reinterpret_cast<const void*>(&k_linear_splitk<T, 4, 8, PRO>),
                       reinterpret_cast<const void*>(&k_linear_head_chunked<T, 2, HEAD_WIDE_NT>),
                       reinterpret_cast<const void*>(&k_linear_head_chunked<T, 3, HEAD_WIDE_NT>),
                       reinterpret_cast<const void*>(&k_linear_head_chunked<T, 4, HEAD_WIDE_NT>),
                       reinterpret_cast<const void*>(&k_linear_mfma<T, PRO, EPI, 1>),
                       reinterpret_cast<const void*>(&k_linear_mfma<T, PRO, EPI, 2>),
                       reinterpret_cast<const void*>(&k_linear_mfma<T, PRO, EPI, 3>),
                       reinterpret_cast<const void*>(&k_linear_mfma<T, PRO, EPI, 4>)};
  bool ok = true;
  for (const void* f : fns) ok &= hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
  return ok;
}


// Dynamic LDS available to one linear workgroup: the device's per-block limit, raised to the
// opt-in limit when every linear kernel accepted it (failed opt-ins are cleared and ignored).
hipError_t configure_kernels(int bf16) {
  int dev = 0, base = 0, optin = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
  if (hipDeviceGetAttribute(&base, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && base > 0)
    g_lds_limit = (size_t)base;
  if (hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, dev) == hipSuccess &&
      (size_t)optin > g_lds_limit) {
    bool ok;
    if (bf16) {
      ok = allow_big_lds<uint16_t, PRO_NORM, EPI_QKV>(optin) & allow_big_lds<uint16_t, PRO_NORM, EPI_SWIGLU>(optin) &
           allow_big_lds<uint16_t, PRO_NORM, EPI_HEAD>(optin) & allow_big_lds<uint16_t, PRO_PLAIN, EPI_RESID>(optin);
    } else {
      ok = allow_big_lds<float, PRO_NORM, EPI_QKV>(optin) & allow_big_lds<float, PRO_NORM, EPI_SWIGLU>(optin) &
           allow_big_lds<float, PRO_NORM, EPI_HEAD>(optin) & allow_big_lds<float, PRO_PLAIN, EPI_RESID>(optin);
    }
    if (ok) g_lds_limit = (size_t)optin;
  }
  (void)hipGetLastError();
  return hipSuccess;
}

size_t linear_lds_limit() { return g_lds_limit; }

template void launch_linear<uint16_t>(const LinArgs&, int, int, int, hipStream_t, const LaunchEvents*);
template void launch_linear<float>(const LinArgs&, int, int, int, hipStream_t, const LaunchEvents*);

}  // namespace seedk
