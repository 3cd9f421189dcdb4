// The LM head (vocabulary-wide linear layer with RMSNorm, logits and argmax): weights streamed once, a
// wave per n-tile (16 tokens of the vocabulary) over all of K, activation rows staged in LDS as MFMA
// B-operand slots.
//
//  * k_head_lds      rows that fit LDS whole (M <= 16)
//  * k_head_chunked  up to 64 rows, staged in double-buffered chunks of K
//
// Both accumulate every logit as one MFMA chain in k order, so a row's logits are bit-identical however
// many rows share the pass: verifying d drafts gives the same logits, row by row, as plain greedy
// decoding (d = 0). Small vocabularies take the row kernel (rows.hip) for every row count instead.
#include "device_common.h"

#include <algorithm>

namespace seedk {

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

// A staged B-operand slot: 32 bytes of LDS holding one row's 8 values of k-group kg of k-tile kt
// (rest = kt * 4 + kg), the two 16-byte halves of the packed activation slot side by side.
struct Slot {
  uint4 p0, p1;
};
__device__ __forceinline__ Slot load_slot(const void* X, int KT, bool frag, int row, int rest) {
  const char* p = reinterpret_cast<const char*>(X) + ((size_t)(row >> 4) * KT + (rest >> 2)) * ACT_TILE +
                  act_slot(frag, row & 15, rest & 3);
  return Slot{*reinterpret_cast<const uint4*>(p), *reinterpret_cast<const uint4*>(p + act_plane(frag))};
}
__device__ __forceinline__ void store_slot(char* p, const Slot& v) {
  reinterpret_cast<uint4*>(p)[0] = v.p0;
  reinterpret_cast<uint4*>(p)[1] = v.p1;
}
template <typename T>
__device__ __forceinline__ typename ET<T>::B lds_slot(const char* p) {
  return ET<T>::join(reinterpret_cast<const uint4*>(p)[0], reinterpret_cast<const uint4*>(p)[1]);
}

__device__ inline size_t lds_x_bytes(int M, int nkt) { return (size_t)nkt * 4 * M * 32 + 32; }

// ---------------------------------------------------------------------------------------------
// M <= 16 rows (one MFMA tile): the workgroup (8 waves, one n-tile each) issues its first weight
// tiles, then stages the activation rows into LDS: slot (kt, kg, r) = 32 bytes, the two planes of
// x[r][32kt + 8kg .. +7], plus one zero slot for the token columns r >= M. Waves then stream weight
// tiles with P in flight, reading their B operands from LDS.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64 * HEAD_NT) k_head_lds(LinArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int P = 8;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int KT = a.K >> 5, n_tiles = a.N >> 4, M = a.M;
  const int tl = lane & 15, kg = lane >> 4;
  const int nt = blockIdx.x * HEAD_NT + wave;
  const int nk = nt < n_tiles ? KT : 0;   // weight tiles this wave streams
  const T* w0 = reinterpret_cast<const T*>(a.W) + (size_t)min(nt, n_tiles - 1) * KT * 512 + lane * 8;

  // ---- weight prefetch ----
  typename ET<T>::A wb[P];
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (p < nk) wb[p] = ET<T>::load_nt(w0 + (size_t)p * 512);
  float ssv[4] = {0.f, 0.f, 0.f, 0.f};
  const bool pre = preload_row_ssq(a, wave, ssv);

  // ---- stage X into LDS ----
  const size_t zero_off = (size_t)KT * 4 * M * 32;
  float* Y = reinterpret_cast<float*>(lds + lds_x_bytes(M, KT));   // [HEAD_NT][M][16], then the row scales
  float* s_rs = Y + (size_t)HEAD_NT * M * 16;
  {
    // two batches of 2 slots per thread per round trip: both batches' loads are issued before
    // either is written, so a workgroup whose rows take several batches (more than 3 rows of 2560)
    // pays half the round trips. Loads are branch-free (slots past the end reload
    // the last one and are not written) and none is issued after a wait: a load under a branch
    // makes the compiler wait for every load in flight before each write, and a surplus load
    // issued after the first wait would add a round trip to the one-batch case.
    const int items = KT * 4 * M, bs = 2 * (int)blockDim.x;
    Slot xa[2], xb[2];
    auto ld = [&](Slot (&xv)[2], int q0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = min(q0 + u * (int)blockDim.x + tid, items - 1);
        xv[u] = load_slot(a.X, KT, false, q % M, q / M);
      }
    };
    auto st = [&](const Slot (&xv)[2], int q0) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = q0 + u * (int)blockDim.x + tid;
        if (q < items) store_slot(lds + (size_t)q * 32, xv[u]);
      }
    };
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
    if (tid < 2) *reinterpret_cast<float4*>(lds + zero_off + tid * 16) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();

  // ---- stream ----
  const bool live_col = tl < M;
  const char* xa = lds + (live_col ? ((size_t)kg * M + tl) * 32 : zero_off);
  const size_t xs = live_col ? (size_t)4 * M * 32 : 0;  // bytes per k-tile
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto consume = [&](int slot, int j) { ET<T>::mma(acc, wb[slot], lds_slot<T>(xa + j * xs)); };
  int s0 = 0;
  for (; s0 + 2 * P <= nk; s0 += P) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      consume(p, s0 + p);
      wb[p] = ET<T>::load_nt(w0 + (size_t)(s0 + p + P) * 512);
      // keep each refill next to its consumption (the scheduler would otherwise sink all refills
      // below the last MFMA and drain the pipeline once per P tiles)
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

  // ---- RMSNorm row scales, epilogue ----
  for (int m = wave; m < M; m += HEAD_NT) {
    const float r = wave_row_scale(a, m, ssv, pre && m == wave);
    if (lane == 0) s_rs[m] = r;
  }
  __syncthreads();
  if (live_col) {
    const float rs = s_rs[tl];
    *reinterpret_cast<float4*>(Y + ((size_t)wave * M + tl) * 16 + 4 * kg) =
        make_float4(acc[0] * rs, acc[1] * rs, acc[2] * rs, acc[3] * rs);
  }
  __syncthreads();
  head_epilogue(a, blockIdx.x, HEAD_NT, Y, M * 16);
}

// ---------------------------------------------------------------------------------------------
// Up to 64 rows (batched verification, draft trees): the rows of all M tokens do not fit LDS whole, so they
// are staged in chunks of HEAD_CK k-tiles, double-buffered: the loads of chunk c+1 are issued before chunk
// c is consumed and written to the other buffer after it. The 8 waves of a workgroup take NT n-tiles
// each (8 NT neighbouring ones together), so that a staged fragment serves NT weight tiles and a
// vocabulary of 151936 makes one round of 238 workgroups; D k-tiles of weights are in flight. Every load
// is unconditional and clamped (surplus ones re-read the last k-tile and are never consumed): under a
// data-dependent branch the compiler's wait counts assume the path without it, and every refill would
// wait for the whole ring. Bound by the weight stream and the one barrier per chunk: 31 rows of the
// 28-layer shape (622 MB) 146 -> 120 us (5.2 TB/s) against 16 waves of one n-tile each, 594 workgroups in 2.3
// rounds; 8 k-tiles of weights in flight instead of 4 changed nothing (125 us).
// ---------------------------------------------------------------------------------------------
template <typename T, int TT, int NT, int D>
__global__ void __launch_bounds__(64 * HEAD_NT) k_head_chunked(LinArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ float s_rs[64];
  constexpr int NTH = 64 * HEAD_NT;
  constexpr int TILES = TT * HEAD_CK, CHUNK = TILES * ACT_TILE, XI = CHUNK / 16 / NTH;   // pieces per thread and chunk
  static_assert(HEAD_CK % D == 0 && CHUNK % (16 * NTH) == 0, "ring slots and pieces are static");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int KT = a.K >> 5, n_tiles = a.N >> 4, M = a.M, m_tiles = (M + 15) >> 4;
  const int tl = lane & 15, kg = lane >> 4;
  const int nt0 = blockIdx.x * NT * HEAD_NT + wave;   // this wave's n-tiles: nt0 + i * HEAD_NT
  const int NC = (KT + HEAD_CK - 1) / HEAD_CK;

  // ---- the rows' sums of squares: rows wave, wave + 8, .. ----
  float ssv[64 / HEAD_NT][4];
#pragma unroll
  for (int r = 0; r < 64 / HEAD_NT; ++r)
    if (r * HEAD_NT < M) preload_row_ssq(a, min(wave + r * HEAD_NT, M - 1), ssv[r]);
  __builtin_amdgcn_sched_barrier(0);

  // chunk c: tile (mt, ktl) at (mt * HEAD_CK + ktl) * ACT_TILE of its buffer
  u32x4 xv[XI];
  auto stage_load = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < XI; ++u) {
      const int o = (u * NTH + tid) * 16, tile = o / ACT_TILE;
      const int mt = min(tile / HEAD_CK, m_tiles - 1), kt = min(c * HEAD_CK + tile % HEAD_CK, KT - 1);
      xv[u] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.X) + ((size_t)mt * KT + kt) * ACT_TILE + o % ACT_TILE);
    }
  };
  auto stage_store = [&](int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < XI; ++u)
      *reinterpret_cast<u32x4*>(lds + (size_t)(c & 1) * CHUNK + (size_t)(u * NTH + tid) * 16) = xv[u];
  };
  const T* wp[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
    wp[i] = reinterpret_cast<const T*>(a.W) + (size_t)min(nt0 + i * HEAD_NT, n_tiles - 1) * KT * 512 + lane * 8;
  typename ET<T>::A w[D][NT];
  auto wload = [&](typename ET<T>::A (&wv)[NT], int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NT; ++i) wv[i] = ET<T>::load_nt(wp[i] + (size_t)min(kt, KT - 1) * 512);
    __builtin_amdgcn_sched_barrier(0);
  };
  stage_load(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < D; ++p) wload(w[p], p);
#pragma unroll
  for (int r = 0; r < 64 / HEAD_NT; ++r) {
    const int m = wave + r * HEAD_NT;
    if (r * HEAD_NT < M) {
      const float rs = wave_row_scale(a, min(m, M - 1), ssv[r], a.nssq <= 256);
      if (lane == 0 && m < M) s_rs[m] = rs;
    }
  }
  stage_store(0);
  __syncthreads();

  f32x4 acc[NT][TT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fo = act_slot(act_frag(M), tl, kg), fp = act_plane(act_frag(M));
  for (int c = 0; c < NC; ++c) {
    stage_load(c + 1);
    __builtin_amdgcn_sched_barrier(0);
    const char* buf = lds + (size_t)(c & 1) * CHUNK + fo;
    const int nkc = min(HEAD_CK, KT - c * HEAD_CK);
#pragma unroll
    for (int p = 0; p < HEAD_CK; ++p) {
      if (p < nkc) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          u32x4 xb[TT];
#pragma unroll
          for (int t = 0; t < TT; ++t)
            xb[t] = *reinterpret_cast<const u32x4*>(buf + (t * HEAD_CK + p) * ACT_TILE + q * fp);
#pragma unroll
          for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int t = 0; t < TT; ++t) ET<T>::mma_plane(acc[i][t], w[p % D][i], xb[t], q);
        }
      }
      wload(w[p % D], c * HEAD_CK + p + D);
    }
    stage_store(c + 1);
    __syncthreads();
  }

  // lane (tl, kg) holds features 4kg..4kg+3 of token t*16+tl: Y[wave][m][16] over the buffers, one of the
  // waves' NT n-tiles at a time (8 neighbouring n-tiles together)
  float* Y = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int m = t * 16 + tl;
      if (m < M) {
        const float rs = s_rs[m];
        *reinterpret_cast<float4*>(Y + ((size_t)wave * M + m) * 16 + 4 * kg) =
            make_float4(acc[i][t][0] * rs, acc[i][t][1] * rs, acc[i][t][2] * rs, acc[i][t][3] * rs);
      }
    }
    __syncthreads();
    const int g = blockIdx.x * NT + i;
    if (g * HEAD_NT < n_tiles) head_epilogue(a, g, HEAD_NT, Y, M * 16);
    __syncthreads();
  }
}

// Reduce per-n-group argmax partials of one row; lowest token id wins among equal maxima. One round trip for
// up to 2048 partials (151936 tokens make 1187): 8 clamped loads in flight per thread, then butterflies.
__global__ void __launch_bounds__(256) k_argmax_finalize(const float* val, const int* idx, int stride, int n_parts,
                                                         int* tok_out, int tok_stride, int* host_out, int host_stride) {
  constexpr int U = 8;
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ float s_v[4];
  __shared__ int s_i[4];
  float best = NEG_INF;
  int bi = -1;
  auto take = [&](float v, int i) {
    if (i >= 0 && (bi < 0 || v > best || (v == best && i < bi))) { best = v; bi = i; }
  };
  for (int j0 = 0; j0 < n_parts; j0 += U * 256) {
    float v[U];
    int i[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * 256 + tid, n_parts - 1);   // a partial taken twice changes nothing
      v[u] = val[(size_t)m * stride + j];
      i[u] = idx[(size_t)m * stride + j];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) take(v[u], i[u]);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float ov = __shfl_xor(best, o);
    const int oi = __shfl_xor(bi, o);
    take(ov, oi);
  }
  if (lane == 0) {
    s_v[wave] = best;
    s_i[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w) take(s_v[w], s_i[w]);
    const int tok = bi < 0 ? 0 : bi;
    tok_out[m * tok_stride] = tok;
    if (host_out) host_out[m * host_stride] = tok;
  }
}

// ---------------------------------------------------------------------------------------------
// Launchers (head_plan in dispatch.h).
// ---------------------------------------------------------------------------------------------
template <typename T, int TT>
static void launch_head_chunked(const LinArgs& a, const HeadPlan& p, hipStream_t s, const LaunchEvents* ev) {
  if constexpr (sizeof(T) == 2) {
    if (p.NT == 5) {
      launch(k_head_chunked<T, TT, 5, 4>, dim3(p.grid), dim3(64 * HEAD_NT), p.lds, s, ev, a);
      return;
    }
  }
  launch(k_head_chunked<T, TT, 1, 4>, dim3(p.grid), dim3(64 * HEAD_NT), p.lds, s, ev, a);
}

template <typename T>
static void launch_head(const LinArgs& a, hipStream_t s, const LaunchEvents* ev) {
  const HeadPlan p = head_plan(a.N, a.K, a.M, sizeof(T));
  if (!p.chunked) {
    launch(k_head_lds<T>, dim3(p.grid), dim3(64 * HEAD_NT), p.lds, s, ev, a);
    return;
  }
  switch ((a.M + 15) / 16) {
    case 1: launch_head_chunked<T, 1>(a, p, s, ev); break;
    case 2: launch_head_chunked<T, 2>(a, p, s, ev); break;
    case 3: launch_head_chunked<T, 3>(a, p, s, ev); break;
    default: launch_head_chunked<T, 4>(a, p, s, ev); break;
  }
}

template <typename T>
void launch_linear(const LinArgs& a, int epilogue, hipStream_t s, const LaunchEvents* ev) {
  if (a.M > 64) launch_linear_wide<T>(a, epilogue, s, ev);
  else if (epilogue == EPI_HEAD && !head_by_rows(a.N)) launch_head<T>(a, s, ev);
  else launch_linear_rows<T>(a, epilogue, s, ev);
}

void launch_argmax_finalize(const float* val, const int* idx, int stride, int n_parts, int M, int* tok_out,
                            int tok_stride, int* host_out, int host_stride, hipStream_t s) {
  hipLaunchKernelGGL(k_argmax_finalize, dim3(M), dim3(256), 0, s, val, idx, stride, n_parts, tok_out, tok_stride, host_out,
                     host_stride);
}

hipError_t check_device() {
  int dev = 0, lds = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  return (size_t)lds >= LDS_MAX ? hipSuccess : hipErrorInvalidDevice;
}

template void launch_linear<uint16_t>(const LinArgs&, int, hipStream_t, const LaunchEvents*);
template void launch_linear<float>(const LinArgs&, int, hipStream_t, const LaunchEvents*);

}  // namespace seedk
