// Linear layers of decode passes (at most 64 rows: draft steps, verification, draft trees): Y = X W^T
// streamed from memory once, with the epilogues (RoPE + paged K/V write, residual, SwiGLU) in the same
// launch.
#include "device_common.h"

#include <algorithm>

namespace seedk {

// The values an epilogue item needs besides its sums, loaded ahead of the weight stream for a thread's
// first item.
struct RowsPre {
  float4 a, b;     // EPI_RESID: residual and next-norm gain; EPI_QKV: RoPE cos and sin
  int pos, blk;    // EPI_QKV: cache slot and KV block of the row
};

// Item (lt, m, cq) of NT n-tiles x M rows: EPI_RESID features 4cq..4cq+3 (4 items per row), else features
// 4cq..4cq+3 and their partners 8 further (rotary pairs, gate and up; 2 items per row).
template <int EPI>
__device__ __forceinline__ void rows_item(int e, int M, int& lt, int& m, int& cq) {
  constexpr int Q = EPI == EPI_RESID || EPI == EPI_HEAD ? 4 : 2;
  cq = e % Q;
  const int r = e / Q;
  lt = r / M;
  m = r - lt * M;
}

template <int EPI>
__device__ __forceinline__ void rows_pre(const LinArgs& a, int nt, int m, int cq, RowsPre& p) {
  if constexpr (EPI == EPI_RESID) {
    p.a = *reinterpret_cast<const float4*>(a.h + (size_t)m * a.N + nt * 16 + 4 * cq);
    p.b = *reinterpret_cast<const float4*>(a.gain_next + nt * 16 + 4 * cq);
  } else if constexpr (EPI == EPI_QKV) {
    int sec, head, j;
    qkv_tile(a, nt, sec, head, j);
    p.pos = a.row_slot[m];   // the cache slot (the rotary position enters through row_rope)
    p.blk = a.row_blk[m];
    const float* rope = a.row_rope + (size_t)m * a.head_dim + 8 * j + 4 * cq;
    p.a = *reinterpret_cast<const float4*>(rope);
    p.b = *reinterpret_cast<const float4*>(rope + (a.head_dim >> 1));
  }
}

// h += y, the packed x * gain of the next norm's consumer, and the tile's share of its sum of squares
template <typename T>
__device__ __forceinline__ void rows_resid(const LinArgs& a, bool frag, int nt, int m, int cq, const float (&y)[4], const RowsPre& pre) {
  const float4 v = make_float4(pre.a.x + y[0], pre.a.y + y[1], pre.a.z + y[2], pre.a.w + y[3]);
  *reinterpret_cast<float4*>(a.h + (size_t)m * a.N + nt * 16 + 4 * cq) = v;
  act_put4<T>(a.xg, a.N >> 5, frag, m, nt * 16 + 4 * cq,
              make_float4(v.x * pre.b.x, v.y * pre.b.y, v.z * pre.b.z, v.w * pre.b.w));
  // the 4 items of a tile's row are neighbouring lanes of one wave in the same iteration
  float s = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  if (cq == 0) a.ssq_out[(size_t)m * (a.N >> 4) + nt] = s;
}

// ---------------------------------------------------------------------------------------------
// A workgroup owns NT n-tiles (16 output features each) for all of K; its KS waves (KS depends on the
// weight shape only) take a k-range each, for every n-tile and all TT token tiles of 16 rows. Both
// operands go from memory straight to registers, D k-tiles ahead: weights are used by one wave only, and
// a wave's k-range of the packed activations is its own too, so nothing is staged in LDS and no wave
// waits for another before its stream begins. Rows past the pass re-read its last row (never stored).
// The KS partial sums meet in LDS (PART: in memory, k_rows_reduce) and are added in k-range order from 0,
// so a row's output is bit-identical however many rows share the pass: verifying d drafts gives the same
// logits, row by row, as plain greedy decoding.
// Bound by the stream: HBM for a few rows (gate/up of the 4B shape, 99.6 MB, 17.9 us at 5 rows = 5.6 TB/s; QKV
// 31.5 MB 9.0, O 21 MB 8.2: start-up, the first burst and the sums are about 5 us of each), and the CU's
// vector memory once the rows' activations outweigh its weights. Measured against kernels that staged the
// rows in LDS first (and, from 17 rows or for long K, split K over workgroups with a reduction launch):
// at 5 rows gate/up 19.5 -> 17.9, QKV 10.9 -> 9.0, O 10.4 -> 8.2; at 40 rows gate/up 42.2 -> 23.3, QKV 22.7 ->
// 16.6, O 14.2 -> 14.5 in one launch, down 24.5 -> 19.1.
// ---------------------------------------------------------------------------------------------
template <typename T, int EPI, int NT, int TT, int D, int MAXT, bool PART>
__global__ void __launch_bounds__(MAXT) k_linear_rows(LinArgs a) {
  extern __shared__ __attribute__((aligned(16))) float part[];   // [NT][KS][M][16]
  __shared__ float s_rs[64];
  const int tid = threadIdx.x, lane = tid & 63, ks = (tid >> 6) + (PART ? blockIdx.y * (blockDim.x >> 6) : 0);
  const int tl = lane & 15, kg = lane >> 4;
  const int M = a.M, KS = a.KS, KT = a.K >> 5, n_tiles = a.N >> 4;
  const int nt0 = blockIdx.x * NT, nts = min(NT, n_tiles - nt0);
  const int ksc = PART ? min(ks, KS - 1) : ks;   // (a last workgroup's surplus wave repeats the last range)
  const int kt0 = (ksc * KT) / KS, nk = ((ksc + 1) * KT) / KS - kt0;

  // ---- RMSNorm row scales: rows ks, ks + KS, ..; their sums of squares are requested first ----
  constexpr int RR = 2;   // rows in flight per wave
  float ssv[RR][4];
  auto ssload = [&](int m0) {
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = lane + 64 * i;
        ssv[r][i] = a.ssq[(size_t)min(m0 + r * KS, M - 1) * a.nssq + min(j, a.nssq - 1)];
      }
  };
  if constexpr (EPI != EPI_RESID) ssload(ks);
  __builtin_amdgcn_sched_barrier(0);

  // ---- the stream ----
  typedef typename ET<T>::A WA;
  const T* wp[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
    wp[i] = reinterpret_cast<const T*>(a.W) + ((size_t)min(nt0 + i, n_tiles - 1) * KT + kt0) * 512 + lane * 8;
  const char* xp[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const int row = min(t * 16 + tl, M - 1);
    xp[t] = reinterpret_cast<const char*>(a.X) + ((size_t)(row >> 4) * KT + kt0) * ACT_TILE + act_slot(TT > 1, row & 15, kg);
  }
  WA w[D][NT];
  u32x4 x[D][TT][2];
  f32x4 acc[NT][TT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto issue = [&](WA (&wv)[NT], u32x4 (&xv)[TT][2], int j) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int p = 0; p < 2; ++p)
        xv[t][p] = *reinterpret_cast<const u32x4*>(xp[t] + (size_t)j * ACT_TILE + p * act_plane(TT > 1));
#pragma unroll
    for (int i = 0; i < NT; ++i) wv[i] = ET<T>::load_nt(wp[i] + (size_t)j * 512);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto consume = [&](const WA (&wv)[NT], const u32x4 (&xv)[TT][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int t = 0; t < TT; ++t) ET<T>::mma_plane(acc[i][t], wv[i], xv[t][p], p);
  };
#pragma unroll
  for (int p = 0; p < D; ++p) issue(w[p], x[p], min(p, nk - 1));   // surplus slots re-read the last k-tile, never consumed

  RowsPre pre{};
  if constexpr (!PART) {
    int lt, m, cq;
    rows_item<EPI>(tid, M, lt, m, cq);
    if (lt < nts) rows_pre<EPI>(a, nt0 + lt, m, cq, pre);
  }
  if constexpr (EPI != EPI_RESID) {
    for (int m0 = ks; m0 < M; m0 += RR * KS) {
      if (m0 != ks) ssload(m0);
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        float s = 0.f;
        if (a.nssq <= 256) {
#pragma unroll
          for (int i = 0; i < 4; ++i) s += lane + 64 * i < a.nssq ? ssv[r][i] : 0.f;
        } else {
          for (int j = lane; j < a.nssq; j += 64) s += a.ssq[(size_t)min(m0 + r * KS, M - 1) * a.nssq + j];
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
        const int m = m0 + r * KS;
        if (lane == 0 && m < M) s_rs[m] = rsqrtf(s / (float)a.K + a.eps);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  int b = 0;
  for (; b + 2 * D <= nk; b += D) {   // every refill is a k-tile of the range
#pragma unroll
    for (int p = 0; p < D; ++p) {
      consume(w[p], x[p]);
      issue(w[p], x[p], b + p + D);
    }
  }
#pragma unroll
  for (int p = 0; p < D; ++p)
    if (b + p < nk) {
      consume(w[p], x[p]);
      if (b + p + D < nk) issue(w[p], x[p], b + p + D);
    }
#pragma unroll
  for (int p = 0; p < D; ++p)
    if (b + D + p < nk) consume(w[p], x[p]);

  // ---- partial sums, lane (tl, kg): features 4kg..4kg+3 of row t*16 + tl ----
  if constexpr (PART) {   // to memory, [KS][M][N]: k_rows_reduce adds them and runs the epilogue
    if (ks >= KS) return;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int m = t * 16 + tl;
      float* pp = a.part + ((size_t)ks * M + m) * a.N + nt0 * 16 + 4 * kg;
#pragma unroll
      for (int i = 0; i < NT; ++i)
        if (m < M && i < nts) *reinterpret_cast<float4*>(pp + i * 16) = make_float4(acc[i][t][0], acc[i][t][1], acc[i][t][2], acc[i][t][3]);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      const int m = t * 16 + tl;
      if (m < M)
        *reinterpret_cast<float4*>(part + ((size_t)(i * KS + ks) * M + m) * 16 + 4 * kg) =
            make_float4(acc[i][t][0], acc[i][t][1], acc[i][t][2], acc[i][t][3]);
    }
  __syncthreads();

  // ---- sums over the k-ranges and the epilogue ----
  constexpr int Q = EPI == EPI_RESID || EPI == EPI_HEAD ? 4 : 2;
  const size_t stride = (size_t)M * 16;
  for (int e = tid; e < nts * M * Q; e += blockDim.x) {
    int lt, m, cq;
    rows_item<EPI>(e, M, lt, m, cq);
    const int nt = nt0 + lt;
    if (e != tid) rows_pre<EPI>(a, nt, m, cq, pre);
    float* pp = part + ((size_t)lt * KS * M + m) * 16 + 4 * cq;
    float y[4] = {0.f, 0.f, 0.f, 0.f}, z[4] = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < KS; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(pp + k * stride);
      y[0] += v.x; y[1] += v.y; y[2] += v.z; y[3] += v.w;
      if constexpr (Q == 2) {
        const float4 u = *reinterpret_cast<const float4*>(pp + k * stride + 8);
        z[0] += u.x; z[1] += u.y; z[2] += u.z; z[3] += u.w;
      }
    }
    if constexpr (EPI == EPI_RESID) {
      rows_resid<T>(a, TT > 1, nt, m, cq, y, pre);
    } else {
      const float rs = s_rs[m];
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] *= rs, z[q] *= rs;
      if constexpr (EPI == EPI_HEAD) {   // back to the item's first partial
        *reinterpret_cast<float4*>(pp) = make_float4(y[0], y[1], y[2], y[3]);
      } else if constexpr (EPI == EPI_SWIGLU) {
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = y[q] / (1.f + __expf(-y[q])) * z[q];
        act_put4<T>(a.act, a.N >> 6, TT > 1, m, nt * 8 + 4 * cq, make_float4(v[0], v[1], v[2], v[3]));
      } else {   // EPI_QKV
        const int HD = a.head_dim, half = HD >> 1;
        int sec, head, j;
        qkv_tile(a, nt, sec, head, j);
        const int d = 8 * j + 4 * cq;
        if (sec < 2) {
          const float cs[4] = {pre.a.x, pre.a.y, pre.a.z, pre.a.w}, sn[4] = {pre.b.x, pre.b.y, pre.b.z, pre.b.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float y0 = y[q], z0 = z[q];
            y[q] = y0 * cs[q] - z0 * sn[q];
            z[q] = z0 * cs[q] + y0 * sn[q];
          }
        }
        if (sec == 0) {
          float* qp = a.q + (size_t)m * a.n_heads * HD + head * HD + d;
          *reinterpret_cast<float4*>(qp) = make_float4(y[0], y[1], y[2], y[3]);
          *reinterpret_cast<float4*>(qp + half) = make_float4(z[0], z[1], z[2], z[3]);
        } else {
          T* kvp = reinterpret_cast<T*>(a.kv);
          const size_t base = ((size_t)(a.layer * a.n_blocks + pre.blk) * 2 + (sec - 1)) * a.n_kv + head;
          const int s = pre.pos & 15;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (sec == 1) {
              kvp[base * 16 * HD + s * HD + d + q] = ET<T>::from_f32(y[q]);
              kvp[base * 16 * HD + s * HD + half + d + q] = ET<T>::from_f32(z[q]);
            } else {
              kvp[base * HD * 16 + (d + q) * 16 + s] = ET<T>::from_f32(y[q]);
              kvp[base * HD * 16 + (half + d + q) * 16 + s] = ET<T>::from_f32(z[q]);
            }
          }
        }
      }
    }
  }
  if constexpr (EPI == EPI_HEAD) {
    __syncthreads();
    head_epilogue(a, blockIdx.x, NT, part, KS * M * 16);
  }
}

// The partials of a residual projection whose k-ranges went to different workgroups, added in k-range order
// from 0, and the epilogue: a thread per 4 outputs, all its loads in flight at once.
template <typename T>
__global__ void __launch_bounds__(256) k_rows_reduce(LinArgs a) {
  const int e = blockIdx.x * 256 + threadIdx.x, M = a.M, n_tiles = a.N >> 4;
  const int cq = e & 3, r = e >> 2, m = r % M, nt = r / M;
  if (nt >= n_tiles) return;   // the 4 lanes of a tile's row leave together
  RowsPre pre;
  rows_pre<EPI_RESID>(a, nt, m, cq, pre);
  const float* pp = a.part + (size_t)m * a.N + nt * 16 + 4 * cq;
  const size_t stride = (size_t)M * a.N;
  float4 v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (k < a.KS) v[k] = *reinterpret_cast<const float4*>(pp + k * stride);
  float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (k < a.KS) y[0] += v[k].x, y[1] += v[k].y, y[2] += v[k].z, y[3] += v[k].w;
  rows_resid<T>(a, act_frag(M), nt, m, cq, y, pre);
}

// ---------------------------------------------------------------------------------------------
// Launchers (rows_plan in dispatch.h).
// ---------------------------------------------------------------------------------------------
// k-tiles in flight per wave: what 256 registers (8 waves per CU) leave beside the sums
static constexpr int rows_depth(int NT, int TT) {
  return NT == 5 ? (TT == 1 ? 5 : TT == 2 ? 4 : 3) : NT == 3 ? (TT <= 2 ? 5 : 3) : NT == 2 && TT == 4 ? 4 : 5;
}

template <typename T, int EPI, int NT, int TT, int D>
static void launch_rows(const LinArgs& a, const RowsPlan& p, hipStream_t s, const LaunchEvents* ev) {
  launch(k_linear_rows<T, EPI, NT, TT, D, ROWS_THREADS, false>, dim3(p.gx), dim3(p.threads), p.lds, s, ev, a);
}

template <typename T, int NT, int TT, int D>
static void launch_rows_part(const LinArgs& a, const RowsPlan& p, hipStream_t s, const LaunchEvents* ev) {
  const LaunchEvents e0{ev ? ev->start : nullptr, nullptr}, e1{nullptr, ev ? ev->stop : nullptr};
  launch(k_linear_rows<T, EPI_RESID, NT, TT, D, ROWS_PART_THREADS, true>, dim3(p.gx, p.gy), dim3(p.threads), 0, s,
         ev ? &e0 : nullptr, a);
  launch(k_rows_reduce<T>, dim3((unsigned)(((a.N >> 4) * a.M * 4 + 255) / 256)), dim3(256), 0, s, ev ? &e1 : nullptr, a);
}

template <typename T, int EPI, int TT>
static void launch_rows_tt(const LinArgs& a, const RowsPlan& p, hipStream_t s, const LaunchEvents* ev) {
  if constexpr (EPI == EPI_RESID) {
    if (p.part) {
      if constexpr (sizeof(T) == 4) launch_rows_part<T, 2, TT, 2>(a, p, s, ev);
      else if (p.NT == 5) launch_rows_part<T, 5, TT, TT == 1 ? 8 : TT == 4 ? 5 : 6>(a, p, s, ev);
      else launch_rows_part<T, 2, TT, TT == 1 ? 10 : 6>(a, p, s, ev);
      return;
    }
  }
  if constexpr (EPI == EPI_HEAD) {
    launch_rows<T, EPI, ROWS_HEAD_NT, TT, sizeof(T) == 4 ? 2 : rows_depth(ROWS_HEAD_NT, TT)>(a, p, s, ev);
  } else if constexpr (sizeof(T) == 4) {
    launch_rows<T, EPI, 1, TT, 2>(a, p, s, ev);
  } else {
    const bool by8 = (a.K >> 5) % (8 * a.KS) == 0;   // ranges of whole 8-tile blocks: 8 in flight, no remainder
    switch (p.NT) {
      case 5:
        if constexpr (TT <= 3) launch_rows<T, EPI, 5, TT, rows_depth(5, TT)>(a, p, s, ev);
        break;
      case 3: launch_rows<T, EPI, 3, TT, rows_depth(3, TT)>(a, p, s, ev); break;
      case 2:
        if (TT == 1 && by8) launch_rows<T, EPI, 2, TT, TT == 1 ? 8 : rows_depth(2, TT)>(a, p, s, ev);
        else launch_rows<T, EPI, 2, TT, rows_depth(2, TT)>(a, p, s, ev);
        break;
      default:
        if (TT <= 2 && by8) launch_rows<T, EPI, 1, TT, TT <= 2 ? 8 : rows_depth(1, TT)>(a, p, s, ev);
        else launch_rows<T, EPI, 1, TT, rows_depth(1, TT)>(a, p, s, ev);
    }
  }
}

template <typename T, int EPI>
static void launch_rows_epi(LinArgs a, hipStream_t s, const LaunchEvents* ev) {
  const RowsPlan p = rows_plan(a.N, a.K, a.M, EPI, sizeof(T));
  a.KS = p.KS;
  switch ((a.M + 15) / 16) {
    case 1: launch_rows_tt<T, EPI, 1>(a, p, s, ev); break;
    case 2: launch_rows_tt<T, EPI, 2>(a, p, s, ev); break;
    case 3: launch_rows_tt<T, EPI, 3>(a, p, s, ev); break;
    default: launch_rows_tt<T, EPI, 4>(a, p, s, ev); break;
  }
}

template <typename T>
void launch_linear_rows(const LinArgs& a, int epilogue, hipStream_t s, const LaunchEvents* ev) {
  switch (epilogue) {
    case EPI_QKV: launch_rows_epi<T, EPI_QKV>(a, s, ev); break;
    case EPI_SWIGLU: launch_rows_epi<T, EPI_SWIGLU>(a, s, ev); break;
    case EPI_HEAD: launch_rows_epi<T, EPI_HEAD>(a, s, ev); break;
    default: launch_rows_epi<T, EPI_RESID>(a, s, ev); break;
  }
}

template void launch_linear_rows<uint16_t>(const LinArgs&, int, hipStream_t, const LaunchEvents*);
template void launch_linear_rows<float>(const LinArgs&, int, hipStream_t, const LaunchEvents*);

}  // namespace seedk
