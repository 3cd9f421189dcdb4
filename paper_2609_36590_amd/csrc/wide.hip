// Linear layers of passes of more than 64 rows (the prompts' prefill, the drafting objective's
// decoder pass): a compute-bound MFMA GEMM, Y[M, N] = X[M, K] W^T, with the epilogues (RoPE + paged
// K/V write, SwiGLU, logits) done in registers, and the residual projections' reduction.
#include "device_common.h"

#include <algorithm>

namespace seedk {

// ---------------------------------------------------------------------------------------------
// A workgroup of 4 waves owns 4*NI n-tiles (16 output features each) x MJ = 4 token tiles (16 rows):
// wave w accumulates n-tiles w*NI .. w*NI+NI-1 for all MJ token tiles; two workgroups share a CU, so
// that one computes while the other waits at its barrier. Both operands are stored as
// MFMA fragments (packed weights, packed activations), so nothing is converted or shuffled here:
//  * weights go from memory straight to registers: every fragment is used by one wave only, two
//    k-tiles ahead, each refilled as soon as its last MFMA has taken it;
//  * activations are used by all 4 waves: each fragment is fetched once per workgroup (two k-tiles
//    in flight in registers), written to one of two LDS slots, and read back one k-tile ahead into
//    the second of two register sets, so that the MFMAs of a k-tile wait for nothing issued in it.
// One barrier per k-tile. By count the matrix cores are the nearest limit: 16 cycles per MFMA against,
// per CU, 64 bytes of LDS per cycle at NI = 5 (of 128) and about 45 of vector memory (of 64). They are
// busy 55% of the time in gate/up, 40% in QKV, 44% in O and down, 58% in the LM head (MfmaUtil, 1024
// rows): the rest goes to a barrier per 40 MFMAs of a wave, the vector-memory path close behind, and
// the last round of workgroups. Measured (MI355X, 1024 rows, 4B shapes, passes in a row; the first
// pass after a pause takes 5-10% longer): gate/up 269 -> 167 us (1.23 PFLOP/s of MFMA work, counting
// both planes), QKV 122 -> 65, O and down 106 -> 63 (mean), the LM head with logits 2110 -> 1245 us,
// against a kernel that converted fp32 rows to operand pairs in every workgroup; a library bf16 GEMM
// of the gate/up shape runs at 1.04 PFLOP/s on the same card. Every output is one MFMA chain over its k-range, hi before lo in every
// k-tile; these passes write the prompt's cache and the objective's logits, which no decode pass has
// to reproduce bit for bit.
// Workgroup order: the token tiles of one n-group are consecutive workgroups of one XCD (workgroup
// w runs on XCD w mod 8), so that the n-group's weights come from HBM once and from that XCD's L2
// for its other token tiles; wider passes go through all n-groups for 1024 rows at a time, so that an
// XCD's 64 resident workgroups share activations too (4096 rows: gate/up 763 us with all 4096 rows of
// an n-group in a row, 734 in blocks of 1024, 739 of 512, 763 of 2048).
// ---------------------------------------------------------------------------------------------
constexpr int WIDE_MTB = 16;  // workgroups (1024 rows) of one n-group in a row

template <typename T, int EPI, int NI>
__global__ void __launch_bounds__(256, 2) k_linear_wide(LinArgs a) {
  constexpr int MJ = WIDE_MJ;
  constexpr int WN = 4 * NI;          // n-tiles per workgroup
  constexpr int XU = MJ / 2;          // fragments each wave fetches per k-tile (2 planes x MJ / 4 waves)
  constexpr int SLOT = 2 * MJ * 1024;   // bytes of one LDS slot (a k-tile's activations)
  constexpr int ACT_IMG = EPI == EPI_SWIGLU ? MJ * NI * ACT_TILE : 0;   // the workgroup's packed outputs
  __shared__ __attribute__((aligned(16))) char lds[2 * SLOT > ACT_IMG ? 2 * SLOT : ACT_IMG];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tl = lane & 15, kg = lane >> 4;
  const int KTF = a.K >> 5, n_tiles = a.N >> 4, m_tiles = (a.M + 15) >> 4;
  const int NG = (n_tiles + WN - 1) / WN, MT = (m_tiles + MJ - 1) / MJ;
  // K in S k-ranges (residual projections), each (n-group, k-range) pair a virtual n-group of its own
  const int S = EPI == EPI_RESID ? a.KS : 1;
  const int b = blockIdx.x, xcd = b & 7, r = b >> 3;
  const int MTB = min(MT, WIDE_MTB), per = (NG * S + 7) / 8 * MTB, mb = r / per, rb = r - mb * per;
  const int mt = mb * MTB + rb % MTB, gv = (rb / MTB) * 8 + xcd;
  if (gv >= NG * S || mt >= MT) return;   // padding of the grid to whole XCD rounds; the workgroup leaves together
  const int g = gv / S, ks = gv - g * S;
  const int kt0 = (ks * KTF) / S, KT = ((ks + 1) * KTF) / S - kt0;   // this workgroup's k-tiles

  // n-tiles past the last one re-read it and token tiles past the pass re-read its last one: neither
  // is stored
  const T* wp[NI];
  const int nt0 = g * WN + wave * NI;
#pragma unroll
  for (int i = 0; i < NI; ++i)
    wp[i] = reinterpret_cast<const T*>(a.W) + ((size_t)min(nt0 + i, n_tiles - 1) * KTF + kt0) * 512 + lane * 8;
  const char* xp[XU];
  char* xl[XU];
#pragma unroll
  for (int u = 0; u < XU; ++u) {
    const int f = u * 4 + wave;   // fragment: token tile f / 2, plane f % 2
    xp[u] = reinterpret_cast<const char*>(a.X) + ((size_t)min(mt * MJ + (f >> 1), m_tiles - 1) * KTF + kt0) * ACT_TILE +
            (f & 1) * 1024 + lane * 16;
    xl[u] = lds + f * 1024 + lane * 16;
  }
  typedef typename ET<T>::A WA;
  WA w0[NI], w1[NI];
  u32x4 x0[XU], x1[XU], b0[MJ][2], b1[MJ][2];
  f32x4 acc[NI][MJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < MJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // every load is unconditional (k-tiles past the range re-read its last one, never consumed): under
  // a data-dependent branch the compiler's wait counts assume the path without the load, and each
  // use would wait for everything in flight
  auto wload = [&](WA& w, int i, int t) __attribute__((always_inline)) {
    w = ET<T>::load(wp[i] + (size_t)min(t, KT - 1) * 512);
  };
  auto xload = [&](u32x4 (&x)[XU], int t) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < XU; ++u) x[u] = *reinterpret_cast<const u32x4*>(xp[u] + (size_t)min(t, KT - 1) * ACT_TILE);
  };
  auto xstore = [&](const u32x4 (&x)[XU], int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < XU; ++u) *reinterpret_cast<u32x4*>(xl[u] + slot * SLOT) = x[u];
  };
  auto bread = [&](u32x4 (&bf)[MJ][2], int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < MJ; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p)
        bf[j][p] = *reinterpret_cast<const u32x4*>(lds + slot * SLOT + (j * 2 + p) * 1024 + lane * 16);
  };
  // k-tile t: operands in w and bf; x holds k-tile t + 2's activations, slot p = t & 1 is free (every
  // wave read it before the last barrier) and slot p ^ 1 holds k-tile t + 1's
  auto step = [&](WA (&w)[NI], u32x4 (&x)[XU], const u32x4 (&bf)[MJ][2], u32x4 (&bn)[MJ][2], int p, int t)
                  __attribute__((always_inline)) {
    bread(bn, p ^ 1);
    xstore(x, p);
    xload(x, t + 4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < MJ; ++j) ET<T>::mma_plane(acc[i][j], w[i], bf[j][q], q);
      wload(w[i], i, t + 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  };

  xload(x0, 0);
  xload(x1, 1);
  xstore(x0, 0);
  xstore(x1, 1);
  // in the order the loop issues them: in another order, the compiler's wait counts for the loop's
  // first pass would hold every later pass to waiting for newer loads
  __builtin_amdgcn_sched_barrier(0);
  xload(x0, 2);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    wload(w0[i], i, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  xload(x1, 3);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    wload(w1[i], i, 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  bread(b0, 0);
  __syncthreads();
  int t = 0;
  for (; t + 1 < KT; t += 2) {
    step(w0, x0, b0, b1, 0, t);
    step(w1, x1, b1, b0, 1, t + 1);
  }
  if (t < KT) step(w0, x0, b0, b1, 0, t);

  // ---- epilogue: lane (tl, kg) holds features 4kg..4kg+3 of its n-tiles for row tl of its token
  // tiles. A QKV or gate/up tile pairs features c and c + 8 (rotary partners; gate and up), which
  // lane ^ 32 holds. ----
  const int hf = kg >> 1, c4 = (kg & 1) * 4;
#pragma unroll
  for (int j = 0; j < MJ; ++j) {
    const int row = (mt * MJ + j) * 16 + tl;
    const bool live = row < a.M;
    const int rowc = min(row, a.M - 1);
    if constexpr (EPI == EPI_RESID) {
      // the k-range's partial sums, [S][M][N]; k_wide_resid adds them
      float* pp = a.part + ((size_t)ks * a.M + rowc) * a.N + nt0 * 16 + 4 * kg;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        if (live && nt0 + i < n_tiles)
          *reinterpret_cast<float4*>(pp + i * 16) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    } else {
      const float rs = a.rs[rowc];
      float* lp = EPI == EPI_HEAD ? a.logits + (long long)rowc * a.ld_logits + nt0 * 16 + 4 * kg : nullptr;
      int pos = 0, blk = 0;
      if constexpr (EPI == EPI_QKV) {
        pos = a.row_slot[rowc];
        blk = a.row_blk[rowc];
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        float y[4], o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) y[q] = acc[i][j][q] * rs;
        const bool ok = live && nt0 + i < n_tiles;
        if constexpr (EPI == EPI_HEAD) {
          if (ok) {
            if (((uintptr_t)a.logits & 15) == 0) {   // rows are whole multiples of 16 floats
              *reinterpret_cast<float4*>(lp + i * 16) = make_float4(y[0], y[1], y[2], y[3]);
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) lp[i * 16 + q] = y[q];
            }
          }
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) o[q] = __shfl_xor(y[q], 32);
          if constexpr (EPI == EPI_SWIGLU) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float gv = hf ? o[q] : y[q], uv = hf ? y[q] : o[q];
              v[q] = gv / (1.f + __expf(-gv)) * uv;
            }
            // both lanes of a pair hold the 4 values: each writes one plane of them. The workgroup's
            // 32 NI features are NI whole k-tiles of the output, assembled in LDS and copied out below
            const int k = (wave * NI + i) * 8 + c4;
            ET<T>::put4_plane(lds + (j * NI + (k >> 5)) * ACT_TILE + act_slot(true, tl, (k >> 3) & 3), act_plane(true), k,
                              make_float4(v[0], v[1], v[2], v[3]), hf);
          } else {   // EPI_QKV
            const int HD = a.head_dim, half = HD >> 1;
            int sec, head, jt;
            qkv_tile(a, min((nt0 + i), n_tiles - 1), sec, head, jt);
            const int fi = 8 * jt + c4, d = hf * half + fi;
            if (sec < 2) {
              const float4 cs = *reinterpret_cast<const float4*>(a.row_rope + (size_t)rowc * HD + fi);
              const float4 sn = *reinterpret_cast<const float4*>(a.row_rope + (size_t)rowc * HD + half + fi);
              const float cv[4] = {cs.x, cs.y, cs.z, cs.w}, sv[4] = {sn.x, sn.y, sn.z, sn.w};
#pragma unroll
              for (int q = 0; q < 4; ++q) y[q] = hf ? y[q] * cv[q] + o[q] * sv[q] : y[q] * cv[q] - o[q] * sv[q];
            }
            if (ok) {
              if (sec == 0) {
                *reinterpret_cast<float4*>(a.q + (size_t)row * a.n_heads * HD + head * HD + d) =
                    make_float4(y[0], y[1], y[2], y[3]);
              } else {
                T* kvp = reinterpret_cast<T*>(a.kv);
                const size_t base = ((size_t)(a.layer * a.n_blocks + blk) * 2 + (sec - 1)) * a.n_kv + head;
                if (sec == 1) {
                  struct __attribute__((aligned(4 * sizeof(T)))) K4 {
                    T v[4];
                  };
                  K4 kv4;
#pragma unroll
                  for (int q = 0; q < 4; ++q) kv4.v[q] = ET<T>::from_f32(y[q]);
                  *reinterpret_cast<K4*>(kvp + base * 16 * HD + (pos & 15) * HD + d) = kv4;
                } else {
#pragma unroll
                  for (int q = 0; q < 4; ++q) kvp[base * HD * 16 + (d + q) * 16 + (pos & 15)] = ET<T>::from_f32(y[q]);
                }
              }
            }
          }
        }
      }
    }
  }
  if constexpr (EPI == EPI_SWIGLU) {
    __syncthreads();
    const int KTO = a.N >> 6;   // k-tiles of the output (N / 2 features)
    for (int t = wave; t < MJ * NI; t += 4) {
      const int m = mt * MJ + t / NI, kt = g * NI + t % NI;
      if (m < m_tiles && kt < KTO) {
        char* out = reinterpret_cast<char*>(a.act) + ((size_t)m * KTO + kt) * ACT_TILE + lane * 16;
        const char* img = lds + t * ACT_TILE + lane * 16;
        const u32x4 v0 = *reinterpret_cast<const u32x4*>(img), v1 = *reinterpret_cast<const u32x4*>(img + 1024);
        *reinterpret_cast<u32x4*>(out) = v0;
        *reinterpret_cast<u32x4*>(out + 1024) = v1;
      }
    }
  }
}

// Residual update of a wide pass: the k-range partials added in k-range order from 0, h += y, the
// packed x * gain of the next norm's consumer and that norm's row scale. A workgroup takes 4 whole rows (so
// that their sums of squares need no other kernel), each wave a quarter of the features, 16 lanes to a
// row (4 rows' slots side by side); the 4 workgroups of a token tile are on one XCD (their slots share
// lines). Bound by memory: 12 us for 1024 rows x 2560 (52 MB).
template <typename T>
__global__ void __launch_bounds__(256) k_wide_resid(LinArgs a) {
  __shared__ float s_ss[4][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int b = blockIdx.x, idx = b >> 3, rr = lane >> 4;
  const int m = ((idx >> 2) * 8 + (b & 7)) * 16 + (idx & 3) * 4 + rr, mc = min(m, a.M - 1);   // rows past the pass: never stored
  const int N = a.N, S = a.KS;
  const size_t stride = (size_t)a.M * N;
  const float* pp = a.part + (size_t)mc * N;
  float* hp = a.h + (size_t)mc * N;
  float ss = 0.f;
  constexpr int U = 5;   // 64-feature steps in flight
  const int steps = (N + 63) / 64, w0 = wave * steps / 4, w1 = (wave + 1) * steps / 4;
  for (int t0 = w0; t0 < w1; t0 += U) {
    float4 v[U][WIDE_SPLIT_MAX], hv[U], gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = min((t0 + u) * 64 + (lane & 15) * 4, N - 4);   // steps past the row re-read its end, never stored
#pragma unroll
      for (int k = 0; k < WIDE_SPLIT_MAX; ++k)
        if (k < S) v[u][k] = *reinterpret_cast<const float4*>(pp + k * stride + f);
      hv[u] = *reinterpret_cast<const float4*>(hp + f);
      gv[u] = *reinterpret_cast<const float4*>(a.gain_next + f);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = (t0 + u) * 64 + (lane & 15) * 4;
      float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < WIDE_SPLIT_MAX; ++k)
        if (k < S) y.x += v[u][k].x, y.y += v[u][k].y, y.z += v[u][k].z, y.w += v[u][k].w;
      const float4 h = make_float4(hv[u].x + y.x, hv[u].y + y.y, hv[u].z + y.z, hv[u].w + y.w);
      if (t0 + u < w1 && f < N && m < a.M) {
        *reinterpret_cast<float4*>(hp + f) = h;
        act_put4<T>(a.xg, N >> 5, true, m, f, make_float4(h.x * gv[u].x, h.y * gv[u].y, h.z * gv[u].z, h.w * gv[u].w));
        ss += (h.x * h.x + h.y * h.y) + (h.z * h.z + h.w * h.w);
      }
    }
  }
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
  if ((lane & 15) == 0) s_ss[wave][rr] = ss;
  __syncthreads();
  if (wave == 0 && (lane & 15) == 0 && m < a.M)
    a.rs_out[m] = rsqrtf((((s_ss[0][rr] + s_ss[1][rr]) + s_ss[2][rr]) + s_ss[3][rr]) / (float)N + a.eps);
}

// ---------------------------------------------------------------------------------------------
// Launchers (wide_split and wide_ni in dispatch.h).
// ---------------------------------------------------------------------------------------------
template <typename T, int EPI, int NI>
static void launch_wide_tile(const LinArgs& a, hipStream_t s, const LaunchEvents* ev) {
  const int n_tiles = a.N >> 4, m_tiles = (a.M + 15) >> 4;
  const int NG = (n_tiles + 4 * NI - 1) / (4 * NI), MT = (m_tiles + WIDE_MJ - 1) / WIDE_MJ, S = EPI == EPI_RESID ? a.KS : 1;
  const int MTB = std::min(MT, WIDE_MTB);
  launch(k_linear_wide<T, EPI, NI>, dim3((unsigned)((NG * S + 7) / 8 * 8 * MTB * ((MT + MTB - 1) / MTB))), dim3(256), 0,
         s, ev, a);
}

template <typename T, int EPI>
static void launch_wide_epi(const LinArgs& a, hipStream_t s, const LaunchEvents* ev) {
  if constexpr (sizeof(T) == 4) {   // fp32 operands take twice the registers
    launch_wide_tile<T, EPI, 2>(a, s, ev);
  } else {
    switch (wide_ni(a.N >> 4, a.M, EPI == EPI_RESID ? a.KS : 1)) {
      case 6: launch_wide_tile<T, EPI, 6>(a, s, ev); break;
      case 5: launch_wide_tile<T, EPI, 5>(a, s, ev); break;
      case 4: launch_wide_tile<T, EPI, 4>(a, s, ev); break;
      case 3: launch_wide_tile<T, EPI, 3>(a, s, ev); break;
      case 2: launch_wide_tile<T, EPI, 2>(a, s, ev); break;
      default: launch_wide_tile<T, EPI, 1>(a, s, ev); break;
    }
  }
}

template <typename T>
void launch_linear_wide(const LinArgs& a0, int epilogue, hipStream_t s, const LaunchEvents* ev) {
  LinArgs a = a0;
  switch (epilogue) {
    case EPI_QKV: launch_wide_epi<T, EPI_QKV>(a, s, ev); break;
    case EPI_SWIGLU: launch_wide_epi<T, EPI_SWIGLU>(a, s, ev); break;
    case EPI_HEAD: launch_wide_epi<T, EPI_HEAD>(a, s, ev); break;
    default: {
      a.KS = wide_split(a.N >> 4, a.K >> 5);
      const LaunchEvents e0{ev ? ev->start : nullptr, nullptr}, e1{nullptr, ev ? ev->stop : nullptr};
      launch_wide_epi<T, EPI_RESID>(a, s, ev ? &e0 : nullptr);
      const int m_tiles = (a.M + 15) >> 4;
      launch(k_wide_resid<T>, dim3((unsigned)((m_tiles + 7) / 8 * 32)), dim3(256), 0, s, ev ? &e1 : nullptr, a);
    }
  }
}

template void launch_linear_wide<uint16_t>(const LinArgs&, int, hipStream_t, const LaunchEvents*);
template void launch_linear_wide<float>(const LinArgs&, int, hipStream_t, const LaunchEvents*);

}  // namespace seedk
