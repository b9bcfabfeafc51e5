// Linear ops of the hybrid batch: one matmul over all C+B rows (Sec. 4.3,
// "fuse all the linear operations"), y = x W^T with W stored [N, K].
//
// bf16, K a multiple of 64 (every LLaMA / GPT-3 shape): gemm_ws_kernel, a
// block of producer waves that move both operands from global memory into an
// LDS ring with LDS DMA (global_load_lds_dwordx4) and consumer waves that run
// v_mfma_f32_16x16x32_bf16 on LDS-staged tiles (16-byte chunks XOR-swizzled
// by row so the operand reads are bank-conflict free).  Both operands are
// K-contiguous, so every lane moves 16 contiguous bytes.  Epilogues fuse the
// residual add (postproj, ffn_ln2), SiLU*mul (SwiGLU ffn_ln1) and GELU.
// Split-K stores one fp32 partial per split; a separate pass adds residual +
// partials in a fixed order, so results do not depend on scheduling.  Large
// batches: gemm_quad_kernel, tiles of up to 256 x 256.  fp32: gemm_ws_kernel on
// v_mfma_f32_16x16x4_f32.
//
// What bounds these: a CU keeps ~45 KB of loads in flight whatever the ring
// depth or the number of producers, and returns them in order, so operand rows
// that hit in L2 wait behind weight rows that come from HBM: ~30 bytes per
// clock and CU (64 when everything hits).  Under full matrix load the power
// limit holds the clock at 1.7-2.1 GHz, which slows that path too.
//
// bf16 with a ragged K, or operands of 4 GiB and more: gemm_bf16_kernel, tiles
// loaded through registers (k-chunks past K zeroed).  fp32 operands of 4 GiB
// and more: a plain LDS-tiled FMA kernel.
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace sarathi {

enum Epi { EPI_STORE = 0, EPI_GELU = 1, EPI_SWIGLU = 2, EPI_RESID_TO_F32 = 3, EPI_RESIDF32_TO_ACT = 4,
           EPI_PARTIAL = 5, EPI_ROPE_KV = 6 };

struct GemmP {
  const void* A;        // [M, K]
  const void* W;        // [N or 2N, K]
  int M, N, K;          // N = output columns (SwiGLU: F)
  int k_split, n_split; // K elements per split; number of splits
  int tiles_m, tiles_n, n_tiles;
  int rotate_k;         // gemm_ws_kernel: 0, or the distance (in k-tiles) by which the M-tiles of a W panel
                        // rotate their k-tile order
  void* out;            // [M, N]: dtype, or fp32 for EPI_RESID_TO_F32; EPI_PARTIAL: fp32 [n_split][M, N]
  const void* resid;    // EPI_RESID_TO_F32: dtype [M,N]; EPI_RESIDF32_TO_ACT: fp32 [M,N]
  int wide_blocks;      // gemm_quad_kernel with a tail: blocks of the wide tiles (a multiple of 8), then
  int tail_tiles, tail_n0;   // tail_tiles narrower tiles of the output columns from tail_n0
  int vec4, vec8;       // N a multiple of 4 / 8 and out, resid 16-byte aligned: wide stores
  RopeArgs rope;        // EPI_ROPE_KV: rotary embedding + KV append of the preproj output
};

// Output element handling shared by both kernels.
template <typename T, int EPI>
__device__ __forceinline__ void epi_store(const GemmP& p, int r, int c, float v, int split = 0) {
  const size_t idx = (size_t)r * p.N + c;
  if (EPI == EPI_STORE) {
    reinterpret_cast<T*>(p.out)[idx] = from_f<T>(v);
  } else if (EPI == EPI_GELU) {
    reinterpret_cast<T*>(p.out)[idx] = from_f<T>(gelu_f(v));
  } else if (EPI == EPI_RESID_TO_F32) {
    reinterpret_cast<float*>(p.out)[idx] = to_f<T>(reinterpret_cast<const T*>(p.resid)[idx]) + v;
  } else if (EPI == EPI_RESIDF32_TO_ACT) {
    reinterpret_cast<T*>(p.out)[idx] = from_f<T>(reinterpret_cast<const float*>(p.resid)[idx] + v);
  } else if (EPI == EPI_PARTIAL) {
    reinterpret_cast<float*>(p.out)[(size_t)split * p.M * p.N + idx] = v;
  }
}

// ============================================================================ bf16 MFMA, register-staged
// Block tile BM x BN (W rows) x 64, WGM x WGN waves, PD register stages of
// prefetch.  Loads are unconditional (addresses clamped into the operands) so
// the compiler can keep PD tiles in flight with partial vmcnt waits; rows and
// k-chunks outside the operands are zeroed when the registers are written to
// LDS.  The k-loop runs whole groups of U tiles (tiles past the end are zero
// and add nothing), keeping every register-stage index static.
__device__ __forceinline__ uint4 mask4(const uint4& v, bool ok) {
  return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

template <int BM, int BN, int WGM, int WGN, int PD, int EPI>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_kernel(GemmP p) {
  constexpr int NT = 64 * WGM * WGN;
  constexpr int BK = 64;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 16, FN = WTN / 16;
  constexpr int RPL = NT / 8;                  // rows covered by one 16-byte load per thread
  constexpr int AL = BM / RPL, BL = BN / RPL;
  constexpr int U = (PD % 2 == 0) ? PD : 2 * PD;
  static_assert(BM % RPL == 0 && BN % RPL == 0, "load split");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0 && (EPI != EPI_SWIGLU || FN % 2 == 0), "wave tile");
  extern __shared__ uint4 lds[];   // [2][(BM + BN) * 8] 16-byte chunks

  // XCD-aware order: block b runs on XCD b % 8.  Consecutive tiles (the
  // M-tiles that share a W panel) are given to blocks of one XCD so the panel
  // is fetched into that XCD's L2 once.
  const int per = gridDim.x / 8;
  const int t = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (t >= p.n_tiles) return;
  const int tile_m = t % p.tiles_m;
  const int rest = t / p.tiles_m;
  const int split = rest % p.n_split;
  const int tile_n = rest / p.n_split;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int m0 = tile_m * BM;
  const int n0_out = tile_n * (EPI == EPI_SWIGLU ? BN / 2 : BN);
  const int kbeg = split * p.k_split;
  const int kend = min(p.K, kbeg + p.k_split);
  const int nk = (kend - kbeg + BK - 1) / BK;

  const bf16* A = reinterpret_cast<const bf16*>(p.A);
  const bf16* W = reinterpret_cast<const bf16*>(p.W);
  const int lc = tid & 7, lr = tid >> 3;

  const bf16* a_src[AL];
  bool a_ok[AL];
#pragma unroll
  for (int i = 0; i < AL; ++i) {
    const int r = m0 + lr + RPL * i;
    a_ok[i] = r < p.M;
    a_src[i] = A + (size_t)(a_ok[i] ? r : 0) * p.K;
  }
  const bf16* b_src[BL];
  bool b_ok[BL];
#pragma unroll
  for (int i = 0; i < BL; ++i) {
    const int nl = lr + RPL * i;
    int wrow;
    if (EPI == EPI_SWIGLU) {
      // each wave's WTN columns: first half gate rows, second half up rows
      const int q = nl / WTN, w = nl % WTN, half = WTN / 2;
      const int j = n0_out + q * half + (w % half);
      b_ok[i] = j < p.N;
      wrow = (w < half) ? j : p.N + j;
    } else {
      wrow = n0_out + nl;
      b_ok[i] = wrow < p.N;
    }
    b_src[i] = W + (size_t)(b_ok[i] ? wrow : 0) * p.K;
  }

  uint4 R[PD][AL + BL];
  auto gload = [&](uint4* r, int kt) {
    const int kc = min(kt, nk - 1);
    const int kk = min(kbeg + kc * BK + lc * 8, p.K - 8);
#pragma unroll
    for (int i = 0; i < AL; ++i) r[i] = *reinterpret_cast<const uint4*>(a_src[i] + kk);
#pragma unroll
    for (int i = 0; i < BL; ++i) r[AL + i] = *reinterpret_cast<const uint4*>(b_src[i] + kk);
  };
  auto sstore = [&](int buf, const uint4* r, int kt) {
    uint4* s = lds + buf * (BM + BN) * 8;
    const bool kok = kbeg + kt * BK + lc * 8 < kend;
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      const int row = lr + RPL * i;
      s[row * 8 + (lc ^ (row & 7))] = mask4(r[i], a_ok[i] && kok);
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      const int row = BM + lr + RPL * i;
      s[row * 8 + (lc ^ (row & 7))] = mask4(r[AL + i], b_ok[i] && kok);
    }
  };

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int buf) {
    const uint4* s = lds + buf * (BM + BN) * 8;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int ch = ks * 4 + (lane >> 4);
      bf16x8_t af[FM], bfr[FN];
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        const int r = wm * WTM + fm * 16 + (lane & 15);
        af[fm] = __builtin_bit_cast(bf16x8_t, s[r * 8 + (ch ^ (r & 7))]);
      }
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const int r = BM + wn * WTN + fn * 16 + (lane & 15);
        bfr[fn] = __builtin_bit_cast(bf16x8_t, s[r * 8 + (ch ^ (r & 7))]);
      }
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
          acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[fm], bfr[fn], acc[fm][fn], 0, 0, 0);
    }
  };

  if (nk > 0) {
#pragma unroll
    for (int st = 0; st < PD; ++st) gload(R[st], st);
    sstore(0, R[0], 0);
    gload(R[0], PD);
    __syncthreads();
    for (int kb = 0; kb < nk; kb += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kt = kb + u;
        compute(u & 1);
        sstore((u + 1) & 1, R[(u + 1) % PD], kt + 1);
        gload(R[(u + 1) % PD], kt + 1 + PD);
        __syncthreads();
      }
    }
  }

  // Epilogue.  acc[fm][fn][i] = C[row 4*(lane/16)+i][col lane%16] of the 16x16 tile.
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = m0 + wm * WTM + fm * 16 + 4 * (lane >> 4) + i;
      if (r >= p.M) continue;
      if (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int fn = 0; fn < FN / 2; ++fn) {
          const int c = n0_out + wn * (WTN / 2) + fn * 16 + (lane & 15);
          if (c < p.N) {
            const float v = silu_f(acc[fm][fn][i]) * acc[fm][fn + FN / 2][i];
            reinterpret_cast<bf16*>(p.out)[(size_t)r * p.N + c] = f2bf(v);
          }
        }
      } else {
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int c = n0_out + wn * WTN + fn * 16 + (lane & 15);
          if (c < p.N) epi_store<bf16, EPI>(p, r, c, acc[fm][fn][i], split);
        }
      }
    }
  }
}

// ============================================================================ bf16 MFMA, producer/consumer waves
// The memory pipeline of a CU holds a bounded number of outstanding cache-line
// requests, and a wave that issues a load while it is full stalls at the
// issue.  When the same waves load and multiply, those stalls serialise the
// operand feed with the MFMAs.  Here NP producer waves only issue LDS DMA
// loads (and wait for them) while WGM x WGN consumer waves only read LDS and
// run MFMAs; one barrier per k-tile hands a filled stage to the consumers
// and the consumed stage back to the producers.  S-stage LDS ring, K a
// multiple of 64.
template <int EPI, int WTN>
__device__ __forceinline__ int w_row_of(int nl, int n0_out, int N) {
  if (EPI == EPI_SWIGLU) {
    // each consumer wave's WTN columns: first half gate rows, second half up rows
    const int q = nl / WTN, w = nl % WTN, half = WTN / 2;
    const int jj = n0_out + q * half + (w % half);
    return jj < N ? ((w < half) ? jj : N + jj) : 0;
  }
  return min(n0_out + nl, N - 1);
}

// Preproj with the rotary embedding and the KV append fused (the "others" of
// Sec. 2.1 that follow the QKV matmul).  The rotary pairs are (d, d + hd/2)
// of a head; so that any tile holds whole pairs, the producers load W's rows
// in pair order: within each head, logical columns 16g .. 16g+7 are physical
// columns 8g .. 8g+7 and logical 16g+8 .. 16g+15 are physical hd/2 + 8g ..
// hd/2 + 8g+7.  Every 16-column group of a tile is then 8 complete pairs of
// one head of q, k or v (hd a multiple of 16).
__device__ __forceinline__ int rope_w_row(int n, int N, int hd) {
  n = min(n, N - 1);
  const int c = n % hd;
  return n - c + ((c >> 3) & 1) * (hd / 2) + (c >> 4) * 8 + (c & 7);
}

// The epilogue: the block's tile goes to LDS in the output type (the rounding
// the separate kernel would read; 16-byte chunks XOR-swizzled by row); each thread
// then keeps one 16-column group (8 complete pairs of one head) and walks
// rows, four at a time so that their loads share a round trip: q is rotated
// into the output, k rotated and v copied into the KV cache at the row's
// (slot, position), 16 bytes per access, both halves of the pairs back at
// their physical columns.  The sines come from the call's rotary table.  The
// k and v columns of the output are not written (attention reads them from
// the cache).
template <int BN, int E = 8>                                // E elements per 16-byte chunk
__device__ __forceinline__ int tile_chunk(int r, int c) {   // 16-byte chunk c of tile row r
  constexpr int MASK = (BN / E) % 8 == 0 ? 7 : 3;          // the XOR stays within the row's chunks
  static_assert(BN / E % (MASK + 1) == 0, "chunks per row");
  return r * (BN / E) + (c ^ (r & MASK));
}

// Eight consecutive elements as fp32 <-> 16-byte chunks.
__device__ __forceinline__ void pack8(const float* f, uint4 (&v)[1]) {
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f2bf(f[2 * i]) | ((uint32_t)f2bf(f[2 * i + 1]) << 16);
  v[0] = make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ void pack8(const float* f, uint4 (&v)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
    v[i] = make_uint4(__float_as_uint(f[4 * i]), __float_as_uint(f[4 * i + 1]), __float_as_uint(f[4 * i + 2]),
                      __float_as_uint(f[4 * i + 3]));
}

template <typename T, int BM, int BN, int NT>
__device__ __forceinline__ void rope_kv_walk(const GemmP& p, int m0, int n0, int tid) {
  extern __shared__ uint4 lds[];
  constexpr int JG = BN / 16;                               // 16-column groups per tile row
  constexpr int RS = NT / JG;                               // rows in flight
  constexpr int U = 4;                                      // rows per round trip
  static_assert(RS > 0, "16-column groups");
  const int j = tid % JG, r0 = tid / JG;
  const int n = n0 + 16 * j;
  if (r0 >= RS || n >= p.N) return;
  const RopeArgs& a = p.rope;
  const int hd = a.hd, half = hd / 2, QD = a.nh * hd;
  const int part = n / QD, head = (n % QD) / hd;            // part 0 q, 1 k, 2 v
  const int d0 = (n % hd) / 2;                              // first pair of the group
  const bool rot = part < 2 && a.rope;
  constexpr int E = 16 / sizeof(T), NV = 8 / E;             // elements per chunk; chunks per half group
  T* cache = reinterpret_cast<T*>(a.kv_layer);
  const size_t kv_off = (part == 2 ? a.st.kv : 0) + (size_t)head * a.st.head;
  const int rows = min(BM, p.M - m0);
  for (int rb = r0; rb < rows; rb += U * RS) {
    int slot[U], pos[U];
    float4 cs[U][4];                                        // (cos, sin) of two pairs each
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = m0 + min(rb + u * RS, rows - 1);
      slot[u] = a.row_slot[row];
      pos[u] = a.row_pos[row];
      if (rot) {
        const float4* tab = reinterpret_cast<const float4*>(a.table + row * a.table_stride + d0);
#pragma unroll
        for (int i = 0; i < 4; ++i) cs[u][i] = tab[i];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = rb + u * RS;
      if (r >= rows) break;
      uint4 lo[NV], hi[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        lo[i] = lds[tile_chunk<BN, E>(r, 2 * NV * j + i)];
        hi[i] = lds[tile_chunk<BN, E>(r, 2 * NV * j + NV + i)];
      }
      if (rot) {
        float x0[8], x1[8], y0[8], y1[8];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          Vec16<T>::unpack(lo[i], x0 + E * i);
          Vec16<T>::unpack(hi[i], x1 + E * i);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float c = e & 1 ? cs[u][e / 2].z : cs[u][e / 2].x, sn = e & 1 ? cs[u][e / 2].w : cs[u][e / 2].y;
          y0[e] = x0[e] * c - x1[e] * sn;
          y1[e] = x0[e] * sn + x1[e] * c;
        }
        pack8(y0, lo);
        pack8(y1, hi);
      }
      T* dst = part == 0 ? reinterpret_cast<T*>(p.out) + (size_t)(m0 + r) * p.N + (n - n % hd)
                         : cache + (size_t)slot[u] * a.st.slot + kv_off + (size_t)pos[u] * a.st.pos;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        *reinterpret_cast<uint4*>(dst + d0 + E * i) = lo[i];
        *reinterpret_cast<uint4*>(dst + half + d0 + E * i) = hi[i];
      }
    }
  }
}

//
// fp32 (T = float): the same tiles of 128-byte k-rows (32 floats), products on
// v_mfma_f32_16x16x4_f32 (full fp32 inputs and sums).  A lane's 16-byte chunk
// holds four consecutive k of its row; product j of a chunk takes element j
// of every lane, so each 16x16x4 product sums k = {j, 4 + j, 8 + j, 12 + j} of
// a 16-wide step for both operands alike.  K need only be a multiple of 4:
// the last k-tile's chunks past K are read from the row's last chunk and
// zeroed in registers.  Bound by the fp32 matrix rate (157 TFLOP/s), 8x the
// time per operand byte of bf16.
//
// STREAM: W is loaded non-temporally (read once: one M-tile).  A template
// argument and not a run-time choice: with both producer loops in one kernel
// the 224-wide tiles (22 or 24 requests per wave and k-tile) spill 17-49
// scalar registers, in launches that never stream too.
template <typename T, int BM, int BN, int WGM, int WGN, int NP, int S, int EPI, bool STREAM>
__global__ __launch_bounds__(64 * (WGM * WGN + NP)) void gemm_ws_kernel(GemmP p) {
  constexpr int NC = WGM * WGN;
  constexpr int ES = sizeof(T);
  constexpr int BK = 128 / ES;
  constexpr bool F32 = ES == 4;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int FM = WTM / 16, FN = WTN / 16;
  constexpr int ROWS = BM + BN;
  constexpr int G = ROWS / 8, GA = BM / 8;
  constexpr int IHI = (G + NP - 1) / NP, ILO = G / NP, RHI = G % NP;
  static_assert(BM % 8 == 0 && BN % 8 == 0 && ILO > 0, "8-row groups");
  static_assert(WTM % 16 == 0 && WTN % 16 == 0 && (EPI != EPI_SWIGLU || FN % 2 == 0), "wave tile");
  static_assert((S - 2) * IHI < 64 && S >= 2, "stages");
  static_assert(EPI != EPI_ROPE_KV || BM * BN * ES <= S * ROWS * 128, "the RoPE epilogue stages the tile in the ring's LDS");
  extern __shared__ uint4 lds[];                 // [S][ROWS * 8] 16-byte chunks

  const int per = gridDim.x / 8;
  const int t = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (t >= p.n_tiles) return;
  const int tile_m = t % p.tiles_m;
  const int rest = t / p.tiles_m;
  const int split = rest % p.n_split;
  const int tile_n = rest / p.n_split;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = tile_m * BM;
  const int n0_out = tile_n * (EPI == EPI_SWIGLU ? BN / 2 : BN);
  const int kbeg = split * p.k_split;
  const int kend = min(p.K, kbeg + p.k_split);
  const int nk = (kend - kbeg + BK - 1) / BK;    // bf16: whole k-tiles; fp32: the last may be short

  if (wave >= NC) {
    // ---------------- producer
    // The wave index is uniform: the LDS destinations (m0) and the matrix
    // bases are scalar, and each lane keeps one 32-bit byte offset per row
    // group, so a request costs no vector instruction (global_load_lds with
    // a scalar base; the launcher keeps both matrices below 4 GiB).
    const int q = __builtin_amdgcn_readfirstlane(wave - NC);
    const char* A = reinterpret_cast<const char*>(p.A) + (size_t)kbeg * ES;
    const char* W = reinterpret_cast<const char*>(p.W) + (size_t)kbeg * ES;
    const int lchunk = (lane & 7) ^ (lane >> 3);
    uint32_t off[IHI];
#pragma unroll
    for (int j = 0; j < IHI; ++j) {
      const int g = min(j * NP + q, G - 1);
      const int row = g * 8 + (lane >> 3);
      const int nl = row - BM;
      const size_t r = g < GA                  ? (size_t)min(m0 + row, p.M - 1)
                       : EPI == EPI_ROPE_KV ? (size_t)rope_w_row(n0_out + nl, p.N, p.rope.hd)
                                            : (size_t)w_row_of<EPI, WTN>(nl, n0_out, p.N);
      off[j] = (uint32_t)(r * p.K * ES + lchunk * 16);
    }
    const bool extra = q < RHI;
    // With rotate_k, the G = tiles_m blocks that share a W panel take each
    // group of G k-tiles in rotated orders (block m starts at m), so every
    // k-tile of the panel is first requested by one block -- which pays the
    // HBM latency -- and found in L2 by the others a step later, instead of
    // all G waiting on the same miss.
    const int G = p.rotate_k ? p.tiles_m : 1, RD = p.rotate_k, GR = G * RD;
    auto issue = [&](int stage, int kt) {
      if (G > 1) {
        const int base = kt / GR * GR;
        if (base + GR <= nk) kt = base + (kt - base + tile_m * RD) % GR;
      }
      uint4* dst = lds + stage * ROWS * 8;
      const char* a_k = A + (size_t)kt * BK * ES;
      const char* w_k = W + (size_t)kt * BK * ES;
      // fp32: a short last k-tile's lanes past K re-read their row's last chunk
      const uint32_t back =
          F32 && kbeg + (kt + 1) * BK > kend ? 16u * max(lchunk - ((kend - kbeg - kt * BK) / 4 - 1), 0) : 0u;
#pragma unroll
      for (int j = IHI - 1; j >= 0; --j)
        if (j < ILO || extra) {
          // the matrix is chosen on the scalar bases, before the lane's offset
          const bool is_a = min(j * NP + q, ROWS / 8 - 1) < GA;
          if (STREAM && !is_a) dma16_stream(w_k + (off[j] - back), dst + (j * NP + q) * 64);
          else dma16((is_a ? a_k : w_k) + (off[j] - back), dst + (j * NP + q) * 64);
        }
    };
    auto wait_next = [&](bool all) {   // all but the newest S - 2 stages landed
      if (all) wait_vmcnt<0>();
      else if (extra) wait_vmcnt<(S - 2) * IHI>();
      else wait_vmcnt<(S - 2) * ILO>();
    };
#pragma unroll
    for (int st = 0; st < S - 1; ++st)
      if (st < nk) issue(st, st);
    wait_next(S - 2 >= nk);
    lds_barrier();
    int nbuf = S - 1;
    for (int kt = 0; kt < nk; ++kt) {
      const bool more = kt + S - 1 < nk;
      if (more) issue(nbuf, kt + S - 1);
      wait_next(!more);
      lds_barrier();
      nbuf = (nbuf + 1 == S) ? 0 : nbuf + 1;
    }
    if constexpr (EPI == EPI_ROPE_KV) lds_barrier();   // pairs with the consumers' epilogue barrier
    return;
  }

  // ---------------- consumer
  const int wm = wave / WGN, wn = wave % WGN;
  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  lds_barrier();
  int buf = 0;
  if constexpr (F32) {
    // The fragments of the other half k-tile are read while this one's
    // products run (one consumer wave per SIMD: nothing else hides the reads).
    floatx4 af[2][FM], bfr[2][FN];
    auto read = [&](auto h, int at, int kt) {
      constexpr int HF = decltype(h)::value;
      const uint4* s = lds + at * ROWS * 8;
      const int ch = HF * 4 + (lane >> 4);
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        const int r = wm * WTM + fm * 16 + (lane & 15);
        af[HF][fm] = __builtin_bit_cast(floatx4, s[r * 8 + (ch ^ (r & 7))]);
      }
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const int r = BM + wn * WTN + fn * 16 + (lane & 15);
        bfr[HF][fn] = __builtin_bit_cast(floatx4, s[r * 8 + (ch ^ (r & 7))]);
      }
      if (kbeg + (kt + 1) * BK > kend && kbeg + kt * BK + ch * 4 >= kend) {   // chunks past K: both operands zero
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) af[HF][fm] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) bfr[HF][fn] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    };
    auto products = [&](auto h) {
      constexpr int HF = decltype(h)::value;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[HF][fm][j], bfr[HF][fn][j], acc[fm][fn], 0, 0, 0);
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    read(H0{}, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      read(H1{}, buf, kt);
      products(H0{});
      lds_read_barrier();
      buf = (buf + 1 == S) ? 0 : buf + 1;
      if (kt + 1 < nk) read(H0{}, buf, kt + 1);
      products(H1{});
    }
  } else {
    for (int kt = 0; kt < nk; ++kt) {
      const uint4* s = lds + buf * ROWS * 8;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int ch = ks * 4 + (lane >> 4);
        bf16x8_t af[FM], bfr[FN];
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
          const int r = wm * WTM + fm * 16 + (lane & 15);
          af[fm] = __builtin_bit_cast(bf16x8_t, s[r * 8 + (ch ^ (r & 7))]);
        }
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int r = BM + wn * WTN + fn * 16 + (lane & 15);
          bfr[fn] = __builtin_bit_cast(bf16x8_t, s[r * 8 + (ch ^ (r & 7))]);
        }
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
            acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[fm], bfr[fn], acc[fm][fn], 0, 0, 0);
      }
      lds_read_barrier();
      buf = (buf + 1 == S) ? 0 : buf + 1;
    }
  }

  if constexpr (EPI == EPI_ROPE_KV) {
    constexpr int E = 16 / ES;
    T* tile = reinterpret_cast<T*>(lds);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = wm * WTM + fm * 16 + 4 * (lane >> 4) + i;
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int c = wn * WTN + fn * 16 + (lane & 15);
          tile[tile_chunk<BN, E>(r, c / E) * E + c % E] = from_f<T>(acc[fm][fn][i]);
        }
      }
    lds_read_barrier();                  // the producers pass their last barrier too
    rope_kv_walk<T, BM, BN, 64 * NC>(p, m0, tile_n * BN, tid);
    return;
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = m0 + wm * WTM + fm * 16 + 4 * (lane >> 4) + i;
      if (r >= p.M) continue;
      if (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int fn = 0; fn < FN / 2; ++fn) {
          const int c = n0_out + wn * (WTN / 2) + fn * 16 + (lane & 15);
          if (c < p.N) {
            const float v = silu_f(acc[fm][fn][i]) * acc[fm][fn + FN / 2][i];
            reinterpret_cast<T*>(p.out)[(size_t)r * p.N + c] = from_f<T>(v);
          }
        }
      } else {
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
          const int c = n0_out + wn * WTN + fn * 16 + (lane & 15);
          if (c < p.N) epi_store<T, EPI>(p, r, c, acc[fm][fn][i], split);
        }
      }
    }
  }
}

// ============================================================================ bf16 MFMA, quadrant tiles
// Large batches (192 and 256 rows by 256 W rows per block, 288 by 192).  With
// operands resident the 256 x 256 loop is bound by the matrix cores and the
// chip's power (a probe: 97% of the matrix issue rate, at the ~1.8 GHz that the
// power limit leaves); in the layers the matrix cores are busy 44-57% of the
// cycles, 0.9-1.3 PFLOP/s (an 8192^3 library product: 1.24-1.34 on these
// cards).  What the smaller tiles lack is operand feed: a CU keeps ~45 KB
// of loads in flight, ~30 bytes per clock at HBM latency, and 160 x 256 needs
// 41 per matrix clock where 256 x 256 needs 32.
//
// 8 waves of WGM x WGN, no producers (the accumulators and two halves of each
// operand fill the 256 registers that two waves per SIMD leave).  A k-tile of
// 64 is two half stages: rows of every wave's first row half and column half
// (A0, B0), then the second halves (A1, B1), two stages in LDS.  The wave
// multiplies the quadrants A0B0, A0B1 | A1B1, A1B0, reading each half from LDS
// while the quadrant before it runs, so a half stage is free as soon as it is
// in registers: with one barrier per two quadrants its successor is requested
// 1.5 k-tiles ahead of its use (a plain two-stage ring, 0.75 ahead, ran 143 us
// where this runs 121 on 1024 x 15360 x 5120; 160 x 256 producer tiles 158).
//
// Hazards, for half stage (kt, h): requested after the barrier that follows
// the reads of (kt - 2, h) by every wave; read after every wave waited for its
// own requests (all but the newest two half stages) and passed a barrier.
// Requests past the last k-tile re-read it into stages that nothing reads.
//
// The products take W as the first operand, so a lane holds four consecutive
// columns of one row: 8- and 16-byte stores.
template <int N>
__device__ __forceinline__ void pin_regs(u32x4 (&r)[N]) {   // no use of r moves above this point
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(r[i]));
}
// LDS reads as inline assembly with the waits written out: the compiler would
// take them to overlap the half stages that LDS DMA fills and drain those.
template <int OFF>
__device__ __forceinline__ u32x4 lds_read16(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "i"(OFF));
  return v;
}
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Four consecutive columns c .. c + 3 of row r (residual kinds and partials).
template <int EPI>
__device__ __forceinline__ void epi_store4(const GemmP& p, int r, int c, const floatx4& v, int split) {
  if (p.vec4) {
    const size_t idx = (size_t)r * p.N + c;
    if (EPI == EPI_PARTIAL) {
      *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + (size_t)split * p.M * p.N + idx) = v;
    } else if (EPI == EPI_RESID_TO_F32) {
      const uint2 x = *reinterpret_cast<const uint2*>(reinterpret_cast<const bf16*>(p.resid) + idx);
      *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + idx) =
          floatx4{__uint_as_float(x.x << 16) + v[0], __uint_as_float(x.x & 0xffff0000u) + v[1],
                  __uint_as_float(x.y << 16) + v[2], __uint_as_float(x.y & 0xffff0000u) + v[3]};
    } else {
      const floatx4 x = *reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(p.resid) + idx) + v;
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16*>(p.out) + idx) =
          make_uint2((uint32_t)f2bf(x[0]) | ((uint32_t)f2bf(x[1]) << 16),
                     (uint32_t)f2bf(x[2]) | ((uint32_t)f2bf(x[3]) << 16));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (c + i < p.N) epi_store<bf16, EPI>(p, r, c + i, v[i], split);
  }
}

// One tile: output columns from n0_out.
template <int FM, int FN, int EPI>
__device__ __forceinline__ void quad_tile(const GemmP& p, int tile_m, int split, int n0_out) {
  constexpr int WGM = 2, WGN = 4, BM = WGM * FM * 16, BN = WGN * FN * 16, BK = 64;
  constexpr int WTM = FM * 16, WTN = FN * 16;
  constexpr int FM0 = (FM + 1) / 2, FM1 = FM / 2, FN0 = (FN + 1) / 2, FN1 = FN / 2;   // 16-row groups per half
  constexpr int AH0 = WGM * FM0 * 16, AH1 = WGM * FM1 * 16, BH0 = WGN * FN0 * 16, BH1 = WGN * FN1 * 16;   // rows
  constexpr int HG0 = (AH0 + BH0) / 8, HG1 = (AH1 + BH1) / 8;       // 1 KB requests (8 rows) per half stage
  constexpr int I0H = (HG0 + 7) / 8, I1H = (HG1 + 7) / 8;           // per wave: at most,
  constexpr int I0L = HG0 / 8, I1L = HG1 / 8;                       // and at least
  constexpr int Q00 = 2 * FM0 * FN0, Q11 = 2 * FM1 * FN1, Q10 = 2 * FM1 * FN0;   // products of the quadrants
  static_assert(FM1 > 0 && FN1 > 0, "two halves each way");
  static_assert(Q00 >= 2 * FN1 + 2 * FM1 && Q11 + Q10 >= 2 * FM0 + 2 * FN0 && Q10 >= 2 * FN0, "reads per phase");
  static_assert(Q00 / 2 >= I0H && (Q11 + Q10) / 2 >= I1H && I0H + 2 * I1H < 64, "requests per phase");
  static_assert(HG0 * 1024 + FM0 * 2048 < 65536, "immediate LDS offsets");
  // [stage][half][AH0 A rows, BH0 W rows][8] 16-byte chunks: a wave's rows start
  // at the same place in both halves (a smaller second half leaves gaps), so
  // one LDS address per operand and k-step serves both
  extern __shared__ uint4 lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int m0 = tile_m * BM;
  const int kbeg = split * p.k_split;
  const int kend = min(p.K, kbeg + p.k_split);
  const int nk = (kend - kbeg) / BK;

  // requests: as gemm_ws_kernel's producers (scalar bases, 32-bit row offsets)
  const char* A = reinterpret_cast<const char*>(p.A) + (size_t)kbeg * 2;
  const char* W = reinterpret_cast<const char*>(p.W) + (size_t)kbeg * 2;
  const int lchunk = (lane & 7) ^ (lane >> 3);
  // SwiGLU: every 16 W rows of the tile are 8 gate rows and their 8 up rows
  auto w_row = [&](int nl) -> size_t {
    if (EPI == EPI_ROPE_KV) return rope_w_row(n0_out + nl, p.N, p.rope.hd);
    if (EPI == EPI_SWIGLU) {
      const int j = min(n0_out + (nl >> 4) * 8 + (nl & 7), p.N - 1);
      return (nl & 8) ? p.N + j : j;
    }
    return min(n0_out + nl, p.N - 1);
  };
  auto offset = [&](int h, int j) -> uint32_t {
    const int ah = h ? AH1 : AH0, arow = (h ? FM1 : FM0) * 16, brow = (h ? FN1 : FN0) * 16;
    const int g = min(j * 8 + wave, (h ? HG1 : HG0) - 1), row = g * 8 + (lane >> 3);
    size_t r;
    if (g * 8 < ah) {
      r = (size_t)min(m0 + (row / arow) * WTM + (h ? FM0 * 16 : 0) + row % arow, p.M - 1);
    } else {
      const int q = row - ah;
      r = w_row((q / brow) * WTN + (h ? FN0 * 16 : 0) + q % brow);
    }
    return (uint32_t)(r * p.K * 2 + lchunk * 16);
  };
  uint32_t off0[I0H], off1[I1H];
#pragma unroll
  for (int j = 0; j < I0H; ++j) off0[j] = offset(0, j);
#pragma unroll
  for (int j = 0; j < I1H; ++j) off1[j] = offset(1, j);
  constexpr int HALF = HG0 * 64, STAGE = 2 * HALF;  // 16-byte chunks
  auto request0 = [&](int kt, int j) {
    const int g = j * 8 + wave;
    if (j < I0L || g < HG0)
      dma16((g * 8 < AH0 ? A : W) + (size_t)min(kt, nk - 1) * BK * 2 + off0[j], lds + (kt & 1) * STAGE + g * 64);
  };
  auto request1 = [&](int kt, int j) {
    const int g = j * 8 + wave, row = g * 8;
    const int at = row < AH1 ? (row / (FM1 * 16)) * (FM0 * 16) + row % (FM1 * 16)
                             : AH0 + ((row - AH1) / (FN1 * 16)) * (FN0 * 16) + (row - AH1) % (FN1 * 16);
    if (j < I1L || g < HG1)
      dma16((row < AH1 ? A : W) + (size_t)min(kt, nk - 1) * BK * 2 + off1[j],
            lds + (kt & 1) * STAGE + HALF + at * 8);
  };
  // this wave's requests but the newest half stage of each kind (EXTRA more half 1s) have landed
  const bool more0 = wave < HG0 % 8, more1 = wave < HG1 % 8;
  auto wait_but = [&](auto n1) {
    constexpr int N1 = decltype(n1)::value;
    if (more0) {
      if (more1) wait_vmcnt<I0L + 1 + N1 * (I1L + 1)>();
      else wait_vmcnt<I0L + 1 + N1 * I1L>();
    } else {
      if (more1) wait_vmcnt<I0L + N1 * (I1L + 1)>();
      else wait_vmcnt<I0L + N1 * I1L>();
    }
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using C2 = std::integral_constant<int, 2>;

  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const uint32_t l0 = (uint32_t)(uintptr_t)lds;
  const uint32_t ax = l0 + (wm * FM0 * 16 + (lane & 15)) * 128 + ((lane >> 4) ^ (lane & 7)) * 16;
  const uint32_t bx = ax + (AH0 + wn * FN0 * 16 - wm * FM0 * 16) * 128;
  // k-step 0 and 1 of a row (chunks 0-3 and 4-7: bit 6 of the swizzled address)
  const uint32_t a_at[2] = {ax, ax ^ 64u}, b_at[2] = {bx, bx ^ 64u};
  constexpr int HOFF = HALF * 16;
  u32x4 fa[2][2 * FM0], fb[2][2 * FN0];             // fragments of a half: [k-step][16-row group]
  auto read_a0 = [&](uint32_t st, auto f) {
    constexpr int F = decltype(f)::value;
    fa[0][F] = lds_read16<(F % FM0) * 2048>(a_at[F / FM0] + st);
  };
  auto read_a1 = [&](uint32_t st, auto f) {
    constexpr int F = decltype(f)::value;
    fa[1][F] = lds_read16<HOFF + (F % FM1) * 2048>(a_at[F / FM1] + st);
  };
  auto read_b0 = [&](u32x4 (&d)[2 * FN0], uint32_t st, auto f) {
    constexpr int F = decltype(f)::value;
    d[F] = lds_read16<(F % FN0) * 2048>(b_at[F / FN0] + st);
  };
  auto read_b1 = [&](u32x4 (&d)[2 * FN0], uint32_t st, auto f) {
    constexpr int F = decltype(f)::value;
    d[F] = lds_read16<HOFF + (F % FN1) * 2048>(b_at[F / FN1] + st);
  };
  // the products of quadrant (mh, nh), with act(i) issued after product i
  auto quadrant = [&](const u32x4* a, const u32x4* b, auto mh, auto nh, auto&& act) {
    constexpr int MH = decltype(mh)::value, NH = decltype(nh)::value;
    constexpr int QM = MH ? FM1 : FM0, QW = NH ? FN1 : FN0;
    static_for<0, 2 * QM * QW>([&](auto i) {
      constexpr int I = decltype(i)::value, ks = I / (QM * QW), r = I % (QM * QW), fm = r / QW, fn = r % QW;
      floatx4& c = acc[MH * FM0 + fm][NH * FN0 + fn];
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b[ks * QW + fn]),
                                                  __builtin_bit_cast(bf16x8_t, a[ks * QM + fm]), c, 0, 0, 0);
      act(i);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto lds_landed = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
    for (int j = 0; j < I0H; ++j) request0(kt, j);
#pragma unroll
    for (int j = 0; j < I1H; ++j) request1(kt, j);
  }
  wait_but(C2{});                                   // (0, 0); newest (0, 1), (1, 0), (1, 1)
  lds_barrier();
  static_for<0, 2 * FM0>([&](auto f) { read_a0(0, f); });
  static_for<0, 2 * FN0>([&](auto f) { read_b0(fb[0], 0, f); });
  lds_landed();
  pin_regs(fa[0]);
  pin_regs(fb[0]);

  // One k-tile.  A0 is in fa[0] and B0 in fb[P]; B1 is read into fb[1 - P],
  // A1 into fa[1], then the next tile's A0 into fa[0] and B0 into fb[1 - P].
  auto tile = [&](int kt, auto pc) {
    constexpr int P = decltype(pc)::value;
    const uint32_t cur = (uint32_t)(kt & 1) * (STAGE * 16), nxt = (uint32_t)((kt + 1) & 1) * (STAGE * 16);
    wait_but(C1{});                                 // (kt, 1); newest (kt + 1, 0), (kt + 1, 1)
    lds_barrier();
    __builtin_amdgcn_s_setprio(1);
    quadrant(fa[0], fb[P], C0{}, C0{}, [&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I < 2 * FN1) read_b1(fb[1 - P], cur, i);
      else if constexpr (I < 2 * FN1 + 2 * FM1) read_a1(cur, std::integral_constant<int, I - 2 * FN1>{});
      if constexpr (I % 2 == 1 && I / 2 < I0H) request0(kt + 2, I / 2);
    });
    lds_landed();
    pin_regs(fb[1 - P]);
    pin_regs(fa[1]);
    quadrant(fa[0], fb[1 - P], C0{}, C1{}, [](auto) {});
    __builtin_amdgcn_s_setprio(0);
    wait_but(C1{});                                 // (kt + 1, 0); newest (kt + 1, 1), (kt + 2, 0)
    lds_barrier();
    __builtin_amdgcn_s_setprio(1);
    quadrant(fa[1], fb[1 - P], C1{}, C1{}, [&](auto i) {
      constexpr int I = decltype(i)::value;
      if constexpr (I < 2 * FM0) read_a0(nxt, i);
      if constexpr (I % 2 == 1 && I / 2 < I1H) request1(kt + 2, I / 2);
    });
    // past the last tile the reads return stale values, which are not used
    quadrant(fa[1], fb[P], C1{}, C0{}, [&](auto i) {
      constexpr int I = decltype(i)::value, LEFT = 2 * FM0 > Q11 ? 2 * FM0 - Q11 : 0, J = Q11 + I;
      if constexpr (I < LEFT) read_a0(nxt, std::integral_constant<int, (I < LEFT ? Q11 + I : 0)>{});
      else if constexpr (I - LEFT < 2 * FN0) read_b0(fb[1 - P], nxt, std::integral_constant<int, I - LEFT>{});
      if constexpr (J % 2 == 1 && J / 2 < I1H) request1(kt + 2, J / 2);
    });
    __builtin_amdgcn_s_setprio(0);
    lds_landed();
    pin_regs(fa[0]);
    pin_regs(fb[1 - P]);
  };
  for (int kt = 0; kt < nk; kt += 2) {
    tile(kt, C0{});
    if (kt + 1 < nk) tile(kt + 1, C1{});
  }
  wait_vmcnt<0>();                                  // requests past the end still fill the stages

  // acc[fm][fn][i] = C[row r16][column 4 cg + i] of the 16 x 16 tile.  (The lane
  // is taken anew: it needs no register through the loop.)
  const int le = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), te = wave * 64 + le;
  const int r16 = le & 15, cg = le >> 4;
  if constexpr (EPI == EPI_ROPE_KV || EPI == EPI_STORE || EPI == EPI_GELU || EPI == EPI_SWIGLU) {
    // bf16 results go to LDS and leave in whole rows, 16 bytes per lane
    // (storing from the registers writes 16- and 32-byte pieces of a line:
    // +14 us on the 1021-row ffn_ln1)
    constexpr int BO = EPI == EPI_SWIGLU ? BN / 2 : BN;
    lds_barrier();                                  // every wave's requests have landed and its reads are done
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        const int r = wm * WTM + fm * 16 + r16;
        floatx4 v = acc[fm][fn];
        if constexpr (EPI == EPI_SWIGLU) {
          // columns 0-7 (lanes 0-31) are gate rows, 8-15 (lane + 32) their up
          // rows; swapping halves gives lanes 0-31 both of columns 4 (cg & 1)
          // and + 1, lanes 32-63 both of + 2 and + 3
          float m[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const auto gu = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + 2]), false,
                                                             false);
            m[i] = silu_f(__uint_as_float(gu[0])) * __uint_as_float(gu[1]);
          }
          const int c = (wn * FN + fn) * 8 + 4 * (cg & 1) + (cg & 2);
          reinterpret_cast<uint32_t*>(lds)[tile_chunk<BO>(r, c >> 3) * 4 + ((c >> 1) & 3)] =
              (uint32_t)f2bf(m[0]) | ((uint32_t)f2bf(m[1]) << 16);
        } else {
          if (EPI == EPI_GELU) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = gelu_f(v[i]);
          }
          const int c = wn * WTN + fn * 16 + 4 * cg;
          reinterpret_cast<uint2*>(lds)[tile_chunk<BO>(r, c >> 3) * 2 + ((c >> 2) & 1)] =
              make_uint2((uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                         (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16));
        }
      }
    lds_read_barrier();
    if constexpr (EPI == EPI_ROPE_KV) {
      rope_kv_walk<bf16, BM, BN, 512>(p, m0, n0_out, te);
    } else {
      constexpr int CH = BO / 8;                    // 16-byte chunks per row
      bf16* out = reinterpret_cast<bf16*>(p.out);
      for (int i = te; i < BM * CH; i += 512) {
        const int r = i / CH, c = i % CH;
        const int row = m0 + r, col = n0_out + 8 * c;
        if (row >= p.M || col >= p.N) continue;
        const uint4 v = lds[tile_chunk<BO>(r, c)];
        bf16* dst = out + (size_t)row * p.N + col;
        if (p.vec8) {
          *reinterpret_cast<uint4*>(dst) = v;
        } else {
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (col + e < p.N) dst[e] = (bf16)(w[e / 2] >> (16 * (e & 1)));
        }
      }
    }
    return;
  }
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int r = m0 + wm * WTM + fm * 16 + r16;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int c = n0_out + wn * WTN + fn * 16 + 4 * cg;
      if (r < p.M && c < p.N) epi_store4<EPI>(p, r, c, acc[fm][fn], split);
    }
  }
}

// Tiles of FN groups per wave, XCD-aware order as in gemm_ws_kernel; behind them
// (FT > 0) the tail: the columns from p.tail_n0 on as tiles of FT groups.  Whole
// rounds of one block per CU take the wide tiles and the rest one round of
// narrower ones, where a last round of wide tiles would leave CUs idle
// (LLaMA-13B ffn_ln1 at 1021 rows: 432 wide tiles are 1.69 rounds; 256 and a
// tail of 236: layer 640 -> 627 us; LLaMA-33B at 544 rows 924 -> 906).
template <int FM, int FN, int FT, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_quad_kernel(GemmP p) {
  int b = blockIdx.x, blocks = gridDim.x;
  if constexpr (FT > 0) {
    if (b >= p.wide_blocks) {
      b -= p.wide_blocks;
      blocks -= p.wide_blocks;
      const int t = (b % 8) * (blocks / 8) + b / 8;
      if (t >= p.tail_tiles) return;
      quad_tile<FM, FT, EPI>(p, t % p.tiles_m, 0, p.tail_n0 + t / p.tiles_m * (EPI == EPI_SWIGLU ? 32 * FT : 64 * FT));
      return;
    }
    blocks = p.wide_blocks;
  }
  const int t = (b % 8) * (blocks / 8) + b / 8;
  if (t >= p.n_tiles) return;
  const int rest = t / p.tiles_m;
  quad_tile<FM, FN, EPI>(p, t % p.tiles_m, rest % p.n_split,
                         rest / p.n_split * (EPI == EPI_SWIGLU ? 32 * FN : 64 * FN));
}

// ============================================================================ fp32 FMA
// 64x64 tile of W rows (SwiGLU: 32 gate + 32 up rows -> 32 outputs), BK 64
// (few k-steps: the small fp32 matmuls run few blocks and are latency-bound),
// 16x16 threads with 4x4 results each.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmP p) {
  constexpr int BK = 64;
  __shared__ float As[BK][64 + 4];
  __shared__ float Ws[BK][64 + 4];
  const int tile_m = blockIdx.x, tile_n = blockIdx.y;
  // split-K (EPI_PARTIAL): blockIdx.z takes k in [z * k_split, (z + 1) * k_split)
  const int split = blockIdx.z;
  const int kbeg = split * p.k_split, kend = min(p.K, kbeg + p.k_split);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int m0 = tile_m * 64;
  const int n0_out = tile_n * (EPI == EPI_SWIGLU ? 32 : 64);
  const float* A = reinterpret_cast<const float*>(p.A);
  const float* W = reinterpret_cast<const float*>(p.W);
  int cols[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) cols[j] = (EPI == EPI_SWIGLU) ? ((j < 2) ? 2 * tx + j : 32 + 2 * tx + j - 2) : 4 * tx + j;
  float acc[4][4] = {};
  // Each thread stages PER elements of A and of W per k-step.  All loads are
  // issued before any is used (addresses clamped into the operands, values
  // outside them zeroed afterwards), so a k-step waits for one memory round
  // trip rather than one per element.
  constexpr int PER = 64 * BK / 256;
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    float ra[PER], rw[PER];
    bool oka[PER], okw[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + i * 256;
      const int r = e / BK, kk = e % BK;
      const int gr = m0 + r, gk = k0 + kk;
      const int ck = min(gk, p.K - 1);
      int wrow, jn;
      if (EPI == EPI_SWIGLU) {
        jn = n0_out + (r % 32);
        wrow = (r < 32) ? min(jn, p.N - 1) : p.N + min(jn, p.N - 1);
      } else {
        jn = n0_out + r;
        wrow = min(jn, p.N - 1);
      }
      oka[i] = gr < p.M && gk < kend;
      okw[i] = jn < p.N && gk < kend;
      ra[i] = A[(size_t)min(gr, p.M - 1) * p.K + ck];
      rw[i] = W[(size_t)wrow * p.K + ck];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + i * 256;
      const int r = e / BK, kk = e % BK;
      As[kk][r] = oka[i] ? ra[i] : 0.f;
      Ws[kk][r] = okw[i] ? rw[i] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][4 * ty + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Ws[kk][cols[j]];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = m0 + 4 * ty + i;
    if (r >= p.M) continue;
    if (EPI == EPI_SWIGLU) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = n0_out + 2 * tx + j;
        if (c < p.N)
          reinterpret_cast<float*>(p.out)[(size_t)r * p.N + c] = silu_f(acc[i][j]) * acc[i][j + 2];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = n0_out + 4 * tx + j;
        if (c < p.N) epi_store<float, EPI>(p, r, c, acc[i][j], split);
      }
    }
  }
}

// ============================================================================ launch
// Tile configurations of the bf16 kernel (BM x BN W rows, waves, prefetch stages).
enum TileCfg { CFG_160x128 = 0, CFG_320x128 = 1, CFG_64x128 = 2, CFG_96x128 = 3 };

template <int BM, int BN, int WGM, int WGN, int PD, int EPI>
static hipError_t run_bf16(GemmP p, hipStream_t s) {
  const size_t lds_bytes = 2 * (BM + BN) * 8 * sizeof(uint4);
  static std::atomic<uint64_t> lds_set{0};   // devices on which this instance's LDS limit is raised
  hipError_t e = ensure_dynamic_lds((const void*)gemm_bf16_kernel<BM, BN, WGM, WGN, PD, EPI>, (int)lds_bytes, lds_set);
  if (e != hipSuccess) return e;
  const int grid = (p.n_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, PD, EPI>), dim3(grid), dim3(64 * WGM * WGN), lds_bytes,
                     s, p);
  return hipGetLastError();
}

template <typename T, int BM, int BN, int WGM, int WGN, int NP, int S, int EPI, bool STREAM>
static hipError_t run_ws_as(const GemmP& p, hipStream_t s) {
  const size_t lds_bytes = (size_t)S * (BM + BN) * 8 * sizeof(uint4);
  static std::atomic<uint64_t> lds_set{0};   // devices on which this instance's LDS limit is raised
  hipError_t e = ensure_dynamic_lds((const void*)gemm_ws_kernel<T, BM, BN, WGM, WGN, NP, S, EPI, STREAM>, (int)lds_bytes, lds_set);
  if (e != hipSuccess) return e;
  const int grid = (p.n_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_ws_kernel<T, BM, BN, WGM, WGN, NP, S, EPI, STREAM>), dim3(grid),
                     dim3(64 * (WGM * WGN + NP)), lds_bytes, s, p);
  return hipGetLastError();
}

template <typename T, int BM, int BN, int WGM, int WGN, int NP, int S, int EPI>
static hipError_t run_ws(const GemmP& p, bool stream_w, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if (stream_w) return run_ws_as<T, BM, BN, WGM, WGN, NP, S, EPI, true>(p, s);
  }
  return run_ws_as<T, BM, BN, WGM, WGN, NP, S, EPI, false>(p, s);
}

constexpr int QUAD_TAIL = 3;   // a tail's tiles: 192 W rows
template <int FM, int FN, int FT, int EPI>
static hipError_t run_quad_as(const GemmP& p, hipStream_t s) {
  // two stages of two halves (the RoPE epilogue's tile fits there)
  constexpr int ROWS0 = (2 * ((FM + 1) / 2) + 4 * ((FN + 1) / 2)) * 16;   // rows of a half stage
  static_assert((FT + 1) / 2 <= (FN + 1) / 2, "the tail's tiles need no more LDS");
  const size_t lds_bytes = (size_t)4 * ROWS0 * 128;
  static std::atomic<uint64_t> lds_set{0};   // devices on which this instance's LDS limit is raised
  hipError_t e = ensure_dynamic_lds((const void*)gemm_quad_kernel<FM, FN, FT, EPI>, (int)lds_bytes, lds_set);
  if (e != hipSuccess) return e;
  const int grid = FT > 0 ? p.wide_blocks + (p.tail_tiles + 7) / 8 * 8 : (p.n_tiles + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_quad_kernel<FM, FN, FT, EPI>), dim3(grid), dim3(512), lds_bytes, s, p);
  return hipGetLastError();
}

template <int FM, int FN, int EPI>
static hipError_t run_quad(const GemmP& p, bool tail, hipStream_t s) {
  if constexpr (FN == 4 && EPI != EPI_PARTIAL) {
    if (tail) return run_quad_as<FM, FN, QUAD_TAIL, EPI>(p, s);
  }
  return run_quad_as<FM, FN, 0, EPI>(p, s);
}

template <int BM, int BN, int WGM, int WGN, int PD>
static hipError_t run_bf16_epi(int epi, const GemmP& p, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return run_bf16<BM, BN, WGM, WGN, PD, EPI_STORE>(p, s);
    case EPI_GELU: return run_bf16<BM, BN, WGM, WGN, PD, EPI_GELU>(p, s);
    case EPI_SWIGLU: return run_bf16<BM, BN, WGM, WGN, PD, EPI_SWIGLU>(p, s);
    case EPI_RESID_TO_F32: return run_bf16<BM, BN, WGM, WGN, PD, EPI_RESID_TO_F32>(p, s);
    case EPI_RESIDF32_TO_ACT: return run_bf16<BM, BN, WGM, WGN, PD, EPI_RESIDF32_TO_ACT>(p, s);
    default: return run_bf16<BM, BN, WGM, WGN, PD, EPI_PARTIAL>(p, s);
  }
}

template <int EPI>
static hipError_t run_f32(const GemmP& p, hipStream_t s) {
  const int out_per_tile = (EPI == EPI_SWIGLU) ? 32 : 64;
  dim3 grid((p.M + 63) / 64, (p.N + out_per_tile - 1) / out_per_tile, p.n_split);
  hipLaunchKernelGGL(gemm_f32_kernel<EPI>, grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

static int cfg_bm(int cfg) {
  switch (cfg) {
    case CFG_320x128: return 320;
    case CFG_64x128: return 64;
    case CFG_96x128: return 96;
    default: return 160;
  }
}

// Tile choice for the skinny matmuls of the hybrid batch (M = C + B rows).
// Many W panels (>= 180 tiles of 128 rows) and M in (160, 320]: one block
// covers all rows (W read once per block, 8 waves).  A middle count: 160-row
// blocks.  Few panels (postproj / ffn_ln2 at N = hidden): 64-row blocks with
// split-K -- or, when split-K scratch is available and M in (160, 320],
// 320-row blocks split over K (chosen by the caller).  Small M: the block
// height that pads M least.
static int pick_cfg(int M, int n_panels) {
  if (M <= 64) return CFG_64x128;
  if (M <= 96) return CFG_96x128;
  if (n_panels >= 180 && M > 160 && M <= 320) return CFG_320x128;
  if (n_panels >= 100) {
    const int pad160 = (M + 159) / 160 * 160, pad96 = (M + 95) / 96 * 96;
    return pad96 < pad160 ? CFG_96x128 : CFG_160x128;
  }
  return CFG_64x128;
}

// Producer/consumer tiles (BM x BN W rows; consumer waves 2 x (BN / 32), or
// 2 x 2 for BN = 64; 4 producer waves, 2 beside 14 consumers) and their LDS
// ring depth (~100-156 KB).
struct WsTile {
  int bm, bn;
};
constexpr WsTile kWsTiles[] = {{64, 64},   {64, 128},  {64, 256},  {96, 128},  {96, 192},  {96, 256},
                               {128, 128}, {128, 192}, {128, 224}, {128, 256}, {160, 128}, {160, 192},
                               {160, 224}, {160, 256}, {288, 192}, {192, 256}, {256, 256}};
constexpr int kFirstQuadTile = 14;   // the rest run gemm_quad_kernel
// Their price per 64-wide k-tile, and per block beyond the producer tiles' 3 us
// (us; on the scale of the producer tiles' prices, which run 1-30% above what
// those measure, most where a round leaves CUs idle).  Fitted to every tile and K-split of the twelve matmuls at 33
// row counts of 8-1536: the picks then take 1.2% more than the fastest tile, and
// 1.7% at the loop's own 1.27 / 1.17 / 1.5 without the extra fill (LLaMA-33B
// layer of 192 rows 364 -> 350 us, 288 rows 406 -> 393, GPT-3 of 400 rows
// 1648 -> 1619: producer tiles where those took quadrant ones).
constexpr double kQuadTileUs[] = {1.37, 1.22, 1.56};
constexpr double kQuadFillUs = 3.5;
constexpr int kNumWsTiles = sizeof(kWsTiles) / sizeof(kWsTiles[0]);

// Variants of a launch: gemm_ws_kernel with W loaded non-temporally, and
// gemm_quad_kernel with a tail of narrower tiles.
struct WsLaunch {
  bool stream_w, tail;
};

template <int EPI>
static hipError_t run_ws_cfg(int cfg, const GemmP& p, const WsLaunch& how, hipStream_t s) {
  switch (cfg) {
    case 0: return run_ws<bf16, 64, 64, 2, 2, 4, 6, EPI>(p, how.stream_w, s);
    case 1: return run_ws<bf16, 64, 128, 2, 4, 4, 6, EPI>(p, how.stream_w, s);
    case 2: return run_ws<bf16, 64, 256, 2, 4, 4, 3, EPI>(p, how.stream_w, s);
    case 3: return run_ws<bf16, 96, 128, 2, 4, 4, 5, EPI>(p, how.stream_w, s);
    case 4: return run_ws<bf16, 96, 192, 2, 6, 4, 4, EPI>(p, how.stream_w, s);
    case 5: return run_ws<bf16, 96, 256, 2, 4, 4, 3, EPI>(p, how.stream_w, s);
    case 6: return run_ws<bf16, 128, 128, 2, 4, 4, 4, EPI>(p, how.stream_w, s);
    case 7: return run_ws<bf16, 128, 192, 2, 6, 4, 3, EPI>(p, how.stream_w, s);
    case 8: return run_ws<bf16, 128, 224, 2, 7, 2, 3, EPI>(p, how.stream_w, s);
    case 9: return run_ws<bf16, 128, 256, 2, 4, 4, 3, EPI>(p, how.stream_w, s);
    case 10: return run_ws<bf16, 160, 128, 2, 4, 4, 4, EPI>(p, how.stream_w, s);
    case 11: return run_ws<bf16, 160, 192, 2, 6, 4, 3, EPI>(p, how.stream_w, s);
    case 12: return run_ws<bf16, 160, 224, 2, 7, 2, 3, EPI>(p, how.stream_w, s);
    case 13: return run_ws<bf16, 160, 256, 2, 4, 4, 3, EPI>(p, how.stream_w, s);
    case 14: return run_quad<9, 3, EPI>(p, how.tail, s);
    case 15: return run_quad<6, 4, EPI>(p, how.tail, s);
    default: return run_quad<8, 4, EPI>(p, how.tail, s);
  }
}

static hipError_t run_ws_epi(int epi, int cfg, const GemmP& p, const WsLaunch& how, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return run_ws_cfg<EPI_STORE>(cfg, p, how, s);
    case EPI_GELU: return run_ws_cfg<EPI_GELU>(cfg, p, how, s);
    case EPI_SWIGLU: return run_ws_cfg<EPI_SWIGLU>(cfg, p, how, s);
    case EPI_RESID_TO_F32: return run_ws_cfg<EPI_RESID_TO_F32>(cfg, p, how, s);
    case EPI_RESIDF32_TO_ACT: return run_ws_cfg<EPI_RESIDF32_TO_ACT>(cfg, p, how, s);
    case EPI_ROPE_KV: return run_ws_cfg<EPI_ROPE_KV>(cfg, p, how, s);
    default: return run_ws_cfg<EPI_PARTIAL>(cfg, p, how, s);
  }
}

// fp32 tiles of the same kernel (4 consumer waves of 2 x 2, or 8 of 2 x 4; the
// 32-row ones 2 x 1 and 2 x 2), and their ring depth (48-112 KB; the 32-row
// tiles leave room for two or three blocks per CU).
constexpr WsTile kF32Tiles[] = {{32, 32}, {32, 64}, {64, 64}, {96, 64}, {160, 64}, {96, 128}, {160, 128}};
constexpr int kNumF32Tiles = sizeof(kF32Tiles) / sizeof(kF32Tiles[0]);

template <int EPI>
static hipError_t run_ws_f32_cfg(int cfg, const GemmP& p, hipStream_t s) {
  switch (cfg) {
    case 0: return run_ws<float, 32, 32, 2, 1, 2, 6, EPI>(p, false, s);
    case 1: return run_ws<float, 32, 64, 2, 2, 2, 6, EPI>(p, false, s);
    case 2: return run_ws<float, 64, 64, 2, 2, 4, 6, EPI>(p, false, s);
    case 3: return run_ws<float, 96, 64, 2, 2, 4, 5, EPI>(p, false, s);
    case 4: return run_ws<float, 160, 64, 2, 2, 4, 4, EPI>(p, false, s);
    case 5: return run_ws<float, 96, 128, 2, 4, 4, 4, EPI>(p, false, s);
    default: return run_ws<float, 160, 128, 2, 4, 4, 3, EPI>(p, false, s);
  }
}

static hipError_t run_ws_f32(int epi, int cfg, const GemmP& p, hipStream_t s) {
  switch (epi) {
    case EPI_STORE: return run_ws_f32_cfg<EPI_STORE>(cfg, p, s);
    case EPI_GELU: return run_ws_f32_cfg<EPI_GELU>(cfg, p, s);
    case EPI_SWIGLU: return run_ws_f32_cfg<EPI_SWIGLU>(cfg, p, s);
    case EPI_RESID_TO_F32: return run_ws_f32_cfg<EPI_RESID_TO_F32>(cfg, p, s);
    case EPI_RESIDF32_TO_ACT: return run_ws_f32_cfg<EPI_RESIDF32_TO_ACT>(cfg, p, s);
    case EPI_ROPE_KV: return run_ws_f32_cfg<EPI_ROPE_KV>(cfg, p, s);
    default: return run_ws_f32_cfg<EPI_PARTIAL>(cfg, p, s);
  }
}

// Tile (and K-split) choice from a cost model of the operand feed, fitted to
// MI355X measurements of the LLaMA-13B / 33B shapes.  Each CU runs one block
// at a time and is bound by its outstanding memory requests: a 64-wide k-tile
// costs ~1.9 ns per A row (L2 hits) and ~3.1 ns per W row when two M-tiles
// share the W panel (~4.2 ns when one block streams it alone, every row an HBM
// miss: taken before such loads were non-temporal, which made them 9-12%
// faster); a block adds ~3 us of pipeline fill plus its output writes
// (~40 GB/s per CU); blocks beyond the first 256 run as another round.  The
// quadrant kernel's tiles have prices of their own (above).  A
// split-K op's reduction pass reads the fp32 partials and writes the result
// at ~5.5 TB/s.  postproj's takes in the norm that follows, which costs a pass
// of its own without a split (LLaMA-13B layer of 1024 rows: 614 us with a split
// 192 x 256, 628 with an unsplit 128 x 192 that runs postproj alone as fast);
// the pass counts by its traffic, without its launch, so that a small op called
// alone is not split for it (200 x 5120 x 704: 11.0 us, 13.2 in two splits).
struct WsChoice {
  int cfg, n_split;
  int wide_n = 0;      // quadrant tiles: > 0, that many W panels of them and a tail of narrower tiles
};
static WsChoice pick_ws(int M, int N, int K, bool swiglu, bool norm_follows, int max_split) {
  WsChoice best{10, 1};
  double best_t = 1e300;
  const int nk = K / 64;
  const double norm_us = norm_follows ? 6.0 * (double)M * N / 5.5e6 : 0.0;
  for (int c = 0; c < kNumWsTiles; ++c) {
    const int bm = kWsTiles[c].bm, bn = kWsTiles[c].bn;
    if (bm == 64 && M > 128) continue;   // 64-row tiles only for short batches
    // 128-row tiles: two cover 256 rows where 160-row ones pad to 320 (LLaMA-13B
    // at 256 rows, alone: preproj 55.7 -> 52.4 us, ffn_ln1 84.2 -> 77.2, ffn_ln2
    // 51.0 -> 49.2; 200 x 15360 x 512 10.7 -> 9.6, 200 x 19968 x 960 18.8 -> 17.1).
    if (bm == 128 && M <= 96) continue;
    if (c >= kFirstQuadTile && M <= 160) continue;
    const int per = swiglu ? bn / 2 : bn;
    const int tiles_m = (M + bm - 1) / bm;
    const long tiles = (long)tiles_m * ((N + per - 1) / per);
    const double per_k = c >= kFirstQuadTile ? kQuadTileUs[c - kFirstQuadTile]
                                             : 1.9e-3 * bm + (tiles_m >= 2 ? 3.1e-3 : 4.2e-3) * bn;   // us per k-tile
    const double fill = 3.0 + (c >= kFirstQuadTile ? kQuadFillUs : 0.0);
    for (int ns = 1; ns <= max_split; ++ns) {
      const double rounds = (double)((tiles * ns + 255) / 256);
      const double k_tiles = 2.0 * ((nk / 2 + ns - 1) / ns);               // whole pairs per split
      const double out_bytes = (double)bm * (swiglu ? bn / 2 : bn) * (ns > 1 ? 4.0 : 2.0);
      double t = rounds * (k_tiles * per_k + fill + out_bytes / 4.0e4);
      t += ns > 1 ? (ns * 4.0 + 6.0) * (double)M * N / 5.5e6 + 2.0 : norm_us;
      if (t < best_t * 0.999) {
        best_t = t;
        best = {c, ns};
      }
    }
    // 256-wide quadrant tiles whose last round is not full: whole rounds of
    // them, then one round of 192-wide tiles over the columns left
    if (c < kFirstQuadTile || bn != 256 || tiles <= 256 || tiles % 256 == 0) continue;
    const int rounds = (int)(tiles / 256), wide_n = rounds * 256 / tiles_m;
    const int pert = per / 4 * QUAD_TAIL, left = N - wide_n * per;
    if (left <= 0 || (long)tiles_m * ((left + pert - 1) / pert) > 256) continue;
    const double out_us = (double)bm * per * 2.0 / 4.0e4;
    const double tail_us = nk * (bm == 256 ? 1.15 : 0.95) + fill + out_us * 0.75;
    const double t = rounds * (nk * per_k + fill + out_us) + tail_us + norm_us;
    if (t < best_t * 0.999) {
      best_t = t;
      best = {c, 1, wide_n};
    }
  }
  return best;
}

// The same for fp32: a 32-wide k-tile costs its products at the fp32 matrix
// rate (256 flop per clock and CU) or its operand feed, whichever is longer,
// and at least a barrier round trip; small shapes are bound by the fill and
// the number of k-tiles in a row, so they take many small tiles.
static WsChoice pick_f32(int M, int N, int K, bool swiglu, int max_split) {
  WsChoice best{0, 1};
  double best_t = 1e300;
  for (int c = 0; c < kNumF32Tiles; ++c) {
    const int bm = kF32Tiles[c].bm, bn = kF32Tiles[c].bn;
    const int per = swiglu ? bn / 2 : bn;
    const long tiles = (long)((M + bm - 1) / bm) * ((N + per - 1) / per);
    const double per_k = std::max(std::max(1.04e-4 * bm * bn * 1.1, 1.9e-3 * bm + 4.2e-3 * bn), 0.15);   // us
    for (int ns = 1; ns <= max_split; ++ns) {
      const double rounds = (double)((tiles * ns + 255) / 256);
      const double k_tiles = 4.0 * (((K + 127) / 128 + ns - 1) / ns);        // whole groups of four per split
      double t = rounds * (k_tiles * per_k + 2.0 + (double)bm * per * 4.0 / 4.0e4);
      if (ns > 1) t += (ns + 2) * 4.0 * (double)M * N / 5.5e6 + 3.0;
      if (t < best_t * 0.999) {
        best_t = t;
        best = {c, ns};
      }
    }
  }
  return best;
}

int linear_tile_count() { return kNumWsTiles; }
bool linear_tile_shape(int tile, int* bm, int* bn) {
  if (tile < 0 || tile >= kNumWsTiles) return false;
  *bm = kWsTiles[tile].bm;
  *bn = kWsTiles[tile].bn;
  return true;
}

hipError_t launch_linear(int dtype, const LinearArgs& a, hipStream_t s, int force_tile, int force_split,
                         LinearPlan* plan) {
  if (plan) *plan = LinearPlan{};
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  GemmP p{};
  p.A = a.x; p.W = a.w; p.M = a.M; p.N = a.N; p.K = a.K;
  p.out = a.out; p.resid = a.resid;
  p.k_split = a.K; p.n_split = 1;

  if (dtype == 0) {
    const bool resid_kind = a.kind == LIN_RESID || a.kind == LIN_RESID_F32IN;
    const bool swiglu = a.kind == LIN_SWIGLU;
    // Split-K of the residual ops: fp32 partials per split of whole groups of
    // four 32-wide k-tiles, then residual + partials added in split order
    // (deterministic).
    int max_split = 1;
    if (resid_kind && a.parts != nullptr) {
      max_split = std::min(MAX_SPLIT, (a.K + 127) / 128);
      max_split = (int)std::min<size_t>((size_t)max_split, a.parts_cap / ((size_t)a.M * a.N));
      max_split = std::max(max_split, 1);
    }
    // matrix-core kernel: x and W each under 4 GiB (32-bit row offsets);
    // sizes past that take the register-staged vector kernel
    const size_t w_rows = swiglu ? 2 * (size_t)a.N : (size_t)a.N;
    const bool ws = (size_t)a.M * a.K * 4 < (1ull << 32) && w_rows * a.K * 4 < (1ull << 32);
    WsChoice ch{2, 1};
    if (ws) {
      ch = pick_f32(a.M, a.N, a.K, swiglu, max_split);
    } else {
      const int tiles = ((a.M + 63) / 64) * ((a.N + 63) / 64);
      if (tiles < 64) ch.n_split = std::min(max_split, (64 + tiles - 1) / tiles);
    }
    const int bm = ws ? kF32Tiles[ch.cfg].bm : 64, bn = ws ? kF32Tiles[ch.cfg].bn : 64;
    const int groups = (a.K + 127) / 128;
    if (ch.n_split > 1) {
      p.k_split = (groups + ch.n_split - 1) / ch.n_split * 128;
      p.n_split = (a.K + p.k_split - 1) / p.k_split;
    }
    if (plan) {
      *plan = LinearPlan{bm, bn, p.n_split, 0, 0};
      return hipSuccess;
    }
    const bool split = p.n_split > 1;
    if (split) p.out = a.parts;
    // preproj with the rotary embedding and KV append in its epilogue
    const bool rope = ws && a.kind == LIN_PLAIN && a.rope != nullptr && a.rope->hd % 16 == 0 &&
                      a.N == 3 * a.rope->nh * a.rope->hd;
    if (rope) {
      p.rope = *a.rope;
      if (a.rope_done) *a.rope_done = true;
    }
    const int epi = split                      ? EPI_PARTIAL
                    : rope                     ? EPI_ROPE_KV
                    : a.kind == LIN_PLAIN      ? EPI_STORE
                    : a.kind == LIN_GELU       ? EPI_GELU
                    : a.kind == LIN_SWIGLU     ? EPI_SWIGLU
                    : a.kind == LIN_RESID      ? EPI_RESID_TO_F32
                                               : EPI_RESIDF32_TO_ACT;
    hipError_t e;
    if (ws) {
      p.tiles_m = (a.M + bm - 1) / bm;
      p.tiles_n = (a.N + (swiglu ? bn / 2 : bn) - 1) / (swiglu ? bn / 2 : bn);
      p.n_tiles = p.tiles_m * p.tiles_n * p.n_split;
      e = run_ws_f32(epi, ch.cfg, p, s);
    } else {
      switch (epi) {
        case EPI_STORE: e = run_f32<EPI_STORE>(p, s); break;
        case EPI_GELU: e = run_f32<EPI_GELU>(p, s); break;
        case EPI_SWIGLU: e = run_f32<EPI_SWIGLU>(p, s); break;
        case EPI_RESID_TO_F32: e = run_f32<EPI_RESID_TO_F32>(p, s); break;
        case EPI_RESIDF32_TO_ACT: e = run_f32<EPI_RESIDF32_TO_ACT>(p, s); break;
        default: e = run_f32<EPI_PARTIAL>(p, s); break;
      }
    }
    if (e != hipSuccess || !split) return e;
    return launch_split_reduce(0, a.kind == LIN_RESID_F32IN, a.kind == LIN_RESID, a.resid, a.parts, p.n_split,
                               (size_t)a.M * a.N, a.out, s);
  }

  int epi;
  switch (a.kind) {
    case LIN_PLAIN: epi = EPI_STORE; break;
    case LIN_GELU: epi = EPI_GELU; break;
    case LIN_SWIGLU: epi = EPI_SWIGLU; break;
    case LIN_RESID: epi = EPI_RESID_TO_F32; break;
    default: epi = EPI_RESIDF32_TO_ACT; break;
  }
  const bool swiglu = a.kind == LIN_SWIGLU;
  const bool resid_kind = a.kind == LIN_RESID || a.kind == LIN_RESID_F32IN;
  // producer/consumer kernel: whole 64-wide k-tiles, and x and W each under
  // 4 GiB (its producers address rows by 32-bit byte offsets)
  const size_t w_rows = swiglu ? 2 * (size_t)a.N : (size_t)a.N;
  const bool ws = (a.K % 64) == 0 && (size_t)a.M * a.K * 2 < (1ull << 32) && w_rows * a.K * 2 < (1ull << 32);

  // splits available to the residual ops: whole groups of two k-tiles per
  // split, partials must fit the scratch
  int max_split = 1;
  if (resid_kind && a.parts != nullptr) {
    max_split = std::min(MAX_SPLIT, (a.K + 127) / 128 / 2);
    max_split = (int)std::min<size_t>((size_t)max_split, a.parts_cap / ((size_t)a.M * a.N));
    max_split = std::max(max_split, 1);
  }
  int cfg, BM, BN, ws_split = 1, wide_n = 0;
  if (ws) {
    WsChoice ch = pick_ws(a.M, a.N, a.K, swiglu, a.kind == LIN_RESID, max_split);
    if (force_tile >= 0 && force_tile < kNumWsTiles) ch = {force_tile, std::min(std::max(force_split, 1), max_split)};
    cfg = ch.cfg;
    ws_split = ch.n_split;
    wide_n = ch.wide_n;
    BM = kWsTiles[cfg].bm;
    BN = kWsTiles[cfg].bn;
  } else {
    BN = 128;
    const int n_panels = (a.N + (swiglu ? BN / 2 : BN) - 1) / (swiglu ? BN / 2 : BN);
    const bool split_kind = resid_kind && a.parts != nullptr;
    cfg = (split_kind && a.M > 160 && a.M <= 320 && n_panels < 256) ? CFG_320x128 : pick_cfg(a.M, n_panels);
    BM = cfg_bm(cfg);
  }
  const int out_per_tile = swiglu ? BN / 2 : BN;
  p.tiles_m = (a.M + BM - 1) / BM;
  p.tiles_n = (a.N + out_per_tile - 1) / out_per_tile;
  // preproj with the rotary embedding and KV append in its epilogue (W rows
  // loaded in rotary-pair order, any tile)
  if (ws && a.kind == LIN_PLAIN && a.rope != nullptr) {
    const int hd = a.rope->hd, QD = a.rope->nh * hd;
    if (hd % 16 == 0 && a.N == 3 * QD) {
      epi = EPI_ROPE_KV;
      p.rope = *a.rope;
      if (a.rope_done) *a.rope_done = true;
    }
  }

  // Split-K for the residual ops when the tile grid leaves CUs idle: every
  // split stores its fp32 partial, then one pass adds residual + partials in
  // split order (deterministic).  Each split covers whole groups of two
  // 64-wide k-tiles.  Blocks of ~150 KB of LDS run one per CU, so the split
  // count keeps the grid within one wave of blocks over the 256 CUs.
  const int tiles = p.tiles_m * p.tiles_n;
  int n_split = 1;
  if (resid_kind && a.parts != nullptr && (ws ? ws_split > 1 : tiles < 256)) {
    const int kgroups = (a.K + 127) / 128;
    int ns = ws ? ws_split : (cfg == CFG_320x128 ? 256 / tiles : (400 + tiles - 1) / tiles);
    if (ns > kgroups / 2) ns = kgroups / 2;
    if (ns > MAX_SPLIT) ns = MAX_SPLIT;
    if ((size_t)ns * a.M * a.N > a.parts_cap) ns = (int)(a.parts_cap / ((size_t)a.M * a.N));
    if (ns > 1) {
      const int g_per = (kgroups + ns - 1) / ns;
      p.k_split = g_per * 128;
      p.n_split = (a.K + p.k_split - 1) / p.k_split;
      n_split = p.n_split;
      epi = EPI_PARTIAL;
      p.out = a.parts;
    }
  }
  if (wide_n > 0) {
    const int per_tail = out_per_tile / 4 * QUAD_TAIL;
    p.tail_n0 = wide_n * out_per_tile;
    p.tail_tiles = p.tiles_m * ((a.N - p.tail_n0 + per_tail - 1) / per_tail);
    p.tiles_n = wide_n;
    p.wide_blocks = (p.tiles_m * wide_n + 7) / 8 * 8;
  }
  p.n_tiles = p.tiles_m * p.tiles_n * p.n_split;
  p.vec4 = a.N % 4 == 0 && ((reinterpret_cast<uintptr_t>(p.out) | reinterpret_cast<uintptr_t>(p.resid)) & 15) == 0;
  p.vec8 = p.vec4 && a.N % 8 == 0;
  // One M-tile: every W line is read once, so it is loaded non-temporally
  // (alone, weights from HBM: LLaMA-13B 4 rows ffn_ln1 49.5 -> 44.4 us, 5.7 ->
  // 6.4 TB/s; LLaMA-33B 160 rows ffn_ln1 107 -> 97; GPT-3 30 rows ffn_ln2 215 ->
  // 189; the quadrant tiles gain nothing).  Not below 32 MB: the weights of such a model can stay in the 256 MB
  // memory-side cache from call to call.  Two M-tiles meet in L2 instead.
  const bool stream_w = ws && cfg < kFirstQuadTile && p.tiles_m == 1 && w_rows * a.K * 2 >= (32u << 20);
  // Rotated k order for the two M-tiles of a W panel, when a block runs at
  // most 192 k-tiles.  Measured in the layers: LLaMA-13B preproj -13% and
  // ffn_ln1 -2%; LLaMA-33B at 288 rows every op -2..-5% (layer -4%); GPT-3
  // preproj, postproj and ffn_ln1 -2..-6% (96-192 k-tiles); but GPT-3 ffn_ln2
  // (384 k-tiles per split) +6%.  Four M-tiles: no gain.
  {
    const int nk_block = (n_split > 1 ? p.k_split : a.K) / 64;
    p.rotate_k = (ws && cfg < kFirstQuadTile && p.tiles_m == 2 && nk_block <= 192) ? 1 : 0;
  }
  if (plan) {
    *plan = LinearPlan{BM, BN, p.n_split, wide_n > 0 ? a.N - p.tail_n0 : 0, wide_n > 0 ? BN / 4 * QUAD_TAIL : 0};
    return hipSuccess;
  }
  hipError_t e;
  if (ws) {
    e = run_ws_epi(epi, cfg, p, WsLaunch{stream_w, wide_n > 0}, s);
  } else {
    switch (cfg) {
      case CFG_320x128: e = run_bf16_epi<320, 128, 4, 2, 2>(epi, p, s); break;
      case CFG_64x128: e = run_bf16_epi<64, 128, 2, 2, 2>(epi, p, s); break;
      case CFG_96x128: e = run_bf16_epi<96, 128, 2, 2, 2>(epi, p, s); break;
      default: e = run_bf16_epi<160, 128, 2, 2, 2>(epi, p, s); break;
    }
  }
  if (e != hipSuccess) return e;
  if (n_split > 1) {
    if (a.norm != nullptr && resid_kind && dtype == 1) {
      e = launch_split_reduce_norm(a.resid, a.kind == LIN_RESID_F32IN, a.parts, n_split, a.M, a.N, a.out, *a.norm, s);
      if (e == hipSuccess && a.norm_done) *a.norm_done = true;
      if (e != hipErrorNotSupported) return e;
    }
    return launch_split_reduce(dtype, a.kind == LIN_RESID_F32IN, a.kind == LIN_RESID, a.resid, a.parts, n_split,
                               (size_t)a.M * a.N, a.out, s);
  }
  return hipSuccess;
}

}  // namespace sarathi
