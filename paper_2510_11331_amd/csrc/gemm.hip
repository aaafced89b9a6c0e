// Skinny GEMM for the projections of the draft and verify passes:
// out[M, N] = A[M, K] * W[N, K]^T with M = rows of the pass (a few to a few
// dozen; 64 per block), fp32 accumulation.  Passes of more rows, and wide
// projections it does not fit, run on the row-tiled GEMM below.
//
// The pass is bound by streaming W from HBM, so the kernel is organised
// around that stream:
//   * W and A are stored in the MFMA-tile layout (W packed once by
//     sd_pack_linear, A written that way by the producing kernels), so every
//     fragment load of a wave is one contiguous 1 KB block;
//   * a workgroup owns one column tile (16*NT output columns = 16*NT rows
//     of W; NT in {1, 2, 3, 4}, wider tiles re-read the activations less
//     often) and splits K over its KW waves (up to 4), interleaved in
//     groups of U k-steps; each wave streams its share of the tile straight
//     into registers, one step group ahead of the MFMAs;
//   * or, in balanced mode (one M block), the grid is one workgroup per CU
//     and the N / 16 column tiles are dealt out evenly, up to NT = 6 per
//     workgroup: at 33-48 rows the activation re-reads from L2 then cost a
//     third as much, and no CU holds more work than another by more than
//     one deal unit;
//   * the matching activation fragments are loaded the same way (they are
//     small and stay in L2), so the main loop has no LDS traffic and no
//     barriers; it has no branches either (padding rows and groups past a
//     wave's share are out-of-range buffer loads that return zero), so
//     vmcnt only ever waits for the older step group;
//   * bf16 models (operands in fp16, see f16_t): one v_mfma_f32_16x16x32_f16
//     per 16-byte unit; fp32: four v_mfma_f32_16x16x4_f32;
//   * the KW partial tiles are added in wave order through LDS in one round
//     (deterministic); K is never split across workgroups (a cross-workgroup
//     reduction needs a device-scope release per workgroup, which costs more
//     than it recovers at these sizes);
//   * for projections with few column tiles, K may also be split over
//     gridDim.y workgroups that store fp32 partial sums; the RMSNorm that
//     follows adds them to the residual stream in split order (no
//     cross-workgroup synchronisation, deterministic);
//   * epilogues: store fp32, add into the fp32 residual stream, SwiGLU over
//     interleaved gate/up rows (written in the model dtype), or, for the QKV
//     projection, the rotary embedding of q and k (rows in rotary pair
//     order: the two halves of a pair sit 8 columns apart in one tile and
//     meet through a lane exchange) with q stored in fp32 and k, v appended
//     to the paged KV cache.
#include "sd_internal.h"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace sd {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<f16_t> {
  __device__ __forceinline__ static f32x4 step(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                  0, 0);
  }
};
template <> struct Mfma<float> {
  __device__ __forceinline__ static f32x4 step(u32x4 a, u32x4 b, f32x4 c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

__device__ __forceinline__ float silu(float g) { return g / (1.0f + expf(-g)); }

// register budget the compiler plans for: narrow tiles as for 16 waves
// (128 VGPRs, several workgroups per CU), wider ones as for 8 (256 VGPRs);
// a launch runs at most 4 waves
template <int MT, int NT> struct GemmBounds {
  static constexpr int threads = (MT * NT <= 4 && MT < 4 && NT < 4) ? 1024 : 512;
};

// Buffer resource over `bytes` bytes at p: raw (unswizzled) addressing with
// range checking, so a load at an offset >= bytes returns zero and reads no
// memory.  The main loop uses such offsets for padding rows and for step
// groups past a wave's share instead of branches: a load under a branch makes
// the compiler wait for every outstanding load before the next MFMA, which
// serialises the stream.
constexpr uint32_t OOB = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
// 16-byte buffer load; NT: non-temporal (streamed once, not kept in the caches)
template <bool NT> __device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, NT ? 2 : 0));
}

// QKV projection epilogue, shared by both GEMM kernels.  Output columns are
// the fused [q heads | k heads | v heads] rows of the weight, q and k in
// rotary pair order: column r16 < 8 of a 16-column tile of a q or k head is
// dim 8 b + r16 of the head, column r16 + 8 its partner dim hd/2 + 8 b + r16,
// so the two halves of a pair meet in one lane exchange (r16 ^ 8).
// qkv_column classifies column c0 + r16 of this lane once per tile: kind (0
// q, 1 k, 2 v), the q column, the rotary frequency index f, and the K/V
// element offset of (token 0, block 0); a row adds its block and token.
template <typename T>
__device__ __forceinline__ void qkv_column(const RopeParams& rp, int c0, int r16, int& kind, int& qcol, int& f,
                                           size_t& kvb) {
  const int hd = rp.hd, half = hd / 2, Nq = rp.H * hd, Nqk = Nq + rp.KV * hd;
  c0 += rp.col0;
  kind = c0 < Nq ? 0 : c0 < Nqk ? 1 : 2;
  qcol = 0;
  f = 0;
  kvb = 0;
  if (c0 < Nqk) {
    const int h = c0 / hd;
    f = 8 * ((c0 % hd) / 16) + (r16 & 7);
    const int d = r16 < 8 ? f : f + half;
    if (h < rp.H) qcol = h * hd + d;
    else kvb = kv_tile_off(h - rp.H, 0, 0, rp.nblk, hd) + kv_key_off<T>(0, d, hd);
  } else {
    const int cv = c0 + r16 - Nqk;
    kvb = kv_tile_off(cv / hd, 0, 1, rp.nblk, hd) + kv_val_off<T>(0, cv % hd, hd);
  }
}

// Rotary embedding of row m (position pos, KV block blk or -1) for the NT
// tiles of a lane: o = this lane's projection, pr = its pair partner's, cs =
// (cos, sin) of the lane's frequency; q goes to rp.q (fp32), k and v are
// appended to the cache (skipped when blk < 0: over capacity, flagged).
template <typename T, int NT>
__device__ __forceinline__ void qkv_store(const RopeParams& rp, int m, int pos, int blk, int r16, const float (&o)[NT],
                                          const float (&pr)[NT], const float2 (&cs)[NT], const int (&kind)[NT],
                                          const int (&qcol)[NT], const size_t (&kvb)[NT], int nt = NT) {
  const int off = pos & 15;
  T* kv = (T*)rp.kv;
  const size_t brow = (size_t)max(blk, 0) * 32 * rp.hd;   // block offset inside a head's run
  const size_t Nq = (size_t)rp.H * rp.hd;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    if (j >= nt) continue;                                // columns at or past N
    const float a = r16 < 8 ? o[j] : pr[j], b = r16 < 8 ? pr[j] : o[j];
    const float y = r16 < 8 ? a * cs[j].x - b * cs[j].y : a * cs[j].y + b * cs[j].x;
    if (kind[j] == 0) rp.q[(size_t)m * Nq + qcol[j]] = y;
    else if (blk < 0) continue;
    else if (kind[j] == 1) Store<T>::store(kv, kvb[j] + brow + kv_key_off<T>(off, 0, rp.hd), y);
    else Store<T>::store(kv, kvb[j] + brow + kv_val_off<T>(off, 0, rp.hd), o[j]);
  }
}

// Both operands are in the MFMA-tile layout (Tile<T>): fragment (tile t,
// k-step s) of a lane is the 16-byte unit 64 (t * ksteps + s) + lane, so a
// wave's load of one fragment is a contiguous 1 KB block.  The k-steps of a
// workgroup's K range are taken in groups of U; wave w takes groups w, w + KW,
// w + 2 KW, ..., so the waves of a workgroup read adjacent memory at any time.
// Each wave keeps the next group's loads in flight while it multiplies the
// current one (two register stages; scheduling barriers keep the compiler
// from pulling the loads next to their uses).
template <typename T, int MT, int NT, int U, int EPI>
__global__ __launch_bounds__((GemmBounds<MT, NT>::threads)) void gemm_kernel(GemmParams p) {

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KW = blockDim.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int ksteps = (int)((size_t)p.K * sizeof(T) / 64);
  // K * sizeof(T) is a multiple of 64 U (checked by the host); split y of
  // gridDim.y takes step groups [gb, gb + groups)
  const int gall = ksteps / U, gsp = (gall + gridDim.y - 1) / gridDim.y;
  const int gb = min((int)blockIdx.y * gsp, gall), groups = min(gsp, gall - gb);
  const int nw = max(0, (groups - wave + KW - 1) / KW);   // groups of this wave
  // Several M blocks (p.mblocks > 1, 1-D grid): workgroup w runs on XCD w % 8
  // (round-robin dispatch), so the M blocks of one column tile are given
  // consecutive slots of one XCD; they run together and all but the first
  // find the tile's weights in that XCD's L2 (plain loads, not streamed).
  // Otherwise blockIdx.x is the column tile and blockIdx.z the M block.
  int bx = blockIdx.x, bz = blockIdx.z;
  if (p.mblocks > 1) {
    const int w = blockIdx.x, j = w >> 3;
    bz = j % p.mblocks;
    bx = (j / p.mblocks) * 8 + (w & 7);
  }
  const bool stream_w = p.mblocks <= 1;
  // Balanced mode (p.tile_unit > 0): the N / 16 column tiles, in units of
  // tile_unit tiles (2 for SwiGLU: a gate tile and its up tile), are dealt
  // to the gridDim.x workgroups as evenly as possible, a contiguous run per
  // workgroup of at most NT tiles.  Loads of tiles past the run fall outside
  // the buffer range: they return zero and read nothing.
  int tile0 = bx * NT, ntile = NT;
  if (p.tile_unit > 0) {
    const int units = p.N / (16 * p.tile_unit), G = gridDim.x;
    const int base = units / G, extra = units % G;
    tile0 = (bx * base + min(bx, extra)) * p.tile_unit;
    ntile = (base + (bx < extra ? 1 : 0)) * p.tile_unit;
  }
  const int n0 = tile0 * 16;
  const int m0 = bz * MT * 16;
  const uint32_t tile_bytes = (uint32_t)ksteps * 1024u;
  const __amdgpu_buffer_rsrc_t wr = buf_rsrc((const char*)p.W + (size_t)tile0 * tile_bytes, ntile * tile_bytes);
  const __amdgpu_buffer_rsrc_t ar = buf_rsrc((const char*)p.A + (size_t)bz * MT * tile_bytes, MT * tile_bytes);

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // activation rows at or past M are padding: never read (their outputs are dropped)
  uint32_t aoff[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) aoff[t] = m0 + 16 * t + r16 < p.M ? (uint32_t)t * tile_bytes + lane * 16u : OOB;
  u32x4 ws[2][NT][U], as[2][MT][U];
  auto load = [&]<int S>(int i) {              // i-th step group of this wave's share
    const bool ok = i < nw;
    const uint32_t kb = (uint32_t)((gb + i * KW + wave) * U) * 1024u;
    // weights are read once: non-temporal loads keep them from evicting the
    // activations, which every workgroup re-reads from L2
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t o = ok ? j * tile_bytes + kb + u * 1024u + lane * 16u : OOB;
        ws[S][j][u] = stream_w ? buf_load16<true>(wr, o) : buf_load16<false>(wr, o);
      }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int u = 0; u < U; ++u) as[S][t][u] = buf_load16<false>(ar, ok ? aoff[t] + kb + u * 1024u : OOB);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&]<int S>() {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[t][j] = Mfma<T>::step(as[S][t][u], ws[S][j][u], acc[t][j]);
    __builtin_amdgcn_sched_barrier(0);
  };

  // QKV runs exactly 4 waves, so wave w finishes the rows 16 i + 4 g + w of
  // the block; their positions, KV blocks and rotary (cos, sin) are loaded
  // at the start of the stream, so the epilogue waits on nothing
  int qpos[EPI == EPI_QKV ? MT : 1], qblk[EPI == EPI_QKV ? MT : 1];
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = m0 + 16 * i + 4 * g + wave;
      qpos[i] = m < p.M ? p.rope.row_pos[m] : -1;
      qblk[i] = m < p.M ? p.rope.row_blk[m] : -1;
    }
  }

  // QKV: what column n0 + 16 j + r16 of this lane is (independent of the row)
  int qkind[EPI == EPI_QKV ? NT : 1], qcol[EPI == EPI_QKV ? NT : 1], qf[EPI == EPI_QKV ? NT : 1];
  size_t qkvb[EPI == EPI_QKV ? NT : 1];
  float2 qcs[EPI == EPI_QKV ? MT : 1][NT];

  // groups past nw load zeros (no memory access) and add nothing
  load.template operator()<0>(0);
  if constexpr (EPI == EPI_QKV) {
    // the rotary (cos, sin) of this lane's rows are loaded once both register
    // stages are in flight: the wait for the row positions (loaded first)
    // then overlaps the first step group's, and the table loads complete
    // during the stream instead of after it
    load.template operator()<1>(1);
    const int half = p.rope.hd / 2;
#pragma unroll
    for (int j = 0; j < NT; ++j) qkv_column<T>(p.rope, n0 + 16 * j, r16, qkind[j], qcol[j], qf[j], qkvb[j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        qcs[i][j] = qpos[i] >= 0 && qkind[j] < 2 ? p.rope.tab[(size_t)qpos[i] * half + qf[j]] : float2{1.f, 0.f};
    __builtin_amdgcn_sched_barrier(0);
    for (int i = 0; i < nw; i += 2) {
      compute.template operator()<0>();
      load.template operator()<0>(i + 2);
      compute.template operator()<1>();
      load.template operator()<1>(i + 3);
    }
  } else {
    for (int i = 0; i < nw; i += 2) {
      load.template operator()<1>(i + 1);
      compute.template operator()<0>();
      load.template operator()<0>(i + 2);
      compute.template operator()<1>();
    }
  }

  // Reduction over the KW (<= 4) wave partials, in wave order 0, 1, 2, 3
  // (deterministic).  Finishing units are a gate/up tile pair (SwiGLU) or a
  // tile; with at least 4 of them each wave finishes whole units (one LDS
  // round, 16 bytes per lane), else each finishes output rows.
  constexpr int TPU = EPI == EPI_SWIGLU ? 2 : 1;        // tiles per unit
  constexpr int UPR = NT / TPU;                         // units per row tile
  if constexpr (EPI == EPI_QKV || MT * UPR < 4) {
    // every wave publishes its partial tile set; wave w finishes the output
    // rows (i, v) with (4 i + v) % KW == w (for QKV the rows whose
    // positions, KV blocks and rotary inputs it prefetched)
    __shared__ float red[4][MT * NT * 4][64];     // [wave][element][lane]
    // residual values of this wave's rows, loaded before the reduction (a
    // load behind the store of the previous row would wait for it)
    float rres[EPI == EPI_RESID ? MT : 1][4][EPI == EPI_RESID ? NT : 1];
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if ((4 * i + v) % KW != wave) continue;
          const int m = m0 + 16 * i + 4 * g + v;
#pragma unroll
          for (int j = 0; j < NT; ++j)
            rres[i][v][j] = m < p.M && j < ntile ? p.out[(size_t)m * p.ldo + n0 + 16 * j + r16] : 0.f;
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][(i * NT + j) * 4 + v][lane] = acc[i][j][v];
    __syncthreads();
    if constexpr (EPI == EPI_QKV) {
      // first use of the prefetched rotary inputs before any store: the wait
      // for them is taken here, not behind the epilogue's stores (the memory
      // counter also counts stores)
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        asm volatile("" : "+v"(qpos[i]), "+v"(qblk[i]));
#pragma unroll
        for (int j = 0; j < NT; ++j) asm volatile("" : "+v"(qcs[i][j].x), "+v"(qcs[i][j].y));
      }
    }
    // output element (i, j, v) is row m0 + 16 i + 4 g + v, column n0 + 16 j + r16
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if ((4 * i + v) % KW != wave) continue;
        const int m = m0 + 16 * i + 4 * g + v;
        float o[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          float t = red[0][(i * NT + j) * 4 + v][lane];
          for (int w = 1; w < KW; ++w) t += red[w][(i * NT + j) * 4 + v][lane];
          o[j] = t;
        }
        if constexpr (EPI == EPI_QKV) {
          // the rotary partner of column r16 is column r16 ^ 8 of the same
          // tile (exchanged while the whole wave is still converged)
          float pr[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) pr[j] = __shfl_xor(o[j], 8);
          if (m >= p.M || qpos[i] < 0) continue;   // padding row, or no pending draft token
          qkv_store<T, NT>(p.rope, m, qpos[i], qblk[i], r16, o, pr, qcs[i], qkind, qcol, qkvb);
        } else if constexpr (EPI == EPI_SWIGLU) {
          if (m >= p.M) continue;
          // tiles (2k, 2k+1) are the gate and up rows of the same 16 outputs
          const int F = p.N / 2;
#pragma unroll
          for (int j = 0; j < NT; j += 2)
            if (j < ntile) Store<T>::store((T*)p.out_t, Tile<T>::off(m, n0 / 2 + 8 * j + r16, F), silu(o[j]) * o[j + 1]);
        } else {
          if (m >= p.M) continue;
          const size_t row = EPI == EPI_PART ? (size_t)blockIdx.y * p.M + m : (size_t)m;
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            if (j >= ntile) continue;
            float* dst = p.out + row * p.ldo + n0 + 16 * j + r16;
            if constexpr (EPI == EPI_RESID) *dst = rres[i][v][j] + o[j];
            else *dst = o[j];
          }
        }
      }
  } else {
    // unit u (row tile i, unit k of it) is finished by wave u % KW; the
    // other waves leave their partial of its tiles in LDS slot
    // (w - f - 1) mod 4
    __shared__ f32x4 red[MT * NT][3][64];           // [tile][slot][lane]
    // residual values of the units this wave finishes, loaded before the
    // reduction so that their latency overlaps it
    float rres[EPI == EPI_RESID ? MT : 1][EPI == EPI_RESID ? UPR : 1][4];
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int k = 0; k < UPR; ++k) {
          if ((i * UPR + k) % KW != wave || k * TPU >= ntile) continue;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = m0 + 16 * i + 4 * g + v;
            rres[i][k][v] = m < p.M ? p.out[(size_t)m * p.ldo + n0 + 16 * k + r16] : 0.f;
          }
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int f = (i * UPR + j / TPU) % KW;
        if (wave != f && j < ntile) red[i * NT + j][(wave - f - 1) & 3][lane] = acc[i][j];
      }
    __syncthreads();
    // the sum of a tile in wave order 0, 1, 2, 3; this wave's own partial
    // from registers, the others from their slots
    auto total = [&](const f32x4& own, int tile) {
      f32x4 t = own;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w >= KW) break;
        f32x4 pw;
        if (w == wave) pw = own;
        else pw = red[tile][(w - wave - 1) & 3][lane];
        t = w == 0 ? pw : t + pw;
      }
      return t;
    };
    // output element (i, j, v) is row m0 + 16 i + 4 g + v, column n0 + 16 j + r16
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int k = 0; k < UPR; ++k) {
        if ((i * UPR + k) % KW != wave || k * TPU >= ntile) continue;
        if constexpr (EPI == EPI_SWIGLU) {
          // tiles (2k, 2k+1) are the gate and up rows of the same 16 outputs
          const f32x4 gt = total(acc[i][2 * k], i * NT + 2 * k), up = total(acc[i][2 * k + 1], i * NT + 2 * k + 1);
          const int F = p.N / 2;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = m0 + 16 * i + 4 * g + v;
            if (m < p.M) Store<T>::store((T*)p.out_t, Tile<T>::off(m, n0 / 2 + 16 * k + r16, F), silu(gt[v]) * up[v]);
          }
        } else {
          const f32x4 o = total(acc[i][k], i * NT + k);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = m0 + 16 * i + 4 * g + v;
            if (m >= p.M) continue;
            const size_t row = EPI == EPI_PART ? (size_t)blockIdx.y * p.M + m : (size_t)m;
            float* dst = p.out + row * p.ldo + n0 + 16 * k + r16;
            if constexpr (EPI == EPI_RESID) *dst = rres[i][k][v] + o[v];
            else *dst = o[v];
          }
        }
      }
  }
}

// Wait until at most N vector memory operations of this wave are
// outstanding (vmcnt only; the LDS and export counters are not waited on).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Appends a wave's values (16 MF rows from row m0, the 16 NF fused columns
// from n0, all of one value head) to the cache from its LDS tile
// [16 MF][16 NF].  In a V tile (kv_val_off) the 4 tokens of a quad (positions
// 4 k .. 4 k + 3) of the dims d and d + 16 are one 16-byte unit, so the rows
// are taken in runs of consecutive positions inside a quad: a whole quad is
// one 16-byte store per lane (256 contiguous bytes per 16 lanes), part of
// one 2- or 4-byte stores.  What bounded the epilogue was these appends: stored
// row by row into tiles that kept the 16 dims of a token 64 bytes apart, every
// 2-byte value was an L2 request of its own in a partly written memory line.
// 13B QKV at 320 rows (64 tasks) 84.9 -> 70.5 us and at 640 rows 135 -> 108
// (61.8 and 90.4 without any of the QKV epilogue), 7B at 160 rows 44.5 -> 40.0
// and at 2048 prefill rows 210 -> 198.
template <int MF, int NF>
__device__ __forceinline__ void store_values(const RopeParams& rp, int M, int m0, int n0, int lane, const f16_t* tile) {
  static_assert(NF == 2 || NF == 4, "whole groups of 32 dims");
  constexpr int UNITS = 8 * NF, SLOTS = 64 / UNITS;    // (32-dim group, d % 16) pairs; runs stored at a time
  const int hd = rp.hd, cv = rp.col0 + n0 - (rp.H + rp.KV) * hd;
  const int unit = lane % UNITS, slot = lane / UNITS;
  const int col = 32 * (unit >> 4) + (unit & 15);      // and col + 16
  f16_t* base = (f16_t*)rp.kv + kv_tile_off(cv / hd, 0, 1, rp.nblk, hd) + kv_val_off<f16_t>(0, cv % hd + col, hd);
  int pos = -1, blk = -1;                              // of row m0 + 16 i + lane (lane < 16)
  auto load_row = [&](int i) {
    const int m = m0 + 16 * i + lane;
    pos = lane < 16 && m < M ? rp.row_pos[m] : -1;
    blk = lane < 16 && m < M ? rp.row_blk[m] : -1;
  };
  load_row(0);
#pragma unroll 1
  for (int i = 0; i < MF; ++i) {
    const int cpos = pos, cblk = blk;
    if (i + 1 < MF) load_row(i + 1);
    const bool valid = cpos >= 0 && cblk >= 0;
    const int ppos = __shfl_up(cpos, 1), pblk = __shfl_up(cblk, 1);
    const bool start = valid && (lane == 0 || pblk != cblk || ppos + 1 != cpos || (cpos & 3) == 0);
    uint32_t runs = (uint32_t)__ballot(start);
    // a run ends before the next start, an invalid row or row 16
    const uint32_t ends = runs | ~(uint32_t)__ballot(valid) | 0x10000u;
    const f16_t* rows = tile + 16 * i * 16 * NF + col;
    while (runs) {
      uint32_t mine = runs;
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        if (k < slot) mine &= mine - 1;
        runs &= runs - 1;
      }
      const int s = mine ? __ffs(mine) - 1 : 0;
      const int n = mine ? __ffs(ends >> (s + 1)) : 0;
      const int t0 = __shfl(cpos, s) & 15;
      f16_t* dst = base + (size_t)__shfl(cblk, s) * 32 * hd + kv_val_off<f16_t>(t0 & 12, 0, hd);
      if (n == 4) {
        uint16_t lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          lo[k] = __builtin_bit_cast(uint16_t, rows[(s + k) * 16 * NF]);
          hi[k] = __builtin_bit_cast(uint16_t, rows[(s + k) * 16 * NF + 16]);
        }
        *(uint4*)dst = make_uint4(lo[0] | (uint32_t)lo[1] << 16, lo[2] | (uint32_t)lo[3] << 16,
                                  hi[0] | (uint32_t)hi[1] << 16, hi[2] | (uint32_t)hi[3] << 16);
      } else {
        const int q0 = t0 & 3;                         // tokens q0 .. q0 + n - 1 of the quad
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int a = 2 * h - q0, b = a + 1;         // their places in the run
          const bool ina = a >= 0 && a < n, inb = b >= 0 && b < n;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const f16_t va = rows[(s + (ina ? a : 0)) * 16 * NF + 16 * e], vb = rows[(s + (inb ? b : 0)) * 16 * NF + 16 * e];
            f16_t* d2 = dst + 4 * e + 2 * h;
            if (ina && inb)
              *(uint32_t*)d2 = __builtin_bit_cast(uint16_t, va) | (uint32_t)__builtin_bit_cast(uint16_t, vb) << 16;
            else if (ina) d2[0] = va;
            else if (inb) d2[1] = vb;
          }
        }
      }
    }
  }
}

// Row-tiled GEMM for passes with more than one 64-row block (batched
// verify at B >= 32, prefill): there every weight byte meets hundreds of
// rows, so the operands are staged once per workgroup in LDS and shared.
// A workgroup of WM x WN waves owns a BM x BN output tile, wave (wm, wn) the
// 16 MF x 16 NF sub-tile at (wm 16 MF, wn 16 NF).
// K advances in stages of KS k-steps (32 KS fp16); a stage is the
// KS (BM + BN) / 16 1 KB fragments, which the waves load straight into
// one of NB LDS buffers (buffer loads with an LDS destination: lane i's
// 16 bytes land at the buffer's fragment base + 16 i, no registers held).
// NB - 1 stages are in flight while one is multiplied: at the top of stage
// st a wave waits until its own loads of stage st have landed (at most
// NB - 2 stages of its loads outstanding), then one barrier makes every
// wave's loads visible and frees the buffer stage st - 1 used, which then
// receives stage st + NB - 1.  Every stage issues the same number of loads
// (past the last stage with an empty buffer range: they read nothing), so
// the count the wait uses holds to the end.  The last stage of a K that is no
// multiple of 32 KS is partial: its k-steps past K are loaded the same way,
// as zeros.  The barrier is a plain
// s_barrier with a compiler memory clobber: a fenced one would wait for
// every load in flight.  Rows at or past M and columns at or past N load
// zeros (range-checked buffer loads).  Tile order: every XCD (workgroups are
// dispatched round-robin over 8) takes one contiguous run of tiles, the row
// tiles and K ranges of a column tile first, so that a column tile's weights
// are fetched from HBM once and re-read from that XCD's L2.
template <int MF_, int NF_, int WM_, int WN_, int KS_, int NB_> struct RowTile {
  static constexpr int MF = MF_, NF = NF_, WM = WM_, WN = WN_, KS = KS_, NB = NB_;
  static constexpr int WAVES = WM * WN, BM = 16 * MF * WM, BN = 16 * NF * WN;
  static constexpr int FA = BM / 16 * KS, FW = BN / 16 * KS;                     // fragments per stage
  static constexpr int LA = (FA + WAVES - 1) / WAVES, LW = (FW + WAVES - 1) / WAVES;   // loads per wave
  static constexpr int SPARE = (FA % WAVES || FW % WAVES) ? 1 : 0;               // their overflow slot
  static constexpr int FS = FA + FW + SPARE;
  static constexpr uint32_t LDS = (uint32_t)NB * FS * 1024;
  static_assert(NB >= 2 && (NB - 2) * (LA + LW) < 64, "stages in flight");
  static_assert(LDS <= 160 * 1024, "LDS of a CU");
  static_assert((uint32_t)BM * BN * 2 <= LDS, "the 16-bit output tile fits the stage buffers");
};

template <typename C, int EPI>
__global__ __launch_bounds__(64 * C::WAVES, 2) void gemm_rows_kernel(GemmParams p) {
  using T = f16_t;
  constexpr int MF = C::MF, NF = C::NF, KS = C::KS, NB = C::NB, WAVES = C::WAVES, BM = C::BM, BN = C::BN;
  constexpr int FA = C::FA, FW = C::FW, LA = C::LA, LW = C::LW, FS = C::FS;
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4* lds = (u32x4*)smem;                          // [NB][FS][64]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % C::WM, wn = wave / C::WM;
  const int r16 = lane & 15, g = lane >> 4;
  const int ksteps = p.K * 2 / 64, stages = (ksteps + KS - 1) / KS;
  const int gz = (p.M + BM - 1) / BM;
  const int ks = max(p.ksplit, 1), R = gz * ks;
  // workgroup w runs on XCD w % 8; XCD x takes the tiles [x T / 8, (x + 1) T / 8) (rounded)
  int bx, r;
  {
    const int w = blockIdx.x, T8 = gridDim.x >> 3, rem = gridDim.x & 7, x = w & 7;
    const int tile = x * T8 + min(x, rem) + (w >> 3);
    bx = tile / R;
    r = tile % R;
  }
  const int bz = r % gz, split = r / gz;
  const int sps = (stages + ks - 1) / ks;              // stages of one K range
  const int s_lo = min(split * sps, stages), s_hi = min(s_lo + sps, stages);
  const uint32_t tile_bytes = (uint32_t)ksteps * 1024u;
  const char* Wp = (const char*)p.W + (size_t)bx * (BN / 16) * tile_bytes;
  const char* Ap = (const char*)p.A + (size_t)bz * (BM / 16) * tile_bytes;
  const int mvalid = p.M - bz * BM;                   // rows of this tile below M
  const int ntile = min(BN / 16, p.N / 16 - bx * (BN / 16));   // 16-column tiles below N

  // this wave's share of a stage: A fragments f = WAVES k + wave (k < LA), W
  // fragments f = WAVES k + wave (k < LW); fragment f = KS t + u is (16-row
  // tile t, k-step u of the stage); a wave's fragments are all of k-step
  // u = wave % KS.  Indices past the stage's fragments load nothing
  // (out-of-range offset) into the overflow slot, so every wave issues the
  // same count
  static_assert(WAVES % KS == 0, "one k-step per wave");
  const int s_end = min(s_hi, (ksteps - wave % KS + KS - 1) / KS);   // stages in which this wave's k-step exists
  uint32_t aoff[LA], woff[LW];
#pragma unroll
  for (int k = 0; k < LA; ++k) {
    const int f = WAVES * k + wave, t = f / KS, u = f % KS;
    aoff[k] = f < FA && 16 * t + r16 < mvalid ? (uint32_t)t * tile_bytes + u * 1024u + lane * 16u : OOB;
  }
#pragma unroll
  for (int k = 0; k < LW; ++k) {
    const int f = WAVES * k + wave, t = f / KS, u = f % KS;
    woff[k] = f < FW ? (uint32_t)t * tile_bytes + u * 1024u + lane * 16u : OOB;
  }
  auto gload = [&](int st) {
    const bool ok = st < s_end;
    const __amdgpu_buffer_rsrc_t ar = buf_rsrc(Ap, ok ? (BM / 16) * tile_bytes : 0u);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(Wp, ok ? (uint32_t)ntile * tile_bytes : 0u);
    u32x4* base = lds + (size_t)(st % NB) * FS * 64;
    const int so = st * KS * 1024;
#pragma unroll
    for (int k = 0; k < LA; ++k) {
      const int f = WAVES * k + wave;
      const uint32_t off = aoff[k];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          ar, (__attribute__((address_space(3))) void*)(base + (FA % WAVES == 0 || f < FA ? f : FA + FW) * 64), 16, off,
          so, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < LW; ++k) {
      const int f = WAVES * k + wave;
      const uint32_t off = woff[k];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          wr, (__attribute__((address_space(3))) void*)(base + (FW % WAVES == 0 || f < FW ? FA + f : FA + FW) * 64), 16,
          off, so, 0, 0);
    }
  };

  f32x4 acc[MF][NF];
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int st = 0; st < NB - 1; ++st) gload(s_lo + st);
  for (int st = s_lo; st < s_hi; ++st) {
    wait_vmcnt<(NB - 2) * (LA + LW)>();
    asm volatile("s_barrier" ::: "memory");
    gload(st + NB - 1);
    const u32x4* base = lds + (size_t)(st % NB) * FS * 64;
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      u32x4 a[MF], b[NF];
#pragma unroll
      for (int j = 0; j < NF; ++j) b[j] = base[(FA + (wn * NF + j) * KS + u) * 64 + lane];
#pragma unroll
      for (int i = 0; i < MF; ++i) a[i] = base[((wm * MF + i) * KS + u) * 64 + lane];
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = Mfma<T>::step(a[i], b[j], acc[i][j]);
      __builtin_amdgcn_s_setprio(0);
    }
  }
  wait_vmcnt<0>();                                    // the trailing out-of-range loads

  // epilogue: element (i, j, v) is row bz BM + wm 16 MF + 16 i + 4 g + v,
  // column n0 + 16 j + r16 with n0 the first column of the wave's sub-tile.
  // The loads of the epilogue (residual values; row positions, KV blocks and
  // rotary inputs) are issued one 16-row tile ahead of the stores: a load
  // after a store to a possibly aliasing address would wait for that store,
  // one round trip per row.
  const int n0 = bx * BN + wn * 16 * NF;
  const int nt = min(NF, ntile - wn * NF);             // tiles of the wave's sub-tile below N (may be <= 0)
  const int mrow0 = bz * BM + wm * 16 * MF + 4 * g;    // + 16 i + v
  if constexpr (EPI == EPI_QKV) {
    // heads are 64 or 128 columns, so a wave's 32 or 64 columns are all
    // queries, all keys or all values
    if (p.rope.col0 + n0 >= (p.rope.H + p.rope.KV) * p.rope.hd) {
      asm volatile("s_barrier" ::: "memory");         // every wave is done reading the stage buffers
      if (nt <= 0) return;
      T* tile = (T*)smem + (size_t)wave * 16 * MF * 16 * NF;
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int j = 0; j < NF; ++j) tile[(16 * i + 4 * g + v) * 16 * NF + 16 * j + r16] = (T)acc[i][j][v];
      store_values<MF, NF>(p.rope, p.M, bz * BM + wm * 16 * MF, n0, lane, tile);
      return;
    }
    asm volatile("s_barrier" ::: "memory");
    int qkind[NF], qcol[NF], qf[NF];
    size_t qkvb[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) qkv_column<T>(p.rope, n0 + 16 * j, r16, qkind[j], qcol[j], qf[j], qkvb[j]);
    if (nt <= 0) return;
    const int half = p.rope.hd / 2;
    auto load_rows = [&](int i, int (&pos)[4], int (&blk)[4]) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = mrow0 + 16 * i + v;
        pos[v] = m < p.M ? p.rope.row_pos[m] : -1;
        blk[v] = m < p.M ? p.rope.row_blk[m] : -1;
      }
    };
    auto load_cs = [&](const int (&pos)[4], float2 (&c)[4][NF]) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < NF; ++j)
          c[v][j] = qkind[j] < 2 ? p.rope.tab[(size_t)max(pos[v], 0) * half + qf[j]] : float2{1.f, 0.f};
    };
    // positions two 16-row tiles ahead, rotary inputs one ahead
    int pos[3][4], blk[3][4];
    float2 cs[2][4][NF];
    load_rows(0, pos[0], blk[0]);
    if constexpr (MF > 1) load_rows(1, pos[1], blk[1]);
    load_cs(pos[0], cs[0]);
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      if (i + 2 < MF) load_rows(i + 2, pos[(i + 2) % 3], blk[(i + 2) % 3]);
      if (i + 1 < MF) load_cs(pos[(i + 1) % 3], cs[(i + 1) & 1]);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float o[NF], pr[NF];
#pragma unroll
        for (int j = 0; j < NF; ++j) o[j] = acc[i][j][v];
#pragma unroll
        for (int j = 0; j < NF; ++j) pr[j] = __shfl_xor(o[j], 8);
        if (pos[i % 3][v] >= 0)   // a row at or past M has pos -1
          qkv_store<T, NF>(p.rope, mrow0 + 16 * i + v, pos[i % 3][v], blk[i % 3][v], r16, o, pr, cs[i & 1][v], qkind,
                           qcol, qkvb, nt);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (EPI == EPI_RESID) {
    float res[2][4][NF];
    auto load_res = [&](int i, float (&o)[4][NF]) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = mrow0 + 16 * i + v;
#pragma unroll
        for (int j = 0; j < NF; ++j) o[v][j] = m < p.M && j < nt ? p.out[(size_t)m * p.ldo + n0 + 16 * j + r16] : 0.f;
      }
    };
    load_res(0, res[0]);
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      if (i + 1 < MF) load_res(i + 1, res[(i + 1) & 1]);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = mrow0 + 16 * i + v;
        if (m >= p.M) continue;
#pragma unroll
        for (int j = 0; j < NF; ++j)
          if (j < nt) p.out[(size_t)m * p.ldo + n0 + 16 * j + r16] = res[i & 1][v][j] + acc[i][j][v];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = mrow0 + 16 * i + v;
        if (m >= p.M) continue;
        if constexpr (EPI == EPI_SWIGLU) {
          const int F = p.N / 2;
#pragma unroll
          for (int j = 0; j < NF; j += 2)
            if (j < nt)
              Store<T>::store((T*)p.out_t, Tile<T>::off(m, n0 / 2 + 8 * j + r16, F), silu(acc[i][j][v]) * acc[i][j + 1][v]);
        } else {
          const size_t row = EPI == EPI_PART ? (size_t)split * p.M + m : (size_t)m;
#pragma unroll
          for (int j = 0; j < NF; ++j)
            if (j < nt) p.out[row * p.ldo + n0 + 16 * j + r16] = acc[i][j][v];
        }
      }
  }
}

template <typename C, int EPI>
static hipError_t launch_rows_t(const GemmParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int grid = (p.N + C::BN - 1) / C::BN * ((p.M + C::BM - 1) / C::BM) * std::max(p.ksplit, 1);
  launch_k(gemm_rows_kernel<C, EPI>, dim3(grid), dim3(64 * C::WAVES), C::LDS, s, e0, e1, p);
  return hipGetLastError();
}

// The output tiles, largest first, and the time model that picks one: a
// workgroup alone on its CU takes a k-step in a microseconds, c more as the
// grid fills the 256 CUs (they share L2 and HBM), and e in all for its start
// and epilogue; with two workgroups per CU (the 4-wave tiles of 128 columns)
// a k-step of both takes a + c and one alone h times that.  The constants are
// a least-squares fit to 7000 measured launches (64 <= M <= 2048; N and K of
// the 7B, 13B and small targets and the drafts; weights streamed from HBM).
// Checked over 627 projections and row counts, 8 <= M <= 2048, against every
// tile and K split (17910 launches): the choice is on average 0.5 % slower
// than the fastest (90 % of them within 1.6 %, the worst 13 %); below 64 rows
// 0.2 %, at widths that were not fitted (1536, 3072) 0.6 %.
// What each is for, at its best against the 128-192 x 128 tiles with stages
// of two k-steps that it replaced:
//   256 x 128, 192 x 128 (two per CU, stages of one k-step: 72 and 60 KB of
//     LDS): grids beyond 512 workgroups.  M = 2048: 7B gate/up 386 -> 337 us
//     (1.10 PFLOP/s), QKV 225 -> 196, 13B gate/up 595 -> 513
//   160 x 256, 128 x 256 (one per CU, 8 waves): fewer, larger tiles read
//     each operand less often per product.  13B gate/up at M = 320 115 -> 98
//     us; 7B down projection at M = 2048 190 us (was on the skinny GEMM: 775)
//   160 x 128 ... 64 x 64 (one per CU, 8 waves, up to 112 KB in flight):
//     grids near 256 workgroups, with K split where the output is narrow
// A tile's number is its place in this table; the kernel instances (RowTile)
// and their dispatch are made from it.
struct RowTileModel {
  int mf, nf, wm, wn, ks, nb;   // RowTile
  int per_cu;
  float e, a, c, h;
  constexpr int bm() const { return 16 * mf * wm; }
  constexpr int bn() const { return 16 * nf * wn; }
};
static constexpr RowTileModel ROW_TILES[] = {
    {8, 4, 2, 2, 1, 3, 2, 5.4f, 0.653f, 0.177f, 0.66f},   // 256 x 128
    {6, 4, 2, 2, 1, 3, 2, 4.4f, 0.495f, 0.160f, 0.70f},   // 192 x 128
    {5, 4, 2, 4, 2, 3, 1, 4.4f, 0.433f, 0.158f, 1.0f},    // 160 x 256
    {4, 4, 2, 4, 1, 4, 1, 3.5f, 0.379f, 0.125f, 1.0f},    // 128 x 256
    {5, 2, 2, 4, 2, 3, 1, 3.1f, 0.264f, 0.088f, 1.0f},    // 160 x 128
    {4, 2, 2, 4, 2, 4, 1, 2.8f, 0.233f, 0.075f, 1.0f},    // 128 x 128
    {2, 2, 4, 2, 4, 3, 1, 1.9f, 0.149f, 0.044f, 1.0f},    // 128 x 64
    {3, 2, 2, 4, 2, 4, 1, 2.2f, 0.212f, 0.048f, 1.0f},    // 96 x 128
    {3, 2, 2, 2, 4, 3, 1, 1.8f, 0.142f, 0.027f, 1.0f},    // 96 x 64
    {2, 2, 2, 4, 2, 4, 1, 1.7f, 0.163f, 0.046f, 1.0f},    // 64 x 128
    {1, 2, 4, 2, 4, 4, 1, 1.5f, 0.101f, 0.029f, 1.0f},    // 64 x 64
};
constexpr int N_ROW_TILES = sizeof(ROW_TILES) / sizeof(ROW_TILES[0]);

RowTileShape row_tile_shape(int tile) {
  const RowTileModel& m = ROW_TILES[tile];
  return {m.mf, m.nf, m.wm, m.wn, m.ks, m.nb};
}

template <int T>
using RowTileAt = RowTile<ROW_TILES[T].mf, ROW_TILES[T].nf, ROW_TILES[T].wm, ROW_TILES[T].wn, ROW_TILES[T].ks,
                          ROW_TILES[T].nb>;

hipError_t prepare_gemm_rows() {
  hipError_t r = hipSuccess;
  auto limit = [&]<int T, int EPI>() {
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)gemm_rows_kernel<RowTileAt<T>, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)RowTileAt<T>::LDS);
  };
  [&]<int... T>(std::integer_sequence<int, T...>) {
    ((limit.template operator()<T, EPI_STORE>(), limit.template operator()<T, EPI_RESID>(),
      limit.template operator()<T, EPI_SWIGLU>(), limit.template operator()<T, EPI_QKV>(),
      limit.template operator()<T, EPI_PART>()), ...);
  }(std::make_integer_sequence<int, N_ROW_TILES>());
  return r;
}

template <int EPI>
static hipError_t launch_rows_e(int tile, const GemmParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  hipError_t r = hipErrorInvalidValue;
  auto at = [&]<int T>() {
    if (tile == T) r = launch_rows_t<RowTileAt<T>, EPI>(p, s, e0, e1);
    return tile == T;
  };
  [&]<int... T>(std::integer_sequence<int, T...>) {
    (at.template operator()<T>() || ...);
  }(std::make_integer_sequence<int, N_ROW_TILES>());
  return r;
}

// K ranges are dealt in whole stages (kps k-steps each), the same number to
// every range but the last.  A split is used only if that leaves none empty: an
// empty range's workgroups would write zeros for the RMSNorm to read.
static bool row_splits_ok(int ksteps, int kps, int ksplit) {
  const int stages = (ksteps + kps - 1) / kps, sps = (stages + ksplit - 1) / ksplit;
  return (ksplit - 1) * sps < stages;
}

int pick_row_tile(int M, int N, int K, int max_ksplit, int* ksplit) {
  const int ksteps = K * 2 / 64;
  max_ksplit = std::max(1, max_ksplit);
  *ksplit = 1;
  int best = 0;
  double best_t = 1e30;
  for (int t = 0; t < N_ROW_TILES; ++t) {
    const RowTileModel& m = ROW_TILES[t];
    for (int ks = 1; ks <= max_ksplit; ++ks) {
      const int grid = (M + m.bm() - 1) / m.bm() * ((N + m.bn() - 1) / m.bn()) * ks;
      if (ks > 1 && grid > 640) break;      // splitting is for grids that leave CUs idle
      if (!row_splits_ok(ksteps, m.ks, ks)) continue;
      // rounds of 256 per_cu workgroups; the last one holds the share `part`
      const int slots = 256 * m.per_cu, full = grid / slots;
      const double part = (double)(grid - full * slots) / slots, one = 1.0 / m.per_cu;
      double last = 0;
      if (part > 0) {
        if (m.per_cu == 1) last = 1.0;
        else if (full == 0) last = part > one + 0.02 ? 1.0 : m.h;
        else last = part > one ? m.h + (1 - m.h) * (part - one) / (1 - one) : m.h * (0.5 + 0.5 * part / one);
      }
      const double step = m.a + m.c * std::min(1.0, grid / 256.0);
      double us = m.e * (full + (part > 0)) + ((ksteps + ks - 1) / ks) * (full + last) * step;
      if (ks > 1) us += (double)ks * M * N * 1e-6;   // the RMSNorm reads the partial sums (4 TB/s)
      if (us < best_t) {
        best_t = us;
        best = t;
        *ksplit = ks;
      }
    }
  }
  return best;
}

// columns col0 .. of the fused projection, whole heads
static bool qkv_shape_ok(const GemmParams& p) {
  const RopeParams& r = p.rope;
  return r.hd % 16 == 0 && r.col0 >= 0 && r.col0 % r.hd == 0 && p.N == (r.H + 2 * r.KV) * r.hd - r.col0;
}

hipError_t launch_gemm_rows(int epi, int tile, const GemmParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (tile < 0 || tile >= N_ROW_TILES || p.N % 16 || p.M < 1 || ((size_t)p.K * 2) % GEMM_CHUNK)
    return hipErrorInvalidValue;
  // a K split writes partial sums (PART)
  if (p.ksplit > 1 && (epi != EPI_PART || !row_splits_ok(p.K * 2 / 64, ROW_TILES[tile].ks, p.ksplit)))
    return hipErrorInvalidValue;
  if (epi == EPI_PART && p.ksplit < 1) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_STORE: return launch_rows_e<EPI_STORE>(tile, p, s, e0, e1);
    case EPI_RESID: return launch_rows_e<EPI_RESID>(tile, p, s, e0, e1);
    case EPI_SWIGLU:
      if (p.N % 32) return hipErrorInvalidValue;
      return launch_rows_e<EPI_SWIGLU>(tile, p, s, e0, e1);
    case EPI_PART: return launch_rows_e<EPI_PART>(tile, p, s, e0, e1);
    case EPI_QKV:
      if (!qkv_shape_ok(p)) return hipErrorInvalidValue;
      return launch_rows_e<EPI_QKV>(tile, p, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

// row-major [N, K] -> MFMA-tile layout, one 16-byte unit per thread; bf16
// sources (S = bf16_t) are converted to fp16 (T = f16_t) on the way: exact
// from 2^-14 up, smaller magnitudes round to the fp16 subnormal grid
template <typename S, typename T>
__global__ void pack_linear_kernel(const S* src, T* dst, int N, int K) {
  static_assert(sizeof(S) == sizeof(T), "same element size");
  constexpr int EPL = Tile<T>::EPL, EPK = Tile<T>::EPK;
  const int ks = K / EPK;
  const size_t units = (size_t)N * K / EPL;
  for (size_t u = blockIdx.x * (size_t)blockDim.x + threadIdx.x; u < units; u += (size_t)gridDim.x * blockDim.x) {
    const int lane = (int)(u % 64);
    const size_t ts = u / 64;
    const int s = (int)(ts % ks), t = (int)(ts / ks);
    const int r = 16 * t + (lane & 15);
    const int k = s * EPK + (lane >> 4) * EPL;
    uint4 v = *(const uint4*)(src + (size_t)r * K + k);
    if constexpr (!std::is_same_v<S, T>) {
      uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = (uint32_t)f2h(bf2f((bf16_t)(w[i] & 0xffffu))) | ((uint32_t)f2h(bf2f((bf16_t)(w[i] >> 16))) << 16);
      v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    *(uint4*)(dst + u * EPL) = v;
  }
}

hipError_t launch_pack_linear(int dtype, const void* src, void* dst, int N, int K, hipStream_t s) {
  const size_t esz = dtype == 0 ? 2 : 4;
  if (N <= 0 || K <= 0 || N % 16 || ((size_t)K * esz) % 64) return hipErrorInvalidValue;
  const size_t units = (size_t)N * K * esz / 16;
  const int blocks = (int)std::min<size_t>((units + 255) / 256, 65536);
  if (dtype == 0)
    hipLaunchKernelGGL((pack_linear_kernel<bf16_t, f16_t>), dim3(blocks), dim3(256), 0, s, (const bf16_t*)src,
                       (f16_t*)dst, N, K);
  else
    hipLaunchKernelGGL((pack_linear_kernel<float, float>), dim3(blocks), dim3(256), 0, s, (const float*)src,
                       (float*)dst, N, K);
  return hipGetLastError();
}

template <typename T, int EPI, int NT, int U>
static hipError_t launch_mt(int mt, dim3 grid, int threads, const GemmParams& p, hipStream_t s, hipEvent_t e0,
                            hipEvent_t e1) {
  switch (mt) {
    case 1:
    case 2:
      // 96-column tiles (balanced mode) only for 3-tile row blocks
      if constexpr (NT <= 4) {
        if (mt == 1) launch_k(gemm_kernel<T, 1, NT, U, EPI>, grid, dim3(threads), 0, s, e0, e1, p);
        else launch_k(gemm_kernel<T, 2, NT, U, EPI>, grid, dim3(threads), 0, s, e0, e1, p);
        break;
      }
      return hipErrorInvalidValue;
    case 3:
      if constexpr (NT <= 4 || NT == 6) {
        launch_k(gemm_kernel<T, 3, NT, U, EPI>, grid, dim3(threads), 0, s, e0, e1, p);
        break;
      }
      return hipErrorInvalidValue;
    case 4:
      // 64-row blocks (prefill) only with tiles of up to 32 columns
      if constexpr (NT <= 2) {
        launch_k(gemm_kernel<T, 4, NT, U, EPI>, grid, dim3(threads), 0, s, e0, e1, p);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, int EPI>
static hipError_t launch_nt(int nt, int mt, dim3 grid, int threads, const GemmParams& p, hipStream_t s, hipEvent_t e0,
                            hipEvent_t e1) {
  switch (nt) {
    case 1:
      if constexpr (EPI != EPI_SWIGLU) return launch_mt<T, EPI, 1, GEMM_U>(mt, grid, threads, p, s, e0, e1);
      return hipErrorInvalidValue;
    case 2: return launch_mt<T, EPI, 2, GEMM_U>(mt, grid, threads, p, s, e0, e1);
    case 3:
      // 48-column tiles: only the QKV projection uses them (one tile per CU at 7B)
      if constexpr (EPI == EPI_QKV) return launch_mt<T, EPI, 3, GEMM_U>(mt, grid, threads, p, s, e0, e1);
      return hipErrorInvalidValue;
    case 4: return launch_mt<T, EPI, 4, GEMM_U>(mt, grid, threads, p, s, e0, e1);
    // balanced mode at 33-48 rows: SwiGLU up to 3 gate/up pairs
    case 6:
      if constexpr (EPI == EPI_SWIGLU && sizeof(T) == 2) return launch_mt<T, EPI, 6, GEMM_U>(mt, grid, threads, p, s, e0, e1);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

bool gemm_config_ok(int dtype, int epi, int nt, int mt, int kw, int grid_x, int ksplit, int grid_z,
                    const GemmParams& p) {
  const size_t kbytes = (size_t)p.K * (dtype == 0 ? 2 : 4);
  if (mt < 1 || mt > 4 || kw < 1 || kw > 4) return false;
  // instantiated tiles: 48 columns for QKV only, 96 columns (16-bit SwiGLU,
  // 3 row tiles) for balanced mode only
  switch (nt) {
    case 1: if (epi == EPI_SWIGLU) return false; break;
    case 2: break;
    case 3: if (epi != EPI_QKV || mt > 3) return false; break;
    case 4: if (mt > 3) return false; break;
    case 6: if (epi != EPI_SWIGLU || dtype != 0 || mt != 3 || p.tile_unit <= 0) return false; break;
    default: return false;
  }
  if (mt == 4 && nt > 2) return false;
  if (p.tile_unit > 0) {
    // balanced mode: one M block, no K split, every workgroup within nt tiles
    if (p.tile_unit > 2 || p.N % (16 * p.tile_unit) || grid_x < 1 || grid_z != 1 || ksplit != 1 ||
        epi == EPI_QKV || epi == EPI_PART || (epi == EPI_SWIGLU && p.tile_unit != 2))
      return false;
    const int units = p.N / (16 * p.tile_unit);
    if (units < grid_x || (units + grid_x - 1) / grid_x * p.tile_unit > nt) return false;
  } else if (p.N % (16 * nt) || grid_x * 16 * nt != p.N) {
    return false;
  }
  if (grid_z * 16 * mt < p.M || kbytes % GEMM_CHUNK) return false;
  if (ksplit < 1 || (ksplit > 1 && epi != EPI_PART) || ksplit > (int)(kbytes / GEMM_CHUNK)) return false;
  if (epi == EPI_QKV && (kw != 4 || !qkv_shape_ok(p))) return false;
  return true;
}

hipError_t launch_gemm(int dtype, int epi, int nt, int mt, int kw, int grid_x, int ksplit, int grid_z,
                       const GemmParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (!gemm_config_ok(dtype, epi, nt, mt, kw, grid_x, ksplit, grid_z, p)) return hipErrorInvalidValue;
  // several M blocks over column tiles in groups of 8: the XCD-aware 1-D grid
  GemmParams q = p;
  q.mblocks = 1;
  dim3 grid(grid_x, ksplit, grid_z);
  if (grid_z > 1 && ksplit == 1 && grid_x % 8 == 0) {
    q.mblocks = grid_z;
    grid = dim3(grid_x * grid_z, 1, 1);
  }
  const int threads = 64 * kw;
  if (dtype == 0) {
    if (epi == EPI_STORE) return launch_nt<f16_t, EPI_STORE>(nt, mt, grid, threads, q, s, e0, e1);
    if (epi == EPI_RESID) return launch_nt<f16_t, EPI_RESID>(nt, mt, grid, threads, q, s, e0, e1);
    if (epi == EPI_QKV) return launch_nt<f16_t, EPI_QKV>(nt, mt, grid, threads, q, s, e0, e1);
    if (epi == EPI_PART) return launch_nt<f16_t, EPI_PART>(nt, mt, grid, threads, q, s, e0, e1);
    return launch_nt<f16_t, EPI_SWIGLU>(nt, mt, grid, threads, q, s, e0, e1);
  }
  if (epi == EPI_STORE) return launch_nt<float, EPI_STORE>(nt, mt, grid, threads, q, s, e0, e1);
  if (epi == EPI_RESID) return launch_nt<float, EPI_RESID>(nt, mt, grid, threads, q, s, e0, e1);
  if (epi == EPI_QKV) return launch_nt<float, EPI_QKV>(nt, mt, grid, threads, q, s, e0, e1);
  if (epi == EPI_PART) return launch_nt<float, EPI_PART>(nt, mt, grid, threads, q, s, e0, e1);
  return launch_nt<float, EPI_SWIGLU>(nt, mt, grid, threads, q, s, e0, e1);
}

}  // namespace sd
