// Causal multi-query attention over the paged KV cache (Section II-A: eq.
// d_kv grows the cache by concatenation, done by the QKV projection's
// epilogue; eq. d_atte / f21 attend with softmax(q K^T / sqrt(d0)) V), and
// the rotary (cos, sin) table that epilogue reads.
//
// Paged layout of one layer's pool: head-major tiles [kv head][block][K|V]
// (kv_tile_off), so that the blocks of one task and head, allocated in
// order, are one contiguous run; K in the layout of the S = K Q^T matrix
// instruction for 16-bit caches (kv_key_off: every wave load of a key k-step
// is a contiguous 1 KB) or as [16 tokens][hd] for fp32; V transposed so that
// the P*V operand of a matrix instruction is 4 consecutive tokens of one
// dimension (kv_val_off: for 16-bit caches two such quads per 16-byte unit,
// 1 KB per wave load; [hd][16 tokens] for fp32); a slot's block table maps
// position / 16 to a block.
//
// Attention work item = (row block, kv head, key split).  A row block is a
// run of consecutive rows of one task (the gamma+1 verify rows of a task, its
// 1-2 draft rows, or a run of prefill rows); all G query heads of the kv
// head and all rows of the block are one set of query vectors that shares
// every K/V tile.  Query i only sees keys at positions <= its own.  Each work
// item keeps an online softmax (running max, running sum, rescaled output);
// when the keys are split (evenly over the item's context), partial (max,
// sum, output) triples go to a workspace with device-scope stores, and the
// last split of the item to finish merges them in split order.
//
// bf16 models (fp16 KV cache, see f16_t): S^T = K Q^T and O^T += V^T P^T on
// v_mfma_f32_16x16x32_f16; q and p enter the matrix instruction as fp16 hi + lo
// pairs, which keeps them at ~2^-22 relative precision.  Decode passes stream
// the keys from the cache straight into registers 32 at a time (two blocks),
// one step ahead, with non-temporal loads (each cache byte is read once per
// pass); prefill passes share K/V tiles in LDS between eight waves of 16 query
// vectors.  fp32 models: a vector kernel with K/V staged in LDS.
#include "sd_internal.h"

#include <algorithm>

namespace sd {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// rotary (cos, sin) table: angle pos * theta^(-2i/hd) in float64, rounded to
// float32 once (the rotation itself is done in float32 by the QKV epilogue)
__global__ void rope_table_kernel(float2* tab, int n_pos, int half, double theta) {
  const size_t n = (size_t)n_pos * half;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
    const int pos = (int)(idx / half), i = (int)(idx % half);
    const double ang = (double)pos * pow(theta, -2.0 * (double)i / (double)(2 * half));
    double s, c;
    sincos(ang, &s, &c);
    tab[idx] = make_float2((float)c, (float)s);
  }
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// the vector kernel serves fp32 caches only (16-bit caches run on the matrix kernel)
template <typename T> struct KvT;
template <> struct KvT<float> {
  static constexpr int KST_PAD = 1;
  static constexpr int EPU = 4;
};

// dynamic LDS layout, in bytes
__host__ __device__ inline size_t attn_lds_bytes(int hd, int esz, int qmax) {
  const int kst = hd + (esz == 2 ? 2 : 1);
  size_t b = (size_t)64 * kst * esz + (size_t)64 * hd * esz;
  b = (b + 15) & ~(size_t)15;
  b += (size_t)qmax * hd * 4 + (size_t)qmax * 65 * 4 + (size_t)qmax * 4 * 4;
  return b;
}

template <typename T, int HD>
__global__ __launch_bounds__(256) void attention_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int KST = HD + KvT<T>::KST_PAD;
  constexpr int EPU = KvT<T>::EPU;
  constexpr int NQG = 256 / HD;            // query groups in the P*V phase
  constexpr int QPT = ATTN_QMAX / NQG;     // query vectors per thread in P*V

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rbk = blockIdx.x;
  const int rb = rbk / p.KV, kvh = rbk % p.KV;
  const int split = blockIdx.y;
  int row0, nr;
  if (p.rowblocks) {
    row0 = p.rowblocks[2 * rb];
    nr = p.rowblocks[2 * rb + 1];
  } else {
    row0 = rb * p.R;
    nr = p.R;
  }
  const int G = p.H / p.KV;
  const int Qn = nr * G;
  const int qmax = p.qmax;

  T* Ks = (T*)smem;
  T* Vs = Ks + 64 * KST;
  size_t off = ((size_t)64 * KST + (size_t)64 * HD) * sizeof(T);
  off = (off + 15) & ~(size_t)15;
  float* Qs = (float*)(smem + off);
  float* Ss = Qs + qmax * HD;
  float* Ms = Ss + qmax * 65;
  float* Ls = Ms + qmax;
  float* As = Ls + qmax;
  int* Ps = (int*)(As + qmax);

  int maxpos = -1;
  for (int r = 0; r < nr; ++r) maxpos = max(maxpos, p.row_pos[row0 + r]);
  const int slot = p.row_bt ? 0 : p.row_slot[row0];   // decode passes: the row block's own table row
  const int k_begin = split * p.keys_per_split;
  // keys never extend past the slot's block-table row
  const int k_end = min(min(k_begin + p.keys_per_split, maxpos + 1), p.mbps * 16);
  const int Hq = p.H * HD;

  for (int idx = tid; idx < Qn * HD; idx += 256) {
    const int qi = idx / HD, d = idx % HD;
    const int row = row0 + qi / G, h = kvh * G + qi % G;
    Qs[qi * HD + d] = p.q[(size_t)row * Hq + h * HD + d] * p.scale;
  }
  for (int qi = tid; qi < Qn; qi += 256) {
    Ps[qi] = p.row_pos[row0 + qi / G];
    Ms[qi] = -INFINITY;
    Ls[qi] = 0.f;
  }

  const int dd = tid % HD, qg = tid / HD;
  float o[QPT];
#pragma unroll
  for (int k = 0; k < QPT; ++k) o[k] = 0.f;

  const T* kv = (const T*)p.kv;
  const int32_t* bt = (p.row_bt ? p.row_bt + (size_t)rb * p.mbps : p.block_table + (size_t)slot * p.mbps);

  for (int c = k_begin; c < k_end; c += 64) {
    __syncthreads();
    // stage 64 keys of K and V
    constexpr int UPR = HD / EPU;      // 16-byte units per key row
    for (int idx = tid; idx < 64 * UPR; idx += 256) {
      const int j = idx / UPR, e = (idx % UPR) * EPU;
      const int kp = c + j;
      uint4 kk = make_uint4(0, 0, 0, 0);
      T vv[EPU];
#pragma unroll
      for (int t = 0; t < EPU; ++t) vv[t] = T(0);
      if (kp < k_end) {
        const int blk = bt[kp / 16];
        const size_t base = kv_tile_off(kvh, blk, 0, p.nblk, HD) + (size_t)(kp % 16) * HD + e;
        const size_t vtb = kv_tile_off(kvh, blk, 1, p.nblk, HD);
        kk = *(const uint4*)(kv + base);
#pragma unroll
        for (int t = 0; t < EPU; ++t) vv[t] = kv[vtb + kv_val_off<T>(kp % 16, e + t, HD)];
      }
      uint32_t* kd = (uint32_t*)(Ks + j * KST + e);   // KST*esz is a multiple of 4
      kd[0] = kk.x; kd[1] = kk.y; kd[2] = kk.z; kd[3] = kk.w;
#pragma unroll
      for (int t = 0; t < EPU; ++t) Vs[j * HD + e + t] = vv[t];
    }
    __syncthreads();
    // scores and online softmax: wave w takes query vectors w, w+4, ...; lane = key
    const int kp = c + lane;
    for (int qi = wave; qi < Qn; qi += 4) {
      const float* qv = Qs + qi * HD;
      const T* kr = Ks + lane * KST;
      float s = 0.f;
#pragma unroll 8
      for (int d = 0; d < HD; ++d) s += qv[d] * Store<T>::load(kr, d);
      const bool ok = kp < k_end && kp <= Ps[qi];
      s = ok ? s : -INFINITY;
      const float mold = Ms[qi];
      const float mnew = fmaxf(mold, wave_max(s));
      const float pj = ok ? expf(s - mnew) : 0.f;
      const float psum = wave_sum(pj);
      const float alpha = mold == -INFINITY ? 0.f : expf(mold - mnew);
      Ss[qi * 65 + lane] = pj;
      if (lane == 0) {
        Ms[qi] = mnew;
        Ls[qi] = Ls[qi] * alpha + psum;
        As[qi] = alpha;
      }
    }
    __syncthreads();
    // P*V: thread (dd, qg) accumulates dimension dd of query vectors qg, qg+NQG, ...
#pragma unroll
    for (int k = 0; k < QPT; ++k) {
      const int qi = qg + NQG * k;
      if (qi < Qn) {
        float a = o[k] * As[qi];
        const float* pr = Ss + qi * 65;
#pragma unroll 8
        for (int j = 0; j < 64; ++j) a += pr[j] * Store<T>::load(Vs, j * HD + dd);
        o[k] = a;
      }
    }
  }
  __syncthreads();

  auto emit = [&](int qi, float val) {
    const int row = row0 + qi / G, h = kvh * G + qi % G;
    Store<T>::store((T*)p.out, Tile<T>::off(row, h * HD + dd, Hq), val);
  };

  if (p.splits == 1) {
#pragma unroll
    for (int k = 0; k < QPT; ++k) {
      const int qi = qg + NQG * k;
      if (qi < Qn) {
        const float L = Ls[qi];
        emit(qi, L > 0.f ? o[k] / L : 0.f);
      }
    }
    return;
  }

  // key split: this workgroup's partial (output, max, sum) goes out with
  // device-scope accesses, which the L2 of another XCD does not serve stale;
  // the item's last split to finish (counted once the stores have been waited
  // for) merges them.  A merge kernel of its own cost a launch per layer and
  // draft or verify call (tiny pair, prompt and four steps: 1194 -> 1161 us)
  const size_t base = (size_t)rbk * p.splits * qmax, item = base + (size_t)split * qmax;
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int qi = qg + NQG * k;
    if (qi < Qn)
      __hip_atomic_store(p.part_o + (item + qi) * HD + dd, o[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int qi = tid; qi < Qn; qi += 256) {
    __hip_atomic_store(p.part_ml + (item + qi) * 2, Ms[qi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p.part_ml + (item + qi) * 2 + 1, Ls[qi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __shared__ int s_last;
  __builtin_amdgcn_s_waitcnt(0);      // this wave's partial stores have reached device scope
  __syncthreads();
  if (tid == 0) {
    const int old = __hip_atomic_fetch_add(p.cnt + rbk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = old == p.splits - 1;
    if (last) __hip_atomic_store(p.cnt + rbk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;

  // merge, in split order: O = sum_s o_s e^(m_s - M) / sum_s l_s e^(m_s - M),
  // M = max_s m_s; every load of an output element is issued before any is used
  for (int qi = qg; qi < Qn; qi += NQG) {
    float ms[ATTN_MAX_SPLITS], ls[ATTN_MAX_SPLITS], os[ATTN_MAX_SPLITS];
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp) {
      const size_t it = base + (size_t)(sp < p.splits ? sp : 0) * qmax + qi;
      ms[sp] = __hip_atomic_load(p.part_ml + it * 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ls[sp] = __hip_atomic_load(p.part_ml + it * 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      os[sp] = __hip_atomic_load(p.part_o + it * HD + dd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    float M = -INFINITY, L = 0.f, O = 0.f;
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp)
      if (sp < p.splits) M = fmaxf(M, ms[sp]);
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp) {
      if (sp >= p.splits || ms[sp] == -INFINITY) continue;
      const float w = expf(ms[sp] - M);
      L += ls[sp] * w;
      O += os[sp] * w;
    }
    emit(qi, L > 0.f ? O / L : 0.f);
  }
}

// fp16 hi + lo pair of 8 floats (hi = x rounded, lo = the rest rounded),
// packed as two f16x8 operands
__device__ __forceinline__ void split8(const float (&x)[8], u32x4& hi, u32x4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint16_t a0 = f2h(x[2 * k]), a1 = f2h(x[2 * k + 1]);
    const uint16_t b0 = f2h(x[2 * k] - h2f(a0)), b1 = f2h(x[2 * k + 1] - h2f(a1));
    h[k] = (uint32_t)a0 | ((uint32_t)a1 << 16);
    l[k] = (uint32_t)b0 | ((uint32_t)b1 << 16);
  }
  hi = u32x4{h[0], h[1], h[2], h[3]};
  lo = u32x4{l[0], l[1], l[2], l[3]};
}

__device__ __forceinline__ f32x4 mfma_f16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                0, 0);
}

// A workgroup's query tiles (16 query vectors each, QT of them) are taken
// `per` to a wave: wave w takes tiles (w % QG) per .. + per - 1 and key group
// w / QG, the 32-key steps kb = k_begin + 32 (kg + KG j).  per is 1 for short
// key ranges: the QT waves of a key group then load the same keys.  From
// QPW_KEYS keys on it is QPW (> 1 for hd 64 with 2 or 3 tiles): each key tile
// is loaded once for all of them, so the loads in flight that hide the memory
// latency are of QT times as many keys (small target, two tasks at 15500
// keys, gamma = 8, four layers: verify pass 338 -> 321 us), but more key groups
// are merged at the end (the same target at 520 keys, 16 layers: step 1271 ->
// 1301 us, hence the limit).
// Lane (r16, g): query r16 of a tile; in S^T it holds keys 4g..4g+3 of
// both blocks of the step, in O^T dimensions 16 dt + 4g .. +3.
constexpr int QPW_KEYS = 512;            // 8 key groups of two 32-key steps

template <int HD, int WAVES, int QPW>
__global__ __launch_bounds__(64 * WAVES, 8 / WAVES) void attention_mfma_kernel(AttnParams p) {
  constexpr int UPG = HD / 32;             // 16-byte K units per lane group (HD/4 dims)
  constexpr int DT = HD / 16;              // 16-dimension output tiles
  constexpr int NSLOT = WAVES / 2;         // merge slots: half the waves hand over in the first round
  __shared__ float s_o[NSLOT * QPW][16][HD + 4];
  __shared__ float s_m[NSLOT * QPW][16], s_l[NSLOT * QPW][16];

  __shared__ int s_bt[ATTN_BT_CAP];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int rbk = blockIdx.x;
  const int rb = rbk / p.KV, kvh = rbk % p.KV;
  const int split = blockIdx.y;
  const int row0 = rb * p.R, nr = p.R;
  const int G = p.H / p.KV;
  const int Qn = nr * G;
  const int QT = (Qn + 15) >> 4;
  // the block's rows (nr <= 64: Qn is at most 64 query vectors) in parallel
  int maxpos = lane < nr ? p.row_pos[row0 + lane] : -1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) maxpos = max(maxpos, __shfl_xor(maxpos, o));
  maxpos = __builtin_amdgcn_readfirstlane(maxpos);
  // the item's keys (positions 0 .. maxpos) are dealt out evenly over the
  // splits in 32-key steps, at most the host's keys_per_split per split
  // (which bounds the staged block ids)
  const int kps = p.splits > 1 ? min(p.keys_per_split, ((maxpos + p.splits) / p.splits + 31) / 32 * 32)
                               : p.keys_per_split;
  const int k_begin = split * kps;
  const int k_end = min(min(k_begin + kps, maxpos + 1), p.mbps * 16);

  const int per = QPW > 1 && k_end - k_begin >= QPW_KEYS ? QPW : 1;
  const int QGn = (QT + per - 1) / per;    // wave groups (1 .. 4; 3 take the waves of 4)
  const int QG = QGn == 3 ? 4 : QGn;
  const int KG = WAVES / QG;
  const int qg = wave % QG, kg = wave / QG;
  const bool wave_on = qg < QGn;

  // block ids of the split's key range, staged in LDS (the host keeps a
  // split within ATTN_BT_CAP blocks): a key load then never waits on the
  // memory counter behind the keys still in flight
  const int32_t* bt = p.row_bt + (size_t)rb * p.mbps;   // the row block's own table row
  const int bfirst = k_begin / 16, nbr = max(0, (k_end + 15) / 16 - bfirst);
  for (int i = tid; i < min(nbr, ATTN_BT_CAP); i += blockDim.x) s_bt[i] = bt[bfirst + i];
  __syncthreads();

  int qi[QPW], qrow[QPW], qh[QPW], qpos[QPW];
  bool qvalid[QPW];
  u32x4 qhi[QPW][UPG], qlo[QPW][UPG];
#pragma unroll
  for (int t = 0; t < QPW; ++t) {
    qi[t] = (qg * per + t) * 16 + r16;
    qvalid[t] = wave_on && t < per && qi[t] < Qn;
    qrow[t] = row0 + (qvalid[t] ? qi[t] / G : 0);
    qh[t] = kvh * G + (qvalid[t] ? qi[t] % G : 0);
    qpos[t] = qvalid[t] ? p.row_pos[qrow[t]] : -1;
    // always-valid address (row0, head kvh G for idle lanes), zeroed after the load
    const float4* qs = (const float4*)(p.q + (size_t)qrow[t] * p.H * HD + (size_t)qh[t] * HD + g * (HD / 4));
    float4 xv[2 * UPG];
#pragma unroll
    for (int s = 0; s < 2 * UPG; ++s) xv[s] = qs[s];
#pragma unroll
    for (int s = 0; s < UPG; ++s) {
      // scores in log2 units (q pre-scaled by log2 e): the softmax then
      // uses the hardware base-2 exponential
      const float sc = qvalid[t] ? p.scale * 1.4426950408889634f : 0.f;
      float x[8] = {xv[2 * s].x * sc, xv[2 * s].y * sc, xv[2 * s].z * sc, xv[2 * s].w * sc,
                    xv[2 * s + 1].x * sc, xv[2 * s + 1].y * sc, xv[2 * s + 1].z * sc, xv[2 * s + 1].w * sc};
      split8(x, qhi[t][s], qlo[t][s]);
    }
  }

  float m_run[QPW], l_run[QPW];
  f32x4 o[QPW][DT];
#pragma unroll
  for (int t = 0; t < QPW; ++t) {
    m_run[t] = -INFINITY;
    l_run[t] = 0.f;
#pragma unroll
    for (int d = 0; d < DT; ++d) o[t][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // this kv head's region of the pool ([blocks][K|V][16 x HD], 2 x 16 HD
  // fp16 per block) as a range-checked buffer: steps past the key range
  // load at an out-of-range offset, which returns zero and reads nothing
  constexpr uint32_t BLK_BYTES = 2u * 16u * HD * 2u;
  const __amdgpu_buffer_rsrc_t kvr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<f16_t*>((const f16_t*)p.kv + kv_tile_off(kvh, 0, 0, p.nblk, HD)), (short)0,
      (int)((uint32_t)p.nblk * BLK_BYTES), 0x00020000);
  // key tile in the matrix-instruction layout: k-step s is the 1 KB run at
  // unit 64 s, this lane's 16 bytes at unit 64 s + lane (token r16, dims
  // g HD/4 + 8 s .. + 8); the V tile follows the K tile of the same block
  const uint32_t koff = (uint32_t)lane * 16u;
  // V tile (kv_val_off): unit 16 g + r16 of 32-dim group dp holds tokens
  // 4g..4g+3 of dims 32 dp + r16 and 32 dp + 16 + r16 (the 64 lanes read the
  // group's 1 KB)
  const uint32_t voff = 16u * HD * 2u + (uint32_t)lane * 16u;

  // two register stages of one 32-key step: K rows (two blocks), V^T quads
  // as loaded, and the masks of the V entries past the key range (applied
  // by the step, so a load is not consumed the moment it is issued)
  u32x4 Kf[2][2][UPG], Vr[2][2][DT / 2];
  uint32_t Vm[2][2][2];

  auto load = [&]<int S>(int kb) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kt = kb + 16 * t;
      const bool ok = kt < k_end;
      const uint32_t base = ok ? (uint32_t)s_bt[kt / 16 - bfirst] * BLK_BYTES : 0x80000000u;
#pragma unroll
      for (int s = 0; s < UPG; ++s)
        Kf[S][t][s] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(kvr, base + koff + 1024u * s, 0, 2));
      // keys at or past k_end were never written: their scores are masked, and
      // their V entries are zeroed so that p = 0 never meets a NaN/Inf pattern
      const int nq = min(max(k_end - (kt + 4 * g), 0), 4);
      Vm[S][t][0] = nq >= 2 ? 0xffffffffu : (nq == 1 ? 0xffffu : 0u);
      Vm[S][t][1] = nq >= 4 ? 0xffffffffu : (nq == 3 ? 0xffffu : 0u);
#pragma unroll
      for (int dp = 0; dp < DT / 2; ++dp)
        Vr[S][t][dp] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(kvr, base + voff + 1024u * dp, 0, 2));
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&]<int S>(int kb) {
#pragma unroll
    for (int t = 0; t < QPW; ++t) {
      if (t >= per) continue;
      // four independent accumulation chains (the hi and lo parts of q for
      // each of the two key blocks), so that consecutive matrix instructions
      // do not wait on each other's results; the parts are added at the end
      f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0, s0l = s0, s1l = s0;
#pragma unroll
      for (int s = 0; s < UPG; ++s) {
        s0 = mfma_f16(Kf[S][0][s], qhi[t][s], s0);
        s1 = mfma_f16(Kf[S][1][s], qhi[t][s], s1);
        s0l = mfma_f16(Kf[S][0][s], qlo[t][s], s0l);
        s1l = mfma_f16(Kf[S][1][s], qlo[t][s], s1l);
      }
      s0 += s0l;
      s1 += s1l;
      float sc[8];
      bool ok[8];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k0 = kb + 4 * g + v, k1 = k0 + 16;
        ok[v] = k0 < k_end && k0 <= qpos[t];
        ok[4 + v] = k1 < k_end && k1 <= qpos[t];
        sc[v] = s0[v];
        sc[4 + v] = s1[v];
      }
      float mx = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = ok[e] ? fmaxf(mx, sc[e]) : mx;
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mnew = fmaxf(m_run[t], mx);
      float pe[8], sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pe[e] = ok[e] ? exp2f(sc[e] - mnew) : 0.f;
        sum += pe[e];
      }
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      const float alpha = m_run[t] == -INFINITY ? 0.f : exp2f(m_run[t] - mnew);
      l_run[t] = l_run[t] * alpha + sum;
      m_run[t] = mnew;
      u32x4 phi, plo;
      split8(pe, phi, plo);
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        o[t][d] *= alpha;
        // dims d (even d: x, y of the unit) of tokens 4g..4g+3 of both blocks
        const u32x4 v0 = Vr[S][0][d / 2], v1 = Vr[S][1][d / 2];
        const u32x4 va = (d & 1) ? u32x4{v0.z & Vm[S][0][0], v0.w & Vm[S][0][1], v1.z & Vm[S][1][0], v1.w & Vm[S][1][1]}
                                 : u32x4{v0.x & Vm[S][0][0], v0.y & Vm[S][0][1], v1.x & Vm[S][1][0], v1.y & Vm[S][1][1]};
        o[t][d] = mfma_f16(va, phi, o[t][d]);
        o[t][d] = mfma_f16(va, plo, o[t][d]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // loads are issued unconditionally (past the key range they read
  // nothing), so the compiler keeps the next step in flight during a step
  const int kstep = 32 * KG;
  int kb = k_begin + 32 * kg;
  if (wave_on && kb < k_end) {
    load.template operator()<0>(kb);
    for (; kb < k_end; kb += 2 * kstep) {
      const int kb1 = kb + kstep;
      load.template operator()<1>(kb1);
      step.template operator()<0>(kb);
      if (kb1 >= k_end) break;
      load.template operator()<0>(kb1 + kstep);
      step.template operator()<1>(kb1);
    }
  }

  // merge the key groups of each query tile into key group 0 as a binary
  // tree (fixed order): in the round of stride h, key group kg with
  // kg % 2h == h hands its state to kg - h through slot qg KG/2 + kg / 2h
  for (int h = 1; h < KG; h *= 2) {
    const int sl = (qg * (KG / 2) + kg / (2 * h)) * QPW;
    if (wave_on && kg % (2 * h) == h) {
#pragma unroll
      for (int t = 0; t < QPW; ++t) {
        if (t >= per) continue;
        if (g == 0) {
          s_m[sl + t][r16] = m_run[t];
          s_l[sl + t][r16] = l_run[t];
        }
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int v = 0; v < 4; ++v) s_o[sl + t][r16][16 * d + 4 * g + v] = o[t][d][v];
      }
    }
    __syncthreads();
    if (wave_on && kg % (2 * h) == 0) {
#pragma unroll
      for (int t = 0; t < QPW; ++t) {
        if (t >= per) continue;
        const float mb = s_m[sl + t][r16], lb = s_l[sl + t][r16];
        const float M = fmaxf(m_run[t], mb);
        const float a = m_run[t] == -INFINITY ? 0.f : exp2f(m_run[t] - M);
        const float b = mb == -INFINITY ? 0.f : exp2f(mb - M);
        l_run[t] = l_run[t] * a + lb * b;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int v = 0; v < 4; ++v) o[t][d][v] = o[t][d][v] * a + s_o[sl + t][r16][16 * d + 4 * g + v] * b;
        m_run[t] = M;
      }
    }
    __syncthreads();
  }
  const bool first = wave_on && kg == 0;     // holds the merged state of its tiles

  if (p.splits == 1) {
    if (first) {
#pragma unroll
      for (int t = 0; t < QPW; ++t) {
        if (!qvalid[t]) continue;
        const float inv = l_run[t] > 0.f ? 1.0f / l_run[t] : 0.f;
        // four consecutive output dimensions of this lane's query, MFMA-tile layout
#pragma unroll
        for (int d = 0; d < DT; ++d) {
          const size_t off = Tile<f16_t>::off(qrow[t], qh[t] * HD + 16 * d + 4 * g, p.H * HD);
          *(uint2*)((f16_t*)p.out + off) =
              make_uint2((uint32_t)f2h(o[t][d][0] * inv) | ((uint32_t)f2h(o[t][d][1] * inv) << 16),
                         (uint32_t)f2h(o[t][d][2] * inv) | ((uint32_t)f2h(o[t][d][3] * inv) << 16));
        }
      }
    }
    return;
  }

  // key split: this workgroup's partial (output, max, sum) goes out with
  // device-scope stores; the item's last split to finish merges them.  Every
  // value handed over is written and read with device-scope (sc1) accesses,
  // which the L2 of another XCD does not serve stale, so waiting for the
  // stores before counting is all the ordering needed (a release / acquire
  // fence would also write back and invalidate the whole L2, which only data
  // written with plain stores needs).  16 bytes at a time: the hand-over and
  // the merge are a chain of memory round trips, and 4-byte accesses made
  // several rounds of each (verify pass of two 7B layers at B = 1 255 -> 250 us,
  // of the small target's 16 at B = 8 with its drafts 1321 -> 1271)
  constexpr int SC1 = 16;
  const size_t base = (size_t)rbk * p.splits * p.qmax;
  const uint32_t nvec = (uint32_t)p.splits * p.qmax;
  const __amdgpu_buffer_rsrc_t por =
      __builtin_amdgcn_make_buffer_rsrc(p.part_o + base * HD, (short)0, (int)(nvec * HD * 4u), 0x00020000);
  const __amdgpu_buffer_rsrc_t pmr =
      __builtin_amdgcn_make_buffer_rsrc(p.part_ml + base * 2, (short)0, (int)(nvec * 8u), 0x00020000);
  if (first) {
#pragma unroll
    for (int t = 0; t < QPW; ++t) {
      if (!qvalid[t]) continue;
      const uint32_t item = (uint32_t)(split * p.qmax + qi[t]);
#pragma unroll
      for (int d = 0; d < DT; ++d)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[t][d]), por,
                                               (item * HD + 16u * d + 4u * g) * 4u, 0, SC1);
      if (g == 0)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(m_run[t]), __float_as_uint(l_run[t])}, pmr,
                                              item * 8u, 0, SC1);
    }
  }
  __shared__ int s_last;
  __builtin_amdgcn_s_waitcnt(0);      // this wave's partial stores have reached device scope
  __syncthreads();
  if (tid == 0) {
    const int old = __hip_atomic_fetch_add(p.cnt + rbk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int last = old == p.splits - 1;
    if (last) __hip_atomic_store(p.cnt + rbk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;

  // merge, in split order: O = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M),
  // M = max_s m_s (log2 units); every load of four output dimensions of a
  // query (all splits' max, sum and output) is issued before any is used
  for (int idx = tid; idx < Qn * (HD / 4); idx += 64 * WAVES) {
    const int qj = idx / (HD / 4), c = idx % (HD / 4);
    u32x2 ml[ATTN_MAX_SPLITS];
    u32x4 os[ATTN_MAX_SPLITS];
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp) {
      // splits past the last read nothing (out-of-range offset: zeros)
      const uint32_t it = (uint32_t)(sp * p.qmax + qj);
      ml[sp] = __builtin_bit_cast(
          u32x2, __builtin_amdgcn_raw_buffer_load_b64(pmr, sp < p.splits ? it * 8u : 0x80000000u, 0, SC1));
      os[sp] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(por, sp < p.splits ? (it * HD + 4u * c) * 4u : 0x80000000u, 0, SC1));
    }
    float M = -INFINITY;
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp)
      if (sp < p.splits) M = fmaxf(M, __uint_as_float(ml[sp].x));
    float L = 0.f;
    float O[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sp = 0; sp < ATTN_MAX_SPLITS; ++sp) {
      const float ms = __uint_as_float(ml[sp].x);
      const float w = sp < p.splits && ms != -INFINITY ? exp2f(ms - M) : 0.f;
      L += __uint_as_float(ml[sp].y) * w;
#pragma unroll
      for (int e = 0; e < 4; ++e) O[e] += __uint_as_float(os[sp][e]) * w;
    }
    const int row = row0 + qj / G, h = kvh * G + qj % G;
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    *(uint2*)((f16_t*)p.out + Tile<f16_t>::off(row, h * HD + 4 * c, p.H * HD)) =
        make_uint2((uint32_t)f2h(O[0] * inv) | ((uint32_t)f2h(O[1] * inv) << 16),
                   (uint32_t)f2h(O[2] * inv) | ((uint32_t)f2h(O[3] * inv) << 16));
  }
}

// Prefill attention of 16-bit caches: up to ATTN_PREFILL_Q query vectors (a
// run of rows of one task, all query heads of one kv head) per workgroup of
// eight waves, one tile of 16 per wave.  Here every key meets more than a
// hundred queries, so the matrix instructions bound the kernel and not the
// cache stream: the K/V tiles are loaded into LDS once per workgroup (64 keys a
// stage, half a block per wave, two stages) and each operand a wave reads from
// there feeds both fp16 parts of q or p.  What is left beside them is the
// softmax, kept small: no masks on steps all of a wave's queries see, row sums
// left per lane until the end, and the running maximum only raised (with its
// lane exchanges and the rescaling of the output) when a score passes it by
// more than 8 in log2 units (the conditional rescaling published with
// FlashAttention-4), so p stays within 2^8 and every step in between is exact
// relative to the same reference.  Row blocks run last to first: the
// ones with the most keys start first.
// Measured per layer (the decode kernel, which streams the keys into each
// wave's registers, before): 7B, a 2048-row chunk of ragged prompts 178 -> 80
// us, one prompt of 1024 tokens 64 -> 39; the small target's last chunk of
// 15000 tokens 1024 -> 310.  Four waves with two tiles each (half the LDS
// reads per matrix instruction): 87, 46 and 351 us.
constexpr int PF_KEYS = 64;

template <int HD>
__global__ __launch_bounds__(512, 2) void attention_prefill_kernel(AttnParams p) {
  constexpr int UPG = HD / 32, DT = HD / 16, WAVES = ATTN_PREFILL_Q / 16;
  constexpr uint32_t BLK_BYTES = 2u * 16u * HD * 2u;   // K and V tile of a block
  constexpr int WPB = WAVES * 16 / PF_KEYS;            // waves that load a block of a stage
  constexpr int NL = (int)BLK_BYTES / 1024 / WPB;      // loads of a wave per stage
  constexpr int UNITS = (int)BLK_BYTES / 16;           // 16-byte units of a block
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  u32x4* lds = (u32x4*)smem;                           // [2][PF_KEYS / 16][UNITS]
  __shared__ int s_bt[ATTN_BT_CAP];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int rb = p.nrb - 1 - (int)blockIdx.x / p.KV, kvh = blockIdx.x % p.KV;
  const int row0 = p.rowblocks[2 * rb], nr = p.rowblocks[2 * rb + 1];
  const int G = p.H / p.KV;
  const int Qn = nr * G;

  int maxpos = lane < nr ? p.row_pos[row0 + lane] : -1;
  if (lane + 64 < nr) maxpos = max(maxpos, p.row_pos[row0 + lane + 64]);   // nr <= ATTN_PREFILL_Q
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) maxpos = max(maxpos, __shfl_xor(maxpos, o));
  maxpos = __builtin_amdgcn_readfirstlane(maxpos);
  const int k_end = min(maxpos + 1, p.mbps * 16);
  const int stages = (k_end + PF_KEYS - 1) / PF_KEYS;
  const int32_t* bt = p.block_table + (size_t)p.row_slot[row0] * p.mbps;
  for (int i = tid; i < min((k_end + 15) / 16, ATTN_BT_CAP); i += 64 * WAVES) s_bt[i] = bt[i];
  __syncthreads();

  const int qi = wave * 16 + r16;
  const bool qvalid = qi < Qn;
  const int qrow = row0 + (qvalid ? qi / G : 0), qh = kvh * G + (qvalid ? qi % G : 0);
  const int qpos = qvalid ? p.row_pos[qrow] : -1;
  u32x4 qhi[UPG], qlo[UPG];
  {
    const float4* qs = (const float4*)(p.q + (size_t)qrow * p.H * HD + (size_t)qh * HD + g * (HD / 4));
    float4 xv[2 * UPG];
#pragma unroll
    for (int s = 0; s < 2 * UPG; ++s) xv[s] = qs[s];
    const float sc = qvalid ? p.scale * 1.4426950408889634f : 0.f;   // scores in log2 units
#pragma unroll
    for (int s = 0; s < UPG; ++s) {
      float x[8] = {xv[2 * s].x * sc, xv[2 * s].y * sc, xv[2 * s].z * sc, xv[2 * s].w * sc,
                    xv[2 * s + 1].x * sc, xv[2 * s + 1].y * sc, xv[2 * s + 1].z * sc, xv[2 * s + 1].w * sc};
      split8(x, qhi[s], qlo[s]);
    }
  }
  float m_run = -1e30f, l_lane = 0.f;
  f32x4 o[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  // positions of the wave's queries: past wmax there is nothing to see, up to
  // wmin nothing to mask
  int wmax = qpos, wmin = qvalid ? qpos : 0x7fffffff;
#pragma unroll
  for (int x = 1; x < 16; x <<= 1) {
    wmax = max(wmax, __shfl_xor(wmax, x));
    wmin = min(wmin, __shfl_xor(wmin, x));
  }
  wmax = __builtin_amdgcn_readfirstlane(wmax);
  wmin = __builtin_amdgcn_readfirstlane(wmin);

  const __amdgpu_buffer_rsrc_t kvr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<f16_t*>((const f16_t*)p.kv + kv_tile_off(kvh, 0, 0, p.nblk, HD)), (short)0,
      (int)((uint32_t)p.nblk * BLK_BYTES), 0x00020000);
  // this wave's share of stage st (part wave % WPB of block wave / WPB) into
  // its place; blocks past the keys load zeros
  const int lb = wave / WPB, lc = wave % WPB * NL * 64;
  auto gload = [&](int st) {
    const int kt = PF_KEYS * st + 16 * lb;
    const uint32_t base = kt < k_end ? (uint32_t)s_bt[kt / 16] * BLK_BYTES + (lc + lane) * 16u : 0x80000000u;
    u32x4* dst = lds + (size_t)((st & 1) * (PF_KEYS / 16) + lb) * UNITS + lc;
#pragma unroll
    for (int c = 0; c < NL; ++c) {
      const uint32_t off = base + 1024u * c;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kvr, (__attribute__((address_space(3))) void*)(dst + 64 * c), 16, off, 0,
                                               0, 0);
    }
  };

  gload(0);
  for (int st = 0; st < stages; ++st) {
    __builtin_amdgcn_s_waitcnt(0x0f70);                // vmcnt 0: this wave's loads of stage st
    asm volatile("s_barrier" ::: "memory");            // every block is there; stage st - 1 has been read
    gload(st + 1);                                     // (past the last stage: zeros)
    const u32x4* buf = lds + (size_t)(st & 1) * (PF_KEYS / 16) * UNITS;
    if (st == stages - 1 && (k_end & 15)) {
      // values past the last key were never written: zero them, so that their
      // p = 0 never meets a NaN or Inf pattern (their scores are masked)
      f16_t* vt = (f16_t*)(buf + ((k_end / 16) & 3) * UNITS) + 16 * HD;
      for (int i = tid; i < 16 * HD; i += 64 * WAVES)
        if ((i & 15) >= (k_end & 15)) vt[kv_val_off<f16_t>(i & 15, i >> 4, HD)] = (f16_t)0.f;
      __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt 0
      asm volatile("s_barrier" ::: "memory");
    }
#pragma unroll
    for (int h = 0; h < PF_KEYS / 32; ++h) {
      const int kb = PF_KEYS * st + 32 * h;
      if (kb > wmax) break;
      const u32x4* b0 = buf + (2 * h) * UNITS + lane;  // the step's two blocks
      const u32x4* b1 = b0 + UNITS;
      // four independent chains: the two blocks, the hi and lo part of q
      f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0, s0l = s0, s1l = s0;
#pragma unroll
      for (int s = 0; s < UPG; ++s) {
        const u32x4 k0 = b0[64 * s], k1 = b1[64 * s];
        s0 = mfma_f16(k0, qhi[s], s0);
        s1 = mfma_f16(k1, qhi[s], s1);
        s0l = mfma_f16(k0, qlo[s], s0l);
        s1l = mfma_f16(k1, qlo[s], s1l);
      }
      s0 += s0l;
      s1 += s1l;
      float sc[8];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sc[v] = s0[v];
        sc[4 + v] = s1[v];
      }
      if (kb + 31 > wmin) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          sc[v] = kb + 4 * g + v <= qpos ? sc[v] : -INFINITY;
          sc[4 + v] = kb + 16 + 4 * g + v <= qpos ? sc[4 + v] : -INFINITY;
        }
      }
      float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
      if (__any(mx > m_run + 8.0f)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mnew = fmaxf(m_run, mx);
        const float alpha = exp2f(m_run - mnew);
        m_run = mnew;
        l_lane *= alpha;
#pragma unroll
        for (int d = 0; d < DT; ++d) o[d] *= alpha;
      }
      float pe[8], sum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pe[e] = __builtin_amdgcn_exp2f(sc[e] - m_run);
        sum += pe[e];
      }
      l_lane += sum;
      u32x4 phi, plo;
      split8(pe, phi, plo);
#pragma unroll
      for (int dp = 0; dp < DT / 2; ++dp) {
        const u32x4 v0 = b0[UNITS / 2 + 64 * dp], v1 = b1[UNITS / 2 + 64 * dp];
        // dims 32 dp + (lane's 4g + v) and + 16 of tokens 4g..4g+3 of both blocks
        const u32x4 va = u32x4{v0.x, v0.y, v1.x, v1.y}, vb = u32x4{v0.z, v0.w, v1.z, v1.w};
        o[2 * dp] = mfma_f16(va, phi, o[2 * dp]);
        o[2 * dp + 1] = mfma_f16(vb, phi, o[2 * dp + 1]);
        o[2 * dp] = mfma_f16(va, plo, o[2 * dp]);
        o[2 * dp + 1] = mfma_f16(vb, plo, o[2 * dp + 1]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);                  // the loads past the last stage

  float l = l_lane;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (!qvalid) return;
  const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
  for (int d = 0; d < DT; ++d) {
    const size_t off = Tile<f16_t>::off(qrow, qh * HD + 16 * d + 4 * g, p.H * HD);
    *(uint2*)((f16_t*)p.out + off) = make_uint2((uint32_t)f2h(o[d][0] * inv) | ((uint32_t)f2h(o[d][1] * inv) << 16),
                                                (uint32_t)f2h(o[d][2] * inv) | ((uint32_t)f2h(o[d][3] * inv) << 16));
  }
}

hipError_t launch_rope_table(float2* tab, int n_pos, int half, double theta, hipStream_t s) {
  if (n_pos <= 0 || half <= 0) return hipErrorInvalidValue;
  const size_t n = (size_t)n_pos * half;
  const int blocks = (int)std::min<size_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(rope_table_kernel, dim3(blocks), dim3(256), 0, s, tab, n_pos, half, theta);
  return hipGetLastError();
}

template <typename T, int HD>
static hipError_t launch_attn_t(const AttnParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const size_t lds = attn_lds_bytes(HD, sizeof(T), p.qmax);
  launch_k(attention_kernel<T, HD>, dim3(p.nrb * p.KV, p.splits), dim3(256), (uint32_t)lds, s, e0, e1, p);
  return hipGetLastError();
}

template <int HD> constexpr int PF_LDS = 2 * PF_KEYS * 2 * HD * (int)sizeof(f16_t);

template <int HD>
static hipError_t launch_prefill(const AttnParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  launch_k(attention_prefill_kernel<HD>, dim3(p.nrb * p.KV), dim3(512), (uint32_t)PF_LDS<HD>, s, e0, e1, p);
  return hipGetLastError();
}

hipError_t prepare_attention() {
  hipError_t r = hipSuccess;
  auto limit = [&](const void* kern, size_t lds) {
    if (r == hipSuccess) r = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  };
  limit((const void*)attention_prefill_kernel<64>, PF_LDS<64>);
  limit((const void*)attention_prefill_kernel<128>, PF_LDS<128>);
  limit((const void*)attention_kernel<float, 64>, attn_lds_bytes(64, sizeof(float), ATTN_QMAX));
  limit((const void*)attention_kernel<float, 128>, attn_lds_bytes(128, sizeof(float), ATTN_QMAX));
  return r;
}

hipError_t launch_attention(int dtype, const AttnParams& p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (p.nrb <= 0) return hipSuccess;
  if (p.keys_per_split % 64 || p.keys_per_split > ATTN_BT_CAP * 16) return hipErrorInvalidValue;
  const dim3 grid(p.nrb * p.KV, p.splits);
  if (dtype == 0 && p.rowblocks) {
    if (p.qmax > ATTN_PREFILL_Q || p.splits != 1) return hipErrorInvalidValue;
    return p.hd == 64    ? launch_prefill<64>(p, s, e0, e1)
           : p.hd == 128 ? launch_prefill<128>(p, s, e0, e1)
                         : hipErrorInvalidValue;
  }
  if (p.qmax > ATTN_QMAX) return hipErrorInvalidValue;
  // a split item's last workgroup merges: every split needs the counter, and
  // the merge holds at most ATTN_MAX_SPLITS partials per query
  if (p.splits > 1 && (!p.cnt || p.splits > ATTN_MAX_SPLITS)) return hipErrorInvalidValue;
  if (dtype == 0) {
    if (!p.row_bt) return hipErrorInvalidValue;
    // four waves per workgroup for large grids (hd 64: 1024 or more
    // workgroups, hd 128: 2048): two then share a CU, and one's start and
    // merge overlap the other's stream.  13B B = 64 (2560 verify and 1024
    // draft workgroups): step 19.73 -> 18.38 ms; 7B paged B = 32 (1024
    // verify workgroups) is 0.7 % slower with four, so keeps eight.  Split
    // hd 128 items (7B B = 1: a few hundred keys per split) also take four:
    // a two-round key-group merge instead of three, 14.2 -> 13.9 us per
    // layer (with twice the splits on them, 14.8)
    const bool many = grid.x * grid.y >= (p.hd == 64 ? 1024u : 2048u) || (p.hd == 128 && p.splits > 1);
    // hd 64, more than one query tile (grouped KV heads, long speculation): up
    // to three tiles in one wave where its key range is long (QPW_KEYS).  hd 128
    // has no registers for a second tile
    const int qt = (p.qmax + 15) / 16, qpw = p.hd == 64 && qt > 1 ? (qt == 3 ? 3 : 2) : 1;
#define SD_ATTN(HDv, Wv, Qv) launch_k(attention_mfma_kernel<HDv, Wv, Qv>, grid, dim3(64 * Wv), 0, s, e0, e1, p)
    if (p.hd == 64) {
      if (many) {
        if (qpw == 1) SD_ATTN(64, 4, 1);
        else if (qpw == 2) SD_ATTN(64, 4, 2);
        else SD_ATTN(64, 4, 3);
      } else {
        if (qpw == 1) SD_ATTN(64, 8, 1);
        else if (qpw == 2) SD_ATTN(64, 8, 2);
        else SD_ATTN(64, 8, 3);
      }
    } else if (p.hd == 128) {
      if (many) SD_ATTN(128, 4, 1);
      else SD_ATTN(128, 8, 1);
    } else {
      return hipErrorInvalidValue;
    }
#undef SD_ATTN
    return hipGetLastError();
  }
  if (p.hd == 64) return launch_attn_t<float, 64>(p, s, e0, e1);
  if (p.hd == 128) return launch_attn_t<float, 128>(p, s, e0, e1);
  return hipErrorInvalidValue;
}

size_t attention_lds_bytes(int hd, int esz, int qmax) { return attn_lds_bytes(hd, esz, qmax); }

}  // namespace sd
