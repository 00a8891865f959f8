// gfx950 (CDNA4) kernels for decode attention over a block-wise low-rank KV
// cache (MILO, Sec. 4.2 Eq. 3 factors; Sec. 4.4 Alg. 1 inference stage; the
// attention itself is Sec. 4.1 Eq. 1).
//
//  pack_kernel    repacks row-major bf16 factors into MFMA-fragment order.
//  attend_kernel  persistent: one workgroup (8 waves) per compute unit runs a
//                 host-built list of work items, its fragment streams flowing
//                 across items:
//     block item (block b, a tile of up to 64 head-major query columns of
//     one or more KV heads, a run of 256-token tiles):
//       projection  Qt = scale*log2(e) * R^K_b[:, g] q          (MFMA, into LDS;
//                   per KV head g of the tile)
//       scores      S  = P^K_b Qt, 32 tokens per wave and tile  (MFMA)
//       softmax     running max per column shared by the waves, W = 2^(S - m)
//       latent V    Ot = sum_t W_t P^V_b[t]                      (MFMA, waves split
//                   token segments x rank tiles)
//       up-project  o  = R^V_b[:, g]^T Ot                        (MFMA, 16-dim slice
//                   per wave; per KV head g of the tile)
//       -> folded into the workgroup's partial (m, l, o) per column for its
//          current column tile; written when the group ends
//     tail item (request i, KV head g, kTailChunk-token chunk of the request's
//     own KV): plain attention of the group's query heads over the chunk
//     (MFMA scores, VALU values) -> partial (m, l, o) per column
//  merge_kernel   log-sum-exp merge of every partial of a column into O (fp32).
//
// Scores are kept in log2 units (the scale folds log2(e)), so every exponential
// is one v_exp_f32.
#include <hip/hip_ext.h>

#include <type_traits>

#include "milo_internal.h"

namespace milo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 ld_bf16x8(const void* p) { return *reinterpret_cast<const bf16x8*>(p); }

// eight int8 codes (little-endian in two dwords) as bf16, exactly
__device__ __forceinline__ bf16x8 i8_to_bf16x8(uint2 raw) {
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = (__bf16)(float)(int8_t)(raw.x >> (8 * e));
    v[4 + e] = (__bf16)(float)(int8_t)(raw.y >> (8 * e));
  }
  return v;
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// the same product on operands that hold fp16 bit patterns (rebuilt keys and
// the query of dense items)
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x16 mfma32_f16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                0, 0);
}
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t u) {
  return __uint_as_float(static_cast<uint32_t>(u) << 16);
}

// sixteen zeros set where they stand (opaque to the optimiser, which would
// otherwise keep one zero accumulator live across the loops that need it)
__device__ __forceinline__ f32x16 zero16() {
  float z;
  asm volatile("v_mov_b32 %0, 0" : "=v"(z));
  f32x16 v;
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = z;
  return v;
}

// v, as a value the optimiser cannot trace: addresses derived from it are formed
// where they are used instead of staying live across a loop
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// ends x's life without an instruction: its registers are free until the next write
template <typename T>
__device__ __forceinline__ void forget(T& x) { asm volatile("" : "=v"(x)); }
__device__ __forceinline__ void forget(uint2& x) { asm volatile("" : "=v"(x.x), "=v"(x.y)); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// n / d for a divisor whose floor(2^32 / d) (2^32 - 1 for d = 1) the host
// computed: the product is at most one short (n < 2^32)
__device__ __forceinline__ int div_by(int n, int d, uint32_t m) {
  const int q = (int)__umulhi((uint32_t)n, m);
  return n - q * d >= d ? q + 1 : q;
}
// query row i * H_q + h of head-major column c = g * N_g + i * G + (h mod G)
__device__ __forceinline__ int64_t query_row(const AttendArgs& a, int c) {
  const int g = div_by(c, a.N_g, a.N_g_inv), rem = c - g * a.N_g, i = div_by(rem, a.G, a.G_inv);
  return (int64_t)i * a.H_q + g * a.G + (rem - i * a.G);
}

// Workgroup barrier for the attention kernel: every wave's LDS reads and
// writes issued before it are complete.  Global loads in flight (the waves'
// fragment streams) are deliberately not waited for; __syncthreads() would
// drain them (vmcnt(0)).  The "memory" clobber keeps the compiler from moving
// memory accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------
// Packing
// ---------------------------------------------------------------------------
// bf16 factor: the 8 elements of lane `lane` of fragment `frag`, one 16-byte store
__device__ __forceinline__ void pack_bf16_fragment(const PackArgs& a, int64_t frag, int lane) {
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int row, col;
    frag_source(a.geom, frag, lane, e, &row, &col);
    v[e] = (row < a.geom.rows && col < a.geom.cols) ? a.src[(int64_t)row * a.geom.cols + col] : 0;
  }
  uint4 out;
  out.x = v[0] | ((uint32_t)v[1] << 16);
  out.y = v[2] | ((uint32_t)v[3] << 16);
  out.z = v[4] | ((uint32_t)v[5] << 16);
  out.w = v[6] | ((uint32_t)v[7] << 16);
  *reinterpret_cast<uint4*>(a.dst + frag * kFragElems + lane * 8) = out;
}

__global__ __launch_bounds__(256) void pack_kernel(PackArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t frag = gid >> 6;
  const int lane = (int)(gid & 63);
  if (frag >= a.n_frags) return;
  if (a.row_scale) {
    // INT8 P factor: code = round-to-nearest-even(P / s_row) in fp32 (correctly
    // rounded division), |code| <= 127; 8 codes per lane at byte 8 lane of the
    // fragment's 512 bytes
    uint32_t w[2] = {0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int row, col;
      frag_source(a.geom, frag, lane, e, &row, &col);
      int code = 0;
      if (row < a.geom.rows && col < a.geom.cols) {
        const float sc = a.row_scale[row];
        if (sc > 0.f) {
          const float x = bf16_to_f32(a.src[(int64_t)row * a.geom.cols + col]);
          code = (int)fminf(127.f, fmaxf(-127.f, rintf(__fdiv_rn(x, sc))));
        }
      }
      w[e >> 2] |= (uint32_t)(code & 0xff) << (8 * (e & 3));
    }
    *reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(a.dst) + frag * kFragElems + lane * 8) =
        make_uint2(w[0], w[1]);
    return;
  }
  pack_bf16_fragment(a, frag, lane);
}

// Many bf16 factors in one launch: job j packs fragments
// starts[j] .. starts[j + 1] - 1 of a flat fragment range that begins at
// starts[0]; 4 fragments per workgroup, each lane finding its job by binary search.
__global__ __launch_bounds__(256) void pack_batch_kernel(const PackArgs* jobs, const int64_t* starts, int n_jobs) {
  const int64_t g = starts[0] + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = (int)(threadIdx.x & 63);
  if (g >= starts[n_jobs]) return;
  int lo = 0, hi = n_jobs - 1;  // the last job whose start is <= g
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= g) lo = mid;
    else hi = mid - 1;
  }
  pack_bf16_fragment(jobs[lo], g - starts[lo], lane);
}

// INT8 P factors: per-row scale s = max |P[row][:]| / 127 (fp32, correctly
// rounded division); rows past `rows` up to rows_pad get 0; a non-finite row sets *bad.
__global__ __launch_bounds__(256) void row_scale_kernel(const uint16_t* src, int rows, int cols, int rows_pad,
                                                        float* scale, int* bad) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows_pad) return;
  float m = 0.f;
  if (r < rows) {
    for (int c = 0; c < cols; ++c) m = fmaxf(m, fabsf(bf16_to_f32(src[(int64_t)r * cols + c])));
    bool finite = true;
    for (int c = 0; c < cols; ++c) finite = finite && isfinite(bf16_to_f32(src[(int64_t)r * cols + c]));
    if (!finite) {
      atomicOr(bad, 1);
      m = 0.f;
    }
  }
  scale[r] = __fdiv_rn(m, 127.f);
}

// INT8 P factors: the 256-byte scale unit of (tile t, wave w) holds the K then
// the V scales of tokens 256 t + 32 w + m, m = 0..31
__global__ __launch_bounds__(256) void scale_units_kernel(const float* ks, const float* vs, int T_pad, float* dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // float index in the units
  if (i >= T_pad * 2) return;
  const int unit = i / 64, m = i % 64;                  // unit = t * kWaves + w
  const int tok = 32 * unit + (m & 31);
  dst[i] = m < 32 ? ks[tok] : vs[tok];
}

// ---------------------------------------------------------------------------
// Tail work item: attention of the G query heads of KV head g of request i over
// tokens [t0, t0 + nt) of that request's uncompressed KV (nt <= kTailChunk
// follows from the call's tail length; an item past the tail does nothing).  Wave w takes tokens t0 + 32w .. t0 + 32w + 31; every load of the
// item is issued up front (rows past the chunk's end re-read its last row and
// are masked), then:
//   scores  S = K q^T  (one 32x32x16 MFMA per 16 dims: 32 tokens x 32 head
//           columns, heads past G read the last head and are discarded)
//   softmax column max / sum over the 4 waves through LDS, W = 2^(S - m)
//   values  o[h] = sum_t W[t][h] V[t]  (VALU: lane owns D/64 dims, the weights
//           of a token are broadcast from LDS), summed over the waves in LDS.
// ---------------------------------------------------------------------------
// Value pass of a tail item for one wave: o[h][e] = sum over the wave's 32
// tokens of W[t][h] * V[t][e] for NH heads and this lane's D/64 dims, written
// to the wave's partial-output rows (row stride D).  Fully unrolled, so the
// per-token registers are addressed statically.
template <int D, int NH>
__device__ __forceinline__ void tail_values(const float* wt, const uint32_t (&vraw)[kTailChunk / kWaves],
                                            float* out) {
  constexpr int DL = D / 64;
  float acc[NH][DL];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int e = 0; e < DL; ++e) acc[h][e] = 0.f;
#pragma unroll
  for (int tt = 0; tt < kTailChunk / kWaves; ++tt) {
    float vf[DL];
    vf[0] = __uint_as_float(vraw[tt] << 16);
    if constexpr (DL == 2) vf[1] = __uint_as_float(vraw[tt] & 0xffff0000u);
    const float4* wr = reinterpret_cast<const float4*>(wt + tt * 32);
#pragma unroll
    for (int q4 = 0; q4 < NH / 4; ++q4) {
      const float4 w4 = wr[q4];
      const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < DL; ++e) acc[4 * q4 + u][e] += wv[u] * vf[e];
    }
  }
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int e = 0; e < DL; ++e) out[h * D + e] = acc[h][e];
}

template <int D>
__device__ __forceinline__ void tail_item(const AttendArgs& a, const WorkItem& it, unsigned char* smem,
                                          const int tid) {
  constexpr int NK = D / 16;                // 16-dim steps of the score MFMA
  constexpr int DL = D / 64;                // dims per lane in the value pass
  constexpr int kTokW = kTailChunk / kWaves;  // tokens per wave (32)
  static_assert(kTokW == 32, "one 32-row MFMA tile of tokens per wave");
  const int i = it.req, slot = a.n_block_slots + it.slot, g = it.g, G = a.G;
  const int wave = tid >> 6, lane = tid & 63, lrow = lane & 31, lhi = lane >> 5;
  // the chunk's rows come from this call's tail length: the plan holds chunks
  // up to its planned capacity, and chunks past the request's tail are empty
  const int t0 = it.sub * kTailChunk;
  const int nt = min(kTailChunk, tail_len_of(a.tl, i) - t0);
  if (nt <= 0) return;
  float* red = reinterpret_cast<float*>(smem);   // [kWaves][32] column maxima
  float* lred = red + kWaves * 32;               // [kWaves][32] column sums
  float* wt = lred + kWaves * 32;                // [kTailChunk][32] weights, token-major
  float* op = wt + kTailChunk * 32;              // [kWaves][kMaxGroup][D] partial outputs

  const int64_t rs = (int64_t)a.H_kv * D;      // row stride of the tail K / V
  const int64_t row0 = (int64_t)i * a.tail_stride + t0;
  const int tk = min(kTokW * wave + lrow, nt - 1);   // this lane's token row (clamped)
  const int hh = min(lrow, G - 1);                    // this lane's head column (clamped)
  const uint16_t* krow = a.tail_k + (row0 + tk) * rs + (int64_t)g * D + 8 * lhi;
  const uint16_t* qrow = a.q + ((int64_t)i * a.H_q + g * G + hh) * D + 8 * lhi;
  const uint16_t* vcol = a.tail_v + row0 * rs + (int64_t)g * D + DL * lane;
  bf16x8 kf[NK], qf[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    kf[k] = ld_bf16x8(krow + 16 * k);
    qf[k] = ld_bf16x8(qrow + 16 * k);
  }
  uint32_t vraw[kTokW];  // V[token][DL*lane .. +DL-1] as bf16 bits
#pragma unroll
  for (int tt = 0; tt < kTokW; ++tt) {
    const int64_t r = min(kTokW * wave + tt, nt - 1);
    if constexpr (DL == 2) vraw[tt] = *reinterpret_cast<const uint32_t*>(vcol + r * rs);
    else vraw[tt] = vcol[r * rs];
  }
  // scores: lane holds head column lrow, token rows 8(v/4) + 4 lhi + v%4 of the wave's 32
  f32x16 sc = {};
#pragma unroll
  for (int k = 0; k < NK; ++k) sc = mfma32(kf[k], qf[k], sc);
  float mx = -INFINITY;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int tw = 8 * (v >> 2) + 4 * lhi + (v & 3);
    const float x = kTokW * wave + tw < nt ? sc[v] * a.qscale : -INFINITY;
    sc[v] = x;
    mx = fmaxf(mx, x);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  red[wave * 32 + lrow] = mx;  // both lane halves hold the same value
  lds_barrier();
  float m = red[lrow];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) m = fmaxf(m, red[w * 32 + lrow]);
  float lsum = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int tw = 8 * (v >> 2) + 4 * lhi + (v & 3);
    const float w = fast_exp2(sc[v] - m);  // masked tokens: 2^-inf = 0
    lsum += w;
    wt[(kTokW * wave + tw) * 32 + lrow] = w;
  }
  lsum += __shfl_xor(lsum, 32);
  lred[wave * 32 + lrow] = lsum;
  lds_barrier();
  // values over the wave's own tokens (heads rounded up to 8 or 16)
  if (G <= 8) tail_values<D, 8>(wt + kTokW * wave * 32, vraw, op + wave * kMaxGroup * D + DL * lane);
  else tail_values<D, kMaxGroup>(wt + kTokW * wave * 32, vraw, op + wave * kMaxGroup * D + DL * lane);
  lds_barrier();
  for (unsigned x = tid; x < (unsigned)(G * D); x += kThreads) {
    const int h = x / D, dd = x % D;
    float o = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) o += op[(w * kMaxGroup + h) * D + dd];
    const int64_t col = (int64_t)i * a.H_q + g * G + h;
    a.part_o[(col * a.n_slots + slot) * D + dd] = o;
    if (dd == 0) {
      float mm = red[h], ll = 0.f;
#pragma unroll
      for (int w = 1; w < kWaves; ++w) mm = fmaxf(mm, red[w * 32 + h]);
#pragma unroll
      for (int w = 0; w < kWaves; ++w) ll += lred[w * 32 + h];
      a.part_ml[col * a.n_slots + slot] = make_float2(mm, ll);
    }
  }
}

// a work item read from LDS into wave-uniform registers
__device__ __forceinline__ WorkItem lds_item(const unsigned char* p) {
  static_assert(sizeof(WorkItem) == 80, "a work item is five 16-byte chunks");
  int32_t w[20];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int4 v = reinterpret_cast<const int4*>(p)[i];
    w[4 * i + 0] = __builtin_amdgcn_readfirstlane(v.x);
    w[4 * i + 1] = __builtin_amdgcn_readfirstlane(v.y);
    w[4 * i + 2] = __builtin_amdgcn_readfirstlane(v.z);
    w[4 * i + 3] = __builtin_amdgcn_readfirstlane(v.w);
  }
  WorkItem it;
  __builtin_memcpy(&it, w, sizeof(WorkItem));
  return it;
}

// A wave's fragment streams.  Fragments go from global memory straight into
// registers, each in its lane's MFMA operand layout, through two sets of slots
// that run ahead of the MFMAs: `ks` for R^K and P^K (projection and scores),
// `vs` for P^V (value pass).  A run of n steps ends on the last slot of a set of
// N: step f sits in slot (f - n) mod N, so a run takes first its n mod N odd
// steps from the last slots, then whole rounds from slot 0, and each slot is
// reloaded as it is consumed, with the step a round later or, past the run's
// end, with its step of the next run of that set (the next tiles, or the next
// item's first run).  Loads are issued in the order of use on every path, which
// is what lets the compiler wait for the slot in use alone (s_waitcnt vmcnt
// counts in order).  The set sizes are what the registers hold without a spill:
// a spilled value's scratch loads sit in the same in-order count and stop the
// streams.  A run's loads go through a buffer that ends with it, so the slots a
// short run leaves out read nothing (7B layer of 32 requests 193 -> 191 us, prefill
// of 45 tokens 84.4 -> 82.7, against reading on).
// (Streaming through per-wave LDS rings by direct global->LDS loads, as this
// kernel did before, cost two LDS passes and ~16 scalar instructions per
// fragment.)
//
// Measured, register streams against the LDS rings: 14B layer of 64 requests (ranks
// to 768) 2796 -> 1697 us, 7B layer of 32 requests 199 -> 172, prefill of 256 tokens
// 864 -> 743, 1M tokens 1574 -> 1371; one-tile blocks of ranks 17 .. 44 under a
// prefill of 228 tokens, where an item's set-up is all its time, 215 -> 214.
// (Two tiles per step, which halves the LDS reads per score, was measured too: the
// registers it takes send the group's output through memory, and it gained 2-5% on
// long items and lost up to 14% on short ones.)
// INT8 P factors: a slot holds the 8 codes of a lane, half the bytes, so there are
// twice as many where registers allow (four left 2 KiB of a wave's codes in flight:
// 7B layer of 8 requests 56.0 -> 52.4 us); R^K, which is bf16, has registers of its own.
template <bool I8, int MAX_RT>
struct Streams {
  using Slot = std::conditional_t<I8, uint2, bf16x8>;
  static constexpr int KD = I8 && MAX_RT < 4 ? 8 : 4;  // steps in a round of ks
  static constexpr int VD = KD;  // P^V fragments loaded ahead across tiles
  Slot ks[KD], vs[VD];
};

// f(integral constant i) for i = FROM, FROM + STEP, .. below TO
template <int FROM, int TO, int STEP, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (FROM < TO) {
    f(std::integral_constant<int, FROM>{});
    static_for<FROM + STEP, TO, STEP>(f);
  }
}

// A wave-uniform fragment address p + off loaded by every lane: buffer loads
// take the base and offset in scalar registers, the lane's part in one vector
// register.  wanted is -1, or 0: nothing is read (an empty buffer), the slot
// gets zeros; or the bytes of p's run, past which nothing is read either; as
// arithmetic on a scalar it costs no branch in the loops.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t frag_buffer(const unsigned char* p, int wanted) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(p), 0, __builtin_amdgcn_readfirstlane(wanted),
                                           0x00020000);
}
// -1 where a < b (both far from the ends of the int range), else 0
__device__ __forceinline__ int mask_lt(int a, int b) { return (a - b) >> 31; }
__device__ __forceinline__ bf16x8 load_frag16(const unsigned char* p, int off, int lane16, int wanted = -1) {
  return __builtin_bit_cast(bf16x8,
                            __builtin_amdgcn_raw_buffer_load_b128(frag_buffer(p, wanted), lane16, off, 0));
}
__device__ __forceinline__ uint2 load_frag8(const unsigned char* p, int off, int lane8, int wanted) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(frag_buffer(p, wanted), lane8, off, 0));
}
// Behind a slot's reload in the rounds of the tile loop: neither memory accesses
// nor MFMAs move across it (VALU, SALU and LDS may).  The scheduler otherwise
// gathers a round's reloads behind its MFMAs, which leaves 2 to 5 loads in flight
// where 7 could be.  Not where an item starts: there it costs a short item 2%.
__device__ __forceinline__ void pin_load() { __builtin_amdgcn_sched_barrier(0x0086); }
// Where the slots of a set of N find their first steps of a run of n steps at p
// (fragments of B bytes): slot s holds step (s + n) mod N.  n = 0: no run.
template <int N, int B>
struct RunStart {
  const unsigned char* p;
  int odd, wanted;  // wanted: the bytes of the run
  __device__ __forceinline__ RunStart(const unsigned char* p_, int n) : p(p_), odd(n & (N - 1)), wanted(n * B) {}
  __device__ __forceinline__ int off(int s) const { return (s + odd - (s + odd >= N ? N : 0)) * B; }
};
// Consume a run of n steps (an even number) at p through slots 0 .. N-1: use(f, s)
// takes slot s for step f + s, load(s, q, off, wanted) reloads it from q + off;
// next: the set's next run.  The odd steps before the whole rounds are one
// straight piece of code per count, so that their operand reads overlap; step by
// step behind branches they cost as much as two rounds.
template <int N, int B, typename Use, typename Load>
__device__ __forceinline__ void consume_run(const unsigned char* p, int n, const RunStart<N, B>& next, Use&& use,
                                            Load&& load) {
  const int odd = n & (N - 1);
  const bool more = n >= N;
  static_for<2, N, 2>([&](auto odd_c) {
    constexpr int ODD = decltype(odd_c)::value;
    if (odd != ODD) return;
    if (!more) {  // a run shorter than a round: the slots it leaves out move on too
      static_for<0, N - ODD, 1>([&](auto s) { load(s, next.p, next.off(s), next.wanted); });
    }
    const unsigned char* q = more ? p : next.p;
    const int wanted = more ? n * B : next.wanted;
    static_for<N - ODD, N, 1>([&](auto s) {
      use(ODD - N, s);
      load(s, q, more ? (ODD + s) * B : next.off(s), wanted);
    });
  });
#pragma clang loop unroll(disable)
  for (int f = odd; f < n; f += N) {
    const bool last = f + N >= n;
    const int wanted = last ? next.wanted : n * B;
    const unsigned char* q = last ? next.p : p;
    const int lo = last ? next.odd * B : (f + N) * B, hi = last ? lo - N * B : lo, wrap = N - next.odd;
    static_for<0, N, 1>([&](auto s) {
      use(f, s);
      load(s, q, (s < wrap ? lo : hi) + s * B, wanted);
      pin_load();
    });
  }
}

// The first run of a block item (bf16 P factors) for wave `wave`, at p: R^K if
// the wave owns projection rank tiles, else the first tile's P^K
__device__ __forceinline__ RunStart<Streams<false, 2>::KD, kFragElems * 2> item_first_run(const WorkItem* it, int wave,
                                                                                   const unsigned char* p) {
  const int rk_pad = __builtin_amdgcn_readfirstlane(it->blk.rk_pad);
  const bool dense = (__builtin_amdgcn_readfirstlane(it->flags) & kItemDense) != 0;
  const bool rk = !dense && owned_tiles(rk_pad >> 5, wave, kWaves) > 0;
  return RunStart<Streams<false, 2>::KD, kFragElems * 2>(p, rk ? Streams<false, 2>::KD : rk_pad >> 4);
}

// The waves' run lists: for each of its block items a wave finds the first
// fragment of the runs it consumes (block_runs) in an LDS buffer that the last wave
// fills for all eight (RunDeriver) two block items ahead, four buffers
// used in turn: the buffer being refilled is two items behind, and the next
// item's list is complete while the current item runs.  After the last block
// item a run of the buffer's first fragments follows (loaded, never used).
struct RunList {
  const int2* rbuf;  // this wave's kRunBufs buffers of run_cap entries
  int run_cap, rb;   // entries per buffer; the current item's buffer
  __device__ __forceinline__ int first(int k) const { return __builtin_amdgcn_readfirstlane(rbuf[rb * run_cap + k].x); }
  __device__ __forceinline__ int next_first() const {
    return __builtin_amdgcn_readfirstlane(rbuf[((rb + 1) % kRunBufs) * run_cap].x);
  }
  __device__ __forceinline__ void advance() { rb = (rb + 1) % kRunBufs; }
};

// Derivation of the run lists, done by the last wave for all eight (lane w
// derives wave w's runs, in vector registers) while the others project: it owns
// the fewest projection rank tiles, none up to rank 224: the runs of the workgroup's
// next block item, or the closing run after the last one, into every wave's
// buffer gb.  Runs are read by their wave only after a later workgroup
// barrier.
template <int D>
struct RunDeriver {
  const unsigned char* items;  // the workgroup's work items (LDS)
  int n_items;
  int gk;                      // next item to look at
  int gb;                      // buffer the next derivation fills
  int2* rbuf;                  // all waves' run buffers: [wave][kRunBufs][run_cap]
  int run_cap;
  int recon_delta;             // fragments from the factor buffer to the reconstruction buffer

  __device__ void derive(int lane) {
    WorkItem it{};
    bool found = false;
    while (gk < n_items) {
      it = lds_item(items + (size_t)gk * sizeof(WorkItem));
      ++gk;
      if (it.kind == kItemBlock) {
        found = true;
        break;
      }
    }
    if (lane < kWaves) {
      int2* out = rbuf + ((size_t)lane * kRunBufs + gb) * run_cap;
      int n = 0;
      auto put = [&](int x, int cnt) { out[n++] = make_int2(x, cnt); };
      if (found)
        block_runs(it.blk, it.g, ((it.flags >> kItemHeadsShift) & 7) + 1, it.tile0, it.ntile, lane, D,
                   (it.flags >> kItemLgNgShift) & 3, (it.flags & kItemInt8) != 0, put, (it.flags & kItemDense) != 0,
                   recon_delta);
      else put(0, 0);
    }
    gb = (gb + 1) % kRunBufs;
  }
};

// A workgroup's running partial for its current group of block items (one KV
// head and column tile): the output in the up-projection's layout (NCB 16-column
// blocks of two 16-dim slices), the per-column maximum in the score layout (32 ch +
// lane % 32; every wave holds it), the per-column sum in wave 0 (thread t: column
// t).  Only plans of at most two rank tiles per wave fold items into groups.
// (Folding in place in the group's slot instead cost a short item 1.1 of its 10 us:
// the stores sit in the same in-order count as the streams' loads.)
template <int NCB>
struct GroupAcc {
  f32x4 o[NCB][2];
  float m[2];
  float l;
};
template <int D>
constexpr int up_col_blocks() {
  return D / 64;  // 16-column blocks per wave in the up-projection (two slices)
}
// 16-byte chunks of an item's query rows a thread loads, and the load: chunk x
// of the 64 rows of a column tile (first column c0, cn columns)
template <int D>
constexpr int query_loads() {
  return kCols * (D / 8) / kThreads;
}
template <int D>
__device__ __forceinline__ void load_queries(const AttendArgs& a, int c0, int cn, int tid,
                                             bf16x8 (&qv)[query_loads<D>()]) {
#pragma unroll
  for (int u = 0; u < query_loads<D>(); ++u) {
    const unsigned x = opaque(tid) + u * kThreads, cl = x / (D / 8), j = x % (D / 8);
    qv[u] = ld_bf16x8(a.q + query_row(a, c0 + min((int)cl, cn - 1)) * D + 8 * j);
  }
}

// ---------------------------------------------------------------------------
// Block work item: latent-space attention of one column tile (at most 64
// consecutive head-major query columns, of up to kMaxTileHeads KV heads) over
// the tiles [tile0, tile0 + ntile) of block b.  The scores and the latent
// value pass do not depend on the head (P^K and P^V are shared by all KV
// heads); the projection and the up-projection run once per KV head of the
// tile, each column keeping the result of its own head.
//
// Eight waves (two per SIMD).  Scores: wave w takes the 32 tokens 32w..32w+31
// of every 256-token tile against all 64 columns.  Latent V: the waves form
// nseg token segments x ng rank groups (see the packed layout), so each wave
// accumulates its own rank tiles over its own tokens; the segments' partial
// sums are then combined in LDS and the latent result goes to LDS as bf16.
// Up-projection: each wave computes a 16-dim slice of the output for all 64
// columns over all ranks.  Every factor fragment a wave consumes (R^K for the
// projection, P^K and P^V per tile, R^V for the up-projection) comes through
// the wave's register slots (Streams above); the item's queries are loaded into
// LDS at its start.
// ---------------------------------------------------------------------------
// MODE: 0 bf16 P factors, 1 INT8 P factors, 2 bf16 P factors with the
// projection as a wavefront GEMV (kernel variants, so no branch of one costs
// the others registers)
// FETCH: the gang's workgroups fetch the coming tile's P into L2 between them
template <int D, int MAX_RT, bool FETCH, int MODE>
__device__ __forceinline__ void block_item(const AttendArgs& a, const WorkItem& it, unsigned char* smem,
                                           Streams<MODE == 1, MAX_RT>& fs, RunList& rl, RunDeriver<D>& rd,
                                           GroupAcc<up_col_blocks<D>()>& acc, bf16x8 (&qv)[query_loads<D>()], const WorkItem* next_item,
                                           const int tid) {
  constexpr bool I8 = MODE == 1, GV = MODE == 2;
  constexpr int NK = D / 16;
  constexpr int KD = Streams<I8, MAX_RT>::KD, VD = Streams<I8, MAX_RT>::VD;
  using Slot = typename Streams<I8, MAX_RT>::Slot;
  static_assert(I8 || NK == KD || NK == 2 * KD, "an R^K rank tile is one or two rounds");
  const BlockMeta& bm = it.blk;
  const int slot = it.slot, g0 = it.g, c0 = it.req;
  const int cn = ((it.flags >> kItemColsShift) & 63) + 1;  // columns of the tile
  const int nh = ((it.flags >> kItemHeadsShift) & 7) + 1;  // KV heads of the tile
  // a reconstructed block: bm names K_{b,g} / V_{b,g} of the tile's one KV head
  // (rank d); the query takes the projection's place and the value pass gives
  // the output
  const bool dense = (it.flags & kItemDense) != 0;
  const bool causal = (it.flags & kItemCausal) != 0;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 31, lhi = lane >> 5;
  const int G = a.G, N_g = a.N_g;
  const int qsd = a.qt_stride;
  const int nrt_k = bm.rk_pad >> 5, nks = bm.rk_pad >> 4;
  const int nrt_v = bm.rv_pad >> 5;
  const int own_k = owned_tiles(nrt_k, wave, kWaves);
  // the split of the value pass, nseg = 8 / ng segments x ng = 2^lg_ng rank groups
  // (v_segments); shifts, since divisions by ng cost a short item half a microsecond
  const int lg_ng = (it.flags >> kItemLgNgShift) & 3, ng = 1 << lg_ng, nseg = kWaves >> lg_ng;
  const int rg = wave & (ng - 1), sg = wave >> lg_ng;
  const int own_v = (nrt_v >> lg_ng) + (rg < (nrt_v & (ng - 1)) ? 1 : 0);
  const int nst = 2 << lg_ng;               // 16-token steps of the wave's segment per tile
  const int T = bm.T;
  constexpr int kTouches = FETCH ? 2 : 0;  // lines a lane fetches ahead for the gang per tile
  const int gang_at = (it.flags >> kItemGangShift) & 31;
  const int ntiles = it.ntile, tile0 = it.tile0;  // tiles this item covers
  // causal limits of this lane's two columns (32 ch + lane % 32; request (c mod N_g) / G)
  // and the smallest over the tile (wave-uniform), past which tokens need masking
  int lim[2] = {T, T}, lim_min = T;
  if (causal) {
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      const int c = c0 + min(32 * ch + (lane & 31), cn - 1);
      lim[ch] = tail_len_of(a.tl, div_by(c - div_by(c, N_g, a.N_g_inv) * N_g, G, a.G_inv));
    }
    lim_min = min(lim[0], lim[1]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lim_min = min(lim_min, __shfl_xor(lim_min, off));
  }
  __bf16* qt = reinterpret_cast<__bf16*>(smem);             // [kCols][qsd]
  constexpr int kWS = kWStride;
  __bf16* wl = qt + kCols * qsd;                            // [kCols][kWS] the tile's weights
  float* red = reinterpret_cast<float*>(wl + kCols * kWS);  // [kWaves][kCols]

  // the runs of this item (first unit of each; P^K and P^V of consecutive tiles
  // follow at constant strides) and the first run of the next one
  const unsigned char* data = reinterpret_cast<const unsigned char*>(a.data);
  constexpr int kFragBytes = kFragElems * 2;
  constexpr int kPBytes = I8 ? kFragElems : kFragElems * 2;  // a P^K / P^V fragment
  const int n_rk = own_k > 0 && !dense ? nh : 0, per_tile = 1 + (I8 ? 1 : 0) + (own_v > 0 ? 1 : 0);
  const unsigned char* rkp = data + (int64_t)rl.first(0) * kFragBytes;
  const unsigned char* pkp = data + (int64_t)rl.first(n_rk) * kPBytes;
  const unsigned char* pvp = data + (own_v > 0 ? (int64_t)rl.first(n_rk + 1 + (I8 ? 1 : 0)) * kPBytes : 0);
  const unsigned char* scp = data + (I8 ? (int64_t)rl.first(n_rk + 1) * kScaleUnitBytes : 0);
  const RunStart<KD, kPBytes> pk_first(pkp, nks);
  const int lane16 = 16 * lane;
  auto ldf = [&](const unsigned char* p, int off, int wanted = -1) {  // a bf16 fragment
    return load_frag16(p, off, lane16, wanted);
  };
  // a P^K / P^V fragment: bf16, or int8 codes (converted exactly as they are used)
  auto ldp = [&](const unsigned char* p, int off, int wanted = -1) -> Slot {
    if constexpr (I8) return load_frag8(p, off, lane16 >> 1, wanted);
    else return load_frag16(p, off, lane16, wanted);
  };
  auto use_p = [&](const Slot& x) -> bf16x8 {
    if constexpr (I8) return i8_to_bf16x8(x);
    else return x;
  };
  // f(rank tiles this wave owns in the value pass, 16-token steps in a round of
  // it), as integral constants: a round is up to eight fragments, the first VD
  // of them loaded across tiles (vs), the rest within a tile.  A wave owns three
  // tiles or more only in a single segment of 16 steps (v_segments)
  static_assert(v_segments(1) == 8 && v_segments(2) == 4 && v_segments(3) == 2 && v_segments(4) == 2 &&
                v_segments(5) == 2 && v_segments(8) == 2 && v_segments(9) == 1, "rounds of the value pass");
  auto with_own = [&](auto&& f) {
    if (own_v == 1) {
      if (nst >= 8) f(std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{});
      else if (nst == 4) f(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
      else f(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
    } else if (own_v == 2) {
      f(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    }
    if constexpr (MAX_RT >= 3)
      if (own_v == 3) f(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{});
    if constexpr (MAX_RT >= 4)
      if (own_v == 4) f(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
  };

  // ---- the item's 64 query rows (qv, loaded during the previous item) -> LDS
  // (in the weight tile's area, idle until the first tile).  Row-major
  // [column][D]; the 16-byte chunk j of column c is stored at chunk position
  // j ^ (c % kRowChunks), so the projection's operand reads (same chunk, 32
  // columns) hit distinct banks.  Columns past the tile's
  // last one re-read the last column's query and count as its head (their
  // results are never stored).
  constexpr int kRowChunks = D / 8;  // 16-byte chunks per query row
  constexpr int kQLoads = query_loads<D>();
  __bf16* qimg = wl;
  // steps kRkSlots .. of an R^K rank tile (those before sit in ks; INT8: none do)
  constexpr int kRkSlots = I8 ? 0 : KD, kMoreRk = NK - kRkSlots;
  bf16x8 rk_more[kMoreRk > 0 ? kMoreRk : 1];
  {
#pragma unroll
    for (int u = 0; u < kQLoads; ++u) {
      const unsigned x = opaque(tid) + u * kThreads, cl = x / kRowChunks, j = x % kRowChunks;
      *reinterpret_cast<bf16x8*>(qimg + cl * D + 8 * (j ^ (cl % kRowChunks))) = qv[u];
    }
    // the rest of the first R^K rank tile, then (INT8: the previous item could not
    // load it) the first tile's P^K, then its P^V
    static_for<0, kMoreRk, 1>([&](auto i) {
      rk_more[decltype(i)::value] = ldf(rkp, (i + kRkSlots) * kFragBytes, mask_lt(0, n_rk));
    });
    if constexpr (I8)
      static_for<0, KD, 1>([&](auto i) { fs.ks[decltype(i)::value] = ldp(pk_first.p, pk_first.off(i), pk_first.wanted); });
    static_for<0, VD, 1>([&](auto x) { forget(fs.vs[decltype(x)::value]); });
    with_own([&](auto own_c, auto cs_c) {
      constexpr int n = decltype(own_c)::value * decltype(cs_c)::value;
      static_for<0, (n < VD ? n : VD), 1>([&](auto x) { fs.vs[decltype(x)::value] = ldp(pvp, x * kPBytes); });
    });
    lds_barrier();
    if (wave == kWaves - 1) rd.derive(lane);  // the runs of the block item two ahead
  }

  auto load_pk_first = [&]() {
    static_for<0, KD, 1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      fs.ks[i] = ldp(pk_first.p, pk_first.off(i), pk_first.wanted);
    });
  };
  // ---- projection: Qt[rank][col] (stored [col][rank]), once per KV head of
  // the tile; each column stores its own head's result.  Dense items: Qt is
  // the query itself times the sign of the scale, as fp16 (exact for the
  // bf16 query in fp16's normal range; saturated at +-65504) to meet the
  // rebuilt keys, which are fp16 too, in the fp16 score MFMA; the scale's
  // magnitude goes onto the fp32 scores (sscale below).  A scaled query
  // rounded to 16 bits would put a relative rounding error on every score,
  // which a peaked softmax magnifies ----
  if (dense) {
    const float sgn = a.qscale > 0.f ? 1.f : a.qscale < 0.f ? -1.f : 0.f;
    for (int x = tid; x < kCols * kRowChunks; x += kThreads) {
      const int cl = x / kRowChunks, j = x % kRowChunks;
      const bf16x8 v = ld_bf16x8(qimg + cl * D + 8 * (j ^ (cl % kRowChunks)));
      f16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (_Float16)fminf(fmaxf((float)v[e] * sgn, -65504.f), 65504.f);
      *reinterpret_cast<f16x8*>(qt + cl * qsd + 8 * j) = o;
    }
  } else if (GV && own_k > 0) {
    // small batches (a tile of at most kGemvCols columns): the projection as a
    // wavefront GEMV.  Lane (c, m) of an R^K fragment holds rank 32 rt + m, dims
    // 16 k + 8 c .. +7; it dots them with the same dims of every column of the
    // current head (the query row chunk is one LDS broadcast), the two lane
    // halves are summed, and lanes m < 32 store their rank of the head's columns.
    // Columns past the tile's last one get zeros.
    for (int x = 0; x < nh * own_k; ++x) {
      const int hh = x / own_k, rt = wave + kWaves * (x - hh * own_k);
      // the head's columns are the consecutive range [lo, hi) of the tile
      const int lo = max(0, (g0 + hh) * N_g - c0), hi = min(cn, (g0 + hh + 1) * N_g - c0);
      float acc[kGemvCols];
#pragma unroll
      for (int cl = 0; cl < kGemvCols; ++cl) acc[cl] = 0.f;
      const unsigned char* rp = rkp + ((int64_t)hh * nrt_k * NK + (x - hh * own_k) * NK) * kFragBytes;
      for (int k = 0; k < NK; ++k) {
        const bf16x8 af = ldf(rp, k * kFragBytes);
        float rf[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) rf[e] = (float)af[e];
        // every one of the kGemvCols query rows (rows past the tile's columns
        // hold a copy of its last one); only the head's columns are stored
#pragma unroll
        for (int cl = 0; cl < kGemvCols; ++cl) {
          const bf16x8 qv = ld_bf16x8(qimg + cl * D + 8 * ((2 * k + lhi) ^ (cl % kRowChunks)));
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[cl] = fmaf(rf[e], (float)qv[e], acc[cl]);
        }
      }
#pragma unroll
      for (int cl = 0; cl < kGemvCols; ++cl) {
        acc[cl] += __shfl_xor(acc[cl], 32);
        if (lhi == 0 && cl >= lo && cl < hi) qt[cl * qsd + 32 * rt + lrow] = (__bf16)(acc[cl] * a.qscale);
      }
      if (hh == 0)
        for (int cl = cn + lhi; cl < kCols; cl += 2) qt[cl * qsd + 32 * rt + lrow] = (__bf16)0.f;
    }
    load_pk_first();
  } else if (own_k > 0) {
    const int ln = opaque(lane), lrow = ln & 31, lhi = ln >> 5;
    bf16x8 qf[NK][2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch)
#pragma unroll
      for (int k = 0; k < NK; ++k)
        qf[k][ch] = ld_bf16x8(qimg + (32 * ch + lrow) * D + 8 * ((2 * k + lhi) ^ (lrow % kRowChunks)));
    // KV head (relative to g0) of this lane's two columns 32 ch + lrow
    const int hq0 = div_by(c0 + min(lrow, cn - 1), N_g, a.N_g_inv) - g0;
    const int hq1 = div_by(c0 + min(32 + lrow, cn - 1), N_g, a.N_g_inv) - g0;
    const int nx = nh * own_k;
    for (int x = 0, hh = 0, j = 0; x < nx; ++x) {
      const int rt = wave + kWaves * j;
      // each step's slot is reloaded with the same step of the next rank tile (the
      // next head's run starts nrt_k NK fragments on; past the last, P^K)
      const unsigned char* after = rkp + (j + 1 < own_k ? (int64_t)hh * nrt_k + j + 1 : (int64_t)(hh + 1) * nrt_k) * NK * kFragBytes;
      const bool to_pk = x + 1 == nx;
      f32x16 acc0 = zero16(), acc1 = zero16();
      static_for<0, NK, 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k >= kRkSlots) {
          bf16x8& slot = rk_more[k - kRkSlots];
          acc0 = mfma32(slot, qf[k][0], acc0);
          acc1 = mfma32(slot, qf[k][1], acc1);
          slot = ldf(after, k * kFragBytes, mask_lt(x + 1, nx));
        } else if constexpr (!I8) {
          acc0 = mfma32(fs.ks[k], qf[k][0], acc0);
          acc1 = mfma32(fs.ks[k], qf[k][1], acc1);
          fs.ks[k] = ldf(to_pk ? pk_first.p : after, to_pk ? pk_first.off(k) : k * kFragBytes,
                         to_pk ? pk_first.wanted : mask_lt(x + 1, nx));
        }
      });
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        bf16x4 v0, v1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          v0[u] = (__bf16)(acc0[4 * jj + u] * a.qscale);
          v1[u] = (__bf16)(acc1[4 * jj + u] * a.qscale);
        }
        const int r = 32 * rt + 8 * jj + 4 * lhi;
        if (hq0 == hh) *reinterpret_cast<bf16x4*>(qt + lrow * qsd + r) = v0;
        if (hq1 == hh) *reinterpret_cast<bf16x4*>(qt + (32 + lrow) * qsd + r) = v1;
      }
      if (++j == own_k) j = 0, ++hh;
    }
  }
  lds_barrier();

  // ---- scores, online softmax, latent V: the tile loop, then the value pass's
  // result into LDS.  One instance per number of rank tiles a wave owns in the
  // value pass, and one for dense items, so that each keeps its own accumulators
  // and nothing else in registers ----
  float m_run[2] = {-INFINITY, -INFINITY};
  float l_run[2] = {0.f, 0.f};
  float* lred = reinterpret_cast<float*>(smem + a.work_bytes) - kWaves * kCols;  // [kWaves][kCols]
  // up-projection: a wave takes two 16-dim slices of the output for a half
  // (d = 128) or a quarter (d = 64) of the columns, so that each latent operand
  // read from LDS feeds two MFMAs; rounds of kRvSteps 32-rank steps
  constexpr int NDS = D / 16, kRvSteps = 4;
  // (a tile of at most 32 columns, in its first half: one slice per wave, and the
  // second fragment of a slot is the same slice kRvSteps steps on)
  const bool narrow = cn <= 32;
  const int ds0 = narrow ? wave % NDS : 2 * (wave % (NDS / 2));  // the first slice
  const int nk_v = bm.rv_pad >> 5;
  const unsigned char* rvp = data + rv_frag(bm, D, g0, ds0, 0) * kFragBytes;
  bf16x8 rv[kRvSteps][2];
  // its first round: a slice's steps past the ranks lie past the end of its
  // buffer and are not read
  auto load_rv_first = [&]() {
    const int end = nk_v * kFragBytes;
    const int end2 = narrow ? max(end - kRvSteps * kFragBytes, 0) : end;
    const __amdgpu_buffer_rsrc_t r0 = frag_buffer(rvp, end);
    const __amdgpu_buffer_rsrc_t r1 = frag_buffer(rvp + (narrow ? kRvSteps : nk_v) * kFragBytes, end2);
    static_for<0, kRvSteps, 1>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      rv[i][0] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r0, lane16 + i * kFragBytes, 0, 0));
      rv[i][1] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r1, lane16 + i * kFragBytes, 0, 0));
    });
  };
  auto tiles = [&](auto own_c, auto cs_c, auto dense_c) {
    constexpr int OWN = decltype(own_c)::value, CS = decltype(cs_c)::value;
    constexpr bool DENSE = decltype(dense_c)::value;
    f32x16 oacc[OWN > 0 ? OWN : 1][2];
#pragma unroll
    for (int r = 0; r < OWN; ++r) oacc[r][0] = oacc[r][1] = zero16();
    // factor (> 0) from the MFMA's raw scores to scores in log2 units: the
    // magnitude of the scale for dense items, 1 otherwise (the projection
    // carries it); applied in the column maximum and the weights' exponent
    const float sscale = DENSE && a.qscale != 0.f ? fabsf(a.qscale) : 1.f;

    for (int tt = 0; tt < ntiles; ++tt) {
      const int after = tt + 1;
      float scale_unit = 0.f;  // INT8: this lane's entry of the wave's scale unit
      if constexpr (I8) scale_unit = reinterpret_cast<const float*>(scp + (int64_t)tt * kWaves * kScaleUnitBytes)[lane];
      // rank step k (P^K sub-tile, or rebuilt keys) times the two column halves
      // of Qt; dense items multiply fp16 operands.  The next K run: the next
      // tile's, then the next item's first (INT8: loaded by that item)
      f32x16 sc[2] = {zero16(), zero16()};
      {
        const int ln = opaque(lane);
        const __bf16* qr0 = qt + (ln & 31) * qsd + 8 * (ln >> 5);
        const __bf16* qr1 = qr0 + 32 * qsd;
        const unsigned char* kb = pkp + (int64_t)tt * nks * kPBytes;
        RunStart<KD, kPBytes> kn(kb + (int64_t)nks * kPBytes, nks);
        if (after >= ntiles) {
          kn.wanted = 0;
          if constexpr (!I8)
            if (next_item) kn = item_first_run(next_item, wave, data + (int64_t)rl.next_first() * kPBytes);
        }
        auto use = [&](int f, auto slot) {
          constexpr int i = decltype(slot)::value;
          const bf16x8 b0 = ld_bf16x8(qr0 + 16 * f + 16 * i), b1 = ld_bf16x8(qr1 + 16 * f + 16 * i);
          const bf16x8 ak = use_p(fs.ks[i]);
          sc[0] = DENSE ? mfma32_f16(ak, b0, sc[0]) : mfma32(ak, b0, sc[0]);
          sc[1] = DENSE ? mfma32_f16(ak, b1, sc[1]) : mfma32(ak, b1, sc[1]);
        };
        consume_run(kb, nks, kn, use, [&](auto slot, const unsigned char* q, int off, int wanted) {
          fs.ks[decltype(slot)::value] = ldp(q, off, wanted);
        });
      }
      const int ln = opaque(lane), lrow = ln & 31, lhi = ln >> 5;
      // INT8 P factors: the scores of int8 codes times each token's K scale (lane:
      // tokens 8 j + 4 lhi + v of the wave's 32, j, v = 0..3); the V scales fold
      // into the weights below.  The unit is spread through the wave's own maxima
      // row, which nobody reads before the maxima below are in it
      float vsc[16];
      if constexpr (I8) {
        float* su = red + wave * kCols;
        su[ln] = scale_unit;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 k4 = *reinterpret_cast<const float4*>(su + 8 * j + 4 * lhi);
          const float4 v4 = *reinterpret_cast<const float4*>(su + 32 + 8 * j + 4 * lhi);
          const float kk[4] = {k4.x, k4.y, k4.z, k4.w};
          vsc[4 * j] = v4.x, vsc[4 * j + 1] = v4.y, vsc[4 * j + 2] = v4.z, vsc[4 * j + 3] = v4.w;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            sc[0][4 * j + v] *= kk[v];
            sc[1][4 * j + v] *= kk[v];
          }
        }
      }
      // mask tokens past the end of the block (only the block's last tile can
      // hold any; the test is wave-uniform), and for a prefill chunk's shared
      // tail the tokens past each column's causal limit; wave-local column max
      float mx[2] = {-INFINITY, -INFINITY};
      const int tw = (tile0 + tt) * kTile + wave * kTokWave;
      if (tw + kTokWave > T || (DENSE && causal && tw + kTokWave > lim_min)) {
#pragma unroll
        for (int ch = 0; ch < 2; ++ch)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int tok = tw + 8 * (v >> 2) + 4 * lhi + (v & 3);
            if (tok >= T || (DENSE && tok >= lim[ch])) sc[ch][v] = -INFINITY;
          }
      }
#pragma unroll
      for (int ch = 0; ch < 2; ++ch)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx[ch] = fmaxf(mx[ch], sc[ch][v]);
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        mx[ch] = fmaxf(mx[ch], __shfl_xor(mx[ch], 32)) * sscale;
        red[wave * kCols + 32 * ch + lrow] = mx[ch];  // both lane halves hold the same value
      }
      lds_barrier();
      // The gang's workgroups read the same P at the same time, so what they have
      // in flight from HBM together is only one workgroup's: each fetches its share
      // of the wave's coming fragments (this tile's P^V, then the next one's P^K,
      // in 64 lines of 128 bytes) into the XCD's L2.  Loads return in order, so the
      // value pass' first fragments past the slots (vx below) wait for the fetch
      // too; issued after that pass it came too late to help.  Dense items of one
      // gang read different K and V and fetch nothing
      uint32_t touched[kTouches > 0 ? kTouches : 1];
      if constexpr (kTouches > 0) {
        const int lane128 = 128 * opaque(lane);
        const int v_lines = OWN > 0 ? nst * OWN * (kPBytes / 128) : 0, v_chunks = (v_lines + 63) >> 6;
        const int k_lines = after < ntiles ? nks * (kPBytes / 128) : 0;
#pragma unroll
        for (int l = 0; l < kTouches; ++l) {
          const int c = gang_at + l * a.gang;
          const bool k_part = c >= v_chunks;
          const int at = (k_part ? c - v_chunks : c) * 8192;
          const unsigned char* base = k_part ? pkp + (int64_t)after * nks * kPBytes : pvp + (int64_t)tt * 16 * OWN * kPBytes;
          // an empty buffer past the part's end, and for a gang of one
          const int bytes = !DENSE && a.gang > 1 ? max(0, min(8192, (k_part ? k_lines : v_lines) * 128 - at)) : 0;
          const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
              const_cast<unsigned char*>(base) + at, 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
          touched[l] = __builtin_amdgcn_raw_buffer_load_b32(r, lane128, 0, 0);
        }
      }
      float alpha[2];
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        float tm = red[32 * ch + lrow];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) tm = fmaxf(tm, red[w * kCols + 32 * ch + lrow]);
        const float mn = fmaxf(m_run[ch], tm);
        // a column with no key so far (a causal column before its first token)
        // keeps m = -inf and zero weights
        alpha[ch] = mn == -INFINITY ? 1.f : fast_exp2(m_run[ch] - mn);
        m_run[ch] = mn;
      }
      // weights W = 2^(s - m) (bf16) to LDS as [col][token]
#pragma unroll
      for (int ch = 0; ch < 2; ++ch) {
        float lsum = 0.f;
        const float mref = m_run[ch] == -INFINITY ? 0.f : m_run[ch];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          bf16x4 wv;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float w = fast_exp2(fmaf(sc[ch][4 * j + v], sscale, -mref));
            lsum += w;
            if constexpr (I8) wv[v] = (__bf16)(w * vsc[4 * j + v]);
            else wv[v] = (__bf16)w;
          }
          *reinterpret_cast<bf16x4*>(wl + (32 * ch + lrow) * kWS + wave * kTokWave + 8 * j + 4 * lhi) = wv;
        }
        l_run[ch] = l_run[ch] * alpha[ch] + lsum;
        // summed here: left to itself the compiler keeps all the weights to sum them later
        asm volatile("" : "+v"(l_run[ch]));
      }
      if constexpr (OWN > 0) {
        // latent V over the wave's token segment of each tile: 16-token step st is
        // slots st % CS (its OWN rank tiles), reloaded a round ahead: this tile's,
        // then the next tile's; the slots past VD hold a step's fragments only
        // here (the scores' registers are free)
        constexpr int NF = CS * OWN;  // fragments in a round
        Slot vx[NF > VD ? NF - VD : 1];
        const unsigned char* vb = pvp + (int64_t)tt * 16 * OWN * kPBytes;
        static_for<VD, NF, 1>([&](auto x) { vx[decltype(x)::value - VD] = ldp(vb, x * kPBytes); });
        lds_barrier();
        // rescale the latent accumulators to the new running maximum; skipped on
        // the first tiles (they are zero) and when no column's maximum moved
        if (tt > 0 && __any(alpha[0] != 1.f || alpha[1] != 1.f)) {
#pragma unroll
          for (int r = 0; r < OWN; ++r) {
            oacc[r][0] *= alpha[0];
            oacc[r][1] *= alpha[1];
          }
        }
        const int steps = OWN > 2 ? 16 : nst;  // a whole number of rounds
        // weight operand rows of the wave's segment (relative step st at 16 st)
        const __bf16* wr0 = wl + lrow * kWS + 8 * lhi + 16 * nst * sg;
        const __bf16* wr1 = wr0 + 32 * kWS;
#pragma clang loop unroll(disable)
        for (int st = 0; st < steps; st += CS) {
          const int in_step = mask_lt(st + CS, steps);
          const int wanted = in_step | mask_lt(after, ntiles);
          const int on = (st + CS >= steps ? 16 : st + CS) * OWN * kPBytes;
          static_for<0, CS, 1>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const bf16x8 w0 = ld_bf16x8(wr0 + 16 * st + 16 * i), w1 = ld_bf16x8(wr1 + 16 * st + 16 * i);
            static_for<0, OWN, 1>([&](auto rc) {
              constexpr int r = decltype(rc)::value, x = i * OWN + r;
              Slot& slot = [&]() -> Slot& {
                if constexpr (x < VD) return fs.vs[x];
                else return vx[x - VD];
              }();
              const bf16x8 pa = use_p(slot);
              oacc[r][0] = mfma32(pa, w0, oacc[r][0]);
              oacc[r][1] = mfma32(pa, w1, oacc[r][1]);
              slot = ldp(vb, on + x * kPBytes, x < VD ? wanted : in_step);
              pin_load();
            });
          });
        }
      } else {
        lds_barrier();
      }
#pragma unroll
      for (int l = 0; l < kTouches; ++l) asm volatile("" ::"v"(touched[l]));
    }

    // the up-projection's first R^V steps load while the partials are combined
    if constexpr (!DENSE) load_rv_first();
    const int ln = opaque(lane), lrow = ln & 31, lhi = ln >> 5;
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) l_run[ch] += __shfl_xor(l_run[ch], 32);
    lds_barrier();  // every wave is done with qt / wl
    lred[wave * kCols + lrow] = l_run[0];  // both lane halves hold the sums
    lred[wave * kCols + 32 + lrow] = l_run[1];
    // combine the token segments' latent partials (pairwise rounds through LDS,
    // fp32): the waves of segments [h, 2h) hand theirs to segments [0, h)
    if (nseg > 1) {
      float4* segbuf = reinterpret_cast<float4*>(smem);  // [slot][owned tile][ch][4][64 lanes]
      const int own_max = (nrt_v + ng - 1) >> lg_ng;    // slot size: the largest rank group's tiles
      for (int h = nseg / 2; h >= 1; h /= 2) {
        if (sg >= h && sg < 2 * h) {
          float4* dst = segbuf + ((sg - h) * ng + rg) * own_max * 2 * 4 * 64 + ln;
#pragma unroll
          for (int r = 0; r < OWN; ++r)
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
              for (int v = 0; v < 4; ++v)
                dst[((r * 2 + ch) * 4 + v) * 64] = make_float4(oacc[r][ch][4 * v], oacc[r][ch][4 * v + 1],
                                                               oacc[r][ch][4 * v + 2], oacc[r][ch][4 * v + 3]);
        }
        lds_barrier();
        if (sg < h) {
          const float4* src = segbuf + (sg * ng + rg) * own_max * 2 * 4 * 64 + ln;
#pragma unroll
          for (int r = 0; r < OWN; ++r)
#pragma unroll
            for (int ch = 0; ch < 2; ++ch)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const float4 x = src[((r * 2 + ch) * 4 + v) * 64];
                oacc[r][ch][4 * v] += x.x;
                oacc[r][ch][4 * v + 1] += x.y;
                oacc[r][ch][4 * v + 2] += x.z;
                oacc[r][ch][4 * v + 3] += x.w;
              }
        }
        lds_barrier();
      }
    }
    if (sg == 0) {
      if constexpr (DENSE) {
        // the value pass already produced the output: its accumulators (fp32,
        // [col][dim]) through LDS into the up-projection's lane layout
        float* of = reinterpret_cast<float*>(smem);
        constexpr int ofs = D + 4;
#pragma unroll
        for (int r = 0; r < OWN; ++r)
#pragma unroll
          for (int ch = 0; ch < 2; ++ch)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
              *reinterpret_cast<float4*>(of + (32 * ch + lrow) * ofs + 32 * (rg + ng * r) + 8 * jj + 4 * lhi) =
                  make_float4(oacc[r][ch][4 * jj], oacc[r][ch][4 * jj + 1], oacc[r][ch][4 * jj + 2],
                              oacc[r][ch][4 * jj + 3]);
      } else {
        // the latent accumulator of every rank tile -> LDS as bf16 [col][rank]
        __bf16* olat = reinterpret_cast<__bf16*>(smem);
        const int ols = bm.rv_pad + 8;
#pragma unroll
        for (int r = 0; r < OWN; ++r)
#pragma unroll
          for (int ch = 0; ch < 2; ++ch)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
              bf16x4 v;
#pragma unroll
              for (int u = 0; u < 4; ++u) v[u] = (__bf16)oacc[r][ch][4 * jj + u];
              *reinterpret_cast<bf16x4*>(olat + (32 * ch + lrow) * ols + 32 * (rg + ng * r) + 8 * jj + 4 * lhi) = v;
            }
      }
    }
    lds_barrier();
  };
  if (!I8 && dense) {
    // at rank d every wave owns one rank tile over 8 (d = 128) or 4 (d = 64) steps
    if constexpr (!I8)
      tiles(std::integral_constant<int, 1>{}, std::integral_constant<int, D == 128 ? 8 : 4>{}, std::true_type{});
  } else if (own_v == 0) {
    tiles(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, std::false_type{});
  } else {
    with_own([&](auto own_c, auto cs_c) { tiles(own_c, cs_c, std::false_type{}); });
  }

  // ---- up-projection through R^V and the partial (m, l, o) ----
  const int ln = opaque(lane);
  constexpr int NCB = up_col_blocks<D>();
  constexpr bool kFold = MAX_RT == 2;  // (plans of more rank tiles per wave do not)
  const int cb0 = wave / (narrow ? NDS : NDS / 2) * NCB;  // the first of them
  // this thread's output dims of its columns in the slot
  auto slot_o = [&](int cb, int sl) {
    const int64_t row = query_row(a, c0 + min(16 * (cb0 + cb) + (ln & 15), cn - 1));
    return reinterpret_cast<float4*>(a.part_o + (row * a.n_slots + slot) * D + 16 * (ds0 + sl) + 4 * (ln >> 4));
  };
  // the next item's queries
  if (next_item) {
    const int nc0 = __builtin_amdgcn_readfirstlane(next_item->req), nf = __builtin_amdgcn_readfirstlane(next_item->flags);
    load_queries<D>(a, nc0, ((nf >> kItemColsShift) & 63) + 1, tid, qv);
  } else {
#pragma unroll
    for (int u = 0; u < kQLoads; ++u) forget(qv[u]);
  }
  f32x4 uacc[NCB][2];
  if (dense) {
    const float* of = reinterpret_cast<const float*>(smem);
    constexpr int ofs = D + 4;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int sl = 0; sl < (narrow ? 1 : 2); ++sl) {
        const float4 v = *reinterpret_cast<const float4*>(of + (16 * (cb0 + cb) + (ln & 15)) * ofs +
                                                          16 * (ds0 + sl) + 4 * (ln >> 4));
        uacc[cb][sl] = f32x4{v.x, v.y, v.z, v.w};
      }
  } else {
    // output dims 32 dp .. + 31 of the wave's columns, over all ranks (16x16x32
    // MFMAs: R^V fragment x latent columns from LDS)
    const __bf16* olat = reinterpret_cast<const __bf16*>(smem);
    const int ols = bm.rv_pad + 8;
    // KV head (relative to g0) of this lane's output columns
    int hu[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) hu[cb] = div_by(c0 + min(16 * (cb0 + cb) + (ln & 15), cn - 1), N_g, a.N_g_inv) - g0;
    const __bf16* ob = olat + (16 * cb0 + (ln & 15)) * ols + 8 * (ln >> 4);
    for (int hh = 0; hh < nh; ++hh) {
      f32x4 t[NCB][2];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) t[cb][0] = t[cb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      // the head's runs of the two slices, kRvSteps at a time; a slot is reloaded
      // with the step a round later, or the next head's (NDS nk_v fragments on)
      const unsigned char* rb = rvp + (int64_t)hh * NDS * nk_v * kFragBytes;
      const int round = narrow ? 2 * kRvSteps : kRvSteps;
      for (int k = 0; k < nk_v; k += round) {
        const bool last = k + round >= nk_v;
        const unsigned char* q = rb + (int64_t)(last ? NDS * nk_v : k + round) * kFragBytes;
        const int have = last ? hh + 1 < nh ? nk_v : 0 : nk_v - k - round;  // steps at q
        static_for<0, kRvSteps, 1>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          bf16x8 b[NCB];  // past the ranks: read, not used
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) b[cb] = ld_bf16x8(ob + 16 * cb * ols + 32 * (k + i));
          if (k + i < nk_v) {
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) t[cb][0] = mfma16(rv[i][0], b[cb], t[cb][0]);
            if (!narrow) {
#pragma unroll
              for (int cb = 0; cb < NCB; ++cb) t[cb][1] = mfma16(rv[i][1], b[cb], t[cb][1]);
            }
          }
          rv[i][0] = ldf(q, i * kFragBytes, mask_lt(i, have));
          if (!narrow) rv[i][1] = ldf(q, (nk_v + i) * kFragBytes, mask_lt(i, have));
        });
        if (narrow)
          static_for<0, kRvSteps, 1>([&](auto ic) {
            constexpr int i = decltype(ic)::value + kRvSteps;
            bf16x8 b[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) b[cb] = ld_bf16x8(ob + 16 * cb * ols + 32 * (k + i));
            if (k + i < nk_v) {
#pragma unroll
              for (int cb = 0; cb < NCB; ++cb) t[cb][0] = mfma16(rv[i - kRvSteps][1], b[cb], t[cb][0]);
            }
            rv[i - kRvSteps][1] = ldf(q, i * kFragBytes, mask_lt(i, have));
          });
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        if (hh == 0 || hu[cb] == hh) uacc[cb][0] = t[cb][0], uacc[cb][1] = t[cb][1];
    }
  }  // latent up-projection
  // the item's partial: per-column maximum m_run (score layout), sum (thread
  // tid < kCols: column tid), output uacc (up-projection layout)
  float l_item = 0.f;
  if (tid < kCols) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) l_item += lred[w * kCols + tid];
  }
  {
    // fold into the group's running partial (log-sum-exp)
    const bool first = !kFold || (it.flags & kItemFirst) != 0;
    float fa[2], fb[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      const float mn = first ? m_run[ch] : fmaxf(acc.m[ch], m_run[ch]);
      fa[ch] = first || mn == -INFINITY ? 0.f : fast_exp2(acc.m[ch] - mn);
      fb[ch] = mn == -INFINITY ? 0.f : fast_exp2(m_run[ch] - mn);
      acc.m[ch] = mn;
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int cc = 16 * (cb0 + cb) + (ln & 15);  // column within the tile
      const bool hi = ((cb0 + cb) >> 1) != 0;        // wave-uniform: column half
      const float sa = __shfl(hi ? fa[1] : fa[0], cc & 31);
      const float sb = __shfl(hi ? fb[1] : fb[0], cc & 31);
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) {
        uacc[cb][sl] *= sb;
        if constexpr (kFold) acc.o[cb][sl] = uacc[cb][sl] = first ? uacc[cb][sl] : acc.o[cb][sl] * sa + uacc[cb][sl];
      }
    }
    if (tid < kCols) {
      const int ch = tid >> 5;
      acc.l = first ? l_item * fb[ch] : acc.l * fa[ch] + l_item * fb[ch];
    }
  }
  if (!kFold || (it.flags & kItemFlush)) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
      if (16 * (cb0 + cb) + (ln & 15) < cn) {
#pragma unroll
        for (int sl = 0; sl < (narrow ? 1 : 2); ++sl)
          *slot_o(cb, sl) = make_float4(uacc[cb][sl][0], uacc[cb][sl][1], uacc[cb][sl][2], uacc[cb][sl][3]);
      }
  }
  if ((it.flags & kItemFlush) && tid < cn) {
    const int64_t colg = query_row(a, c0 + tid);
    a.part_ml[colg * a.n_slots + slot] = make_float2(tid < 32 ? acc.m[0] : acc.m[1], acc.l);
  }
  rl.advance();
}

template <int D, int MAX_RT, bool FETCH, int MODE>
__global__ __launch_bounds__(kThreads, 1) void attend_kernel(AttendArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const WgProgram p = a.wg[blockIdx.x];
  if (p.n_items == 0) return;
  {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.prog + p.off);
    uint32_t* dst = reinterpret_cast<uint32_t*>(smem);
    for (int i = threadIdx.x; i < p.words; i += kThreads) dst[i] = src[i];
  }
  lds_barrier();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char* work = smem + a.prog_bytes;
  Streams<MODE == 1, MAX_RT> fs;
  GroupAcc<up_col_blocks<D>()> acc;
  RunDeriver<D> rd;
  rd.items = smem;
  rd.n_items = p.n_items;
  rd.gk = 0;
  rd.gb = 0;
  rd.rbuf = reinterpret_cast<int2*>(smem + (size_t)p.n_items * sizeof(WorkItem));
  rd.recon_delta = a.recon_delta;
  rd.run_cap = a.run_cap;
  if (wave == kWaves - 1) {
    rd.derive(threadIdx.x & 63);
    rd.derive(threadIdx.x & 63);
  }
  lds_barrier();
  RunList rl;
  rl.rbuf = rd.rbuf + (size_t)wave * kRunBufs * a.run_cap;
  rl.run_cap = a.run_cap;
  rl.rb = 0;
  bf16x8 qv[query_loads<D>()];
  // the first block item's queries and first K run load while the tail items,
  // which come before it, run
  if (p.first_block < p.n_items) {
    const WorkItem* it = reinterpret_cast<const WorkItem*>(smem) + p.first_block;
    const int c0 = __builtin_amdgcn_readfirstlane(it->req), fl = __builtin_amdgcn_readfirstlane(it->flags);
    load_queries<D>(a, c0, ((fl >> kItemColsShift) & 63) + 1, threadIdx.x, qv);
    if constexpr (MODE != 1) {  // INT8 items load their first K run themselves
      const int lane16 = 16 * (threadIdx.x & 63);
      const auto run = item_first_run(it, wave, reinterpret_cast<const unsigned char*>(a.data) +
                                                       (int64_t)rl.first(0) * kFragElems * 2);
      static_for<0, Streams<false, 2>::KD, 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        fs.ks[i] = load_frag16(run.p, run.off(i), lane16, run.wanted);
      });
    }
  }
  for (int k = 0; k < p.n_items; ++k) {
    const WorkItem it = lds_item(smem + (size_t)k * sizeof(WorkItem));
    if (k > 0) lds_barrier();  // the previous item's LDS reads are done
    // the thread index is re-derived per item (opaque to the optimiser), so no
    // lane-dependent address of one item kind stays live across the other
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (it.kind == kItemBlock) {
      const WorkItem* next = k + 1 < p.n_items ? reinterpret_cast<const WorkItem*>(smem) + k + 1 : nullptr;
      block_item<D, MAX_RT, FETCH, MODE>(a, it, work, fs, rl, rd, acc, qv, next, tid);
    } else if (it.kind == kItemTail) {
      tail_item<D>(a, it, work, tid);
    }
  }
}

// ---------------------------------------------------------------------------
// Log-sum-exp merge: one workgroup per query column (i, h).  Its partials are
// the block-group slots [0, nb) of its column tile, then request i's tail
// chunks at n_block_slots + chunk.  Thread t takes the
// 4 output dims 4 (t % (D/4)) of the slots s = t / (D/4) (mod slots per pass),
// so every load is one 16-byte vector and a wave reads whole slots; the loads
// of kMergeUnroll passes are issued before any is used, and each thread keeps
// a running (max, sum, output) over its slots.  The slot lanes are then merged
// in a fixed order through LDS, so the result is deterministic.
// ---------------------------------------------------------------------------
constexpr int kMergeThreads = 256;
constexpr int kMergeUnroll = 8;
template <int D>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeArgs a) {
  constexpr int TPS = D / 4;                // threads per slot
  constexpr int SPP = kMergeThreads / TPS;  // slots per pass
  __shared__ float red_m[SPP], red_l[SPP];
  __shared__ float4 red_o[SPP][TPS];
  const int col = blockIdx.x, tid = threadIdx.x;
  const int dq = tid % TPS, sl = tid / TPS;
  const int i = col / a.H_q, h = col % a.H_q;
  const int cf = (h / a.G) * a.tiles.N_g + i * a.G + h % a.G;  // head-major column
  const int nb = a.slot_count[tile_of(a.tiles, cf)];         // block-group slots of its column tile
  const int n_valid = nb + (tail_len_of(a.tl, i) + kTailChunk - 1) / kTailChunk;
  const float2* ml = a.part_ml + (int64_t)col * a.n_slots;
  const float4* po = reinterpret_cast<const float4*>(a.part_o + (int64_t)col * a.n_slots * D) + dq;
  float m = -INFINITY, l = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = sl; s0 < n_valid; s0 += SPP * kMergeUnroll) {
    float2 mm[kMergeUnroll];
    float4 oo[kMergeUnroll];
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      const int v = s0 + u * SPP;
      if (v < n_valid) {
        const int s = v < nb ? v : a.n_block_slots + (v - nb);
        mm[u] = ml[s];
        oo[u] = po[(int64_t)s * TPS];
      } else {
        mm[u] = make_float2(-INFINITY, 0.f);
        oo[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int u = 0; u < kMergeUnroll; ++u) {
      if (mm[u].x == -INFINITY) continue;  // past the last slot
      const float mn = fmaxf(m, mm[u].x);
      const float fo = fast_exp2(m - mn);  // m = -inf before the first slot: 0
      const float fn = fast_exp2(mm[u].x - mn);
      l = l * fo + mm[u].y * fn;
      o.x = o.x * fo + oo[u].x * fn;
      o.y = o.y * fo + oo[u].y * fn;
      o.z = o.z * fo + oo[u].z * fn;
      o.w = o.w * fo + oo[u].w * fn;
      m = mn;
    }
  }
  // every thread of a slot lane holds the same (m, l)
  if (dq == 0) {
    red_m[sl] = m;
    red_l[sl] = l;
  }
  red_o[sl][dq] = o;
  __syncthreads();
  if (tid < TPS) {
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < SPP; ++k) mx = fmaxf(mx, red_m[k]);
    float den = 0.f;
    float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < SPP; ++k) {
      if (red_m[k] == -INFINITY) continue;  // a lane without slots
      const float f = fast_exp2(red_m[k] - mx);
      den += red_l[k] * f;
      const float4 v = red_o[k][tid];
      num.x += v.x * f;
      num.y += v.y * f;
      num.z += v.z * f;
      num.w += v.w * f;
    }
    const float inv = 1.f / den;
    reinterpret_cast<float4*>(a.out + (int64_t)col * D)[tid] =
        make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_pack_batch(const PackArgs* jobs, const int64_t* starts, int n_jobs, int64_t n_frags,
                             hipStream_t s) {
  if (n_jobs == 0 || n_frags == 0) return hipSuccess;
  const int64_t groups = (n_frags + 3) / 4;
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_batch_kernel, dim3((unsigned)groups), dim3(256), 0, s, jobs, starts, n_jobs);
  return hipGetLastError();
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s) {
  if (a.n_frags == 0) return hipSuccess;
  const int64_t threads = a.n_frags * 64;
  const unsigned grid = (unsigned)((threads + 255) / 256);
  hipLaunchKernelGGL(pack_kernel, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_row_scales(const uint16_t* src, int rows, int cols, int rows_pad, float* scale, int* bad,
                             hipStream_t s) {
  if (rows_pad == 0) return hipSuccess;
  hipLaunchKernelGGL(row_scale_kernel, dim3((rows_pad + 255) / 256), dim3(256), 0, s, src, rows, cols, rows_pad,
                     scale, bad);
  return hipGetLastError();
}

hipError_t launch_scale_units(const float* ks, const float* vs, int T_pad, float* dst, hipStream_t s) {
  if (T_pad == 0) return hipSuccess;
  hipLaunchKernelGGL(scale_units_kernel, dim3((2 * T_pad + 255) / 256), dim3(256), 0, s, ks, vs, T_pad, dst);
  return hipGetLastError();
}


template <int D, int MAX_RT, bool FETCH, int MODE>
static hipError_t launch_attend_t(const AttendArgs& a, int grid, size_t lds, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1) {
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_kernel<D, MAX_RT, FETCH, MODE>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipExtLaunchKernelGGL((attend_kernel<D, MAX_RT, FETCH, MODE>), dim3(grid), dim3(kThreads), (uint32_t)lds, s, e0, e1, 0, a);
  return hipGetLastError();
}

template <int D, int MODE>
static hipError_t launch_attend_d(const AttendArgs& a, int max_rt, bool fetch, int grid, size_t lds, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1) {
  switch (max_rt) {
    case 2:
      if constexpr (MODE != 2)
        if (fetch) return launch_attend_t<D, 2, true, MODE>(a, grid, lds, s, e0, e1);
      return launch_attend_t<D, 2, false, MODE>(a, grid, lds, s, e0, e1);
    case 3: return launch_attend_t<D, 3, true, MODE>(a, grid, lds, s, e0, e1);
    case 4: return launch_attend_t<D, 4, true, MODE>(a, grid, lds, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

template <int D>
static hipError_t launch_attend_m(const AttendArgs& a, int max_rt, bool fetch, bool p_int8, bool gemv, int grid, size_t lds,
                                  hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (p_int8) return launch_attend_d<D, 1>(a, max_rt, fetch, grid, lds, s, e0, e1);
  if (gemv) return launch_attend_d<D, 2>(a, max_rt, fetch, grid, lds, s, e0, e1);
  return launch_attend_d<D, 0>(a, max_rt, fetch, grid, lds, s, e0, e1);
}

hipError_t launch_attend(const AttendArgs& a, int head_dim, int max_rt, bool fetch, bool p_int8, bool gemv, int grid,
                         size_t lds_bytes, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (grid == 0) return hipSuccess;
  if (head_dim == 64) return launch_attend_m<64>(a, max_rt, fetch, p_int8, gemv, grid, lds_bytes, s, e0, e1);
  if (head_dim == 128) return launch_attend_m<128>(a, max_rt, fetch, p_int8, gemv, grid, lds_bytes, s, e0, e1);
  return hipErrorInvalidValue;
}

hipError_t launch_merge(const MergeArgs& a, int head_dim, int n_cols, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (head_dim == 64) {
    hipExtLaunchKernelGGL(merge_kernel<64>, dim3(n_cols), dim3(kMergeThreads), 0, s, e0, e1, 0, a);
  } else if (head_dim == 128) {
    hipExtLaunchKernelGGL(merge_kernel<128>, dim3(n_cols), dim3(kMergeThreads), 0, s, e0, e1, 0, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace milo
