// KV append into the paged cache (+ 3D RoPE on keys) and the RoPE table.
//
// One page slot holds one latent frame of one state: K[head][token][d] then
// V[head][d][token].  Keys are rotated at their absolute positions (time =
// chunk * pages_per_chunk + frame, height = n / grid_w, width = n % grid_w)
// with interleaved channel pairs split over the three axes.
#include "device.h"
#include "internal.h"

namespace sc {

// cos/sin of pos * theta^(-2 i / dim_a) for every (position, pair) of the
// three axes, computed in double and stored as fp32 (cos, sin).
__global__ void rope_table_kernel(float2* table, int32_t pt, int32_t ph, int32_t pw, int64_t off_h,
                                  int64_t off_w, int64_t total, float theta) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  int32_t pos, i, dim;
  if (e < off_h) {
    pos = (int32_t)(e / pt); i = (int32_t)(e % pt); dim = 2 * pt;
  } else if (e < off_w) {
    pos = (int32_t)((e - off_h) / ph); i = (int32_t)((e - off_h) % ph); dim = 2 * ph;
  } else {
    pos = (int32_t)((e - off_w) / pw); i = (int32_t)((e - off_w) % pw); dim = 2 * pw;
  }
  const double freq = pow((double)theta, -2.0 * (double)i / (double)dim);
  const double ang = (double)pos * freq;
  table[e] = make_float2((float)cos(ang), (float)sin(ang));
}

int launch_rope_table(const sc_rope_desc* d, void* table, hipStream_t stream) {
  RopeLayout L = rope_layout(d);
  if (L.total == 0) return SC_OK;
  const int threads = 256;
  const int64_t blocks = (L.total + threads - 1) / threads;
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)blocks), dim3(threads), 0, stream,
                     static_cast<float2*>(table), L.pairs_t, L.pairs_h, L.pairs_w, L.off_h, L.off_w,
                     L.total, d->theta);
  SC_HIP(hipGetLastError());
  return SC_OK;
}

struct RopeArgs {
  const float2* table;
  int32_t grid_w, pairs_t, pairs_h, pairs_w;
  int64_t off_h, off_w;
  int32_t frame0;  // absolute latent frame of the state's first page
  DivMagic gw_div;
};

struct SlotList {
  int32_t slot[32];
};

// 16 bytes of a tensor that is only aligned to its element type (the hardware
// takes unaligned 16-byte accesses), and its values as fp32.
template <typename T> struct Vec;
template <> struct Vec<uint16_t> {
  static constexpr int N = 8;
  typedef uint32_t V __attribute__((ext_vector_type(4), aligned(2)));
  static __device__ __forceinline__ void ld(const V& v, float (&f)[N]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      f[2 * k] = __uint_as_float(v[k] << 16);
      f[2 * k + 1] = __uint_as_float(v[k] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ V st(const float (&f)[N]) {
    V v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = pack_bf16x2(f[2 * k], f[2 * k + 1]);
    return v;
  }
  static __device__ __forceinline__ uint16_t elt(const V& v, int e) { return (uint16_t)(v[e >> 1] >> (16 * (e & 1))); }
};
template <> struct Vec<float> {
  static constexpr int N = 4;
  typedef float V __attribute__((ext_vector_type(4), aligned(4)));
  static __device__ __forceinline__ void ld(const V& v, float (&f)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) f[k] = v[k];
  }
  static __device__ __forceinline__ V st(const float (&f)[N]) { return V{f[0], f[1], f[2], f[3]}; }
  static __device__ __forceinline__ float elt(const V& v, int e) { return v[e]; }
};

// A work-group: 64 tokens of one page and head.  Grid: x = page (frame) x token
// blocks, y = head.  Tokens of the source: [frame * tpp + t][head][d].
// A thread takes one 16-byte run of channels of every (256 / runs per row)th
// token: all its loads (keys, values, rotations) go out before the first is
// used.  Keys are rotated and stored as they are; values cross LDS, where the
// 16-byte token segments of channel row d are XORed with the row's run index, and
// leave as 16-byte runs of one channel's tokens (pages hold a multiple of 8 tokens,
// so a run stays in one).  The reads meet no bank conflict; of the 2-byte writes,
// runs r and r + 8 share banks and token pairs a word (conflicts in 44 % of the LDS
// cycles by the counters, hidden behind memory).
// Bound by memory: a Wan chunk (57.5 MB read and written) 11.2 us, 5.1 TB/s,
// against 27.4 for 2-byte accesses; a small page by its chain of latencies.
template <typename T, int HD, bool ROPE>
__global__ __launch_bounds__(256) void append_kernel(const T* __restrict__ k, const T* __restrict__ v,
                                                     char* __restrict__ layer_base, size_t slot_bytes,
                                                     size_t kv_half, SlotList slots, int32_t n_heads,
                                                     int32_t tpp, RopeArgs rope) {
  using V = typename Vec<T>::V;
  constexpr int TB = 64, N = Vec<T>::N, RUNS = HD / N, SEGS = TB / N;
  constexpr int STEP = 256 / RUNS, IT = TB / STEP;  // tokens per pass, passes
  __shared__ __attribute__((aligned(16))) T vt[HD][TB];
  const int32_t blocks_per_page = (tpp + TB - 1) / TB;
  const int32_t page = blockIdx.x / blocks_per_page;
  const int32_t t0 = (blockIdx.x % blocks_per_page) * TB;
  const int32_t h = blockIdx.y;
  const int32_t ntok = min(TB, tpp - t0);
  char* slot_base = layer_base + (size_t)slots.slot[page] * slot_bytes;
  T* kdst = reinterpret_cast<T*>(slot_base) + ((size_t)h * tpp + t0) * HD;
  T* vdst = reinterpret_cast<T*>(slot_base + kv_half) + (size_t)h * HD * tpp + t0;
  const size_t row_stride = (size_t)n_heads * HD;
  const int32_t run = threadIdx.x % RUNS, tok0 = threadIdx.x / RUNS;
  const size_t src0 = ((size_t)page * tpp + t0) * row_stride + (size_t)h * HD + N * run;
  V kv[IT], vv[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const size_t src = src0 + (size_t)min(tok0 + STEP * i, ntok - 1) * row_stride;  // past the end: the last token
    kv[i] = *reinterpret_cast<const V*>(k + src);
    vv[i] = *reinterpret_cast<const V*>(v + src);
  }
  // the rotations of this thread's channel pairs: the axis and its table are
  // fixed, the position changes with the token
  float2 cs[ROPE ? IT : 1][N / 2];
  if constexpr (ROPE) {
    int32_t ax[N / 2];
    int64_t base[N / 2];
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
      int32_t p = N / 2 * run + j;
      ax[j] = p < rope.pairs_t ? 0 : p < rope.pairs_t + rope.pairs_h ? 1 : 2;
      base[j] = ax[j] == 0 ? (int64_t)(rope.frame0 + page) * rope.pairs_t + p
                : ax[j] == 1 ? rope.off_h + p - rope.pairs_t : rope.off_w + p - rope.pairs_t - rope.pairs_h;
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int32_t tok = t0 + min(tok0 + STEP * i, ntok - 1);
      const int32_t hh = (int32_t)fast_div((uint32_t)tok, rope.gw_div), ww = tok - hh * rope.grid_w;
#pragma unroll
      for (int j = 0; j < N / 2; ++j)
        cs[i][j] = rope.table[base[j] + (ax[j] == 0 ? 0 : ax[j] == 1 ? hh * rope.pairs_h : ww * rope.pairs_w)];
    }
  }
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int32_t tok = tok0 + STEP * i;
    if (tok >= ntok) continue;
    if constexpr (ROPE) {
      float f[N];
      Vec<T>::ld(kv[i], f);
#pragma unroll
      for (int j = 0; j < N / 2; ++j) {
        const float x0 = f[2 * j], x1 = f[2 * j + 1];
        // written out, so that a key's bits do not hang on how the compiler contracts these
        f[2 * j] = fmaf(x0, cs[i][j].x, -(x1 * cs[i][j].y));
        f[2 * j + 1] = fmaf(x0, cs[i][j].y, x1 * cs[i][j].x);
      }
      kv[i] = Vec<T>::st(f);
    }
    *reinterpret_cast<V*>(kdst + (size_t)tok * HD + N * run) = kv[i];
    const int32_t col = ((tok / N) ^ (run & (SEGS - 1))) * N + tok % N;
#pragma unroll
    for (int e = 0; e < N; ++e) vt[N * run + e][col] = Vec<T>::elt(vv[i], e);
  }
  __syncthreads();
  // values transposed: V[head][d][token]
#pragma unroll
  for (int i = 0; i < HD * SEGS / 256; ++i) {
    const int32_t e = threadIdx.x + 256 * i, d = e / SEGS, seg = e % SEGS;
    if (seg * N >= ntok) continue;
    const V r = *reinterpret_cast<const V*>(&vt[d][(seg ^ ((d / N) & (SEGS - 1))) * N]);
    *reinterpret_cast<V*>(vdst + (size_t)d * tpp + seg * N) = r;
  }
}

template <typename T, int HD>
static void launch_append_t(dim3 grid, const sc_cache* c, char* layer_base, const SlotList& sl, const void* k,
                            const void* v, bool use_rope, const RopeArgs& ra, hipStream_t stream) {
  const T *kt = static_cast<const T*>(k), *vt = static_cast<const T*>(v);
  if (use_rope)
    hipLaunchKernelGGL((append_kernel<T, HD, true>), grid, dim3(256), 0, stream, kt, vt, layer_base, c->slot_bytes,
                       c->kv_half, sl, c->d.n_heads, c->d.tokens_per_page, ra);
  else
    hipLaunchKernelGGL((append_kernel<T, HD, false>), grid, dim3(256), 0, stream, kt, vt, layer_base, c->slot_bytes,
                       c->kv_half, sl, c->d.n_heads, c->d.tokens_per_page, ra);
}

int launch_append(const sc_cache* c, int32_t layer, const int32_t* slots, int32_t chunk,
                  const void* k, const void* v, const sc_rope* rope, hipStream_t stream) {
  const sc_cache_desc& d = c->d;
  if (d.pages_per_chunk > 32) return fail(SC_EUNSUPPORTED, "pages_per_chunk > 32");
  SlotList sl;
  for (int i = 0; i < d.pages_per_chunk; ++i) sl.slot[i] = slots[i];
  RopeArgs ra{};
  if (rope) {
    RopeLayout L = rope_layout(&rope->desc);
    ra.table = static_cast<const float2*>(rope->dev_table);
    ra.grid_w = rope->desc.grid_w;
    ra.pairs_t = L.pairs_t;
    ra.pairs_h = L.pairs_h;
    ra.pairs_w = L.pairs_w;
    ra.off_h = L.off_h;
    ra.off_w = L.off_w;
    ra.frame0 = chunk * d.pages_per_chunk;
    ra.gw_div = magic_div((uint32_t)rope->desc.grid_w);
  }
  char* layer_base = c->pool + (size_t)layer * d.n_slots * c->slot_bytes;
  dim3 grid(d.pages_per_chunk * ((d.tokens_per_page + 63) / 64), d.n_heads);
  timer_begin(TK_APPEND, stream);
  if (d.dtype == SC_DTYPE_BF16) {
    if (d.head_dim == 128)
      launch_append_t<uint16_t, 128>(grid, c, layer_base, sl, k, v, rope, ra, stream);
    else
      launch_append_t<uint16_t, 64>(grid, c, layer_base, sl, k, v, rope, ra, stream);
  } else {
    if (d.head_dim == 128)
      launch_append_t<float, 128>(grid, c, layer_base, sl, k, v, rope, ra, stream);
    else
      launch_append_t<float, 64>(grid, c, layer_base, sl, k, v, rope, ra, stream);
  }
  timer_end(TK_APPEND, stream);
  SC_HIP(hipGetLastError());
  return SC_OK;
}

}  // namespace sc
