// Pooling and upsampling over SC(f, s) connections (Sec. 4.1 "Other
// operators": MP takes the maximum of the zero vector and the active input
// vectors of a receptive field, AP f^-d times their sum; Sec. 5: the FCN
// upsamples by nearest neighbour).  All of them, and their gradients, are
// reductions over the pairs of a rule book direction:
//
//   AP forward      sum over the SC direction, scale f^-d (1 / K)
//   AP backward     sum over the transposed direction, scale f^-d
//   MP forward      max over the SC direction (records the winning offset)
//   MP backward     over the transposed direction: the gradient of an
//                   output element goes to the input at its winning offset
//   upsample        sum over the transposed direction (one pair per row, f = s)
//   its backward    sum over the SC direction
//
// Two output-stationary kernels cover all of them (k_pool_walk for what has
// many offsets and few pairs).  The main one, k_pool: a workgroup owns 64
// output rows (one tile of the direction's storage) and a run of channels.
// It first writes the tile's pairs into an LDS table (input row by offset and
// output row, -1 for none; within one offset every output row has at most one
// pair), and then every thread takes 16 bytes of an output row and walks the
// offsets in order, with the reads of four of them in flight and the result
// in registers.  Each output element is written once: no atomics,
// deterministic.
// Memory-bound: every pair reads one input row piece, every output row is
// written once.  Measured at 99,515 sites -> 30,041, 64 fp32 channels, MP and
// AP forward and backward, upsampling and its gradient, six calls together:
// 81 us.  (The tile's rows in LDS, all offsets in turn with a barrier after
// each and 4 bytes a lane, were bound by that walk's latency: 231 us.)
#include "internal.h"
#include "numeric.h"
#include "routes.h"

namespace sscn {

namespace {

enum PoolMode { kSum = 0, kMax = 1, kMaxBack = 2 };
constexpr int kPoolCols = 64;
constexpr uint8_t kNoArg = 255;  // the zero vector is the maximum

// V consecutive values of a row, or of its winning offsets.
template <typename T, int V> struct Piece {
  static __device__ __forceinline__ void load(const T* p, float (&v)[V]) {
    if constexpr (V == 1) {
      v[0] = ld(p);
    } else {
      const uint4 q = *reinterpret_cast<const uint4*>(p);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (V == 4) {
          v[i] = __uint_as_float(w[i]);
        } else {
          v[2 * i] = __uint_as_float(w[i] << 16);
          v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
      }
    }
  }
  static __device__ __forceinline__ void store(T* p, const float (&v)[V]) {
    if constexpr (V == 1) {
      st(p, v[0]);
    } else {
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (V == 4) w[i] = __float_as_uint(v[i]);
        else w[i] = (uint32_t)f32_bf16_bits(v[2 * i]) | ((uint32_t)f32_bf16_bits(v[2 * i + 1]) << 16);
      }
      *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
};
template <int V>
__device__ __forceinline__ void load_arg(const uint8_t* p, uint8_t (&a)[V]) {
  if constexpr (V == 1) {
    a[0] = *p;
  } else {
#pragma unroll
    for (int i = 0; i < V / 4; ++i) {
      const uint32_t w = reinterpret_cast<const uint32_t*>(p)[i];
#pragma unroll
      for (int b = 0; b < 4; ++b) a[4 * i + b] = (uint8_t)(w >> (8 * b));
    }
  }
}
template <int V>
__device__ __forceinline__ void store_arg(uint8_t* p, const uint8_t (&a)[V]) {
  if constexpr (V == 1) {
    *p = a[0];
  } else {
#pragma unroll
    for (int i = 0; i < V / 4; ++i)
      reinterpret_cast<uint32_t*>(p)[i] = (uint32_t)a[4 * i] | ((uint32_t)a[4 * i + 1] << 8) |
                                          ((uint32_t)a[4 * i + 2] << 16) | ((uint32_t)a[4 * i + 3] << 24);
  }
}

// X: rows of the direction's input side (n_in x c); arg_in (kMaxBack): the
// forward's winning offsets, indexed like X.  Y: n_out x c; arg_out (kMax):
// n_out x c winning offsets.  V channels per thread (16 bytes, or 1 where
// rows are not whole aligned pieces); a workgroup takes 2^pb pieces of every
// row of its tile.  LDS: K x 64 words.
template <typename T, int MODE, int V>
__global__ __launch_bounds__(256) void k_pool(const T* __restrict__ X, const uint8_t* __restrict__ arg_in,
                                              const int64_t* __restrict__ seg, int64_t n_tiles,
                                              const int32_t* __restrict__ in_rows, const int32_t* __restrict__ out_rows,
                                              int K, int mirror, int64_t n_out, int c, int pb, float scale,
                                              T* __restrict__ Y, uint8_t* __restrict__ arg_out) {
  extern __shared__ int32_t src[];  // [o][row of the tile]
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t row0 = t * kPlanRows;
  // A tile holds at most 64 pairs of an offset, in increasing output row: one
  // lane per pair.  The table's rows belong to one wavefront each, whose LDS
  // accesses keep their order, so no barrier is needed between the two stores.
  constexpr int U = 4;  // offsets in flight per wavefront
  for (int o0 = wave; o0 < K; o0 += 4 * U) {
    int64_t p0[U];
    int n[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int o = min(o0 + 4 * u, K - 1), so = mirror ? K - 1 - o : o;
      p0[u] = seg[(int64_t)so * n_tiles + t];
      n[u] = (int)(seg[(int64_t)so * n_tiles + t + 1] - p0[u]);
    }
    int32_t j[U], r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = o0 + 4 * u < K && lane < n[u];
      j[u] = ok ? in_rows[p0[u] + lane] : -1;
      r[u] = ok ? (int32_t)(out_rows[p0[u] + lane] - row0) : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (o0 + 4 * u >= K) break;
      int32_t* dst = src + (o0 + 4 * u) * kPlanRows;
      dst[lane] = -1;
      __builtin_amdgcn_wave_barrier();
      if (j[u] >= 0) dst[r[u]] = j[u];
    }
  }
  __syncthreads();
  const int piece = (int)blockIdx.y * (1 << pb) + (tid & ((1 << pb) - 1));
  const int col = piece * V;
  if (col >= c) return;
  for (int r = tid >> pb; r < kPlanRows; r += 256 >> pb) {
    const int64_t row = row0 + r;
    if (row >= n_out) break;
    float acc[V];
    uint8_t arg[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      acc[i] = 0.f;
      arg[i] = kNoArg;
    }
    for (int o = 0; o < K; o += 4) {
      int32_t j[4];
      float v[4][V];
      uint8_t a[4][V];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        j[u] = o + u < K ? src[(o + u) * kPlanRows + r] : -1;
        if (j[u] >= 0) {
          Piece<T, V>::load(X + (int64_t)j[u] * c + col, v[u]);
          if constexpr (MODE == kMaxBack) load_arg<V>(arg_in + (int64_t)j[u] * c + col, a[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j[u] < 0) continue;
#pragma unroll
        for (int i = 0; i < V; ++i) {
          if constexpr (MODE == kSum) {
            acc[i] += v[u][i];
          } else if constexpr (MODE == kMax) {
            if (v[u][i] > acc[i]) {
              acc[i] = v[u][i];
              arg[i] = (uint8_t)(o + u);
            }
          } else {
            if (a[u][i] == (uint8_t)(o + u)) acc[i] += v[u][i];
          }
        }
      }
    }
    if constexpr (MODE == kSum) {
#pragma unroll
      for (int i = 0; i < V; ++i) acc[i] *= scale;
    }
    Piece<T, V>::store(Y + row * c + col, acc);
    if constexpr (MODE == kMax) store_arg<V>(arg_out + row * c + col, arg);
  }
}

// The same results, bit for bit, by a walk over the pairs: the tile's rows and
// 64 channels of them in LDS, the offsets in order, the four wavefronts taking
// an offset's pairs in turn (a row has one at most), a barrier after each
// offset.  For many offsets with a pair at few of them, and for long rows of
// single channels: its time goes with the offsets of a tile and the pairs, not
// with the offsets of every row (pool_takes_table).
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_pool_walk(const T* __restrict__ X, const uint8_t* __restrict__ arg_in,
                                                   const int64_t* __restrict__ seg, int64_t n_tiles,
                                                   const int32_t* __restrict__ in_rows,
                                                   const int32_t* __restrict__ out_rows, int K, int mirror,
                                                   int64_t n_out, int c, float scale, T* __restrict__ Y,
                                                   uint8_t* __restrict__ arg_out) {
  __shared__ float acc[kPlanRows][kPoolCols];
  __shared__ uint8_t arg[kPlanRows][kPoolCols];
  const int64_t t = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.y * kPoolCols + lane;
  const bool live = col < c;
  const int64_t row0 = t * kPlanRows;
  for (int r = wave; r < kPlanRows; r += 4) {
    acc[r][lane] = 0.f;
    arg[r][lane] = kNoArg;
  }
  __syncthreads();
  for (int o = 0; o < K; ++o) {
    const int so = mirror ? K - 1 - o : o;
    const int64_t p0 = seg[(int64_t)so * n_tiles + t], p1 = seg[(int64_t)so * n_tiles + t + 1];
    for (int64_t p = p0 + wave; p < p1; p += 4) {
      const int64_t j = in_rows[p];
      const int r = (int)(out_rows[p] - row0);
      if (!live) continue;
      const float v = ld(X + j * c + col);
      if constexpr (MODE == kSum) {
        acc[r][lane] += v;
      } else if constexpr (MODE == kMax) {
        if (v > acc[r][lane]) {
          acc[r][lane] = v;
          arg[r][lane] = (uint8_t)o;
        }
      } else {
        if (arg_in[j * c + col] == (uint8_t)o) acc[r][lane] += v;
      }
    }
    __syncthreads();
  }
  if (!live) return;
  for (int r = wave; r < kPlanRows; r += 4) {
    const int64_t row = row0 + r;
    if (row >= n_out) break;
    st(Y + row * c + col, MODE == kSum ? acc[r][lane] * scale : acc[r][lane]);
    if constexpr (MODE == kMax) arg_out[row * c + col] = arg[r][lane];
  }
}

template <typename T, int MODE>
sscn_status launch_pool(const View& v, const void* X, const uint8_t* arg_in, int c, float scale, void* Y,
                        uint8_t* arg_out, hipStream_t s) {
  const int64_t tiles = v.st->n_tiles;
  if (tiles == 0) return SSCN_OK;
  if (tiles > 0x7fffffff) return fail(SSCN_ERR_INVALID_ARG, "too many output rows");
  // 16-byte pieces where rows are whole ones on both sides (and the winning
  // offsets' words aligned), else a channel per thread
  constexpr int V = 16 / (int)sizeof(T);
  const auto addr = [](const void* p) { return reinterpret_cast<uintptr_t>(p); };
  const bool vec = c % V == 0 && addr(X) % 16 == 0 && addr(Y) % 16 == 0 && addr(arg_in) % 4 == 0 && addr(arg_out) % 4 == 0;
  const int pieces = vec ? c / V : c;
  // pieces per workgroup: 128 bytes of every row (64 channels one by one);
  // fewer where the rows are shorter
  int pb = vec ? 3 : 6;
  while (pb > 0 && (1 << (pb - 1)) >= pieces) --pb;
  if (!pool_takes_table(v.K, v.n_pairs, v.n_out, tiles, pieces, pb)) {
    const dim3 grid((unsigned)tiles, (unsigned)ceil_div(c, kPoolCols));
    k_pool_walk<T, MODE><<<grid, 256, 0, s>>>((const T*)X, arg_in, v.st->seg, tiles, v.st->in_rows, v.st->out_rows,
                                              v.K, v.mirror ? 1 : 0, v.n_out, c, scale, (T*)Y, arg_out);
    SSCN_HIP(hipGetLastError());
    return SSCN_OK;
  }
  const dim3 grid((unsigned)tiles, (unsigned)ceil_div(pieces, 1 << pb));
  const size_t lds = sizeof(int32_t) * kPlanRows * (size_t)v.K;
  auto kern = vec ? k_pool<T, MODE, V> : k_pool<T, MODE, 1>;
  kern<<<grid, 256, lds, s>>>((const T*)X, arg_in, v.st->seg, tiles, v.st->in_rows, v.st->out_rows, v.K,
                              v.mirror ? 1 : 0, v.n_out, c, pb, scale, (T*)Y, arg_out);
  SSCN_HIP(hipGetLastError());
  return SSCN_OK;
}

template <int MODE>
sscn_status launch_pool_t(sscn_dtype dtype, const View& v, const void* X, const uint8_t* arg_in, int c, float scale,
                          void* Y, uint8_t* arg_out, hipStream_t s) {
  if (dtype == SSCN_F32) return launch_pool<float, MODE>(v, X, arg_in, c, scale, Y, arg_out, s);
  return launch_pool<uint16_t, MODE>(v, X, arg_in, c, scale, Y, arg_out, s);
}

sscn_status check_pool(sscn_rulebook rb, int32_t c, sscn_dtype dtype) {
  if (!rb) return fail(SSCN_ERR_INVALID_ARG, "NULL rule book");
  if (c < 1 || c > 65536) return fail(SSCN_ERR_INVALID_ARG, "channel count must be in [1, 65536]");
  if (dtype != SSCN_F32 && dtype != SSCN_BF16) return fail(SSCN_ERR_INVALID_ARG, "unknown dtype");
  if (rb->d->submanifold) return fail(SSCN_ERR_INVALID_ARG, "pooling and upsampling take an SC(f, s) rule book");
  if (rb->transposed) return fail(SSCN_ERR_INVALID_ARG, "pass the SC rule book itself, not its transpose");
  return SSCN_OK;
}

View direction(sscn_rulebook rb, bool transposed) {
  sscn_rulebook_s t{rb->d, transposed};
  return view_of(&t);
}

}  // namespace
}  // namespace sscn

using namespace sscn;

extern "C" sscn_status sscn_pool_forward(const void* features, sscn_rulebook rb, int32_t c, sscn_dtype dtype,
                                         sscn_pool_mode mode, void* out, uint8_t* argmax, hipStream_t stream) {
  SSCN_TRY(check_pool(rb, c, dtype));
  if (mode != SSCN_POOL_MAX && mode != SSCN_POOL_AVG) return fail(SSCN_ERR_INVALID_ARG, "unknown pooling mode");
  const RulebookData* d = rb->d;
  if (mode == SSCN_POOL_MAX && d->K >= kNoArg) return fail(SSCN_ERR_INVALID_ARG, "max pooling takes at most 254 offsets");
  if (d->n_out == 0) return SSCN_OK;
  if (!out || (d->n_in > 0 && !features) || (mode == SSCN_POOL_MAX && !argmax))
    return fail(SSCN_ERR_INVALID_ARG, "NULL features, out or argmax");
  UseNote note{rb->d, stream};
  const View v = direction(rb, false);
  if (mode == SSCN_POOL_AVG)
    return launch_pool_t<kSum>(dtype, v, features, nullptr, c, 1.0f / (float)d->K, out, nullptr, stream);
  return launch_pool_t<kMax>(dtype, v, features, nullptr, c, 1.0f, out, argmax, stream);
}

extern "C" sscn_status sscn_pool_backward(const void* dout, const uint8_t* argmax, sscn_rulebook rb, int32_t c,
                                          sscn_dtype dtype, sscn_pool_mode mode, void* dgrad, hipStream_t stream) {
  SSCN_TRY(check_pool(rb, c, dtype));
  if (mode != SSCN_POOL_MAX && mode != SSCN_POOL_AVG) return fail(SSCN_ERR_INVALID_ARG, "unknown pooling mode");
  const RulebookData* d = rb->d;
  if (mode == SSCN_POOL_MAX && d->K >= kNoArg) return fail(SSCN_ERR_INVALID_ARG, "max pooling takes at most 254 offsets");
  if (d->n_in == 0) return SSCN_OK;
  if (!dgrad || (d->n_out > 0 && !dout) || (mode == SSCN_POOL_MAX && d->n_out > 0 && !argmax))
    return fail(SSCN_ERR_INVALID_ARG, "NULL dout, dgrad or argmax");
  UseNote note{rb->d, stream};
  const View v = direction(rb, true);
  if (mode == SSCN_POOL_AVG)
    return launch_pool_t<kSum>(dtype, v, dout, nullptr, c, 1.0f / (float)d->K, dgrad, nullptr, stream);
  return launch_pool_t<kMaxBack>(dtype, v, dout, argmax, c, 1.0f, dgrad, nullptr, stream);
}

extern "C" sscn_status sscn_upsample_forward(const void* features, sscn_rulebook rb, int32_t c, sscn_dtype dtype,
                                             void* out, hipStream_t stream) {
  SSCN_TRY(check_pool(rb, c, dtype));
  const RulebookData* d = rb->d;
  if (d->f != d->stride) return fail(SSCN_ERR_INVALID_ARG, "nearest-neighbour upsampling inverts an SC(s, s) rule book");
  if (d->n_in == 0) return SSCN_OK;
  if (!out || (d->n_out > 0 && !features)) return fail(SSCN_ERR_INVALID_ARG, "NULL features or out");
  UseNote note{rb->d, stream};
  return launch_pool_t<kSum>(dtype, direction(rb, true), features, nullptr, c, 1.0f, out, nullptr, stream);
}

extern "C" sscn_status sscn_upsample_backward(const void* dout, sscn_rulebook rb, int32_t c, sscn_dtype dtype,
                                              void* dgrad, hipStream_t stream) {
  SSCN_TRY(check_pool(rb, c, dtype));
  const RulebookData* d = rb->d;
  if (d->f != d->stride) return fail(SSCN_ERR_INVALID_ARG, "nearest-neighbour upsampling inverts an SC(s, s) rule book");
  if (d->n_out == 0) return SSCN_OK;
  if (!dgrad || (d->n_in > 0 && !dout)) return fail(SSCN_ERR_INVALID_ARG, "NULL dout or dgrad");
  UseNote note{rb->d, stream};
  return launch_pool_t<kSum>(dtype, direction(rb, false), dout, nullptr, c, 1.0f, dgrad, nullptr, stream);
}
