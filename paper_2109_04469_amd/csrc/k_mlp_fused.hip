// The warm-start network in two launches per training step and one per
// prediction, for networks whose rows fit the LDS.
//
// A network of a few hundred features on a batch of up to a few hundred rows
// is nothing but latency: one product per layer and launch spent 15 to 20 us
// on each of 22 launches of a training step (4 layers of 256, 512 outputs, 96
// rows: 440 us per step) for 0.1 GFLOP. So a workgroup here takes 2 to 32 rows
// through all layers, forward and back, with the rows' activations as BF16 in
// LDS, and what crosses rows (weight gradients, biases, loss) and the optimiser
// follow in one second launch: 29.5 + 8.6 us, and 14 us for a prediction of 16
// rows. What bounds the first is a compute unit's own pace: a hidden layer of
// 256 takes 2.3 us, of which its 128 KB of weights at 64 bytes per clock are
// 0.9 and the chain product, GELU, LDS, barrier (1.1 us at width 64) the rest.
//
// Arithmetic as in the layer-by-layer kernels, to the last bit: operands
// rounded to BF16, v_mfma_f32_32x32x16_bf16 in ascending k from a zero
// accumulator, the same epilogues in FP32, bias gradients summed over the rows
// in order, the loss in the same tree.
//
// Weights and the operands of the weight gradients are kept packed in fragment
// order: the 16 bytes each lane feeds to a product are consecutive over the
// lanes, so a fragment is one 1 KB read straight to registers and no LDS round
// trip or barrier is spent on it. A wave asks for the first eight fragments of
// its next tile (of the next layer, too: weights depend on nothing) before the
// epilogue of the current one, which hides most of the L2 latency (sixteen
// ahead: 32.6 us, the registers cost more than they hide).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlp_dev.h"
#include "mlp_internal.h"

namespace pic {

namespace {

constexpr int kRowThreads = 512;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kCus = 256;
constexpr int kAhead = 8;  // fragments in flight per wave
constexpr int kUpdateThreads = 256;  // 128: 11.7 us per launch, 256: 8.6, 512: 10.1
constexpr int kUpdateWaves = kUpdateThreads / 64;

// position of (feature f, k) in a packed matrix of `ks` k-steps
__device__ __forceinline__ int64_t frag_at(int f, int k, int ks) {
  return (((int64_t)(f >> 5) * ks + (k >> 4)) * 64 + ((k >> 3) & 1) * 32 + (f & 31)) * 8 + (k & 7);
}

__device__ __forceinline__ void fetch(short8 (&b)[kAhead], const uint16_t* __restrict__ tile,
                                      int k0, int ks, int lane) {
#pragma unroll
  for (int q = 0; q < kAhead; ++q)
    if (k0 + q < ks)
      b[q] = *reinterpret_cast<const short8*>(tile + ((int64_t)(k0 + q) * 64 + lane) * 8);
}

__device__ __forceinline__ f32x16 mfma(short8 a, short8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 32 rows of LDS (`row`: this lane's, at its eight k) times a packed tile of
// 32 features whose first fragments are in b.
__device__ __forceinline__ f32x16 product(short8 (&b)[kAhead], const uint16_t* __restrict__ tile,
                                          int ks, const uint16_t* row, int lane) {
  f32x16 acc = {};
  for (int k0 = 0; k0 < ks; k0 += kAhead) {
    short8 nb[kAhead];
    fetch(nb, tile, k0 + kAhead, ks, lane);
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
      if (k0 + q < ks)
        acc = mfma(*reinterpret_cast<const short8*>(row + (k0 + q) * 16), b[q], acc);
#pragma unroll
    for (int q = 0; q < kAhead; ++q) b[q] = nb[q];
  }
  return acc;
}

// start of the next tile of this wave: `nt` of a layer's `tiles`, else its
// first tile in the layer after it
__device__ __forceinline__ void fetch_next(short8 (&b)[kAhead], const uint16_t* here, int nt,
                                           int tiles, int ks, const uint16_t* next, int next_tiles,
                                           int next_ks, int wave, int lane) {
  if (nt < tiles)
    fetch(b, here + (int64_t)nt * ks * 512, 0, ks, lane);
  else if (wave < next_tiles)
    fetch(b, next + (int64_t)wave * next_ks * 512, 0, next_ks, lane);
}

// Q consecutive k from k0 (a multiple of Q) of feature f
template <int Q>
__device__ __forceinline__ void store_run(uint16_t* base, int f, int k0, int ks,
                                          const uint16_t (&q)[Q]) {
  uint16_t* p = base + frag_at(f, k0, ks);
  if (Q == 4)
    *reinterpret_cast<uint2*>(p) = make_uint2((uint32_t)q[0] | ((uint32_t)q[1 % Q] << 16),
                                              (uint32_t)q[2 % Q] | ((uint32_t)q[3 % Q] << 16));
  else if (Q == 2)
    *reinterpret_cast<uint32_t*>(p) = (uint32_t)q[0] | ((uint32_t)q[1 % Q] << 16);
  else
    *p = q[0];
}

// Accumulator order: lane j + 32 ((i / 4) % 2) and register (i % 4) + 4 (i / 8)
// hold row i, column j of the 32 x 32 product. A workgroup fills 2 E of the 32
// rows, E per lane: rows 8 j + 4 h + q with q < Q = min(E, 4), j < E / Q, which
// hold the batch's rows 2 Q j + Q h + q of the workgroup's.
template <bool TRAIN, int E>
__global__ __launch_bounds__(kRowThreads) void k_mlp_rows(MlpArgs a, int ld) {
  constexpr int Q = E < 4 ? E : 4, J = E / Q, R = 2 * E;
  extern __shared__ __align__(16) uint16_t sRows[];  // two buffers of 32 rows of ld
  const int lane = threadIdx.x & 63;
  const int wave = !TRAIN && E == 16 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int waves = TRAIN || E < 16 ? kRowWaves : blockDim.x >> 6;
  const int col = lane & 31, h = lane >> 5;
  const int rb = blockIdx.x, row0 = rb * R;
  const int L = a.d.depth;
  const int ksb = a.rows >> 4;  // k-steps of the operands over rows
  const int pin = pad32(a.d.n_in), pw = pad32(a.d.width), po = pad32(a.d.n_out);
  uint16_t* sIn = sRows;
  uint16_t* sOut = sRows + 32 * ld;

  short8 b[kAhead];
  fetch_next(b, a.wf, 0, 0, 0, a.wf, (L == 0 ? po : pw) >> 5, pin >> 4, wave, lane);

  if constexpr (!TRAIN && E == 16) {
    // many rows: 64 inputs of a row to a wave at a time, eight of those on
    // their way (a division per element takes longer than these loads)
    const int per_row = (pin + 63) >> 6, chunks = R * per_row;
    for (int c0 = wave; c0 < chunks; c0 += 8 * waves) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int c = c0 + q * waves, r = c / per_row, k = (c - r * per_row) * 64 + lane;
        v[q] = (c < chunks && row0 + r < a.batch && k < a.d.n_in)
                   ? a.x[(int64_t)(row0 + r) * a.d.n_in + k] : 0.0f;
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int c = c0 + q * waves, r = c / per_row, k = (c - r * per_row) * 64 + lane;
        if (c < chunks && k < pin)
          sIn[(8 * (r / (2 * Q)) + 4 * ((r / Q) & 1) + r % Q) * ld + k] = to_bf16(v[q]);
      }
    }
  } else {
    for (int e = threadIdx.x; e < R * pin; e += kRowThreads) {
      const int r = e / pin, k = e - r * pin;
      const float v = (row0 + r < a.batch && k < a.d.n_in)
                          ? a.x[(int64_t)(row0 + r) * a.d.n_in + k] : 0.0f;
      const uint16_t q = to_bf16(v);
      sIn[(8 * (r / (2 * Q)) + 4 * ((r / Q) & 1) + r % Q) * ld + k] = q;
      if (TRAIN) a.xf[frag_at(k, row0 + r, ksb)] = q;
    }
  }
  __syncthreads();

  const float scale = 2.0f / (float)((int64_t)a.batch * a.d.n_out);
  for (int l = 0; l <= L; ++l) {
    const MlpLayer lay = mlp_layer(a.d, l);
    const bool last = l == L;
    const int ks = pad32(lay.di) >> 4, tiles = pad32(lay.dn) >> 5;
    const uint16_t* wl = a.wf + lay.packed;
    // what follows this layer: the next one, or the way back from the last
    const uint16_t* nw = nullptr;
    int ntiles = 0, nks = 0;
    if (!last) {
      nw = a.wf + mlp_layer(a.d, l + 1).packed;
      ntiles = (l + 1 == L ? po : pw) >> 5;
      nks = pw >> 4;
    } else if (TRAIN && L > 0) {
      nw = a.wt + lay.packed;
      ntiles = pw >> 5;
      nks = po >> 4;
    }
    const float* bias = a.par + lay.w + (int64_t)lay.di * lay.dn;
    const uint16_t* row = sIn + col * ld + h * 8;
    for (int nt = wave; nt < tiles; nt += waves) {
      const int n = nt * 32 + col;
      // what the epilogue needs, on its way during the product
      const float bn = n < lay.dn ? bias[n] : 0.0f;
      float tg[E];
      if (TRAIN && last) {
#pragma unroll
        for (int q = 0; q < E; ++q) {
          const int r = row0 + 2 * Q * (q / Q) + Q * h + q % Q;
          tg[q] = r < a.batch && n < a.d.n_out ? a.target[(int64_t)r * a.d.n_out + n] : 0.0f;
        }
      }
      const f32x16 acc = product(b, wl + (int64_t)nt * ks * 512, ks, row, lane);
      fetch_next(b, wl, nt + waves, tiles, ks, nw, ntiles, nks, wave, lane);
      if (!last) {
        float* gg = nullptr;
        if (TRAIN) gg = a.gg + ((int64_t)l * a.rows + row0) * pw + ((int64_t)nt * 64 + lane) * E;
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int r = row0 + 2 * Q * j + Q * h;
          uint16_t qv[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const float z = acc[4 * j + q] + bn;
            // the padding stays zero whatever the row holds: zero weights times
            // an infinite activation are not a number, and the next layer's
            // padded products would spread it over the row
            const uint16_t v = n < lay.dn ? to_bf16(gelu(z)) : (uint16_t)0;
            sOut[(8 * j + 4 * h + q) * ld + n] = v;
            if (TRAIN) {
              qv[q] = r + q < a.batch ? v : (uint16_t)0;
              gg[Q * j + q] = gelu_grad(z);
            }
          }
          if (TRAIN)
            store_run<Q>(a.xf + ((int64_t)pin + (int64_t)l * pw) * a.rows, n, r, ksb, qv);
        }
      } else {
        float* dz = TRAIN ? a.dz + (int64_t)L * pw * a.rows : nullptr;
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int r = row0 + 2 * Q * j + Q * h;
          uint16_t qv[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const bool in = r + q < a.batch && n < a.d.n_out;
            const int64_t o = (int64_t)(r + q) * a.d.n_out + n;
            const float v = acc[4 * j + q] + bn;
            if (in) a.y[o] = v;
            if (TRAIN) {
              const float t = in ? scale * (v - tg[Q * j + q]) : 0.0f;
              dz[(int64_t)(r + q) * po + n] = t;
              qv[q] = to_bf16(t);
              sOut[(8 * j + 4 * h + q) * ld + n] = qv[q];
            }
          }
          if (TRAIN) store_run<Q>(a.dzf + (int64_t)L * pw * a.rows, n, r, ksb, qv);
        }
      }
    }
    if (wave >= tiles) fetch_next(b, nullptr, 0, 0, 0, nw, ntiles, nks, wave, lane);
    __syncthreads();
    uint16_t* t = sIn;
    sIn = sOut;
    sOut = t;
  }
  if (!TRAIN) return;

  // dZ_{l-1} = (dZ_l W_l) gelu'(Z_{l-1})
  for (int l = L; l > 0; --l) {
    const int ks = (l == L ? po : pw) >> 4, tiles = pw >> 5;
    const uint16_t* wl = a.wt + mlp_layer(a.d, l).packed;
    const uint16_t* nw = l > 1 ? a.wt + mlp_layer(a.d, l - 1).packed : nullptr;
    const int ntiles = l > 1 ? pw >> 5 : 0, nks = pw >> 4;
    const uint16_t* row = sIn + col * ld + h * 8;
    float* dz = a.dz + (int64_t)(l - 1) * pw * a.rows;
    for (int nt = wave; nt < tiles; nt += waves) {
      // written by this same lane on the way forward
      const float* gg = a.gg + ((int64_t)(l - 1) * a.rows + row0) * pw + ((int64_t)nt * 64 + lane) * E;
      float g[E];
#pragma unroll
      for (int q = 0; q < E; ++q) g[q] = gg[q];
      const f32x16 acc = product(b, wl + (int64_t)nt * ks * 512, ks, row, lane);
      fetch_next(b, wl, nt + waves, tiles, ks, nw, ntiles, nks, wave, lane);
      const int n = nt * 32 + col;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int r = row0 + 2 * Q * j + Q * h;
        uint16_t qv[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          float v = acc[4 * j + q] * g[Q * j + q];
          if (r + q >= a.batch || n >= a.d.width) v = 0.0f;
          dz[(int64_t)(r + q) * pw + n] = v;
          qv[q] = to_bf16(v);
          sOut[(8 * j + 4 * h + q) * ld + n] = qv[q];
        }
        store_run<Q>(a.dzf + (int64_t)(l - 1) * pw * a.rows, n, r, ksb, qv);
      }
    }
    if (wave >= tiles) fetch_next(b, nullptr, 0, 0, 0, nw, ntiles, nks, wave, lane);
    __syncthreads();
    uint16_t* t = sIn;
    sIn = sOut;
    sOut = t;
  }
}

// Everything that crosses rows, one wave per 32 x 32 tile of a weight gradient
// or per 64 biases, and workgroup 0 for the loss. ADAM: the parameters the
// wave has just computed the gradient of are stepped and repacked.
template <bool ADAM>
__global__ __launch_bounds__(kUpdateThreads) void k_mlp_update(MlpArgs a, AdamArgs ad, uint16_t* wf,
                                                    uint16_t* wt, int tiles) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int pin = pad32(a.d.n_in), pw = pad32(a.d.width), po = pad32(a.d.n_out);
  const int L = a.d.depth;
  if (blockIdx.x == 0) {
    // mean squared error: 1024 partial sums, P per thread, in 16 groups of 64
    constexpr int P = 1024 / kUpdateThreads;
    __shared__ float s_part[16];
    const int64_t count = (int64_t)a.batch * a.d.n_out;
    float s[P] = {};
    int64_t i = threadIdx.x;
    for (; i + 31 * kUpdateThreads < count; i += 32 * kUpdateThreads) {
      float y[32], t[32];
#pragma unroll
      for (int q = 0; q < 32; ++q) {
        y[q] = a.y[i + kUpdateThreads * q];
        t[q] = a.target[i + kUpdateThreads * q];
      }
#pragma unroll
      for (int q = 0; q < 32; ++q) {
        const float d = y[q] - t[q];
        s[q % P] += d * d;
      }
    }
    for (; i < count; i += 1024) {
#pragma unroll
      for (int q = 0; q < P; ++q)
        if (i + kUpdateThreads * q < count) {
          const float d = a.y[i + kUpdateThreads * q] - a.target[i + kUpdateThreads * q];
          s[q] += d * d;
        }
    }
#pragma unroll
    for (int q = 0; q < P; ++q) {
      for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
      if (lane == 0) s_part[wave + kUpdateWaves * q] = s[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = 0.0f;
      for (int w = 0; w < 16; ++w) t += s_part[w];
      *a.loss = t / (float)count;
    }
    return;
  }

  int job = (blockIdx.x - 1) * kUpdateWaves + wave;
  if (job >= tiles) {
    // db[n] = sum over the rows, in order
    const int c = (job - tiles) * 64 + lane;
    const int l = a.d.depth > 0 && c / a.d.width < L ? c / a.d.width : L;
    const MlpLayer lay = mlp_layer(a.d, l);
    const int n = c - l * a.d.width;
    if (n >= lay.dn) return;
    const int ld = l == L ? po : pw;
    const float* dz = a.dz + (int64_t)l * pw * a.rows + n;
    float s = 0.0f;
    int m = 0;
    for (; m + 32 <= a.batch; m += 32) {
      float v[32];
#pragma unroll
      for (int q = 0; q < 32; ++q) v[q] = dz[(int64_t)(m + q) * ld];
#pragma unroll
      for (int q = 0; q < 32; ++q) s += v[q];
    }
    for (; m < a.batch; ++m) s += dz[(int64_t)m * ld];
    const int64_t w = lay.w + (int64_t)lay.di * lay.dn + n;
    a.grad[w] = s;
    if (ADAM) (void)adam_step(ad, w, s, ad.w[w], ad.m[w], ad.v[w]);
    return;
  }

  // dW[o][i] = sum over the rows of dZ[m][o] X[m][i]
  int l = 0, ti = pin >> 5, to = (L == 0 ? po : pw) >> 5;
  while (job >= ti * to) {
    job -= ti * to;
    ++l;
    ti = pw >> 5;
    to = (l == L ? po : pw) >> 5;
  }
  const MlpLayer lay = mlp_layer(a.d, l);
  const int tile_o = job / ti, tile_i = job - tile_o * ti;
  const int ksb = a.rows >> 4;
  const uint16_t* pa = a.dzf + (int64_t)l * pw * a.rows + (int64_t)tile_o * ksb * 512 + lane * 8;
  const uint16_t* pb = a.xf + (l == 0 ? 0 : ((int64_t)pin + (int64_t)(l - 1) * pw) * a.rows) +
                       (int64_t)tile_i * ksb * 512 + lane * 8;
  const int h = lane >> 5;
  const int i = tile_i * 32 + (lane & 31);
  // the parameters and their moments, on their way during the product
  float pw_[16], pm[16], pv[16];
  if (ADAM) {
#pragma unroll
    for (int g = 0; g < 16; ++g) {
      const int o = tile_o * 32 + 8 * (g >> 2) + 4 * h + (g & 3);
      const bool in = i < lay.di && o < lay.dn;
      const int64_t w = in ? lay.w + (int64_t)o * lay.di + i : 0;
      pw_[g] = ad.w[w];
      pm[g] = ad.m[w];
      pv[g] = ad.v[w];
    }
  }
  f32x16 acc = {};
  for (int k = 0; k < ksb; k += 4) {
    short8 fa[4], fb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k + q < ksb) {
        fa[q] = *reinterpret_cast<const short8*>(pa + (int64_t)(k + q) * 512);
        fb[q] = *reinterpret_cast<const short8*>(pb + (int64_t)(k + q) * 512);
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k + q < ksb) acc = mfma(fa[q], fb[q], acc);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint16_t q4[4] = {0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = tile_o * 32 + 8 * j + 4 * h + q;
      if (i >= lay.di || o >= lay.dn) continue;
      const int64_t w = lay.w + (int64_t)o * lay.di + i;
      a.grad[w] = acc[4 * j + q];
      if (ADAM) {
        q4[q] = to_bf16(adam_step(ad, w, acc[4 * j + q], pw_[4 * j + q], pm[4 * j + q], pv[4 * j + q]));
        wf[lay.packed + frag_at(o, i, pad32(lay.di) >> 4)] = q4[q];
      }
    }
    if (ADAM) store_run<4>(wt + lay.packed, i, tile_o * 32 + 8 * j + 4 * h, pad32(lay.dn) >> 4, q4);
  }
}

// Packed weights from the parameter vector, eight per thread, padding zero.
__global__ __launch_bounds__(256) void k_mlp_pack(MlpDims d, const float* __restrict__ par,
                                                  uint16_t* __restrict__ wf,
                                                  uint16_t* __restrict__ wt) {
  const int64_t total = mlp_packed(d) / 8;
  int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool back = e >= total;
  if (back) e -= total;
  if (e >= total || (back && !wt)) return;
  const int64_t first = mlp_layer(d, d.depth > 0 ? 1 : 0).packed / 8;
  const int64_t hidden = (int64_t)pad32(d.width) * pad32(d.width) / 8;
  int l = 0;
  if (d.depth > 0 && e >= first) {
    const int64_t q = 1 + (e - first) / hidden;
    l = q < d.depth ? (int)q : d.depth;
  }
  const MlpLayer lay = mlp_layer(d, l);
  const int64_t r = e - lay.packed / 8;  // fragment lanes into the layer
  const int ks = pad32(back ? lay.dn : lay.di) >> 4;
  const int lane = (int)(r & 63);
  const int64_t blk = r >> 6;
  const int f = (int)(blk / ks) * 32 + (lane & 31);
  const int k0 = (int)(blk % ks) * 16 + (lane >> 5) * 8;
  const float* w = par + lay.w;
  uint32_t v[4];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int n = back ? k0 + q : f, i = back ? f : k0 + q;
    const uint32_t u = n < lay.dn && i < lay.di ? to_bf16(w[(int64_t)n * lay.di + i]) : 0u;
    v[q >> 1] = (q & 1) ? v[q >> 1] | (u << 16) : u;
  }
  *reinterpret_cast<uint4*>((back ? wt : wf) + e * 8) = make_uint4(v[0], v[1], v[2], v[3]);
}

}  // namespace

size_t mlp_xf_elems(const MlpDims& d, int rows) {
  return ((size_t)pad32(d.n_in) + (size_t)d.depth * pad32(d.width)) * rows;
}
size_t mlp_dz_elems(const MlpDims& d, int rows) {
  return ((size_t)d.depth * pad32(d.width) + (size_t)pad32(d.n_out)) * rows;
}
size_t mlp_gg_elems(const MlpDims& d, int rows) {
  return (size_t)d.depth * pad32(d.width) * rows;
}

hipError_t launch_mlp_pack(const MlpDims& d, const float* par, uint16_t* wf, uint16_t* wt,
                           hipStream_t s) {
  const int64_t n = mlp_packed(d) / 8 * (wt ? 2 : 1);
  hipLaunchKernelGGL(k_mlp_pack, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, par, wf, wt);
  return hipGetLastError();
}

// Waves of a workgroup of a prediction with 32 rows each. A layer of few tiles
// leaves the waves beyond them idle, and a CU holds about sixteen of this
// kernel, so where there are more workgroups than CUs the fewest rounds of tiles
// decide: the tiles of a wave over all layers (a wave stages four inputs of a
// lane per row like a tile), times the workgroups that wait for their turn. us
// for 65536 rows, eight waves / these / layer by layer: (6, 2 x 32, 32) 99 / 41
// / 55, (6, 16, 1) 76 / 36 / 38, (6, 4 x 32, 512) 171 / 85 / 150, (256, 2 x 32,
// 32) 159 / 86 / 100, (1024, 32, 32) 381 / 236 / 233, (6, 3 x 200, 512) 208 /
// 138 / 754.
static int row_waves(const MlpDims& d, int groups, size_t lds) {
  int best = kRowWaves;
  double cost = 0.0;
  for (int w = kRowWaves; w >= 1; w >>= 1) {
    int tiles = ((pad32(d.n_in) >> 7) + w - 1) / w;
    for (int l = 0; l <= d.depth; ++l) tiles += ((pad32(mlp_layer(d, l).dn) >> 5) + w - 1) / w;
    const int fit = (int)((160 << 10) / lds), held = 16 / w < fit ? 16 / w : fit;
    const double rounds = (double)groups / ((double)kCus * held);
    const double c = tiles * (rounds > 1.0 ? rounds : 1.0);
    if (w == kRowWaves || c < cost || (c == cost && groups > kCus)) {
      cost = c;
      best = w;
    }
  }
  return best;
}

template <bool TRAIN, int E>
static hipError_t launch_rows(const MlpArgs& a, hipStream_t s) {
  // 8 more per row: rows start on different banks, 16-byte aligned
  const int ld = mlp_row(a.d, TRAIN) + 8;
  // training covers the rows of the padding too, whose deltas have to be zero
  const int rows = TRAIN ? a.rows : a.batch;
  const int groups = (rows + 2 * E - 1) / (2 * E);
  const size_t lds = (size_t)ld * 2 * 32 * 2;
  const int waves = TRAIN || E < 16 ? kRowWaves : row_waves(a.d, groups, lds);
  hipLaunchKernelGGL((k_mlp_rows<TRAIN, E>), dim3(groups), dim3(64 * waves), lds, s, a, ld);
  return hipGetLastError();
}

// Rows per lane: the fewest with which a workgroup per compute unit takes the
// whole batch, as the epilogues (GELU, about 100 instructions per element) are
// the larger part of a workgroup's time beyond a few rows. Training step of
// (6, 4 x 256, 512) with 1 / 2 / 4 / 16 elements per lane, us: 96 rows 40 / 43
// / 47 / 71, 512 rows 55 / 57 / 61 / 87, 1024 rows 102 / 78 / 81 / 108, 2048
// rows 197 / 148 / 121 / 150, 4096 rows 388 / 290 / 237 / 235; forward pass of
// 2048 rows 39 / 22 / 18 / 29, of 4096 rows 75 / 40 / 34 / 29.
template <bool TRAIN>
static hipError_t pick_rows(const MlpArgs& a, hipStream_t s) {
  if (a.batch < 1 || a.rows != pad32(a.batch) || mlp_row(a.d, TRAIN) > kMlpMaxRow)
    return hipErrorInvalidValue;
  const int e = (a.batch + 2 * kCus - 1) / (2 * kCus);
  if (e <= 1) return launch_rows<TRAIN, 1>(a, s);
  if (e <= 2) return launch_rows<TRAIN, 2>(a, s);
  if (e <= 4) return launch_rows<TRAIN, 4>(a, s);
  return launch_rows<TRAIN, 16>(a, s);
}

hipError_t launch_mlp_forward(const MlpArgs& a, hipStream_t s) { return pick_rows<false>(a, s); }
hipError_t launch_mlp_deltas(const MlpArgs& a, hipStream_t s) { return pick_rows<true>(a, s); }

hipError_t launch_mlp_update(const MlpArgs& a, const AdamArgs* adam, uint16_t* wf, uint16_t* wt,
                             hipStream_t s) {
  int tiles = 0;
  for (int l = 0; l <= a.d.depth; ++l) {
    const MlpLayer lay = mlp_layer(a.d, l);
    tiles += (pad32(lay.di) >> 5) * (pad32(lay.dn) >> 5);
  }
  const int cols = (a.d.depth * a.d.width + a.d.n_out + 63) / 64;
  const dim3 g(1 + (unsigned)((tiles + cols + kUpdateWaves - 1) / kUpdateWaves));
  if (adam)
    hipLaunchKernelGGL(k_mlp_update<true>, g, dim3(kUpdateThreads), 0, s, a, *adam, wf, wt, tiles);
  else
    hipLaunchKernelGGL(k_mlp_update<false>, g, dim3(kUpdateThreads), 0, s, a, AdamArgs{}, nullptr, nullptr, tiles);
  return hipGetLastError();
}

}  // namespace pic
