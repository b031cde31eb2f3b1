// FP32 training of the networks that the chained kernels take (hidden width 64, 128 or 256, at most 64
// inputs and 192 outputs): the forward, the backward down to dX and the weight products of a batch in
// three launches and a reduction, on v_mfma_f32_16x16x4f32.  Included by train.hip.
//
//   k_pack_f32t     weights in operand order, forward and transposed, and padded biases
//   k_f32_fwd       X -> hidden outputs (kept for the backward) -> sigmoid heads, the layers chained in
//                   registers
//   k_f32_bwd       dZ of the head -> dZ of every hidden layer -> dX, chained the same way
//   k_f32_dw        dW_k = dZ_k^T H_{k-1} and db_k of every layer in one launch, 64 x 64 tiles, the batch
//                   split into ranges; k_train_dw_reduce adds the ranges in a fixed order (no atomics)
//
// A wave owns 16 positions: lane (j, g) = (lane % 16, lane / 16).  Positions are the columns of every
// product, neurons its rows: accumulator v of output tile t is neuron 16t + 4g + v of position j, and the B
// operand of K-step s is row 4s + g.  The weights stream through LDS in chunks of kF32Chunk output tiles
// over the full K (double-buffered, fetched by direct DMA under the previous chunk's products); a lane's A
// values of four K-steps are one 16-byte read.
//
// The forward sums each output in K order from zero and adds the bias last, so its heads do not depend on
// how the batch is tiled (the loss takes hard choices on them): a layer's accumulators are turned into the
// next layer's operands in natural order by a 4 x 4 exchange among the lane groups (two half-wave and two
// quarter-wave register swaps for four registers).  The backward has no choices to keep: its operands stay
// where they are, and its weights are packed with the columns in that order.
//
//   k_f32_fwd_narrow, k_f32_bwd_dw
//                   for the narrow networks of the two-network layout (width 64, three SELU layers, at most 16
//                   inputs and 48 outputs) the features and the forward as one, and the last two as one: neither dZ nor
//                   a second read of the layer inputs passes through memory
//
// What it replaces: a product a launch for every layer and direction, 64 x 64 tiles with one 16-deep slice
// in flight, activations read back between the layers, and weight products adding to one matrix with
// float atomics.  16,384 positions, 48-128x3-162: 380 -> 125 us of products; the matrix cores need
// 38 us for them at the FP32 rate.

constexpr int kF32Waves = 4;
constexpr int kF32Threads = 64 * kF32Waves;
constexpr int kF32Pos = 16 * kF32Waves;  // positions per workgroup
constexpr int kF32MaxChunks = 80;        // width 256: 16 chunks a hidden layer, at most 12 for the head
constexpr int kF32HeadTiles = 12;
constexpr int kF32Groups = 4;            // groups of 16 first-layer inputs

template <int H>
constexpr int f32_chunk_tiles() {
  return H == 256 ? 1 : 2;
}

struct F32Chunks {
  int n, cap;  // chunks; u32x4 slots of one chunk buffer
  int src[kF32MaxChunks], len[kF32MaxChunks];
};

struct F32PackArgs {
  const float* w;
  int n_layers;
  int in_dim[kFMaxLayers], out_dim[kFMaxLayers];
  int64_t w_off[kFMaxLayers], b_off[kFMaxLayers];
  int f_tiles[kFMaxLayers], f_groups[kFMaxLayers], f_off[kFMaxLayers];  // forward: row tiles, K groups of 16, u32x4 offset
  int b_tiles[kFMaxLayers], b_groups[kFMaxLayers], b_off2[kFMaxLayers];
  int bias_off[kFMaxLayers];
  u32x4* pack;
  float* bias;
  float* zero5;  // when set, five floats that block (0, 0) zeroes (a step's loss sums and flag)
};

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Unit (tile t, group q, lane l), element v: forward W[16t + l%16][16q + 4v + l/16] (natural K order),
// transposed W[16q + 4 (l/16) + v][16t + l%16] (the accumulators' order).
__global__ void __launch_bounds__(256) k_pack_f32t(F32PackArgs a) {
  if (a.zero5 != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 5) a.zero5[threadIdx.x] = 0.0f;
  const int layer = blockIdx.y >> 1;
  const bool bwd = (blockIdx.y & 1) != 0;
  if (layer >= a.n_layers) return;
  const int in = a.in_dim[layer], out = a.out_dim[layer];
  const float* w = a.w + a.w_off[layer];
  const int groups = bwd ? a.b_groups[layer] : a.f_groups[layer];
  const int total = (bwd ? a.b_tiles[layer] : a.f_tiles[layer]) * groups * 64;
  u32x4* dst = a.pack + (bwd ? a.b_off2[layer] : a.f_off[layer]);
  for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int l = e & 63, tq = e >> 6, t = tq / groups, q = tq - t * groups;
    const int m = 16 * t + (l & 15), g = l >> 4;
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int row = bwd ? 16 * q + 4 * g + k : m, col = bwd ? m : 16 * q + 4 * k + g;
      v[k] = row < out && col < in ? w[(int64_t)row * in + col] : 0.0f;
    }
    dst[e] = u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
  }
  if (!bwd)
    for (int i = blockIdx.x * 256 + threadIdx.x; i < a.f_tiles[layer] * 16; i += gridDim.x * 256)
      a.bias[a.bias_off[layer] + i] = i < out ? a.w[a.b_off[layer] + i] : 0.0f;
}

struct F32FwdArgs {
  const float* x;  // [n][in_dim]
  int in_dim, n_layers, head_dim, head_tiles;
  int64_t n;
  const u32x4* wpack;
  const float* bias;
  int bias_off[kFMaxLayers], n_bias;
  float* h[kFMaxLayers - 1];  // hidden outputs [n][H]
  float* y;                   // [n][head_dim]
  F32Chunks ct;
};

struct F32BwdArgs {
  const float* dz;  // [n][head_dim]
  int in_dim, n_layers, head_dim, head_tiles;
  int64_t n;
  const u32x4* wpack;
  const float* h[kFMaxLayers - 1];
  float* dh[kFMaxLayers - 1];  // dZ of the hidden layers [n][H]
  float* dx;                   // [n][in_dim]
  F32Chunks ct;
};

__device__ __forceinline__ void f32_dma(const u32x4* __restrict__ wp, const F32Chunks& ct, int c, u32x4* dst, int tid) {
  if (c >= ct.n) return;
  const int wave_base = __builtin_amdgcn_readfirstlane(tid & ~63);
  const int len = ct.len[c];
  const u32x4* src = wp + ct.src[c];
  for (int r = 0; r * kF32Threads < len; ++r) {
    const int e = tid + kF32Threads * r;
    if (e < len)
      __builtin_amdgcn_global_load_lds(src + e, (__attribute__((address_space(3))) void*)(dst + wave_base + kF32Threads * r),
                                       16, 0, 0);
  }
}

// out[v] of lane group g = in[g] of lane group v.
__device__ __forceinline__ f32x4_t f32_natural(const f32x4_t& r) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(r[0]), __float_as_uint(r[2]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(r[1]), __float_as_uint(r[3]), false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return f32x4_t{__uint_as_float(c[0]), __uint_as_float(c[1]), __uint_as_float(d[0]), __uint_as_float(d[1])};
}

// Elements c .. c+3 of a row of `cols` floats (zero past its end; rows need not be 16-byte aligned).
__device__ __forceinline__ f32x4_t f32_row4(const float* row, int c, int cols) {
  if (c + 3 < cols) return *reinterpret_cast<const f32x4_a4*>(row + c);
  f32x4_t r{};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (c + k < cols) r[k] = row[c + k];
  return r;
}

__device__ __forceinline__ void f32_put4(float* row, int c, int cols, const f32x4_t& v) {
  if (c + 3 < cols) {
    *reinterpret_cast<f32x4_a4*>(row + c) = v;
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (c + k < cols) row[c + k] = v[k];
}

// CT output tiles (those below `valid`) from the chunk at wb over Q groups of 16 K values, of which the first
// `groups` are in the chunk.
template <int CT, int Q>
__device__ __forceinline__ void f32_products(const u32x4* wb, const f32x4_t (&b)[Q], int groups, int valid, int lane,
                                             f32x4_t (&acc)[CT]) {
#pragma unroll
  for (int u = 0; u < CT; ++u) acc[u] = f32x4_t{};
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q < groups) {
      f32x4_t w[CT];
#pragma unroll
      for (int u = 0; u < CT; ++u)
        if (u < valid) w[u] = __builtin_bit_cast(f32x4_t, wb[(u * groups + q) * 64 + lane]);
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int u = 0; u < CT; ++u)
          if (u < valid) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][v], b[q][v], acc[u], 0, 0, 0);
    }
  }
}

// One hidden layer: products, bias, activation; the outputs go to `store` (row-major, the lane's row) and,
// in natural order, into `out`.
template <int H, int Q>
__device__ __forceinline__ void f32_fwd_layer(const F32FwdArgs& a, const f32x4_t (&in)[Q], f32x4_t (&out)[H / 16], const float* bl,
                                              float* store, bool valid, u32x4* smem, int& c, int tid, int lane) {
  constexpr int CT = f32_chunk_tiles<H>();
  const int g = lane >> 4;
#pragma unroll
  for (int tc = 0; tc < H / 16 / CT; ++tc) {
    f32_dma(a.wpack, a.ct, c + 1, smem + ((c + 1) & 1) * a.ct.cap, tid);
    f32x4_t acc[CT];
    f32_products<CT, Q>(smem + (c & 1) * a.ct.cap, in, Q, CT, lane, acc);
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      const int t = CT * tc + u;
      const float4 b = *reinterpret_cast<const float4*>(bl + 16 * t + 4 * g);
      const float bv[4] = {b.x, b.y, b.z, b.w};
      f32x4_t r;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float z = acc[u][v] + bv[v];
        r[v] = z < 0.0f ? 0.0f : z;  // ReLU that keeps NaN
      }
      if (valid) *reinterpret_cast<f32x4_t*>(store + 16 * t + 4 * g) = r;
      out[t] = f32_natural(r);
    }
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

template <int H, int KQ>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(H == 256 ? 2 : (H == 128 ? 3 : 4))))
k_f32_fwd(F32FwdArgs a) {
  constexpr int CT = f32_chunk_tiles<H>(), Q = H / 16;
  extern __shared__ u32x4 smem[];
  float* bias_s = reinterpret_cast<float*>(smem + 2 * a.ct.cap);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int64_t p = ((int64_t)blockIdx.x * kF32Waves + wave) * 16 + j;
  const bool valid = p < a.n;
  const int64_t pc = valid ? p : a.n - 1;
  f32_dma(a.wpack, a.ct, 0, smem, tid);
  for (int i = tid; i < a.n_bias; i += kF32Threads) bias_s[i] = a.bias[i];
  f32x4_t x0[KQ];
#pragma unroll
  for (int q = 0; q < KQ; ++q) x0[q] = f32_natural(f32_row4(a.x + pc * a.in_dim, 16 * q + 4 * g, a.in_dim));
  fwait_dma();
  __syncthreads();
  int c = 0;
  f32x4_t in[Q], out[Q];
  f32_fwd_layer<H, KQ>(a, x0, in, bias_s + a.bias_off[0], a.h[0] + pc * H, valid, smem, c, tid, lane);
  for (int layer = 1; layer < a.n_layers - 1; ++layer) {
    f32_fwd_layer<H, Q>(a, in, out, bias_s + a.bias_off[layer], a.h[layer] + pc * H, valid, smem, c, tid, lane);
#pragma unroll
    for (int q = 0; q < Q; ++q) in[q] = out[q];
  }
  const float* bl = bias_s + a.bias_off[a.n_layers - 1];
  for (int t0 = 0; t0 < a.head_tiles; t0 += CT) {
    f32_dma(a.wpack, a.ct, c + 1, smem + ((c + 1) & 1) * a.ct.cap, tid);
    f32x4_t acc[CT];
    f32_products<CT, Q>(smem + (c & 1) * a.ct.cap, in, Q, a.head_tiles - t0, lane, acc);
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      if (t0 + u >= a.head_tiles) continue;
      const int n0 = 16 * (t0 + u) + 4 * g;
      f32x4_t r;
#pragma unroll
      for (int v = 0; v < 4; ++v) r[v] = 1.0f / (1.0f + expf(-(acc[u][v] + bl[n0 + v])));
      if (valid) f32_put4(a.y + p * a.head_dim, n0, a.head_dim, r);
    }
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

// dZ of a hidden layer: the products of Wᵀ with the layer above's dZ (the first `groups` groups of `in`),
// times the activation's derivative, taken from the layer's outputs h.
template <int H, int QI>
__device__ __forceinline__ void f32_bwd_layer(const F32BwdArgs& a, const f32x4_t (&in)[QI], int groups, f32x4_t (&out)[H / 16],
                                              const float* h, float* store, bool valid, u32x4* smem, int& c, int tid, int lane) {
  constexpr int CT = f32_chunk_tiles<H>();
  const int g = lane >> 4;
#pragma unroll
  for (int tc = 0; tc < H / 16 / CT; ++tc) {
    f32x4_t hv[CT];
#pragma unroll
    for (int u = 0; u < CT; ++u) hv[u] = *reinterpret_cast<const f32x4_t*>(h + 16 * (CT * tc + u) + 4 * g);
    f32_dma(a.wpack, a.ct, c + 1, smem + ((c + 1) & 1) * a.ct.cap, tid);
    f32x4_t acc[CT];
    f32_products<CT, QI>(smem + (c & 1) * a.ct.cap, in, groups, CT, lane, acc);
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      const int t = CT * tc + u;
      f32x4_t r;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        r[v] = hv[u][v] > 0.0f ? acc[u][v] : 0.0f;
      if (valid) *reinterpret_cast<f32x4_t*>(store + 16 * t + 4 * g) = r;
      out[t] = r;
    }
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

template <int H, int KQ>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(H == 256 ? 2 : (H == 128 ? 3 : 4))))
k_f32_bwd(F32BwdArgs a) {
  constexpr int CT = f32_chunk_tiles<H>(), Q = H / 16;
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j = lane & 15, g = lane >> 4;
  const int64_t p = ((int64_t)blockIdx.x * kF32Waves + wave) * 16 + j;
  const bool valid = p < a.n;
  const int64_t pc = valid ? p : a.n - 1;
  f32_dma(a.wpack, a.ct, 0, smem, tid);
  f32x4_t out[Q];
  int c = 0, layer = a.n_layers - 2;
  {
    f32x4_t head[kF32HeadTiles];
#pragma unroll
    for (int q = 0; q < kF32HeadTiles; ++q)
      head[q] = q < a.head_tiles ? f32_row4(a.dz + pc * a.head_dim, 16 * q + 4 * g, a.head_dim) : f32x4_t{};
    fwait_dma();
    __syncthreads();
    f32_bwd_layer<H, kF32HeadTiles>(a, head, a.head_tiles, out, a.h[layer] + pc * H, a.dh[layer] + pc * H, valid, smem, c,
                                          tid, lane);
  }
  for (--layer; layer >= 0; --layer) {
    f32x4_t in[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) in[q] = out[q];
    f32_bwd_layer<H, Q>(a, in, Q, out, a.h[layer] + pc * H, a.dh[layer] + pc * H, valid, smem, c, tid, lane);
  }
#pragma unroll
  for (int t0 = 0; t0 < KQ; t0 += CT) {
    f32_dma(a.wpack, a.ct, c + 1, smem + ((c + 1) & 1) * a.ct.cap, tid);
    f32x4_t acc[CT];
    f32_products<CT, Q>(smem + (c & 1) * a.ct.cap, out, Q, KQ - t0, lane, acc);
#pragma unroll
    for (int u = 0; u < CT; ++u)
      if (t0 + u < KQ && valid) f32_put4(a.dx + p * a.in_dim, 16 * (t0 + u) + 4 * g, a.in_dim, acc[u]);
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

// Weight products, FP32: block = (tile, batch range).  Four waves, each a 32 x 32 quadrant as 2 x 2 products;
// slices of 16 positions of both operands (row-major: the contraction index is the row) go through two LDS
// buffers, the next slice in registers meanwhile.  Rows 80 floats apart put the four lane groups of a read
// on different banks.
constexpr int kF32DwTile = 64, kF32DwK = 16, kF32DwLd = 80;

struct F32DwJob {
  const float *a, *b;  // dZ [n][M], layer inputs [n][N]
  int M, N, tiles_n, tile0;
};

struct F32DwArgs {
  F32DwJob job[kFMaxLayers];
  int n_jobs, n_tiles, splits, k_split;
  int64_t n;
  float *part, *dbpart;  // [n_tiles][splits][64 * 64], [n_tiles][splits][64]
};

__global__ void __launch_bounds__(256) k_f32_dw(F32DwArgs a) {
  __shared__ __align__(16) float As[2][kF32DwK][kF32DwLd];
  __shared__ __align__(16) float Bs[2][kF32DwK][kF32DwLd];
  // as in k_train_dw: each XCD takes a contiguous run of (range, tile) pairs, tiles fastest
  const int nwg = (int)gridDim.x, per = nwg / 8, extra = nwg % 8, x = (int)blockIdx.x % 8, kx = (int)blockIdx.x / 8;
  const int flat = x * per + (x < extra ? x : extra) + kx;
  const int tile = flat % a.n_tiles, split = flat / a.n_tiles;
  int jb = 0;
  while (jb + 1 < a.n_jobs && tile >= a.job[jb + 1].tile0) ++jb;
  const F32DwJob& J = a.job[jb];
  const int lt = tile - J.tile0, tm = lt / J.tiles_n, tn = lt % J.tiles_n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32, li = lane & 15, g = lane >> 4;
  const int64_t k0 = (int64_t)split * a.k_split, k1 = k0 + a.k_split < a.n ? k0 + a.k_split : a.n;
  // the thread's four columns of slice row tid / 16
  const int sr = tid >> 4, sc = (tid & 15) * 4, am = tm * kF32DwTile + sc, bn = tn * kF32DwTile + sc;
  f32x4_t ra{}, rb{}, cs{};
  auto load = [&](int64_t k) {
    const bool in = k + sr < k1;
    ra = in && am < J.M ? f32_row4(J.a + (k + sr) * J.M, am, J.M) : f32x4_t{};
    rb = in && bn < J.N ? f32_row4(J.b + (k + sr) * J.N, bn, J.N) : f32x4_t{};
  };
  auto store = [&](int buf) {
    cs += ra;
    *reinterpret_cast<f32x4_t*>(&As[buf][sr][sc]) = ra;
    *reinterpret_cast<f32x4_t*>(&Bs[buf][sr][sc]) = rb;
  };
  f32x4_t acc[2][2] = {};
  if (k0 < k1) {
    load(k0);
    store(0);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t k = k0; k < k1; k += kF32DwK) {
    const bool more = k + kF32DwK < k1;
    if (more) load(k + kF32DwK);
#pragma unroll
    for (int s = 0; s < kF32DwK / 4; ++s) {
      float af[2], bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = As[buf][4 * s + g][wm + 16 * i + li];
        bf[i] = Bs[buf][4 * s + g][wn + 16 * i + li];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[jj], acc[i][jj], 0, 0, 0);
    }
    if (more) store(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  float* part = a.part + ((int64_t)tile * a.splits + split) * (kF32DwTile * kF32DwTile);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[(wm + 16 * i + 4 * g + v) * kF32DwTile + wn + 16 * jj + li] = acc[i][jj][v];
  if (tn == 0) {
    // bias gradient: the sixteen threads of a column group hold its slice rows' sums
    *reinterpret_cast<f32x4_t*>(&As[0][sr][sc]) = cs;
    __syncthreads();
    if (tid < kF32DwTile) {
      float t = 0.0f;
#pragma unroll
      for (int r = 0; r < kF32DwK; ++r) t += As[0][r][tid];
      a.dbpart[((int64_t)tile * a.splits + split) * kF32DwTile + tid] = t;
    }
  }
}

// ------------------------------------------------------------------------------------------ width 64: backward and dW
// dZ of the head -> dX and dW, db of every layer, for the networks of the two-network layout.  Their layers are
// so narrow that the two kernels above are bound by memory (65,536 * 16 texels: 0.8 GB of dZ written, read back
// beside the layer inputs' second 0.8 GB; 0.40 + 0.59 ms, where the matrix cores need 0.28 for both).  Here all
// weights stay in LDS and a wave keeps the weight products of its positions in accumulators: 10 to 13 tiles of
// 16 x 16 a layer column, 176 registers with 32 outputs, so one wave a SIMD with all 512
// (a step of 65,536 blocks: 0.98 ms -> 0.51, the matrix cores busy for 0.29).  A workgroup a CU takes
// groups of 16 positions in turn; the next group's rows are loaded under this one's products.  dZ and the layer
// inputs pass through a patch of LDS per wave, from a position's row a lane to a neuron a lane.  Nothing in the
// loop waits for another wave.  At the end the four waves' sums are added in order and each workgroup
// writes one partial, which k_train_dw_reduce adds in workgroup order.
constexpr int kF32NarrowBlocks = 256;  // a CU each
constexpr int kF32NarrowLd = 72;       // floats between the rows of a patch: rows and columns both over the banks
constexpr int kF32NarrowHidden = 3, kF32NarrowHeadTiles = 3;  // eight BC1 textures: 48 endpoint values

struct F32NarrowArgs {
  const float *dz, *x;  // [n][head_dim], [n][in_dim]
  const float* h[kF32NarrowHidden];
  float* dx;
  int in_dim, head_dim;
  int64_t n;
  const u32x4* wpack;
  int src[kF32NarrowHidden + 1];  // u32x4 offsets of the layers' transposed weights
  float *part, *dbpart;           // [layer][gridDim.x][64 * 64], [layer][gridDim.x][64]
};

constexpr int f32_narrow_units(int ht) { return (4 * ht + 2 * 16 + 4) * 64; }
constexpr size_t f32_narrow_lds(int ht) {
  return (size_t)f32_narrow_units(ht) * 16 + (size_t)kF32Waves * 2 * 16 * kF32NarrowLd * 4;
}

// The forward of the same networks: features (as k_features), layers and heads of 16 positions a wave, all weights in
// LDS, sixteen waves a CU that wait for nobody.  A lane gathers the four features it takes as an operand; what is
// written is what the backward reads (features, hidden outputs) and the heads.  Features and streamed
// weights as two launches: 0.12 + 0.35 ms for both networks of 65,536 blocks, now 0.38.  Bound by issue: 1,800 VALU
// instructions a group, over half of them the exponentials of SELU, beside 160 products of 32 cycles.
constexpr int kF32NarrowWaves = 8;

struct F32NarrowFwdArgs {
  FeatArgs f;
  int in_dim, head_dim, head_tiles, n_bias;
  const u32x4* wpack;
  const float* bias;
  int src[kF32NarrowHidden + 1], bias_off[kF32NarrowHidden + 1];
  float* h[kF32NarrowHidden];
  float* y;
};

constexpr int f32_narrow_fwd_units(int ht) { return (4 + 2 * 16 + 4 * ht) * 64; }

// Features c0 .. c0+3 of a position (two levels of two), zero past in_dim; the corners' values with QAT's rounding
// and the sum as in k_features.
__device__ __forceinline__ f32x4_t f32_features(const FeatArgs& a, int id, int c0, int in_dim) {
  f32x4_t r{};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (c0 + 2 * h >= in_dim) continue;
    const int l = c0 / 2 + h;
    const Tap t = grid_tap_id(a, id, l);
    float c[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) dev::load_f32<2>(a.grid + t.vtx[k] * 2, c[k]);
    if (a.stats) {
      const float s = reinterpret_cast<const float*>(a.stats)[2 * NTBC_MAX_LEVELS + l];
      const int z = a.stats[3 * NTBC_MAX_LEVELS + l];
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          bool inside;
          c[k][m] = fake_quant(c[k][m], s, z, &inside);
        }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
      r[2 * h + m] = fmaf(t.w[0], c[0][m], fmaf(t.w[1], c[1][m], fmaf(t.w[2], c[2][m], t.w[3] * c[3][m])));
  }
  return r;
}

template <int Q>
__device__ __forceinline__ void f32_narrow_fwd_layer(const u32x4* w, const float* bias, const f32x4_t (&in)[Q], f32x4_t (&out)[4],
                                                     float* store, bool valid, int lane) {
  const int g = lane >> 4;
#pragma unroll
  for (int t0 = 0; t0 < 4; t0 += 2) {
    f32x4_t acc[2];
    f32_products<2, Q>(w + t0 * Q * 64, in, Q, 2, lane, acc);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = t0 + u;
      const f32x4_t b = *reinterpret_cast<const f32x4_t*>(bias + 16 * t + 4 * g);
      f32x4_t r;
#pragma unroll
      for (int v = 0; v < 4; ++v) r[v] = selu_f(acc[u][v] + b[v]);
      if (valid) *reinterpret_cast<f32x4_t*>(store + 16 * t + 4 * g) = r;
      out[t] = f32_natural(r);
    }
  }
}

__global__ void __launch_bounds__(64 * kF32NarrowWaves) __attribute__((amdgpu_waves_per_eu(4))) k_f32_fwd_narrow(F32NarrowFwdArgs a) {
  extern __shared__ u32x4 smem[];
  constexpr int kW1 = 4 * 64, kW2 = kW1 + 16 * 64, kW3 = kW2 + 16 * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int units = f32_narrow_fwd_units(a.head_tiles);
  for (int at = 64 * wave; at < units; at += 64 * kF32NarrowWaves) {
    const u32x4* from = a.wpack + (at < kW1 ? a.src[0] + at : at < kW2 ? a.src[1] + at - kW1 : at < kW3 ? a.src[2] + at - kW2 : a.src[3] + at - kW3);
    __builtin_amdgcn_global_load_lds(from + lane, (__attribute__((address_space(3))) void*)(smem + at), 16, 0, 0);
  }
  float* bias = reinterpret_cast<float*>(smem + units);
  for (int i = tid; i < a.n_bias; i += 64 * kF32NarrowWaves) bias[i] = a.bias[i];
  fwait_dma();
  __syncthreads();
  const int64_t n = a.f.n, groups = (n + 15) / 16, npos = (int64_t)a.f.blocks_w * a.f.blocks_h;
  for (int64_t grp = (int64_t)blockIdx.x * kF32NarrowWaves + wave; grp < groups; grp += (int64_t)gridDim.x * kF32NarrowWaves) {
    int zero = 0;  // opaque: the weights are to be read in each turn, not kept in registers over the loop
    asm volatile("" : "+v"(zero));
    const int g = (lane >> 4) + zero, j = (lane & 15) + zero;
    const int64_t p = grp * 16 + j;
    const bool valid = p < n;
    const int64_t pc = valid ? p : n - 1;
    const u32x4* w = smem + zero;
    const float* bl = bias + zero;
    const f32x4_t x = f32_features(a.f, clamp_id(a.f.ids[pc], npos), 4 * g, a.in_dim);
    if (valid) f32_put4(a.f.x + p * a.in_dim, 4 * g, a.in_dim, x);
    const f32x4_t x0[1] = {f32_natural(x)};
    f32x4_t u[4], v[4];
    f32_narrow_fwd_layer(w, bl + a.bias_off[0], x0, u, a.h[0] + pc * 64, valid, lane + zero);
    f32_narrow_fwd_layer(w + kW1, bl + a.bias_off[1], u, v, a.h[1] + pc * 64, valid, lane + zero);
    f32_narrow_fwd_layer(w + kW2, bl + a.bias_off[2], v, u, a.h[2] + pc * 64, valid, lane + zero);
    for (int t = 0; t < a.head_tiles; ++t) {
      f32x4_t acc[1], r;
      f32_products<1, 4>(w + kW3 + t * 256, u, 4, 1, lane, acc);
      const int n0 = 16 * t + 4 * g;
#pragma unroll
      for (int k = 0; k < 4; ++k) r[k] = 1.0f / (1.0f + expf(-(acc[0][k] + bl[a.bias_off[3] + n0 + k])));
      if (valid) f32_put4(a.y + p * a.head_dim, n0, a.head_dim, r);
    }
  }
}

template <int HT>
struct F32Rows {  // of one group: a lane's four of every sixteen elements
  f32x4_t dz[HT], x, h[kF32NarrowHidden][4];
};

template <int HT>
__device__ __forceinline__ void f32_narrow_load(const F32NarrowArgs& a, int64_t grp, int lane, F32Rows<HT>* r) {
  const int j = lane & 15, g = lane >> 4;
  const int64_t p = grp * 16 + j, pc = p < a.n ? p : a.n - 1;
#pragma unroll
  for (int q = 0; q < HT; ++q) {
    r->dz[q] = f32_row4(a.dz + pc * a.head_dim, 16 * q + 4 * g, a.head_dim);
    if (p >= a.n) r->dz[q] = f32x4_t{};  // and with it every dZ of the lane's position
  }
  r->x = f32_row4(a.x + pc * a.in_dim, 4 * g, a.in_dim);
#pragma unroll
  for (int k = 0; k < kF32NarrowHidden; ++k)
#pragma unroll
    for (int t = 0; t < 4; ++t) r->h[k][t] = *reinterpret_cast<const f32x4_t*>(a.h[k] + pc * 64 + 16 * t + 4 * g);
}

template <int T>
__device__ __forceinline__ void f32_patch_put(float* patch, const f32x4_t (&v)[T], int lane) {
#pragma unroll
  for (int t = 0; t < T; ++t)
    *reinterpret_cast<f32x4_t*>(patch + (lane & 15) * kF32NarrowLd + 16 * t + 4 * (lane >> 4)) = v[t];
}

// The patches are one wave's: its LDS accesses complete in order, so only the compiler has to keep them so.
__device__ __forceinline__ void f32_patch_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Both operands of the weight products over a patch's 16 positions, K-step s = positions 4s .. 4s+3.
template <int MT, int NT>
struct F32Frags {
  float a[4][MT], b[4][NT];
};

template <int MT, int NT>
__device__ __forceinline__ void f32_patch_get(const float* z, const float* h, int lane, F32Frags<MT, NT>* f) {
  const int li = lane & 15, g = lane >> 4;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int i = 0; i < MT; ++i) f->a[s][i] = z[(4 * s + g) * kF32NarrowLd + 16 * i + li];
#pragma unroll
    for (int k = 0; k < NT; ++k) f->b[s][k] = h[(4 * s + g) * kF32NarrowLd + 16 * k + li];
  }
}

// acc[i][k] += dZ^T H, bs the lane's share of the row sums of dZ^T.
template <int MT, int NT>
__device__ __forceinline__ void f32_patch_dw(const F32Frags<MT, NT>& f, f32x4_t (&acc)[MT][NT], float (&bs)[MT]) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      bs[i] += f.a[s][i];
#pragma unroll
      for (int k = 0; k < NT; ++k) acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[s][i], f.b[s][k], acc[i][k], 0, 0, 0);
    }
}

// T tiles over Q groups of 16 K values, as f32_products, the next group's weights read under this one's products.
template <int T, int Q>
__device__ __forceinline__ void f32_narrow_products(const u32x4* wb, const f32x4_t (&b)[Q], int lane, f32x4_t (&acc)[T]) {
  f32x4_t w[2][T];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    acc[u] = f32x4_t{};
    w[0][u] = __builtin_bit_cast(f32x4_t, wb[u * Q * 64 + lane]);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q + 1 < Q)
#pragma unroll
      for (int u = 0; u < T; ++u) w[(q + 1) & 1][u] = __builtin_bit_cast(f32x4_t, wb[(u * Q + q + 1) * 64 + lane]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int u = 0; u < T; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q & 1][u][v], b[q][v], acc[u], 0, 0, 0);
    if (q + 1 < Q) __builtin_amdgcn_sched_barrier(0);
  }
}

// dZ of a hidden layer from the layer above's, with all four tiles of its weights at w.
template <int Q>
__device__ __forceinline__ void f32_narrow_layer(const u32x4* w, const f32x4_t (&in)[Q], const f32x4_t (&h)[4], int lane,
                                                 f32x4_t (&out)[4]) {
  f32x4_t acc[4];
  f32_narrow_products<4, Q>(w, in, lane, acc);
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) out[t][v] = acc[t][v] * selu_grad_of_out(h[t][v]);
}

// The sums of a layer over the workgroup, wave 0's first, in wave 0's registers; buf holds a wave's sums.
template <int MT, int NT>
__device__ __forceinline__ void f32_wave_put(f32x4_t* buf, int& o, int lane, const f32x4_t (&acc)[MT][NT], const float (&bs)[MT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int k = 0; k < NT; ++k) buf[(o++) * 64 + lane] = acc[i][k];
    buf[(o++) * 64 + lane] = f32x4_t{bs[i], 0.0f, 0.0f, 0.0f};
  }
}

template <int MT, int NT>
__device__ __forceinline__ void f32_wave_add(const f32x4_t* buf, int& o, int lane, f32x4_t (&acc)[MT][NT], float (&bs)[MT]) {
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[i][k] += buf[(o++) * 64 + lane];
    bs[i] += buf[(o++) * 64 + lane][0];
  }
}

template <int MT, int NT>
__device__ __forceinline__ void f32_narrow_part(const F32NarrowArgs& a, int layer, int lane, const f32x4_t (&acc)[MT][NT],
                                                const float (&bs)[MT]) {
  const int li = lane & 15, g = lane >> 4;
  const int64_t slot = (int64_t)layer * gridDim.x + blockIdx.x;
  float* part = a.part + slot * 4096;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[(16 * i + 4 * g + v) * 64 + 16 * k + li] = acc[i][k][v];
    float b = bs[i];
    b += __shfl_xor(b, 16);
    b += __shfl_xor(b, 32);
    if (g == 0) a.dbpart[slot * 64 + 16 * i + li] = b;
  }
}

template <int HT>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(1, 1))) k_f32_bwd_dw(F32NarrowArgs a) {
  extern __shared__ u32x4 smem[];
  constexpr int kW2 = 4 * HT * 64, kW1 = kW2 + 16 * 64, kW0 = kW1 + 16 * 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int u = wave; u < f32_narrow_units(HT) / 64; u += kF32Waves) {
    const int at = 64 * u;
    const u32x4* from = a.wpack + (at < kW2 ? a.src[3] + at : at < kW1 ? a.src[2] + at - kW2 : at < kW0 ? a.src[1] + at - kW1 : a.src[0] + at - kW0);
    __builtin_amdgcn_global_load_lds(from + lane, (__attribute__((address_space(3))) void*)(smem + at), 16, 0, 0);
  }
  float* zp = reinterpret_cast<float*>(smem + f32_narrow_units(HT)) + wave * 2 * 16 * kF32NarrowLd;
  float* hp = zp + 16 * kF32NarrowLd;
  f32x4_t w3[HT][4] = {}, w2[4][4] = {}, w1[4][4] = {}, w0[4][1] = {};
  float b3[HT] = {}, b2[4] = {}, b1[4] = {}, b0[4] = {};
  const int64_t groups = (a.n + 15) / 16, step = (int64_t)gridDim.x * kF32Waves;
  int64_t grp = (int64_t)blockIdx.x * kF32Waves + wave;
  F32Rows<HT> next{};
  if (grp < groups) f32_narrow_load(a, grp, lane, &next);
  fwait_dma();
  __syncthreads();
  for (; grp < groups; grp += step) {
    const F32Rows<HT> r = next;
    f32_narrow_load(a, grp + step < groups ? grp + step : grp, lane, &next);
    f32x4_t d2[4], d1[4], d0[4], dx[1];
    const f32x4_t x[1] = {r.x};
    f32_patch_put(zp, r.dz, lane);
    f32_patch_put(hp, r.h[2], lane);
    f32_patch_order();
    F32Frags<HT, 4> f3;
    f32_patch_get(zp, hp, lane, &f3);
    f32_narrow_layer(smem, r.dz, r.h[2], lane, d2);
    f32_patch_dw(f3, w3, b3);
    f32_patch_order();
    f32_patch_put(zp, d2, lane);
    f32_patch_put(hp, r.h[1], lane);
    f32_patch_order();
    F32Frags<4, 4> f2;
    f32_patch_get(zp, hp, lane, &f2);
    f32_narrow_layer(smem + kW2, d2, r.h[1], lane, d1);
    f32_patch_dw(f2, w2, b2);
    f32_patch_order();
    f32_patch_put(zp, d1, lane);
    f32_patch_put(hp, r.h[0], lane);
    f32_patch_order();
    F32Frags<4, 4> f1;
    f32_patch_get(zp, hp, lane, &f1);
    f32_narrow_layer(smem + kW1, d1, r.h[0], lane, d0);
    f32_patch_dw(f1, w1, b1);
    f32_patch_order();
    f32_patch_put(zp, d0, lane);
    f32_patch_put(hp, x, lane);
    f32_patch_order();
    F32Frags<4, 1> f0;
    f32_patch_get(zp, hp, lane, &f0);
    f32_narrow_products<1, 4>(smem + kW0, d0, lane, dx);
    f32_patch_dw(f0, w0, b0);
    f32_patch_order();
    const int64_t p = grp * 16 + (lane & 15);
    if (p < a.n) f32_put4(a.dx + p * a.in_dim, 4 * (lane >> 4), a.in_dim, dx[0]);
  }
  f32x4_t* buf = reinterpret_cast<f32x4_t*>(smem);
  static_assert((size_t)(HT * 5 + 20 + 20 + 8) * 64 * 16 <= f32_narrow_lds(HT), "a wave's sums");
  for (int w = 1; w < kF32Waves; ++w) {
    __syncthreads();
    int o = 0;
    if (wave == w) {
      f32_wave_put(buf, o, lane, w3, b3);
      f32_wave_put(buf, o, lane, w2, b2);
      f32_wave_put(buf, o, lane, w1, b1);
      f32_wave_put(buf, o, lane, w0, b0);
    }
    __syncthreads();
    if (wave == 0) {
      f32_wave_add(buf, o, lane, w3, b3);
      f32_wave_add(buf, o, lane, w2, b2);
      f32_wave_add(buf, o, lane, w1, b1);
      f32_wave_add(buf, o, lane, w0, b0);
    }
  }
  if (wave == 0) {
    f32_narrow_part(a, 3, lane, w3, b3);
    f32_narrow_part(a, 2, lane, w2, b2);
    f32_narrow_part(a, 1, lane, w1, b1);
    f32_narrow_part(a, 0, lane, w0, b0);
  }
}
