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
template <int H, int Q, bool SELU>
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
        r[v] = SELU ? selu_f(z) : (z < 0.0f ? 0.0f : z);  // ReLU that keeps NaN
      }
      if (valid) *reinterpret_cast<f32x4_t*>(store + 16 * t + 4 * g) = r;
      out[t] = f32_natural(r);
    }
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

template <int H, int KQ, bool SELU>
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
  f32_fwd_layer<H, KQ, SELU>(a, x0, in, bias_s + a.bias_off[0], a.h[0] + pc * H, valid, smem, c, tid, lane);
  for (int layer = 1; layer < a.n_layers - 1; ++layer) {
    f32_fwd_layer<H, Q, SELU>(a, in, out, bias_s + a.bias_off[layer], a.h[layer] + pc * H, valid, smem, c, tid, lane);
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
template <int H, int QI, bool SELU>
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
        r[v] = SELU ? acc[u][v] * selu_grad_of_out(hv[u][v]) : (hv[u][v] > 0.0f ? acc[u][v] : 0.0f);
      if (valid) *reinterpret_cast<f32x4_t*>(store + 16 * t + 4 * g) = r;
      out[t] = r;
    }
    fwait_dma();
    __syncthreads();
    ++c;
  }
}

template <int H, int KQ, bool SELU>
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
    f32_bwd_layer<H, kF32HeadTiles, SELU>(a, head, a.head_tiles, out, a.h[layer] + pc * H, a.dh[layer] + pc * H, valid, smem, c,
                                          tid, lane);
  }
  for (--layer; layer >= 0; --layer) {
    f32x4_t in[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) in[q] = out[q];
    f32_bwd_layer<H, Q, SELU>(a, in, Q, out, a.h[layer] + pc * H, a.dh[layer] + pc * H, valid, smem, c, tid, lane);
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
