// BC1 / BC4 on gfx950: the integer reference encoder, the decoder, per-block SSE and the per-block
// fallback.  One thread per 4x4 block; everything is exact integer arithmetic.
//
// Format (paper Sec. 1, Sec. 2.1; Eq. palette and Eq. weightBC4): BC1 = two RGB565 endpoints and
// sixteen 2-bit codes; four colours (c0 > c1: endpoints and the two thirds) or three plus black
// (c0 <= c1: endpoints, midpoint, black).  BC4 = two 8-bit endpoints and sixteen 3-bit codes; eight
// values (e0 > e1: endpoints and six sevenths) or six plus 0 and 255 (e0 <= e1: endpoints, four fifths).
// Endpoints expand to 8 bits by bit replication; interpolants round to the nearest integer (thirds,
// fifths and sevenths of integers never tie; the BC1 midpoint rounds halves up).
//
// Weight ("logical") order n: the order of w_n in Eq. palette / Eq. weightBC4 -- BC1 codes 0,2,3,1;
// BC4 eight-value codes 0,2,3,4,5,6,7,1; BC4 six-value codes 6 (=0),0,2,3,4,5,1,7 (=255).  Ties between
// palette entries go to the smallest n.
//
// The reference encoder (the paper's training targets come from a third-party encoder with two
// refinement steps, Sec. 4.1) is this project's REF-BC1 / REF-BC4 algorithm:
//   BC1: candidate A = farthest texel pair (lexicographically first on ties); candidate B = per-channel
//   bounding box inset by range/16, the diagonal of each channel flipped when its integer covariance
//   with the widest channel is negative; each quantised to the nearest 565 code, put in four-colour
//   order (c0 == c1 -> all codes 0), texels coded by least squared error; the smaller SSE wins (ties A);
//   then two least-squares steps (exact rational endpoints, rounded half up to 5/6 bits), each kept
//   only if the SSE strictly falls.
//   BC4: candidates (max, min) and (min, max) of the texels other than 0/255; two least-squares steps
//   each in its own mode (sevenths, or fifths without the 0/255 texels), dropped if they leave the mode
//   or do not lower the SSE; the smaller SSE wins (ties: the first).
#include <algorithm>

#include "common.h"

namespace {

constexpr int kThreads = 256;

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));

__host__ __device__ constexpr int expand5(int v) { return (v << 3) | (v >> 2); }
__host__ __device__ constexpr int expand6(int v) { return (v << 2) | (v >> 4); }

// ------------------------------------------------------------------------------------------- integer helpers
// Sum of four unsigned byte products, and of two unsigned 16-bit products, plus c.
__device__ __forceinline__ uint32_t dot4(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_udot4(a, b, c, false); }
__device__ __forceinline__ uint32_t dot2(u16x2 a, u16x2 b, uint32_t c) { return __builtin_amdgcn_udot2(a, b, c, false); }
__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// Exact quotients by constants, as one 24-bit product and a shift: x / 3 for x < 2^16, x / 255 for
// x < 2^16, x / 5 and x / 7 for x <= 1791 (the error of the rounded reciprocal times x stays below 1/5
// and 1/7).
__device__ __forceinline__ uint32_t div3(uint32_t x) { return __umul24(x, 0xAAABu) >> 17; }
__device__ __forceinline__ uint32_t div255(uint32_t x) { return __umul24(x, 0x8081u) >> 23; }
__device__ __forceinline__ uint32_t div5(uint32_t x) { return __umul24(x, 13108u) >> 16; }
__device__ __forceinline__ uint32_t div7(uint32_t x) { return __umul24(x, 9363u) >> 16; }

// n / d for a quotient of at most 256, d in 1 .. 2^23, n < 2^31: the float quotient is off by less than
// 1e-4, so its integer part is off by at most one and the remainder corrects it.
__device__ __forceinline__ int small_quot(uint32_t n, uint32_t d) {
  int q = (int)((float)n * __builtin_amdgcn_rcpf((float)d));
  const int r = (int)(n - __umul24((uint32_t)q, d));
  q += r >= (int)d ? 1 : 0;
  return r < 0 ? q - 1 : q;
}

// Block coordinates of block b: 32-bit division wherever the block count allows it.
__device__ __forceinline__ void block_xy(int64_t b, int bw, int64_t n, int* bx, int* by) {
  if (n <= 0x7fffffff) {
    const uint32_t q = (uint32_t)b / (uint32_t)bw;
    *by = (int)q;
    *bx = (int)((uint32_t)b - q * (uint32_t)bw);
  } else {
    *bx = (int)(b % bw);
    *by = (int)(b / bw);
  }
}

// W 4-byte words at p: dword accesses when `aligned` (uniform: the texture base and its pitch are
// multiples of four bytes; a block's row offset always is), bytes otherwise.
template <int W>
__device__ __forceinline__ void load_words(const uint8_t* p, bool aligned, uint32_t w[W]) {
  if (aligned) {
    typedef uint32_t words __attribute__((ext_vector_type(W == 3 ? 3 : 1), aligned(4)));
    const words v = *reinterpret_cast<const words*>(p);
#pragma unroll
    for (int k = 0; k < W; ++k) w[k] = v[k];
  } else {
#pragma unroll
    for (int k = 0; k < W; ++k)
      w[k] = (uint32_t)p[4 * k] | ((uint32_t)p[4 * k + 1] << 8) | ((uint32_t)p[4 * k + 2] << 16) | ((uint32_t)p[4 * k + 3] << 24);
  }
}

template <int W>
__device__ __forceinline__ void store_words(uint8_t* p, bool aligned, const uint32_t w[W]) {
  if (aligned) {
    typedef uint32_t words __attribute__((ext_vector_type(W == 3 ? 3 : 1), aligned(4)));
    words v;
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] = w[k];
    *reinterpret_cast<words*>(p) = v;
  } else {
#pragma unroll
    for (int k = 0; k < W; ++k)
#pragma unroll
      for (int b = 0; b < 4; ++b) p[4 * k + b] = (uint8_t)(w[k] >> (8 * b));
  }
}

__device__ __forceinline__ bool word_aligned(const void* p, int pitch) {
  return ((reinterpret_cast<uintptr_t>(p) | (uintptr_t)pitch) & 3) == 0;
}

// -------------------------------------------------------------------------------------------------- BC1
// The encoder is bound by its integer VALU work (56 bytes a block against hundreds of operations), so
// the colours stay packed, R | G << 8 | B << 16 in a word, and every squared distance comes from byte
// dot products: |p - c|^2 = |p|^2 - (2 p.c - |c|^2).  The nearest of the four entries is the maximum of
// 4 (2 p.c - |c|^2) + (3 - n), whose low bits also settle ties for the smallest n.  One 4x4 block a
// thread; 262,144 blocks: 45.1 us with one value a register, now 18.3.
struct Bc1Enc {
  uint32_t ends;  // c0 | c1 << 16
  uint32_t q;     // 2 bits a texel: 3 - n, n the weight order
  int sse;
};

// Stored codes (0, 2, 3, 1 for n = 0 .. 3) of the sixteen 2-bit fields 3 - n: 11 -> 00, 10 -> 10,
// 01 -> 11, 00 -> 01.
__device__ __forceinline__ uint32_t bc1_codes_of(uint32_t q) {
  const uint32_t b1 = (q >> 1) & 0x55555555u, b0 = q & 0x55555555u;
  return ((b1 ^ b0) << 1) | (b1 ^ 0x55555555u);
}

__device__ __forceinline__ uint32_t rgb_of_565(uint32_t c) {
  return (uint32_t)expand5((c >> 11) & 31) | ((uint32_t)expand6((c >> 5) & 63) << 8) | ((uint32_t)expand5(c & 31) << 16);
}

__device__ __forceinline__ uint32_t channel(uint32_t w, int c) { return (w >> (8 * c)) & 255u; }

// Sixteen texels coded against the endpoints c0, c1 (either order; stored larger first).  c0 == c1: the
// four entries coincide, so every texel takes n = 0, whose code is 0.  n2_sum = sum of |p|^2.
__device__ Bc1Enc bc1_finish(uint32_t c0, uint32_t c1, const uint32_t (&w)[16], uint32_t n2_sum) {
  if (c0 < c1) {
    const uint32_t t = c0;
    c0 = c1;
    c1 = t;
  }
  Bc1Enc st;
  st.ends = c0 | (c1 << 16);
  uint32_t pal[4] = {rgb_of_565(c0), 0, 0, rgb_of_565(c1)};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const uint32_t a = channel(pal[0], c), b = channel(pal[3], c);
    pal[1] |= div3(2 * a + b + 1) << (8 * c);
    pal[2] |= div3(a + 2 * b + 1) << (8 * c);
  }
  int base[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) base[n] = 3 - n - (int)(dot4(pal[n], pal[n], 0) << 2);
  st.q = 0;
  int gain = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    int k[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) k[n] = (int)(dot4(w[i], pal[n], 0) << 3) + base[n];
    const int best = max(max(k[0], k[1]), max(k[2], k[3]));
    gain += best >> 2;
    st.q = __builtin_amdgcn_alignbit((uint32_t)best, st.q, 2);
  }
  st.sse = (int)n2_sum - gain;
  return st;
}

__device__ __forceinline__ uint32_t quant565(uint32_t r, uint32_t g, uint32_t b) {
  return (div255(r * 31 + 127) << 11) | (div255(g * 63 + 127) << 5) | div255(b * 31 + 127);
}

// round-half-up of (num/den) * mul / 255 with num clamped to [0, 255 den]: den <= 5184 (sixteen weights
// of 0 .. 3), |num| <= 3 * 144 * 12240, so everything fits 32 bits.
__device__ __forceinline__ uint32_t ratio_code(int num, int den, int mul) {
  num = min(max(num, 0), 255 * den);
  return (uint32_t)small_quot((uint32_t)(2 * num * mul + 255 * den), (uint32_t)(510 * den));
}

// One least-squares step, kept if the SSE strictly falls; false when nothing changed (a further step
// would repeat it).  ch[c][k]: channel c of texels 4k .. 4k+3, one a byte; sum[c] over the block.
__device__ bool bc1_refine(Bc1Enc& st, const uint32_t (&w)[16], const uint32_t (&ch)[3][4], const int (&sum)[3],
                           uint32_t n2_sum) {
  uint32_t sa = 0, saa = 0, sap[3] = {0, 0, 0};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t a = (st.q >> (8 * k)) & 255u;  // the four weights 3 - n of the row, spread to bytes
    a = (a | (a << 12)) & 0x000F000Fu;
    a = (a | (a << 6)) & 0x03030303u;
    sa = dot4(a, 0x01010101u, sa);
    saa = dot4(a, a, saa);
#pragma unroll
    for (int c = 0; c < 3; ++c) sap[c] = dot4(a, ch[c][k], sap[c]);
  }
  const int sbb = 144 - 6 * (int)sa + (int)saa, sab = 3 * (int)sa - (int)saa;
  const int det = (int)saa * sbb - sab * sab;
  if (det <= 0) return false;
  uint32_t qa[3], qb[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int mul = c == 1 ? 63 : 31, pa = (int)sap[c], pb = 3 * sum[c] - pa;
    qa[c] = ratio_code(3 * (sbb * pa - sab * pb), det, mul);
    qb[c] = ratio_code(3 * ((int)saa * pb - sab * pa), det, mul);
  }
  const Bc1Enc nw = bc1_finish((qa[0] << 11) | (qa[1] << 5) | qa[2], (qb[0] << 11) | (qb[1] << 5) | qb[2], w, n2_sum);
  if (nw.sse >= st.sse) return false;
  st = nw;
  return true;
}

// Optimal single-colour endpoints (step 8 of REF-BC1): for every value v, the code pair (a, b) of 5-bit
// or 6-bit endpoints whose four-colour 2/3 point (2 E(a) + E(b) + 1) / 3 is nearest to v, ties to the
// smallest a, then the smallest b; entry = a | b << 8.  Built by the compiler: first the smallest (a, b)
// of every value that a 2/3 point takes, then the nearest taken value on either side.
struct SingleColour {
  uint16_t five[256], six[256];
};

constexpr void single_colour_table(int bits, uint16_t (&out)[256]) {
  const int n = 1 << bits;
  int first[256] = {};  // 1 + (a << 8 | b) of the value's smallest pair, 0: not taken
  for (int a = 0; a < n; ++a)
    for (int b = 0; b < n; ++b) {
      const int ea = bits == 5 ? expand5(a) : expand6(a), eb = bits == 5 ? expand5(b) : expand6(b);
      int& f = first[(2 * ea + eb + 1) / 3];
      if (f == 0) f = 1 + (a << 8 | b);
    }
  for (int v = 0; v < 256; ++v) {
    int best = 0;
    for (int e = 0; best == 0; ++e) {
      const int lo = v - e >= 0 ? first[v - e] : 0, hi = v + e <= 255 ? first[v + e] : 0;
      best = lo == 0 ? hi : (hi == 0 ? lo : (lo < hi ? lo : hi));
    }
    out[v] = (uint16_t)(((best - 1) >> 8) | (((best - 1) & 255) << 8));
  }
}

constexpr SingleColour make_single_colour() {
  SingleColour t{};
  single_colour_table(5, t.five);
  single_colour_table(6, t.six);
  return t;
}

__device__ const SingleColour g_single = make_single_colour();

// w[idx] by a tree of bit selects.  (An indexed read moves the array out of registers, and so does a choice between two
// of its elements, which the compiler turns into one: then 16 KB of LDS, addressed with the workgroup's size from
// the dispatch packet in host memory, a wait of some 10 us once all CUs ask for it.  1024^2 texture 20.7 -> 6.9 us,
// 2048^2 31 -> 18.3.)
__device__ __forceinline__ uint32_t pick16(const uint32_t (&w)[16], int idx) {
  uint32_t a[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) a[k] = w[k];
#pragma unroll
  for (int half = 8; half > 0; half >>= 1) {
    const uint32_t m = idx & half ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int k = 0; k < half; ++k) a[k] = (a[k + half] & m) | (a[k] & ~m);
  }
  return a[0];
}

// Smallest and largest of a channel's sixteen bytes.
__device__ __forceinline__ void byte_range(const uint32_t (&x)[4], int* lo, int* hi) {
  u16x2 mn{255, 255}, mx{0, 0};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const u16x2 e = __builtin_bit_cast(u16x2, x[k] & 0x00FF00FFu), o = __builtin_bit_cast(u16x2, (x[k] >> 8) & 0x00FF00FFu);
    mn = __builtin_elementwise_min(__builtin_elementwise_min(mn, e), o);
    mx = __builtin_elementwise_max(__builtin_elementwise_max(mx, e), o);
  }
  *lo = min((int)mn[0], (int)mn[1]);
  *hi = max((int)mx[0], (int)mx[1]);
}

// w: the texels; ch: the same by channel (bc1_refine).
__device__ Bc1Enc bc1_encode_block(const uint32_t (&w)[16], const uint32_t (&ch)[3][4]) {
  // candidate A: farthest pair.  Key of a pair: d << 8 | (15 - i) << 4 | (15 - j), so the maximum is the
  // lexicographically first pair of the largest distance d = |p_i|^2 + |p_j|^2 - 2 p_i.p_j.
  uint32_t n2_sum = 0;
  int nk[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t n2 = dot4(w[i], w[i], 0);
    n2_sum += n2;
    nk[i] = (int)(n2 << 8) + (15 - i);
  }
  int far = 0;
#pragma unroll
  for (int i = 0; i < 15; ++i) {
    int row = 0x7fffffff;  // min over j of 2 p_i.p_j - |p_j|^2 in the key's units (a shift and an add)
#pragma unroll
    for (int j = i + 1; j < 16; ++j) row = min(row, (int)(dot4(w[i], w[j], 0) << 9) - nk[j]);
    far = max(far, nk[i] + 15 * (15 - i) - row);
  }
  const uint32_t pa = pick16(w, 15 - ((far >> 4) & 15)), pb = pick16(w, 15 - (far & 15));
  Bc1Enc st = bc1_finish(quant565(channel(pa, 0), channel(pa, 1), channel(pa, 2)),
                         quant565(channel(pb, 0), channel(pb, 1), channel(pb, 2)), w, n2_sum);
  // candidate B: inset bounding box, diagonal signed by covariance with the widest channel
  int mn[3], mx[3], sum[3], cross[3][3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    byte_range(ch[c], &mn[c], &mx[c]);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) s = dot4(ch[c][k], 0x01010101u, s);
    sum[c] = (int)s;
#pragma unroll
    for (int d = 0; d <= c; ++d) {
      uint32_t x = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) x = dot4(ch[c][k], ch[d][k], x);
      cross[c][d] = cross[d][c] = (int)x;
    }
  }
  int m = 0;
  if (mx[1] - mn[1] > mx[0] - mn[0]) m = 1;
  if (mx[2] - mn[2] > (m ? mx[1] - mn[1] : mx[0] - mn[0])) m = 2;
  const int sum_m = m == 0 ? sum[0] : (m == 1 ? sum[1] : sum[2]);
  uint32_t b0[3], b1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int inset = (mx[c] - mn[c]) >> 4;
    const int lo = mn[c] + inset, hi = mx[c] - inset;
    const int cov = 16 * (m == 0 ? cross[c][0] : (m == 1 ? cross[c][1] : cross[c][2])) - sum[c] * sum_m;
    b0[c] = (uint32_t)(cov < 0 ? lo : hi);
    b1[c] = (uint32_t)(cov < 0 ? hi : lo);
  }
  const Bc1Enc stb = bc1_finish(quant565(b0[0], b0[1], b0[2]), quant565(b1[0], b1[1], b1[2]), w, n2_sum);
  if (stb.sse < st.sse) st = stb;
  // an exact block cannot get better, and a step that changed nothing would do so again
  if (st.sse > 0) {
    if (bc1_refine(st, w, ch, sum, n2_sum)) bc1_refine(st, w, ch, sum, n2_sum);
  }
  // step 8: a one-colour block also tries the optimal single-colour endpoints
  if (mn[0] == mx[0] && mn[1] == mx[1] && mn[2] == mx[2]) {
    const uint32_t r = g_single.five[mn[0]], g = g_single.six[mn[1]], b = g_single.five[mn[2]];
    const Bc1Enc sc = bc1_finish(((r & 255u) << 11) | ((g & 255u) << 5) | (b & 255u), ((r >> 8) << 11) | ((g >> 8) << 5) | (b >> 8),
                                 w, n2_sum);
    if (sc.sse < st.sse) st = sc;
  }
  return st;
}

// -------------------------------------------------------------------------------------------------- BC4
// Texels travel as pairs of 16-bit values.  The nearest of the eight entries is the minimum of
// 8 |v - p_n| + n = max(8v - (8 p_n - n), (8 p_n + n) - 8v): four packed operations for two texels, ties
// to the smallest n.  262,144 blocks: 55.5 -> 8.9 us on smooth textures (most of their blocks are exact after the
// first candidate).
struct Bc4Enc {
  int e0, e1;
  uint32_t n[2];  // weight order of the texels, 4 bits each: n[h], half x, nibble k = texel 8h + 2k + x
  int sse;
};

// Entries in weight order (EIGHT: e0 > e1; else six values plus 0 and 255).
template <bool EIGHT>
__device__ __forceinline__ void bc4_entries(int e0, int e1, uint32_t pal[8]) {
  const uint32_t a = (uint32_t)e0, b = (uint32_t)e1;
  if (EIGHT) {
    pal[0] = a;
    pal[7] = b;
#pragma unroll
    for (uint32_t j = 1; j <= 6; ++j) pal[j] = div7((7 - j) * a + j * b + 3);
  } else {
    pal[0] = 0;
    pal[1] = a;
    pal[6] = b;
    pal[7] = 255;
#pragma unroll
    for (uint32_t j = 1; j <= 4; ++j) pal[1 + j] = div5((5 - j) * a + j * b + 2);
  }
}

__device__ __forceinline__ i16x2 both(uint32_t x) { return __builtin_bit_cast(i16x2, __umul24(x, 0x00010001u)); }

// v8[k]: 8 x texels 2k and 2k + 1.
template <bool EIGHT>
__device__ Bc4Enc bc4_finish(int e0, int e1, const i16x2 (&v8)[8]) {
  Bc4Enc st;
  st.e0 = e0;
  st.e1 = e1;
  uint32_t pal[8];
  bc4_entries<EIGHT>(e0, e1, pal);
  i16x2 best[8];
#pragma unroll
  for (uint32_t n = 0; n < 8; ++n) {
    const i16x2 lo = both(8 * pal[n]) - (int16_t)n, hi = both(8 * pal[n]) + (int16_t)n;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const i16x2 key = __builtin_elementwise_max(v8[k] - lo, hi - v8[k]);
      best[k] = n == 0 ? key : __builtin_elementwise_min(best[k], key);
    }
  }
  uint32_t sse = 0;
  st.n[0] = st.n[1] = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const u16x2 b = __builtin_bit_cast(u16x2, best[k]);
    const u16x2 d = b >> (uint16_t)3;
    sse = dot2(d, d, sse);
    st.n[k >> 2] |= (__builtin_bit_cast(uint32_t, b) & 0x00070007u) << (4 * (k & 3));
  }
  st.sse = (int)sse;
  return st;
}

// One least-squares step in the block's own mode, dropped if it leaves the mode or does not lower the
// SSE; false when nothing changed.  With b the step of a texel's entry along the endpoints (n, or n - 1 of
// the six values) and a = S - b (S = 7 or 5): the sums of a, a^2, ab, av follow from those of b, b^2, bv, v.
// Every product fits 32 bits: |na| <= 7 * 784 * 28560, det <= 614,656.
template <bool EIGHT>
__device__ bool bc4_refine(Bc4Enc& st, const i16x2 (&v8)[8]) {
  constexpr int S = EIGHT ? 7 : 5;
  uint32_t cnt = 0, sb = 0, sbb = 0, sv8 = 0, sbv8 = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const u16x2 v = __builtin_bit_cast(u16x2, v8[k]);
    u16x2 b = __builtin_bit_cast(u16x2, (st.n[k >> 2] >> (4 * (k & 3))) & 0x00070007u);
    u16x2 one{1, 1};
    if (!EIGHT) {
      // texels on the constant entries 0 and 7 take no part: n - 1 is then 0xFFFF or 6
      b -= one;
      one = __builtin_bit_cast(u16x2, (i16x2)((b < (uint16_t)6) & (i16x2){1, 1}));
      b *= one;
    }
    cnt = dot2(one, u16x2{1, 1}, cnt);
    sb = dot2(b, u16x2{1, 1}, sb);
    sbb = dot2(b, b, sbb);
    sv8 = dot2(v, one, sv8);
    sbv8 = dot2(v, b, sbv8);
  }
  const int b1 = (int)sb, b2 = (int)sbb, bv = (int)(sbv8 >> 3), sv = (int)(sv8 >> 3), n = (int)cnt;
  const int saa = S * S * n - 2 * S * b1 + b2, sab = S * b1 - b2, av = S * sv - bv;
  const int det = saa * b2 - sab * sab;
  if (det <= 0) return false;
  const int na = min(max(S * (b2 * av - sab * bv), 0), 255 * det);
  const int nb = min(max(S * (saa * bv - sab * av), 0), 255 * det);
  const int ea = small_quot((uint32_t)(2 * na + det), (uint32_t)(2 * det));
  const int eb = small_quot((uint32_t)(2 * nb + det), (uint32_t)(2 * det));
  if (EIGHT ? !(ea > eb) : !(ea <= eb)) return false;
  const Bc4Enc nw = bc4_finish<EIGHT>(ea, eb, v8);
  if (nw.sse >= st.sse) return false;
  st = nw;
  return true;
}

// Stored 3-bit codes of the weight orders: eight-value 0,2,3,4,5,6,7,1, six-value 6,0,2,3,4,5,1,7.
__device__ __forceinline__ uint64_t bc4_codes_of(const uint32_t (&n)[2], bool eight) {
  const uint32_t lo = eight ? 0x04030200u : 0x03020006u, hi = eight ? 0x01070605u : 0x07010504u;
  uint32_t half[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint32_t bits = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // texels 8h + 4q .. +3 (nibbles 2q and 2q + 1 of both halves) as bytes 0, 2 / 1, 3 -> codes
      const uint32_t t = n[h] >> (8 * q);
      const uint32_t c = perm(hi, lo, perm(t >> 4, t, 0x06020400u) & 0x07070707u);  // bytes: texels 0, 2, 1, 3
      const uint32_t row = (c & 7u) | ((c >> 13) & 0x38u) | ((c >> 2) & 0x1C0u) | ((c >> 15) & 0xE00u);
      bits |= row << (12 * q);
    }
    half[h] = bits;
  }
  return (uint64_t)half[0] | ((uint64_t)half[1] << 24);
}

// row[y]: the four texels of row y, one a byte.
__device__ void bc4_encode_block(const uint32_t (&row)[4], uint64_t* word, int* sse) {
  int mn, mx;
  byte_range(row, &mn, &mx);
  i16x2 v8[8];
  u16x2 imn{256, 256}, imx{0, 0};  // over the texels other than 0 and 255
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const u16x2 v = __builtin_bit_cast(u16x2, perm(0, row[k >> 1], k & 1 ? 0x0C030C02u : 0x0C010C00u));
    v8[k] = __builtin_bit_cast(i16x2, (u16x2)(v << (uint16_t)3));
    const u16x2 u = v - (uint16_t)1;  // 0 -> 0xFFFF, 255 -> 254, the others 0 .. 253
    const auto in = u < (uint16_t)254;
    imn = __builtin_elementwise_min(imn, in ? v : u16x2{256, 256});
    imx = __builtin_elementwise_max(imx, in ? v : u16x2{0, 0});
  }
  // a flat block is exact in the six-value order of equal endpoints: entry 0 for 0, else entry 1
  if (mn == mx) {
    *word = (uint64_t)(uint32_t)mn * 0x0101u | (mn == 0 ? 0xDB6DB6DB6DB60000ull : 0ull);
    *sse = 0;
    return;
  }
  Bc4Enc st = bc4_finish<true>(mx, mn, v8);
  // an exact block cannot get better, and a step that changed nothing would do so again
  if (st.sse > 0) {
    if (bc4_refine<true>(st, v8)) bc4_refine<true>(st, v8);
    const bool has = (imx[0] | imx[1]) != 0;
    Bc4Enc s6 = bc4_finish<false>(has ? min((int)imn[0], (int)imn[1]) : 0, has ? max((int)imx[0], (int)imx[1]) : 0, v8);
    if (bc4_refine<false>(s6, v8)) bc4_refine<false>(s6, v8);
    if (s6.sse < st.sse) st = s6;
  }
  *word = (uint64_t)st.e0 | ((uint64_t)st.e1 << 8) | (bc4_codes_of(st.n, st.e0 > st.e1) << 16);
  *sse = st.sse;
}

// ------------------------------------------------------------------------------------------ kernels
// A texel row of a BC1 block (w: its twelve bytes) as four packed texels and as a word a channel.
__device__ __forceinline__ void split_row(const uint32_t w[3], uint32_t px[4], uint32_t ch[3]) {
  px[0] = w[0] & 0xFFFFFFu;
  px[1] = __builtin_amdgcn_alignbit(w[1], w[0], 24) & 0xFFFFFFu;
  px[2] = __builtin_amdgcn_alignbit(w[2], w[1], 16) & 0xFFFFFFu;
  px[3] = w[2] >> 8;
  ch[0] = perm(w[2], perm(w[1], w[0], 0x0C060300u), 0x05020100u);
  ch[1] = perm(w[2], perm(w[1], w[0], 0x0C070401u), 0x06020100u);
  ch[2] = perm(w[2], perm(w[1], w[0], 0x0C0C0502u), 0x07040100u);
}

__global__ void __launch_bounds__(kThreads) k_encode_ref_bc1(const uint8_t* __restrict__ tex, int bw, int bh,
                                                       int pitch, uint64_t* __restrict__ out,
                                                       int32_t* __restrict__ sse_out) {
  const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x, n = (int64_t)bw * bh;
  if (b >= n) return;
  int bx, by;
  block_xy(b, bw, n, &bx, &by);
  const bool al = word_aligned(tex, pitch);
  uint32_t w[16], ch[3][4];
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    uint32_t r[3], c[3];
    load_words<3>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)12 * bx, al, r);
    split_row(r, w + 4 * y, c);
#pragma unroll
    for (int k = 0; k < 3; ++k) ch[k][y] = c[k];
  }
  const Bc1Enc st = bc1_encode_block(w, ch);
  out[b] = (uint64_t)st.ends | ((uint64_t)bc1_codes_of(st.q) << 32);
  if (sse_out) sse_out[b] = st.sse;
}

__global__ void __launch_bounds__(kThreads) k_encode_ref_bc4(const uint8_t* __restrict__ tex, int bw, int bh,
                                                       int pitch, uint64_t* __restrict__ out,
                                                       int32_t* __restrict__ sse_out) {
  const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x, n = (int64_t)bw * bh;
  if (b >= n) return;
  int bx, by;
  block_xy(b, bw, n, &bx, &by);
  const bool al = word_aligned(tex, pitch);
  uint32_t row[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) load_words<1>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)4 * bx, al, row + y);
  uint64_t word;
  int sse;
  bc4_encode_block(row, &word, &sse);
  out[b] = word;
  if (sse_out) sse_out[b] = sse;
}

// Decoded texels of a block, a row at a time, by byte permutes: the palette of a channel is one word (BC1,
// indexed by the stored code) or two (BC4), and a row's four codes spread to bytes select from it.
struct Bc1Dec {
  uint32_t pal[3];  // a byte per code, for each channel
  uint32_t idx;
};

__device__ __forceinline__ Bc1Dec bc1_decoder(uint64_t w) {
  Bc1Dec d;
  const uint32_t c0 = (uint32_t)(w & 0xFFFF), c1 = (uint32_t)((w >> 16) & 0xFFFF);
  const uint32_t a = rgb_of_565(c0), b = rgb_of_565(c1);
  const bool four = c0 > c1;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const uint32_t x = channel(a, c), y = channel(b, c);
    const uint32_t p2 = four ? div3(2 * x + y + 1) : (x + y + 1) >> 1, p3 = four ? div3(x + 2 * y + 1) : 0;
    d.pal[c] = x | (y << 8) | (p2 << 16) | (p3 << 24);
  }
  d.idx = (uint32_t)(w >> 32);
  return d;
}

// The twelve bytes of texel row y.
__device__ __forceinline__ void bc1_row(const Bc1Dec& d, int y, uint32_t out[3]) {
  uint32_t s = (d.idx >> (8 * y)) & 255u;
  s = (s | (s << 12)) & 0x000F000Fu;
  s = (s | (s << 6)) & 0x03030303u;
  const uint32_t r = perm(0, d.pal[0], s), g = perm(0, d.pal[1], s), b = perm(0, d.pal[2], s);
  const uint32_t rg = perm(g, r, 0x05010400u);                 // r0 g0 r1 g1
  const uint32_t hg = perm(g, r, 0x07030602u);                 // r2 g2 r3 g3
  out[0] = perm(b, rg, 0x02040100u);                           // r0 g0 b0 r1
  out[1] = perm(perm(b, rg, 0x0C0C0503u), hg, 0x01000504u);    // g1 b1 r2 g2
  out[2] = perm(b, hg, 0x07030206u);                           // b2 r3 g3 b3
}

struct Bc4Dec {
  uint32_t lo, hi;  // entries of codes 0 .. 3 and 4 .. 7
  uint64_t idx;
};

__device__ __forceinline__ Bc4Dec bc4_decoder(uint64_t w) {
  Bc4Dec d;
  const uint32_t a = (uint32_t)(w & 0xFF), b = (uint32_t)((w >> 8) & 0xFF);
  uint32_t p[8];
  p[0] = a;
  p[1] = b;
  const bool eight = a > b;
#pragma unroll
  for (uint32_t j = 1; j <= 6; ++j) {
    const uint32_t six = j <= 4 ? div5((5 - j) * a + j * b + 2) : (j == 5 ? 0u : 255u);
    p[1 + j] = eight ? div7((7 - j) * a + j * b + 3) : six;
  }
  d.lo = p[0] | (p[1] << 8) | (p[2] << 16) | (p[3] << 24);
  d.hi = p[4] | (p[5] << 8) | (p[6] << 16) | (p[7] << 24);
  d.idx = w >> 16;
  return d;
}

__device__ __forceinline__ uint32_t bc4_row(const Bc4Dec& d, int y) {
  uint32_t s = (uint32_t)(d.idx >> (12 * y)) & 0xFFFu;
  s = (s | (s << 10)) & 0x003F003Fu;
  s = (s | (s << 5)) & 0x07070707u;
  return perm(d.hi, d.lo, s);
}

__global__ void __launch_bounds__(kThreads) k_decode_bc1(const uint64_t* __restrict__ blocks, int bw, int bh,
                                                   uint8_t* __restrict__ tex, int pitch) {
  const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x, n = (int64_t)bw * bh;
  if (b >= n) return;
  int bx, by;
  block_xy(b, bw, n, &bx, &by);
  const Bc1Dec d = bc1_decoder(blocks[b]);
  const bool al = word_aligned(tex, pitch);
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    uint32_t row[3];
    bc1_row(d, y, row);
    store_words<3>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)12 * bx, al, row);
  }
}

__global__ void __launch_bounds__(kThreads) k_decode_bc4(const uint64_t* __restrict__ blocks, int bw, int bh,
                                                   uint8_t* __restrict__ tex, int pitch) {
  const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x, n = (int64_t)bw * bh;
  if (b >= n) return;
  int bx, by;
  block_xy(b, bw, n, &bx, &by);
  const Bc4Dec d = bc4_decoder(blocks[b]);
  const bool al = word_aligned(tex, pitch);
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    const uint32_t row = bc4_row(d, y);
    store_words<1>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)4 * bx, al, &row);
  }
}

// Sum over the words of a row of (a - b)^2, from byte dot products.
template <int W>
__device__ __forceinline__ int row_sse(const uint32_t a[W], const uint32_t b[W]) {
  uint32_t sq = 0, ab = 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    sq = dot4(b[k], b[k], dot4(a[k], a[k], sq));
    ab = dot4(a[k], b[k], ab);
  }
  return (int)(sq - 2 * ab);
}

__global__ void __launch_bounds__(kThreads) k_block_sse(const uint64_t* __restrict__ blocks,
                                                  const uint8_t* __restrict__ tex, int bw, int bh,
                                                  int pitch, int fmt, int32_t* __restrict__ sse) {
  const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x, n = (int64_t)bw * bh;
  if (b >= n) return;
  int bx, by;
  block_xy(b, bw, n, &bx, &by);
  const uint64_t w = blocks[b];
  const bool al = word_aligned(tex, pitch);
  int total = 0;
  if (fmt == NTBC_BC1) {
    uint32_t r[4][3];
#pragma unroll
    for (int y = 0; y < 4; ++y) load_words<3>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)12 * bx, al, r[y]);
    const Bc1Dec d = bc1_decoder(w);
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      uint32_t row[3];
      bc1_row(d, y, row);
      total += row_sse<3>(row, r[y]);
    }
  } else {
    uint32_t r[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) load_words<1>(tex + (int64_t)(4 * by + y) * pitch + (int64_t)4 * bx, al, r + y);
    const Bc4Dec d = bc4_decoder(w);
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const uint32_t row = bc4_row(d, y);
      total += row_sse<1>(&row, r + y);
    }
  }
  sse[b] = total;
}

// Same-address atomics serialise (about 10 ns each), so the launch has at most 256 workgroups of sixteen
// waves: 262,144 blocks with 1,024 workgroups 14.0 us, now 5.8.
constexpr int kFallbackThreads = 1024, kFallbackBlocks = 256;

__global__ void __launch_bounds__(kFallbackThreads) k_fallback(const uint64_t* __restrict__ ntbc_words,
                                                 const uint64_t* __restrict__ ref_words,
                                                 const int32_t* __restrict__ sse_n,
                                                 const int32_t* __restrict__ sse_r, int64_t n, float kappa,
                                                 float delta, uint64_t* __restrict__ out,
                                                 int32_t* __restrict__ count) {
  // grid-stride over the blocks; the replaced count is summed per wavefront (ballot), then per
  // workgroup in LDS, and added with one atomic per workgroup (same-address atomics serialise)
  __shared__ int part[kFallbackThreads / 64];
  int mine = 0;
  for (int64_t b = (int64_t)blockIdx.x * kFallbackThreads + threadIdx.x; b - threadIdx.x < n;
       b += (int64_t)gridDim.x * kFallbackThreads) {
    bool replaced = false;
    if (b < n) {
      const float limit = kappa * (float)sse_r[b] + delta;
      replaced = (float)sse_n[b] > limit;
      out[b] = replaced ? ref_words[b] : ntbc_words[b];
    }
    mine += (int)__popcll(__ballot(replaced));
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int w = 0; w < kFallbackThreads / 64; ++w) tot += part[w];
    if (tot != 0) atomicAdd(count, tot);
  }
}

int check_texture(const void* tex, int32_t width, int32_t height, int32_t pitch, int32_t format) {
  NTBC_REQUIRE(tex != nullptr, "texture pointer is NULL");
  NTBC_REQUIRE(format == NTBC_BC1 || format == NTBC_BC4, "format %d is not NTBC_BC1 or NTBC_BC4", format);
  NTBC_REQUIRE(width > 0 && height > 0 && width % 4 == 0 && height % 4 == 0,
               "texture %dx%d must be positive multiples of 4", width, height);
  const int ch = format == NTBC_BC1 ? 3 : 1;
  NTBC_REQUIRE(pitch >= width * ch, "row_pitch %d smaller than width*channels %d", pitch, width * ch);
  return NTBC_OK;
}

}  // namespace

extern "C" int ntbc_bc_encode_ref(const uint8_t* texels, int32_t width, int32_t height, int32_t row_pitch,
                                  int32_t format, uint64_t* blocks_out, int32_t* sse_out, void* stream) {
  int st = check_texture(texels, width, height, row_pitch, format);
  if (st != NTBC_OK) return st;
  NTBC_REQUIRE(blocks_out != nullptr, "blocks_out is NULL");
  const int bw = width / 4, bh = height / 4;
  const int64_t n = (int64_t)bw * bh;
  const dim3 grid((unsigned)ntbc::ceil_div(n, kThreads));
  if (format == NTBC_BC1)
    hipLaunchKernelGGL(k_encode_ref_bc1, grid, dim3(kThreads), 0, ntbc::as_stream(stream), texels, bw, bh,
                       row_pitch, blocks_out, sse_out);
  else
    hipLaunchKernelGGL(k_encode_ref_bc4, grid, dim3(kThreads), 0, ntbc::as_stream(stream), texels, bw, bh,
                       row_pitch, blocks_out, sse_out);
  return ntbc::check_launch("ntbc_bc_encode_ref");
}

// One thread per (block, texel row): the row's 4 texels (4 * ch bytes) to their place in the block-major copy.
__global__ void __launch_bounds__(kThreads) k_texels_to_blocks(const uint8_t* __restrict__ tex, int bw, int bh, int pitch,
                                                               int ch, uint8_t* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= (int64_t)bw * bh * 4) return;
  const int64_t b = e >> 2;
  const int y = (int)(e & 3);
  const int bx = (int)(b % bw), by = (int)(b / bw);
  const uint8_t* src = tex + (int64_t)(4 * by + y) * pitch + (int64_t)(4 * bx) * ch;
  uint8_t* dst = out + (b * 16 + 4 * y) * ch;
  for (int k = 0; k < 4 * ch; ++k) dst[k] = src[k];
}

extern "C" int ntbc_texels_to_blocks(const uint8_t* texels, int32_t width, int32_t height, int32_t row_pitch,
                                     int32_t format, uint8_t* blocks_out, void* stream) {
  int st = check_texture(texels, width, height, row_pitch, format);
  if (st != NTBC_OK) return st;
  NTBC_REQUIRE(blocks_out != nullptr, "blocks_out is NULL");
  const int bw = width / 4, bh = height / 4;
  const int64_t n = (int64_t)bw * bh * 4;
  if (n == 0) return NTBC_OK;
  hipLaunchKernelGGL(k_texels_to_blocks, dim3((unsigned)ntbc::ceil_div(n, kThreads)), dim3(kThreads), 0,
                     ntbc::as_stream(stream), texels, bw, bh, row_pitch, format == NTBC_BC1 ? 3 : 1, blocks_out);
  return ntbc::check_launch("ntbc_texels_to_blocks");
}

extern "C" int ntbc_bc_decode(const uint64_t* blocks, int32_t width, int32_t height, int32_t format,
                              uint8_t* texels_out, int32_t row_pitch, void* stream) {
  int st = check_texture(texels_out, width, height, row_pitch, format);
  if (st != NTBC_OK) return st;
  NTBC_REQUIRE(blocks != nullptr, "blocks is NULL");
  const int bw = width / 4, bh = height / 4;
  const int64_t n = (int64_t)bw * bh;
  const dim3 grid((unsigned)ntbc::ceil_div(n, kThreads));
  if (format == NTBC_BC1)
    hipLaunchKernelGGL(k_decode_bc1, grid, dim3(kThreads), 0, ntbc::as_stream(stream), blocks, bw, bh,
                       texels_out, row_pitch);
  else
    hipLaunchKernelGGL(k_decode_bc4, grid, dim3(kThreads), 0, ntbc::as_stream(stream), blocks, bw, bh,
                       texels_out, row_pitch);
  return ntbc::check_launch("ntbc_bc_decode");
}

extern "C" int ntbc_block_sse(const uint64_t* blocks, const uint8_t* texels, int32_t width, int32_t height,
                              int32_t row_pitch, int32_t format, int32_t* sse_out, void* stream) {
  int st = check_texture(texels, width, height, row_pitch, format);
  if (st != NTBC_OK) return st;
  NTBC_REQUIRE(blocks != nullptr && sse_out != nullptr, "blocks or sse_out is NULL");
  const int bw = width / 4, bh = height / 4;
  const int64_t n = (int64_t)bw * bh;
  hipLaunchKernelGGL(k_block_sse, dim3((unsigned)ntbc::ceil_div(n, kThreads)), dim3(kThreads), 0,
                     ntbc::as_stream(stream), blocks, texels, bw, bh, row_pitch, format, sse_out);
  return ntbc::check_launch("ntbc_block_sse");
}

extern "C" int ntbc_fallback(const uint64_t* ntbc_words, const uint64_t* ref, const int32_t* sse_ntbc,
                             const int32_t* sse_ref, int64_t n_blocks, float kappa, float delta, uint64_t* out,
                             int32_t* n_fallback, void* stream) {
  NTBC_REQUIRE(ntbc_words && ref && sse_ntbc && sse_ref && out && n_fallback, "NULL pointer argument");
  NTBC_REQUIRE(n_blocks >= 0, "n_blocks %lld < 0", (long long)n_blocks);
  if (n_blocks == 0) return NTBC_OK;
  hipLaunchKernelGGL(k_fallback, dim3((unsigned)std::min<int64_t>(ntbc::ceil_div(n_blocks, kFallbackThreads), kFallbackBlocks)), dim3(kFallbackThreads), 0,
                     ntbc::as_stream(stream), ntbc_words, ref, sse_ntbc, sse_ref, n_blocks, kappa, delta, out,
                     n_fallback);
  return ntbc::check_launch("ntbc_fallback");
}
