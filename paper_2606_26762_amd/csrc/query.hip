// Query path of libprotokv for gfx950: pseudo-token synthesis and the
// mass-aware readout.
//
// Paper: Section "Residual Statistics and Pseudo-Token Interface" (pseudo
// tokens, mass-aware bias, Eq. attn_logit), Eq. pq and Appendix Algorithms
// "DecodeTopSResidualModes" and "ProtoKV Query-Time Pseudo-Token Decoding
// and Attention".
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "pkv_internal.h"

namespace pkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t q_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float q_from_bf16(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// cos and sin of the rotary angle pos * inv (inv = theta^(-2i/D)): the angle
// in float64, whole turns taken off in float64, the rest (|r| <= pi) to
// float32 sincos.  Stream positions reach 10^6 and more, where a float32
// angle would already be off by tenths of a radian.
__device__ __forceinline__ void rope_cs(double pos, double inv, float& c, float& s) {
  const double a = pos * inv;
  const double turns = rint(a * 0.15915494309189535);  // 1 / (2 pi)
  const float r = (float)fma(-turns, 6.283185307179586, a);
  sincosf(r, &s, &c);
}

// Rotate-half rotation of the pair (x1 = dim i, x2 = dim i + D/2):
// lo = x1 c - x2 s, hi = x2 c + x1 s (float32, one rounding per operation).
__device__ __forceinline__ void rope_pair(float x1, float x2, float c, float s, float& lo, float& hi) {
  lo = x1 * c - x2 * s;
  hi = x2 * c + x1 * s;
}

// ---------------------------------------------------------------------------
// Exact top-S decoding of one PQ histogram.
//
// With eps = 1 the smoothed probability is (H[g][c]+1)/(n_res+C), so a code
// tuple's log-score sum_g log P(g, z_g) orders tuples exactly as the integer
// prod_g (H[g][z_g]+1); the denominator is common to every tuple.  Equal
// scores are ordered by the code tuple, lexicographically ascending.
//
// The beam of Alg. DecodeTopSResidualModes returns the exact top-S for any
// beam width B >= S (a prefix of a top-S tuple always ranks within the top S
// prefixes: otherwise S better prefixes, each completed with the same
// suffix, would give S better tuples).  So the beam here has width S: at
// subspace g the new beam is the best S of {prefix_i x rank_r}, taken by a
// merge over the prefixes (each prefix's extensions are already ordered by
// the codewords' rank (count desc, code asc)).
//
// Products are exact 192-bit integers (three 64-bit limbs): factors are
// < 2^24 and there are 8 of them.  Code tuples are packed one nibble per
// subspace, subspace 0 in the most significant nibble, so comparing packed
// values compares tuples lexicographically.
// ---------------------------------------------------------------------------
struct Big {
  uint64_t w0, w1, w2;  // little-endian limbs
};

__device__ __forceinline__ Big big_mul(const Big& a, uint32_t f) {
  Big r;
  unsigned __int128 t = (unsigned __int128)a.w0 * f;
  r.w0 = (uint64_t)t;
  t = (unsigned __int128)a.w1 * f + (uint64_t)(t >> 64);
  r.w1 = (uint64_t)t;
  t = (unsigned __int128)a.w2 * f + (uint64_t)(t >> 64);
  r.w2 = (uint64_t)t;
  return r;
}

// true if candidate (pa, ca) ranks before (pb, cb): larger product, then
// smaller packed code tuple.
__device__ __forceinline__ bool ranks_before(const Big& pa, uint32_t ca, const Big& pb, uint32_t cb) {
  if (pa.w2 != pb.w2) return pa.w2 > pb.w2;
  if (pa.w1 != pb.w1) return pa.w1 > pb.w1;
  if (pa.w0 != pb.w0) return pa.w0 > pb.w0;
  return ca < cb;
}

constexpr int SYN_P = 32;  // prototypes per workgroup (one wave: 32 x {keys, values})

// Per-thread beam state in dynamic LDS, planes [buf][entry][thread] so the
// 64 threads touch consecutive words: three 64-bit limbs and the packed code.
struct BeamView {
  uint64_t* w0;
  uint64_t* w1;
  uint64_t* w2;
  uint32_t* code;
  int S;
  __device__ __forceinline__ int at(int buf, int e, int tl) const { return (buf * S + e) * 64 + tl; }
};

__device__ void decode_top_s(const uint32_t* hist /* [G][CMAX] */, int C, int S, const BeamView& bv, int tl,
                             uint32_t* out_codes /* S */) {
  int nb = 1;
  int cur = 0;
  bv.w0[bv.at(0, 0, tl)] = 1;
  bv.w1[bv.at(0, 0, tl)] = 0;
  bv.w2[bv.at(0, 0, tl)] = 0;
  bv.code[bv.at(0, 0, tl)] = 0;
  for (int g = 0; g < G; ++g) {
    // rank the codewords of subspace g: count desc, code asc (top min(S, C))
    uint32_t h[CMAX];
#pragma unroll
    for (int c = 0; c < CMAX; ++c) h[c] = c < C ? hist[g * CMAX + c] : 0u;
    const int nr = S < C ? S : C;
    uint32_t rfac[SMAX], rcode[SMAX];
    uint32_t used = 0;
    for (int r = 0; r < nr; ++r) {
      int bc = -1;
      uint32_t bh = 0;
#pragma unroll
      for (int c = 0; c < CMAX; ++c) {
        const bool ok = c < C && !((used >> c) & 1u);
        if (ok && (bc < 0 || h[c] > bh)) { bc = c; bh = h[c]; }
      }
      used |= 1u << bc;
      rfac[r] = bh + 1u;
      rcode[r] = (uint32_t)bc;
    }
    // merge: row i = beam prefix i, column = rank
    int ptr[SMAX];
#pragma unroll
    for (int i = 0; i < SMAX; ++i) ptr[i] = 0;
    const int shift = 4 * (G - 1 - g);
    const int total = nb * nr;
    const int nout = S < total ? S : total;
    const int nxt = cur ^ 1;
    for (int o = 0; o < nout; ++o) {
      int bi = -1;
      Big bp{0, 0, 0};
      uint32_t bcode = 0;
      for (int i = 0; i < nb; ++i) {
        if (ptr[i] >= nr) continue;
        const int a = bv.at(cur, i, tl);
        Big p{bv.w0[a], bv.w1[a], bv.w2[a]};
        Big cand = big_mul(p, rfac[ptr[i]]);
        uint32_t code = bv.code[a] | (rcode[ptr[i]] << shift);
        if (bi < 0 || ranks_before(cand, code, bp, bcode)) { bi = i; bp = cand; bcode = code; }
      }
      ptr[bi] += 1;
      const int w = bv.at(nxt, o, tl);
      bv.w0[w] = bp.w0;
      bv.w1[w] = bp.w1;
      bv.w2[w] = bp.w2;
      bv.code[w] = bcode;
    }
    nb = nout;
    cur = nxt;
  }
  for (int s = 0; s < S; ++s) out_codes[s] = s < nb ? bv.code[bv.at(cur, s, tl)] : 0u;
}

// Exchanges within a quad of lanes (DPP quad_perm, no LDS round trip).
template <int CTRL>
__device__ __forceinline__ uint32_t qperm(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ uint64_t qperm64(uint64_t x) {
  return (uint64_t)qperm<CTRL>((uint32_t)x) | ((uint64_t)qperm<CTRL>((uint32_t)(x >> 32)) << 32);
}
constexpr int QP_XOR1 = 0xB1;  // lanes (1, 0, 3, 2)

__device__ __forceinline__ uint64_t sel64(bool t, uint64_t a, uint64_t b) {
  const uint64_t m = 0ull - (uint64_t)t;
  return (a & m) | (b & ~m);
}

// Decoding by halves: the top SM tuples of subspaces 0..3 and of subspaces
// 4..7, then the top SM of their products (the pairs with (i + 1)(j + 1) <= SM,
// as above).  A product of four factors below 2^37 is a float64 integer whose
// 16 low mantissa bits are free: they hold the half's code tuple, inverted, so
// that a candidate is one float64 product and one OR, and one v_max_f64 /
// v_min_f64 pair orders two candidates by (product desc, tuple asc).  The
// codeword ranks come from 16-bit keys (H + 1) << 4 | (15 - c), two subspaces
// in the halves of one register.  Half products from 2^37 (the four largest
// counts of a half 600 in the geometric mean) are 64-bit integers above the
// tuple instead, ordered by compares and selects; with counts above 4094 the
// keys are whole registers and the tuple lies beside the 64-bit product, ordered
// by both (slots of 60 000 residuals: 112 units x 256, S = 8, 28 us; 256 x 2 048,
// S = 8, 320, and S = 12, 1 008; a beam search on two lanes in this kernel, which
// took counts above 4094 before, 43, 578 and 2 940, and the kernels before the
// decode by halves 53, 379 and 1 430).
//
// The joined product's ties are broken by the first half's tuple, then the
// second's, whose order within one first half is its rank j: a tag of 2
// log2(SM) bits (the tuple's rank among the SM first halves, SM - 1 - j).
// Products below 2^53 / 2^tag carry it in the mantissa like the others; larger
// ones are compared as 54 + 42 bits (below 2^96) or 128 bits (large counts) with
// the tag below.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// a <- the first in rank order of a and b, b <- the other
__device__ __forceinline__ void order2(u16x2& a, u16x2& b) {
  const u16x2 hi = __builtin_elementwise_max(a, b), lo = __builtin_elementwise_min(a, b);
  a = hi;
  b = lo;
}
// (raw instructions: fmax / fmin would first quiet operands that are never NaN)
__device__ __forceinline__ double max64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double min64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ void order2(double& a, double& b) {
  const double hi = max64(a, b), lo = min64(a, b);
  a = hi;
  b = lo;
}
__device__ __forceinline__ void first2(double& a, double b) { a = max64(a, b); }
__device__ __forceinline__ void order2(uint64_t& a, uint64_t& b) {
  const bool sw = b > a;
  const uint64_t t = a;
  a = sel64(sw, b, a);
  b = sel64(sw, t, b);
}
__device__ __forceinline__ void first2(uint64_t& a, uint64_t b) { a = sel64(b > a, b, a); }
// a product of two half products: P >> 42, and the low 42 bits above an 8-bit tag
struct Wide {
  uint64_t hi, lo;
};
__device__ __forceinline__ void order2(Wide& a, Wide& b) {
  const bool sw = (b.hi > a.hi) | ((b.hi == a.hi) & (b.lo > a.lo));
  const Wide t = a;
  a.hi = sel64(sw, b.hi, a.hi);
  a.lo = sel64(sw, b.lo, a.lo);
  b.hi = sel64(sw, t.hi, b.hi);
  b.lo = sel64(sw, t.lo, b.lo);
}
__device__ __forceinline__ void first2(Wide& a, const Wide& b) {
  const bool sw = (b.hi > a.hi) | ((b.hi == a.hi) & (b.lo > a.lo));
  a.hi = sel64(sw, b.hi, a.hi);
  a.lo = sel64(sw, b.lo, a.lo);
}
// Half products of large counts beside their inverted tuple, and products of two
// of them beside their tag.
struct Tagged64 {
  uint64_t p;
  uint32_t tag;
};
struct Tagged128 {
  uint64_t hi, lo;
  uint32_t tag;
};
// b comes before a in rank order
__device__ __forceinline__ bool swapped(const Tagged64& a, const Tagged64& b) {
  return (b.p > a.p) | ((b.p == a.p) & (b.tag > a.tag));
}
__device__ __forceinline__ bool swapped(const Tagged128& a, const Tagged128& b) {
  return (b.hi > a.hi) | ((b.hi == a.hi) & ((b.lo > a.lo) | ((b.lo == a.lo) & (b.tag > a.tag))));
}
__device__ __forceinline__ Tagged64 pick(bool t, const Tagged64& a, const Tagged64& b) {
  return Tagged64{t ? a.p : b.p, t ? a.tag : b.tag};
}
__device__ __forceinline__ Tagged128 pick(bool t, const Tagged128& a, const Tagged128& b) {
  return Tagged128{t ? a.hi : b.hi, t ? a.lo : b.lo, t ? a.tag : b.tag};
}
template <typename E>
__device__ __forceinline__ auto order2(E& a, E& b) -> decltype(pick(true, a, b), void()) {
  const bool sw = swapped(a, b);
  const E t = a;
  a = pick(sw, b, a);
  b = pick(sw, t, b);
}
template <typename E>
__device__ __forceinline__ auto first2(E& a, const E& b) -> decltype(pick(true, a, b), void()) {
  a = pick(swapped(a, b), b, a);
}
__device__ __forceinline__ void order2(uint32_t& a, uint32_t& b) {
  const uint32_t hi = max(a, b), lo = min(a, b);
  a = hi;
  b = lo;
}
// bitonic sequence a[0..N-1] -> rank order
template <int N, typename E>
__device__ __forceinline__ void bitonic(E* a) {
#pragma unroll
  for (int j = N / 2; j > 0; j >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if ((i & j) == 0) order2(a[i], a[i + j]);
}
// a <- the first N in rank order of a[0..N-1] and b[0..M-1], both in order
template <int N, int M, typename E>
__device__ __forceinline__ void keep_top(E (&a)[N], const E (&b)[M]) {
#pragma unroll
  for (int i = N - M; i < N; ++i) first2(a[i], b[N - 1 - i]);
  bitonic<N>(a);
}
// Eight keys into rank order (Batcher's odd-even merge sort, 19 exchanges).
template <typename E>
__device__ __forceinline__ void sort8(E* a) {
  constexpr int X[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                            {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int i = 0; i < 19; ++i) order2(a[X[i][0]], a[X[i][1]]);
}
// The top N of the candidates cand(i, j), i, j < N, in rank order: both
// factors are in order, so candidate (i, j) has (i + 1)(j + 1) - 1 before it and
// only those with (i + 1)(j + 1) <= N count.  Each column j (prefixes 0 ..
// N / (j + 1) - 1) is in order, and so is row 0.
template <typename E, typename F>
__device__ __forceinline__ void top_products(E (&r)[8], F cand) {
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = cand(i, 0);
  E b[4] = {cand(0, 1), cand(1, 1), cand(2, 1), cand(3, 1)};
  keep_top(r, b);
  E c[4] = {cand(0, 2), cand(1, 2), cand(1, 3), cand(0, 3)};
  bitonic<4>(c);
  keep_top(r, c);
  E d[4] = {cand(0, 4), cand(0, 5), cand(0, 6), cand(0, 7)};
  keep_top(r, d);
}
template <typename E, typename F>
__device__ __forceinline__ void top_products(E (&r)[16], F cand) {
#pragma unroll
  for (int i = 0; i < 16; ++i) r[i] = cand(i, 0);
  {
    E b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = cand(i, 1);
    keep_top(r, b);
  }
  {  // columns 2 (five), 7 (two)
    E b[8] = {cand(0, 2), cand(1, 2), cand(2, 2), cand(3, 2), cand(4, 2), E{}, cand(1, 7), cand(0, 7)};
    bitonic<8>(b);
    keep_top(r, b);
  }
  {  // columns 3 (four), 4 (three)
    E b[8] = {cand(0, 3), cand(1, 3), cand(2, 3), cand(3, 3), E{}, cand(2, 4), cand(1, 4), cand(0, 4)};
    bitonic<8>(b);
    keep_top(r, b);
  }
  {  // columns 5, 6 (two each)
    E b[4] = {cand(0, 5), cand(1, 5), cand(1, 6), cand(0, 6)};
    bitonic<4>(b);
    keep_top(r, b);
  }
  {
    E b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = cand(0, 8 + j);
    keep_top(r, b);
  }
}

constexpr double HALF_MAX = 0x1p37;        // half products in float64 stay below this
constexpr uint32_t HALF_COUNT = 4094;      // counts up to this (half products below 2^48)
constexpr uint32_t HALF_TAG = 0xFFFFu;     // the inverted tuple in a half product's low bits

__device__ __forceinline__ uint32_t lo32(double x) { return (uint32_t)__double_as_longlong(x); }
__device__ __forceinline__ uint32_t lo32(uint64_t x) { return (uint32_t)x; }
__device__ __forceinline__ uint32_t lo32(const Tagged64& x) { return x.tag; }
__device__ __forceinline__ double with_lo32(double x, uint32_t lo) {
  return __longlong_as_double((__double_as_longlong(x) & ~0xFFFFFFFFll) | lo);
}
__device__ __forceinline__ uint64_t with_lo32(uint64_t x, uint32_t lo) { return (x & ~0xFFFFFFFFull) | lo; }
__device__ __forceinline__ Tagged64 with_lo32(const Tagged64& x, uint32_t lo) { return Tagged64{x.p, lo}; }
// a half product x (tag clear) as an integer
__device__ __forceinline__ uint64_t half_int(double x) { return (uint64_t)x; }
__device__ __forceinline__ uint64_t half_int(uint64_t x) { return x >> 16; }
__device__ __forceinline__ uint64_t half_int(const Tagged64& x) { return x.p; }
// the value of lane CTRL's pattern in the quad
template <int CTRL>
__device__ __forceinline__ double half_perm(double x) {
  return __longlong_as_double((long long)qperm64<CTRL>((uint64_t)__double_as_longlong(x)));
}
template <int CTRL>
__device__ __forceinline__ uint64_t half_perm(uint64_t x) { return qperm64<CTRL>(x); }
template <int CTRL>
__device__ __forceinline__ Tagged64 half_perm(const Tagged64& x) {
  return Tagged64{qperm64<CTRL>(x.p), qperm<CTRL>(x.tag)};
}

// The counts of four subspaces, and the largest half product and count they
// can give.
struct HalfCounts {
  uint4 h[4][4];
  double bound;
  uint32_t most;
};

// The top SM tuples of one half, in rank order: product | inverted tuple (E:
// float64, or uint64_t with the product shifted up by 16).
template <int SM, typename E>
__device__ __forceinline__ void decode_half(const HalfCounts& hc, int C, E (&p)[SM]) {
  using F = std::conditional_t<std::is_same_v<E, double>, double, uint32_t>;
#pragma unroll
  for (int pr = 0; pr < 2; ++pr) {  // subspaces 2 pr (low halves) and 2 pr + 1
    u16x2 key[16];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint4 a = hc.h[2 * pr][v], b = hc.h[2 * pr + 1][v];
      const uint32_t x[4] = {a.x | b.x << 16, a.y | b.y << 16, a.z | b.z << 16, a.w | b.w << 16};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * v + e;
        const uint32_t k = (x[e] << 4) + (uint32_t)(16 + 15 - c) * 0x10001u;
        key[c] = __builtin_bit_cast(u16x2, c < C ? k : 0u);
      }
    }
    sort8(key);
    sort8(key + 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (SM == 16) order2(key[i], key[15 - i]);
      else key[i] = __builtin_elementwise_max(key[i], key[15 - i]);
    }
    bitonic<8>(key);
    if (SM == 16) {
      bitonic<8>(key + 8);  // (in reversed places: still a bitonic sequence)
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int g = 2 * pr + s;
      F f[SM];
      uint32_t z[SM];
#pragma unroll
      for (int j = 0; j < SM; ++j) {
        const uint32_t k = __builtin_bit_cast(uint32_t, key[j]);
        f[j] = (F)((k >> (16 * s + 4)) & 0xFFFu);
        z[j] = ((k >> (16 * s)) & 15u) << (12 - 4 * g);
      }
      if (g == 0) {
#pragma unroll
        for (int j = 0; j < SM; ++j) {
          const E x = (E)f[j] * (E)(std::is_same_v<E, double> ? 1 : 65536);
          p[j] = with_lo32(x, lo32(x) | z[j]);
        }
        continue;
      }
      E b[SM];
      uint32_t t[SM];
#pragma unroll
      for (int i = 0; i < SM; ++i) {
        t[i] = lo32(p[i]) & HALF_TAG;
        b[i] = with_lo32(p[i], lo32(p[i]) & ~HALF_TAG);
      }
      top_products(p, [&](int i, int j) {
        const E x = b[i] * f[j];
        return with_lo32(x, lo32(x) | t[i] | z[j]);
      });
    }
  }
}

// The same for counts up to 65534, read again from LDS: unit 4 g + v of the
// half at `unit`.  One rolled loop over the subspaces, from the empty tuple.
template <int SM, typename F>
__device__ __forceinline__ void decode_half_large(F unit, int C, Tagged64 (&p)[SM]) {
#pragma unroll
  for (int i = 0; i < SM; ++i) p[i] = Tagged64{i == 0 ? 1ull : 0ull, 0u};
#pragma nounroll
  for (int g = 0; g < 4; ++g) {
    uint32_t key[16];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint4 h = unit(4 * g + v);
      const uint32_t x[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 4 * v + e;
        key[c] = c < C ? (x[e] << 4) + (uint32_t)(16 + 15 - c) : 0u;
      }
    }
    sort8(key);
    sort8(key + 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (SM == 16) order2(key[i], key[15 - i]);
      else key[i] = max(key[i], key[15 - i]);
    }
    bitonic<8>(key);
    if (SM == 16) bitonic<8>(key + 8);  // (in reversed places: still a bitonic sequence)
    const int sh = 12 - 4 * g;
    Tagged64 b[SM];
#pragma unroll
    for (int i = 0; i < SM; ++i) b[i] = p[i];
    top_products(p, [&](int i, int j) {
      return Tagged64{b[i].p * (key[j] >> 4), b[i].tag | (key[j] & 15u) << sh};
    });
  }
}

// The top S tuples from the halves' top SM (pa: subspaces 0..3, pb: 4..7), lane
// q of the pair writing those of its parity.  `wide`: uniform, some lane's
// product may not fit the mantissa beside its tag.  codes: 4 SM words of LDS per
// lane at a stride of 64 words.
template <int SM, typename E>
__device__ __forceinline__ void decode_join(const E (&pa)[SM], const E (&pb)[SM], bool wide, bool mine, int S, int q,
                                            uint32_t* codes, uint32_t* out) {
  constexpr int LB = SM == 8 ? 3 : 4;
  uint32_t ra[SM];  // rank of the first half's tuple among the SM, larger = earlier tuple
#pragma unroll
  for (int i = 0; i < SM; ++i) ra[i] = 0;
#pragma unroll
  for (int i = 0; i < SM; ++i)
#pragma unroll
    for (int k = 0; k < i; ++k) {
      const uint32_t t = (lo32(pa[k]) & HALF_TAG) < (lo32(pa[i]) & HALF_TAG) ? 1u : 0u;
      ra[i] += t;
      ra[k] += 1u - t;
    }
  E a[SM], b[SM];
#pragma unroll
  for (int i = 0; i < SM; ++i) {
    codes[ra[i] * 64] = (~lo32(pa[i]) & HALF_TAG) << 16;
    codes[(2 * SM - 1 - i) * 64] = ~lo32(pb[i]) & HALF_TAG;
    a[i] = with_lo32(pa[i], lo32(pa[i]) & ~HALF_TAG);
    b[i] = with_lo32(pb[i], lo32(pb[i]) & ~HALF_TAG);
    ra[i] <<= LB;
  }
  uint32_t tag[SM];
  bool done = false;
  if constexpr (std::is_same_v<E, double>) {
    if (!wide) {
      double r[SM];
      top_products(r, [&](int i, int j) {
        const double x = a[i] * b[j];
        return with_lo32(x, lo32(x) | ra[i] | (uint32_t)(SM - 1 - j));
      });
#pragma unroll
      for (int o = 0; o < SM; ++o) tag[o] = lo32(r[o]) & (SM * SM - 1);
      done = true;
    }
  }
  if (!done) {
    uint64_t ia[SM], ib[SM];
#pragma unroll
    for (int i = 0; i < SM; ++i) {
      ia[i] = half_int(a[i]);
      ib[i] = half_int(b[i]);
    }
    if constexpr (std::is_same_v<E, Tagged64>) {
      // (the second halves in LDS: SM = 16 then fits 256 registers, two waves
      // a SIMD)
      uint32_t* second_half = codes + 2 * SM * 64;
#pragma unroll
      for (int j = 0; j < SM; ++j) {
        second_half[2 * j * 64] = (uint32_t)ib[j];
        second_half[(2 * j + 1) * 64] = (uint32_t)(ib[j] >> 32);
      }
      asm volatile("" ::: "memory");
      Tagged128 r[SM];
      top_products(r, [&](int i, int j) {
        const uint64_t b = (uint64_t)second_half[(2 * j + 1) * 64] << 32 | second_half[2 * j * 64];
        const unsigned __int128 x = (unsigned __int128)ia[i] * b;
        return Tagged128{(uint64_t)(x >> 64), (uint64_t)x, ra[i] | (uint32_t)(SM - 1 - j)};
      });
#pragma unroll
      for (int o = 0; o < SM; ++o) {
        tag[o] = r[o].tag;
        asm("" : "+v"(tag[o]));
      }
    } else {
      Wide r[SM];
      top_products(r, [&](int i, int j) {
        const unsigned __int128 x = (unsigned __int128)ia[i] * ib[j];
        return Wide{(uint64_t)(x >> 42), ((uint64_t)x & ((1ull << 42) - 1)) << 8 | ra[i] | (uint32_t)(SM - 1 - j)};
      });
#pragma unroll
      for (int o = 0; o < SM; ++o) tag[o] = (uint32_t)r[o].lo & (SM * SM - 1);
    }
  }
  if (mine) {
#pragma unroll
    for (int o = 0; o < SM; ++o)
      if (o < S && (o & 1) == q)
        out[o] = codes[(tag[o] >> LB) * 64] | codes[(SM + (tag[o] & (SM - 1))) * 64];
    if (q == 0) out[SMAX] = 0u;
  }
}

// Two lanes per (slot, K/V) beam, 16 slots per wave: each lane takes a half and
// both join them.  The wave's histograms (1 KiB per slot) come into LDS by DMA,
// whole lines at a time: loaded from registers, 16 bytes per lane 256 bytes apart,
// every line went through L1 several times over.  Lane l of a slot's load brings
// the 16-byte unit that leaves unit v of (K/V, half) r at 16 r + (v + 4 i + r) %
// 16, so that lanes reading one unit of different slots fall on different banks.
// With `centres` (rows formed by the readout) it also writes each slot's bias,
// tau_k into the key record's spare word and n into the value record's.
// Bound by the histograms' bytes (256 units x 2 048 slots, 0.6 GB: 159 us, with
// loads into registers 195, 197 with one lane per beam and sorting networks on
// 64-bit products) or, on few slots, by one wave's 1 530 VALU instructions
// (112 units x 256 slots: 32 -> 17 us; 64 slots 25 -> 7 us; S = 16 on 2 000
// slots, two lanes and merge pops before, 63 -> 13.5 us).  Two waves a SIMD, as the
// LDS allows: with 262 registers S > 8 had one (112 x 256, S = 16, 49 -> 38 us).
// Those are times of one query after another.  A wave runs straight through its
// code once, so a query after eight folds, or with other data through the caches
// since, waits for instructions too (by events, S = 8: 64 slots 10 and 17 us, 28 and
// 42 by the kernels before; 112 x 256 17 and 25, before 35 and 54; 256 x 1 024 90 and
// 121, before 114 and 139; S = 16, 112 x 256, 37 and 51, before 88 and 136).
template <int SM>
__global__ __launch_bounds__(256, 2) void k_decode(Dims dm, Workspace ws, int sid, int n_active, int centres) {
  constexpr int SPW = 16;  // slots per wave
  __shared__ __attribute__((aligned(16))) uint8_t s_mem[4][SPW * 1024];
  static_assert(4 * SM * 64 * 4 <= SPW * 1024, "tuples and halves reuse the histograms' LDS");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nslots = dm.units * n_active;
  const int slot0 = ((int)blockIdx.x * 4 + wave) * SPW;  // unit * n_active + slot
  if (slot0 >= nslots) return;  // uniform, and waves do not synchronise below
  uint8_t* mem = s_mem[wave];
  const uint8_t* bank = ws.bank + (size_t)sid * dm.units * dm.K * ROW;
  {
    int u = slot0 / n_active, p = slot0 % n_active;  // uniform
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      const int r = lane >> 4, v = ((lane & 15) - (4 * i + r)) & 15;
      lds_dma16(bank + ((size_t)u * dm.K + p) * ROW + ROW_HK + (16 * r + v) * 16, mem + i * 1024);
      if (slot0 + i + 1 < nslots) {  // past the last slot the loads repeat it
        const bool next = p + 1 == n_active;
        p = next ? 0 : p + 1;
        u += next ? 1 : 0;
      }
    }
  }
  const int q = lane & 1, kv = (lane >> 1) & 1;
  const bool bvalid = slot0 + (lane >> 2) < nslots;
  const int sl = min(slot0 + (lane >> 2), nslots - 1);
  const int u = sl / n_active, p = sl % n_active;
  const uint8_t* row = bank + ((size_t)u * dm.K + p) * ROW;
  const RowMeta m = *reinterpret_cast<const RowMeta*>(row + ROW_META);
  uint32_t* out = ws.pcodes + (((size_t)u * dm.K + p) * 2 + kv) * PCW;
  const bool pq = (dm.flags & PROTOKV_FLAG_PQ) != 0;
  const int S = dm.S, C = dm.C;
  const bool nores = !pq || m.n_res == 0;
  if (bvalid && q == 0 && nores) out[SMAX] = 1u;
  if (centres && bvalid && q == 0) {  // centres: uniform
    if (kv == 0) {
      const bool mb = (dm.flags & PROTOKV_FLAG_MASS_BIAS) != 0;
      ws.pbias[(size_t)u * dm.K + p] = mb ? logf((float)m.n) : 0.f;
      // tau_k in the key record's spare word: the readout rotates the
      // slot's formed pseudo-keys at it
      out[SMAX + 1] = (uint32_t)m.tau;
    } else {
      // n in the value record's spare word: the readout divides the slot's
      // sums by it
      out[SMAX + 1] = m.n;
    }
  }
  // (k_decode_wide takes the others)
  const bool mine = bvalid && !nores && m.n_res <= 65534u && S <= SM;
  wait_vm<0>();  // the histograms have landed
  asm volatile("" ::: "memory");
  auto unit = [&](int i) {  // 16 bytes of this lane's half
    return *reinterpret_cast<const uint4*>(mem + (lane >> 2) * 1024 + (lane & 3) * 256 + ((i + lane) & 15) * 16);
  };
  HalfCounts hc;
  hc.bound = 1.0;
  hc.most = 0;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    uint32_t mx = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint4 x = unit(4 * g + v);
      hc.h[g][v] = x;
      mx = max(max(mx, max(x.x, x.y)), max(x.z, x.w));
    }
    hc.most = max(hc.most, mx);
    hc.bound *= (double)mx + 1.0;
  }
  const double bound = hc.bound * __longlong_as_double((long long)qperm64<QP_XOR1>((uint64_t)__double_as_longlong(hc.bound)));
  const bool wide = !__all(!mine || bound < 0x1p53 / (SM * SM));
  auto halves = [&](auto e) {
    using E = decltype(e);
    E pa[SM], pb[SM];
    if constexpr (std::is_same_v<E, Tagged64>) decode_half_large<SM>(unit, C, pa);
    else decode_half<SM, E>(hc, C, pa);
#pragma unroll
    for (int i = 0; i < SM; ++i) {  // lanes (1, 1, 3, 3) and (0, 0, 2, 2) of each quad
      pb[i] = half_perm<0xF5>(pa[i]);
      pa[i] = half_perm<0xA0>(pa[i]);
    }
    decode_join<SM, E>(pa, pb, wide, mine, S, q, reinterpret_cast<uint32_t*>(mem) + lane, out);
  };
  if (__all(!mine || hc.bound < HALF_MAX) && __all(!mine || hc.most <= HALF_COUNT))
    halves(0.0);
  else if (__all(!mine || hc.most <= HALF_COUNT))
    halves((uint64_t)0);
  else
    halves(Tagged64{});
}

// Decoding, wide path (prototypes with more than 65534 residuals, whose
// products need 192 bits): one thread per (slot, K/V) of one (layer, kv
// head), 32 slots per
// workgroup (lanes 0-31 keys, 32-63 values).  Codes go to ws.pcodes
// [units][K][2][SMAX] (packed tuples, subspace 0 in the top nibble) and a flag
// word per (slot, K/V): 1 if the slot has no residual statistics.
template <int SM>
__global__ __launch_bounds__(64) void k_decode_wide(Dims dm, Workspace ws, int sid, int n_active, int blocks_per_unit) {
  extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
  const int lane = threadIdx.x;
  const int u = blockIdx.x / blocks_per_unit;
  const int p = (blockIdx.x % blocks_per_unit) * SYN_P + (lane & 31);
  const int kv = lane >> 5;
  if (p >= n_active) return;
  const size_t unit = (size_t)sid * dm.units + u;
  const int S = dm.S;
  const uint8_t* row = ws.bank + (unit * dm.K + p) * ROW;
  const RowMeta m = *reinterpret_cast<const RowMeta*>(row + ROW_META);
  uint32_t* out = ws.pcodes + (((size_t)u * dm.K + p) * 2 + kv) * PCW;
  const bool pq = (dm.flags & PROTOKV_FLAG_PQ) != 0;
  if (!pq || m.n_res == 0) return;             // flagged by k_decode
  if (m.n_res <= 65534u && S <= SM) return;    // decoded by k_decode
  out[SMAX] = 0u;
  const uint32_t* hist = reinterpret_cast<const uint32_t*>(row + (kv ? ROW_HV : ROW_HK));
  uint32_t codes[SMAX];
  {
    BeamView bv;
    bv.S = S;
    bv.w0 = reinterpret_cast<uint64_t*>(s_dyn);
    bv.w1 = bv.w0 + 2 * S * 64;
    bv.w2 = bv.w1 + 2 * S * 64;
    bv.code = reinterpret_cast<uint32_t*>(bv.w2 + 2 * S * 64);
    decode_top_s(hist, dm.C, S, bv, lane, codes);
  }
  for (int s2 = 0; s2 < S; ++s2) out[s2] = codes[s2];
}

// Pseudo-tokens: one wave per slot, lane l writes components 2l, 2l+1 of each
// of the 2S rows: k~_s = kv_dtype(float32(c + r^K_s)), v~_s likewise, with
// c = float32(sum / n) (EMA centres: the stored c) and r_s = concatenated
// codewords; bias = log n.
template <int FP32>
__global__ __launch_bounds__(256) void k_materialize(Dims dm, Workspace ws, int sid, int n_active) {
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int u = gw / dm.K, p = gw % dm.K;
  if (u >= dm.units || p >= n_active) return;
  const size_t unit = (size_t)sid * dm.units + u;
  // S_k rows from row rb of the unit (variance-aware allocation), else S from p S
  const bool var = ws.ps_count != nullptr;
  const int S = var ? ws.ps_count[(size_t)u * dm.K + p] : dm.S;
  const size_t rb = var ? (size_t)ws.ps_off[(size_t)u * dm.K + p] : (size_t)p * dm.S;
  const size_t es = FP32 ? 4 : 2;
  const uint8_t* row = ws.bank + (unit * dm.K + p) * ROW;
  const RowMeta m = *reinterpret_cast<const RowMeta*>(row + ROW_META);
  const float nf = (float)m.n;
  const float2 sk = reinterpret_cast<const float2*>(row + ROW_SUMK)[lane];
  const float2 sv = reinterpret_cast<const float2*>(row + ROW_SUMV)[lane];
  const float* cbk = ws.codebooks + unit * (2 * G * CMAX * DP);
  const int g = lane >> 3, u16 = (2 * lane) & 15;
  // rotary positions: the pseudo-keys turn at tau_k; lane l holds dims 2l,
  // 2l + 1, pair index 2 (l % 32) + {0, 1}, its partner in lane l ^ 32
  const bool rope = ws.rope_inv != nullptr;
  float rc[2] = {1.f, 1.f}, rs[2] = {0.f, 0.f};
  if (rope)
    for (int e = 0; e < 2; ++e) rope_cs((double)m.tau, ws.rope_inv[2 * (lane & 31) + e], rc[e], rs[e]);
  {
    const bool mb = (dm.flags & PROTOKV_FLAG_MASS_BIAS) != 0;
    const float bias = mb ? logf(nf) : 0.f;
    if (lane == 0) ws.pbias[(size_t)u * dm.K + p] = bias;
    if (var && lane < S) ws.prow_bias[(size_t)u * dm.K * dm.S + rb + lane] = bias;
  }
  // the decoded tuples of K and V first (all loads in flight together)
  const uint32_t* codes_k = ws.pcodes + (((size_t)u * dm.K + p) * 2) * PCW;
  const uint32_t* codes_v = codes_k + PCW;
  uint32_t ck[SMAX], cv[SMAX];
#pragma unroll
  for (int s2 = 0; s2 < SMAX; ++s2) {
    ck[s2] = s2 < S ? codes_k[s2] : 0u;
    cv[s2] = s2 < S ? codes_v[s2] : 0u;
  }
  const bool nores_k = codes_k[SMAX] != 0u, nores_v = codes_v[SMAX] != 0u;
  const int sh = 4 * (G - 1 - g);
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const float cd = (dm.flags & PROTOKV_FLAG_EMA_CENTRES) ? 1.f : nf;  // EMA centres are stored
    const float2 c = w ? make_float2(sv.x / cd, sv.y / cd) : make_float2(sk.x / cd, sk.y / cd);
    const bool nores = w ? nores_v : nores_k;
    const float* cbw = cbk + ((size_t)w * G + g) * CMAX * DP + u16;
    uint8_t* out = (w ? ws.pv : ws.pk) + ((size_t)u * dm.K * dm.S + rb) * D * es;
#pragma unroll
    for (int s2 = 0; s2 < SMAX; ++s2) {
      if (s2 < S) {
        float2 val = c;
        if (!nores) {
          const int z = ((w ? cv[s2] : ck[s2]) >> sh) & 15;
          const float2 cw = *reinterpret_cast<const float2*>(cbw + z * DP);
          val.x = c.x + cw.x;
          val.y = c.y + cw.y;
        }
        if (rope && w == 0) {  // rotate the key as rounded to the KV dtype
          if (!FP32) {
            val.x = q_from_bf16(q_to_bf16(val.x));
            val.y = q_from_bf16(q_to_bf16(val.y));
          }
          const float px = __shfl_xor(val.x, 32, 64), py = __shfl_xor(val.y, 32, 64);
          float lo, hi;
          if (lane < 32) {
            rope_pair(val.x, px, rc[0], rs[0], lo, hi);
            val.x = lo;
            rope_pair(val.y, py, rc[1], rs[1], lo, hi);
            val.y = lo;
          } else {
            rope_pair(px, val.x, rc[0], rs[0], lo, hi);
            val.x = hi;
            rope_pair(py, val.y, rc[1], rs[1], lo, hi);
            val.y = hi;
          }
        }
        if (FP32) {
          reinterpret_cast<float2*>(out + (size_t)s2 * D * 4)[lane] = val;
        } else {
          const uint32_t packed = (uint32_t)q_to_bf16(val.x) | ((uint32_t)q_to_bf16(val.y) << 16);
          reinterpret_cast<uint32_t*>(out + (size_t)s2 * D * 2)[lane] = packed;
        }
      }
    }
  }
}

// bf16 pseudo-tokens, one wave per slot with 16-byte stores: lane l writes
// dims [8 (l % 16), 8 (l % 16) + 8) of rows s = l / 16 + 4 i (i = 0, 1, ...)
// of K and of V, so each store instruction covers four whole rows.  The
// values and their rounding are those of k_materialize.
__global__ __launch_bounds__(256) void k_materialize16(Dims dm, Workspace ws, int sid, int n_active) {
  const int lane = threadIdx.x & 63;
  const int gw = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int u = gw / dm.K, p = gw % dm.K;
  if (u >= dm.units || p >= n_active) return;
  const size_t unit = (size_t)sid * dm.units + u;
  // S_k rows from row rb of the unit (variance-aware allocation), else S from p S
  const bool var = ws.ps_count != nullptr;
  const int S = var ? ws.ps_count[(size_t)u * dm.K + p] : dm.S;
  const size_t rb = var ? (size_t)ws.ps_off[(size_t)u * dm.K + p] : (size_t)p * dm.S;
  const int dq = lane & 15, r0 = lane >> 4;
  const int g = dq >> 1, hsub = (dq & 1) * 8;  // subspace of these 8 dims, offset inside it
  const uint8_t* row = ws.bank + (unit * dm.K + p) * ROW;
  const float nf = (float)reinterpret_cast<const RowMeta*>(row + ROW_META)->n;
  const uint32_t* codes = ws.pcodes + (((size_t)u * dm.K + p) * 2) * PCW;
  // rotary positions: the pseudo-keys turn at tau_k; this lane's dims are
  // pair indices 8 (dq % 8) + e, the partners in lane dq ^ 8
  const bool rope = ws.rope_inv != nullptr;
  float rc[8], rs[8];
  if (rope) {
    const double tau = (double)reinterpret_cast<const RowMeta*>(row + ROW_META)->tau;
#pragma unroll
    for (int e = 0; e < 8; ++e) rope_cs(tau, ws.rope_inv[8 * (dq & 7) + e], rc[e], rs[e]);
  }
  const float* cbk = ws.codebooks + unit * (2 * G * CMAX * DP);
  {
    const bool mb = (dm.flags & PROTOKV_FLAG_MASS_BIAS) != 0;
    const float bias = mb ? logf(nf) : 0.f;
    if (lane == 0) ws.pbias[(size_t)u * dm.K + p] = bias;
    if (var && lane < S) ws.prow_bias[(size_t)u * dm.K * dm.S + rb + lane] = bias;
  }
  // everything this lane needs first: its 8 dims of both sums, the no-residual
  // flags and the tuples of its rows
  float4 sr[2][2];
  uint32_t tup[2][SMAX / 4];
  bool nores[2];
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const float* sums = reinterpret_cast<const float*>(row + (w ? ROW_SUMV : ROW_SUMK)) + 8 * dq;
    sr[w][0] = reinterpret_cast<const float4*>(sums)[0];
    sr[w][1] = reinterpret_cast<const float4*>(sums)[1];
    const uint32_t* cw = codes + w * PCW;
    nores[w] = cw[SMAX] != 0u;
#pragma unroll
    for (int i = 0; i < SMAX / 4; ++i) {
      const int s2 = r0 + 4 * i;
      tup[w][i] = s2 < S ? cw[s2] : 0u;
    }
  }
  const int sh = 4 * (G - 1 - g);
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const float cd = (dm.flags & PROTOKV_FLAG_EMA_CENTRES) ? 1.f : nf;  // EMA centres are stored
    const float c[8] = {sr[w][0].x / cd, sr[w][0].y / cd, sr[w][0].z / cd, sr[w][0].w / cd,
                        sr[w][1].x / cd, sr[w][1].y / cd, sr[w][1].z / cd, sr[w][1].w / cd};
    const float* cbw = cbk + ((size_t)w * G + g) * CMAX * DP + hsub;
    uint8_t* out = (w ? ws.pv : ws.pk) + ((size_t)u * dm.K * dm.S + rb) * D * 2 + dq * 16;
#pragma unroll
    for (int i = 0; i < SMAX / 4; ++i) {
      const int s2 = r0 + 4 * i;
      if (s2 < S) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c[e];
        if (!nores[w]) {
          const int z = (tup[w][i] >> sh) & 15;
          const float4 a = reinterpret_cast<const float4*>(cbw + z * DP)[0];
          const float4 b = reinterpret_cast<const float4*>(cbw + z * DP)[1];
          v[0] = c[0] + a.x; v[1] = c[1] + a.y; v[2] = c[2] + a.z; v[3] = c[3] + a.w;
          v[4] = c[4] + b.x; v[5] = c[5] + b.y; v[6] = c[6] + b.z; v[7] = c[7] + b.w;
        }
        if (rope && w == 0) {  // rotate the key as rounded to bf16
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = q_from_bf16(q_to_bf16(v[e]));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float pv = __shfl_xor(v[e], 8, 64);
            float lo, hi;
            if (dq < 8) {
              rope_pair(v[e], pv, rc[e], rs[e], lo, hi);
              v[e] = lo;
            } else {
              rope_pair(pv, v[e], rc[e], rs[e], lo, hi);
              v[e] = hi;
            }
          }
        }
        uint4 o;
        o.x = (uint32_t)q_to_bf16(v[0]) | ((uint32_t)q_to_bf16(v[1]) << 16);
        o.y = (uint32_t)q_to_bf16(v[2]) | ((uint32_t)q_to_bf16(v[3]) << 16);
        o.z = (uint32_t)q_to_bf16(v[4]) | ((uint32_t)q_to_bf16(v[5]) << 16);
        o.w = (uint32_t)q_to_bf16(v[6]) | ((uint32_t)q_to_bf16(v[7]) << 16);
        *reinterpret_cast<uint4*>(out + (size_t)s2 * D * 2) = o;
      }
    }
  }
}

hipError_t launch_decode(const Dims& dm, const Workspace& ws, int sid, int n_active, bool centres, bool wide,
                         hipStream_t st) {
  if (n_active <= 0) return hipSuccess;
  const int bpu = (n_active + SYN_P - 1) / SYN_P;
  const size_t lds = (size_t)2 * dm.S * 64 * (3 * sizeof(uint64_t) + sizeof(uint32_t));
  const dim3 grid((unsigned)((dm.units * n_active + 63) / 64));  // 64 slots per workgroup
  if (dm.S <= 8) {
    hipLaunchKernelGGL(k_decode<8>, grid, dim3(256), 0, st, dm, ws, sid, n_active, centres ? 1 : 0);
    if (wide) hipLaunchKernelGGL(k_decode_wide<8>, dim3(dm.units * bpu), dim3(64), lds, st, dm, ws, sid, n_active, bpu);
  } else {
    hipLaunchKernelGGL(k_decode<16>, grid, dim3(256), 0, st, dm, ws, sid, n_active, centres ? 1 : 0);
    if (wide) hipLaunchKernelGGL(k_decode_wide<16>, dim3(dm.units * bpu), dim3(64), lds, st, dm, ws, sid, n_active, bpu);
  }
  return hipGetLastError();
}

// Eight consecutive KV elements at element offset e of `base` as float, and back.
template <int FP32>
__device__ __forceinline__ void ld8kv(const uint8_t* base, size_t e, float (&x)[8]) {
  if (FP32) {
    const float4 a = reinterpret_cast<const float4*>(base + e * 4)[0];
    const float4 b = reinterpret_cast<const float4*>(base + e * 4)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  } else {
    const uint4 w = *reinterpret_cast<const uint4*>(base + e * 2);
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[2 * q] = __uint_as_float(ww[q] << 16);
      x[2 * q + 1] = __uint_as_float(ww[q] & 0xFFFF0000u);
    }
  }
}
template <int FP32>
__device__ __forceinline__ void st8kv(uint8_t* base, size_t e, const float (&x)[8]) {
  if (FP32) {
    reinterpret_cast<float4*>(base + e * 4)[0] = make_float4(x[0], x[1], x[2], x[3]);
    reinterpret_cast<float4*>(base + e * 4)[1] = make_float4(x[4], x[5], x[6], x[7]);
  } else {
    uint4 o;
    o.x = (uint32_t)q_to_bf16(x[0]) | ((uint32_t)q_to_bf16(x[1]) << 16);
    o.y = (uint32_t)q_to_bf16(x[2]) | ((uint32_t)q_to_bf16(x[3]) << 16);
    o.z = (uint32_t)q_to_bf16(x[4]) | ((uint32_t)q_to_bf16(x[5]) << 16);
    o.w = (uint32_t)q_to_bf16(x[6]) | ((uint32_t)q_to_bf16(x[7]) << 16);
    *reinterpret_cast<uint4*>(base + e * 2) = o;
  }
}

// Rotates the rows of one token vector: pair indices [8 c, 8 c + 8) (dims
// 8c.. and D/2 + 8c..) of the row at element offset `e0`, at position pos.
template <int FP32>
__device__ __forceinline__ void rope_row8(const uint8_t* src, uint8_t* dst, size_t e0, int c, double pos,
                                          const double* inv) {
  float x1[8], x2[8], y1[8], y2[8];
  ld8kv<FP32>(src, e0 + 8 * c, x1);
  ld8kv<FP32>(src, e0 + D / 2 + 8 * c, x2);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float cs, sn;
    rope_cs(pos, inv[8 * c + e], cs, sn);
    rope_pair(x1[e], x2[e], cs, sn, y1[e], y2[e]);
  }
  st8kv<FP32>(dst, e0 + 8 * c, y1);
  st8kv<FP32>(dst, e0 + D / 2 + 8 * c, y2);
}

// The query [L][tq][Hq][D] rotated into qrot: thread = (row, pair block c);
// token t at position p0 + t.
template <int FP32>
__global__ __launch_bounds__(256) void k_rope_q(Dims dm, Workspace ws, const uint8_t* q, int tq, long long p0) {
  const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t row = gid >> 3;
  if (row >= (size_t)dm.L * tq * dm.Hq) return;
  const int c = (int)(gid & 7);
  const int t = (int)((row / dm.Hq) % tq);
  rope_row8<FP32>(q, ws.qrot, row * D, c, (double)(p0 + t), ws.rope_inv);
}

// Ring insert with rotary positions, in one pass: thread = (entry, unit,
// token j, pair block c) copies the token's K and V chunks [8c, 8c + 8) and
// [D/2 + 8c, D/2 + 8c + 8) into the ring and writes the K pair rotated at
// its stream position f * T + j into ring_kr.
template <int FP32>
__global__ __launch_bounds__(256) void k_ring_insert_rope(Dims dm, Workspace ws, AppendBatch ab,
                                                          const uint8_t* k, const uint8_t* v) {
  const size_t gid = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t per = (size_t)dm.units * dm.T * 8;
  const int e = (int)(gid / per);
  if (e >= ab.n) return;
  const size_t r = gid % per;
  const int c = (int)(r & 7), j = (int)((r >> 3) % dm.T), u = (int)((r >> 3) / dm.T);
  const size_t es = FP32 ? 4 : 2;
  const size_t s0 = (((size_t)e * dm.units + u) * dm.T + j) * (size_t)D;
  const size_t d0 = ((((size_t)ab.sid[e] * dm.units + u) * (dm.W + 1) + ab.slot[e]) * dm.T + j) * (size_t)D;
  constexpr int W16 = FP32 ? 2 : 1;  // 16-byte words per 8 elements
  uint4 ka[W16], kb[W16], va[W16], vb[W16];
#pragma unroll
  for (int w = 0; w < W16; ++w) {
    ka[w] = reinterpret_cast<const uint4*>(k + (s0 + 8 * c) * es)[w];
    kb[w] = reinterpret_cast<const uint4*>(k + (s0 + D / 2 + 8 * c) * es)[w];
    va[w] = reinterpret_cast<const uint4*>(v + (s0 + 8 * c) * es)[w];
    vb[w] = reinterpret_cast<const uint4*>(v + (s0 + D / 2 + 8 * c) * es)[w];
  }
#pragma unroll
  for (int w = 0; w < W16; ++w) {
    reinterpret_cast<uint4*>(ws.ring_k + (d0 + 8 * c) * es)[w] = ka[w];
    reinterpret_cast<uint4*>(ws.ring_k + (d0 + D / 2 + 8 * c) * es)[w] = kb[w];
    reinterpret_cast<uint4*>(ws.ring_v + (d0 + 8 * c) * es)[w] = va[w];
    reinterpret_cast<uint4*>(ws.ring_v + (d0 + D / 2 + 8 * c) * es)[w] = vb[w];
  }
  float x1[8], x2[8], y1[8], y2[8];
  ld8kv<FP32>(reinterpret_cast<const uint8_t*>(ka), 0, x1);
  ld8kv<FP32>(reinterpret_cast<const uint8_t*>(kb), 0, x2);
  const double pos = (double)ab.frame[e] * dm.T + j;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    float cs, sn;
    rope_cs(pos, ws.rope_inv[8 * c + q], cs, sn);
    rope_pair(x1[q], x2[q], cs, sn, y1[q], y2[q]);
  }
  st8kv<FP32>(ws.ring_kr, d0 + 8 * c, y1);
  st8kv<FP32>(ws.ring_kr, d0 + D / 2 + 8 * c, y2);
}

hipError_t launch_ring_insert_rope(const Dims& dm, const Workspace& ws, const AppendBatch& ab, const void* k,
                                   const void* v, hipStream_t st) {
  const size_t n = (size_t)ab.n * dm.units * dm.T * 8;
  const dim3 grid((unsigned)((n + 255) / 256));
  const uint8_t* kb = static_cast<const uint8_t*>(k);
  const uint8_t* vb = static_cast<const uint8_t*>(v);
  if (dm.kv_fp32)
    hipLaunchKernelGGL(k_ring_insert_rope<1>, grid, dim3(256), 0, st, dm, ws, ab, kb, vb);
  else
    hipLaunchKernelGGL(k_ring_insert_rope<0>, grid, dim3(256), 0, st, dm, ws, ab, kb, vb);
  return hipGetLastError();
}

hipError_t launch_rope_q(const Dims& dm, const Workspace& ws, const void* q, int tq, long long p0,
                         hipStream_t st) {
  const size_t n = (size_t)dm.L * tq * dm.Hq * 8;
  const dim3 grid((unsigned)((n + 255) / 256));
  const uint8_t* qb = static_cast<const uint8_t*>(q);
  if (dm.kv_fp32)
    hipLaunchKernelGGL(k_rope_q<1>, grid, dim3(256), 0, st, dm, ws, qb, tq, p0);
  else
    hipLaunchKernelGGL(k_rope_q<0>, grid, dim3(256), 0, st, dm, ws, qb, tq, p0);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Variance-aware pseudo-token counts (appendix "Dynamic Pseudo-Token
// Allocation"), in float64 with every sum in the order the definition gives it.
// k_alloc_var: Var(H_k), 16 lanes per slot, one per (side, subspace), codewords
// and dims ascending; the sixteen terms are then added in order.  k_alloc:
// workgroup = one (layer, kv head); the sums over slots run in slot order in one
// wave (water-filling of the shares over the cap, then cumulative rounding), their
// operands read from LDS ahead of the chain of additions; the shares are computed
// by all threads.  With one thread per slot for the variances and one thread
// reading and adding slot by slot, 6 units x 333 slots took 210 us; now 27 (the
// chains of additions are 20 of them).
// ---------------------------------------------------------------------------
constexpr int AV_STRIDE = CMAX * DP + 4;  // floats per (side, subspace) in LDS: 16 of them on 16 different bank quads

__global__ __launch_bounds__(256) void k_alloc_var(Dims dm, Workspace ws, int sid, int A, int blocks_per_unit) {
  __shared__ __attribute__((aligned(16))) float s_cb[2 * G * AV_STRIDE];
  __shared__ double s_n2[2 * G][CMAX + 1];
  const int tid = threadIdx.x;
  const int u = blockIdx.x / blocks_per_unit, blk = blockIdx.x % blocks_per_unit;
  const size_t unit = (size_t)sid * dm.units + u;
  const float* cbk = ws.codebooks + unit * (2 * G * CMAX * DP);
  for (int i = tid; i < 2 * G * CMAX * DP; i += 256) s_cb[(i >> 8) * AV_STRIDE + (i & 255)] = cbk[i];
  __syncthreads();
  {
    double n2 = 0.0;
#pragma unroll
    for (int d = 0; d < DP; ++d) {
      const double c = (double)s_cb[(tid >> 4) * AV_STRIDE + (tid & 15) * DP + d];
      n2 = n2 + c * c;
    }
    s_n2[tid >> 4][tid & 15] = n2;
  }
  __syncthreads();
  const int sg = tid & 15, lane0 = (tid & 63) & ~15;
  const float* cb = s_cb + sg * AV_STRIDE;
  // 16 slots per pass; every lane of a group runs the same passes
  for (int k = blk * 16 + (tid >> 4); k < A; k += blocks_per_unit * 16) {
    const uint8_t* row = ws.bank + (unit * dm.K + k) * ROW;
    const uint32_t nres = reinterpret_cast<const RowMeta*>(row + ROW_META)->n_res;
    const double den = (double)nres;
    uint32_t h[CMAX];  // K's subspaces, then V's (the histograms are adjacent)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint4 x = reinterpret_cast<const uint4*>(row + ROW_HK + sg * CMAX * 4)[v];
      h[4 * v] = x.x; h[4 * v + 1] = x.y; h[4 * v + 2] = x.z; h[4 * v + 3] = x.w;
    }
    double e2 = 0.0, mean[DP];
#pragma unroll
    for (int d = 0; d < DP; ++d) mean[d] = 0.0;
#pragma unroll
    for (int c = 0; c < CMAX; ++c) {
      if (c < dm.C) {  // uniform
        const double pc = (double)h[c] / den;
        e2 = e2 + pc * s_n2[sg][c];
#pragma unroll
        for (int d = 0; d < DP; ++d) mean[d] = mean[d] + pc * (double)cb[c * DP + d];
      }
    }
    double m2 = 0.0;
#pragma unroll
    for (int d = 0; d < DP; ++d) m2 = m2 + mean[d] * mean[d];
    const double x = e2 - m2, v = x > 0.0 ? x : 0.0;
    double total = 0.0;
#pragma unroll
    for (int i = 0; i < 2 * G; ++i) total = total + __shfl(v, lane0 + i, 64);
    if (sg == 0) ws.ps_var[(size_t)u * dm.K + k] = nres > 0 ? total : 0.0;
  }
}

// Sums a[0..n) in order, n a multiple of 16 (LDS, the tail zeros), and calls
// each(k, sum up to and with k).  One wave, every lane the same.
template <typename F>
__device__ __forceinline__ double sum_in_order(const double* a, int n, F each) {
  double next[16], acc = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) next[i] = a[i];
  for (int k = 0; k < n; k += 16) {
    double cur[16];
    const int kn = min(k + 16, n - 16);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      cur[i] = next[i];
      next[i] = a[kn + i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      acc = acc + cur[i];
      each(k + i, acc);
    }
  }
  return acc;
}

__global__ __launch_bounds__(256) void k_alloc(Dims dm, Workspace ws, int sid, int A) {
  __shared__ __attribute__((aligned(16))) double s_var[AL_KMAX];  // 0 once capped
  __shared__ __attribute__((aligned(16))) double s_x[AL_KMAX];
  __shared__ uint8_t s_cap[AL_KMAX];
  __shared__ double s_w;
  __shared__ int s_ncap, s_total;
  const int tid = threadIdx.x, u = blockIdx.x, lane = tid & 63;
  const int S = dm.S, smax = dm.pseudo_max, A64 = (A + 63) & ~63;
  for (int k = tid; k < A64; k += 256) {
    s_var[k] = k < A ? ws.ps_var[(size_t)u * dm.K + k] : 0.0;
    s_cap[k] = 0;
    s_x[k] = 0.0;
  }
  if (tid == 0) s_ncap = 0;
  int32_t* cnt = ws.ps_count + (size_t)u * dm.K;
  int32_t* off = ws.ps_off + (size_t)u * dm.K;
  __syncthreads();
  const int tot = A * S;
  bool novar = false;
  for (int ncap = 0, pass = 0;; ++pass) {  // uniform
    if (tid < 64) {
      const double w = sum_in_order(s_var, A64, [](int, double) {});
      if (tid == 0) s_w = w;
    }
    __syncthreads();
    const double w = s_w, rest = (double)(tot - A - ncap * (smax - 1)), nunc = (double)(A - ncap);
    if (pass == 0 && w == 0.0) {  // no variance at all: every S_k = S
      novar = true;
      break;
    }
    for (int k = tid; k < A; k += 256) {
      double x;
      if (s_cap[k]) x = (double)smax;
      else if (w > 0.0) x = 1.0 + rest * s_var[k] / w;
      else x = 1.0 + rest / nunc;
      s_x[k] = x;
      if (!s_cap[k] && x > (double)smax) {
        s_cap[k] = 1;
        s_var[k] = 0.0;
        atomicAdd(&s_ncap, 1);
      }
    }
    __syncthreads();
    const int now = s_ncap;
    __syncthreads();
    if (now == ncap) break;
    ncap = now;
  }
  if (tid < 64) {
    // cumulative rounding: S_k = floor(X_k + 1/2) - floor(X_(k-1) + 1/2)
    int prev = 0;
    double mine = 0.0;
    if (novar) {
      prev = tot;
    } else {
      sum_in_order(s_x, A64, [&](int k, double X) {
        mine = (k & 63) == lane ? X : mine;
        if ((k & 63) == 63) {  // uniform: 64 slots done, lane i holds X of slot k - 63 + i
          const int cur = (int)floor(mine + 0.5);
          int before = __shfl_up(cur, 1, 64);
          if (lane == 0) before = prev;
          const int slot = k - 63 + lane;
          if (slot < A) {
            off[slot] = before;
            cnt[slot] = cur - before;
          }
          prev = __shfl(cur, 63, 64);
        }
      });
    }
    if (tid == 0) s_total = prev;
  }
  __syncthreads();
  for (int k = tid; k < dm.K; k += 256) {
    if (k >= A) {
      cnt[k] = 0;
      off[k] = s_total;
    } else if (novar) {
      cnt[k] = S;
      off[k] = k * S;
    }
  }
}

hipError_t launch_alloc(const Dims& dm, const Workspace& ws, int sid, int n_active, hipStream_t st) {
  if (n_active > 0) {
    // about 2048 workgroups, each staging its unit's codebooks once
    const int bpu = std::max(1, std::min((n_active + 15) / 16, 2048 / dm.units));
    hipLaunchKernelGGL(k_alloc_var, dim3(dm.units * bpu), dim3(256), 0, st, dm, ws, sid, n_active, bpu);
  }
  hipLaunchKernelGGL(k_alloc, dim3(dm.units), dim3(256), 0, st, dm, ws, sid, n_active);
  return hipGetLastError();
}

hipError_t launch_materialize(const Dims& dm, const Workspace& ws, int sid, int n_active, hipStream_t st) {
  if (n_active <= 0) return hipSuccess;
  const int waves = dm.units * dm.K;
  if (dm.kv_fp32)
    hipLaunchKernelGGL(k_materialize<1>, dim3((waves + 3) / 4), dim3(256), 0, st, dm, ws, sid, n_active);
  else
    hipLaunchKernelGGL(k_materialize16, dim3((waves + 3) / 4), dim3(256), 0, st, dm, ws, sid, n_active);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Readout.  Context of kv head u: near tokens (frames f_first.. in ring
// slots f mod (W+1)), then pseudo-tokens; logit = q.k/sqrt(D) + bias with
// bias 0 on near tokens and log n_k on the pseudo-tokens of slot k.
// Query rows of one kv head: r = t * (Hq/Hkv) + g  (query head u_h*grp + g).
// ---------------------------------------------------------------------------
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float SQRT_D = 11.313708498984761f;  // a logit in units of q.k

// bf16 path.  Workgroup = eight waves for one (kv head, context split,
// block of query rows): one wave per 32 rows for up to 256 rows (KH = 1), or
// for at most 128 rows two waves per 32 rows, each taking one 32-key half
// of every tile, their results merged at the end (KH = 2), so each SIMD
// runs two waves either way.  A context tile of 64
// keys sits in LDS in two layouts under which every operand read is a per-lane
// base plus compile-time offsets and touches distinct banks:
//   K chunk-major: 16-byte chunk c (dims 8c .. 8c+7) of row r at c * 1024 + r * 16;
//   V by 32-dim block: dims 32b .. 32b+31 of row r at b * 4096 + r * 64.
// Near-window tiles go straight from global memory into these layouts
// (global_load_lds_dwordx4), three tiles ahead of the one computed.
// S^T = K Q^T and O^T = V^T P with v_mfma_f32_32x32x16_bf16; the V^T operand
// comes through ds_read_b64_tr_b16.  Each lane holds one query column, so the
// online softmax is lane-local plus one exchange with the partner lane.  With
// several splits, every workgroup writes its partial (unnormalised O, running
// max, sum) for k_attend_merge.
constexpr int AT_KEYS = 64;
constexpr int AT_ROWS = 256;  // query rows per workgroup
constexpr int AT_TILE_BYTES = AT_KEYS * D * 2;   // one K or V tile, 16 KB

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// Barrier for LDS traffic only: waits for this wave's LDS operations, not
// for its outstanding global loads (the tiles in flight).  The asm memory
// clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  asm volatile("s_barrier" ::: "memory");
}
constexpr int A32_CW = 80;        // bytes from codeword to codeword in LDS (16 of padding: 16 of them on 16 different bank quads)
constexpr int AT_NBUF = 4;        // tile buffers: tile t computes while t+1..t+3 load
constexpr int AT_NTAB = 5;        // row-table entries (written 3 tiles ahead)
constexpr int AT_PB_MAX = 2048;   // pseudo-token biases staged in LDS up to this capacity

template <int NW, int KH>
__global__ __launch_bounds__(NW * 64, 1) void k_attend_bf16(Dims dm, Workspace ws, AttendArgs aa, int rows, int rblocks) {
  constexpr int LPT = 32 / NW;  // load instructions per wave per tile
  constexpr int RPW = NW * 32 / KH;  // query rows per workgroup
  __shared__ __attribute__((aligned(16))) uint8_t s_kv[AT_NBUF][2][AT_TILE_BYTES];   // [buffer][K,V]
  __shared__ __attribute__((aligned(16))) float s_bias[AT_NTAB][AT_KEYS];           // bias in units of q.k, -inf past the context
  __shared__ const uint8_t* s_rowp[AT_NTAB][2][AT_KEYS];                             // K and V address of each tile row
  __shared__ float s_pb[AT_PB_MAX];                                                  // ln n_k of this unit in units of q.k
  // rotary positions: (cos, sin) of tau_k * theta^(-2i/D) for the slots of
  // a formed tile, two tiles' tables (the next one's is written ahead)
  __shared__ float2 s_rtab[2][PS_SLOTS][D / 2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // blocks of one kv head land on one XCD (dispatch is round-robin over 8)
  const int nblk = gridDim.x, per = nblk / 8;
  const int lbid = (int)blockIdx.x < per * 8 ? ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8 : (int)blockIdx.x;
  const int split = lbid % aa.splits;
  const int rb = (lbid / aa.splits) % rblocks;
  const int u = lbid / (aa.splits * rblocks);
  const size_t unit = (size_t)aa.sid * dm.units + u;
  const int grp = dm.Hq / dm.Hkv;
  const int l = u / dm.Hkv, kvh = u % dm.Hkv;
  const int ctx = aa.n_near + aa.n_far;
  // rows [c0, c1n) stream through LDS by DMA: with aa.gen the split's share
  // of the near window (the pseudo-token rows [ps0, ps1) of its share are
  // formed in LDS from the synthesized centres, decode records and
  // codebooks), else context rows [c0, c1) of the near window followed by
  // the written pseudo-token rows
  const int c0 = aa.gen ? min(aa.n_near, split * aa.near_chunk) : split * aa.chunk;
  const int c1n = aa.gen ? min(aa.n_near, c0 + aa.near_chunk) : min(ctx, c0 + aa.chunk);
  const int ntiles = c1n > c0 ? (c1n - c0 + AT_KEYS - 1) / AT_KEYS : 0;
  const bool pb_lds = dm.K <= AT_PB_MAX;
  if (pb_lds)
    for (int k = tid; k < dm.K; k += NW * 64) s_pb[k] = ws.pbias[(size_t)u * dm.K + k] * SQRT_D;

  const int col = lane & 31, half = lane >> 5;
  // KH = 2: waves w and w + NW / 2 take the same 32 query rows and the two
  // 32-key halves of every tile
  const int rblk = KH == 2 ? wave % (NW / 2) : wave, kh = KH == 2 ? wave / (NW / 2) : 0;
  const int r = rb * RPW + rblk * 32 + col;  // query row of this lane
  const bool rvalid = r < rows;
  const bool wvalid = rb * RPW + rblk * 32 < rows;  // uniform: the wave has query rows
  bf16x8 bq[8];
  {
    const int t = rvalid ? r / grp : 0, gg = rvalid ? r % grp : 0;
    const uint16_t* qr = reinterpret_cast<const uint16_t*>(aa.q) +
                         ((((size_t)l * aa.tq + t) * dm.Hq + kvh * grp + gg) * D);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      u16x8 v = *reinterpret_cast<const u16x8*>(qr + kk * 16 + half * 8);
      if (!rvalid) v = (u16x8)0;
      bq[kk] = __builtin_bit_cast(bf16x8, v);
    }
  }
  __syncthreads();  // s_pb staged (and the query loads complete)

  // Per-tile row table: wave 0 resolves each tile row (one lane per row) to its
  // K and V addresses and its bias once, three tiles ahead.  Rows past the
  // context read row c0 and carry bias -inf.
  const float invS = 1.0f / (float)dm.S;
  auto resolve = [&](int t, const uint8_t*& kp, const uint8_t*& vp, float& bv) {
    const int idx = c0 + t * AT_KEYS + lane;
    const int pos = idx < c1n ? idx : c0;
    bv = idx < c1n ? 0.f : -INFINITY;
    if (pos < aa.n_near) {
      const int fo = pos / dm.T;
      const int slot = (aa.f_first + fo) % (dm.W + 1);
      const size_t off = (((unit * (dm.W + 1) + slot) * dm.T + (pos - fo * dm.T)) * (size_t)D) * 2;
      kp = aa.near_k + off;
      vp = ws.ring_v + off;
    } else {
      const int prow = pos - aa.n_near;
      const size_t off = (((size_t)u * dm.K * dm.S + prow) * (size_t)D) * 2;
      kp = ws.pk + off;
      vp = ws.pv + off;
      if (aa.rowbias) {
        if (idx < c1n) bv = aa.rowbias[(size_t)u * dm.K * dm.S + prow] * SQRT_D;
      } else {
        int k = (int)((float)prow * invS);
        k -= k * dm.S > prow ? 1 : 0;
        k += (k + 1) * dm.S <= prow ? 1 : 0;
        if (idx < c1n) bv = pb_lds ? s_pb[k] : ws.pbias[(size_t)u * dm.K + k] * SQRT_D;
      }
    }
  };
  auto publish = [&](int t, const uint8_t* kp, const uint8_t* vp, float bv) {
    const int e = t % AT_NTAB;
    s_rowp[e][0][lane] = kp;
    s_rowp[e][1][lane] = vp;
    s_bias[e][lane] = bv;
  };
  // Loads of tile t into LDS buffer t % AT_NBUF: instruction i = wave + q * NW
  // (q < LPT) moves 1 KiB, K chunk i of all 64 rows (lane = row) for i < 16,
  // else V block j = i - 16: dims 32 (j / 4) .. +31 of rows 16 (j % 4) ..
  // +15 (lane / 4 = row, lane % 4 = 16-byte part).
  auto issue = [&](int t) {
    const int e = t % AT_NTAB, buf = t % AT_NBUF;
#pragma unroll
    for (int q = 0; q < LPT; ++q) {
      const int i = wave + q * NW;  // uniform
      const uint8_t* src;
      if (i < 16) {
        src = s_rowp[e][0][lane] + i * 16;
      } else {
        const int j = i - 16;
        src = s_rowp[e][1][(j & 3) * 16 + (lane >> 2)] + ((j >> 2) * 4 + (lane & 3)) * 16;
      }
      lds_dma16(src, &s_kv[buf][i >> 4][(i & 15) * 1024]);
    }
  };

  const float scale = LOG2E / sqrtf((float)D);
  f32x16 oacc[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) oacc[b] = (f32x16){0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // Reference max (log2 units) with a finite floor: masked keys score -inf and
  // give exp2(-inf) = 0 without special cases.  The reference is raised only
  // when a row's max exceeds it by more than 8, so p <= 2^8 and the output
  // accumulators are rescaled rarely.
  float mref = -1e30f, lrun = 0.f;

  // per-lane operand bases: K row h*32 + col, chunk 2 kk + half at
  // koff + kk * 2048 + h * 512; V (transposed reads, see below) at
  // voff + b * 4096 + st * 1024 (+ 512 for keys 8 .. 15 of the step)
  const int grp16 = lane >> 4, s16 = lane & 15;
  const int koff = half * 1024 + col * 16;
  const int voff = (4 * half + (s16 >> 2)) * 64 + (grp16 & 1) * 32 + (s16 & 3) * 8;
  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // one 64-key tile in LDS (K at kt, V at vt): S^T = K Q^T, online softmax,
  // O^T += V^T P.  BIAS: the products start from the keys' biases (the tile's
  // bias entries, in units of q.k); a full tile of near-window keys starts
  // from 0.
  auto compute_tile = [&](const uint8_t* kt, const uint8_t* vt, int tb, auto bias_tag) {
    constexpr bool BIAS = decltype(bias_tag)::value;
    const uint8_t* kl = kt + koff;
    const uint8_t* vl = vt + voff;
    // S^T for the wave's 32-key halves of the tile (both, or half kh)
    constexpr int NH = 2 / KH;
    f32x16 sacc[NH];
  #pragma unroll
    for (int hh = 0; hh < NH; ++hh) {
      const int h = KH == 2 ? kh : hh;
      sacc[hh] = (f32x16){0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if constexpr (BIAS) {
        // element i is key h * 32 + (i / 4) * 8 + half * 4 + i % 4
  #pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const float4 bb = *reinterpret_cast<const float4*>(&s_bias[tb][h * 32 + i4 * 8 + half * 4]);
          sacc[hh][i4 * 4] = bb.x;
          sacc[hh][i4 * 4 + 1] = bb.y;
          sacc[hh][i4 * 4 + 2] = bb.z;
          sacc[hh][i4 * 4 + 3] = bb.w;
        }
      }
  #pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        const bf16x8 ak = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(kl + kk * 2048 + h * 512));
        sacc[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak, bq[kk], sacc[hh], 0, 0, 0);
      }
    }
    // V operands read before the softmax (their LDS latency under its
    // arithmetic): all of a half tile's, or the first of four 32-dim blocks
    constexpr int VP = KH == 2 ? 4 : 1;
    v8i16 va[4][2 * NH];
    auto read_v = [&](int b) {
  #pragma unroll
      for (int st = 0; st < 2 * NH; ++st) {
        const int sk = KH == 2 ? 2 * kh + st : st;  // 16-key step of the tile
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vl + b * 4096 + sk * 1024));
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vl + b * 4096 + sk * 1024 + 512));
        va[b][st] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    };
  #pragma unroll
    for (int b = 0; b < VP; ++b) read_v(b);
    __builtin_amdgcn_sched_barrier(0);
    float tmax = -1e30f;
  #pragma unroll
    for (int hh = 0; hh < NH; ++hh)
  #pragma unroll
      for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, sacc[hh][i]);
    tmax = fmaxf(tmax, xor32(tmax)) * scale;
    // the reference moves up only when a row's max exceeds it by more than 8
    const bool grow = tmax > mref + 8.0f;
    if (__ballot(grow)) {  // uniform
      const float mnew = grow ? tmax : mref;
      const float alpha = __builtin_amdgcn_exp2f(mref - mnew);
      lrun *= alpha;
  #pragma unroll
      for (int b = 0; b < 4; ++b)
  #pragma unroll
        for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
      mref = mnew;
    }
    const float nm = -mref;
    // P in bf16; the row sum is taken over the rounded values the products use
    bf16x8 pb[2 * NH];
  #pragma unroll
    for (int hh = 0; hh < NH; ++hh)
  #pragma unroll
      for (int i = 0; i < 16; ++i)
        pb[2 * hh + (i >> 3)][i & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sacc[hh][i], scale, nm));
    float sum0 = 0.f, sum1 = 0.f;
  #pragma unroll
    for (int j = 0; j < 2 * NH; ++j) {
      sum0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 0, 1), ones2, sum0, false);
      sum1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 2, 3), ones2, sum1, false);
      sum0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 4, 5), ones2, sum0, false);
      sum1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 6, 7), ones2, sum1, false);
    }
    float psum = sum0 + sum1;
    psum += xor32(psum);
    lrun += psum;
    // O^T = V^T P.  k positions half*8 + i of step st <-> keys 16 st + 4 half + {0..3}
    // (i < 4) and 16 st + 8 + 4 half + {0..3} (i >= 4), matching P's layout.  Each
    // 4-key part is one ds_read_b64_tr_b16 per 16-lane group: source lane s reads
    // key key0 + s/4, dims d0 + 4(s%4) .. +3 (d0 = 32 b + 16 (lane/16 % 2)); lane i
    // then holds dim d0 + i of the 4 keys.
  #pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (b + VP < 4) read_v(b + VP);
  #pragma unroll
      for (int st = 0; st < 2 * NH; ++st)
        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va[b][st]), pb[st], oacc[b], 0, 0, 0);
    }
  };

  // prologue: rows of tiles 0..2 published, their loads issued; tile 3 resolved
  const uint8_t *nk = nullptr, *nv = nullptr;
  float nb = -INFINITY;
  if (wave == 0) {
    for (int t = 0; t < 3 && t < ntiles; ++t) {
      resolve(t, nk, nv, nb);
      publish(t, nk, nv, nb);
    }
    if (ntiles > 3) resolve(3, nk, nv, nb);
  }
  wait_vm<0>();  // the query operands are in registers before any tile is in flight
  lds_barrier();
  for (int t = 0; t < 3 && t < ntiles; ++t) issue(t);

  for (int t = 0; t < ntiles; ++t) {
    const int buf = t % AT_NBUF, tb = t % AT_NTAB;
    // this wave's loads of tile t have landed; tiles t+1, t+2 may still be in flight
    if (t + 2 < ntiles) wait_vm<2 * LPT>();
    else if (t + 1 < ntiles) wait_vm<LPT>();
    else wait_vm<0>();
    // entry (t + 3) % 5 was last read for tile t - 2 (before the previous barrier)
    if (wave == 0 && t + 3 < ntiles) publish(t + 3, nk, nv, nb);
    lds_barrier();
    // buffer (t + 3) % 4 held tile t - 1, finished by every wave before this barrier
    if (t + 3 < ntiles) issue(t + 3);
    if (wave == 0 && t + 4 < ntiles) resolve(t + 4, nk, nv, nb);
    if (!wvalid) continue;  // uniform: a loader-only wave
    // a full tile of near-window keys has all biases 0
    if (c0 + (t + 1) * AT_KEYS <= min(c1n, aa.n_near))
      compute_tile(s_kv[buf][0], s_kv[buf][1], tb, std::false_type{});
    else
      compute_tile(s_kv[buf][0], s_kv[buf][1], tb, std::true_type{});
  }

  // Pseudo-token tiles formed in LDS (aa.gen): row (k, s) of K is
  // bf16(c_k + concat_g C^K_g[z_{s,g}]) (c_k alone when the slot has no
  // residual), the values k_materialize writes; likewise V.  A tile is 64 / S
  // whole slots, so that a thread's row belongs to the same slot of every tile
  // and everything it derives from its row (centre, tuple, codebook and store
  // addresses) is computed once (tiles of 64 rows across slots, derived anew for
  // every 16 bytes: high resolution 740 us against 614, 448 rows over K = 1024
  // 507 against 443, 7B 95 against 89; that is S = 8, where no row stays empty.
  // Least is left of it at S = 11, 55 rows a tile: 448 rows over K = 1024, before
  // whole slots and with all that has changed since, 600 -> 586, at S = 13 694 -> 657).  The inputs of a tile (the
  // bank rows' float32 sums, 1 KiB per slot, and decode records of its slots)
  // go by DMA into one of three staging buffers three tiles ahead; two tiles
  // ahead the sums are turned into centres in place.  Iteration t: wait for
  // tile t+2's inputs, barrier, issue tile t+3's, convert tile t+2's, form tile
  // t+1 into buffer (t+1) % 2, compute tile t: the forming of the next tile
  // overlaps the MFMA work of the current one.
  // LDS: buffers 0, 1 the formed tiles, buffers 2 and 3 the unit's codebooks
  // and the staging buffers.  Slots at PS_CS and codewords at A32_CW bytes from
  // each other: lanes reading one part of different ones hit different banks.
  const int nsl = 64 / dm.S;
  const int nact = aa.n_far / dm.S;
  const int ks0 = min(nact, split * aa.far_slots), ks1 = min(nact, ks0 + aa.far_slots);
  const int npt = aa.gen && ks1 > ks0 ? (ks1 - ks0 + nsl - 1) / nsl : 0;
  if (npt > 0) {  // uniform
    constexpr int PS_CS = 1024 + 32;                    // bytes of one slot's centres, K then V (32 of padding)
    constexpr int PS_REC = PS_SLOTS * PS_CS;            // records at this offset of a stage
    constexpr int PS_STAGE = PS_REC + 2 * 1024;
    constexpr int CB_BYTES = 2 * G * CMAX * A32_CW;
    static_assert(NW == 8, "a thread forms one row's chunks c and c + 8 of K and of V");
    static_assert(2 * PCW * 4 * PS_SLOTS <= 2 * 1024 && CB_BYTES + 3 * PS_STAGE <= 4 * AT_TILE_BYTES, "LDS layout");
    static_assert(CB_BYTES % 1024 == 0 && PS_STAGE % 16 == 0, "DMA of whole KiB to 16-byte places");
    const int S = dm.S;
    uint8_t* s_cbb = s_kv[2][0];
    uint8_t* s_stage = s_cbb + CB_BYTES;
    const size_t ubase = (size_t)u * dm.K;
    auto stage = [&](int t) {
      const int k0 = ks0 + t * nsl, nk = min(nsl, ks1 - k0);
      uint8_t* sb = s_stage + (t % 3) * PS_STAGE;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int i = wave + q * NW;  // uniform: 0 .. PS_SLOTS - 1 sums, then two of records
        if (i < nsl) {
          // slots past the split's last repeat it
          lds_dma16(ws.bank + (unit * dm.K + k0 + min(i, nk - 1)) * ROW + ROW_SUMK + lane * 16, sb + i * PS_CS);
        } else if (i >= PS_SLOTS && i < PS_SLOTS + 2) {
          // past the last slot: its last 16 bytes (n in their last word)
          const int ch = min((i - PS_SLOTS) * 64 + lane, nk * (2 * PCW / 4) - 1);
          lds_dma16(reinterpret_cast<const uint8_t*>(ws.pcodes + (ubase + k0) * 2 * PCW) + ch * 16,
                    sb + PS_REC + (i - PS_SLOTS) * 1024);
        }
      }
    };
    // The staged sums of tile t's slots become their float32 centres
    // sum / n (IEEE division; EMA centres are stored as such) in place, n
    // from the staged value records.
    const bool ema = (dm.flags & PROTOKV_FLAG_EMA_CENTRES) != 0;
    auto convert = [&](int t) {
      const int nk = min(nsl, ks1 - ks0 - t * nsl);
      uint8_t* sb = s_stage + (t % 3) * PS_STAGE;
      const uint32_t* recs = reinterpret_cast<const uint32_t*>(sb + PS_REC);
      if (ema) return;
      for (int i = wave; i < nk; i += NW) {  // uniform
        float4* c4 = reinterpret_cast<float4*>(sb + i * PS_CS) + lane;
        const float nf = (float)recs[(i * 2 + 1) * PCW + SMAX + 1];
        const float4 v = *c4;
        *c4 = make_float4(v.x / nf, v.y / nf, v.z / nf, v.w / nf);
      }
    };
    // Tile t from stage t % 3 into buffer t % 2, in the layouts of the near
    // tiles: a thread forms K row tid % 64, chunks tid / 64 and + 8 (dims i
    // and i + D / 2: with rotary positions each key, rounded to bf16 as
    // written, is turned at tau_k in registers, with the roundings of
    // k_materialize16, and rounded again), and V row tid / 4 % 64, chunks
    // 4 (tid / 256) + tid % 4 and + 8: each store instruction writes 1 KiB
    // contiguous per wave.
    const bool rope = ws.rope_inv != nullptr;  // uniform
    struct Mine {
      int row, j, cen, tup, flag, cw, shift;  // byte offsets in a stage and in the codebooks
    } mine[2];
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
      const int row = kv ? (tid >> 2) & 63 : tid & 63;
      const int chunk = kv ? 4 * (tid >> 8) + (tid & 3) : tid >> 6;
      const int j = min(row / S, nsl - 1), s2 = min(row - j * S, S - 1), g = chunk >> 1;
      mine[kv].row = row;
      mine[kv].j = j;
      mine[kv].cen = j * PS_CS + kv * 512 + chunk * 32;
      mine[kv].tup = PS_REC + ((j * 2 + kv) * PCW + s2) * 4;
      mine[kv].flag = PS_REC + ((j * 2 + kv) * PCW + SMAX) * 4;
      mine[kv].cw = (kv * G + g) * CMAX * A32_CW + (chunk & 1) * 32;
      mine[kv].shift = 4 * (G - 1 - g);
    }
    auto form = [&](int t) {
      const int k0 = ks0 + t * nsl;
      const uint8_t* sb = s_stage + (t % 3) * PS_STAGE;
      const int pb = t & 1;
      const bool tail = nsl * S < 64 || k0 + nsl > ks1;  // uniform: rows past the tile's slots
      // 8 values at centre c, codeword w: exactly c + w or (m 0) c
      auto values = [](const uint8_t* c, const uint8_t* w, float m, float (&x)[8]) {
        const float4 ca = reinterpret_cast<const float4*>(c)[0], cb = reinterpret_cast<const float4*>(c)[1];
        const float4 wa = reinterpret_cast<const float4*>(w)[0], wb = reinterpret_cast<const float4*>(w)[1];
        x[0] = fmaf(wa.x, m, ca.x); x[1] = fmaf(wa.y, m, ca.y); x[2] = fmaf(wa.z, m, ca.z); x[3] = fmaf(wa.w, m, ca.w);
        x[4] = fmaf(wb.x, m, cb.x); x[5] = fmaf(wb.y, m, cb.y); x[6] = fmaf(wb.z, m, cb.z); x[7] = fmaf(wb.w, m, cb.w);
      };
      auto store8 = [&](int kv, int e, const float (&x)[8]) {
        const bf16x2 o0 = {(__bf16)x[0], (__bf16)x[1]}, o1 = {(__bf16)x[2], (__bf16)x[3]};
        const bf16x2 o2 = {(__bf16)x[4], (__bf16)x[5]}, o3 = {(__bf16)x[6], (__bf16)x[7]};
        *reinterpret_cast<uint4*>(s_kv[pb][kv] + (tid + e * 512) * 16) =
            make_uint4(__builtin_bit_cast(uint32_t, o0), __builtin_bit_cast(uint32_t, o1),
                       __builtin_bit_cast(uint32_t, o2), __builtin_bit_cast(uint32_t, o3));
      };
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        const Mine& mn = mine[kv];
        const uint32_t tup = *reinterpret_cast<const uint32_t*>(sb + mn.tup) >> mn.shift;  // chunk's nibble lowest
        const uint32_t tup8 = *reinterpret_cast<const uint32_t*>(sb + mn.tup) >> (mn.shift - 16);  // chunk + 8's
        const float m = *reinterpret_cast<const uint32_t*>(sb + mn.flag) != 0u ? 0.f : 1.f;  // no residual: the centre alone
        float xl[8], xh[8];
        values(sb + mn.cen, s_cbb + mn.cw + (tup & 15) * A32_CW, m, xl);
        values(sb + mn.cen + 256, s_cbb + mn.cw + 4 * CMAX * A32_CW + (tup8 & 15) * A32_CW, m, xh);
        const bool ok = mn.row < nsl * S && k0 + mn.j < ks1;
        if (kv == 0 && rope) {
          const float4* cs = reinterpret_cast<const float4*>(&s_rtab[pb][mn.j][8 * (tid >> 6)]);
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2) {
            const float4 a = cs[i2];  // (cos, sin) of two pair indices
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int i = 2 * i2 + h;
              const float c = h ? a.z : a.x, sn = h ? a.w : a.y;
              const float x1 = (float)(__bf16)xl[i], x2 = (float)(__bf16)xh[i];
              float lo, hi;
              rope_pair(x1, x2, c, sn, lo, hi);
              xl[i] = lo;
              xh[i] = hi;
            }
          }
        }
        if (tail) {  // score -inf and weight 0, but unwritten centres or rotation tables may hold inf or NaN
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            xl[i] = ok ? xl[i] : 0.f;
            xh[i] = ok ? xh[i] : 0.f;
          }
        }
        store8(kv, 0, xl);
        store8(kv, 1, xh);
        if (kv == 0 && tid < AT_KEYS) {  // row == tid
          const int k = min(k0 + mn.j, ks1 - 1);
          s_bias[pb][tid] = ok ? (pb_lds ? s_pb[k] : ws.pbias[ubase + k] * SQRT_D) : -INFINITY;
        }
      }
    };
    // (cos, sin) table of tile t's slots from tau_k in the staged key
    // records (stage t % 3), into table t % 2: lane = pair index
    const double rinv = rope ? ws.rope_inv[lane] : 0.0;
    auto rtab = [&](int t) {
      const int nk = min(nsl, ks1 - ks0 - t * nsl);
      const uint32_t* recs = reinterpret_cast<const uint32_t*>(s_stage + (t % 3) * PS_STAGE + PS_REC);
      for (int i = wave; i < nk; i += NW) {  // uniform
        const double tau = (double)(int32_t)recs[i * 2 * PCW + SMAX + 1];
        float c, sn;
        rope_cs(tau, rinv, c, sn);
        s_rtab[t & 1][i][lane] = make_float2(c, sn);
      }
    };

    lds_barrier();  // every wave is done with the near tiles (buffers and bias entries are reused)
    // codebooks [K/V][subspace][codeword] at A32_CW: 16-byte unit x is part
    // x % 5 of codeword x / 5 (the fifth is padding)
#pragma unroll
    for (int q = 0; q < (CB_BYTES / 1024 + NW - 1) / NW; ++q) {
      const int i = wave + q * NW;  // uniform
      if (i < CB_BYTES / 1024) {
        const int x = i * 64 + lane, z = x / 5;
        lds_dma16(reinterpret_cast<const uint8_t*>(ws.codebooks + unit * (2 * G * CMAX * DP)) + z * 64 + min(x - 5 * z, 3) * 16,
                  s_cbb + i * 1024);
      }
    }
    stage(0);
    if (npt > 1) stage(1);
    // codebooks and tiles 0 and 1's inputs have landed: both are converted
    // (and with rotary positions get their tables) before tile 0 is formed
    wait_vm<0>();
    lds_barrier();
    if (npt > 2) stage(2);
    convert(0);
    if (npt > 1) convert(1);
    if (rope) {
      rtab(0);
      if (npt > 1) rtab(1);
    }
    lds_barrier();
    form(0);
    for (int t = 0; t < npt; ++t) {
      // this wave's loads of tile t+2's inputs have landed (converted, and
      // with rotary positions tabled, now; tile t+1's were converted in the
      // previous iteration)
      wait_vm<0>();
      // tile t formed everywhere; stage t % 3 (read by form(t)), formed
      // buffer (t+1) % 2 (read by compute(t-1)) and table t % 2 (read by
      // form(t)) are free
      lds_barrier();
      if (t + 3 < npt) stage(t + 3);
      if (t + 2 < npt) convert(t + 2);
      if (rope && t + 2 < npt) rtab(t + 2);
      // waves w and w + 4 share a SIMD: one forms before computing, the other
      // after, so the forming overlaps the partner's matrix work
      const bool form_first = wave < 4 || !wvalid;  // uniform
      if (form_first && t + 1 < npt) form(t + 1);
      if (wvalid) compute_tile(s_kv[t & 1][0], s_kv[t & 1][1], t & 1, std::true_type{});
      if (!form_first && t + 1 < npt) form(t + 1);
    }
  }
  if constexpr (KH == 2) {
    // waves of key half 1 hand (reference, sum, O) to their half-0 partner
    // through LDS; both are relative to their own reference, so
    // O = 2^(m1 - m) O1 + 2^(m2 - m) O2, l likewise, m = max(m1, m2)
    __syncthreads();  // every wave is done with the tiles (LDS reused)
    float* s_part = reinterpret_cast<float*>(&s_kv[0][0][0]) + (size_t)rblk * 66 * 64;
    if (kh == 1) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) s_part[(b * 16 + i) * 64 + lane] = oacc[b][i];
      s_part[64 * 64 + lane] = mref;
      s_part[65 * 64 + lane] = lrun;
    }
    __syncthreads();
    if (kh == 1) return;
    const float m2 = s_part[64 * 64 + lane], l2 = s_part[65 * 64 + lane];
    const float m = fmaxf(mref, m2);
    const float a1 = __builtin_amdgcn_exp2f(mref - m), a2 = __builtin_amdgcn_exp2f(m2 - m);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[b][i] = oacc[b][i] * a1 + s_part[(b * 16 + i) * 64 + lane] * a2;
    lrun = lrun * a1 + l2 * a2;
    mref = m;
  }
  const float mrun = mref;

  const size_t orow_t = rvalid ? (size_t)(r / grp) : 0;
  const int ogg = rvalid ? r % grp : 0;
  const size_t orow = (((size_t)l * aa.tq + orow_t) * dm.Hq + kvh * grp + ogg) * D;
  if (aa.splits == 1) {
    if (rvalid) {
      const float inv = lrun > 0.f ? 1.0f / lrun : 0.f;
      uint16_t* o = reinterpret_cast<uint16_t*>(aa.o) + orow;
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[b * 32 + (i >> 2) * 8 + half * 4 + (i & 3)] = q_to_bf16(oacc[b][i] * inv);
      if (half == 0 && aa.lse) aa.lse[((size_t)l * aa.tq + orow_t) * dm.Hq + kvh * grp + ogg] = (mrun + log2f(lrun)) * LN2;
    }
    return;
  }
  if (rvalid) {
    float* po = ws.part_o + (((size_t)u * dm.max_splits + split) * dm.max_rows + r) * D;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) po[b * 32 + (i >> 2) * 8 + half * 4 + (i & 3)] = oacc[b][i];
    if (half == 0) {
      float* pml = ws.part_ml + (((size_t)u * dm.max_splits + split) * dm.max_rows + r) * 2;
      pml[0] = mrun;
      pml[1] = lrun;
    }
  }
}

// bf16 path for at most 32 query rows per kv head (the tokens of an answer).
// With one block of rows there is nothing for waves to share but the context, so
// every wave takes tiles of its own, 32 keys each, and nothing synchronises until
// the end, where the workgroup's eight partial outputs are merged through LDS:
// with the tiles shared by the workgroup, two of eight waves computed and each
// tile cost a barrier and the whole load - product - softmax - product chain.
// Tile t of a kv head goes to wave t mod (8 splits): first the tiles that are
// loaded (near window; also written pseudo-token rows), then those formed.
//   Loaded: K rows straight into the A operand (lane (m, h): row m, dims 16 kk +
//   8 h .. + 7), V rows through registers into the wave's LDS tile (by 32-dim
//   block) for the transposed reads; the next tile's K and V load meanwhile.
//   Formed: NSL = min(5, 32 / S) whole slots.  The next tile's sums, records and
//   biases load into registers meanwhile; the centres sum / n go to LDS once per
//   slot, then each lane forms its row of K in the A operand and half its row of
//   V in the LDS tile, with the roundings of k_materialize16.
// Bound by the bytes read (112 kv heads, 7 rows, 1 568 near keys and 256 slots:
// 123 MB, 26 us at the rate of a copy) and the forming's arithmetic (14 us by
// itself): 34.8 us, 66.7 with shared tiles.
constexpr int A32_W = 8;                       // waves per workgroup
constexpr int A32_VB = 32 * 64 + 64;           // bytes of one 32-dim block of a V tile (64 of padding: bank spread)
constexpr int A32_SLOTS = 5;                   // slots per formed tile, at most
constexpr int A32_CS = 1024 + 64;              // bytes of one slot's centres, K then V (64 of padding)
constexpr int A32_CEN = 4 * A32_VB;            // wave's LDS: V tile, centres, records, row biases, rotary table
constexpr int A32_REC = A32_CEN + A32_SLOTS * A32_CS;
constexpr int A32_BIAS = A32_REC + 768;        // 5 records of 144 bytes
constexpr int A32_ROPE = A32_BIAS + 128;
constexpr int A32_WAVE = A32_ROPE + A32_SLOTS * 512;
constexpr int A32_LDS = A32_W * A32_WAVE + 2 * G * CMAX * A32_CW;
static_assert(A32_SLOTS * 2 * PCW * 4 <= 768 && A32_WAVE % 16 == 0 && A32_LDS <= 163840, "LDS layout");
static_assert(A32_W * 66 * 64 * 4 <= A32_LDS, "the merge reuses the tiles");

// Orders the LDS accesses of one wave's lanes (no instruction: a wave's LDS
// operations complete in order).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(A32_W * 64, 2) void k_attend_rows32(Dims dm, Workspace ws, AttendArgs aa, int rows) {
  __shared__ __attribute__((aligned(16))) uint8_t s_mem[A32_LDS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // splits of one kv head land on one XCD (dispatch is round-robin over 8)
  const int nblk = gridDim.x, per = nblk / 8;
  const int lbid = (int)blockIdx.x < per * 8 ? ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8 : (int)blockIdx.x;
  const int split = lbid % aa.splits, u = lbid / aa.splits;
  const size_t unit = (size_t)aa.sid * dm.units + u;
  const int grp = dm.Hq / dm.Hkv;
  const int l = u / dm.Hkv, kvh = u % dm.Hkv;
  const int m = lane & 31, half = lane >> 5;
  const bool rvalid = m < rows;
  const int rt = rvalid ? m / grp : 0, gg = rvalid ? m % grp : 0;
  const size_t orow = ((size_t)l * aa.tq + rt) * dm.Hq + kvh * grp + gg;
  uint8_t* mem = s_mem + wave * A32_WAVE;
  uint8_t* s_cb = s_mem + A32_W * A32_WAVE;  // [K/V][subspace][codeword] at A32_CW
  const int w0 = split * A32_W + wave, nw = aa.splits * A32_W;  // this wave's tiles: w0, w0 + nw, ...
  const int nload = aa.gen ? aa.n_near : aa.n_near + aa.n_far;
  const int ltiles = (nload + 31) / 32;
  const int nsl = aa.gen ? min(A32_SLOTS, 32 / dm.S) : 1;
  const int nact = aa.gen ? aa.n_far / dm.S : 0;
  const int ftiles = (nact + nsl - 1) / nsl;
  const bool ema = (dm.flags & PROTOKV_FLAG_EMA_CENTRES) != 0;
  const bool rope = ws.rope_inv != nullptr;  // uniform

  // the unit's codebooks (two 16-byte parts per thread), the query, and below the
  // first tiles: all loads in flight before the first wait
  constexpr int CBP = 2 * G * CMAX * DP / 4 / (A32_W * 64);
  float4 cbr[CBP];
#pragma unroll
  for (int i = 0; i < CBP; ++i)
    cbr[i] = reinterpret_cast<const float4*>(ws.codebooks + unit * (2 * G * CMAX * DP))[tid + i * A32_W * 64];
  bf16x8 bq[8];
  {
    const u16x8* qr = reinterpret_cast<const u16x8*>(reinterpret_cast<const uint16_t*>(aa.q) + orow * D);
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) bq[kk] = __builtin_bit_cast(bf16x8, qr[2 * kk + half]);  // lanes past the rows repeat row 0
  }

  const float scale = LOG2E / sqrtf((float)D);
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 oacc[4] = {zero, zero, zero, zero};
  float mref = -1e30f, lrun = 0.f;  // as in k_attend_bf16
  const int grp16 = lane >> 4, s16 = lane & 15;
  const uint8_t* vl = mem + (4 * half + (s16 >> 2)) * 64 + (grp16 & 1) * 32 + (s16 & 3) * 8;
  const float4* s_bias = reinterpret_cast<const float4*>(mem + A32_BIAS);
  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // the products S^T of a tile start from the keys' biases (in units of q.k)
  auto biases = [&]() {
    f32x16 s;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const float4 b4 = s_bias[i4 * 2 + half];
      s[i4 * 4] = b4.x;
      s[i4 * 4 + 1] = b4.y;
      s[i4 * 4 + 2] = b4.z;
      s[i4 * 4 + 3] = b4.w;
    }
    return s;
  };
  // softmax of the scores s (S^T of 32 keys) and O^T += V^T P from the LDS tile
  auto weigh = [&](const f32x16& s) {
    float tmax = -1e30f;
#pragma unroll
    for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
    tmax = fmaxf(tmax, xor32(tmax)) * scale;
    const bool grow = tmax > mref + 8.0f;
    if (__ballot(grow)) {  // uniform
      const float mnew = grow ? tmax : mref;
      const float alpha = __builtin_amdgcn_exp2f(mref - mnew);
      lrun *= alpha;
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[b][i] *= alpha;
      mref = mnew;
    }
    const float nm = -mref;
    bf16x8 pb[2];
#pragma unroll
    for (int i = 0; i < 16; ++i) pb[i >> 3][i & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[i], scale, nm));
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      sum0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 0, 1), ones2, sum0, false);
      sum1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 2, 3), ones2, sum1, false);
      sum0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 4, 5), ones2, sum0, false);
      sum1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[j], pb[j], 6, 7), ones2, sum1, false);
    }
    lrun += sum0 + sum1;  // this half's keys
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vl + b * A32_VB + st * 1024));
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vl + b * A32_VB + st * 1024 + 512));
        const v8i16 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pb[st], oacc[b], 0, 0, 0);
      }
  };

  // formed tiles: this tile's inputs in registers (sums: unit `lane` of slot
  // i's 64; records: words lane, lane + 64, lane + 128; bias of slot m)
  const size_t ubase = (size_t)u * dm.K;
  auto load_slots = [&](int ft, float4 (&fs)[A32_SLOTS], uint32_t (&fr)[3], float& fb) {
    const int k0 = ft * nsl, last = nact - 1;
#pragma unroll
    for (int i = 0; i < A32_SLOTS; ++i)
      if (i < nsl)  // uniform
        fs[i] = reinterpret_cast<const float4*>(ws.bank + (unit * dm.K + min(k0 + i, last)) * ROW + ROW_SUMK)[lane];
#pragma unroll
    for (int i = 0; i < 3; ++i)  // past the last slot: its value record's last word, n
      fr[i] = ws.pcodes[ubase * 2 * PCW + min(k0 * 2 * PCW + lane + 64 * i, nact * 2 * PCW - 1)];
    fb = ws.pbias[ubase + min(k0 + min(m, nsl - 1), last)];
  };

  // loaded tiles
  auto row_of = [&](int t, float& bias) {  // ring row, or -1 - pseudo-token row, of this lane's key m
    const int idx = t * 32 + m, pos = min(idx, nload - 1);
    int row;
    bias = 0.f;
    if (pos < aa.n_near) {
      const int fo = pos / dm.T;
      row = ((aa.f_first + fo) % (dm.W + 1)) * dm.T + (pos - fo * dm.T);
    } else {
      const int pr = pos - aa.n_near;
      row = -1 - pr;
      bias = (aa.rowbias ? aa.rowbias[ubase * dm.S + pr] : ws.pbias[ubase + pr / dm.S]) * SQRT_D;
    }
    if (idx >= nload) bias = -INFINITY;
    return row;
  };
  const u16x8* nk = reinterpret_cast<const u16x8*>(aa.near_k + unit * (dm.W + 1) * dm.T * (size_t)(D * 2));
  const u16x8* nv = reinterpret_cast<const u16x8*>(ws.ring_v + unit * (dm.W + 1) * dm.T * (size_t)(D * 2));
  const u16x8* pk = reinterpret_cast<const u16x8*>(ws.pk + ubase * dm.S * (size_t)(D * 2));
  const u16x8* pv = reinterpret_cast<const u16x8*>(ws.pv + ubase * dm.S * (size_t)(D * 2));
  auto load_k = [&](int row, u16x8 (&kr)[8]) {
    const u16x8* p = row >= 0 ? nk + (size_t)row * 16 : pk + (size_t)(-1 - row) * 16;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kr[kk] = p[2 * kk + half];
  };
  auto load_v = [&](int row, u16x8 (&vr)[8]) {  // unit i: row 4 i + lane / 16, 16-byte chunk lane % 16
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = __builtin_amdgcn_ds_bpermute(4 * (lane >> 4) + 16 * i, row);
      vr[i] = (r >= 0 ? nv + (size_t)r * 16 : pv + (size_t)(-1 - r) * 16)[lane & 15];
    }
  };
#pragma unroll
  for (int i = 0; i < CBP; ++i) {
    const int x = tid + i * A32_W * 64;
    *reinterpret_cast<float4*>(s_cb + (x >> 2) * A32_CW + (x & 3) * 16) = cbr[i];
  }
  // formed tiles: row m is pseudo-token s2 of the tile's slot j
  const int j = min(m / dm.S, nsl - 1), s2 = m - j * dm.S;
  // this lane's chunks: of K 2 kk + half, of V 8 half + e
  const uint8_t* cenk = mem + A32_CEN + j * A32_CS + half * 32;
  const uint8_t* cenv = mem + A32_CEN + j * A32_CS + 512 + half * 256;
  const uint8_t* cbk = s_cb + half * 32;
  const uint8_t* cbv = s_cb + (G + half * 4) * CMAX * A32_CW;
  const uint32_t* rec = reinterpret_cast<const uint32_t*>(mem + A32_REC) + j * 2 * PCW;
  const double rinv = rope ? ws.rope_inv[lane] : 0.0;
  auto loaded_tiles = [&](bool first) {
    u16x8 kr[8], vr[8];
    int t = w0, row = 0;
    float bias = 0.f;
    if (t < ltiles) {
      row = row_of(t, bias);
      load_v(row, vr);
      load_k(row, kr);
    }
    if (first) lds_barrier();  // the codebooks are staged
    for (; t < ltiles; t += nw) {
      const int tn = t + nw < ltiles ? t + nw : t;  // past the last tile the loads repeat it
      float nbias;
      row = row_of(tn, nbias);
      const bool biased = (t + 1) * 32 > aa.n_near;  // uniform
      {
        if ((t + 1) * 32 > nload) {  // uniform: keys past the context have weight 0, but 0 x inf would not be 0
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (t * 32 + 4 * i + (lane >> 4) >= nload) vr[i] = (u16x8)0;
        }
        uint8_t* vw = mem + ((lane & 15) >> 2) * A32_VB + (lane >> 4) * 64 + (lane & 3) * 16;
        wave_lds_order();
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u16x8*>(vw + i * 256) = vr[i];
        if (biased && half == 0) reinterpret_cast<float*>(mem + A32_BIAS)[m] = bias;
        wave_lds_order();
      }
      load_v(row, vr);
      f32x16 s = zero;
      if (biased) s = biases();
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kr[kk]), bq[kk], s, 0, 0, 0);
      load_k(row, kr);
      weigh(s);
      bias = nbias;
    }
  };
  auto formed_tiles = [&](bool first) {
    float4 fs[A32_SLOTS];
    uint32_t fr[3];
    float fb = 0.f;
    int ft = ((w0 - ltiles) % nw + nw) % nw;  // tile ltiles + ft = w0 mod nw
    if (ft < ftiles) load_slots(ft, fs, fr, fb);
    if (first) lds_barrier();
    for (; ft < ftiles; ft += nw) {
      wave_lds_order();
      // centres sum / n (IEEE division)
#pragma unroll
      for (int i = 0; i < A32_SLOTS; ++i) {
        if (i < nsl) {  // uniform
          constexpr int LAST = PCW + SMAX + 1;  // n in the value record, tau in the key record
          const int wn = i * 2 * PCW + LAST, wt = i * 2 * PCW + SMAX + 1;
          const float nf = ema ? 1.f : (float)(uint32_t)__builtin_amdgcn_readlane((int)fr[wn >> 6], wn & 63);
          reinterpret_cast<float4*>(mem + A32_CEN + i * A32_CS)[lane] =
              make_float4(fs[i].x / nf, fs[i].y / nf, fs[i].z / nf, fs[i].w / nf);
          if (rope) {
            float c, sn;
            rope_cs((double)__builtin_amdgcn_readlane((int)fr[wt >> 6], wt & 63), rinv, c, sn);
            reinterpret_cast<float2*>(mem + A32_ROPE)[i * 64 + lane] = make_float2(c, sn);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int w = lane + 64 * i;
        if (w < A32_SLOTS * 2 * PCW) reinterpret_cast<uint32_t*>(mem + A32_REC)[w] = fr[i];
      }
      const bool ok = m < nsl * dm.S && ft * nsl + j < nact;  // row m is a pseudo-token
      {
        const float b = __shfl(fb, j, 64) * SQRT_D;
        if (half == 0) reinterpret_cast<float*>(mem + A32_BIAS)[m] = ok ? b : -INFINITY;
      }
      wave_lds_order();
      if (ft + nw < ftiles) load_slots(ft + nw, fs, fr, fb);
      const bool tail = nsl * dm.S < 32 || (ft + 1) * nsl > nact;  // uniform
      // rows past the tile's last slot repeat a valid tuple (bias -inf)
      const int sv = min(s2, dm.S - 1);
      const uint32_t tk = rec[sv], tv = rec[PCW + sv] >> (16 - 16 * half);  // V: this half's four subspaces
      const float mk = rec[SMAX] != 0u ? 0.f : 1.f, mv = rec[PCW + SMAX] != 0u ? 0.f : 1.f;  // no residual: the centre alone
      // 8 values at centre c, codeword w: exactly c + w or (mul 0) c
      auto chunk = [&](const uint8_t* c, const uint8_t* w, float mul, float (&x)[8]) {
        const float4 ca = reinterpret_cast<const float4*>(c)[0], cb = reinterpret_cast<const float4*>(c)[1];
        const float4 wa = reinterpret_cast<const float4*>(w)[0], wb = reinterpret_cast<const float4*>(w)[1];
        x[0] = fmaf(wa.x, mul, ca.x); x[1] = fmaf(wa.y, mul, ca.y); x[2] = fmaf(wa.z, mul, ca.z); x[3] = fmaf(wa.w, mul, ca.w);
        x[4] = fmaf(wb.x, mul, cb.x); x[5] = fmaf(wb.y, mul, cb.y); x[6] = fmaf(wb.z, mul, cb.z); x[7] = fmaf(wb.w, mul, cb.w);
      };
      auto keyc = [&](int kk, float (&x)[8]) {  // dims 16 kk + 8 half .. + 7
        chunk(cenk + kk * 64, cbk + kk * CMAX * A32_CW + ((tk >> (4 * (G - 1 - kk))) & 15) * A32_CW, mk, x);
      };
      auto round8 = [](const float (&x)[8]) {
        bf16x8 r;
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = (__bf16)x[e];
        return r;
      };
      f32x16 s = biases();
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        // chunks of rotate-half pairs: dims i and i + D / 2
        float x1[8], x2[8];
        keyc(kk, x1);
        keyc(kk + 4, x2);
        bf16x8 a1 = round8(x1), a2 = round8(x2);
        if (rope) {  // each key, rounded to bf16 as written, turned at tau_k and rounded again
          const float4* cs = reinterpret_cast<const float4*>(mem + A32_ROPE) + (j * 64 + 16 * kk + 8 * half) / 2;
#pragma unroll
          for (int e2 = 0; e2 < 4; ++e2) {
            const float4 c4 = cs[e2];  // (cos, sin) of two pairs
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const int e = 2 * e2 + h;
              rope_pair((float)a1[e], (float)a2[e], h ? c4.z : c4.x, h ? c4.w : c4.y, x1[e], x2[e]);
            }
          }
          a1 = round8(x1);
          a2 = round8(x2);
        }
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, bq[kk], s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, bq[kk + 4], s, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x[8];
        chunk(cenv + e * 32, cbv + (e >> 1) * CMAX * A32_CW + (e & 1) * 32 + ((tv >> (12 - 4 * (e >> 1))) & 15) * A32_CW, mv, x);
        if (tail) {
#pragma unroll
          for (int y = 0; y < 8; ++y) x[y] = ok ? x[y] : 0.f;  // (0 x inf, as above)
        }
        *reinterpret_cast<bf16x8*>(mem + (2 * half + (e >> 2)) * A32_VB + m * 64 + (e & 3) * 16) = round8(x);
      }
      wave_lds_order();
      weigh(s);
    }
  };
  // Waves w and w + 4 share a SIMD: one takes the loaded tiles first, the other the
  // formed ones, so that the one's memory latency meets the other's arithmetic
  // (all loaded tiles first: 37.8 us against 34.8).
  if (wave < A32_W / 2) {  // uniform
    loaded_tiles(true);
    formed_tiles(false);
  } else {
    formed_tiles(true);
    loaded_tiles(false);
  }

  // merge of the eight waves (each relative to its own reference)
  lrun += xor32(lrun);
  __syncthreads();  // the tiles' LDS is reused
  float* part = reinterpret_cast<float*>(s_mem);
  if (rvalid) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) part[(wave * 66 + b * 16 + i) * 64 + lane] = oacc[b][i];
    part[(wave * 66 + 64) * 64 + lane] = mref;
    part[(wave * 66 + 65) * 64 + lane] = lrun;
  }
  __syncthreads();
  if (!rvalid) return;
  float M = -INFINITY, L = 0.f, wgt[A32_W];
#pragma unroll
  for (int w = 0; w < A32_W; ++w) M = fmaxf(M, part[(w * 66 + 64) * 64 + lane]);
#pragma unroll
  for (int w = 0; w < A32_W; ++w) {
    wgt[w] = __builtin_amdgcn_exp2f(part[(w * 66 + 64) * 64 + lane] - M);
    L += wgt[w] * part[(w * 66 + 65) * 64 + lane];
  }
  // wave w's registers 8 w .. 8 w + 7: two runs of four dims
  const bool whole = aa.splits == 1;
  const float inv = whole ? (L > 0.f ? 1.0f / L : 0.f) : 1.0f;
  const size_t prow = ((size_t)u * dm.max_splits + split) * dm.max_rows + m;
#pragma unroll
  for (int run = 0; run < 2; ++run) {
    float o[4];
    const int i0 = wave * 8 + run * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = 0.f;
#pragma unroll
      for (int w = 0; w < A32_W; ++w) o[e] += wgt[w] * part[(w * 66 + i0 + e) * 64 + lane];
    }
    const int dim = (i0 >> 4) * 32 + ((i0 & 15) >> 2) * 8 + half * 4;
    if (whole)
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(aa.o) + orow * D + dim) =
          make_uint2((uint32_t)q_to_bf16(o[0] * inv) | ((uint32_t)q_to_bf16(o[1] * inv) << 16),
                     (uint32_t)q_to_bf16(o[2] * inv) | ((uint32_t)q_to_bf16(o[3] * inv) << 16));
    else
      *reinterpret_cast<float4*>(ws.part_o + prow * D + dim) = make_float4(o[0], o[1], o[2], o[3]);
  }
  if (wave == 0 && half == 0) {
    if (!whole) {
      ws.part_ml[prow * 2] = M;
      ws.part_ml[prow * 2 + 1] = L;
    } else if (aa.lse) {
      aa.lse[orow] = (M + log2f(L)) * LN2;
    }
  }
}

// Combines the splits' partials of output row r, dims 4 d4 .. 4 d4 + 3, of
// kv head u: O = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^(m_s - max m).
// NSP: the number of splits when known at compile time (0: aa.splits).
template <int FP32, int NSP>
__device__ __forceinline__ void merge_row4(const Dims& dm, const Workspace& ws, const AttendArgs& aa, int u, int r,
                                           int d4) {
  constexpr int NS = NSP ? NSP : MAX_SPLITS;
  const int nsplit = NSP ? NSP : aa.splits;
  const int grp = dm.Hq / dm.Hkv;
  const int l = u / dm.Hkv, kvh = u % dm.Hkv;
  float ms[NS], ls[NS];
  float4 ov[NS];
  float M = -INFINITY;
#pragma unroll
  for (int s2 = 0; s2 < NS; ++s2) {
    if (s2 < nsplit) {
      const size_t pr = ((size_t)u * dm.max_splits + s2) * dm.max_rows + r;
      ms[s2] = ws.part_ml[pr * 2];
      ls[s2] = ws.part_ml[pr * 2 + 1];
      ov[s2] = reinterpret_cast<const float4*>(ws.part_o + pr * D)[d4];
      M = fmaxf(M, ms[s2]);
    }
  }
  float Lsum = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int s2 = 0; s2 < NS; ++s2) {
    if (s2 < nsplit) {
      const float w = ms[s2] == -INFINITY ? 0.f : exp2f(ms[s2] - M);
      Lsum += w * ls[s2];
      o.x += w * ov[s2].x;
      o.y += w * ov[s2].y;
      o.z += w * ov[s2].z;
      o.w += w * ov[s2].w;
    }
  }
  const float inv = Lsum > 0.f ? 1.0f / Lsum : 0.f;
  const int t = r / grp, gg = r % grp;
  const size_t orow = (((size_t)l * aa.tq + t) * dm.Hq + kvh * grp + gg) * D;
  if (FP32) {
    reinterpret_cast<float4*>(reinterpret_cast<float*>(aa.o) + orow)[d4] =
        make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
  } else {
    const uint2 packed = make_uint2((uint32_t)q_to_bf16(o.x * inv) | ((uint32_t)q_to_bf16(o.y * inv) << 16),
                                    (uint32_t)q_to_bf16(o.z * inv) | ((uint32_t)q_to_bf16(o.w * inv) << 16));
    reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(aa.o) + orow)[d4] = packed;
  }
  if (d4 == 0 && aa.lse) aa.lse[((size_t)l * aa.tq + t) * dm.Hq + kvh * grp + gg] = (M + log2f(Lsum)) * LN2;
}

template <int FP32, int NSP>
__global__ __launch_bounds__(256) void k_attend_merge(Dims dm, Workspace ws, AttendArgs aa, int rows) {
  // thread = (kv head, query row, 4 output dims); every split's (m, l) and
  // partial O are loaded together (units * rows * D / 4 < 2^31)
  const int gt = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (gt >= dm.units * rows * (D / 4)) return;
  const int d4 = gt & (D / 4 - 1);
  const int rr = gt / (D / 4);
  const int r = rr % rows;
  const int u = rr / rows;
  merge_row4<FP32, NSP>(dm, ws, aa, u, r, d4);
}

// float32 path: S^T = K Q^T and O^T = V^T P on v_mfma_f32_32x32x2_f32 (float32
// products and sums).  One wave = one work item (kv head, context split, 32
// query rows), 32 keys per tile, four independent waves per workgroup.  A
// float32 MFMA holds the matrix core for 64 cycles and takes 4 bytes per lane of
// each operand, so K and V go straight from global memory into the operand
// registers, 16 bytes per lane and load, half a tile at a time and two half
// products ahead; only the query sits in LDS (each lane reads back what it wrote).
//   K: lane (m = lane % 32, h = lane / 32) loads dims 8 j + 4 h .. + 3 of key m,
//      so step (j, e) contracts dims 8 j + e (h = 0) and 8 j + 4 + e (h = 1);
//      Q is laid out the same way.
//   P: register i of S^T holds key 8 (i / 4) + 4 h + i % 4 of query lane % 32: as
//      it stands the B operand of a step over the keys 8 (i / 4) + i % 4 (h = 0)
//      and + 4 (h = 1).
//   V: for that step lane (m, h) loads dims 4 m .. 4 m + 3 of its half's key; row
//      m of accumulator b is dim 4 m + b, so the output is stored 16 bytes at a
//      time.
// A dot product is the sum of eight 16-dim chains, four and four: its rounding
// error is that of a pairwise sum (one chain of 64 steps would carry several
// times as much into the exponent).  Bound by the float32 matrix rate: 32 kv
// heads x 224 rows x 3 616 keys (13.3 GFLOP) take 149 us (157 under the counters,
// by which the matrix cores are busy 54% of it; one wave per query row with a
// shuffled dot product per key took 4 311 us); its error against 64 bits fell from 2.3e-6 to 7e-7.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const f32x4 gbl_f32x4;

__global__ __launch_bounds__(256, 2) void k_attend_f32(Dims dm, Workspace ws, AttendArgs aa, int rows, int rblocks) {
  __shared__ f32x4 s_q[4][16][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nblk = gridDim.x, per = nblk / 8;
  // blocks of one kv head land on one XCD (dispatch is round-robin over 8)
  const int lbid = (int)blockIdx.x < per * 8 ? ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8 : (int)blockIdx.x;
  const int item = lbid * 4 + wave;
  if (item >= dm.units * aa.splits * rblocks) return;  // uniform, and nothing below synchronises waves
  const int rb = item % rblocks, split = (item / rblocks) % aa.splits, u = item / (rblocks * aa.splits);
  const size_t unit = (size_t)aa.sid * dm.units + u;
  const int grp = dm.Hq / dm.Hkv;
  const int l = u / dm.Hkv, kvh = u % dm.Hkv;
  const int ctx = aa.n_near + aa.n_far;
  const int c0 = split * aa.chunk, c1 = min(ctx, c0 + aa.chunk);
  const int ntiles = (c1 - c0 + F32_KEYS - 1) / F32_KEYS;
  const int m = lane & 31, half = lane >> 5;
  const int r = rb * 32 + m;  // query row of this lane
  const bool rvalid = r < rows;
  // lanes past the last row repeat row 0 and store nothing
  const int t = rvalid ? r / grp : 0, gg = rvalid ? r % grp : 0;
  const size_t orow = ((size_t)l * aa.tq + t) * dm.Hq + kvh * grp + gg;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    s_q[wave][j][lane] = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(aa.q) + orow * D)[2 * j + half];
  // the K and V rows of this lane's key of tile tl (keys past the split repeat
  // its last one) and the key's bias in log2 units
  auto resolve = [&](int tl, const float*& kp, const float*& vp, float& bias) {
    const int idx = c0 + tl * F32_KEYS + m;
    const int pos = min(idx, c1 - 1);
    bias = 0.f;
    if (pos < aa.n_near) {
      const int fo = pos / dm.T;
      const size_t row = (unit * (dm.W + 1) + (aa.f_first + fo) % (dm.W + 1)) * dm.T + (pos - fo * dm.T);
      kp = reinterpret_cast<const float*>(aa.near_k) + row * D;
      vp = reinterpret_cast<const float*>(ws.ring_v) + row * D;
    } else {
      const int pr = pos - aa.n_near;
      const size_t row = (size_t)u * dm.K * dm.S + pr;
      kp = reinterpret_cast<const float*>(ws.pk) + row * D;
      vp = reinterpret_cast<const float*>(ws.pv) + row * D;
      bias = (aa.rowbias ? aa.rowbias[row] : ws.pbias[(size_t)u * dm.K + pr / dm.S]) * LOG2E;
    }
    if (idx >= c1) bias = -INFINITY;
  };
  // half h of a tile: dims 64 h .. 64 h + 63 of K; registers 8 h .. 8 h + 7 of V,
  // register i's key being lane 8 (i / 4) + 4 half + i % 4's
  auto load_k = [&](const float* kp, int h, f32x4 (&kr)[8]) {
    gbl_f32x4* p = (gbl_f32x4*)(uintptr_t)kp + half + 16 * h;
#pragma unroll
    for (int j = 0; j < 8; ++j) kr[j] = p[2 * j];
  };
  // value of register i's key (lane addresses in bytes)
  auto of_key = [&](int x, int i) {
    return __builtin_amdgcn_ds_bpermute(16 * half + 4 * (8 * (i >> 2) + (i & 3)), x);
  };
  auto load_v = [&](const float* vp, int h, f32x4 (&vr)[8]) {
    const uint64_t a = reinterpret_cast<uint64_t>(vp);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t lo = of_key((int)(uint32_t)a, 8 * h + i), hi = of_key((int)(uint32_t)(a >> 32), 8 * h + i);
      vr[i] = ((gbl_f32x4*)(uintptr_t)((uint64_t)hi << 32 | lo))[m];
    }
  };
  const float scale = LOG2E / sqrtf((float)D);
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 oacc[4] = {zero, zero, zero, zero};
  float mrun = -INFINITY, lrun = 0.f;  // log2 units; lrun: this half's keys
  // four chains over the dims of half h
  auto dots = [&](const f32x4 (&kr)[8], int h) {
    f32x16 s = zero;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x16 a = zero;
#pragma unroll
      for (int j = 2 * g; j < 2 * g + 2; ++j) {
        const f32x4 qv = s_q[wave][8 * h + j][lane];
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j].x, qv.x, a, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j].y, qv.y, a, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j].z, qv.z, a, 0, 0, 0);
        a = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j].w, qv.w, a, 0, 0, 0);
      }
      s = g ? s + a : a;
      asm("" : "+v"(s));  // summed here, not after every chain is done
    }
    return s;
  };
  auto weigh = [&](const f32x4 (&vr)[8], const f32x16& p, int h) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      oacc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i].x, p[8 * h + i], oacc[0], 0, 0, 0);
      oacc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i].y, p[8 * h + i], oacc[1], 0, 0, 0);
      oacc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i].z, p[8 * h + i], oacc[2], 0, 0, 0);
      oacc[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i].w, p[8 * h + i], oacc[3], 0, 0, 0);
    }
  };
  // keys past the split have weight 0, but 0 x inf would not be 0
  auto mask = [&](f32x4 (&vr)[8], const f32x16& bv, int h) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t keep = bv[8 * h + i] == -INFINITY ? 0u : ~0u;
      vr[i].x = __uint_as_float(__float_as_uint(vr[i].x) & keep);
      vr[i].y = __uint_as_float(__float_as_uint(vr[i].y) & keep);
      vr[i].z = __uint_as_float(__float_as_uint(vr[i].z) & keep);
      vr[i].w = __uint_as_float(__float_as_uint(vr[i].w) & keep);
    }
  };
  f32x4 k0[8], k1[8], v0[8], v1[8];
  const float *kp, *vp;
  float bias;
  resolve(0, kp, vp, bias);
  load_k(kp, 0, k0);
  load_k(kp, 1, k1);
  for (int tl = 0; tl < ntiles; ++tl) {
    load_v(vp, 0, v0);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s = dots(k0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(vp, 1, v1);
    __builtin_amdgcn_sched_barrier(0);
    s = s + dots(k1, 1);
    // bias of register i's key; -inf past the split
    f32x16 bv;
#pragma unroll
    for (int i = 0; i < 16; ++i) bv[i] = __int_as_float(of_key(__float_as_int(bias), i));
    // the next tile's keys load while this tile's values are used (past the
    // last tile the loads repeat it)
    resolve(min(tl + 1, ntiles - 1), kp, vp, bias);
    load_k(kp, 0, k0);
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, fmaf(s[i], scale, bv[i]));
    tmax = fmaxf(tmax, xor32(tmax));
    const float mnew = fmaxf(mrun, tmax);
    if (__ballot(!(mnew <= mrun))) {  // uniform
      const float alpha = __builtin_amdgcn_exp2f(mrun - mnew);
      lrun *= alpha;
#pragma unroll
      for (int b = 0; b < 4; ++b) oacc[b] *= alpha;
      mrun = mnew;
    }
    // relative to the maximum before the bias is added: one rounding at the
    // size of the difference, not of the logit
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = __builtin_amdgcn_exp2f(fmaf(s[i], scale, -mrun) + bv[i]);
      part[i & 3] += s[i];
    }
    lrun += (part[0] + part[1]) + (part[2] + part[3]);
    if (c0 + (tl + 1) * F32_KEYS > c1) {  // uniform: the last tile is short
      mask(v0, bv, 0);
      mask(v1, bv, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    weigh(v0, s, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_k(kp, 1, k1);
    __builtin_amdgcn_sched_barrier(0);
    weigh(v1, s, 1);
  }
  lrun += xor32(lrun);
  if (!rvalid) return;
  // register i of oacc[0..3]: dims 4 mm .. 4 mm + 3 with mm = 8 (i / 4) + 4 half + i % 4
  const bool whole = aa.splits == 1;
  const float w = whole ? (lrun > 0.f ? 1.0f / lrun : 0.f) : 1.0f;
  const size_t pr = ((size_t)u * dm.max_splits + split) * dm.max_rows + r;
  float* out = whole ? reinterpret_cast<float*>(aa.o) + orow * D : ws.part_o + pr * D;
#pragma unroll
  for (int i = 0; i < 16; ++i)
    reinterpret_cast<float4*>(out)[8 * (i >> 2) + 4 * half + (i & 3)] =
        make_float4(oacc[0][i] * w, oacc[1][i] * w, oacc[2][i] * w, oacc[3][i] * w);
  if (half == 0) {
    if (!whole) {
      ws.part_ml[pr * 2] = mrun;
      ws.part_ml[pr * 2 + 1] = lrun;
    } else if (aa.lse) {
      aa.lse[orow] = (mrun + log2f(lrun)) * LN2;
    }
  }
}

hipError_t launch_attend(const Dims& dm, const Workspace& ws, const AttendArgs& aa, hipStream_t st) {
  const int grp = dm.Hq / dm.Hkv;
  const int rows = aa.tq * grp;
  if (dm.kv_fp32) {
    const int rblocks = (rows + 31) / 32, items = dm.units * aa.splits * rblocks;
    hipLaunchKernelGGL(k_attend_f32, dim3((items + 3) / 4), dim3(256), 0, st, dm, ws, aa, rows, rblocks);
  } else {
    // 8 waves per workgroup: 256 query rows, or at most 128 rows with the
    // tiles' key halves split between wave pairs; at most 32 rows, the one block
    // a wave holds, a wave per tile (28 rows, 112 x 256 slots, S = 8: 66 us with key
    // halves, 34 so; 32 rows, 256 x 2 048: 642 and 253, and 33 rows there 509 now)
    const int rblocks = (rows + AT_ROWS - 1) / AT_ROWS;
    if (rows <= 32)
      hipLaunchKernelGGL(k_attend_rows32, dim3(dm.units * aa.splits), dim3(A32_W * 64), 0, st, dm, ws, aa, rows);
    else if (rows > 128)
      hipLaunchKernelGGL((k_attend_bf16<8, 1>), dim3(dm.units * aa.splits * rblocks), dim3(512), 0, st, dm, ws, aa,
                         rows, rblocks);
    else
      hipLaunchKernelGGL((k_attend_bf16<8, 2>), dim3(dm.units * aa.splits), dim3(512), 0, st, dm, ws, aa, rows, 1);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of protokv_attend_static (callers that cannot allocate): the split
// partials and the rotated query live in this file-scope device array instead
// of the workspace.  Every device the library runs on holds its own copy
// until the process ends; host code must use the address from
// static_scratch_ptr, never the array's name.
// ---------------------------------------------------------------------------
static __device__ __align__(256) uint8_t scratch[PROTOKV_STATIC_SCRATCH_BYTES];

hipError_t static_scratch_ptr(void** out) {
  static std::mutex mu;
  static void* per_device[MAX_DEVICES] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    per_device[dev] = p;
  }
  *out = per_device[dev];
  return hipSuccess;
}

hipError_t launch_attend_merge(const Dims& dm, const Workspace& ws, const AttendArgs& aa, hipStream_t st) {
  if (aa.splits == 1) return hipSuccess;  // the readout wrote O directly
  const int rows = aa.tq * (dm.Hq / dm.Hkv);
  const int nb = (int)(((size_t)dm.units * rows * (D / 4) + 255) / 256);
  if (dm.kv_fp32)
    hipLaunchKernelGGL((k_attend_merge<1, 0>), dim3(nb), dim3(256), 0, st, dm, ws, aa, rows);
  else if (aa.splits == 2)
    hipLaunchKernelGGL((k_attend_merge<0, 2>), dim3(nb), dim3(256), 0, st, dm, ws, aa, rows);
  else
    hipLaunchKernelGGL((k_attend_merge<0, 0>), dim3(nb), dim3(256), 0, st, dm, ws, aa, rows);
  return hipGetLastError();
}

}  // namespace pkv
