// Wide-k products on the matrix cores (gfx950): R = A.W and out = (G^T A)^T for
// batches of up to 256 tuples whose used columns are filled densely enough.
//
// The matrix cores run bf16 products with binary32 accumulation at 16 times the
// vector units' rate, so a batch is expanded on the chip, 32 of its used columns at
// a time, into LDS tiles of bf16, and never in memory.  Operands keep their 24-bit
// significands: a binary32 value is split exactly into three bf16 parts (Henry, Tang and
// Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for
// higher-precision computations", ARITH 2019), x = x1 + x2 + x3 with |x2| < 2^-7 |x|,
// |x3| < 2^-15 |x| (the dense operand's are rounded to nearest: half of these), and a
// product x.y is the sum of all products of parts but x3y3, which is below 2^-31 |x||y|.
// With six of them, up to x1y3, x2y2 and x3y1, a sum of one term was off by 1.9e-7 of
// itself at most, where one fma gives 6.0e-8.  A chunk whose values all have
// x2 = x3 = 0 (integers below 256, 1.0, sixteenths) takes the three products of x1
// alone, which are exact; the entries loaded past a column's end are looked at too, so
// some chunks take eight that need not.
//
// Sums are formed in blocks: the right product adds the 32 terms of a chunk to an output
// at once, the left product those of all tuples.  Both keep the products of smaller
// parts apart from the leading ones x1y1 until then: the matrix cores cut a sum off where
// they add to it instead of rounding it, which with one accumulator for all parts left
// sums of one term off by 1.1e-7.  Kept apart, sums of one term are as good as the
// vector kernels' (largest 6.0e-8, RMS 2.5e-8), of two 1.6e-7 at most where those have
// 1.2e-7 (RMS 3.0e-8 and 2.9e-8), and the products of 250-row batches are closer to
// 64 bits (2-norm; vector kernels, then these): image-like right 1.1e-7, 8.0e-8, left
// 1.1e-7, 5.3e-8; dense quantised right 1.6e-7, 1.1e-7, left 1.2e-7, 8.8e-8.
//
// Parts of values near the ends of the exponent range would be lost, and an
// infinity or NaN of the dense operand must not reach tuples without that column
// (0 times infinity): a tile whose operands hold a non-finite value, or a nonzero
// one outside the ranges below, is computed term by term in binary32 instead.  The
// ranges hold what occurs: an image with values outside theirs stays with the vector
// kernels (toc_map_values can still move some out), and the dense operand is scaled,
// G column by column, so that its smallest nonzero value may be 2^-129 of the column's
// largest (saturated gradients; 400 image-like batches at k = 300 with 1 % of 1e-25
// took 12.9 ms while these went term by term, 0.3 now).  What is left is dear: with an
// infinity in one row of G that call takes 0.6 ms, in one row of W 1.0 ms, with 1 % of W
// beyond its range 4.7 ms (vector kernels 0.48 and 0.42 ms).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "toc_internal.h"

using toc::fail;

namespace {

constexpr int kWave = 64;
constexpr int kXcd = 8;
constexpr int kThreads = 512;                 // 8 waves, 2 per SIMD: 256 registers each
constexpr int kChunk = 32;                    // used columns per LDS tile
constexpr uint32_t kRowMask = 0x3fffffffu;    // row of a leaf occurrence word
constexpr uint32_t kRoot = 0xffffffffu;       // parent of a code of depth 1
constexpr int kExpandCols = 16384;            // columns whose counts the LDS holds
constexpr uint32_t kLeftRow = (kChunk + 4) * 16;   // bytes of a slot row of the left product's tile
constexpr uint32_t kSpare = kWave * 4;         // bytes after a plane: a word per lane without an entry

// |x| of the compressed values in [2^-32, 2^50], of the scaled dense operand in
// [2^-62, 2^68), zeros apart: products are then at least 2^-94, so that what parts and
// products lose below the smallest normal number 2^-126 is below 2^-32 of them, and no
// sum of 256 overflows.  G is scaled column by column, W by 2^30 (to [2^-92, 2^38)).
constexpr uint32_t kValLo = toc::kMfmaValLo, kValHi = toc::kMfmaValHi;
constexpr int kDenseTop = 68;
constexpr float kDenseLo = 0x1p-62f, kWUp = 0x1p30f;
constexpr uint32_t kWLo = (127 - 62 - 30) << 23, kWHi = ((127 + kDenseTop - 30) << 23) - 1;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// stores of both kinds go to one LDS tile
typedef uint16_t __attribute__((may_alias)) tile_u16;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x4 __attribute__((may_alias)) tile_u32x4;
typedef u32x2 __attribute__((may_alias)) tile_u32x2;
typedef __attribute__((address_space(3))) tile_u16 lds_u16;

__device__ inline uint32_t lds_address(const char *p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const char *)p;
}

__device__ inline f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Three bf16 parts of 8 values, rounded to nearest.
__device__ inline void split8(const float (&x)[8], u32x4 (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], c = x[2 * i + 1];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const f32x2 v = {a, c};
      const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
      p[s][i] = w;
      a -= __uint_as_float(w << 16);
      c -= __uint_as_float(w & 0xffff0000u);
    }
  }
}

// Running bounds of |x| over nonzero x, on the bits.
struct Range {
  uint32_t hi = 0, lo = 0xffffffffu;
  __device__ void add(uint32_t bits) {
    const uint32_t a = bits & 0x7fffffffu;
    hi = max(hi, a);
    lo = min(lo, a - 1u);           // a zero wraps to the top
  }
  __device__ bool outside(uint32_t low, uint32_t high) const { return hi > high || lo < low - 1u; }
};

__device__ inline int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

struct MfmaImg {
  const toc_batch *batches;
  const toc_key *key;
  const toc_link *link;
  const uint32_t *span, *dcodes, *centry, *cval, *occ_off, *tlist, *cols, *tchild;
  // expanded tree codes (tree_expand_kernel) of batches b0 ..: the pairs (tuple, value
  // bits) column by column, room for x_stride of them to a batch, and each column's
  // first (and the end), xoff_stride words to a batch
  const uint32_t *xoff;
  const uint2 *xpair;
  int64_t b0, xoff_stride, x_stride;
};

// One batch's column entries and tree, in wave-uniform registers.
struct Batch {
  const uint32_t *ce, *cv;       // entries and their values
  __amdgpu_buffer_rsrc_t ce_res, cv_res, x_res;   // range-checked; x: expanded pairs
  const uint32_t *xoff;          // per column: expanded pairs before it
  const toc_key *key;
  const uint32_t *occ, *tf;      // per column: leaf occurrences before it, tree-list start
  const uint32_t *order;         // columns, most entries first, those without last
  const uint32_t *to, *tch, *tl; // per tree row: occurrences, children; tree codes by column
  uint32_t n_used, ni, n1, n_tree, tbase;
  int n_rows;
  int64_t row_base;
};

__device__ inline Batch load_batch(const MfmaImg &im, int64_t b, int m) {
  const toc_batch *p = im.batches + b;
  Batch t;
  const int64_t code_base = uniform64(p->code_base), d_base = uniform64(p->d_base),
                tree_base = uniform64(p->tree_base);
  t.row_base = uniform64(p->row_base);
  t.n_rows = __builtin_amdgcn_readfirstlane(p->n_rows);
  t.ni = (uint32_t)__builtin_amdgcn_readfirstlane(p->n_int1);
  t.n1 = (uint32_t)__builtin_amdgcn_readfirstlane(p->n_lvl1);
  t.n_used = (uint32_t)__builtin_amdgcn_readfirstlane(p->n_ucols);
  t.ce = im.centry + d_base + tree_base;
  t.cv = im.cval + d_base + tree_base;
  const uint32_t *c = im.cols + b * 4 * (int64_t)(m + 1);
  t.n_tree = t.ni + (uint32_t)__builtin_amdgcn_readfirstlane(p->n_codes) - t.n1;
  const int n_entries = __builtin_amdgcn_readfirstlane(p->n_d) + (int)t.n_tree;
  t.ce_res = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(t.ce), (short)0, n_entries * 4,
                                               0x00020000);
  t.cv_res = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(t.cv), (short)0, n_entries * 4,
                                               0x00020000);
  t.occ = c + (m + 1);
  t.tf = c + 2 * (int64_t)(m + 1);
  t.order = c + 3 * (int64_t)(m + 1);
  t.tbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)t.occ[m]);
  t.to = im.occ_off + code_base + 2 * b + (t.n1 - t.ni) + 1;
  t.tch = im.tchild + tree_base + b;
  t.tl = im.tlist + tree_base;
  t.x_res = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint2 *>(im.xpair + (b - im.b0) * im.x_stride), (short)0, (int)(im.x_stride * 8),
      0x00020000);
  t.xoff = im.xoff + (b - im.b0) * im.xoff_stride;
  t.key = im.key + code_base;
  return t;
}

// The pairs of a column's tree codes, in a fixed order, by a wave: lane l walks the
// subtree of the l-th code (its own occurrences, then each level's below it: the
// descendants one level down are consecutive codes and so are their occurrences), all
// lanes a step at a time; put(row, value bits) for each pair, uniform.
template <typename F>
__device__ inline void tree_pairs(const Batch &t, uint32_t s0, uint32_t s1, F put) {
  const uint32_t lane = threadIdx.x % kWave;
  for (; s0 < s1; s0 += kWave) {
    uint32_t v = 0, o = 0, oe = 0, c = 0, ce = 0;
    if (s0 + lane < s1) {
      const uint32_t y = t.tl[s0 + lane], a = y < t.ni ? y : y - t.n1 + t.ni;
      v = t.cv[t.tbase + s0 + lane];
      o = t.to[a], oe = t.to[a + 1], c = t.tch[a], ce = t.tch[a + 1];
    }
    while (__any(o < oe || c < ce)) {
      const bool on = o < oe;
      const uint32_t row = on ? t.ce[o] & kRowMask : 0u;
      if (on) {
        ++o;
      } else if (c < ce) {
        const uint32_t a = c - t.n1 + t.ni, e = ce - t.n1 + t.ni;
        o = t.to[a], oe = t.to[e], c = t.tch[a], ce = t.tch[e];
      }
      for (uint64_t m = __ballot(on); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        put(__builtin_amdgcn_readlane((int)row, l), __builtin_amdgcn_readlane((int)v, l));
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The tree codes of the batches, expanded column by column: for every column the
// tuples whose sequences pass through one of its tree codes, with the code's value.  They
// are a small part of a batch's pairs (2 % of an image-like batch, 14 % of a dense
// quantised one), but each is found through dependent loads: done here once per call
// instead of inside the products' pipelines once per tile of columns (there it took half
// of the dense quantised batches' time).  A workgroup takes a batch and walks from every
// tree code that tuples hold up to the root, twice: first the pairs of each column are
// counted, in LDS, then, from the counts' running sums, written.  So a batch takes the
// room of its pairs (a place for every cell took 25 to 150 times as much, and no scan).
// kExpandCodes walks of a thread are in flight at a time.  The order of a column's pairs
// varies from run to run and does not matter: each fills a tile cell of its own.
//
// What bounds it is a cache line per lane of nearly every load and store, at one line a
// clock and CU, and the chain of loads of a deep code: so the tree codes (a tree row's
// parent row, column and value, 8 bytes) are first copied to LDS, where they fit.  Few
// batches of many codes are shared by `parts` workgroups each: every one counts all
// pairs and writes those of its part of the codes.
// ---------------------------------------------------------------------------
constexpr int kExpandThreads = 1024;
constexpr int kExpandCodes = 4;

template <bool LDS>
__global__ __launch_bounds__(kExpandThreads) void tree_expand_kernel(MfmaImg im, int m, int max_tree,
                                                                     int parts,
                                                                     uint32_t *__restrict__ xoff,
                                                                     uint2 *__restrict__ xpair) {
  extern __shared__ uint32_t next[];            // per column: its pairs, then its next place
  __shared__ uint32_t wave_sum[kExpandThreads / kWave];
  uint32_t *before = next + m;                  // (parts > 1) per column: pairs of the parts before
  uint32_t *up_col = next + (parts > 1 ? 2 * m : m), *key_val = up_col + max_tree;   // (up 0xffff: the root)
  const int64_t bi = blockIdx.x / parts, b = im.b0 + bi;
  const uint32_t part = blockIdx.x % parts;
  const Batch t = load_batch(im, b, m);
  const toc_link *link = im.link + (uniform64(im.batches[b].deep_base) - (int64_t)t.n1);
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  // tree row h: its column and value, and the tree row of its parent
  auto node = [&](uint32_t h, uint32_t &up, uint32_t &col, uint32_t &val) {
    const uint32_t c = h < t.ni ? h : h - t.ni + t.n1;
    const toc_key k = t.key[c];
    const uint32_t p = c >= t.n1 ? link[c].parent : kRoot;
    up = p == kRoot || p < t.n1 ? p : p - t.n1 + t.ni;
    col = k.col;
    val = __float_as_uint(k.val);
  };
  const uint32_t lo = part * t.n_tree / parts, hi = (part + 1) * t.n_tree / parts;
  // put(u, column, value bits, first occurrence, their number) for every code on the way up
  // to the root from every one of tree codes a .. e-1 that tuples hold, the u-th of the
  // thread's in flight; begin() before each set of those
  auto walk = [&](uint32_t a, uint32_t e, auto begin, auto put) {
    for (uint32_t h0 = a + tid; h0 < e; h0 += kExpandCodes * kExpandThreads) {
      uint32_t o[kExpandCodes], n[kExpandCodes], h[kExpandCodes];
#pragma unroll
      for (int u = 0; u < kExpandCodes; ++u) {
        h[u] = h0 + (uint32_t)(u * kExpandThreads);
        o[u] = h[u] < e ? t.to[h[u]] : 0u;
        n[u] = h[u] < e ? t.to[h[u] + 1] - o[u] : 0u;
        if (n[u] == 0u) h[u] = kRoot;
      }
      begin(o, n);
      while (true) {
        uint32_t up[kExpandCodes], col[kExpandCodes], val[kExpandCodes];
        bool any = false;
#pragma unroll
        for (int u = 0; u < kExpandCodes; ++u) {
          up[u] = kRoot;
          col[u] = val[u] = 0u;
          if (h[u] == kRoot) continue;
          any = true;
          if (LDS) {
            const uint32_t w = up_col[h[u]];
            up[u] = w >> 16 == 0xffffu ? kRoot : w >> 16;
            col[u] = w & 0xffffu;
            val[u] = key_val[h[u]];
          } else {
            node(h[u], up[u], col[u], val[u]);
          }
        }
        if (!any) break;
#pragma unroll
        for (int u = 0; u < kExpandCodes; ++u) {
          if (h[u] != kRoot) put(u, col[u], val[u], o[u], n[u]);
          h[u] = up[u];
        }
      }
    }
  };
  for (int j = tid; j < (parts > 1 ? 2 * m : m); j += kExpandThreads) next[j] = 0u;
  if (LDS)
    for (uint32_t h = tid; h < t.n_tree; h += kExpandThreads) {
      uint32_t up, col;
      node(h, up, col, key_val[h]);
      up_col[h] = up << 16 | col;
    }
  __syncthreads();
  auto none = [](auto &, auto &) {};
  auto count = [&](int, uint32_t j, uint32_t, uint32_t, uint32_t n) { atomicAdd(&next[j], n); };
  if (parts > 1) {
    walk(0, lo, none, [&](int, uint32_t j, uint32_t, uint32_t, uint32_t n) { atomicAdd(&before[j], n); });
    walk(lo, t.n_tree, none, count);
    __syncthreads();
    for (int j = tid; j < m; j += kExpandThreads) next[j] += before[j];
  } else {
    walk(0, t.n_tree, none, count);
  }
  __syncthreads();
  // running sums: a thread's columns are neighbours
  const int per = (m + kExpandThreads - 1) / kExpandThreads;
  const int j0 = min(m, tid * per), j1 = min(m, j0 + per);
  uint32_t sum = 0;
  for (int j = j0; j < j1; ++j) sum += next[j];
  uint32_t at0 = sum;
#pragma unroll
  for (int s = 1; s < kWave; s *= 2) {
    const uint32_t u = (uint32_t)__shfl_up((int)at0, s, kWave);
    if (lane >= s) at0 += u;
  }
  if (lane == kWave - 1) wave_sum[wave] = at0;
  __syncthreads();
  at0 -= sum;
  for (int w = 0; w < wave; ++w) at0 += wave_sum[w];
  uint32_t *off = xoff + bi * im.xoff_stride;
  for (int j = j0; j < j1; ++j) {
    const uint32_t n = next[j];
    next[j] = at0 + (parts > 1 ? before[j] : 0u);
    if (part == 0) off[j] = at0;
    at0 += n;
  }
  if (part == 0 && tid == kExpandThreads - 1) off[m] = at0;   // (its columns, if any, are the last)
  __syncthreads();
  uint2 *const x = xpair + bi * im.x_stride;
  // (in bounds whatever the bytes that the image was built from hold)
  auto store = [&](uint32_t at, uint32_t row, uint32_t bits) {
    if (at < (uint64_t)im.x_stride) x[at] = make_uint2(row & kRowMask, bits);
  };
  uint32_t row[kExpandCodes][2];                     // the first tuples of each code
  walk(
      lo, hi,
      [&](auto &o, auto &n) {
#pragma unroll
        for (int u = 0; u < kExpandCodes; ++u)
#pragma unroll
          for (uint32_t i = 0; i < 2; ++i) row[u][i] = i < n[u] ? t.ce[o[u] + i] : 0u;
      },
      [&](int u, uint32_t j, uint32_t bits, uint32_t o, uint32_t n) {
        const uint32_t at = atomicAdd(&next[j], n);
        store(at, row[u][0], bits);
        if (n > 1) store(at + 1, row[u][1], bits);
        for (uint32_t i0 = 2; i0 < n; i0 += 4) {
          uint32_t r[4];
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i) r[i] = i0 + i < n ? t.ce[o + i0 + i] : 0u;
#pragma unroll
          for (uint32_t i = 0; i < 4; ++i)
            if (i0 + i < n) store(at + i0 + i, r[i], bits);
        }
      });
}

// Where the used columns of the chunks in flight find their entries: written by the
// first wave, from the column index loaded one and two chunks before.
constexpr int kRing = 6;
struct Ring {
  u32x4 at[kRing][kChunk];        // leaf occurrences: first and number; pairs: first and number
  uint32_t off[kRing][kChunk];    // byte offset of the column's row of W or out, or kNone
  uint32_t steps[kRing][kChunk];  // of 4 columns: most 16-entry steps of leaves, of pairs << 16
};
constexpr uint32_t kNone = 0x80000000u;

struct RingLoad {
  uint32_t jn, jp, l0, l1, x0, x1;
  __device__ void places(const Batch &t) {
    l0 = l1 = x0 = x1 = 0;
    if (jp != 0xffffffffu) {
      l0 = t.occ[jp];
      l1 = t.occ[jp + 1];
      x0 = t.xoff[jp];
      x1 = t.xoff[jp + 1];
    }
  }
  __device__ void publish(const Batch &t, Ring &ring, int slot, uint32_t i, uint32_t row_bytes) {
    ring.off[slot][i] = jp == 0xffffffffu ? kNone : jp * row_bytes;
    ring.at[slot][i] = u32x4{l0, l1 - l0, x0, x1 - x0};
    uint32_t a = (l1 - l0 + 15u) / 16u, b = (x1 - x0 + 15u) / 16u;
    a = max(a, (uint32_t)__shfl_xor((int)a, 1, kWave));
    b = max(b, (uint32_t)__shfl_xor((int)b, 1, kWave));
    a = max(a, (uint32_t)__shfl_xor((int)a, 2, kWave));
    b = max(b, (uint32_t)__shfl_xor((int)b, 2, kWave));
    ring.steps[slot][i] = a | b << 16;
  }
  __device__ static uint32_t column(const Batch &t, uint32_t at) {
    return at < t.n_used ? t.order[at] : 0xffffffffu;
  }
  // the first three chunks' places, by the first wave (before a barrier); the loads
  // of the fourth's and of the fifth's columns on their way
  __device__ void start(const Batch &t, Ring &ring, uint32_t row_bytes) {
    if (threadIdx.x >= kWave) return;
    const uint32_t i = threadIdx.x;
    jp = column(t, i);
    const uint32_t j2 = column(t, 2 * kChunk + i % kChunk);
    const uint32_t j3 = column(t, 3 * kChunk + i % kChunk);
    jn = column(t, 4 * kChunk + i % kChunk);
    places(t);
    publish(t, ring, (int)(i / kChunk), i % kChunk, row_bytes);
    jp = j2;
    places(t);
    publish(t, ring, 2, i % kChunk, row_bytes);
    jp = j3;
    places(t);
  }
  // one step per chunk: the places of chunk c + 4 to the ring, c + 5's from the
  // index, c + 6's columns from the order
  __device__ void step(const Batch &t, Ring &ring, int c, uint32_t row_bytes) {
    if (threadIdx.x >= kChunk) return;
    const uint32_t i = threadIdx.x;
    publish(t, ring, (c + 4) % kRing, i, row_bytes);
    jp = jn;
    places(t);
    jn = column(t, (uint32_t)(c + 6) * kChunk + i);
  }
};

// The entries of a chunk's columns on their way from memory to the LDS tile: a 16-lane
// group takes column kk of every chunk, its leaf occurrences from the image and its
// expanded pairs from the workspace.  load() issues the loads, a chunk's time
// before store() uses them: STEPS x 16 leaf occurrences and kXSteps x 16 pairs; a
// column with more has the rest loaded by store().
//
// store() is the serial part of a workgroup's time (one wave per SIMD runs it while
// the other multiplies), so its steps are short and free of branches: address, the
// value's high half to plane 0 (lanes without an entry write to a spare word), and the
// low halves gathered to see whether planes 1 and 2 are needed at all; they are
// written by a second pass over the same registers.
template <int STEPS>
struct Feed {
  static constexpr int kXSteps = 2;
  u32x4 at;                              // of the ring; [0] and [2] as byte offsets
  uint32_t steps, xsteps;
  uint32_t w[STEPS], v[STEPS], xw[kXSteps], xv[kXSteps];

  __device__ void load(const Batch &t, const Ring &ring, int c, uint32_t kk, uint32_t sub) {
    at = ring.at[c % kRing][kk];
    const uint32_t n =
        (uint32_t)__builtin_amdgcn_readfirstlane((int)ring.steps[c % kRing][kk & ~3u]);
    at[0] = (at[0] + 2u * sub) * 4u;
    at[2] = (at[2] + sub) * 8u;
    steps = n & 0xffffu, xsteps = n >> 16;
#pragma unroll
    for (int i = 0; i < STEPS; i += 2) {
      if ((uint32_t)i < steps) {
        // two entries a lane; past the column's end: some other entry or none, not stored
        const auto y = __builtin_amdgcn_raw_buffer_load_b64(t.ce_res, at[0], 64 * i, 0);
        const auto z = __builtin_amdgcn_raw_buffer_load_b64(t.cv_res, at[0], 64 * i, 0);
        w[i] = y[0], w[i + 1] = y[1];
        v[i] = z[0], v[i + 1] = z[1];
      }
    }
#pragma unroll
    for (int i = 0; i < kXSteps; ++i) {
      if ((uint32_t)i < xsteps) {
        const auto y = __builtin_amdgcn_raw_buffer_load_b64(t.x_res, at[2], 128 * i, 0);
        xw[i] = y[0];
        xv[i] = y[1];
      }
    }
  }

  // place(word): the LDS address of the entry's cell in plane 0; spare: an address for
  // lanes without an entry.  Returns whether the wave wrote planes 1 and 2.
  template <typename P>
  __device__ bool store(const Batch &t, uint32_t sub, uint32_t plane, uint32_t spare, Range &range,
                        P place) const {
    uint32_t low = 0;
    auto high = [&](uint32_t word, uint32_t bits, uint32_t i, uint32_t n) {
      const uint32_t to = i < n ? place(word) : spare;
      *(lds_u16 *)(size_t)to = (uint16_t)(bits >> 16);
      low |= bits << 16;
      range.add(bits);
    };
#pragma unroll
    for (int i = 0; i < STEPS; i += 2) {
      if ((uint32_t)i < steps) {
        high(w[i], v[i], 16u * i + 2u * sub, at[1]);
        high(w[i + 1], v[i + 1], 16u * i + 2u * sub + 1u, at[1]);
      }
    }
#pragma unroll
    for (int i = 0; i < kXSteps; ++i)
      if ((uint32_t)i < xsteps)
        high(xw[i], 16u * i + sub < at[3] ? xv[i] : 0u, 16u * i + sub, at[3]);
    bool both = __any(low != 0);
    auto rest = [&](uint32_t word, uint32_t bits, uint32_t i, uint32_t n) {
      const uint32_t to = i < n ? place(word) : spare;
      const float x = __uint_as_float(bits);
      const float r = x - __uint_as_float(bits & 0xffff0000u);
      const uint32_t rb = __float_as_uint(r);
      const float q = r - __uint_as_float(rb & 0xffff0000u);
      *(lds_u16 *)(size_t)(to + plane) = (uint16_t)(rb >> 16);
      *(lds_u16 *)(size_t)(to + 2 * plane) = (uint16_t)(__float_as_uint(q) >> 16);
    };
    if (both) {
#pragma unroll
      for (int i = 0; i < STEPS; i += 2) {
        if ((uint32_t)i < steps) {
          rest(w[i], v[i], 16u * i + 2u * sub, at[1]);
          rest(w[i + 1], v[i + 1], 16u * i + 2u * sub + 1u, at[1]);
        }
      }
#pragma unroll
      for (int i = 0; i < kXSteps; ++i)
        if ((uint32_t)i < xsteps) rest(xw[i], xv[i], 16u * i + sub, at[3]);
    }
    for (uint32_t i = kXSteps; i < xsteps; i += 4) {
      uint32_t y[4], z[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const auto p = __builtin_amdgcn_raw_buffer_load_b64(t.x_res, at[2] + 128u * i, 128 * u, 0);
        y[u] = p[0];
        z[u] = p[1];
      }
      low = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        high(y[u], 16u * (i + u) + sub < at[3] ? z[u] : 0u, 16u * (i + u) + sub, at[3]);
      if (__any(low != 0)) {
        both = true;
#pragma unroll
        for (int u = 0; u < 4; ++u) rest(y[u], z[u], 16u * (i + u) + sub, at[3]);
      }
    }
    return both;
  }
};

// ---------------------------------------------------------------------------
// Left product (Theorem 2): out[j, q] = sum over tuples of A[i, j] G[i, q].
// A workgroup takes a batch and 128 columns of G, 16 per wave.  A wave keeps the
// three parts of its columns of G for all tuples in registers (12 per 32 tuples)
// and the workgroup streams the used columns of A through LDS, 32 at a time, in two
// buffers: one is multiplied while the other is cleared and filled (by the 16-lane
// groups, a column each, so that one barrier per chunk is enough) from entry words
// that were loaded a chunk ahead.  So G is read once per batch and A once per 128
// columns of G, by workgroups of one XCD that run at the same time and share it in
// the L2.  250-row batches, vector kernel then this one with the expansion: 400 image-like
// batches at k = 300 417 -> 294 us (639 MB, 2.2 TB/s), 100 dense quantised ones at k = 200
// 1393 -> 264 us, of which 59 the expansion.  What is left is the serial part of a chunk:
// two waves per SIMD, whose fill (LDS writes of single values) and matrix work overlap
// little (matrix cores 18 and 22 % busy, LDS 27 and 42 %, more than half of it bank
// conflicts).  In an earlier form of this kernel, which took 338 us, one wave of a SIMD
// filling while the other multiplies, half a chunk apart, took 347 us, and bringing the
// next chunk's lines into the L2 first 401.
// Tile: [tuples / 8][32 columns] slots of 8 tuples (16 bytes), 36 slots to a row: a
// matrix operand is one 16-byte read per lane, and a wave's writes (four columns, 32
// tuples each) fall into different banks.
// ---------------------------------------------------------------------------
template <int KS>
// (64 tuples: 128 registers, so that two workgroups share a CU)
__global__ __launch_bounds__(kThreads, KS == 2 ? 4 : 2) void left_mfma_kernel(
    MfmaImg im, int64_t nb, int n_tiles, int m, const float *__restrict__ G, int64_t ldg,
    int k, float *__restrict__ out, int64_t ldo, int accumulate) {
  constexpr uint32_t kPlane = KS * 4 * kLeftRow + kSpare;
  extern __shared__ __align__(16) char lds[];   // [2 buffers][3 planes][kPlane]
  __shared__ __align__(16) Ring ring;
  __shared__ uint32_t parts[4], bad[4], bad_g;  // of chunk c at c % 4
  __shared__ uint32_t slow[kExpandCols / kChunk / 32 + 1];   // a bit per chunk left to the end; any
  const int64_t i = blockIdx.x / kXcd;
  const int64_t b = im.b0 + (i / n_tiles) * kXcd + blockIdx.x % kXcd;
  if (b >= im.b0 + nb) return;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int sub = lane % 16, grp = lane / 16;
  const int qz = (int)(i % n_tiles) * 128;
  const int q = qz + wave * 16 + sub;           // this lane's column of G and out
  const Batch t = load_batch(im, b, m);
  const float *Gb = G + t.row_base * ldg;
  float *ob = out + b * m * ldo;
  const int n_chunks = (int)((t.n_used + kChunk - 1) / kChunk);
  // Columns without entries get zeros, a wave every eighth row: the first 512 with the
  // chunks (a lane of the wave holds the column of one row), the others at the end.
  const uint32_t n_zero = accumulate ? 0u : (uint32_t)m - t.n_used;
  auto zero_row = [&](uint32_t j) {
    float *o = ob + (int64_t)j * ldo + qz;
    if (qz + lane < k) o[lane] = 0.0f;
    if (qz + lane + kWave < k) o[lane + kWave] = 0.0f;
  };
  const uint32_t zr = (uint32_t)(wave + 8 * lane);
  const uint32_t zcol = zr < n_zero ? t.order[t.n_used + zr] : 0u;
  const uint32_t z_mine = n_zero > (uint32_t)wave ? min((n_zero - wave + 7) / 8, 64u) : 0u;
  const uint32_t z_per = n_chunks ? (z_mine + n_chunks - 1) / n_chunks : 64u;
  uint32_t z = 0;
  auto zero_some = [&]() {
    for (uint32_t e = min(z + z_per, z_mine); z < e; ++z)
      zero_row((uint32_t)__builtin_amdgcn_readlane((int)zcol, (int)z));
  };
  auto zero_rest = [&]() {
    while (z < z_mine) zero_some();
    for (uint32_t r = 512 + wave; r < n_zero; r += 8)
      zero_row((uint32_t)__builtin_amdgcn_readfirstlane((int)t.order[t.n_used + r]));
  };
  if (n_chunks == 0) zero_rest();
  if (n_chunks == 0) return;            // (a batch without tuples has no row of G either)

  if (threadIdx.x < 4) parts[threadIdx.x] = bad[threadIdx.x] = 0;
  if (threadIdx.x == 0) bad_g = 0;
  constexpr int kSlow = kExpandCols / kChunk / 32;
  if (threadIdx.x <= kSlow) slow[threadIdx.x] = 0;
  RingLoad index;
  index.start(t, ring, (uint32_t)ldo * 4u);
  const uint32_t kk = (uint32_t)(wave * 4 + grp);
  Feed<2 * KS> feed;

  // G: lane holds tuples 32 s + 8 grp .. + 7 of column q, scaled by 2^shift so that the
  // column's largest value is in the topmost binade
  u32x4 g[KS][3];
  Range range;
  int shift;
  {
    float x[KS][8];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = 32 * s + 8 * grp + e;
        const bool ok = r < t.n_rows && q < k;
        const float y = Gb[ok ? (int64_t)r * ldg + q : 0];
        x[s][e] = ok ? y : 0.0f;
        range.add(__float_as_uint(x[s][e]));
      }
    }
    // (the four lanes of a column)
    uint32_t top = max(range.hi, (uint32_t)__shfl_xor((int)range.hi, 16, kWave));
    top = max(top, (uint32_t)__shfl_xor((int)top, 32, kWave));
    shift = top ? kDenseTop - 1 + 127 - (int)(top >> 23) : 0;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[s][e] = ldexpf(x[s][e], shift);
      split8(x[s], g[s]);
    }
  }
  __syncthreads();
  if (range.hi >= 0x7f800000u ||
      (range.hi && fabsf(ldexpf(__uint_as_float(range.lo + 1u), shift)) < kDenseLo))
    bad_g = 1;
  feed.load(t, ring, 0, kk, sub);

  const auto ores = __builtin_amdgcn_make_buffer_rsrc(
      ob, (short)0, (int)(((int64_t)(m - 1) * ldo + k) * 4), 0x00020000);
  const uint32_t qoff = q < k ? (uint32_t)q * 4u : 0x40000000u;   // beyond the buffer: not stored
  uint32_t used = 3;                    // buffers (a bit each) whose planes 1 and 2 are not clear
  // chunk c's results, stored by the wave's next half so that no wait for that half's
  // entry words includes them
  float res[2][4];
  int res_chunk = -1;
  auto put_out = [&]() {
    if (res_chunk < 0) return;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      const u32x4 off = *(const tile_u32x4 *)&ring.off[res_chunk % kRing][mt * 16 + grp * 4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float r = res[mt][e];
        if (accumulate)
          r += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ores, off[e] + qoff, 0, 0));
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r), ores, off[e] + qoff, 0, 0);
      }
    }
    res_chunk = -1;
  };
  auto produce = [&](int c) {
    if (c + 1 < n_chunks) {
      // the group's column of chunk c + 1's buffer cleared, then the loaded words
      // written to it (a wave's LDS operations stay in order)
      char *tile = lds + ((c + 1) & 1) * 3 * kPlane;
      const uint32_t bit = 1u << ((c + 1) & 1);
#pragma unroll
      for (int h = 0; h < KS / 4 + (KS < 4); ++h) {
        const uint32_t rg = sub + 16u * h;
        char *o = tile + rg * kLeftRow + kk * 16u;
        if (KS >= 4 || rg < KS * 4) {
          *(tile_u32x4 *)o = u32x4{0, 0, 0, 0};
          if (used & bit) {
            *(tile_u32x4 *)(o + kPlane) = u32x4{0, 0, 0, 0};
            *(tile_u32x4 *)(o + 2 * kPlane) = u32x4{0, 0, 0, 0};
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      Range vr;
      const uint32_t base = lds_address(tile) + kk * 16u;
      const uint32_t spare = lds_address(tile) + kPlane - kSpare + (uint32_t)lane * 4u;
      const bool low = feed.store(t, sub, kPlane, spare, vr, [&](uint32_t word) {
        return base + (word >> 3 & (4u * KS - 1u)) * kLeftRow + (word & 7u) * 2u;
      });
      used &= ~bit;
      if (low) {
        used |= bit;
        parts[(c + 1) & 3] = 1;
      }
      if (vr.outside(kValLo, kValHi)) bad[(c + 1) & 3] = 1;
    }
    if (threadIdx.x == 0) parts[(c + 2) & 3] = bad[(c + 2) & 3] = 0;
    index.step(t, ring, c, (uint32_t)ldo * 4u);
    put_out();
    zero_some();
    if (c + 2 < n_chunks) {
      feed.load(t, ring, c + 2, kk, sub);
    }
  };
  auto consume = [&](int c) {
    const char *tile = lds + (c & 1) * 3 * kPlane;
    // the chunk's two halves of 16 columns in turn, the next operand read while the
    // last is multiplied; lo, lo2: the small products
    f32x4 hi[2] = {}, lo[2] = {}, lo2[2] = {};
    const char *ta = tile + grp * kLeftRow + sub * 16;
    auto operand = [&](int at, int plane) {
      return *(const tile_u32x4 *)(ta + plane * kPlane + (at / 2) * (4 * kLeftRow) + (at % 2) * 256);
    };
    if (__builtin_amdgcn_readfirstlane((int)parts[c & 3]) == 0) {
      u32x4 next = operand(0, 0), next2 = operand(1, 0);
#pragma unroll
      for (int at = 0; at < 2 * KS; ++at) {
        const int s = at / 2, mt = at % 2;
        const u32x4 a = next;
        next = next2;
        if (at + 2 < 2 * KS) next2 = operand(at + 2, 0);
        lo[mt] = mfma(a, g[s][2], lo[mt]);
        hi[mt] = mfma(a, g[s][0], hi[mt]);
        lo2[mt] = mfma(a, g[s][1], lo2[mt]);
      }
    } else {
      u32x4 next[3];
#pragma unroll
      for (int pl = 0; pl < 3; ++pl) next[pl] = operand(0, pl);
#pragma unroll
      for (int at = 0; at < 2 * KS; ++at) {
        const int s = at / 2, mt = at % 2;
        const u32x4 a1 = next[0], a2 = next[1], a3 = next[2];
        if (at + 1 < 2 * KS) {
#pragma unroll
          for (int pl = 0; pl < 3; ++pl) next[pl] = operand(at + 1, pl);
        }
        lo[mt] = mfma(a2, g[s][2], lo[mt]);
        hi[mt] = mfma(a1, g[s][0], hi[mt]);
        lo2[mt] = mfma(a1, g[s][1], lo2[mt]);
        lo[mt] = mfma(a3, g[s][1], lo[mt]);
        lo2[mt] = mfma(a2, g[s][0], lo2[mt]);
        lo[mt] = mfma(a1, g[s][2], lo[mt]);
        lo[mt] = mfma(a2, g[s][1], lo[mt]);
        lo[mt] = mfma(a3, g[s][0], lo[mt]);
      }
    }
    if (__builtin_amdgcn_readfirstlane((int)(bad[c & 3] | bad_g)) == 0) {
      res_chunk = c;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          res[mt][e] = ldexpf(hi[mt][e] + (lo[mt][e] + lo2[mt][e]), -shift);
    } else if (threadIdx.x == 0) {
      slow[c / 32] |= 1u << (c % 32);
      slow[kSlow] = 1;
    }
  };
  for (int c = -1; c < n_chunks; ++c) {
    if (c >= 0) consume(c);
    produce(c);
    __syncthreads();
  }
  put_out();
  zero_rest();
  if (!__builtin_amdgcn_readfirstlane((int)slow[kSlow])) return;
  // The chunks left, term by term: 64 columns of G at a time in LDS, a wave per column of
  // A, its leaf occurrences 64 at a time and then its tree codes' pairs.
  float *Gs = (float *)lds;
  for (int h = 0; h < 128 && qz + h < k; h += kWave) {
    const int qq = qz + h + lane;
    __syncthreads();
    for (int r = wave; r < t.n_rows; r += kThreads / kWave)
      Gs[r * kWave + lane] = Gb[(int64_t)r * ldg + min(qq, k - 1)];
    __syncthreads();
    for (int c = 0; c < n_chunks; ++c) {
      if (!((uint32_t)__builtin_amdgcn_readfirstlane((int)slow[c / 32]) >> (c % 32) & 1u)) continue;
      // (the wave's four columns' first entries are loaded together)
      uint32_t j[4], o[4], end[4];
      int row[4], v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t at = (uint32_t)c * kChunk + (uint32_t)(wave * 4 + i);
        j[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)t.order[min(at, t.n_used - 1)]);
      }
      auto load = [&](int i) {
        const uint32_t x = min(o[i] + (uint32_t)lane, max(end[i], 1u) - 1);
        row[i] = (int)(t.ce[x] & kRowMask) * kWave;
        v[i] = (int)t.cv[x];
      };
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = t.occ[j[i]], end[i] = t.occ[j[i] + 1];
#pragma unroll
      for (int i = 0; i < 4; ++i) load(i);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if ((uint32_t)c * kChunk + (uint32_t)(wave * 4 + i) >= t.n_used) break;
        float sum = 0.0f, part = 0.0f;
        uint32_t n = 0;
        auto term = [&](int x, float y) {
          part = fmaf(__int_as_float(x), y, part);
          if ((++n & 15u) == 0) sum += part, part = 0.0f;
        };
        while (o[i] < end[i]) {
          const int count = (int)min(end[i] - o[i], (uint32_t)kWave);
          int u = 0;
          for (; u + 16 <= count; u += 16) {
            float y[16];
#pragma unroll
            for (int x = 0; x < 16; ++x) y[x] = Gs[__builtin_amdgcn_readlane(row[i], u + x) + lane];
#pragma unroll
            for (int x = 0; x < 16; ++x) term(__builtin_amdgcn_readlane(v[i], u + x), y[x]);
          }
          for (; u < count; ++u)
            term(__builtin_amdgcn_readlane(v[i], u), Gs[__builtin_amdgcn_readlane(row[i], u) + lane]);
          o[i] += kWave;
          if (o[i] < end[i]) load(i);
        }
        tree_pairs(t, t.tf[j[i]], t.tf[j[i] + 1], [&](int r, int x) { term(x, Gs[r * kWave + lane]); });
        sum += part;
        if (qq < k) {
          float *p = ob + (int64_t)j[i] * ldo + qq;
          *p = accumulate ? *p + sum : sum;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Right product (Theorem 1): R[i, q] = sum over used columns of A[i, j] W[j, q].
// A workgroup takes a batch and N = 16 NF (8 / WM) columns of W and keeps that
// part of R in registers (a wave: 64 tuples x 16 NF columns); the used columns of A
// and the rows of W they name stream through LDS, 32 at a time, double-buffered as
// in the left product.  W is split into its parts on the way (it stays in the L2).
// 400 image-like batches at k = 300 382 -> 262 us, 100 dense quantised ones at k = 200
// 1278 -> 247 us (matrix cores 22 and 24 % busy).  NF = 5 (two tiles instead of three at
// k = 300) spills: 434 us.
// Tiles: A [8][64 WM tuples] slots of 4 columns (8 bytes), W [4][N] slots of 8 rows; a
// wave owns the 4 columns of one slot row, which it clears and fills by itself.
// ---------------------------------------------------------------------------
template <int WM, int NF>
__global__ __launch_bounds__(kThreads) void right_mfma_kernel(
    MfmaImg im, int64_t nb, int n_tiles, int m, const float *__restrict__ W, int64_t ldw,
    int k, float *__restrict__ R, int64_t ldr) {
  constexpr int kRows = 64 * WM, kWn = 8 / WM, N = 16 * NF * kWn;
  constexpr int kSteps = kRows / 16;
  constexpr uint32_t kPlane = 4 * kRows * 16 + kSpare, kBPlane = 4 * N * 16;
  constexpr int kTasks = (4 * N + kThreads - 1) / kThreads;   // slots of W per thread
  extern __shared__ __align__(16) char lds[];          // A [2][3][kPlane], W [2][3][kBPlane]
  __shared__ __align__(16) Ring ring;
  __shared__ uint32_t parts[4], bad;     // parts of chunk c at c % 4
  const int64_t i = blockIdx.x / kXcd;
  const int64_t b = im.b0 + (i / n_tiles) * kXcd + blockIdx.x % kXcd;
  if (b >= im.b0 + nb) return;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int sub = lane % 16, grp = lane / 16;
  const int wm = wave % WM, wn = wave / WM;
  const int q0 = (int)(i % n_tiles) * N;
  const Batch t = load_batch(im, b, m);
  const int n_chunks = (int)((t.n_used + kChunk - 1) / kChunk);
  const auto wres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float *>(W), (short)0, (int)(((int64_t)(m - 1) * ldw + k) * 4), 0x00020000);
  char *ldsB = lds + 6 * kPlane;

  if (threadIdx.x < 4) parts[threadIdx.x] = 0;
  if (threadIdx.x == 0) bad = 0;
  const uint32_t kk = (uint32_t)(wave * 4 + grp);   // this group's column within a chunk
  RingLoad index;
  index.start(t, ring, (uint32_t)ldw * 4u);
  Feed<kSteps> feed;

  float w[kTasks][8];
  Range range;
  auto load_w = [&](int c) {
#pragma unroll
    for (int e = 0; e < kTasks; ++e) {
      const int task = threadIdx.x + e * kThreads;
      if (task < 4 * N) {
        const uint32_t n = (uint32_t)(task % N);
        const uint32_t *rows = ring.off[c % kRing] + 8 * (task / N);
        // a row that is not there, or a column beyond k: outside the buffer, read as 0
        const uint32_t off = q0 + (int)n < k ? (uint32_t)(q0 + n) * 4u : 0x40000000u;
#pragma unroll
        for (int r = 0; r < 8; ++r)
          w[e][r] =
              __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wres, rows[r] + off, 0, 0));
      }
    }
  };
  auto store_w = [&](int c) {
    char *tile = ldsB + (c & 1) * 3 * kBPlane;
#pragma unroll
    for (int e = 0; e < kTasks; ++e) {
      const int task = threadIdx.x + e * kThreads;
      if (task < 4 * N) {
        u32x4 p[3];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          range.add(__float_as_uint(w[e][r]));
          w[e][r] *= kWUp;
        }
        split8(w[e], p);
#pragma unroll
        for (int s = 0; s < 3; ++s) *(u32x4 *)(tile + s * kBPlane + task * 16) = p[s];
      }
    }
  };
  bool out_of_range = false;
  f32x4 acc[4][NF] = {};
  uint32_t used = 3;                     // buffers whose planes 1 and 2 are not clear
  auto produce = [&](int c) {
    if (c + 1 < n_chunks) {
      char *tile = lds + ((c + 1) & 1) * 3 * kPlane + wave * (kRows * 8);
      const uint32_t bit = 1u << ((c + 1) & 1);
#pragma unroll
      for (int o = 0; o < kRows * 8; o += kWave * 16) {
        if (kRows * 8 >= kWave * 16 || lane * 16 < kRows * 8) {
          *(tile_u32x4 *)(tile + o + lane * 16) = u32x4{0, 0, 0, 0};
          if (used & bit) {
            *(tile_u32x4 *)(tile + kPlane + o + lane * 16) = u32x4{0, 0, 0, 0};
            *(tile_u32x4 *)(tile + 2 * kPlane + o + lane * 16) = u32x4{0, 0, 0, 0};
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      Range vr;
      const uint32_t base = lds_address(tile) + (uint32_t)grp * 2u;
      const uint32_t spare = lds_address(lds) + ((c + 1) & 1) * 3 * kPlane + kPlane - kSpare +
                             (uint32_t)lane * 4u;
      const bool low = feed.store(t, sub, kPlane, spare, vr, [&](uint32_t word) {
        return base + (word & (kRows - 1u)) * 8u;
      });
      used &= ~bit;
      if (low) {
        used |= bit;
        parts[(c + 1) & 3] = 1;
      }
      out_of_range |= vr.outside(kValLo, kValHi);
      store_w(c + 1);
    }
    if (threadIdx.x == 0) parts[(c + 2) & 3] = 0;
    index.step(t, ring, c, (uint32_t)ldw * 4u);
    if (c + 2 < n_chunks) {
      load_w(c + 2);
      feed.load(t, ring, c + 2, kk, sub);
    }
  };
  auto consume = [&](int c) {
    // lane (sub, grp): columns 8 grp .. + 7 of a tuple, in two slots
    const char *ta = lds + (c & 1) * 3 * kPlane + (2 * grp * kRows + wm * 64 + sub) * 8;
    const char *tb = ldsB + (c & 1) * 3 * kBPlane + (grp * N + wn * 16 * NF + sub) * 16;
    auto load_a = [&](int s, int x) {
      const u32x2 l = *(const tile_u32x2 *)(ta + s * kPlane + x * 128);
      const u32x2 h = *(const tile_u32x2 *)(ta + s * kPlane + x * 128 + kRows * 8);
      return u32x4{l[0], l[1], h[0], h[1]};
    };
    if (__builtin_amdgcn_readfirstlane((int)parts[c & 3]) == 0) {
      u32x4 a[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) a[x] = load_a(0, x);
      u32x4 next[3];
#pragma unroll
      for (int s = 0; s < 3; ++s) next[s] = *(const tile_u32x4 *)(tb + s * kBPlane);
#pragma unroll
      for (int n = 0; n < NF; ++n) {
        u32x4 w3[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          w3[s] = next[s];
          if (n + 1 < NF) next[s] = *(const tile_u32x4 *)(tb + s * kBPlane + (n + 1) * 256);
        }
        f32x4 hi[4] = {}, lo[4] = {};
#pragma unroll
        for (int x = 0; x < 4; ++x) lo[x] = mfma(a[x], w3[2], lo[x]);
#pragma unroll
        for (int x = 0; x < 4; ++x) hi[x] = mfma(a[x], w3[0], hi[x]);
#pragma unroll
        for (int x = 0; x < 4; ++x) lo[x] = mfma(a[x], w3[1], lo[x]);
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[x][n] += hi[x] + lo[x];
      }
    } else {
#pragma unroll
      for (int xh = 0; xh < 4; xh += 2) {
        u32x4 a[2][3];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int s = 0; s < 3; ++s) a[x][s] = load_a(s, xh + x);
#pragma unroll
        for (int n = 0; n < NF; ++n) {
          u32x4 w3[3];
#pragma unroll
          for (int s = 0; s < 3; ++s) w3[s] = *(const tile_u32x4 *)(tb + s * kBPlane + n * 256);
          f32x4 hi[2] = {}, lo[2] = {};
          auto small = [&](int p, int r) {
#pragma unroll
            for (int x = 0; x < 2; ++x) lo[x] = mfma(a[x][p], w3[r], lo[x]);
          };
          small(2, 1);
          small(1, 2);
          small(2, 0);
          small(1, 1);
          small(0, 2);
          small(1, 0);
          small(0, 1);
#pragma unroll
          for (int x = 0; x < 2; ++x) hi[x] = mfma(a[x][0], w3[0], hi[x]);
#pragma unroll
          for (int x = 0; x < 2; ++x) acc[xh + x][n] += hi[x] + lo[x];
          __builtin_amdgcn_sched_barrier(0);   // (loads hoisted further ahead spill)
        }
      }
    }
  };
  __syncthreads();
  if (n_chunks) {
    load_w(0);
    feed.load(t, ring, 0, kk, sub);
  }
  for (int c = n_chunks ? -1 : 0; c < n_chunks; ++c) {
    if (c >= 0) consume(c);
    produce(c);
    __syncthreads();
  }
  if (out_of_range || range.outside(kWLo, kWHi)) bad = 1;
  __syncthreads();
  float *Rb = R + t.row_base * ldr;
  if (!bad) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = wm * 64 + x * 16 + grp * 4 + e;
#pragma unroll
        for (int n = 0; n < NF; ++n) {
          const int q = q0 + (wn * NF + n) * 16 + sub;
          if (r < t.n_rows && q < k) Rb[(int64_t)r * ldr + q] = acc[x][n][e] * (1.0f / kWUp);
        }
      }
    }
    return;
  }
  // term by term: a wave per tuple, a lane per code, all walked to the root together; the
  // rows of W of eight pairs are loaded together
  const toc_batch *bp = im.batches + b;
  const uint32_t *span = im.span + uniform64(bp->span_base);
  const uint32_t *D = im.dcodes + uniform64(bp->d_base);
  const toc_key *key = im.key + uniform64(bp->code_base);
  const toc_link *link = im.link + (uniform64(bp->deep_base) - (int64_t)t.n1);
  constexpr int kH = (N + kWave - 1) / kWave;            // 64-column parts of the tile
  const int parts_k = min(kH, (k - q0 + kWave - 1) / kWave);
  for (int r = wave; r < t.n_rows; r += kThreads / kWave) {
    float sum[kH] = {}, part[kH] = {};
    uint32_t n = 0;
    const uint32_t end = span[r + 1];
    for (uint32_t e = span[r]; e < end; e += kWave) {
      uint32_t c = e + (uint32_t)lane < end ? D[e + (uint32_t)lane] : kRoot;
      uint64_t on;
      while ((on = __ballot(c != kRoot)) != 0) {
        const toc_key y = c != kRoot ? key[c] : toc_key{0u, 0.0f};
        c = c != kRoot && c >= t.n1 ? link[c].parent : kRoot;
        const int col = (int)y.col, val = __float_as_int(y.val);
        while (on) {
          float x[8][kH];
          int v[8];
          const int count = min((int)__popcll(on), 8);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int l = __builtin_ctzll(on | 1ull << 63);      // (past the last: any lane)
            if (u < count) on &= on - 1;
            v[u] = __builtin_amdgcn_readlane(val, l);
            const float *Wr = W + (int64_t)__builtin_amdgcn_readlane(col, l) * ldw;
#pragma unroll
            for (int h = 0; h < kH; ++h)
              if (h < parts_k) x[u][h] = Wr[min(q0 + h * kWave + lane, k - 1)];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (u >= count) break;
            ++n;
#pragma unroll
            for (int h = 0; h < kH; ++h) {
              if (h < parts_k) part[h] = fmaf(__int_as_float(v[u]), x[u][h], part[h]);
              if ((n & 15u) == 0) sum[h] += part[h], part[h] = 0.0f;
            }
          }
        }
      }
    }
#pragma unroll
    for (int h = 0; h < kH; ++h) {
      const int q = h * kWave + lane;
      if (q < N && q0 + q < k) Rb[(int64_t)r * ldr + q0 + q] = sum[h] + part[h];
    }
  }
}

MfmaImg image_of(const toc_dev *d) {
  const uint8_t *p = (const uint8_t *)d->buf;
  const toc_layout &L = d->layout;
  MfmaImg im{};
  im.batches = (const toc_batch *)(p + L.batches);
  im.key = (const toc_key *)(p + L.key);
  im.link = (const toc_link *)(p + L.link);
  im.span = (const uint32_t *)(p + L.span);
  im.dcodes = (const uint32_t *)(p + L.dcodes);
  im.centry = (const uint32_t *)(p + L.centry);
  im.cval = (const uint32_t *)(p + L.cval);
  im.occ_off = (const uint32_t *)(p + L.occ_off);
  im.tlist = (const uint32_t *)(p + L.tlist);
  im.cols = (const uint32_t *)(p + L.cols);
  im.tchild = (const uint32_t *)(p + L.tchild);
  return im;
}

// Workspace of a run of n batches: their columns' first pairs (m + 1 words a batch,
// rounded up to 16 bytes), then room for the pairs of the batch with the most.
int64_t offsets_words(const toc_dev *d) { return ((int64_t)d->info.n_cols + 4) / 4 * 4; }
size_t pass_bytes(const toc_dev *d, int64_t n) {
  return (size_t)(n * (4 * offsets_words(d) + 8 * std::max<int64_t>(d->max_tree_pairs, 1)));
}
// Asked for at most; more is used when given.
constexpr size_t kPassBytes = TOC_NOALLOC_SCRATCH_BYTES;
constexpr size_t kExpandLds = 152 * 1024;

// Batches full of deep codes (dense quantised ones).
bool many_deep(const toc_dev *d) {
  const toc_dev_info &n = d->info;
  return n.nnz * 2 >= n.n_rows * d->max_ucols && n.n_deep * 32 > n.n_stored;
}

// The batches that a pass has to hold: enough for 192 pairs of batch and 128-column tile,
// three quarters of the chip's CUs (1,200 image-like batches at k = 300, left: passes of
// 21 batches 3.8 ms, of 42 1.9 ms, one pass 0.87 ms, vector kernel 1.3 ms), or for 64
// where the vector kernels are four times slower (200 dense quantised batches at k = 200,
// left: passes of 34 batches 1.5 ms, one pass 0.53 ms, vector kernel 2.7 ms).
int64_t least_batches(const toc_dev *d, int32_t k, bool right) {
  const int64_t pairs = many_deep(d) || (right && k < 4) ? 64 : 192, tiles = (k + 127) / 128;
  return std::min(d->info.n_batches, (pairs + tiles - 1) / tiles);
}

// Workgroups that share a batch's tree codes in a pass of n batches: one where a workgroup
// has them all in flight, else as many as the chip's CUs allow (dense quantised batches of
// 15,005 tree codes, k = 200, right and left with one workgroup, then with several: one
// batch 214 -> 196 and 227 -> 207 us, 100 223 -> 204 and 275 -> 260; 200 batches with two
// each 487 -> 525 and 529 -> 550).
int expand_parts(const toc_dev *d, int64_t n) {
  return d->max_tree <= kExpandCodes * kExpandThreads
             ? 1
             : (int)std::max<int64_t>(1, std::min<int64_t>(256 / n, 8));
}

// Per pass of batches, of one size: their tree codes expanded into the workspace, then
// `kernel` over all (batch, tile) pairs, the tiles of a batch on one XCD.
template <typename K, typename... Args>
toc_status run(const char *name, K kernel, size_t lds, const toc_dev *d, int n_tiles, void *ws,
               size_t ws_bytes, hipStream_t s, Args... args) {
  const int64_t nb = d->info.n_batches, m = d->info.n_cols;
  // the tree codes in LDS, where it holds them beside the columns' counts; see expand_parts
  const size_t lds_t = 8 * (size_t)m + 8 * (size_t)d->max_tree;
  const bool tree_lds = d->max_tree < 0xffff && lds_t <= kExpandLds;
  const size_t lds_x = tree_lds ? lds_t : 8 * (size_t)m;
  const auto expand = tree_lds ? tree_expand_kernel<true> : tree_expand_kernel<false>;
  auto allow = [](const void *f, size_t bytes) {
    return bytes <= 48 * 1024 ||
           hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
  };
  if (!allow((const void *)kernel, lds) || !allow((const void *)expand, lds_x))
    return fail(TOC_EDEVICE, "cannot raise dynamic LDS to %zu bytes", std::max(lds, lds_x));
  const int64_t most = std::min<int64_t>(((int64_t)1 << 21) / n_tiles, (int64_t)(ws_bytes / pass_bytes(d, 1)));
  const int64_t n_passes = (nb + most - 1) / most, per = (nb + n_passes - 1) / n_passes;
  for (int64_t b0 = 0; b0 < nb; b0 += per) {
    const int64_t n = std::min(nb - b0, per);
    MfmaImg im = image_of(d);
    im.b0 = b0;
    im.xoff_stride = offsets_words(d);
    im.x_stride = std::max<int64_t>(d->max_tree_pairs, 1);
    uint32_t *xoff = (uint32_t *)ws;
    uint2 *xpair = (uint2 *)(xoff + n * im.xoff_stride);
    im.xoff = xoff;
    im.xpair = xpair;
    const int parts = tree_lds ? expand_parts(d, n) : 1;
    hipLaunchKernelGGL(expand, dim3((unsigned)(n * parts)), dim3(kExpandThreads), lds_x, s, im, (int)m,
                       (int)d->max_tree, parts, xoff, xpair);
    const unsigned grid = (unsigned)((n + kXcd - 1) / kXcd * kXcd * n_tiles);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), lds, s, im, n, n_tiles, args...);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(TOC_EDEVICE, "%s: %s", name, hipGetErrorString(e));
  return TOC_OK;
}

}  // namespace

namespace {

// Tiles of a right product and the 16-column fragments of a wave; returns the waves along
// the tuples.
int right_tiles(const toc_dev *d, int32_t k, int &n_tiles, int &f) {
  const int wm = d->max_rows <= 64 ? 1 : d->max_rows <= 128 ? 2 : 4;
  const int wn = 8 / wm, most = wm == 1 ? 2 : 4;
  const int nf = (k + 15) / 16;
  n_tiles = (nf + wn * most - 1) / (wn * most);
  f = (nf + wn * n_tiles - 1) / (wn * n_tiles);
  return wm;
}

// Whether these kernels are the faster ones for batches that are mostly leaves (image-like).
// They multiply whole tiles: 64, 128 or 256 tuples whatever a batch has, in rounds of as
// many workgroups as the CUs hold, and where values are not one bf16 number, eight products
// instead of three; the vector kernels' time follows the nonzeros, in rounds of a batch and
// 64 columns to a CU.  So with batches of 130 tuples of fractional values calls take longer
// here (300 batches, k = 300, right 303 us against 194, left 343 against 240), with whole
// numbers the same (197 and 194), and with 250 tuples less (234 and 329).  Both times (us)
// are fitted to 75 to 1,000 image-like batches of 10 to 250 tuples, k of 66 to 300 and both
// kinds of values, and are right to 5 % (RMS); the calls of that range that go to the slower
// kernel lose 1 % on average.
bool mfma_faster(const toc_dev *d, int32_t k, bool right) {
  const int64_t nb = d->info.n_batches;
  const int size = d->max_rows <= 64 ? 0 : d->max_rows <= 128 ? 1 : 2, parts = d->any_parts;
  const int64_t chunks = (d->total_ucols + nb * kChunk - 1) / (nb * kChunk);
  int64_t groups, at_once = 256;
  double chunk;                             // a chunk of a round of workgroups
  if (right) {
    static const double us[2][3][4] = {
        {{1.65, 2.35, 2.35, 2.35}, {2.0, 2.25, 2.6, 3.1}, {2.0, 2.4, 2.7, 3.0}},
        {{2.35, 3.3, 3.3, 3.3}, {2.6, 3.2, 3.9, 4.9}, {2.7, 3.4, 4.2, 4.8}}};
    int n_tiles, f;
    right_tiles(d, k, n_tiles, f);
    groups = nb * n_tiles;
    chunk = us[parts][size][f - 1];
    if (size == 0 && f == 1 && groups > 256) chunk *= 0.75;   // (two workgroups to a CU)
  } else {
    static const double us[2][3] = {{4.0, 2.8, 3.3}, {4.9, 3.7, 5.6}};
    groups = nb * ((k + 127) / 128);
    if (size == 0) at_once = 512;
    chunk = us[parts][size];
    if (size == 0 && groups <= 512) chunk *= groups <= 256 ? 0.55 : 0.65;
  }
  const double here = 20 + (double)((groups + at_once - 1) / at_once) * (double)chunks * chunk;
  const int64_t items = nb * ((k + 63) / 64), whole = (items + 255) / 256;
  const double pairs = (double)d->info.nnz / (double)nb * 1e-3, part = (double)items / 256;
  const double there = right
                           ? 16.5 + (0.8 * (double)whole + 0.2 * part) * (1.07 * pairs + 8.7)
                           : 14.9 + (0.7 * (double)whole + 0.3 * part) * (1.16 * pairs + 13.5);
  return here < there;
}

}  // namespace

namespace toc {

// Where these kernels are the faster ones.  Against the vector kernels of
// toc_device.hip (right / left, us a call alone, vector then matrix; 250-row batches):
//  - dense quantised batches, whose many deep codes cost those a table row each:
//    always (100 batches, k = 200: 1305 -> 259, 1416 -> 287; one batch, k = 8: 311 -> 138,
//    414 -> 210).  A right product of batches with far fewer codes than nonzeros
//    runs on the codes instead (400 census batches, k = 20: 132 both ways, 50 of 100 rows,
//    k = 10: 41 against 78; their left products 370 -> 154 and 116 -> 82);
//  - others (image-like, one-hot): when the pairs of batches and 64-column tiles fill
//    the chip and more than one tile shares a batch's expansion, and, of batches that are
//    mostly leaves, when mfma_faster says so (400 image-like
//    batches, k = 300: 445 -> 278, 494 -> 320; 64 batches: 114 -> 73, 124 -> 75; 150, k =
//    100: 113 -> 73, 123 -> 76; one-hot batches, left: 400, k = 100 406 -> 186, k = 300
//    814 -> 394, 150, k = 130 198 -> 160; but 64 image-like batches at k = 128: 66 and 69
//    against 68 and 73, 400 of 100 rows at k = 20: 44 and 72 against 74 and 89);
//  - right products of 2 and 3 columns, which only the general kernel took (400
//    image-like batches, k = 2: 2382 -> 87).
// Below a sixteenth of the tiles' cells filled (sparse text) the expansion is mostly zeros.
bool mfma_suits(const toc_dev *d, int32_t k, bool right) {
  const toc_dev_info &n = d->info;
  if (k < 2 || d->max_rows > 256 || d->max_ucols < 1) return false;
  // a tile has one cell for a tuple and a column
  if (d->max_tree_pairs < 0) return false;
  if (n.n_cols > kExpandCols || pass_bytes(d, least_batches(d, k, right)) > kPassBytes) return false;
  const int64_t cells = n.n_rows * d->max_ucols;
  if (n.nnz * 16 < cells) return false;
  if (right && k < 4) return true;
  if (right && n.n_codes * 10 < n.nnz * 9) return false;
  if (many_deep(d)) return true;
  if (k <= 64 || n.n_batches * ((k + 63) / 64) < 300) return false;
  return d->max_tree * 8 > d->max_codes || mfma_faster(d, k, right);
}

size_t mfma_workspace(const toc_dev *d) {
  return std::min(pass_bytes(d, d->info.n_batches), kPassBytes);
}

bool mfma_fits(const toc_dev *d, int32_t k, bool right, int64_t ld, const void *ws,
               size_t ws_bytes) {
  // 32-bit byte offsets into W and a batch's block of out
  if (!mfma_suits(d, k, right) || (int64_t)d->info.n_cols * ld >= ((int64_t)1 << 28)) return false;
  return ws && ((uintptr_t)ws & 15) == 0 && ws_bytes >= pass_bytes(d, least_batches(d, k, right));
}

toc_status left_mfma(const toc_dev *d, const float *G, int32_t k, int64_t ldg, float *out, int64_t ldo,
                     int32_t accumulate, void *ws, size_t ws_bytes, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const int n_tiles = (k + 127) / 128;
  const int ks = d->max_rows <= 64 ? 2 : d->max_rows <= 128 ? 4 : 8;
  const size_t lds = (size_t)6 * (ks * 4 * kLeftRow + kSpare);
  const int m = d->info.n_cols;
#define TOC_LM(KS)                                                                              \
  return run("left_mfma_kernel", left_mfma_kernel<KS>, lds, d, n_tiles, ws, ws_bytes, s, m, G, ldg, \
             (int)k, out, ldo, (int)accumulate)
  if (ks == 2) TOC_LM(2);
  if (ks == 4) TOC_LM(4);
  TOC_LM(8);
#undef TOC_LM
}

toc_status right_mfma(const toc_dev *d, const float *W, int32_t k, int64_t ldw, float *R, int64_t ldr,
                      void *ws, size_t ws_bytes, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  int n_tiles, f;
  const int wm = right_tiles(d, k, n_tiles, f), wn = 8 / wm;
  const size_t lds = (size_t)6 * (4 * 16 * (64 * wm + 16 * f * wn) + kSpare);
  const int m = d->info.n_cols;
#define TOC_RM(WM, NF)                                                                          \
  if (wm == WM && f == NF)                                                                      \
    return run("right_mfma_kernel", right_mfma_kernel<WM, NF>, lds, d, n_tiles, ws, ws_bytes, s, m, W, \
               ldw, (int)k, R, ldr)
  TOC_RM(4, 1);
  TOC_RM(4, 2);
  TOC_RM(4, 3);
  TOC_RM(4, 4);
  TOC_RM(2, 1);
  TOC_RM(2, 2);
  TOC_RM(2, 3);
  TOC_RM(2, 4);
  TOC_RM(1, 1);
  TOC_RM(1, 2);
#undef TOC_RM
  return fail(TOC_EINVAL, "no right_mfma_kernel for %d fragments", f);
}

}  // namespace toc
