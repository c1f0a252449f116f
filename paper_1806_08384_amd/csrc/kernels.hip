// kernels.hip -- gfx950 kernels of the exact-selectivity path.
//
//  k_scan<M_COUNT>      fused predicate evaluation + COUNT(*)   (Ch.3 sec.3.1)
//  k_scan<M_MASK>       same, also writing the per-row result mask and the
//                       per-tile TRUE counts that materialisation needs
//                       (Algorithm 1: count first, then materialise)
//  k_scan<M_KEYBITMAP>  same, setting bit (key - key_min) for every TRUE
//                       row of a pushed-down dimension (Ch.3 sec.3.3)
//  k_chunk_scan         exclusive scan of the per-tile counts in chunks (tables
//                       of more than one tile per wave)
//  k_compact            mask -> ascending row ids
//  k_gather             projected columns at given row ids
//  k_luts, k_lbatch     many programs over several tables, one count each:
//                       one lookup per column and row serves them all
//  k_tables, k_batch    the same for programs outside conjunctive form
//
// Evaluation is bit-sliced: each lane owns 32 rows of a 2048-row wave tile
// (sel_device.h) and every truth value of SQL's three-valued logic is a pair
// of 32-bit words (t, f): bit set in t = TRUE, in f = FALSE, in neither =
// UNKNOWN.  Kleene AND is (t1 & t2, f1 | f2), OR is (t1 | t2, f1 & f2), NOT
// swaps the words.  The postfix program is wave-uniform, so its dispatch is
// scalar; only the leaf tests touch per-row data.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "sel_device.h"

using namespace sel;

typedef int32_t v2i __attribute__((ext_vector_type(2)));
typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Pointers read from memory are generic to the compiler; casting them to
// the global (1) or constant (4) address space gives global_load / s_load
// instead of flat loads.
#define GLOBAL __attribute__((address_space(1)))
#define CONSTANT __attribute__((address_space(4)))
typedef const CONSTANT DevInstr* CInstr;

namespace {

template <class T>
__device__ __forceinline__ const GLOBAL T* gptr(const void* p) {
  return (const GLOBAL T*)p;
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// Constants of the program staged in the workgroup's LDS: a leaf whose
// lds_word lies in the staged words reads the copy there (of a bitmap,
// followed by a zero word) instead.
struct StageView {
  const uint32_t* lds;
  uint32_t words;
};

// An instruction in scalar registers, from one 64-byte scalar load: read field
// by field where each is needed, a leaf was a chain of eight scalar-cache
// round trips, and they, not the columns' loads, took most of a short scan.
struct Ins {
  uint32_t op, type, flags, n;
  const void* data;
  const uint32_t* valid;
  int64_t lo;
  uint64_t span;
  const void* aux;
  uint32_t lds_word;
};
typedef uint32_t v8u __attribute__((ext_vector_type(8)));
typedef uint32_t v16u __attribute__((ext_vector_type(16)));
__device__ __forceinline__ uint64_t pair64(v16u w, int k) { return ((uint64_t)w[k + 1] << 32) | w[k]; }
__device__ __forceinline__ Ins decode(v16u w) {
  return Ins{w[0], w[1], w[2], w[3], (const void*)pair64(w, 4), (const uint32_t*)pair64(w, 6), (int64_t)pair64(w, 8),
             pair64(w, 10), (const void*)pair64(w, 12), w[15]};
}
__device__ __forceinline__ Ins load_ins(CInstr p) { return decode(*(const CONSTANT v16u*)p); }

// ---------------------------------------------------------------- loads --
// A wave takes NS steps of 256 rows at a time: a whole 2048-row tile (NS =
// kSteps), or in a small table a quarter of one (kSmallSteps), so that four
// times as many waves share it.
//
// Raw storage of one lane's 4 NS rows of a column.  All loads of a column are
// issued before any is used, so each lane keeps its rows' loads in flight;
// a tile's are nontemporal (streamed once, not re-read).  int64 columns are
// loaded in groups of at most four steps (8 x 16 B per lane).
template <int TY, int NS> struct Raw;
template <int NS> struct Raw<T_I8, NS> { uint32_t w[NS]; };
template <int NS> struct Raw<T_I16, NS> { v2i w[NS]; };
template <int NS> struct Raw<T_I32, NS> { v4i w[NS]; };
constexpr int group64(int ns) { return ns < 4 ? ns : 4; }
template <int NS> struct Raw<T_I64, NS> { v4i w[2 * group64(NS)]; };

constexpr int kNt = 2;   // buffer-load cache policy: nontemporal (streamed once)

// A streamed load: nontemporal (NT, the default) or through the caches as
// usual; which one is faster is left to the tuner.
template <bool NT, class T>
__device__ __forceinline__ T ldg(const GLOBAL T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <int TY>
constexpr uint32_t type_width() { return TY == T_I8 ? 1u : TY == T_I16 ? 2u : TY == T_I32 ? 4u : 8u; }

constexpr uint32_t kOutOfBounds = 1u << 30;   // past any col_rsrc

// Buffer resource over rows [tb, min(tb + span, nrows)) of a column: 32-bit
// offsets from row tb, and a read past the table's last row returns zero
// without touching memory.  The bound is in whole dwords, since the hardware
// zeroes a dword that crosses it; the bytes up to the next 4-byte boundary
// may be read.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t col_rsrc(const void* data, uint32_t width, uint64_t tb,
                                                           uint64_t nrows, uint32_t span) {
  const uint32_t rows = nrows - tb < (uint64_t)span ? (uint32_t)(nrows - tb) : span;
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)data + tb * width), (short)0,
                                           (int)uni((rows * width + 3u) & ~3u), 0x00020000);
}

// Steps j0 .. of a column: every load of r, whole tiles by global loads, the
// small scan's quarters by bounded buffer loads (3 % slower in the mask scan
// of 300M rows, but right for a table's last rows too).
template <int TY, int NS, bool NT>
__device__ __forceinline__ void load_raw(Raw<TY, NS>& r, const void* data, uint64_t tb, uint64_t nrows,
                                         uint32_t lane, int j0) {
  using W = std::remove_reference_t<decltype(r.w[0])>;
  constexpr int N = sizeof(r.w) / sizeof(W);
  if constexpr (NS == kSteps) {
    const GLOBAL W* p = gptr<W>((const char*)data + tb * type_width<TY>());
#pragma unroll
    for (int k = 0; k < N; ++k)
      r.w[k] = TY == T_I64 ? ldg<NT>(p + 2 * lane + 128 * (j0 + (k >> 1)) + (k & 1)) : ldg<NT>(p + lane + 64 * (j0 + k));
  } else {
    const __amdgpu_buffer_rsrc_t rs = col_rsrc(data, type_width<TY>(), tb, nrows, 256u * NS);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const uint32_t off = TY == T_I64 ? 32u * lane + 2048u * (uint32_t)(j0 + (k >> 1)) + 16u * (uint32_t)(k & 1)
                                       : type_width<TY>() * (4u * lane + 256u * (uint32_t)(j0 + k));
      if constexpr (TY == T_I8) r.w[k] = (W)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0);
      else if constexpr (TY == T_I16) r.w[k] = (W)__builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
      else r.w[k] = (W)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    }
  }
}

// value of row bit b (= 4*j + i) from the raw registers; b is a constant
// after unrolling.  Narrow types are sign-extended to int32.
template <int TY, int NS>
__device__ __forceinline__ auto get(const Raw<TY, NS>& r, int b) {
  const int j = b >> 2, i = b & 3;
  if constexpr (TY == T_I8) {
    return (int32_t)(int8_t)(r.w[j] >> (8 * i));
  } else if constexpr (TY == T_I16) {
    return (int32_t)(int16_t)((uint32_t)r.w[j][i >> 1] >> (16 * (i & 1)));
  } else if constexpr (TY == T_I32) {
    return (int32_t)r.w[j][i];
  } else {  // b indexes the loaded group
    const v4i& q = r.w[2 * j + (i >> 1)];
    const int k = 2 * (i & 1);
    return (int64_t)(((uint64_t)(uint32_t)q[k + 1] << 32) | (uint32_t)q[k]);
  }
}

__device__ __forceinline__ uint64_t row_of(uint64_t tb, uint32_t lane, int b) {
  return tb + 256u * (uint32_t)(b >> 2) + 4u * lane + (uint32_t)(b & 3);
}

// Predicate bits of one lane's rows: bit b = pred(value of row b).  The word
// is built highest row first as P = 2P + bit, one add-with-carry per row
// after the compare.  Rows past the table (small scans) test a zero; the
// caller drops them.
template <int TY, int NS, bool NT, class Pred>
__device__ __forceinline__ uint32_t pred_bits(const void* data, uint64_t tb, uint64_t nrows, uint32_t lane, Pred pred) {
  uint32_t P = 0;
  if constexpr (TY == T_I64) {
    constexpr int G = group64(NS);
#pragma unroll
    for (int h = NS / G - 1; h >= 0; --h) {
      Raw<TY, NS> r;
      load_raw<TY, NS, NT>(r, data, tb, nrows, lane, G * h);
#pragma unroll
      for (int b = 4 * G - 1; b >= 0; --b) P = (P << 1) + (uint32_t)pred(get<TY, NS>(r, b), 4 * G * h + b);
    }
  } else {
    Raw<TY, NS> r;
    load_raw<TY, NS, NT>(r, data, tb, nrows, lane, 0);
#pragma unroll
    for (int b = 4 * NS - 1; b >= 0; --b) P = (P << 1) + (uint32_t)pred(get<TY, NS>(r, b), b);
  }
  return P;
}

// Validity bits of the lane's rows (all ones for a column without NULLs).
template <bool FULL, int NS = kSteps>
__device__ __forceinline__ uint32_t valid_bits(const uint32_t* valid, uint64_t tb, uint32_t lane,
                                               uint64_t nrows) {
  if (valid == nullptr) return ~0u;
  const GLOBAL uint32_t* vw = gptr<uint32_t>(valid) + tb / 32 + (lane >> 3);
  const uint32_t sh = 4 * (lane & 7);
  uint32_t V = 0;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    if (FULL || tb + 256u * j + 4u * lane < nrows)
      V |= ((vw[8 * j] >> sh) & 0xFu) << (4 * j);
  }
  return V;
}

// The lane's rows that the table holds.
template <int NS>
__device__ __forceinline__ uint32_t inrange_bits(uint64_t tb, uint32_t lane, uint64_t nrows) {
  const int rows = nrows - tb < 256ull * NS ? (int)(nrows - tb) : 256 * NS;
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < NS; ++j)
    m |= ((1u << min(max(rows - (int)(256u * (uint32_t)j + 4u * lane), 0), 4)) - 1u) << (4 * j);
  return m;
}

// Values of rows 8q .. 8q + 7 of the lane (steps 2q, 2q + 1), as int64:
// wide loads on a whole tile as for a range test; where the table may end the
// same loads through a bounded buffer resource.
template <int TY, bool FULL, bool NT>
__device__ __forceinline__ void load8(const void* data, uint64_t tb, uint32_t lane, uint64_t nrows, int q,
                                      int64_t (&x)[8]) {
  constexpr uint32_t width = type_width<TY>();
  const char* base = (const char*)data + tb * width;
  const __amdgpu_buffer_rsrc_t rs = col_rsrc(data, width, tb, nrows, (uint32_t)kTileRows);
#pragma unroll
  for (int js = 0; js < 2; ++js) {
    const uint32_t at = width * (256u * (uint32_t)(2 * q + js) + 4u * lane);   // byte offset of the lane's four rows
    if constexpr (TY == T_I8) {
      uint32_t w;
      if constexpr (FULL) w = ldg<NT>((const GLOBAL uint32_t*)(gptr<char>(base) + at));
      else w = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)at, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * js + i] = (int64_t)(int8_t)(w >> (8 * i));
    } else if constexpr (TY == T_I16) {
      v2i w;
      if constexpr (FULL) w = ldg<NT>((const GLOBAL v2i*)(gptr<char>(base) + at));
      else w = (v2i)__builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * js + i] = (int64_t)(int16_t)((uint32_t)w[i >> 1] >> (16 * (i & 1)));
    } else if constexpr (TY == T_I32) {
      v4i w;
      if constexpr (FULL) w = ldg<NT>((const GLOBAL v4i*)(gptr<char>(base) + at));
      else w = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)at, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * js + i] = (int64_t)w[i];
    } else {
      v4i w[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if constexpr (FULL) w[h] = ldg<NT>((const GLOBAL v4i*)(gptr<char>(base) + at) + h);
        else w[h] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + 16u * (uint32_t)h), 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const v4i& v = w[i >> 1];
        x[4 * js + i] = (int64_t)(((uint64_t)(uint32_t)v[2 * (i & 1) + 1] << 32) | (uint32_t)v[2 * (i & 1)]);
      }
    }
  }
}

// Bitmap, hashed-list or sorted-list test of eight values, appended to P: the
// constants at `words`, which are 64-bit `values` to the lists, in LDS or in
// device memory.
template <bool HASHED, class Words, class Values>
__device__ __forceinline__ uint32_t const_bits8(uint32_t P, const Ins& I, const int64_t (&x)[8], Words words, Values values) {
  if (I.op == D_BITMAP) {
#pragma unroll
    for (int k = 7; k >= 0; --k) {
      const uint64_t d = (uint64_t)x[k] - (uint64_t)I.lo;
      const uint32_t at = d < I.span ? (uint32_t)d : 0u;   // nbits <= 2^32
      P = (P << 1) + ((uint32_t)(d < I.span) & ((words[at >> 5] >> (at & 31)) & 1u));
    }
  } else if (HASHED && (I.flags & F_HASHED)) {
    const uint32_t f = I.flags, b = in_hash_bits(f);
    const uint32_t c1 = kInHashMul[in_hash_pair(f)][0], c2 = kInHashMul[in_hash_pair(f)][1];
#pragma unroll
    for (int k = 7; k >= 0; --k) {
      const int64_t h1 = values[in_hash(x[k], c1, b)], h2 = values[(1u << b) + in_hash(x[k], c2, b)];
      P = (P << 1) + ((uint32_t)(h1 == x[k]) | (uint32_t)(h2 == x[k]));
    }
  } else {  // D_INLIST: lower bound in the sorted list
    uint32_t base[8] = {};
    for (uint32_t len = I.n; len > 1;) {
      const uint32_t half = len >> 1;
#pragma unroll
      for (int k = 0; k < 8; ++k) base[k] = values[base[k] + half] <= x[k] ? base[k] + half : base[k];
      len -= half;
    }
#pragma unroll
    for (int k = 7; k >= 0; --k) P = (P << 1) + (uint32_t)(values[base[k]] == x[k]);
  }
  return P;
}

// One leaf on the partial last tile of its table, eight rows of a lane at a
// time (rows past the table test a zero and are not counted).  The values are
// widened to int64, so that one short body serves every type and test: the
// wide bodies of whole tiles are not doubled, and keep their registers.
// Four loads in turn per leaf; element loads, one row of a lane after
// another, were 32 (six leaves over 10 007 rows: 37 us, with these 19, and
// 9 with the quarter tiles of small tables).
// Staged constants are read from LDS here too: a sorted list's searches are
// 4 log2(n) dependent reads, which in device memory made this one tile outlast
// the rest of the scan (60M int64 rows against 1500 values: 214 us).
// SCAN: a scan's leaf, whose flags are DevFlags and whose constants may be
// staged (a batch's copies of the leaves reuse these words, and read an IN
// list through its sorted values in device memory).
template <bool SCAN>
__device__ __forceinline__ uint32_t partial_leaf(const Ins& I, uint32_t ty, uint64_t tb, uint32_t lane, uint64_t nrows,
                                                 const StageView& sv) {
  const void* data = I.data;
  uint32_t P = 0;
#pragma unroll 1
  for (int q = 3; q >= 0; --q) {
    int64_t x[8];
    switch (ty) {
      case T_I8: load8<T_I8, false, true>(data, tb, lane, nrows, q, x); break;
      case T_I16: load8<T_I16, false, true>(data, tb, lane, nrows, q, x); break;
      case T_I32: load8<T_I32, false, true>(data, tb, lane, nrows, q, x); break;
      default: load8<T_I64, false, true>(data, tb, lane, nrows, q, x); break;
    }
    // the ranges' code stays beside the loads': where each wave takes one tile,
    // this one's instruction fetches end the scan
    if (__builtin_expect(I.op == D_RANGE, 1)) {
#pragma unroll
      for (int k = 7; k >= 0; --k) P = (P << 1) + (uint32_t)((uint64_t)x[k] - (uint64_t)I.lo <= I.span);
    } else if (SCAN && I.lds_word < sv.words) {
      const uint32_t* copy = sv.lds + I.lds_word;
      P = const_bits8<SCAN>(P, I, x, copy, (const int64_t*)copy);
    } else {
      const bool tables = SCAN && I.op == D_INLIST && (I.flags & F_HASHED);   // they follow the list
      P = const_bits8<SCAN>(P, I, x, gptr<uint32_t>(I.aux), gptr<int64_t>(I.aux) + (tables ? I.n : 0u));
    }
  }
  return P;
}

// IN-list test of a lane's rows against a sorted list of n values (in
// LDS or device memory): wide loads of the column as for a range test, then
// a branch-free lower bound that moves the eight rows of two steps one
// search step at a time, so that their list reads are in flight together.
template <int TY, int NS, bool NT, class List>
__device__ __forceinline__ uint32_t inlist_bits(const void* data, uint64_t tb, uint64_t nrows, uint32_t lane,
                                                List list, uint32_t n, uint32_t need) {
  // the next instruction's load must not be in flight across the searches: the
  // scalar and LDS loads share a counter, and each group of list reads would
  // be waited for whole (60M rows against 5000 values: 172 us, without 165)
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  uint32_t P = 0;
#pragma unroll 1
  for (int q = NS / 2 - 1; q >= 0; --q) {   // bits 8q .. 8q + 7: steps 2q, 2q + 1
    int64_t x[8];
    load8<TY, NS == kSteps, NT>(data, tb, lane, nrows, q, x);
    uint32_t base[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) base[k] = 0;
    for (uint32_t len = n; len > 1;) {
      const uint32_t half = len >> 1;
#pragma unroll
      for (int k = 0; k < 8; ++k) base[k] = list[base[k] + half] <= x[k] ? base[k] + half : base[k];
      len -= half;
    }
#pragma unroll
    for (int k = 7; k >= 0; --k)
      P = (P << 1) + (uint32_t)(((need >> (8 * q + k)) & 1u) && list[base[k]] == x[k]);
  }
  return P;
}

// The same test through the list's two cuckoo tables of 2^b slots each (T
// then T + 2^b, in LDS or device memory): a value is in the list if and
// only if it sits in its slot of either table, so two reads per row answer
// it (empty slots hold a list value, which can only match a member).
template <int TY, int NS, bool NT, class Tab>
__device__ __forceinline__ uint32_t inhash_bits(const void* data, uint64_t tb, uint64_t nrows, uint32_t lane, Tab T,
                                                uint32_t b, uint32_t c1, uint32_t c2, uint32_t need) {
  const uint32_t m = 1u << b;
  uint32_t P = 0;
#pragma unroll 1
  for (int q = NS / 2 - 1; q >= 0; --q) {
    int64_t x[8];
    load8<TY, NS == kSteps, NT>(data, tb, lane, nrows, q, x);
#pragma unroll
    for (int k = 7; k >= 0; --k) {
      const bool hit = T[in_hash(x[k], c1, b)] == x[k] || T[m + in_hash(x[k], c2, b)] == x[k];
      P = (P << 1) + (uint32_t)(((need >> (8 * q + k)) & 1u) && hit);
    }
  }
  return P;
}

// ---------------------------------------------------------------- leaves --
// A scan's leaf on a whole tile, or on a small scan's quarter of one.
template <int TY, int NS, bool NT>
__device__ __forceinline__ uint32_t leaf_pred(const Ins& I, uint64_t tb, uint64_t nrows, uint32_t lane, uint32_t need,
                                              const StageView& sv) {
  const uint32_t op = I.op;
  const void* data = I.data;
  const int64_t lo = I.lo;
  const uint64_t span = I.span;
  const bool staged = I.lds_word < sv.words;
  const uint32_t* copy = sv.lds + I.lds_word;
  if (op == D_INLIST) {
    const uint32_t f = I.flags;
    if (f & F_HASHED) {
      // the cuckoo tables after the sorted list: their LDS copy if staged
      const uint32_t b = in_hash_bits(f), c1 = kInHashMul[in_hash_pair(f)][0], c2 = kInHashMul[in_hash_pair(f)][1];
      if (staged) return inhash_bits<TY, NS, NT>(data, tb, nrows, lane, (const int64_t*)copy, b, c1, c2, need);
      return inhash_bits<TY, NS, NT>(data, tb, nrows, lane, gptr<int64_t>((const int64_t*)I.aux + I.n), b, c1, c2, need);
    }
    if (staged) return inlist_bits<TY, NS, NT>(data, tb, nrows, lane, (const int64_t*)copy, I.n, need);
    return inlist_bits<TY, NS, NT>(data, tb, nrows, lane, gptr<int64_t>(I.aux), I.n, need);
  }
  if (op == D_BITMAP && staged) {
    // an offset outside the window, or a row the guard skips, reads the
    // zero bit z after the copy; for narrow columns the window lies inside
    // int32 (the host stages only such bitmaps)
    const uint32_t z = (uint32_t)((span + 31u) & ~31ull);
    if constexpr (TY == T_I64) {
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int64_t x, int b) -> uint32_t {
        const uint64_t d = (uint64_t)x - (uint64_t)lo;
        const uint32_t k = ((need >> b) & 1u) && d < z ? (uint32_t)d : z;
        return (copy[k >> 5] >> (k & 31)) & 1u;
      });
    } else {
      const uint32_t lo32 = (uint32_t)lo;
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int32_t x, int b) -> uint32_t {
        const uint32_t d = (uint32_t)x - lo32;
        const uint32_t k = ((need >> b) & 1u) && d < z ? d : z;
        return (copy[k >> 5] >> (k & 31)) & 1u;
      });
    }
  }
  if (op == D_RANGE) {
    if constexpr (TY == T_I64) {
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int64_t x, int) {
        return (uint64_t)x - (uint64_t)lo <= span;
      });
    } else {
      const uint32_t lo32 = (uint32_t)lo, span32 = (uint32_t)span;
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int32_t x, int) {
        return (uint32_t)x - lo32 <= span32;
      });
    }
  } else if (op == D_BITMAP) {
    // rows that need no test (guard) or fall outside [lo, lo + nbits) read
    // word 0 and are masked: no branch, so all 32 lookups issue together
    const GLOBAL uint32_t* bits = gptr<uint32_t>(I.aux);
    if constexpr (TY == T_I64) {
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int64_t x, int b) -> uint32_t {
        const uint64_t d = (uint64_t)x - (uint64_t)lo;
        const bool ok = d < span && ((need >> b) & 1u);
        const uint32_t k = ok ? (uint32_t)d : 0u;  // nbits <= 2^32
        return ok & ((bits[k >> 5] >> (k & 31)) & 1u);
      });
    } else {
      // x - lo in 64 bits: a negative key must not alias a bit when nbits
      // exceeds 2^31
      return pred_bits<TY, NS, NT>(data, tb, nrows, lane, [=](int32_t x, int b) -> uint32_t {
        const uint64_t d = (uint64_t)((int64_t)x - lo);
        const bool ok = d < span && ((need >> b) & 1u);
        const uint32_t k = ok ? (uint32_t)d : 0u;
        return ok & ((bits[k >> 5] >> (k & 31)) & 1u);
      });
    }
  } else {  // D_INLIST, handled above
    return 0u;
  }
}

template <int NS, bool PARTIAL, bool NT>
__device__ __forceinline__ void eval_leaf(const Ins& I, uint64_t tb, uint32_t lane,
                                          uint64_t nrows, uint32_t tos_t, uint32_t tos_f,
                                          uint32_t& t, uint32_t& f, const StageView& sv) {
  const uint32_t op = I.op;
  const uint32_t V = valid_bits<NS == kSteps && !PARTIAL, NS>(I.valid, tb, lane, nrows);
  if (op >= D_NN_TRUE) {
    switch (op) {
      case D_NN_TRUE: t = V; f = 0; return;
      case D_NN_FALSE: t = 0; f = V; return;
      case D_ISNULL: t = ~V; f = V; return;
      default: t = V; f = ~V; return;  // D_NOTNULL
    }
  }
  const uint32_t flags = I.flags;
  uint32_t need = ~0u;
  if (flags & F_GUARD_AND) need = ~tos_f;
  else if (flags & F_GUARD_OR) need = ~tos_t;
  uint32_t P;
  if constexpr (PARTIAL) {
    P = partial_leaf<true>(I, I.type, tb, lane, nrows, sv);
  } else {
    switch (I.type) {
      case T_I8: P = leaf_pred<T_I8, NS, NT>(I, tb, nrows, lane, need, sv); break;
      case T_I16: P = leaf_pred<T_I16, NS, NT>(I, tb, nrows, lane, need, sv); break;
      case T_I32: P = leaf_pred<T_I32, NS, NT>(I, tb, nrows, lane, need, sv); break;
      default: P = leaf_pred<T_I64, NS, NT>(I, tb, nrows, lane, need, sv); break;
    }
  }
  t = P & V;
  f = ~P & V;
}

// ---------------------------------------------------------- interpreter --
// The stack below its two top values is held in registers; its index is
// uniform, so the unrolled selects below compile to scalar branches and no
// private memory is used.  Few programs get there: the top two have
// registers of their own.
constexpr int kDeep = kMaxDepth - 2;
__device__ __forceinline__ void spill(uint32_t (&st)[kDeep], uint32_t (&sf)[kDeep],
                                      int idx, uint32_t t, uint32_t f) {
#pragma unroll
  for (int k = 0; k < kDeep; ++k)
    if (k == idx) { st[k] = t; sf[k] = f; }
}
__device__ __forceinline__ void fill(const uint32_t (&st)[kDeep], const uint32_t (&sf)[kDeep],
                                     int idx, uint32_t& t, uint32_t& f) {
  t = 0; f = 0;
#pragma unroll
  for (int k = 0; k < kDeep; ++k)
    if (k == idx) { t = st[k]; f = sf[k]; }
}

// TRUE bits of the lane's rows of the NS steps from row tb (bits past them,
// and of rows past the table, are to be dropped by the caller unless the tile
// is whole).  The host has folded a NOT, AND or OR that follows a leaf into
// the leaf (scan_code), so that most programs run an instruction per leaf.
template <int NS, bool PARTIAL, bool NT>
__device__ __forceinline__ uint32_t eval_tile(CInstr prog, uint32_t nins, uint64_t tb,
                                              uint32_t lane, uint64_t nrows, const StageView& sv) {
  uint32_t st[kDeep], sf[kDeep];
  uint32_t tt = 0, tf = 0, ut = 0, uf = 0;
  int d = 0;  // values on the stack; the top is (tt, tf), below it (ut, uf)
  // the next instruction is asked for before the current one runs
  v16u next = *(const CONSTANT v16u*)prog;
  for (uint32_t pc = 0; pc < nins; ++pc) {
    v16u cur = next;
    asm volatile("" : "+s"(cur));
    next = *(const CONSTANT v16u*)(prog + min(pc + 1u, nins - 1u));
    const Ins I = decode(cur);
    const uint32_t op = I.op;
    if (op < D_AND || op >= D_TRUE) {
      uint32_t t, f;
      if (op == D_TRUE) { t = ~0u; f = 0; }
      else if (op == D_FALSE) { t = 0; f = ~0u; }
      else eval_leaf<NS, PARTIAL, NT>(I, tb, lane, nrows, tt, tf, t, f, sv);
      if (I.flags & F_THEN_NOT) { const uint32_t x = t; t = f; f = x; }
      if (I.flags & F_THEN_AND) {
        tt &= t;
        tf |= f;
      } else if (I.flags & F_THEN_OR) {
        tt |= t;
        tf &= f;
      } else {
        if (d >= 2) spill(st, sf, d - 2, ut, uf);
        ut = tt; uf = tf;
        tt = t; tf = f;
        ++d;
      }
    } else if (op == D_NOT) {
      const uint32_t x = tt; tt = tf; tf = x;
    } else if (op == D_ISUNK) {
      const uint32_t k = tt | tf; tt = ~k; tf = k;
    } else {
      if (op == D_AND) { tt &= ut; tf |= uf; }
      else { tt |= ut; tf &= uf; }
      --d;
      if (d >= 2) fill(st, sf, d - 2, ut, uf);
    }
  }
  return tt;
}

// ------------------------------------------------------------ reductions --
// Wait until this thread's earlier memory operations, atomics included,
// have completed.  The end-of-launch ticket hand-offs below need no more:
// what one workgroup passes to the last one travels only through
// device-scope atomics, which are coherent by themselves, so the cache
// write-back and invalidation of a device-scope fence (issued by every
// workgroup, tens of microseconds at the end of a short scan) are not
// needed.  Plain stores (results, masks) are read after the launch.
__device__ __forceinline__ void atomics_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sum over the 64 lanes: DPP within quads and 16-lane rows, then the four
// row sums by readlane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // quad_perm 1,0,3,2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // quad_perm 2,3,0,1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);  // row_ror:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);  // row_ror:8
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
         (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}

// A result word in pinned host memory: a system-scope store, so that a host
// thread polling the word sees it without waiting for the launch to retire.
__device__ __forceinline__ void put_host(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Block sum and one device atomic per workgroup, which adds its count and
// takes its ticket at once (kSlotTicket): the workgroup that sees all other
// tickets also holds the total, publishes it and resets the slot for the next
// launch.  Separate atomics (add, wait, ticket, read back) were four memory
// latencies at the end of every launch instead of one.  Atomics on one word
// take 9 ns each in turn, so that a grid of 768 workgroups that end together
// waited 7 us: the workgroups share kSlotParts words, and the last of each
// part adds its sum to the slot's.  The second count (rare: out-of-range keys
// and ids) is added before the ticket.
__device__ void finish(DevSlot* slot, unsigned long long* out, unsigned long long* host, uint32_t c0, uint32_t c1,
                       bool two) {
  __shared__ unsigned long long red0[16], red1[16];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t s0 = wave_sum(c0);
  const uint32_t s1 = two ? wave_sum(c1) : 0u;
  if (lane == 0) { red0[wave] = s0; red1[wave] = s1; }
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long b0 = 0, b1 = 0;
  for (uint32_t w = 0; w < (blockDim.x >> 6); ++w) { b0 += red0[w]; b1 += red1[w]; }
  if (b1) {
    atomicAdd(&slot->acc2, b1);
    atomics_done();
  }
  const uint32_t parts = min(gridDim.x, kSlotParts), part = blockIdx.x % kSlotParts;
  unsigned long long* p = &slot->part[part * kSlotStride];
  const unsigned long long here = atomicAdd(p, kSlotTicket + b0);
  if (here / kSlotTicket != (gridDim.x - 1u - part) / kSlotParts) return;
  atomicExch(p, 0ull);
  const unsigned long long sum = here % kSlotTicket + b0;
  const unsigned long long old = atomicAdd(&slot->acc, kSlotTicket + sum);
  if (old / kSlotTicket != parts - 1u) return;
  const unsigned long long total = old % kSlotTicket + sum;
  const unsigned long long second = two ? atomicExch(&slot->acc2, 0ull) : 0ull;
  if (out) {
    out[0] = total;
    if (two) out[1] = second;
  }
  if (host) {
    if (two) put_host(host + 1, second);
    put_host(host, total);
  }
  atomicExch(&slot->acc, 0ull);
}

// Key-bitmap push-down of one wave's rows, with one atomic for a lane's
// neighbouring keys in one word.  Where every lane has few TRUE rows it loads
// their keys alone, four at a time; else the keys of all steps in a few wide
// loads, those without a TRUE row of the lane sent out of bounds.  100M rows,
// int64 keys in order: a row at a time, each waited for by itself, took 105 us
// for 0.5 % of them and 1210 us for half; every key by wide loads and every bit
// tested 227 and 624 us; now 96 and 618.  The line lies at a quarter of a
// lane's rows: at an eighth 5 % of the rows take 211 us against 176, at a half
// 13 % take 294 against 290.
constexpr uint32_t kKeysAtOnce = 4;
template <int TY, int NS>
__device__ __forceinline__ uint32_t put_keys(const ScanArgs& a, uint32_t T, uint64_t tb, uint32_t lane) {
  const __amdgpu_buffer_rsrc_t rs = col_rsrc(a.key_data, type_width<TY>(), tb, a.nrows, 256u * NS);
  uint32_t oor = 0, word = 0, bits = 0;
  auto put = [&](int64_t key) {
    const uint64_t d = (uint64_t)key - (uint64_t)a.key_min;
    if (d >= a.nbits) {
      ++oor;
      return;
    }
    const uint32_t at = (uint32_t)(d >> 5);
    if (at != word && bits) {
      atomicOr(&a.bitmap[word], bits);
      bits = 0;
    }
    word = at;
    bits |= 1u << (d & 31);
  };
  if (__ballot(__builtin_popcount(T) > NS) == 0ull) {
    for (uint32_t m = T; __ballot(m != 0u);) {
      int64_t key[kKeysAtOnce];
      bool row[kKeysAtOnce];
#pragma unroll
      for (uint32_t u = 0; u < kKeysAtOnce; ++u) {
        row[u] = m != 0u;
        const uint32_t b = (uint32_t)__builtin_ctz(m | 0x80000000u);
        const uint32_t at = row[u] ? type_width<TY>() * (256u * (b >> 2) + 4u * lane + (b & 3u)) : kOutOfBounds;
        if constexpr (TY == T_I64) {
          const v2u w = (v2u)__builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, 0, 0);
          key[u] = (int64_t)(((uint64_t)w[1] << 32) | w[0]);
        } else {
          key[u] = (int64_t)(int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)at, 0, 0);
        }
        m &= m - 1u;
      }
#pragma unroll
      for (uint32_t u = 0; u < kKeysAtOnce; ++u)
        if (row[u]) put(key[u]);
    }
  } else {
    constexpr int G = TY == T_I64 ? group64(NS) : NS;
#pragma unroll
    for (int g = 0; g < NS / G; ++g) {
      v4i w[TY == T_I64 ? 2 * G : G];
#pragma unroll
      for (int k = 0; k < (int)(sizeof w / sizeof w[0]); ++k) {
        const uint32_t rows = TY == T_I64 ? T >> (4 * G * g + 2 * k) & 3u : T >> (4 * (G * g + k)) & 0xFu;
        const uint32_t at = TY == T_I64 ? 32u * lane + 2048u * (uint32_t)(G * g + (k >> 1)) + 16u * (uint32_t)(k & 1)
                                        : 16u * lane + 1024u * (uint32_t)(G * g + k);
        w[k] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)(rows ? at : kOutOfBounds), 0, 0);
      }
#pragma unroll
      for (int b = 0; b < 4 * G; ++b) {
        if (!((T >> (4 * G * g + b)) & 1u)) continue;
        const int j = b >> 2, i = b & 3;
        if constexpr (TY == T_I64) {
          const v4i& q = w[2 * j + (i >> 1)];
          put((int64_t)(((uint64_t)(uint32_t)q[2 * (i & 1) + 1] << 32) | (uint32_t)q[2 * (i & 1)]));
        } else {
          put((int64_t)w[j][i]);
        }
      }
    }
  }
  if (bits) atomicOr(&a.bitmap[word], bits);
  return oor;
}

// NS = kSteps: tiles, by as many waves as fill the chip.  NS = kSmallSteps:
// quarters of tiles, for tables where that many waves would have a tile or
// two each: latency bounds those (six leaves in turn took 13 us a tile), so
// more and shorter waves share the table (a 1M-row push-down's scan: 14.5 us,
// now 7.6).
template <int MODE, bool NT, int NS>
__global__ void __launch_bounds__(256) k_scan(const DevInstr* __restrict__ prog_, ScanArgs a) {
  constexpr bool SMALL = NS != kSteps;
  constexpr uint32_t kRows = 256u * NS, kWords = 8u * NS;   // of a tile, or a quarter
  CInstr prog = (CInstr)prog_;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t nw = blockDim.x >> 6;
  const uint64_t W = (uint64_t)gridDim.x * nw;
  const uint64_t wid = uni64((uint64_t)blockIdx.x * nw + (threadIdx.x >> 6));
  extern __shared__ __align__(16) uint32_t sbm[];
  const StageView sv{sbm, a.stage_words};
  if (a.nstage) {
    // the program's small bitmaps, each followed by a zero word
    for (uint32_t k = 0; k < a.nstage; ++k) {
      const CONSTANT BatchBitmap* B = (const CONSTANT BatchBitmap*)a.stage + k;
      const uint32_t n = B->words, last = B->last_mask;
      const GLOBAL uint32_t* src = gptr<uint32_t>(B->src);
      uint32_t* dst = sbm + B->lds_word;
      for (uint32_t i = threadIdx.x; i <= n; i += blockDim.x) {
        uint32_t w = 0;
        if (i < n) w = i + 1 == n ? src[i] & last : src[i];
        dst[i] = w;
      }
    }
    __syncthreads();
  }
  uint32_t cnt = 0, oor = 0;
  // M_MASK: the nonzero words of the wave's tiles go to one packed stream
  // per group of kMaskGroup turns, its pending words in `hold` (word l of the
  // current block of 64 in lane l, `cur` of them), each turn's word map,
  // count and offset in the lane of that number; blocks and groups are stored
  // whole.  Each tile's words, count and map stored at its own place
  // were three partly written cache lines a tile: the six-leaf mask scan over
  // 300M rows took 1033 us, now 1009 (963 with no store at all).
  uint32_t hold = 0, cur = 0, blocks = 0, turn = 0, meta = 0;
  uint64_t words = 0, place = 0;
  if constexpr (MODE == M_MASK) place = wave_place(a.order, (uint32_t)uni((uint32_t)(blockIdx.x * nw + (threadIdx.x >> 6))));
  auto put_group = [&](uint32_t turns) {
    if (lane < cur) a.mask[place * kWords + (uint64_t)blocks * kWave + lane] = hold;
    if (lane < turns) {
      a.tile_words[place + lane] = words;
      a.tile_meta[place + lane] = meta;
    }
    place += turns;
    cur = blocks = 0;
  };
  // Each wave takes runs of tps consecutive whole tiles, W runs apart.  A
  // partial last tile goes to the last wave, which has the fewest, before its
  // others: at the end of the scan every other wave would wait for it.  (A
  // quarter's loads are bounded: the last one is like the others.)
  const uint64_t tps = a.tiles_per_step ? a.tiles_per_step : 1;
  const uint64_t nfull = SMALL ? a.ntiles : a.nrows / kTileRows;
  uint64_t run = wid * tps;
  uint32_t k = 0;
  bool partial = !SMALL && wid == W - 1 && nfull < a.ntiles;
  for (;;) {
    uint64_t tile = nfull;
    if (!partial) {
      if (k == tps) {
        run += W * tps;
        k = 0;
      }
      tile = run + k++;
      if (tile >= nfull) break;
    }
    const uint64_t tb = tile * kRows;
    uint32_t T;
    if constexpr (SMALL) {
      T = eval_tile<NS, false, NT>(prog, a.nins, tb, lane, a.nrows, sv) & inrange_bits<NS>(tb, lane, a.nrows);
    } else if (!partial) {
      T = eval_tile<NS, false, NT>(prog, a.nins, tb, lane, a.nrows, sv);
    } else {
      T = eval_tile<NS, true, NT>(prog, a.nins, tb, lane, a.nrows, sv) & inrange_bits<NS>(tb, lane, a.nrows);
      partial = false;
    }
    cnt += __builtin_popcount(T);
    if constexpr (MODE == M_MASK) {
      // from the lanes' words to words of 32 rows in table order: word r
      // holds step r / 8 of lanes 8 (r % 8) .. + 7
      uint32_t R = 0;
      if (__ballot(T != 0u)) {
#pragma unroll
        for (uint32_t l = 0; l < 8; ++l) {
          const uint32_t w = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * (8u * (lane & 7u) + l)), (int)T);
          R |= ((w >> (4u * (lane >> 3))) & 0xFu) << (4 * l);
        }
      }
      // a lane with a nonzero word sends it to the next free place of the
      // block, the others to the places after those
      const uint64_t nz = __ballot(R != 0u);
      const uint32_t n = (uint32_t)__popcll(nz);
      const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(nz >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)nz, 0u));
      const uint32_t to = (cur + (R != 0u ? pos : n + lane - pos)) & 63u;
      const uint32_t v = (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)R);
      const uint32_t at = blocks * kWave + cur;
      hold = lane < cur ? hold : v;
      if (cur + n >= kWave) {
        a.mask[place * kWords + (uint64_t)blocks * kWave + lane] = hold;
        ++blocks;
        hold = v;
      }
      cur = (cur + n) & 63u;
      const uint32_t tc = wave_sum(__builtin_popcount(T));
      if (lane == turn) {
        words = nz;
        meta = tc | (at << kMetaShift);
      }
      if (++turn == kMaskGroup) {
        put_group(turn);
        turn = 0;
      }
    } else if constexpr (MODE == M_KEYBITMAP) {
      if (__ballot(T != 0u))
        oor += a.key_type == T_I64 ? put_keys<T_I64, NS>(a, T, tb, lane) : put_keys<T_I32, NS>(a, T, tb, lane);
    }
  }
  if constexpr (MODE == M_MASK) {
    if (turn) put_group(turn);
  }
  finish(a.slot, a.out, a.host, cnt, oor, MODE == M_KEYBITMAP);
}

// Exclusive scan of the tile counts: one workgroup of 1024 threads per chunk
// of 1024 tiles writes each tile's offset within its chunk and the chunk's
// total (at most 2048 chunks for 2^32 rows), which the compaction's waves add
// up themselves.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, uint32_t lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= (uint32_t)off) x += y;
  }
  return x;
}

// exclusive prefix of v over the (up to 1024) threads of the block
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v) {
  __shared__ uint32_t wsum[16];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v, lane);
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  if (wave == 0) {
    const uint32_t nw = blockDim.x >> 6;
    const uint32_t w = lane < nw ? wsum[lane] : 0u;
    const uint32_t wi = wave_incl_scan(w, lane);
    if (lane < nw) wsum[lane] = wi - w;
  }
  __syncthreads();
  return wsum[wave] + inc - v;
}

__global__ void __launch_bounds__(1024) k_chunk_scan(MaskOrder order, const uint32_t* __restrict__ meta,
                                                     uint32_t* __restrict__ offsets,
                                                     uint32_t* __restrict__ chunk_sums, uint32_t n) {
  const uint32_t i = blockIdx.x * 1024u + threadIdx.x;
  uint32_t turn, v = 0;
  if (i < n) v = meta[tile_place(order, i, turn)] & kMetaCount;
  const uint32_t ex = block_excl_scan(v);
  if (i < n) offsets[i] = ex;
  if (threadIdx.x == 1023) chunk_sums[blockIdx.x] = ex + v;
}

// Inclusive sum over the 64 lanes: DPP shifts within each 16-lane row, then
// the row totals by readlane.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x, uint32_t lane, uint32_t& total) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);  // row_shr:8
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)x, 47);
  const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  total = r0 + r1 + r2 + r3;
  const uint32_t row = lane >> 4;
  return x + (row == 0 ? 0u : row == 1 ? r0 : row == 2 ? r0 + r1 : r0 + r1 + r2);
}

// Row ids of TRUE rows in ascending order.  The packed words are in table
// order, so a word's first id comes after the ids of the words before it: one
// prefix sum of their popcounts.  Each wave takes one tile, or four of a
// larger table, and adds up the counts before its first (of the tiles when
// there are few, else of the chunks).

// The set bits of each lane's word, lane by lane: ids are first + bit, the
// lane's from out[pos].
__device__ __forceinline__ void put_bits(uint32_t w, uint32_t pos, uint32_t first, uint32_t* __restrict__ out) {
  while (__ballot(w != 0u)) {
    if (w != 0u) {
      out[pos++] = first + (uint32_t)__builtin_ctz(w);
      w &= w - 1u;
    }
  }
}

// The same for the words of lanes 0 .. n - 1 (the other lanes' are zero), two
// words at once, so that every store fills consecutive ids: from out[base].
__device__ __forceinline__ void put_words(uint32_t w, uint32_t first, uint32_t n, uint32_t base, uint32_t lane,
                                          uint32_t* __restrict__ out) {
  for (uint32_t k = 0; k < n; k += 2) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)w, (int)k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)w, (int)k + 1);
    const uint32_t f0 = (uint32_t)__builtin_amdgcn_readlane((int)first, (int)k);
    const uint32_t f1 = (uint32_t)__builtin_amdgcn_readlane((int)first, (int)k + 1);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    if (((lane & 32u ? hi : lo) >> (lane & 31u)) & 1u) out[base + rank] = (lane & 32u ? f1 : f0) + (lane & 31u);
    base += (uint32_t)(__builtin_popcount(lo) + __builtin_popcount(hi));
  }
}

// One tile: word r of 32 rows in lane r.  With many TRUE rows the wave goes
// through them 64 rows at a time, two words at once, so that every store
// fills consecutive ids; with few, each lane walks its own word.  (Every lane
// storing its own rows took 32 stores of scattered ids a tile, 51 us for the
// 30M ids of half of 60M rows; now 31.)
__device__ __forceinline__ void compact_tile(uint32_t w, uint32_t base, uint32_t tile, uint32_t lane,
                                             uint32_t* __restrict__ out) {
  const uint32_t tb = tile * (uint32_t)kTileRows;
  const uint32_t c = __builtin_popcount(w);
  uint32_t run;
  const uint32_t pos = wave_incl_sum(c, lane, run) - c;
  if (run <= 192u) {
    put_bits(w, base + pos, tb + 32u * lane, out);
    return;
  }
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * k + 1);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    if (((lane & 32u ? hi : lo) >> (lane & 31u)) & 1u) out[base + rank] = tb + 64u * (uint32_t)k + lane;
    base += (uint32_t)(__builtin_popcount(lo) + __builtin_popcount(hi));
  }
}

__global__ void __launch_bounds__(256) k_compact(CompactArgs a) {
  // the limit check of Algorithm 1 on the device: an empty or over-limit
  // selection writes no id, so the host learns the outcome with one wait
  const uint64_t total = *a.total;
  if (total == 0 || total > a.limit) return;
  const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  const uint32_t tpw = a.tiles_per_wave;
  const uint32_t t0 = (blockIdx.x * 4u + wave) * tpw;
  if (t0 >= a.ntiles) return;
  const uint32_t nt = min(tpw, a.ntiles - t0);
  // lane q (q < nt) looks up tile t0 + q: its word map, count and first word
  const uint32_t tile = t0 + (lane < nt ? lane : 0u);
  uint32_t turn;
  const uint32_t place = tile_place(a.order, tile, turn);
  const uint64_t nz = lane < nt ? a.tile_words[place] : 0ull;
  const uint32_t meta = a.tile_meta[place];
  const uint32_t word0 = (place - turn % kMaskGroup) * (a.quarters ? 8u * kSmallSteps : (uint32_t)kWave) +
                         (meta >> kMetaShift);   // < 2^27
  // ids before the wave's first tile
  uint32_t before = 0;
  if (a.offsets) {
    if (lane == 0) before = a.offsets[t0];
    for (uint32_t i = lane; i < (t0 >> 10); i += kWave) before += a.chunk_sums[i];
  } else {
#pragma unroll 4
    for (uint32_t i = lane; i < t0; i += kWave) before += a.tile_meta[i] & kMetaCount;
  }
  // tile q's map, first word and the words of the tiles before it
  uint32_t lo[4], hi[4], w0[4], sum[5];
  sum[0] = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    lo[q] = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)nz, q);
    hi[q] = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(nz >> 32), q);
    w0[q] = (uint32_t)__builtin_amdgcn_readlane((int)word0, q);
    sum[q + 1] = sum[q] + (uint32_t)(__builtin_popcount(lo[q]) + __builtin_popcount(hi[q]));
  }
  if (a.quarters) {
    // a small scan's four quarters make a tile: word r of it in lane r
    const uint32_t mlo = lo[0] | (lo[1] << 16), mhi = lo[2] | (lo[3] << 16);
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, 0u));
    const uint32_t q = lane >> 4;
    const uint32_t from = (q == 0 ? w0[0] : q == 1 ? w0[1] - sum[1] : q == 2 ? w0[2] - sum[2] : w0[3] - sum[3]) + rank;
    const bool set = (((lane & 32u ? mhi : mlo) >> (lane & 31u)) & 1u) != 0u;
    const uint32_t w = set ? a.mask[from] : 0u;
    compact_tile(w, wave_sum(before), t0 / 4u, lane, a.out);
    return;
  }
  if (sum[4] <= (uint32_t)kWave) {
    // All the wave's words at once, lane x the x-th: the tile it belongs to,
    // its word (the tile's words are packed), and its number in the tile,
    // which the set lane of that number in the tile's map sends to x; the
    // other lanes send zeros to the places left.  A tile at a time, with the
    // eight prefix sums that lane-ordered words needed, was 63 us for the
    // 1.6M ids of 300M rows; now 26.
    const uint32_t q = (lane >= sum[1]) + (lane >= sum[2]) + (lane >= sum[3]);
    const uint32_t from = (q == 0 ? w0[0] : q == 1 ? w0[1] - sum[1] : q == 2 ? w0[2] - sum[2] : w0[3] - sum[3]) + lane;
    const uint32_t w = lane < sum[4] ? a.mask[from] : 0u;
    const uint32_t base = wave_sum(before);
    uint32_t number = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi[k], __builtin_amdgcn_mbcnt_lo(lo[k], 0u));
      const bool set = (((lane & 32u ? hi[k] : lo[k]) >> (lane & 31u)) & 1u) != 0u;
      const uint32_t to = (set ? sum[k] + rank : sum[k + 1] + lane - rank) & 63u;
      number |= (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)(set ? lane : 0u));
    }
    const uint32_t c = __builtin_popcount(w), first = (t0 + q) * (uint32_t)kTileRows + 32u * number;
    // a lane's word at a time takes as many stores as the fullest word has
    // rows, each to as many lines as there are full words; two words at a time
    // half as many stores as words, each to one or two lines.  12 % of 200M
    // rows in runs of 700: 192 us word by word, 110 in pairs; 3 % in runs of 8
    // 103 and 107.
    if (__ballot(2u * c > sum[4])) {
      put_words(w, first, sum[4], base, lane, a.out);
      return;
    }
    uint32_t run;
    const uint32_t pos = wave_incl_sum(c, lane, run) - c;
    put_bits(w, base + pos, first, a.out);
    return;
  }
  uint32_t base = wave_sum(before);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if ((lo[k] | hi[k]) == 0u) continue;  // no TRUE row in the tile
    // word r is packed at its rank among the nonzero ones
    const uint32_t raw = lane < sum[k + 1] - sum[k] ? a.mask[w0[k] + lane] : 0u;
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(hi[k], __builtin_amdgcn_mbcnt_lo(lo[k], 0u));
    const uint32_t word = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(rank << 2), (int)raw);
    const bool set = (((lane & 32u ? hi[k] : lo[k]) >> (lane & 31u)) & 1u) != 0u;
    compact_tile(set ? word : 0u, base, t0 + (uint32_t)k, lane, a.out);
    base += (uint32_t)__builtin_amdgcn_readlane((int)meta, k) & kMetaCount;
  }
}

// ---------------------------------------------------- projected columns --
// Materialised sigma(R) with its projected columns (Ch.3 sec.3.3): each wave
// takes kGatherUnroll x 64 consecutive outputs, loads all their row ids
// first (coalesced; ascending ids make neighbouring lanes read neighbouring
// rows), then per column issues every gather before any store; the validity
// bits of each 64 outputs are one ballot, written as two words.  An id past
// the table's rows gives 0 and NULL and is counted.
constexpr int kGatherUnroll = 4;

template <class T>
__device__ __forceinline__ void gather_col(const GatherCol& C, uint64_t base, uint32_t lane,
                                           const uint32_t (&row)[kGatherUnroll],
                                           const bool (&in)[kGatherUnroll],
                                           const bool (&ok)[kGatherUnroll]) {
  const GLOBAL T* src = gptr<T>(C.src);
  T v[kGatherUnroll];
#pragma unroll
  for (int j = 0; j < kGatherUnroll; ++j) v[j] = ok[j] ? src[row[j]] : (T)0;
#pragma unroll
  for (int j = 0; j < kGatherUnroll; ++j)
    if (in[j]) ((T*)C.out)[base + 64 * j + lane] = v[j];
}

__global__ void __launch_bounds__(256) k_gather(GatherArgs a) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * kGatherUnroll;
  uint32_t bad = 0;
  for (uint64_t base = ((uint64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u)) * kGatherUnroll;
       base < a.count; base += stride) {
    uint32_t row[kGatherUnroll];
    bool in[kGatherUnroll], ok[kGatherUnroll];
#pragma unroll
    for (int j = 0; j < kGatherUnroll; ++j) {
      const uint64_t k = base + 64 * j + lane;
      in[j] = k < a.count;
      row[j] = in[j] ? __builtin_nontemporal_load(gptr<uint32_t>(a.ids) + k) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kGatherUnroll; ++j) {
      ok[j] = in[j] && row[j] < a.nrows;
      bad += (in[j] && !ok[j]) ? 1u : 0u;
    }
    for (uint32_t c = 0; c < a.ncols; ++c) {
      const GatherCol& C = a.cols[c];
      switch (C.width) {
        case 1: gather_col<uint8_t>(C, base, lane, row, in, ok); break;
        case 2: gather_col<uint16_t>(C, base, lane, row, in, ok); break;
        case 4: gather_col<uint32_t>(C, base, lane, row, in, ok); break;
        default: gather_col<uint64_t>(C, base, lane, row, in, ok); break;
      }
      if (C.out_valid) {
        uint32_t vw[kGatherUnroll];
#pragma unroll
        for (int j = 0; j < kGatherUnroll; ++j)
          vw[j] = ok[j] && C.valid != nullptr ? gptr<uint32_t>(C.valid)[row[j] >> 5] : ~0u;
#pragma unroll
        for (int j = 0; j < kGatherUnroll; ++j) {
          const bool v = ok[j] && ((vw[j] >> (row[j] & 31)) & 1u);
          const uint64_t m = __ballot(v);
          const uint64_t w = (base + 64 * j) >> 5;
          if (lane == 0 && in[j]) C.out_valid[w] = (uint32_t)m;
          if (lane == 32 && in[j]) C.out_valid[w + 1] = (uint32_t)(m >> 32);
        }
      }
    }
  }
  finish(a.slot, nullptr, a.host, 0u, bad, true);
}

// --------------------------------------------------------- batched count --
// Column values of one pipeline segment: a full tile of a narrow column or
// half a tile of an int64 column, 128 B per lane at most.  Narrow types use
// the leading components of each step's vector.
struct Seg { v4i w[kSteps]; };

template <int TY>
__device__ __forceinline__ auto seg_get(const Seg& r, int b) {
  const int j = b >> 2, i = b & 3;
  if constexpr (TY == T_I8) {
    return (int32_t)(int8_t)((uint32_t)r.w[j][0] >> (8 * i));
  } else if constexpr (TY == T_I16) {
    return (int32_t)(int16_t)((uint32_t)r.w[j][i >> 1] >> (16 * (i & 1)));
  } else if constexpr (TY == T_I32) {
    return (int32_t)r.w[j][i];
  } else {  // b indexes the loaded half: 0..15
    const v4i& q = r.w[2 * j + (i >> 1)];
    const int k = 2 * (i & 1);
    return (int64_t)(((uint64_t)(uint32_t)q[k + 1] << 32) | (uint32_t)q[k]);
  }
}

// Issue the loads of a segment (and, with a column's first segment, of its
// validity word); nothing waits for them here.
__device__ __forceinline__ void seg_issue(Seg& r, uint32_t& V, const CONSTANT BatchCol* C, int h,
                                          uint64_t tb, uint32_t lane) {
  const void* data = C->data;
  switch (C->type) {
    case T_I8: {
      const GLOBAL uint32_t* p = gptr<uint32_t>((const int8_t*)data + tb) + lane;
#pragma unroll
      for (int j = 0; j < kSteps; ++j) r.w[j][0] = (int32_t)__builtin_nontemporal_load(p + 64 * j);
      break;
    }
    case T_I16: {
      const GLOBAL v2i* p = gptr<v2i>((const int16_t*)data + tb) + lane;
#pragma unroll
      for (int j = 0; j < kSteps; ++j) {
        const v2i x = __builtin_nontemporal_load(p + 64 * j);
        r.w[j][0] = x[0];
        r.w[j][1] = x[1];
      }
      break;
    }
    case T_I32: {
      const GLOBAL v4i* p = gptr<v4i>((const int32_t*)data + tb) + lane;
#pragma unroll
      for (int j = 0; j < kSteps; ++j) r.w[j] = __builtin_nontemporal_load(p + 64 * j);
      break;
    }
    default: {  // int64: h = 0 loads steps 4..7 (bits 16..31), h = 1 steps 0..3
      const GLOBAL v4i* p = gptr<v4i>((const int64_t*)data + tb) + 2 * lane + 128 * 4 * (1 - h);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        r.w[2 * j] = __builtin_nontemporal_load(p + 128 * j);
        r.w[2 * j + 1] = __builtin_nontemporal_load(p + 128 * j + 1);
      }
      break;
    }
  }
  if (h == 0 && C->vslot != kNoSlot) V = valid_bits<true>(C->valid, tb, lane, tb + kTileRows);
}

// Rows a direct factor of a conjunction still needs tested: those its
// program's accumulator still holds TRUE.
__device__ __forceinline__ uint32_t acc_need(uint32_t sl, const uint32_t* wl, uint32_t lane) {
  return wl[(sl & 0xFFFu) * kWave + lane];
}

// Validity word of a leaf's column (all ones without NULLs).
__device__ __forceinline__ uint32_t leaf_valid(uint32_t sl, const uint32_t* wl, uint32_t lane) {
  const uint32_t vs = (sl >> 24) & 0x7Fu;
  return vs == kAccNoValid ? ~0u : wl[vs * kWave + lane];
}

// *w &= x and *w |= x on the lane's own LDS word, by the LDS itself: nothing
// is read back and waited for.
__device__ __forceinline__ void lds_and(uint32_t* w, uint32_t x) {
  __hip_atomic_fetch_and(w, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void lds_or(uint32_t* w, uint32_t x) {
  __hip_atomic_fetch_or(w, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// Stores a leaf's TRUE word (its test on non-NULL rows): into its slot, or
// for a direct factor of a conjunction ANDed into its program's accumulator,
// or for a leaf of an OR factor of narrow tests ORed into that factor's word.
__device__ __forceinline__ void put_leaf(uint32_t* wl, uint32_t lane, uint32_t sl, uint32_t P) {
  const uint32_t T = P & leaf_valid(sl, wl, lane);
  uint32_t* w = wl + (sl & 0xFFFu) * kWave + lane;
  if (!(sl & kAccTarget)) *w = T;
  else if (sl & kAccOr) lds_or(w, T);
  else lds_and(w, T);
}

// Resets the accumulators of an entry's programs for a new tile.
__device__ __forceinline__ void reset_acc(const CONSTANT BatchTable* E, const CONSTANT uint32_t* ops,
                                          uint32_t* wl, uint32_t lane) {
  const uint32_t ib = E->init_begin, in = E->init_count;
  for (uint32_t k = 0; k < in; k += kSlotGroup) {
    const v8u w = *(const CONSTANT v8u*)(ops + ib + k);
#pragma unroll
    for (uint32_t q = 0; q < kSlotGroup; ++q)
      wl[(w[q] & 0xFFFu) * kWave + lane] = (w[q] & kInitTrue) ? ~0u : 0u;
  }
}

// Value tests of one leaf on a segment: bits [0, nb) of the result, highest
// row first.  A bitmap leaf in global memory that is a direct factor of a
// conjunction looks up only rows its program's accumulator does not hold
// FALSE; the others read word 0 and test FALSE.  `gshift` places the
// segment's rows in the guard word (16 for the upper half of an int64
// column).
template <int TY>
__device__ __forceinline__ uint32_t seg_leaf(const Seg& r, uint32_t op, CInstr I,
                                             const uint32_t* bmlds, const uint32_t* wl,
                                             uint32_t lane, int gshift) {
  constexpr int nb = TY == T_I64 ? 16 : 32;
  const int64_t lo = I->lo;
  const uint64_t span = I->span;
  uint32_t P = 0;
  if (op == D_BITMAP && I->lds_word != kNoLds) {
    // staged copy: an offset past the window is clamped to the zero bit z
    // that follows the copied words, so no test or select is needed.  For
    // narrow columns the window lies inside int32 (the host stages only
    // such bitmaps), so 32-bit differences are exact.
    const uint32_t* bm = bmlds + I->lds_word;
    const uint32_t z = I->n;
    if constexpr (TY == T_I64) {
#pragma unroll
      for (int b = nb - 1; b >= 0; --b) {
        const uint64_t d = (uint64_t)seg_get<TY>(r, b) - (uint64_t)lo;
        const uint32_t k = d < z ? (uint32_t)d : z;
        P = (P << 1) + ((bm[k >> 5] >> (k & 31)) & 1u);
      }
    } else {
      // eight rows at a time: their LDS reads are all issued before the
      // first bit is taken, so one wait covers eight round trips
      const uint32_t lo32 = (uint32_t)lo;
#pragma unroll
      for (int g = nb - 8; g >= 0; g -= 8) {
        uint32_t k[8], w[8];
#pragma unroll
        for (int q = 7; q >= 0; --q) {
          const uint32_t d = (uint32_t)seg_get<TY>(r, g + q) - lo32;
          k[q] = d < z ? d : z;
        }
#pragma unroll
        for (int q = 7; q >= 0; --q) w[q] = bm[k[q] >> 5];
#pragma unroll
        for (int q = 7; q >= 0; --q) P = (P << 1) + ((w[q] >> (k[q] & 31)) & 1u);
      }
    }
  } else if (op == D_RANGE) {
    if constexpr (TY == T_I64) {
      // one-sided ranges (x >= lo, x <= hi) need one compare per row
      if ((uint64_t)lo + span == (uint64_t)INT64_MAX) {
#pragma unroll
        for (int b = nb - 1; b >= 0; --b) P = (P << 1) + (uint32_t)(seg_get<TY>(r, b) >= lo);
      } else if (lo == INT64_MIN) {
        const int64_t hi = (int64_t)((uint64_t)lo + span);
#pragma unroll
        for (int b = nb - 1; b >= 0; --b) P = (P << 1) + (uint32_t)(seg_get<TY>(r, b) <= hi);
      } else {
#pragma unroll
        for (int b = nb - 1; b >= 0; --b)
          P = (P << 1) + (uint32_t)((uint64_t)seg_get<TY>(r, b) - (uint64_t)lo <= span);
      }
    } else {
      const uint32_t lo32 = (uint32_t)lo, span32 = (uint32_t)span;
#pragma unroll
      for (int b = nb - 1; b >= 0; --b)
        P = (P << 1) + (uint32_t)((uint32_t)seg_get<TY>(r, b) - lo32 <= span32);
    }
  } else {  // D_BITMAP in global memory
    const GLOBAL uint32_t* bits = gptr<uint32_t>(I->aux);
    uint32_t need = ~0u;
    if (I->flags == kAccGuard) need = acc_need(I->slot, wl, lane) >> gshift;
#pragma unroll
    for (int b = nb - 1; b >= 0; --b) {
      uint64_t d;
      if constexpr (TY == T_I64) d = (uint64_t)seg_get<TY>(r, b) - (uint64_t)lo;
      else d = (uint64_t)((int64_t)seg_get<TY>(r, b) - lo);
      const bool ok = d < span && ((need >> b) & 1u);
      const uint32_t k = ok ? (uint32_t)d : 0u;
      P = (P << 1) + (ok & ((bits[k >> 5] >> (k & 31)) & 1u));
    }
  }
  return P;
}

// In-register transpose of a 32 x 32 bit matrix: on return a[c] bit r is
// what a[r] bit c was.  Each stage swaps, in every 2s x 2s block, the s x s
// block above the diagonal with the one below it.
// Only words 0 .. NOUT-1 of the result are wanted: later stages mix words
// within blocks of S, so a stage updates only the words below
// ceil(NOUT / S) * S.
template <int S, int NOUT>
__device__ __forceinline__ void transpose_stage(uint32_t (&a)[32], uint32_t m) {
  constexpr int R = (NOUT + S - 1) / S * S;
#pragma unroll
  for (int g = 0; g < 32; g += 2 * S) {
#pragma unroll
    for (int k = g; k < g + S; ++k) {
      if (k >= R) continue;
      const uint32_t t = ((a[k] >> S) ^ a[k + S]) & m;
      if (k + S < R) a[k + S] ^= t;
      a[k] ^= t << S;
    }
  }
}

template <int NOUT>
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
  transpose_stage<16, NOUT>(a, 0x0000FFFFu);
  transpose_stage<8, NOUT>(a, 0x00FF00FFu);
  transpose_stage<4, NOUT>(a, 0x0F0F0F0Fu);
  transpose_stage<2, NOUT>(a, 0x33333333u);
  transpose_stage<1, NOUT>(a, 0x55555555u);
}

// The table leaves of a narrow column on one segment: one lookup per row
// (entries of E: one bit per leaf, NOUT >= the leaf count) serves them all;
// transposed, word i holds leaf i's truth bits.
template <class E, int NOUT, int TY>
__device__ __forceinline__ void tab_leaves(const Seg& r, const CONSTANT BatchCol* C,
                                           const CONSTANT uint32_t* ops,
                                           const uint32_t* bmlds, uint32_t* wl, uint32_t lane) {
  const uint32_t L32 = (uint32_t)C->tab_lo, n = C->tab_n, m = C->tab_count;
  uint32_t sl[NOUT];   // uniform
#pragma unroll
  for (int i = 0; i < NOUT; i += (int)kSlotGroup) {
    const v8u s = *(const CONSTANT v8u*)(ops + C->tab_slots + i);
#pragma unroll
    for (int q = 0; q < (int)kSlotGroup; ++q) sl[i + q] = s[q];
  }
  uint32_t T[32];
  if (C->tab_word != kNoLds) {
    const E* tab = (const E*)(bmlds + C->tab_word);
#pragma unroll
    for (int b = 0; b < 32; ++b) {
      const uint32_t d = (uint32_t)seg_get<TY>(r, b) - L32;
      T[b] = tab[d < n ? d : n];
    }
  } else {
    // 32-bit byte offsets from the table's uniform base (device tables
    // are at most 32 MB)
    const GLOBAL char* tab = gptr<char>(C->gtab);
    if (C->tab_flags & kTabGuarded) {
      // rows no table leaf needs (the complement of the union of the
      // leaves' guards) read the zero entry n: with g all ones on such a
      // row, min(d | g, n) is n, and on the others it is min(d, n)
      uint32_t need = 0;
#pragma unroll
      for (int i = 0; i < NOUT; ++i) need |= acc_need(sl[i], wl, lane);
      const uint32_t skip = ~need;
#pragma unroll
      for (int b = 0; b < 32; ++b) {
        const uint32_t d = (uint32_t)seg_get<TY>(r, b) - L32;
        const uint32_t g = (uint32_t)((int32_t)(skip << (31 - b)) >> 31);
        const uint32_t k = min(d | g, n);
        T[b] = *(const GLOBAL E*)(tab + k * (uint32_t)sizeof(E));
      }
    } else {
#pragma unroll
      for (int b = 0; b < 32; ++b) {
        const uint32_t d = (uint32_t)seg_get<TY>(r, b) - L32;
        const uint32_t k = min(d, n);
        T[b] = *(const GLOBAL E*)(tab + k * (uint32_t)sizeof(E));
      }
    }
  }
  // row b's entry holds leaf i in bit i; transposed, T[i] holds leaf i's
  // word (bit b = row b)
  transpose32<NOUT>(T);
  if (C->tab_flags & kTabFactors) {
    const uint32_t V = leaf_valid(sl[0], wl, lane);
#pragma unroll
    for (int i = 0; i < NOUT; ++i)
      if ((uint32_t)i < m) lds_and(wl + (sl[i] & 0xFFFu) * kWave + lane, T[i] & V);
  } else {
#pragma unroll
    for (int i = 0; i < NOUT; ++i)
      if ((uint32_t)i < m) put_leaf(wl, lane, sl[i], T[i]);
  }
}

// A sparse IN-list leaf of the batched kernel (its registers are spent on the
// column pipeline): the four rows of a step at a time, loop kept rolled.  A row
// at a time, a step's lines were read four times over, from L1 as long as the
// other waves' lines left them there: six int64 lists of 12 values, 200M rows,
// 6.40 ms, now 4.81.
template <int TY>
__device__ __noinline__ uint32_t inlist_rows(CInstr I_, uint64_t tb_, uint32_t lane) {
  const CInstr I = (CInstr)uni64((uint64_t)I_);
  const uint64_t tb = uni64(tb_);
  const GLOBAL int64_t* list = gptr<int64_t>(I->aux);
  const uint32_t n = I->n;
  const GLOBAL char* data = gptr<char>(I->data) + tb * type_width<TY>();
  uint32_t P = 0;
#pragma unroll 1
  for (int j = kSteps - 1; j >= 0; --j) {
    const uint32_t at = type_width<TY>() * (256u * (uint32_t)j + 4u * lane);
    int64_t x[4];
    if constexpr (TY == T_I8) {
      const uint32_t w = *(const GLOBAL uint32_t*)(data + at);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (int64_t)(int8_t)(w >> (8 * i));
    } else if constexpr (TY == T_I16) {
      const v2i w = *(const GLOBAL v2i*)(data + at);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (int64_t)(int16_t)((uint32_t)w[i >> 1] >> (16 * (i & 1)));
    } else if constexpr (TY == T_I32) {
      const v4i w = *(const GLOBAL v4i*)(data + at);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (int64_t)w[i];
    } else {
      const v4i w[2] = {*(const GLOBAL v4i*)(data + at), *((const GLOBAL v4i*)(data + at) + 1)};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const v4i& v = w[i >> 1];
        x[i] = (int64_t)(((uint64_t)(uint32_t)v[2 * (i & 1) + 1] << 32) | (uint32_t)v[2 * (i & 1)]);
      }
    }
    uint32_t base[4] = {};
    for (uint32_t len = n; len > 1;) {
      const uint32_t half = len >> 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) base[i] = list[base[i] + half] <= x[i] ? base[i] + half : base[i];
      len -= half;
    }
#pragma unroll
    for (int i = 3; i >= 0; --i) P = (P << 1) + (list[base[i]] == x[i] ? 1u : 0u);
  }
  return P;
}

// Every leaf of one segment; truth words go to the wave's slots.  An int64
// column's upper half (h = 0) writes bits 16..31, its lower half completes
// them.  Sparse value lists take the element path once, with the last
// segment of their column.
template <int TY>
__device__ __forceinline__ void seg_leaves(const Seg& r, const CONSTANT BatchCol* C, int h,
                                           CInstr leaves, const CONSTANT uint32_t* ops,
                                           uint64_t tb, uint32_t lane,
                                           uint32_t* wl, const uint32_t* bmlds) {
  const uint32_t lb = C->leaf_begin, ln = C->leaf_count;
  const uint32_t tw = TY != T_I64 ? C->tab_word : kNoLds;
  const bool tabled = TY != T_I64 && (tw != kNoLds || C->gtab != nullptr);
  // leaves outside the table first: the values die once the table is read
  for (uint32_t k = tabled ? C->tab_count : 0u; k < ln; ++k) {
    CInstr I = leaves + lb + k;
    const uint32_t op = I->op;
    if (op == D_INLIST) {
      if (TY != T_I64 || h == 1) put_leaf(wl, lane, I->slot, inlist_rows<TY>(I, tb, lane));
      continue;
    }
    const uint32_t P = seg_leaf<TY>(r, op, I, bmlds, wl, lane, TY == T_I64 && h == 0 ? 16 : 0);
    if constexpr (TY != T_I64) {
      put_leaf(wl, lane, I->slot, P);
    } else {  // int64 leaves always have a slot of their own
      const uint32_t sl = I->slot;
      uint32_t* w = wl + (sl & 0xFFFu) * kWave + lane;
      if (h == 0) *w = P;
      else *w = ((*w << 16) | P) & leaf_valid(sl, wl, lane);
    }
  }
  if constexpr (TY != T_I64) {
    if (tw != kNoLds || C->gtab != nullptr) {
      const uint32_t m = C->tab_count;
      if (m <= 8) tab_leaves<uint8_t, 8, TY>(r, C, ops, bmlds, wl, lane);
      else if (m <= 16) tab_leaves<uint16_t, 16, TY>(r, C, ops, bmlds, wl, lane);
      else tab_leaves<uint32_t, 32, TY>(r, C, ops, bmlds, wl, lane);
    }
  }
}

// All leaf tests of an entry on a full tile, as a software pipeline over
// the segments of the columns that have leaves: the loads of the next
// segment are in flight while the leaves of the current one run.
__device__ __forceinline__ void entry_leaves_full(const CONSTANT BatchTable* E,
                                                  const CONSTANT BatchCol* cols, CInstr leaves,
                                                  uint64_t tb, uint32_t lane, uint32_t* wl,
                                                  const uint32_t* bmlds, const CONSTANT uint32_t* ops) {
  const uint32_t cb = E->col_begin, cn = E->col_count;
  reset_acc(E, ops, wl, lane);
  // columns that only null tests read: validity alone
  for (uint32_t c = 0; c < cn; ++c) {
    const CONSTANT BatchCol* C = cols + cb + c;
    if (!C->leaf_count && C->vslot != kNoSlot)
      wl[C->vslot * kWave + lane] = valid_bits<true>(C->valid, tb, lane, tb + kTileRows);
  }
  uint32_t c = 0;
  while (c < cn && !cols[cb + c].leaf_count) ++c;
  if (c == cn) return;
  Seg cur;
  uint32_t curV = ~0u;
  int h = 0;
  seg_issue(cur, curV, cols + cb + c, h, tb, lane);
  for (;;) {
    const CONSTANT BatchCol* C = cols + cb + c;
    const uint32_t ty = C->type;
    uint32_t nc = c;
    int nh = 0;
    if (ty == T_I64 && h == 0) {
      nh = 1;
    } else {
      ++nc;
      while (nc < cn && !cols[cb + nc].leaf_count) ++nc;
    }
    const bool more = nc < cn;
    Seg nxt;
    uint32_t nxtV = ~0u;
    if (more) seg_issue(nxt, nxtV, cols + cb + nc, nh, tb, lane);
    if (h == 0 && C->vslot != kNoSlot) wl[C->vslot * kWave + lane] = curV;
    switch (ty) {
      case T_I8: seg_leaves<T_I8>(cur, C, h, leaves, ops, tb, lane, wl, bmlds); break;
      case T_I16: seg_leaves<T_I16>(cur, C, h, leaves, ops, tb, lane, wl, bmlds); break;
      case T_I32: seg_leaves<T_I32>(cur, C, h, leaves, ops, tb, lane, wl, bmlds); break;
      default: seg_leaves<T_I64>(cur, C, h, leaves, ops, tb, lane, wl, bmlds); break;
    }
    if (!more) break;
    cur = nxt;
    curV = nxtV;
    c = nc;
    h = nh;
  }
}

// All leaf tests of an entry on the partial last tile of its table.
__device__ __forceinline__ void entry_leaves_partial(const CONSTANT BatchTable* E,
                                                     const CONSTANT BatchCol* cols, CInstr leaves,
                                                     uint64_t tb, uint32_t lane, uint64_t nrows,
                                                     uint32_t* wl, const CONSTANT uint32_t* ops) {
  const uint32_t cb = E->col_begin, cn = E->col_count;
  reset_acc(E, ops, wl, lane);
  for (uint32_t c = 0; c < cn; ++c) {
    const CONSTANT BatchCol* C = cols + cb + c;
    const uint32_t lb = C->leaf_begin, ln = C->leaf_count;
    // validity first: direct factors read it when they are stored
    const uint32_t vs = C->vslot;
    if (vs != kNoSlot) wl[vs * kWave + lane] = valid_bits<false>(C->valid, tb, lane, nrows);
    for (uint32_t k = 0; k < ln; ++k) {
      CInstr I = leaves + lb + k;
      const uint32_t P = partial_leaf<false>(load_ins(I), C->type, tb, lane, nrows, StageView{});
      put_leaf(wl, lane, I->slot, P);
    }
  }
}

// TRUE bits of the lane's rows for one batched program: its postfix
// combinators over the leaf and validity words in the wave's slots.
__device__ __forceinline__ uint32_t run_ops(const CONSTANT uint32_t* ops, uint32_t nops,
                                            const uint32_t* wl, uint32_t lane) {
  uint32_t st[kMaxDepth], sf[kMaxDepth];
  uint32_t tt = 0, tf = 0;
  int d = 0;
  for (uint32_t pc = 0; pc < nops; ++pc) {
    const uint32_t w = ops[pc];
    const uint32_t op = w & 0xFFu;
    if (op == B_AND_LEAF || op == B_OR_LEAF) {
      const uint32_t vs = w >> 20;
      const uint32_t V = vs == kNoSlot ? ~0u : wl[vs * kWave + lane];
      const uint32_t P = wl[((w >> 8) & 0xFFFu) * kWave + lane];
      if (op == B_AND_LEAF) { tt &= P & V; tf |= ~P & V; }
      else { tt |= P & V; tf &= ~P & V; }
    } else if (op == B_ACC || op == B_AND_ACC) {
      const uint32_t fs = w >> 20;
      const uint32_t T = wl[((w >> 8) & 0xFFFu) * kWave + lane];
      const uint32_t F = fs == kNoSlot ? ~T : wl[fs * kWave + lane];
      if (op == B_AND_ACC) {
        tt &= T; tf |= F;
      } else {
        if (d > 0) {
          st[uni(d - 1)] = tt;
          sf[uni(d - 1)] = tf;
        }
        tt = T; tf = F;
        ++d;
      }
    } else if (op < D_AND || op == D_TRUE || op == D_FALSE) {
      uint32_t t, f;
      const uint32_t vs = w >> 20;
      const uint32_t V = (vs == kNoSlot || op >= D_TRUE) ? ~0u : wl[vs * kWave + lane];
      switch (op) {
        case D_RANGE: {
          const uint32_t P = wl[((w >> 8) & 0xFFFu) * kWave + lane];
          t = P & V; f = ~P & V;
          break;
        }
        case D_NN_TRUE: t = V; f = 0; break;
        case D_NN_FALSE: t = 0; f = V; break;
        case D_ISNULL: t = ~V; f = V; break;
        case D_NOTNULL: t = V; f = ~V; break;
        case D_TRUE: t = ~0u; f = 0; break;
        default: t = 0; f = ~0u; break;  // D_FALSE
      }
      if (d > 0) {
        st[uni(d - 1)] = tt;
        sf[uni(d - 1)] = tf;
      }
      tt = t; tf = f;
      ++d;
    } else if (op == D_NOT) {
      const uint32_t x = tt; tt = tf; tf = x;
    } else if (op == D_ISUNK) {
      const uint32_t k = tt | tf; tt = ~k; tf = k;
    } else {
      const uint32_t at = st[uni(d - 2)], af = sf[uni(d - 2)];
      if (op == D_AND) { tt &= at; tf |= af; }
      else { tt |= at; tf &= af; }
      --d;
    }
  }
  return tt;
}

// The same for a program with no NOT and no IS UNKNOWN: the TRUE word of an
// AND or OR is the AND or OR of its operands' TRUE words, so the TRUE words
// of leaves (NULL rows cleared) and null tests are all it needs, one word
// per stack entry.
__device__ __forceinline__ uint32_t run_ops2(const CONSTANT uint32_t* ops, uint32_t nops,
                                             const uint32_t* wl, uint32_t lane) {
  uint32_t st[kMaxDepth];
  uint32_t tt = 0;
  int d = 0;
  for (uint32_t pc = 0; pc < nops; ++pc) {
    const uint32_t w = ops[pc];
    const uint32_t op = w & 0xFFu;
    if (op >= B_AND_LEAF) {   // fused leaves and the accumulator
      const uint32_t P = wl[((w >> 8) & 0xFFFu) * kWave + lane];
      if (op == B_AND_LEAF || op == B_AND_ACC) {
        tt &= P;
      } else if (op == B_OR_LEAF) {
        tt |= P;
      } else {  // B_ACC
        if (d > 0) st[uni(d - 1)] = tt;
        tt = P;
        ++d;
      }
    } else if (op < D_AND || op == D_TRUE || op == D_FALSE) {
      uint32_t t;
      if (op == D_RANGE) {
        t = wl[((w >> 8) & 0xFFFu) * kWave + lane];
      } else {
        const uint32_t vs = w >> 20;
        const uint32_t V = (vs == kNoSlot || op >= D_TRUE) ? ~0u : wl[vs * kWave + lane];
        t = (op == D_NN_TRUE || op == D_NOTNULL) ? V : op == D_ISNULL ? ~V : op == D_TRUE ? ~0u : 0u;
      }
      if (d > 0) st[uni(d - 1)] = tt;
      tt = t;
      ++d;
    } else if (op == D_NOT) {
      tt = ~tt;
    } else if (op == D_ISUNK) {
      tt = 0;
    } else {
      const uint32_t at = st[uni(d - 2)];
      if (op == D_AND) tt &= at;
      else tt |= at;
      --d;
    }
  }
  return tt;
}

// Star programs (one lookup per dimension and row serves 16 of them) over 160M
// rows: 230 us with the two dimensions whose tables fit LDS, at the rate of the
// columns' bytes; a third of 200,000 keys (400 KB) adds 460 us, all of them
// lines of 128 bytes that L2 sends the CU for two bytes each (0.42 lines a
// cycle and CU with no row skipped, of 0.5 that 64 bytes a cycle allow), and a
// fourth of 3.2M keys 250 us.  What a tile does besides is kept off that path:
// slots are read eight at a time by one scalar load, words combine in the LDS,
// and programs of one word are counted sixteen at a time (1690 scalar
// instructions and 219 scalar loads a tile became 800 and 75; 985 -> 943 us).
//
// Per workgroup, per-program counts accumulate in LDS; at the end each
// workgroup adds them to per-program accumulator lines (128 bytes each, so
// atomics on different programs do not contend), and the last workgroup by
// ticket moves the finished lines out and zeroes them.  Entries may be
// chunks of tables (row_begin), and lines not finished by this launch keep
// accumulating: a cooperative scan adds one chunk per launch.
__global__ void __launch_bounds__(768) k_batch(BatchArgs a) {
  // LDS: per-program counters, tables and staged bitmaps, each wave's slots
  extern __shared__ __align__(16) uint32_t dyn[];
  // the wave's number is made scalar, so that its slots' address is: in a
  // vector register it was spilled, and reloaded five times a tile (one star
  // program over four dimensions, 200M rows: 766 us, now 730)
  const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  const uint32_t nw = blockDim.x >> 6;
  const uint32_t nacc = a.acc_words;   // min(nprogs, kBatchMaxProgs)
  uint32_t* acc = dyn;
  uint32_t* bmlds = dyn + nacc;
  uint32_t* wl = bmlds;   // this wave's slots, placed by each pass's layout
  for (uint32_t p = threadIdx.x; p < nacc; p += blockDim.x) acc[p] = 0;
  __syncthreads();
  const CONSTANT BatchTable* tables = (const CONSTANT BatchTable*)a.tables;
  const CONSTANT BatchCol* cols = (const CONSTANT BatchCol*)a.cols;
  CInstr leaves = (CInstr)a.leaves;
  const CONSTANT BatchProg* progs = (const CONSTANT BatchProg*)a.progs;
  const CONSTANT BatchBitmap* bms = (const CONSTANT BatchBitmap*)a.bms;
  // the workgroup takes groups of nw consecutive tiles; entry ranges are
  // padded to multiples of kBatchTileAlign, so a group never straddles two
  // entries and the loop below (with its barriers) is uniform over the
  // workgroup
  const uint64_t ngroups = a.total_tiles / nw;
  uint32_t staged = 0xFFFFFFFFu;
  uint32_t word0 = 0;   // LDS offset of the TRUE word of the pass's program lane / 4
  for (uint64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
    const uint64_t flat = g * nw + wave;
    // entry holding this tile: last e with tile_begin <= flat (uniform search)
    uint32_t lo = 0, hi = a.ntables;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (tables[mid].tile_begin <= flat) lo = mid; else hi = mid;
    }
    lo = uni(lo);
    const CONSTANT BatchTable* E = tables + lo;
    if (lo != staged) {
      // a new pass: its own LDS layout (tables, bitmaps, slots), so every
      // wave must be done with the previous one's first
      __syncthreads();
      wl = bmlds + E->bm_words + wave * E->slot_words;
      if (E->words_begin != kNoLds)
        word0 = gptr<uint32_t>(a.ops)[E->words_begin + min(lane >> 2, E->prog_count - 1)];
      if (E->bm_count || E->ntab) {
        // lookup tables: copies of the ones k_tables built in device memory
        for (uint32_t c = 0; c < E->col_count; ++c) {
          const CONSTANT BatchCol* C = cols + E->col_begin + c;
          if (C->tab_word == kNoLds) continue;
          const uint32_t words = ((C->tab_n + 1) * tab_entry_bytes(C->tab_count) + 3) / 4;
          const GLOBAL uint32_t* src = gptr<uint32_t>(C->gtab);
          uint32_t* dst = bmlds + C->tab_word;
          for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) dst[i] = src[i];
        }
        for (uint32_t k = 0; k < E->bm_count; ++k) {
          const CONSTANT BatchBitmap* B = bms + E->bm_begin + k;
          const uint32_t n = B->words, last = B->last_mask;
          const GLOBAL uint32_t* src = gptr<uint32_t>(B->src);
          uint32_t* dst = bmlds + B->lds_word;
          for (uint32_t i = threadIdx.x; i <= n; i += blockDim.x) {
            uint32_t w = 0;
            if (i < n) w = i + 1 == n ? src[i] & last : src[i];
            dst[i] = w;
          }
        }
        __syncthreads();
      }
      staged = lo;
    }
    const uint64_t local = flat - E->tile_begin;
    if (local >= E->ntiles) continue;   // padding
    const uint64_t nrows = E->nrows;
    const uint64_t tb = E->row_begin + local * kTileRows;
    const uint32_t pb = E->prog_begin, pn = E->prog_count;
    const bool full = tb + kTileRows <= nrows;
    uint32_t inr = ~0u;
    if (full) {
      entry_leaves_full(E, cols, leaves, tb, lane, wl, bmlds, (const CONSTANT uint32_t*)a.ops);
    } else {
      entry_leaves_partial(E, cols, leaves, tb, lane, nrows, wl, (const CONSTANT uint32_t*)a.ops);
      inr = inrange_bits<kSteps>(tb, lane, nrows);
    }
    if (full && E->words_begin != kNoLds) {
      // every program is one TRUE word: sixteen at a time, a lane counts 16
      // of the 64 lanes' words of its program, each lane of a program from
      // another word on (64 banks)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      for (uint32_t k0 = 0; k0 < pn; k0 += 16) {
        const uint32_t j = lane >> 2, k = k0 + j;
        const uint32_t off = k0 ? gptr<uint32_t>(a.ops)[E->words_begin + min(k, pn - 1)] : word0;
        const uint32_t* w = wl + off + (lane & 3u) * 16u;
        uint32_t c = 0;
#pragma unroll
        for (uint32_t i = 0; i < 16; ++i) c += __builtin_popcount(w[(i + j) & 15u]);
        c += __builtin_amdgcn_update_dpp(0u, c, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
        c += __builtin_amdgcn_update_dpp(0u, c, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
        if ((lane & 3u) == 0 && k < pn && c) {
          if (pb + k < nacc) atomicAdd(&acc[pb + k], c);
          else atomicAdd(&a.acc[(uint64_t)progs[pb + k].acc_index * kBatchAccStride], (unsigned long long)c);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      continue;
    }
    // programs in pairs: both popcounts (at most 2048 per wave each) share
    // one wave reduction, 16 bits apart
    for (uint32_t k = 0; k < pn; k += 2) {
      uint32_t T[2] = {0u, 0u};
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (k + q >= pn) break;
        const CONSTANT BatchProg* P = progs + pb + k + q;
        const uint32_t nops = P->nops;
        const CONSTANT uint32_t* ops = (const CONSTANT uint32_t*)P->ops;
        uint32_t t;
        if (nops & kAndList) {   // a conjunction of TRUE words at these offsets
          const uint32_t n = nops & ~kAndList;
          t = wl[ops[0] + lane];
          for (uint32_t j = 1; j < n; ++j) t &= wl[ops[j] + lane];
        } else if (nops & kTwoValued) {
          t = run_ops2(ops, nops & ~kTwoValued, wl, lane);
        } else {
          t = run_ops(ops, nops, wl, lane);
        }
        T[q] = t & inr;
      }
      const uint32_t c2 = wave_sum(__builtin_popcount(T[0]) | (__builtin_popcount(T[1]) << 16));
      if (lane == 0 && c2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t c = q ? c2 >> 16 : c2 & 0xFFFFu;
          if (!c) continue;
          if (pb + k + q < nacc) {
            atomicAdd(&acc[pb + k + q], c);
          } else {  // beyond the LDS table: straight to the accumulator line
            atomicAdd(&a.acc[(uint64_t)progs[pb + k + q].acc_index * kBatchAccStride], (unsigned long long)c);
          }
        }
      }
    }
  }
  __syncthreads();
  for (uint32_t p = threadIdx.x; p < nacc; p += blockDim.x)
    if (acc[p]) atomicAdd(&a.acc[(uint64_t)progs[p].acc_index * kBatchAccStride], (unsigned long long)acc[p]);
  atomics_done();
  __syncthreads();
  __shared__ bool last;
  if (threadIdx.x == 0) {
    const unsigned int ticket = atomicAdd(&a.slot->ticket, 1u);
    last = ticket == gridDim.x - 1;
  }
  __syncthreads();
  if (last) {
    for (uint32_t k = threadIdx.x; k < a.ndone; k += blockDim.x) {
      const uint64_t line = a.done ? a.done[k] : k;
      put_host(&a.out[k], atomicExch(&a.acc[line * kBatchAccStride], 0ull));
    }
    atomics_done();
    __syncthreads();
    if (threadIdx.x == 0) atomicExch(&a.slot->ticket, 0u);
  }
}

// Bits r (of 32) with a <= r < b.
__device__ __forceinline__ uint32_t span_bits(int64_t a, int64_t b) {
  const uint32_t lo = (uint32_t)(a < 0 ? 0 : a > 32 ? 32 : a), hi = (uint32_t)(b < 0 ? 0 : b > 32 ? 32 : b);
  const uint32_t below = hi < 32u ? (1u << hi) - 1u : ~0u;
  return lo < 32u ? below & (~0u << lo) : 0u;
}

// Device-memory lookup tables of a batch: a thread takes 32 entries, for which
// each leaf's truth is one word (a range's bits, or two neighbouring words of
// its bitmap), and transposes the leaves' words into entries.  A wave works on
// one table, so the leaves are scalar loads, and all bitmap words are in
// flight together.  (A thread per entry, testing one leaf after another, took
// 93 us for the tables of 16 star programs over a 3.2M-key dimension; now 17.)
__global__ void __launch_bounds__(256) k_tables(const TableBuild* __restrict__ tb_, uint32_t nb, uint64_t nunits) {
  const CONSTANT TableBuild* tb = (const CONSTANT TableBuild*)tb_;
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t unit = uni64((uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6));
  if (unit >= nunits) return;
  uint32_t lo = 0, hi = nb;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (tb[mid].unit_begin <= unit) lo = mid; else hi = mid;
  }
  const CONSTANT TableBuild* B = tb + uni(lo);
  const uint64_t e0 = (unit - B->unit_begin) * kTableUnit + 32u * lane;   // first entry
  const uint64_t n = B->n;
  const uint32_t m = B->m;
  if (e0 > n) return;
  const int64_t x0 = B->lo + (int64_t)e0;
  const uint32_t inside = span_bits(0, (int64_t)(n - e0));   // entry n is zero
  CInstr leaves = (CInstr)B->leaves;
  uint32_t a[32];
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    a[k] = 0;
    if ((uint32_t)k >= m) continue;
    CInstr I = leaves + k;
    const int64_t at = (int64_t)((uint64_t)I->lo - (uint64_t)x0);
    if (I->op == D_RANGE) {
      a[k] = span_bits(at, at + (int64_t)I->span + 1) & inside;
    } else {  // D_BITMAP
      const GLOBAL uint32_t* bits = gptr<uint32_t>(I->aux);
      const int64_t span = (int64_t)I->span, w = -at >> 5, words = (span + 31) >> 5;   // floor
      const uint32_t sh = (uint32_t)-at & 31u;
      const uint32_t w0 = w >= 0 && w < words ? bits[w] : 0u;
      const uint32_t w1 = w + 1 >= 0 && w + 1 < words ? bits[w + 1] : 0u;
      a[k] = (uint32_t)((((uint64_t)w1 << 32) | w0) >> sh) & span_bits(at, at + span) & inside;
    }
  }
  transpose32<32>(a);
  const uint32_t eb = tab_entry_bytes(m);
  uint8_t* dst = (uint8_t*)B->dst + e0 * eb;
  const uint32_t cnt = n + 1 - e0 < 32u ? (uint32_t)(n + 1 - e0) : 32u;
  if (cnt < 32u) {
#pragma unroll
    for (int r = 0; r < 32; ++r) {
      if ((uint32_t)r >= cnt) continue;
      if (eb == 1) dst[r] = (uint8_t)a[r];
      else if (eb == 2) ((uint16_t*)dst)[r] = (uint16_t)a[r];
      else ((uint32_t*)dst)[r] = a[r];
    }
  } else if (eb == 4) {
#pragma unroll
    for (int r = 0; r < 32; r += 4) ((v4u*)dst)[r / 4] = v4u{a[r], a[r + 1], a[r + 2], a[r + 3]};
  } else if (eb == 2) {
#pragma unroll
    for (int r = 0; r < 32; r += 8)
      ((v4u*)dst)[r / 8] = v4u{a[r] | (a[r + 1] << 16), a[r + 2] | (a[r + 3] << 16), a[r + 4] | (a[r + 5] << 16),
                               a[r + 6] | (a[r + 7] << 16)};
  } else {
#pragma unroll
    for (int r = 0; r < 32; r += 16) {
      v4u q;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        q[c] = a[r + 4 * c] | (a[r + 4 * c + 1] << 8) | (a[r + 4 * c + 2] << 16) | (a[r + 4 * c + 3] << 24);
      ((v4u*)dst)[r / 16] = q;
    }
  }
}

// ------------------------------------------ batched count, column tables --
// A program of a pass owns one bit of each word of a row's accumulator (its
// single-column clauses that failed, and one word per clause spanning
// columns); a column ORs into it the entry of its value in its lookup table,
// so one lookup serves every program of the pass on that column.

// Truth of a literal (a leaf test, possibly negated) on a row: `nonnull`
// says whether the row's value is present, `inwin` whether x lies in the
// window of the column's value tests (outside it every value test is FALSE).
__device__ __forceinline__ bool lit_true(CInstr L, bool nonnull, bool inwin, int64_t x) {
  const bool neg = (L->flags & kLitNeg) != 0u;
  switch (L->op) {
    case D_NN_TRUE: return nonnull && !neg;
    case D_NN_FALSE: return nonnull && neg;
    case D_ISNULL: return nonnull ? neg : !neg;
    case D_NOTNULL: return nonnull ? !neg : neg;
    default: break;
  }
  if (!nonnull) return false;   // a value test on NULL is UNKNOWN, negated or not
  bool v = false;
  if (inwin) {
    const uint64_t d = (uint64_t)x - (uint64_t)L->lo;
    if (L->op == D_RANGE) {
      v = d <= L->span;
    } else if (L->op == D_BITMAP) {
      v = d < L->span && ((gptr<uint32_t>(L->aux)[d >> 5] >> (d & 31)) & 1u);
    } else {  // D_INLIST: lower bound in the sorted list
      const GLOBAL int64_t* list = gptr<int64_t>(L->aux);
      uint32_t base = 0, len = L->n;
      while (len > 1) {
        const uint32_t half = len >> 1;
        base = list[base + half] <= x ? base + half : base;
        len -= half;
      }
      v = list[base] == x;
    }
  }
  return v != neg;
}

// Lookup tables of a launch, in device memory.  A workgroup takes 64 entries
// of one column, an entry per lane, and its waves share the column's atoms,
// whose literals are then scalar loads; their bits meet in LDS.  (A thread per
// entry, one atom after another by vector loads, was a chain of some sixty
// memory latencies: 33 us before every batch of 64 programs, now 8.)
constexpr uint32_t kLutWaves = 8;
__global__ void __launch_bounds__(kLutWaves * 64) k_luts(LutArgs a) {
  __shared__ uint32_t out[4 * 64];
  const uint32_t lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  const CONSTANT LutBuild* builds = (const CONSTANT LutBuild*)a.builds;
  uint32_t lo = 0, hi = a.nbuilds;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (builds[mid].unit_begin <= blockIdx.x) lo = mid; else hi = mid;
  }
  const CONSTANT LutBuild* B = builds + uni(lo);
  const CONSTANT LutCol* C = (const CONSTANT LutCol*)a.cols + B->col;
  const uint32_t i = (blockIdx.x - (uint32_t)B->unit_begin) * kLutUnit + lane;
  const uint32_t kind = C->kind, n = C->n, ents = B->nentries;
  bool zero = i >= ents, nonnull = true, inwin = true;
  int64_t x = 0;
  if (kind == LK_DIRECT) {
    // 0: below the window, 1..n: values lo.., n+1: above, n+2: NULL, n+3: zero
    if (i == 0 || i == n + 1) inwin = false;
    else if (i == n + 2) nonnull = false;
    else if (i == n + 3) zero = true;
    else x = C->lo + (int64_t)(i - 1);
  } else if (kind == LK_RANK) {
    // 0..n: by rank, n+1: NULL, n+2: zero
    if (i == n + 1) nonnull = false;
    else if (i == n + 2) zero = true;
    else if (!zero) x = a.reps[B->reps + i];
  } else {  // LK_VALID: 0 non-NULL, 1 NULL
    nonnull = i == 0;
    inwin = false;
  }
  for (uint32_t k = threadIdx.x; k < 4 * 64; k += blockDim.x) out[k] = 0;
  __syncthreads();
  const CONSTANT LutAtom* atoms = (const CONSTANT LutAtom*)a.atoms + C->atom_begin;
  const uint32_t an = C->atom_count;
  for (uint32_t k = wave; k < an; k += kLutWaves) {
    const uint32_t lb = atoms[k].lit_begin, ln = atoms[k].lit_count, bit = atoms[k].bit;
    bool any = false;
    for (uint32_t l = 0; l < ln; ++l) any |= lit_true((CInstr)a.lits + lb + l, nonnull, inwin && !zero, x);
    if (!zero && any == (atoms[k].kind == LA_SAT)) atomicOr(&out[(bit >> 5) * 64 + lane], 1u << (bit & 31));
  }
  __syncthreads();
  const uint32_t D = B->dwords;
  for (uint32_t k = threadIdx.x; k < 64 * D; k += blockDim.x) {
    const uint32_t e = (blockIdx.x - (uint32_t)B->unit_begin) * kLutUnit + k / D;
    if (e < ents) B->dst[(uint64_t)e * D + k % D] = out[(k % D) * 64 + k / D];
  }
}

// A pass column in scalar registers, from one 64-byte scalar load.
struct ColD {
  const void* data;
  const uint32_t* valid;
  uint32_t type, kind;
  int64_t lo;
  uint32_t n, lds_word;
  const uint32_t* gtab;
  uint32_t first, guard;
};
__device__ __forceinline__ ColD decode_col(v16u w) {
  return ColD{(const void*)pair64(w, 0), (const uint32_t*)pair64(w, 2), w[4], w[5], (int64_t)pair64(w, 6),
              w[8], w[9], (const uint32_t*)pair64(w, 10), w[12], w[15]};
}

// One column's loads for S steps of the tile: per step one 16-byte load at the
// lane's first row, whatever the column's width, so that the registers do not
// depend on a branch (which would make the compiler wait for the loads in
// flight).  A narrow column reads its neighbours' rows too (the same cache
// lines); an int64 column's rows 2 and 3 of each step are four more loads.
// Bounded to the table's rows: past them the loads return zero without
// touching memory.
template <int S, bool WIDE>
struct Stage {
  v4i w[WIDE ? 2 * S : S];
  uint32_t vr[WIDE ? S : 1];   // validity words of the lane's rows
};

template <int S, bool WIDE>
__device__ __forceinline__ void lut_issue(Stage<S, WIDE>& g, const ColD& c, uint64_t tb, uint64_t nrows, uint32_t lane, int j0,
                                          bool on = true) {
  const uint32_t width = c.type == T_I8 ? 1u : c.type == T_I16 ? 2u : c.type == T_I32 ? 4u : 8u;
  const __amdgpu_buffer_rsrc_t rs = col_rsrc(c.data, width, tb, nrows, on ? (uint32_t)kTileRows : 0u);
  const uint32_t at = width * (4u * lane + 256u * (uint32_t)j0), step = width * 256u;
#pragma unroll
  for (int s = 0; s < S; ++s) g.w[s] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + step * (uint32_t)s), 0, kNt);
  if (WIDE && c.type == T_I64) {
#pragma unroll
    for (int s = 0; s < S; ++s)
      g.w[(WIDE ? S : 0) + s] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + 16u + step * (uint32_t)s), 0, kNt);
  }
  if (WIDE && c.valid) {
    const uint32_t rows = nrows - tb < (uint64_t)kTileRows ? (uint32_t)(nrows - tb) : (uint32_t)kTileRows;
    const __amdgpu_buffer_rsrc_t vs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(c.valid + tb / 32), (short)0, (int)uni((rows + 31u) / 32u * 4u), 0x00020000);
#pragma unroll
    for (int s = 0; s < S; ++s)
      g.vr[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(vs, (int)(4u * ((lane >> 3) + 8u * (uint32_t)(j0 + s))), 0, 0);
  }
}

// value of row r (step r / 4) of a stage
template <int TY, int S, bool WIDE>
__device__ __forceinline__ auto sget(const Stage<S, WIDE>& g, int r) {
  const int s = r >> 2, i = r & 3;
  if constexpr (TY == T_I8) {
    return (int32_t)(int8_t)((uint32_t)g.w[s][0] >> (8 * i));
  } else if constexpr (TY == T_I16) {
    return (int32_t)(int16_t)((uint32_t)g.w[s][i >> 1] >> (16 * (i & 1)));
  } else if constexpr (TY == T_I32) {
    return (int32_t)g.w[s][i];
  } else {
    const v4i& q = g.w[S * (i >> 1) + s];
    const int k = 2 * (i & 1);
    return (int64_t)(((uint64_t)(uint32_t)q[k + 1] << 32) | (uint32_t)q[k]);
  }
}

// Validity of R rows of the lane from step j0: bit b = row b is not NULL (0
// past the table).
template <int R>
__device__ __forceinline__ uint32_t lseg_valid(const uint32_t* valid, uint64_t tb, int j0, uint32_t lane,
                                               uint64_t nrows, bool full) {
  constexpr int S = R / 4;
  const GLOBAL uint32_t* vw = gptr<uint32_t>(valid) + tb / 32 + (lane >> 3) + 8 * j0;
  const uint32_t sh = 4 * (lane & 7);
  uint32_t V = 0;
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (full || tb + 256u * (uint32_t)(j0 + s) + 4u * lane < nrows) V |= ((vw[8 * s] >> sh) & 0xFu) << (4 * s);
  return V;
}

#define LDS_PTR(T) __attribute__((address_space(3))) T*

// The entry at LDS byte address e ORed into the accumulators.
template <int D>
__device__ __forceinline__ void ent_or_lds(LDS_PTR(const char) e, uint32_t (&acc)[D]) {
  if constexpr (D == 1) {
    acc[0] |= *(LDS_PTR(const uint32_t))e;
  } else if constexpr (D == 2) {
    const v2u x = *(LDS_PTR(const v2u))e;
    acc[0] |= x[0];
    acc[1] |= x[1];
  } else {
    const v4u x = *(LDS_PTR(const v4u))e;
#pragma unroll
    for (int d = 0; d < 4; ++d) acc[d] |= x[d];
  }
}

// Entry idx of a device-memory table through a buffer resource: a 32-bit
// offset per lane instead of a 64-bit address, and an offset past the
// table reads zero.
template <int D>
__device__ __forceinline__ void gent_or(__amdgpu_buffer_rsrc_t tab, uint32_t idx, uint32_t (&acc)[D]) {
  if constexpr (D == 1) {
    acc[0] |= __builtin_amdgcn_raw_buffer_load_b32(tab, (int)(idx * 4u), 0, 0);
  } else if constexpr (D == 2) {
    const v2u e = __builtin_amdgcn_raw_buffer_load_b64(tab, (int)(idx * 8u), 0, 0);
    acc[0] |= e[0];
    acc[1] |= e[1];
  } else {
    const v4u e = __builtin_amdgcn_raw_buffer_load_b128(tab, (int)(idx * 16u), 0, 0);
#pragma unroll
    for (int d = 0; d < 4; ++d) acc[d] |= e[d];
  }
}

// Buffer resource of a device table of `entries` D-dword entries (gfx9
// raw buffer: stride 0, bounds checked against the byte size).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t table_rsrc(const uint32_t* tab, uint32_t entries, uint32_t dwords) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)tab, (short)0, (int)(entries * dwords * 4u), 0x00020000);
}

// Table indices of eight rows to entries, ORed into the accumulators of rows
// off .. off + 7: from LDS, or from device memory where a guarded table is
// read only on rows some program of the pass can still count (the others read
// the zero entry).
template <int D, int R>
__device__ __forceinline__ void lookup_or(const ColD& c, const uint32_t* lds, uint32_t (&idx)[8], uint32_t zero,
                                          const CONSTANT LutPass* P, uint32_t (&acc)[R][D], int off) {
  if (c.lds_word != kNoLds) {
    const LDS_PTR(char) l3 = (LDS_PTR(char))lds;
#pragma unroll
    for (int r = 0; r < 8; ++r)
      ent_or_lds<D>((LDS_PTR(const char))(l3 + (c.lds_word * 4u + idx[r] * (4u * D))), acc[off + r]);
  } else {
    const __amdgpu_buffer_rsrc_t tab = table_rsrc(c.gtab, zero + 1, D);
    if (c.guard) {
      // a row some program can still count: a failure bit (word 0 of a
      // dword) still clear
      uint32_t am[D];
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const uint32_t g = (P->fold[d] >> 8) & 0xFFu;
        am[d] = g >= 32 ? ~0u : (1u << g) - 1u;
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        uint32_t alive = 0;
#pragma unroll
        for (int d = 0; d < D; ++d) alive |= ~acc[off + r][d] & am[d];
        idx[r] = alive ? idx[r] : zero;
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) gent_or<D>(tab, idx[r], acc[off + r]);
  }
}

// One column on the segment's rows of the lane: every row's
// entry ORed into its accumulator.
// Eight rows at a time (a scheduling barrier between them): more entries in
// flight would spill the accumulators.
template <int D, int R, int TY, bool WIDE>
__device__ __forceinline__ void lut_col(const Stage<R / 4, WIDE>& raw, const ColD& c, const LutArgs& a, uint32_t lane, const uint32_t* lds,
                                        const CONSTANT LutPass* P, uint32_t (&acc)[R][D]) {
  const uint32_t n = c.n;
  const int64_t lo = c.lo;
  const bool nullable = WIDE && c.valid != nullptr;
  uint32_t V = 0;   // the rows' validity
  if (nullable) {
#pragma unroll
    for (int s = 0; s < R / 4; ++s) V |= ((raw.vr[WIDE ? s : 0] >> (4u * (lane & 7u))) & 0xFu) << (4 * s);
  }
  if (c.kind == LK_DIRECT) {
    constexpr int64_t tmin = TY == T_I8 ? INT8_MIN : TY == T_I16 ? INT16_MIN : INT32_MIN;
    constexpr int64_t tmax = TY == T_I8 ? INT8_MAX : TY == T_I16 ? INT16_MAX : INT32_MAX;
    const int32_t cl = (int32_t)(lo - 1 < tmin ? tmin : lo - 1);
    const int32_t ch = (int32_t)(lo + (int64_t)n > tmax ? tmax : lo + (int64_t)n);
    if constexpr (TY != T_I64) {
      if (c.lds_word != kNoLds && !nullable) {
        // clamped value straight to the entry's LDS byte address: the
        // table's address less (lo - 1) entries, plus the value's entries
        const LDS_PTR(char) l3 = (LDS_PTR(char))lds;
        const uint32_t abase = c.lds_word * 4u - (uint32_t)(lo - 1) * (4u * D);
        int32_t chv = ch;   // in a vector register once: one scalar operand per VALU op
        asm volatile("v_mov_b32 %0, %1" : "=v"(chv) : "s"(ch));
#pragma unroll
        for (int g = 0; g < R; g += 8) {
#pragma unroll
          for (int r = g; r < g + 8; ++r) {
            const int32_t x = sget<TY>(raw, r);
            int32_t m;
            asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(x), "s"(cl), "v"(chv));
            ent_or_lds<D>((LDS_PTR(const char))(l3 + (abase + (uint32_t)m * (4u * D))), acc[r]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        return;
      }
    }
#pragma unroll
    for (int g = 0; g < R; g += 8) {
      uint32_t idx[8];
      if constexpr (TY != T_I64) {
        // clamp to [lo - 1, lo + n] (inside the type), then offset: entry 0
        // below the window, n + 1 above it
        const uint32_t base = (uint32_t)(lo - 1);
#pragma unroll
        for (int r = 0; r < 8; ++r) idx[r] = (uint32_t)min(max((int32_t)sget<TY>(raw, g + r), cl), ch) - base;
      } else {
        const int64_t cl8 = lo == INT64_MIN ? lo : lo - 1;
        const int64_t ch8 = lo + (int64_t)n;   // the planned window ends below INT64_MAX
        const uint64_t base = (uint64_t)lo - 1u;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const int64_t x = sget<TY>(raw, g + r);
          const int64_t m = x < cl8 ? cl8 : x > ch8 ? ch8 : x;
          idx[r] = (uint32_t)((uint64_t)m - base);
        }
      }
      if (nullable) {
#pragma unroll
        for (int r = 0; r < 8; ++r) idx[r] = (V >> (g + r)) & 1u ? idx[r] : n + 2;
      }
      lookup_or<D, R>(c, lds, idx, n + 3, P, acc, g);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {  // LK_RANK: the number of bounds at or below the value
    // bounds in blocks of eight (the list is padded to whole blocks), one
    // scalar load per block
    const CONSTANT int64_t* b = (const CONSTANT int64_t*)a.bounds + c.first;
    uint32_t idx[R / 8][8] = {};
    for (uint32_t k0 = 0; k0 < n; k0 += 8) {
      int64_t bb[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) bb[j] = b[k0 + j];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (k0 + j >= n) break;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (TY != T_I64) idx[r >> 3][r & 7] += (int32_t)sget<TY>(raw, r) >= (int32_t)bb[j] ? 1u : 0u;
          else idx[r >> 3][r & 7] += sget<TY>(raw, r) >= bb[j] ? 1u : 0u;
        }
      }
    }
#pragma unroll
    for (int g = 0; g < R / 8; ++g) {
      if (nullable) {
#pragma unroll
        for (int r = 0; r < 8; ++r) idx[g][r] = (V >> (8 * g + r)) & 1u ? idx[g][r] : n + 1;
      }
      lookup_or<D, R>(c, lds, idx[g], n + 2, P, acc, 8 * g);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Per-lane carry-save counters of T bits: planes of weight 1, 2, 4, 8 and
// a vertical counter of weight 16 * 2^k (at most 2047 per bit position
// between reads).
constexpr int kHsLevels = 7;
struct Hs {
  uint32_t ones, twos, fours, eights;
  uint32_t h[kHsLevels];
};

__device__ __forceinline__ void csa(uint32_t& carry, uint32_t& sum, uint32_t a, uint32_t b, uint32_t c) {
  const uint32_t u = a ^ b;
  carry = (u & c) | (~u & a);   // one bit-field insert
  sum = u ^ c;
}

__device__ __forceinline__ void hs_sixteens(Hs& s, uint32_t c) {
#pragma unroll
  for (int k = 0; k < kHsLevels; ++k) {
    const uint32_t t = s.h[k] & c;
    s.h[k] ^= c;
    c = t;
  }
}

// Add NW words (NW = 2, 4 or a multiple of 8), each bit position counting 0 or 1.
template <int NW>
__device__ __forceinline__ void hs_add(Hs& s, const uint32_t* w) {
  if constexpr (NW > 8) {
    static_assert(NW % 8 == 0, "blocks of eight words");
#pragma unroll
    for (int k = 0; k < NW; k += 8) hs_add<8>(s, w + k);
  } else if constexpr (NW == 8) {
    uint32_t ta, tb, fa, fb, e;
    csa(ta, s.ones, s.ones, w[0], w[1]);
    csa(tb, s.ones, s.ones, w[2], w[3]);
    csa(fa, s.twos, s.twos, ta, tb);
    csa(ta, s.ones, s.ones, w[4], w[5]);
    csa(tb, s.ones, s.ones, w[6], w[7]);
    csa(fb, s.twos, s.twos, ta, tb);
    csa(e, s.fours, s.fours, fa, fb);
    const uint32_t c = s.eights & e;
    s.eights ^= e;
    hs_sixteens(s, c);
  } else if constexpr (NW == 4) {
    uint32_t ta, tb, f;
    csa(ta, s.ones, s.ones, w[0], w[1]);
    csa(tb, s.ones, s.ones, w[2], w[3]);
    csa(f, s.twos, s.twos, ta, tb);
    const uint32_t e = s.fours & f;
    s.fours ^= f;
    const uint32_t c = s.eights & e;
    s.eights ^= e;
    hs_sixteens(s, c);
  } else {
    static_assert(NW == 2, "two, four or a multiple of eight words");
    uint32_t t;
    csa(t, s.ones, s.ones, w[0], w[1]);
    const uint32_t f = s.twos & t;
    s.twos ^= t;
    const uint32_t e = s.fours & f;
    s.fours ^= f;
    const uint32_t c = s.eights & e;
    s.eights ^= e;
    hs_sixteens(s, c);
  }
}

// Rows' accumulators to their T words (bit p: program p counts the row), eight
// rows at a time, packed 32 / B rows to a word, into the counters.  Within
// dword d, word 0 is inverted and the b_d-bit words are ANDed together by
// folding.
template <int D, int R>
__device__ __forceinline__ void lut_count(uint32_t (&acc)[R][D], const CONSTANT LutPass* P, uint32_t inr,
                                          Hs& hs) {
  const uint32_t B = P->bits;
  uint32_t nm[D], gm[D], ps[D], bw[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const uint32_t f = P->fold[d];
    bw[d] = f & 0xFFu;
    const uint32_t g = (f >> 8) & 0xFFu;
    ps[d] = f >> 16;
    nm[d] = bw[d] >= 32 ? ~0u : (1u << bw[d]) - 1u;
    gm[d] = g >= 32 ? ~0u : (1u << g) - 1u;
  }
  // each dword folded in place; its width is a uniform branch around all rows
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (bw[d] >= 32) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r][d] = ~acc[r][d];
    } else if (bw[d] == 16) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r][d] = (acc[r][d] >> 16) & ~acc[r][d];
    } else if (bw[d] == 8) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        uint32_t t = acc[r][d] ^ nm[d];
        t &= t >> 16;
        acc[r][d] = t & (t >> 8);
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        uint32_t t = acc[r][d] ^ nm[d];
        t &= t >> 16;
        t &= t >> 8;
        acc[r][d] = t & (t >> 4);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    acc[r][0] = (acc[r][0] & gm[0]) << ps[0];
#pragma unroll
    for (int d = 1; d < D; ++d) acc[r][0] |= (acc[r][d] & gm[d]) << ps[d];
  }
  if (inr != ~0u) {
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r][0] = (inr >> r) & 1u ? acc[r][0] : 0u;
  }
  if (B == 32) {
#pragma unroll
    for (int g = 0; g < R; g += 8) {
      uint32_t w[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) w[k] = acc[g + k][0];
      hs_add<8>(hs, w);
    }
  } else if (B == 16) {
    uint32_t w[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) w[k] = acc[2 * k][0] | (acc[2 * k + 1][0] << 16);
    hs_add<R / 2>(hs, w);
  } else {
    uint32_t w[R / 4];
#pragma unroll
    for (int k = 0; k < R / 4; ++k)
      w[k] = acc[4 * k][0] | (acc[4 * k + 1][0] << 8) | (acc[4 * k + 2][0] << 16) | (acc[4 * k + 3][0] << 24);
    hs_add<R / 4>(hs, w);
  }
}

// Reads the counters out (wave-wide bit counts per position), adds each
// program's count to its LDS counter or accumulator line, and clears them.
// Program p's rows are counted at bit positions p, p + B, ... of the words.
__device__ __forceinline__ void hs_flush(Hs& s, const CONSTANT LutPass* P, unsigned long long* gacc,
                         const uint32_t* acc_index, uint32_t* accl, uint32_t nacc, uint32_t lane) {
  uint32_t planes[4 + kHsLevels] = {s.ones, s.twos, s.fours, s.eights};
#pragma unroll
  for (int k = 0; k < kHsLevels; ++k) planes[4 + k] = s.h[k];
  uint32_t used = 0;   // planes with a bit set in some lane
#pragma unroll
  for (int k = 0; k < 4 + kHsLevels; ++k) used |= (__ballot(planes[k] != 0u) != 0ull ? 1u : 0u) << k;
  const uint32_t B = P->bits, pb = P->prog_begin, pn = P->prog_count;
  for (uint32_t p = 0; p < pn; ++p) {
    uint32_t c = 0;
    for (uint32_t q = p; q < 32; q += B) {
#pragma unroll
      for (int k = 0; k < 4 + kHsLevels; ++k)
        if ((used >> k) & 1u) c += (uint32_t)__popcll(__ballot((planes[k] >> q) & 1u)) << k;
    }
    if (lane == 0 && c) {
      if (pb + p < nacc) atomicAdd(&accl[pb + p], c);
      else atomicAdd(&gacc[(uint64_t)acc_index[pb + p] * kBatchAccStride], (unsigned long long)c);
    }
  }
  s = Hs{};
}

// Every column of a pass on one tile, R rows of the lane at a time (half of
// the tile, or a quarter): the loads of a column and, if it is narrow and has
// no NULLs, of the one after it, then every row's lookups.  The rows'
// accumulators stay in registers, and a column's description is read once for
// all of them.  With every column of eight rows loaded together, the
// descriptions of eight columns did not fit the scalar registers: a third of
// the vector instructions moved them to vector lanes and back (124 a row, now
// 79), and 64 programs over four tables took 1.87 ms, now 1.38
// (5.8 TB/s; the kernel alone 1.81, now 1.33).  Vector issue
// and memory latency share the time: one column at a time took 1.57 ms, three
// 1.51 (spills), whole tiles (32 rows a lane) 2.1 (spills), the next column
// loaded or touched ahead 1.7 to 2.4.  The second column's loads are issued
// whether or not there is one (with no bytes in bounds), so that the compiler
// knows how many are in flight and waits for the first column's alone.  Rows
// past the table read zeros and are not counted.
template <int D, int R>
__device__ __forceinline__ void lut_tile(const CONSTANT LutPass* P, const CONSTANT LutCol* cols,
                                         const LutArgs& a, uint64_t tb, uint32_t lane,
                                         const uint32_t* lds, Hs& hs) {
  static_assert(R == 8 || R == 16, "a quarter tile or half of one");
  constexpr int S = R / 4;
  const uint64_t nrows = P->nrows;
  const bool full = tb + kTileRows <= nrows;
  const CONSTANT LutCol* cb = cols + P->col_begin;
  const uint32_t nd = P->ndata, cn = P->col_count;
  uint32_t acc[R][D];
  auto start = [&](int j0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const uint32_t v = P->init[d];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r][d] = v;
    }
    // columns that only null tests read (no data) come last in the pass
    for (uint32_t c = nd; c < cn; ++c) {
      const CONSTANT LutCol* C = cb + c;
      const uint32_t V = lseg_valid<R>(C->valid, tb, j0, lane, nrows, full);
      const CONSTANT uint32_t* e = (const CONSTANT uint32_t*)C->gtab;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const uint32_t e0 = e[d], e1 = e[D + d];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r][d] |= (V >> r) & 1u ? e0 : e1;
      }
    }
  };
  auto count = [&](int j0) {
    lut_count<D, R>(acc, P, full ? ~0u : inrange_bits<kSteps>(tb, lane, nrows) >> (4 * j0), hs);
  };
  auto use = [&](auto& g, const ColD& c) {
    constexpr bool WIDE = sizeof g.w / sizeof g.w[0] == 2 * S;
    if (WIDE && c.type == T_I64) {
      if constexpr (WIDE) lut_col<D, R, T_I64, WIDE>(g, c, a, lane, lds, P, acc);
    } else if (c.type == T_I32) {
      lut_col<D, R, T_I32, WIDE>(g, c, a, lane, lds, P, acc);
    } else if (c.type == T_I8) {
      lut_col<D, R, T_I8, WIDE>(g, c, a, lane, lds, P, acc);
    } else {
      lut_col<D, R, T_I16, WIDE>(g, c, a, lane, lds, P, acc);
    }
  };
  for (int j0 = 0; j0 < kSteps; j0 += S) {
    start(j0);
    for (uint32_t c = 0; c < nd;) {
      const ColD ca = decode_col(*(const CONSTANT v16u*)(cb + c));
      const ColD cc = decode_col(*(const CONSTANT v16u*)(cb + min(c + 1, nd - 1)));
      const bool two = c + 1 < nd && cc.type != T_I64 && !cc.valid;
      Stage<S, true> A;
      Stage<S, false> B;
      lut_issue<S, true>(A, ca, tb, nrows, lane, j0);
      lut_issue<S, false>(B, cc, tb, nrows, lane, j0, two);
      use(A, ca);
      if (two) use(B, cc);
      c += two ? 2 : 1;
    }
    count(j0);
  }
}

// Per workgroup, per-program counts accumulate in LDS and go to the
// accumulator lines at the end, as in k_batch; the last workgroup by ticket
// moves the finished lines out.  The workgroup takes groups of nw tiles
// (pass ranges are padded to kLutTileAlign), and copies a pass's LDS tables
// from device memory when it moves to that pass.
// Workgroup of the lookup-table kernel (one per CU, whose LDS it takes):
// twelve waves, three per SIMD (168 vector registers each); sixteen waves of
// eight rows a lane (the tuner's other choice) fit 128 registers where the
// rows have one or two accumulator dwords (1.44 ms for the 64 programs,
// against 1.38).
constexpr uint32_t lbatch_threads(uint32_t dwords, uint32_t rows) { return rows == 8 && dwords < 4 ? 1024u : 768u; }

template <int D, int R>
__global__ void __launch_bounds__((lbatch_threads(D, R))) k_lbatch(LutArgs a) {
  extern __shared__ __align__(16) uint32_t dyn[];
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t nw = blockDim.x >> 6;
  const uint32_t nacc = a.acc_words;
  uint32_t* accl = dyn;
  uint32_t* lds = dyn + nacc;
  for (uint32_t p = threadIdx.x; p < nacc; p += blockDim.x) accl[p] = 0;
  __syncthreads();
  const CONSTANT LutPass* passes = (const CONSTANT LutPass*)a.passes;
  const CONSTANT LutCol* cols = (const CONSTANT LutCol*)a.cols;
  const uint64_t ngroups = a.total_tiles / nw;
  uint32_t staged = 0xFFFFFFFFu;
  const CONSTANT LutPass* P = nullptr;
  Hs hs{};
  uint32_t since = 0;
  for (uint64_t g = blockIdx.x; g < ngroups; g += gridDim.x) {
    const uint64_t flat = g * nw + wave;
    uint32_t lo = 0, hi = a.npasses;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (passes[mid].tile_begin <= flat) lo = mid; else hi = mid;
    }
    lo = uni(lo);
    if (passes[lo].dwords != (uint32_t)D) continue;   // another launch's pass
    if (lo != staged) {
      if (P) {
        hs_flush(hs, P, a.acc, a.acc_index, accl, nacc, lane);
        since = 0;
      }
      P = passes + lo;
      __syncthreads();
      for (uint32_t c = 0; c < P->col_count; ++c) {
        const CONSTANT LutCol* C = cols + P->col_begin + c;
        if (C->lds_word == kNoLds) continue;
        const uint32_t entries = C->kind == LK_DIRECT ? C->n + 4 : C->n + 3;
        const uint32_t words = entries * P->dwords;
        const GLOBAL uint32_t* src = gptr<uint32_t>(C->gtab);
        uint32_t* dst = lds + C->lds_word;
        for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) dst[i] = src[i];
      }
      __syncthreads();
      staged = lo;
    }
    const uint64_t local = flat - P->tile_begin;
    if (local >= P->ntiles) continue;   // padding
    // the wave's tile start is wave-uniform: say so, so that the buffer
    // resources built from it stay in scalar registers
    const uint64_t tb = uni64(P->row_begin + local * kTileRows);
    lut_tile<D, R>(P, cols, a, tb, lane, lds, hs);
    if (++since == kLutFlushTiles) {
      hs_flush(hs, P, a.acc, a.acc_index, accl, nacc, lane);
      since = 0;
    }
  }
  if (P) hs_flush(hs, P, a.acc, a.acc_index, accl, nacc, lane);
  __syncthreads();
  for (uint32_t p = threadIdx.x; p < nacc && p < a.nprogs; p += blockDim.x)
    if (accl[p]) atomicAdd(&a.acc[(uint64_t)a.acc_index[p] * kBatchAccStride], (unsigned long long)accl[p]);
  atomics_done();
  __syncthreads();
  __shared__ bool last;
  if (threadIdx.x == 0) {
    const unsigned int ticket = atomicAdd(&a.slot->ticket, 1u);
    last = ticket == gridDim.x - 1;
  }
  __syncthreads();
  if (last) {
    for (uint32_t k = threadIdx.x; k < a.ndone; k += blockDim.x) {
      const uint64_t line = a.done ? a.done[k] : k;
      put_host(&a.out[k], atomicExch(&a.acc[line * kBatchAccStride], 0ull));
    }
    atomics_done();
    __syncthreads();
    if (threadIdx.x == 0) atomicExch(&a.slot->ticket, 0u);
  }
}

__global__ void k_fill(uint32_t* __restrict__ p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

}  // namespace

// Workspace of sel_pushdown_rowids_noalloc: a fixed array in each device's
// copy of the code object, for callers that cannot allocate device memory.
// In host code `scratch` names a host-side stand-in, not a device address;
// kernels receive the address that sel_noalloc_scratch looked up for the
// current device.
static __device__ __align__(256) uint8_t scratch[sel::kNoAllocScratchBytes];

int sel_noalloc_scratch(int device, void** ptr) {
  static std::mutex mu;
  static std::map<int, void*> addr;  // device -> address of its array
  std::lock_guard<std::mutex> lock(mu);
  auto it = addr.find(device);
  if (it == addr.end()) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (p == nullptr) return (int)hipErrorInvalidSymbol;
    it = addr.emplace(device, p).first;
  }
  *ptr = it->second;
  return 0;
}

int sel_launch_scan(int mode, const ScanArgs& a, uint32_t grid, uint32_t block, void* stream) {
  if (grid >= kSlotMaxGrid) return (int)hipErrorInvalidValue;
  hipStream_t s = (hipStream_t)stream;
  const uint32_t lds = a.nstage ? 4u * a.stage_words : 0u;
  const bool nt = !a.cached;
  if (a.small && block != 256) return (int)hipErrorInvalidValue;
#define SCAN(...) hipLaunchKernelGGL((k_scan<__VA_ARGS__>), dim3(grid), dim3(block), lds, s, a.prog, a)
  switch (mode) {
    case M_COUNT:
      if (a.small) SCAN(M_COUNT, false, kSmallSteps);
      else if (nt) SCAN(M_COUNT, true, kSteps);
      else SCAN(M_COUNT, false, kSteps);
      break;
    case M_MASK:
      if (a.small) SCAN(M_MASK, false, kSmallSteps);
      else if (nt) SCAN(M_MASK, true, kSteps);
      else SCAN(M_MASK, false, kSteps);
      break;
    default:
      if (a.small) SCAN(M_KEYBITMAP, false, kSmallSteps);
      else SCAN(M_KEYBITMAP, true, kSteps);
      break;
  }
#undef SCAN
  return (int)hipGetLastError();
}

int sel_launch_scan_tiles(const MaskOrder& order, const uint32_t* tile_meta, uint32_t* offsets, uint32_t* chunk_sums,
                          uint32_t ntiles, void* stream) {
  const uint32_t nchunks = (ntiles + 1023) / 1024;
  if (nchunks == 0) return 0;
  if (nchunks > 2048) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_chunk_scan, dim3(nchunks), dim3(1024), 0, (hipStream_t)stream, order, tile_meta, offsets,
                     chunk_sums, ntiles);
  return (int)hipGetLastError();
}

int sel_launch_compact(const CompactArgs& a, void* stream) {
  if (a.tiles_per_wave != 1 && a.tiles_per_wave != 4) return (int)hipErrorInvalidValue;
  const uint32_t per_group = 4 * a.tiles_per_wave;
  const uint32_t grid = a.ntiles ? (a.ntiles + per_group - 1) / per_group : 1u;
  hipLaunchKernelGGL(k_compact, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int sel_launch_gather(const GatherArgs& a, uint32_t grid, uint32_t block, void* stream) {
  if (grid >= kSlotMaxGrid) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gather, dim3(grid), dim3(block), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int sel_launch_tables(const TableBuild* d_builds, uint32_t nbuilds, uint64_t nunits, void* stream) {
  if (nbuilds == 0 || nunits == 0) return 0;
  const uint64_t blocks = (nunits + 3) / 4;
  if (blocks >= 1ull << 31) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_tables, dim3((uint32_t)blocks), dim3(256), 0, (hipStream_t)stream, d_builds, nbuilds, nunits);
  return (int)hipGetLastError();
}

int sel_launch_fill(uint32_t* p, uint64_t nwords, uint32_t value, void* stream) {
  if (nwords == 0) return 0;
  uint64_t blocks = (nwords + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill, dim3((uint32_t)blocks), dim3(256), 0, (hipStream_t)stream, p, nwords, value);
  return (int)hipGetLastError();
}

int sel_scan_occupancy(int mode, uint32_t block, int* blocks_per_cu) {
  const void* k = mode == M_COUNT  ? (const void*)k_scan<M_COUNT, true, kSteps>
                  : mode == M_MASK ? (const void*)k_scan<M_MASK, true, kSteps>
                                   : (const void*)k_scan<M_KEYBITMAP, true, kSteps>;
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, block, 0);
}

int sel_launch_batch(const BatchArgs& a, uint32_t grid, uint32_t block, uint32_t lds_bytes,
                     void* stream) {
  hipLaunchKernelGGL(k_batch, dim3(grid), dim3(block), lds_bytes, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int sel_batch_occupancy(uint32_t block, uint32_t lds_bytes, int* blocks_per_cu) {
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_batch, block, lds_bytes);
}

int sel_launch_luts(const LutArgs& a, void* stream) {
  if (a.nbuilds == 0 || a.nunits == 0) return 0;
  if (a.nunits >= 1ull << 31) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL(k_luts, dim3((uint32_t)a.nunits), dim3(kLutWaves * 64), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

// The lookup-table kernel for passes of `dwords` accumulator dwords per row.
// `rows` is the launch configuration's: 8 for sixteen rows per lane at a time,
// 4 for eight.
namespace {
const void* lbatch_kernel(uint32_t dwords, uint32_t rows) {
  switch (dwords) {
    case 1: return rows == 4 ? (const void*)k_lbatch<1, 8> : (const void*)k_lbatch<1, 16>;
    case 2: return rows == 4 ? (const void*)k_lbatch<2, 8> : (const void*)k_lbatch<2, 16>;
    default: return (const void*)k_lbatch<4, 8>;   // sixteen rows' accumulators would not fit
  }
}
}  // namespace

int sel_launch_lbatch(const LutArgs& a, uint32_t dwords, uint32_t rows, uint32_t grid, uint32_t block,
                      uint32_t lds_bytes, void* stream) {
  if (block == 0 || block > sel_lbatch_block(dwords, rows) || block % kWave) return (int)hipErrorInvalidValue;
  LutArgs args = a;
  void* kargs[] = {&args};
  return (int)hipLaunchKernel(lbatch_kernel(dwords, rows), dim3(grid), dim3(block), kargs, lds_bytes,
                              (hipStream_t)stream);
}

uint32_t sel_lbatch_block(uint32_t dwords, uint32_t rows) { return lbatch_threads(dwords, rows == 4 || dwords == 4 ? 8 : 16); }

int sel_lbatch_occupancy(uint32_t dwords, uint32_t rows, uint32_t block, uint32_t lds_bytes, int* blocks_per_cu) {
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, lbatch_kernel(dwords, rows), block,
                                                           lds_bytes);
}
