// Narrow products (N <= 8192) on gfx950, with presence bitmaps of B's rows.
//
// A dense enough B row is cheaper to read as N bits than as a list of
// columns, and the union of B rows is then an OR of registers:
//   k_narrow_prepare   per row of B: its bitmap and a slot of fixed size with
//                    its entries (once per call)
//   k_narrow_symbolic  per row of the tile: C_i's bitmap (the OR), nnz(C_i)
//                    and P_i (popcounts), in place of the analysis and of the
//                    symbolic phase
//   k_narrow_rows    numeric, a wavefront per row: S lanes take one B row, the
//                    64 / S lane groups different ones, each group adding
//                    into a dense LDS row of its own by plain reads and
//                    writes (the columns of a B row are distinct, and a
//                    wavefront's LDS operations complete in order); C_i's
//                    bitmap gives the output positions
//   k_narrow_block   numeric, heavier rows: a workgroup per row, or per part
//                    of a row that adds into a dense slot in global memory
#include "device.h"
#include "kernels.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace aires {
namespace kern {
namespace {

// the value of lane i
__device__ __forceinline__ int64_t lane_i64(int64_t v, int i) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, i);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), i);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// -------------------------------------------------- B's bitmaps and slots

// A slot holds a B row's first cap entries: cap values, then cap 16-bit
// column words, padded to whole 64-byte blocks.  A column word is the byte
// offset of the column's sums in a wavefront's dense rows (64 / lanes floats a
// column, below GOES_ON), so that the add loop uses it as it is; unused
// entries point behind the last column (and hold the value 0).  Its top bit
// says that the row goes on after the entry.
constexpr uint32_t GOES_ON = 0x8000u;

__host__ __device__ constexpr int padded_cols(int64_t N) { return (int)((N + 63) / 64 * 64); }

constexpr int64_t PREPARE_LONG = 256;  // entries of a row of B

// One pass over B writes both.  16 lanes per row; bitmaps and slots of the
// workgroup's rows are put together in LDS and go out as whole lines.
template <typename RB>
__global__ __launch_bounds__(256) void k_narrow_prepare(const void* brp, const int32_t* bcol, const float* bval,
                                                        int64_t K, int64_t N, const NarrowView nv, int rows) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int words = nv.words, cap = nv.cap, slot = nv.slot;
  const uint32_t col_bytes = slot ? 4u * (WAVE / nv.lanes) : 0u;
  const uint32_t no_col = (uint32_t)padded_cols(N) * col_bytes;
  uint32_t* bm = reinterpret_cast<uint32_t*>(smem);
  unsigned char* sl = smem + (size_t)rows * words * 4;
  const int sub = threadIdx.x & 15, sg = threadIdx.x >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * rows;
  const int nr = (int)(K - r0 < rows ? K - r0 : rows);
  for (int i = threadIdx.x; i < rows * words; i += 256) bm[i] = 0u;
  __syncthreads();
  // entries from q on, `step` apart, of row r: [s, s + len) of B's arrays
  auto put_row = [&](int r, int64_t s, int64_t len, int64_t q, int step) {
    float* sv = reinterpret_cast<float*>(sl + (size_t)r * slot);
    uint16_t* sc = reinterpret_cast<uint16_t*>(sv + cap);
    for (; q < len || q < cap; q += step) {
      uint32_t c = no_col;
      float v = 0.f;
      if (q < len) {
        const int j = bcol[s + q];
        atomicOr(&bm[r * words + (j >> 5)], 1u << (j & 31));
        c = (uint32_t)j * col_bytes | (q + 1 < len ? GOES_ON : 0u);
        if (q < cap) v = bval[s + q];
      }
      if (q < cap) {
        sv[q] = v;
        sc[q] = (uint16_t)c;
      }
    }
  };
  for (int rb = 0; rb < nr; rb += 16) {
    const int r = rb + sg;
    int64_t s = 0, len = -1;
    if (r < nr) {
      s = ld_rp<RB>(brp, r0 + r);
      len = ld_rp<RB>(brp, r0 + r + 1) - s;
    }
    const bool is_long = len > PREPARE_LONG;
    if (r < nr && !is_long) put_row(r, s, len, sub, 16);
    // long rows by the whole wavefront (30 K rows, 60 of them of 8000 entries: 147
    // us with 16 lanes to each)
    for (uint64_t todo = __ballot(is_long && sub == 0); todo; todo &= todo - 1u) {
      const int l = __builtin_ctzll(todo);
      put_row(__builtin_amdgcn_readlane(r, l), lane_i64(s, l), lane_i64(len, l), lane_id(), WAVE);
    }
  }
  __syncthreads();
  const uint4* src = reinterpret_cast<const uint4*>(bm);
  uint4* dst = reinterpret_cast<uint4*>(const_cast<uint32_t*>(nv.bbm) + r0 * words);
  for (int i = threadIdx.x; i < nr * (words / 4); i += 256) dst[i] = src[i];
  if (slot) {
    src = reinterpret_cast<const uint4*>(sl);
    dst = reinterpret_cast<uint4*>(const_cast<unsigned char*>(nv.slots) + r0 * slot);
    for (int i = threadIdx.x; i < nr * (slot / 16); i += 256) dst[i] = src[i];
  }
}

// ---------------------------------------------------------------- symbolic

// Lanes that share a row in the symbolic phase: 16, or all 64 where a bitmap
// takes more than 16 lanes of 16 bytes (L = words / 4).
template <int L>
constexpr int row_lanes() {
  return L <= 16 ? 16 : WAVE;
}

// The OR of the bitmaps of the B rows named by A entries [p0, p1), over a
// group of GR lanes: lane sub holds words 4 (sub % L) .. + 3 (L lanes to a
// bitmap, GR / L bitmaps side by side) in acc, and the products in pc.  Both
// are the lane's own part: reduce with group_or.
template <int L>
__device__ __forceinline__ void or_rows(const int32_t* acol, int64_t p0, int64_t p1, const uint4* bbm, uint4& acc,
                                        uint32_t& pc) {
  constexpr int GR = row_lanes<L>();
  constexpr int EP = GR / L;                       // entries side by side
  constexpr int UB = L == 1 ? 4 : L == 2 ? 2 : 1;  // batches of GR entries in flight
  constexpr int H = L < 8 ? L : 8;                 // loads in flight per batch
  const int sub = threadIdx.x & (GR - 1);
  for (int64_t p = p0; p < p1; p += GR * UB) {
    int k[UB];
#pragma unroll
    for (int b = 0; b < UB; ++b) k[b] = p + GR * b + sub < p1 ? acol[p + GR * b + sub] : -1;
#pragma unroll
    for (int b = 0; b < UB; ++b)
      for (int h = 0; h < L; h += H) {
        if (L > H && p + GR * b + h * EP >= p1) break;  // uniform over the group
        uint4 x[H];
        bool ok[H];
#pragma unroll
        for (int s = 0; s < H; ++s) {
          const int kk = __shfl(k[b], (h + s) * EP + sub / L, GR);
          ok[s] = kk >= 0;
          x[s] = bbm[(int64_t)(ok[s] ? kk : 0) * L + sub % L];
        }
#pragma unroll
        for (int s = 0; s < H; ++s) {
          const uint32_t m = ok[s] ? ~0u : 0u;
          x[s].x &= m; x[s].y &= m; x[s].z &= m; x[s].w &= m;
          acc.x |= x[s].x; acc.y |= x[s].y; acc.z |= x[s].z; acc.w |= x[s].w;
          pc += __popc(x[s].x) + __popc(x[s].y) + __popc(x[s].z) + __popc(x[s].w);
        }
      }
  }
}

template <int L>
__device__ __forceinline__ void group_or(uint4& acc, uint32_t& pc) {
  constexpr int GR = row_lanes<L>();
#pragma unroll
  for (int o = L; o < GR; o <<= 1) {
    acc.x |= __shfl_xor(acc.x, o, GR);
    acc.y |= __shfl_xor(acc.y, o, GR);
    acc.z |= __shfl_xor(acc.z, o, GR);
    acc.w |= __shfl_xor(acc.w, o, GR);
  }
#pragma unroll
  for (int o = 1; o < GR; o <<= 1) pc += __shfl_xor(pc, o, GR);
}

// A lane group per row; rows above NARROW_LONG entries are pushed as parts of
// NARROW_PART entries for k_narrow_long, with counts[row] = -1 (k_bin_count
// sums those rows' popcounts once every part has been added).
template <typename RA, int L>
__global__ __launch_bounds__(256) void k_narrow_symbolic(const Operands op, int64_t nrows, const NarrowView nv,
                                                         int64_t* P, int64_t* counts, unsigned long long* total) {
  __shared__ int64_t red[256 / WAVE];
  constexpr int GR = row_lanes<L>();
  const int sub = threadIdx.x & (GR - 1);
  const int64_t nsub = (int64_t)gridDim.x * (256 / GR);
  const uint4* bbm = reinterpret_cast<const uint4*>(nv.bbm);
  uint4* cbm = reinterpret_cast<uint4*>(nv.cbm);
  int64_t mine = 0;
  for (int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / GR; row < nrows; row += nsub) {
    const int64_t p0 = ld_rp<RA>(op.arp, row) - op.a_base;
    const int64_t p1 = ld_rp<RA>(op.arp, row + 1) - op.a_base;
    uint4 acc = make_uint4(0u, 0u, 0u, 0u);
    if (p1 - p0 > NARROW_LONG) {  // uniform over the group
      if (sub == 0) {
        const int np = (int)((p1 - p0 + NARROW_PART - 1) / NARROW_PART);
        const int at = atomicAdd(nv.nparts, np);
        for (int i = 0; i < np; ++i) nv.parts[at + i] = NarrowPart{(int32_t)row, i};
        P[row] = 0;
        counts[row] = -1;
      }
      if (sub < L) cbm[row * L + sub] = acc;
      continue;
    }
    uint32_t pc = 0;
    or_rows<L>(op.acol, p0, p1, bbm, acc, pc);
    group_or<L>(acc, pc);
    int c = sub < L ? __popc(acc.x) + __popc(acc.y) + __popc(acc.z) + __popc(acc.w) : 0;
#pragma unroll
    for (int o = 1; o < L; o <<= 1) c += __shfl_xor(c, o, GR);
    if (sub < L) cbm[row * L + sub] = acc;
    if (sub == 0) {
      counts[row] = c;
      P[row] = pc;
      mine += pc;
    }
  }
  mine = wave_sum(mine);
  if (lane_id() == 0) red[threadIdx.x / WAVE] = mine;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int i = 0; i < 256 / WAVE; ++i) t += red[i];
    if (t) atomicAdd(total, (unsigned long long)t);
  }
}

// One part of a long row per workgroup, an equal share per lane group; ORed and added into the row's bitmap and products.
template <typename RA, int L>
__global__ __launch_bounds__(256) void k_narrow_long(const Operands op, const NarrowView nv, int64_t* P,
                                                     unsigned long long* total) {
  constexpr int W = 4 * L;
  __shared__ uint32_t bm[W];
  constexpr int GR = row_lanes<L>();
  __shared__ uint32_t sum;
  const int sub = threadIdx.x & (GR - 1), sg = threadIdx.x / GR;
  const int n = *nv.nparts;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const NarrowPart pt = nv.parts[it];
    const int64_t p0 = ld_rp<RA>(op.arp, pt.row) - op.a_base;
    const int64_t p1 = ld_rp<RA>(op.arp, pt.row + 1) - op.a_base;
    constexpr int SHARE = NARROW_PART / (256 / GR);  // entries of one group
    const int64_t q0 = min(p1, p0 + (int64_t)pt.part * NARROW_PART + sg * SHARE);
    const int64_t q1 = min(p1, q0 + SHARE);
    for (int i = threadIdx.x; i < W; i += 256) bm[i] = 0u;
    if (threadIdx.x == 0) sum = 0u;
    __syncthreads();
    uint4 acc = make_uint4(0u, 0u, 0u, 0u);
    uint32_t pc = 0;
    or_rows<L>(op.acol, q0, q1, reinterpret_cast<const uint4*>(nv.bbm), acc, pc);
    group_or<L>(acc, pc);
    if (sub < L) {
      if (acc.x) atomicOr(&bm[4 * sub], acc.x);
      if (acc.y) atomicOr(&bm[4 * sub + 1], acc.y);
      if (acc.z) atomicOr(&bm[4 * sub + 2], acc.z);
      if (acc.w) atomicOr(&bm[4 * sub + 3], acc.w);
    }
    if (sub == 0 && pc) atomicAdd(&sum, pc);
    __syncthreads();
    for (int i = threadIdx.x; i < W; i += 256)
      if (bm[i]) atomicOr(&nv.cbm[(int64_t)pt.row * W + i], bm[i]);
    if (threadIdx.x == 0 && sum) {
      atomicAdd(reinterpret_cast<unsigned long long*>(&P[pt.row]), (unsigned long long)sum);
      atomicAdd(total, (unsigned long long)sum);
    }
    __syncthreads();
  }
}

// ----------------------------------------------------------------- numeric

__device__ __forceinline__ int lanes_below(uint64_t bits) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, 0u));
}

// 64 words of a row's bitmap from word 64 i on, one per lane
__device__ __forceinline__ uint32_t row_word(const NarrowView& nv, int64_t row, int i) {
  const int w = 64 * i + lane_id();
  return w < nv.words ? nv.cbm[row * nv.words + w] : 0u;
}

// the 64 presence bits of the c-th 64 columns of those words: lane w holds word w
__device__ __forceinline__ uint64_t chunk_bits(uint32_t word, int c) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)word, 2 * c);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)word, 2 * c + 1);
  return ((uint64_t)hi << 32) | lo;
}

struct Entry {  // of A: the byte offset of its B row's slot, and its value
  uint32_t at;
  float a;
};

constexpr int WINDOW = 128;  // entries of A a wavefront holds in LDS
constexpr int WINDOW_PAD = 32;  // entries past a window that a step may read (and not use)
constexpr int WPL = WINDOW / WAVE;

// A wavefront's LDS: its dense rows, column c of lane group g at acc[c * G +
// g], so that the G sums of a column are one vector, with one column more for
// what is not used; then a window of A's entries.  S lanes take one B row:
// entry sl and, where slots hold more than S (TWO: S < cap <= 2 S), entry S +
// sl; rows above cap go on in B's arrays, with O loads of each array in flight
// where DEEP (k_narrow_block; rows of 600 entries in slots of 106, 47 M
// products: 312 us with one at a time).  In k_narrow_rows, whose rows are short
// and registers few, that cost 5 % (N = 4000, 240 M products: 1154 -> 1203 us).
template <typename RB, int S, bool TWO, bool DEEP = false>
struct DenseRows {
  static constexpr int G = WAVE / S;
  static constexpr int U = 4;  // steps (of G entries) in flight together
  static constexpr int O = 4;
  static_assert(G * U <= WINDOW_PAD, "a step reads at most the padding past the window");
  unsigned char* acc;
  Entry* win;
  const unsigned char* slots;
  int cap, slot;
  uint32_t no_col;

  static __host__ __device__ constexpr size_t acc_bytes(int Np) { return sizeof(float) * G * (size_t)(Np + 4); }
  static __host__ __device__ constexpr size_t bytes(int Np) {
    return acc_bytes(Np) + sizeof(Entry) * (WINDOW + WINDOW_PAD);
  }
  __device__ __forceinline__ DenseRows(unsigned char* base, const NarrowView& nv, int Np)
      : acc(base),
        win(reinterpret_cast<Entry*>(base + acc_bytes(Np))),
        slots(nv.slots),
        cap(nv.cap),
        slot(nv.slot),
        no_col((uint32_t)(4 * G * Np)) {}
  __device__ __forceinline__ void clear(int Np) {
    for (int i = lane_id(); i < Np * G; i += WAVE) reinterpret_cast<float*>(acc)[i] = 0.f;
  }

  // entries [p, pe) of A into the window, as far as it holds them; the rest
  // of it and its padding name an entry that is there
  __device__ __forceinline__ void fill(const Operands& op, int64_t p, int64_t pe) {
    int k[WPL];
    float a[WPL];
#pragma unroll
    for (int i = 0; i < WPL; ++i) {
      const int64_t q = p + i * WAVE + lane_id();
      k[i] = op.acol[q < pe ? q : p];
      a[i] = op.aval[q < pe ? q : p];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < WPL; ++i) win[i * WAVE + lane_id()] = Entry{(uint32_t)k[i] * (uint32_t)slot, a[i]};
    if (lane_id() < WINDOW_PAD) win[WINDOW + lane_id()] = Entry{(uint32_t)k[0] * (uint32_t)slot, 0.f};
    wave_sync();
  }

  // adds a * v at column word c
  __device__ __forceinline__ void put(uint32_t c, float a, float v) {
    float* x = reinterpret_cast<float*>(acc + ((c & (GOES_ON - 1u)) | (uint32_t)(lane_id() / S * 4)));
    *x = fmaf(a, v, *x);
    wave_sync();
  }

  // adds entries [j, min(j1, j + G U)) of the window.  No branch between the
  // loads, so that they are in flight together: a lane past the slot repeats
  // its last entry (a read past it would fetch the next slot's cache line),
  // and what is not an entry of the lane's own goes to the spare column.
  template <bool FULL>
  __device__ __forceinline__ void add(const Operands& op, int j, int j1) {
    const int lane = lane_id(), g = lane / S, sl = lane % S;
    const uint32_t i1 = (uint32_t)(TWO || sl < cap ? sl : cap - 1), i2 = (uint32_t)(S + sl < cap ? S + sl : cap - 1);
    const unsigned char* cols = slots + 4 * cap;
    uint32_t c[U], c2[TWO ? U : 1];
    float v[U], v2[TWO ? U : 1], a[U];
    const Entry* w = win + j + g;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Entry en = w[u * G];
      a[u] = en.a;
      v[u] = *reinterpret_cast<const float*>(slots + (en.at + 4u * i1));
      c[u] = *reinterpret_cast<const uint16_t*>(cols + (en.at + 2u * i1));
      if constexpr (TWO) {
        v2[u] = *reinterpret_cast<const float*>(slots + (en.at + 4u * i2));
        c2[u] = *reinterpret_cast<const uint16_t*>(cols + (en.at + 2u * i2));
      }
    }
    wave_sync();  // the loads stay above what follows
    const bool in1 = TWO || sl < cap, in2 = sl < cap - S;
    uint32_t over = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!FULL && j + u * G >= j1) break;  // uniform
      const bool on = FULL || j + u * G + g < j1;
      over |= TWO ? c2[u] : c[u];
      put(on && in1 ? c[u] : no_col, a[u], v[u]);
      if constexpr (TWO) {
        const uint32_t d = on && in2 ? c2[u] : no_col;
        if (__any((d & (GOES_ON - 1u)) != no_col)) put(d, a[u], v2[u]);
      }
    }
    // rows longer than their slot: the top bit of the slot's last column word
    if (__any((over & GOES_ON) && sl == (TWO ? cap - 1 - S : cap - 1))) {
#pragma unroll 1
      for (int u = 0; u < U; ++u) {
        const int e = j + u * G + g;
        int64_t q = 0, end = 0;
        float x = 0.f;
        if (e < j1) {
          const Entry en = win[e];
          const int64_t k = en.at / (uint32_t)slot;
          x = en.a;
          q = ld_rp<RB>(op.brp, k) + cap + sl;
          end = ld_rp<RB>(op.brp, k + 1);
        }
        if constexpr (DEEP) {
          for (; __any(q < end); q += O * S) {
            uint32_t col[O];
            float b[O];
#pragma unroll
            for (int i = 0; i < O; ++i) {
              const int64_t at = q + i * S < end ? q + i * S : 0;
              col[i] = (uint32_t)op.bcol[at] * (4u * G);
              b[i] = op.bval[at];
            }
            wave_sync();
#pragma unroll
            for (int i = 0; i < O; ++i) {
              if (i && !__any(q + i * S < end)) break;
              put(q + i * S < end ? col[i] : no_col, x, b[i]);
            }
          }
          continue;
        }
        for (; __any(q < end); q += S) {
          uint32_t col = no_col;
          float b = 0.f;
          if (q < end) {
            col = (uint32_t)op.bcol[q] * (4u * G);
            b = op.bval[q];
          }
          put(col, x, b);
        }
      }
    }
  }

  // adds entries [j, j1) of the window
  __device__ __forceinline__ void add_all(const Operands& op, int j, int j1) {
    for (; j + G * U <= j1; j += G * U) add<true>(op, j, j1);
    if (j < j1) add<false>(op, j, j1);
  }

  // the sum of column c over the groups; the slots are cleared
  __device__ __forceinline__ float take(int c) {
    float v;
    if constexpr (G == 1) {
      float* x = reinterpret_cast<float*>(acc) + c;
      v = *x;
      *x = 0.f;
    } else if constexpr (G == 2) {
      float2* x = reinterpret_cast<float2*>(acc) + c;
      v = x->x + x->y;
      *x = make_float2(0.f, 0.f);
    } else {
      float4* x = reinterpret_cast<float4*>(acc) + c * (G / 4);
      v = 0.f;
#pragma unroll
      for (int i = 0; i < G / 4; ++i) {
        const float4 y = x[i];
        v += (y.x + y.y) + (y.z + y.w);
        x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    return v;
  }
};

constexpr int MAX_ROWS_PER_TURN = 16;   // consecutive rows a wavefront takes at a time

// Rows with 0 < P_i <= max_p, `turn` consecutive ones to a wavefront.
// Rows of a single entry (isolated vertices: their C row is a_ik times B_k)
// come first, a lane group each.  The entries of the others are one run of A,
// read a window at a time whatever rows they belong to.
template <typename RA, typename RB, int S, bool TWO>
__global__ __launch_bounds__(WAVE, 8) void k_narrow_rows(const Operands op, const NarrowView nv, const int64_t* P,
                                                         int64_t nrows, int64_t max_p, int turn, const Outputs out) {
  extern __shared__ __align__(16) unsigned char smem[];
  using DR = DenseRows<RB, S, TWO>;
  const int N = (int)op.N, Np = padded_cols(N);
  const int lane = lane_id(), sl = lane % S;
  DR D(smem, nv, Np);
  D.clear(Np);
  for (int64_t r0 = (int64_t)blockIdx.x * turn; r0 < nrows; r0 += (int64_t)gridDim.x * turn) {
    const int nr = (int)(nrows - r0 < turn ? nrows - r0 : turn);
    int64_t rp = 0, crp = 0, prods = 0;
    if (lane <= nr) rp = ld_rp<RA>(op.arp, r0 + lane) - op.a_base;
    if (lane < nr) {
      crp = out.crp[r0 + lane];
      prods = P[r0 + lane];
    }
    const int64_t rp1 = __shfl(rp, lane + 1);
    const bool mine = prods > 0 && prods <= max_p;
    const uint64_t ones = __ballot(mine && rp1 - rp == 1);
    uint64_t todo = __ballot(mine) & ~ones;
    for (uint64_t left = ones; left;) {
      // lane group g takes the g-th row left
      int row = -1;
      uint64_t b = left;
#pragma unroll
      for (int g = 0; g < DR::G; ++g) {
        if (lane / S == g && b) row = __builtin_ctzll(b);
        b &= b - 1u;
      }
      left = b;
      const int64_t p = __shfl(rp, row < 0 ? 0 : row), o = __shfl(crp, row < 0 ? 0 : row);
      if (row < 0) continue;
      const int64_t k = op.acol[p];
      const float a = op.aval[p];
      const unsigned char* s = D.slots + k * D.slot;
      const uint16_t* cols = reinterpret_cast<const uint16_t*>(s + 4 * D.cap);
      for (int q = sl; q < D.cap; q += S) {
        const uint32_t c = cols[q] & (GOES_ON - 1u);
        if (c == D.no_col) break;
        const float x = a * reinterpret_cast<const float*>(s)[q];
        store_stream(&out.ccol[o + q], (int32_t)(c / (4u * DR::G)));
        store_stream(&out.cval[o + q], 0.f + x);
      }
      if (cols[D.cap - 1] & GOES_ON) {  // longer than its slot
        const int64_t lo = ld_rp<RB>(op.brp, k), len = ld_rp<RB>(op.brp, k + 1) - lo;
        for (int64_t q = D.cap + sl; q < len; q += S) {
          const float x = a * op.bval[lo + q];
          store_stream(&out.ccol[o + q], op.bcol[lo + q]);
          store_stream(&out.cval[o + q], 0.f + x);
        }
      }
    }
    if (!todo) continue;
    const int last = 63 - __builtin_clzll(todo);
    const int64_t pend = lane_i64(rp, last + 1);
    int64_t w0 = lane_i64(rp, __builtin_ctzll(todo));  // the window's first entry
    D.fill(op, w0, pend);
    while (todo) {
      const int i = __builtin_ctzll(todo);
      todo &= todo - 1u;
      const int64_t row = r0 + i;
      const int64_t s = lane_i64(rp, i), e = lane_i64(rp, i + 1);
      int64_t o0 = lane_i64(crp, i);
      uint32_t word = row_word(nv, row, 0);
      for (int64_t p = s; p < e;) {
        if (p >= w0 + WINDOW) {
          w0 = p;
          D.fill(op, w0, pend);
        }
        const int j1 = (int)(e - w0 < WINDOW ? e - w0 : WINDOW);
        D.add_all(op, (int)(p - w0), j1);
        p = w0 + j1;
      }
      wave_sync();
      for (int c0 = 0; c0 < Np / 64; c0 += 32) {  // 64 words hold 32 times 64 columns
        if (c0) word = row_word(nv, row, c0 / 32);
        const int nc = Np / 64 - c0 < 32 ? Np / 64 - c0 : 32;
        for (int c = 0; c < nc; ++c) {
          const uint64_t bits = chunk_bits(word, c);
          if (!bits) continue;
          const int col = (c0 + c) * 64 + lane;
          const float v = D.take(col);
          if ((bits >> lane) & 1u) {
            const int64_t o = o0 + lanes_below(bits);
            store_stream(&out.ccol[o], col);
            store_stream(&out.cval[o], v);
          }
          o0 += __popcll(bits);
        }
      }
      wave_sync();
    }
  }
}

// wavefronts of a k_narrow_block workgroup: eight, or four where their dense
// rows (up to 16 KB each) would leave one workgroup to a CU otherwise
constexpr int block_waves(int64_t N) { return N <= 2048 ? 8 : 4; }

// Rows of a bin, a workgroup per row (SPLIT: per part of a row, NARROW_PARTS
// of them, added into the row's dense slot): the wavefronts take windows of
// entries in turn, each into dense rows of its own, added up at the end.
template <typename RA, typename RB, int S, bool TWO, bool SPLIT, int NWV>
__global__ __launch_bounds__(NWV* WAVE, NWV) void k_narrow_block(const Operands op, const NarrowView nv, const BinView bv,
                                                               const SplitWs sw, const Outputs out) {
  extern __shared__ __align__(16) unsigned char smem[];
  using DR = DenseRows<RB, S, TWO, true>;
  const int N = (int)op.N, Np = padded_cols(N);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int lane = lane_id();
  const size_t per = DR::bytes(Np);
  DR D(smem + wv * per, nv, Np);
  D.clear(Np);
  const int32_t* list = bv.list + bv.binoff[bv.bin];
  int64_t cnt = bv.binoff[bv.bin + 1] - bv.binoff[bv.bin];
  if (SPLIT) cnt = min(cnt, sw.cap) * NARROW_PARTS;
  for (int64_t it = blockIdx.x + (SPLIT ? 0 : bv.skip); it < cnt; it += gridDim.x) {
    const int64_t d = SPLIT ? it / NARROW_PARTS : it;
    const int64_t row = list[d];
    int64_t p0 = ld_rp<RA>(op.arp, row) - op.a_base;
    int64_t p1 = ld_rp<RA>(op.arp, row + 1) - op.a_base;
    if (SPLIT) {
      const int64_t share = (p1 - p0 + NARROW_PARTS - 1) / NARROW_PARTS;
      p0 = min(p1, p0 + (it - d * NARROW_PARTS) * share);
      p1 = min(p1, p0 + share);
      if (p0 == p1) continue;  // uniform over the workgroup
    }
    uint32_t word = row_word(nv, row, 0);
    // the wavefronts' equal shares, a window at a time
    const int64_t share = ((p1 - p0 + NWV - 1) / NWV + DR::G - 1) / DR::G * DR::G;
    const int64_t q0 = min(p1, p0 + wv * share), q1 = min(p1, q0 + share);
    for (int64_t q = q0; q < q1; q += WINDOW) {
      D.fill(op, q, q1);
      const int j1 = (int)(q1 - q < WINDOW ? q1 - q : WINDOW);
      D.add_all(op, 0, j1);
    }
    __syncthreads();
    // sums over the wavefronts and groups, 64 columns to a wavefront
    int64_t o0 = SPLIT ? 0 : out.crp[row];
    for (int c0 = 0; c0 < Np / 64; c0 += 32) {  // 64 words hold 32 times 64 columns
      if (c0) word = row_word(nv, row, c0 / 32);
      const int pc = __popc(word);
      const int incl = wave_incl_scan(pc);
      const int pre = incl - pc;
      const int nc = Np / 64 - c0 < 32 ? Np / 64 - c0 : 32;
      for (int c = wv; c < nc; c += NWV) {
        const uint64_t bits = chunk_bits(word, c);
        if (!bits) continue;
        const int col = (c0 + c) * 64 + lane;
        float v = 0.f;
#pragma unroll 2
        for (int w = 0; w < NWV; ++w) v += DR(smem + w * per, nv, Np).take(col);
        if ((bits >> lane) & 1u) {
          if constexpr (SPLIT) {
            if (v != 0.f) atomicAdd(&sw.acc[d * N + col], v);
          } else {
            const int64_t o = o0 + __builtin_amdgcn_readlane(pre, 2 * c) + lanes_below(bits);
            store_stream(&out.ccol[o], col);
            store_stream(&out.cval[o], v);
          }
        }
      }
      o0 += wave_last(incl);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_narrow_clear(const BinView bv, SplitWs sw, int32_t N) {
  const int64_t cnt = min((int64_t)(bv.binoff[bv.bin + 1] - bv.binoff[bv.bin]), sw.cap);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt * N; i += stride) sw.acc[i] = 0.f;
}

// One wavefront per split row writes its slot in column order.
__global__ __launch_bounds__(256) void k_narrow_finish(const BinView bv, const SplitWs sw, const NarrowView nv,
                                                       int32_t N, const Outputs out) {
  const int32_t* list = bv.list + bv.binoff[bv.bin];
  const int64_t cnt = min((int64_t)(bv.binoff[bv.bin + 1] - bv.binoff[bv.bin]), sw.cap);
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x / WAVE);
  const int lane = lane_id();
  for (int64_t d = (int64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE; d < cnt; d += nw) {
    const int64_t row = list[d];
    int64_t o0 = out.crp[row];
    for (int c0 = 0; c0 < padded_cols(N) / 64; c0 += 32) {
      const uint32_t word = row_word(nv, row, c0 / 32);
      const int nc = padded_cols(N) / 64 - c0 < 32 ? padded_cols(N) / 64 - c0 : 32;
      for (int c = 0; c < nc; ++c) {
        const uint64_t bits = chunk_bits(word, c);
        if ((bits >> lane) & 1u) {
          const int64_t o = o0 + lanes_below(bits);
          store_stream(&out.ccol[o], (c0 + c) * 64 + lane);
          store_stream(&out.cval[o], sw.acc[d * N + (c0 + c) * 64 + lane]);
        }
        o0 += __popcll(bits);
      }
    }
  }
}

// ---------------------------------------------------------------- launches

template <typename RA, int L>
hipError_t symbolic_t(const Operands& op, int64_t nrows, int64_t nnz, const NarrowView& nv, int64_t* P,
                      int64_t* counts, unsigned long long* total, hipStream_t s) {
  int64_t grid = (nrows * row_lanes<L>() + 255) / 256;
  if (grid > 8192) grid = 8192;
  hipLaunchKernelGGL((k_narrow_symbolic<RA, L>), dim3((unsigned)grid), dim3(256), 0, s, op, nrows, nv, P, counts,
                     total);
  int64_t lg = std::min<int64_t>(nnz / NARROW_LONG, 4096);  // no long rows below NARROW_LONG entries
  if (lg > 0) hipLaunchKernelGGL((k_narrow_long<RA, L>), dim3((unsigned)lg), dim3(256), 0, s, op, nv, P, total);
  return hipGetLastError();
}

template <typename RA>
hipError_t symbolic_l(const Operands& op, int64_t nrows, int64_t nnz, const NarrowView& nv, int64_t* P,
                      int64_t* counts, unsigned long long* total, hipStream_t s) {
  switch (nv.words / 4) {
    case 1: return symbolic_t<RA, 1>(op, nrows, nnz, nv, P, counts, total, s);
    case 2: return symbolic_t<RA, 2>(op, nrows, nnz, nv, P, counts, total, s);
    case 4: return symbolic_t<RA, 4>(op, nrows, nnz, nv, P, counts, total, s);
    case 8: return symbolic_t<RA, 8>(op, nrows, nnz, nv, P, counts, total, s);
    case 16: return symbolic_t<RA, 16>(op, nrows, nnz, nv, P, counts, total, s);
    case 32: return symbolic_t<RA, 32>(op, nrows, nnz, nv, P, counts, total, s);
    case 64: return symbolic_t<RA, 64>(op, nrows, nnz, nv, P, counts, total, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename K>
int64_t resident_blocks(K kern, int block, size_t lds) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, block, lds) != hipSuccess || per_cu <= 0) per_cu = 1;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  return (int64_t)per_cu * cus;
}

template <typename K>
hipError_t allow_lds(K kern, size_t lds) {
  return lds > 65536 ? hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
                     : hipSuccess;
}

template <typename RA, typename RB, int S, bool TWO>
hipError_t rows_t(const Operands& op, const NarrowView& nv, const int64_t* P, int64_t nrows, int64_t max_p,
                  const Outputs& out, hipStream_t s) {
  auto kern = k_narrow_rows<RA, RB, S, TWO>;
  const int Np = padded_cols(op.N);
  const size_t lds = DenseRows<RB, S, TWO>::bytes(Np);
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  // few rows: fewer to a turn, so that every wavefront slot of the chip has some
  const int64_t slots = resident_blocks(kern, WAVE, lds);
  const int turn = (int)std::max<int64_t>(1, std::min<int64_t>(MAX_ROWS_PER_TURN, nrows / slots));
  const int64_t need = (nrows + turn - 1) / turn;
  const int64_t grid = std::min<int64_t>(need, 1 << 20);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WAVE), lds, s, op, nv, P, nrows, max_p, turn,
                     out);
  return hipGetLastError();
}

template <typename RA, typename RB, int S, bool TWO, int NWV>
hipError_t block_w(const Operands& op, const NarrowView& nv, const BinView& bv, const SplitWs* sw, int64_t rows,
                   const Outputs& out, hipStream_t s) {
  const size_t lds = NWV * DenseRows<RB, S, TWO>::bytes(padded_cols(op.N));
  if constexpr (NWV == 8) {
    if (sw && sw->cap > 0) {
      const int64_t cap = std::min(rows, sw->cap);
      const int64_t cg = std::min<int64_t>((cap * op.N + 255) / 256, 4096);
      hipLaunchKernelGGL(k_narrow_clear, dim3((unsigned)cg), dim3(256), 0, s, bv, *sw, (int32_t)op.N);
      auto kern = k_narrow_block<RA, RB, S, TWO, true, NWV>;
      hipError_t e = allow_lds(kern, lds);
      if (e != hipSuccess) return e;
      const int64_t grid = std::min(cap * NARROW_PARTS, 4 * resident_blocks(kern, NWV * WAVE, lds));
      hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NWV * WAVE), lds, s, op, nv, bv, *sw, out);
      const int64_t fg = std::min<int64_t>((cap + 3) / 4, 8192);
      hipLaunchKernelGGL(k_narrow_finish, dim3((unsigned)fg), dim3(256), 0, s, bv, *sw, nv, (int32_t)op.N, out);
      e = hipGetLastError();
      if (e != hipSuccess || rows <= sw->cap) return e;
    }
  }
  // a workgroup per row (of a split bin: the rows beyond its slots)
  BinView rest = bv;
  rest.skip = sw ? (int32_t)sw->cap : 0;
  const int64_t left = rows - rest.skip;
  auto kern = k_narrow_block<RA, RB, S, TWO, false, NWV>;
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int64_t grid = std::min(left, 4 * resident_blocks(kern, NWV * WAVE, lds));
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NWV * WAVE), lds, s, op, nv, rest, SplitWs{}, out);
  return hipGetLastError();
}

template <typename RA, typename RB, int S, bool TWO>
hipError_t block_t(const Operands& op, const NarrowView& nv, const BinView& bv, const SplitWs* sw, int64_t rows,
                   const Outputs& out, hipStream_t s) {
  if constexpr (S == WAVE)  // above 2048 columns the lanes are always 64
    if (block_waves(op.N) == 4) return block_w<RA, RB, S, TWO, 4>(op, nv, bv, nullptr, rows, out, s);
  return block_w<RA, RB, S, TWO, 8>(op, nv, bv, sw, rows, out, s);
}

// fn<RA, RB, S, TWO>(...) for the operands' row-pointer widths and the slots
#define NARROW_DISPATCH(op, S, TWO, FN, ...)                                                    \
  ((op).rpa64 ? ((op).rpb64 ? FN<int64_t, int64_t, S, TWO>(__VA_ARGS__)                         \
                            : FN<int64_t, int32_t, S, TWO>(__VA_ARGS__))                        \
              : ((op).rpb64 ? FN<int32_t, int64_t, S, TWO>(__VA_ARGS__)                         \
                            : FN<int32_t, int32_t, S, TWO>(__VA_ARGS__)))
#define NARROW_LANES(op, nv, S, FN, ...)                                 \
  case S:                                                                \
    return (nv).cap > S ? NARROW_DISPATCH(op, S, true, FN, __VA_ARGS__)  \
                        : NARROW_DISPATCH(op, S, false, FN, __VA_ARGS__);
#define NARROW_SWITCH(op, nv, FN, ...)        \
  switch ((nv).lanes) {                       \
    NARROW_LANES(op, nv, 8, FN, __VA_ARGS__)  \
    NARROW_LANES(op, nv, 16, FN, __VA_ARGS__) \
    NARROW_LANES(op, nv, 32, FN, __VA_ARGS__) \
    NARROW_LANES(op, nv, 64, FN, __VA_ARGS__) \
    default: return hipErrorInvalidValue;     \
  }

}  // namespace

int32_t narrow_words(int64_t N) {
  int32_t w = 4;
  while ((int64_t)w * 32 < N) w *= 2;
  return w;
}

// Slots for B rows of mean length mu: room for mu + 2.2 sqrt(mu) entries (few
// rows of a feature matrix are longer), in whole 64-byte blocks, for at most
// twice the lanes that take a row.  The lanes: the power of two from 1.25 mu
// on, at least 8, and enough that a wavefront's dense rows (64 / lanes of N
// floats) stay within 8 KB (above 2048 columns: 64 lanes, up to 16 KB).
bool narrow_slots(int64_t N, int64_t K, int64_t nnz, NarrowView* nv) {
  nv->lanes = nv->cap = nv->slot = 0;
  if (K <= 0 || nnz <= 0 || N > NARROW_SLOT_COLS) return false;
  const double mu = (double)nnz / (double)K;
  if (N > 2048 && mu < WAVE / 2) return false;  // 64 lanes a row from there on (see NARROW_SLOT_COLS)
  const double want = mu + 2.2 * std::sqrt(mu);
  int S = 8;
  while (S < WAVE && ((double)S < 1.25 * mu || N * (WAVE / S) > 2048)) S *= 2;
  static_assert(4 * padded_cols(NARROW_SLOT_COLS) < GOES_ON, "column words hold every column and the spare one");
  if (want > 2.0 * S) return false;
  const int slot = ((int)std::ceil(6.0 * want) + 63) / 64 * 64;
  if ((int64_t)slot * K >= (int64_t)1 << 32) return false;  // offsets in 32 bits
  nv->lanes = S;
  nv->slot = slot;
  nv->cap = std::min(2 * S, slot / 6 / 2 * 2);
  return true;
}

hipError_t narrow_prepare(const void* brp, int rpb64, const int32_t* bcol, const float* bval, int64_t K, int64_t N,
                          const NarrowView& nv, hipStream_t s) {
  if (K <= 0) return hipSuccess;
  int rows = 64;  // per workgroup, within 32 KB of LDS
  const size_t per = (size_t)nv.words * 4 + nv.slot;
  while (rows > 16 && rows * per > 32768) rows /= 2;
  const dim3 grid((unsigned)((K + rows - 1) / rows));
  if (rpb64)
    hipLaunchKernelGGL(k_narrow_prepare<int64_t>, grid, dim3(256), rows * per, s, brp, bcol, bval, K, N, nv, rows);
  else
    hipLaunchKernelGGL(k_narrow_prepare<int32_t>, grid, dim3(256), rows * per, s, brp, bcol, bval, K, N, nv, rows);
  return hipGetLastError();
}

hipError_t narrow_symbolic(const Operands& op, int64_t nrows, int64_t nnz, const NarrowView& nv, int64_t* P,
                           int64_t* counts, unsigned long long* total, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  return op.rpa64 ? symbolic_l<int64_t>(op, nrows, nnz, nv, P, counts, total, s)
                  : symbolic_l<int32_t>(op, nrows, nnz, nv, P, counts, total, s);
}

hipError_t narrow_rows(const Operands& op, const NarrowView& nv, const int64_t* P, int64_t nrows, int64_t max_p,
                       const Outputs& out, hipStream_t s) {
  if (nrows <= 0) return hipSuccess;
  NARROW_SWITCH(op, nv, rows_t, op, nv, P, nrows, max_p, out, s)
}

hipError_t narrow_block(const Operands& op, const NarrowView& nv, const BinView& bv, const SplitWs* sw, int64_t rows,
                        const Outputs& out, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  NARROW_SWITCH(op, nv, block_t, op, nv, bv, sw, rows, out, s)
}

}  // namespace kern
}  // namespace aires
