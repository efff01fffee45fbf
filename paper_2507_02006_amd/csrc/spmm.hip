// Sparse-times-dense product Y = act(A * W) on gfx950: the combination step
// of a GCN layer (Sec. II-A, Eq. 3: the aggregated features times the
// layer's weights, then the activation) and, with a dense feature matrix,
// the aggregation of Eq. 1.  A is CSR (32- or 64-bit row pointers), W and
// Y are dense row-major with leading dimensions ldw and ldy.
//
// Entry gather (sparse A): L lanes own one entry's row of W, V columns a
// lane, and the 64 / L lane groups of a wavefront take different entries of
// the row of A; their partial rows are added across the groups at the end.
// Rows with at most kHeavy entries (more where rows are long on average) take
// one wavefront each; longer rows take the eight wavefronts of a workgroup, per
// block of 64 columns, and come first in the same launch.  Dense tiles: see
// below.  The activation is applied before the store; every element of Y is
// written exactly once.
#include "kernels.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace aires {
namespace kern {
namespace {

constexpr int WAVE = 64;
constexpr int SPMM_BLOCK = 512;  // eight wavefronts
// Longer rows are split over a workgroup: 128 and 512 were slower (4000 rows,
// F = 256: 29.6 and 19.3 us against 12.8; 150 K rows: 231 and 241 against 225).
constexpr int64_t kHeavy = 256;
// Where rows are long on average the limit is twice the mean, as far as that is
// no more than an even share of the work for 3072 wavefronts (about half of
// those the chip holds): rows of like length keep the wavefronts busy by
// themselves (20 K rows of 300 entries, F = 64 / 256: 61 / 219 us a wavefront
// each, 100 / 373 split).
constexpr int64_t kHeavyShare = 3072;
// The workgroups for heavy rows look for them in groups of at most 512 rows. A
// group's heavy rows come one after the other, so there are at least
// kHeavyGroups groups where each can have kHeavyGroup entries (256 rows of 900
// entries, F = 64: 877 us in one group, 11 so). More would make the light rows
// of a small launch wait (4000 rows of 200, F = 64: 12.3 us with 8 groups,
// 12.5 with 256, 15.5 with 512). Four blocks of columns and more make as many
// workgroups of a group; there the large groups stay where rows are short on
// average (symmetric R-MAT, 8000 rows of 13, F = 256: 18.8 us, 19.7 with small
// groups; F = 128: 13.3 and 13.4, and 20000 rows of 13: 28.0 and 21.3).
constexpr int64_t kHeavyGroups = 256;
constexpr int64_t kHeavyGroup = 1024;
constexpr int64_t kHeavyMean = 48;
constexpr int64_t kMaxCols = int64_t(1) << 20;  // columns of one launch
constexpr unsigned NXCD = 8;     // gfx950 hands workgroups round-robin to its 8 XCDs

template <typename RP>
__device__ __forceinline__ int64_t rp_at(const void* rp, int64_t i) {
  return (int64_t) static_cast<const RP*>(rp)[i];
}

// Four floats at any 4-byte boundary: one 16-byte load or store (global
// memory takes 16-byte accesses at 4-byte alignment), so that row strides and
// bases need no alignment of their own.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

template <int V>
__device__ __forceinline__ void load_cols(const float* p, float (&w)[V]) {
  if constexpr (V == 4) {
    const f32x4_any x = *reinterpret_cast<const f32x4_any*>(p);
    w[0] = x[0]; w[1] = x[1]; w[2] = x[2]; w[3] = x[3];
  } else {
    w[0] = *p;
  }
}

// One wavefront's share of columns [cb, ce) of a row of Y: L lanes per
// entry, V columns per lane (from cb + l * V), E = 64 / L entries side by
// side.  A lane's vector that would end past ce is moved back to end there:
// every load is a whole vector inside the row of W (ce >= V), and the store
// keeps only the columns that are the lane's own.
template <int L, int V>
struct RowPart {
  static constexpr int E = WAVE / L;
  static constexpr int U = E < 8 ? 8 : 4;  // steps of E entries in flight
  int col;                                 // first column loaded
  float acc[V];

  __device__ __forceinline__ void start(int cb, int ce) {
    const int c = cb + (int)(threadIdx.x % L) * V;
    col = c + V <= ce ? c : ce - V;
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
  }

  // acc += a_ik W[k, .] for N steps of E entries from j on; kl, al hold the
  // cnt entries of a batch, one per lane.  Past the batch's last entry a
  // group repeats that entry's load and adds nothing.
  template <int N>
  __device__ __forceinline__ void steps(int kl, float al, int j, int cnt, const float* W, int64_t ldw) {
    float w[N][V], a[N];
    bool ok[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if constexpr (E == 1) {
        a[u] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(al), j + u));
        ok[u] = true;
        load_cols<V>(W + (int64_t)__builtin_amdgcn_readlane(kl, j + u) * ldw + col, w[u]);
      } else {
        const int e = j + u * E + (int)(threadIdx.x % WAVE) / L;
        ok[u] = e < cnt;
        const int ec = ok[u] ? e : cnt - 1;
        a[u] = __shfl(al, ec);
        load_cols<V>(W + (int64_t)__shfl(kl, ec) * ldw + col, w[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float x = fmaf(a[u], w[u][v], acc[v]);
        acc[v] = ok[u] ? x : acc[v];
      }
  }

  // a batch of 1 ... 64 entries; kl, al as above
  __device__ __forceinline__ void batch(int kl, float al, int cnt, const float* W, int64_t ldw) {
    int j = 0;
    for (; j + (U - 1) * E < cnt; j += U * E) steps<U>(kl, al, j, cnt, W, ldw);
    if (U > 4 && j + 3 * E < cnt) { steps<4>(kl, al, j, cnt, W, ldw); j += 4 * E; }
    if (j + E < cnt) { steps<2>(kl, al, j, cnt, W, ldw); j += 2 * E; }
    if (j < cnt) steps<1>(kl, al, j, cnt, W, ldw);
  }

  // the groups' partial rows added up, in every group
  __device__ __forceinline__ void combine_groups() {
#pragma unroll
    for (int o = L; o < WAVE; o <<= 1)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += __shfl_xor(acc[v], o);
  }

  // the first group writes its columns of the row
  __device__ __forceinline__ void store(float* yr, int cb, int ce, int relu) {
    const int lane = threadIdx.x % WAVE;
    if (lane >= L) return;
    const int c = cb + lane * V;
    float y[V];
#pragma unroll
    for (int v = 0; v < V; ++v) y[v] = relu ? fmaxf(acc[v], 0.f) : acc[v];
    if constexpr (V == 4) {
      if (c + V <= ce) {
        *reinterpret_cast<f32x4_any*>(yr + c) = f32x4_any{y[0], y[1], y[2], y[3]};
        return;
      }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (col + v >= c) yr[col + v] = y[v];
  }
};

// Gather bound: every entry reads 4 F bytes of W from L2 or beyond.  With
// one lane per column and one entry at a time a narrow row (F = 16 ... 64)
// left most lanes idle or moved 4 bytes a lane; L lanes of 16 bytes keep the
// loads wide and 64 / L entries side by side.  Blocks [0, hblocks) do the
// heavy rows: block b scans groups of hrows rows for them and takes column block
// b mod hcb (64 columns) with all eight wavefronts, so that a hub row's time is divided
// by 8 * hcb and runs beside the light rows instead of after them.  Measured
// on symmetric R-MAT graphs against a column per lane with the heavy rows in
// a launch of their own: 1 M rows, 17.1 M entries, F = 256: 3.65 -> 2.05 ms
// (8.5 TB/s of gathered rows); 150 K rows, 2.1 M entries, F = 41: 351 -> 81 us.
template <typename RP, int L, int V>
__global__ __launch_bounds__(SPMM_BLOCK, 6) void k_spmm_rows(const void* arp, const int32_t* acol, const float* aval,
                                                              int64_t m, const float* W, int64_t ldw, int F, float* Y,
                                                              int64_t ldy, int relu, unsigned hblocks, unsigned hcb,
                                                              int hrows, int64_t heavy, unsigned ncb, int cw) {
  constexpr int NWV = SPMM_BLOCK / WAVE;
  constexpr int LH = L < 16 ? L : 16;  // heavy rows: lanes per entry
  constexpr int HC = LH * V;           // and columns of a block
  __shared__ float part[NWV - 1][HC];
  __shared__ int32_t found[SPMM_BLOCK];
  __shared__ int nfound;
  const int lane = threadIdx.x % WAVE;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  if (blockIdx.x < hblocks) {
    const int cb = (int)(blockIdx.x % hcb) * HC, ce = cb + HC < F ? cb + HC : F;
    for (int64_t r0 = (int64_t)(blockIdx.x / hcb) * hrows; r0 < m; r0 += (int64_t)(hblocks / hcb) * hrows) {
      if (threadIdx.x == 0) nfound = 0;
      __syncthreads();
      const int64_t mine = r0 + threadIdx.x;
      if ((int)threadIdx.x < hrows && mine < m && rp_at<RP>(arp, mine + 1) - rp_at<RP>(arp, mine) > heavy)
        found[atomicAdd(&nfound, 1)] = (int32_t)threadIdx.x;
      __syncthreads();
      const int n = nfound;
      for (int x = 0; x < n; ++x) {
        const int64_t row = r0 + found[x];
        const int64_t p0 = rp_at<RP>(arp, row), p1 = rp_at<RP>(arp, row + 1);
        RowPart<LH, V> r;
        r.start(cb, ce);
        // 64 entries at a time, the wavefronts in turn
        for (int64_t p = p0 + wv * WAVE; p < p1; p += NWV * WAVE) {
          const int cnt = (int)(p1 - p < WAVE ? p1 - p : WAVE);
          const int64_t q = p + (lane < cnt ? lane : cnt - 1);
          r.batch(acol[q], aval[q], cnt, W, ldw);
        }
        r.combine_groups();
        if (wv > 0 && lane < LH)
#pragma unroll
          for (int v = 0; v < V; ++v) part[wv - 1][lane * V + v] = r.acc[v];
        __syncthreads();
        if (wv == 0) {
          if (lane < LH)
#pragma unroll
            for (int i = 0; i < NWV - 1; ++i)
#pragma unroll
              for (int v = 0; v < V; ++v) r.acc[v] += part[i][lane * V + v];
          r.store(Y + row * ldy, cb, ce, relu);
        }
        __syncthreads();
      }
    }
    return;
  }
  // light rows, a wavefront per row and column block; the next row's first
  // entries and the row pointers of the one after it are in flight while a
  // row is added up
  const unsigned b = blockIdx.x - hblocks;  // hblocks and the light blocks are multiples of NXCD
  const unsigned nside = NXCD / (ncb < NXCD ? ncb : NXCD);
  const unsigned x = b % NXCD;
  const int64_t nw = (int64_t)((gridDim.x - hblocks) / NXCD) * nside * NWV;
  const int64_t row0 = ((int64_t)(b / NXCD) * nside + x / (NXCD / nside)) * NWV + wv;
  if (row0 >= m) return;
  auto entries = [&](int64_t p0, int64_t p1, int& k, float& a) {
    k = 0;
    a = 0.f;
    if (p0 + lane < p1) {
      k = acol[p0 + lane];
      a = aval[p0 + lane];
    }
  };
  for (unsigned c = x % (NXCD / nside); c < ncb; c += NXCD) {
    const int cb = (int)c * cw, ce = cb + cw < F ? cb + cw : F;
    int64_t row = row0;
    int64_t p0 = rp_at<RP>(arp, row), p1 = rp_at<RP>(arp, row + 1);
    int64_t q0 = 0, q1 = 0;
    if (row + nw < m) {
      q0 = rp_at<RP>(arp, row + nw);
      q1 = rp_at<RP>(arp, row + nw + 1);
    }
    int kl;
    float al;
    entries(p0, p1, kl, al);
    for (; row < m; row += nw) {
      int kn;
      float an;
      entries(q0, q1, kn, an);
      int64_t s0 = 0, s1 = 0;
      if (row + 2 * nw < m) {
        s0 = rp_at<RP>(arp, row + 2 * nw);
        s1 = rp_at<RP>(arp, row + 2 * nw + 1);
      }
      if (p1 - p0 <= heavy) {
        RowPart<L, V> r;
        r.start(cb, ce);
        if (p1 > p0) r.batch(kl, al, (int)(p1 - p0 < WAVE ? p1 - p0 : WAVE), W, ldw);
        for (int64_t p = p0 + WAVE; p < p1; p += WAVE) {
          const int cnt = (int)(p1 - p < WAVE ? p1 - p : WAVE);
          int k2;
          float a2;
          entries(p, p1, k2, a2);
          r.batch(k2, a2, cnt, W, ldw);
        }
        r.combine_groups();
        r.store(Y + row * ldy, cb, ce, relu);
      }
      p0 = q0; p1 = q1; q0 = s0; q1 = s1;
      kl = kn; al = an;
    }
  }
}

// ---------------------------------------------------------------------------
// Dense tiles on the matrix cores.  When A is dense enough (the aggregated
// features of Eq. 3 typically are), reading one row of W per entry of A
// costs more than a dense product over the zeros: a workgroup takes a
// 64-row x 16*NT-column tile of Y, densifies A's rows 32 columns at a time
// into LDS, stages the matching 32 x 16*NT block of W (transposed, k
// contiguous), and accumulates with v_mfma_f32_32x32x2_f32 (it sustains a
// larger share of the fp32 matrix peak than the 16x16x4 form).  Each
// wavefront owns 32 rows and 8*NT columns (NT/4 blocks of 32) of the tile.
//
// k order: for an 8-wide block of k, lane l (h = l / 32, c = l % 32) reads
// k = 4h .. 4h+3 of its row (A) and of its column (W) as one 16-byte LDS
// load, and the four MFMA steps take those four k's in turn, so every
// product a_ik w_kj meets its partner in the same step.  Absent entries are
// zeros in the tile, and x + 0 * w = x exactly for finite w, so each
// element is still a sum of the row's own products.
//
// Pipeline: LDS holds two chunks.  While the wavefronts multiply chunk c
// from one buffer they write chunk c+1 (loaded during chunk c-1) into the
// other and issue the loads of chunk c+2, so one barrier per chunk
// suffices and the staging work interleaves with the MFMAs.  Every load
// goes through a buffer resource: out-of-range offsets read 0 without
// touching memory, so the loop body has no branches.
constexpr int DT_M = 64;        // rows per tile
constexpr int DT_K = 32;        // k per LDS chunk
constexpr int DT_BLOCK = 256;   // four wavefronts, 16 rows each
constexpr int DT_ENTRIES = DT_K / 4;  // four threads per row: one round of loads covers a chunk
constexpr int kOutOfRange = INT32_MIN;  // a buffer offset no resource here reaches (reads 0)

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Row layout of a tile chunk in LDS (element k of row r, DT_K per row).
// Padded: rows of DT_K + 4 floats, so the 16-byte operand reads of 16 rows
// fall on distinct banks; column DT_K of each row takes the entries of later
// chunks.  Swizzled (less LDS, used where it buys one more workgroup per
// CU): unpadded rows whose 16-byte groups are permuted by the row's low
// three bits, so eight consecutive rows' reads of one group fall on
// distinct banks; one dump slot per row after the rows.
template <bool SWZ>
struct TileLayout {
  static constexpr int S = SWZ ? DT_K : DT_K + 4;                // floats per row
  static constexpr int A_FLOATS = SWZ ? DT_M * DT_K + DT_M : DT_M * S;
  __device__ static __forceinline__ int at(int r, int k) {
    if constexpr (SWZ) return r * DT_K + ((((k >> 2) ^ (r & 7)) << 2) | (k & 3));
    else return r * S + k;
  }
  __device__ static __forceinline__ int dump(int r) { return SWZ ? DT_M * DT_K + r : r * S + DT_K; }
};

// a wavefront-uniform 64-bit value in scalar registers
__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// raw buffer over `bytes` bytes (gfx9 resource word 3: 32-bit data format)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Occupancy is LDS-bound (two chunks per workgroup): four workgroups per CU
// at NT = 4, three at NT = 8; the register budget is set to match.
template <typename RP, int NT, bool VEC, bool RELU>
__global__ __launch_bounds__(DT_BLOCK, NT > 4 ? 3 : 4) void k_spmm_dense(
    const void* arp, const int32_t* acol, const float* aval, int64_t m, int K, const float* W, int64_t ldw, int F,
    float* Y, int64_t ldy, int64_t nrt, int64_t nct, int64_t ntiles) {
  constexpr int BN = 16 * NT;
  constexpr int WL = NT / 2;  // 16-byte W loads per thread per chunk (32 x BN floats over 256 threads)
  using L = TileLayout<(NT > 4)>;
  __shared__ __align__(16) float As[2][L::A_FLOATS];  // [row][k]
  __shared__ __align__(16) float Wt[2][BN * L::S];    // [column][k]
  constexpr int NB = BN / 64;  // 32-column MFMA blocks per wavefront
  const int t = threadIdx.x, lane = t % WAVE, wv = t / WAVE;
  const int r = t / 4, q = t % 4;             // densify: four threads per row
  const int h = lane / 32, c = lane % 32;     // MFMA operand position
  const int mr = 32 * (wv >> 1), mc = (wv & 1) * (BN / 2);  // the wavefront's rows and columns
  // W staging: the thread takes row wk of the chunk and, for e < WL, the
  // columns wc + 16e .. +3; a row's 64 bytes come from four lanes, and the
  // transposed LDS stores of a wavefront hit 64 distinct banks.
  const int wk = lane % 16 + 16 * (wv & 1);
  const int wc = (wv >> 1) * (BN / 2) + 4 * (lane / 16);
  const int nch = (K + DT_K - 1) / DT_K;
  // The grid is a multiple of 8 blocks, so a block's tiles all have its
  // index mod 8 and stay on its XCD; the column tiles of one row tile are
  // consecutive there and share A's entries through that XCD's L2.
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t x = tile % NXCD, i = tile / NXCD;
    const int64_t rt = (i / nct) * NXCD + x, ct = i % nct;
    if (rt >= nrt) continue;  // uniform over the workgroup
    const int64_t row0 = rt * DT_M;
    const int n0 = (int)ct * BN;
    // A's entries of the tile (< 2^26 of them: K <= 2^20), positions relative to e0
    const int64_t e0 = uniform64(rp_at<RP>(arp, row0));
    const int64_t e1 = uniform64(rp_at<RP>(arp, row0 + DT_M < m ? row0 + DT_M : m));
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(acol + e0, 4 * (e1 - e0));
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(aval + e0, 4 * (e1 - e0));
    // the row's entries as tile-local positions [cur, p1)
    int cur = 0, p1 = 0;
    if (row0 + r < m) {
      cur = (int)(rp_at<RP>(arp, row0 + r) - e0);
      p1 = (int)(rp_at<RP>(arp, row0 + r + 1) - e0);
    }
    int kc[DT_ENTRIES];
    float kv[DT_ENTRIES];
    int nval = 0;  // kc[e] belongs to the row while 4e < nval
    f32x4 w[WL];
    // the row's next 32 entries; nothing here waits for the loads
    auto load_entries = [&]() {
      nval = p1 - cur - q;  // entries of the row at or after this thread's first
      const int off = 4 * (cur + q);
#pragma unroll
      for (int e = 0; e < DT_ENTRIES; ++e) {
        kc[e] = __builtin_amdgcn_raw_buffer_load_b32(rc, off + 16 * e, 0, 0);
        kv[e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rv, off + 16 * e, 0, 0));
      }
    };
    // this thread's share of rows k0 .. k0+32 of W[:, n0 .. n0+BN): rows
    // past K are outside the resource, columns past F get an out-of-range
    // offset, so both read as zeros (F <= ldw < 2^23 keeps offsets in int)
    auto load_w = [&](int k0) {
      const int rows = K - k0 < DT_K ? (K - k0 > 0 ? K - k0 : 0) : DT_K;
      const __amdgpu_buffer_rsrc_t rw = make_rsrc(W + (int64_t)k0 * ldw + n0, 4 * (int64_t)rows * ldw);
#pragma unroll
      for (int e = 0; e < WL; ++e) {
        const int n = wc + 16 * e;  // column within the tile
        const int base = 4 * (wk * (int)ldw + n);
        if constexpr (VEC) {
          // n0 + n, F and ldw are multiples of 4: the 16 bytes are all
          // columns below F or all past it
          w[e] = __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, n0 + n < F ? base : kOutOfRange, 0, 0));
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            w[e][u] = __int_as_float(
                __builtin_amdgcn_raw_buffer_load_b32(rw, n0 + n + u < F ? base + 4 * u : kOutOfRange, 0, 0));
        }
      }
    };
    // chunk k0 from the registers into LDS buffer b, in two parts.
    // A: zero this thread's quarter of its row; the scatter runs in the same
    // wavefront after it, and LDS executes a wavefront's accesses in order.
    // 32 entries cover the 32 columns: every entry of the row in the chunk is
    // here.  Each is stored; one of a later chunk lands in the row's dump
    // slot, which the products never read.
    auto write_a = [&](int b, int k0) {
#pragma unroll
      for (int e = 0; e < DT_K / 16; ++e)
        *reinterpret_cast<f32x4*>(&As[b][L::at(r, q * (DT_K / 4) + 4 * e)]) = f32x4{0.f, 0.f, 0.f, 0.f};
      int n_in = 0;
#pragma unroll
      for (int e = 0; e < DT_ENTRIES; ++e) {
        // a canonical row has no column below k0 left, so this is kc < kend
        const bool in = 4 * e < nval && (unsigned)(kc[e] - k0) < (unsigned)DT_K;
        As[b][in ? L::at(r, kc[e] - k0) : L::dump(r)] = kv[e];
        n_in += in;
      }
      n_in += __shfl_xor(n_in, 1);
      n_in += __shfl_xor(n_in, 2);
      cur += n_in;
    };
    auto write_w = [&](int b, int e0, int e1) {
#pragma unroll
      for (int e = e0; e < e1; ++e)
#pragma unroll
        for (int u = 0; u < 4; ++u) Wt[b][L::at(wc + 16 * e + u, wk)] = w[e][u];
    };
    f32x16 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    if (nch > 0) {
      load_entries();
      load_w(0);
      write_w(0, 0, WL);
      write_a(0, 0);
      load_entries();
      load_w(DT_K);
      __syncthreads();
    }
    for (int ch = 0; ch < nch; ++ch) {
      const int b = ch & 1;
#pragma unroll
      for (int kb = 0; kb < DT_K; kb += 8) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(&As[b][L::at(mr + c, kb + 4 * h)]);
        f32x4 bw[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
          bw[j] = *reinterpret_cast<const f32x4*>(&Wt[b][L::at(mc + 32 * j + c, kb + 4 * h)]);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s], bw[j][s], acc[j], 0, 0, 0);
        // chunk ch+1 into the other buffer (read last in chunk ch-1, before
        // the barrier), then the loads of chunk ch+2.  Past the last chunk
        // both are harmless: the rows are exhausted and W's rows are out of
        // range.  128-column tiles do this in parts between the products of
        // the chunk's four k blocks, so that a wavefront's own staging runs
        // under its products; with 64-column tiles, whose four workgroups per
        // CU cover it, it comes after them (262144 x 512, parts / after:
        // F = 256 701 / 715 us, F = 512 1365 / 1393, F = 64 237 / 221).
        if constexpr (NT > 4) {
          if (kb == 0) {
            write_a(b ^ 1, (ch + 1) * DT_K);
            load_entries();
          } else if (kb == 8) {
            write_w(b ^ 1, 0, WL / 2);
          } else if (kb == 16) {
            write_w(b ^ 1, WL / 2, WL);
            load_w((ch + 2) * DT_K);
          }
        }
      }
      if constexpr (NT <= 4) {
        write_w(b ^ 1, 0, WL);
        write_a(b ^ 1, (ch + 1) * DT_K);
        load_entries();
        load_w((ch + 2) * DT_K);
      }
      __syncthreads();
    }
    // register v of block j holds row 8(v/4) + 4h + v%4 of the wavefront's
    // 32, column c of the block
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int col = n0 + mc + 32 * j + c;
      if (col >= F) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = row0 + mr + 8 * (v / 4) + 4 * h + v % 4;
        if (row < m) Y[row * ldy + col] = RELU ? fmaxf(acc[j][v], 0.f) : acc[j][v];
      }
    }
  }
}

template <typename RP, int L, int V>
hipError_t spmm_t(int relu, const void* arp, const int32_t* acol, const float* aval, int64_t m, int64_t nnz,
                  const float* W, int64_t ldw, int F, float* Y, int64_t ldy, int64_t ncb, hipStream_t s) {
  constexpr int NWV = SPMM_BLOCK / WAVE;
  const int cw = (int)(((F + V - 1) / V + ncb - 1) / ncb * V);
  constexpr int HC = (L < 16 ? L : 16) * V;
  const int64_t hcb = (F + HC - 1) / HC;
  const int64_t heavy = std::max(kHeavy, std::min(2 * (nnz / m), nnz * ncb / kHeavyShare));
  int64_t hx = (m + SPMM_BLOCK - 1) / SPMM_BLOCK;
  if (hcb < 4 || nnz >= kHeavyMean * m)
    hx = std::max(hx, std::min({m, nnz / kHeavyGroup, kHeavyGroups, 4 * kHeavyGroups / hcb}));
  hx = std::min(hx, hcb < 512 ? 4096 / hcb : 8);
  hx = (hx + NXCD - 1) / NXCD * NXCD;
  int hrows = (int)std::min<int64_t>(SPMM_BLOCK, (m + hx - 1) / hx);
  if (hrows > SPMM_BLOCK / 2) hrows = SPMM_BLOCK;
  const int64_t hblocks = hx * hcb;
  const int64_t nside = NXCD / (ncb < NXCD ? ncb : NXCD);
  int64_t g = (m + nside * NWV - 1) / (nside * NWV);
  if (g > 512) g = 512;
  hipLaunchKernelGGL((k_spmm_rows<RP, L, V>), dim3((unsigned)(hblocks + g * NXCD)), dim3(SPMM_BLOCK), 0, s, arp, acol,
                     aval, m, W, ldw, F, Y, ldy, relu, (unsigned)hblocks, (unsigned)hcb, hrows, heavy,
                     (unsigned)ncb, cw);
  return hipGetLastError();
}

template <typename RP>
hipError_t spmm_rp(int relu, const void* arp, const int32_t* acol, const float* aval, int64_t m, int64_t nnz,
                   const float* W, int64_t ldw, int F, float* Y, int64_t ldy, hipStream_t s) {
  if (F < 4) return spmm_t<RP, 4, 1>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, 1, s);
  // Column blocks of at most 64 vectors, a power of two of them up to the
  // number of XCDs (each XCD then gathers from a part of W's columns), and
  // two where both halves of a row are whole cache lines (1 M rows, F = 256:
  // 2.14 -> 2.06 ms); halves that share lines cost more than they save
  // (150 K rows, F = 200: 222 against 236 us), as do blocks below 128 columns.
  const int64_t vec = (F + 3) / 4;
  const bool lines = F > 128 && F % 64 == 0 && ldw % 32 == 0 && reinterpret_cast<uintptr_t>(W) % 128 == 0;
  int64_t ncb = lines ? 2 : 1;
  while (ncb < NXCD && vec > ncb * 64) ncb *= 2;
  if (vec > ncb * 64) ncb = (vec + 63) / 64;
  const int64_t cv = (vec + ncb - 1) / ncb;
  if (cv <= 2) return spmm_t<RP, 2, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
  if (cv <= 4) return spmm_t<RP, 4, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
  if (cv <= 8) return spmm_t<RP, 8, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
  if (cv <= 16) return spmm_t<RP, 16, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
  if (cv <= 32) return spmm_t<RP, 32, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
  return spmm_t<RP, 64, 4>(relu, arp, acol, aval, m, nnz, W, ldw, F, Y, ldy, ncb, s);
}

template <typename RP, int NT, bool VEC>
hipError_t dense_t(int relu, const void* arp, const int32_t* acol, const float* aval, int64_t m, int K,
                   const float* W, int64_t ldw, int F, float* Y, int64_t ldy, hipStream_t s) {
  const int64_t nrt = (m + DT_M - 1) / DT_M, nct = (F + 16 * NT - 1) / (16 * NT);
  const int64_t ntiles = (nrt + NXCD - 1) / NXCD * NXCD * nct;  // a multiple of NXCD
  const int64_t grid = ntiles < 65536 ? ntiles : 65536;          // so is this
  if (relu)
    hipLaunchKernelGGL((k_spmm_dense<RP, NT, VEC, true>), dim3((unsigned)grid), dim3(DT_BLOCK), 0, s, arp, acol,
                       aval, m, K, W, ldw, F, Y, ldy, nrt, nct, ntiles);
  else
    hipLaunchKernelGGL((k_spmm_dense<RP, NT, VEC, false>), dim3((unsigned)grid), dim3(DT_BLOCK), 0, s, arp, acol,
                       aval, m, K, W, ldw, F, Y, ldy, nrt, nct, ntiles);
  return hipGetLastError();
}

template <typename RP>
hipError_t dense_rp(int relu, const void* arp, const int32_t* acol, const float* aval, int64_t m, int K,
                    const float* W, int64_t ldw, int F, float* Y, int64_t ldy, hipStream_t s) {
  const bool vec = ldw % 4 == 0 && F % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0;
  if (F > 64)
    return vec ? dense_t<RP, 8, true>(relu, arp, acol, aval, m, K, W, ldw, F, Y, ldy, s)
               : dense_t<RP, 8, false>(relu, arp, acol, aval, m, K, W, ldw, F, Y, ldy, s);
  return vec ? dense_t<RP, 4, true>(relu, arp, acol, aval, m, K, W, ldw, F, Y, ldy, s)
             : dense_t<RP, 4, false>(relu, arp, acol, aval, m, K, W, ldw, F, Y, ldy, s);
}

}  // namespace

bool spmm_dense_fits(int64_t K, int64_t ldw) {
  return K >= 0 && K <= (int64_t(1) << 20) && ldw < (int64_t(1) << 23);
}

hipError_t spmm(const void* arp, int rpa64, const int32_t* acol, const float* aval, int64_t m, int64_t K, int64_t nnz,
                const float* W, int64_t ldw, int64_t F, float* Y, int64_t ldy, int relu, int dense, hipStream_t s) {
  if (m <= 0 || F <= 0) return hipSuccess;
  if (dense) {
    if (!spmm_dense_fits(K, ldw)) return hipErrorInvalidValue;
    return rpa64 ? dense_rp<int64_t>(relu, arp, acol, aval, m, (int)K, W, ldw, (int)F, Y, ldy, s)
                 : dense_rp<int32_t>(relu, arp, acol, aval, m, (int)K, W, ldw, (int)F, Y, ldy, s);
  }
  // a launch takes at most kMaxCols columns: its workgroups for heavy rows, eight
  // or more to 64 columns, stay far below the 2^32 threads that a launch holds
  // and column numbers past the end of a row below the largest int
  hipError_t e = hipSuccess;
  for (int64_t f0 = 0; f0 < F && e == hipSuccess; f0 += kMaxCols) {
    const int f = (int)std::min(F - f0, kMaxCols);
    e = rpa64 ? spmm_rp<int64_t>(relu, arp, acol, aval, m, nnz, W ? W + f0 : W, ldw, f, Y + f0, ldy, s)
              : spmm_rp<int32_t>(relu, arp, acol, aval, m, nnz, W ? W + f0 : W, ldw, f, Y + f0, ldy, s);
  }
  return e;
}

}  // namespace kern
}  // namespace aires
