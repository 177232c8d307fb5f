// kernels_mix.hip -- the stochastic reduce (Appendix A, update equation
// (A.2), second line): W'[i] = sum_{j in N_in(i)} P_ij W[j].
//
// The reduce is a low fan-in streaming product: every output element is
// deg+1 fused multiply-adds over rows that are each read by deg+1 outputs.
// It is bound by HBM bandwidth (arithmetic intensity < 1 flop/byte), so MFMA
// has no role here.  What matters is that every model byte crosses HBM once.
//
// slab kernel (n a power of two in [8, 1024], rows of at most 17 entries):
// each workgroup owns a contiguous range of column chunks; a chunk holds all
// n rows of a column range, sized so that it holds a whole 128-byte line of
// every row (128 KiB above 512 rows, 64 KiB above 256, else 32 KiB), and is
// staged in LDS, so each neighbour re-read is an LDS read.  The loads of the
// next chunk (two below 1024 rows) are in flight while one is computed.  A
// thread keeps the neighbour lists of its output rows in registers (two
// weights per row when all of a row's entries but its own share one weight).
// LDS slots of a row are XOR-swizzled by the row's low bits so that lanes
// reading random rows spread over the banks.  Results are transposed across
// groups of 8 lanes (DPP) so that each store writes a whole 128-byte line of
// a row rather than 16 bytes in each of 64 rows.
//
// column kernel (other graphs of up to 1024 workers, but for the sizes that
// launch_mix_cols names): a workgroup takes all n rows of a narrow column range
// through LDS, see mix_cols_kernel.
//
// tile kernel (n above 1024 and what the column kernel leaves): a tile is one
// 1 KiB segment of 16 consecutive output rows, one wave per row segment with
// 16-byte loads; the tiles of one column range go to one XCD so that re-reads of
// a neighbour's segment hit its L2.
//
// Precision: the slab kernel accumulates its at most 17 terms with fp32
// fused multiply-adds (error below 17 ulp of sum_j |P_ij w_j|); the tile and
// mean kernels take rows of any length (a hub, the complete graph) and
// accumulate in fp64, rounding once.
//
// NOTIFY-ACK (Section 4) on one device: a row is reduced only if every
// in-neighbour carries the tag "published in this round" in buffer e; a row
// with a stale neighbour is not reduced and the mismatch is counted in the
// device error words.  Rows that are reduced get the next round's tag in buffer
// e^1.  The column kernel and the slab kernel's narrow variants read the tags
// themselves; for the 17-entry slab variant and the tile kernel a small kernel
// ahead of them (the WAIT) records the verdict in row_ok.
#include "asap_launch.h"

namespace asap {
namespace {

constexpr int kSegFloats = 256;  // one wave x float4
constexpr int kTileRows = 16;
constexpr int kMixThreads = 256;

// Blocks are dealt round-robin to the 8 XCDs (blockIdx % 8).  Give XCD x the
// contiguous tile range [x*T/8, (x+1)*T/8) so that consecutive tiles of a
// column range stay in one L2.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t bid, uint32_t total) {
  if (total % 8u) return bid;
  return (bid % 8u) * (total / 8u) + bid / 8u;
}

// Non-temporal 16-byte accesses, for data a reduce reads or writes exactly
// once (the slab kernel's staging loads and result stores): 4-5% faster
// than plain accesses for 1024 x 2^20 models.
typedef float nt4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ld_nt(const float4* p) {
  const nt4 x = __builtin_nontemporal_load(reinterpret_cast<const nt4*>(p));
  return make_float4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ void st_nt(float4* p, const float4& v) {
  const nt4 x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, reinterpret_cast<nt4*>(p));
}

__device__ __forceinline__ void fma4(float4& acc, float w, const float4& x) {
  acc.x = fmaf(w, x.x, acc.x);
  acc.y = fmaf(w, x.y, acc.y);
  acc.z = fmaf(w, x.z, acc.z);
  acc.w = fmaf(w, x.w, acc.w);
}

// fp64 accumulator of one float4 slot: rows of any length (the tile and mean
// kernels) sum without fp32 error growth; the result is rounded once
struct Acc4 {
  double x = 0.0, y = 0.0, z = 0.0, w = 0.0;
  __device__ void fma(double wt, const float4& v) {
    x = ::fma(wt, double(v.x), x);
    y = ::fma(wt, double(v.y), y);
    z = ::fma(wt, double(v.z), z);
    w = ::fma(wt, double(v.w), w);
  }
  __device__ float4 round() const { return make_float4(float(x), float(y), float(z), float(w)); }
};

__device__ __forceinline__ void store_tail(float* d, const float4& v, int64_t c, int64_t dim) {
  if (c + 4 <= dim) {
    *reinterpret_cast<float4*>(d) = v;
  } else {
    d[0] = v.x;
    if (c + 1 < dim) d[1] = v.y;
    if (c + 2 < dim) d[2] = v.z;
  }
}

// NOTIFY-ACK: whether every in-neighbour of a row carries the tag "published
// in this round"; a row for which it does not is not reduced.  Every block of
// the slab and column kernels checks the rows it needs itself, beside its
// first loads (a launch of its own cost 4-6 us a reduce); one block reports.
__device__ __forceinline__ bool row_published(const MixArgs& a, int row) {
  bool ok = true;
  for (int p = a.nbr_ptr[row], p1 = a.nbr_ptr[row + 1]; p < p1; p += 4) {
    int j[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) j[u] = a.nbr_idx[min(p + u, p1 - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) ok &= a.tag_src[j[u]] == a.expect;
  }
  return ok;
}
__device__ __forceinline__ void report_stale(const MixArgs& a, int row) {
  atomicAdd(&a.err[kErrEpochCount], 1);
  atomicMin(&a.err[kErrEpochWorker], row);
}

// The same as a launch of its own, one wave per row, for the tile kernel (more
// rows than a block can check) and the slab kernel's longest rows.
__global__ __launch_bounds__(64) void epoch_check_kernel(MixArgs a) {
  const int r = int(blockIdx.x), lane = int(threadIdx.x);
  const int p0 = a.nbr_ptr[r], p1 = a.nbr_ptr[r + 1];
  int ok = 1;
  for (int p = p0 + lane; p < p1; p += 64) ok &= (a.tag_src[a.nbr_idx[p]] == a.expect);
  ok = __all(ok);
  if (lane == 0) {
    a.row_ok[r] = ok;
    if (!ok) report_stale(a, r);
  }
}

__global__ __launch_bounds__(kMixThreads) void mix_kernel(MixArgs a, uint32_t nseg, uint32_t nrg) {
  const uint32_t tile = xcd_tile(blockIdx.x, nseg * nrg);
  const uint32_t seg = tile / nrg, rg = tile % nrg;
  const int row0 = int(rg) * kTileRows;
  const int row1 = min(row0 + kTileRows, a.n);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t c = int64_t(seg) * kSegFloats + lane * 4;
  for (int r = row0 + wave; r < row1; r += kMixThreads / 64) {
    if (!a.row_ok[r]) continue;
    if (c < a.dim) {
      Acc4 acc;
      const int p0 = a.nbr_ptr[r], p1 = a.nbr_ptr[r + 1];
      for (int p = p0; p < p1; ++p) {
        const int j = a.nbr_idx[p];
        double wt = a.nbr_w[p];
        if (a.scale) wt *= double(a.scale[j]);
        acc.fma(wt, *reinterpret_cast<const float4*>(a.src + int64_t(j) * a.ld + c));
      }
      store_tail(a.dst + int64_t(r) * a.ld + c, acc.round(), c, a.dim);
    }
    if (seg == 0 && lane == 0) a.tag_dst[r] = a.next;
  }
}

// Barrier that orders LDS only: global loads stay in flight across it, and
// global stores need not have landed.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Column kernel: any graph of up to 1024 workers that the slab kernel does not
// take.  A block walks a contiguous range of column chunks; a chunk is all n
// rows of 4 LPR columns (LPR lanes of a float4 each per row: 64 up to 128
// rows, then 32, 16, 8, so that a chunk is at most 128 KiB, and fewer where
// there are few columns, see launch_mix_cols), staged in LDS, so
// every model byte crosses HBM once and a neighbour is an LDS read.  Thread t
// stages and computes float4 slots t + T m of the chunk (m < PF): slot s is
// float4 s mod LPR of row s div LPR.  The loads of the next chunk are in
// flight while one is computed, so nothing else may be loaded through the
// vector path meanwhile (loads complete in order: a list entry would wait for
// the chunk): with LPR = 64 a wave has one row at a time and its list comes
// through the scalar cache, otherwise the lists are in LDS behind the chunk
// (graphs whose lists do not fit there run the tile kernel).  Sums run in fp64 in row order,
// rounded once, as in the tile kernel, which re-read every neighbour through
// the L2 with one load in flight per wave: 25 x 11000003, root expander, 0.908
// -> 0.456 ms (4.8 TB/s); 6 x 11738470 0.209 -> 0.122; 100 x 500009, d = 6, 0.222
// -> 0.115; 300 x 500009, d = 4, 0.531 -> 0.309; 1000 x 300007, d = 4, 1.058 ->
// 0.641 ms.  Above 64 rows, where one block fills a compute unit, its 1024
// threads matter: with 512 the last three took 0.148, 0.427 and 1.058 ms.
constexpr int kColsMaxRows = 1024;
typedef const int32_t __attribute__((address_space(4))) * ConstI32;
typedef const float __attribute__((address_space(4))) * ConstF32;

template <int LPR, int PF>
__global__ __launch_bounds__(1024) void mix_cols_kernel(MixArgs a, int nchunks) {
  extern __shared__ float4 chunk[];  // [n][LPR], then (LPR < 64) the lists
  const int nnz = LPR < 64 ? a.nbr_ptr[a.n] : 0;
  float* lw = reinterpret_cast<float*>(chunk + a.n * LPR);       // [nnz] weights
  float* lscale = lw + nnz;                                      // [n] scales, if any
  uint16_t* lptr = reinterpret_cast<uint16_t*>(lscale + (a.scale ? a.n : 0));  // [n + 1]
  uint16_t* lidx = lptr + a.n + 1;                               // [nnz]
  __shared__ uint32_t okw[kColsMaxRows / 32];
  const int T = int(blockDim.x), tid = int(threadIdx.x), n = a.n;
  const int q = tid % LPR, r0 = tid / LPR, rstep = T / LPR;
  constexpr int C = 4 * LPR;
  const int per = (nchunks + int(gridDim.x) - 1) / int(gridDim.x);
  const int ch0 = int(blockIdx.x) * per, ch1 = min(nchunks, ch0 + per);
  auto load = [&](float4 (&buf)[PF], int ch) {
    const int64_t c = int64_t(ch) * C + 4 * q;
    const bool in = ch < ch1 && c < a.dim;
#pragma unroll
    for (int m = 0; m < PF; ++m) {
      const int r = r0 + m * rstep;
      if (in && r < n) buf[m] = ld_nt(reinterpret_cast<const float4*>(a.src + int64_t(r) * a.ld + c));
    }
  };
  float4 buf[PF];
#pragma unroll
  for (int m = 0; m < PF; ++m) buf[m] = make_float4(0.f, 0.f, 0.f, 0.f);
  load(buf, ch0);
  for (int k = tid; k < kColsMaxRows / 32; k += T) okw[k] = 0u;
  if constexpr (LPR < 64) {
    for (int p = tid; p < nnz; p += T) {
      lw[p] = a.nbr_w[p];
      lidx[p] = uint16_t(a.nbr_idx[p]);
    }
    for (int r = tid; r <= n; r += T) {
      lptr[r] = uint16_t(a.nbr_ptr[r]);
      if (a.scale && r < n) lscale[r] = a.scale[r];
    }
  }
  __syncthreads();
  for (int r = tid; r < n; r += T) {
    if (row_published(a, r))
      atomicOr(&okw[r >> 5], 1u << (r & 31));
    else if (blockIdx.x == 0)
      report_stale(a, r);
  }
  for (int ch = ch0; ch < ch1; ++ch) {
    lds_barrier();  // the previous chunk is no longer read (and the verdicts are there)
#pragma unroll
    for (int m = 0; m < PF; ++m)
      if (r0 + m * rstep < n) chunk[tid + m * T] = buf[m];
    lds_barrier();
    load(buf, ch + 1);
    const int64_t c = int64_t(ch) * C + 4 * q;
#pragma unroll 1
    for (int m = 0; m < PF; ++m) {
      const int rl = r0 + m * rstep, r = LPR == 64 ? __builtin_amdgcn_readfirstlane(rl) : rl;
      if (r >= n || c >= a.dim || !((okw[r >> 5] >> (r & 31)) & 1u)) continue;
      Acc4 acc;
      int p0, p1;
      if constexpr (LPR == 64) {
        p0 = ((ConstI32)(uintptr_t)a.nbr_ptr)[r];
        p1 = ((ConstI32)(uintptr_t)a.nbr_ptr)[r + 1];
      } else {
        p0 = lptr[r];
        p1 = lptr[r + 1];
      }
      // four entries at a time: their reads are issued before the first sum
      for (int p = p0; p < p1; p += 4) {
        float4 x[4];
        double wt[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int pu = min(p + u, p1 - 1);
          int j;
          if constexpr (LPR == 64) {
            j = ((ConstI32)(uintptr_t)a.nbr_idx)[pu];
            wt[u] = ((ConstF32)(uintptr_t)a.nbr_w)[pu];
            if (a.scale) wt[u] *= double(((ConstF32)(uintptr_t)a.scale)[j]);
          } else {
            j = lidx[pu];
            wt[u] = lw[pu];
            if (a.scale) wt[u] *= double(lscale[j]);
          }
          x[u] = chunk[j * LPR + q];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (p + u < p1) acc.fma(wt[u], x[u]);
      }
      const float4 v = acc.round();
      float* d = a.dst + int64_t(r) * a.ld + c;
      if (c + 4 <= a.dim)
        st_nt(reinterpret_cast<float4*>(d), v);
      else
        store_tail(d, v, c, a.dim);
    }
  }
  if (blockIdx.x == 0)
    for (int r = tid; r < n; r += T)
      if ((okw[r >> 5] >> (r & 31)) & 1u) a.tag_dst[r] = a.next;
}

// Complete graph with uniform weights (all-reduce, Figure 2a): every output
// row is the same weighted column sum, so compute it once per column and
// broadcast it: n reads and n writes per column instead of n^2 reads.  The
// sum runs over j ascending with the same fp64 fused multiply-adds as
// mix_kernel, so both kernels produce identical bits on this graph.  On the
// complete graph one stale worker makes every row stale.
__global__ __launch_bounds__(64) void mean_kernel(MixArgs a, uint32_t nseg) {
  const uint32_t seg = xcd_tile(blockIdx.x, nseg);
  const int lane = threadIdx.x;
  const int64_t c = int64_t(seg) * kSegFloats + lane * 4;
  // nothing waits for the tags before the rows are loading (with few workers the
  // wait was much of a wave's time: 1 x 2^24 48.4 -> 33.4 us, 3 x 2^24 147 -> 114)
  const int64_t tag = a.tag_src[min(lane, a.n - 1)];
  Acc4 acc;
  if (c < a.dim) {
    const double w0 = a.nbr_w[0];
    // 32 rows' loads in flight per wave (one wave per segment leaves few
    // waves on a CU): 256 workers x 2^18 beside the next round's planning,
    // 0.32 -> 0.24 ms; the order of the sum is unchanged
#pragma unroll 32
    for (int j = 0; j < a.n; ++j) {
      double wt = w0;
      if (a.scale) wt *= double(a.scale[j]);
      acc.fma(wt, *reinterpret_cast<const float4*>(a.src + int64_t(j) * a.ld + c));
    }
  }
  int stale = tag != a.expect;
  for (int j = lane + 64; j < a.n; j += 64) stale |= a.tag_src[j] != a.expect;
  if (__ballot(stale) != 0ull) {
    if (seg == 0)
      for (int j = lane; j < a.n; j += 64) report_stale(a, j);
    return;
  }
  if (c < a.dim) {
    const float4 out = acc.round();
#pragma unroll 4
    for (int j = 0; j < a.n; ++j) store_tail(a.dst + int64_t(j) * a.ld + c, out, c, a.dim);
  }
  if (seg == 0)
    for (int j = lane; j < a.n; j += 64) a.tag_dst[j] = a.next;
}

constexpr int kOut = 8;                             // outputs transposed and stored together

// x of lane i ^ S (S = 1, 2, 4) by DPP moves: quad_perm [1,0,3,2] and
// [2,3,0,1] are the xor-1 and xor-2 exchanges; xor 4 is the mirror inside
// each 8-lane half-row (i -> i ^ 7) followed by quad_perm [3,2,1,0]
// (i -> i ^ 3).
template <int S>
__device__ __forceinline__ float xor_lane(float x) {
  int v = __builtin_bit_cast(int, x);
  if constexpr (S == 1) {
    v = __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
  } else if constexpr (S == 2) {
    v = __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
  } else {
    static_assert(S == 4, "xor_lane: S in {1, 2, 4}");
    v = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);
    v = __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, false);
  }
  return __builtin_bit_cast(float, v);
}

template <int S>
__device__ __forceinline__ float4 xor_lane4(const float4& x) {
  return make_float4(xor_lane<S>(x.x), xor_lane<S>(x.y), xor_lane<S>(x.z), xor_lane<S>(x.w));
}

__device__ __forceinline__ float4 sel4(bool c, const float4& a, const float4& b) {
  return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}

// v[k] of lane i <- v[i] of lane k, within aligned groups of 8 lanes:
// butterfly exchanges with the lanes i ^ s, s = 4, 2, 1.
template <int S>
__device__ __forceinline__ void transpose_stage(float4 (&v)[kOut], int lane_in) {
  const bool hi = lane_in & S;
#pragma unroll
  for (int k = 0; k < kOut; ++k) {
    if (k & S) continue;
    // a lane keeps the slot whose bit S matches its own and sends the other
    // (value selects only: a select of the slot to write would put v in
    // scratch memory)
    const float4 lo_v = v[k], hi_v = v[k | S];
    const float4 recv = xor_lane4<S>(sel4(hi, lo_v, hi_v));
    v[k] = sel4(hi, recv, lo_v);
    v[k | S] = sel4(hi, hi_v, recv);
  }
}

__device__ __forceinline__ void transpose8(float4 (&v)[kOut], int lane_in) {
  transpose_stage<4>(v, lane_in);
  transpose_stage<2>(v, lane_in);
  transpose_stage<1>(v, lane_in);
}

// 1 to 3 leading components of v (a row's ragged last float4)
__device__ __forceinline__ void store_partial(float* d, float4 v, int k) {
  d[0] = v.x;
  if (k > 1) d[1] = v.y;
  if (k > 2) d[2] = v.z;
}

// LDS reads in flight per thread
template <int DEG, int R> constexpr int slab_group() { return DEG <= 5 ? DEG : (R == 2 && DEG > 9 ? 1 : 4); }

// Slab kernel.  A THREADS-thread workgroup walks a contiguous
// range of column chunks; a chunk is all n rows of 4 VEC / n columns (VEC
// float4), staged in LDS.  Thread t stages float4 slots t + THREADS m of the
// chunk (m < VEC / THREADS); NBUF register buffers keep the loads of the
// next NBUF chunks in flight while one is computed.  Outputs: with R = 2
// (n = 2 THREADS) thread t computes rows t and t + THREADS, the whole chunk
// of each; with R = 1 row t mod n, VEC / THREADS float4 of it from
// (t div n) VEC / THREADS on.  Groups of 8 outputs of 8 consecutive lanes (8
// consecutive rows) are transposed across the lanes, so that each store
// instruction writes whole 128-byte lines: 8 lanes fill 128 contiguous
// bytes of one row.  With UNI every entry of a row but its own carries one
// weight, so a row keeps two weights instead of DEG.
template <int DEG, int R, int THREADS, int NBUF, int VEC, bool UNI>
__global__ __launch_bounds__(THREADS) void mix_slab_kernel(MixArgs a, int nchunks) {
  constexpr int kSlabThreads = THREADS;
  constexpr int kSlabVec = VEC;
  constexpr int kSlabPF = kSlabVec / THREADS;      // float4 staged per thread per chunk
  __shared__ float4 slab[kSlabVec];
  const int n = a.n;
  const int Q = kSlabVec / n;                // float4 per row per chunk (>= 8)
  const int C = 4 * Q;                       // columns per chunk
  const int X = min(Q, 8) - 1;               // swizzle mask
  const int tid = threadIdx.x;
  constexpr int OPR = kSlabPF / R;           // outputs per row per thread per chunk
  static_assert(OPR >= kOut && OPR % kOut == 0, "mix_slab_kernel: whole groups of transposed outputs");
  constexpr int G = slab_group<DEG, R>();
  constexpr bool kOwnCheck = DEG <= 9;
  // this thread's output rows and first float4
  int orow[R];
  int oq0;
  if constexpr (R == 2) {
    orow[0] = tid;
    orow[1] = tid + kSlabThreads;
    oq0 = 0;
  } else {
    orow[0] = tid % n;
    oq0 = (tid / n) * OPR;
  }
  const int per = (nchunks + int(gridDim.x) - 1) / int(gridDim.x);
  const int ch0 = int(blockIdx.x) * per, ch1 = min(nchunks, ch0 + per);

  // Staging: slot s = tid + THREADS m of a chunk is float4 s mod Q of row s div
  // Q.  The per-thread part of the address is a 32-bit byte offset below
  // 2^31 (the launcher checks it); the rest is wave-uniform.
  const int lq = __builtin_ctz(Q);
  const bool wideq = Q > kSlabThreads;       // n == 8: Q = 1024
  const int q0 = wideq ? tid : (tid & (Q - 1));
  const int r0 = wideq ? 0 : (tid >> lq);
  const uint32_t voff = (uint32_t(r0) * uint32_t(a.ld) + 4u * uint32_t(q0)) * 4u;
  auto srow = [&](int m) {                   // uniform row offset of slot m
    return wideq ? (m >> 1) : m * (kSlabThreads >> lq);
  };
  auto sq = [&](int m) {                     // uniform float4 offset of slot m
    return wideq ? (m & 1) * kSlabThreads : 0;
  };
  auto load = [&](float4 (&buf)[kSlabPF], int ch) {
    const bool live = ch < ch1;
    const int64_t off = int64_t(live ? ch : ch0) * C;
    // an empty asm makes voff opaque per chunk, so the compiler does not
    // hoist 16 64-bit row addresses out of the chunk loop
    uint32_t vo = voff;
    asm volatile("" : "+v"(vo));
#pragma unroll
    for (int m = 0; m < kSlabPF; ++m) {
      const bool in = live && off + 4 * (q0 + sq(m)) < a.dim;
      const char* base = reinterpret_cast<const char*>(a.src + off + int64_t(srow(m)) * a.ld + 4 * sq(m));
      buf[m] = in ? ld_nt(reinterpret_cast<const float4*>(base + vo)) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  // The first chunks' loads go out before the lists and tags are read; where the
  // lists leave no registers, after them, and after the verdicts' ballot, which
  // would wait for the rows (128 x 65536, d = 10: 41.8 us with the loads ahead of
  // it, 38.8 behind).
  float4 bufA[kSlabPF], bufB[NBUF == 2 ? kSlabPF : 1];
  auto first_loads = [&]() {
    load(bufA, ch0);
    if constexpr (NBUF == 2) load(bufB, ch0 + 1);
  };
  if constexpr (kOwnCheck) first_loads();
  // jq = j*Q | (j & X): the slot of float4 q of row j is jq ^ q, because
  // X < Q and Q is a power of two (see the staging writes below).
  // jq < n*Q = 8192, so two of them share a register.
  // Weights: with UNI every entry of a row but its own has one weight (the
  // launcher checked it bit for bit, and no scale applies), so a row keeps
  // (own weight, other weight, own position, length) and weight p is picked
  // by selects, the same value as the general table would give.
  uint32_t jq2[R][(DEG + 1) / 2];
  float nw[R][UNI ? 1 : DEG];
  float uw_self[R], uw_off[R];
  int upos[R], ulen[R];
  bool ok[R];
#pragma unroll
  for (int rr = 0; rr < R; ++rr) {
    const int row = orow[rr];
#pragma unroll
    for (int u = 0; u < (DEG + 1) / 2; ++u) jq2[rr][u] = 0u;
    const int p0 = a.nbr_ptr[row], deg = a.nbr_ptr[row + 1] - p0;
    uw_self[rr] = 0.f;
    uw_off[rr] = 0.f;
    upos[rr] = -1;
    ulen[rr] = deg;
    // NOTIFY-ACK: every in-neighbour carries this round's tag (rows of up to
    // 17 entries have no registers for that: 1024 x 2^18, d = 16, 664 -> 674
    // us with it, so the check stays a launch of its own there)
    ok[rr] = kOwnCheck || a.row_ok[row] != 0;
#pragma unroll
    for (int u = 0; u < DEG; ++u) {
      const bool has = u < deg;  // padding: own row, weight 0
      const int j = has ? a.nbr_idx[p0 + u] : row;
      float wt = has ? a.nbr_w[p0 + u] : 0.f;
      if (a.scale && has) wt *= a.scale[j];
      if constexpr (kOwnCheck) ok[rr] &= !has || a.tag_src[j] == a.expect;
      jq2[rr][u / 2] |= uint32_t(j * Q | (j & X)) << (16 * (u & 1));
      if constexpr (UNI) {
        if (has && j == row) {
          uw_self[rr] = wt;
          upos[rr] = u;
        } else if (has) {
          uw_off[rr] = wt;
        }
      } else {
        nw[rr][u] = wt;
      }
    }
  }
  if (kOwnCheck && blockIdx.x == 0) {
    const bool head = R == 2 || tid < n;
#pragma unroll
    for (int rr = 0; rr < R; ++rr)
      if (head && !ok[rr]) report_stale(a, orow[rr]);
  }
  auto stage = [&](const float4 (&buf)[kSlabPF]) {
#pragma unroll
    for (int m = 0; m < kSlabPF; ++m) {
      const int r = r0 + srow(m), q = q0 + sq(m);
      slab[(r * Q | (r & X)) ^ q] = buf[m];
    }
  };
  // Output float4 q of row rr of this thread from the staged chunk.  Padding
  // entries read the own row with weight 0, which adds an exact zero, so the
  // reads of a group issue back to back with no branches.
  // the state of the row being computed, copied out of the per-row arrays
  // by selects (a runtime row index into those arrays would put them in
  // scratch memory)
  uint32_t jl[(DEG + 1) / 2];
  float nl[UNI ? 1 : DEG];
  float ls_self = 0.f, ls_off = 0.f;
  int lpos = 0, llen = 0;
  auto select_row = [&](int rr) {
    const bool second = R == 2 && rr == 1;
#pragma unroll
    for (int k = 0; k < (DEG + 1) / 2; ++k) jl[k] = second ? jq2[R - 1][k] : jq2[0][k];
    if constexpr (UNI) {
      ls_self = second ? uw_self[R - 1] : uw_self[0];
      ls_off = second ? uw_off[R - 1] : uw_off[0];
      lpos = second ? upos[R - 1] : upos[0];
      llen = second ? ulen[R - 1] : ulen[0];
    } else {
#pragma unroll
      for (int k = 0; k < DEG; ++k) nl[k] = second ? nw[R - 1][k] : nw[0][k];
    }
  };
  auto lweight = [&](int p) -> float {
    if constexpr (UNI) {
      const float w_in = p == lpos ? ls_self : ls_off;
      return p < llen ? w_in : 0.f;
    } else {
      return nl[p];
    }
  };
  auto slab_row = [&](int q) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    // Empty asm statements pin the register plan: the packed slots stay
    // packed and the weights stay in registers (not reloaded from memory),
    // and the reads of one group are not hoisted above the previous group.
#pragma unroll
    for (int k = 0; k < (DEG + 1) / 2; ++k) asm volatile("" : "+v"(jl[k]));
    if constexpr (UNI) {
      asm volatile("" : "+v"(ls_self), "+v"(ls_off), "+v"(lpos), "+v"(llen));
    } else {
#pragma unroll
      for (int k = 0; k < DEG; ++k) asm volatile("" : "+v"(nl[k]));
    }
#pragma unroll
    for (int p0 = 0; p0 < DEG; p0 += G) {
      if (p0 > 0) asm volatile("" ::: "memory");
      float4 x[G];
#pragma unroll
      for (int p = p0; p < p0 + G && p < DEG; ++p)
        x[p - p0] = slab[((jl[p / 2] >> (16 * (p & 1))) & 0xffffu) ^ q];
#pragma unroll
      for (int p = p0; p < p0 + G && p < DEG; ++p) fma4(acc, lweight(p), x[p - p0]);
    }
    // all four components here, or the compiler splits 16-byte LDS reads
    asm volatile("" : "+v"(acc.x), "+v"(acc.y), "+v"(acc.z), "+v"(acc.w));
    return acc;
  };
  const int lane = int(threadIdx.x) & 63;
  const int lane_in = lane & (kOut - 1);
  uint64_t okmask[R];
#pragma unroll
  for (int rr = 0; rr < R; ++rr) okmask[rr] = __ballot(ok[rr]);
  if constexpr (!kOwnCheck) first_loads();
  // one transposed group of 8 outputs: rows row_base + k, columns from c
  auto store_group = [&](const float4 (&res)[kOut], int64_t c, int row_base, uint64_t okm) {
    if (c < a.dim) {
      const bool full = c + 4 <= a.dim;
      const int k_tail = int(min<int64_t>(a.dim - c, 4));
#pragma unroll
      for (int k = 0; k < kOut; ++k) {
        if ((okm >> (lane - lane_in + k)) & 1) {
          float* d = a.dst + int64_t(row_base + k) * a.ld + c;
          if (full) {
            st_nt(reinterpret_cast<float4*>(d), res[k]);
          } else {
            store_partial(d, res[k], k_tail);
          }
        }
      }
    }
  };
  // With two output rows per thread and up to 5 entries per row, the second
  // row's group is held back and stored after the next chunk's loads are
  // issued, so that the wait for those loads at the next staging does not
  // also wait for these stores to drain (1024 x 2^20: d = 2 1.745 -> 1.714
  // ms, d = 4 1.772 -> 1.755 ms; with 9 entries, holding the whole group or
  // half of it made d = 8 slower: its longer neighbour sums let the stores
  // drain anyway).
  constexpr bool kDefer = R == 2 && DEG <= 5 && OPR == kOut;
  float4 pend[kDefer ? kOut : 1];
  int64_t pend_c = -1;
  auto compute = [&](int ch) {
    // one row at a time (R = 2: the second row's state is selected in, not
    // kept beside the first's while its outputs are computed)
#pragma unroll 1
    for (int rr = 0; rr < R; ++rr) {
      select_row(rr);
      const int row_base = (R == 2 && rr == 1 ? orow[R - 1] : orow[0]) & ~(kOut - 1);
      const uint64_t okm = R == 2 && rr == 1 ? okmask[R - 1] : okmask[0];
#pragma unroll 1
      for (int h = 0; h < OPR / kOut; ++h) {
        float4 res[kOut];
#pragma unroll
        for (int u = 0; u < kOut; ++u) res[u] = slab_row(oq0 + h * kOut + u);
        transpose8(res, lane_in);
        const int64_t c = int64_t(ch) * C + 4 * (oq0 + h * kOut + lane_in);
        if (kDefer && rr == R - 1) {
#pragma unroll
          for (int u = 0; u < (kDefer ? kOut : 1); ++u) pend[u] = res[u];
          pend_c = c;
        } else {
          store_group(res, c, row_base, okm);
        }
      }
    }
  };
  auto flush = [&]() {
    if constexpr (kDefer) {
      if (pend_c >= 0) store_group(pend, pend_c, orow[R - 1] & ~(kOut - 1), okmask[R - 1]);
      pend_c = -1;
    }
  };
  if constexpr (NBUF == 2) {
    for (int ch = ch0; ch < ch1; ch += 2) {
      lds_barrier();  // the previous chunk is no longer read
      stage(bufA);
      lds_barrier();
      load(bufA, ch + 2);
      compute(ch);
      if (ch + 1 < ch1) {
        lds_barrier();
        stage(bufB);
        lds_barrier();
        load(bufB, ch + 3);
        compute(ch + 1);
      }
    }
  } else {
    for (int ch = ch0; ch < ch1; ++ch) {
      lds_barrier();  // the previous chunk is no longer read
      stage(bufA);
      lds_barrier();
      load(bufA, ch + 1);
      flush();
      compute(ch);
    }
    flush();
  }
  if (blockIdx.x == 0) {
    const bool head = R == 2 || tid < n;
#pragma unroll
    for (int rr = 0; rr < R; ++rr)
      if (head && ok[rr]) a.tag_dst[orow[rr]] = a.next;
  }
}

template <class T>
__global__ void fill_kernel(T* p, int64_t count, T value) {
  for (int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < count;
       k += int64_t(gridDim.x) * blockDim.x)
    p[k] = value;
}

template <class T>
hipError_t fill(T* p, int64_t count, T value, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((count + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_kernel<T>, dim3(uint32_t(blocks)), dim3(256), 0, s, p, count, value);
  return hipGetLastError();
}

}  // namespace

namespace {
hipError_t launch_epoch_check(const MixArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(epoch_check_kernel, dim3(uint32_t(a.n)), dim3(64), 0, s, a);
  return hipGetLastError();
}

// whether the slab kernel takes this graph: n a power of two in [8, 1024]
// and rows of at most 17 entries
bool slab_graph(int n, int max_deg) { return n >= 8 && n <= 1024 && !(n & (n - 1)) && max_deg <= 17; }

// Shapes: above 256 rows one 512-thread workgroup per CU with a 128 KiB
// (above 512 rows) or 64 KiB chunk; up to 256 rows 256-thread workgroups
// with 32 KiB chunks, up to four per CU.  Every chunk holds a whole 128-byte
// line of every row (Q >= 8 float4).  Small workgroups leave room on a CU for
// the kernels that plan the next round beside the reduce: 256 workers x
// 2^18, random 8-regular: reduce 0.32 -> 0.29 ms, round 1.36 -> 1.32 ms.
int slab_threads(int n) { return n > 256 ? 512 : 256; }
int slab_vec(int n) { return n > 512 ? 8192 : n > 256 ? 4096 : 2048; }
int slab_per_cu(int n) { return n > 256 ? 1 : 4; }

// per-thread staging offset (rows below THREADS/Q, float4 slots below Q) and
// chunk count within 31 bits
bool slab_fits(const MixArgs& a) {
  const int T = slab_threads(a.n);
  const int Q = slab_vec(a.n) / a.n, C = 4 * Q;
  const int rows = Q > T ? 1 : T / Q;
  if ((int64_t(rows - 1) * a.ld + 4 * int64_t(std::min(Q, T))) * 4 >= (int64_t(1) << 31)) return false;
  return (a.dim + C - 1) / C < (int64_t(1) << 31);
}
}  // namespace

bool mix_slab_applies(const MixArgs& a, int max_deg) { return slab_graph(a.n, max_deg) && slab_fits(a); }

// Slab kernel when n is a power of two in [8, 1024] and every row has at most
// 17 entries (returns hipErrorNotSupported otherwise).
template <int DEG>
hipError_t launch_slab(const MixArgs& a, int n_cu, hipStream_t s) {
  if (!slab_fits(a)) return hipErrorNotSupported;
  if (DEG > 9)
    if (hipError_t e = launch_epoch_check(a, s)) return e;
  const int C = 4 * (slab_vec(a.n) / a.n);
  const int nchunks = int((a.dim + C - 1) / C);
  const int grid = std::max(1, std::min(nchunks, slab_per_cu(a.n) * n_cu));
  const dim3 g(grid), b(slab_threads(a.n));
  if (a.n > 512) {
    if (a.uniform_rows)
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 2, 512, 1, 8192, true>), g, b, 0, s, a, nchunks);
    else
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 2, 512, 1, 8192, false>), g, b, 0, s, a, nchunks);
  } else if (a.n > 256) {
    if (a.uniform_rows)
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 1, 512, 2, 4096, true>), g, b, 0, s, a, nchunks);
    else
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 1, 512, 2, 4096, false>), g, b, 0, s, a, nchunks);
  } else {
    if (a.uniform_rows)
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 1, 256, 2, 2048, true>), g, b, 0, s, a, nchunks);
    else
      hipLaunchKernelGGL((mix_slab_kernel<DEG, 1, 256, 2, 2048, false>), g, b, 0, s, a, nchunks);
  }
  return hipGetLastError();
}

hipError_t launch_mix_slab(const MixArgs& a, int max_deg, int n_cu, hipStream_t s) {
  if (!slab_graph(a.n, max_deg)) return hipErrorNotSupported;
  if (max_deg <= 3) return launch_slab<3>(a, n_cu, s);
  if (max_deg <= 5) return launch_slab<5>(a, n_cu, s);
  if (max_deg <= 9) return launch_slab<9>(a, n_cu, s);
  return launch_slab<17>(a, n_cu, s);
}

// Threads for about four slots each, 64 to 1024; blocks per compute unit as LDS
// and threads allow.
constexpr size_t kColsLds = (160 << 10) - 512;  // of a compute unit's 160 KiB, beside the verdicts
size_t cols_lds(const MixArgs& a, int lanes, int64_t nnz) {
  const size_t lists = lanes < 64 ? size_t(nnz) * 6 + size_t(a.n) * (a.scale ? 6 : 2) + 16 : 0;
  return size_t(a.n) * size_t(lanes) * 16 + lists;
}
template <int LPR>
hipError_t launch_cols(const MixArgs& a, int64_t nnz, int n_cu, hipStream_t s) {
  const int slots = a.n * LPR, C = 4 * LPR;
  const int64_t chunks = (a.dim + C - 1) / C;
  if (chunks >= (int64_t(1) << 31)) return hipErrorNotSupported;
  int T = 64;
  while (T < 1024 && T * 4 < slots) T *= 2;
  const int pf = (slots + T - 1) / T;  // <= 8
  const size_t lds = cols_lds(a, LPR, nnz);
  if (lds > kColsLds || nnz > 65535) return hipErrorNotSupported;
  const int per_cu = int(std::max<size_t>(1, std::min<size_t>((size_t(160) << 10) / (lds + 256), size_t(1024 / T))));
  const dim3 g(uint32_t(std::min<int64_t>(chunks, int64_t(per_cu) * n_cu))), b(static_cast<uint32_t>(T));
  auto go = [&](auto kernel) -> hipError_t {
    if (lds > (64u << 10)) {  // has to be asked for
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(kColsLds));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, g, b, lds, s, a, int(chunks));
    return hipGetLastError();
  };
  if (pf <= 4) return go(mix_cols_kernel<LPR, 4>);
  return go(mix_cols_kernel<LPR, 8>);
}

// Column kernel when there are at most 1024 rows (hipErrorNotSupported
// otherwise).  Lanes per row: the most that keep a chunk within 128 KiB.
hipError_t launch_mix_cols(const MixArgs& a, int64_t nnz, int n_cu, hipStream_t s) {
  if (a.n > kColsMaxRows) return hipErrorNotSupported;
  const int most = a.n <= 128 ? 64 : a.n <= 256 ? 32 : a.n <= 512 ? 16 : 8;
  int lanes = most;
  // Above 64 rows a block has 1024 threads and takes all rows of a chunk one
  // after the other, so models with fewer chunks than compute units get
  // narrower ones (tile kernel / most lanes / this, us a reduce): 100 x 4096,
  // 8 neighbours 12.8 / 16.2 / 9.4; 128 x 4096, 64 neighbours 54 / 84 / 37;
  // 200 x 4096, 16 neighbours 19.2 / 25.1 / 14.1.
  auto chunks = [&](int l) { return (a.dim + 4 * l - 1) / (4 * l); };
  if (a.n > 64)
    while (lanes > 8 && chunks(lanes) < n_cu) lanes /= 2;
  if (cols_lds(a, lanes, nnz) > kColsLds) lanes = most;
  // With 8 lanes there are no narrower ones, and few blocks for many rows are
  // slower than the tile kernel: 1000 x 4096, 4 neighbours 16.3 and 20.8 us,
  // 800 x 1000 12.7 and 15.2, 576 x 1000, 16 neighbours, 21.5 and 22.4; 520 x
  // 1000, 4 neighbours, 14.6 and 10.9.  With a chunk for every compute unit the
  // column kernel is ahead (1000 x 16384, 4 neighbours, 45 and 39).
  if (a.n > 544 && chunks(lanes) < n_cu) return hipErrorNotSupported;
  // Rows of up to three entries whose models stay in the memory-side cache
  // (256 MB): the tile kernel's second and third read of a row cost little, and
  // it has no chunk to stage first and no last round of chunks that fills the
  // device in part.  Both buffers of 105 to 260 MB, from 48 MB above 128 workers
  // (tile / column kernel, chain and ring, us): 100 x 200000 34.0 / 47.7 and
  // 39.6 / 48.0; 200 x 33000 15.7 / 19.5 and 17.7 / 20.3; 500 x 33000 30.9 /
  // 41.6 and 35.5 / 42.4.  Below, 100 x 131072 24.3 / 22.4 and 28.0 / 22.5;
  // above, 500 x 65536 76.9 / 62.3 and 84.4 / 63.7; five entries, 100 x 200000
  // 71.0 / 51.5.
  // From 40 MB where the last round of chunks leaves more than 30% of all
  // rounds idle: 100 x 80000 17.3 / 20.3 and 19.6 / 20.6, 160 x 33000 14.2 / 16.3.
  const int64_t both = 8 * int64_t(a.n) * a.dim, rounds = (chunks(lanes) + n_cu - 1) / n_cu;
  const bool uneven = 10 * chunks(lanes) < 7 * rounds * n_cu;
  if (a.n > 64 && nnz <= 3 * int64_t(a.n) && both <= 260000000 &&
      both >= (uneven ? 40000000 : a.n > 128 ? 48000000 : 105000000))
    return hipErrorNotSupported;
  if (lanes == 64) return launch_cols<64>(a, nnz, n_cu, s);
  if (lanes == 32) return launch_cols<32>(a, nnz, n_cu, s);
  if (lanes == 16) return launch_cols<16>(a, nnz, n_cu, s);
  return launch_cols<8>(a, nnz, n_cu, s);
}

// Tile kernel: any number of rows, after its own epoch check.
hipError_t launch_mix(const MixArgs& a, hipStream_t s) {
  const uint32_t nseg = uint32_t((a.dim + kSegFloats - 1) / kSegFloats);
  const uint32_t nrg = uint32_t((a.n + kTileRows - 1) / kTileRows);
  const uint64_t total = uint64_t(nseg) * nrg;
  if (total >= (1ull << 31)) return hipErrorInvalidValue;
  if (hipError_t e = launch_epoch_check(a, s)) return e;
  hipLaunchKernelGGL(mix_kernel, dim3(uint32_t(total)), dim3(kMixThreads), 0, s, a, nseg, nrg);
  return hipGetLastError();
}

hipError_t launch_mean(const MixArgs& a, hipStream_t s) {
  const uint32_t nseg = uint32_t((a.dim + kSegFloats - 1) / kSegFloats);
  hipLaunchKernelGGL(mean_kernel, dim3(nseg), dim3(64), 0, s, a, nseg);
  return hipGetLastError();
}

hipError_t launch_fill_i64(int64_t* p, int64_t count, int64_t value, hipStream_t s) {
  return fill<int64_t>(p, count, value, s);
}
hipError_t launch_fill_f32(float* p, int64_t count, float value, hipStream_t s) {
  return fill<float>(p, count, value, s);
}
hipError_t launch_fill_i32(int32_t* p, int64_t count, int32_t value, hipStream_t s) {
  return fill<int32_t>(p, count, value, s);
}

}  // namespace asap
