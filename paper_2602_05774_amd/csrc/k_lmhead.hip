// Fused LM-head variant: the draft and target logits X = H_d W_d^T and
// Y = H_t W_t^T (bf16 operands, fp32 accumulation on MFMA) are never written
// to memory.
//
// Matrix core tiling.  A workgroup of eight wavefronts (two per SIMD) owns a
// 256x256 output tile, computed as v_mfma_f32_32x32x16_bf16 tiles from LDS
// stages of 64 K values per row (nt_stream below).  K-major operands (the
// weight in dH = g W_d, both in dW_d = g^T H_d) are read with the gfx950
// transpose load (ds_read_b64_tr_b16, two per fragment).
//
// Forward.  One launch covers both models.  A workgroup owns 256 rows and one
// slice of a vocabulary; every 256-column logit tile of the slice is consumed
// in the accumulator registers: the online log-sum-exp (row softmax
// normalisers, Sec. "Preliminary"), the Gumbel-max draws with the exact
// candidate filter (Alg. 1 draws z~ ~ q and z' ~ p under the library's
// normative sampler) and the greedy maximum (Alg. 2).  A row's running state
// stays in registers across the tiles of the slice; the slice's result goes
// to a partial record.  A combine kernel merges the slices, forms the drawn
// tokens' logits by dot products (H_r . W_z) and writes tokens and the
// per-row statistics (log q, log alpha of Eq. acc).
//
// Backward (derivative of Eq. advance through the LM head).  The draft
// logits are recomputed tile by tile; g = loss_scale/T_q ((a+b) q - a e_z~ -
// b e_z') is written in bf16 (the gradient with respect to the logits); then
// dH_d = g W_d and, when asked for, dW_d = g^T H_d (fp32).
#include "vsd_device.hpp"
#include "vsd_kernels.hpp"
#include "vsd_topk.hpp"

namespace vsd {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int TM = 256, TN = 256, TK = 64;   // workgroup tile and K per stage
constexpr int kThreads = 512;                // eight wavefronts
constexpr int kHalfElems = TM / 2 * TK;      // nt_stream: half an operand's stage (128 rows)
constexpr int kBufElems = 4 * kHalfElems;    // one stage: U0 U1 V0 V1
constexpr int kNtLdsBytes = 2 * kBufElems * 2;
constexpr int kXcds = 8;                     // MI355X: 8 XCDs, workgroups dealt round-robin
constexpr int64_t kBigStride = 1ll << 27;    // gradient row strides (elements) past which 8 rows exceed 2^31 bytes
constexpr int kGroupRows = 4;                // row tiles per L2 reuse group
static_assert(kLmTile == TN && kLmTile == TM, "tile width shared with the host");
constexpr int kLmSegM = 6;                   // KL term: list length of one row segment
static_assert(kLmRedoM >= kMaxTopK, "a recompute record holds every member a slice can have");
static_assert(TM * 2 * kLmRedoM * 8 <= kNtLdsBytes, "the recompute's segment lists fit");
static_assert(kLmRedoM * 2 >= 16, "the recompute's list covers the stash");
static_assert(TM * 2 * 32 + TM * 4 * (kLmSegM * 8 + 4) <= kNtLdsBytes, "the slice merge's row states and KL lists fit");

__device__ __forceinline__ f32x16 mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Workgroup -> (row tile, column index) so that the workgroups resident on
// one XCD at a time share few operand tiles: the dispatcher deals workgroup
// ids round-robin over the XCDs, so ids are first regrouped per XCD
// (a bijection), then walked in groups of kGroupRows row tiles, column index
// fastest within a group.
__device__ __forceinline__ void tile_of(int pid, int nrt, int ncol, int& rt, int& col) {
  const int total = nrt * ncol;
  const int xcd = pid % kXcds, local = pid / kXcds;
  const int per = total / kXcds, extra = total % kXcds;
  const int lpid = xcd * per + min(xcd, extra) + local;
  const int gsize = kGroupRows * ncol;
  const int g = lpid / gsize, in = lpid % gsize;
  const int first = g * kGroupRows;
  const int rows = min(nrt - first, kGroupRows);
  rt = first + in % rows;
  col = in / rows;
}

// -------------------------------------------------------------- nt_stream ---
// acc[m][n] = sum_k U[m][k] V[n][k] (bf16, fp32 sums over k in order) for a run
// of 256-row tiles of U (in the forward: weight rows, i.e. vocabulary columns)
// against one 256-row tile of V (hidden states); epi(tile, acc) consumes each
// tile.
//
// Bound: matrix-core issue (2048 cycles per 64-K stage of a tile) against the
// rate at which operands reach LDS.  The eight wavefronts form two groups of
// four (wr = 0, 1: one wavefront of each per SIMD) that run half a phase
// apart: while one group reads fragments and issues loads, the other issues
// MFMAs.  A stage has four phases, one quadrant of the tile each (U half x V
// half; a wavefront owns 64 U rows and 32 V rows of a quadrant: eight MFMAs),
// with two barriers per phase.  Every phase refills the half operand whose
// last reader is past: 48 KB stay in flight and no wait ever drains them.
//   phase  reads (ds_read_b128)  refills           multiplies   waits for
//   1      U0(t)       8         U1(t+1)           U0 V0
//   2      V1(t)       4         V0(t+2)           U0 V1
//   3      U1(t)       8         U0(t+2)           U1 V0        V0(t+1)
//   4      V0(t+1)     4         V1(t+2)           U1 V1        all of t+1
// A refill is safe because the trailing group is at most one barrier behind:
// it has passed the lgkmcnt(0) of the phase that read the half (for V0 the
// phase before; the first stage's, read before the loop, is waited for there).
// A read is safe because both groups waited for their loads before the barrier
// that precedes it.  Loads past the last stage repeat it,
// so the loop has no tail case.
// The loads are buffer loads into LDS: the per-lane offset is 32-bit and the K
// offset scalar.  With 64-bit addresses (global_load_lds) the same loop took
// 9.08 M instead of 7.30 M cycles for 24576 x 32000 x 4096 (matrix cores busy 68
// against 84 %): the address operands slow the issue of every load.
// Without any load it takes 7.24 M.  Output stored: 1390 against 1275 TFLOP/s, and
// 1150-1170 for a loop that loads a whole stage per barrier.
//
// LDS rows are 64 K values (128 B) of eight 16-byte chunks; chunk c of row r
// sits at position c ^ swz(r), so 16 lanes reading a chunk of their rows meet
// every bank once.  The lane of a V fragment reads row lane % 32.  The lane of
// a U fragment i reads row 32 b + 16 i + 4 a + c for lane % 32 = 8 a + 4 b + c,
// which gives accumulator lane (n, b) the 16 consecutive U rows
// 32 b + 16 i + 0..15 of V row n (register 4 a + c).
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_void;

__device__ __forceinline__ int swz_u(int r) { return ((r >> 1) & 3) | (((r >> 5) & 1) << 2); }
__device__ __forceinline__ int swz_v(int r) { return (r >> 1) & 7; }

// A workgroup barrier alone: no wait for outstanding loads, and nothing moves
// across it.
__device__ __forceinline__ void phase_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
// s_waitcnt immediates: vmcnt bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8.
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Operand sources of nt_stream.  A source keeps a cursor per operand (U, V): first()
// sets both to stage 0, advance() moves both on by one stage, the last stage
// repeating; load_u / load_v issue this wavefront's loads of half h of the
// stage a cursor stands at (L: where they go).  kTr: the operand is K-major
// and read with transpose loads.  tail(): the values of the last, partial
// stage (K % 64), formed in registers, zeros past the ends.
//
// Operands as they lie in memory: U rows tile * 256 .. of [nu, K], V rows row0
// .. of [nv, K], for the tiles t_begin .. t_end - 1; K a multiple of 64.  Rows
// past the ends are out of the descriptors' range: no access is made, and what
// their LDS rows then hold reaches only results that the callers discard.
struct NtRows {
  static constexpr bool kTrU = false, kTrV = false, kTail = false;
  const bf16_t* pu;
  const bf16_t* pv;
  int nu;
  int64_t row0, nv;
  int K, t_begin, t_end;
  int t2;                  // tile of the U cursor
  int ou[2][2], ov[2][2];  // lane's byte offset of half h, load j
  __amdgpu_buffer_rsrc_t rv;
  struct U {
    __amdgpu_buffer_rsrc_t r;
    int k;  // byte offset of the stage
  };
  struct V {
    int k;
  };

  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows(const bf16_t* base, int64_t n) const {
    return row_rsrc(base, (uint32_t)min(n, (int64_t)TM) * (uint32_t)K * 2u);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t tile(int t) const {
    return rows(pu + (int64_t)t * TN * K, nu - t * TN);
  }
  __device__ __forceinline__ int stages() const { return K / TK; }
  __device__ __forceinline__ void first(U& u, V& v) {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int r = h * 128 + w * 16 + j * 8 + (lane >> 3);
        ou[h][j] = (r * K + (((lane & 7) ^ swz_u(r)) << 3)) * 2;
        ov[h][j] = (r * K + (((lane & 7) ^ swz_v(r)) << 3)) * 2;
      }
    rv = rows(pv + row0 * K, nv - row0);
    t2 = t_begin;
    u = U{tile(t_begin), 0};
    v = V{0};
  }
  __device__ __forceinline__ void advance(U& u, V& v) {
    int k = u.k + TK * 2;
    if (k == K * 2) {
      if (t2 + 1 < t_end) {
        u.r = tile(++t2);
        k = 0;
      } else {
        k -= TK * 2;
      }
    }
    u.k = v.k = __builtin_amdgcn_readfirstlane(k);  // a scalar operand of the loads
  }
  __device__ __forceinline__ void load_u(int h, const U& u, bf16_t* L) const {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(u.r, (lds_void*)(L + j * 8 * TK), 16, ou[h][j], u.k, 0, 0);
  }
  __device__ __forceinline__ void load_v(int h, const V& v, bf16_t* L) const {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void*)(L + j * 8 * TK), 16, ov[h][j], v.k, 0, 0);
  }
  __device__ __forceinline__ void tail(bf16_t*) const {}
};

// The same gathered through row lists: U row j is row urow[j] of pu (null: j;
// an entry outside [0, urow_n) reads row 0), V row i is row vrow[i] of pv.
// Rows past the ends read the last one.
struct NtGather {
  static constexpr bool kTrU = false, kTrV = false, kTail = false;
  const bf16_t* pu;
  const bf16_t* pv;
  const int32_t* urow;
  int urow_n;
  const int32_t* vrow;
  int nu;
  int64_t row0, nv;
  int K, t_begin, t_end;
  const bf16_t* at[2][2];
  struct U {
    int t, k;
  };
  struct V {
    int k;
  };

  __device__ __forceinline__ int stages() const { return K / TK; }
  __device__ __forceinline__ void first(U& u, V& v) {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int r = h * 128 + w * 16 + j * 8 + (lane >> 3);
        at[h][j] = pv + (int64_t)vrow[min(row0 + r, nv - 1)] * K + (((lane & 7) ^ swz_v(r)) << 3);
      }
    u = U{t_begin, 0};
    v = V{0};
  }
  __device__ __forceinline__ void advance(U& u, V& v) const {
    if (u.k + TK < K)
      u.k += TK;
    else if (u.t + 1 < t_end)
      u = U{u.t + 1, 0};
    v.k = u.k;
  }
  __device__ __forceinline__ void load_u(int h, const U& c, bf16_t* L) const {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = h * 128 + w * 16 + j * 8 + (lane >> 3);
      int u = min(c.t * TN + r, nu - 1);
      if (urow != nullptr) {
        u = urow[u];
        u = (uint32_t)u < (uint32_t)urow_n ? u : 0;
      }
      const bf16_t* p = pu + (int64_t)u * K + (((lane & 7) ^ swz_u(r)) << 3) + c.k;
      __builtin_amdgcn_global_load_lds((const global_void*)p, (lds_void*)(L + j * 8 * TK), 16, 0, 0);
    }
  }
  __device__ __forceinline__ void load_v(int h, const V& v, bf16_t* L) const {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_global_load_lds((const global_void*)(at[h][j] + v.k), (lds_void*)(L + j * 8 * TK), 16, 0, 0);
  }
  __device__ __forceinline__ void tail(bf16_t*) const {}
};

// A K-major operand [K, n] (stride ld), columns c0 .. c0 + 255.  A stage's half
// lies in LDS as 64 rows of 128 columns (256 B, sixteen 16-byte chunks), chunk
// c of row k at position c ^ swz(k): the transpose load's 32 lanes read four
// rows (64 B each), which the swizzle spreads over all banks.  Each load has a
// descriptor of its own four rows up to the last one's column n, so a lane's
// offset covers three rows at most; columns past n read the next row or, in the
// last one, nothing (what lies there may belong to another buffer), and reach
// only results that the callers discard.  BIG: strides past a descriptor's
// 32-bit offsets, by 64-bit addresses with the columns clamped.
template <bool IS_U, bool BIG>
struct KMajor {
  const bf16_t* p;
  int64_t ld;
  int n, c0, K;
  int off[2];           // lane's byte offset of half h (BIG: element offset within the row)
  const bf16_t* at[2];  // first row of load j in stage 0 (BIG: the lane's)
  __device__ __forceinline__ static int swz(int k) { return IS_U ? ((k & 1) << 3) ^ (k & 2) : (k & 3) << 2; }

  __device__ __forceinline__ void init() {
    const int lane = threadIdx.x & 63;
    const int r = lane >> 4;  // (a load's first row is a multiple of 4)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = c0 + h * 128 + (((lane & 15) ^ swz(r)) << 3);
      off[h] = BIG ? min(c, (n - 1) & ~7) : (int)((r * ld + c) * 2);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) at[j] = p + (int64_t)(wave_id() * 8 + j * 4 + (BIG ? r : 0)) * ld;
  }
  // (a whole stage: all four rows of a load exist)
  __device__ __forceinline__ void load(int h, int k, bf16_t* L) const {
    const int64_t ahead = (int64_t)k * ld;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      lds_void* const to = (lds_void*)(L + j * 4 * 128);
      if constexpr (BIG)
        __builtin_amdgcn_global_load_lds((const global_void*)(at[j] + ahead + off[h]), to, 16, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(row_rsrc(at[j] + ahead, lm_kmajor_bytes(ld, n)), to, 16, off[h], 0,
                                                 0, 0);
    }
  }
  // the partial last stage: rows k0 .. K-1, zeros after them and past column n
  __device__ __forceinline__ void tail(int k0, bf16_t* half0) const {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = w * 8 + j * 4 + (lane >> 4);
        const int c = c0 + h * 128 + (((lane & 15) ^ swz(k)) << 3);
        uint32_t v[4] = {0, 0, 0, 0};
        for (int e = 0; e < 8; ++e)
          if (k0 + k < K && c + e < n) v[e >> 1] |= (uint32_t)p[(int64_t)(k0 + k) * ld + c + e] << (16 * (e & 1));
        *reinterpret_cast<uint4*>(half0 + h * kHalfElems + w * 16 * TK + j * 4 * 128 + lane * 8) =
            make_uint4(v[0], v[1], v[2], v[3]);
      }
  }
};

// A K-contiguous operand V [nv, K] of any row stride ld (a multiple of 8), rows
// row0 .. row0 + 255: a descriptor per load (BIG: addresses, rows past the end
// reading the last one), as above.
template <bool BIG>
struct KRows {
  const bf16_t* p;
  int64_t ld, row0, nv;
  int K;
  const bf16_t* at[2][2];  // first row of half h, load j (BIG: the lane's)
  uint32_t bytes[2][2];    // of the rows that exist
  int off[2];

  __device__ __forceinline__ void init() {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = ((lane & 7) ^ swz_v(j * 8 + (lane >> 3))) << 3;
      off[j] = (int)(((lane >> 3) * ld + c) * 2);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t first = row0 + h * 128 + w * 16 + j * 8;
        if constexpr (BIG) {
          at[h][j] = p + min(first + (lane >> 3), nv - 1) * ld + c;
          continue;
        }
        const int64_t r0 = min(first, nv);
        at[h][j] = p + r0 * ld;
        bytes[h][j] = (uint32_t)(min((int64_t)8, nv - r0) * ld * 2);
      }
    }
  }
  __device__ __forceinline__ void load(int h, int koff, bf16_t* L) const {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      lds_void* const to = (lds_void*)(L + j * 8 * TK);
      if constexpr (BIG)
        __builtin_amdgcn_global_load_lds((const global_void*)(at[h][j] + (koff >> 1)), to, 16, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(row_rsrc(at[h][j], bytes[h][j]), to, 16, off[j], koff, 0, 0);
    }
  }
  __device__ __forceinline__ void tail(int k0, bf16_t* half0) const {
    const int lane = threadIdx.x & 63, w = wave_id();
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int lr = w * 16 + j * 8 + (lane >> 3);
        const int64_t row = row0 + h * 128 + lr;
        const int k = k0 + (((lane & 7) ^ swz_v(lr)) << 3);
        uint32_t v[4] = {0, 0, 0, 0};
        for (int e = 0; e < 8; ++e)
          if (row < nv && k + e < K) v[e >> 1] |= (uint32_t)p[row * ld + k + e] << (16 * (e & 1));
        *reinterpret_cast<uint4*>(half0 + h * kHalfElems + lr * TK + (lane & 7) * 8) = make_uint4(v[0], v[1], v[2], v[3]);
      }
  }
};

// One 256 x 256 tile of a product over any K: U K-major; V K-contiguous (OpV =
// KRows) or K-major.  With K-major operands loaded straight into LDS (they went
// through registers and padded LDS rows before, one stage per barrier) dH of
// 24 576 x 4096, K = 32 000, takes 4.39 ms (1467 TFLOP/s) against 6.5-6.9, and
// dW_d of 32 000 x 4096, K = 3072, 0.71 against 0.86-0.98 ms.
template <class OpV, bool TR_V>
struct NtTile {
  static constexpr bool kTrU = true, kTrV = TR_V, kTail = true;
  KMajor<true, false> u;
  OpV v;
  int K;
  static constexpr int t_begin = 0, t_end = 1;
  struct U {
    int k;
  };
  struct V {
    int k;
  };

  __device__ __forceinline__ int stages() const { return K / TK; }
  __device__ __forceinline__ void first(U& a, V& b) {
    u.init();
    v.init();
    a.k = b.k = 0;
  }
  __device__ __forceinline__ void advance(U& a, V& b) const {
    const int k = a.k + 2 * TK <= K ? a.k + TK : a.k;
    a.k = b.k = __builtin_amdgcn_readfirstlane(k);
  }
  __device__ __forceinline__ void load_u(int h, const U& a, bf16_t* L) const { u.load(h, a.k, L); }
  __device__ __forceinline__ void load_v(int h, const V& b, bf16_t* L) const {
    v.load(h, TR_V ? b.k : b.k * 2, L);
  }
  __device__ __forceinline__ void tail(bf16_t* lds) const {
    const int k0 = K / TK * TK;
    u.tail(k0, lds);
    v.tail(k0, lds + 2 * kHalfElems);
  }
};

// A tile's accumulators of one wavefront: acc[h][g][i] = U rows h*128 + wr*64 +
// (fragment i), V rows g*128 + wc*32 + lane % 32.
typedef f32x16 NtAcc[2][2][2];

// Transpose loads (ds_read_b64_tr_b16): in each 16-lane group, source lane s
// names K row s / 4 and four consecutive columns; lane i of the group then
// holds the rows of column i, i.e. of source lane i / 4's (i % 4)th column.
// Two loads (rows +0 and +4, 1024 B apart) give a lane the eight K values of a
// fragment, and a K step of 16 rows lies 4096 B further.  The four K steps of
// one column group are read, and waited for, in one asm block: before the
// builtin the compiler waits for every load into LDS still in flight, which is
// what the loop below avoids.
__device__ __forceinline__ void frag_tr4(const bf16_t* p, bf16x8 (&f)[4]) {
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const bf16_t*)p;
  u32x2 r[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:4096\n\t"
      "ds_read_b64_tr_b16 %3, %8 offset:5120\n\t"
      "ds_read_b64_tr_b16 %4, %8 offset:8192\n\t"
      "ds_read_b64_tr_b16 %5, %8 offset:9216\n\t"
      "ds_read_b64_tr_b16 %6, %8 offset:12288\n\t"
      "ds_read_b64_tr_b16 %7, %8 offset:13312\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a)
      : "memory");
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    f[ks] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, r[2 * ks]), __builtin_bit_cast(bf16x4, r[2 * ks + 1]), 0,
                                    1, 2, 3, 4, 5, 6, 7);
}
// Two column groups at once (one wait).
__device__ __forceinline__ void frag_tr8(const bf16_t* p, const bf16_t* q, bf16x8 (&f)[2][4]) {
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  const uint32_t a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const bf16_t*)p;
  const uint32_t b = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const bf16_t*)q;
  u32x2 r[16];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16\n\t"
      "ds_read_b64_tr_b16 %1, %16 offset:1024\n\t"
      "ds_read_b64_tr_b16 %2, %16 offset:4096\n\t"
      "ds_read_b64_tr_b16 %3, %16 offset:5120\n\t"
      "ds_read_b64_tr_b16 %4, %16 offset:8192\n\t"
      "ds_read_b64_tr_b16 %5, %16 offset:9216\n\t"
      "ds_read_b64_tr_b16 %6, %16 offset:12288\n\t"
      "ds_read_b64_tr_b16 %7, %16 offset:13312\n\t"
      "ds_read_b64_tr_b16 %8, %17\n\t"
      "ds_read_b64_tr_b16 %9, %17 offset:1024\n\t"
      "ds_read_b64_tr_b16 %10, %17 offset:4096\n\t"
      "ds_read_b64_tr_b16 %11, %17 offset:5120\n\t"
      "ds_read_b64_tr_b16 %12, %17 offset:8192\n\t"
      "ds_read_b64_tr_b16 %13, %17 offset:9216\n\t"
      "ds_read_b64_tr_b16 %14, %17 offset:12288\n\t"
      "ds_read_b64_tr_b16 %15, %17 offset:13312\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
        "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11]), "=&v"(r[12]), "=&v"(r[13]), "=&v"(r[14]), "=&v"(r[15])
      : "v"(a), "v"(b)
      : "memory");
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      f[i][ks] = __builtin_shufflevector(__builtin_bit_cast(bf16x4, r[i * 8 + 2 * ks]),
                                         __builtin_bit_cast(bf16x4, r[i * 8 + 2 * ks + 1]), 0, 1, 2, 3, 4, 5, 6, 7);
}

template <class Src, class Epi>
__device__ __forceinline__ void nt_stream(bf16_t* lds, Src& src, Epi&& epi) {
  const int lane = threadIdx.x & 63;
  const int w = wave_id();
  const int wr = w >> 2, wc = w & 3;
  const int nk = src.stages();
  bf16_t* const mine = lds + w * 16 * TK;  // where this wavefront's loads of a half go
  // a lane's fragment addresses, per K step of 16 (K-major: of the first step,
  // for U per fragment i)
  int fu_off[4], fv_off[4];
  {
    const int m = lane & 31, b = (m >> 2) & 1;
    const int ru = 32 * b + 4 * (m >> 3) + (m & 3);
    const int g = lane >> 4, s = lane & 15, kr = (g >> 1) * 8 + (s >> 2);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int c = ks * 2 + (lane >> 5);
      // K-major U: the four quads of a group's 16 columns, in the order of ru
      const int cu = wr * 8 + (s & 1) * 4 + (ks & 1) * 2 + (g & 1);
      const int cv = wc * 4 + (g & 1) * 2 + ((s & 3) >> 1);
      fu_off[ks] = Src::kTrU ? kr * 128 + ((cu ^ KMajor<true, false>::swz(kr)) << 3) + 4 * ((s >> 1) & 1)
                             : (wr * 64 + ru) * TK + ((c ^ swz_u(ru)) << 3);
      fv_off[ks] = 2 * kHalfElems + (Src::kTrV ? kr * 128 + ((cv ^ KMajor<false, false>::swz(kr)) << 3) + 4 * (s & 1)
                                               : (wc * 32 + m) * TK + ((c ^ swz_v(m)) << 3));
    }
  }
  auto frag = [&](int off) { return *reinterpret_cast<const bf16x8*>(lds + off); };
  NtAcc acc;
  bf16x8 fu[2][4], fv0[4], fv1[4];
  auto read_u = [&](int buf, int half) {
    const int at = buf * kBufElems + half * kHalfElems;
    if constexpr (Src::kTrU) {
      frag_tr8(lds + at + fu_off[0], lds + at + fu_off[1], fu);
    } else {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i) fu[i][ks] = frag(at + fu_off[ks] + i * 16 * TK);
    }
  };
  auto read_v = [&](bf16x8 (&f)[4], int buf, int half) {
    const int at = buf * kBufElems + half * kHalfElems;
    if constexpr (Src::kTrV) {
      frag_tr4(lds + at + fv_off[0], f);
    } else {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) f[ks] = frag(at + fv_off[ks]);
    }
  };
  // (the empty asm ties the products between the barriers of their phase)
  auto mult = [&](f32x16 (&c)[2], const bf16x8 (&v)[4]) {
    asm volatile("" : "+v"(c[0]), "+v"(c[1]));
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) c[i] = mfma(fu[i][ks], v[ks], c[i]);
    asm volatile("" : "+v"(c[0]), "+v"(c[1]));
    __builtin_amdgcn_s_setprio(0);
  };
  const bool tail = Src::kTail && src.K % TK != 0;
  auto clear = [&]() {
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q >> 2][(q >> 1) & 1][q & 1] = f32x16{};
  };
  if (nk > 0) {
    // cursors of the stages one and two ahead
    typename Src::U u1, u2;
    typename Src::V v1, v2;
    src.first(u2, v2);
    src.load_v(0, v2, mine + 2 * kHalfElems);
    src.load_u(0, u2, mine);
    src.load_v(1, v2, mine + 3 * kHalfElems);
    src.load_u(1, u2, mine + kHalfElems);
    src.advance(u2, v2);
    u1 = u2;
    v1 = v2;
    src.advance(u2, v2);
    src.load_v(0, v1, mine + kBufElems + 2 * kHalfElems);
    src.load_u(0, u1, mine + kBufElems);
    src.load_v(1, v1, mine + kBufElems + 3 * kHalfElems);
    wait_loads<6>();
    phase_barrier();
    if (wr == 1) phase_barrier();  // from here on this group runs half a phase behind
    read_v(fv0, 0, 0);
    wait_lds();  // phase 2 refills this half, one barrier on for the group behind
    int p = 0;
    for (int tile = src.t_begin; tile < src.t_end; ++tile) {
      clear();
      for (int k = 0; k < nk; ++k, p ^= 1) {
        bf16_t* const cur = mine + p * kBufElems;
        src.load_u(1, u1, mine + (p ^ 1) * kBufElems + kHalfElems);
        read_u(p, 0);
        phase_barrier();
        wait_lds();
        mult(acc[0][0], fv0);
        phase_barrier();

        src.load_v(0, v2, cur + 2 * kHalfElems);
        read_v(fv1, p, 1);
        phase_barrier();
        wait_lds();
        mult(acc[0][1], fv1);
        phase_barrier();

        src.load_u(0, u2, cur);
        read_u(p, 1);
        wait_loads<10>();
        phase_barrier();
        wait_lds();
        mult(acc[1][0], fv0);
        phase_barrier();

        src.load_v(1, v2, cur + 3 * kHalfElems);
        read_v(fv0, p ^ 1, 0);
        wait_loads<6>();
        phase_barrier();
        wait_lds();
        mult(acc[1][1], fv1);
        u1 = u2;
        src.advance(u2, v2);
        // both groups consume the finished tile between the same two barriers
        if (wr == 0) phase_barrier();
        if (!tail && k + 1 == nk) epi(tile, acc);
        if (wr == 1) phase_barrier();
      }
    }
    if (wr == 0) phase_barrier();
    wait_loads<0>();  // the repeated loads have landed ...
    __syncthreads();  // ... in every wavefront: LDS is free
  } else {
    clear();
  }
  if (tail) {  // the partial stage, once per tile and not pipelined
    src.tail(lds);
    __syncthreads();
    read_u(0, 0);
    read_v(fv0, 0, 0);
    read_v(fv1, 0, 1);
    mult(acc[0][0], fv0);
    mult(acc[0][1], fv1);
    read_u(0, 1);
    mult(acc[1][0], fv0);
    mult(acc[1][1], fv1);
    epi(src.t_begin, acc);
  }
}

// Give every lane one V row: after this lane l holds, for V row (l / 32) * 128 +
// wc * 32 + l % 32, the 64 consecutive U rows h*128 + wr*64 + 0..63 of each h
// in acc[h][0][0], acc[h][0][1], acc[h][1][0], acc[h][1][1] (v_permlane32_swap
// exchanges the two V rows' upper and lower halves of the columns).
__device__ __forceinline__ void nt_row_per_lane(NtAcc& acc) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[h][0][i][e]),
                                                        __float_as_uint(acc[h][1][i][e]), false, false);
        acc[h][0][i][e] = __uint_as_float(s[0]);
        acc[h][1][i][e] = __uint_as_float(s[1]);
      }
}
__device__ __forceinline__ int nt_lane_row() {
  const int lane = threadIdx.x & 63;
  return (lane >> 5) * 128 + (wave_id() & 3) * 32 + (lane & 31);
}
// Chunk CH (of 16) of a lane's row: columns (CH / 8) * 128 + wr * 64 + (CH % 8) * 8 .. +7.
template <int CH>
__device__ __forceinline__ void nt_take(const NtAcc& acc, float (&x)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = acc[CH >> 3][(CH >> 2) & 1][(CH >> 1) & 1][(CH & 1) * 8 + e];
}
// The same for a wavefront-uniform chunk number: one copy of the code that
// consumes a chunk serves all sixteen.
__device__ __forceinline__ void nt_chunk(const NtAcc& acc, int ch, float (&x)[8]) {
  switch (ch) {
    case 0: nt_take<0>(acc, x); break;
    case 1: nt_take<1>(acc, x); break;
    case 2: nt_take<2>(acc, x); break;
    case 3: nt_take<3>(acc, x); break;
    case 4: nt_take<4>(acc, x); break;
    case 5: nt_take<5>(acc, x); break;
    case 6: nt_take<6>(acc, x); break;
    case 7: nt_take<7>(acc, x); break;
    case 8: nt_take<8>(acc, x); break;
    case 9: nt_take<9>(acc, x); break;
    case 10: nt_take<10>(acc, x); break;
    case 11: nt_take<11>(acc, x); break;
    case 12: nt_take<12>(acc, x); break;
    case 13: nt_take<13>(acc, x); break;
    case 14: nt_take<14>(acc, x); break;
    default: nt_take<15>(acc, x); break;
  }
}
__device__ __forceinline__ int nt_chunk_col(int ch) { return (ch >> 3) * 128 + (wave_id() >> 2) * 64 + (ch & 7) * 8; }

// --------------------------------------------------------- epilogue helpers ---
__device__ __forceinline__ uint32_t word_of(const uint4& p, int k) {
  return k == 0 ? p.x : k == 1 ? p.y : k == 2 ? p.z : p.w;
}

// Candidate filter of the Gumbel-max draw.  With u from word w and
// j' = (~w) >> 8 <= 2^24 (1 - u), the variate obeys
// G = -ln(-ln u) <= -ln(1 - u) <= (24 - log2 j') ln 2, so an element whose
// bound x/T + (24 - log2 j') ln 2 stays below the best key so far, thr, less
// a rounding margin, cannot win.  (thr - margin) log2(e) is folded into the
// bound's constant; the margin 2e-3 + 2e-6 |thr| exceeds every rounding
// involved for |x/T| <= |thr| + 100, and an element with x/T < thr - 100
// cannot reach thr because G < 16.7.
__device__ __forceinline__ float bound_offset(float thr) {
  return 24.0f - (thr - (2e-3f + 2e-6f * fabsf(thr))) * kLog2e;
}

__device__ __forceinline__ bool bound_ok(float v, uint32_t w, float c2, float off) {
  return fmaf(v, c2, off) >= __builtin_amdgcn_logf((float)((~w) >> 8));
}

__device__ __forceinline__ void lse_merge(float& mraw, float& mc, float& s, float omraw, float omc, float os) {
  lse2_merge(mc, s, omc, os);
  mraw = fmaxf(mraw, omraw);
}

__device__ __forceinline__ void best_merge(float& key, int& idx, float okey, int oidx) {
  if (okey > key || (okey == key && oidx < idx)) {
    key = okey;
    idx = oidx;
  }
}

struct RowState {
  float mraw, mc, s;  // log-sum-exp: raw maximum, its scaled value, sum of exp2(x c2 - mc)
  float key;          // best Gumbel key so far
  int idx;            // its draft index
  float gval;         // target: greedy maximum (raw logit) ...
  int gidx;           // ... and its draft index
  int pad;
};
static_assert(sizeof(RowState) == sizeof(LmPartial), "partial record layout");

__device__ __forceinline__ RowState empty_state() {
  return RowState{kNegBig, kNegBig, 0.0f, -INFINITY, 0x7FFFFFFF, -INFINITY, 0x7FFFFFFF, 0};
}

__device__ __forceinline__ void state_merge(RowState& a, const RowState& b) {
  lse_merge(a.mraw, a.mc, a.s, b.mraw, b.mc, b.s);
  best_merge(a.key, a.idx, b.key, b.idx);
  best_merge(a.gval, a.gidx, b.gval, b.gidx);
}

// KL term (Eq. klv): the M best (value, draft index) pairs offered to one row
// segment (M = kLmSegM) or kept by one slice (M = kLmKlM), ordered as the
// top-K orders them (larger value first, equal values by the smaller index);
// n counts the finite values offered, so n > M means some were dropped,
// every one of them at most v[M - 1].  Only finite values take part (a token
// of zero target probability is not a member).
template <int M>
struct KlList {
  float v[M];
  int i[M];
  int n;

  __device__ __forceinline__ void init() {
#pragma unroll
    for (int j = 0; j < M; ++j) {
      v[j] = -INFINITY;
      i[j] = 0x7FFFFFFF;
    }
    n = 0;
  }
  __device__ __forceinline__ static bool beats(float a, int ia, float b, int ib) {
    return a > b || (a == b && ia < ib);
  }
  __device__ __forceinline__ void offer(float x, int idx) {
    if (!(x > -INFINITY)) return;
    ++n;
    if (!beats(x, idx, v[M - 1], i[M - 1])) return;
    v[M - 1] = x;
    i[M - 1] = idx;
#pragma unroll
    for (int j = M - 1; j > 0; --j) {  // one bubble pass keeps the list ordered
      const bool up = beats(v[j], i[j], v[j - 1], i[j - 1]);
      const float tv = v[j];
      const int ti = i[j];
      v[j] = up ? v[j - 1] : tv;
      i[j] = up ? i[j - 1] : ti;
      v[j - 1] = up ? tv : v[j - 1];
      i[j - 1] = up ? ti : i[j - 1];
    }
  }
  // an upper bound of every dropped value (-inf: nothing dropped)
  __device__ __forceinline__ float bound() const { return n > M ? v[M - 1] : -INFINITY; }
};

// Per-thread words kept in LDS while nt_stream multiplies: its accumulators and
// fragments leave room for the running state of a row but not for the KL lists
// beside it (kept in registers they spilled inside the loop: 30.8 ms for a
// forward that takes 4.6).  Word j of every thread is a row of kThreads words.
constexpr int kStashWords = 16;
struct Stash {
  uint32_t* p;  // LDS [kStashWords][kThreads], at the calling thread
  __device__ __forceinline__ void put(int j, float v) { p[j * kThreads] = __float_as_uint(v); }
  __device__ __forceinline__ void put(int j, int v) { p[j * kThreads] = (uint32_t)v; }
  __device__ __forceinline__ void get(int j, float& v) const { v = __uint_as_float(p[j * kThreads]); }
  __device__ __forceinline__ void get(int j, int& v) const { v = (int)p[j * kThreads]; }
};
constexpr int kStashBytes = kStashWords * kThreads * 4;
static_assert(kNtLdsBytes + kStashBytes <= 160 * 1024, "operand stages and stash fit the LDS");

// Fold eight consecutive columns c .. c+7 of row r (values x; columns past
// the vocabulary hold -inf) into the running state st of one row segment.
// Every lane of a wavefront works on the same columns of a different row, so
// map lookups and Philox group changes are uniform across the wavefront.
// TARGET = false: keys of family 0 over every column.  TARGET = true: keys of
// family 1 and the greedy maximum over the mapped columns, each identified by
// its draft index; the last Philox call (group cg, words cw) is reused, and
// for an ascending map the draft indices increase along the row, so a new
// call is made once per four mapped columns.
template <bool TARGET, bool KL>
__device__ __forceinline__ void fold8(const LmFwdArgs& a, const float (&x)[8], uint32_t r, int c, int nvalid,
                                      float inv_t, float c2, RowState& st, int& cg, uint4& cw, KlList<kLmSegM>& kl) {
  float cm = x[0];
#pragma unroll
  for (int k = 1; k < 8; ++k) cm = fmaxf(cm, x[k]);
  if (cm > st.mraw) {
    const float nmc = cm * c2;
    st.s = lse_scaled(st.s, st.mc - nmc);
    st.mc = nmc;
    st.mraw = cm;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) st.s += __builtin_amdgcn_exp2f(fmaf(x[k], c2, -st.mc));
  if (TARGET && KL) {  // the mapped columns' logits, for the row's top-K set
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int vk = k < nvalid ? (a.inv == nullptr ? c + k : a.inv[c + k]) : -1;
      if (vk >= 0) kl.offer(x[k], vk);
    }
  }
  if (!a.sample) return;
  const float off = bound_offset(st.key);
  if (!TARGET) {
    const uint32_t c0 = (uint32_t)c >> 2;
    const uint4 p0 = philox4x32_10(c0, r, 0u, a.offset, a.k0, a.k1);
    const uint4 p1 = philox4x32_10(c0 + 1, r, 0u, a.offset, a.k0, a.k1);
    uint32_t cand = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      cand |= (k < nvalid && bound_ok(x[k], word_of(k < 4 ? p0 : p1, k & 3), c2, off)) ? (1u << k) : 0u;
    if (__ballot(cand != 0u) != 0ull) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (cand & (1u << k)) {  // columns increase along the row: strict > keeps the smallest index
          const float key = gumbel_key(x[k], inv_t, word_of(k < 4 ? p0 : p1, k & 3));
          if (key > st.key) {
            st.key = key;
            st.idx = c + k;
          }
        }
      }
    }
  } else {
    int v[8];
    if (a.inv == nullptr) {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = k < nvalid ? c + k : -1;
    } else if (nvalid == 8) {
      load8(a.inv + c, v);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = k < nvalid ? a.inv[c + k] : -1;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (v[k] >= 0) {
        const int grp = v[k] >> 2;
        if (grp != cg) {
          cg = grp;
          cw = philox4x32_10((uint32_t)grp, r, 1u, a.offset, a.k0, a.k1);
        }
        const uint32_t wk = word_of(cw, v[k] & 3);
        best_merge(st.gval, st.gidx, x[k], v[k]);
        if (bound_ok(x[k], wk, c2, off)) best_merge(st.key, st.idx, gumbel_key(x[k], inv_t, wk), v[k]);
      }
    }
  }
}

// One slice of one model for rows row0 .. row0+255.  TARGET = false: draft
// logits; TARGET = true: target logits (log-sum-exp over every column, draws
// and greedy maximum over the mapped ones).  A lane owns one row and the 128
// columns h*128 + wr*64 .. +63 (h = 0, 1) of every tile, in increasing order;
// every lane of a wavefront works on the same columns.  A tile's log-sum-exp is
// formed by itself and then merged into the slice's, tile by tile; the two
// column segments (wr) of a row are merged once, at the end, through LDS.
// Consuming a tile in the accumulators (no LDS round trip, no barrier, and the
// next tile's operands already in flight) with nt_stream's loop took the
// forward of 24 576 rows (H 4096, 128 256 + 32 000 columns) from 31.0 to 27.8
// ms; without draws, 24.0 ms.
// First tile of a slice of a pass of V columns.
__device__ __forceinline__ int slice_begin(int V, int nslice, int slice) {
  return (int)((int64_t)((V + TN - 1) / TN) * slice / nslice);
}

// TILES: `slice` is a run of a.run_tiles tiles, whose states go to a.tile_part
// one by one; the stores are issued next to the stream's loads, whose waits
// count both and so wait for no less than they did.  The KL lists run on over
// the run's tiles and are a run's as they are a slice's.
template <bool TARGET, bool KL, bool TILES>
__device__ void lm_pass(const LmFwdArgs& a, int64_t row0, int slice, bf16_t* lds, Stash stash) {
  const int wr = wave_id() >> 2;
  const int V = TARGET ? a.Vt : a.Vd;
  const int nslice = TARGET ? a.nslice_t : a.nslice_d;
  const int ntiles = (V + TN - 1) / TN;
  const int t_begin = TILES ? slice * a.run_tiles : slice_begin(V, nslice, slice);
  const int t_end = TILES ? min(ntiles, t_begin + a.run_tiles) : slice_begin(V, nslice, slice + 1);
  const float inv_t = TARGET ? a.inv_tp : a.inv_tq;
  const float c2 = inv_t * kLog2e;
  const int lrow = nt_lane_row();
  const int64_t r = row0 + lrow;
  RowState st = empty_state();
  KlList<kLmSegM> kl[2];  // one list per 64-column half of the lane's columns
  // the second list and the slice's log-sum-exp wait in the stash between tiles
  // (TILES: the log-sum-exp is done with the tile)
  auto save = [&]() {
#pragma unroll
    for (int j = 0; j < kLmSegM; ++j) {
      stash.put(2 * j, kl[1].v[j]);
      stash.put(2 * j + 1, kl[1].i[j]);
    }
    stash.put(2 * kLmSegM, kl[1].n);
    stash.put(2 * kLmSegM + 1, st.mraw);
    stash.put(2 * kLmSegM + 2, st.mc);
    stash.put(2 * kLmSegM + 3, st.s);
  };
  auto load = [&]() {
#pragma unroll
    for (int j = 0; j < kLmSegM; ++j) {
      stash.get(2 * j, kl[1].v[j]);
      stash.get(2 * j + 1, kl[1].i[j]);
    }
    stash.get(2 * kLmSegM, kl[1].n);
    stash.get(2 * kLmSegM + 1, st.mraw);
    stash.get(2 * kLmSegM + 2, st.mc);
    stash.get(2 * kLmSegM + 3, st.s);
  };
  if (TARGET && KL) {
    kl[0].init();
    kl[1].init();
    save();
  }
  NtRows src{static_cast<const bf16_t*>(TARGET ? a.Wt : a.Wd), static_cast<const bf16_t*>(TARGET ? a.Ht : a.Hd), V,
             row0, a.R, a.H, t_begin, t_end};
  nt_stream(lds, src, [&](int tile, NtAcc& acc) {
    nt_row_per_lane(acc);
    if (r >= a.R) return;
    if (TARGET && KL) load();
    float cmraw = st.mraw, cmc = st.mc, cs = st.s;
    st.mraw = kNegBig;
    st.mc = kNegBig;
    st.s = 0.0f;
    int cg = -1;
    uint4 cw = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll 1
      for (int ch = 0; ch < 8; ++ch) {
        const int c = tile * TN + nt_chunk_col(h * 8 + ch);
        const int nvalid = min(8, V - c);
        if (nvalid <= 0) break;
        float x[8];
        nt_chunk(acc, h * 8 + ch, x);
        if (nvalid < 8) {
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (k >= nvalid) x[k] = -INFINITY;
        }
        fold8<TARGET, KL>(a, x, (uint32_t)r, c, nvalid, inv_t, c2, st, cg, cw, kl[h]);
      }
    }
    if (TILES) {
      const int64_t at = (int64_t)((TARGET ? 0 : (a.Vt + TN - 1) / TN) + tile) * 2 + wr;
      a.tile_part[at * a.R + r] = LmPartial{st.mraw, st.mc, st.s, st.key, st.idx, st.gval, st.gidx, 0};
      if (TARGET && KL) save();
      return;
    }
    lse_merge(cmraw, cmc, cs, st.mraw, st.mc, st.s);
    st.mraw = cmraw;
    st.mc = cmc;
    st.s = cs;
    if (TARGET && KL) save();
  });
  if (TILES && !(TARGET && KL)) return;
  if (TARGET && KL) load();
  RowState* red = reinterpret_cast<RowState*>(lds);  // [TM rows][2 segments]
  LmKlEntry* klred = reinterpret_cast<LmKlEntry*>(red + TM * 2);  // [TM rows][4 segments][kLmSegM]
  float* klbnd = reinterpret_cast<float*>(klred + TM * 4 * kLmSegM);  // [TM rows][4 segments]
  red[lrow * 2 + wr] = st;
  if (TARGET && KL) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int q = lrow * 4 + wr * 2 + h;
#pragma unroll
      for (int j = 0; j < kLmSegM; ++j) klred[q * kLmSegM + j] = LmKlEntry{kl[h].v[j], kl[h].i[j]};
      klbnd[q] = kl[h].bound();
    }
  }
  __syncthreads();
  if (threadIdx.x >= TM || row0 + threadIdx.x >= a.R) return;
  const int64_t row = row0 + threadIdx.x;
  if (TARGET && KL) {
    // the slice's list: the best kLmKlM of its four segments' lists; its
    // bound covers what the segments dropped and what this merge drops
    KlList<kLmKlM> m;
    m.init();
    float bnd = -INFINITY;
#pragma unroll 1
    for (int sg = 0; sg < 4; ++sg) {
      const int q = threadIdx.x * 4 + sg;
      bnd = fmaxf(bnd, klbnd[q]);
#pragma unroll
      for (int j = 0; j < kLmSegM; ++j) {
        const LmKlEntry e = klred[q * kLmSegM + j];
        m.offer(e.val, e.idx);
      }
    }
#pragma unroll
    for (int j = 0; j < kLmKlM; ++j) a.kl_part[row * a.kl_stride + slice * kLmKlM + j] = LmKlEntry{m.v[j], m.i[j]};
    a.kl_bound[row * a.kl_lists + slice] = fmaxf(bnd, m.bound());
  }
  if (TILES) return;
  RowState m = red[threadIdx.x * 2];
  state_merge(m, red[threadIdx.x * 2 + 1]);
  const int col = TARGET ? slice : a.nslice_t + slice;
  a.part[row * (a.nslice_t + a.nslice_d) + col] = LmPartial{m.mraw, m.mc, m.s, m.key, m.idx, m.gval, m.gidx, 0};
}

template <bool KL, bool TILES>
__global__ __launch_bounds__(kThreads, 1) void k_lm_fwd(LmFwdArgs a) {
  __shared__ __align__(16) bf16_t lds[2 * kBufElems + (KL ? kStashBytes / 2 : 0)];
  const Stash stash{reinterpret_cast<uint32_t*>(lds + 2 * kBufElems) + threadIdx.x};
  const int nrt = (int)((a.R + TM - 1) / TM);
  auto runs = [&](int V) { return ((V + TN - 1) / TN + a.run_tiles - 1) / a.run_tiles; };
  const int cols_t = TILES ? runs(a.Vt) : a.nslice_t, cols_d = TILES ? runs(a.Vd) : a.nslice_d;
  int rt, col;
  tile_of(blockIdx.x, nrt, cols_t + cols_d, rt, col);
  if (col < cols_t)
    lm_pass<true, KL, TILES>(a, (int64_t)rt * TM, col, lds, stash);
  else
    lm_pass<false, false, TILES>(a, (int64_t)rt * TM, col - cols_t, lds, stash);
}

// The slices' states from the tiles' (one thread per slice and row): the
// tiles of a wavefront group merge in order, then the two groups, as in a
// workgroup that walks the slice.
__global__ __launch_bounds__(256) void k_lm_fold(LmFwdArgs a) {
  const int nsl = a.nslice_t + a.nslice_d;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= a.R * nsl) return;
  const int64_t r = t % a.R;
  const int sl = (int)(t / a.R);
  const bool target = sl < a.nslice_t;
  const int V = target ? a.Vt : a.Vd, n = target ? a.nslice_t : a.nslice_d, k = target ? sl : sl - a.nslice_t;
  const int first = target ? 0 : (a.Vt + TN - 1) / TN;
  const int begin = slice_begin(V, n, k), end = slice_begin(V, n, k + 1);
  RowState m[2] = {empty_state(), empty_state()};
  for (int tile = begin; tile < end; ++tile) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const LmPartial p = a.tile_part[((int64_t)(first + tile) * 2 + g) * a.R + r];
      state_merge(m[g], RowState{p.mraw, p.mc, p.s, p.key, p.idx, p.gval, p.gidx, 0});
    }
  }
  state_merge(m[0], m[1]);
  a.part[r * nsl + sl] = LmPartial{m[0].mraw, m[0].mc, m[0].s, m[0].key, m[0].idx, m[0].gval, m[0].gidx, 0};
}

// Inverse of the draft->target map: inv[t] = v where d2t[v] = t, else -1.
// The map must be injective: a second draft index claiming a target slot
// finds it taken (compare-and-swap against the fill value) and reports
// VSD_DEVERR_MAP_DUPLICATE instead of overwriting it.
// The inverse map in one launch: workgroup b owns target columns
// [b kInvCols, (b + 1) kInvCols), gathers their draft indices in LDS from a
// pass over the whole map (L2-resident; 0.13 MB for 32 000 entries) and
// writes its part of inv, -1 where no entry points.  (A fill and a scatter in
// two launches took 4.9 + 4.6 us and the gap between them.)
constexpr int kInvThreads = 1024, kInvCols = 4096;
__global__ __launch_bounds__(kInvThreads) void k_lm_inv(const int32_t* d2t, int Vd, int Vt, int32_t* inv,
                                                        int32_t* err, uint32_t* clear, int nclear) {
  __shared__ int32_t own[kInvCols];
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < nclear; k += kInvThreads) clear[k] = 0u;
  const int64_t lo = (int64_t)blockIdx.x * kInvCols;
  for (int k = threadIdx.x; k < kInvCols; k += kInvThreads) own[k] = -1;
  __syncthreads();
  constexpr int U = 32;  // map entries in flight per thread: one round trip for 32 768 entries
  for (int v0 = threadIdx.x; v0 - (int)threadIdx.x < Vd; v0 += U * kInvThreads) {
    int32_t t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = v0 + u * kInvThreads < Vd ? d2t[v0 + u * kInvThreads] : (int32_t)lo - 1;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * kInvThreads;
      if (v >= Vd) continue;
      if ((uint32_t)t[u] >= (uint32_t)Vt) {
        if (blockIdx.x == 0) report_error(err, VSD_DEVERR_MAP_RANGE);
        continue;
      }
      const int64_t at = (int64_t)t[u] - lo;
      if (at >= 0 && at < kInvCols && atomicCAS(own + at, -1, v) != -1) report_error(err, VSD_DEVERR_MAP_DUPLICATE);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kInvCols && lo + k < Vt; k += kInvThreads) inv[lo + k] = own[k];
}

// Dot product of two bf16 rows of length H (H % 8 == 0), one wavefront; the
// result is the same in every lane.
__device__ __forceinline__ float wave_dot(const bf16_t* x, const bf16_t* y, int H, int lane) {
  float acc = 0.0f;
  for (int k = lane * 8; k < H; k += kWave * 8) {
    float xv[8], yv[8];
    load8(x + k, xv);
    load8(y + k, yv);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc = fmaf(xv[j], yv[j], acc);
  }
  return wave_sum(acc);
}

// The KL term of row r from its members in tk (after finish()): the draft
// logits at the members by dot products, then the row term (Eq. klv).
__device__ void lm_kl_row(const LmCombineArgs& a, const WaveTopK& tk, int64_t r, int lane) {
  const bf16_t* hd = static_cast<const bf16_t*>(a.Hd) + r * a.H;
  const bf16_t* Wd = static_cast<const bf16_t*>(a.Wd);
  const int n = min(tk.n, a.kl_k);
  float x = -INFINITY;
  for (int k = 0; k < n; ++k) {
    const int v = tk.bi[k];
    const float xk = (uint32_t)v < (uint32_t)a.Vd ? wave_dot(hd, Wd + (int64_t)v * a.H, a.H, lane) : -INFINITY;
    x = lane == k ? xk : x;
  }
  const bool mine = lane < n;
  int v = mine ? tk.bi[lane] : -1;
  v = (uint32_t)v < (uint32_t)a.Vd ? v : -1;
  const float y = mine ? tk.bv[lane] : -INFINITY;
  kl_row_term_xy(mine, v, y, x, a.kl_k, a.inv_tq, a.inv_tp, a.kl_gscale, a.kl_idx + r * a.kl_k,
                 a.kl_grad + r * a.kl_k, a.kl_row + r, lane);
}

// Offer ne (value, draft index) entries to tk, 8 per lane per round
// (non-finite values take no part).
__device__ __forceinline__ void offer_entries(WaveTopK& tk, const LmKlEntry* ent, int ne, int lane) {
  typedef __attribute__((ext_vector_type(8))) int i32x8;  // a register vector, never a private array
  for (int e0 = 0; e0 < ne; e0 += 8 * kWave) {
    float x[8];
    i32x8 ix;
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = e0 + lane * 8 + k;
      const LmKlEntry en = e < ne ? ent[e] : LmKlEntry{-INFINITY, 0x7FFFFFFF};
      x[k] = en.val;
      ix[k] = en.idx;
      bits |= en.val > -INFINITY ? (1u << k) : 0u;
    }
    tk.offer8(x, 0, bits, [&](int k) { return ix[k]; }, lane);
  }
}

// Merge the slices of both models, write tokens (sampling) and the row
// statistics.  One wavefront per row.  With the KL term, the slices' lists
// are merged into the row's top-K set: exact unless some slice dropped a
// value reaching the set's K-th value; such a row is appended to kl_list
// and its term is left to k_lm_kl_redo and k_lm_kl_redo_select.
template <bool KL>
__global__ __launch_bounds__(256) void k_lm_combine(LmCombineArgs a) {
  __shared__ float kl_bv[KL ? 4 * kTopKCap : 1];
  __shared__ int kl_bi[KL ? 4 * kTopKCap : 1];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int64_t r = (int64_t)blockIdx.x * 4 + wave;
  if (r >= a.R) return;
  const int i = (int)(r % a.L);
  int d = a.L;
  if (a.depth != nullptr) {
    d = a.depth[r / a.L];
    if (d < 1 || d > a.L) {
      if (lane == 0) report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  const bool sampling = a.tok_in[0] == nullptr;
  if (i >= d) {  // masked slot: tokens -1 (sampling), every statistic 0
    if (lane < 3) {
      a.la[r * 3 + lane] = 0.0f;
      a.lq[r * 3 + lane] = 0.0f;
      if (sampling) a.tok_out[lane][r] = -1;
    }
    if (lane == 0) {
      a.lse_q[r] = 0.0f;
      if (a.lse_p != nullptr) a.lse_p[r] = 0.0f;
    }
    if (KL) {
      if (lane < a.kl_k) {
        a.kl_idx[r * a.kl_k + lane] = -1;
        a.kl_grad[r * a.kl_k + lane] = 0.0f;
      }
      if (lane == 0) {
        a.kl_row[r] = 0.0f;
      }
    }
    return;
  }
  const int nsl = a.nslice_t + a.nslice_d;
  const LmPartial* pr = a.part + r * nsl;
  // slices in index order, so equal keys resolve to the smaller index as in one pass
  float pmraw = kNegBig, pmc = kNegBig, ps = 0.0f, tkey = -INFINITY, gval = -INFINITY;
  int tidx = 0x7FFFFFFF, gidx = 0x7FFFFFFF;
  for (int sl = 0; sl < a.nslice_t; ++sl) {
    const LmPartial p = pr[sl];
    lse_merge(pmraw, pmc, ps, p.mraw, p.mc, p.s);
    best_merge(tkey, tidx, p.key, p.idx);
    best_merge(gval, gidx, p.gval, p.gidx);
  }
  float qmraw = kNegBig, qmc = kNegBig, qs = 0.0f, dkey = -INFINITY;
  int didx = 0x7FFFFFFF;
  for (int sl = 0; sl < a.nslice_d; ++sl) {
    const LmPartial p = pr[a.nslice_t + sl];
    lse_merge(qmraw, qmc, qs, p.mraw, p.mc, p.s);
    best_merge(dkey, didx, p.key, p.idx);
  }
  const float cq2 = a.inv_tq * kLog2e, cp2 = a.inv_tp * kLog2e;
  const float qt = (log2f(qs) - fmaf(qmraw, cq2, -qmc)) * kLn2;
  const float pt = (log2f(ps) - fmaf(pmraw, cp2, -pmc)) * kLn2;
  int tok[3];
  if (sampling) {
    tok[0] = didx;
    tok[1] = tidx;
    tok[2] = gidx;
  } else {
#pragma unroll
    for (int f = 0; f < 3; ++f) tok[f] = a.tok_in[f][r];
  }
  const bf16_t* hd = static_cast<const bf16_t*>(a.Hd) + r * a.H;
  const bf16_t* ht = static_cast<const bf16_t*>(a.Ht) + r * a.H;
  const bf16_t* Wd = static_cast<const bf16_t*>(a.Wd);
  const bf16_t* Wt = static_cast<const bf16_t*>(a.Wt);
  const float gap = lse_gap(pmraw, pt, a.inv_tp, qmraw, qt, a.inv_tq);
  float lqv[3], lav[3];
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    const int z = tok[f];
    lqv[f] = 0.0f;
    lav[f] = 0.0f;
    if ((uint32_t)z >= (uint32_t)a.Vd) {
      if (lane == 0) report_error(a.err, VSD_DEVERR_TOKEN_RANGE);
      continue;
    }
    const int zt = a.d2t != nullptr ? a.d2t[z] : z;
    if ((uint32_t)zt >= (uint32_t)a.Vt) {
      if (lane == 0) report_error(a.err, VSD_DEVERR_MAP_RANGE);
      continue;
    }
    const float xz = wave_dot(hd, Wd + (int64_t)z * a.H, a.H, lane);
    const float yz = wave_dot(ht, Wt + (int64_t)zt * a.H, a.H, lane);
    lqv[f] = (xz - qmraw) * a.inv_tq - qt;
    lav[f] = log_alpha_of(xz, yz, a.inv_tq, a.inv_tp, gap);
  }
  if (lane < 3) {
    a.la[r * 3 + lane] = lane == 0 ? lav[0] : lane == 1 ? lav[1] : lav[2];
    a.lq[r * 3 + lane] = lane == 0 ? lqv[0] : lane == 1 ? lqv[1] : lqv[2];
    if (sampling) a.tok_out[lane][r] = lane == 0 ? tok[0] : lane == 1 ? tok[1] : tok[2];
  }
  if (lane == 0) {
    a.lse_q[r] = qmraw * a.inv_tq + qt;
    if (a.lse_p != nullptr) a.lse_p[r] = pmraw * a.inv_tp + pt;
  }
  if (KL) {
    WaveTopK tk;
    tk.init(kl_bv + wave * kTopKCap, kl_bi + wave * kTopKCap, a.kl_k);
    offer_entries(tk, a.kl_in + r * a.kl_in_stride, a.kl_lists * kLmKlM, lane);
    tk.finish(lane);
    const float tau = tk.n >= a.kl_k ? tk.bv[a.kl_k - 1] : -INFINITY;
    float bmax = -INFINITY;
    for (int k = lane; k < a.kl_lists; k += kWave) bmax = fmaxf(bmax, a.kl_bound[r * a.kl_lists + k]);
    bmax = wave_max(bmax);
    // a dropped value at or above the K-th member (or any, with fewer than K
    // members) might belong to the set
    const bool redo = tk.n >= a.kl_k ? bmax >= tau : bmax > -INFINITY;
    if (redo) {
      if (lane == 0) a.kl_list[atomicAdd(a.kl_count, 1)] = (int)r;
    } else {
      lm_kl_row(a, tk, r, lane);
    }
  }
}

__global__ void k_lm_kl_reset(int32_t* count) {
  if (threadIdx.x == 0) *count = 0;
}

// Exact recompute of the rows k_lm_combine<KL> listed.  A workgroup takes
// 256 listed rows (tile row i: H_t row kl_list[row0 + i]) and one of
// kl_nslice slices of the draft vocabulary's 256-column tiles (tile column
// j: draft index v, W_t row d2t[v]).  Operands, K order and matrix-core
// arithmetic are those of the forward's target tiles, so each value equals
// the one the forward formed for (row, d2t[v]).  Each thread keeps the
// kLmRedoM best (value, v) of its row segment (128 columns of every tile),
// which holds every member of the row's top-K that lies there, since K <=
// kLmRedoM; the two segments of a row merge into the slice's record in
// kl_part (where the forward's slice lists lay, already consumed).
// Workgroups past the listed rows return at once (the grid is sized for
// every row listed).
__global__ __launch_bounds__(kThreads, 1) void k_lm_kl_redo(LmCombineArgs a) {
  __shared__ __align__(16) bf16_t lds[2 * kBufElems + kStashBytes / 2];
  Stash stash{reinterpret_cast<uint32_t*>(lds + 2 * kBufElems) + threadIdx.x};
  // workgroup ids row tile by row tile (slices fastest): the busy ones, the
  // first ceil(n / 256) row tiles, are the lowest ids, which the dispatcher
  // deals round-robin over all the XCDs (a per-XCD regrouping as in the
  // forward would put them all on the first XCDs)
  const int n = *a.kl_count;
  const int rt = (int)(blockIdx.x / (unsigned)a.kl_nslice), sl = (int)(blockIdx.x % (unsigned)a.kl_nslice);
  const int64_t row0 = (int64_t)rt * TM;
  if (row0 >= n) return;
  const int wr = wave_id() >> 2;
  const int ntiles = (a.Vd + TN - 1) / TN;
  const int per = (ntiles + a.kl_nslice - 1) / a.kl_nslice;
  const int t_begin = sl * per, t_end = min(ntiles, (sl + 1) * per);
  const int lrow = nt_lane_row();
  KlList<kLmRedoM> kl;
  kl.init();
  auto save = [&]() {
#pragma unroll
    for (int j = 0; j < kStashWords / 2; ++j) {
      stash.put(2 * j, kl.v[j]);
      stash.put(2 * j + 1, kl.i[j]);
    }
  };
  auto load = [&]() {
#pragma unroll
    for (int j = 0; j < kStashWords / 2; ++j) {
      stash.get(2 * j, kl.v[j]);
      stash.get(2 * j + 1, kl.i[j]);
    }
  };
  save();
  if (t_begin < t_end) {
    NtGather src{static_cast<const bf16_t*>(a.Wt), static_cast<const bf16_t*>(a.Ht), a.d2t, a.Vt, a.kl_list, a.Vd,
                 row0, n, a.H, t_begin, t_end};
    nt_stream(lds, src, [&](int tile, NtAcc& acc) {
      nt_row_per_lane(acc);
      if (row0 + lrow >= n) return;
      load();
#pragma unroll 1
      for (int ch = 0; ch < 16; ++ch) {
        const int c = tile * TN + nt_chunk_col(ch);
        if (c >= a.Vd) break;
        float x[8];
        nt_chunk(acc, ch, x);
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (c + k < a.Vd) kl.offer(x[k], c + k);
      }
      save();
    });
  }
  load();
  LmKlEntry* klred = reinterpret_cast<LmKlEntry*>(lds);  // [TM rows][2 segments][kLmRedoM]
#pragma unroll
  for (int j = 0; j < kLmRedoM; ++j) klred[(lrow * 2 + wr) * kLmRedoM + j] = LmKlEntry{kl.v[j], kl.i[j]};
  __syncthreads();
  if (threadIdx.x < TM && row0 + threadIdx.x < n) {
    KlList<kLmRedoM> m;
    m.init();
#pragma unroll 1
    for (int e = 0; e < 2 * kLmRedoM; ++e) {
      const LmKlEntry en = klred[threadIdx.x * 2 * kLmRedoM + e];
      m.offer(en.val, en.idx);
    }
    const int64_t r = a.kl_list[row0 + threadIdx.x];
    LmKlEntry* rec = a.kl_part + r * a.kl_stride + sl * kLmRedoM;
#pragma unroll
    for (int j = 0; j < kLmRedoM; ++j) rec[j] = LmKlEntry{m.v[j], m.i[j]};
  }
}

// The KL term of each listed row from its slice records: an exact wavefront
// top-K over the records' entries, then the row term.  One wavefront per
// listed row; the grid is sized for every row listed.
__global__ __launch_bounds__(256) void k_lm_kl_redo_select(LmCombineArgs a) {
  __shared__ float kl_bv[4 * kTopKCap];
  __shared__ int kl_bi[4 * kTopKCap];
  const int lane = threadIdx.x & 63;
  const int wave = wave_id();
  const int64_t f = (int64_t)blockIdx.x * 4 + wave;
  if (f >= *a.kl_count) return;
  WaveTopK tk;
  tk.init(kl_bv + wave * kTopKCap, kl_bi + wave * kTopKCap, a.kl_k);
  const int64_t r = a.kl_list[f];
  offer_entries(tk, a.kl_part + r * a.kl_stride, a.kl_nslice * kLmRedoM, lane);
  tk.finish(lane);
  lm_kl_row(a, tk, r, lane);
}

// ----------------------------------------------------------- backward pass ---
// g for one 256x256 tile of the recomputed draft logits, written in bf16 to
// G [R, ldg] (columns [0, Vd) only).
__global__ __launch_bounds__(kThreads, 1) void k_lm_bwd_g(LmBwdArgs a) {
  __shared__ __align__(16) bf16_t lds[2 * kBufElems];
  const int nrt = (int)((a.R + TM - 1) / TM);
  int rt, ct;
  tile_of(blockIdx.x, nrt, (a.Vd + TN - 1) / TN, rt, ct);
  const int64_t row0 = (int64_t)rt * TM;
  const int64_t r = row0 + nt_lane_row();
  NtRows src{static_cast<const bf16_t*>(a.Wd), static_cast<const bf16_t*>(a.Hd), a.Vd, row0, a.R, a.H, ct,
             ct + 1};
  nt_stream(lds, src, [&](int tile, NtAcc& acc) {
    nt_row_per_lane(acc);
    if (r >= a.R) return;
    const float c2 = a.inv_tq * kLog2e;
    const float k = a.scale * a.inv_tq;
    const float ca = a.coef_a[r], cb = a.coef_b[r];
    const bool zero = ca == 0.0f && cb == 0.0f;
    const float lse2 = a.lse_q[r] * kLog2e;
    const float kab = k * (ca + cb), ka = k * ca, kb = k * cb;
    const int zd = a.tok_d[r], zt = a.tok_t[r];
    bf16_t* G = static_cast<bf16_t*>(a.G) + r * a.ldg;
#pragma unroll 1
    for (int ch = 0; ch < 16; ++ch) {
      const int c = tile * TN + nt_chunk_col(ch);
      const int nvalid = min(8, a.Vd - c);
      if (nvalid <= 0) break;
      float x[8], gv[8];
      nt_chunk(acc, ch, x);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float t = kab * __builtin_amdgcn_exp2f(fmaf(x[j], c2, -lse2));
        t -= (c + j == zd) ? ka : 0.0f;
        t -= (c + j == zt) ? kb : 0.0f;
        gv[j] = zero ? 0.0f : t;
      }
      if (nvalid == 8) {
        store8(G + c, gv);
      } else {
        for (int j = 0; j < nvalid; ++j) store1(G + c + j, gv[j]);
      }
    }
  });
}

// With the KL term: g at the row's top-K members, recomputed in fp32 with the
// term's sparse gradient added, then rounded once (the entries k_lm_bwd_g
// wrote there are replaced).  One wavefront per row.
__global__ __launch_bounds__(256) void k_lm_kl_fix(LmBwdArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + wave_id();
  if (r >= a.R) return;
  const bf16_t* hd = static_cast<const bf16_t*>(a.Hd) + r * a.H;
  const bf16_t* Wd = static_cast<const bf16_t*>(a.Wd);
  const float ca = a.coef_a[r], cb = a.coef_b[r];
  const float c2 = a.inv_tq * kLog2e;
  const float k = a.scale * a.inv_tq;
  const float kab = k * (ca + cb), ka = k * ca, kb = k * cb;
  const float lse2 = a.lse_q[r] * kLog2e;
  const int zd = a.tok_d[r], zt = a.tok_t[r];
  bf16_t* G = static_cast<bf16_t*>(a.G) + r * a.ldg;
  for (int j = 0; j < a.kl_k; ++j) {
    const int v = a.kl_idx[r * a.kl_k + j];
    if ((uint32_t)v >= (uint32_t)a.Vd) continue;
    float t = 0.0f;
    if (ca != 0.0f || cb != 0.0f) {
      const float x = wave_dot(hd, Wd + (int64_t)v * a.H, a.H, lane);
      t = kab * __builtin_amdgcn_exp2f(fmaf(x, c2, -lse2));
      t -= (v == zd) ? ka : 0.0f;
      t -= (v == zt) ? kb : 0.0f;
    }
    t += a.kl_grad[r * a.kl_k + j];
    if (lane == 0) store1(G + v, t);
  }
}

// dH[R, H] = G[R, Vd] W_d[Vd, H] (bf16 in, fp32 accumulation, bf16 out): one
// 256x256 tile per workgroup, W_d (K-major) as U, G as V: a lane owns a row of
// dH and stores 16 consecutive columns at a time.
template <bool BIG>
__global__ __launch_bounds__(kThreads, 1) void k_lm_gemm_nn(LmGemmNNArgs a) {
  __shared__ __align__(16) bf16_t lds[2 * kBufElems];
  const int lane = threadIdx.x & 63, w = wave_id();
  const int nrt = (int)((a.M + TM - 1) / TM);
  int rt, ct;
  tile_of(blockIdx.x, nrt, (a.N + TN - 1) / TN, rt, ct);
  const int64_t row0 = (int64_t)rt * TM;
  const int n0 = ct * TN;
  NtTile<KRows<BIG>, false> src{{static_cast<const bf16_t*>(a.B), a.ldb, a.N, n0, a.K},
                           {static_cast<const bf16_t*>(a.A), a.lda, row0, a.M, a.K},
                           a.K};
  nt_stream(lds, src, [&](int, NtAcc& acc) {
    bf16_t* C = static_cast<bf16_t*>(a.C);
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int64_t row = row0 + g * 128 + (w & 3) * 32 + (lane & 31);
      if (row >= a.M) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = n0 + (q >> 1) * 128 + (w >> 2) * 64 + (lane >> 5) * 32 + (q & 1) * 16;
        if (col >= a.N) continue;  // N and col are multiples of 16
        const f32x16& c = acc[q >> 1][g][q & 1];
#pragma unroll
        for (int e = 0; e < 16; e += 8) {
          const float v[8] = {c[e], c[e + 1], c[e + 2], c[e + 3], c[e + 4], c[e + 5], c[e + 6], c[e + 7]};
          store8(C + row * a.ldc + col + e, v);
        }
      }
    }
  });
}

// dW = A^T B (fp32): A = g [R, ldg] (K = R rows, M = V_d columns), B = H_d
// [R, H], both K-major: B as U, A as V.
template <bool BIG>
__global__ __launch_bounds__(kThreads, 1) void k_lm_gemm_tn(LmGemmTNArgs a) {
  __shared__ __align__(16) bf16_t lds[2 * kBufElems];
  const int lane = threadIdx.x & 63, w = wave_id();
  const int nrt = (int)((a.M + TM - 1) / TM);
  int rt, ct;
  tile_of(blockIdx.x, nrt, (a.N + TN - 1) / TN, rt, ct);
  const int64_t row0 = (int64_t)rt * TM;
  const int n0 = ct * TN;
  NtTile<KMajor<false, BIG>, true> src{{static_cast<const bf16_t*>(a.B), a.ldb, a.N, n0, a.K},
                                  {static_cast<const bf16_t*>(a.A), a.lda, (int)a.M, (int)row0, a.K},
                                  a.K};
  nt_stream(lds, src, [&](int, NtAcc& acc) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int64_t row = row0 + g * 128 + (w & 3) * 32 + (lane & 31);
      if (row >= a.M) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = n0 + (q >> 1) * 128 + (w >> 2) * 64 + (lane >> 5) * 32 + (q & 1) * 16;
        if (col >= a.N) continue;  // N and col are multiples of 16
        const f32x16& c = acc[q >> 1][g][q & 1];
#pragma unroll
        for (int e = 0; e < 16; e += 4)
          *reinterpret_cast<float4*>(a.C + row * a.ldc + col + e) = make_float4(c[e], c[e + 1], c[e + 2], c[e + 3]);
      }
    }
  });
}

}  // namespace

hipError_t launch_lm_inv(const int32_t* d2t, int Vd, int Vt, int32_t* inv, int32_t* err, uint32_t* clear, int nclear,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_lm_inv, dim3((unsigned)((Vt + kInvCols - 1) / kInvCols)), dim3(kInvThreads), 0, s, d2t, Vd, Vt,
                     inv, err, clear, nclear);
  return hipGetLastError();
}

hipError_t launch_lm_fwd(const LmFwdArgs& a, hipStream_t s) {
  const int64_t nrt = (a.R + TM - 1) / TM;
  if (a.tile_part != nullptr) {
    const dim3 grid((unsigned)(nrt * (lm_runs(a.Vt, a.run_tiles) + lm_runs(a.Vd, a.run_tiles))));
    if (a.kl_part != nullptr)
      hipLaunchKernelGGL((k_lm_fwd<true, true>), grid, dim3(kThreads), 0, s, a);
    else
      hipLaunchKernelGGL((k_lm_fwd<false, true>), grid, dim3(kThreads), 0, s, a);
    const int64_t n = a.R * (a.nslice_t + a.nslice_d);
    hipLaunchKernelGGL(k_lm_fold, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)(nrt * (a.nslice_t + a.nslice_d)));
  if (a.kl_part != nullptr)
    hipLaunchKernelGGL((k_lm_fwd<true, false>), grid, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((k_lm_fwd<false, false>), grid, dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lm_combine(const LmCombineArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.R + 3) / 4));
  if (a.kl_k > 0)
    hipLaunchKernelGGL(k_lm_combine<true>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_lm_combine<false>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lm_kl_reset(const LmCombineArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_lm_kl_reset, dim3(1), dim3(64), 0, s, a.kl_count);
  return hipGetLastError();
}

hipError_t launch_lm_kl_redo(const LmCombineArgs& a, hipStream_t s) {
  const unsigned nrt = (unsigned)((a.R + TM - 1) / TM);
  hipLaunchKernelGGL(k_lm_kl_redo, dim3(nrt * (unsigned)a.kl_nslice), dim3(kThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_lm_kl_redo_select, dim3((unsigned)((a.R + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lm_bwd(const LmBwdArgs& a, hipStream_t s) {
  const int64_t nrt = (a.R + TM - 1) / TM;
  hipLaunchKernelGGL(k_lm_bwd_g, dim3((unsigned)(nrt * ((a.Vd + TN - 1) / TN))), dim3(kThreads), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.kl_idx != nullptr) {
    hipLaunchKernelGGL(k_lm_kl_fix, dim3((unsigned)((a.R + 3) / 4)), dim3(256), 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  LmGemmNNArgs gm{a.G, a.Wd, a.dH, a.R, a.ldg, a.H, a.H, a.H, a.Vd};
  const bool big = a.ldg >= kBigStride;
  hipLaunchKernelGGL(big ? k_lm_gemm_nn<true> : k_lm_gemm_nn<false>, dim3((unsigned)(nrt * ((a.H + TN - 1) / TN))),
                     dim3(kThreads), 0, s, gm);
  e = hipGetLastError();
  if (e != hipSuccess || a.dW == nullptr) return e;
  LmGemmTNArgs tn{a.G, a.Hd, a.dW, a.Vd, a.ldg, a.H, a.H, a.H, (int32_t)a.R};
  const int64_t nvt = (a.Vd + TM - 1) / TM;
  hipLaunchKernelGGL(big ? k_lm_gemm_tn<true> : k_lm_gemm_tn<false>, dim3((unsigned)(nvt * ((a.H + TN - 1) / TN))),
                     dim3(kThreads), 0, s, tn);
  return hipGetLastError();
}

}  // namespace vsd
