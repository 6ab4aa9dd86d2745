// E-step sampling (Alg. 1 proposal z~ ~ q and correction z' ~ p; Alg. 2
// greedy reference z-bar), optionally fused with the row statistics of path
// scoring (log-sum-exps and the drawn tokens' log q / log alpha).
//
// A pair of wavefronts per row (or per span of a row, below): the draft
// wavefront draws z~ from X (and, fused, accumulates the draft log-sum-exp);
// the target wavefront draws z' and z-bar from the mapped target logits.  Fused with a map, the target row is streamed
// for its log-sum-exp in lock-step with the draft chunks (2048 target
// elements per 512-element chunk, half by each wavefront), so the mapped
// gathers of a chunk find its cache lines in L2 and every logit is read from
// memory once.  The wavefronts meet at a barrier at the end of the row.
//
// A row is a serial chain of chunks, so few rows are split over 4 or 2 pairs,
// each on its span of the row's chunks.  The tokens are maxima and do not
// depend on the split; the log-sum-exps are summed over segments of chunks
// that depend on V_d only, against one reference per row, and the segments'
// sums are added in order, so every split gives bitwise the same floats.
//
// Each lane owns 8 consecutive vocabulary indices of every 512-element chunk
// (128-bit loads; the Philox counters of the sampler definition cover 4
// consecutive indices) and draws the Philox word of every element.  The
// normative key float(x/T) + G costs two logarithms with a correctly rounded
// division each, so it is evaluated only for elements that can still win:
// with d = 1 - u (exact on the 2^-24 grid), G = -ln(-ln(1 - d)) <= -ln(d)
// because -ln(1 - d) >= d, and -ln(d) <= (24 - log2 j') ln 2 for the integer
// j' = (~w) >> 8 <= 2^24 d.  An element whose bound x/T - ln(d) + margin is
// below the running maximum (the lane's own, or the wavefront's, refreshed
// whenever a lane improves on it) cannot be the argmax; every other element
// gets its exact key.  The margin exceeds every rounding involved, so the
// tokens are exactly those of the definition.  Lanes visit indices in
// increasing order and keep the first of equal keys; a butterfly reduction
// with the same tie rule yields the row's tokens, independent of geometry.
//
// Mapped target logits are gathered in lane-strided order (gather k of a
// chunk loads indices chunk + 64k + lane: a few consecutive cache lines per
// instruction) and transposed to the lane-contiguous layout through a
// per-row LDS tile.  Chunks are software pipelined: the next chunk's map
// entries and rows are loaded while the current chunk is drawn, and the target
// gathers of the next chunk are issued at the end of the current one.
//
// k_sample_step draws one depth of a rollout with exact context: three
// wavefronts per path, each on its own row (z~ from the draft row along z~,
// z' from the target row along z', z-bar from the target row along z-bar),
// with the counters of the slot's global row, so equal rows give exactly the
// tokens k_sample draws.
//
// With the top-K renormalised KL term (one-pass mode), the target wavefront
// also offers each chunk's mapped target logits, already in draft-index
// order, to an exact wavefront top-K (vsd_topk.hpp) and, after the row, forms
// the term over the K (as k_score_rows does).
#include "vsd_device.hpp"
#include "vsd_kernels.hpp"
#include "vsd_draw.hpp"
#include "vsd_topk.hpp"

namespace vsd {

namespace {

constexpr int kRowsPerBlock = 2;   // 256 threads = 2 rows x 2 wavefronts
constexpr int kChunk = 8 * kWave;  // draft elements per wavefront step
constexpr int64_t kStepPathsW16 = 128, kStepPathsW4 = 768;  // most paths of a k_sample_step launch with W = 16, 4
constexpr int kStream = 2 * kChunk;  // target elements each wavefront streams per chunk (fused, mapped)

template <typename T>
__device__ __forceinline__ T neg_inf();
template <>
__device__ __forceinline__ float neg_inf<float>() { return -INFINITY; }
template <>
__device__ __forceinline__ bf16_t neg_inf<bf16_t>() { return (bf16_t)0xFF80u; }

// Per-lane log-sum-exp of v/T in the scorer's exactly consistent form:
// mraw = a raw reference value, mc = float(mraw * c), s = sum of
// exp2(fma(v, c, -mc)), c = log2(e)/T.  Elements equal to -inf add nothing.
// Every identity used after the row (the reduction, the rounding correction
// of mc, log q) holds for any reference, so the reference need not be the
// maximum.  It is the same in every lane (scalar registers) and begins each
// segment at the largest value of the row's first chunk:
//   add8_lazy   moves it only when some lane's largest value (already known to
//               the caller) exceeds it by more than 16 / c, to that value, until
//               none does: one compare per slice, and an exponent below 16, so
//               that the multiply-add rounds little.  On peaked rows every
//               segment moves it one or two times, so a move takes one lane
//               read and no reduction or division (51 -> 16 VALU instructions);
//               with an unsplit row's reference from the chunk at hand, 32 768
//               rows of 32k + 32k peaked columns, 44 % of them masked, take 779
//               us (824 before, 811 with one running sum per lane and row);
//               (PER_LANE: to each lane's own largest value.  An unmapped row
//               of one segment is short: finding its first reference took 3 %
//               of the kernel.)
//   add8_fixed  keeps it and tracks nothing: one fma, exp2 and add per
//               element (a stream whose maxima nobody needs);
//   add8        moves a lane's own up to its running maximum (the careful
//               form).
// A lane whose sum leaves [0, 2^64] (an element about 64 / c above a fixed
// reference, a first chunk of -inf, or a NaN) is recomputed with add8
// (bad()).  Its reference then lies above those of lanes that were not, and
// merging scales their sums by 2^(difference), which underflows past 2^-126:
// sums below 2^64 lose nothing there (with a limit of 2^120 up to a
// percent of a row's sum was lost).
__device__ __forceinline__ float uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
template <bool PER_LANE>
struct LaneLse {
  static constexpr bool kPerLane = PER_LANE;
  float mraw = kNegBig, mc = kNegBig, s = 0.0f;
  float lim = kNegBig;  // add8_lazy's threshold in raw units, mraw + 16 / c
  float ref = kNegBig, ref_mc = kNegBig, ref_lim = kNegBig;  // where every segment begins
  float closed_mraw = kNegBig, closed_mc = kNegBig, closed = 0.0f;  // the segments merged so far

  __device__ __forceinline__ static float scaled(float m, float c) { return m > kNegBig ? m * c : kNegBig; }

  // m: the same in every lane (1/c within an ulp: the threshold need not be exact)
  __device__ __forceinline__ void move(float m, float c) {
    mraw = uniform_f(fmaxf(m, kNegBig));
    mc = uniform_f(scaled(m, c));
    lim = uniform_f(fmaf(16.0f, __builtin_amdgcn_rcpf(c), mraw));
  }
  __device__ __forceinline__ void refer(float m, float c) {
    move(m, c);
    ref = closed_mraw = mraw;
    ref_mc = closed_mc = mc;
    ref_lim = lim;
  }
  __device__ __forceinline__ void next_segment() {
    s = 0.0f;
    mraw = ref;
    mc = ref_mc;
    lim = ref_lim;
  }
  __device__ __forceinline__ void merge_closed(float omraw, float omc, float os) {
    if (omc == closed_mc) {  // nearly always: no reference moved
      closed += os;
      return;
    }
    lse2_merge(closed_mc, closed, omc, os);
    closed_mraw = fmaxf(closed_mraw, omraw);
  }
  __device__ __forceinline__ void take_closed() {
    mraw = closed_mraw;
    mc = closed_mc;
    s = closed;
  }

  __device__ __forceinline__ void add8_lazy(const float (&v)[8], float vmax, float c) {
    if (PER_LANE) {
      if (__builtin_expect(__ballot(vmax > lim) != 0ull, 0) && vmax > lim) {
        const float nmc = vmax * c;
        s = lse_scaled(s, mc - nmc);
        mc = nmc;
        mraw = vmax;
        lim = fmaf(16.0f, __builtin_amdgcn_rcpf(c), vmax);
      }
      add8_fixed(v, c);
      return;
    }
    uint64_t over = __ballot(vmax > lim);
    while (__builtin_expect(over != 0ull, 0)) {
      const float omc = mc;
      move(lane_f(vmax, __builtin_ctzll(over)), c);
      s = lse_scaled(s, omc - mc);
      over = __ballot(vmax > lim);
    }
    add8_fixed(v, c);
  }

  __device__ __forceinline__ void add8_fixed(const float (&v)[8], float c) {
#pragma unroll
    for (int k = 0; k < 8; ++k) s += __builtin_amdgcn_exp2f(fmaf(v[k], c, -mc));
  }

  __device__ __forceinline__ bool bad() const { return !(s <= 0x1p64f); }

  __device__ __forceinline__ void add8(const float (&v)[8], float c) {
    const float cm = max8(v);
    if (cm > mraw) {
      const float nmc = cm * c;
      s = lse_scaled(s, mc - nmc);
      mc = nmc;
      mraw = cm;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s += __builtin_amdgcn_exp2f(fmaf(v[k], c, -mc));
  }

  // Wavefront reduction (every lane ends with the row's values).
  __device__ __forceinline__ void reduce() {
    wave_lse2(mc, s);
    mraw = wave_max(mraw);
  }
};

// What the two wavefronts of a row hand to the epilogue.
struct RowShared {
  Best d, t, g;
  float q_mraw, q_mc, q_s;   // draft log-sum-exp (reduced)
  float p_mraw[2], p_mc[2], p_s[2];  // target log-sum-exp partials of the two wavefronts
};

// The lane's slice of a row at g (elements past n read as -inf).
template <typename T>
__device__ __forceinline__ void load_slice(const T* Y, int g, int n, float (&v)[8]) {
  if (g + 8 <= n) {
    load8(Y + g, v);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = (g + k < n) ? load1(Y + g + k) : -INFINITY;
  }
}

// Log-sum-exp of target elements [lo, hi) of a row (guarded at both ends);
// FIXED: against the lane's fixed reference, a whole range without guards.
template <bool FIXED, typename T, class Lse>
__device__ __forceinline__ void stream_lse(const T* Y, int lo, int hi, int lane, float c2, Lse& acc) {
  if (FIXED && hi - lo == kStream) {
    float v0[8], v1[8];
    load8(Y + lo + lane * 8, v0);
    load8(Y + lo + kChunk + lane * 8, v1);
    acc.add8_fixed(v0, c2);
    acc.add8_fixed(v1, c2);
    return;
  }
  for (int g = lo + lane * 8; g - lane * 8 < hi; g += kChunk) {
    float v[8];
    load_slice(Y, g, hi, v);
    if (FIXED)
      acc.add8_fixed(v, c2);
    else
      acc.add8(v, c2);
  }
}

// The reference of a row's fixed-reference sums: the largest value of its
// first chunk (in every lane).
template <typename T>
__device__ __forceinline__ float first_max(const T* row, int n, int lane) {
  float v[8];
  load_slice(row, lane * 8, n, v);
  return wave_max(max8(v));
}

// The same from the row's first whole chunk when that is at hand (an unsplit
// row: a load of its own would be a serial step more for every row; a row
// shorter than a chunk keeps the empty reference, which its first slice moves).
template <typename T>
__device__ __forceinline__ float slice_max(const Raw8<T>& r) {
  float v[8];
  r.unpack(v);
  return wave_max(max8(v));
}

// Wavefront w of a pair streams the target ranges [lo, lo + kStream) with
// lo = w kStream + j 2 kStream; the careful recomputation repeats every range.
template <typename T, class Lse>
__device__ void stream_redo(const T* Y, int w, int Vt, int lane, float c2, Lse& acc) {
  acc = Lse{};
  for (int lo = w * kStream; lo < Vt; lo += 2 * kStream) stream_lse<false>(Y, lo, min(lo + kStream, Vt), lane, c2, acc);
}

// Careful recomputation over the lane's slices g = lane 8 + j kChunk of a row
// of n elements (the chunk layout of both wavefronts).
template <typename T, class Lse>
__device__ void row_redo(const T* X, int n, int lane, float c, Lse& acc) {
  acc = Lse{};
  for (int g = lane * 8; g < n; g += kChunk) {
    float v[8];
    load_slice(X, g, n, v);
    acc.add8(v, c);
  }
}

// log2 of the segments of a row with n whole chunks (a function of its length only).
constexpr int kMaxSegShift = 2;
__device__ __host__ inline int seg_shift(int n) { return n >= 8 ? kMaxSegShift : 0; }

// The whole chunks [begin, end) of a row that one wavefront takes, made of the
// segments from `seg` on; the last span of a row also takes what follows the
// whole chunks, as part of the last segment.
struct Span {
  int begin, end;
  bool last;
  int seg, shift;  // the row has 2^shift segments
  __device__ __forceinline__ int segs() const { return 1 << shift; }
  __device__ __forceinline__ int seg_end(int n, int g) const { return (n * (g + 1)) >> shift; }
};
// Part p of 2^w_shift of a row with n whole chunks; the segments are at least
// as many, or, where no sums are taken, the parts.
__device__ __forceinline__ Span span_of(int n, int p, int w_shift, bool fused) {
  const int shift = fused ? seg_shift(n) : w_shift, g = p << (shift - w_shift), g_end = (p + 1) << (shift - w_shift);
  return Span{(n * g) >> shift, (n * g_end) >> shift, p == (1 << w_shift) - 1, g, shift};
}
constexpr int log2_of(int w) { return w <= 1 ? 0 : 1 + log2_of(w / 2); }

// The draft wavefront of a row: z~ and, fused, the draft log-sum-exp and one
// half of the target stream.
template <typename T, bool MAPPED, bool FUSED, bool SPLIT, class Lse, class Close>
__device__ void draft_wave(const T* X, const T* Y, int Vd, int Vt, Span sp, FamilyDraw& f, Lse& lq, Lse& lp,
                           float cp2, int lane, Close&& close) {
  const int nfull = Vd / kChunk;
  int seg = sp.seg, seg_end = sp.seg_end(nfull, seg);
  if (FUSED && (SPLIT || MAPPED)) lq.refer(first_max(X, Vd, lane), f.c2);
  if (FUSED && MAPPED) lp.refer(first_max(Y, Vt, lane), cp2);
  if (sp.begin < sp.end) {
    Raw8<T> xr;
    xr.load(X + sp.begin * kChunk + lane * 8);
    if (FUSED && !SPLIT && !MAPPED && !Lse::kPerLane) lq.refer(slice_max(xr), f.c2);
    for (int it = sp.begin; it < sp.end; ++it) {
      const int base = it * kChunk + lane * 8;
      Raw8<T> xn;
      if (it + 1 < sp.end) xn.load(X + base + kChunk);
      float x[8];
      xr.unpack(x);
      if (FUSED && MAPPED) {  // before the draws: the target wavefront's gathers of this
        // block's mapped elements then find its lines in L2 more often
        const int lo = it * 2 * kStream;
        stream_lse<true>(Y, min(lo, Vt), min(lo + kStream, Vt), lane, cp2, lp);
      }
      const float xmax = max8(x);
      if (FUSED) lq.add8_lazy(x, xmax, f.c2);
      f.draw8(base, x, xmax, it == sp.begin);
      xr = xn;
      if (FUSED && __builtin_expect(it + 1 == seg_end, 0) && seg + 1 < sp.segs()) {
        close(seg);
        seg_end = sp.seg_end(nfull, ++seg);
      }
    }
  }
  if (sp.last && nfull * kChunk < Vd) {  // the partial last chunk
    const int base = nfull * kChunk + lane * 8;
    const int nvalid = min(8, max(0, Vd - base));
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = k < nvalid ? load1(X + base + k) : -INFINITY;
    if (FUSED) lq.add8_lazy(x, max8(x), f.c2);
    f.draw(base, x, nvalid);
    if (FUSED && MAPPED) {
      const int lo = nfull * 2 * kStream;
      stream_lse<true>(Y, min(lo, Vt), min(lo + kStream, Vt), lane, cp2, lp);
    }
  }
  if (FUSED && MAPPED && sp.last) {  // target elements past the last chunk's block: even half-blocks
    const int nchunks = (Vd + kChunk - 1) / kChunk;
    for (int lo = nchunks * 2 * kStream; lo < Vt; lo += 2 * kStream)
      stream_lse<true>(Y, lo, min(lo + kStream, Vt), lane, cp2, lp);
  }
  if (FUSED && sp.last) close(seg);
}

// The target wavefront of a row: z' and z-bar and, fused, the target
// log-sum-exp (unmapped) or the other half of the target stream (mapped).
template <typename T, bool MAPPED, bool FUSED, bool SPLIT, bool KL, bool DRAW, class Lse, class Close>
__device__ void target_wave(const T* Y, const int32_t* d2t, T* tile, int Vd, int Vt, Span sp, FamilyDraw& f,
                            Best& bg, Lse& lp, bool& map_bad, WaveTopK& tk, int lane, Close&& close) {
  auto same = [](int col) { return col; };
  const int nfull = Vd / kChunk;
  // Greedy maximum: each lane keeps the first of its largest values, gw is the
  // wavefront's largest so far.  A chunk in which no lane's maximum ymax
  // (elements past nvalid hold -inf) exceeds gw changes nothing: an element
  // below gw cannot be the row's maximum, and one equal to gw comes after the
  // element that reached gw (every earlier chunk holds smaller indices), so it
  // loses the tie.  gw rises a few times per row (each a new record of the
  // row so far), whereas some lane of 64 improves on its own maximum in
  // almost every chunk.
  float gw = -INFINITY;
  auto greedy = [&](int base, const float (&y)[8], int nvalid, float ymax) {
    if (__ballot(ymax > gw) == 0ull) return;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool better = k < nvalid && y[k] > bg.key;
      bg.key = better ? y[k] : bg.key;
      bg.idx = better ? base + k : bg.idx;
    }
    gw = wave_max(bg.key);
  };
  int seg = sp.seg, seg_end = sp.seg_end(nfull, seg);
  if (FUSED && (SPLIT || MAPPED)) lp.refer(first_max(Y, Vt, lane), f.c2);
  if (sp.begin < sp.end) {
    uint32_t t[8];
    T g[8];
    Raw8<T> yr;
    auto load_map = [&](int chunk, uint32_t (&tt)[8]) {
#pragma unroll
      for (int k = 0; k < 8; ++k) tt[k] = (uint32_t)d2t[chunk + k * kWave + lane];
    };
    // map entries are range-checked once at the kernel's start; the buffer's
    // range check keeps every access in the row
    const __amdgpu_buffer_rsrc_t yrow = row_rsrc(Y, row_bytes(Y, Vt));
    auto gather = [&](const uint32_t (&tt)[8]) {
#pragma unroll
      for (int k = 0; k < 8; ++k) buf_gather(yrow, tt[k], g[k]);
    };
    if (MAPPED) {
      load_map(sp.begin * kChunk, t);
      gather(t);
    } else {
      yr.load(Y + sp.begin * kChunk + lane * 8);
      if (FUSED && !SPLIT && !Lse::kPerLane) lp.refer(slice_max(yr), f.c2);
    }
    for (int it = sp.begin; it < sp.end; ++it) {
      const int chunk = it * kChunk;
      const int base = chunk + lane * 8;
      const bool next = it + 1 < sp.end;
      uint32_t tn[8];
      Raw8<T> yn;
      if (next) {
        if (MAPPED)
          load_map(chunk + kChunk, tn);
        else
          yn.load(Y + base + kChunk);
      }
      if (FUSED && MAPPED) {  // this chunk's target block, second half
        const int lo = it * 2 * kStream + kStream;
        stream_lse<true>(Y, min(lo, Vt), min(lo + kStream, Vt), lane, f.c2, lp);
      }
      float y[8];
      if (MAPPED) {
        // transpose the gathered values through the LDS tile; LDS operations
        // of one wavefront execute in order, so no barrier is needed
#pragma unroll
        for (int k = 0; k < 8; ++k) tile[k * kWave + lane] = g[k];
        load8(tile + lane * 8, y);
      } else {
        yr.unpack(y);
      }
      const float ymax = max8(y);
      if (FUSED && !MAPPED) lp.add8_lazy(y, ymax, f.c2);
      greedy(base, y, 8, ymax);
      if (DRAW) f.draw8(base, y, ymax, it == sp.begin);
      if (KL) {  // a slice whose largest mapped value is below the top-K threshold offers nothing
        if (it == sp.begin) tk.seed_lane_max(ymax, lane);
        if (it == sp.begin || __ballot(ymax >= tk.thv) != 0ull) tk.append8(y, base, 0xFFu, same, lane);
      }
      if (next) {
        if (MAPPED)
          gather(tn);
        else
          yr = yn;
      }
      if (FUSED && __builtin_expect(it + 1 == seg_end, 0) && seg + 1 < sp.segs()) {
        close(seg);
        seg_end = sp.seg_end(nfull, ++seg);
      }
    }
  }
  if (sp.last && nfull * kChunk < Vd) {  // the partial last chunk
    const int chunk = nfull * kChunk;
    const int base = chunk + lane * 8;
    const int nvalid = min(8, max(0, Vd - base));
    if (FUSED && MAPPED) {
      const int lo = nfull * 2 * kStream + kStream;
      stream_lse<true>(Y, min(lo, Vt), min(lo + kStream, Vt), lane, f.c2, lp);
    }
    if (MAPPED) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int v = chunk + k * kWave + lane;
        const bool in = v < Vd;
        const uint32_t t = (uint32_t)d2t[in ? v : 0];
        const bool ok = t < (uint32_t)Vt;
        map_bad |= in && !ok;
        const T val = Y[ok ? t : 0u];
        tile[k * kWave + lane] = (in && ok) ? val : neg_inf<T>();
      }
    }
    float y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool in = k < nvalid;
      y[k] = in ? (MAPPED ? load1(tile + lane * 8 + k) : load1(Y + base + k)) : -INFINITY;
    }
    if (FUSED && !MAPPED) lp.add8_lazy(y, max8(y), f.c2);
    greedy(base, y, nvalid, max8(y));
    if (DRAW) f.draw(base, y, nvalid);
    if (KL) tk.offer8(y, base, nvalid > 0 ? (1u << nvalid) - 1u : 0u, same, lane);
  }
  if (FUSED && MAPPED && sp.last) {  // target elements past the last chunk's block: odd half-blocks
    const int nchunks = (Vd + kChunk - 1) / kChunk;
    for (int lo = nchunks * 2 * kStream + kStream; lo < Vt; lo += 2 * kStream)
      stream_lse<true>(Y, lo, min(lo + kStream, Vt), lane, f.c2, lp);
  }
  if (FUSED && sp.last) close(seg);
}

// Every entry of the map is range-checked once per launch (the gathers do not
// test theirs): thread t of n takes entries t, t + n, ...
__device__ __forceinline__ void check_map(const int32_t* d2t, int Vd, int Vt, int32_t* err, int64_t t, int64_t n) {
  for (; t < Vd; t += n)
    if ((uint32_t)d2t[t] >= (uint32_t)Vt) report_error(err, VSD_DEVERR_MAP_RANGE);
}

// W pairs of wavefronts per row; W = 1: kRowsPerBlock rows per workgroup.
// Wavefront 2 p is pair p's draft wavefront, 2 p + 1 its target wavefront.
// (Unmapped bf16 rows with W = 1 fill 96 scalar registers: with 97 a SIMD holds 7
// of these wavefronts instead of 8, and peaked rows took 5 % longer.)
// SEGS: the rows' sums have several segments (or there are none: the draws
// alone); without, W is 1 and a wavefront's accumulator is its row's sum.
template <typename T, bool MAPPED, bool FUSED, bool KL, int W, bool SEGS>
__global__ __launch_bounds__(W == 1 ? 256 : 2 * W * kWave) void k_sample(SampleArgs a) {
  constexpr int kRows = W == 1 ? kRowsPerBlock : 1, kPairs = W == 1 ? kRowsPerBlock : W;
  constexpr int kMaxSegs = 1 << kMaxSegShift;
  __shared__ __align__(16) T ytile[kPairs][kChunk];
  __shared__ RowShared sh[kRows];
  __shared__ float kl_bv[KL ? kPairs * kTopKCap : 1];
  __shared__ int kl_bi[KL ? kPairs * kTopKCap : 1];
  constexpr bool kParts = W > 1;
  __shared__ Best part[kParts ? W : 1][3];                            // the pairs' z~, z', z-bar
  __shared__ float part_s[kParts && FUSED ? kMaxSegs : 1][3][kWave];  // segment sums: lq, lp of both wavefronts
  __shared__ float part_m[kParts && FUSED ? kMaxSegs : 1][3];         // and their references
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int pair = wave >> 1;
  const int slot = W == 1 ? pair : 0;  // row within the block
  const bool draft_role = (wave & 1) == 0;
  if (MAPPED)
    check_map(a.d2t, a.Vd, a.Vt, a.err, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
              (int64_t)gridDim.x * blockDim.x);
  const int64_t r = (int64_t)blockIdx.x * kRows + slot;
  const bool active = r < a.R;
  bool live = false;
  if (active) {
    const int i = (int)(r % a.L);
    int d = a.L;
    if (a.depth != nullptr) {
      d = a.depth[r / a.L];
      if (d < 1 || d > a.L) {
        if (lane == 0 && draft_role && (W == 1 || pair == 0)) report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
        d = 0;
      }
    }
    live = i < d;
  }
  const T* X = static_cast<const T*>(a.X) + (active ? r : 0) * a.ld_d;
  const T* Y = static_cast<const T*>(a.Y) + (active ? r : 0) * a.ld_t;
  const float cq2 = a.inv_tq * kLog2e, cp2 = a.inv_tp * kLog2e;
  typedef LaneLse<!SEGS && !MAPPED> Lse;
  Lse lq, lp;
  WaveTopK tk;
  // A segment's sum: merged in place (W = 1) or left for the pairs' merge.
  auto close_acc = [&](Lse& l, int which, int seg) {
    if (!SEGS) return;
    if (kParts) {
      part_s[FUSED ? seg : 0][which][lane] = l.s;
      if (lane == 0) part_m[FUSED ? seg : 0][which] = l.mraw;
    } else {
      l.merge_closed(l.mraw, l.mc, l.s);
    }
    l.next_segment();
  };
  auto closed = [&](Lse& l, int which, float c) {
    if (!SEGS) return;
    if (kParts) {
      const int segs = 1 << seg_shift(a.Vd / kChunk);
      for (int g = 0; g < segs; ++g) {
        const float m = part_m[FUSED ? g : 0][which];
        l.merge_closed(m, Lse::scaled(m, c), part_s[FUSED ? g : 0][which][lane]);
      }
    }
    l.take_closed();
  };
  // The row's draft (target) results from the first pair's draft (target)
  // wavefront, whose references are those of every pair.
  auto finish_draft = [&](Best best) {
    if (FUSED) {
      closed(lq, 0, cq2);
      if (lq.bad()) row_redo(X, a.Vd, lane, cq2, lq);
      lq.reduce();
      if (MAPPED) {
        closed(lp, 1, cp2);
        if (lp.bad()) stream_redo(Y, 0, a.Vt, lane, cp2, lp);
      }
      lp.reduce();
    }
    if (lane == 0) {
      RowShared& o = sh[slot];
      o.d = best;
      o.q_mraw = lq.mraw;
      o.q_mc = lq.mc;
      o.q_s = lq.s;
      o.p_mraw[0] = lp.mraw;
      o.p_mc[0] = lp.mc;
      o.p_s[0] = lp.s;
    }
  };
  auto finish_target = [&](Best best, Best bg) {
    if (FUSED) {
      closed(lp, 2, cp2);
      if (lp.bad()) {
        if (MAPPED)
          stream_redo(Y, 1, a.Vt, lane, cp2, lp);
        else
          row_redo(Y, a.Vt, lane, cp2, lp);
      }
      lp.reduce();
    }
    if (lane == 0) {
      RowShared& o = sh[slot];
      o.t = best;
      o.g = bg;
      o.p_mraw[1] = lp.mraw;
      o.p_mc[1] = lp.mc;
      o.p_s[1] = lp.s;
    }
  };
  auto kl_term = [&]() {
    tk.finish(lane);
    kl_row_term(tk, X, a.Vd, a.inv_tq, a.inv_tp, a.kl_gscale, a.kl_idx + r * a.kl_k, a.kl_grad + r * a.kl_k,
                a.kl_row + r, lane);
  };
  if (live) {
    // without sums every pair takes an equal share of the chunks
    const Span sp = SEGS ? span_of(a.Vd / kChunk, W == 1 ? 0 : pair, log2_of(W), FUSED)
                         : Span{0, a.Vd / kChunk, true, 0, 0};
    if (draft_role) {
      FamilyDraw f{(uint32_t)r, 0u, a.offset, a.k0, a.k1, a.inv_tq, cq2};
      draft_wave<T, MAPPED, FUSED, kParts>(X, Y, a.Vd, a.Vt, sp, f, lq, lp, cp2, lane, [&](int seg) {
        close_acc(lq, 0, seg);
        if (MAPPED) close_acc(lp, 1, seg);
      });
      wave_argmax(f.best.key, f.best.idx);
      if (!kParts)
        finish_draft(f.best);
      else if (lane == 0)
        part[pair][0] = f.best;
    } else {
      FamilyDraw f{(uint32_t)r, 1u, a.offset, a.k0, a.k1, a.inv_tp, cp2};
      Best bg{-INFINITY, 0x7FFFFFFF};
      bool map_bad = false;
      if (KL) tk.init(kl_bv + pair * kTopKCap, kl_bi + pair * kTopKCap, a.kl_k);
      target_wave<T, MAPPED, FUSED, kParts, KL, true>(Y, a.d2t, ytile[pair], a.Vd, a.Vt, sp, f, bg, lp, map_bad, tk, lane,
                                              [&](int seg) { close_acc(lp, 2, seg); });
      if (map_bad) report_error(a.err, VSD_DEVERR_MAP_RANGE);
      wave_argmax(f.best.key, f.best.idx);
      wave_argmax(bg.key, bg.idx);
      if (!kParts) {
        if (KL) kl_term();
        finish_target(f.best, bg);
      } else {
        if (KL) tk.finish(lane);
        if (lane == 0) {
          part[pair][1] = f.best;
          part[pair][2] = bg;
        }
      }
    }
    if (kParts) {  // the pairs meet (a workgroup holds one row, so all its wavefronts are here)
      __syncthreads();
      auto merged = [&](int which) {  // the pairs' maxima: lane p holds pair p's
        Best b = lane < W ? part[kParts ? lane : 0][which] : Best{-INFINITY, 0x7FFFFFFF};
        wave_argmax(b.key, b.idx);
        return b;
      };
      if (wave == 0) finish_draft(merged(0));
      if (wave == 1) finish_target(merged(1), merged(2));
      if (KL && !draft_role && lane < a.kl_k) {  // every pair's best K into the first one's buffer (-inf: no entry)
        const bool has = lane < tk.n;
        if (pair > 0 || !has) {
          const float v = has ? tk.bv[lane] : -INFINITY;
          const int id = has ? tk.bi[lane] : 0x7FFFFFFF;
          kl_bv[pair * a.kl_k + lane] = v;
          kl_bi[pair * a.kl_k + lane] = id;
        }
      }
    }
  }
  __syncthreads();
  if (!active || draft_role || (kParts && pair > 0)) return;
  if (KL && kParts && live) {
    tk.n = W * a.kl_k;  // <= 64 of the buffer's 640 entries
    kl_term();
  }
  // epilogue, by the (first) target wavefront's first three lanes
  if (!live) {  // masked slot: tokens -1, score outputs 0, nothing read
    if (lane == 0) {
      a.tok_d[r] = -1;
      a.tok_t[r] = -1;
      a.tok_g[r] = -1;
    }
    if (FUSED) {
      if (lane < 3) {
        a.la[r * 3 + lane] = 0.0f;
        a.lq[r * 3 + lane] = 0.0f;
      }
      if (lane == 0) {
        a.lse_q[r] = 0.0f;
        if (a.lse_p != nullptr) a.lse_p[r] = 0.0f;
      }
    }
    if (KL) {
      if (lane < a.kl_k) {
        a.kl_idx[r * a.kl_k + lane] = -1;
        a.kl_grad[r * a.kl_k + lane] = 0.0f;
      }
      if (lane == 0) a.kl_row[r] = 0.0f;
    }
    return;
  }
  const RowShared& s = sh[slot];
  if (lane == 0) {
    a.tok_d[r] = s.d.idx;
    a.tok_t[r] = s.t.idx;
    a.tok_g[r] = s.g.idx;
  }
  if (FUSED && lane < 3) {
    // row statistics in the scorer's shifted form: log q(z) = (x_z - max)/T
    // - ln sum exp((x - max)/T), the scaled maximum's rounding corrected
    const float qt = (log2f(s.q_s) - fmaf(s.q_mraw, cq2, -s.q_mc)) * kLn2;
    const float pmc = fmaxf(s.p_mc[0], s.p_mc[1]);
    const float ps = s.p_s[0] * __builtin_amdgcn_exp2f(s.p_mc[0] - pmc) +
                     s.p_s[1] * __builtin_amdgcn_exp2f(s.p_mc[1] - pmc);
    const float pmraw = fmaxf(s.p_mraw[0], s.p_mraw[1]);
    const float pt = (log2f(ps) - fmaf(pmraw, cp2, -pmc)) * kLn2;
    const int z = lane == 0 ? s.d.idx : lane == 1 ? s.t.idx : s.g.idx;
    const float gap = lse_gap(pmraw, pt, a.inv_tp, s.q_mraw, qt, a.inv_tq);
    float lqv = 0.0f, lav = 0.0f;
    if ((uint32_t)z < (uint32_t)a.Vd) {
      const int32_t zt = MAPPED ? a.d2t[z] : z;
      if ((uint32_t)zt < (uint32_t)a.Vt) {
        const float xz = load1(X + z);
        lqv = (xz - s.q_mraw) * a.inv_tq - qt;
        lav = log_alpha_of(xz, load1(Y + zt), a.inv_tq, a.inv_tp, gap);
      }
    }
    a.la[r * 3 + lane] = lav;
    a.lq[r * 3 + lane] = lqv;
    if (lane == 0) {
      a.lse_q[r] = s.q_mraw * a.inv_tq + qt;
      if (a.lse_p != nullptr) a.lse_p[r] = pmraw * a.inv_tp + pt;
    }
  }
}

// W wavefronts per row, each on a contiguous span of its chunks, F rows
// (families) per workgroup: family = blockIdx.y with F = 1.  The spans'
// (key, index) maxima merge in index order, so the tokens do not depend on W.
template <typename T, bool MAPPED, int W, int F>
__global__ __launch_bounds__(F* W* kWave) void k_sample_step(SampleStepArgs a) {
  static_assert(F == 1 || W == 1, "several families only with one wavefront each");
  __shared__ __align__(16) T ytile[F * W][kChunk];
  __shared__ Best part[W];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int fam = F == 1 ? (int)blockIdx.y : wave;  // 0: z~, 1: z', 2: z-bar
  const int64_t path = blockIdx.x;                  // the grid has exactly one column per path
  if (MAPPED)
    check_map(a.d2t, a.Vd, a.Vt, a.err, ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x,
              (int64_t)gridDim.x * gridDim.y * blockDim.x);
  int d = a.L;
  if (a.depth != nullptr) {
    d = a.depth[path];
    if (d < 1 || d > a.L) {
      if (lane == 0 && wave == 0 && fam == 0) report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  const int64_t r = path * a.L + a.step;
  int32_t* out = fam == 0 ? a.tok_d : fam == 1 ? a.tok_t : a.tok_g;
  if (a.step >= d) {  // masked slot (the whole workgroup)
    if (lane == 0) out[r] = -1;
    return;
  }
  const Span sp = span_of(a.Vd / kChunk, F == 1 ? wave : 0, log2_of(W), false);
  auto no_sums = [](int) {};
  LaneLse<false> unused_q, unused_p;
  Best best{-INFINITY, 0x7FFFFFFF};
  if (fam == 0) {
    const T* X = static_cast<const T*>(a.X) + path * a.ld_d;
    FamilyDraw f{(uint32_t)r, 0u, a.offset, a.k0, a.k1, a.inv_tq, a.inv_tq * kLog2e};
    draft_wave<T, MAPPED, false, false>(X, nullptr, a.Vd, a.Vt, sp, f, unused_q, unused_p, 0.0f, lane, no_sums);
    best = f.best;
  } else {
    const T* Y = static_cast<const T*>(fam == 1 ? a.Y : a.Yg) + path * a.ld_t;
    FamilyDraw f{(uint32_t)r, 1u, a.offset, a.k0, a.k1, a.inv_tp, a.inv_tp * kLog2e};
    bool map_bad = false;
    WaveTopK unused_tk;
    if (fam == 1) {
      Best unused_bg{-INFINITY, 0x7FFFFFFF};
      target_wave<T, MAPPED, false, false, false, true>(Y, a.d2t, ytile[wave], a.Vd, a.Vt, sp, f, unused_bg, unused_p,
                                                 map_bad, unused_tk, lane, no_sums);
      best = f.best;
    } else {
      target_wave<T, MAPPED, false, false, false, false>(Y, a.d2t, ytile[wave], a.Vd, a.Vt, sp, f, best, unused_p, map_bad,
                                                  unused_tk, lane, no_sums);
    }
    if (map_bad) report_error(a.err, VSD_DEVERR_MAP_RANGE);
  }
  wave_argmax(best.key, best.idx);
  if (W > 1) {
    if (lane == 0) part[wave] = best;
    __syncthreads();
    if (wave != 0) return;
    // lane w holds span w's maximum; equal keys resolve to the smaller index
    best = lane < W ? part[lane] : Best{-INFINITY, 0x7FFFFFFF};
    wave_argmax(best.key, best.idx);
  }
  if (lane == 0) out[r] = best.idx;
}

template <typename T, int W, int F>
void launch_step_w(const SampleStepArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)a.paths, 3 / F);
  if (a.d2t != nullptr)
    hipLaunchKernelGGL((k_sample_step<T, true, W, F>), grid, dim3(F * W * kWave), 0, s, a);
  else
    hipLaunchKernelGGL((k_sample_step<T, false, W, F>), grid, dim3(F * W * kWave), 0, s, a);
}

// A row is a serial chain of chunks (load latency: about 0.85 us each), so
// few paths want many wavefronts per row and many paths one (each wavefront
// seeds and refines a filter threshold of its own).
// 32 000 draft and 128 256 target columns, us a depth, by W (the three
// wavefronts of a path in one workgroup and the map's check in a launch of
// its own took 56 us up to 128 paths, 110 at 1024):
//   paths    1     4    16
//      64   55    23    18
//     128   56    24    23
//     256   72    35    47
//     512   79    57    89
//    1024  109   112   174
// W wavefronts want at least a chunk each.
template <typename T>
hipError_t launch_step_t(const SampleStepArgs& a, hipStream_t s) {
  if (a.paths <= kStepPathsW16 && a.Vd >= 16 * kChunk)
    launch_step_w<T, 16, 1>(a, s);
  else if (a.paths <= kStepPathsW4 && a.Vd >= 4 * kChunk)
    launch_step_w<T, 4, 1>(a, s);
  else
    launch_step_w<T, 1, 3>(a, s);
  return hipGetLastError();
}

template <typename T, bool FUSED, bool KL, int W, bool SEGS>
void launch_w(const SampleArgs& a, hipStream_t s) {
  constexpr int rows = W == 1 ? kRowsPerBlock : 1;
  const dim3 grid((unsigned)((a.R + rows - 1) / rows)), block(W == 1 ? 256 : 2 * W * kWave);
  if (a.d2t != nullptr)
    hipLaunchKernelGGL((k_sample<T, true, FUSED, KL, W, SEGS>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_sample<T, false, FUSED, KL, W, SEGS>), grid, block, 0, s, a);
}

// Pairs per row.  A pair is a serial chain of chunks (1 to 1.5 us each, load
// latency), so few rows want several pairs; each pair seeds and refines filter
// thresholds (and a top-K list) of its own, so many rows want one.  us of
// vsd_sample_score_paths by W:
//                        rows      1       2       4
//   32k + 128k            256    75.2    51.7    41.8
//                         640    91.6    73.8    71.3
//                         768    95.0    75.2    71.9
//                         896   106.0    93.1    91.7
//                        1024   109.7    96.1    95.1
//                        1280   131.6   114.4   114.7
//                        1536   133.4   130.9   135.8
//                        2048   164.0   177.0   175.3
//   32k + 128k, KL        256    92.4    61.0    52.1
//                         640   109.0    86.4    87.7
//                         768   112.5    88.3    88.1
//                         896   123.2   106.4   111.4
//                        1280   147.5   127.8   135.0
//                        1536   152.0   143.7   157.5
//                        2048   181.3   194.7   202.3
//   32k + 32k             512    59.1    46.1    44.3
//                         768    70.0    55.8    55.9
//                         896    70.2    65.1    67.2
//                        1280    88.1    75.9    81.0
//                        1536    88.6    86.8    92.3
//   16k + 65k             512    46.9    40.0    37.5
//                         768    55.8    48.6    48.0
//                        1280    68.8    64.7    67.1
//                        1536    70.4    72.5    77.5
//   8k + 16k              512    28.7    26.2    25.0
//                         768    33.6    32.8    31.5
//   3k + 9k               512    20.1    20.2    21.0
// (The steps lie at multiples of the 256 CUs; from 896 to 1280 rows W = 4 is 1 %
// ahead on 32k + 128k and 3 to 7 % behind elsewhere.)
// Rows of one segment (below 8 chunks, where nothing splits) have kernels without
// the segments' bookkeeping: 15 624 rows of 1535 + 1535 columns 80.1 -> 75.6 us,
// of 4095 + 4095 122.8 -> 115.0 (76.6 and 118.8 before sums had segments).
constexpr int64_t kRowsW4 = 768, kRowsW2 = 1536, kShortRowsW4 = 512;
constexpr int kLongRow = 32;  // chunks
template <typename T, bool FUSED, bool KL>
hipError_t launch_t(const SampleArgs& a, hipStream_t s) {
  const int n = a.Vd / kChunk;
  const bool splits = seg_shift(n) == 2, lng = n >= kLongRow;
  if (splits && a.R <= (lng ? kRowsW4 : kShortRowsW4))
    launch_w<T, FUSED, KL, 4, true>(a, s);
  else if (splits && lng && a.R <= kRowsW2)
    launch_w<T, FUSED, KL, 2, true>(a, s);
  else if (splits || !FUSED)
    launch_w<T, FUSED, KL, 1, true>(a, s);
  else
    launch_w<T, FUSED, KL, 1, !FUSED>(a, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_sample(const SampleArgs& a, bool bf16, hipStream_t s) {
  const bool fused = a.lse_q != nullptr;
  const bool kl = fused && a.kl_k > 0;
  if (bf16) {
    if (kl) return launch_t<bf16_t, true, true>(a, s);
    return fused ? launch_t<bf16_t, true, false>(a, s) : launch_t<bf16_t, false, false>(a, s);
  }
  if (kl) return launch_t<float, true, true>(a, s);
  return fused ? launch_t<float, true, false>(a, s) : launch_t<float, false, false>(a, s);
}

hipError_t launch_sample_step(const SampleStepArgs& a, bool bf16, hipStream_t s) {
  return bf16 ? launch_step_t<bf16_t>(a, s) : launch_step_t<float>(a, s);
}

}  // namespace vsd
