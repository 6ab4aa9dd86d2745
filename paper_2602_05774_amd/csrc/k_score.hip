// Path scoring (vsd_score_paths).
//
// k_score_rows   W wavefronts per row: online log-sum-exp of X/T_q over the
//                draft vocabulary and of Y/T_p over the whole target
//                vocabulary (128-bit loads, exp2 with folded scales, per-lane
//                chunk max), then the token gathers giving log q, log p and
//                log alpha = min(0, log p - log q) of the three families
//                (Sec. "Preliminary", Eq. acc).
// k_combine      one workgroup per position, one thread per path: prefix sums
//                over depth (Eqs. kappa, survival_def, accepted_len_cond), the
//                oracle gate and the correction (Alg. 2, Alg. 1), ARW beta
//                (Eq. beta_update), CAR zeta (Eq. zeta_update), the loss of
//                Eq. advance / Eq. basic and the per-row coefficients a, b.
//                k_combine_small takes up to 64 paths of depth up to 8.
// k_loss_total   one workgroup: loss_scale * sum over positions, fixed order
//                (k_combine_small forms it itself for few positions).
//
// With the top-K renormalised KL term on (VSD (KL) variant, Eq. klv),
// k_score_rows also selects, while it streams the target row, the K mapped
// target tokens with the largest logits (exact wavefront top-K, vsd_topk.hpp;
// the mapped values are gathered through the map next to the blocks being
// streamed), then forms p_hat and q_hat renormalised over them, the row's term
// -sum p_hat log q_hat and its gradient coefficients; k_combine adds the
// per-position average over paths to the loss.
#include "vsd_device.hpp"
#include "vsd_kernels.hpp"
#include "vsd_topk.hpp"

namespace vsd {

namespace {

constexpr int kStep = 8 * kWave;     // columns of one chunk: 8 per lane
constexpr int kU = 4;                // chunks of a block, in flight together
constexpr int kBlockCols = kU * kStep;
// A row's log-sum-exp is summed over segments of whole blocks, lane by lane:
// the segments of a group merge in order, the groups merge in order, the
// lanes meet last.  The segments depend on the row's length only: 4 groups of
// 4 from kSegs16Blocks blocks on, 4 groups of one down to 4 blocks, else one
// segment.  Of W = 16 wavefronts each takes one place of a group, of W = 4
// each a group, so every W gives bitwise the same sums (a place without a
// segment adds nothing).
constexpr int kGroups = kScoreGroups, kSegs16Blocks = kScoreSegs16Blocks;
static_assert(kBlockCols == kScoreBlockCols, "blocks as score_waves counts them");

__device__ __host__ inline int blocks_of(int V) { return (V + kBlockCols - 1) / kBlockCols; }
struct Segs {
  int groups, per;  // segments per group
};
__device__ __host__ inline Segs segs_of(int blocks) {
  return blocks >= kSegs16Blocks ? Segs{kGroups, 4} : blocks >= kGroups ? Segs{kGroups, 1} : Segs{1, 1};
}

// Online log-sum-exp of the columns one lane has seen.
//
// With c = float(log2(e) / T), each lane keeps mraw (its largest raw logit),
// mc = float(mraw * c) and s = sum_v exp2(fma(x_v, c, -mc)); the fused
// multiply-add forms x_v * c exactly, so s is exactly consistent with mc.
// Because float(mraw * c) differs from mraw * c by delta = fma(mraw, c, -mc)
// (exactly representable), log2 sum_v 2^((x_v - mraw) c) = log2(s) - delta.
// Callers then form log q(z) = (x_z - mraw)/T - ln2 (log2 s - delta), which
// keeps full float32 precision even when |x/T| is in the hundreds (the
// shifted difference never rounds against a large log-sum-exp).
struct LseState {
  float mraw = kNegBig, mc = kNegBig, s = 0.0f;

  // 8 columns x with largest value cm (columns past the row hold -inf)
  __device__ __forceinline__ void add8(const float (&x)[8], float cm, float c) {
    if (cm > mraw) {
      const float nmc = cm * c;
      s = lse_scaled(s, mc - nmc);
      mc = nmc;
      mraw = cm;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) s += __builtin_amdgcn_exp2f(fmaf(x[k], c, -mc));
  }
  __device__ __forceinline__ void merge(const LseState& o) {
    lse2_merge(mc, s, o.mc, o.s);
    mraw = fmaxf(mraw, o.mraw);
  }
};

struct RowLse {
  float mraw;  // wavefront max of the raw logits
  float tail;  // ln sum_v exp((x_v - mraw)/T)  (>= 0)
};
__device__ __forceinline__ RowLse reduce_lse(LseState t, float c) {
  wave_lse2(t.mc, t.s);        // every lane's mc = float(its mraw * c): the max commutes
  t.mraw = wave_max(t.mraw);
  const float delta = fmaf(t.mraw, c, -t.mc);
  return RowLse{t.mraw, (log2f(t.s) - delta) * kLn2};
}

// Wavefront w of W: its segments of the row, merged as far as they are its
// own.  Each chunk's values also go to seen(x, column of the lane's first
// value, valid columns, largest value); before() runs once a block's loads
// are issued, after() once it is summed.
template <int W, typename T, class Before, class Seen, class After>
__device__ __forceinline__ LseState segments_lse(const T* row, int V, int w, float c, int lane, Before&& before,
                                                 Seen&& seen, After&& after) {
  static_assert(W == 1 || W == kGroups || W == 4 * kGroups, "a row, a group or a segment");
  const int blocks = blocks_of(V), whole = V / kBlockCols;
  const Segs n = segs_of(blocks);
  const int segs = n.groups * n.per;
  int seg = 0, last = segs;
  if (W == kGroups) {
    seg = w * n.per;
    last = w < n.groups ? seg + n.per : seg;
  } else if (W > 1) {
    seg = (w >> 2) * n.per + (w & 3);
    last = (w >> 2) < n.groups && (w & 3) < n.per ? seg + 1 : seg;
  }
  LseState sum, group;
  int in_group = 0, groups = 0;
  for (; seg < last; ++seg) {
    LseState st;
    int b = blocks * seg / segs;
    const int end = blocks * (seg + 1) / segs, whole_end = min(end, whole);
    for (; b < whole_end; ++b) {
      const int col = b * kBlockCols + lane * 8;
      float x[kU][8];
#pragma unroll
      for (int u = 0; u < kU; ++u) load8(row + col + u * kStep, x[u]);
      before();
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const float cm = max8(x[u]);
        st.add8(x[u], cm, c);
        seen(x[u], col + u * kStep, 8, cm);
      }
      after();
    }
    if (b < end) {  // the row's partial last block
      before();
      for (int chunk = b * kBlockCols; chunk < V; chunk += kStep) {
        const int base = chunk + lane * 8, nvalid = min(8, V - base);
        float x[8];
        if (nvalid >= 8) {
          load8(row + base, x);
        } else {
#pragma unroll
          for (int k = 0; k < 8; ++k) x[k] = k < nvalid ? load1(row + base + k) : -INFINITY;
        }
        const float cm = max8(x);
        st.add8(x, cm, c);
        seen(x, base, nvalid, cm);
      }
      after();
    }
    if (in_group == 0)
      group = st;
    else
      group.merge(st);
    if (W <= kGroups && ++in_group == n.per) {
      if (groups == 0)
        sum = group;
      else
        sum.merge(group);
      ++groups;
      in_group = 0;
    }
  }
  return W <= kGroups ? sum : group;
}

// The states the W > 1 wavefronts of a row left in LDS, merged as W = 1 does.
template <int W>
struct LseParts {
  float mraw[W][kWave], s[W][kWave];
  __device__ __forceinline__ void put(int w, int lane, const LseState& st) {
    mraw[w][lane] = st.mraw;
    s[w][lane] = st.s;
  }
  __device__ __forceinline__ LseState get(int w, int lane, float c) const {
    const float m = mraw[w][lane];
    return LseState{m, m == kNegBig ? kNegBig : m * c, s[w][lane]};  // mc is always float(mraw c) once a column was seen
  }
  __device__ __forceinline__ LseState merged(int lane, float c) const {
    constexpr int n = W / kGroups;  // parts of a group
    LseState row;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      LseState group = get(g * n, lane, c);
#pragma unroll
      for (int k = 1; k < n; ++k) group.merge(get(g * n + k, lane, c));
      if (g == 0) row = group; else row.merge(group);
    }
    return row;
  }
};

// Wavefront w of W: the target row's segments, also selecting the K mapped
// target logits of largest value (wavefront top-K; value = raw target logit,
// index = its draft index).  With a map, block by block of the stream the
// wavefront offers the next of its draft chunks (512 indices): each lane
// gathers Y[d2t[v]] for v = 512 chunk + 64 k + lane, k < 8.  For an ascending
// map (about four target columns per draft index) those columns lie near the
// block just streamed, so the gathers find their lines in L2.  Draft chunks
// left when the stream ends (a map onto fewer columns than 4 per index) are
// offered after it.  Without a map the streamed values themselves are
// offered.  Only values at or above the top-K threshold are ever appended, so
// a slice whose largest value is below it in every lane offers nothing: one
// ballot decides.  Map entries are range-checked at the kernel's start.
template <typename T, bool MAPPED, int W>
__device__ LseState row_lse_topk(const T* row, int V, float c, int lane, int w, WaveTopK& tk, const int32_t* d2t,
                                 int Vd) {
  bool seeded = false;
  auto offer = [&](const float (&x)[8], int base, uint32_t bits, float vmax, auto idx_of) {
    if (!seeded) {  // the threshold from the lanes' largest offered values of the first slice
      seeded = true;
      tk.seed_lane_max(vmax, lane);
      tk.offer8(x, base, bits, idx_of, lane);
      return;
    }
    if (__ballot(vmax >= tk.thv) == 0ull) return;  // vmax: the lane's largest offered value
    tk.append8(x, base, bits, idx_of, lane);
  };
  // Draft chunk dc (512 indices; lane-strided: k-th value of a lane is draft
  // index 512 dc + 64 k + lane) is offered from gathered raw values.  Its map
  // entries are loaded one iteration ahead and its gathers are issued right
  // after the stream loads of the iteration that offers it, so the
  // log-sum-exp work of the block covers their latency.  The gathers go
  // through the row's buffer resource, which keeps every access in the row.
  // Only the last chunk can hold indices past V_d (their slots offer
  // nothing).
  const int chunks = MAPPED ? (Vd + kStep - 1) / kStep : 0;
  const int nfull_dc = MAPPED ? Vd / kStep : 0;
  const int dc_end = chunks * (w + 1) / W;
  int dc = chunks * w / W;
  uint32_t tmap[8];
  T graw[8];
  const __amdgpu_buffer_rsrc_t yrow = row_rsrc(row, row_bytes(row, V));
  auto load_map = [&](int d) {
    if (d < nfull_dc) {
#pragma unroll
      for (int k = 0; k < 8; ++k) tmap[k] = (uint32_t)d2t[d * kStep + k * kWave + lane];
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int v = d * kStep + k * kWave + lane;
        tmap[k] = v < Vd ? (uint32_t)d2t[v] : 0u;
      }
    }
  };
  auto gather = [&]() {
#pragma unroll
    for (int k = 0; k < 8; ++k) buf_gather(yrow, tmap[k], graw[k]);
  };
  auto offer_gathered = [&](int d) {
    float y[8];
    uint32_t bits = 0xFFu;
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = load1(&graw[k]);
    if (d >= nfull_dc) {
      bits = 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool in = d * kStep + k * kWave + lane < Vd;
        y[k] = in ? y[k] : -INFINITY;
        bits |= in ? (1u << k) : 0u;
      }
    }
    const int base = d * kStep + lane;
    offer(y, 0, bits, max8(y), [&](int k) { return base + k * kWave; });
  };
  if (MAPPED && dc < dc_end) load_map(dc);
  bool gathered = false;
  const LseState st = segments_lse<W>(
      row, V, w, c, lane,
      [&] {
        gathered = MAPPED && dc < dc_end;
        if (gathered) gather();
      },
      [&](const float (&x)[8], int base, int nvalid, float cm) {
        if (MAPPED) return;
        const uint32_t bits = nvalid <= 0 ? 0u : nvalid >= 8 ? 0xFFu : (1u << nvalid) - 1u;
        offer(x, base, bits, cm, [](int col) { return col; });
      },
      [&] {
        if (!gathered) return;
        offer_gathered(dc);
        if (++dc < dc_end) load_map(dc);
      });
  for (; MAPPED && dc < dc_end;) {  // draft chunks past the streamed blocks
    gather();
    offer_gathered(dc);
    if (++dc < dc_end) load_map(dc);
  }
  return st;
}

template <typename T, bool MAPPED, bool KL, int W>
__global__ __launch_bounds__(W == 1 ? 256 : W * kWave) void k_score_rows(ScoreRowArgs a) {
  constexpr int kWaves = W == 1 ? 4 : W;  // W = 1: four rows per workgroup
  __shared__ float kl_bv[KL ? kWaves * kTopKCap : 1];
  __shared__ int kl_bi[KL ? kWaves * kTopKCap : 1];
  __shared__ LseParts<W == 1 ? 1 : W> qpart, ppart;
  __shared__ float prow[2];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int w = W == 1 ? 0 : wave;
  if (KL && MAPPED) {  // every map entry is range-checked once per launch (the top-K gathers do not test theirs)
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < a.Vd; v += (int64_t)gridDim.x * blockDim.x)
      if ((uint32_t)a.d2t[v] >= (uint32_t)a.Vt) report_error(a.err, VSD_DEVERR_MAP_RANGE);
  }
  const int64_t r = W == 1 ? (int64_t)blockIdx.x * kWaves + wave : (int64_t)blockIdx.x;
  if (r >= a.R) return;
  const int i = (int)(r % a.L);
  const int64_t path = r / a.L;
  int d = a.L;
  if (a.depth != nullptr) {
    d = a.depth[path];
    if (d < 1 || d > a.L) {
      if (lane == 0 && w == 0) report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  if (i >= d) {  // masked slot (W > 1: the whole workgroup): nothing is read, every output is zero
    if (w != 0) return;
    if (lane < 3) {
      a.la[r * 3 + lane] = 0.0f;
      a.lq[r * 3 + lane] = 0.0f;
    }
    if (lane == 0) {
      if (a.lse_q != nullptr) a.lse_q[r] = 0.0f;
      if (a.lse_p != nullptr) a.lse_p[r] = 0.0f;
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
  const T* X = static_cast<const T*>(a.X) + r * a.ld_d;
  const T* Y = static_cast<const T*>(a.Y) + r * a.ld_t;
  const float cq = a.inv_tq * kLog2e, cp = a.inv_tp * kLog2e;
  auto stream = [&](const T* row, int V, float c) {
    return segments_lse<W>(row, V, w, c, lane, [] {}, [](const float(&)[8], int, int, float) {}, [] {});
  };
  LseState qs = stream(X, a.Vd, cq), ps;
  WaveTopK tk;
  if (KL) {
    tk.init(kl_bv + wave * kTopKCap, kl_bi + wave * kTopKCap, a.kl_k);
    ps = row_lse_topk<T, MAPPED, W>(Y, a.Vt, cp, lane, w, tk, a.d2t, a.Vd);
  } else {
    ps = stream(Y, a.Vt, cp);
  }
  RowLse q, p;
  if (W == 1) {
    q = reduce_lse(qs, cq);
    p = reduce_lse(ps, cp);
    if (KL) tk.finish(lane);
  } else {
    qpart.put(w, lane, qs);
    ppart.put(w, lane, ps);
    if (KL) tk.finish(lane);
    __syncthreads();
    if (KL && w != 0 && lane < a.kl_k) {  // each wavefront's best K into the first one's buffer (-inf: no entry)
      kl_bv[w * a.kl_k + lane] = lane < tk.n ? tk.bv[lane] : -INFINITY;
      kl_bi[w * a.kl_k + lane] = lane < tk.n ? tk.bi[lane] : 0x7FFFFFFF;
    }
    if (w == 1) {  // the second wavefront forms the target's statistics next to the first
      p = reduce_lse(ppart.merged(lane, cp), cp);
      if (lane == 0) {
        prow[0] = p.mraw;
        prow[1] = p.tail;
      }
    }
    if (w == 0) {
      q = reduce_lse(qpart.merged(lane, cq), cq);
      if (KL && lane >= tk.n && lane < a.kl_k) kl_bv[lane] = -INFINITY;
    }
    __syncthreads();
    if (w != 0) return;
    p = RowLse{prow[0], prow[1]};
    if (KL) {
      tk.n = W * a.kl_k;  // <= 256 of the buffer's 640 entries
      tk.finish(lane);
    }
  }
  const float lse_q = q.mraw * a.inv_tq + q.tail;
  const float lse_p = p.mraw * a.inv_tp + p.tail;
  const float gap = lse_gap(p.mraw, p.tail, a.inv_tp, q.mraw, q.tail, a.inv_tq);
  if (lane >= a.fam_lo && lane < a.fam_hi) {  // lane f gathers family f
    const int32_t z = a.tok[lane][r];
    float lq = 0.0f, la = 0.0f;
    if ((uint32_t)z >= (uint32_t)a.Vd) {
      report_error(a.err, VSD_DEVERR_TOKEN_RANGE);
    } else {
      const int32_t zt = a.d2t != nullptr ? a.d2t[z] : z;
      if ((uint32_t)zt >= (uint32_t)a.Vt) {
        report_error(a.err, VSD_DEVERR_MAP_RANGE);
      } else {
        const float xz = load1(X + z);
        lq = (xz - q.mraw) * a.inv_tq - q.tail;
        la = log_alpha_of(xz, load1(Y + zt), a.inv_tq, a.inv_tp, gap);
      }
    }
    a.la[r * 3 + lane] = la;
    a.lq[r * 3 + lane] = lq;
  }
  if (lane == 0) {
    if (a.lse_q != nullptr) a.lse_q[r] = lse_q;
    if (a.lse_p != nullptr) a.lse_p[r] = lse_p;
  }
  if (KL)
    kl_row_term(tk, X, a.Vd, a.inv_tq, a.inv_tp, a.kl_gscale, a.kl_idx + r * a.kl_k, a.kl_grad + r * a.kl_k,
                a.kl_row + r, lane);
}

// Deterministic block reductions: butterfly within each wavefront, then the
// per-wavefront partials combined in wavefront order by every thread.
__device__ __forceinline__ float block_sum(float v, float* smem) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) smem[w] = v;
  __syncthreads();
  float t = 0.0f;
  for (int k = 0; k < nw; ++k) t += smem[k];
  return t;
}

__device__ __forceinline__ float block_max(float v, float* smem) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_max(v);
  __syncthreads();
  if (lane == 0) smem[w] = v;
  __syncthreads();
  float t = kNegBig;
  for (int k = 0; k < nw; ++k) t = fmaxf(t, smem[k]);
  return t;
}

__device__ __forceinline__ int block_sum_int(int v, int* smem) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  v = wave_sum_int(v);
  __syncthreads();
  if (lane == 0) smem[w] = v;
  __syncthreads();
  int t = 0;
  for (int k = 0; k < nw; ++k) t += smem[k];
  return t;
}

__global__ __launch_bounds__(1024) void k_combine(CombineArgs a) {
  __shared__ float redf[16];
  __shared__ int redi[16];
  const int pos = blockIdx.x;
  const int s = threadIdx.x;
  const bool real = s < a.N;
  int d = 0;
  if (real) {
    d = a.depth != nullptr ? a.depth[(int64_t)pos * a.N + s] : a.L;
    if (d < 1 || d > a.L) {
      report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  const int64_t row0 = ((int64_t)pos * a.N + s) * a.L;
  float LSd = 0.0f, LSt = 0.0f, LSg = 0.0f, LQd = 0.0f, LQt = 0.0f;
  float ea = 0.0f, wsum = 0.0f, lsum = 0.0f, klsum = 0.0f;
  for (int l = 0; l < a.L; ++l) {
    const bool live = real && l < d;
    const int64_t row = row0 + l;
    if (live && a.kl_row != nullptr) klsum += a.kl_row[row];
    if (live) {  // prefix sums of log alpha (log survival) and of log q
      LSd += a.la[row * 3 + 0];
      LSt += a.la[row * 3 + 1];
      LSg += a.la[row * 3 + 2];
      LQd += a.lq[row * 3 + 0];
      LQt += a.lq[row * 3 + 1];
    }
    // Alg. 2 gate on z~; Alg. 1 substitutes z' when it fails.
    const bool acc = live && (LSd >= LSg);
    const bool val = live && (acc || LSt >= LSg);
    // ARW: leave-one-out acceptance rate among live paths with o' > 0; all
    // o' at one level share w(l), which cancels (acc implies val).
    const int n_acc = block_sum_int(acc ? 1 : 0, redi);
    const int n_val = block_sum_int(val ? 1 : 0, redi);
    const int num = n_acc - (acc ? 1 : 0);
    const int den = n_val - (val ? 1 : 0);
    const float beta = (live && den > 0) ? (float)num / (float)den : 0.0f;
    // CAR: softmax over live paths of confidence / tau.
    const float conf = a.car_input == VSD_CAR_PROB ? expf(LQd) : LQd;
    const float cmax = block_max(live ? conf : kNegBig, redf);
    const float e = live ? expf((conf - cmax) * a.inv_tau) : 0.0f;
    const float esum = block_sum(e, redf);
    const float zeta = live ? e / esum : 0.0f;
    const float c = a.mode == VSD_GRAD_ARW_CAR ? beta * zeta : a.mode == VSD_GRAD_ARW ? beta : 0.0f;
    const float o = val ? a.w[l] : 0.0f;
    const float surv = live ? expf(LSd) : 0.0f;
    ea += surv;
    wsum += o;
    if (live) lsum += o * ((acc ? LQd : LQt) - c * LQd);
    if (real) {
      if (a.survival) a.survival[row] = surv;
      if (a.acc_flag) a.acc_flag[row] = acc ? 1 : 0;
      if (a.val_flag) a.val_flag[row] = val ? 1 : 0;
      if (a.o_prime) a.o_prime[row] = o;
      if (a.beta) a.beta[row] = beta;
      if (a.zeta) a.zeta[row] = zeta;
      // level-l terms of the coefficient suffix sums, finished below
      a.coef_a[row] = o * ((acc ? 1.0f : 0.0f) - c);
      a.coef_b[row] = o * (acc ? 0.0f : 1.0f);
    }
  }
  const float W = block_sum(wsum, redf);
  const float total = block_sum(lsum, redf);
  if (real) {
    // a_{s,i} = (1/W) sum_{l>=i} o'(I~ - c),  b_{s,i} = (1/W) sum_{l>=i} o'(1 - I~)
    float acc_a = 0.0f, acc_b = 0.0f;
    for (int l = a.L - 1; l >= 0; --l) {
      const int64_t row = row0 + l;
      if (l < d && W > 0.0f) {
        acc_a += a.coef_a[row];
        acc_b += a.coef_b[row];
        a.coef_a[row] = acc_a / W;
        a.coef_b[row] = acc_b / W;
      } else {
        a.coef_a[row] = 0.0f;
        a.coef_b[row] = 0.0f;
      }
    }
    if (a.ea) a.ea[(int64_t)pos * a.N + s] = ea;
  }
  if (a.kl_row != nullptr) {
    // KL_x = (1/N) sum over live slots of the row terms, weighted into the loss
    const float kl = block_sum(klsum, redf) / (float)a.N;
    if (threadIdx.x == 0) {
      a.loss_pos[pos] = (W > 0.0f ? -total / W : 0.0f) + a.kl_weight * kl;
      if (a.kl_pos != nullptr) a.kl_pos[pos] = kl;
    }
  } else if (threadIdx.x == 0) {
    a.loss_pos[pos] = W > 0.0f ? -total / W : 0.0f;
  }
}

__global__ __launch_bounds__(256) void k_loss_total(const float* loss_pos, int32_t P, float scale, float* out) {
  __shared__ float red[16];
  float t = 0.0f;
  for (int p = threadIdx.x; p < P; p += blockDim.x) t += loss_pos[p];
  t = block_sum(t, red);
  if (threadIdx.x == 0) *out = scale * t;
}

// Sum and maximum over groups of G lanes.  G = 8 takes the first three steps
// of the wavefront's reduction; the remaining ones would only add zeros (keep
// the maximum), so a group's result is that of k_combine's workgroup.
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(G == 8 || G == kWave, "eight lanes or the wavefront");
  if (G == kWave) return wave_sum(v);
  v += dpp_f<kDppQuad1>(v);
  v += dpp_f<kDppQuad2>(v);
  v += dpp_f<kDppHalfMirror>(v);
  return v;
}
template <int G>
__device__ __forceinline__ float group_max(float v) {
  if (G == kWave) return wave_max(v);
  v = fmaxf(v, dpp_f<kDppQuad1>(v));
  v = fmaxf(v, dpp_f<kDppQuad2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  return v;
}
template <int G>
__device__ __forceinline__ int group_count(bool b) {
  const uint64_t m = __ballot(b);
  return G == kWave ? __builtin_popcountll(m)
                    : __builtin_popcount((uint32_t)(m >> (threadIdx.x & (kWave - G))) & ((1u << (G & 31)) - 1u));
}

// k_combine for N <= G paths of depth L <= 8: G lanes per position, several
// positions per wavefront, the path's values and coefficient terms in
// registers.  The kernel is a chain of latencies: k_combine reads a level,
// reduces it over a workgroup (ten barriers) and goes on, then reads its
// coefficient terms back; here all levels load at once and no step needs a
// barrier.  Every operation and its order are k_combine's, so are the results.
// 512 positions of 8 paths, depth 8: 15.8 -> 9.9 us.
// Up to kSmallOneRows rows one workgroup holds all positions and also forms the
// total (16 positions of 4 paths, depth 3: 7.6 + 1.5 -> 5.1 us and a launch
// less; 128 positions of 8 paths, depth 5, in one workgroup: 3 us slower than
// spread over the CUs with the total in its own launch).
constexpr int kSmallL = 8, kSmallThreads = 1024;
constexpr int64_t kSmallOneRows = 2048;
template <int G>
__global__ __launch_bounds__(kSmallThreads) void k_combine_small(CombineArgs a) {
  __shared__ float loss[kSmallThreads / G];
  const int per_block = (int)blockDim.x / G;
  const int here = (int)threadIdx.x / G;
  const int64_t pos = (int64_t)blockIdx.x * per_block + here;
  const int s = threadIdx.x % G;
  const bool real = pos < a.P && s < a.N;  // lanes without a path take part in the reductions
  const int64_t path = pos * a.N + s, row0 = path * a.L;
  int d = 0;
  if (real) {
    d = a.depth != nullptr ? a.depth[path] : a.L;
    if (d < 1 || d > a.L) {
      report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  float la[kSmallL][3], lq[kSmallL][2], kl[kSmallL];
#pragma unroll
  for (int l = 0; l < kSmallL; ++l) {
    const bool live = l < d;
    const int64_t row = row0 + l;
#pragma unroll
    for (int f = 0; f < 3; ++f) la[l][f] = live ? a.la[row * 3 + f] : 0.0f;
#pragma unroll
    for (int f = 0; f < 2; ++f) lq[l][f] = live ? a.lq[row * 3 + f] : 0.0f;
    kl[l] = live && a.kl_row != nullptr ? a.kl_row[row] : 0.0f;
  }
  float LSd = 0.0f, LSt = 0.0f, LSg = 0.0f, LQd = 0.0f, LQt = 0.0f;
  float ea = 0.0f, wsum = 0.0f, lsum = 0.0f, klsum = 0.0f;
  float ta[kSmallL], tb[kSmallL];
#pragma unroll
  for (int l = 0; l < kSmallL; ++l) {
    if (l >= a.L) break;
    const bool live = l < d;
    const int64_t row = row0 + l;
    if (live) {  // prefix sums of log alpha (log survival) and of log q
      klsum += kl[l];
      LSd += la[l][0];
      LSt += la[l][1];
      LSg += la[l][2];
      LQd += lq[l][0];
      LQt += lq[l][1];
    }
    const bool acc = live && (LSd >= LSg);
    const bool val = live && (acc || LSt >= LSg);
    const int num = group_count<G>(acc) - (acc ? 1 : 0);
    const int den = group_count<G>(val) - (val ? 1 : 0);
    const float beta = (live && den > 0) ? (float)num / (float)den : 0.0f;
    const float conf = a.car_input == VSD_CAR_PROB ? expf(LQd) : LQd;
    const float cmax = group_max<G>(live ? conf : kNegBig);
    const float e = live ? expf((conf - cmax) * a.inv_tau) : 0.0f;
    const float esum = group_sum<G>(e);
    const float zeta = live ? e / esum : 0.0f;
    const float c = a.mode == VSD_GRAD_ARW_CAR ? beta * zeta : a.mode == VSD_GRAD_ARW ? beta : 0.0f;
    const float o = val ? a.w[l] : 0.0f;
    const float surv = live ? expf(LSd) : 0.0f;
    ea += surv;
    wsum += o;
    if (live) lsum += o * ((acc ? LQd : LQt) - c * LQd);
    ta[l] = o * ((acc ? 1.0f : 0.0f) - c);
    tb[l] = o * (acc ? 0.0f : 1.0f);
    if (real) {
      if (a.survival) a.survival[row] = surv;
      if (a.acc_flag) a.acc_flag[row] = acc ? 1 : 0;
      if (a.val_flag) a.val_flag[row] = val ? 1 : 0;
      if (a.o_prime) a.o_prime[row] = o;
      if (a.beta) a.beta[row] = beta;
      if (a.zeta) a.zeta[row] = zeta;
    }
  }
  const float W = group_sum<G>(wsum);
  const float total = group_sum<G>(lsum);
  if (real) {
    float acc_a = 0.0f, acc_b = 0.0f;
#pragma unroll
    for (int l = kSmallL - 1; l >= 0; --l) {
      if (l >= a.L) continue;
      const bool on = l < d && W > 0.0f;
      acc_a = on ? acc_a + ta[l] : acc_a;
      acc_b = on ? acc_b + tb[l] : acc_b;
      a.coef_a[row0 + l] = on ? acc_a / W : 0.0f;
      a.coef_b[row0 + l] = on ? acc_b / W : 0.0f;
    }
    if (a.ea) a.ea[path] = ea;
  }
  float loss_pos = W > 0.0f ? -total / W : 0.0f;
  if (a.kl_row != nullptr) {
    const float klx = group_sum<G>(klsum) / (float)a.N;
    loss_pos += a.kl_weight * klx;
    if (real && s == 0 && a.kl_pos != nullptr) a.kl_pos[pos] = klx;
  }
  if (real && s == 0) a.loss_pos[pos] = loss_pos;
  if (a.loss_total == nullptr || gridDim.x != 1) return;
  if (s == 0) loss[here] = real ? loss_pos : 0.0f;
  __syncthreads();
  if (threadIdx.x < kWave) {  // k_loss_total's sum: wavefronts of positions, then in order
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < kSmallThreads / G; k += kWave) {
      const int p = k + (int)threadIdx.x;
      t += wave_sum(p < per_block ? loss[p] : 0.0f);
    }
    if (threadIdx.x == 0) *a.loss_total = a.loss_scale * t;
  }
}

// true: the launch also formed the total
template <int G>
bool launch_combine_small(const CombineArgs& a, hipStream_t s) {
  const int64_t threads = (int64_t)a.P * G;
  const bool one = threads <= kSmallThreads && (int64_t)a.P * a.N * a.L <= kSmallOneRows;
  const unsigned block = one ? (unsigned)((threads + kWave - 1) / kWave * kWave) : kWave;
  hipLaunchKernelGGL(k_combine_small<G>, dim3((unsigned)((threads + block - 1) / block)), dim3(block), 0, s, a);
  return one;
}

template <typename T, int W>
void launch_rows_w(const ScoreRowArgs& a, hipStream_t s) {
  constexpr int rows = W == 1 ? 4 : 1;
  const dim3 grid((unsigned)((a.R + rows - 1) / rows)), block(W == 1 ? 256 : W * kWave);
  if (a.kl_k == 0)  // without the KL term the map is read only for the tokens
    hipLaunchKernelGGL((k_score_rows<T, false, false, W>), grid, block, 0, s, a);
  else if (a.d2t != nullptr)
    hipLaunchKernelGGL((k_score_rows<T, true, true, W>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((k_score_rows<T, false, true, W>), grid, block, 0, s, a);
}

// (score_waves holds the rule and its measurements.)
template <typename T>
hipError_t launch_rows_t(const ScoreRowArgs& a, hipStream_t s) {
  switch (score_waves(a.R, a.Vd, a.Vt, (int)sizeof(T), a.kl_k > 0, a.depth != nullptr)) {
    case 16: launch_rows_w<T, 16>(a, s); break;
    case 4: launch_rows_w<T, 4>(a, s); break;
    default: launch_rows_w<T, 1>(a, s); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_rows(const ScoreRowArgs& a, bool bf16, hipStream_t s) {
  return bf16 ? launch_rows_t<bf16_t>(a, s) : launch_rows_t<float>(a, s);
}

hipError_t launch_combine(const CombineArgs& a, hipStream_t s) {
  bool total = false;
  if (a.N <= kWave && a.L <= kSmallL) {
    total = a.N <= 8 ? launch_combine_small<8>(a, s) : launch_combine_small<kWave>(a, s);
  } else {
    const int threads = ((a.N + kWave - 1) / kWave) * kWave;
    hipLaunchKernelGGL(k_combine, dim3((unsigned)a.P), dim3(threads), 0, s, a);
  }
  if (a.loss_total != nullptr && !total)
    hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(256), 0, s, a.loss_pos, a.P, a.loss_scale, a.loss_total);
  return hipGetLastError();
}

}  // namespace vsd
