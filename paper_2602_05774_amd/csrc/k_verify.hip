// Decode-time verification of the draft paths (vsd_verify_paths).
//
// Speculative decoding keeps the draft token z~_i with probability
// alpha_i = min(1, p(z~_i) / q(z~_i)) (Sec. "Preliminary", Eq. acc) and, at
// the first rejection, draws a replacement from the residual distribution
// norm(max(0, p - q)) over the target vocabulary, which ends the path.  The
// count of kept tokens is an unbiased draw of the accepted length whose mean
// given the path is sum_k S_k (Eq. accepted_len_cond).
//
// One workgroup of W wavefronts per path.  Lane i < d_s draws slot i's
// acceptance uniform (Philox counter (0, row, 2, offset), word 0) and tests
// Lambda(u) < log alpha (the normative log; log alpha from scoring); a ballot
// gives the first rejection (every wavefront of the workgroup takes the same
// decisions).  The wavefronts then stream contiguous ranges of the
// rejected row's target logits (8 consecutive target indices per lane,
// 128-bit loads), form p(t) and q(t) (draft logit through the inverse map, 0
// for target tokens the draft cannot propose) from the row's log-sum-exps,
// and draw the residual token by Gumbel-max over log(max(0, p - q)) with the
// sampler's exact candidate filter (family 3, counters over the target
// index); the ranges' (key, index) maxima merge in index order, so the token
// does not depend on W.  The draft logits are gathered through the inverse
// map by every lane (an unmapped column reads nothing and is answered with
// 0), so a slice's eight gathers are in flight together, and the next
// chunk's target logits and map entries load under the current one.
//
// Wavefronts per path: a path is a serial chain of chunks (about 0.8 us each,
// load latency) and a CU takes 23 us of VALU work for 128 256 columns, so few
// paths want several workgroups each and many paths few wavefronts (each
// seeds and refines a filter threshold of its own).  With a map and a
// workspace that also holds a result slot per path, up to kPathsSplit paths are
// split over workgroups of 4: their maxima meet in the slot by an atomic
// maximum of (key, smaller index), and the last workgroup to finish writes the
// token.  Without a map there is no workspace and a path has one workgroup.
//
// 128 256 target logits, map of 32 000, us of scoring and verification:
//   paths   one workgroup of 16   split over 256 / 1024 / 2048 workgroups in all
//       4        76                  42     42     42
//      64        77                  58     67     89
//     128        80                  75
//     256        92                        107    129
//   paths   one workgroup of 2      4     16  (scoring not yet split)
//     512       243                183    173
//    1024       329                270    285
//    4096       720                701    759

#include "vsd_device.hpp"
#include "vsd_draw.hpp"
#include "vsd_kernels.hpp"

namespace vsd {

namespace {

constexpr int64_t kPathsW16 = 512;  // most paths a launch of W = 16 takes
constexpr int64_t kSplitGroups = 256;  // workgroups of 4 a split launch aims at: one per CU
constexpr int kChunkV = 8 * kWave;  // target indices per chunk: 8 per lane

// One 8-element slice of the residual draw with its values formed only where
// the filter needs them.  vmax is the log of the slice's largest residual:
// the logarithm is increasing, so it is the slice's largest value, and it
// takes the slice test; the eight logarithms are taken only when some lane's
// slice passes that test or the slice seeds the threshold.  Otherwise the
// steps and their order are those of FamilyDraw::draw8.
template <class Vals>
__device__ __forceinline__ void draw8_lazy(FamilyDraw& f, int base, float vmax, bool seed, Vals&& vals) {
  float v[8];
  if (seed) {
    vals(v);
    f.draw8(base, v, vmax, true);
    return;
  }
  if (!f.reachable(vmax)) return;
  const uint32_t c0 = (uint32_t)base >> 2;
  const uint4 p0 = f.philox(c0), p1 = f.philox(c0 + 1);
  const uint32_t wmax = max(max(max(p0.x, p0.y), max(p0.z, p0.w)), max(max(p1.x, p1.y), max(p1.z, p1.w)));
  const bool maybe = fmaf(vmax, f.c2, f.off) >= __builtin_amdgcn_logf((float)((~wmax) >> 8));
  if (__ballot(maybe) == 0ull) return;
  vals(v);
  f.exact(base, v, c0,
          maybe ? FamilyDraw::cand4(p0, v, f.c2, f.off) | (FamilyDraw::cand4(p1, v + 4, f.c2, f.off) << 4) : 0u);
}

// A chunk's raw operands of one lane: 8 target logits and, with a map, the
// inverse map's entries and the draft logits gathered through them.
template <typename T, bool MAPPED>
struct ResSlice {
  Raw8<T> y, x;
  int32_t iv[8];
  T xg[8];
  __device__ __forceinline__ void load(const T* Y, const T* X, const int32_t* inv, int base) {
    y.load(Y + base);
    if (MAPPED)
      load8(inv + base, iv);
    else
      x.load(X + base);
  }
  // every lane loads, so the eight gathers issue together instead of one per
  // branch; they go through the draft row's buffer resource, which answers
  // an unmapped column's index (-1) with 0 without an access
  __device__ __forceinline__ void gather(__amdgpu_buffer_rsrc_t xrow) {
    if (MAPPED) {
#pragma unroll
      for (int k = 0; k < 8; ++k) buf_gather(xrow, (uint32_t)iv[k], xg[k]);
    }
  }
};

// A draw's maximum as one integer: larger keys first, equal keys by the
// smaller index (-0 and +0 are equal keys); 0 is below every finite key.
__device__ __forceinline__ unsigned long long pack_best(const Best& b) {
  const uint32_t u = __float_as_uint(b.key + 0.0f);
  const uint32_t ord = (u & 0x80000000u) != 0u ? ~u : u | 0x80000000u;
  return ((unsigned long long)ord << 32) | (0xFFFFFFFFu - (uint32_t)b.idx);
}

// SPLIT: gridDim.y workgroups per path
template <typename T, bool MAPPED, int W, bool SPLIT>
__global__ __launch_bounds__(W * kWave) void k_verify(VerifyArgs a) {
  __shared__ Best part[W];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int64_t path = blockIdx.x;
  if (path >= a.paths) return;
  int d = a.L;
  if (a.depth != nullptr) {
    d = a.depth[path];
    if (d < 1 || d > a.L) {
      if (threadIdx.x == 0 && blockIdx.y == 0) report_error(a.err, VSD_DEVERR_DEPTH_RANGE);
      d = 0;
    }
  }
  // every wavefront of the block takes the same acceptance decisions
  bool reject = false;
  if (lane < d) {  // L <= 64: one slot per lane
    const int64_t r = path * a.L + lane;
    const uint4 w = philox4x32_10(0u, (uint32_t)r, 2u, a.offset, a.k0, a.k1);
    reject = !(spec_log(uniform_from_word(w.x)) < a.la[r * 3]);
  }
  const uint64_t rej = __ballot(reject);
  const int j = rej != 0ull ? __builtin_ctzll(rej) : d;
  if (j >= d) {
    if (threadIdx.x == 0 && blockIdx.y == 0) {
      a.accept_len[path] = j;
      a.resample[path] = -1;
    }
    return;
  }
  // residual draw at the rejected slot
  const int64_t r = path * a.L + j;
  const T* X = static_cast<const T*>(a.X) + r * a.ld_d;
  const T* Y = static_cast<const T*>(a.Y) + r * a.ld_t;
  const float cq2 = a.inv_tq * kLog2e, cp2 = a.inv_tp * kLog2e;
  const float lq2 = a.lse_q[r] * kLog2e, lp2 = a.lse_p[r] * kLog2e;
  FamilyDraw f{(uint32_t)r, 3u, a.offset, a.k0, a.k1, 1.0f, kLog2e};
  const __amdgpu_buffer_rsrc_t xrow = row_rsrc(X, row_bytes(X, a.Vd));
  // max(0, p - q) of a slice's 8 target indices (p from the target logit, q
  // from the draft logit through the inverse map, 0 if unmapped)
  auto residual = [&](const ResSlice<T, MAPPED>& c, float (&res)[8]) {
    float y[8], x[8];
    c.y.unpack(y);
    if (MAPPED) {
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = load1(&c.xg[k]);
    } else {
      c.x.unpack(x);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool mapped = !MAPPED || (uint32_t)c.iv[k] < (uint32_t)a.Vd;
      const float p = __builtin_amdgcn_exp2f(fmaf(y[k], cp2, -lp2));
      const float q = mapped ? __builtin_amdgcn_exp2f(fmaf(x[k], cq2, -lq2)) : 0.0f;
      res[k] = fmaxf(p - q, 0.0f);
    }
  };
  // log(max(0, p - q)), -inf where p <= q
  auto log_res = [](float r) { return r > 0.0f ? __builtin_amdgcn_logf(r) * kLn2 : -INFINITY; };
  // the whole chunks are split into contiguous ranges, one per
  // wavefront, with every lane active (the draw's wavefront reductions,
  // including each range's seed, need all lanes); the last wavefront then
  // takes the partial chunk, in which every lane takes part with its valid
  // count
  const int nfull = a.Vt / kChunkV;
  const int parts = SPLIT ? W * (int)gridDim.y : W, part_no = SPLIT ? W * (int)blockIdx.y + wave : wave;
  const int c_begin = (int)((int64_t)nfull * part_no / parts);
  const int c_end = (int)((int64_t)nfull * (part_no + 1) / parts);
  if (c_begin < c_end) {
    ResSlice<T, MAPPED> cur;
    cur.load(Y, X, a.inv, c_begin * kChunkV + lane * 8);
    cur.gather(xrow);
    for (int it = c_begin; it < c_end; ++it) {
      const int base = it * kChunkV + lane * 8;
      const bool next = it + 1 < c_end;
      ResSlice<T, MAPPED> nxt;
      if (next) nxt.load(Y, X, a.inv, base + kChunkV);
      float res[8];
      residual(cur, res);
      draw8_lazy(f, base, log_res(max8(res)), it == c_begin, [&](float (&v)[8]) {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = log_res(res[k]);
      });
      if (next) {
        nxt.gather(xrow);
        cur = nxt;
      }
    }
  }
  if (part_no == parts - 1 && nfull * kChunkV < a.Vt) {
    const int base = nfull * kChunkV + lane * 8;
    const int nvalid = min(8, max(0, a.Vt - base));
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool in = k < nvalid;
      const float y = in ? load1(Y + base + k) : 0.0f;
      const int32_t iv = MAPPED ? (in ? a.inv[base + k] : -1) : (in ? base + k : -1);
      const bool mapped = (uint32_t)iv < (uint32_t)a.Vd;
      const float x = mapped ? load1(X + iv) : 0.0f;
      const float p = __builtin_amdgcn_exp2f(fmaf(y, cp2, -lp2));
      const float q = mapped ? __builtin_amdgcn_exp2f(fmaf(x, cq2, -lq2)) : 0.0f;
      v[k] = in ? log_res(fmaxf(p - q, 0.0f)) : -INFINITY;
    }
    f.draw(base, v, nvalid);
  }
  wave_argmax(f.best.key, f.best.idx);
  if (lane == 0) part[wave] = f.best;
  __syncthreads();
  if (threadIdx.x == 0) {
    // the wavefronts' ranges are in index order, so the strict comparison
    // keeps the smallest index among equal keys
    Best b = part[0];
#pragma unroll
    for (int w = 1; w < W; ++w)
      if (part[w].key > b.key) b = part[w];
    if (SPLIT) {
      if (b.key > -INFINITY)
        __hip_atomic_fetch_max(a.slot_best + path, pack_best(b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // released after this workgroup's maximum, acquired after every one's
      const uint32_t done =
          __hip_atomic_fetch_add(a.slot_done + path, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      if (done != gridDim.y - 1) return;
      const unsigned long long best =
          __hip_atomic_load(a.slot_best + path, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      a.accept_len[path] = j;
      a.resample[path] = best == 0ull ? -1 : (int32_t)(0xFFFFFFFFu - (uint32_t)best);
      return;
    }
    a.accept_len[path] = j;
    // no candidate at all: the residual mass vanished in float32 (alpha
    // rounds to 1 but the uniform exceeded it); reported as no replacement
    a.resample[path] = b.key == -INFINITY ? -1 : b.idx;
  }
}

template <typename T, int W>
void launch_w(const VerifyArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)a.paths);
  if (a.inv != nullptr)
    hipLaunchKernelGGL((k_verify<T, true, W, false>), grid, dim3(W * kWave), 0, s, a);
  else
    hipLaunchKernelGGL((k_verify<T, false, W, false>), grid, dim3(W * kWave), 0, s, a);
}

template <typename T>
hipError_t launch_t(const VerifyArgs& a, hipStream_t s) {
  // see above; every wavefront wants a chunk or two
  const int chunks = a.Vt / kChunkV;
  const int groups = (int)(kSplitGroups / a.paths < chunks / 8 ? kSplitGroups / a.paths : chunks / 8);
  if (a.slot_best != nullptr && groups > 1)
    hipLaunchKernelGGL((k_verify<T, true, 4, true>), dim3((unsigned)a.paths, (unsigned)groups), dim3(4 * kWave), 0, s,
                       a);
  else if (a.paths <= kPathsW16 && chunks >= 16)
    launch_w<T, 16>(a, s);
  else
    launch_w<T, 4>(a, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_verify(const VerifyArgs& a, bool bf16, hipStream_t s) {
  return bf16 ? launch_t<bf16_t>(a, s) : launch_t<float>(a, s);
}

}  // namespace vsd
