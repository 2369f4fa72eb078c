// Tiled candidate sweep of dense features: 16 source points per pass, moments on the vector ALU.
//
// As in the class-id sweep (sweep.hip), lane l of a wavefront works for source point s = l % 16 and candidate
// stream g = l / 16; the cell rows around the pass's box are walked 64 at a time into one candidate list, consumed
// in tiles of 64 candidates and sub-tiles of 16.  Feature rows never pass through LDS: the matrix-core operand of a
// sub-tile is read from the frame's rows straight into the registers that the instruction takes (rows are stored so
// that lane (s, g)'s elements of candidate s are contiguous), one sub-tile ahead of its use and across tiles.
// Staged through LDS, a tile of 64-dimensional FP32 rows took 16.6 KB and 64 registers, and two wavefronts per SIMD
// were in flight (now four): 8 x 30,000 points, 28 edges 2054 -> 1695 us per sweep.
//
// Spread passes.  A pass whose sources lie in a few places far apart (a jump of the Morton order, isolated points)
// walks the rows of a box that spans them all, alone for many times a compact pass's duration, at the end of the
// launch.  A first small kernel (k_split) finds such passes and lists them as items, one per quad of the pass's
// sources (one per source where a quad is spread itself); the sweep's first workgroups take items (kFrontItems), the
// others the remaining passes in their order.  An item walks only the row batches that its own sources are near, and
// only the tiles with a candidate that they reach.  What it leaves out adds exact zeros to its sources' moments, and
// what it keeps has the pass's own order, so the moments are the same bit for bit, whether a pass is split or not.
// Sweeps with staged rows and whole passes -> now: 8 x 30,000 points, 23 dimensions 995 -> 844 us; 6 x 17,001, 64
// dimensions 552 -> 402; 5 x 12,345 fp8 161 -> 102; 4 x 8,000, 20 dimensions 101 -> 70; 3 x 9,000 bfloat16 74 -> 48.
// Small launches are bound by the candidates of their longest pass, one after another (about 1.5 us per 64), large
// ones by the vector ALU, which FP32 matrix instructions occupy too (6 of 16x16x4 take 212 cycles per SIMD alone and
// 96 FMAs 408, together 610).
#include "sweep_device.h"

namespace rkhsba {
namespace {

// The operand of one sub-tile that a lane holds: the elements of one row that its column g of the matrix
// instructions takes.
template <int FEAT, int DP>
struct Operand {
  // FP32: elements 4k + g of the row, one 16x16x4 instruction per k.  bfloat16, fp8: elements 32k + 8g ..
  // 32k + 8g + 7, one 16x16x32 instruction per k.
  static constexpr int N = FEAT == FEAT_DENSE ? DP / 4 : DP / 32;
  static constexpr int ROWB = FEAT == FEAT_DENSE ? 4 * DP : FEAT == FEAT_BF16 ? 2 * DP : DP;
  typedef typename std::conditional<
      FEAT == FEAT_DENSE, float, typename std::conditional<FEAT == FEAT_BF16, bf16x8, long>::type>::type Elem;
  Elem e[N];
  __device__ void clear() {
#pragma unroll
    for (int k = 0; k < N; ++k) e[k] = Elem{};
  }
  __device__ void load(const uint8_t* __restrict__ row, int g) {
    if constexpr (FEAT == FEAT_DENSE) {  // stored column by column (feat_slot)
      const float* p = reinterpret_cast<const float*>(row) + g * N;
      if constexpr (N % 4 == 0) {
#pragma unroll
        for (int k = 0; k < N; k += 4) {
          const float4 v = *reinterpret_cast<const float4*>(p + k);
          e[k] = v.x; e[k + 1] = v.y; e[k + 2] = v.z; e[k + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int k = 0; k < N; k += 2) {
          const float2 v = *reinterpret_cast<const float2*>(p + k);
          e[k] = v.x; e[k + 1] = v.y;
        }
      }
    } else {
      constexpr int OB = FEAT == FEAT_BF16 ? 16 : 8;
#pragma unroll
      for (int k = 0; k < N; ++k) e[k] = *reinterpret_cast<const Elem*>(row + (4 * k + g) * OB);
    }
  }
};

// Inner products of the sub-tile's 16 candidates (a) with the pass's 16 sources (b): candidate 4g + r, source s.
template <int FEAT, int DP>
__device__ inline floatx4 products(const Operand<FEAT, DP>& a, const Operand<FEAT, DP>& b) {
  floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < Operand<FEAT, DP>::N; ++k) {
    if constexpr (FEAT == FEAT_DENSE) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a.e[k], b.e[k], c, 0, 0, 0);
    else if constexpr (FEAT == FEAT_BF16) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.e[k], b.e[k], c, 0, 0, 0);
    else c = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a.e[k], b.e[k], c, 0, 0, 0);
  }
  return c;
}

struct Shared {
  uint32_t row_j0[kLanes];
  uint32_t row_off[kLanes];
  uint32_t marker[kLanes];
  float4 tpos[kTile];  // position, and the candidate's index in the frame
};

// Finds the spread passes: 16 lanes per pass (four passes per wavefront).  a.split[pass] = 1 for a pass that went to
// the list, 0 for the others.
__global__ __launch_bounds__(256) void k_split(PairArgs a) {
  const int t = (int)(blockIdx.x * 256 + threadIdx.x);
  const int pass = t >> 4, s = t & 15, lane = threadIdx.x & 63;
  const bool live = pass < a.n_pass;  // (whole groups of 16 lanes; the wavefront stays together below)
  const PassInfo pi = a.passes[a.pass0 + (live ? pass : 0)];
  const FrameInfo Fn = a.frames[pi.tgt];
  const KConst kc = a.kcs[pi.prob];
  const bool in_range = live && s < pi.count;
  bool valid = in_range;
  float3 q = make_float3(0.f, 0.f, 0.f);
  if (valid) {
    const float4 x = a.pts[pi.src_off + a.vals[pi.entry0 + s]];
    q = rule_q32(a.xf[pi.e], x.x, x.y, x.z);
    valid = source_in_grid(q, Fn, kc);
  }
  const float3 l = make_float3(valid ? q.x : FLT_MAX, valid ? q.y : FLT_MAX, valid ? q.z : FLT_MAX);
  const float3 h = make_float3(valid ? q.x : -FLT_MAX, valid ? q.y : -FLT_MAX, valid ? q.z : -FLT_MAX);
  const float3 lo = make_float3(group_min<16>(l.x), group_min<16>(l.y), group_min<16>(l.z));
  const float3 hi = make_float3(group_max<16>(h.x), group_max<16>(h.y), group_max<16>(h.z));
  // extents (negative without a valid source)
  const float quad = fmaxf(quad_max(h.x) - quad_min(l.x), fmaxf(quad_max(h.y) - quad_min(l.y),
                                                                quad_max(h.z) - quad_min(l.z)));
  const float all = fmaxf(hi.x - lo.x, fmaxf(hi.y - lo.y, hi.z - lo.z));
  const float limit = a.split_factor * kc.r_c;
  bool spread = live && lo.x <= hi.x && all > limit;
  if (spread) spread = row_box(Fn, kc, lo, hi).n > kSplitRows;
  const bool wide = quad > limit;  // goes source by source
  const uint64_t emit = __builtin_amdgcn_ballot_w64(spread && in_range && (wide || (s & 3) == 0));
  const uint32_t n = (uint32_t)__popcll(emit);
  uint32_t at = 0;
  if (n > 0) {
    if (lane == 0) at = atomicAdd(a.n_items, n);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
  }
  const bool fits = at + n <= a.item_cap;  // otherwise the wavefront's slots stay empty, its passes whole
  if ((emit >> lane) & 1ull) {
    const uint32_t slot = at + (uint32_t)__popcll(emit & ((1ull << lane) - 1ull));
    if (slot < a.item_cap) a.items[slot] = make_uint2((uint32_t)pass, !fits ? 0u : wide ? 1u << s : 0xfu << s);
  }
  if (live && s == 0) a.split[pass] = spread && fits ? 1 : 0;
}

// Items come first, but no more of them than half of the wavefronts that the chip holds (256 CUs of 16): the first
// passes behind them then start while places are free, spread evenly over the SIMDs.  Behind an item list that fills
// the chip they started where the short items ended first, and a dense edge's long passes ended up on few SIMDs: 8 x
// 30,000 points, 64 dimensions, 6 cells per r_c (2,837 items, half of the pairs in the first 1,875 passes) FP32 3.17
// -> 2.55 ms, bfloat16 1.45 -> 1.24, fp8 1.12 -> 0.95; with at most 1,024 items first 3.14, 1.45 and 1.12; no items
// first loses 0.15 ms on fp8 at 4 and 8 cells.  Lists of up to kFrontItems are as they were.
constexpr uint32_t kFrontItems = 2048;

// CM: inner products as computed (0), negative ones clamped to 0 (1), or known to be positive (2: the pair count
// needs no c != 0 test).  SC: every source's own pair count is stored.
template <int MODE, int FEAT, int DP, int CM, bool SC>
__global__ __launch_bounds__(kLanes) void k_sweep_dense(PairArgs a) {
  __shared__ Shared sh;
  uint32_t pass = blockIdx.x, smask = 0xffffu;  // (uniform) the sources this wavefront works for
  bool item = false;
  if (a.items) {
    const uint32_t n = min(*a.n_items, a.item_cap);
    // kFrontItems items, as many passes, the other items, the other passes
    const uint32_t front = min(n, kFrontItems), fp = min((uint32_t)a.n_pass, kFrontItems);
    if (pass >= front && pass < n + fp) pass = pass < front + fp ? pass - front + n : pass - fp;
    if (pass < n) {
      const uint2 it = a.items[pass];
      pass = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.x);
      smask = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.y);
      if (smask == 0u) return;
      item = true;
    } else {
      pass -= n;
      if (pass >= (uint32_t)a.n_pass || a.split[pass]) return;
    }
  }
  typedef Operand<FEAT, DP> Op;
  const int lane = threadIdx.x;
  const PassInfo pi = a.passes[a.pass0 + pass];
  const EdgeXf X = a.xf[pi.e];
  const FrameInfo Fn = a.frames[pi.tgt];
  const KConst kc = a.kcs[pi.prob];
  const int s = lane & 15, g = lane >> 4;
  const int64_t entry = pi.entry0 + s;
  const bool in_range = s < pi.count;
  bool valid = in_range;
  const uint32_t src = in_range ? a.vals[entry] : 0u;
  float3 q = make_float3(0.f, 0.f, 0.f);
  const uint8_t* __restrict__ feat = static_cast<const uint8_t*>(a.feat);
  Op b;
  b.clear();
  if (valid) {
    const float4 x = a.pts[pi.src_off + src];
    q = rule_q32(X, x.x, x.y, x.z);
    valid = source_in_grid(q, Fn, kc);
    b.load(feat + (pi.src_off + src) * (int64_t)Op::ROWB, g);
  }
  const bool mine = in_range && ((smask >> s) & 1u);  // entries that this wavefront writes
  float3 lo, hi;
  lo.x = uniform_f(group_min<16>(valid ? q.x : FLT_MAX));
  lo.y = uniform_f(group_min<16>(valid ? q.y : FLT_MAX));
  lo.z = uniform_f(group_min<16>(valid ? q.z : FLT_MAX));
  hi.x = uniform_f(group_max<16>(valid ? q.x : -FLT_MAX));
  hi.y = uniform_f(group_max<16>(valid ? q.y : -FLT_MAX));
  hi.z = uniform_f(group_max<16>(valid ? q.z : -FLT_MAX));
  if (!(lo.x <= hi.x)) {  // no valid source point in this pass (uniform)
    if (g == 0 && mine) {
      a.cnt[entry] = 0u;
      store_zero_moments<MODE>(a, entry);
    }
    return;
  }
  const RowBox rbx = row_box(Fn, kc, lo, hi);
  // A lane without a valid source point (or with another item's) gets q at -1e18 (padding candidates sit at +1e18):
  // it fails every membership test at a finite distance.
  const bool active = valid && mine;
  if (!active) q = make_float3(-1.0e18f, -1.0e18f, -1.0e18f);
  float3 ilo = lo, ihi = hi;  // box of the wavefront's own sources
  if (item) {
    ilo.x = uniform_f(group_min<16>(active ? q.x : FLT_MAX)); ihi.x = uniform_f(group_max<16>(active ? q.x : -FLT_MAX));
    ilo.y = uniform_f(group_min<16>(active ? q.y : FLT_MAX)); ihi.y = uniform_f(group_max<16>(active ? q.y : -FLT_MAX));
    ilo.z = uniform_f(group_min<16>(active ? q.z : FLT_MAX)); ihi.z = uniform_f(group_max<16>(active ? q.z : -FLT_MAX));
  }

  const float rc2 = kc.rc2, alpha = kc.alpha;
  float A = 0.f, Bx = 0.f, By = 0.f, Bz = 0.f;
  float Cxx = 0.f, Cxy = 0.f, Cxz = 0.f, Cyy = 0.f, Cyz = 0.f, Wr2 = 0.f;
  uint32_t cnt = 0;  // pairs of the wavefront
  uint32_t own = 0;  // pairs of this lane (SC)
  const float4* __restrict__ tp = a.pts + Fn.pt_off;
  const uint8_t* __restrict__ trow = feat + Fn.pt_off * (int64_t)Op::ROWB;
  const int4* __restrict__ trows = a.rows + Fn.row_off;
  const float far_ = 1.0e18f;

  // The pairs of one sub-tile: this lane's four candidates with their inner products.
  auto pairs = [&](const float4 (&z4)[4], const floatx4& cur) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float4 z = z4[r];
      float dx, dy, dz;
      const float s2 = rule_s2(q, z.x, z.y, z.z, dx, dy, dz);
      const bool in = s2 <= rc2;
      const float c = CM == 1 ? fmaxf(cur[r], 0.f) : cur[r];
      const float k = __builtin_amdgcn_exp2f(-alpha * s2);
      const float w = in ? c * k : 0.f;
      if constexpr (SC) {
        own += (in && (CM == 2 || c != 0.f)) ? 1u : 0u;
      } else if constexpr (CM == 2) {
        cnt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(in));
      } else {
        cnt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(in) & __builtin_amdgcn_ballot_w64(c != 0.f));
      }
      A += w;
      if constexpr (MODE == MODE_NORMAL) {
        const float wx = w * dx, wy = w * dy;
        Bx += wx; By += wy; Bz = fmaf(w, dz, Bz);
        Cxx = fmaf(wx, dx, Cxx); Cxy = fmaf(wx, dy, Cxy); Cxz = fmaf(wx, dz, Cxz);
        Cyy = fmaf(wy, dy, Cyy); Cyz = fmaf(wy, dz, Cyz); Wr2 = fmaf(w, s2, Wr2);
      }
    }
  };

  // operands in flight, each replaced as it is consumed: two sub-tiles ahead, one for the longest rows
  constexpr int NB = Op::ROWB <= (FEAT == FEAT_DENSE ? 128 : 256) ? 2 : 1;
  Op oa[NB];
  uint64_t batches = 0;  // of the 64 batches of 64 rows that rb lies in: those with a row near a source
  for (int rb = 0; rb < rbx.n; rb += kLanes) {
    if (rbx.n > kManyRows) {  // uniform
      if ((rb & (64 * kLanes - 1)) == 0) batches = near_batches<16>(Fn, kc, rbx, q, active, rb, kLanes);
      const uint64_t ahead = batches >> ((rb / kLanes) & 63);
      if (!(ahead & 1ull)) {  // on to the next batch near a source, or to the next 64
        rb = ahead ? rb + kLanes * (__builtin_ctzll(ahead) - 1) : rb | (64 * kLanes - kLanes);
        continue;
      }
    }
    // ---- one row per lane: its contiguous candidate range
    uint32_t j0 = 0, cntr = 0;
    const int r = rb + lane;
    if (r < rbx.n) {
      int oz, oy;
      rbx.split(r, oz, oy);
      row_range(Fn, kc, trows, a.xtab, lo, hi, rbx.z0 + oz, rbx.y0 + oy, j0, cntr);
    }
    const uint32_t incl = wave_inclusive_scan(cntr);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    const uint32_t my_off = incl - cntr;
    if (total == 0) continue;
    wave_sync();  // earlier reads of row_j0 / row_off are done
    sh.row_j0[lane] = j0;
    sh.row_off[lane] = my_off;
    wave_sync();
    // ---- tiles of 64 candidates, the next one fetched while the current one is processed (the first step of the
    // loop fetches only).  The row of every candidate of a tile: rows mark the first position they cover, and a
    // candidate belongs to the last row marked at or before it.  Padding lanes read the frame's first point; the
    // consumer moves it far away.
    float4 npos = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t nj = 0;
    bool npad = true;
    auto load_row = [&](Op& o, uint32_t j, int sub) __attribute__((always_inline)) {
      // (__shfl forms the lane's byte address anew, 2 of a sub-tile's 65 vector instructions in the loss sweep: at
      // 5e9 pairs a sweep, 64 dimensions fp8 0.98 of the staged sweep's speed with it and 0.99 without, FP32 at 6
      // cells 0.99 and 1.00)
      o.load(trow + (int64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(4 * s + 64 * sub, (int)j) * Op::ROWB, g);
    };
    uint32_t left = 0;  // candidates from the fetched tile on (0: none fetched)
    for (uint32_t nb = 0; left > 0 || nb < total;) {
      // a tile without a candidate within reach of the item's sources adds nothing
      bool proc = left > 0;  // uniform
      if (proc && item) proc = __builtin_amdgcn_ballot_w64(!npad && box_s2(ilo, ihi, npos) <= rc2) != 0ull;
      const int n_sub = left >= (uint32_t)kTile ? 4 : (int)((left + 15) / 16);
      const uint32_t j = nj;
      floatx4 cv = {0.f, 0.f, 0.f, 0.f};
      if (proc) {
        sh.tpos[lane] = npad ? make_float4(far_, far_, far_, 0.f) : npos;
        cv = products<FEAT, DP>(oa[0], b);
        if (n_sub > NB) load_row(oa[0], j, NB);
      }
      const bool more = nb < total;
      left = 0;
      if (more) {
        sh.marker[lane] = 0u;
        wave_sync();
        if (cntr > 0 && my_off < nb + (uint32_t)kTile && my_off + cntr > nb)
          sh.marker[my_off > nb ? my_off - nb : 0u] = (uint32_t)lane + 1u;
        wave_sync();
        const uint32_t mr = wave_inclusive_max(sh.marker[lane]);
        const int rid = (int)min(max(mr, 1u), (uint32_t)kLanes) - 1;
        const uint32_t c = nb + (uint32_t)lane;
        const uint32_t jc = sh.row_j0[rid] + (c - sh.row_off[rid]);
        npad = c >= total || jc >= (uint32_t)Fn.n;  // the second test only bounds the reads
        nj = npad ? 0u : jc;
        npos = tp[nj];
        left = total - nb;
        nb += kTile;
      }
      wave_sync();  // tile positions written, markers read
      if (proc) {
        // unrolled: the products and the LDS offsets of each sub-tile get registers and immediates of their own
#pragma unroll
        for (int sub = 0; sub < 4; ++sub) {
          if (sub >= n_sub) break;  // uniform
          // this lane's four candidates, read before the products of the next sub-tile are waited for
          const float4* zp = sh.tpos + 16 * sub + 4 * g;
          float4 z4[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) z4[r] = zp[r];
          const floatx4 cur = cv;
          if (sub + 1 < n_sub) {  // the next sub-tile's products, and the operand that replaces theirs requested
            Op& o = oa[(sub + 1) % NB];
            cv = products<FEAT, DP>(o, b);
            if (sub + 1 + NB < 4) {
              if (sub + 1 + NB < n_sub) load_row(o, j, sub + 1 + NB);
            } else if (more) {  // (then this tile is a full one)
              load_row(o, nj, sub + 1 + NB - 4);
            }
          }
          pairs(z4, cur);
        }
      }
      if (more && !proc) {
#pragma unroll
        for (int k = 0; k < NB; ++k) load_row(oa[k], nj, k);
      }
      wave_sync();  // the tile buffer is rewritten next
    }
  }

  // the four candidate streams of each source point
  auto sum_streams = [&](auto xa) __attribute__((always_inline)) {
    A = xa(A);
    if constexpr (MODE == MODE_NORMAL) {
      Bx = xa(Bx); By = xa(By); Bz = xa(Bz);
      Cxx = xa(Cxx); Cxy = xa(Cxy); Cxz = xa(Cxz);
      Cyy = xa(Cyy); Cyz = xa(Cyz); Wr2 = xa(Wr2);
    }
  };
  sum_streams([](float v) { return xor_add<16>(v); });
  sum_streams([](float v) { return xor_add<32>(v); });
  if constexpr (SC) {
    own = xor_add<16>(own);
    own = xor_add<32>(own);
  }
  if (g == 0 && mine) {
    // every source's own count, or the wavefront's on its first entry; zero moments for a source outside the grid
    const int first = __builtin_ctz(smask);
    a.cnt[entry] = SC ? (valid ? own : 0u) : s == first ? cnt : 0u;
    const int64_t N = a.n_entries;
    auto v = [&](float m) { return valid ? m : 0.f; };
    a.mom[entry] = v(A);
    if constexpr (MODE == MODE_NORMAL) {
      a.mom[1 * N + entry] = v(Bx); a.mom[2 * N + entry] = v(By); a.mom[3 * N + entry] = v(Bz);
      a.mom[4 * N + entry] = v(Cxx); a.mom[5 * N + entry] = v(Cxy); a.mom[6 * N + entry] = v(Cxz);
      a.mom[7 * N + entry] = v(Cyy); a.mom[8 * N + entry] = v(Cyz); a.mom[9 * N + entry] = v(Wr2);
    }
  }
}

template <int MODE, int FEAT, int DP, int CM, bool SC>
hipError_t launch(const PairArgs& a, hipStream_t st) {
  k_sweep_dense<MODE, FEAT, DP, CM, SC>
      <<<(unsigned)a.n_pass + (a.items ? a.item_cap : 0u), kLanes, 0, st>>>(a);
  return hipGetLastError();
}

template <int MODE, int FEAT, int CM, bool SC>
hipError_t launch_dp(const PairArgs& a, hipStream_t st) {
  const int DP = a.kc.Dp;
  if constexpr (FEAT == FEAT_DENSE) {
    if (DP <= 8) return launch<MODE, FEAT, 8, CM, SC>(a, st);
    if (DP <= 16) return launch<MODE, FEAT, 16, CM, SC>(a, st);
    if (DP <= 24) return launch<MODE, FEAT, 24, CM, SC>(a, st);
  }
  if (DP <= 32) return launch<MODE, FEAT, 32, CM, SC>(a, st);
  return launch<MODE, FEAT, 64, CM, SC>(a, st);
}

// clamped, known-positive (FP32 features) or plain inner products
template <int MODE, int FEAT, bool SC>
hipError_t launch_cm(const PairArgs& a, hipStream_t st) {
  if (a.kc.clamp) return launch_dp<MODE, FEAT, 1, SC>(a, st);
  if constexpr (FEAT == FEAT_DENSE)
    if (a.kc.c_positive) return launch_dp<MODE, FEAT, 2, SC>(a, st);
  return launch_dp<MODE, FEAT, 0, SC>(a, st);
}

template <int FEAT>
hipError_t launch_mode(const PairArgs& a, int mode, bool source_counts, hipStream_t st) {
  if (source_counts) return launch_cm<MODE_NORMAL, FEAT, true>(a, st);
  return mode == MODE_LOSS ? launch_cm<MODE_LOSS, FEAT, false>(a, st) : launch_cm<MODE_NORMAL, FEAT, false>(a, st);
}

}  // namespace

hipError_t launch_sweep_dense(const PairArgs& a, int mode, int feat_path, bool source_counts, hipStream_t st) {
  if (a.n_pass == 0) return hipSuccess;
  if (a.items) k_split<<<(unsigned)(((int64_t)a.n_pass * 16 + 255) / 256), 256, 0, st>>>(a);
  switch (feat_path) {
    case FEAT_DENSE: return launch_mode<FEAT_DENSE>(a, mode, source_counts, st);
    case FEAT_BF16: return launch_mode<FEAT_BF16>(a, mode, source_counts, st);
    case FEAT_FP8: return launch_mode<FEAT_FP8>(a, mode, source_counts, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rkhsba
