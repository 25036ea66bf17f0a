// bcjr_lin_kernels.h -- forward-backward and VJP kernels in the linear domain
// for the trellises below 65536 states, dCodebook included.
//
// The recursions are those of fb_kernel_lin (sums of Boltzmann weights, one
// exponential per state and sweep, an exact power-of-two rescale per step),
// for every super-group shape (k = 1, 2, 3) up to S / K = 8192 groups.  All
// of it is bound by VALU issue, so what differs is there to issue less:
//  * dCodebook is accumulated inside the forward sweep: the states a lane
//    owns never change, so their sums stay in its registers, and the step's
//    normalisation is known before the step (Z from the backward sweep, the
//    exponents from the rescales).  fb_kernel's third sweep over stored
//    (G, A) rows moved 40 bytes of history per group-step, this 16.
//  * both tangents are centred on the weights: E[F] is then one number of the
//    block, known after the backward sweep, and no step needs the moments of
//    the one before it (but for dCodebook, see there).
//  * the moments of a step therefore only feed its outputs.  Each lane leaves
//    its partial sums of Q steps in LDS, and a wave sums them with its lanes
//    spread over steps: about 7 instructions per step instead of 6 lane
//    permutes for each of 4 moments; the divisions of the Q steps run side by
//    side as well.
//  * the distance to the codebook's range (0 inside it) is taken out of every
//    exponent of a step, so that a weight outside does not underflow the
//    whole vector; logZ gets the sum back.
//  * a block of at most 64 lanes lies inside one wave: its steps need no
//    workgroup barrier, only the wave's own LDS order, and waves run free of
//    each other.
//
// lin_group_kernel: one lane per group (S / K <= 64).  Backward lane v sums
//   the K successors of group v, forward lane v the K predecessors; the
//   history entry (H_t(v), H B_t(v)) is private to the lane.
// lin_sg_kernel: SGT super-groups per lane (S / K > 64), one block per
//   workgroup above 64 lanes, one or several per one-wave workgroup below.
//
// A block whose vectors leave the number range -- a step's largest entry
// below a floor, the forward mass sum_s alpha_t beta_t / Z away from 1, alpha H
// of a step so small that a better path may have been lost (kScaleMax), a weight
// far outside the codebook, moments that are not finite -- is marked in
// a.flags and recomputed by a second launch of the log-domain kernels.  The
// tangents' range does not depend on the gradient's: a power of two per block
// is taken out of g when its rows are read and put back at dW and dCodebook
// (see grad_exp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bcjr_device.h"
#include "bcjr_internal.h"

namespace bcjr {
namespace {
namespace lin {

// LDS order inside one wave: its LDS operations complete in issue order; the
// fence keeps the compiler from moving them across a step.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <bool MW>
__device__ __forceinline__ void block_sync() {
  if constexpr (MW) {
    __syncthreads();
  } else {
    wave_sync();
  }
}

// threads per workgroup of lin_sg_kernel
constexpr int sg_threads(int n, int KB, int SGT) {
  const int tpb = (1 << (n - 2 * KB)) / SGT;
  return tpb > 64 ? tpb : 64;
}

// waves per SIMD the register budget is cut for: 128 registers for 16 states per
// lane, 256 for 64; at n = 15 the LDS holds one workgroup of two waves per SIMD
// anyway.  With dCodebook's sums the budget does not hold all values everywhere:
// the compiler spills 32 and 35 registers at n = 14 and 9 of k = 2, 15 and 21 at
// n = 8 and 9 of k = 1, and 35 to 88 at k = 3; without dCodebook 0 to 11.
constexpr int min_waves(int KB, int SGT, bool VJP) {
  const int states = SGT << (2 * KB);
  return states <= 32 && SGT <= 4 ? (VJP ? 4 : 5) : VJP ? 2 : 3;
}

// Where several waves share vectors of over 1024 groups, the moments (1 KiB
// per wave and step) would cost a workgroup per CU: batches are of 2 steps
// instead of 4 there, and two lanes' moments are added before they are stored.
constexpr bool tight(int n, int KB, int SGT) {
  return (1 << (n - 2 * KB)) / SGT >= 256 && (1 << (n - KB)) > 1024;
}
constexpr int batch(int n, int KB, int SGT) { return tight(n, KB, SGT) ? 2 : 4; }

// LDS bytes of lin_sg_kernel: the ping-ponged vectors, the moments, for several
// waves their partial sums and maxima, for several blocks their powers of two
constexpr size_t sg_lds(int n, int KB, int SGT, bool VJP) {
  const size_t gs = (size_t)1 << (n - KB);
  const int tpb = (1 << (n - 2 * KB)) / SGT, waves = tpb > 64 ? tpb / 64 : 1, bpw = tpb > 64 ? 1 : 64 / tpb;
  return bpw * 2 * (VJP ? 2 : 1) * gs * 4 +
         (size_t)waves * batch(n, KB, SGT) * (tight(n, KB, SGT) ? 32 : 64) * (VJP ? 16 : 8) +
         (waves > 1 ? (size_t)waves * (2 * batch(n, KB, SGT) * 16 + 2 * 4) : 0) + (bpw > 1 ? 4 * bpw : 0);
}

// A rescale puts the largest entry at 2^90.  A step may lower it to 2^-36 (a
// weight that few states emit, after states far from them): 90 log2 units
// below it then still hold, and below that the block is marked.  H takes the
// exponents of both vectors and Z in one ldexp before it meets alpha.
constexpr int kTopExp = 90;
constexpr float kTop = 0x1p90f;
constexpr uint32_t kFloorBits = 0x2D800000u;  // 2^-36
constexpr uint32_t kCeilBits = 0x79800000u;   // 2^116
// With Z's mantissa in [1, 2), alpha H of a step's states sums to 2^-es in the
// stored units.  A path with an exponential below 2^-126 is lost, which may weigh
// up to 2^62 there (the vectors' entries reach 2^91 and, unscaled, 2^94), and
// both sweeps lose the same ones, so that the mass does not show it: against 64
// bits (256 steps, T = 0.0225 to 0.1) no block of 2000 is over 2e-5 off with all
// es below -70; from there up 4 % are, by up to the codebook's range.
constexpr int kScaleMax = -75;
// log2 units of a weight's distance outside the codebook (its exponents round
// at 6e-8 of them); beyond, the block is marked
constexpr float kFarMax = 4096.f;
constexpr float kMassTol = 1.4e-4f;     // departure of the forward mass from Z

// how far a weight lies above (below, negative) the range [lo, hi]
__device__ __forceinline__ float beyond(float w, float lo, float hi) { return w - fminf(fmaxf(w, lo), hi); }

// Holds a step's uniform values in vector registers: on gfx950 v_fma_f32,
// v_mul_f32 and v_add_f32 with vector operands only issue every 2.4 clocks per
// SIMD, with one scalar operand every 4.2 (2 and more waves per SIMD).
__device__ __forceinline__ void to_vgpr(float& a, float& b, float& c) {
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c));
}

// 1 / x to one rounding
__device__ __forceinline__ float inv(float x) {
  const float r = rcp(x);
  return fmaf(fmaf(-x, r, 1.f), r, r);
}

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}

// largest of the bit patterns of non-negative floats over W aligned lanes, in
// every lane (W = 64: a scalar).  A NaN's pattern is above every number's.
template <int W>
__device__ __forceinline__ uint32_t max_bits(uint32_t v) {
  if constexpr (W >= 2) v = umax(v, dpp_u<0xB1>(v));    // quad_perm [1,0,3,2]
  if constexpr (W >= 4) v = umax(v, dpp_u<0x4E>(v));    // quad_perm [2,3,0,1]
  if constexpr (W >= 8) v = umax(v, dpp_u<0x141>(v));   // row_half_mirror
  if constexpr (W >= 16) v = umax(v, dpp_u<0x140>(v));  // row_mirror
  if constexpr (W == 32) v = umax(v, (uint32_t)__shfl_xor((int)v, 16));
  if constexpr (W == 64) {
    v = umax(v, dpp_u<0x142, 0xA>(v));                  // row 0 -> 1, row 2 -> 3
    v = umax(v, dpp_u<0x143, 0xC>(v));                  // row 1 -> 2, 3
    v = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
  }
  return v;
}

// The exponent a rescale takes out after a step whose largest entry has these
// bits; 0 (and the block marked) where it is out of range.
__device__ __forceinline__ int rescale(uint32_t bits, bool& bad) {
  const bool in = bits >= kFloorBits && bits <= kCeilBits;
  bad = bad || !in;
  return in ? (int)(bits >> 23) - 127 - kTopExp : 0;
}

// The rows of a block, W = 64 or the lanes of its segment: lane l holds entry
// base + l of w' and g, and for a weight outside the codebook's range how far
// (m) and the whole log2 units (f) that the step's exponents leave out.  Such
// a step's tangent terms and moments are taken about the edge of the range,
// not the weight: d - m stays of the size of the codewords' own differences.
template <int W, bool VJP>
struct Rows {
  static constexpr int kChunk = W;
  const float* w;
  const float* g;
  int L;
  float kap, lo, hi;
  int li, seg0;          // lane in the segment, its first lane
  int gs;                // the power of two taken out of g: a scalar (W = 64), or
  int* gexp;             // each block's in LDS (a register less across the steps)
  float cw, cg, cf, cm, nw, ng;
  int base;

  __device__ __forceinline__ void load(int b, float& x, float& y) const {
    const int i = b + li;
    const bool in = i >= 0 && i < L;
    x = in ? w[i] : 0.f;
    if constexpr (VJP) y = in ? g[i] : 0.f;
  }
  // from the row's largest |g|, four loads in flight (every lane of a block
  // stores the same)
  __device__ __forceinline__ void scale() {
    float m = 0.f;
    for (int b = 0; b < L; b += 4 * W) {
      float y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] = g[b + q * W + li < L ? b + q * W + li : L - 1];
#pragma unroll
      for (int q = 0; q < 4; ++q) m = fmaxf(m, fabsf(y[q]));
    }
    const int e = grad_exp(seg_reduce<true>(m, W), L);
    if constexpr (W == 64) {
      gs = __builtin_amdgcn_readfirstlane(e);
    } else {
      gexp[lane_id() / W] = e;
      wave_sync();
    }
  }
  __device__ __forceinline__ int ge() const {
    if constexpr (W == 64) return gs;
    return gexp[lane_id() / W];  // (the lane index rebuilt: no register holds it)
  }
  // takes the prefetched chunk as [b, b + W) and fetches the one at `next`
  __device__ __forceinline__ void take(int b, int next, bool& bad) {
    base = b;
    cw = nw * kap;
    if constexpr (VJP) cg = ldexpf(ng, -ge());
    cm = b + li < L ? beyond(cw, lo, hi) : 0.f;
    cf = floorf(cm * cm);  // (whole, so that both sweeps take out the same)
    if (!(cf <= kFarMax)) bad = true;
    load(next, nw, ng);
  }
  __device__ __forceinline__ float at(float v, int t) const {
    if constexpr (W == 64) return read_lane(v, t - base);
    return __shfl(v, seg0 + t - base);
  }
  __device__ __forceinline__ int at_i(int v, int t) const {
    if constexpr (W == 64) return __builtin_amdgcn_readlane(v, t - base);
    return __shfl(v, seg0 + t - base);
  }
  // sets this chunk's entry of step t in the lane that holds it
  __device__ __forceinline__ void put_i(int& v, int x, int t) const {
    v = li == t - base ? x : v;
  }
};

// Sums over a wave of Q steps' moments m[q][E entries]: the segments of W
// lanes (E W / 64 entries) yield Q x 64 / W sums, one per LPO = W / Q lanes; a
// lane of segment s sums for segment s.  NM = 4 (VJP) or 2 values per entry.
template <int W, int Q, int NM, int E = 64>
__device__ __forceinline__ void sum_batch(const float* m, int lane, float (&r)[NM]) {
  constexpr int LPO = W / Q, PER = E * W / 64;
  static_assert(PER >= LPO, "an entry per lane");
  const int o = lane / LPO, p = lane % LPO;
  const float* src = m + ((o % Q) * E + (o / Q) * PER + p) * NM;
#pragma unroll
  for (int i = 0; i < PER / LPO; ++i) {
    float x[NM];
    ld_vec<NM>(src + i * LPO * NM, x);
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] = i ? r[c] + x[c] : x[c];
  }
  if constexpr (LPO > 1) {
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] += dpp<0xB1>(r[c]);
  }
  if constexpr (LPO > 2) {
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] += dpp<0x4E>(r[c]);
  }
  if constexpr (LPO > 4) {
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] += dpp<0x141>(r[c]);
  }
  if constexpr (LPO > 8) {
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] += dpp<0x140>(r[c]);
  }
  if constexpr (LPO > 16) {
#pragma unroll
    for (int c = 0; c < NM; ++c) r[c] += __shfl_xor(r[c], 16);
  }
}

// w_soft_t and dW_t from a step's moments sum P d, sum P, sum P (X - E X),
// sum P (X - E X) d (P normalised by Z: sum P is the forward mass); wt = w'_t, or the
// edge of the range that the moments are about; ge: the power of two to put back
template <bool VJP>
__device__ __forceinline__ void step_outputs(const LinArgs& a, int64_t at, float wt, int ge, const float* r,
                                             bool& bad) {
  const float mass = r[1];
  if (!(fabsf(mass - 1.f) <= kMassTol)) bad = true;
  const float r1 = inv(mass), md = r[0] * r1;
  if (a.w_soft) a.w_soft[at] = (wt - md) * a.inv_kap;
  if constexpr (VJP) {
    if (!(fabsf(r[2]) + fabsf(r[3]) < INFINITY)) bad = true;
    if (a.dW) a.dW[at] = ldexpf(fmaf(r[2] * r1, r[0], -r[3]) * r1 * a.dws, ge);
  }
}

// e with x = m 2^e, 1 <= m < 2, for a positive normal x
__device__ __forceinline__ int exp_bits(float x) { return (int)((as_u(x) >> 23) & 0xFFu) - 127; }

__device__ __forceinline__ double pow2_d(int e) { return __longlong_as_double((long long)(e + 1023) << 52); }

__device__ __forceinline__ double seg_sum_d(double v, int width) {
  for (int o = 1; o < width; o <<= 1) v += __shfl_xor(v, o);
  return v;
}

}  // namespace lin
}  // namespace

// ---------------------------------------------------------------------------
// One lane per group.  GS = S / K lanes per block, 64 / GS blocks per wave;
// one wave per workgroup, free of the others.  Against the log-domain kernel
// with its third sweep: 64 blocks of 16 steps at S = 16 with dCodebook 106 ->
// 24 us for the call (15 us in here, the latency of 32 dependent steps; the
// rest launches); S = 256, 4096 blocks of 256, w_soft + logZ + dW 687 -> 378 us.
// ---------------------------------------------------------------------------
template <int KB, int n, bool VJP, bool DC>
__global__ void __launch_bounds__(64, KB == 3 ? 3 : 4) lin_group_kernel(LinArgs a) {
  constexpr int K = 1 << KB;
  constexpr int GS = 1 << (n - KB), NSG = GS >> KB;
  constexpr int Q = 4;                       // steps per batch, and history entries in flight
  constexpr bool BATCH = GS >= Q;            // (two-lane blocks sum their moments directly)
  constexpr int NM = VJP ? 4 : 2;
  __shared__ float2 xw[64];                  // (value, tangent) of each lane's group
  __shared__ __align__(16) float mom[BATCH ? Q * 64 * NM : 4];
  __shared__ int gexp[64 / GS];              // (see Rows)
  const int lane = threadIdx.x;
  const int v = lane & (GS - 1);             // the lane's group
  const int seg0 = lane & ~(GS - 1);
  constexpr int bpw = 64 >> (n - KB);        // blocks per wave
  const int64_t nslots = (int64_t)gridDim.x * bpw;
  const int64_t slot = (int64_t)blockIdx.x * bpw + (lane >> (n - KB));
  const int L = (int)a.L;                    // (L x S / K x 12 bytes is below 2^31)
  const float kap = a.kap;
  // d' = kappa (w - c) as fma(-kappa, c, kappa w): one rounding, relative to d'
  float nkap = -kap;
  pin(nkap);
  float dws = a.dws;
  if constexpr (DC) pin(dws);                // (a vector register, see to_vgpr)
  const int rowi = seg0 + ((v << KB) & (GS - 1));   // H(v K + b): K consecutive groups
  const int coli = seg0 + (v >> KB);                // G(j NSG + (v >> KB))

  // the K states of each sweep: v K + b (backward), j GS + v (forward)
  float cb[K], cf[K], acc[DC ? K : 1];
  float clo = INFINITY, chi = -INFINITY;
#pragma unroll
  for (int b = 0; b < K; ++b) {
    cb[b] = a.c[v * K + b];
    cf[b] = a.c[b * GS + v];
    const float cs = cf[b] * kap;
    clo = fminf(clo, cs);
    chi = fmaxf(chi, cs);
    if (slot == 0) a.cs[b * GS + v] = cs;
  }
  clo = -seg_reduce<true>(-clo, GS);
  chi = seg_reduce<true>(chi, GS);
  double* const part = DC ? a.dc_part + slot * ((int64_t)K * GS) : nullptr;
  if constexpr (DC) {
#pragma unroll
    for (int j = 0; j < K; ++j) part[j * GS + v] = 0.0;
  }
  // (H, H B) of step t at hist + t * GS + v
  float2* const hist2 = reinterpret_cast<float2*>(a.hist) + slot * L * GS + v;
  float* const hist1 = a.hist + slot * L * GS + v;
  int32_t* const exps = a.exps + slot * L;

  for (int64_t base = (int64_t)blockIdx.x * bpw; base < a.B; base += nslots) {
    const int64_t blk = base + (lane >> (n - KB));
    const bool valid = blk < a.B;
    const int64_t bb = valid ? blk : a.B - 1;
    lin::Rows<GS, VJP> rw;
    rw.w = a.w + bb * L;
    rw.g = VJP ? a.g + bb * L : nullptr;
    rw.L = L;
    rw.kap = kap;
    rw.lo = clo;
    rw.hi = chi;
    rw.li = v;
    rw.gexp = gexp;
    rw.seg0 = seg0;
    bool bad = false;

    // ------------------------------------------------------------ backward
    xw[lane] = make_float2(lin::kTop, 0.f);
    if constexpr (VJP) {
      hist2[(L - 1) * GS] = make_float2(lin::kTop, 0.f);
    } else {
      hist1[(L - 1) * GS] = lin::kTop;
    }
    lin::wave_sync();
    int ex = lin::kTopExp, off = 0, ev = ex;
    double far = 0.0;                        // what the exponents leave out
    {
      const int top = (L - 1) / GS * GS;
      if constexpr (VJP) rw.scale();
      rw.load(top, rw.nw, rw.ng);
      rw.take(top, top - GS, bad);
      far += (double)rw.cf;
    }
    for (int t = L - 1; t >= 1; --t) {
      if (t < rw.base) {
        if (rw.base + v < L) exps[rw.base + v] = ev;
        rw.take(rw.base - GS, rw.base - 2 * GS, bad);
        far += (double)rw.cf;
      }
      rw.put_i(ev, ex, t);
      float wt = rw.at(rw.cw, t);
      float gt = VJP ? rw.at(rw.cg, t) : 0.f;
      float mf = rw.at(rw.cm, t);
      lin::to_vgpr(wt, gt, mf);
      const float noff = rw.at(rw.cf, t) - (float)off;
      float2 in[K];
#pragma unroll
      for (int b = 0; b < K; ++b) in[b] = xw[rowi + b];
      float hv = 0.f, bv = 0.f;
#pragma unroll
      for (int b = 0; b < K; ++b) {
        const float d = fmaf(nkap, cb[b], wt);
        const float e = ex2(fmaf(-d, d, noff));
        hv = fmaf(e, in[b].x, hv);
        if constexpr (VJP) bv = fmaf(e, fmaf(-gt * in[b].x, d - mf, in[b].y), bv);
      }
      lin::wave_sync();
      xw[lane] = make_float2(hv, bv);
      if constexpr (VJP) {
        hist2[(t - 1) * GS] = make_float2(hv, bv);
      } else {
        hist1[(t - 1) * GS] = hv;
      }
      ex -= off;
      off = lin::rescale(lin::max_bits<GS>(as_u(hv)), bad);
      lin::wave_sync();
    }
    // (L > 1 leaves the last chunk's entries 1 .. in place; step 0 follows)
    if (0 < rw.base) {
      if (rw.base + v < L) exps[rw.base + v] = ev;
      rw.take(rw.base - GS, rw.base - 2 * GS, bad);
      far += (double)rw.cf;
    }
    rw.put_i(ev, ex, 0);
    if (v < L) exps[v] = ev;
    // Z = sum_s alpha_0(s) beta_0(s) = sum_v sum_j e(j GS + v) H_0(v), E_p[F]
    float xbar = 0.f, rz;
    int exz;
    {
      const float wt = rw.at(rw.cw, 0), gt = VJP ? rw.at(rw.cg, 0) : 0.f, mf = rw.at(rw.cm, 0);
      const float noff = rw.at(rw.cf, 0) - (float)off;
      const float2 in = xw[lane];
      float ls = 0.f, ly = 0.f;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const float d = fmaf(nkap, cf[j], wt);
        const float e = ex2(fmaf(-d, d, noff));
        ls = fmaf(e, in.x, ls);
        if constexpr (VJP) ly = fmaf(e, fmaf(-gt * in.x, d - mf, in.y), ly);
      }
      ls = seg_reduce<false>(ls, GS);
      if constexpr (VJP) ly = seg_reduce<false>(ly, GS);
      if (!(ls > 0.f && ls < INFINITY)) bad = true;
      const int ez = lin::exp_bits(ls);
      ls = ldexpf(ls, -ez);
      rz = lin::inv(ls);
      exz = ex - off - ez;
      xbar = ldexpf(ly, -ez) * rz;
      far = lin::seg_sum_d(far, GS);
      if (v == 0 && valid && a.logZ)
        a.logZ[bb] = (float)(((double)lg2(ls) - (double)exz - far) * 0.69314718055994530942);
    }

    // ------------------------------------------------------------- forward
    lin::wave_sync();
    xw[lane] = make_float2(lin::kTop, 0.f);
    lin::wave_sync();
    if constexpr (DC) {
#pragma unroll
      for (int j = 0; j < K; ++j) acc[j] = 0.f;
    }
    ex = lin::kTopExp;
    off = 0;
    rw.load(0, rw.nw, rw.ng);
    rw.take(0, GS, bad);
    int ec = exps[v < L ? v : L - 1];
    int en = exps[GS + v < L ? GS + v : L - 1];
    float2 ph[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int tq = q < L ? q : L - 1;
      ph[q] = VJP ? hist2[tq * GS] : make_float2(hist1[tq * GS], 0.f);
    }
    for (int t0 = 0; t0 < L; t0 += Q) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int t = t0 + q;
        if (t < L) {
          if (t >= rw.base + GS) {
            const int nb = rw.base + 2 * GS;
            rw.take(rw.base + GS, nb, bad);
            ec = en;
            en = exps[nb + v < L ? nb + v : L - 1];
          }
          float wt = rw.at(rw.cw, t);
          float gt = VJP ? rw.at(rw.cg, t) : 0.f;
          float mf = rw.at(rw.cm, t);
          lin::to_vgpr(wt, gt, mf);
          const float noff = rw.at(rw.cf, t) - (float)off;
          // alpha_t beta_t / Z = alpha H sc, exponents of both vectors and Z;
          // (ex - off: of alpha_t; the stored H_t carries no rescale of its own)
          const int es = exz - (ex - off) - rw.at_i(ec, t);
          if (es > lin::kScaleMax) bad = true;
          const float H = ph[q].x, HB = ph[q].y;
          {
            const int tn = t + Q < L ? t + Q : L - 1;
            ph[q] = VJP ? hist2[tn * GS] : make_float2(hist1[tn * GS], 0.f);
          }
          float al[K], qq[K], dd[K], dw[K];  // d about the edge of the range, and about the weight
#pragma unroll
          for (int j = 0; j < K; ++j) {
            const float2 in = xw[coli + j * NSG];
            dw[j] = fmaf(nkap, cf[j], wt);
            dd[j] = dw[j] - mf;
            const float e = ex2(fmaf(-dw[j], dw[j], noff));
            al[j] = e * in.x;
            if constexpr (VJP) qq[j] = e * fmaf(-gt * in.x, dd[j], in.y);
          }
          float go = al[0], sad = al[0] * dd[0], ao = 0.f, sqd = 0.f;
          if constexpr (VJP) {
            ao = qq[0];
            sqd = qq[0] * dd[0];
          }
#pragma unroll
          for (int j = 1; j < K; ++j) {
            go += al[j];
            sad = fmaf(al[j], dd[j], sad);
            if constexpr (VJP) {
              ao += qq[j];
              sqd = fmaf(qq[j], dd[j], sqd);
            }
          }
          lin::wave_sync();
          xw[lane] = make_float2(go, ao);
          const float Hs = ldexpf(H, es) * rz;
          float m[NM];
          m[0] = Hs * sad;
          m[1] = Hs * go;
          if constexpr (VJP) {
            const float bx = fmaf(-xbar, Hs, ldexpf(HB, es) * rz);
            m[VJP ? 2 : 0] = fmaf(go, bx, Hs * ao);
            m[VJP ? 3 : 0] = fmaf(sad, bx, Hs * sqd);
            if constexpr (DC) {
              // p (g + d (X - E X) / (kappa^2 T)) of the lane's K states
              const float aq = Hs * gt, bq = bx * dws, cq = Hs * dws;
#pragma unroll
              for (int j = 0; j < K; ++j) {
                acc[j] = fmaf(dw[j], fmaf(al[j], bq, qq[j] * cq), fmaf(al[j], aq, acc[j]));
                pin(acc[j]);  // (or it sinks out of the step, its inputs live across)
              }
            }
          }
          // E[F] anew from the step's own sum: with one value for the whole block its
          // rounding adds up coherently over the steps of dCodebook (2 to 4 times the error)
          if constexpr (DC) xbar += seg_reduce<false>(m[VJP ? 2 : 0], GS);
          ex -= off;
          {
            bool out = false;
            off = lin::rescale(lin::max_bits<GS>(as_u(go)), out);
            if (out && t + 1 < L) bad = true;
          }
          if constexpr (BATCH) {
            st_vec<NM>(mom + (q * 64 + lane) * NM, m);
          } else {
#pragma unroll
            for (int c = 0; c < NM; ++c) m[c] = seg_reduce<false>(m[c], GS);
            if (v == 0 && valid) lin::step_outputs<VJP>(a, bb * L + t, wt - mf, rw.ge(), m, bad);
          }
          lin::wave_sync();
        }
      }
      if constexpr (BATCH) {
        // lane (segment, step, part): every lane of a step's LPO holds its sums
        const int ln = lane_id(), lv = ln & (GS - 1);
        float r[NM];
        lin::sum_batch<GS, Q, NM>(mom, ln, r);
        const int t = t0 + (lv / (GS / Q));
        const float wt = __shfl(rw.cw - rw.cm, (ln & ~(GS - 1)) + t - rw.base);
        if (t < L && valid && lv % (GS / Q) == 0)
          lin::step_outputs<VJP>(a, bb * L + t, wt, rw.ge(), r, bad);
        lin::wave_sync();
      }
    }
    {  // the block is marked when any of its lanes is
      const uint64_t any = __ballot(bad) >> seg0;
      bad = (GS == 64 ? any : any & ((1ull << GS) - 1)) != 0;
    }
    if (v == 0 && valid) a.flags[bb] = bad ? 1 : 0;
    if constexpr (DC) {
      if (valid && !bad) {
        const double pow2 = lin::pow2_d(rw.ge());
#pragma unroll
        for (int j = 0; j < K; ++j) part[j * GS + v] = fma((double)acc[j], pow2, part[j * GS + v]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// SGT super-groups per lane.  MW: one block per workgroup of TPB = NSG / SGT
// > 64 lanes, one barrier per step; otherwise TPB <= 64 lanes per block and
// independent waves.  The vectors are ping-ponged between two LDS copies,
// values and tangents in planes of their own: a row access (K consecutive
// groups) is then 16 bytes at a 16-byte lane stride, a column access one
// dword per lane, both without bank conflicts.  Bound by VALU issue.  Against
// the log-domain kernel: S = 4096, 16384 blocks with dCodebook 41.1 -> 20.0 ms;
// S = 16384, 1800 blocks of 200, Viterbi + VJP 15.3 -> 10.0 ms.  Reducing all
// moments in every step took 24.4 ms at S = 4096.
// ---------------------------------------------------------------------------
template <int KB, int n, int SGT, bool VJP, bool DC>
__global__ void __launch_bounds__(lin::sg_threads(n, KB, SGT), lin::min_waves(KB, SGT, VJP))
    lin_sg_kernel(LinArgs a) {
  constexpr int K = 1 << KB;
  extern __shared__ float lds[];
  constexpr int GS = 1 << (n - KB), NSG = GS >> KB;
  constexpr int TPB = NSG / SGT;
  constexpr bool MW = TPB > 64;
  constexpr int W = MW ? 64 : TPB;           // lanes of a block inside a wave
  constexpr int NW = MW ? TPB / 64 : 1;      // waves of a block
  constexpr int Q = lin::batch(n, KB, SGT), NM = VJP ? 4 : 2;
  constexpr bool HALF = lin::tight(n, KB, SGT);
  constexpr int E = HALF ? 32 : 64;          // stored moments per step and wave
  static_assert(W >= Q, "a batch needs a lane per step");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tb = MW ? (int)threadIdx.x : lane & (TPB - 1);
  const int seg0 = MW ? 0 : lane & ~(TPB - 1);
  constexpr int bpw = MW ? 1 : 64 / TPB;     // blocks per workgroup
  const int64_t unit = blockIdx.x;
  const int64_t nslots = (int64_t)gridDim.x * bpw;
  const int sub = MW ? 0 : lane / TPB;       // block inside the wave
  const int64_t slot = unit * bpw + sub;
  const int L = (int)a.L;                    // (L x S / K x 12 bytes is below 2^31)
  const float kap = a.kap;
  // d' = kappa (w - c) as fma(-kappa, c, kappa w): one rounding, relative to d'
  float nkap = -kap;
  pin(nkap);
  float dws = a.dws;
  if constexpr (DC) pin(dws);                // (a vector register, see to_vgpr)

  // LDS: per block [2 copies][value, tangent][GS], each wave's moments of a
  // batch, the waves' sums of a batch and their maxima of a step (each with
  // two parities: one barrier per step); several blocks' powers of two
  constexpr int PL = VJP ? 2 : 1;            // planes
  float* const vb = lds + sub * 2 * PL * GS;
  float* const mom = lds + bpw * 2 * PL * GS + wave * Q * E * NM;
  float* const wsum = lds + bpw * 2 * PL * GS + NW * Q * E * NM;
  uint32_t* const wmax = reinterpret_cast<uint32_t*>(wsum + 2 * NW * Q * NM);
  int* const gexp = reinterpret_cast<int*>(wsum);  // (one wave: no sums of waves)
  // largest entry over the block, from each wave's; call around the barrier
  auto max_pre = [&](float m, int par) -> uint32_t {
    const uint32_t b = lin::max_bits<W>(as_u(m));
    if constexpr (MW) {
      if (lane == 0) wmax[par * NW + wave] = b;
    }
    return b;
  };
  auto max_post = [&](uint32_t b, int par) -> uint32_t {
    if constexpr (MW) {
      uint32_t x = wmax[par * NW];
#pragma unroll
      for (int i = 1; i < NW; ++i) x = lin::umax(x, wmax[par * NW + i]);
      return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
    }
    return b;
  };
  RedCtx rc;                                 // once-per-block sums
  rc.width = W;
  rc.rw = NW;
  rc.wave = wave;
  rc.red = mom - wave * Q * E * NM;         // (over the moments, between the sweeps)

  const rsrc_t cbk = make_rsrc(a.c, (uint32_t)4 << n);
  const uint32_t voK = (uint32_t)tb << (KB + 2);
  float cc[SGT][K][K], acc[DC ? SGT : 1][K][K];
  float clo = INFINITY, chi = -INFINITY;
#pragma unroll
  for (int i = 0; i < SGT; ++i) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const uint32_t so = ((j << (n - KB)) + ((i * TPB) << KB)) * 4;
      buf_ld<K>(cbk, voK, so, cc[i][j]);
      float cs[K];
#pragma unroll
      for (int u = 0; u < K; ++u) {
        cs[u] = cc[i][j][u] * kap;
        clo = fminf(clo, cs[u]);
        chi = fmaxf(chi, cs[u]);
      }
      if (slot == 0) st_vec<K>(a.cs + (voK + so) / 4, cs);
    }
  }
  {  // the codebook's range over the block
    float mm[2] = {-clo, chi};
    red_pre<2, 3u>(mm, rc);
    lin::block_sync<MW>();
    red_post<2, 3u>(mm, rc);
    clo = -mm[0];
    chi = mm[1];
    lin::block_sync<MW>();
  }
  // the slot's dCodebook partial, state (j, i, tb, u) at row (j, i) + tb K + u;
  // the lane's offset is rebuilt at each use, so that no address stays live
  double* const part = DC ? a.dc_part + (unit * bpw << n) : nullptr;
  auto part_at = [&](int i, int j) {
    uint32_t o = (uint32_t)((sub << n) + (tb << KB));
    pin_u(o);
    return part + (o + (uint32_t)((j << (n - KB)) + ((i * TPB) << KB)));
  };
  if constexpr (DC) {
#pragma unroll
    for (int i = 0; i < SGT; ++i)
#pragma unroll
      for (int j = 0; j < K; ++j) {
        double* const pj = part_at(i, j);
#pragma unroll
        for (int u = 0; u < K; ++u) pj[u] = 0.0;
      }
  }
  constexpr uint32_t hstep = (uint32_t)GS * PL;  // floats per history step: H, then H B
  const int64_t slot0 = unit * bpw;
  const rsrc_t hist = make_rsrc(a.hist + slot0 * L * hstep, (uint32_t)bpw * (uint32_t)L * hstep * 4u);
  const uint32_t voS = (uint32_t)sub * (uint32_t)L * hstep * 4u;
  const uint32_t voR = voS + (uint32_t)tb * K * 4u;      // row form
  const uint32_t voC = voS + (uint32_t)tb * 4u;          // column form
  int32_t* const exps = a.exps + slot * L;

  for (int64_t base = unit * bpw; base < a.B; base += nslots) {
    const int64_t blk = base + sub;
    const bool valid = blk < a.B;
    const int64_t bb = valid ? blk : a.B - 1;
    lin::Rows<W, VJP> rw;
    rw.w = a.w + bb * L;
    rw.g = VJP ? a.g + bb * L : nullptr;
    rw.L = L;
    rw.kap = kap;
    rw.lo = clo;
    rw.hi = chi;
    rw.li = lane & (W - 1);
    rw.gexp = gexp;
    rw.seg0 = seg0;
    bool bad = false;
    const bool first_wave = !MW || wave == 0;

    // ------------------------------------------------------------ backward
#pragma unroll 1
    for (int i = tb; i < GS; i += TPB) {
      vb[i] = lin::kTop;
      if constexpr (VJP) vb[GS + i] = 0.f;
      const float one[1] = {lin::kTop}, zero[1] = {0.f};
      const uint32_t so = (uint32_t)(L - 1) * hstep * 4u;
      buf_st<1, kStream>(hist, voS + (uint32_t)i * 4u, so, one);
      if constexpr (VJP) buf_st<1, kStream>(hist, voS + (uint32_t)i * 4u, so + (uint32_t)GS * 4u, zero);
    }
    lin::block_sync<MW>();
    int ex = lin::kTopExp, off = 0, ev = ex;
    double far = 0.0;
    int par = 0;                             // the copy being read
    {
      const int top = (L - 1) / W * W;
      if constexpr (VJP) rw.scale();
      rw.load(top, rw.nw, rw.ng);
      rw.take(top, top - W, bad);
      far += (double)rw.cf;
    }
    for (int t = L - 1; t >= 1; --t) {
      if (t < rw.base) {
        if (first_wave && rw.base + rw.li < L) exps[rw.base + rw.li] = ev;
        rw.take(rw.base - W, rw.base - 2 * W, bad);
        far += (double)rw.cf;
      }
      rw.put_i(ev, ex, t);
      float wt = rw.at(rw.cw, t);
      float gt = VJP ? rw.at(rw.cg, t) : 0.f;
      float mf = rw.at(rw.cm, t);
      lin::to_vgpr(wt, gt, mf);
      const float noff = rw.at(rw.cf, t) - (float)off;
      const float* const rd = vb + par * PL * GS;
      float* const wr = vb + (par ^ 1) * PL * GS;
      const uint32_t so = (uint32_t)(t - 1) * hstep * 4u;
      float vmax = 0.f;
#pragma unroll
      for (int i = 0; i < SGT; ++i) {
        float wtl = wt;
        pin(wtl);  // one super-group at a time: no value of another is worked out ahead
        float Hin[K], Bin[K], gH[K];
        ld_vec<K>(rd + (tb + i * TPB) * K, Hin);
        if constexpr (VJP) ld_vec<K>(rd + GS + (tb + i * TPB) * K, Bin);
#pragma unroll
        for (int b = 0; b < K; ++b) gH[b] = VJP ? gt * Hin[b] : 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) {
          float e[K], d[K];
#pragma unroll
          for (int b = 0; b < K; ++b) {
            d[b] = fmaf(nkap, cc[i][j][b], wtl);
            e[b] = ex2(fmaf(-d[b], d[b], noff));
            if constexpr (VJP) d[b] -= mf;
          }
          float hv[1] = {e[0] * Hin[0]};
#pragma unroll
          for (int b = 1; b < K; ++b) hv[0] = fmaf(e[b], Hin[b], hv[0]);
          vmax = as_f(lin::umax(as_u(vmax), as_u(hv[0])));
          const int ci = j * NSG + i * TPB;
          wr[ci + tb] = hv[0];
          buf_st<1, kStream>(hist, voC, so + (uint32_t)ci * 4u, hv);
          if constexpr (VJP) {
            float bv[1] = {e[0] * fmaf(-gH[0], d[0], Bin[0])};
#pragma unroll
            for (int b = 1; b < K; ++b) bv[0] = fmaf(e[b], fmaf(-gH[b], d[b], Bin[b]), bv[0]);
            wr[GS + ci + tb] = bv[0];
            buf_st<1, kStream>(hist, voC, so + (uint32_t)(ci + GS) * 4u, bv);
          }
          if constexpr (KB == 3 || SGT > 1) __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" ::: "memory");
      }
      const uint32_t mb = max_pre(vmax, par);
      lin::block_sync<MW>();
      ex -= off;
      off = lin::rescale(max_post(mb, par), bad);
      par ^= 1;
    }
    if (0 < rw.base) {
      if (first_wave && rw.base + rw.li < L) exps[rw.base + rw.li] = ev;
      rw.take(rw.base - W, rw.base - 2 * W, bad);
      far += (double)rw.cf;
    }
    rw.put_i(ev, ex, 0);
    if (first_wave && rw.li < L) exps[rw.li] = ev;
    float xbar = 0.f, rz;
    int exz;
    {
      const float wt = rw.at(rw.cw, 0);
      const float gt = VJP ? rw.at(rw.cg, 0) : 0.f, mf = rw.at(rw.cm, 0);
      const float noff = rw.at(rw.cf, 0) - (float)off;
      const float* const rd = vb + par * PL * GS;
      float sv[2] = {0.f, 0.f};
#pragma unroll
      for (int i = 0; i < SGT; ++i) {
        float Hin[K], Bin[K];
        ld_vec<K>(rd + (tb + i * TPB) * K, Hin);
        if constexpr (VJP) ld_vec<K>(rd + GS + (tb + i * TPB) * K, Bin);
#pragma unroll
        for (int j = 0; j < K; ++j) {
#pragma unroll
          for (int b = 0; b < K; ++b) {
            const float d = fmaf(nkap, cc[i][j][b], wt);
            const float e = ex2(fmaf(-d, d, noff));
            sv[0] = fmaf(e, Hin[b], sv[0]);
            if constexpr (VJP) sv[1] = fmaf(e, fmaf(-gt * (d - mf), Hin[b], Bin[b]), sv[1]);
          }
        }
        asm volatile("" ::: "memory");
      }
      red_pre<2, 0u>(sv, rc);
      lin::block_sync<MW>();
      red_post<2, 0u>(sv, rc);
      if (!(sv[0] > 0.f && sv[0] < INFINITY)) bad = true;
      const int ez = lin::exp_bits(sv[0]);
      sv[0] = ldexpf(sv[0], -ez);
      rz = lin::inv(sv[0]);
      exz = ex - off - ez;
      xbar = ldexpf(sv[1], -ez) * rz;
      far = lin::seg_sum_d(far, W);
      if (tb == 0 && valid && a.logZ)
        a.logZ[bb] = (float)(((double)lg2(sv[0]) - (double)exz - far) * 0.69314718055994530942);
      lin::block_sync<MW>();
    }

    // ------------------------------------------------------------- forward
#pragma unroll 1
    for (int i = tb; i < GS; i += TPB) {
      vb[i] = lin::kTop;
      if constexpr (VJP) vb[GS + i] = 0.f;
    }
    if constexpr (DC) {
#pragma unroll
      for (int i = 0; i < SGT; ++i)
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
          for (int u = 0; u < K; ++u) acc[i][j][u] = 0.f;
    }
    lin::block_sync<MW>();
    ex = lin::kTopExp;
    off = 0;
    par = 0;
    rw.load(0, rw.nw, rw.ng);
    rw.take(0, W, bad);
    int ec = exps[rw.li < L ? rw.li : L - 1];
    int en = exps[W + rw.li < L ? W + rw.li : L - 1];
    float pH[K], pB[K];
    hist_row<K, VJP>(hist, voR, 0, 0, (uint32_t)GS * 4u, pH, pB);
    for (int t = 0; t < L; ++t) {
      if (t >= rw.base + W) {
        const int nb = rw.base + 2 * W;
        rw.take(rw.base + W, nb, bad);
        ec = en;
        en = exps[nb + rw.li < L ? nb + rw.li : L - 1];
      }
      float wt = rw.at(rw.cw, t);
      float gt = VJP ? rw.at(rw.cg, t) : 0.f;
      float mf = rw.at(rw.cm, t);
      lin::to_vgpr(wt, gt, mf);
      const float noff = rw.at(rw.cf, t) - (float)off;
      const int es = exz - (ex - off) - rw.at_i(ec, t);
      if (es > lin::kScaleMax) bad = true;
      const float grz = gt * rz, drz = dws * rz;
      const float* const rd = vb + par * PL * GS;
      float* const wr = vb + (par ^ 1) * PL * GS;
      const int tn = t + 1 < L ? t + 1 : t;
      // max G_{t+1}; sum P d, sum P, sum P (X - xbar), sum P (X - xbar) d
      float vmax = 0.f, m[NM];
#pragma unroll
      for (int q = 0; q < NM; ++q) m[q] = 0.f;
#pragma unroll
      for (int i = 0; i < SGT; ++i) {
        float wtl = wt;
        pin(wtl);
        float Gin[K], Ain[K], gG[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
          Gin[j] = rd[j * NSG + i * TPB + tb];
          if constexpr (VJP) {
            Ain[j] = rd[GS + j * NSG + i * TPB + tb];
            gG[j] = gt * Gin[j];
          }
        }
        float Hc[K], Bc[K];
#pragma unroll
        for (int u = 0; u < K; ++u) {
          Hc[u] = ldexpf(pH[u], es);
          Bc[u] = VJP ? ldexpf(pB[u], es) : 0.f;
        }
        {  // the next super-group's history row (the next step's first after the last)
          const bool last = i + 1 >= SGT;
          hist_row<K, VJP>(hist, voR, (uint32_t)(last ? tn : t) * hstep * 4u,
                           last ? 0u : (uint32_t)(i + 1) * TPB * K * 4u, (uint32_t)GS * 4u, pH, pB);
        }
        float gov[K], aov[K];
#pragma unroll
        for (int u = 0; u < K; ++u) {
          float al[K], qq[K], dd[K], dw[K];  // d about the edge of the range, and about the weight
#pragma unroll
          for (int j = 0; j < K; ++j) {
            dw[j] = fmaf(nkap, cc[i][j][u], wtl);
            dd[j] = dw[j] - mf;
            const float e = ex2(fmaf(-dw[j], dw[j], noff));
            al[j] = e * Gin[j];
            if constexpr (VJP) qq[j] = e * fmaf(-gG[j], dd[j], Ain[j]);
          }
          float go = al[0], sad = al[0] * dd[0], ao = 0.f, sqd = 0.f;
          if constexpr (VJP) {
            ao = qq[0];
            sqd = qq[0] * dd[0];
          }
#pragma unroll
          for (int j = 1; j < K; ++j) {
            go += al[j];
            sad = fmaf(al[j], dd[j], sad);
            if constexpr (VJP) {
              ao += qq[j];
              sqd = fmaf(qq[j], dd[j], sqd);
            }
          }
          gov[u] = go;
          aov[u] = ao;
          const float Hu = Hc[u];
          vmax = as_f(lin::umax(as_u(vmax), as_u(go)));
          m[0] = fmaf(Hu, sad, m[0]);
          m[1] = fmaf(Hu, go, m[1]);
          if constexpr (VJP) {
            const float bx = fmaf(-xbar, Hu, Bc[u]);
            m[VJP ? 2 : 0] = fmaf(go, bx, fmaf(Hu, ao, m[VJP ? 2 : 0]));
            m[VJP ? 3 : 0] = fmaf(sad, bx, fmaf(Hu, sqd, m[VJP ? 3 : 0]));
            if constexpr (DC) {
              // p (g + d (X - E X) / (kappa^2 T)) of the group's K states
              const float aq = Hu * grz, bq = bx * drz, cq = Hu * drz;
#pragma unroll
              for (int j = 0; j < K; ++j) {
                acc[i][j][u] = fmaf(dw[j], fmaf(al[j], bq, qq[j] * cq), fmaf(al[j], aq, acc[i][j][u]));
                pin(acc[i][j][u]);  // (or it sinks below the barrier, its inputs live across)
              }
            }
          }
          if constexpr (KB == 3 || SGT > 1) __builtin_amdgcn_sched_barrier(0);
        }
        st_vec<K>(wr + (tb + i * TPB) * K, gov);
        if constexpr (VJP) st_vec<K>(wr + GS + (tb + i * TPB) * K, aov);
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int c = 0; c < NM; ++c) m[c] *= rz;
      const int q = t & (Q - 1);
      if constexpr (HALF) {
#pragma unroll
        for (int c = 0; c < NM; ++c) m[c] += dpp<0xB1>(m[c]);
        st_vec<NM>(mom + (q * E + (lane >> 1)) * NM, m);
      } else {
        st_vec<NM>(mom + (q * E + lane) * NM, m);
      }
      const bool end = q == Q - 1 || t + 1 == L;
      float r[NM];
      if (end) {  // the wave's sums of the batch (the lane index rebuilt: no address of it stays live)
        const int ln = lane_id();
        lin::wave_sync();
        lin::sum_batch<W, Q, NM, E>(mom, ln, r);
        if constexpr (MW) {
          if (ln % (64 / Q) == 0) st_vec<NM>(wsum + ((par * NW + wave) * Q + ln / (64 / Q)) * NM, r);
        }
      }
      const uint32_t mb = max_pre(vmax, par);
      lin::block_sync<MW>();
      if (end) {
        const int t0 = t - q;
        const int ln = lane_id();
        if constexpr (DC) {
          // E[F] anew from the batch's mean: with one value for the whole block its
          // rounding adds up coherently over the steps of dCodebook (2 to 4 times the error)
          float x = r[VJP ? 2 : 0];
          if constexpr (MW) x = wsum[(par * NW * Q + (ln & (NW * Q - 1))) * NM + (VJP ? 2 : 0)];
          x = seg_reduce<false>(x, MW ? NW * Q : W) * (1.f / (MW ? Q : W));
          if (q == Q - 1) xbar += x;
        }
        if constexpr (MW) {
          if (wave == 0) {
            const float ws = __shfl(rw.cw - rw.cm, t0 - rw.base + (ln & (Q - 1)));
            if (ln < Q) {
              ld_vec<NM>(wsum + (par * NW * Q + ln) * NM, r);
#pragma unroll
              for (int i = 1; i < NW; ++i) {
                float x[NM];
                ld_vec<NM>(wsum + ((par * NW + i) * Q + ln) * NM, x);
#pragma unroll
                for (int c = 0; c < NM; ++c) r[c] += x[c];
              }
              if (t0 + ln < L) lin::step_outputs<VJP>(a, bb * L + t0 + ln, ws, rw.ge(), r, bad);
            }
          }
        } else {
          const int ts = t0 + (ln & (W - 1)) / (W / Q);
          const float ws = __shfl(rw.cw - rw.cm, (ln & ~(W - 1)) + ts - rw.base);
          if (ts < L && valid && (ln & (W - 1)) % (W / Q) == 0)
            lin::step_outputs<VJP>(a, bb * L + ts, ws, rw.ge(), r, bad);
        }
      }
      ex -= off;
      {
        bool out = false;
        off = lin::rescale(max_post(mb, par), out);
        if (out && t + 1 < L) bad = true;
      }
      par ^= 1;
    }
    if constexpr (MW) {
      bad = __syncthreads_or(bad);
    } else {
      const uint64_t any = __ballot(bad) >> seg0;
      bad = (W == 64 ? any : any & ((1ull << W) - 1)) != 0;
      lin::wave_sync();
    }
    if (tb == 0 && valid) a.flags[bb] = bad ? 1 : 0;
    if constexpr (DC) {
      if (valid && !bad) {
        const double pow2 = lin::pow2_d(rw.ge());
#pragma unroll
        for (int i = 0; i < SGT; ++i)
#pragma unroll
          for (int j = 0; j < K; ++j) {
            double* const pj = part_at(i, j);
#pragma unroll
            for (int u = 0; u < K; ++u) pj[u] = fma((double)acc[i][j][u], pow2, pj[u]);
            asm volatile("" ::: "memory");
          }
      }
    }
  }
}

}  // namespace bcjr
