// Drafting with the draft model resident in one workgroup's registers (§4.3
// "Drafting", the inner loop of Algorithm 1): small draft models (d_head 16,
// width 16, 32 or 64, one or two layers; THP, or AttNHP without FFN).
//
// One workgroup runs all gamma draft steps of a sequence. The model's matrices
// are loaded once into MFMA operand registers, spread over the workgroup's
// waves (a 64-wide, two-layer bf16 model with F = 256 is 234 fragments of 16
// outputs x 32 inputs: with tiles dealt out whole 32 per wave over eight waves,
// 128 of the 256 registers),
// so that a step's products read only the activations, from LDS. Weights are
// the products' first operand: lane (r, g) of a result holds outputs 4 g .. + 3
// of token r (one token, two in the first step, which re-encodes the last two
// committed events; the other columns repeat one).
//
// What bounds it: instructions (every wave issues the row-local work of every
// phase again) and the chain of phases, each a barrier, an LDS round trip and
// two or more dependent matrix instructions, five per layer and three for the
// decoder and the draw; then the stream of cached keys and values. So
//  - the residual stream is one element per lane in every wave's registers;
//    LayerNorms, the merge of the attention's partials and the residual sums
//    take a few dozen instructions there and go to operand layout through a
//    wave's own LDS row, instead of taking phases (barriers) of their own;
//  - products with few output tiles split K over the waves and leave their
//    partial sums to the next phase's readers;
//  - the keys and values of committed positions do not change during the
//    launch: a batch of them is always in flight across the phases before the
//    attention that takes it. The round's own positions (at most gamma + 1)
//    are kept in LDS;
//  - the scores of 64 keys come out one per lane (the query sits in a
//    different row of the operand for each group of 16 keys), so that the
//    softmax costs one exponential per 64 keys and wave, and go back through
//    LDS as the operand of the value product;
//  - the draw runs the mixture chain and the type chain on two waves, a third
//    forms the record.
// Measured, 10 drafts (before: one workgroup with weights in LDS or L2, for
// AttNHP the per-step kernels): fp32 d = 32, 64 sequences of 40 events 118 ->
// 56 us; bf16 d = 64, two layers, 256 sequences of 576 events 333 -> 178 us (of
// these some 95 us are the cache at 8 TB/s); AttNHP d = 64, two layers, 256
// sequences of 580 events 417 -> 146 us.
// Rounding points are those of the layered kernels, but for THP's attention
// probabilities, which are not rounded (as in the other one-launch kernels).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "tppsd_device.h"
#include "tppsd_philox.h"
#include "../../include/tppsd.h"

namespace tppsd {

namespace {

constexpr int DG_TAIL = 64;   // positions of the round kept in LDS (gamma + 1 <= 33), one step of 64
constexpr int DG_HEAD_TILES = 8;   // 16-row tiles of the decoder heads

template <typename ELT> struct DgFrag;
template <> struct DgFrag<bf16_t> {
  typedef bf16x8_t frag;
  static __device__ __forceinline__ frag pack(const float *v) {
    return __builtin_bit_cast(frag, make_uint4(pk2bf(v[0], v[1]), pk2bf(v[2], v[3]), pk2bf(v[4], v[5]),
                                               pk2bf(v[6], v[7])));
  }
};
template <> struct DgFrag<float> {
  typedef f32x4_t frag;
  static __device__ __forceinline__ frag pack(const float *v) { return (f32x4_t){v[0], v[1], v[2], v[3]}; }
};

// Attention over 64 consecutive cached positions of one head, d_head = 16:
// keys kt + lane scored one per lane; probabilities come back from LDS.
// bf16: MFMA. Lane (r, g) holds dims 4 g .. + 3 of keys 16 m + r (m = 0..3) and,
// as the value operand, positions 32 c + 8 g .. + 7 of column r; group m's
// product puts the queries in rows 4 m, 4 m + 1 of its first operand, so that
// lane (r, g) ends up with the scores of key 16 g + r. THP's probabilities stay
// in fp32, as the other one-launch drafting kernels have them: each is cut into
// three bf16 parts, which hold all of its 24 bits, with a product each (the
// three sums do not wait for one another). AttNHP's are rounded to bf16, as in
// the layered kernels that serve its other sizes. Their sum is kept by the lane.
// (Ten drafts of 256 sequences after 576 events, d = 64, two layers: 178 us,
// with rounded probabilities 169.)
// fp32: vector ALU (an fp32 matrix instruction with one query in 16 rows takes
// eight times the cycles of the FMAs): lane holds its key's row and, for the
// value sums, positions 16 g + s of column r.
template <typename ELT> struct DgStep;
template <> struct DgStep<bf16_t> {
  uint2 k[4];
  uint4 v[2];
  // last: the last valid position (loads are clamped to it)
  __device__ __forceinline__ void load_k(const bf16_t *kc, int kt, int last, int lane) {
    const int rr = lane & 15, g = lane >> 4;
    const bf16_t *p = kc + kt * 16;
    const int off = rr * 16 + 4 * g;
    if (kt + 63 <= last) {   // (uniform)
#pragma unroll
      for (int m = 0; m < 4; ++m) k[m] = *(const uint2 *)(p + off + 256 * m);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) k[m] = *(const uint2 *)(p + min(16 * m + rr, last - kt) * 16 + 4 * g);
    }
  }
  __device__ __forceinline__ void load_v(const bf16_t *vc, int kt, int last, int lane) {
    const int rr = lane & 15, g = lane >> 4;
    const bf16_t *p = vc + kt * 16;
    const int n8 = (last - kt) >> 3;   // (the last block of the step)
#pragma unroll
    for (int c = 0; c < 2; ++c) v[c] = *(const uint4 *)(p + min(4 * c + g, n8) * 128 + rr * 8);
  }
};
template <> struct DgStep<float> {
  float4 k[4];
  float v[16];
  __device__ __forceinline__ void load_k(const float *kc, int kt, int last, int lane) {
    const float *p = kc + kt * 16 + min(lane, last - kt) * 16;
#pragma unroll
    for (int c = 0; c < 4; ++c) k[c] = *(const float4 *)(p + 4 * c);
  }
  __device__ __forceinline__ void load_v(const float *vc, int kt, int last, int lane) {
    const int rr = lane & 15, g = lane >> 4;
    const float *p = vc + kt * 16;
    if (kt + 63 <= last) {   // (uniform)
#pragma unroll
      for (int s = 0; s < 16; ++s) v[s] = p[256 * g + rr + 16 * s];
    } else {
#pragma unroll
      for (int s = 0; s < 16; ++s) v[s] = p[min(16 * g + s, last - kt) * 16 + rr];
    }
  }
};

// the one or two queries of a wave's head and their running sums
// NPL: parts of a bf16 kernel's probability
template <typename ELT, int NPL> struct DgAttn;
template <int NPL> struct DgAttn<bf16_t, NPL> {
  uint2 q[4];
  f32x4_t o[NPL];
  float l[2];
  // qs: query rows in LDS, this head's 16 dims
  __device__ __forceinline__ void init(const bf16_t *q0, int ld, int P, int lane) {
    const int rr = lane & 15, g = lane >> 4;
    const uint2 qv = *(const uint2 *)(q0 + min(rr & 3, P - 1) * ld + 4 * g);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bool in = (rr >> 2) == m && (rr & 3) < P;
      q[m] = make_uint2(in ? qv.x : 0u, in ? qv.y : 0u);
    }
#pragma unroll
    for (int i = 0; i < NPL; ++i) o[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    l[0] = l[1] = 0.f;
  }
  __device__ __forceinline__ void scores(const DgStep<bf16_t> &st, int P, float &s0, float &s1) const {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 4; ++m)
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, q[m]),
                                                      __builtin_bit_cast(short4_t, st.k[m]), acc, 0, 0, 0);
    s0 = acc[0];
    s1 = acc[1];
  }
  __device__ __forceinline__ void rescale(float a0, float a1, int lane) {
    const float a = (lane & 15) == 1 ? a1 : a0;   // column r is query r
#pragma unroll
    for (int i = 0; i < NPL; ++i) o[i] *= a;
    l[0] *= a0, l[1] *= a1;
  }
  // the lane's probability of a step for query t, to the parts' rows (ldl apart)
  __device__ __forceinline__ void keep(int t, float p, bf16_t *row, int ldl) {
    if constexpr (NPL == 1) {
      *row = f2bf(p);
      l[t] += rnd_act<bf16_t>(p);
    } else {
      const float m = p - __uint_as_float(__float_as_uint(p) & 0xFFFF0000u);
      const float s = m - __uint_as_float(__float_as_uint(m) & 0xFFFF0000u);
      row[0] = (bf16_t)(__float_as_uint(p) >> 16);
      row[ldl] = (bf16_t)(__float_as_uint(m) >> 16);
      row[2 * ldl] = (bf16_t)(__float_as_uint(s) >> 16);
      l[t] += p;
    }
  }
  // p: the queries' rows of probabilities in LDS (parts ldl apart); nv: valid positions of the step
  __device__ __forceinline__ void apply(const DgStep<bf16_t> &st, const bf16_t *p, int ldl, int P, int nv, int lane) {
    const int rr = lane & 15, g = lane >> 4;
    const bf16_t *pr = p + min(rr, P - 1) * NPL * ldl + 8 * g;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      u32x4_t w = {st.v[c].x, st.v[c].y, st.v[c].z, st.v[c].w};
      if (nv < 64) {   // (uniform: values past the range may be any bits)
        const int n8 = nv - 32 * c - 8 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = 2 * i >= n8 ? 0u : (2 * i + 1 >= n8 ? w[i] & 0xFFFFu : w[i]);
      }
#pragma unroll
      for (int i = 0; i < NPL; ++i)
        o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w),
                                                       *(const bf16x8_t *)(pr + i * ldl + 32 * c), o[i], 0, 0, 0);
    }
  }
  // r: [2][ld] per query (max, sum, -, -, 16 sums)
  __device__ __forceinline__ void finish(float *r, int ld, int P, int lane) const {
    const int rr = lane & 15, g = lane >> 4;
    f32x4_t sum = o[0];
    if constexpr (NPL == 3) sum += o[1] + o[2];
    if (rr < P) *(f32x4_t *)(r + rr * ld + 4 + 4 * g) = sum;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= P) break;
      const float sl = lanes_sum<64>(l[t]);
      if (lane == 0) r[t * ld + 1] = sl;
    }
  }
};
template <int NPL> struct DgAttn<float, NPL> {
  float4 q0[4];
  const float *q1;   // the second query's row, read where it is used
  float o[2], l[2];
  __device__ __forceinline__ void init(const float *qr, int ld, int P, int lane) {
#pragma unroll
    for (int c = 0; c < 4; ++c) q0[c] = *(const float4 *)(qr + 4 * c);
    q1 = qr + ld;
    o[0] = o[1] = l[0] = l[1] = 0.f;
  }
  static __device__ __forceinline__ float dot(const float4 *a, const float4 *b) {
    float s[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = fmaf(a[c].w, b[c].w, fmaf(a[c].z, b[c].z, fmaf(a[c].y, b[c].y, a[c].x * b[c].x)));
    return (s[0] + s[1]) + (s[2] + s[3]);
  }
  __device__ __forceinline__ void scores(const DgStep<float> &st, int P, float &s0, float &s1) const {
    s0 = dot(q0, st.k);
    s1 = 0.f;
    if (P == 2) {   // (uniform)
      float4 q[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) q[c] = *(const float4 *)(q1 + 4 * c);
      s1 = dot(q, st.k);
    }
  }
  __device__ __forceinline__ void rescale(float a0, float a1, int) {
    o[0] *= a0, l[0] *= a0;
    o[1] *= a1, l[1] *= a1;
  }
  __device__ __forceinline__ void keep(int, float p, float *row, int) { *row = p; }
  // (values past the range were clamped to its last position: finite, times a probability of 0)
  __device__ __forceinline__ void apply(const DgStep<float> &st, const float *p, int ldp, int P, int nv, int lane) {
    const int g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= P) break;   // uniform
      float so[4], sl[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float4 w = *(const float4 *)(p + t * ldp + 16 * g + 4 * c);
        so[c] = fmaf(w.w, st.v[4 * c + 3], fmaf(w.z, st.v[4 * c + 2], fmaf(w.y, st.v[4 * c + 1], w.x * st.v[4 * c])));
        sl[c] = (w.x + w.y) + (w.z + w.w);
      }
      o[t] += (so[0] + so[1]) + (so[2] + so[3]);
      l[t] += (sl[0] + sl[1]) + (sl[2] + sl[3]);
    }
  }
  __device__ __forceinline__ void finish(float *r, int ld, int P, int lane) const {
    const int rr = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= P) break;
      const float so = xor32_sum(xor16_sum(o[t])), sl = xor32_sum(xor16_sum(l[t]));
      if (g == 0) r[t * ld + 4 + rr] = so;
      if (lane == 0) r[t * ld + 1] = sl;
    }
  }
};

// A 16-row tile of matrix-vector products over NK k-steps. w: the tile's
// fragments; act(t, s): token t's operand fragment of k-step s. Outputs of a
// lane: NE rows from n0, for token tk (in use where tk < P).
// bf16: MFMA, lane (r, g): rows 4 g .. + 3 of token r. fp32: FMAs over the
// lane's k values, summed over its row's four lanes; lane (r, g): row r of token g.
template <typename ELT> struct DgTile;
template <> struct DgTile<bf16_t> {
  static constexpr int NE = 4;
  static __device__ __forceinline__ int n0(int lane) { return 4 * (lane >> 4); }
  static __device__ __forceinline__ int tk(int lane) { return lane & 15; }
  template <int NK, typename A>
  static __device__ __forceinline__ void mul(const bf16x8_t *w, A act, int P, int lane, float (&y)[NE]) {
    const int t = min(lane & 15, P - 1);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NK; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], act(t, s), acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NE; ++i) y[i] = acc[i];
  }
  // NE consecutive elements
  static __device__ __forceinline__ void store(bf16_t *p, const float (&v)[NE]) {
    *(uint2 *)p = make_uint2(pk2bf(v[0], v[1]), pk2bf(v[2], v[3]));
  }
  static __device__ __forceinline__ void store(float *p, const float (&v)[NE]) {
    *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <> struct DgTile<float> {
  static constexpr int NE = 1;
  static __device__ __forceinline__ int n0(int lane) { return lane & 15; }
  static __device__ __forceinline__ int tk(int lane) { return lane >> 4; }
  template <int NK, typename A>
  static __device__ __forceinline__ void mul(const f32x4_t *w, A act, int P, int lane, float (&y)[NE]) {
    float r[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= P) break;   // uniform
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < NK; ++s) {
        const f32x4_t x = act(t, s);
        v += fmaf(w[s][3], x[3], fmaf(w[s][2], x[2], fmaf(w[s][1], x[1], w[s][0] * x[0])));
      }
      r[t] = xor32_sum(xor16_sum(v));
    }
    y[0] = (lane >> 4) == 1 ? r[1] : r[0];
  }
  static __device__ __forceinline__ void store(float *p, const float (&v)[NE]) { *p = v[0]; }
};

// D: model width, F: FFN width (0: AttNHP), L: layers, NW: waves
template <typename ELT, int D, int F, int L, int NW>
__global__ __launch_bounds__(64 * NW) void k_draft_regs(DraftArgs a) {
  typedef MfmaStep<ELT> S;
  typedef DgFrag<ELT> X;
  typedef typename X::frag frag;
  typedef DgTile<ELT> Tile;
  constexpr int NPL = sizeof(ELT) == 2 && F != 0 ? 3 : 1;
  constexpr int NE = Tile::NE;
  constexpr bool NHP = F == 0;
  constexpr int KS = S::KSTEP, VE = 16 / sizeof(ELT), DH = 16, H = D / 16;
  constexpr int DK = NHP ? 2 * D : D;                  // input width of q, k, v
  constexpr int KD = D / KS, KQ = DK / KS, KF = NHP ? 1 : F / KS;
  constexpr int TQ = 3 * D / 16, TPQ = (TQ + NW - 1) / NW;
  constexpr int TF = F / 16, TPF = NHP ? 1 : (TF + NW - 1) / NW;
  constexpr int TE = 4 * D / 16, TPE = (TE + NW - 1) / NW;
  constexpr int TPH = DG_HEAD_TILES / NW;
  constexpr int DT = D / 16, KG = NW / DT;             // narrow products: D / 16 tiles, K over KG waves each
  constexpr int KGO = KG < KD ? KG : KD, NO = KD / KGO;
  constexpr int KGF = KG < KF ? KG : KF, NF = KF / KGF;
  constexpr int WPH = NW / H;                          // waves per head
  // 64-key steps per batch: what fits beside the weights without a spill
  constexpr int NB = sizeof(ELT) != 2 || (D == 64 && L == 2 && !NHP) ? 2 : D == 64 && F == 256 ? 3 : 4;
  constexpr int LV = NHP ? 3 * D : 9 * D + F;          // small vectors per layer
  constexpr int NP = D == 64 ? 2 : 1;                  // registers of the residual stream per lane
  static_assert(NW % DT == 0 && NW % H == 0 && KD >= 1 && TPH >= 1 && (NHP || KF % KGF == 0), "shapes");
  __shared__ __attribute__((aligned(16))) float pA[KGO][2][D], pB[KGF][2][D], zs[2][D];
  __shared__ __attribute__((aligned(16))) ELT as[NW][2][D];   // each wave's operand rows
  __shared__ __attribute__((aligned(16))) float pm[NW][2][DH + 4];
  __shared__ __attribute__((aligned(16))) ELT qs[2][D], hs[2][NHP ? 4 : F], es[4 * D], pbuf[NW][2][NPL][NB * 64];
  __shared__ __attribute__((aligned(16))) ELT kt_s[L][H][DG_TAIL * DH], vt_s[L][H][DG_TAIL * DH];
  __shared__ __attribute__((aligned(16))) float vec[L * LV + 4 * D + DG_HEAD_TILES * 16], hv[DG_HEAD_TILES * 16];
  __shared__ __attribute__((aligned(16))) ELT emb[TPPSD_MAX_TYPES * D];
  __shared__ float pu[TPPSD_MAX_GAMMA][4];
  __shared__ int tok_k[2];
  const int b = blockIdx.x;
  if (a.done[b]) return;
  const int tid = threadIdx.x;
  int lane = tid & 63, rr = lane & 15, g = lane >> 4;
  int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (scalar: its branches and addresses are uniform)
  const int M = a.M, K = a.K;
  const int n = a.n[b], base = a.lenD[b];
  int ne0 = Tile::n0(lane), tk = Tile::tk(lane);   // a product's rows and token in this lane
  const int Mt = (M + 15) / 16, Kt = (K + 15) / 16;
  int j = lane & (D - 1), tok = D == 64 ? 0 : (lane / D) & 1;   // element and token of the lane's stream
  int tn = wave % DT, kg = wave / DT;             // narrow products: this wave's tile and K group
  int head = wave / WPH, sub = wave % WPH;        // attention: its head and place among the head's waves
  // Everything derived from the lane and the wave is formed again in each
  // phase: as values known over the whole loop they (LDS addresses above all)
  // would be kept in some 90 registers, and the weights spilled for them.
  auto phase = [&]() {
    asm volatile("" : "+v"(lane), "+s"(wave));
    rr = lane & 15;
    g = lane >> 4;
    ne0 = Tile::n0(lane);
    tk = Tile::tk(lane);
    j = lane & (D - 1);
    tok = D == 64 ? 0 : (lane / D) & 1;
    tn = wave % DT;
    kg = wave / DT;
    head = wave / WPH;
    sub = wave % WPH;
  };

  // ---- the model into registers -------------------------------------------
  auto wfrag = [&](const void *W, int row, int ld, int s) -> frag {
    return *(const frag *)((const ELT *)W + (size_t)row * ld + KS * s + VE * g);
  };
  frag wq[L][TPQ][KQ], wo[NHP ? 1 : L][NO], w1[NHP ? 1 : L][TPF][KD], w2[NHP ? 1 : L][NF], we[TPE][KD], wh[TPH][KD];
#pragma unroll
  for (int ly = 0; ly < L; ++ly) {
    const FusedLayerW &w = a.layer[ly];
#pragma unroll
    for (int i = 0; i < TPQ; ++i)
#pragma unroll
      for (int s = 0; s < KQ; ++s) wq[ly][i][s] = wfrag(w.qkv_w, 16 * min(wave + NW * i, TQ - 1) + rr, DK, s);
    if constexpr (!NHP) {
#pragma unroll
      for (int s = 0; s < NO; ++s) wo[ly][s] = wfrag(w.out_w, 16 * tn + rr, D, min(kg, KGO - 1) * NO + s);
#pragma unroll
      for (int i = 0; i < TPF; ++i)
#pragma unroll
        for (int s = 0; s < KD; ++s) w1[ly][i][s] = wfrag(w.ffn1_w, 16 * min(wave + NW * i, TF - 1) + rr, D, s);
#pragma unroll
      for (int s = 0; s < NF; ++s) w2[ly][s] = wfrag(w.ffn2_w, 16 * tn + rr, F, min(kg, KGF - 1) * NF + s);
    }
  }
#pragma unroll
  for (int i = 0; i < TPE; ++i)
#pragma unroll
    for (int s = 0; s < KD; ++s) we[i][s] = wfrag(a.Ek1_w, 16 * min(wave + NW * i, TE - 1) + rr, D, s);
  // head tile t: 16 rows of V_w, V_mu, V_sigma (on e1, e2, e3) or V_k2 (on the
  // tanh row); rows past a head's count repeat its last and are not used
#pragma unroll
  for (int i = 0; i < TPH; ++i) {
    const int t = wave + NW * i, c = min(t / Mt, 3);
    const ELT *hw = c < 3 ? (const ELT *)a.mix_w + (size_t)c * M * D : (const ELT *)a.k2_w;
    const int row = c < 3 ? min(16 * (t % Mt) + rr, M - 1) : min(16 * (t - 3 * Mt) + rr, K - 1);
#pragma unroll
    for (int s = 0; s < KD; ++s) wh[i][s] = wfrag(hw, row, D, s);
  }

  // ---- cached keys and values: the first batch of layer 0 -----------------
  auto slab = [&]() { return ((size_t)b * H + head) * a.cap * DH; };
  auto kcache = [&](int ly) { return (const ELT *)(a.kc + a.layer_bytes * ly) + slab(); };
  auto vcache = [&](int ly) { return (const ELT *)(a.vc + a.layer_bytes * ly) + slab(); };
  const int nst = (base + 63) / 64;                                   // steps of committed positions
  const int mine = nst > sub ? (nst - sub + WPH - 1) / WPH : 0;       // this wave's
  DgStep<ELT> kv[NB];
  auto fetch_k = [&](int ly, int bt) {
    if (nst == 0) return;   // (uniform)
#pragma unroll
    for (int i = 0; i < NB; ++i)
      kv[i].load_k(kcache(ly), 64 * min(sub + WPH * (bt * NB + i), nst - 1), base - 1, lane);
  };
  auto fetch_v = [&](int ly, int bt) {
    if (nst == 0) return;
#pragma unroll
    for (int i = 0; i < NB; ++i)
      kv[i].load_v(vcache(ly), 64 * min(sub + WPH * (bt * NB + i), nst - 1), base - 1, lane);
  };
  fetch_k(0, 0);
  fetch_v(0, 0);

  // ---- small vectors, embeddings, draw numbers, the first step's tokens ---
  float t_last = a.ev_t[(size_t)b * a.ev_stride + n - 1];
  {
    auto cp = [&](float *dst, const float *src, int cnt) {
      for (int i = tid; i < cnt; i += 64 * NW) dst[i] = src[i];
    };
    for (int ly = 0; ly < L; ++ly) {
      const FusedLayerW &w = a.layer[ly];
      float *v = vec + ly * LV;
      cp(v, w.qkv_b, 3 * D);
      if constexpr (!NHP) {
        cp(v + 3 * D, w.ln1_g, D);
        cp(v + 4 * D, w.ln1_b, D);
        cp(v + 5 * D, w.out_b, D);
        cp(v + 6 * D, w.ln2_g, D);
        cp(v + 7 * D, w.ln2_b, D);
        cp(v + 8 * D, w.ffn2_b, D);
        cp(v + 9 * D, w.ffn1_b, F);
      }
    }
    float *v = vec + L * LV;
    if constexpr (!NHP) {
      cp(v, a.lnf_g, D);
      cp(v + D, a.lnf_b, D);
    }
    cp(v + 2 * D, a.k1_b, D);
    cp(v + 3 * D, a.freq, D);
    cp(v + 4 * D, a.mix_b, 3 * M);
    cp(v + 4 * D + 3 * M, a.k2_b, K);
    const ELT *we_g = (const ELT *)a.type_emb;
    for (int i = tid; i < K * D; i += 64 * NW) emb[i] = we_g[i];
    for (int i = tid; i < L * H * DG_TAIL * DH; i += 64 * NW) {
      (&kt_s[0][0][0])[i] = 0;
      (&vt_s[0][0][0])[i] = 0;
    }
  }
  const float *hvec = vec + L * LV;
  const float *freq = hvec + 3 * D, *head_b = hvec + 4 * D;
  if (tid < a.gamma) {   // the draws' numbers depend only on the counters
    float u[4];
    philox_uniforms(a.seed, (uint64_t)b, (uint64_t)a.rnd[b], (uint64_t)(tid + 1), TAG_DRAFT, u);
    pu[tid][0] = u[0];
    pu[tid][1] = sqrtf(-2.f * logf(u[1])) * cosf(6.28318530717958647692f * u[2]);   // Box-Muller deviate
    pu[tid][2] = u[3];
  }
  for (int i = tid; i < 2 * D; i += 64 * NW) {
    const int p = i / D, j = i - p * D;
    const float arg = a.ev_t[(size_t)b * a.ev_stride + n - 2 + p] * a.freq[j];
    zs[p][j] = (j & 1) ? cosf(arg) : sinf(arg);
  }
  if (tid < 2) tok_k[tid] = min(max(a.ev_k[(size_t)b * a.ev_stride + n - 2 + tid], 0), K - 1);
  lds_barrier();

  const float scale = sizeof(ELT) == 2 ? 0.25f * 1.4426950408889634f : 0.25f;   // 1 / sqrt(16) (base-2 units)
  for (int l = 1; l <= a.gamma; ++l) {
    const int P = (l == 1) ? 2 : 1;
    const int pos0 = (l == 1) ? base : base + l, off0 = pos0 - base;
    auto k_of = [&](int s) { return KS * s + VE * g; };
    // the residual stream: element (token, j) of lane; a wave of 64 lanes holds
    // one row of 64 (the second token in the second register), or both rows
    float x[NP];
    // pending partial sums and their bias into the stream
    auto add = [&](const float (*parts)[2][D], int np, const float *bias) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        if (i >= P) break;   // uniform
        const int t = D == 64 ? i : tok;
        float v = parts[0][t][j];
        for (int q = 1; q < np; ++q) v += parts[q][t][j];
        x[i] += v + bias[j];
      }
    };
    auto to_operand = [&](int i, float v) { st(&as[wave][D == 64 ? i : tok][0], j, v); };
    // LayerNorm of the stream (biased variance, two passes) into the operand rows
    auto norm = [&](const float *gn, const float *bt) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        if (i >= P) break;
        const float mean = lanes_sum<D>(x[i]) / (float)D, c = x[i] - mean;
        const float rstd = rsqrt_nr(lanes_sum<D>(c * c) / (float)D + 1e-5f);
        to_operand(i, c * rstd * gn[j] + bt[j]);
      }
      wave_lds_order();
    };
    auto operand = [&](int t, int s) -> frag { return *(const frag *)&as[wave][t][k_of(s)]; };
    // this lane's element of the attention output of the layer whose partials are in pm
    auto merged = [&](int i) -> float {
      const int t = D == 64 ? i : tok, hh = j / DH;
      float m[WPH], Mx = NHP ? 0.f : -INFINITY;   // (AttNHP: the extra key of score 0, value 0)
#pragma unroll
      for (int w = 0; w < WPH; ++w) {
        m[w] = pm[hh * WPH + w][t][0];
        Mx = fmaxf(Mx, m[w]);
      }
      float Ls = NHP ? exp_score<ELT>(-Mx) : 0.f, o = 0.f;
#pragma unroll
      for (int w = 0; w < WPH; ++w) {
        const float *r = pm[hh * WPH + w][t];
        const float f = (m[w] == -INFINITY) ? 0.f : exp_score<ELT>(m[w] - Mx);
        Ls += r[1] * f;
        o += r[4 + j % DH] * f;
      }
      return rnd_act<ELT>(Ls > 0.f ? o * rcp_nr(Ls) : 0.f);
    };

#pragma unroll
    for (int ly = 0; ly < L; ++ly) {
      const float *lv = vec + ly * LV;
      phase();
      // ---- q, k, v ---------------------------------------------------------
      if (ly == 0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const int t = D == 64 ? i : tok;
          x[i] = ld(emb, tok_k[t] * D + j) + (NHP ? 0.f : zs[t][j]);
        }
      }
      if constexpr (NHP) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          if (i >= P) break;
          if (ly > 0) x[i] += tanhf(merged(i));
          to_operand(i, x[i]);
        }
        wave_lds_order();
      } else {
        if (ly > 0) add(pB, KGF, lv - LV + 8 * D);
        norm(lv + 3 * D, lv + 4 * D);
      }
      // (AttNHP: u = [z(t); h])
      auto in = [&](int t, int s) -> frag { return NHP && s < KD ? X::pack(&zs[t][k_of(s)]) : operand(t, NHP ? s - KD : s); };
#pragma unroll
      for (int i = 0; i < TPQ; ++i) {
        const int t = wave + NW * i;
        if (t >= TQ) break;   // uniform across the wave
        float y[NE];
        Tile::template mul<KQ>(wq[ly][i], in, P, lane, y);
        if (tk < P) {
          const int which = t / DT, hh = t % DT;
#pragma unroll
          for (int c = 0; c < NE; ++c) y[c] += lv[16 * t + ne0 + c];
          const int pt = off0 + tk, pos = pos0 + tk;
          if (which == 0) {
            Tile::store(&qs[tk][16 * hh + ne0], y);
          } else {
            const bool fits = pos < a.cap;
            if (!fits) atomicOr(a.status, TPPSD_STATUS_CAPACITY);
            const size_t row0 = ((size_t)b * H + hh) * a.cap * DH;   // (uniform)
            if (which == 1) {
              Tile::store(&kt_s[ly][hh][pt * DH + ne0], y);
              if (fits) Tile::store((ELT *)(a.kc + a.layer_bytes * ly) + row0 + (pos * DH + ne0), y);
            } else {
              ELT *gv = (ELT *)(a.vc + a.layer_bytes * ly) + row0;
#pragma unroll
              for (int c = 0; c < NE; ++c) {
                st(&vt_s[ly][hh][0], v_at<ELT>(0, pt, ne0 + c, DH), y[c]);
                if (fits) st(gv, (int)v_at<ELT>(0, pos, ne0 + c, DH), y[c]);
              }
            }
          }
        }
      }
      lds_barrier();
      phase();
      // ---- attention: this wave's share of its head's keys ------------------
      {
        DgAttn<ELT, NPL> at;
        at.init(&qs[0][16 * head], D, P, lane);
        float m_run[2] = {-INFINITY, -INFINITY};
        // ns steps whose scores are in sc: running maxima, rescaled sums, probabilities to LDS
        auto softmax = [&](float (&sc)[2][NB], int ns) {
          float al[2] = {1.f, 1.f};
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            if (p >= P) break;   // uniform
            float mx = sc[p][0];
#pragma unroll
            for (int i = 1; i < NB; ++i) mx = fmaxf(mx, sc[p][i]);
            const float m_new = fmaxf(m_run[p], lanes_max(mx));
            al[p] = exp_score<ELT>(m_run[p] - (m_new == -INFINITY ? 0.f : m_new));
            m_run[p] = m_new;
          }
          at.rescale(al[0], al[1], lane);
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            if (p >= P) break;
            const float m_ref = m_run[p] == -INFINITY ? 0.f : m_run[p];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              if (i >= ns) break;   // uniform
              at.keep(p, exp_score<ELT>(sc[p][i] - m_ref), &pbuf[wave][p][0][64 * i + lane], NB * 64);
            }
          }
          wave_lds_order();
        };
        const int nbt = (mine + NB - 1) / NB;
        const int nly = ly + 1 == L ? 0 : ly + 1;    // the next attention's layer
        for (int bt = 0; bt < nbt; ++bt) {
          float sc[2][NB];
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int idx = bt * NB + i, key = 64 * (sub + WPH * idx) + lane;
            sc[0][i] = sc[1][i] = -INFINITY;
            if (idx >= mine) continue;   // uniform
            float s0, s1;
            at.scores(kv[i], P, s0, s1);
            sc[0][i] = key < base ? s0 * scale : -INFINITY;
            sc[1][i] = key < base ? s1 * scale : -INFINITY;
          }
          const bool more = bt + 1 < nbt;
          fetch_k(more ? ly : nly, more ? bt + 1 : 0);
          softmax(sc, min(NB, mine - bt * NB));
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int idx = bt * NB + i;
            if (idx >= mine) break;   // uniform
            at.apply(kv[i], &pbuf[wave][0][0][64 * i], NB * 64, P, base - 64 * (sub + WPH * idx), lane);
          }
          wave_lds_order();
          fetch_v(more ? ly : nly, more ? bt + 1 : 0);
        }
        if (sub == nst % WPH) {
          // the round's own positions, one step from LDS
          DgStep<ELT> tl;
          tl.load_k(&kt_s[ly][head][0], 0, DG_TAIL - 1, lane);
          tl.load_v(&vt_s[ly][head][0], 0, DG_TAIL - 1, lane);
          float sc[2][NB], s0, s1;
#pragma unroll
          for (int i = 0; i < NB; ++i) sc[0][i] = sc[1][i] = -INFINITY;
          at.scores(tl, P, s0, s1);
          const bool in_cap = base + lane < a.cap;
          sc[0][0] = in_cap && lane <= off0 ? s0 * scale : -INFINITY;
          sc[1][0] = in_cap && lane <= off0 + 1 ? s1 * scale : -INFINITY;
          softmax(sc, 1);
          at.apply(tl, &pbuf[wave][0][0][0], NB * 64, P, 64, lane);
          wave_lds_order();
        }
        at.finish(&pm[wave][0][0], DH + 4, P, lane);
        if (lane == 0) {
          pm[wave][0][0] = m_run[0];
          pm[wave][1][0] = m_run[1];
        }
      }
      lds_barrier();
      phase();
      if constexpr (!NHP) {
        // ---- output projection (K over the waves of a tile) -----------------
        if (kg < KGO) {
#pragma unroll
          for (int i = 0; i < NP; ++i) {
            if (i >= P) break;
            to_operand(i, merged(i));
          }
          wave_lds_order();
          float y[NE];
          Tile::template mul<NO>(wo[ly], [&](int t, int s) -> frag { return operand(t, kg * NO + s); }, P, lane, y);
          if (tk < P) Tile::store(&pA[kg][tk][16 * tn + ne0], y);
          wave_lds_order();
        }
        lds_barrier();
        phase();
        // ---- feed-forward block ---------------------------------------------
        add(pA, KGO, lv + 5 * D);
        norm(lv + 6 * D, lv + 7 * D);
#pragma unroll
        for (int i = 0; i < TPF; ++i) {
          const int t = wave + NW * i;
          if (t >= TF) break;
          float y[NE];
          Tile::template mul<KD>(w1[ly][i], operand, P, lane, y);
          if (tk < P) {
#pragma unroll
            for (int c = 0; c < NE; ++c) y[c] = fmaxf(y[c] + lv[9 * D + 16 * t + ne0 + c], 0.f);
            Tile::store(&hs[tk][16 * t + ne0], y);
          }
        }
        lds_barrier();
        phase();
        if (kg < KGF) {
          float y[NE];
          Tile::template mul<NF>(
              w2[ly], [&](int t, int s) -> frag { return *(const frag *)&hs[t][KS * (kg * NF + s) + VE * g]; }, P, lane, y);
          if (tk < P) Tile::store(&pB[kg][tk][16 * tn + ne0], y);
        }
        lds_barrier();
      }
    }
    phase();
    // ---- decoder of the last token: [E; V_k1], tanh ------------------------
    if constexpr (NHP) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        if (i >= P) break;
        x[i] += tanhf(merged(i));
        to_operand(i, x[i]);
      }
      wave_lds_order();
    } else {
      add(pB, KGF, vec + (L - 1) * LV + 8 * D);
      norm(hvec, hvec + D);
    }
#pragma unroll
    for (int i = 0; i < TPE; ++i) {
      const int t = wave + NW * i;
      if (t >= TE) break;
      float y[NE];
      Tile::template mul<KD>(we[i], [&](int, int s) -> frag { return operand(P - 1, s); }, 1, lane, y);
      if (16 * t >= 3 * D) {   // (uniform: a tile of V_k1)
        // every column of a bf16 tile holds the token: column r finishes row 4 g + r mod 4
        float v = y[0];
        int e = 16 * t + ne0;
        if constexpr (NE == 4) {
          v = (rr & 2) ? ((rr & 1) ? y[3] : y[2]) : ((rr & 1) ? y[1] : y[0]);
          e += rr & 3;
        }
        st(&es[0], e, tanhf(v + hvec[2 * D + e - 3 * D]));
      } else if (tk == 0) {
        Tile::store(&es[16 * t + ne0], y);
      }
    }
    lds_barrier();
    phase();
    // ---- mixture and type logits --------------------------------------------
#pragma unroll
    for (int i = 0; i < TPH; ++i) {
      const int t = wave + NW * i;
      if (t >= 3 * Mt + Kt) break;
      const int c = min(t / Mt, 3);
      float y[NE];
      Tile::template mul<KD>(wh[i], [&](int, int s) -> frag { return *(const frag *)&es[c * D + k_of(s)]; }, 1, lane, y);
      if (tk == 0) {
        const int r0 = 16 * (c < 3 ? t % Mt : t - 3 * Mt) + ne0, cnt = c < 3 ? M : K, o0 = c < 3 ? c * M : 3 * M;
#pragma unroll
        for (int q = 0; q < NE; ++q)
          if (r0 + q < cnt) hv[o0 + r0 + q] = y[q] + head_b[o0 + r0 + q];
      }
    }
    lds_barrier();
    phase();
    // ---- the draw -------------------------------------------------------------
    const size_t di = (size_t)b * a.MG + (l - 1);
    // lane's logit -> the log of the softmax's denominator (in lse) and the
    // first index whose running sum exceeds u times the total
    auto draw = [&](float lp, int cnt, float u, float &lse) {
      const float mx = lanes_max(lp);
      const float c = wave_cumsum(lane < cnt ? expf(lp - mx) : 0.f);
      const float tot = lane_val(c, cnt - 1);
      const unsigned long long hit = __ballot(lane < cnt && u * tot < c);
      lse = mx + logf(tot);
      return hit ? (int)__builtin_ctzll(hit) : cnt - 1;
    };
    if (wave == 0 || wave == 2) {
      // component and interval (both waves); wave 0 goes on to the next
      // token's time encoding, wave 2 to the record
      const float lw = lane < M ? hv[lane] : -INFINITY;
      const float mu_l = lane < M ? hv[M + lane] : 0.f, s_l = lane < M ? hv[2 * M + lane] : 0.f;
      float lse;
      const int z = draw(lw, M, pu[l - 1][0], lse);
      const float nlw = lw - lse;
      const float tau = expf(lane_val(mu_l, z) + expf(lane_val(s_l, z)) * pu[l - 1][1]);
      const float t_new = t_last + tau;
      t_last = t_new;
      if (wave == 0) {
        if (lane < D) {
          float zsin, zcos;
          sincosf(t_new * freq[lane], &zsin, &zcos);
          zs[0][lane] = (lane & 1) ? zcos : zsin;
        }
        if (lane == 0) {
          a.d_tau[di] = tau;
          a.d_t[di] = t_new;
          if (!isfinite(tau)) atomicOr(a.status, TPPSD_STATUS_NONFINITE);
        }
      } else {
        if (lane < M) {
          a.d_mix[di * 3 * M + lane] = nlw;
          a.d_mix[di * 3 * M + M + lane] = mu_l;
          a.d_mix[di * 3 * M + 2 * M + lane] = s_l;
        }
        // log g of the drawn interval under the draft mixture
        const float lt = logf(tau);
        float c = -INFINITY;
        if (lane < M) {
          const float zz = lt - mu_l;
          c = nlw - s_l - 0.918938533204672742f - lt - 0.5f * zz * zz * expf(-2.f * s_l);
        }
        const float cm = lanes_max(c);
        const float lg = cm + logf(lanes_sum<64>(lane < M ? expf(c - cm) : 0.f));
        if (lane == 0) a.d_logg[di] = lg;
      }
    } else if (wave == 1) {
      const float lk = lane < K ? hv[3 * M + lane] : -INFINITY;
      float lse;
      const int kk = draw(lk, K, pu[l - 1][2], lse);
      const float nlk = lk - lse;
      if (lane < K) a.d_logtype[di * K + lane] = nlk;
      if (lane == 0) {
        a.d_k[di] = kk;
        a.d_logf[di] = lane_val(nlk, kk);
        tok_k[0] = kk;
      }
    }
    lds_barrier();
  }
}

template <typename ELT, int D, int F, int NW>
void dg_launch(const DraftArgs &a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  if (a.L == 1)
    hipExtLaunchKernelGGL((k_draft_regs<ELT, D, F, 1, NW>), dim3(a.B), dim3(64 * NW), 0, s, ev0, ev1, 0, a);
  else
    hipExtLaunchKernelGGL((k_draft_regs<ELT, D, F, 2, NW>), dim3(a.B), dim3(64 * NW), 0, s, ev0, ev1, 0, a);
}

}  // namespace

bool regs_draft_ok(int attnhp, int bf16, int L, int d, int H, int F, int M, int K) {
  const bool width = bf16 ? (d == 32 || d == 64) : (d == 16 || d == 32);
  return L >= 1 && L <= 2 && width && d == 16 * H && (attnhp || F == 2 * d || F == 4 * d) &&
         3 * ((M + 15) / 16) + (K + 15) / 16 <= DG_HEAD_TILES && 3 * M + K <= DG_HEAD_TILES * 16;
}

void launch_draft_regs(const DraftArgs &a, int attnhp, int bf16, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const int f = attnhp ? 0 : a.F / a.d;   // 0, 2 or 4
  if (bf16 && a.d == 64) {
    if (f == 0) dg_launch<bf16_t, 64, 0, 8>(a, s, ev0, ev1);
    else if (f == 2) dg_launch<bf16_t, 64, 128, 8>(a, s, ev0, ev1);
    else dg_launch<bf16_t, 64, 256, 8>(a, s, ev0, ev1);
  } else if (bf16) {
    if (f == 0) dg_launch<bf16_t, 32, 0, 4>(a, s, ev0, ev1);
    else if (f == 2) dg_launch<bf16_t, 32, 64, 4>(a, s, ev0, ev1);
    else dg_launch<bf16_t, 32, 128, 4>(a, s, ev0, ev1);
  } else if (a.d == 32) {
    if (f == 0) dg_launch<float, 32, 0, 4>(a, s, ev0, ev1);
    else if (f == 2) dg_launch<float, 32, 64, 4>(a, s, ev0, ev1);
    else dg_launch<float, 32, 128, 4>(a, s, ev0, ev1);
  } else {
    if (f == 0) dg_launch<float, 16, 0, 4>(a, s, ev0, ev1);
    else if (f == 2) dg_launch<float, 16, 32, 4>(a, s, ev0, ev1);
    else dg_launch<float, 16, 64, 4>(a, s, ev0, ev1);
  }
}

}  // namespace tppsd
