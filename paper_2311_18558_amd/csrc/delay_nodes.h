// Gathering a link's paths on a grid of half taps of the delay axis, and
// interpolating from it (fused_cir.hip, the long-link kernels of cfr.hip).
//
// With x = N df tau a path's delay in taps, its contribution to anything
// band-limited to the grid's N subcarriers about their midpoint -- the
// subcarriers' exponentials exp(-j 2 pi n' x / N), |n'| <= (N-1)/2, and their
// transforms -- is, in x, band-limited to half the rate of half taps, so
//     f(x) = sum_j psi(p_j - x) f(p_j),   p_j = e0 + j / 2,
//     psi(t) = sinc(2 t) exp(b (sqrt(1 - (t / 5.5)^2) - 1)), |t| < 5.5, b = 17.16,
// to 6e-9 rms and 2.9e-8 at most (the window and b minimise it at 22 nodes;
// measured over 300 delays).  A kernel contracts over the link's nodes, a few
// per tap its delays span, instead of its paths.
#pragma once

#include <type_traits>

#include "cfr_common.h"
#include "dev_common.h"
#include "split_f16.h"

namespace rtc {

constexpr int kNodeReach = 5;              // positions before a path's tap that psi reaches
// a path's weights in LDS: half taps at words 1..12
// (positions X - 5 .. X + 6), whole taps at 15..26, zeros at 0, 13, 14, 27;
// an odd row length spreads the lanes over the banks
constexpr int kNodeRow = 29;

// exp(-j 2 pi x) for an FP64 phase in cycles, to ~4e-8 (expm2pi_f64_hw's
// 1.3e-7 and the rounding of its reduced phase would be the largest errors
// here): reduced to an eighth of a turn in FP64, then polynomials.
RTC_DEV float2 expm2pi_f64_acc(double x) {
  const double fr = __builtin_amdgcn_fract(x);
  const double q = rint(4.0 * fr);
  const float r = (float)fma(q, -0.25, fr);
  float s, c;
  sincos2pi(r, &s, &c);  // |r| <= 1/8: no further reduction
  const int qi = (int)q;
  const float cs = (qi & 1) ? -s : c, sn = (qi & 1) ? c : s;
  return (qi & 2) ? make_float2(-cs, sn) : make_float2(cs, -sn);
}

// A path's place on the tap axis: whole tap X (relative to an origin), the
// rest f in (0, 1) -- kept off 0, 1/2 and 1, where psi and D are 0/0 (the
// shift is below f's own rounding) -- and sin(2 pi f) / (2 pi) or, without
// nodes, the path's factor of D, both times the operand's 2^14.
struct PathTap {
  float X, f, S;
};

// x = W tau relative to the nodes' first position e0
RTC_DEV PathTap node_tap(double x, double e0) {
  const double X = floor(x);
  PathTap r;
  r.X = (float)(X - e0);
  r.f = fminf(fmaxf((float)(x - X), 1e-20f), 0.99999994f);
  if (r.f == 0.5f) r.f = 0.50000006f;
  float s, c;
  sincos2pi(r.f, &s, &c);
  r.S = s * (16384.0f * 0.15915494309189535f);
  return r;
}

// Word w (1..12 half taps, 15..26 whole taps) of a path's weights: psi at
// t = position - x (taps) times 2^14, sin(2 pi t) = +-sin(2 pi f); b (sqrt(s)
// - 1) is written without cancellation.
RTC_DEV float node_weight(int w, const PathTap& pt) {
  const bool odd = w < 14;
  const float t = (float)(odd ? w - 6 : w - 20) + ((odd ? 0.5f : 0.0f) - pt.f);
  const float u = t * t * (1.0f / 30.25f);
  const float s = 1.0f - u;
  constexpr float b = 17.16f * 1.4426950408889634f;
  const float e = __builtin_amdgcn_exp2f(
      -b * u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_sqrtf(fmaxf(s, 0.0f))));
  float r = __builtin_amdgcn_rcpf(t);
  r = fmaf(fmaf(-t, r, 1.0f), r, r);
  return s > 0.0f ? (odd ? pt.S : -pt.S) * r * e : 0.0f;
}

// A lane's eight operand values from the weights: psi of eight paths at the
// lane's node, or of eight nodes for the lane's path.  at[j]: byte address,
// already clamped to the row.
RTC_DEV void node_values(const char* base, const int (&at)[8], float (&w)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = *reinterpret_cast<const float*>(base + at[j]);
}

// x in three FP16 parts (the third what the first two leave)
struct Split3 {
  Split2 s;
  halfx8 m;
};
RTC_DEV Split3 split3(const float (&x)[8]) {
  u32x4 H, L, Q;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = x[2 * j], b = x[2 * j + 1];
    H[j] = pack_f16(a, b);
    const float ra = sub_f16<true>(a, H[j]), rb = sub_f16<false>(b, H[j]);
    L[j] = pack_f16(ra, rb);
    Q[j] = pack_f16(sub_f16<true>(ra, L[j]), sub_f16<false>(rb, L[j]));
  }
  Split3 r;
  r.s.h = __builtin_bit_cast(halfx8, H);
  r.s.l = __builtin_bit_cast(halfx8, L);
  r.m = __builtin_bit_cast(halfx8, Q);
  return r;
}
RTC_DEV floatx16 mac5(const Split3& a, const Split3& b, floatx16 c) {
  c = mfma_f16(a.m, b.s.h, c);
  c = mfma_f16(a.s.h, b.m, c);
  return mac3(a.s, b.s, c);
}
// three parts of a chunk's operand (re, or im 3 x 1 KB on) of lane `lane`
RTC_DEV Split3 read_split3(const char* op, int lane) {
  const u32x4* o = reinterpret_cast<const u32x4*>(op) + lane;
  Split3 r;
  r.s.h = __builtin_bit_cast(halfx8, o[0]);
  r.s.l = __builtin_bit_cast(halfx8, o[64]);
  r.m = __builtin_bit_cast(halfx8, o[128]);
  return r;
}

RTC_DEV int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

// MFMA row (0..31) -> position within a 32-row tile whose lane registers
// 8 c .. 8 c + 7 are to be eight consecutive positions: register 4 q + i of
// lane half h is row 8 q + 4 h + i, and position 16 (q / 2) + 8 h + 4 (q % 2) + i
RTC_DEV int tile_pos(int row) {
  return 16 * (row >> 4) + 8 * ((row >> 2) & 1) + 4 * ((row >> 3) & 1) + (row & 3);
}

// Wave-wide maxima by DPP (the LDS crossbar's shuffles take several hundred
// cycles for the six steps), the same value on every lane.
template <typename T, typename F>
RTC_DEV T wave_red_dpp(T v, F op) {
  auto mv = [](T x, auto ctrl) {
    const int b = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(b, b, decltype(ctrl)::value, 0xf, 0xf, false));
  };
  v = op(v, mv(v, std::integral_constant<int, 0x111>()));  // row_shr 1, 2, 4, 8
  v = op(v, mv(v, std::integral_constant<int, 0x112>()));
  v = op(v, mv(v, std::integral_constant<int, 0x114>()));
  v = op(v, mv(v, std::integral_constant<int, 0x118>()));
  v = op(v, mv(v, std::integral_constant<int, 0x142>()));  // row_bcast 15, 31
  v = op(v, mv(v, std::integral_constant<int, 0x143>()));
  return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
RTC_DEV float wave_max_dpp(float v) {
  return wave_red_dpp(v, [](float a, float b) { return fmaxf(a, b); });
}
RTC_DEV int wave_max_dpp(int v) {
  return wave_red_dpp(v, [](int a, int b) { return max(a, b); });
}

// The span of a link's delays in whole taps and its largest |Re|, |Im| of a;
// bad: a delay that is not finite (or beyond 1e9 taps).  Called by every
// thread of an eight-wave workgroup; the same on all of them.  U: loads in
// flight per thread.
struct LinkSpan {
  int imin, imax, bad;
  float am;
};
template <int U = 1>
RTC_DEV LinkSpan link_span(const float2* a, const double* tau, double bw, int64_t off0, int64_t off1,
                           int* ired, float* wmax) {
  const int tid = threadIdx.x, wv = tid >> 6;
  LinkSpan s{0x7fffffff, -0x7fffffff, 0, 0.0f};
  for (int64_t p = off0 + tid; p < off1; p += 512 * U) {
    float2 v[U];
    double x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int64_t q = k ? min(p + 512 * k, off1 - 1) : p;
      v[k] = a[q];
      x[k] = bw * tau[q];
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      s.am = fmaxf(s.am, fmaxf(fabsf(v[k].x), fabsf(v[k].y)));
      s.bad |= !(fabs(x[k]) < 1e9);
      const int i = (int)floor(fmin(fmax(x[k], -2e9), 2e9));
      s.imin = min(s.imin, i);
      s.imax = max(s.imax, i);
    }
  }
  s.am = wave_max_dpp(s.am);
  s.imin = -wave_max_dpp(-s.imin);
  s.imax = wave_max_dpp(s.imax);
  s.bad = __ballot(s.bad) != 0;
  if ((tid & 63) == 0) {
    wmax[wv] = s.am;
    ired[3 * wv] = s.imin;
    ired[3 * wv + 1] = s.imax;
    ired[3 * wv + 2] = s.bad;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    s.am = fmaxf(s.am, wmax[w]);
    s.imin = min(s.imin, ired[3 * w]);
    s.imax = max(s.imax, ired[3 * w + 1]);
    s.bad |= ired[3 * w + 2];
  }
  s.imin = __builtin_amdgcn_readfirstlane(s.imin);
  s.imax = __builtin_amdgcn_readfirstlane(s.imax);
  s.bad = __builtin_amdgcn_readfirstlane(s.bad);
  return s;
}

// The path operand A'[i, m] = a_i g_m exp(j psi_i (m - c)) exp(-j 2 pi (f_ref
// tau_i + ph0)) of a stage of 64 paths, formed by an eight-wave workgroup in
// the MFMA's operand layout, three FP16 parts of re and im (6 KB per 16
// paths): thread t takes path t / 8, elements m_base + 4 (t % 8) .. + 3, one
// accurate phase and three steps; the threads of paths 2 k and 2 k + 1 (eight
// lanes apart) swap half their values, so that each stores two elements'
// pairs as one word per part.  The next stage's path loads into registers
// while the current one's products run.
struct PathStage {
  const float2* a;
  const float* psi;
  const double* tau;
  double fref, ph0, mc_cyc;
  int64_t off1;
  int wp, m0;
  float2 g4[4];
  float2 fa;
  float fpsi;
  double ftau;

  RTC_DEV PathStage(const float2* a_, const float* psi_, const double* tau_, const float2* g, int M,
                    int m_base, double cm, double fref_, double ph0_, int sx, int64_t off1_)
      : a(a_), psi(psi_), tau(tau_), fref(fref_), ph0(ph0_), off1(off1_) {
    wp = threadIdx.x >> 3;
    m0 = 4 * (threadIdx.x & 7);
    mc_cyc = ((double)(m_base + m0) - cm) * kInv2Pi;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m_base + m0 + i;
      const float2 gv = m < M ? g[m] : make_float2(0.0f, 0.0f);
      g4[i] = make_float2(ldexpf(gv.x, sx), ldexpf(gv.y, sx));
    }
    fa = make_float2(0.0f, 0.0f);
    fpsi = 0.0f;
    ftau = 0.0;
  }
  // the stage's path (the link's last one beyond it: a valid address)
  RTC_DEV void fetch(int64_t s0) {
    const int64_t p = s0 + wp < off1 ? s0 + wp : off1 - 1;
    fa = a[p];
    fpsi = psi[p];
    ftau = tau[p];
  }
  template <bool THIRD = true>
  RTC_DEV void store(int64_t s0, unsigned* opnd) const {
    const int oddp = wp & 1;
    const float2 b0 = expm2pi_f64_acc(fma(fref, ftau, fma(-(double)fpsi, mc_cyc, ph0)));
    const float2 step = expm2pi_f64_acc(-(double)fpsi * kInv2Pi);
    float2 v[4];
    float2 b = cmul(fa, b0);
    if (s0 + wp >= off1) b = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = cmul(b, g4[i]);
      if (i < 3) b = cmul(b, step);
    }
    const int c = wp >> 4, h = (wp & 15) >> 3, w32 = (wp & 7) >> 1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float2 keep = oddp ? v[2 + k] : v[k], send = oddp ? v[k] : v[2 + k];
      auto ror8 = [](float x) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, false));
      };
      const float2 got = make_float2(ror8(send.x), ror8(send.y));
      const float2 e = oddp ? got : keep, o = oddp ? keep : got;  // the even and the odd path
      unsigned* d = opnd + (c * 384 + m0 + 2 * oddp + k + 32 * h) * 4 + w32;
#pragma unroll
      for (int part = 0; part < 2; ++part) {  // re, im
        float x = part ? e.y : e.x, y = part ? o.y : o.x;
#pragma unroll
        for (int i = 0; i < (THIRD ? 3 : 2); ++i) {
          const unsigned w = pack_f16(x, y);
          d[(part * 3 + i) * 256] = w;
          x = sub_f16<true>(x, w);
          y = sub_f16<false>(y, w);
        }
      }
    }
  }
  // the rows' zero words, once (the whole workgroup)
  RTC_DEV void zero_words(char* W) const {
    if (threadIdx.x < 256) {
      const int z = threadIdx.x & 3;
      reinterpret_cast<float*>(W)[(threadIdx.x >> 2) * kNodeRow + (z == 0 ? 0 : z == 3 ? 27 : 12 + z)] = 0.0f;
    }
  }
  // the stage's weights (three words per thread) and 4 x the paths' taps,
  // relative to e0; a path beyond the link weighs nothing
  RTC_DEV void weights(int64_t s0, double bw, int e0, char* Xs, char* Ws) const {
    const int w0 = (threadIdx.x & 3) * 3 + ((threadIdx.x & 4) ? 15 : 1);
    PathTap pt = node_tap(bw * ftau, (double)e0);
    if (s0 + wp >= off1) pt.S = 0.0f;
    float* W = reinterpret_cast<float*>(Ws) + wp * kNodeRow + w0;
#pragma unroll
    for (int i = 0; i < 3; ++i) W[i] = node_weight(w0 + i, pt);
    if ((threadIdx.x & 7) == 0) reinterpret_cast<int*>(Xs)[wp] = 4 * (int)pt.X;
  }
};

// Chunk c (16 paths) of a stage onto a 16-position block of nodes: acc += psi
// A', rows = nodes (registers 0..7 the half taps, 8..15 the whole taps of
// positions 8 (lane / 32) + 0..7), columns = elements.  pos: the lane row's
// position relative to e0, 16 block + 8 ((col / 4) % 2) + 4 ((col / 8) % 2) +
// col % 4.  THIRD: with the third FP16 parts of psi and A'.
template <bool THIRD = true>
RTC_DEV void spread_chunk(const char* opnd, const char* Xs, const char* Ws, int c, int pos,
                          floatx16 (&acc)[2]) {
  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  const Split3 AR = read_split3(opnd + c * 6144, lane), AI = read_split3(opnd + c * 6144 + 3072, lane);
  const int4* X4 = reinterpret_cast<const int4*>(Xs) + 4 * c + 2 * half;
  const int4 xa = X4[0], xb = X4[1];
  const int X[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
  // byte place of the row's word for a path at X: 4 (pos - X + 6) within the
  // half taps' or the whole taps' words
  const int at0 = 4 * (pos + 6), lo = col < 16 ? 0 : 4 * 14;
  int at[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) at[j] = clampi(at0 - X[j], 0, 4 * 13) + (lo + 4 * kNodeRow * j);
  float w[8];
  node_values(Ws + (16 * c + 8 * half) * 4 * kNodeRow, at, w);
  if constexpr (THIRD) {
    const Split3 W = split3(w);
    acc[0] = mac5(W, AR, acc[0]);
    acc[1] = mac5(W, AI, acc[1]);
  } else {
    const Split2 W = split2(w);
    acc[0] = mac3(W, AR.s, acc[0]);
    acc[1] = mac3(W, AI.s, acc[1]);
  }
}

// The nodes' G (operand opg: chunk `stride` b + .. of block b's half taps, and
// `whole` further on its whole taps) interpolated to the lane's path pt of a
// 32-path tile: rows = elements, columns = paths.  W: the wave's own LDS rows
// (32 of kNodeRow words), no barrier.
RTC_DEV void interpolate_tile(float* W, const PathTap& pt, const unsigned* opg, int nt, int stride,
                              int whole, floatx16& gr, floatx16& gi) {
  const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
  W += col * kNodeRow;
  {
    const int w0 = half ? 14 : 0;  // lane (col, half): the half taps or the whole taps
    W[w0] = 0.0f;
    W[w0 + 13] = 0.0f;
#pragma unroll
    for (int i = 1; i < 13; ++i) W[w0 + i] = node_weight(w0 + i, pt);
  }
  __builtin_amdgcn_wave_barrier();
  const int at0 = 4 * (8 * half + 6 - (int)pt.X);
#pragma unroll 1
  for (int b = 0; b < nt; ++b) {
#pragma unroll
    for (int par = 0; par < 2; ++par) {
      int at[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) at[j] = clampi(at0 + 64 * b + 4 * j, 0, 4 * 13) + (par ? 0 : 4 * 14);
      float w[8];
      node_values(reinterpret_cast<const char*>(W), at, w);
      const Split2 Wv = split2(w);
      Split2 GR, GI;
      path_stage_read(opg, stride * b + (par ? 0 : whole), lane, GR, GI);
      gr = mac3(GR, Wv, gr);
      gi = mac3(GI, Wv, gi);
    }
  }
}

}  // namespace rtc
