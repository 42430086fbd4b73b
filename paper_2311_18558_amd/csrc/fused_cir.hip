// The calibration step's channel part fused per link, with the targets in the
// delay domain (rtc_cfr_loss_adjoint_cir): CFR, workload loss with its
// gradient, and CFR adjoint, without the CFR itself ever being formed.
//
// The loss and its gradient are functions of each row's transform X_k =
// sum_n H[n] exp(+j 2 pi n k / N) alone (by Parseval sum |H - H*|^2 =
// sum |X - X*|^2 / N; the PDP is |X|^2 / N), and X is linear in the paths:
// with x_i = N df tau_i the path's delay in taps and the phase reference at
// the middle of the grid,
//     X_k = exp(j pi (N-1) k / N) sum_i A'[m, i] D(k - x_i),
//     D(y) = sin(pi y) / sin(pi y / N),
//     A'[m, i] = a_i g_m exp(j psi_i (m - c)) exp(-j 2 pi f_ref tau_i),
// D real (Eq. cfr_cont at the subcarriers of Sec. II-A, then the IDFT of
// Sec. II-A).  So the forward product gives X directly, the loss is
// elementwise, dL/dX is the adjoint product's operand, and no transform is
// left (two per row before: the H-domain pass measured ~154 k cycles a link
// at 1,024 subcarriers and 186 paths, 69 k of them the transforms).
//
// Nodes.  A link's delays span far fewer taps than N (42 of 1,024 on the
// scale workload), so its paths are first gathered on a grid of half taps:
// D(k - x) is band-limited in x to half the grid's rate, and the windowed
// sinc
//     D(k - x) = sum_j psi(p_j - x) D(k - p_j),   p_j = e0 + j / 2,
//     psi(t) = sinc(2 t) exp(b (sqrt(1 - (t / 5.5)^2) - 1)), |t| < 5.5, b = 17.16
// reproduces it to 6e-9 rms (2.9e-8 largest, in the unit of D's spectrum),
// below the rounding of the split products (~1e-7).  At the whole taps
// D(k - p) = N delta(k, p): those nodes only add to their own tap.  At the
// half taps D depends on k - p alone and is the same for every link: a table
// of FP16-split operand vectors, built at compile time and copied to LDS,
// serves as the matrix operand of both products with no vector work.  The
// products contract over 16 nt half taps instead of the link's paths (64
// instead of 186 on the scale workload), two real products per complex one.
// A link whose delays span more than kDlPos taps (or are not finite) takes
// the paths themselves as the contraction axis, D evaluated per (path, tap).
//
// One workgroup of eight waves owns one link; wave w owns taps N/8 w ..
// N/8 (w + 1) - 1 of a window of N taps around the link's delays, as TPW
// tiles of 32 taps x 32 elements.  The accumulators hold X transposed (lane =
// element, register = tap): the layout the adjoint takes its operand in.  The
// taps of a tile are spread over the MFMA's rows so that a lane's registers
// 8 c .. 8 c + 7 are the eight consecutive taps 16 c + 8 (lane/32) + 0..7:
// 64 contiguous bytes of X*, and directly one K-vector of the adjoint.
//
//  1. Spread: per stage of 64 paths the workgroup forms A' in LDS
//     and the paths' weights psi; the waves contract chunks of 16 paths
//     with psi, each for one node block; their sums meet in LDS, get one
//     power-of-two scale per link and are stored as FP16 parts (half
//     taps) and FP32 (whole taps).
//  2. Forward: acc = sum over half taps; the whole taps are its start value.
//  3. Loss on the accumulators, X* read once from HBM, a tile ahead.
//  4. Adjoint to the nodes: the waves' partial sums meet in LDS; the whole
//     taps' values are dL/dX itself.
//  5. Interpolation to the paths with the same psi, a wave per 32 paths;
//     path phase, array phase and gain give dL/da and dL/dg (FP64).
// Measured (MI355X, 32 elements, 205 paths a link, 1,024 subcarriers): 8,192
// links 1.50 ms, 2.36 ms before (H-domain pass with two transforms a row);
// 512 links 109 us, 178 before; 2,048 links at 256 subcarriers 269 us, 449
// before.  Clock probes, cycles a link: delays and table 5 k, spread 18 k, the
// nodes' sums 5 k, forward 9 k, loss 19 k, scale 10 k, adjoint 11 k, its scale
// 2 k, interpolation 9 k, dL/dg 8 k: latency and vector work between the
// barriers of one workgroup per CU; the matrix cores are busy a fifth of it.
// Links wider than the nodes: 4,096 links 1.65 ms, 1.36 before (those do pay).
#include <cmath>

#include "api_common.h"
#include "cfr_common.h"
#include "delay_nodes.h"
#include "dev_common.h"
#include "split_f16.h"

namespace rtc {

constexpr int kDlWaves = 8;
constexpr int kDlThreads = kDlWaves * 64;
constexpr int kDlBlocks = 8;             // node blocks of 16 positions at most
constexpr int kDlPos = 16 * kDlBlocks;   // positions (whole and half taps each)

template <int LOGN>
struct Dl {
  static constexpr int N = 1 << LOGN;
  static constexpr int TPW = N / (32 * kDlWaves);  // 32-tap tiles per wave
  static constexpr int NCH = 2 * TPW;              // 16-tap chunks per wave
  static constexpr int TV = N + 160;               // operand vectors of the D table
  static constexpr int T0 = N / 2 + 80;            // the one that starts at y = 1/2
  static constexpr int TM = 256;                   // third parts: y = -TM + 1/2 .. TM - 1/2
  // LDS: the table's three parts, the targets' factors, the gains,
  // then the region the phases share
  static constexpr int OFF_TM = TV * 32;
  static constexpr int OFF_PH = OFF_TM + 2 * TM * 16;
  static constexpr int OFF_G = OFF_PH + N * 8;
  static constexpr int OFF_RED = OFF_G + 256;
  static constexpr int OFF_R = OFF_RED + 256;
  // the region: two stages of the spread (A' in the operand layout, its
  // paths' taps, delays and weights); the waves' sums of the nodes; the nodes'
  // operand (half taps) and values (whole taps); the adjoint's partial sums
  // and, behind them, the whole taps' dL/dX; the nodes' dL/dC operand and,
  // behind it, each wave's weights of a path tile
  static constexpr int ST_X = 4 * 6 * 1024;  // four chunks of three parts, re and im
  static constexpr int ST_W = ST_X + 64 * 4;
  static constexpr int ST_BYTES = ST_W + 64 * kNodeRow * 4;
  static constexpr int R_BYTES = kDlWaves * 8192 + kDlPos * 256;
  static constexpr int R_EVEN = kDlBlocks * 4096;   // whole taps' C
  static constexpr int R_GEVEN = kDlWaves * 8192;   // whole taps' dL/dX
  static constexpr int R_TW = 2 * kDlBlocks * 4096; // path tiles' weights
  static_assert(2 * ST_BYTES <= R_BYTES && R_EVEN + kDlPos * 256 <= R_GEVEN, "regions");
  static_assert(R_TW + kDlWaves * 32 * kNodeRow * 4 <= R_BYTES, "regions");
  // at the end: every path lane's dL/dg, [wave][32 paths][32 rows x 2 + 2]
  static constexpr int DG_LD = 66;
  static constexpr int DG_BYTES = kDlWaves * 32 * DG_LD * 8;
  static constexpr int SMEM =
      (OFF_R + R_BYTES > DG_BYTES + 4096 ? OFF_R + R_BYTES : DG_BYTES + 4096);
  static_assert(SMEM <= 160 * 1024, "LDS");
};

// The half taps' operand vectors: entry s holds D'(y), D' = D 2^14 / N, at
// y = s - T0 + 1/2 + 0 .. 7, as three FP16 parts.  (X is concentrated in a few
// taps, so a rounding error there is not averaged over the row as one of H's
// is over its subcarriers, and the table's is the same for every path: with
// two parts dL/dg was up to 4x further from 64 bits where X is near X*.  The
// forward takes the third part of D, and the spread those of A' and psi; the
// reverse products act on the difference and take two.)  (sin(pi y) = +-1 there, so D' is
// (+-1) 2^14 / (N sin(pi y / N)): between 2^14 / N and 0.64 x 2^14).
template <int LOGN>
struct alignas(16) DlTable {
  unsigned short h[Dl<LOGN>::TV * 8];
  unsigned short l[Dl<LOGN>::TV * 8];
  unsigned short m[2 * Dl<LOGN>::TM * 8];
};

constexpr double dl_sin(double x) {  // Taylor, |x| <= 0.6 pi
  double t = x, s = x;
  for (int m = 2; m < 44; m += 2) {
    t *= -x * x / (double)(m * (m + 1));
    s += t;
  }
  return s;
}

template <int LOGN>
constexpr DlTable<LOGN> make_dl_table() {
  using F = Dl<LOGN>;
  constexpr double kPi = 3.14159265358979323846264338327950288;
  DlTable<LOGN> t{};
  // scalars first: value i is y = i - T0 + 1/2
  unsigned short h[F::TV + 8] = {}, l[F::TV + 8] = {}, m[F::TV + 8] = {};
  for (int i = 0; i < F::TV + 8; ++i) {
    const int k = i - F::T0;  // y = k + 1/2, D even in y
    const double y = k < 0 ? -((double)k + 0.5) : (double)k + 0.5;
    const int r = k < 0 ? -k - 1 : k;
    const double yy = y > 0.5 * F::N ? F::N - y : y;  // sin(pi y / N), y < N
    const double v = (r % 2 ? -1.0 : 1.0) * 16384.0 / ((double)F::N * dl_sin(kPi * yy / (double)F::N));
    const _Float16 hv = (_Float16)v;
    const _Float16 lv = (_Float16)(v - (double)hv);
    h[i] = __builtin_bit_cast(unsigned short, hv);
    l[i] = __builtin_bit_cast(unsigned short, lv);
    m[i] = __builtin_bit_cast(unsigned short, (_Float16)(v - (double)hv - (double)lv));
  }
  for (int s = 0; s < F::TV; ++s)
    for (int j = 0; j < 8; ++j) {
      t.h[8 * s + j] = h[s + j];
      t.l[8 * s + j] = l[s + j];
    }
  for (int s = 0; s < 2 * F::TM; ++s)
    for (int j = 0; j < 8; ++j) {
      const int i = s - F::TM + F::T0 + j;  // beyond the row: 0 (not read there)
      t.m[8 * s + j] = i >= 0 && i < F::TV + 8 ? m[i] : (unsigned short)0;
    }
  return t;
}

__device__ const DlTable<8> kDlTable8 = make_dl_table<8>();
__device__ const DlTable<9> kDlTable9 = make_dl_table<9>();
__device__ const DlTable<10> kDlTable10 = make_dl_table<10>();
template <int LOGN>
RTC_DEV const DlTable<LOGN>* dl_table() {
  if constexpr (LOGN == 8)
    return &kDlTable8;
  else if constexpr (LOGN == 9)
    return &kDlTable9;
  else
    return &kDlTable10;
}

struct DelayArgs {
  int n_links, M;
  const int64_t* link_off;
  const float2* a;
  const float* psi;
  const double* tau;
  const float2* g;
  const float2* Xt;   // targets' transforms X* c64 [L, M, N], natural tap order
  const double* Z;    // {sum |H*|^2, sum (p*)^2} over the batch
  float w_coh, w_pdp;
  double fref, cm;    // grid midpoint, (M-1)/2
  double bw;          // N df: taps per second of delay
  double* rows;       // [L][K]: two loss sums, then M complex dL/dg (K = 2 without)
  int K;
  float2* dLda;       // [P] or null
};

// without nodes: x reduced to [0, N) (D(y + N) = -D(y)), S = -(+-1) (-1)^X
// sin(pi f) 2^14 / N, so that D'(k - x) = S (-1)^k / sin(pi (k - X - f) / N)
RTC_DEV PathTap direct_tap(double x, double N) {
  const double w = floor(x / N);
  const double xr = x - w * N;
  const double X = floor(xr);
  PathTap r;
  r.X = (float)X;
  r.f = fminf(fmaxf((float)(xr - X), 1e-20f), 0.99999994f);
  float s, c;
  sincos2pi(0.5f * r.f, &s, &c);
  const bool odd = ((long long)X + (long long)w) & 1;
  r.S = (odd ? s : -s) * (float)(16384.0 / N);
  if (!(fabs(x) < 1e300)) r.S = __builtin_nanf("");  // a delay that is not finite
  return r;
}

RTC_DEV float direct_weight(float d, float f, float S, float N) {
  const float invN = 1.0f / N;
  // d = k - X in (-N, N), wrapped to half a period while it is whole
  const float k = rintf(d * invN);
  const float v = (fmaf(-k, N, d) - f) * invN, v2 = v * v;
  // sin(pi v) / v to 4e-6 |v| relative (fitted over |v| <= 1/2): D falls as
  // 1 / |v|, so its error stays below 1.3e-9 of its peak
  float p = -0.5624642f;
  p = fmaf(p, v2, 2.5452757f);
  p = fmaf(p, v2, -5.1675433f);
  p = fmaf(p, v2, 3.1415926f);
  return S * fmaf(-2.0f, fabsf(k), 1.0f) * __builtin_amdgcn_rcpf(p * v);
}

RTC_DEV Split2 ld_split(const char* hi, const char* lo, int idx) {
  Split2 s;
  s.h = __builtin_bit_cast(halfx8, reinterpret_cast<const u32x4*>(hi)[idx]);
  s.l = __builtin_bit_cast(halfx8, reinterpret_cast<const u32x4*>(lo)[idx]);
  return s;
}

// four values, FP16-split, as 4 consecutive elements (4 sub .. ) of an
// operand vector: part (high; low 64 vectors on) of lane `lane`
RTC_DEV void put_split4(unsigned* op, int lane, int sub, const float (&v)[4]) {
  const unsigned h0 = pack_f16(v[0], v[1]), h1 = pack_f16(v[2], v[3]);
  const unsigned l0 = pack_f16(sub_f16<true>(v[0], h0), sub_f16<false>(v[1], h0));
  const unsigned l1 = pack_f16(sub_f16<true>(v[2], h1), sub_f16<false>(v[3], h1));
  *reinterpret_cast<uint2*>(op + lane * 4 + 2 * sub) = make_uint2(h0, h1);
  *reinterpret_cast<uint2*>(op + (64 + lane) * 4 + 2 * sub) = make_uint2(l0, l1);
}

// Eight consecutive X* values of a row, as 16-byte loads: global loads take
// any 4-byte address, and a tensor of complex values starts at 8 bytes at
// least (a branch on the alignment moved the loads of all tiles together,
// and their registers to scratch memory).
typedef float floatx4_a8 __attribute__((ext_vector_type(4), aligned(8)));
RTC_DEV void load_run(const float2* p, float4 (&v)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const floatx4_a8 x = reinterpret_cast<const floatx4_a8*>(p)[i];
    v[i] = make_float4(x.x, x.y, x.z, x.w);
  }
}

template <int LOGN>
__global__ void __launch_bounds__(kDlThreads) cfr_delay_kernel(DelayArgs A) {
  using F = Dl<LOGN>;
  constexpr int N = F::N, NW = kDlWaves, NT = kDlThreads, TPW = F::TPW, NCH = F::NCH;
  __shared__ __align__(16) char smem[F::SMEM];
  const char* th = smem;
  const char* tl = smem + F::TV * 16;
  const char* tm = smem + F::OFF_TM;
  float2* phs = reinterpret_cast<float2*>(smem + F::OFF_PH);
  float2* gs = reinterpret_cast<float2*>(smem + F::OFF_G);
  double* red = reinterpret_cast<double*>(smem + F::OFF_RED);   // [NW][2]
  float* wmax = reinterpret_cast<float*>(smem + F::OFF_RED + 128);
  char* R = smem + F::OFF_R;

  const int tid = threadIdx.x;
  const int lane = tid & 63, half = lane >> 5, col = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t l = blockIdx.x;
  const int M = A.M;
  const int64_t off0 = A.link_off[l], off1 = A.link_off[l + 1];
  const int kw = wv * 32 * TPW;  // the wave's first tap of the window

  {  // the table and the gains (read after the barriers below)
    const float4* src = reinterpret_cast<const float4*>(dl_table<LOGN>());
    float4* dst = reinterpret_cast<float4*>(smem);
    constexpr int NW16 = 2 * F::TV + 2 * F::TM;  // 16-byte vectors
    constexpr int NV = (NW16 + NT - 1) / NT;
    float4 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = src[min(tid + i * NT, NW16 - 1)];
#pragma unroll
    for (int i = 0; i < NV; ++i) dst[min(tid + i * NT, NW16 - 1)] = v[i];
    // exp(-j pi (N-1) k / N): the targets come into the products' phase by it
    for (int k = tid; k < N; k += NT) {
      float s, c;
      sincos2pi((float)k * (0.5f / (float)N), &s, &c);
      phs[k] = (k & 1) ? make_float2(-c, -s) : make_float2(c, s);
    }
    if (tid < 32) gs[tid] = tid < M ? A.g[tid] : make_float2(0.0f, 0.0f);
  }

  // ------------------------------------------------- the link's delays, scale
  const LinkSpan sp = link_span(A.a, A.tau, A.bw, off0, off1, reinterpret_cast<int*>(red), wmax);
  const int imin = sp.imin, imax = sp.imax;
  const float2 g_row = col < M ? A.g[col] : make_float2(0.0f, 0.0f);
  const float gx = wave_max_dpp(fmaxf(fabsf(g_row.x), fabsf(g_row.y)));
  int ea = 0;
  frexpf(2.0f * sp.am * gx, &ea);  // |A'| < 2^ea
  const int sx = __builtin_amdgcn_readfirstlane(14 - min(max(ea, -100), 100));
  // node blocks, or none: the workgroup's waves agree (all saw every path)
  const int64_t n_pos = (int64_t)imax - imin + 12;
  const bool nodes = off0 < off1 && sp.bad == 0 && n_pos <= kDlPos;
  const int nt = nodes ? (int)((n_pos + 15) >> 4) : 0;
  const int e0 = nodes ? imin - kNodeReach : 0;
  // the window's first tap, a multiple of eight, the nodes in its middle
  const int ks = nodes ? (e0 + 8 * nt - N / 2) & ~7 : 0;
  const int po = e0 - ks;
  // exp(j pi (N-1) ks / N) goes into the path phases
  const double ph0 = -(double)(N - 1) * (double)ks / (2.0 * (double)N);

  // ------------------------------------------------------ 1. spread, 2. forward
  floatx16 acc[TPW][2];
  float us;  // X = us acc
  {
    // stages of 64 paths: A' in three parts (PathStage)
    PathStage st(A.a, A.psi, A.tau, A.g, M, 0, A.cm, A.fref, ph0, sx, off1);
    if (off0 < off1) st.fetch(off0);
    if (nodes) {
      // a stage of 64 paths: A' and the paths' weights (thread t: three words
      // of path t / 8); two stages alternate in LDS, one barrier each
      st.zero_words(R + F::ST_W);
      st.zero_words(R + F::ST_BYTES + F::ST_W);
      auto stage = [&](int64_t s0, int buf) {
        char* B = R + buf * F::ST_BYTES;
        st.store(s0, reinterpret_cast<unsigned*>(B));
        st.weights(s0, A.bw, e0, B + F::ST_X, B + F::ST_W);
        if (s0 + 64 < off1) st.fetch(s0 + 64);
      };
      // waves to node blocks of 16 positions: pw waves share a block, each
      // taking every pw-th chunk of 16 paths
      const int pw = nt <= 2 ? 4 : nt <= 4 ? 2 : 1;
      const int blk = wv / pw, pc0 = wv % pw;
      // node rows of a block: registers 0..7 the half taps, 8..15 the whole
      // taps of positions 8 half + 0..7
      const int pos = 16 * blk + 8 * ((col >> 2) & 1) + 4 * ((col >> 3) & 1) + (col & 3);
      floatx16 cacc[2] = {floatx16{0}, floatx16{0}};
      int buf = 0;
      for (int64_t s0 = off0; s0 < off1; s0 += 64, buf ^= 1) {
        stage(s0, buf);
        __syncthreads();
        if (blk < nt) {
          const char* B = R + buf * F::ST_BYTES;
#pragma unroll 1
          for (int c = pc0; c < 4 && s0 + 16 * c < off1; c += pw) {
            spread_chunk(B, B + F::ST_X, B + F::ST_W, c, pos, cacc);
          }
        }
      }
      // the sums of each block's waves meet in LDS: thread (q, part, lane) gets
      // registers 4 q .. 4 q + 3
      const int q = tid >> 7, part = (tid >> 6) & 1;
      float4 v[kDlBlocks];
      __syncthreads();
      if (blk < nt) {
        float4* dst = reinterpret_cast<float4*>(R) + wv * 512 + lane;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            dst[(2 * i + k) * 64] =
                make_float4(cacc[k][4 * i], cacc[k][4 * i + 1], cacc[k][4 * i + 2], cacc[k][4 * i + 3]);
      }
      __syncthreads();
#pragma unroll
      for (int t = 0; t < kDlBlocks; ++t)
        if (t < nt) {
          const float4* src = reinterpret_cast<const float4*>(R) + t * pw * 512 + tid;
          float4 s = src[0];
          for (int c = 1; c < pw; ++c) {
            const float4 o = src[c * 512];
            s = make_float4(s.x + o.x, s.y + o.y, s.z + o.z, s.w + o.w);
          }
          v[t] = s;
        }
      float mx = 0.0f;
#pragma unroll
      for (int t = 0; t < kDlBlocks; ++t)
        if (t < nt)
          mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[t].x), fabsf(v[t].y)), fmaxf(fabsf(v[t].z), fabsf(v[t].w))));
      mx = wave_max_dpp(mx);
      if (lane == 0) wmax[wv] = mx;
      __syncthreads();
      mx = wmax[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) mx = fmaxf(mx, wmax[w]);
      int ec = 14;
      if (mx > 0.0f) frexpf(mx, &ec);  // |C| < 2^ec in the accumulators' unit
      ec = __builtin_amdgcn_readfirstlane(min(max(ec, -100), 120));
      const float sc = ldexpf(1.0f, 14 - ec);
      us = ldexpf(1.0f, LOGN - 14 - (14 - ec) - 14 - sx);
      float* even = reinterpret_cast<float*>(R + F::R_EVEN);
      unsigned* opnd = reinterpret_cast<unsigned*>(R);
      const int sub = q & 1;
#pragma unroll
      for (int t = 0; t < kDlBlocks; ++t)
        if (t < nt) {
          const float o[4] = {v[t].x * sc, v[t].y * sc, v[t].z * sc, v[t].w * sc};
          if (q < 2) {
            put_split4(opnd + (t * 4 + part * 2) * 256, lane, sub, o);
          } else {
            float* e = even + (16 * t + 8 * half + 4 * sub) * 64 + part * 32 + col;
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i * 64] = o[i] * 16384.0f;
          }
        }
      __syncthreads();
      // forward: the whole taps start the accumulators of their own tap
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        acc[t][0] = acc[t][1] = floatx16{0};
        const int t0 = kw + 32 * t;
        if (t0 + 32 > po && t0 < po + 16 * nt) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int p = t0 + 16 * (r >> 3) + 8 * half + (r & 7) - po;
            const bool in = p >= 0 && p < 16 * nt;
            const float* e = even + (in ? p : 0) * 64 + col;
            acc[t][0][r] = in ? e[0] : 0.0f;
            acc[t][1][r] = in ? e[32] : 0.0f;
          }
        }
      }
      // entry of the table for (tap row, half-tap chunk): y = p + 1/2 - tap
      const int idx = po + 8 * half - kw - tile_pos(col) + F::T0;
#pragma unroll 1
      for (int c = 0; c < nt; ++c) {
        Split2 CR, CI;
        path_stage_read(opnd, c, lane, CR, CI);
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
          const int i = idx + 16 * c - 32 * t;
          const Split2 T = ld_split(th, tl, i);
          // the third part where D is not small (1/300 of its peak beyond)
          const int d = kw + 32 * t - po;
          if (d > -128 && d < 16 * nt + 96) {
            const halfx8 Tm =
                __builtin_bit_cast(halfx8, reinterpret_cast<const u32x4*>(tm)[i - F::T0 + F::TM]);
            acc[t][0] = mfma_f16(Tm, CR.h, acc[t][0]);
            acc[t][1] = mfma_f16(Tm, CI.h, acc[t][1]);
          }
          acc[t][0] = mac3(T, CR, acc[t][0]);
          acc[t][1] = mac3(T, CI, acc[t][1]);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < TPW; ++t) acc[t][0] = acc[t][1] = floatx16{0};
      us = ldexpf(1.0f, LOGN - 14 - sx);
      const float tap0 = (float)(kw + tile_pos(col));
      unsigned* opnd = reinterpret_cast<unsigned*>(R);
      float* inX = reinterpret_cast<float*>(R + F::ST_X);
      float* inF = inX + 64;
      float* inS = inF + 64;
      auto info8 = [&](const float* v, int c, float (&o)[8]) {
        const float4* q = reinterpret_cast<const float4*>(v + 16 * c + 8 * half);
        const float4 x = q[0], y = q[1];
        o[0] = x.x, o[1] = x.y, o[2] = x.z, o[3] = x.w;
        o[4] = y.x, o[5] = y.y, o[6] = y.z, o[7] = y.w;
      };
      for (int64_t s0 = off0; s0 < off1; s0 += 64) {
        __syncthreads();  // the previous stage is consumed
        st.store(s0, opnd);
        if (tid < 64) {
          const int64_t p = s0 + tid;
          PathTap pt = PathTap{0.0f, 0.25f, 0.0f};  // beyond the link: weight 0
          if (p < off1) pt = direct_tap(A.bw * A.tau[p], (double)N);
          inX[tid] = pt.X;
          inF[tid] = pt.f;
          inS[tid] = pt.S;
        }
        __syncthreads();
        if (s0 + 64 < off1) st.fetch(s0 + 64);
        const int nch = (int)min((int64_t)4, (off1 - s0 + 15) >> 4);
        for (int c = 0; c < nch; ++c) {
          const Split3 AR = read_split3(R + c * 6144, lane), AI = read_split3(R + c * 6144 + 3072, lane);
          float X[8], f[8], S[8];
          info8(inX, c, X);
          info8(inF, c, f);
          info8(inS, c, S);
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            float w[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
              w[j] = direct_weight(tap0 + (float)(32 * t) - X[j], f[j], (col & 1) ? -S[j] : S[j], (float)N);
            const Split3 W = split3(w);
            acc[t][0] = mac5(W, AR, acc[t][0]);
            acc[t][1] = mac5(W, AI, acc[t][1]);
          }
        }
      }
      __syncthreads();
    }
  }

  // ------------------------------------------------------------------ 3. loss
  const float invN = 1.0f / (float)N;
  const float gcn = (float)(2.0 * (double)A.w_coh / A.Z[0]) * invN;
  const float gp = (float)(4.0 * (double)A.w_pdp / (A.Z[1] * (double)N));
  const bool row_ok = col < M;  // lanes beyond M compute on row 0's target, weighted 0 below
  const float2* xrow = A.Xt + (l * M + (row_ok ? col : 0)) * (int64_t)N;
  float4 xs[2][4];
  auto load_chunk = [&](int t, int c) {
    load_run(xrow + ((ks + kw + 32 * t + 16 * c + 8 * half) & (N - 1)), xs[c]);
  };
  load_chunk(0, 0);
  load_chunk(0, 1);
  double sums[2] = {0.0, 0.0};
  float mx = 0.0f;
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    float ec = 0.0f, ep = 0.0f;
    const float4* ph = reinterpret_cast<const float4*>(phs + kw + 32 * t + 8 * half);
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      if (r % 4 == 0) asm volatile("" ::: "memory");
      if (r == 8 && t + 1 < TPW) load_chunk(t + 1, 0);
      const float4 x2 = xs[r >> 3][(r & 7) >> 1];
      const float4 p2 = ph[(16 * (r >> 3) + (r & 7)) / 2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float2 T = cmul(e ? make_float2(x2.z, x2.w) : make_float2(x2.x, x2.y),
                              e ? make_float2(p2.z, p2.w) : make_float2(p2.x, p2.y));
        const float2 X = make_float2(acc[t][0][r + e] * us, acc[t][1][r + e] * us);
        const float2 dx = csub(X, T);
        ec += cabs2(dx);
        const float d = (cabs2(X) - cabs2(T)) * invN;  // p - p*
        ep += d * d;
        const float w = gp * d;
        float2 G = make_float2(fmaf(w, X.x, gcn * dx.x), fmaf(w, X.y, gcn * dx.y));
        mx = fmaxf(mx, fmaxf(fabsf(G.x), fabsf(G.y)));
        // computed here, tap by tap: the compiler would otherwise move all
        // tiles' loads together and the sums to the end, and keep what they
        // take in scratch memory (one link's 3 KB a wave thrash the L2)
        asm volatile("" : "+v"(G.x), "+v"(G.y), "+v"(ec), "+v"(ep), "+v"(mx));
        acc[t][0][r + e] = G.x;
        acc[t][1][r + e] = G.y;
      }
    }
    if (t + 1 < TPW) load_chunk(t + 1, 1);
    sums[0] += (double)ec;
    sums[1] += (double)ep;
  }
  if (row_ok) {
    sums[0] *= (double)invN;  // sum |X - X*|^2 / N = sum |H - H*|^2
  } else {
    sums[0] = sums[1] = 0.0;
    mx = 0.0f;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) sums[k] = wave_sum_f64(sums[k]);
  mx = wave_max_dpp(mx);
  __syncthreads();  // wmax was read for the nodes' scale
  if (lane == 0) {
    red[2 * wv] = sums[0];
    red[2 * wv + 1] = sums[1];
    wmax[wv] = mx;
  }
  __syncthreads();
  mx = wmax[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) mx = fmaxf(mx, wmax[w]);
  double* out = A.rows + l * A.K;
  if (tid < 2) {
    double s = red[tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[2 * w + tid];
    out[tid] = s;
  }

  // --------------------------------------------------------------- 4. adjoint
  // one power-of-two scale for the link's dL/dX, its largest value below 2^14
  int sa = 0;
  if (mx > 0.0f) {
    int e = 0;
    frexpf(mx, &e);
    sa = 14 - min(max(e, -100), 100);
  }
  sa = __builtin_amdgcn_readfirstlane(sa);
  const float sca = row_ok ? ldexpf(1.0f, sa) : 0.0f;
  Split2 SR[NCH], SI[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    float sr[8], si[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sr[j] = acc[c >> 1][0][8 * (c & 1) + j] * sca;
      si[j] = acc[c >> 1][1][8 * (c & 1) + j] * sca;
    }
    SR[c] = split2(sr);
    SI[c] = split2(si);
    // packed here: the FP32 values die before the adjoint's loops
    asm volatile("" : "+v"(SR[c].h), "+v"(SR[c].l), "+v"(SI[c].h), "+v"(SI[c].l));
  }
  float* geven = reinterpret_cast<float*>(R + F::R_GEVEN);
  // dL/dX at the whole taps among the nodes, from the operand's two parts
  // (taken from the accumulators in the loss loop it made that loop spill)
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int t0 = kw + 32 * t - po;
    if (t0 > -32 && t0 < 16 * nt) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int p = t0 + 16 * (r >> 3) + 8 * half + (r & 7), c = 2 * t + (r >> 3), j = r & 7;
        if (p >= 0 && p < 16 * nt) {
          geven[p * 64 + col] = (float)SR[c].h[j] + (float)SR[c].l[j];
          geven[p * 64 + 32 + col] = (float)SI[c].h[j] + (float)SI[c].l[j];
        }
      }
    }
  }
  const int n_tiles = (int)((off1 - off0 + 31) >> 5);
  const bool want_g = A.K > 2;
  // the lane's path of a tile, loaded without a branch (zero past the link)
  auto tile_path = [&](int T, float2& ai, double& psi_cyc, double& tau) {
    const int64_t p = off0 + 32 * (int64_t)T + col;
    const bool ok = p < off1;
    const int64_t pc = ok ? p : off1 - 1;
    ai = ok ? A.a[pc] : make_float2(0.0f, 0.0f);
    psi_cyc = (double)(ok ? A.psi[pc] : 0.0f) * kInv2Pi;
    tau = ok ? A.tau[pc] : 0.0;
  };
  if (nodes) {
    const int na = (nt + 1) >> 1;  // tiles of 32 half taps
    const int q = tid >> 7, part = (tid >> 6) & 1;
    float4* parts = reinterpret_cast<float4*>(R);
    float4 vo[kDlBlocks / 2];
    // y = tap + 1/2 - (p + 1): the table is even in y
    const int idx = kw + 8 * half - po - tile_pos(col) - 1 + F::T0;
#pragma unroll
    for (int ta = 0; ta < kDlBlocks / 2; ++ta) {
      if (ta < na) {
        floatx16 gr = floatx16{0}, gi = floatx16{0};
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const Split2 T = ld_split(th, tl, idx + 16 * c - 32 * ta);
          gr = mac3(T, SR[c], gr);
          gi = mac3(T, SI[c], gi);
        }
        if (ta > 0) __syncthreads();  // the previous tile's sums are read
        float4* dst = parts + wv * 512 + lane;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          dst[(2 * i) * 64] = make_float4(gr[4 * i], gr[4 * i + 1], gr[4 * i + 2], gr[4 * i + 3]);
          dst[(2 * i + 1) * 64] = make_float4(gi[4 * i], gi[4 * i + 1], gi[4 * i + 2], gi[4 * i + 3]);
        }
        __syncthreads();
        float4 s = parts[tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          const float4 o = parts[w * 512 + tid];
          s = make_float4(s.x + o.x, s.y + o.y, s.z + o.z, s.w + o.w);
        }
        vo[ta] = s;
      }
    }
    // thread (q, part, lane): positions 16 (2 ta + q/2) + 8 half + 4 (q%2) + 0..3
    constexpr float se = 16384.0f;
    float4 ve[kDlBlocks / 2];
    float gmx = 0.0f;
#pragma unroll
    for (int ta = 0; ta < kDlBlocks / 2; ++ta)
      if (ta < na) {
        const int b = 2 * ta + (q >> 1);
        const float* e = geven + ((b < nt ? 16 * b : 0) + 8 * half + 4 * (q & 1)) * 64 + part * 32 + col;
        ve[ta] = make_float4(e[0] * se, e[64] * se, e[128] * se, e[192] * se);
        gmx = fmaxf(gmx, fmaxf(fmaxf(fabsf(vo[ta].x), fabsf(vo[ta].y)), fmaxf(fabsf(vo[ta].z), fabsf(vo[ta].w))));
        gmx = fmaxf(gmx, fmaxf(fmaxf(fabsf(ve[ta].x), fabsf(ve[ta].y)), fmaxf(fabsf(ve[ta].z), fabsf(ve[ta].w))));
      }
    gmx = wave_max_dpp(gmx);
    __syncthreads();  // the last tile's sums and the scale's wmax are read
    if (lane == 0) wmax[wv] = gmx;
    __syncthreads();
    gmx = wmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) gmx = fmaxf(gmx, wmax[w]);
    int eg = 14;
    if (gmx > 0.0f) frexpf(gmx, &eg);
    eg = __builtin_amdgcn_readfirstlane(min(max(eg, -100), 120));
    const float sg = ldexpf(1.0f, 14 - eg);
    // G = N 2^-14 (value) / (sca), its operand times sg, psi times 2^14
    const float ug = ldexpf(1.0f, LOGN - 14 - sa - (14 - eg) - 14);
    unsigned* opg = reinterpret_cast<unsigned*>(R);
#pragma unroll
    for (int ta = 0; ta < kDlBlocks / 2; ++ta)
      if (ta < na) {
        const int b = 2 * ta + (q >> 1);
        const float o[4] = {vo[ta].x * sg, vo[ta].y * sg, vo[ta].z * sg, vo[ta].w * sg};
        const float e[4] = {ve[ta].x * sg, ve[ta].y * sg, ve[ta].z * sg, ve[ta].w * sg};
        put_split4(opg + (b * 4 + part * 2) * 256, lane, q & 1, o);
        put_split4(opg + ((kDlBlocks + b) * 4 + part * 2) * 256, lane, q & 1, e);
      }
    __syncthreads();
    // ------------------------------------------------------ 5. interpolation
    double dgw[16][2];
#pragma unroll
    for (int r = 0; r < 16; ++r) dgw[r][0] = dgw[r][1] = 0.0;
    for (int T = wv; T < n_tiles; T += NW) {
      float2 ai;
      double psi_cyc, tau;
      tile_path(T, ai, psi_cyc, tau);
      const bool ok = off0 + 32 * (int64_t)T + col < off1;
      const PathTap pt = node_tap(ok ? A.bw * tau : (double)e0 + kNodeReach, (double)e0);
      floatx16 gr = floatx16{0}, gi = floatx16{0};
      interpolate_tile(reinterpret_cast<float*>(R + F::R_TW) + wv * 32 * kNodeRow, pt, opg, nt, 1,
                       kDlBlocks, gr, gi);
      const float2 cc = cconj(expm2pi_f64_acc(fma(A.fref, tau, ph0)));
      const float2 step = expm2pi_f64_acc(psi_cyc);
      float2 da = make_float2(0.0f, 0.0f), ph;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = 8 * (r >> 2) + 4 * half + (r & 3);
        if ((r & 3) == 0)
          ph = expm2pi_f64_acc(psi_cyc * ((double)m - A.cm));
        else
          ph = cmul(ph, step);
        const float2 Gph = cmul(cmul(cc, make_float2(gr[r] * ug, gi[r] * ug)), ph);
        da = cadd(da, cmulc(gs[m], Gph));
        const float2 tg = cmulc(ai, Gph);
        dgw[r][0] += (double)tg.x;
        dgw[r][1] += (double)tg.y;
      }
      da.x += __shfl_xor(da.x, 32, 64);
      da.y += __shfl_xor(da.y, 32, 64);
      if (half == 0 && ok && A.dLda) A.dLda[off0 + 32 * (int64_t)T + col] = da;
    }
    if (want_g) {
      // every lane's sums over its paths, added over lanes and waves in order
      __syncthreads();
      double* dg = reinterpret_cast<double*>(smem);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = 8 * (r >> 2) + 4 * half + (r & 3);
        *reinterpret_cast<double2*>(dg + (wv * 32 + col) * F::DG_LD + 2 * m) =
            make_double2(dgw[r][0], dgw[r][1]);
      }
      __syncthreads();
      double s = 0.0;
#pragma unroll 8
      for (int i = 0; i < 32; ++i) s += dg[(wv * 32 + i) * F::DG_LD + lane];
      double* seg = reinterpret_cast<double*>(smem + F::DG_BYTES);
      seg[tid] = s;
      __syncthreads();
      if (tid < 2 * M) {
        s = seg[tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += seg[w * 64 + tid];
        out[2 + tid] = s;
      }
    }
    return;
  }
  // without nodes: a tile of 32 paths at a time, every wave over its own taps
  const float ug = ldexpf(1.0f, LOGN - 14 - sa);
  float* parts = reinterpret_cast<float*>(R);
  float2* das = reinterpret_cast<float2*>(R + F::R_GEVEN);  // [NW][64]
  const int r0 = 4 * (wv >> 1) + 2 * (wv & 1);              // this wave's two rows (registers)
  double dgw[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  for (int T = 0; T < n_tiles; ++T) {
    float2 ai;
    double psi_cyc, tau;
    tile_path(T, ai, psi_cyc, tau);
    const PathTap pt = direct_tap(A.bw * tau, (double)N);
    const float d0 = (float)(kw + 8 * half) - pt.X;
    floatx16 gr = floatx16{0}, gi = floatx16{0};
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      float w[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        w[j] = direct_weight(d0 + (float)(16 * c + j), pt.f, (j & 1) ? -pt.S : pt.S, (float)N);
      const Split2 W = split2(w);
      gr = mac3(SR[c], W, gr);
      gi = mac3(SI[c], W, gi);
    }
    __syncthreads();  // the previous tile's sums and shares are read
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      parts[wv * 2048 + r * 64 + lane] = gr[r];
      parts[wv * 2048 + (16 + r) * 64 + lane] = gi[r];
    }
    __syncthreads();
    const float2 cc = cconj(expm2pi_f64_acc(fma(A.fref, tau, ph0)));
    float2 da = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = r0 + i, m = 8 * (r >> 2) + 4 * half + (r & 3);
      float g0 = 0.0f, g1 = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        g0 += parts[w * 2048 + r * 64 + lane];
        g1 += parts[w * 2048 + (16 + r) * 64 + lane];
      }
      const float2 ph = expm2pi_f64_acc(psi_cyc * ((double)m - A.cm));
      const float2 Gph = cmul(cmul(cc, make_float2(g0 * ug, g1 * ug)), ph);
      da = cadd(da, cmulc(gs[m], Gph));
      const float2 tg = cmulc(ai, Gph);
      dgw[i][0] += (double)tg.x;
      dgw[i][1] += (double)tg.y;
    }
    das[wv * 64 + lane] = da;
    __syncthreads();
    const int64_t p = off0 + 32 * (int64_t)T + tid;
    if (tid < 32 && p < off1 && A.dLda) {
      float2 d = cadd(das[tid], das[32 + tid]);
#pragma unroll
      for (int w = 1; w < NW; ++w) d = cadd(d, cadd(das[w * 64 + tid], das[w * 64 + 32 + tid]));
      A.dLda[p] = d;
    }
  }
  if (want_g) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = r0 + i, m = 8 * (r >> 2) + 4 * half + (r & 3);
      const double re = half_sum_f64(dgw[i][0]), im = half_sum_f64(dgw[i][1]);
      if (col == 0 && m < M) {
        out[2 + 2 * m] = re;
        out[3 + 2 * m] = im;
      }
    }
  }
}

// From the batch's sums {two loss sums, M complex dL/dg} to the outputs.
__global__ void cfr_delay_finish_kernel(const double* sums, const double* Z, float w_coh, float w_pdp,
                                        int M, double* loss, float2* dLdg) {
  const int t = threadIdx.x;
  if (t == 0) {
    const double coh = sums[0] / Z[0], pdp = sums[1] / Z[1];
    loss[0] = (double)w_coh * coh + (double)w_pdp * pdp;
    loss[1] = coh;
    loss[2] = pdp;
  }
  if (dLdg && t < M) dLdg[t] = make_float2((float)sums[2 + 2 * t], (float)sums[3 + 2 * t]);
}

}  // namespace rtc

using namespace rtc;

extern "C" rtc_status rtc_cfr_loss_adjoint_cir(const rtc_radio* radio, const rtc_paths* paths,
                                               const void* a, const float* psi, const void* g,
                                               const void* X_tgt, const double* tgt_stats,
                                               float w_coh, float w_pdp, double* loss,
                                               void* dLda, void* dLdg, void* ws,
                                               size_t ws_bytes, void* stream) {
  const char* fn = "rtc_cfr_loss_adjoint_cir";
  RTC_REQUIRE(X_tgt, RTC_ERR_INVALID_ARG, "%s: X_tgt is required", fn);
  rtc_status st;
  if ((st = check_fused(fn, radio, paths, a, psi, g, tgt_stats, loss, ws, ws_bytes)) != RTC_OK)
    return st;
  hipStream_t s = as_stream(stream);
  const int64_t L = paths->n_links;
  const int M = radio->n_elem, N = radio->n_sc;
  DelayArgs A;
  A.n_links = paths->n_links;
  A.M = M;
  A.link_off = paths->link_off;
  A.a = reinterpret_cast<const float2*>(a);
  A.psi = psi;
  A.tau = paths->tau;
  A.g = reinterpret_cast<const float2*>(g);
  A.Xt = reinterpret_cast<const float2*>(X_tgt);
  A.Z = tgt_stats;
  A.w_coh = w_coh;
  A.w_pdp = w_pdp;
  A.fref = radio->fc_hz - (double)(N / 2) * radio->df_hz + 0.5 * (double)(N - 1) * radio->df_hz;
  A.cm = 0.5 * (double)(M - 1);
  A.bw = (double)N * radio->df_hz;
  A.K = dLdg ? 2 + 2 * M : 2;
  A.dLda = reinterpret_cast<float2*>(dLda);
  // workspace: rows [L][K] | their reduction's scratch | sums [K] (doubles)
  A.rows = reinterpret_cast<double*>(ws);
  double* rtmp = A.rows + L * A.K;
  double* sums = rtmp + reduce_tmp_doubles(L, A.K);
  const dim3 grid((unsigned)L), block(kDlThreads);
  switch (N) {
    case 256:
      hipLaunchKernelGGL((cfr_delay_kernel<8>), grid, block, 0, s, A);
      break;
    case 512:
      hipLaunchKernelGGL((cfr_delay_kernel<9>), grid, block, 0, s, A);
      break;
    default:
      hipLaunchKernelGGL((cfr_delay_kernel<10>), grid, block, 0, s, A);
  }
  if ((st = check_launch(fn)) != RTC_OK) return st;
  if ((st = reduce_all(A.rows, L, A.K, rtmp, sums, s, fn)) != RTC_OK) return st;
  hipLaunchKernelGGL(cfr_delay_finish_kernel, dim3(1), dim3(64), 0, s, sums, tgt_stats, w_coh, w_pdp,
                     M, loss, reinterpret_cast<float2*>(dLdg));
  return check_launch(fn);
}
