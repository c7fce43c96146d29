// NASGabor appearance evaluator: forward, backward and fused forward+backward
// kernels for gfx950.
//
// Work mapping: each primitive owns P consecutive lanes of a wavefront. A
// view chunk of P * VPL views is split into P view slots (slot j holds views
// v0 + j + P*t, t < VPL: the direction, upstream gradient, colour and
// direction-gradient accumulators, in registers). Lobes are taken P at a time
// and lane j owns lobe lc + j: it loads that lobe (structure-of-arrays,
// coalesced across primitives) and prepares its constants once (the FP64 frame,
// normaliser and its log-derivatives). Then, P times, every lane evaluates its
// own lobe against the view slot it holds and passes the slot on to the next
// lane of the group (ds_bpermute), so each owned lobe meets every view of the
// chunk and each slot ends back in its home lane. A lobe's gradient sums never
// leave its lane and a view's sums travel with its slot: no cross-lane
// reduction per lobe, no atomics, a fixed summation order.
//
// Numerics: the view direction, the frame axes, d.x, the squared chord
// |d + z|^2 = 4 kappa (relatively accurate next to the antipode, where
// 1 + d.z would cancel), h = 1 - d.z and 1 - (d.z)^2 are FP64 (the lobes reach
// lambda (1 + a) ~ 1e6, where FP32 rounding of d.z alone moves G by ~1e-4);
// the carrier's half phase is reduced in FP64 to an exact offset, of which the
// carrier and the zeta gradient's two cancelling terms are formed in FP64 up to
// FP32 corrections, relatively accurate at the carrier's peaks and zeros; the
// envelope exponent ln(p E) is formed in FP64 (exp turns its absolute error into
// a relative error of G) and only its final exponential, the other gradient
// factors and all accumulations are FP32. The normaliser and its log-derivatives are
// formed once per lobe: in FP32 where lam >= 1/2 and lam (1 + a) >= 3/2
// (with the cancellation-prone pieces in FP64), in FP64 elsewhere.
//
// Value (Section 5.1): G = N p E c, kappa = (d.z + 1)/2,
//   tau = a (d.x)^2 / (1 - (d.z)^2), E = kappa^tau, p = exp(2 lam (E kappa - 1)),
//   c = (1 + cos(k d.x + zeta)) / 2.
// Gradients (Supplementary F): with ln kappa = L and E kappa = 1 + em1,
//   dG/dlam = 2 G em1 + G dlnN/dlam            (dp/dlam = 2 p (E kappa - 1))
//   dG/da   = G (2 lam E kappa + 1) L dtau/da + G dlnN/da
//   dG/dk   = N p E dc/dk + G dlnN/dk,  dG/dzeta = N p E dc/dzeta + G dlnN/dzeta
//   dG/dx   = s_x d,  s_x = G (2 lam E kappa + 1) L 2 a d.x/(1-(d.z)^2) + k N p E dc/dtheta
//   dG/dz   = s_z d,  s_z = G [lam (1+tau) E + tau/(2 kappa)
//                             + (2 lam E kappa + 1) L tau 2 d.z/(1-(d.z)^2)]
//                         = G [(2 lam E kappa + 1) tau Q + lam E],
//                       Q = 1/(2 kappa) + 2 d.z L/(1-(d.z)^2)  (formed in FP64)
//   dG/dd   = s_x x + s_z z.
#include <hip/hip_runtime.h>

#include "nasg_device.hpp"
#include "nasg_launch.hpp"
#include "nasg_skeleton.hpp"

namespace nasg {

// The paper's raw lobe values activated (Supplementary C): lam = e^u,
// a = e^u, k = 20 (tanh u + 1), w = tanh u, with the derivatives of k and w.
// With the frame's three cosines they are nine exponentials a lobe, over a
// third of the instructions of a lobe with one view. Exponentials that a
// division follows are carried as a fraction and the forward leaves out the
// derivatives: 270 -> 196 FP64 instructions (K = 8, 1 M x 1: forward 223 -> 202
// us, backward 301 -> 287).
// Inlined where two waves per SIMD leave the registers (backward 287 -> 273, x 2
// 318 -> 299; forward x 2 246 -> 224); at three waves, and with four views per
// lane in the backward, it would spill (202 -> 284; 374 -> 395) and is called.
struct Activated {
  double lam, a, k;
  float dk;
  float w[3], dw[3];
};
template <bool BWD>
__device__ __forceinline__ Activated activate(float4 sh, float w0, float w1, float w2, bool car) {
  Activated r;
  r.lam = exp_full(sh.x);
  r.a = exp_full(sh.y);
  r.k = 0.0;
  r.dk = 0.f;
  if (car) k_activation(sh.z, r.k, r.dk);
  const float w[3] = {w0, w1, w2};
  for (int c = 0; c < 3; ++c) {
    tanh_f32(w[c], r.w[c], r.dw[c]);
    if constexpr (!BWD) r.dw[c] = 0.f;
  }
  if constexpr (!BWD) r.dk = 0.f;
  return r;
}

template <bool BWD>
__device__ __noinline__ Activated activate_call(float4 sh, float w0, float w1, float w2, bool car) {
  return activate<BWD>(sh, w0, w1, w2, car);
}

// Waves per SIMD that a lane mapping is compiled for. A view slot takes 19
// registers. With at most two per lane the kernel fits the 168 registers of
// three waves, given that the view chunks are no loop where one holds all views
// (ONE), that c0 and the mean are read again per chunk and that two polynomial
// constants are not kept in registers. The third wave covers the dependent FP64
// chains that two leave bare, and fewer spills leave room for it (backward: K =
// 8, 3 M x 16 on (8, 2) 2069 -> 1892 us, where (4, 4) at two waves takes 2027; K
// = 16 in bfloat16, 2 M x 8 on (4, 2) 1580 -> 1398; K = 8, 1.5 M x 2 on (1, 2)
// 274 -> 240; the FP64 terms of the zeta gradient have since added 5 %). With four views per lane, or the paper's raw values (six more
// registers of activation derivatives; backward, K = 2, 1 M x 1: 98 us at three
// waves, 87 at two), the spills cost more than the wave brings; four waves of
// 128 registers spill too (forward K = 8, 1 M x 1: 139 us against 80).
constexpr int mapping_waves(int lanes, int vpl, bool bc, bool ang, bool bwd) {
  return bc || (lanes == 1 && vpl == 1 && !(ang && bwd)) ||
                 (vpl <= 2 && !(lanes == 2 && vpl == 2) && (!ang || (lanes == 8 && vpl == 1)))
             ? 3 : 2;
}

// One primitive-lane-group's work: primitive `prim` (may be >= n for tail
// lanes, which compute on a real primitive and write nothing), lane j of P.
// NOCAR: the NASG lobe (Supplementary E): no carrier (k = zeta = 0) and the
// NASG normaliser, which is exact for it.
// BC (views broadcast): the P lanes of a primitive own its lobes as usual but
// every lane holds the same VPL views, so each lane evaluates its lobes
// against all of them with no slot transfer, and the per-view colour and
// direction-gradient partials are summed over the lane group at the end (DPP);
// the forward instead adds each lobe's colour in lobe order, in every lane of
// the group, so that its bits are those of the one-lane mapping. For few views
// this spreads a primitive over P lanes (P lobes prepared and loaded at once)
// instead of one lane walking all of them.
template <int P, int VPL, bool BWD, bool BF16, bool ANG, bool NOCAR = false, bool BC = false,
          bool ONE = false, bool ONCE = false,
          bool PF = (ONE && (!BWD || P == 1 || VPL == 1)) || mapping_waves(P, VPL, false, ANG, BWD) == 2>
__device__ __forceinline__ void nasg_body(const NasgArgs& a, int64_t prim, int j,
                                          const LogEntry* ltab) {
  using S = Store<BF16>;
  const int64_t N = a.n;
  const bool valid = prim < N;
  const int64_t i = valid ? prim : N - 1;  // tail lanes compute on a real primitive, write nothing
  const int V = a.v;
  const int K = a.k;
  const int rot_addr = group_next_addr<P>();
  // (two registers each that three waves per SIMD cannot spare)
  constexpr bool kKeep = mapping_waves(P, VPL, BC, ANG, BWD) == 2;
  const double k_c3 = kKeep ? vreg_const(kLog2C3) : kLog2C3;
  const double k_c8 = kKeep ? vreg_const(kExp2C8) : kExp2C8;

  const float* bp = a.dirs != nullptr ? a.dirs : a.means;

  constexpr int kChunk = BC ? VPL : P * VPL;
  for (int v0 = 0; v0 < (ONE ? kChunk : V); v0 += kChunk) {
    // read again for every view chunk: nine registers that need not live
    // through the lobes
    const float c0v[3] = {a.c0[3 * i + 0], a.c0[3 * i + 1], a.c0[3 * i + 2]};
    const double base[3] = {bp[3 * i + 0], bp[3 * i + 1], bp[3 * i + 2]};
    // gradients of later view chunks accumulate onto the first chunk's
    const bool acc_mode = a.accumulate || v0 > 0;
    ViewSlots<VPL> sl;
    slots_setup<P, VPL, BWD, BC, ONCE>(a, i, v0, j, base, c0v, sl);

    // ---- lobes, P at a time: lane j owns lobe lc + j. The view slots travel
    // round the lane group (lane j takes over the slot of lane j + 1 after
    // every step), so after P steps every owned lobe has met every view of the
    // chunk and every slot is back in its home lane. A lobe's gradient sums
    // stay in the lane that owns it; a view's colour and direction gradient
    // travel with its slot. A lane with no lobe left (K not a multiple of P)
    // carries a zero normaliser and adds nothing.
    // Records in their storage type: widened where they are used. Widened
    // where they are loaded, a bfloat16 record is waited for there, and loading
    // it ahead covers nothing (K = 8, forward 1 M x 4: 174 -> 122 us, x 1 82 ->
    // 67; K = 16 backward x 2 341 -> 305).
    using Raw4 = typename S::Raw4;
    using Raw1 = typename S::Raw1;
    auto load_rec = [&](int lc_, Raw4& q_, Raw4& sh_, Raw1& w0_, Raw1& w1_, Raw1& w2_) {
      const int lo_ = lc_ + j < K ? lc_ + j : K - 1;
      const int64_t oi_ = static_cast<int64_t>(lo_) * N + i;
      q_ = S::template raw4<ONCE>(a.quat, oi_);
      sh_ = S::template raw4<ONCE>(a.shape, oi_);
      w0_ = S::template raw1<ONCE>(a.rgbw, (static_cast<int64_t>(lo_) * 3 + 0) * N + i);
      w1_ = S::template raw1<ONCE>(a.rgbw, (static_cast<int64_t>(lo_) * 3 + 1) * N + i);
      w2_ = S::template raw1<ONCE>(a.rgbw, (static_cast<int64_t>(lo_) * 3 + 2) * N + i);
    };
    // PF: the next lobe group's records are loaded while the current group
    // is evaluated, where the 11 registers are there (at two waves, and in the
    // forward or on one lane with a single chunk: forward K = 8, 1 M x 1 91 ->
    // 82 us, raw values K = 2, 3 M x 1, both directions 311 -> 287).
    Raw4 nq, nsh;
    Raw1 nw0, nw1, nw2;
    if constexpr (PF) load_rec(0, nq, nsh, nw0, nw1, nw2);
    for (int lc = 0; lc < K; lc += P) {
      const bool own = lc + j < K;
      if constexpr (!PF) load_rec(lc, nq, nsh, nw0, nw1, nw2);
      const float4 q = S::wide(nq), sh = S::wide(nsh);
      float w0 = S::wide(nw0), w1 = S::wide(nw1), w2 = S::wide(nw2);
      if constexpr (PF) {
        if (lc + P < K) load_rec(lc + P, nq, nsh, nw0, nw1, nw2);
      }
      double xa[3], za[3], lamd, ad, kd;
      // what the gradient write-out needs besides the sums: the frame's own
      // parameters (f) and, for the paper's raw values, the derivative of
      // each value's activation
      float f[6];
      float dlam_du = 1.f, da_du = 1.f, dk_du = 1.f, dw0 = 1.f, dw1 = 1.f, dw2 = 1.f;
      lobe_frame<ANG>(q, xa, za, f);
      if constexpr (ANG) {
        constexpr bool kInline = kKeep && (!BWD || VPL <= 2);
        const Activated act = kInline ? activate<BWD>(sh, w0, w1, w2, !NOCAR)
                                      : activate_call<BWD>(sh, w0, w1, w2, !NOCAR);
        lamd = act.lam;
        ad = act.a;
        kd = act.k;
        w0 = act.w[0];
        w1 = act.w[1];
        w2 = act.w[2];
        dw0 = act.dw[0];
        dw1 = act.dw[1];
        dw2 = act.dw[2];
        dlam_du = static_cast<float>(lamd);
        da_du = static_cast<float>(ad);
        dk_du = act.dk;
      } else {
        lamd = sh.x;
        ad = sh.y;
        kd = NOCAR ? 0.0 : static_cast<double>(sh.z);
      }
      const double xa0 = xa[0], xa1 = xa[1], xa2 = xa[2];
      const double za0 = za[0], za1 = za[1], za2 = za[2];
      const double zd = NOCAR ? 0.0 : static_cast<double>(sh.w);
      const double kh = kd * kInvTwoPi;
      const double zh = zd * kInvTwoPi;
      const LobeNorm nm = lobe_norm_any<!NOCAR>(lamd, ad, kd, zd, NOCAR ? 1 : a.norm);
      const float Nn = own ? nm.n : 0.f;
      const float kf = static_cast<float>((-2.0 / kPi) * kd);
      const float dzf = static_cast<float>(nm.dz);
      const float two_lam = static_cast<float>(2.0 * lamd);
      const double two_laml = lamd * (2.0 * kLog2e);
      const double a2 = 2.0 * ad;
      const float a_ln2 = static_cast<float>(4.0 * kLn2 * ad);
      const float xf0 = static_cast<float>(xa0), xf1 = static_cast<float>(xa1),
                  xf2 = static_cast<float>(xa2);
      const float zf0 = static_cast<float>(2.0 * za0), zf1 = static_cast<float>(2.0 * za1),
                  zf2 = static_cast<float>(2.0 * za2);   // 2 z

      // gradient sums of the owned lobe
      float acc_w0 = 0.f, acc_w1 = 0.f, acc_w2 = 0.f, acc_G = 0.f, acc_l = 0.f, acc_a = 0.f;
      float acc_k = 0.f, acc_z = 0.f;
      float ax0 = 0.f, ax1 = 0.f, ax2 = 0.f, az0 = 0.f, az1 = 0.f, az2 = 0.f;
      float Gt[BC && !BWD ? VPL : 1];   // the owned lobe's G, for the sum in lobe order

#pragma unroll 2
      for (int step = 0; step < (BC ? 1 : P); ++step) {
#pragma unroll
        for (int t = 0; t < VPL; ++t) {
          // Branch-free. A view slot beyond V carries a real direction and a zero
          // upstream gradient, so it adds nothing but its (unwritten) colour; at
          // d = -z (kappa = 0) G and every gradient are forced to 0.
          const double dxd = sl.dd[t][0] * xa0 + sl.dd[t][1] * xa1 + sl.dd[t][2] * xa2;
          // q = |d + z|^2 = 2 (1 + d.z) = 4 kappa from the chord: relatively
          // accurate next to the antipode, where 1 + d.z would cancel. Every
          // other quantity derives from q: kappa = q/4 (exact), h = 1 - d.z =
          // 2 - q/2 (exact where q >= 2, Sterbenz), so kappa and h are
          // consistent and the table log needs no correction for kappa's own
          // rounding. Next to the axis h keeps an absolute error ~2e-16;
          // nothing below is sensitive to h's relative error there (G, s_x
          // and a's gradient depend on tau only through tau ln kappa and ln
          // kappa/(1 - (d.z)^2), s_z through tau Q, all smooth in h), given that
          // both ln kappa and h come from a q below 4: rounded to 4 or above (d
          // within 2e-8 of z, where d.x is up to that and tau up to a) it would
          // take ln kappa from the bucket above, 3e-13 instead of -1e-16, and h
          // would be 0. The largest q below 4 gives ln kappa/(1 - (d.z)^2) = -1/4,
          // its limit.
          // At d = -z (q = 0) 1/(h q) is not a number, of which the two minima below
          // take their limits, and everything is multiplied by G = 0. Next to it q
          // may be any positive number and G keeps its limit N e^{-2 lam} kappa^tau:
          // tau = 2 a (d.x)^2/(h q) is held to a, its largest value (a rounding of
          // d.x would take it beyond), and 1/(h q) to 1e35 where it goes into FP32.
          const double e0 = sl.dd[t][0] + za0;
          const double e1 = sl.dd[t][1] + za1;
          const double e2 = sl.dd[t][2] + za2;
          const double qr = fma(e0, e0, fma(e1, e1, e2 * e2));
          const bool live = qr > 0.0;
          const double q = fmin(qr, 0x1.fffffffffffffp+1);
          const double hd = fma(q, -0.5, 2.0);
          // kappa = lm 2^le. The table entry is fetched first, its use comes
          // after the carrier and 1/(h q).
          const int le = __builtin_amdgcn_frexp_exp(q) - 2;
          const double lm = __builtin_amdgcn_frexp_mant(q);
          const LogEntry lt = ltab[log_bucket(lm)];
          __builtin_amdgcn_sched_barrier(0);   // keep the table read ahead of the carrier work
          const double dend = hd * q;                // 2 (1 - (d.z)^2)
          const float dx = static_cast<float>(dxd);
          // carrier c = cos^2(theta/2), theta = k d.x + zeta; its half phase in units
          // of pi is reduced to an offset r in [-1/2, 1/2], exact in FP64, whose
          // cosine and sine have the dropped integer's sign in common, so c and
          // dc/dtheta = -sin cos stay relatively accurate at the carrier's peaks and
          // zeros alike. car, scp and cz are c, -dc/dtheta and c d ln N/d zeta +
          // dc/dzeta in units of pi^2, 2 pi and 2 pi; those factors are in Nn, kf and
          // the write-out. cz's two terms cancel where Psi is near 1 (in FP32 one lobe
          // next to a zero of its carrier put its rounding into the whole zeta
          // gradient), so their difference is taken in FP64 up to uc and us, which are
          // small where it is small: dz v - r.
          float car = 1.f, scp = 0.f, cz = 0.f;
          if constexpr (!NOCAR) {
            const double th = fma(dxd, kh, zh);
            const double r = th - rint(th);
            const double v = quarter_less_sq(r);
            const float vf = static_cast<float>(v);
            const float uc = cos_pi_u(vf);
            const double cr = fma(v, static_cast<double>(uc), v);
            car = static_cast<float>(cr * cr);
            if constexpr (BWD) {
              const float cf = fmaf(vf, uc, vf);
              const float rf = static_cast<float>(r);
              const float ru = rf * sin_pi_u(vf);
              scp = cf * (rf + ru);
              cz = cf * (static_cast<float>(fma(nm.dz, v, -r)) + fmaf(dzf * vf, uc, -ru));
            }
          }
          // envelope exponent in FP64, base 2: X log2(e) = 2 lam log2(e) (E kappa
          // - 1) + tau log2 kappa
          const double rden = rcp64(dend);           // 1 / (2 (1 - (d.z)^2))
          const double taud = a2 * fmin(dxd * dxd * rden, 0.5);
          const double Ld = log2_finish(lm, le, lt, 0.0, k_c3);
          const double Ad = taud * Ld;               // log2 E
          double Ekd, em1d;
          env_exp2(Ad + Ld, Ekd, em1d, k_c8);        // E kappa and E kappa - 1
          const float pE = exp2_neg(fma(two_laml, em1d, Ad));
          const float Npe = live ? Nn * pE : 0.f;
          const float G = Npe * car;
          if constexpr (BC && !BWD) {
            Gt[t] = G;
          } else {
            sl.col[t][0] = fmaf(w0, G, sl.col[t][0]);
            sl.col[t][1] = fmaf(w1, G, sl.col[t][1]);
            sl.col[t][2] = fmaf(w2, G, sl.col[t][2]);
          }
          if constexpr (BWD) {
            // log2 kappa/(2 (1 - (d.z)^2)); the factor 2 ln2 of ln kappa/(1 -
            // (d.z)^2) is in a_ln2 and in a's sum
            const double rdf = fmin(rden, 1e35);
            const float LR = static_cast<float>(Ld * rdf);
            // Q/2, Q = 1/(2 kappa) + 2 d.z ln kappa/(1 - (d.z)^2) = (h + 2 d.z ln
            // kappa)/(1 - (d.z)^2) in FP64: its two terms (each ~1/2) cancel next
            // to the axis, where Q -> 3h/8 (2 d.z = q - 2)
            const float Qh = static_cast<float>(fma((q - 2.0) * kLn2, Ld, hd) * rdf);
            const float tau = static_cast<float>(taud);
            const float em1 = static_cast<float>(em1d);
            const float g0 = sl.gr[t][0], g1 = sl.gr[t][1], g2 = sl.gr[t][2];
            const float gG = fmaf(g0, w0, fmaf(g1, w1, g2 * w2));
            acc_w0 = fmaf(g0, G, acc_w0);
            acc_w1 = fmaf(g1, G, acc_w1);
            acc_w2 = fmaf(g2, G, acc_w2);
            const float qG = gG * G;
            acc_G += qG;
            acc_l = fmaf(qG, em1, acc_l);
            // E kappa itself, not 1 + (E kappa - 1): near d = -z kappa is small and
            // the FP32 difference would carry its absolute error into E kappa
            const float Ek = static_cast<float>(Ekd);
            const float T2 = fmaf(two_lam, Ek, 1.f);   // 2 lam E kappa + 1
            const float gP = gG * Npe;
            const float gS = gP * scp;                 // dL/dG N p E dc/dtheta, times -pi/2
            acc_k = fmaf(gS, dx, acc_k);
            acc_z = fmaf(gP, cz, acc_z);
            // qT = dL/dG G (2 lam E kappa + 1); uu = qT LR d.x with LR as above:
            // a's sum takes uu d.x (ln kappa dtau/da = 2 ln2 LR (d.x)^2), and
            // dL/dG s_x = uu 4 a ln2 + dL/dG N p E dc/dtheta k (kf = -2 k/pi)
            const float qT = qG * T2;
            const float uu = qT * LR * dx;
            acc_a = fmaf(uu, dx, acc_a);
            const float gsx = fmaf(uu, a_ln2, gS * kf);
            const float iq = static_cast<float>(hd * rdf);    // 1/q
            // half of dL/dG s_z = dL/dG G [(2 lam E kappa + 1) tau Q + lam E],
            // lam E = 2 (2 lam E kappa)/q; the factor 2 is in zf0..2 and where
            // az is used
            const float gsz = fmaf(qT * tau, Qh, qG * (two_lam * Ek * iq));
            ax0 = fmaf(gsx, sl.df[t][0], ax0);
            ax1 = fmaf(gsx, sl.df[t][1], ax1);
            ax2 = fmaf(gsx, sl.df[t][2], ax2);
            az0 = fmaf(gsz, sl.df[t][0], az0);
            az1 = fmaf(gsz, sl.df[t][1], az1);
            az2 = fmaf(gsz, sl.df[t][2], az2);
            sl.gdir[t][0] = fmaf(gsx, xf0, fmaf(gsz, zf0, sl.gdir[t][0]));
            sl.gdir[t][1] = fmaf(gsx, xf1, fmaf(gsz, zf1, sl.gdir[t][1]));
            sl.gdir[t][2] = fmaf(gsx, xf2, fmaf(gsz, zf2, sl.gdir[t][2]));
          }
          // pass this view slot on (this lane takes the slot of lane j + 1) as
          // soon as it is done, so the transfer overlaps the next view's work
          if constexpr (P > 1 && !BC) {
            slot_pass<P, VPL, BWD>(sl, t, rot_addr);
          }
        }
      }

      if constexpr (BC && !BWD) {
#pragma unroll
        for (int m = 0; m < P; ++m) {
          if (lc + m >= K) continue;  // uniform
          const float m0 = __shfl(w0, m, P), m1 = __shfl(w1, m, P), m2 = __shfl(w2, m, P);
#pragma unroll
          for (int t = 0; t < VPL; ++t) {
            const float Gm = __shfl(Gt[t], m, P);
            sl.col[t][0] = fmaf(m0, Gm, sl.col[t][0]);
            sl.col[t][1] = fmaf(m1, Gm, sl.col[t][1]);
            sl.col[t][2] = fmaf(m2, Gm, sl.col[t][2]);
          }
        }
      }

      // the owning lane writes its lobe's gradients, as streaming data in the
      // ONCE flavour (each written once: acc_mode is false there)
      if constexpr (BWD) {
        if (valid && own) {
          const int64_t li = static_cast<int64_t>(lc + j) * N + i;
          if (a.g_shape != nullptr) {
            put4<ONCE>(a.g_shape, li,
                       make_float4(fmaf(nm.dl, acc_G, 2.f * acc_l) * dlam_du,
                                   fmaf(nm.da, acc_G, static_cast<float>(2.0 * kLn2) * acc_a) * da_du,
                                   fmaf(nm.dk, acc_G, static_cast<float>(-2.0 / kPi) * acc_k) * dk_du,
                                   static_cast<float>(2.0 / kPi) * acc_z),
                       acc_mode);
          }
          if (a.g_quat != nullptr) {
            const float xf[3] = {xf0, xf1, xf2}, zf[3] = {0.5f * zf0, 0.5f * zf1, 0.5f * zf2};
            const float gx[3] = {ax0, ax1, ax2}, gz[3] = {2.f * az0, 2.f * az1, 2.f * az2};
            put4<ONCE>(a.g_quat, li, frame_grad<ANG>(f, xf, zf, gx, gz), acc_mode);
          }
          if (a.g_rgbw != nullptr)
            put_rgbw<ONCE>(a.g_rgbw, lc + j, N, i, acc_w0 * dw0, acc_w1 * dw1,
                                   acc_w2 * dw2, acc_mode);
        }
      }
    }

    slots_finish<P, VPL, BWD, BC, ONCE>(a, i, valid, v0, j, acc_mode, sl);
  }
}

template <int P, int VPL, bool BWD, bool BF16, bool ANG, bool NOCAR, bool BC, bool ONE, bool ONCE>
// ONE: one chunk holds all views. ONCE (one lane per primitive, one chunk only):
// and nothing accumulates onto earlier results, so the lobe records are read and
// every output is written exactly once, all as streaming data.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    mapping_waves(P, VPL, BC, ANG, BWD))))
void nasg_kernel(const NasgArgs a) {
  static_assert(!ONCE || (P == 1 && ONE), "the streaming flavour: one lane per primitive, one chunk");
  __shared__ LogEntry ltab[kLogEntries];
  load_log_table(ltab);
  const int64_t gt = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  nasg_body<P, VPL, BWD, BF16, ANG, NOCAR, BC, ONE, ONCE>(a, gt / P,
                                                          static_cast<int>(gt & (P - 1)), ltab);
}

// ------------------------------------------------------- persistent batch

template <int P, int VPL, bool ANG>
__device__ __forceinline__ void batch_tile(const NasgArgs& a, int64_t start, int iters,
                                           const LogEntry* ltab) {
  constexpr int kPrimsPerPass = 256 / P;
  for (int m = 0; m < iters; ++m) {
    const int64_t base = start + static_cast<int64_t>(m) * kPrimsPerPass;
    if (base >= a.n) break;  // uniform across the block
    // Records ahead with up to two views per lane, which leave the registers at two
    // waves (24 scenes of 1e4 to 1e6 primitives 2719 -> 2640 us, K = 8, 24 of 60 000
    // x 1 294 -> 274); with four 30 registers spill (x 4 421 -> 474).
    nasg_body<P, VPL, true, false, ANG, false, false, false, false, VPL <= 2>(
        a, base + threadIdx.x / P, static_cast<int>(threadIdx.x & (P - 1)), ltab);
  }
}

__global__ void batch_reset(uint32_t* counter) { *counter = 0u; }

// Loads a record that every lane of the wave reads at the same address and
// pins each 32-bit word to a scalar register. Without it the compiler sees an
// index that came through LDS as divergent and keeps the scene's pointers and
// sizes in vector registers, with vector address arithmetic on every access.
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "record size must be a multiple of 4 bytes");
  constexpr int kWords = sizeof(T) / 4;
  uint32_t w[kWords];
  __builtin_memcpy(w, p, sizeof(T));
#pragma unroll
  for (int i = 0; i < kWords; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  T out;
  __builtin_memcpy(&out, w, sizeof(T));
  return out;
}

// Pulls tiles from the queue until it is empty; every block exits when the
// head passes n_items. A plan whose token does not match is not run.
// Two waves per SIMD: the inlined lane mappings would otherwise need more
// registers than that occupancy allows (a second kernel and queue at three
// waves for the mappings that fit them alone spills 36 registers here, where
// the scene's record is in scalar ones, and adds a tail: 32 large scenes 5.7 ->
// 6.1 ms). RAW: the plan has scenes with the paper's raw values, so the lane
// mappings are inlined for both parametrisations; without them only the
// quaternion mappings are, and an item of a raw-value scene, which such a plan
// never holds, is skipped.
template <bool RAW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void nasg_batched_kernel(const BatchHeader* hdr, const BatchScene* scenes, const BatchItem* items,
                         uint32_t* counter, uint64_t token) {
  __shared__ int s_item;
  __shared__ LogEntry ltab[kLogEntries];
  if (hdr->token != token) return;
  load_log_table(ltab);
  const int n_items = hdr->n_items;
  for (;;) {
    if (threadIdx.x == 0) s_item = static_cast<int>(atomicAdd(counter, 1u));
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
    if (it >= n_items) break;
    const BatchItem item = load_uniform(items + it);
    const BatchScene sc = load_uniform(scenes + item.scene);
    switch (sc.variant) {
      case 0: batch_tile<1, 1, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      case 1: batch_tile<1, 2, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      case 2: batch_tile<1, 4, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      case 3: batch_tile<4, 2, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      case 4: batch_tile<4, 4, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      case 5: batch_tile<8, 2, false>(sc.args, item.start, sc.tile_iters, ltab); break;
      default:
        if constexpr (RAW) {
          switch (sc.variant) {
            case 6: batch_tile<1, 1, true>(sc.args, item.start, sc.tile_iters, ltab); break;
            case 7: batch_tile<1, 2, true>(sc.args, item.start, sc.tile_iters, ltab); break;
            case 8: batch_tile<1, 4, true>(sc.args, item.start, sc.tile_iters, ltab); break;
            case 9: batch_tile<4, 2, true>(sc.args, item.start, sc.tile_iters, ltab); break;
            case 10: batch_tile<4, 4, true>(sc.args, item.start, sc.tile_iters, ltab); break;
            default: batch_tile<8, 2, true>(sc.args, item.start, sc.tile_iters, ltab); break;
          }
        }
        break;
    }
  }
}

hipError_t launch_batched(const BatchHeader* hdr, const BatchScene* scenes, const BatchItem* items,
                          uint32_t* counter, uint64_t token, int grid, bool raw, hipStream_t s) {
  hipLaunchKernelGGL(batch_reset, dim3(1), dim3(1), 0, s, counter);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (raw) {
    hipLaunchKernelGGL(nasg_batched_kernel<true>, dim3(grid), dim3(256), 0, s, hdr, scenes, items,
                       counter, token);
  } else {
    hipLaunchKernelGGL(nasg_batched_kernel<false>, dim3(grid), dim3(256), 0, s, hdr, scenes, items,
                       counter, token);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------ instantiation

template <int P, int VPL, bool BWD, bool BF16, bool ANG, bool NOCAR, bool BC>
static hipError_t launch_one(const NasgArgs& a, int block, hipStream_t s) {
  const int64_t threads = a.n * P;
  const int64_t grid = (threads + block - 1) / block;
  // The streaming flavour (ONCE): one lane per primitive, so that a wave's
  // accesses cover whole cache lines, and a launch that reads every record
  // and writes every output once: all views in one chunk and no accumulation
  // onto earlier results (so acc_mode is always false in it).
  const bool one = a.v <= (BC ? VPL : P * VPL);
  const dim3 g(static_cast<unsigned>(grid)), b(block);
  if (one && P == 1 && !a.accumulate) {
    hipLaunchKernelGGL((nasg_kernel<P, VPL, BWD, BF16, ANG, NOCAR, BC, true, P == 1>), g, b, 0, s, a);
  } else if (one) {
    hipLaunchKernelGGL((nasg_kernel<P, VPL, BWD, BF16, ANG, NOCAR, BC, true, false>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((nasg_kernel<P, VPL, BWD, BF16, ANG, NOCAR, BC, false, false>), g, b, 0, s, a);
  }
  return hipGetLastError();
}

template <int P, int VPL, bool ANG, bool NOCAR, bool BC>
static hipError_t launch_pa(const NasgArgs& a, bool bwd, bool bf16, int block, hipStream_t s) {
  if (bwd) return bf16 ? launch_one<P, VPL, true, true, ANG, NOCAR, BC>(a, block, s)
                       : launch_one<P, VPL, true, false, ANG, NOCAR, BC>(a, block, s);
  return bf16 ? launch_one<P, VPL, false, true, ANG, NOCAR, BC>(a, block, s)
              : launch_one<P, VPL, false, false, ANG, NOCAR, BC>(a, block, s);
}

template <int P, int VPL, bool NOCAR, bool BC = false>
static hipError_t launch_pv(const NasgArgs& a, bool bwd, bool bf16, int block, hipStream_t s) {
  return a.param == kParamAngles ? launch_pa<P, VPL, true, NOCAR, BC>(a, bwd, bf16, block, s)
                                 : launch_pa<P, VPL, false, NOCAR, BC>(a, bwd, bf16, block, s);
}

hipError_t launch_nasg(const NasgArgs& a, int lanes, int vpl, bool bcast, bool bwd, bool bf16,
                       int block, hipStream_t s) {
  if (a.family == kFamNasg) {
    // NASG lobes: the compiled family mappings
    int fl, fv;
    family_mapping(bwd, a.n, a.k, a.v, fl, fv);
    switch (fl) {
      case 1: return launch_pv<1, 1, true>(a, bwd, bf16, block, s);
      case 2: return launch_pv<2, 2, true>(a, bwd, bf16, block, s);
      case 4: return launch_pv<4, 2, true>(a, bwd, bf16, block, s);
      default: return launch_pv<8, 2, true>(a, bwd, bf16, block, s);
    }
  }
  if (a.family != kFamNasgabor) return launch_family(a, bwd, bf16, block, s);
  if (bcast) {
#define NASG_BC_CASE(P_, V_) \
    if (lanes == P_ && vpl == V_) return launch_pv<P_, V_, false, true>(a, bwd, bf16, block, s);
    NASG_FOR_EACH_BCAST_CONFIG(NASG_BC_CASE)
#undef NASG_BC_CASE
    return hipErrorInvalidValue;
  }
#define NASG_CASE(P_, V_) \
  if (lanes == P_ && vpl == V_) return launch_pv<P_, V_, false>(a, bwd, bf16, block, s);
  NASG_FOR_EACH_CONFIG(NASG_CASE)
#undef NASG_CASE
  return hipErrorInvalidValue;
}

}  // namespace nasg
