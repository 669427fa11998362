// surrogate.hip -- multilayer-perceptron surrogate of the cloak transit:
// entry ray on the outer cylinder -> exit ray and optical path length.
//
// Network: 6 inputs -> 256 -> 256 -> 256 -> 256 -> 5 outputs, SiLU after the
// four hidden layers; inputs and targets are standardized with offsets and
// scales stored in the model. Precision by layer:
//   layer 1 (6 -> 256) and layer 5 (256 -> 5): FP32 on the vector units
//     (too thin for matrix cores; FP32 keeps the inputs' and outputs'
//     precision),
//   layers 2-4 (256 -> 256, 98% of the flops): BF16 x BF16 products with
//     FP32 accumulation on MFMA (v_mfma_f32_16x16x32_bf16).
// Training minimizes the mean squared error of the standardized targets
// with AdamW on FP32 master weights; the BF16 copies of W2..W4 are refreshed
// after every step.
//
// The surrogate is not part of the paper. The exact integrator
// (rt_transit_exact) labels its training data, judges its error, and
// replaces its prediction wherever the gate rejects it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <new>
#include <random>
#include <string>
#include <vector>

#include "../../include/rt.h"
#include "internal.h"

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace sg {

constexpr int NIN = 6, HID = 256, NOUT = 5;
// FP32 parameter vector, weights stored (fan_in, fan_out) row-major:
// W1 [6][256], b1, W2 [256][256], b2, W3, b3, W4, b4, W5 [256][5], b5 [5]
constexpr long long OFF_W1 = 0;
constexpr long long OFF_B1 = OFF_W1 + NIN * HID;
constexpr long long OFF_W2 = OFF_B1 + HID;
constexpr long long OFF_B2 = OFF_W2 + HID * HID;
constexpr long long OFF_W3 = OFF_B2 + HID;
constexpr long long OFF_B3 = OFF_W3 + HID * HID;
constexpr long long OFF_W4 = OFF_B3 + HID;
constexpr long long OFF_B4 = OFF_W4 + HID * HID;
constexpr long long OFF_W5 = OFF_B4 + HID;
constexpr long long OFF_B5 = OFF_W5 + HID * NOUT;
constexpr long long NPARAM = OFF_B5 + NOUT;  // 200,453
static_assert(OFF_B1 == OFF_W1 + NIN * HID, "W1, b1 are contiguous");
// BF16 copies of W2, W3, W4, twice in MFMA operand order (frag_index): with
// the outputs as units (forward), then with the inputs as units (backward
// through the layer); NBF per copy
constexpr long long NBF = 3LL * HID * HID;
// scaling block: in_off[6], in_scale[6], out_mean[5], out_std[5], then the loss
constexpr int S_INOFF = 0, S_INSCALE = 6, S_OMEAN = 12, S_OSTD = 17, S_LOSS = 22, NSCAL = 24;
// trust map of the side job: (axis, branch) x alpha cells x beta cells
constexpr int NCELL_A = 128, NCELL_B = 128, NCOMBO = 4;
constexpr int NCELLS = NCOMBO * NCELL_A * NCELL_B;
// trust map of the cap job: (axis, branch) x alpha x |beta| x cap-fraction
// cells, as many as the side job's
constexpr int CAP_A = 32, CAP_B = 16, CAP_U = 32;
static_assert(NCOMBO * CAP_A * CAP_B * CAP_U == NCELLS, "both jobs' trust maps have NCELLS cells");
constexpr float OUT_STD_FLOOR = 1e-3f;
constexpr float PI_F = 3.14159265358979f;

}  // namespace sg

// the library's thread-local error message (shared with the tracer)
void rt_set_error_message(const char *msg);

namespace sg {

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  rt_set_error_message(buf);
  return code;
}

// SiLU and its derivative with the hardware reciprocal (about 1 ulp): the
// activations are rounded to BF16 or feed FP32 layers whose inputs carry
// far more error than that, and an IEEE division would cost ~10
// instructions per activation. Training and inference share these; the
// derivative takes s = sigmoid(z), which its callers have.
__device__ __forceinline__ float sigmoid_f(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }
__device__ __forceinline__ float dsilu_f(float z, float s) { return s * (1.0f + z * (1.0f - s)); }

// ---------------------------------------------------------------------------
// Target encoding. Entry (phi, z, alpha, beta) on r = b, exit (phi', z',
// alpha', beta') on r = b, optical path T between them:
//   t0 = dtheta - dtheta_0,  t1 = dz - dz_0,  t2 = alpha' - alpha,
//   t3 = beta' - beta,       t4 = T - T_0,
// with dz = z' - z and dtheta the signed azimuth swept by the ray. The
// conserved angular momentum p_theta keeps its sign along the path (the
// inner mirror reflects radially), so theta is monotonic with the sign s of
// alpha, and dtheta = s * ((s (phi' - phi)) mod 2 pi) unwraps exactly for
// transits of less than a full turn. All five residuals are bounded: the
// refraction into the cloak keeps the rise and the path inside finite even
// for entries at grazing elevation, so they enter unscaled (a residual
// divided by cos(beta) would multiply the network's error by 1 / cos(beta)).
//
// (dtheta_0, dz_0, T_0) is the closed-form transit where one exists (zero
// otherwise), so that the network learns a residual:
//  - radial cloak, ordinary branch: M = kappa I (Eq. (14): eps_o = kappa),
//    a homogeneous medium of index n = sqrt(kappa) = b / (b - a); the ray is
//    straight inside, with horizontal wave number k_h = sqrt(n^2 - k_z^2)
//    and horizontal impact parameter p = b |k_theta| / k_h, and reflects
//    specularly off the metal cylinder when p <= a (Sect. 4);
//  - azimuthal cloak, extraordinary branch: M = diag(kappa, kappa s, kappa)
//    (Eq. (15)) makes the line element drho^2 + rho^2 dtheta^2 + dzeta^2 with
//    rho = sqrt(kappa) (r - a), zeta = sqrt(kappa) z: a straight line in
//    (rho, theta, zeta) at unit speed, entering at rho = b with tangential
//    speed k_theta and axial speed k_z / sqrt(kappa).
//  - radial cloak, extraordinary branch, and azimuthal cloak, ordinary
//    branch: both have m_theta = m_z = kappa s, so with p = b k_theta the
//    Hamiltonian constraint gives m_r rdot^2 = Q(r) / (kappa (r - a)^2) for
//    the quadratic Q(r) = kappa (r - a)^2 - p^2 - k_z^2 r^2, which equals
//    (b k_n)^2 at r = b; the turning point is its larger root. The sweep,
//    the rise and the optical path per unit r are
//      radial e (m_r = kappa):      p / (u sqrt Q), k_z r^2 / (u sqrt Q),
//                                   kappa u / sqrt Q            (u = r - a),
//      azimuthal o (m_r = kappa s): p / (r sqrt Q), k_z r / sqrt Q,
//                                   kappa u^2 / (r sqrt Q),
//    sums of 1 / sqrt Q, x / sqrt Q and 1 / (x sqrt Q) for Q quadratic in x,
//    integrated in closed form from the root to r = b (asinh, atan2 and
//    asinh(sqrt y) / sqrt y, the last continued through y = 0 as
//    asin(sqrt -y) / sqrt -y).
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wrap2pi(float a) {
  a = fmodf(a, 2.0f * PI_F);
  return a < 0.0f ? a + 2.0f * PI_F : a;
}

// half the azimuth swept along a chord of a circle of radius 1 with impact
// parameter u in [0, 1]: acos(u), in a form accurate near u = 1
__device__ __forceinline__ float half_sweep(float u) { return atan2f(sqrtf(fmaxf(0.f, (1.f - u) * (1.f + u))), u); }

__device__ __forceinline__ void baseline(int kind, float al, float be, float a, float b, float &dth, float &dz,
                                         float &T) {
  dth = 0.f; dz = 0.f; T = 0.f;
  const float s = al < 0.0f ? -1.0f : 1.0f;
  const float kt = fabsf(cosf(be) * sinf(al)), kz = sinf(be);
  const float n = b / (b - a), kap = n * n;
  if (kind == 0) {
    const float kh = sqrtf(kap - kz * kz);
    const float u = kt / kh;  // p / b
    float sweep = half_sweep(u), lh = b * sqrtf(fmaxf(0.f, (1.f - u) * (1.f + u)));
    const float ua = u * (b / a);  // p / a
    if (ua <= 1.0f) {
      sweep -= half_sweep(ua);
      lh -= a * sqrtf(fmaxf(0.f, (1.f - ua) * (1.f + ua)));
    }
    dth = 2.0f * s * sweep;
    dz = 2.0f * lh * kz / kh;
    T = 2.0f * lh * kap / kh;
  } else if (kind == 3) {
    const float h = sqrtf(1.0f - kz * kz / kap);
    const float u = kt / h;
    dth = 2.0f * s * half_sweep(u);
    T = 2.0f * b * sqrtf(fmaxf(0.f, (1.f - u) * (1.f + u))) / h;
    dz = T * kz / kap;
  } else {
    const float p = b * kt, A = kap - kz * kz, kza2 = kz * kz * a * a;
    const float S = sqrtf(fmaf(A, p * p, kap * kza2));  // half the root of the discriminant of Q
    const float sq = b * cosf(al) * cosf(be);           // sqrt Q(b)
    const float sA = sqrtf(A);
    const float J0 = asinhf(sA * sq / S) / sA;          // int dx / sqrt Q from the root
    if (kind == 1) {                                    // x = u: Q = A u^2 - 2 a k_z^2 u - (p^2 + k_z^2 a^2)
      const float mC = fmaf(p, p, kza2), rm = sqrtf(mC);
      const float J1 = fmaf(a * kz * kz, J0, sq) / A;   // int u du / sqrt Q
      const float Jm = atan2f(rm * sq, fmaf(a * kz * kz, b - a, mC)) / rm;  // int du / (u sqrt Q)
      dth = 2.0f * s * p * Jm;
      dz = 2.0f * kz * (J1 + 2.0f * a * J0 + a * a * Jm);
      T = 2.0f * kap * J1;
    } else {                                            // x = r: Q = A r^2 - 2 kappa a r + kappa a^2 - p^2
      const float C = fmaf(kap * a, a, -p * p);
      const float y = C * sq * sq / (b * b * S * S);
      float g;                                          // asinh(sqrt y) / sqrt y
      if (fabsf(y) < 1e-3f) g = fmaf(y, fmaf(y, 0.075f, -1.0f / 6.0f), 1.0f);
      else if (y > 0.0f) g = asinhf(sqrtf(y)) / sqrtf(y);
      else g = asinf(sqrtf(-y)) / sqrtf(-y);
      const float Jm = sq / (b * S) * g;                // int dr / (r sqrt Q)
      const float J1 = fmaf(kap * a, J0, sq) / A;       // int r dr / sqrt Q
      dth = 2.0f * s * p * Jm;
      dz = 2.0f * kz * J1;
      T = 2.0f * kap * (J1 - 2.0f * a * J0 + a * a * Jm);
    }
  }
}

__device__ __forceinline__ int kind_of(float pol, float axis) {
  return (axis == 0.0f ? 0 : 2) + (pol == 0.0f ? 0 : 1);
}

__device__ __forceinline__ bool entry_ok(float phi, float z, float al, float be, float pol, float axis) {
  return isfinite(phi) && isfinite(z) && fabsf(al) < 0.5f * PI_F && fabsf(be) < 0.5f * PI_F &&
         (pol == 0.0f || pol == 1.0f) && (axis == 0.0f || axis == 1.0f);
}

// A model's job and the geometry it needs besides an entry: RT_SUR_SIDE
// (side-to-side transits of the infinite cylinder, no geometry) or
// RT_SUR_CAP (side entries whose path meets an end cap of the cloak with
// radii a < b and material height [z0, z1]).
struct JobP {
  int job;
  float a, b, z0, z1;
};

// Fraction u of the closed-form infinite-cylinder transit's rise that the
// entry's headroom allows: h / |dz_0| with h the distance from the entry
// height to the cap the ray climbs (or sinks) towards. z is monotonic along
// a transit (p_z keeps its sign), so the path meets that cap exactly when
// u < 1. Clamped to [0, 2] (u >= 1 never meets a cap).
__device__ __forceinline__ float cap_fraction(float z, float al, float be, int kind, const JobP &jp) {
  float dth0, dz0, T0;
  baseline(kind, al, be, jp.a, jp.b, dth0, dz0, T0);
  const float h = be >= 0.0f ? jp.z1 - z : z - jp.z0;
  const float u = h / fabsf(dz0);
  return u < 2.0f ? fmaxf(u, 0.0f) : 2.0f;  // NaN (dz_0 = 0 = h) -> 2
}

// Chord model of the path up to the cap, at rise fraction u, for the cap
// job's baselines. The infinite-cylinder path is symmetric about its
// turning point, which it reaches at u = 1/2, so it is modelled by the
// straight chord through the entry with the path's impact parameter w, the
// radius traversed at fraction u being sqrt(w^2 + (b^2 - w^2)(1 - 2u)^2):
//  - radial extraordinary and azimuthal ordinary branches: w the turning
//    radius, the larger root (kappa a + S) / (kappa - k_z^2) of the
//    quadratic Q of the closed-form transit (S as there);
//  - azimuthal extraordinary branch: the path is a straight line in
//    (rho = sqrt(kappa) (r - a), theta, zeta = sqrt(kappa) z) at unit speed
//    (Eq. (15)), so the chord in rho, with w = b k_theta / sqrt(1 - k_z^2 /
//    kappa) and rho_b = b, is exact, as are the sweep fraction and the
//    optical-path fraction u;
//  - radial ordinary branch: the straight chord (its paths never leave
//    through a cap: with n = 2 it is totally reflected at every cap).
// The swept azimuth is the chord's share frac of the whole sweep, the radial
// wave number at the modelled radius r_c comes from the dispersion relation
// k_r^2 / m_r + k_theta^2 / m_theta + k_z^2 / m_z = 1 (k_theta = p_theta /
// r_c, k_z conserved; the metric of Eqs. (14)/(15): m = kappa (1, 1, 1),
// kappa (1, s, s), kappa s (1, 1, 1), kappa (1, s, 1) for the radial o, e
// and azimuthal o, e branches, s = ((r - a) / r)^2) with the sign of the leg
// (inwards before the turning point), and it is the vacuum direction's d_r
// after the cap (tangential continuity, Sect. 3), with |d_z| from
// normalization.
__device__ __forceinline__ void cap_chord(int kind, float al, float be, float u, float a, float b, float &frac,
                                          float &rc, float &dr, float &adz) {
  const float kap = (b / (b - a)) * (b / (b - a)), skap = b / (b - a);
  const float kt = fabsf(cosf(be) * sinf(al)), kz = sinf(be), p = b * kt;
  const float A = kap - kz * kz;
  float w;
  if (kind == 3) {
    w = b * kt / sqrtf(1.0f - kz * kz / kap);
  } else if (kind == 0) {
    w = p / sqrtf(A);
  } else {
    w = (kap * a + sqrtf(fmaf(A, p * p, kap * kz * kz * a * a))) / A;
  }
  w = fminf(w, b);
  const float v = 1.0f - 2.0f * u;
  const float wb = sqrtf(fmaxf(0.0f, (b - w) * (b + w)));
  const float rr = sqrtf(fmaf(wb * wb, v * v, w * w));
  rc = kind == 3 ? a + rr / skap : rr;
  const float half = atan2f(wb, w);
  frac = half > 1e-6f ? 0.5f * (1.0f - atan2f(wb * v, w) / half) : u;
  // k_r^2 vanishes at the turning point, where its terms cancel; written
  // with the factor rr - w = wb^2 v^2 / (rr + w) taken out it is v^2 times a
  // smooth positive function, so d_r = -v (...) runs linearly through it:
  //  - radial ordinary, azimuthal extraordinary (straight in r or rho):
  //    k_r^2 = (kappa - k_z^2)(rr^2 - w^2) / rr^2;
  //  - radial extraordinary, azimuthal ordinary: k_r^2 = m_r Q(r) /
  //    (kappa (r - a)^2) with Q = (kappa - k_z^2)(r - w)(r - r_s), r_s the
  //    smaller root (kappa a^2 - p^2) / ((kappa - k_z^2) w).
  if (kind == 0 || kind == 3) {
    dr = -v * wb * sqrtf(A) / rr;
  } else {
    const float rs = (kap * a * a - p * p) / (A * w);
    const float g = sqrtf(fmaxf(0.0f, A * (rc - rs) / (rc + w)));
    dr = -v * wb * g / (kind == 1 ? rc - a : rc);
  }
  const float kth = p / rc;
  adz = sqrtf(fmaxf(0.0f, 1.0f - dr * dr - kth * kth));
}

// Network input features of entry i. The transit of the infinite cylinder
// is invariant under rotation about and translation along its axis, so the
// exit offsets do not depend on phi or z; those two slots carry instead the
// entry's tangential wave numbers k_theta = cos(beta) sin(alpha) and
// k_z = sin(beta), the invariants p_theta / r2 and p_z of the transit:
//   side job: f = (k_theta, k_z, alpha, beta, branch bit, axis bit).
// A path that meets a cap depends on the height as well; the cloak is also
// symmetric under the mirror z -> z0 + z1 - z, which flips beta, so the cap
// job takes |k_z| and the cap fraction u (cap_fraction) instead:
//   cap job:  f = (k_theta, |k_z|, u, alpha, branch bit, axis bit).
__device__ __forceinline__ void features(const float *__restrict__ x6, long long ld, long long i, const JobP &jp,
                                         float f[NIN]) {
  const float al = x6[2 * ld + i], be = x6[3 * ld + i];
  f[0] = cosf(be) * sinf(al);
  f[1] = sinf(be);
  f[2] = al;
  f[3] = be;
  f[4] = x6[4 * ld + i];
  f[5] = x6[5 * ld + i];
  if (jp.job == RT_SUR_CAP) {
    f[1] = fabsf(f[1]);
    f[2] = cap_fraction(x6[ld + i], al, be, kind_of(f[4], f[5]), jp);
    f[3] = al;
  }
}

__global__ void k_fill(float *p, long long n, float v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_u32(unsigned int *p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

__device__ __forceinline__ bool is_bias(long long i) {
  return (i >= OFF_B1 && i < OFF_W2) || (i >= OFF_B2 && i < OFF_W3) || (i >= OFF_B3 && i < OFF_W4) ||
         (i >= OFF_B4 && i < OFF_W5) || i >= OFF_B5;
}

// The BF16 weights of a hidden layer are kept in the order the matrix cores
// take them: an operand fragment is 16 units x 32 consecutive k, lane (q, c16)
// holding unit c16, k = 8 q..8 q + 7, and a fragment's 64 x 16 bytes are
// contiguous, so that a wave's load of one is 8 full cache lines (as rows of
// 256 k it touched half of 16).
__host__ __device__ __forceinline__ constexpr int frag_index(int unit, int k) {
  return ((unit >> 4) * (HID / 32) + (k >> 5)) * 512 + (16 * (k >> 3 & 3) + (unit & 15)) * 8 + (k & 7);
}

// index of FP32 parameter i in the BF16 copy whose units are the layer's
// outputs (k its inputs: forward); -1: no copy. Its index in the copy with
// units and k exchanged (backward) goes to back.
__device__ __forceinline__ long long bf16_index(long long i, long long &back) {
  long long l, e;
  if (i >= OFF_W2 && i < OFF_B2) { l = 0; e = i - OFF_W2; }
  else if (i >= OFF_W3 && i < OFF_B3) { l = 1; e = i - OFF_W3; }
  else if (i >= OFF_W4 && i < OFF_B4) { l = 2; e = i - OFF_W4; }
  else return -1;
  const int in = (int)(e / HID), out = (int)(e - in * HID);
  back = NBF + l * HID * HID + frag_index(in, out);
  return l * HID * HID + frag_index(out, in);
}

// AdamW (decoupled weight decay on the weights, not the biases) on the FP32
// master weights, then the BF16 copy of each updated W2..W4 entry
__global__ void k_adamw(float *__restrict__ P, const float *__restrict__ G, float *__restrict__ m,
                        float *__restrict__ v, bf16 *__restrict__ Pb, float lr, float wd, float b1, float b2,
                        float c1, float c2, float eps) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NPARAM) return;
  const float g = G[i];
  const float mi = b1 * m[i] + (1.0f - b1) * g;
  const float vi = b2 * v[i] + (1.0f - b2) * g * g;
  m[i] = mi;
  v[i] = vi;
  float p = P[i];
  if (!is_bias(i)) p -= lr * wd * p;
  p -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  P[i] = p;
  long long kr;
  const long long k = bf16_index(i, kr);
  if (k >= 0) {
    Pb[k] = (bf16)p;
    Pb[kr] = (bf16)p;
  }
}

__global__ void k_refresh_bf16(const float *__restrict__ P, bf16 *__restrict__ Pb) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= NPARAM) return;
  long long kr;
  const long long k = bf16_index(i, kr);
  if (k >= 0) {
    Pb[k] = (bf16)P[i];
    Pb[kr] = (bf16)P[i];
  }
}

// masked first and second moments of the 6 input features and 5 targets (FP64 sums)
constexpr int NMOM = 2 * (NIN + NOUT) + 1;
__global__ void __launch_bounds__(256) k_moments(const float *__restrict__ x, const float *__restrict__ t, long long ld,
                                                 const float *__restrict__ wrow, int n, JobP jp,
                                                 double *__restrict__ acc) {
  double s[NMOM];
#pragma unroll
  for (int k = 0; k < NMOM; ++k) s[k] = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const double wr = wrow ? wrow[i] : 1.0;
    if (wr == 0.0) continue;
    s[NMOM - 1] += wr;
    float f[NIN];
    features(x, ld, i, jp, f);
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      const double v = f[k];
      s[2 * k] += wr * v;
      s[2 * k + 1] += wr * v * v;
    }
#pragma unroll
    for (int o = 0; o < NOUT; ++o) {
      const double v = t[o * ld + i];
      s[2 * (NIN + o)] += wr * v;
      s[2 * (NIN + o) + 1] += wr * v * v;
    }
  }
#pragma unroll
  for (int k = 0; k < NMOM; ++k) {
    double v = s[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(&acc[k], v);
  }
}

__global__ void k_fill_f64(double *p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// exit point and unit direction from exit parameters
__device__ __forceinline__ void exit_ray(const float *p, float b, float x[3], float d[3]) {
  float sp, cp, sa, ca, sb, cbt;
  sincosf(p[0], &sp, &cp);
  sincosf(p[2], &sa, &ca);
  sincosf(p[3], &sb, &cbt);
  x[0] = b * cp; x[1] = b * sp; x[2] = p[1];
  d[0] = cbt * (ca * cp - sa * sp);
  d[1] = cbt * (ca * sp + sa * cp);
  d[2] = sb;
}

__global__ void __launch_bounds__(256) k_encode(const float *__restrict__ x6, const float *__restrict__ y5,
                                                const int *__restrict__ status, long long ld, long long n, float a,
                                                float b, float *__restrict__ t5, float *__restrict__ wrow) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float phi = x6[i], z = x6[ld + i], al = x6[2 * ld + i], be = x6[3 * ld + i];
  const float pol = x6[4 * ld + i], axis = x6[5 * ld + i];
  float t[NOUT] = {0.f, 0.f, 0.f, 0.f, 0.f};
  bool ok = status[i] == RT_RAY_EXITED && entry_ok(phi, z, al, be, pol, axis);
  if (ok) {
    const float s = al < 0.0f ? -1.0f : 1.0f;
    const float dth = s * wrap2pi(s * (y5[i] - phi));
    float dth0, dz0, T0;
    baseline(kind_of(pol, axis), al, be, a, b, dth0, dz0, T0);
    t[0] = dth - dth0;
    t[1] = (y5[ld + i] - z) - dz0;
    t[2] = y5[2 * ld + i] - al;
    t[3] = y5[3 * ld + i] - be;
    t[4] = y5[4 * ld + i] - T0;
#pragma unroll
    for (int o = 0; o < NOUT; ++o) ok = ok && isfinite(t[o]);
  }
#pragma unroll
  for (int o = 0; o < NOUT; ++o) t5[o * ld + i] = ok ? t[o] : 0.0f;
  wrow[i] = ok ? 1.0f : 0.0f;
}

// Cap-job targets. A side entry whose path leaves through an end cap exits
// as the vacuum ray from its cap point, given where that ray crosses r = b;
// the straight vacuum leg back to the cap plane recovers the cap point
// (r_c, theta_c) and the optical path T_c up to it. The cap's refraction
// keeps the tangential wave vector (k_r, k_theta), so the vacuum direction
// there has d_theta = b k_theta / r_c (the conserved angular momentum) and
// |d_z| from normalization: the exit is fixed by (theta_c, r_c, d_r, T_c).
// With u the cap fraction (cap_fraction) and (dtheta_0, T_0) the closed-form
// transit of the infinite cylinder, whose share u the path covers before the
// cap in rise, the state (dtheta_c, r_c, d_r, T_c) and |d_z| (a second
// estimate, checked against the normalization by the gate) enter as
// residuals,
// dtheta_c the signed azimuth swept from the entry to the cap point (sign of
// alpha), each against the chord model of the path (cap_chord):
//   t0 = dtheta_c - frac dtheta_0,  t1 = r_c - r_c^chord,
//   t2 = d_r - d_r^chord,           t3 = T_c - u T_0,
//   t4 = |d_z| - |d_z|^chord.
// Rows that do not leave through the cap they head for get w = 0.
__global__ void __launch_bounds__(256) k_encode_cap(const float *__restrict__ x6, const float *__restrict__ y5,
                                                    const int *__restrict__ status, long long ld, long long n,
                                                    JobP jp, float *__restrict__ t5, float *__restrict__ wrow) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float phi = x6[i], z = x6[ld + i], al = x6[2 * ld + i], be = x6[3 * ld + i];
  const float pol = x6[4 * ld + i], axis = x6[5 * ld + i];
  float t[NOUT] = {0.f, 0.f, 0.f, 0.f, 0.f};
  const float ze = y5[ld + i];
  const bool up = be >= 0.0f;
  bool ok = status[i] == RT_RAY_EXITED && entry_ok(phi, z, al, be, pol, axis) && z >= jp.z0 && z <= jp.z1 &&
            (up ? ze > jp.z1 : ze < jp.z0);
  if (ok) {
    float ex[NOUT], xe[3], de[3];
#pragma unroll
    for (int o = 0; o < NOUT; ++o) ex[o] = y5[o * ld + i];
    exit_ray(ex, jp.b, xe, de);
    const float tb = (xe[2] - (up ? jp.z1 : jp.z0)) / de[2];  // vacuum leg back to the cap plane
    const float cx = fmaf(-tb, de[0], xe[0]), cy = fmaf(-tb, de[1], xe[1]);
    const float rc = sqrtf(fmaf(cx, cx, cy * cy));
    const float s = al < 0.0f ? -1.0f : 1.0f;
    float dth = s * wrap2pi(s * (atan2f(cy, cx) - phi));
    if (s * dth > 2.0f * PI_F - 1e-3f) dth -= s * 2.0f * PI_F;  // a sweep rounded to just below zero
    const int kind = kind_of(pol, axis);
    float dth0, dz0, T0;
    baseline(kind, al, be, jp.a, jp.b, dth0, dz0, T0);
    const float u = cap_fraction(z, al, be, kind, jp);
    float frac, rcb, drb, adzb;
    cap_chord(kind, al, be, u, jp.a, jp.b, frac, rcb, drb, adzb);
    t[0] = fmaf(-frac, dth0, dth);
    t[1] = rc - rcb;
    t[2] = fmaf(cx, de[0], cy * de[1]) / rc - drb;
    t[3] = fmaf(-u, T0, ex[4] - tb);
    t[4] = fabsf(de[2]) - adzb;
    ok = tb >= 0.0f && u < 1.0f;
#pragma unroll
    for (int o = 0; o < NOUT; ++o) ok = ok && isfinite(t[o]);
  }
#pragma unroll
  for (int o = 0; o < NOUT; ++o) t5[o * ld + i] = ok ? t[o] : 0.0f;
  wrow[i] = ok ? 1.0f : 0.0f;
}

// standardized network outputs -> exit parameters (phi', z', alpha', beta', T)
__device__ __forceinline__ void decode(const float *yrow, const float *sc, float phi, float z, float al, float be,
                                       int kind, float a, float b, float out[NOUT]) {
  float t[NOUT];
#pragma unroll
  for (int o = 0; o < NOUT; ++o) t[o] = fmaf(yrow[o], sc[S_OSTD + o], sc[S_OMEAN + o]);
  float dth0, dz0, T0;
  baseline(kind, al, be, a, b, dth0, dz0, T0);
  out[0] = wrap2pi(phi + t[0] + dth0);
  out[1] = z + (dz0 + t[1]);
  out[2] = al + t[2];
  out[3] = be + t[3];
  out[4] = T0 + t[4];
}

// Cap-job prediction -> exit parameters: the cap point and the vacuum
// direction from the targets of k_encode_cap, then the straight vacuum leg
// to r = b. Returns false where the prediction is no usable cap exit: a cap
// point within `margin` of the rims r = a, r = b of the cap, a vacuum
// direction within |d_z| < 0.05 of grazing the cap (the refraction is
// ill-conditioned next to total reflection) or with a horizontal speed
// below 0.05 (a vacuum leg longer than ~2 b / 0.05), or the two estimates
// of |d_z| (normalization, output t4) apart by more than CAP_DZ_CHECK: a
// network that contradicts itself that much is outside what it learned.
constexpr float CAP_DZ_CHECK = 1e-2f;
__device__ __forceinline__ bool decode_cap(const float *yrow, const float *sc, float phi, float z, float al,
                                           float be, int kind, const JobP &jp, float margin, float out[NOUT]) {
  float t[NOUT];
#pragma unroll
  for (int o = 0; o < NOUT; ++o) t[o] = fmaf(yrow[o], sc[S_OSTD + o], sc[S_OMEAN + o]);
  float dth0, dz0, T0;
  baseline(kind, al, be, jp.a, jp.b, dth0, dz0, T0);
  const float u = cap_fraction(z, al, be, kind, jp);
  float frac, rcb, drb, adzb;
  cap_chord(kind, al, be, u, jp.a, jp.b, frac, rcb, drb, adzb);
  const bool up = be >= 0.0f;
  const float thc = phi + fmaf(frac, dth0, t[0]);
  const float rc = rcb + t[1], dr = drb + t[2];
  const float dt = jp.b * cosf(be) * sinf(al) / rc;
  const float q = fmaf(dr, dr, dt * dt);  // horizontal speed squared
  const float adz = sqrtf(fmaxf(0.0f, 1.0f - q));
  float st, ct;
  sincosf(thc, &st, &ct);
  const float cx = rc * ct, cy = rc * st;
  const float dx = dr * ct - dt * st, dy = dr * st + dt * ct;
  // vacuum leg: |(c + s d)_xy| = b with s > 0 from a cap point inside
  // (r_c < b), in the form without cancellation for either sign of d_r
  const float qb = rc * dr, qc = (rc - jp.b) * (rc + jp.b);
  const float disc = sqrtf(fmaxf(0.0f, fmaf(qb, qb, -q * qc)));
  const float s = qb >= 0.0f ? -qc / (qb + disc) : (disc - qb) / q;
  const float px = fmaf(s, dx, cx), py = fmaf(s, dy, cy);
  const float ph = wrap2pi(atan2f(py, px));
  float sph, cph;
  sincosf(ph, &sph, &cph);
  out[0] = ph;
  out[1] = fmaf(s, up ? adz : -adz, up ? jp.z1 : jp.z0);
  out[2] = atan2f(dy * cph - dx * sph, fmaf(dx, cph, dy * sph));
  out[3] = up ? asinf(fminf(1.0f, adz)) : -asinf(fminf(1.0f, adz));
  out[4] = fmaf(u, T0, t[3]) + s;
  return rc > jp.a + margin && rc < jp.b - margin && adz >= 0.05f && q >= 0.0025f &&
         fabsf(adzb + t[4] - adz) <= CAP_DZ_CHECK;
}

// cell of the side job's trust map: (axis, branch) x alpha x beta
__device__ __forceinline__ int cell_of(int kind, float al, float be) {
  int ia = (int)floorf((al + 0.5f * PI_F) * (NCELL_A / PI_F));
  int ib = (int)floorf((be + 0.5f * PI_F) * (NCELL_B / PI_F));
  ia = min(max(ia, 0), NCELL_A - 1);
  ib = min(max(ib, 0), NCELL_B - 1);
  return (kind * NCELL_A + ia) * NCELL_B + ib;
}

// cell of the cap job's trust map: (axis, branch) x alpha x |beta| x u
__device__ __forceinline__ int cell_cap(int kind, float al, float be, float u) {
  int ia = (int)floorf((al + 0.5f * PI_F) * (CAP_A / PI_F));
  int ib = (int)floorf(fabsf(be) * (2.0f * CAP_B / PI_F));
  int iu = (int)floorf(u * (float)CAP_U);
  ia = min(max(ia, 0), CAP_A - 1);
  ib = min(max(ib, 0), CAP_B - 1);
  iu = min(max(iu, 0), CAP_U - 1);
  return ((kind * CAP_A + ia) * CAP_B + ib) * CAP_U + iu;
}

struct GateP {
  float a, b, z0, z1;  // cloak radii r1, r2 and material height range
  float hres_max;    // conservation residual limit
  float cap_margin;  // distance of the predicted exit height from a cap (side job), of the cap point from the rims (cap job)
  float p_min;       // near-singular band of the conserved wave number
};

// Outside the near-singular band: the conserved wave number that keeps the
// path away from r = a (k_theta for the azimuthal cloak's extraordinary
// branch, whose metric is singular in theta only; |(k_theta, k_z)| for the
// radial extraordinary and azimuthal ordinary branches, singular in theta
// and z; the radial cloak's ordinary branch is homogeneous) is >= p_min.
__device__ __forceinline__ bool outside_band(int kind, float al, float be, float p_min) {
  if (kind == 0 || !(p_min > 0.0f)) return true;
  const float kt = cosf(be) * sinf(al), kz = sinf(be);
  const float p = kind == 3 ? fabsf(kt) : sqrtf(fmaf(kt, kt, kz * kz));
  return p >= p_min;
}

// The input half of the gate: a valid entry inside the material's height
// range, outside the near-singular band, in a trusted cell of the model's
// trust map and, for the cap job, heading for a cap (u < 1).
__device__ __forceinline__ bool gate_inputs(float phi, float z, float al, float be, float pol, float axis,
                                            const unsigned char *__restrict__ map, const GateP &gp, const JobP &jp) {
  if (!(entry_ok(phi, z, al, be, pol, axis) && z >= gp.z0 && z <= gp.z1)) return false;
  const int kind = kind_of(pol, axis);
  if (!outside_band(kind, al, be, gp.p_min)) return false;
  if (jp.job == RT_SUR_CAP) {
    const float u = cap_fraction(z, al, be, kind, jp);
    return u < 1.0f && map[cell_cap(kind, al, be, u)] != 0;
  }
  return map[cell_of(kind, al, be)] != 0;
}

// Gate and write the accepted predictions. A prediction is rejected (and
// the exact integrator traces the ray) when its input fails gate_inputs or
//  - side job: the predicted exit ray violates the conservation of the
//    tangential wave numbers (p_theta / b and p_z, equal at entry and exit
//    on r = b for every side-to-side transit) by more than hres_max, or the
//    predicted exit height lies within cap_margin of an end cap or beyond
//    it (z is monotonic along a transit since p_z keeps its sign, so an exit
//    height inside the material with margin means the whole path stayed
//    inside);
//  - cap job: the prediction is no usable cap exit (decode_cap).
__device__ __forceinline__ void gate_row(long long i, const float *__restrict__ x6, long long ld,
                                         const float *yrow, const float *__restrict__ sc,
                                         const unsigned char *__restrict__ map, const GateP &gp, const JobP &jp,
                                         float *__restrict__ y5, unsigned char *__restrict__ fallback,
                                         int *__restrict__ status) {
  const float phi = x6[i], z = x6[ld + i], al = x6[2 * ld + i], be = x6[3 * ld + i];
  const float pol = x6[4 * ld + i], axis = x6[5 * ld + i];
  bool acc = gate_inputs(phi, z, al, be, pol, axis, map, gp, jp);
  float out[NOUT];
  if (acc) {
    const int kind = kind_of(pol, axis);
    if (jp.job == RT_SUR_CAP) {
      acc = decode_cap(yrow, sc, phi, z, al, be, kind, jp, gp.cap_margin, out);
    } else {
      decode(yrow, sc, phi, z, al, be, kind, gp.a, gp.b, out);
      const float kt = cosf(be) * sinf(al), kz = sinf(be);
      const float kt2 = cosf(out[3]) * sinf(out[2]), kz2 = sinf(out[3]);
      const float res = fmaxf(fabsf(kt2 - kt), fabsf(kz2 - kz));
      acc = res <= gp.hres_max && out[1] >= gp.z0 + gp.cap_margin && out[1] <= gp.z1 - gp.cap_margin;
    }
#pragma unroll
    for (int o = 0; o < NOUT; ++o) acc = acc && isfinite(out[o]);
  }
  fallback[i] = acc ? 0 : 1;
  if (acc) {
#pragma unroll
    for (int o = 0; o < NOUT; ++o) y5[o * ld + i] = out[o];
    status[i] = RT_RAY_EXITED;
  }
}

// First half of the gate, on the inputs alone: entries that pass
// gate_inputs are appended to idx for the network; the others go to the
// exact transit (fallback = 1). With `chained`, only the rows an earlier
// model rejected (fallback != 0) are considered; the others keep fallback 0.
__global__ void __launch_bounds__(256) k_pregate(const float *__restrict__ x6, long long ld, int n,
                                                 const unsigned char *__restrict__ map, GateP gp, JobP jp,
                                                 int chained, unsigned char *__restrict__ fallback,
                                                 int *__restrict__ idx, unsigned int *__restrict__ count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  bool take = false;
  if (i < n && (!chained || fallback[i] != 0)) {
    take = gate_inputs(x6[i], x6[ld + i], x6[2 * ld + i], x6[3 * ld + i], x6[4 * ld + i], x6[5 * ld + i], map, gp,
                       jp);
    fallback[i] = take ? 0 : 1;
  }
  const unsigned long long m = __ballot(take);
  unsigned int base = 0;
  if (m != 0ull) {
    const int leader = __ffsll((unsigned long long)m) - 1;
    if ((int)__lane_id() == leader) base = atomicAdd(count, (unsigned int)__popcll(m));
    base = __shfl(base, leader);
  }
  const unsigned int lane = __lane_id();
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  if (take) idx[base + (unsigned int)__popcll(m & below)] = (int)i;
}

// second half of the gate on the network's outputs of the compacted entries
__global__ void __launch_bounds__(256) k_gate_idx(const float *__restrict__ x6, long long ld,
                                                  const int *__restrict__ idx, const unsigned int *count,
                                                  const float *__restrict__ y, const float *__restrict__ sc,
                                                  const unsigned char *__restrict__ map, GateP gp, JobP jp,
                                                  float *__restrict__ y5, unsigned char *__restrict__ fallback,
                                                  int *__restrict__ status) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < (long long)*count) gate_row(idx[p], x6, ld, y + p * NOUT, sc, map, gp, jp, y5, fallback, status);
}

// ---------------------------------------------------------------------------
// Fused inference: the whole network for FR rows per block, activations
// resident in LDS (BF16, FR x 256, rows padded to 264 so that the 16 rows
// an operand read touches fall in distinct banks). Each hidden layer is
// computed transposed, out^T = W^T act^T, so that an MFMA 16x16x32 tile's
// A operand is 8 consecutive inputs of one output unit (one 16-byte load of
// the BF16 weights in operand order, streamed from L2), its B operand 8
// consecutive inputs of one row (one 16-byte LDS read), and each lane's 4
// results are 4 consecutive output units of one row (one 8-byte LDS store).
// Wave w owns output units 64w..64w+63: 4 unit tiles x 8 row tiles, 128 FP32
// accumulators per lane. Layer 1 (FP32) fills the tile; layer 5 (FP32)
// reduces the layer-4 accumulators over each lane's 16 units, across the 4
// lane groups of a wave, then across the 4 waves through LDS, and the block
// writes the standardized outputs (n x 5) or the targets themselves.
//
// The vector instructions bound it (the 1024 SiLUs of an entry above all: 400
// us of issue for 2^20 entries, at the 2.2 GHz it runs at), but one wave's SiLUs
// and products (matrix cores: 165 us) followed each other, and the two waves of
// a SIMD did not make up for it. So the tile is worked on in two halves of 64
// rows, one layer step apart: every step multiplies one half and applies the
// previous step's SiLUs to the other in the same instruction stream, 16 matrix
// instructions and the SiLUs of 8 values per lane for each 32 inputs. Weights
// come FDEPTH such groups ahead, across steps (1 to 3: 552, 540, 568 us).
// 2^20 entries: 634 -> 540 us, 18 of them for the targets written from here
// instead of by a launch of their own, 40 for the weights in operand order. It
// uses all 256 registers and spills 10 (44 bytes of scratch per lane).
// ---------------------------------------------------------------------------
constexpr int FR = 128, FH = FR / 2, ALD = HID + 8, FDEPTH = 2;

// With idx != NULL, row r of the network is entry idx[r] for r < *count
// (a compacted subset); otherwise row r is entry r, r < n. With t != NULL the
// outputs go there as targets (5 x ldt), else to yout.
__global__ void __launch_bounds__(256, 2) k_mlp_fused(const float *__restrict__ x6, long long ld, int n,
                                                      const int *__restrict__ idx, const unsigned int *count,
                                                      const float *__restrict__ P, const bf16 *__restrict__ Wt,
                                                      const float *__restrict__ sc, JobP jp,
                                                      float *__restrict__ yout, float *__restrict__ t,
                                                      long long ldt) {
  __shared__ __attribute__((aligned(16))) bf16 act[FR * ALD];
  __shared__ float xn[FR * NIN];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int q = lane >> 4, c16 = lane & 15, ub = 64 * w;
  const long long row0 = (long long)blockIdx.x * FR;
  if (idx) n = (int)*count;  // block-uniform
  if (row0 >= n) return;
  // weights of group g = (step, 32 inputs): ring of FDEPTH + 1
  constexpr int KS = HID / 32;
  bf16x8 wf[FDEPTH + 1][4];
  const auto load_group = [&](int g) {
    const bf16 *W = Wt + (g / (2 * KS)) * HID * HID + (4 * w * KS + g % KS) * 512 + 8 * lane;
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
      wf[g % (FDEPTH + 1)][ti] = *reinterpret_cast<const bf16x8 *>(W + ti * KS * 512);
  };
#pragma unroll
  for (int g = 0; g < FDEPTH; ++g) load_group(g);
  // standardized input features of the tile (rows past n read as zeros)
  if (tid < FR) {
    const long long i = row0 + tid;
    float f[NIN] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (i < n) {
      features(x6, ld, idx ? (long long)idx[i] : i, jp, f);
#pragma unroll
      for (int k = 0; k < NIN; ++k) f[k] = (f[k] - sc[S_INOFF + k]) * sc[S_INSCALE + k];
    }
#pragma unroll
    for (int k = 0; k < NIN; ++k) xn[tid * NIN + k] = f[k];
  }
  __syncthreads();
  // layer 1 (FP32): thread = pair of hidden units x half of a half's rows
  float w0[NIN], w1[NIN], b0, b1;
  {
    const int u = 2 * (tid & 127);
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      w0[k] = P[OFF_W1 + k * HID + u];
      w1[k] = P[OFF_W1 + k * HID + u + 1];
    }
    b0 = P[OFF_B1 + u];
    b1 = P[OFF_B1 + u + 1];
  }
  const auto layer1 = [&](int r) {
    float z0 = b0, z1 = b1;
#pragma unroll
    for (int k = 0; k < NIN; ++k) {
      z0 = fmaf(xn[r * NIN + k], w0[k], z0);
      z1 = fmaf(xn[r * NIN + k], w1[k], z1);
    }
    bf16x2 pr;
    pr[0] = (bf16)silu_f(z0);
    pr[1] = (bf16)silu_f(z1);
    *reinterpret_cast<bf16x2 *>(&act[r * ALD + 2 * (tid & 127)]) = pr;
  };
  const int r1 = (tid >> 7) * (FH / 2);
#pragma unroll 4
  for (int j = 0; j < FH / 2; ++j) layer1(r1 + j);
  __syncthreads();
  f32x4 acc[2][4][4];  // [half][unit tile][row tile]
  // biases of the elementwise steps: 4 consecutive units per unit tile
  f32x4 bias[4];
  const auto load_bias = [&](long long off) {
#pragma unroll
    for (int ti = 0; ti < 4; ++ti)
#pragma unroll
      for (int r = 0; r < 4; ++r) bias[ti][r] = P[off + ub + 16 * ti + 4 * q + r];
  };
  // SiLU of unit tile ti, row tile tj of a half into the tile
  const auto silu_tile = [&](int h, int ti, int tj) {
    bf16x4 pk;
#pragma unroll
    for (int r = 0; r < 4; ++r) pk[r] = (bf16)silu_f(acc[h][ti][tj][r] + bias[ti][r]);
    *reinterpret_cast<bf16x4 *>(&act[(h * FH + 16 * tj + c16) * ALD + ub + 16 * ti + 4 * q]) = pk;
  };
  float s5[4][NOUT];  // layer 5: partial sums over this lane's 16 units for each of a half's rows
  const auto out_tile = [&](int h, int ti, int tj, const float w5[4][NOUT]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a4 = silu_f(acc[h][ti][tj][r] + bias[ti][r]);
#pragma unroll
      for (int o = 0; o < NOUT; ++o) s5[tj][o] = fmaf(a4, w5[r][o], s5[tj][o]);
    }
  };
  const auto load_w5 = [&](int ti, float w5[4][NOUT]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int o = 0; o < NOUT; ++o) w5[r][o] = P[OFF_W5 + (ub + 16 * ti + 4 * q + r) * NOUT + o];
  };
  float *red = reinterpret_cast<float *>(act);  // [half][wave][FH][NOUT], once the tile is not read any more
  const auto reduce_half = [&](int h) {
#pragma unroll
    for (int tj = 0; tj < 4; ++tj) {
#pragma unroll
      for (int o = 0; o < NOUT; ++o) {
        s5[tj][o] += __shfl_xor(s5[tj][o], 16);
        s5[tj][o] += __shfl_xor(s5[tj][o], 32);
      }
      if (q == 0) {
#pragma unroll
        for (int o = 0; o < NOUT; ++o) red[((h * 4 + w) * FH + 16 * tj + c16) * NOUT + o] = s5[tj][o];
      }
    }
  };
  // step st multiplies half st & 1 by layer 2 + st / 2
#pragma unroll
  for (int st = 0; st < 6; ++st) {
    const int h = st & 1, o = 1 - h;
    if (st >= 1) load_bias((st - 1) / 2 == 0 ? OFF_B2 : (st - 1) / 2 == 1 ? OFF_B3 : OFF_B4);
    if (st == 5) {
#pragma unroll
      for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int k = 0; k < NOUT; ++k) s5[tj][k] = 0.0f;
    }
    float w5[4][NOUT];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int g = st * KS + ks;
      if (g + FDEPTH < 6 * KS) load_group(g + FDEPTH);
      bf16x8 bop[4];
#pragma unroll
      for (int tj = 0; tj < 4; ++tj)
        bop[tj] = *reinterpret_cast<const bf16x8 *>(&act[(h * FH + 16 * tj + c16) * ALD + 32 * ks + 8 * q]);
#pragma unroll
      for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int ti = 0; ti < 4; ++ti)
          acc[h][ti][tj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              wf[g % (FDEPTH + 1)][ti], bop[tj], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[h][ti][tj], 0, 0, 0);
      if (st == 0) {
#pragma unroll
        for (int j = 0; j < FH / 2 / KS; ++j) layer1(FH + r1 + ks * (FH / 2 / KS) + j);
      } else if (st < 5) {
        silu_tile(o, ks >> 1, 2 * (ks & 1));
        silu_tile(o, ks >> 1, 2 * (ks & 1) + 1);
      } else {
        if (!(ks & 1)) load_w5(ks >> 1, w5);
        out_tile(o, ks >> 1, 2 * (ks & 1), w5);
        out_tile(o, ks >> 1, 2 * (ks & 1) + 1, w5);
      }
    }
    __syncthreads();  // the other half's tile is written, this half's read
  }
  reduce_half(0);
  load_bias(OFF_B4);
#pragma unroll
  for (int tj = 0; tj < 4; ++tj)
#pragma unroll
    for (int k = 0; k < NOUT; ++k) s5[tj][k] = 0.0f;
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) {
    float w5[4][NOUT];
    load_w5(ti, w5);
#pragma unroll
    for (int tj = 0; tj < 4; ++tj) out_tile(1, ti, tj, w5);
  }
  reduce_half(1);
  __syncthreads();
  if (tid < FR) {
    const long long i = row0 + tid;
    const float *rd = red + (tid / FH * 4 * FH + tid % FH) * NOUT;
    if (i < n) {
#pragma unroll
      for (int o = 0; o < NOUT; ++o) {
        const float y = P[OFF_B5 + o] + ((rd[o] + rd[FH * NOUT + o]) + (rd[2 * FH * NOUT + o] + rd[3 * FH * NOUT + o]));
        if (t)
          t[o * ldt + i] = fmaf(y, sc[S_OSTD + o], sc[S_OMEAN + o]);
        else
          yout[i * NOUT + o] = y;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Training: three launches make the gradient of a batch.
//  1. k_mlp_train: forward and backward of the whole network for R rows at a
//     time, activations and their gradients resident in one LDS tile, the
//     SiLU derivatives of layers 1 to 3 (FP32) in registers. It leaves what
//     the weight gradients are made of, a1..a3 and dz2..dz4 (BF16, row-major),
//     and per block the sums over its rows of everything thin: W1, the biases,
//     W5 and the loss.
//  2. k_weight_grad: dW_l = a_{l-1}^T dz_l, the three layers in one launch, split
//     over the rows.
//  3. k_grad_reduce: adds up both kernels' partial sums (fixed order, no
//     atomics: the same batch gives the same gradient bit for bit).
// One launch per layer product (FP32 pre-activations and both layouts of
// every dz through HBM, 0.9 GB at 65,536 rows, 14 launches) took 446 us for a
// gradient and step at 65,536 rows and 134 us at 1000; this takes 197 (173 when
// one model's buffers stay in the last-level cache) and 34.
// ---------------------------------------------------------------------------
// columns of a block's row of partial sums: W1 and b1, b2, b3, then b4, W5, b5
// (contiguous in the parameter vector each), and the loss's parts
constexpr int PS_W1 = 0, PS_B1 = NIN * HID, PS_B2 = PS_B1 + HID, PS_B3 = PS_B2 + HID, PS_B4 = PS_B3 + HID,
              PS_W5 = PS_B4 + HID, PS_B5 = PS_W5 + HID * NOUT, PS_LOSS = PS_B5 + NOUT, PS_N = PS_LOSS + 1;
constexpr int PS_LD = (PS_N + 3) / 4 * 4;
constexpr int TRAIN_THREADS = 512, TRAIN_BLOCKS = 256;  // one block per CU, taking tiles in turn
static_assert(OFF_W5 == OFF_B4 + HID && OFF_B5 == OFF_W5 + HID * NOUT, "b4, W5, b5 are contiguous");

// the parameter of a column (of PS_LOSS such)
__device__ __forceinline__ long long thin_param(int col) {
  return col < PS_B2 ? OFF_W1 + col
         : col < PS_B3 ? OFF_B2 + (col - PS_B2)
         : col < PS_B4 ? OFF_B3 + (col - PS_B3) : OFF_B4 + (col - PS_B4);
}

// The rows of a batch: targets t (SoA 5 x ldt) with row weights w (NULL = 1)
// and what k_mlp_train leaves. Loss per element d = y - (t - out_mean) /
// out_std: d^2, or for huber = delta > 0 the Huber function (d^2 up to |d| =
// delta, then 2 delta |d| - delta^2, gradient clipped to 2 delta sign(d)),
// times the row weight; loss and gradient divided by n.
struct TrainSink {
  const float *t;
  long long ldt;
  const float *w;
  float huber;
  bf16 *a[3], *dz[3];  // a1..a3 and dz2..dz4, [n][256]
  float *part;         // [blocks][PS_LD]
};

// Sums over the 16 rows a DPP row of lanes holds, of 8 values per lane: each
// fold adds two values over a pair of lanes and leaves one of the sums in
// either, so that three levels of folds and one addition leave lane c16 the
// sum of value t(c16), in 8 instead of 32 additions. Partners are lanes ^15,
// ^7, ^3, ^1; bits 3, 2, 1 of the lane choose the value.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ float fold(float v0, float v1, bool upper) {
  return (upper ? v1 : v0) + dpp<CTRL>(upper ? v0 : v1);
}
// sums of v0 over lanes l and l ^ 32 in lanes 0..31, of v1 in lanes 32..63;
// and over lanes l and l ^ 16, v0 in the even rows of 16 lanes and v1 in the odd
__device__ __forceinline__ float fold32(float v0, float v1) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float v0, float v1) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
struct RowFold {
  bool b3, b2, b1;
  __device__ explicit RowFold(int c16) : b3(c16 & 8), b2(c16 & 4), b1(c16 & 2) {}
  // units r = 0..3 of a unit tile, then both unit tiles of the wave
  __device__ float units(const float v[4]) const {
    return fold<0x141>(fold<0x140>(v[0], v[1], b3), fold<0x140>(v[2], v[3], b3), b2);
  }
  __device__ float tiles(const float v[2]) const {
    const float s = fold<0x1B>(v[0], v[1], b1);
    return s + dpp<0xB1>(s);
  }
  // the unit (of the wave's 32) whose sum this lane ends up with
  __device__ int unit(int q) const { return 16 * b1 + 4 * q + b3 + 2 * b2; }
};

// Keeps loads and addresses of one phase of k_mlp_train in that phase: without
// it the compiler moves everything the tile loop reads ahead of the loop and
// spills 2.5 KB of registers per lane.
template <typename T>
using GlobalPtr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ GlobalPtr<T> here(const T *p) {
  asm volatile("" : "+s"(p));
  return (GlobalPtr<T>)p;
}
// one register now: otherwise what it is computed from may be kept instead (z
// and sigmoid(z) for a derivative that is needed much later)
__device__ __forceinline__ float pin(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// the block's activation tile of R rows, the first `rows` of them in the
// batch, to rows row0.. of dst [n][256], 16 bytes per lane
template <int R>
__device__ __forceinline__ void store_tile(const bf16 *act, bf16 *__restrict__ dst, long long row0, int rows,
                                           int tid) {
  constexpr int STEP = TRAIN_THREADS / 32;
  const int c = 8 * (tid & 31), r0 = tid >> 5;
  bf16 *d = dst + row0 * HID + c;
  if (rows == R) {
    bf16x8 v[R / STEP];
#pragma unroll
    for (int k = 0; k < R / STEP; ++k) v[k] = *reinterpret_cast<const bf16x8 *>(&act[(r0 + k * STEP) * ALD + c]);
#pragma unroll
    for (int k = 0; k < R / STEP; ++k) *reinterpret_cast<bf16x8 *>(d + (r0 + k * STEP) * HID) = v[k];
  } else {
    for (int r = r0; r < rows; r += STEP)
      *reinterpret_cast<bf16x8 *>(d + r * HID) = *reinterpret_cast<const bf16x8 *>(&act[r * ALD + c]);
  }
}

// One block of 8 waves per CU; R = 16 NT rows per tile. Products are computed
// transposed as in the fused inference, wave w owning units 32 w..32 w + 31:
// a lane's results are 4 consecutive units (u0 + 0..3) of one row (16 tj + c16)
// per pair of tiles, and every elementwise step keeps that layout. What bounds
// it is the chain of seven phases per tile between barriers, so that nothing
// in it waits for memory: a wave's share of the next product's weights (64
// registers) is loaded during the elementwise phase before it, the thin
// parameters are in LDS, and inputs and targets of the next 512 rows are
// fetched, and the inputs' sines and cosines taken, by all threads at once.
// 65,536 rows: 127 us, of which the matrix products need 21 and the vector
// instructions 54 (SiLU and its derivative, 5 exponentials and reciprocals
// per unit and row); as 4 waves of 64 units with the weights loaded where
// they are used, 250; with each operand read from LDS waited for (a product
// 4400 clocks instead of 2700), 142. With 64 rows it uses all 256 registers and
// spills 14 (60 bytes of scratch per lane), with 32 and 16 it uses 225 and 185.
template <int NT>
__global__ void __launch_bounds__(TRAIN_THREADS, 2) k_mlp_train(const float *__restrict__ x6, long long ld, int n,
                                                                const float *__restrict__ P, const bf16 *Wt,
                                                                const bf16 *Wr, const float *__restrict__ sc,
                                                                JobP jp, TrainSink ts) {
  constexpr int R = 16 * NT, GT = TRAIN_THREADS / R, RED = R * NOUT;
  __shared__ __attribute__((aligned(16))) bf16 act[R * ALD];
  __shared__ __attribute__((aligned(16))) float th[PS_LD], ps[PS_LD];
  __shared__ __attribute__((aligned(16))) float xn[TRAIN_THREADS * NIN], tn[TRAIN_THREADS * (NOUT + 1)];
  __shared__ float red[8 * RED], dys[RED], lossp[NOUT];
  for (int e = threadIdx.x; e < PS_LD; e += TRAIN_THREADS) {
    th[e] = e < PS_LOSS ? P[thin_param(e)] : 0.0f;
    ps[e] = 0.0f;
  }
  if (threadIdx.x < NOUT) lossp[threadIdx.x] = 0.0f;
  const int ntiles = (n + R - 1) / R;
  int slot = GT;  // of the tile in the staged group
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x, ++slot) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // as for here(): no address leaves the loop
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, c16 = lane & 15, ub = 32 * w;
    const RowFold rf(c16);
    const int um = ub + rf.unit(q);       // the unit whose sums this lane has,
    const bool keeps = (c16 & 1) == 0;    // and adds
    if (slot == GT) {  // stage the inputs and targets of this and the next GT - 1 tiles
      slot = 0;
      const long long t = tile + (long long)(tid / R) * gridDim.x, i = t * R + tid % R;
      float f[NIN] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, tg[NOUT + 1] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (i < n) {
        tg[NOUT] = ts.w ? ts.w[i] : 1.0f;
        if (tg[NOUT] != 0.0f) {
#pragma unroll
          for (int o = 0; o < NOUT; ++o) tg[o] = (ts.t[o * ts.ldt + i] - sc[S_OMEAN + o]) / sc[S_OSTD + o];
        }
        features(x6, ld, i, jp, f);
#pragma unroll
        for (int k = 0; k < NIN; ++k) f[k] = (f[k] - sc[S_INOFF + k]) * sc[S_INSCALE + k];
      }
#pragma unroll
      for (int k = 0; k < NIN; ++k) xn[tid * NIN + k] = f[k];
#pragma unroll
      for (int o = 0; o <= NOUT; ++o) tn[tid * (NOUT + 1) + o] = tg[o];
    }
    const long long row0 = (long long)tile * R;
    const int rows = (int)min((long long)R, n - row0);
    bf16x8 wf[2][HID / 32];  // the wave's weights of the next product
    const auto load_weights = [&](const bf16 *W) {
      const GlobalPtr<bf16x8> p = (GlobalPtr<bf16x8>)here(W) + 2 * w * (HID / 32) * 64 + lane;
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int ks = 0; ks < HID / 32; ++ks) wf[ti][ks] = p[(ti * (HID / 32) + ks) * 64];
    };
    f32x4 acc[2][NT];  // [unit tile][row tile]
    const auto product = [&]() {
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < NT; ++tj) acc[ti][tj] = f32x4{0.f, 0.f, 0.f, 0.f};
      // the rows' operands come one group of 32 inputs ahead
      bf16x8 bop[2][NT];
      const auto load_rows = [&](int ks) {
#pragma unroll
        for (int tj = 0; tj < NT; ++tj)
          bop[ks & 1][tj] = *reinterpret_cast<const bf16x8 *>(&act[(16 * tj + c16) * ALD + 32 * ks + 8 * q]);
      };
      load_rows(0);
#pragma unroll
      for (int ks = 0; ks < HID / 32; ++ks) {
        if (ks + 1 < HID / 32) load_rows(ks + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tj = 0; tj < NT; ++tj)
#pragma unroll
          for (int ti = 0; ti < 2; ++ti)
            acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ti][ks], bop[ks & 1][tj], acc[ti][tj], 0, 0, 0);
      }
    };
    const auto vec = [&](int col) { return *reinterpret_cast<const f32x4 *>(&th[col]); };
    load_weights(Wt);
    __syncthreads();
    f32x4 ds1[2][NT], ds2[2][NT], ds3[2][NT];  // SiLU derivatives of layers 1 to 3
    {
      float xr[NT][NIN];
#pragma unroll
      for (int tj = 0; tj < NT; ++tj)
#pragma unroll
        for (int k = 0; k < NIN; ++k) xr[tj][k] = xn[(slot * R + 16 * tj + c16) * NIN + k];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const int u0 = ub + 16 * ti + 4 * q;
        const f32x4 b = vec(PS_B1 + u0);
        f32x4 w1[NIN];
#pragma unroll
        for (int k = 0; k < NIN; ++k) w1[k] = vec(PS_W1 + k * HID + u0);
#pragma unroll
        for (int tj = 0; tj < NT; ++tj) {
          bf16x4 pk;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            float z = b[r];
#pragma unroll
            for (int k = 0; k < NIN; ++k) z = fmaf(xr[tj][k], w1[k][r], z);
            const float s = sigmoid_f(z);
            pk[r] = (bf16)(z * s);
            ds1[ti][tj][r] = pin(dsilu_f(z, s));
          }
          *reinterpret_cast<bf16x4 *>(&act[(16 * tj + c16) * ALD + u0]) = pk;
        }
      }
    }
    __syncthreads();
    const auto hidden = [&](bf16 *a, const bf16 *next, int bias_col, f32x4 (&ds)[2][NT]) {
      store_tile<R>(act, a, row0, rows, tid);
      product();
      load_weights(next);
      __syncthreads();  // every wave has read the layer's input tile
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const int u0 = ub + 16 * ti + 4 * q;
        const f32x4 bias = vec(bias_col + u0);
#pragma unroll
        for (int tj = 0; tj < NT; ++tj) {
          bf16x4 pk;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = acc[ti][tj][r] + bias[r], s = sigmoid_f(z);
            pk[r] = (bf16)(z * s);
            ds[ti][tj][r] = pin(dsilu_f(z, s));
          }
          *reinterpret_cast<bf16x4 *>(&act[(16 * tj + c16) * ALD + u0]) = pk;
        }
      }
      __syncthreads();
    };
    hidden(ts.a[0], Wt + HID * HID, PS_B2, ds2);
    hidden(ts.a[1], Wt + 2 * HID * HID, PS_B3, ds3);
    store_tile<R>(act, ts.a[2], row0, rows, tid);
    product();
    {
      // layer 5 (FP32) on a4 = silu(z4): partial sums over this lane's 8
      // units for each of its rows, then over the 4 lane groups and 8 waves
      float s5[NT][NOUT];
#pragma unroll
      for (int tj = 0; tj < NT; ++tj)
#pragma unroll
        for (int o = 0; o < NOUT; ++o) s5[tj][o] = 0.0f;
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const int u0 = ub + 16 * ti + 4 * q;
        const f32x4 bias = vec(PS_B4 + u0);
        f32x4 w5[NOUT];  // the 4 x 5 weights of units u0 + 0..3 in memory order
#pragma unroll
        for (int o = 0; o < NOUT; ++o) w5[o] = vec(PS_W5 + u0 * NOUT + 4 * o);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int tj = 0; tj < NT; ++tj) {
            const float z = acc[ti][tj][r] + bias[r];
            acc[ti][tj][r] = pin(z);  // z4, kept for the way back
            const float a4 = silu_f(z);
#pragma unroll
            for (int o = 0; o < NOUT; ++o)
              s5[tj][o] = fmaf(a4, w5[(r * NOUT + o) / 4][(r * NOUT + o) % 4], s5[tj][o]);
          }
      }
      if constexpr (NT == 4) {
        // fold the 4 row tiles over the 4 lane groups: lane group q ends up
        // with row tile 2 (q & 1) + (q >> 1)
#pragma unroll
        for (int o = 0; o < NOUT; ++o) {
          const float lo = fold32(s5[0][o], s5[1][o]), hi = fold32(s5[2][o], s5[3][o]);
          red[w * RED + (16 * (2 * (q & 1) + (q >> 1)) + c16) * NOUT + o] = fold16(lo, hi);
        }
      } else {
#pragma unroll
        for (int tj = 0; tj < NT; ++tj)
#pragma unroll
          for (int o = 0; o < NOUT; ++o) {
            s5[tj][o] += __shfl_xor(s5[tj][o], 16);
            s5[tj][o] += __shfl_xor(s5[tj][o], 32);
            if (q == 0) red[w * RED + (16 * tj + c16) * NOUT + o] = s5[tj][o];
          }
      }
    }
    load_weights(Wr + 2 * HID * HID);
    __syncthreads();
    if (tid < RED) {  // outputs, loss and dy: thread = output x row
      const int o = tid / R, row = tid % R, e = row * NOUT + o;
      float v[8], l = 0.0f, g = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = red[k * RED + e];
      const float y = th[PS_B5 + o] + (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
      const float *tr = &tn[(slot * R + row) * (NOUT + 1)];
      const float wrow = tr[NOUT];
      if (wrow != 0.0f) {
        const float d = y - tr[o];
        if (ts.huber > 0.0f && fabsf(d) > ts.huber) {
          l = wrow * (2.0f * ts.huber * fabsf(d) - ts.huber * ts.huber);
          g = 2.0f * wrow * copysignf(ts.huber, d);
        } else {
          l = wrow * d * d;
          g = 2.0f * wrow * d;
        }
      }
      l = l / (float)n;
      g = g / (float)n;
      dys[e] = g;
#pragma unroll
      for (int off = R / 2; off > 0; off >>= 1) {
        l += __shfl_xor(l, off);
        g += __shfl_xor(g, off);
      }
      if (row == 0) {
        lossp[o] += l;
        ps[PS_B5 + o] += g;
      }
    }
    __syncthreads();
    // layer 5 backwards: dz4 = (dy W5^T) silu'(z4), dW5 = a4^T dy, db4 = sum dz4
    {
      float dy[NT][NOUT], sz[2], sw[NOUT][2];
#pragma unroll
      for (int tj = 0; tj < NT; ++tj)
#pragma unroll
        for (int o = 0; o < NOUT; ++o) dy[tj][o] = dys[(16 * tj + c16) * NOUT + o];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const int u0 = ub + 16 * ti + 4 * q;
        bf16x4 pk[NT];
        float gw[NOUT][4], gz[4];
        f32x4 w5[NOUT];
#pragma unroll
        for (int o = 0; o < NOUT; ++o) w5[o] = vec(PS_W5 + u0 * NOUT + 4 * o);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gz[r] = 0.0f;
#pragma unroll
          for (int o = 0; o < NOUT; ++o) gw[o][r] = 0.0f;
#pragma unroll
          for (int tj = 0; tj < NT; ++tj) {
            const float z = acc[ti][tj][r], s = sigmoid_f(z), a4 = z * s;
            float da = 0.f;
#pragma unroll
            for (int o = 0; o < NOUT; ++o) {
              da = fmaf(dy[tj][o], w5[(r * NOUT + o) / 4][(r * NOUT + o) % 4], da);
              gw[o][r] = fmaf(a4, dy[tj][o], gw[o][r]);
            }
            const float g = da * dsilu_f(z, s);
            gz[r] += g;
            pk[tj][r] = (bf16)g;
          }
        }
        sz[ti] = rf.units(gz);
#pragma unroll
        for (int o = 0; o < NOUT; ++o) sw[o][ti] = rf.units(gw[o]);
#pragma unroll
        for (int tj = 0; tj < NT; ++tj) *reinterpret_cast<bf16x4 *>(&act[(16 * tj + c16) * ALD + u0]) = pk[tj];
      }
      const float s = rf.tiles(sz);
      if (keeps) ps[PS_B4 + um] += s;
#pragma unroll
      for (int o = 0; o < NOUT; ++o) {
        const float so = rf.tiles(sw[o]);
        if (keeps) ps[PS_W5 + um * NOUT + o] += so;
      }
    }
    __syncthreads();
    // hidden layers: dz_l = (dz_{l+1} W_{l+1}^T) silu'(z_l), db_l = sum dz_l
    const auto hidden_back = [&](bf16 *dz, const bf16 *next, int sums, const f32x4 (&ds)[2][NT]) {
      store_tile<R>(act, dz, row0, rows, tid);
      product();
      load_weights(next);
      __syncthreads();
      float sz[2];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        const int u0 = ub + 16 * ti + 4 * q;
        float gz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tj = 0; tj < NT; ++tj) {
          bf16x4 pk;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float g = acc[ti][tj][r] * ds[ti][tj][r];
            gz[r] += g;
            pk[r] = (bf16)g;
          }
          *reinterpret_cast<bf16x4 *>(&act[(16 * tj + c16) * ALD + u0]) = pk;
        }
        sz[ti] = rf.units(gz);
      }
      const float s = rf.tiles(sz);
      if (keeps) ps[sums + um] += s;
      __syncthreads();
    };
    hidden_back(ts.dz[2], Wr + HID * HID, PS_B3, ds3);
    hidden_back(ts.dz[1], Wr, PS_B2, ds2);
    // dz1 never leaves its registers: dW1 = x^T dz1, db1 = sum dz1
    store_tile<R>(act, ts.dz[0], row0, rows, tid);
    product();
    {
      float xr[NT][NIN], sz[2], sw[NIN][2];
#pragma unroll
      for (int tj = 0; tj < NT; ++tj)
#pragma unroll
        for (int k = 0; k < NIN; ++k) xr[tj][k] = xn[(slot * R + 16 * tj + c16) * NIN + k];
#pragma unroll
      for (int ti = 0; ti < 2; ++ti) {
        float gw[NIN][4], gz[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gz[r] = 0.0f;
#pragma unroll
          for (int k = 0; k < NIN; ++k) gw[k][r] = 0.0f;
#pragma unroll
          for (int tj = 0; tj < NT; ++tj) {
            const float g = acc[ti][tj][r] * ds1[ti][tj][r];
            gz[r] += g;
#pragma unroll
            for (int k = 0; k < NIN; ++k) gw[k][r] = fmaf(xr[tj][k], g, gw[k][r]);
          }
        }
        sz[ti] = rf.units(gz);
#pragma unroll
        for (int k = 0; k < NIN; ++k) sw[k][ti] = rf.units(gw[k]);
      }
      const float s = rf.tiles(sz);
      if (keeps) ps[PS_B1 + um] += s;
#pragma unroll
      for (int k = 0; k < NIN; ++k) {
        const float sk = rf.tiles(sw[k]);
        if (keeps) ps[PS_W1 + k * HID + um] += sk;
      }
    }
    __syncthreads();  // act, xn and dys are free for the next tile
  }
  float *out = ts.part + (long long)blockIdx.x * PS_LD;
  for (int e = threadIdx.x; e < PS_LOSS; e += TRAIN_THREADS) out[e] = ps[e];
  if (threadIdx.x == 0) out[PS_LOSS] = ((lossp[0] + lossp[1]) + (lossp[2] + lossp[3])) + lossp[4];
}

// dW_l(i, j) = sum over rows of a_{l-1}(row, i) dz_l(row, j) for l = 2..4: 128 x
// 128 tiles, 4 waves of 64 x 64, rows in steps of 64 through double-buffered
// LDS, split over the rows. Both operands are row-major, rows being the sum
// index; an MFMA lane needs 8 consecutive rows of one unit, which two
// transposing LDS reads give (ds_read_b64_tr_b16: 16 lanes fetch a 4 x 16
// block, 4 units each, and lane i gets unit i of the 4 rows), so no transposed
// copy of either exists in memory. The 4 tiles of a (layer, split) are next to
// each other on one XCD, whose L2 then reads each operand from memory once:
// 65,536 rows (0.2 GB) take 40 us, and 62 where those tiles are on different
// XCDs. The transposing reads (64 bytes a clock) bound the rest.
constexpr int WG_T = 128, WG_K = 64, WG_LD = WG_T + 16, WG_TILES = 4, WG_SPLITS = 42;
struct WGrad {
  const bf16 *a[3], *dz[3];
  float *part;  // [split][layer][256 * 256]
  int n, kchunk, tiles;
};

// 64 rows from k0 of 128 columns, rows past kend as zeros: a buffer load checks
// its offset against the resource's size, so that the loop has no branches. All
// of the offset is in the vector operand: the scalar one is not part of what
// the instruction promises to check, and rows past kend hold an earlier, larger
// batch's values.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void wg_load(u32x4 v[4], const bf16 *src, int k0, int kend, int col0, int tid) {
  // (all uniform; said so, as the compiler takes vector instructions for parts of it)
  const int rows = __builtin_amdgcn_readfirstlane(max(0, min(WG_K, kend - k0)));
  const unsigned long long base = (unsigned long long)(src + (long long)k0 * HID);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)base);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(base >> 32));
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((unsigned long long)hi << 32 | lo), 0, rows * HID * (int)sizeof(bf16), 0x00027000);
  const int off = ((tid >> 4) * HID + 8 * (tid & 15) + col0) * (int)sizeof(bf16);
#pragma unroll
  for (int p = 0; p < 4; ++p)
    v[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * p * HID * (int)sizeof(bf16), 0, 0);
}

__device__ __forceinline__ void wg_store(bf16 *T, const u32x4 v[4], int tid) {
#pragma unroll
  for (int p = 0; p < 4; ++p)
    *reinterpret_cast<u32x4 *>(&T[(16 * p + (tid >> 4)) * WG_LD + 8 * (tid & 15)]) = v[p];
}

// 8 rows of unit u0 + c16 for lane (q, c16): k0 + 4 q + 0..3 and k0 + 16 + 4 q +
// 0..3. Which k of the product's 32 a lane holds is free as long as both
// operands agree, and 16 consecutive rows a read fall in distinct banks.
__device__ __forceinline__ bf16x8 wg_operand(const bf16 *T, int k0, int u0, int q, int c16) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s16x4 *LdsPtr;
  const bf16 *p = &T[(k0 + 4 * q + (c16 >> 2)) * WG_LD + u0 + 4 * (c16 & 3)];
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)(p + 16 * WG_LD));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ void __launch_bounds__(256, 2) k_weight_grad(WGrad g) {
  __shared__ __attribute__((aligned(16))) bf16 sm[2][2][WG_K * WG_LD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, c16 = lane & 15;
  // an eighth of the tiles per XCD (consecutive blocks go to different ones)
  const unsigned t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (t >= (unsigned)g.tiles) return;
  const int tile = (int)(t % WG_TILES), ls = __builtin_amdgcn_readfirstlane((int)(t / WG_TILES));
  const int split = __builtin_amdgcn_readfirstlane(ls / 3), layer = ls - 3 * split;
  const int i0 = (tile >> 1) * WG_T, j0 = (tile & 1) * WG_T, im = 64 * (w >> 1), jm = 64 * (w & 1);
  const int kbeg = split * g.kchunk, kend = min(g.n, kbeg + g.kchunk);
  const bf16 *A = layer == 0 ? g.a[0] : (layer == 1 ? g.a[1] : g.a[2]);
  const bf16 *B = layer == 0 ? g.dz[0] : (layer == 1 ? g.dz[1] : g.dz[2]);
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nk = (kend - kbeg + WG_K - 1) / WG_K;
  // two steps in flight (rows past kend read as zeros, so that an odd number
  // of steps adds an empty one)
  u32x4 ra[2][4], rb[2][4];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    wg_load(ra[p], A, kbeg + p * WG_K, kend, i0, tid);
    wg_load(rb[p], B, kbeg + p * WG_K, kend, j0, tid);
  }
  for (int it = 0; it < nk; it += 2)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      bf16 *As = sm[p][0], *Bs = sm[p][1];
      wg_store(As, ra[p], tid);
      wg_store(Bs, rb[p], tid);
      __syncthreads();  // also: every wave is done with the stage's previous use
      wg_load(ra[p], A, kbeg + (it + 2 + p) * WG_K, kend, i0, tid);
      wg_load(rb[p], B, kbeg + (it + 2 + p) * WG_K, kend, j0, tid);
      __builtin_amdgcn_sched_barrier(0);  // issued before the products, not after them
#pragma unroll
      for (int ks = 0; ks < WG_K; ks += 32) {
        bf16x8 af[4], bf_[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          af[i] = wg_operand(As, ks, im + 16 * i, q, c16);
          bf_[i] = wg_operand(Bs, ks, jm + 16 * i, q, c16);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf_[j], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  // lane holds D[4 q + r][c16] of each tile
  float *o = g.part + ((long long)split * 3 + layer) * HID * HID;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        o[(i0 + im + 16 * i + 4 * q + r) * HID + j0 + jm + 16 * j + c16] = acc[i][j][r];
}

// The gradient from the partial sums: blocks 0..191 the 3 x 256 x 256 weights
// of the hidden layers (256 float4 columns x 4 groups of splits), the others 64
// of the thin columns each (x 16 groups of blocks). G, and where the caller
// asks for them its gradient vector and loss.
constexpr int GR_THREADS = 1024, GR_WBLOCKS = 3 * HID * HID / 1024, GR_BLOCKS = GR_WBLOCKS + (PS_N + 63) / 64;
__global__ void __launch_bounds__(GR_THREADS) k_grad_reduce(const float *__restrict__ wpart, int splits,
                                                            const float *__restrict__ part, int blocks,
                                                            float *__restrict__ G, float *__restrict__ grads,
                                                            float *__restrict__ loss, float *__restrict__ loss_out) {
  __shared__ float4 sh4[3][256];
  __shared__ float sh[16][64];
  const int tid = threadIdx.x;
  if (blockIdx.x < GR_WBLOCKS) {
    const int c = tid & 255, grp = tid >> 8;
    const long long e = (long long)blockIdx.x * 1024 + 4 * c;
    float4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k = grp; k < splits; k += 4) {
      const float4 v = *reinterpret_cast<const float4 *>(&wpart[(long long)k * 3 * HID * HID + e]);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    if (grp) sh4[grp - 1][c] = s;
    __syncthreads();
    if (grp) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float4 v = sh4[k][c];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    const long long l = e / (HID * HID), off = l == 0 ? OFF_W2 : (l == 1 ? OFF_W3 : OFF_W4);
    const long long o = off + e % (HID * HID);
    *reinterpret_cast<float4 *>(&G[o]) = s;
    if (grads) {  // a caller's vector need not be 16-byte aligned
      grads[o] = s.x; grads[o + 1] = s.y; grads[o + 2] = s.z; grads[o + 3] = s.w;
    }
    return;
  }
  const int c = tid & 63, grp = tid >> 6, col = (blockIdx.x - GR_WBLOCKS) * 64 + c;
  float s = 0.f;
  if (col < PS_N) {
#pragma unroll 4
    for (int k = grp; k < blocks; k += 16) s += part[(long long)k * PS_LD + col];
  }
  sh[grp][c] = s;
  __syncthreads();
  if (grp || col >= PS_N) return;
  s = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) s += sh[k][c];
  if (col == PS_LOSS) {
    *loss = s;
    if (loss_out) *loss_out = s;
    return;
  }
  const long long o = thin_param(col);
  G[o] = s;
  if (grads) grads[o] = s;
}

// error of the decoded prediction against the exact exit, per trust-map cell:
// err = max(|x - x_exact| / b, angle(d, d_exact)); a ray the exact
// integrator did not carry to an exit (absorbed, reflected, ...) makes its
// cell untrusted. The cap job counts only the rows its gate would offer the
// network (heading for a cap, u < 1) and whose prediction is a usable cap
// exit (decode_cap with the gate's margin): the gate rejects the
// others whatever their cell, so they neither count towards nor fail it.
__global__ void __launch_bounds__(256) k_calib(const float *__restrict__ x6, long long ld, int n,
                                               const float *__restrict__ y, const float *__restrict__ sc,
                                               const float *__restrict__ ye, const int *__restrict__ st,
                                               const float *__restrict__ hres, float unresolved, bool infinite,
                                               JobP jp, float margin, unsigned int *__restrict__ cmax,
                                               unsigned int *__restrict__ ccnt) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float phi = x6[i], z = x6[ld + i], al = x6[2 * ld + i], be = x6[3 * ld + i];
  const float pol = x6[4 * ld + i], axis = x6[5 * ld + i];
  if (!entry_ok(phi, z, al, be, pol, axis)) return;
  // an exit the integrator did not resolve is no reference: a drifted
  // Hamiltonian, or total internal reflection at the exit of a side entry
  // into the infinite cylinder (impossible in exact arithmetic: the
  // tangential wave numbers the ray entered with are conserved, so the exit
  // refraction transmits; only drift beyond a grazing entry's normal wave
  // number turns it evanescent)
  if (hres && st[i] == RT_RAY_EXITED && !(hres[i] <= unresolved)) return;
  if (hres && infinite && st[i] == RT_RAY_TIR) return;
  const int kind = kind_of(pol, axis);
  const float b = jp.b;
  int cell;
  float out[NOUT];
  bool usable = true;
  if (jp.job == RT_SUR_CAP) {
    if (!(z >= jp.z0 && z <= jp.z1)) return;
    const float u = cap_fraction(z, al, be, kind, jp);
    if (!(u < 1.0f)) return;
    cell = cell_cap(kind, al, be, u);
    usable = decode_cap(y + i * NOUT, sc, phi, z, al, be, kind, jp, margin, out);
  } else {
    cell = cell_of(kind, al, be);
    decode(y + i * NOUT, sc, phi, z, al, be, kind, jp.a, b, out);
  }
  float err = INFINITY;
  if (st[i] == RT_RAY_EXITED) {
    if (!usable) return;
    float ex[NOUT], xp[3], dp[3], xe[3], de[3];
#pragma unroll
    for (int o = 0; o < NOUT; ++o) ex[o] = ye[o * ld + i];
    exit_ray(out, b, xp, dp);
    exit_ray(ex, b, xe, de);
    float ex2 = 0.f, dd2 = 0.f;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      ex2 += (xp[j] - xe[j]) * (xp[j] - xe[j]);
      dd2 += (dp[j] - de[j]) * (dp[j] - de[j]);
    }
    const float dang = 2.0f * asinf(fminf(1.0f, 0.5f * sqrtf(dd2)));
    err = fmaxf(sqrtf(ex2) / b, dang);
    if (!isfinite(err)) err = INFINITY;
  }
  atomicMax(&cmax[cell], __float_as_uint(err));  // err >= 0: uint order = float order
  atomicAdd(&ccnt[cell], 1u);
}

unsigned int gblocks(long long n, int b) { return (unsigned int)std::max(1LL, (n + b - 1) / b); }

}  // namespace sg

using namespace sg;

struct rt_model_s {
  int device = -1;
  void *base = nullptr;
  float *P = nullptr, *G = nullptr, *m = nullptr, *v = nullptr;  // FP32 [NPARAM]
  bf16 *Pb = nullptr;                                            // BF16 W2..W4
  float *scal = nullptr;                                         // [NSCAL]
  unsigned char *map = nullptr;                                  // trust map [NCELLS]
  unsigned int *cal = nullptr;                                   // calibration max/count [2 * NCELLS]
  double *mom = nullptr;                                         // moments [NMOM]
  float h_scal[NSCAL] = {0};
  std::vector<unsigned char> h_map;
  int map_valid = 0;
  int job = RT_SUR_SIDE;
  float geo[4] = {0.f, 0.f, 0.f, 0.f};  // cap job: r1, r2, z0, z1 of the cloak it was set up for
  rt_model next = nullptr;              // rt_surrogate_chain: rows this model rejects go to next
  rt_model prev = nullptr;              // the model whose rejected rows come here
  rt_gate_opts gate{};
  long long step = 0;
  // activations for up to `cap` rows
  long long cap = 0;
  void *act = nullptr;
  bf16 *a[3] = {nullptr, nullptr, nullptr};   // a1..a3 [cap][256]
  bf16 *dz[3] = {nullptr, nullptr, nullptr};  // dz2..dz4 [cap][256]
  float *part = nullptr;                      // thin partial sums [TRAIN_BLOCKS][PS_LD]
  float *wpart = nullptr;                     // weight-gradient partial sums [WG_SPLITS][3][256 * 256]
  // standardized outputs of the fused inference kernel, and the compacted
  // entry list of the gated inference
  long long ycap = 0;
  float *yinf = nullptr;
  int *idx = nullptr;
  unsigned int *count = nullptr;
};

namespace {

int reserve_acts(rt_model mo, long long n) {
  if (n <= mo->cap) return RT_OK;
  if (mo->act) {
    (void)hipDeviceSynchronize();
    (void)hipFree(mo->act);
    mo->act = nullptr;
    mo->cap = 0;
  }
  const long long cap = std::max(n, 4096LL);
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t ab = al(sizeof(bf16) * cap * HID), pb = al(sizeof(float) * TRAIN_BLOCKS * PS_LD);
  const size_t wb = al(sizeof(float) * WG_SPLITS * 3 * HID * HID);
  const size_t bytes = 6 * ab + pb + wb;
  void *p = nullptr;
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(RT_E_NOMEM, "hipMalloc of %zu bytes for activations failed", bytes);
  }
  char *c = (char *)p;
  size_t off = 0;
  for (int l = 0; l < 3; ++l) { mo->a[l] = (bf16 *)(c + off); off += ab; }
  for (int l = 0; l < 3; ++l) { mo->dz[l] = (bf16 *)(c + off); off += ab; }
  mo->part = (float *)(c + off); off += pb;
  mo->wpart = (float *)(c + off);
  mo->act = p;
  mo->cap = cap;
  return RT_OK;
}

int reserve_yinf(rt_model mo, long long n) {
  if (n <= mo->ycap) return RT_OK;
  if (mo->yinf) {
    (void)hipDeviceSynchronize();
    (void)hipFree(mo->yinf);
    mo->yinf = nullptr;
    mo->ycap = 0;
  }
  const long long cap = std::max(n, 4096LL);
  const size_t yb = (sizeof(float) * cap * NOUT + 255) & ~(size_t)255;
  if (hipMalloc((void **)&mo->yinf, yb + sizeof(int) * cap + 256) != hipSuccess) {
    (void)hipGetLastError();
    return fail(RT_E_NOMEM, "hipMalloc for %lld inference outputs failed", cap);
  }
  mo->idx = (int *)((char *)mo->yinf + yb);
  mo->count = (unsigned int *)((char *)mo->idx + ((sizeof(int) * cap + 255) & ~(size_t)255));
  mo->ycap = cap;
  return RT_OK;
}

// The job parameters of a model's kernels: the cap job carries the
// geometry it was set up for; the side job's features need none, and its
// decoding takes the radii of the cloak description d (if given).
JobP job_for(rt_model mo, const rt_cloak_desc *d) {
  if (mo->job == RT_SUR_CAP) return JobP{RT_SUR_CAP, mo->geo[0], mo->geo[1], mo->geo[2], mo->geo[3]};
  if (!d) return JobP{RT_SUR_SIDE, 0.0f, 0.0f, 0.0f, 0.0f};
  return JobP{RT_SUR_SIDE, (float)d->r1, (float)d->r2, std::isfinite(d->z0) ? (float)d->z0 : -INFINITY,
              std::isfinite(d->z1) ? (float)d->z1 : INFINITY};
}

// outputs of n rows (fused kernel): targets into t (5 x ldt), or where t is
// NULL standardized into mo->yinf
void infer_outputs(rt_model mo, const float *x, long long ld, int n, float *t, long long ldt, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_fused, dim3(gblocks(n, FR)), dim3(256), 0, s, x, ld, n, nullptr, nullptr, mo->P, mo->Pb,
                     mo->scal, job_for(mo, nullptr), mo->yinf, t, ldt);
}

// BF16 weights of W2 (l = 0), W3 (1), W4 (2) for the backward products (mo->Pb: forward)
const bf16 *wr(rt_model mo) { return mo->Pb + NBF; }

// gradient and loss of a batch of n rows into mo->G and scal[S_LOSS], and to
// the caller's vectors (may be NULL)
void forward_backward(rt_model mo, const float *x, const float *t, long long ld, const float *wrow, int n,
                      float huber, float *grads, float *loss, hipStream_t s) {
  TrainSink ts{t, ld, wrow, huber, {mo->a[0], mo->a[1], mo->a[2]}, {mo->dz[0], mo->dz[1], mo->dz[2]}, mo->part};
  // Rows per tile: the fewest whose tiles go over the chip once, as a tile's
  // chain of layers takes 21, 25 and 35 us at 16, 32 and 64 rows and the work
  // beyond it shares the CU no better; past 8192 rows, 64, which read the
  // weights least often. Gradient and step at 4096 / 8192 / 16384 / 65536 rows,
  // one model's buffers, us: 41 / 54 / 84 / 257 with 16, 44 / 46 / 68 / 191 with
  // 32, 52 / 54 / 65 / 173 with 64.
  const int rows = n <= 16 * TRAIN_BLOCKS ? 16 : n <= 32 * TRAIN_BLOCKS ? 32 : 64;
  const int blocks = std::min((int)gblocks(n, rows), TRAIN_BLOCKS);
  const auto kern = rows == 64 ? k_mlp_train<4> : rows == 32 ? k_mlp_train<2> : k_mlp_train<1>;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(TRAIN_THREADS), 0, s, x, ld, n, mo->P, mo->Pb, wr(mo), mo->scal,
                     job_for(mo, nullptr), ts);
  // splits of two or more steps of 64 rows (the last takes what is left), two
  // blocks per CU for large batches
  int splits = std::min(WG_SPLITS, std::max(1, n / (2 * WG_K)));
  const int kchunk = ((n + splits - 1) / splits + WG_K - 1) / WG_K * WG_K;
  splits = (n + kchunk - 1) / kchunk;
  WGrad g{{mo->a[0], mo->a[1], mo->a[2]}, {mo->dz[0], mo->dz[1], mo->dz[2]}, mo->wpart, n, kchunk,
          3 * WG_TILES * splits};
  // (whole groups of WG_TILES per XCD)
  hipLaunchKernelGGL(k_weight_grad, dim3(8 * WG_TILES * (unsigned)gblocks(3 * splits, 8)), dim3(256), 0, s, g);
  hipLaunchKernelGGL(k_grad_reduce, dim3(GR_BLOCKS), dim3(GR_THREADS), 0, s, mo->wpart, splits, mo->part, blocks,
                     mo->G, grads, mo->scal + S_LOSS, loss);
}

int check_model(rt_model mo) {
  if (!mo || !mo->P) return fail(RT_E_INVALID, "model is NULL");
  int dev = -1;
  (void)hipGetDevice(&dev);
  if (dev != mo->device) return fail(RT_E_INVALID, "model was created on device %d, current is %d", mo->device, dev);
  return RT_OK;
}

int check_rows(long long n, long long ld, const void *x6) {
  if (n < 1 || n > (1LL << 24)) return fail(RT_E_INVALID, "n must be in [1, 2^24]");
  if (ld < n) return fail(RT_E_INVALID, "ld must be >= n");
  if (!x6) return fail(RT_E_INVALID, "x6 is required");
  return RT_OK;
}

int upload_scal(rt_model mo) {
  if (hipMemcpy(mo->scal, mo->h_scal, sizeof(float) * S_LOSS, hipMemcpyHostToDevice) != hipSuccess)
    return fail(RT_E_DEVICE, "copy of the scaling failed");
  return RT_OK;
}

int upload_map(rt_model mo) {
  if (hipMemcpy(mo->map, mo->h_map.data(), NCELLS, hipMemcpyHostToDevice) != hipSuccess)
    return fail(RT_E_DEVICE, "copy of the trust map failed");
  return RT_OK;
}

int cloak_geometry(const rt_cloak *cloaks, int32_t n_cloaks, rt_cloak_desc &d) {
  if (n_cloaks < 1 || n_cloaks > 2 || !cloaks || !cloaks[0]) return fail(RT_E_INVALID, "need 1 or 2 cloak handles");
  if (rt_cloak_get_desc(cloaks[0], &d) != RT_OK) return fail(RT_E_INVALID, "bad cloak handle");
  return RT_OK;
}

int launch_err(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(RT_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
  return RT_OK;
}

// A cap model works on cloaks of the geometry it was set up for.
int check_geometry(rt_model mo, const rt_cloak_desc &d) {
  if (mo->job != RT_SUR_CAP) return RT_OK;
  if ((float)d.r1 != mo->geo[0] || (float)d.r2 != mo->geo[1] || (float)d.z0 != mo->geo[2] ||
      (float)d.z1 != mo->geo[3])
    return fail(RT_E_INVALID, "the cloaks' geometry (r1 %g, r2 %g, z %g..%g) is not the one the cap model was set "
                              "up for (r1 %g, r2 %g, z %g..%g)", d.r1, d.r2, d.z0, d.z1, mo->geo[0], mo->geo[1],
                mo->geo[2], mo->geo[3]);
  return RT_OK;
}

}  // namespace

int surrogate_check_ready(rt_model mo) {
  for (rt_model m = mo; m; m = m == mo ? mo->next : nullptr) {
    int e = check_model(m);
    if (e) return e;
    if (!m->map_valid)
      return fail(RT_E_INVALID, "the %smodel has no calibrated trust map (rt_surrogate_calibrate)",
                  m == mo ? "" : "chained ");
  }
  return RT_OK;
}

double surrogate_exit_tolerance(rt_model mo) {
  return mo->next ? std::max(mo->gate.tol, mo->next->gate.tol) : mo->gate.tol;
}

int surrogate_predict_gated(rt_model mo, const rt_cloak_desc &d, int64_t n, int64_t ld, const float *x6, float *y5,
                            uint8_t *fallback, int32_t *status, hipStream_t s) {
  int e = surrogate_check_ready(mo);
  if (!e) e = check_geometry(mo, d);
  if (!e && mo->next) e = check_geometry(mo->next, d);
  if (e) return e;
  if (n == 0) return RT_OK;
  if (n < 0 || ld < n || !x6 || !y5 || !fallback || !status)
    return fail(RT_E_INVALID, "bad rows for the surrogate (n, ld or a NULL array)");
  const long long batch = std::min<long long>(n, 1LL << 24);
  // the model, then the chained one on the rows the first rejected
  for (rt_model m = mo; m; m = m == mo ? mo->next : nullptr) {
    GateP gp;
    gp.a = (float)d.r1;
    gp.b = (float)d.r2;
    gp.z0 = std::isfinite(d.z0) ? (float)d.z0 : -INFINITY;
    gp.z1 = std::isfinite(d.z1) ? (float)d.z1 : INFINITY;
    gp.hres_max = (float)m->gate.hres_max;
    gp.cap_margin = (float)m->gate.cap_margin;
    gp.p_min = (float)m->gate.p_min;
    const JobP jp = job_for(m, &d);
    e = reserve_yinf(m, batch);
    if (e) return e;
    for (long long off = 0; off < n; off += batch) {
      const int rows = (int)std::min<long long>(batch, n - off);
      const float *x = x6 + off;
      // entries that pass the input gate only go through the network
      // (compacted), then the output half of the gate
      hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, m->count, 1LL);
      hipLaunchKernelGGL(k_pregate, dim3(gblocks(rows, 256)), dim3(256), 0, s, x, (long long)ld, rows, m->map, gp, jp,
                         m == mo ? 0 : 1, fallback + off, m->idx, m->count);
      hipLaunchKernelGGL(k_mlp_fused, dim3(gblocks(rows, FR)), dim3(256), 0, s, x, (long long)ld, rows, m->idx,
                         m->count, m->P, m->Pb, m->scal, jp, m->yinf, nullptr, 0LL);
      hipLaunchKernelGGL(k_gate_idx, dim3(gblocks(rows, 256)), dim3(256), 0, s, x, (long long)ld, m->idx, m->count,
                         m->yinf, m->scal, m->map, gp, jp, y5 + off, fallback + off, status + off);
    }
  }
  return launch_err("surrogate launch");
}

extern "C" {

int rt_surrogate_create(uint64_t seed, rt_model *out) {
  if (!out) return fail(RT_E_INVALID, "out is NULL");
  *out = nullptr;
  rt_model mo = new (std::nothrow) rt_model_s;
  if (!mo) return fail(RT_E_NOMEM, "host allocation failed");
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t pb = al(sizeof(float) * NPARAM), bb = al(sizeof(bf16) * 2 * NBF), sb = al(sizeof(float) * NSCAL),
               mb = al(NCELLS), cb = al(sizeof(unsigned int) * 2 * NCELLS), ob = al(sizeof(double) * NMOM);
  const size_t bytes = 4 * pb + bb + sb + mb + cb + ob;
  if (hipMalloc(&mo->base, bytes) != hipSuccess) {
    (void)hipGetLastError();
    delete mo;
    return fail(RT_E_NOMEM, "hipMalloc of the model failed");
  }
  (void)hipGetDevice(&mo->device);
  char *c = (char *)mo->base;
  size_t off = 0;
  mo->P = (float *)(c + off); off += pb;
  mo->G = (float *)(c + off); off += pb;
  mo->m = (float *)(c + off); off += pb;
  mo->v = (float *)(c + off); off += pb;
  mo->Pb = (bf16 *)(c + off); off += bb;
  mo->scal = (float *)(c + off); off += sb;
  mo->map = (unsigned char *)(c + off); off += mb;
  mo->cal = (unsigned int *)(c + off); off += cb;
  mo->mom = (double *)(c + off); off += ob;
  // weights and biases uniform in +-1/sqrt(fan_in) from a seeded Mersenne
  // twister, drawn layer by layer (weights row-major, then biases)
  std::vector<float> h(NPARAM, 0.0f);
  std::mt19937_64 rng(seed);
  const int fan_in[5] = {NIN, HID, HID, HID, HID}, fan_out[5] = {HID, HID, HID, HID, NOUT};
  const long long offw[5] = {OFF_W1, OFF_W2, OFF_W3, OFF_W4, OFF_W5};
  const long long offb[5] = {OFF_B1, OFF_B2, OFF_B3, OFF_B4, OFF_B5};
  for (int l = 0; l < 5; ++l) {
    const float k = 1.0f / std::sqrt((float)fan_in[l]);
    std::uniform_real_distribution<float> U(-k, k);
    for (long long e = 0; e < (long long)fan_in[l] * fan_out[l]; ++e) h[offw[l] + e] = U(rng);
    for (int j = 0; j < fan_out[l]; ++j) h[offb[l] + j] = U(rng);
  }
  for (int k = 0; k < NIN; ++k) { mo->h_scal[S_INOFF + k] = 0.0f; mo->h_scal[S_INSCALE + k] = 1.0f; }
  for (int o = 0; o < NOUT; ++o) { mo->h_scal[S_OMEAN + o] = 0.0f; mo->h_scal[S_OSTD + o] = 1.0f; }
  mo->h_map.assign(NCELLS, 0);
  mo->gate.tol = 1e-3;
  mo->gate.hres_max = 1e-4;
  mo->gate.cap_margin = 1e-2;
  mo->gate.min_count = 8;
  mo->gate.p_min = 1e-4;
  bool ok = hipMemcpy(mo->P, h.data(), sizeof(float) * NPARAM, hipMemcpyHostToDevice) == hipSuccess &&
            upload_scal(mo) == RT_OK && upload_map(mo) == RT_OK;
  if (ok) {
    hipLaunchKernelGGL(k_fill, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->m, NPARAM, 0.0f);
    hipLaunchKernelGGL(k_fill, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->v, NPARAM, 0.0f);
    hipLaunchKernelGGL(k_refresh_bf16, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->P, mo->Pb);
    ok = hipDeviceSynchronize() == hipSuccess;
  }
  if (!ok) {
    (void)hipFree(mo->base);
    delete mo;
    return fail(RT_E_DEVICE, "model initialization failed");
  }
  *out = mo;
  return RT_OK;
}

int rt_surrogate_free(rt_model mo) {
  if (!mo) return RT_OK;
  (void)hipDeviceSynchronize();
  if (mo->prev) mo->prev->next = nullptr;
  if (mo->next) mo->next->prev = nullptr;
  if (mo->act) (void)hipFree(mo->act);
  if (mo->yinf) (void)hipFree(mo->yinf);
  if (mo->base) (void)hipFree(mo->base);
  delete mo;
  return RT_OK;
}

int rt_surrogate_nparams(int64_t *count) {
  if (!count) return fail(RT_E_INVALID, "count is NULL");
  *count = NPARAM;
  return RT_OK;
}

int rt_surrogate_get_params(rt_model mo, float *host) {
  int e = check_model(mo);
  if (e) return e;
  if (!host) return fail(RT_E_INVALID, "host is NULL");
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(host, mo->P, sizeof(float) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess)
    return fail(RT_E_DEVICE, "copy failed");
  return RT_OK;
}

int rt_surrogate_set_params(rt_model mo, const float *host) {
  int e = check_model(mo);
  if (e) return e;
  if (!host) return fail(RT_E_INVALID, "host is NULL");
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(mo->P, host, sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess)
    return fail(RT_E_DEVICE, "copy failed");
  hipLaunchKernelGGL(k_refresh_bf16, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->P, mo->Pb);
  hipLaunchKernelGGL(k_fill, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->m, NPARAM, 0.0f);
  hipLaunchKernelGGL(k_fill, dim3(gblocks(NPARAM, 256)), dim3(256), 0, 0, mo->v, NPARAM, 0.0f);
  if (hipDeviceSynchronize() != hipSuccess) return fail(RT_E_DEVICE, "refresh failed");
  mo->step = 0;
  return RT_OK;
}

int rt_surrogate_get_scaling(rt_model mo, float *scaling22) {
  int e = check_model(mo);
  if (e) return e;
  if (!scaling22) return fail(RT_E_INVALID, "scaling is NULL");
  memcpy(scaling22, mo->h_scal, sizeof(float) * S_LOSS);
  return RT_OK;
}

int rt_surrogate_set_scaling(rt_model mo, const float *scaling22) {
  int e = check_model(mo);
  if (e) return e;
  if (!scaling22) return fail(RT_E_INVALID, "scaling is NULL");
  for (int k = 0; k < S_LOSS; ++k)
    if (!std::isfinite(scaling22[k])) return fail(RT_E_INVALID, "scaling values must be finite");
  for (int o = 0; o < NOUT; ++o)
    if (!(scaling22[S_OSTD + o] > 0.0f)) return fail(RT_E_INVALID, "out_std must be > 0");
  memcpy(mo->h_scal, scaling22, sizeof(float) * S_LOSS);
  if (hipDeviceSynchronize() != hipSuccess) return fail(RT_E_DEVICE, "synchronize failed");
  return upload_scal(mo);
}

int rt_surrogate_fit_scaling(rt_model mo, int64_t n, int64_t ld, const float *x6, const float *t5, const float *w,
                             void *stream) {
  int e = check_model(mo);
  if (!e) e = check_rows(n, ld, x6);
  if (e) return e;
  if (!t5) return fail(RT_E_INVALID, "t5 is required");
  hipStream_t s = (hipStream_t)stream;
  double h[NMOM];
  hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, mo->mom, NMOM);
  hipLaunchKernelGGL(k_moments, dim3(std::min(gblocks(n, 256), 1024u)), dim3(256), 0, s, x6, t5, (long long)ld, w,
                     (int)n, job_for(mo, nullptr), mo->mom);
  if (hipMemcpyAsync(h, mo->mom, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return fail(RT_E_DEVICE, "moments failed");
  const double W = h[NMOM - 1];
  if (!(W > 0.0)) return fail(RT_E_INVALID, "no row has a nonzero weight");
  for (int k = 0; k < NIN + NOUT; ++k) {
    const double mean = h[2 * k] / W;
    const double var = std::max(0.0, h[2 * k + 1] / W - mean * mean);
    const double sd = std::sqrt(var);
    if (k < NIN) {
      mo->h_scal[S_INOFF + k] = (float)mean;
      mo->h_scal[S_INSCALE + k] = (float)(1.0 / std::max(sd, 1e-6));
    } else {
      mo->h_scal[S_OMEAN + (k - NIN)] = (float)mean;
      mo->h_scal[S_OSTD + (k - NIN)] = std::max((float)sd, OUT_STD_FLOOR);
    }
  }
  return upload_scal(mo);
}

int grad_impl(rt_model mo, int64_t n, int64_t ld, const float *x6, const float *t5, const float *w, float huber,
              float *grads, float *loss, void *stream);

int rt_surrogate_grad(rt_model mo, int64_t n, int64_t ld, const float *x6, const float *t5, const float *w,
                      float huber, float *grads, float *loss, void *stream) {
  if (!(huber >= 0.0f)) return fail(RT_E_INVALID, "huber must be >= 0");
  return grad_impl(mo, n, ld, x6, t5, w, huber, grads, loss, stream);
}

int grad_impl(rt_model mo, int64_t n, int64_t ld, const float *x6, const float *t5, const float *w, float huber,
              float *grads, float *loss, void *stream) {
  int e = check_model(mo);
  if (!e) e = check_rows(n, ld, x6);
  if (e) return e;
  if (!t5) return fail(RT_E_INVALID, "t5 is required");
  e = reserve_acts(mo, n);
  if (e) return e;
  hipStream_t s = (hipStream_t)stream;
  forward_backward(mo, x6, t5, ld, w, (int)n, huber, grads, loss, s);
  return launch_err("gradient launch");
}

int check_train_opts(const rt_train_opts *opts) {
  if (!opts) return fail(RT_E_INVALID, "opts is NULL");
  if (!(opts->lr >= 0.0f) || !(opts->beta1 >= 0.0f && opts->beta1 < 1.0f) ||
      !(opts->beta2 >= 0.0f && opts->beta2 < 1.0f) || !(opts->eps > 0.0f) || !(opts->weight_decay >= 0.0f) ||
      !(opts->huber >= 0.0f))
    return fail(RT_E_INVALID, "need lr >= 0, 0 <= beta1, beta2 < 1, eps > 0, weight_decay >= 0, huber >= 0");
  return RT_OK;
}

// one AdamW step with the gradient G (device, NPARAM floats); advances the
// step count that the bias corrections use
int adamw_step(rt_model mo, const float *G, const rt_train_opts *opts, hipStream_t s) {
  mo->step += 1;
  // bias corrections 1 - beta^t formed in FP64 and rounded once: 1 - beta2^t
  // cancels for early steps (0.039 at beta2 = 0.995, t = 8), and rounding
  // beta2^t to FP32 first would cost it 2^-24 / 0.039 relative
  const float c1 = (float)(1.0 - std::pow((double)opts->beta1, (double)mo->step));
  const float c2 = (float)(1.0 - std::pow((double)opts->beta2, (double)mo->step));
  hipLaunchKernelGGL(k_adamw, dim3(gblocks(NPARAM, 256)), dim3(256), 0, s, mo->P, G, mo->m, mo->v, mo->Pb,
                     opts->lr, opts->weight_decay, opts->beta1, opts->beta2, c1, c2, opts->eps);
  return launch_err("optimizer launch");
}

int rt_surrogate_train(rt_model mo, int64_t n, int64_t ld, const float *x6, const float *t5, const float *w,
                       const rt_train_opts *opts, float *loss, void *stream) {
  int e = check_train_opts(opts);
  if (e) return e;
  e = grad_impl(mo, n, ld, x6, t5, w, opts->huber, nullptr, loss, stream);
  if (e) return e;
  return adamw_step(mo, mo->G, opts, (hipStream_t)stream);
}

int rt_surrogate_step(rt_model mo, const float *grads, const rt_train_opts *opts, void *stream) {
  int e = check_model(mo);
  if (!e) e = check_train_opts(opts);
  if (e) return e;
  if (!grads) return fail(RT_E_INVALID, "grads is NULL");
  return adamw_step(mo, grads, opts, (hipStream_t)stream);
}

int rt_surrogate_get_state(rt_model mo, float *m_host, float *v_host, int64_t *step) {
  int e = check_model(mo);
  if (e) return e;
  if (hipDeviceSynchronize() != hipSuccess) return fail(RT_E_DEVICE, "synchronize failed");
  if ((m_host && hipMemcpy(m_host, mo->m, sizeof(float) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess) ||
      (v_host && hipMemcpy(v_host, mo->v, sizeof(float) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess))
    return fail(RT_E_DEVICE, "copy failed");
  if (step) *step = mo->step;
  return RT_OK;
}

int rt_surrogate_set_state(rt_model mo, const float *m_host, const float *v_host, int64_t step) {
  int e = check_model(mo);
  if (e) return e;
  if (!m_host || !v_host) return fail(RT_E_INVALID, "m and v are required");
  if (step < 0) return fail(RT_E_INVALID, "step must be >= 0");
  for (long long i = 0; i < NPARAM; ++i)
    if (!std::isfinite(m_host[i]) || !(v_host[i] >= 0.0f) || !std::isfinite(v_host[i]))
      return fail(RT_E_INVALID, "moments must be finite and v >= 0 (entry %lld)", i);
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(mo->m, m_host, sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(mo->v, v_host, sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess)
    return fail(RT_E_DEVICE, "copy failed");
  mo->step = step;
  return RT_OK;
}

int rt_surrogate_forward(rt_model mo, int64_t n, int64_t ld, const float *x6, float *t5, void *stream) {
  int e = check_model(mo);
  if (!e) e = check_rows(n, ld, x6);
  if (e) return e;
  if (!t5) return fail(RT_E_INVALID, "t5 is required");
  infer_outputs(mo, x6, ld, (int)n, t5, ld, (hipStream_t)stream);
  return launch_err("forward launch");
}

int rt_surrogate_encode_job(int32_t job, const rt_cloak *cloaks, int32_t n_cloaks, int64_t n, int64_t ld,
                            const float *x6, const float *y5, const int32_t *status, float *t5, float *w,
                            void *stream) {
  rt_cloak_desc d;
  int e = cloak_geometry(cloaks, n_cloaks, d);
  if (e) return e;
  if (job != RT_SUR_SIDE && job != RT_SUR_CAP) return fail(RT_E_INVALID, "job must be RT_SUR_SIDE or RT_SUR_CAP");
  if (job == RT_SUR_CAP && (!std::isfinite(d.z0) || !std::isfinite(d.z1) || !(d.z1 > d.z0)))
    return fail(RT_E_INVALID, "the cap job needs cloaks of finite height");
  if (n == 0) return RT_OK;
  e = check_rows(n, ld, x6);
  if (e) return e;
  if (!y5 || !status || !t5 || !w) return fail(RT_E_INVALID, "y5, status, t5 and w are required");
  if (job == RT_SUR_CAP) {
    const JobP jp{RT_SUR_CAP, (float)d.r1, (float)d.r2, (float)d.z0, (float)d.z1};
    hipLaunchKernelGGL(k_encode_cap, dim3(gblocks(n, 256)), dim3(256), 0, (hipStream_t)stream, x6, y5, status,
                       (long long)ld, (long long)n, jp, t5, w);
  } else {
    hipLaunchKernelGGL(k_encode, dim3(gblocks(n, 256)), dim3(256), 0, (hipStream_t)stream, x6, y5, status,
                       (long long)ld, (long long)n, (float)d.r1, (float)d.r2, t5, w);
  }
  return launch_err("encode launch");
}

int rt_surrogate_encode(const rt_cloak *cloaks, int32_t n_cloaks, int64_t n, int64_t ld, const float *x6,
                        const float *y5, const int32_t *status, float *t5, float *w, void *stream) {
  return rt_surrogate_encode_job(RT_SUR_SIDE, cloaks, n_cloaks, n, ld, x6, y5, status, t5, w, stream);
}

int rt_surrogate_calibrate(rt_model mo, const rt_cloak *cloaks, int32_t n_cloaks, int64_t n, int64_t ld,
                           const float *x6, const float *y5_exact, const int32_t *status_exact,
                           const float *hres_exact, const rt_gate_opts *gate, double *trusted_fraction,
                           void *stream) {
  int e = check_model(mo);
  if (e) return e;
  rt_cloak_desc d;
  e = cloak_geometry(cloaks, n_cloaks, d);
  if (!e) e = check_geometry(mo, d);
  if (!e) e = check_rows(n, ld, x6);
  if (e) return e;
  if (!y5_exact || !status_exact || !gate) return fail(RT_E_INVALID, "y5_exact, status_exact and gate are required");
  if (!(gate->tol > 0.0) || !(gate->hres_max > 0.0) || !(gate->cap_margin >= 0.0) || gate->min_count < 1 ||
      gate->dilate < 0 || gate->dilate > 8 || (hres_exact && !(gate->unresolved > 0.0)) ||
      !(gate->p_min >= 0.0 && gate->p_min < 1.0))
    return fail(RT_E_INVALID, "gate needs tol > 0, hres_max > 0, cap_margin >= 0, min_count >= 1, "
                              "0 <= dilate <= 8, 0 <= p_min < 1 and, with hres_exact, unresolved > 0");
  e = reserve_yinf(mo, n);
  if (e) return e;
  hipStream_t s = (hipStream_t)stream;
  infer_outputs(mo, x6, ld, (int)n, nullptr, 0, s);
  hipLaunchKernelGGL(k_fill_u32, dim3(gblocks(2LL * NCELLS, 256)), dim3(256), 0, s, mo->cal, 2LL * NCELLS);
  hipLaunchKernelGGL(k_calib, dim3(gblocks(n, 256)), dim3(256), 0, s, x6, (long long)ld, (int)n, mo->yinf, mo->scal,
                     y5_exact, status_exact, hres_exact, (float)gate->unresolved,
                     !std::isfinite(d.z0) && !std::isfinite(d.z1), job_for(mo, &d), (float)gate->cap_margin, mo->cal,
                     mo->cal + NCELLS);
  std::vector<unsigned int> h(2 * NCELLS);
  if (hipMemcpyAsync(h.data(), mo->cal, sizeof(unsigned int) * 2 * NCELLS, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return fail(RT_E_DEVICE, "calibration failed");
  std::vector<unsigned char> good(NCELLS);
  for (int c = 0; c < NCELLS; ++c) {
    float mx;
    memcpy(&mx, &h[c], sizeof(float));
    good[c] = h[NCELLS + c] >= (unsigned int)gate->min_count && mx <= (float)gate->tol;
  }
  // dilation within each (axis, branch) block over the cell grid's
  // dimensions: (alpha, beta) for the side job, (alpha, |beta|, u) for the
  // cap job
  const int dl = gate->dilate;
  const bool capj = mo->job == RT_SUR_CAP;
  const int na = capj ? CAP_A : NCELL_A, nb = capj ? CAP_B : NCELL_B, nu = capj ? CAP_U : 1;
  const int du = capj ? dl : 0;
  long long trusted = 0;
  for (int k = 0; k < NCOMBO; ++k)
    for (int ia = 0; ia < na; ++ia)
      for (int ib = 0; ib < nb; ++ib)
        for (int iu = 0; iu < nu; ++iu) {
          bool ok = true;
          for (int da = -dl; da <= dl && ok; ++da)
            for (int db = -dl; db <= dl && ok; ++db)
              for (int dv = -du; dv <= du && ok; ++dv) {
                const int ja = ia + da, jb = ib + db, ju = iu + dv;
                if (ja < 0 || ja >= na || jb < 0 || jb >= nb || ju < 0 || ju >= nu) continue;
                ok = good[((k * na + ja) * nb + jb) * nu + ju] != 0;
              }
          mo->h_map[((k * na + ia) * nb + ib) * nu + iu] = ok ? 1 : 0;
          trusted += ok;
        }
  mo->gate = *gate;
  mo->map_valid = 1;
  if (trusted_fraction) *trusted_fraction = (double)trusted / NCELLS;
  return upload_map(mo);
}

int rt_surrogate_get_map(rt_model mo, uint8_t *host, int32_t *cells_alpha, int32_t *cells_beta, int32_t *cells_u) {
  int e = check_model(mo);
  if (e) return e;
  const bool capj = mo->job == RT_SUR_CAP;
  if (cells_alpha) *cells_alpha = capj ? CAP_A : NCELL_A;
  if (cells_beta) *cells_beta = capj ? CAP_B : NCELL_B;
  if (cells_u) *cells_u = capj ? CAP_U : 1;
  if (host) memcpy(host, mo->h_map.data(), NCELLS);
  return RT_OK;
}

int rt_surrogate_set_job(rt_model mo, int32_t job, rt_cloak cloak) {
  int e = check_model(mo);
  if (e) return e;
  if (job != RT_SUR_SIDE && job != RT_SUR_CAP) return fail(RT_E_INVALID, "job must be RT_SUR_SIDE or RT_SUR_CAP");
  float geo[4] = {0.f, 0.f, 0.f, 0.f};
  if (job == RT_SUR_CAP) {
    rt_cloak_desc d;
    if (!cloak || rt_cloak_get_desc(cloak, &d) != RT_OK) return fail(RT_E_INVALID, "the cap job needs a cloak handle");
    if (!std::isfinite(d.z0) || !std::isfinite(d.z1) || !(d.z1 > d.z0))
      return fail(RT_E_INVALID, "the cap job needs a cloak of finite height");
    geo[0] = (float)d.r1;
    geo[1] = (float)d.r2;
    geo[2] = (float)d.z0;
    geo[3] = (float)d.z1;
  }
  mo->job = job;
  memcpy(mo->geo, geo, sizeof(geo));
  // the cells of the trust map change meaning
  std::fill(mo->h_map.begin(), mo->h_map.end(), 0);
  mo->map_valid = 0;
  return upload_map(mo);
}

int rt_surrogate_get_job(rt_model mo, int32_t *job) {
  int e = check_model(mo);
  if (e) return e;
  if (!job) return fail(RT_E_INVALID, "job is NULL");
  *job = mo->job;
  return RT_OK;
}

int rt_surrogate_chain(rt_model first, rt_model next) {
  int e = check_model(first);
  if (e) return e;
  if (next) {
    e = check_model(next);
    if (e) return e;
    if (next == first) return fail(RT_E_INVALID, "a model cannot follow itself");
    if (next->next || first->prev) return fail(RT_E_INVALID, "chains hold two models");
    if (next->prev && next->prev != first) return fail(RT_E_INVALID, "next already follows another model");
  }
  if (first->next) first->next->prev = nullptr;
  first->next = next;
  if (next) next->prev = first;
  return RT_OK;
}

int rt_surrogate_infer(rt_model mo, const rt_cloak *cloaks, int32_t n_cloaks, const rt_trace_opts *opts, int64_t n,
                       int64_t ld, const float *x6, float *y5, uint8_t *fallback, int32_t *status, void *stream) {
  int e = check_model(mo);
  if (e) return e;
  rt_cloak_desc d;
  e = cloak_geometry(cloaks, n_cloaks, d);
  if (e) return e;
  if (!opts) return fail(RT_E_INVALID, "opts is NULL");
  if (n == 0) return RT_OK;
  e = check_rows(n, ld, x6);
  if (e) return e;
  if (!y5 || !fallback || !status) return fail(RT_E_INVALID, "y5, fallback and status are required");
  e = surrogate_predict_gated(mo, d, n, ld, x6, y5, fallback, status, (hipStream_t)stream);
  if (e) return e;
  // the exact integrator traces the rejected rays (one persistent launch)
  return rt_transit_exact(cloaks, n_cloaks, opts, n, ld, x6, fallback, y5, status, nullptr, nullptr, stream);
}

int rt_surrogate_save(rt_model mo, const char *path) {
  int e = check_model(mo);
  if (e) return e;
  if (!path) return fail(RT_E_INVALID, "path is NULL");
  std::vector<float> h(NPARAM);
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(h.data(), mo->P, sizeof(float) * NPARAM, hipMemcpyDeviceToHost) != hipSuccess)
    return fail(RT_E_DEVICE, "copy failed");
  FILE *f = fopen(path, "wb");
  if (!f) return fail(RT_E_INVALID, "cannot open %s", path);
  const char magic[8] = {'R', 'T', 'M', 'L', 'P', '0', '5', '\0'};
  const long long np = NPARAM, nc = NCELLS;
  const int valid = mo->map_valid;
  bool ok = fwrite(magic, 1, 8, f) == 8 && fwrite(&np, sizeof(np), 1, f) == 1 &&
            fwrite(mo->h_scal, sizeof(float), S_LOSS, f) == (size_t)S_LOSS &&
            fwrite(h.data(), sizeof(float), NPARAM, f) == (size_t)NPARAM && fwrite(&nc, sizeof(nc), 1, f) == 1 &&
            fwrite(&valid, sizeof(valid), 1, f) == 1 && fwrite(&mo->gate, sizeof(mo->gate), 1, f) == 1 &&
            fwrite(mo->h_map.data(), 1, NCELLS, f) == (size_t)NCELLS && fwrite(&mo->job, sizeof(int), 1, f) == 1 &&
            fwrite(mo->geo, sizeof(float), 4, f) == 4;
  ok = (fclose(f) == 0) && ok;
  return ok ? RT_OK : fail(RT_E_INVALID, "write to %s failed", path);
}

int rt_surrogate_load(const char *path, rt_model *out) {
  if (!path || !out) return fail(RT_E_INVALID, "path and out are required");
  *out = nullptr;
  FILE *f = fopen(path, "rb");
  if (!f) return fail(RT_E_INVALID, "cannot open %s", path);
  char magic[8];
  long long np = 0, nc = 0;
  int valid = 0, job = RT_SUR_SIDE;
  float scal[S_LOSS], geo[4];
  rt_gate_opts gate;
  std::vector<float> h(NPARAM);
  std::vector<unsigned char> map(NCELLS);
  bool ok = fread(magic, 1, 8, f) == 8 && memcmp(magic, "RTMLP05", 8) == 0 && fread(&np, sizeof(np), 1, f) == 1 &&
            np == NPARAM && fread(scal, sizeof(float), S_LOSS, f) == (size_t)S_LOSS &&
            fread(h.data(), sizeof(float), NPARAM, f) == (size_t)NPARAM && fread(&nc, sizeof(nc), 1, f) == 1 &&
            nc == NCELLS && fread(&valid, sizeof(valid), 1, f) == 1 && fread(&gate, sizeof(gate), 1, f) == 1 &&
            fread(map.data(), 1, NCELLS, f) == (size_t)NCELLS && fread(&job, sizeof(int), 1, f) == 1 &&
            fread(geo, sizeof(float), 4, f) == 4 && (job == RT_SUR_SIDE || job == RT_SUR_CAP);
  fclose(f);
  if (!ok) return fail(RT_E_INVALID, "%s is not a surrogate file of this layout", path);
  rt_model mo = nullptr;
  int e = rt_surrogate_create(0, &mo);
  if (e) return e;
  e = rt_surrogate_set_scaling(mo, scal);
  if (!e) e = rt_surrogate_set_params(mo, h.data());
  if (!e) {
    mo->h_map = map;
    mo->map_valid = valid;
    mo->gate = gate;
    mo->job = job;
    memcpy(mo->geo, geo, sizeof(geo));
    e = upload_map(mo);
  }
  if (e) {
    rt_surrogate_free(mo);
    return e;
  }
  *out = mo;
  return RT_OK;
}

}  // extern "C"
