// Device-side physics of one element for the TLED + Pennes step, single
// precision, written in "small quantities" so that nothing is formed by
// subtracting nearly equal O(1) numbers:
//   - the displacement gradient H = F - I is kept, not F;
//   - the elastic part is H_e = F_e - I, twice the Green strain
//     G = C - I = H_e + H_e^T + H_e^T H_e;
//   - J - 1 = tr H + i2(H) + det H (exact expansion of det(I + H));
//   - J^(-2/3) - 1 = expm1(-2/3 log1p(J - 1));
//   - N = I - C^-1 = (G - adj G + (det C - 1 - tr G) I) / det C, det C = J^2
//     (adj(I + G) = I + tr G I - G + adj G): every term is of the order of the
//     strain, so N keeps its relative accuracy, and C^-1 = I - N;
//   - I - I1/3 C^-1 = 2 C^-1 dev E = N (1 + tr G / 3) - (tr G / 3) I and
//     I4bar - 1 = (J^-2/3 - 1) + J^-2/3 a.G.a.
// Algebraically these are the textbook forms of the Table 5 model (Eq. 9)
// evaluated on the elastic deformation (Eq. 8) and pulled back (Eq. 10).
// The T4 patch kernel is limited by vector instruction issue (80 % of its issue
// slots at 732 instructions per element when S was formed from C^-1 dev E by
// matrix products and the conduction tensor from the total C): with N the stress
// is two scalars times N and I, and for isotropic expansion the same N serves the
// conduction, which leaves 548 (1M-tet ellipsoid: 28.5 -> 26.4 us per launch, 69 %
// of the issue slots; the rest is memory and LDS latency).  Taking the strain of an
// isotropically heated element from the total gradient, with the thermal part
// subtracted from the invariants, needs no fewer and loses accuracy: at a thermal
// strain of 1e-2 and an elastic one of 1e-4 the stress error rose from 7.0e-6 to
// 1.0e-5 of the stress, under a shrinkage of -0.05 from 3.5e-6 to 7.2e-6.
#pragma once

#include <hip/hip_runtime.h>

namespace tled {

// Kernel-side material constants (single precision, derived on the host).
struct KMat {
    float mu, kappa, eta;         // moduli at T0
    float alpha, alpha_m, alpha_n; // expansion coefficients (alpha_m: along the fibre m, alpha_n: along n)
    float k, k_m;                 // conductivities
    // Temperature laws are evaluated on the rise dT = T - T0 with the ramp start
    // as an offset from T0 formed in FP64 on the host (off = T0 - T_start): an
    // absolute temperature in FP32 is quantised to 3e-5 K near 310 K, which the
    // steep shrinkage ramp would turn into strain errors.
    float muT_off, muT_inv, muT_drop;
    float sh_off, sh_inv, sh_eps;
    float ck_off, ck_inv;         // c(T), k(T) ramp
    float c_lo, c_hi, kr_hi;      // c at lo/hi; k_hi / k
    float pc1[4], pc2[4];         // Prony: dt g/(dt + tau), tau/(dt + tau)
    float hgk;                    // hourglass: hg_coef (kappa + 4 mu / 3)
    int n_prony;
    int expan_mode, cond_mode, muT_on, shrink_on, ckT_on;
};

// Expansion and conduction modes compiled into a kernel: isotropic only; also transversely
// isotropic about the fibre; also orthotropic expansion and tensor conduction.
constexpr int kIso = 0, kTi = 1, kOrtho = 2;

struct Sym3 {
    float xx, yy, zz, xy, yz, xz;
};

__device__ __forceinline__ float clamp01f(float x) { return fminf(fmaxf(x, 0.0f), 1.0f); }

// Hardware reciprocal (v_rcp_f32, within 1 ulp).  Every reciprocal here is of a
// quantity near 1 or of a well-scaled determinant, so the IEEE division
// sequence is not needed.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// (1 + x)^(-2/3) - 1.  Binomial series to x^5 for |x| < 0.02 (truncation below
// 3e-11, i.e. < 3e-9 relative).  Up to |x| = 0.5 (thermal shrinkage) one Newton step
// on (1 + w)^3 (1 + x)^2 = 1 from the hardware base-2 exponential and logarithm, with
// both powers in small quantities (P = (1 + w)^3 - 1, Q = (1 + x)^2 - 1, residual
// P + Q + P Q), which leaves the rounding of the residual, an ulp of w; it takes 15
// instructions where expm1(-2/3 log1p(x)) takes 154.  Beyond, that form.
__device__ __forceinline__ float pow_m23_m1(float x) {
    float w = x * (-2.0f / 3.0f +
                   x * (5.0f / 9.0f + x * (-40.0f / 81.0f + x * (110.0f / 243.0f + x * (-308.0f / 729.0f)))));
    if (!(fabsf(x) < 0.02f)) {
        if (fabsf(x) < 0.5f) {
            w = __builtin_amdgcn_exp2f((-2.0f / 3.0f) * __builtin_amdgcn_logf(1.0f + x)) - 1.0f;
            const float P = w * (3.0f + w * (3.0f + w)), Q = x * (2.0f + x);
            w -= (P + Q + P * Q) * (1.0f + w) * (1.0f / 3.0f);
        } else {
            w = expm1f(-(2.0f / 3.0f) * log1pf(x));
        }
    }
    return w;
}

// (J - 1) of I + A from the invariants of A.
__device__ __forceinline__ float det_m1(const float A[9]) {
    const float m0 = A[4] * A[8] - A[5] * A[7];
    const float i2 = m0 + A[0] * A[8] - A[2] * A[6] + A[0] * A[4] - A[1] * A[3];
    const float i3 = A[0] * m0 - A[1] * (A[3] * A[8] - A[5] * A[6]) + A[2] * (A[3] * A[7] - A[4] * A[6]);
    return A[0] + A[4] + A[8] + (i2 + i3);
}

// G = C - I = A + A^T + A^T A for the displacement gradient A of a deformation I + A.
__device__ __forceinline__ Sym3 strain2(const float A[9]) {
    return Sym3{A[0] * A[0] + A[3] * A[3] + A[6] * A[6] + 2.0f * A[0],
                A[1] * A[1] + A[4] * A[4] + A[7] * A[7] + 2.0f * A[4],
                A[2] * A[2] + A[5] * A[5] + A[8] * A[8] + 2.0f * A[8],
                A[1] + A[3] + A[0] * A[1] + A[3] * A[4] + A[6] * A[7],
                A[5] + A[7] + A[1] * A[2] + A[4] * A[5] + A[7] * A[8],
                A[2] + A[6] + A[0] * A[2] + A[3] * A[5] + A[6] * A[8]};
}

// N = I - (I + G)^-1 for det(I + G) = J^2, J = 1 + Jm1.
__device__ __forceinline__ Sym3 one_minus_inverse(const Sym3 &G, float Jm1, float trG) {
    const float J = 1.0f + Jm1;
    const float w = rcp(J * J);
    const float s = Jm1 * (2.0f + Jm1) - trG;
    return Sym3{w * (s + G.xx + G.yz * G.yz - G.yy * G.zz), w * (s + G.yy + G.xz * G.xz - G.xx * G.zz),
                w * (s + G.zz + G.xy * G.xy - G.xx * G.yy), w * (G.xy + G.xy * G.zz - G.xz * G.yz),
                w * (G.yz + G.xx * G.yz - G.xy * G.xz), w * (G.xz + G.xz * G.yy - G.xy * G.yz)};
}

// scale (I - N) g: the pulled-back conduction of an isotropic tensor.
__device__ __forceinline__ void inverse_apply(const Sym3 &N, const float g[3], float scale, float q[3]) {
    q[0] = scale * (g[0] - N.xx * g[0] - N.xy * g[1] - N.xz * g[2]);
    q[1] = scale * (g[1] - N.xy * g[0] - N.yy * g[1] - N.yz * g[2]);
    q[2] = scale * (g[2] - N.xz * g[0] - N.yz * g[1] - N.zz * g[2]);
}

// Result of the per-element physics: PV = V0 F S~ (first Piola times volume,
// row-major 3x3), qV = V0 K0 grad T (pulled-back heat flux times volume),
// psiV = V0 det(Fth) Psi (only when requested), Jmin = min(det F, J_el).
struct ElemOut {
    float PV[9];
    float qV[3];
    float psiV;
    float Jmin;
};

// Thermal stretch (Section 3.2): lambda - 1 = alpha dT for the expansion
// coefficient of one axis, times the optional shrinkage factor.
__device__ __forceinline__ float stretch_m1(const KMat &m, float alpha, float dTe) {
    float a = alpha * dTe;
    if (m.shrink_on) {
        const float s1 = m.sh_eps * clamp01f((dTe + m.sh_off) * m.sh_inv);
        a = a + s1 + s1 * a;
    }
    return a;
}

// Octahedral decoding of a unit vector stored as two floats.
__device__ __forceinline__ void oct_decode(float x, float y, float a[3]) {
    float z = 1.0f - fabsf(x) - fabsf(y);
    float t = fmaxf(-z, 0.0f);
    x -= copysignf(t, x);
    y -= copysignf(t, y);
    float r = rsqrtf(x * x + y * y + z * z);
    a[0] = x * r; a[1] = y * r; a[2] = z * r;
}

// He += beta (F v) (x) v for a unit axis v (F = I + H): one axis term of
// F F_th^-1 with F_th^-1 = I / lambda_i + sum_v beta_v v (x) v (Eq. 11).
__device__ __forceinline__ void add_axis_term(float He[9], const float H[9], const float v[3], float beta) {
    const float Fv[3] = {v[0] + H[0] * v[0] + H[1] * v[1] + H[2] * v[2],
                         v[1] + H[3] * v[0] + H[4] * v[1] + H[5] * v[2],
                         v[2] + H[6] * v[0] + H[7] * v[1] + H[8] * v[2]};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) He[3 * i + j] += beta * Fv[i] * v[j];
}

// Per-element physics.  H: displacement gradient (row-major), gT: reference
// temperature gradient, dTe: element temperature rise over T0, a: unit fibre,
// theta: Prony state (n_prony x 6, updated in place), aniso + 2 e: the
// element's two float4 of anisotropy data (second expansion axis in
// octahedral coordinates, conductivity tensor: (n.x, n.y, Dxx, Dyy),
// (Dzz, Dxy, Dyz, Dxz)), read only inside the orthotropic expansion and tensor
// conduction branches.  MODE (kIso, kTi, kOrtho) says which expansion and conduction
// modes are compiled in: every mode a problem does not use costs registers in the
// others' code (the H8 patch kernel takes 127 VGPRs with kIso and 126 with kTi, the
// T4 one with two Prony terms 88 and 93; 64^3 H8 cube: 16.7 -> 14.9 us per launch
// against all modes in one kernel that spilled).
template <int NP, int MODE>
__device__ __forceinline__ void element_physics(const KMat &m, const float H[9], const float gT[3],
                                                float dTe, const float a[3], float V0, float *theta,
                                                bool want_psi, ElemOut &o, const float4 *__restrict__ aniso,
                                                int e) {
    constexpr bool ANISO = MODE == kOrtho;
    const int expan_mode = MODE == kIso ? 0 : m.expan_mode, cond_mode = MODE == kIso ? 0 : m.cond_mode;
    // ---- conduction with the total F, Eq. 16: qV = V0 J F^-1 D F^-T grad T
    float kscale = 1.0f;
    if (m.ckT_on) kscale = 1.0f + clamp01f((dTe + m.ck_off) * m.ck_inv) * (m.kr_hi - 1.0f);
    const bool iso = cond_mode == 0 && expan_mode == 0;   // then from the N of the stress below
    float Jt;
    if (!iso) {
        const float Jt1 = det_m1(H);
        Jt = 1.0f + Jt1;
        if (cond_mode == 0) {
            const Sym3 Gt = strain2(H);
            const Sym3 Nt = one_minus_inverse(Gt, Jt1, Gt.xx + Gt.yy + Gt.zz);
            inverse_apply(Nt, gT, V0 * m.k * kscale * Jt, o.qV);
        } else {
            // adj(F) D adj(F)^T gT / J, from the right
            const float F[9] = {1.0f + H[0], H[1], H[2], H[3], 1.0f + H[4], H[5], H[6], H[7], 1.0f + H[8]};
            const float Ad[9] = {F[4] * F[8] - F[5] * F[7], F[2] * F[7] - F[1] * F[8], F[1] * F[5] - F[2] * F[4],
                                 F[5] * F[6] - F[3] * F[8], F[0] * F[8] - F[2] * F[6], F[2] * F[3] - F[0] * F[5],
                                 F[3] * F[7] - F[4] * F[6], F[1] * F[6] - F[0] * F[7], F[0] * F[4] - F[1] * F[3]};
            float y[3], z[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) y[j] = Ad[j] * gT[0] + Ad[3 + j] * gT[1] + Ad[6 + j] * gT[2];
            const float f = V0 * kscale * rcp(Jt);
            if (!ANISO || cond_mode == 1) {
                // D = k I + (k_m - k) a a
                const float ay = (m.k_m - m.k) * (a[0] * y[0] + a[1] * y[1] + a[2] * y[2]);
#pragma unroll
                for (int j = 0; j < 3; ++j) z[j] = f * (m.k * y[j] + ay * a[j]);
            } else {
                // the element's tensor D (times k(T)/k)
                const float4 d0 = aniso[2 * size_t(e)], d1 = aniso[2 * size_t(e) + 1];
                z[0] = f * (d0.z * y[0] + d1.y * y[1] + d1.w * y[2]);
                z[1] = f * (d1.y * y[0] + d0.w * y[1] + d1.z * y[2]);
                z[2] = f * (d1.w * y[0] + d1.z * y[1] + d1.x * y[2]);
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) o.qV[i] = Ad[3 * i] * z[0] + Ad[3 * i + 1] * z[1] + Ad[3 * i + 2] * z[2];
        }
    }
    // ---- thermal split, Eqs. 7-8, 11: A = F_e - I
    const float li1 = stretch_m1(m, m.alpha, dTe);
    const float li = 1.0f + li1, inv_li = rcp(li);
    float A[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) A[i] = H[i] * inv_li;
    A[0] -= li1 * inv_li;
    A[4] -= li1 * inv_li;
    A[8] -= li1 * inv_li;
    float beta = 0.0f, lm = 1.0f;
    if (expan_mode != 0) {
        // F_e = F/li + b_m (F m) (x) m [+ b_n (F n) (x) n], b = 1/l - 1/li = (li1 - l1)/(li l)
        const float lm1 = stretch_m1(m, m.alpha_m, dTe);
        lm = 1.0f + lm1;
        beta = (li1 - lm1) * inv_li * rcp(lm);
        add_axis_term(A, H, a, beta);
        if (ANISO && expan_mode == 2) {
            float nv[3];
            const float4 q = aniso[2 * size_t(e)];
            oct_decode(q.x, q.y, nv);
            const float ln1 = stretch_m1(m, m.alpha_n, dTe);
            add_axis_term(A, H, nv, (li1 - ln1) * inv_li * rcp(1.0f + ln1));
        }
    }
    // ---- elastic strain and stress S_i (Eq. 9)
    const Sym3 G = strain2(A);
    const float Jm1 = det_m1(A);
    const float J = 1.0f + Jm1;
    const float trG = G.xx + G.yy + G.zz;
    const Sym3 N = one_minus_inverse(G, Jm1, trG);
    if (iso) {   // F = l_i F_e: J F^-1 F^-T = l_i J_e C_e^-1
        const float Jl = J * li;
        Jt = Jl * (li * li);
        inverse_apply(N, gT, V0 * m.k * kscale * Jl, o.qV);
    }
    const Sym3 aa{a[0] * a[0], a[1] * a[1], a[2] * a[2], a[0] * a[1], a[1] * a[2], a[0] * a[2]};
    float scale = 1.0f;
    if (m.muT_on) scale = 1.0f - m.muT_drop * clamp01f((dTe + m.muT_off) * m.muT_inv);
    const float mu = m.mu * scale, eta = m.eta * scale;
    const float aGa = 2.0f * (G.xy * aa.xy + G.yz * aa.yz + G.xz * aa.xz) + G.xx * aa.xx + G.yy * aa.yy + G.zz * aa.zz;
    const float j23m1 = pow_m23_m1(Jm1);
    const float j23 = 1.0f + j23m1;
    const float I4 = 1.0f + aGa;
    const float I4b1 = j23m1 + j23 * aGa;  // I4bar - 1
    const float ciso = mu * j23;
    const float cvol = m.kappa * J * Jm1;
    // S_i = cN N + cI I + cA a (x) a: mu J^-2/3 (I - I1/3 C^-1), the fibre term and kappa J (J - 1) C^-1;
    // with isotropic expansion the pull-back det(Fth) / l_i^2 = l_i (Eq. 10) goes into the scalars
    float cA = 2.0f * eta * I4b1 * j23;
    const float cfc = cvol - cA * I4 * (1.0f / 3.0f);
    const float t3 = trG * (1.0f / 3.0f);
    float cN = ciso * (1.0f + t3) - cfc, cI = cfc - ciso * t3;
    if (expan_mode == 0) {
        cA *= li;
        cI *= li;
        cN *= li;
    }
    Sym3 S;
    S.xx = cA * aa.xx + (cN * N.xx + cI);
    S.yy = cA * aa.yy + (cN * N.yy + cI);
    S.zz = cA * aa.zz + (cN * N.zz + cI);
    S.xy = cA * aa.xy + cN * N.xy;
    S.yz = cA * aa.yz + cN * N.yz;
    S.xz = cA * aa.xz + cN * N.xz;
    // ---- pull-back, Eq. 10
    float detFth;
    if (expan_mode == 0) {
        detFth = li * li * li;   // S already holds the pull-back
    } else if (!ANISO) {
        // det(Fth) Fth^-1 S Fth^-T, Fth^-1 = I/li + beta a(x)a
        detFth = li * li * lm;
        float Sa[3] = {S.xx * a[0] + S.xy * a[1] + S.xz * a[2], S.xy * a[0] + S.yy * a[1] + S.yz * a[2],
                       S.xz * a[0] + S.yz * a[1] + S.zz * a[2]};
        float aSa = a[0] * Sa[0] + a[1] * Sa[1] + a[2] * Sa[2];
        float c0 = detFth * inv_li * inv_li, c1 = detFth * beta * inv_li, c2 = detFth * beta * beta * aSa;
        S = Sym3{c0 * S.xx + c1 * 2.0f * a[0] * Sa[0] + c2 * a[0] * a[0],
                 c0 * S.yy + c1 * 2.0f * a[1] * Sa[1] + c2 * a[1] * a[1],
                 c0 * S.zz + c1 * 2.0f * a[2] * Sa[2] + c2 * a[2] * a[2],
                 c0 * S.xy + c1 * (a[0] * Sa[1] + Sa[0] * a[1]) + c2 * a[0] * a[1],
                 c0 * S.yz + c1 * (a[1] * Sa[2] + Sa[1] * a[2]) + c2 * a[1] * a[2],
                 c0 * S.xz + c1 * (a[0] * Sa[2] + Sa[0] * a[2]) + c2 * a[0] * a[2]};
    } else {
        // det(Fth) P S P with P = Fth^-1 = I/li + b_m m (x) m + b_n n (x) n (m = a; b_n = 0
        // in the transversely isotropic mode):
        //   P S P = S/li^2 + (1/li) sum_v b_v (v (S v)^T + (S v) v^T) + sum_{v,w} b_v b_w (v.S w) v (x) w
        const float lm1 = stretch_m1(m, m.alpha_m, dTe), lm = 1.0f + lm1;
        const float bm = (li1 - lm1) * inv_li * rcp(lm);
        float nv[3] = {0.0f, 0.0f, 0.0f}, bn = 0.0f, ln = li;
        if (expan_mode == 2) {
            const float4 q = aniso[2 * size_t(e)];
            oct_decode(q.x, q.y, nv);
            const float ln1 = stretch_m1(m, m.alpha_n, dTe);
            ln = 1.0f + ln1;
            bn = (li1 - ln1) * inv_li * rcp(ln);
        }
        detFth = li * lm * ln;
        const float Sa[3] = {S.xx * a[0] + S.xy * a[1] + S.xz * a[2], S.xy * a[0] + S.yy * a[1] + S.yz * a[2],
                             S.xz * a[0] + S.yz * a[1] + S.zz * a[2]};
        const float Sn[3] = {S.xx * nv[0] + S.xy * nv[1] + S.xz * nv[2], S.xy * nv[0] + S.yy * nv[1] + S.yz * nv[2],
                             S.xz * nv[0] + S.yz * nv[1] + S.zz * nv[2]};
        const float aSa = a[0] * Sa[0] + a[1] * Sa[1] + a[2] * Sa[2];
        const float nSn = nv[0] * Sn[0] + nv[1] * Sn[1] + nv[2] * Sn[2];
        const float aSn = a[0] * Sn[0] + a[1] * Sn[1] + a[2] * Sn[2];
        const float c0 = detFth * inv_li * inv_li, cm = detFth * bm * inv_li, cn = detFth * bn * inv_li;
        const float cmm = detFth * bm * bm * aSa, cnn = detFth * bn * bn * nSn, cmn = detFth * bm * bn * aSn;
#define TLED_PSP(i, j)                                                                                       \
    (cm * (a[i] * Sa[j] + Sa[i] * a[j]) + cn * (nv[i] * Sn[j] + Sn[i] * nv[j]) + cmm * a[i] * a[j] +            \
     cnn * nv[i] * nv[j] + cmn * (a[i] * nv[j] + nv[i] * a[j]))
        S = Sym3{c0 * S.xx + TLED_PSP(0, 0), c0 * S.yy + TLED_PSP(1, 1), c0 * S.zz + TLED_PSP(2, 2),
                 c0 * S.xy + TLED_PSP(0, 1), c0 * S.yz + TLED_PSP(1, 2), c0 * S.xz + TLED_PSP(0, 2)};
#undef TLED_PSP
    }
    if (want_psi) {
        float I1b3 = 3.0f * j23m1 + j23 * trG;  // I1bar - 3
        o.psiV = V0 * detFth * (0.5f * mu * I1b3 + 0.5f * eta * I4b1 * I4b1 + 0.5f * m.kappa * Jm1 * Jm1);
    }
    // ---- Prony relaxation on the total stress
    Sym3 St = S;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        float *t = theta + 6 * p;
        const float c1 = m.pc1[p], c2 = m.pc2[p];
        t[0] = c1 * S.xx + c2 * t[0];
        t[1] = c1 * S.yy + c2 * t[1];
        t[2] = c1 * S.zz + c2 * t[2];
        t[3] = c1 * S.xy + c2 * t[3];
        t[4] = c1 * S.yz + c2 * t[4];
        t[5] = c1 * S.xz + c2 * t[5];
        St.xx -= t[0]; St.yy -= t[1]; St.zz -= t[2]; St.xy -= t[3]; St.yz -= t[4]; St.xz -= t[5];
    }
    // ---- PV = (I + H) (V0 S~)
    St.xx *= V0; St.yy *= V0; St.zz *= V0; St.xy *= V0; St.yz *= V0; St.xz *= V0;
    const float Sm[9] = {St.xx, St.xy, St.xz, St.xy, St.yy, St.yz, St.xz, St.yz, St.zz};
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            o.PV[3 * i + j] = Sm[3 * i + j] + H[3 * i] * Sm[j] + H[3 * i + 1] * Sm[3 + j] + H[3 * i + 2] * Sm[6 + j];
    o.Jmin = fminf(J, Jt);
}

}  // namespace tled
