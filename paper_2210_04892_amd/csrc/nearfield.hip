// Double-precision set-up kernels: leaf radiation/receive patterns and the
// near-field blocks (regular triangle pairs by the 7-point rule on both
// triangles, touching pairs by singularity-cancelling transformations of the
// 4-D integral followed by tensor Gauss-Legendre rules).
#include "nearfield.hpp"

namespace mlfma {

// Radon's 7-point degree-5 rule: barycentric points and weights (sum 1)
__host__ __device__ inline void radon7(int p, double &l0, double &l1, double &l2, double &w)
{
    const double s15 = 3.872983346207417;   // sqrt(15)
    const double a = (6.0 - s15) / 21.0, b = (6.0 + s15) / 21.0;
    const double wa = (155.0 - s15) / 1200.0, wb = (155.0 + s15) / 1200.0;
    switch (p) {
        case 0: l0 = l1 = l2 = 1.0 / 3.0; w = 9.0 / 40.0; break;
        case 1: l0 = a; l1 = a; l2 = 1 - 2 * a; w = wa; break;
        case 2: l0 = a; l1 = 1 - 2 * a; l2 = a; w = wa; break;
        case 3: l0 = 1 - 2 * a; l1 = a; l2 = a; w = wa; break;
        case 4: l0 = b; l1 = b; l2 = 1 - 2 * b; w = wb; break;
        case 5: l0 = b; l1 = 1 - 2 * b; l2 = b; w = wb; break;
        default: l0 = 1 - 2 * b; l1 = b; l2 = b; w = wb; break;
    }
}

struct V3 { double x, y, z; };
__host__ __device__ inline V3 v3(const double *p) { return {p[0], p[1], p[2]}; }
__host__ __device__ inline V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__host__ __device__ inline V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__host__ __device__ inline V3 operator*(double s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
__host__ __device__ inline double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__host__ __device__ inline V3 cross(V3 a, V3 b) { return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x}; }

// ---------------------------------------------------------------- patterns
// R_n(k) = Int f_n e^{+jk khat.(r - r_b)} (theta, phi components) and the
// receive pattern of the C block Q_n = conj(Rg_n) - khat x conj(R_n) with
// Rg_n = Int (n x f_n) e^{+jk khat.(r - r_b)}; both by the 7-point rule.
__global__ void k_patterns(int N, int K, int nph, const double *__restrict__ ct, double k,
                           const int *__restrict__ rtri, const double *__restrict__ rcoef, const int *__restrict__ rloc,
                           const double *__restrict__ tri_v, const double *__restrict__ tri_n,
                           const double *__restrict__ tri_a, const double *__restrict__ centre,
                           cpx<double> *__restrict__ R, cpx<double> *__restrict__ Q)
{
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (long long)N * K) return;
    const int n = (int)(g / K), q = (int)(g % K);
    const int it = q / nph, ip = q % nph;
    const double c = ct[it], s = sqrt(fmax(0.0, 1 - c * c));
    double sp, cp;
    sincos(2.0 * M_PI * ip / nph, &sp, &cp);
    const V3 kh = {s * cp, s * sp, c}, th = {c * cp, c * sp, -s}, ph = {-sp, cp, 0.0};
    const V3 rb = v3(centre + 3 * (long long)n);
    cpx<double> Rt{0, 0}, Rp{0, 0}, Gt{0, 0}, Gp{0, 0};
    for (int h = 0; h < 2; h++) {
        const int t = rtri[2 * n + h];
        const double cf = rcoef[2 * n + h] * tri_a[t];
        const V3 P0 = v3(tri_v + 9 * (long long)t), P1 = v3(tri_v + 9 * (long long)t + 3),
                 P2 = v3(tri_v + 9 * (long long)t + 6);
        const V3 pf = v3(tri_v + 9 * (long long)t + 3 * rloc[2 * n + h]);
        const V3 nt = v3(tri_n + 3 * (long long)t);
        for (int p = 0; p < 7; p++) {
            double l0, l1, l2, w;
            radon7(p, l0, l1, l2, w);
            const V3 r = l0 * P0 + l1 * P1 + l2 * P2;
            const V3 f = (w * cf) * (r - pf);
            const V3 tw = cross(nt, f);
            double sn, cs;
            sincos(k * dot(kh, r - rb), &sn, &cs);
            const double ft = dot(f, th), fp = dot(f, ph), gt = dot(tw, th), gp = dot(tw, ph);
            Rt.re += ft * cs; Rt.im += ft * sn;
            Rp.re += fp * cs; Rp.im += fp * sn;
            Gt.re += gt * cs; Gt.im += gt * sn;
            Gp.re += gp * cs; Gp.im += gp * sn;
        }
    }
    R[2 * g] = Rt;
    R[2 * g + 1] = Rp;
    // Q = conj(Rg) - khat x conj(R),  khat x (v_t, v_p) = (-v_p, v_t)
    Q[2 * g] = conjg(Gt) + conjg(Rp);
    Q[2 * g + 1] = conjg(Gp) - conjg(Rt);
}

// ----------------------------------------------------------- touching pairs
// Reference coordinates: x = P0 + s1 (P1-P0) + s2 (P2-P0),
//                        y = Q0 + t1 (Q1-Q0) + t2 (Q2-Q0).
// rel 1 (shared vertex P0 = Q0): polar coordinates about the vertex on both
//   triangles, radial square split on its diagonal; weight xi^3 eta.
// rel 2 (shared edge P0P1 = Q0P1): each triangle swept from the edge to its
//   apex, x = (1-h)(P0 + sigma (P1-P0)) + h P2; split on the order of the two
//   edge abscissae, then the cube (offset, h_t, h_s) into three pyramids;
//   weight xi^2 (1 - offset) (1 - h_t) (1 - h_s).
// rel 3 (same triangle): difference vector over the hexagon S - S in polar
//   form; weight xi (1 - xi)^2 t1; each point also evaluated with x and y
//   exchanged (the opposite hexagon edge), so odd 1/R^2 parts cancel in pairs.
// The innermost Gauss coordinate tau (u3) moves the points along a line: s1,
// s2, t1, t2 = c0 + c1 tau with the coefficients of the other three.
struct TouchLine {
    double s1[2], s2[2], t1[2], t2[2], w;   // w: weight without tau's own
};
template <int REL>
__device__ inline TouchLine touch_line(int region, double u0, double u1, double u2)
{
    TouchLine l;
    if constexpr (REL == 1) {
        const double xi = u0, eta = u1;
        const double r1 = region == 0 ? xi : xi * eta, r2 = region == 0 ? xi * eta : xi;
        l = {{r1 * (1 - u2), 0}, {r1 * u2, 0}, {r2, -r2}, {0, r2}, xi * xi * xi * eta};
    } else if constexpr (REL == 2) {
        const int ord = region / 3, pyr = region % 3;
        const double a = u0 * u1, b = u0 * u2;
        const double off = pyr == 0 ? u0 : a, ht = pyr == 1 ? u0 : (pyr == 0 ? a : b), hs = pyr == 2 ? u0 : b;
        // edge abscissae off + (1 - off) tau and (1 - off) tau
        const double st = ord == 0 ? off : 0, ss = ord == 0 ? 0 : off;
        l = {{(1 - ht) * st, (1 - ht) * (1 - off)}, {ht, 0}, {(1 - hs) * ss, (1 - hs) * (1 - off)}, {hs, 0},
             u0 * u0 * (1 - off) * (1 - ht) * (1 - hs)};
    } else {
        const double xi = u0, eta = u1, pu = (1 - xi) * u2;
        // hexagon edge `region` as a - b with a, b on the boundary of
        // S = {0 <= v <= u <= 1} (coordinates (u, v)); (u, v) -> reference (u - v, v)
        const double au = region == 2 ? 1 - eta : 1, av = region == 0 ? eta : (region == 1 ? 1 : 1 - eta);
        const double bu = region == 0 ? 0 : (region == 1 ? eta : 1);
        l = {{pu + xi * bu, -pu}, {0, pu}, {pu + xi * (au - av), -pu}, {xi * av, pu}, xi * (1 - xi) * (1 - xi) * u2};
    }
    return l;
}

// 1 / sqrt(x) for normal x > 0: the hardware estimate (about 26 bits) and one
// third-order Newton step, x y^2 = 1 - e: y (1 + e/2 + 3 e^2/8).
__device__ inline double rsqrt3(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-x * y, y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// cos x and sin x / x from z = x^2 <= 4: power series in -z up to z^12
// (the next terms are below 3e-18).
__device__ inline void cos_sinc(double z, double &c, double &s)
{
    constexpr int NT = 12;
    double fc = 1, fs = 1;      // (2 n)!, (2 n + 1)! for n = NT
#pragma unroll
    for (int n = 1; n <= NT; n++) {
        fc *= (2.0 * n - 1) * (2.0 * n);
        fs *= (2.0 * n) * (2.0 * n + 1);
    }
    c = 1 / fc;
    s = 1 / fs;
#pragma unroll
    for (int n = NT; n >= 1; n--) {
        fc /= (2.0 * n - 1) * (2.0 * n);
        fs /= (2.0 * n) * (2.0 * n + 1);
        c = __builtin_fma(-z, c, 1 / fc);
        s = __builtin_fma(-z, s, 1 / fs);
    }
}

// The moments of one pair over this thread's lines: acc[v][3 a + b] += Sum w
// value_v phi_a psi_b, values G re, im, grad G re x, y, z, im x, y, z.  SERIES:
// the kernel's cosine and sine by cos_sinc (all k R of the pair at most 2).
template <int REL, bool SERIES>
__device__ inline void touch_moments(int n, double k, const double *gx, const double *gw, V3 e1, V3 e2, V3 f1, V3 f2,
                                     double (&acc)[8][9])
{
    const int nreg = REL == 1 ? 2 : (REL == 2 ? 6 : 3), count = nreg * n * n * n;
    // mixed-radix digits (i2, i1, i0, region) of this thread's line and of
    // the stride of 256 lines
    int d2 = threadIdx.x % n, d1 = threadIdx.x / n % n, d0 = threadIdx.x / (n * n) % n, reg = threadIdx.x / (n * n * n);
    const int p2 = 256 % n, p1 = 256 / n % n, p0 = 256 / (n * n) % n, pr = 256 / (n * n * n);
    const double k2 = k * k;
    for (int idx = threadIdx.x; idx < count; idx += 256) {
        const TouchLine l = touch_line<REL>(reg, gx[d0], gx[d1], gx[d2]);
        const double w = l.w * (gw[d0] * gw[d1] * gw[d2]);
        d2 += p2;
        int carry = d2 >= n;
        d2 -= carry ? n : 0;
        d1 += p1 + carry;
        carry = d1 >= n;
        d1 -= carry ? n : 0;
        d0 += p0 + carry;
        carry = d0 >= n;
        d0 -= carry ? n : 0;
        reg += pr + carry;
        V3 o[2];   // x - y = o[0] + o[1] tau
#pragma unroll
        for (int e = 0; e < 2; e++)
            o[e] = {l.s1[e] * e1.x + l.s2[e] * e2.x - l.t1[e] * f1.x - l.t2[e] * f2.x,
                    l.s1[e] * e1.y + l.s2[e] * e2.y - l.t1[e] * f1.y - l.t2[e] * f2.y,
                    l.s1[e] * e1.z + l.s2[e] * e2.z - l.t1[e] * f1.z - l.t2[e] * f2.z};
        // Sum over tau of G tau^m and g tau^m (grad G = g (x - y)); both
        // functions linear in tau except for a shared vertex, where x is fixed
        constexpr int NM = REL == 1 ? 2 : 3;
        double Gr[NM], Gi[NM], gr[NM + 1], gi[NM + 1];
#pragma unroll
        for (int m = 0; m < NM; m++) Gr[m] = Gi[m] = 0;
#pragma unroll
        for (int m = 0; m <= NM; m++) gr[m] = gi[m] = 0;
        auto point = [&](int i3) {
            const double tau = gx[i3];
            const V3 d = {fmad(tau, o[1].x, o[0].x), fmad(tau, o[1].y, o[0].y), fmad(tau, o[1].z, o[0].z)};
            const double r2 = dot(d, d), ir = rsqrt3(r2), kr = k * (r2 * ir);
            double sn, cs;
            if constexpr (SERIES) {
                cos_sinc(k2 * r2, cs, sn);
                sn *= kr;
            } else {
                sincos(kr, &sn, &cs);
            }
            const double inv = gw[i3] * ir, i3r = inv * (ir * ir);
            double vr = cs * inv, vi = -sn * inv, hr = -fmad(kr, sn, cs) * i3r, hi = fmad(-kr, cs, sn) * i3r;
#pragma unroll
            for (int m = 0; m < NM; m++) {
                Gr[m] += vr;
                Gi[m] += vi;
                gr[m] += hr;
                gi[m] += hi;
                vr *= tau;
                vi *= tau;
                hr *= tau;
                hi *= tau;
            }
            gr[NM] += hr;
            gi[NM] += hi;
        };
        for (int i3 = 0; i3 < n; i3 += 2) {   // two at a time (n is even)
            point(i3);
            point(i3 + 1);
        }
        // value moments V[v][m], m < NM
        double V[8][NM];
#pragma unroll
        for (int m = 0; m < NM; m++) {
            V[0][m] = Gr[m];
            V[1][m] = Gi[m];
            V[2][m] = fmad(o[1].x, gr[m + 1], o[0].x * gr[m]);
            V[3][m] = fmad(o[1].y, gr[m + 1], o[0].y * gr[m]);
            V[4][m] = fmad(o[1].z, gr[m + 1], o[0].z * gr[m]);
            V[5][m] = fmad(o[1].x, gi[m + 1], o[0].x * gi[m]);
            V[6][m] = fmad(o[1].y, gi[m + 1], o[0].y * gi[m]);
            V[7][m] = fmad(o[1].z, gi[m + 1], o[0].z * gi[m]);
        }
        // phi_a psi_b as polynomials in tau
        const double one[2] = {1, 0};
        const double *ph[3] = {one, l.s1, l.s2}, *ps[3] = {one, l.t1, l.t2};
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                double c[3] = {w * (ph[a][0] * ps[b][0]), w * (ph[a][0] * ps[b][1] + ph[a][1] * ps[b][0]),
                               w * (ph[a][1] * ps[b][1])};
                double cd[3] = {c[0], c[1], c[2]};
                if constexpr (REL == 3) {
                    // the point with x and y exchanged: same G, opposite gradient
                    const double q[3] = {w * (ps[a][0] * ph[b][0]), w * (ps[a][0] * ph[b][1] + ps[a][1] * ph[b][0]),
                                         w * (ps[a][1] * ph[b][1])};
#pragma unroll
                    for (int m = 0; m < 3; m++) {
                        cd[m] = c[m] - q[m];
                        c[m] += q[m];
                    }
                }
#pragma unroll
                for (int v = 0; v < 8; v++)
#pragma unroll
                    for (int m = 0; m < NM; m++) acc[v][3 * a + b] = fmad(v < 2 ? c[m] : cd[m], V[v][m], acc[v][3 * a + b]);
            }
    }
}

// One workgroup per touching pair, threads over the rule's lines.  The test
// and source functions are linear on their triangles, so the 36 entries (4
// operators x 3 x 3 edges) are combinations of 36 complex moments,
//   M[0][a][b] = Sum w G phi_a psi_b,  M[1 + c][a][b] = Sum w (grad G)_c phi_a psi_b,
// phi = (1, s1, s2), psi = (1, t1, t2).  Along a line (the innermost Gauss
// coordinate) x - y is linear and phi psi at most quadratic, so a point costs
// its kernel and 10 or 14 sums; the moments are formed once per line.  A
// pair's triangles share P[0] = Q[0], so x - y comes from the edge vectors
// alone.  Bound by FP64 issue, about 70 operations per point: a wave issues
// vector instructions in 0.46 of its time (0.76 of the slots), and 256 registers,
// 41 of them spilled (140 bytes a lane), leave two waves per SIMD.  MI355X, box of
// 3 456 triangles (45 000 pairs, mostly order 14): 194 ms with the nine dyads
// of cross products and 64-bit index divisions per point, 51 ms with the
// moments per point, 20.5 ms with the moments per line.
__global__ __launch_bounds__(256, 2) void k_touch(int npairs, const TouchPair *__restrict__ pairs, double k,
                                                  const double *__restrict__ gnodes, const int *__restrict__ goff,
                                                  cpx<double> *__restrict__ out)
{
    __shared__ double nodes[2 * TOUCH_MAX_ORDER];
    __shared__ double red[4][72];
    __shared__ double mom[72];
    const int p = blockIdx.x;
    if (p >= npairs) return;
    const TouchPair &tp = pairs[p];
    const int n = tp.order, rel = tp.rel;
    for (int i = threadIdx.x; i < 2 * n; i += 256) nodes[i] = gnodes[goff[n] + i];
    __syncthreads();
    const double *gx = nodes, *gw = nodes + n;
    const V3 P0 = v3(tp.P), e1 = v3(tp.P + 3) - P0, e2 = v3(tp.P + 6) - P0;
    const V3 Q0 = v3(tp.Q), f1 = v3(tp.Q + 3) - Q0, f2 = v3(tp.Q + 6) - Q0;
    double acc[8][9];
#pragma unroll
    for (int v = 0; v < 8; v++)
#pragma unroll
        for (int e = 0; e < 9; e++) acc[v][e] = 0;
    // the largest distance of two points of the triangles is one of corners
    double r2max = 0;
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            const V3 d = v3(tp.P + 3 * a) - v3(tp.Q + 3 * b);
            r2max = fmax(r2max, dot(d, d));
        }
    const bool series = k * k * r2max <= 4.0;
    if (rel == 1) {
        if (series) touch_moments<1, true>(n, k, gx, gw, e1, e2, f1, f2, acc);
        else touch_moments<1, false>(n, k, gx, gw, e1, e2, f1, f2, acc);
    } else if (rel == 2) {
        if (series) touch_moments<2, true>(n, k, gx, gw, e1, e2, f1, f2, acc);
        else touch_moments<2, false>(n, k, gx, gw, e1, e2, f1, f2, acc);
    } else {
        if (series) touch_moments<3, true>(n, k, gx, gw, e1, e2, f1, f2, acc);
        else touch_moments<3, false>(n, k, gx, gw, e1, e2, f1, f2, acc);
    }
    // block reduction: waves by shuffles, then across waves through LDS
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
#pragma unroll
    for (int c = 0; c < 8; c++)
#pragma unroll
        for (int e = 0; e < 9; e++) {
            double v = acc[c][e];
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
            if (lane == 0) red[wave][9 * c + e] = v;
        }
    __syncthreads();
    // (2 A_t)(2 A_s): reference -> physical, and the kernel's 1 / (4 pi)
    const double scale = tp.At * tp.As / M_PI;
    if (threadIdx.x < 72)
        mom[threadIdx.x] = scale * (red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x]);
    __syncthreads();
    if (threadIdx.x >= 9) return;
    // entry (i, j) from the moments: x - p_i = Sum phi_a U_a, y - q_j = Sum psi_b W_b
    const int i = threadIdx.x / 3, j = threadIdx.x % 3;
    const V3 U[3] = {P0 - v3(tp.P + 3 * i), e1, e2}, W[3] = {Q0 - v3(tp.Q + 3 * j), f1, f2};
    const V3 nt = v3(tp.nt);
    cpx<double> ab = {0, 0}, twb = {0, 0}, Kv = {0, 0}, Kx = {0, 0}, twd = {0, 0};
    for (int a = 0; a < 3; a++) {
        const V3 tw = cross(nt, U[a]);   // n_t x (x - p_i)
        for (int b = 0; b < 3; b++) {
            const int e = 3 * a + b;
            const cpx<double> G = {mom[e], mom[9 + e]};
            const V3 gr = {mom[18 + e], mom[27 + e], mom[36 + e]}, gi = {mom[45 + e], mom[54 + e], mom[63 + e]};
            axpy_to(ab, dot(U[a], W[b]), G);
            axpy_to(twb, dot(tw, W[b]), G);
            const V3 cr = cross(gr, W[b]), ci = cross(gi, W[b]);
            Kv.re += dot(U[a], cr);
            Kv.im += dot(U[a], ci);
            Kx.re -= dot(tw, cr);
            Kx.im -= dot(tw, ci);
            if (b == 0) {
                twd.re += dot(tw, gr);
                twd.im += dot(tw, gi);
            }
        }
    }
    const double f4 = 4.0 / (k * k);
    const cpx<double> T = {k * (ab.im - f4 * mom[9]), -k * (ab.re - f4 * mom[0])};   // -jk (a.b - 4/k^2) G
    const cpx<double> Tx = {-k * twb.im - (2.0 / k) * twd.im, k * twb.re + (2.0 / k) * twd.re};
    // result stored as [op][original test edge][original source edge]; K and
    // n x Kbar vanish on one flat triangle
    cpx<double> *dst = out + 36LL * p + 3 * tp.pi[i] + tp.qi[j];
    dst[0] = T;
    dst[9] = rel == 3 ? mk<double>(0, 0) : Kv;
    dst[18] = Tx;
    dst[27] = rel == 3 ? mk<double>(0, 0) : Kx;
}

// --------------------------------------------------------------- near slots
// cos x and sin x for 0 <= x < 1e4: x less the nearest multiple of pi / 2 (in
// two parts), then the power series on [-pi/4, pi/4] (next terms below 3e-18).
__device__ inline void cos_sin(double x, double &c, double &s)
{
    constexpr double PIO2 = 1.5707963267948966, PIO2_LO = 6.123233995736766e-17;   // pi / 2 = PIO2 + PIO2_LO
    const double m = __builtin_rint(x * (2 / M_PI));
    const double r = __builtin_fma(-m, PIO2_LO, __builtin_fma(-m, PIO2, x)), z = r * r;
    constexpr int NT = 9;
    double cr = 0, sr = 0, fc = 1, fs = 1;
#pragma unroll
    for (int n = 1; n <= NT; n++) {
        fc *= (2.0 * n - 1) * (2.0 * n);
        fs *= (2.0 * n) * (2.0 * n + 1);
    }
    cr = 1 / fc;
    sr = 1 / fs;
#pragma unroll
    for (int n = NT; n >= 1; n--) {
        fc /= (2.0 * n - 1) * (2.0 * n);
        fs /= (2.0 * n) * (2.0 * n + 1);
        cr = __builtin_fma(-z, cr, 1 / fc);
        sr = __builtin_fma(-z, sr, 1 / fs);
    }
    sr *= r;
    const int q = (int)m & 3;
    c = q & 1 ? sr : cr;
    s = q & 1 ? cr : sr;
    if (q == 1 || q == 2) c = -c;
    if (q >= 2) s = -s;
}

// The 7 x 7 points of a pair of triangles without a common corner, for test
// edge i and source edge j.  With a = x - p_i and b = y - q_j the operators
// need, per test point, only S0 = Sum w G, S1 = Sum w G b, H0 = Sum w g and H1
// = Sum w g b: Sum w grad G = (x - q_j) H0 - H1, Sum w grad G x b = (x - q_j) x H1.
// Bound by FP64 issue, about 75 operations per point pair (a wave issues vector
// instructions in 0.53 of its time).  MI355X, box of 3 456 triangles (the launch of k_slots): 13.9 ms with the dyads and library
// functions at every point pair, 5.9 ms like this.
__device__ inline void regular_pair(const double *Pv, const double *Qv, const double *nt, double At, double As, int i,
                                    int j, double k, cpx<double> out[4])
{
    const V3 P0 = v3(Pv), P1 = v3(Pv + 3), P2 = v3(Pv + 6), Q0 = v3(Qv), Q1 = v3(Qv + 3), Q2 = v3(Qv + 6);
    const V3 pi = v3(Pv + 3 * i), qj = v3(Qv + 3 * j), n = v3(nt);
    V3 b[7];
    double wb[7];
#pragma unroll
    for (int q = 0; q < 7; q++) {
        double b0, b1, b2;
        radon7(q, b0, b1, b2, wb[q]);
        b[q] = b0 * Q0 + b1 * Q1 + b2 * Q2 - qj;
    }
    cpx<double> T = {0, 0}, Kv = {0, 0}, Tx = {0, 0}, Kx = {0, 0}, sd = {0, 0}, s0 = {0, 0};
#pragma unroll 1
    for (int p = 0; p < 7; p++) {
        double a0, a1, a2, wp;
        radon7(p, a0, a1, a2, wp);
        const V3 x = a0 * P0 + a1 * P1 + a2 * P2, a = x - pi, xq = x - qj, tw = cross(n, a);
        double S[4][2] = {{0}}, H[4][2] = {{0}};
#pragma unroll
        for (int q = 0; q < 7; q++) {
            const V3 d = xq - b[q];
            const double r2 = dot(d, d), ir = rsqrt3(r2), kr = k * (r2 * ir);
            double cs, sn;
            cos_sin(kr, cs, sn);
            const double inv = wb[q] * ir, i3 = inv * (ir * ir);
            const double gr = cs * inv, gi = -sn * inv, hr = -fmad(kr, sn, cs) * i3, hi = fmad(-kr, cs, sn) * i3;
            const double v[4] = {1.0, b[q].x, b[q].y, b[q].z};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                S[e][0] = fmad(v[e], gr, S[e][0]);
                S[e][1] = fmad(v[e], gi, S[e][1]);
                H[e][0] = fmad(v[e], hr, H[e][0]);
                H[e][1] = fmad(v[e], hi, H[e][1]);
            }
        }
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const V3 s1 = {S[1][c], S[2][c], S[3][c]}, h1 = {H[1][c], H[2][c], H[3][c]}, xh = cross(xq, h1);
            (c ? s0.im : s0.re) += wp * S[0][c];
            (c ? T.im : T.re) += wp * dot(a, s1);
            (c ? Tx.im : Tx.re) += wp * dot(tw, s1);
            (c ? sd.im : sd.re) += wp * (dot(tw, xq) * H[0][c] - dot(tw, h1));
            (c ? Kv.im : Kv.re) += wp * dot(a, xh);
            (c ? Kx.im : Kx.re) -= wp * dot(tw, xh);
        }
    }
    const double w = At * As / (4.0 * M_PI), f4 = 4.0 / (k * k);
    out[0] = w * mk<double>(k * (T.im - f4 * s0.im), -k * (T.re - f4 * s0.re));   // -jk (a.b - 4/k^2) G
    out[1] = w * Kv;                                                              // a . (grad G x b)
    out[2] = w * mk<double>(-k * Tx.im - (2.0 / k) * sd.im, k * Tx.re + (2.0 / k) * sd.re);   // jk tw.b G + (2j/k) tw.grad G
    out[3] = w * Kx;                                                              // -tw . (grad G x b)
}

// One workgroup per leaf box; threads over the (row, near column) slots of the
// box.  Each slot sums the four triangle pairs of its two RWGs.
__global__ __launch_bounds__(256) void k_slots(const int *__restrict__ box_start, const int *__restrict__ near_start,
                                               const int *__restrict__ near_box, const long long *__restrict__ val_off,
                                               const int *__restrict__ rtri, const int *__restrict__ rloc,
                                               const double *__restrict__ rcoef, const double *__restrict__ tri_v,
                                               const double *__restrict__ tri_n, const double *__restrict__ tri_a,
                                               const int *__restrict__ tp_start, const int *__restrict__ tp_s,
                                               const cpx<double> *__restrict__ touch, double k,
                                               cpx<double> *__restrict__ em64, cpx<double> *__restrict__ c64,
                                               cpx<float> *__restrict__ em32, cpx<float> *__restrict__ c32)
{
    __shared__ int cstart[32];
    __shared__ int pre[33];
    const int b = blockIdx.x;
    const int nn = near_start[b + 1] - near_start[b];
    if (threadIdx.x == 0) {
        pre[0] = 0;
        for (int q = 0; q < nn; q++) {
            int nb = near_box[near_start[b] + q];
            cstart[q] = box_start[nb];
            pre[q + 1] = pre[q] + box_start[nb + 1] - box_start[nb];
        }
    }
    __syncthreads();
    const int ncols = pre[nn];
    const int m0 = box_start[b];
    const long long nslot = (long long)(box_start[b + 1] - m0) * ncols;
    for (long long sl = threadIdx.x; sl < nslot; sl += blockDim.x) {
        const int m = m0 + (int)(sl / ncols), jc = (int)(sl % ncols);
        int q = 0;
        while (jc >= pre[q + 1]) q++;
        const int n = cstart[q] + (jc - pre[q]);
        cpx<double> acc[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
        for (int h1 = 0; h1 < 2; h1++)
            for (int h2 = 0; h2 < 2; h2++) {
                const int t = rtri[2 * m + h1], s = rtri[2 * n + h2];
                const int i = rloc[2 * m + h1], j = rloc[2 * n + h2];
                const double cc = rcoef[2 * m + h1] * rcoef[2 * n + h2];
                int hit = -1;
                for (int e = tp_start[t]; e < tp_start[t + 1]; e++)
                    if (tp_s[e] == s) { hit = e; break; }
                cpx<double> part[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
                if (hit >= 0) {
                    for (int o = 0; o < 4; o++) part[o] = touch[36LL * hit + 9 * o + 3 * i + j];
                } else {
                    regular_pair(tri_v + 9LL * t, tri_v + 9LL * s, tri_n + 3LL * t, tri_a[t], tri_a[s], i, j, k, part);
                }
                for (int o = 0; o < 4; o++) acc[o] = acc[o] + cc * part[o];
            }
        const cpx<double> T = acc[0], Kk = acc[1], Tx = acc[2], Kx = acc[3];
        const cpx<double> A = -0.5 * (T + Kx), B = 0.5 * (Tx - Kk);
        const long long slot = val_off[b] + sl;
        em64[2 * slot] = T;
        em64[2 * slot + 1] = Kk;
        c64[2 * slot] = A;
        c64[2 * slot + 1] = B;
        em32[2 * slot] = {(float)T.re, (float)T.im};
        em32[2 * slot + 1] = {(float)Kk.re, (float)Kk.im};
        c32[2 * slot] = {(float)A.re, (float)A.im};
        c32[2 * slot + 1] = {(float)B.re, (float)B.im};
    }
}

// ------------------------------------------------------------- conversions
__global__ void k_to_float(const cpx<double> *__restrict__ a, cpx<float> *__restrict__ b, long long n)
{
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n) b[g] = {(float)a[g].re, (float)a[g].im};
}

// ------------------------------------------------------------- plane waves
// b^J = <f, E/2 + n x H/2>, b^M = <f, H/2 - n x E/2>, E = p e^{-jk khat.r},
// H = khat x p e^{-jk khat.r}; 7-point rule on both triangles of the RWG.
template <class T>
__global__ void k_plane_wave(int N, int nrhs, double k, const int *__restrict__ perm, const int *__restrict__ rtri,
                             const int *__restrict__ rloc, const double *__restrict__ rcoef,
                             const double *__restrict__ tri_v, const double *__restrict__ tri_n,
                             const double *__restrict__ tri_a, const double *__restrict__ dirs,
                             cpx<T> *__restrict__ b, long long ldb)
{
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (long long)N * nrhs) return;
    const int i = (int)(g % N), r = (int)(g / N);
    const V3 kh = v3(dirs + 6 * r), p = v3(dirs + 6 * r + 3);
    const V3 h = cross(kh, p);
    cpx<double> bj{0, 0}, bm{0, 0};
    for (int s = 0; s < 2; s++) {
        const int t = rtri[2 * i + s];
        const double cf = rcoef[2 * i + s] * tri_a[t];
        const V3 P0 = v3(tri_v + 9LL * t), P1 = v3(tri_v + 9LL * t + 3), P2 = v3(tri_v + 9LL * t + 6);
        const V3 pf = v3(tri_v + 9LL * t + 3 * rloc[2 * i + s]);
        const V3 n = v3(tri_n + 3LL * t);
        const V3 nxe = cross(n, p), nxh = cross(n, h);
        for (int q = 0; q < 7; q++) {
            double l0, l1, l2, w;
            radon7(q, l0, l1, l2, w);
            const V3 x = l0 * P0 + l1 * P1 + l2 * P2;
            const V3 a = x - pf;
            double sn, cs;
            sincos(k * dot(kh, x), &sn, &cs);
            const double fj = 0.5 * w * cf * (dot(a, p) + dot(a, nxh));
            const double fm = 0.5 * w * cf * (dot(a, h) - dot(a, nxe));
            bj.re += fj * cs; bj.im -= fj * sn;
            bm.re += fm * cs; bm.im -= fm * sn;
        }
    }
    const int u = perm[i];
    b[(long long)r * ldb + u] = {(T)bj.re, (T)bj.im};
    b[(long long)r * ldb + N + u] = {(T)bm.re, (T)bm.im};
}

// -------------------------------------------------------------- far field
// F(khat) = (-jk/4pi)[P_J - khat (khat . P_J) - khat x P_M], the far-zone
// limit of E = L{J} - K{M} (plane-wave limits L -> -jk(I - khat khat),
// K -> -jk khat x); P_X = Int X exp(+jk khat . r) ds with the 7-point rule on
// both triangles of every RWG; the radar cross section of Sec. III is
// 4 pi |F|^2.  Workgroup = (direction, right-hand side), threads over RWGs,
// double-precision sums reduced in LDS; output F . theta_hat, F . phi_hat.
template <class T>
__global__ __launch_bounds__(256) void k_far_field(int N, double k, const int *__restrict__ perm,
                                                   const int *__restrict__ rtri, const int *__restrict__ rloc,
                                                   const double *__restrict__ rcoef, const double *__restrict__ tri_v,
                                                   const double *__restrict__ tri_a, const double *__restrict__ dirs,
                                                   const cpx<T> *__restrict__ x, long long ldx, cpx<T> *__restrict__ F,
                                                   int nrhs)
{
    __shared__ double red[12][256];
    const int d = blockIdx.x, r = blockIdx.y;
    const V3 kh = v3(dirs + 3 * d);
    double acc[12] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};   // P_J (re, im) xyz, then P_M
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        const int u = perm[i];
        const cpx<T> xj = x[(long long)r * ldx + u], xm = x[(long long)r * ldx + N + u];
        for (int s2 = 0; s2 < 2; s2++) {
            const int t = rtri[2 * i + s2];
            const double cf = rcoef[2 * i + s2] * tri_a[t];
            const V3 P0 = v3(tri_v + 9LL * t), P1 = v3(tri_v + 9LL * t + 3), P2 = v3(tri_v + 9LL * t + 6);
            const V3 pf = v3(tri_v + 9LL * t + 3 * rloc[2 * i + s2]);
            for (int q = 0; q < 7; q++) {
                double l0, l1, l2, w;
                radon7(q, l0, l1, l2, w);
                const V3 xq = l0 * P0 + l1 * P1 + l2 * P2;
                const V3 a = (w * cf) * (xq - pf);
                double sn, cs;
                sincos(k * dot(kh, xq), &sn, &cs);
                // a e^{+j phase} times the coefficients
                const double pjr = cs * xj.re - sn * xj.im, pji = cs * xj.im + sn * xj.re;
                const double pmr = cs * xm.re - sn * xm.im, pmi = cs * xm.im + sn * xm.re;
                const double av[3] = {a.x, a.y, a.z};
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    acc[2 * c] += av[c] * pjr;
                    acc[2 * c + 1] += av[c] * pji;
                    acc[6 + 2 * c] += av[c] * pmr;
                    acc[6 + 2 * c + 1] += av[c] * pmi;
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 12; c++) red[c][threadIdx.x] = acc[c];
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st)
#pragma unroll
            for (int c = 0; c < 12; c++) red[c][threadIdx.x] += red[c][threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double kk[3] = {kh.x, kh.y, kh.z};
    double PJr[3], PJi[3], PMr[3], PMi[3];
    for (int c = 0; c < 3; c++) {
        PJr[c] = red[2 * c][0];
        PJi[c] = red[2 * c + 1][0];
        PMr[c] = red[6 + 2 * c][0];
        PMi[c] = red[6 + 2 * c + 1][0];
    }
    const double kpr = kk[0] * PJr[0] + kk[1] * PJr[1] + kk[2] * PJr[2];
    const double kpi = kk[0] * PJi[0] + kk[1] * PJi[1] + kk[2] * PJi[2];
    double Fr[3], Fi[3];
    for (int c = 0; c < 3; c++) {
        const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        Fr[c] = PJr[c] - kk[c] * kpr - (kk[c1] * PMr[c2] - kk[c2] * PMr[c1]);
        Fi[c] = PJi[c] - kk[c] * kpi - (kk[c1] * PMi[c2] - kk[c2] * PMi[c1]);
    }
    const double th = acos(fmax(-1.0, fmin(1.0, kk[2]))), ph = atan2(kk[1], kk[0]);
    const double tv[3] = {cos(th) * cos(ph), cos(th) * sin(ph), -sin(th)}, pv[3] = {-sin(ph), cos(ph), 0.0};
    const double pre = k / (4 * M_PI);   // F = -j pre (...)
    double ftr = 0, fti = 0, fpr = 0, fpi = 0;
    for (int c = 0; c < 3; c++) {
        ftr += Fr[c] * tv[c];
        fti += Fi[c] * tv[c];
        fpr += Fr[c] * pv[c];
        fpi += Fi[c] * pv[c];
    }
    // -j (a + jb) = b - ja
    F[((long long)d * 2) * nrhs + r] = {(T)(pre * fti), (T)(-pre * ftr)};
    F[((long long)d * 2 + 1) * nrhs + r] = {(T)(pre * fpi), (T)(-pre * fpr)};
}

// ---------------------------------------------------------------- launchers
void launch_far_field(bool single, int N, double k, const int *perm, const int *rtri, const int *rloc,
                      const double *rcoef, const double *tri_v, const double *tri_a, const double *dirs, int ndir,
                      const void *x, long long ldx, void *F, int nrhs, hipStream_t s)
{
    if (ndir <= 0 || nrhs <= 0) return;
    const dim3 grid(ndir, nrhs);
    if (single)
        hipLaunchKernelGGL(k_far_field<float>, grid, dim3(256), 0, s, N, k, perm, rtri, rloc, rcoef, tri_v, tri_a,
                           dirs, (const cpx<float> *)x, ldx, (cpx<float> *)F, nrhs);
    else
        hipLaunchKernelGGL(k_far_field<double>, grid, dim3(256), 0, s, N, k, perm, rtri, rloc, rcoef, tri_v, tri_a,
                           dirs, (const cpx<double> *)x, ldx, (cpx<double> *)F, nrhs);
}

void launch_plane_wave(bool single, int N, int nrhs, double k, const int *perm, const int *rtri, const int *rloc,
                       const double *rcoef, const double *tri_v, const double *tri_n, const double *tri_a,
                       const double *dirs, void *b, long long ldb, hipStream_t s)
{
    long long n = (long long)N * nrhs;
    dim3 grid((unsigned)((n + 255) / 256));
    if (single)
        hipLaunchKernelGGL(k_plane_wave<float>, grid, dim3(256), 0, s, N, nrhs, k, perm, rtri, rloc, rcoef, tri_v,
                           tri_n, tri_a, dirs, (cpx<float> *)b, ldb);
    else
        hipLaunchKernelGGL(k_plane_wave<double>, grid, dim3(256), 0, s, N, nrhs, k, perm, rtri, rloc, rcoef, tri_v,
                           tri_n, tri_a, dirs, (cpx<double> *)b, ldb);
}

void launch_patterns(int N, int K, int nph, const double *ct, double k, const int *rtri, const double *rcoef,
                     const int *rloc, const double *tri_v, const double *tri_n, const double *tri_a,
                     const double *centre, cpx<double> *R, cpx<double> *Q, hipStream_t s)
{
    long long n = (long long)N * K;
    hipLaunchKernelGGL(k_patterns, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, N, K, nph, ct, k, rtri, rcoef,
                       rloc, tri_v, tri_n, tri_a, centre, R, Q);
}

void launch_touch(int npairs, const TouchPair *pairs, double k, const double *gnodes, const int *goff,
                  cpx<double> *out, hipStream_t s)
{
    if (npairs > 0)
        hipLaunchKernelGGL(k_touch, dim3(npairs), dim3(256), 0, s, npairs, pairs, k, gnodes, goff, out);
}

void launch_slots(int nbox, const int *box_start, const int *near_start, const int *near_box, const long long *val_off,
                  const int *rtri, const int *rloc, const double *rcoef, const double *tri_v, const double *tri_n,
                  const double *tri_a, const int *tp_start, const int *tp_s, const cpx<double> *touch, double k,
                  cpx<double> *em64, cpx<double> *c64, cpx<float> *em32, cpx<float> *c32, hipStream_t s)
{
    hipLaunchKernelGGL(k_slots, dim3(nbox), dim3(256), 0, s, box_start, near_start, near_box, val_off, rtri, rloc,
                       rcoef, tri_v, tri_n, tri_a, tp_start, tp_s, touch, k, em64, c64, em32, c32);
}

void launch_to_float(const cpx<double> *a, cpx<float> *b, long long n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_to_float, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, b, n);
}

}  // namespace mlfma
