// Radiation for two, near field for three, receive for four or more right-hand
// sides on the matrix cores.
//
// With nrhs right-hand sides both steps are dense complex products per leaf
// box b (Sec. II-E; the single-pattern far field of the C block and the L/K
// pair):
//   radiation  U_b[c](q, r) = sum_{n in b} alpha_n(r) R_n[c](q) + beta_n(r) (khat x R_n)[c](q)
//   receive    y_(m,h)(r)   += sum_{c, q} P_(m,h)[c](q) V_b[c](q, r)
// Each complex product is four real 16x16x4 MFMAs (real part: re*re and
// -im*im, imaginary part: re*im and im*re), FP32 for complex64 and FP64 for
// complex128.  Lane layout (wave64, both checked on the device): lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16]; it holds D[(l / 16) * 4 +
// v][l % 16] (v_mfma_f32_16x16x4f32) or D[l / 16 + 4 v][l % 16]
// (v_mfma_f64_16x16x4f64), v = 0..3.
#include "device.hpp"
#include "mfma_ops.hpp"
#include "../../include/mlfma.h"

namespace mlfma {

namespace {

constexpr int NXCD_M = 8;
__device__ inline long long xcd_block_m(long long nblk)
{
    const long long per = (nblk + NXCD_M - 1) / NXCD_M;
    const long long hw = blockIdx.x;
    const long long lb = (hw % NXCD_M) * per + hw / NXCD_M;
    return lb < nblk ? lb : -1;
}
inline unsigned xcd_grid_m(long long nblk) { return (unsigned)(((nblk + NXCD_M - 1) / NXCD_M) * NXCD_M); }

__device__ inline long long pidx_m(long long b, int c, int r, int q, int nrhs, int ks)
{
    return ((b * 2 + c) * nrhs + r) * (long long)ks + q;
}

// complex D += A B on RT accumulator pairs sharing the B operand
template <class T, int RT>
__device__ inline void cmfma(typename Mf<T>::v4 (&dre)[RT], typename Mf<T>::v4 (&dim)[RT], const cpx<T> (&a)[RT],
                             cpx<T> b)
{
#pragma unroll
    for (int t = 0; t < RT; t++) dre[t] = Mf<T>::mma(a[t].re, b.re, dre[t]);
#pragma unroll
    for (int t = 0; t < RT; t++) dim[t] = Mf<T>::mma(a[t].re, b.im, dim[t]);
#pragma unroll
    for (int t = 0; t < RT; t++) dre[t] = Mf<T>::mma(-a[t].im, b.im, dre[t]);
#pragma unroll
    for (int t = 0; t < RT; t++) dim[t] = Mf<T>::mma(a[t].im, b.re, dim[t]);
}

// packed columns' products (d1, d2) -> (real, imaginary) in columns 0..7
template <class A>
__device__ inline void fold_cols(A &d1, A &d2)
{
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const auto o1 = __shfl_xor(d1[v], 8), o2 = __shfl_xor(d2[v], 8);
        const auto re = d1[v] - o2, im = o1 + d2[v];
        d1[v] = re;
        d2[v] = im;
    }
}

// the same for packed rows in double precision (rows 0..7 real, 8..15 imaginary
// parts of the packed operand; d1, d2 its products with the real and imaginary
// part of the other one): row r + 8 is the same lane's slot v + 2
template <int RT, class A>
__device__ inline void fold_rows(A (&d1)[RT], A (&d2)[RT])
{
#pragma unroll
    for (int u = 0; u < RT; u++)
#pragma unroll
        for (int v = 0; v < 2; v++) {
            const double re = d1[u][v] - d2[u][v + 2], im = d1[u][v + 2] + d2[u][v];
            d1[u][v] = re;
            d2[u][v] = im;
        }
}

// The right-hand-side operand of a complex product: full (a lane holds a
// complex value of one of 16 right-hand sides, four real MFMAs per step) or
// packed (at most 8 right-hand sides: lanes 0..7 of the 16 hold the real
// parts, lanes 8..15 the imaginary parts, so that two real MFMAs with the
// other operand's real and imaginary part form all four partial products;
// fold_* combines them once, after the sum).  Up to 8 right-hand sides the
// packed form takes half the matrix-core time.  Ellipsoid of 48 000 RWGs, 7
// right-hand sides, complex64 (complex128): near field 0.413 (0.686) ms on
// the vector units, 0.185 (0.33) full, 0.138 (0.214) packed with the inner
// index split (NEAR_SPLIT_BELOW; complex64 with sums in double, as they are
// now, 0.164); radiation in complex128 0.400, 0.168, 0.116
// (complex64: k_radiate_few); receive 0.350 (0.625), 0.113 (0.202), 0.084
// (0.141; complex64 with sums in double, as they are now, 0.110).
template <class T, bool PK>
struct Pk;
template <class T>
struct Pk<T, false> {
    typedef cpx<T> elem;
    typedef typename Mf<T>::v4 v4;
    static __device__ inline elem get(const cpx<T> *p, int) { return *p; }
    static __device__ inline void mma(cpx<T> a, elem b, v4 &dre, v4 &dim)
    {
        dre = Mf<T>::mma(a.re, b.re, dre);
        dim = Mf<T>::mma(a.re, b.im, dim);
        dre = Mf<T>::mma(-a.im, b.im, dre);
        dim = Mf<T>::mma(a.im, b.re, dim);
    }
};
template <class T>
struct Pk<T, true> {
    typedef T elem;
    typedef typename Mf<T>::v4 v4;
    static __device__ inline elem get(const cpx<T> *p, int lo) { return reinterpret_cast<const T *>(p)[lo >> 3]; }
    // packed columns: d1 = a.re [b.re | b.im], d2 = a.im [b.re | b.im]
    static __device__ inline void mma(cpx<T> a, elem b, v4 &d1, v4 &d2)
    {
        d1 = Mf<T>::mma(a.re, b, d1);
        d2 = Mf<T>::mma(a.im, b, d2);
    }
};

// Radiation.  Wave = (box, tile of 16 samples, both components) x RT tiles of
// 16 right-hand sides (packed: one tile of 8); D[i = rhs][j = sample], inner
// index k = (RWG, alpha|beta): one MFMA step covers two RWGs.  EM pair: alpha
// = x1, beta = -x2; C block: alpha = x2 / 2, beta = x1 / 2.  A lane's pattern
// sample feeds both components (alpha lanes R[c], beta lanes (khat x R)[c],
// the other component up to the sign), so it is one load of both and the x
// values of a step serve both.  Bound by the vector memory path (texture data
// unit busy 0.88 with one component per wave): sphere of radius 8 wavelengths
// (276 480 RWGs), 16 right-hand sides, complex64 0.605 ms with one component
// per wave and two sample tiles, 0.553 ms like this; two tiles per wave here
// 0.581 (complex128 1.07, 1.07, 1.22 ms).  Steps with both RWGs in the box
// load without predicates, the next step's operands in flight while the
// current one is multiplied (two register sets taking turns; past the last
// step the loads repeat it).
template <class T, int RT, bool PK>
__global__ __launch_bounds__(256) void k_radiate_mfma(int op, int nbox, int K, int ks, int nqt,
                                                      const int *__restrict__ box_start,
                                                      const cpx<T> *__restrict__ R,
                                                      const cpx<T> *__restrict__ X, cpx<T> *__restrict__ U,
                                                      int nrhs)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per_box = (nqt + 3) / 4;
    const int nrg = (nrhs + 16 * RT - 1) / (16 * RT);
    const long long blk = xcd_block_m((long long)nbox * per_box * nrg);
    if (blk < 0) return;
    const int rg = (int)(blk % nrg);
    const long long bt = blk / nrg;
    const int b = (int)(bt / per_box), qt = (int)(bt % per_box) * 4 + wave;
    if (qt >= nqt) return;
    const int lo = lane & 15, kk = lane >> 4;
    const int q = qt * 16 + lo;                      // this lane's sample
    const long long qo = 2LL * min(q, K - 1);        // its pattern offset, clamped to a valid sample
    const int s = kk & 1;
    // which half of X feeds this lane's alpha/beta, and its factor
    const int h = op == MLFMA_OP_EM ? s : 1 - s;
    const T fac = op == MLFMA_OP_EM ? (s ? T(-1) : T(1)) : T(0.5);
    const int n0 = box_start[b], n1 = box_start[b + 1];
    int rr[RT];   // this lane's right-hand side per tile, clamped
#pragma unroll
    for (int u = 0; u < RT; u++) rr[u] = min(PK ? lo & 7 : (rg * RT + u) * 16 + lo, nrhs - 1);
    typename Mf<T>::v4 dre[2][RT], dim[2][RT];
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int u = 0; u < RT; u++) dre[c][u] = dim[c][u] = typename Mf<T>::v4{0, 0, 0, 0};
    struct Step {
        cpx<T> v[2];
        typename Pk<T, PK>::elem x[RT];
    };
    auto load = [&](int nn, Step &o) {
        load_pair(R + (long long)nn * K * 2 + qo, o.v[0], o.v[1]);
        const cpx<T> *xn = X + ((long long)nn * 2 + h) * nrhs;
#pragma unroll
        for (int u = 0; u < RT; u++) o.x[u] = Pk<T, PK>::get(xn + rr[u], lo);
    };
    auto mult = [&](const Step &o) {
        typename Pk<T, PK>::elem av[RT];
#pragma unroll
        for (int u = 0; u < RT; u++) av[u] = fac * o.x[u];
#pragma unroll
        for (int c = 0; c < 2; c++) {
            // alpha lanes take R[c]; beta lanes (khat x R)[c]: (-R_phi, R_theta)
            const cpx<T> oth = o.v[1 - c];
            const cpx<T> bv = s == 0 ? o.v[c] : (c == 0 ? mk<T>(-oth.re, -oth.im) : oth);
            if constexpr (PK) {
#pragma unroll
                for (int u = 0; u < RT; u++) {
                    dre[c][u] = Mf<T>::mma(av[u], bv.re, dre[c][u]);
                    dim[c][u] = Mf<T>::mma(av[u], bv.im, dim[c][u]);
                }
            } else {
                cmfma<T, RT>(dre[c], dim[c], av, bv);
            }
        }
    };
    // steps with both RWGs inside the box (samples past K and right-hand
    // sides past nrhs read clamped, valid elements; only their own outputs,
    // which are never stored, see them)
    const int nfull = (n1 - n0) / 2;
    auto rwg = [&](int step) { return n0 + 2 * min(step, nfull - 1) + (kk >> 1); };
    if (nfull > 0) {
        Step s0, s1;
        load(rwg(0), s0);
        for (int step = 0; step < nfull; step += 2) {
            load(rwg(step + 1), s1);
            mult(s0);
            if (step + 1 >= nfull) break;
            load(rwg(step + 2), s0);
            mult(s1);
        }
    }
    if (n0 + 2 * nfull < n1) {   // the last RWG of an odd box: lanes of the absent second RWG feed zeros
        const int nn = n0 + 2 * nfull + (kk >> 1);
        Step o;
        load(min(nn, n1 - 1), o);
        if (nn >= n1) {
            o.v[0] = o.v[1] = mk<T>(0, 0);
#pragma unroll
            for (int u = 0; u < RT; u++) o.x[u] = typename Pk<T, PK>::elem{};
        }
        mult(o);
    }
#pragma unroll
    for (int c = 0; c < 2; c++) {
        if constexpr (PK) fold_rows<RT>(dre[c], dim[c]);
        if (q >= K) continue;
#pragma unroll
        for (int u = 0; u < RT; u++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int r = (rg * RT + u) * 16 + Mf<T>::row(kk, v);
                if (r < nrhs) U[pidx_m(b, c, r, q, nrhs, ks)] = mk<T>(dre[c][u][v], dim[c][u][v]);
            }
    }
}

// Radiation of 2 to 15 right-hand sides in single precision, on the 16-block
// 4 x 4 x 1 product: lane l holds sample l of the wave's 64 as the block's
// column and right-hand side l % 4 of a group as its row, and gets its sample's
// sums for the group's four right-hand sides.  Every MFMA is one fused
// multiply-add per sum, so the sums
//   U_t += alpha R_t - beta R_p,  U_p += alpha R_p + beta R_t
// (EM pair: alpha = x1, beta = -x2; C block: alpha = x2 / 2, beta = x1 / 2) are
// those of the one-right-hand-side kernel term for term: a vector's patterns do
// not depend on how many others share the product.  (The translation amplifies
// their rounding by 1e4 to 1e5, so that other orders differ by 1e-5 of the
// product.)  Wave = (box, 64 samples) x NG groups; a pattern sample is loaded
// once for all groups.  Two RWGs are multiplied while the next two are loaded.
// Sphere of radius 8 wavelengths (276 480 RWGs), 2 right-hand sides: 0.319 ms on
// the vector units, 0.266 ms like this; ellipsoid of 48 000, 7:
// 0.219, 0.084 ms (0.071 on packed 16 x 16 x 4 tiles, which add up two RWGs at once).
template <int NG>
__global__ __launch_bounds__(256) void k_radiate_few(int op, int nbox, int K, int ks, int nqc,
                                                     const int *__restrict__ box_start,
                                                     const cpx<float> *__restrict__ R,
                                                     const cpx<float> *__restrict__ X, cpx<float> *__restrict__ U,
                                                     int nrhs)
{
    typedef Mf<float>::v4 v4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long blk = xcd_block_m(((long long)nbox * nqc + 3) / 4);
    if (blk < 0) return;
    const long long w = blk * 4 + wave;
    if (w >= (long long)nbox * nqc) return;
    const int b = (int)(w / nqc), q = (int)(w % nqc) * 64 + lane;
    const cpx<float> *Rq = R + 2LL * min(q, K - 1);   // samples past K read a valid one, store nothing
    const int n0 = box_start[b], n1 = box_start[b + 1];
    const int ha = op == MLFMA_OP_EM ? 0 : 1;         // half of X that gives alpha
    const float fa = op == MLFMA_OP_EM ? 1.f : 0.5f, fb = op == MLFMA_OP_EM ? -1.f : 0.5f;
    int rr[NG];
#pragma unroll
    for (int g = 0; g < NG; g++) rr[g] = min(g * 4 + (lane & 3), nrhs - 1);
    v4 tre[NG], tim[NG], pre[NG], pim[NG];
#pragma unroll
    for (int g = 0; g < NG; g++) tre[g] = tim[g] = pre[g] = pim[g] = v4{0, 0, 0, 0};
    struct Step {
        cpx<float> t[2], p[2], a[2][NG], b[2][NG];
    };
    auto load = [&](int n, Step &o) {
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int nn = min(n + u, n1 - 1);
            load_pair(Rq + (long long)nn * K * 2, o.t[u], o.p[u]);
            const cpx<float> *xa = X + (2LL * nn + ha) * nrhs, *xb = X + (2LL * nn + 1 - ha) * nrhs;
#pragma unroll
            for (int g = 0; g < NG; g++) {
                o.a[u][g] = xa[rr[g]];
                o.b[u][g] = xb[rr[g]];
            }
        }
    };
    auto mma = [](float a, float v, v4 c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(a, v, c, 0, 0, 0); };
    auto one = [&](const Step &o, int u) {
        const cpx<float> t = o.t[u], p = o.p[u];
#pragma unroll
        for (int g = 0; g < NG; g++) {
            const cpx<float> al = fa * o.a[u][g], be = fb * o.b[u][g];
            tre[g] = mma(al.re, t.re, tre[g]);
            tim[g] = mma(al.re, t.im, tim[g]);
            pre[g] = mma(al.re, p.re, pre[g]);
            pim[g] = mma(al.re, p.im, pim[g]);
            tre[g] = mma(-al.im, t.im, tre[g]);
            tim[g] = mma(al.im, t.re, tim[g]);
            pre[g] = mma(-al.im, p.im, pre[g]);
            pim[g] = mma(al.im, p.re, pim[g]);
            tre[g] = mma(-be.re, p.re, tre[g]);
            tim[g] = mma(-be.re, p.im, tim[g]);
            pre[g] = mma(be.re, t.re, pre[g]);
            pim[g] = mma(be.re, t.im, pim[g]);
            tre[g] = mma(be.im, p.im, tre[g]);
            tim[g] = mma(-be.im, p.re, tim[g]);
            pre[g] = mma(-be.im, t.im, pre[g]);
            pim[g] = mma(be.im, t.re, pim[g]);
        }
    };
    auto mult = [&](int n, const Step &o) {
        one(o, 0);
        if (n + 1 < n1) one(o, 1);
    };
    Step s0, s1;
    load(n0, s0);
    for (int n = n0; n < n1; n += 4) {
        load(n + 2, s1);
        mult(n, s0);
        if (n + 2 >= n1) break;
        load(n + 4, s0);
        mult(n + 2, s1);
    }
    if (q >= K) return;
#pragma unroll
    for (int g = 0; g < NG; g++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int r = g * 4 + v;
            if (r >= nrhs) continue;
            U[pidx_m(b, 0, r, q, nrhs, ks)] = mk<float>(tre[g][v], tim[g][v]);
            U[pidx_m(b, 1, r, q, nrhs, ks)] = mk<float>(pre[g][v], pim[g][v]);
        }
}

// Sum of the four waves' accumulators of one work item, in wave order, left
// in wave 0 (true there, false in the others).
template <class T, class A>
__device__ inline bool sum_parts(int wave, int lane, A &dre, A &dim)
{
    __shared__ T red[3][8][64];
    if (wave > 0)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            red[wave - 1][v][lane] = dre[v];
            red[wave - 1][4 + v][lane] = dim[v];
        }
    __syncthreads();
    if (wave > 0) return false;
#pragma unroll
    for (int p = 0; p < 3; p++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            dre[v] += red[p][v][lane];
            dim[v] += red[p][4 + v][lane];
        }
    return true;
}

// Below this many (item, right-hand-side tile) pairs the receive and the near
// field give each to a workgroup of four waves that share its inner index
// (SPLIT = 4), instead of one wave each: with few waves the chip waits on the
// serial chain over the inner index.  The receive's chain is short (16 blocks
// of samples), so the sum over LDS pays only below two waves per SIMD (1 080
// RWGs, 5 right-hand sides, complex128: 21 -> 11.5 us; 17 280 RWGs, 2 300
// pairs and more: 60 -> 72 us); the near field's is a few hundred columns
// (1 080 RWGs: 30 -> 13.5 us; 48 000 RWGs, complex64, 16 right-hand sides: 185
// -> 161 us), up to where the waves fill the chip by themselves (box of 27 225
// RWGs, 64 right-hand sides, 14 900 pairs, complex128: 537 -> 556 us; sphere of
// 122 880, 16: 403 -> 495 us).
constexpr long long RECEIVE_SPLIT_BELOW = 2048, NEAR_SPLIT_BELOW = 12288;

// Receive.  Work item = (leaf box, row tile of 16 rows (RWG m, half h),
// tile of 16 right-hand sides), one per wave, right-hand-side tiles
// innermost; D[i = (m, h)][j = rhs], inner index k = (component, sample).
// Rows: h = 0 uses (Pt, Pp), h = 1 uses (Pp, -Pt), with P = conj(R) for the
// EM pair and P = Q for the C block, weights wq folded in.  The samples go
// in blocks of 16: lane group kk (lanes 16 kk .. 16 kk + 15) loads samples
// 4 kk .. 4 kk + 3 of the block for its row (both components, 64 contiguous
// bytes) and for its right-hand side (32 bytes per component), and step u
// of the block takes sample 4 kk + u in every lane group: the same order of
// the inner index for the A and B operands, so that each lane reads whole
// runs of samples.  Two blocks are in flight while one is multiplied.
// V holds large terms that cancel in the sum over the samples, so in complex64
// the rounding of that sum shows in the product (1e-5 of it on coarse meshes).
// Up to 15 right-hand sides (from 4 on: RECEIVE_ROWS_MAX) WIDE multiplies and adds in double (the operands
// are exact there): 0.110 ms on the ellipsoid of 48 000 RWGs, 7 right-hand
// sides, against 0.084 with single-precision sums, whose products differ from
// those of one right-hand side by up to 1.2e-5 instead of 7e-6.  From 16 on
// the sums are single ones in sample order, never split.
template <class T, bool PK, int SPLIT, bool WIDE>
__global__ __launch_bounds__(256) void k_receive_mfma(int op, int nitem, const int2 *__restrict__ items, int K, int ks,
                                                      const int *__restrict__ box_start,
                                                      const cpx<T> *__restrict__ R,
                                                      const cpx<T> *__restrict__ Q, const T *__restrict__ wq,
                                                      const cpx<T> *__restrict__ V, cpx<T> *__restrict__ Y,
                                                      int nrhs)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nrt = (nrhs + 15) / 16;
    const long long blk = xcd_block_m(((long long)nitem * nrt * SPLIT + 3) / 4);
    if (blk < 0) return;
    const long long w = SPLIT == 4 ? blk : blk * 4 + wave;
    if (w >= (long long)nitem * nrt) return;
    const int part = SPLIT == 4 ? wave : 0;   // this wave's share of the inner index
    const int2 it = items[w / nrt];
    const int rt = (int)(w % nrt);
    const int b = it.x, tile = it.y;
    const int n0 = box_start[b], rows = 2 * (box_start[b + 1] - n0);
    const int lo = lane & 15, kk = lane >> 4;
    const cpx<T> *pat = op == MLFMA_OP_EM ? R : Q;
    const bool cj = op == MLFMA_OP_EM;
    const int row = tile * 16 + lo, r = PK ? lo & 7 : rt * 16 + lo;
    const bool mok = row < rows, rok = r < nrhs;
    const int h = row & 1;
    const cpx<T> *pm = pat + (long long)(n0 + (mok ? row / 2 : 0)) * K * 2;
    const cpx<T> *v0 = V + ((long long)(b * 2) * nrhs + (rok ? r : 0)) * ks;
    const long long vstep = (long long)nrhs * ks;   // second component of V
    const int nblk = (K + 15) / 16;
    // the lane's A operand in component pass c is one component of its row's
    // pattern: theta for (h, c) = (0, 0), phi for (0, 1) and (1, 0), minus
    // theta for (1, 1)
    const int comp0 = h == 0 ? 0 : 1, comp1 = h == 0 ? 1 : 0;
    const T sg1 = h == 1 ? T(-1) : T(1);
    struct Blk {
        cpx<T> q[4][2];   // pattern, samples x components
        typename Pk<T, PK>::elem v[2][4];   // V, components x samples
        T w[4];
    };
    auto load = [&](int bk, Blk &o) {
        const int q0 = bk * 16 + kk * 4;
        if (bk * 16 + 16 <= K) {   // the whole block (wave-uniform: one path per block)
            // rows past the box and right-hand sides past nrhs read row 0 /
            // right-hand side 0 (pm, v0 are clamped): they feed only D rows
            // and columns that are never stored
#pragma unroll
            for (int u = 0; u < 4; u++) {
                o.w[u] = wq[q0 + u];
                o.q[u][0] = pm[2 * (q0 + u)];
                o.q[u][1] = pm[2 * (q0 + u) + 1];
                o.v[0][u] = Pk<T, PK>::get(v0 + q0 + u, lo);
                o.v[1][u] = Pk<T, PK>::get(v0 + vstep + q0 + u, lo);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int q = q0 + u;
                const bool qok = q < K;
                o.w[u] = qok ? wq[q] : T(0);
                o.q[u][0] = mok && qok ? pm[2 * q] : mk<T>(0, 0);
                o.q[u][1] = mok && qok ? pm[2 * q + 1] : mk<T>(0, 0);
                o.v[0][u] = o.v[1][u] = typename Pk<T, PK>::elem{};
                if (rok && qok) {
                    o.v[0][u] = Pk<T, PK>::get(v0 + q, lo);
                    o.v[1][u] = Pk<T, PK>::get(v0 + vstep + q, lo);
                }
            }
        }
    };
    using A = std::conditional_t<WIDE, double, T>;   // the sums' type
    typedef typename Mf<A>::v4 v4;
    v4 dre = {0, 0, 0, 0}, dim = {0, 0, 0, 0};
    // DEPTH blocks in flight: block bk + DEPTH is loaded while block bk is
    // multiplied (one in double precision, where a block takes 72
    // registers).  The register sets take turns (no copies), and every path
    // issues the same loads (past the last block they repeat it), so that
    // the wait before a product counts the newer blocks' loads as in flight.
    constexpr int DEPTH = sizeof(T) == 8 ? 1 : 2;
    auto mult = [&](const Blk &cur) {
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int cp = c == 0 ? comp0 : comp1;
                cpx<T> p = cp ? cur.q[u][1] : cur.q[u][0];   // a select, not a dynamic register index
                if (cj) p = conjg(p);
                const cpx<T> a = ((c == 1 ? sg1 : T(1)) * cur.w[u]) * p;
                const cpx<A> aw = {(A)a.re, (A)a.im};
                if constexpr (PK) Pk<A, true>::mma(aw, (A)cur.v[c][u], dre, dim);
                else Pk<A, false>::mma(aw, {(A)cur.v[c][u].re, (A)cur.v[c][u].im}, dre, dim);
            }
    };
    const int bk0 = part * nblk / SPLIT, bk1 = (part + 1) * nblk / SPLIT;
    auto at = [&](int bk) { return min(bk, bk1 - 1); };
    if (bk0 < bk1) {
        Blk b0, b1, b2;
        load(bk0, b0);
        if constexpr (DEPTH == 2) {
            load(at(bk0 + 1), b1);
            for (int bk = bk0; bk < bk1; bk += 3) {
                load(at(bk + 2), b2);
                mult(b0);
                if (bk + 1 >= bk1) break;
                load(at(bk + 3), b0);
                mult(b1);
                if (bk + 2 >= bk1) break;
                load(at(bk + 4), b1);
                mult(b2);
            }
        } else {
            for (int bk = bk0; bk < bk1; bk += 2) {
                load(at(bk + 1), b1);
                mult(b0);
                if (bk + 1 >= bk1) break;
                load(at(bk + 2), b0);
                mult(b1);
            }
        }
    }
    if constexpr (SPLIT == 4)
        if (!sum_parts<A>(wave, lane, dre, dim)) return;
    if constexpr (PK) fold_cols(dre, dim);
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const int orow = tile * 16 + Mf<A>::row(kk, v);
        if (orow < rows && rok && (!PK || lo < 8)) {
            cpx<T> &y = Y[((long long)(n0 + orow / 2) * 2 + (orow & 1)) * nrhs + r];
            y = mk<T>((T)(y.re + dre[v]), (T)(y.im + dim[v]));
        }
    }
}

// Near field.  Work item = (leaf box b, row tile of 16 rows (RWG m, half
// h), tile of 16 right-hand sides), one per wave, right-hand-side tiles
// innermost so that neighbouring waves share the value rows.  The box's
// columns are the RWGs of its <= 27 adjacent boxes, concatenated (the order
// the stored (A, B) rows follow), listed in cols[col_off[b] ..].
// D[i = (m, h)][j = rhs] with inner index k = (column, half h'): two columns
// per MFMA step, taken in blocks of eight columns (four steps) whose inner
// index is permuted so that each lane reads its row's entries as runs.  The
// 2 x 2 block of a pair is [[A, -B], [B, A]].  The identity
// terms of the C block (Gram and rotated Gram, same triangle only) are added
// in the epilogue; Y is overwritten.
// A row sums several hundred products one after another, where the vector
// kernel of one right-hand side adds up 64 short sums in a tree.  Single
// precision throughout leaves complex64 2 to 5 times as far from the
// complex128 product (sphere of 122 880 RWGs, EM pair: 3.8e-7 packed, 5.4e-7
// full, against 0.98e-7), so from 3 (NEAR_TILE_MAX) to 15 right-hand sides WIDE
// sums in double:
// packed, on FP64 matrix cores (0.36e-7), full, the eight products of a step in
// single precision and the steps in double on the vector units (0.54e-7).
// Ellipsoid of 48 000 RWGs: 7 right-hand sides 0.138 -> 0.164 ms (in steps,
// 0.172), 15 0.161 -> 0.202 ms (on FP64 matrix cores 0.262), both at 8 and 6 waves
// per SIMD (7 and 5 without the bound: 0.167, 0.218).  Then the vector units are
// the bound: 84 instructions per 8 columns, 12 of them conversions.
template <class T, bool PK, int SPLIT, bool WIDE>
__global__ __launch_bounds__(256, WIDE ? (PK ? 8 : 6) : 1) void k_near_mfma(int nitem, const int2 *__restrict__ items,
                                                   const int *__restrict__ box_start,
                                                   const int *__restrict__ col_off, const int *__restrict__ cols,
                                                   const long long *__restrict__ val_off,
                                                   const cpx<T> *__restrict__ vals,
                                                   const int *__restrict__ id_start, const int *__restrict__ id_col,
                                                   const T *__restrict__ id_w, const cpx<T> *__restrict__ X,
                                                   cpx<T> *__restrict__ Y, int nrhs)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nrt = (nrhs + 15) / 16;
    const long long blk = xcd_block_m(((long long)nitem * nrt * SPLIT + 3) / 4);
    if (blk < 0) return;
    const long long w = SPLIT == 4 ? blk : blk * 4 + wave;
    if (w >= (long long)nitem * nrt) return;
    const int part = SPLIT == 4 ? wave : 0;   // this wave's share of the inner index
    const int2 it = items[w / nrt];
    const int rt = (int)(w % nrt);
    const int b = it.x, tile = it.y;
    const int n0 = box_start[b], rows = 2 * (box_start[b + 1] - n0);
    const int *cl = cols + col_off[b];
    const int ncols = col_off[b + 1] - col_off[b];
    const int lo = lane & 15, kk = lane >> 4;
    const int jc = kk >> 1, hp = kk & 1;
    const int row = tile * 16 + lo, r = PK ? lo & 7 : rt * 16 + lo;
    const bool mok = row < rows, rok = r < nrhs;
    const int h = row & 1;
    const cpx<T> *vr = vals + 2 * (val_off[b] + (long long)(mok ? row / 2 : 0) * ncols);
    const int vsel = h == hp ? 0 : 1;
    const T vsg = (h == 0 && hp == 1) ? T(-1) : T(1);
    // column indices 64 at a time, one per lane, handed out by lane shuffles
    // (so the x load of a step does not wait for an index load)
    int cbase = -64, myc = 0;
    auto cols_for = [&](int j0) {
        if (j0 >= cbase + 64) {   // j0 is even: a step never straddles two groups
            cbase = j0 - j0 % 64;
            myc = cl[min(cbase + lane, ncols - 1)];
        }
    };
    using M = std::conditional_t<WIDE && PK, double, T>;   // the products' type
    using A = std::conditional_t<WIDE, double, T>;         // the sums' type
    typename Mf<A>::v4 dre = {0, 0, 0, 0}, dim = {0, 0, 0, 0};
    typedef typename Pk<T, PK>::elem elem;
    auto mma = [&](cpx<T> a, elem bv) {
        if constexpr (PK) {
            Pk<M, true>::mma({(M)a.re, (M)a.im}, (M)bv, dre, dim);
        } else if constexpr (WIDE) {
            typename Mf<T>::v4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};   // one step's eight products per sum
            Pk<T, false>::mma(a, bv, re, im);
#pragma unroll
            for (int v = 0; v < 4; v++) {
                dre[v] += (A)re[v];
                dim[v] += (A)im[v];
            }
        } else {
            Pk<T, false>::mma(a, bv, dre, dim);
        }
    };
    const int rc = rok ? r : 0;
    // Blocks of 8 columns, four MFMA steps: lane group kk takes columns
    // j = j0 + 2 kk + c (c = 0, 1) and step u = 2 c + h' feeds column
    // j0 + 2 kk + c, half h' -- the same inner index for the A and B operands
    // -- so that a lane reads the (A, B) entries of its two columns as one
    // run of its row (rows past the tile and right-hand sides past nrhs read
    // clamped, valid elements that only feed outputs never stored).  The next
    // block's operands are in flight while a block is multiplied (two
    // register sets taking turns; past the last block the loads repeat it).
    const int nb8 = ncols / 8;
    const T sgb = h == 0 ? T(-1) : T(1);   // B's sign where h' != h
    struct Blk8 {
        cpx<T> v[4];   // A, B of the lane's first column, A, B of its second
        elem x[4];     // x of (column c, half h') at 2 c + h'
    };
    auto load8 = [&](int bi, Blk8 &o) {
        const int j0 = bi * 8, j = j0 + 2 * kk;
        cols_for(j0);
#pragma unroll
        for (int e = 0; e < 4; e++) o.v[e] = vr[2 * j + e];
        const int c0 = __shfl(myc, j - cbase), c1 = __shfl(myc, j + 1 - cbase);
#pragma unroll
        for (int hh = 0; hh < 2; hh++) {
            o.x[hh] = Pk<T, PK>::get(X + ((long long)c0 * 2 + hh) * nrhs + rc, lo);
            o.x[2 + hh] = Pk<T, PK>::get(X + ((long long)c1 * 2 + hh) * nrhs + rc, lo);
        }
    };
    auto mult8 = [&](const Blk8 &o) {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int c = u >> 1, hh = u & 1;
            const cpx<T> av = hh == h ? o.v[2 * c] : sgb * o.v[2 * c + 1];
            mma(av, o.x[u]);
        }
    };
    const int bi0 = part * nb8 / SPLIT, bi1 = (part + 1) * nb8 / SPLIT;
    if (bi0 < bi1) {
        Blk8 s0, s1;
        load8(bi0, s0);
        for (int bi = bi0; bi < bi1; bi += 2) {
            load8(min(bi + 1, bi1 - 1), s1);
            mult8(s0);
            if (bi + 1 >= bi1) break;
            load8(min(bi + 2, bi1 - 1), s0);
            mult8(s1);
        }
    }
    // the last ncols % 8 columns, two per step (lane group kk: column j0 +
    // kk / 2, half kk % 2)
    auto load = [&](int j0, cpx<T> &a, elem &bv) {
        cols_for(j0);
        const int j = j0 + jc;
        const bool jok = j < ncols;
        const int col = __shfl(myc, min(j, ncols - 1) - cbase);
        a = mk<T>(0, 0);
        bv = elem{};
        if (jok && mok) {
            // [[A, -B], [B, A]]: the lane needs A on the diagonal, B (or -B) off it
            const cpx<T> v = vr[2 * j + vsel];
            a = mk<T>(vsg * v.re, vsg * v.im);
        }
        if (jok && rok) bv = Pk<T, PK>::get(X + ((long long)col * 2 + hp) * nrhs + r, lo);
    };
    for (int j0 = part == SPLIT - 1 ? nb8 * 8 : ncols; j0 < ncols; j0 += 2) {
        cpx<T> a;
        elem bv;
        load(j0, a, bv);
        mma(a, bv);
    }
    if constexpr (SPLIT == 4)
        if (!sum_parts<A>(wave, lane, dre, dim)) return;
    if constexpr (PK) fold_cols(dre, dim);
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const int orow = tile * 16 + Mf<M>::row(kk, v);
        if (orow >= rows || !rok || (PK && lo >= 8)) continue;
        const int m = n0 + orow / 2, oh = orow & 1;
        cpx<T> y = mk<T>((T)dre[v], (T)dim[v]);
        if (id_start) {
            for (int e = id_start[m]; e < id_start[m + 1]; e++) {
                const long long col = id_col[e];
                const T g = id_w[2 * e], gx = id_w[2 * e + 1];
                const cpx<T> x1 = X[(col * 2) * nrhs + r], x2 = X[(col * 2 + 1) * nrhs + r];
                if (oh == 0) {
                    axpy_to(y, g, x1);
                    axpy_to(y, T(0.5) * gx, x2);
                } else {
                    axpy_to(y, T(0.5) * g, x2);
                }
            }
        }
        Y[((long long)m * 2 + oh) * nrhs + r] = y;
    }
}

}  // namespace

template <class T>
void launch_near_mfma(int nitem, const int2 *items, const int *box_start, const int *col_off, const int *cols,
                      const long long *val_off, const cpx<T> *vals, const int *id_start, const int *id_col,
                      const T *id_w, const cpx<T> *X, cpx<T> *Y, int nrhs, hipStream_t s)
{
    const long long nw = (long long)nitem * ((nrhs + 15) / 16);
    const bool split = nw < NEAR_SPLIT_BELOW;
    const long long nblk = split ? nw : (nw + 3) / 4;
    if (nblk <= 0) return;
#define NEAR(PK_, SPLIT_, WIDE_)                                                                                     \
    hipLaunchKernelGGL((k_near_mfma<T, PK_, SPLIT_, WIDE_>), dim3(xcd_grid_m(nblk)), dim3(256), 0, s, nitem, items,   \
                       box_start, col_off, cols, val_off, vals, id_start, id_col, id_w, X, Y, nrhs)
    constexpr bool W = sizeof(T) == 4;
    if (nrhs <= 8) {
        if (split) NEAR(true, 4, W);
        else NEAR(true, 1, W);
    } else if (nrhs < 16) {
        if (split) NEAR(false, 4, W);
        else NEAR(false, 1, W);
    } else {
        if (split) NEAR(false, 4, false);
        else NEAR(false, 1, false);
    }
#undef NEAR
}

template <class T>
void launch_radiate_mfma(int op, int nbox, int K, int ks, const int *box_start, const cpx<T> *R, const cpx<T> *X, cpx<T> *U,
                         int nrhs, hipStream_t s)
{
    const int nqt = (K + 15) / 16;
    const int rt = nrhs >= 32 ? 2 : 1;   // right-hand-side tiles per wave
    const long long nblk = (long long)nbox * ((nqt + 3) / 4) * ((nrhs + 16 * rt - 1) / (16 * rt));
    if (nblk <= 0) return;
    const dim3 grid(xcd_grid_m(nblk)), block(256);
#define RADIATE(RT_, PK_) \
    hipLaunchKernelGGL((k_radiate_mfma<T, RT_, PK_>), grid, block, 0, s, op, nbox, K, ks, nqt, box_start, R, X, U, nrhs)
    if constexpr (sizeof(T) == 4) {
        if (rt == 2) RADIATE(2, false);
        else if (nrhs >= 16) RADIATE(1, false);
        else {
            const int nqc = (K + 63) / 64;
            const dim3 gridf(xcd_grid_m(((long long)nbox * nqc + 3) / 4));
#define FEW(NG_) \
    hipLaunchKernelGGL((k_radiate_few<NG_>), gridf, block, 0, s, op, nbox, K, ks, nqc, box_start, R, X, U, nrhs)
            if (nrhs <= 4) FEW(1);
            else if (nrhs <= 8) FEW(2);
            else if (nrhs <= 12) FEW(3);
            else FEW(4);
#undef FEW
        }
    } else {
        if (rt == 2) RADIATE(2, false);
        else if (nrhs > 8) RADIATE(1, false);
        else RADIATE(1, true);
    }
#undef RADIATE
}

template <class T>
void launch_receive_mfma(int op, int nitem, const int2 *items, int K, int ks, const int *box_start, const cpx<T> *R,
                         const cpx<T> *Q, const T *wq, const cpx<T> *V, cpx<T> *Y, int nrhs, hipStream_t s)
{
    const long long nw = (long long)nitem * ((nrhs + 15) / 16);
    const bool wide = sizeof(T) == 4 && nrhs < 16, split = nw < RECEIVE_SPLIT_BELOW && (wide || sizeof(T) == 8);
    const long long nblk = split ? nw : (nw + 3) / 4;
    if (nblk <= 0) return;
#define RECEIVE(PK_, SPLIT_, WIDE_)                                                                                 \
    hipLaunchKernelGGL((k_receive_mfma<T, PK_, SPLIT_, WIDE_>), dim3(xcd_grid_m(nblk)), dim3(256), 0, s, op, nitem, \
                       items, K, ks, box_start, R, Q, wq, V, Y, nrhs)
    constexpr bool W = sizeof(T) == 4;
    if (nrhs <= 8) {
        if (split) RECEIVE(true, 4, W);
        else RECEIVE(true, 1, W);
    } else if (wide || sizeof(T) == 8) {
        if (split) RECEIVE(false, 4, W);
        else RECEIVE(false, 1, W);
    } else {
        RECEIVE(false, 1, false);
    }
#undef RECEIVE
}

#define MFMA_INST(T)                                                                                                 \
    template void launch_near_mfma<T>(int, const int2 *, const int *, const int *, const int *, const long long *,    \
                                      const cpx<T> *, const int *, const int *, const T *, const cpx<T> *, cpx<T> *,  \
                                      int, hipStream_t);                                                              \
    template void launch_radiate_mfma<T>(int, int, int, int, const int *, const cpx<T> *, const cpx<T> *, cpx<T> *, int,   \
                                         hipStream_t);                                                                \
    template void launch_receive_mfma<T>(int, int, const int2 *, int, int, const int *, const cpx<T> *, const cpx<T> *,    \
                                         const T *, const cpx<T> *, cpx<T> *, int, hipStream_t);
MFMA_INST(float)
MFMA_INST(double)
#undef MFMA_INST

}  // namespace mlfma
