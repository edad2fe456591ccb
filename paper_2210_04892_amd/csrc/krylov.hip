// Vector kernels of the outer GMRES (restarted, one Krylov space per
// right-hand-side column).  Vectors are column-major blocks: element (n, r)
// of a block with leading dimension ld sits at r * ld + n.  Inner products
// are accumulated in double precision in a fixed order (partial sums per
// chunk of rows, then a second pass over the chunks), so results do not
// depend on the launch.
//
// Bound by latency: the vectors of an Arnoldi step (77 760 unknowns: 0.6 MB
// each) take a microsecond or two to read.  So a step is six kernels with no
// host round trip (inner products, their sum, w -= V h with the next inner
// products of the rows just written, their sum, the second pass with |w|^2,
// the normalisation) and one fetch of all its numbers, the inner products are
// spread over vectors as well as rows, and chunks are summed by a wave each.
// 38 880 RWGs, complex64, one column, ten steps with products of 0.23 ms: 4.92
// ms with nine kernels and four round trips a step on a quarter of the
// workgroups, 3.88 ms like this.
#include "device.hpp"

namespace mlfma {

namespace {

constexpr int KT = 256;

__device__ inline double wave_sum_d(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// this wave's part of the inner product of rows n0 .. n1 of two vectors
template <class T>
__device__ inline cpx<double> wave_dot(const cpx<T> *v, const cpx<T> *w, long long n0, long long n1)
{
    double sre = 0, sim = 0;
    for (long long k = n0 + threadIdx.x; k < n1; k += KT) {
        const cpx<T> a = v[k], b = w[k];
        sre += (double)a.re * (double)b.re + (double)a.im * (double)b.im;
        sim += (double)a.re * (double)b.im - (double)a.im * (double)b.re;
    }
    return {wave_sum_d(sre), wave_sum_d(sim)};
}

// one row chunk's sums of up to DOT_BATCH inner products: lane 0 of every wave
// leaves its part in red, and after one barrier a thread per product adds the
// waves' parts up
constexpr int DOT_BATCH = 4;
template <class T, class F>
__device__ inline void chunk_dots(int i0, int i1, long long n0, long long n1, const cpx<T> *wr, F vec,
                                  cpx<double> *part, int nchunk, int c, int nrhs, int r)
{
    __shared__ cpx<double> red[DOT_BATCH][KT / 64];
    for (int ib = i0; ib < i1; ib += DOT_BATCH) {
        const int nb = min(DOT_BATCH, i1 - ib);
        for (int i = 0; i < nb; i++) {
            const cpx<double> d = wave_dot<T>(vec(ib + i), wr, n0, n1);
            if ((threadIdx.x & 63) == 0) red[i][threadIdx.x >> 6] = d;
        }
        __syncthreads();
        if ((int)threadIdx.x < nb) {
            double a = 0, b = 0;
            for (int k = 0; k < KT / 64; k++) {
                a += red[threadIdx.x][k].re;
                b += red[threadIdx.x][k].im;
            }
            part[((long long)(ib + threadIdx.x) * nchunk + c) * nrhs + r] = {a, b};
        }
        __syncthreads();
    }
}

// part[(i * nchunk + c) * nrhs + r] = sum over rows of chunk c of
// conj(V_i(n, r)) w(n, r); workgroup = (chunk, column, DOT_BATCH vectors)
template <class T>
__global__ __launch_bounds__(KT) void k_dots(const cpx<T> *__restrict__ V, long long vstride, long long ldv, int nv,
                                             const cpx<T> *__restrict__ w, long long ldw, long long n, long long chunk,
                                             cpx<double> *__restrict__ part, int nchunk, int nrhs)
{
    const int c = blockIdx.x, r = blockIdx.y, i0 = blockIdx.z * DOT_BATCH;
    const long long n0 = (long long)c * chunk, n1 = n0 + chunk < n ? n0 + chunk : n;
    chunk_dots<T>(i0, min(nv, i0 + DOT_BATCH), n0, n1, w + (long long)r * ldw,
                  [&](int i) { return V + i * vstride + (long long)r * ldv; }, part, nchunk, c, nrhs, r);
}

// sum over the chunks of one product's parts, in all lanes of the wave
__device__ inline cpx<double> sum_chunks(const cpx<double> *part, int nchunk, int nrhs)
{
    double a = 0, b = 0;
    for (int c = threadIdx.x & 63; c < nchunk; c += 64) {
        const cpx<double> p = part[(long long)c * nrhs];
        a += p.re;
        b += p.im;
    }
    return {wave_sum_d(a), wave_sum_d(b)};
}

// out[i * nrhs + r] = sum over chunks of part, a wave each
__global__ __launch_bounds__(KT) void k_sum_parts(const cpx<double> *__restrict__ part, int nv, int nchunk, int nrhs,
                                                  cpx<double> *__restrict__ out)
{
    const int g = blockIdx.x * (KT / 64) + (threadIdx.x >> 6);
    if (g >= nv * nrhs) return;
    const cpx<double> s = sum_chunks(part + (long long)(g / nrhs) * nchunk * nrhs + g % nrhs, nchunk, nrhs);
    if ((threadIdx.x & 63) == 0) out[g] = s;
}

// one row of w(n, r) + sign * sum_{i < nv} V_i(n, r) h[i * nrhs + r]
template <class T>
__device__ inline cpx<T> combine_row(const cpx<T> *v, long long vstride, int nv, const cpx<double> *h, int nrhs,
                                     double sign, cpx<T> o)
{
    double are = 0, aim = 0;
    for (int i = 0; i < nv; i++) {
        const cpx<T> x = v[i * vstride];
        const cpx<double> c = h[(long long)i * nrhs];
        are += (double)x.re * c.re - (double)x.im * c.im;
        aim += (double)x.re * c.im + (double)x.im * c.re;
    }
    return {(T)((double)o.re + sign * are), (T)((double)o.im + sign * aim)};
}

// w(n, r) += sign * sum_{i < nv} V_i(n, r) h[i * nrhs + r]
template <class T>
__global__ __launch_bounds__(KT) void k_combine(const cpx<T> *__restrict__ V, long long vstride, long long ldv, int nv,
                                                const cpx<double> *__restrict__ h, double sign, cpx<T> *__restrict__ w,
                                                long long ldw, long long n, int nrhs)
{
    const long long g = (long long)blockIdx.x * KT + threadIdx.x;
    if (g >= n * nrhs) return;
    const int r = (int)(g / n);
    const long long k = g % n;
    cpx<T> &o = w[(long long)r * ldw + k];
    o = combine_row<T>(V + (long long)r * ldv + k, vstride, nv, h + r, nrhs, sign, o);
}

// A Gram-Schmidt pass on one row chunk of a column: w -= V h, then the chunk's
// part of the next inner products of the new w, with V_i (norm = 0) or with
// itself (norm = 1): its rows are done when the workgroup's threads, each of
// which reads only rows it wrote, come to them.
template <class T>
__global__ __launch_bounds__(KT) void k_orthogonalise(const cpx<T> *__restrict__ V, long long vstride, int nv,
                                                      const cpx<double> *__restrict__ h, cpx<T> *w, long long n,
                                                      long long chunk, cpx<double> *__restrict__ part, int nchunk,
                                                      int nrhs, int norm)
{
    const int c = blockIdx.x, r = blockIdx.y;
    const long long n0 = (long long)c * chunk, n1 = n0 + chunk < n ? n0 + chunk : n;
    const cpx<T> *vr = V + (long long)r * n;
    cpx<T> *wr = w + (long long)r * n;
    for (long long k = n0 + threadIdx.x; k < n1; k += KT)
        wr[k] = combine_row<T>(vr + k, vstride, nv, h + r, nrhs, -1.0, wr[k]);
    if (norm)
        chunk_dots<T>(0, 1, n0, n1, wr, [&](int) { return (const cpx<T> *)wr; }, part, nchunk, c, nrhs, r);
    else
        chunk_dots<T>(0, nv, n0, n1, wr, [&](int i) { return vr + i * vstride; }, part, nchunk, c, nrhs, r);
}

// y(:, r) = w(:, r) / |w(:, r)| (0 where the norm is 0) from the chunks' parts of
// |w|^2, whose sum goes to sq[r]
template <class T>
__global__ __launch_bounds__(KT) void k_normalise(const cpx<T> *w, long long n, long long chunk,
                                                  const cpx<double> *__restrict__ part, int nchunk, int nrhs,
                                                  cpx<double> *__restrict__ sq, cpx<T> *y)
{
    const int c = blockIdx.x, r = blockIdx.y;
    const long long n0 = (long long)c * chunk, n1 = n0 + chunk < n ? n0 + chunk : n;
    const cpx<double> s = sum_chunks(part + r, nchunk, nrhs);
    if (c == 0 && threadIdx.x == 0) sq[r] = s;
    const double nrm = sqrt(s.re > 0 ? s.re : 0.0), f = nrm > 0 ? 1.0 / nrm : 0.0;
    const cpx<T> *wr = w + (long long)r * n;
    cpx<T> *yr = y + (long long)r * n;
    for (long long k = n0 + threadIdx.x; k < n1; k += KT) {
        const cpx<T> v = wr[k];
        yr[k] = {(T)(f * v.re), (T)(f * v.im)};
    }
}

// y(n, r) = a[r] x(n, r) + b[r] z(n, r)  (z may be null: b ignored)
template <class T>
__global__ __launch_bounds__(KT) void k_axpby(const cpx<double> *__restrict__ a, const cpx<T> *__restrict__ x,
                                              long long ldx, const cpx<double> *__restrict__ b,
                                              const cpx<T> *__restrict__ z, long long ldz, cpx<T> *__restrict__ y,
                                              long long ldy, long long n, int nrhs)
{
    const long long g = (long long)blockIdx.x * KT + threadIdx.x;
    if (g >= n * nrhs) return;
    const int r = (int)(g / n);
    const long long k = g % n;
    const cpx<T> xv = x[(long long)r * ldx + k];
    double re = a[r].re * xv.re - a[r].im * xv.im, im = a[r].re * xv.im + a[r].im * xv.re;
    if (z) {
        const cpx<T> zv = z[(long long)r * ldz + k];
        re += b[r].re * zv.re - b[r].im * zv.im;
        im += b[r].re * zv.im + b[r].im * zv.re;
    }
    y[(long long)r * ldy + k] = {(T)re, (T)im};
}

// y(i, r) = alpha * sum_k val[k] x(col[k], r) over row i's entries of a CSR
// matrix (plus y(i, r) when accumulate); thread per (row, right-hand side),
// rows fastest so a wave writes consecutive elements of one column.
template <class T>
__global__ __launch_bounds__(KT) void k_csr_spmm(long long nrows, int nrhs, const long long *__restrict__ ptr,
                                                 const int *__restrict__ col, const cpx<T> *__restrict__ val,
                                                 const cpx<T> *__restrict__ x, long long ldx, cpx<T> *__restrict__ y,
                                                 long long ldy, double alpha, int accumulate)
{
    const long long g = (long long)blockIdx.x * KT + threadIdx.x;
    if (g >= nrows * nrhs) return;
    const int r = (int)(g / nrows);
    const long long i = g % nrows;
    const cpx<T> *xr = x + (long long)r * ldx;
    double re = 0, im = 0;
    for (long long k = ptr[i]; k < ptr[i + 1]; k++) {
        const cpx<T> a = val[k], b = xr[col[k]];
        re += (double)a.re * b.re - (double)a.im * b.im;
        im += (double)a.re * b.im + (double)a.im * b.re;
    }
    cpx<T> &o = y[(long long)r * ldy + i];
    if (accumulate) o = {(T)((double)o.re + alpha * re), (T)((double)o.im + alpha * im)};
    else o = {(T)(alpha * re), (T)(alpha * im)};
}

// b(:, r) = (complex float) a(:, r)  (rows n, leading dimensions lda, ldb)
__global__ __launch_bounds__(KT) void k_to_single(const cpx<double> *__restrict__ a, long long lda,
                                                  cpx<float> *__restrict__ b, long long ldb, long long n, int nrhs)
{
    const long long g = (long long)blockIdx.x * KT + threadIdx.x;
    if (g >= n * nrhs) return;
    const int r = (int)(g / n);
    const long long k = g % n;
    const cpx<double> v = a[(long long)r * lda + k];
    b[(long long)r * ldb + k] = {(float)v.re, (float)v.im};
}

// a(:, r) = b(:, r), or a(:, r) += b(:, r) with add  (complex double from complex float)
__global__ __launch_bounds__(KT) void k_from_single(cpx<double> *__restrict__ a, long long lda,
                                                    const cpx<float> *__restrict__ b, long long ldb, long long n,
                                                    int nrhs, int add)
{
    const long long g = (long long)blockIdx.x * KT + threadIdx.x;
    if (g >= n * nrhs) return;
    const int r = (int)(g / n);
    const long long k = g % n;
    const cpx<float> v = b[(long long)r * ldb + k];
    cpx<double> &o = a[(long long)r * lda + k];
    if (add) o = {o.re + (double)v.re, o.im + (double)v.im};
    else o = {(double)v.re, (double)v.im};
}

inline unsigned blocks(long long n) { return (unsigned)((n + KT - 1) / KT); }

}  // namespace

void launch_to_single(const cpx<double> *a, long long lda, cpx<float> *b, long long ldb, long long n, int nrhs,
                      hipStream_t s)
{
    if (n * nrhs > 0) hipLaunchKernelGGL(k_to_single, dim3(blocks(n * nrhs)), dim3(KT), 0, s, a, lda, b, ldb, n, nrhs);
}

void launch_from_single(cpx<double> *a, long long lda, const cpx<float> *b, long long ldb, long long n, int nrhs,
                        bool add, hipStream_t s)
{
    if (n * nrhs > 0)
        hipLaunchKernelGGL(k_from_single, dim3(blocks(n * nrhs)), dim3(KT), 0, s, a, lda, b, ldb, n, nrhs, add ? 1 : 0);
}

template <class T>
void launch_csr_spmm(long long nrows, int nrhs, const long long *ptr, const int *col, const cpx<T> *val,
                     const cpx<T> *x, long long ldx, cpx<T> *y, long long ldy, double alpha, bool accumulate,
                     hipStream_t s)
{
    if (nrows <= 0) return;
    hipLaunchKernelGGL(k_csr_spmm<T>, dim3(blocks(nrows * nrhs)), dim3(KT), 0, s, nrows, nrhs, ptr, col, val, x, ldx,
                       y, ldy, alpha, accumulate ? 1 : 0);
}

template <class T>
void krylov_dots(const cpx<T> *V, long long vstride, long long ldv, int nv, const cpx<T> *w, long long ldw, long long n,
                 int nrhs, cpx<double> *part, int nchunk, cpx<double> *out, hipStream_t s)
{
    const long long chunk = (n + nchunk - 1) / nchunk;
    hipLaunchKernelGGL(k_dots<T>, dim3(nchunk, nrhs, (nv + DOT_BATCH - 1) / DOT_BATCH), dim3(KT), 0, s, V, vstride, ldv,
                       nv, w, ldw, n, chunk, part, nchunk, nrhs);
    const int wpb = KT / 64;
    hipLaunchKernelGGL(k_sum_parts, dim3((nv * nrhs + wpb - 1) / wpb), dim3(KT), 0, s, part, nv, nchunk, nrhs, out);
}

template <class T>
void krylov_step(const cpx<T> *V, int nv, cpx<T> *w, cpx<T> *next, long long n, int nrhs, cpx<double> *part, int nchunk,
                 cpx<double> *sq, cpx<double> *h1, cpx<double> *h2, hipStream_t s)
{
    const long long chunk = (n + nchunk - 1) / nchunk, vstride = n * nrhs;
    const int wpb = KT / 64, nsum = (nv * nrhs + wpb - 1) / wpb;
    const dim3 grid(nchunk, nrhs);
    krylov_dots<T>(V, vstride, n, nv, w, n, n, nrhs, part, nchunk, h1, s);
    hipLaunchKernelGGL(k_orthogonalise<T>, grid, dim3(KT), 0, s, V, vstride, nv, h1, w, n, chunk, part, nchunk, nrhs, 0);
    hipLaunchKernelGGL(k_sum_parts, dim3(nsum), dim3(KT), 0, s, part, nv, nchunk, nrhs, h2);
    hipLaunchKernelGGL(k_orthogonalise<T>, grid, dim3(KT), 0, s, V, vstride, nv, h2, w, n, chunk, part, nchunk, nrhs, 1);
    hipLaunchKernelGGL(k_normalise<T>, grid, dim3(KT), 0, s, w, n, chunk, part, nchunk, nrhs, sq, next);
}

template <class T>
void krylov_normalise(const cpx<T> *w, cpx<T> *y, long long n, int nrhs, cpx<double> *part, int nchunk, cpx<double> *sq,
                      hipStream_t s)
{
    const long long chunk = (n + nchunk - 1) / nchunk;
    hipLaunchKernelGGL(k_dots<T>, dim3(nchunk, nrhs), dim3(KT), 0, s, w, 0, n, 1, w, n, n, chunk, part, nchunk, nrhs);
    hipLaunchKernelGGL(k_normalise<T>, dim3(nchunk, nrhs), dim3(KT), 0, s, w, n, chunk, part, nchunk, nrhs, sq, y);
}

template <class T>
void krylov_combine(const cpx<T> *V, long long vstride, long long ldv, int nv, const cpx<double> *h, double sign,
                    cpx<T> *w, long long ldw, long long n, int nrhs, hipStream_t s)
{
    hipLaunchKernelGGL(k_combine<T>, dim3(blocks(n * nrhs)), dim3(KT), 0, s, V, vstride, ldv, nv, h, sign, w, ldw, n,
                       nrhs);
}

template <class T>
void krylov_axpby(const cpx<double> *a, const cpx<T> *x, long long ldx, const cpx<double> *b, const cpx<T> *z,
                  long long ldz, cpx<T> *y, long long ldy, long long n, int nrhs, hipStream_t s)
{
    hipLaunchKernelGGL(k_axpby<T>, dim3(blocks(n * nrhs)), dim3(KT), 0, s, a, x, ldx, b, z, ldz, y, ldy, n, nrhs);
}

#define KRYLOV_INST(T)                                                                                              \
    template void krylov_dots<T>(const cpx<T> *, long long, long long, int, const cpx<T> *, long long, long long,  \
                                 int, cpx<double> *, int, cpx<double> *, hipStream_t);                             \
    template void krylov_step<T>(const cpx<T> *, int, cpx<T> *, cpx<T> *, long long, int, cpx<double> *, int,       \
                                 cpx<double> *, cpx<double> *, cpx<double> *, hipStream_t);                         \
    template void krylov_normalise<T>(const cpx<T> *, cpx<T> *, long long, int, cpx<double> *, int, cpx<double> *,  \
                                      hipStream_t);                                                                 \
    template void krylov_combine<T>(const cpx<T> *, long long, long long, int, const cpx<double> *, double,       \
                                    cpx<T> *, long long, long long, int, hipStream_t);                             \
    template void krylov_axpby<T>(const cpx<double> *, const cpx<T> *, long long, const cpx<double> *,           \
                                  const cpx<T> *, long long, cpx<T> *, long long, long long, int, hipStream_t);   \
    template void launch_csr_spmm<T>(long long, int, const long long *, const int *, const cpx<T> *,             \
                                     const cpx<T> *, long long, cpx<T> *, long long, double, bool, hipStream_t);
KRYLOV_INST(float)
KRYLOV_INST(double)

}  // namespace mlfma
