// Disaggregation between octree levels with a box's whole intermediate in LDS.
//
// The step is the one of levels.hip, term for term: for a child box c of P and
// each of its 2 nrhs vectors (component, right-hand side)
//   X(i, jp)   = conj(shift_c(i, jp)) V_P(i, jp)
//   mid(i, jc) = rowf(i) sum_jp D_phi(jc, jp) X(i, jp)
//   V_c(ic, jc) += sum_(i, turn) D_th(ic, i, turn) mid(i, jc + turn * half a circle)
// Workgroup = (child, slice of the vectors), NV vectors per pass.  Both sums
// are banded and their weights depend on the output alone, so that a wave
// takes 64 rows (columns) as its lanes and a group of G outputs: an input is
// read from LDS once for the G sums it enters, and its G weights are the same
// in all lanes (scalar loads, no vector register or LDS traffic).  On a coarse
// level the theta window of a chunk of child rows is most of the box, and the
// chunked kernels form its intermediate rows several times over; here each is
// formed once.  Bound by vector instructions (0.66 of the issue slots), the
// texture data unit (busy 0.64: windows in, old values and rows out) and the
// waits between the short phases (0.34 of a wave's time): sphere of radius 8 wavelengths (276 480 RWGs), 16 right-hand sides,
// complex64 (complex128), step by step from 58 x 116 parent samples to 34 x 68,
// 21 x 42 and 14 x 28: chunked 0.70, 0.42, 0.53 (1.48, 1.41, 1.28) ms, here
// 0.29, 0.42, 0.50 (0.57, 0.66, 0.78) ms; the step to 11 x 22 stays chunked:
// 0.69 against 0.91 (1.32, 1.41) ms.  On the matrix cores (16 outputs per
// group, the same sums) 0.31, 0.44, 0.55, 1.14 (0.63, 0.78, 0.93, 1.84) ms.
#include <algorithm>
#include <cmath>

#include "device.hpp"

namespace mlfma {

namespace {

constexpr int NXCD_B = 8;
constexpr int BOX_NS = 8;                     // window samples per thread at most
constexpr size_t BOX_LDS_MAX = 160 * 1024;
__device__ inline long long xcd_block_b(long long nblk)
{
    const long long per = (nblk + NXCD_B - 1) / NXCD_B;
    const long long hw = blockIdx.x;
    const long long lb = (hw % NXCD_B) * per + hw / NXCD_B;
    return lb < nblk ? lb : -1;
}
inline unsigned xcd_grid_b(long long nblk) { return (unsigned)(((nblk + NXCD_B - 1) / NXCD_B) * NXCD_B); }

// the scalar unit's view of read-only tables
template <class T>
using table = const __attribute__((address_space(4))) T *;
template <class T>
__device__ inline table<T> as_table(const T *p)
{
    return (table<T>)(p);
}

// sums of one group over its entries: input p[turn][(key / 2) * pitch], U
// entries' loads in flight together
template <class T, int G>
__device__ inline void group_sums(cpx<T> (&acc)[G], const cpx<T> *p0, const cpx<T> *p1, int pitch, table<int> key,
                                  table<T> w, int n0, int n1)
{
    constexpr int U = G * sizeof(T) <= 32 ? 4 : 2;
#pragma unroll
    for (int k = 0; k < G; k++) acc[k] = mk<T>(0, 0);
    for (int n = n0; n < n1; n += U) {
        cpx<T> x[U];
        T wt[U][G];
        int e[U];
#pragma unroll
        for (int u = 0; u < U; u++) e[u] = key[n + u];
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int k = 0; k < G; k++) wt[u][k] = w[(n + u) * G + k];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = ((e[u] & 1) ? p1 : p0)[(e[u] >> 1) * pitch];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int k = 0; k < G; k++) axpy_to(acc[k], wt[u][k], x[u]);
    }
}

template <class T, int G>
__device__ inline void dis_phi(const LevelStep<T> &a, const BoxPlan<T> &b, const cpx<T> *X, cpx<T> *mid,
                               const int *s_row, const T *s_rowf, int i0, int wave, int nwave, int lane)
{
    const int nrow = b.nv * b.cr, nrb = (nrow + 63) / 64;
    for (int task = wave; task < nrb * b.phi.ng; task += nwave) {
        const int g = task / nrb, row = (task - g * nrb) * 64 + lane, rr = min(row, nrow - 1);
        const cpx<T> *x = X + rr;
        cpx<T> acc[G];
        table<int> st = as_table(b.phi.start);
        group_sums<T, G>(acc, x, x, b.pitch_x, as_table(b.phi.key), as_table(b.phi.w), st[g], st[g + 1]);
        const int rec = s_row[rr], i = i0 + (rec & 0xffff), v = rec >> 16;
        if (row < nrow && i < a.nth_p) {
            const T f = s_rowf[i];
            cpx<T> *m = mid + i * b.pitch_m + v * a.nph_c + g * G;
#pragma unroll
            for (int k = 0; k < G; k++)
                if (g * G + k < a.nph_c) m[k] = f * acc[k];
        }
    }
}

template <class T, int G>
__device__ inline void dis_theta(const LevelStep<T> &a, const BoxPlan<T> &b, const cpx<T> *mid, const int *s_col,
                                 cpx<T> *out, int nv, int wave, int nwave, int lane)
{
    const int ncol = nv * a.nph_c, ncb = (ncol + 63) / 64;
    for (int task = wave; task < ncb * b.th.ng; task += nwave) {
        const int g = task / ncb, col = (task - g * ncb) * 64 + lane, cc = min(col, ncol - 1);
        const int rec = s_col[cc], v = rec >> 16, jc = rec & 0xffff;
        const int turn = cc + (2 * jc < a.nph_c ? a.nph_c / 2 : -(a.nph_c / 2));
        cpx<T> *o = out + v * a.ks_c + g * G * a.nph_c + jc;
        cpx<T> old[G], acc[G];
#pragma unroll
        for (int k = 0; k < G; k++) old[k] = o[min(k, a.nth_c - 1 - g * G) * a.nph_c];
        table<int> st = as_table(b.th.start);
        group_sums<T, G>(acc, mid + cc, mid + turn, b.pitch_m, as_table(b.th.key), as_table(b.th.w), st[g], st[g + 1]);
        if (col < ncol)
#pragma unroll
            for (int k = 0; k < G; k++)
                if (g * G + k < a.nth_c) o[k * a.nph_c] = old[k] + acc[k];
    }
}

// NS: samples of a chunk's window that a thread holds
template <class T, int NS>
__global__ __launch_bounds__(1024) void k_disaggregate_box(const LevelStep<T> a, const BoxPlan<T> b, int nrhs)
{
    extern __shared__ double box_lds_raw[];
    const long long c = xcd_block_b(a.nbox);
    if (c < 0) return;
    const int nvec = 2 * nrhs, vs0 = blockIdx.y * b.per, vs1 = min(nvec, vs0 + b.per);
    if (vs0 >= vs1) return;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nt >> 6;
    const int Kp = a.nth_p * a.nph_p, win = b.cr * a.nph_p, nslot = b.nv * win;
    cpx<T> *X = reinterpret_cast<cpx<T> *>(box_lds_raw);      // [nph_p][pitch_x]: column, (vector, chunk row)
    cpx<T> *mid = X + (size_t)a.nph_p * b.pitch_x;             // [nth_p][pitch_m]: row, (vector, child column)
    T *s_rowf = reinterpret_cast<T *>(mid + (size_t)a.nth_p * b.pitch_m);   // [nth_p]
    int *s_row = reinterpret_cast<int *>(s_rowf + a.nth_p);    // [nv * cr]: chunk row, vector
    int *s_col = s_row + b.nv * b.cr;                          // [nv * nph_c]: child column, vector
    for (int i = tid; i < a.nth_p; i += nt) s_rowf[i] = a.rowf[i];
    for (int i = tid; i < b.nv * b.cr; i += nt) s_row[i] = (i / b.cr) << 16 | i % b.cr;
    for (int i = tid; i < b.nv * a.nph_c; i += nt) s_col[i] = (i / a.nph_c) << 16 | i % a.nph_c;
    // window sample of slot s: its offset in the vectors, in the shift and in X
    int off[NS], xo[NS], lo[NS];
#pragma unroll
    for (int s = 0; s < NS; s++) {
        const int e = min(tid + s * nt, nslot - 1), v = e / win, x = e - v * win, i = x / a.nph_p, jp = x - i * a.nph_p;
        off[s] = v * a.ks_p + x;
        xo[s] = x;
        lo[s] = jp * b.pitch_x + v * b.cr + i;
    }
    const cpx<T> *pin = a.in + (long long)a.parent[c] * nvec * a.ks_p;
    const cpx<T> *sh = a.shift + (long long)a.oct[c] * Kp;
    cpx<T> *out = a.out + c * nvec * a.ks_c;
    for (int v0 = vs0; v0 < vs1; v0 += b.nv) {
        for (int ch = 0; ch < b.nch; ch++) {
            const int i0 = ch * b.cr;
            const int o0 = i0 * a.nph_p, last = Kp - 1 - o0, lastv = (vs1 - 1 - v0) * a.ks_p + last;
            const cpx<T> *p = pin + (long long)v0 * a.ks_p + o0;
            cpx<T> pf[NS], sf[NS];
            // clamped (valid) addresses, no predicates: samples past the box
            // or the slice feed rows and columns that are never stored
#pragma unroll
            for (int s = 0; s < NS; s++) pf[s] = p[min(off[s], lastv)];
#pragma unroll
            for (int s = 0; s < NS; s++) sf[s] = sh[o0 + min(xo[s], last)];
#pragma unroll
            for (int s = 0; s < NS; s++)
                if (tid + s * nt < nslot) X[lo[s]] = conjg(sf[s]) * pf[s];
            __syncthreads();
            if (b.gphi == 0) dis_phi<T, 4>(a, b, X, mid, s_row, s_rowf, i0, wave, nwave, lane);
            else if (b.gphi == 1) dis_phi<T, 6>(a, b, X, mid, s_row, s_rowf, i0, wave, nwave, lane);
            else dis_phi<T, 8>(a, b, X, mid, s_row, s_rowf, i0, wave, nwave, lane);
            __syncthreads();
        }
        cpx<T> *o = out + (long long)v0 * a.ks_c;
        const int nv = min(b.nv, vs1 - v0);
        if (b.gth == 0) dis_theta<T, 4>(a, b, mid, s_col, o, nv, wave, nwave, lane);
        else if (b.gth == 1) dis_theta<T, 6>(a, b, mid, s_col, o, nv, wave, nwave, lane);
        else dis_theta<T, 8>(a, b, mid, s_col, o, nv, wave, nwave, lane);
    }
}

template <class T>
size_t box_lds(const LevelStep<T> &a, const BoxPlan<T> &p)
{
    return ((size_t)a.nph_p * p.pitch_x + (size_t)a.nth_p * p.pitch_m) * sizeof(cpx<T>) + a.nth_p * sizeof(T) +
           (size_t)p.nv * (p.cr + a.nph_c) * sizeof(int);
}

template <class T>
auto box_kernel(const LevelStep<T> &a, const BoxPlan<T> &p)
{
    return p.nv * p.cr * a.nph_p <= 4 * p.nt ? k_disaggregate_box<T, 4> : k_disaggregate_box<T, BOX_NS>;
}

}  // namespace

// The plan of least estimated time per vector.  A pass takes the longest
// wave's tasks (serial: a wave's reads are short chains) shared by the
// workgroups on a CU, plus the issue cycles of all; the constants put the
// measured plans of four geometries, 1 to 64 right-hand sides, in their order
// (the plan taken is within 15 % of the best one in most, 24 % in the worst).
template <class T>
bool plan_disaggregate_box(const LevelStep<T> &a, const GroupTable<T> &phi, const GroupTable<T> &th, int nrhs,
                           BoxPlan<T> &best)
{
    if (!phi.ng[0] || !th.ng[0] || a.nph_p >= 1 << 15 || a.nbox <= 0) return false;
    const int nvec = 2 * nrhs;
    const double f = sizeof(T) == 4 ? 4 : 8;   // cycles of a complex-by-real product and sum
    double best_cost = 1e300;
    for (int nt : {256, 512, 1024})
        for (int nv = 1; nv <= std::min(nvec, 8); nv++)
            for (int nch = 1; nch <= 4; nch++) {
                BoxPlan<T> p{};
                p.nt = nt;
                p.nv = nv;
                p.cr = (a.nth_p + nch - 1) / nch;
                p.nch = (a.nth_p + p.cr - 1) / p.cr;
                if (p.nch != nch || (long long)nv * p.cr * a.nph_p > (long long)BOX_NS * nt) continue;
                p.pitch_x = nv * p.cr | 1;
                p.pitch_m = nv * a.nph_c | 1;
                const size_t lds = box_lds(a, p);
                if (lds > BOX_LDS_MAX) continue;
                const int nw = nt / 64, nrb = (nv * p.cr + 63) / 64, ncb = (nv * a.nph_c + 63) / 64;
                const int regw = sizeof(T) == 4 ? 24 : 16;   // waves per CU by registers
                const int occ = std::max(1, std::min<int>(regw / nw, BOX_LDS_MAX / lds));
                const double wgs = (double)a.nbox * ((nvec + nv - 1) / nv) / 256;   // workgroups per CU
                const double share = std::max(1.0, std::min<double>(occ, wgs));
                double bp = 1e300, bt = 1e300;
                auto phase = [&](const GroupTable<T> &t, int g, int blocks) {
                    const int G = STEP_GROUP[g], tasks = blocks * t.ng[g];
                    const double len = (double)t.len[g] / t.ng[g];
                    const double issue = len * (G * f + 24) + 24 * G + 100, wait = len * 60 + 600;
                    return (tasks + nw - 1) / nw * (issue + wait) / share + tasks * issue / 4;
                };
                for (int g = 0; g < 3; g++) {
                    const double cp = p.nch * phase(phi, g, nrb), ct = phase(th, g, ncb);
                    if (cp < bp) bp = cp, p.gphi = g;
                    if (ct < bt) bt = ct, p.gth = g;
                }
                const double slots = std::ceil((double)nv * p.cr * a.nph_p / nt);
                const double x = p.nch * ((1200 + slots * 60) / share + slots * nw * 15);
                const double cost = (bp + bt + x) * std::ceil((double)nvec / nv) * std::ceil(wgs / share) / wgs * share;
                if (cost < best_cost) {
                    best_cost = cost;
                    best = p;
                }
            }
    if (best_cost == 1e300) return false;
    best.phi = {phi.ng[best.gphi], phi.start[best.gphi], phi.key[best.gphi], phi.w[best.gphi]};
    best.th = {th.ng[best.gth], th.start[best.gth], th.key[best.gth], th.w[best.gth]};
    // more than the default dynamic LDS: allowed here, once, not at a launch
    // that may be captured
    if (box_lds(a, best) > 64 * 1024 &&
        hipFuncSetAttribute((const void *)box_kernel(a, best), hipFuncAttributeMaxDynamicSharedMemorySize,
                            BOX_LDS_MAX) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

template <class T>
bool launch_disaggregate_box(const LevelStep<T> &a, int nrhs, hipStream_t s)
{
    if (!a.box) return false;
    if (a.nbox <= 0 || nrhs <= 0) return true;
    BoxPlan<T> p = *a.box;
    const int nvec = 2 * nrhs;
    // slices of the vectors: about eight workgroups per CU
    const int pass = (nvec + p.nv - 1) / p.nv;
    const int slices = (int)std::min<long long>(pass, std::max<long long>(1, (2048 + a.nbox - 1) / a.nbox));
    p.per = (pass + slices - 1) / slices * p.nv;
    hipLaunchKernelGGL(box_kernel(a, p), dim3(xcd_grid_b(a.nbox), (nvec + p.per - 1) / p.per), dim3(p.nt),
                       box_lds(a, p), s, a, p, nrhs);
    return true;
}

#define BOX_INST(T)                                                                                                  \
    template bool plan_disaggregate_box<T>(const LevelStep<T> &, const GroupTable<T> &, const GroupTable<T> &, int,   \
                                           BoxPlan<T> &);                                                             \
    template bool launch_disaggregate_box<T>(const LevelStep<T> &, int, hipStream_t);
BOX_INST(float)
BOX_INST(double)
#undef BOX_INST

}  // namespace mlfma
