// Diagonal translation by sibling groups, register-blocked over targets.
//
// V_A(k) = sum_{(B, o) in IL(A)} T_o(k) U_B(k)  (Sec. II-E, MLFMA far field;
// diagonal in k).  Siblings share most of their interaction lists (the
// children of their parent's neighbours, less the boxes adjacent to each),
// so a group of up to TG siblings streams the union of its sources once:
// every lane loads a source's samples and applies them to every target of
// the group that has the source in its list, keeping all targets' sums in
// registers.  Nothing is staged in LDS and there are no barriers; a source's
// value is loaded once per group instead of once per (target, source) pair.
//
// Lanes: QW = 64 / RW consecutive samples x RW right-hand sides; each lane
// handles RB right-hand sides (rbase + j RW).  Fewer samples per wave (more
// lanes over the right-hand sides) load each operator value for fewer sums
// but keep fewer sums per lane (more waves resident): the autotuner picks.
// A workgroup of four waves takes four consecutive sample chunks of one
// group.  Workgroups are ordered sample chunk first, group second, and every
// XCD takes a contiguous range of each level: consecutive groups (Morton
// order) share sources through the XCD's L2, and the operator rows of one
// sample chunk stay resident there.
//
// Two variants share the group tables: k_translate_lds stages the operator
// rows of a sample chunk in LDS for a workgroup of eight groups (only source
// samples then travel through the vector memory path), and k_translate_mfma
// forms the sums of a 16-target group as one complex product per sample on
// the matrix cores.
#include "device.hpp"
#include "mfma_ops.hpp"

namespace mlfma {

namespace {

constexpr int WAVE = 64;     // lanes of a wavefront
constexpr int NXCD = 8;      // dies (XCDs); hardware block b runs on XCD b mod 8
constexpr int GWAVES = 4, LWAVES = 8;   // waves per workgroup: register kernel, LDS-operator kernel

typedef const __attribute__((address_space(4))) int cint_g;
__device__ inline int ldu(const int *p, int i) { return ((cint_g *)p)[i]; }

// Raw buffer loads: a resource descriptor for a uniform base address (no
// range check: every offset used lies inside the array) and a per-lane
// 32-bit byte offset, so that a loop's loads need no 64-bit vector address
// arithmetic.  Descriptor word 3 = 0x00020000 (the gfx9 family's 32-bit
// data format, no swizzle).
__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00020000);
}
template <class T>
__device__ inline cpx<T> bload(__amdgpu_buffer_rsrc_t r, unsigned off);
template <>
__device__ inline cpx<float> bload<float>(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return __builtin_bit_cast(cpx<float>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <>
__device__ inline cpx<double> bload<double>(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return __builtin_bit_cast(cpx<double>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

template <class T, int TG, int RW, int RB>
__global__ __launch_bounds__(GWAVES * WAVE) void k_translate_groups(const GroupArgs<T> a, int nrhs)
{
    constexpr int QW = WAVE / RW;
    const int xcd = blockIdx.x % NXCD, pos = blockIdx.x / NXCD;
    if (pos >= a.nblocks) return;
    int l = 0;
    while (l + 1 < a.nlev && pos >= a.lv[l + 1].first) l++;
    const GroupLevel<T> &L = a.lv[l];
    const int nblk = L.ngroup * L.nqc, per = (nblk + NXCD - 1) / NXCD;
    const int lb = xcd * per + (pos - L.first);
    if (lb >= nblk) return;
    const int g = lb % L.ngroup, qc = lb / L.ngroup;
    const int K = L.K;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int qi = lane % QW, ri = lane / QW;
    const int q = (qc * GWAVES + wave) * QW + qi;
    const bool qok = q < K;
    const int qr = qok ? q : K - 1;   // lanes past the last sample read a valid element, store nothing
    const int rbase = blockIdx.y * RW * RB + ri;
    const int ks = L.ks;
    const long long S = 2LL * nrhs * ks;   // one box's patterns
    const long long half = (long long)nrhs * ks;   // second component
    // per-lane byte offsets within a box's patterns and within an operator
    // row: every load takes a uniform 64-bit base (scalar registers, from
    // the record's source and offset ids) and one of these 32-bit offsets
    unsigned rob[RB];
#pragma unroll
    for (int j = 0; j < RB; j++)
        rob[j] = (unsigned)(((long long)min(rbase + j * RW, nrhs - 1) * ks + qr) * (long long)sizeof(cpx<T>));
    const unsigned qb = (unsigned)(qr * sizeof(cpx<T>));
    const int t0 = ldu(L.first_tgt, g), nt = ldu(L.count, g);
    const int r0 = ldu(L.rec_start, g), r1 = ldu(L.rec_start, g + 1);
    cpx<T> acc[TG][2][RB];
#pragma unroll
    for (int t = 0; t < TG; t++)
#pragma unroll
        for (int j = 0; j < RB; j++) acc[t][0][j] = acc[t][1][j] = mk<T>(0, 0);
    // a record: its source's samples, the group's operator values and offset
    // ids; the next record is loaded while the current one is summed (two
    // register sets used in turn)
    struct Rec {
        cpx<T> u0[RB], u1[RB], op[TG];
        int off[TG];
    };
    const int *srcp = L.src, *offp = L.off;
    const cpx<T> *Ub = L.U, *Tb = L.trans;
    auto load = [&](int r, Rec &o) {
        const cpx<T> *us = Ub + (long long)ldu(srcp, r) * S;
        const auto ru0 = rsrc(us), ru1 = rsrc(us + half);
#pragma unroll
        for (int j = 0; j < RB; j++) {
            o.u0[j] = bload<T>(ru0, rob[j]);
            o.u1[j] = bload<T>(ru1, rob[j]);
        }
#pragma unroll
        for (int t = 0; t < TG; t++) {
            o.off[t] = ldu(offp, r * TG + t);
            // a valid row also where the source is absent
            o.op[t] = bload<T>(rsrc(Tb + (long long)max(o.off[t], 0) * L.tks), qb);
        }
    };
    auto sum = [&](const Rec &c) {
#pragma unroll
        for (int t = 0; t < TG; t++) {
            if (c.off[t] < 0) continue;   // uniform: the source is not in target t's list
#pragma unroll
            for (int j = 0; j < RB; j++) {
                fma_to(acc[t][0][j], c.op[t], c.u0[j]);
                fma_to(acc[t][1][j], c.op[t], c.u1[j]);
            }
        }
    };
    // the loads of the next record are issued on every path (past the last
    // record they repeat it), so that the wait before a sum counts the other
    // set's loads as in flight instead of merging with a path without them
    Rec ra, rb2;
    if (r0 < r1) load(r0, ra);
    for (int r = r0; r < r1; r += 2) {
        load(min(r + 1, r1 - 1), rb2);
        sum(ra);
        if (r + 1 >= r1) break;
        load(min(r + 2, r1 - 1), ra);
        sum(rb2);
    }
    if (!qok) return;
#pragma unroll
    for (int t = 0; t < TG; t++) {
        if (t >= nt) break;
        cpx<T> *vt = L.V + (long long)(t0 + t) * S;
#pragma unroll
        for (int j = 0; j < RB; j++) {
            const int rr = rbase + j * RW;
            if (rr >= nrhs) continue;
            vt[(long long)rr * ks + q] = acc[t][0][j];
            vt[half + (long long)rr * ks + q] = acc[t][1][j];
        }
    }
}


// SV consecutive samples of one lane (SV = 2 in single precision: one 16-byte
// access; rows start at even samples, as K is even)
template <class T, int SV>
struct alignas(SV * sizeof(cpx<T>)) Smp {
    cpx<T> s[SV];
};
template <class T, int SV>
__device__ inline Smp<T, SV> sload(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    if constexpr (SV == 2) return __builtin_bit_cast(Smp<T, SV>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    else return Smp<T, SV>{{bload<T>(r, off)}};
}

// The sibling-group kernel with the operator values in LDS.  A workgroup
// takes eight consecutive groups (one per wave) at one chunk of QW samples and
// first stages the operator rows of all 343 offsets for that chunk in LDS
// (343 QW complex values, 44 KB); the record loop then loads only source
// samples through the vector memory path, in runs of 128 bytes that are one
// line each (row_stride), and 16 bytes per lane (SV samples).  DEPTH records
// are in flight per wave in a ring of register sets, and nothing else in the
// loop waits on memory: the offset ids of 64 / TG records sit in one vector
// register (a lane each), loaded a batch ahead, and the source ids of 64
// records in another; both are handed out by readlane.  A record's operator
// values are read from LDS for all targets at once (absent ones read row 0)
// and the sums of absent targets are skipped by a scalar bit test.  Bound by
// the vector memory path into the CUs (texture data unit busy 0.88 of the time,
// addresser 0.54) and the vector units (0.69 of their issue slots); 16 right-hand
// sides in complex64 as below.  Sphere of radius 8 wavelengths (276 480 RWGs), 16 right-hand sides, all
// levels: complex64 3.25 ms (best earlier shape, rows of K samples, 12 to 19 GB
// fetched past L2), 2.69 with padded rows (7.5 GB), 2.47 with 16 bytes per
// lane, 2.3 with eight waves per staged table and two records in flight (10 GB)
// (one: 2.9, four: 2.4; four waves: 2.7, sixteen: 2.3; 16-target groups 3.5);
// complex128 5.5 -> 4.4.
template <class T, int TG, int RW, int RB, int SV>
__global__ __launch_bounds__(LWAVES * WAVE) void k_translate_lds(const GroupArgs<T> a, int nrhs)
{
    constexpr int QL = WAVE / RW, QW = QL * SV;   // lanes over the samples, samples of a wave
    typedef Smp<T, SV> smp;
    constexpr int BATCH = WAVE / TG;   // records per register of offset ids
    constexpr int DEPTH = 2;           // records in flight
    static_assert(BATCH % DEPTH == 0, "ring positions are compile-time");
    __shared__ cpx<T> tl[343 * QW];
    const int xcd = blockIdx.x % NXCD, pos = blockIdx.x / NXCD;
    if (pos >= a.nblocks) return;
    int l = 0;
    while (l + 1 < a.nlev && pos >= a.lv[l + 1].first) l++;
    const GroupLevel<T> &L = a.lv[l];
    const int ngb = (L.ngroup + LWAVES - 1) / LWAVES;
    const int nblk = ngb * L.nqc, per = (nblk + NXCD - 1) / NXCD;
    const int lb = xcd * per + (pos - L.first);
    if (lb >= nblk) return;
    const int gb = lb % ngb, qc = lb / ngb;
    const int K = L.K, q0 = qc * QW;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int g = gb * LWAVES + wave;
    const int gc = min(g, L.ngroup - 1);   // waves past the last group load its records and store nothing
    const int qi = lane % QL * SV, ri = lane / QL;
    const int q = q0 + qi;
    const int qr = min(q, K - SV);   // lanes past the last sample read valid elements, store nothing
    const int rbase = blockIdx.y * RW * RB + ri;
    const int ks = L.ks;
    const long long S = 2LL * nrhs * ks;   // one box's patterns
    const long long half = (long long)nrhs * ks;   // second component
    unsigned rob[RB];
#pragma unroll
    for (int j = 0; j < RB; j++)
        rob[j] = (unsigned)(((long long)min(rbase + j * RW, nrhs - 1) * ks + qr) * (long long)sizeof(cpx<T>));
    const int r0 = ldu(L.rec_start, gc), r1 = ldu(L.rec_start, gc + 1);
    smp acc[TG][2][RB];
#pragma unroll
    for (int t = 0; t < TG; t++)
#pragma unroll
        for (int j = 0; j < RB; j++) acc[t][0][j] = acc[t][1][j] = smp{};
    // ids: lane l holds source r + l, and offset id l % TG of record r + l / TG
    const auto rsrcs = rsrc(L.src + r0);
    const auto roffs = rsrc(L.off + (long long)r0 * TG);
    const int nrec = r1 - r0;
    auto load_src = [&](int r) { return __builtin_amdgcn_raw_buffer_load_b32(rsrcs, 4u * min(r + lane, max(nrec - 1, 0)), 0, 0); };
    auto load_off = [&](int r) {
        const int e = r * TG + lane, last = max(nrec * TG - 1, 0);
        const int o = __builtin_amdgcn_raw_buffer_load_b32(roffs, 4u * min(e, last), 0, 0);
        return e <= last ? o : -1;
    };
    struct Rec {
        smp u0[RB], u1[RB];
    };
    Rec ring[DEPTH];
    auto load = [&](int sb, Rec &o) {
        const cpx<T> *us = L.U + (long long)sb * S;
        const auto ru0 = rsrc(us), ru1 = rsrc(us + half);
#pragma unroll
        for (int j = 0; j < RB; j++) {
            o.u0[j] = sload<T, SV>(ru0, rob[j]);
            o.u1[j] = sload<T, SV>(ru1, rob[j]);
        }
    };
    // sources 0 .. 63 and, from the middle of a window on, 64 .. 127 ahead
    int srcv = 0, offv = -1;
    if (nrec > 0) {
        srcv = load_src(0);
        offv = load_off(0);
#pragma unroll
        for (int d = 0; d < DEPTH; d++) load(__builtin_amdgcn_readlane(srcv, min(d, nrec - 1)), ring[d]);
    }
    // stage the chunk's operator rows (samples past K as zeros)
    for (int i = threadIdx.x; i < 343 * QW; i += LWAVES * WAVE) {
        const int o = i / QW, qq = q0 + i % QW;
        tl[i] = qq < K ? L.trans[(long long)o * L.tks + qq] : mk<T>(0, 0);
    }
    __syncthreads();
    const char *tq = reinterpret_cast<const char *>(tl + qi);
    // windows of 64 records; within one, batches of BATCH records whose ring
    // positions are compile-time
    for (int w0 = 0; w0 < nrec; w0 += WAVE) {
        const int srcn = load_src(w0 + WAVE);   // the next window's sources (past the end: the last one)
        const int wend = min(nrec - w0, WAVE);
#pragma unroll 1
        for (int b0 = 0; b0 < wend; b0 += BATCH) {
            const int offn = load_off(w0 + b0 + BATCH);
            const unsigned long long present = __ballot(offv >= 0);
            const int offb = max(offv, 0) * (int)(QW * sizeof(cpx<T>));
#pragma unroll
            for (int k = 0; k < BATCH; k++) {
                Rec &c = ring[k % DEPTH];
                smp op[TG];
#pragma unroll
                for (int t = 0; t < TG; t++)
                    op[t] = *reinterpret_cast<const smp *>(tq + __builtin_amdgcn_readlane(offb, k * TG + t));
#pragma unroll
                for (int t = 0; t < TG; t++)
                    if (present >> (k * TG + t) & 1) {   // uniform: the source is in target t's list
#pragma unroll
                        for (int j = 0; j < RB; j++) {
#pragma unroll
                            for (int v = 0; v < SV; v++) {
                                fma_to(acc[t][0][j].s[v], op[t].s[v], c.u0[j].s[v]);
                                fma_to(acc[t][1][j].s[v], op[t].s[v], c.u1[j].s[v]);
                            }
                        }
                    }
                // the record DEPTH ahead takes this one's registers
                const int n = b0 + k + DEPTH;
                load(n < WAVE ? __builtin_amdgcn_readlane(srcv, n & (WAVE - 1))
                              : __builtin_amdgcn_readlane(srcn, n & (WAVE - 1)),
                     c);
            }
            offv = offn;
        }
        srcv = srcn;
    }
    if (g >= L.ngroup || q >= K) return;
    const int t0 = ldu(L.first_tgt, g), nt = ldu(L.count, g);
#pragma unroll
    for (int t = 0; t < TG; t++) {
        if (t < nt) {
            cpx<T> *vt = L.V + (long long)(t0 + t) * S;
#pragma unroll
            for (int j = 0; j < RB; j++) {
                const int rr = rbase + j * RW;
                if (rr < nrhs) {
                    *reinterpret_cast<smp *>(vt + (long long)rr * ks + q) = acc[t][0][j];
                    *reinterpret_cast<smp *>(vt + half + (long long)rr * ks + q) = acc[t][1][j];
                }
            }
        }
    }
}

// Translation on the matrix cores, for groups of up to 16 targets (whole
// sibling sets merged).  For one sample q a group's sums are a complex
// product
//   D[col][t] = sum_s U_s[col](q) T_{o(t, s)}(q),
// col = (component, right-hand side) and s running over the union of the
// targets' sources, four sources per MFMA step (T = 0 where s is not in
// t's list).  A wave takes QT consecutive samples (one accumulator pair per
// sample) and CT tiles of 16 columns; lane l feeds column and target l % 16
// and source slot l / 16 of a step, and loads its QT samples of one U row
// and one operator row as a run.  The next step's operands are loaded while
// the current step's MFMAs run.  Workgroups are ordered as in the
// sibling-group kernel (group innermost, every XCD a contiguous range).
template <class T, int QT, int CT>
__global__ __launch_bounds__(GWAVES * WAVE) void k_translate_mfma(const GroupArgs<T> a, int nrhs)
{
    typedef typename Mf<T>::v4 v4;
    const int xcd = blockIdx.x % NXCD, pos = blockIdx.x / NXCD;
    if (pos >= a.nblocks) return;
    int l = 0;
    while (l + 1 < a.nlev && pos >= a.lv[l + 1].first) l++;
    const GroupLevel<T> &L = a.lv[l];
    const int ncol = 2 * nrhs, nct = (ncol + 16 * CT - 1) / (16 * CT);
    const int nblk = L.ngroup * nct * L.nqc, per = (nblk + NXCD - 1) / NXCD;
    const int lb = xcd * per + (pos - L.first);
    if (lb >= nblk) return;
    const int g = lb % L.ngroup, rest = lb / L.ngroup;
    const int ct = rest % nct, qc = rest / nct;
    const int K = L.K;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int q0 = (qc * GWAVES + wave) * QT;
    if (q0 >= K) return;
    const bool full = q0 + QT <= K;
    const int qlast = K - 1 - q0;   // last valid sample of the run
    const int lo = lane & 15, kk = lane >> 4;
    const int ks = L.ks;
    const long long S = (long long)ncol * ks;   // one box's patterns
    long long co[CT];   // this lane's column rows (clamped to a valid one)
#pragma unroll
    for (int c = 0; c < CT; c++) co[c] = (long long)min((ct * CT + c) * 16 + lo, ncol - 1) * ks + q0;
    const int t0 = ldu(L.first_tgt, g), nt = ldu(L.count, g);
    const int r0 = ldu(L.rec_start, g), r1 = ldu(L.rec_start, g + 1);
    v4 dre[CT][QT], dim[CT][QT];
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int u = 0; u < QT; u++) dre[c][u] = dim[c][u] = v4{0, 0, 0, 0};
    cpx<T> un[CT][QT], tn[QT];
    const int *srcp = L.src, *offp = L.off;
    const cpx<T> *Ub = L.U, *Tb = L.trans + q0;
    auto load = [&](int r) {
        const int rec = r + kk;
        const bool ok = rec < r1;
        const int sb = srcp[ok ? rec : r0];
        const int o = ok ? offp[(long long)rec * 16 + lo] : -1;
        const cpx<T> *us = Ub + (long long)sb * S;
        const cpx<T> *tp = Tb + (long long)max(o, 0) * L.tks;
        if (full) {
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int u = 0; u < QT; u++) un[c][u] = us[co[c] + u];
#pragma unroll
            for (int u = 0; u < QT; u++) tn[u] = tp[u];
        } else {
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int u = 0; u < QT; u++) un[c][u] = us[co[c] + min(u, qlast)];
#pragma unroll
            for (int u = 0; u < QT; u++) tn[u] = tp[min(u, qlast)];
        }
        if (o < 0)
#pragma unroll
            for (int u = 0; u < QT; u++) tn[u] = mk<T>(0, 0);
    };
    if (r0 < r1) load(r0);
    for (int r = r0; r < r1; r += 4) {
        cpx<T> uc[CT][QT], tc[QT];
#pragma unroll
        for (int u = 0; u < QT; u++) {
            tc[u] = tn[u];
#pragma unroll
            for (int c = 0; c < CT; c++) uc[c][u] = un[c][u];
        }
        if (r + 4 < r1) load(r + 4);
#pragma unroll
        for (int u = 0; u < QT; u++)
#pragma unroll
            for (int c = 0; c < CT; c++) dre[c][u] = Mf<T>::mma(uc[c][u].re, tc[u].re, dre[c][u]);
#pragma unroll
        for (int u = 0; u < QT; u++)
#pragma unroll
            for (int c = 0; c < CT; c++) dim[c][u] = Mf<T>::mma(uc[c][u].re, tc[u].im, dim[c][u]);
#pragma unroll
        for (int u = 0; u < QT; u++)
#pragma unroll
            for (int c = 0; c < CT; c++) dre[c][u] = Mf<T>::mma(-uc[c][u].im, tc[u].im, dre[c][u]);
#pragma unroll
        for (int u = 0; u < QT; u++)
#pragma unroll
            for (int c = 0; c < CT; c++) dim[c][u] = Mf<T>::mma(uc[c][u].im, tc[u].re, dim[c][u]);
    }
    if (lo >= nt) return;
    cpx<T> *vt = L.V + (long long)(t0 + lo) * S + q0;
#pragma unroll
    for (int c = 0; c < CT; c++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int col = (ct * CT + c) * 16 + Mf<T>::row(kk, v);
            if (col >= ncol) continue;
#pragma unroll
            for (int u = 0; u < QT; u++)
                if (full || u <= qlast) vt[(long long)col * ks + u] = mk<T>(dre[c][u][v], dim[c][u][v]);
        }
}

}  // namespace


// The LDS-operator kernel: groups of 8 targets, (lanes over the RHS, RHS per
// lane) in {(8, 1), (8, 2)} and, in single precision, {(4, 1), (4, 2), (4, 4)};
// 16 samples per workgroup in single precision, 8 in double (128-byte runs).
inline bool lds_shape_ok(bool single, int tg, int rw, int rb)
{
    return tg == 8 && ((rw == 8 && (rb == 1 || rb == 2)) || (single && rw == 4 && (rb == 1 || rb == 2 || rb == 4)));
}
template <class T>
bool launch_translate_lds(const GroupArgs<T> &args, int nrhs, hipStream_t s)
{
    constexpr bool single = sizeof(T) == 4;
    int rw = args.rw, rb = args.rb;
    if (!lds_shape_ok(single, args.tg, rw, rb)) return false;
    if (args.nlev <= 0 || nrhs <= 0) return true;
    // a shape tuned for more right-hand sides than this call has gives way
    // to the narrowest that leaves under half of the lanes idle (with fewer
    // right-hand sides than that needs, trans_shape takes another kernel)
    if (rw * rb > nrhs) {
        if (nrhs < (single ? 2 : 5)) return false;
        rw = nrhs >= 5 ? 8 : 4;
        rb = 1;
    }
    for (int l = 0; l < args.nlev; l++)   // 32-bit byte offsets within one box's patterns
        if (2.0 * nrhs * args.lv[l].ks * sizeof(cpx<T>) >= 4294967296.0) return false;
    constexpr int QW = single ? 16 : 8;
    GroupArgs<T> a = args;
    a.nblocks = 0;
    for (int l = 0; l < a.nlev; l++) {
        const int ngb = (a.lv[l].ngroup + LWAVES - 1) / LWAVES;
        a.lv[l].nqc = (a.lv[l].K + QW - 1) / QW;
        a.lv[l].first = a.nblocks;
        a.nblocks += (ngb * a.lv[l].nqc + NXCD - 1) / NXCD;
    }
    if (a.nblocks <= 0) return true;
    const dim3 grid((unsigned)a.nblocks * NXCD, (nrhs + rw * rb - 1) / (rw * rb)), block(LWAVES * WAVE);
#define LDS_LAUNCH(RW_, RB_, SV_) hipLaunchKernelGGL((k_translate_lds<T, 8, RW_, RB_, SV_>), grid, block, 0, s, a, nrhs)
    if constexpr (single) {
        if (rw == 8 && rb == 2) LDS_LAUNCH(8, 2, 2);
        else if (rw == 8) LDS_LAUNCH(8, 1, 2);
        else if (rb == 4) LDS_LAUNCH(4, 4, 1);
        else if (rb == 2) LDS_LAUNCH(4, 2, 1);
        else LDS_LAUNCH(4, 1, 1);
    } else {
        if (rb == 2) LDS_LAUNCH(8, 2, 1);
        else LDS_LAUNCH(8, 1, 1);
    }
#undef LDS_LAUNCH
    return true;
}

// the matrix-core kernel: args.rb = samples per wave (QT), args.rw = tiles of
// 16 columns per wave (CT)
template <class T>
bool launch_translate_mfma(const GroupArgs<T> &args, int nrhs, hipStream_t s)
{
    const int qt = args.rb, ct = args.rw;
    const bool ok = sizeof(T) == 4 ? ((qt == 4 || qt == 8) && (ct == 1 || ct == 2))
                                   : ((qt == 4 && (ct == 1 || ct == 2)) || (qt == 2 && ct == 2));
    if (!ok) return false;
    if (args.nlev <= 0 || nrhs <= 0) return true;
    const int nct = (2 * nrhs + 16 * ct - 1) / (16 * ct);
    GroupArgs<T> a = args;
    a.nblocks = 0;
    for (int l = 0; l < a.nlev; l++) {
        a.lv[l].nqc = (a.lv[l].K + GWAVES * qt - 1) / (GWAVES * qt);
        a.lv[l].first = a.nblocks;
        a.nblocks += (a.lv[l].ngroup * nct * a.lv[l].nqc + NXCD - 1) / NXCD;
    }
    if (a.nblocks <= 0) return true;
    const dim3 grid((unsigned)a.nblocks * NXCD), block(GWAVES * WAVE);
#define MFMA_LAUNCH(QT_, CT_) hipLaunchKernelGGL((k_translate_mfma<T, QT_, CT_>), grid, block, 0, s, a, nrhs)
    if constexpr (sizeof(T) == 4) {
        if (qt == 8 && ct == 2) MFMA_LAUNCH(8, 2);
        else if (qt == 8) MFMA_LAUNCH(8, 1);
        else if (ct == 2) MFMA_LAUNCH(4, 2);
        else MFMA_LAUNCH(4, 1);
    } else {
        if (qt == 2) MFMA_LAUNCH(2, 2);
        else if (ct == 2) MFMA_LAUNCH(4, 2);
        else MFMA_LAUNCH(4, 1);
    }
#undef MFMA_LAUNCH
    return true;
}

template <class T>
bool launch_translate_groups(const GroupArgs<T> &args, int nrhs, hipStream_t s)
{
    const int tg = args.tg;
    if (args.lds) return launch_translate_lds<T>(args, nrhs, s);
    if (tg == 16) return launch_translate_mfma<T>(args, nrhs, s);
    int rb = args.rb, rw = args.rw > 0 ? args.rw : trans_rw(nrhs);
    if (tg != 4 && tg != 8) return false;
    // (lanes over the RHS, RHS per lane) with a kernel
    auto valid = [&](int w, int b) {
        return (b == 1 && (w == 1 || w == 2 || w == 4 || w == 8 || w == 16)) || (w == 4 && (b == 2 || b == 4)) ||
               (w == 8 && b == 2) || (w == 2 && b == 8 && tg == 4 && sizeof(T) == 4);
    };
    if (!valid(rw, rb)) return false;
    // a shape tuned for more right-hand sides than this call has: fewer per
    // lane, else the default lane split (no lanes idle for lack of them)
    if (rw * rb > nrhs && nrhs > 0) {
        while (rb > 1 && (rw * rb > nrhs || !valid(rw, rb))) rb /= 2;
        if (rw * rb > nrhs) {
            rw = trans_rw(nrhs);
            rb = 1;
        }
    }
    if (args.nlev <= 0 || nrhs <= 0) return true;
    for (int l = 0; l < args.nlev; l++)   // 32-bit byte offsets within one box's patterns
        if (2.0 * nrhs * args.lv[l].ks * sizeof(cpx<T>) >= 4294967296.0) return false;
    const int qw = WAVE / rw;
    GroupArgs<T> a = args;
    a.rb = rb;
    a.rw = rw;
    a.nblocks = 0;
    for (int l = 0; l < a.nlev; l++) {
        a.lv[l].nqc = (a.lv[l].K + GWAVES * qw - 1) / (GWAVES * qw);
        a.lv[l].first = a.nblocks;
        a.nblocks += (a.lv[l].ngroup * a.lv[l].nqc + NXCD - 1) / NXCD;
    }
    if (a.nblocks <= 0) return true;
    const dim3 grid((unsigned)a.nblocks * NXCD, (nrhs + rw * rb - 1) / (rw * rb)), block(GWAVES * WAVE);
#define GROUP_LAUNCH(TG_, RW_, RB_) hipLaunchKernelGGL((k_translate_groups<T, TG_, RW_, RB_>), grid, block, 0, s, a, nrhs)
#define GROUP_SHAPES(TG_)                          \
    if (rw == 4 && rb == 4) GROUP_LAUNCH(TG_, 4, 4);       \
    else if (rw == 4 && rb == 2) GROUP_LAUNCH(TG_, 4, 2);  \
    else if (rw == 8 && rb == 2) GROUP_LAUNCH(TG_, 8, 2);  \
    else if (rw == 16) GROUP_LAUNCH(TG_, 16, 1);           \
    else if (rw == 8) GROUP_LAUNCH(TG_, 8, 1);             \
    else if (rw == 4) GROUP_LAUNCH(TG_, 4, 1);             \
    else if (rw == 2) GROUP_LAUNCH(TG_, 2, 1);             \
    else GROUP_LAUNCH(TG_, 1, 1);
    if (tg == 4 && rw == 2 && rb == 8) {
        if constexpr (sizeof(T) == 4) GROUP_LAUNCH(4, 2, 8);   // single precision only (register budget)
    } else if (tg == 4) {
        GROUP_SHAPES(4)
    } else {
        GROUP_SHAPES(8)
    }
#undef GROUP_SHAPES
#undef GROUP_LAUNCH
    return true;
}

template bool launch_translate_groups<float>(const GroupArgs<float> &, int, hipStream_t);
template bool launch_translate_groups<double>(const GroupArgs<double> &, int, hipStream_t);

}  // namespace mlfma
