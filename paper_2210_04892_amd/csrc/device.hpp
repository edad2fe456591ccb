// Device-side types and kernel launchers shared by the HIP sources.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

namespace mlfma {

template <class T>
struct alignas(2 * sizeof(T)) cpx {
    T re, im;
};

template <class T>
__host__ __device__ inline cpx<T> mk(T r, T i) { return cpx<T>{r, i}; }
template <class T>
__host__ __device__ inline cpx<T> operator+(cpx<T> a, cpx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <class T>
__host__ __device__ inline cpx<T> operator-(cpx<T> a, cpx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <class T>
__host__ __device__ inline cpx<T> operator*(cpx<T> a, cpx<T> b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <class T>
__host__ __device__ inline cpx<T> operator*(T s, cpx<T> a) { return {s * a.re, s * a.im}; }
template <class T>
__host__ __device__ inline cpx<T> conjg(cpx<T> a) { return {a.re, -a.im}; }
// fused multiply-add a b + c, rounded once
template <class T>
__host__ __device__ inline T fmad(T a, T b, T c);
template <>
__host__ __device__ inline float fmad<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <>
__host__ __device__ inline double fmad<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }

// p[0], p[1] with one 16-byte load in single precision (p must be 16-byte
// aligned there: an even index into a buffer from the allocator)
__device__ inline void load_pair(const cpx<float> *p, cpx<float> &a, cpx<float> &b)
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    a = {v.x, v.y};
    b = {v.z, v.w};
}
__device__ inline void load_pair(const cpx<double> *p, cpx<double> &a, cpx<double> &b)
{
    a = p[0];
    b = p[1];
}
// the same for data read once (non-temporal: streamed past the caches)
typedef float nt_f4 __attribute__((ext_vector_type(4)));
__device__ inline void load_pair_once(const cpx<float> *p, cpx<float> &a, cpx<float> &b)
{
    const nt_f4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f4 *>(p));
    a = {v.x, v.y};
    b = {v.z, v.w};
}
// (double pairs: plain loads measured faster)
__device__ inline void load_pair_once(const cpx<double> *p, cpx<double> &a, cpx<double> &b) { load_pair(p, a, b); }

// acc += a b (four fused multiply-adds)
template <class T>
__host__ __device__ inline void fma_to(cpx<T> &acc, cpx<T> a, cpx<T> b)
{
    acc.re = fmad(a.re, b.re, acc.re);
    acc.re = fmad(-a.im, b.im, acc.re);
    acc.im = fmad(a.re, b.im, acc.im);
    acc.im = fmad(a.im, b.re, acc.im);
}
// acc -= a b
template <class T>
__host__ __device__ inline void fms_to(cpx<T> &acc, cpx<T> a, cpx<T> b)
{
    acc.re = fmad(-a.re, b.re, acc.re);
    acc.re = fmad(a.im, b.im, acc.re);
    acc.im = fmad(-a.re, b.im, acc.im);
    acc.im = fmad(-a.im, b.re, acc.im);
}
// acc += s x for real s
template <class T>
__host__ __device__ inline void axpy_to(cpx<T> &acc, T s, cpx<T> x)
{
    acc.re = fmad(s, x.re, acc.re);
    acc.im = fmad(s, x.im, acc.im);
}

// Launchers of the hot path (matvec.hip).  X, Y internal vectors
// [rwg][half][rhs]; U, V patterns [box][component][rhs][sample], rows of K
// samples with stride ks >= K (the workspace's row_stride).
template <class T>
void launch_perm_in(const cpx<T> *x, long long ldx, cpx<T> *X, const int *perm, const int *iperm, int N, int nrhs,
                    hipStream_t s);
template <class T>
void launch_perm_out(const cpx<T> *Y, cpx<T> *y, long long ldy, const int *iperm, int N, int nrhs, hipStream_t s);
// Near field of 1 to NEAR_TILE_MAX right-hand sides: wave per (leaf box, tile of
// 8 RWGs) work item, columns of the box from cols[col_off[b] ..].  More go to
// the matrix cores, which at two multiply mostly empty columns.  Matrix cores
// (sums in double) against waves, us: sphere of 38 880 RWGs, complex64
// (complex128), two 88, 75 (111, 102), three 90, 104 (111, 142); of 122 880 two
// 232, 208 (303, 291), three 238, 295 (304, 434); ellipsoid of 48 000 with leaf
// boxes of 0.5 two 519, 291 (661, 566), three 522, 349 (672, 668).
constexpr int NEAR_TILE_MAX = 2;
template <class T>
void launch_near_tile(int nitem, const int2 *items, const int *box_start, const int *col_off, const int *cols,
                      const long long *val_off, const cpx<T> *vals, const int *id_start, const int *id_col,
                      const T *id_w, const cpx<T> *X, cpx<T> *Y, int nrhs, hipStream_t s);
template <class T>
void launch_radiate1(int op, int nbox, int K, int ks, const int *box_start, const cpx<T> *R, const cpx<T> *X, cpx<T> *U,
                     hipStream_t s);
template <class T>
void launch_interp(int nbox, int rows, int in_ks, int out_ks, const int *st, const int *col, const T *w, const cpx<T> *in,
                   cpx<T> *out, int nrhs, bool accumulate, hipStream_t s);
// fixed-size forward stencils (taps = interpolation order 6, 8 or 10);
// return false when the order has no fixed-size kernel
template <class T>
bool launch_interp_fixed(int taps, int nbox, int rows, int in_ks, const int *col, const T *w, const cpx<T> *in,
                         cpx<T> *out, int nrhs, hipStream_t s);
template <class T>
bool launch_agg_phi_fixed(int taps, int nparent, int Kp, int ks_p, int mid_len, const int *child_start, const int *child_oct,
                          const cpx<T> *shift, const int *col, const T *w, const cpx<T> *mid, cpx<T> *Up, int nrhs,
                          hipStream_t s);
template <class T>
void launch_agg_phi(int nparent, int Kp, int ks_p, int mid_len, const int *child_start, const int *child_oct,
                    const cpx<T> *shift, const int *st, const int *col, const T *w, const cpx<T> *mid, cpx<T> *Up,
                    int nrhs, hipStream_t s);
// Tiled translation of every level in one launch.  Per level: the tile
// tables of build_translation_tiles (device copies), the level's translation
// operators (343 offsets x K samples) and its outgoing/incoming patterns.
constexpr int TRANS_MAXLEV = 20;   // the octree has at most 20 levels
// Tile shape of the translation: tmax targets per tile (= waves per
// workgroup, at most TRANS_TMAX_MAX), smax sources per LDS batch and rb
// right-hand sides per lane (1, 2 or 4; above 1 only with four right-hand
// sides across the lanes of a wave).  A target's entries in one batch are
// fetched by the lanes of one wave, so smax <= 64, and each wave stages at
// most TRANS_ROWS rows of 64 lanes, so 2 smax rb <= TRANS_ROWS tmax.
constexpr int TRANS_TMAX_MAX = 16;
constexpr int TRANS_ROWS = 8;
inline bool trans_shape_ok(int tmax, int smax, int rb)
{
    return tmax >= 1 && tmax <= TRANS_TMAX_MAX && smax >= 1 && smax <= 64 && (rb == 1 || rb == 2 || rb == 4) &&
           2 * smax * rb <= TRANS_ROWS * tmax;
}
template <class T>
inline size_t trans_lds_bytes(int smax, int rb) { return (size_t)smax * 2 * 64 * rb * sizeof(cpx<T>); }
// right-hand sides across the lanes of a wave
inline int trans_rw(int nrhs) { return nrhs >= 4 ? 4 : (nrhs >= 2 ? 2 : 1); }
template <class T>
struct TransLevel {
    int K = 0, ks = 0, ntile = 0;   // samples, row stride of U and V
    int nqc = 0, first = 0;     // sample chunks; first position in each XCD's workgroup sequence (launcher)
    const int *tile_tgt = nullptr, *tile_bat = nullptr, *bat_src = nullptr, *src = nullptr;
    const int *bat_row = nullptr, *row = nullptr, *ent = nullptr;
    const cpx<T> *trans = nullptr, *U = nullptr;
    cpx<T> *V = nullptr;
};
template <class T>
struct TransArgs {
    int nlev = 0, nblocks = 0, smax = 0, tmax = 0, rb = 1;   // nblocks: workgroups per XCD
    TransLevel<T> lv[TRANS_MAXLEV];
};
// false when the tile shape is invalid
template <class T>
bool launch_translate_tiled(const TransArgs<T> &a, int nrhs, hipStream_t s);

// A step's stencils in groups of STEP_GROUP[.] outputs (StencilGroups on the
// host): per size the groups, their entries in all and the device tables.
// Keys of a phi table: 2 * column; of a theta table: 2 * row + (1: half a turn
// further in phi).
constexpr int STEP_GROUP[3] = {4, 6, 8};
template <class T>
struct GroupTable {
    int ng[3] = {0, 0, 0}, len[3] = {0, 0, 0};
    const int *start[3] = {}, *key[3] = {};
    const T *w[3] = {};
};
// Launch plan of a whole-box step (levels_box.hip)
template <class T>
struct BoxPlan {
    struct Groups {
        int ng;
        const int *start, *key;
        const T *w;
    };
    int nt = 0, nv = 0;                 // threads per workgroup, vectors per pass
    int cr = 0, nch = 0;                // parent rows per chunk, chunks
    int gphi = 0, gth = 0;              // group sizes STEP_GROUP[.]
    int pitch_x = 0, pitch_m = 0;       // LDS pitches
    int per = 0;                        // vectors per workgroup (per call)
    Groups phi = {}, th = {};
};
// Register-blocked translation over sibling groups (translate.hip; tables
// of GroupTiles in setup.hpp): every lane keeps the sums of all targets of
// its group and streams the group's source records, so a source value is
// loaded once for all the targets whose interaction lists hold it.
template <class T>
struct GroupLevel {
    int K = 0, ks = 0, tks = 0, ngroup = 0;   // samples, row strides of U and V and of the operators
    int nqc = 0, first = 0;     // sample chunks of a workgroup; first position per XCD (launcher)
    const int *first_tgt = nullptr, *count = nullptr, *rec_start = nullptr, *src = nullptr;
    const int *off = nullptr;   // per record tg offset ids, -1 = not in that target's list
    const cpx<T> *trans = nullptr, *U = nullptr;
    cpx<T> *V = nullptr;
};
template <class T>
struct GroupArgs {
    int nlev = 0, nblocks = 0, tg = 4, rb = 1;   // tg: targets per group (4 or 8); rb: RHS per lane
    int rw = 0;                                  // lanes over the RHS (1, 2, 4, 8, 16; 0: trans_rw(nrhs))
    int lds = 0;                                 // 1: operator values staged in LDS (k_translate_lds)
    GroupLevel<T> lv[TRANS_MAXLEV];
};
// false when (tg, rw, rb) has no kernel
template <class T>
bool launch_translate_groups(const GroupArgs<T> &a, int nrhs, hipStream_t s);
// One octree step of aggregation (children at level l+1 -> parents at l) or
// disaggregation (parents -> children), done per box and chunk of theta rows
// in LDS (levels.hip).  Sample index = theta row * nph + phi column.
//  aggregation: workgroup = (parent, chunk of `rows` parent theta rows); the
//    chunk needs child theta rows win[2 c] .. win[2 c + 1] (exclusive);
//  disaggregation: workgroup = (child, chunk of `rows` child theta rows); the
//    chunk needs parent (and intermediate) theta rows win[2 c] .. win[2 c + 1].
// `wrows` is the largest window of any chunk.
template <class T>
struct LevelStep {
    int nbox = 0;                       // parents (aggregation) or children (disaggregation)
    int nth_p = 0, nph_p = 0, nth_c = 0, nph_c = 0;
    int ks_p = 0, ks_c = 0;             // row strides of the parents' and children's patterns
    int rows = 0, nchunk = 0, wrows = 0, taps = 0;
    int rb = 0;                         // right-hand sides per workgroup (0: the launcher's choice)
    int group = 0;                      // aggregation: children staged together (0: the launcher's choice)
    int pipe = 0;                       // > 0: the pipelined kernel; per pass this many vectors (component x
                                        // right-hand side; 1, 2, 4) in the disaggregation, right-hand sides
                                        // (1, 2; 4 counts as 2) in the aggregation
    const int *win = nullptr;
    const int *child_start = nullptr;   // aggregation: children of each parent
    const int *parent = nullptr;        // disaggregation: parent of each child
    const int *oct = nullptr;           // octant of each child in its parent
    // aggregation: theta and phi stencils with `taps` entries per row
    const int *c1 = nullptr, *c2 = nullptr;
    const T *w1 = nullptr, *w2 = nullptr;
    // disaggregation: separable transposed stencils (SepStencil on the host)
    int tphi = 0, tth = 0;
    const int *phi_col = nullptr, *th_row = nullptr, *th_sh = nullptr;
    const T *phi_w = nullptr, *rowf = nullptr, *th_w = nullptr;
    const cpx<T> *shift = nullptr;      // exp(+jk khat.(r_child - r_parent)), 8 x Kp
    const cpx<T> *in = nullptr;
    cpx<T> *out = nullptr;
    const BoxPlan<T> *box = nullptr;    // host: the whole-box kernel's plan, where it is to be used
};
// LDS bytes of a step (both components of the window and of the intermediate)
template <class T>
inline size_t agg_lds_bytes(int wrows, int rows, int nph_c) { return 2 * (size_t)(wrows + rows) * nph_c * sizeof(cpx<T>); }
template <class T>
inline size_t dis_lds_bytes(int wrows, int nph_p, int nph_c) { return 2 * (size_t)wrows * (nph_p + nph_c) * sizeof(cpx<T>); }
constexpr size_t STEP_LDS_MAX = 64 * 1024;
// The whole-box disaggregation (levels_box.hip): a step's plan for nrhs
// right-hand sides or more (false where the step does not fit the kernel) and
// its launch with a.box
template <class T>
bool plan_disaggregate_box(const LevelStep<T> &a, const GroupTable<T> &phi, const GroupTable<T> &th, int nrhs,
                           BoxPlan<T> &plan);
template <class T>
bool launch_disaggregate_box(const LevelStep<T> &a, int nrhs, hipStream_t s);
// One level step on the matrix cores (levels_mfma.hip, complex64): the
// stencils as dense, zero-padded real matrices (see the kernels).  ok = 0
// when the step's stencils are not separable in that form or exceed the
// kernels' tile limits (16 x 8 parent phi columns, 16 x 4 parent theta rows).
struct StepMfma {
    int ok = 0;
    int nbox = 0;                       // parents (aggregation) or children (disaggregation)
    int nth_p = 0, nph_p = 0, nth_c = 0, nph_c = 0;
    int ks_p = 0, ks_c = 0;             // row strides of the parents' and children's patterns (per call)
    const int *child_start = nullptr, *parent = nullptr, *oct = nullptr;
    const cpx<float> *shift = nullptr;
    int njt = 0;                        // tiles of 16 child phi columns
    // aggregation: theta over the child rows extended across the poles
    int nit = 0, ne = 0, e_pad = 0, jc_pad = 0;
    const int *ext_row = nullptr, *ext_sh = nullptr, *ks_lo = nullptr, *ks_hi = nullptr;
    const float *ath = nullptr;         // [nit * 16][e_pad]
    const float *bph = nullptr;         // [16 * ceil(nph_p / 16)][jc_pad]
    const unsigned *bmask = nullptr;    // per child phi tile: bit p = block p of bph is non-zero
    // disaggregation
    int nks = 0, jp_pad = 0, nict = 0, ip_pad = 0;
    unsigned rmask = 0;                 // parent theta tiles reached across a pole
    const unsigned long long *kmask = nullptr, *kmask_s = nullptr;   // per child phi tile: non-zero k-steps
    const float *dph = nullptr;         // [njt * 16][jp_pad]
    const float *rowf = nullptr;        // [ip_pad]
    const float *dthd = nullptr, *dthr = nullptr;   // [nict * 16][ip_pad]
    const unsigned *dmask = nullptr, *rmask_c = nullptr;   // per child theta tile
};
bool launch_aggregate_mfma(const StepMfma &a, const cpx<float> *in, cpx<float> *out, int nrhs, hipStream_t s);
bool launch_disaggregate_mfma(const StepMfma &a, const cpx<float> *in, cpx<float> *out, int nrhs, hipStream_t s);

// return false when the step has no fused kernel (taps or LDS size)
template <class T>
bool launch_aggregate_step(const LevelStep<T> &a, int nrhs, hipStream_t s);
template <class T>
bool launch_disaggregate_step(const LevelStep<T> &a, int nrhs, hipStream_t s);

// Radiation of two or more right-hand sides, on the matrix cores (mfma.hip):
// FP32 MFMAs for complex float, FP64 MFMAs for complex double
template <class T>
void launch_radiate_mfma(int op, int nbox, int K, int ks, const int *box_start, const cpx<T> *R, const cpx<T> *X, cpx<T> *U,
                         int nrhs, hipStream_t s);
// Near field of more than NEAR_TILE_MAX and receive of more than
// RECEIVE_ROWS_MAX right-hand sides.
// items = (leaf box, row tile of 16 rows) pairs; cols[col_off[b] ..] = the
// RWGs of leaf box b's adjacent boxes in block-row order.
template <class T>
void launch_near_mfma(int nitem, const int2 *items, const int *box_start, const int *col_off, const int *cols,
                      const long long *val_off, const cpx<T> *vals, const int *id_start, const int *id_col,
                      const T *id_w, const cpx<T> *X, cpx<T> *Y, int nrhs, hipStream_t s);
template <class T>
void launch_receive_mfma(int op, int nitem, const int2 *items, int K, int ks, const int *box_start, const cpx<T> *R,
                         const cpx<T> *Q, const T *wq, const cpx<T> *V, cpx<T> *Y, int nrhs, hipStream_t s);

// Outer GMRES vector kernels (krylov.hip); column-major blocks, element
// (n, r) at r * ld + n; basis vector i of V starts at V + i * vstride.
// out[i * nrhs + r] = <V_i(:, r), w(:, r)> (conjugate-linear in V), i < nv,
// accumulated in double; part holds nv x nchunk x nrhs partial sums.
template <class T>
void krylov_dots(const cpx<T> *V, long long vstride, long long ldv, int nv, const cpx<T> *w, long long ldw, long long n,
                 int nrhs, cpx<double> *part, int nchunk, cpx<double> *out, hipStream_t s);
// One Arnoldi step's orthogonalisation (vectors of n rows, stride n nrhs, no
// padding): w against V_0 .. V_(nv - 1) twice, next = w / |w|; the coefficients
// of the two passes in h1, h2 ([i][rhs]), |w|^2 in sq.  And w / |w| alone.
template <class T>
void krylov_step(const cpx<T> *V, int nv, cpx<T> *w, cpx<T> *next, long long n, int nrhs, cpx<double> *part, int nchunk,
                 cpx<double> *sq, cpx<double> *h1, cpx<double> *h2, hipStream_t s);
template <class T>
void krylov_normalise(const cpx<T> *w, cpx<T> *y, long long n, int nrhs, cpx<double> *part, int nchunk, cpx<double> *sq,
                      hipStream_t s);
// w(:, r) += sign * sum_i V_i(:, r) h[i * nrhs + r]
template <class T>
void krylov_combine(const cpx<T> *V, long long vstride, long long ldv, int nv, const cpx<double> *h, double sign,
                    cpx<T> *w, long long ldw, long long n, int nrhs, hipStream_t s);
// y(:, r) = a[r] x(:, r) + b[r] z(:, r)  (z = null: the second term is dropped)
template <class T>
void krylov_axpby(const cpx<double> *a, const cpx<T> *x, long long ldx, const cpx<double> *b, const cpx<T> *z,
                  long long ldz, cpx<T> *y, long long ldy, long long n, int nrhs, hipStream_t s);

// Column-major blocks between precisions: b = (complex float) a; a = b, or
// a += b with add.
void launch_to_single(const cpx<double> *a, long long lda, cpx<float> *b, long long ldb, long long n, int nrhs,
                      hipStream_t s);
void launch_from_single(cpx<double> *a, long long lda, const cpx<float> *b, long long ldb, long long n, int nrhs,
                        bool add, hipStream_t s);

// Sparse (CSR) times a column-major block: y(i, r) = alpha * sum_k val[k]
// x(col[k], r) (+ y(i, r) with accumulate), rows i < nrows.
template <class T>
void launch_csr_spmm(long long nrows, int nrhs, const long long *ptr, const int *col, const cpx<T> *val,
                     const cpx<T> *x, long long ldx, cpx<T> *y, long long ldy, double alpha, bool accumulate,
                     hipStream_t s);

template <class T>
void launch_disagg_mid(int nchild, int mid_len, int Kp, int ks_p, const int *parent, const int *oct, const cpx<T> *shift,
                       const int *st, const int *col, const T *w, const cpx<T> *Vp, cpx<T> *mid, int nrhs,
                       hipStream_t s);
template <class T>
void launch_zero(cpx<T> *p, long long n, hipStream_t s);
// Receive of 1 to RECEIVE_ROWS_MAX right-hand sides, a wave per RWG.  More go
// to the matrix cores, whose tiles of 16 rows and 8 right-hand sides are mostly
// empty at two and three.  Matrix cores against waves, us: sphere of 38 880
// RWGs, complex64 (complex128), two 89, 54 (109, 81), three 91, 77 (112, 98),
// four 92, 107 (114, 116); of 122 880 271, 157 (323, 238), 274, 222 (334, 294),
// 278, 327 (348, 345); ellipsoid of 48 000 with leaf boxes of 0.5 183, 107 (228,
// 182), 187, 137 (239, 211), 191, 171 (256, 241).
constexpr int RECEIVE_ROWS_MAX = 3;
template <class T>
void launch_receive_rows(int op, int N, int K, int ks, const int *leaf_of, const cpx<T> *R, const cpx<T> *Q, const T *wq,
                         const cpx<T> *V, cpx<T> *Y, int nrhs, hipStream_t s);
// One right-hand side with the permutations folded in: the radiation reads
// the caller's vector x (user order, J half then M half) through perm (tree
// position -> user RWG) and also stores it in tree order in X; the receive
// adds the far field to the tree-order near field Y and writes the sum to y
// in user order.
template <class T>
void launch_radiate1_user(int op, int nbox, int K, int ks, const int *box_start, const cpx<T> *R, const cpx<T> *x,
                          const int *perm, int N, cpx<T> *X, cpx<T> *U, hipStream_t s);
template <class T>
void launch_receive1_user(int op, int N, int K, int ks, const int *leaf_of, const cpx<T> *R, const cpx<T> *Q, const T *wq,
                          const cpx<T> *V, const cpx<T> *Y, cpx<T> *y, const int *perm, hipStream_t s);

}  // namespace mlfma
