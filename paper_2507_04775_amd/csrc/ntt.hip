// Negacyclic NTT / inverse NTT for gfx950 (paper Sec. III-F.4).
//
// Forward: radix-2 Cooley-Tukey with the psi twist merged into the
// butterflies, natural coefficients -> bit-reversed evaluations.  Inverse:
// Gentleman-Sande butterflies, bit-reversed -> natural, times N^-1.  The
// butterfly of stage m at index j uses w = psi^br(m + j div 2t) from the
// context tables.
//
// Layout of the work: threads own a few elements each and run several radix-2
// stages on them in registers ("rounds"); rounds exchange data through LDS.
// N = 2^12 fits one workgroup of 512 threads with 8 elements each (four rounds
// of three stages); inside key switches it runs as 64 x 64 in two passes.  N = 2^16 is the paper's 2-D / hierarchical scheme:
// viewed as a 256 x 256 matrix, a column pass runs the first eight stages
// (each column is an independent 256-point problem) and a row pass runs the
// last eight (each row of 256 contiguous elements is independent, with its own
// twiddle subset).  Each pass reads and writes every element once: four global
// accesses per element in total.  A pass workgroup holds 16 columns (rows) with
// 32 threads on each and 8 elements per thread, in rounds of 3, 3 and 2
// stages: short dependency chains per thread and twice the waves of a
// 16-element layout, which matters most for the slower integer path.
//
// Two arithmetic paths, chosen per limb (uniform per workgroup):
// - primes below 2^50: exact FP64 arithmetic (modarith.h).  Values are
//   signed representatives; a centred reduction at the start of each round
//   keeps |x| <= q/2 + 1, after which four forward stages stay below 5.3 q
//   (7.1 q when a round starts from canonical input) and four inverse stages,
//   with the sums of the third stage re-centred, below 4 q; all < 2^53.
// - other primes (up to 2^61): 64-bit integers with Shoup twiddles and lazy
//   butterflies after Harvey ([0, 8q) forward, [0, 4q) inverse).
// Outputs of every transform are canonical.
#include <atomic>

#include "coef_units.h"
#include "internal.h"
#include "unit_map.h"

namespace ckks {

namespace {

// SwitchModulo of the rescale: u in [0, q_l) lifted centred and reduced mod q
__device__ __forceinline__ uint64_t switch_modulo(uint64_t u, uint64_t half, uint64_t qlmod, const Prime &P)
{
    uint64_t um = csub(u - mul_hi(u, P.one_s) * P.q, P.q);
    return u <= half ? um : submod(um, qlmod, P.q);
}

// ----------------------------------------------------------- integer path

struct IntArith {
    typedef uint64_t V;
    typedef ulonglong2 W;
    const ulonglong2 *T;
    uint64_t q, q4, nq, fc, fc_s;  // 4q, 2^64 - q; fc: constant of the last inverse multiplication

    __device__ __forceinline__ V from_u64(uint64_t x) const { return x; }
    __device__ __forceinline__ V from_bits(uint64_t x) const { return x; }
    __device__ __forceinline__ uint64_t to_bits(V x) const { return x; }
    __device__ __forceinline__ W tw(uint32_t i) const { return T[i]; }
    // the twiddle at hi + k (k below the lowest set bit of hi): read from the table
    __device__ __forceinline__ W tw_split(uint32_t hi, uint32_t k) const { return T[hi + k]; }
    // the same twiddle for all lanes, through the scalar cache
    __device__ __forceinline__ W tw_uniform(uint32_t i) const
    {
        const auto *t = (const __attribute__((address_space(4))) uint64_t *)T;
        return make_ulonglong2(t[2 * i], t[2 * i + 1]);
    }
    // [x y]_q of two canonical residues (HMult's d2 = a1 b1 as it is loaded)
    __device__ __forceinline__ V product(uint64_t x, uint64_t y, const Prime &P) const
    {
        return reduce128(mul_wide(x, y), P);
    }
    template <int NV>
    __device__ __forceinline__ void reduce_all(V (&)[NV]) const {}
    // Butterflies after Harvey, with shoup_add's products in [0, 4q): forward x, y in [0, 8q) ->
    // [0, 8q) (x brought below 4q, x + t formed by the product's own multiply-adds), inverse x, y in
    // [0, 4q) -> [0, 4q).  8q fits a word (q < 2^61).
    __device__ __forceinline__ void ct(V &x, V &y, W w) const
    {
        const uint64_t a = csub_sign(x, 4 * nq);
        x = shoup_add(a, y, w.x, w.y, nq);
        y = shl_add<1>(a, q4) - x;
    }
    __device__ __forceinline__ void gs(V &x, V &y, W w, int) const
    {
        const uint64_t d = x + q4 - y;
        x = csub_sign(x + y, 4 * nq);
        y = shoup_add(0, d, w.x, w.y, nq);
    }
    __device__ __forceinline__ uint64_t fwd_final(V x) const
    {
        return csub_sign(csub_sign(csub_sign(x, 4 * nq), 2 * nq), nq);
    }
    __device__ __forceinline__ uint64_t inv_final(V x) const
    {
        return csub_sign(csub_sign(shoup_add(0, x, fc, fc_s, nq), 2 * nq), nq);
    }
    __device__ __forceinline__ uint64_t modulus() const { return q; }
    // exact sums of products with canonical residues k, reduced once (at most kMaxDigits + 2 terms)
    typedef u128 Sum;
    __device__ __forceinline__ void sum_start(Sum &s) const { s = {0, 0}; }
    __device__ __forceinline__ void sum_add(Sum &s, V x, uint64_t k) const { s = add128(s, mul_wide(x, k)); }
    __device__ __forceinline__ void sum_centre(Sum &) const {}
    __device__ __forceinline__ V sum_value(const Sum &s, const Prime &P) const { return reduce128(s, P); }
    __device__ __forceinline__ V sum_input(V x) const { return fwd_final(x); }  // of a forward output
    // c (aux - x) + add for a forward output x and canonical aux, add: P^-1 (acc - Conv) + add of
    // ModDown, q_l^-1 (c - .) of Rescale
    __device__ __forceinline__ uint64_t scaled_difference(V x, V aux, uint64_t add, ulonglong2 c) const
    {
        const uint64_t r = shoup_add(add, aux + q - fwd_final(x), c.x, c.y, nq);  // below 5q
        return csub_sign(csub_sign(csub_sign(r, 4 * nq), 2 * nq), nq);
    }
    // SwitchModulo of the rescale: u in [0, q_l) lifted centred and reduced
    __device__ __forceinline__ V lift(uint64_t u, uint64_t ql, uint64_t qlmod, const Prime &P) const
    {
        return switch_modulo(u, (ql - 1) >> 1, qlmod, P);
    }
};

// ----------------------------------------------------------- FP64 path

struct FpArith {
    typedef double V;
    typedef double W;
    const double *T;
    FpMod m;
    double fc;  // constant of the last inverse multiplication

    __device__ __forceinline__ V from_u64(uint64_t x) const { return fp_from_word(x); }
    __device__ __forceinline__ V from_bits(uint64_t x) const { return __longlong_as_double((long long)x); }
    __device__ __forceinline__ uint64_t to_bits(V x) const { return (uint64_t)__double_as_longlong(x); }
    __device__ __forceinline__ W tw(uint32_t i) const { return T[i]; }
    // the twiddle at hi + k, k below the lowest set bit of hi: the table holds psi^br(i) (or its
    // inverse), and br(hi + k) = br(hi) + br(k) for such k, so it is T[hi] T[k], formed here (a
    // centred representative) from the row's one entry and the first entries shared by every row
    __device__ __forceinline__ W tw_split(uint32_t hi, uint32_t k) const { return fp_mulmod(T[hi], T[k], m); }
    __device__ __forceinline__ W tw_uniform(uint32_t i) const
    {
        return ((const __attribute__((address_space(4))) double *)T)[i];
    }
    // [x y]_q of two canonical residues below 2^50, a centred representative
    __device__ __forceinline__ V product(uint64_t x, uint64_t y, const Prime &) const
    {
        return fp_mulmod(fp_from_word(x), fp_from_word(y), m);
    }
    template <int NV>
    __device__ __forceinline__ void reduce_all(V (&v)[NV]) const
    {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = fp_reduce(v[i], m);
    }
    __device__ __forceinline__ void ct(V &x, V &y, W w) const
    {
        double t = fp_mulmod(y, w, m);
        double a = x;
        x = a + t;
        y = a - t;
    }
    // the sums of the third stage of a round (st == 2) are re-centred
    __device__ __forceinline__ void gs(V &x, V &y, W w, int st) const
    {
        double s = x + y, d = x - y;
        x = st == 2 ? fp_reduce(s, m) : s;
        y = fp_mulmod(d, w, m);
    }
    __device__ __forceinline__ uint64_t fwd_final(V x) const { return fp_canonical(x, m); }
    __device__ __forceinline__ uint64_t inv_final(V x) const { return fp_canonical(fp_mulmod(x, fc, m), m); }
    __device__ __forceinline__ uint64_t modulus() const { return (uint64_t)m.q; }
    // sums of products, each below 2.9 q: sum_centre after every second term at the latest
    typedef double Sum;
    __device__ __forceinline__ void sum_start(Sum &s) const { s = 0.0; }
    __device__ __forceinline__ void sum_add(Sum &s, V x, uint64_t k) const { s += fp_mulmod(x, fp_from_word(k), m); }
    __device__ __forceinline__ void sum_centre(Sum &s) const { s = fp_reduce(s, m); }
    __device__ __forceinline__ V sum_value(const Sum &s, const Prime &) const { return fp_reduce(s, m); }
    __device__ __forceinline__ V sum_input(V x) const { return x; }
    // as IntArith's; |x| < 5.3 q, |aux| <= q leave the difference below 2^53 and the product below 2.9 q
    __device__ __forceinline__ uint64_t scaled_difference(V x, V aux, uint64_t add, ulonglong2 c) const
    {
        return fp_canonical(fp_mulmod(aux - x, (double)c.x, m) + fp_from_word(add), m);
    }
    __device__ __forceinline__ V lift(uint64_t u, uint64_t ql, uint64_t qlmod, const Prime &P) const
    {
        if (ql < kFpMaxPrime) {  // the centred lift itself, below 2^49
            const double d = fp_from_word(u), l = (double)ql;
            return d > 0.5 * l ? d - l : d;
        }
        return from_u64(switch_modulo(u, (ql - 1) >> 1, qlmod, P));
    }
};

// Stores the last inverse pass's outputs: coefficients (ys_mode 0), or a base
// conversion's inputs, cut for its sums (cut_word).  For ModDown's centred
// conversion (ys_mode 2) each canonical y of the special limb p goes in as y + p
// when y <= (p - 1)/2, else as y: the centred representative plus p, in
// [(p + 1)/2, 3 (p - 1)/2], below 2^62, so the sums take no per-term comparison
// (their constant rows remove the shift).
template <int NV, class A, class Idx>
__device__ __forceinline__ void inv_store(uint64_t *dst, const typename A::V (&v)[NV], const A &ar, uint32_t ys_mode,
                                          Idx idx)
{
    if (ys_mode == 2) {
        const uint64_t q = ar.modulus(), half = q >> 1;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const uint64_t y = ar.inv_final(v[i]);
            dst[idx(i)] = cut_word(y <= half ? y + q : y);
        }
    } else if (ys_mode == 1) {
#pragma unroll
        for (int i = 0; i < NV; ++i) dst[idx(i)] = cut_word(ar.inv_final(v[i]));
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) dst[idx(i)] = ar.inv_final(v[i]);
    }
}

// LOG forward stages on v[i] = element base + STRIDE i (i < 2^LOG) of an
// NS-point problem: t = 2^(LOG-1) STRIDE, ..., STRIDE.  base = a 2^LOG STRIDE
// + s with s < STRIDE.  Twiddles come from T[m B + j div 2t], m = NS / 2t.
// tw_fwd loads the 2^LOG - 1 twiddles a round uses (stage by stage, group by
// group) and fwd_rw applies them, so a pass can issue a round's twiddle loads
// before the barrier that precedes the round.
//
// Row passes (ROW, B = 256 + row) take the stages with NS / 2t >= kTwSplit
// groups per row as tw_split(m B, j div 2t): one table entry per row and
// stage, and the first entries of the table, which every row shares.  A row
// then reads 34 of its 255 twiddles from the table instead of all of them.
constexpr uint32_t kTwSplit = 32;

template <int LOG, int NS, int STRIDE, class A, bool ROW = false>
__device__ __forceinline__ void tw_fwd(typename A::W *w, uint32_t base, const A &ar, uint32_t B)
{
    int k = 0;
#pragma unroll
    for (int st = 0; st < LOG; ++st) {
        const uint32_t t = ((1u << (LOG - 1)) >> st) * STRIDE;
        const uint32_t hi = (NS / (2 * t)) * B, g0 = base / (2 * t);
#pragma unroll
        for (int g = 0; g < (1 << st); ++g)
            w[k++] = ROW && NS / (2 * t) >= kTwSplit ? ar.tw_split(hi, g0 + g) : ar.tw(hi + g0 + g);
    }
}

template <int LOG, class A>
__device__ __forceinline__ void fwd_rw(typename A::V *v, const typename A::W *w, const A &ar)
{
    int k = 0;
#pragma unroll
    for (int st = 0; st < LOG; ++st) {
        const int h = (1 << (LOG - 1)) >> st;
#pragma unroll
        for (int g = 0; g < (1 << st); ++g) {
            const typename A::W ww = w[k++];
#pragma unroll
            for (int kk = 0; kk < h; ++kk) ar.ct(v[g * 2 * h + kk], v[g * 2 * h + kk + h], ww);
        }
    }
}

// LOG inverse stages: t = STRIDE, 2 STRIDE, ..., 2^(LOG-1) STRIDE.  Rounds
// of four stages re-centre the sums of their third stage (FP64 path); three
// stages from a centred start stay below 4 q + 8 without it.
template <int LOG, int NS, int STRIDE, class A, bool ROW = false>
__device__ __forceinline__ void tw_inv(typename A::W *w, uint32_t base, const A &ar, uint32_t B)
{
    int k = 0;
#pragma unroll
    for (int st = 0; st < LOG; ++st) {
        const uint32_t t = (1u << st) * STRIDE;
        const uint32_t hi = (NS / (2 * t)) * B, g0 = base / (2 * t);
#pragma unroll
        for (int g = 0; g < ((1 << (LOG - 1)) >> st); ++g)
            w[k++] = ROW && NS / (2 * t) >= kTwSplit ? ar.tw_split(hi, g0 + g) : ar.tw(hi + g0 + g);
    }
}

template <int LOG, class A>
__device__ __forceinline__ void inv_rw(typename A::V *v, const typename A::W *w, const A &ar)
{
    int k = 0;
#pragma unroll
    for (int st = 0; st < LOG; ++st) {
        const int h = 1 << st;
#pragma unroll
        for (int g = 0; g < ((1 << (LOG - 1)) >> st); ++g) {
            const typename A::W ww = w[k++];
#pragma unroll
            for (int kk = 0; kk < h; ++kk) ar.gs(v[g * 2 * h + kk], v[g * 2 * h + kk + h], ww, LOG == 4 ? st : -1);
        }
    }
}

// The thread's index, opaque to loop-invariant code motion, for the pass
// bodies of the persistent kernels at N = 2^16.  Those run a body once per
// claimed unit; offsets derived from threadIdx.x and hoisted out of that loop
// stay live in vector registers across the whole body (ModDown's conversion
// pass needed 154 per thread that way, 124 with this index, and the forward
// column pass 118 against 70).  Grid kernels pass threadIdx.x itself.
__device__ __forceinline__ uint32_t thread_index()
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

struct LimbPos {
    uint32_t poly, row, prime;
    bool skip;
};

// Field of polynomial p (0 or 1) of a two-entry argument array, as a select:
// the argument block then has no dynamically indexed field and a persistent
// kernel keeps it in scalar registers.
template <class T>
__device__ __forceinline__ T pick(T const (&v)[2], uint32_t p)
{
    return p ? v[1] : v[0];
}

__host__ __device__ __forceinline__ LimbPos limb_pos(const LimbMap &m, uint32_t limb)
{
    LimbPos p;
    if (m.dense && m.skip_alpha) {
        // the limb-th row that is not skipped: polynomial j leaves out its rows
        // [j alpha, min(j alpha + alpha, level + 1)) (row0 = 0 in such launches)
        uint32_t rem = limb, poly = 0;
        for (;;) {
            const uint32_t lo = poly * m.skip_alpha;
            const uint32_t hi = lo + m.skip_alpha < m.level + 1 ? lo + m.skip_alpha : m.level + 1;
            const uint32_t gap = hi > lo ? hi - lo : 0, kept = m.rows - gap;
            if (rem < kept) {
                p.poly = poly;
                p.row = rem < lo ? rem : rem + gap;
                break;
            }
            rem -= kept;
            ++poly;
        }
        p.skip = false;
    } else {
        p.poly = limb / m.rows;
        p.row = limb - p.poly * m.rows;
        p.skip = limb_skipped(m, p.poly, p.row);
    }
    p.prime = limb_prime(m, p.row);
    return p;
}

template <int PRO, class A>
__device__ __forceinline__ typename A::V load_fwd(const NttArgs &a, const LimbPos &lp, const A &ar, const uint64_t *src,
                                                  uint32_t e, const Prime &P)
{
    if (PRO == PRO_RESCALE) return ar.lift(pick(a.rs_src, lp.poly)[e], a.rs_ql, a.rs_qlmod[lp.prime], P);
    return ar.from_u64(src[e]);
}

// What a forward pass leaves for its store: the canonical residue, or the value
// itself where an epilogue goes on with it.
template <int EPI, class A>
__device__ __forceinline__ uint64_t fwd_out(const A &ar, typename A::V v)
{
    return EPI == EPI_PLAIN ? ar.fwd_final(v) : ar.to_bits(v);
}

// Final forward value (fwd_out's x) at element e of the limb; `addv` is the
// addend of the ModDown epilogue (already gathered, 0 without addend).
template <int EPI, class A>
__device__ __forceinline__ void store_fwd(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *dst, uint32_t e,
                                          uint64_t x, uint64_t addv, uint64_t auxv, size_t N)
{
    if (EPI == EPI_PLAIN) {
        dst[e] = x;
    } else {
        pick(a.out, lp.poly)[(size_t)lp.row * N + e] =
            ar.scaled_difference(ar.from_bits(x), ar.from_u64(auxv), EPI == EPI_MODDOWN ? addv : 0, a.cst[lp.prime]);
    }
}

__device__ __forceinline__ IntArith int_arith(const ulonglong2 *tw, const Prime &P, uint32_t prime, uint32_t N)
{
    IntArith r;
    r.T = tw + (size_t)prime * N;
    r.q = P.q;
    r.q4 = 2 * P.two_q;
    r.nq = 0 - P.q;
    r.fc = P.ninv;
    r.fc_s = P.ninv_s;
    return r;
}

__device__ __forceinline__ FpArith fp_arith(const double *twd, const Prime &P, uint32_t prime, uint32_t N)
{
    FpArith r;
    r.T = twd + (size_t)prime * N;
    r.m.q = (double)P.q;
    r.m.qinv = P.qinv;
    r.fc = (double)P.ninv;
    return r;
}

__device__ __forceinline__ IntArith int_arith(const NttArgs &a, const Prime &P, uint32_t prime, uint32_t N)
{
    return int_arith(a.tw, P, prime, N);
}

__device__ __forceinline__ FpArith fp_arith(const NttArgs &a, const Prime &P, uint32_t prime, uint32_t N)
{
    return fp_arith(a.twd, P, prime, N);
}

// Constant of the last inverse multiplication of a limb: N^-1, or the
// base-conversion input scale N^-1 [(B/b_i)^-1]_{b_i} (ys_mode 1 / 2).
__device__ __forceinline__ uint32_t ys_index(const NttArgs &a, const LimbPos &lp)
{
    if (a.ys_mode == 1) {
        const uint32_t r = lp.row + a.map.row0, j = r / a.alpha, lo = j * a.alpha;
        const uint32_t ns = min(a.alpha, a.nlev - lo);
        return (j * a.alpha + ns - 1) * kMaxDigitPrimes + (r - lo);
    }
    return a.pset * kMaxDigitPrimes + lp.row;
}

__device__ __forceinline__ IntArith inv_int_arith(const NttArgs &a, const LimbPos &lp, const Prime &P, uint32_t N)
{
    IntArith r = int_arith(a, P, lp.prime, N);
    if (a.ys_mode) {
        const ulonglong2 c = a.ys[ys_index(a, lp)];
        r.fc = c.x;
        r.fc_s = c.y;
    }
    return r;
}

__device__ __forceinline__ FpArith inv_fp_arith(const NttArgs &a, const LimbPos &lp, const Prime &P, uint32_t N)
{
    FpArith r = fp_arith(a, P, lp.prime, N);
    if (a.ys_mode) r.fc = a.ysd[ys_index(a, lp)];
    return r;
}

// Source of a base conversion computed in the first forward pass (PRO_BCONV).
struct BcSrc {
    const uint64_t *y;   // ns scaled source rows, stride N
    const uint64_t *hm;  // the target prime's constant row (kConvRow)
    uint32_t ns;
};

__device__ __forceinline__ BcSrc bc_source(const NttArgs &a, uint32_t poly, uint32_t prime)
{
    BcSrc b;
    b.ns = a.nprimes - a.map.nq;
    b.y = a.bc_src + (int64_t)poly * a.bc_poly_stride;
    b.hm = a.hmod + ((size_t)a.pset * a.nprimes + prime) * kConvRow;
    return b;
}

typedef const __attribute__((address_space(4))) uint64_t ConvWord;  // constants through the scalar cache

// Accumulator of one converted element: the sum of its terms, then its value
// in the limb's arithmetic.  FoldAcc, FoldWideAcc: two columns and an FP64
// quotient (four multiply-adds a term, 14 and 20 instructions for the residue).
// WideAcc, where those do not hold the sum: exact 128-bit sums reduced once, by
// MacSplit's carry-free columns below 2^50 and by MacCols (carries counted) above.
struct FoldAcc {
    FoldSum s;
    __device__ __forceinline__ void start(ConvWord *h) { s.a = h[kConvStart], s.b = h[kConvStart + 1]; }
    __device__ __forceinline__ void add(uint64_t y, ConvWord *h, uint32_t k) { s.add(y, h[2 * k], h[2 * k + 1]); }
    __device__ __forceinline__ double value(const FpArith &ar, ConvWord *, const Prime &) const { return s.residue(ar.m); }
};
struct FoldWideAcc {
    FoldSumWide s;
    __device__ __forceinline__ void start(ConvWord *h) { s.a = 0, s.b = h[kConvStart + 1]; }
    __device__ __forceinline__ void add(uint64_t y, ConvWord *h, uint32_t k) { s.add(y, h[2 * k], h[2 * k + 1]); }
    __device__ __forceinline__ uint64_t value(const IntArith &, ConvWord *, const Prime &P) const
    {
        return s.residue(P.q, P.qinv);
    }
};
template <class Acc>
struct WideAcc {
    Acc s;
    __device__ __forceinline__ void start(ConvWord *) {}
    __device__ __forceinline__ void add(uint64_t y, ConvWord *h, uint32_t k) { s.add(join_word(y), h[k]); }
    template <class A>
    __device__ __forceinline__ typename A::V value(const A &ar, ConvWord *h, const Prime &P) const
    {
        return ar.from_u64(addmod(reduce128(s.total(), P), h[kConvStart + 1], P.q));
    }
};

// v[i] = Conv(y)[pos(i)]: sum_k y_k[pos] [B/b_k]_q, reduced once.  Groups of
// four elements keep the column sums in few registers; a group's loads are
// issued four source rows at a time, before the first of their products, so a
// group waits once for every four rows.
constexpr uint32_t kConvBatch = 4;

template <class Acc, int NV, class A, class Pos>
__device__ __forceinline__ void bconv_acc(typename A::V (&v)[NV], const A &ar, const BcSrc &b, const Prime &P,
                                          size_t N, Pos pos)
{
    constexpr int G = 4;
    static_assert(NV % G == 0, "groups of four elements");
    ConvWord *h = (ConvWord *)b.hm;
#pragma unroll
    for (int grp = 0; grp < NV / G; ++grp) {
        Acc acc[G];
#pragma unroll
        for (int i = 0; i < G; ++i) acc[i].start(h);
        for (uint32_t k0 = 0; k0 < b.ns; k0 += kConvBatch) {
            uint64_t y[kConvBatch][G];
#pragma unroll
            for (uint32_t t = 0; t < kConvBatch; ++t)
                if (k0 + t < b.ns) {
                    const uint64_t *row = b.y + (size_t)(k0 + t) * N;
#pragma unroll
                    for (int i = 0; i < G; ++i) y[t][i] = row[pos(G * grp + i)];
                }
#pragma unroll
            for (uint32_t t = 0; t < kConvBatch; ++t)
                if (k0 + t < b.ns) {
#pragma unroll
                    for (int i = 0; i < G; ++i) acc[i].add(y[t][i], h, k0 + t);
                }
        }
#pragma unroll
        for (int i = 0; i < G; ++i) v[G * grp + i] = acc[i].value(ar, h, P);
    }
}

template <int NV, class Pos>
__device__ __forceinline__ void bconv_load(double (&v)[NV], const FpArith &ar, const BcSrc &b, const Prime &P,
                                           size_t N, Pos pos)
{
    if (b.ns <= kFoldMaxTerms)
        bconv_acc<FoldAcc>(v, ar, b, P, N, pos);
    else
        bconv_acc<WideAcc<MacSplit>>(v, ar, b, P, N, pos);
}

template <int NV, class Pos>
__device__ __forceinline__ void bconv_load(uint64_t (&v)[NV], const IntArith &ar, const BcSrc &b, const Prime &P,
                                           size_t N, Pos pos)
{
    if (((ConvWord *)b.hm)[kConvStart])
        bconv_acc<FoldWideAcc>(v, ar, b, P, N, pos);
    else
        bconv_acc<WideAcc<MacColsAcc>>(v, ar, b, P, N, pos);
}

// ------------------------------------------------------------------ N = 2^16
// Every kernel body processes one "unit": tile `tile` (16 columns or 16 rows
// of the 256 x 256 view) of limb `limb` of a launch described by NttArgs.
// Grid kernels take (tile, limb) from (blockIdx.x, blockIdx.y); persistent
// kernels claim units from a work queue (see the end of this file).
//
// A unit runs on 512 threads: 32 per column (row), each holding 8 of its 256
// elements.  Element positions within the 256-point problem in the three
// layouts a thread s < 32 takes:
//   wide   s + 32 i          (stages t = 128, 64, 32; coalesced global access)
//   mid    32 (s/4) + s%4 + 4 i (stages t = 16, 8, 4)
//   narrow 8 s + i            (stages t = 2, 1 as two radix-4 groups)
// Between layouts each thread stores what it holds and, after one barrier,
// loads the next layout; a thread only ever overwrites slots it loaded itself,
// so one barrier per exchange suffices.

constexpr int kThreads16 = 512;

// The 32 threads of a row lie in one 64-wide wave (a wave holds two rows), so
// the row passes exchange data through LDS within the wave: a release fence,
// a wave barrier and an acquire fence order the LDS stores before the loads of
// other lanes, with no workgroup barrier.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t pos_wide(uint32_t s, int i) { return s + 32 * i; }
__device__ __forceinline__ uint32_t pos_mid(uint32_t s, int i) { return 32 * (s >> 2) + (s & 3) + 4 * i; }
__device__ __forceinline__ uint32_t pos_narrow(uint32_t s, int i) { return 8 * s + i; }

// LDS slot of element e of column `col` in a column pass over a tile of TW
// columns: the columns interleaved (element-major) and every group of 8
// elements padded by one word.  A half-wave (TW columns x 32/TW threads) then
// touches 32 consecutive words in the wide and mid layouts and 32 / TW groups
// of TW words spread over all banks in the narrow one (TW = 16, 8, 4).
template <int TW>
__device__ __forceinline__ uint32_t col_slot(uint32_t e, uint32_t col) { return TW * (e + (e >> 3)) + col; }
constexpr int kColLds = 16 * (255 + 31 + 1);

// LDS slot of element e of a row (256 words per row): the low five bits are
// XOR-swizzled with f(e / 32), f(h) = h ^ 4h, so that the 32 threads of a row
// (one half-wave) hit 32 distinct banks in each of the three layouts.
__device__ __forceinline__ uint32_t row_slot(uint32_t e)
{
    const uint32_t h = e >> 5;
    return (e & ~31u) | ((e ^ h ^ (h << 2)) & 31u);
}
constexpr int kLds16 = kColLds > 16 * 256 ? kColLds : 16 * 256;
// Tile widths: 16 columns (rows) of the 256 x 256 view per workgroup of 512
// threads, the layout of every persistent pass and of grid launches over many
// limbs; 8 or 4 per workgroup of 256 or 128 threads for launches over few
// limbs, which then have two or four times the workgroups to spread over the
// 256 CUs.  LDS per workgroup: TW (255 + 31 + 1) words.
template <int TW>
constexpr int lds_words() { return TW * (255 + 31 + 1); }

// Where the row passes keep the values between a transform's two passes.
// Natural: row b of 256 words, as the column passes read it.  Tiled (a.tiled):
// tiles of 4 columns x 256 rows in 8 KB each, for the column launch (k16_cols),
// whose wave takes one tile; in a tile the rows come as 16 (b mod 16) + b / 16,
// so that its round on rows 16 s + i reads and writes 512 consecutive bytes.
// A row pass's workgroup then takes rows with the same b mod 16: its accesses
// run over 32 TW bytes of every tile.  Such a pass does not work in place.
struct MidRow {
    uint64_t *p;      // the thread's first value, column s
    uint32_t step;    // to column s + step columns
};
template <int STEP>
__device__ __forceinline__ MidRow mid_row(const NttArgs &a, uint64_t *limb, uint32_t b, uint32_t s)
{
    MidRow m;
    m.p = limb + (a.tiled ? (s >> 2) * 1024 + (b & 15) * 64 + (b >> 4) * 4 + (s & 3) : b * 256 + s);
    m.step = a.tiled ? STEP * 256 : STEP;
    return m;
}
template <int TW>
__device__ __forceinline__ uint32_t pass_row(const NttArgs &a, uint32_t tile, uint32_t blk)
{
    constexpr uint32_t G = 16 / TW;
    return a.tiled ? 16 * ((tile % G) * TW + blk) + tile / G : tile * TW + blk;
}

template <int PRO, int TW, class A>
__device__ __forceinline__ void fwd_col_body(const NttArgs &a, const LimbPos &lp, const Prime &P, const A &ar,
                                             uint64_t *lds, uint32_t tile, uint32_t tx)
{
    const uint32_t col = tx & (TW - 1), s = tx / TW, c = tile * TW + col;
    const uint64_t *src = a.src + (int64_t)lp.poly * a.map.src_poly_stride + (size_t)lp.row * 65536;
    typename A::W wa[7], wb[7], wc[6];
    typename A::V v[8];
    if (PRO == PRO_BCONV) {  // the twiddles after the conversion: not live across its loop
        bconv_load(v, ar, bc_source(a, lp.poly, lp.prime), P, 65536,
                   [&](int i) { return pos_wide(s, i) * 256 + c; });
        tw_fwd<3, 256, 32>(wa, s, ar, 1);
    } else {
        tw_fwd<3, 256, 32>(wa, s, ar, 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = load_fwd<PRO>(a, lp, ar, src, pos_wide(s, i) * 256 + c, P);
    }
    fwd_rw<3>(v, wa, ar);
    tw_fwd<3, 256, 4>(wb, pos_mid(s, 0), ar, 1);  // in flight across the exchange
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[col_slot<TW>(pos_wide(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[col_slot<TW>(pos_mid(s, i), col)]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wb, ar);
    tw_fwd<2, 256, 1>(wc, 8 * s, ar, 1);
    tw_fwd<2, 256, 1>(wc + 3, 8 * s + 4, ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[col_slot<TW>(pos_mid(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[col_slot<TW>(pos_narrow(s, i), col)]);
    ar.reduce_all(v);
    fwd_rw<2>(v, wc, ar);
    fwd_rw<2>(v + 4, wc + 3, ar);
    uint64_t *m = a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536;
#pragma unroll
    for (int i = 0; i < 8; ++i) m[pos_narrow(s, i) * 256 + c] = ar.to_bits(v[i]);
}

template <int PRO, int TW = 16>
__device__ __forceinline__ void fwd_col_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                             uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        fwd_col_body<PRO, TW>(a, lp, P, fp_arith(a, P, lp.prime, 65536), lds, tile, tx);
    else
        fwd_col_body<PRO, TW>(a, lp, P, int_arith(a, P, lp.prime, 65536), lds, tile, tx);
}

template <int EPI, int TW, class A>
__device__ __forceinline__ void fwd_row_body(const NttArgs &a, const LimbPos &lp, const Prime &P, const A &ar,
                                             uint64_t *lds, uint32_t tile, uint32_t tx)
{
    const uint32_t blk = tx >> 5, s = tx & 31, b = pass_row<TW>(a, tile, blk);
    const MidRow m = mid_row<32>(a, a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536, b, s);
    uint64_t *L = lds + blk * 256;
    typename A::W wa[7], wb[7], wc[6];
    tw_fwd<3, 256, 32, A, true>(wa, s, ar, 256 + b);
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(m.p[i * m.step]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wa, ar);
    tw_fwd<3, 256, 4, A, true>(wb, pos_mid(s, 0), ar, 256 + b);  // in flight across the exchange
#pragma unroll
    for (int i = 0; i < 8; ++i) L[row_slot(pos_wide(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(L[row_slot(pos_mid(s, i))]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wb, ar);
    // the epilogue's operands are loaded here, so their latency overlaps the last round: the
    // subtrahend row (ModDown, Rescale) and the addend (ModDown; block b's addend under X -> X^g
    // comes from one block sb and is permuted through LDS at the end)
    uint64_t auxv[8], addv[8];
    const uint64_t *add = EPI == EPI_MODDOWN ? pick(a.add, lp.poly) : nullptr;
    uint32_t sb = b * 256;
#pragma unroll
    for (int i = 0; i < 8; ++i) auxv[i] = addv[i] = 0;
    if (EPI != EPI_PLAIN) {
        const uint64_t *ax = pick(a.aux, lp.poly) + (size_t)lp.row * 65536 + b * 256;
#pragma unroll
        for (int i = 0; i < 8; ++i) auxv[i] = ax[pos_wide(s, i)];
    }
    if (add) {
        add += (size_t)lp.row * 65536;
        if (a.galois != 1) sb = galois_src(b * 256, a.galois, 16) & ~255u;
#pragma unroll
        for (int i = 0; i < 8; ++i) addv[i] = add[sb + pos_wide(s, i)];
    }
    tw_fwd<2, 256, 1, A, true>(wc, 8 * s, ar, 256 + b);
    tw_fwd<2, 256, 1, A, true>(wc + 3, 8 * s + 4, ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 8; ++i) L[row_slot(pos_mid(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(L[row_slot(pos_narrow(s, i))]);
    ar.reduce_all(v);
    fwd_rw<2>(v, wc, ar);
    fwd_rw<2>(v + 4, wc + 3, ar);
#pragma unroll
    for (int i = 0; i < 8; ++i) L[row_slot(pos_narrow(s, i))] = fwd_out<EPI>(ar, v[i]);
    wave_sync();
    uint64_t x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = L[row_slot(pos_wide(s, i))];
    if (add && a.galois != 1) {
        wave_sync();
#pragma unroll
        for (int i = 0; i < 8; ++i) L[row_slot(pos_wide(s, i))] = addv[i];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 8; ++i) addv[i] = L[row_slot(galois_src(b * 256 + pos_wide(s, i), a.galois, 16) - sb)];
    }
    uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + (size_t)lp.row * 65536;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        store_fwd<EPI>(a, lp, ar, dst, b * 256 + pos_wide(s, i), x[i], addv[i], auxv[i], 65536);
}

template <int EPI, int TW = 16>
__device__ __forceinline__ void fwd_row_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                             uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        fwd_row_body<EPI, TW>(a, lp, P, fp_arith(a, P, lp.prime, 65536), lds, tile, tx);
    else
        fwd_row_body<EPI, TW>(a, lp, P, int_arith(a, P, lp.prime, 65536), lds, tile, tx);
}

// The rounds of row b from the narrow layout on, output m (mid_row<32>); wa: the first round's
// twiddles, L the row's scratch.
template <class A>
__device__ __forceinline__ void inv_row_rounds(const A &ar, typename A::V (&v)[8], const typename A::W (&wa)[6],
                                               uint64_t *L, uint32_t s, uint32_t b, MidRow m)
{
    typename A::W wb[7], wc[7];
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    inv_rw<2>(v + 4, wa + 3, ar);
    tw_inv<3, 256, 4, A, true>(wb, pos_mid(s, 0), ar, 256 + b);  // in flight across the exchange
#pragma unroll
    for (int i = 0; i < 8; ++i) L[row_slot(pos_narrow(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(L[row_slot(pos_mid(s, i))]);
    ar.reduce_all(v);
    inv_rw<3>(v, wb, ar);
    tw_inv<3, 256, 32, A, true>(wc, s, ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 8; ++i) L[row_slot(pos_mid(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(L[row_slot(pos_wide(s, i))]);
    ar.reduce_all(v);
    inv_rw<3>(v, wc, ar);
#pragma unroll
    for (int i = 0; i < 8; ++i) m.p[i * m.step] = ar.to_bits(v[i]);
}

template <int PRO, int TW, class A>
__device__ __forceinline__ void inv_row_body(const NttArgs &a, const LimbPos &lp, const Prime &P, const A &ar,
                                             uint64_t *lds, uint32_t tile, uint32_t tx)
{
    const uint32_t blk = tx >> 5, s = tx & 31, b = pass_row<TW>(a, tile, blk);
    const size_t row_off = (int64_t)lp.poly * a.map.src_poly_stride + (size_t)lp.row * 65536;
    const uint64_t *src = a.src + row_off;
    uint64_t *L = lds + blk * 256;
    typename A::W wa[6];
    tw_inv<2, 256, 1, A, true>(wa, 8 * s, ar, 256 + b);
    tw_inv<2, 256, 1, A, true>(wa + 3, 8 * s + 4, ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t e = b * 256 + pos_wide(s, i);
        if (PRO == PRO_TENSOR)  // HMult's d2 = a1 b1, formed on the fly in the limb's arithmetic
            L[row_slot(pos_wide(s, i))] = ar.to_bits(ar.product(src[e], a.src2[row_off + e], P));
        else
            L[row_slot(pos_wide(s, i))] = src[PRO == PRO_GALOIS ? galois_src(e, a.galois, 16) : e];
    }
    wave_sync();
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
        v[i] = PRO == PRO_TENSOR ? ar.from_bits(L[row_slot(pos_narrow(s, i))]) : ar.from_u64(L[row_slot(pos_narrow(s, i))]);
    inv_row_rounds(ar, v, wa, L, s, b,
                   mid_row<32>(a, a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536, b, s));
}

template <int PRO, int TW = 16>
__device__ __forceinline__ void inv_row_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                             uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv_row_body<PRO, TW>(a, lp, P, fp_arith(a, P, lp.prime, 65536), lds, tile, tx);
    else
        inv_row_body<PRO, TW>(a, lp, P, int_arith(a, P, lp.prime, 65536), lds, tile, tx);
}

template <int TW, class A>
__device__ __forceinline__ void inv_col_body(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *lds,
                                             uint32_t tile, uint32_t tx)
{
    const uint32_t col = tx & (TW - 1), s = tx / TW, c = tile * TW + col;
    const uint64_t *m = a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536;
    typename A::W wa[6], wb[7], wc[7];
    tw_inv<2, 256, 1>(wa, 8 * s, ar, 1);
    tw_inv<2, 256, 1>(wa + 3, 8 * s + 4, ar, 1);
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(m[pos_narrow(s, i) * 256 + c]);
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    inv_rw<2>(v + 4, wa + 3, ar);
    tw_inv<3, 256, 4>(wb, pos_mid(s, 0), ar, 1);  // in flight across the exchange
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[col_slot<TW>(pos_narrow(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[col_slot<TW>(pos_mid(s, i), col)]);
    ar.reduce_all(v);
    inv_rw<3>(v, wb, ar);
    tw_inv<3, 256, 32>(wc, s, ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[col_slot<TW>(pos_mid(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[col_slot<TW>(pos_wide(s, i), col)]);
    ar.reduce_all(v);
    inv_rw<3>(v, wc, ar);
    uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + (size_t)lp.row * 65536;
    inv_store(dst, v, ar, a.ys_mode, [&](int i) { return pos_wide(s, i) * 256 + c; });
}

template <int TW = 16>
__device__ __forceinline__ void inv_col_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                             uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv_col_body<TW>(a, lp, inv_fp_arith(a, lp, P, 65536), lds, tile, tx);
    else
        inv_col_body<TW>(a, lp, inv_int_arith(a, lp, P, 65536), lds, tile, tx);
}

// Inverse passes with 4 elements per thread, 64 threads per 256-point problem,
// for launches over few limbs: those are latency-bound with one wave per SIMD
// in the 8-element layout, and this one gives them twice the waves.  A
// workgroup of 512 threads takes 8 rows (one wave each) or 8 columns.  Rounds
// of two stages (t = 1, 2 | 4, 8 | 16, 32 | 64, 128) in four layouts, thread
// s < 64 holding positions
//   A 4s + i,  B 16 (s/4) + s%4 + 4i,  C 64 (s/16) + s%16 + 16i,  D s + 64i.
__device__ __forceinline__ uint32_t p4a(uint32_t s, int i) { return 4 * s + i; }
__device__ __forceinline__ uint32_t p4b(uint32_t s, int i) { return 16 * (s >> 2) + (s & 3) + 4 * i; }
__device__ __forceinline__ uint32_t p4c(uint32_t s, int i) { return 64 * (s >> 4) + (s & 15) + 16 * i; }
__device__ __forceinline__ uint32_t p4d(uint32_t s, int i) { return s + 64 * i; }
// LDS slot of element e of a row (256 words): the low five bits XOR-ed with
// 9 (e/32) and 4 (e/64) (mod 32), so that each half-wave hits 32 distinct
// 8-byte banks in all four layouts (checked exhaustively on the host).
__device__ __forceinline__ uint32_t row4_slot(uint32_t e)
{
    return (e & ~31u) | ((e ^ (9 * (e >> 5)) ^ (4 * (e >> 6))) & 31u);
}
// LDS slot of element e of column `col` of an 8-column tile: columns
// interleaved, one word of padding every 4 elements (conflict-free likewise).
__device__ __forceinline__ uint32_t col4_slot(uint32_t e, uint32_t col) { return 8 * (e + (e >> 2)) + col; }
constexpr int kLds4 = 8 * (255 + 63 + 1);

// The rounds of one row: thread s < 64 of the row's wave, values
// value(i) at position p4a(s, i), scratch L (256 words), output m (mid_row<64>).
template <class A, class Value>
__device__ __forceinline__ void inv_row4_values(const A &ar, uint64_t *L, uint32_t s, uint32_t b, Value value, MidRow m)
{
    typename A::W wa[3], wb[3];
    typename A::V v[4];
    tw_inv<2, 256, 1, A, true>(wa, p4a(s, 0), ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = value(i);
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    tw_inv<2, 256, 4, A, true>(wb, p4b(s, 0), ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4a(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4b(s, i))]);
    ar.reduce_all(v);
    inv_rw<2>(v, wb, ar);
    tw_inv<2, 256, 16, A, true>(wa, p4c(s, 0), ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4b(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4c(s, i))]);
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    tw_inv<2, 256, 64, A, true>(wb, p4d(s, 0), ar, 256 + b);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4c(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4d(s, i))]);
    ar.reduce_all(v);
    inv_rw<2>(v, wb, ar);
#pragma unroll
    for (int i = 0; i < 4; ++i) m.p[i * m.step] = ar.to_bits(v[i]);
}

template <class A, class Load>
__device__ __forceinline__ void inv_row4_rounds(const A &ar, uint64_t *L, uint32_t s, uint32_t b, Load load, MidRow m)
{
    inv_row4_values(ar, L, s, b, [&](int i) { return ar.from_u64(load(i)); }, m);
}

template <class A>
__device__ __forceinline__ void inv_row4_body(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *lds,
                                              uint32_t tile, uint32_t tx)
{
    const uint32_t blk = tx >> 6, s = tx & 63, b = pass_row<8>(a, tile, blk);
    const uint64_t *src = a.src + (int64_t)lp.poly * a.map.src_poly_stride + (size_t)lp.row * 65536 + b * 256;
    const MidRow m = mid_row<64>(a, a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536, b, s);
    inv_row4_rounds(ar, lds + blk * 256, s, b, [&](int i) { return src[p4a(s, i)]; }, m);
}

template <class A>
__device__ __forceinline__ void inv_col4_body(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *lds,
                                              uint32_t tile, uint32_t tx)
{
    const uint32_t col = tx & 7, s = tx >> 3, c = tile * 8 + col;
    const uint64_t *m = a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 65536;
    typename A::W wa[3], wb[3];
    typename A::V v[4];
    tw_inv<2, 256, 1>(wa, p4a(s, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(m[p4a(s, i) * 256 + c]);
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    tw_inv<2, 256, 4>(wb, p4b(s, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[col4_slot(p4a(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(lds[col4_slot(p4b(s, i), col)]);
    ar.reduce_all(v);
    inv_rw<2>(v, wb, ar);
    tw_inv<2, 256, 16>(wa, p4c(s, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[col4_slot(p4b(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(lds[col4_slot(p4c(s, i), col)]);
    ar.reduce_all(v);
    inv_rw<2>(v, wa, ar);
    tw_inv<2, 256, 64>(wb, p4d(s, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds[col4_slot(p4c(s, i), col)] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(lds[col4_slot(p4d(s, i), col)]);
    ar.reduce_all(v);
    inv_rw<2>(v, wb, ar);
    uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + (size_t)lp.row * 65536;
    inv_store(dst, v, ar, a.ys_mode, [&](int i) { return p4d(s, i) * 256 + c; });
}

__device__ __forceinline__ void inv_row4_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                              uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv_row4_body(a, lp, fp_arith(a, P, lp.prime, 65536), lds, tile, tx);
    else
        inv_row4_body(a, lp, int_arith(a, P, lp.prime, 65536), lds, tile, tx);
}

__device__ __forceinline__ void inv_col4_unit(const NttArgs &a, uint32_t limb, uint32_t tile, uint64_t *lds,
                                              uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv_col4_body(a, lp, inv_fp_arith(a, lp, P, 65536), lds, tile, tx);
    else
        inv_col4_body(a, lp, inv_int_arith(a, lp, P, 65536), lds, tile, tx);
}

// ------------------------------------------------------------------ N = 2^12
// One workgroup of 512 threads per limb, 8 elements per thread, four rounds of
// three stages in the layouts
//   0: t + 512 i,  1: 512 (t/64) + t%64 + 64 i,  2: 64 (t/8) + t%8 + 8 i,  3: 8 t + i.
// Layouts 1, 2 and 3 of a wave cover the same 512 elements, so only the exchange
// with layout 0 takes a workgroup barrier; layout 3 reads and writes 64
// consecutive bytes per thread.  A launch has as many workgroups as limbs, far
// fewer than CUs, so a limb's own time is all that counts: two waves per SIMD
// with four independent butterflies each, and the twiddles of a round loaded
// before the exchange that precedes it.  (256 threads with 16 elements, one
// wave per SIMD and three rounds with a barrier each: 9.3 us for the four limbs
// of the small set, 7.7 us this way.)
constexpr int kThreads12 = 512;
constexpr int kLds12 = 4096;

__device__ __forceinline__ uint32_t p12a(uint32_t t, int i) { return t + 512 * i; }
__device__ __forceinline__ uint32_t p12b(uint32_t t, int i) { return 512 * (t >> 6) + (t & 63) + 64 * i; }
__device__ __forceinline__ uint32_t p12c(uint32_t t, int i) { return 64 * (t >> 3) + (t & 7) + 8 * i; }
__device__ __forceinline__ uint32_t p12d(uint32_t t, int i) { return 8 * t + i; }

// LDS slot of element e: its low five bits XOR-ed with bits 5 to 7, so that
// each half-wave hits 32 distinct 8-byte banks in all four layouts (bits 3, 4
// identify a thread's group in layout 3, bits 6, 7 in layout 2).
__device__ __forceinline__ uint32_t slot12(uint32_t e)
{
    const uint32_t h = (e >> 5) & 7;
    return e ^ h ^ ((h >> 1) << 3);
}

template <int PRO, int EPI, class A>
__device__ __forceinline__ void fwd12_body(const NttArgs &a, const LimbPos &lp, const Prime &P, const A &ar,
                                           uint64_t *lds, uint32_t t)
{
    const size_t off = (size_t)lp.row * 4096;
    typename A::W wa[7], wb[7];
    typename A::V v[8], aux[8];
    tw_fwd<3, 4096, 512>(wa, 0, ar, 1);
    if (PRO == PRO_BCONV) {
        bconv_load(v, ar, bc_source(a, lp.poly, lp.prime), P, 4096, [&](int i) { return p12a(t, i); });
    } else {
        const uint64_t *src = a.src + (int64_t)lp.poly * a.map.src_poly_stride + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = load_fwd<PRO>(a, lp, ar, src, p12a(t, i), P);
    }
    fwd_rw<3>(v, wa, ar);
    tw_fwd<3, 4096, 64>(wb, p12b(t, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12a(t, i))] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12b(t, i))]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wb, ar);
    tw_fwd<3, 4096, 8>(wa, p12c(t, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12b(t, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12c(t, i))]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wa, ar);
    // the epilogue's operands, in flight across the last round
    uint64_t addv[8];
    const uint64_t *add = EPI == EPI_MODDOWN ? pick(a.add, lp.poly) : nullptr;
#pragma unroll
    for (int i = 0; i < 8; ++i) addv[i] = 0;
    if (EPI != EPI_PLAIN) {
        const uint64_t *ax = pick(a.aux, lp.poly) + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) aux[i] = ar.from_u64(ax[p12d(t, i)]);
    }
    if (add) {
        add += off;
#pragma unroll
        for (int i = 0; i < 8; ++i) addv[i] = add[a.galois == 1 ? p12d(t, i) : galois_src(p12d(t, i), a.galois, 12)];
    }
    tw_fwd<3, 4096, 1>(wb, 8 * t, ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12c(t, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12d(t, i))]);
    ar.reduce_all(v);
    fwd_rw<3>(v, wb, ar);
    if (EPI == EPI_PLAIN) {
        uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) dst[p12d(t, i)] = ar.fwd_final(v[i]);
    } else {
        const ulonglong2 c = a.cst[lp.prime];
        uint64_t *out = pick(a.out, lp.poly) + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) out[p12d(t, i)] = ar.scaled_difference(v[i], aux[i], addv[i], c);
    }
}

template <int PRO, int EPI>
__device__ __forceinline__ void fwd12_unit(const NttArgs &a, uint32_t limb, uint32_t, uint64_t *lds, uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        fwd12_body<PRO, EPI>(a, lp, P, fp_arith(a, P, lp.prime, 4096), lds, tx);
    else
        fwd12_body<PRO, EPI>(a, lp, P, int_arith(a, P, lp.prime, 4096), lds, tx);
}

template <int PRO, class A>
__device__ __forceinline__ void inv12_body(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *lds, uint32_t t)
{
    const uint64_t *src = a.src + (int64_t)lp.poly * a.map.src_poly_stride + (size_t)lp.row * 4096;
    typename A::W wa[7], wb[7];
    typename A::V v[8];
    tw_inv<3, 4096, 1>(wa, 8 * t, ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        v[i] = ar.from_u64(src[PRO == PRO_GALOIS ? galois_src(p12d(t, i), a.galois, 12) : p12d(t, i)]);
    ar.reduce_all(v);
    inv_rw<3>(v, wa, ar);
    tw_inv<3, 4096, 8>(wb, p12c(t, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12d(t, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12c(t, i))]);
    ar.reduce_all(v);
    inv_rw<3>(v, wb, ar);
    tw_inv<3, 4096, 64>(wa, p12b(t, 0), ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12c(t, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12b(t, i))]);
    ar.reduce_all(v);
    inv_rw<3>(v, wa, ar);
    tw_inv<3, 4096, 512>(wb, 0, ar, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) lds[slot12(p12b(t, i))] = ar.to_bits(v[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(lds[slot12(p12a(t, i))]);
    ar.reduce_all(v);
    inv_rw<3>(v, wb, ar);
    uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + (size_t)lp.row * 4096;
    inv_store(dst, v, ar, a.ys_mode, [&](int i) { return p12a(t, i); });
}

template <int PRO>
__device__ __forceinline__ void inv12_unit(const NttArgs &a, uint32_t limb, uint32_t, uint64_t *lds, uint32_t tx)
{
    const LimbPos lp = limb_pos(a.map, limb);
    if (lp.skip) return;
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv12_body<PRO>(a, lp, inv_fp_arith(a, lp, P, 4096), lds, tx);
    else
        inv12_body<PRO>(a, lp, inv_int_arith(a, lp, P, 4096), lds, tx);
}

// ------------------------------------- N = 2^12, transforms in two launches
// The single key switch, ModDown and Rescale at N = 2^12 are latency-bound: a
// whole limb per workgroup (above) leaves most CUs idle and takes 7 to 20 us
// on one of them.  Here a limb is a 64 x 64 matrix and a wave owns 8 columns
// (or 8 rows) of it, 8 elements per lane, two rounds of three stages with one
// exchange inside the wave.  What is local to columns shares a launch, and so
// does what is local to rows:
//   inverse rows | inverse columns, conversion, forward columns |
//   forward rows, inner product, inverse rows of the special rows |
//   inverse columns, conversion, forward columns | forward rows, P^-1 (x - .) + add
// (Rescale: inverse rows | inverse columns, lift, forward columns | forward
// rows, q_l^-1 (x - .)).  HMult of the small set (four limbs) went from 58 us
// in seven launches to 32 us in these five, a rotation at K = 2 from 62 to 28 us.
// Lane layouts (s = 0..7 along the 64-point problem): A: s + 8 i, B: 8 s + i.
// Columns: col = lane % 8, s = lane / 8, element e = 8 row + col of the tile;
// rows: row = lane / 8, s = lane % 8, e = 64 row + position.  slot12 keeps the
// exchanges conflict-free in all of them.
constexpr uint32_t kTile12 = 512;  // elements of a wave's tile

// exchange of a wave's tile: v[i] at element from(i) becomes the one at to(i)
template <class A, class From, class To>
__device__ __forceinline__ void exchange12(const A &ar, typename A::V (&v)[8], uint64_t *L, From from, To to)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) L[slot12(from(i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(L[slot12(to(i))]);
    ar.reduce_all(v);
}

// 64-point transforms over layout s; e(p) is the tile element of position p of
// the lane's problem, B the twiddle block (1 for columns, 64 + row for rows).
// Forward A -> B, inverse B -> A; the caller has centred the inverse's input.
template <class A, class E>
__device__ __forceinline__ void fwd64(const A &ar, typename A::V (&v)[8], uint64_t *L, uint32_t s, uint32_t B, E e)
{
    typename A::W wa[7], wb[7];
    tw_fwd<3, 64, 8>(wa, s, ar, B);
    tw_fwd<3, 64, 1>(wb, 8 * s, ar, B);
    fwd_rw<3>(v, wa, ar);
    exchange12(ar, v, L, [&](int i) { return e(s + 8 * i); }, [&](int i) { return e(8 * s + i); });
    fwd_rw<3>(v, wb, ar);
}

template <class A, class E>
__device__ __forceinline__ void inv64(const A &ar, typename A::V (&v)[8], uint64_t *L, uint32_t s, uint32_t B, E e)
{
    typename A::W wa[7], wb[7];
    tw_inv<3, 64, 1>(wb, 8 * s, ar, B);
    tw_inv<3, 64, 8>(wa, s, ar, B);
    inv_rw<3>(v, wb, ar);
    exchange12(ar, v, L, [&](int i) { return e(8 * s + i); }, [&](int i) { return e(s + 8 * i); });
    inv_rw<3>(v, wa, ar);
}

// First inverse pass of 8 rows (tile) of a limb's evaluations src (gathered
// through X -> X^g, or times src2: HMult's d2 = a1 b1), in layout A.
template <int PRO, class A>
__device__ __forceinline__ void inv_row_tile12(typename A::V (&v)[8], const A &ar, const Prime &P, const uint64_t *src,
                                               const uint64_t *src2, uint32_t g, uint64_t *L, uint32_t tile,
                                               uint32_t lane)
{
    const uint32_t row = lane >> 3, s = lane & 7, e0 = tile * kTile12 + 64 * row + 8 * s;
    uint64_t x[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = src[PRO == PRO_GALOIS ? galois_src(e0 + i, g, 12) : e0 + i];
    if (PRO == PRO_TENSOR) {
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = src2[e0 + i];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = PRO == PRO_TENSOR ? ar.product(x[i], y[i], P) : ar.from_u64(x[i]);
    ar.reduce_all(v);
    inv64(ar, v, L, s, 64 + 8 * tile + row, [&](uint32_t p) { return 64 * row + p; });
}

// Inverse rows: 8 rows of a limb from its evaluations to a.mid.
template <int PRO, class A>
__device__ __forceinline__ void inv_rows12(const NttArgs &a, const LimbPos &lp, const Prime &P, const A &ar, uint64_t *L,
                                           uint32_t tile, uint32_t lane)
{
    const size_t row_off = (int64_t)lp.poly * a.map.src_poly_stride + (size_t)lp.row * 4096;
    typename A::V v[8];
    inv_row_tile12<PRO>(v, ar, P, a.src + row_off, PRO == PRO_TENSOR ? a.src2 + row_off : nullptr, a.galois, L, tile, lane);
    const uint32_t row = lane >> 3, s = lane & 7;
    uint64_t *m = a.mid + (int64_t)lp.poly * a.mid_stride + (size_t)lp.row * 4096 + tile * kTile12;
#pragma unroll
    for (int i = 0; i < 8; ++i) m[64 * row + s + 8 * i] = ar.to_bits(v[i]);
}

template <int PRO>
__global__ __launch_bounds__(64) void k12_inv_rows(NttArgs a)
{
    __shared__ uint64_t L[kTile12];
    const LimbPos lp = limb_pos(a.map, blockIdx.y);
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        inv_rows12<PRO>(a, lp, P, fp_arith(a, P, lp.prime, 4096), L, blockIdx.x, threadIdx.x);
    else
        inv_rows12<PRO>(a, lp, P, int_arith(a, P, lp.prime, 4096), L, blockIdx.x, threadIdx.x);
}

// Forward rows: 8 rows of a limb from a.mid to its evaluations, with the epilogue.
template <int EPI, class A>
__device__ __forceinline__ void fwd_rows12(const NttArgs &a, const LimbPos &lp, const A &ar, uint64_t *L, uint32_t tile,
                                           uint32_t lane)
{
    const uint32_t row = lane >> 3, s = lane & 7, e0 = tile * kTile12 + 64 * row + 8 * s;
    const size_t off = (size_t)lp.row * 4096;
    const uint64_t *m = a.mid + (int64_t)lp.poly * a.mid_stride + off + tile * kTile12;
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(m[64 * row + s + 8 * i]);
    // the epilogue's operands, in flight across the rounds
    uint64_t auxv[8], addv[8];
    const uint64_t *add = EPI == EPI_MODDOWN ? pick(a.add, lp.poly) : nullptr;
#pragma unroll
    for (int i = 0; i < 8; ++i) auxv[i] = EPI != EPI_PLAIN ? pick(a.aux, lp.poly)[off + e0 + i] : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        addv[i] = add ? add[off + (a.galois == 1 ? e0 + i : galois_src(e0 + i, a.galois, 12))] : 0;
    ar.reduce_all(v);
    fwd64(ar, v, L, s, 64 + 8 * tile + row, [&](uint32_t p) { return 64 * row + p; });
    if (EPI == EPI_PLAIN) {
        uint64_t *dst = a.dst + (int64_t)lp.poly * a.map.dst_poly_stride + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) dst[e0 + i] = ar.fwd_final(v[i]);
    } else {
        const ulonglong2 c = a.cst[lp.prime];
        uint64_t *out = pick(a.out, lp.poly) + off;
#pragma unroll
        for (int i = 0; i < 8; ++i) out[e0 + i] = ar.scaled_difference(v[i], ar.from_u64(auxv[i]), addv[i], c);
    }
}

template <int EPI>
__global__ __launch_bounds__(64) void k12_fwd_rows(NttArgs a)
{
    __shared__ uint64_t L[kTile12];
    const LimbPos lp = limb_pos(a.map, blockIdx.y);
    const Prime P = a.primes[lp.prime];
    if (P.q < kFpMaxPrime)
        fwd_rows12<EPI>(a, lp, fp_arith(a, P, lp.prime, 4096), L, blockIdx.x, threadIdx.x);
    else
        fwd_rows12<EPI>(a, lp, int_arith(a, P, lp.prime, 4096), L, blockIdx.x, threadIdx.x);
}

// inv_store's mode for a conversion's sources (Rescale lifts plain coefficients)
template <int MODE>
constexpr uint32_t kSourceMode = MODE == COLS_MODDOWN ? 2 : MODE == COLS_MODUP ? 1 : 0;

// Second inverse pass of a source row's 8 columns, scaled: canonical inputs of
// the conversion (shifted for ModDown) to the tile y, element lane + 64 i.  The
// first pass's output comes from m, or (ROWS) is in y already, element 8 row + col.
template <int MODE, bool ROWS, class A>
__device__ __forceinline__ void source_cols12(const A &ar, const uint64_t *m, uint64_t *y, uint32_t tile, uint32_t lane)
{
    const uint32_t col = lane & 7, s = lane >> 3, c = 8 * tile + col;
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = ar.from_bits(ROWS ? y[8 * (8 * s + i) + col] : m[64 * (8 * s + i) + c]);
    if (ROWS) wave_sync();  // read before the exchange reuses the tile
    ar.reduce_all(v);
    inv64(ar, v, y, s, 1, [&](uint32_t p) { return 8 * p + col; });
    wave_sync();  // the exchange's reads are done: the tile takes the result
    inv_store(y, v, ar, kSourceMode<MODE>, [&](int i) { return lane + 64 * i; });
}

// First inverse pass of a source row by one of the workgroup's waves (its row
// tile `rows`), of which the column tile keeps 8 columns: col + 8 i, i = tile.
template <int PRO, class A>
__device__ __forceinline__ void source_rows12(const ColsArgs &a, const A &ar, const Prime &P, const uint64_t *src,
                                              const uint64_t *src2, uint64_t *L, uint64_t *y, uint32_t tile,
                                              uint32_t rows, uint32_t lane)
{
    typename A::V v[8];
    inv_row_tile12<PRO>(v, ar, P, src, src2, a.galois, L, rows, lane);
    typename A::V x = v[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) x = (uint32_t)i == tile ? v[i] : x;
    y[8 * (8 * rows + (lane >> 3)) + (lane & 7)] = ar.to_bits(x);
    wave_sync();  // the next source's exchange reuses L
}

// v[i] = Conv(y)[lane + 64 i] from the source tiles in LDS.
template <class Acc, class A>
__device__ __forceinline__ void conv12_acc(typename A::V (&v)[8], const A &ar, const uint64_t *y, uint32_t ns,
                                           ConvWord *h, const Prime &P, uint32_t lane)
{
    Acc acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i].start(h);
    for (uint32_t k = 0; k < ns; ++k) {
        uint64_t x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = y[k * kTile12 + lane + 64 * i];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i].add(x[i], h, k);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = acc[i].value(ar, h, P);
}
__device__ __forceinline__ void conv12(double (&v)[8], const FpArith &ar, const uint64_t *y, uint32_t ns, ConvWord *h,
                                       const Prime &P, uint32_t lane)
{
    if (ns <= kFoldMaxTerms)
        conv12_acc<FoldAcc>(v, ar, y, ns, h, P, lane);
    else
        conv12_acc<WideAcc<MacSplit>>(v, ar, y, ns, h, P, lane);
}
__device__ __forceinline__ void conv12(uint64_t (&v)[8], const IntArith &ar, const uint64_t *y, uint32_t ns, ConvWord *h,
                                       const Prime &P, uint32_t lane)
{
    if (h[kConvStart])
        conv12_acc<FoldWideAcc>(v, ar, y, ns, h, P, lane);
    else
        conv12_acc<WideAcc<MacColsAcc>>(v, ar, y, ns, h, P, lane);
}

// First forward pass of a target row's 8 columns, converted from the sources.
template <int MODE, class A>
__device__ __forceinline__ void target_cols12(const A &ar, const Prime &P, const uint64_t *y, uint32_t ns, ConvWord *h,
                                              uint64_t qlmod, uint64_t ql, uint64_t *L, uint64_t *m, uint32_t tile,
                                              uint32_t lane)
{
    const uint32_t col = lane & 7, s = lane >> 3, c = 8 * tile + col;
    typename A::V v[8];
    if (MODE == COLS_RESCALE) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = ar.lift(y[lane + 64 * i], ql, qlmod, P);
    } else {
        conv12(v, ar, y, ns, h, P, lane);
    }
    fwd64(ar, v, L, s, 1, [&](uint32_t p) { return 8 * p + col; });
#pragma unroll
    for (int i = 0; i < 8; ++i) m[64 * (8 * s + i) + c] = ar.to_bits(v[i]);
}

// A workgroup of 8 waves: a job's sources for one tile (each wave a row, two
// when there are more than eight), then one target row per wave.  A job with
// more than eight targets takes several workgroups, which all form the sources:
// that costs no time, since they do it side by side.  With PRO the sources are
// evaluations and the workgroup runs their first inverse pass as well, a row tile
// per wave: no launch for it, but ns passes one after another in each of the
// workgroups, so only for few sources.
constexpr uint32_t kColsWaves = 8;

template <int MODE, int PRO>
__global__ __launch_bounds__(64 * kColsWaves) void k12_cols(ColsArgs a)
{
    constexpr bool kRows = PRO != PRO_MID;
    extern __shared__ uint64_t lds12[];  // ns source tiles, then a tile per wave
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t tile = blockIdx.x, job = blockIdx.y, n = a.level + 1;
    uint32_t lo = 0, ns = 1, set = a.pset, prime0 = a.level, ntgt = a.level;
    if (MODE == COLS_MODUP) {
        lo = job * a.alpha;
        ns = min(a.alpha, n - lo);
        set = job * a.alpha + ns - 1;
        prime0 = lo;
        ntgt = n + a.np - ns;
    } else if (MODE == COLS_MODDOWN) {
        ns = a.np;
        prime0 = a.nq;
        ntgt = n;
    }
    const int64_t src_off = MODE == COLS_MODUP ? (int64_t)lo * 4096 : (int64_t)job * a.src_stride;
    const uint64_t *src = a.src + src_off;
    if (kRows) {
        uint64_t *L = lds12 + (ns + w) * kTile12;
        for (uint32_t k = 0; k < ns; ++k) {
            const uint32_t pi = prime0 + k;
            const Prime P = a.primes[pi];
            const uint64_t *x = src + (size_t)k * 4096, *x2 = PRO == PRO_TENSOR ? a.src2 + src_off + (size_t)k * 4096 : nullptr;
            if (P.q < kFpMaxPrime)
                source_rows12<PRO>(a, fp_arith(a.twdi, P, pi, 4096), P, x, x2, L, lds12 + k * kTile12, tile, w, lane);
            else
                source_rows12<PRO>(a, int_arith(a.twi, P, pi, 4096), P, x, x2, L, lds12 + k * kTile12, tile, w, lane);
        }
        __syncthreads();
    }
    for (uint32_t k = w; k < ns; k += kColsWaves) {
        const uint32_t pi = prime0 + k;
        const Prime P = a.primes[pi];
        uint64_t *y = lds12 + k * kTile12;
        if (P.q < kFpMaxPrime) {
            FpArith ar = fp_arith(a.twdi, P, pi, 4096);
            if (MODE != COLS_RESCALE) ar.fc = a.ysd[set * kMaxDigitPrimes + k];
            source_cols12<MODE, kRows>(ar, src + (size_t)k * 4096, y, tile, lane);
        } else {
            IntArith ar = int_arith(a.twi, P, pi, 4096);
            if (MODE != COLS_RESCALE) {
                const ulonglong2 f = a.ys[set * kMaxDigitPrimes + k];
                ar.fc = f.x;
                ar.fc_s = f.y;
            }
            source_cols12<MODE, kRows>(ar, src + (size_t)k * 4096, y, tile, lane);
        }
    }
    __syncthreads();
    const uint32_t idx = blockIdx.z * kColsWaves + w;
    if (idx >= ntgt) return;
    const uint32_t r = MODE == COLS_MODUP && idx >= lo ? idx + ns : idx;
    const uint32_t pi = coef::row_prime(r, a.level, a.nq);
    const Prime P = a.primes[pi];
    ConvWord *h = (ConvWord *)(a.hmod + ((size_t)set * (a.nq + a.np) + pi) * kConvRow);
    const uint64_t qlmod = MODE == COLS_RESCALE ? a.rs_qlmod[pi] : 0, ql = MODE == COLS_RESCALE ? a.primes[a.level].q : 0;
    uint64_t *L = lds12 + (ns + w) * kTile12, *m = a.dst + (int64_t)job * a.dst_stride + (size_t)r * 4096;
    if (P.q < kFpMaxPrime)
        target_cols12<MODE>(fp_arith(a.twdf, P, pi, 4096), P, lds12, ns, h, qlmod, ql, L, m, tile, lane);
    else
        target_cols12<MODE>(int_arith(a.twf, P, pi, 4096), P, lds12, ns, h, qlmod, ql, L, m, tile, lane);
}

// Half `half` of the inner product of extended row r on 8 rows of its matrix
// (layout B: eight consecutive positions per lane): sum_j x_j[r] key[j][half][r],
// x_j the digit's row (READY: finished, gathered through ip.galois; else its
// last forward pass runs here), its own row of ip.own (gathered through
// ip.own_galois) or, with a tensor, the product a1 b1; rows q_0..q_l of a
// tensor also take [P]_q d_half (see IpArgs).  A special row goes on to
// ModDown's first inverse pass.  fwd, inv: the row's two directions.
template <bool READY, class A>
__device__ __forceinline__ void ip_rows12(const IpArgs &ip, const NttArgs &ia, const A &fwd, const A &inv, const Prime &P,
                                          uint32_t half, uint32_t r, uint32_t pi, uint64_t *L, uint32_t tile,
                                          uint32_t lane)
{
    const bool qrow = r <= ip.level;
    const uint32_t row = lane >> 3, s = lane & 7, e0 = tile * kTile12 + 64 * row + 8 * s;
    const size_t krows = ip.nq + ip.np, off = (size_t)r * 4096;
    auto elem = [&](uint32_t p) { return 64 * row + p; };
    typename A::Sum sum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) fwd.sum_start(sum[i]);
    for (uint32_t j = 0; j < ip.beta; ++j) {
        const uint64_t *key = ip.key + (((size_t)j * 2 + half) * krows + pi) * 4096 + e0;
        const bool own = qrow && r >= j * ip.alpha && r < j * ip.alpha + ip.alpha && (ip.own || ip.ta0);
        uint64_t k[8], x[8];
        typename A::V v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) k[i] = key[i];
        if (own && ip.ta0) {
            uint64_t y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = ip.ta1[off + e0 + i], y[i] = ip.tb1[off + e0 + i];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fwd.product(x[i], y[i], P);
        } else if (own || READY) {
            const uint64_t *xr = own ? ip.own + off : ip.ext + ((size_t)j * ip.rows + r) * 4096;
            const uint32_t g = own ? ip.own_galois : ip.galois;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fwd.from_u64(xr[g == 1 ? e0 + i : galois_src(e0 + i, g, 12)]);
        } else {
            const uint64_t *m = ip.ext + ((size_t)j * ip.rows + r) * 4096 + tile * kTile12;
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fwd.from_bits(m[64 * row + s + 8 * i]);
            fwd.reduce_all(v);
            wave_sync();  // the previous digit's exchange is read
            fwd64(fwd, v, L, s, 64 + 8 * tile + row, elem);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fwd.sum_input(v[i]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) fwd.sum_add(sum[i], v[i], k[i]);
        if (j & 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) fwd.sum_centre(sum[i]);
        }
    }
    if (qrow && ip.ta0) {
        const uint64_t pm = ip.pmod[pi];
        uint64_t x[8], y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) fwd.sum_centre(sum[i]);
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = ip.ta0[off + e0 + i], y[i] = (half ? ip.tb1 : ip.tb0)[off + e0 + i];
#pragma unroll
        for (int i = 0; i < 8; ++i) fwd.sum_add(sum[i], fwd.product(x[i], y[i], P), pm);
        if (half) {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = ip.ta1[off + e0 + i], y[i] = ip.tb0[off + e0 + i];
#pragma unroll
            for (int i = 0; i < 8; ++i) fwd.sum_add(sum[i], fwd.product(x[i], y[i], P), pm);
        }
    }
    typename A::V v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fwd.sum_value(sum[i], P);
    if (qrow) {
        uint64_t *acc = ip.acc + ((size_t)half * ip.rows + r) * 4096 + e0;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = fwd.fwd_final(v[i]);
        return;
    }
    wave_sync();
    inv64(inv, v, L, s, 64 + 8 * tile + row, elem);
    uint64_t *m = ia.mid + (int64_t)half * ia.mid_stride + (size_t)(r - ip.level - 1) * 4096 + tile * kTile12;
#pragma unroll
    for (int i = 0; i < 8; ++i) m[64 * row + s + 8 * i] = inv.to_bits(v[i]);
}

template <bool READY>
__global__ __launch_bounds__(64) void k12_ip_rows(IpArgs ip, NttArgs ia, const ulonglong2 *twf, const double *twdf)
{
    __shared__ uint64_t L[kTile12];
    const uint32_t half = blockIdx.z, r = blockIdx.y, pi = coef::row_prime(r, ip.level, ip.nq);
    const Prime P = ip.primes[pi];
    if (P.q < kFpMaxPrime)
        ip_rows12<READY>(ip, ia, fp_arith(twdf, P, pi, 4096), fp_arith(ia.twd, P, pi, 4096), P, half, r, pi, L, blockIdx.x,
                         threadIdx.x);
    else
        ip_rows12<READY>(ip, ia, int_arith(twf, P, pi, 4096), int_arith(ia.tw, P, pi, 4096), P, half, r, pi, L, blockIdx.x,
                         threadIdx.x);
}

// ----------------------------- N = 2^16, the columns of a conversion in one launch
// Between the row passes of a key switch everything is local to a column: the
// second inverse pass of the source rows, the base conversion, the first
// forward pass of the target rows.  A workgroup takes a tile of 4 columns of one
// job (a digit, a polynomial): its waves bring the sources' tiles to scaled
// coefficients in LDS, then each takes target rows, converts and transforms
// them.  A wave works a tile of a row alone, 16 elements per lane in two rounds
// of four stages with one exchange inside the wave.  No scaled coefficient or
// converted row goes through memory, three launches are one, and a wave has
// nothing to wait for but its LDS: the separate passes wrote and read every row
// once more and spent half their time between loads and stores.  ModUp's three
// passes of HMult at l = 30 (digits of 11, 11 and 9, K = 4) took 67 us, this launch 44;
// ModDown's two 38, this 27; Rescale's two at l = 12 17, this 12.  What bounds it
// is the VALU: ModUp's issues 10.4 M wave instructions, 23 us at the card's rate
// for 64-bit multiply-adds, over 192 workgroups of a digit's tile each (a CU
// takes one: LDS), 66 % of the issue slots of the CUs that have one; the rest is
// the wait for the sources and the first loads.  Not kept: two targets per wave
// over each source read from LDS (46 us; LDS does not bound it) and Rescale with
// two workgroups per CU (128 registers spill: 20 us).
// Lane layouts (col = lane % 4, s = lane / 4, element e = 4 row + col): A rows
// s + 16 i, e = lane + 64 i; B rows 16 s + i, stored at 64 i + lane (mid_row).
constexpr uint32_t kTile16 = 1024;
constexpr uint32_t kCols16Waves = 8;

// LDS slot of element e: bits 2 to 4 XOR-ed with bits 6 to 8, so that a half-wave
// hits 32 distinct 8-byte banks in both layouts.
__device__ __forceinline__ uint32_t slot16(uint32_t e) { return e ^ (((e >> 6) & 7) << 2); }

// wb: tw_fwd<4, 256, 1> of the lane, loaded by the caller ahead of the input.
template <class A>
__device__ __forceinline__ void fwd256(const A &ar, typename A::V (&v)[16], const typename A::W (&wb)[15], uint64_t *L,
                                       uint32_t lane)
{
    const uint32_t col = lane & 3, s = lane >> 2;
    typename A::W wa[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) wa[i] = ar.tw_uniform(1 + i);  // tw_fwd<4, 256, 16>: the same for all lanes
    fwd_rw<4>(v, wa, ar);
#pragma unroll
    for (int i = 0; i < 16; ++i) L[slot16(lane + 64 * i)] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = ar.from_bits(L[slot16(64 * s + 4 * i + col)]);
    wave_sync();
    ar.reduce_all(v);
    fwd_rw<4>(v, wb, ar);
}

template <class A>
__device__ __forceinline__ void inv256(const A &ar, typename A::V (&v)[16], uint64_t *L, uint32_t lane)
{
    const uint32_t col = lane & 3, s = lane >> 2;
    typename A::W wa[15], wb[15];
    tw_inv<4, 256, 1>(wb, 16 * s, ar, 1);
#pragma unroll
    for (int i = 0; i < 15; ++i) wa[i] = ar.tw_uniform(i < 8 ? 8 + i : i < 12 ? i - 4 : i < 14 ? i - 10 : 1);
    inv_rw<4>(v, wb, ar);
#pragma unroll
    for (int i = 0; i < 16; ++i) L[slot16(64 * s + 4 * i + col)] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = ar.from_bits(L[slot16(lane + 64 * i)]);
    wave_sync();
    ar.reduce_all(v);
    inv_rw<4>(v, wa, ar);
}

// Second inverse pass of a source tile m, scaled, to y (element lane + 64 i).
template <int MODE, class A>
__device__ __forceinline__ void source_cols16(const A &ar, const uint64_t *m, uint64_t *y, uint32_t lane)
{
    typename A::V v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = ar.from_bits(m[lane + 64 * i]);
    ar.reduce_all(v);
    inv256(ar, v, y, lane);
    inv_store(y, v, ar, kSourceMode<MODE>, [&](int i) { return lane + 64 * i; });
}

// v[i] = Conv(y)[lane + 64 i], G elements at a time: all 16 where two columns hold
// a sum, so that a source's constants are fetched once (with 8, ModUp's launch of
// HMult at l = 30 takes 46.3 us in place of 44.4), 4 with 128-bit sums.
template <class Acc, int G, class A>
__device__ __forceinline__ void conv16_acc(typename A::V (&v)[16], const A &ar, const uint64_t *y, uint32_t ns,
                                           ConvWord *h, const Prime &P, uint32_t lane)
{
#pragma unroll
    for (int g = 0; g < 16; g += G) {
        Acc acc[G];
#pragma unroll
        for (int i = 0; i < G; ++i) acc[i].start(h);
        for (uint32_t k = 0; k < ns; ++k) {
            uint64_t x[G];
#pragma unroll
            for (int i = 0; i < G; ++i) x[i] = y[k * kTile16 + lane + 64 * (g + i)];
#pragma unroll
            for (int i = 0; i < G; ++i) acc[i].add(x[i], h, k);
        }
#pragma unroll
        for (int i = 0; i < G; ++i) v[g + i] = acc[i].value(ar, h, P);
    }
}
__device__ __forceinline__ void conv16(double (&v)[16], const FpArith &ar, const uint64_t *y, uint32_t ns, ConvWord *h,
                                       const Prime &P, uint32_t lane)
{
    conv16_acc<FoldAcc, 16>(v, ar, y, ns, h, P, lane);
}
__device__ __forceinline__ void conv16(uint64_t (&v)[16], const IntArith &ar, const uint64_t *y, uint32_t ns, ConvWord *h,
                                       const Prime &P, uint32_t lane)
{
    if (h[kConvStart])
        conv16_acc<FoldWideAcc, 16>(v, ar, y, ns, h, P, lane);
    else
        conv16_acc<WideAcc<MacColsAcc>, 4>(v, ar, y, ns, h, P, lane);
}

// First forward pass of a target tile to m, converted from the sources (lifted
// from the one source by Rescale).
template <int MODE, class A>
__device__ __forceinline__ void target_cols16(const A &ar, const Prime &P, const uint64_t *y, uint32_t ns, ConvWord *h,
                                              uint64_t qlmod, uint64_t ql, uint64_t *L, uint64_t *m, uint32_t lane)
{
    typename A::V v[16];
    typename A::W wb[15];
    tw_fwd<4, 256, 1>(wb, 16 * (lane >> 2), ar, 1);
    if (MODE == COLS_RESCALE) {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = ar.lift(y[lane + 64 * i], ql, qlmod, P);
    } else {
        conv16(v, ar, y, ns, h, P, lane);
    }
    fwd256(ar, v, wb, L, lane);
#pragma unroll
    for (int i = 0; i < 16; ++i) m[lane + 64 * i] = ar.to_bits(v[i]);
}

// The k-th set bit of m (k below its population).
__device__ __forceinline__ uint32_t nth_bit(uint64_t m, uint32_t k)
{
    for (; k; --k) m &= m - 1;
    return (uint32_t)__builtin_ctzll(m);
}

// blockIdx: (tile, job, part); the parts of a job share its targets and each
// form the sources.  Targets on the integer path, about twice the work of the
// others, come first in the order in which the waves take them.
template <int MODE>
__global__ __launch_bounds__(64 * kCols16Waves) void k16_cols(ColsArgs a)
{
    extern __shared__ uint64_t lds16[];  // ns source tiles, then a tile per wave
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const uint32_t tile = blockIdx.x, job = blockIdx.y, n = a.level + 1;
    uint32_t lo = 0, ns = 1, set = a.pset, prime0 = a.level;
    uint64_t targets = (1ull << a.level) - 1;  // by prime; Rescale: q_0..q_{l-1}
    if (MODE == COLS_MODUP) {
        lo = job * a.alpha;
        ns = min(a.alpha, n - lo);
        set = job * a.alpha + ns - 1;
        prime0 = lo;
        const uint64_t own = ((1ull << ns) - 1) << lo, special = ((1ull << a.np) - 1) << a.nq;
        targets = (((2ull << a.level) - 1) & ~own) | special;
    } else if (MODE == COLS_MODDOWN) {
        ns = a.np;
        prime0 = a.nq;
        targets = (2ull << a.level) - 1;
    }
    const uint64_t *src = a.src + (MODE == COLS_MODUP ? (int64_t)lo * 65536 : (int64_t)job * a.src_stride) + tile * kTile16;
    for (uint32_t k = w; k < ns; k += kCols16Waves) {
        const uint32_t pi = prime0 + k;
        const Prime P = a.primes[pi];
        uint64_t *y = lds16 + k * kTile16;
        const uint64_t *m = src + (size_t)k * 65536;
        if (P.q < kFpMaxPrime) {
            FpArith ar = fp_arith(a.twdi, P, pi, 65536);
            if (MODE != COLS_RESCALE) ar.fc = a.ysd[set * kMaxDigitPrimes + k];
            source_cols16<MODE>(ar, m, y, lane);
        } else {
            IntArith ar = int_arith(a.twi, P, pi, 65536);
            if (MODE != COLS_RESCALE) {
                const ulonglong2 f = a.ys[set * kMaxDigitPrimes + k];
                ar.fc = f.x;
                ar.fc_s = f.y;
            }
            source_cols16<MODE>(ar, m, y, lane);
        }
    }
    __syncthreads();
    const uint64_t heavy = targets & a.int_primes, light = targets & ~a.int_primes;
    const uint32_t nh = (uint32_t)__builtin_popcountll(heavy), nt = (uint32_t)__builtin_popcountll(targets);
    uint64_t *L = lds16 + (ns + w) * kTile16, *dst = a.dst + (int64_t)job * a.dst_stride + tile * kTile16;
    for (uint32_t t = blockIdx.z + gridDim.z * w; t < nt; t += gridDim.z * kCols16Waves) {
        const uint32_t pi = t < nh ? nth_bit(heavy, t) : nth_bit(light, t - nh);
        const uint32_t r = pi <= a.level ? pi : pi - a.nq + n;
        const Prime P = a.primes[pi];
        ConvWord *h = (ConvWord *)(a.hmod + ((size_t)set * (a.nq + a.np) + pi) * kConvRow);
        const uint64_t qlmod = MODE == COLS_RESCALE ? a.rs_qlmod[pi] : 0;
        const uint64_t ql = MODE == COLS_RESCALE ? a.primes[a.level].q : 0;
        uint64_t *m = dst + (size_t)r * 65536;
        if (P.q < kFpMaxPrime)
            target_cols16<MODE>(fp_arith(a.twdf, P, pi, 65536), P, lds16, ns, h, qlmod, ql, L, m, lane);
        else
            target_cols16<MODE>(int_arith(a.twf, P, pi, 65536), P, lds16, ns, h, qlmod, ql, L, m, lane);
    }
}

// The key inner product at N = 2^16 on ModUp's tiles: the last forward pass of
// every digit's row runs here, so the finished transforms never go through
// memory.  A wave takes one row of the 256 x 256 view of extended row r, 4
// elements per lane in the layouts of the 4-element inverse passes (D, C, B, A);
// it ends in A, four consecutive positions, in which the keys are read and the
// sums stored, and from which ModDown's first inverse pass starts.  (With 8
// elements per lane the sums of both halves, 64 registers on the integer path,
// leave one wave per SIMD.)  A digit's own row comes from ip.own (gathered
// through ip.own_galois) or, with a tensor, is the product a1 b1.
// IP_MODDOWN, IP_TENSOR: the special rows, whose workgroups come first, go on to
// ModDown's first inverse pass.  IP_EXTENDED: all rows' sums are stored, or
// accumulated (see IpArgs).
enum IpMode { IP_MODDOWN, IP_TENSOR, IP_EXTENDED };
// Four rows a workgroup read 128-byte runs of the tiles: 56 us at l = 30 with a
// tensor (three digits, 35 rows; 294 MB moved, 250 MB of them operands, at the
// rate of a copy) where eight
// rows take 58, two 60, sixteen 65, and the row pass and the inner product apart
// 25 + 47.  A rotation's at l = 17 takes 24 us for 12 + 20.
// Loading the next digit's row ahead of this one's rounds gains nothing (58.3 us
// against 57.7): the other waves cover the wait.
constexpr uint32_t kIpRows = 4;

// The rounds of a forward row pass from layout D to layout A.
template <class A>
__device__ __forceinline__ void fwd_row4_rounds(const A &ar, typename A::V (&v)[4], uint64_t *L, uint32_t s, uint32_t b)
{
    typename A::W w[3], w2[3];
    tw_fwd<2, 256, 64, A, true>(w, p4d(s, 0), ar, 256 + b);
    tw_fwd<2, 256, 16, A, true>(w2, p4c(s, 0), ar, 256 + b);
    ar.reduce_all(v);
    fwd_rw<2>(v, w, ar);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4d(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4c(s, i))]);
    tw_fwd<2, 256, 4, A, true>(w, p4b(s, 0), ar, 256 + b);
    fwd_rw<2>(v, w2, ar);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4c(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4b(s, i))]);
    tw_fwd<2, 256, 1, A, true>(w2, p4a(s, 0), ar, 256 + b);
    ar.reduce_all(v);
    fwd_rw<2>(v, w, ar);
#pragma unroll
    for (int i = 0; i < 4; ++i) L[row4_slot(p4b(s, i))] = ar.to_bits(v[i]);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = ar.from_bits(L[row4_slot(p4a(s, i))]);
    wave_sync();
    fwd_rw<2>(v, w2, ar);
}

template <IpMode MODE, class A>
__device__ __forceinline__ void ip_rows16(const IpArgs &ip, const NttArgs &ia, const A &fwd, const A &inv, const Prime &P,
                                          uint32_t r, uint32_t pi, uint64_t *L, uint32_t b, uint32_t s)
{
    const bool qrow = r <= ip.level;
    const uint32_t own = qrow ? r / ip.alpha : ~0u, e0 = b * 256 + 4 * s;
    const size_t off = (size_t)r * 65536, kstep = (size_t)(ip.nq + ip.np) * 65536;
    const uint32_t g = ip.own_galois, sb = MODE == IP_TENSOR || g == 1 ? b * 256 : galois_src(b * 256, g, 16) & ~255u;
    const uint64_t *mid = ip.ext + off + (s >> 2) * 1024 + (b & 15) * 64 + (b >> 4) * 4 + (s & 3);
    auto read = [&](uint64_t (&x)[4], const uint64_t *p) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = p[i];
    };
    auto gather = [&](uint64_t (&x)[4], const uint64_t *row) {  // x = phi_g(row) at e0
        read(x, row + sb + 4 * s);
        if (g == 1) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) L[row4_slot(p4a(s, i))] = x[i];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = L[row4_slot(galois_src(e0 + i, g, 16) - sb)];
        wave_sync();
    };
    typename A::Sum s0[4], s1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) fwd.sum_start(s0[i]), fwd.sum_start(s1[i]);
    for (uint32_t j = 0; j < ip.beta; ++j) {
        const uint64_t *key = ip.key + (size_t)j * 2 * kstep + (size_t)pi * 65536 + e0;
        uint64_t k0[4], k1[4], x[4];
        typename A::V v[4];
        if (j != own) {
            const uint64_t *m = mid + (size_t)j * ip.rows * 65536;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = m[i * 16384];
            read(k0, key);
            read(k1, key + kstep);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fwd.from_bits(x[i]);
            fwd_row4_rounds(fwd, v, L, s, b);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fwd.sum_input(v[i]);
        } else {
            read(k0, key);
            read(k1, key + kstep);
            if (MODE == IP_TENSOR) {
                uint64_t y[4];
                read(x, ip.ta1 + off + e0);
                read(y, ip.tb1 + off + e0);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = fwd.product(x[i], y[i], P);
            } else {
                gather(x, ip.own + off);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = fwd.from_u64(x[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) fwd.sum_add(s0[i], v[i], k0[i]), fwd.sum_add(s1[i], v[i], k1[i]);
        if (j & 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) fwd.sum_centre(s0[i]), fwd.sum_centre(s1[i]);
        }
    }
    if (MODE == IP_TENSOR && qrow) {
        const uint64_t pm = ip.pmod[pi];
        uint64_t a0[4], a1[4], b0[4], b1[4];
        read(a0, ip.ta0 + off + e0);
        read(b0, ip.tb0 + off + e0);
        read(a1, ip.ta1 + off + e0);
        read(b1, ip.tb1 + off + e0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fwd.sum_centre(s0[i]), fwd.sum_centre(s1[i]);
            fwd.sum_add(s0[i], fwd.product(a0[i], b0[i], P), pm);
            fwd.sum_add(s1[i], fwd.product(a0[i], b1[i], P), pm);
            fwd.sum_add(s1[i], fwd.product(a1[i], b0[i], P), pm);
        }
    }
    if (MODE == IP_EXTENDED && ip.fold_tot && ip.fold_c0 && qrow) {
        const uint64_t pm = ip.pmod[pi];
        uint64_t x[4];
        gather(x, ip.fold_c0 + off);
#pragma unroll
        for (int i = 0; i < 4; ++i) fwd.sum_centre(s0[i]), fwd.sum_add(s0[i], fwd.from_u64(x[i]), pm);
    }
    if (MODE == IP_EXTENDED || qrow) {
        const bool fold = MODE == IP_EXTENDED && ip.fold_tot, more = fold && !ip.fold_first;
        uint64_t *out = (fold ? ip.fold_tot : ip.acc) + off + e0;
        const size_t half = (size_t)ip.rows * 65536;
        uint64_t t0[4] = {}, t1[4] = {};
        if (more) {
            read(t0, out);
            read(t1, out + half);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t y0 = fwd.fwd_final(fwd.sum_value(s0[i], P)), y1 = fwd.fwd_final(fwd.sum_value(s1[i], P));
            t0[i] = more ? addmod(t0[i], y0, P.q) : y0;
            t1[i] = more ? addmod(t1[i], y1, P.q) : y1;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = t0[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) out[half + i] = t1[i];
        return;
    }
#pragma unroll
    for (uint32_t t = 0; t < 2; ++t) {
        uint64_t *limb = ia.mid + (int64_t)t * ia.mid_stride + (size_t)(r - ip.level - 1) * 65536;
        wave_sync();
        inv_row4_values(inv, L, s, b, [&](int i) { return fwd.sum_value(t ? s1[i] : s0[i], P); }, mid_row<64>(ia, limb, b, s));
    }
}

template <IpMode MODE>
__global__ __launch_bounds__(64 * kIpRows) void k16_ip_rows(IpArgs ip, NttArgs ia, const ulonglong2 *twf, const double *twdf)
{
    __shared__ uint64_t lds[kIpRows * 256];
    const uint32_t y = blockIdx.y, nqr = ip.level + 1, nsp = ip.rows - nqr, r = y < nsp ? nqr + y : y - nsp;
    const uint32_t pi = coef::row_prime(r, ip.level, ip.nq), s = threadIdx.x & 63;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), groups = 16 / kIpRows;
    const uint32_t b = 16 * (blockIdx.x % groups * kIpRows + w) + blockIdx.x / groups;
    uint64_t *L = lds + w * 256;
    const Prime P = ip.primes[pi];
    if (P.q < kFpMaxPrime)
        ip_rows16<MODE>(ip, ia, fp_arith(twdf, P, pi, 65536), fp_arith(ia.twd, P, pi, 65536), P, r, pi, L, b, s);
    else
        ip_rows16<MODE>(ip, ia, int_arith(twf, P, pi, 65536), int_arith(ia.tw, P, pi, 65536), P, r, pi, L, b, s);
}

// ---------------------------------------------------- kernels: grid and queue
// Every NTT stage exists as a grid kernel (one launch = one NttArgs, unit =
// (blockIdx.x, blockIdx.y)) and as a persistent kernel that claims units
// (instance, limb, tile) of many launches from a work queue, so a whole batch
// of ciphertexts at different levels goes through one launch per stage.

__device__ __forceinline__ UnitId grid_unit(const NttArgs &a)
{
    if (gridDim.x != 16 || a.by_tile || (a.map.skip_alpha != 0 && !a.map.dense)) {  // or N = 2^12, or skipped limbs
        UnitId u;
        u.limb = blockIdx.y;
        u.tile = blockIdx.x;
        return u;
    }
    return unit_of(blockIdx.y * 16 + blockIdx.x, gridDim.y, a.n_heavy, a.heavy);
}

#define NTT_GRID(NAME, LDS, THREADS, ATTR, ...)                                                  \
    __global__ __launch_bounds__(THREADS) ATTR void k_##NAME(NttArgs a)                          \
    {                                                                                             \
        __shared__ uint64_t lds[LDS];                                                             \
        const UnitId u = grid_unit(a);                                                            \
        __VA_ARGS__(a, u.limb, u.tile, lds, threadIdx.x);                                         \
    }
// two workgroups per CU: at most 128 VGPRs
#define NTT_QUEUE(NAME, LDS, THREADS, ...)                                                       \
    __global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(4))) void           \
        q_##NAME(const NttArgs *insts, WorkQueue q)                                              \
    {                                                                                             \
        __shared__ uint64_t lds[LDS];                                                             \
        __shared__ uint32_t claim;                                                                \
        run_work_queue_uniform(insts, q, &claim, [&](const NttArgs &a, uint32_t limb, uint32_t tile) { \
            __VA_ARGS__(a, limb, tile, lds, thread_index());                                      \
        });                                                                                       \
    }
#define NTT_KERNELS(NAME, LDS, THREADS, ATTR, ...)                                               \
    NTT_GRID(NAME, LDS, THREADS, ATTR, __VA_ARGS__)                                               \
    NTT_QUEUE(NAME, LDS, THREADS, __VA_ARGS__)

// Three 512-thread workgroups per CU for the plain passes: the column passes
// fit in 72 VGPRs; the row passes spill 12 to 16 bytes per lane and still gain
// over 35 limbs (not over 74, and the tensor prologue's pass loses, so it
// keeps two workgroups per CU).
#define OCC6 __attribute__((amdgpu_waves_per_eu(6)))
#define OCC4 __attribute__((amdgpu_waves_per_eu(4)))  // two: 128 VGPRs

NTT_KERNELS(fwd_col_plain, kLds16, kThreads16, OCC6, fwd_col_unit<PRO_PLAIN>)
NTT_GRID(fwd_col_rescale, kLds16, kThreads16, , fwd_col_unit<PRO_RESCALE>)
NTT_KERNELS(fwd_col_bconv, kLds16, kThreads16, , fwd_col_unit<PRO_BCONV>)
NTT_KERNELS(fwd_row_plain, kLds16, kThreads16, OCC6, fwd_row_unit<EPI_PLAIN>)
NTT_KERNELS(fwd_row_moddown, kLds16, kThreads16, OCC4, fwd_row_unit<EPI_MODDOWN>)
NTT_GRID(fwd_row_rescale, kLds16, kThreads16, , fwd_row_unit<EPI_RESCALE>)
NTT_KERNELS(inv_row_plain, kLds16, kThreads16, OCC6, inv_row_unit<PRO_PLAIN>)
NTT_KERNELS(inv_row_galois, kLds16, kThreads16, , inv_row_unit<PRO_GALOIS>)
NTT_GRID(inv_row_tensor, kLds16, kThreads16, , inv_row_unit<PRO_TENSOR>)
NTT_KERNELS(inv_col, kLds16, kThreads16, OCC6, inv_col_unit)
// Grid kernels with narrower tiles (TW = 8, 4 columns or rows per workgroup of
// 32 TW threads), for launches over few limbs; unit = (blockIdx.x, blockIdx.y).
#define NTT_NARROW(NAME, UNIT_T)                                                                    \
    __global__ __launch_bounds__(256) OCC4 void k_##NAME##_w8(NttArgs a)                                \
    {                                                                                               \
        __shared__ uint64_t lds[lds_words<8>()];                                                    \
        UNIT_T(8)(a, blockIdx.y, blockIdx.x, lds, threadIdx.x);                                     \
    }                                                                                               \
    __global__ __launch_bounds__(128) OCC4 void k_##NAME##_w4(NttArgs a)                                \
    {                                                                                               \
        __shared__ uint64_t lds[lds_words<4>()];                                                    \
        UNIT_T(4)(a, blockIdx.y, blockIdx.x, lds, threadIdx.x);                                     \
    }
// The 4-element inverse passes (tile code 2: 8 rows or columns, 512 threads).
__global__ __launch_bounds__(512) void k_inv_row4(NttArgs a)
{
    __shared__ uint64_t lds[kLds4];
    inv_row4_unit(a, blockIdx.y, blockIdx.x, lds, threadIdx.x);
}
__global__ __launch_bounds__(512) void k_inv_col4(NttArgs a)
{
    __shared__ uint64_t lds[kLds4];
    inv_col4_unit(a, blockIdx.y, blockIdx.x, lds, threadIdx.x);
}
#define U_FCP(W) fwd_col_unit<PRO_PLAIN, W>
#define U_FCR(W) fwd_col_unit<PRO_RESCALE, W>
#define U_FCB(W) fwd_col_unit<PRO_BCONV, W>
#define U_FRP(W) fwd_row_unit<EPI_PLAIN, W>
#define U_FRM(W) fwd_row_unit<EPI_MODDOWN, W>
#define U_FRR(W) fwd_row_unit<EPI_RESCALE, W>
#define U_IRP(W) inv_row_unit<PRO_PLAIN, W>
#define U_IRG(W) inv_row_unit<PRO_GALOIS, W>
#define U_IRT(W) inv_row_unit<PRO_TENSOR, W>
#define U_IC(W) inv_col_unit<W>
NTT_NARROW(fwd_col_plain, U_FCP)
NTT_NARROW(fwd_col_rescale, U_FCR)
NTT_NARROW(fwd_col_bconv, U_FCB)
NTT_NARROW(fwd_row_plain, U_FRP)
NTT_NARROW(fwd_row_moddown, U_FRM)
NTT_NARROW(fwd_row_rescale, U_FRR)
NTT_NARROW(inv_row_plain, U_IRP)
NTT_NARROW(inv_row_galois, U_IRG)
NTT_NARROW(inv_row_tensor, U_IRT)
NTT_NARROW(inv_col, U_IC)
#undef U_FCP
#undef U_FCR
#undef U_FCB
#undef U_FRP
#undef U_FRM
#undef U_FRR
#undef U_IRP
#undef U_IRG
#undef U_IRT
#undef U_IC
#undef NTT_NARROW

#define FWD12_PP fwd12_unit<PRO_PLAIN, EPI_PLAIN>
#define FWD12_RP fwd12_unit<PRO_RESCALE, EPI_PLAIN>
#define FWD12_BM fwd12_unit<PRO_BCONV, EPI_MODDOWN>
NTT_KERNELS(fwd12_plain, kLds12, kThreads12, , FWD12_PP)
NTT_GRID(fwd12_lift, kLds12, kThreads12, , FWD12_RP)
NTT_QUEUE(fwd12_bconv_moddown, kLds12, kThreads12, FWD12_BM)
NTT_KERNELS(inv12_plain, kLds12, kThreads12, , inv12_unit<PRO_PLAIN>)
NTT_QUEUE(inv12_galois, kLds12, kThreads12, inv12_unit<PRO_GALOIS>)
#undef FWD12_PP
#undef FWD12_RP
#undef FWD12_BM
#undef NTT_KERNELS
#undef NTT_GRID
#undef NTT_QUEUE
#undef OCC6
#undef OCC4

// ------------------------------------------- one launch for a whole batch
// The persistent kernel of a batch of key switches in one launch (N = 2^16):
// every step of every key switch is a group of units in one list, and a unit
// starts once the group it depends on (the previous step of the same key
// switch) is done, so the steps of different key switches overlap instead of
// meeting at eleven launch boundaries.  Dependencies go through per-group
// counters: a unit's stores are complete in every wave before the workgroup
// counts it done with an agent-scope release, and a waiting workgroup
// acquires at agent scope before it reads, which makes the data of other
// workgroups, on any XCD, visible.  The coefficient-wise steps run their
// 256-thread units on the two halves of the 512-thread workgroup, each half
// taking eight of the unit's sixteen 256-coefficient blocks.
//
constexpr uint32_t kFusedIpStage = 2 * coef::kIpStage * coef::kCoefThreads;
constexpr int kFusedLds = kLds16 > (int)kFusedIpStage ? kLds16 : (int)kFusedIpStage;
static_assert(kQueueBlocks % 2 == 0, "the two halves take half of a unit's blocks each");

__shared__ uint64_t g_fused_lds[kFusedLds];

// Completions a workgroup has not yet published: up to f.publish_every
// (at most kFusedPending) groups with their unit counts, kept by thread 0.
// Publishing costs one agent-scope release (a write-back of the XCD's L2), so
// it is done for several units at once: when publish_every groups are
// pending, before the workgroup blocks on a wait, and when it runs out of
// units.  A workgroup that blocks has published everything it finished, so
// the earliest unfinished unit can always proceed, and a workgroup that does
// not block publishes within publish_every units.
constexpr uint32_t kFusedPending = 32;
constexpr uint32_t kFusedSeen = 4;
struct Pending {
    uint32_t group[kFusedPending], count[kFusedPending], n;
    // groups this workgroup has seen complete (and acquired after): a later unit waiting for one of
    // them needs neither a poll nor another acquire, since a complete group's data no longer changes
    uint32_t seen[kFusedSeen], seen_next;
};

__device__ __forceinline__ void fused_publish(const FusedArgs &f, Pending &p)
{
    if (p.n == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    for (uint32_t i = 0; i < p.n; ++i)
        __hip_atomic_fetch_add(f.done + (size_t)p.group[i] * f.done_stride, p.count[i], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    p.n = 0;
}

__device__ __forceinline__ void fused_finished(const FusedArgs &f, Pending &p, uint32_t g)
{
    for (uint32_t i = 0; i < p.n; ++i)
        if (p.group[i] == g) {
            ++p.count[i];
            return;
        }
    p.group[p.n] = g;
    p.count[p.n] = 1;
    if (++p.n >= f.publish_every) fused_publish(f, p);
}

// Waits (thread 0 only) until every unit of group g is done, publishing the
// workgroup's own completions first if it has to wait; gives up after
// spin_limit polls and raises the fault flag, so that the launch always ends.
__device__ __forceinline__ void fused_wait(const FusedArgs &f, Pending &p, uint32_t g)
{
    for (uint32_t i = 0; i < kFusedSeen; ++i)
        if (p.seen[i] == g) return;
    const uint32_t want = f.target[g];
    const uint32_t *cnt = f.done + (size_t)g * f.done_stride;
    if (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) {
        fused_publish(f, p);
        uint32_t polls = 0;
        while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) {
            if (++polls > f.spin_limit) {
                __hip_atomic_store(f.fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    p.seen[p.seen_next] = g;
    p.seen_next = (p.seen_next + 1) % kFusedSeen;
}

// The argument block of the unit's step: the pointer passes through an empty
// asm statement, so that the scalar loads of one step's block are not
// hoisted above the switch (speculated for every step, the blocks of all
// steps would be live at once).
template <class Args>
__device__ __forceinline__ Args step_args(const Args *base, uint32_t inst)
{
    uint64_t p = (uint64_t)(uintptr_t)base;
    asm volatile("" : "+s"(p));
    return uniform_args((const Args *)(uintptr_t)p + inst);
}

__global__ __launch_bounds__(kThreads16) __attribute__((amdgpu_waves_per_eu(4))) void q_fused16(FusedArgs f)
{
    typedef const __attribute__((address_space(4))) uint32_t ConstWord;
    __shared__ uint32_t claim;
    __shared__ Pending pend;  // thread 0's
    if (threadIdx.x == 0) {
        claim = atomicAdd(f.claim, 1u);
        pend.n = 0;
        for (uint32_t i = 0; i < kFusedSeen; ++i) pend.seen[i] = kNoGroup;
        pend.seen_next = 0;
    }
    __syncthreads();
    uint32_t u = __builtin_amdgcn_readfirstlane(claim);
    while (u < f.nunits) {
        ConstWord *w = (ConstWord *)((uintptr_t)f.units + (uintptr_t)u * sizeof(FusedUnit));
        const uint32_t inst = __builtin_amdgcn_readfirstlane(w[0]);
        const uint32_t code = __builtin_amdgcn_readfirstlane(w[1]);
        const uint32_t wait = __builtin_amdgcn_readfirstlane(w[2]);
        const uint32_t signal = __builtin_amdgcn_readfirstlane(w[3]);
        __syncthreads();  // every thread has read claim and is done with the previous unit's LDS
        if (threadIdx.x == 0) claim = atomicAdd(f.claim, 1u);
        if (wait != kNoGroup) {
            if (threadIdx.x == 0) fused_wait(f, pend, wait);
            __syncthreads();
        }
        const uint32_t step = code >> 28, tile = (code >> 16) & 0xFFFu, limb = code & 0xFFFFu;
        // the thread index is taken anew for every unit: offsets derived from it and hoisted out of
        // the loop would stay live across every step's body
        const uint32_t tx = thread_index();
        switch (step) {
        case QI_TENSOR: {
            const TensorArgs a = step_args(f.tensor, inst);
            for (uint32_t i = tx / coef::kCoefThreads; i < kQueueBlocks; i += 2)
                coef::tensor_unit(a, limb, tile * kQueueBlocks + i, tx % coef::kCoefThreads);
            break;
        }
        case QI_UP_INTT0_PLAIN: inv_row_unit<PRO_PLAIN>(step_args(f.ntt[0], inst), limb, tile, g_fused_lds, tx); break;
        case QI_UP_INTT0_GALOIS: inv_row_unit<PRO_GALOIS>(step_args(f.ntt[0], inst), limb, tile, g_fused_lds, tx); break;
        case QI_UP_INTT1: inv_col_unit(step_args(f.ntt[0], inst), limb, tile, g_fused_lds, tx); break;
        case QI_UP_BCONV: {
            const BconvCommon c = uniform_args(&f.bconv[inst].c);
            const BconvJob J = uniform_args(&f.bconv[inst].job[limb]);
            const uint32_t nb = c.N / (coef::kCoefThreads * kQueueBlocks);
            for (uint32_t i = tx / coef::kCoefThreads; i < kQueueBlocks; i += 2)
                coef::bconv_unit(c, J, (tile % nb) * kQueueBlocks + i, tile / nb, tx % coef::kCoefThreads);
            break;
        }
        case QI_UP_NTT0: fwd_col_unit<PRO_PLAIN>(step_args(f.ntt[1], inst), limb, tile, g_fused_lds, tx); break;
        case QI_UP_NTT1: fwd_row_unit<EPI_PLAIN>(step_args(f.ntt[1], inst), limb, tile, g_fused_lds, tx); break;
        case QI_IP: {
            const uint32_t half = tx / coef::kCoefThreads;
            coef::ip_blocks(step_args(f.ip, inst), limb, tile * kQueueBlocks + half * (kQueueBlocks / 2),
                            kQueueBlocks / 2, g_fused_lds + half * coef::kIpStage * coef::kCoefThreads,
                            tx % coef::kCoefThreads);
            break;
        }
        case QI_DN_INTT0: inv_row_unit<PRO_PLAIN>(step_args(f.ntt[2], inst), limb, tile, g_fused_lds, tx); break;
        case QI_DN_INTT1: inv_col_unit(step_args(f.ntt[2], inst), limb, tile, g_fused_lds, tx); break;
        case QI_DN_NTT0: fwd_col_unit<PRO_BCONV>(step_args(f.ntt[3], inst), limb, tile, g_fused_lds, tx); break;
        case QI_DN_NTT1: fwd_row_unit<EPI_MODDOWN>(step_args(f.ntt[3], inst), limb, tile, g_fused_lds, tx); break;
        default: break;
        }
        // the barrier does not wait for global stores: every wave waits for its own first, so
        // the unit's stores are complete before thread 0 records (and later publishes) it
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        if (threadIdx.x == 0) fused_finished(f, pend, signal);
        u = __builtin_amdgcn_readfirstlane(claim);
    }
    if (threadIdx.x == 0) fused_publish(f, pend);
}

typedef void (*GridKernel)(NttArgs);
typedef void (*QueueKernel)(const NttArgs *, WorkQueue);

struct StageKernels {
    GridKernel grid;
    QueueKernel queue;
};

// The key inner product (N = 2^16) with the first inverse pass of ModDown's
// special rows run by the same workgroups (Sec. III-F.5: the inner product
// feeds ModDown directly).  A block bx of 256 coefficients of a row is the
// 256-point row problem b = bx of that row's inverse NTT, so a workgroup of a
// special row reduces its sums over two blocks, stages them in LDS, and its
// four waves run the row passes (4 elements per thread), writing their output
// where ModDown's INTT keeps it; the INTT then runs its column pass only.  The
// special rows' accumulators never reach memory.  Their workgroups come first
// in the launch, so their longer units overlap the q-rows' streaming instead
// of forming its tail.  `ia` is ModDown's INTT (the rows p_0..p_{K-1} of both
// accumulators, in that order).
constexpr uint32_t kIpRowpassLds = coef::kIpStage * coef::kCoefThreads + 4 * 256;

template <bool TENSOR>
__device__ __forceinline__ void ip_rowpass_unit(const IpArgs &ip, const NttArgs &ia, uint32_t y, uint32_t bx,
                                                uint64_t *lds, uint32_t tid)
{
    const uint32_t nqr = ip.level + 1, nsp = ip.rows - nqr;
    const uint32_t r = y < nsp ? nqr + y : y - nsp;
    if (r < nqr) {
        if (TENSOR)
            coef::ip_unit_tensor(ip, r, bx, tid);
        else
            coef::ip_unit(ip, r, bx, lds, tid);
        return;
    }
    // a special row: blocks 2 bx and 2 bx + 1 (the upper half of the grid row has no work), so
    // that all four waves run a row pass (block 2 bx + w / 2, polynomial w % 2)
    if (bx >= (1u << ip.logn) / (2 * coef::kCoefThreads)) return;
    uint64_t v[4];
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
        const coef::RegStore st{&v[2 * h], &v[2 * h + 1]};
        if (TENSOR)
            coef::ip_unit_tensor(ip, r, 2 * bx + h, tid, st);
        else
            coef::ip_unit(ip, r, 2 * bx + h, lds, tid, st);
    }
    // the four rows' inputs; after the barrier the staging area is the row passes' scratch
    uint64_t *in = lds + coef::kIpStage * coef::kCoefThreads;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) in[i * coef::kCoefThreads + tid] = v[i];
    __syncthreads();
    const uint32_t w = tid >> 6, s = tid & 63, k = r - nqr, prime = ip.nq + k;
    const uint32_t poly = w & 1, b = 2 * bx + (w >> 1);
    const Prime P = ia.primes[prime];
    const uint64_t *x = in + ((w >> 1) * 2 + poly) * coef::kCoefThreads;
    uint64_t *L = lds + w * 256;
    const MidRow m = mid_row<64>(ia, ia.mid + (int64_t)poly * ia.mid_stride + (size_t)k * 65536, b, s);
    auto load = [&](int i) { return x[p4a(s, i)]; };
    if (P.q < kFpMaxPrime)
        inv_row4_rounds(fp_arith(ia, P, prime, 65536), L, s, b, load, m);
    else
        inv_row4_rounds(int_arith(ia, P, prime, 65536), L, s, b, load, m);
}

__global__ __launch_bounds__(coef::kCoefThreads) void k_inner_product_rowpass(IpArgs ip, NttArgs ia)
{
    __shared__ uint64_t lds[kIpRowpassLds];
    ip_rowpass_unit<false>(ip, ia, blockIdx.y, blockIdx.x, lds, threadIdx.x);
}

__global__ __launch_bounds__(coef::kCoefThreads) void k_inner_product_tensor_rowpass(IpArgs ip, NttArgs ia)
{
    __shared__ uint64_t lds[kIpRowpassLds];
    ip_rowpass_unit<true>(ip, ia, blockIdx.y, blockIdx.x, lds, threadIdx.x);
}

// The kernel that runs one pass of a stage (pass 0 = first, 1 = second at N =
// 2^16) with tiles of tw columns (rows); the narrow tiles have grid kernels only.
bool stage_kernels(NttStage st, uint32_t logn, int pass, StageKernels &k, uint32_t tw = 16)
{
#define SK(GRID, QUEUE) \
    k.grid = GRID; \
    k.queue = QUEUE; \
    return true;
#define SK_TILES(G) tw == 8 ? k_##G##_w8 : tw == 4 ? k_##G##_w4 : k_##G
#define SK16(G) SK(SK_TILES(G), tw == 16 ? q_##G : nullptr)
#define SK16_GRID(G) SK(SK_TILES(G), nullptr)
    if (logn == 12) {  // whole limbs; the split transforms have launches of their own
        if (pass != 0) return false;
        switch (st) {
        case STAGE_FWD_PLAIN: SK(k_fwd12_plain, q_fwd12_plain)
        case STAGE_FWD_LIFT: SK(k_fwd12_lift, nullptr)
        case STAGE_FWD_BCONV_MODDOWN: SK(nullptr, q_fwd12_bconv_moddown)
        case STAGE_INV_PLAIN: SK(k_inv12_plain, q_inv12_plain)
        case STAGE_INV_GALOIS: SK(nullptr, q_inv12_galois)
        default: return false;
        }
    }
    if (tw == 2) {  // 4 elements per thread: the column pass of every inverse, the plain row pass
        const bool inv = st == STAGE_INV_PLAIN || st == STAGE_INV_GALOIS || st == STAGE_INV_TENSOR;
        if (inv && (pass == 1 || st == STAGE_INV_PLAIN)) {
            k.grid = pass == 0 ? k_inv_row4 : k_inv_col4;
            k.queue = nullptr;
            return true;
        }
        tw = 8;  // the other row passes take tiles of 8
    }
    switch (st) {
    case STAGE_FWD_PLAIN:
        if (pass == 0) { SK16(fwd_col_plain) } else { SK16(fwd_row_plain) }
    case STAGE_FWD_RESCALE:  // the first pass: launch_cols16
        if (pass == 0) return false;
        SK16_GRID(fwd_row_rescale)
    case STAGE_FWD_LIFT:
        if (pass == 0) { SK16_GRID(fwd_col_rescale) } else { SK16(fwd_row_plain) }
    case STAGE_FWD_BCONV_MODDOWN:
        if (pass == 0) { SK16(fwd_col_bconv) } else { SK16(fwd_row_moddown) }
    case STAGE_INV_PLAIN:
        if (pass == 0) { SK16(inv_row_plain) } else { SK16(inv_col) }
    case STAGE_INV_GALOIS:
        if (pass == 0) { SK16(inv_row_galois) } else { SK16(inv_col) }
    case STAGE_INV_TENSOR:
        if (pass == 0) { SK16_GRID(inv_row_tensor) } else { SK16(inv_col) }
    default: return false;
    }
#undef SK
#undef SK_TILES
#undef SK16
#undef SK16_GRID
}

}  // namespace

uint32_t ntt_passes(uint32_t logn) { return logn == 12 ? 1 : 2; }
uint32_t ntt_tiles(uint32_t logn) { return logn == 12 ? 1 : 16; }
static uint32_t ntt_threads(uint32_t logn) { return logn == 12 ? kThreads12 : kThreads16; }

// Fills a.heavy with the launch limbs on the integer path.  It leaves none when
// they do not fit the list, when every limb is on that path, or in launches of
// more than kHeavyMaxLimbs limbs: the assignment is then the whole-limb one.
// Measured side by side on whole transforms, placing the heavy limbs apart makes
// the passes over 31 and 35 limbs 5 to 12 % faster, leaves those over 62 limbs
// unchanged and makes those over 74 limbs 2 to 4 % slower: they run in more than
// one round of workgroups per CU, where the position of a workgroup in the launch
// no longer decides its CU.
constexpr uint32_t kHeavyMaxLimbs = 48;
static void set_heavy(NttArgs &a, uint32_t nlimbs)
{
    a.n_heavy = 0;
    if (a.logn != 16 || (a.map.skip_alpha != 0 && !a.map.dense) || nlimbs > kHeavyMaxLimbs) return;
    uint32_t nh = 0;
    for (uint32_t l = 0; l < nlimbs; ++l) {
        const LimbPos lp = limb_pos(a.map, l);
        if (lp.prime >= 64 || !((a.int_primes >> lp.prime) & 1)) continue;
        if (nh == (uint32_t)kMaxHeavy) return;
        a.heavy[nh++] = (uint8_t)l;
    }
    a.n_heavy = nh < nlimbs ? nh : 0;  // all limbs alike: whole-limb placement
}

// Tile width of the grid launches at N = 2^16, per kind (CKKS_TILE_TRANSFORM: both passes of a
// transform; CKKS_TILE_ROWS: a row pass next to a column launch), direction and launch size (0: the
// default rule below).  Set by ckks_ntt_tile_set (both kinds) and ckks_ntt_tile_set_kind (the
// autotuner), read by every grid launch.
static std::atomic<uint8_t> g_tile[2][2][kMaxTileLimbs + 1];

// The default.  Whole transforms: a column pass reads runs of 8 TW bytes, so 16
// columns (whole lines) from 8 limbs on (12 limbs 12.4 us, 16.9 with 8, 18.8 with
// 4), with rows alike, so that unit_of places a limb's passes on one XCD (24
// limbs inverse 17.8 us, 21 with rows of 8); 8 below, for twice the workgroups (4
// limbs 10.2 us, 11.7 with 16, 11.2 with 4).  A row pass alone (next to a column
// launch) reads whole rows at any width: 8 rows, which spread more evenly than 16
// (ModDown's over 36 limbs 18.2 us, 19.8 with 16, 18.1 to 23.4 with 4; Rescale's
// over 24 limbs 11.9, 12.8, 12.7; the tensor's first inverse pass within HMult of
// 31, 24 and 9 limbs 157.4, 129.9 and 69.3 us, 157.2, 130.9 and 69.9 with 16; the
// gathered one within a rotation of 31, 24 and 12 limbs 144.4, 121.4 and 73.7 us,
// 144.5, 122.4 and 75.0), 4 below 8 limbs (4 limbs 5.1 us, 5.8 with 8).
// ModDown's conversion in the column pass (13 to 16 special primes) computes more
// than it reads, and half as wide tiles fill the chip up to 24 limbs (ModDown at K =
// 14 over 8, 18 and 24 limbs 40.6, 50.0 and 54.4 us, 45.5, 55.2 and 56.1 with 16; over
// 26 and 30 limbs 58.3 and 58.8, 56.1 and 56.5 with 16).
static uint32_t default_tile(NttStage st, bool row_alone, uint32_t nlimbs)
{
    if (row_alone) return nlimbs >= 8 ? 8 : 4;
    if (st == STAGE_FWD_BCONV_MODDOWN) return nlimbs > 24 ? 16 : 8;
    return nlimbs >= 8 ? 16 : 8;
}

// tile code 2 (the 4-element inverse passes) applies to inverse stages only; a pass without a
// 4-element kernel (the gathered or tensor row passes) runs with tiles of 8
static uint32_t effective_tile(NttStage st, uint32_t tw)
{
    const bool inv = st == STAGE_INV_PLAIN || st == STAGE_INV_GALOIS || st == STAGE_INV_TENSOR;
    return tw == 2 && !inv ? 8 : tw;
}
static bool four_element_pass(NttStage st, uint32_t pass, uint32_t tw)
{
    return tw == 2 && (pass == 1 || st == STAGE_INV_PLAIN);
}

static uint32_t tile_width(NttStage st, uint32_t logn, uint32_t nlimbs, bool row_alone)
{
    if (logn != 16) return 16;
    const int inv = st == STAGE_INV_PLAIN || st == STAGE_INV_GALOIS || st == STAGE_INV_TENSOR;
    const uint32_t t = nlimbs <= kMaxTileLimbs ? g_tile[row_alone][inv][nlimbs].load(std::memory_order_relaxed) : 0;
    if (t) return t;
    return inv && nlimbs <= 8 ? 2 : default_tile(st, row_alone, nlimbs);
}

hipError_t launch_ntt_stage(NttStage st, const NttArgs &a0, uint32_t nlimbs, hipStream_t stream, uint32_t first_pass,
                            uint32_t last_pass)
{
    if (nlimbs == 0) return hipSuccess;
    if (first_pass >= ntt_passes(a0.logn)) return hipErrorInvalidValue;
    NttArgs a = a0;
    const bool inverse = st == STAGE_INV_PLAIN || st == STAGE_INV_GALOIS || st == STAGE_INV_TENSOR;
    const uint32_t tw = effective_tile(st, tile_width(st, a.logn, nlimbs, inverse ? last_pass == 0 : first_pass == 1));
    if (tw == 16) set_heavy(a, nlimbs);
    else a.n_heavy = 0;
    for (uint32_t pass = first_pass; pass < ntt_passes(a.logn) && pass <= last_pass; ++pass) {
        StageKernels k;
        if (!stage_kernels(st, a.logn, pass, k, tw) || !k.grid) return hipErrorInvalidValue;
        const bool four = a.logn == 16 && four_element_pass(st, pass, tw);
        const uint32_t pw = tw == 2 ? 8 : tw;  // rows or columns per workgroup
        const uint32_t tiles = a.logn == 12 ? 1 : 256 / pw;
        const uint32_t threads = a.logn == 12 ? kThreads12 : four ? 512 : 32 * pw;
        // ModDown's conversion (here with 13 to 16 special primes) reads the same K source rows for every
        // limb: workgroups in (tile, limb) order send a column tile of every limb to one XCD, whose L2
        // then holds that tile of the sources (whole limbs per XCD read all K rows, 6.5 MB at K = 13,
        // against 4 MB of L2).  Key switches at K = 13 and l = 30 take 228 us so and 232 without, at
        // K = 16 and l = 39 300 and 313.
        a.by_tile = st == STAGE_FWD_BCONV_MODDOWN && pass == 0;
        hipLaunchKernelGGL(k.grid, dim3(tiles, nlimbs), dim3(threads), 0, stream, a);
    }
    return hipGetLastError();
}

hipError_t launch_split12_inv_rows(NttStage st, const NttArgs &a, uint32_t nlimbs, hipStream_t stream)
{
    if (a.logn != 12 || !a.mid) return hipErrorInvalidValue;
    const dim3 grid(8, nlimbs), block(64);
    switch (st) {
    case STAGE_INV_PLAIN: hipLaunchKernelGGL(k12_inv_rows<PRO_PLAIN>, grid, block, 0, stream, a); break;
    case STAGE_INV_GALOIS: hipLaunchKernelGGL(k12_inv_rows<PRO_GALOIS>, grid, block, 0, stream, a); break;
    case STAGE_INV_TENSOR: hipLaunchKernelGGL(k12_inv_rows<PRO_TENSOR>, grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Sources whose first inverse pass the column launch runs itself.  A launch costs about 4 us of GPU
// time and 2 of the host's.  One source (Rescale, digits of one prime): Rescale at l = 17 takes 12.4 us
// so, 15 with a launch for it, a key switch at level 0 27.6 us against 28.4.  Two sources run their
// passes one after the other in every workgroup: HMult of the small set 33.6 us against 31.8.
uint32_t split12_row_sources() { return 1; }

hipError_t launch_split12_cols(ColsMode mode, NttPro pro, const ColsArgs &a, uint32_t njobs, hipStream_t stream)
{
    const uint32_t n = a.level + 1;
    // the most sources and targets of a job; LDS holds a tile per source and per wave (96 KB at most)
    const uint32_t ns = mode == COLS_MODUP ? (a.alpha < n ? a.alpha : n) : mode == COLS_MODDOWN ? a.np : 1;
    const uint32_t least = mode == COLS_MODUP ? (n % a.alpha ? n % a.alpha : ns) : 0;
    const uint32_t targets = mode == COLS_MODUP ? n + a.np - least : mode == COLS_MODDOWN ? n : a.level;
    if (targets == 0 || njobs == 0) return hipSuccess;
    const dim3 grid(8, njobs, (targets + kColsWaves - 1) / kColsWaves), block(64 * kColsWaves);
    const size_t lds = (size_t)(ns + kColsWaves) * kTile12 * 8;
#define COLS12(M, PRO) \
    if (mode == M && pro == PRO) { \
        hipLaunchKernelGGL((k12_cols<M, PRO>), grid, block, lds, stream, a); \
        return hipGetLastError(); \
    }
    COLS12(COLS_MODUP, PRO_MID)
    COLS12(COLS_MODUP, PRO_PLAIN)
    COLS12(COLS_MODUP, PRO_GALOIS)
    COLS12(COLS_MODUP, PRO_TENSOR)
    COLS12(COLS_MODDOWN, PRO_MID)
    COLS12(COLS_RESCALE, PRO_PLAIN)
#undef COLS12
    return hipErrorInvalidValue;
}

// Parts of a job: workgroups fill LDS, one to a CU, so as many parts as the CUs take at once.
constexpr uint32_t kCols16Parts = 256;

// LDS holds a tile per source and one per wave, 160 KB at 12 sources; more (whose sums
// the two columns do not hold either) go through the separate passes.
bool cols16_fits(uint32_t ns) { return ns <= kFoldMaxTerms; }

hipError_t launch_cols16(ColsMode mode, const ColsArgs &a, uint32_t njobs, hipStream_t stream)
{
    const uint32_t n = a.level + 1, ns = mode == COLS_MODUP ? (a.alpha < n ? a.alpha : n) : mode == COLS_MODDOWN ? a.np : 1;
    if (!cols16_fits(ns) || a.nq + a.np > 64) return hipErrorInvalidValue;
    if (njobs == 0 || (mode == COLS_RESCALE && a.level == 0)) return hipSuccess;
    const uint32_t parts = njobs < kCols16Parts / 64 ? kCols16Parts / 64 / njobs : 1;
    const dim3 grid(64, njobs, parts), block(64 * kCols16Waves);
    const size_t lds = (size_t)(ns + kCols16Waves) * kTile16 * 8;
    switch (mode) {
    case COLS_MODUP: hipLaunchKernelGGL(k16_cols<COLS_MODUP>, grid, block, lds, stream, a); break;
    case COLS_MODDOWN: hipLaunchKernelGGL(k16_cols<COLS_MODDOWN>, grid, block, lds, stream, a); break;
    case COLS_RESCALE: hipLaunchKernelGGL(k16_cols<COLS_RESCALE>, grid, block, lds, stream, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_split12_fwd_rows(NttEpi epi, const NttArgs &a, uint32_t nlimbs, hipStream_t stream)
{
    if (a.logn != 12 || !a.mid || (a.map.skip_alpha && !a.map.dense)) return hipErrorInvalidValue;
    const dim3 grid(8, nlimbs), block(64);
    switch (epi) {
    case EPI_PLAIN: hipLaunchKernelGGL(k12_fwd_rows<EPI_PLAIN>, grid, block, 0, stream, a); break;
    case EPI_MODDOWN: hipLaunchKernelGGL(k12_fwd_rows<EPI_MODDOWN>, grid, block, 0, stream, a); break;
    case EPI_RESCALE: hipLaunchKernelGGL(k12_fwd_rows<EPI_RESCALE>, grid, block, 0, stream, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_split12_ip(const IpArgs &ip, const NttArgs &ia, const NttArgs &fa, bool ready, hipStream_t stream)
{
    if (ip.logn != 12 || ia.logn != 12 || ip.fold_tot || ip.rows != ip.level + 1 + ip.np || ia.map.rows != ip.np ||
        !ia.mid || (!ready && ip.galois != 1) ||
        (ip.ta0 && (ip.galois != 1 || !ip.ta1 || !ip.tb0 || !ip.tb1 || !ip.pmod)))
        return hipErrorInvalidValue;
    const dim3 grid(8, ip.rows, 2), block(64);
    if (ready)
        hipLaunchKernelGGL(k12_ip_rows<true>, grid, block, 0, stream, ip, ia, fa.tw, fa.twd);
    else
        hipLaunchKernelGGL(k12_ip_rows<false>, grid, block, 0, stream, ip, ia, fa.tw, fa.twd);
    return hipGetLastError();
}

bool ntt_tile_set(uint32_t kind, uint32_t inverse, uint32_t nlimbs, uint32_t tile)
{
    if (kind > CKKS_TILE_ROWS || inverse > 1 || nlimbs == 0 || nlimbs > kMaxTileLimbs ||
        !(tile == 0 || tile == 4 || tile == 8 || tile == 16 || (tile == 2 && inverse == 1)))
        return false;
    g_tile[kind][inverse][nlimbs].store((uint8_t)tile, std::memory_order_relaxed);
    return true;
}

uint32_t ntt_tile_get(uint32_t kind, uint32_t inverse, uint32_t nlimbs)
{
    return tile_width(inverse ? STAGE_INV_PLAIN : STAGE_FWD_PLAIN, 16, nlimbs, kind == CKKS_TILE_ROWS);
}

hipError_t launch_inner_product_rowpass(const IpArgs &ip, const NttArgs &ia, hipStream_t stream)
{
    if (ip.logn != 16 || ia.logn != 16 || ip.fold_tot || ip.rows != ip.level + 1 + ip.np || ia.map.rows != ip.np ||
        ia.ys_mode != 2 || !ia.mid)
        return hipErrorInvalidValue;
    const dim3 grid((1u << ip.logn) / coef::kCoefThreads, ip.rows);
    if (ip.ta0) {
        if (ip.galois != 1 || !ip.ta1 || !ip.tb0 || !ip.tb1 || !ip.pmod) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_inner_product_tensor_rowpass, grid, dim3(coef::kCoefThreads), 0, stream, ip, ia);
    } else {
        hipLaunchKernelGGL(k_inner_product_rowpass, grid, dim3(coef::kCoefThreads), 0, stream, ip, ia);
    }
    return hipGetLastError();
}

hipError_t launch_ip_rows16(const IpArgs &ip, const NttArgs &ia, const NttArgs &fa, hipStream_t stream)
{
    const bool extended = !ia.mid;
    if (ip.logn != 16 || ip.galois != 1 || ip.rows != ip.level + 1 + ip.np || (!ip.own && !ip.ta0) ||
        (extended ? ip.ta0 != nullptr : ip.fold_tot || ia.logn != 16 || ia.map.rows != ip.np || ia.ys_mode != 2) ||
        (ip.ta0 && (!ip.ta1 || !ip.tb0 || !ip.tb1 || !ip.pmod)))
        return hipErrorInvalidValue;
    const dim3 grid(256 / kIpRows, ip.rows), block(64 * kIpRows);
    if (extended)
        hipLaunchKernelGGL(k16_ip_rows<IP_EXTENDED>, grid, block, 0, stream, ip, ia, fa.tw, fa.twd);
    else if (ip.ta0)
        hipLaunchKernelGGL(k16_ip_rows<IP_TENSOR>, grid, block, 0, stream, ip, ia, fa.tw, fa.twd);
    else
        hipLaunchKernelGGL(k16_ip_rows<IP_MODDOWN>, grid, block, 0, stream, ip, ia, fa.tw, fa.twd);
    return hipGetLastError();
}

hipError_t launch_ntt_stage_queue(NttStage st, uint32_t logn, uint32_t pass, const NttArgs *insts,
                                  const WorkQueue &q, uint32_t grid, hipStream_t stream)
{
    StageKernels k;
    if (!stage_kernels(st, logn, pass, k) || !k.queue) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k.queue, dim3(grid), dim3(ntt_threads(logn)), 0, stream, insts, q);
    return hipGetLastError();
}

hipError_t launch_fused_batch(const FusedArgs &f, uint32_t grid, hipStream_t stream)
{
    if (f.nunits == 0) return hipSuccess;
    hipLaunchKernelGGL(q_fused16, dim3(grid), dim3(kThreads16), 0, stream, f);
    return hipGetLastError();
}

// Whole transforms between limbs in one buffer each: plain, or of the centred lift (PRO_RESCALE).
hipError_t launch_ntt_fwd(const NttArgs &a0, uint32_t nlimbs, NttPro pro, hipStream_t stream, uint64_t *mid,
                          int64_t mid_poly_stride)
{
    NttArgs a = a0;
    a.mid = mid;
    a.mid_stride = mid_poly_stride;
    if (pro != PRO_PLAIN && pro != PRO_RESCALE) return hipErrorInvalidValue;
    return launch_ntt_stage(pro == PRO_PLAIN ? STAGE_FWD_PLAIN : STAGE_FWD_LIFT, a, nlimbs, stream);
}

hipError_t launch_ntt_inv(const NttArgs &a0, uint32_t nlimbs, hipStream_t stream, uint64_t *mid, int64_t mid_poly_stride)
{
    NttArgs a = a0;
    a.mid = mid;
    a.mid_stride = mid_poly_stride;
    return launch_ntt_stage(STAGE_INV_PLAIN, a, nlimbs, stream);
}

}  // namespace ckks
