// 32-bit word limbs (the paper's limb type is templated on the word size,
// Sec. III-C; only 64-bit words are verified there): the key-switching path
// with every residue in a 32-bit word, for primes below 2^30 at N = 2^16.
//
// Half the bytes of the 64-bit path per limb, and every modular product is
// native: a twiddle multiplication is Shoup's method on 32-bit words (one
// high multiply, two multiplies, one subtract), the butterflies are Harvey's
// lazy forms ([0, 4q) forward, [0, 2q) inverse, below 2^32 since q < 2^30), and
// sums of products (base conversion, inner product, tensor) accumulate exact
// 64-bit sums reduced once by an FP64 quotient (reduce64).  The same modulus
// budget takes about twice the limbs.
//
// Operations (include/ckks.h, ckks32_*): NTT / INTT, ModUp, ModDown, key
// switching, HMult with relinearisation, Rescale and the Galois automorphism
// with its key switch, all on limb-major [limbs][N] u32 polynomials.
//
// Kernels:
// - NTT passes: N = 2^16 as a 256 x 256 matrix, a column pass (the first
//   eight stages, each column an independent 256-point transform) and a row
//   pass (the last eight), four global accesses per element as in the paper.
//   A workgroup of 512 threads takes 32 columns (rows), 16 threads per column
//   (row) with 16 elements each, in two register rounds of four stages with an
//   exchange through LDS; a row's threads lie in one wave, so the row passes
//   exchange without workgroup barriers.  A pass over 188 rows issues 8 to 9 M
//   wave instructions (about 18 us of VALU time) and moves 98 MB; the column
//   pass takes 23 us and the row pass 31, whose twiddles are two words per
//   word of data: the limbs of one prime are neighbours in a launch, so that
//   they find them in L2.
// - Base conversion: two coefficients per thread.  Inner product: one.
// - Fused into the passes: HMult's d2 = a1 b1 and the automorphism into the
//   first inverse pass's load (and the inner product's own rows), Rescale's
//   lift into the first forward pass's load, ModDown's P^-1 (x - Conv(x)) (+
//   add) and Rescale's q_l^-1 (c - .) into the last forward pass's store.
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "internal.h"

namespace ckks {
ckks_status fail(ckks_status s, const std::string &msg);
}

using namespace ckks;

namespace {

constexpr uint32_t kN = 65536;
constexpr uint32_t kLogN = 16;
constexpr int kT = 512;                 // threads per pass workgroup
constexpr uint32_t kMaxPrimes32 = 64;   // q and p together
constexpr uint32_t kMaxRows32 = 64;     // rows of one polynomial in a launch (l + 1 + K)
constexpr uint32_t kMaxLaunch32 = 256;  // rows of one launch (polynomials x rows)
constexpr uint32_t kMaxDigit32 = 16;    // primes per digit and in the special basis
constexpr uint32_t kQBound = 1u << 30;

struct Pair32 {
    uint32_t w, s;  // a constant and its Shoup companion floor(w 2^32 / q)
};

struct Prime32 {
    uint32_t q, pad;
    double qinv;  // 1 / q, for the quotient of 64-bit sums
};

// -------------------------------------------------------- modular arithmetic

// x - q if x >= q, else x, for x < 2q (x - q wraps above x otherwise)
__device__ __forceinline__ uint32_t csub(uint32_t x, uint32_t q) { return min(x, x - q); }

// floor(ws y / 2^32) q - w y = -(w y mod q) or -(w y mod q) - q, modulo 2^32 (Shoup), any y
__device__ __forceinline__ uint32_t shoup_neg(uint32_t y, Pair32 w, uint32_t q) { return __umulhi(w.s, y) * q - w.w * y; }

// w y - floor(ws y / 2^32) q: in [0, 2q) for every y < 2^32
__device__ __forceinline__ uint32_t shoup_lazy(uint32_t y, Pair32 w, uint32_t q) { return w.w * y - __umulhi(w.s, y) * q; }

__device__ __forceinline__ uint32_t shoup(uint32_t y, Pair32 w, uint32_t q) { return csub(shoup_lazy(y, w, q), q); }

// x mod q for a 64-bit x (SIGNED: two's complement).  k = round(x / q) comes
// from the low word of 1.5 2^52 + x (1/q).  The callers' sums, at most 16 products
// of words below 2^30 and residues, are below 2^34 q, so that it is within 1/2 +
// 2^-17 of x / q (x and 1/q are rounded to 53 bits) and x - k q, taken in 32 bits,
// is the centred residue: eight instructions, where Barrett with a 64-bit product takes about
// sixteen.
template <bool SIGNED = false>
__device__ __forceinline__ uint32_t reduce64(uint64_t x, const Prime32 &P)
{
    const uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    const double d = fma(SIGNED ? (double)(int32_t)hi : (double)hi, 0x1p32, (double)lo);
    const uint32_t k = (uint32_t)__double_as_longlong(fma(d, P.qinv, 0x1.8p52));
    const uint32_t r = lo - k * P.q;
    return min(r, r + P.q);
}

__device__ __forceinline__ uint64_t mul32(uint32_t a, uint32_t b) { return (uint64_t)a * b; }

// The threads of a row share a wave: their exchanges through LDS need its
// order only.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Prime index of a launch's row: prime0 + r below `split`, prime1 + r - split
// from there on (q_0..q_l, then p_0..p_{K-1}).  Formed, not looked up: a byte of
// the argument block is a vector load in front of everything a row needs.
struct RowMap32 {
    uint32_t prime0, split, prime1;
};
__host__ __device__ __forceinline__ uint32_t row_prime32(const RowMap32 &m, uint32_t r)
{
    return r < m.split ? m.prime0 + r : m.prime1 + r - m.split;
}

// ------------------------------------------------------------- NTT passes

// Launch row y = r npoly + poly: polynomial `poly`, row r under prime map(r)
// (the polynomials' limbs of one prime follow each other); rows whose bit
// poly * rows + r is set in skip are left alone.
struct Ntt32Args {
    const uint32_t *src;
    uint32_t *dst;              // pass 0 writes here, pass 1 transforms it in place
    int64_t src_poly_stride, dst_poly_stride;
    uint32_t rows, npoly;
    const Prime32 *primes;
    const Pair32 *tw;           // [n_primes][N]: psi^(+-br(i))
    // last inverse multiplication (N^-1, times a conversion scale) per row r
    Pair32 scale[kMaxRows32];
    // forward epilogue: 0 plain; 1 ModDown out_p = cst (aux_p - x) + add_p; 2 Rescale out_p = cst (aux_p - x)
    uint32_t epi;
    const uint32_t *aux[2];
    const uint32_t *add[2];
    uint32_t *out[2];
    const Pair32 *cst;          // per prime index
    const uint32_t *src2;       // first inverse pass: the input is [src src2]_q (HMult's d2)
    uint32_t galois;            // first inverse pass and ModDown's addend: gathered through X -> X^g (1 = none)
    // first forward pass of Rescale: its input is the centred lift of src (one limb per polynomial,
    // coefficients under ql)
    uint32_t lift_ql;
    uint32_t centred;           // last inverse pass: stores centred signed values (ModDown's conversion)
    uint32_t skip[kMaxLaunch32 / 32];
    RowMap32 map;
};

struct RowPos {
    uint32_t poly, r, pi;
    bool skip;
};

__device__ __forceinline__ RowPos row_pos(const Ntt32Args &a, uint32_t y)
{
    RowPos p;
    p.r = y / a.npoly;
    p.poly = y - p.r * a.npoly;
    p.pi = row_prime32(a.map, p.r);
    const uint32_t bit = p.poly * a.rows + p.r;
    p.skip = (a.skip[bit >> 5] >> (bit & 31)) & 1;
    return p;
}

// Stage k (0..7) of a 256-point transform on element e of block B: the
// butterfly's twiddle is T[(B << k) + (e >> (8 - k))] (B = 1 for the column
// pass, 256 + row for the row pass), its partner e + (128 >> k).
__device__ __forceinline__ Pair32 twk(const Pair32 *T, uint32_t B, int k, uint32_t e)
{
    return T[(B << k) + (e >> (8 - k))];
}

// Four forward (Cooley-Tukey) stages k0..k0+3 on v[i], element e(i) =
// base + stride i, partners i + (8 >> (k - k0)).  Values stay in [0, 4q).
template <class E>
__device__ __forceinline__ void fwd4(uint32_t (&v)[16], const Pair32 *T, uint32_t B, int k0, uint32_t q, E e)
{
    const uint32_t q2 = 2 * q;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int h = 8 >> st;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i & h) continue;
            const Pair32 w = twk(T, B, k0 + st, e(i));
            const uint32_t x = csub(v[i], q2);
            const uint32_t t = shoup_neg(v[i + h], w, q);
            v[i] = x - t;
            v[i + h] = x + q2 + t;
        }
    }
}

// Four inverse (Gentleman-Sande) stages k0, k0-1, .., k0-3, partners i + (1 << st).
// Values stay in [0, 2q).
template <class E>
__device__ __forceinline__ void inv4(uint32_t (&v)[16], const Pair32 *T, uint32_t B, int k0, uint32_t q, E e)
{
    const uint32_t q2 = 2 * q;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int h = 1 << st;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i & h) continue;
            const Pair32 w = twk(T, B, k0 - st, e(i));
            const uint32_t x = v[i], y = v[i + h];
            v[i] = csub(x + y, q2);
            v[i + h] = shoup_lazy(x - y + q2, w, q);
        }
    }
}

constexpr uint32_t kColStride = 33;               // LDS words per matrix row in a column pass (32 + 1)
constexpr uint32_t kRowStride = 256 + 16;         // LDS words per row in a row pass
__device__ __forceinline__ uint32_t rslot(uint32_t e) { return e + (e >> 4); }  // conflict-free both ways

// Forward column pass: 32 columns per workgroup; round 1 on rows s + 16 i,
// round 2 on rows 16 s + i.  LIFT: Rescale's SwitchModulo of the input,
// u - q_l [u > (q_l - 1) / 2] mod q.
template <bool LIFT>
__global__ __launch_bounds__(kT) void k32_fwd_col(Ntt32Args a)
{
    __shared__ uint32_t L[256 * kColStride];
    const RowPos p = row_pos(a, blockIdx.y);
    if (p.skip) return;
    const Prime32 P = a.primes[p.pi];
    const uint32_t q = P.q;
    const Pair32 *T = a.tw + (size_t)p.pi * kN;
    const uint32_t col = threadIdx.x & 31, s = threadIdx.x >> 5, c = blockIdx.x * 32 + col;
    const uint32_t *src = a.src + p.poly * a.src_poly_stride + (LIFT ? 0 : (size_t)p.r * kN);
    uint32_t v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = src[(s + 16 * i) * 256 + c];
    if (LIFT) {
        const uint32_t half = (a.lift_ql - 1) / 2;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int32_t u = (int32_t)(v[i] > half ? v[i] - a.lift_ql : v[i]);
            v[i] = reduce64<true>((uint64_t)(int64_t)u, P);
        }
    }
    fwd4(v, T, 1, 0, q, [&](int i) { return s + 16 * i; });
#pragma unroll
    for (int i = 0; i < 16; ++i) L[(s + 16 * i) * kColStride + col] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = L[(16 * s + i) * kColStride + col];
    fwd4(v, T, 1, 4, q, [&](int i) { return 16 * s + i; });
    uint32_t *dst = a.dst + p.poly * a.dst_poly_stride + (size_t)p.r * kN;
#pragma unroll
    for (int i = 0; i < 16; ++i) dst[(16 * s + i) * 256 + c] = v[i];
}

__device__ __forceinline__ void load16(uint32_t (&v)[16], const uint32_t *m)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint4 x = ((const uint4 *)m)[j];
        v[4 * j] = x.x;
        v[4 * j + 1] = x.y;
        v[4 * j + 2] = x.z;
        v[4 * j + 3] = x.w;
    }
}

__device__ __forceinline__ void store16(uint32_t *m, const uint32_t (&v)[16])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) ((uint4 *)m)[j] = make_uint4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
}

// Forward row pass: 32 rows per workgroup, 16 threads per row: round 1 on e =
// s + 16 i as loaded, round 2 on e = 16 s + i, stored as 16 consecutive words
// per thread (with the epilogue).
__global__ __launch_bounds__(kT) void k32_fwd_row(Ntt32Args a)
{
    __shared__ uint32_t L[32 * kRowStride];
    const RowPos p = row_pos(a, blockIdx.y);
    if (p.skip) return;
    const uint32_t q = a.primes[p.pi].q;
    const Pair32 *T = a.tw + (size_t)p.pi * kN;
    const uint32_t rw = threadIdx.x >> 4, s = threadIdx.x & 15, b = blockIdx.x * 32 + rw;
    uint32_t *m = a.dst + p.poly * a.dst_poly_stride + (size_t)p.r * kN + b * 256;
    uint32_t *Lr = L + rw * kRowStride;
    uint32_t v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = m[s + 16 * i];
    fwd4(v, T, 256 + b, 0, q, [&](int i) { return s + 16 * i; });
#pragma unroll
    for (int i = 0; i < 16; ++i) Lr[rslot(s + 16 * i)] = v[i];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = Lr[rslot(16 * s + i)];
    fwd4(v, T, 256 + b, 4, q, [&](int i) { return 16 * s + i; });
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = csub(csub(v[i], 2 * q), q);
    const size_t off = (size_t)p.r * kN + b * 256 + 16 * s;
    if (a.epi == 0) {
        store16(m + 16 * s, v);
        return;
    }
    const Pair32 c = a.cst[p.pi];
    uint32_t x[16], o[16];
    load16(x, (p.poly ? a.aux[1] : a.aux[0]) + off);
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = shoup(x[i] - v[i] + q, c, q);
    const uint32_t *add = p.poly ? a.add[1] : a.add[0];
    if (a.epi == 1 && add) {
        if (a.galois == 1) {
            load16(x, add + off);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = add[(size_t)p.r * kN + galois_src(b * 256 + 16 * s + i, a.galois, kLogN)];
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] = csub(o[i] + x[i], q);
    }
    store16((p.poly ? a.out[1] : a.out[0]) + off, o);
}

// Inverse row pass: round 1 (stages 7..4) on e = 16 s + i as loaded, round 2
// (stages 3..0) on e = s + 16 i; stored from that layout.  IN_GALOIS gathers
// the input (a block of 256 positions comes from one source block), IN_TENSOR
// forms HMult's d2.
enum Inv32 { IN_PLAIN = 0, IN_GALOIS = 1, IN_TENSOR = 2 };

template <int IN>
__global__ __launch_bounds__(kT) void k32_inv_row(Ntt32Args a)
{
    __shared__ uint32_t L[32 * kRowStride];
    const RowPos p = row_pos(a, blockIdx.y);
    if (p.skip) return;
    const Prime32 P = a.primes[p.pi];
    const uint32_t q = P.q;
    const Pair32 *T = a.tw + (size_t)p.pi * kN;
    const uint32_t rw = threadIdx.x >> 4, s = threadIdx.x & 15, b = blockIdx.x * 32 + rw;
    const size_t off = p.poly * a.src_poly_stride + (size_t)p.r * kN;
    uint32_t *Lr = L + rw * kRowStride;
    uint32_t v[16];
    if (IN == IN_GALOIS) {
        const uint32_t sb = galois_src(b * 256, a.galois, kLogN) & ~255u;
        load16(v, a.src + off + sb + 16 * s);
#pragma unroll
        for (int i = 0; i < 16; ++i) Lr[rslot(16 * s + i)] = v[i];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = Lr[rslot(galois_src(b * 256 + 16 * s + i, a.galois, kLogN) - sb)];
        wave_sync();
    } else {
        load16(v, a.src + off + b * 256 + 16 * s);
        if (IN == IN_TENSOR) {
            uint32_t y[16];
            load16(y, a.src2 + off + b * 256 + 16 * s);
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = reduce64(mul32(v[i], y[i]), P);
        }
    }
    inv4(v, T, 256 + b, 7, q, [&](int i) { return 16 * s + i; });
#pragma unroll
    for (int i = 0; i < 16; ++i) Lr[rslot(16 * s + i)] = v[i];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = Lr[rslot(s + 16 * i)];
    inv4(v, T, 256 + b, 3, q, [&](int i) { return s + 16 * i; });
    uint32_t *d = a.dst + p.poly * a.dst_poly_stride + (size_t)p.r * kN + b * 256;
#pragma unroll
    for (int i = 0; i < 16; ++i) d[s + 16 * i] = v[i];
}

// Inverse column pass: round 1 (stages 7..4) on rows 16 s + i, round 2 (3..0)
// on rows s + 16 i, then the last multiplication (N^-1 and the row's scale).
__global__ __launch_bounds__(kT) void k32_inv_col(Ntt32Args a)
{
    __shared__ uint32_t L[256 * kColStride];
    const RowPos p = row_pos(a, blockIdx.y);
    if (p.skip) return;
    const uint32_t q = a.primes[p.pi].q;
    const Pair32 *T = a.tw + (size_t)p.pi * kN;
    const uint32_t col = threadIdx.x & 31, s = threadIdx.x >> 5, c = blockIdx.x * 32 + col;
    uint32_t *d = a.dst + p.poly * a.dst_poly_stride + (size_t)p.r * kN;
    uint32_t v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = d[(16 * s + i) * 256 + c];
    inv4(v, T, 1, 7, q, [&](int i) { return 16 * s + i; });
#pragma unroll
    for (int i = 0; i < 16; ++i) L[(16 * s + i) * kColStride + col] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = L[(s + 16 * i) * kColStride + col];
    inv4(v, T, 1, 3, q, [&](int i) { return s + 16 * i; });
    const Pair32 f = a.scale[p.r];
    const uint32_t half = a.centred ? q >> 1 : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t y = shoup(v[i], f, q);
        d[(s + 16 * i) * 256 + c] = y > half ? y - q : y;
    }
}

// ----------------------------------------------------- coefficient kernels

constexpr int kB = 256;

// Fast base conversion (Eq. (1)) of job j = blockIdx.y: y_i = src row i (already
// scaled by [(B/b_i)^-1]_{b_i} in the inverse NTT), out row c = [sum_i y_i [B/b_i]_c]_c
// for the rows c outside [lo, hi), in groups of a.group rows (blockIdx.z).
// ModDown's inputs are centred (CENTRED: signed words, sums below 2^63 over 16
// terms; ModUp's unsigned sums stay below 2^64).  The source count is a template
// parameter, the constants come through the scalar cache, and a thread takes two
// coefficients: a term is one multiply-add, a reduction eight instructions, and
// the rows' stores are what is left (4 digits of 13 rows into 47 each: 63 us
// with the counts at run time and one coefficient per thread, 22 us so).
struct Bconv32Job {
    const uint32_t *src;
    uint32_t *dst;
    const uint32_t *hmod;       // [prime][kMaxDigit32]: [B/b_i]_{prime}
    uint32_t ns, lo, hi, pad;
};

struct Bconv32Args {
    Bconv32Job job[kMaxDigit32];
    const Prime32 *primes;
    uint32_t nrows, group;      // output rows, and how many of them a workgroup takes
    RowMap32 map;
};

typedef const __attribute__((address_space(4))) uint32_t Const32;

// A target row's constants in scalar registers.
template <int NS>
struct ConvRow32 {
    Prime32 P;
    uint32_t h[NS];
};

template <int NS>
__device__ __forceinline__ ConvRow32<NS> conv_row32(const Bconv32Args &a, const Bconv32Job &J, uint32_t r)
{
    const uint32_t pi = row_prime32(a.map, r);
    Const32 *w = (Const32 *)(a.primes + pi), *h = (Const32 *)(J.hmod + (size_t)pi * kMaxDigit32);
    ConvRow32<NS> c;
    c.P.q = w[0];
    c.P.pad = 0;
    c.P.qinv = __hiloint2double((int)w[3], (int)w[2]);
#pragma unroll
    for (int i = 0; i < NS; ++i) c.h[i] = h[i];
    return c;
}

// s + y c, y and c signed (the compiler widens one of two such products to 64 bits)
__device__ __forceinline__ uint64_t mad_signed(uint32_t y, uint32_t c, uint64_t s)
{
    uint64_t k;
    asm("v_mad_i64_i32 %0, %1, %2, %3, %0" : "+v"(s), "=s"(k) : "v"(y), "s"(c));
    return s;
}

template <bool CENTRED, int NS>
__device__ __forceinline__ void bconv32_rows(const Bconv32Args &a, const Bconv32Job &J, uint32_t n, uint32_t r0)
{
    uint2 y[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) y[i] = *(const uint2 *)(J.src + (size_t)i * kN + n);
    const uint32_t r1 = min(r0 + a.group, a.nrows);
    auto next = [&](uint32_t r) { return r >= J.lo && r < J.hi ? J.hi : r; };  // rows [lo, hi) are the sources
    uint32_t r = next(r0);
    if (r >= r1) return;
    ConvRow32<NS> c = conv_row32<NS>(a, J, r);
    while (r < r1) {
        // the next row's constants are on their way while this one is summed
        const uint32_t rn = next(r + 1);
        const ConvRow32<NS> cn = conv_row32<NS>(a, J, min(rn, r1 - 1));
        uint64_t s0 = 0, s1 = 0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            s0 = CENTRED ? mad_signed(y[i].x, c.h[i], s0) : s0 + mul32(y[i].x, c.h[i]);
            s1 = CENTRED ? mad_signed(y[i].y, c.h[i], s1) : s1 + mul32(y[i].y, c.h[i]);
        }
        *(uint2 *)(J.dst + (size_t)r * kN + n) = make_uint2(reduce64<CENTRED>(s0, c.P), reduce64<CENTRED>(s1, c.P));
        r = rn;
        c = cn;
    }
}

template <bool CENTRED>
__global__ __launch_bounds__(kB) void k32_bconv(Bconv32Args a)
{
    const Bconv32Job &J = a.job[blockIdx.y];
    const uint32_t n = 2 * (blockIdx.x * kB + threadIdx.x), r0 = blockIdx.z * a.group;
    if (r0 >= a.nrows) return;
    switch (J.ns) {
#define BC32(k) \
    case k: bconv32_rows<CENTRED, k>(a, J, n, r0); break;
        BC32(1) BC32(2) BC32(3) BC32(4) BC32(5) BC32(6) BC32(7) BC32(8)
        BC32(9) BC32(10) BC32(11) BC32(12) BC32(13) BC32(14) BC32(15) BC32(16)
#undef BC32
    default: break;
    }
}

// Key inner product: acc_t[r] = sum_j x_j[r] key[j][t][prime(r)], x_j[r] = d[r]
// for the digit's own rows (d at level l, evaluation domain, gathered through X
// -> X^galois), ext_j[r] else.  HMult (ta0 set): d = a1 b1 is formed here, and
// rows q_0..q_l also take [P]_q d0 and [P]_q d1 (d0 = a0 b0, d1 = a0 b1 + a1 b0),
// so that ModDown's P^-1 (acc - Conv) leaves KS(d2) + (d0, d1).
struct Ip32Args {
    const uint32_t *ext, *d, *key;
    uint32_t *acc;
    const Prime32 *primes;
    const uint32_t *ta0, *ta1, *tb0, *tb1, *pmod;
    uint32_t beta, rows, n, alpha, krows, galois;
    RowMap32 map;
};

template <bool TENSOR>
__global__ __launch_bounds__(kB) void k32_inner_product(Ip32Args a)
{
    const uint32_t n = blockIdx.x * kB + threadIdx.x, r = blockIdx.y, pi = row_prime32(a.map, r);
    const Prime32 P = a.primes[pi];
    const bool qrow = r < a.n;
    uint32_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    if (TENSOR && qrow) {
        const size_t i = (size_t)r * kN + n;
        a0 = a.ta0[i], a1 = a.ta1[i], b0 = a.tb0[i], b1 = a.tb1[i];
    }
    uint64_t s0 = 0, s1 = 0;
#pragma unroll 4
    for (uint32_t j = 0; j < a.beta; ++j) {
        const bool own = qrow && r >= j * a.alpha && r < j * a.alpha + a.alpha;
        const uint32_t k0 = a.key[(((size_t)j * 2 + 0) * a.krows + pi) * kN + n];
        const uint32_t k1 = a.key[(((size_t)j * 2 + 1) * a.krows + pi) * kN + n];
        uint32_t x;
        if (!own) x = a.ext[((size_t)j * a.rows + r) * kN + n];
        else if (TENSOR) x = reduce64(mul32(a1, b1), P);
        else x = a.d[(size_t)r * kN + (a.galois == 1 ? n : galois_src(n, a.galois, kLogN))];
        s0 += mul32(x, k0);
        s1 += mul32(x, k1);
    }
    if (TENSOR && qrow) {
        // one term more: 16 in all at most, since beta (l + 1 + K) <= kMaxLaunch32 keeps beta below 16
        const uint32_t pm = a.pmod[pi];
        s0 += mul32(reduce64(mul32(a0, b0), P), pm);
        s1 += mul32(reduce64(mul32(a0, b1) + mul32(a1, b0), P), pm);
    }
    a.acc[(size_t)r * kN + n] = reduce64(s0, P);
    a.acc[((size_t)a.rows + r) * kN + n] = reduce64(s1, P);
}

// out[limb][e] = in[limb][src of e under X -> X^g] (evaluation domain), for a
// rotation whose outputs overlap c0
__global__ __launch_bounds__(kB) void k32_automorph(const uint32_t *in, uint32_t *out, uint32_t g)
{
    const uint32_t e = blockIdx.x * kB + threadIdx.x;
    const size_t row = (size_t)blockIdx.y * kN;
    out[row + e] = in[row + galois_src(e, g, kLogN)];
}

}  // namespace

// --------------------------------------------------------------- host side

struct ckks32_ctx {
    int device = 0;
    uint32_t nq = 0, np = 0, dnum = 0, alpha = 0;
    std::vector<uint32_t> primes;  // q_0..q_L, p_0..p_{K-1}
    void *dev = nullptr;
    Prime32 *d_primes = nullptr;
    Pair32 *d_tw_fwd = nullptr, *d_tw_inv = nullptr;
    uint32_t *d_hmod = nullptr;    // [nsets][n_primes][kMaxDigit32]
    uint32_t *d_pmod = nullptr;    // [n_primes]: P mod prime
    Pair32 *d_pinv = nullptr;      // [n_primes]: P^-1 mod q_i
    Pair32 *d_qlinv = nullptr;     // [nq][nq]: (l, i) -> q_l^-1 mod q_i
    // host copies of per-set constants
    std::vector<Pair32> ys;        // [nsets][kMaxDigit32]: N^-1 [(B/b_i)^-1]_{b_i}
    std::vector<Pair32> ninv;      // [n_primes]
    std::vector<Pair32> qlinv;     // [nq][nq]
    uint32_t nsets = 0;
    uint32_t set_index(uint32_t digit, uint32_t size) const { return digit * alpha + size - 1; }
    uint32_t pset() const { return dnum * alpha; }
};

namespace {

#define TRY32(x)                        \
    do {                                \
        ckks_status _s = (x);           \
        if (_s != CKKS_OK) return _s;   \
    } while (0)

Pair32 pair32(uint64_t w, uint64_t q)
{
    Pair32 p;
    p.w = (uint32_t)w;
    p.s = (uint32_t)((w << 32) / q);
    return p;
}

ckks_status dev32(hipError_t e, const char *what)
{
    if (e == hipSuccess) return CKKS_OK;
    return fail(CKKS_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Sizes32 {
    uint32_t n, rows, beta;
};

Sizes32 sizes(const ckks32_ctx *c, uint32_t level)
{
    Sizes32 s;
    s.n = level + 1;
    s.rows = s.n + c->np;
    s.beta = (s.n + c->alpha - 1) / c->alpha;
    return s;
}

// rows of an extended polynomial at `level`; n rows from prime `first` on
RowMap32 ext_map(const ckks32_ctx *c, uint32_t level) { return RowMap32{0, level + 1, c->nq}; }
RowMap32 plain_map(uint32_t first) { return RowMap32{first, 0xFFFFFFFFu, 0}; }

Ntt32Args base_args(const ckks32_ctx *c, bool inverse)
{
    Ntt32Args a;
    memset(&a, 0, sizeof(a));
    a.primes = c->d_primes;
    a.tw = inverse ? c->d_tw_inv : c->d_tw_fwd;
    a.galois = 1;
    return a;
}

hipError_t launch_ntt32(const Ntt32Args &a, bool inverse, hipStream_t st)
{
    const uint32_t ny = a.npoly * a.rows;
    if (ny == 0) return hipSuccess;
    if (ny > kMaxLaunch32 || a.rows > kMaxRows32) return hipErrorInvalidValue;
    const dim3 grid(8, ny), block(kT);
    if (inverse) {
        if (a.src2) hipLaunchKernelGGL(k32_inv_row<IN_TENSOR>, grid, block, 0, st, a);
        else if (a.galois != 1) hipLaunchKernelGGL(k32_inv_row<IN_GALOIS>, grid, block, 0, st, a);
        else hipLaunchKernelGGL(k32_inv_row<IN_PLAIN>, grid, block, 0, st, a);
        hipLaunchKernelGGL(k32_inv_col, grid, block, 0, st, a);
    } else {
        if (a.lift_ql) hipLaunchKernelGGL(k32_fwd_col<true>, grid, block, 0, st, a);
        else hipLaunchKernelGGL(k32_fwd_col<false>, grid, block, 0, st, a);
        hipLaunchKernelGGL(k32_fwd_row, grid, block, 0, st, a);
    }
    return hipGetLastError();
}

ckks_status check_ptr32(const void *p, const char *what)
{
    if (!p || ((uintptr_t)p & 15)) return fail(CKKS_E_ARG, std::string(what) + ": null or not 16-byte aligned");
    return CKKS_OK;
}

// whether [a, a + bytes) and [b, b + bytes) overlap
bool overlap32(const void *a, const void *b, size_t bytes)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + bytes && y < x + bytes;
}

// Workspace layout of a key switch at `level` (words): dc [n], ext [beta][rows],
// acc [2][rows], pc [2][K], conv [2][n].
struct Ws32 {
    uint32_t *dc, *ext, *acc, *pc, *conv;
};

size_t ks_words(const ckks32_ctx *c, uint32_t level)
{
    const Sizes32 s = sizes(c, level);
    return ((size_t)s.n + (size_t)s.beta * s.rows + 2 * (size_t)s.rows + 2 * (size_t)c->np + 2 * (size_t)s.n) * kN;
}

size_t ks_bytes(const ckks32_ctx *c, uint32_t level) { return align256(ks_words(c, level) * 4); }

Ws32 ks_ws(const ckks32_ctx *c, uint32_t level, void *ws)
{
    const Sizes32 s = sizes(c, level);
    Ws32 w;
    w.dc = (uint32_t *)ws;
    w.ext = w.dc + (size_t)s.n * kN;
    w.acc = w.ext + (size_t)s.beta * s.rows * kN;
    w.pc = w.acc + 2 * (size_t)s.rows * kN;
    w.conv = w.pc + 2 * (size_t)c->np * kN;
    return w;
}

constexpr uint32_t kConvGroups32 = 2048;
// Rows per workgroup: as many as leave 2,048 workgroups, eight per CU.  Flat around that: the two
// conversions of a key switch at l = 51 take 36, 35, 34 and 36 us for 1,024, 2,048, 4,096 and 8,192
// workgroups, those at l = 24 15, 15, 17 and 22 us (their stores, 49 and 14 MB, are most of it).
hipError_t launch_bconv32(Bconv32Args &a, uint32_t njobs, bool centred, hipStream_t st)
{
    static_assert(sizeof(Bconv32Args) <= 4096, "the conversion's argument block is a kernel argument");
    const uint32_t want = std::max(1u, kConvGroups32 / (kN / (2 * kB) * njobs));
    a.group = (a.nrows + want - 1) / want;
    const dim3 grid(kN / (2 * kB), njobs, (a.nrows + a.group - 1) / a.group);
    if (centred) hipLaunchKernelGGL(k32_bconv<true>, grid, dim3(kB), 0, st, a);
    else hipLaunchKernelGGL(k32_bconv<false>, grid, dim3(kB), 0, st, a);
    return hipGetLastError();
}

// HMult's operands, whose product a1 b1 is key-switched.
struct Tensor32 {
    const uint32_t *a0, *a1, *b0, *b1;
};

// ModUp of phi_g(d), or of a1 b1 with tin (evaluation domain, level l), into ext
// (evaluation domain, the digits' own rows left out: the inner product reads or
// forms them).
hipError_t modup32(const ckks32_ctx *c, const uint32_t *d, uint32_t g, const Tensor32 *tin, uint32_t level, const Ws32 &w,
                   hipStream_t st)
{
    const Sizes32 s = sizes(c, level);
    Ntt32Args ia = base_args(c, true);
    ia.src = tin ? tin->a1 : d;
    ia.src2 = tin ? tin->b1 : nullptr;
    ia.galois = g;
    ia.dst = w.dc;
    ia.rows = s.n;
    ia.npoly = 1;
    ia.map = plain_map(0);
    for (uint32_t i = 0; i < s.n; ++i) {
        const uint32_t j = i / c->alpha, lo = j * c->alpha, hi = std::min(lo + c->alpha, s.n);
        ia.scale[i] = c->ys[(size_t)c->set_index(j, hi - lo) * kMaxDigit32 + (i - lo)];
    }
    hipError_t e = launch_ntt32(ia, true, st);
    if (e != hipSuccess) return e;
    Bconv32Args bh;
    memset(&bh, 0, sizeof(bh));
    bh.primes = c->d_primes;
    bh.nrows = s.rows;
    const size_t hstride = (size_t)(c->nq + c->np) * kMaxDigit32;
    bh.map = ext_map(c, level);
    for (uint32_t j = 0; j < s.beta; ++j) {
        const uint32_t lo = j * c->alpha, hi = std::min(lo + c->alpha, s.n);
        Bconv32Job &J = bh.job[j];
        J.src = w.dc + (size_t)lo * kN;
        J.dst = w.ext + (size_t)j * s.rows * kN;
        J.hmod = c->d_hmod + (size_t)c->set_index(j, hi - lo) * hstride;
        J.ns = hi - lo;
        J.lo = lo;
        J.hi = hi;
    }
    e = launch_bconv32(bh, s.beta, false, st);
    if (e != hipSuccess) return e;
    Ntt32Args fa = base_args(c, false);
    fa.src = fa.dst = w.ext;
    fa.src_poly_stride = fa.dst_poly_stride = (int64_t)s.rows * kN;
    fa.rows = s.rows;
    fa.npoly = s.beta;
    fa.map = ext_map(c, level);
    for (uint32_t j = 0; j < s.beta; ++j)
        for (uint32_t r = j * c->alpha; r < std::min(j * c->alpha + c->alpha, s.n); ++r) {
            const uint32_t y = j * s.rows + r;
            fa.skip[y >> 5] |= 1u << (y & 31);
        }
    return launch_ntt32(fa, false, st);
}

// ModDown of the pair acc [2][rows] into out_t = P^-1 (acc_t - Conv(acc_t|P)) + phi_g(add_t).
hipError_t moddown32(const ckks32_ctx *c, const uint32_t *acc, uint32_t level, const Ws32 &w, uint32_t *out0,
                     uint32_t *out1, const uint32_t *add0, uint32_t g, hipStream_t st)
{
    const Sizes32 s = sizes(c, level);
    const uint32_t K = c->np;
    Ntt32Args ia = base_args(c, true);
    ia.src = acc + (size_t)s.n * kN;
    ia.dst = w.pc;
    ia.src_poly_stride = (int64_t)s.rows * kN;
    ia.dst_poly_stride = (int64_t)K * kN;
    ia.rows = K;
    ia.npoly = 2;
    ia.centred = 1;
    ia.map = plain_map(c->nq);
    for (uint32_t k = 0; k < K; ++k) {
        ia.scale[k] = c->ys[(size_t)c->pset() * kMaxDigit32 + k];
    }
    hipError_t e = launch_ntt32(ia, true, st);
    if (e != hipSuccess) return e;
    Bconv32Args bh;
    memset(&bh, 0, sizeof(bh));
    bh.primes = c->d_primes;
    bh.nrows = s.n;
    bh.map = plain_map(0);
    const size_t hstride = (size_t)(c->nq + c->np) * kMaxDigit32;
    for (uint32_t t = 0; t < 2; ++t) {
        Bconv32Job &J = bh.job[t];
        J.src = w.pc + (size_t)t * K * kN;
        J.dst = w.conv + (size_t)t * s.n * kN;
        J.hmod = c->d_hmod + (size_t)c->pset() * hstride;
        J.ns = K;
        J.lo = J.hi = 0xFFFFFFFFu;
    }
    e = launch_bconv32(bh, 2, true, st);
    if (e != hipSuccess) return e;
    Ntt32Args fa = base_args(c, false);
    fa.src = fa.dst = w.conv;
    fa.src_poly_stride = fa.dst_poly_stride = (int64_t)s.n * kN;
    fa.rows = s.n;
    fa.npoly = 2;
    fa.map = plain_map(0);
    fa.epi = 1;
    fa.aux[0] = acc;
    fa.aux[1] = acc + (size_t)s.rows * kN;
    fa.add[0] = add0;
    fa.galois = g;
    fa.out[0] = out0;
    fa.out[1] = out1;
    fa.cst = c->d_pinv;
    return launch_ntt32(fa, false, st);
}

hipError_t inner_product32(const ckks32_ctx *c, const uint32_t *d, uint32_t g, const Tensor32 *tin, uint32_t level,
                           const uint32_t *key, const Ws32 &w, hipStream_t st)
{
    const Sizes32 s = sizes(c, level);
    Ip32Args a;
    memset(&a, 0, sizeof(a));
    a.ext = w.ext;
    a.d = d;
    a.key = key;
    a.acc = w.acc;
    a.primes = c->d_primes;
    a.beta = s.beta;
    a.rows = s.rows;
    a.n = s.n;
    a.alpha = c->alpha;
    a.krows = c->nq + c->np;
    a.galois = g;
    a.pmod = c->d_pmod;
    a.map = ext_map(c, level);
    const dim3 grid(kN / kB, s.rows), block(kB);
    if (tin) {
        a.ta0 = tin->a0, a.ta1 = tin->a1, a.tb0 = tin->b0, a.tb1 = tin->b1;
        hipLaunchKernelGGL(k32_inner_product<true>, grid, block, 0, st, a);
    } else {
        hipLaunchKernelGGL(k32_inner_product<false>, grid, block, 0, st, a);
    }
    return hipGetLastError();
}

// out_t = KS_t + phi_g_add(add_t) with KS the key switch of phi_g(d), or with tin
// the relinearised product (d, add0 null, g = 1); add_1 = 0.  With g_add other than
// 1 the outputs may not overlap add0: its blocks are gathered as they are written.
hipError_t keyswitch32(ckks32_ctx *c, const uint32_t *d, uint32_t g, const Tensor32 *tin, uint32_t level,
                       const uint32_t *key, uint32_t *out0, uint32_t *out1, const uint32_t *add0, uint32_t g_add, void *ws,
                       hipStream_t st)
{
    const Ws32 w = ks_ws(c, level, ws);
    hipError_t e = modup32(c, d, g, tin, level, w, st);
    if (e == hipSuccess) e = inner_product32(c, d, g, tin, level, key, w, st);
    if (e == hipSuccess) e = moddown32(c, w.acc, level, w, out0, out1, add0, g_add, st);
    return e;
}

ckks_status check_ctx32(const ckks32_ctx *c, uint32_t level)
{
    if (!c) return fail(CKKS_E_ARG, "ckks32: null context");
    if (level >= c->nq) return fail(CKKS_E_LEVEL, "ckks32: level " + std::to_string(level) + " out of range");
    return CKKS_OK;
}

}  // namespace

extern "C" ckks_status ckks32_ctx_create(uint32_t log_n, const uint32_t *q, uint32_t n_q, const uint32_t *p,
                                         uint32_t n_p, uint32_t dnum, int hip_device, ckks32_ctx **out)
{
    if (!out || !q || !p) return fail(CKKS_E_ARG, "ckks32_ctx_create: null pointer");
    *out = nullptr;
    if (log_n != kLogN) return fail(CKKS_E_UNSUPPORTED, "ckks32_ctx_create: log_n must be 16");
    if (n_q < 1 || n_p < 1 || dnum < 1 || dnum > n_q)
        return fail(CKKS_E_ARG, "ckks32_ctx_create: need n_q >= 1, n_p >= 1, 1 <= dnum <= n_q");
    const uint32_t alpha = (n_q + dnum - 1) / dnum;
    if (n_q + n_p > kMaxPrimes32 || alpha > kMaxDigit32 || n_p > kMaxDigit32 || dnum > kMaxDigit32 ||
        n_q + n_p > kMaxRows32)
        return fail(CKKS_E_UNSUPPORTED, "ckks32_ctx_create: at most 64 primes, 16 per digit, 16 special, 16 digits");
    std::vector<uint32_t> primes(q, q + n_q);
    primes.insert(primes.end(), p, p + n_p);
    const uint64_t N = kN, two_n = 2 * N;
    for (size_t i = 0; i < primes.size(); ++i) {
        const uint64_t m = primes[i];
        if (m >= kQBound || m % two_n != 1 || !probably_prime(m))
            return fail(CKKS_E_ARG, "ckks32_ctx_create: prime " + std::to_string(i) +
                                        " is not a prime below 2^30 congruent to 1 mod 2N");
        for (size_t k = 0; k < i; ++k)
            if (primes[k] == m) return fail(CKKS_E_ARG, "ckks32_ctx_create: primes must be distinct");
    }
    if (hipSetDevice(hip_device) != hipSuccess) return fail(CKKS_E_DEVICE, "ckks32_ctx_create: hipSetDevice failed");
    ckks32_ctx *c = new ckks32_ctx();
    c->device = hip_device;
    c->nq = n_q;
    c->np = n_p;
    c->dnum = dnum;
    c->alpha = alpha;
    c->primes = primes;
    const uint32_t np_all = n_q + n_p;
    c->nsets = dnum * alpha + 1;

    std::vector<Prime32> pr(np_all);
    std::vector<Pair32> twf((size_t)np_all * N), twi((size_t)np_all * N);
    c->ninv.resize(np_all);
    for (uint32_t i = 0; i < np_all; ++i) {
        const uint64_t m = primes[i];
        pr[i].q = (uint32_t)m;
        pr[i].pad = 0;
        pr[i].qinv = 1.0 / (double)m;
        const uint64_t psi = smallest_2n_root(m, two_n), psi_inv = inv_mod(psi, m);
        uint64_t a = 1, b = 1;
        std::vector<uint64_t> pw(N), pwi(N);
        for (uint64_t k = 0; k < N; ++k, a = mul_mod(a, psi, m), b = mul_mod(b, psi_inv, m)) {
            pw[k] = a;
            pwi[k] = b;
        }
        for (uint32_t k = 0; k < N; ++k) {
            const uint32_t e = reverse_bits(k, kLogN);
            twf[(size_t)i * N + k] = pair32(pw[e], m);
            twi[(size_t)i * N + k] = pair32(pwi[e], m);
        }
        c->ninv[i] = pair32(inv_mod(N % m, m), m);
    }
    // conversion constants: digit sets (j, size) and the special basis
    std::vector<uint32_t> hmod((size_t)c->nsets * np_all * kMaxDigit32, 0);
    c->ys.assign((size_t)c->nsets * kMaxDigit32, Pair32{0, 0});
    auto fill_set = [&](uint32_t set, const std::vector<uint32_t> &src) {
        for (size_t i = 0; i < src.size(); ++i) {
            const uint64_t bi = primes[src[i]];
            uint64_t hat_i = 1;  // (B / b_i) mod b_i
            for (size_t k = 0; k < src.size(); ++k)
                if (k != i) hat_i = mul_mod(hat_i, primes[src[k]] % bi, bi);
            const uint64_t y = mul_mod(inv_mod(hat_i, bi), c->ninv[src[i]].w, bi);
            c->ys[(size_t)set * kMaxDigit32 + i] = pair32(y, bi);
            for (uint32_t t = 0; t < np_all; ++t) {
                const uint64_t qt = primes[t];
                uint64_t h = 1;
                for (size_t k = 0; k < src.size(); ++k)
                    if (k != i) h = mul_mod(h, primes[src[k]] % qt, qt);
                hmod[((size_t)set * np_all + t) * kMaxDigit32 + i] = (uint32_t)h;
            }
        }
    };
    for (uint32_t j = 0; j < dnum; ++j)
        for (uint32_t size = 1; size <= alpha; ++size) {
            if (j * alpha + size > n_q) continue;
            std::vector<uint32_t> src;
            for (uint32_t i = 0; i < size; ++i) src.push_back(j * alpha + i);
            fill_set(c->set_index(j, size), src);
        }
    {
        std::vector<uint32_t> src;
        for (uint32_t k = 0; k < n_p; ++k) src.push_back(n_q + k);
        fill_set(c->pset(), src);
    }
    std::vector<uint32_t> pmod(np_all);
    std::vector<Pair32> pinv(np_all);
    for (uint32_t t = 0; t < np_all; ++t) {
        const uint64_t qt = primes[t];
        uint64_t P = 1;
        for (uint32_t k = 0; k < n_p; ++k) P = mul_mod(P, primes[n_q + k] % qt, qt);
        pmod[t] = (uint32_t)P;
        pinv[t] = t < n_q ? pair32(inv_mod(P, qt), qt) : Pair32{0, 0};
    }
    std::vector<Pair32> qlinv((size_t)n_q * n_q, Pair32{0, 0});
    for (uint32_t l = 1; l < n_q; ++l)
        for (uint32_t i = 0; i < l; ++i) {
            qlinv[(size_t)l * n_q + i] = pair32(inv_mod(primes[l] % primes[i], primes[i]), primes[i]);
        }
    c->qlinv = qlinv;

    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    const size_t o_pr = take(pr.size() * sizeof(Prime32)), o_twf = take(twf.size() * sizeof(Pair32)),
                 o_twi = take(twi.size() * sizeof(Pair32)), o_hm = take(hmod.size() * 4),
                 o_pm = take(pmod.size() * 4), o_pi = take(pinv.size() * sizeof(Pair32)),
                 o_ql = take(qlinv.size() * sizeof(Pair32));
    if (hipMalloc(&c->dev, off) != hipSuccess) {
        delete c;
        return fail(CKKS_E_NOMEM, "ckks32_ctx_create: table allocation failed");
    }
    char *base = (char *)c->dev;
    c->d_primes = (Prime32 *)(base + o_pr);
    c->d_tw_fwd = (Pair32 *)(base + o_twf);
    c->d_tw_inv = (Pair32 *)(base + o_twi);
    c->d_hmod = (uint32_t *)(base + o_hm);
    c->d_pmod = (uint32_t *)(base + o_pm);
    c->d_pinv = (Pair32 *)(base + o_pi);
    c->d_qlinv = (Pair32 *)(base + o_ql);
    hipError_t e = hipMemcpy(c->d_primes, pr.data(), pr.size() * sizeof(Prime32), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_tw_fwd, twf.data(), twf.size() * sizeof(Pair32), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_tw_inv, twi.data(), twi.size() * sizeof(Pair32), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_hmod, hmod.data(), hmod.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_pmod, pmod.data(), pmod.size() * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_pinv, pinv.data(), pinv.size() * sizeof(Pair32), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(c->d_qlinv, qlinv.data(), qlinv.size() * sizeof(Pair32), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(c->dev);
        delete c;
        return fail(CKKS_E_DEVICE, "ckks32_ctx_create: table upload failed");
    }
    *out = c;
    return CKKS_OK;
}

extern "C" void ckks32_ctx_destroy(ckks32_ctx *c)
{
    if (!c) return;
    if (c->dev) {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(c->device);
        (void)hipFree(c->dev);
        (void)hipSetDevice(cur);
    }
    delete c;
}

extern "C" size_t ckks32_workspace_bytes(const ckks32_ctx *c, uint32_t op, uint32_t level)
{
    if (!c || level >= c->nq) return 0;
    const size_t n = level + 1;
    switch (op) {
    case CKKS_OP_KEYSWITCH: return ks_bytes(c, level);
    case CKKS_OP_HMULT:  // as ROTATE, whose rows behind the key switch's hold phi_g(c0) in place
    case CKKS_OP_ROTATE: return ks_bytes(c, level) + align256(2 * n * kN * 4);
    case CKKS_OP_RESCALE: return (2 + 2 * (size_t)level) * kN * 4;
    default: return 0;
    }
}

static ckks_status ntt32_common(ckks32_ctx *c, uint32_t *poly, uint32_t limb0, uint32_t n_limbs, void *stream,
                                bool inverse)
{
    if (!c) return fail(CKKS_E_ARG, "ckks32_(i)ntt: null context");
    TRY32(check_ptr32(poly, "ckks32_(i)ntt poly"));
    if (n_limbs == 0 || limb0 + n_limbs > c->nq + c->np || n_limbs > kMaxRows32)
        return fail(CKKS_E_ARG, "ckks32_(i)ntt: limb range outside q_0..q_L, p_0..p_{K-1}");
    Ntt32Args a = base_args(c, inverse);
    a.src = a.dst = poly;
    a.rows = n_limbs;
    a.npoly = 1;
    a.map = plain_map(limb0);
    for (uint32_t r = 0; r < n_limbs; ++r) {
        a.scale[r] = c->ninv[limb0 + r];
    }
    return dev32(launch_ntt32(a, inverse, (hipStream_t)stream), inverse ? "ckks32_intt" : "ckks32_ntt");
}

extern "C" ckks_status ckks32_ntt(ckks32_ctx *c, uint32_t *poly, uint32_t limb0, uint32_t n_limbs, void *stream)
{
    return ntt32_common(c, poly, limb0, n_limbs, stream, false);
}

extern "C" ckks_status ckks32_intt(ckks32_ctx *c, uint32_t *poly, uint32_t limb0, uint32_t n_limbs, void *stream)
{
    return ntt32_common(c, poly, limb0, n_limbs, stream, true);
}

extern "C" ckks_status ckks32_modup(ckks32_ctx *c, const uint32_t *d, uint32_t level, uint32_t *ext, void *ws,
                                    void *stream)
{
    TRY32(check_ctx32(c, level));
    TRY32(check_ptr32(d, "ckks32_modup d"));
    TRY32(check_ptr32(ext, "ckks32_modup ext"));
    TRY32(check_ptr32(ws, "ckks32_modup ws"));
    const hipStream_t st = (hipStream_t)stream;
    const Sizes32 s = sizes(c, level);
    Ws32 w = ks_ws(c, level, ws);
    w.ext = ext;  // the caller's buffer: its own rows are copied from d afterwards
    hipError_t e = modup32(c, d, 1, nullptr, level, w, st);
    for (uint32_t j = 0; j < s.beta && e == hipSuccess; ++j) {
        const uint32_t lo = j * c->alpha, hi = std::min(lo + c->alpha, s.n);
        e = hipMemcpyAsync(ext + ((size_t)j * s.rows + lo) * kN, d + (size_t)lo * kN, (size_t)(hi - lo) * kN * 4,
                           hipMemcpyDeviceToDevice, st);
    }
    return dev32(e, "ckks32_modup");
}

extern "C" ckks_status ckks32_moddown(ckks32_ctx *c, const uint32_t *x, uint32_t level, uint32_t *out0,
                                      uint32_t *out1, void *ws, void *stream)
{
    TRY32(check_ctx32(c, level));
    TRY32(check_ptr32(x, "ckks32_moddown x"));
    TRY32(check_ptr32(out0, "ckks32_moddown out0"));
    TRY32(check_ptr32(out1, "ckks32_moddown out1"));
    TRY32(check_ptr32(ws, "ckks32_moddown ws"));
    const hipStream_t st = (hipStream_t)stream;
    const Ws32 w = ks_ws(c, level, ws);
    return dev32(moddown32(c, x, level, w, out0, out1, nullptr, 1, st), "ckks32_moddown");
}

extern "C" ckks_status ckks32_keyswitch(ckks32_ctx *c, const uint32_t *d, uint32_t level, const uint32_t *key,
                                        uint32_t *out0, uint32_t *out1, void *ws, void *stream)
{
    TRY32(check_ctx32(c, level));
    TRY32(check_ptr32(d, "ckks32_keyswitch d"));
    TRY32(check_ptr32(key, "ckks32_keyswitch key"));
    TRY32(check_ptr32(out0, "ckks32_keyswitch out0"));
    TRY32(check_ptr32(out1, "ckks32_keyswitch out1"));
    TRY32(check_ptr32(ws, "ckks32_keyswitch ws"));
    return dev32(keyswitch32(c, d, 1, nullptr, level, key, out0, out1, nullptr, 1, ws, (hipStream_t)stream),
                 "ckks32_keyswitch");
}

extern "C" ckks_status ckks32_hmult_relin(ckks32_ctx *c, const uint32_t *a0, const uint32_t *a1, const uint32_t *b0,
                                          const uint32_t *b1, uint32_t level, const uint32_t *rlk, uint32_t *out0,
                                          uint32_t *out1, void *ws, void *stream)
{
    TRY32(check_ctx32(c, level));
    const void *ptrs[] = {a0, a1, b0, b1, rlk, out0, out1, ws};
    for (const void *q : ptrs) TRY32(check_ptr32(q, "ckks32_hmult_relin"));
    const Tensor32 tin = {a0, a1, b0, b1};
    const hipError_t e = keyswitch32(c, nullptr, 1, &tin, level, rlk, out0, out1, nullptr, 1, ws, (hipStream_t)stream);
    return dev32(e, "ckks32_hmult_relin");
}

extern "C" ckks_status ckks32_apply_galois(ckks32_ctx *c, const uint32_t *c0, const uint32_t *c1, uint32_t level,
                                           uint32_t galois, const uint32_t *key, uint32_t *out0, uint32_t *out1,
                                           void *ws, void *stream)
{
    TRY32(check_ctx32(c, level));
    const void *ptrs[] = {c0, c1, key, out0, out1, ws};
    for (const void *q : ptrs) TRY32(check_ptr32(q, "ckks32_apply_galois"));
    if (galois % 2 == 0 || galois >= 2 * kN) return fail(CKKS_E_ARG, "ckks32_apply_galois: galois must be odd, below 2N");
    const hipStream_t st = (hipStream_t)stream;
    const size_t bytes = (size_t)(level + 1) * kN * 4;
    const uint32_t *add = c0;
    uint32_t g_add = galois;
    hipError_t e = hipSuccess;
    // c1 is read out before the last launch, which writes the outputs, but c0 is gathered by it: where an
    // output overlaps c0, phi_g(c0) goes to the workspace behind the key switch's first
    if (overlap32(c0, out0, bytes) || overlap32(c0, out1, bytes)) {
        uint32_t *g0 = (uint32_t *)((char *)ws + ks_bytes(c, level));
        hipLaunchKernelGGL(k32_automorph, dim3(kN / kB, level + 1), dim3(kB), 0, st, c0, g0, galois);
        e = hipGetLastError();
        add = g0;
        g_add = 1;
    }
    if (e == hipSuccess) e = keyswitch32(c, c1, galois, nullptr, level, key, out0, out1, add, g_add, ws, st);
    return dev32(e, "ckks32_apply_galois");
}

extern "C" ckks_status ckks32_rescale(ckks32_ctx *c, const uint32_t *c0, const uint32_t *c1, uint32_t level,
                                      uint32_t *out0, uint32_t *out1, void *ws, void *stream)
{
    TRY32(check_ctx32(c, level));
    if (level < 1) return fail(CKKS_E_LEVEL, "ckks32_rescale: level 0 cannot be rescaled");
    const void *ptrs[] = {c0, c1, out0, out1, ws};
    for (const void *q : ptrs) TRY32(check_ptr32(q, "ckks32_rescale"));
    const hipStream_t st = (hipStream_t)stream;
    const uint32_t l = level;
    uint32_t *v = (uint32_t *)ws, *lift = v + 2 * (size_t)kN;
    // v_t = INTT_{q_l}(c_t[l])
    Ntt32Args ia = base_args(c, true);
    ia.src = c0 + (size_t)l * kN;
    ia.src_poly_stride = (int64_t)(c1 - c0);
    ia.dst = v;
    ia.dst_poly_stride = kN;
    ia.rows = 1;
    ia.npoly = 2;
    ia.map = plain_map(l);
    ia.scale[0] = c->ninv[l];
    const hipError_t e = launch_ntt32(ia, true, st);
    if (e != hipSuccess) return dev32(e, "ckks32_rescale");
    Ntt32Args fa = base_args(c, false);
    fa.src = v;
    fa.src_poly_stride = kN;
    fa.lift_ql = c->primes[l];
    fa.dst = lift;
    fa.dst_poly_stride = (int64_t)l * kN;
    fa.rows = l;
    fa.npoly = 2;
    fa.map = plain_map(0);
    fa.epi = 2;
    fa.aux[0] = c0;
    fa.aux[1] = c1;
    fa.out[0] = out0;
    fa.out[1] = out1;
    fa.cst = c->d_qlinv + (size_t)l * c->nq;
    return dev32(launch_ntt32(fa, false, st), "ckks32_rescale");
}
