// Blind rotation + sample extraction with exact negacyclic products by
// double-precision transforms (gfx950), for rings of 1024 and 2048
// coefficients and, at 32-bit words, of 256.
//
// TFHE bootstrapping (ePrint 2018/421, Alg. 3 / Sec. 4): for i = 0..n-1,
//   ACC <- ACC + ExtProd(BSK_i, X^{abar_i} ACC - ACC),
// ExtProd(G, C)_v = sum_{u,p} Dec_p(C_u) * G[u*l+p-1][v] (negacyclic products).
//
// Why it is exact.  A real polynomial mod X^N + 1 is taken as M = N/2 complex
// points a_j + i a_{j+M} mod X^M - i, whose M values are formed by radix-2
// splittings X^{2m} - w^2 = (X^m - w)(X^m + w).  The key words are split into
// balanced limbs (2 of 16 bits at q = 32, 3 of 22 bits at q = 64), each limb's
// spectrum is kept in double precision, and the sums over the 2l digit
// polynomials of every limb are transformed back and rounded to the nearest
// integer.  Those sums are integers of magnitude at most
// S = 2l 2^{bg-1} 2^{b-1} N (b = 16 or 22): 2^33.6 at n = 630, N = 1024,
// l = 3, Bg = 2^7; at most 2^35.6 (q = 32) and 2^41.6 (q = 64) over every
// parameter set a context accepts.  With u = 2^-53, a butterfly with its
// twiddle held as (cos, tan) adds at most 6 u of its output's l2 norm going
// forward and 7 u going back (twiddles accurate to 2 u), so that a transform
// of 10 levels adds 60 u and 70 u, the accumulated products (2l + 2) 1.5 u,
// and every output is within 60 u + 60 u + 96 u + 70 u < 300 u of S (Cauchy-
// Schwarz over the digit and key polynomials): 2^-9 at q = 32 and 2^-3.2 at
// q = 64, below the 1/2 at which rounding would go wrong, for any input.  So
// every rounded value is the integer itself and the output bits are those of
// the schoolbook product.
//
// Transform.  One wave transforms one polynomial with R = M/64 points per
// lane: radix R in registers (uniform twiddles), an exchange through the
// wave's own LDS buffer, radix R again, then the lane bits that are left but
// one come into registers by lane swaps (v_permlane32_swap and
// v_permlane16_swap) for another radix 4 (R = 8) or 2 (R = 16).  The last
// radix-2 level is done by the thread that multiplies: it reads the pair from
// the wave's buffer, so that a thread holds the same two frequencies of all G
// ciphertexts and outputs of its workgroup, and each key value read from
// memory serves G ciphertexts.  The inverse runs the same steps backwards.
// A butterfly is 6 fused multiply-adds (x +- w y with w = c (1 + i t)).
// Published methods used: the folding of a real polynomial mod X^N + 1 into N/2
// complex points (a weighted transform: Crandall and Fagin, "Discrete weighted
// transforms and large-integer arithmetic", Math. Comp. 62, 1994) and twiddles as
// cosine and tangent for fused multiply-adds (Linzer and Feig, "Implementation of
// efficient FFT algorithms on fused multiply-add architectures", IEEE Trans.
// Signal Processing 41, 1993).
//
// Workgroup: G ciphertexts, W waves, W/G polynomials of each at a time; the
// accumulators stay in LDS, natural order, for all n steps.
//
// What it is for: the dense Toeplitz product on the int8 matrix cores ran at
// 72% of their peak but needs 2N (k+1)l N limbs operations where the
// transforms need about 1/100 of them.  Measured, int8 path -> this one,
// identical bits: n = 630, N = 1024, l = 3, q = 32: 1 ciphertext 8.4 -> 2.36 ms,
// 256 30.8 -> 2.38 ms, 1024 50 -> 8.3 ms, 4096 77 -> 27.7 ms; n = 750, N = 2048,
// l = 4, q = 64: 1 ciphertext 34 -> 10.2 ms, 256 158 -> 10.1 ms, 1000 355 -> 40.4 ms.
//
// What bounds it: double-precision vector issue (about 4450 vector
// instructions per ciphertext and step at N = 1024, l = 3, q = 32, 3000 of them
// double precision at 4.3-4.7 cycles of their SIMD; the vector units are 73%
// busy in a launch of 4096) and the LDS exchanges beside it; for one ciphertext
// per workgroup the chain of a step (digits, transform, products, transform
// back, five barriers) and the key reads (64 bytes per cycle and CU: 3100 of
// the 8800 cycles of a step at N = 1024, 12,300 of 32,000 at N = 2048, q = 64,
// l = 4), which find their lines in L2: the workgroups of an XCD ask for a
// step's lines together, each a share, while they transform the step before
// back.  Values of the next step held in registers across its transforms, as
// before that, cost more than the L2 hits do now (B = 1 2.87 ms, against 2.66).
#include <algorithm>
#include <cmath>

#include "fhesql_internal.h"

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));

template <int R>
struct Plan {
    static constexpr int L = R == 8 ? 3 : 4;  // log2 R
    static constexpr int M = 64 * R, N = 128 * R;
    static constexpr int NT2 = R / 2;             // twiddles of a radix-R pass in registers
    static constexpr int NT3 = R == 8 ? 3 : 4;    // twiddles of the swapped levels
    // twiddle table, (cos, tan) entries: second pass [R blocks][NT2], swapped
    // levels [32 lane pairs][NT3], last level [M/2 pairs]
    static constexpr int T3 = R * NT2;
    static constexpr int T4 = T3 + 32 * NT3;
    static constexpr int TN = T4 + M / 2;
};

template <typename T> struct Limb;
template <> struct Limb<uint32_t> {
    static constexpr int BITS = 16, COUNT = 2;
};
template <> struct Limb<uint64_t> {
    static constexpr int BITS = 22, COUNT = 3;
};

// cos and tan of the first pass's angles (turns 1/8, 1/16, 1/32, 5/32, 1/64,
// 9/64, 5/64, 13/64): the root of X^M - i
constexpr double kC1[8] = {0.70710678118654752440, 0.92387953251128675613, 0.98078528040323044913,
                           0.55557023301960222474, 0.99518472667219688624, 0.63439328416364549822,
                           0.88192126434835502971, 0.29028467725446236764};
constexpr double kT1[8] = {1.0, 0.41421356237309504880, 0.19891236737965800691, 1.49660576266548901760,
                           0.09849140335716425308, 1.21850352558797634480, 0.53451113595079164109,
                           3.29655820893832042688};

// (x, y) -> (x + w y, x - w y), w = c (1 + i t), times i when ROT
template <bool ROT>
FHE_DEV void bf_fwd(double& xr, double& xi, double& yr, double& yi, double c, double t) {
    const double a = __builtin_fma(-t, yi, yr), b = __builtin_fma(t, yr, yi);
    const double pr = ROT ? -b : a, pi = ROT ? a : b;
    yr = __builtin_fma(-c, pr, xr);
    yi = __builtin_fma(-c, pi, xi);
    xr = __builtin_fma(c, pr, xr);
    xi = __builtin_fma(c, pi, xi);
}

// (x, y) -> (x + y, conj(w) (x - y))
template <bool ROT>
FHE_DEV void bf_inv(double& xr, double& xi, double& yr, double& yi, double c, double t) {
    const double dr = xr - yr, di = xi - yi;
    xr += yr;
    xi += yi;
    const double pr = c * __builtin_fma(t, di, dr), pi = c * __builtin_fma(-t, dr, di);
    yr = ROT ? pi : pr;
    yi = ROT ? -pr : pi;
}

// Radix-R pass in registers: level m (1..L) pairs indices R >> m apart; block
// b of level m has the path bits b, its twiddle the index below and a factor
// i when the last path bit is set.
template <int R>
FHE_DEV void lane_fwd(double (&re)[R], double (&im)[R], const double* c, const double* t) {
    constexpr int L = Plan<R>::L;
#pragma unroll
    for (int m = 1; m <= L; m++) {
        const int half = R >> m;
#pragma unroll
        for (int b = 0; b < (1 << (m - 1)); b++) {
            const int k = m == 1 ? 0 : (1 << (m - 2)) + (b >> 1);
#pragma unroll
            for (int x = 0; x < half; x++) {
                const int i = 2 * b * half + x, j = i + half;
                if (b & 1) bf_fwd<true>(re[i], im[i], re[j], im[j], c[k], t[k]);
                else bf_fwd<false>(re[i], im[i], re[j], im[j], c[k], t[k]);
            }
        }
    }
}

template <int R>
FHE_DEV void lane_inv(double (&re)[R], double (&im)[R], const double* c, const double* t) {
    constexpr int L = Plan<R>::L;
#pragma unroll
    for (int m = L; m >= 1; m--) {
        const int half = R >> m;
#pragma unroll
        for (int b = 0; b < (1 << (m - 1)); b++) {
            const int k = m == 1 ? 0 : (1 << (m - 2)) + (b >> 1);
#pragma unroll
            for (int x = 0; x < half; x++) {
                const int i = 2 * b * half + x, j = i + half;
                if (b & 1) bf_inv<true>(re[i], im[i], re[j], im[j], c[k], t[k]);
                else bf_inv<false>(re[i], im[i], re[j], im[j], c[k], t[k]);
            }
        }
    }
}

// The first pass (uniform twiddles) backwards, its factors c left to the end:
// a butterfly keeps y / c, two elements of different factors are combined with
// their ratio, and element r has to be multiplied by sc[r] (all constants),
// which the rounding does for nothing.
template <int R>
FHE_DEV void lane_inv_first(double (&re)[R], double (&im)[R], double (&sc)[R]) {
#pragma unroll
    for (int r = 0; r < R; r++) sc[r] = 1.0;
#pragma unroll
    for (int m = Plan<R>::L; m >= 1; m--) {
        const int half = R >> m;
#pragma unroll
        for (int b = 0; b < (1 << (m - 1)); b++) {
            const int k = m == 1 ? 0 : (1 << (m - 2)) + (b >> 1);
#pragma unroll
            for (int x = 0; x < half; x++) {
                const int i = 2 * b * half + x, j = i + half;
                const double q = sc[j] / sc[i], t = kT1[k];
                const double dr = __builtin_fma(-q, re[j], re[i]), di = __builtin_fma(-q, im[j], im[i]);
                re[i] = __builtin_fma(q, re[j], re[i]);
                im[i] = __builtin_fma(q, im[j], im[i]);
                const double pr = __builtin_fma(t, di, dr), pi = __builtin_fma(-t, dr, di);
                re[j] = b & 1 ? pi : pr;
                im[j] = b & 1 ? -pr : pi;
                sc[j] = sc[i] * kC1[k];
            }
        }
    }
}

// x sc to the nearest integer, as the 64-bit difference from kMagic's bits:
// integers below 2^51 end up in the low bits of the sum with 1.5 * 2^52
constexpr double kMagic = 6755399441055744.0;
FHE_DEV uint64_t nearest(double x, double sc) {
    return __builtin_bit_cast(uint64_t, __builtin_fma(x, sc, kMagic)) - __builtin_bit_cast(uint64_t, kMagic);
}

// Exchange lane bit 5 (4) with the register bit that tells a from b.
FHE_DEV void swap32(double& a, double& b) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    a = __builtin_bit_cast(double, u2{lo[0], hi[0]});
    b = __builtin_bit_cast(double, u2{lo[1], hi[1]});
}
FHE_DEV void swap16(double& a, double& b) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    a = __builtin_bit_cast(double, u2{lo[0], hi[0]});
    b = __builtin_bit_cast(double, u2{lo[1], hi[1]});
}

template <int R>
FHE_DEV void lane_swaps(double (&re)[R], double (&im)[R]) {
#pragma unroll
    for (int i = 0; i < R / 2; i++) {
        swap32(re[i], re[i + R / 2]);
        swap32(im[i], im[i + R / 2]);
    }
    if constexpr (R == 8) {
#pragma unroll
        for (int i = 0; i < R; i++)
            if (!(i & 2)) {
                swap16(re[i], re[i + 2]);
                swap16(im[i], im[i + 2]);
            }
    }
}

// The levels after the swaps.  R = 8: register bits (b2, b1, e3), e3 the last
// path bit of the second pass; R = 16: (b1, e2, e3, e4).
template <int R>
FHE_DEV void swapped_fwd(double (&re)[R], double (&im)[R], const double* c, const double* t) {
    if constexpr (R == 8) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (i & 1) bf_fwd<true>(re[i], im[i], re[i + 4], im[i + 4], c[0], t[0]);
            else bf_fwd<false>(re[i], im[i], re[i + 4], im[i + 4], c[0], t[0]);
        }
#pragma unroll
        for (int f = 0; f < 2; f++)
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const int i = 4 * f + e;
                if (f) bf_fwd<true>(re[i], im[i], re[i + 2], im[i + 2], c[1 + e], t[1 + e]);
                else bf_fwd<false>(re[i], im[i], re[i + 2], im[i + 2], c[1 + e], t[1 + e]);
            }
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if (i & 1) bf_fwd<true>(re[i], im[i], re[i + 8], im[i + 8], c[i >> 1], t[i >> 1]);
            else bf_fwd<false>(re[i], im[i], re[i + 8], im[i + 8], c[i >> 1], t[i >> 1]);
        }
    }
}

template <int R>
FHE_DEV void swapped_inv(double (&re)[R], double (&im)[R], const double* c, const double* t) {
    if constexpr (R == 8) {
#pragma unroll
        for (int f = 0; f < 2; f++)
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const int i = 4 * f + e;
                if (f) bf_inv<true>(re[i], im[i], re[i + 2], im[i + 2], c[1 + e], t[1 + e]);
                else bf_inv<false>(re[i], im[i], re[i + 2], im[i + 2], c[1 + e], t[1 + e]);
            }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (i & 1) bf_inv<true>(re[i], im[i], re[i + 4], im[i + 4], c[0], t[0]);
            else bf_inv<false>(re[i], im[i], re[i + 4], im[i + 4], c[0], t[0]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if (i & 1) bf_inv<true>(re[i], im[i], re[i + 8], im[i + 8], c[i >> 1], t[i >> 1]);
            else bf_inv<false>(re[i], im[i], re[i + 8], im[i + 8], c[i >> 1], t[i >> 1]);
        }
    }
}

// LDS accesses of one wave are executed in order: only the compiler has to
// keep a wave's writes before its reads.
FHE_DEV void wave_order() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier that orders LDS only (loads from global memory stay in flight).
FHE_DEV void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Where a transform's per-lane twiddles come from: registers, an LDS copy read
// at each use (where registers are scarce), or global memory (where the LDS is
// full as well), requested before the transform's first pass.
enum TwiddleSource { TW_REG, TW_LDS, TW_GLOBAL };

// A wave's part of a transform: its twiddles and its byte offsets in LDS.
// Exchange buffer: point j of block k at 64 k + (j ^ 2 (k & 7)), and pairs of
// the last level in two member planes, the second one's index ^ 4: with these
// swizzles no lanes of a read or write meet in an LDS bank (measured for one
// 1 KB wave access per CU: reads 1.9 ns, writes 5.6 ns; with blocks 66 points
// apart and planes M/2 + 8 apart the exchange read took 3.6 ns, the pair write
// 7.0 ns).
template <int R, TwiddleSource TWS>
struct WaveFft {
    using P = Plan<R>;
    static constexpr bool REG = TWS == TW_REG;
    static constexpr int S2 = P::NT2 + (R == 8 ? 1 : 0);  // entries per block of the LDS copy (5: no bank conflicts)
    double c2[REG ? P::NT2 : 1], t2[REG ? P::NT2 : 1], c3[REG ? P::NT3 : 1], t3[REG ? P::NT3 : 1];
    uint8_t* lds;
    uint32_t wb, rb, pb;  // write / read of the exchange, pairs
    uint32_t tw2, tw3;    // this lane's twiddles: LDS offsets or table entries
    const d2* twg;

    // buf: offset of the wave's buffer; twl: offset of the LDS copy of the
    // second pass's and the swapped levels' twiddles
    FHE_DEV void init(const d2* tw, uint8_t* lds_, uint32_t buf, uint32_t twl) {
        const int lane = threadIdx.x & 63;
        const int k = (lane >> 1) & (R - 1);
        const int bb = R == 8 ? (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + (lane & 1) : (lane >> 5) * 2 + (lane & 1);
        lds = lds_;
        wb = buf + lane * 16;
        rb = buf + (k * 64 + (bb ^ ((k & 7) * 2))) * 16;
        pb = buf + pair_off(lane & 1, lane >> 1);
        if constexpr (TWS == TW_LDS) {
            tw2 = twl + k * S2 * 16;
            tw3 = twl + (R * S2 + (lane >> 1) * P::NT3) * 16;
        } else {
            twg = tw;
            tw2 = k * P::NT2;
            tw3 = P::T3 + (lane >> 1) * P::NT3;
            if constexpr (REG) {
                fetch2(c2, t2);
                fetch3(c3, t3);
            }
        }
    }
    template <int K>
    FHE_DEV void fetch(uint32_t off, double (&c)[K], double (&t)[K]) const {
#pragma unroll
        for (int i = 0; i < K; i++) {
            const d2 w = TWS == TW_LDS ? at(off + i * 16) : twg[off + i];
            c[i] = w.x;
            t[i] = w.y;
        }
    }
    FHE_DEV void fetch2(double (&c)[P::NT2], double (&t)[P::NT2]) const { fetch(tw2, c, t); }
    FHE_DEV void fetch3(double (&c)[P::NT3], double (&t)[P::NT3]) const { fetch(tw3, c, t); }
    FHE_DEV d2& at(uint32_t off) const { return *(d2*)(lds + off); }
    // (an opaque copy keeps the swizzled addresses from being held in
    // registers across the step loop)
    FHE_DEV static uint32_t opaque(uint32_t x) {
        __asm__ volatile("" : "+v"(x));
        return x;
    }
    FHE_DEV void put_blocks(const double (&re)[R], const double (&im)[R]) const {  // point `lane` of block r
        const uint32_t b = opaque(wb);
#pragma unroll
        for (int r = 0; r < R; r++) at((b ^ ((r & 7) * 32)) + r * 64 * 16) = d2{re[r], im[r]};
    }
    FHE_DEV void get_blocks(double (&re)[R], double (&im)[R]) const {
        const uint32_t b = opaque(wb);
#pragma unroll
        for (int r = 0; r < R; r++) {
            const d2 v = at((b ^ ((r & 7) * 32)) + r * 64 * 16);
            re[r] = v.x;
            im[r] = v.y;
        }
    }
    FHE_DEV void put_points(const double (&re)[R], const double (&im)[R]) const {  // points of this lane's block
        const uint32_t b = opaque(rb);
#pragma unroll
        for (int r = 0; r < R; r++) at(b ^ (r * (64 / R) * 16)) = d2{re[r], im[r]};
    }
    FHE_DEV void get_points(double (&re)[R], double (&im)[R]) const {
        const uint32_t b = opaque(rb);
#pragma unroll
        for (int r = 0; r < R; r++) {
            const d2 v = at(b ^ (r * (64 / R) * 16));
            re[r] = v.x;
            im[r] = v.y;
        }
    }

    // points j = 64 r + lane in -> pairs of the last level in the buffer
    FHE_DEV void forward(double (&re)[R], double (&im)[R]) const {
        double c[P::NT2], t[P::NT2], cs[P::NT3], ts[P::NT3];
        if constexpr (TWS == TW_GLOBAL) {
            fetch2(c, t);
            fetch3(cs, ts);
            __builtin_amdgcn_sched_barrier(0);
        }
        lane_fwd<R>(re, im, kC1, kT1);
        put_blocks(re, im);
        wave_order();
        get_points(re, im);
        if constexpr (TWS == TW_LDS) fetch2(c, t);
        lane_fwd<R>(re, im, REG ? c2 : c, REG ? t2 : t);
        if constexpr (TWS == TW_LDS) fetch3(cs, ts);
        lane_swaps<R>(re, im);
        swapped_fwd<R>(re, im, REG ? c3 : cs, REG ? t3 : ts);
        wave_order();
#pragma unroll
        for (int r = 0; r < R; r++) at(pb + r * 32 * 16) = d2{re[r], im[r]};
    }
    struct Twiddles {
        double c2[P::NT2], t2[P::NT2], c3[P::NT3], t3[P::NT3];
    };
    // requests the inverse's twiddles (TW_GLOBAL)
    FHE_DEV void request(Twiddles& w) const {
        if constexpr (TWS == TW_GLOBAL) {
            fetch3(w.c3, w.t3);
            fetch2(w.c2, w.t2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // pairs in the buffer -> the first pass's inputs in registers
    FHE_DEV void inverse_to_first(double (&re)[R], double (&im)[R], Twiddles& w) const {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const d2 v = at(pb + r * 32 * 16);
            re[r] = v.x;
            im[r] = v.y;
        }
        if constexpr (TWS == TW_LDS) fetch3(w.c3, w.t3);
        swapped_inv<R>(re, im, REG ? c3 : w.c3, REG ? t3 : w.t3);
        if constexpr (TWS == TW_LDS) fetch2(w.c2, w.t2);
        lane_swaps<R>(re, im);
        lane_inv<R>(re, im, REG ? c2 : w.c2, REG ? t2 : w.t2);
        wave_order();
        put_points(re, im);
        wave_order();
        get_blocks(re, im);
    }
    // offset of member e of pair g in a buffer
    FHE_DEV static uint32_t pair_off(int e, int g) { return (e * (P::M / 2) + (g ^ (e * 4))) * 16; }
};

// -------------------------------------------------------- key spectra

// fkey[poly][limb][member][pair]: spectrum of limb `limb` of key polynomial
// `poly` = BSK[i][r][v], scaled by 1/M; member e of pair g as a thread of the
// blind rotation reads them.  One wave per (poly, limb).
template <typename T, int R>
__global__ __launch_bounds__(64) void fft_key_kernel(const T* bsk, const d2* tw, d2* fkey) {
    using P = Plan<R>;
    using F = WaveFft<R, TW_REG>;
    __shared__ d2 buf[P::M];
    const int lane = threadIdx.x;
    const int limb = blockIdx.x % Limb<T>::COUNT;
    const size_t poly = blockIdx.x / Limb<T>::COUNT;
    const T* K = bsk + poly * P::N;
    F f;
    f.init(tw, (uint8_t*)buf, 0, 0);
    auto part = [&](int j) -> double {
        T x = K[j];
        constexpr int b = Limb<T>::BITS;
        int64_t v = 0;
        for (int m = 0; m <= limb; m++) {
            // the last limb holds the bits that are left, as a signed number
            const int w = m + 1 < Limb<T>::COUNT ? b : Torus<T>::Q - b * (Limb<T>::COUNT - 1);
            const int sh = 64 - w;
            v = (int64_t)((uint64_t)x << sh) >> sh;
            x = (T)((T)(x - (T)v) >> b);
        }
        return (double)v;
    };
    double re[R], im[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        re[r] = part(64 * r + lane);
        im[r] = part(64 * r + lane + P::M);
    }
    f.forward(re, im);
    __syncthreads();
    d2* out = fkey + (size_t)blockIdx.x * P::M;
    constexpr double scale = 1.0 / P::M;
    for (int g = lane; g < P::M / 2; g += 64) {
        const d2 x = f.at(F::pair_off(0, g)), y = f.at(F::pair_off(1, g)), w = tw[P::T4 + g];
        double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
        bf_fwd<false>(xr, xi, yr, yi, w.x, w.y);
        out[g] = d2{xr * scale, xi * scale};
        out[P::M / 2 + g] = d2{yr * scale, yi * scale};
    }
}

// ------------------------------------------------------ blind rotation

struct FftArgs {
    const void* lwe;          // [B][n+1] words
    const d2* fkey;           // [n][2l][2][limbs][M]
    const d2* tw;             // twiddle table
    const void* tv;           // test polynomials [ntv][N] words
    const int32_t* tv_index;  // [B] or null
    void* out;                // [B][N+1] words
    int B, n, l, bg_bits, cus;
};

// One configuration: W waves and G ciphertexts per workgroup; KD: a thread's
// ring of key values, in polynomials, filled when the transform's registers are
// free.
template <typename T_, int R_, int W_, int G_, int L_, int KD_, TwiddleSource TWS_, int WPE_ = 2>
struct Cfg {
    using T = T_;
    static constexpr int R = R_, W = W_, G = G_, L = L_, KD = KD_, WPE = WPE_;
    static constexpr TwiddleSource TWS = TWS_;
    using P = Plan<R>;
    using F = WaveFft<R, TWS>;
    // Key lines into L2 a step ahead (8-wave workgroups; with 4 waves, several
    // workgroups per CU hide the latency: 1500 ciphertexts 13.6 ms both ways).
    // Held by lane AHEAD at a time by waves W/2.., a step's lines need HELP
    // workgroups, 8 XCDs' worth; a smaller batch is topped up with copies.
    // Without the lines, B = 1 took 3.07 ms (3.62 with the key in HBM), at N =
    // 2048, q = 64 15.5 ms; with lines and 16 workgroups 2.87 and 13.0, with 32
    // 2.50 and 11.7, 64 2.52 and 10.7, 128 2.53 and 10.7.
    static constexpr int HELP = W == 8 && G == 1 ? (R == 8 ? 32 : 64) : 0;
    static constexpr int LINES = 2 * (L ? L : Limb<T>::COUNT + 1) * 2 * Limb<T>::COUNT * P::M / 8;
    static constexpr int AHEAD = W < 8 ? 0 : HELP ? (LINES + HELP / 8 * 256 - 1) / (HELP / 8 * 256) : 1;
    static constexpr uint32_t BUF = P::M * 16;                            // bytes of a wave's buffer
    static constexpr uint32_t ACC = W * BUF;                              // accumulators [G][2][N]
    static constexpr uint32_t TW = ACC + G * 2 * P::N * (uint32_t)sizeof(T);  // twiddles (TW_LDS)
    static constexpr uint32_t ZS = TW + (TWS == TW_LDS ? (uint32_t)(R * F::S2 + 32 * P::NT3) * 16 : 0);
    // Digit words [G][2][N], formed once for all levels: behind the rest if LDS
    // has room, else in the first buffers if one round reads them all.
    static constexpr uint32_t ZBYTES = G * 2 * P::N * 4;
    static constexpr bool ZROOM = W == 8 && ZS + ZBYTES <= 160 * 1024;
    static constexpr bool SHARE = ZROOM || (W == 8 && L && 2 * L * G <= W);
    static constexpr uint32_t LDS = ZS + (ZROOM ? ZBYTES : 0);
};

template <typename CF>
__global__ __launch_bounds__(64 * CF::W) __attribute__((amdgpu_waves_per_eu(CF::WPE, CF::WPE))) void br_fft_kernel(FftArgs a) {
    using T = typename CF::T;
    using P = typename CF::P;
    using WF = typename CF::F;
    constexpr int R = CF::R, W = CF::W, G = CF::G, KD = CF::KD;
    constexpr int N = P::N, M = P::M, LN = __builtin_ctz(N);
    constexpr int Q = Torus<T>::Q;
    constexpr int OUT = 2 * Limb<T>::COUNT;       // outputs: component, limb
    constexpr int PPR = W / G;                    // polynomials of a ciphertext per round
    constexpr int OS = 64 * W / (M / 2);          // thread sets that share the pairs' outputs
    constexpr int OT = OUT / OS;                  // outputs of a thread
    constexpr int IR = (OUT + PPR - 1) / PPR;     // inverse rounds
    static_assert(W % G == 0 && 64 * W % (M / 2) == 0 && OUT % OS == 0, "work split");
    static_assert(OS == 1 || PPR >= OUT, "one inverse round when the outputs are split over threads");
    static_assert(PPR % KD == 0, "key ring");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n, l = CF::L ? CF::L : a.l, NB = 2 * l;
    // copies (HELP) work on a ciphertext of the batch again and store nothing
    const int ct0 = CF::HELP ? blockIdx.x % a.B : blockIdx.x * G;

    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    T* accs = (T*)(smem + CF::ACC);  // [G][2][N]

    // this wave's ciphertext and its place among that ciphertext's waves
    const int ct = wave % G, pq0 = wave / G;
    const bool live = ct0 + ct < a.B;
    const T* lwe = (const T*)a.lwe + (size_t)(live ? ct0 + ct : 0) * (n + 1);
    T* const acc_ct = accs + (size_t)ct * 2 * N;

    // accumulator = (0, X^{-bbar} testv)
    for (int idx = tid; idx < G * N; idx += 64 * W) {
        const int c = idx / N, j = idx & (N - 1);
        const int gi = ct0 + c;
        T body = 0;
        if (gi < a.B) {
            const int bb = (int)mod_switch<T>(((const T*)a.lwe)[(size_t)gi * (n + 1) + n], LN + 1);
            const int e = (2 * N - bb) & (2 * N - 1);
            const T* tv = (const T*)a.tv + (size_t)(a.tv_index ? a.tv_index[gi] : 0) * N;
            body = monomial_coef<T>([&](int s) -> T { return tv[s]; }, N, e, j);
        }
        accs[(size_t)c * 2 * N + j] = 0;
        accs[(size_t)c * 2 * N + N + j] = body;
    }
    if constexpr (CF::TWS == TW_LDS)
        for (int idx = tid; idx < P::T4; idx += 64 * W)
            ((d2*)(smem + CF::TW))[idx < P::T3 ? idx + idx / P::NT2 * (WF::S2 - P::NT2) : idx + R * WF::S2 - P::T3] = a.tw[idx];

    WF f;
    f.init(a.tw, smem, wave * CF::BUF, CF::TW);
    const int g = tid & (M / 2 - 1), os = OS == 1 ? 0 : tid / (M / 2);
    const d2 w4 = a.tw[P::T4 + g];
    // this thread's pairs in buffer 0
    const uint32_t px = WF::pair_off(0, g), py = WF::pair_off(1, g);

    // gadget digits as in the int8 path: field p of z, read as a signed number
    const int bgb = a.bg_bits;
    const int shr = Q - l * bgb;
    uint32_t off = 0;
    for (int p = 0; p < l; p++) off += (uint32_t)(1 << (bgb - 1)) << (p * bgb);
    const T F = (T)off << shr;
    const T C = ((T)1 << (shr - 1)) + F;
    const int fb = Q == 32 ? shr : shr - 32;

    // digit words of X^{ab} ACC_u - ACC_u at coefficients j0 + 64 r + lane, r < CNT
    auto form_words = [&](auto& z, int u, int j0, int ab) {
        constexpr int CNT = sizeof(z) / 4;
        const T* acc = acc_ct + (size_t)u * N;
        int x0 = j0 + lane;
        __asm__ volatile("" : "+v"(x0));
        const T* own = acc + x0;
        x0 -= ab;
#pragma unroll
        for (int r = 0; r < CNT; r++) {
            const int x = x0 + 64 * r;
            const T v = acc[x & (N - 1)];
            const T m = (T)(int64_t)(int32_t)__builtin_amdgcn_sbfe(x, LN, 1);  // all ones: negate
            const T zz = (T)((T)(C - own[64 * r]) + (T)((v ^ m) - m)) ^ F;
            z[r] = Q == 32 ? (uint32_t)zz : (uint32_t)((uint64_t)zz >> 32);
        }
    };
    auto form = [&](uint32_t (&z)[2 * R], int u, int ab) { form_words(z, u, 0, ab); };
    // SHARE: a ciphertext's waves form an equal part of its words each, once for
    // all levels.  About 170 of a digit polynomial's 500 vector instructions were
    // its words, formed again per level, on the SIMDs with two of a step's six
    // transforms: 1 ciphertext 2.51 -> 2.36 ms, 512 4.41 -> 4.14; N = 2048, q = 64
    // 10.7 -> 10.2.
    constexpr bool SHARE = CF::SHARE;
    uint32_t* const zs = (uint32_t*)(smem + (CF::ZROOM ? CF::ZS : 0)) + ct * 2 * N + lane;
    auto form_share = [&](int ab) {
        constexpr int CNT = 2 * N / (64 * PPR);
        const int u = pq0 / (PPR / 2), j0 = pq0 % (PPR / 2) * (64 * CNT);
        uint32_t z[CNT];
        form_words(z, u, j0, ab);
#pragma unroll
        for (int r = 0; r < CNT; r++) zs[u * N + j0 + 64 * r] = z[r];
    };
    auto transform = [&](const uint32_t (&z)[2 * R], int p) {
        const int pos = fb + (l - 1 - p) * bgb;
        double re[R], im[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            re[r] = (double)(int)__builtin_amdgcn_sbfe((int)z[r], pos, bgb);
            im[r] = (double)(int)__builtin_amdgcn_sbfe((int)z[R + r], pos, bgb);
        }
        f.forward(re, im);
    };

    // key values of this thread: 2 OT per polynomial, KD polynomials
    const d2* const key0 = a.fkey + (size_t)os * OT * M + g;
    d2 kv[KD][OT][2];
    auto key_load = [&](d2 (&k)[OT][2], int i, int pq) {
        const d2* kp = key0 + ((size_t)i * NB + pq) * (OUT * M);
#pragma unroll
        for (int o = 0; o < OT; o++)
#pragma unroll
            for (int e = 0; e < 2; e++) k[o][e] = kp[o * M + e * (M / 2)];
    };
    // Key lines of step i, one dword of each, so that they are in this XCD's L2
    // when the step loads them.  Consecutive workgroups run on different XCDs:
    // workgroups 8 apart share the lines, and every fourth of a share is a wave's.
    constexpr int AHEAD = CF::AHEAD;
    uint32_t line[AHEAD ? AHEAD : 1] = {};
    const int sharers = min(((int)gridDim.x + 7) / 8, 32);
    const int lines = NB * OUT * M / 8, share = (lines + sharers - 1) / sharers;
    const int line0 = (int)(blockIdx.x / 8) % sharers * share, line1 = min(line0 + share, lines);
    auto request_lines = [&](int i) {
        if (!AHEAD || wave < W / 2) return;
        const uint8_t* kb = (const uint8_t*)(a.fkey + (size_t)min(i, n - 1) * NB * OUT * M);
#pragma unroll
        for (int t = 0; t < AHEAD; t++) {
            const int x = line0 + (wave - W / 2 + t * (W / 2)) * 64;
            if (x < line1) line[t] = *(const uint32_t*)(kb + (size_t)min(x + lane, line1 - 1) * 128);
        }
    };
    auto lines_arrived = [&] {
#pragma unroll
        for (int t = 0; t < AHEAD; t++) __asm__ volatile("" ::"v"(line[t]));
    };

    // Where the ring holds a whole step (one ciphertext, l = 3), the waves that
    // have no output to transform back load the next step's values meanwhile: the
    // loads of a step take 3000 cycles of the CU's path to L2, 800 of them after
    // the last transform otherwise (64 ciphertexts 2.67 -> 2.51 ms).  The other
    // waves have none to spare: issuing loads holds up their transforms (all
    // loads ahead of the transforms: 3.1 ms).
    constexpr bool EARLY = CF::L && 2 * CF::L <= KD && IR == 1 && PPR > OUT;
    auto key_step = [&](int i) {
#pragma unroll
        for (int pp = 0; pp < KD; pp++)
            if (pp < NB) key_load(kv[pp], i, pp);
    };

    int abv = 0;  // abar of steps 64 (i/64) + lane
    // Workgroups that share a CU start together and run their phases at the same
    // time, one in the other's way (a launch of one round 15.5 ms, of eight
    // rounds, where they drift apart, 14.2 per round).  So the second to come to
    // a CU goes first for 5/8 of the steps and then the other one, so that both
    // end together: 2048 ciphertexts 15.5 -> 13.9 ms, 4096 29.7 -> 27.7, 16,384
    // 113.5 -> 111.0.  (1/2^k of the steps in turn: 14.9 at 1 and 16 steps, 14.6 at
    // 256; 11/16, 3/4, 13/16, all: 13.8, 14.0, 14.4, 15.5, and 28.6 at 4096 for
    // 11/16; three workgroups of two ciphertexts per CU: 1% slower with it.)
    const bool second = blockIdx.x / a.cus & 1;
    const int swap_at = n * 5 / 8;
    if (EARLY && pq0 >= OUT) key_step(0);
    lds_barrier();
    for (int i = 0; i < n; i++) {
        if ((i & 63) == 0) abv = live && i + lane < n ? (int)mod_switch<T>(lwe[i + lane], LN + 1) : 0;
        const int ab = __builtin_amdgcn_readlane(abv, i & 63);
        if constexpr (G == 4) {
            if (i == 0 || i == swap_at) {
                if (second == (i == 0)) __builtin_amdgcn_s_setprio(2);
                else __builtin_amdgcn_s_setprio(0);
            }
        }
        double ar[OT][2][G], ai[OT][2][G];
#pragma unroll
        for (int o = 0; o < OT; o++)
#pragma unroll
            for (int e = 0; e < 2; e++)
#pragma unroll
                for (int c = 0; c < G; c++) ar[o][e][c] = ai[o][e][c] = 0;

        // pairs of polynomial pp of every ciphertext
        auto pairs = [&](d2 (&x)[G], d2 (&y)[G], int pp) {
#pragma unroll
            for (int c = 0; c < G; c++) {
                x[c] = f.at(px + (pp * G + c) * CF::BUF);
                y[c] = f.at(py + (pp * G + c) * CF::BUF);
            }
        };
        auto products = [&](const d2 (&x)[G], const d2 (&y)[G], const d2 (&k)[OT][2]) {
            double dr[2][G], di[2][G];
#pragma unroll
            for (int c = 0; c < G; c++) {
                dr[0][c] = x[c].x;
                di[0][c] = x[c].y;
                dr[1][c] = y[c].x;
                di[1][c] = y[c].y;
                bf_fwd<false>(dr[0][c], di[0][c], dr[1][c], di[1][c], w4.x, w4.y);
            }
#pragma unroll
            for (int o = 0; o < OT; o++)
#pragma unroll
                for (int e = 0; e < 2; e++)
#pragma unroll
                    for (int c = 0; c < G; c++) {
                        ar[o][e][c] = __builtin_fma(dr[e][c], k[o][e].x, ar[o][e][c]);
                        ai[o][e][c] = __builtin_fma(dr[e][c], k[o][e].y, ai[o][e][c]);
                        ar[o][e][c] = __builtin_fma(-di[e][c], k[o][e].y, ar[o][e][c]);
                        ai[o][e][c] = __builtin_fma(di[e][c], k[o][e].x, ai[o][e][c]);
                    }
        };

        if constexpr (PPR == 1) {
            for (int u = 0; u < 2; u++) {
                uint32_t z[2 * R];
                form(z, u, ab);
                for (int p = 0; p < l; p++) {
                    transform(z, p);
                    if (p + u == 0) lines_arrived();
                    __builtin_amdgcn_sched_barrier(0);  // (not earlier: the transform needs the registers)
                    key_load(kv[0], i, u * l + p);
                    lds_barrier();
                    d2 x[G], y[G];
                    pairs(x, y, 0);
                    lds_barrier();
                    products(x, y, kv[0]);
                }
            }
        } else {
            if constexpr (SHARE) {
                form_share(ab);
                lds_barrier();
            }
            for (int q0 = 0; q0 < NB; q0 += PPR) {
                const bool any = q0 + pq0 < NB;
                const int u = q0 + pq0 >= l;
                uint32_t z[2 * R];
                if (any) {
                    if constexpr (SHARE) {
#pragma unroll
                        for (int r = 0; r < 2 * R; r++) z[r] = zs[u * N + 64 * r];
                    } else {
                        form(z, u, ab);
                    }
                }
                if (SHARE && !CF::ZROOM) lds_barrier();  // the words lie in the buffers
                if (any) transform(z, q0 + pq0 - u * l);
                if (q0 == 0) lines_arrived();
                __builtin_amdgcn_sched_barrier(0);  // (not earlier: the transform needs the registers)
                if (!EARLY || pq0 < OUT)
#pragma unroll
                    for (int pp = 0; pp < KD; pp++)
                        if (q0 + pp < NB) key_load(kv[pp], i, q0 + pp);
                lds_barrier();
#pragma unroll
                for (int pp = 0; pp < PPR; pp++) {
                    if (q0 + pp < NB) {
                        d2 x[G], y[G];
                        pairs(x, y, pp);
                        products(x, y, kv[pp % KD]);
                    }
                    if (pp + KD < PPR && q0 + pp + KD < NB) key_load(kv[pp % KD], i, q0 + pp + KD);
                }
                lds_barrier();
            }
        }

        // back: one output of a ciphertext per wave and round
#pragma unroll
        for (int rd = 0; rd < IR; rd++) {
#pragma unroll
            for (int o = 0; o < OT; o++) {
                if (OS == 1 && o / PPR != rd) continue;
                const int slot = OS == 1 ? o % PPR : os * OT + o;
#pragma unroll
                for (int c = 0; c < G; c++) {
                    bf_inv<false>(ar[o][0][c], ai[o][0][c], ar[o][1][c], ai[o][1][c], w4.x, w4.y);
                    f.at(px + (slot * G + c) * CF::BUF) = d2{ar[o][0][c], ai[o][0][c]};
                    f.at(py + (slot * G + c) * CF::BUF) = d2{ar[o][1][c], ai[o][1][c]};
                }
            }
            lds_barrier();
            const int o = rd * PPR + pq0;
            const bool mine = OUT % PPR == 0 || o < OUT;
            double re[R], im[R];
            typename WF::Twiddles tw;
            f.request(tw);
            if (EARLY && pq0 >= OUT) key_step(i + 1 < n ? i + 1 : 0);
            if (rd == 0) request_lines(i + (EARLY ? 2 : 1));
            if (mine) f.inverse_to_first(re, im, tw);
            if (rd + 1 < IR) lds_barrier();
            if (mine) {
                double sc[R];
                lane_inv_first<R>(re, im, sc);
                constexpr int LC = Limb<T>::COUNT;
                T* acc = acc_ct + (size_t)(o / LC) * N + lane;
                const int sh = (o % LC) * Limb<T>::BITS;
#pragma unroll
                for (int r = 0; r < R; r++) {
                    atomicAdd(acc + 64 * r, (T)nearest(re[r], sc[r]) << sh);
                    atomicAdd(acc + 64 * r + M, (T)nearest(im[r], sc[r]) << sh);
                }
            }
        }
        // with one wave per ciphertext only that wave reads its accumulator
        if (W > G) lds_barrier();
        else wave_order();
    }

    // ---- sample extraction: a'_0 = A[0], a'_j = -A[N-j], b' = B[0]
    lds_barrier();
    if (CF::HELP && (int)blockIdx.x >= a.B) return;
    T* out = (T*)a.out;
    for (int c = 0; c < G && ct0 + c < a.B; c++) {
        const T* A = accs + (size_t)c * 2 * N;
        for (int j = tid; j <= N; j += 64 * W)
            out[(size_t)(ct0 + c) * (N + 1) + j] = j == 0 ? A[0] : j < N ? (T)(0 - A[N - j]) : A[N];
    }
}

// ---------------------------------------------- small ring (N = 256, q = 32)
//
// A transform of M = 128 points takes 16 lanes with 8 points each, so one wave
// transforms 4 polynomials at a time: the digits of a ciphertext (l = 2: all of
// them), or its 4 outputs on the way back.  Radix 8, an exchange, radix 8, and
// the last level in the lane that multiplies (64 pairs, a lane each).  A wave
// needs no other: no barrier, one wave per workgroup and ciphertext.
//
// Bounded by its chain while a SIMD has fewer than three waves (a step of one
// alone takes 4900 cycles, of twelve on a CU 14,800), then by double-precision
// issue (530 of about 780 vector instructions per ciphertext and step).
// Measured at n = 64, l = 2 against the int8 kernel (whose workgroup runs 16
// ciphertexts, so that its time goes in steps of 16 per CU): 1 ciphertext 0.447
// -> 0.131 ms, 1024 0.467 -> 0.183 ms, 2597 0.454 -> 0.372 ms, 5904 0.775 ->
// 0.715 ms; 8192 0.886 against 0.960 ms and 65,536 6.74 against 7.6 ms, where
// the int8 kernel stays (small_pays).  All of a step's key values a step ahead
// with two waves per SIMD: 4250 0.604 ms against 0.575; two ciphertexts per wave
// 0.687, 65,536 7.4.
struct Small {
    static constexpr int N = 256, M = 128;
    static constexpr int T4 = 32, TN = 32 + 64;  // twiddle table: [8 blocks][4], [64 pairs]
};

// L: gadget levels when compile-time (then a polynomial's key values are
// requested while the one before is multiplied, the first one's ahead of the
// last pass forward), else 0.
template <int L>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void br_fft256_kernel(FftArgs a) {
    using T = uint32_t;
    constexpr int N = Small::N, M = Small::M, LN = 8, OUT = 4;
    constexpr int KD = L ? 2 : 1;
    const int lane = threadIdx.x;
    const int n = a.n, l = L ? L : a.l, NB = 2 * l;
    __shared__ d2 buf[4 * M];  // [polynomial][M]
    __shared__ T accs[2 * N];
    const T* const lwe = (const T*)a.lwe + (size_t)blockIdx.x * (n + 1);

    const int bb = (int)mod_switch<T>(lwe[n], LN + 1);
    const T* tv = (const T*)a.tv + (size_t)(a.tv_index ? a.tv_index[blockIdx.x] : 0) * N;
    for (int j = lane; j < N; j += 64) {
        accs[j] = 0;
        accs[N + j] = monomial_coef<T>([&](int s) -> T { return tv[s]; }, N, (2 * N - bb) & (2 * N - 1), j);
    }

    // lane: polynomial pl of the pass; point j4 (of 16) or block k, member b0
    const int pl = lane >> 4, j4 = lane & 15, k = j4 >> 1, b0 = j4 & 1;
    double c2[4], t2[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const d2 w = a.tw[k * 4 + i];
        c2[i] = w.x;
        t2[i] = w.y;
    }
    const d2 w4 = a.tw[Small::T4 + lane];
    // exchange: point j of block k at 16 k + (j ^ 2 k); pairs: member planes of
    // 64, the second one's index ^ 4
    const int wr = pl * M + j4, rd = pl * M + k * 16 + (b0 ^ (2 * k)), pr = pl * M + b0 * 64 + (k ^ (b0 * 4));

    const int bgb = a.bg_bits;
    const int shr = 32 - l * bgb;
    uint32_t off = 0;
    for (int p = 0; p < l; p++) off += (uint32_t)(1 << (bgb - 1)) << (p * bgb);
    const T F = off << shr;
    const T C = (1u << (shr - 1)) + F;

    const d2* const key0 = a.fkey + lane;  // [n][2l][OUT][2 members][64 pairs]
    d2 kv[KD][OUT][2];
    auto key_load = [&](d2 (&v)[OUT][2], int i, int pq) {
        const d2* kp = key0 + ((size_t)i * NB + pq) * (OUT * M);
#pragma unroll
        for (int o = 0; o < OUT; o++)
#pragma unroll
            for (int e = 0; e < 2; e++) v[o][e] = kp[o * M + e * 64];
    };
    int abv = 0;  // abar of steps 64 (i/64) + lane
    wave_order();
    for (int i = 0; i < n; i++) {
        if ((i & 63) == 0) abv = i + lane < n ? (int)mod_switch<T>(lwe[i + lane], LN + 1) : 0;
        const int ab = __builtin_amdgcn_readlane(abv, i & 63);
        double ar[OUT][2], ai[OUT][2];
#pragma unroll
        for (int o = 0; o < OUT; o++)
#pragma unroll
            for (int e = 0; e < 2; e++) ar[o][e] = ai[o][e] = 0;
        for (int q0 = 0; q0 < NB; q0 += 4) {
            // digits and transforms of polynomials q0 .. q0 + 3 (a lane's past
            // the last one repeats it; it is not read)
            const int pq = min(q0 + pl, NB - 1), u = pq >= l ? 1 : 0;
            const int pos = shr + (l - 1 - (pq - u * l)) * bgb;
            const T* acc = accs + u * N;
            // digit word of coefficient 16 r + x0
            int x0 = L == 2 ? j4 + (pl & 1) * M : j4;
            __asm__ volatile("" : "+v"(x0));
            const T* own = acc + x0;
            x0 -= ab;
            auto word = [&](int r) -> int {
                const int x = x0 + 16 * r;
                const T v = acc[x & (N - 1)];
                const T m = (T)(int32_t)__builtin_amdgcn_sbfe(x, LN, 1);
                return (int)(((C - own[16 * r]) + ((v ^ m) - m)) ^ F);
            };
            double re[8], im[8];
#pragma unroll
            for (int r = 0; r < 8; r++) {
                int zr, zi;
                if constexpr (L == 2) {
                    // the two levels of a component (lane rows 2u, 2u + 1)
                    // form a half of its words each and swap copies
                    const int z = word(r);
                    const auto zz = __builtin_amdgcn_permlane16_swap(z, z, false, false);
                    zr = (int)zz[0];
                    zi = (int)zz[1];
                } else {
                    zr = word(r);
                    zi = word(r + 8);
                }
                re[r] = (double)(int)__builtin_amdgcn_sbfe(zr, pos, bgb);
                im[r] = (double)(int)__builtin_amdgcn_sbfe(zi, pos, bgb);
            }
            lane_fwd<8>(re, im, kC1, kT1);
#pragma unroll
            for (int r = 0; r < 8; r++) buf[(wr ^ (2 * r)) + r * 16] = d2{re[r], im[r]};
            wave_order();
#pragma unroll
            for (int r = 0; r < 8; r++) {
                const d2 v = buf[rd ^ (2 * r)];
                re[r] = v.x;
                im[r] = v.y;
            }
            if (KD == 2) key_load(kv[0], i, 0);
            lane_fwd<8>(re, im, c2, t2);
            wave_order();
#pragma unroll
            for (int r = 0; r < 8; r++) buf[pr + r * 8] = d2{re[r], im[r]};
            wave_order();
#pragma unroll
            for (int pp = 0; pp < 4; pp++) {
                if (L ? pp >= 2 * L : q0 + pp >= NB) break;
                if (KD == 1) key_load(kv[0], i, q0 + pp);
                if (KD == 2 && pp + 1 < 2 * L) key_load(kv[(pp + 1) % KD], i, pp + 1);
                const d2 x = buf[pp * M + lane], y = buf[pp * M + 64 + (lane ^ 4)];
                double dr[2] = {x.x, y.x}, di[2] = {x.y, y.y};
                bf_fwd<false>(dr[0], di[0], dr[1], di[1], w4.x, w4.y);
#pragma unroll
                for (int o = 0; o < OUT; o++)
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        const d2 w = kv[pp % KD][o][e];
                        ar[o][e] = __builtin_fma(dr[e], w.x, ar[o][e]);
                        ai[o][e] = __builtin_fma(dr[e], w.y, ai[o][e]);
                        ar[o][e] = __builtin_fma(-di[e], w.y, ar[o][e]);
                        ai[o][e] = __builtin_fma(di[e], w.x, ai[o][e]);
                    }
            }
            wave_order();
        }
        // back: the lanes of group pl transform output pl (component pl / 2, limb pl % 2)
#pragma unroll
        for (int o = 0; o < OUT; o++) {
            bf_inv<false>(ar[o][0], ai[o][0], ar[o][1], ai[o][1], w4.x, w4.y);
            buf[o * M + lane] = d2{ar[o][0], ai[o][0]};
            buf[o * M + 64 + (lane ^ 4)] = d2{ar[o][1], ai[o][1]};
        }
        wave_order();
        double re[8], im[8];
#pragma unroll
        for (int r = 0; r < 8; r++) {
            const d2 v = buf[pr + r * 8];
            re[r] = v.x;
            im[r] = v.y;
        }
        lane_inv<8>(re, im, c2, t2);
        wave_order();
#pragma unroll
        for (int r = 0; r < 8; r++) buf[rd ^ (2 * r)] = d2{re[r], im[r]};
        wave_order();
#pragma unroll
        for (int r = 0; r < 8; r++) {
            const d2 v = buf[(wr ^ (2 * r)) + r * 16];
            re[r] = v.x;
            im[r] = v.y;
        }
        double sc[8];
        lane_inv_first<8>(re, im, sc);
        T* acc = accs + (pl >> 1) * N + j4;
        const int sh = (pl & 1) * 16;
#pragma unroll
        for (int r = 0; r < 8; r++) {
            atomicAdd(acc + 16 * r, (T)nearest(re[r], sc[r]) << sh);
            atomicAdd(acc + 16 * r + M, (T)nearest(im[r], sc[r]) << sh);
        }
        wave_order();
    }

    T* out = (T*)a.out + (size_t)blockIdx.x * (N + 1);
    for (int j = lane; j <= N; j += 64) out[j] = j == 0 ? accs[0] : j < N ? 0 - accs[N - j] : accs[N];
}

// Key spectra of the small ring: 16 lanes per (polynomial, limb), 4 per wave.
__global__ __launch_bounds__(64) void fft256_key_kernel(const uint32_t* bsk, const d2* tw, d2* fkey, int total) {
    constexpr int N = Small::N, M = Small::M;
    __shared__ d2 buf[4 * M];
    const int lane = threadIdx.x, pl = lane >> 4, j4 = lane & 15, k = j4 >> 1, b0 = j4 & 1;
    const int id = min((int)blockIdx.x * 4 + pl, total - 1);  // polynomial * 2 + limb
    const uint32_t* K = bsk + (size_t)(id >> 1) * N;
    const int limb = id & 1;
    double c2[4], t2[4];
    for (int i = 0; i < 4; i++) {
        c2[i] = tw[k * 4 + i].x;
        t2[i] = tw[k * 4 + i].y;
    }
    auto part = [&](int j) -> double {
        const uint32_t x = K[j];
        const int lo = (int16_t)x;
        return limb ? (double)(int16_t)((x - (uint32_t)lo) >> 16) : (double)lo;
    };
    double re[8], im[8];
#pragma unroll
    for (int r = 0; r < 8; r++) {
        re[r] = part(16 * r + j4);
        im[r] = part(16 * r + j4 + M);
    }
    const int wr = pl * M + j4, rd = pl * M + k * 16 + (b0 ^ (2 * k)), pr = pl * M + b0 * 64 + (k ^ (b0 * 4));
    lane_fwd<8>(re, im, kC1, kT1);
#pragma unroll
    for (int r = 0; r < 8; r++) buf[(wr ^ (2 * r)) + r * 16] = d2{re[r], im[r]};
    wave_order();
#pragma unroll
    for (int r = 0; r < 8; r++) {
        const d2 v = buf[rd ^ (2 * r)];
        re[r] = v.x;
        im[r] = v.y;
    }
    lane_fwd<8>(re, im, c2, t2);
    wave_order();
#pragma unroll
    for (int r = 0; r < 8; r++) buf[pr + r * 8] = d2{re[r], im[r]};
    wave_order();
    const d2 w = tw[Small::T4 + lane];
    constexpr double scale = 1.0 / M;
    for (int q = 0; q < 4 && (int)blockIdx.x * 4 + q < total; q++) {
        const d2 x = buf[q * M + lane], y = buf[q * M + 64 + (lane ^ 4)];
        double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
        bf_fwd<false>(xr, xi, yr, yi, w.x, w.y);
        d2* out = fkey + (size_t)(blockIdx.x * 4 + q) * M;
        out[lane] = d2{xr * scale, xi * scale};
        out[64 + lane] = d2{yr * scale, yi * scale};
    }
}

template <typename CF>
int launch_fft_t(tfhe_ctx* c, const FftArgs& a, hipStream_t s) {
    auto k = br_fft_kernel<CF>;
    static_assert(CF::LDS <= 160 * 1024, "LDS");
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CF::LDS);
    if (e != hipSuccess) return hip_check(c, e, "hipFuncSetAttribute(br_fft)");
    if (CF::L && CF::L != a.l) return ctx_fail(c, TFHE_EINVAL, "transform kernel of another level count");
    hipLaunchKernelGGL(k, dim3(std::max((a.B + CF::G - 1) / CF::G, CF::HELP)), dim3(64 * CF::W), CF::LDS, s, a);
    return hip_check(c, hipGetLastError(), "launch br_fft");
}

// cos and tan of `turns` (dyadic, never a quarter turn's odd multiple)
d2 twiddle(long double turns) {
    const long double x = 2.0L * 3.14159265358979323846264338327950288L * turns;
    return d2{(double)cosl(x), (double)(sinl(x) / cosl(x))};
}

// Angles (in turns): after t levels the block with path bits d1..dt is mod
// X^m - e^{2 pi i theta}, theta = 1/(4 2^t) + sum_i d_i 2^{i-1-t}, and the next
// level's twiddle has the angle theta/2.
long double theta(const std::vector<int>& d) {
    const int t = (int)d.size();
    long double x = 0.25L;
    for (int i = 0; i < t; i++) x += d[i] * (long double)(1 << i);
    return x / (long double)(1 << t);
}
void bits(std::vector<int>& d, int v, int count) {  // first path bit = top bit
    for (int b = count - 1; b >= 0; b--) d.push_back((v >> b) & 1);
}

// the second pass's twiddles of every block of the first
template <int R>
void second_pass(d2* tw) {
    using P = Plan<R>;
    for (int k = 0; k < R; k++)
        for (int m = 1; m <= P::L; m++)
            for (int q = 0; q < (m == 1 ? 1 : 1 << (m - 2)); q++) {
                std::vector<int> d;
                bits(d, k, P::L);
                if (m > 1) {
                    bits(d, q, m - 2);
                    d.push_back(0);
                }
                tw[(size_t)k * P::NT2 + (m == 1 ? 0 : (1 << (m - 2)) + q)] = twiddle(theta(d) / 2);
            }
}

template <int R>
std::vector<d2> twiddle_table() {
    using P = Plan<R>;
    std::vector<d2> tw(P::TN);
    second_pass<R>(tw.data());
    for (int x = 0; x < 32; x++)
        for (int q = 0; q < P::NT3; q++) {
            std::vector<int> d;
            bits(d, x & (R - 1), P::L);  // first pass
            if (R == 8) {
                bits(d, x >> 3, 2);               // e1 e2
                d.push_back(q == 2 ? 1 : 0);      // e3 (a factor i for the first swapped level)
                if (q) d.push_back(0);            // f1 (a factor i for the second)
            } else {
                d.push_back(x >> 4);  // e1
                bits(d, q, 2);        // e2 e3
                d.push_back(0);       // e4 (a factor i)
            }
            tw[P::T3 + (size_t)x * P::NT3 + q] = twiddle(theta(d) / 2);
        }
    for (int g = 0; g < P::M / 2; g++) {
        const int r = g >> 5, x = g & 31;
        std::vector<int> d;
        bits(d, x & (R - 1), P::L);
        if (R == 8) {
            bits(d, x >> 3, 2);
            d.push_back(r & 1);
            bits(d, r >> 1, 2);  // f1 f2
        } else {
            d.push_back(x >> 4);
            bits(d, r & 7, 3);       // e2 e3 e4
            d.push_back(r >> 3);     // f1
        }
        tw[P::T4 + g] = twiddle(theta(d) / 2);
    }
    return tw;
}

// The small ring: [8 blocks][4] and the last level's [64 pairs], path bits (k, e).
std::vector<d2> small_table() {
    std::vector<d2> tw(Small::TN);
    second_pass<8>(tw.data());
    for (int g = 0; g < 64; g++) {
        std::vector<int> d;
        bits(d, g & 7, 3);
        bits(d, g >> 3, 3);
        tw[Small::T4 + g] = twiddle(theta(d) / 2);
    }
    return tw;
}

// Allocates the key spectra of `per_poly` values per key polynomial with the
// twiddles behind them, and uploads those; no room leaves d_fkey null.
int setup_tables(tfhe_ctx* c, size_t per_poly, const std::vector<d2>& tw) {
    const size_t key_bytes = (size_t)c->p.n * 2 * c->p.l * 2 * per_poly * sizeof(d2);
    const size_t bytes = key_bytes + tw.size() * sizeof(d2);
    if (hipMalloc(&c->d_fkey, bytes) != hipSuccess) {
        (void)hipGetLastError();
        c->d_fkey = nullptr;
        return TFHE_OK;
    }
    c->fkey_bytes = bytes;
    c->d_ftw = (uint8_t*)c->d_fkey + key_bytes;
    return hip_check(c, hipMemcpy(c->d_ftw, tw.data(), tw.size() * sizeof(d2), hipMemcpyHostToDevice),
                     "copy twiddles");
}

template <typename T, int R>
int setup_t(tfhe_ctx* c, hipStream_t s) {
    constexpr int LC = Limb<T>::COUNT;
    const int rc = setup_tables(c, (size_t)LC * Plan<R>::M, twiddle_table<R>());
    if (rc || !c->d_fkey) return rc;
    auto k = fft_key_kernel<T, R>;
    hipLaunchKernelGGL(k, dim3(c->p.n * 2 * c->p.l * 2 * LC), dim3(64), 0, s, (const T*)c->d_bsk, (const d2*)c->d_ftw,
                       (d2*)c->d_fkey);
    return hip_check(c, hipGetLastError(), "launch fft_key");
}

int setup_small(tfhe_ctx* c, hipStream_t s) {
    const int rc = setup_tables(c, 2 * Small::M, small_table());
    if (rc || !c->d_fkey) return rc;
    const int total = (int)(c->p.n * 2 * c->p.l * 2 * 2);
    hipLaunchKernelGGL(fft256_key_kernel, dim3((total + 3) / 4), dim3(64), 0, s, (const uint32_t*)c->d_bsk,
                       (const d2*)c->d_ftw, (d2*)c->d_fkey, total);
    return hip_check(c, hipGetLastError(), "launch fft256_key");
}

}  // namespace

// Key spectra and twiddles of a context whose ring has 1024 or 2048
// coefficients, or 256 at 32-bit words (none without room for them: the int8
// path is used then).
int fft_setup(tfhe_ctx* c, hipStream_t s) {
    if (c->p.N == 256 && c->q == 32) return setup_small(c, s);
    if (c->p.N == 1024) return c->q == 32 ? setup_t<uint32_t, 8>(c, s) : setup_t<uint64_t, 8>(c, s);
    if (c->p.N == 2048) return c->q == 32 ? setup_t<uint32_t, 16>(c, s) : setup_t<uint64_t, 16>(c, s);
    return TFHE_OK;
}

// The small ring's transform kernel against the int8 one: linear in the batch
// against steps of 16 ciphertexts per CU.  At n = 64, l = 2 on 256 CUs (step
// 4096), int8 / transform in ms: 2560 0.454 / 0.404, 3072 0.447 / 0.412, 3328
// 0.459 / 0.483, 4352 0.750 / 0.583, 6144 0.783 / 0.727, 6656 0.804 / 0.820, 9216
// 1.32 / 1.08, 10,240 1.33 / 1.21, 14,336 1.66 / 1.64, 18,432 2.17 / 2.13, 22,528
// 2.54 / 2.61.  So it is taken in the first three quarters of the first step and
// the first half of the next four.  At other level counts (l = 3: 2048 0.784 /
// 0.489, 5: 1.21 / 0.69, 1: 0.321 / 0.293) up to half a step.
static bool small_pays(const tfhe_ctx* c, uint32_t B) {
    const uint64_t step = 16ull * (c->prop.multiProcessorCount > 0 ? c->prop.multiProcessorCount : 256);
    if (c->p.l != 2) return B <= step / 2;
    const uint64_t full = B / step, rem = B % step;
    return full == 0 ? rem <= step * 3 / 4 : full <= 4 && rem <= step / 2 && rem > 0;
}

// Whether the context's batches take the transform path at all: with key spectra
// and no tuning knob that asks for a shape of the int8 kernels -- a row pass that
// is not the ring's default or a digit grouping.  (The default row pass and
// "never split", which earlier tunings saved, do not.)
static bool fft_selected(const tfhe_ctx* c) {
    const int default_rp = c->p.N == 2048 ? 8 : c->q == 64 || c->p.N == 256 ? 4 : 16;
    return c->d_fkey && c->digit_blocks == 0 && (c->row_pass == 0 || c->row_pass == default_rp);
}

// Whether a batch of B takes it: if no positive split threshold covers the batch
// and, at N = 256, where it is faster.
bool fft_usable(const tfhe_ctx* c, uint32_t B) {
    if (!fft_selected(c) || (c->p.N == 256 && !small_pays(c, B))) return false;
    return !(c->split_groups > 0 && ((uint64_t)B + 15) / 16 <= (uint64_t)c->split_groups);
}

// A bound on the batches of at most Bmax that do not take it (0: all do).
uint32_t fft_leaves_upto(const tfhe_ctx* c, uint32_t Bmax) {
    const uint32_t cus = c->prop.multiProcessorCount > 0 ? c->prop.multiProcessorCount : 256;
    if (!fft_selected(c) || (c->p.N == 256 && !(Bmax <= 16 * cus && small_pays(c, Bmax)))) return Bmax;
    return c->split_groups > 0 ? (uint32_t)std::min<uint64_t>(Bmax, 16 * (uint64_t)c->split_groups) : 0;
}

int launch_br_fft(tfhe_ctx* c, const void* lwe_in, const void* tv, const int32_t* tv_index, void* big_out, uint32_t B,
                  hipStream_t s) {
    FftArgs a;
    a.lwe = lwe_in;
    a.fkey = (const d2*)c->d_fkey;
    a.tw = (const d2*)c->d_ftw;
    a.tv = tv;
    a.tv_index = tv_index;
    a.out = big_out;
    a.B = (int)B;
    a.n = (int)c->p.n;
    a.l = (int)c->p.l;
    a.bg_bits = (int)c->p.bg_bits;
    a.cus = c->prop.multiProcessorCount > 0 ? c->prop.multiProcessorCount : 256;
    // The ciphertexts per workgroup follow the batch, so that every one is
    // resident if it can be.  At N = 1024, q = 32, on 256 CUs: one (8 waves) up
    // to a ciphertext per CU (2.4 ms at l = 3), two of the same up to two per CU
    // (512: 4.1 ms) and in rounds of those up to six per CU (1024: 8.3 ms, 1500:
    // 12.3; four in 4 waves 14.0), above that four in 4 waves, two workgroups per
    // CU, whose key reads serve four (1600: 14.0 ms, 15.0 in pairs; 2048: 14.1;
    // 4096: 27.7).  What is left after full rounds of those is launched by the
    // same rule: 700 as 512 in pairs and 188 by ones (6.6 ms, 9.1 in one launch of
    // two in 4 waves), 1100 10.9 (13.1), 2300 16.5 (24.3 all by fours), 2900 22.5
    // (23.4), 3600 28.4 (30.5).  At another l, two in 4 waves, three workgroups per
    // CU, stand for the pairs (l = 4: 1500 16.5 ms, 16.9 by fours; 2600 28.2, 28.6
    // all by fours).
    // The gadget levels of the named parameter sets (l = 3 at 32-bit words, 4 at
    // 64-bit) are compile-time where the ring holds several polynomials: one
    // ciphertext took 2.66 ms, 2.88 with l a run-time value, and 512 4.39 and 4.76.
    const int l = (int)c->p.l;
    const uint32_t cus = (uint32_t)a.cus;
    if (c->p.N == 256) {
        hipLaunchKernelGGL(l == 2 ? br_fft256_kernel<2> : br_fft256_kernel<0>, dim3(B), dim3(64), 0, s, a);
        return hip_check(c, hipGetLastError(), "launch br_fft256");
    }
    // The next `count` ciphertexts, per_wg of them per workgroup, in launches of at
    // most 2^22 workgroups of 512 threads: HIP launches no grid of 2^32 work-items.
    uint32_t done = 0;
    const auto part = [&](uint32_t count, uint32_t per_wg, int (*launch)(tfhe_ctx*, const FftArgs&, hipStream_t)) {
        int rc = TFHE_OK;
        while (count && !rc) {
            FftArgs p = a;
            p.lwe = (const uint8_t*)a.lwe + (size_t)done * (a.n + 1) * word_bytes(c);
            if (a.tv_index) p.tv_index = a.tv_index + done;
            p.out = (uint8_t*)a.out + (size_t)done * (c->p.N + 1) * word_bytes(c);
            p.B = (int)std::min(count, per_wg << 22);
            done += (uint32_t)p.B;
            count -= (uint32_t)p.B;
            rc = launch(c, p, s);
        }
        return rc;
    };
    //                                                       T         R   W  G  L  KD twiddles WPE
    if (c->q == 32) {
        if (c->p.N == 2048) return part(B, 1, l == 3 ? launch_fft_t<Cfg<uint32_t, 16, 8, 1, 3, 2, TW_LDS>>
                                                     : launch_fft_t<Cfg<uint32_t, 16, 8, 1, 0, 1, TW_LDS>>);
        const uint32_t fours = B % (8 * cus) > 6 * cus ? B : B - B % (8 * cus);
        int rc = part(fours, 4, launch_fft_t<Cfg<uint32_t, 8, 4, 4, 0, 1, TW_LDS>>);
        const uint32_t rest = B - done;
        if (rc || !rest) return rc;
        if (l != 3) return rest > 2 * cus ? part(rest, 2, launch_fft_t<Cfg<uint32_t, 8, 4, 2, 0, 1, TW_LDS, 3>>)
                                          : part(rest, 1, launch_fft_t<Cfg<uint32_t, 8, 8, 1, 0, 2, TW_REG>>);
        const uint32_t pairs = rest % (2 * cus) > cus ? rest : rest - rest % (2 * cus);
        rc = part(pairs, 2, launch_fft_t<Cfg<uint32_t, 8, 8, 2, 3, 4, TW_REG>>);
        return rc ? rc : part(B - done, 1, launch_fft_t<Cfg<uint32_t, 8, 8, 1, 3, 8, TW_REG>>);
    }
    if (c->p.N == 2048) return part(B, 1, l == 4 ? launch_fft_t<Cfg<uint64_t, 16, 8, 1, 4, 2, TW_GLOBAL>>
                                                 : launch_fft_t<Cfg<uint64_t, 16, 8, 1, 0, 1, TW_GLOBAL>>);
    return part(B, 1, launch_fft_t<Cfg<uint64_t, 8, 8, 1, 0, 4, TW_REG>>);
}
