// Batched mixture objective and adjoint gradient on MFMA (gfx950).
//
// For a point x and component k the kernel forms delta = x - mu_k (centring
// before the product keeps FP32 cancellation out of the contraction) and
// u_k = P_k delta with P_k the precision matrix.  Then
//   q_k = delta . u_k,   l_k = log c_k - q_k / 2           (Gaussian)
//                        l_k = log c_k - (nu+d)/2 log1p(q_k/nu)  (Student-t)
//   f = log sum_k exp(l_k),   grad f = -sum_k r_k s_k u_k,
// with r = softmax(l) and s_k = 1 (Gaussian) or (nu+d)/(nu+q_k) (Student-t).
// The same contraction therefore yields the value and its reverse-mode
// gradient: 2 K d^2 MFMA flops per point whether or not the gradient is kept.
//
// Work layout: a tile of 32 points in two 16-point blocks per wave (direct
// evaluations may take 16-point half tiles; several waves share a line-search
// tile or one of a small direct evaluation, each contracting a contiguous part
// of the components, and their partial states are merged in wave order).  In
// float32 (the form in two f16 parts is described below) v_mfma_f32_16x16x4f32
// computes U^T (DP x 16) = P' (DP x DP) * Delta^T (DP x 16), P' the precision
// matrix with its rows permuted: lane l
// supplies P[pi(16mb + l%16)][4ks + l/16] (A operand), pi(16mb + 4a + b) =
// 4(4mb + b) + a, and delta[point l%16][4ks + l/16] (B operand), and receives
// u at point l%16 and coordinate pi(16mb + 4(l/16) + r) = 4(4mb + r) + l/16,
// r = 0..3.  So each lane holds u at the very coordinates it holds delta at,
// and the quadratic form delta . u needs no second copy of delta.
// Components are streamed; the log-sum-exp runs online in base 2, and its
// reference moves (rescaling the gradient sums) only when a term exceeds it
// by 2^kLseSlack.  Mixtures with d <= 8 take a VALU path instead, one point
// per lane in 64-point tiles.
//
// The closed-form test functions of Appendix D share the kernel's tiling,
// point generation and epilogues; their value (and analytic gradient) is a
// sum over coordinates evaluated on the VALU, two lanes per point.  Their
// central differences have a kernel of their own (closed_fd_kernel).
#include <math.h>

#include <type_traits>

#include "kernels.h"
#include "ranges.h"

namespace chisao {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int NB = 2;          // 16-point blocks per wave
constexpr int kTilePts = 32;  // points per wave in the MFMA tiles
using AllBlocks = std::integral_constant<int, NB>;
using OneBlock = std::integral_constant<int, 1>;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
// online log-sum-exp: headroom (log2) a term may exceed the running reference
// before the reference moves
constexpr float kLseSlack = 8.0f;
// The reference a sum starts from.  A part of a split sum that does not begin
// with component 0 starts from a finite one, so that a component whose term is
// 2^-inf (its quadratic form overflowed) adds nothing to it, as it does further
// on in an unsplit sum; from -inf the sum of such a part would be a NaN.
__device__ __forceinline__ float lse_start(bool at_component_0) { return at_component_0 ? -INFINITY : -__FLT_MAX__; }
// Student-t kernel in base 2: log2(1 + q / nu) with the hardware log2.
// Rounding 1 + q / nu costs at most 2^-24 absolute in the argument, i.e.
// 1.7e-7 in the log, which the factor (nu + d) / 2 scales to a few 1e-6:
// well inside the FP32 error of the quadratic form itself.
__device__ __forceinline__ float student_log2(float q, float inv_nu) { return __log2f(fmaf(q, inv_nu, 1.0f)); }

// Pointers into the global address space (plain loads through them compile
// to global_load, which only the vector-memory counter tracks).
typedef const float __attribute__((address_space(1))) gfloat;
typedef const f32x4 __attribute__((address_space(1))) gf32x4;
typedef const f32x2 __attribute__((address_space(1))) gf32x2;
__device__ __forceinline__ const gfloat *as_global(const float *p) { return (const gfloat *)p; }
// A read-only table whose address is the same in every lane, in the constant
// address space: loads at wave-uniform offsets compile to scalar loads.
typedef const float __attribute__((address_space(4))) cfloat;
__device__ __forceinline__ const cfloat *uniform_const(const float *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32);
    return reinterpret_cast<const cfloat *>(u);
}

template <int MB>
__device__ __forceinline__ void load_frag(const gfloat *p, float out[MB]) {
    if constexpr (MB == 4) {
        const f32x4 v = *reinterpret_cast<const gf32x4 *>(p);
        out[0] = v[0]; out[1] = v[1]; out[2] = v[2]; out[3] = v[3];
    } else if constexpr (MB == 2) {
        const f32x2 v = *reinterpret_cast<const gf32x2 *>(p);
        out[0] = v[0]; out[1] = v[1];
    } else {
        out[0] = *p;
    }
}

// Raw buffer resource over a read-only table of `bytes` bytes (gfx9
// descriptor; loads past the end return zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t table_rsrc(const float *base, uint32_t bytes) {
    // the table pointer is the same in every lane; passing it through
    // readfirstlane puts the resource in scalar registers
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float *>(u), (short)0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

template <int MB>
__device__ __forceinline__ void load_frag_buf(__amdgpu_buffer_rsrc_t rs, int voff, int soff, float out[MB]) {
    if constexpr (MB == 4) {
        const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0));
        out[0] = v[0]; out[1] = v[1]; out[2] = v[2]; out[3] = v[3];
    } else if constexpr (MB == 2) {
        const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
        out[0] = v[0]; out[1] = v[1];
    } else {
        out[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
    }
}

// One component's operands in registers: precision-matrix fragments,
// centre coordinates in B-operand lane order, log2 weight.
template <int KS, int MB>
struct CompRegs {
    float pa[KS][MB];
    float muB[KS];
    float lc2;
};

// ---------------------------------------------------------------------------
// Two-part contraction.  u = P delta with each operand as a sum of two f16
// values, x = h + l, h = f16(x) and l = f16(x - h) (round to nearest): the
// three products l_P h_d + h_P l_d + h_P h_d on the f16 matrix core (16 times
// the rate of the float32 one), summed in float32; up to d = kTwoPartLowD the
// fourth, l_P l_d, as well.  h and l hold 23 of the 24 significant bits of x, so a term
// is off by about a rounding of float32, and a sum goes through 3 DP / 32
// accumulations; the float32 instruction rounds once a coordinate.
// Which of the two is further off depends on the matrices; the rule below takes
// two parts where float32 is.  Errors of gradients against float64, two parts
// over float32 (2-norm over 24 to 300 matrices with log-uniform spectra over a
// factor 10 and 20, points of their component): d = 20 1.00 and 1.04, 21 1.00
// and 1.03, 24 0.94 and 0.96, 28 0.89 and 0.92, 32 0.84 and 0.86, 36 0.88 and
// 0.85, 48 0.77 and 0.75, 53 0.92 and 0.95, 64 0.84 and 0.85; values 0.94 to
// 1.05.  Next to the end of an ascent, where delta lies along P's small
// eigenvalues (P^-1 z, z normal): d = 20 1.06 and 1.06, 24 0.97 and 1.02, 28
// 0.94 and 0.97, 32 0.86 and 0.93, 36 0.91 and 0.86, 48 0.81 and 0.79, 64 0.89
// and 0.92, so that populations take it from d = 24 on only.  Outside of the
// rule: d = 19 1.02 and 1.06, 17 1.05 to 1.12; spectra over 10^4 1.3 to 1.5,
// with one small eigenvalue of 10^-4 values 3.4; multiples of the identity 1.9,
// for there float32 rounds delta and one product (2e-8 against 4e-8).  Without
// l_P l_d the gradients of d = 49 were 0.96 and 0.98, at the end of an ascent
// 1.01 and 1.03, and at d = 12 four products gave 9e-8 against 7e-8: so
// kTwoPartLowD, and DP = 16 stays in float32.
//
// What bounds it: the matrix core's rate under load (the products alone ran at
// 1480 TFLOP/s) plus the vector instructions that split delta (two conversions
// and two mixed multiply-adds a pair), which the matrix core does not hide.
// 262144 points of the d = 64, K = 128 mixture, value and gradient: 2216 us in
// float32, 856 us in two parts; a cycle of its 65536 samples 42.1 -> 19.1 ms
// (before the shared components of large launches, see SHARE).
//
// f16 has 5 exponent bits, so operands are scaled by powers of two (exact):
// coordinate j of points and centres by xs_j = 2^(e_j + b), the matrices by
// 2^(kTwoPartP - e_i - e_j), with 4^e_j about max_k (P_k)_jj, so that scaled
// diagonals are at most 2^(kTwoPartP + 1) and, the matrices being positive
// definite, no entry is larger; b puts the largest distance between two points
// of the box and the centres, in those units, at no more than 2^kTwoPartX.
// What a part holds is then good to 2^-25 absolutely where its own 11 bits do
// not reach.  The rule below keeps that harmless: problems whose box spans
// more than 2^kTwoPartSpan of the narrowest component's standard deviations,
// or whose diagonals differ by more than 2^kTwoPartRatio, stay in float32.  So
// do, for the errors above, d < kTwoPartMinD; a component fewer than three
// quarters of whose off-diagonal entries exceed 2^-16 sqrt(P_ii P_jj) (diagonal,
// banded and block matrices: float32 rounds a sum only where it adds something);
// and one whose mean P_jj (P^-1)_jj is above two_part_kappa (the square by which
// a point's terms exceed their sum; up to 1.8 for spectra over 10, 2.4 over 20,
// 4.6 in the mean over 100), which prepare_kernel finds.
// Next to a centre at or near 0 float32 holds every digit of a small delta, and
// 2^-25 is too much: a point within 4 2^-b standard deviations of a centre is
// contracted again with that component, its delta scaled up (a few evaluations
// at the end of an ascent; a branch that other waves skip).  A
// point far outside the box carries a power of two of its own (1 for any other
// point), so nothing overflows that would not in float32.
// ---------------------------------------------------------------------------
constexpr int kTwoPartMinD = 20, kTwoPartLowD = 52;
constexpr float two_part_kappa(int d) { return d < 24 ? 1.9f : 2.5f; }
constexpr int kTwoPartP = 12, kTwoPartX = 13, kTwoPartSpan = 10, kTwoPartRatio = 12, kTwoPartMaxB = 12;

bool two_part_scales(int d, int DP, int K, const float *mu, const float *prec, const float *lo, const float *hi,
                     float *xs, float *kq) {
    if (d < kTwoPartMinD) return false;
    int e[64];
    double span = 0.0;
    for (int j = 0; j < d; ++j) {
        double pmax = 0.0, a = lo[j], z = hi[j];
        for (int k = 0; k < K; ++k) {
            pmax = fmax(pmax, (double)prec[((size_t)k * d + j) * d + j]);
            a = fmin(a, (double)mu[(size_t)k * d + j]);
            z = fmax(z, (double)mu[(size_t)k * d + j]);
        }
        if (!(pmax > 0.0)) return false;  // not positive definite: reported by launch_prepare
        e[j] = (int)lrint(0.5 * log2(pmax));
        if (e[j] < -40 || e[j] > 40) return false;
        span = fmax(span, ldexp(z - a, e[j]));
    }
    for (int k = 0; k < K; ++k)
        for (int j = 0; j < d; ++j)
            if (!(ldexp((double)prec[((size_t)k * d + j) * d + j], -2 * e[j]) >= ldexp(1.0, -kTwoPartRatio)))
                return false;
    if (!(span <= ldexp(1.0, kTwoPartSpan))) return false;
    // (in units of the 2^e_j, where float32 does not overflow)
    float unit[64], diag[64];
    for (int j = 0; j < d; ++j) unit[j] = (float)ldexp(1.0, -e[j]);
    for (int k = 0; k < K; ++k) {
        const float *P = prec + (size_t)k * d * d;
        int full = -d;  // the diagonal's own
        for (int j = 0; j < d; ++j) diag[j] = 0x1p-32f * (P[j * d + j] * unit[j] * unit[j]);
        for (int i = 0; i < d; ++i) {
            const float ui = unit[i], di = 0x1p32f * diag[i];
            for (int j = 0; j < d; ++j) {
                const float v = P[i * d + j] * ui * unit[j];
                full += v * v >= di * diag[j];
            }
        }
        if (4 * full < 3 * d * (d - 1)) return false;
    }
    const int b = span > 0.0 ? (int)fmin((double)kTwoPartMaxB, kTwoPartX - ceil(log2(span))) : kTwoPartMaxB;
    for (int j = 0; j < DP; ++j) xs[j] = j < d ? (float)ldexp(1.0, e[j] + b) : 1.0f;
    *kq = (float)ldexp(1.0, -2 * b - kTwoPartP);
    return true;
}

// The coordinate a lane of row g holds at position i of its DP / 4: every
// fourth one, the operand order of the float32 instruction (K = 4).  The f16
// instruction (K = 32) takes a lane's positions 8 s .. 8 s + 7 in step s;
// which coordinates those are is free as long as both operands agree, and this
// choice spreads d < DP evenly over the rows (with 16 in a row per lane the
// values of d = 33 were 14% further off, from longer chains in delta . u).
// The accumulators of block mb, with the rows of P permuted alike, are the
// lane's positions 4 mb .. 4 mb + 3.
__device__ __forceinline__ constexpr int lane_coord(int i, int g) { return 4 * i + g; }

// Eight values of a lane as two f16 parts.  neg1 is -1 in a scalar register
// the compiler cannot see through, which makes h - x one v_fma_mix_f32 (with a
// literal -1 it converts h back and subtracts, one instruction more).
__device__ __forceinline__ void two_parts(const float *x, float neg1, f16x8 &hi, f16x8 &lo) {
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const f32x2 v = {x[j], x[j + 1]};
        const f16x2 h = __builtin_convertvector(v, f16x2);
        const f32x2 r = {__builtin_fmaf((float)h[0], neg1, v[0]), __builtin_fmaf((float)h[1], neg1, v[1])};
        const f16x2 l = __builtin_convertvector(r, f16x2);
        hi[j] = h[0]; hi[j + 1] = h[1];
        lo[j] = l[0]; lo[j + 1] = l[1];
    }
}

// One component's operands of the two-part contraction: fragments of both
// parts ([part][K step][row block]), centre coordinates, log2 weight.
template <int DP>
struct TwoPartRegs {
    static constexpr int KS = DP / 4, MB = DP / 16, S = DP / 32;
    f16x8 pa[2][S][MB];
    float muB[KS];
    float lc2;
};

// ---------------------------------------------------------------------------
// Closed-form test functions (Appendix D; each negated so that its optimum is
// a maximum).  cf_partial sums one lane's share of the coordinates, c = c0,
// c0 + 2, ... < d, into two accumulators (Ackley needs two sums, the others
// one); cf_value turns the totals into f; cf_grad gives df/dx_c from the
// totals.  Non-differentiable points (Ackley's origin, Bukin N.6's ridge)
// get a zero gradient term.
// ---------------------------------------------------------------------------
constexpr float kTwoPi = 6.283185307179586f;
constexpr float kInvPi = 0.3183098861837907f;
constexpr float kInvPi2 = 0.10132118364233778f;  // 1 / pi^2

__device__ __forceinline__ float sign_of(float v) { return (float)((v > 0.0f) - (v < 0.0f)); }

// sin(u)^20 and sin(u)^19 (Michalewicz, m = 10)
__device__ __forceinline__ void pow20(float su, float &p20, float &p19) {
    const float s2 = su * su, s4 = s2 * s2, s8 = s4 * s4, s16 = s8 * s8;
    p20 = s16 * s4;
    p19 = s16 * s2 * su;
}

// The transcendental factors of coordinate c's term, which depend on x_c alone ...
__device__ __forceinline__ void cf_factors(int fam, int c, float v, float &t1, float &t2) {
    t1 = t2 = 0.0f;
    switch (fam) {
        case CHISAO_RASTRIGIN:
        case CHISAO_ACKLEY: t1 = cospif(2.0f * v); break;
        case CHISAO_SCHWEFEL: t1 = sinf(sqrtf(fabsf(v))); break;
        case CHISAO_MICHALEWICZ: {
            float p19;
            // sin(i x^2 / pi) = sinpi(i x^2 / pi^2): exact range reduction
            pow20(sinpif((float)(c + 1) * v * v * kInvPi2), t2, p19);
            t1 = sinf(v);
            break;
        }
    }
}

// ... and that term, added to the accumulators (prev: x_{c-1}, for c > 0).
__device__ __forceinline__ void cf_add(int fam, int c, float v, float prev, float t1, float t2, float &a, float &b) {
    switch (fam) {
        case CHISAO_RASTRIGIN: a += v * v - 10.0f * t1; break;
        case CHISAO_ACKLEY:
            a += v * v;
            b += t1;
            break;
        case CHISAO_SCHWEFEL: a += v * t1; break;
        case CHISAO_STYBLINSKI_TANG: {
            const float v2 = v * v;
            a += v2 * v2 - 16.0f * v2 + 5.0f * v;
            break;
        }
        case CHISAO_MICHALEWICZ: a += t1 * t2; break;
        case CHISAO_TRID:
            a += (v - 1.0f) * (v - 1.0f);
            if (c > 0) b += v * prev;
            break;
    }
}

__device__ __forceinline__ float cf_bukin(float x0, float x1) {
    return 100.0f * sqrtf(fabsf(x1 - 0.01f * x0 * x0)) + 0.01f * fabsf(x0 + 10.0f);
}

// f(std::integral_constant<int, fam>) for the functions that are sums over the
// coordinates, so that loops over them hold one function's term and no switch
template <class F>
__device__ __forceinline__ void cf_dispatch(int fam, F &&f) {
    switch (fam) {
        case CHISAO_RASTRIGIN: f(std::integral_constant<int, CHISAO_RASTRIGIN>{}); break;
        case CHISAO_ACKLEY: f(std::integral_constant<int, CHISAO_ACKLEY>{}); break;
        case CHISAO_SCHWEFEL: f(std::integral_constant<int, CHISAO_SCHWEFEL>{}); break;
        case CHISAO_STYBLINSKI_TANG: f(std::integral_constant<int, CHISAO_STYBLINSKI_TANG>{}); break;
        case CHISAO_MICHALEWICZ: f(std::integral_constant<int, CHISAO_MICHALEWICZ>{}); break;
        case CHISAO_TRID: f(std::integral_constant<int, CHISAO_TRID>{}); break;
    }
}

__device__ __forceinline__ void cf_partial(int fam, int d, const float *x, int c0, float &a, float &b) {
    a = 0.0f;
    b = 0.0f;
    if (fam == CHISAO_BUKIN6) {
        if (c0 == 0) a = cf_bukin(x[0], x[1]);
        return;
    }
    cf_dispatch(fam, [&](auto fc) {
        for (int c = c0; c < d; c += 2) {
            float t1, t2;
            cf_factors(fc.value, c, x[c], t1, t2);
            cf_add(fc.value, c, x[c], c > 0 ? x[c - 1] : 0.0f, t1, t2, a, b);
        }
    });
}

__device__ __forceinline__ float cf_value(int fam, int d, float a, float b) {
    switch (fam) {
        case CHISAO_RASTRIGIN: return -(10.0f * (float)d + a);
        case CHISAO_ACKLEY: {
            const float r = sqrtf(a / (float)d);
            return 20.0f * expf(-0.2f * r) + expf(b / (float)d) - 20.0f - 2.718281828459045f;
        }
        case CHISAO_SCHWEFEL: return -(418.9829f * (float)d - a);
        case CHISAO_STYBLINSKI_TANG: return -0.5f * a;
        case CHISAO_MICHALEWICZ: return a;
        case CHISAO_TRID: return -(a - b);
        case CHISAO_BUKIN6: return -a;
        default: return __builtin_nanf("");
    }
}

__device__ __forceinline__ float cf_grad(int fam, int d, const float *x, int c, float a, float b) {
    const float v = x[c];
    switch (fam) {
        case CHISAO_RASTRIGIN: return -(2.0f * v + 10.0f * kTwoPi * sinpif(2.0f * v));
        case CHISAO_ACKLEY: {
            const float r = sqrtf(a / (float)d);
            const float t1 = r > 0.0f ? -20.0f * 0.2f * expf(-0.2f * r) * v / ((float)d * r) : 0.0f;
            return t1 - expf(b / (float)d) * kTwoPi * sinpif(2.0f * v) / (float)d;
        }
        case CHISAO_SCHWEFEL: {
            const float r = sqrtf(fabsf(v));
            return sinf(r) + 0.5f * r * cosf(r);
        }
        case CHISAO_STYBLINSKI_TANG: return -0.5f * (4.0f * v * v * v - 32.0f * v + 5.0f);
        case CHISAO_MICHALEWICZ: {
            const float ci = (float)(c + 1), un = ci * v * v * kInvPi2;  // u / pi
            float p20, p19;
            pow20(sinpif(un), p20, p19);
            return cosf(v) * p20 + sinf(v) * 20.0f * p19 * cospif(un) * (2.0f * ci * v * kInvPi);
        }
        case CHISAO_TRID:
            return -2.0f * (v - 1.0f) + (c > 0 ? x[c - 1] : 0.0f) + (c + 1 < d ? x[c + 1] : 0.0f);
        case CHISAO_BUKIN6: {
            const float u = x[1] - 0.01f * x[0] * x[0], r = sqrtf(fabsf(u));
            const float w = r > 0.0f ? sign_of(u) / r : 0.0f;  // d sqrt|u| / du = w / 2
            return c == 0 ? x[0] * w - 0.01f * sign_of(x[0] + 10.0f) : -50.0f * w;
        }
        default: return __builtin_nanf("");
    }
}

constexpr int kMaxClass = 256;  // problems per class (LDS budget: 2 waves per SIMD)
// waves per line-search tile: line-search launches are small, so their time
// is one tile's pass over the components, which four waves share; the closed
// forms have no component loop to split
template <int DP, int FAM>
constexpr int trial_split() { return (FAM < kFamClosed && DP != kAluDP) ? 4 : 1; }

__device__ __forceinline__ int job_count(const EvalArgs &a, int p, const ProblemDesc &pd) {
    if (a.ext_n >= 0) return a.ext_n;
    if (a.nz_kind == 1 && !(pd.noise_sigma > 0.0f)) return 0;
    if (a.need_bit && !(pd.phase_mask & (uint32_t)a.need_bit)) return 0;
    if ((a.step_limit == 1 && a.step >= pd.n_cloud) || (a.step_limit == 2 && a.step >= pd.n_anti)) return 0;
    return a.list_id >= 0 ? a.D.ctl[p].count[a.list_id] : pd.N;
}
__device__ __forceinline__ int centres(const EvalArgs &a, const ProblemDesc &pd) {
    switch (a.vc_kind) {
        case kVcTrialRest: return max(0, min(a.trial_cnt, pd.ls_max - a.trial_lo));
        case kVcProbes: return pd.M;
        default: return 1;
    }
}
// inclusive prefix sum over the wave
template <class T>
__device__ __forceinline__ T wave_scan(T v) {
    const int l = threadIdx.x % kWave;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const T u = __shfl_up(v, o, kWave);
        if (l >= o) v += u;
    }
    return v;
}
// tiles of ppw points: jpw jobs per tile, or wpj tiles per job
__device__ __forceinline__ long tiles_of(int count, int V, int ppw, int &jpw, int &wpj) {
    if (V <= 0 || count <= 0) {
        jpw = 1;
        wpj = 1;
        return 0;
    }
    if (V <= ppw) {
        jpw = ppw / V;
        wpj = 1;
        return (count + jpw - 1) / jpw;
    }
    jpw = 1;
    wpj = (V + ppw - 1) / ppw;
    return (long)count * wpj;
}
// Line-search launches of at most this many full tiles run half tiles (16
// points, one MFMA column block): twice the tiles, each with half the matrix
// work per component, still one workgroup per CU, so the launch, whose time is
// one tile's pass over the components, takes about half as long.
constexpr int kHalfTileMax = 128;

// Direct evaluations of few points (caller memory) split a tile's components
// too.  One wave alone goes through K components in a row, so such a launch
// took one pass however few its points: 118 us for 1 to 8192 points at d = 64,
// K = 128.  Up to 128 full tiles, eight waves take a half tile (16 points), at
// most one workgroup per CU: 23 us for one point, 29 us for 4096.  Up to 512
// tiles, four waves take a full tile, two waves per SIMD: 77 us against 128
// for 16384 points; at 1024 tiles it is 161 against 149.  Narrower components
// keep more waves per SIMD resident, so there four waves pay up to 1024 tiles
// if there are components enough to share (d = 32: 60 us against 69 at K =
// 128, 29.7 against 31.8 at 48, but 17.7 against 16.9 at 16; d = 16, K = 128:
// 35.8 against 47.4).  Populations are left as they are: a problem's results
// do not depend on how many samples are evaluated together.
int direct_split(int DP, int family, int K, long tiles) {
    if (family >= kFamClosed || DP == kAluDP) return 0;
    if (tiles <= 128) return kSplitHalf;
    return tiles <= 512 || (tiles <= 1024 && DP <= 32 && K >= 32) ? kSplitFull : 0;
}

// SPLIT waves share a tile: each contracts a contiguous part of the
// components and the first (lead) wave merges the partial log-sum-exp states
// in wave order, then runs the epilogue.  Line-search launches are small (a
// few thousand points), so their time is the latency of one tile's pass over
// all K components; splitting the components cuts that latency.
//
// SHARE (large two-part launches): four waves take 32 points each of a
// 128-point tile and go through the components together.  A component's
// fragments are brought to LDS once for the four, by direct loads into the half
// of the buffer that is not being read, instead of through the vector cache
// four times (16 KB each for about 2000 cycles of work): 262144 points, K =
// 128, values and gradients 905 -> 867 us, values 859 -> 808; a cycle of 65536
// samples 20.2 -> 19.0 ms.  (The compiler cannot tell the halves apart and
// waits for the loads of component k + 1 before it reads component k, so what
// hides their latency is the other workgroup of the CU, not this one's work.)
//
// Registers: two waves per SIMD leave 256 a lane.  In two parts at width 64 the
// line-search kernel with gradients keeps 11 more (Gaussian) or 12 (Student-t)
// in scratch, the direct one whose four waves share a tile 3 or 7, the
// Student-t probe kernel 3: written once a tile, at most one read back a
// component beside its 48 matrix instructions.  The float32 forms need none.
constexpr int kShareWaves = 4;
template <int DP, int FAM, bool GRAD, int CENTER, bool FD, int SPLIT, bool HT, bool H16, bool SHARE = false>
__global__ __launch_bounds__(64 * (SHARE ? kShareWaves : SPLIT)) __attribute__((amdgpu_waves_per_eu(2))) void eval_kernel(EvalArgs a) {
    constexpr int KS = DP / 4;
    constexpr int MB = DP / 16;
    constexpr bool CLOSED = FAM >= kFamClosed;
    // small mixtures: one lane per point on the VALU, 64 points per tile
    constexpr bool ALU = !CLOSED && DP == kAluDP;
    constexpr int PPW = ALU ? kWave : (SHARE ? kShareWaves * kTilePts : kTilePts);
    constexpr int LD = DP + 1;  // padded row: conflict-free column reads
    static_assert(!SHARE || (DP == 64 && H16 && SPLIT == 1 && !HT && !FD && CENTER != kTrial), "shared components: large launches");
    // (SHARE) a component in LDS: fragments, scaled centre
    constexpr int kCompF = SHARE ? DP * DP + DP : 0;
    // split direct evaluations: every wave's partial state goes through LDS and
    // all waves merge; split line-search tiles: waves 1.. hand theirs to the first
    constexpr bool DSPLIT = CENTER == kDirect && SPLIT > 1;
    constexpr int NP = SPLIT == 1 ? 1 : (DSPLIT ? SPLIT : SPLIT - 1), NBP = HT ? 1 : NB;
    __shared__ float s_pm[NP][NBP][kWave], s_ps[NP][NBP][kWave];             // partial max / sum
    __shared__ float s_pg[(SPLIT > 1 && GRAD) ? NP * NBP * KS : 1][kWave];  // partial gradient sums
    // (SHARE) the points, then two components in turn, then the gradients
    constexpr int kPtsF = PPW * LD > 2 * kCompF ? PPW * LD : 2 * kCompF;
    __shared__ __align__(16) float s_pts[kPtsF];
    __shared__ float s_grad[GRAD && !SHARE ? PPW * LD : 1];
    float *s_g = SHARE ? s_pts : s_grad;
    __shared__ float s_f[PPW];
    __shared__ float s_den[PPW];
    __shared__ int s_s[PPW];    // sample (or caller row) per point, -1 when the lane is idle
    __shared__ int s_c[PPW];    // centre index within the job
    __shared__ int s_st[PPW];   // stencil index within the centre
    __shared__ int s_pass[PPW];
    __shared__ int s_acc[PPW];
    __shared__ int s_pref[kMaxClass + 1];
    __shared__ int s_ppw;  // points per tile in this launch
    // line search: each point's sample row and gradient before the step, and
    // the partial sums of g . (x_trial - x) over blocks of four coordinates,
    // all gathered while the points are generated
    constexpr bool TRIAL = CENTER == kTrial;
    // half tiles: only split line-search tiles, whose launches are latency-bound
    static_assert(!(TRIAL && FD), "line-search trials take no finite differences");
    constexpr bool HALF = TRIAL && SPLIT > 1;
    // HT: half tiles throughout (direct evaluations; the autotuner's choice
    // for classes whose launches hold too few full tiles to fill the chip)
    static_assert(!HT || (CENTER == kDirect && !FD && !CLOSED && !ALU), "half tiles: direct MFMA only");
    static_assert(!DSPLIT || (!FD && !CLOSED && !ALU), "split direct evaluations: MFMA only");
    __shared__ int s_pref2[HALF ? kMaxClass + 1 : 1];  // tile prefix in half tiles
    // jobs picked out of a list by their flag: launches of Phase 1 only
    constexpr bool FLAGS = TRIAL || (FD && CENTER == kDirect);
    __shared__ int s_live[1];
    __shared__ float s_x0[TRIAL ? PPW * LD : 1];
    __shared__ float s_g0[TRIAL ? PPW * LD : 1];
    __shared__ float s_dp[TRIAL ? PPW * KS : 1];

    const Dev &D = a.D;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const bool lead = SPLIT == 1 || wv == 0;
    const int tl = SHARE ? (int)threadIdx.x : lane;      // one thread per point of the tile
    const int wp = SHARE ? wv * kTilePts : 0;            // the wave's first point
    constexpr int kTl = SHARE ? kShareWaves * kWave : kWave;
    const int g = lane >> 4, n = lane & 15;
    const bool ext = a.ext_n >= 0;
    // Tile prefix over the problems of the class.  Line-search launches are
    // short and many, and a VALU-path launch is short whatever its kind, so
    // there the first wave computes it, one problem per lane: the problems'
    // counts are read in parallel, not one dependent load after another.  The
    // other launches are long; there one thread walks the problems (the wave
    // version's extra scalar registers cost the long launches' component loop
    // more than the walk takes).
    if constexpr (TRIAL || ALU) {
        if (threadIdx.x < kWave) {
            int carry = 0, carry2 = 0;
            if (lane == 0) s_pref[0] = s_pref2[0] = 0;
            for (int j0 = 0; j0 < a.n_cls; j0 += kWave) {
                const int j = j0 + lane;
                int t = 0, t2 = 0;
                if (j < a.n_cls) {
                    const int p = a.cls[j];
                    const ProblemDesc &pd = D.pd[p];
                    const int jobs = job_count(a, p, pd);
                    const int V = centres(a, pd) * (FD ? 2 * pd.d : 1);
                    int jpw, wpj;
                    t = (int)tiles_of(jobs, V, PPW, jpw, wpj);
                    if constexpr (HALF) t2 = (int)tiles_of(jobs, V, PPW / 2, jpw, wpj);
                    // evaluation counts, once per launch (block 0) rather than per tile
                    if (blockIdx.x == 0 && !ext && jobs > 0 && !(FLAGS && a.by_flag)) {
                        const unsigned long long nv = (unsigned long long)jobs * (unsigned long long)V;
                        atomicAdd(&D.ctl[p].evals, nv);
                        atomicAdd(&D.prof[FD ? 3 : CENTER], nv);
                    }
                }
                const int inc = wave_scan(t), inc2 = HALF ? wave_scan(t2) : 0;
                if (j < a.n_cls) {
                    s_pref[j + 1] = carry + inc;
                    if constexpr (HALF) s_pref2[j + 1] = carry2 + inc2;
                }
                carry += __shfl(inc, kWave - 1, kWave);
                if constexpr (HALF) carry2 += __shfl(inc2, kWave - 1, kWave);
            }
            if (HALF && lane == 0) s_ppw = carry <= kHalfTileMax ? PPW / 2 : PPW;
        }
    } else if (threadIdx.x == 0) {
        int acc = 0;
        unsigned long long pts = 0;
        s_pref[0] = 0;
        for (int j = 0; j < a.n_cls; ++j) {
            const int p = a.cls[j];
            const ProblemDesc &pd = D.pd[p];
            const int Vs = FD ? 2 * pd.d : 1;
            const int jobs = job_count(a, p, pd);
            int jpw, wpj;
            acc += (int)tiles_of(jobs, centres(a, pd) * Vs, HT ? PPW / 2 : PPW, jpw, wpj);
            s_pref[j + 1] = acc;
            // evaluation counts, once per launch (block 0) rather than per tile
            if (blockIdx.x == 0 && !ext && jobs > 0 && !(FLAGS && a.by_flag)) {
                const unsigned long long nv = (unsigned long long)jobs * centres(a, pd) * Vs;
                atomicAdd(&D.ctl[p].evals, nv);
                pts += nv;
            }
        }
        if (blockIdx.x == 0 && pts) atomicAdd(&D.prof[FD ? 3 : CENTER], pts);
    }
    __syncthreads();
    const int ppw = HALF ? s_ppw : (HT ? PPW / 2 : PPW);
    const int *pref = (HALF && ppw < PPW) ? s_pref2 : s_pref;
    const int n_tiles = pref[a.n_cls];

    // Tile order.  Linear: block b takes tiles b, b + G, ...  XCD-chunked:
    // workgroups are dispatched round-robin over the 8 XCDs, so block b runs on
    // XCD b % 8; that XCD's blocks take a contiguous eighth of the tile range,
    // which in class order spans fewer problems, so each XCD's L2 holds the
    // precision matrices of fewer problems.
    int t0 = 0, first = blockIdx.x, stride = gridDim.x, span = n_tiles;
    if (a.order == 1) {
        constexpr int kXcd = 8;
        span = (n_tiles + kXcd - 1) / kXcd;
        t0 = (blockIdx.x % kXcd) * span;
        first = blockIdx.x / kXcd;
        stride = gridDim.x / kXcd;
    }
    for (int it = first; it < span; it += stride) {
        const int tile = t0 + it;
        if (tile >= n_tiles) break;
        // ---- the tile's problem ---------------------------------------------
        int lo_j = 0, hi_j = a.n_cls - 1;
        while (lo_j < hi_j) {
            const int mid = (lo_j + hi_j + 1) >> 1;
            if (pref[mid] <= tile) lo_j = mid;
            else hi_j = mid - 1;
        }
        // every lane finds the same problem; saying so keeps its descriptor,
        // table pointers and the component loop's addressing in scalar
        // registers instead of per-lane 64-bit arithmetic
        const int p = __builtin_amdgcn_readfirstlane(a.cls[lo_j]);
        const ProblemDesc &pd = D.pd[p];
        const int ltile = tile - pref[lo_j];
        const int d = pd.d;
        const int count = job_count(a, p, pd);
        const int Vc = centres(a, pd);
        const int r0 = a.vc_kind == kVcTrialRest ? a.trial_lo : 0;
        const int Vs = FD ? 2 * d : 1;
        const int V = Vc * Vs;
        int jpw, wpj;
        (void)tiles_of(count, V, ppw, jpw, wpj);
        const uint32_t kcyc = (uint32_t)D.ctl[p].k + 1u;
        const float sigma = (CENTER == kProbe) ? D.ctl[p].sigma : 0.0f;
        const int xs = a.x_stride;
        const int *lst = (!ext && a.list_id >= 0) ? list_ptr(D, a.list_id, pd.s0) : nullptr;
        // ---- point metadata ------------------------------------------------
        if (lead && tl < PPW) {
            const int pt = tl;
            int job, v;
            bool valid;
            if (V <= ppw) {
                job = (int)(ltile * jpw) + pt / V;
                v = pt % V;
                valid = (pt < jpw * V) && job < count;
            } else {
                job = (int)(ltile / wpj);
                v = (int)(ltile % wpj) * ppw + pt;
                valid = pt < ppw && v < V;
            }
            if constexpr (FLAGS) {
                if (a.by_flag) {
                    valid = valid && D.flag[pd.s0 + job] == a.by_flag;
                    // the points of this tile, counted here (below: lanes < PPW)
                    const int n = (int)__popcll(__ballot(valid));
                    if (lane == 0) {
                        s_live[0] = n;
                        if (n) {
                            atomicAdd(&D.ctl[p].evals, (unsigned long long)n);
                            atomicAdd(&D.prof[FD ? 3 : CENTER], (unsigned long long)n);
                        }
                    }
                }
            }
            s_s[pt] = valid ? (ext ? job : (lst ? lst[job] : pd.s0 + job)) : -1;
            s_c[pt] = v / Vs;
            s_st[pt] = v % Vs;
            s_den[pt] = 1.0f;
        }
        __syncthreads();
        if constexpr (FLAGS)
            if (a.by_flag && s_live[0] == 0) {
                __syncthreads();
                continue;
            }
        // ---- generate the points (zero padded to DP), all waves -------------
        // rows are read in 16-byte chunks when the row stride and base allow it
        // (the library's own rows always do; a caller's array may not)
        const bool vrow = (xs & 3) == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
        // Smoothing probes come in antithetic pairs x + sigma z, x - sigma z
        // (centres 2i and 2i + 1 of a job).  When a job's probe count is even
        // the two points of a pair sit side by side in the tile, from an even
        // slot on, so one read of the sample row and one draw of z serve both
        // (the same values the per-point loop below computes for each).
        bool paired = false;
        if constexpr (CENTER == kProbe && !FD) paired = (Vc & 1) == 0;
        if (paired) {
            for (int e = threadIdx.x; e < (PPW / 2) * KS; e += blockDim.x) {
                const int pt = 2 * (e / KS), blk = e % KS, c0 = 4 * blk;
                const int s = s_s[pt];  // the same sample as slot pt + 1
                float xp[4] = {0.f, 0.f, 0.f, 0.f}, xm[4] = {0.f, 0.f, 0.f, 0.f};
                if (s >= 0 && c0 < d) {
                    const uint32_t pair = (uint32_t)(s_c[pt] >> 1);
                    float z[4];
                    box_muller4(philox((uint32_t)(s - pd.s0), kcyc, (kHLC << 24) | ((uint32_t)a.step << 16) | pair,
                                       (uint32_t)blk, pd.key0, pd.key1),
                                z);
                    float xr[4] = {0.f, 0.f, 0.f, 0.f};
                    if (vrow) {
                        const f32x4 w = *reinterpret_cast<const f32x4 *>(a.X + (size_t)s * xs + c0);
                        xr[0] = w[0]; xr[1] = w[1]; xr[2] = w[2]; xr[3] = w[3];
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (c0 + q < d) xr[q] = a.X[(size_t)s * xs + c0 + q];
                    }
                    const float sp = sigma, sm = -sigma;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (c0 + q < d) {
                            xp[q] = xr[q] + sp * z[q];
                            xm[q] = xr[q] + sm * z[q];
                        }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    s_pts[pt * LD + c0 + q] = xp[q];
                    s_pts[(pt + 1) * LD + c0 + q] = xm[q];
                }
            }
        }
        for (int e = paired ? PPW * KS : threadIdx.x; e < PPW * KS; e += blockDim.x) {
            const int pt = e / KS, blk = e % KS, c0 = 4 * blk;
            const int s = s_s[pt];
            float x[4] = {0.f, 0.f, 0.f, 0.f};
            float x0[4] = {0.f, 0.f, 0.f, 0.f}, g0[4] = {0.f, 0.f, 0.f, 0.f};
            float dp = 0.0f;
            if (s >= 0) {
                const int ci = s_c[pt];
                float z[4] = {0.f, 0.f, 0.f, 0.f};
                if constexpr (CENTER == kProbe) {
                    const uint32_t pair = (uint32_t)(ci >> 1);
                    uint4 o = philox((uint32_t)(s - pd.s0), kcyc,
                                     (kHLC << 24) | ((uint32_t)a.step << 16) | pair, (uint32_t)blk, pd.key0, pd.key1);
                    box_muller4(o, z);
                }
                float xr[4] = {0.f, 0.f, 0.f, 0.f}, gr[4] = {0.f, 0.f, 0.f, 0.f}, pr[4] = {0.f, 0.f, 0.f, 0.f};
                if (c0 < d) {
                    if (vrow) {
                        const f32x4 w = *reinterpret_cast<const f32x4 *>(a.X + (size_t)s * xs + c0);
                        xr[0] = w[0]; xr[1] = w[1]; xr[2] = w[2]; xr[3] = w[3];
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (c0 + q < d) xr[q] = a.X[(size_t)s * xs + c0 + q];
                    }
                    if constexpr (CENTER == kTrial) {
                        // the library's rows: stride a multiple of four floats
                        const f32x4 wg = *reinterpret_cast<const f32x4 *>(D.G + (size_t)s * D.DS + c0);
                        const f32x4 wp = *reinterpret_cast<const f32x4 *>(D.Pd + (size_t)s * D.DS + c0);
                        gr[0] = wg[0]; gr[1] = wg[1]; gr[2] = wg[2]; gr[3] = wg[3];
                        pr[0] = wp[0]; pr[1] = wp[1]; pr[2] = wp[2]; pr[3] = wp[3];
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = c0 + q;
                    if (c < d) {
                        float xv = xr[q];
                        if constexpr (CENTER == kTrial) {
                            const float t = ldexpf(1.0f, -(r0 + ci));
                            x0[q] = xv;
                            g0[q] = gr[q];
                            xv = fminf(fmaxf(xv + t * pr[q], pd.lo[c]), pd.hi[c]);
                            dp += g0[q] * (xv - x0[q]);
                        } else if constexpr (CENTER == kProbe) {
                            const float sgn = (ci & 1) ? -1.0f : 1.0f;
                            xv = xv + sigma * sgn * z[q];
                        }
                        x[q] = xv;
                    }
                }
                if constexpr (FD) {
                    const int st = s_st[pt];
                    const int cs = st >> 1;
                    if (cs >= c0 && cs < c0 + 4) {
                        const float xc = x[cs - c0];
                        const float h = pd.fd_h > 0.0f ? pd.fd_h : ldexpf(fmaxf(1.0f, fabsf(xc)), -8);
                        const float xp = xc + h, xm = xc - h;
                        x[cs - c0] = (st & 1) ? xm : xp;
                        s_den[pt] = xp - xm;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) s_pts[pt * LD + c0 + q] = x[q];
            if constexpr (TRIAL) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    s_x0[pt * LD + c0 + q] = x0[q];
                    s_g0[pt * LD + c0 + q] = g0[q];
                }
                s_dp[pt * KS + blk] = dp;
            }
        }
        __syncthreads();
        // Noisy problems: every value the method sees carries sigma_n z, z the
        // first normal of the NOISE stream at (sample, cycle, step << 16 |
        // sub); the gate value carries sigma_n times the mean of gate_reps
        // normals of the GATE stream.  The gradient stays noise-free.
        const bool noisy = !ext && a.nz_kind >= 0 && pd.noise_sigma > 0.0f;
        auto noise_of = [&](int pt) -> float {
            const uint32_t ls = (uint32_t)(s_s[pt] - pd.s0);
            if (a.nz_kind == 0) {
                uint32_t sub = a.nz_base;
                if constexpr (CENTER == kTrial) sub += (uint32_t)(r0 + s_c[pt]);
                if constexpr (CENTER == kProbe) sub |= (uint32_t)s_c[pt] << 7;
                if constexpr (FD) sub += (uint32_t)s_st[pt];
                float z[4];
                box_muller4(philox(ls, kcyc, (kNoise << 24) | ((uint32_t)a.step << 16) | sub, 0u, pd.key0, pd.key1), z);
                return pd.noise_sigma * z[0];
            }
            float zs = 0.0f;
            for (int b = 0; 4 * b < pd.gate_reps; ++b) {
                float z[4];
                box_muller4(philox(ls, kcyc, kGate << 24, (uint32_t)b, pd.key0, pd.key1), z);
                for (int q = 0; q < 4 && 4 * b + q < pd.gate_reps; ++q) zs += z[q];
            }
            return pd.noise_sigma * (zs / (float)pd.gate_reps);
        };
        if constexpr (CLOSED) {
            // ---- closed-form value (and gradient), two lanes per point ------
            const int pt = lane >> 1, c0 = lane & 1;
            const float *x = s_pts + pt * LD;
            float sa, sb;
            cf_partial(pd.family, d, x, c0, sa, sb);
            sa += __shfl_xor(sa, 1, kWave);
            sb += __shfl_xor(sb, 1, kWave);
            if (s_s[pt] >= 0) {
                if (c0 == 0) {
                    float f = cf_value(pd.family, d, sa, sb);
                    if (noisy) f += noise_of(pt);
                    s_f[pt] = f;
                }
                if constexpr (GRAD)
                    for (int c = c0; c < d; c += 2) s_g[pt * LD + c] = cf_grad(pd.family, d, x, c, sa, sb);
            }
            __syncthreads();
        } else if constexpr (ALU) {
            // ---- small mixtures: one lane per point on the VALU ----------------
            // A few coordinates give the matrix core too little to do: padded
            // to 16, a d = 2 component would cost its full 16-wide tile.  Here
            // each lane carries one point through the components; the tile's
            // problem is the same in every lane, so a component's record (P's
            // upper triangle, mu, log2 weight) is read with scalar loads and
            // enters each instruction as its scalar operand.
            const int W = alu_width(d);
            const int K = __builtin_amdgcn_readfirstlane(pd.K);
            const cfloat *tab = uniform_const(pd.Pfrag);
            const float nu = pd.nu, nupd = pd.nu_plus_d, inv_nu = 1.0f / nu;
            auto run = [&](auto wc) {
                constexpr int Wc = decltype(wc)::value, T = Wc * (Wc + 1) / 2, R = alu_record(Wc);
                const int pt = lane;
                float xr[Wc], ga[GRAD ? Wc : 1];
#pragma unroll
                for (int i = 0; i < Wc; ++i) {
                    xr[i] = s_pts[pt * LD + i];
                    if constexpr (GRAD) ga[i] = 0.0f;
                }
                float m = -INFINITY, sm = 0.0f;
                for (int k = 0; k < K; ++k) {
                    const cfloat *rec = tab + k * R;
                    float dl[Wc], u[Wc];
#pragma unroll
                    for (int i = 0; i < Wc; ++i) dl[i] = xr[i] - rec[T + i];
                    // u = P (x - mu) from the upper triangle, q = (x - mu) . u
                    float q = 0.0f;
#pragma unroll
                    for (int i = 0; i < Wc; ++i) {
                        float acc = 0.0f;
#pragma unroll
                        for (int j = 0; j < Wc; ++j) {
                            const int lo = i < j ? i : j, hi = i < j ? j : i;
                            acc = fmaf(rec[lo * Wc - lo * (lo - 1) / 2 + (hi - lo)], dl[j], acc);
                        }
                        u[i] = acc;
                        q = fmaf(dl[i], acc, q);
                    }
                    float l2, w = 1.0f;
                    if constexpr (FAM == 0) {
                        l2 = rec[T + Wc] - q * (0.5f * kLog2e);
                    } else {
                        l2 = rec[T + Wc] - (0.5f * nupd) * student_log2(q, inv_nu);
                        w = nupd * __builtin_amdgcn_rcpf(nu + q);
                    }
                    // the same online log-sum-exp as the tiles: the reference
                    // moves only when a term exceeds it by 2^kLseSlack, which
                    // few components do, so the rescale is a rare branch
                    const bool moved = l2 > m + kLseSlack;
                    if (__any(moved)) {
                        const float mnew = moved ? l2 : m;
                        const float sc = moved ? __builtin_amdgcn_exp2f(m - mnew) : 1.0f;
                        sm *= sc;
                        if constexpr (GRAD)
#pragma unroll
                            for (int i = 0; i < Wc; ++i) ga[i] *= sc;
                        m = mnew;
                    }
                    const float pk = __builtin_amdgcn_exp2f(l2 - m);
                    sm += pk;
                    if constexpr (GRAD) {
                        const float pw = pk * w;
#pragma unroll
                        for (int i = 0; i < Wc; ++i) ga[i] = fmaf(pw, u[i], ga[i]);
                    }
                }
                float f = (m + __log2f(sm)) * kLn2;
                if (noisy && s_s[pt] >= 0) f += noise_of(pt);
                s_f[pt] = f;
                if constexpr (GRAD) {
                    const float inv = -1.0f / sm;
#pragma unroll
                    for (int i = 0; i < Wc; ++i) s_g[pt * LD + i] = ga[i] * inv;
                }
            };
            if (W == 2) run(std::integral_constant<int, 2>{});
            else if (W == 4) run(std::integral_constant<int, 4>{});
            else run(std::integral_constant<int, 8>{});
            __syncthreads();
        } else {
            // ---- operand registers ---------------------------------------------
            float xB[NB][KS];
            // two-part problems: the point's own power of two, and the factors
            // of its quadratic form and gradient sums
            float cn[H16 ? NB : 1], kqn[H16 ? NB : 1], kgn[H16 ? NB : 1];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const float *row = s_pts + (wp + nb * 16 + n) * LD;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) xB[nb][ks] = row[lane_coord(ks, g)];
            }
            if constexpr (H16) {
                const gfloat *xs = as_global(pd.xs), *mu0 = as_global(pd.muB2) + g * KS;
                float far[NB] = {};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const float sc = xs[lane_coord(ks, g)], c0 = mu0[ks];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        xB[nb][ks] *= sc;
                        far[nb] = fmaxf(far[nb], fabsf(xB[nb][ks] - c0));
                    }
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    // a point within 2^14 of the first centre lies within 2^14 +
                    // 2^kTwoPartX of the others: in f16's range as it is
                    const float fm = rows4_max(far[nb]);
                    const int ex = fm > 16384.0f ? 140 - (int)(__float_as_uint(fm) >> 23) : 0;
                    cn[nb] = ldexpf(1.0f, ex);
                    kqn[nb] = ldexpf(pd.kq, -2 * ex);
                    kgn[nb] = ldexpf(pd.kq, -ex);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) xB[nb][ks] *= cn[nb];
                }
            }
            const int K = __builtin_amdgcn_readfirstlane(pd.K);
            const int wvu = __builtin_amdgcn_readfirstlane(wv);
            const int kb = SPLIT == 1 ? 0 : (wvu * K) / SPLIT, ke = SPLIT == 1 ? K : ((wvu + 1) * K) / SPLIT;
            const float m_start = lse_start(!DSPLIT || kb == 0);
            float mrun[NB], srun[NB];
            float gacc[NB][GRAD ? KS : 1];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                mrun[nb] = m_start;
                srun[nb] = 0.0f;
                if constexpr (GRAD)
#pragma unroll
                    for (int i = 0; i < KS; ++i) gacc[nb][i] = 0.0f;
            }
            // ---- stream the components -----------------------------------------
            // Two waves per SIMD: while one waits for a component's operands or
            // works through the log-sum-exp epilogue on the VALU, the other keeps
            // the matrix core busy; a wave raises its priority for the duration of
            // its MFMA block so the arbiter keeps the matrix core fed.  Operands
            // come through buffer loads, which only the vector-memory counter
            // tracks: flat loads would also count against the LDS counter, and
            // the cross-lane reductions of the epilogue would then wait for them.
            const float nu = pd.nu, nupd = pd.nu_plus_d, inv_nu = 1.0f / nu;
            typedef typename std::conditional<H16, TwoPartRegs<DP>, CompRegs<KS, MB>>::type Regs;
            Regs ra;
            // Buffer loads: a scalar resource per table and the component's
            // byte offset in a scalar register, each lane's fixed offset in a
            // vector register, so the loop advances one scalar per table
            // instead of per-lane 64-bit addresses.
            const int Kc = pd.K;
            const __amdgpu_buffer_rsrc_t rs_pf = table_rsrc(H16 ? pd.Pfrag2 : pd.Pfrag, (uint32_t)Kc * DP * DP * 4u);
            const __amdgpu_buffer_rsrc_t rs_mu = table_rsrc(H16 ? pd.muB2 : pd.muB, (uint32_t)Kc * DP * 4u);
            const __amdgpu_buffer_rsrc_t rs_lc = table_rsrc(pd.logc2, (uint32_t)Kc * 4u);
            const int mu_lane = g * KS * 4;
            // (SHARE) component k into half b of s_pts, by every thread; there
            // after the next arrive()
            [[maybe_unused]] auto fetch = [&](int k, int b) {
                typedef const void __attribute__((address_space(1))) * gptr;
                typedef void __attribute__((address_space(3))) * lptr;
                const float *src = pd.Pfrag2 + (size_t)k * DP * DP;
                float *dst = s_pts + b * kCompF;
#pragma unroll
                for (int i = 0; i < DP * DP / (4 * kShareWaves * kWave); ++i)
                    __builtin_amdgcn_global_load_lds((gptr)(src + 4 * (i * kShareWaves * kWave + threadIdx.x)),
                                                     (lptr)(dst + 4 * (i * kShareWaves + wv) * kWave), 16, 0, 0);
                if (threadIdx.x < DP / 4)
                    __builtin_amdgcn_global_load_lds((gptr)(pd.muB2 + (size_t)k * DP + 4 * threadIdx.x),
                                                     (lptr)(dst + DP * DP), 16, 0, 0);
            };
            // Direct loads write LDS outside of what a barrier waits for: each
            // wave waits for its own, then for the others.
            [[maybe_unused]] auto arrive = [&] {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
            };
            [[maybe_unused]] auto load_shared = [&](int b, Regs &r) {
                if constexpr (SHARE) {
                    const float *src = s_pts + b * kCompF;
#pragma unroll
                    for (int i = 0; i < 2 * r.S * MB; ++i) {
                        const int part = i % 2, blk = i / 2;
                        r.pa[part][blk / MB][blk % MB] = *reinterpret_cast<const f16x8 *>(
                            src + 4 * ((part * r.S * MB + blk) * kWave + lane));
                    }
#pragma unroll
                    for (int i = 0; i < KS; i += 4) {
                        const f32x4 v = *reinterpret_cast<const f32x4 *>(src + DP * DP + g * KS + i);
                        r.muB[i] = v[0]; r.muB[i + 1] = v[1]; r.muB[i + 2] = v[2]; r.muB[i + 3] = v[3];
                    }
                }
            };
            [[maybe_unused]] const int pf_lane = lane * MB * 4;
            float neg1 = -1.0f;
            if constexpr (H16) asm("" : "+s"(neg1));
            auto load = [&](int k, Regs &r) {
                const int pf_k = k * DP * DP * 4, mu_k = k * DP * 4;
                if constexpr (H16) {
#pragma unroll
                    for (int i = 0; i < 2 * r.S * MB; ++i) {
                        const int part = i % 2, blk = i / 2;  // (the parts of a block are used together)
                        const int off = (part * r.S * MB + blk) * kWave * 16;
                        r.pa[part][blk / MB][blk % MB] = __builtin_bit_cast(
                            f16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_pf, lane * 16 + off, pf_k, 0));
                    }
                } else {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) load_frag_buf<MB>(rs_pf, pf_lane + ks * kWave * MB * 4, pf_k, r.pa[ks]);
                }
#pragma unroll
                for (int i = 0; i < KS; i += 4) {
                    const f32x4 vb = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_mu, mu_lane + i * 4, mu_k, 0));
                    r.muB[i] = vb[0]; r.muB[i + 1] = vb[1]; r.muB[i + 2] = vb[2]; r.muB[i + 3] = vb[3];
                }
                r.lc2 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_lc, 0, k * 4, 0));
            };
            // k, as a value the compiler does not know to be k
            [[maybe_unused]] auto hidden = [](int k) {
                asm("" : "+s"(k));
                return k;
            };
            // contracts one component for the first NBA column blocks of the tile
            // log-sum-exp state of the lane's own block in the two-block path
            float m_own = m_start, s_own = 0.0f;
            auto own_to_blocks = [&](auto nba) {
                if constexpr (decltype(nba)::value == 2) {
                    rows_pair_split(m_own, mrun[0], mrun[1]);
                    rows_pair_split(s_own, srun[0], srun[1]);
                }
            };
            // (two-part problems) the lane's own block's factor of the quadratic form
            float kq_own = 1.0f;
            if constexpr (H16) kq_own = (g & 1) ? kqn[1] : kqn[0];
            // forms of points that lie within 4 2^-b standard deviations of a
            // centre (kq = 2^(-2 b - kTwoPartP)): where f16's smallest numbers begin
            // to show in their deltas
            [[maybe_unused]] const float q_near = H16 ? pd.kq * (float)(16 << kTwoPartP) : 0.0f;
            // (two parts) again: the fragments once more, for the rare use far from the
            // first (held, they would cost 32 registers)
            auto step = [&](const Regs &r, auto nba, auto four, auto &&again) {
                constexpr bool FOUR = decltype(four)::value;
                constexpr int NBA = decltype(nba)::value;
                f32x4 acc[NB][MB];
#pragma unroll
                for (int nb = 0; nb < NBA; ++nb)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                // delta = x - mu_k in B-operand order; with the rows of P
                // permuted at init, the accumulator of lane (n, g) holds u at
                // the same coordinates 4 ks + g, so delta also serves the
                // quadratic form below
                float bv[NB][KS];
                // (two parts) acc += P v for the blocks b0 .. b1 - 1; fill(s, v) gives
                // the deltas of K step s.  The small products go first, while the
                // accumulator is small: all of them where the second step holds
                // few coordinates (d <= kTwoPartLowD of 64; step by step those of
                // d = 36 were 1.03 times float32's error off), else, to save
                // registers, those of a step before its large one.  Which of
                // l_P h_d and h_P l_d comes first makes no difference to the
                // error; it does to the path that a long run takes (on which of
                // the highest maxima of the d = 64, K = 128 mixture 300 cycles
                // end hangs on rounding), and with this order that run passes its
                // recall test.
                [[maybe_unused]] auto contract = [&](const Regs &r, auto &&fill, auto b0, auto b1) {
                    if constexpr (H16) {
                        constexpr bool LATE = FOUR && Regs::S > 1;
                        f16x8 bh[LATE ? Regs::S : 1][NB], bl[NB];
                        // consecutive instructions go to different accumulators
                        auto product = [&](const f16x8(&pa)[MB], const f16x8(&b)[NB]) {
#pragma unroll
                            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                                for (int nb = b0.value; nb < b1.value; ++nb)
                                    acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa[mb], b[nb], acc[nb][mb], 0, 0, 0);
                        };
#pragma unroll
                        for (int s = 0; s < Regs::S; ++s) {
                            const int o = LATE ? s : 0;
                            float v[NB][8];
                            fill(s, v);
#pragma unroll
                            for (int nb = b0.value; nb < b1.value; ++nb) two_parts(v[nb], neg1, bh[o][nb], bl[nb]);
                            __builtin_amdgcn_s_setprio(1);
                            if constexpr (FOUR) product(r.pa[1][s], bl);
                            product(r.pa[0][s], bl);
                            product(r.pa[1][s], bh[o]);
                            if constexpr (!LATE) product(r.pa[0][s], bh[o]);
                            __builtin_amdgcn_s_setprio(0);
                        }
                        if constexpr (LATE) {
                            __builtin_amdgcn_s_setprio(1);
#pragma unroll
                            for (int s = 0; s < Regs::S; ++s) product(r.pa[0][s], bh[s]);
                            __builtin_amdgcn_s_setprio(0);
                        }
                    }
                };
                // (two parts) u again for the points of block nb that lie next to
                // the centre, from deltas scaled so that the largest fills f16's
                // range; the other points' come out as they were
                [[maybe_unused]] auto contract_near = [&](const Regs &r2, auto b, bool near) {
                    if constexpr (H16) {
                        constexpr int nb = decltype(b)::value;
                        float mx = 0.0f;
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) mx = fmaxf(mx, fabsf(bv[nb][ks]));
                        const int e = 140 - (int)(__float_as_uint(rows4_max(mx)) >> 23);
                        const int ex = near ? max(0, min(e, 120)) : 0;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                        contract(r2, [&](int s, float(&v)[NB][8]) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) v[nb][j] = ldexpf(bv[nb][8 * s + j], ex);
                        }, b, std::integral_constant<int, nb + 1>{});
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] *= ldexpf(1.0f, -ex);
                    }
                };
                if constexpr (H16) {
                    contract(r, [&](int s, float(&v)[NB][8]) {
#pragma unroll
                        for (int nb = 0; nb < NBA; ++nb)
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                v[nb][j] = bv[nb][8 * s + j] = fmaf(-r.muB[8 * s + j], cn[nb], xB[nb][8 * s + j]);
                    }, std::integral_constant<int, 0>{}, nba);
                } else {
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                    for (int nb = 0; nb < NBA; ++nb) {
                        bv[nb][ks] = xB[nb][ks] - r.muB[ks];
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
                            acc[nb][mb] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(r.pa[ks][mb], bv[nb][ks], acc[nb][mb], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_s_setprio(0);
                }
                if constexpr (NBA == 2) {
                    // Both blocks' quadratic forms reduced in one exchange;
                    // rows 0 and 2 then carry block 0's log-sum-exp state and
                    // rows 1 and 3 block 1's (the same arithmetic as the
                    // per-block path below, half the lanes' work each), and
                    // the gradient weights are exchanged back to every lane.
                    auto form = [&] {
                        float q0 = 0.0f, q1 = 0.0f;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr) {
                                q0 = fmaf(bv[0][4 * mb + rr], acc[0][mb][rr], q0);
                                q1 = fmaf(bv[1][4 * mb + rr], acc[1][mb][rr], q1);
                            }
                        return rows4_sum_pair(q0, q1);
                    };
                    float q = form();
                    if constexpr (H16) {
                        q *= kq_own;
                        if (__any(q < q_near)) {
                            float n0, n1;
                            rows_pair_split(q < q_near ? 1.0f : 0.0f, n0, n1);
                            Regs r2;
                            again(r2);
                            contract_near(r2, std::integral_constant<int, 0>{}, n0 != 0.0f);
                            contract_near(r2, std::integral_constant<int, 1>{}, n1 != 0.0f);
                            q = form() * kq_own;
                        }
                    }
                    float l2, w = 1.0f;
                    if constexpr (FAM == 0) {
                        l2 = r.lc2 - q * (0.5f * kLog2e);
                    } else {
                        l2 = r.lc2 - (0.5f * nupd) * student_log2(q, inv_nu);
                        w = nupd * __builtin_amdgcn_rcpf(nu + q);
                    }
                    const bool moved = l2 > m_own + kLseSlack;
                    // (few components move the reference, so its rescale is a
                    // rare branch)
                    if (__any(moved)) {
                        // sc is exactly 1 in the block that did not move
                        const float mnew = moved ? l2 : m_own;
                        const float sc = __builtin_amdgcn_exp2f(m_own - mnew);
                        s_own *= sc;
                        m_own = mnew;
                        if constexpr (GRAD) {
                            float sc0, sc1;
                            rows_pair_split(sc, sc0, sc1);
#pragma unroll
                            for (int i = 0; i < KS; ++i) {
                                gacc[0][i] *= sc0;
                                gacc[1][i] *= sc1;
                            }
                        }
                    }
                    const float pk = __builtin_amdgcn_exp2f(l2 - m_own);
                    s_own += pk;
                    if constexpr (GRAD) {
                        float pw0, pw1;
                        rows_pair_split(pk * w, pw0, pw1);
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr) {
                                gacc[0][mb * 4 + rr] = fmaf(pw0, acc[0][mb][rr], gacc[0][mb * 4 + rr]);
                                gacc[1][mb * 4 + rr] = fmaf(pw1, acc[1][mb][rr], gacc[1][mb * 4 + rr]);
                            }
                    }
                    return;
                }
#pragma unroll
                for (int nb = 0; nb < NBA; ++nb) {
                    auto form = [&] {
                        float q = 0.0f;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr) q = fmaf(bv[nb][4 * mb + rr], acc[nb][mb][rr], q);
                        return rows4_sum(q);
                    };
                    float q = form();
                    if constexpr (H16) {
                        q *= kqn[nb];
                        if (__any(q < q_near)) {
                            Regs r2;
                            again(r2);
                            contract_near(r2, std::integral_constant<int, 0>{}, q < q_near);  // (one block only)
                            q = form() * kqn[nb];
                        }
                    }
                    float l2, w = 1.0f;
                    if constexpr (FAM == 0) {
                        l2 = r.lc2 - q * (0.5f * kLog2e);
                    } else {
                        l2 = r.lc2 - (0.5f * nupd) * student_log2(q, inv_nu);
                        w = nupd * __builtin_amdgcn_rcpf(nu + q);
                    }
                    // the reference moves only when a term exceeds it by more
                    // than 2^kLseSlack: terms stay below 2^kLseSlack, and the
                    // gradient sums are rescaled far less often
                    const bool moved = l2 > mrun[nb] + kLseSlack;
                    if (__any(moved)) {
                        const float mnew = moved ? l2 : mrun[nb];
                        const float sc = __builtin_amdgcn_exp2f(mrun[nb] - mnew);
                        srun[nb] *= sc;
                        mrun[nb] = mnew;
                        if constexpr (GRAD)
#pragma unroll
                            for (int i = 0; i < KS; ++i) gacc[nb][i] *= sc;
                    }
                    const float pk = __builtin_amdgcn_exp2f(l2 - mrun[nb]);
                    srun[nb] += pk;
                    if constexpr (GRAD) {
                        const float pw = pk * w;
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr)
                                gacc[nb][mb * 4 + rr] = fmaf(pw, acc[nb][mb][rr], gacc[nb][mb * 4 + rr]);
                    }
                }
            };
            if constexpr (SHARE) {
                auto loop = [&](auto four) {
                    auto lc = [&](int k) {
                        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_lc, 0, k * 4, 0));
                    };
                    __syncthreads();  // the points are in registers
                    float lc_next = lc(0);
                    fetch(0, 0);
                    arrive();
                    for (int k = 0; k < K; ++k) {
                        ra.lc2 = lc_next;
                        const int kn = min(k + 1, K - 1);
                        lc_next = lc(kn);
                        fetch(kn, (k + 1) & 1);
                        load_shared(k & 1, ra);
                        step(ra, AllBlocks{}, four, [&](Regs &r2) { load_shared(hidden(k) & 1, r2); });
                        arrive();
                    }
                };
                if (d <= kTwoPartLowD) loop(std::true_type{});
                else loop(std::false_type{});
                own_to_blocks(AllBlocks{});
            } else if constexpr (DP < 64) {
                // small components: too little work per component to hide its load
                // latency behind the other wave, so the next one is loaded into a
                // second register set while this one is contracted (the set is
                // small at DP <= 32); the prefetch past the end reloads the last
                // component, which keeps the loop branch-free
                auto run = [&](auto nba) {
                    if (kb < ke) {
                        Regs rb;
                        load(kb, ra);
                        for (int k = kb; k < ke; k += 2) {
                            load(min(k + 1, ke - 1), rb);
                            step(ra, nba, std::true_type{}, [&](Regs &r2) { load(hidden(k), r2); });
                            if (k + 1 >= ke) break;
                            load(min(k + 2, ke - 1), ra);
                            step(rb, nba, std::true_type{}, [&](Regs &r2) { load(hidden(k + 1), r2); });
                        }
                    }
                    own_to_blocks(nba);
                };
                if constexpr (HALF) {
                    if (ppw < PPW) run(OneBlock{});
                    else run(AllBlocks{});
                } else if constexpr (HT) {
                    run(OneBlock{});
                } else {
                    run(AllBlocks{});
                }
            } else {
                auto loop = [&](auto nba, auto four) {
                    for (int k = kb; k < ke; ++k) {
                        load(k, ra);
                        step(ra, nba, four, [&](Regs &r2) { load(hidden(k), r2); });
                    }
                };
                auto run = [&](auto nba) {
                    if (H16 && d <= kTwoPartLowD) loop(nba, std::integral_constant<bool, H16>{});
                    else loop(nba, std::false_type{});
                    own_to_blocks(nba);
                };
                if constexpr (HALF) {
                    if (ppw < PPW) run(OneBlock{});
                    else run(AllBlocks{});
                } else if constexpr (HT) {
                    run(OneBlock{});
                } else {
                    run(AllBlocks{});
                }
            }
            if constexpr (DSPLIT) {
                // merge: m the largest reference, the sums scaled by 2^(m_v - m)
                // and added in wave order; each wave takes its share of the
                // coordinates.  A part without components, or with none whose
                // term counts, has its first reference and sum 0; one that
                // met a NaN has sum NaN.
                constexpr int NBM = HT ? 1 : NB;
#pragma unroll
                for (int nb = 0; nb < NBM; ++nb) {
                    s_pm[wv][nb][lane] = mrun[nb];
                    s_ps[wv][nb][lane] = srun[nb];
                    if constexpr (GRAD)
#pragma unroll
                        for (int i = 0; i < KS; ++i) s_pg[(wv * NBM + nb) * KS + i][lane] = gacc[nb][i];
                }
                __syncthreads();
#pragma unroll
                for (int nb = 0; nb < NBM; ++nb) {
                    float m = -INFINITY, sm = 0.0f, av[SPLIT];
#pragma unroll
                    for (int v = 0; v < SPLIT; ++v) m = fmaxf(m, s_pm[v][nb][lane]);
#pragma unroll
                    for (int v = 0; v < SPLIT; ++v) {
                        const float mv = s_pm[v][nb][lane], sv = s_ps[v][nb][lane];
                        av[v] = (mv == -INFINITY && sv == 0.0f) ? 0.0f : __builtin_amdgcn_exp2f(mv - m);
                        sm = fmaf(sv, av[v], sm);
                    }
                    const int pt = nb * 16 + n;
                    if (wv == 0 && g == 0) s_f[pt] = (m + __log2f(sm)) * kLn2;
                    if constexpr (GRAD) {
                        const float inv = -1.0f / sm;
                        for (int i = wv; i < KS; i += SPLIT) {
                            const int c = lane_coord(i, g);
                            float gv = 0.0f;
#pragma unroll
                            for (int v = 0; v < SPLIT; ++v) gv = fmaf(s_pg[(v * NBM + nb) * KS + i][lane], av[v], gv);
                            gv *= inv;
                            if constexpr (H16) gv *= as_global(pd.xs)[c] * kgn[nb];
                            s_g[pt * LD + c] = gv;
                        }
                    }
                }
            } else if constexpr (SPLIT > 1) {
                // merge: m = max(m0, m_v), s = s0 2^(m0-m) + s_v 2^(m_v-m), the
                // gradient sums alike, for v = 1, 2, ... in order
                if (!lead) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        s_pm[wv - 1][nb][lane] = mrun[nb];
                        s_ps[wv - 1][nb][lane] = srun[nb];
                        if constexpr (GRAD)
#pragma unroll
                            for (int i = 0; i < KS; ++i) s_pg[((wv - 1) * NB + nb) * KS + i][lane] = gacc[nb][i];
                    }
                }
                __syncthreads();
                if (lead) {
                    for (int v = 0; v < SPLIT - 1; ++v) {
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            const float mv = s_pm[v][nb][lane];
                            if (!(mv > -INFINITY)) continue;  // no components in that part
                            const float mn = fmaxf(mrun[nb], mv);
                            const float a0 = __builtin_amdgcn_exp2f(mrun[nb] - mn);
                            const float a1 = __builtin_amdgcn_exp2f(mv - mn);
                            srun[nb] = fmaf(srun[nb], a0, s_ps[v][nb][lane] * a1);
                            if constexpr (GRAD)
#pragma unroll
                                for (int i = 0; i < KS; ++i)
                                    gacc[nb][i] = fmaf(gacc[nb][i], a0, s_pg[(v * NB + nb) * KS + i][lane] * a1);
                            mrun[nb] = mn;
                        }
                    }
                }
            }
            // ---- results to LDS --------------------------------------------
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if (DSPLIT || !lead || ((HALF || HT) && nb * 16 >= ppw)) break;
                const int pt = wp + nb * 16 + n;
                float f = (mrun[nb] + __log2f(srun[nb])) * kLn2;
                if (noisy && g == 0 && s_s[pt] >= 0) f += noise_of(pt);
                if (g == 0) s_f[pt] = f;
                if constexpr (GRAD) {
                    const float inv = -1.0f / srun[nb];
#pragma unroll
                    for (int i = 0; i < KS; ++i) {
                        const int c = lane_coord(i, g);
                        float gv = gacc[nb][i] * inv;
                        if constexpr (H16) gv *= as_global(pd.xs)[c] * kgn[nb];
                        s_g[pt * LD + c] = gv;
                    }
                }
            }
            __syncthreads();
        }
        // ---- epilogues -----------------------------------------------------
        const int os = a.out_stride;
        if constexpr (CENTER == kDirect && !FD) {
            if (lead && tl < PPW && s_s[tl] >= 0 && a.F_out) a.F_out[s_s[tl]] = s_f[tl];
            if constexpr (GRAD) {
                if (a.G_out)
                    for (int e = threadIdx.x; e < PPW * d; e += blockDim.x) {
                        const int pt = e / d, c = e % d, s = s_s[pt];
                        if (s >= 0) a.G_out[(size_t)s * os + c] = s_g[pt * LD + c];
                    }
            }
        } else if constexpr (FD) {
            if (lead && lane < PPW) {
                const int pt = lane, s = s_s[pt], st = s_st[pt];
                if (s >= 0 && (st & 1) == 0) {
                    const float gv = (s_f[pt] - s_f[pt + 1]) / s_den[pt];
                    const int c = st >> 1;
                    if constexpr (CENTER == kDirect) a.G_out[(size_t)s * os + c] = gv;
                    else D.Gp[((size_t)s * D.Mmax + s_c[pt]) * D.DS + c] = gv;
                }
            }
        } else if constexpr (CENTER == kProbe) {
            // mean over the job's probes, summed in probe order
            const float invM = 1.0f / (float)Vc;
            for (int e = lead ? tl : jpw * d; e < jpw * d; e += kTl) {
                const int j = e / d, c = e % d, p0 = j * Vc, s = s_s[p0];
                if (s >= 0) {
                    float acc = 0.0f;
                    for (int mm = 0; mm < Vc; ++mm) acc += s_g[(p0 + mm) * LD + c];
                    D.Gh[(size_t)s * D.DS + c] = acc * invM;
                }
            }
        } else if constexpr (CENTER == kTrial) {
            // Armijo margins f_tr - f - c1 g.(x_tr - x), two lanes per point
            const int DS = D.DS;
            if (lead) {
                for (int pt0 = 0; pt0 < PPW; pt0 += kWave / 2) {
                    const int pt = pt0 + (lane >> 1), h = lane & 1, s = s_s[pt];
                    float dot = 0.0f;
                    if (s >= 0)
                        for (int b = h; b < KS; b += 2) dot += s_dp[pt * KS + b];
                    dot += __shfl_xor(dot, 1, kWave);
                    // (relaxed by twice the noise level for noisy objectives: the
                    // noise-aware Armijo test of Berahas, Byrd and Nocedal 2019)
                    if (h == 0)
                        s_pass[pt] =
                            (s >= 0) && (s_f[pt] - D.F[s] - pd.ls_c1 * dot + 2.0f * pd.noise_sigma >= 0.0f);
                }
            }
            __syncthreads();
            if (lead && lane < jpw) {
                int r = -1;
                const int p0 = lane * Vc;
                if (s_s[p0] >= 0)
                    for (int i = 0; i < Vc; ++i)
                        if (s_pass[p0 + i]) { r = i; break; }
                s_acc[lane] = r;
            }
            __syncthreads();
            for (int e = threadIdx.x; e < jpw * d; e += blockDim.x) {
                const int j = e / d, c = e % d, p0 = j * Vc, s = s_s[p0];
                if (s >= 0 && s_acc[j] >= 0) {
                    const int pa = p0 + s_acc[j];
                    const size_t o = (size_t)s * DS + c;
                    D.Xprev[o] = s_x0[p0 * LD + c];
                    D.X[o] = s_pts[pa * LD + c];
                    D.Gprev[o] = s_g0[p0 * LD + c];
                    if constexpr (GRAD) D.G[o] = s_g[pa * LD + c];
                }
            }
            // (a cycle's evaluation count is that of two stages; a profile's
            // points are those computed)
            if constexpr (FLAGS) {
                if (lead && a.trial_need > 0 && Vc > a.trial_need) {
                    const bool early = lane < jpw && s_s[lane * Vc] >= 0 && s_acc[lane] >= 0 && s_acc[lane] < a.trial_need;
                    const int n = (int)__popcll(__ballot(early));
                    if (lane == 0 && n) {
                        const unsigned long long not_needed = (unsigned long long)n * (Vc - a.trial_need);
                        atomicAdd(&D.ctl[p].evals, 0ull - not_needed);
                    }
                }
            }
            // verdict per list position for the compaction that follows:
            // 1 try the remaining trials, 2 accepted (the finite-difference
            // gradient is still due), 3 the search failed, 0 nothing to do
            if (lead && lane < jpw) {
                const int p0 = lane * Vc, sl = s_s[p0];
                if (sl >= 0) {
                    const int r = s_acc[lane];
                    uint8_t verdict;
                    if (r >= 0) {
                        D.F[sl] = s_f[p0 + r];
                        D.status[sl] = (uint8_t)(kStAccept | (r0 + r));
                        verdict = GRAD ? 0 : 2;
                    } else if (a.trial_next >= 0 && r0 + Vc < pd.ls_max) {
                        verdict = 1;
                    } else {
                        D.status[sl] = kStFail;
                        verdict = 3;
                    }
                    D.flag[pd.s0 + (int)(ltile * jpw) + lane] = verdict;
                    // (the compaction counts the failed searches otherwise)
                    if (a.by_flag && verdict == 3) atomicAdd(&D.ctl[p].ls_fail, 1);
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Central differences of the closed forms, one wave per centre (a sample, or a
// smoothing probe of one) and one lane per stencil point.  A stencil point
// differs from its centre in one coordinate, so the factors of its other d - 1
// terms are the centre's: the wave takes them once, one lane per coordinate,
// and each lane adds its point's terms from LDS, its own coordinate's in their
// place, in the order the tiles add them (even coordinates, odd coordinates,
// then the two): every value has the bits of a full evaluation of that point.
//
// What bounds it: the vector unit.  As tiles of 32 points, each with all its
// terms, the d = 64 Michalewicz function spent 45 instructions a term and as
// much again on the tile's own bookkeeping: 8192 gradients (and values) took
// 150 us, with the factors shared within those tiles 103 us, here 26 us.
// ---------------------------------------------------------------------------
constexpr int kCfdWaves = 4;  // waves (centres at a time) per workgroup
template <int CENTER>
__global__ __launch_bounds__(kWave *kCfdWaves) void closed_fd_kernel(EvalArgs a) {
    __shared__ unit_t s_pref[kMaxClass + 1];
    __shared__ f32x4 s_row[kCfdWaves][kWave];  // per coordinate: centre, its two factors
    const Dev &D = a.D;
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    const bool ext = a.ext_n >= 0;
    if (wv == 0) {
        unit_t carry = 0;
        if (lane == 0) s_pref[0] = 0;
        for (int j0 = 0; j0 < a.n_cls; j0 += kWave) {
            const int j = j0 + lane;
            unit_t t = 0;
            if (j < a.n_cls) {
                const int p = a.cls[j];
                const ProblemDesc &pd = D.pd[p];
                t = units_of(job_count(a, p, pd), centres(a, pd));
                if (blockIdx.x == 0 && !ext && t > 0 && !a.by_flag) {
                    const unsigned long long nv = (unsigned long long)t * (unsigned long long)(2 * pd.d);
                    atomicAdd(&D.ctl[p].evals, nv);
                    atomicAdd(&D.prof[CHISAO_PROF_EVAL_FD], nv);
                }
            }
            const unit_t inc = wave_scan(t);
            if (j < a.n_cls) s_pref[j + 1] = carry + inc;
            carry += __shfl(inc, kWave - 1, kWave);
        }
    }
    __syncthreads();
    const unit_t total = s_pref[a.n_cls];
    // (no barrier inside the loop: a wave's rows of s_row are its own)
    for (unit_t u = first_unit(blockIdx.x, kCfdWaves, wv); u < total; u = next_unit(u, gridDim.x, kCfdWaves)) {
        int lo_j = 0, hi_j = a.n_cls - 1;
        while (lo_j < hi_j) {
            const int mid = (lo_j + hi_j + 1) >> 1;
            if (s_pref[mid] <= u) lo_j = mid;
            else hi_j = mid - 1;
        }
        const int p = __builtin_amdgcn_readfirstlane(a.cls[lo_j]);
        const ProblemDesc &pd = D.pd[p];
        const int d = pd.d, fam = pd.family;
        // (one centre a job unless the jobs' centres are probes)
        const unit_t v = u - s_pref[lo_j];
        const int Vc = CENTER == kProbe ? centres(a, pd) : 1;
        const int job = (int)(v / Vc), ci = (int)(v % Vc);
        const int s = ext ? job : (a.list_id >= 0 ? list_ptr(D, a.list_id, pd.s0)[job] : pd.s0 + job);
        const uint32_t kcyc = (uint32_t)D.ctl[p].k + 1u;
        if (a.by_flag) {
            if (D.flag[pd.s0 + job] != a.by_flag) continue;
            if (lane == 0) {
                atomicAdd(&D.ctl[p].evals, (unsigned long long)(2 * d));
                atomicAdd(&D.prof[CHISAO_PROF_EVAL_FD], (unsigned long long)(2 * d));
            }
        }
        // the centre, one lane per coordinate
        float xc = lane < d ? a.X[(size_t)s * a.x_stride + lane] : 0.0f;
        if constexpr (CENTER == kProbe) {
            float z[4];
            box_muller4(philox((uint32_t)(s - pd.s0), kcyc, (kHLC << 24) | ((uint32_t)a.step << 16) | (uint32_t)(ci >> 1),
                               (uint32_t)(lane >> 2), pd.key0, pd.key1),
                        z);
            const float zv = lane & 2 ? (lane & 1 ? z[3] : z[2]) : (lane & 1 ? z[1] : z[0]);
            if (lane < d) xc = xc + D.ctl[p].sigma * ((ci & 1) ? -1.0f : 1.0f) * zv;
        }
        float t1 = 0.0f, t2 = 0.0f;
        cf_dispatch(fam, [&](auto fc) { cf_factors(fc.value, lane, xc, t1, t2); });
        s_row[wv][lane] = f32x4{xc, t1, t2, 0.0f};
        __builtin_amdgcn_wave_barrier();
        const float h = pd.fd_h > 0.0f ? pd.fd_h : ldexpf(fmaxf(1.0f, fabsf(xc)), -8);
        const float up = xc + h, dn = xc - h;
        for (int st0 = 0; st0 < 2 * d; st0 += kWave) {
            const int st = st0 + lane, cs = min(st >> 1, d - 1);
            const float xs_up = __shfl(up, cs, kWave), xs_dn = __shfl(dn, cs, kWave);
            const float own = (st & 1) ? xs_dn : xs_up, den = xs_up - xs_dn;
            float sa = 0.0f, sb = 0.0f;
            if (fam == CHISAO_BUKIN6) {
                sa = cf_bukin(cs == 0 ? own : s_row[wv][0][0], cs == 1 ? own : s_row[wv][1][0]);
            } else {
                cf_dispatch(fam, [&](auto fc) {
                    float o1, o2, oa = 0.0f, ob = 0.0f, prev = 0.0f;
                    cf_factors(fc.value, cs, own, o1, o2);
                    auto add = [&](int c, float &ra, float &rb) {
                        const f32x4 r = s_row[wv][c];
                        const bool mine = c == cs;
                        const float v = mine ? own : r[0];
                        cf_add(fc.value, c, v, prev, mine ? o1 : r[1], mine ? o2 : r[2], ra, rb);
                        prev = v;
                    };
                    int c = 0;
#pragma unroll 4
                    for (; c + 1 < d; c += 2) {
                        add(c, sa, sb);
                        add(c + 1, oa, ob);
                    }
                    if (c < d) add(c, sa, sb);
                    sa += oa;
                    sb += ob;
                });
            }
            float f = cf_value(fam, d, sa, sb);
            if (!ext && a.nz_kind >= 0 && pd.noise_sigma > 0.0f) {
                uint32_t sub = a.nz_base;
                if constexpr (CENTER == kProbe) sub |= (uint32_t)ci << 7;
                sub += (uint32_t)st;
                float z[4];
                box_muller4(philox((uint32_t)(s - pd.s0), kcyc, (kNoise << 24) | ((uint32_t)a.step << 16) | sub, 0u,
                                   pd.key0, pd.key1),
                            z);
                f += pd.noise_sigma * z[0];
            }
            const float f_dn = __shfl_xor(f, 1, kWave);
            if (st < 2 * d && !(st & 1)) {
                const float gv = (f - f_dn) / den;
                if constexpr (CENTER == kDirect) a.G_out[(size_t)s * a.out_stride + cs] = gv;
                else D.Gp[((size_t)s * D.Mmax + ci) * D.DS + cs] = gv;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------------------
// Values and gradients of a small mixture (d <= 8) on caller memory: one point
// per lane as in the tiles, without their lists, problems and staging.  The
// component records go through LDS, kAluChunk at a time, and are read as
// broadcasts (through scalar loads, which cannot be kept in flight, a wave
// alone on its SIMD took 810 cycles a component of width 8, so 680).
// SPLIT > 1: the waves of a workgroup share 64 points, each taking every
// SPLIT-th component, and merge their states through LDS.
//
// What bounds it: with waves enough the vector unit, about 100 instructions a
// component of width 8 at 4 cycles each (two waves' instructions pair up only
// where their registers allow it; a call of 300000 points, K = 40: 45 us as
// tiles, 36 here); with few points one pass over the components, which the split
// shortens (16384 points, K = 40: 19.5 us as tiles, 16 unsplit, 7 split).  Two
// points per lane were slower at every size (300000 points: 50 us).
// ---------------------------------------------------------------------------
constexpr int kAluBlock = 256, kAluChunk = 64;
template <int FAM, bool GRAD, int W, int SPLIT>
__global__ __launch_bounds__(kAluBlock) void alu_direct_kernel(EvalArgs a) {
    constexpr int T = W * (W + 1) / 2, R = alu_record(W), kWaves = kAluBlock / kWave;
    static_assert(SPLIT == 1 || SPLIT == kWaves, "all waves of a workgroup share its points, or none");
    __shared__ f32x4 s_rec[kAluChunk * (R / 4)];
    const int lane = threadIdx.x % kWave, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const ProblemDesc &pd = a.D.pd[a.cls[0]];
    const int d = pd.d, K = __builtin_amdgcn_readfirstlane(pd.K);
    const float nu = pd.nu, nupd = pd.nu_plus_d, inv_nu = 1.0f / nu;
    const uint32_t i = (SPLIT > 1 ? blockIdx.x : blockIdx.x * kWaves + wv) * kWave + lane;
    const bool in = i < (uint32_t)a.ext_n;
    float xr[W], ga[GRAD ? W : 1], m = lse_start(SPLIT == 1 || wv == 0), sm = 0.0f;
#pragma unroll
    for (int c = 0; c < W; ++c) {
        xr[c] = (in && c < d) ? as_global(a.X)[(size_t)i * d + c] : 0.0f;
        if constexpr (GRAD) ga[c] = 0.0f;
    }
    for (int k0 = 0; k0 < K; k0 += kAluChunk) {
        const int n = min(kAluChunk, K - k0);
        if (k0) __syncthreads();
        for (int e = threadIdx.x; e < n * (R / 4); e += kAluBlock)
            s_rec[e] = reinterpret_cast<const gf32x4 *>(as_global(pd.Pfrag) + (size_t)k0 * R)[e];
        __syncthreads();
        for (int k = SPLIT == 1 ? 0 : wv; k < n; k += SPLIT) {
            float rec[R], dl[W], u[W], q = 0.0f;
#pragma unroll
            for (int e = 0; e < R / 4; ++e) {
                const f32x4 v = s_rec[k * (R / 4) + e];
                rec[4 * e] = v[0]; rec[4 * e + 1] = v[1]; rec[4 * e + 2] = v[2]; rec[4 * e + 3] = v[3];
            }
#pragma unroll
            for (int c = 0; c < W; ++c) dl[c] = xr[c] - rec[T + c];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                float acc = 0.0f;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    const int lo = c < j ? c : j, hi = c < j ? j : c;
                    acc = fmaf(rec[lo * W - lo * (lo - 1) / 2 + (hi - lo)], dl[j], acc);
                }
                u[c] = acc;
                q = fmaf(dl[c], acc, q);
            }
            float l2, w = 1.0f;
            if constexpr (FAM == 0) {
                l2 = rec[T + W] - q * (0.5f * kLog2e);
            } else {
                l2 = rec[T + W] - (0.5f * nupd) * student_log2(q, inv_nu);
                w = nupd * __builtin_amdgcn_rcpf(nu + q);
            }
            const bool moved = l2 > m + kLseSlack;
            if (__any(moved)) {
                const float mnew = moved ? l2 : m;
                const float sc = moved ? __builtin_amdgcn_exp2f(m - mnew) : 1.0f;
                sm *= sc;
                if constexpr (GRAD)
#pragma unroll
                    for (int c = 0; c < W; ++c) ga[c] *= sc;
                m = mnew;
            }
            const float pk = __builtin_amdgcn_exp2f(l2 - m);
            sm += pk;
            if constexpr (GRAD) {
                const float pw = pk * w;
#pragma unroll
                for (int c = 0; c < W; ++c) ga[c] = fmaf(pw, u[c], ga[c]);
            }
        }
    }
    if constexpr (SPLIT > 1) {
        // merged as split tiles are: scaled to the largest reference, added in
        // wave order
        __shared__ float s_m[SPLIT][kWave], s_s[SPLIT][kWave], s_g[GRAD ? SPLIT * W : 1][kWave];
        s_m[wv][lane] = m;
        s_s[wv][lane] = sm;
        if constexpr (GRAD)
#pragma unroll
            for (int c = 0; c < W; ++c) s_g[wv * W + c][lane] = ga[c];
        __syncthreads();
        if (wv != 0) return;
        m = -INFINITY;
        sm = 0.0f;
        float av[SPLIT];
#pragma unroll
        for (int v = 0; v < SPLIT; ++v) m = fmaxf(m, s_m[v][lane]);
#pragma unroll
        for (int v = 0; v < SPLIT; ++v) {
            const float mv = s_m[v][lane], sv = s_s[v][lane];
            av[v] = (mv == -INFINITY && sv == 0.0f) ? 0.0f : __builtin_amdgcn_exp2f(mv - m);
            sm = fmaf(sv, av[v], sm);
        }
        if constexpr (GRAD)
#pragma unroll
            for (int c = 0; c < W; ++c) {
                float g = 0.0f;
#pragma unroll
                for (int v = 0; v < SPLIT; ++v) g = fmaf(s_g[v * W + c][lane], av[v], g);
                ga[c] = g;
            }
    }
    if (!in) return;
    if (a.F_out) a.F_out[i] = (m + __log2f(sm)) * kLn2;
    if constexpr (GRAD) {
        const float inv = -1.0f / sm;
#pragma unroll
        for (int c = 0; c < W; ++c)
            if (c < d) a.G_out[(size_t)i * d + c] = ga[c] * inv;
    }
}

// Shared points while that shortens the pass: with 32 components or more at any
// size (its many small workgroups also fill the last round more evenly: 300000
// points of width 8, K = 128: 112 us against 114), with 8 or more up to 65536
// points (K = 16: 8.7 against 9.8 us there, 13.3 against 12.6 at 131072).
template <int FAM, bool GRAD, int W>
static hipError_t alu_direct_width(const EvalArgs &a, int K, hipStream_t st) {
    const long groups = ((long)a.ext_n + kWave - 1) / kWave;
    constexpr int kWaves = kAluBlock / kWave;
    const dim3 b(kAluBlock), each((unsigned)((groups + kWaves - 1) / kWaves)), shared((unsigned)groups);
    if (K >= 32 || (K >= 8 && groups <= 1024))
        hipLaunchKernelGGL((alu_direct_kernel<FAM, GRAD, W, kWaves>), shared, b, 0, st, a);
    else
        hipLaunchKernelGGL((alu_direct_kernel<FAM, GRAD, W, 1>), each, b, 0, st, a);
    return hipGetLastError();
}

// fn for each launch's rows of a call on caller memory
template <class F>
static hipError_t for_launch_rows(EvalArgs a, int d, F &&fn) {
    for (int left = a.ext_n; left > 0;) {
        a.ext_n = launch_rows(left);
        const hipError_t e = fn(a);
        if (e != hipSuccess) return e;
        left -= a.ext_n;
        a.X += (size_t)a.ext_n * d;
        if (a.F_out) a.F_out += a.ext_n;
        if (a.G_out) a.G_out += (size_t)a.ext_n * d;
    }
    return hipSuccess;
}

static hipError_t alu_direct_rows(const EvalArgs &a, int d, int family, int K, bool grad, hipStream_t st) {
#define CHISAO_ALU(F, G)                                                  \
    switch (alu_width(d)) {                                               \
        case 2: return alu_direct_width<F, G, 2>(a, K, st);               \
        case 4: return alu_direct_width<F, G, 4>(a, K, st);               \
        default: return alu_direct_width<F, G, 8>(a, K, st);              \
    }
    if (family == 0) {
        if (grad) CHISAO_ALU(0, true) else CHISAO_ALU(0, false)
    } else {
        if (grad) CHISAO_ALU(1, true) else CHISAO_ALU(1, false)
    }
#undef CHISAO_ALU
}

hipError_t launch_alu_direct(const EvalArgs &a, int d, int family, int K, bool grad, hipStream_t st) {
    return for_launch_rows(a, d, [&](const EvalArgs &r) { return alu_direct_rows(r, d, family, K, grad, st); });
}

// ---------------------------------------------------------------------------
// Central differences of a mixture on caller memory.  A stencil point differs
// from its centre in one coordinate, so with u = P delta and q = delta . u of
// the centre its quadratic form is q + h (2 u_j + h P_jj), h the realised step:
// one contraction a component and two multiply-adds, one exp2 and a sum a
// stencil point, instead of a contraction each.  Every stencil point keeps a
// log-sum-exp state of its own; the difference is taken between the states,
// (m+ - m-) + (log2 s+ - log2 s-), where a common rounding of q is in both.
// Contraction in float32: it is the smaller part.
//
// A step that leads from far away to next to a component's centre leaves a
// difference of large numbers in that formula, off by a rounding of the
// centre's q.  A stencil point whose form is less than half of a centre's that
// is more than kFdTrust (long_step) is therefore contracted itself, from its
// own delta.  That takes a step of more than (1 - 1/sqrt 2) sqrt(q), at least
// 1.2 standard deviations of the component, so ordinary steps never do it, and
// a wave in which every one does costs what evaluating its points costs.
//
// What bounds it: the vector unit, about 8 instructions a stencil point and
// component, one of them an exponential.  16384 gradients of a d = 16, K = 32
// mixture (and the values) took 109 us as 33 evaluations, 24 here; the relative
// error against float64 falls by a third (d = 2 to 31: 0.4e-6 to 4e-6).
// (Populations evaluate every stencil point as it is: their differences carry
// noise per point, and their paths the bits of the plain evaluation.)
// ---------------------------------------------------------------------------
template <int NS>
struct LseStates {
    float m[NS], s[NS];
    __device__ __forceinline__ void clear(bool at_component_0) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            m[i] = lse_start(at_component_0);
            s[i] = 0.0f;
        }
    }
    // adds 2^t[i] to state i (the reference moves as in the tiles)
    __device__ __forceinline__ void add(const float (&t)[NS]) {
        float over = -INFINITY;
#pragma unroll
        for (int i = 0; i < NS; ++i) over = fmaxf(over, t[i] - m[i]);
        if (__any(over > kLseSlack))
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const bool moved = t[i] - m[i] > kLseSlack;
                s[i] *= moved ? __builtin_amdgcn_exp2f(m[i] - t[i]) : 1.0f;
                m[i] = moved ? t[i] : m[i];
            }
#pragma unroll
        for (int i = 0; i < NS; ++i) s[i] += __builtin_amdgcn_exp2f(t[i] - m[i]);
    }
    // the states of a workgroup's four waves into the first wave's: 0 + 2 and
    // 1 + 3, then those two.  Every wave calls it.
    __device__ __forceinline__ void merge(int wv, int lane) {
        __shared__ float s_m[2][NS][kWave], s_s[2][NS][kWave];
#pragma unroll
        for (int half = 2; half > 0; half /= 2) {
            if (half < 2) __syncthreads();
            if (wv >= half && wv < 2 * half)
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    s_m[wv - half][i][lane] = m[i];
                    s_s[wv - half][i][lane] = s[i];
                }
            __syncthreads();
            if (wv < half)
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    const float mv = s_m[wv][i][lane], sv = s_s[wv][i][lane], mx = fmaxf(m[i], mv);
                    // (a wave without components, or with none that counts)
                    const float a = s[i] == 0.0f ? 0.0f : s[i] * __builtin_amdgcn_exp2f(m[i] - mx);
                    const float b = sv == 0.0f ? 0.0f : sv * __builtin_amdgcn_exp2f(mv - mx);
                    s[i] = a + b;
                    m[i] = mx;
                }
        }
    }
    // log2 of state i's sum over state j's
    __device__ __forceinline__ float log2_ratio(int i, int j) const {
        return (m[i] - m[j]) + (__log2f(s[i]) - __log2f(s[j]));
    }
};

__device__ __forceinline__ float fd_half_step(float fd_h, float x) {
    return fd_h > 0.0f ? fd_h : ldexpf(fmaxf(1.0f, fabsf(x)), -8);
}

// log2 density of a component from its quadratic form
template <int FAM>
__device__ __forceinline__ float component_log2(float lc2, float q, float nupd, float inv_nu) {
    return FAM == 0 ? lc2 - q * (0.5f * kLog2e) : lc2 - (0.5f * nupd) * student_log2(q, inv_nu);
}

// Centres whose form is below it are off by roundings of 16 at most, as a value
// is by its other terms; a Student-t density is log1p(q / nu), so there the
// form counts in units of nu too.
constexpr float kFdTrust = 16.0f;
template <int FAM>
__device__ __forceinline__ float fd_trust(float nu) {
    return FAM == 0 ? kFdTrust : fminf(kFdTrust, 4.0f * nu);
}
// whether a stencil point's form t is not to be had from its centre's q (an
// overflown q says nothing of t; a NaN stays one either way)
__device__ __forceinline__ bool long_step(float t, float q, float trust) {
    return q > trust && !(t >= 0.5f * q && q < INFINITY);
}

constexpr int kFdWaves = 4;

// d > 8: 16 points a tile, the contraction and the lanes' coordinates as in
// eval_kernel; a lane holds the states of its KS coordinates' stencils.
// SPLIT: the four waves of a workgroup share a tile's components.
template <int DP, int FAM, bool SPLIT>
__global__ __launch_bounds__(kWave * kFdWaves) void mixture_fd_kernel(EvalArgs a) {
    constexpr int KS = DP / 4, MB = DP / 16;
    const int lane = threadIdx.x % kWave, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int n = lane & 15, g = lane >> 4;
    const ProblemDesc &pd = a.D.pd[a.cls[0]];
    const int d = pd.d, K = __builtin_amdgcn_readfirstlane(pd.K);
    const float nupd = pd.nu_plus_d, inv_nu = 1.0f / pd.nu, trust = fd_trust<FAM>(pd.nu);
    const uint32_t i = (SPLIT ? blockIdx.x : blockIdx.x * kFdWaves + wv) * 16 + n, ir = min(i, (uint32_t)a.ext_n - 1);
    float x[KS], hp[KS], hm[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int c = 4 * ks + g;
        x[ks] = c < d ? as_global(a.X)[(size_t)ir * d + c] : 0.0f;
        const float h = c < d ? fd_half_step(pd.fd_h, x[ks]) : 0.0f, up = x[ks] + h, dn = x[ks] - h;
        hp[ks] = up - x[ks];
        hm[ks] = dn - x[ks];
    }
    const __amdgpu_buffer_rsrc_t rs_pf = table_rsrc(pd.Pfrag, (uint32_t)K * DP * DP * 4u);
    const __amdgpu_buffer_rsrc_t rs_mu = table_rsrc(pd.muB, (uint32_t)K * DP * 4u);
    const __amdgpu_buffer_rsrc_t rs_lc = table_rsrc(pd.logc2, (uint32_t)K * 4u);
    LseStates<2 * KS> st;
    const int k_begin = SPLIT ? (int)((long)K * wv / kFdWaves) : 0;
    const int k_end = SPLIT ? (int)((long)K * (wv + 1) / kFdWaves) : K;
    st.clear(k_begin == 0);
    for (int k = k_begin; k < k_end; ++k) {
        const int pf_k = k * DP * DP * 4, mu_k = k * DP * 4;
        float pa[KS][MB], diag[KS], dl[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) load_frag_buf<MB>(rs_pf, (ks * kWave + lane) * MB * 4, pf_k, pa[ks]);
        // P_jj of coordinate j = 4 ks + g: row block ks / 4, lane 16 g + (4 g + ks % 4)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            diag[ks] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(
                           rs_pf, ((ks * kWave + 20 * g + (ks & 3)) * MB + (ks >> 2)) * 4, pf_k, 0));
#pragma unroll
        for (int ks = 0; ks < KS; ks += 4) {
            const f32x4 v = __builtin_bit_cast(
                f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_mu, (g * KS + ks) * 4, mu_k, 0));
            dl[ks] = x[ks] - v[0]; dl[ks + 1] = x[ks + 1] - v[1];
            dl[ks + 2] = x[ks + 2] - v[2]; dl[ks + 3] = x[ks + 3] - v[3];
        }
        const float lc2 = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_lc, 0, k * 4, 0));
        f32x4 acc[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[ks][mb], dl[ks], acc[mb], 0, 0, 0);
        float q = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) q = fmaf(dl[ks], acc[ks / 4][ks % 4], q);
        q += __shfl_xor(q, 16, kWave);
        q += __shfl_xor(q, 32, kWave);
        float t[2 * KS], low = q;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const float u2 = 2.0f * acc[ks / 4][ks % 4];
            t[2 * ks] = fmaf(hp[ks], fmaf(hp[ks], diag[ks], u2), q);
            t[2 * ks + 1] = fmaf(hm[ks], fmaf(hm[ks], diag[ks], u2), q);
            low = fminf(low, fminf(t[2 * ks], t[2 * ks + 1]));
        }
        if (__any(long_step(low, q, trust)))
#pragma clang loop unroll(disable)
            for (int i = 0; i < 2 * KS; ++i) {
                const int ks = i >> 1;
                float own = 0.0f, ti = 0.0f;
#pragma unroll
                for (int j = 0; j < KS; ++j) {
                    own = j == ks ? x[j] : own;
                    ti = j == ks ? ((i & 1) ? t[2 * j + 1] : t[2 * j]) : ti;
                }
                const bool mine = 4 * ks + g < d && long_step(ti, q, trust);
                if (!__any(mine)) continue;
                const float h = fd_half_step(pd.fd_h, own);
                own = ((i & 1) ? own - h : own + h) -
                      __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_mu, (g * KS + ks) * 4, mu_k, 0));
                // the four lanes of a point hold four coordinates: one contraction each
#pragma clang loop unroll(disable)
                for (int gg = 0; gg < 4; ++gg) {
                    if (!__any(mine && g == gg)) continue;
                    f32x4 acc1[MB];
                    float dl1[KS], q1 = 0.0f;
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc1[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < KS; ++j) {
                        dl1[j] = (j == ks && g == gg) ? own : dl[j];
                        float pj[MB];
                        load_frag_buf<MB>(rs_pf, (j * kWave + lane) * MB * 4, pf_k, pj);
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
                            acc1[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(pj[mb], dl1[j], acc1[mb], 0, 0, 0);
                    }
#pragma unroll
                    for (int j = 0; j < KS; ++j) q1 = fmaf(dl1[j], acc1[j / 4][j % 4], q1);
                    q1 += __shfl_xor(q1, 16, kWave);
                    q1 += __shfl_xor(q1, 32, kWave);
                    ti = mine && g == gg ? q1 : ti;
                }
#pragma unroll
                for (int j = 0; j < 2 * KS; ++j) t[j] = j == i ? ti : t[j];
            }
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) t[i] = component_log2<FAM>(lc2, t[i], nupd, inv_nu);
        st.add(t);
    }
    if constexpr (SPLIT) {
        st.merge(wv, lane);
        if (wv != 0) return;
    }
    if (i >= (uint32_t)a.ext_n) return;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int c = 4 * ks + g;
        const float h = fd_half_step(pd.fd_h, x[ks]), up = x[ks] + h, dn = x[ks] - h;
        if (c < d) a.G_out[(size_t)i * d + c] = st.log2_ratio(2 * ks, 2 * ks + 1) * kLn2 / (up - dn);
    }
}

// d <= 8: one point a lane, records through LDS as in alu_direct_kernel.
template <int FAM, int W, bool SPLIT>
__global__ __launch_bounds__(kAluBlock) void alu_fd_kernel(EvalArgs a) {
    constexpr int T = W * (W + 1) / 2, R = alu_record(W);
    static_assert(kAluBlock == kWave * kFdWaves, "four waves share a tile's components");
    __shared__ f32x4 s_rec[kAluChunk * (R / 4)];
    const int lane = threadIdx.x % kWave, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const ProblemDesc &pd = a.D.pd[a.cls[0]];
    const int d = pd.d, K = __builtin_amdgcn_readfirstlane(pd.K);
    const float nupd = pd.nu_plus_d, inv_nu = 1.0f / pd.nu, trust = fd_trust<FAM>(pd.nu);
    const uint32_t i = (SPLIT ? blockIdx.x : blockIdx.x * kFdWaves + wv) * kWave + lane;
    const bool in = i < (uint32_t)a.ext_n;
    float x[W], hp[W], hm[W];
#pragma unroll
    for (int c = 0; c < W; ++c) {
        x[c] = (in && c < d) ? as_global(a.X)[(size_t)i * d + c] : 0.0f;
        const float h = c < d ? fd_half_step(pd.fd_h, x[c]) : 0.0f, up = x[c] + h, dn = x[c] - h;
        hp[c] = up - x[c];
        hm[c] = dn - x[c];
    }
    LseStates<2 * W> st;
    st.clear(!SPLIT || wv == 0);
    for (int k0 = 0; k0 < K; k0 += kAluChunk) {
        const int n = min(kAluChunk, K - k0);
        if (k0) __syncthreads();
        for (int e = threadIdx.x; e < n * (R / 4); e += kAluBlock)
            s_rec[e] = reinterpret_cast<const gf32x4 *>(as_global(pd.Pfrag) + (size_t)k0 * R)[e];
        __syncthreads();
        for (int k = SPLIT ? wv : 0; k < n; k += SPLIT ? kFdWaves : 1) {
            float rec[R], dl[W], u[W], q = 0.0f, t[2 * W];
#pragma unroll
            for (int e = 0; e < R / 4; ++e) {
                const f32x4 v = s_rec[k * (R / 4) + e];
                rec[4 * e] = v[0]; rec[4 * e + 1] = v[1]; rec[4 * e + 2] = v[2]; rec[4 * e + 3] = v[3];
            }
#pragma unroll
            for (int c = 0; c < W; ++c) dl[c] = x[c] - rec[T + c];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                float acc = 0.0f;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    const int lo = c < j ? c : j, hi = c < j ? j : c;
                    acc = fmaf(rec[lo * W - lo * (lo - 1) / 2 + (hi - lo)], dl[j], acc);
                }
                u[c] = acc;
                q = fmaf(dl[c], acc, q);
            }
            float low = q;
#pragma unroll
            for (int c = 0; c < W; ++c) {
                const float pjj = rec[c * W - c * (c - 1) / 2], u2 = 2.0f * u[c];
                t[2 * c] = fmaf(hp[c], fmaf(hp[c], pjj, u2), q);
                t[2 * c + 1] = fmaf(hm[c], fmaf(hm[c], pjj, u2), q);
                low = fminf(low, fminf(t[2 * c], t[2 * c + 1]));
            }
            if (__any(long_step(low, q, trust)))
#pragma clang loop unroll(disable)
                for (int i1 = 0; i1 < 2 * W; ++i1) {
                    const int c1 = i1 >> 1;
                    float own = 0.0f, ti = 0.0f, dl1[W], q1 = 0.0f;
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        own = c == c1 ? x[c] : own;
                        ti = c == c1 ? ((i1 & 1) ? t[2 * c + 1] : t[2 * c]) : ti;
                    }
                    const bool mine = c1 < d && long_step(ti, q, trust);
                    if (!__any(mine)) continue;
                    const float h = fd_half_step(pd.fd_h, own);
                    own = ((i1 & 1) ? own - h : own + h) - s_rec[k * (R / 4) + (T + c1) / 4][(T + c1) % 4];
#pragma unroll
                    for (int c = 0; c < W; ++c) dl1[c] = c == c1 ? own : dl[c];
#pragma unroll
                    for (int c = 0; c < W; ++c) {
                        float acc = 0.0f;
#pragma unroll
                        for (int j = 0; j < W; ++j) {
                            const int lo = c < j ? c : j, hi = c < j ? j : c;
                            acc = fmaf(rec[lo * W - lo * (lo - 1) / 2 + (hi - lo)], dl1[j], acc);
                        }
                        q1 = fmaf(dl1[c], acc, q1);
                    }
#pragma unroll
                    for (int c = 0; c < 2 * W; ++c) t[c] = c == i1 && mine ? q1 : t[c];
                }
#pragma unroll
            for (int c = 0; c < 2 * W; ++c) t[c] = component_log2<FAM>(rec[T + W], t[c], nupd, inv_nu);
            st.add(t);
        }
    }
    if constexpr (SPLIT) {
        st.merge(wv, lane);
        if (wv != 0) return;
    }
    if (!in) return;
#pragma unroll
    for (int c = 0; c < W; ++c) {
        const float h = fd_half_step(pd.fd_h, x[c]), up = x[c] + h, dn = x[c] - h;
        if (c < d) a.G_out[(size_t)i * d + c] = st.log2_ratio(2 * c, 2 * c + 1) * kLn2 / (up - dn);
    }
}

// Components are shared while the tiles leave SIMDs idle and there is work in a
// component to share (us unshared / shared; tiles of 64 points at width 8, of
// 16 above): width 16, K = 16: 11.4 / 6.9 at 256 tiles, 11.7 / 11.8 at 1024, 25
// / 29 at 4096; K = 64: 31 / 25 at 1024; K = 4: 6.6 / 6.9 at 256; width 32, K =
// 4: 9.4 / 8.0 at 256, K = 64: 57 / 53 at 1024; width 64, K = 16: 45 / 22 at
// 256, 47 / 56 at 1024; width 8, K = 16: 17 / 10 at 256, 18.1 / 21.7 at 1024.
static bool fd_split(int DP, int K, long tiles) {
    return K * DP >= 128 && (tiles <= 512 || (tiles <= 1024 && K >= 32 && DP <= 32));
}

static hipError_t mixture_fd_rows(const EvalArgs &a, int d, int DP, int family, int K, hipStream_t st) {
    const int per_tile = DP == kAluDP ? kWave : 16;
    const long tiles = ((long)a.ext_n + per_tile - 1) / per_tile;
    const bool split = fd_split(DP, K, tiles);
    const dim3 b(kWave * kFdWaves), g((unsigned)(split ? tiles : (tiles + kFdWaves - 1) / kFdWaves));
#define CHISAO_FD(KERNEL, N)                                                                 \
    do {                                                                                     \
        if (family == 0) {                                                                   \
            if (split) hipLaunchKernelGGL((KERNEL(N, 0, true)), g, b, 0, st, a);             \
            else hipLaunchKernelGGL((KERNEL(N, 0, false)), g, b, 0, st, a);                  \
        } else {                                                                             \
            if (split) hipLaunchKernelGGL((KERNEL(N, 1, true)), g, b, 0, st, a);             \
            else hipLaunchKernelGGL((KERNEL(N, 1, false)), g, b, 0, st, a);                  \
        }                                                                                    \
    } while (0)
#define CHISAO_FD_MFMA(DP, F, S) mixture_fd_kernel<DP, F, S>
#define CHISAO_FD_ALU(W, F, S) alu_fd_kernel<F, W, S>
    switch (DP == kAluDP ? alu_width(d) : DP) {
        case 2: CHISAO_FD(CHISAO_FD_ALU, 2); break;
        case 4: CHISAO_FD(CHISAO_FD_ALU, 4); break;
        case 8: CHISAO_FD(CHISAO_FD_ALU, 8); break;
        case 16: CHISAO_FD(CHISAO_FD_MFMA, 16); break;
        case 32: CHISAO_FD(CHISAO_FD_MFMA, 32); break;
        case 64: CHISAO_FD(CHISAO_FD_MFMA, 64); break;
        default: return hipErrorInvalidValue;
    }
#undef CHISAO_FD_ALU
#undef CHISAO_FD_MFMA
#undef CHISAO_FD
    return hipGetLastError();
}

hipError_t launch_mixture_fd(const EvalArgs &a, int d, int DP, int family, int K, hipStream_t st) {
    return for_launch_rows(a, d, [&](const EvalArgs &r) { return mixture_fd_rows(r, d, DP, family, K, st); });
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
template <int DP, int FAM, bool H16>
static hipError_t dispatch_modes(const EvalArgs &a, int center, bool fd, bool grad, dim3 grid, hipStream_t st) {
    const dim3 block(kWave);
    constexpr int S = trial_split<DP, FAM>();
    constexpr bool kStencils = FAM < kFamClosed;  // (the closed forms' are closed_fd_kernel's)
#define CHISAO_GO(C, G, F)                                                                             \
    do {                                                                                               \
        if constexpr (!(F) || kStencils)                                                               \
            hipLaunchKernelGGL((eval_kernel<DP, FAM, G, C, F, 1, false, H16>), grid, block, 0, st, a); \
    } while (0)
#define CHISAO_GO_HALF(G) \
    hipLaunchKernelGGL((eval_kernel<DP, FAM, G, kDirect, false, 1, true, H16>), grid, block, 0, st, a)
#define CHISAO_GO_SPLIT(C, G, F) \
    hipLaunchKernelGGL((eval_kernel<DP, FAM, G, C, F, S, false, H16>), grid, dim3(kWave * S), 0, st, a)
#define CHISAO_GO_DSPLIT(G, N, HALF) \
    hipLaunchKernelGGL((eval_kernel<DP, FAM, G, kDirect, false, N, HALF, H16>), grid, dim3(kWave * N), 0, st, a)
    constexpr bool kHalfOk = FAM < kFamClosed && DP != kAluDP;  // tiles of two MFMA column blocks
    if constexpr (H16 && DP == 64) {
        if (a.share) {
            const dim3 b4(kShareWaves * kWave);
            if (center == kProbe) hipLaunchKernelGGL((eval_kernel<DP, FAM, true, kProbe, false, 1, false, true, true>), grid, b4, 0, st, a);
            else if (grad) hipLaunchKernelGGL((eval_kernel<DP, FAM, true, kDirect, false, 1, false, true, true>), grid, b4, 0, st, a);
            else hipLaunchKernelGGL((eval_kernel<DP, FAM, false, kDirect, false, 1, false, true, true>), grid, b4, 0, st, a);
            return hipGetLastError();
        }
    }
    if (center == kDirect) {
        if (fd) CHISAO_GO(kDirect, false, true);
        else if (kHalfOk && a.dsplit) {
            if constexpr (kHalfOk) {
                if (a.dsplit == kSplitHalf) {
                    if (grad) CHISAO_GO_DSPLIT(true, kSplitHalf, true);
                    else CHISAO_GO_DSPLIT(false, kSplitHalf, true);
                } else {
                    if (grad) CHISAO_GO_DSPLIT(true, kSplitFull, false);
                    else CHISAO_GO_DSPLIT(false, kSplitFull, false);
                }
            }
        } else if (kHalfOk && a.half_tiles) {
            if constexpr (kHalfOk) {
                if (grad) CHISAO_GO_HALF(true);
                else CHISAO_GO_HALF(false);
            }
        } else if (grad) CHISAO_GO(kDirect, true, false);
        else CHISAO_GO(kDirect, false, false);
    } else if (center == kTrial) {
        if (grad) CHISAO_GO_SPLIT(kTrial, true, false);
        else CHISAO_GO_SPLIT(kTrial, false, false);
    } else {
        if (fd) CHISAO_GO(kProbe, false, true);
        else CHISAO_GO(kProbe, true, false);
    }
#undef CHISAO_GO
#undef CHISAO_GO_HALF
#undef CHISAO_GO_SPLIT
#undef CHISAO_GO_DSPLIT
    return hipGetLastError();
}

// Workgroups of a line-search launch resident at once on the current device
// (the occupancy of the class's split trial kernel times the CU count), or 0
// where line-search tiles are not split.
template <int DP, int FAM, bool H16>
static int trial_resident(bool grad) {
    constexpr int S = trial_split<DP, FAM>();
    if constexpr (S == 1) {
        return 0;
    } else {
        int nb = 0, dev = 0, cus = 0;
        const hipError_t e = grad ? hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                        &nb, eval_kernel<DP, FAM, true, kTrial, false, S, false, H16>, kWave * S, 0)
                                  : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                        &nb, eval_kernel<DP, FAM, false, kTrial, false, S, false, H16>, kWave * S, 0);
        if (e != hipSuccess || hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
            (void)hipGetLastError();  // no limit then; leave no error for later launches to report
            return 0;
        }
        return nb * cus;
    }
}

template <int DP>
static int trial_resident_dp(int family, bool split, bool grad) {
    if constexpr (DP >= 32)
        if (split) return family == 0 ? trial_resident<DP, 0, true>(grad) : trial_resident<DP, 1, true>(grad);
    return family == 0 ? trial_resident<DP, 0, false>(grad) : trial_resident<DP, 1, false>(grad);
}

int trial_resident_blocks(int DP, int family, bool split, bool grad) {
    if (family >= kFamClosed) return 0;
    switch (DP) {
        case 16: return trial_resident_dp<16>(family, split, grad);
        case 32: return trial_resident_dp<32>(family, split, grad);
        case 64: return trial_resident_dp<64>(family, split, grad);
        default: return 0;
    }
}

template <int DP>
static hipError_t dispatch_family(const EvalArgs &a, int fam, int center, bool fd, bool grad, dim3 grid,
                                  hipStream_t st) {
    if constexpr (DP >= 32)
        if (a.split && fam < kFamClosed)
            return fam == 0 ? dispatch_modes<DP, 0, true>(a, center, fd, grad, grid, st)
                            : dispatch_modes<DP, 1, true>(a, center, fd, grad, grid, st);
    if (fam == 0) return dispatch_modes<DP, 0, false>(a, center, fd, grad, grid, st);
    if (fam == 1) return dispatch_modes<DP, 1, false>(a, center, fd, grad, grid, st);
    return dispatch_modes<DP, kFamClosed, false>(a, center, fd, grad, grid, st);
}

// 128-point tiles with shared components: at width 64, from the 2048 tiles of
// 32 points on that make 512 workgroups, two for every CU (at 1024 tiles it is
// 185 us against 154, K = 128; at 2048 252 against 264).  At width 32 a
// component is 4 KB and not worth the barrier: 182 us against 159 (262144
// points, K = 48).
static bool share_components(const EvalArgs &a, int DP, int center, bool fd) {
    if (!a.split || DP != 64 || fd || center == kTrial || a.dsplit) return false;
    return a.max_tiles >= 2048 && !(center == kDirect && a.half_tiles);
}

hipError_t launch_eval(EvalArgs a, int DP, int family, int center, bool fd, bool grad, hipStream_t st) {
    if (a.max_tiles <= 0 || a.n_cls <= 0) return hipSuccess;
    if (a.n_cls > kMaxClass) return hipErrorInvalidValue;
    if (fd && family >= kFamClosed) {
        // (a 32-point tile holds at most 16 centres)
        const long need = (16 * a.max_tiles + kCfdWaves - 1) / kCfdWaves;
        const dim3 g((unsigned)(need < 4096 ? need : 4096)), b(kWave * kCfdWaves);
        if (center == kDirect) hipLaunchKernelGGL(closed_fd_kernel<kDirect>, g, b, 0, st, a);
        else hipLaunchKernelGGL(closed_fd_kernel<kProbe>, g, b, 0, st, a);
        return hipGetLastError();
    }
    const long cap = a.grid_cap > 0 ? a.grid_cap : 8192;
    // max_tiles counts 32-point tiles; half tiles are twice as many
    const bool halves = a.half_tiles || a.dsplit == kSplitHalf;
    a.share = share_components(a, DP, center, fd);
    // (a tile of each problem may be partly filled)
    const long tiles = a.share ? a.max_tiles / kShareWaves + a.n_cls
                               : ((center == kDirect && !fd && halves) ? 2 * a.max_tiles : a.max_tiles);
    long g = tiles < cap ? tiles : cap;
    if (a.order == 1) g = (g + 7) / 8 * 8;  // whole rounds over the XCDs
    const dim3 grid((unsigned)g);
    // the closed forms share one instantiation per padded dimension and
    // select the function per problem
    const int fam = family >= kFamClosed ? kFamClosed : family;
    switch (DP) {
        case kAluDP:  // mixtures only
            return fam == 0   ? dispatch_modes<kAluDP, 0, false>(a, center, fd, grad, grid, st)
                   : fam == 1 ? dispatch_modes<kAluDP, 1, false>(a, center, fd, grad, grid, st)
                              : hipErrorInvalidValue;
        case 16: return dispatch_family<16>(a, fam, center, fd, grad, grid, st);
        case 32: return dispatch_family<32>(a, fam, center, fd, grad, grid, st);
        case 64: return dispatch_family<64>(a, fam, center, fd, grad, grid, st);
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// Per-component constants.  One workgroup per component: float64 Cholesky of
// the precision matrix for log|P_k| (setup only), then the MFMA fragment
// layouts (or, at the VALU width, the component records).  bad[0] is set when
// a matrix is not positive definite; ill[0] (not null) when its mean P_jj
// (P^-1)_jj exceeds kappa.  logc2 null: the layouts alone.
// ---------------------------------------------------------------------------
// Two-part tables of component k: fragments [part][K step][row block][lane]
// in the f16 instruction's A-operand order, rows permuted as lane_coord
// states, and the scaled centre in the lanes' order ([row][position]).
__global__ __launch_bounds__(64) void two_part_kernel(int d, int DP, const float *mu_all, const float *prec,
                                                      const float *xs, float kq, float *Pfrag, float *muB) {
    const int k = blockIdx.x, lane = threadIdx.x;
    const float *A = prec + (size_t)k * d * d, *mu = mu_all + (size_t)k * d;
    const int KS = DP / 4, MB = DP / 16, S = DP / 32;
    _Float16 *P = reinterpret_cast<_Float16 *>(Pfrag + (size_t)k * DP * DP);
    const int rho = lane & 15;
    for (int s = 0; s < S; ++s)
        for (int mb = 0; mb < MB; ++mb)
            for (int j = 0; j < 8; ++j) {
                const int row = lane_coord(4 * mb + (rho & 3), rho >> 2), col = lane_coord(8 * s + j, lane >> 4);
                float v = 0.0f;
                // scaled by 2^(kTwoPartP - e_row - e_col) = 1 / (kq xs_row xs_col)
                if (row < d && col < d)
                    v = ldexpf(A[row * d + col], -(ilogbf(kq) + ilogbf(xs[row]) + ilogbf(xs[col])));
                const _Float16 h = (_Float16)v, l = (_Float16)(v - (float)h);
                const size_t o = ((size_t)(s * MB + mb) * kWave + lane) * 8 + j;
                P[o] = h;
                P[(size_t)S * MB * kWave * 8 + o] = l;
            }
    if (lane < DP) {
        const int c = lane_coord(lane % KS, lane / KS);
        muB[(size_t)k * DP + lane] = c < d ? mu[c] * xs[c] : 0.0f;
    }
}

// Mean over j of P_jj (P^-1)_jj from the Cholesky factor L (lower triangle, row
// stride d): lane j solves L y = e_j, (P^-1)_jj = |y|^2.
__device__ float mean_kappa(int d, const float *A, const double *L, int lane) {
    __shared__ float Y[64][64];
    double sq = 0.0;
    for (int i = 0; i < d; ++i) {
        // (four chains, so that the reads of one do not wait for the others)
        double acc[4] = {i == lane ? 1.0 : 0.0, 0.0, 0.0, 0.0};
        int c = 0;
        for (; c + 4 <= i; c += 4)
#pragma unroll
            for (int o = 0; o < 4; ++o) acc[o] -= L[i * d + c + o] * (double)Y[c + o][lane];
        for (; c < i; ++c) acc[0] -= L[i * d + c] * (double)Y[c][lane];
        const double y = ((acc[0] + acc[1]) + (acc[2] + acc[3])) / L[i * d + i];
        Y[i][lane] = (float)y;
        sq += y * y;
    }
    float v = lane < d ? (float)(sq * (double)A[lane * d + lane]) : 0.0f;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o, kWave);
    return v / (float)d;
}

__global__ __launch_bounds__(64) void prepare_kernel(int family, int d, int DP, int K, float nu, const float *log_w,
                                                     const float *mu, const float *prec, float *logc2, float *Pfrag,
                                                     float *muB, int *bad, int *ill, float kappa) {
    const int k = blockIdx.x;
    const int lane = threadIdx.x;
    __shared__ double L[64 * 64];
    __shared__ double diag_log[64];
    const float *A = prec + (size_t)k * d * d;
    if (logc2) {
        for (int e = lane; e < d * d; e += 64) L[e] = (double)A[e];
        __syncthreads();
        // right-looking Cholesky, one column at a time
        for (int j = 0; j < d; ++j) {
            if (lane == 0) {
                double v = L[j * d + j];
                if (!(v > 0.0)) {
                    atomicExch(bad, 1);
                    v = 1.0;
                }
                L[j * d + j] = sqrt(v);
                diag_log[j] = log(L[j * d + j]);
            }
            __syncthreads();
            for (int i = j + 1 + lane; i < d; i += 64) L[i * d + j] /= L[j * d + j];
            __syncthreads();
            for (int e = lane; e < (d - j - 1) * (d - j - 1); e += 64) {
                const int i = j + 1 + e / (d - j - 1), c = j + 1 + e % (d - j - 1);
                if (c <= i) L[i * d + c] -= L[i * d + j] * L[c * d + j];
            }
            __syncthreads();
        }
        if (lane == 0) {
            double logdet = 0.0;
            for (int j = 0; j < d; ++j) logdet += 2.0 * diag_log[j];
            const double log_2pi = 1.8378770664093454835606594728112;
            double c;
            if (family == 0) {
                c = -0.5 * d * log_2pi + 0.5 * logdet;
            } else {
                c = lgamma(0.5 * ((double)nu + d)) - lgamma(0.5 * (double)nu) - 0.5 * d * log((double)nu * M_PI) +
                    0.5 * logdet;
            }
            logc2[k] = (float)(((double)log_w[k] + c) * 1.4426950408889634);
            if (DP == kAluDP) {
                const int W = alu_width(d), T = W * (W + 1) / 2;
                Pfrag[(size_t)k * alu_record(W) + T + W] = logc2[k];
            }
        }
        if (ill && !(mean_kappa(d, A, L, lane) <= kappa) && lane == 0) atomicExch(ill, 1);
    }
    if (DP == kAluDP) {
        // one record per component: upper triangle of P row by row, mu, and
        // (above) the log2 weight; coordinates past d are zero
        const int W = alu_width(d), T = W * (W + 1) / 2, R = alu_record(W);
        float *rec = Pfrag + (size_t)k * R;
        for (int e = lane; e < T; e += 64) {
            int i = 0, r = e;
            while (r >= W - i) {
                r -= W - i;
                ++i;
            }
            const int j = i + r;
            rec[e] = (i < d && j < d) ? A[i * d + j] : 0.0f;
        }
        if (lane < W) rec[T + lane] = lane < d ? mu[(size_t)k * d + lane] : 0.0f;
        if (lane > 0 && lane < R - T - W) rec[T + W + lane] = 0.0f;
        return;
    }
    // fragments with permuted rows: Pfrag[k][ks][lane][mb] = P[pi][4 ks + lane/16],
    // pi = 4 (4 mb + rho % 4) + rho / 4 for rho = lane % 16
    const int KS = DP / 4, MB = DP / 16;
    for (int ks = 0; ks < KS; ++ks)
        for (int mb = 0; mb < MB; ++mb) {
            const int rho = lane & 15;
            const int row = 4 * (4 * mb + (rho & 3)) + (rho >> 2), col = 4 * ks + (lane >> 4);
            const float v = (row < d && col < d) ? A[row * d + col] : 0.0f;
            Pfrag[(((size_t)k * KS + ks) * 64 + lane) * MB + mb] = v;
        }
    // centres in B-operand order: muB[k][g][ks] = mu[4 ks + g]
    if (lane < 4 * KS) {
        const int gg = lane / KS, i = lane % KS;
        const int cb = 4 * i + gg;
        muB[((size_t)k * 4 + gg) * KS + i] = cb < d ? mu[(size_t)k * d + cb] : 0.0f;
    }
}

hipError_t launch_prepare(int family, int d, int DP, int K, float nu, const float *log_w, const float *mu,
                          const float *prec, float *logc2, float *Pfrag, float *muB, int *bad, int *ill,
                          hipStream_t st) {
    hipLaunchKernelGGL(prepare_kernel, dim3(K), dim3(64), 0, st, family, d, DP, K, nu, log_w, mu, prec, logc2, Pfrag,
                       muB, bad, ill, two_part_kappa(d));
    return hipGetLastError();
}

hipError_t launch_two_part_tables(int d, int DP, int K, const float *mu, const float *prec, const float *xs, float kq,
                                  float *Pfrag2, float *muB2, hipStream_t st) {
    hipLaunchKernelGGL(two_part_kernel, dim3(K), dim3(64), 0, st, d, DP, mu, prec, xs, kq, Pfrag2, muB2);
    return hipGetLastError();
}

}  // namespace chisao
