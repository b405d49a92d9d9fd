// Library functions of the wide kernel, shared by the kernel and the host
// emulator that checks the scheduler.  Adjoint rules follow Appendix C, table
// tab:adjoints; w is the adjoint so far, or +0.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace ndvm {
namespace wide {

#define NDVM_WIDE_HD __host__ __device__ __forceinline__

NDVM_WIDE_HD double clamp_eps(double x) { return x < 1e-8 ? 1e-8 : x; }
NDVM_WIDE_HD double f_logc(double x) { return log(clamp_eps(x)); }
NDVM_WIDE_HD double f_sqrtc(double x) { return sqrt(clamp_eps(x)); }
NDVM_WIDE_HD double f_accsin(double x, double y, double w) {
    const double c = cos(y);
    return x != 0.0 ? w + x * c : w;
}
NDVM_WIDE_HD double f_acccos(double x, double y, double w) {
    const double s = -sin(y);
    return x != 0.0 ? w + x * s : w;
}
NDVM_WIDE_HD double f_acclog(double x, double y, double w) { return ((x != 0.0) & (y > 1e-8)) ? w + x / y : w; }
NDVM_WIDE_HD double f_accabs(double x, double y, double w) {
    const double d = y > 0.0 ? x : (y < 0.0 ? -x : 0.0);
    return x != 0.0 ? w + d : w;
}
NDVM_WIDE_HD double f_accpow(double x, double y, double z, double w) {
    const double c = log(y);
    return x != 0.0 ? w + z * c : w;
}
NDVM_WIDE_HD double f_accsqrt(double x, double y, double z, double w) {
    const double d = 2.0 * z;
    return ((x != 0.0) & (y > 1e-8)) ? w + x / d : w;
}

}  // namespace wide
}  // namespace ndvm

// ---- small matrices (at most 4 x 4), in memory M: M::ld(p, e) and M::st(p, e, v)
// access element e of the matrix at p.  Contractions are fma chains over the
// summation index in ascending order with a plain product as the first term.
// The forms below take one row (or element) each; a lane's four threads share
// a matrix.
namespace ndvm {
namespace wide {

// Immediate: rows and columns m, k, n (z = A[m, k] B[k, n]), or n elements as
// quads of 4 in the bits of m, k and n together; then flags.
constexpr uint32_t kFirstBit = 1u << 9, kNegBit = 1u << 10;
constexpr uint32_t mat_imm(uint32_t m, uint32_t k, uint32_t n) { return m | k << 3 | n << 6; }

// row `r` of d = A B
template <uint32_t K, uint32_t N, class M>
NDVM_WIDE_HD void mm_row(const M &mem, uint32_t a, uint32_t b, uint32_t d, uint32_t r) {
    double X[K], Y[K][N];
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) X[k] = mem.ld(a, r * K + k);
#pragma unroll
    for (uint32_t k = 0; k < K; ++k)
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) Y[k][j] = mem.ld(b, k * N + j);
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) {
        double s = X[0] * Y[0][j];
#pragma unroll
        for (uint32_t k = 1; k < K; ++k) s = fma(X[k], Y[k][j], s);
        mem.st(d, r * N + j, s);
    }
}
// row `r` of the adjoint of A: t[r, p] += sum over j of G[r, j] B[p, j] where `gate`(G has a nonzero)
template <uint32_t K, uint32_t N, class M, class G>
NDVM_WIDE_HD void mma_row(const M &mem, uint32_t g, uint32_t b, uint32_t t, uint32_t r, bool first, G gate) {
    double X[N], Y[K][N], base[K];
    bool nz = false;
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) X[j] = mem.ld(g, r * N + j);
#pragma unroll
    for (uint32_t p = 0; p < K; ++p) {
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) Y[p][j] = mem.ld(b, p * N + j);
        base[p] = 0.0;
    }
    if (!first)
#pragma unroll
        for (uint32_t p = 0; p < K; ++p) base[p] = mem.ld(t, r * K + p);
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) nz |= X[j] != 0.0;
    const bool on = gate(nz);
#pragma unroll
    for (uint32_t p = 0; p < K; ++p) {
        double s = X[0] * Y[p][0];
#pragma unroll
        for (uint32_t j = 1; j < N; ++j) s = fma(X[j], Y[p][j], s);
        mem.st(t, r * K + p, on ? base[p] + s : base[p]);
    }
}
// row `p` of the adjoint of B: t[p, j] += sum over i of A[i, p] G[i, j] where G has a nonzero
template <uint32_t R, uint32_t N, class M>
NDVM_WIDE_HD void mmb_row(const M &mem, uint32_t a, uint32_t g, uint32_t t, uint32_t p, uint32_t K, bool first) {
    double X[R], Y[R][N], base[N];
    bool nz = false;
#pragma unroll
    for (uint32_t i = 0; i < R; ++i) X[i] = mem.ld(a, i * K + p);
#pragma unroll
    for (uint32_t i = 0; i < R; ++i)
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) Y[i][j] = mem.ld(g, i * N + j);
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) base[j] = 0.0;
    if (!first)
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) base[j] = mem.ld(t, p * N + j);
#pragma unroll
    for (uint32_t i = 0; i < R; ++i)
#pragma unroll
        for (uint32_t j = 0; j < N; ++j) nz |= Y[i][j] != 0.0;
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) {
        double s = X[0] * Y[0][j];
#pragma unroll
        for (uint32_t i = 1; i < R; ++i) s = fma(X[i], Y[i][j], s);
        mem.st(t, p * N + j, nz ? base[j] + s : base[j]);
    }
}
// calls f<K, N> for sides 1 .. 4
#define NDVM_WIDE_SIDES(a, b, CALL) \
    switch ((a) * 8 + (b)) { \
        case 9: CALL(1, 1); break; case 10: CALL(1, 2); break; case 11: CALL(1, 3); break; case 12: CALL(1, 4); break; \
        case 17: CALL(2, 1); break; case 18: CALL(2, 2); break; case 19: CALL(2, 3); break; case 20: CALL(2, 4); break; \
        case 25: CALL(3, 1); break; case 26: CALL(3, 2); break; case 27: CALL(3, 3); break; case 28: CALL(3, 4); break; \
        case 33: CALL(4, 1); break; case 34: CALL(4, 2); break; case 35: CALL(4, 3); break; default: CALL(4, 4); break; \
    }

// elements e, e + 4, ... of the elementwise forms over `quads` quads
template <class M>
NDVM_WIDE_HD void vadd(const M &mem, uint32_t a, uint32_t b, uint32_t d, uint32_t e, uint32_t imm) {
    const uint32_t quads = imm & 511u;
    const bool neg = imm & kNegBit;
    for (uint32_t i = 0; i < quads; ++i, e += 4) {
        const double x = mem.ld(a, e), y = mem.ld(b, e);
        mem.st(d, e, x + (neg ? -y : y));
    }
}
// t += (+/-) g (adding a zero changes no adjoint, so no gate)
template <class M>
NDVM_WIDE_HD void vacc(const M &mem, uint32_t g, uint32_t t, uint32_t e, uint32_t imm) {
    const uint32_t quads = imm & 511u;
    const bool neg = imm & kNegBit, first = imm & kFirstBit;
    for (uint32_t i = 0; i < quads; ++i, e += 4) {
        const double x = mem.ld(g, e), base = first ? 0.0 : mem.ld(t, e);
        mem.st(t, e, base + (neg ? -x : x));
    }
}
template <class M>
NDVM_WIDE_HD void vscale(const M &mem, uint32_t a, uint32_t d, double s, uint32_t e, uint32_t imm) {
    const uint32_t quads = imm & 511u;
    for (uint32_t i = 0; i < quads; ++i, e += 4) {
        const double p = s * mem.ld(a, e);
        mem.st(d, e, p + -0.0);
    }
}
// t += g * s where some element of g is nonzero (n elements; e runs over them all)
template <class M>
NDVM_WIDE_HD bool any_of(const M &mem, uint32_t g, uint32_t n) {
    bool nz = false;
    for (uint32_t e = 0; e < n; ++e) nz |= mem.ld(g, e) != 0.0;
    return nz;
}
template <class M>
NDVM_WIDE_HD void vaccs(const M &mem, uint32_t g, uint32_t t, double s, uint32_t e, uint32_t n, bool first, bool on) {
    for (; e < n; e += 4) {
        const double x = mem.ld(g, e), base = first ? 0.0 : mem.ld(t, e), p = x * s;
        mem.st(t, e, on ? base + p : base);
    }
}
// sum of g[e] m[e] where some element of g is nonzero, else +0
template <class M>
NDVM_WIDE_HD double sdot(const M &mem, uint32_t g, uint32_t a, uint32_t n) {
    double x = mem.ld(g, 0), s = x * mem.ld(a, 0);
    bool nz = x != 0.0;
    for (uint32_t e = 1; e < n; ++e) {
        x = mem.ld(g, e);
        nz |= x != 0.0;
        s = fma(x, mem.ld(a, e), s);
    }
    return nz ? s : 0.0;
}
// element (i, j) of d = the transpose of A[m, q]; of its adjoint
template <class M>
NDVM_WIDE_HD void transpose(const M &mem, uint32_t a, uint32_t d, uint32_t e, uint32_t imm) {
    const uint32_t m = imm & 7u, q = (imm >> 3) & 7u;
    for (; e < m * q; e += 4) mem.st(d, e, mem.ld(a, e % m * q + e / m));
}
template <class M>
NDVM_WIDE_HD void transpose_acc(const M &mem, uint32_t g, uint32_t t, uint32_t e, uint32_t imm) {
    const uint32_t m = imm & 7u, q = (imm >> 3) & 7u;
    for (; e < m * q; e += 4) {   // t[i, j] += g[j, i]
        const double x = mem.ld(g, e % q * m + e / q), base = (imm & kFirstBit) ? 0.0 : mem.ld(t, e);
        mem.st(t, e, base + x);
    }
}
struct Inv2 {
    double det, v[4];
};
// determinant and inverse of the 2 x 2 matrix a: the adjugate times 1 / det
NDVM_WIDE_HD double det2(const double a[4]) {
    const double t1 = a[0] * a[3], t2 = a[1] * a[2];
    return t1 - t2;
}
NDVM_WIDE_HD Inv2 inverse2(const double a[4]) {
    Inv2 o;
    o.det = det2(a);
    const double r = 1.0 / o.det, nr = r * -1.0;
    o.v[0] = a[3] * r;
    o.v[1] = a[1] * nr;
    o.v[2] = a[2] * nr;
    o.v[3] = a[0] * r;
    return o;
}
template <class M>
NDVM_WIDE_HD void load4(const M &mem, uint32_t a, double v[4]) {
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) v[e] = mem.ld(a, e);
}
template <class M>
NDVM_WIDE_HD void inv2(const M &mem, uint32_t a, uint32_t d) {
    double v[4];
    load4(mem, a, v);
    const Inv2 o = inverse2(v);
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) mem.st(d, e, o.v[e]);
}
// adjoint of an inverse z: M1 = z^T g, then t -= M1 z^T where g has a nonzero
template <class M>
NDVM_WIDE_HD void inv2_acc(const M &mem, uint32_t z, uint32_t g, uint32_t t, uint32_t imm) {
    double Z[4], G[4], m1[4], base[4] = {0.0, 0.0, 0.0, 0.0};
    load4(mem, z, Z);
    load4(mem, g, G);
    if (!(imm & kFirstBit)) load4(mem, t, base);
    const bool on = (G[0] != 0.0) | (G[1] != 0.0) | (G[2] != 0.0) | (G[3] != 0.0);
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j) m1[i * 2 + j] = fma(Z[2 + i], G[2 + j], Z[i] * G[j]);
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j) {
            const double s = -fma(m1[i * 2 + 1], Z[j * 2 + 1], m1[i * 2] * Z[j * 2]);
            mem.st(t, i * 2 + j, on ? base[i * 2 + j] + s : base[i * 2 + j]);
        }
}
// adjoint of log det a: t += g a^-T where g != 0 and det > 1e-8
template <class M>
NDVM_WIDE_HD void logdet2_acc(const M &mem, uint32_t a, uint32_t t, double g, uint32_t imm) {
    double v[4], base[4] = {0.0, 0.0, 0.0, 0.0};
    load4(mem, a, v);
    if (!(imm & kFirstBit)) load4(mem, t, base);
    const Inv2 o = inverse2(v);
    const bool on = (g != 0.0) & (o.det > 1e-8);
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
#pragma unroll
        for (uint32_t j = 0; j < 2; ++j) {
            const double p = g * o.v[j * 2 + i];
            mem.st(t, i * 2 + j, on ? base[i * 2 + j] + p : base[i * 2 + j]);
        }
}

}  // namespace wide
}  // namespace ndvm
