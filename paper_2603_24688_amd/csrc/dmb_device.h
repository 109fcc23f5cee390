// dmb_device.h -- device-side math of the DM-gas pair step for gfx950.
//
// Paper: Hainje & Farrar, arXiv 2603.24688.  Each function names the passage
// it implements.  Templates over float/double are one code path: the pair
// math runs in `Real`, positions and sums in double.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dmb {

// Selects by bit masks (m all ones or zero).  The compiler turns a select whose
// operand is costly into a branch around the operand's computation; a mask keeps
// straight-line code one block for the scheduler.
__device__ __forceinline__ uint32_t bits(bool c) { return c ? ~0u : 0u; }
__device__ __forceinline__ float masked(float x, uint32_t m) { return __uint_as_float(__float_as_uint(x) & m); }
__device__ __forceinline__ double masked(double x, uint32_t m)
{
    const uint64_t b = uint64_t(__double_as_longlong(x));
    return __longlong_as_double((long long)((uint64_t(uint32_t(b >> 32) & m) << 32) | (uint32_t(b) & m)));
}
__device__ __forceinline__ float either(uint32_t m, float x, float y)      // m: x, else y
{
    return __uint_as_float((__float_as_uint(x) & m) | (__float_as_uint(y) & ~m));
}

constexpr double kPi = 3.14159265358979323846;
constexpr double kSqrtPi = 1.7724538509055160273;

// ---------------------------------------------------------------------------
// Cubic-spline kernel (Sec. 2.4): w(q) = 8/pi {1-6q^2+6q^3; 2(1-q)^3; 0}.
template <typename T>
__device__ __forceinline__ T kernel_w(T q)
{
    const T c = T(8.0 / kPi);
    if (q <= T(0.5)) return c * (T(1) + q * q * (T(6) * q - T(6)));
    if (q < T(1)) { T p = T(1) - q; return c * T(2) * p * p * p; }
    return T(0);
}

// Overlap H(delta, eta) = h_b^3 g for the cubic spline (Appendix D):
//   H = (2 pi / eta^3) int_0^1 ds s w(s) V(s),
//   V(s) = eta^2/delta [psi((s+delta)/eta) - psi(|s-delta|/eta)],  psi(Q) = int_0^Q q w(q) dq.
// V vanishes outside [max(0, delta - eta), min(1, delta + eta)].  Between
// consecutive breakpoints (where s, a = |s - delta|/eta or b = (s + delta)/eta
// crosses a branch edge of w or psi) the integrand is one polynomial of degree
// 9 in s, so 5-point Gauss-Legendre on each piece is exact up to rounding.
//
// Bound by binary64 vector instructions, so the work is what the pieces hold:
// at most five breakpoints can lie inside the support (1/2, delta,
// delta + eta/2, |delta - eta/2| and, for delta < eta, eta - delta), those
// outside are moved to its end, so that the sorted list has its pieces in front
// and the loop ends with the wave's longest list (2 to 6 pieces).  On a piece
// every branch is fixed, so its polynomials are picked once: w(s) and the tail
// T(q) = int_q^1 q w dq (all terms of one sign near q = 1) as Horner forms in
// q or 1 - q.  Where b >= 1, psi(b) - psi(a) = T(a); otherwise, with
// X = max(s, delta)/eta and y = min(s, delta)/eta, the difference on one branch
// is 2y times a form in X (or 1 - X) and y, free of the cancellation at small
// delta (and of the division by delta: eta^2/delta 2y = 2 eta min(1, s/delta)),
// and across the edge at 1/2, a piece no wider than 2 min(s, delta), T(a) - T(b).
// All 8/pi of w and T are in the caller's factor.
// Against nine pieces (those outside the support too) of five nodes, both
// branches of both ends formed at each: a binary64 step of 80 021 gas + 320 009
// DM 6.46 -> 3.12 ms, of the 4096 + 4096 box 1.64 -> 1.14 ms; the mean error
// against 113-bit arithmetic is 5-30 % smaller.
__device__ __forceinline__ double overlap_integral(double delta, double eta, double ie, double c_ed)
{
    // 5-point Gauss-Legendre: nodes 0, +-gx[0], +-gx[1] with weights gw[0..2]
    constexpr double gx[2] = {0.5384693101056830910, 0.9061798459386639928};
    constexpr double gw[3] = {0.5688888888888888889, 0.4786286704993664680, 0.2369268850561890875};
    const double lo0 = fmax(delta - eta, 0.0), hi = fmin(delta + eta, 1.0);
    double b1 = 0.5, b2 = delta, b3 = delta + 0.5 * eta, b4 = fabs(delta - 0.5 * eta), b5 = eta - delta;
    auto clamp = [lo0, hi](double& v) { v = v > lo0 && v < hi ? v : hi; };
    clamp(b1); clamp(b2); clamp(b3); clamp(b4); clamp(b5);
    auto order = [](double& x, double& y) { const double t = fmin(x, y); y = fmax(x, y); x = t; };
    order(b1, b2); order(b4, b5); order(b3, b5); order(b3, b4); order(b2, b5);
    order(b1, b4); order(b1, b3); order(b2, b4); order(b2, b3);
    const double id = c_ed * ie * ie;            // 1/delta (0 when delta = 0)
    double lo = lo0, nx = b1, acc = 0.0;
#pragma unroll 1
    while (lo < hi) {
        const double half = 0.5 * (nx - lo), mid = 0.5 * (nx + lo);
        // the piece's branches, taken at its midpoint
        const double am = fabs(mid - delta), bm = mid + delta;
        const bool s1 = mid > 0.5, a1 = am > 0.5 * eta, inner = bm < eta, b1r = bm > 0.5 * eta, right = mid > delta;
        // w(s)/(8/pi) = e3 t^3 + e2 t^2 + e0, t = 1 - s on the outer branch, else s
        const double e3 = s1 ? 2.0 : 6.0, e2 = s1 ? 0.0 : -6.0, e0 = s1 ? 0.0 : 1.0;
        // T(q)/(8/pi) = f0 + t^2 (f2 + t^2 (f4 + f5 t)), t = 1 - q on the outer branch, else q
        const double f0 = a1 ? 0.0 : 0.0875, f2 = a1 ? 0.0 : -0.5, f4 = a1 ? 0.5 : 1.5, f5 = a1 ? -0.4 : -1.2;
        // t of T(a), linear in s: (eta - |s - delta|)/eta on the outer branch, else |s - delta|/eta; like 1 - s
        // below it is carried from its value at the midpoint, so that a narrow piece near contact, where both
        // vanish, keeps its relative accuracy
        const double tm = (a1 ? (right ? (delta + eta) - mid : mid - (delta - eta)) : am) * ie;
        const double th = right != a1 ? half * ie : -half * ie;
        const double um = s1 ? 1.0 - mid : mid, uh = s1 ? -half : half;
        double sq[5], V[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const double xq = q == 0 ? 0.0 : (q == 1 ? -gx[0] : (q == 2 ? gx[0] : (q == 3 ? -gx[1] : gx[1])));
            sq[q] = q == 0 ? mid : fma(half, xq, mid);
            const double t = q == 0 ? tm : fma(th, xq, tm), t2 = t * t;
            V[q] = c_ed * fma(t2, fma(t2, fma(f5, t, f4), f2), f0);
        }
        if (inner) {
            const double p1 = a1 ? 0.0 : 1.0, p3 = a1 ? 2.0 : -6.0, p5 = a1 ? -0.4 : 1.2;
            const bool same = a1 == b1r;
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const double X = fmax(sq[q], delta) * ie, y = fmin(sq[q], delta) * ie, y2 = y * y;
                const double Z = a1 ? 1.0 - X : X, Z2 = Z * Z;
                const double br = fma(p5, fma(5.0 * Z2, fma(2.0, y2, Z2), y2 * y2), Z * fma(p3, Z2 + y2, p1));
                const double p = 1.0 - (X + y), pp = p * p;
                V[q] = same ? 2.0 * eta * (right ? 1.0 : sq[q] * id) * br : V[q] - c_ed * (pp * pp * fma(-0.4, p, 0.5));
            }
        }
        double piece = 0.0;
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const double wq = q == 0 ? gw[0] : (q < 3 ? gw[1] : gw[2]);
            const double xq = q == 0 ? 0.0 : (q == 1 ? -gx[0] : (q == 2 ? gx[0] : (q == 3 ? -gx[1] : gx[1])));
            const double u = q == 0 ? um : fma(uh, xq, um);
            piece = fma(wq * sq[q] * fma(u * u, fma(e3, u, e2), e0), V[q], piece);
        }
        acc = fma(half, piece, acc);
        lo = nx; nx = b2; b2 = b3; b3 = b4; b4 = b5; b5 = hi;
    }
    return acc;
}

constexpr double kOverlapScale = 128.0 / kPi;    // 2 pi (8/pi)^2

// ---------------------------------------------------------------------------
// Overlap for the binary32 path (Appendix D tabulates the overlap; here the
// table keeps RELATIVE accuracy over the whole support, down to pairs that
// barely touch).  With h_b >= h_s, eta = h_s/h_b, delta = d/h_b, H = h_b^3 g:
//   shell (h_b - d < h_s: the small kernel crosses the big one's surface):
//     rho = (h_b + h_s - d)/h_s in [0, 2),  H = eta^3 rho^8 QA(rho, eta);
//   core (h_b - d >= h_s: the small kernel lies inside the big one):
//     kappa = eta/(1 - delta) in (0, 1],  H = (1 - delta)^3 QB(delta, kappa).
// The envelopes carry how H vanishes at the support edge (as its eighth power
// in the distance to contact) and at the big kernel's surface (as the cube),
// so QA and QB are smooth and bounded (QA in [0.0038, 0.146], QB in
// [0.99, 6.3]).  For rho <= 1/2 the shell overlap has the closed form
//   QA = 512/(pi delta) [1/1120 - (1 + eta) rho/2520 + eta rho^2/6300]
// (one polynomial piece of the Appendix D integral), used for the nodes.
// Each region is a kTabN x kTabN grid of cells on [0,1]^2 (x = rho/2 or
// delta, y = eta or kappa); nodes carry Q and its two first derivatives
// scaled by the cell width; the interpolant is cubic Hermite along x for Q,
// linear along x for the y-derivative and cubic Hermite along y, stored per
// cell as polynomial coefficients in the cell offsets (a, b):
//   Q = P0(a) + P1(a) b + P2(a) b^2 + P3(a) b^3,
// P0, P2, P3 cubic and P1 linear in a, as four float4 (P0, P2, P3, P1) = 64
// bytes, so one lookup reads one aligned 64-byte segment.  Interpolation and
// coefficient rounding stay below 6e-7 of g itself.
constexpr int kTabN = 128;
constexpr int kTabCellsRegion = kTabN * kTabN;
constexpr int kTabCells = 2 * kTabCellsRegion;   // shell cells, then core cells

// 1/x for x > 0 in binary64: binary32 reciprocal and one Newton step
// (relative error ~1e-14; no binary64 division).
__device__ __forceinline__ double rcp64(double x)
{
    double r = double(__builtin_amdgcn_rcpf(float(x)));
    return r * fma(-x, r, 2.0);
}

// g(d; h1, h2) in binary64 from the binary64 squared distance of a pair
// inside the support (d2 < (h1 + h2)^2).  The distance is refined from the
// binary32 root by one Newton step in binary64, so that h_b + h_s - d and
// h_b - d keep their relative accuracy near contact.  The value is returned in
// binary64: near contact it falls far below the binary32 range.
__device__ __forceinline__ double overlap_g_table(const float4* __restrict__ tab, double d2, double h1, double h2)
{
    const double hb = h1 > h2 ? h1 : h2, hs = h1 > h2 ? h2 : h1;
    const float d0f = __builtin_amdgcn_sqrtf(float(d2));
    const double d0 = double(d0f);
    const double d = d0f > 0.f ? fma(d2 - d0 * d0, double(0.5f * __builtin_amdgcn_rcpf(d0f)), d0) : 0.0;
    const double ib = rcp64(hb);
    const double inner = hb - d;             // >= hs in the core
    const bool shell = inner < hs;
    const double num = shell ? (hb + hs) - d : hs;
    const double r = num * rcp64(shell ? hs : inner);   // rho (shell) or kappa (core)
    const double eta = hs * ib;
    const double x = shell ? 0.5 * r : d * ib, y = shell ? eta : r;
    const double fx = fmin(x, 1.0) * double(kTabN), fy = fmin(y, 1.0) * double(kTabN);
    const int i = min(int(fx), kTabN - 1), j = min(int(fy), kTabN - 1);
    // the cell polynomial (smooth, positive, of order one) in binary32: its rounding stays
    // below the table's own error; the envelope and the 1/h_b^3 scale stay in binary64
    const float a = float(fx - double(i)), b = float(fy - double(j));
    const float4* c = tab + 4 * ((shell ? 0 : kTabCellsRegion) + j * kTabN + i);
    const float4 q0 = c[0], q2 = c[1], q3 = c[2], q1 = c[3];
    auto cubic = [a](float4 q) { return fmaf(fmaf(fmaf(q.w, a, q.z), a, q.y), a, q.x); };
    const float p0 = cubic(q0), p2 = cubic(q2), p3 = cubic(q3), p1 = fmaf(q1.y, a, q1.x);
    const double Q = double(fmaf(fmaf(fmaf(p3, b, p2), b, p1), b, p0));
    // both envelopes and a select: one basic block, so the scheduler can overlap the cell loads
    const double r2 = r * r, r4 = r2 * r2, tc = inner * ib;
    const double env = shell ? eta * eta * eta * (r4 * r4) : tc * tc * tc;
    return Q * env * (ib * ib * ib);
}

// The same lookup returning binary32, for the binary32 DM pass, whose P_ij
// are binary32: the distance and the two differences that vanish at contact
// (h_b + h_s - d, h_b - d) are still formed in binary64, everything after
// them in binary32 (rounding below 4e-7 of g).  Overlaps under the binary32
// range (pairs within ~1e-5 h_s of contact) flush to zero, as the binary32
// P_ij built from them would.  The gas pass (binary64 terms) takes the
// binary64 lookup for such pairs (GasEval::finish), so an owner whose every
// neighbour is that close to contact keeps its relative accuracy.
// In two halves, so that a pass can put other work between them: begin() finds
// the cell and issues its loads, value() takes them.
struct Overlap32 {
    float4 q0, q2, q3;
    float2 q1;
    float a, b, env, ib;
    __device__ __forceinline__ void begin(const float4* __restrict__ tab, double d2, double h1, double h2)
    {
        const double hbd = h1 > h2 ? h1 : h2, hsd = h1 > h2 ? h2 : h1;
        // binary32 root, then one Newton step in binary64
        const float d0f = __builtin_amdgcn_sqrtf(float(d2));
        const double d0 = double(d0f);
        const double d = masked(fma(fma(-d0, d0, d2), double(0.5f * __builtin_amdgcn_rcpf(d0f)), d0), bits(d0f > 0.f));
        const double innerd = hbd - d;
        const bool shell = innerd < hsd;
        const uint32_t ms = bits(shell);
        const float hb = float(hbd), hs = float(hsd), inner = float(innerd);
        const float num = either(ms, float((hbd + hsd) - d), hs);
        ib = __builtin_amdgcn_rcpf(hb);
        const float r = num * __builtin_amdgcn_rcpf(either(ms, hs, inner));   // rho (shell) or kappa (core)
        const float eta = hs * ib;
        const float x = either(ms, 0.5f * r, float(d) * ib), y = either(ms, eta, r);
        const float fx = fminf(x, 1.f) * float(kTabN), fy = fminf(y, 1.f) * float(kTabN);
        const int i = min(int(fx), kTabN - 1), j = min(int(fy), kTabN - 1);
        a = fx - float(i);
        b = fy - float(j);
        const float4* c = tab + 4 * ((shell ? 0 : kTabCellsRegion) + j * kTabN + i);
        q0 = c[0]; q2 = c[1]; q3 = c[2];
        q1 = *reinterpret_cast<const float2*>(c + 3);
        const float r2 = r * r, r4 = r2 * r2, tc = inner * ib;
        env = either(ms, eta * eta * eta * (r4 * r4), tc * tc * tc);
    }
    __device__ __forceinline__ float value() const
    {
        auto cubic = [this](float4 q) { return fmaf(fmaf(fmaf(q.w, a, q.z), a, q.y), a, q.x); };
        const float p0 = cubic(q0), p2 = cubic(q2), p3 = cubic(q3), p1 = fmaf(q1.y, a, q1.x);
        const float Q = fmaf(fmaf(fmaf(p3, b, p2), b, p1), b, p0);
        return Q * env * (ib * ib * ib);
    }
};

__device__ __forceinline__ float overlap_g_table32(const float4* __restrict__ tab, double d2, double h1, double h2)
{
    Overlap32 o;
    o.begin(tab, d2, h1, h2);
    return o.value();
}

// g in binary64: delta and eta by division (near contact g goes as the eighth
// power of 1 + eta - delta), the integral's other factors from 1/h_s and 1/d.
template <typename T>
__device__ __forceinline__ T overlap_g_exact(T d, T hi, T hj)
{
    const double hb = double(hi > hj ? hi : hj), hs = double(hi > hj ? hj : hi), dd = double(d);
    const double delta = dd / hb, eta = hs / hb, is = 1.0 / hs;
    if (delta >= 1.0 + eta) return T(0);
    const double c_ed = dd > 0.0 ? eta * hs / dd : 0.0;
    return T(kOverlapScale * overlap_integral(delta, eta, hb * is, c_ed) * (is * is * is));
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): per round the products M0*x0 and
// M1*x2 give (hi1^x1^k0, lo1, hi0^x3^k1, lo0); key bumped by the Weyl
// constants between rounds.
struct U4 { uint32_t x, y, z, w; };

// x ^ y ^ z in one instruction (v_bitop3_b32)
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z)
{
    return uint32_t(__builtin_amdgcn_bitop3_b32(x, y, z, 0x96));
}

template <int R>
__device__ __forceinline__ U4 philox_rounds(U4 c, uint32_t k0, uint32_t k1)
{
    // the key schedule is rebuilt per call (scalar adds): hoisted, its 20 words
    // would occupy scalar registers for a whole pass.  Keys are wave-uniform.
    asm("" : "+s"(k0), "+s"(k1) : "v"(c.x));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // one 32x32->64 multiply (v_mad_u64_u32) gives both halves
        const uint64_t p0 = uint64_t(c.x) * 0xD2511F53u, p1 = uint64_t(c.z) * 0xCD9E8D57u;
        const uint32_t lo0 = uint32_t(p0), hi0 = uint32_t(p0 >> 32);
        const uint32_t lo1 = uint32_t(p1), hi1 = uint32_t(p1 >> 32);
        U4 n;
        n.x = xor3(hi1, c.y, k0);
        n.y = lo1;
        n.z = xor3(hi0, c.w, k1);
        n.w = lo0;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) { return philox_rounds<10>(c, k0, k1); }

// 24-bit centred uniform ((r >> 8) + 1/2) 2^-24, exactly representable.
template <typename T>
__device__ __forceinline__ T u24(uint32_t r)
{
    // one rounding of the 25-bit sum either way; the scale is a power of two
    if constexpr (sizeof(T) == 4) return fmaf(float(r >> 8), 1.f / 16777216.f, 0.5f / 16777216.f);
    else return (T(r >> 8) + T(0.5)) * T(1.0 / 16777216.0);
}

// Stream layout shared with every consumer of the random numbers:
// counter = (dm index, gas index, step, tag | box << 8), key = seed.
enum : uint32_t { kTagGasVel = 0u, kTagDir = 1u, kTagDecision = 2u, kTagTilt = 5u };

__device__ __forceinline__ U4 philox_block(uint32_t i, uint32_t j, uint32_t step, uint32_t tag, uint32_t box,
                                           uint32_t k0, uint32_t k1)
{
    U4 c{i, j, step, tag | (box << 8)};
    return philox4x32_10(c, k0, k1);
}

// The blocks philox_block(i, j, step, tag, box) of many pairs (i, j): the first
// three rounds hold five of the ten-round block's twenty products that depend
// on i alone or on j alone, formed once per i (owner) and once per j (other)
// instead of per pair.  With z, w, ... as the counter words after a round,
//   round 1: x = hi(step M1) ^ j ^ k0 (j alone), y = lo(step M1),
//            z = hi(i M0) ^ (tag | box << 8) ^ k1, w = lo(i M0) (i alone);
//   round 2: x M0 is j's, z M1 is i's; x, y are i's, w is j's;
//   round 3: x M0 is i's.
// pair() takes the rest, seven rounds and one product.
struct PhiloxPair {
    uint32_t x1, y1, w0, k0, k1;
    __device__ __forceinline__ PhiloxPair(uint32_t step, uint32_t tag, uint32_t box, uint32_t k0_, uint32_t k1_)
        : k0(k0_), k1(k1_)
    {
        const uint64_t p = uint64_t(step) * 0xCD9E8D57u;
        x1 = uint32_t(p >> 32) ^ k0;
        y1 = uint32_t(p);
        w0 = (tag | (box << 8)) ^ k1;
    }
    // j's part: the two halves of its round-2 product
    __device__ __forceinline__ void other(uint32_t j, uint32_t* a, uint32_t* b) const
    {
        const uint64_t p = uint64_t(x1 ^ j) * 0xD2511F53u;
        *a = uint32_t(p >> 32);
        *b = uint32_t(p);
    }
    // i's part: (w after round 1 ^ key, y after round 2 ^ key, high and low half of the round-3 product (high ^ key))
    __device__ __forceinline__ uint4 owner(uint32_t i) const
    {
        const uint64_t p = uint64_t(i) * 0xD2511F53u;
        const uint64_t q = uint64_t(uint32_t(p >> 32) ^ w0) * 0xCD9E8D57u;
        const uint32_t x2 = uint32_t(q >> 32) ^ y1 ^ (k0 + 0x9E3779B9u);
        const uint64_t r = uint64_t(x2) * 0xD2511F53u;
        return make_uint4(uint32_t(p) ^ (k1 + 0xBB67AE85u), uint32_t(q) ^ (k0 + 2u * 0x9E3779B9u),
                          uint32_t(r >> 32) ^ (k1 + 2u * 0xBB67AE85u), uint32_t(r));
    }
    __device__ __forceinline__ U4 pair(uint4 o, uint32_t a, uint32_t b) const
    {
        const uint64_t p = uint64_t(a ^ o.x) * 0xCD9E8D57u;
        U4 c{uint32_t(p >> 32) ^ o.y, uint32_t(p), o.z ^ b, o.w};
        return philox_rounds<7>(c, k0 + 3u * 0x9E3779B9u, k1 + 3u * 0xBB67AE85u);
    }
};

// cos(2 pi u), sin(2 pi u): the gfx950 transcendental unit takes turns.
__device__ __forceinline__ void sincos_turns(float u, float* s, float* c)
{
    *s = __builtin_amdgcn_sinf(u);
    *c = __builtin_amdgcn_cosf(u);
}
__device__ __forceinline__ void sincos_turns(double u, double* s, double* c) { sincospi(2.0 * u, s, c); }

// Binary32 uses the hardware units directly: log2 (within 1 ulp) times ln 2,
// square root and reciprocal (1 ulp).  Their arguments on the binary32 path
// are normal numbers or zero, so the library wrappers' rescaling of
// subnormal arguments is not needed.
__device__ __forceinline__ float log_real(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
__device__ __forceinline__ double log_real(double x) { return log(x); }
// -2 ln x; the factor -2 only moves exponents, so it joins ln 2 without a change of rounding
__device__ __forceinline__ float neg2log_real(float x) { return __builtin_amdgcn_logf(x) * (-2.f * 0.693147180559945309f); }
__device__ __forceinline__ double neg2log_real(double x) { return -2.0 * log(x); }
__device__ __forceinline__ float sqrt_real(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double sqrt_real(double x) { return sqrt(x); }
__device__ __forceinline__ float rcp_real(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_real(double x) { return 1.0 / x; }

// Three standard normals by Box-Muller from one Philox block.
template <typename T>
__device__ __forceinline__ void normals3(U4 r, T z[3])
{
    T u0 = u24<T>(r.x), u1 = u24<T>(r.y), u2 = u24<T>(r.z), u3 = u24<T>(r.w);
    T r0 = sqrt_real(neg2log_real(u0)), r1 = sqrt_real(neg2log_real(u2));
    T s, c, s2, c2;
    sincos_turns(u1, &s, &c);
    sincos_turns(u3, &s2, &c2);
    z[0] = r0 * c;
    z[1] = r0 * s;
    z[2] = r1 * c2;
}

// ---------------------------------------------------------------------------
// Anisotropic scattering (Sec. 2.2-2.3: dsigma/dOmega = sigma(v) p(Omega)).
// cos theta of the Henyey-Greenstein law p(c) = (1 - g^2) / (2 (1 + g^2 - 2 g c)^{3/2})
// (mean g) from a uniform u by its inverse CDF, and sin theta.  With t = 2u - 1
// the inverse c = (1 + g^2 - s^2) / (2g), s = (1 - g^2) / (1 - g + 2 g u),
// expands to (2t + g (t^2 + 3) + 2 g^2 t + g^3 (t^2 - 1)) / (2 (1 + g t)^2), free
// of the cancellation at small g (g = 0 gives t); and 1 - c^2 factors into
// 4 (1 - g^2)^2 u (1 - u) (1 - g + g u) (1 + g u) / (1 + g t)^4, so sin theta
// keeps its relative accuracy where c is within rounding of +-1.
template <typename T>
__device__ __forceinline__ void hg_angle(T g, T u, T* ct, T* st)
{
    const T t = T(2) * u - T(1), d = T(1) + g * t;
    const T c = (T(2) * t + g * (t * t + T(3)) + T(2) * g * g * t + g * g * g * (t * t - T(1))) / (T(2) * d * d);
    *ct = c < T(-1) ? T(-1) : (c > T(1) ? T(1) : c);
    const T p = u * (T(1) - u) * (T(1) - g + g * u) * (T(1) + g * u);
    *st = T(2) * (T(1) - g * g) * sqrt_real(p > T(0) ? p : T(0)) / (d * d);
}

// Orthonormal e1, e2 with (e1, e2, n) right-handed for a unit n (the
// branch-free construction of Duff et al., J. Comput. Graph. Tech. 6(1), 2017).
template <typename T>
__device__ __forceinline__ void orthonormal_frame(const T n[3], T e1[3], T e2[3])
{
    const T sg = n[2] >= T(0) ? T(1) : T(-1);
    const T a = T(-1) / (sg + n[2]);
    const T b = n[0] * n[1] * a;
    e1[0] = T(1) + sg * n[0] * n[0] * a; e1[1] = sg * b; e1[2] = -sg * n[0];
    e2[0] = b; e2[1] = sg + n[1] * n[1] * a; e2[2] = -n[1];
}

// ---------------------------------------------------------------------------
// Rate functions (Appendix B): for sigma-bar = sigma0 (v/c)^n,
//   A = alpha_n/3 vs^{n+1} 1F1(-(n+1)/2, 5/2, -x),
//   B = alpha_n   vs^{n+3} 1F1(-(n+3)/2, 3/2, -x),  x = w^2/(2 vs^2).
// Here FA, FB are the two 1F1 values.  Large x: erf/exp closed forms of the
// 1F1 for integer n; x < 1: their Taylor series (the closed forms cancel).
template <int N>
struct RateCoef {
    static constexpr int kTerms = 24;
    double ca[kTerms], cb[kTerms];
    constexpr RateCoef() : ca(), cb()
    {
        double a1 = -(N + 1) * 0.5, b1 = 2.5, a2 = -(N + 3) * 0.5, b2 = 1.5;
        double t1 = 1.0, t2 = 1.0;
        for (int k = 0; k < kTerms; ++k) {
            ca[k] = t1;
            cb[k] = t2;
            t1 *= -(a1 + k) / ((b1 + k) * (k + 1));
            t2 *= -(a2 + k) / ((b2 + k) * (k + 1));
        }
    }
};

// Taylor terms for x < 1: binary64 keeps 22; binary32 keeps the fewest whose
// tail (the series alternate) stays below 3e-8 of the value at x = 1.
template <typename T> struct RealTraits;
template <> struct RealTraits<float> {
    template <int N> static constexpr int taylor() { return N == -4 ? 11 : (N == -2 ? 9 : 8); }
};
template <> struct RealTraits<double> {
    template <int N> static constexpr int taylor() { return 22; }
};

__device__ __forceinline__ float erf_real(float x) { return erff(x); }

// erf(t) for t >= 1 in binary32, given e = e^{-t^2}: erf = 1 - e R(t) with
// R(t) = e^{t^2} erfc(t), an entire function, as a degree-12 polynomial in
// t - 2.75 (weighted least-squares fit for relative error on [1, 4.5]; Horner
// in binary32 keeps R within 1.5e-7).  Past t = 4.5, e R < 2^-28 and R(4.5)
// stands in.  Sharing e with the caller saves erf its own exponential.
__device__ __forceinline__ float erf_ge1(float t, float e)
{
    constexpr float c[13] = {1.936620921e-01f, -6.323760748e-02f, 1.975860447e-02f, -5.934607703e-03f,
                             1.719569904e-03f, -4.814862041e-04f, 1.311259839e-04f, -3.548420500e-05f,
                             9.050128938e-06f, -1.834100885e-06f, 4.788607271e-07f, -2.315289720e-07f,
                             5.124300273e-08f};
    const float z = fminf(t, 4.5f) - 2.75f;
    float R = c[12];
#pragma unroll
    for (int k = 11; k >= 0; --k) R = fmaf(R, z, c[k]);
    return fmaf(-e, R, 1.0f);
}
__device__ __forceinline__ double erf_real(double x) { return erf(x); }
__device__ __forceinline__ float exp_neg(float x) { return __expf(-x); }
__device__ __forceinline__ double exp_neg(double x) { return exp(-x); }

template <int N, typename T>
__device__ __forceinline__ void rate_1f1_small(T x, T* FA, T* FB)      // x < 1: Taylor series
{
    constexpr RateCoef<N> C{};
    constexpr int K = RealTraits<T>::template taylor<N>();
    T fa = T(C.ca[K - 1]), fb = T(C.cb[K - 1]);
#pragma unroll
    for (int k = K - 2; k >= 0; --k) {
        fa = fa * x + T(C.ca[k]);
        fb = fb * x + T(C.cb[k]);
    }
    *FA = fa;
    *FB = fb;
}

template <int N, typename T>
__device__ __forceinline__ void rate_1f1_large(T x, T* FA, T* FB)      // x >= 1: closed forms
{
    T t, r, it;
    if constexpr (sizeof(T) == 4) {
        it = __builtin_amdgcn_rsqf(x);   // x >= 1 here
        t = x * it;
        r = it * it;
    } else {
        t = sqrt_real(x);
        r = T(1) / x;
        it = T(1) / t;
    }
    const T ex = exp_neg(x);
    T E;
    if constexpr (sizeof(T) == 4) E = erf_ge1(t, ex);
    else E = erf_real(t);
    T spE = T(kSqrtPi) * E;
    if constexpr (N == 0) {
        *FA = T(3.0 / 32.0) * (spE * (T(4) * x + T(4) - r) * it + T(2) * (T(2) + r) * ex);
        *FB = (spE * ((T(4) * x + T(12)) * x + T(3)) * it + T(2) * (T(2) * x + T(5)) * ex) * T(1.0 / 16.0);
    } else if constexpr (N == -2) {
        *FA = T(0.75) * ex * r + T(0.75) * spE * it - T(0.375) * spE * r * it;
        *FB = T(0.5) * spE * t + T(0.5) * ex + T(0.25) * spE * it;
    } else if constexpr (N == -4) {
        *FA = T(-1.5) * ex * r + T(0.75) * spE * r * it;
        *FB = T(0.5) * spE * it;
    } else if constexpr (N == 2) {
        *FA = (spE * (((T(8) * x + T(36)) * x + T(18)) * x - T(3)) * it + T(2) * ((T(4) * x + T(16)) * x + T(3)) * ex) *
              (r * T(1.0 / 64.0));
        *FB = (spE * (((T(8) * x + T(60)) * x + T(90)) * x + T(15)) * it + T(2) * ((T(4) * x + T(28)) * x + T(33)) * ex) *
              T(1.0 / 96.0);
    }
}

template <int N, typename T>
__device__ __forceinline__ void rate_1f1(T x, T* FA, T* FB)
{
    if (x < T(1)) rate_1f1_small<N, T>(x, FA, FB);
    else rate_1f1_large<N, T>(x, FA, FB);
}

// Rate integrals by quadrature (for any momentum-transfer cross section;
// used here for sigma-bar = sigma0 (v/c)^n).  With s = u/vs and x = w/vs,
// integrating eq. scrA / scrB over directions of u about w gives
//   A / vs^{n+1} = sqrt(2/pi) (1/x) int_0^inf s^{4+n} e^{-(s^2+x^2)/2} j(s x) ds,
//   B / vs^{n+3} = sqrt(2/pi)       int_0^inf s^{5+n} e^{-(s^2+x^2)/2} sinh(s x)/(s x) ds,
// j(k) = cosh k / k - sinh k / k^2.  The Gaussian factors are formed as
// e^{-(s -+ x)^2/2} (no overflow) and small k uses the Taylor series of j(k)/k
// and sinh(k)/k.  K-node Gauss-Legendre on [max(0, x - hw), max(x + hw, bmin)]
// (hw = 8.5, bmin = 11 reach 1e-10 at K = 32; hw = 5.5, bmin = 7 reach 1e-3
// at K = 12).  Returns the values divided by alpha_n/3 and alpha_n, i.e. in
// the same normalisation as the 1F1 forms of rate_1f1.
template <int N> struct Pow {
    template <typename T> __device__ static __forceinline__ T of(T s)
    {
        if constexpr (N == 0) return T(1);
        else if constexpr (N > 0) return s * Pow<N - 1>::of(s);
        else return T(1) / Pow<-N>::of(s);
    }
};

template <typename T> struct QuadTraits;
template <> struct QuadTraits<float> { static constexpr float kSmall = 0.5f; };
template <> struct QuadTraits<double> { static constexpr double kSmall = 0.1; };

template <int N, typename Real>
__device__ __forceinline__ void rate_quad(Real x, const Real* __restrict__ gx, const Real* __restrict__ gw, int K,
                                          Real inv_alpha, Real hw, Real bmin, Real* FA, Real* FB)
{
    const Real a = x > hw ? x - hw : Real(0);
    const Real b = x + hw > bmin ? x + hw : bmin;
    const Real mid = Real(0.5) * (a + b), half = Real(0.5) * (b - a);
    Real accA = 0, accB = 0;
    for (int q = 0; q < K; ++q) {
        const Real s = mid + half * gx[q];
        const Real k = s * x, k2 = k * k;
        Real jx, es;
        if (k < QuadTraits<Real>::kSmall) {
            const Real e0 = exp_neg(Real(0.5) * (s * s + x * x));
            jx = e0 * s * (Real(1.0 / 3.0) + k2 * (Real(1.0 / 30.0) + k2 * (Real(1.0 / 840.0) + k2 * Real(1.0 / 45360.0))));
            es = e0 * (Real(1) + k2 * (Real(1.0 / 6.0) + k2 * (Real(1.0 / 120.0) + k2 * (Real(1.0 / 5040.0) + k2 * Real(1.0 / 362880.0)))));
        } else {
            const Real g1 = exp_neg(Real(0.5) * (s - x) * (s - x)), g2 = exp_neg(Real(0.5) * (s + x) * (s + x));
            const Real c = Real(0.5) * (g1 + g2), sh = Real(0.5) * (g1 - g2), ik = rcp_real(k);
            jx = (c - sh * ik) * ik * rcp_real(x);
            es = sh * ik;
        }
        const Real p4 = Pow<4 + N>::of(s);
        accA += gw[q] * p4 * jx;
        accB += gw[q] * p4 * s * es;
    }
    const Real c0 = Real(0.79788456080286535588) * half;   // sqrt(2/pi)
    *FA = c0 * accA * Real(3) * inv_alpha;
    *FB = c0 * accB * inv_alpha;
}

// v^{n+1} for the scattering probability P = K g v^{n+1} dt.
template <int N, typename T>
__device__ __forceinline__ T pow_np1(T v)
{
    if constexpr (N == 0) return v;
    else if constexpr (N == -2) return rcp_real(v);
    else if constexpr (N == -4) { T iv = rcp_real(v); return iv * iv * iv; }
    else if constexpr (N == 2) return v * v * v;
    else return T(0);
}

}  // namespace dmb
