// k_interp.hip -- the G-Interp predictor-quantiser (compression) and its
// replay (decompression) on gfx950 (Sec. V-A, V-B, V-D; Sec. III-A).
//
// One wave64 per window, kWaves windows per workgroup.  A window owns the
// points [lo, lo + W) of each dimension; its block adds the far faces
// (lo + W), which the next window owns.  Neighbours are searched inside the
// point's own window interval along the pass dimension only, so a face point
// is computed identically by both windows that hold it and windows are
// independent.  A wave stages its block in LDS, runs the passes (levels from
// stride S/2 down to 1, one pass per dimension in the planned order) without
// any workgroup barrier, and writes out the points it owns.  The block of
// the wave's next window is loaded into registers while the current one is
// processed.
//
// A pass along dimension d at stride s works on lines: block points that
// share every coordinate but d.  The targets of a line are its odd multiples
// of s, its knowns the even ones.  A lane takes K consecutive targets of one
// line, reads the K + 3 knowns around them once, and predicts all K; every
// LDS offset along the line is a compile-time constant.
//
// Arithmetic: every FP32 expression is evaluated in the order written, one
// rounding per operation (the library is built with -ffp-contract=off).
#include "dev_common.h"

#include <type_traits>

namespace szi {

constexpr int kWaves = kWinPerGroup;    // windows in flight per workgroup, one per wave
static_assert(kWaves * 64 == kThreads, "one wave per window of a group");
constexpr int kPad = 8;                 // guard floats on both sides of a block in LDS
constexpr int kXcds = 8;                // L2 domains; workgroup i runs on domain i % kXcds

template <int ND>
constexpr int vlen() { return kPad + Geo<ND>::BN + kPad; }

// The window a wave works on.  Every member is wave-uniform.
struct Win {
    uint64_t gbase;          // linear index of the window origin
    uint32_t n0, n01;        // field strides
    int lo0, lo1, lo2;       // origin
    int e0, e1, e2;          // block extents (owned points + far face where present)
    uint32_t op;             // owned extents o0 | o1 << 8 | o2 << 16 (each at most 64)
    bool full;
    __device__ int own(int d) const { return (int)((op >> (8 * d)) & 255u); }
};

template <int ND>
__device__ __forceinline__ Win make_win(const FieldDesc& f, uint32_t w) {
    using G = Geo<ND>;
    Win wi;
    const uint32_t nw0 = (uint32_t)f.nwin[0];
    const uint32_t nw01 = nw0 * (uint32_t)f.nwin[1];
    // w / nw01 and r / nw0: the product with floor(2^32 / m) is the
    // quotient or one less
    uint32_t wz = __umulhi(w, f.wmag[1]), r = w - wz * nw01;
    if (r >= nw01) {
        ++wz;
        r -= nw01;
    }
    uint32_t wy = __umulhi(r, f.wmag[0]), wx = r - wy * nw0;
    if (wx >= nw0) {
        ++wy;
        wx -= nw0;
    }
    wi.n0 = (uint32_t)f.n[0];
    wi.n01 = wi.n0 * (uint32_t)f.n[1];
    wi.lo0 = (int)wx * G::W0;
    wi.lo1 = (int)wy * G::W1;
    wi.lo2 = ND == 3 ? (int)wz * G::W2 : 0;
    const int s0 = f.n[0] - 1 - wi.lo0, s1 = f.n[1] - 1 - wi.lo1;
    const int s2 = ND == 3 ? f.n[2] - 1 - wi.lo2 : 0;
    wi.e0 = (s0 < G::W0 ? s0 : G::W0) + 1;
    wi.e1 = (s1 < G::W1 ? s1 : G::W1) + 1;
    wi.e2 = ND == 3 ? (s2 < G::W2 ? s2 : G::W2) + 1 : 1;
    const int o0 = wi.e0 < G::W0 ? wi.e0 : G::W0;
    const int o1 = wi.e1 < G::W1 ? wi.e1 : G::W1;
    const int o2 = ND == 3 ? (wi.e2 < G::W2 ? wi.e2 : G::W2) : 1;
    static_assert(G::W0 < 256 && G::W1 < 256 && G::W2 < 256, "owned extents fit 8 bits");
    wi.op = (uint32_t)o0 | ((uint32_t)o1 << 8) | ((uint32_t)o2 << 16);
    wi.full = wi.e0 == G::B0 && wi.e1 == G::B1 && (ND == 2 || wi.e2 == G::B2);
    wi.gbase = (uint64_t)wi.lo0 + (uint64_t)wi.lo1 * wi.n0 + (uint64_t)wi.lo2 * wi.n01;
    return wi;
}

// byte offset from a window origin: the 64-bit base stays in scalar
// registers and the per-lane part is a 32-bit offset (the host bounds the
// span of a window below 4 GiB)
template <class T>
__device__ __forceinline__ const SZI_G T* at(const SZI_G T* base, uint32_t off) {
    return (const SZI_G T*)((const SZI_G char*)base + (off * (uint32_t)sizeof(T)));
}
template <class T>
__device__ __forceinline__ SZI_G T* at(SZI_G T* base, uint32_t off) {
    return (SZI_G T*)((SZI_G char*)base + (off * (uint32_t)sizeof(T)));
}

// ------------------------------------------------------------ block staging
// Slots of the replay's code load, NPRE per lane; slot k of a lane is a (global
// offset from the window origin, LDS index) pair and whether the lane holds
// a point of the block there (of its in-extent part, for partial windows).
// 3D: slots 0-35 hold rows (y, z) and (y, z + 4) of planes 0-7 (lanes 0-31
// and 32-63, x = lane % 32), slots 36-40 rows (y, 8) and (y + 5, 8), slots
// 41-42 the x = 32 column (row = lane and lane + 64).  2D: slots 0-16 rows
// y (x = lane), slot 17 the x = 64 column (row = lane).
template <int ND>
struct LaneMap;

template <>
struct LaneMap<3> {
    uint32_t x, hi;
    uint32_t gA, gB, gC0, gC1;   // per-lane global offsets
    int yc0, zc0, yc1, zc1;      // column rows
    __device__ __forceinline__ void init(uint32_t lane, uint32_t n0, uint32_t n01) {
        x = lane & 31u;
        hi = lane >> 5;
        gA = x + hi * 4u * n01;
        gB = x + hi * 5u * n0;
        yc0 = (int)(lane % 9u);
        zc0 = (int)(lane / 9u);
        yc1 = (int)((lane + 64u) % 9u);
        zc1 = (int)((lane + 64u) / 9u);
        gC0 = 32u + (uint32_t)yc0 * n0 + (uint32_t)zc0 * n01;
        gC1 = 32u + (uint32_t)yc1 * n0 + (uint32_t)zc1 * n01;
    }
    template <bool FULL>
    __device__ __forceinline__ bool slot(int k, const Win& wi, uint32_t& g, int& l) const {
        if (k < 36) {
            const int zl = k / 9, y = k % 9;
            g = (uint32_t)y * wi.n0 + (uint32_t)zl * wi.n01 + gA;
            l = zl * 297 + y * 33 + (int)x + (int)hi * (4 * 297);
            return FULL || ((int)x < wi.e0 && y < wi.e1 && zl + 4 * (int)hi < wi.e2);
        } else if (k < 41) {
            const int p = k - 36;
            g = (uint32_t)p * wi.n0 + 8u * wi.n01 + gB;
            l = 8 * 297 + p * 33 + (int)x + (int)hi * (5 * 33);
            const bool exists = p + 5 * (int)hi <= 8;
            return exists && (FULL || ((int)x < wi.e0 && p + 5 * (int)hi < wi.e1 && 8 < wi.e2));
        } else {
            const bool c1 = k == 42;
            const int r = (int)(x + 32u * hi) + (c1 ? 64 : 0);
            g = c1 ? gC1 : gC0;
            l = 32 + 33 * r;
            const int y = c1 ? yc1 : yc0, z = c1 ? zc1 : zc0;
            return r < 81 && (FULL || (32 < wi.e0 && y < wi.e1 && z < wi.e2));
        }
    }
};

template <>
struct LaneMap<2> {
    uint32_t x;
    uint32_t gC;
    __device__ __forceinline__ void init(uint32_t lane, uint32_t n0, uint32_t) {
        x = lane;
        gC = 64u + lane * n0;
    }
    template <bool FULL>
    __device__ __forceinline__ bool slot(int k, const Win& wi, uint32_t& g, int& l) const {
        if (k < 17) {
            g = (uint32_t)k * wi.n0 + x;
            l = k * 65 + (int)x;
            return FULL || ((int)x < wi.e0 && k < wi.e1);
        }
        g = gC;
        l = 64 + 65 * (int)x;
        return x < 17u && (FULL || (64 < wi.e0 && (int)x < wi.e1));
    }
};

// 16-byte staging of the FP32 block (rows at any float's address): lane =
// (quad q of x, row).  3D: slots 0-8 hold planes z = 0-8 at rows y = lane /
// 8, slot 9 rows y = 8 of planes lane / 8, slot 10 row (8, 8); then the x =
// 32 column in two scalar slots.  2D: slots 0-4 rows 4k + lane / 16, then
// the x = 64 column.  NQ quads and NC column values per lane, the quads
// first in the register array.
template <int ND>
struct QuadMap;

template <>
struct QuadMap<3> {
    static constexpr int NQ = 11, NC = 2, N = 4 * NQ + NC;
    uint32_t gq, gy8, gc0, gc1;   // per-lane global offsets
    int lq, ly8;                  // per-lane LDS offsets
    bool c1v;
    __device__ __forceinline__ void init(uint32_t lane, uint32_t n0, uint32_t n01) {
        const uint32_t q = lane & 7u, r = lane >> 3;
        gq = 4u * q + r * n0;
        lq = 4 * (int)q + 33 * (int)r;
        gy8 = 4u * q + 8u * n0 + r * n01;
        ly8 = 4 * (int)q + 8 * 33 + 297 * (int)r;
        gc0 = 32u + (lane % 9u) * n0 + (lane / 9u) * n01;
        gc1 = 32u + ((lane + 64u) % 9u) * n0 + ((lane + 64u) / 9u) * n01;
        c1v = lane + 64u < 81u;
    }
    // quad slot k: global offset and LDS index of its first value
    __device__ __forceinline__ bool quad(int k, uint32_t lane, uint32_t n01, uint32_t& g,
                                         int& l) const {
        if (k < 9) {
            g = gq + (uint32_t)k * n01;
            l = lq + 297 * k;
            return true;
        }
        if (k == 9) {
            g = gy8;
            l = ly8;
            return true;
        }
        g = gy8 + 8u * n01 - (lane >> 3) * n01;   // row (8, 8)
        l = 4 * (int)(lane & 7u) + 8 * 33 + 8 * 297;
        return lane < 8u;
    }
    // values of quad slot k inside a partial window's block
    __device__ __forceinline__ int inside(int k, uint32_t lane, const Win& wi) const {
        const int r = (int)(lane >> 3);
        const int y = k < 9 ? r : 8, z = k < 9 ? k : (k == 9 ? r : 8);
        return y < wi.e1 && z < wi.e2 ? wi.e0 - 4 * (int)(lane & 7u) : 0;
    }
    __device__ __forceinline__ bool col(int k, uint32_t lane, uint32_t& g, int& l) const {
        g = k == 0 ? gc0 : gc1;
        l = 32 + 33 * ((int)lane + 64 * k);
        return k == 0 || c1v;
    }
    __device__ __forceinline__ bool col_inside(int k, uint32_t lane, const Win& wi) const {
        const uint32_t r = lane + 64u * (uint32_t)k;
        return 32 < wi.e0 && (int)(r % 9u) < wi.e1 && (int)(r / 9u) < wi.e2;
    }
};

template <>
struct QuadMap<2> {
    static constexpr int NQ = 5, NC = 1, N = 4 * NQ + NC;
    uint32_t gq, gc0, n0;
    int lq;
    uint32_t r;
    __device__ __forceinline__ void init(uint32_t lane, uint32_t nn0, uint32_t) {
        const uint32_t q = lane & 15u;
        r = lane >> 4;
        n0 = nn0;
        gq = 4u * q + r * nn0;
        lq = 4 * (int)q + 65 * (int)r;
        gc0 = 64u + lane * nn0;
    }
    __device__ __forceinline__ bool quad(int k, uint32_t lane, uint32_t, uint32_t& g,
                                         int& l) const {
        g = gq + (uint32_t)(4 * k) * n0;
        l = lq + 65 * 4 * k;
        return 4 * k + (int)r < 17;
    }
    __device__ __forceinline__ int inside(int k, uint32_t lane, const Win& wi) const {
        return 4 * k + (int)r < wi.e1 ? wi.e0 - 4 * (int)(lane & 15u) : 0;
    }
    __device__ __forceinline__ bool col(int, uint32_t lane, uint32_t& g, int& l) const {
        g = gc0;
        l = 64 + 65 * (int)lane;
        return lane < 17u;
    }
    __device__ __forceinline__ bool col_inside(int, uint32_t lane, const Win& wi) const {
        return 64 < wi.e0 && (int)lane < wi.e1;
    }
};

// FULL: the whole block lies in the field; else quads that cross its end
// load the values inside it one by one, the others hold zeros
template <int ND, bool FULL>
__device__ __forceinline__ void load_quads(float* pre, const SZI_G float* wb, const QuadMap<ND>& qm,
                                           uint32_t lane, const Win& wi) {
    using Q = QuadMap<ND>;
#pragma unroll
    for (int k = 0; k < Q::NQ; ++k) {
        uint32_t g;
        int l;
        vf4 t = {0.0f, 0.0f, 0.0f, 0.0f};
        const bool slot = qm.quad(k, lane, wi.n01, g, l);
        const int in = FULL ? 4 : (slot ? qm.inside(k, lane, wi) : 0);
        if (FULL ? slot : in >= 4) t = *(const SZI_G vf4a4*)at(wb, g);
        if (!FULL && in > 0 && in < 4) {
            t.x = *at(wb, g);
            if (in > 1) t.y = *at(wb, g + 1u);
            if (in > 2) t.z = *at(wb, g + 2u);
        }
        pre[4 * k] = t.x;
        pre[4 * k + 1] = t.y;
        pre[4 * k + 2] = t.z;
        pre[4 * k + 3] = t.w;
    }
#pragma unroll
    for (int k = 0; k < Q::NC; ++k) {
        uint32_t g;
        int l;
        float t = 0.0f;
        if (qm.col(k, lane, g, l) && (FULL || qm.col_inside(k, lane, wi))) t = *at(wb, g);
        pre[4 * Q::NQ + k] = t;
    }
}

template <int ND>
__device__ __forceinline__ void commit_quads(float* v, const float* pre, const QuadMap<ND>& qm,
                                             uint32_t lane, uint32_t n01) {
    using Q = QuadMap<ND>;
#pragma unroll
    for (int k = 0; k < Q::NQ; ++k) {
        uint32_t g;
        int l;
        if (qm.quad(k, lane, n01, g, l)) {
            v[l] = pre[4 * k];
            v[l + 1] = pre[4 * k + 1];
            v[l + 2] = pre[4 * k + 2];
            v[l + 3] = pre[4 * k + 3];
        }
    }
#pragma unroll
    for (int k = 0; k < Q::NC; ++k) {
        uint32_t g;
        int l;
        if (qm.col(k, lane, g, l)) v[l] = pre[4 * Q::NQ + k];
    }
}

// Slots a lane does not load keep the value fill.
template <int ND, bool FULL, class T, class U>
__device__ __forceinline__ void load_block(U* pre, const SZI_G T* wb, const LaneMap<ND>& lm,
                                           const Win& wi, U fill) {
#pragma unroll
    for (int k = 0; k < Geo<ND>::NPRE; ++k) {
        uint32_t g;
        int l;
        U t = fill;
        if (lm.template slot<FULL>(k, wi, g, l)) t = (U)*at(wb, g);
        pre[k] = t;
    }
}

// anchors of the block (Sec. V-A: stored losslessly), one per lane
template <int ND>
__device__ __forceinline__ bool anchor_slot(uint32_t lane, const FieldDesc& f, const Win& wi,
                                            uint32_t& gi, int& li) {
    using G = Geo<ND>;
    constexpr int S = 1 << G::SHS;
    const int ax = (int)(lane % 5u);
    const int ay = ND == 3 ? (int)((lane / 5u) & 1u) : (int)(lane / 5u);
    const int az = ND == 3 ? (int)(lane / 10u) : 0;
    li = ax * S + ay * S * G::SY + az * S * G::SZ;
    gi = (uint32_t)((wi.lo0 >> G::SHS) + ax) +
         (uint32_t)f.na[0] * ((uint32_t)((wi.lo1 >> G::SHS) + ay) +
                              (uint32_t)f.na[1] * (uint32_t)((wi.lo2 >> G::SHS) + az));
    return lane < (uint32_t)G::NANCH && ax * S < wi.e0 && ay * S < wi.e1 && az * S < wi.e2;
}

// ------------------------------------------------------------------ passes
// Division by 40 in the natural cubic, as a multiply by RN(1/40) followed
// by one fused multiply-add correction (Brisebarre, Muller and Raina,
// "Accelerating correctly rounded floating-point division when the divisor
// is known in advance", IEEE Trans. Computers 53(8), 2004).  Checked
// exhaustively over all FP32 inputs: equal to the correctly rounded x / 40
// for 2^-123 <= |x| < inf.  Smaller numerators (zeros included) take the
// division.  An infinite numerator gives NaN instead of an infinity; both
// make the point an outlier (the quantiser's range test fails on either),
// so compression and replay are unchanged.
__device__ __forceinline__ float div40_fast(float x) {
    const float c = 0.025f;
    const float q0 = x * c;
    const float r = fmaf(-q0, 40.0f, x);
    return fmaf(r, c, q0);
}

// Sec. V-B.1 splines by neighbour availability (a = x[-3s], b = x[-s],
// c = x[+s], d = x[+3s]); with one neighbour the value of x[-s].  num
// receives the natural cubic's numerator where that cubic gives the
// prediction, else 1 (a value the fast division handles).  The stencil is
// picked by selects, not branches: where the flags are compile-time
// constants only the chosen formula remains, elsewhere the wave computes
// the candidates and keeps one per lane.
template <int SPL>
__device__ __forceinline__ float predict(bool m3, bool p1, bool p3, float a, float b, float c,
                                         float d, float& num) {
    const float sbc = b + c;
    float p = sbc * 0.5f;   // linear
    num = 1.0f;
    if (SPL != SPL_LIN) {
        const float ql = ((6.0f * b + 3.0f * c) - a) * 0.125f;   // quadratic on a, b, c
        const float qr = ((3.0f * b + 6.0f * c) - d) * 0.125f;   // quadratic on b, c, d
        float cu;
        if (SPL == SPL_NAT) {
            const float n = 23.0f * sbc - 3.0f * (a + d);       // natural cubic, / 40
            cu = div40_fast(n);
            num = m3 && p3 && p1 ? n : 1.0f;
        } else {
            cu = (9.0f * sbc - (a + d)) * 0.0625f;              // not-a-knot cubic
        }
        p = m3 ? (p3 ? cu : ql) : (p3 ? qr : p);
    }
    return p1 ? p : b;
}

// Natural cubics whose numerators lie below the fast division's range (a
// NaN passes the minimum by: either division keeps it a NaN): rare, so one
// test for all targets of all lanes.
template <int K>
__device__ __forceinline__ void divide_small(float (&pr)[K], const float (&nm)[K]) {
    float least = fabsf(nm[0]);
#pragma unroll
    for (int j = 1; j < K; ++j) least = fminf(least, fabsf(nm[j]));
    if (wave_any(!(least >= 0x1p-123f))) {
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (!(fabsf(nm[j]) >= 0x1p-123f)) pr[j] = nm[j] / 40.0f;
    }
}

// Closed-loop quantisation of K targets of a lane against e_l (Sec. III-A):
// reconstructed values xr and codes cd from predictions pr and originals
// xv.  With e_l = 0, inv = 0 gives q = 0 and xr = p + 0, so only exact
// predictions pass the bound test.  |rint(qf)| < R holds iff |qf| < R and
// |q| < R; NaN fails it.  The FP64 bound test |x - xr| <= e_l is decided in
// FP32 where the rounded difference is below e_l (then so is the exact one),
// in FP64 otherwise.  One test of the largest |q| and |x - xr| of all
// targets of all lanes (in[j] false: a target outside the field, left out)
// decides whether any target has to be looked at by itself.
template <int K>
__device__ __forceinline__ void quantise(const float (&pr)[K], const float (&xv)[K],
                                         const bool (&in)[K], float el, float ebx2, float inv,
                                         int R, float (&xr)[K], uint32_t (&cd)[K]) {
    const float Rf = (float)R;
    float qr[K], dm = 0.0f, qm = 0.0f;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        qr[j] = rintf((xv[j] - pr[j]) * inv);   // round half to even
        xr[j] = pr[j] + qr[j] * ebx2;           // (float)(int)q == q in range
        // this maximum keeps a NaN (a prediction past the largest float)
        qm = __builtin_elementwise_maximum(qm, in[j] ? fabsf(qr[j]) : 0.0f);
        dm = __builtin_elementwise_maximum(dm, in[j] ? fabsf(xv[j] - xr[j]) : 0.0f);
        cd[j] = (uint32_t)((int)qr[j] + R);
    }
    if (wave_any(!(dm < el && qm < Rf))) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            // (no short-circuits: selects only, no nested branches)
            const bool inr = fabsf(qr[j]) < Rf;
            const bool in32 = fabsf(xv[j] - xr[j]) < el;
            const bool in64 = fabs((double)xv[j] - (double)xr[j]) <= (double)el;
            const bool good = inr & (in32 | in64);
            xr[j] = good ? xr[j] : xv[j];
            cd[j] = good ? cd[j] : 0u;
        }
    }
}

// Makes the compiler wait here for loads into these registers, so that it
// places no wait for them further on (where it would also hold for every
// store and load issued since).
template <class T, int N>
__device__ __forceinline__ void settle(T (&r)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : "+v"(r[k]));
}

// A pass's descriptor in scalar registers, from the wave's register that
// holds the passes of its field a word a lane (a scalar load per pass would
// cost its latency nine times a window).
struct Pass {
    uint32_t kind, lines, magic;
    float el, ebx2, inv;
};
__device__ __forceinline__ Pass get_pass(uint32_t words, int np) {
    const int l = np * kPassWords;
    auto rd = [&](int i) SZI_INLINE { return (uint32_t)__builtin_amdgcn_readlane((int)words, l + i); };
    return Pass{rd(0), rd(1), rd(2), __uint_as_float(rd(3)), __uint_as_float(rd(4)), __uint_as_float(rd(5))};
}
__device__ __forceinline__ uint32_t load_passes(const FieldPlan& p, uint32_t lane) {
    uint32_t w[1] = {gp(reinterpret_cast<const uint32_t*>(p.pass))[lane]};
    settle(w);
    return w[0];
}

// LDS values of one task: K targets of one line (segment seg, starting at
// LDS index base), the K + 3 knowns around them and the targets' original
// values (compression) or quant-codes (decompression).
template <int K>
struct Task {
    int base;       // LDS index of the segment start
    uint32_t gl;    // compression: its global offset from the window origin
    uint32_t t;     // the task's number
    bool own;       // the line lies in the window's owned part (compression)
    float kn[K + 3];
    float xt[K];
    uint32_t ct[K];
};

// Where a pass leaves its results besides the block: compression stores
// the quant-code of every owned target in the codes array and counts it in
// the histogram; the replay finds outliers' values in the output array.
struct PassOut {
    SZI_G uint16_t* cb;       // the window's codes (compression)
    const SZI_G float* ob;    // the window's output values (replay)
    uint32_t* hist;           // LDS histogram (compression)
};

// a * b modulo 2^32 for a < 2^16, from 24-bit multiplies (full rate; a
// 32-bit multiply issues at a quarter of it), the halves of b uniform (the
// empty asm keeps the compiler from joining them to the 32-bit product)
__device__ __forceinline__ uint32_t mul16x32(uint32_t a, uint32_t b) {
    uint32_t hi = __umul24(a, b >> 16);
    asm("" : "+v"(hi));
    return __umul24(a, b & 0xFFFFu) + (hi << 16);
}

// Targets per task: a lane reads K + 3 knowns for K targets, so long tasks
// save LDS reads and task set-up where a pass has many lines (stride 1),
// and short ones fill the wave where it has few: at the coarse strides a
// pass has less than a wave of targets, and each task's time is its K
// predictions one after another.  At stride 1 four; in 2D compression two
// (24 climate fields: interpolation 349 us against 391-402 with four and 413
// with eight along y; the replay 301 with four against 317 and 357; in 3D
// two take 337 and 268 us at 512^3 against 330 and 246).
template <int ND, bool COMP, int T, int SH>
constexpr int task_targets() {
    constexpr int most = SH == 0 ? (ND == 2 && COMP ? 2 : 4) : (SH == 1 ? 2 : 1);
    return T < most ? T : most;
}

// One pass: dimension D, stride s = 1 << SH, spline SPL.  FULL: the window
// interval along D is the whole block, so the stencil flags are constants
// (in whole lines) or follow from the segment.  store: the pass's values
// are read by a later one (compression only; the last pass's are not).
// Tasks are software-pipelined: the LDS reads of a lane's next task are
// issued before the current one is computed.  Within a pass no task reads a
// point another task writes (targets never neighbour each other along D and
// knowns are not written), so the reordering is safe.
//
// The block holds a value at every known point.  In the replay a point not
// yet reconstructed holds its quant-code instead (as the bits of the
// float), which the pass reading it as a target replaces by the value.
//
// Bound by instruction issue (about 2000 vector and 1200 scalar
// instructions a 3D window), so the common case is kept short: one test per
// task decides whether every target of every lane is in range and inside
// the bound in FP32; only otherwise are outliers and the FP64 test looked
// at target by target.
template <int ND, int D, int SH, int SPL, bool COMP, bool FULL>
__device__ __forceinline__ void pass_lines(float* v, uint32_t lane, const Pass& pd,
                                           const Win& wi, int ed, int R, const PassOut& po,
                                           bool store) {
    using G = Geo<ND>;
    constexpr int s = 1 << SH;
    constexpr int W = D == 0 ? G::W0 : (D == 1 ? G::W1 : G::W2);
    constexpr int SD = D == 0 ? 1 : (D == 1 ? G::SY : G::SZ);
    constexpr int T = W / (2 * s);   // targets per line
    constexpr int K = task_targets<ND, COMP, T, SH>();
    constexpr int NSEG = T / K;
    static_assert(NSEG * K == T && (NSEG & (NSEG - 1)) == 0, "whole power-of-two segments");
    // a split line's end segments have knowns past the line: along x at
    // small strides the guard band or the next row absorbs the read, else
    // it is moved onto the line (the flags drop the value either way)
    constexpr bool kGuard = D == 0 && 2 * s <= kPad;
    // the dimensions of the lines, e < g: LDS strides, global strides,
    // owned extents
    constexpr int DE = D == 0 ? 1 : 0, DG = D == 2 ? 1 : 2;
    constexpr uint32_t SE = DE == 0 ? 1 : G::SY, SG = DG == 1 ? G::SY : G::SZ;
    const uint32_t gse = DE == 0 ? 1u : wi.n0, gsg = DG == 1 ? wi.n0 : wi.n01;
    const uint32_t owne = (uint32_t)wi.own(DE), owng = (uint32_t)wi.own(DG);
    const uint32_t ne = pd.lines >> 16, magic = pd.magic;
    const uint32_t she = (pd.kind >> 4) & 15u, shg = (pd.kind >> 8) & 15u;
    const uint32_t ntask = (pd.lines & 0xFFFFu) * (uint32_t)NSEG;
    const float ebx2 = pd.ebx2, inv = pd.inv;
    const float el = pd.el;
    const uint32_t gsd = D == 0 ? 1u : (D == 1 ? wi.n0 : wi.n01);   // global stride along D

    auto seg_of = [&](uint32_t t) SZI_INLINE { return NSEG > 1 ? (t & (uint32_t)(NSEG - 1)) : 0u; };
    // coordinates of a task's line along e and g
    auto line_of = [&](uint32_t t, uint32_t& ce, uint32_t& cg) SZI_INLINE {
        const uint32_t ln = t / (uint32_t)NSEG;
        const uint32_t i1 = ND == 2 ? 0u : __umul24(ln, magic) >> 16;   // ln / ne
        ce = (ND == 2 ? ln : ln - __umul24(i1, ne)) << she;
        cg = i1 << shg;
    };
    // global offset of the segment start from the window origin
    auto global_of = [&](uint32_t ce, uint32_t cg, uint32_t seg) SZI_INLINE {
        uint32_t g = seg * (uint32_t)(2 * K * s) * gsd + (DE == 0 ? ce : mul16x32(ce, gse));
        if (ND == 3) g += mul16x32(cg, gsg);
        return g;
    };

    auto fetch = [&](uint32_t t, Task<K>& tk) SZI_INLINE {
        uint32_t ce, cg;
        line_of(t, ce, cg);
        const uint32_t seg = seg_of(t);
        tk.t = t;
        uint32_t base = (SE == 1 ? ce : __umul24(ce, SE)) + __umul24(seg, (uint32_t)(2 * K * s * SD));
        if (ND == 3) base += __umul24(cg, SG);
        tk.base = (int)base;
        if (COMP) {
            tk.gl = global_of(ce, cg, seg);
            tk.own = ce < owne && (ND == 2 || cg < owng);
        }
        // knowns at (2i - 2) s from the segment start; whole lines read only
        // the ones inside the block
#pragma unroll
        for (int i = 0; i < K + 3; ++i) {
            const int pos = (2 * i - 2) * s;
            if (NSEG == 1) {
                tk.kn[i] = pos >= 0 && pos <= W ? v[tk.base + pos * SD] : 0.0f;
            } else if (kGuard || (i > 0 && i < K + 2)) {
                tk.kn[i] = v[tk.base + pos * SD];
            } else {
                const bool in = i == 0 ? seg > 0u : seg < (uint32_t)(NSEG - 1);
                tk.kn[i] = v[tk.base + (in ? pos : (i == 0 ? 0 : pos - 2 * s)) * SD];
            }
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int li = tk.base + (2 * j + 1) * s * SD;
            if (COMP)
                tk.xt[j] = v[li];
            else
                tk.ct[j] = __float_as_uint(v[li]);
        }
    };

    auto compute = [&](const Task<K>& tk) SZI_INLINE {
        const uint32_t seg = seg_of(tk.t);
        const int p0 = (int)seg * (2 * K * s);   // segment start along D
        float pr[K], nm[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int pos = (2 * j + 1) * s;   // target position in the segment
            const bool m3 = NSEG > 1 ? (j >= 1 || seg > 0u) : (j >= 1);
            bool p3 = NSEG > 1 ? (j <= K - 2 || seg < (uint32_t)(NSEG - 1))
                               : ((2 * j + 4) * s <= W);
            bool p1 = true;
            if (!FULL) {   // the window interval ends at ed - 1
                p1 = p0 + pos + s <= ed - 1;
                p3 = p0 + pos + 3 * s <= ed - 1;
            }
            pr[j] = predict<SPL>(m3, p1, p3, tk.kn[j], tk.kn[j + 1], tk.kn[j + 2], tk.kn[j + 3],
                                 nm[j]);
        }
        if (SPL == SPL_NAT) divide_small<K>(pr, nm);
        float* vb = v + tk.base;
        if (COMP) {
            float xr[K];
            uint32_t cd[K];
            bool in[K];
#pragma unroll
            for (int j = 0; j < K; ++j) in[j] = FULL || p0 + (2 * j + 1) * s < ed;
            quantise<K>(pr, tk.xt, in, el, ebx2, inv, R, xr, cd);
            if (store) {
#pragma unroll
                for (int j = 0; j < K; ++j) vb[(2 * j + 1) * s * SD] = xr[j];
            }
            // owned targets: the quant-codes, and the histogram, where the
            // centre code goes to a bin of the lane's own past the 2R
            // symbols (no two lanes share an address).  The window interval
            // along D ends at ed - 1.
            if (tk.own) {
                const uint32_t rb = (uint32_t)(2 * R) + lane;
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const int pos = (2 * j + 1) * s;
                    if (FULL || p0 + pos < ed) {
                        // a uniform base per target and the lane's 32-bit offset
                        SZI_G uint16_t* cj = po.cb + (uint64_t)((uint32_t)pos * gsd);
                        *at(cj, tk.gl) = (uint16_t)cd[j];
                        atomicAdd(&po.hist[cd[j] != (uint32_t)R ? cd[j] : rb], 1u);
                    }
                }
            }
        } else {
            uint32_t least = tk.ct[0];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                pr[j] = pr[j] + (float)((int)tk.ct[j] - R) * ebx2;
                least = tk.ct[j] < least ? tk.ct[j] : least;
            }
            // code 0: an outlier, whose value the scatter step put in the
            // output array (points outside the field hold a code no point
            // takes, so the load stays inside it); rare, so one uniform test
            if (wave_any(least == 0u)) {
                uint32_t ce, cg;
                line_of(tk.t, ce, cg);
                const uint32_t gl = global_of(ce, cg, seg);
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const int pos = (2 * j + 1) * s;
                    if (tk.ct[j] == 0u) pr[j] = *at(po.ob, gl + (uint32_t)pos * gsd);
                }
                // the values are waited for in here: a wait behind the
                // branch would hold every task for the next window's loads
                // (replay 254 -> 246 us at 512^3 with it here and
                // below, the passes in a register and the shorter index sums)
                settle(pr);
            }
#pragma unroll
            for (int j = 0; j < K; ++j) vb[(2 * j + 1) * s * SD] = pr[j];
        }
    };

    // two task slots in turn, so that no values are copied between them
    uint32_t t = lane;
    if (t >= ntask) return;
    Task<K> ta, tb;
    fetch(t, ta);
#pragma unroll 1
    while (true) {
        t += 64;
        bool more = t < ntask;
        if (more) fetch(t, tb);
        compute(ta);
        if (!more) break;
        t += 64;
        more = t < ntask;
        if (more) fetch(t, ta);
        compute(tb);
        if (!more) break;
    }
}

template <int ND, int D, int SH, bool COMP>
__device__ __forceinline__ void run_pass(float* v, uint32_t lane, const Pass& pd, const Win& wi,
                                         int R, const PassOut& po, bool store) {
    using G = Geo<ND>;
    constexpr int W = D == 0 ? G::W0 : (D == 1 ? G::W1 : G::W2);
    const int ed = D == 0 ? wi.e0 : (D == 1 ? wi.e1 : wi.e2);
    const uint32_t spl = (pd.kind >> 2) & 3u;
    // the stencil flags depend on the extent along D only
    if (ed == W + 1) {
        if (spl == SPL_LIN)
            pass_lines<ND, D, SH, SPL_LIN, COMP, true>(v, lane, pd, wi, ed, R, po, store);
        else if (spl == SPL_NAT)
            pass_lines<ND, D, SH, SPL_NAT, COMP, true>(v, lane, pd, wi, ed, R, po, store);
        else
            pass_lines<ND, D, SH, SPL_NAK, COMP, true>(v, lane, pd, wi, ed, R, po, store);
    } else {
        if (spl == SPL_LIN)
            pass_lines<ND, D, SH, SPL_LIN, COMP, false>(v, lane, pd, wi, ed, R, po, store);
        else if (spl == SPL_NAT)
            pass_lines<ND, D, SH, SPL_NAT, COMP, false>(v, lane, pd, wi, ed, R, po, store);
        else
            pass_lines<ND, D, SH, SPL_NAK, COMP, false>(v, lane, pd, wi, ed, R, po, store);
    }
}

// A wave's own LDS accesses execute in program order; this keeps the
// compiler from moving them across a pass boundary.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The passes of one level (stride 1 << SH), in the planned order.
template <int ND, int SH, bool COMP>
__device__ __forceinline__ void run_level(float* v, uint32_t lane, uint32_t passes, int R,
                                          const Win& wi, const PassOut& po) {
    constexpr int L = ND == 3 ? 3 : 4;
#pragma unroll 1
    for (int k = 0; k < ND; ++k) {
        const Pass pd = get_pass(passes, (L - 1 - SH) * ND + k);
        const bool store = SH > 0 || k + 1 < ND;   // the last pass's values are read by none
        const uint32_t d = pd.kind & 3u;
        if (d == 0) run_pass<ND, 0, SH, COMP>(v, lane, pd, wi, R, po, store);
        else if (ND == 2 || d == 1) run_pass<ND, 1, SH, COMP>(v, lane, pd, wi, R, po, store);
        else if constexpr (ND == 3) run_pass<ND, 2, SH, COMP>(v, lane, pd, wi, R, po, store);
        wave_sync();
    }
}

template <int ND, bool COMP>
__device__ __forceinline__ void run_levels(float* v, uint32_t lane, uint32_t passes, int R,
                                           const Win& wi, const PassOut& po) {
    if constexpr (ND == 2) run_level<ND, 3, COMP>(v, lane, passes, R, wi, po);
    run_level<ND, 2, COMP>(v, lane, passes, R, wi, po);
    run_level<ND, 1, COMP>(v, lane, passes, R, wi, po);
    run_level<ND, 0, COMP>(v, lane, passes, R, wi, po);
}

// ---------------------------------------------------------------- write-out
// Rows of the owned part are covered in slots of RPS rows; a slot's rows
// lie in one plane.  Lane = (sub, x-group).
template <int ND, int PER_ROW>
struct OutMap {
    using G = Geo<ND>;
    static constexpr int RPS = 64 / PER_ROW;
    static constexpr int NS = G::W1 * (ND == 3 ? G::W2 : 1) / RPS;
    static constexpr int y0(int k) { return (k * RPS) % G::W1; }
    static constexpr int z0(int k) { return (k * RPS) / G::W1; }
};

// Owned anchors: x = 0, S, 2S, 3S of row 0.  Their values go to the anchor
// array (Sec. V-A: stored losslessly); their quant-code is R (counted in
// the histogram like every owned code, Sec. VI-A).  The passes store the
// codes of all other owned points.
template <int ND>
__device__ __forceinline__ void write_anchors(const float* v, uint32_t lane, const FieldDesc& f,
                                              const Win& wi, uint32_t* hist) {
    using G = Geo<ND>;
    constexpr int S = 1 << G::SHS;
    if (lane < (uint32_t)(G::W0 / S) && (int)lane * S < wi.own(0)) {
        const uint32_t ai = (uint32_t)(wi.lo0 >> G::SHS) + lane +
                            (uint32_t)f.na[0] * ((uint32_t)(wi.lo1 >> G::SHS) +
                                                 (uint32_t)f.na[1] * (uint32_t)(wi.lo2 >> G::SHS));
        gp(f.anchors)[ai] = v[(int)lane * S];
        *at(gp(f.codes) + wi.gbase, lane * (uint32_t)S) = (uint16_t)f.R;
        atomicAdd(&hist[2 * f.R + lane], 1u);   // the lane's centre-code bin
    }
}

// Owned reconstructed values.
template <int ND, bool FULL>
__device__ __forceinline__ void write_values(const float* v, uint32_t lane, const FieldDesc& f,
                                             const Win& wi) {
    using G = Geo<ND>;
    using M = OutMap<ND, G::W0 / 4>;    // x-quads
    SZI_G float* ob = gp(f.out) + wi.gbase;
    const uint32_t sub = lane / (uint32_t)(G::W0 / 4);
    const int x = 4 * (int)(lane % (uint32_t)(G::W0 / 4));
    const int lq = x + (int)sub * G::SY;
    const uint32_t gq = (uint32_t)x + sub * wi.n0;
    if (FULL) {
#pragma unroll
        for (int k = 0; k < M::NS; ++k) {
            const int l = lq + M::y0(k) * G::SY + M::z0(k) * G::SZ;
            vf4 o;
            o.x = v[l];
            o.y = v[l + 1];
            o.z = v[l + 2];
            o.w = v[l + 3];
            const uint32_t g = gq + (uint32_t)M::y0(k) * wi.n0 + (uint32_t)M::z0(k) * wi.n01;
            *(SZI_G vf4a4*)at(ob, g) = o;
        }
    } else {
#pragma unroll 1
        for (int k = 0; k < M::NS; ++k) {
            const int y = M::y0(k) + (int)sub, z = M::z0(k);
            if (y >= wi.own(1) || z >= wi.own(2)) continue;
            const int l = x + y * G::SY + z * G::SZ;
            const uint32_t g = (uint32_t)x + (uint32_t)y * wi.n0 + (uint32_t)z * wi.n01;
            if (x + 4 <= wi.own(0)) {
                *(SZI_G vf4a4*)at(ob, g) = vf4{v[l], v[l + 1], v[l + 2], v[l + 3]};
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (x + i < wi.own(0)) *at(ob, g + (uint32_t)i) = v[l + i];
            }
        }
    }
}

// ------------------------------------------------------------ group order
// Work is handed out in groups of kWaves windows of one field (the host
// pads each field to whole groups).  Workgroups on one L2 domain take one
// contiguous eighth of the groups, so that windows sharing faces are
// processed close in time on the same L2: in round k its S workgroups take
// the k-th run of S groups, workgroup j the group (j + k) mod S of the run.
// The rotation, and that of the wave slots within a group every kWaves
// rounds, spread windows of one kind (the field's far boundary along x
// always falls in the same slot of every fourth group) over all waves.  A
// fixed group and slot per workgroup and wave sent all of them to a
// quarter of the workgroups, one wave each, which finished a fifth later
// than the rest.
struct GroupSeq {
    uint64_t lo, end;   // the L2 domain's groups
    uint32_t S, j, k;   // workgroups in the domain, this one's index, round
    uint32_t rot;       // (j + k) mod S
    uint64_t g;         // the round's group, lo + k S + rot (increasing; past end: done)
    __device__ __forceinline__ bool ok() const { return g < end; }
    __device__ __forceinline__ void next() {
        ++k;
        const bool wrap = rot + 1u == S;
        rot = wrap ? 0u : rot + 1u;
        g += wrap ? 1u : S + 1u;   // S further, and the rotation's step
    }
    // the window slot of a wave in the round's group
    __device__ __forceinline__ uint32_t slot(int wave) const {
        return ((uint32_t)wave + k / (uint32_t)kWaves) % (uint32_t)kWaves;
    }
    // Issue priority of the round.  A SIMD issues from its oldest wave
    // first, so with equal work the workgroups dispatched first on a CU
    // finish first and the last ones run on alone.  Dispatch fills the
    // domain's 32 CUs one workgroup each before it places second ones, so
    // the T = S / 32 workgroups that share a CU are j, j + 32, .. of the
    // domain; with priority (k + j / 32) mod T they hold the highest
    // priority in turn, one round each.
    __device__ __forceinline__ void set_priority() const {
        constexpr uint32_t kCusPerDomain = 32;   // 256 CUs in 8 L2 domains
        uint32_t T = S / kCusPerDomain;
        T = T < 1u ? 1u : (T > 4u ? 4u : T);
        const uint32_t p = (k + j / kCusPerDomain) % T;
        if (p == 0u) __builtin_amdgcn_s_setprio(0);
        else if (p == 1u) __builtin_amdgcn_s_setprio(1);
        else if (p == 2u) __builtin_amdgcn_s_setprio(2);
        else __builtin_amdgcn_s_setprio(3);
    }
};
__device__ __forceinline__ GroupSeq group_seq(uint64_t ngroups) {
    const uint32_t G = gridDim.x, b = blockIdx.x;
    GroupSeq s;
    if (G >= (uint32_t)kXcds && G % (uint32_t)kXcds == 0u) {
        const uint64_t chunk = (ngroups + kXcds - 1) / kXcds;
        s.lo = (uint64_t)(b % (uint32_t)kXcds) * chunk;
        s.end = s.lo + chunk < ngroups ? s.lo + chunk : ngroups;
        s.S = G / (uint32_t)kXcds;
        s.j = b / (uint32_t)kXcds;
    } else {
        s.lo = 0;
        s.end = ngroups;
        s.S = G;
        s.j = b;
    }
    s.k = 0;
    s.rot = s.j;   // j < S
    s.g = s.lo + s.j;
    return s;
}

// --------------------------------------------------------------- kernels
// LDS histogram of a workgroup: the 2R symbols, then one bin per lane that
// collects the centre code; the flush folds the lane bins into the centre
// bin.
__device__ __forceinline__ void clear_hist(uint32_t* hist, int R) {
#pragma unroll 1
    for (int b = threadIdx.x; b < 2 * R + 64; b += kThreads) hist[b] = 0;
}
__device__ __forceinline__ void flush_hist(uint32_t* hist, const FieldDesc& fd) {
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t c = wave_sum(hist[2 * fd.R + threadIdx.x]);
        if (threadIdx.x == 0) atomicAdd(&hist[fd.R], c);
    }
    __syncthreads();
#pragma unroll 1
    for (int b = threadIdx.x; b < 2 * fd.R; b += kThreads)
        if (hist[b]) gatomic_add(gp(fd.hist) + b, hist[b]);
    __syncthreads();
}

// WPE waves per SIMD: the register budget that leaves (3: 168 VGPRs, 4:
// 128) is what a kernel variant is compiled for.  With the block alone in
// LDS (and the histogram of compression), three workgroups of four 3D
// windows fit a CU; 2D blocks are small enough for four.
#define SZI_WINDOW_KERNEL \
    __global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(WPE)))

template <int ND, int WPE>
SZI_WINDOW_KERNEL void k_compress(const FieldDesc* __restrict__ F, const FieldPlan* __restrict__ P,
                                  const uint64_t* __restrict__ goff, uint64_t ngroups) {
    using G = Geo<ND>;
    __shared__ float vbuf[kWaves][vlen<ND>()];
    extern __shared__ uint32_t hist[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave] + kPad;
    GroupSeq gs = group_seq(ngroups);
    if (!gs.ok()) return;
    int f = 0;
    float pre[QuadMap<ND>::N];   // block of the next window
    QuadMap<ND> qm;
    Win wn;
    bool valid;
    // window of group g for this wave, and the start of its block load
    auto fetch = [&]() {
        while (gs.g >= goff[f + 1]) ++f;
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        valid = w < (uint32_t)(F[f].nwin[0] * F[f].nwin[1] * F[f].nwin[2]);
        if (valid) {
            wn = make_win<ND>(F[f], w);
            const SZI_G float* wb = gp(F[f].in) + wn.gbase;
            qm.init(lane, wn.n0, wn.n01);
            if (wn.full) load_quads<ND, true>(pre, wb, qm, lane, wn);
            else load_quads<ND, false>(pre, wb, qm, lane, wn);
        }
    };
    fetch();
    int hf = -1;         // field whose histogram the workgroup accumulates
    uint32_t passes = 0;
    while (true) {
        const int fc = f;
        const Win wc = wn;
        const bool vc = valid;
        if (fc != hf) {   // uniform over the workgroup: groups never span fields
            if (hf >= 0) flush_hist(hist, F[hf]);
            clear_hist(hist, F[fc].R);
            __syncthreads();
            hf = fc;
            passes = load_passes(P[fc], lane);
        }
        if (vc) commit_quads<ND>(v, pre, qm, lane, wc.n01);
        gs.next();
        gs.set_priority();
        const bool more = gs.ok();
        if (more) fetch();   // in flight during the passes below
        if (vc) {
            wave_sync();
            const FieldDesc& fd = F[fc];
            const PassOut po{gp(fd.codes) + wc.gbase, nullptr, hist};
            run_levels<ND, true>(v, lane, passes, fd.R, wc, po);
            write_anchors<ND>(v, lane, fd, wc, hist);
            wave_sync();
        }
        if (!more) break;
    }
    flush_hist(hist, F[hf]);
}

template <int ND, int WPE>
SZI_WINDOW_KERNEL void k_decompress(const FieldDesc* __restrict__ F,
                                    const FieldPlan* __restrict__ P,
                                    const uint64_t* __restrict__ goff, uint64_t ngroups) {
    using G = Geo<ND>;
    __shared__ float vbuf[kWaves][vlen<ND>()];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave] + kPad;
    GroupSeq gs = group_seq(ngroups);
    if (!gs.ok()) return;
    int f = 0;
    // codes of the next window's block; block points outside the field
    // hold a value no code takes
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    uint32_t pre[G::NPRE];
    float apre = 0.0f;   // one anchor per lane
    LaneMap<ND> lm;
    Win wn;
    bool valid;
    auto fetch = [&]() {
        while (gs.g >= goff[f + 1]) ++f;
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        valid = w < (uint32_t)(F[f].nwin[0] * F[f].nwin[1] * F[f].nwin[2]);
        if (valid) {
            wn = make_win<ND>(F[f], w);
            lm.init(lane, wn.n0, wn.n01);
            const SZI_G uint16_t* cb = gp(F[f].codes) + wn.gbase;
            if (wn.full) load_block<ND, true>(pre, cb, lm, wn, kNone);
            else load_block<ND, false>(pre, cb, lm, wn, kNone);
            uint32_t ga;
            int la;
            if (anchor_slot<ND>(lane, F[f], wn, ga, la)) apre = gp(F[f].anchors)[ga];
        }
    };
    fetch();
    int pf = -1;   // the field that passes belongs to
    uint32_t passes = 0;
    while (true) {
        // 2D: lane-dependent addresses are formed anew for each window: kept
        // in registers they cost the fifth wave a SIMD (137 -> 95 registers,
        // 24 climate fields 301 -> 274 us; in 3D, where LDS bounds the
        // waves, 247 -> 250)
        if (ND == 2) asm volatile("" : "+v"(lane));
        const int fc = f;
        const Win wc = wn;
        const bool vc = valid;
        if (fc != pf) {
            passes = load_passes(P[fc], lane);
            pf = fc;
        }
        if (vc) {
            // every point of the block takes its code (as float bits), those
            // outside the field the value kNone; the anchors then their values
#pragma unroll
            for (int k = 0; k < G::NPRE; ++k) {
                uint32_t gg;
                int l;
                if (lm.template slot<true>(k, wc, gg, l)) v[l] = __uint_as_float(pre[k]);
            }
            uint32_t ga;
            int la;
            if (anchor_slot<ND>(lane, F[fc], wc, ga, la)) v[la] = apre;
        }
        gs.next();
        gs.set_priority();
        const bool more = gs.ok();
        if (more) fetch();   // in flight during the passes below
        if (vc) {
            wave_sync();
            const FieldDesc& fd = F[fc];
            const PassOut po{nullptr, gp((const float*)fd.out) + wc.gbase, nullptr};
            run_levels<ND, false>(v, lane, passes, fd.R, wc, po);
            // the next block's codes are here by now: waited for ahead of
            // the stores of this window's values, not behind them
            settle(pre);
            asm volatile("" : "+v"(apre));
            if (wc.full) write_values<ND, true>(v, lane, fd, wc);
            else write_values<ND, false>(v, lane, fd, wc);
            wave_sync();
        }
        if (!more) break;
    }
}

// ------------------------------------------------------------ 1D fields
// Sec. V-A in one dimension: anchors every kS1 = 512 points, nine levels
// (strides 256 .. 1), one pass per level.  A window is four chunks, 2048
// points, plus the far anchor, as the 3D and 2D windows span four chunks
// along x; one wave per window.
//
// Lane t holds points 32 t .. 32 t + 31 in registers.  The levels of stride
// 16 and below lie inside the lanes: a lane's targets read its own points
// and three of its neighbours' (lane moves), every index a compile-time
// constant; those five levels hold 31 of 32 points.  The four coarse levels
// work on the lanes' first points, one target a lane, through LDS.  Values
// and codes cross between this layout and coalesced 16-byte global accesses
// through a wave's LDS rows of 32 words, the 16-byte groups of a row
// permuted by the row so that neither side meets bank conflicts.
// Bound by instruction issue and, near it, by memory: 2^26 points, rel 1e-3:
// compression 112 us (3.6 TB/s of values and codes), replay 96 us; one target
// per lane at a time with its four neighbours read from LDS took 250 and
// 217 us.
constexpr int kS1 = 512, kW1 = 4 * kS1;
constexpr int kP1 = kW1 / 64;   // points per lane
static_assert(kP1 == 32, "a lane's points are one LDS row");

struct Win1 {
    uint32_t lo;   // first point
    int e;         // block extent: owned points, and the far anchor where present
    int o;         // owned extent
};

__device__ __forceinline__ Win1 make_win1(const FieldDesc& f, uint32_t w) {
    Win1 wi;
    // a field has fewer than 2^32 points (the compiler drops the scalar
    // condition of the 64-bit comparison)
    wi.lo = w * (uint32_t)kW1;
    const uint32_t left = (uint32_t)f.npts - 1u - wi.lo;
    wi.e = (int)(left < (uint32_t)kW1 ? left : (uint32_t)kW1) + 1;
    wi.o = wi.e < kW1 ? wi.e : kW1;
    return wi;
}

// word of point i of a window in the LDS rows
__device__ __forceinline__ uint32_t row_word(uint32_t i) {
    const uint32_t r = i >> 5, g = (i >> 2) & 7u;
    return r * 32u + 4u * (g ^ (r & 7u)) + (i & 3u);
}
// word that holds the 16-bit codes i and i ^ 1 in the LDS rows of 16 words
__device__ __forceinline__ uint32_t code_word(uint32_t i) {
    const uint32_t r = i >> 5, g = (i >> 3) & 3u;
    return r * 16u + 4u * (g ^ ((r >> 2) & 3u)) + ((i >> 1) & 3u);
}
// the value of the lane below / above (lanes 0 and 63 get no meaningful one)
__device__ __forceinline__ float lane_below(float x) {
    constexpr int kWaveShr = 0x138;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kWaveShr, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_above(float x) {
    constexpr int kWaveShl = 0x130;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kWaveShl, 0xF, 0xF, false));
}

// What the passes of a window need besides its values: codes of the lane's
// points, two a word (written in compression, read in the replay).
struct Lane1 {
    float r[kP1];          // the lane's points
    uint32_t pk[kP1 / 2];  // their codes
    float far;             // the far anchor
};

// Finishes K targets at the lane's points o0, o0 + so, ..: quantises and
// counts them (compression) or adds their residuals (replay).
template <int SPL, bool COMP, bool FULL, int K>
__device__ __forceinline__ void finish1(Lane1& L, uint32_t lane, int o0, int so, float (&pr)[K],
                                        const float (&nm)[K], const bool (&in)[K], const Win1& wi,
                                        float el, float ebx2, float inv, int R,
                                        const SZI_G float* ob, uint32_t* hist) {
    if (SPL == SPL_NAT) divide_small<K>(pr, nm);
    if (COMP) {
        float xv[K], xr[K];
        uint32_t cd[K];
#pragma unroll
        for (int j = 0; j < K; ++j) xv[j] = L.r[o0 + j * so];
        quantise<K>(pr, xv, in, el, ebx2, inv, R, xr, cd);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int o = o0 + j * so;
            L.r[o] = xr[j];
            if (o & 1) L.pk[o >> 1] |= cd[j] << 16;
            else L.pk[o >> 1] |= cd[j];
            // the centre code goes to the lane's own bin
            const uint32_t bin = cd[j] != (uint32_t)R ? cd[j] : (uint32_t)(2 * R) + lane;
            if (FULL || kP1 * (int)lane + o < wi.o) atomicAdd(&hist[bin], 1u);
        }
    } else {
        uint32_t least = 0xFFFFu, cd[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int o = o0 + j * so;
            cd[j] = (o & 1) ? L.pk[o >> 1] >> 16 : L.pk[o >> 1] & 0xFFFFu;
            L.r[o] = pr[j] + (float)((int)cd[j] - R) * ebx2;
            least = cd[j] < least ? cd[j] : least;
        }
        // code 0: an outlier, whose value the scatter step put in the output
        // (points outside the field hold a code no point takes)
        if (wave_any(least == 0u)) {
            float v[K];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                v[j] = L.r[o0 + j * so];
                if (cd[j] == 0u) v[j] = *at(ob, (uint32_t)(kP1 * (int)lane + o0 + j * so));
            }
            settle(v);
#pragma unroll
            for (int j = 0; j < K; ++j) L.r[o0 + j * so] = v[j];
        }
    }
}

// One level of stride S1 <= 16, inside the lanes; next0: the first point of
// the lane above.
template <int S1, int SPL, bool COMP, bool FULL>
__device__ __forceinline__ void fine_level1(Lane1& L, uint32_t lane, float next0, const FieldPlan& pl,
                                            const Win1& wi, int R, const SZI_G float* ob,
                                            uint32_t* hist) {
    constexpr int lvl = S1 == 1 ? 0 : S1 == 2 ? 1 : S1 == 4 ? 2 : S1 == 8 ? 3 : 4;
    constexpr int N = kP1 / (2 * S1);        // targets per lane
    constexpr int K = N < 4 ? N : 4;         // finished together
    const float el = pl.el[lvl], ebx2 = pl.ebx2[lvl];
    const float inv = el == 0.0f ? 0.0f : pl.inv[lvl];
    // the known before the lane's first point, and the one past next0
    const float below = lane_below(L.r[(kP1 - 2 * S1) % kP1]);
    const float above = lane_above(S1 == 16 ? next0 : L.r[(2 * S1) % kP1]);
    // lane 63's step past next0 would leave the window; lane 62 of stride
    // 16 reaches the far anchor, which only next0 of lane 63 holds
    const int last = wi.e - 1;
    auto known = [&](int o) SZI_INLINE {
        return o < 0 ? below : (o < kP1 ? L.r[o] : (o == kP1 ? next0 : above));
    };
#pragma unroll
    for (int j0 = 0; j0 < N; j0 += K) {
        float pr[K], nm[K];
        bool in[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int i = j0 + j, o = (2 * i + 1) * S1;
            const int pos = kP1 * (int)lane + o;
            const bool m3 = i > 0 || lane > 0u;
            const bool p1 = FULL || pos + S1 <= last;
            const bool p3 = FULL ? (i < N - 1 || lane < 63u) : pos + 3 * S1 <= last;
            in[j] = FULL || pos <= last;
            pr[j] = predict<SPL>(m3, p1, p3, known(o - 3 * S1), known(o - S1), known(o + S1),
                                 known(o + 3 * S1), nm[j]);
        }
        finish1<SPL, COMP, FULL, K>(L, lane, (2 * j0 + 1) * S1, 2 * S1, pr, nm, in, wi, el, ebx2, inv,
                                    R, ob, hist);
        // targets finished later are not predicted ahead (their registers
        // would not fit)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// All levels of a window.  c: 66 words of the wave's LDS.
template <int SPL, bool COMP, bool FULL>
__device__ __forceinline__ void levels1(Lane1& L, float* c, uint32_t lane, const FieldPlan& pl,
                                        const Win1& wi, int R, const SZI_G float* ob,
                                        uint32_t* hist) {
    const int last = wi.e - 1;
    const int pos = kP1 * (int)lane;
    if (lane == 0) c[64] = L.far;
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) {   // strides 32 m: 256, 128, 64, 32
        constexpr int kLvl[9] = {0, 5, 6, 0, 7, 0, 0, 0, 8};
        const int lvl = kLvl[m], s = kP1 * m;
        const float el = pl.el[lvl], ebx2 = pl.ebx2[lvl];
        const float inv = el == 0.0f ? 0.0f : pl.inv[lvl];
        c[lane] = L.r[0];
        wave_sync();
        const int t = (int)lane;
        const float a = c[t >= 3 * m ? t - 3 * m : 0], b = c[t >= m ? t - m : 0];
        const float cc = c[t + m < 64 ? t + m : 64], d = c[t + 3 * m < 64 ? t + 3 * m : 64];
        wave_sync();
        if ((t & (2 * m - 1)) == m) {
            float pr[1], nm[1];
            bool in[1] = {FULL || pos <= last};
            pr[0] = predict<SPL>(pos >= 3 * s, pos + s <= last, pos + 3 * s <= last, a, b, cc, d, nm[0]);
            finish1<SPL, COMP, FULL, 1>(L, lane, 0, 1, pr, nm, in, wi, el, ebx2, inv, R, ob, hist);
        }
    }
    const float up = lane_above(L.r[0]);
    const float next0 = lane == 63u ? L.far : up;
    fine_level1<16, SPL, COMP, FULL>(L, lane, next0, pl, wi, R, ob, hist);
    fine_level1<8, SPL, COMP, FULL>(L, lane, next0, pl, wi, R, ob, hist);
    fine_level1<4, SPL, COMP, FULL>(L, lane, next0, pl, wi, R, ob, hist);
    fine_level1<2, SPL, COMP, FULL>(L, lane, next0, pl, wi, R, ob, hist);
    fine_level1<1, SPL, COMP, FULL>(L, lane, next0, pl, wi, R, ob, hist);
}

template <bool COMP, bool FULL>
__device__ __forceinline__ void levels1_spline(Lane1& L, float* c, uint32_t lane, const FieldPlan& pl,
                                               const Win1& wi, int R, const SZI_G float* ob,
                                               uint32_t* hist) {
    const int spl = pl.spline[0];
    if (spl == SPL_LIN) levels1<SPL_LIN, COMP, FULL>(L, c, lane, pl, wi, R, ob, hist);
    else if (spl == SPL_NAK) levels1<SPL_NAK, COMP, FULL>(L, c, lane, pl, wi, R, ob, hist);
    else levels1<SPL_NAT, COMP, FULL>(L, c, lane, pl, wi, R, ob, hist);
}

// The next window of a wave: whole windows on 16-byte boundaries are loaded
// ahead, 16 bytes a lane, while the current one is processed; others when
// their turn comes, value by value.
struct Next1 {
    Win1 wi;
    int f;
    bool valid, ahead;
};

// (compression holds the block, its codes and the next block: 166 registers
// without spills; four waves a SIMD spilled the next block, 199 us)
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_compress1d(
    const FieldDesc* __restrict__ F, const FieldPlan* __restrict__ P,
    const uint64_t* __restrict__ goff, uint64_t ngroups) {
    __shared__ __align__(16) float vbuf[kWaves][kW1];
    extern __shared__ uint32_t hist[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave];
    GroupSeq gs = group_seq(ngroups);
    if (!gs.ok()) return;
    int f = 0, hf = -1;
    Next1 nx;
    vf4 pre[8];
    float farp = 0.0f;
    auto fetch = [&]() SZI_INLINE {
        while (gs.g >= goff[f + 1]) ++f;
        const FieldDesc& fd = F[f];
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        nx.f = f;
        nx.valid = w < (uint32_t)fd.nwin[0];
        nx.ahead = false;
        if (nx.valid) {
            nx.wi = make_win1(fd, w);
            nx.ahead = nx.wi.o == kW1 && ((uintptr_t)fd.in & 15u) == 0u;
            const SZI_G float* in = gp(fd.in) + nx.wi.lo;
            if (nx.ahead) {
#pragma unroll
                for (int k = 0; k < 8; ++k) pre[k] = *at((const SZI_G vf4*)in, 64u * k + lane);
            }
            if (nx.wi.e > kW1) farp = in[kW1];
        }
    };
    fetch();
    while (true) {
        asm volatile("" : "+v"(lane));   // LDS addresses are formed anew, not kept in registers
        const Next1 cu = nx;
        Lane1 L;
        L.far = farp;
        if (cu.f != hf) {   // uniform over the workgroup: groups never span fields
            if (hf >= 0) flush_hist(hist, F[hf]);
            clear_hist(hist, F[cu.f].R);
            __syncthreads();
            hf = cu.f;
        }
        const FieldDesc& fd = F[cu.f];
        if (cu.valid) {
            if (cu.ahead) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    *reinterpret_cast<vf4*>(v + row_word(256u * k + 4u * lane)) = pre[k];
            } else {
                const SZI_G float* in = gp(fd.in) + cu.wi.lo;
#pragma unroll 4
                for (int i = (int)lane; i < kW1; i += 64) v[row_word((uint32_t)i)] = i < cu.wi.o ? in[i] : 0.0f;
            }
            wave_sync();
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const vf4 q = *reinterpret_cast<const vf4*>(v + row_word(32u * lane + 4u * g));
                L.r[4 * g] = q.x;
                L.r[4 * g + 1] = q.y;
                L.r[4 * g + 2] = q.z;
                L.r[4 * g + 3] = q.w;
            }
            wave_sync();
        }
        gs.next();
        const bool more = gs.ok();
        if (more) fetch();   // in flight during the passes below
        if (cu.valid) {
            const int R = fd.R;
#pragma unroll
            for (int k = 0; k < kP1 / 2; ++k) L.pk[k] = 0u;
            // owned anchors: their values losslessly, quant-code R, counted
            const int pos = kP1 * (int)lane;
            if ((pos & (kS1 - 1)) == 0 && pos < cu.wi.o) {
                gp(fd.anchors)[(cu.wi.lo + (uint32_t)pos) / (uint32_t)kS1] = L.r[0];
                L.pk[0] = (uint32_t)R;
                atomicAdd(&hist[2 * R + (int)lane], 1u);
            }
            if (cu.wi.e > kW1) levels1_spline<true, true>(L, v, lane, P[cu.f], cu.wi, R, nullptr, hist);
            else levels1_spline<true, false>(L, v, lane, P[cu.f], cu.wi, R, nullptr, hist);
            // the codes, two a word, through LDS to coalesced stores
            wave_sync();
            uint32_t* u = reinterpret_cast<uint32_t*>(v);
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<vu4*>(u + code_word(32u * lane + 8u * g)) =
                    vu4{L.pk[4 * g], L.pk[4 * g + 1], L.pk[4 * g + 2], L.pk[4 * g + 3]};
            wave_sync();
            SZI_G uint16_t* cb = gp(fd.codes) + cu.wi.lo;   // 16-byte aligned
            if (cu.wi.o == kW1) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *at((SZI_G vu4*)cb, 64u * k + lane) =
                        *reinterpret_cast<const vu4*>(u + code_word(512u * k + 8u * lane));
            } else {
                for (int i = (int)lane; i < cu.wi.o; i += 64)
                    cb[i] = (uint16_t)(u[code_word((uint32_t)i)] >> (16 * (i & 1)));
            }
            wave_sync();
        }
        if (!more) break;
    }
    flush_hist(hist, F[hf]);
}

__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_decompress1d(
    const FieldDesc* __restrict__ F, const FieldPlan* __restrict__ P,
    const uint64_t* __restrict__ goff, uint64_t ngroups) {
    __shared__ __align__(16) float vbuf[kWaves][kW1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave];
    uint32_t* u = reinterpret_cast<uint32_t*>(v);
    GroupSeq gs = group_seq(ngroups);
    if (!gs.ok()) return;
    int f = 0;
    Next1 nx;
    vu4 pre[4];
    float ancp = 0.0f, farp = 0.0f;
    auto fetch = [&]() SZI_INLINE {
        while (gs.g >= goff[f + 1]) ++f;
        const FieldDesc& fd = F[f];
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        nx.f = f;
        nx.valid = w < (uint32_t)fd.nwin[0];
        nx.ahead = false;
        if (nx.valid) {
            nx.wi = make_win1(fd, w);
            nx.ahead = nx.wi.o == kW1;
            const SZI_G uint16_t* cb = gp((const uint16_t*)fd.codes) + nx.wi.lo;   // 16-byte aligned
            if (nx.ahead) {
#pragma unroll
                for (int k = 0; k < 4; ++k) pre[k] = *at((const SZI_G vu4*)cb, 64u * k + lane);
            }
            const int pos = kP1 * (int)lane;
            const SZI_G float* anc = gp((const float*)fd.anchors) + nx.wi.lo / (uint32_t)kS1;
            if ((pos & (kS1 - 1)) == 0 && pos < nx.wi.o) ancp = anc[pos / kS1];
            if (nx.wi.e > kW1) farp = anc[kW1 / kS1];
        }
    };
    fetch();
    while (true) {
        asm volatile("" : "+v"(lane));   // LDS addresses are formed anew, not kept in registers
        const Next1 cu = nx;
        const FieldDesc& fd = F[cu.f];
        Lane1 L;
        L.far = farp;
        L.r[0] = ancp;
        if (cu.valid) {
            if (cu.ahead) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<vu4*>(u + code_word(512u * k + 8u * lane)) = pre[k];
            } else {
                // points outside the field hold a code no point takes
                const SZI_G uint16_t* cb = gp((const uint16_t*)fd.codes) + cu.wi.lo;
                uint16_t* h = reinterpret_cast<uint16_t*>(u);
                for (int i = (int)lane; i < kW1; i += 64)
                    h[2u * code_word((uint32_t)i) + (uint32_t)(i & 1)] = i < cu.wi.o ? cb[i] : (uint16_t)0xFFFFu;
            }
            wave_sync();
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const vu4 q = *reinterpret_cast<const vu4*>(u + code_word(32u * lane + 8u * g));
                L.pk[4 * g] = q.x;
                L.pk[4 * g + 1] = q.y;
                L.pk[4 * g + 2] = q.z;
                L.pk[4 * g + 3] = q.w;
            }
            wave_sync();
        }
        gs.next();
        const bool more = gs.ok();
        if (more) fetch();   // in flight during the passes below
        if (cu.valid) {
            const int R = fd.R;
            SZI_G float* ob = gp(fd.out) + cu.wi.lo;
            if (cu.wi.e > kW1) levels1_spline<false, true>(L, v, lane, P[cu.f], cu.wi, R, ob, nullptr);
            else levels1_spline<false, false>(L, v, lane, P[cu.f], cu.wi, R, ob, nullptr);
            wave_sync();
#pragma unroll
            for (int g = 0; g < 8; ++g)
                *reinterpret_cast<vf4*>(v + row_word(32u * lane + 4u * g)) =
                    vf4{L.r[4 * g], L.r[4 * g + 1], L.r[4 * g + 2], L.r[4 * g + 3]};
            wave_sync();
            // the next window's codes are here by now: waited for ahead of
            // the stores, not behind them
            settle(pre);
            if (cu.wi.o == kW1 && ((uintptr_t)fd.out & 15u) == 0u) {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    *at((SZI_G vf4*)ob, 64u * k + lane) =
                        *reinterpret_cast<const vf4*>(v + row_word(256u * k + 4u * lane));
            } else {
                for (int i = (int)lane; i < cu.wi.o; i += 64) ob[i] = v[row_word((uint32_t)i)];
            }
            wave_sync();
        }
        if (!more) break;
    }
}

// ------------------------------------------------------------ any window
// Fields whose anchor stride or window is not the default one (Sec. V-A and
// V-D leave both open: the window trades prediction accuracy at its faces
// against parallelism) run a generic pair of kernels with the geometry read
// from the field descriptor: one wave per window, its block (window + far
// faces) in LDS.  The passes work on lines as those above, K consecutive
// targets of a line per task, with run-time strides; stencils, quantiser and
// histogram are the same.  Bound by instruction issue: 16x16x8 windows of a
// 256x384x384 field, rel 1e-3, compression 216 us and replay 194 us, against
// 449 and 370 with one target a lane, its coordinates by two 32-bit
// multiplies at a quarter of the rate, and 64 KB of LDS a workgroup whatever
// the block.
struct WinG {
    uint64_t gbase;
    uint32_t n0, n01;
    int lo[3], e[3], o[3];   // origin, block extent, owned extent per dimension
    int B0, B01;             // LDS strides
};

__device__ __forceinline__ WinG make_wing(const FieldDesc& f, uint32_t w) {
    WinG wi;
    const uint32_t nw0 = (uint32_t)f.nwin[0], nw01 = nw0 * (uint32_t)f.nwin[1];
    const uint32_t wz = w / nw01, r = w - wz * nw01, wy = r / nw0, wx = r - wy * nw0;
    const uint32_t wc[3] = {wx, wy, wz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        wi.lo[k] = (int)wc[k] * f.w[k];
        const int sk = f.n[k] - 1 - wi.lo[k];
        wi.e[k] = (sk < f.w[k] ? sk : f.w[k]) + 1;
        wi.o[k] = wi.e[k] < f.w[k] ? wi.e[k] : f.w[k];
    }
    wi.n0 = (uint32_t)f.n[0];
    wi.n01 = wi.n0 * (uint32_t)f.n[1];
    wi.B0 = f.ndim >= 1 ? f.w[0] + 1 : 1;
    wi.B01 = wi.B0 * (f.ndim >= 2 ? f.w[1] + 1 : 1);
    wi.gbase = (uint64_t)wi.lo[0] + (uint64_t)wi.lo[1] * wi.n0 + (uint64_t)wi.lo[2] * wi.n01;
    return wi;
}

// t / m for t <= 2^12 and m < kMagicN, from the high half of a 24-bit product:
// (t 2^8) ceil(2^24 / m) / 2^32, exact because t m < 2^24 (24-bit multiplies
// issue at full rate)
struct Div24 {
    uint32_t m, mg;
    __device__ __forceinline__ void set(uint32_t mm) {
        m = mm;
        mg = (kMagic.v[mm] + 0xFFu) >> 8;
    }
    __device__ __forceinline__ uint32_t div(uint32_t t) const {
        const uint32_t a = (t << 8) & 0xFFFFFFu, b = mg & 0xFFFFFFu;
        return m > 1 ? (uint32_t)(((uint64_t)a * b) >> 32) : t;
    }
};
static_assert((uint64_t)kGenMaxBlock * (kGenMaxExtent + 1) < (1ull << 24) && kGenMaxBlock <= (1 << 12),
              "block points times an extent stay below 2^24");

// a point's block coordinates from its number among m0 x m1 x m2 grid
// points with the given spacing per dimension
struct Grid3 {
    Div24 f0, f1;
    int step;
    __device__ __forceinline__ void at(uint32_t t, uint32_t* c) const {
        const uint32_t t1 = f0.div(t), i0 = t - __umul24(t1, f0.m);
        const uint32_t i2 = f1.div(t1), i1 = t1 - __umul24(i2, f1.m);
        c[0] = i0 * (uint32_t)step;
        c[1] = i1 * (uint32_t)step;
        c[2] = i2 * (uint32_t)step;
    }
};
// index of block coordinates in LDS and from the window origin in the field
// (fewer than 2^32 points, so 32 bits hold it; its bytes may need more)
__device__ __forceinline__ uint32_t lds_index(const WinG& wi, const uint32_t* c) {
    return c[0] + __umul24(c[1], (uint32_t)wi.B0) + __umul24(c[2], (uint32_t)wi.B01);
}
__device__ __forceinline__ uint32_t field_index(const WinG& wi, const uint32_t* c) {
    return c[0] + mul16x32(c[1], wi.n0) + mul16x32(c[2], wi.n01);
}

// One pass of the generic kernels along D at stride s: nseg tasks of K
// targets per line, lines ne x ng along the other dimensions e < g, spaced
// ste and stg (Sec. V-A: s where this level has passed the dimension, 2 s
// where not).  FULL: the window interval along D is the whole block and K
// divides its targets.
template <int D, int SPL, bool COMP, bool FULL, int K>
__device__ __forceinline__ void lines_gen(float* v, uint32_t lane, const WinG& wi, int s, uint32_t nseg,
                                          uint32_t ne, uint32_t ng, uint32_t ste, uint32_t stg,
                                          bool store, float el, float ebx2, float inv, int R,
                                          SZI_G uint16_t* cb, const SZI_G float* ob, uint32_t* hist) {
    constexpr int DE = D == 0 ? 1 : 0, DG = D == 2 ? 1 : 2;
    const int SD = D == 0 ? 1 : (D == 1 ? wi.B0 : wi.B01);
    const uint32_t SE = DE == 0 ? 1u : (uint32_t)wi.B0, SG = (uint32_t)(DG == 1 ? wi.B0 : wi.B01);
    const uint32_t gsd = D == 0 ? 1u : (D == 1 ? wi.n0 : wi.n01);
    const uint32_t gse = DE == 0 ? 1u : wi.n0, gsg = DG == 1 ? wi.n0 : wi.n01;
    const uint32_t owne = (uint32_t)wi.o[DE], owng = (uint32_t)wi.o[DG];
    const int lim = wi.e[D] - 1;
    Div24 fs, fe;
    fs.set(nseg);
    fe.set(ne);
    const uint32_t nt = nseg * ne * ng;
#pragma unroll 1
    for (uint32_t t = lane; t < nt; t += 64) {
        const uint32_t ln = fs.div(t), seg = t - __umul24(ln, nseg);
        const uint32_t i1 = fe.div(ln), i0 = ln - __umul24(i1, ne);
        const uint32_t ce = __umul24(i0, ste), cg = __umul24(i1, stg);
        const int base = (int)(__umul24(ce, SE) + __umul24(cg, SG));
        const int p0 = (int)__umul24(seg, (uint32_t)(2 * K) * (uint32_t)s);   // segment start along D
        // the K + 3 knowns around the targets; those outside the block are
        // read at its ends (the flags drop them)
        float kn[K + 3], xt[K], pr[K], nm[K];
#pragma unroll
        for (int i = 0; i < K + 3; ++i) {
            int p = p0 + (2 * i - 2) * s;
            if (!FULL || i == 0) p = p < 0 ? 0 : p;
            if (!FULL || i == K + 2) p = p > lim ? lim : p;
            kn[i] = v[base + __mul24(p, SD)];
        }
        bool in[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int p = p0 + (2 * j + 1) * s;
            in[j] = FULL || p <= lim;
            xt[j] = v[base + __mul24(FULL || p <= lim ? p : lim, SD)];
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int p = p0 + (2 * j + 1) * s;
            pr[j] = predict<SPL>(j > 0 || seg > 0u, FULL || p + s <= lim,
                                 FULL && j < K - 1 ? true : p + 3 * s <= lim, kn[j], kn[j + 1],
                                 kn[j + 2], kn[j + 3], nm[j]);
        }
        if (SPL == SPL_NAT) divide_small<K>(pr, nm);
        if (COMP) {
            float xr[K];
            uint32_t cd[K];
            quantise<K>(pr, xt, in, el, ebx2, inv, R, xr, cd);
            if (store) {
#pragma unroll
                for (int j = 0; j < K; ++j)
                    if (in[j]) v[base + __mul24(p0 + (2 * j + 1) * s, SD)] = xr[j];
            }
            if (ce < owne && cg < owng) {
                const uint32_t rb = (uint32_t)(2 * R) + lane;
                const uint32_t gl = mul16x32((uint32_t)p0, gsd) + mul16x32(ce, gse) + mul16x32(cg, gsg);
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const uint32_t q = (uint32_t)((2 * j + 1) * s);
                    if (p0 + (int)q < wi.o[D]) {
                        cb[gl + mul16x32(q, gsd)] = (uint16_t)cd[j];
                        atomicAdd(&hist[cd[j] != (uint32_t)R ? cd[j] : rb], 1u);
                    }
                }
            }
        } else {
            uint32_t least = 1u;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t code = __float_as_uint(xt[j]);
                pr[j] = pr[j] + (float)((int)code - R) * ebx2;
                if (in[j]) least = code < least ? code : least;
            }
            // code 0: an outlier, whose value the scatter step put in the
            // output (rare)
            if (wave_any(least == 0u)) {
                const uint32_t gl = mul16x32((uint32_t)p0, gsd) + mul16x32(ce, gse) + mul16x32(cg, gsg);
#pragma unroll
                for (int j = 0; j < K; ++j)
                    if (in[j] && __float_as_uint(xt[j]) == 0u)
                        pr[j] = ob[gl + mul16x32((uint32_t)((2 * j + 1) * s), gsd)];
                settle(pr);
            }
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (in[j]) v[base + __mul24(p0 + (2 * j + 1) * s, SD)] = pr[j];
        }
    }
}

template <int D, int SPL, bool COMP>
__device__ __forceinline__ void pass_gen(float* v, uint32_t lane, const FieldDesc& fd, const WinG& wi,
                                         int s, const bool* passed, bool store, float el, float ebx2,
                                         float inv, SZI_G uint16_t* cb, const SZI_G float* ob,
                                         uint32_t* hist) {
    constexpr int DE = D == 0 ? 1 : 0, DG = D == 2 ? 1 : 2;
    const int lim = wi.e[D] - 1;
    if (lim < s) return;   // no targets
    const uint32_t m = (uint32_t)((lim - s) / (2 * s) + 1);   // targets per line
    // at the finest level no later pass reads the far face of a dimension
    // already passed
    auto lines = [&](int j) SZI_INLINE {
        const int last = s == 1 && passed[j] ? wi.o[j] - 1 : wi.e[j] - 1;
        return (uint32_t)(last / (passed[j] ? s : 2 * s) + 1);
    };
    const uint32_t ne = lines(DE), ng = lines(DG);
    const uint32_t ste = (uint32_t)(passed[DE] ? s : 2 * s), stg = (uint32_t)(passed[DG] ? s : 2 * s);
    // long tasks where the pass has more than a few waves of targets: they
    // share knowns and the task's set-up
    const uint32_t all = m * ne * ng;
    const bool full = wi.e[D] == fd.w[D] + 1;
    auto go = [&](auto k) SZI_INLINE {
        constexpr int K = decltype(k)::value;
        if (full && m % (uint32_t)K == 0u)
            lines_gen<D, SPL, COMP, true, K>(v, lane, wi, s, m / (uint32_t)K, ne, ng, ste, stg, store, el,
                                             ebx2, inv, fd.R, cb, ob, hist);
        else
            lines_gen<D, SPL, COMP, false, K>(v, lane, wi, s, (m + (uint32_t)K - 1) / (uint32_t)K, ne, ng,
                                              ste, stg, store, el, ebx2, inv, fd.R, cb, ob, hist);
    };
    if (all >= 192u && m >= 3u) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 1>{});
}

template <int D, bool COMP>
__device__ __forceinline__ void pass_gen_spline(float* v, uint32_t lane, const FieldDesc& fd,
                                                const WinG& wi, int spl, int s, const bool* passed,
                                                bool store, float el, float ebx2, float inv,
                                                SZI_G uint16_t* cb, const SZI_G float* ob,
                                                uint32_t* hist) {
    if (spl == SPL_LIN)
        pass_gen<D, SPL_LIN, COMP>(v, lane, fd, wi, s, passed, store, el, ebx2, inv, cb, ob, hist);
    else if (spl == SPL_NAK)
        pass_gen<D, SPL_NAK, COMP>(v, lane, fd, wi, s, passed, store, el, ebx2, inv, cb, ob, hist);
    else
        pass_gen<D, SPL_NAT, COMP>(v, lane, fd, wi, s, passed, store, el, ebx2, inv, cb, ob, hist);
}

template <bool COMP>
__device__ __forceinline__ void levels_gen(float* v, uint32_t lane, const FieldDesc& fd,
                                           const FieldPlan& pl, const WinG& wi, SZI_G uint16_t* cb,
                                           const SZI_G float* ob, uint32_t* hist) {
#pragma unroll 1
    for (int l = fd.L; l >= 1; --l) {
        const int s = 1 << (l - 1);
        const float el = pl.el[l - 1], ebx2 = pl.ebx2[l - 1];
        const float inv = el == 0.0f ? 0.0f : pl.inv[l - 1];
        bool passed[3] = {false, false, false};
#pragma unroll 1
        for (int k = 0; k < fd.ndim; ++k) {
            const int d = pl.order[k];
            const int spl = pl.spline[d];
            const bool store = l > 1 || k + 1 < fd.ndim;   // the last pass's values are read by none
            if (d == 0) {
                pass_gen_spline<0, COMP>(v, lane, fd, wi, spl, s, passed, store, el, ebx2, inv, cb, ob, hist);
                passed[0] = true;
            } else if (d == 1) {
                pass_gen_spline<1, COMP>(v, lane, fd, wi, spl, s, passed, store, el, ebx2, inv, cb, ob, hist);
                passed[1] = true;
            } else {
                pass_gen_spline<2, COMP>(v, lane, fd, wi, spl, s, passed, store, el, ebx2, inv, cb, ob, hist);
                passed[2] = true;
            }
            wave_sync();
        }
    }
}

// the block's points (a grid of step 1), or its anchor points (step S) up
// to an extent per dimension
__device__ __forceinline__ Grid3 block_grid(const int* ext, int step, uint32_t& n) {
    Grid3 gr;
    uint32_t m[3];
    gr.step = step;
#pragma unroll
    for (int j = 0; j < 3; ++j) m[j] = (uint32_t)((ext[j] - 1) / step + 1);
    gr.f0.set(m[0]);
    gr.f1.set(m[1]);
    n = m[0] * m[1] * m[2];
    return gr;
}

__device__ __forceinline__ uint32_t anchor_index(const FieldDesc& fd, const WinG& wi, const uint32_t* c) {
    return ((uint32_t)wi.lo[0] + c[0]) / (uint32_t)fd.S +
           (uint32_t)fd.na[0] * (((uint32_t)wi.lo[1] + c[1]) / (uint32_t)fd.S +
                                 (uint32_t)fd.na[1] * (((uint32_t)wi.lo[2] + c[2]) / (uint32_t)fd.S));
}

// BW: LDS words per wave, at least the largest block of the launch
template <int BW>
__global__ __launch_bounds__(kThreads) void k_compress_gen(const FieldDesc* __restrict__ F,
                                                           const FieldPlan* __restrict__ P,
                                                           const uint64_t* __restrict__ goff,
                                                           uint64_t ngroups) {
    __shared__ float vbuf[kWaves][BW];
    extern __shared__ uint32_t hist[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave];
    int f = 0, hf = -1;
#pragma unroll 1
    for (GroupSeq gs = group_seq(ngroups); gs.ok(); gs.next()) {
        while (gs.g >= goff[f + 1]) ++f;
        if (f != hf) {   // uniform over the workgroup: groups never span fields
            if (hf >= 0) flush_hist(hist, F[hf]);
            clear_hist(hist, F[f].R);
            __syncthreads();
            hf = f;
        }
        const FieldDesc& fd = F[f];
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        if (w >= (uint32_t)(fd.nwin[0] * fd.nwin[1] * fd.nwin[2])) continue;
        const WinG wi = make_wing(fd, w);
        const SZI_G float* in = gp(fd.in) + wi.gbase;
        uint32_t nb;
        const Grid3 bg = block_grid(wi.e, 1, nb);
#pragma unroll 1
        for (uint32_t t = lane; t < nb; t += 512) {   // eight loads in flight
            float x[8];
            uint32_t li[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t c[3];
                bg.at(t + 64u * k < nb ? t + 64u * k : nb - 1u, c);
                li[k] = lds_index(wi, c);
                x[k] = in[field_index(wi, c)];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) v[li[k]] = x[k];   // past the end: the last point again
        }
        wave_sync();
        SZI_G uint16_t* cb = gp(fd.codes) + wi.gbase;
        levels_gen<true>(v, lane, fd, P[f], wi, cb, nullptr, hist);
        // owned anchors: their values losslessly, quant-code R, counted
        uint32_t na;
        const Grid3 ag = block_grid(wi.o, fd.S, na);
#pragma unroll 1
        for (uint32_t t = lane; t < na; t += 64) {
            uint32_t c[3];
            ag.at(t, c);
            gp(fd.anchors)[anchor_index(fd, wi, c)] = v[lds_index(wi, c)];
            cb[field_index(wi, c)] = (uint16_t)fd.R;
            atomicAdd(&hist[2 * fd.R + lane], 1u);
        }
        wave_sync();
    }
    if (hf >= 0) flush_hist(hist, F[hf]);
}

template <int BW>
__global__ __launch_bounds__(kThreads) void k_decompress_gen(const FieldDesc* __restrict__ F,
                                                             const FieldPlan* __restrict__ P,
                                                             const uint64_t* __restrict__ goff,
                                                             uint64_t ngroups) {
    __shared__ float vbuf[kWaves][BW];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63u;
    float* v = vbuf[wave];
    int f = 0;
#pragma unroll 1
    for (GroupSeq gs = group_seq(ngroups); gs.ok(); gs.next()) {
        while (gs.g >= goff[f + 1]) ++f;
        const FieldDesc& fd = F[f];
        const uint32_t w = (uint32_t)(gs.g - goff[f]) * kWaves + gs.slot(wave);
        if (w >= (uint32_t)(fd.nwin[0] * fd.nwin[1] * fd.nwin[2])) continue;
        const WinG wi = make_wing(fd, w);
        // every point takes its code (as float bits), the anchors their values
        const SZI_G uint16_t* cb = gp((const uint16_t*)fd.codes) + wi.gbase;
        uint32_t nb;
        const Grid3 bg = block_grid(wi.e, 1, nb);
#pragma unroll 1
        for (uint32_t t = lane; t < nb; t += 512) {   // eight loads in flight
            uint32_t x[8], li[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                uint32_t c[3];
                bg.at(t + 64u * k < nb ? t + 64u * k : nb - 1u, c);
                li[k] = lds_index(wi, c);
                x[k] = (uint32_t)cb[field_index(wi, c)];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) v[li[k]] = __uint_as_float(x[k]);
        }
        wave_sync();
        uint32_t na;
        const Grid3 ag = block_grid(wi.e, fd.S, na);
#pragma unroll 1
        for (uint32_t t = lane; t < na; t += 64) {
            uint32_t c[3];
            ag.at(t, c);
            v[lds_index(wi, c)] = gp((const float*)fd.anchors)[anchor_index(fd, wi, c)];
        }
        wave_sync();
        SZI_G float* ob = gp(fd.out) + wi.gbase;
        levels_gen<false>(v, lane, fd, P[f], wi, nullptr, ob, nullptr);
        uint32_t no;
        const Grid3 og = block_grid(wi.o, 1, no);
#pragma unroll 4
        for (uint32_t t = lane; t < no; t += 64) {
            uint32_t c[3];
            og.at(t, c);
            ob[field_index(wi, c)] = v[lds_index(wi, c)];
        }
        wave_sync();
    }
}

// ------------------------------------------------------- launchers
// The persistent grid is the number of workgroups resident at once
// (occupancy from the runtime x compute units) unless per_cu overrides it,
// rounded to whole L2 domains.
template <class K>
static uint64_t resident_grid(K kernel, size_t lds, int num_cus, int per_cu, uint64_t ngroups) {
    const int occ = per_cu > 0 ? per_cu : resident_per_cu(kernel, lds);
    uint64_t grid = (uint64_t)num_cus * (uint64_t)occ;
    if (grid > ngroups) grid = ngroups;
    if (grid > (uint64_t)kXcds) grid -= grid % kXcds;
    return grid;
}

hipError_t launch_compress(int ndim, const FieldDesc* d_fields, const FieldPlan* d_plans,
                           const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                           LaunchShape shape, int max_R, hipStream_t st) {
    if (ngroups == 0) return hipSuccess;
    const size_t lds = (size_t)(2 * max_R + 64) * sizeof(uint32_t);
    auto go = [&](auto k) {
        const uint64_t grid = resident_grid(k, lds, num_cus, shape.per_cu, ngroups);
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), lds, st, d_fields, d_plans,
                           d_goff, ngroups);
    };
    if (ndim == 3) go(k_compress<3, 3>);
    else if (ndim == 1) go(k_compress1d);
    else if (shape.variant == 1) go(k_compress<2, 4>);
    else go(k_compress<2, 3>);
    return hipGetLastError();
}

// The generic kernels by the LDS their blocks need: up to 1152 words a wave
// leave seven workgroups a CU, up to 2816 three, the largest blocks two.
template <class Fn>
static void by_block(uint64_t block, Fn&& go) {
    if (block <= 1152) go(std::integral_constant<int, 1152>{});
    else if (block <= 2816) go(std::integral_constant<int, 2816>{});
    else go(std::integral_constant<int, kGenMaxBlock>{});
}

hipError_t launch_compress_gen(const FieldDesc* d_fields, const FieldPlan* d_plans,
                               const uint64_t* d_goff, uint64_t ngroups, int num_cus, int max_R,
                               uint64_t block, hipStream_t st) {
    if (ngroups == 0) return hipSuccess;
    if (block > (uint64_t)kGenMaxBlock) return hipErrorInvalidValue;
    const size_t lds = (size_t)(2 * max_R + 64) * sizeof(uint32_t);
    by_block(block, [&](auto bw) {
        auto k = k_compress_gen<decltype(bw)::value>;
        const uint64_t grid = resident_grid(k, lds, num_cus, 0, ngroups);
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), lds, st, d_fields, d_plans, d_goff,
                           ngroups);
    });
    return hipGetLastError();
}

hipError_t launch_decompress_gen(const FieldDesc* d_fields, const FieldPlan* d_plans,
                                 const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                                 uint64_t block, hipStream_t st) {
    if (ngroups == 0) return hipSuccess;
    if (block > (uint64_t)kGenMaxBlock) return hipErrorInvalidValue;
    by_block(block, [&](auto bw) {
        auto k = k_decompress_gen<decltype(bw)::value>;
        const uint64_t grid = resident_grid(k, 0, num_cus, 0, ngroups);
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), 0, st, d_fields, d_plans, d_goff,
                           ngroups);
    });
    return hipGetLastError();
}

hipError_t launch_decompress(int ndim, const FieldDesc* d_fields, const FieldPlan* d_plans,
                             const uint64_t* d_goff, uint64_t ngroups, int num_cus,
                             LaunchShape shape, hipStream_t st) {
    if (ngroups == 0) return hipSuccess;
    auto go = [&](auto k) {
        const uint64_t grid = resident_grid(k, 0, num_cus, shape.per_cu, ngroups);
        hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(kThreads), 0, st, d_fields, d_plans,
                           d_goff, ngroups);
    };
    if (ndim == 3) go(k_decompress<3, 3>);
    else if (ndim == 1) go(k_decompress1d);
    else if (shape.variant == 1) go(k_decompress<2, 4>);
    else go(k_decompress<2, 3>);
    return hipGetLastError();
}

}  // namespace szi
