// A 4096-point complex fp64 transform by one workgroup of 512 threads, eight
// points each: four radix-8 passes in registers, exchanged through LDS with one
// barrier (the last three passes stay inside a wavefront).  Included only by
// translation units compiled with -ffp-contract=off.
//
// Rounding, in units u of the norm: a radix-8 pass is three levels of additions
// (u each) with exact turns or a product with sqrt(1/2) (3 u), then one
// multiplication (2.3 u) with a twiddle accurate to 17 u (table entries within 2
// ulp a component, so 4 u; a product adds the errors of both and 2.3 u, and w^7 is
// made of two): 25 u at most.  The bounds charge three radix-2 stages of 21.7 u for
// it, so a transform of 2^k points errs by less than half of the k + 1 stages that
// they count.
#pragma once

#include "fft_common.h"

namespace gpoeo {
namespace {

constexpr int kP = 4096;                     // points
constexpr int kT = 512;                      // threads
constexpr int kTw = kP / 2;                  // twiddles e^(-2 pi i e / 4096), e < 2048
static_assert(kP == 8 * kT && kT == 8 * kWave, "four radix-8 passes");

// Eight-point transforms in registers, y_m = sum_r v_r W^(r m), W = e^(-2 pi i / 8)
// (or its conjugate), natural order in and out; kHalf: v_4 .. v_7 are zero.
template <bool kInverse, bool kHalf>
__device__ __forceinline__ void dft8(double2 (&v)[8]) {
    constexpr double c = 0.70710678118654752440;
    auto turn = [](double2 z) {   // z times -i (forward) or i
        return kInverse ? make_double2(-z.y, z.x) : make_double2(z.y, -z.x);
    };
    auto w1 = [&](double2 z) {    // z W
        return kInverse ? make_double2((z.x - z.y) * c, (z.x + z.y) * c)
                        : make_double2((z.x + z.y) * c, (z.y - z.x) * c);
    };
    const double2 a0 = kHalf ? v[0] : cadd(v[0], v[4]), a1 = kHalf ? v[0] : csub(v[0], v[4]);
    const double2 a2 = kHalf ? v[2] : cadd(v[2], v[6]), a3 = turn(kHalf ? v[2] : csub(v[2], v[6]));
    const double2 b0 = kHalf ? v[1] : cadd(v[1], v[5]), b1 = kHalf ? v[1] : csub(v[1], v[5]);
    const double2 b2 = kHalf ? v[3] : cadd(v[3], v[7]), b3 = turn(kHalf ? v[3] : csub(v[3], v[7]));
    const double2 e0 = cadd(a0, a2), e2 = csub(a0, a2), e1 = cadd(a1, a3), e3 = csub(a1, a3);
    const double2 o0 = cadd(b0, b2), o2 = turn(csub(b0, b2));
    const double2 o1 = w1(cadd(b1, b3)), o3 = turn(w1(csub(b1, b3)));
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
}

// The twiddles of a radix-8 pass, w^m for m = 1 .. 7: w, w^2 and w^4 from the
// table (w = W_4096^e), the others as products of two of them or of one and a
// product, each within 17 u.
struct Twiddles {
    double2 w1, w2, w4;
    __device__ __forceinline__ void load(const double2* __restrict__ tw, int e) {
        w1 = tw[e];
        w2 = tw[2 * e];
        w4 = tw[4 * e];
    }
};
template <bool kInverse>
__device__ __forceinline__ void twiddle8(double2 (&v)[8], const Twiddles& t) {
    const double2 w3 = cmul(t.w1, t.w2), w5 = cmul(t.w1, t.w4), w6 = cmul(t.w2, t.w4);
    const double2 w7 = cmul(w3, t.w4);
    auto mul = [](double2 z, double2 w) { return kInverse ? cmul_conj(z, w) : cmul(z, w); };
    v[1] = mul(v[1], t.w1);
    v[2] = mul(v[2], t.w2);
    v[3] = mul(v[3], w3);
    v[4] = mul(v[4], t.w4);
    v[5] = mul(v[5], w5);
    v[6] = mul(v[6], w6);
    v[7] = mul(v[7], w7);
}

// LDS slots of point i, one free slot after every 8 and one more after every
// 64: each of the accesses below then touches all banks evenly.  Thread t =
// 64 w + c, c = 8 p + q, holds eight points a pass (r = 0 .. 7):
//   pass 1  t + 512 r               pass 2  512 w + c + 64 r
//   pass 3  512 w + 64 p + q + 8 r  pass 4  512 w + 8 c + r
// (decimation in frequency: 4096 natural points in, frequency w + 8 p + 64 q +
// 512 r of the point at 512 w + 64 p + 8 q + r out), so passes 2 to 4 exchange
// points inside a wavefront only.
constexpr int kSlots = kP + kP / 8 + kP / 64;
struct Lanes {
    int t, s1, s2, s3, s4, sk, sm;
    __device__ __forceinline__ explicit Lanes(int thread) {
        t = thread;
        const int w = t >> 6, c = t & 63, p = c >> 3, q = c & 7;
        s1 = t + (t >> 3) + (t >> 6);            // + 584 r
        s2 = 584 * w + c + p;                    // + 73 r
        s3 = 584 * w + 73 * p + q;               // + 9 r
        s4 = 584 * w + 9 * c + p;                // + r
        // slots of this thread's frequencies k = w + 8 p + 64 q + 512 r, and of
        // their mirrors 4096 - k (for thread 0, whose k = 0 is no mirror of
        // another, from r = 1 on)
        sk = w + 9 * p + 73 * q;                 // + 584 r
        const int u = kT - (w + 8 * p + 64 * q);
        sm = u + (u >> 3) + (u >> 6);            // + 584 (7 - r)
    }
};
template <int kStep>
__device__ __forceinline__ void put8(double2* lds, int s, const double2 (&v)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) lds[s + kStep * r] = v[r];
}
template <int kStep>
__device__ __forceinline__ void get8(const double2* lds, int s, double2 (&v)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = lds[s + kStep * r];
}
// Orders this wavefront's LDS writes before its next reads (its LDS operations
// run in order; no other wavefront's points are involved).
__device__ __forceinline__ void wave_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The first pass of a forward transform from the points t + 512 r in v to the
// LDS; kHalf: v_4 .. v_7 are zero.  The caller's barrier follows.
template <bool kHalf>
__device__ __forceinline__ void forward_first(double2* lds, const Lanes& at, double2 (&v)[8],
                                              const Twiddles& t1) {
    dft8<false, kHalf>(v);
    twiddle8<false>(v, t1);
    put8<584>(lds, at.s1, v);
}
// The other three, to the frequencies of this thread in v (tw512: W_512^e, e < 256).
__device__ __forceinline__ void forward_rest(double2* lds, const Lanes& at, double2 (&v)[8],
                                             const double2* tw512) {
    const int c = at.t & 63;
    Twiddles tw;
    tw.load(tw512, c);
    get8<73>(lds, at.s2, v);
    dft8<false, false>(v);
    twiddle8<false>(v, tw);
    put8<73>(lds, at.s2, v);
    wave_exchange();
    tw.load(tw512, 8 * (c & 7));
    get8<9>(lds, at.s3, v);
    dft8<false, false>(v);
    twiddle8<false>(v, tw);
    put8<9>(lds, at.s3, v);
    wave_exchange();
    get8<1>(lds, at.s4, v);
    dft8<false, false>(v);
}

}  // namespace
}  // namespace gpoeo
