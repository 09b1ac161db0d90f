// Generated by gen_icdf_table.py: polynomials of the plain sampler.
#pragma once

namespace cs {

// P(sigma) = sum_k 2 sigma^k / (2k + 3) on [0, 1/4]
constexpr int kTailPolyTerms = 16;
__constant__ constexpr double kTailPoly[16] = {
    6.66666666666666630e-01,
    4.00000000000000078e-01,
    2.85714285714250782e-01,
    2.22222222226894417e-01,
    1.81818181490559644e-01,
    1.53846167702629405e-01,
    1.33332949808410622e-01,
    1.17654366514060499e-01,
    1.05164229066601764e-01,
    9.62069398098493317e-02,
    8.00458838642351400e-02,
    1.15740849501449292e-01,
    -5.75081827186928393e-02,
    4.00305665397085453e-01,
    -4.60916898759158367e-01,
    4.88564573373308109e-01,
};

// (8/3) s(x) about x = 0, for x < kSmallX
constexpr double kSmallX = 0.00390625;
constexpr int kSmallZTerms = 8;
__constant__ constexpr double kSmallZ[8] = {
    2.66666666666666652e+00,
    -5.33333333333333304e+00,
    1.38666666666666671e+01,
    -3.54666666666666686e+01,
    8.71619047619047649e+01,
    -2.07238095238095241e+02,
    4.80507936507936506e+02,
    -1.09297777777777787e+03,
};

// the same in powers of x - kMidC, for kSmallX <= x < kMidX
constexpr double kMidX = 0.125, kMidC = 0.06666851043701172;
constexpr int kMidZTerms = 14;
__constant__ constexpr double kMidZ[14] = {
    2.36371039173310171e+00,
    -3.87124334961286065e+00,
    8.60070829245241519e+00,
    -1.91943691639883376e+01,
    4.14460160206864074e+01,
    -8.67955543987861660e+01,
    1.77426473765123063e+02,
    -3.55955114485484614e+02,
    7.03684685697307941e+02,
    -1.37485154058525904e+03,
    2.65804434265405007e+03,
    -5.08969110728220221e+03,
    1.01846937630780321e+04,
    -2.05014720342007313e+04,
};

// h(w, t), t = L / (L + kStartShift): relative error of v 1.0e-02
constexpr float kStartShift = 2.0f;
constexpr int kStartRows = 5;
constexpr int kStartDeg[5] = {5, 5, 5, 4, 3};
constexpr float kStart[5][6] = {
    {6.7338948e-01f, 1.8934626e-01f, 1.6715588e+00f, -1.9947739e-01f, -3.7444221e+00f, 2.4196518e+00f},
    {-8.5401163e-01f, 3.1280259e+00f, -2.8401510e+01f, 5.7891194e+01f, -3.2344132e+01f, 3.2329546e-01f},
    {1.3910877e+00f, -8.8784142e+00f, 6.8702337e+01f, -1.5399867e+02f, 1.0127913e+02f, -7.3322275e+00f},
    {-2.5959562e-01f, 2.3858932e+00f, -1.7914398e+01f, 7.3041258e+01f, -5.9058455e+01f, 0.0000000e+00f},
    {-5.4391230e-01f, 7.8093019e+00f, -3.4709717e+01f, 2.8357882e+01f, 0.0000000e+00f, 0.0000000e+00f},
};

// v / w for x < kSmallX: A(w) + x B(w), relative error 8.0e-04
constexpr int kStartSmallA = 8, kStartSmallB = 2;
constexpr float kStartA[9] = {1.3341255e+00f, 7.4438954e-01f, 4.3784783e+00f, -3.1663911e+01f, 1.3672623e+02f, -2.9335611e+02f, 3.1722786e+02f, -1.6838893e+02f, 3.4996256e+01f};
constexpr float kStartB[3] = {-2.5679278e+00f, -4.1998718e+00f, 7.4457755e+00f};

// P(sigma) on [0, 1/4] in FP32, relative error 5.2e-08
constexpr int kStartTailDeg = 5;
constexpr float kStartTail[6] = {6.6666663e-01f, 4.0000977e-01f, 2.8526977e-01f, 2.2950884e-01f, 1.2935588e-01f, 3.1586435e-01f};

}  // namespace cs
