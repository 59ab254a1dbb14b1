/* Generated by gen_cutoff_fits.py -- do not edit. */
#pragma once
/* erfcx(s) ~= u * sum_k VFMM_ERFCX_C[k] u^k, u = 1/s, s in [1.0, 6.3];
   max error it causes in P(3/2, s^2), P(5/2, s^2), relative: 1.08e-07 (float64 coefs) /
   1.55e-07 (float32 Horner). */
#define VFMM_ERFCX_DEG 5
static constexpr float VFMM_ERFCX_C[6] = {5.643908978e-01f, 1.107340306e-02f, -3.891636133e-01f, 3.861538768e-01f, -1.787817478e-01f, 3.391078115e-02f};
/* 1F1(1; 7/2; x) ~= sum_k VFMM_M2_C[k] x^k, x in [0, 1.0];
   max rel. error 3.46e-08 (float64 coefs) / 1.09e-07 (float32 Horner). */
#define VFMM_M2_DEG 5
static constexpr float VFMM_M2_C[6] = {9.999999404e-01f, 2.857158482e-01f, 6.347598135e-02f, 1.160909701e-02f, 1.655175467e-03f, 3.381539718e-04f};
/* branch point s = 1.0 (x = s^2) between the two forms */
#define VFMM_CUTOFF_XSPLIT 1.000000000e+00f
/* Float64 form, x = s^2.  x < 3: sum_k x^k / Gamma(k + 7/2), relative error 4.6e-17 (of the
   coefficients as doubles, in exact arithmetic). */
static constexpr double VFMM64_M2_C[16] = {3.00901111225470030e-01, 8.59717460644202902e-02, 1.91048324587514209e-02, 3.47360590169250652e-03, 5.34400907331056404e-04, 7.12534566086119134e-05, 8.38275404415027230e-06, 8.82404419199664462e-07, 8.40275412384677721e-08, 7.31618739783582931e-09, 5.79341542772324383e-10, 4.56607144285361020e-11, 2.23280868293570230e-12, 3.59064214941747448e-13, -1.18924337992684033e-14, 2.47330239076380958e-15};
/* 3 <= x <= 43: s erfcx(s) in t = SCALE u + SHIFT, u = 1/s; relative error it causes in P(3/2, x) and
   P(5/2, x): 1.6e-17.  1 - P(5/2, 43) = 4.6e-17. */
static constexpr double VFMM64_PE_C[12] = {5.32378135318474999e-01, -3.17951270644215092e-02, -4.39824684240165253e-03, 1.74374659322701266e-03, -2.32272761475324095e-04, -2.17224790795246132e-05, 1.97194677241051423e-05, -5.19610162480154226e-06, 5.17207667947055751e-07, 1.53842734492292529e-07, -7.50528175982086695e-08, 1.11742654212069868e-08};
#define VFMM64_PE_SCALE 4.70752501491838604e+00
#define VFMM64_PE_SHIFT -1.71789083458002745e+00
#define VFMM64_XSPLIT 3.0
#define VFMM64_XMAX 43.0
/* ln 2 = HI + LO, HI of 40 bits */
#define VFMM64_LN2_HI 6.93147180559208209e-01
#define VFMM64_LN2_LO 7.37100256516779890e-13
