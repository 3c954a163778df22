// Generated by gen_constants.py; do not edit.
// D2Q37 velocity set, quadrature weights and Hermite tables (exact doubles).
#pragma once

namespace d2q37 {

constexpr int Q = 37;
// integer hops e_l = (EX[l], EY[l]); lattice velocity c_l = R * e_l
constexpr int EX[Q] = {3, 3, 3, 2, 2, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0, 0, 0, 0, -1, -1, -1, -1, -1, -1, -1, -2, -2, -2, -2, -2, -3, -3, -3};
constexpr int EY[Q] = {-1, 0, 1, -2, -1, 0, 1, 2, -3, -2, -1, 0, 1, 2, 3, -3, -2, -1, 0, 1, 2, 3, -3, -2, -1, 0, 1, 2, 3, -2, -1, 0, 1, 2, -1, 0, 1};
// quadrature weights w_l
constexpr double W[Q] = {
    0x1.292e6f2a5028ap-12, 0x1.01377e4533417p-12, 0x1.292e6f2a5028ap-12,
    0x1.0945fb76e9ba5p-10, 0x1.5ed142641e9d8p-8, 0x1.d19327de15f21p-7,
    0x1.5ed142641e9d8p-8, 0x1.0945fb76e9ba5p-10, 0x1.292e6f2a5028ap-12,
    0x1.5ed142641e9d8p-8, 0x1.d86a448815fd3p-5, 0x1.b786979d5dd9dp-4,
    0x1.d86a448815fd3p-5, 0x1.5ed142641e9d8p-8, 0x1.292e6f2a5028ap-12,
    0x1.01377e4533417p-12, 0x1.d19327de15f21p-7, 0x1.b786979d5dd9dp-4,
    0x1.dd7e1917b6364p-3, 0x1.b786979d5dd9dp-4, 0x1.d19327de15f21p-7,
    0x1.01377e4533417p-12, 0x1.292e6f2a5028ap-12, 0x1.5ed142641e9d8p-8,
    0x1.d86a448815fd3p-5, 0x1.b786979d5dd9dp-4, 0x1.d86a448815fd3p-5,
    0x1.5ed142641e9d8p-8, 0x1.292e6f2a5028ap-12, 0x1.0945fb76e9ba5p-10,
    0x1.5ed142641e9d8p-8, 0x1.d19327de15f21p-7, 0x1.5ed142641e9d8p-8,
    0x1.0945fb76e9ba5p-10, 0x1.292e6f2a5028ap-12, 0x1.01377e4533417p-12,
    0x1.292e6f2a5028ap-12,
};
constexpr double R = 0x1.326d4427cfd50p+0;  // 1.196979770393074358972388
// HE[k][n] = He_n(R k), k = 0..3 (He_n(-x) = (-1)^n He_n(x))
constexpr double HE[4][5] = {
    {0x1.0000000000000p+0, 0.0, -0x1.0000000000000p+0, 0.0, 0x1.8000000000000p+1},
    {0x1.0000000000000p+0, 0x1.326d4427cfd50p+0, 0x1.bb25964923953p-2, -0x1.e03e83a7cba48p+0, -0x1.c599f24762767p+1},
    {0x1.0000000000000p+0, 0x1.326d4427cfd50p+1, 0x1.2ec9659248e55p+2, 0x1.a26eab638ff56p+2, 0x1.7566483831aeap+0},
    {0x1.0000000000000p+0, 0x1.cba3e63bb7bf7p+1, 0x1.7ca292449201fp+3, 0x1.1c411a43ffcc6p+5, 0x1.6fa1c056bacfep+6},
};
// HEF[k][n] = He_n(R k) / n!
constexpr double HEF[4][5] = {
    {0x1.0000000000000p+0, 0.0, -0x1.0000000000000p-1, 0.0, 0x1.0000000000000p-3},
    {0x1.0000000000000p+0, 0x1.326d4427cfd50p+0, 0x1.bb25964923953p-3, -0x1.4029ad1a87c30p-2, -0x1.2e66a184ec4efp-3},
    {0x1.0000000000000p+0, 0x1.326d4427cfd50p+1, 0x1.2ec9659248e55p+1, 0x1.16f472425ff8fp+0, 0x1.f1ddb5a0423e3p-5},
    {0x1.0000000000000p+0, 0x1.cba3e63bb7bf7p+1, 0x1.7ca292449201fp+2, 0x1.7b01785aaa65ep+2, 0x1.ea2d0073a3bfep+1},
};
// INVFAC[n] = 1 / n!
constexpr double INVFAC[5] = {0x1.0000000000000p+0, 0x1.0000000000000p+0, 0x1.0000000000000p-1, 0x1.5555555555555p-3, 0x1.5555555555555p-5};
// powers of r (R2 = r^2, R6_6 = r^6 / 6, IR2_3 = 3 r^-2, ...)
constexpr double R2 = 0x1.6ec9659248e55p+0;
constexpr double R4 = 0x1.06c23e6f78397p+1;
constexpr double R6 = 0x1.78786c072ba31p+1;
constexpr double R8 = 0x1.0db22b2eda41fp+2;
constexpr double R6_6 = 0x1.f5f5e55ee4d97p-2;
constexpr double R8_6 = 0x1.67983993cdad4p-1;
constexpr double R8_24 = 0x1.67983993cdad4p-3;
constexpr double IR2 = 0x1.655a23486b0e9p-1;
constexpr double IR2_3 = 0x1.0c039a76504afp+1;
constexpr double IR2_6 = 0x1.0c039a76504afp+2;
// sum w e_x^2, sum w e_x^4, sum w e_x^2 e_y^2
constexpr double G20 = 0x1.655a23486b0e9p-1;
constexpr double G40 = 0x1.761f649b9ac71p+0;
constexpr double G22 = 0x1.f2d48624ce5ecp-2;

}  // namespace d2q37
