// First row of the inverse of a periodic mass matrix (host code, no HIP).
#pragma once

#include <cmath>
#include <cstdlib>
#include <vector>

namespace ecpic2d {

// The matrix is dx times the circulant of M points with the symmetric stencil mass (offsets
// -d .. d).  From its eigenvalues lam_k: c_m = (1/M) sum_k cos(2 pi k m / M) / lam_k, which
// decay geometrically; kept while above 1e-18 c_0 (the whole period if that is shorter).
// Everything up to the entries is in long double: eigenvalues rounded to double would
// leave entries of about 1e-18 c_0 behind the decay, and the length to chance.  Offsets
// hi, hi - 1, ..: M a power of two; 65, 101, 135, 169 and 205 entries for degrees 1 to 5
// on a long enough period.
inline std::vector<double> inverse_row(int M, const std::vector<double> &mass, double dx, int &hi) {
    const long double PI = 3.14159265358979323846264338327950288L;
    const int d = (int)mass.size() / 2;
    // eigenvalues and cosines are even in k: half of them, the inner ones twice
    std::vector<long double> cs(M), inv(M / 2 + 1);
    for (int k = 0; k <= M / 2; ++k) cs[k] = cs[(M - k) & (M - 1)] = cosl(2 * PI * k / M);
    for (int k = 0; k <= M / 2; ++k) {
        long double lam = mass[d];
        for (int q = 1; q <= d; ++q) lam += 2 * (long double)mass[d + q] * cs[(k * q) & (M - 1)];
        inv[k] = (k == 0 || k == M / 2 ? 1.0L : 2.0L) / (lam * dx);
    }
    auto entry = [&](int m) {
        long double v = 0;
        for (int k = 0, i = 0; k <= M / 2; ++k, i = (i + m) & (M - 1)) v += inv[k] * cs[i];
        return (double)(v / M);
    };
    std::vector<double> half(1, entry(0));
    while ((int)half.size() < M / 2 && std::fabs(half.back()) > 1e-18 * half[0]) half.push_back(entry((int)half.size()));
    const bool whole = (int)half.size() >= M / 2;
    const int lo = whole ? M / 2 - 1 : (int)half.size() - 1;   // offsets -lo .. hi
    hi = whole ? M / 2 : lo;
    if (whole) half.resize(M / 2), half.push_back(entry(M / 2));
    std::vector<double> row(lo + hi + 1);
    for (int m = -lo; m <= hi; ++m) row[hi - m] = half[std::abs(m)];
    return row;
}

}  // namespace ecpic2d
