// Minimax polynomials of the direct inverse square root (k_isqrt.hip), formed
// once on the host (plain C++, shared with their test).
#pragma once
#include <algorithm>
#include <cmath>

#define ISQ_CLASSES 10     // spectral classes (largest kappa) with a plan each
#define ISQ_OPMAX 17       // products of the longest program

// Stage s: W_s (s = 0) or W_s - I (later stages) = sum_j b[s][j] X^j, X = (P - mid)/hw.
struct IsqClass {
    double kappa;
    int deg[3];
    double b[3][10], mid[3], hw[3];
};
struct IsqTable {
    IsqClass cls[ISQ_CLASSES];
};

typedef long double isq_ld;

// Coefficients b_0..b_d in X = (x - mid)/hw of the W of degree d with least
// max |1 - t W(t^2)| on t in [l, u], by the Remez exchange; returns the error.
// In extended precision: the last stages' errors are below FP64 rounding.
inline isq_ld isq_remez(isq_ld l, isq_ld u, int d, isq_ld* b, isq_ld* mid, isq_ld* hw) {
    const int n = d + 2, G = 1500;
    *mid = 0.5L * (l * l + u * u);
    *hw = 0.5L * (u * u - l * l);
    const isq_ld pi = 3.14159265358979323846264338327950288L;
    isq_ld t[16], A[16][17], x[16], res[1501];
    for (int i = 0; i < n; i++) t[i] = 0.5L * (l + u) - 0.5L * (u - l) * std::cos(pi * i / (n - 1));
    isq_ld E = 0.0L;
    for (int it = 0; it < 40; it++) {
        // t_i W(t_i^2) + (-1)^i E = 1 in the Chebyshev basis
        for (int i = 0; i < n; i++) {
            const isq_ld X = (t[i] * t[i] - *mid) / *hw;
            isq_ld t0 = 1.0L, t1 = X;
            for (int k = 0; k <= d; k++) {
                A[i][k] = t[i] * t0;
                const isq_ld t2 = 2.0L * X * t1 - t0;
                t0 = t1;
                t1 = t2;
            }
            A[i][d + 1] = (i & 1) ? -1.0L : 1.0L;
            A[i][n] = 1.0L;
        }
        for (int p = 0; p < n; p++) {
            int q = p;
            for (int r = p + 1; r < n; r++)
                if (std::fabs(A[r][p]) > std::fabs(A[q][p])) q = r;
            for (int k = 0; k <= n; k++) std::swap(A[p][k], A[q][k]);
            for (int r = p + 1; r < n; r++) {
                const isq_ld f = A[r][p] / A[p][p];
                for (int k = p; k <= n; k++) A[r][k] -= f * A[p][k];
            }
        }
        for (int p = n - 1; p >= 0; p--) {
            isq_ld s = A[p][n];
            for (int k = p + 1; k < n; k++) s -= A[p][k] * x[k];
            x[p] = s / A[p][p];
        }
        E = std::fabs(x[d + 1]);
        // new reference: the extremum of each run of equal sign
        isq_ld big = 0.0L, pts[17];
        int np = 0, start = 0;
        for (int g = 0; g <= G; g++) {
            const isq_ld tg = 0.5L * (l + u) - 0.5L * (u - l) * std::cos(pi * g / G);
            const isq_ld X = (tg * tg - *mid) / *hw;
            isq_ld t0 = 1.0L, t1 = X, s = 0.0L;
            for (int k = 0; k <= d; k++) {
                s += x[k] * t0;
                const isq_ld t2 = 2.0L * X * t1 - t0;
                t0 = t1;
                t1 = t2;
            }
            res[g] = 1.0L - tg * s;
        }
        for (int g = 1; g <= G + 1; g++) {
            if (g <= G && res[g] * res[g - 1] >= 0.0L) continue;
            int m = start;
            for (int k = start; k < g; k++)
                if (std::fabs(res[k]) > std::fabs(res[m])) m = k;
            if (np < 17) pts[np] = 0.5L * (l + u) - 0.5L * (u - l) * std::cos(pi * m / G);
            np++;
            big = std::max(big, std::fabs(res[m]));
            start = g;
        }
        if (np != n) break;  // rounding level: the error no longer alternates cleanly
        for (int i = 0; i < n; i++) t[i] = pts[i];
        if (big <= E * 1.002L) break;
    }
    // Chebyshev to monomial coefficients in X
    isq_ld Tk[2][16] = {{1.0L}, {0.0L, 1.0L}};
    for (int k = 0; k <= d; k++) b[k] = 0.0L;
    for (int k = 0; k <= d; k++) {
        isq_ld* cur = Tk[k & 1];
        if (k >= 2) {
            isq_ld nxt[16];
            for (int j = 0; j <= k; j++)
                nxt[j] = (j ? 2.0L * Tk[(k - 1) & 1][j - 1] : 0.0L) - (j <= k - 2 ? Tk[k & 1][j] : 0.0L);
            for (int j = 0; j <= k; j++) cur[j] = nxt[j];
        }
        for (int j = 0; j <= k; j++) b[j] += x[k] * cur[j];
    }
    return E;
}

// Stage degrees per largest kappa: the fewest products whose composed error
// stays below 1e-16, half a unit of FP64's last place (`kappa`), or below 6e-15
// (`wide`: for operands rounded to 46 bits).
inline IsqTable isq_build_table(bool wide) {
    static const struct { double kappa, wide; int deg[3]; } plan[ISQ_CLASSES] = {
        {5.4, 6.5, {4, 6, 0}},       {11.0, 14.0, {4, 9, 0}},     {22.0, 29.0, {6, 9, 0}},    {45.0, 60.0, {9, 9, 0}},
        {93.0, 125.0, {4, 4, 4}},    {200.0, 265.0, {4, 4, 6}},   {450.0, 600.0, {4, 4, 9}},  {930.0, 1200.0, {6, 4, 9}},
        {1850.0, 2400.0, {6, 6, 9}}, {3700.0, 4700.0, {6, 9, 9}},
    };
    IsqTable tab;
    for (int c = 0; c < ISQ_CLASSES; c++) {
        IsqClass& k = tab.cls[c];
        k.kappa = wide ? plan[c].wide : plan[c].kappa;
        isq_ld l = 1.0L / std::sqrt((isq_ld)k.kappa), u = 1.0L;
        for (int s = 0; s < 3; s++) {
            const int d = k.deg[s] = plan[c].deg[s];
            if (!d) break;
            isq_ld b[10], mid, hw;
            const isq_ld e = isq_remez(l, u, d, b, &mid, &hw);
            if (s) b[0] -= 1.0L;
            for (int j = 0; j <= d; j++) k.b[s][j] = (double)b[j];
            k.mid[s] = (double)mid;
            k.hw[s] = (double)hw;
            // the next stage's interval, a little wider than the error left
            l = 1.0L - 1.05L * e - 1e-12L;
            u = 1.0L + 1.05L * e + 1e-12L;
        }
    }
    return tab;
}
