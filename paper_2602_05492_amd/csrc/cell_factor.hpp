// cell_factor.hpp - the factor of a cell's Gramian in the normal equations over cells (jtj_cells.hip).
//
// With Phi [64][n] the interpolation weights of a cell's n samples, G = Phi Phi^T = D^T M D, M the Gramian of the products
// T_a(xi) T_b(eta) and D the nodes' Chebyshev coefficients.  cell_factor gives R and C with R R^T = G and R Q = Phi for
// Q = C T(x), both to rounding, whatever the samples: fewer than nodes, in a corner, in a strip, along a line.  G is
// singular to rounding then, so the elimination takes the largest remaining diagonal entry as its pivot and stops at the
// first below kPivotFloor of the largest; the columns of R and the rows of C beyond stay zero.  (In node order, skipping
// small pivots, the Schur complement is multiplied up by pivots that are rounding: R R^T was off by up to 110 times G.)
// Over 4,000 cells of 1 to 400 samples of those kinds: R R^T - G up to 1.0e-13 of the largest entry of G,
// R Q - Phi up to 1.8e-6 (what the floor leaves out: its square root times the samples' share), |Q| <= 1.
//
// A template over the threads that share the work, so that the same code runs in a workgroup and in host-side unit tests.
#pragma once

#include "seg_math.hpp"

namespace bem {

constexpr int kFactorSide = 8, kFactorNodes = kFactorSide * kFactorSide;
constexpr int kMom = 16;                       // moments a side (15 used)
// of the largest diagonal entry: far above G's rounding (1e-15 of it), its square root below the features' 22 bits a
// sample of a cell at the floor
constexpr double kPivotFloor = 1e-13;

// rows padded by one against bank conflicts
struct CellFactor {
    double A[kFactorNodes][kFactorNodes + 1];       // working matrix, then C [k][ab]
    double R[kFactorNodes][kFactorNodes + 1];       // [node][k]
    double mu[kMom * kMom];                         // in: mu[q kMom + p] = sum T_p(xi) T_q(eta)
    double d[kFactorSide][kFactorSide];             // in: d[a][i] = s_a T_a(t_i)
    double inv[kFactorNodes];                       // 1 / R[node[k]][k]
    int node[kFactorNodes], step[kFactorNodes];     // node of step k; step of a node, or -1
};

// Team: t of n threads, sync(), and largest(A, step): the node of the largest positive A[i][i] among those with
// step[i] < 0 (-1: none), the same in every thread.  Nodes and products: node (i, j) is j 8 + i, T_a T_b is b 8 + a.
template <class Team>
BEM_HD inline void cell_factor(const Team& tm, CellFactor& w)
{
    constexpr int Q = kFactorSide, NN = kFactorNodes;
    double(*A)[NN + 1] = w.A, (*R)[NN + 1] = w.R;
    // T_a T_a' is the mean of T_{a + a'} and T_{|a - a'|}
    for (int e = tm.t; e < NN * NN; e += tm.n) {
        const int r = e / NN, q = e % NN;
        const int a = r % Q, b = r / Q, a2 = q % Q, b2 = q / Q;
        const int ad = a > a2 ? a - a2 : a2 - a, bd = b > b2 ? b - b2 : b2 - b;
        A[r][q] = 0.25 * ((w.mu[(b + b2) * kMom + a + a2] + w.mu[(b + b2) * kMom + ad]) +
                          (w.mu[bd * kMom + a + a2] + w.mu[bd * kMom + ad]));
    }
    tm.sync();
    // the four index transforms a -> i, b -> j, a' -> i', b' -> j'
    for (int e = tm.t; e < NN * NN; e += tm.n) {
        const int r = e / NN, q = e % NN, i = r % Q, b = r / Q;
        double v = 0.0;
        for (int a = 0; a < Q; ++a) v += w.d[a][i] * A[b * Q + a][q];
        R[r][q] = v;
    }
    tm.sync();
    for (int e = tm.t; e < NN * NN; e += tm.n) {
        const int r = e / NN, q = e % NN, i = r % Q, j = r / Q;
        double v = 0.0;
        for (int b = 0; b < Q; ++b) v += w.d[b][j] * R[b * Q + i][q];
        A[r][q] = v;
    }
    tm.sync();
    for (int e = tm.t; e < NN * NN; e += tm.n) {
        const int r = e / NN, q = e % NN, i = q % Q, b = q / Q;
        double v = 0.0;
        for (int a = 0; a < Q; ++a) v += w.d[a][i] * A[r][b * Q + a];
        R[r][q] = v;
    }
    tm.sync();
    for (int e = tm.t; e < NN * NN; e += tm.n) {
        const int r = e / NN, q = e % NN, i = q % Q, j = q / Q;
        double v = 0.0;
        for (int b = 0; b < Q; ++b) v += w.d[b][j] * R[r][b * Q + i];
        A[r][q] = v;
    }
    for (int i = tm.t; i < NN; i += tm.n) w.step[i] = -1;
    tm.sync();
    // R by columns, right-looking on the whole matrix (an eliminated node's entries of R are zero from then on)
    double floor = 0.0;
    int rank = 0;
    for (; rank < NN; ++rank) {
        const int p = tm.largest(A, w.step);
        if (p < 0) break;
        const double piv = A[p][p];
        if (rank == 0) floor = kPivotFloor * piv;
        if (!(piv > floor)) break;
        const double inv = 1.0 / sqrt(piv);
        for (int i = tm.t; i < NN; i += tm.n) R[i][rank] = w.step[i] < 0 ? A[i][p] * inv : 0.0;
        tm.sync();
        if (tm.t == 0) {
            w.step[p] = rank;
            w.node[rank] = p;
            w.inv[rank] = inv;
        }
        for (int e = tm.t; e < NN * NN; e += tm.n) A[e / NN][e % NN] -= R[e / NN][rank] * R[e % NN][rank];
        tm.sync();
    }
    for (int e = tm.t; e < NN * (NN - rank); e += tm.n) R[e % NN][rank + e / NN] = 0.0;
    tm.sync();                                       // (A is C's from here on)
    // C = R^-1 D^T over the pivots' rows, column ab by forward substitution
    for (int t = tm.t; t < NN; t += tm.n) {
        const int a = t % Q, b = t / Q;
        for (int k = 0; k < rank; ++k) {
            const int n = w.node[k];
            double v = w.d[a][n % Q] * w.d[b][n / Q];
            for (int m = 0; m < k; ++m) v -= R[n][m] * A[m][t];
            A[k][t] = v * w.inv[k];
        }
        for (int k = rank; k < NN; ++k) A[k][t] = 0.0;
    }
    tm.sync();
}

}  // namespace bem
