// Host build of the factor of a cell's Gramian (cell_factor.hpp), by one thread.  Test infrastructure only.
#define BEM_HD
#include <cmath>
#include <cstdint>

#include "../../paper_2602_05492_amd/csrc/cell_factor.hpp"

namespace {
using namespace bem;

struct OneThread {
    static constexpr int t = 0, n = 1;
    void sync() const {}
    int largest(const double (*A)[kFactorNodes + 1], const int* step) const
    {
        int p = -1;
        for (int i = 0; i < kFactorNodes; ++i)
            if (step[i] < 0 && A[i][i] > 0.0 && (p < 0 || A[i][i] > A[p][p])) p = i;
        return p;
    }
};
}  // namespace

// Samples x [n][2] of the cell [-1, 1]^2; R [node][k], C [k][ab]
extern "C" void hm_cell_factor(const double* x, int64_t n, double* R, double* C)
{
    static CellFactor w;
    for (double& m : w.mu) m = 0.0;
    for (int64_t i = 0; i < n; ++i) {
        double T[2][kMom];
        for (int d = 0; d < 2; ++d) {
            T[d][0] = 1.0;
            T[d][1] = x[2 * i + d];
            for (int k = 2; k < kMom; ++k) T[d][k] = 2.0 * T[d][1] * T[d][k - 1] - T[d][k - 2];
        }
        for (int q = 0; q < kMom; ++q)
            for (int p = 0; p < kMom; ++p) w.mu[q * kMom + p] += T[0][p] * T[1][q];
    }
    const int Q = kFactorSide;
    for (int a = 0; a < Q; ++a)
        for (int i = 0; i < Q; ++i) w.d[a][i] = std::cos(a * (2 * i + 1) * kPi / (2 * Q)) * (a == 0 ? 1.0 / Q : 2.0 / Q);
    cell_factor(OneThread{}, w);
    for (int i = 0; i < kFactorNodes; ++i)
        for (int k = 0; k < kFactorNodes; ++k) {
            R[i * kFactorNodes + k] = w.R[i][k];
            C[i * kFactorNodes + k] = w.A[i][k];
        }
}
extern "C" double hm_pivot_floor() { return kPivotFloor; }
