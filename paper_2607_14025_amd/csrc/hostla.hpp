// Host work of the iterative eigensolvers (no GPU types): dense eigensolvers of their small projected matrices,
// cyclic Jacobi rotations for real symmetric and complex Hermitian matrices, and their random starts.
#pragma once
#include <complex>
#include <cstddef>
#include <random>
#include <vector>

namespace stern {

// Eigenvalues (ascending) and eigenvectors (columns of V, row-major n x n) of a real symmetric
// matrix A [n][n] (row-major).
void jacobi_eigh(std::vector<double> A, int n, std::vector<double>& w, std::vector<double>& V);
// The same for a complex Hermitian matrix.
void jacobi_zheev(std::vector<std::complex<double>> A, int n, std::vector<double>& w,
                  std::vector<std::complex<double>>& V);

// n standard normal deviates, by Marsaglia's polar method on the engine's words: the same values, bit for bit, as a fresh
// std::normal_distribution<double> gives. Starts of tens of millions of values are drawn in one go, and the library's
// function, called once per value, costs what its place in the binary makes it cost: on an EPYC host 36 ns a value at
// one alignment of the same instructions and 67 at another (a Davidson start of 34.6 million: 1.3 and 2.4 s). In a loop of its
// own: 6.6 ns at any alignment.
void fill_normal(std::mt19937_64& rng, double* x, std::size_t n);

}  // namespace stern
