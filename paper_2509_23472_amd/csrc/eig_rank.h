// Order of the eigenvalues of a positive semidefinite matrix.  Plain C++ (a constexpr function also runs
// on the device), so that it can be tested without a GPU.
#pragma once

// Rank of lam[i] among lam[0 .. l-1], descending, ties by index.  The ranks are a permutation of 0 .. l-1
// whatever the bits of lam are, because the results index other arrays: what is not positive counts
// as zero, and so does NaN (an activation with a NaN makes all of them NaN), which comparisons alone would
// give rank 0 everywhere.
constexpr int ej_rank_of(const double* lam, int l, int i) {
  const double vi = lam[i] > 0.0 ? lam[i] : 0.0;
  int rank = 0;
  for (int j = 0; j < l; ++j) {
    const double vj = lam[j] > 0.0 ? lam[j] : 0.0;
    rank += (vj > vi) || (vj == vi && j < i);
  }
  return rank;
}
