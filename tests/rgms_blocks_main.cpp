// Rows of Y per block and columns per pass of RGMS (csrc/rgms_blocks.h, compiled alone), for test_rgms_blocks.py.
//   waves: reads lines "kind ordered workgroups tiles_each" and prints the wavefronts of a workgroup (kind 1: a large block, 2: large matrices W[r])
//   otherwise reads lines "n_rows n_rel nnz workspace" and prints "rows columns power columns_of_power" of each: the block's rows, the columns beside
//   them, the power of two that the rule on entries names, and the columns beside that
#include <stdio.h>

#include "rgms_blocks.h"

int main(int argc, char**) {
  long long n_rows, n_rel, nnz;
  int workspace;
  if (argc > 1) {
    while (scanf("%lld %lld %lld %d", &n_rows, &n_rel, &nnz, &workspace) == 4)
      printf("%d\n", sptir::wavefronts_per_workgroup(n_rows == 1, n_rows == 2, nnz, workspace, n_rel != 0));
    return 0;
  }
  while (scanf("%lld %lld %lld %d", &n_rows, &n_rel, &nnz, &workspace) == 4) {
    const int32_t rows = sptir::rows_of_a_block(n_rows, n_rel, nnz, workspace != 0);
    const int32_t power = 1 << sptir::log2_block_rows(n_rows, n_rel, nnz, workspace != 0);
    printf("%d %d %d %d\n", rows, sptir::columns_beside(rows), power, sptir::columns_beside(power));
  }
  return 0;
}
