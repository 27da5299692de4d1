// Arguments shared by the coarse-solve kernels.
#pragma once
#include "common.h"

namespace stomsfem {

struct CoarseArgs {
  int32_t ncx, ncy;
  int64_t nsamples;
  const double* S;
  const double* load;
  double* U;
  int32_t* status;
  double* work;  // nsamples * (nU * (ncx+1) + 1) doubles (one launch's samples)
};

// Symmetric systems with 4 <= ncx <= 32 (coarse_rows.hip): the forward and
// backward pass of the samples of `a`.
bool coarse_rows_supports(int ncx);
hipError_t launch_coarse_rows(const CoarseArgs& a, hipStream_t st);

}  // namespace stomsfem
