// Compensated FP64 sums (Neumaier) shared by the reductions.
#pragma once
#include <hip/hip_runtime.h>

namespace qs {

struct Acc {
  double s, c;
};

__device__ __forceinline__ void nadd(Acc& a, double x) {
  const double t = a.s + x;
  if (fabs(a.s) >= fabs(x))
    a.c += (a.s - t) + x;
  else
    a.c += (x - t) + a.s;
  a.s = t;
}
__device__ __forceinline__ Acc ncombine(Acc a, const Acc& b) {
  nadd(a, b.s);
  a.c += b.c;
  return a;
}

}  // namespace qs
