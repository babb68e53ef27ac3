// The small integer arrays a call hands to its kernels (offsets, counts): by value in the kernel's arguments when they
// fit, else from the context's device plan buffer.
#ifndef OTAS_PLAN_ARGS_H_
#define OTAS_PLAN_ARGS_H_

#include <cstring>

#include "kernels.h"

namespace otas {

// In a kernel's arguments.  A copy to the device buffer costs a launch of
// its own (4 - 6 us on the GPU and, with the event that guards the staging slot, about 10 us on the host), which for the
// calls that launch one or two kernels is a third of the call: otas_token_merge of 64 queries of 197 tokens, back to
// back, 32.6 us with the copy, 25.3 without (MI355X).
struct ArgInts {
  int32_t v[kArgInts];
  __device__ int32_t operator[](int i) const { return v[i]; }
};
struct DevInts {
  const int32_t* p;
  __device__ int32_t operator[](int i) const { return p[i]; }
};

// f(ArgInts) or f(DevInts), whichever plan_in_args picked.
template <typename F>
inline hipError_t with_plan(const int32_t* plan, size_t count, const int32_t* d_plan, F f) {
  if (!plan_in_args(count)) return f(DevInts{d_plan});
  ArgInts a;
  std::memcpy(a.v, plan, count * sizeof(int32_t));
  return f(a);
}

}  // namespace otas
#endif  // OTAS_PLAN_ARGS_H_
