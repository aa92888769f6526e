// One part of the update's kernels (HET_PART of HET_APPLY_PARTS): the library's longest compilation, cut to run side by side.
#include "cache_kernels.hpp"

namespace het {

static_assert(HET_PARTS == HET_APPLY_PARTS, "the build compiles other parts than there are: kernels would be missing in the library");
#define HET_LISTED(part, ...) static_assert(part < HET_APPLY_PARTS, "a part beyond the last");
HET_APPLY_VARIANTS(HET_LISTED)
#undef HET_LISTED

#if HET_PART == 0
#define HET_PART_0(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_0(...)
#endif
#if HET_PART == 1
#define HET_PART_1(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_1(...)
#endif
#if HET_PART == 2
#define HET_PART_2(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_2(...)
#endif
#if HET_PART == 3
#define HET_PART_3(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_3(...)
#endif
#if HET_PART == 4
#define HET_PART_4(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_4(...)
#endif
#if HET_PART == 5
#define HET_PART_5(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_5(...)
#endif
#if HET_PART == 6
#define HET_PART_6(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_6(...)
#endif
#if HET_PART == 7
#define HET_PART_7(...) HET_APPLY_KERNEL(__VA_ARGS__)
#else
#define HET_PART_7(...)
#endif
#define HET_HERE(part, ...) HET_PART_##part(__VA_ARGS__)
HET_APPLY_VARIANTS(HET_HERE)

} // namespace het
