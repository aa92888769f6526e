// One part of the lookup's second kernel (HET_PART of HET_FILL_PARTS), see apply_variants.hip.
#include "cache_kernels.hpp"

namespace het {

static_assert(HET_PARTS == HET_FILL_PARTS, "the build compiles other parts than there are: kernels would be missing in the library");
#define HET_LISTED(part, ...) static_assert(part < HET_FILL_PARTS, "a part beyond the last");
HET_FILL_VARIANTS(HET_LISTED)
#undef HET_LISTED

#if HET_PART == 0
#define HET_PART_0(...) HET_FILL_KERNEL(__VA_ARGS__)
#else
#define HET_PART_0(...)
#endif
#if HET_PART == 1
#define HET_PART_1(...) HET_FILL_KERNEL(__VA_ARGS__)
#else
#define HET_PART_1(...)
#endif
#define HET_HERE(part, ...) HET_PART_##part(__VA_ARGS__)
HET_FILL_VARIANTS(HET_HERE)

} // namespace het
