// The count kernel's variants whose search stacks are in LDS (k <= 12).
#define CITRON_COUNT_UNIT kStackLds
#include "kernels_count.hip"
