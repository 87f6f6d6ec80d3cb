// The count kernel's variants whose search stacks are in device memory (k > 12).
#define CITRON_COUNT_UNIT kStackGlobal
#include "kernels_count.hip"
