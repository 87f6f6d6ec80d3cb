// The count kernel's variants whose light stacks are two levels of registers
// (k = 7).
#define CITRON_COUNT_UNIT kStackReg
#include "kernels_count.hip"
