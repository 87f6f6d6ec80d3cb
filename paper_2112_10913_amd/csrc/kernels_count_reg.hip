// The count kernel's variants whose light stacks are four levels of registers
// (k = 7..9).
#define CITRON_COUNT_UNIT kStackReg
#include "kernels_count.hip"
