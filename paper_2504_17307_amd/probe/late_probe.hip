// Measurement and test aid, not part of the product: the kernels of group_probe.hip with a first workgroup that comes late.
#define UCCL_GROUP_LEADS 2
#define UCCL_PROBE(name) name##_late
#include "group_probe.hip"
