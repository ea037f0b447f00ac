// The fused adjoint's instances that read click-pattern gradients (threshold
// detectors; arXiv 2602.11092, Sec. II-B) through the states' patterns, built
// in a translation unit of their own so that the standard instances' code does
// not change and the two compile in parallel.
#define SLOS_FUSED_CLICK_INSTANCES
#include "slos_fused.hip"
