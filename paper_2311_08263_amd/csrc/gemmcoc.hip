// The column-owner GEMM (gemmco_k.h) over coded weights; a file of its own because its kernels take as long to compile as the
// others together.
#include "gemmco_k.h"

hipError_t fc_gemmco_coded(int epi, const GemmCoArgs& a, int G, hipStream_t st) { return launch_co<WCoded>(epi, a, G, st); }
