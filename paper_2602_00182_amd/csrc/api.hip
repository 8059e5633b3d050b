// Library identification and per-thread error state.
#include <hip/hip_version.h>

#include "common.h"
#include "geometry.h"

namespace det {
static thread_local int g_last_hip_error = 0;
void set_last_hip_error(int e) { g_last_hip_error = e; }
}  // namespace det

#define DET_STR2(x) #x
#define DET_STR(x) DET_STR2(x)

extern "C" const char* det_fingerprint(void)
{
    return "libdetinfer gfx950 hip-" DET_STR(HIP_VERSION_MAJOR) "." DET_STR(HIP_VERSION_MINOR) "." DET_STR(
        HIP_VERSION_PATCH) " canon-2 gemm-16x16x32-k64"
        // launch geometry revision: which tile shapes and kernel forms the row count (GEMM), the batch
        // (attention) select.  They move no output byte, but a receipt pins them all the same, so a change of
        // what det_gemm_tile() or det_qgemm_tile() answers for any launch, or of the forms and grids the quantized GEMM and attention
        // take, is a new revision.
        " tiles-9(gemm:n256@rounds,n128@256wg,rowcut8,n64@m65|m64r64|m161,reads@m96|m192,norm-in-kernel@4rows;"
        "qgemm:few@" DET_STR(DET_QGEMM_FEW_ROWS) "rows,norm@" DET_STR(DET_QGEMM_NORM_ROWS) "rows,norm128@" DET_STR(
            DET_QGEMM_FEW_ROWS) "rows,mid@" DET_STR(DET_QGEMM_MID16_ROWS) "rows|" DET_STR(DET_QGEMM_MID32_ROWS) "rows,"
        "32x64+64x64@768wg,64x128;"
        "attn:chunk,rows8@" DET_STR(DET_ATTN_NAMED_ROWS) "rows,walk@" DET_STR(DET_ATTN_WALK_WGS) "wg,few@" DET_STR(
            DET_ATTN_FEW_PAIRS) "pairs,turn@" DET_STR(DET_ATTN_TURN_CHUNKS) "chunks)";
}

extern "C" int det_last_hip_error(void) { return det::g_last_hip_error; }
