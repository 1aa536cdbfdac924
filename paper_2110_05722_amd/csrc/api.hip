// Entry points that launch nothing: workspace sizing and status names.
#include "host.hpp"

extern "C" size_t lsq_workspace_bytes(int32_t op, int64_t rows, int32_t cols)
{
    using namespace lsq;
    if (rows <= 0 || cols <= 0) return 0;
    switch (op) {
        case LSQ_OP_LAYERNORM_BWD:
            // one [2][cols] fp32 partial row (dgamma, dbeta) per workgroup
            return ln_bwd_bytes(rows, cols, 2);
        case LSQ_OP_BDR_LAYERNORM_BWD:
            // one [3][cols] fp32 partial row (dgamma, dbeta, dbias) per workgroup; also enough for the
            // two separate operators that serve row lengths without a register bucket
            {
                const size_t fused = ln_bwd_bytes(rows, cols, 3), apart = bdr_bwd_bytes_upto(rows, cols);
                return fused > apart ? fused : apart;
            }
        // one [cols] fp32 partial row (dbias) per row block, or per workgroup of the flat walk
        case LSQ_OP_BIAS_DROPOUT_RESIDUAL_BWD: return bdr_bwd_bytes_upto(rows, cols);
        case LSQ_OP_BIAS_ACT_DROPOUT_BWD: return bad_bwd_bytes_upto(rows, cols);
        case LSQ_OP_SPLIT_HEADS_BWD: return heads_bwd_bytes_upto(rows, cols);
        case LSQ_OP_EMBEDDING_BWD:
            // sorted order, the sort's second buffer and digit counts, the partial rows of long calls
            return emb_bwd_plan(rows, cols).total();
        default:
            return 0;
    }
}

extern "C" const char* lsq_status_string(lsq_status s)
{
    switch (s) {
        case LSQ_OK: return "LSQ_OK";
        case LSQ_INVALID_ARG: return "LSQ_INVALID_ARG";
        case LSQ_UNSUPPORTED_DTYPE: return "LSQ_UNSUPPORTED_DTYPE";
        case LSQ_MISALIGNED: return "LSQ_MISALIGNED";
        case LSQ_WORKSPACE_TOO_SMALL: return "LSQ_WORKSPACE_TOO_SMALL";
        case LSQ_LAUNCH_FAILED: return "LSQ_LAUNCH_FAILED";
        default: return "LSQ_UNKNOWN_STATUS";
    }
}
