// Prints what make_plan decides for shapes read from stdin, one "G H_kv H_q d_h r_k r_v L k batch dtype" a line, as
// name=value pairs.  Linked with the library's objects by tests/test_plan.py; host only.
#include <cstdio>

#include "xkv_common.h"

int main()
{
    xkv_shape s{};
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d", &s.G, &s.H_kv, &s.H_q, &s.d_h, &s.r_k, &s.r_v, &s.L, &s.k, &s.batch,
                      &s.dtype) == 10) {
        xkv::Plan p;
        if (xkv::make_plan(s, p) != XKV_OK) return 1;
        std::printf("absorb=%d occ=%d splits=%d chunk=%d lds=%d max_splits=%d sr_splits=%d merge_limit=%d tail_parts=%d "
                    "absorbed=%d absorbed_q4=%d kept_0=%d kept_4=%d kept_3=%d regs_0=%d regs_4=%d regs_3=%d waves=%d ak_splits=%d ak_chunk=%d "
                    "stream=%d score_tpw=%d score_hist=%d topk_row=%d topk_chunk=%d factor_kept=%d\n", (int)p.absorb,
                    p.ab_occ, p.ab_splits, p.ab_chunk, (int)p.ab_lds, p.max_splits, p.sr_splits, xkv::kMaxCombineParts, xkv::kTailParts,
                    (int)(p.absorb && xkv::absorbed_mfma_pays(s, false)), (int)(p.absorb && xkv::absorbed_mfma_pays(s, true)),
                    (int)p.rope_kept[0], (int)p.rope_kept[1], (int)p.rope_kept[2], (int)p.rope_regs[0], (int)p.rope_regs[1],
                    (int)p.rope_regs[2], p.ga_waves, p.ak_splits, p.ak_chunk,
                    (int)p.score_stream, p.score_tpw, (int)p.score_hist, (int)p.topk_row, p.topk_chunk,
                    (int)xkv::reconstruct_keeps_factor(s, s.r_k));
    }
    return 0;
}
