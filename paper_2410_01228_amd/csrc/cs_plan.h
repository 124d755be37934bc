// The launch plans of the attention call and the host functions around them that more than one file
// uses (cs_api.hip makes the plans; cs_run_layers.hip runs them over several layers at a time).
#pragma once
#include "cs_common.h"

namespace cs {

// How a batch with both kinds of work is launched (see cs_mixed.hip): as two kernels in a row, as
// one grid with the decode pairs behind the tiles, or as one grid with a decode workgroup per CU
// beside the tiles.  mode: cs_set_mixed_fusion's (0 never fuse, 1 choose, 2 always behind, 3
// always beside).
struct FusePlan {
    int32_t arrangement;       // 0 two kernels, 1 decode behind the tiles, 2 decode beside the tiles
    int32_t prio;              // 0, or the higher of the two issue priorities the tiles alternate between (1, 2)
    int32_t persistent_wgs;    // arrangement 2: decode workgroups (one per CU)
};

struct Plans {
    DecodePlan d;
    PrefillPlan p;
    FusePlan f;
    size_t decode_bytes, need;     // workspace: the decode side's, all of it
};

// The plan of a batch for launches of `layers` layers each (remembered per thread; the reference is
// good until the thread asks for six more).  Sequences and tiles are cut as for one layer, whatever
// `layers` is: how many layers share a launch changes no bit of their results.
const Plans& plans_for(const cs_batch* b, int32_t Hq, int32_t Hkv, int32_t D, int32_t layers = 1);

// The workspace a launch of `layers` layers may need: at least plans_for(..., layers).need, without making
// that plan; nothing where one layer needs nothing.
size_t workspace_for_layers(const cs_batch* b, int32_t Hq, int32_t Hkv, int32_t D, int32_t layers);

int attention_shape_ok(int32_t Hq, int32_t Hkv, int32_t D);

// The first num_online_seqs sequences of a batch over the same arrays (what is left of an
// iteration once it is preempted: paper Sec. 4.3).
cs_batch online_prefix(const cs_batch& b, int32_t num_online_seqs);

int attention_mixed(const cs_kv_pool* pool, int32_t layer, const cs_batch* batch,
                    const void* q, void* out, int32_t Hq, float softmax_scale,
                    void* workspace, size_t workspace_bytes, void* stream, bool f16);

}  // namespace cs
