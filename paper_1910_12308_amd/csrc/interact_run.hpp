// A run of Algorithm 1 in one launch (interact_run.hip): what the host hands over.
#pragma once
#include "internal.h"
#include "objectives.h"

namespace swarm {

// One interaction of the run.  nodes: initiator | responder << 16; event: the interaction number that keys its
// random streams; flags: SEQ_HAS_DELTA, RUN_*, bits 8-15 = the initiator's number of local steps; turn:
// how many interactions of the run touch the initiator (low half) and the responder (high half) before this one.
struct RunDesc {
    uint32_t nodes, event, flags, turn;
};
constexpr uint32_t RUN_LAST_OF_I = 2u, RUN_LAST_OF_J = 4u;        // no later interaction of the run touches the node
constexpr uint32_t RUN_SNAPSHOT_IS_MODEL = 8u;    // the node's interaction before this one was its own: Xhat_i = X_i
constexpr uint32_t RUN_SNAPSHOT_SHORT = 16u;      // so is the next one that touches it: nobody reads the snapshot
constexpr uint32_t RUN_MAX_NODES = 78;            // 2 KiB of local memory per node, 160 KiB per compute unit

struct RunArgs {
    GossipArgs g;
    const RunDesc *descs;     // device: in an order in which every interaction follows those it depends on
    uint32_t count;           // at most 65535, so that `turn` holds
    const float *A, *C;       // n x d objective data (LOCAL only)
    float sigma, lr;
};

// local: take the initiators' local steps of this diagonal objective in registers, or null.
hipError_t launch_interact_run(const GossipArgs &g, uint32_t bits, const RunDesc *descs_dev, uint32_t count,
                               const DiagObjective *local, float lr, hipStream_t st);

}  // namespace swarm
