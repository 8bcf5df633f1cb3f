// A run of Algorithm 1 in one launch (interact_run.hip, lsq_run.hip): what the host hands over.
#pragma once
#include "internal.h"
#include "objectives.h"

namespace swarm {

// One interaction of the run.  nodes: initiator | responder << 16; event: the interaction number that keys its
// random streams; flags: SEQ_HAS_DELTA, RUN_*, bits 8-15 = the initiator's number of local steps; turn:
// how many interactions of the run touch the initiator (low half) and the responder (high half) before this one; in
// least-squares runs how many interactions have ended, in the order of the descriptors, when the initiator's snapshot is there.
struct RunDesc {
    uint32_t nodes, event, flags, turn;
};
constexpr uint32_t RUN_LAST_OF_I = 2u, RUN_LAST_OF_J = 4u;        // no later interaction of the run touches the node
constexpr uint32_t RUN_SNAPSHOT_IS_MODEL = 8u;    // the node's interaction before this one was its own: Xhat_i = X_i
constexpr uint32_t RUN_SNAPSHOT_SHORT = 16u;      // so is the next one that touches it: nobody reads the snapshot
constexpr uint32_t RUN_LAST_LED = 32u;            // no later interaction of the run is the initiator's own
constexpr uint32_t RUN_READY_SHIFT = 16;          // bits 16-31: how many of the run's interactions the initiator has been through when its snapshot is there
constexpr uint32_t RUN_MAX_NODES = 78;            // two tiles of 256 coordinates (1 KiB per node) per compute unit of 160 KiB

#if defined(__HIPCC__)
// Descriptor k, or one of no consequence past the end.  Written before the launch and never by it: a scalar load.
__device__ __forceinline__ RunDesc run_desc(const RunDesc *descs, uint32_t k, uint32_t count) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const u4 v = ((const __attribute__((address_space(4))) u4 *)descs)[k < count ? k : 0u];
    return RunDesc{first_lane(v.x), first_lane(v.y), first_lane(v.z), first_lane(v.w)};
}
#endif

struct RunArgs {
    GossipArgs g;
    const RunDesc *descs;     // device: in an order in which every interaction follows those it depends on
    uint32_t count;           // at most 65535, so that `turn` holds
    const float *A, *C;       // n x d objective data (LOCAL only)
    float sigma, lr;
};

// Whether launch_interact_run is sooner done than a launch per level (H: mean number of local steps, 0 without).
bool interact_run_pays(uint64_t d, uint32_t n, uint32_t H, uint32_t m, uint32_t levels);
// local: take the initiators' local steps of this diagonal objective in registers, or null.
hipError_t launch_interact_run(const GossipArgs &g, uint32_t bits, const RunDesc *descs_dev, uint32_t count,
                               const DiagObjective *local, float lr, hipStream_t st);

// The same for small least-squares swarms (those whose objective has words to exchange, LsqObjective::run_part), steps
// included: descs_dev, or the single interaction `one` when it is null.  total_steps: of all interactions together.
hipError_t launch_lsq_run(const GossipArgs &g, uint32_t bits, const RunDesc *descs_dev, RunDesc one, uint32_t count,
                          uint32_t total_steps, LsqObjective &o, float lr, hipStream_t st);
bool lsq_run_fits(uint64_t d, uint32_t n, uint32_t batch);
size_t lsq_run_bytes(uint64_t d, uint32_t batch);

}  // namespace swarm
