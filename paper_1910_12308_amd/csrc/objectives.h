// Node objectives: borrowed data pointers, workspaces and the local-step launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swarm {

struct DiagObjective { const float *a; const float *c; float sigma; };

constexpr uint32_t LSQ_MAX_BATCH = 64;
struct LsqTeams;
struct LsqObjective {
    const float *A = nullptr;    // n x m_rows x d
    const float *b = nullptr;    // n x m_rows
    uint32_t m_rows = 0, batch = 0;
    // split form (small swarms): tagged partial residuals exchanged between the workgroups of a node
    // (owned; null when the wide form is used)
    unsigned long long *part = nullptr;
    size_t part_bytes = 0;
    uint32_t launches = 0;          // launches of the split form so far (24 bits, tags the exchanged words)
    // runs of Algorithm 1 in one launch: words its waves exchange (owned; null when the swarm does not fit that form) and
    // the tag of the next step
    unsigned long long *run_part = nullptr;
    size_t run_part_bytes = 0;
    uint32_t run_tag = 0;
    // wide form (all other swarms): partial residuals, two steps' worth of wide_rows x LSQ_MAX_BATCH (owned),
    // wide_rows = nodes x wide_slices
    float *wide_part = nullptr;
    uint64_t wide_rows = 0;
    uint32_t wide_slices = 0;
    bool by_rows = false;           // wide form with a wave per row of the batch instead
    // teams of workgroups (lsq_team.hip), where these are the better form; not for steps that update the models themselves
    LsqTeams *teams = nullptr;
    unsigned long long patience = 2000000;        // 100 MHz ticks a workgroup waits for the others of its team: 20 ms
};

struct MlpSplitSpace;
struct MlpObjective {
    uint32_t n_in = 0, n_hid = 0, n_out = 0, batch = 0;
    const float *means = nullptr;   // n_out x n_in
    const float *cdf = nullptr;     // n x n_out
    float data_sigma = 0.f;
    // workspace for all nodes (owned): inputs, labels, hidden activations, logits gradient, hidden gradient; the bf16x3 steps keep
    // packed operands in x, hid, dhid and dlogits
    float *x = nullptr, *hid = nullptr, *dlogits = nullptr, *dhid = nullptr;
    uint32_t *labels = nullptr;
    uint32_t n_nodes = 0;
    bool bf16x3 = false;            // products as three bf16 products per term instead of float32 matrix instructions
    MlpSplitSpace *split = nullptr; // their workspace (owned), there while they are chosen
};

// Whole round in one pass (local steps + quantized gossip) for the diagonal objective; bits in {2,4,8,16}.
struct GossipArgs;
hipError_t launch_fused_pairs(const GossipArgs &g, const DiagObjective &o, uint32_t bits, bool inplace, uint32_t H,
                              float lr, int stale_mode, uint32_t npairs, hipStream_t st);
hipError_t launch_fused_singles(const GossipArgs &g, const DiagObjective &o, uint32_t bits, bool inplace, uint32_t H,
                                float lr, uint32_t nsingles, hipStream_t st);

struct LocalSlots;
struct DeviceCounters;
struct SeqDesc;
// Allocates the exchange buffers of the split form when ceil(d / 512) * n workgroups are few enough to be
// resident together (they wait for one another inside the kernel), and with merge_runs also those of the form that takes
// a run of Algorithm 1 in one launch (lsq_run_fits).
hipError_t alloc_lsq(LsqObjective &o, uint64_t d, uint32_t n, uint32_t H, bool merge_runs);
hipError_t launch_local_lsq(const float *base, float *W, LsqObjective &o, const LocalSlots &slots,
                            DeviceCounters *counters, uint32_t count, uint64_t d, uint32_t H, float lr, uint64_t seed,
                            uint32_t event, hipStream_t st);
// Steps of Algorithm 1 on disjoint nodes in one kernel (split form only): each initiator's local steps
// (count taken from its descriptor) from its snapshot, then its interaction.  descs_dev, or the single interaction
// `one` when it is null.
hipError_t launch_lsq_interact(const GossipArgs &g, uint32_t bits, const SeqDesc *descs_dev, const SeqDesc &one, uint32_t count,
                               LsqObjective &o, float lr, hipStream_t st);
void free_lsq(LsqObjective &o);
void alloc_lsq_teams(LsqObjective &o, uint64_t d, uint32_t n, bool at_once);
void free_lsq_teams(LsqObjective &o);
hipError_t launch_lsq_teams(const float *base, float *W, const LsqObjective &o, const LocalSlots &slots, DeviceCounters *counters,
                            uint32_t count, uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event, hipStream_t st);

hipError_t alloc_mlp(MlpObjective &o, uint32_t n_nodes);
void free_mlp(MlpObjective &o);
hipError_t launch_local_mlp(const float *base, float *W, const MlpObjective &o, const LocalSlots &slots,
                            uint32_t count, uint32_t n, uint64_t d, uint32_t H, float lr, uint64_t seed,
                            uint32_t event, hipStream_t st);
// The same with bf16x3 products; alloc_mlp_split is called when they are chosen and does nothing a second time, free_mlp_split when
// they no longer are.
hipError_t alloc_mlp_split(MlpObjective &o);
void free_mlp_split(MlpObjective &o);
hipError_t launch_local_mlp_split(const float *base, float *W, const MlpObjective &o, const LocalSlots &slots, uint32_t count,
                                  uint64_t d, uint32_t H, float lr, uint64_t seed, uint32_t event, hipStream_t st);

}  // namespace swarm
