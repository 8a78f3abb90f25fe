// Host-side declarations shared by the library's translation units.
#pragma once

#include <string>
#include <vector>

#include "../../include/wfstdec.h"
#include "wd_common.h"

struct wd_graph {
  wd::DevGraph dg;
  int32_t S = 0;
  int64_t A = 0;
  uint64_t Ae = 0, Ax = 0;
  uint32_t nlevels = 0;
  uint32_t P = 0;
  std::vector<uint32_t> level_base;  // host copy, nlevels + 1 entries
  size_t bytes = 0;
};

namespace wd {

void set_error(const std::string& msg);
wd_status fail(wd_status st, const std::string& msg);
wd_status hip_check(hipError_t e, const char* what);

// The frames received and not decoded yet, of at most `frames` each.
void launch_forward(const DevGraph& g, const LaneDesc* lanes, int B, int frames, const Params& prm,
                    const uint32_t* bad, hipStream_t s);
// Lattice links of one-workgroup decodes, from the node store, after the
// forward pass (all frames at once); before launch_lattice.
void launch_links(const DevGraph& g, const LaneDesc* lanes, int B, const Params& prm, hipStream_t s);
// Backward pruning sweep over the live nodes only, for the utterances that
// sparse_lane chooses; before launch_links, which then forms their kept links.
void launch_sweep(const DevGraph& g, const LaneDesc* lanes, int B, const Params& prm, hipStream_t s);
void launch_lattice(const DevGraph& g, const LaneDesc* lanes, int B, const Params& prm, hipStream_t s);
// The control block of an utterance's workgroup cluster.
size_t cluster_ctl_bytes();
// Workgroups of a launch of B leaders that brings helpers: one per CU in all.
int cluster_grid(int B);
size_t grid_lane_bytes();
// Chip-wide forward pass in three steps, so that a stream can decode frames as
// they arrive: begin (per-utterance state), frames t_from..t_to (any number of
// calls, in order), end.
void grid_begin(const LaneDesc* lanes, void* grid, int B, const uint32_t* bad, hipStream_t s);
void grid_frames(const DevGraph& g, const LaneDesc* lanes, void* grid, int B, const Params& prm, const uint32_t* bad,
                 int t_from, int t_to, hipStream_t s);
void grid_end(const LaneDesc* lanes, void* grid, int B, hipStream_t s);
void launch_grid_sweep(const DevGraph& g, const LaneDesc* lanes, void* grid, int B, int maxT, const Params& prm,
                       hipStream_t s);
void launch_grid_nodes(const LaneDesc* lanes, void* grid, int B, hipStream_t s);
void launch_check_loglikes(const LaneDesc* lanes, int B, uint32_t P, uint32_t* bad, hipStream_t s);
// Packs the links, nodes and words of every finished lane into dst (device),
// lane after lane, each lane's part 16-byte aligned.
void launch_pack_results(const LaneDesc* lanes, int B, void* dst, hipStream_t s);
// Sets T, t0 and open of lanes[0..B) (streaming) from host values passed as
// kernel arguments.
void launch_set_frames(LaneDesc* lanes, int B, const int32_t* T, const int32_t* t0, int32_t open, hipStream_t s);
// Resets what a decode reads before writing (launch_set_frames resets the
// cluster headers again for a stream's advances).
void launch_setup(const LaneDesc* lanes, int B, uint32_t* bad, uint64_t used_words, uint64_t S, uint64_t bitmap_words,
                  bool chip, hipStream_t s);

inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

}  // namespace wd
