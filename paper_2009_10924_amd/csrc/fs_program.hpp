// An explored program: the fusion plan of a multi-pattern graph, made executable (built by fs_explore.cpp, run by
// fs_program.cpp).
#pragma once

#include <vector>

#include "fs_internal.hpp"

extern "C" {
void fs_plan_destroy(fs_plan* p);
void fs_pack_destroy(fs_pack* p);
}

using namespace fs;

constexpr size_t kMergedMaxOperands = 256;   // 2 KB of kernel arguments

struct fs_program {
  struct Step {
    std::vector<int> ops;               // graph op indices
    double f = 0;                       // delta-evaluator gain (microseconds), 0 for a single op
    fs_plan* plan = nullptr;
    std::vector<BufRef> in, out;        // where each plan input / output lives: graph input, graph output or workspace offset
    int64_t plan_ws_offset = 0;
    int32_t pack = -1;                  // index into packs, -1 = runs on its own
    size_t own_launches = 0;            // launches of the plan issued at the step itself (the rest are joint folds)
    int32_t stage = 0;                  // external computations that must have run before it (longest chain of them)
  };
  struct JointFold { int step; size_t launch; };   // a K_COLFOLD launch of a step's plan, issued after the last step
  struct Pack {
    fs_pack* pack = nullptr;
    std::vector<int> steps;
  };
  std::vector<Step> steps;              // dependence order
  std::vector<Pack> packs;
  std::vector<std::vector<JointFold>> joint_folds;   // one launch each, at most kFoldManyMax folds in it
  // the last step's kernel carries the joint folds along (see carry_folds): they have no launch of their own
  struct Carrier {
    int step = -1;
    std::shared_ptr<GenKernel> kernel;
    LaunchShape shape;
  } carrier;
  // The whole program in fewer launches than step by step: each one kernel over steps (and folds of earlier ones' column sums)
  // that do not depend on each other (see merge_steps).  Empty: none, the steps run one by one.
  struct Merged {
    std::vector<int> steps;
    std::vector<JointFold> folds;
    struct Operand { int step; BufRef ref; };   // of one of the step's launches
    std::vector<Operand> operands;              // in the order of the kernel's parameters
    std::string entry;                          // the kernel's name
    std::shared_ptr<GenKernel> kernel;
    LaunchShape shape;
  };
  std::vector<Merged> merged;
  std::vector<int64_t> input_bytes, output_bytes;
  fs_program_info info{};
  int32_t n_inputs = 0, n_outputs = 0;
  ~fs_program() {
    for (Step& s : steps) fs_plan_destroy(s.plan);
    for (Pack& p : packs) fs_pack_destroy(p.pack);
  }
};
