// The decoder pass of a small model over a few rows in one launch (kernels_relay.hip): layers whose weights are a few megabytes, so
// that a launch per step costs more than the step.
#pragma once
#include "common.h"

namespace mtad {

constexpr int RELAY_MAX_LAYERS = 48;  // weight pointers travel in the kernel arguments; below 63 (tags)
constexpr int RELAY_MAX_ROWS = 8;     // rows of a pass, all sequences together
constexpr int RELAY_MAX_SPLITS = 8;   // key splits of an attention unit
constexpr int RELAY_MAX_GROUPS = 512;  // workgroups

// Steps of a layer; the units of a step are numbered, unit u of step s belongs to workgroup (first[s] + u) % (workgroups).
enum : int { RS_QKV = 0, RS_ATTN = 1, RS_O = 2, RS_GU = 3, RS_DOWN = 4, RS_STEPS = 5 };

// What workgroups hand to each other: 8-byte words (tag << 32 | 32 bits of payload), written and read whole.  A word is there when its
// tag is the one of this pass and layer.  Two layers' words alternate (a step's words are written again two layers later, which
// takes every reader's own results of the layer between); the second copy of all of them is for a pass that starts over.
struct RelayMail {
  uint64_t* words;
  int qkv, att, part, hm, act, hd;  // first word of: q, k, v [rows][packed features]; attention [rows][d]; its splits; residual stream after o; act; after down
  int slot;                         // words of a layer
};
// Words that say who takes part (uint32_t unless noted); epoch: the number of this pass, counted by the row descriptors' kernel (PassCount).
//   [0] epoch   [1] last pass that was given up   [2] last pass whose workgroups were counted   [3] passes that have started over
//   [64 + b]    state of workgroup b: epoch * 4 + 1 present, 2 past layer 0, 3 present and counted, 0 done without having been past layer 0
//   [64 + RELAY_MAX_GROUPS + 2 b]  (uint64_t) epoch << 32 | number of workgroups that start over << 16 | rank of b (0xFFFF: not one of
//                                  them); no workgroups: the pass goes on
constexpr int RELAY_SYNC_WORDS = 64 + 3 * RELAY_MAX_GROUPS;

// A word's tag is epoch << 6 | layer + 1, so that it comes round after 2^26 passes (an hour and a half of short ones).  Whenever the low 26 bits
// of the epoch become 0 all words become 0, which no tag is, as they are when a workspace is bound, and the states those of the pass
// before: nothing that is found with a pass's tag is older than the pass.
struct PassCount {
  uint32_t* sync;  // null: not counted
  uint64_t* words;
  size_t n;
};
__device__ __forceinline__ uint32_t last_pass(const PassCount& c) { return c.sync ? c.sync[0] : 0; }  // (requested before the rows, used after them)
__device__ __forceinline__ void count_pass(const PassCount& c, uint32_t last, int lane) {  // one wave, before the pass
  if (!c.sync) return;
  const uint32_t epoch = (uint32_t)__builtin_amdgcn_readfirstlane((int)last) + 1u;
  if (lane == 0) c.sync[0] = epoch;
  if (epoch << 6) return;
  for (size_t i = lane; i < c.n; i += 64) c.words[i] = 0;
  for (int i = lane; i < RELAY_MAX_GROUPS; i += 64) {
    c.sync[64 + i] = epoch * 4u - 1u;
    ((uint64_t*)(c.sync + 64 + RELAY_MAX_GROUPS))[i] = (uint64_t)(epoch - 1u) << 32;
  }
  if (lane == 0) c.sync[1] = c.sync[2] = epoch - 1u;
}

struct RelayArgs {
  const void* w[RELAY_MAX_LAYERS * 6 + 3];  // the model's weight list (order of mtad_model.weights)
  int n_layers, d, f, H, KVH, vocab;
  float eps;
  double inv_freq[64];  // radians a rotary pair turns by per position
  int rows, Rseq, B, ncg;
  int units[RS_STEPS];   // units of a step
  int first[RS_STEPS];   // workgroup of a step's unit 0
  int strips[RS_STEPS];  // strips of 16 features per unit (1 or 2)
  int pairs, splits;     // attention: (query head, row) pairs of a unit, key splits offered
  KvView kv;
  RowDesc rd;
  RelayMail mail;
  uint32_t* sync;
  uint32_t* status;
  float* h;       // float32 models: the hidden states
  bf16_t* xg;     // bf16 models: h * final gain as hi / lo terms (act_offset), and
  float* ssq;     // sums of squares of h per strip, [rows][d / 16]
  unsigned patience;  // ticks of the 100 MHz clock after which a workgroup whose wait in layer 0 lasts counts those that have started
  unsigned give_up;   // ticks after which one whose wait lasts gives the pass up
  int present;        // workgroups that take part (all but in tests)
};

int relay_mail_words(int rows, int d, int f, int H, int KVH, int hd, int splits, RelayMail* m);  // lays a layer's words out
// Units, their places and the key splits of a pass (n_layers, a.rows, Rseq, B, d, f, H, KVH are set); returns the workgroups, 0: no such pass, or
// one that is no faster (any: that one too)
int relay_plan(RelayArgs& a, int dtype, int hd, int max_context, bool any);
hipError_t launch_relay(const RelayArgs& a, int dtype, int hd, int groups, hipStream_t s);

}  // namespace mtad
