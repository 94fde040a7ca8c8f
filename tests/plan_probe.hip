// Test infrastructure: says which kernels the entry points' plans pick, from the planning code itself (its structures are
// internal to fdl_api.hip).  Host code; linked with the library's other objects by test_routes_host.py.
#include "../paper_2509_14279_amd/csrc/fdl_api.hip"

#include <string>

namespace {
std::string product(int mid, int skinny, int pad, int tiled, int split, int copied) {
  if (mid) return split > 1 ? "mid split" : "mid";
  if (skinny) return "few rows";
  if (!pad && !tiled) return "generic";
  return std::string(pad ? "padded" : "tiled") + (split > 1 ? " split" : "") + (copied && !pad ? " from blocks" : "");
}
std::string gradients(const GradPlan& g) {
  if (g.dt == kF32) return g.s64_a.small && g.s64_b.small ? "32 x 32" : "64 x 64";
  if (g.mid) return std::string("mid") + (g.split_a > 1 ? " dx-split" : "") + (g.split_b > 1 ? " dw-split" : "");
  std::string s = g.pair ? "pair" : (std::string(g.b3_fast ? "tiled" : "generic") + " and " + (g.b4_fast ? "tiled" : "generic"));
  if (g.pad) s += g.stage_x ? " padded-x" : " padded";
  if (g.extra) s += " extra";
  if (g.blocked) s += " blocked";
  return s;
}
std::string text;
}  // namespace

// "forward product | gradients | pitch of dZ" of the block (op 0) and of Linear+ReLU (op 1), "gate | down" of the feed-forward
// block (op 2), for a workspace of the size asked for
extern "C" __attribute__((visibility("default"))) const char* plan_probe(int op, int dt, int64_t M, int64_t K, int64_t N) {
  if (op == 0) {
    Plan p;
    if (!make_plan(dt, M, K, N, Room::kAll, &p)) return "";
    text = product(p.f1_mid, p.f1_skinny, p.pad, p.f1_fast, p.f1_split, 0) + " | " + gradients(p.g) + " | " + std::to_string(p.g.ldz);
  } else if (op == 1) {
    ReluPlan p = {};
    if (!make_relu_plan(dt, M, K, N, Room::kAll, &p)) return "";
    text = product(p.f1_mid, p.f1_skinny, p.pad, p.f1_fast, p.f1_split, 0) + " | " + gradients(p.g) + " | " + std::to_string(p.g.ldz);
  } else {
    FfnPlan p = {};
    if (!make_ffn_plan(dt, M, K, N, Room::kAll, &p)) return "";
    text = product(p.gate_mid, p.gate_skinny, p.gate_pad, p.gate_fused, 1, 0) + " | " +
           product(p.down_mid, p.down_skinny, p.down_pad, p.down_fast, p.down_split, p.g_blocked);
  }
  return text.c_str();
}
