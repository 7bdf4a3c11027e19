// launch_trace.cpp - walks the host side of librl_policy.so without a GPU: the HIP runtime's entry points are defined here, ahead of the real
// ones, and a launch is a line in a list.  For every call of the grid below each operand of a backward contraction has to be an input or an array that
// an earlier launch of the same call wrote, and a contraction that reads an input itself must not write a gradient that shares memory with it.
//   launch_trace LIBRARY G L N S ..     prints which kernel encodes L vectors of each of G groups in N stages of S entries, "few" or "many", a line for each four
//   launch_trace LIBRARY     prints the kinds of contraction it met, how often, and every operand that nothing wrote; 0 if there is none
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "../include/rl_policy.h"

struct dim3 { unsigned x, y, z; };

static std::map<const void*, std::string> g_names;      // (mangled)
static dim3 g_grid, g_block;
static std::set<const void*> g_written;
static std::map<std::string, long> g_met;
static std::string g_case;
static long g_bad = 0;
static const void *g_x, *g_w;
static bool g_no_small, g_no_k_major;      // gradients meet what these launches read while they write them

template <class T> static T arg(void** args, int i, size_t offset = 0) {
  T v;
  memcpy(&v, static_cast<const char*>(args[i]) + offset, sizeof v);
  return v;
}
static const void* ptr(void** args, int i, size_t offset = 0) { return arg<const void*>(args, i, offset); }

static void bad(const std::string& what) {
  if (g_bad++ < 20) printf("%s: %s\n", g_case.c_str(), what.c_str());
}
static void reads(const char* kind, const char* which, const void* p) {
  if (p != g_x && p != g_w && !g_written.count(p)) bad(std::string(kind) + " reads " + which + ", which nothing wrote");
}

static void launch(const std::string& n, void** a) {
  auto is = [&](const char* s) { return n.find(s) != std::string::npos; };
  if (is("rvq_few_kernel")) printf("few\n");
  if (is("rvq_encode_kernel")) printf("many\n");
  auto writes = [&](const void* p) { if (p) g_written.insert(p); };
  // epilogues that store an operand: EpiDS {ids, lse, c, dS, stride, dS^T, ..}, EpiFwdStash {ref, part, stride, E, ..}
  if (is("EpiDSI")) { writes(ptr(a, 3, 24)); if (is("EpiDSIf")) writes(ptr(a, 3, 40)); }
  else if (is("EpiFwdStashI")) writes(ptr(a, 3, 24));
  else if (is("loss_prep_kernel")) {          // (LossJob, W: TransposeJob, int, workgroups, X: TransposeJob, int, workgroups, ..)
    for (int i : {1, 4}) if (arg<int>(a, i + 2) > 0) writes(ptr(a, i, 64));
  } else if (is("transpose_kernelI")) writes(ptr(a, 0, 64));
  else if (is("transpose_bf16_kernel")) writes(ptr(a, 10));
  else if (is("kept_ds_f32_kernel")) { writes(ptr(a, 1)); writes(ptr(a, 3)); }
  else if (is("kept_ds_t_kernel")) writes(ptr(a, 1));
  else if (is("kept_ds_kernel")) writes(ptr(a, 3));
  const bool pair = is("pair_kernelI");
  if (!is("splitk_reduce") && (pair || is("EpiDXIf") || is("EpiDWE"))) {
    const char* kind = is("small_pair") ? "small pair" : pair ? "bf16 pair" : is("EpiDWE") ? "dW" : is("gemm_nt_f32_kernelINS_5EpiDXIfEELb0ELb1E") ? "dX K-major" : "dX";
    ++g_met[kind];
    if (g_no_k_major && !strcmp(kind, "dX K-major")) bad("dX is written over W, which its launch reads");
    reads(kind, "A", ptr(a, 0)); reads(kind, "B", ptr(a, 1));
    if (pair) { reads(kind, "the second A", ptr(a, 5)); reads(kind, "the second B", ptr(a, 6)); }
  }
  if (is("small_grads_kernel")) {
    ++g_met["small grads"];
    if (g_no_small) bad("gradients are written over what their launch reads");
  }
}

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, void*) { g_grid = grid; g_block = block; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) { *grid = g_grid; *block = g_block; *lds = 0; *stream = nullptr; return 0; }
int hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, void*) { launch(g_names.at(f), args); return 0; }
int hipGetLastError() { return 0; }
}

int main(int argc, char** argv) {
  void* lib = argc >= 2 && argc % 4 == 2 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : nullptr;
  if (!lib) { fprintf(stderr, "%s\n", argc >= 2 && argc % 4 == 2 ? dlerror() : "usage: launch_trace LIBRARY [G L N S ..]"); return 2; }
  const auto bytes = reinterpret_cast<decltype(&rl_workspace_bytes)>(dlsym(lib, "rl_workspace_bytes"));
  const auto call = reinterpret_cast<decltype(&rl_policy_loss_fwd_bwd)>(dlsym(lib, "rl_policy_loss_fwd_bwd"));
  if (g_names.empty()) { fprintf(stderr, "the library registered no kernel here\n"); return 2; }
  // addresses that nothing follows, far apart
  auto at = [](int i, int off = 0) { return reinterpret_cast<void*>(((uintptr_t)(i + 1) << 40) + off); };
  if (argc > 2) {
    const auto encode = reinterpret_cast<decltype(&rl_rvq_encode)>(dlsym(lib, "rl_rvq_encode"));
    for (int i = 2; i + 3 < argc; i += 4)
      if (encode(at(0), at(1), (const float*)at(2), atoi(argv[i]), atoi(argv[i + 1]), 128, atoi(argv[i + 2]), atoi(argv[i + 3]), (int32_t*)at(3), at(4), nullptr) != RL_OK) printf("refused\n");
    return 0;
  }
  long calls = 0, before = 0, apart = 0;
  for (int dtype : {RL_F32, RL_BF16})
    for (int64_t R : {1, 200, 356, 1000, 1025, 2048, 2600, 3072, 4096, 5400, 8192, 16384, 33000})
      for (int H : {4, 8, 16, 32, 40, 64, 72, 80, 128, 264, 512, 712, 1024})
        for (int V : {5, 300, 1000, 2048, 2064, 3000, 3199, 4096, 5400, 8000, 8192, 16384, 33024, 50257})
          for (int chunk : {0, 256, 2048, 3072, 5120})
            for (int off : {0, 4})
              for (int promise : {0, 100})
              for (int place = 0; place < 8; ++place) {
                if (dtype == RL_BF16 && H % 8) continue;
                if (dtype == RL_F32 && promise) continue;
                if (place && (dtype != RL_F32 || off || R > 5400)) continue;
                rl_batch b{};
                b.R = R; b.H = H; b.V = V; b.B = 4; b.P = 2; b.dtype = dtype;
                b.hidden = g_x = at(0); b.weight = g_w = at(1, off); b.token_ids = (const int32_t*)at(2); b.mask = (const uint8_t*)at(3);
                b.cu_seqlens = (const int32_t*)at(4); b.group_idx = (const int32_t*)at(5); b.rewards = (const float*)at(6);
                b.old_logprob = (const float*)at(7); b.ref_logprob = (const float*)at(8); b.log_z = (const float*)at(9);
                rl_params p{};
                p.clip_eps = 0.2f; p.adv_eps = 1e-6f; p.chunk_rows = chunk; p.max_seq_len = promise;
                rl_outputs o{};
                o.loss = (float*)at(10); o.d_hidden = at(11); o.d_weight = (float*)at(12);
                // gradients beside the inputs, in their place, over their first or last bytes
                const size_t xb = 4 * (size_t)R * H, wb = 4 * (size_t)V * H;
                char *X = (char*)at(0), *W = (char*)at(1, off);
                if (place == 1) { o.d_hidden = X + xb; o.d_weight = (float*)(W - wb); }
                if (place == 2) o.d_hidden = X;
                if (place == 3) o.d_weight = (float*)W;
                if (place == 4) o.d_hidden = W + wb - 4;
                if (place == 5) o.d_weight = (float*)(X - wb + 4);
                if (place == 6) o.d_hidden = (char*)at(5) + 12;
                if (place == 7) o.d_hidden = W - xb + 4;
                g_no_small = place > 1; g_no_k_major = place == 4 || place == 7;
                size_t n = 0;
                char text[160];
                snprintf(text, sizeof text, "%s, %ld rows, H %d, V %d, chunks of %d, weight + %d, lengths up to %d, place %d", dtype == RL_F32 ? "f32" : "bf16", (long)R, H, V, chunk, off, promise, place);
                g_case = text;
                g_written.clear();
                if (bytes(&b, &p, 1, &n) != RL_OK || call(&b, &p, RL_OBJ_FLOW, &o, at(20), n, nullptr) != RL_OK) bad("refused");
                ++calls;
                if (place == 0) apart = g_met["small grads"] + g_met["dX K-major"] - before;
                if (place == 1 && g_met["small grads"] + g_met["dX K-major"] - before != apart) bad("gradients beside the inputs take another path");
                before = g_met["small grads"] + g_met["dX K-major"];
              }
  printf("%ld calls\n", calls);
  for (auto& m : g_met) printf("%s: %ld\n", m.first.c_str(), m.second);
  printf("%ld faults\n", g_bad);
  return g_bad ? 1 : 0;
}
