// The host side of the library (csrc/fc_api.hip, csrc/fc_plan.cpp) without a GPU: a HIP
// runtime whose allocations can be made to fail, and launchers that only say that they
// were called.  Like HIP's, an error of a call stays behind for the next hipGetLastError,
// which is what a launcher returns.  Built and checked by test_api_host.py; the argument
// names the scenario.  Compiled with -x hip --offload-host-only.
#include <hip/hip_runtime.h>
#undef __device__
#define __device__

#include "../paper_2503_08461_amd/csrc/fc_api.hip"

#include <cstdlib>
#include <string>

static hipError_t g_last = hipSuccess;
static size_t g_largest = ~(size_t)0;  // largest device allocation that succeeds
static int g_allocations = 0;  // device allocations and waits
static bool g_capturing = false;
static std::string g_launched;

static hipError_t give(void** out, size_t size) {
  if (size > g_largest) return g_last = hipErrorOutOfMemory;
  *out = calloc(1, size);
  return hipSuccess;
}
extern "C" {
hipError_t hipMalloc(void** out, size_t size) {
  ++g_allocations;
  return give(out, size);
}
hipError_t hipHostMalloc(void** out, size_t size, unsigned) { *out = calloc(1, size); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  g_launched += "copy ";
  memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  ++g_allocations;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** out, const void* symbol) { *out = const_cast<void*>(symbol); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

namespace fc {
static hipError_t launched(const char* name) {
  g_launched += name;
  g_launched += ' ';
  return hipGetLastError();
}
hipError_t kernels_one_time_setup() { return hipSuccess; }
hipError_t mlp_one_time_setup() { return hipSuccess; }
size_t mlp_w1p_elems(int, int, int) { return 1; }
size_t mlp_w2p_elems(int, int) { return 1; }
int mlp_rows_per_tile(int, int) { return 256; }
int mlp_workgroups_per_cu(int, int) { return 1; }
hipError_t launch_stack_init(int32_t*, int, hipStream_t) { return launched("stack_init"); }
hipError_t launch_pool_pop(const int32_t*, int, int, int32_t*, int32_t*, int, int32_t*, hipStream_t) { return launched("pop"); }
hipError_t launch_pool_push(int32_t*, int, int, const int32_t*, int32_t*, int, hipStream_t) { return launched("push"); }
hipError_t launch_owner_init(int32_t*, const int32_t*, int, int, hipStream_t) { return launched("owner_init"); }
hipError_t launch_owner_check_ids(const int32_t*, int, int, int32_t*, int32_t*, bool, hipStream_t) { return launched("check_ids"); }
hipError_t launch_owner_check_tables(const BatchParams&, int32_t*, bool, hipStream_t) { return launched("check_tables"); }
hipError_t launch_plan_alloc(const BatchParams&, const MetaChunk* c, int, hipStream_t) { return launched(c ? "plan_inline" : "plan"); }
hipError_t launch_snapkv_score(const BatchParams&, hipStream_t) { return launched("snapkv_score"); }
hipError_t launch_zero_ints(int32_t*, int, hipStream_t) { return launched("zero"); }
hipError_t launch_knorm_score(const BatchParams&, hipStream_t) { return launched("knorm_score"); }
hipError_t launch_split_scores(const BatchParams&, hipStream_t) { return launched("split_scores"); }
hipError_t launch_select(const BatchParams&, int, bool, hipStream_t) { return launched("select"); }
// (+reclaim: told to take the old blocks back in passing)
static hipError_t launched_main(const BatchParams& p, const char* name) {
  return launched((std::string(name) + (p.main_reclaims ? "+reclaim" : "")).c_str());
}
hipError_t launch_gather(const BatchParams& p, hipStream_t) { return launched_main(p, "gather"); }
hipError_t launch_fused(BatchParams p, int, int, int, bool wide, hipStream_t) { return launched_main(p, wide ? "fused_wide" : "fused_narrow"); }
hipError_t launch_reclaim(const BatchParams&, hipStream_t) { return launched("reclaim"); }
hipError_t launch_meta_upload(const MetaChunk&, char*, int, hipStream_t) { return launched("upload"); }
hipError_t launch_append(const DecodeParams& p, const DecodeReqs&, hipStream_t) { return launched(p.reqs ? "append" : "append_inline"); }
hipError_t launch_decode_attention(const DecodeParams& p, const DecodeReqs&, hipStream_t) {
  return launched((std::string(p.reqs ? "attention" : "attention_inline") + ":" + std::to_string(p.n_seg)).c_str());
}
hipError_t launch_mlp_permute_weights(const _Float16*, const _Float16*, _Float16*, _Float16*, int, int, int, hipStream_t) { return launched("permute"); }
hipError_t launch_mlp_compress(const BatchParams& p, const MlpParams&, hipStream_t) { return launched_main(p, "mlp"); }
}  // namespace fc

static void report(const char* what, int rc) {
  printf("%s %d %s\n", what, rc, g_launched.c_str());
  g_launched.clear();
}

// (addresses that nothing behind the launchers reads)
template <typename T>
static T* somewhere() {
  return reinterpret_cast<T*>((uintptr_t)1 << 30);
}

int main(int argc, char** argv) {
  const std::string scenario = argc > 1 ? argv[1] : "";
  fc_pool* pool = nullptr;
  auto create = [&] {
    return fc_pool_create(&pool, somewhere<void>(), ~(size_t)0, 4096, 16, 1, 32, 128, FC_DTYPE_F16);
  };
  const int32_t method[2] = {FC_METHOD_SNAPKV, FC_METHOD_KNORM}, budget[2] = {1500, 1400};
  auto compress = [&](const char* what, int32_t* kept) {
    int32_t lens[2] = {7001, 8000};
    const int rc = fc_compress_batch(pool, somewhere<int32_t>(), 512, lens, somewhere<void>(), 32, method, budget, 2, 7,
                                     0.f, nullptr, kept, nullptr);
    report(what, rc);
    fc_pool_import_state_dev(pool, somewhere<int32_t>(), 4096, nullptr);
    g_launched.clear();
  };
  if (scenario == "no_room_for_split_scores") {
    report("create", create());
    // what any call of this size needs is there: only few long heads into fresh blocks are split
    fc_set_compaction_mode(pool, FC_COMPACT_IN_PLACE);
    compress("in_place", nullptr);
    fc_set_compaction_mode(pool, FC_COMPACT_FRESH);
    g_largest = 0;
    compress("full", nullptr);
    compress("full_kept_out", somewhere<int32_t>());
    printf("error [%s]\n", fc_last_error());
    g_allocations = 0;
    compress("full_again", nullptr);
    printf("error %d\n", g_allocations);
    g_largest = ~(size_t)0;
    fc_pool_destroy(pool);
    report("create_with_room", create());
    fc_set_compaction_mode(pool, FC_COMPACT_IN_PLACE);
    compress("in_place_again", nullptr);
    fc_set_compaction_mode(pool, FC_COMPACT_FRESH);
    g_capturing = true;
    g_allocations = 0;
    compress("captured", nullptr);
    printf("error %d\n", g_allocations);
    g_capturing = false;
    compress("room", nullptr);
    g_capturing = true;
    compress("captured_warm", nullptr);
    g_capturing = false;
  } else if (scenario == "no_room_for_decode_segments") {
    const int32_t lens[2] = {8000, 30000};
    auto attention = [&](const char* what) {
      report(what, fc_decode_attention(pool, somewhere<int32_t>(), 2048, lens, somewhere<void>(), somewhere<float>(), 2,
                                       0.f, nullptr));
    };
    g_largest = 1 << 20;
    report("create", create());
    attention("whole");
    fc_pool_destroy(pool);
    g_largest = ~(size_t)0;
    report("create_with_room", create());
    attention("cut");
  } else if (scenario == "decode_requests") {
    report("create", create());
    for (int n : {149, 150}) {
      std::vector<int32_t> lens(n, 20);
      auto step = [&](const char* what) {
        report(what, fc_decode_attention(pool, somewhere<int32_t>(), 2, lens.data(), somewhere<void>(),
                                         somewhere<float>(), n, 0.f, nullptr));
      };
      step(n == 149 ? "few" : "many");
      g_capturing = true;
      step(n == 149 ? "few_captured" : "many_captured");
      g_capturing = false;
    }
  } else if (scenario == "reclaim") {
    report("create", create());
    const _Float16 w1[256 * 128] = {}, w2[128 * 256] = {};
    const float b1[256] = {}, b2[128] = {};
    const fc_mlp_weights weights = {1, 256, FC_ACT_GELU_ERF, {w1, w1}, {b1, b1}, {w2, w2}, {b2, b2}};
    report("weights", fc_mlp_set_weights(pool, &weights, nullptr));
    fc_set_profiling(pool, 1);
    // few requests (descriptors as an argument of plan_alloc), many, few with ownership checks
    for (const char* how : {"few", "many", "checked"}) {
      const int n = std::string(how) == "many" ? 60 : 2;
      fc_set_debug_checks(pool, std::string(how) == "checked");
      // a head in one workgroup, heads split over workgroups, the separate kernels next to a streaming request, the MLP
      for (const char* what : {"fused", "split", "separate", "mlp"}) {
        const std::string name = what;
        std::vector<int32_t> lens(n, name == "split" ? 4000 : 500), budgets(n, 100), methods(n, FC_METHOD_KNORM), zeros(n, 0);
        if (name == "split" && n == 60) continue;  // (more heads than are split)
        if (name == "separate") methods[0] = FC_METHOD_STREAMING;
        fc_set_score_mode(pool, name == "separate" ? FC_SCORE_TWO_PASS : FC_SCORE_AUTO);
        fc_pool_import_state_dev(pool, somewhere<int32_t>(), 4096, nullptr);
        g_launched.clear();
        const int rc = name == "mlp" ? fc_compress_batch_mlp(pool, somewhere<int32_t>(), 512, lens.data(), zeros.data(),
                                                             lens.data(), nullptr, n, nullptr)
                                     : fc_compress_batch(pool, somewhere<int32_t>(), 512, lens.data(), nullptr, 32,
                                                         methods.data(), budgets.data(), n, 7, 0.f, nullptr, nullptr, nullptr);
        report((name + "_" + how).c_str(), rc);
        float ms[FC_N_KERNELS];
        fc_get_kernel_times(pool, ms);
        report((name + "_" + how + "_timed").c_str(), (int)ms[K_RECLAIM]);
        fc_set_profiling(pool, 1);  // (counts from here)
      }
    }
  } else {
    return 2;
  }
  fc_pool_destroy(pool);
  return 0;
}
