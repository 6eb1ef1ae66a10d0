// A recording stand-in for the HIP runtime, for tests of what the library's
// host code does without a GPU: memory is address space only, copies do
// nothing, and every launch is written to stdout, one event a line:
//   launch <device> <capture 0/1> <lds bytes> <start event> <stop event> <gx> <gy> <kernel>
//   limit <device> <capture 0/1> <lds bytes> <kernel>     (dynamic LDS limit raised)
//   alloc <base> <bytes> / fill <base> <bytes>            (hipMalloc / hipMemset)
//   parts <base> <bytes>   (partials that a launch writes for the next kernel: K or key splits,
//                           sums of squares, argmax)
//   mark <text>                                            (a step of the scenario)
// The executable's definitions come before libamdhip64's for libaxon.so too.
// Usage: recorded_hip <scenario> [number ...].
#include <cxxabi.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <string>
#include <vector>

#include "axon.h"
#include "kernels.h"

using namespace axon;

namespace {

int g_device = 0, g_capture = 0;
uint64_t g_next = 1ull << 40, g_event = 1;

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}

const char* name_of(const void* f) {
  auto it = names().find(f);
  return it == names().end() ? "?" : it->second.c_str();
}

void* reserve(size_t bytes) {
  void* p = (void*)g_next;
  g_next += (bytes + 4095) / 4096 * 4096;
  printf("alloc %llu %zu\n", (unsigned long long)p, bytes);
  return p;
}

// the partials written by a launch, from its arguments
void partials(const std::string& k, dim3 grid, void** args) {
  auto say = [](const void* p, int64_t words) {
    if (p) printf("parts %llu %lld\n", (unsigned long long)p, (long long)words * 4);
  };
  auto is = [&](const char* part) { return k.find(part) != std::string::npos; };
  const int64_t wgs = grid.x;
  if (is("gemv_wide_kernel<")) {
    const GemvArgs& a = *(const GemvArgs*)args[0];
    if (!a.g_off) say(a.part, (int64_t)grid.y * a.M * a.N);
  } else if (is("gemv_fused_kernel<") || is("gemv_split_resid_kernel")) {
    const GemvArgs& a = *(const GemvArgs*)args[0];
    say(a.ss_out, wgs * a.M);
    say(a.am_val, wgs * a.M);
    say(a.am_idx, wgs * a.M);
  } else if (is("gemm_ring_kernel<") || is("gemm_bf16_256_kernel<")) {
    const int64_t N = *(const int*)args[2], M = *(const int*)args[3];
    const EpiArgs& e = *(const EpiArgs*)args[5];
    if (grid.y > 1) say(e.out_f32, (grid.y - 1) * e.part_stride + M * N);
    if (is("gemm_ring_kernel<8")) {
      const int rows = few_head_rows((int)N, (int)M, *(const int*)args[4]);
      say(e.am_val, M * ((N + rows - 1) / rows));
      say(e.am_idx, M * ((N + rows - 1) / rows));
    }
  } else if (is("argmax_part_kernel")) {
    say(*(void**)args[2], wgs * grid.y);
    say(*(void**)args[3], wgs * grid.y);
  } else if (is("attn_decode_bf16_kernel")) {
    const KVView& kv = *(const KVView*)args[1];
    const int64_t H = *(const int*)args[5];
    say(*(void**)args[3], wgs * grid.z * H * (kv.hd + 2));
    say(*(void**)args[4], (int64_t)grid.z * grid.y);
  }
}

void launched(const void* f, dim3 grid, size_t lds, hipEvent_t a, hipEvent_t b, void** args) {
  partials(name_of(f), grid, args);
  printf("launch %d %d %zu %llu %llu %u %u %s\n", g_device, g_capture, lds, (unsigned long long)a,
         (unsigned long long)b, grid.x, grid.y, name_of(f));
}

struct Call {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
} g_call;

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* dev, unsigned, void*, void*, void*, void*,
                           int*) {
  int st = 0;
  char* d = abi::__cxa_demangle(dev, nullptr, nullptr, &st);
  std::string n = st == 0 ? d : dev;
  free(d);
  names()[host] = n;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_call = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_call.grid;
  *b = g_call.block;
  *lds = g_call.lds;
  *s = g_call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void** args, size_t lds, hipStream_t) {
  launched(f, g, lds, nullptr, nullptr, args);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3, void** args, size_t lds, hipStream_t, hipEvent_t a,
                              hipEvent_t b, int) {
  launched(f, g, lds, a, b, args);
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int bytes) {
  printf("limit %d %d %d %s\n", g_device, g_capture, bytes, name_of(f));
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = reserve(n);
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int, size_t n, hipStream_t) {
  printf("fill %llu %zu\n", (unsigned long long)p, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = g_device;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = reserve(AXON_NOALLOC_SCRATCH_BYTES);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)g_event++;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)1;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_capture = 1;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_capture = 0;
  *g = (hipGraph_t)1;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)1;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
}

namespace {

void mark(const std::string& what) { printf("mark %s\n", what.c_str()); }

void check(int rc, const char* what) {
  if (rc < 0) {
    printf("error %s: %s\n", what, axon_last_error());
    exit(1);
  }
}

axon_config llama(int D, int H, int KV, int hd, int I, int V) {
  axon_config c;
  memset(&c, 0, sizeof(c));
  c.hidden = D;
  c.n_layers = 1;
  c.n_heads = H;
  c.n_kv_heads = KV;
  c.head_dim = hd;
  c.intermediate = I;
  c.vocab = V;
  c.rms_eps = 1e-5f;
  c.rope_theta = 1e4;
  c.tie_embeddings = 1;
  c.dtype = AXON_BF16;
  return c;
}

// the weight map of a one-layer model, as device pointers
struct Map {
  std::vector<std::string> names;
  std::vector<axon_weight> w;
  Map(const axon_config& c, int dtype) {
    const int64_t D = c.hidden, H = c.n_heads, KV = c.n_kv_heads, hd = c.head_dim, I = c.intermediate;
    const std::string p = c.arch == AXON_ARCH_GPT2 ? "transformer.h.0." : "model.layers.0.";
    std::vector<std::pair<std::string, std::pair<int64_t, int64_t>>> l;
    if (c.arch == AXON_ARCH_GPT2) {
      l = {
        {"transformer.wte.weight", {c.vocab, D}}, {"transformer.wpe.weight", {c.max_positions, D}},
        {p + "ln_1.weight", {D, 0}}, {p + "ln_1.bias", {D, 0}},
        {p + "attn.c_attn.weight", {D, 3 * D}}, {p + "attn.c_attn.bias", {3 * D, 0}},
        {p + "attn.c_proj.weight", {D, D}}, {p + "attn.c_proj.bias", {D, 0}},
        {p + "ln_2.weight", {D, 0}}, {p + "ln_2.bias", {D, 0}},
        {p + "mlp.c_fc.weight", {D, I}}, {p + "mlp.c_fc.bias", {I, 0}},
        {p + "mlp.c_proj.weight", {I, D}}, {p + "mlp.c_proj.bias", {D, 0}},
        {"transformer.ln_f.weight", {D, 0}}, {"transformer.ln_f.bias", {D, 0}}};
    } else {
      l = {
        {"model.embed_tokens.weight", {c.vocab, D}},
        {"model.norm.weight", {D, 0}},
        {p + "input_layernorm.weight", {D, 0}},
        {p + "post_attention_layernorm.weight", {D, 0}},
        {p + "self_attn.q_proj.weight", {H * hd, D}},
        {p + "self_attn.k_proj.weight", {KV * hd, D}},
        {p + "self_attn.v_proj.weight", {KV * hd, D}},
        {p + "self_attn.o_proj.weight", {D, H * hd}}};
    }
    if (!c.tie_embeddings) l.push_back({"lm_head.weight", {c.vocab, D}});
    const bool gpt2 = c.arch == AXON_ARCH_GPT2;
    if (c.qkv_bias && !gpt2)
      for (auto& b : {std::make_pair("q", H), std::make_pair("k", KV), std::make_pair("v", KV)})
        l.push_back({p + "self_attn." + b.first + "_proj.bias", {b.second * hd, 0}});
    auto mlp = [&](const std::string& q, int64_t ii) {
      l.push_back({q + "gate_proj.weight", {ii, D}});
      l.push_back({q + "up_proj.weight", {ii, D}});
      l.push_back({q + "down_proj.weight", {D, ii}});
    };
    if (c.n_experts > 0) {
      l.push_back({p + "mlp.gate.weight", {c.n_experts, D}});
      for (int e = 0; e < c.n_experts; ++e) mlp(p + "mlp.experts." + std::to_string(e) + ".", c.moe_intermediate);
    } else if (!gpt2) {
      mlp(p + "mlp.", I);
    }
    for (auto& x : l) names.push_back(x.first);
    for (size_t i = 0; i < l.size(); ++i) {
      axon_weight a;
      memset(&a, 0, sizeof(a));
      a.name = names[i].c_str();
      a.data = (void*)(uintptr_t)0x10000;
      a.dtype = dtype;
      a.ndim = l[i].second.second ? 2 : 1;
      a.shape[0] = l[i].second.first;
      a.shape[1] = l[i].second.second;
      a.on_device = 1;
      w.push_back(a);
    }
  }
};

axon_model* make(const axon_config& c) {
  Map m(c, c.dtype);
  axon_model* out = nullptr;
  check(axon_init_model(&c, m.w.data(), (int)m.w.size(), nullptr, &out), "axon_init_model");
  return out;
}

int32_t* const TOK = (int32_t*)(uintptr_t)0x20000;
float* const LOGITS = (float*)(uintptr_t)0x30000;

void prefill(axon_model* m, int batch, int len, int all = 0) {
  std::vector<int32_t> cu;
  for (int b = 0; b <= batch; ++b) cu.push_back(b * len);
  check(axon_prefill(m, batch, TOK, TOK, cu.data(), nullptr, 0, all, LOGITS, TOK, nullptr), "axon_prefill");
}

void train(axon_model* m, const axon_config& c, const std::vector<int32_t>& cu) {
  Map g(c, AXON_F32);
  check(axon_loss_and_grads(m, (int)cu.size() - 1, TOK, TOK, cu.data(), TOK, LOGITS, g.w.data(), (int)g.w.size(), nullptr),
        "axon_loss_and_grads");
}

void train(axon_model* m, const axon_config& c, int batch, int len) {
  std::vector<int32_t> cu;
  for (int b = 0; b <= batch; ++b) cu.push_back(b * len);
  train(m, c, cu);
}

// calls of many sizes on two devices, one after the other in this process
void two_devices() {
  for (int d = 0; d < 2; ++d) {
    g_device = d;
    mark("device " + std::to_string(d));
    axon_config c = llama(1024, 16, 4, 64, 4096, 20000);
    c.max_batch = 160;
    c.max_seq = 2048;
    c.max_tokens = 8192;
    axon_model* m = make(c);
    mark("ready");
    for (int len : {1, 20, 70, 200, 700, 2000}) prefill(m, 4, len);
    prefill(m, 2, 300, 1);
    for (int b : {8, 24, 40, 64, 160}) {
      prefill(m, b, 16);
      mark("decode " + std::to_string(b));
      check(axon_decode_step(m, b, TOK, LOGITS, TOK, nullptr), "axon_decode_step");
      if (b <= 64) {
        mark("noalloc " + std::to_string(b));
        check(axon_decode_step_noalloc(m, b, TOK, LOGITS, TOK, nullptr), "axon_decode_step_noalloc");
      }
    }
    for (int len : {40, 500, 2000}) {
      mark("train " + std::to_string(len));
      train(m, c, 4, len);
    }
    axon_free(m);
  }
}

// float rows of an ungrouped few-token projection: raw partials only
void raw_rows() {
  for (int K : {64, 1024})
    for (int M : {1, 16, 17, 64}) {
      GemvArgs a{};
      a.W = a.X = (const bf16*)TOK;
      a.N = 64;
      a.K = K;
      a.M = M;
      a.ldo = a.N;
      a.out_f32 = LOGITS;
      a.part = LOGITS;
      for (int epi : {GV_F32, GV_PART}) {
        mark("raw " + std::to_string(epi) + " " + std::to_string(K) + " " + std::to_string(M));
        const bool ok = launch_gemv_fused(a, epi, nullptr);
        mark(ok ? "launched" : "refused");
        if (epi == GV_PART && (int64_t)gemv_shape(a.N, K, M, epi).ksplit * M * a.N > gemv_workspace_floats(a.N, K, M, epi))
          mark("workspace too small");
      }
    }
}

// a timed training step whose weight gradients split over the tokens
void timed_train() {
  axon_config c = llama(512, 8, 2, 64, 1024, 3000);
  c.max_batch = 2;
  c.max_seq = 1024;
  axon_model* m = make(c);
  check(axon_timing_enable(m, 1), "axon_timing_enable");
  mark("train");
  train(m, c, 2, 1000);
}

// the same decode step of a wide batch before and after a training step
void decode_after_training() {
  axon_config c = llama(4160, 16, 16, 64, 16384, 1000);
  c.max_batch = 1024;
  c.max_seq = 4;
  axon_model* m = make(c);
  for (int pass = 0; pass < 2; ++pass) {
    prefill(m, 1024, 1);
    mark("decode");
    check(axon_decode_step(m, 1024, TOK, LOGITS + 4 * pass, TOK, nullptr), "axon_decode_step");
    mark("end");
    train(m, c, 1024, 2);
  }
}

// a mixture-of-experts model's buffers: 7 tokens x 3 choices, 4 experts
void moe_init() {
  axon_config c = llama(128, 2, 2, 64, 64, 100);
  c.n_experts = 4;
  c.top_k = 3;
  c.moe_intermediate = 64;
  c.max_batch = 1;
  c.max_seq = 7;
  make(c);
}

// prompts, decode steps and mixed steps of models with few and many sequence
// slots: a dense one of each head dimension, a float32 one, a mixture of experts and GPT-2
void partials_of_many_sizes() {
  for (int max_batch : {1, 3, 40, 64, 65, 300})
    for (int kind = 0; kind < 5; ++kind) {
      axon_config c = kind == 1 ? llama(3584, 28, 4, 128, 18944, 1000) : llama(512, 8, 2, 64, 1536, 1000);
      if (kind == 2) c.dtype = AXON_F32;
      if (kind == 3) {
        c.n_experts = 256;
        c.top_k = 8;
        c.moe_intermediate = 64;
      }
      if (kind == 4) {
        c = llama(1600, 25, 25, 64, 6400, 1001);
        c.arch = AXON_ARCH_GPT2;
        c.qkv_bias = 1;
        c.max_positions = 3000;
      }
      c.max_batch = max_batch;
      c.max_seq = max_batch <= 40 ? 3000 : 82;  // (long: the decode attention splits the keys)
      c.max_tokens = 300 * 82;
      axon_model* m = make(c);
      for (int len : {1, 2, 4, 12, 16, 21, 33, 64, 79}) {
        for (int b : {1, 3, 40, 64, 65, 300})
          if (b <= max_batch) {
            mark("max_batch " + std::to_string(max_batch) + " kind " + std::to_string(kind) + " " + std::to_string(b) +
                 " x " + std::to_string(len));
            prefill(m, b, len);
            check(axon_decode_step(m, b, TOK, LOGITS, TOK, nullptr), "axon_decode_step");
            if (b <= 64 && kind < 2)
              check(axon_decode_step_noalloc(m, b, TOK, LOGITS, TOK, nullptr), "axon_decode_step_noalloc");
            // a step of prompt chunks in the even slots and decode tokens in the odd ones
            std::vector<int32_t> slots, fresh, cu{0};
            for (int i = 0; i < b; ++i) {
              slots.push_back(i);
              fresh.push_back(i % 2 == 0);
              cu.push_back(cu.back() + (i % 2 == 0 ? len : 1));
            }
            if (len <= 64)
              check(axon_step(m, b, slots.data(), fresh.data(), TOK, TOK, cu.data(), nullptr, 0, LOGITS, TOK, nullptr),
                    "axon_step");
          }
      }
      axon_free(m);
    }
}

// one training step: hidden, heads, kv heads, head dimension, intermediate,
// vocabulary, biases, tied head, sequence lengths
void train_step(const std::vector<int>& v) {
  axon_config c = llama(v[0], v[1], v[2], v[3], v[4], v[5]);
  c.qkv_bias = v[6];
  c.tie_embeddings = v[7];
  std::vector<int32_t> cu{0};
  for (size_t i = 8; i < v.size(); ++i) {
    cu.push_back(cu.back() + v[i]);
    c.max_seq = std::max(c.max_seq, (int32_t)v[i]);
  }
  c.max_batch = (int)cu.size() - 1;
  axon_model* m = make(c);
  mark("train");
  train(m, c, cu);
}

// a second training step of a model with an untied head
void train_twice() {
  axon_config c = llama(256, 4, 2, 64, 256, 1000);
  c.tie_embeddings = 0;
  c.max_batch = 2;
  c.max_seq = 64;
  axon_model* m = make(c);
  train(m, c, 2, 50);
  mark("second");
  train(m, c, 2, 60);
}

}  // namespace

int main(int argc, char** argv) {
  setvbuf(stdout, nullptr, _IOFBF, 1 << 20);
  const std::string s = argc > 1 ? argv[1] : "";
  std::vector<int> v;
  for (int i = 2; i < argc; ++i) v.push_back(atoi(argv[i]));
  if (s == "two_devices") two_devices();
  else if (s == "raw_rows") raw_rows();
  else if (s == "train_step" && v.size() > 8) train_step(v);
  else if (s == "train_twice") train_twice();
  else if (s == "timed_train") timed_train();
  else if (s == "partials") partials_of_many_sizes();
  else if (s == "moe_init") moe_init();
  else if (s == "decode_after_training") decode_after_training();
  else return 2;
  printf("done\n");
  return 0;
}
