// Host-side check of merged-adapter state over HIP calls that fail.  Builds the
// library's runtime (model.cpp) against stand-ins for the HIP calls and kernel
// launchers it makes: "device" memory is host memory, streams run at once, a
// merge adds a number that names its slot to every weight, and any merge launch,
// copy or synchronisation can be told to fail.  Whatever failed, the weights that
// a prefill is allowed to run on are the unmerged ones with at most one adapter.
#include "model.cpp"

#include <cstdlib>

namespace {

enum Fail { NONE, LAUNCH, LAUNCH_HALF, SYNC, COPY, COPY_HALF };
Fail g_fail = NONE;  // what the next call of that kind does (then NONE again)
bool g_armed = false;  // synchronisations fail only inside a merge or unmerge

bool take(Fail f) {
    if (g_fail != f || !g_armed) return false;
    g_fail = NONE;
    return true;
}

}  // namespace

extern "C" {
// the device array of model.cpp has no device image here
extern const char __hip_fatbin[8] = {};
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { *t = 0.f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)3; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return take(SYNC) ? hipErrorUnknown : hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
    a->type = hipMemoryTypeHost;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, hipMemcpyKind,
                            hipStream_t) {
    if (take(COPY)) return hipErrorUnknown;
    const bool half = take(COPY_HALF);
    for (size_t i = 0; i < (half ? h / 2 : h); ++i) std::memcpy((char*)d + i * dp, (const char*)s + i * sp, w);
    return half ? hipErrorUnknown : hipSuccess;
}
}

namespace pb {

thread_local LaunchTiming g_launch_timing = {nullptr, nullptr};

int lm_head_blocks(int) { return 1; }
int lm_head_mfma_blocks(int) { return 1; }
bool lm_head_use_mfma(int, int, int) { return false; }
size_t lm_head_mfma_scratch(int) { return 0; }
hipError_t launch_gemm(int, int, int, const GemmParams&, const GemmWorkspace&, hipStream_t) { return hipSuccess; }
hipError_t launch_attention(int, const void*, void*, int, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_attention_kv(int, const void*, const void*, int64_t, int64_t, void*, int, int, int, int,
                               hipStream_t) { return hipSuccess; }
hipError_t launch_embed(int, const int32_t*, const void*, const void*, float*, int, int, int, const int32_t*,
                        hipStream_t) { return hipSuccess; }
hipError_t launch_decode_attention(int, const void*, const void*, int64_t, int, int, int, const int32_t*, void*,
                                   hipStream_t) { return hipSuccess; }
hipError_t launch_layernorm(int, const float*, int64_t, int64_t, const void*, const void*, void*, bool, int, int,
                            float, hipStream_t, const RowShrink*) { return hipSuccess; }
hipError_t launch_row_shrink(int, const void*, const RowShrink&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lm_head(int, const float*, int, const void*, int, int, float*, float*, int*, hipStream_t) {
    return hipSuccess;
}
hipError_t launch_lm_head_mfma(int, const float*, int, const void*, int, int, float*, float*, int*, void*,
                               hipStream_t) { return hipSuccess; }
hipError_t launch_argmax(const float*, const int*, int, int, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_lora_pack(int, const void*, size_t, int, int, int, uint32_t, int, int, int, void*, void*,
                            hipStream_t) { return hipSuccess; }
hipError_t launch_lora_merge(int, const MergeParams& p, hipStream_t) {
    if (take(LAUNCH)) return hipErrorUnknown;
    const bool half = take(LAUNCH_HALF);
    const size_t dd = (size_t)p.d * p.d;
    for (int l = 0; l < (half ? p.layers / 2 : p.layers); ++l)
        for (int t = 0; t < 4; ++t) {
            const bool merge = (p.merge_mask >> t) & 1u;
            if (!merge && !((p.copy_mask >> t) & 1u)) continue;
            const uint16_t* s = (const uint16_t*)(p.src + l * p.src_stride) + t * dd;
            uint16_t* d = (uint16_t*)(p.dst + l * p.dst_stride) + t * dd;
            for (size_t i = 0; i < dd; ++i) d[i] = (uint16_t)(s[i] + (merge ? 100 * (p.slot + 1) : 0));
        }
    return half ? hipErrorUnknown : hipSuccess;
}

}  // namespace pb

namespace {

int failures = 0;

#define CHECK(cond)                                                                          \
    do {                                                                                     \
        if (!(cond)) {                                                                       \
            ++failures;                                                                      \
            std::printf("FAIL line %d (%s): %s; %s\n", __LINE__, what, #cond, g_err.c_str()); \
        }                                                                                    \
    } while (0)

constexpr uint32_t MASKS[3] = {PB_LORA_Q | PB_LORA_V, PB_LORA_K | PB_LORA_O, PB_LORA_Q};

struct World {
    pb_config c{};
    pb_model* m = nullptr;
    void* arena = nullptr;
    std::vector<char> layer, globals, lora;
    std::vector<const void*> layers, loras;

    explicit World(bool shadow) {
        c.n_layers = 2; c.d_model = 128; c.n_heads = 2; c.d_ffn = 64; c.vocab = 8; c.max_pos = 2;
        c.max_tokens = 2; c.max_batch = 1; c.max_adapters = 3; c.max_rank = 8; c.dtype = PB_F16;
        c.ln_eps = 1e-5f; c.merge_shadow = shadow;
        const size_t n = pb_arena_bytes(&c);
        arena = std::aligned_alloc(256, n);
        pb_model_create(&c, arena, n, (void*)1, (void*)2, &m);
        pb_set_graph_replay(m, 0);
        layer.assign(pb_layer_bytes(&c), 7);
        globals.assign(pb_globals_bytes(&c), 7);
        lora.assign(pb_lora_layer_bytes(&c, 8, 0xF), 0);
        layers = {layer.data(), layer.data()};
        loras = {lora.data(), lora.data()};
        for (int s = 0; s < 3; ++s) pb_attach_lora(m, s, 8, 8.f, MASKS[s], loras.data());
        load();
    }
    ~World() {
        pb_destroy(m);
        std::free(arena);
    }
    int load() {
        const int32_t order[2] = {0, 1};
        return pb_stream_layers(m, order, 2, layers.data(), globals.data());
    }
    int merge(int slot, Fail f = NONE) {
        g_fail = f;
        g_armed = true;
        const int rc = pb_merge_lora(m, slot);
        g_armed = false;
        return rc;
    }
    int unmerge(Fail f = NONE) {
        g_fail = f;
        g_armed = true;
        const int rc = pb_unmerge_lora(m);
        g_armed = false;
        return rc;
    }
    int prefill(int adapter = -1) {
        const int32_t tok[2] = {1, 2};
        const int32_t ad[1] = {adapter};
        int32_t out[1];
        return pb_prefill_first_token(m, tok, 1, 2, ad, out, nullptr);
    }
    // every layer holds the streamed weights, with `slot` (-1: none) merged once
    bool holds(int slot) {
        const int tensors[4] = {PB_T_WQ, PB_T_WK, PB_T_WV, PB_T_WO};
        for (int l = 0; l < 2; ++l)
            for (int t = 0; t < 4; ++t) {
                const uint16_t want = 0x0707 + (slot >= 0 && ((MASKS[slot] >> t) & 1u) ? 100 * (slot + 1) : 0);
                const uint16_t* w = (const uint16_t*)m->ltensor(l, tensors[t]);
                for (size_t i = 0; i < 128 * 128; ++i)
                    if (w[i] != want) return false;
            }
        return true;
    }
};

}  // namespace

int main() {
    const Fail kinds[] = {LAUNCH, LAUNCH_HALF, SYNC};
    const char* names[] = {"launch", "launch after half", "synchronisation"};
    for (int k = 0; k < 3; ++k) {
        const char* what = names[k];
        {  // a switch that fails, then another merge
            World w(true);
            CHECK(w.merge(0) == PB_OK && w.holds(0) && w.prefill() == PB_OK);
            CHECK(w.merge(1, kinds[k]) == PB_EHIP);
            CHECK(w.prefill() == PB_ESTATE && w.prefill(2) == PB_ESTATE);
            CHECK(w.merge(2) == PB_OK && w.holds(2) && w.prefill() == PB_OK);
            CHECK(w.merge(1) == PB_OK && w.holds(1));
        }
        {  // a switch that fails, then the unmerged model
            World w(true);
            CHECK(w.merge(0) == PB_OK);
            CHECK(w.merge(1, kinds[k]) == PB_EHIP);
            CHECK(w.unmerge() == PB_OK && w.holds(-1) && w.prefill() == PB_OK && w.prefill(1) == PB_OK);
            CHECK(w.unmerge() == PB_ESTATE);
            CHECK(w.merge(0) == PB_OK && w.holds(0));
        }
        {  // two in a row, then the layers again
            World w(true);
            CHECK(w.merge(2) == PB_OK);
            CHECK(w.merge(1, kinds[k]) == PB_EHIP && w.merge(0, kinds[k]) == PB_EHIP);
            CHECK(w.load() == PB_OK && w.holds(-1) && w.prefill() == PB_OK);
            CHECK(w.merge(1) == PB_OK && w.holds(1));
        }
        {  // the first merge of a load fails: a merge or unmerge works if the shadow was written
            World w(true);
            CHECK(w.merge(0, kinds[k]) == PB_EHIP && w.prefill() == PB_ESTATE);
            const bool written = kinds[k] != SYNC;
            CHECK(w.merge(1) == (written ? PB_OK : PB_ESTATE));
            if (written) CHECK(w.holds(1));
            CHECK(w.unmerge() == (written ? PB_OK : PB_ESTATE));
            if (written) CHECK(w.holds(-1));
            CHECK(w.load() == PB_OK && w.merge(2) == PB_OK && w.holds(2));
        }
        {  // no shadow: only streaming the layers helps
            World w(false);
            CHECK(w.merge(0, kinds[k]) == PB_EHIP);
            CHECK(w.prefill() == PB_ESTATE && w.merge(1) == PB_ESTATE && w.unmerge() == PB_ESTATE);
            CHECK(w.load() == PB_OK && w.holds(-1) && w.prefill() == PB_OK);
            CHECK(w.merge(1) == PB_OK && w.holds(1) && w.merge(0) == PB_ESTATE && w.prefill() == PB_OK);
        }
    }
    for (Fail f : {COPY, COPY_HALF, SYNC}) {
        const char* what = "unmerge";
        World w(true);
        CHECK(w.merge(0) == PB_OK);
        CHECK(w.unmerge(f) == PB_EHIP);
        CHECK(w.prefill() == PB_ESTATE);
        CHECK(w.unmerge() == PB_OK && w.holds(-1) && w.prefill() == PB_OK);
        CHECK(w.merge(1) == PB_OK && w.unmerge(f) == PB_EHIP);
        CHECK(w.merge(2) == PB_OK && w.holds(2));
    }
    {
        const char* what = "copy to the shadow";
        World w(true);
        CHECK(w.merge(0, COPY_HALF) == PB_EHIP);  // nothing merged yet
        CHECK(w.prefill() == PB_OK && w.holds(-1));
        CHECK(w.merge(0) == PB_OK && w.holds(0) && w.unmerge() == PB_OK && w.holds(-1));
    }
    std::printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
