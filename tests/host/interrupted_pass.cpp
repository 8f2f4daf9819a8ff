// A call of the resident pass whose second launch fails must not leave words that the next call takes for its own.  Drives the
// host side of the library (adasum_api.cpp, adasum_plan.cpp) on the CPU: "device" memory is host memory, and the launches are
// stand-ins that follow the pass's protocol -- the first sends words under the call's tag, the last moves the tag on.  Every
// call checks that no word carries its tag before it sends any.  Built and run by tests/test_interrupted_pass_cpu.py.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "adasum_host.h"

using namespace adasum;

#define CHECK(cond)                                                                           \
    do {                                                                                      \
        if (!(cond)) {                                                                        \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);     \
            std::exit(1);                                                                     \
        }                                                                                     \
    } while (0)

namespace {
enum { kNothing, kFirst, kSecond };
int fail_at = kNothing;          // which launch of the next resident pass fails
bool capturing = false;          // the caller's stream is being captured: launches are recorded, not run
std::vector<std::pair<int32_t*, int64_t>> cleared;   // runs of zero words
int passes = 0;

int stand_in(const ResidentCall& c) {
    if (fail_at == kFirst) return hipErrorLaunchFailure;
    ++passes;
    if (capturing) return hipSuccess;
    const int64_t words = (c.state.sums - c.state.partials);
    const unsigned long long tag = static_cast<unsigned>(*c.state.epoch) + 1u;
    for (int64_t i = 0; i < words; ++i) CHECK(c.state.partials[i] >> 32 != tag);
    for (int64_t i = 0; i < words; ++i) c.state.partials[i] = tag << 32 | 7u;
    if (fail_at == kSecond) return hipErrorLaunchFailure;
    *c.state.epoch += 1;
    return hipSuccess;
}
}  // namespace

namespace adasum {
int launch_resident_bf16(const ResidentCall& c, void*) { return stand_in(c); }
int launch_resident_f32(const ResidentCall& c, void*) { return stand_in(c); }
int launch_resident_wide_bf16(const ResidentCall& c, void*) { return stand_in(c); }
const char* kernel_name(const char*, int, int, int, bool, char* buf, size_t n) {
    if (n > 0) buf[0] = 0;
    return buf;
}
int launch_zero_words(int32_t* p, int64_t n, void*) {
    cleared.emplace_back(p, n);
    if (!capturing) std::memset(p, 0, static_cast<size_t>(n) * 4);
    return hipSuccess;
}
}  // namespace adasum

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
    std::memset(*p, 0x5a, (n + 255) / 256 * 256);
    return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = kResidentCus; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(16); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}

int main() {
    struct Case {
        int K, dtype, form;
        std::vector<int64_t> offsets;
    };
    const std::vector<Case> cases = {{2, ADASUM_BF16, 2, {0, 20000000, 25000000, 25000009}},
                                     {8, ADASUM_F32, 3, {0, 3000000, 6000000, 6000100}},
                                     {16, ADASUM_BF16, 3, {0, 900000, 1800000, 4000000}}};
    void* const stream = reinterpret_cast<void*>(32);
    for (const Case& t : cases) {
        const int L = static_cast<int>(t.offsets.size()) - 1;
        CHECK(plan_resident(t.K, {t.K}, t.dtype, false, t.offsets.data(), L).form >= 2);
        // (no buffer is read)
        std::vector<void*> grads;
        for (int k = 0; k < t.K; ++k) grads.push_back(reinterpret_cast<void*>((k + 2ull) << 40));
        void* const out = reinterpret_cast<void*>(1ull << 40);
        adasum_plan* plan = nullptr;
        CHECK(adasum_plan_create(t.K, t.offsets.data(), L, t.dtype, nullptr, &plan) == ADASUM_OK);
        auto execute = [&](int fail) {
            fail_at = fail;
            const int rc = adasum_plan_execute(plan, grads.data(), out, nullptr, nullptr, stream);
            fail_at = kNothing;
            return rc;
        };
        cleared.clear();
        for (int i = 0; i < 3; ++i) CHECK(execute(kNothing) == ADASUM_OK);
        CHECK(cleared.empty());
        // the second launch fails: the next call starts from a cleared section, and the one after it goes on as ever
        CHECK(execute(kSecond) == ADASUM_ERR_HIP && adasum_last_hip_error() == hipErrorLaunchFailure);
        CHECK(execute(kNothing) == ADASUM_OK && cleared.size() == 1);
        CHECK(execute(kNothing) == ADASUM_OK && cleared.size() == 1);
        // two failures in a row, and one in the first launch
        CHECK(execute(kSecond) == ADASUM_ERR_HIP && execute(kSecond) == ADASUM_ERR_HIP && execute(kFirst) == ADASUM_ERR_HIP);
        CHECK(execute(kNothing) == ADASUM_OK && execute(kNothing) == ADASUM_OK);
        // a call that is captured next records the clearing, and the next eager one clears too
        CHECK(execute(kSecond) == ADASUM_ERR_HIP);
        cleared.clear();
        capturing = true;
        CHECK(execute(kNothing) == ADASUM_OK && cleared.size() == 1);
        capturing = false;
        CHECK(execute(kNothing) == ADASUM_OK && cleared.size() == 2);
        CHECK(execute(kNothing) == ADASUM_OK && cleared.size() == 2);
        CHECK(adasum_plan_destroy(plan) == ADASUM_OK);

        // the library's own plan of the same shape
        for (int fail : {int(kNothing), int(kSecond), int(kNothing), int(kNothing)}) {
            fail_at = fail;
            CHECK(adasum_reduce(grads.data(), t.K, t.offsets.data(), L, t.dtype, out, stream) == (fail ? ADASUM_ERR_HIP : ADASUM_OK));
        }
        fail_at = kNothing;
        CHECK(adasum_shutdown() == ADASUM_OK);
    }
    std::printf("interrupted passes ok: %d passes\n", passes);
    return 0;
}
