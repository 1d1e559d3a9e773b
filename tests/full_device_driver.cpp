// Driver of test_full_device_cpu.py: the library's host code against a device that lives in host
// memory and can be full.  hipMalloc fails beyond `room` bytes; the launches that the calls below
// need before the device fills up do nothing, and any other is left unresolved.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "sg.h"
#include "sg_internal.h"

static size_t room = (size_t)1 << 40;
static int32_t *apt_perm;      // slot -> buffer of the last APT context made
static int mlp_chunk, mlp_calls;

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    *p = n <= room ? std::malloc(n) : nullptr;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)&room; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)&room; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}

namespace sg {
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return hipSuccess;
}
hipError_t launch_fill_i64(int64_t *p, int64_t v, int64_t n, hipStream_t)
{
    for (int64_t i = 0; i < n; ++i) p[i] = v;
    return hipSuccess;
}
hipError_t launch_apt_init(const InstDev *, const QuadDesc *, int, uint8_t *, const int32_t *perm, uint32_t, uint32_t,
                           uint32_t, hipStream_t)
{
    apt_perm = const_cast<int32_t *>(perm);
    return hipSuccess;
}
hipError_t launch_apt_quad(const AptArgs &, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_sqa_init(const SqaArgs &, int, hipStream_t) { return hipSuccess; }
hipError_t mlp_scratch(float **p)
{
    static float a[4];
    *p = a;
    return hipSuccess;
}
hipError_t launch_mlp_grad(float *, const float *, const float *, const int *, int batch, const MlpWork &w, float *loss,
                           float *, const MlpAdam *, hipStream_t)
{
    mlp_chunk = w.chunk;
    ++mlp_calls;
    std::memset(w.rec, 0, sizeof(float) * kMlpRecFloats * (size_t)w.chunk);
    for (int q = 0; q < (batch < kMlpGroups ? batch : kMlpGroups); ++q) loss[q] = 33.f;
    return hipSuccess;
}
}  // namespace sg

#define CHECK(x)                                                       \
    do {                                                               \
        if (!(x)) {                                                    \
            std::printf("line %d: %s failed\n", __LINE__, #x);         \
            return 1;                                                  \
        }                                                              \
    } while (0)

// Spins in, out, in parts and through a checkpoint while nothing can be allocated on the device.
static int spins(int mode)
{
    const int shape[3][3] = {{5, 7, 3}, {4, 4, 4}, {3, 1, 1}};
    std::vector<int8_t> J[3];
    sg_lattice lat[3];
    for (int i = 0; i < 3; ++i) {
        J[i].assign((size_t)3 * shape[i][0] * shape[i][1] * shape[i][2], 1);
        lat[i] = {shape[i][0], shape[i][1], shape[i][2], 7u, J[i].data(), nullptr};
    }
    const double one[5] = {0.2, 0.5, 1.0, 2.0, 3.0};
    std::vector<double> beta;
    for (int i = 0; i < 3; ++i) beta.insert(beta.end(), one, one + 5);
    const int M = mode == SG_APT ? 1 : 33, R = mode == SG_APT ? 10 : 4, n_max = 105;
    sg_config cfg{};
    cfg.mode = mode;
    cfg.n_inst = 3;
    cfg.inst = lat;
    cfg.n_beta = 5;
    cfg.beta = beta.data();
    cfg.reps_per_beta = 2;
    cfg.M = M;
    cfg.R = R;
    cfg.sqa_beta = 2.0;
    cfg.seed = 1;
    sg_ctx *c = nullptr;
    room = (size_t)1 << 40;
    CHECK(sg_create(&cfg, &c) == SG_OK);
    room = 0;
    std::mt19937 rng(2);
    const size_t row = (size_t)M * n_max, total = 3 * R * row;
    std::vector<int8_t> s(total, 0), got(total, 9);
    for (int i = 0; i < 3; ++i)
        for (size_t r = 0; r < (size_t)R * M; ++r)
            for (int j = 0; j < lat[i].Lx * lat[i].Ly * lat[i].Lz; ++j)
                s[((size_t)i * R * M + r) * n_max + j] = rng() & 1 ? 1 : -1;
    CHECK(sg_set_spins(c, s.data()) == SG_OK);
    CHECK(sg_get_spins(c, got.data()) == SG_OK && got == s);
    const int n1 = 64;
    std::vector<int8_t> part((size_t)2 * M * n1);
    CHECK(sg_get_spins_range(c, 1, 1, 2, part.data()) == SG_OK);
    for (int r = 0; r < 2 * M; ++r)
        CHECK(std::memcmp(&part[(size_t)r * n1], &s[((size_t)(R + 1) * M + r) * n_max], n1) == 0);
    std::vector<int8_t> bad = s;
    bad[(2 * R + R - 1) * row + row - n_max + 2] = 0;
    CHECK(sg_set_spins(c, bad.data()) == SG_EINVAL);
    CHECK(sg_get_spins(c, got.data()) == SG_OK && got == s);
    size_t len = 0;
    CHECK(sg_get_state(c, nullptr, &len) == SG_OK);
    std::vector<char> blob(len);
    CHECK(sg_get_state(c, blob.data(), &len) == SG_OK);
    std::vector<int8_t> other = s;
    for (int8_t &v : other) v = (int8_t)-v;
    CHECK(sg_set_spins(c, other.data()) == SG_OK);
    CHECK(sg_set_state(c, blob.data(), len) == SG_OK);
    CHECK(sg_get_spins(c, got.data()) == SG_OK && got == s);
    if (mode == SG_APT) {   // slots 0 and 1 of instance 2 trade buffers
        std::swap(apt_perm[2 * 12], apt_perm[2 * 12 + 1]);
        CHECK(sg_get_spins(c, got.data()) == SG_OK);
        for (size_t j = 0; j < row; ++j)
            CHECK(got[(2 * R) * row + j] == s[(2 * R + 1) * row + j] && got[(2 * R + 1) * row + j] == s[2 * R * row + j]);
    }
    sg_destroy(c);
    return 0;
}

// Gradient and training with room for few records and for the losses of one epoch at a time.
static int training()
{
    room = (size_t)1 << 40;
    sg_mlp *m = nullptr;
    CHECK(sg_mlp_create(nullptr, 1, nullptr, &m) == SG_OK);
    const int n = 9000;
    std::vector<float> x(4 * n, 1.f), y(33 * n, 1.f), g(SG_MLP_NPARAM);
    room = 33 * 4 * n;   // the targets: the largest array of the caller's data
    float loss = 0.f;
    CHECK(sg_mlp_loss_grad(m, x.data(), y.data(), n, &loss, g.data()) == SG_OK);
    CHECK(mlp_chunk >= 512 && (size_t)mlp_chunk * sg::kMlpRecFloats * 4 <= room);
    mlp_calls = 0;
    const int epochs = 80;
    std::vector<float> per(epochs, 0.f);
    CHECK(sg_mlp_train(m, x.data(), y.data(), n, 1, epochs, 1e-3f, per.data()) == SG_OK);
    CHECK(mlp_calls == epochs * n);
    for (float v : per) CHECK(v == 1.f);
    sg_mlp_destroy(m);
    return 0;
}

int main() { return spins(SG_APT) || spins(SG_SQA) || training(); }
