// The host side of the library on a machine without a GPU: lc_api.hip with launchers and HIP calls that do nothing
// but count, one of which fails when it is told to.  Exit code 0: what the callers of a failed call are promised holds.
#include <stdio.h>

#include "lc_internal.h"

static int gathers, fails_at, broadcasts, averages;

namespace lc {
hipError_t launch_gather(lc_handle*, bool, int64_t, int) { return ++gathers == fails_at ? hipErrorLaunchFailure : hipSuccess; }
hipError_t launch_broadcast_xbar(lc_handle*) { ++broadcasts; return hipSuccess; }
hipError_t launch_average(lc_handle*, const float*, float*, float*) { ++averages; return hipSuccess; }
hipError_t launch_update_from_grad(lc_handle*) { return hipSuccess; }
hipError_t launch_update_and_average(lc_handle*) { return hipSuccess; }
hipError_t launch_quad_step(lc_handle*) { return hipSuccess; }
hipError_t launch_quad_loss(lc_handle*, int*) { return hipSuccess; }
hipError_t launch_forward(lc_handle*, bool, int, int) { return hipSuccess; }
bool eval_layer_ok(const lc_handle*, int) { return false; }
hipError_t launch_eval_layer(lc_handle*, int) { return hipSuccess; }
bool forward_fuses_softmax(const lc_handle*) { return true; }
hipError_t launch_softmax(lc_handle*, bool, int) { return hipSuccess; }
hipError_t launch_backward(lc_handle*, int, bool) { return hipSuccess; }
size_t backward_share_floats(const lc_handle*) { return 0; }
bool first_layer_kernel_ok(const lc_handle*) { return false; }
hipError_t launch_first_layer(lc_handle*) { return hipSuccess; }
bool implicit_layer_ok(const lc_handle*, int) { return false; }
bool sync_layer_ok(const lc_handle*, int l) { return l == 1; }
hipError_t launch_sync_layer(lc_handle*, int) { return hipSuccess; }
bool head_is_fused(const lc_handle*) { return false; }
hipError_t launch_head(lc_handle*) { return hipSuccess; }
bool resident_shape_ok(const lc_handle*) { return false; }
int compute_units() { return 256; }
bool net_shape_ok(const lc_handle*) { return false; }
hipError_t launch_net(lc_handle*, int, int) { return hipSuccess; }
size_t resident_exchange_floats(const lc_handle*) { return 0; }
hipError_t probe_block_placement(lc_handle*) { return hipSuccess; }
bool exchange_is_local(const lc_handle*) { return false; }
hipError_t launch_resident(lc_handle*, int, int, int) { return hipSuccess; }
}  // namespace lc

extern "C" {
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
}

#define EXPECT(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    lc_model md = {};
    md.kind = LC_KIND_MLP;
    md.n_layers = 2;
    md.dims[0] = 64; md.dims[1] = 64; md.dims[2] = 10;
    md.B = 16; md.N = 100; md.E = 10; md.lr = 0.1f;
    for (int lazy = 0; lazy < 2; ++lazy) {
        lc_handle* h = nullptr;
        EXPECT(lc_init(2, lc_param_count(&md), &md, 1, &h) == LC_OK);
        void* p = reinterpret_cast<void*>(uintptr_t{4096});   // never touched here
        EXPECT(lc_attach(h, p, p, p, lc_workspace_bytes(h), p, static_cast<int32_t*>(p), nullptr) == LC_OK);
        EXPECT(lc_set_lazy_broadcast(h, lazy) == LC_OK);
        gathers = broadcasts = averages = 0;
        fails_at = 2;   // averaged models of many iterations are behind it, none copied to the rows yet
        EXPECT(lc_local_periods(h, 1, 1000) == LC_ERR_HIP);
        EXPECT(lc_last_hip_error(h) == hipErrorLaunchFailure);
        EXPECT(averages > 0);
        if (lazy) {   // asked for: the rows wait for lc_materialize()
            EXPECT(broadcasts == 0);
            EXPECT(lc_materialize(h) == LC_OK && broadcasts == 1);
        } else {      // who never asked for a deferred broadcast finds the averaged model in the rows
            EXPECT(broadcasts == 1);
            EXPECT(lc_materialize(h) == LC_OK && broadcasts == 1);
        }
        lc_destroy(h);
    }
    printf("ok\n");
    return 0;
}
