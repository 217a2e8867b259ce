// Host-only probe of the tile rules at wide row pitches (no kernel runs, no
// device call): for each "nx ny nz pitch" on the command line, the tile of
// every sweep kind (0 to 3) and of the reactive sweep (4), its chunk, its
// height's bytes per element and whether its launch takes the pitch.
#include <cstdlib>

#include "waves.hip"

extern "C" {
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
extern const char __hip_fatbin[64] = {};
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
hipError_t hipDeviceGetAttribute(int*, hipDeviceAttribute_t, int) { return hipErrorNoDevice; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}
namespace ptk {
hipError_t launch_copy(const double*, double*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_reduce_max(const double*, int64_t, double*, hipStream_t) { return hipSuccess; }
}

int main(int argc, char** argv) {
    for (int a = 1; a + 3 < argc; a += 4) {
        Geom g{};
        g.nx = atoi(argv[a]); g.ny = atoi(argv[a + 1]); g.nz = atoi(argv[a + 2]);
        g.P = atoll(argv[a + 3]); g.S = g.P * (g.ny + 1);
        const Tiling t = make_tiling(g);
        for (int k = 0; k < 5; ++k) {
            const TileShape s = k < 4 ? t.shape[k] : waves_tile(g);
            const int elem = k == SK_F32 || k == SK_NORM32 ? 4 : 8;
            // the reactive sweep's launch, as the library makes it
            int taken = -1;
            if (k == 4) {
                pt_waves w{};
                w.geom = g;
                w.tile = s;
                w.blocks = sweep_blocks(g, s);
                taken = launch_waves<false>(&w, WavesPtrs{}) == hipSuccess;
            }
            printf("%d %d %d %lld %d %d %d %d %d %d\n", g.nx, g.ny, g.nz, (long long)g.P, k, s.w, s.h, s.kz, elem, taken);
        }
    }
    return 0;
}
