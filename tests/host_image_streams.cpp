// Host replay of an image whose context can get no further streams: launches
// and HIP calls are stood in for, stream creation fails, and the control block
// says that every channel stopped at rank 0.  No device is touched.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdio>

static int streams = 0, pinned = 0, allow_streams = 0;
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)0
#define hipGetLastError() hipSuccess
#define hipStreamCreateWithFlags(s, f) (++streams, streams <= allow_streams ? (*(s) = (hipStream_t)8, hipSuccess) : hipErrorOutOfMemory)
#define hipStreamDestroy(s) hipSuccess
#define hipEventCreateWithFlags(e, f) (*(e) = (hipEvent_t)8, hipSuccess)
#define hipEventDestroy(e) hipSuccess
#define hipEventRecord(...) hipSuccess
#define hipStreamWaitEvent(...) hipSuccess
#define hipStreamSynchronize(s) hipSuccess
#define hipMemcpyAsync(...) hipSuccess
#define hipHostMalloc(p, n, f) (++pinned, hipErrorOutOfMemory)
#define hipHostFree(p) hipSuccess
#include "eodabe.hip"

int main() {
  for (int fail_at = 0; fail_at < 2; ++fail_at) {      // the first stream, or the pinned memory behind it
    streams = pinned = 0;
    allow_streams = fail_at;
    State host{};
    host.stop_block = 0;
    eodabe_ctx ctx{};
    eodabe_default_opts(&ctx.o);
    ctx.host_state = &host;
    ctx.images = IMG_OVERLAP_AFTER;
    const int c = 3;
    const int64_t h = 90, w = 70, n = eodabe_image_workspace_size(&ctx, c, h, w);
    eodabe_image_info info;
    const int st = eodabe_compress_image(&ctx, (const float*)4096, c, h, w, 1e-3, (void*)4096, n, (float*)4096,
                                         (int64_t)c * w * (h + w + w), (float*)4096, &info);
    printf("streams asked for %d, pinned %d, status %d, ranks %ld %ld %ld\n", streams, pinned, st, (long)info.rank[0],
           (long)info.rank[1], (long)info.rank[2]);
    if (st != 0 || streams < 1 || pinned != fail_at || ctx.last_hip != 0) return 1;
    for (auto* x : ctx.chan)
      if (x) return 2;
  }
  return 0;
}
