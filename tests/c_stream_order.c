/* A client of libwb that stands in for the parts of the HIP runtime the library
 * calls, so that the order of its work on several streams can be read without
 * a GPU: this program's definitions come before the runtime's, write one line
 * per call and run nothing. Built and run by tests/test_stream_order_cpu.py.
 *
 * Usage: c_stream_order STEP...  with STEP = <stream><set>, e.g. A0 B0: pack
 * the tensors of that set (their addresses only; none is read) on that stream.
 */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "wb.h"

static hipStream_t stream_of(char c) { return (hipStream_t)(uintptr_t)c; }
static char name_of(hipStream_t s) { return s ? (char)(uintptr_t)s : '-'; }

static struct { dim3 g, b; size_t lds; hipStream_t s; } launch;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  launch.g = g, launch.b = b, launch.lds = lds, launch.s = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = launch.g, *b = launch.b, *lds = launch.lds, *s = launch.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  (void)f, (void)g, (void)b, (void)args, (void)lds;
  printf("launch %c\n", name_of(s));
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  (void)p;
  memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  *base = p, *size = (size_t)1 << 40;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
  (void)flags;
  return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t s) {
  (void)src, (void)n, (void)kind;
  printf("copy %c %p\n", name_of(s), dst);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { return printf("sync %c\n", name_of(s)), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
  *e = (hipEvent_t)malloc(1);
  printf("event %p 0x%x\n", (void*)*e, flags);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return free((void*)e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return printf("record %c %p\n", name_of(s), (void*)e), hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { return printf("hostwait %p\n", (void*)e), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned flags) {
  (void)flags;
  return printf("wait %c %p\n", name_of(s), (void*)e), hipSuccess;
}

static void check(int rc, const char* what) {
  if (rc == WB_OK) return;
  fprintf(stderr, "%s: status %d: %s\n", what, rc, wb_last_error());
  exit(1);
}

int main(int argc, char** argv) {
  const wb_model_shapes model = {WB_FAMILY_DENSE, 2, 256, 4, 4, 64, 1024, 1024, 0, 0};
  const wb_parallelism trainer = {WB_STYLE_FSDP_FLAT, WB_F32, 1, 1, 2, 1, 0, WB_DTYPE_NONE, 0};
  const wb_parallelism rollout = {WB_STYLE_SERVING, WB_BF16, 2, 1, 1, 1, 0, WB_DTYPE_NONE, 0};
  wb_layout_t *lt = NULL, *lr = NULL;
  wb_plan_t* plan = NULL;
  int64_t ws = 0;
  int32_t n = 0;
  check(wb_describe_layout(&model, &trainer, &lt), "trainer layout");
  check(wb_describe_layout(&model, &rollout, &lr), "rollout layout");
  check(wb_plan(lt, lr, WB_SENDER, 0, &plan), "plan");
  check(wb_plan_workspace_bytes(plan, &ws), "workspace size");
  check(wb_plan_num_local_tensors(plan, &n), "local tensors");
  check(wb_plan_upload(plan, (void*)(uintptr_t)(1 << 20), (size_t)ws, stream_of('U')), "upload");
  for (int i = 1; i < argc; ++i) {
    const void** src = malloc((size_t)n * sizeof *src);
    if (!src) return 1;
    for (int u = 0; u < n; ++u) src[u] = (const void*)(((uintptr_t)(argv[i][1] - '0' + 1) << 40) + ((uintptr_t)u << 30));
    printf("step %s\n", argv[i]);
    check(wb_pack(plan, src, (void*)((uintptr_t)1 << 39), stream_of(argv[i][0])), argv[i]);
    free(src);
  }
  wb_plan_destroy(plan);
  wb_layout_destroy(lr);
  wb_layout_destroy(lt);
  return 0;
}
