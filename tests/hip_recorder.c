/* Stands in for the HIP runtime where a test looks at the order in which the library hands work to streams: nothing runs, and every
 * call that orders work is written down, one line each:
 *   launch <kernel> <stream> <stop event or nil> <grid> <captured>
 *   record <event> <stream> <captured>
 *   wait   <event> <stream> <captured>
 *   sync
 * Device memory is not modelled, except for what the library asks its device about where blocks run: rec_where() says what a launch of
 * where_kernel leaves there.
 * A stream is captured from rec_capture on, or from a wait for an event that was recorded in the capture (streams join a capture
 * that way); rec_end_capture ends it for all of them.  As in the runtime, the stop event of a launch that is captured is no
 * node of the capture. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define MAX 4096
typedef struct { unsigned x, y, z; } dim3_t;
typedef struct { int captured; } event_t;

static char log_text[1 << 20];
static size_t log_len;
static const void* stubs[MAX];
static const char* names[MAX];
static int n_stubs, n_captured;
static unsigned long long n_captures;
static void* captured[64];

static int is_captured(void* s) {
  for (int i = 0; i < n_captured; ++i)
    if (captured[i] == s) return 1;
  return 0;
}
#define LOG(...) (log_len += (size_t)snprintf(log_text + log_len, sizeof log_text - log_len, __VA_ARGS__))

void rec_capture(void* s) { if (!is_captured(s)) captured[n_captured++] = s; }
void rec_end_capture(void) { n_captured = 0; n_captures += 1; }
const char* rec_log(void) { return log_text; }

/* what where_kernel does: 0 writes block numbers modulo 8, 1 other numbers, 2 is refused, 3 writes nothing; 4 is 0, after a call of
 * the program's own that failed */
static int where_mode, where_ran, where_fill, last_error;
void rec_where(int mode) { where_mode = mode; last_error = mode == 4 ? 98 : 0; }

static const char* name_of(const void* stub) {
  for (int i = 0; i < n_stubs; ++i)
    if (stubs[i] == stub) return names[i];
  return "?";
}
static void launched(const void* stub, dim3_t grid, void* stream, event_t* stop) {
  LOG("launch %s %p %p %ux%ux%u %d\n", name_of(stub), stream, (void*)stop, grid.x, grid.y, grid.z, is_captured(stream));
  if (stop) stop->captured = 0;
}

/* what compiled host code registers and calls for a launch */
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* stub, char* dev, const char* name, unsigned t, void* a, void* b, void* c, void* d, int* w) {
  (void)h; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_stubs < MAX) { stubs[n_stubs] = stub; names[n_stubs++] = name; }
}
void __hipRegisterVar(void** h, void* var, char* a, char* b, int c, size_t d, int e, int f) {
  (void)h; (void)var; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f;
}
static struct { dim3_t grid, block; size_t lds; void* stream; } pushed;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* stub, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)block; (void)args; (void)lds;
  if (strstr(name_of(stub), "where_kernel")) {
    if (where_mode == 2) return last_error = 98;
    where_ran = where_mode != 3;
  }
  launched(stub, grid, stream, NULL);
  return 0;
}
int hipExtLaunchKernel(const void* stub, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream, void* start, void* stop, int flags) {
  (void)block; (void)args; (void)lds; (void)start; (void)flags;
  launched(stub, grid, stream, stop);
  return 0;
}

int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; *e = calloc(1, sizeof(event_t)); return 0; }
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* stream) {
  ((event_t*)e)->captured = is_captured(stream);
  LOG("record %p %p %d\n", e, stream, is_captured(stream));
  return 0;
}
int hipStreamWaitEvent(void* stream, void* e, unsigned flags) {
  (void)flags;
  if (((event_t*)e)->captured && n_captured > 0) rec_capture(stream);
  LOG("wait %p %p %d\n", e, stream, is_captured(stream));
  return 0;
}
int hipStreamIsCapturing(void* stream, int* status) { *status = is_captured(stream); return 0; }
int hipStreamGetCaptureInfo(void* stream, int* status, unsigned long long* id) {
  *status = is_captured(stream);
  *id = n_captures;
  return 0;
}
int hipEventSynchronize(void* e) { (void)e; LOG("sync\n"); return 0; }
int hipStreamSynchronize(void* s) { (void)s; LOG("sync\n"); return 0; }
int hipDeviceSynchronize(void) { LOG("sync\n"); return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }

int hipMemcpy(void* d, const void* s, size_t n, int kind) {
  (void)s;
  if (kind != 2) return 0;
  memset(d, where_fill, n);
  for (size_t i = 0; where_ran && i < n / 4; ++i) ((unsigned*)d)[i] = (unsigned)(where_mode == 1 ? i / 2 % 8 : i % 8);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)d; (void)s; (void)n; (void)kind; (void)st; return 0; }
int hipMemset(void* d, int v, size_t n) { (void)d; (void)n; where_fill = v; return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)d; (void)v; (void)n; (void)st; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 160 * 1024; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int v) { (void)f; (void)attr; (void)v; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = (void*)0x1000; return 0; }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { (void)e; return "recorded"; }
