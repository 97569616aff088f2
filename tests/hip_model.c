/* A model of the HIP runtime for tests without a GPU: devices, streams and
 * events, no work.  Loaded before libmppi.so (dlopen with RTLD_GLOBAL), so that
 * the library's calls come here.  Every call on a stream is a line of the log:
 *   launch DEV STREAM GRIDX GRIDY GRIDZ THREADS KERNEL | copy DEV STREAM DST SRC |
 *   record EVENT DEV STREAM | wait DEV STREAM EVENT
 * Stream 0 is the null stream of the device that is current at the call.  What
 * HIP refuses is refused: an event recorded on a stream of another device. */
#include <stdarg.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { int dev, id; } object; /* a stream or an event */
typedef struct { uint32_t x, y, z; } dim3;

static int current;
static char log_text[1 << 20];
static size_t log_len;

static void line(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  log_len += (size_t)vsnprintf(log_text + log_len, sizeof log_text - log_len, fmt, ap);
  va_end(ap);
}
static int dev_of(void* stream) { return stream ? ((object*)stream)->dev : current; }
static int id_of(void* stream) { return stream ? ((object*)stream)->id : 0; }
static void* new_object(int dev) {
  static int next = 1;
  object* o = malloc(sizeof *o);
  o->dev = dev;
  o->id = next++;
  return o;
}

static struct { const void* fn; char name[512]; } kernel[4096];
static int kernels;

/* for the test */
const char* model_log(void) { return log_text; }
void model_clear(void) { log_len = 0; log_text[0] = 0; }
void* model_stream(int dev) { return new_object(dev); }
int model_id(void* o) { return id_of(o); }
int model_current(void) { return current; }

/* the runtime */
int hipGetDevice(int* dev) { *dev = current; return 0; }
int hipSetDevice(int dev) { current = dev; return 0; }
int hipStreamGetDevice(void* s, int* dev) { *dev = dev_of(s); return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = new_object(current); return 0; }
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) {
  if (((object*)e)->dev != dev_of(s)) return 400; /* hipErrorInvalidHandle */
  line("record %d %d %d\n", ((object*)e)->id, dev_of(s), id_of(s));
  return 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned f) {
  (void)f;
  line("wait %d %d %d\n", dev_of(s), id_of(s), ((object*)e)->id);
  return 0;
}
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
const char* hipGetErrorString(int e) { return e == 400 ? "invalid resource handle" : "error"; }
int hipGetLastError(void) { return 0; }
int hipMemcpyAsync(void* d, const void* src, size_t n, int kind, void* s) {
  (void)n; (void)kind;
  line("copy %d %d %p %p\n", dev_of(s), id_of(s), d, src);
  return 0;
}
int hipMemcpy2DAsync(void* d, size_t dp, const void* src, size_t sp, size_t w, size_t h, int kind,
                     void* s) {
  (void)dp; (void)sp; (void)w; (void)h;
  return hipMemcpyAsync(d, src, 0, kind, s);
}
int hipMemsetAsync(void* d, int v, size_t n, void* s) {
  (void)v; (void)n;
  line("copy %d %d %p %p\n", dev_of(s), id_of(s), d, (void*)0);
  return 0;
}
int hipLaunchKernel(const void* fn, dim3 g, dim3 b, void** args, size_t lds, void* s) {
  (void)args; (void)lds;
  const char* name = "?";
  for (int i = 0; i < kernels; ++i)
    if (kernel[i].fn == fn) name = kernel[i].name;
  line("launch %d %d %u %u %u %u %s\n", dev_of(s), id_of(s), g.x, g.y, g.z, b.x * b.y * b.z, name);
  return 0;
}
int hipFuncSetAttribute(const void* fn, int a, int v) { (void)fn; (void)a; (void)v; return 0; }
int hipGetSymbolAddress(void** p, const void* sym) {
  (void)sym;
  static char scratch[512];
  *p = (void*)(((uintptr_t)scratch + 255) & ~(uintptr_t)255);
  return 0;
}
int hipStreamBeginCapture(void* s, int mode) { (void)s; (void)mode; return 0; }
int hipStreamEndCapture(void* s, void** g) { *g = s; return 0; }
int hipGraphInstantiate(void** e, void* g, void* n, char* l, size_t len) {
  (void)g; (void)n; (void)l; (void)len;
  *e = new_object(current);
  return 0;
}
int hipGraphDestroy(void* g) { (void)g; return 0; }
int hipGraphExecDestroy(void* e) { free(e); return 0; }
int hipGraphLaunch(void* e, void* s) {
  (void)e;
  line("launch %d %d\n", dev_of(s), id_of(s));
  return 0;
}

/* the compiler's registration and launch hooks */
static struct { dim3 g, b; size_t lds; void* s; } pushed;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) {
  pushed.g = g; pushed.b = b; pushed.lds = lds; pushed.s = s;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
  *g = pushed.g; *b = pushed.b; *lds = pushed.lds; *s = pushed.s;
  return 0;
}
void** __hipRegisterFatBinary(const void* data) { (void)data; static void* h; return &h; }
void __hipRegisterFunction(void** m, const void* f, char* df, const char* n, unsigned t, void* a,
                           void* b, void* c, void* d, int* w) {
  (void)m; (void)df; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (kernels == 4096) abort();
  kernel[kernels].fn = f;
  snprintf(kernel[kernels++].name, sizeof kernel[0].name, "%s", n);
}
void __hipRegisterVar(void** m, void* v, char* h, char* n, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
