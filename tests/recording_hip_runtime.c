/* Stands in for the HIP runtime under libmsgemm.so on a machine without a GPU: several devices, no memory behind the
 * addresses, launches and copies do nothing.  What it keeps is, for every call that uses a device, which device was current
 * and on what kind of stream the work went.  Loaded with its symbols global before libmsgemm.so, it is found first. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

enum { kAlloc = 1, kLaunch = 2, kWork = 3, kEvent = 4 };
static int current_device, capturing, count;
static uintptr_t next_address = 0x100000000ull;
static struct { int kind, device, own_stream; const void* kernel; } calls[65536];
static struct { const void* host; char name[320]; } kernels[8192];
static int kernels_known;
static char streams[64];
static int streams_made;

static int note_kernel(int kind, const void* stream, const void* kernel)
{
    if (count < 65536) {
        calls[count].kind = kind;
        calls[count].device = current_device;
        calls[count].own_stream = (const char*)stream >= streams && (const char*)stream < streams + sizeof(streams);
        calls[count].kernel = kernel;
        ++count;
    }
    return 0;
}
static int note(int kind, const void* stream) { return note_kernel(kind, stream, 0); }

/* for the test */
int rec_count(void) { return count; }
int rec_kind(int i) { return calls[i].kind; }
int rec_device(int i) { return calls[i].device; }
int rec_own_stream(int i) { return calls[i].own_stream; }
void rec_capture(int on) { capturing = on; }
const char* rec_kernel(int i)          /* name of the kernel that call i launches, as the compiler made it */
{
    for (int j = 0; j < kernels_known; ++j)
        if (kernels[j].host == calls[i].kernel) return kernels[j].name;
    return "";
}
int rec_kernels(void) { return kernels_known; }   /* the library's own */
const char* rec_name(int j) { return kernels[j].name; }
void rec_forget(void) { count = 0; }

/* the runtime */
void __hipRegisterFunction(void** module, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           void* block, void* grid, int* size)
{
    (void)module; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
    if (kernels_known == 8192) return;
    kernels[kernels_known].host = host;
    strncpy(kernels[kernels_known].name, name, sizeof(kernels[0].name) - 1);
    ++kernels_known;
}
int hipGetDevice(int* d) { *d = current_device; return 0; }
int hipSetDevice(int d) { current_device = d; return 0; }
int hipDeviceGetAttribute(int* v, int attribute, int device) { (void)attribute; (void)device; *v = 256; return 0; }
int hipGetDevicePropertiesR0600(void* p, int device) { (void)p; (void)device; return 1; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void** p, size_t n)
{
    *p = (void*)next_address;
    next_address += (n + 0xfffffu) & ~(uintptr_t)0xfffffu;
    return note(kAlloc, 0);
}
int hipFree(void* p) { (void)p; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { (void)d; (void)s; (void)n; (void)kind; return note(kWork, 0); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream)
{
    (void)s;
    if (kind == 2) memset(d, 0, n);   /* device to host */
    return note(kWork, stream);
}
int hipMemsetAsync(void* d, int v, size_t n, void* stream) { (void)d; (void)v; (void)n; return note(kWork, stream); }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; *e = &count; return note(kEvent, 0); }
int hipEventRecord(void* e, void* stream) { (void)e; (void)stream; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipStreamWaitEvent(void* stream, void* e, unsigned flags) { (void)e; (void)flags; return note(kWork, stream); }
int hipStreamCreateWithFlags(void** s, unsigned flags)
{
    (void)flags;
    *s = streams + streams_made++ % (int)sizeof(streams);
    return 0;
}
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* status) { *status = 0; return capturing && !s ? 900 : 0; }
int hipThreadExchangeStreamCaptureMode(int* mode) { (void)mode; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int block, size_t lds)
{
    (void)f; (void)block; (void)lds;
    *n = 2;
    return 0;
}
int hipGetSymbolAddress(void** p, const void* symbol) { *p = (void*)symbol; return 0; }
struct dim { unsigned x, y, z; };
static struct { struct dim grid, block; size_t lds; void* stream; } pushed;
int __hipPushCallConfiguration(struct dim g, struct dim b, size_t lds, void* stream)
{
    pushed.grid = g;
    pushed.block = b;
    pushed.lds = lds;
    pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(struct dim* g, struct dim* b, size_t* lds, void** stream)
{
    *g = pushed.grid;
    *b = pushed.block;
    *lds = pushed.lds;
    *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void* f, struct dim g, struct dim b, void** args, size_t lds, void* stream)
{
    (void)g; (void)b; (void)args; (void)lds;
    return note_kernel(kLaunch, stream, f);
}
