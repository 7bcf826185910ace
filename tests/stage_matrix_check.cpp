// Host check of stage_matrix: it reads no byte behind the caller's buffer.
// Buffers of odd sizes end at an inaccessible page; HIP's copies are memcpy.
// Exit status 0 = all passed.
#include "../paper_2308_01999_amd/csrc/sv_api.cpp"

#include <signal.h>
#include <sys/mman.h>
#include <unistd.h>

extern "C" {
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
}

static void read_behind(int)
{
    const char text[] = "read behind the buffer\n";
    (void)!write(1, text, sizeof text - 1);
    _exit(1);
}

int main()
{
    signal(SIGSEGV, read_behind);
    const size_t page = size_t(sysconf(_SC_PAGESIZE)), room = 4 << 20;
    char* base = static_cast<char*>(mmap(nullptr, room + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
    if (base == MAP_FAILED || mprotect(base + room, page, PROT_NONE)) return 2;
    for (size_t i = 0; i < room; ++i) base[i] = char(i * 7 + 1);
    std::vector<char> ws(kMinWorkspace), pinned(kMatRingBytes);
    sv_handle_s h;
    h.ws = ws.data();
    h.ws_bytes = ws.size();
    h.pinned = pinned.data();
    for (size_t bytes : {size_t(1), size_t(64), size_t(256), size_t(1344), size_t(1) << 20, (size_t(1) << 20) + 8}) {
        const char* from = base + room - bytes;
        const void* to = sv::stage_matrix(&h, from, bytes);
        if (std::memcmp(to, from, bytes)) return 3;
        if ((static_cast<const char*>(to) - h.ws) % 256) return 4;
    }
    std::puts("passed");
    return 0;
}
