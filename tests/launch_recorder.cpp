// Stands in for the HIP runtime's launch call in a process without a GPU: loaded with
// global visibility before libndq.so, it takes the library's launches and notes, in order,
// which kernel was launched on which grid.  Nothing runs.
#include <cstdint>
#include <map>
#include <string>

struct Dim3 { uint32_t x, y, z; };

static std::map<const void*, std::string>& names()
{
    static std::map<const void*, std::string> n;
    return n;
}
static std::string& log_text()
{
    static std::string t;
    return t;
}

extern "C" {

void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned, void*, void*, void*,
                           void*, int*)
{
    names()[host] = device_name;
}

int hipLaunchKernel(const void* host, Dim3 grid, Dim3, void**, size_t, void*)
{
    log_text() += names()[host] + " " + std::to_string(grid.x) + " " + std::to_string(grid.y) + "\n";
    return 0;
}

const char* recorder_log() { return log_text().c_str(); }
void recorder_clear() { log_text().clear(); }

}  // extern "C"
