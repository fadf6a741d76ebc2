// Test infrastructure: the few entry points of the HIP runtime that libogq.so uses, for a machine without a GPU.  Preloaded
// in front of the runtime, they write down the kernels that the library brings and the launches that its calls make;
// nothing reaches a device.
#include <cstddef>
#include <cstdint>
#include <string>
#include <unordered_map>
#include <vector>

namespace {

struct Kernel {
    std::string name;  // as registered (mangled)
    uint64_t launches = 0;
};

std::vector<Kernel>& kernels()
{
    static std::vector<Kernel> list;
    return list;
}

std::unordered_map<const void*, size_t>& index_of()
{
    static std::unordered_map<const void*, size_t> map;
    return map;
}

struct Size {
    uint32_t x, y, z;
};

uint64_t launches = 0, unknown = 0;
size_t last = 0;
Size last_grid{}, last_block{};

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}

void __hipUnregisterFatBinary(void**) {}

void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    index_of()[host] = kernels().size();
    kernels().push_back(Kernel{name});
}

int hipLaunchKernel(const void* host, Size grid, Size block, void**, size_t, void*)
{
    ++launches;
    const auto at = index_of().find(host);
    if (at == index_of().end()) {
        ++unknown;
        return 98;  // hipErrorInvalidDeviceFunction
    }
    last = at->second;
    last_grid = grid;
    last_block = block;
    ++kernels()[last].launches;
    return 0;
}

// What was written down.
uint64_t recorded_launches(void) { return launches; }
uint64_t recorded_unknown(void) { return unknown; }
size_t recorded_kernels(void) { return kernels().size(); }
const char* recorded_name(size_t i) { return kernels()[i].name.c_str(); }
uint64_t recorded_launches_of(size_t i) { return kernels()[i].launches; }
size_t recorded_last(void) { return last; }
uint32_t recorded_last_blocks(void) { return last_grid.x; }
uint32_t recorded_last_threads(void) { return last_block.x; }

}  // extern "C"
