// What the entry points for several products launch, for tests on the CPU: reads "fused|list batch count" and then "M K b" per item,
// writes the launches of that call as "kernel:items" ("alu_list", "tile_list", "alu_fused", "tile_fused", "single"), then "clean" if
// nothing past the items of a work list was left as it was found on the stack, else "dirty".
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/apgemv.h"
#include "../../paper_2402_10517_amd/csrc/dense_gemm.h"
#include "../../paper_2402_10517_amd/csrc/handle.h"
#include "../../paper_2402_10517_amd/csrc/kernels.h"

static std::string seen;
static bool clean;

static hipError_t note(const char *kernel, int items)
{
    seen += std::string(kernel) + ":" + std::to_string(items) + " ";
    return hipSuccess;
}

static hipError_t note_list(const char *kernel, const apgemv::ListArgs &a)
{
    static const apgemv::ListItem none[apgemv::kMaxListItems] = {};
    if (std::memcmp(a.item + a.count, none, (apgemv::kMaxListItems - a.count) * sizeof(none[0])) != 0) clean = false;
    return note(kernel, a.count);
}

namespace apgemv {
hipError_t launch_gemv(const GemvArgs &, hipStream_t) { return note("single", 1); }
hipError_t launch_gemv_multi(const MultiArgs &a, int, int, hipStream_t) { return note("alu_fused", a.count); }
hipError_t launch_matrix_tile_multi(const MultiArgs &a, int, hipStream_t) { return note("tile_fused", a.count); }
hipError_t launch_matrix_tile_list(ListArgs &a, int, int, hipStream_t) { return note_list("tile_list", a); }
hipError_t launch_gemv_list(ListArgs &a, int, hipStream_t) { return note_list("alu_list", a); }
hipError_t launch_dequantize(const GemvArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_probe_read(const void *, size_t, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_probe_issue(int, int, hipStream_t) { return hipErrorInvalidValue; }
bool static_scratch_setup() { return false; }
bool dense_gemm_f16(const void *, const void *, void *, int, int, int, hipStream_t) { return false; }
} // namespace apgemv

static void fill_the_stack()
{
    volatile char used[1 << 16];
    for (size_t i = 0; i < sizeof(used); ++i) used[i] = 0x5a;
}

int main()
{
    char kind[16];
    int batch, count;
    while (std::scanf("%15s %d %d", kind, &batch, &count) == 3) {
        std::vector<ap_matrix> m(count);
        std::vector<ap_gemv_item> fused(count);
        std::vector<ap_gemv_list_item> list(count);
        char *fake = reinterpret_cast<char *>(0x100000);
        int b = 0;
        for (int i = 0; i < count; ++i) {
            std::memset(&m[i], 0, sizeof(m[i]));
            m[i].tag = apgemv::kHandleTag;
            m[i].hdr.n = 8;
            m[i].hdr.lut_mask = 0x1f8;
            m[i].dev = reinterpret_cast<uint8_t *>(fake);
            m[i].row_groups_per_wg = -1;
            if (std::scanf("%d %d %d", &m[i].hdr.M, &m[i].hdr.K, &b) != 3) return 1;
            fused[i] = {&m[i], fake, fake};
            list[i] = {&m[i], b, fake, fake};
        }
        seen.clear();
        clean = true;
        fill_the_stack();
        const ap_status s = !std::strcmp(kind, "fused") ? ap_gemv_multi(fused.data(), count, b, batch, nullptr)
                                                        : ap_gemv_list_batch(list.data(), count, batch, nullptr);
        if (s != AP_OK) return 2;
        std::printf("%s%s\n", seen.c_str(), clean ? "clean" : "dirty");
    }
    return 0;
}
