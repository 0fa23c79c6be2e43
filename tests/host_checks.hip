// The C ABI of the codec with the launches recorded instead of made, for tests/test_launch_plans.py (a library of its own; needs
// no device): the host side of division.hip over bridges that write down what they are handed.
#define DIVISION_PART 3
#include "../paper_2208_04187_amd/csrc/division.hip"

struct check_launch {
    int what;                     // 0 compress, 1 decompress, 2 decompress of several shapes, 3 relu
    int kind, dt, waves;
    uint32_t gx, gy, walked;      // walked: maps whose planes the workgroups walk over together (0: none)
    uint32_t shapes, maps;        // of a launch of several shapes
    const void* out;              // the first map's output
};
static std::vector<check_launch> recorded;

static hipError_t note_compress(const void* p, int dt, int what) {
    const CompLaunch& c = *static_cast<const CompLaunch*>(p);
    recorded.push_back({what, c.kind, dt, c.kind == REGS || c.kind == UNITS ? c.nw : 0, c.gx, c.gy, c.kind == REGS ? c.ra.maps : 0u, 1, c.gy, nullptr});
    return hipSuccess;
}
static hipError_t note_decompress(const void* p, int dt) {
    const DecLaunch& c = *static_cast<const DecLaunch*>(p);
    recorded.push_back({1, c.kind, dt, 0, c.gx, c.gy, 0, 1, c.gy, c.a.tab.xhat[0]});
    return hipSuccess;
}
static hipError_t note_mixed(const void* p, int dt) {
    const MixLaunch& c = *static_cast<const MixLaunch*>(p);
    uint32_t shapes = 0, chunks = 0, maps = 0;
    while (shapes < (uint32_t)kMixShapes && c.a.first[shapes] != 0xffffffffu) ++shapes;
    for (uint32_t i = 0; i < shapes; ++i) {
        const uint32_t end = i + 1 < shapes ? c.a.first[i + 1] : c.grid;
        chunks = end - c.a.first[i];
        maps += chunks / c.a.chunks[i];
    }
    recorded.push_back({2, 0, dt, 0, c.grid, 1, 0, shapes, maps, c.a.xhat[0]});
    return hipSuccess;
}
#define BRIDGES(name, dt) \
    hipError_t division_bridge_compress_##name(const void* c, int) { return note_compress(c, dt, 0); } \
    hipError_t division_bridge_decompress_##name(const void* c, int) { return note_decompress(c, dt); } \
    hipError_t division_bridge_decompress_mixed_##name(const void* c, int) { return note_mixed(c, dt); } \
    hipError_t division_bridge_relu_##name(const void* c, int) { return note_compress(c, dt, 3); }
BRIDGES(f32, 0)
BRIDGES(bf16, 1)
BRIDGES(c16, 2)

extern "C" {
size_t division_mask_bytes(int64_t n) { return n < 0 ? 0 : 4 * (((size_t)n + 31) / 32); }
int division_relu_forward(const void*, int64_t, division_dtype, void*, void*, size_t, void*) { return DIVISION_OK; }

// copies up to cap recorded launches, forgets all of them and returns how many there were
int check_take_launches(check_launch* out, int cap) {
    const int n = (int)recorded.size();
    for (int i = 0; i < n && i < cap; ++i) out[i] = recorded[(size_t)i];
    recorded.clear();
    return n;
}
int check_cus(void) { return num_cus(); }
// what compress_rowstrip reads of a round: elements of the map in front of it, bytes from there on
uint32_t check_round_span(uint32_t p0, uint32_t planes, uint32_t HW, uint32_t es, uint32_t* bytes) {
    const RoundSpan span = round_span(p0, planes, HW, es);
    *bytes = span.bytes;
    return span.before;
}
}
