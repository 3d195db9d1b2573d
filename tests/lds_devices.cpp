// Stands in for the HIP runtime's device, attribute and launch calls (the executable's own definitions come before the
// library's): launches prefill kernels with more than 64 KB of dynamic LDS on two pretended devices and checks that
// each launch was preceded, on its device, by the permission for that kernel and size.  Nothing runs on a GPU.
#include <cstdio>
#include <cstring>
#include <map>
#include <utility>

#include "../include/attn.h"

static int g_device = 0;
static std::map<std::pair<int, const void *>, int> g_allowed;
static int g_launches = 0, g_refused = 0;

struct Dim3 {
    unsigned x, y, z;
};

extern "C" {
int hipGetDevice(int *d)
{
    *d = g_device;
    return 0;
}
int hipFuncSetAttribute(const void *f, int, int value)
{
    g_allowed[{g_device, f}] = value;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **, size_t lds, void *)
{
    ++g_launches;
    const auto it = g_allowed.find({g_device, f});
    if (lds > 65536 && (it == g_allowed.end() || (size_t)it->second < lds)) ++g_refused;
    return 0;
}
int hipGetLastError(void) { return 0; }
// the compiler's kernel launch: configuration pushed, then popped by the kernel's host stub, which calls hipLaunchKernel
static Dim3 g_grid, g_block;
static size_t g_lds;
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *)
{
    g_grid = grid;
    g_block = block;
    g_lds = lds;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = g_grid;
    *block = g_block;
    *lds = g_lds;
    *stream = nullptr;
    return 0;
}
}

int main()
{
    attn_args a;
    memset(&a, 0, sizeof a);
    a.struct_bytes = sizeof a;
    a.num_seqs = 64;
    a.num_q_heads = 32;
    a.num_kv_heads = 8;
    a.q = a.k = a.v = a.out = (void *)0x1000;
    a.query_start_loc = a.seq_lens = (const int32_t *)0x2000;
    a.scale = 0.1f;
    a.causal = 1;
    for (int device = 0; device < 3; ++device)
        for (int repeat = 0; repeat < 2; ++repeat)
            for (int dtype = 0; dtype < 3; ++dtype)
                for (int d = 64; d <= 128; d += 64)
                    for (int len = 100; len <= 6000; len *= 60) {  // short: key split or small workgroups; long: large ones
                        g_device = device;
                        a.dtype = dtype;
                        a.head_dim = d;
                        a.max_q_len = a.max_kv_len = len;
                        a.total_q = len * a.num_seqs;
                        a.q_stride_tok = a.o_stride_tok = 32 * d;
                        a.kv_stride_tok = 8 * d;
                        a.q_stride_head = a.o_stride_head = a.kv_stride_head = d;
                        if (attn_prefill_varlen(&a, nullptr) != ATTN_OK) return 2;
                    }
    printf("%d launches, %d without permission\n", g_launches, g_refused);
    return g_refused != 0 || g_launches != 72;
}
