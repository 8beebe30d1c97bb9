/* Host-only check of what the entry points ask HIP for.  This program defines the few HIP functions through which libdream sets
 * kernel attributes and launches, so its definitions are used instead of the runtime's and nothing reaches a device.
 *
 *   - dream_init() raises, for the current device, the dynamic-LDS limit of every kernel that needs it: no later call raises one (it
 *     might be under capture);
 *   - no launch asks for more LDS than its kernel's limit (64 KB where none was raised), nor for an empty or oversized grid.
 */
#include <stdio.h>
#include <stdlib.h>
#include "dream.h"

typedef struct { unsigned x, y, z; } grid3;

enum { MAX_FUNCS = 256 };
static const void *func[MAX_FUNCS];
static int limits[2][MAX_FUNCS], launched[MAX_FUNCS], n_funcs, initialised, late, bad, device;   /* two devices, each with limits of its own */
static long launches;

static int index_of(const void *f)
{
    int i = 0;
    while (i < n_funcs && func[i] != f)
        i++;
    if (i == MAX_FUNCS)
        exit(3);
    if (i == n_funcs) {
        func[n_funcs] = f;
        limits[0][n_funcs] = limits[1][n_funcs] = 65536;
        n_funcs++;
    }
    return i;
}
int hipGetDevice(int *current) { *current = device; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = (void *)0x10000; return 0; }
int hipFuncSetAttribute(const void *f, int attribute, int value)
{
    (void)attribute;
    late += initialised;
    limits[device][index_of(f)] = value > 65536 ? value : 65536;
    return 0;
}
/* (a launch is these two around the kernel's host stub, which calls hipLaunchKernel) */
static struct { grid3 grid, block; size_t lds; void *stream; } config;
int __hipPushCallConfiguration(grid3 grid, grid3 block, size_t lds, void *stream)
{
    config.grid = grid;
    config.block = block;
    config.lds = lds;
    config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(grid3 *grid, grid3 *block, size_t *lds, void **stream)
{
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, grid3 grid, grid3 block, void **args, size_t lds, void *stream)
{
    const int i = index_of(f), limit = limits[device][i];
    (void)args; (void)stream;
    launches++;
    launched[i]++;
    if (lds > (size_t)limit || lds > 163840 || !grid.x || !grid.y || !grid.z || grid.y > 65535 || grid.z > 65535 || block.x * block.y * block.z > 1024) {
        printf("launch %ld: %zu bytes of LDS with a limit of %d, grid %u x %u x %u\n", launches, lds, limit, grid.x, grid.y, grid.z);
        bad++;
    }
    return 0;
}

static void expect(int status, int line)
{
    if (status) {
        printf("line %d: status %d, %s\n", line, status, dream_last_error());
        bad++;
    }
}
#define OK(call) expect(call, __LINE__)

static void sweep(void)
{
    static const int dims[3] = {64, 128, 256};
    void *const p = (void *)0x10000;         /* never dereferenced: nothing runs */
    const size_t all = (size_t)1 << 40;
    int i, j, b;
    for (i = 0; i < 3; i++) {
        static const int rows[] = {1, 16, 17, 32, 33, 48, 64, 65, 80, 96, 97, 112, 113, 128, 129, 300};
        static const int heads[] = {1, 8, 32, 64, 200};
        const int d = dims[i];
        for (j = 0; j < (int)(sizeof rows / sizeof *rows); j++)
            for (b = 0; b < (int)(sizeof heads / sizeof *heads); b++) {
                const dream_attn_desc desc = {1, heads[b], heads[b], d, DREAM_BF16, 0.0f, 500};
                OK(dream_project_rows(&desc, p, rows[j], 1024, p, heads[b], p, NULL, p, NULL));
            }
        for (b = 1; b <= 40; b = b < 9 ? b + 1 : b * 2) {
            static const int group[][2] = {{1, 1}, {8, 8}, {8, 4}, {32, 32}, {32, 8}, {28, 4}, {64, 8}};
            static const int trees[] = {1, 10, 17, 60, 64, 100, 256};
            static const int keys[] = {300, 770, 1340, 4100};
            for (j = 0; j < (int)(sizeof group / sizeof *group); j++) {
                const dream_attn_desc desc = {b, group[j][0], group[j][1], d, DREAM_BF16, 0.0f, 4200};
                int t, k;
                for (t = 0; t < (int)(sizeof trees / sizeof *trees); t++)
                    for (k = 0; k < (int)(sizeof keys / sizeof *keys); k++) {
                        OK(dream_tree_verify_attn(&desc, p, p, p, p, trees[t], p, NULL, keys[k], p, NULL, p, all, NULL));
                        OK(dream_draft_xattn(&desc, p, p, p, p, 200, p, trees[t], p, keys[k], p, p, all, NULL));
                    }
                for (k = 0; k < (int)(sizeof keys / sizeof *keys); k++) {
                    OK(dream_visual_compress(&desc, p, NULL, keys[k], p, keys[k], 0, keys[k] - 30, 1, 4, NULL, NULL, p, p, NULL, NULL, 0, NULL, 0, p, all, NULL));
                    OK(dream_visual_compress(&desc, p, p, 40, (char *)p + 2, keys[k], 3, 200, 1, 4, NULL, p, p, p, NULL, NULL, 0, NULL, 0, p, all, NULL));
                    OK(dream_attention_entropy(&desc, p, NULL, keys[k], p, keys[k], p, p, p, all, NULL));
                }
            }
        }
    }
    for (i = 1; i <= DREAM_MAX_VISUAL; i = i * 3 + 1) {
        const dream_attn_desc desc = {3, 1, 1, 64, DREAM_BF16, 0.0f, 20000};
        OK(dream_visual_compress(&desc, NULL, NULL, 0, NULL, 0, 0, i < 5000 ? i : DREAM_MAX_VISUAL, 1, 2, p, NULL, NULL, p, NULL, NULL, 0, NULL, 0, p, all, NULL));
    }
    for (i = 0; i < 2; i++)
        for (j = 100; j < 600000; j *= 7) {
            OK(dream_accept_path(p, i, 2, 60, j, p, p, 6, p, p, p, p, p, all, NULL));
            OK(dream_accept_path_static(p, i, 2, 60, j, p, p, 6, p, p, p, p, NULL));
            OK(dream_spec_accept(p, p, i, 2, 60, j, p, p, p, p, 6, 1.0f, p, p, p, p, all, NULL));
            OK(dream_tree_expand_level(p, i, 2, 10, j / 4, p, 5, p, p, p, p, all, NULL));
        }
    for (i = 1; i <= DREAM_MAX_POOL; i *= 2)
        OK(dream_tree_finalize(p, p, p, 4, i, 59, p, p, p, NULL, NULL));
}

int main(void)
{
    int i, used, raised;
    for (device = 0; device < 2; device++) {
        launches = 0;
        initialised = raised = used = 0;
        OK(dream_init());
        initialised = 1;
        for (i = 0; i < n_funcs; i++) {
            raised += limits[device][i] > 65536;
            launched[i] = 0;
        }
        sweep();
        for (i = 0; i < n_funcs; i++)
            used += launched[i] > 0 && limits[device][i] > 65536;
        printf("device %d: %d kernels with a raised limit, %d of them launched; raised after dream_init: %d; bad: %d; kernels seen: %d; launches: %ld\n",
               device, raised, used, late, bad, n_funcs, launches);
        if (late || bad || !launches || !used)
            return 1;
    }
    return 0;
}
