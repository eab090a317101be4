// The table of chosen kernels (pc_choice of pc_internal.h) on the host: entries of one network do not drive each other out.
// Prints, for every network, how many of its shapes had to be planned again in a second iteration.
#include "pc_internal.h"

int main()
{
    for (int net = 0; net < 3; ++net) {
        pc_ctx *ctx = new pc_ctx();
        memset(ctx, 0, sizeof(*ctx));
        int again = 0, wrong = 0;
        for (int step = 0; step < 2; ++step) {
            int c = 64, h = net == 2 ? 56 : 32, l = 0;
            const int N = net == 2 ? 64 : 128;
            for (int s = 0; s < 4; ++s)
                for (int k = 0; k < (net ? 4 : 2); ++k, ++l) {
                    const int f = 64 << s, st = s && k == 0 ? 2 : 1, o = (h - 1) / st + 1;
                    const int32_t keys[3][PC_CHOICE_KEY] = {{5, N, h, h, c, f, o, o, st * 16 + 1, 6},
                                                            {st == 2 ? 6 : 5, N, o, o, f, st == 2 ? h : c, h, st == 2 ? c : h, st == 2 ? 0 : 17, st == 2 ? 0 : 7},
                                                            {7, N, h, h, c, f, st, f * c / 4, 0, 0}};
                    for (int q = 0; q < 3; ++q) {
                        bool hit;
                        int32_t *e = pc_choice(ctx, keys[q], &hit);
                        if (hit && *e < 0) ++wrong;
                        if (step && !hit) ++again;
                        *e = l;
                    }
                    c = f;
                    h = o;
                }
        }
        // more shapes than there are places: an entry that is found is the one that was stored
        for (int i = 0; i < 5000; ++i)
            for (int back = 0; back < 2; ++back) {
                const int v = i - 700 * back;
                if (v < 0) continue;
                const int32_t key[PC_CHOICE_KEY] = {5, 1, v, v, 8, 8, v, v, 17, 6};
                bool hit;
                int32_t *e = pc_choice(ctx, key, &hit);
                if (hit ? *e != v : *e != -1) ++wrong;
                *e = v;
            }
        printf("%d %d\n", again, wrong);
        delete ctx;
    }
}
