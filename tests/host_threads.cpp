// Driver for the schedules' enqueue threads under ThreadSanitizer: a chain of fully connected layers cut into Z stages, every mode,
// several steps each, on tests/lanes' runtime with launches not run.  An event record writes to the event and a wait reads it, so a
// wait that is not ordered behind its record is a race, too.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lpm.h"

extern "C" void lanes_host_only(int);
extern "C" long lanes_complaints();

#define CHECK(call)                                                                                     \
    do {                                                                                                \
        const int32_t rc__ = (call);                                                                    \
        if (rc__ < 0) { printf("%s: %d %s\n", #call, rc__, lpm_last_error()); return 1; }               \
    } while (0)

static void* mem(size_t n) { return aligned_alloc(256, (n + 255 + 256) & ~(size_t)255); }

static int run(int Z, int M, int window, int m, int steps) {
    std::vector<lpm_layer> net;
    for (int i = 0; i <= Z; ++i) {
        lpm_layer l{};
        l.kind = i == Z ? LPM_SOFTMAX_CE : LPM_FC;
        l.cin = l.cout = 128;
        l.kh = l.kw = l.stride = l.h_in = l.w_in = l.d_in = l.kd = 1;
        l.flags = i == Z ? 0 : LPM_BIAS | (i + 1 < Z ? LPM_RELU : 0);
        l.src = i - 1;
        l.add_src = LPM_NONE;
        l.cut_allowed_after = i + 1 < Z;
        net.push_back(l);
    }
    std::vector<lpm_stage*> st((size_t)Z);
    std::vector<lpm_stage_buffers> buf((size_t)Z);
    for (int z = 0; z < Z; ++z) {
        CHECK(lpm_stage_create(net.data(), (int32_t)net.size(), z, z + 1 < Z ? z + 1 : Z + 1, m, LPM_BF16, &st[(size_t)z]));
        size_t v[8];
        CHECK(lpm_stage_sizes(st[(size_t)z], &v[0], &v[1], &v[2], &v[3], &v[4], &v[5], &v[6], &v[7]));
        lpm_stage_buffers& b = buf[(size_t)z];
        memset(&b, 0, sizeof b);
        b.params = (float*)mem(v[0]); b.lowp = mem(v[1]); b.grads = (float*)mem(v[2]); b.momentum = (float*)mem(v[2]);
        b.fwd_ws = mem(v[4]); b.bwd_ws = mem(v[5]); b.params_alt = (float*)mem(v[0]); b.lowp_alt = mem(v[1]);
        for (int w = 0; w < window; ++w) { b.stash[w] = mem(v[3]); b.act_out[w] = mem(v[7]); b.grad_in[w] = mem(v[6]); }
    }
    void* x = mem((size_t)M * m * 128 * 2);
    int32_t* labels = (int32_t*)mem((size_t)M * m * 4);
    float* loss = (float*)mem(256);
    std::vector<int> modes = {LPM_LOCKED, LPM_OVERLAPPED, LPM_PIPELINED};
    if (window <= 2) modes.insert(modes.end(), {LPM_LOCKED | LPM_ASYNC_UPDATE, LPM_OVERLAPPED | LPM_ASYNC_UPDATE});
    lpm_schedule* s = nullptr;
    CHECK(lpm_schedule_create(st.data(), Z, M, window, &s));
    for (int mode : modes)
        for (int k = 0; k < (mode == LPM_PIPELINED ? 8 : steps); ++k)          // (one after the other without a pause: a thread may still be on its way out of the step before)
            CHECK(lpm_schedule_run(s, mode, x, labels, nullptr, buf.data(), 0, 0.1f, 0.9f, loss, (void*)0x10, (void*)0x20));
    CHECK(lpm_schedule_destroy(s));
    for (lpm_stage* q : st) CHECK(lpm_stage_destroy(q));
    return 0;
}

int main() {
    lanes_host_only(1);
    for (int Z : {1, 2, 3, 6, 40})
        for (int window : {1, 2, 3})
            for (int M : {1, 5}) {
                if (run(Z, M, window, 16, Z == 40 && M == 1 ? 100 : 8)) return 1;
                printf("Z %d window %d M %d\n", Z, window, M);
            }
    printf("done, %ld complaints\n", lanes_complaints());
    return 0;
}
