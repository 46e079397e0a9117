// What the library launches, on the host alone: the runtime's entry points below take the place of the real ones (256 compute
// units, launches are counted, the n-th one can be made to fail), so nothing reaches a GPU.  Prints one line per question.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>

#include "../include/balancekv.h"
#include "../paper_2502_07861_amd/csrc/bkv_host.h"

static int launches, fail_at;
static hipError_t last;

extern "C" {
hipError_t hipGetDevice(int* dev) { *dev = 0; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) { memset(p, 0, sizeof(*p)); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) { *grid = dim3(1); *block = dim3(1); *lds = 0; *st = nullptr; return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return last = ++launches == fail_at ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
}

static bkv_params params(int d, int block, int rounds, int dtype) {
    bkv_params p;
    memset(&p, 0, sizeof(p));
    p.d = d; p.block = block; p.rounds = rounds; p.dtype = dtype; p.flags = BKV_CENTER_KEYS | BKV_STRICT_HALF;
    return p;
}
static void* const some = (void*)(uintptr_t)0x100000;                 // an address that nothing reads
static bkv_stream* stream(const bkv_params& p, int64_t n_seq) {
    const int64_t cap_num = 4 * p.block, cap_den = 8 * p.block;
    bkv_stream* h = nullptr;
    const int rc = bkv_stream_init(&h, &p, n_seq, 0, 4, cap_num, cap_den, 0, 0.f, 0.f, some, bkv_stream_bytes(&p, n_seq, 4, cap_num, cap_den), nullptr);
    if (rc != BKV_OK) printf("init %d\n", rc);
    return h;
}

int main() {
    // launches of the tokens b - 1, b, b + 1 and 2 b (counted from 1)
    for (int T : {0, 1, 2})
        for (int64_t n_seq : {1, 256, 257, 4096}) {
            const bkv_params p = params(128, 64, T, BKV_BF16);
            bkv_stream* h = stream(p, n_seq);
            int n[130];
            for (int j = 1; j <= 128; ++j) n[j] = bkv_stream_append(h, some, some, nullptr, nullptr, nullptr);
            printf("append T=%d n_seq=%d: %d %d %d %d, seen %d\n", T, (int)n_seq, n[63], n[64], n[65], n[128], (int)bkv_stream_tokens_seen(h));
            bkv_stream_free(h);
        }
    // the launch that takes the token in fails: the token is not counted, the next call takes it
    for (int64_t n_seq : {1, 257})
        for (int at : {1, 64}) {
            const bkv_params p = params(64, 64, 1, BKV_F32);
            bkv_stream* h = stream(p, n_seq);
            for (int j = 1; j < at; ++j) bkv_stream_append(h, some, some, nullptr, nullptr, nullptr);
            launches = 0; fail_at = 1;
            const int rc = bkv_stream_append(h, some, some, nullptr, nullptr, nullptr);
            const int seen = (int)bkv_stream_tokens_seen(h);
            fail_at = 0;
            const bool again = bkv_stream_append(h, some, some, nullptr, nullptr, nullptr) > 0;
            printf("failed n_seq=%d at=%d: %s, seen %d, again %d, seen %d\n", (int)n_seq, at, rc == BKV_EHIP ? "EHIP" : "?", seen, (int)again,
                   (int)bkv_stream_tokens_seen(h));
            bkv_stream_free(h);
        }
    // a halving launch that is to take a token in, with one of the things it needs left out: refused, nothing launched
    for (int without = 0; without < 5; ++without) {
        bkv::CompressArgs a;
        memset(&a, 0, sizeof(a));
        a.b = 64; a.flags = without == 3 ? 0 : BKV_VALUE_GRAM; a.blocks_per_seq = 1; a.desc = (bkv::InstDesc*)some;
        a.K = a.V = (const char*)some; a.tok_k = (const char*)some; a.tok_v = without == 1 ? nullptr : (const char*)some;
        a.carry_w = without == 2 ? nullptr : (float*)some; a.carry_idx = a.carry_cnt = (int32_t*)some;
        a.stream.n_seq = without == 4 ? 7 : 8;
        launches = 0;
        const hipError_t e = bkv::launch_compress(BKV_BF16, 128, false, a, 8, nullptr);
        printf("token without=%d: %s, %d launches\n", without, e == hipSuccess ? "ok" : e == hipErrorInvalidValue ? "invalid" : "?", launches);
    }
    return 0;
}
