// rtcc_rotated_nms: the NMS kernels of the join, on caller-provided records.
// Argument checks, scratch allocation and the launch only; the work is in
// kernels/nms.hip.
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/rtcc.h"
#include "kernels/kernels.hpp"

namespace rtcc {
void set_thread_error(const std::string &msg);
}

namespace {

// The call's device memory, one allocation for every part.
struct Scratch {
    void *base = nullptr;
    size_t bytes = 0;
    size_t part(size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) & ~size_t(255);
        return at;
    }
    template <class T>
    T *at(size_t off) const {
        return reinterpret_cast<T *>(static_cast<char *>(base) + off);
    }
    ~Scratch() {
        if (base) (void)hipFree(base);
    }
};

rtcc_status fail(rtcc_status s, const std::string &msg) {
    rtcc::set_thread_error(msg);
    return s;
}

rtcc_status hip_fail(hipError_t e, const char *what) {
    return fail(e == hipErrorOutOfMemory ? RTCC_E_NOMEM : RTCC_E_HIP,
                std::string(what) + " failed: " + hipGetErrorString(e));
}

}  // namespace

extern "C" RTCC_API rtcc_status rtcc_rotated_nms(const float *device_records, int64_t n, int32_t max_candidates,
                                                 float iou_threshold, float *device_out, int64_t *kept) {
    if (!kept) return fail(RTCC_E_ARG, "kept is NULL");
    *kept = 0;
    if (n < 0 || n > 2147483647) return fail(RTCC_E_ARG, "n out of range");
    if (max_candidates < 1 || max_candidates > rtcc::kern::kNmsMaxCandidates)
        return fail(RTCC_E_ARG, "max_candidates must be in [1, 16384]");
    if (!(iou_threshold >= 0.f && iou_threshold <= 1.f)) return fail(RTCC_E_ARG, "iou_threshold must be in [0, 1]");
    if (n == 0) return RTCC_OK;
    if (!device_records || !device_out) return fail(RTCC_E_ARG, "NULL records or output");

    const size_t m = size_t(max_candidates), listed = rtcc::kern::nms_listed(max_candidates);
    Scratch sc;
    const size_t o_count = sc.part(64), o_key = sc.part(size_t(n) * 4), o_order = sc.part(m * 4);
    const size_t o_foot = sc.part(m * rtcc::kern::kNmsFootDoubles * 8), o_mask_t = sc.part(m * 8);
    const size_t o_rows = sc.part(listed * 4), o_words = sc.part(listed * 8), o_colcount = sc.part((m + 63) / 64 * 4);
    hipError_t e = hipMalloc(&sc.base, sc.bytes);
    if (e != hipSuccess) return hip_fail(e, "hipMalloc");
    hipStream_t s = nullptr;
    e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    if (e != hipSuccess) return hip_fail(e, "hipStreamCreateWithFlags");
    int32_t *count = sc.at<int32_t>(o_count);  // n, kept, NaN-score flag
    int32_t host_out[2] = {0, 0};
    rtcc::kern::NmsArgs a{};
    a.rec = device_records;
    a.count = count;
    a.key = sc.at<uint32_t>(o_key);
    a.order = sc.at<int32_t>(o_order);
    a.foot = sc.at<double>(o_foot);
    a.mask_t = sc.at<unsigned long long>(o_mask_t);
    a.colrows = sc.at<int32_t>(o_rows);
    a.colwords = sc.at<unsigned long long>(o_words);
    a.colcount = sc.at<int32_t>(o_colcount);
    a.out = device_out;
    a.out_count = count + 1;
    a.bad_score = count + 2;
    a.iou_threshold = double(iou_threshold);
    a.max_candidates = max_candidates;
    e = rtcc::kern::nms_keys(device_records, int32_t(n), sc.at<uint32_t>(o_key), count, s);
    if (e == hipSuccess) e = rtcc::kern::rotated_nms(a, n, s);
    if (e == hipSuccess) e = hipMemcpyAsync(host_out, count + 1, sizeof(host_out), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
    if (e != hipSuccess) return hip_fail(e, "rotated NMS");
    if (host_out[1]) return fail(RTCC_E_ARG, "a record's score is NaN (no defined ranking)");
    *kept = host_out[0];
    return RTCC_OK;
}
