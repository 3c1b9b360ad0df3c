// Launch helpers that the device translation units of libsaq.so share.  Not
// part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.hpp"

namespace saq {

// The plan must be uploaded, and to the current device.
saq_status check_uploaded(const saq_plan* p, const char* what);
saq_status hip_status(hipError_t e, const char* what);

inline const SegEntry* device_segments(const saq_plan* p) {
    return reinterpret_cast<const SegEntry*>(static_cast<const char*>(p->dev) + p->layout.off_seg);
}
inline const float* device_weights(const saq_plan* p) {
    return reinterpret_cast<const float*>(static_cast<const char*>(p->dev) + p->layout.off_weight);
}

// Projected queries Qp [nq x max(D_kept, 1)] and ||q - c||^2 [nq], against
// the plan's c or, when ref is given, against that one row.
saq_status project_queries(const saq_plan* p, const float* Q, int32_t nq, const float* ref,
                           float* Qp, float* qn2, hipStream_t st);

// One dataset's rows to project.
struct ProjectItem {
    const float* X;             // [n x D]
    int64_t n;
    const void* M_split;        // device plan
    const float* c;
    const float* refs;          // per-row references (null: the plan's c)
    const int32_t* ref_ids;
    float* O;
    int64_t ld;
    float* norm2;               // null: not wanted
    int32_t D, k_pad, dk, n_refs;
    int32_t acc64, fill;        // fill: store the rows of the last 64-row tile past n too
};
// Whether the items are few enough for one workgroup per 32 x 32 block of the
// output, and that launch (project_few.hip); all items with references or none.
bool few_rows(const ProjectItem* items, int count);
saq_status launch_project_few(const ProjectItem* items, int count, int layout, hipStream_t st);

// One dataset's projected rows to quantize, adjust and pack.
struct QuantItem {
    const float* O;             // projected rows, leading dimension ld, in `layout`
    int64_t ld, n;
    const SegEntry* segs;       // device
    const float* norm2;
    uint8_t* codes;
    float* factors;
    int64_t code_bytes;
    int32_t layout, n_kept, dk, max_w;
};
// Whether the items are few enough for one wave per vector and segment, and
// that launch (quantize_few.hip).
bool few_vectors(const QuantItem* items, int count);
saq_status launch_quantize_few(const QuantItem* items, int count, int rounds, hipStream_t st);

// The plain scan on split bf16 operands (device.hip), for checked arguments and
// a workspace of saq_estimate_workspace_bytes.
saq_status scan_split(const saq_plan* p, const float* Q, int32_t nq, const float* ref,
                      const uint8_t* codes, const float* factors, int64_t n, int32_t prefix_bits,
                      float* out, void* ws, hipStream_t st);

// Device scratch of the integer scan for nq queries (scan.hip).
int64_t scan_workspace_bytes(const saq_plan* p, int32_t nq);

}  // namespace saq
