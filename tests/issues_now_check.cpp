// Host-only driver of tests/test_launch_rules.py: issues_now (csrc/adagc_internal.h) with the runtime's two calls stood in for, so that
// a stream's state and the error left behind are known.  Prints nothing and returns 0 if all is as it should be.
#include <cstdio>

#include "adagc_internal.h"

static hipError_t             answer, last_error;
static hipStreamCaptureStatus state;

hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* out)
{
    if (answer == hipSuccess) *out = state;
    else last_error = answer;
    return answer;
}

hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}

static int check(hipError_t e, hipStreamCaptureStatus s, bool expected)
{
    answer = e;
    state = s;
    last_error = hipSuccess;
    const bool now = adagc::issues_now(nullptr);
    if (now == expected && last_error == hipSuccess) return 0;
    std::printf("answer %d, state %d: issues_now %d, error left behind %d\n", (int)e, (int)s, (int)now, (int)last_error);
    return 1;
}

int main()
{
    return check(hipSuccess, hipStreamCaptureStatusNone, true) + check(hipSuccess, hipStreamCaptureStatusActive, false) +
           check(hipSuccess, hipStreamCaptureStatusInvalidated, false) + check(hipErrorStreamCaptureImplicit, hipStreamCaptureStatusNone, false) +
           check(hipErrorInvalidHandle, hipStreamCaptureStatusNone, false);
}
