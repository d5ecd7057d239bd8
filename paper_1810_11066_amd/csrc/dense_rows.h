// Matrix products of few rows (dense_rows.hip).
#pragma once

#include "bs_internal.h"

namespace bs {
namespace rows {

// Rows up to which the kernel may serve a product of at least so many words per
// plane.  Measured per launch against the kernel that serves it otherwise
// (n = 4096, k = 4096, A2W2): 1 row 4.2 against 13.1 us, 16 rows 6.1 against
// 13.3, 32 rows 10.3 against 13.3, 48 rows 14.2 against 13.2; n = 1000, k =
// 800, A4W4: 1 row 4.0 against 6.5, 16 rows 5.0 against 6.9, 32 rows 8.2
// against 7.0.  At 16 words (k = 512) and at 1024 x 1 bit both take the 4 us
// an empty launch takes here.
constexpr int kFewRows = 16, kFewWords = 24;
constexpr int kMoreRows = 32, kMoreWords = 96;

// True for a matrix product (1x1, stride 1, no padding) the kernel serves on a
// device of cus compute units; pixel: the pixel kernel would serve it otherwise
// (the tiled kernel, if not).
bool covers(const ConvShape& s, int cus, bool pixel);

hipError_t launch_rows(const ConvShape& s, const uint32_t* act,
                       const uint32_t* wts, int32_t* out, hipStream_t st);

// The launch as text (snprintf semantics); enc names the encodings.
int describe(const ConvShape& s, const char* enc, char* buf, size_t len);

}  // namespace rows
}  // namespace bs
