// When create may take device memory for another form of the blocks (the compressed
// copy of the passes, the SYRK's nonzero lists).  Plain C++, so that it can be checked
// on the host.
#pragma once

namespace ahlp {

// need: bytes of the copy; free: bytes free on the device; later: bytes the handle
// allocates at first use (FP32 factors and blocks, tuning).  A copy takes an eighth
// of what is left beside those at most, so that a problem that fits without it still
// does.
inline bool copy_fits(double need, double free, double later) { return 8.0 * need <= free - later; }

}  // namespace ahlp
