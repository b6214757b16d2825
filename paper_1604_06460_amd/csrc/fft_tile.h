// FFT passes on register tiles (fft_tile.hip) as fft.hip's dispatch sees them.
#pragma once

struct qs_state;

namespace qs {
namespace fftdev {
struct PassArgs;
}

// Whether the pass can run there (states of 10 qubits or more).
bool fft_tile_applies(int n, const fftdev::PassArgs &pa);

// Enqueues the pass from src to dst (which may be src unless the pass is
// final). Only the pass's digit, twiddle and order are used; columns are the
// launcher's own.
int launch_fft_tile(qs_state *h, const fftdev::PassArgs &pa, const void *src, void *dst);

}  // namespace qs
