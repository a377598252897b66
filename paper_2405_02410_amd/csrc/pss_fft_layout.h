// LDS sizes of the line transforms (pss_fft.h), shared with the host code
// that sizes the kernels' dynamic LDS.
#pragma once

// one pad element after every 2^PSS_FFT_PAD elements of an exchange region
#ifndef PSS_FFT_PAD
#define PSS_FFT_PAD 3
#endif

namespace pss {

// pad shift (a step of 256 lattices of 128^2 held in LDS: 20.0 us with one pad
// element in 8, 20.6 with one in 16, 20.9 in 32, 22.4 without)
constexpr int kFftPad = PSS_FFT_PAD;

// D(t): the first output index that thread t of L/P holds after a transform
// of a line of L (LineFFT::drev, pss_fft.h), on the host
inline int fft_drev(int L, int P, int t) {
    int M = 1;
    while (M * P <= L) M *= P;
    int Ls = L, G = L / P, R = L / M > 1 ? L / M : P, d = 0, mul = 1;
    while (Ls > R) {
        const int Gn = G / R;
        if (G > 1) {
            d += mul * (t / Gn);
            mul *= R;
            t &= Gn - 1;
        }
        Ls /= R;
        G /= R;
        R = P;
    }
    return d;
}

// elements of one exchange region of a line of L points
constexpr int fft_region(int L) { return L + (L >> kFftPad); }

// Exchange regions of a line held by L/P threads: one within a wave; a line
// of several waves adds two block buffers used in turn, or, from 2048 points
// at 8 or more a thread, one that is guarded by a second barrier.  With three
// regions a line of 4096 left room for one block of four waves per CU, with
// two it is two blocks of eight.
constexpr bool fft_one_buffer(int L, int P) { return L >= 2048 && P >= 8; }
constexpr int fft_regions(int L, int P) { return L / P <= 64 ? 1 : (fft_one_buffer(L, P) ? 2 : 3); }

// LDS elements of the line transforms of `lines` lines of L points held by
// L/P threads each
constexpr int fft_lds_elems(int L, int P, int lines) {
    return lines * fft_regions(L, P) * fft_region(L);
}
// the packed line's exchange: its own L elements, or the line's block buffer
constexpr int fft_xbuf_elems(int L, int P) { return L / P > 64 && fft_one_buffer(L, P) ? 0 : L; }

// Where the twiddles of a line held P points a thread live.  Up to 8 points:
// in registers (at most 20 complex values, read once and used by every
// transform of the kernel), except that lines of 2048 and more keep only the
// first stage's there and the later stages' (a table of 512) in LDS (the
// update kernel then takes 148 registers and not 180).  16 points: an LDS
// copy of the table (30 values would halve the waves in flight).
constexpr int kTwRegs = 0, kTwSplit = 1, kTwTable = 2;
constexpr int fft_tw_form(int L, int P) { return P > 8 ? kTwTable : (L >= 2048 && P == 8 ? kTwSplit : kTwRegs); }
constexpr int fft_tw_elems(int L, int P) {
    return fft_tw_form(L, P) == kTwRegs ? 0 : (fft_tw_form(L, P) == kTwSplit ? 512 : L);
}

}  // namespace pss
