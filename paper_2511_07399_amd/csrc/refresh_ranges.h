// How the launches of a sink / RoPE refresh cut caches whose element counts exceed what a launch can index: kernels count
// 16-byte pieces in 32 bits, and a grid has at most 65535 rows.  Host code without dependencies.
#pragma once

namespace sdv2 {

constexpr long long kMaxPieces = 1ll << 31;      // 16-byte pieces of a launch
constexpr int kMaxGridRows = 65535;              // heads of a launch that has one grid row per head

// f(h0, heads, t0, tokens) for ranges that cover H heads x T tokens of `pieces` pieces each, every range at most kMaxPieces
// pieces and max_heads heads.  One range wherever everything fits.
template <typename F>
void for_refresh_ranges(int H, int T, int pieces, int max_heads, F&& f) {
    const long long most_tokens = kMaxPieces / pieces;
    const int tokens = T < most_tokens ? T : (int)most_tokens;
    long long heads = kMaxPieces / ((long long)tokens * pieces);
    if (heads > max_heads) heads = max_heads;
    for (int h0 = 0; h0 < H;) {
        const int hn = H - h0 < heads ? H - h0 : (int)heads;
        for (int t0 = 0; t0 < T;) {
            const int tn = T - t0 < tokens ? T - t0 : tokens;
            f(h0, hn, t0, tn);
            t0 += tn;
        }
        h0 += hn;
    }
}

}  // namespace sdv2
