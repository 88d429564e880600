// Numbers of the light frames (fltop_beam_light.inc): plain C++, the same on the host, where the choice
// of a build needs them and tests run them under the sanitizers.  (Constant-expression functions are
// device functions as well.)
#ifndef FLTOP_LIGHT_H_
#define FLTOP_LIGHT_H_

#include <cstdint>

namespace fltop {

constexpr int kLightBins = 256;  // bins of their selection, 16 bits each

// How a light frame lays its candidates out: wavefronts with the stays, one thread per beam entry, and
// behind them blocks of 1 << lg threads, each with the beam's extensions by one non-blank survivor, in up to
// kLightRounds rounds.
constexpr int kLightRounds = 3;  // most extensions per thread
struct LightShape {
    int lg, stay_waves, blocks;
};
constexpr LightShape light_shape(int beam, int threads) {
    LightShape s{0, 1, 0};
    while ((1 << s.lg) < beam) ++s.lg;
    s.stay_waves = ((1 << s.lg) + 63) / 64;
    s.blocks = (threads - s.stay_waves * 64) >> s.lg;
    return s;
}
// Places of their scores: the stays', then each round's.
constexpr int light_candidates(int beam, int threads) {
    const int stays = light_shape(beam, threads).stay_waves * 64;
    return stays + kLightRounds * (threads - stays);
}
// Frames that go through the tokens that can reach the beam only: how many such tokens at most (a lane holds
// one), and how many candidates that makes, in up to kReachRounds rounds.  With 256 threads a frame of more than
// 20 tokens is left to the general path: its candidates crowd about the cut, where they are ranked one by one
// (64 utterances x 500 frames, V = 32, beam 32, every token kept, which now have 512 threads: 848 us; up to 12 tokens
// 792, up to 31 1040; 16 utterances, beam 42: 941 / 974 / 929 us).  With 512 threads all have a place (128 x 400, V = 1024, beam 64,
// table in memory, R = 0.01: 64 tokens 819 us, 20 869, 12 904).
constexpr int kReachRounds = 8;
constexpr int reach_list_places(int blocks, int threads, int vocabulary) {
    const int most = threads > 256 ? 64 : 20;
    int n = kReachRounds * blocks;
    if (n > vocabulary - 1) n = vocabulary - 1;
    return n < most ? n : most;
}
constexpr int reach_candidates(int beam, int threads, int vocabulary) {
    const LightShape s = light_shape(beam, threads);
    const int stays = s.stay_waves * 64;
    const int n = s.blocks > 0 ? (reach_list_places(s.blocks, threads, vocabulary) + s.blocks - 1) / s.blocks : 0;
    return stays + n * (threads - stays);
}
// Where an entry's last token stands in the table of survivors by token.  The empty prefix has none (-1), and behind the
// beam's end anything may stand in its place: what LDS, or a stream's record, held before.
constexpr int light_token_row(bool there, int32_t last) { return there && last > 0 ? last : 0; }
// Rounds for so many non-blank survivors; more than kLightRounds: not a light frame.
constexpr int light_rounds(int blocks, int others) {
    int rounds = blocks > 0 ? 1 : kLightRounds + 1;
    while (rounds <= kLightRounds && rounds * blocks < others) ++rounds;
    return rounds;
}
// Whether a frame that keeps `kept` tokens can be one (blank may or may not be among them), in a build whose
// headers hold `inline_survivors`.
constexpr bool light_possible(int kept, int beam, int threads, int inline_survivors) {
    return kept <= inline_survivors && light_rounds(light_shape(beam, threads).blocks, kept - 1) <= kLightRounds;
}

// Bin of a candidate whose score lies `x` bins below the reference.  What has no mass lies infinitely
// far below, masked tokens farther than any integer counts, and a score may come out a little above
// the reference: the clamp has to come before the conversion, whose result is undefined outside the
// integer's range.
constexpr uint32_t light_bin(float x) {
    return (uint32_t)__builtin_fminf(__builtin_fmaxf(x, 0.0f), (float)(kLightBins - 1));
}

// What a light frame's bins cover is the spread of the beam's scores and a margin; both the width of a
// bin and its reciprocal have to stay finite.  The spread at least doubles while the cut lies in the
// last bin, which masked tokens in the beam can keep up for any number of frames, and a frame without
// candidates has none.  (1e30 nats in 256 bins: no farther than fp32 reaches by a wide margin, and the
// frames whose scores lie wider apart find theirs in the last bin.)
constexpr float kWidestSpread = 1e30f;
constexpr float light_spread_of(float spread) {
    return __builtin_fminf(__builtin_fmaxf(spread, 0.0f), kWidestSpread);
}
// Whether that leaves a spread as it is, with what its rounding adds (NaN: no).
constexpr bool spread_is_kept(double spread) { return spread < 0.5 * (double)kWidestSpread; }

}  // namespace fltop

#endif
