"""The numbers that light frames work with, compiled for the host from the kernel's own header and run
under UndefinedBehaviorSanitizer (conversions out of an integer's range included): any report fails."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "fltop_light.h"
using namespace fltop;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\\n", __LINE__, #c); std::exit(1); } } while (0)
"""


def run(tmp_path, body):
    source, exe = tmp_path / "numbers.cpp", tmp_path / "numbers"
    source.write_text(HEAD + "int main() {\n" + body + "\nreturn 0; }\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined,float-cast-overflow",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2510_09085_amd", "csrc"),
                    str(source), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr[-2000:]


@pytest.mark.parametrize("x, bin_", [
    ("INFINITY", 255), ("3.4e38f", 255), ("4294967296.0f", 255), ("256.0f", 255), ("255.9f", 255),
    ("254.9f", 254), ("1.0f", 1), ("0.99f", 0), ("0.0f", 0), ("-0.5f", 0), ("-7.0f", 0),
    ("-3.4e38f", 0), ("-INFINITY", 0), ("NAN", 0)])
def test_every_distance_has_a_bin(tmp_path, x, bin_):
    """No mass, masked tokens, scores above the reference: inside the table, and defined."""
    run(tmp_path, f"volatile float x = {x}; CHECK(light_bin(x) == {bin_}u);")


@pytest.mark.parametrize("first", ["1.0f", "3.4e38f", "INFINITY", "NAN"])
def test_bins_stay_finite_however_long_the_cut_lies_in_the_last_one(tmp_path, first):
    """The recurrence of a light frame whose cut lies in the last row of bins (its spread becomes 512 of
    them), 2000 times, then one without candidates; `first` is the spread it is entered with."""
    run(tmp_path, f"""
    volatile float margin = 1.6f;
    float spread = light_spread_of({first});
    for (int frame = 0; frame < 2000; ++frame) {{
        const float scale = (float)kLightBins * (1.0f / (spread + margin)), width = 1.0f / scale;
        CHECK(scale > 1.2e-38f && std::isfinite(width));  // (the reciprocal flushes subnormals)
        CHECK(light_bin((float)1e41 * scale) == 255u && light_bin(-1.0f * scale) == 0u);
        spread = light_spread_of(width * 512.0f);
        CHECK(spread >= 0.0f);
    }}
    CHECK(light_spread_of((float)-62 * 4.0f) == 0.0f);""")


@pytest.mark.parametrize("threads", [128, 256])
def test_a_build_without_light_frames_is_taken_only_where_none_can_be_one(tmp_path, threads):
    """Frames that all keep the same number of tokens (R = 0), against the layout spelled out: threads behind
    those of the stays, one per beam entry (a power of two) and token, three times over at most."""
    run(tmp_path, f"""
    for (int beam = 1; beam <= {threads} / 2; ++beam) {{
        int size = 1;
        while (size < beam) size *= 2;
        const int behind = {threads} - (size <= 64 ? 64 : 128);
        for (int kept = 2; kept <= 12; ++kept) {{
            const bool fits = kept <= 6 && 3 * (behind / size) >= kept - 1;
            CHECK(light_possible(kept, beam, {threads}, 6) == fits);
        }}
        CHECK(light_rounds(light_shape(beam, {threads}).blocks, 1) <= kLightRounds);
    }}""")


@pytest.mark.parametrize("threads", [128, 256])
def test_scores_of_every_round_have_a_place(tmp_path, threads):
    """The last thread's last round, at the index the kernel writes it to."""
    run(tmp_path, f"""
    for (int beam = 1; beam <= {threads} / 2; ++beam) {{
        const LightShape s = light_shape(beam, {threads});
        const int stays = 64 * s.stay_waves, behind = {threads} - stays;
        CHECK(beam <= stays && s.blocks << s.lg <= behind);
        CHECK({threads} - 1 + (kLightRounds - 1) * behind < light_candidates(beam, {threads}));
    }}""")


def test_a_spread_that_is_held_back_is_no_bound(tmp_path):
    """What `spread_is_kept` says of a spread in fp64, against what becomes of it in fp32."""
    run(tmp_path, """
    const double spreads[] = {0.0, 1.0, 1e9, 1e20, 4.9e29, 5.1e29, 1e30, 1e38, 1e39, 1e300, INFINITY, NAN};
    for (double spread : spreads) {
        const bool kept = spread_is_kept(spread);
        if (kept) CHECK((double)light_spread_of((float)spread * 1.0001f + 2e-3f) > spread);
        CHECK(kept == (spread < 5e29));
    }""")


def test_what_stands_behind_the_beam_is_no_index(tmp_path):
    """The place of an entry's last token in a table of V + 1: inside, whatever the place of an entry that was
    never written holds."""
    run(tmp_path, """
    const int32_t left_behind[] = {-1, 0, 5, 31, 32, 4096, 1 << 28, 2147483647, -2147483647 - 1};
    for (int32_t last : left_behind) {
        CHECK(light_token_row(false, last) == 0);
        if (last < 32) CHECK(light_token_row(true, last) == (last > 0 ? last : 0));
    }""")


@pytest.mark.parametrize("threads", [256, 512])
def test_everything_of_a_listed_token_has_a_place(tmp_path, threads):
    """Frames that go through a list of tokens: the last thread's last round, and the notes of the list's last token, at
    the indices the kernel writes them to."""
    run(tmp_path, f"""
    const int vocabularies[] = {{2, 5, 21, 29, 64, 65, 300, 2048}};
    for (int V : vocabularies)
        for (int beam = 1; beam <= 128; ++beam) {{
            const LightShape s = light_shape(beam, {threads});
            const int stays = 64 * s.stay_waves, behind = {threads} - stays;
            CHECK(s.blocks > 0 && s.blocks << s.lg == behind && beam <= 1 << s.lg);
            const int places = reach_list_places(s.blocks, {threads}, V);
            CHECK(places >= 1 && places <= 64 && places < V);  // (a lane each)
            int last_score = stays - 1, last_note = 0;
            for (int tid = stays; tid < {threads}; ++tid) {{
                const int k0 = (tid - stays) >> s.lg, own = (tid - stays) & ((1 << s.lg) - 1);
                for (int k = k0, slot = tid; k - k0 < places; k += s.blocks, slot += behind) {{
                    if (slot > last_score) last_score = slot;
                    const int note = ((k < places ? k : places - 1) << s.lg) + own;
                    if (note > last_note) last_note = note;
                }}
            }}
            CHECK(last_score < reach_candidates(beam, {threads}, V));
            CHECK(last_note < places << s.lg);
        }}""")
