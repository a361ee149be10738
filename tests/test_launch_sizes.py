"""The host's launch arithmetic (csrc/launch_sizes.h), compiled with the host compiler and swept over its whole range."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_10111_amd", "csrc")


def _sweep(tmp_path, body):
    """Runs `body` (statements of a main() that print what is wrong) and returns what it printed."""
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text('#include <cstdio>\n#include "launch_sizes.h"\nusing namespace dq;\nint main() {\n' + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout


def test_a_prepared_mini_batch_fits_its_room_in_the_workspace(tmp_path):
    """CSR features, every width the library takes, margins cached or not: the entries that a block may prepare ahead fit the
    words the workspace holds per worker, and the staging buffer of the step that reads them; the plans fit in LDS."""
    out = _sweep(tmp_path, """
    long wider = 0;
    for (int64_t d = 1; d < (1ll << kColBits); ++d)
        for (int second = 0; second < 2; ++second) {
            CsrPlan p;
            if (!csr_plan(d, second, p)) { std::printf("no plan %ld\\n", (long)d); return 0; }
            const int cap = csr_prep_cap(d, p);
            if (cap < 1 || cap > p.cap || kPrepInts(cap) > csr_prep_stride(d)) std::printf("room %ld %d\\n", (long)d, second);
            if ((int64_t)p.lds > kLdsBudget - kCsrFixedLds || p.win % 4 || (int64_t)p.win * p.nwin < d || p.cap > kMaxStage)
                std::printf("lds %ld %d\\n", (long)d, second);
            wider += kPrepInts(p.cap) > csr_prep_stride(d);
        }
    if (wider == 0) std::printf("no width whose plan stages more than the workspace has room for\\n");
    CsrPlan p;
    if (csr_plan(1ll << kColBits, false, p)) std::printf("too wide\\n");
    """)
    assert out == "", out[:2000]


def test_the_full_gradient_masks_every_column_that_can_pass_the_end(tmp_path):
    """Dense features, every width above 1024: the shape covers the row, and the columns that are not masked hold whole quads
    of it for every thread."""
    out = _sweep(tmp_path, """
    for (int64_t d = 1025; d <= 16384; ++d) {
        const FullShape s = full_shape(d);
        if (s.threads < 256 || s.threads > 512 || s.threads % 64 || (int64_t)s.threads * s.cols < ceil_div(d, 4)) std::printf("shape %ld\\n", (long)d);
        if ((int64_t)s.threads * full_whole_cols(s.cols) > d / 4) std::printf("mask %ld\\n", (long)d);
        if (d < 2048 && 256 * full_whole_cols(2) > d / 4) std::printf("mask of 256 threads %ld\\n", (long)d);
    }
    """)
    assert out == "", out[:2000]


def test_both_sets_of_prepared_mini_batches_fit_the_workspace_of_a_run(tmp_path):
    """CSR features, with and without the row of differences: two sets of M mini-batches fit what the workspace holds behind
    its rows, a mini-batch's entries and their snapshot values fit its room, and no mini-batch is given less than before."""
    out = _sweep(tmp_path, """
    const int workers[] = {1, 2, 3, 8, 16, 63, 127}, rows[] = {1, 2, 31, 32, 255, 256};
    for (int64_t d = 1; d < (1ll << kColBits); d += 1 + d / 97)
        for (int second = 0; second < 2; ++second)
            for (int M : workers)
                for (int B : rows)
                    for (int snaps = 0; snaps < 2; ++snaps) {
                        CsrPlan p;
                        csr_plan(d, second, p);
                        const PrepRoom r = csr_prep_room(d, M, B, p, snaps);
                        const int64_t words = pad4(d) + 2 * M * csr_prep_stride(d), at = PrepLayout(B).entries;
                        bool ok = r.stride % 4 == 0 && (snaps ? 0 : pad4(d)) + 2 * M * r.stride <= words && r.cap <= p.cap;
                        ok = ok && at + 2ll * r.cap <= r.stride && (!snaps || (at + 3ll * r.snap_cap <= r.stride && r.snap_cap >= 1));
                        ok = ok && r.cap >= csr_prep_cap(d, p) && PrepLayout(B).dev_max < PrepLayout(B).y && PrepLayout(B).dev_max > PrepLayout(B).pre + B;
                        if (!ok) std::printf("d %ld M %d B %d %d %d\\n", (long)d, M, B, second, snaps);
                    }
    """)
    assert out == "", out[:2000]


def test_the_word_that_the_master_leaves_beside_a_prepared_mini_batch_is_in_none_of_its_tables(tmp_path):
    """CSR features: the master of a round writes PrepLayout::dev_max of a mini-batch prepared for B rows; the launch that left
    it and the one that reads it lay it out for B rows or for as many as a block takes.  In either layout the word is
    in no table, the tables hold their rows and do not overlap, and none reaches into the header or the entries."""
    out = _sweep(tmp_path, """
    for (int B = 1; B <= kCsrMaxRows; ++B)
        for (int rows = B; rows <= kCsrMaxRows; rows += rows < kCsrMaxRows ? kCsrMaxRows - rows : 1) {
            const PrepLayout at(rows);
            const int word = PrepLayout(B).dev_max;
            const int first[] = {0, at.row, at.len, at.pre, at.y, at.z, at.entries}, size[] = {4, B, B, B + 1, B, B, 1 << 20};
            for (int i = 0; i < 7; ++i) {
                if (word >= first[i] && word < first[i] + size[i]) std::printf("B %d of %d: word %d in table %d\\n", B, rows, word, i);
                if (first[i] % 4) std::printf("B %d of %d: table %d not on a quad\\n", B, rows, i);
                for (int j = 0; j < i; ++j)
                    if (first[i] < first[j] + size[j] && first[j] < first[i] + size[i]) std::printf("B %d of %d: tables %d %d\\n", B, rows, j, i);
            }
        }
    """)
    assert out == "", out[:2000]


def test_the_model_is_quantized_by_the_worker_for_light_mini_batches_only(tmp_path):
    """CSR features: little more entries on average than a block keeps in registers, no more than the width leaves room to prepare."""
    out = _sweep(tmp_path, """
    for (int64_t d = 4096; d <= 32768; d += 97)
        for (int B = 1; B <= 256; ++B)
            for (int per_row = 0; per_row <= 300; per_row += 1 + per_row / 8) {
                CsrPlan p;
                csr_plan(d, false, p);
                const bool light = csr_light_batches(B, 1000, 1000ll * per_row, 4096, p.cap);
                const int mean = B * (per_row ? per_row : 100);
                if (light && (mean > 4096 * 5 / 4 || mean > p.cap)) std::printf("heavy: d %ld B %d, %d a row\\n", (long)d, B, per_row);
                if (!light && mean <= 4096 && mean * 8 < p.cap * 7) std::printf("light: d %ld B %d, %d a row\\n", (long)d, B, per_row);
            }
    if (csr_light_batches(1, 1, 1ll << 60, 4096, 8192) || !csr_light_batches(1, 1ll << 40, 1, 4096, 8192)) std::printf("ends\\n");
    """)
    assert out == "", out[:2000]


def test_rounds_on_one_die_fit_the_workspace_and_the_chip(tmp_path):
    """CSR rounds in one launch, every width and number of workers: what the members share lies behind the rows of a step and inside a run's
    workspace; slices, chunks and threads cover every column; members, LDS and what a wavefront quantizes are within bounds."""
    out = _sweep(tmp_path, """
    const int rows[] = {1, 8, 32, 128}, widths[] = {2, 3, 8, 11, 16};
    const int64_t per_row[] = {0, 1, 9, 52, 400};
    long taken = 0;
    for (int64_t d = 1; d < (1ll << kColBits); d += 1 + d / 997)
        for (int M = 1; M <= 33; ++M) {
            const int64_t at = csr_run_offset(d, M);
            if (at % 16 || at < M * pad4(d) * 4 + M * 2 * kMaxSlices * 4 || at + kRoundsControl > csr_run_bytes(d, M)) std::printf("room d %ld M %d\\n", (long)d, M);
            for (int B : rows)
                for (int b_x : widths)
                    for (int64_t each : per_row) {
                        CsrRoundsShape s;
                        if (!csr_rounds_shape(d, 1000, 1000 * each, M, B, b_x, 8, s)) continue;
                        ++taken;
                        bool ok = M <= kDieUnits && s.want >= 1 && s.want <= kDieUnits && M * s.S <= s.want && s.S <= 16 && s.win % 256 == 0;
                        ok = ok && (int64_t)s.S * s.win >= d && (int64_t)(s.S - 1) * s.win < d && (int64_t)s.want * s.chunks * kChunk >= d;
                        ok = ok && s.chunks <= kMostChunks && M * s.chunks <= kPasses * kUnitWaves && s.room % 64 == 0 && s.room >= M * s.chunks * 64;
                        ok = ok && s.lds > 160 * 1024 / 2 - kRoundsFixedLds && s.lds + kRoundsFixedLds <= 160 * 1024;
                        ok = ok && s.lds >= 4 * (s.win + (d * b_x + 31) / 32 + 1 + s.room + pad4(d)) && s.cap <= kMaxStage;
                        if (!ok) std::printf("d %ld M %d B %d b_x %d %ld\\n", (long)d, M, B, b_x, (long)each);
                    }
        }
    CsrRoundsShape s;
    if (!taken || csr_rounds_shape(20958, 1000, 52000, 8, 32, 8, 7, s) || csr_rounds_shape(20958, 1000, 52000, 8, 32, 17, 8, s) ||
        csr_rounds_shape(20958, 1000, 52000, 8, 129, 8, 8, s) || !csr_rounds_shape(20958, 1000, 52000, 8, 32, 8, 8, s)) std::printf("ends\\n");
    """)
    assert out == "", out[:2000]


def test_launches_with_equal_parts_of_all_dies_pick_different_ones(tmp_path):
    """Two launches that begin together hold as many blocks on every die: which one a launch keeps is by lot, over all of them.  One that
    has more on a die keeps that one, and one without any its own."""
    out = _sweep(tmp_path, """
    int times[kDies] = {};
    for (uint32_t lot = 0; lot < 800; ++lot) {
        ++times[die_pick([](uint32_t i) { return i < 8 ? 16u : 0u; }, 3, lot)];
        for (uint32_t most = 0; most < kDies; ++most)
            if (die_pick([&](uint32_t i) { return i == most ? 17u : 16u; }, 3, lot) != most) std::printf("most %u lot %u\\n", most, lot);
        if (die_pick([](uint32_t) { return 0u; }, 3, lot) != 3) std::printf("none, lot %u\\n", lot);
    }
    for (uint32_t i = 0; i < kDies; ++i)
        if (times[i] != (i < 8 ? 100 : 0)) std::printf("die %u: %d\\n", i, times[i]);
    """)
    assert out == "", out[:2000]
