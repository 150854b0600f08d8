"""Host-side check of the launchers' rules (csrc/launch_rules.h), compiled with the host compiler as they stand."""
import subprocess
from pathlib import Path

from paper_2406_09827_amd import build

CSRC = Path(__file__).resolve().parents[1] / "paper_2406_09827_amd" / "csrc"


def run(tmp_path, body: str) -> str:
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include "launch_rules.h"\n#include <cstdio>\n#include <initializer_list>\nusing namespace hipattn;\nint main() {\n' + body + "\nreturn 0; }\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", str(CSRC), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_row_offsets_of_the_prefill_attention_stay_within_32_bits(tmp_path):
    # the largest offset a lane forms (last row, last 16-byte chunk, load without an instruction offset) for lengths on either
    # side of the bound, and that a slice well below 4 GB is still taken
    out = run(tmp_path, r"""
    for (int d : {64, 128})
        for (int64_t row : {2LL * d, 512LL, 1024LL, 2048LL, 4096LL, 8192LL, 65536LL}) {
            const int64_t edge = (1LL << 32) / row;
            for (int64_t T = edge - 40 > 2 ? edge - 40 : 2; T <= edge + 2; ++T) {
                const int64_t largest = (T - 1) * row + (2 * d - 16) + kRowBias;
                if (rows_by_lane_offset(T, row, d) && (largest >= 1LL << 32 || T >= 1 << 24)) { std::printf("wraps: d %d row %lld T %lld\n", d, (long long)row, (long long)T); return 1; }
            }
            if (!rows_by_lane_offset(edge * 9 / 10 < (1 << 24) ? edge * 9 / 10 : (1 << 24) - 1, row, d)) { std::printf("refused: d %d row %lld\n", d, (long long)row); return 1; }
        }
    // lengths that the sum without the bias would let through
    const int64_t past[][2] = {{16777205, 256}, {16777215, 256}, {8388603, 512}, {8388607, 512}, {4194302, 1024}, {4194303, 1024}};
    for (auto &c : past) if (rows_by_lane_offset(c[0], c[1], 128)) { std::printf("taken: %lld\n", (long long)c[0]); return 1; }
    std::printf("ok %d\n", (int)rows_by_lane_offset(4194301, 1024, 128));
    """)
    assert out.strip() == "ok 1"


def test_workgroups_per_compute_unit_follow_the_bytes_of_keys(tmp_path):
    # 128 channels: 24 MB are 98304 tokens, 128 MB 524288; what a paged table or a cache with lengths on the device could hold cuts
    # nothing, and the pitch of the rows does not come into it
    out = run(tmp_path, r"""
    struct { int64_t T; int d; bool known; int want; } c[] = {
        {32768, 128, true, 0}, {65536, 128, true, 0}, {98304, 128, true, 0}, {98305, 128, true, 2}, {524288, 128, true, 2}, {524289, 128, true, 1},
        {1 << 20, 128, true, 1}, {131072, 64, true, 0}, {1 << 20, 64, true, 0}, {(1 << 20) + 1, 64, true, 2},
        {131072, 128, false, 0}, {1 << 20, 128, false, 0}, {1 << 23, 64, false, 0}};
    for (auto &x : c) if (mask_workgroups_per_cu(x.T, x.d, x.known) != x.want) { std::printf("%lld %d\n", (long long)x.T, x.d); return 1; }
    std::printf("ok\n");
    """)
    assert out.strip() == "ok"
    src = (CSRC / "mask_mfma_impl.h").read_text()
    assert "mask_workgroups_per_cu(p.max_kv_len, D, p.kv_lens == nullptr)" in src and "p.max_kv_len * p.ks_r" not in src


def test_workgroup_or_wave_per_item_of_the_prefill_mask(tmp_path):
    out = run(tmp_path, r"""
    struct { int64_t units; int kb, d; bool two_tiles, paged; int groups, gc; int64_t T; bool want; } c[] = {
        // blocks of a round, query tiles
        {1, 1024, 128, 0, 0, 8, 8, 1 << 20, 1}, {512, 16, 64, 1, 1, 5, 0, 1 << 20, 1}, {513, 32, 128, 0, 0, 8, 8, 16384, 0}, {513, 33, 128, 1, 1, 8, 8, 16384, 1},
        {768, 100, 128, 1, 0, 8, 8, 16384, 1}, {769, 128, 128, 1, 0, 8, 8, 16384, 0}, {769, 129, 128, 1, 0, 8, 8, 16384, 1}, {1024, 33, 64, 1, 0, 8, 8, 16384, 1},
        {1024, 33, 128, 0, 1, 8, 8, 16384, 1}, {1025, 128, 128, 0, 1, 8, 8, 16384, 0}, {1025, 129, 128, 0, 1, 8, 8, 16384, 1}, {1536, 512, 64, 0, 0, 8, 8, 16384, 1},
        {1537, 256, 128, 0, 1, 8, 8, 16384, 0}, {1024, 1024, 64, 0, 1, 8, 8, 16384, 1}, {1025, 1024, 64, 0, 1, 8, 8, 16384, 0}, {1025, 1024, 128, 0, 0, 8, 8, 16384, 0},
        {100000, 513, 128, 1, 1, 3, 0, 1 << 20, 1}, {100000, 512, 128, 1, 1, 8, 8, 16384, 0},
        // keys that an XCD reads at a time
        {768, 256, 128, 0, 0, 8, 8, 1 << 20, 1}, {769, 256, 128, 0, 0, 8, 8, 65536, 1}, {769, 256, 128, 0, 0, 8, 8, 65537, 0}, {1025, 256, 128, 0, 0, 8, 8, 32768, 1},
        {1025, 256, 128, 0, 0, 8, 8, 32769, 0}, {1025, 256, 64, 0, 0, 8, 8, 65536, 1}, {900, 256, 128, 0, 0, 12, 4, 32768, 1}, {900, 256, 128, 0, 0, 12, 4, 32769, 0},
        {900, 256, 128, 0, 0, 6, 2, 16384, 1}, {900, 256, 128, 0, 0, 6, 2, 32768, 0}, {1400, 256, 128, 0, 1, 6, 2, 1 << 20, 1}, {513, 256, 128, 0, 0, 1, 0, 49152, 1},
        {513, 256, 128, 0, 0, 1, 0, 49153, 0}, {513, 256, 128, 0, 1, 5, 0, 16384, 0}, {1400, 256, 128, 0, 0, 3, 0, 16384, 1}};
    for (auto &x : c)
        if (mask_item_per_workgroup(x.units, x.kb, x.d, x.two_tiles, x.paged, x.groups, x.gc, x.T) != x.want) {
            std::printf("%lld items, k/bk %d, %d groups, %lld tokens\n", (long long)x.units, x.kb, x.groups, (long long)x.T);
            return 1;
        }
    std::printf("ok\n");
    """)
    assert out.strip() == "ok"
    assert "mask_item_per_workgroup(units, p.kb, p.d, !one_tile, p.page_table != nullptr, groups, gc, p.max_kv_len)" in (CSRC / "mask_mfma_impl.h").read_text()


def test_waves_per_item_of_the_prefill_attention(tmp_path):
    out = run(tmp_path, r"""
    struct { int64_t items; int n_keys, d; bool paged; int groups, gc, T, want; } c[] = {
        {1, 64, 128, 0, 8, 8, 16384, 4}, {512, 2048, 64, 1, 5, 0, 16384, 4}, {513, 256, 128, 0, 8, 8, 16384, 1}, {513, 257, 128, 0, 8, 8, 16384, 2},
        {1024, 128, 128, 1, 8, 8, 16384, 1}, {1024, 129, 128, 1, 8, 8, 16384, 2}, {1024, 128, 64, 0, 8, 8, 16384, 1}, {1024, 256, 64, 0, 8, 8, 16384, 2},
        {1025, 512, 128, 1, 8, 8, 16384, 1}, {900, 512, 128, 0, 3, 0, 16384, 2}, {900, 512, 128, 0, 5, 0, 16384, 1}, {900, 512, 128, 1, 5, 0, 16384, 2}};
    for (auto &x : c) if (attn_waves_per_item(x.items, x.n_keys, x.d, x.paged, x.groups, x.gc, x.T) != x.want) { std::printf("%lld %d\n", (long long)x.items, x.n_keys); return 1; }
    std::printf("ok\n");
    """)
    assert out.strip() == "ok"
    assert "attn_waves_per_item(waves, p.kb * p.bk, p.d, p.page_table != nullptr, groups, gc, p.max_kv_len)" in (CSRC / "attn_mfma.hip").read_text()


def test_waves_of_the_decode_mask(tmp_path):
    # the lines between sixteen, four and one wave per problem
    out = run(tmp_path, r"""
    const Slice N = Slice::narrow, W = Slice::wide, P = Slice::paged;
    struct { int64_t problems; int kb, d; Slice slice; int want; } c[] = {
        {1, 256, 128, N, 16}, {256, 256, 128, W, 16}, {256, 256, 64, P, 16}, {257, 256, 128, N, 4}, {257, 256, 128, W, 4}, {32, 16, 128, N, 4}, {32, 17, 128, N, 16},
        {32, 512, 128, P, 16}, {32, 513, 128, P, 4}, {8192, 16, 64, P, 4}, {8193, 256, 128, N, 4}, {8193, 256, 128, P, 1}, {8193, 256, 64, N, 1}, {8193, 257, 128, N, 1},
        {16384, 64, 128, N, 4}, {16384, 63, 128, N, 1}, {16384, 16, 64, P, 1}, {16385, 256, 128, N, 1}, {16385, 256, 128, W, 4}};
    for (auto &x : c) {   // bk = 2: stages of four and of eight rows
        const int rpw = 512 / x.d, got = decode_mask_waves(x.problems, x.kb, x.d, rpw * 2, rpw * 4, x.slice);
        if (got != x.want) { std::printf("%lld problems, k/bk %d, d %d: %d\n", (long long)x.problems, x.kb, x.d, got); return 1; }
    }
    std::printf("ok\n");
    """)
    assert out.strip() == "ok"
    assert "decode_mask_waves(problems, p.kb, D, STEP, 512 / D * (8 / BK), slice)" in (CSRC / "mask_decode_impl.h").read_text()


def test_the_prefill_attention_uses_the_rule_it_is_tested_with():
    src = (CSRC / "attn_mfma.hip").read_text()
    assert "rows_by_lane_offset(p.max_kv_len, p.ks_r * 2, p.d)" in src
    assert src.count("kRowBias - back") == 1 and src.count(": Kseq) - kRowBias") == 1 and "3072" not in src


def occupancy_failures(source: str) -> list:
    """The kernels of a source that the compiler could not give the waves per SIMD they ask for (it then gives up on a target)."""
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c", str(CSRC / source),
                        "-o", "/dev/null"], capture_output=True, text=True)
    assert r.returncode == 0 and "Occupancy [waves/SIMD]" in r.stderr, r.stderr
    return [line for line in r.stderr.splitlines() if "failed to meet occupancy target" in line]


def test_attention_kernels_get_the_waves_they_ask_for():
    assert occupancy_failures("attn_mfma.hip") == []
