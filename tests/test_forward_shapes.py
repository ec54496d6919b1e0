"""The one-launch forward requests the first layer's weights in whole 128-byte pieces; which networks it may serve is a rule
on their shape (csrc/fwd_shape.h).  Here every request of a preference is walked on the host, lane by lane, for every width,
output width and element type: what the rule accepts must end inside that preference's matrices.  And which tiles a call takes
is a rule too: what it plans must be compiled and cover every row."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_09237_amd", "csrc")

# The walk repeats the kernel's request pattern: wave w, request b of lane l = chunk (l & 7) ^ ((l >> 4) & 3) (odd b: the
# other half of the line) of feature 64 w + 8 b + (l >> 3), features beyond W reading the last row.  Chunks behind the end of
# a hidden row are not requested.  A bf16 first layer of at most 32 columns is read as 32 consecutive elements a row instead,
# where another kernel did so before.
PROGRAM = r"""
#include <cstdio>
#include "fwd_shape.h"
static long last_of_matrix(int es, int W, int ld, int steps, long off, bool hidden) {
    const int VE = 16 / es, KS = 8 * VE;
    long last = 0;
    for (int w = 0; w < fwd_waves(W); ++w)
        for (int s = 0; s < steps; ++s)
            for (int b = 0; b < 8; ++b)
                for (int l = 0; l < 64; ++l) {
                    const int f = 64 * w + 8 * b + (l >> 3);
                    const int chunk = ((l & 7) ^ ((l >> 4) & 3)) ^ (4 * (b & 1));
                    if (hidden && s * KS + chunk * VE >= ld) continue;
                    const long e = off + (long)(f < W ? f : W - 1) * ld + s * KS + chunk * VE + VE - 1;
                    if (e > last) last = e;
                }
    return last;
}
int main() {
    const int Os[] = {1, 2, 3, 8, 11, 19, 31, 32, 33, 45, 63, 64, 65, 100, 127, 513, 1024};
    long n = 0, wrong = 0, refused = 0, refused_wide = 0;
    for (int es = 2; es <= 4; es += 2)
        for (int W = 16; W <= 2048; W += 16)
            for (int L = 1; L <= 8; L += L < 3 ? 1 : 5)
                for (int O : Os) {
                    const int KS = 128 / es;
                    long last = 0;
                    if (W <= kFwdMaxWidth) {
                        last = last_of_matrix(es, W, O, (O + KS - 1) / KS, 0, false);
                        if (es == 2 && O <= 32 && (long)(W - 1) * O + 31 > last) last = (long)(W - 1) * O + 31;
                        for (int l = 1; l < L; ++l) {
                            const long e = last_of_matrix(es, W, W, 64 * fwd_waves(W) / KS, (long)W * O + (long)(l - 1) * W * W, true);
                            if (e > last) last = e;
                        }
                    }
                    for (int out = 1; out <= 16; ++out) {
                        const long mat_len = (long)W * O + (long)(L - 1) * W * W + (long)out * W;
                        const bool ok = fwd_reads_inside(es, W, L, out);
                        ++n;
                        if (W > kFwdMaxWidth) refused_wide += ok ? 0 : 1, wrong += ok ? 1 : 0;
                        else if (!ok) ++refused;
                        else if (last >= mat_len && wrong++ < 10)
                            printf("reads element %ld of %ld: %d bytes, W %d, O %d, %d hidden, output %d\n", last, mat_len, es, W, O, L, out);
                    }
                }
    printf("shapes %ld wrong %ld refused %ld\n", n, wrong, refused);
    return wrong ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_accepted_networks_are_read_inside_their_matrices(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    # refused: one hidden layer of width 16, 32 or 48 and 3, 1 or 1 outputs at most (bf16), of width 16 and 1 output (fp32)
    refused = int(r.stdout.split("refused")[1])
    assert refused == (3 + 1 + 1 + 1) * 17, r.stdout


# The same for fp32 networks on split operands (csrc/fused_fwd_split.h): request b of lane l = sixteen bytes of row 8 b + (l >> 3)
# of a wave's 32 features, whole super-steps of 32 elements to the end of the waves' features.
SPLIT_PROGRAM = r"""
#include <cstdio>
#include "fwd_shape.h"
int main() {
    const int Os[] = {1, 2, 8, 11, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 300, 513, 1024};
    long n = 0, wrong = 0;
    for (int W = 16; W <= kSplitMaxWidth; W += 16)
        for (int L = 1; L <= 8; ++L)
            for (int O : Os)
                for (int out = 1; out <= 16; ++out) {
                    if (!fwd_reads_inside(4, W, L, out)) continue;
                    const int nw = split_waves(W);
                    const long mat_len = (long)W * O + (long)(L - 1) * W * W + (long)out * W;
                    long last = (long)(W - 1) * O + (O + 31) / 32 * 32 - 1;                     // first layer
                    if (L > 1) last = (long)W * O + (long)(L - 2) * W * W + (long)(W - 1) * W + 32 * nw - 1;
                    if (L > 1 && (long)(W - 1) * O + (O + 31) / 32 * 32 - 1 > last) last = (long)(W - 1) * O + (O + 31) / 32 * 32 - 1;
                    // the tile: chunks of sixteen bytes inside a row's pitch, whatever they are XORed with (3, 7 or 15)
                    const int ks[] = {O, 32 * nw};
                    for (int k : ks) {
                        const int pitch = split_pitch(k), x = pitch == 64 ? 3 : (pitch & 128) ? 7 : 15;
                        if (((((k + 31) / 32 * 4 - 1) | x) + 1) * 16 > pitch) ++wrong;
                    }
                    ++n;
                    if (32 * nw < W || last >= mat_len) ++wrong;
                }
    printf("shapes %ld wrong %ld\n", n, wrong);
    return wrong ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_split_networks_are_read_inside_their_matrices(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(SPLIT_PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


# The rule on tiles: what it asks for is compiled, and each compiled variant is asked for by something; a workgroup's LDS holds the
# tile; and the workgroups that the launch counts cover every row, once, whatever their number.
PLAN_PROGRAM = r"""
#include <cstdio>
#include "fwd_shape.h"
int main() {
    const int Os[] = {1, 8, 27, 32, 33, 64, 65, 100, 128, 129, 300, 513, 700, 1024}, Ps[] = {2, 3, 10, 16, 24, 64, 200, 4096, 65535};
    const int cuss[] = {64, 256, 304};
    const long Ms[] = {1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 129, 255, 257, 512, 700, 1025, 2048, 4095, 4096, 4100, 8192, 100001};
    long n = 0, wrong = 0, rt_seen[5][9][5] = {}, split_seen[9][4] = {};
    for (int es = 2; es <= 4; es += 2)
        for (int W = 16; W <= 560; W += 16)
            for (int L = 1; L <= 4; ++L)
                for (int O : Os) for (int P : Ps) for (long M : Ms) for (int cus : cuss) for (int tall = 0; tall < 2; ++tall) {
                    const FwdPlan f = fwd_plan(es, W, L, O, 4, P, M, cus, es == 2 && tall);
                    ++n;
                    if (f.rt == 0) { wrong += f.split != 0; continue; }
                    const int nw = fwd_waves(W), snw = split_waves(W);
                    bool ok;
                    if (f.split) {
                        // (up to 64 features: not where the first layer is so much longer than the hidden ones)
                        ok = es == 4 && W <= kSplitMaxWidth && f.split <= split_most(snw) && f.rt == 2 * f.split &&
                             split_lds_bytes(O, W, L, f.split) <= 160 * 1024 && (W > 64 || O <= 64 * L);
                        if (ok) ++split_seen[snw][f.split];
                    } else {
                        ok = W <= kFwdMaxWidth && f.rt == fwd_compiled(es, nw, f.rt) && fwd_lds_bytes(es, O, W, L, f.rt) <= 160 * 1024;
                        if (ok) ++rt_seen[es][nw][f.rt];
                    }
                    const long th = 16 * (f.split ? 2 * f.split : fwd_compiled(es, nw, f.rt)), planned = (M + 16 * f.rt - 1) / (16 * f.rt);
                    if (!ok || planned * th < M || (planned - 1) * th >= M)
                        if (wrong++ < 10)
                            printf("W %d O %d L %d, %d x %ld, %d bytes, %d CUs: row tiles %d, split %d: %ld tiles of %ld rows\n", W, O, L, P,
                                   M, es, cus, f.rt, f.split, planned, th);
                }
    for (int es = 2; es <= 4; es += 2)
        for (int W = 16; W <= kFwdMaxWidth; W += 16)
            for (int rt = fwd_low(es); rt <= 4; rt *= 2)
                if (rt == fwd_compiled(es, fwd_waves(W), rt) && !rt_seen[es][fwd_waves(W)][rt] && ++wrong)
                    printf("nothing takes %d row tiles of %d waves, %d bytes\n", rt, fwd_waves(W), es);
    for (int W = 16; W <= kSplitMaxWidth; W += 16)
        for (int rb = 1; rb <= split_most(split_waves(W)); ++rb)
            if (!split_seen[split_waves(W)][rb] && ++wrong) printf("nothing takes %d blocks of %d split waves\n", rb, split_waves(W));
    printf("shapes %ld wrong %ld\n", n, wrong);
    return wrong ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_planned_tiles_are_compiled_and_cover_all_rows(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PLAN_PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
