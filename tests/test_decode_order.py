"""The order in which the paged decode kernels deal out their workgroups (csrc/decode_order.h), on the host: every (layer, request,
KV head, split) is done exactly once and nothing outside the grid is named, also where a length on the device has outgrown the
max_blocks that the launch and the room for the splits' states are sized for."""
import subprocess

import pytest

from paper_2601_03067_amd import build as kbuild

CHECK = r"""
#include "decode_order.h"
#include <cstdio>
using namespace kvfuse;

int main()
{
    uint32_t st = 99u;
    auto rnd = [&](uint32_t m) { st = st * 1664525u + 1013904223u; return (st >> 8) % m; };
    long outside = 0, left_out = 0;
    for (int trial = 0; trial < 3000; ++trial) {
        const int layers = 1 + rnd(9), heads = 1 + rnd(11), B = 1 + rnd(20), nsplit = 1 + rnd(trial % 3 == 0 ? 64 : 6);
        const int tokens = 16 * (1 + (int)rnd(30));                        // of a split
        DecodeOrder o;
        o.by_xcd = trial % 8 != 0;
        o.nsplit = nsplit;
        o.groups = GroupsByXcd((int64_t)layers * heads, (int64_t)B * nsplit);
        o.requests = Divisor(B);
        o.heads = Divisor(heads);
        o.split_tokens = Divisor(tokens);
        std::vector<int32_t> ctx(B);
        for (int &c : ctx) {
            const int kind = rnd(6);
            c = kind == 0 ? 0 : kind == 1 ? nsplit * tokens : kind == 2 && LONGER ? nsplit * tokens + 1 + (int)rnd(4 * nsplit * tokens)
                : kind == 3 && LONGER ? INT32_MAX - (int)rnd(3) : (int)rnd(nsplit * tokens + 1);
        }
        std::vector<int> seen((size_t)layers * heads * B * nsplit, 0);
        for (int z = 0; z < layers; ++z)
            for (int y = 0; y < B * heads; ++y)
                for (int x = 0; x < nsplit; ++x) {
                    const DecodeOrder::Place p = o.place(x, y, z, ctx.data());
                    if (p.split < 0 || p.split >= nsplit || p.b < 0 || p.b >= B || p.kvh < 0 || p.kvh >= heads || p.li < 0 || p.li >= layers)
                        ++outside;
                    else
                        ++seen[(((size_t)p.li * B + p.b) * heads + p.kvh) * nsplit + p.split];
                }
        for (int s : seen)
            left_out += s != 1;
    }
    std::printf("outside %ld left out %ld\n", outside, left_out);
    return 0;
}
"""


@pytest.mark.parametrize("longer", [0, 1])
def test_every_place_is_taken_once(tmp_path, longer):
    try:
        hipcc = kbuild._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc here")
    src, exe = tmp_path / "order.hip", tmp_path / "order"
    src.write_text(CHECK)
    subprocess.check_call([hipcc, *kbuild.FLAGS, f"-DLONGER={longer}", "--offload-host-only", "-I", kbuild.CSRC, str(src), "-o", str(exe)])
    assert subprocess.check_output([str(exe)], text=True) == "outside 0 left out 0\n"
