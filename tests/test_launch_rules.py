"""The rules by which the launchers choose a kernel's shape (csrc/launch_rules.h), compiled as a host
program and checked over their ranges."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_05589_amd", "csrc")
WAVES = 2048


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(lines) -> one list of integers per line "name arguments..."."""
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(r'''
#include <cstdio>
#include <cstring>
#include "launch_rules.h"
using namespace copris;
int main() {
  char name[32];
  while (std::scanf("%31s", name) == 1) {
    long long a[8] = {};
    if (!std::strcmp(name, "share")) {
      std::scanf("%lld %lld %lld %lld", a, a + 1, a + 2, a + 3);
      const int total = static_cast<int>(a[0]), longest = static_cast<int>(a[1]), group = static_cast<int>(a[3]);
      std::printf("%d %d\n", attn_share(total, longest, group), attn_most_waves(a[2], group));
    }
  }
}
''')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-result", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def ask(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        return [[int(x) for x in l.split()] for l in out.splitlines()]
    return ask


@pytest.mark.parametrize("group", [1, 2, 16])
def test_attention_shares(rules, group):
    totals = sorted({0, 1, 2, 256, 257, 1536, 1537, 2047, 2048, 2049, 4096, 4097, 6144, 6145, 8192, 8193, 100000, 2**31 - 1}
                    | {int(1.37 ** k) for k in range(1, 60)})
    cases = [(t, l) for t in totals for l in (0, 1, 4, 64, 65, 128, 129, 2048, 10**6) if l <= t]
    for (t, l), (s, _) in zip(cases, rules([f"share {t} {l} 1 {group}" for t, l in cases])):
        equal = -(-t // WAVES)
        assert 1 <= s and s * WAVES >= t, (t, l, s)                     # the wavefronts cover the slots
        assert s == equal if equal >= 4 else equal <= s <= 4, (t, l, s)
        if t <= 256 and l <= 64:
            assert s == 1, (t, l, s)                                    # little to merge: no serial chain
        assert s >= 4 or l <= 64 * s, (t, l, s)                         # partials of a context


@pytest.mark.parametrize("group", [1, 2, 16])
def test_attention_launches_enough_wavefronts(rules, group):
    # for every pool that a table of some capacity admits
    totals = list(range(1, 9000)) + [10**5, 10**7, 2**31 - 1]
    caps = [1, 2, 255, 256, 257, 600, 767, 768, 769, 1535, 1536, 1537, 2047, 2048, 2049, 3071, 3072, 3073, 4096, 4097, 6144, 6145, 8192, 8193, 10**5, 2**31 - 1]
    most = {c: m for c, (_, m) in zip(caps, rules([f"share 1 1 {c} {group}" for c in caps]))}
    need = [-(-t // s) for t, (s, _) in zip(totals, rules([f"share {t} 1 1 {group}" for t in totals]))]
    for c in caps:
        worst = max(n for t, n in zip(totals, need) if t <= c)
        assert worst <= most[c] <= WAVES, (c, worst, most[c])
