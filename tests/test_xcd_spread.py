"""The order in which Deflate chunks are dealt to workgroups takes every chunk
once, and gives each of eight XCDs its share of the chunks of any small period."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _spread():
    """The rule of the source, read as Python."""
    with open(os.path.join(ROOT, "paper_2307_03760_amd", "csrc", "codag.hip")) as f:
        text = f.read()
    body = re.search(r"uint32_t spread_over_xcds\(uint32_t b, uint32_t n\) \{(.*?)\n\}", text, re.S).group(1)
    g, cond, own, other = re.search(r"g = (.*?);\s*return (.*?) \? (.*?) : (.*?);", body, re.S).groups()
    py = lambda e: e.replace("/", "//")
    return eval(f"lambda b, n: (lambda g: ({py(own)}) if ({py(cond)}) else ({py(other)}))({py(g)})")


def test_every_chunk_once():
    f = _spread()
    for n in list(range(1, 70)) + [513, 4095, 4096, 4103]:
        assert sorted(f(b, n) for b in range(n)) == list(range(n))


def test_periods():
    f, n = _spread(), 8192
    for period in (2, 4, 8, 16, 80):
        for phase in range(period):
            count = [0] * 8
            for b in range(n):
                if f(b, n) % period == phase:
                    count[b % 8] += 1
            assert max(count) <= 1.3 * n / period / 8, (period, phase, count)
