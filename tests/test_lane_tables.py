"""The LJ lane tables: the tuner's rule, and that the committed tables follow it on the times
written beside them (a count that a full batch bears; relaxations by the fastest alone)."""
import re

import pytest

from paper_2510_16721_amd import tune_lanes as T


def test_allowed_counts():
    t = {1: 30.0, 2: 20.0, 4: 14.0, 8: 10.0}
    assert T.allowed(t, None) == t
    # eight lanes cost the batch too much; four, the fastest left, are not within MARGIN of them
    assert T.allowed(t, {1: 100.0, 2: 101.0, 4: 110.0, 8: 118.0}) == {4: 14.0}
    assert T.allowed(t, {1: 100.0, 2: 101.0, 4: 126.0, 8: 118.0}) == {2: 20.0}
    assert T.allowed(t, {1: 100.0, 2: 101.0, 4: 110.0, 8: 116.0}) == {8: 10.0}
    # within MARGIN of the fastest of all
    assert T.allowed({1: 11.0, 2: 10.5, 4: 10.0, 8: 12.0}, dict.fromkeys((1, 2, 4, 8), 1.0)) == {1: 11.0, 2: 10.5, 4: 10.0}
    # a larger size never takes more lanes than a smaller one
    assert T.table_rows([(10, {1: 2.0, 4: 1.0}), (40, {1: 1.0, 4: 1.0}), (160, {1: 2.0, 4: 1.0})]) == [(20, 4), (None, 1)]


@pytest.mark.parametrize("bits", [32, 64])
def test_committed_tables_follow_the_rule(bits):
    src = open(T.TABLE).read()

    def rows(name):
        body = re.search(name + r"\[\] = \{(.*?)\};", src, re.S).group(1)
        return [(int(a), int(k)) for a, k in re.findall(r"\{(\d+)(?:LL)?, (\d+)\}", body)]

    def section(title):
        body = src[src.index(title):].split("\n")[1:]
        out, batch = [], {}
        for line in body:
            times = {int(k): float(v) for k, v in re.findall(r"(\d+): +([\d.]+)", line)}
            if not times:
                break
            if "batch" in line:
                batch[out[-1][0]] = times
            else:
                out.append((int(line.split()[1]), times))
        return out, batch

    def lanes(table, work):
        return next(k for limit, k in table if work <= limit)

    bands, batch = section(f"// FP{bits} bands")
    table = rows("kLjLanesFp64" if bits == 64 else "kLjLanesTable")
    assert len(bands) > 10 and len(batch) > 10
    for work, t in bands:
        k = lanes(table, work)
        assert k in T.BAND_LANES
        if work in batch:
            b = batch[work]
            assert b[k] <= min(b.values()) * (1.0 + T.BATCH_MARGIN.get(k, 1.0))
    relax, _ = section(f"// FP{bits} relaxations")
    rtable = rows("kLjLanesRelaxFp64" if bits == 64 else "kLjLanesRelax")
    assert len(relax) > 10
    for work, t in relax:
        assert t[lanes(rtable, work)] <= 1.15 * min(t.values())
    for tab in (table, rtable):
        assert [w for w, _ in tab] == sorted(w for w, _ in tab) and tab[-1][0] >= 2**31 - 1
        assert [k for _, k in tab] == sorted((k for _, k in tab), reverse=True)
