"""The shipped cost table is what calibrate.py writes: its measured entries, and in place of some
of them the ones it keeps."""
import re

from paper_1711_07295_amd import calibrate


def _shipped():
    text = open(calibrate.TABLE).read()
    values = {m[0]: [float(v) for v in m[1].strip("{}").split(",")]
              for m in re.findall(r"constexpr \w+ (k\w+)(?:\[6\])? = (\{[^}]*\}|[^;]*);", text)}
    return text, values


def test_calibrate_writes_the_shipped_table(tmp_path):
    text, v = _shipped()
    device, date = re.search(r"// Device: (.*); (\S+)\.\n", text).groups()
    res = {"device": device, "entry_ns": v["kSlowEntryNs"][0], "survivor_ns": v["kSurvivorNs"][0]}
    for key, name in (("filter_ns", "kFilterNsPerPair"), ("launch_ns", "kClassLaunchNs"),
                      ("wave_ns", "kSurvivorWaveNs"), ("tile_cols", "kClassTileCols")):
        res[key] = dict(zip(calibrate.WIDTHS, v[name]))
    res["tile_cols"] = {b: int(t) for b, t in res["tile_cols"].items()}
    # a measurement's values where the table keeps others
    measured = re.findall(r"// b = (\d+): kept.*\n// (\S+) ns per pair, (\d+) pairs a step and "
                          r"(\S+) ns a launch", text)
    assert [int(m[0]) for m in measured] == list(calibrate.KEPT)
    for b, ns, pairs, launch in measured:
        res["filter_ns"][int(b)], res["launch_ns"][int(b)] = float(ns), float(launch)
        assert int(pairs) == calibrate.PAIRS_PER_STEP[int(b)]
    out = calibrate.write_table(res, tmp_path / "table.h", date)
    assert open(out).read() == text
    for b, kept in calibrate.KEPT.items():
        k = calibrate.WIDTHS.index(b)
        assert (v["kFilterNsPerPair"][k], v["kPairsPerStep"][k], v["kClassLaunchNs"][k]) == \
            (kept["filter_ns"], kept["pairs"], kept["launch_ns"])
