"""The tracked profiler summaries that bench.py and the design notes quote must belong to the kernels in the tree:
the HBM-traffic summary names the mover source it was taken with, and bench.py reads its figures from it."""
import hashlib
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TRAFFIC = os.path.join(ROOT, "profiles", "bench_dsv3_hbm_traffic_pmc.txt")
MOVERS = os.path.join(ROOT, "paper_2512_22036_amd", "csrc", "movers.h")


def test_traffic_summary_was_taken_with_the_movers_in_the_tree():
    text = open(TRAFFIC).read()
    m = re.search(r"^movers\.h sha256: ([0-9a-f]{64})$", text, flags=re.M)
    assert m, "the summary must name the mover source it was measured with"
    assert m.group(1) == hashlib.sha256(open(MOVERS, "rb").read()).hexdigest(), \
        "csrc/movers.h changed since profiles/bench_dsv3_hbm_traffic_pmc.txt was taken: profile again"


def test_bench_reads_its_traffic_figures_from_the_summary():
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    got = bench.measured_traffic("dsv3")
    algorithmic = (8192 + 65536) * 14336
    assert set(got) == {"dispatch", "combine"}
    # combine: every row once - no wasted re-reads, and nothing the counters could have missed
    assert algorithmic <= got["combine"] <= 1.01 * algorithmic, got
    # dispatch: a tile's source rows are fetched once and stay in the XCD's L2 (write-through non-temporal stores do
    # not displace them; with plain non-temporal stores the figure was 1.047)
    assert algorithmic <= got["dispatch"] <= 1.01 * algorithmic, got
    assert bench.measured_traffic("qwen3") == {}          # no summary for other workloads: reported as null
    assert "MEASURED_TRAFFIC_BYTES" not in open(os.path.join(ROOT, "bench.py")).read()


def table_rows(heading):
    """The rows of the first table behind a heading of the design notes, as lists of cells by the first cell's first word."""
    text = open(os.path.join(ROOT, "DESIGN.md")).read()
    lines = iter(text[text.index("\n" + heading) + 1:].split("\n")[1:])
    line = next(lines)
    while not line.startswith("|"):
        line = next(lines)
    width, rows = line.count("|"), {}
    next(lines)
    for line in lines:
        if not line.startswith("|"):
            break
        assert line.count("|") == width, line
        cells = [c.strip() for c in line.strip("|").split("|")]
        rows[cells[0].split()[0]] = cells[1:]
    return rows


def test_input_table_describes_the_configurations():
    import workloads
    rows = table_rows("## 4. Synthetic inputs")
    assert set(rows) == set(workloads.CONFIGS)
    for name, (n, hidden, ekd, *_) in rows.items():
        cfg = workloads.CONFIGS[name]
        assert int(n) == cfg.N and int(hidden.split()[0]) == cfg.H, name
        assert [int(v) for v in ekd.split("/")] == [cfg.E, cfg.k, cfg.D], name


def test_configuration_table_holds_the_measured_summary():
    import workloads
    summary = open(os.path.join(ROOT, "profiles", "bench_all_configs.txt")).read()
    rows = table_rows("### 6.6 All five configurations")
    assert set(rows) == set(workloads.CONFIGS)

    def span(cell):   # "1.5–2.5" or "1.5", in the notes or the summary; a span of equal ends is written either way
        ends = [float(v) for v in re.split("[-–]", cell)]
        return ends[0], ends[-1]

    for name, (step, rate, plan, dispatch, combine, share) in rows.items():
        m = re.search(rf"^{name}  +(\S+)  +(\S+)  +(\S+)  +(\S+)  +(\S+)$", summary, flags=re.M)
        assert m, f"no row of {name} in the summary"
        assert [span(c) for c in (step, dispatch, combine, plan)] == [span(m.group(i)) for i in (1, 2, 3, 5)], name
        per_us = [workloads.CONFIGS[name].N / v for v in reversed(span(m.group(1)))]
        figure = rate.split()[0].split("–")
        for cell, want in zip((figure[0], figure[-1]), per_us):
            # both are rounded to their last digit: N / step of the summary, whose steps are given to 0.1 us
            digit = 10.0 ** -len(cell.partition(".")[2])
            assert abs(float(cell) - want) <= 0.5 * digit + want * want / workloads.CONFIGS[name].N * 0.05 + 1e-9, (name, rate)
        if not share.startswith("latency"):
            assert span(share.split()[0]) == span(m.group(4)), name
