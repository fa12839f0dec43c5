"""Host-side checks of bench.py: the schedule each workload gets by default,
explicit flags taking precedence, and step boundaries over several streams (no
GPU, no torch)."""

import os
import sys

import pytest

import bench


def parsed(*argv):
    old = sys.argv
    sys.argv = ["bench.py", *argv]
    try:
        return bench.parse()
    finally:
        sys.argv = old


@pytest.mark.parametrize("argv,streams,assign,queues", [
    ((), 6, "balance", 8),                         # Llama-600M set, input side
    (("--sides", "both"), 6, "balance", 8),
    (("--ef",), 8, "balance", 8),                  # error feedback: eight streams
    (("--config", "4"), 4, "round-robin", 4),      # Llama-300M set keeps the four-stream deal
    (("--config", "2"), 4, "round-robin", 4),
    (("--hw-queues", "4", "--streams", "4", "--assign", "round-robin"), 4, "round-robin", 4),
    (("--streams", "3"), 3, "balance", 8),
    (("--config", "4", "--hw-queues", "0"), 4, "round-robin", 0),
])
def test_schedule_defaults(argv, streams, assign, queues):
    a = parsed(*argv)
    assert (a.streams, a.assign, a.hw_queues) == (streams, assign, queues)


def test_more_than_one_gpu_is_refused(capsys, monkeypatch):
    monkeypatch.delenv("GPU_MAX_HW_QUEUES", raising=False)
    old = sys.argv
    sys.argv = ["bench.py", "--gpus", "2"]
    try:
        with pytest.raises(SystemExit) as e:
            bench.main()
    finally:
        sys.argv = old
    assert e.value.code == 2
    assert "one GPU" in capsys.readouterr().err
    assert "GPU_MAX_HW_QUEUES" not in os.environ   # refused before touching it


class Stream:
    """A queue in virtual time: work runs after what it waits for."""

    def __init__(self):
        self.now = 0.0

    def run(self, duration):
        self.now += duration

    def wait_event(self, ev):
        self.now = max(self.now, ev.at)


class Event:
    def record(self, stream):
        self.at = stream.now


@pytest.mark.parametrize("durations", [(1.0, 3.0), (3.0, 1.0, 2.0), (2.0,)])
def test_steps_begin_on_every_stream(durations):
    """Each step takes as long as its slowest stream, whichever that is in that
    step, and its interval on the main stream says so."""
    streams = [Stream() for _ in durations]
    main = streams[0]
    for step in range(4):
        bench.join(main, streams, Event)
        begin = main.now
        bench.start_together(main, streams, Event)
        assert all(st.now == begin for st in streams)
        for i, st in enumerate(streams):
            st.run(durations[(i + step) % len(durations)])
        bench.join(main, streams, Event)
        assert main.now - begin == max(durations)


@pytest.mark.parametrize("used", [[1, 2], [0], [2, 2, 0], []])
def test_steps_wait_for_streams_with_work(used):
    """Streams that get no work are neither waited for nor held: a step ends
    with the streams that have some."""
    streams = [Stream() for _ in range(4)]
    main = streams[0]
    busy = bench.with_work(streams, used)
    assert busy == [streams[i] for i in sorted(set(used))]
    for step in range(3):
        bench.join(main, busy, Event)
        begin = main.now
        bench.start_together(main, busy, Event)
        for i in set(used):
            streams[i].run(1.0 + i)
        bench.join(main, busy, Event)
        assert main.now - begin == max([1.0 + i for i in used], default=0.0)
    assert all(streams[i].now == 0.0 for i in range(1, 4) if i not in used)


def test_traffic_goes_with_its_sources(tmp_path, monkeypatch):
    """A counted HBM figure is reported while every source of its family is the
    one it was counted on, and no longer."""
    for name in ("a.hip", "b.hip"):
        (tmp_path / name).write_text(name)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "FAMILY_SOURCE", {"update_amax": ("a.hip", "b.hip")})
    monkeypatch.setattr(bench, "TRAFFIC_GLOB", str(tmp_path / "*.md"))
    line = "traffic: family=update_amax workload=w bytes_per_launch=12 sha256=%s\n"
    (tmp_path / "t.md").write_text(line % bench.source_sha256(("a.hip", "b.hip")))
    assert bench.measured_traffic("update_amax", "w") == 12
    assert bench.measured_traffic("update_amax", "v") is None
    (tmp_path / "a.hip").write_text("c")
    assert bench.measured_traffic("update_amax", "w") is None


def test_families_name_files_that_are_there():
    for rel in bench.FAMILY_SOURCE.values():
        assert len(bench.source_sha256(rel)) == 64
    assert "paper_2607_07494_amd/csrc/k_strip.hip" in bench.FAMILY_SOURCE["update_quant"]
