"""bench.py's launch counts: each launch once, however the library books one of
seven terms."""
import bench
import paper_2307_12276_amd as A


class Booked:
    """Counters of two sweeps of three launches: six terms (100 us), seven and
    seven (210 us each), booked by the library as groups of three and one."""

    def profile_read_kind(self, kind):
        return {A.LAUNCH_FIRST: (0.2, 2, 12.0, 12), A.LAUNCH_THREE: (0.72, 8, 24.0, 24),
                A.LAUNCH_ONE: (0.12, 4, 4.0, 4)}.get(kind, (0.0, 0, 0.0, 0))

    def profile_read(self):
        return 1.04, 6, 40.0


def test_each_launch_counts_once():
    ms, launches, nbytes, terms, kinds = bench.read_launches(Booked())
    assert (ms, launches, nbytes, terms) == (1.04, 6, 40.0, 40)
    assert kinds["first"]["launches"] == 2 and kinds["first"]["terms"] == 12
    assert kinds["later"]["launches"] == 4 and kinds["later"]["terms"] == 28
    assert abs(kinds["first"]["avg_us"] - 100.0) < 1e-9 and abs(kinds["later"]["avg_us"] - 210.0) < 1e-9
