"""bench.py reports the measured HBM traffic of its dominant kernels only while
their sources are those that were measured: a change to them has to come with
a new measurement (or the same one confirmed), or the figure is silently null
(CPU only)."""
import bench


def test_traffic_records_are_of_the_present_sources():
    for workload, kernel in bench.MEASURED_TRAFFIC:
        assert bench.measured_traffic(workload, kernel) is not None, kernel
