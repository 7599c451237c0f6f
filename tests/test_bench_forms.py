"""bench.py's byte counts follow the form of the step that was timed (no GPU): the
form is told by the launches, and each count is the list of the fields that the
launch reads or writes."""
import bench


def test_form_is_told_by_the_launches():
    flux = [("k_prep", 10, 1.0), ("k_lb", 10, 9.0), ("k_uend", 10, 8.0), ("k_stage", 10, 2.0)]
    phases = flux[:3] + [("k_stage", 20, 5.0)]
    assert bench.step_form(flux, 10) == "flux"
    assert bench.step_form(phases, 10) == "phases"
    assert bench.step_form([("k_half1", 10, 1.0), ("k_half2", 10, 1.0)], 10) == "halves"
    assert bench.step_form([], 10) == "phases"


def test_bytes_of_the_flux_form():
    w, fused = bench.WORKLOADS[bench.DEFAULT_WORKLOAD], {"overlap": 3}

    def count(name):
        return bench.kernel_alg_bytes_per_site(name, w, schedule=fused, form="flux")

    # populations, psi, mu, flux; stage velocity, stage output, rate
    assert count("k_uend") == (19 + 1 + 1 + 3 + 3 + 1 + 1) * 8 == 232
    # stage output, rate, stage velocity; psi
    assert count("k_stage") == (1 + 1 + 3 + 1) * 8 == 48
    assert count("k_lb") == (19 + 1 + 1 + 19 + 3) * 8 == 344
    assert count("k_prep") == 16


def test_bytes_of_the_halves():
    w = dict(bench.WORKLOADS[bench.DEFAULT_WORKLOAD], lattice=9, precision=1)
    # populations, psi; populations, stage output, rate
    assert bench.kernel_alg_bytes_per_site("k_half1", w, form="halves") == (9 + 1 + 9 + 2) * 4
    # populations, psi, stage output, rate; psi
    assert bench.kernel_alg_bytes_per_site("k_half2", w, form="halves") == (9 + 3 + 1) * 4
