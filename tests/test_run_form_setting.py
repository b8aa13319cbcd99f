"""cola_plan_set_run_form / cola_plan_get_run_form (host-only)."""
import pytest

import paper_1301_0322_amd as cola


def test_run_form_setting():
    with cola.Plan(cola.Config(np=16, nm=32)) as p:
        default = p.get_run_form()
        assert default in (0, 1)
        for form in (0, 1):
            p.set_run_form(form)
            assert p.get_run_form() == form
        for bad in (-2, 2):
            with pytest.raises(cola.ColaError):
                p.set_run_form(bad)
        p.set_run_form(-1)
        assert p.get_run_form() == default
    lib = cola.lib()
    assert lib.cola_plan_set_run_form(None, 0) == -1 and lib.cola_plan_get_run_form(None, None) == -1
