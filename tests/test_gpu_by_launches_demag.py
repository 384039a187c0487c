"""The local magnetostatic solve by launches (by_launches.py)."""
from by_launches import by_launches  # noqa: F401
from test_gpu_demag_local import (case, pytestmark, test_mixed_form_matches_fp64,  # noqa: F401
                                  test_operator_and_solve_match_oracle, test_steps_match_oracle)
