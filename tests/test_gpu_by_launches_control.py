"""Control paths of CG, the mixed form and deterministic mode, solving by launches (by_launches.py)."""
from by_launches import by_launches  # noqa: F401
from test_gpu_cg_control import (case, pytestmark, test_budget_exhaustion_returns_the_oracle_iterate,  # noqa: F401
                                 test_elastic_iterations_and_solution_match_oracle,
                                 test_zero_rhs_and_converged_start)
from test_gpu_deterministic import (test_deterministic_steps_match_oracle,  # noqa: F401
                                    test_repeat_and_split_runs_are_bitwise_identical)
from test_gpu_mixed import test_mixed_solves_reach_true_residual  # noqa: F401
