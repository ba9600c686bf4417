// Which kernel the host side of libwd chooses for a configuration, for tests that run without a GPU.
#include "wd_api.hip"

#include <cstdio>

// out: one line "kernel teams threads strips wide apart reach lds"; `recording`: a call of wd_rollout.  Returns a status of wd.h.
extern "C" int wd_test_route(const wd_config* c, int recording, char* out, int len) {
  const int rc = check_config(c);
  if (rc != WD_OK) return rc;
  wd_buffers none = {};
  wd::Params p;
  const int filled = fill_params(*c, none, &p, true);
  if (filled != WD_OK) return filled;
  const bool multi = recording && wd::rollout_available(p);
  const char* kernel = p.crew_threads                     ? "crew_env_kernel"
                       : p.wave_envs == wd::kSmallEnvs    ? "small_env_kernel"
                       : p.wave_envs                      ? ((recording ? p.quad_roll : p.quad_single) ? "quad_env_kernel" : "wave_env_kernel")
                       : p.big                            ? (p.big_spread ? "spread_obs_kernel" : "big_obs_kernel")
                       : multi                            ? "rollout_kernel"
                                                          : "env_kernel";
  const bool env_per_team = !p.crew_threads && !p.wave_envs;
  std::snprintf(out, size_t(len), "%s %d %d %d %d %d %d %d", kernel, env_per_team ? p.teams_per_wg : 1,
                p.crew_threads ? p.crew_threads : env_per_team ? p.wg_size : 64, env_per_team || p.crew_threads ? p.strips : 0, p.wide,
                p.obs_mode == wd::kObsFullSplit ? 1 : 0, p.crew_threads ? p.crew_reach_words : 0,
                p.crew_threads ? p.crew_lds : env_per_team ? p.lds_bytes : 0);
  return WD_OK;
}
