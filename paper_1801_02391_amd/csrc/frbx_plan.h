// How many DM trials and whole baselines share a dedispersed tile: sizes
// only, no device code (a plain C++ header).
#ifndef FRBX_PLAN_H
#define FRBX_PLAN_H

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace frbx {

// Most segments, or (segment, rate) tasks of a screening pass, of one launch:
// the kernels count them in int and round up to work-groups and sweeps over
// the grid, so the limit stays a grid's worth below 2^31.
constexpr int64_t kLaunchMost = (int64_t(1) << 31) - (1 << 16);

// DM trials of a tile: as many of D as fit `most` bytes at per_trial bytes
// each (at least one), within a launch of `tasks` per trial.
inline int tile_trials(size_t most, size_t per_trial, int D, int64_t tasks) {
  if (per_trial == 0) return 1;
  int dt = int(std::max<size_t>(1, std::min<size_t>(size_t(D), most / per_trial)));
  while (dt > 1 && int64_t(dt) * tasks > kLaunchMost) dt /= 2;
  return dt;
}

// A tile that holds every DM trial of a baseline takes further baselines as
// long as it stays within `most` bytes and its tasks within a launch: few
// trials of a short scan would otherwise be one small launch per baseline.
inline int whole_baselines(int dt, size_t per_trial, int D, int B, int64_t tasks, size_t most) {
  if (dt < D || per_trial == 0) return dt;
  int nb = int(std::min<size_t>(size_t(B), std::max<size_t>(1, most / (per_trial * size_t(D)))));
  while (nb > 1 && int64_t(nb) * D * tasks > kLaunchMost) --nb;
  return nb * D;
}

// The tile of a search: its DM trials (a multiple of D where it holds whole
// baselines) and whether it is screened.
struct TilePlan {
  int dt = 1;
  bool records = false;
};

// per_tile, per_rec: bytes of a DM trial's dedispersed spectra and of its
// screening records (0: not screened), rec_extra bytes of records once; S
// segments of a trial with n_rate screening tasks each.  Tiles and records
// share the budget.  Where a trial's do not fit together it is searched without
// records; a budget that is not strict holds any one trial, whose records may
// then take as much again as its spectra.  Baselines share a tile up to `merge`
// bytes of spectra.
inline TilePlan plan_tiles(size_t budget, bool strict, size_t merge, size_t per_tile, size_t per_rec, size_t rec_extra,
                           int D, int B, int64_t S, int n_rate) {
  TilePlan p;
  const size_t room = strict ? budget : std::max(budget, 2 * per_tile);
  p.records = per_rec > 0 && S * n_rate <= kLaunchMost && per_tile + per_rec + rec_extra <= room;
  const size_t per = per_tile + (p.records ? per_rec : 0), most = budget - std::min(budget, p.records ? rec_extra : 0);
  const int64_t tasks = S * (p.records ? n_rate : 1);
  p.dt = tile_trials(most, per, D, tasks);
  p.dt = std::min(whole_baselines(p.dt, per, D, B, tasks, most),
                  whole_baselines(p.dt, per_tile, D, B, tasks, std::min(budget, merge)));
  return p;
}

}  // namespace frbx

#endif
