// Which form of the class kernel is the fastest for a batch: plain functions of integers.
#pragma once

namespace gs {

// Costs of a layer front in microseconds, for `used` 64-row tiles with work per instance:
//   one launch per front        max(launch, base + tile x B x used): the tiles spread evenly over the
//                               chip, a launch costs its four microseconds whatever it does
//   several fronts per launch   base8 + tile8 x load with eight waves per tile, base4 + tile4 x load with
//                               four, load = ceil(B / 8) x used tiles of the fullest XCD (an instance
//                               is bound to one); and more over a range of loads, where the tiles of one
//                               front, or of two, about fill the XCD (44 strategies, 8 instances, 23
//                               fronts, eight waves: 32 tiles 105 us, 56 159, 80 163, 110 104, 126 113;
//                               four waves: 94 195, 126 248, 180 119).  The range is measured, its cause
//                               not shown; polling less often does not change it.
// Fitted to whole searches of 9 to 96 layers, 12 to 242 strategies, 1 to 157 instances, 4 to 257 tiles, 0.3
// to all of them with work, equal and ragged budgets (17 thousand shapes, every form measured at
// each): the form picked takes 1.010 times the best one's time on average, the same over three thousand
// shapes left out of the fit, and more than 1.1 times in one of 25.  (Always one launch per front: 1.22
// times; always several, eight or four waves by the strategies alone: 1.11.)
//
// Beyond a load of 500 to 700 tiles, outside the fit, one launch per front: its workgroups fill the chip
// evenly and stay full, the other form's wait for each other as before.  500 shapes of 60 to 2000
// instances, several fronts at the better wave count / one launch, loads of 400 to 1000 and beyond: 16 to
// 32 strategies 1.03 to 1.19 / 1.3 to 1.6, 48 to 96 0.92 to 1.14 / 1.12 to 1.35, 128 and more 1.03 to 1.14 /
// 1.1 to 1.4; the form picked takes 1.010 times the best one's time, 1.012 over 400 shapes that the limits
// were not chosen by, 1.028 by the costs alone (815 instances, 20 strategies, 51 tiles, 27 layers: 3084 ->
// 1903 us).  Under eight layers the rule of gsearch_api.hip stays.
struct ClassCosts {
  float launch, base, tile, base8, tile8, base4, tile4;
};

// 16, 24, 32, 48, 64, 96, 128, 192, 256 padded strategies (the last two have no four-wave form)
constexpr ClassCosts kClassCosts[2][9] = {
    {// min-only
     {5.00f, 3.85f, 0.00051f, 1.93f, 0.018f, 1.87f, 0.0069f},
     {4.49f, 4.05f, 0.00085f, 1.08f, 0.022f, 3.41f, 0.0075f},
     {4.56f, 3.78f, 0.00099f, 1.32f, 0.02f, 3.14f, 0.0084f},
     {3.59f, 2.56f, 0.0021f, 1.26f, 0.02f, 2.50f, 0.013f},
     {4.47f, 2.59f, 0.0044f, 1.68f, 0.028f, 4.76f, 0.013f},
     {4.44f, 2.61f, 0.0061f, 1.06f, 0.038f, 2.62f, 0.03f},
     {4.19f, 2.69f, 0.0065f, 0.80f, 0.044f, 3.18f, 0.029f},
     {4.25f, 5.22f, 0.0088f, 0.94f, 0.081f, 0.00f, 0.0f},
     {8.91f, 6.53f, 0.015f, 1.24f, 0.123f, 0.00f, 0.0f}},
    {// with backpointers
     {4.01f, 4.64f, 0.0014f, 0.60f, 0.033f, 2.40f, 0.014f},
     {4.16f, 4.07f, 0.0016f, 0.78f, 0.028f, 2.47f, 0.013f},
     {3.08f, 4.20f, 0.0017f, 0.39f, 0.033f, 2.38f, 0.015f},
     {3.75f, 4.08f, 0.0019f, 2.12f, 0.02f, 2.77f, 0.016f},
     {4.16f, 3.32f, 0.0042f, 0.88f, 0.032f, 2.03f, 0.023f},
     {5.35f, 4.13f, 0.0051f, 0.36f, 0.052f, 0.43f, 0.086f},
     {5.87f, 4.60f, 0.0078f, 0.17f, 0.067f, -0.42f, 0.227f},
     {7.59f, 5.48f, 0.023f, -2.91f, 0.234f, 0.00f, 0.0f},
     {8.78f, 6.97f, 0.04f, -3.63f, 0.344f, 0.00f, 0.0f}}};

constexpr int class_cost_row(int SP) {
  return SP <= 16 ? 0 : SP <= 24 ? 1 : SP <= 32 ? 2 : SP <= 48 ? 3 : SP <= 64 ? 4
         : SP <= 96 ? 5 : SP <= 128 ? 6 : SP <= 192 ? 7 : 8;
}

struct ClassTimes {
  float single, four, eight; // one launch per front; several, four and eight waves per tile
};

constexpr ClassTimes class_times(int B, int L, int SP, bool with_bp, float used) {
  const ClassCosts &c = kClassCosts[with_bp ? 1 : 0][class_cost_row(SP)];
  const int q = (B + 7) / 8;
  const float load = (float)q * used, spread = c.base + c.tile * (float)B * used;
  const bool full8 = with_bp ? load > 37.f && load < 94.f : load > 40.f && load < 113.f;
  const bool full4 = with_bp ? load > 29.f && load < 178.f : load > 39.f && load < 219.f;
  const float more8 = !full8 || q > 3 ? 0.f : q == 1 ? 2.5f : 0.9f;
  const float more4 = !full4 || q > (with_bp ? 3 : 7) ? 0.f : with_bp ? (q == 1 ? 2.f : 1.f) : q == 1 ? 2.6f : 2.1f;
  const float small = 4.f / (float)(L > 1 ? L - 1 : 1); // two small launches more per solve
  return {spread > c.launch ? spread : c.launch, c.base4 + c.tile4 * load + more4 + small,
          c.base8 + c.tile8 * load + more8 + small};
}

struct ClassForm {
  int waves;  // per tile in the several-fronts form: 4 or 8
  bool pays;  // that form is to be taken
};

constexpr bool class_load_is_large(int B, int SP, float used) {
  return (float)((B + 7) / 8) * used > (SP > 32 && SP <= 96 ? 700.f : 500.f);
}

constexpr ClassForm class_form(int B, int L, int SP, bool with_bp, float used) {
  const ClassTimes t = class_times(B, L, SP, with_bp, used);
  const int waves = SP > 128 || t.eight <= t.four ? 8 : 4;
  return {waves, (waves == 8 ? t.eight : t.four) < t.single && !class_load_is_large(B, SP, used)};
}

// The same while nothing is known about how many tiles have work: by the costs for four tenths to all
// of them.  Several fronts per launch find it out, so they are tried where they are up to a tenth
// dearer (the first solve takes 1.033 times the best form's time on average, later ones 1.015).
constexpr ClassForm class_form_unknown(int B, int L, int SP, bool with_bp, int tiles) {
  ClassTimes sum = {0.f, 0.f, 0.f};
  for (int k = 2; k <= 5; ++k) {
    const ClassTimes t = class_times(B, L, SP, with_bp, 0.2f * (float)(k * tiles));
    sum = {sum.single + t.single, sum.four + t.four, sum.eight + t.eight};
  }
  const int waves = SP > 128 || sum.eight <= sum.four ? 8 : 4;
  return {waves, (waves == 8 ? sum.eight : sum.four) <= 1.1f * sum.single &&
                     !class_load_is_large(B, SP, 0.7f * (float)tiles)};
}

} // namespace gs
